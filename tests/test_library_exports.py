"""The C-ABI library loads without a GPU and exports every function include/gear.h declares."""
import ctypes
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "gear.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(gear_[a-z_0-9]+)\s*\(", text)))


def test_header_declares_the_three_named_calls():
    names = declared_functions()
    for required in ("gear_init_tables", "gear_step", "gear_refresh_dfv"):
        assert required in names


def test_library_exports_every_declared_symbol():
    lib = ctypes.CDLL(os.path.join(ROOT, "paper_1806_03925_amd", "libgear.so"))
    for name in declared_functions():
        assert hasattr(lib, name), f"libgear.so does not export {name}"


def test_binding_mirrors_the_header():
    import paper_1806_03925_amd as g
    from paper_1806_03925_amd import binding
    assert sorted(binding.EXPORTS) == declared_functions()
    for name in binding.EXPORTS:
        assert hasattr(binding.lib, name)
    # host-only calls work without a GPU
    cfg = g.make_config(1000, 4096, 2000, 16, 64, (64, 1), max_batch=512, max_nnz=2048)
    assert g.gear_workspace_bytes(cfg) > 0
    assert g.gear_mlp_param_count(cfg) == 96 * 64 + 64 + 64 + 1
    assert g.gear_mlp_param_offset(cfg, 1, 0) == 96 * 64 + 64
    bad = g.make_config(1000, 4096, 2000, 12, 64, (64, 1), max_batch=512, max_nnz=2048)   # emb_dim % 8 != 0
    assert g.gear_workspace_bytes(bad) == 0 and g.gear_mlp_param_count(bad) == -1
    assert binding.lib.gear_status_string(3) == b"workspace or ready list too small"
    # null arguments are reported, not dereferenced
    assert binding.lib.gear_step(None, None, None, None, None, None, 1, 0.1, None, 0, None, None) == g.GEAR_ERR_INVALID


def test_workspace_size_is_a_fixed_rule_of_the_configuration():
    """Callers keep workspaces, and the static scratch array takes what fits in 64 MiB: neither may change."""
    import paper_1806_03925_amd as g
    sizes = []
    for B, nnz, layers, dt, d, D in [(1, 1, (8, 1), "f32", 8, 8), (512, 2048, (64, 1), "f32", 16, 64),
                                     (4096, 32768, (256, 128, 1), "f32", 32, 256),
                                     (16384, 131072, (512, 256, 1), "bf16", 32, 512),
                                     (3699, 490, (216, 200, 16, 16, 16, 1), "f32", 96, 1256),
                                     (700, 900, (512, 512, 512, 512, 512, 1), "bf16", 8, 496),
                                     (65536, 524288, (1024, 256, 1), "bf16", 64, 1024)]:
        sizes.append(g.gear_workspace_bytes(g.make_config(1000, 4096, 2000, d, D, layers, "f32", dt, dt, max_batch=B,
                                                          max_nnz=nnz)))
    assert sizes == [176128, 2080000, 39670016, 163967232, 87716352, 27937280, 793410048]
