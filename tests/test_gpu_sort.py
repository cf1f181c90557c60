"""Grouping at the sizes where its shape changes: tiles of 2048 keys, four tiles per counting workgroup beyond 65 536 keys,
one to four passes of up to twelve bits (kernels for up to nine bits and for more).  Integers: exact."""
import numpy as np
import pytest
import torch

from step_forms import form_of_launches, launches_of

pytestmark = pytest.mark.gpu


def grouped(keys):
    perm = np.argsort(keys, kind="stable")
    unique, start = np.unique(keys[perm], return_index=True)
    return unique, np.append(start, len(keys)), perm


@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 12_345, 65_537, 300_001])
@pytest.mark.parametrize("bits", [1, 9, 10, 12, 13, 21, 22, 23, 31])
def test_groups_of_any_length_and_key_width(n, bits):
    import paper_1806_03925_amd as g
    st = g.GearState(g.make_config(16, 16, 16, 8, 8, (8, 1), max_batch=1, max_nnz=n))
    rng = np.random.default_rng(n + bits)
    span = (1 << bits) - 1
    keys = np.minimum((rng.random(n) ** 6 * span).astype(np.int64), span - 1 if bits > 1 else 1).astype(np.int32)
    keys[rng.integers(0, n, n // 2)] = keys[n // 2]           # a run over many tiles
    keys[-1] = span                                           # the widest key there is
    print(f"group n {n} bits {bits}", flush=True)
    for _ in range(2):                                        # the second time on whatever the first left behind
        unique, segoff, perm, n_unique = g.gear_group_ids(st, torch.from_numpy(keys).cuda(), 1 << bits)
        ru, rs, rp = grouped(keys)
        m = int(n_unique.item())
        assert m == len(ru)
        assert np.array_equal(unique[:m].cpu().numpy(), ru)
        assert np.array_equal(segoff[:m + 1].cpu().numpy(), rs)
        assert np.array_equal(perm.cpu().numpy(), rp)


@pytest.mark.parametrize("name,layers,batch,changes,forms", [      # on one stream; on two, unless the step is short
    ("bf16", (512, 256, 1), 9_001, {}, ("carried", "long blocks")), ("bf16", (72, 1), 9_001, {}, ("carried", "long blocks")),
    ("bf16", (72, 40, 1), 9_001, dict(dfv_dim=2_080), ("carried", "helper")),   # two, three passes
    ("bf16", (40, 1), 18_001, dict(dfv_dim=2_080), ("carried", "helper")),
    ("small", (64, 40, 24, 16, 1), 8_500, {}, ("carried", "helper")), ("small", (256, 1), 8_500, {}, ("carried", "helper")),   # more launches than links, and fewer
    ("tiny", (64, 1), 1, {}, ("blocks",)), ("tiny", (64, 1), 511, {}, ("blocks",)),     # one tile of each list; too short for the helper
    ("tiny", (64, 1), 1, dict(dfv_dim=2_080), ("carried",)), ("tiny", (64, 1), 511, dict(dfv_dim=2_080), ("carried",)),
    ("tiny", (64, 1), 511, dict(dfv_dim=2_080, mlp_dtype="bf16"), ("carried",)),
    ("bf16", (512, 256, 1), 4_600, dict(max_images=10), ("carried",)),                  # short, but a list LDS does not hold
])
def test_a_carried_grouping_gives_the_bits_of_one_on_the_helper_stream(name, layers, batch, changes, forms):
    """Both against numpy, and where the step is long enough to use the helper stream against each other."""
    import paper_1806_03925_amd as g
    from gear_inputs import PageViewSource, get_workload
    wl = get_workload(name).scaled(n_users=100_000, n_urls=1 << 22, n_images=9_000, M=4, layers=layers, **changes)
    outs = []
    for one, form in zip((True, False), forms):
        st = g.GearState(g.config_for(wl, max_batch=batch), debug=True)
        g.gear_init_tables(st)
        g.gear_fill_normal(st.dfv_cache, wl.n_images, wl.dfv_dim, wl.seed, 3, wl.dfv_std)
        st.one_stream = one
        src = PageViewSource(wl)
        for step in range(2):
            b = g.DeviceBatch.from_host(src.batch(step, batch=batch))
            names = launches_of(st, b, wl.M, 0.1)
            # the segments by their name where they are a launch of their own: always but in blocks, or where another carries them
            assert form_of_launches(names) == form and ("accum_plan" in names or form in ("blocks", "carried"))
        assert int(st.status.item()) == 0
        n, m = int(st.n_ready.item()), int(st.dbg[3].item())
        outs.append([t.clone() for t in (st.loss, st.n_ready, st.ready_ids[:n], st.ready_grads[:n], st.grad_accum, st.counts,
                                         st.user_emb, st.url_emb, st.mlp_params, st.dbg[0][:m], st.dbg[1][:m + 1])])
        ru, rs, rp = grouped(b.img_id.cpu().numpy())
        assert np.array_equal(st.dbg[0][:m].cpu().numpy(), ru) and np.array_equal(st.dbg[1][:m + 1].cpu().numpy(), rs)
    for a, b in zip(outs[0], outs[-1]):
        assert torch.equal(a, b)
