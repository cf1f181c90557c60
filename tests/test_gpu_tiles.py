"""Matrix products at the sizes where a tile shape changes or a tile is cut (gemm_tile.hip), against fp64 products of
the same operands.  Accumulation is fp32 over at most 1100 terms: 1e-5 of the row's largest element."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def operands(dtype, M, N, K):
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(M * 31 + N * 7 + K)
    draw = lambda *s: torch.randn(s, generator=gen, device="cuda").to(td)
    return draw(M, K), draw(N, K), draw(M, N), torch.randn(N, generator=gen, device="cuda")


def beside_the_oracle(wl):
    """The comparison of tests/test_gpu_parity.py, also where these tests run by themselves."""
    import paper_1806_03925_amd as g
    import test_gpu_parity as parity
    parity.g = g
    return parity.Pair(wl)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("M,N,K", [
    (1, 8, 8), (63, 72, 24), (65, 64, 64), (64, 56, 72), (129, 200, 136),    # 64 x 64: one piece, one stage, one over
    (16385, 128, 40), (16384, 64, 128),                                       # bf16 from 256 tiles of 128 x 64 on
    (32760, 256, 72), (16390, 256, 32), (65537, 128, 200),                    # 128 x 128, cut in M and in K
    (16390, 320, 40), (20000, 384, 40), (20000, 320, 40),                     # fp32 by rounds: 64 x 64, 128 x 128, 64 x 64
])
def test_products_at_the_edges_of_tiles(dtype, M, N, K):
    import paper_1806_03925_amd as g
    A, B, aux, bias = operands(dtype, M, N, K)
    ref = A.double() @ B.double().T
    scale = ref.abs().amax(dim=1, keepdim=True).clamp_min(1e-30)
    tol = 2.0 ** -8 if dtype == "bf16" else 1e-5            # one rounding of the result to the operand type
    assert ((g.gear_gemm(A, B, 0, 2).double() - ref).abs() <= 1e-5 * scale).all()
    want = torch.relu(ref + bias.double())
    assert ((g.gear_gemm(A, B, 0, 0, bias=bias).double() - want).abs() <= tol * want.abs() + 1e-5 * scale).all()
    want = torch.where(aux.double() > 0, ref, torch.zeros_like(ref))
    assert ((g.gear_gemm(A, B, 0, 1, aux=aux).double() - want).abs() <= tol * want.abs() + 1e-5 * scale).all()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("M,N,K,splits", [(8, 8, 1, 1), (72, 136, 31, 3), (64, 128, 33, 64), (320, 72, 1000, 7), (512, 576, 1099, 5)])
def test_weight_gradients_over_any_number_of_rows(dtype, M, N, K, splits):
    """K rows of a batch in `splits` ranges, the last cut or empty."""
    import paper_1806_03925_amd as g
    A, B, _, _ = operands(dtype, M, N, K)
    ref = A.double() @ B.double().T
    out = g.gear_gemm(A.T.contiguous(), B.T.contiguous(), 1, splits=splits)
    assert ((out.double() - ref).abs() <= 1e-5 * ref.abs().max()).all()


def test_fp32_bits_do_not_depend_on_the_tile_shape():
    """Sums run over k in ascending pairs in every shape: the same rows, once in 64 x 64 tiles, once in 128 x 128."""
    import paper_1806_03925_amd as g
    for K in (8, 72, 320):
        A, B, _, bias = operands("f32", 32760, 256, K)
        big = g.gear_gemm(A, B, 0, 0, bias=bias)
        small = g.gear_gemm(A[:200].contiguous(), B, 0, 0, bias=bias)
        assert torch.equal(big[:200], small)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_weight_gradients_and_bias_sums_that_do_not_fit_at_once(dtype):
    """Five equal hidden layers and a short batch: the partial results of all weight gradients exceed their region, so
    the layers go out in groups; the bias partials fit with 128-row tiles only."""
    from gear_inputs import PageViewSource, get_workload
    wl = get_workload("tiny").scaled(batch=300, layers=(512,) * 5 + (1,), emb_dtype=dtype, dfv_dtype=dtype,
                                     mlp_dtype=dtype)
    pair = beside_the_oracle(wl)
    src = PageViewSource(wl)
    for step in range(2):
        pair.step(src.batch(step), wl.lr, f"deep {dtype} step {step}")


@pytest.mark.parametrize("layers,batch", [
    ((1024,) * 5 + (1,), 2_208),              # 68 tiles of 256 x 256 in three ranges, the shortest batch that takes them
    ((1024,) * 5 + (1,), 2_176),              # a size below: 128 x 128
    ((2048, 2048, 2048, 1024, 1), 2_944),     # 168 large tiles: two launches, of 96 and of 72
])
def test_weight_gradients_of_many_tiles(layers, batch):
    """Wide layers take the large tiles below 32 768 rows too, in groups of layers that fill the CUs."""
    import paper_1806_03925_amd as g
    from gear_inputs import PageViewSource, get_workload
    wl = get_workload("tiny").scaled(batch=batch, layers=layers, emb_dtype="bf16", dfv_dtype="bf16", mlp_dtype="bf16")
    pair = beside_the_oracle(wl)
    pair.st.profile = g.GearProfile()
    pair.step(PageViewSource(wl).batch(0), wl.lr, f"{len(layers)} layers, {batch} views")
    launches = [name for name, _ in pair.st.profile.spans()].count("wgrad_gemm")
    pair.st.profile.close()
    assert launches == (2 if layers[0] == 2048 else 1)


@pytest.mark.parametrize("M,N,K", [(20_000, 768, 512), (28_672, 512, 1_056), (20_000, 576, 1_024), (24_001, 512, 1_024)])
def test_bf16_bits_do_not_depend_on_the_kernel(M, N, K):
    """Long products that leave a few CUs without a 256 x 256 tile take that kernel, the same rows in a short one do not, and
    a step's product goes either way depending on whether it carries other work: every epilogue gives the same bits."""
    import paper_1806_03925_amd as g
    A, B, aux, bias = operands("bf16", M, N, K)
    rows = 500
    a, x = A[:rows].contiguous(), aux[:rows].contiguous()
    for epilogue, many, few in ((0, dict(bias=bias), dict(bias=bias)), (1, dict(aux=aux), dict(aux=x)), (2, {}, {})):
        big = g.gear_gemm(A, B, 0, epilogue, **many)
        assert torch.equal(big[:rows], g.gear_gemm(a, B, 0, epilogue, **few))
        last = g.gear_gemm(A[-rows:].contiguous(), B, 0, epilogue, **(dict(aux=aux[-rows:].contiguous()) if epilogue == 1 else many))
        assert torch.equal(big[-rows:], last)


@pytest.mark.parametrize("batch,layers,d,D", [
    (65_540, (96, 32, 1), 16, 160),   # one, three and six k-tiles; 32, 96 and 192 columns; four rows in the last tile
    (33_028, (288, 1), 16, 224),      # column tiles of 256 and 32
    (65_536, (288, 1), 16, 288),      # dLoss/dx in two products, the transpose in tile order from row 32 on
])
def test_weights_in_the_order_of_large_tiles(batch, layers, d, D):
    """The first quarter of the views as a step of its own takes other kernels, with weights in other orders: the same logits, and
    dLoss/dx four times as large, which is exact (a mean over a quarter of the views)."""
    import paper_1806_03925_amd as g
    from gear_inputs import PageViewSource, get_workload
    from gear_inputs.pageviews import PageViewBatch
    wl = get_workload("tiny").scaled(batch=batch, layers=layers, emb_dim=d, dfv_dim=D, emb_dtype="bf16", dfv_dtype="bf16",
                                     mlp_dtype="bf16", max_images=1)
    full = PageViewSource(wl).batch(0)
    B = batch // 4

    def run(host):
        st = g.GearState(g.config_for(wl))
        g.gear_init_tables(st)
        g.gear_fill_normal(st.dfv_cache, wl.n_images, wl.dfv_dim, wl.seed, 3, wl.dfv_std)
        g.gear_step(st, g.DeviceBatch.from_host(host), wl.M, 0.1)
        torch.cuda.synchronize()
        assert int(st.status.item()) == 0
        return st

    whole = run(full)
    part = run(PageViewBatch(user_id=full.user_id[:B], url_id=full.url_id[:B], img_off=full.img_off[:B + 1],
                             img_id=full.img_id[:full.img_off[B]], label=full.label[:B]))
    assert torch.equal(whole.region("logits", batch)[:B], part.region("logits", B))
    assert torch.equal(4.0 * whole.region("dx", batch)[:B].float(), part.region("dx", B).float())


@pytest.mark.parametrize("M,N,K,splits", [
    (8, 8, 32, 1), (8, 8, 33, 1), (136, 264, 65, 1), (128, 128, 64, 2),      # one round, a half that has none, halves of unlike length
    (136, 40, 1_000, 3), (520, 72, 4_099, 25), (256, 256, 4_096, 64),        # tiles and ranges that nothing divides; 256 workgroups
    (256, 264, 4_096, 64),                                                    # and more: single ones
])
def test_weight_gradients_by_two_halves_of_a_range(M, N, K, splits):
    """bf16 values of few bits, so that all sums are exact."""
    import paper_1806_03925_amd as g
    gen = torch.Generator(device="cuda").manual_seed(K)
    a = torch.randint(-4, 5, (K, M), device="cuda", generator=gen).bfloat16()
    b = torch.randint(-4, 5, (K, N), device="cuda", generator=gen).bfloat16()
    out = g.gear_gemm(a, b, 1, splits=splits)
    assert torch.equal(out.double().cpu(), a.double().cpu().T @ b.double().cpu())
