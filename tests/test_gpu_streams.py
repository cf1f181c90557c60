"""Steps beside other work on the same device: what other streams do to words and stores that a step shares with them."""
import numpy as np
import pytest
import torch

from step_forms import form_of, form_of_launches, launches_of

pytestmark = pytest.mark.gpu


def state_of(name, batch, **changes):
    import paper_1806_03925_amd as g
    from gear_inputs import PageViewSource, get_workload
    wl = get_workload(name).scaled(n_users=50_000, n_urls=1 << 15, n_images=4_000, M=4, **changes)
    st = g.GearState(g.config_for(wl, max_batch=batch))
    g.gear_init_tables(st)
    g.gear_fill_normal(st.dfv_cache, wl.n_images, wl.dfv_dim, wl.seed, 3, wl.dfv_std)
    return wl, st, PageViewSource(wl)


@pytest.mark.parametrize("batch,changes,form", [
    (16_383, dict(layers=(128, 1)), "blocks"), (16_384, dict(layers=(128, 1)), "long blocks"),                 # 49 152 ids
    (16_383, dict(layers=(40, 1), dfv_dim=2_080), "carried"), (16_384, dict(layers=(40, 1), dfv_dim=2_080), "helper"),
    (15_963, {}, "blocks"), (15_964, {}, "long blocks"),                                            # 6.8e9 multiply-adds
    (11_529, dict(layers=(1024, 1)), "divided"),
    (2_882, dict(layers=(1024, 1), mlp_dtype="f32"), "carried"), (2_883, dict(layers=(1024, 1), mlp_dtype="f32"), "helper"),
])
def test_steps_on_either_side_of_the_line_between_their_forms(batch, changes, form):
    """One image a view, so three ids.  Each takes the form it should and gives the bits of the other."""
    import paper_1806_03925_amd as g
    results = []
    for one in (False, True):
        wl, st, src = state_of("bf16", batch, max_images=1, **changes)
        st.one_stream = one
        dev = g.DeviceBatch.from_host(src.batch(0, batch=batch))
        assert form_of(st, dev, wl.M, 0.1) == (form if not one or form == "blocks" else "carried")
        g.gear_step(st, dev, wl.M, 0.1)
        torch.cuda.synchronize()
        assert int(st.status.item()) == 0
        results.append(outputs(st))
    for a, b in zip(*results):
        assert torch.equal(a, b)


def outputs(st):
    n = int(st.n_ready.item())
    return [t.clone() for t in (st.loss, st.n_ready, st.ready_ids[:n], st.ready_grads[:n], st.grad_accum, st.counts,
                                st.user_emb, st.url_emb, st.mlp_params)]


@pytest.mark.parametrize("name,batch,changes,form", [
    ("tiny", 511, {}, "blocks"), ("small", 4_096, {}, "blocks"),
    ("tiny", 511, {"dfv_dim": 2_080}, "carried"),                # one tile of each list
    ("small", 4_096, {"max_images": 12}, "carried"), ("bf16", 4_600, {"max_images": 10}, "carried"),   # several that look back
    ("bf16", 9_001, {}, "long blocks"),                          # lists in counted tiles
    ("bf16", 16_200, {"max_images": 40}, "long blocks"),         # in tiles that look back
    ("bf16", 8_000, {"max_images": 80}, "long blocks"),          # on the caller's stream, beside blocks
    ("bf16", 18_001, {}, "helper"),
    ("large", 8_192, {"max_images": 40}, "divided"),             # helper stream, long lists, dLoss/dx in two products
])
def test_a_step_does_not_read_the_status_word_that_others_write(name, batch, changes, form):
    """Two calls on another stream report bad ids into the step's status word and clear it again, over and over, while the
    steps run.  Workgroups that wait for one another must not decide by that word whether to work: every step has to end
    with the bits it gets when it runs alone."""
    import paper_1806_03925_amd as g
    results = []
    for disturbed in (False, True):
        wl, st, src = state_of(name, batch, **changes)
        dev = [g.DeviceBatch.from_host(src.batch(t, batch=batch)) for t in range(4)]
        other = g.GearState(g.make_config(16, 16, 16, 8, 8, (8, 1), max_batch=1, max_nnz=64))
        other.status = st.status                                   # one word for all that goes on with a cache
        bad = torch.full((64,), 16, dtype=torch.int32, device="cuda")
        rows = torch.zeros((64, 8), device="cuda")
        stamp = torch.zeros(16, dtype=torch.int32, device="cuda")
        good = torch.zeros(1, dtype=torch.int32, device="cuda")
        beside = torch.cuda.Stream()
        torch.cuda.synchronize()
        assert form_of(st, dev[0], wl.M, 0.1) == form
        for t in range(4):
            print(f"{name} disturbed {disturbed} step {t}", flush=True)
            if disturbed:
                with torch.cuda.stream(beside):
                    for _ in range(20):
                        g.gear_refresh_dfv(other, bad, rows)           # sets the word, writes no row
                        g.gear_expired_ids(other, good, stamp, 0, 1)   # clears it
            g.gear_step(st, dev[t], wl.M, 0.1)
        torch.cuda.synchronize()
        results.append(outputs(st))
    assert int(results[0][1].item()) > 0
    for a, b in zip(*results):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])   # without a prologue, with one
def test_what_others_report_while_a_step_runs_stays(dtype):
    """A step clears its status word when it starts and not again: refreshes on another stream that report a bad id from before the
    middle of it on are still seen behind it.  All images are one and no group closes, so that the accumulation is one chain of
    19 000 rows, many times as long as all that comes ahead of it."""
    import paper_1806_03925_amd as g
    from gear_inputs import get_workload
    from gear_inputs.pageviews import PageViewBatch
    B, nnz = 100, 19_000
    wl = get_workload("tiny").scaled(batch=B, layers=(16, 1), emb_dim=8, dfv_dim=8, emb_dtype=dtype, dfv_dtype=dtype, mlp_dtype=dtype,
                                     n_users=1_000, n_urls=1_000, n_images=2_000, max_images=190, M=1 << 20)
    st = g.GearState(g.config_for(wl))
    g.gear_init_tables(st)
    rng = np.random.default_rng(0)
    dev = g.DeviceBatch.from_host(PageViewBatch(
        user_id=rng.integers(0, 1_000, B).astype(np.int32), url_id=rng.integers(0, 1_000, B).astype(np.int32),
        img_off=(190 * np.arange(B + 1)).astype(np.int32), img_id=np.full(nnz, 7, dtype=np.int32), label=np.zeros(B, dtype=np.float32)))
    names = launches_of(st, dev, wl.M, 0.1)
    assert form_of_launches(names) == "blocks" and ("begin" in names) == (dtype == "bf16")
    other = g.GearState(g.make_config(16, 16, 16, 8, 8, (8, 1), max_batch=1, max_nnz=64))
    other.status = st.status
    bad, rows = torch.full((64,), 16, dtype=torch.int32, device="cuda"), torch.zeros((64, 8), device="cuda")
    begin, reported, end = (torch.cuda.Event(enable_timing=True) for _ in range(3))
    # another stream each time: one that shares a queue of the device with the step's runs behind it; fewer refreshes where the host is slow
    for count in 4 * (60, 30, 15):
        beside = torch.cuda.Stream()
        torch.cuda.synchronize()
        begin.record()
        beside.wait_event(begin)
        g.gear_step(st, dev, wl.M, 0.1)
        end.record()
        with torch.cuda.stream(beside):
            for _ in range(count):
                g.gear_refresh_dfv(other, bad, rows)
            reported.record()
        torch.cuda.synchronize()
        at, whole = begin.elapsed_time(reported), begin.elapsed_time(end)
        print(f"{dtype}: reported until {at:.3f} of {whole:.3f} ms", flush=True)
        if 0.2 < at < 0.8 * whole:
            break
    else:
        pytest.fail("no refresh ran beside the step")
    assert int(st.status.item()) == g.GEAR_ERR_RANGE


# views of the bf16 workload: in blocks on one stream (13 000 ids), with the grouping on the helper stream, in counted tiles (58 000)
# or in tiles that look back (365 000), or on the caller's beside blocks on the helper's (340 000), and layer by layer with everything about
# the store on the helper's
SHORT, LONG, BACK, HERE, LAYERS = 2_000, 9_001, 16_200, 8_000, 18_001
FORMS = {SHORT: "blocks", LONG: "long blocks", BACK: "long blocks", HERE: "long blocks", LAYERS: "helper"}
IMAGES = {BACK: dict(max_images=40), HERE: dict(max_images=80)}


@pytest.mark.parametrize("sizes", [(SHORT, SHORT), (SHORT, LONG), (LONG, SHORT), (SHORT, LONG, SHORT), (LONG, LONG),
                                   (HERE, HERE), (SHORT, HERE), (HERE, SHORT), (LONG, HERE), (HERE, LONG), (LAYERS, LAYERS),
                                   (SHORT, LAYERS), (LAYERS, SHORT), (HERE, LAYERS), (LAYERS, HERE), (LAYERS, HERE, LONG, LAYERS),
                                   (BACK, BACK), (BACK, SHORT), (LONG, BACK), (BACK, LAYERS), (LAYERS, BACK), (HERE, BACK, HERE)])
def test_steps_on_streams_of_their_own_share_a_store_in_the_order_they_were_issued(sizes):
    """Each step has tables, workspace and stream of its own and all collect gradients in one store.  The first stream is
    held up ahead of its step, so a step that does not wait for the one issued before it gets there first; which groups of
    an image close in which step, and every sum, then come out differently."""
    import paper_1806_03925_amd as g
    results = []
    for apart in (False, True):
        states = [state_of("bf16", n, **IMAGES.get(n, {})) for n in sizes]
        store = states[0][1]
        for _, st, _ in states[1:]:
            st.grad_accum, st.counts = store.grad_accum, store.counts
        # another batch for each step, on tables of the same initial values
        dev = [[g.DeviceBatch.from_host(src.batch(len(sizes) * t + i, batch=n)) for i, (n, (_, _, src)) in enumerate(zip(sizes, states))]
               for t in range(2)]
        streams = [torch.cuda.Stream() if apart else torch.cuda.current_stream() for _ in sizes]
        torch.cuda.synchronize()
        assert [form_of(st, d, wl.M, 0.1) for (wl, st, _), d in zip(states, dev[0])] == [FORMS[n] for n in sizes]
        lists = []
        for t in range(2):
            print(f"sizes {sizes} apart {apart} round {t}", flush=True)
            for i, (wl, st, _) in enumerate(states):
                with torch.cuda.stream(streams[i]):
                    if i == 0:
                        torch.cuda._sleep(3_000_000)
                    g.gear_step(st, dev[t][i], wl.M, 0.1)
            torch.cuda.synchronize()
            for _, st, _ in states:
                assert int(st.status.item()) == 0
                n = int(st.n_ready.item())
                assert n > 0
                lists += [st.ready_ids[:n].clone(), st.ready_grads[:n].clone()]
        results.append(lists + [x.clone() for _, st, _ in states for x in (st.grad_accum, st.counts, st.user_emb, st.mlp_params)])
    for a, b in zip(*results):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])   # without a prologue, with one
def test_a_step_that_stops_part_way_keeps_its_place_in_the_order(dtype):
    """The last launch of a short step leaves the event by which steps on other streams know their place behind it.  Where that launch, or an
    earlier one, is not enqueued, what the step has done to the store so far still happens ahead of the next step's."""
    import paper_1806_03925_amd as g
    results = []
    for apart in (False, True):
        states = [state_of("tiny", 512, emb_dtype=dtype, dfv_dtype=dtype, mlp_dtype=dtype) for _ in range(2)]
        (wl, first, src), (_, second, _) = states
        second.grad_accum, second.counts = first.grad_accum, first.counts
        dev = [g.DeviceBatch.from_host(src.batch(t, batch=512)) for t in range(10)]
        streams = [torch.cuda.Stream() if apart else torch.cuda.current_stream() for _ in states]
        torch.cuda.synchronize()
        names = launches_of(first, dev[8], wl.M, 0.1)
        assert names == ["begin"] * (dtype == "bf16") + ["view_blocks", "accumulate_wgrad", "param_update"]
        assert launches_of(second, dev[9], wl.M, 0.1) == names
        lists = []
        for nth in range(1, len(names) + 1):
            print(f"{dtype} apart {apart}, without launch {nth}", flush=True)
            with torch.cuda.stream(streams[0]):
                torch.cuda._sleep(3_000_000)
                g.gear_debug_fail_launch(nth)
                try:
                    with pytest.raises(g.GearError):
                        g.gear_step(first, dev[2 * nth - 2], wl.M, 0.1)
                finally:
                    g.gear_debug_fail_launch(0)
            with torch.cuda.stream(streams[1]):
                g.gear_step(second, dev[2 * nth - 1], wl.M, 0.1)
            torch.cuda.synchronize()
            assert int(second.status.item()) == 0
            lists += outputs(second)
        results.append(lists)
    for a, b in zip(*results):
        assert torch.equal(a, b)


# on one stream, in blocks and layer by layer with the sums of blocks; on two, the fork to the helper ahead of all launches and behind the first
@pytest.mark.parametrize("views,one", [(SHORT, False), (LONG, True), (LONG, False), (BACK, False), (HERE, False)])
def test_a_step_recorded_into_a_graph_between_steps_on_other_streams(views, one):
    """Recording takes no event from the order of the steps and leaves none: replays, with eager steps on another stream
    before and between them, give the bits of the same steps issued one after the other."""
    import paper_1806_03925_amd as g
    results = []
    for recorded in (False, True):
        wl, st, src = state_of("bf16", views, **IMAGES.get(views, {}))
        st.one_stream = one
        dev = g.DeviceBatch.from_host(src.batch(0, batch=views))
        wl2, st2, src2 = state_of("bf16", LONG)
        dev2 = g.DeviceBatch.from_host(src2.batch(1, batch=LONG))
        beside = torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(beside):
            g.gear_step(st2, dev2, wl2.M, 0.1)
        g.gear_step(st, dev, wl.M, 0.1)
        torch.cuda.synchronize()
        if recorded:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                g.gear_step(st, dev, wl.M, 0.1)
        for _ in range(3):
            if recorded:
                graph.replay()
            else:
                g.gear_step(st, dev, wl.M, 0.1)
            with torch.cuda.stream(beside):
                g.gear_step(st2, dev2, wl2.M, 0.1)
            torch.cuda.synchronize()
        g.gear_step(st, dev, wl.M, 0.1)
        torch.cuda.synchronize()
        assert int(st.status.item()) == 0 and int(st2.status.item()) == 0
        results.append(outputs(st) + outputs(st2))
        assert form_of(st, dev, wl.M, 0.1) == ("carried" if one else FORMS[views])
    for a, b in zip(*results):
        assert torch.equal(a, b)
