"""The selection of the separate kernels (prr_topk.h) on scores set directly, at the edges of
its group sizes and list, in every form of the entry points that use it; the two-stream
step's update and prediction against prr_predict; the two-stream step captured in a graph."""
import zlib

import numpy as np
import pytest

import oracle as O
import workloads as W
from tests import gpu_support as S
from tests.test_gpu_parity import SELECT_DISTS, _select_values

pytestmark = pytest.mark.gpu


def _score_layer(torch, vals, k, forced, cap_pages=None):
    """A layer whose score of page p of head h is vals[h][p]: mean metadata with the value in
    channel 0, one query head per KV head with 1 there."""
    from paper_2606_30389_amd import runtime as R
    hkv, n = vals.shape
    pc = R.PathConfig(num_q_heads=hkv, num_kv_heads=hkv, page_size=32, num_tokens=n * 32, k_select=k, forced=forced,
                      forced_in_budget=True, dtype="bf16", meta_kind="mean", gamma=0.25, max_pages=cap_pages)
    dev = torch.device("cuda:0")
    st = R.LayerState(pc, dev, k=torch.zeros(hkv, pc.dims().max_pages, 32, 128, dtype=torch.bfloat16, device=dev))
    st.meta[:, :n, 0] = torch.from_numpy(vals).to(dev)
    q = torch.zeros(hkv, 128, dtype=torch.bfloat16, device=dev)
    q[:, 0] = 1.0
    return pc, st, q


# sizes around the direct list (1024, 2048), the two group sizes (8192) and the largest select
SIZES = [(1, 1), (5, 3), (64, 63), (1023, 200), (1025, 40), (1025, 600), (2048, 256), (2049, 255), (2500, 1000),
         (8191, 512), (8193, 1024), (16384, 256), (16384, 1024)]


# (most distributions plant groups of hundreds of pages)
CASES = [(d, n, k) for n, k in SIZES for d in SELECT_DISTS if n >= 700 or d in ("gauss", "constant", "tiny")]


@pytest.mark.parametrize("dist,n,k", CASES)
def test_score_topk_structures(dist, n, k):
    import torch
    from paper_2606_30389_amd import _lib as L
    S.log(f"score_topk {dist}: n={n} k={k}")
    rng = np.random.default_rng(zlib.crc32(f"{dist}/{n}/{k}".encode()))
    vals = np.stack([_select_values(dist, n, rng) for _ in range(3)])
    for forced in ([], sorted({0, n // 2, n - 1})):
        pc, st, q = _score_layer(torch, vals, k, forced)
        want = [O.select_topk(vals[h].astype(np.float64), k, forced, True) for h in range(3)]
        calls = [("workspace", lambda: st.select(q)),
                 # a workspace with room for the arrival counters only
                 ("counters", lambda: L.prr_score_topk(st.dims, q, st.meta, n, k, forced, True, st.scores, st.sel,
                                                       st.sel_count, st.cap, st.workspace, 512)),
                 ("static", lambda: L.prr_score_topk_static(st.dims, q, st.meta, n, k, forced, True, st.scores, st.sel,
                                                            st.sel_count, st.cap))]
        for name, call in calls:
            st.sel.fill_(-5)
            st.sel_count.fill_(-5)
            call()
            torch.cuda.synchronize()
            for h, got in enumerate(S.lists(st)):
                assert np.array_equal(got, want[h]), f"{name}, head {h}: {len(set(got) ^ set(want[h]))} pages differ"
            np.testing.assert_array_equal(S.to_np(st.scores)[:, :n], vals)


def test_score_topk_refuses_less_than_its_counters():
    import torch
    from paper_2606_30389_amd import _lib as L
    _, st, q = _score_layer(torch, np.zeros((3, 40), dtype=np.float32), 4, [])
    with pytest.raises(L.PrrError) as e:
        L.prr_score_topk(st.dims, q, st.meta, 40, 4, [], True, st.scores, st.sel, st.sel_count, st.cap, st.workspace, 256)
    assert e.value.status == L.PRR_ERR_WORKSPACE


@pytest.mark.parametrize("n,k,forced", [(1, 1, []), (250, 20, [0, 249]), (1030, 300, [3]), (2049, 128, []),
                                        (9000, 256, [0, 8998, 8999]), (16384, 700, [])])
def test_prefill_and_two_stream_predictions(n, k, forced):
    """PRR_SCHED_PREFILL and PRR_SCHED_TWO_STREAM update and predict in many workgroups;
    prr_predict, which one workgroup per KV head serves, gives the same state and lists."""
    import torch
    from paper_2606_30389_amd import _lib as L
    from paper_2606_30389_amd import runtime as R
    S.log(f"predictions n={n} k={k}")
    rng = np.random.default_rng(n)
    vals = rng.standard_normal((2, n)).astype(np.float32)
    layers = [_score_layer(torch, vals, k, forced, n + 5) for _ in range(2)]
    (_, a, q), (_, b, _) = layers
    stack = R.DecodeStack([a], [q], torch.device("cuda:0"))
    spec = torch.cuda.Stream()
    for step in range(3):
        new = torch.from_numpy(rng.standard_normal((2, n)).astype(np.float32)).cuda()
        for st in (a, b):
            st.meta[:, :n, 0] = new
        torch.cuda.synchronize()
        stack.step(L.PRR_SCHED_TWO_STREAM if step else L.PRR_SCHED_PREFILL, torch.cuda.current_stream(), spec)
        b.select(q)
        b.predict()
        b.advance()
        torch.cuda.synchronize()
        for name in ("level", "trend", "init_bits", "scores", "sel", "sel_count"):
            assert torch.equal(getattr(a, name), getattr(b, name)), (step, name)
        assert torch.equal(a.pred_count[a.cur], b.pred_count[b.cur])
        for h in range(2):
            m = int(a.pred_count[a.cur][h])
            assert torch.equal(a.pred[a.cur][h, :m], b.pred[b.cur][h, :m]), step


def test_two_stream_step_in_a_graph():
    """The two-stream step under capture, replayed between eager work, equals the eager step."""
    import torch
    from paper_2606_30389_amd import _lib as L
    from paper_2606_30389_amd import runtime as R
    cfg = W.CONFIGS["glm32k"]
    pc = S.path_config(cfg, num_pages=300)
    st, _ = S.make_layer(cfg, pc)
    st.build_meta()
    _, qb = W.query_trajectory(cfg, 0, steps=5)
    q = S.q_tensor(qb[0], pc).clone()
    stack = R.DecodeStack([st], [q], torch.device("cuda:0"))
    s, spec = torch.cuda.Stream(), torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    stack.step(L.PRR_SCHED_PREFILL, s)
    torch.cuda.synchronize()
    keep = ("level", "trend", "init_bits", "scores", "out_o32", "out_m", "out_l", "missed", "wasted")
    state = {n: getattr(st, n).clone() for n in keep}
    lists = [x.clone() for x in st.pred + st.pred_count]
    cur = st.cur
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        stack.step(L.PRR_SCHED_TWO_STREAM, s, spec)
    for t in range(1, 5):
        results = []
        for replay in (False, True):
            for n in keep:
                getattr(st, n).copy_(state[n])
            for x, y in zip(st.pred + st.pred_count, lists):
                x.copy_(y)
            st.cur = cur
            q.copy_(S.q_tensor(qb[t], pc))
            torch.cuda.synchronize()
            if replay:
                graph.replay()
            else:
                stack.step(L.PRR_SCHED_TWO_STREAM, s, spec)
            torch.cuda.synchronize()
            results.append([getattr(st, n).clone() for n in keep] + [st.pred[1 - cur].clone()])
        for x, y in zip(*results):
            assert torch.equal(x, y)


def test_repair_calls_of_other_sizes_share_a_workspace():
    """Serial and exact repairs of several chunk sizes in turn on one workspace: each leaves it
    as the next call needs it."""
    import torch
    from paper_2606_30389_amd import _lib as L
    from paper_2606_30389_amd import runtime as R
    pc = R.PathConfig(num_q_heads=8, num_kv_heads=2, page_size=16, num_tokens=300 * 16 - 3, k_select=70, dtype="f16",
                      chunk_pages=1)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(3)
    k, v = (torch.randn(2, 300, 16, 128, generator=g, device=dev).half() for _ in range(2))
    st = R.LayerState(pc, dev, k=k, v=v)
    q = torch.randn(8, 128, generator=g, device=dev).half()
    order = torch.rand(2, 300, generator=g, device=dev).argsort(dim=-1)
    st.sel[:] = order[:, :70].sort(dim=-1).values
    pred = order[:, 35:105].sort(dim=-1).values.to(torch.int32).contiguous()
    st.sel_count.fill_(70)
    count = st.sel_count.clone()
    results = {True: [], False: []}
    for chunk, serial in [(8, True), (1, False), (16, False), (3, True), (8, False), (1, True), (16, False), (2, True)]:
        S.log(f"repair chunk={chunk} serial={serial}")
        lists = (st.sel, st.sel_count) + ((None, None) if serial else (pred, count))
        if not serial:
            L.prr_spec_attn(st.dims, q, st.k, st.v, None, pc.num_tokens, pred, count, st.cap, chunk, st.part_o, st.part_m,
                            st.part_l, st.page_m)
        for out in (st.out_o32, st.out_m, st.out_l):
            out.fill_(float("nan"))
        L.prr_repair(st.dims, q, st.k, st.v, None, pc.num_tokens, 300, *lists, st.cap, chunk, st.part_o, st.part_m,
                     st.part_l, st.page_m, 0, st.out_o32, st.out_o, st.out_m, st.out_l, st.missed, st.wasted,
                     st.workspace, st.ws_bytes)
        torch.cuda.synchronize()
        results[serial].append((st.out_o32.clone(), st.out_l.clone()))
    for o, l in results[True] + results[False]:
        assert (o - results[True][0][0]).abs().max() < 1e-4 and torch.allclose(l, results[True][0][1], rtol=1e-4)
    assert int(st.workspace[0]) == 0  # no error flag


@pytest.mark.parametrize("events", [True, False])
def test_two_stream_step_that_fails_orders_its_layers(events):
    """A later layer's invalid arguments end the step with its own message; the layers before it
    still run ahead of what the caller enqueues on the speculation stream next."""
    import torch
    from paper_2606_30389_amd import _lib as L
    from paper_2606_30389_amd import runtime as R
    n, reps = 3000, 100
    vals = (45 + np.random.default_rng(5).standard_normal((2, n))).astype(np.float32)
    pc, st, q = _score_layer(torch, vals, 64, [])
    dev = torch.device("cuda:0")
    stack = R.DecodeStack([st] * (reps + 1), [q] * (reps + 1), dev)  # the same layer again and again
    s, spec = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    one = R.DecodeStack([st], [q], dev)
    one.step(L.PRR_SCHED_PREFILL, s)
    torch.cuda.synchronize()
    st.level.zero_()  # (each pass moves it half way towards the scores)
    st.trend.zero_()
    torch.cuda.synchronize()
    stack.io[reps].ws_bytes = 16
    stack.params.epoch = 0
    with pytest.raises(L.PrrError, match="workspace of 16 bytes too small"):
        L.prr_decode_step(stack.dims, stack.params, stack.io, st.cur, L.PRR_SCHED_TWO_STREAM, s, spec,
                          stack.events if events else None)
    with torch.cuda.stream(spec):
        level, trend, count = st.level.clone(), st.trend.clone(), st.pred_count[1 - st.cur].clone()
    torch.cuda.synchronize()
    assert torch.equal(level, st.level) and torch.equal(trend, st.trend)
    assert torch.equal(count, st.pred_count[1 - st.cur]) and int(count[0]) == 64
    assert float((level[:, :n].cpu() - torch.from_numpy(vals)).abs().max()) < 1e-3


def _us(torch, fn, iters=30, reps=5):
    best = float("inf")
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        fn()
        a.record()
        for _ in range(iters):
            fn()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / iters)
    return best


@pytest.mark.parametrize("hkv,n,k", [(1, 4096, 1024), (2, 2500, 625), (2, 4096, 256), (8, 2500, 600), (1, 8192, 1024)])
def test_selection_takes_the_quicker_kernels(hkv, n, k):
    """Where few heads and pages or large budgets make the block-wide kernels the quicker ones, no
    entry takes the others, which need 1.4 to 2.9 times as long there: step 0 against its two
    calls, the selection without scratch against the one with it."""
    import torch
    from paper_2606_30389_amd import _lib as L
    from paper_2606_30389_amd import runtime as R
    rng = np.random.default_rng(n + k)
    vals = (45 + rng.standard_normal((hkv, n))).astype(np.float32)
    pc, st, q = _score_layer(torch, vals, k, [])
    stack = R.DecodeStack([st], [q], torch.device("cuda:0"))
    stream = torch.cuda.current_stream()
    step = _us(torch, lambda: stack.step(L.PRR_SCHED_PREFILL, stream))
    select, predict = _us(torch, lambda: st.select(q)), _us(torch, lambda: st.predict())
    counters = _us(torch, lambda: L.prr_score_topk(st.dims, q, st.meta, n, k, [], True, st.scores, st.sel, st.sel_count,
                                                   st.cap, st.workspace, 512))
    S.log(f"hkv={hkv} n={n} k={k}: step 0 {step:.1f} us, its calls {select:.1f} + {predict:.1f}, counters {counters:.1f}")
    assert step <= 1.15 * (select + predict) and counters <= 1.25 * select
