"""One workspace used by calls of several head shapes, page counts and list capacities in turn."""
import pytest

from tests import gpu_support as S

pytestmark = pytest.mark.gpu

# (KV heads, query heads per KV head, pages, page size, pages selected)
SHAPES = [(1, 1, 8192, 16, 40), (8, 4, 600, 16, 250), (2, 16, 3000, 16, 128), (1, 4, 5000, 16, 900), (8, 8, 2600, 16, 1000),
          (8, 1, 300, 128, 64), (70, 2, 200, 16, 20)]


def _layer(torch, R, shape, workspace=None):
    hkv, g, n, ps, k = shape
    pc = R.PathConfig(num_q_heads=hkv * g, num_kv_heads=hkv, page_size=ps, num_tokens=n * ps - 5, k_select=k, dtype="f16",
                      chunk_pages=max(1, 128 // ps), gamma=0.25)
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(hkv * 100 + g)
    kv = [torch.randn(hkv, n, ps, 128, generator=gen, device=dev, dtype=torch.float16) for _ in range(2)]
    st = R.LayerState(pc, dev, k=kv[0], v=kv[1])
    if workspace is not None:
        assert workspace.numel() * 4 >= st.ws_bytes
        st.workspace = workspace
    st.build_meta()
    q = torch.randn(hkv * g, 128, generator=gen, device=dev).half()
    return st, R.DecodeStack([st], [q], dev), q


def test_head_shapes_share_a_workspace():
    """Selections, predictions and repairs of every shape give on the shared workspace, where
    other shapes' data lies when they begin, bit for bit what they give on one of their own."""
    import torch
    from paper_2606_30389_amd import _lib as L
    from paper_2606_30389_amd import runtime as R
    stream, spec = torch.cuda.current_stream(), torch.cuda.Stream()
    own = [_layer(torch, R, s) for s in SHAPES]
    bytes_ = max(st.ws_bytes for st, _, _ in own)
    shared = torch.empty(bytes_ // 4 + 64, dtype=torch.int32, device="cuda:0")
    L.prr_workspace_init(shared, bytes_)
    both = [(o, _layer(torch, R, s, shared)) for s, o in zip(SHAPES, own)]
    names = ("out_o32", "out_o", "out_m", "out_l", "scores", "level", "trend", "init_bits", "sel", "sel_count", "missed",
             "wasted")
    g = torch.Generator(device="cuda:0").manual_seed(11)
    for step, schedule in enumerate((L.PRR_SCHED_PREFILL, L.PRR_SCHED_TWO_STREAM, L.PRR_SCHED_SERIAL,
                                     L.PRR_SCHED_TWO_STREAM)):
        order = range(len(SHAPES)) if step % 2 == 0 else reversed(range(len(SHAPES)))
        for i in order:
            S.log(f"step {step} shape {SHAPES[i]}")
            noise = 0.5 * torch.randn(both[i][0][2].shape, generator=g, device="cuda:0").half()
            for _, stack, q in both[i]:
                q += noise
                stack.step(schedule, stream, spec)
            torch.cuda.synchronize()
            a, b = both[i][0][0], both[i][1][0]
            for name in names:
                assert torch.equal(getattr(a, name), getattr(b, name)), (SHAPES[i], step, name)
            assert torch.equal(a.pred_count[a.cur], b.pred_count[b.cur]) and torch.equal(a.pred[a.cur], b.pred[b.cur])
            if schedule == L.PRR_SCHED_TWO_STREAM:
                assert int(a.missed.sum()) > 0, "nothing to repair"
            assert int(a.workspace[0]) == 0 and int(b.workspace[0]) == 0, "workspace error flags"
