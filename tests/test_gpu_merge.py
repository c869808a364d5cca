"""prr_merge_states at the edges of its tiles (128 states, 64 channels), of the rule that takes
them, and of the batches (2, 8, 16 states) and vectors (4 channels, aligned) it takes otherwise."""
import numpy as np
import pytest

import oracle as O


@pytest.mark.gpu
@pytest.mark.parametrize("ns,rows,d", [(1, 1, 1), (2, 3, 63), (127, 2, 64), (128, 1, 65), (129, 5, 192), (300, 2, 128),
                                       (7, 1, 1024), (0, 3, 12), (1, 700, 128), (3, 5, 4), (8, 33, 20), (9, 31, 66),
                                       (16, 3, 1000), (17, 272, 64), (17, 273, 64), (64, 513, 128), (300, 1025, 8),
                                       (2, 20000, 13)])
def test_merge_states_edges(ns, rows, d):
    import torch
    import paper_2606_30389_amd as P
    rng = np.random.default_rng(ns * 1000 + d)
    o = rng.standard_normal((ns, rows, d)).astype(np.float32)
    m = (8 * rng.standard_normal((ns, rows))).astype(np.float32)
    l = (0.1 + rng.random((ns, rows))).astype(np.float32)
    empty = rng.random((ns, rows)) < 0.3
    empty[:1] = False
    l[empty], m[empty] = 0.0, -np.inf
    dirty = o.copy()
    dirty[empty] = np.nan  # an empty state's output is never used
    dev = torch.device("cuda:0")
    tt = lambda x: torch.from_numpy(x).to(dev)  # noqa: E731
    out = [torch.full(s, 7.0, device=dev) for s in ((rows, d), (rows,), (rows,))]
    P.prr_merge_states(ns, rows, d, tt(dirty), tt(m), tt(l), *out)
    if ns == 0:
        assert not out[0].any() and torch.all(out[1] == -float("inf")) and not out[2].any()
        return
    if d % 4 == 0:  # the same from outputs that are not 16-byte aligned
        shift = torch.empty(ns * rows * d + 1, device=dev)
        shift[1:] = tt(dirty).flatten()
        again = [torch.full(s, 7.0, device=dev) for s in ((rows, d), (rows,), (rows,))]
        P.prr_merge_states(ns, rows, d, shift[1:].view(ns, rows, d), tt(m), tt(l), *again)
        assert all(torch.equal(x, y) for x, y in zip(out, again))
    ref = O.merge_states([(o[s].astype(np.float64), m[s].astype(np.float64), l[s].astype(np.float64)) for s in range(ns)])
    got = [x.cpu().numpy().astype(np.float64) for x in out]
    # ns float32 products and sums, each rounded to 2^-24, and weights whose exponent (at most
    # about 64 in base 2) is rounded to 2^-24 relative
    bound = (ns + 64) * 2.0 ** -23
    assert np.abs(got[0] - ref[0]).max() <= bound * np.abs(o).max()
    np.testing.assert_array_equal(got[1], ref[1])
    np.testing.assert_allclose(got[2], ref[2], rtol=bound)


@pytest.mark.gpu
def test_merge_of_empty_states():
    import torch
    import paper_2606_30389_amd as P
    dev = torch.device("cuda:0")
    o = torch.full((130, 2, 70), float("nan"), device=dev)
    m, l = torch.full((130, 2), -float("inf"), device=dev), torch.zeros(130, 2, device=dev)
    out = [torch.full(s, 7.0, device=dev) for s in ((2, 70), (2,), (2,))]
    P.prr_merge_states(130, 2, 70, o, m, l, *out)
    assert torch.equal(out[0], torch.zeros(2, 70, device=dev))
    assert torch.equal(out[1], torch.full((2,), -float("inf"), device=dev))
    assert torch.equal(out[2], torch.zeros(2, device=dev))
