"""GPU parity of pool, Gram matrix and max-min around the pool size that one
block takes whole: pools of one frame, of one and two tiles and their edges, one
frame beyond, fewer voted frames than the pool holds, the narrowest and widest
descriptors, several streams."""
import numpy as np
import pytest

import workloads as W
from oracle import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


from parity import dev_bf16, staged_check  # noqa: E402


@pytest.mark.parametrize("Hk,d", [(1, 64), (3, 64), (8, 128)])
@pytest.mark.parametrize("K,mult,F", [(1, 1, 40), (4, 4, 60), (17, 1, 60), (8, 4, 90), (31, 1, 90), (32, 1, 20), (11, 3, 90),
                                      (3, 5, 1)])
def test_pools(Hk, d, K, mult, F):
    import paper_2609_02780_amd as P
    T, k = 6, 25
    gs, os_, qs = [], [], []
    for s in range(2):
        n = F + 7 * s
        cfg = W.Config("tail", 2, 2 * Hk, Hk, d, T, 3, k, K, n_frames=n, n_planted=1, pool_mult=mult)
        q, keys = W.make_stream(cfg, W.stream_specs(cfg)[0], seed=10 * F + s)
        g = P.ShallowIndex(2, 2 * Hk, Hk, d, n, n * T)
        g.append([dev_bf16(x) for x in keys], n, T)
        o = O.Index(2, 2 * Hk, Hk, d)
        o.append(keys, n, T)
        gs.append(g)
        os_.append(o)
        qs.append(q)
    for head_mode in (0, 1):
        out = P.Retriever(gs, k, K, mult, head_mode).debug([[dev_bf16(x) for x in q] for q in qs])
        for s in range(2):
            staged_check(os_[s], qs[s], out, s, k, K, mult, head_mode=head_mode)
            n = out["n_out"][s]
            assert n == min(K, out["pool_n"][s]) and np.all(out["frame_ids"][s, n:] == -1)
            picked = out["frame_ids"][s, :n]
            np.testing.assert_array_equal(out["votes"][s, :n], out["vote_hist"][s][picked])
            np.testing.assert_array_equal(out["mass"][s, :n], out["mass_hist"][s][picked])


@pytest.mark.parametrize("F", [1, 63, 64, 65, 128, 129, 255, 256, 257, 300])
def test_every_frame_voted(F):
    """k beyond the rows: every frame holds votes (equal ones), so the pool is
    the frames of largest mass, at voted counts around those ranked by counting."""
    import paper_2609_02780_amd as P
    T, K, mult = 2, 12, 4
    cfg = W.Config("allvoted", 1, 4, 2, 64, T, 2, 700, K, n_frames=F, n_planted=1, pool_mult=mult)
    q, keys = W.make_stream(cfg, W.stream_specs(cfg)[0], seed=F)
    g = P.ShallowIndex(1, 4, 2, 64, F, F * T)
    g.append([dev_bf16(x) for x in keys], F, T)
    o = O.Index(1, 4, 2, 64)
    o.append(keys, F, T)
    out = P.Retriever([g], 700, K, mult).debug([[dev_bf16(x) for x in q]])
    assert np.all(out["vote_hist"][0, :F] == 4 * T) and out["pool_n"][0] == min(K * mult, F)
    staged_check(o, q, out, 0, 700, K, mult)
