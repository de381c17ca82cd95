"""GPU parity of the sample cut-off over the block sizes it is launched in:
samples of whole lists around the slots of four and of sixteen waves, and long
lists of few and of more than 512 lists, one sample size on each side of every
switch."""
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


def _stream(P, L, Hq, Hk, F, T, k, K, seed):
    cfg = W.Config("cutoff", L, Hq, Hk, 64, T, 3, k, K, n_frames=F, n_planted=1)
    q, keys = W.make_stream(cfg, W.stream_specs(cfg)[0], seed=seed)
    g = P.ShallowIndex(L, Hq, Hk, 64, F, F * T)
    g.append([dev_bf16(x) for x in keys], F, T)
    o = O.Index(L, Hq, Hk, 64)
    o.append(keys, F, T)
    return g, o, q


@pytest.mark.parametrize("n", [1, 63, 255, 256, 257, 1792, 1793, 2047, 2048, 2049, 4096])
def test_whole_list_samples(n):
    """Head-averaged lists of up to 4,096 rows: the sample is the list and the
    cut-off its k-th largest score."""
    import paper_2609_02780_amd as P
    k, K = 100, 4
    g, o, q = _stream(P, 2, 4, 2, n, 1, k, K, seed=n)
    out = P.Retriever([g], k, K, head_mode=1).debug([[dev_bf16(x) for x in q]])
    assert np.all(out["list_stats"][0, :, 1] == 0)
    staged_check(o, q, out, 0, k, K, head_mode=1)


@pytest.mark.parametrize("S", [2, 17])
@pytest.mark.parametrize("F", [1400, 2400, 2900, 5200, 6000])
def test_long_list_samples(F, S):
    """One list set of 140,000 to 600,000 rows (about 1,900 to 8,200 of them
    sampled) beside short ones; 17 streams are 544 lists."""
    import paper_2609_02780_amd as P
    k, K = 100, 4
    parts = [_stream(P, 2, 16, 1, F if s == 1 else 40, 100 if s == 1 else 3, k, K, seed=s) for s in range(S)]
    out = P.Retriever([g for g, _, _ in parts], k, K).debug([[dev_bf16(x) for x in q] for _, _, q in parts])
    for s in (0, 1, S - 1):
        assert np.all(out["list_stats"][s, :, 1] == 0)
        staged_check(parts[s][1], parts[s][2], out, s, k, K)
