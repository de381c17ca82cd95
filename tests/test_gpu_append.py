"""GPU parity of an append's arena entries at the edges of its kernels: head
counts that leave threads idle, fewer tokens than token slices, token counts
around one round of loads, several appends in a row; raw and compressed."""
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


@pytest.mark.parametrize("compress", [None, (4, 2)])
@pytest.mark.parametrize("L,Hk,d,T", [(1, 1, 64, 1), (2, 3, 128, 5), (1, 16, 64, 9), (2, 8, 128, 57), (3, 4, 128, 112),
                                      (2, 4, 128, 113), (1, 5, 64, 256), (2, 1, 128, 196)])
def test_append_entries(L, Hk, d, T, compress):
    import paper_2609_02780_amd as P
    rng = np.random.default_rng(T)
    parts = (2, 1, 3)                                     # frames of each append call
    F, rpf = sum(parts), T if compress is None else min(compress[0], T)
    keys = [W.bf16_bits(rng.standard_normal((Hk, F, T, d)).astype(np.float32)) for _ in range(L)]
    g = P.ShallowIndex(L, 2 * Hk, Hk, d, F, F * rpf)
    f0 = 0
    for n in parts:
        block = [torch.from_numpy(np.ascontiguousarray(k[:, f0:f0 + n]).reshape(Hk, n * T, d).view(np.int16)).cuda() for k in keys]
        assert g.append(block, n, T, compress) == f0
        f0 += n
    ex = g.export()
    assert ex["frame_offsets"] == [rpf * f for f in range(F + 1)]
    X = np.stack([O.decode_bf16(k) for k in keys])        # [L][Hk][F][T][d]
    if compress is None:
        for l in range(L):
            np.testing.assert_array_equal(ex["rows"][l], keys[l].reshape(Hk, F * T, d))
        assert np.all(ex["counts"] == 1)
    # fp32 sums of at most 256 terms against float64: T 2^-24 relative to the sum of magnitudes at worst
    want = X.mean(axis=3).transpose(2, 0, 1, 3)           # [F][L][Hk][d]
    tol = T * 2.0 ** -23 * np.abs(X).mean(axis=3).transpose(2, 0, 1, 3) + 1e-12
    a = g.arena
    lg, al = L * Hk, lambda n: (n + 255) // 256 * 256
    at = al(lg * F * rpf * d * 2)
    at = al(at + lg * F * rpf * 4)
    at = al(at + F * Hk * d * 4)
    pooled = a[at:at + F * lg * d * 4].view(torch.float32).cpu().numpy().reshape(F, L, Hk, d)
    assert np.all(np.abs(pooled - want) <= tol)
    desc = np.array([O.descriptor(X[-1][:, f]) for f in range(F)])
    np.testing.assert_allclose(ex["desc"], desc, atol=T * 2.0 ** -22)
    off = at + al(F * lg * d * 4)
    offs = a[off:off + (F + 1) * 4].view(torch.int32).cpu().numpy()
    np.testing.assert_array_equal(offs, rpf * np.arange(F + 1))
    kmax = a[al(off + (F + 1) * 4):][:4].view(torch.float32).item()
    assert kmax == np.abs(X).max()


@pytest.mark.parametrize("compress", [None, (4, 2)])
@pytest.mark.parametrize("bad", [0x7FC0, 0xFFC0, None])
def test_descriptor_of_a_frame_without_a_norm(bad, compress):
    """A NaN among a frame's last-layer keys, or keys that are all zero: that
    frame's descriptor is zeros, the others' are untouched."""
    import paper_2609_02780_amd as P
    rng = np.random.default_rng(3)
    Hk, F, T, d = 2, 3, 9, 64
    bits = W.bf16_bits(rng.standard_normal((Hk, F, T, d)).astype(np.float32))
    if bad is None:
        bits[:, 1] = 0
    else:
        bits[1, 1, 4, 7] = bad
    g = P.ShallowIndex(1, Hk, Hk, d, F, F * T)
    g.append([torch.from_numpy(bits.reshape(Hk, F * T, d).view(np.int16)).cuda()], F, T, compress)
    desc = g.export()["desc"]
    assert np.all(desc[1] == 0)
    for f in (0, 2):
        np.testing.assert_allclose(desc[f], O.descriptor(O.decode_bf16(bits[:, f])), atol=T * 2.0 ** -22)
