"""GPU parity of the append-time k-means at the edges of its layout: token
counts around the 16-token tiles, the 32-token steps and the 64-token waves,
centroid counts around the 16-centre tiles, and exact ties between tokens of
different tiles and waves."""
import numpy as np
import pytest

import workloads as W
from oracle import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# a decision whose relative margin is below this may fall either way in fp32
# (about ten times the relative error of a 128-term squared distance)
MARGIN = 1e-5


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _compress(bits, T, n_c, n_it):
    """bits [H_kv][F*T][d] -> (rows [H_kv][F][c][d], counts [H_kv][F][c])."""
    import paper_2609_02780_amd as P
    Hk, n, d = bits.shape
    F, c = n // T, min(n_c, T)
    g = P.ShallowIndex(1, Hk, Hk, d, F, F * c)
    g.append([torch.from_numpy(bits.view(np.int16)).cuda()], F, T, (n_c, n_it))
    ex = g.export()
    return ex["rows"][0].reshape(Hk, F, c, d), ex["counts"][0].reshape(Hk, F, c)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T,n_c,n_it", [(1, 1, 2), (15, 3, 2), (16, 16, 3), (17, 17, 1), (31, 16, 4), (33, 20, 4),
                                        (64, 32, 3), (65, 33, 5), (97, 48, 0), (196, 32, 10), (255, 49, 4), (256, 64, 6)])
def test_kmeans_edges(T, n_c, n_it, d):
    rng = np.random.default_rng(1000 * T + n_c)
    Hk, F = 2, 3
    z = rng.standard_normal((Hk, F, 1, d))
    bits = W.bf16_bits((z + 0.5 * rng.standard_normal((Hk, F, T, d))).astype(np.float32).reshape(Hk, F * T, d))
    rows, counts = _compress(bits, T, n_c, n_it)
    exact = 0
    for g in range(Hk):
        for f in range(F):
            X = O.decode_bf16(bits[g, f * T:(f + 1) * T])
            C, cnt, dg = O.kmeans(X, n_c, n_it)
            assert counts[g, f].sum() == (T if n_it else 0)
            if min(dg["init_margin"], dg["assign_margin"]) < MARGIN:
                continue
            exact += 1
            diff = np.abs(rows[g, f].astype(np.int32) - O.round_bf16(C).astype(np.int32))
            assert diff.max() <= 1, (g, f)          # one bf16 unit: the fp32 sums' rounding
            np.testing.assert_array_equal(counts[g, f], cnt)
    assert exact >= 1


@pytest.mark.parametrize("copies", [2, 3, 8, 96])
@pytest.mark.parametrize("n_c", [5, 32, 40])
def test_kmeans_equal_tokens(copies, n_c):
    """Every token of a frame ``copies`` times, the copies a whole number of
    tokens apart (other tiles, other waves): picks and centres tie exactly, and
    the lower token and the lower centre win; centres without members stay."""
    T, d = 96, 128
    rng = np.random.default_rng(copies)
    base = rng.standard_normal((T // copies, d)).astype(np.float32)
    bits = W.bf16_bits(np.tile(base, (copies, 1)))[None]
    rows, counts = _compress(bits, T, n_c, 3)
    C, cnt, _ = O.kmeans(O.decode_bf16(bits[0]), n_c, 3)
    assert np.abs(rows[0, 0].astype(np.int32) - O.round_bf16(C).astype(np.int32)).max() <= 1
    np.testing.assert_array_equal(counts[0, 0], cnt)


@pytest.mark.parametrize("bad", [0x7FC0, 0xFFC0, 0xFFFF, 0x7F80, 0xFF80])
@pytest.mark.parametrize("T,n_c,d", [(17, 4, 64), (70, 16, 128), (196, 33, 128)])
def test_kmeans_non_finite_tokens(T, n_c, d, bad):
    """One NaN or infinity in a frame, of either sign: the mean and every distance
    from it are NaN (or infinite), and the picks must still be distinct tokens of
    the frame (the stored rows of no rounds at all); after rounds every token has
    one centre."""
    rng = np.random.default_rng(bad + T)
    bits = W.bf16_bits(rng.standard_normal((1, 2 * T, d)).astype(np.float32))
    bits[0, T // 2, 3] = bad
    rows, _ = _compress(bits, T, n_c, 0)
    tokens = {t.tobytes(): i for i, t in enumerate(bits[0, :T])}
    picks = [tokens.get(r.tobytes(), -1) for r in rows[0, 0]]
    assert min(picks) >= 0 and len(set(picks)) == n_c, picks
    assert picks[0] in (0, T // 2)                  # equal distances from the mean, or the odd one's NaN above them
    rows, counts = _compress(bits, T, n_c, 3)
    assert np.all(counts.sum(axis=-1) == T)
    C, cnt, dg = O.kmeans(O.decode_bf16(bits[0, T:]), n_c, 3)      # the other frame is untouched by it
    if min(dg["init_margin"], dg["assign_margin"]) >= MARGIN:
        assert np.abs(rows[0, 1].astype(np.int32) - O.round_bf16(C).astype(np.int32)).max() <= 1
        np.testing.assert_array_equal(counts[0, 1], cnt)
