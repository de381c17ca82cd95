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
    assert exact >= 4, exact      # of six; the oracle's margins of these draws leave four to six


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


@pytest.mark.parametrize("common", [3.0, 8.0, 30.0])
@pytest.mark.parametrize("T,n_c,d", [(196, 16, 128), (196, 32, 128), (256, 33, 128), (196, 48, 64), (256, 64, 128),
                                     (250, 64, 64)])
def test_kmeans_common_component(T, n_c, d, common):
    """Tokens around a common vector many times longer than what sets them apart:
    the dot products' bounds are wide, so most picks and many assignments are
    decided again.  Each pick has to be a farthest token, and after one round
    each centre whose members are beyond doubt has to be their mean, up to the
    direct form's rounding (d + 2 roundings of a sum of squares)."""
    rng = np.random.default_rng(int(common) * 1000 + T + n_c)
    F, tol = 2, (d + 2) * 2.0 ** -23
    x = common * rng.standard_normal(d) + 0.5 * rng.standard_normal((F * T, d))
    bits = W.bf16_bits(x.astype(np.float32))[None]
    rows0, _ = _compress(bits, T, n_c, 0)
    rows1, counts = _compress(bits, T, n_c, 1)
    settled = 0
    for f in range(F):
        tok = bits[0, f * T:(f + 1) * T]
        X = O.decode_bf16(tok)
        at = {t.tobytes(): i for i, t in reversed(list(enumerate(tok)))}
        picks = [at[r.tobytes()] for r in rows0[0, f]]
        assert len(set(picks)) == n_c
        far = ((X - X.mean(0)) ** 2).sum(1)
        # the mean is a sum of T terms in fp32, each addition off by at most 2^-24 of the sum
        mean_err = np.sqrt(d) * np.abs(X).max() * T * 2.0 ** -24
        assert far[picks[0]] >= far.max() * (1 - tol) - 2 * np.sqrt(far.max()) * mean_err
        near = np.full(T, np.inf)
        for i, p in enumerate(picks):
            if i:
                free = np.ones(T, bool)
                free[picks[:i]] = False
                assert near[p] >= near[free].max() * (1 - tol), (f, i)
            near = np.minimum(near, ((X - X[p]) ** 2).sum(1))
        dist = ((X[:, None] - X[picks][None]) ** 2).sum(-1)
        two = np.sort(dist, 1)[:, :2]
        doubt = two[:, 1] - two[:, 0] <= tol * two[:, 1]
        member = dist.argmin(1)
        assert counts[0, f].sum() == T
        for c in range(n_c):
            if np.any(doubt & (dist[:, c] <= two[:, 1])):
                continue
            mine = member == c
            settled += 1
            assert counts[0, f, c] == mine.sum()
            diff = np.abs(rows1[0, f, c].astype(np.int32) - O.round_bf16(X[mine].mean(0)).astype(np.int32))
            assert diff.max() <= 1, (f, c)
    assert settled >= 1.8 * n_c   # of 2 n_c centres
