"""GPU parity of lists short enough to be selected from every row's score: list
lengths around the per-thread slots of the selection, k from 1 to more than the
rows, ties, batches of unequal lists, both readings; and the same calls through
the sampled route where the workspace leaves only that one."""
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


@pytest.mark.parametrize("score_mode", [0, 1])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("nqs", [(768,), (769,), (4096,), (3, 1000, 1)])
def test_long_questions(nqs, d, score_mode):
    """Questions around the token count from which the query tiles are formed by a
    kernel of their own, and a batch that mixes them with short ones; both routes."""
    import paper_2609_02780_amd as P
    k, K = 50, 5
    parts = [_stream(P, 2, 6, 2, d, 70 + 9 * i, 13, nq, k, K, seed=i) for i, nq in enumerate(nqs)]
    r = P.Retriever([g for g, _, _ in parts], k, K, score_mode=score_mode)
    outs = [r.debug([[dev_bf16(x) for x in q] for _, _, q in parts], stats=stats) for stats in (False, True)]
    for s, (_, o, q) in enumerate(parts):
        for out in outs:
            staged_check(o, q, out, s, k, K, score_mode=score_mode)
        np.testing.assert_array_equal(outs[0]["topk_pos"][s], outs[1]["topk_pos"][s])
        if score_mode == 0:
            assert np.array_equal(outs[0]["topk_score"][s].view(np.uint32), outs[1]["topk_score"][s].view(np.uint32))


def _stream(P, L, Hq, Hk, d, F, T, nq, k, K, seed, recent=0):
    cfg = W.Config("short", L, Hq, Hk, d, T, nq, k, K, n_frames=F, n_planted=1)
    spec = W.stream_specs(cfg)[0]
    q, keys = W.make_stream(cfg, spec, seed=seed)
    g = P.ShallowIndex(L, Hq, Hk, d, F, F * T, recent)
    g.append([dev_bf16(x) for x in keys], F, T)
    o = O.Index(L, Hq, Hk, d, recent)
    o.append(keys, F, T)
    return g, o, q


@pytest.mark.parametrize("score_mode", [0, 1])
@pytest.mark.parametrize("L,Hq,Hk,d,F,T,k", [
    (1, 2, 1, 64, 1, 1, 5), (2, 4, 2, 64, 3, 5, 16), (1, 7, 1, 128, 16, 16, 200), (2, 4, 4, 64, 41, 25, 257),
    (1, 2, 1, 64, 256, 16, 1024), (1, 2, 1, 128, 241, 17, 64), (1, 4, 1, 64, 512, 16, 1000), (1, 2, 2, 64, 483, 17, 1),
    (1, 2, 1, 64, 1024, 16, 512), (1, 2, 1, 128, 1639, 10, 33), (1, 2, 1, 64, 2048, 16, 700),
    (1, 2, 1, 64, 2048, 16, 1024), (1, 2, 1, 128, 1200, 16, 960), (1, 2, 1, 64, 331, 25, 1024), (1, 2, 1, 64, 300, 15, 1024)])
def test_short_lists(L, Hq, Hk, d, F, T, k, score_mode):
    import paper_2609_02780_amd as P
    g, o, q = _stream(P, L, Hq, Hk, d, F, T, 3, k, 4, seed=F)
    r = P.Retriever([g], k, 4, score_mode=score_mode)
    out = r.debug([[dev_bf16(x) for x in q]], stats=False)
    staged_check(o, q, out, 0, k, 4, score_mode=score_mode)
    plain = r([[dev_bf16(x) for x in q]])
    for key, t in zip(("frame_ids", "votes", "mass", "n_out"), plain):
        assert np.array_equal(t.cpu().numpy().view(np.uint8), out[key].view(np.uint8)), key


@pytest.mark.parametrize("score_mode", [0, 1])
@pytest.mark.parametrize("n,above,tied,k", [(20000, 500, 6000, 1000), (32768, 1023, 9000, 1024), (9000, 0, 8990, 1000),
                                            (20000, 999, 1, 1000), (8192, 100, 4200, 1024)])
def test_many_ties_at_the_cut(n, above, tied, k, score_mode):
    """``above`` rows over ``tied`` equal ones over the rest, k ending among the
    equal ones: more rows reach the cut than are kept for the selection, from
    the first bound and (k near the number of threads) from the closer one."""
    import paper_2609_02780_amd as P
    T = 8
    rng = np.random.default_rng(n + above)
    v = np.concatenate([2.0 + np.arange(above) / 64.0, np.ones(tied), -1.0 - rng.random(n - above - tied)])
    x = np.zeros((1, n, 64), np.float32)
    x[0, :, 5] = rng.permutation(v)
    keys = [W.bf16_bits(x)]
    q = np.zeros((2, 1, 64), np.float32)
    q[0, 0, 5], q[1, 0, 5] = 1.0, 0.25
    q = [W.bf16_bits(q)]
    g = P.ShallowIndex(1, 2, 1, 64, n // T, n)
    g.append([dev_bf16(keys[0])], n // T, T)
    o = O.Index(1, 2, 1, 64)
    o.append(keys, n // T, T)
    out = P.Retriever([g], k, 4, score_mode=score_mode).debug([[dev_bf16(q[0])]], stats=False)
    rep = staged_check(o, q, out, 0, k, 4, score_mode=score_mode)
    assert rep.get("swaps", 0) == 0


def test_unequal_batch_with_an_empty_stream():
    """One launch for lists of 24,000, 4,097, 300 and 8 rows, and a stream whose
    frames are all in its recent window."""
    import paper_2609_02780_amd as P
    k, K = 100, 6
    parts = [_stream(P, 2, 6, 2, 64, F, T, nq, k, K, seed=i, recent=rec)
             for i, (F, T, nq, rec) in enumerate([(1500, 16, 1, 0), (4097, 1, 5, 0), (60, 5, 17, 0), (5, 2, 64, 1), (3, 4, 2, 3)])]
    r = P.Retriever([g for g, _, _ in parts], k, K)
    for stats in (False, True):
        out = r.debug([[dev_bf16(x) for x in q] for _, _, q in parts], stats=stats)
        for s, (_, o, q) in enumerate(parts[:4]):
            staged_check(o, q, out, s, k, K)
        assert out["n_out"][4] == 0 and np.all(out["frame_ids"][4] == -1)


@pytest.mark.parametrize("S", [1, 40])
@pytest.mark.parametrize("score_mode", [0, 1])
def test_stats_are_the_streaming_pass(score_mode, S):
    """Lists of 8,192 rows whose statistics are asked for: the counts are the
    rows at or above the sample's cut-off (about the planner's expectation, more
    than k), not those at or above the k-th score, in a workspace of the size
    that the library asks for."""
    import paper_2609_02780_amd as P
    k = 40
    g, o, q = _stream(P, 1, 2, 1, 64, 512, 16, 3, k, 4, seed=9)
    m, _, cap, E = P.sample_plan(8192, k)
    assert m < 8192 and E > 2 * k
    r = P.Retriever([g] * S, k, 4, score_mode=score_mode)
    out = r.debug([[dev_bf16(x) for x in q]] * S)
    for s in {0, S - 1}:
        stats = out["list_stats"][s]
        assert np.all(stats[:, 1] == 0) and np.all(stats[:, 0] <= cap)
        assert np.all(stats[:, 0] > k + k // 4), stats
        staged_check(o, q, out, s, k, 4, score_mode=score_mode)


@pytest.mark.parametrize("bad", [0x7FC0, 0xFFC0, 0x7F80, 0xFF80])
@pytest.mark.parametrize("n", [3000, 9000, 20000, 32768])
def test_non_finite_keys(n, bad):
    """Three rows with a NaN or an infinity among lists that the other route takes
    whole (3,000 rows) or samples: the same lists and votes on both, and no NaN
    row in the sampled ones."""
    import paper_2609_02780_amd as P
    T, k = 8, 64
    rng = np.random.default_rng(n)
    bits = W.bf16_bits(rng.standard_normal((2, n, 64)).astype(np.float32))
    rows = [7, n // 2, n - 1]
    bits[1, rows, [3, 40, 63]] = bad
    g = P.ShallowIndex(1, 4, 2, 64, n // T, n)
    g.append([dev_bf16(bits)], n // T, T)
    q = [dev_bf16(W.bf16_bits(rng.standard_normal((4, 2, 64)).astype(np.float32)))]
    r = P.Retriever([g], k, 4)
    a, b = r.debug([q], stats=False), r.debug([q])
    np.testing.assert_array_equal(a["topk_pos"], b["topk_pos"])
    np.testing.assert_array_equal(a["vote_hist"], b["vote_hist"])
    assert (P.sample_plan(n, k)[0] < n) == (n > 4096)
    if n > 4096 and (bad & 0x7FFF) > 0x7F80:
        assert not np.isin(a["topk_pos"], rows).any()


@pytest.mark.parametrize("T,dup", [(16, 1), (16, 40), (16, 100000)])
def test_routes_agree(T, dup):
    """The same call on its own route, with a workspace that has no room for every
    row's score, and with the streaming pass's statistics asked for: lists, votes
    and masses bit for bit.  ``dup`` equal
    rows in a row make ties at the cut (with all rows equal the lists are rows
    0 .. k - 1, and more rows tie than either route keeps)."""
    import paper_2609_02780_amd as P
    L, Hq, Hk, d, F, k, K = 1, 4, 2, 64, 2000, 90, 5
    rng = np.random.default_rng(dup)
    x = rng.standard_normal((Hk, F * T, d)).astype(np.float32)[:, np.arange(F * T) // dup * dup]
    g = P.ShallowIndex(L, Hq, Hk, d, F, F * T)
    g.append([dev_bf16(W.bf16_bits(x))], F, T)
    q = [dev_bf16(W.bf16_bits(rng.standard_normal((Hq, 2, d)).astype(np.float32)))]
    for score_mode in (0, 1):
        r = P.Retriever([g], k, K, score_mode=score_mode)
        a = r.debug([q], stats=False)
        need = r.workspace_bytes([2])
        small = P.Retriever([g], k, K, score_mode=score_mode)
        small._ws = torch.empty(need - 256, dtype=torch.uint8, device="cuda")
        small.workspace_bytes = lambda n_q: 1
        b = small.debug([q], stats=False)
        c = small.debug([q])
        if dup > F * T:
            np.testing.assert_array_equal(a["topk_pos"][0], np.tile(np.arange(k), (Hq, 1)))
        keys = ["topk_pos", "vote_hist"] + (["frame_ids", "votes", "topk_score", "mass", "mass_hist"] if score_mode == 0 else [])
        for key in keys:
            assert np.array_equal(a[key].view(np.uint8), b[key].view(np.uint8)), key
        for key in b:   # both the sampled route
            assert np.array_equal(b[key].view(np.uint8), c[key].view(np.uint8)), key
        # probabilities: two fixed-point sums of the normaliser, 2^-40 apart per row, and fp32 exp and log
        np.testing.assert_allclose(a["topk_score"], b["topk_score"], rtol=4e-6)
        np.testing.assert_allclose(a["mass_hist"], b["mass_hist"], rtol=4e-6)


@pytest.mark.parametrize("score_mode", [0, 1])
def test_fallback_of_long_lists_with_equal_rows(score_mode):
    """Zero queries over 40,000 rows, more than the lists selected from every
    score: every row ties at the cut-off, the candidate buffer overflows and
    the exact fallback returns rows 0 .. k - 1."""
    import paper_2609_02780_amd as P
    g, o, q = _stream(P, 1, 2, 1, 64, 2500, 16, 1, 40, 3, seed=5)
    zq = [np.zeros_like(x) for x in q]
    out = P.Retriever([g], 40, 3, score_mode=score_mode).debug([[dev_bf16(x) for x in zq]])
    assert np.all(out["list_stats"][0, :, 1] == 1)
    np.testing.assert_array_equal(out["topk_pos"][0], np.tile(np.arange(40), (2, 1)))
