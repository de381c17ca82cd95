"""The calls whose speed counts: a list of named cases, more of the same ranges on
demand, and a plain 64-bit torch reference of what each returns.

Three kinds of case:

- ``retrieve``: one question per stream against indices that are in place
  (:class:`Retriever`), single streams from a few seconds to an hour and ragged
  batches, raw and k-means compressed, per-head and head-averaged lists, logits
  and attention probabilities;
- ``append``: a stream's frames entering a new index, one call per frame (a live
  stream) or one call per clip, raw or compressed;
- ``session``: a stream that outgrows its detailed window: appends, the byte
  budget, absorption into long-term clusters, compaction, then a question over
  both memories and the evidence for it.

Frames are the workloads' clustered Gaussians (a centroid per frame, layer and
KV head; tokens around it; a few frames planted along the question's mean
query).  In a session neighbouring frames share a scene, as a video's do.
"""
import math
import random

import numpy as np
import torch

from paper_2609_02780_amd.index import LongClusters, PooledRanker, Retriever, ShallowIndex, assemble_evidence

CHUNK = 100        # frames generated and appended at a time when an index is prepared

# n_layers, n_q_heads, n_kv_heads, head_dim
TINY = (2, 4, 2, 64)
QWEN7B = (4, 28, 4, 128)
QWEN3B = (6, 16, 2, 128)
QWEN8B = (5, 32, 8, 128)
MHA64 = (4, 16, 16, 64)


def _shape(s):
    return {"layers": s[0], "q_heads": s[1], "kv_heads": s[2], "dim": s[3]}


def _retrieve(shape, frames, tokens, nq, top_k, select, **more):
    c = {"kind": "retrieve", **_shape(shape), "streams": 1, "frames": frames, "frames_lo": frames, "tokens": tokens,
         "nq": nq, "top_k": top_k, "select": select, "head_mode": 0, "score_mode": 0, "recent": 0,
         "centroids": 0, "iters": 0, "every": 1, "planted_every": 150}
    c.update(more)
    return c


def _append(shape, frames, tokens, step, centroids=0, iters=0):
    return {"kind": "append", **_shape(shape), "frames": frames, "tokens": tokens, "step": step,
            "centroids": centroids, "iters": iters}


def _session(shape, frames, tokens, step, keep, centroids=0, iters=0, **more):
    c = {"kind": "session", **_shape(shape), "frames": frames, "tokens": tokens, "step": step, "keep": keep,
         "centroids": centroids, "iters": iters, "scene": 8, "tau": 0.5, "recent": 6, "nq": 32, "top_k": 64,
         "select": 8, "clusters": 8}
    c.update(more)
    return c


def listed():
    return [
        # the smallest index a test or a first minute of a stream has: launches and latency
        dict(name="retrieve_tiny", **_retrieve(TINY, 64, 16, 8, 32, 4, planted_every=32)),
        # a ten-minute stream at one frame a second, every list kept per query head
        dict(name="retrieve_10min", **_retrieve(QWEN7B, 600, 196, 32, 256, 16, planted_every=75)),
        # the same stream after k-means compression: few rows, all of them from cache
        dict(name="retrieve_10min_compressed", **_retrieve(QWEN7B, 600, 196, 32, 64, 16, centroids=32, iters=10, planted_every=75)),
        # an hour of video: the index streams from memory
        dict(name="retrieve_1h", **_retrieve(QWEN7B, 3600, 196, 64, 512, 32)),
        # sixteen users' streams of 5 to 60 minutes in one call, every other one compressed
        dict(name="retrieve_16_streams", **_retrieve(QWEN3B, 3600, 196, 32, 256, 16, streams=16, frames_lo=300, centroids=32, iters=10, every=2)),
        # the method's own settings on the hour: last prompt token, head-averaged lists, six recent frames left out
        dict(name="retrieve_1h_head_mean", **_retrieve(QWEN7B, 3600, 196, 1, 64, 8, head_mode=1, recent=6)),
        # the same settings read as attention probabilities, at seventeen minutes and an odd token count
        dict(name="retrieve_17min_probabilities", **_retrieve(QWEN7B, 1024, 187, 1, 64, 8, head_mode=1, score_mode=1, recent=6)),
        # a live stream: sixteen frames, one append call for each
        dict(name="append_live", **_append(QWEN7B, 16, 196, 1)),
        # a recorded ten-minute clip entering in one call
        dict(name="append_clip", **_append(QWEN7B, 600, 196, 600)),
        # the live stream with per-frame compression
        dict(name="append_live_compressed", **_append(QWEN7B, 16, 196, 1, 32, 10)),
        # the clip with per-frame compression
        dict(name="append_clip_compressed", **_append(QWEN7B, 600, 196, 600, 32, 10)),
        # a stream that outgrows its window: clusters, compaction, then a question over both memories
        dict(name="session_long_history", **_session(QWEN7B, 400, 196, 50, 150)),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.random()
    if what < 0.40:
        shape = rng.choice([TINY, QWEN7B, QWEN7B, QWEN3B, QWEN8B, MHA64])
        frames, tokens = _log(rng, 64, 3600), rng.randint(16, 256)
        head_mode = 1 if rng.random() < 0.4 and shape[2] <= 8 else 0
        score_mode = 1 if rng.random() < 0.4 and (head_mode == 0 or shape[2] * shape[3] <= 512) else 0
        comp = rng.random() < 0.3
        while frames * tokens * shape[0] * shape[2] * shape[3] * 2 > 3.2e9:
            frames = frames * 2 // 3
        return _retrieve(shape, frames, tokens, _log(rng, 1, 64), _log(rng, 32, 512), rng.randint(4, 32),
                         head_mode=head_mode, score_mode=score_mode, recent=rng.choice([0, 6]),
                         centroids=rng.randint(8, 48) if comp else 0, iters=rng.randint(4, 10) if comp else 0,
                         planted_every=rng.randint(40, 200))
    if what < 0.50:
        shape = rng.choice([QWEN7B, QWEN3B])
        lo, comp = _log(rng, 64, 600), rng.random() < 0.6
        return _retrieve(shape, rng.randint(2 * lo, 1800), rng.randint(49, 196), _log(rng, 1, 64), _log(rng, 32, 512),
                         rng.randint(4, 24), streams=rng.randint(2, 12), frames_lo=lo,
                         centroids=rng.randint(16, 40) if comp else 0, iters=rng.randint(4, 10) if comp else 0, every=2)
    shape = rng.choice([TINY, QWEN7B, QWEN7B, QWEN3B, QWEN8B])
    if what < 0.88:
        tokens = rng.randint(16, 256)
        comp = rng.random() < 0.5
        live = rng.random() < 0.5
        frames = rng.randint(4, 24) if live else _log(rng, 32, 600)
        thirds = rng.random() < 0.5
        centroids, iters = (rng.randint(8, 64), rng.randint(2, 12)) if comp else (0, 0)
        while frames * tokens * shape[0] * shape[2] * shape[3] * min(centroids, tokens) * (1 + iters) > 8e10:
            frames = frames * 2 // 3
        return _append(shape, frames, tokens, 1 if live else max(2, frames // 3) if thirds else frames, centroids, iters)
    comp = rng.random() < 0.5
    keep, step = rng.randint(60, 200), rng.randint(17, 64)
    return _session(shape, keep + rng.randint(60, 250), rng.randint(49, 196), step, keep,
                    rng.randint(16, 32) if comp else 0, rng.randint(4, 10) if comp else 0, top_k=_log(rng, 32, 256),
                    select=rng.randint(4, 16), nq=_log(rng, 1, 64))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------


def _lengths(case):
    """Frames of each stream: the largest first, the others spread over the range."""
    if case["streams"] == 1:
        return [case["frames"]]
    r = random.Random(case["frames"] * 1000 + case["streams"])
    return [case["frames"]] + [r.randint(case["frames_lo"], case["frames"]) for _ in range(case["streams"] - 1)]


def _compress(case, stream=0):
    """(n_centroids, n_iters) of a stream, or None; in a batch every ``every``-th stream is compressed."""
    every = case.get("every", 1)
    return (case["centroids"], case["iters"]) if case["centroids"] and stream % every == every - 1 else None


def _rows(case, stream=0):
    c = _compress(case, stream)
    return min(c[0], case["tokens"]) if c else case["tokens"]


def _generator(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000 + stream)
    return g


def _queries(case, gen):
    shape = (case["q_heads"], case["nq"], case["dim"])
    return [torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(case["layers"])]


def _directions(case, queries):
    """Unit mean query of each (layer, KV head)."""
    m = torch.stack([q.float().reshape(case["kv_heads"], -1, case["dim"]).mean(1) for q in queries])
    return m / m.norm(dim=-1, keepdim=True)


def _tokens(case, gen, z):
    """Per layer [H_kv][n * tokens][d] bfloat16 around the centroids z [n][L][H_kv][d]."""
    n, T, Hk, d = z.shape[0], case["tokens"], case["kv_heads"], case["dim"]
    out = []
    for l in range(case["layers"]):
        x = torch.randn((Hk, n, T, d), generator=gen, device="cuda")
        x.mul_(0.5).add_(z[:, l].transpose(0, 1).unsqueeze(2))
        out.append(x.to(torch.bfloat16).reshape(Hk, n * T, d))
    return out


def _stream_chunks(case, gen, frames, queries, step=CHUNK):
    """A stream's frames in order, ``step`` at a time: (frames, layer keys)."""
    dirs = _directions(case, queries) if queries is not None else None
    n_planted = max(1, frames // case.get("planted_every", 150)) if queries is not None else 0
    planted = {int((i + 0.5) * frames / n_planted) for i in range(n_planted)}
    for f0 in range(0, frames, step):
        n = min(step, frames - f0)
        z = torch.randn((n, case["layers"], case["kv_heads"], case["dim"]), generator=gen, device="cuda")
        for f in range(f0, f0 + n):
            if f in planted:
                z[f - f0] = z[f - f0].norm(dim=-1, keepdim=True) * dirs
        yield n, _tokens(case, gen, z)


def _session_chunks(case, gen):
    """Frames of scenes of ``scene`` frames each: neighbours share most of their centroid."""
    n_scene = -(-case["frames"] // case["scene"])
    dims = (case["layers"], case["kv_heads"], case["dim"])
    scenes = torch.randn((n_scene, *dims), generator=gen, device="cuda")
    for f0 in range(0, case["frames"], case["step"]):
        n = min(case["step"], case["frames"] - f0)
        at = torch.arange(f0, f0 + n, device="cuda") // case["scene"]
        z = scenes[at] + 0.3 * torch.randn((n, *dims), generator=gen, device="cuda")
        yield n, _tokens(case, gen, z)


def _new_index(case, frames, rows, recent=0):
    return ShallowIndex(case["layers"], case["q_heads"], case["kv_heads"], case["dim"], frames, frames * rows, n_recent=recent)


def prepare(case, seed):
    if case["kind"] == "retrieve":
        indices, queries = [], []
        for s, frames in enumerate(_lengths(case)):
            gen = _generator(seed, s)
            q = _queries(case, gen)
            x = _new_index(case, frames, _rows(case, s), case["recent"])
            for n, keys in _stream_chunks(case, gen, frames, q):
                x.append(keys, n, case["tokens"], _compress(case, s))
            indices.append(x)
            queries.append(q)
        return {"case": case, "queries": queries,
                "retriever": Retriever(indices, case["top_k"], case["select"], head_mode=case["head_mode"],
                                       score_mode=case["score_mode"])}
    gen = _generator(seed, 0)
    if case["kind"] == "append":
        return {"case": case, "chunks": list(_stream_chunks(case, gen, case["frames"], None, case["step"]))}
    return {"case": case, "queries": _queries(case, gen), "chunks": list(_session_chunks(case, gen))}


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------


def _carve(arena, parts):
    """Views of the 256-byte aligned parts of an arena, one after another."""
    out, at = [], 0
    for dtype, shape in parts:
        nbytes = math.prod(shape) * dtype.itemsize
        out.append(arena[at:at + nbytes].view(dtype).view(shape))
        at = (at + nbytes + 255) // 256 * 256
    return out


def _index_parts(x):
    """keys, member counts, descriptors, pooled keys and row offsets in an index's arena."""
    d = x.desc
    return _carve(x.arena, [(torch.bfloat16, (d.n_layers, d.n_kv_heads, d.max_rows, d.head_dim)),
                            (torch.int32, (d.n_layers, d.n_kv_heads, d.max_rows)),
                            (torch.float32, (d.max_frames, d.n_kv_heads * d.head_dim)),
                            (torch.float32, (d.max_frames, d.n_layers, d.n_kv_heads, d.head_dim)),
                            (torch.int32, (d.max_frames + 1,))])


def _absorbed(case):
    """(frames that left the detailed window, clusters they form, the set's capacity)."""
    gone = max(0, min(case["frames"] - case["keep"], case["frames"] - case["recent"]))
    return gone, -(-gone // case["scene"]), -(-case["frames"] // case["scene"]) + 1


def _cluster_parts(case, cl):
    """centroids, sizes, member spans and representatives of the clusters in use."""
    used, cap, dim = _absorbed(case)[1], _absorbed(case)[2], case["kv_heads"] * case["dim"]
    parts = _carve(cl.arena, [(torch.int32, (4,)), (torch.float32, (cap, dim)), (torch.int32, (cap,)),
                              (torch.int64, (cap, 2)),
                              (torch.float32, (cap, case["layers"], case["kv_heads"], _rows(case), case["dim"]))])
    return [p[:used] for p in parts[1:]]


def run(state):
    case = state["case"]
    if case["kind"] == "retrieve":
        return state["retriever"](state["queries"])
    if case["kind"] == "append":
        x = _new_index(case, case["frames"], _rows(case))
        for n, keys in state["chunks"]:
            x.append(keys, n, case["tokens"], _compress(case))
        return _index_parts(x)
    rows = _rows(case)
    x = _new_index(case, case["keep"] + case["step"], rows, case["recent"])
    cl = LongClusters(x, rows, _absorbed(case)[2], case["tau"])
    budget = case["keep"] * _frame_bytes(case)
    for n, keys in state["chunks"]:
        x.append(keys, n, case["tokens"], _compress(case))
        first, hi = x.window()[1], x.budget_split(budget)
        if hi > first:
            cl.absorb(hi, hi - first)
            x.compact()
    q = state["queries"]
    found = Retriever([x], case["top_k"], case["select"])([q])
    clusters = cl.retrieve(q, case["clusters"])
    pooled = PooledRanker([x], case["select"])([q])
    units = assemble_evidence([x], found[0], case["recent"], clusters=[cl], cluster_ids=clusters[0].view(1, -1))
    keys, counts, desc, means, off = _index_parts(x)
    held = x.n_rows
    kept = held // rows
    return [found, clusters, pooled, units, [keys[:, :, :held], counts[:, :, :held], desc[:kept], means[:kept], off[:kept + 1]],
            _cluster_parts(case, cl)]


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how far two correct ones differ
# ---------------------------------------------------------------------------


def _frame_bytes(case):
    """Arena bytes of one frame: keys and member counts, descriptor, pooled keys, row offset."""
    lg = case["layers"] * case["kv_heads"]
    return _rows(case) * lg * (2 * case["dim"] + 4) + (case["kv_heads"] + lg) * case["dim"] * 4 + 4


def _append_work(case, frames):
    """Raw keys read, the arena's entries written; per compressed frame the k-means' dot products and sums."""
    lg, T, d = case["layers"] * case["kv_heads"], case["tokens"], case["dim"]
    nbytes = frames * (lg * T * d * 2 + _frame_bytes(case))
    flops = frames * lg * T * d
    if case["centroids"]:
        flops += frames * lg * T * d * (2 * _rows(case) * (1 + case["iters"]) + case["iters"])
    return nbytes, flops


def work(case):
    lg, d = case["layers"] * case["kv_heads"], case["dim"]
    if case["kind"] == "append":
        nbytes, flops = _append_work(case, case["frames"])
        return {"bytes": nbytes, "flops": flops}
    query = case["layers"] * case["q_heads"] * case["nq"] * d * 2
    if case["kind"] == "retrieve":
        rows = sum(max(0, f - case["recent"]) * _rows(case, s) for s, f in enumerate(_lengths(case)))
        out = case["streams"] * (case["select"] * 16 + 4)
        return {"bytes": rows * lg * d * 2 + case["streams"] * query + out,
                "flops": 2 * rows * case["layers"] * case["q_heads"] * d}
    nbytes, flops = _append_work(case, case["frames"])
    gone, used, _ = _absorbed(case)
    rows = (case["frames"] - gone - case["recent"]) * _rows(case)
    # the absorbed rows read again and their clusters' representatives written, then one question over the window
    nbytes += gone * _rows(case) * lg * d * 2 + used * _rows(case) * lg * d * 4 + rows * lg * d * 2 + query
    return {"bytes": nbytes, "flops": flops + 3 * gone * _rows(case) * lg * d + 2 * rows * case["layers"] * case["q_heads"] * d}


def tolerance(case):
    # Raw keys are copied; mass, means, norms and scores are 32-bit sums (up to 4e-7 from 64 bits).
    # Compressed: a centroid is a bfloat16 value of a 32-bit sum, and a token midway between two
    # centroids (or two tokens equally far from the picks) may go either way, which moves whole
    # centroids (up to 3e-3 from 64 bits); what is retrieved over them moves far less.
    if case["centroids"]:
        return {"rel": 1e-3 if case["kind"] == "retrieve" else 1e-2, "max": 0.9, "differ": 0.01}
    return {"rel": 2e-6, "max": 2e-5, "differ": 0.0}


# ---------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------


def _kmeans64(X, C, iters):
    """X [P][T][d] double -> (centroids [P][C][d], counts): farthest-point seeding from the mean, then Lloyd rounds."""
    P, T, d = X.shape
    every = torch.arange(P, device=X.device)
    far = (X - X.mean(1, keepdim=True)).square().sum(-1)
    near = torch.full((P, T), math.inf, dtype=torch.float64, device=X.device)
    taken = torch.zeros((P, T), dtype=torch.bool, device=X.device)
    cen = []
    for c in range(C):
        pick = far.masked_fill(taken, -math.inf).argmax(1)
        taken[every, pick] = True
        p = X[every, pick]
        cen.append(p)
        near = torch.minimum(near, (X - p.unsqueeze(1)).square().sum(-1))
        far = near
    cen = torch.stack(cen, 1)
    x2 = X.square().sum(-1, keepdim=True)
    for _ in range(iters):
        dist = x2 + cen.square().sum(-1).unsqueeze(1) - 2 * torch.bmm(X, cen.transpose(1, 2).contiguous())
        one = torch.nn.functional.one_hot(dist.argmin(-1), C).to(torch.float64).transpose(1, 2).contiguous()
        n = one.sum(-1, keepdim=True)
        cen = torch.where(n > 0, torch.bmm(one, X) / n.clamp(min=1), cen)
    return cen


def _stored64(case, keys, n, comp):
    """The rows an index stores of a chunk, [L][H_kv][n * rows][d] double."""
    Hk, T, d = case["kv_heads"], case["tokens"], case["dim"]
    if comp is None:
        return torch.stack([k.double() for k in keys])
    C = min(comp[0], T)
    out = [_kmeans64(k.double().reshape(Hk * n, T, d), C, comp[1]).reshape(Hk, n * C, d) for k in keys]
    return torch.stack(out).to(torch.bfloat16).double()


def _means64(case, keys, n):
    """Mean raw key of each frame, [n][L][H_kv][d] double."""
    Hk, T, d = case["kv_heads"], case["tokens"], case["dim"]
    return torch.stack([k.double().reshape(Hk, n, T, d).mean(2).transpose(0, 1) for k in keys], 1)


def _descriptors64(means):
    v = means[:, -1].reshape(means.shape[0], -1)
    return v / v.norm(dim=-1, keepdim=True)


def _question64(case, queries):
    """Mean query, [L][H_kv][d][G] double."""
    G = case["q_heads"] // case["kv_heads"]
    return torch.stack([q.double().mean(1).reshape(case["kv_heads"], G, case["dim"]).transpose(1, 2).contiguous() for q in queries])


def _logits64(case, rows, question):
    """[L][H_q][n] scaled logits of rows [L][H_kv][n][d]."""
    out = [torch.bmm(rows[l], question[l]).transpose(1, 2).reshape(case["q_heads"], -1) for l in range(case["layers"])]
    return torch.stack(out) / math.sqrt(case["dim"])


def _evidence64(case, logits, desc, rows):
    """Attention mass of the selected frames in selection order (logits and descriptors of the candidates)."""
    mode = case.get("head_mode", 0)
    v = logits.softmax(-1) if case.get("score_mode", 0) else logits
    v = v.mean(1) if mode else v.reshape(-1, v.shape[-1])
    top, pos = v.topk(min(case["top_k"], v.shape[-1]), dim=-1)
    frame = (pos // rows).reshape(-1)
    votes = torch.bincount(frame, minlength=desc.shape[0]).cpu().numpy()
    mass = torch.zeros(desc.shape[0], dtype=torch.float64, device=v.device).index_add_(0, frame, top.reshape(-1)).cpu().numpy()
    voted = np.nonzero(votes)[0]
    pool = voted[np.lexsort((voted, -mass[voted], -votes[voted]))][:4 * case["select"]]
    D = desc[torch.from_numpy(pool).to(desc.device)]
    far = (1 - D @ D.T).cpu().numpy()
    picked, near = [0], far[0].copy()
    while len(picked) < min(case["select"], len(pool)):
        near[picked] = -np.inf
        picked.append(int(np.argmax(near)))
        near = np.minimum(near, far[picked[-1]])
    out = np.zeros(case["select"])
    out[:len(picked)] = mass[pool[picked]]
    return torch.from_numpy(out)


def exact(case, seed):
    if case["kind"] == "retrieve":
        masses = []
        for s, frames in enumerate(_lengths(case)):
            gen = _generator(seed, s)
            q = _queries(case, gen)
            question = _question64(case, q)
            logits, desc = [], []
            for n, keys in _stream_chunks(case, gen, frames, q):
                logits.append(_logits64(case, _stored64(case, keys, n, _compress(case, s)), question))
                desc.append(_descriptors64(_means64(case, keys, n)))
            use = max(0, frames - case["recent"])
            masses.append(_evidence64(case, torch.cat(logits, -1)[..., :use * _rows(case, s)], torch.cat(desc)[:use], _rows(case, s)))
        return (None, None, torch.stack(masses), None)
    gen = _generator(seed, 0)
    if case["kind"] == "append":
        rows, means = [], []
        for n, keys in _stream_chunks(case, gen, case["frames"], None, case["step"]):
            rows.append(_stored64(case, keys, n, _compress(case)))
            means.append(_means64(case, keys, n))
        means = torch.cat(means)
        return [torch.cat(rows, 2), None, _descriptors64(means), means, None]
    q = _queries(case, gen)
    question = _question64(case, q)
    rows, means = [], []
    for n, keys in _session_chunks(case, gen):
        rows.append(_stored64(case, keys, n, _compress(case)))
        means.append(_means64(case, keys, n))
    rows, means = torch.cat(rows, 2), torch.cat(means)
    desc, R = _descriptors64(means), _rows(case)
    gone, used, _ = _absorbed(case)
    by_frame = rows.reshape(case["layers"], case["kv_heads"], case["frames"], R, case["dim"]).permute(2, 0, 1, 3, 4)
    cen, rep, size = [], [], []
    for f in range(gone):
        if cen and float(desc[f] @ cen[-1]) >= case["tau"]:
            c = (size[-1] * cen[-1] + desc[f]) / (size[-1] + 1)
            cen[-1] = c / c.norm()
            rep[-1] = (size[-1] * rep[-1] + by_frame[f]) / (size[-1] + 1)
            size[-1] += 1
        else:
            cen.append(desc[f])
            rep.append(by_frame[f])
            size.append(1)
    if len(cen) != used:
        return None
    hi = case["frames"] - case["recent"]
    mass = _evidence64(case, _logits64(case, rows[:, :, gone * R:hi * R], question), desc[gone:hi], R)
    weight = question.sum(-1) / (case["q_heads"] * math.sqrt(case["dim"]))        # [L][H_kv][d]
    best = (torch.stack(cen) @ weight[-1].reshape(-1)).sort(descending=True).values[:case["clusters"]]
    scores = torch.zeros(case["clusters"], dtype=torch.float64, device=best.device)
    scores[:len(best)] = best
    frames = (means[gone:hi].reshape(hi - gone, -1) @ weight.reshape(-1)) / case["layers"]
    pooled = frames.sort(descending=True).values[:case["select"]]
    return [[None, None, mass.unsqueeze(0), None], [None, scores, None, None, None], [None, pooled.unsqueeze(0), None], None,
            [rows[:, :, gone * R:], None, desc[gone:], means[gone:], None], [torch.stack(cen), None, None, torch.stack(rep)]]
