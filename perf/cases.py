"""The work a program has this library do, as timed cases: boosted greedy and
beam decoding of batches of streams through the public entry points, over the
real range of sizes, types and call patterns.

A case is a plain dict:

* ``search``: "greedy", "beam" (no recombination) or "stream" (beam with
  recombination and the flattened hypothesis tree);
* ``graph``: "class" (phrases as token ids over case classes) or "pieces"
  (phrases as characters over a piece vocabulary, variative graph);
* ``B`` streams, ``K`` hypotheses each, ``V`` tokens and the blank, ``T`` steps
  in calls of ``chunk`` steps, logits of type ``dtype`` whose rows are padded
  by ``pad`` values;
* ``lists`` phrase lists shared evenly by the streams (lists == B: one each),
  every list ``phrases`` long with 1..``longest`` tokens (or words) per
  phrase, tokens drawn by a Zipf law of exponent ``zipf`` (0: uniform);
* ``std`` and ``blank``: the logits' standard deviation and the blank's offset;
  ``plant``: listed phrases are spelled in the logits, one per 16 steps;
* ``plain``: every plain-th stream carries no list (0: none).

One pass starts the streams (tb_init_states or tb_init_beam_stream) and decodes
all T steps, the states carried from call to call on the device.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2608_21343_amd import capi
from paper_2608_21343_amd.decoder import BoostDecoder

TOKEN_W, END_BONUS, PLANT = 1.0, 2.0, 4.0
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}

_BASE = dict(search="greedy", graph="class", B=1, K=1, V=256, T=16, chunk=16, dtype="f32", pad=0,
             lists=1, phrases=10, longest=4, zipf=1.1, std=1.0, blank=1.5, plant=False, plain=0)


def listed():
    return [
        # one short utterance with a handful of phrases: latency of a single call
        dict(_BASE, name="one_utterance", V=256, T=50, chunk=50, zipf=0.0, blank=0.0),
        # frame-synchronous decoding, where each step's logits depend on the last
        # step's token, so that every step is a call of its own
        dict(_BASE, name="greedy_steps", B=128, V=1024, T=32, chunk=1, lists=128, phrases=1000,
             longest=10),
        # 128 live streams, each with its own list, fed in chunks
        dict(_BASE, name="greedy_chunks", B=128, V=1024, T=256, chunk=16, lists=128, phrases=1000,
             longest=10),
        # the same service over a piece vocabulary with variative graphs
        dict(_BASE, name="pieces_chunks", graph="pieces", B=64, V=1024, T=128, chunk=16, lists=64,
             phrases=400, longest=3, plant=True),
        # an offline batch of whole utterances with short lists
        dict(_BASE, name="greedy_batch", B=32, V=1024, T=500, chunk=500, lists=32, phrases=100,
             longest=6, zipf=1.2, blank=2.0),
        # a full batch of long recordings
        dict(_BASE, name="greedy_long", B=128, V=1024, T=1024, chunk=1024, lists=128, phrases=1000,
             longest=10),
        # odd sizes: a vocabulary, batch and call length that no tile divides,
        # padded rows, and streams without a list between the others
        dict(_BASE, name="greedy_odd", B=37, V=611, T=203, chunk=29, dtype="bf16", pad=5, lists=9,
             phrases=300, longest=8, blank=1.0, plant=True, plain=6),
        # a large vocabulary with long lists, shared by the streams of one customer
        dict(_BASE, name="greedy_wide", B=256, V=8192, T=256, chunk=256, dtype="bf16", lists=64,
             phrases=10000, longest=12, zipf=1.0, blank=0.0, plant=True),
        # beam search over a batch of utterances
        dict(_BASE, name="beam_batch", search="beam", B=64, K=8, V=1024, T=256, chunk=256,
             lists=64, phrases=1000, longest=10, std=1.5, blank=0.0),
        # live streams decoded with the streaming beam
        dict(_BASE, name="stream_chunks", search="stream", B=48, K=5, V=1000, T=96, chunk=16,
             dtype="bf16", lists=48, phrases=500, longest=8, std=1.5, blank=0.5, plant=True),
        # beam search over a large vocabulary
        dict(_BASE, name="beam_wide", search="beam", B=256, K=4, V=8192, T=64, chunk=64,
             dtype="bf16", lists=64, phrases=10000, longest=12, zipf=1.0, blank=0.0, plant=True),
        # the widest beam, 32 hypotheses a stream
        dict(_BASE, name="beam_32", search="beam", B=16, K=32, V=1024, T=32, chunk=32, lists=16,
             phrases=1000, longest=10, std=1.5, blank=0.0),
    ]


#: The logits of the largest listed case, in values.
MOST_VALUES = 256 * 256 * 8193


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    c = dict(_BASE)
    c["search"] = rng.choice(["greedy", "greedy", "beam", "stream"])
    c["dtype"] = rng.choice(["f32", "bf16"])
    c["V"] = _log_int(rng, 200, 8192)
    c["B"] = _log_int(rng, 1, 256)
    c["K"] = 1 if c["search"] == "greedy" else rng.choice([2, 3, 4, 4, 5, 6, 8, 8, 12, 32])
    c["T"] = _log_int(rng, 16, 500)
    c["pad"] = rng.choice([0, 0, 0, 3, 7, 64])
    if c["search"] == "greedy" and rng.random() < 0.2:
        c.update(graph="pieces", V=_log_int(rng, 300, 2000), B=_log_int(rng, 1, 64),
                 phrases=_log_int(rng, 10, 400), longest=rng.randint(1, 3))
    else:
        c.update(phrases=_log_int(rng, 10, 3000), longest=rng.randint(3, 12))
    # the largest work: fewer steps of the slower searches
    room = MOST_VALUES // (1 if c["K"] == 1 else 8 if c["K"] <= 8 else 256)
    c["T"] = max(16, min(c["T"], room // (c["B"] * c["K"] * (c["V"] + 1))))
    if c["B"] * c["K"] * c["T"] * (c["V"] + 1) > room:
        c["B"] = max(1, room // (c["K"] * c["T"] * (c["V"] + 1)))
    c["chunk"] = rng.choice([c["T"], c["T"], 1, 8, 16, rng.randint(2, 64)])
    c["T"] = min(c["T"], 64 * c["chunk"])
    c["chunk"] = min(c["chunk"], c["T"])
    c["lists"] = rng.choice([c["B"], max(1, c["B"] // 4)])
    c["zipf"] = rng.choice([0.0, 1.0, 1.1, 1.2])
    c["std"] = rng.choice([1.0, 1.5])
    c["blank"] = rng.choice([0.0, 1.0, 2.0])
    c["plant"] = rng.random() < 0.5
    c["plain"] = rng.choice([0, 0, 5])
    return c


# ---------------------------------------------------------------------------
# inputs


def _class_map(V):
    """Token -> case class: the first 3 * (V // 9) ids are lower, upper and
    title case blocks, the others are classes of their own; the blank is -1."""
    n = V // 9
    cm = np.arange(V + 1, dtype=np.int32)
    cm[n:2 * n] -= n
    cm[2 * n:3 * n] -= 2 * n
    cm[V] = -1
    return cm


def _zipf(rng, n, V, s):
    if s == 0.0:
        return rng.integers(0, V, size=n)
    cdf = np.cumsum(np.arange(1, V + 1, dtype=np.float64) ** -s)
    return np.minimum(np.searchsorted(cdf, rng.random(n) * cdf[-1]), V - 1)


def _token_lists(c, seed):
    """CSR of the phrase lists: model -> phrases -> tokens."""
    rng = np.random.default_rng([seed, 1])
    n = c["lists"] * c["phrases"]
    lens = rng.integers(1, c["longest"] + 1, size=n)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    toks = _zipf(rng, int(ptr[-1]), c["V"], c["zipf"]).astype(np.int32)
    return np.arange(c["lists"] + 1, dtype=np.int64) * c["phrases"], ptr, toks


def _model_ids(c):
    ids = (np.arange(c["B"]) % c["lists"]).astype(np.int32)
    if c["plain"]:
        ids[c["plain"] - 1::c["plain"]] = -1
    return ids


# Characters of the piece vocabulary: 0..25 lowercase, 26 the word start,
# 27..52 uppercase. Every character is a piece.
_LOWER = np.array(list(range(27)) + list(range(26)), np.int32)


def _upper(p, first_only):
    at = next(i for i, ch in enumerate(p) if ch < 26)
    return tuple(ch + 27 if ch < 26 and (not first_only or i == at) else ch
                 for i, ch in enumerate(p))


def _pieces(c, seed):
    """(pieces, phrase lists): substrings of a random lexicon, some of them
    cased, and lists of one to ``longest`` lexicon words in random casing."""
    rng = np.random.default_rng([seed, 2])
    freq = rng.permutation(1.0 / np.arange(1, 27))
    lens = rng.integers(3, 10, size=1500)
    chars = rng.choice(26, size=int(lens.sum()), p=freq / freq.sum()).tolist()
    ends = np.cumsum(lens).tolist()
    words = [tuple(chars[e - n:e]) for e, n in zip(ends, lens.tolist())]
    count = {}
    for w in words:
        w = (26,) + w
        for i in range(len(w)):
            for k in range(2, min(6, len(w) - i) + 1):
                count[w[i:i + k]] = count.get(w[i:i + k], 0) + 1
    pieces = [(ch,) for ch in range(53)]
    for p in sorted(count, key=lambda s: (-count[s], s)):
        if len(pieces) >= c["V"]:
            break
        pieces.append(p)
        for first_only, share in ((True, 0.3), (False, 0.1)):
            q = _upper(p, first_only)
            if rng.random() < share and q != pieces[-1] and len(pieces) < c["V"]:
                pieces.append(q)
    cdf = np.cumsum(1.0 / np.arange(1, len(words) + 1))
    out = []
    for _ in range(c["lists"]):
        lst = []
        for n in rng.integers(1, c["longest"] + 1, size=c["phrases"]).tolist():
            ph = ()
            for i in np.searchsorted(cdf, rng.random(n) * cdf[-1]).tolist():
                w, u = (26,) + words[min(i, len(words) - 1)], rng.random()
                ph += w if u < 0.7 else _upper(w, u < 0.9)
            lst.append(ph)
        out.append(lst)
    return pieces, out


def _spell(phrase, ids, rng):
    """Token ids of the phrase: the longest piece at every position, in a random casing."""
    low, out, i = tuple(int(_LOWER[ch]) for ch in phrase), [], 0
    while i < len(low):
        m = next(m for m in range(min(6, len(low) - i), 0, -1) if low[i:i + m] in ids)
        same = ids[low[i:i + m]]
        out.append(same[int(rng.integers(len(same)))])
        i += m
    return out


def _planted(c, seed, mids, phrase_of):
    """(step, stream, token) of the phrases spelled in the logits."""
    rng = np.random.default_rng([seed, 3])
    where = []
    for s0 in range(0, c["T"] - 15, 16):
        for b in np.flatnonzero(mids >= 0).tolist():
            sp = phrase_of(int(mids[b]), rng)
            if len(sp) <= 16:
                at = s0 + int(rng.integers(0, 17 - len(sp)))
                where += [(at + i, b, v) for i, v in enumerate(sp)]
    return np.asarray(where, np.int64).reshape(-1, 3)


def _logits(c, seed, where):
    g = torch.Generator(device="cuda").manual_seed(seed * 2 + 1)
    V1, dt = c["V"] + 1, DTYPES[c["dtype"]]
    buf = torch.empty((c["T"], c["B"], c["K"], V1 + c["pad"]), dtype=dt, device="cuda")
    step = max(1, (1 << 27) // max(1, buf[0].numel()))
    for t in range(0, c["T"], step):
        x = torch.randn(buf[t:t + step].shape, generator=g, device="cuda")
        x *= c["std"]
        x[..., c["V"]] += c["blank"]
        at = where[(where[:, 0] >= t) & (where[:, 0] < t + step)]
        if len(at):
            i = torch.from_numpy(at).cuda()
            k = torch.arange(c["K"], device="cuda")
            x.index_put_((i[:, 0:1] - t, i[:, 1:2], k[None, :], i[:, 2:3]),
                         torch.tensor(PLANT, device="cuda"), accumulate=True)
        buf[t:t + step] = x
    return buf[..., :V1]


def _inputs(c, seed):
    """(host lists, pieces or None, model ids, logits [T, B, K, V+1])."""
    mids, where = _model_ids(c), np.zeros((0, 3), np.int64)
    if c["graph"] == "pieces":
        pieces, lists = _pieces(c, seed)
        c = dict(c, V=len(pieces))
        if c["plant"]:
            ids = {}
            for v, p in enumerate(pieces):
                ids.setdefault(tuple(int(_LOWER[ch]) for ch in p), []).append(v)
            where = _planted(c, seed, mids, lambda m, r: _spell(
                lists[m][int(r.integers(len(lists[m])))], ids, r))
        return lists, pieces, mids, _logits(c, seed, where)
    lists = mp, pp, tk = _token_lists(c, seed)
    if c["plant"]:
        n, targets = c["V"] // 9, max(1, c["phrases"] // 10)

        def phrase_of(m, r):
            p = int(mp[m]) + int(r.integers(targets))
            return [int(v) % n + n * int(r.integers(3)) if v < 3 * n else int(v)
                    for v in tk[pp[p]:pp[p + 1]]]

        where = _planted(c, seed, mids, phrase_of)
    return lists, None, mids, _logits(c, seed, where)


def prepare(case, seed):
    lists, pieces, mids, logits = _inputs(case, seed)
    if pieces is not None:
        dec = BoostDecoder.variative(lists, pieces, _LOWER, tau=1.0, token_w=TOKEN_W,
                                     end_bonus=END_BONUS)
    else:
        graphs = capi.tb_compile_graphs(*lists, TOKEN_W, END_BONUS, _class_map(case["V"]))
        dec = BoostDecoder.for_arena(capi.tb_graphs_upload(graphs))
    T, B, K = logits.shape[:3]
    i32 = dict(dtype=torch.int32, device="cuda")
    f32 = dict(dtype=torch.float32, device="cuda")
    s = dict(dec=dec, chunk=case["chunk"], B=B, K=K, search=case["search"])
    if case["search"] == "greedy":
        s["logits"] = logits[:, :, 0]
        s["mids"], s["states"], _ = dec.start(mids)
        s["out"] = [torch.empty((T, B), **i32), torch.empty((T, B), **i32),
                    torch.empty((T, B), **f32)]
    else:
        s["logits"] = logits
        s["out"] = [torch.empty((T, B, K), **i32) for _ in range(3)]
        s["out"] += [torch.empty((T, B, K), **f32) for _ in range(2)]
        if case["search"] == "beam":
            s["mids"], s["states"], s["scores"] = dec.start(mids, K)
        else:
            s["carry"] = dec.start_beam_stream(mids, K, tree_cap=T * K)
    s["calls"] = [(s["logits"][t:t + case["chunk"]], tuple(o[t:t + case["chunk"]] for o in s["out"]))
                  for t in range(0, T, case["chunk"])]
    return s


def run(s):
    dec, arena = s["dec"], s["dec"].arena
    if s["search"] == "greedy":
        capi.tb_init_states(arena, s["B"], 1, s["mids"], s["states"])
        for rows, out in s["calls"]:
            dec.greedy(rows, s["mids"], s["states"], out)
        return s["out"] + [s["states"]]
    if s["search"] == "beam":
        capi.tb_init_states(arena, s["B"], s["K"], s["mids"], s["states"], s["scores"])
        for rows, out in s["calls"]:
            dec.beam(rows, s["mids"], s["states"], s["scores"], out)
        return s["out"] + [s["states"], s["scores"]]
    y = s["carry"]
    capi.tb_init_beam_stream(arena, s["B"], s["K"], y.mids, y.states, y.scores, y.hyps, y.tree_len)
    for rows, out in s["calls"]:
        dec.beam_stream(rows, y, out=out)
    return s["out"] + [y.states, y.scores, y.hyps, y.tree, y.tree_len]


def work(case):
    """Each logit read once, each output and carry written once; one add and
    one exponential a logit. The graphs' records are not counted."""
    rows = case["T"] * case["B"] * case["K"]
    item = 4 if case["dtype"] == "f32" else 2
    per_row = {"greedy": 12, "beam": 20, "stream": 28}[case["search"]]
    carry = {"greedy": 4, "beam": 8, "stream": 32}[case["search"]] * case["B"] * case["K"]
    return {"bytes": rows * ((case["V"] + 1) * item + per_row) + carry + 4 * case["B"],
            "flops": rows * 4.0 * (case["V"] + 1)}


def tolerance(case):
    """Keys and candidates are 32-bit sums in a fixed order, so that tokens,
    parents and states are the same whole numbers; the normaliser is a 32-bit
    sum in greedy search and a 64-bit one, rounded once, in the beams."""
    return {"rel": 1.5e-6, "max": 1e-5}


# ---------------------------------------------------------------------------
# the same pass in plain torch


class _Trie:
    """All lists' phrase tries with suffix links, built level by level. Nodes
    are numbered by level, within one by list, parent and class; the child of
    x on class c is the node of key x * V + c in the ascending ``keys``."""

    def __init__(self, mp, pp, tk, cm, V):
        dev = "cuda"
        self.V, self.n = V, len(mp) - 1
        lens = torch.from_numpy(np.diff(pp)).to(dev)
        start = torch.from_numpy(pp[:-1].copy()).to(dev)
        cls = torch.from_numpy(cm[tk].astype(np.int64)).to(dev)
        cur = torch.repeat_interleave(torch.arange(self.n, device=dev),
                                      torch.from_numpy(np.diff(mp)).to(dev))
        model, parent = [torch.arange(self.n, device=dev)], []
        local = [torch.zeros(self.n, dtype=torch.int64, device=dev)]
        used = torch.ones(self.n, dtype=torch.int64, device=dev)
        keys, end_nodes, levels, base = [], [], [], self.n
        for d in range(int(lens.max()) if len(lens) else 0):
            on = lens > d
            key, inv = torch.unique(cur[on] * V + cls[start[on] + d], return_inverse=True)
            m = torch.cat(model)[key // V]
            first = torch.searchsorted(m, torch.arange(self.n, device=dev))
            i = torch.arange(len(key), device=dev)
            local.append(used[m] + i - first[m])
            used = used + torch.bincount(m, minlength=self.n)
            model.append(m)
            parent.append(key // V)
            keys.append(key)
            cur = cur.clone()
            cur[on] = base + inv
            end_nodes.append(cur[lens == d + 1])
            levels.append((base, base + len(key)))
            base += len(key)
        self.model, self.local = torch.cat(model), torch.cat(local)
        self.keys = torch.cat(keys) if keys else torch.zeros(0, dtype=torch.int64, device=dev)
        end = torch.zeros(base, dtype=torch.bool, device=dev)
        for e in end_nodes:
            end[e] = True
        self.link = self.model.clone()
        kept = torch.zeros(base, dtype=torch.float64, device=dev)   # longest listed prefix
        after = torch.zeros(base, dtype=torch.bool, device=dev)     # a proper suffix is listed
        self.phi = torch.zeros(base, dtype=torch.float64, device=dev)
        self.psi = torch.zeros(base, dtype=torch.float64, device=dev)
        for d, (a, b) in enumerate(levels):
            x = torch.arange(a, b, device=dev)
            up, c = parent[d], keys[d] % V
            if d > 0:
                f, todo = self.link[up], torch.ones(len(x), dtype=torch.bool, device=dev)
                got = self.model[x].clone()
                while bool(todo.any()):
                    y = self.child(f, c)
                    got = torch.where(todo & (y >= 0), y, got)
                    todo = todo & (y < 0) & (f >= self.n)
                    f = self.link[f]
                self.link[a:b] = got
            kept[a:b] = torch.where(end[a:b], float(d + 1), kept[up])
            lk = self.link[a:b]
            after[a:b] = end[lk] | after[lk]
            self.phi[a:b] = TOKEN_W * (d + 1 - kept[a:b])
            bonus = torch.where(end[a:b], TOKEN_W * (d + 1 - kept[up]) + END_BONUS,
                                torch.where(after[a:b], END_BONUS, 0.0))
            self.psi[a:b] = self.phi[a:b] + bonus
        roots = torch.arange(self.n, device=dev)[:, None]
        self.cls = torch.from_numpy(cm[:V].astype(np.int64)).to(dev)
        y = self.child(roots, self.cls[None, :])
        self.root_move = torch.where(y >= 0, y, roots)

    def child(self, x, c):
        """The child of x on class c, or -1."""
        k = x * self.V + c
        if not len(self.keys):
            return torch.full_like(k, -1)
        i = torch.searchsorted(self.keys, k).clamp_(max=len(self.keys) - 1)
        return torch.where(self.keys[i] == k, i + self.n, -1)

    def moves(self, s):
        """[N, V] node reached from node s[i] by every token; -1 for s[i] = -1."""
        live = s >= 0
        out = torch.where(live[:, None], self.root_move[self.model[s.clamp(min=0)]], -1)
        left = torch.nonzero(live & (s >= self.n)).flatten()
        cur, done = s[left], torch.zeros((len(left), self.V), dtype=torch.bool, device=s.device)
        while len(left):
            y = self.child(cur[:, None], self.cls[None, :])
            hit = (y >= 0) & ~done
            out[left] = torch.where(hit, y, out[left])
            done |= hit
            cur = self.link[cur]
            on = cur >= self.n
            left, cur, done = left[on], cur[on], done[on]
        return out


def exact(case, seed):
    """What run returns. Selections follow the documented arithmetic (keys and
    candidates are 32-bit sums, the beam's normaliser is rounded to 32 bits
    first); the scores along the selected path are in 64 bits."""
    rows = case["T"] * case["B"] * case["K"]
    if case["graph"] == "pieces" or rows * (case["V"] + 1) > MOST_VALUES or case["T"] > 1024:
        return None
    lists, _, mids, logits = _inputs(case, seed)
    V, V1, T, B, K = case["V"], case["V"] + 1, case["T"], case["B"], case["K"]
    tr = _Trie(*lists, _class_map(V), V)
    node = torch.from_numpy(np.repeat(mids, K).astype(np.int64)).cuda()  # a list's root is its id
    phi32, psi32 = tr.phi.float(), tr.psi.float()
    i = torch.arange(V1, device="cuda")

    def at(table, x):
        return torch.where(x >= 0, table[x.clamp(min=0)], torch.zeros((), dtype=table.dtype, device="cuda"))

    def local(x):
        return torch.where(x >= 0, tr.local[x.clamp(min=0)], -1).to(torch.int32)

    if case["search"] == "greedy":
        out = [[], [], []]
        for t in range(T):
            z = logits[t, :, 0].float()
            dst = torch.cat([tr.moves(node), node[:, None]], 1)
            gain = at(psi32, dst)
            gain[:, V] = at(phi32, node)
            key = z + gain
            v = torch.where(key == key.amax(1, keepdim=True), i, V1).amin(1, keepdim=True)
            to = dst.gather(1, v)[:, 0]
            boost = torch.where(v[:, 0] == V, 0.0, at(tr.psi, to) - at(tr.phi, node))
            zz = z.double()
            out[2].append(zz.gather(1, v)[:, 0] - torch.logsumexp(zz, 1) + boost)
            node = to
            out[0].append(v[:, 0].to(torch.int32))
            out[1].append(local(node))
        return [torch.stack(o) for o in out] + [local(node)]

    S = torch.full((B, K), -math.inf, device="cuda")
    S[:, 0] = 0.0
    SS = S.double()
    node = node.view(B, K)
    mul = torch.tensor(0x9E3779B97F4A7C15 - (1 << 64), dtype=torch.int64, device="cuda")
    h = torch.zeros((B, K), dtype=torch.int64, device="cuda")
    before, last = h.clone(), torch.full_like(h, -1)
    b_at = torch.arange(B, device="cuda")[:, None]
    out = [[] for _ in range(5)]
    for t in range(T):
        z = logits[t].float()
        zz = z.double()
        dst = torch.cat([tr.moves(node.reshape(-1)).view(B, K, V), node[..., None]], 2)
        gain, gg = at(psi32, dst), at(tr.psi, dst)
        gain[..., V], gg[..., V] = at(phi32, node), at(tr.phi, node)
        lse = torch.logsumexp(zz, 2)
        c = (S - lse.float()) - at(phi32, node)
        cand = c[..., None] + (z + gain)
        step = zz - lse[..., None] + gg - at(tr.phi, node)[..., None]
        full = SS[..., None] + step
        if case["search"] == "stream":
            live = S > -math.inf
            pair = ((before[:, :, None] == h[:, None, :]) & (last >= 0)[:, :, None]
                    & live[:, :, None] & live[:, None, :])
            bi, x, y = torch.nonzero(pair, as_tuple=True)
            v = last[bi, x]
            p, q = cand[bi, x, V], cand[bi, y, v]
            one = torch.logaddexp(p.double(), q.double()).float()
            both = torch.logaddexp(full[bi, x, V], full[bi, y, v])
            keep = (p > q) | ((p == q) & (x * V1 + V < y * V1 + v))
            cand[bi, x, V] = torch.where(keep, one, -math.inf)
            cand[bi, y, v] = torch.where(keep, -math.inf, one)
            full[bi, x, V], full[bi, y, v] = both, both
        top, flat = torch.sort(cand.view(B, K * V1), dim=1, descending=True, stable=True)
        S, flat = top[:, :K].contiguous(), flat[:, :K]
        par, v = flat // V1, flat % V1
        SS = full.view(B, -1).gather(1, flat)
        node = dst.view(B, -1).gather(1, flat)
        out[0].append(v.to(torch.int32))
        out[1].append(par.to(torch.int32))
        out[2].append(local(node))
        out[3].append(step.view(B, -1).gather(1, flat))
        out[4].append(SS)
        if case["search"] == "stream":
            hp, bp, lp = h[b_at, par], before[b_at, par], last[b_at, par]
            emit = v < V
            before = torch.where(emit, hp, bp)
            h = torch.where(emit, hp * mul + v + 1, hp)
            last = torch.where(emit, v, lp)
    got = [torch.stack(o) for o in out] + [local(node).view(-1), SS.reshape(-1)]
    return got + [None, None, None] if case["search"] == "stream" else got
