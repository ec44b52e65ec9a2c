"""Calls of more rows or streams than one launch may have work-items for (2^32
- 1): 2^24 workgroups of 256 threads in the row summaries, 2^22 of 1024 in the
steps of beams above 8 hypotheses. The streams repeat with a period of seven,
so the expected outputs are those of a call of seven streams."""

import numpy as np
import pytest

from tests.gpu_cases import say

pytestmark = pytest.mark.gpu

MIDS = np.array([0, 1, -1, 0, 0, 1, 1], np.int32)


def _decoder(V):
    from paper_2608_21343_amd.decoder import BoostDecoder
    cm = np.arange(V + 1, dtype=np.int32)
    cm[V] = -1
    rng = np.random.default_rng(V)
    lists = [[rng.integers(0, V, size=3).astype(np.int32) for _ in range(4)] for _ in range(2)]
    return BoostDecoder(lists, cm)


def _run(dec, base, B, kind):
    import torch
    T, K = base.shape[0], base.shape[2]
    rows = torch.empty((T, B) + base.shape[2:], dtype=base.dtype, device="cuda")
    full = B // 7 * 7
    for t in range(T):
        rows[t, :full].view(-1, 7, *base.shape[2:]).copy_(base[t][None])
        rows[t, full:] = base[t, :B - full]
    mids = np.resize(MIDS, B)
    if kind == "greedy":
        m, st, _ = dec.start(mids)
        out = dec.greedy(rows[:, :, 0], m, st)
        carry = (st,)
    elif kind == "beam":
        m, st, sc = dec.start(mids, K)
        out = dec.beam(rows, m, st, sc)
        carry = (st.view(B, K), sc.view(B, K))
    else:
        c = dec.start_beam_stream(mids, K, 4)
        out = dec.beam_stream(rows, c)
        carry = (c.states.view(B, K), c.scores.view(B, K), c.hyps.view(B, K, -1), c.tree,
                 c.tree_len)
    torch.cuda.synchronize()
    return [o.transpose(0, 1) for o in out] + list(carry)


def _same(got, want, B):
    import torch
    full = B // 7 * 7
    for g, w in zip(got, want):
        assert g.shape[0] == B
        g, w = (x.contiguous() for x in (g, w))
        if g.dtype == torch.float32:  # bit for bit
            g, w = g.view(torch.int32), w.view(torch.int32)
        assert bool((g[:full].view(-1, 7, *w.shape[1:]) == w[None]).all())
        assert bool((g[full:] == w[:B - full]).all())


# (kind, streams, hypotheses, steps, V+1, type, GB of device memory)
CASES = [("beam", 2 ** 20 + 3, 2, 33, 3, "f32", 8), ("beam", 2 ** 22 + 3, 9, 1, 9, "bf16", 12),
         ("stream", 2 ** 22 + 3, 9, 1, 9, "bf16", 12),
         ("greedy", 2 ** 20 + 3, 1, 17, 2049, "bf16", 90)]


@pytest.mark.parametrize("kind,B,K,T,V1,dtype,gb", CASES)
def test_more_rows_than_one_launch_holds(kind, B, K, T, V1, dtype, gb):
    import torch
    if torch.cuda.mem_get_info()[0] < gb * 1e9:
        pytest.skip(f"needs {gb} GB of device memory")
    say(f"[launch limits] {kind} B={B} K={K} T={T} V+1={V1} {dtype}")
    dec = _decoder(V1 - 1)
    g = torch.Generator(device="cuda")
    g.manual_seed(V1)
    base = torch.randn((T, 7, K, V1), device="cuda", generator=g)
    base = base.to(torch.float32 if dtype == "f32" else torch.bfloat16)
    _same(_run(dec, base, B, kind), _run(dec, base, 7, kind), B)
    torch.cuda.empty_cache()
