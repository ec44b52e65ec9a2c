"""One-step calls whose outputs share memory: the carried states (and beam
scores) advanced in place, and one buffer for two outputs that nobody reads. The
other outputs equal those of calls with buffers of their own."""

import numpy as np
import pytest

import workloads as W
from paper_2608_21343_amd import capi
from tests.gpu_cases import say

pytestmark = pytest.mark.gpu

T = 6


def _case(V1, K):
    from paper_2608_21343_amd.decoder import BoostDecoder, to_device_logits
    cfg = W.Config(9300 + V1 + K, "shared", B=5, K=K, V=V1 - 1, T=T, chunk=1, dtype="f32",
                   n_phrases=80, len_lo=1, len_hi=5, token_dist="zipf", zipf_s=1.1, logit_std=1.0,
                   blank_offset=0.0, n_case=V1 // 6)
    lists = W.phrases(cfg)
    rows = np.array(W.logits(cfg))
    for b in range(5):
        for t, v in enumerate(np.concatenate(lists[b][:6])[:T]):
            rows[t, b, :, int(v)] += np.float32(4.0)
    return BoostDecoder(lists, W.class_map(cfg)), to_device_logits(rows), [0, 1, -1, 3, 4]


@pytest.mark.parametrize("V1", [300, 2305, 12000])
def test_greedy(V1):
    import torch
    say(f"[shared outputs] greedy V+1={V1}")
    dec, rows, mids = _case(V1, 1)
    rows = rows[:, :, 0]
    m, want_st, _ = dec.start(mids)
    want = [dec.greedy(rows[t:t + 1], m, want_st) for t in range(T)]
    m, st, _ = dec.start(mids)
    for t in range(T):
        tok, sc = torch.empty_like(want[t][0]), torch.empty_like(want[t][2])
        capi.tb_boost_step_greedy(dec.arena, rows[t:t + 1], m, st, tok, st, sc)
        assert torch.equal(tok, want[t][0]) and torch.equal(st, want[t][1][0])
        # the reference kernel sums a row's exponentials in another order
        assert torch.allclose(sc, want[t][2], rtol=0, atol=1e-5)
    m, st, _ = dec.start(mids)
    for t in range(T):
        tok, both = torch.empty_like(want[t][0]), torch.empty_like(want[t][0])
        capi.tb_boost_step_greedy(dec.arena, rows[t:t + 1], m, st, tok, both, both.view(torch.float32))
        assert torch.equal(tok, want[t][0]) and torch.equal(st, want[t][1][0])


@pytest.mark.parametrize("V1", [300, 2305])
@pytest.mark.parametrize("K", [3, 8, 12])
@pytest.mark.parametrize("stream", [False, True])
def test_beam(V1, K, stream):
    import torch
    say(f"[shared outputs] beam V+1={V1} K={K} stream={stream}")
    dec, rows, mids = _case(V1, K)

    def start():
        if stream:
            c = dec.start_beam_stream(mids, K, 64)
            return c, c.states, c.scores
        m, st, sc = dec.start(mids, K)
        return m, st, sc

    def step(t, c, st, sc, out):
        x = rows[t:t + 1]
        if stream:
            dec.beam_stream(x, c, out=out)
        else:
            dec.beam(x, c, st, sc, out=out)

    def buffers():
        i32 = dict(dtype=torch.int32, device="cuda")
        return [torch.empty((1, 5, K), **i32) for _ in range(3)] + \
            [torch.empty((1, 5, K), device="cuda") for _ in range(2)]

    c, st, sc = start()
    want = []
    for t in range(T):
        want.append(buffers())
        step(t, c, st, sc, want[-1])
    end = (c.hyps, c.tree, c.tree_len) if stream else ()
    c, st, sc = start()
    for t in range(T):
        out = buffers()
        step(t, c, st, sc, (out[0], out[1], st, out[3], sc))
        for i, o in enumerate((out[0], out[1], st, out[3], sc)):
            assert torch.equal(o.view(-1), want[t][i].view(-1)) or \
                (i == 3 and torch.allclose(o, want[t][i], rtol=0, atol=1e-5)), i
    if stream:
        assert all(torch.equal(a, b) for a, b in zip((c.hyps, c.tree, c.tree_len), end))
    c, st, sc = start()
    for t in range(T):
        out = buffers()
        step(t, c, st, sc, (out[0], out[1], out[1], out[3], out[3]))
        assert torch.equal(out[0], want[t][0]) and torch.equal(st, want[t][2].view(-1))
        assert torch.equal(sc, want[t][4].view(-1))
