"""The beam kernels where their instances and paths change, against the oracle:
rows on both sides of every row-preparation instance, beams on both sides of
every wave layout (4, 8 and 16 waves, two slots a wave), calls with and without
LDS records, rows of equal values (more candidates than the ranked list holds),
rows with fewer finite values than hypotheses (the rounds over every
candidate), and a row with a nan beside clean streams. Tokens, parents, states
and accumulated scores bit for bit; step scores within 1e-5 (float32 sums of
terms below 64: 64 * 2^-24 * 2 = 8e-6)."""

import numpy as np
import pytest

import oracle
import workloads as W
from tests.gpu_cases import compare_beam, gpu_beam, say

pytestmark = pytest.mark.gpu

ATOL = 1e-5
MASKS = {"-1e10": -1e10, "-1e30": -1e30, "lowest": np.finfo(np.float32).min}
EDGES = [2, 3, 256, 257, 512, 513, 768, 769, 1024, 1025, 1280, 1281, 1536, 1537, 1792, 1793, 2048,
         2049, 3072, 3073, 4096, 4097, 5120, 5121, 6144, 6145, 8192, 8193, 10240, 10241, 16384,
         16385]
BEAMS = [8, 1, 4, 5, 9, 16, 17, 32, 12, 3]


def _run(V1, K, kind, fill, dtype, chunk, T=6, atol=ATOL):
    from paper_2608_21343_amd.decoder import BoostDecoder, to_device_logits
    from workloads.synth import _f32_to_bf16_bits
    K = min(K, V1)
    V = V1 - 1
    say(f"[beam edge] V+1={V1} K={K} {kind} {fill} {dtype} chunk={chunk}")
    cfg = W.Config(8100 + V1 + K, "edge", B=3, K=K, V=V, T=T, chunk=chunk, dtype="f32",
                   n_phrases=40, len_lo=1, len_hi=5, token_dist="zipf", zipf_s=1.1, logit_std=1.5,
                   blank_offset=0.5, n_case=V // 6)
    lists, cm = W.phrases(cfg), W.class_map(cfg)
    mids = np.array([0, 1, -1], np.int32)
    rows = np.array(W.logits(cfg))
    rng = np.random.default_rng(V1 * 64 + K)
    for b in range(2):  # spell phrases, so that states have children
        t = 0
        while t < T:
            ph = lists[b][int(rng.integers(len(lists[b])))]
            for i, v in enumerate(ph[:T - t]):
                rows[t + i, b, :, int(v)] += np.float32(4.0)
            t += len(ph)
    if fill == "equal":
        rows[...] = np.float32(0.25)
    elif fill == "masked":
        keep = rng.random(rows.shape) < min(1.0, 1.5 / V1)
        keep[..., V] = rng.random(rows.shape[:-1]) < 0.5
        keep[..., 0] |= ~keep.any(-1)
        rows[~keep] = -np.inf
    elif fill.startswith("offset"):
        rows += np.float32(fill[6:])
    elif fill in MASKS:  # 100 tokens kept, all within one wave's share of a row
        keep = np.zeros(V1, bool)
        keep[V1 // 2 - V1 // 2 % 256:][:100] = True
        rows[..., ~keep] = np.float32(MASKS[fill])
    if dtype == "bf16":
        rows = _f32_to_bf16_bits(rows)
        if fill == "lowest":  # bfloat16's own (the float32 one rounds to -inf)
            rows[..., ~keep] = 0xff7f
    dec = BoostDecoder(lists, cm, token_w=cfg.token_w, end_bonus=cfg.end_bonus)
    graphs = {m: oracle.build_graph(lists[m], cm, token_w=cfg.token_w, end_bonus=cfg.end_bonus)
              for m in (0, 1)}
    dev = to_device_logits(rows)
    if kind == "plain":
        st0, S0 = oracle.init_carry(mids, K)
        compare_beam(gpu_beam(dec, dev, mids, chunk),
                     oracle.beam_decode(graphs, mids, rows, st0, S0), range(cfg.B), atol)
        return
    carry, want = dec.start_beam_stream(mids, K, 24), oracle.init_stream_carry(mids, K)
    for t0 in range(0, T, chunk):
        got = [o.cpu().numpy() for o in dec.beam_stream(dev[t0:t0 + chunk], carry)]
        exp = oracle.beam_decode_stream(graphs, mids, rows[t0:t0 + chunk], want, tree_cap=24)
        compare_beam(got, exp, range(cfg.B), atol)


@pytest.mark.parametrize("i", range(len(EDGES)))
def test_row_instance_edges(i):
    _run(EDGES[i], BEAMS[i % len(BEAMS)], ("plain", "stream")[i % 2], "normal",
         ("f32", "bf16")[i // 2 % 2], (17, 3)[i // 3 % 2], T=17)


@pytest.mark.parametrize("K", [1, 4, 5, 8, 9, 16, 17, 32])
@pytest.mark.parametrize("kind", ["plain", "stream"])
def test_wave_layouts(K, kind):
    _run(601, K, kind, "normal", "f32", 6, T=10)
    _run(601, K, kind, "normal", "bf16", 20, T=20)
    _run(2600, K, kind, "normal", "bf16", 10, T=10)
    _run(2600, K, kind, "normal", "f32", 20, T=20)


@pytest.mark.parametrize("K", [3, 8, 16, 32])
@pytest.mark.parametrize("fill", ["equal", "masked"])
@pytest.mark.parametrize("V1", [70, 1025, 2305])
def test_equal_and_masked_rows(V1, fill, K):
    for kind in ("plain", "stream"):
        _run(V1, K, kind, fill, "f32", 3)


@pytest.mark.parametrize("V1,phrases,members", [(61, 600, 3), (201, 900, 3), (201, 900, 5),
                                                (301, 3000, 3), (2101, 6000, 3)])
@pytest.mark.parametrize("K", [1, 2, 4, 7, 12, 32])
def test_children_for_most_classes(V1, phrases, members, K):
    """Many phrases over few tokens: most of a row's best root moves are
    overridden, by children held one per lane and by larger sets."""
    from paper_2608_21343_amd.decoder import BoostDecoder, to_device_logits
    say(f"[beam edge] dense lists V+1={V1} phrases={phrases} members={members} K={K}")
    V, T = V1 - 1, 18
    cfg = W.Config(8400 + V1 + K, "dense", B=3, K=K, V=V, T=T, chunk=T, dtype="f32",
                   n_phrases=phrases, len_lo=1, len_hi=6, token_dist="zipf", zipf_s=1.1,
                   logit_std=1.5, blank_offset=0.5, n_case=V // 9)
    lists, cm = W.phrases(cfg), W.class_map(cfg)
    if members == 5:
        n = V // 7
        cm = np.arange(V + 1, dtype=np.int32)
        for k in range(1, 5):
            cm[k * n:(k + 1) * n] = np.arange(n)
        cm[V] = -1
    rows = np.array(W.logits(cfg))
    mids = np.array([0, 1, -1], np.int32)
    dec = BoostDecoder(lists, cm, token_w=cfg.token_w, end_bonus=cfg.end_bonus)
    graphs = {m: oracle.build_graph(lists[m], cm, token_w=cfg.token_w, end_bonus=cfg.end_bonus)
              for m in (0, 1)}
    dev = to_device_logits(rows)
    st0, S0 = oracle.init_carry(mids, K)
    compare_beam(gpu_beam(dec, dev, mids, 9), oracle.beam_decode(graphs, mids, rows, st0, S0),
                 range(3), ATOL)
    carry, want = dec.start_beam_stream(mids, K, 64), oracle.init_stream_carry(mids, K)
    got = [o.cpu().numpy() for o in dec.beam_stream(dev, carry)]
    compare_beam(got, oracle.beam_decode_stream(graphs, mids, rows, want, tree_cap=64), range(3),
                 ATOL)


@pytest.mark.parametrize("offset", ["+630", "-630", "+650", "-650", "+720", "-720", "+2000", "-2000"])
@pytest.mark.parametrize("V1", [301, 2305])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rows_far_from_zero(V1, offset, dtype):
    """Rows whose sum of exponentials leaves what is summed without a maximum
    (about e^644 either way), and rows at its edge; accumulated scores bit for
    bit. Step scores are differences of values up to 2000: 2^-13 each."""
    for kind in ("plain", "stream"):
        _run(V1, 4, kind, "offset" + offset, dtype, 3, atol=2.0 ** -12)


@pytest.mark.parametrize("fill", MASKS)
@pytest.mark.parametrize("V1", [1025, 8193])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rows_masked_with_a_finite_value(V1, fill, dtype):
    _run(V1, 4, "plain", fill, dtype, 3)
    _run(V1, 12, "stream", fill, dtype, 3)


@pytest.mark.parametrize("V1", [300, 2305])
def test_nan_row_leaves_other_streams(V1):
    """A nan in one stream's row leaves the other streams' outputs as they are,
    and the stream's own outputs hold valid tokens, parents and states."""
    import torch
    from paper_2608_21343_amd.decoder import BoostDecoder, to_device_logits
    cfg = W.Config(8800 + V1, "nan", B=3, K=5, V=V1 - 1, T=5, chunk=5, dtype="f32", n_phrases=20,
                   len_lo=1, len_hi=4, token_dist="zipf", zipf_s=1.1, logit_std=1.0,
                   blank_offset=0.0, n_case=V1 // 6)
    lists = W.phrases(cfg)
    dec = BoostDecoder(lists, W.class_map(cfg))
    rows = np.array(W.logits(cfg))
    mids = np.arange(3, dtype=np.int32)
    clean = gpu_beam(dec, to_device_logits(rows), mids, 5)
    rows[2, 1, 3, 7] = np.nan
    got = gpu_beam(dec, to_device_logits(rows), mids, 5)
    torch.cuda.synchronize()
    for a, b in zip(clean, got):
        a, b = np.asarray(a).reshape(-1, 3, 5)[:5], np.asarray(b).reshape(-1, 3, 5)[:5]
        assert np.array_equal(a[:, [0, 2]], b[:, [0, 2]])
    tok, par = (np.asarray(got[i]).reshape(-1, 3, 5) for i in (0, 1))
    assert tok.min() >= 0 and tok.max() <= cfg.V and par.min() >= 0 and par.max() < 5


@pytest.mark.parametrize("V1", [300, 2305])
@pytest.mark.parametrize("K", [1, 3, 8, 12, 32])
def test_steps_without_a_candidate(V1, K):
    """A step whose rows are all nan or all -inf leaves no candidate: every slot
    takes the first token from slot 0 and its state, with score -inf, as the
    reference kernel does, and the steps after it go on from there."""
    from paper_2608_21343_amd import capi
    from paper_2608_21343_amd.decoder import BoostDecoder, to_device_logits
    say(f"[beam edge] no candidate V+1={V1} K={K}")
    cfg = W.Config(8900 + V1, "none", B=4, K=K, V=V1 - 1, T=9, chunk=9, dtype="f32", n_phrases=20,
                   len_lo=2, len_hi=4, token_dist="zipf", zipf_s=1.1, logit_std=1.0,
                   blank_offset=0.0, n_case=V1 // 6)
    lists = [list(p) for p in W.phrases(cfg)]
    first = int(lists[0][0][0])
    lists[0].append(np.array([first, 0, 3], np.int32))  # the first token continues a phrase
    rows = np.array(W.logits(cfg))
    mids = np.array([0, 1, -1, 3], np.int32)
    rows[2, :, :, first] += 9.0
    rows[3] = np.nan
    rows[4, 0] = rows[6, 1] = -np.inf
    rows[6, 3, 0, 5] = np.nan
    dec = BoostDecoder(lists, W.class_map(cfg))
    dev = to_device_logits(rows)

    def run(kernel):
        with capi.kernels(beam=kernel):
            carry = dec.start_beam_stream(mids, K, 64)
            out = [np.asarray(o.cpu()) for o in dec.beam_stream(dev, carry)]
            return list(gpu_beam(dec, dev, mids, 9)), out + [
                np.asarray(o.cpu()) for o in (carry.states, carry.scores, carry.hyps, carry.tree,
                                              carry.tree_len)]

    for got, want in zip(run(capi.BEAM_AUTO), run(capi.BEAM_REF)):
        assert (want[0][3] == 0).all() and (want[4][3] == -np.inf).all()
        assert np.isnan(want[3][3]).all()
        for i, (a, b) in enumerate(zip(got, want)):
            assert np.array_equal(a, b, equal_nan=a.dtype == np.float32) if i != 3 else \
                np.allclose(a, b, rtol=0, atol=ATOL, equal_nan=True), i
