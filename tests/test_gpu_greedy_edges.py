"""The wide-row greedy kernels where their instances and paths change, against
the oracle: rows on both sides of every summary instance, calls with and
without LDS records and longer than one piece of LDS row records, rows of
equal values, rows with few finite values or none, and a row with a nan beside
clean streams. Tokens and states bit for bit, scores within 1e-5 (float32 sums
of terms below 64: 64 * 2^-24 * 2 = 8e-6)."""

import numpy as np
import pytest

import oracle
import workloads as W
from tests.gpu_cases import compare_greedy, gpu_greedy, say

pytestmark = pytest.mark.gpu

ATOL = 1e-5
MASKS = {"-1e10": -1e10, "-1e30": -1e30, "lowest": np.finfo(np.float32).min}
EDGES = [2049, 3072, 3073, 4096, 4097, 5120, 5121, 6144, 6145, 8192, 8193, 10240, 10241, 16384,
         16385, 32768]


def _case(V1, T, fill, dtype, seed=0):
    from workloads.synth import _f32_to_bf16_bits
    V = V1 - 1
    cfg = W.Config(8200 + V1 + seed, "edge", B=4, K=1, V=V, T=T, chunk=T, dtype="f32",
                   n_phrases=150, len_lo=1, len_hi=7, token_dist="zipf", zipf_s=1.2, logit_std=1.0,
                   blank_offset=1.0, n_case=V // 6)
    lists, cm = [list(p) for p in W.phrases(cfg)], W.class_map(cfg)
    # nested suffixes: chains of more than four states
    lists[1] += [lists[1][0][i:] for i in range(len(lists[1][0]))]
    long = np.arange(40, 52, dtype=np.int32)
    lists[1] += [long[i:] for i in range(len(long))]
    if seed % 2:  # classes of five members
        n5 = V // 7
        cm = np.arange(V + 1, dtype=np.int32)
        for k in range(1, 5):
            cm[k * n5:(k + 1) * n5] = np.arange(n5)
        cm[V] = -1
    mids = np.array([0, 1, -1, 3], np.int32)
    rows = np.array(W.logits(cfg))[:, :, 0]
    rng = np.random.default_rng(V1 + 7 * T)
    for b in (0, 1, 3):
        t = 0
        while t < T:
            ph = lists[b][int(rng.integers(len(lists[b])))]
            for i, v in enumerate(ph[:T - t]):
                rows[t + i, b, int(v)] += np.float32(4.0)
            t += len(ph)
    if fill == "equal":
        rows[...] = np.float32(0.25)
    elif fill == "masked":
        keep = rng.random(rows.shape) < 2.0 / V1
        keep[..., V] = rng.random(rows.shape[:-1]) < 0.5
        keep[..., 5] |= ~keep.any(-1)
        rows[~keep] = -np.inf
    elif fill in MASKS:  # 100 tokens kept, all within one wave's share of a row
        keep = np.zeros(V1, bool)
        keep[V1 // 2 - V1 // 2 % 256:][:100] = True
        rows[..., ~keep] = np.float32(MASKS[fill])
    if dtype == "bf16":
        rows = _f32_to_bf16_bits(rows)
        if fill == "lowest":  # bfloat16's own (the float32 one rounds to -inf)
            rows[..., ~keep] = 0xff7f
    return cfg, lists, cm, mids, rows


def _check(V1, T, chunk, fill, dtype, seed=0):
    from paper_2608_21343_amd.decoder import BoostDecoder, to_device_logits
    say(f"[greedy edge] V+1={V1} T={T} chunk={chunk} {fill} {dtype}")
    cfg, lists, cm, mids, rows = _case(V1, T, fill, dtype, seed)
    dec = BoostDecoder(lists, cm, token_w=cfg.token_w, end_bonus=cfg.end_bonus)
    graphs = {m: oracle.build_graph(lists[m], cm, token_w=cfg.token_w, end_bonus=cfg.end_bonus)
              for m in (0, 1, 3)}
    st0 = np.where(mids >= 0, 0, -1).astype(np.int32)
    compare_greedy(gpu_greedy(dec, to_device_logits(rows), mids, chunk),
                   oracle.greedy_decode(graphs, mids, rows, st0), range(cfg.B), ATOL)


@pytest.mark.parametrize("i", range(len(EDGES)))
def test_row_instance_edges(i):
    _check(EDGES[i], 20, (20, 7, 1)[i % 3], "normal", ("f32", "bf16")[i % 2], i)
    _check(EDGES[i], 3, 3, "normal", ("bf16", "f32")[i % 2], i)


@pytest.mark.parametrize("T", [1, 2, 15, 16, 17, 63, 64, 65, 200])
def test_call_lengths(T):
    _check(2305, T, T, "normal", "f32", T)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V1", [2049, 3072, 3073, 4096, 4097, 6144, 6145, 8448, 8449, 10496, 10497])
def test_calls_of_few_steps(V1, dtype):
    """Calls of one to seven steps on both sides of the line between the kernel
    that scores every token and the row summaries, which lies where the rows'
    instance, the type and the streams (from 128 and 256 on) set it. The streams
    repeat four streams."""
    from paper_2608_21343_amd.decoder import BoostDecoder, to_device_logits
    T = 14
    cfg, lists, cm, mids, rows = _case(V1, T, "normal", dtype, V1 % 2)
    dec = BoostDecoder(lists, cm, token_w=cfg.token_w, end_bonus=cfg.end_bonus)
    graphs = {m: oracle.build_graph(lists[m], cm, token_w=cfg.token_w, end_bonus=cfg.end_bonus)
              for m in (0, 1, 3)}
    st0 = np.where(mids >= 0, 0, -1).astype(np.int32)
    ref = oracle.greedy_decode(graphs, mids, rows, st0)
    dev = to_device_logits(rows)
    for B, chunks in ((4, (1, 2, 3, 4, 5)), (128, (1, 3, 5)), (256, (1, 2, 4, 6, 7))):
        for chunk in chunks:
            say(f"[greedy edge] few steps V+1={V1} {dtype} B={B} chunk={chunk}")
            got = gpu_greedy(dec, dev.repeat(1, B // 4, 1), np.tile(mids, B // 4), chunk)
            for i in range(0, B, 4):
                compare_greedy(got, ref, range(i, i + 4), ATOL, range(4))


@pytest.mark.parametrize("V1", [65, 1280, 1281, 2048])
def test_boundary_fix_up_of_narrow_rows(V1):
    """Calls of several workgroups a stream through the fix-up kernel, on both
    sides of its change from sixteen waves to eight (1280 values)."""
    _check(V1, 300, 300, "normal", "f32", 1)
    _check(V1, 300, 300, "normal", "bf16", 2)


def test_call_of_several_pieces():
    """More steps than LDS holds row records for (48 bytes each)."""
    _check(2049, 3500, 3500, "normal", "bf16")


@pytest.mark.parametrize("fill", ["equal", "masked"])
@pytest.mark.parametrize("V1", [2049, 4100, 8193])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_equal_and_masked_rows(V1, fill, dtype):
    _check(V1, 12, 12, fill, dtype, 1)
    _check(V1, 12, 12, fill, dtype, 2)


@pytest.mark.parametrize("fill", MASKS)
@pytest.mark.parametrize("V1", [2049, 8193, 12000])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rows_masked_with_a_finite_value(V1, fill, dtype):
    """Three of a row's four waves hold nothing but the mask value: their sums
    weigh nothing, whatever the rounding of such values."""
    _check(V1, 6, 6, fill, dtype, 1)


@pytest.mark.parametrize("V1,dtype,chunk", [(2305, "f32", 14), (2305, "bf16", 1), (8193, "f32", 3),
                                            (8193, "bf16", 14), (3001, "f32", 4), (6001, "f32", 2),
                                            (6001, "bf16", 1), (8193, "f32", 1)])
@pytest.mark.parametrize("seed", [1, 2])
def test_rows_of_nan_and_of_no_finite_value(V1, dtype, chunk, seed):
    """A nan never wins: tokens and states are the oracle's for the same rows
    with -inf in its place. Among rows without a finite key the lowest token
    that is no nan is taken (the blank after the tokens), at its own move. The
    scores of such rows, and of rows that hold a nan, are nan."""
    from paper_2608_21343_amd.decoder import BoostDecoder, to_device_logits
    from workloads.synth import _f32_to_bf16_bits
    T, V = 14, V1 - 1
    cfg, lists, cm, mids, rows = _case(V1, T, "normal", "f32", seed)
    say(f"[greedy edge] nan and -inf rows V+1={V1} {dtype} chunk={chunk} seed={seed}")
    n = V // 7 if seed % 2 else V // 6  # first members of the classes
    rows[2, :, V] = np.nan
    rows[4, :, :n] = np.nan
    rows[4, :, n:2 * n] += np.float32(3.0)
    rows[5, :, 0] = np.nan  # the blank is the best
    rows[5, :, V] = 20.0
    rows[6] = -np.inf
    rows[8, :, :V] = -np.inf
    rows[8, :, :5] = np.nan
    rows[8, :, V] = -np.inf
    rows[9] = np.nan
    rows[11] = np.nan
    rows[11, :, V] = -np.inf
    want = np.where(np.isnan(rows), np.float32(-np.inf), rows)
    want[8, :, 5] = want[11, :, V] = 0.0  # the rows' lowest entries that are no nan
    if dtype == "bf16":
        rows, want = _f32_to_bf16_bits(rows), _f32_to_bf16_bits(want)
    dec = BoostDecoder(lists, cm, token_w=cfg.token_w, end_bonus=cfg.end_bonus)
    graphs = {m: oracle.build_graph(lists[m], cm, token_w=cfg.token_w, end_bonus=cfg.end_bonus)
              for m in (0, 1, 3)}
    st0 = np.where(mids >= 0, 0, -1).astype(np.int32)
    got = gpu_greedy(dec, to_device_logits(rows), mids, chunk)
    with np.errstate(invalid="ignore"):
        ref = oracle.greedy_decode(graphs, mids, want, st0)
    none = np.isin(np.arange(T), [2, 4, 5, 6, 8, 9, 11])
    assert np.isnan(got[2][none]).all()
    compare_greedy([a[~none] for a in got[:3]], [a[~none] for a in ref[:3]], range(cfg.B), ATOL)
    assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])
    assert (got[1][[6, 8], :2] >= 0).all() and (ref[1][:, [0, 1, 3]] > 0).any()


def test_nan_in_a_wave_without_finite_values():
    """The score of a row is nan when its only nan lies in a wave's share that
    holds -inf besides (tokens 256..511 of every 1024 in float32)."""
    from paper_2608_21343_amd.decoder import BoostDecoder, to_device_logits
    cfg, lists, cm, mids, rows = _case(8193, 3, "normal", "f32")
    dec = BoostDecoder(lists, cm)
    rows[1, :, :8192].reshape(4, 8, 4, 256)[:, :, 1] = -np.inf
    rows[1, 0, 300] = rows[1, 2, 300] = np.nan
    tok, _, sc, _ = gpu_greedy(dec, to_device_logits(rows), mids, 3)
    assert np.isnan(sc[1, [0, 2]]).all() and not np.isnan(sc[1, [1, 3]]).any()
    assert not np.isnan(sc[[0, 2]]).any()


@pytest.mark.parametrize("V1", [300, 2305])
def test_nan_row_leaves_other_streams(V1):
    from paper_2608_21343_amd.decoder import BoostDecoder, to_device_logits
    cfg, lists, cm, mids, rows = _case(V1, 18, "normal", "f32")
    dec = BoostDecoder(lists, cm)
    clean = gpu_greedy(dec, to_device_logits(rows), mids, 18)
    rows[7, 1, 9] = np.nan
    got = gpu_greedy(dec, to_device_logits(rows), mids, 18)
    for a, b in zip(clean[:3], got[:3]):
        assert np.array_equal(a[:, [0, 2, 3]], b[:, [0, 2, 3]])
    assert got[0].min() >= 0 and got[0].max() <= cfg.V
