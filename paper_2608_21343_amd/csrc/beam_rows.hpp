// Row summaries of a beam call: the part of a step that does not depend on
// the hypotheses, for every row (t, b, k) of the call at once.
//
//  * the normaliser: log of the float64 sum of exponentials, rounded once to
//    float32 (beam scores are carried and compared, so they follow the exact
//    reading);
//  * the kList best root moves z + psi(root move) in (value descending, token
//    ascending) order (psi of the stream's model; zero for unbiased streams).
//
// They are stored in the call's own output rows of that (t, b, k): out_step
// holds the normaliser and out_tok, out_parent, out_state and out_cum two
// 16-bit token ids each (0xffff: none). The step kernel reads a row's entry
// before it writes the row's outputs, so the call needs no workspace.
//
// One wave per row up to 2048 values, four waves above. The kernel is bound
// by vector instructions, most of them the exponentials (21 a value, 13 in
// float64): 131,072 rows of 1025 float32 take 197 us, 65,536 of 8193 bfloat16
// 569 us, where reading them takes 104 and 207 us at a copy's rate. The sum is
// taken of e^z itself, not of e^(z - max), so that the row is passed once and no
// value waits for a maximum; float64 holds e^z for |z| <= 700, and a row whose
// sum leaves [1e-280, 1e280] (or holds a nan) is summed again relative to its
// maximum.
#pragma once

#include <climits>

#include "beam_list.hpp"
#include "device.hpp"

namespace tbias {
namespace blist {

// e^x in float64 for float32 x, as 2^k e^r with r = x - k ln 2 in
// [-0.3475, 0.3475] and e^r by a degree-11 polynomial (minimax in the relative
// error, by Remez exchange; 1.6e-17 with its coefficients rounded). x is clamped
// to [-700, 700]: 2^k is then added into the exponent field. ln 2 is taken in two
// parts: k times the first, of 15 bits, is subtracted in float32 without an error
// (the difference lies on a grid of which it spans fewer than 2^24 steps).
// Largest relative error 1.5e-16 over the whole range.
__device__ __forceinline__ double exp_f32(float x) {
  x = __builtin_amdgcn_fmed3f(x, -700.0f, 700.0f);
  const float magic = 12582912.0f;  // 1.5 * 2^23: the sum's low bits are the integer
  const float t = __builtin_fmaf(x, 1.44269504f, magic);
  const float k = t - magic;
  const double r = __builtin_fma(-(double)k, 0x1.7f7d1cf79abcap-20,
                                 (double)__builtin_fmaf(-k, 0x1.62e4p-1f, x));
  double p = 0x1.ad64c1d19cd83p-26;
  p = __builtin_fma(p, r, 0x1.28b42b3d7df6ep-22);
  p = __builtin_fma(p, r, 0x1.71df47fc1ca59p-19);
  p = __builtin_fma(p, r, 0x1.a01991a1cec39p-16);
  p = __builtin_fma(p, r, 0x1.a01a010e063f0p-13);
  p = __builtin_fma(p, r, 0x1.6c16c187f1c93p-10);
  p = __builtin_fma(p, r, 0x1.11111111318cbp-7);
  p = __builtin_fma(p, r, 0x1.555555554f156p-5);
  p = __builtin_fma(p, r, 0x1.555555555549dp-3);
  p = __builtin_fma(p, r, 0x1.0000000000010p-1);
  p = __builtin_fma(p, r, 1.0);
  p = __builtin_fma(p, r, 1.0);
  const uint32_t hi = (uint32_t)__double2hiint(p) + ((uint32_t)__float_as_int(t) << 20);
  return __hiloint2double((int)hi, __double2loint(p));
}

// Sum over the wave (row shifts within rows of 16 lanes, then the row
// broadcasts, on both words of a float64), uniform.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_d(double v) {
  return __hiloint2double(dpp_i<CTRL, ROW_MASK>(0, __double2hiint(v)),
                          dpp_i<CTRL, ROW_MASK>(0, __double2loint(v)));
}
__device__ __forceinline__ double wave_sum_dpp_d(double v) {
  v += dpp_d<0x111, 0xf>(v);
  v += dpp_d<0x112, 0xf>(v);
  v += dpp_d<0x114, 0xf>(v);
  v += dpp_d<0x118, 0xf>(v);
  v += dpp_d<0x142, 0xa>(v);
  v += dpp_d<0x143, 0xc>(v);
  return __hiloint2double(rl(__double2hiint(v), 63), rl(__double2loint(v), 63));
}

constexpr int kRowThreads = 256;

// NWR waves per row; a wave's chunk j holds the row's values (j * NWR + q) * 64
// + lane. Chunks below NF lie before the blank for every row that runs this
// instance (no test of the index); those up to NC are tested. Four workgroups a
// CU (128 registers) for all but the longest rows: 131 would leave three.
template <class Ld, int NWR, int NF, int NC>
__global__ __launch_bounds__(kRowThreads, NC <= 40 ? 4 : 1) void beam_rows_kernel(
    ArenaView A, const typename Ld::T* __restrict__ logits, int64_t r0, int64_t n_rows, int32_t B,
    int32_t K, int64_t stride, const int32_t* __restrict__ model_ids,
    const int32_t* __restrict__ states, int32_t* __restrict__ out_tok,
    int32_t* __restrict__ out_parent, int32_t* __restrict__ out_state,
    float* __restrict__ out_step, float* __restrict__ out_cum) {
  constexpr int kWaves = kRowThreads / 64, kRows = kWaves / NWR;
  __shared__ uint64_t g_key[kRows][64];  // moves in (value, token) order: order_key, ~token
  __shared__ double g_sum[kWaves];
  __shared__ float g_max[kWaves][64];
  __shared__ int32_t g_count[kRows];
  lds_poison(g_key, sizeof(g_key));
  lds_poison(g_max, sizeof(g_max));
  const int lane = __lane_id();
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q = wv % NWR, rw = wv / NWR;  // part of the row, row of the workgroup
  const int64_t r = r0 + (int64_t)blockIdx.x * kRows + rw;
  if (r >= n_rows) return;  // uniform per wave (per workgroup when waves share a row)
  const int32_t V1 = A.V1, V = V1 - 1;
  const int32_t b = (int32_t)((r / K) % B);
  // the step kernel's decision: biased when the model id and every carried
  // state of the stream are in range
  const int32_t m = model_ids[b];
  bool biased = m >= 0 && m < A.n_models;
  if (biased) {
    const int32_t n = A.model_n[m];
    const int32_t s = (lane < K) ? states[(int64_t)b * K + lane] : 0;
    biased = __ballot(s < 0 || s >= n) == 0ull;
  }
  const typename Ld::T* row = logits + r * stride + q * 64;
  const float* gpsi = A.root_psi + (int64_t)(biased ? m : 0) * V1 + q * 64;
  auto index = [&](int j) { return (j * NWR + q) * 64 + lane; };
  auto used = [&](int j) { return j < NF || (j * NWR + q) * 64 < opaque(V1); };  // uniform

  // the tested chunks: rows that end within the first one pass over the others
  // with one test
  const bool more = ((NF + 1) * NWR + q) * 64 < V1;
  auto tested = [&](auto f) {
    if (used(NF)) f(NF);
    if (more) {
#pragma unroll
      for (int j = NF + 1; j < NC; ++j)
        if (used(j)) f(j);
    }
  };

  float z[NC], y[NC];
#pragma unroll
  for (int j = 0; j < NF; ++j) z[j] = Ld::get(row, j * NWR * 64 + lane);
#pragma unroll
  for (int j = 0; j < NF; ++j) y[j] = biased ? gpsi[j * NWR * 64 + lane] : 0.f;
#pragma unroll
  for (int j = NF; j < NC; ++j) z[j] = y[j] = kNegInf;
  tested([&](int j) {
    if (index(j) < V1) {
      z[j] = Ld::get(row, j * NWR * 64 + lane);
      y[j] = biased ? gpsi[j * NWR * 64 + lane] : 0.f;
    }
  });

  // normaliser, and every lane's best move (a nan stays)
  double se = 0.0;
  float lm = kNegInf;
  // waves that share a row keep the best of every eight values: few of these
  // groups hold one of the row's best moves
  constexpr int NG = (NC + 7) / 8;
  float group[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) group[g] = kNegInf;
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    se += exp_f32(z[j]);
    y[j] = z[j] + y[j];
    float& best = NWR > 1 ? group[j / 8] : lm;
    best = __builtin_elementwise_maximum(best, y[j]);
  }
#pragma unroll
  for (int g = 0; g < (NWR > 1 ? NG : 0); ++g) lm = __builtin_elementwise_maximum(lm, group[g]);
  bool bad = lm != lm;
  tested([&](int j) {
    const double e = exp_f32(z[j]);
    se += index(j) < V1 ? e : 0.0;
    bad = bad || z[j] != z[j];
    y[j] = index(j) < V ? z[j] + y[j] : kNegInf;
    lm = __builtin_fmaxf(lm, y[j]);
    if (NWR > 1) group[j / 8] = __builtin_elementwise_maximum(group[j / 8], y[j]);
  });
  se = wave_sum_dpp_d(se);
  if (__ballot(bad) != 0ull) {  // nan values: their sum is nan, the other moves are listed
    se = __builtin_nan("");
    lm = kNegInf;
#pragma unroll
    for (int j = 0; j < NC; ++j) lm = __builtin_fmaxf(lm, y[j]);
  }
  float om[NWR > 1 ? NWR : 1];  // the lane maxima of the row's waves
  om[0] = lm;
  if constexpr (NWR > 1) {
    g_max[wv][lane] = lm;
    if (lane == 0) g_sum[wv] = se;
    if (threadIdx.x == 0) g_count[0] = 0;
    __syncthreads();
    se = 0.0;
#pragma unroll
    for (int i = 0; i < NWR; ++i) {
      se += g_sum[i];
      om[i] = g_max[i][lane];
    }
  }
  double lse = 0.0;
  if (!(se > 1e-280 && se < 1e280)) {  // uniform over the row's waves
    float zm = kNegInf;
#pragma unroll 1
    for (int32_t v = lane; v < V1; v += 64) zm = __builtin_fmaxf(zm, Ld::get(row - q * 64, v));
    zm = wave_max_dpp(zm);
    const double zmd = (double)zm;
    double s2 = 0.0;
#pragma unroll 1
    for (int32_t v = lane; v < V1; v += 64) s2 += exp((double)Ld::get(row - q * 64, v) - zmd);
    lse = zmd + log(wave_sum_d(s2));
  } else if (NWR == 1 || q == 0) {
    lse = log(se);
  }

  // the row's kList best root moves. At least kList lanes hold a move that
  // reaches theta, a lane maximum found by bisection over the gap to the best
  // (as the step kernel's bound); the moves that reach it (about ten) are
  // gathered in LDS and ranked.
  float best = kNegInf;
#pragma unroll
  for (int i = 0; i < NWR; ++i) best = __builtin_fmaxf(best, om[i]);
  best = wave_max_dpp(best);
  int32_t bound = 0;
  {
    int32_t gap[NWR];
#pragma unroll
    for (int i = 0; i < NWR; ++i) gap[i] = gap_of(best, om[i]);
#pragma unroll
    for (int bit = 8; bit >= 0; --bit) {
      const int32_t c = bound | (1 << bit);
      int32_t cnt = 0;
#pragma unroll
      for (int i = 0; i < NWR; ++i) cnt += (int32_t)__builtin_popcountll(__ballot(gap[i] < c));
      if (cnt < kList) bound = c;
    }
  }
  int32_t total = INT_MAX;
  auto key_of = [&](float v, int32_t tok) { return ((uint64_t)order_key(v) << 32) | (uint32_t)~tok; };
  if (bound < kNone) {
    float th = kNegInf;  // the smallest lane maximum within the bound
#pragma unroll
    for (int i = 0; i < NWR; ++i) th = __builtin_fmaxf(th, gap_of(best, om[i]) <= bound ? -om[i] : kNegInf);
    const float theta = -wave_max_dpp(th);
    total = 0;
    bool any = true;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      if (NWR > 1 && j % 8 == 0) any = __ballot(!(group[j / 8] < theta)) != 0ull;  // or a nan
      if (!any) continue;
      const bool hit = used(j) && y[j] >= theta;
      const uint64_t in = __ballot(hit);
      if (in == 0ull) continue;
      const int32_t n = (int32_t)__builtin_popcountll(in);
      int32_t base = total;
      if constexpr (NWR > 1) {
        if (lane == 0)
          base = __hip_atomic_fetch_add(&g_count[0], n, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_WORKGROUP);
        base = __builtin_amdgcn_readfirstlane(base);
      }
      total += n;
      const int32_t pos = base + (int32_t)lanes_below(in);
      if (hit && pos < 64) g_key[rw][pos] = key_of(y[j], index(j));
    }
  }
  if constexpr (NWR > 1) {
    __syncthreads();
    if (bound < kNone) total = __builtin_amdgcn_readfirstlane(g_count[0]);
  }
  if (total > 64) {  // uniform over the row's waves
    // fewer than kList lanes with a finite move, or very many equal values:
    // kList rounds of a wave argmax over the moves after the last one taken
    if constexpr (NWR > 1) __syncthreads();  // g_key is rewritten
    float pk = 0.f;
    int32_t pt = -1;
    uint64_t mine = 0ull;
    for (int32_t i = 0; i < kList; ++i) {
      float bk = kNegInf;
      int32_t bt = INT_MAX;
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        const int32_t v = index(j);
        const bool after = i == 0 || y[j] < pk || (y[j] == pk && v > pt);
        if (used(j) && after && y[j] > kNegInf && better(y[j], v, bk, bt)) {
          bk = y[j];
          bt = v;
        }
      }
      wave_argmax_dpp(bk, bt, pk, pt);
      if (pt == INT_MAX) break;
      if (lane == i) mine = key_of(pk, pt);
    }
    if (lane < kList) g_key[rw][q * kList + lane] = mine;  // 0: none
    total = NWR * kList;
    if constexpr (NWR > 1) __syncthreads();
  }
  if (NWR > 1 && q != 0) return;  // no barrier follows
  asm volatile("" ::: "memory");
  const uint64_t key = lane < total ? g_key[rw][lane] : 0ull;
  const int32_t khi = (int32_t)(uint32_t)(key >> 32), klo = (int32_t)(uint32_t)key;
  int32_t rank = 0;
  for (int32_t i = 0; i < total; i += 4) {  // lanes past total hold 0
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint64_t ki = ((uint64_t)(uint32_t)rl(khi, i + u) << 32) | (uint32_t)rl(klo, i + u);
      rank += ki > key ? 1 : 0;
    }
  }
  const int32_t to = 4 * ((key != 0ull && rank < kList) ? rank : 63);
  const int32_t sent = __builtin_amdgcn_ds_permute(to, klo);  // 0 where nothing was sent
  const int32_t tok = lane < kList && sent != 0 ? ~sent : -1;
  // lanes 0..3 store two tokens each
  const int32_t lo = __shfl(tok, 2 * lane, 64), hi = __shfl(tok, 2 * lane + 1, 64);
  const uint32_t word = ((uint32_t)lo & 0xffffu) | ((uint32_t)hi << 16);
  if (lane == 0) {
    out_tok[r] = (int32_t)word;
    out_step[r] = (float)lse;
  }
  if (lane == 1) out_parent[r] = (int32_t)word;
  if (lane == 2) out_state[r] = (int32_t)word;
  if (lane == 3) out_cum[r] = __uint_as_float(word);
}

// ---- launch

typedef hipError_t (*RowsLaunch)(const ArenaView&, const void*, int32_t, int32_t, int32_t, int64_t,
                                 const int32_t*, const int32_t*, int32_t*, int32_t*, int32_t*,
                                 float*, float*, hipStream_t);
typedef hipError_t (*StepLaunch)(const ArenaView&, const void*, int32_t, int32_t, int32_t, int64_t,
                                 const int32_t*, int32_t*, float*, int32_t*, int32_t*, int32_t*,
                                 float*, float*, StreamArgs, hipStream_t);
RowsLaunch rows_launcher_f32(int32_t V1);
RowsLaunch rows_launcher_bf16(int32_t V1);
StepLaunch step_launcher_f32(int32_t K, bool stream, bool rows);
StepLaunch step_launcher_bf16(int32_t K, bool stream, bool rows);

template <class Ld, int NWR, int NF, int NC>
hipError_t launch_rows_t(const ArenaView& A, const void* logits, int32_t T, int32_t B, int32_t K,
                         int64_t stride, const int32_t* model_ids, const int32_t* states,
                         int32_t* out_tok, int32_t* out_parent, int32_t* out_state,
                         float* out_step, float* out_cum, hipStream_t st) {
  // rows [r0, n_rows) in launches of as many workgroups as one may have
  const int64_t n_rows = (int64_t)T * B * K;
  constexpr int64_t kPer = (kRowThreads / 64) / NWR, kMost = kPer * most_groups(kRowThreads);
  for (int64_t r0 = 0; r0 < n_rows; r0 += kMost) {
    const int64_t nr = n_rows - r0 < kMost ? n_rows - r0 : kMost;
    hipLaunchKernelGGL((beam_rows_kernel<Ld, NWR, NF, NC>), dim3((uint32_t)((nr + kPer - 1) / kPer)),
                       dim3(kRowThreads), 0, st, A, static_cast<const typename Ld::T*>(logits), r0,
                       n_rows, B, K, stride, model_ids, states, out_tok, out_parent, out_state,
                       out_step, out_cum);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// The instance for rows of V1 values: its untested chunks lie before the blank
// (NF * NWR * 64 <= V) and its chunks hold the row. Four tested chunks at
// most up to 5120 values; more above, where they weigh less.
template <class Ld>
RowsLaunch rows_launcher_t(int32_t V1) {
  if (V1 <= 64 * 4) return launch_rows_t<Ld, 1, 0, 4>;
  if (V1 <= 64 * 8) return launch_rows_t<Ld, 1, 4, 8>;
  if (V1 <= 64 * 12) return launch_rows_t<Ld, 1, 8, 12>;
  if (V1 <= 64 * 16) return launch_rows_t<Ld, 1, 12, 16>;
  if (V1 <= 64 * 20) return launch_rows_t<Ld, 1, 16, 20>;
  if (V1 <= 64 * 24) return launch_rows_t<Ld, 1, 20, 24>;
  if (V1 <= 64 * 28) return launch_rows_t<Ld, 1, 24, 28>;
  if (V1 <= 64 * 32) return launch_rows_t<Ld, 1, 28, 32>;
  if (V1 <= 256 * 12) return launch_rows_t<Ld, 4, 8, 12>;
  if (V1 <= 256 * 16) return launch_rows_t<Ld, 4, 12, 16>;
  if (V1 <= 256 * 20) return launch_rows_t<Ld, 4, 16, 20>;
  if (V1 <= 256 * 24) return launch_rows_t<Ld, 4, 20, 24>;
  if (V1 <= 256 * 32) return launch_rows_t<Ld, 4, 24, 32>;
  if (V1 <= 256 * 40) return launch_rows_t<Ld, 4, 32, 40>;
  if (V1 <= 256 * 64) return launch_rows_t<Ld, 4, 40, 64>;
  return launch_rows_t<Ld, 4, 64, 128>;
}

// LDS of the step kernel: the rows (ROWS), the class bitmaps, and with what
// is left records of the model's first states. Records are filled once a
// call (20 bytes read per state) and save a trip to the cache per step, so a
// call of fewer than kHotSteps steps does without: with / without them, 64
// streams, 4 hypotheses of 1024 float32, calls of 4, 12, 16, 32 and 64 steps take
// 33 / 30, 64 / 62, 81 / 78, 149 / 149 and 269 / 272 us, 8 hypotheses 38 / 37, 77 / 76,
// 98 / 99, 182 / 185 and 329 / 334, 4 of 8192 bfloat16 48 / 44, 100 / 98, 124 / 123,
// 226 / 229 and 431 / 439; 32 hypotheses of 1000 float32, calls of 4 and 8 steps 93 / 94
// and 264 / 267, so above 16 hypotheses four steps are enough. (A model with a record that does not fit, such as a state
// of 255 children, runs without them: these figures are what that costs.)
constexpr int kHotSteps = 16;
constexpr int kLdsBytes = 160 * 1024;
// LDS given to rows; the records need the rest. Rows in LDS against rows gathered
// from memory, calls of 32 steps: 177 / 196 us (8 hypotheses of 1024 float32, 33 KB),
// 147 / 168 (4 of 500 bfloat16), 205 / 208 (8 of 2000 float32, 64 KB); 16 of 1000
// float32 (64 KB) 334 / 333, and above the line 379 / 358 (12 of 2000 float32, 96 KB)
// and 512 / 490 (16 of them, 128 KB).
constexpr int kMostRows = 72 * 1024;

inline int32_t row_bytes(int32_t V1, size_t item) {
  return (int32_t)(((size_t)V1 * item + 15) / 16 * 16);
}
inline bool rows_in_lds(int32_t V1, int32_t K, size_t item) {
  return K <= 16 && V1 <= 2048 && (int64_t)K * row_bytes(V1, item) <= kMostRows;
}

inline Layout make_layout(const ArenaView& A, int32_t T, int32_t K, size_t item, bool rows,
                          size_t fixed) {
  Layout l;
  l.rows = 0;
  l.row_stride = rows ? row_bytes(A.V1, item) : 0;
  l.marks = K * l.row_stride;
  l.mark_words = (A.V1 + 31) / 32;
  l.hot = (l.marks + 4 * K * l.mark_words + 15) / 16 * 16;
  const int64_t room = (kLdsBytes - 1024 - (int64_t)fixed - l.hot) / 16;
  l.nhot = (T >= (K > 16 ? 4 : kHotSteps) && room > 0) ? (int32_t)(room < 8192 ? room : 8192) : 0;
  if (l.nhot > A.n_states) l.nhot = (int32_t)A.n_states;
  l.total = l.hot + 16 * l.nhot;
  return l;
}

template <class Ld, int NW, int KPW, int NS, bool STREAM, bool ROWS>
hipError_t launch_step_t(const ArenaView& A, const void* logits, int32_t T, int32_t B, int32_t K,
                         int64_t stride, const int32_t* model_ids, int32_t* states, float* scores,
                         int32_t* out_tok, int32_t* out_parent, int32_t* out_state,
                         float* out_step, float* out_cum, StreamArgs sa, hipStream_t st) {
  auto kernel = &beam_list_kernel<Ld, NW, KPW, NS, STREAM, ROWS>;
  const Layout l = make_layout(A, T, K, sizeof(typename Ld::T), ROWS,
                               sizeof(Shared<NW * KPW, NW>));
  allow_dynamic_lds(kernel, (size_t)kLdsBytes - sizeof(Shared<NW * KPW, NW>) - 1024);
  // streams [b0, B) in launches of as many workgroups as one may have
  constexpr int64_t kMost = most_groups(64 * NW);
  for (int64_t b0 = 0; b0 < B; b0 += kMost) {
    const int64_t nb = B - b0 < kMost ? B - b0 : kMost, k0 = b0 * K;
    StreamArgs s = sa;
    if constexpr (STREAM) {
      s.hyps += k0;
      if (s.tree) s.tree += b0 * sa.cap * 2;
      s.tree_len += b0;
    }
    hipLaunchKernelGGL(kernel, dim3((uint32_t)nb), dim3(64 * NW), (size_t)l.total, st, A,
                       static_cast<const typename Ld::T*>(logits) + k0 * stride, T, B, K, stride,
                       model_ids + b0, states + k0, scores + k0, out_tok + k0, out_parent + k0,
                       out_state + k0, out_step + k0, out_cum + k0, s, l);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Waves: one per slot up to 16, then two slots each. Children per lane: two
// (128 children; a fifth of the states of 1000-phrase lists have more than
// 64), four for the wide rows of long lists, one where sixteen waves leave 128
// registers to each.
template <class Ld, bool STREAM>
StepLaunch step_launcher_s(int32_t K, bool rows) {
  if (K <= 4)
    return rows ? launch_step_t<Ld, 4, 1, 2, STREAM, true> : launch_step_t<Ld, 4, 1, 4, STREAM, false>;
  if (K <= 8)
    return rows ? launch_step_t<Ld, 8, 1, 2, STREAM, true> : launch_step_t<Ld, 8, 1, 4, STREAM, false>;
  if (K <= 16)
    return rows ? launch_step_t<Ld, 16, 1, 1, STREAM, true>
                : launch_step_t<Ld, 16, 1, 1, STREAM, false>;
  return launch_step_t<Ld, 16, 2, 1, STREAM, false>;
}

}  // namespace blist
}  // namespace tbias
