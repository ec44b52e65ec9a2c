// Boosted greedy step from row summaries: a summary kernel over all rows of
// the call, then one workgroup per stream that walks its rows in parallel
// segments (templates; instantiated in greedy_list_*.hip).
//
// A call over wide rows should cost one read of the logits. What kept it
// from that was the scoring of every token from the current state, row after
// row (12 thousand cycles a row of 8192 tokens; 256 streams of 256 bfloat16
// rows took 2.40 ms, now 0.37 ms for the summaries and 0.18 ms for the walk,
// where reading the rows takes 0.21 ms). Calls of very few steps are the
// exception (greedy_wide.hip). Only the children along the
// state's suffix chain depend on the state; the normaliser and the best root
// moves do not, and are taken for all rows at once:
//
//  * greedy_rows_kernel: per row the float32 normaliser (maximum, then the
//    sum of exponentials relative to it) and the kBest best root moves z +
//    psi(root move) in (value, token) order, kept in the call's own output
//    rows (out_score: the normaliser; out_tok, out_state: two 16-bit token
//    ids each) until the walk has read them;
//  * greedy_walk_kernel: the stream's summaries go to LDS (one thread per
//    row also gathers the best move's logit, psi, class and target and the
//    blank's logit), then wave w steps through segment w of the rows. A
//    segment that does not start the call begins kWarm rows early from the
//    root: from most states the best move is a root move, so trajectories
//    meet within a few rows. A step gathers the children of the suffix chain
//    (one per lane and register) and compares their best with the blank and
//    with the best root move whose class no child has. Afterwards every
//    segment whose start differs from the previous segment's end is
//    walked again from there until it meets its stored states; rounds of this
//    (all such segments at once) end when no start differs, after which every
//    segment follows from the carried state.
#pragma once

#include <climits>

#include "beam_list.hpp"
#include "device.hpp"
#include "launch.hpp"

namespace tbias {
namespace glist {

using blist::arc_class;
using blist::arc_more;
using blist::gap_of;
using blist::gload;
using blist::kNegInf;
using blist::kNone;
using blist::lanes_below;
using blist::opaque;
using blist::order_key;
using blist::rl;
using blist::rlf;
using blist::sload;

// Root moves listed per row: two words of a row's outputs hold four. With two the
// row is scanned more often: 32 streams of 64 rows of 4097 float32 61 us against 52,
// 256 streams of 64 rows of 8193 bfloat16 169 against 154.
constexpr int kBest = 4;
// Warm-up rows of a guessed segment start. Two, four and seven measure within the
// spread of one another over lists of 1000 and 5000 phrases (128 streams of 64 rows
// of 4097 float32: 83, 81, 81 and 140, 125, 137 us; 256 rows: 195, 197, 204 and 257,
// 260, 263).
constexpr int kWarm = 4;
constexpr int kRowThreads = 256;
constexpr int kWalkThreads = 1024;
constexpr int kLevels = 4;  // chain states whose children are taken one per lane
constexpr float kLog2e = 1.4426950408889634f;

// NWR waves per row. A lane holds NP pieces of PV = 16 / sizeof(element)
// neighbouring values (one 16-byte load each, at the alignment of the
// elements), all before the blank for every row that runs this instance, then
// NC chunks of one value each, which are tested against the row's end. Bound
// by instructions, of which a wave of 8193 bfloat16 values spends fewer on the
// values than on what follows them: passing over the unused chunks with one
// test (407 -> 386 us for 65,536 rows) and over groups of eight values that
// hold none of the best moves (419 -> 407 us) counts.
template <class Ld, int NWR, int NP, int NC>
__global__ __launch_bounds__(kRowThreads) void greedy_rows_kernel(
    ArenaView A, const typename Ld::T* __restrict__ logits, int64_t r0, int64_t n_rows, int32_t B,
    int64_t stride, const int32_t* __restrict__ model_ids, const int32_t* __restrict__ states,
    int32_t* __restrict__ out_tok, int32_t* __restrict__ out_state,
    float* __restrict__ out_score) {
  typedef typename Ld::T LT;
  constexpr int kWaves = kRowThreads / 64, kRows = kWaves / NWR;
  constexpr int PV = 16 / sizeof(LT), NF = NP * PV, NZ = NF + NC;
  __shared__ uint64_t g_key[kRows][64];  // moves in (value, token) order: order_key, ~token
  __shared__ float g_sum[kWaves], g_max[kWaves], g_shift[kWaves], g_top[kWaves][64];
  __shared__ int32_t g_count[kRows];
  lds_poison(g_key, sizeof(g_key));
  lds_poison(g_top, sizeof(g_top));
  const int lane = __lane_id();
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q = wv % NWR, rw = wv / NWR;
  const int64_t r = r0 + (int64_t)blockIdx.x * kRows + rw;
  if (r >= n_rows) return;  // uniform per wave (per workgroup when waves share a row)
  const int32_t V1 = A.V1, V = V1 - 1;
  const int32_t b = (n_rows >> 31) == 0 ? (int32_t)((uint32_t)r % (uint32_t)B) : (int32_t)(r % B);
  const int32_t m = model_ids[b];
  int32_t off, n;
  const bool biased = resolve_stream(A, m, states[b], off, n) == 1;
  const LT* row = logits + r * stride;
  const float* gpsi = A.root_psi + (int64_t)(biased ? m : 0) * V1;
  // value j of this lane: pieces first, then the tested chunks
  const int32_t tail = NP * NWR * 64 * PV;
  auto index = [&](int j) {
    return j < NF ? ((j / PV * NWR + q) * 64 + lane) * PV + j % PV
                  : tail + ((j - NF) * NWR + q) * 64 + lane;
  };
  auto used = [&](int j) {  // uniform
    return j < NF || tail + ((j - NF) * NWR + q) * 64 < opaque(V1);
  };

  // the tested chunks: rows that end within the first one (a piece's edge and
  // the blank) pass over the others with one test
  const bool more = tail + (NWR + q) * 64 < V1;
  auto tested = [&](auto f) {
    if (used(NF)) f(NF);
    if (more) {
#pragma unroll
      for (int j = NF + 1; j < NZ; ++j)
        if (used(j)) f(j);
    }
  };

  float z[NZ], y[NZ];
  blist::Quad<LT> raw[NP > 0 ? NP : 1];
#pragma unroll
  for (int p = 0; p < NP; ++p)
    raw[p] = *reinterpret_cast<const blist::Quad<LT>*>(row + index(p * PV));
#pragma unroll
  for (int j = NF; j < NZ; ++j) z[j] = y[j] = kNegInf;
  tested([&](int j) {
    if (index(j) < V1) z[j] = Ld::get(row, index(j));
  });
#pragma unroll
  for (int p = 0; p < NF / 4; ++p) {
    blist::Quad<float> ps = {{0u, 0u, 0u, 0u}};
    if (biased) ps = *reinterpret_cast<const blist::Quad<float>*>(gpsi + index(4 * p));
#pragma unroll
    for (int e = 0; e < 4; ++e) y[4 * p + e] = __uint_as_float(ps.w[e]);
  }
  tested([&](int j) {
    if (index(j) < V1) y[j] = biased ? gpsi[index(j)] : 0.f;
  });
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int e = 0; e < PV; ++e) {
      const uint32_t wd = raw[p].w[e * sizeof(LT) / 4];
      z[p * PV + e] = __uint_as_float(sizeof(LT) == 4 ? wd : (e & 1) ? wd & 0xffff0000u : wd << 16);
    }
  float zm = kNegInf, top = kNegInf;
  constexpr int NG = (NZ + 7) / 8;
  float group[NG];  // the best of eight values
#pragma unroll
  for (int g = 0; g < NG; ++g) group[g] = kNegInf;
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    zm = __builtin_fmaxf(zm, z[j]);
    y[j] = z[j] + y[j];
    group[j / 8] = __builtin_fmaxf(group[j / 8], y[j]);
  }
  tested([&](int j) {
    zm = __builtin_fmaxf(zm, z[j]);
    y[j] = index(j) < V ? z[j] + y[j] : kNegInf;
    group[j / 8] = __builtin_fmaxf(group[j / 8], y[j]);
  });
#pragma unroll
  for (int g = 0; g < NG; ++g) top = __builtin_fmaxf(top, group[g]);
  // The wave's sum relative to its own maximum. The exponent z log2(e) - mL is
  // one instruction and off by the rounding of mL alone, which is taken out
  // where the waves' sums are added up. Where that rounding is not small (a wave
  // of nothing but mask values such as -1e30, where it exceeds every exponent)
  // the maximum is subtracted first. Largest error of the step scores against
  // float64, 4096 rows of 8193 float32 of deviation 1.5 around 0, 20, 100, 1000:
  // 1.1e-6, 1.5e-6, 4.3e-6, 3.1e-5 (with that rounding left in 1.1e-6, 2.5e-6,
  // 8.5e-6, 6.3e-5).
  static_assert(NWR > 1, "the factors of the waves' sums take the shift out");
  zm = wave_max_dpp(zm);
  const float ref = zm == kNegInf ? 0.f : zm;  // no finite value: the terms are 0 (or nan)
  auto exp_of = [](float x) { return __builtin_amdgcn_exp2f(x * kLog2e); };
  float se = 0.f, shift = 0.f;  // the sum is 2^shift times too large
  auto sum = [&](auto term) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {  // a piece at a time: less rounding than one chain
      float part = 0.f;
#pragma unroll
      for (int e = 0; e < PV; ++e) part += term(z[p * PV + e]);
      se += part;
    }
    tested([&](int j) { se += term(z[j]); });
  };
  if (__builtin_fabsf(ref) < 8192.f) {  // uniform
    const float mL = ref * kLog2e;
    sum([&](float x) { return __builtin_amdgcn_exp2f(__builtin_fmaf(x, kLog2e, -mL)); });
    shift = __builtin_fmaf(ref, kLog2e, -mL);
  } else {
    sum([&](float x) { return exp_of(x - ref); });
  }
  se = wave_sum_dpp(se);

  if constexpr (NWR > 1) {
    g_top[wv][lane] = top;
    if (lane == 0) {
      g_sum[wv] = se;
      g_max[wv] = zm;
      g_shift[wv] = shift;
    }
    if (threadIdx.x == 0) g_count[0] = 0;
    __syncthreads();
    zm = kNegInf;
#pragma unroll
    for (int i = 0; i < NWR; ++i) {
      zm = __builtin_fmaxf(zm, g_max[i]);
      top = __builtin_fmaxf(top, g_top[i][lane]);
    }
    se = 0.f;
#pragma unroll
    for (int i = 0; i < NWR; ++i) {
      const float mi = g_max[i];  // -inf: the wave's sum is 0 (or nan, which stays)
      se += g_sum[i] *
            (mi == kNegInf ? 0.f : __builtin_amdgcn_exp2f(__builtin_fmaf(mi - zm, kLog2e, -g_shift[i])));
    }
  }
  const float lse = zm + __logf(se);

  // the row's kBest best root moves: at least kBest lanes hold a move that
  // reaches theta, the smallest lane maximum (over the row's waves) within a
  // bound found by bisection over the gap to the best; the moves that reach
  // it are gathered in LDS and ranked
  const float best = wave_max_dpp(top);
  const int32_t gap = gap_of(best, top);
  int32_t bound = 0;
#pragma unroll
  for (int bit = 8; bit >= 0; --bit) {
    const int32_t c = bound | (1 << bit);
    if ((int32_t)__builtin_popcountll(__ballot(gap < c)) < kBest) bound = c;
  }
  int32_t total = INT_MAX;
  auto key_of = [&](float v, int32_t tok) { return ((uint64_t)order_key(v) << 32) | (uint32_t)~tok; };
  if (bound < kNone) {
    const float theta = -wave_max_dpp(gap <= bound ? -top : kNegInf);
    total = 0;
    bool any = false;
#pragma unroll
    for (int j = 0; j < NZ; ++j) {
      // few groups of eight hold a hit: the others are passed over
      if (j % 8 == 0) any = __ballot(group[j / 8] >= theta) != 0ull;
      if (!any) continue;
      const bool hit = used(j) && y[j] >= theta;
      const uint64_t in = __ballot(hit);
      if (in == 0ull) continue;
      const int32_t c = (int32_t)__builtin_popcountll(in);
      int32_t base = total;
      if constexpr (NWR > 1) {
        if (lane == 0)
          base = __hip_atomic_fetch_add(&g_count[0], c, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_WORKGROUP);
        base = __builtin_amdgcn_readfirstlane(base);
      }
      total += c;
      const int32_t pos = base + (int32_t)lanes_below(in);
      if (hit && pos < 64) g_key[rw][pos] = key_of(y[j], index(j));
    }
  }
  if constexpr (NWR > 1) {
    __syncthreads();
    if (bound < kNone) total = __builtin_amdgcn_readfirstlane(g_count[0]);
  }
  if (total > 64) {  // uniform over the row's waves
    // fewer than kBest lanes with a finite move, or very many equal values:
    // kBest rounds of a wave argmax over the moves after the last one taken
    if constexpr (NWR > 1) __syncthreads();  // g_key is rewritten
    float pk = 0.f;
    int32_t pt = -1;
    uint64_t mine = 0ull;
    for (int32_t i = 0; i < kBest; ++i) {
      float bk = kNegInf;
      int32_t bt = INT_MAX;
#pragma unroll
      for (int j = 0; j < NZ; ++j) {
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
    if (lane < kBest) g_key[rw][q * kBest + lane] = mine;  // 0: none
    total = NWR * kBest;
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
  const int32_t to = 4 * ((key != 0ull && rank < kBest) ? rank : 63);
  const int32_t sent = __builtin_amdgcn_ds_permute(to, klo);  // 0 where nothing was sent
  const int32_t tok = lane < kBest && sent != 0 ? ~sent : -1;
  const int32_t lo = __shfl(tok, 2 * lane, 64), hi = __shfl(tok, 2 * lane + 1, 64);
  const int32_t word = (int32_t)(((uint32_t)lo & 0xffffu) | ((uint32_t)hi << 16));
  if (lane == 0) {
    out_tok[r] = word;
    out_score[r] = lse;
  }
  if (lane == 1) out_state[r] = word;
}

// A row's summary and its step, in LDS.
struct alignas(16) RowRec {
  float y1, zb, z1, psi1;  // best root move's key, blank's logit, the move's logit and psi
  float lse;
  int32_t dst1, cls1;
  uint32_t t12;            // listed tokens (0xffff: none)
  uint32_t t34;
  int32_t tok, ns;         // the step: token, state after it
  float score;
};

struct Answer {
  int32_t tok, ns;
  float z, b;
};

// What a step reads: the stream's model (records of its first states in LDS)
// and rows.
template <class Ld>
struct Walk {
  const ArenaView& A;
  const blist::Graph& G;
  float root_phi;
  int32_t off, V;
  const typename Ld::T* col;  // row t of the stream: col + t * tstride
  int64_t tstride;
  const float* gpsi;
  const int32_t* gdst;
  uint32_t* marks;  // class bitmap of the wave
  int32_t mark_words;
};

// The step from state x on row t. NS children per lane.
template <class Ld, int NS>
__device__ __forceinline__ Answer walk_step(const Walk<Ld>& W, const RowRec& R, int32_t t, int32_t x) {
  const ArenaView& A = W.A;
  const int32_t off = W.off, V = W.V, V1 = V + 1;
  const int lane = __lane_id();
  const typename Ld::T* row = W.col + (int64_t)t * W.tstride;
  const int32_t tok1 = __builtin_amdgcn_readfirstlane((int32_t)(R.t12 & 0xffffu));
  float rk = R.y1, r_psi = R.psi1, r_z = R.z1;
  int32_t rt = tok1, r_ns = R.dst1;  // tok1 0xffff: none (rk is -inf)
  const blist::Graph::State S0 = x != 0 ? W.G.state(x) : blist::Graph::State{0, 0, 0, W.root_phi, 0.f};
  const float phi = S0.phi;
  const float zb = R.zb, bk = zb + phi;
  float ok = kNegInf, o_psi = 0.f, o_z = 0.f;
  int32_t ot = INT_MAX, o_ns = 0;
  if (x != 0) {
    int32_t fc = S0.fc, nc = S0.nc, link = S0.link;
    bool allhot = fc + nc <= W.G.nhot;
    int32_t f0 = fc, f1 = 0, f2 = 0, f3 = 0, s1 = nc, s2 = nc, s3 = nc, total = nc, levels = 1;
    bool big = false;
    while (link != 0) {
      if (levels == kLevels) {
        big = true;
        break;
      }
      const blist::Graph::State S1 = W.G.state(link);
      fc = S1.fc;
      nc = S1.nc;
      link = S1.link;
      allhot = allhot && fc + nc <= W.G.nhot;
      if (levels == 1) f1 = fc - total;
      else if (levels == 2) f2 = fc - total;
      else f3 = fc - total;
      total += nc;
      if (levels == 1) s2 = s3 = total;
      else if (levels == 2) s3 = total;
      ++levels;
    }
    const int32_t deep = levels == 1 ? 0 : (levels == 2 ? s1 : (levels == 3 ? s2 : s3));
    big = big || total > 64 * NS || deep > 64;
    bool over = false;  // the best root move's class has a child
    // the children, one per lane and register: slot q = 64 g + lane
    int32_t y[NS], lab[NS], lv[NS], tk[NS];
    float py[NS], kb[NS], zk[NS];
    if (total > 0 && !big) {
      uint2 m[NS];
      bool more = false;
#pragma unroll
      for (int g = 0; g < NS; ++g) {
        const int32_t q = 64 * g + lane;
        const bool p1 = levels > 1 && q >= s1, p2 = levels > 2 && q >= s2, p3 = levels > 3 && q >= s3;
        lv[g] = (p1 ? 1 : 0) + (p2 ? 1 : 0) + (p3 ? 1 : 0);
        y[g] = q + (p3 ? f3 : (p2 ? f2 : (p1 ? f1 : f0)));
        m[g] = make_uint2(0u, 0u);
        py[g] = 0.f;
        lab[g] = -3;
        if (64 * g < total) {
          if (allhot) W.G.child_hot(q < total ? y[g] : 1, m[g], py[g]);
          else if (q < total) W.G.child(y[g], m[g], py[g]);
        }
      }
#pragma unroll
      for (int g = 0; g < NS; ++g) {
        if (64 * g + lane < total) {
          more = more || arc_more(m[g]);
          lab[g] = arc_class(m[g]);
        }
      }
      big = __ballot(more) != 0ull;
      if (!big) {
        bool hit = false;
#pragma unroll
        for (int g = 0; g < NS; ++g) {
          kb[g] = kNegInf;
          tk[g] = INT_MAX;
          zk[g] = 0.f;
          if (64 * g + lane < total) {
            const int32_t t0 = (int32_t)(m[g].x & 0xffffu), t1 = (int32_t)(m[g].x >> 16);
            const int32_t t2 = (int32_t)(m[g].y & 0xffffu);
            const float z0 = Ld::get(row, t0), z1 = Ld::get(row, t1), z2 = Ld::get(row, t2);
            const float k0 = z0 + py[g], k1 = z1 + py[g], k2 = z2 + py[g];
            // members ascend: ties keep the lower; a nan is passed over
            if (k0 > kb[g]) { kb[g] = k0; tk[g] = t0; zk[g] = z0; }
            if (k1 > kb[g]) { kb[g] = k1; tk[g] = t1; zk[g] = z1; }
            if (k2 > kb[g]) { kb[g] = k2; tk[g] = t2; zk[g] = z2; }
          }
          hit = hit || lab[g] == R.cls1;
        }
        over = __ballot(hit) != 0ull;
        // A child whose class a deeper chain state also has is dropped. Both
        // have the same tokens, so the best of all children is the answer
        // unless it is such a child, which is tested on the winner alone.
        uint32_t drop = 0u;
        for (;;) {
          float bv = kNegInf;
          int32_t bt = INT_MAX, bg = 0;
#pragma unroll
          for (int g = 0; g < NS; ++g)
            if (!((drop >> g) & 1u) && better(kb[g], tk[g], bv, bt)) {
              bv = kb[g];
              bt = tk[g];
              bg = g;
            }
          const int32_t wl = wave_argmax_dpp(bv, bt, ok, ot);
          const int32_t wg = rl(bg, wl);
          int32_t w_lab = 0, w_lv = 0;
#pragma unroll
          for (int g = 0; g < NS; ++g)
            if (wg == g) {
              w_lab = rl(lab[g], wl);
              w_lv = rl(lv[g], wl);
              o_ns = rl(y[g], wl);
              o_psi = rlf(py[g], wl);
              o_z = rlf(zk[g], wl);
            }
          if (levels == 1 || ot == INT_MAX) break;
          bool sh = false;
#pragma unroll
          for (int g = 0; g < NS; ++g) sh = sh || (lab[g] == w_lab && lv[g] < w_lv);
          if (__ballot(sh) == 0ull) break;
          // drop every child of this class but the deepest
          int32_t dl = INT_MAX;
#pragma unroll
          for (int g = 0; g < NS; ++g)
            if (lab[g] == w_lab) dl = min(dl, lv[g]);
          dl = wave_min_i32_dpp(dl);
#pragma unroll
          for (int g = 0; g < NS; ++g)
            if (lab[g] == w_lab && lv[g] != dl) drop |= 1u << g;
        }
      }
    }
    // level by level with the class bitmap: longer chains, more children,
    // classes of more than three members
    if (big) {
      for (int32_t i = lane; i < W.mark_words; i += 64) W.marks[i] = 0u;
      asm volatile("" ::: "memory");
      float bv = kNegInf, bpsi = 0.f, bz = 0.f;
      int32_t bt = INT_MAX, bns = 0;
      for (int32_t s = x; s != 0; s = sload(A.link + off + s)) {
        const int32_t c0 = sload(A.first_child + off + s), cn = sload(A.n_child + off + s);
        for (int32_t j = lane; j < cn; j += 64) {
          const int32_t yy = c0 + j;
          const uint32_t* p = A.arc_mem + 2 * ((int64_t)off + yy);
          const uint2 m = make_uint2(gload(p), gload(p + 1));
          const float ps = gload(A.psi + off + yy);
          const int32_t c = arc_class(m);
          if ((W.marks[c >> 5] >> (c & 31)) & 1u) continue;  // a deeper state's child has it
          auto offer = [&](int32_t v) {
            const float z = Ld::get(row, v);
            if (better(z + ps, v, bv, bt)) {
              bv = z + ps;
              bt = v;
              bns = yy;
              bpsi = ps;
              bz = z;
            }
          };
          if (!arc_more(m)) {
            offer((int32_t)(m.x & 0xffffu));
            offer((int32_t)(m.x >> 16));
            offer((int32_t)(m.y & 0xffffu));
          } else {
            for (int32_t e = gload(A.cls_ptr + c); e < gload(A.cls_ptr + c + 1); ++e)
              offer(gload(A.cls_tok + e));
          }
        }
        asm volatile("" ::: "memory");
        for (int32_t j = lane; j < cn; j += 64) {
          const int32_t c = gload(A.label + off + c0 + j);
          __hip_atomic_fetch_or(W.marks + (c >> 5), 1u << (c & 31), __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        asm volatile("" ::: "memory");
      }
      const int32_t wl = wave_argmax_dpp(bv, bt, ok, ot);
      o_ns = rl(bns, wl);
      o_psi = rlf(bpsi, wl);
      o_z = rlf(bz, wl);
      const int32_t c1 = R.cls1;
      over = __builtin_amdgcn_readfirstlane(
                 (int32_t)(c1 >= 0 && ((W.marks[c1 >> 5] >> (c1 & 31)) & 1u))) != 0;
    }
    // the best root move is overridden: none of the others exceeds it, so they
    // matter only when neither the best child nor the blank is above it
    if (__builtin_amdgcn_readfirstlane((int32_t)(over && !(ok > rk || bk > rk)))) {
      rk = kNegInf;
      // the listed moves after the first, lane by lane
      const int32_t lt = (int32_t)((lane < 2 ? R.t12 >> (16 * lane) : R.t34 >> (16 * (lane & 1))) & 0xffffu);
      const bool in = lane < kBest && lt < V;
      int32_t lc = -2, ld = 0;
      float lz = 0.f, lp = 0.f;
      if (in) {
        lc = A.class_map[lt];
        ld = W.gdst[lt];
        lz = Ld::get(row, lt);
        lp = W.gpsi[lt];
      }
      bool free_ = in;
      if (big) {
        if (in && lc >= 0) free_ = !((W.marks[lc >> 5] >> (lc & 31)) & 1u);
      } else {
#pragma unroll
        for (int i = 0; i < kBest; ++i) {
          const int32_t ci = rl(lc, i);
          bool h = false;
#pragma unroll
          for (int g = 0; g < NS; ++g) h = h || lab[g] == ci;
          if (__ballot(h) != 0ull && lane == i) free_ = false;
        }
      }
      const uint64_t fm = __ballot(free_), im = __ballot(in);
      if (fm != 0ull) {
        const int32_t i = (int32_t)__builtin_ctzll(fm);
        rt = rl(lt, i);
        r_ns = rl(ld, i);
        r_z = rlf(lz, i);
        r_psi = rlf(lp, i);
        rk = r_z + r_psi;
      } else if ((im >> (kBest - 1)) & 1ull) {
        // all listed moves are overridden: the rest of the row
        if (!big) {
          for (int32_t i = lane; i < W.mark_words; i += 64) W.marks[i] = 0u;
          asm volatile("" ::: "memory");
#pragma unroll
          for (int g = 0; g < NS; ++g)
            if (lab[g] >= 0)
              __hip_atomic_fetch_or(W.marks + (lab[g] >> 5), 1u << (lab[g] & 31), __ATOMIC_RELAXED,
                                    __HIP_MEMORY_SCOPE_WORKGROUP);
          asm volatile("" ::: "memory");
        }
        float bv = kNegInf;
        int32_t bt = INT_MAX;
        constexpr int SC = 16;  // chunks whose loads are in flight together
        for (int32_t v0 = 0; v0 < V; v0 += 64 * SC) {
          float kc[SC];
          int32_t cc[SC];
#pragma unroll
          for (int q = 0; q < SC; ++q) {
            const int32_t v = min(v0 + 64 * q + lane, V);
            kc[q] = Ld::get(row, v) + gload(W.gpsi + v);
            cc[q] = gload(A.class_map + v);
          }
#pragma unroll
          for (int q = 0; q < SC; ++q) {
            const int32_t v = v0 + 64 * q + lane, c = cc[q];
            if (v < V && kc[q] > bv && !(c >= 0 && ((W.marks[c >> 5] >> (c & 31)) & 1u))) {
              bv = kc[q];  // v ascends: ties keep the lower
              bt = v;
            }
          }
        }
        wave_argmax_dpp(bv, bt, rk, rt);
        const int32_t rv = rt < V ? rt : 0;
        r_ns = gload(W.gdst + rv);
        r_psi = gload(W.gpsi + rv);
        r_z = Ld::get(row, rv);
      }
    }
  }
  Answer a;
  a.tok = V;
  a.ns = x;
  a.z = zb;
  a.b = 0.f;
  float k = bk > kNegInf ? bk : kNegInf;  // the blank keeps the state (a nan never wins)
  int32_t v = V;
  if (better(ok, ot, k, v)) {
    k = ok;
    v = ot;
    a.tok = ot;
    a.ns = o_ns;
    a.z = o_z;
    a.b = o_psi - phi;
  }
  if (better(rk, rt, k, v)) {
    a.tok = rt;
    a.ns = r_ns;
    a.z = r_z;
    a.b = r_psi - phi;
    k = rk;
  }
  if (__builtin_amdgcn_readfirstlane((int32_t)(k == kNegInf))) {
    // no key is above -inf: the lowest that is no nan (the first token when all
    // are), at its own move
    int32_t v0 = V1;
    for (int32_t i = 0; i < V1 && v0 == V1; i += 64) {
      const bool in = i + lane < V1;
      const float zi = Ld::get(row, in ? i + lane : 0);
      const uint64_t is = __ballot(in && zi == zi);
      if (is != 0ull) v0 = i + (int32_t)__builtin_ctzll(is);
    }
    if (v0 == V) {
      a.tok = V;
      a.ns = x;
      a.z = zb;
      a.b = 0.f;
      return a;
    }
    if (v0 == V1) v0 = 0;
    const int32_t c = sload(A.class_map + v0);
    int32_t ns = sload(W.gdst + v0);
    bool found = false;
    for (int32_t s = x; s != 0 && c >= 0 && !found; s = sload(A.link + off + s)) {
      const int32_t c0 = sload(A.first_child + off + s), cn = sload(A.n_child + off + s);
      for (int32_t j0 = 0; j0 < cn && !found; j0 += 64) {
        const uint64_t at = __ballot(j0 + lane < cn && gload(A.label + off + c0 + min(j0 + lane, cn - 1)) == c);
        found = at != 0ull;
        if (found) ns = c0 + j0 + (int32_t)__builtin_ctzll(at);
      }
    }
    a.tok = v0;
    a.ns = ns;
    a.z = Ld::get(row, v0);
    a.b = sload(A.psi + off + ns) - phi;
  }
  return a;
}

template <class Ld, int NS>
__global__ __launch_bounds__(kWalkThreads) void greedy_walk_kernel(
    ArenaView A, const typename Ld::T* __restrict__ logits, int32_t T, int32_t B, int64_t stride,
    int32_t L, const int32_t* __restrict__ model_ids, int32_t* __restrict__ states,
    int32_t* __restrict__ out_tok, int32_t* __restrict__ out_state,
    float* __restrict__ out_score, int32_t mark_words, int32_t hot_states, int32_t lds_bytes) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  __shared__ int32_t fin[kWalkThreads / 64];
  __shared__ float vpsi[256], vphi[256];
  lds_poison(dyn, lds_bytes);
  lds_poison(fin, sizeof(fin));
  const int32_t V1 = A.V1, V = V1 - 1;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = __lane_id();
  const int32_t b = blockIdx.x;
  RowRec* rec = reinterpret_cast<RowRec*>(dyn);
  const int32_t m = model_ids[b];
  const int32_t s0 = states[b];
  int32_t off = 0, n = 0;
  const int mode = resolve_stream(A, m, s0, off, n);
  const bool biased = mode == 1;
  const int32_t fixed = unbiased_state(mode, s0 == TB_STATE_TIMEOUT);
  const typename Ld::T* col = logits + (int64_t)b * stride;
  const int64_t tstride = (int64_t)B * stride;
  const float* gpsi = A.root_psi + (int64_t)(biased ? m : 0) * V1;
  const int32_t* gdst = A.root_dst + (int64_t)(biased ? m : 0) * V1;

  // ---- the summaries, one row per thread
  for (int32_t t = threadIdx.x; t < T; t += blockDim.x) {
    const int64_t o = (int64_t)t * B + b;
    const typename Ld::T* row = col + (int64_t)t * tstride;
    RowRec r;
    r.t12 = (uint32_t)out_tok[o];
    r.t34 = (uint32_t)out_state[o];
    r.lse = out_score[o];
    const int32_t t1 = (int32_t)(r.t12 & 0xffffu);
    r.zb = Ld::get(row, V);
    r.y1 = kNegInf;
    r.z1 = r.psi1 = 0.f;
    r.dst1 = biased ? 0 : fixed;
    r.cls1 = -1;
    if (t1 < V) {
      r.z1 = Ld::get(row, t1);
      if (biased) {
        r.psi1 = gpsi[t1];
        r.dst1 = gdst[t1];
        r.cls1 = A.class_map[t1];
      }
      r.y1 = r.z1 + r.psi1;
    }
    if (!biased) {  // the best of the tokens and the blank
      int32_t v = better(r.zb, V, r.y1, t1) ? V : t1;
      float z = v == V ? r.zb : r.z1;
      if (!(r.y1 > kNegInf || r.zb > kNegInf)) {  // as walk_step
        for (v = 0; v < V && Ld::get(row, v) != Ld::get(row, v); ++v) {}
        if (v == V && r.zb != r.zb) v = 0;  // nothing but nan
        z = Ld::get(row, v);
      }
      out_tok[o] = v;
      out_state[o] = fixed;
      out_score[o] = z - r.lse;
    }
    r.tok = 0;
    r.ns = 0;
    r.score = 0.f;
    rec[t] = r;
  }
  if (!biased) {  // uniform over the workgroup
    if (threadIdx.x == 0) states[b] = fixed;
    return;
  }
  // ---- records of the model's first states
  uint4* hot = reinterpret_cast<uint4*>(rec + T);
  int32_t nhot = n < hot_states ? n : hot_states;
  bool unusable = false;
  for (int32_t i = threadIdx.x; i < nhot; i += blockDim.x) {
    const bool ok = blist::hot_record(A, (int64_t)off + i, hot[i]);
    unusable = unusable || (i > 0 && !ok);
  }
  for (int32_t i = threadIdx.x; i < (nhot > 0 ? 512 : 0); i += blockDim.x)
    (i < 256 ? vpsi[i] : vphi[i - 256]) = A.value_tab[512 * (int64_t)m + i];
  if (__syncthreads_or(unusable)) nhot = 0;

  // ---- segments
  const blist::Graph G{A, off, nhot, hot, vpsi, vphi};
  const Walk<Ld> W{A, G, sload(A.phi + off), off, V, col, tstride, gpsi, gdst,
                   reinterpret_cast<uint32_t*>(hot + hot_states) + w * mark_words, mark_words};
  const int32_t t0 = w * L, t1 = min(t0 + L, T);
  int32_t s = w == 0 ? s0 : 0, assumed = s;
  auto step = [&](int32_t t, bool keep) {
    const Answer a = walk_step<Ld, NS>(W, rec[t], t, s);
    if (keep && lane == 0) {
      rec[t].tok = a.tok;
      rec[t].ns = a.ns;
      rec[t].score = (a.z - rec[t].lse) + a.b;
    }
    s = __builtin_amdgcn_readfirstlane(a.ns);
  };
  if (t0 < t1) {
    const int32_t tw = w == 0 ? t0 : max(t0 - kWarm, 0);
    // a warm-up that reaches the call's first row starts exactly
    if (w > 0 && tw == 0) s = s0;
    for (int32_t t = tw; t < t1; ++t) {
      if (t == t0) assumed = s;
      step(t, t >= t0);
    }
  }
  if (lane == 0) fin[w] = s;
  // ---- rounds: a segment whose start is not the previous segment's end is
  // walked again from there until it meets its stored states. After round i
  // the first i + 1 segments are exact, so the rounds end.
  for (;;) {
    __syncthreads();
    const int32_t from = w > 0 ? __builtin_amdgcn_readfirstlane(fin[w - 1]) : s0;
    const bool redo = t0 < t1 && from != assumed;
    if (!__syncthreads_or(redo)) break;
    if (redo) {
      assumed = from;
      s = from;
      bool met = false;
      for (int32_t t = t0; t < t1 && !met; ++t) {
        const int32_t old = __builtin_amdgcn_readfirstlane(rec[t].ns);
        step(t, true);
        met = s == old;
      }
      if (!met && lane == 0) fin[w] = s;
    }
  }
  // ---- outputs
  for (int32_t t = threadIdx.x; t < T; t += blockDim.x) {
    const int64_t o = (int64_t)t * B + b;
    out_tok[o] = rec[t].tok;
    out_state[o] = rec[t].ns;
    out_score[o] = rec[t].score;
  }
  if (threadIdx.x == 0) states[b] = rec[T - 1].ns;
}

// ---- launch

typedef hipError_t (*Launch)(const ArenaView&, const void*, int32_t, int32_t, int64_t,
                             const int32_t*, int32_t*, int32_t*, int32_t*, float*, hipStream_t);
Launch launcher_f32(int32_t V1);
Launch launcher_bf16(int32_t V1);

constexpr int kLdsBytes = 152 * 1024;
// Steps of a call from which the records are worth their filling: with / without
// them calls of 6, 8, 12 and 16 steps take 32 / 30, 34 / 34, 45 / 46 and 51 / 53 us (128
// streams, 4097 float32), 45 / 41, 48 / 47, 61 / 61 and 70 / 72 (256 streams, 8193
// bfloat16); 64 steps 81 / 84 and 154 / 156.
constexpr int kHotSteps = 12;

template <class Ld, int NWR, int NP, int NC>
hipError_t launch_t(const ArenaView& A, const void* logits, int32_t T, int32_t B, int64_t stride,
                    const int32_t* model_ids, int32_t* states, int32_t* out_tok,
                    int32_t* out_state, float* out_score, hipStream_t st) {
  typedef typename Ld::T LT;
  const LT* z = static_cast<const LT*>(logits);
  // rows [r0, n_rows) in launches of as many workgroups as one may have
  const int64_t n_rows = (int64_t)T * B;
  constexpr int64_t kPer = (kRowThreads / 64) / NWR, kMost = kPer * most_groups(kRowThreads);
  for (int64_t r0 = 0; r0 < n_rows; r0 += kMost) {
    const int64_t nr = n_rows - r0 < kMost ? n_rows - r0 : kMost;
    hipLaunchKernelGGL((greedy_rows_kernel<Ld, NWR, NP, NC>),
                       dim3((uint32_t)((nr + kPer - 1) / kPer)), dim3(kRowThreads), 0, st, A, z, r0,
                       n_rows, B, stride, model_ids, states, out_tok, out_state, out_score);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  // The walk: pieces of as many steps as LDS holds records for, one segment
  // per wave.
  constexpr int kWaves = kWalkThreads / 64;
  const int32_t words = (A.V1 + 31) / 32;
  const int32_t most = (kLdsBytes - 4 * kWaves * words) / (int32_t)sizeof(RowRec);
  auto kernel = &greedy_walk_kernel<Ld, 4>;
  allow_dynamic_lds(kernel, (size_t)kLdsBytes);
  for (int32_t t = 0; t < T; t += most) {
    const int32_t n = T - t < most ? T - t : most;
    const int32_t L = (n + kWaves - 1) / kWaves, waves = (n + L - 1) / L;
    const int32_t room = kLdsBytes - n * (int32_t)sizeof(RowRec) - 4 * waves * words;
    int32_t hot = n >= kHotSteps ? (room / 16 < 8192 ? room / 16 : 8192) : 0;
    if (hot > A.n_states) hot = (int32_t)A.n_states;
    const int32_t lds = kLdsBytes - room + 16 * hot;
    // streams [b0, B) in launches of as many workgroups as one may have
    const int64_t group = most_groups(64 * waves);
    for (int64_t b0 = 0; b0 < B; b0 += group) {
      const int64_t nb = B - b0 < group ? B - b0 : group, o = (int64_t)t * B + b0;
      hipLaunchKernelGGL(kernel, dim3((uint32_t)nb), dim3(64 * waves), (size_t)lds, st, A,
                         z + o * stride, n, B, stride, L, model_ids + b0, states + b0, out_tok + o,
                         out_state + o, out_score + o, words, hot, lds);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

// The instance for rows of V1 values: as many 16-byte pieces as lie before the
// blank, chunks for the rest. A piece is 1024 values of four waves in float32,
// 2048 in bfloat16; above 8 (4) pieces the instances double.
template <class Ld>
Launch launcher_t(int32_t V1) {
  constexpr int PV = 16 / sizeof(typename Ld::T), P = 256 * PV;
  const int32_t np = (V1 - 1) / P;
  if constexpr (PV == 4) {
    if (np <= 2) return launch_t<Ld, 4, 2, 4>;
    if (np == 3) return launch_t<Ld, 4, 3, 4>;
    if (np == 4) return launch_t<Ld, 4, 4, 4>;
    if (np == 5) return launch_t<Ld, 4, 5, 4>;
    if (np <= 7) return launch_t<Ld, 4, 6, 8>;
    if (np <= 9) return launch_t<Ld, 4, 8, 8>;
    if (np <= 15) return launch_t<Ld, 4, 10, 24>;
    return launch_t<Ld, 4, 16, 64>;
  } else {
    if (np <= 1) return launch_t<Ld, 4, 1, 8>;
    if (np == 2) return launch_t<Ld, 4, 2, 8>;
    if (np == 3) return launch_t<Ld, 4, 3, 8>;
    if (np == 4) return launch_t<Ld, 4, 4, 8>;
    if (np <= 7) return launch_t<Ld, 4, 5, 24>;
    return launch_t<Ld, 4, 8, 64>;
  }
}

}  // namespace glist
}  // namespace tbias
