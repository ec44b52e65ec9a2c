// Boosted beam step from row summaries, for every row width and beam: a
// row-preparation kernel over all rows of the call (beam_rows.hpp), then one
// workgroup per stream that carries the beam through the steps (templates;
// instantiated in beam_list_*.hip).
//
// What bounds a beam call is the chain of its steps: a stream's step t needs
// the hypotheses that step t-1 kept, so a call takes T times the latency of
// one step, on as many CUs as there are streams. Everything that does not
// depend on the hypotheses is therefore taken out of the chain: slot k reads
// row [t, b, k] whatever was kept, so the row's normaliser and its kList best
// root moves are known before the step (the row summary), and the step
// gathers only
//
//  * the listed root moves (their logit, psi, class and target are loaded a
//    step ahead),
//  * the children along the suffix chain of the slot's state (one per lane),
//  * the blank,
//
// instead of scoring K*(V+1) candidates: a step is some 10 thousand cycles
// (8 hypotheses, 1024 tokens: 4.1 us against 7.0 us when every wave scored its
// whole row; 32 hypotheses: 11 us against 920 us for the reference kernel, which
// took beams above 8 before; 4 hypotheses of 8192 tokens: 8 us against 26 us
// with the rows summarised inside the step). Per step, wave w (slots w and, for
// more than 16 hypotheses, w + 16):
//
//  1. candidates of its slots: c = (S - lse) - phi(s), then c + (z + psi) of
//     the chain's children (deeper states first: a child whose class a deeper
//     chain state also has is dropped) and of the listed root moves whose
//     class no child has, and the blank c + (z[V] + phi(s)). The values of
//     the listed moves and of the blank are posted to the other waves; a listed
//     token whose class a child has is posted with that child's value.
//  2. a bound that at least K posted candidates reach (every wave finds the
//     same one by bisection over the gap to the best posted candidate,
//     rounded to 4 bits of mantissa: 9 ballots per posted register). The
//     candidates of the wave that reach it go to a shared list. A row whose
//     last listed move reaches it may hold further moves that do: the wave
//     scans that row (mostly the call's first step, where one slot is alone).
//  3. every wave ranks the shared list (about 1.5 K entries) in (value,
//     slot, token) order and holds slot j's new hypothesis in lane j, so the
//     hypotheses are replicated and two barriers a step are enough.
//
// When the posted candidates are fewer than K, the rows are searched for such
// a bound; when there is none (fewer than K finite candidates), or more than
// kCap candidates reach it, K rounds of an argmax over every candidate take
// the K best one after the other. All paths order candidates by (value, flat
// index), so the result does not depend on the path.
//
// Rows: in LDS (ROWS, copied a step ahead) when the K rows fit beside the
// model's records, else gathered from memory. States: 16-byte records of the
// model's first states in LDS (built from state_rec and arc_mem), the others
// from the arena. A call of a few steps does not fill them.
#pragma once

#include <climits>

#include "device.hpp"
#include "launch.hpp"
#include "ref_table.hpp"

namespace tbias {

// Carry of the streaming beam (tb_boost_step_beam_stream); unused otherwise.
struct StreamArgs {
  tb_hyp* hyps = nullptr;   // [B*K]
  int32_t* tree = nullptr;  // [B*cap*2] (label, parent record)
  int32_t cap = 0;
  int32_t* tree_len = nullptr;  // [B]
  int32_t recombine = 0;
};

namespace blist {

constexpr int kList = 8;     // best root moves listed per row
constexpr int kCap = 256;    // candidates ranked in one step
constexpr int kNone = 511;   // quantised gap of a candidate that reaches no bound
constexpr uint32_t kNoTok = 0xffffu;
constexpr float kNegInf = -__builtin_huge_valf();

// Float order as unsigned integers (larger float, larger key; both zeros alike).
__device__ __forceinline__ uint32_t order_key(float x) {
  const uint32_t u = __float_as_uint(x + 0.0f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_order_key(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// The gap best - v of a candidate, rounded down to 4 bits of mantissa: 0 for
// gaps below 2^-12 (and above the best), kNone from 2^19.9 on and for -inf.
__device__ __forceinline__ int32_t gap_of(float best, float v) {
  const int32_t q = (__float_as_int(best - v) >> 19) - ((127 - 12) << 4);
  return v > kNegInf ? min(max(q, 0), kNone) : kNone;
}

// log(exp(a) + exp(b)) of two finite float32 values, in float64, rounded once.
__device__ __forceinline__ float logaddexp32(float a, float b) {
  const double hi = (double)(a > b ? a : b), lo = (double)(a > b ? b : a);
  return (float)(hi + log1p(exp(lo - hi)));
}

template <class T>
__device__ __forceinline__ T sload(const T* p) {  // uniform address, scalar cache
  return *(const __attribute__((address_space(4))) T*)(p);
}
// A read through an explicitly global pointer: keeps the compiler from merging
// it with an LDS read of another branch into one generic (flat) load.
template <class T>
__device__ __forceinline__ T gload(const T* p) {
  return *(const __attribute__((address_space(1))) T*)(p);
}
// A uniform value the compiler cannot follow: what is compared with it is
// compared where it is used, instead of one mask per chunk kept in scalar
// registers across the step loop.
__device__ __forceinline__ int32_t opaque(int32_t x) {
  asm volatile("" : "+s"(x));
  return x;
}
__device__ __forceinline__ int32_t rl(int32_t v, int32_t lane) {
  return __builtin_amdgcn_readlane(v, lane);
}
__device__ __forceinline__ float rlf(float v, int32_t lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// ---- LDS layout (dynamic): offsets in bytes from the start.
struct Layout {
  int32_t rows, row_stride;  // K rows of the logits' type, in bytes (ROWS)
  int32_t marks, mark_words; // class bitmap per slot
  int32_t hot, nhot;         // 16-byte records of the first nhot states
  int32_t total;
};

struct Cand {
  uint32_t code;  // ~(slot << 16 | token)
  uint32_t okey;
  int32_t dst;
  float step;
};

template <int MAXK, int NW>
struct alignas(16) Shared {
  Cand cand[kCap];
  float listed[9 * MAXK];  // posted values: kList moves and the blank of every slot
  float c[MAXK], psi[MAXK], a[MAXK];  // streaming beam
  float red_v[2][NW], red_step[2][NW];
  int32_t red_code[2][NW], red_dst[2][NW];
  int32_t bound[MAXK];
  float best;
  int32_t first_bound;
  int32_t count[2];
  int32_t rank[2][64];
  float opsi[NW][kList];  // psi of the children that override listed moves (large sets)
  float vpsi[256], vphi[256];
};

// A non-root state's record: from LDS (x < nhot) or the arena. The LDS records
// are all usable: a model with a record whose fields do not fit (the flag of
// state_rec, the root's aside) runs with nhot = 0.
struct Graph {
  const ArenaView& A;
  int32_t off, nhot;
  const uint4* hot;
  const float* vpsi;
  const float* vphi;

  struct State {
    int32_t fc, nc, link;
    float phi, psi;
  };
  __device__ __forceinline__ State state(int32_t x) const {  // x uniform, not the root
    State r;
    if (x < nhot) {
      const uint2 h = *reinterpret_cast<const uint2*>(hot + x);
      const uint32_t a = __builtin_amdgcn_readfirstlane(h.x);
      const uint32_t b = __builtin_amdgcn_readfirstlane(h.y);
      r.fc = (int32_t)(a & 0xffffu);
      r.nc = (int32_t)((a >> 16) & 0xffu);
      r.link = (int32_t)(b & 0xffffu);
      r.phi = vphi[(b >> 16) & 0xffu];
      r.psi = vpsi[a >> 24];
    } else {
      r.fc = sload(A.first_child + off + x);
      r.nc = sload(A.n_child + off + x);
      r.link = sload(A.link + off + x);
      r.phi = sload(A.phi + off + x);
      r.psi = sload(A.psi + off + x);
    }
    return r;
  }
  // arc record (as arc_mem) and psi of child y of this lane
  __device__ __forceinline__ void child_hot(int32_t y, uint2& m, float& psi) const {
    const uint4 h = hot[y];
    m = make_uint2(h.z, h.w);
    psi = vpsi[h.x >> 24];
  }
  __device__ __forceinline__ void child(int32_t y, uint2& m, float& psi) const {
    if (y < nhot) {
      child_hot(y, m, psi);
    } else {
      const uint32_t* p = A.arc_mem + 2 * ((int64_t)off + y);
      m = make_uint2(gload(p), gload(p + 1));
      psi = gload(A.psi + off + y);
    }
  }
};
__device__ __forceinline__ int32_t arc_class(uint2 m) { return (int32_t)((m.y >> 16) & 0x7fffu); }
__device__ __forceinline__ bool arc_more(uint2 m) { return (m.y >> 31) != 0u; }

// The 16-byte LDS record of global state x: first child | child count << 16 |
// psi index << 24, link | phi index << 16, the arc record. False when a field
// does not fit.
__device__ __forceinline__ bool hot_record(const ArenaView& A, int64_t x, uint4& out) {
  const uint32_t* r = A.state_rec + 3 * x;
  const uint32_t* q = A.arc_mem + 2 * x;
  const uint32_t r2 = r[2];
  out = make_uint4(r[0], (r[1] & 0xffffu) | (((r2 >> 8) & 0xffu) << 16), q[0], q[1]);
  return (r2 >> 31) == 0u;
}

constexpr int kLevels = 4;  // chain states whose children are taken one per lane

// What a wave holds of one of its slots during a step.
template <int NS>
struct Slot {
  // row summary of the step and of the next one, by lane: lanes 0..kList-1
  // the listed moves, lane kList the blank
  int32_t tok, cls, dst;
  float rpsi, z, lse;
  uint32_t word;                 // summary word of the step after
  int32_t n_tok, n_cls, n_dst;   // the next step's
  float n_rpsi, n_z, n_lse;
  // the step's hypothesis
  int32_t s;
  float c, phi, psi;
  // chain children, NS per lane (unless big)
  bool big;  // more than 64 * NS children or kLevels levels, or a class of more than 3 members
  int32_t n;  // children held over the lanes
  int32_t y[NS];
  uint2 m[NS];
  float py[NS], z0[NS], z1[NS], z2[NS];
  uint32_t on;  // bit 3 * i + q: member q of the lane's child i is a candidate
  float top;    // largest value of the lane's children (shadowed ones included)
  float lv;     // value of this lane's listed move or blank
};

// Sixteen bytes of a logit row, at the alignment of its elements.
template <class T>
struct __attribute__((packed, aligned(sizeof(T)))) Quad {
  uint32_t w[4];
};

template <class Ld, int NW, int KPW, int NS, bool STREAM, bool ROWS>
__global__ __launch_bounds__(64 * NW) void beam_list_kernel(
    ArenaView A, const typename Ld::T* __restrict__ logits, int32_t T, int32_t B, int32_t K,
    int64_t stride, const int32_t* __restrict__ model_ids, int32_t* __restrict__ states,
    float* __restrict__ scores, int32_t* __restrict__ out_tok, int32_t* __restrict__ out_parent,
    int32_t* __restrict__ out_state, float* __restrict__ out_step, float* __restrict__ out_cum,
    StreamArgs sa, Layout lay) {
  constexpr int MAXK = NW * KPW;
  constexpr int NV = (9 * MAXK + 63) / 64;  // posted values per lane
  typedef typename Ld::T LT;
  constexpr int QV = 16 / sizeof(LT);       // values in 16 bytes
  constexpr int RC = 2048 / (64 * QV);      // 16-byte pieces of a row a lane carries to LDS (ROWS)
  __shared__ Shared<MAXK, NW> S;
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  lds_poison(&S, sizeof(S));
  lds_poison(dyn, lay.total);
  const int32_t V1 = A.V1, V = V1 - 1;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = __lane_id();
  const int32_t b = blockIdx.x;

  // ---- the carry: every wave holds hypothesis j in lane j
  const int32_t m = model_ids[b];
  int mode = (m == -1) ? 0 : ((m < -1 || m >= A.n_models) ? -1 : 1);
  int32_t off = 0, n = 0;
  if (mode == 1) {
    off = A.model_off[m];
    n = A.model_n[m];
  }
  const bool has = lane < K;
  int32_t hs = has ? states[(int64_t)b * K + lane] : 0;
  float hS = has ? scores[(int64_t)b * K + lane] : kNegInf;
  if (mode == 1 && __ballot(has && (hs < 0 || hs >= n)) != 0ull) mode = -1;
  const bool tmo = __ballot(has && hs == TB_STATE_TIMEOUT) != 0ull;
  const bool biased = mode == 1;
  const int32_t fixed = unbiased_state(mode, tmo);
  if (!biased) hs = fixed;
  uint64_t hh = 0ull, hp = 0ull;
  int32_t hl = -1, hn = -1, tlen = 0;
  if constexpr (STREAM) {
    if (has) {
      const tb_hyp y = sa.hyps[(int64_t)b * K + lane];
      hh = y.hash;
      hp = y.prefix_hash;
      hl = y.last;
      hn = y.node;
    }
    const int32_t l = sa.tree_len[b];  // clamped: records are only written at [0, cap)
    tlen = l < 0 ? 0 : (l > sa.cap ? sa.cap : l);
  }

  // ---- tables
  uint4* hot = reinterpret_cast<uint4*>(dyn + lay.hot);
  int32_t nhot = biased ? (n < lay.nhot ? n : lay.nhot) : 0;
  bool unusable = false;
  for (int32_t i = threadIdx.x; i < nhot; i += 64 * NW) {
    const bool ok = hot_record(A, (int64_t)off + i, hot[i]);
    unusable = unusable || (i > 0 && !ok);
  }
  if (nhot > 0) {
    const float* vt = A.value_tab + 512 * (int64_t)m;
    for (int32_t i = threadIdx.x; i < 512; i += 64 * NW)
      (i < 256 ? S.vpsi[i] : S.vphi[i - 256]) = vt[i];
  }
  if (threadIdx.x < 2) S.count[threadIdx.x] = 0;
  if (threadIdx.x < 128) S.rank[threadIdx.x >> 6][threadIdx.x & 63] = 0;
  if (nhot > 0 && __syncthreads_or(unusable)) nhot = 0;  // nhot is uniform
  const Graph G{A, off, nhot, hot, S.vpsi, S.vphi};
  float root_phi = 0.f, root_psi = 0.f;
  if (biased) {
    root_phi = sload(A.phi + off);
    root_psi = sload(A.psi + off);
  }
  const float* gpsi = A.root_psi + (int64_t)(biased ? m : 0) * V1;
  const int32_t* gdst = A.root_dst + (int64_t)(biased ? m : 0) * V1;

  // ---- row summaries: lane i < kList reads the word of token i, lane kList
  // the normaliser
  const int64_t ostride = (int64_t)B * K;
  const int64_t tstride = ostride * stride;
  const int32_t* word_base =
      lane < 2 ? out_tok
               : (lane < 4 ? out_parent
                           : (lane < 6 ? out_state
                                       : reinterpret_cast<const int32_t*>(lane < 8 ? out_cum : out_step)));
  auto slot_id = [&](int i) { return w + i * NW; };
  const LT* row_p[KPW];        // the slot's row of the current step
  const int32_t* word_p[KPW];  // this lane's summary word two steps ahead
  auto load_word = [&](Slot<NS>& h, int i) {
    if (lane <= kList) h.word = (uint32_t)*word_p[i];
    word_p[i] += ostride;
  };
  // the next step's listed moves from their summary word; row: the next step's
  auto gather = [&](Slot<NS>& h, const LT* row) {
    h.n_lse = rlf(__uint_as_float(h.word), kList);
    int32_t tk = (int32_t)((h.word >> (16 * (lane & 1))) & 0xffffu);
    if (lane == kList) tk = V;
    const bool in = lane <= kList && tk < V1;
    h.n_tok = in ? tk : -1;
    h.n_cls = -2;
    h.n_dst = fixed;
    h.n_rpsi = 0.f;
    h.n_z = kNegInf;
    if (in) {
      if (biased) {
        h.n_rpsi = gpsi[tk];
        h.n_dst = gdst[tk];
        h.n_cls = A.class_map[tk];
      }
      if (!ROWS) h.n_z = Ld::get(row, tk);
    }
  };
  LT* lrow[KPW];
  // this wave's next row (ROWS implies one slot per wave): full pieces of 64 *
  // QV values, then its last values one by one
  Quad<LT> pre[ROWS ? RC : 1];
  LT tail[ROWS ? QV : 1];
  const int32_t n_full = V1 / (64 * QV), n_tail = V1 - n_full * 64 * QV;
  auto load_rows = [&](const LT* r) {
    if constexpr (ROWS) {
      const int32_t nf = opaque(n_full), nt = opaque(n_tail);
#pragma unroll
      for (int j = 0; j < RC; ++j)
        if (j < nf) pre[j] = *reinterpret_cast<const Quad<LT>*>(r + (64 * j + lane) * QV);
      const LT* q = r + nf * 64 * QV;
#pragma unroll
      for (int j = 0; j < QV; ++j)
        if (64 * j < nt) tail[j] = q[min(64 * j + lane, nt - 1)];
    }
  };
  auto store_rows = [&]() {
    if constexpr (ROWS) {
      const int32_t nf = opaque(n_full), nt = opaque(n_tail);
#pragma unroll
      for (int j = 0; j < RC; ++j)
        if (j < nf)
          *reinterpret_cast<uint4*>(lrow[0] + (64 * j + lane) * QV) =
              make_uint4(pre[j].w[0], pre[j].w[1], pre[j].w[2], pre[j].w[3]);
      LT* q = lrow[0] + nf * 64 * QV;
#pragma unroll
      for (int j = 0; j < QV; ++j)
        if (64 * j < nt && 64 * j + lane < nt) q[64 * j + lane] = tail[j];
    }
  };
  auto zat = [&](int i, int32_t v) -> float {
    if constexpr (ROWS) return Ld::get(lrow[i], v);
    else return Ld::get(row_p[i], v);
  };
  Slot<NS> H[KPW];
#pragma unroll
  for (int i = 0; i < KPW; ++i) {
    const int32_t k = slot_id(i);
    lrow[i] = reinterpret_cast<LT*>(dyn + lay.rows + (int64_t)min(k, K - 1) * lay.row_stride);
    H[i].word = kNoTok | (kNoTok << 16);
    row_p[i] = logits + ((int64_t)b * K + min(k, K - 1)) * stride;
    word_p[i] = word_base + (int64_t)b * K + min(k, K - 1);
    if (k < K) {
      load_word(H[i], i);
      gather(H[i], row_p[i]);
      if (T > 1) load_word(H[i], i);
      load_rows(row_p[i]);
      store_rows();
      row_p[i] -= tstride;  // advanced at the start of a step
    }
  }
  uint32_t* marks_of[KPW];
#pragma unroll
  for (int i = 0; i < KPW; ++i)
    marks_of[i] = reinterpret_cast<uint32_t*>(dyn + lay.marks) + min(slot_id(i), K - 1) * lay.mark_words;
  __syncthreads();

  for (int32_t t = 0; t < T; ++t) {
    const int par = t & 1;
    // ---- this step's summaries become current, the next step's are loaded
#pragma unroll
    for (int i = 0; i < KPW; ++i) {
      const int32_t k = slot_id(i);
      if (k >= K) continue;
      Slot<NS>& h = H[i];
      row_p[i] += tstride;
      h.tok = h.n_tok;
      h.cls = h.n_cls;
      h.dst = h.n_dst;
      h.rpsi = h.n_rpsi;
      h.z = h.n_z;
      h.lse = h.n_lse;
      if (t + 1 < T) {
        gather(h, row_p[i] + tstride);
        if (t + 2 < T) load_word(h, i);
        load_rows(row_p[i] + tstride);
      }
    }
    // candidates are (slot, token) codes; a slot's logits and children
    auto mark_clear = [&](uint32_t* mk) {
      for (int32_t i = lane; i < lay.mark_words; i += 64) mk[i] = 0u;
      asm volatile("" ::: "memory");
    };
    auto marked = [&](const uint32_t* mk, int32_t c) { return ((mk[c >> 5] >> (c & 31)) & 1u) != 0u; };
    auto mark = [&](uint32_t* mk, int32_t c) {
      __hip_atomic_fetch_or(mk + (c >> 5), 1u << (c & 31), __ATOMIC_RELAXED,
                            __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    // every override member of state s, level by level (deepest first): the
    // class bitmap mk is cleared first and holds the overridden classes
    // afterwards. f(valid, token, child, psi) runs with all lanes, and before it
    // g(valid, class, psi) for every child that counts.
    auto walk_children = [&](int32_t s, uint32_t* mk, auto f, auto g) {
      mark_clear(mk);
      if (!biased || s == 0) return;
      Graph::State st = G.state(s);
      for (;;) {
        for (int32_t j0 = 0; j0 < st.nc; j0 += 64) {
          const int32_t j = j0 + lane;
          bool take = false;
          uint2 mm = make_uint2(0u, 0u);
          float py = 0.f;
          int32_t nm = 0, q0 = 0, lab = 0;
          const int32_t y = st.fc + j;
          if (j < st.nc) {
            G.child(y, mm, py);
            lab = arc_class(mm);
            take = !marked(mk, lab);
          }
          asm volatile("" ::: "memory");
          if (take) {
            mark(mk, lab);
            if (!arc_more(mm)) {
              nm = (mm.x >> 16) == (mm.x & 0xffffu) ? 1 : ((mm.y & 0xffffu) == (mm.x >> 16) ? 2 : 3);
            } else {
              q0 = A.cls_ptr[lab];
              nm = A.cls_ptr[lab + 1] - q0;
            }
          }
          g(take, lab, py);
          for (int32_t i = 0; __ballot(i < nm) != 0ull; ++i) {
            int32_t tk = 0;
            if (i < nm) {
              if (!arc_more(mm))
                tk = (int32_t)(i == 0 ? (mm.x & 0xffffu) : (i == 1 ? (mm.x >> 16) : (mm.y & 0xffffu)));
              else
                tk = A.cls_tok[q0 + i];
            }
            f(i < nm, tk, y, py);
          }
        }
        asm volatile("" ::: "memory");
        if (st.link == 0) break;
        st = G.state(st.link);
      }
    };

    auto walk = [&](int32_t s, uint32_t* mk, auto f) {
      walk_children(s, mk, f, [](bool, int32_t, float) {});
    };

    // ---- 1. candidates
    // streaming beam: slot x and its prefix slot y (live, holding x's labels
    // without the last) are one hypothesis: x's blank extension and y's
    // extension by x's last label merge. x pairs with its lowest-numbered
    // prefix slot. pair_y: the prefix slot of slot i of this wave (-1: none);
    // pair_x: the slots whose prefix slot it is.
    int32_t pair_y[KPW];
    uint32_t pair_x[KPW];
#pragma unroll
    for (int i = 0; i < KPW; ++i) {
      pair_y[i] = -1;
      pair_x[i] = 0u;
    }
    if constexpr (STREAM) {
      if (sa.recombine) {
        const bool live = has && hS > kNegInf;
        const bool ext = live && hl >= 0 && hl < V;
#pragma unroll
        for (int i = 0; i < KPW; ++i) {
          const int32_t k = slot_id(i);
          if (k >= K) continue;
          auto prefix_of = [&](int32_t x) -> int32_t {  // x's lowest prefix slot, or -1
            const uint32_t lo = (uint32_t)rl((int32_t)(uint32_t)hp, x);
            const uint32_t hi = (uint32_t)rl((int32_t)(uint32_t)(hp >> 32), x);
            const uint64_t want = ((uint64_t)hi << 32) | lo;
            const uint64_t y = __ballot(live && lane != x && hh == want);
            return y ? (int32_t)__builtin_ctzll(y) : -1;
          };
          const uint64_t is_ext = __ballot(ext);
          if ((is_ext >> k) & 1ull) pair_y[i] = prefix_of(k);
          const uint32_t lo = (uint32_t)rl((int32_t)(uint32_t)hh, k);
          const uint32_t hi = (uint32_t)rl((int32_t)(uint32_t)(hh >> 32), k);
          const uint64_t own = ((uint64_t)hi << 32) | lo;
          const bool k_live = (__ballot(live) >> k) & 1ull;
          uint64_t xs = k_live ? __ballot(ext && lane != k && hp == own) : 0ull;
          while (xs) {
            const int32_t x = (int32_t)__builtin_ctzll(xs);
            xs &= xs - 1ull;
            if (prefix_of(x) == k) pair_x[i] |= 1u << x;
          }
        }
      }
    }
    // whether a merge may change slot i's candidate for token v
    auto patched = [&](int i, int32_t v) -> bool {
      bool p = false;
      if constexpr (STREAM) {
        for (uint32_t xs = pair_x[i]; xs; xs &= xs - 1u)
          p = p || rl(hl, (int32_t)__builtin_ctz(xs)) == v;
      }
      return p;
    };

#pragma unroll
    for (int i = 0; i < KPW; ++i) {
      const int32_t k = slot_id(i);
      if (k >= K) continue;
      Slot<NS>& h = H[i];
      h.s = rl(hs, k);
      const float Sk = rlf(hS, k);
      if (ROWS && lane <= kList) h.z = h.tok >= 0 ? Ld::get(lrow[i], h.tok) : kNegInf;
      h.phi = root_phi;
      h.psi = root_psi;
      h.big = false;
      h.n = 0;
      h.on = 0u;
      float top = kNegInf;
      bool over = false;
      float opsi = kNegInf;  // psi of the child that has the listed move's class
      if (biased && h.s != 0) {  // the root's children are the root moves
        Graph::State st = G.state(h.s);
        h.phi = st.phi;
        h.psi = st.psi;
        int32_t f0 = st.fc, f1 = 0, f2 = 0, f3 = 0, s1 = st.nc, s2 = st.nc, s3 = st.nc;
        int32_t total = st.nc, levels = 1;
        bool allhot = st.fc + st.nc <= nhot;
        while (st.link != 0) {
          if (levels == kLevels) {
            h.big = true;
            break;
          }
          st = G.state(st.link);
          allhot = allhot && st.fc + st.nc <= nhot;
          if (levels == 1) f1 = st.fc - total;
          else if (levels == 2) f2 = st.fc - total;
          else f3 = st.fc - total;
          total += st.nc;
          if (levels == 1) s2 = s3 = total;
          else if (levels == 2) s3 = total;
          ++levels;
        }
        // the children of all levels but the shallowest are looked up by lane
        const int32_t deep = levels == 1 ? 0 : (levels == 2 ? s1 : (levels == 3 ? s2 : s3));
        h.big = h.big || total > 64 * NS || deep > 64;
        if (total > 0 && !h.big) {
          // the child of slot q = 64 i + lane: its level by where q lies
          bool in[NS];
          int32_t lv[NS], lab[NS];
#pragma unroll
          for (int g = 0; g < NS; ++g) {
            const int32_t q = 64 * g + lane;
            in[g] = q < total;
            const bool p1 = levels > 1 && q >= s1, p2 = levels > 2 && q >= s2, p3 = levels > 3 && q >= s3;
            lv[g] = (p1 ? 1 : 0) + (p2 ? 1 : 0) + (p3 ? 1 : 0);
            h.y[g] = in[g] ? q + (p3 ? f3 : (p2 ? f2 : (p1 ? f1 : f0))) : f0;
          }
          bool more = false;
#pragma unroll
          for (int g = 0; g < NS; ++g) {
            h.m[g] = make_uint2(0u, 0u);
            h.py[g] = 0.f;
            if (64 * g < total) {
              if (allhot) G.child_hot(in[g] ? h.y[g] : 1, h.m[g], h.py[g]);
              else if (in[g]) G.child(h.y[g], h.m[g], h.py[g]);
            }
            more = more || (in[g] && arc_more(h.m[g]));
          }
          h.big = __ballot(more) != 0ull;
          if (!h.big) {
            h.n = total;
#pragma unroll
            for (int g = 0; g < NS; ++g) {
              h.z0[g] = h.z1[g] = h.z2[g] = kNegInf;
              lab[g] = -3;
              if (64 * g < total) {
                lab[g] = in[g] ? arc_class(h.m[g]) : -3;
                const int32_t t0 = (int32_t)(h.m[g].x & 0xffffu), t1 = (int32_t)(h.m[g].x >> 16);
                const int32_t t2 = (int32_t)(h.m[g].y & 0xffffu);
                if (in[g]) {
                  h.z0[g] = zat(i, t0);
                  h.z1[g] = zat(i, t1);
                  h.z2[g] = zat(i, t2);
                  h.on |= (1u | (t1 != t0 ? 2u : 0u) | (t2 != t1 ? 4u : 0u)) << (3 * g);
                }
                const float zm = __builtin_fmaxf(__builtin_fmaxf(h.z0[g], h.z1[g]), h.z2[g]);
                top = __builtin_fmaxf(top, zm + h.py[g]);
              }
            }
            // the listed moves whose class a child has
            uint32_t om = 0u;
#pragma unroll
            for (int q = 0; q < kList; ++q) {
              const int32_t cq = rl(h.cls, q);
              bool hit = false;
#pragma unroll
              for (int g = 0; g < NS; ++g) hit = hit || lab[g] == cq;
              om |= __ballot(hit) != 0ull ? 1u << q : 0u;
            }
            over = ((om >> lane) & 1u) != 0u && lane < kList;
            // the psi of the deepest such child (the first)
            for (; om != 0u; om &= om - 1u) {
              const int32_t q = (int32_t)__builtin_ctz(om), cq = rl(h.cls, q);
#pragma unroll
              for (int g = NS - 1; g >= 0; --g) {
                const uint64_t at = __ballot(lab[g] == cq);
                if (at != 0ull) {
                  const float pq = rlf(h.py[g], (int32_t)__builtin_ctzll(at));
                  if (lane == q) opsi = pq;
                }
              }
            }
            // drop the children that a deeper state's child shadows
            for (int32_t j = 0; j < deep; ++j) {
              const int32_t cj = rl(lab[0], j);
              const int32_t lj = (j >= s1 ? 1 : 0) + (levels > 2 && j >= s2 ? 1 : 0) +
                                 (levels > 3 && j >= s3 ? 1 : 0);
#pragma unroll
              for (int g = 0; g < NS; ++g)
                if (lab[g] == cj && lv[g] > lj) h.on &= ~(7u << (3 * g));
            }
          }
        }
        if (h.big) {
          // The psi of the children that have a listed move's class. Narrow rows of
          // few waves look the moves up one by one (stream of 5 hypotheses of 1000
          // tokens 536 us a pass against 547 through LDS); else the child leaves
          // its psi in LDS, at the last such move (32 hypotheses: 395 against 406).
          constexpr bool kThroughLds = NW == 16 || !ROWS;
          float* ob = S.opsi[w];
          walk_children(h.s, marks_of[i], [](bool, int32_t, int32_t, float) {},
                        [&](bool take, int32_t lab, float py) {
                          int32_t cls = h.cls;
                          asm volatile("" : "+v"(cls));  // its lanes are not kept across the walk
                          int32_t at = -1;
#pragma unroll
                          for (int q = 0; q < kList; ++q) at = lab == rl(cls, q) ? q : at;
                          if constexpr (kThroughLds) {
                            if (take && at >= 0) ob[at] = py;
                          } else {
                            if (__ballot(take && at >= 0) == 0ull) return;
#pragma unroll 1
                            for (int32_t q = 0; q < kList; ++q) {
                              const uint64_t who = __ballot(take && lab == rl(cls, q));
                              if (who == 0ull) continue;
                              const float pq = rlf(py, (int32_t)__builtin_ctzll(who));
                              if (lane == q) opsi = pq;
                            }
                          }
                        });
          over = h.cls >= 0 && lane < kList && marked(marks_of[i], h.cls);
          if constexpr (kThroughLds) {
            int32_t at = 0;
#pragma unroll
            for (int q = 0; q < kList; ++q) at = h.cls == rl(h.cls, q) ? q : at;
            if (over) opsi = ob[at];
          }
        }
      }
      h.c = (Sk - h.lse) - h.phi;
      h.top = h.c + top;
      h.lv = kNegInf;
      if (lane < kList && h.tok >= 0 && !over) h.lv = h.c + (h.z + h.rpsi);
      if (lane == kList) h.lv = h.c + (h.z + h.phi);
      // A listed token whose class a child has is a candidate with the child's
      // psi. Where most classes have one (many phrases over few tokens) the
      // blanks alone would leave a weak bound, which most of the row reaches (100
      // streams, 2 hypotheses, 1000 phrases over 200 tokens, calls of 16 steps:
      // 154 us without, 86 us with it; 32 hypotheses of 1000 tokens 1680 and 550).
      float post = over && h.tok >= 0 ? h.c + (h.z + opsi) : h.lv;
      if constexpr (STREAM) {
        if (lane == 0) {
          S.c[k] = h.c;
          S.psi[k] = h.psi;
        }
        if (lane == kList) S.a[k] = h.lv;
        // values that a merge may change bound nothing
        if (lane == kList && pair_y[i] >= 0) post = kNegInf;
        if (lane < kList && patched(i, h.tok)) post = kNegInf;
      }
      if (lane <= kList) S.listed[9 * k + lane] = post;
    }
    __syncthreads();

    // ---- 2. the bound, and the candidates that reach it
    float best = kNegInf;
    int32_t bound = 0;  // largest gap value with fewer than K posted candidates below it
    if (NW < 16 || w == 0) {
      float pv[NV];
#pragma unroll
      for (int r = 0; r < NV; ++r) {
        pv[r] = (64 * r + lane < 9 * K) ? S.listed[64 * r + lane] : kNegInf;
        best = __builtin_fmaxf(best, pv[r]);
      }
      best = wave_max_dpp(best);
      int32_t q[NV];
#pragma unroll
      for (int r = 0; r < NV; ++r) q[r] = gap_of(best, pv[r]);
#pragma unroll
      for (int bit = 8; bit >= 0; --bit) {
        const int32_t c = bound | (1 << bit);
        int32_t cnt = 0;
#pragma unroll
        for (int r = 0; r < NV; ++r) cnt += (int32_t)__builtin_popcountll(__ballot(q[r] < c));
        if (cnt < K) bound = c;
      }
    }
    if constexpr (NW == 16) {
      // sixteen waves finding the same bound would share four SIMDs: the first
      // one hands it to the others
      if (w == 0 && lane == 0) {
        S.best = best;
        S.first_bound = bound;
      }
      __syncthreads();
      best = rlf(S.best, 0);
      bound = __builtin_amdgcn_readfirstlane(S.first_bound);
    }
    // streaming beam: the merged values
    float blank_v[KPW];
#pragma unroll
    for (int i = 0; i < KPW; ++i) blank_v[i] = H[i].lv;  // on lane kList
    if constexpr (STREAM) {
#pragma unroll
      for (int i = 0; i < KPW; ++i) {
        const int32_t k = slot_id(i);
        if (k >= K || pair_y[i] < 0) continue;
        const int32_t y = pair_y[i], v = rl(hl, k);
        float zy;
        if constexpr (ROWS)
          zy = Ld::get(reinterpret_cast<const LT*>(dyn + lay.rows + (int64_t)y * lay.row_stride), v);
        else
          zy = Ld::get(row_p[i] + (int64_t)(y - k) * stride, v);
        const float av = S.a[k], bv = S.c[y] + (zy + H[i].psi);
        if (av > kNegInf && bv > kNegInf) {
          const bool keep = av > bv || (av == bv && k < y);
          blank_v[i] = keep ? logaddexp32(av, bv) : kNegInf;
        }
      }
    }
    // y's candidate for token v (the last label of slot x) after the merge
    auto merged_at = [&](int i, int32_t x, float& val, float& zv) {
      const Slot<NS>& h = H[i];
      const int32_t k = slot_id(i), v = rl(hl, x);
      zv = zat(i, v);
      const float av = S.a[x], bv = h.c + (zv + S.psi[x]);
      val = bv;
      if (av > kNegInf && bv > kNegInf) {
        const bool keep_a = av > bv || (av == bv && x < k);
        val = keep_a ? kNegInf : logaddexp32(av, bv);
      }
    };

    bool full = false;  // the rows are scanned whatever their lists hold
    if (bound >= kNone) {
      // fewer than K posted candidates: a slot with K root moves gives a bound
#pragma unroll
      for (int i = 0; i < KPW; ++i) {
        const int32_t k = slot_id(i);
        if (k >= K) continue;
        const Slot<NS>& h = H[i];
        int32_t bk = 0;
        if (best > kNegInf && h.c > kNegInf) {
          walk(h.s, marks_of[i], [](bool, int32_t, int32_t, float) {});
          for (int bit = 8; bit >= 0; --bit) {
            const int32_t c = bk | (1 << bit);
            int32_t cnt = 0;
            for (int32_t v0 = 0; v0 < V; v0 += 64) {
              const int32_t v = v0 + lane;
              bool in = false;
              if (v < V) {
                const float val = h.c + (zat(i, v) + (biased ? gpsi[v] : 0.f));
                in = gap_of(best, val) < c;
                if (in && biased) {
                  const int32_t cl = A.class_map[v];
                  in = !(cl >= 0 && marked(marks_of[i], cl));
                }
                if (in) in = !patched(i, v);
              }
              cnt += (int32_t)__builtin_popcountll(__ballot(in));
            }
            if (cnt < K) bk = c;
          }
        } else {
          bk = kNone;
        }
        if (lane == 0) S.bound[k] = bk;
      }
      __syncthreads();
      const int32_t mine = has ? S.bound[lane] : kNone;
      bound = kNone;
      for (int32_t k = 0; k < K; ++k) bound = min(bound, rl(mine, k));
      full = true;
    }
    const bool rounds = bound >= kNone;  // no bound: the K rounds below

    // places in the shared list, and the candidates of the lanes in mask there
    auto take = [&](int32_t count) -> int32_t {
      int32_t base = 0;
      if (lane == 0)
        base = __hip_atomic_fetch_add(&S.count[par], count, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_WORKGROUP);
      return __builtin_amdgcn_readfirstlane(base);
    };
    auto put = [&](uint64_t mask, int32_t base, int32_t k, int32_t v, float val, int32_t dst,
                   float step) {
      const int32_t pos = base + (int32_t)lanes_below(mask);
      if (((mask >> lane) & 1ull) && pos < kCap) {
        Cand e;
        e.code = ~(((uint32_t)k << 16) | (uint32_t)v);
        e.okey = order_key(val);
        e.dst = dst;
        e.step = step;
        S.cand[pos] = e;
      }
    };
    auto add = [&](bool p, int32_t k, int32_t v, float val, int32_t dst, float step) {
      const uint64_t mask = __ballot(p);
      if (mask != 0ull) put(mask, take((int32_t)__builtin_popcountll(mask)), k, v, val, dst, step);
    };
    if (!rounds) {
#pragma unroll
      for (int i = 0; i < KPW; ++i) {
        const int32_t k = slot_id(i);
        if (k >= K) continue;
        Slot<NS>& h = H[i];
        const float gain = h.rpsi - h.phi;
        // gap_of(best, v) <= bound
        const float reach = __int_as_float((bound + 1 + ((127 - 12) << 4)) << 19);
        auto pass = [&](float v) { return best - v < reach; };
        // the listed moves and the blank, and the children: one place in the
        // shared list for all of the slot's
        {
          const bool blank = lane == kList;
          const float lv = blank ? blank_v[i] : h.lv;
          bool lp = lane <= kList && pass(lv);
          if (STREAM && pair_x[i] && !blank) lp = lp && !patched(i, h.tok);
          const uint64_t lm = __ballot(lp);
          uint64_t cm[3 * NS];
          int32_t need = (int32_t)__builtin_popcountll(lm);
#pragma unroll
          for (int q = 0; q < 3 * NS; ++q) cm[q] = 0ull;
          const bool kids = h.n > 0 && __ballot(pass(h.top)) != 0ull;
          if (kids) {
#pragma unroll
            for (int g = 0; g < NS; ++g) {
              if (64 * g >= h.n) continue;
              const int32_t tk[3] = {(int32_t)(h.m[g].x & 0xffffu), (int32_t)(h.m[g].x >> 16),
                                     (int32_t)(h.m[g].y & 0xffffu)};
              const float zz[3] = {h.z0[g], h.z1[g], h.z2[g]};
#pragma unroll
              for (int q = 0; q < 3; ++q) {
                bool p = ((h.on >> (3 * g + q)) & 1u) && pass(h.c + (zz[q] + h.py[g]));
                if (STREAM && pair_x[i]) p = p && !patched(i, tk[q]);
                cm[3 * g + q] = __ballot(p);
                need += (int32_t)__builtin_popcountll(cm[3 * g + q]);
              }
            }
          }
          if (need > 0) {
            int32_t base = take(need);
            put(lm, base, k, blank ? V : h.tok, lv, blank ? h.s : h.dst,
                (h.z - h.lse) + (blank || !biased ? 0.f : gain));
            base += (int32_t)__builtin_popcountll(lm);
            if (kids) {
#pragma unroll
              for (int g = 0; g < NS; ++g) {
                if (64 * g >= h.n) continue;
                const int32_t tk[3] = {(int32_t)(h.m[g].x & 0xffffu), (int32_t)(h.m[g].x >> 16),
                                       (int32_t)(h.m[g].y & 0xffffu)};
                const float zz[3] = {h.z0[g], h.z1[g], h.z2[g]};
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                  const uint64_t mq = cm[3 * g + q];
                  if (mq != 0ull) {
                    put(mq, base, k, tk[q], h.c + (zz[q] + h.py[g]), h.y[g],
                        (zz[q] - h.lse) + (h.py[g] - h.phi));
                    base += (int32_t)__builtin_popcountll(mq);
                  }
                }
              }
            }
          }
        }
        if (h.big) {
          walk(h.s, marks_of[i], [&](bool valid, int32_t tk, int32_t y, float py) {
            const float z = valid ? zat(i, tk) : kNegInf;
            const float v = h.c + (z + py);
            bool p = valid && pass(v);
            if (STREAM && pair_x[i]) p = p && !patched(i, tk);
            add(p, k, tk, v, y, (z - h.lse) + (py - h.phi));
          });
        }
        if constexpr (STREAM) {
          for (uint32_t xs = pair_x[i]; xs; xs &= xs - 1u) {
            const int32_t x = (int32_t)__builtin_ctz(xs);
            float val, zv;
            merged_at(i, x, val, zv);
            const float px = S.psi[x];
            add(lane == 0 && pass(val), k, rl(hl, x), val, rl(hs, x),
                (zv - h.lse) + (biased ? px - h.phi : 0.f));
          }
        }
        // root moves past the list: none of them exceeds the last listed one
        const int32_t t8 = rl(h.tok, kList - 1);
        const float b8 = h.c + (rlf(h.z, kList - 1) + rlf(h.rpsi, kList - 1));
        if (full || (t8 >= 0 && pass(b8))) {
          bool walked = h.big;  // the bitmap holds the overridden classes
          constexpr int SC = 8;  // chunks whose loads are in flight together
          for (int32_t v0 = 0; v0 < V; v0 += 64 * SC) {
            float zc[SC], pc[SC];
#pragma unroll
            for (int q = 0; q < SC; ++q) {
              const int32_t v = min(v0 + 64 * q + lane, V);
              zc[q] = zat(i, v);
              pc[q] = biased ? gload(gpsi + v) : 0.f;
            }
#pragma unroll
            for (int q = 0; q < SC; ++q) {
              const int32_t v = v0 + 64 * q + lane;
              const float val = h.c + (zc[q] + pc[q]);
              bool p = v < V && pass(val);
              if (__ballot(p) == 0ull) continue;
#pragma unroll
              for (int e = 0; e < kList; ++e) p = p && rl(h.tok, e) != v;
              if (__ballot(p) == 0ull) continue;
              if (!walked) walk(h.s, marks_of[i], [](bool, int32_t, int32_t, float) {});
              walked = true;
              int32_t dst = fixed;
              if (p && biased) {
                const int32_t cl = gload(A.class_map + v);
                p = !(cl >= 0 && marked(marks_of[i], cl));
                dst = gload(gdst + v);
              }
              if (STREAM && pair_x[i]) p = p && !patched(i, v);
              add(p, k, v, val, dst, (zc[q] - h.lse) + (biased ? pc[q] - h.phi : 0.f));
            }
          }
        }
      }
    }
    // the other step's counters: their readers passed this step's first barrier
    if (threadIdx.x == 0) S.count[par ^ 1] = 0;
    if (NW == 16 && w == 0) S.rank[par ^ 1][lane] = 0;
    __syncthreads();

    // ---- 3. the K best: lane j takes rank j
    const int32_t total = __builtin_amdgcn_readfirstlane(S.count[par]);
    uint32_t w_code = ~0u, w_key = 0u;
    int32_t w_dst = fixed;
    float w_step = 0.f, w_val = kNegInf;
    if (!rounds && total <= 64) {
      const bool in = lane < total;
      Cand e = {0u, 0u, 0, 0.f};
      if (in) e = S.cand[lane];
      const uint64_t key = ((uint64_t)e.okey << 32) | e.code;
      // lanes past total hold key 0, which is before no candidate
      int32_t rank = 0;
      auto before = [&](int32_t q0, int32_t step, int32_t end) {
        for (int32_t q = q0; q < end; q += step)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const uint64_t kq = ((uint64_t)(uint32_t)rl((int32_t)e.okey, q + u) << 32) |
                                (uint32_t)rl((int32_t)e.code, q + u);
            rank += kq > key ? 1 : 0;
          }
      };
      if constexpr (NW == 16) {
        // sixteen waves ranking everything would share four SIMDs: each takes
        // four of the candidates and the counts are added up
        before(4 * w, 64, 4 * w < total ? 4 * w + 1 : 0);
        if (rank) __hip_atomic_fetch_add(&S.rank[par][lane], rank, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_WORKGROUP);
        __syncthreads();
        rank = S.rank[par][lane];
      } else {
        before(0, 4, total);
      }
      const int32_t to = 4 * ((in && rank < K) ? rank : 63);  // K <= 32: lane 63 is spare
      w_code = (uint32_t)__builtin_amdgcn_ds_permute(to, (int32_t)e.code);
      w_key = (uint32_t)__builtin_amdgcn_ds_permute(to, (int32_t)e.okey);
      w_dst = __builtin_amdgcn_ds_permute(to, e.dst);
      w_step = __int_as_float(__builtin_amdgcn_ds_permute(to, __float_as_int(e.step)));
      w_val = from_order_key(w_key);
    } else if (!rounds && total <= kCap) {
      int32_t who = 0;
      for (int32_t r0 = 0; r0 < total; r0 += 64) {
        const bool in = r0 + lane < total;
        uint64_t key = 0ull;
        if (in) key = ((uint64_t)S.cand[r0 + lane].okey << 32) | S.cand[r0 + lane].code;
        int32_t rank = 0;
        for (int32_t q = 0; q < total; ++q) {
          const uint64_t kq = ((uint64_t)S.cand[q].okey << 32) | S.cand[q].code;
          rank += kq > key ? 1 : 0;
        }
        const int32_t to = 4 * ((in && rank < K) ? rank : 63);
        who |= __builtin_amdgcn_ds_permute(to, r0 + lane + 1);  // 0 where nothing was sent
      }
      const int32_t at = min(max(who - 1, 0), kCap - 1);
      if (has) {
        const Cand e = S.cand[at];
        w_code = e.code;
        w_dst = e.dst;
        w_step = e.step;
        w_val = from_order_key(e.okey);
      }
    } else {
      // K rounds of an argmax over every candidate after the last one taken
      constexpr int32_t kRootMove = INT_MIN;  // the token's root move, looked up for the best
      float pvl = 0.f;
      int32_t pcode = -1;
      for (int32_t j = 0; j < K; ++j) {
        float bv = kNegInf, bstep = 0.f;
        int32_t bc = INT_MAX, bd = fixed;
        auto offer = [&](bool p, int32_t k, int32_t v, float val, int32_t dst, float step) {
          const int32_t code = (k << 16) | v;
          if (j == 0 && p && code == 0) S.bound[0] = dst == kRootMove ? gdst[0] : dst;  // its place when no candidate is left
          const bool after = j == 0 || val < pvl || (val == pvl && code > pcode);
          if (p && after && better(val, code, bv, bc)) {
            bv = val;
            bc = code;
            bd = dst;
            bstep = step;
          }
        };
#pragma unroll
        for (int i = 0; i < KPW; ++i) {
          const int32_t k = slot_id(i);
          if (k >= K) continue;
          Slot<NS>& h = H[i];
          offer(lane == kList, k, V, blank_v[i], h.s, (h.z - h.lse) + 0.f);
          walk(h.s, marks_of[i], [&](bool valid, int32_t tk, int32_t y, float py) {
            const float z = valid ? zat(i, tk) : kNegInf;
            bool p = valid;
            if (STREAM && pair_x[i]) p = p && !patched(i, tk);
            offer(p, k, tk, h.c + (z + py), y, (z - h.lse) + (py - h.phi));
          });
          if constexpr (STREAM) {
            for (uint32_t xs = pair_x[i]; xs; xs &= xs - 1u) {
              const int32_t x = (int32_t)__builtin_ctz(xs);
              float val, zv;
              merged_at(i, x, val, zv);
              const float px = S.psi[x];
              offer(lane == 0, k, rl(hl, x), val, rl(hs, x),
                    (zv - h.lse) + (biased ? px - h.phi : 0.f));
            }
          }
          constexpr int SC = NW < 16 ? 4 : 1;  // chunks whose loads are in flight together
          for (int32_t v0 = 0; v0 < V; v0 += 64 * SC) {
            float pc[SC];
            int32_t cc[SC];
#pragma unroll
            for (int q = 0; q < SC; ++q) {
              const int32_t v = min(v0 + 64 * q + lane, V);
              pc[q] = biased ? gload(gpsi + v) : 0.f;
              cc[q] = biased ? gload(A.class_map + v) : -1;
            }
#pragma unroll
            for (int q = 0; q < SC; ++q) {
              const int32_t v = v0 + 64 * q + lane;
              bool p = v < V && !(cc[q] >= 0 && marked(marks_of[i], cc[q]));
              if (STREAM && pair_x[i]) p = p && !patched(i, v);
              const float z = zat(i, min(v, V));
              offer(p, k, v, h.c + (z + pc[q]), biased ? kRootMove : fixed,
                    (z - h.lse) + (biased ? pc[q] - h.phi : 0.f));
            }
          }
        }
        float wv;
        int32_t wc;
        const int32_t wl = wave_argmax_dpp(bv, bc, wv, wc);
        int32_t wd = rl(bd, wl);
        if (wd == kRootMove) wd = sload(gdst + (wc & 0xffff));
        const float ws = rlf(bstep, wl);
        const int rp = j & 1;
        if (lane == 0) {
          S.red_v[rp][w] = wv;
          S.red_code[rp][w] = wc;
          S.red_dst[rp][w] = wd;
          S.red_step[rp][w] = ws;
        }
        __syncthreads();
        const bool in = lane < NW;
        float gv;
        int32_t gc;
        const float rv = in ? S.red_v[rp][lane] : kNegInf;
        const int32_t rc = in ? S.red_code[rp][lane] : INT_MAX;
        const int32_t rd = in ? S.red_dst[rp][lane] : 0;
        const float rs = in ? S.red_step[rp][lane] : 0.f;
        const int32_t gl = wave_argmax_dpp(rv, rc, gv, gc);
        const int32_t gd = rl(rd, gl);
        const float gs = rlf(rs, gl);
        if (lane == j) {
          // none left (nan values only): slot 0 by its first token, no score
          w_code = gc == INT_MAX ? ~0u : ~(uint32_t)gc;
          w_dst = gc == INT_MAX ? S.bound[0] : gd;
          w_step = gc == INT_MAX ? __builtin_nanf("") : gs;
          w_val = gv;
        }
        pvl = gv;
        pcode = gc;
      }
    }

    // ---- slot j's hypothesis into lane j; the first wave writes the outputs
    {
      const uint32_t f = ~w_code;
      int32_t k = (int32_t)(f >> 16), v = (int32_t)(f & 0xffffu);
      if (!has || k >= K || v >= V1) {
        k = 0;
        v = 0;
      }
      const int32_t ns = biased ? w_dst : fixed;
      if constexpr (STREAM) {
        const uint64_t ph = ((uint64_t)(uint32_t)__shfl((int32_t)(uint32_t)(hh >> 32), k, 64) << 32) |
                            (uint32_t)__shfl((int32_t)(uint32_t)hh, k, 64);
        const uint64_t pp = ((uint64_t)(uint32_t)__shfl((int32_t)(uint32_t)(hp >> 32), k, 64) << 32) |
                            (uint32_t)__shfl((int32_t)(uint32_t)hp, k, 64);
        const int32_t pl = __shfl(hl, k, 64), pn = __shfl(hn, k, 64);
        const bool emit = has && v != V;
        const uint64_t em = __ballot(emit);
        const int32_t r = tlen + (int32_t)lanes_below(em);
        hh = emit ? ph * (uint64_t)TB_HASH_MUL + (uint64_t)(v + 1) : ph;
        hp = emit ? ph : pp;
        hl = emit ? v : pl;
        hn = emit ? (r < sa.cap ? r : -2) : pn;
        if (w == 0 && emit && r < sa.cap) {
          sa.tree[((int64_t)b * sa.cap + r) * 2] = v;
          sa.tree[((int64_t)b * sa.cap + r) * 2 + 1] = pn;
        }
        tlen += (int32_t)__builtin_popcountll(em);
      }
      hs = ns;
      hS = w_val;
      if (w == 0 && has) {
        const int64_t o = ((int64_t)b * K + lane) + (int64_t)t * ostride;
        out_tok[o] = v;
        out_parent[o] = k;
        out_state[o] = ns;
        out_step[o] = w_step;
        out_cum[o] = w_val;
      }
    }
    // this wave's next row to LDS (the streaming beam's waves read each
    // other's rows only before the second barrier)
    if (t + 1 < T && slot_id(0) < K) store_rows();
  }

  if (w == 0 && has && T > 0) {
    states[(int64_t)b * K + lane] = hs;
    scores[(int64_t)b * K + lane] = hS;
    if constexpr (STREAM) {
      tb_hyp y;
      y.hash = hh;
      y.prefix_hash = hp;
      y.last = hl;
      y.node = hn;
      sa.hyps[(int64_t)b * K + lane] = y;
      if (lane == 0) sa.tree_len[b] = tlen < sa.cap ? tlen : sa.cap;
    }
  }
}

}  // namespace blist
}  // namespace tbias
