// attend_prefill.hip -- multi-query (prefill / denoising) attention over
// bf16 segments on the CDNA4 matrix cores (App. E, "Attention over
// heterogeneous cache segments": one softmax across all segments; packed
// segments are dequantised into a reusable workspace before attention).
//
// Work item: 128 query rows of one (b, h_kv) -- the rows of its G query heads
// are contiguous in q -- in one workgroup of four waves; each wave owns two
// 16-row query tiles.  The workgroup walks every key tile (32 rows) of every
// segment once: the waves stage the K and V rows of later tiles through
// registers (two register sets, so a tile's loads have two iterations to
// arrive) into a four-deep ring of padded LDS tiles.  The loop is a
// three-stage software pipeline: in iteration t a wave issues, interleaved
// (each matrix instruction followed by its share of the softmax),
//   S^T(t+1) = K Q^T    v_mfma_f32_16x16x32_bf16, K rows read from LDS as the
//                       A operand (shared by both query tiles), Q^T in
//                       registers;
//   O^T += V^T P(t-1)   V^T by transposing LDS reads (shared by both query
//                       tiles); fp16 P and V on v_mfma_f32_16x16x32_f16 when
//                       every V value of the call fits fp16 (a range pass sets
//                       a flag the kernel reads), else bf16 V with P as bf16
//                       hi + lo parts;
//   softmax(t)          on the vector ALUs: base-2 exponentials against a
//                       lazily raised reference maximum, running per-segment
//                       sums for seg_lse;
// none of which depends on another, so one wave keeps the matrix cores and
// the vector ALUs busy at once; the probability operands of consecutive
// tiles alternate between two register sets.  The rare raise of the reference
// maximum, and the mask of a tile that a segment's end leaves partial, run
// after the matrix instructions (a raise rescales the accumulators they update).
// Outputs (normalised O, lse, per-segment lse) are written directly; only a
// call with too few query blocks for the chip splits the keys (Split).
// Workgroups are mapped so that those of one (b, h_kv) run on the same XCD and
// share its L2 copy of the head's rows.
//
// Packed segments first go through prepare_kernel: codes -> round_to_bf16(
// fmaf(code, scale, min)) into a [B, Hkv, n_full, D] bf16 workspace (once per
// call, where the query blocks of a head would otherwise each decode every
// packed tile again); their residual tails are read in place.  This
// preparation (with the fp16 V copies and the range flag) is a stage of its
// own, so an execution plan over an unchanged cache runs it once.
#include <string.h>

#include <algorithm>
#include <type_traits>

#include "mfma_util.h"
#include "uc_common.h"

namespace uc {
namespace {

using namespace mf;

constexpr int STAGES = 4;                  // stages in LDS: t-1 .. t+1 in use, t+2 staged
constexpr int SUBB = 2 * TILEB;            // one tile: K rows + V rows
// Layouts: W waves per workgroup, TPS tiles per stage (one barrier per
// stage) and QT 16-row query tiles per wave.  <4, 1, 2>: 128 query rows, two
// workgroups per CU; <8, 2, 2>: 256 query rows, one workgroup per CU, half
// the barriers and staging per query row.  (Four query tiles per wave, one
// wave per SIMD, measured slower than two waves per SIMD with two.)
template <int W, int QT>
constexpr int qrows() { return W * QT * 16; }
constexpr float kLazy = 8.0f;
constexpr float kLazyExp = 256.0f;  // 2^kLazy
constexpr int kMaxViews = 2 * kMaxSeg;
constexpr int kPrepBlocks = 256, kPrepThreads = 1024;  // of prepare_kernel; one flag byte per block

// dense row views of the logical sequence, in order; seg = logical segment
struct View {
  const uint16_t* k;
  const uint16_t* v;
  const uint16_t* vh;  // the V rows converted to fp16 once per call, [BH, n, D]
  int64_t bh_stride;   // elements between consecutive (b, h_kv) of k and v
  int n;               // rows
  int seg;
};

struct Views {
  View v[kMaxViews];
  int n;
  int tiles;  // total key tiles
};

// A call whose query blocks leave CUs idle splits its key tiles: split s of a
// query block takes tiles [s*per, (s+1)*per) and leaves an unnormalised
// record of every query row -- (m, l) in base 2, O, and the log-sum-exp of
// each segment's rows it saw -- for split_merge_kernel.  Record s of query
// row r is number r*n + s.  n = 1: outputs are written directly.
// Every split starts from the reference maximum that an unsplit walk has after
// its first tile, so a probability is rounded to the same 16 bits however the
// keys are split (references of the splits' own moved the results of 203 query
// rows over 6144 by 2.7e-4, as much as that rounding itself); what is left is
// the order of the sums, and rows whose reference is raised later on (3e-5 to
// 8e-5 over calls of 3 to 1000 query rows with outlier keys).  It costs a call
// of 203 rows 0.6 us of 48.
struct Split {
  int n, per;
  float* ml;
  float* o;
  float* seg;
};

struct QState {
  float m, l, ls;  // reference max (base 2), row sum, running sum of the current segment
  f4 acc[8];       // O^T, dims d*16 + g4*4 + j of query column i16
};

// tile t of the sequence -> view index and first row
__device__ inline int tile_view(const Views& vs, int t, int& row0) {
  int i = 0;
  while (i + 1 < vs.n && t >= (vs.v[i].n + TILE - 1) / TILE) {
    t -= (vs.v[i].n + TILE - 1) / TILE;
    ++i;
  }
  row0 = t * TILE;
  return i;
}

// A walk over the logical sequence one 32-row tile at a time.  The current
// view's row count, segment and this (b, h_kv)'s K and V rows stay in
// scalars, so a step reads the view table (kernel arguments) only when it
// crosses into the next view.
template <bool F16>
struct Cursor {
  int vi, row0, n, seg;
  const uint16_t* k;
  const uint16_t* v;
  __device__ inline void load(const Views& vs, int bh) {
    const View& w = vs.v[vi];
    n = w.n;
    seg = w.seg;
    k = w.k + bh * w.bh_stride;
    v = F16 ? w.vh + (int64_t)bh * w.n * D : w.v + bh * w.bh_stride;
  }
  __device__ inline void start(const Views& vs, int bh, int t) {
    vi = tile_view(vs, t, row0);
    load(vs, bh);
  }
  __device__ inline void next(const Views& vs, int bh) {
    row0 += TILE;
    if (row0 >= n && vi + 1 < vs.n) {
      ++vi;
      row0 = 0;
      load(vs, bh);
    }
  }
};

// one thread's share of staging the two tiles of a stage: row tid/16,
// chunk tid%16 of each tile's K and V rows
struct Stage {
  u4 k[2], v[2];
};

// A thread stages two 16-byte chunks of K and of V per stage: chunk i is
// global chunk g = tid + i * NT, tile g / 512 of the stage, row (g % 512) / 16,
// column chunk g % 16 (two rows of one tile with 256 threads, one row of each
// of two tiles with 512).  F16: V comes from the view's fp16 copy.
template <bool F16, int NT, bool V = true>
__device__ inline void stage_load(const Cursor<F16>& cu, Stage& S, int i) {
  const __amdgpu_buffer_rsrc_t rk = rsrc(cu.k, (uint32_t)cu.n * ROWB);
  const __amdgpu_buffer_rsrc_t rv = rsrc(cu.v, (uint32_t)cu.n * ROWB);
  const int g = (threadIdx.x + i * NT) & 511, r = g >> 4, c = g & 15;
  const int off = (cu.row0 + r) * ROWB + c * 16;
  S.k[i] = bload(rk, off);
  if (V) S.v[i] = bload(rv, off);
}

// chunk i into the LDS tile at buf (K rows, V rows at + TILEB)
template <int NT, bool V = true>
__device__ inline void stage_store(char* buf, const Stage& S, int i) {
  const int g = (threadIdx.x + i * NT) & 511, r = g >> 4, c = g & 15;
  *reinterpret_cast<u4*>(buf + toff(r, c)) = S.k[i];
  if (V) *reinterpret_cast<u4*>(buf + TILEB + toff(r, c)) = S.v[i];
}

// LDS tile of tile t of the sequence
template <int TPS>
__device__ inline char* tile_buf(char* lds, int t) {
  return lds + ((t / TPS) % STAGES) * (TPS * SUBB) + (t % TPS) * SUBB;
}

// rows past a view's end, staged as zeros (range-checked loads), take no part:
// logit -inf, probability 0 (their V rows are 0 too).  n_valid: rows of the
// tile.  The lane's rows are formed here, not kept in a register of the loop.
__device__ inline void tile_mask(f4& s0, f4& s1, int n_valid) {
  int row = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)) / 16 * 4;
  asm volatile("" : "+v"(row));
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (row + j >= n_valid) s0[j] = -INFINITY;
    if (row + 16 + j >= n_valid) s1[j] = -INFINITY;
  }
}

// raw logits of one query tile (8 per lane)
__device__ inline void tile_logits(const f4& s0, const f4& s1, float (&p)[8]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    p[j] = s0[j];
    p[4 + j] = s1[j];
  }
}

// common path of the softmax of one query tile: probabilities against the
// current reference; returns the lane's sum.  A lane sum above 2^kLazy
// (every logit more than kLazy above the reference makes one, and a first
// tile's -inf reference makes inf or NaN) sends the wave through tile_raise.
__device__ inline float tile_exp(const QState& st, const f4& s0, const f4& s1, float scale_log2,
                                 float (&e)[8]) {
  float p[8];
  tile_logits(s0, s1, p);
#pragma unroll
  for (int j = 0; j < 8; ++j) e[j] = __builtin_amdgcn_exp2f(fmaf(p[j], scale_log2, -st.m));
  return ((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7]));
}

// largest logit of each query column of a tile, in base 2 (the scale is
// positive, so the maximum of the raw logits gives the maximum)
__device__ inline float column_max(const float (&p)[8], float scale_log2) {
  float mx = fmaxf(fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3])),
                   fmaxf(fmaxf(p[4], p[5]), fmaxf(p[6], p[7]))) * scale_log2;
  mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
  return fmaxf(mx, __shfl_xor(mx, 32, 64));
}

// rare path: raise the reference to the column maximum, rescale the running
// state and recompute the probabilities (they stay below 2^kLazy, well inside
// fp16)
__device__ inline float tile_raise(QState& st, const f4& s0, const f4& s1, float scale_log2,
                                   float (&e)[8]) {
  float p[8];
  tile_logits(s0, s1, p);
  const float m_new = fmaxf(st.m, column_max(p, scale_log2));
  const float alpha = __builtin_amdgcn_exp2f(st.m - m_new);
  st.l *= alpha;
  st.ls *= alpha;
#pragma unroll
  for (int d = 0; d < 8; ++d) st.acc[d] *= alpha;
  st.m = m_new;
#pragma unroll
  for (int j = 0; j < 8; ++j) e[j] = __builtin_amdgcn_exp2f(fmaf(p[j], scale_log2, -st.m));
  return ((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7]));
}

// probability operands of one query tile: fp16 P (F16), else bf16 hi + lo
struct POp {
  u4 hi, lo;
};

template <bool F16>
__device__ inline POp pack_p(const float (&e)[8]) {
  POp r;
  if (F16) {
    r.hi = u4{h2(e[0], e[1]), h2(e[2], e[3]), h2(e[4], e[5]), h2(e[6], e[7])};
    r.lo = r.hi;
  } else {
    split_p(e, r.hi, r.lo);
  }
  return r;
}

// sum of a lane-partial value over the four key-row lanes of a query column
__device__ inline float col_sum(float x) {
  x += __shfl_xor(x, 16, 64);
  x += __shfl_xor(x, 32, 64);
  return x;
}

// K rows of tile buffer lk as A operands (shared by the query tiles)
__device__ inline void load_ka(const char* lk, int i16, int g4, u4 (&ka)[8]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    ka[k] = *reinterpret_cast<const u4*>(lk + toff(i16, k * 4 + g4));
    ka[4 + k] = *reinterpret_cast<const u4*>(lk + toff(16 + i16, k * 4 + g4));
  }
}

// S^T = K Q^T of one tile for one query tile
__device__ inline void qt_scores(const u4 (&ka)[8], const u4 (&q)[4], f4& s0, f4& s1) {
  s0 = f4{0.f, 0.f, 0.f, 0.f};
  s1 = s0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    s0 = mfma(ka[k], q[k], s0);
    s1 = mfma(ka[4 + k], q[k], s1);
  }
}

// S^T = K Q^T of one tile for every query tile of the wave
template <int QT>
__device__ inline void tile_scores(const u4 (&ka)[8], const u4 (&qop)[QT][4], f4 (&s)[QT][2]) {
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) qt_scores(ka, qop[qt], s[qt][0], s[qt][1]);
}

// O^T += V^T P of one tile (V^T operands read from the tile's LDS V rows)
template <bool F16, int QT>
__device__ inline void tile_pv(const char* lv, const POp (&pp)[QT], QState (&st)[QT], int i16,
                               int g4) {
  const char* vb = vt_base(lv, i16, g4);
#pragma unroll
  for (int d = 0; d < 8; ++d) {
    const u4 vt = vt_operand_at(vb, d);
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      if (F16) {
        st[qt].acc[d] = mfma_f16(vt, pp[qt].hi, st[qt].acc[d]);
      } else {
        st[qt].acc[d] = mfma(vt, pp[qt].hi, st[qt].acc[d]);
        st[qt].acc[d] = mfma(vt, pp[qt].lo, st[qt].acc[d]);
      }
    }
  }
}

// Scheduling of one pipeline iteration: N matrix instructions, each followed
// by its even share of about NV vector instructions.
template <int N, int NV, int I = 0>
__device__ inline void interleave() {
  if constexpr (I < N) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
    constexpr int v = (I + 1) * NV / N - I * NV / N;
    if constexpr (v > 0) __builtin_amdgcn_sched_group_barrier(0x002, v, 0);  // VALU
    interleave<N, NV, I + 1>();
  }
}

// One iteration of the pipeline (tile t): scores of tile t+1 and, with PV,
// O += V^T P of tile t-1 (operands pp) on the matrix cores, interleaved with
// the softmax common path of tile t on the vector ALUs; then the rare
// reference raise (which recomputes tile t's scores from its K rows, still in
// LDS, so the scores need not stay in registers) and the running sums.  A
// tile that a view's end leaves partial takes the rare path too, which masks
// it.  sc holds tile t's scores on entry and tile t+1's on exit; tile t's
// probability operands go to pn (the caller alternates two sets, so they
// are never copied).
template <bool F16, int TPS, bool PV, int QT>
__device__ __attribute__((always_inline)) inline void tile_step(
    int t, char* lds, const u4 (&qop)[QT][4], QState (&st)[QT], f4 (&sc)[QT][2],
    const POp (&pp)[QT], POp (&pn)[QT], float scale_log2, int n_valid, int i16, int g4) {
  float psum[QT];
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    float e[8];
    psum[qt] = tile_exp(st[qt], sc[qt][0], sc[qt][1], scale_log2, e);
    pn[qt] = pack_p<F16>(e);
  }
  {
    u4 ka[8];
    load_ka(tile_buf<TPS>(lds, t + 1), i16, g4, ka);
    tile_scores(ka, qop, sc);
  }
  if (PV) tile_pv<F16, QT>(tile_buf<TPS>(lds, t - 1) + TILEB, pp, st, i16, g4);
  // matrix and vector instructions in turn (the softmax takes about 26
  // vector instructions per query tile, 30 with the bf16 split)
  interleave<QT * 8 + (PV ? QT * 8 * (F16 ? 1 : 2) : 0), QT * (F16 ? 26 : 30)>();
  bool rare = false;
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) rare = rare || !(psum[qt] <= kLazyExp);
  if (n_valid < TILE) rare = true;
  if (__builtin_amdgcn_ballot_w64(rare)) {  // rare: mask, raise the reference max
#pragma unroll
    for (int qt = 0; qt < QT; ++qt)
      if (n_valid < TILE || __builtin_amdgcn_ballot_w64(!(psum[qt] <= kLazyExp))) {
        u4 ka[8];
        load_ka(tile_buf<TPS>(lds, t), i16, g4, ka);
        f4 s0, s1;
        qt_scores(ka, qop[qt], s0, s1);
        if (n_valid < TILE) tile_mask(s0, s1, n_valid);
        float e[8];
        psum[qt] = tile_exp(st[qt], s0, s1, scale_log2, e);
        if (__builtin_amdgcn_ballot_w64(!(psum[qt] <= kLazyExp)))
          psum[qt] = tile_raise(st[qt], s0, s1, scale_log2, e);
        pn[qt] = pack_p<F16>(e);
      }
  }
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    st[qt].l += psum[qt];
    st[qt].ls += psum[qt];
  }
}

// the key-tile loop of one workgroup over all tiles or those of its key split
// (see the file comment).  Returns the view of the last tile.
template <bool F16, int W, int TPS, int QT, bool SPLIT>
__device__ __attribute__((always_inline)) inline int tile_loop(
    const Views& vs, const Split& sp, int split, int bh, char* lds, const u4 (&qop)[QT][4],
    QState (&st)[QT], float scale_log2, int r_wave, int nq, int64_t qbase, int nseg,
    float* seg_lse, int i16, int g4) {
  int cur_view = -1, cur_seg = -1;
  const int t_first = SPLIT ? split * sp.per : 0;
  const int T = SPLIT ? min(sp.per, vs.tiles - t_first) : vs.tiles;
  // tiles go through LDS in stages of TPS: stage j holds tiles TPS*j ..
  // TPS*j + TPS - 1; after the last tile of stage j the tiles of stage j + 2
  // are stored, and one barrier per stage publishes them.  During stage j
  // the pipeline reads stages j - 1 .. j + 1.  With two tiles per stage the
  // tiles of stage j + 2 are loaded at the start of stage j; with one, tile
  // t + 3 is loaded at the start of iteration t into the other of two
  // register sets, so a load has two iterations to arrive.
  constexpr int NT = W * 64;
  Cursor<F16> ct, cs;  // tile t (computed) and the next tile to stage
  Stage SA, SB;
  // the sequence's first tile, whose maxima a later split starts from, goes to
  // the last stage (first needed for tile 3)
  static_assert(!SPLIT || (TPS == 1 && STAGES == 4), "the last stage is free at the start");
  char* const first = tile_buf<TPS>(lds, STAGES - 1);
  {
    Stage S;
    if (SPLIT && t_first > 0) {
      cs.start(vs, bh, 0);
      stage_load<F16, NT, false>(cs, SA, 0);
      stage_load<F16, NT, false>(cs, SA, 1);
    }
    ct.start(vs, bh, t_first);
    cs.start(vs, bh, t_first);
    for (int u = 0; u < 2 * TPS && u < T; ++u) {
      // the chunks of tile u (both with one tile per stage)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (TPS == 1 || i == 0) stage_load<F16, NT>(cs, S, i);
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (TPS == 1 || i == 0) stage_store<NT>(tile_buf<TPS>(lds, u), S, i);
      cs.next(vs, bh);
    }
    if (SPLIT && t_first > 0) {
      stage_store<NT, false>(first, SA, 0);
      stage_store<NT, false>(first, SA, 1);
    }
    if (TPS == 1 && T > 2) {
      stage_load<F16, NT>(cs, SA, 0);
      stage_load<F16, NT>(cs, SA, 1);
      cs.next(vs, bh);
    }
  }
  __syncthreads();
  f4 sc[QT][2];
  if (SPLIT && t_first > 0) {
    u4 ka[8];
    load_ka(first, i16, g4, ka);
    tile_scores(ka, qop, sc);
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      float p[8];
      tile_mask(sc[qt][0], sc[qt][1], vs.v[0].n);
      tile_logits(sc[qt][0], sc[qt][1], p);
      st[qt].m = fmaxf(st[qt].m, column_max(p, scale_log2));
    }
  }
  {
    u4 ka[8];
    load_ka(tile_buf<TPS>(lds, 0), i16, g4, ka);
    tile_scores(ka, qop, sc);
  }
  POp pa[QT], pb[QT];  // probability operands of alternate tiles
  int n_pre = 0;  // tiles of the stage in flight (two tiles per stage)
  // one iteration (PV of tile t-1 from pp, P of tile t into pn; with one
  // tile per stage, tile t+2 stored from Sc and tile t+3 loaded into Sn);
  // the first (no previous tile to multiply with V) is peeled
  auto iter = [&](int t, auto pv, const POp (&pp)[QT], POp (&pn)[QT], Stage& Sc, Stage& Sn) {
    if (TPS == 1) {
      if (t + 3 < T) {
        stage_load<F16, NT>(cs, Sn, 0);
        stage_load<F16, NT>(cs, Sn, 1);
        cs.next(vs, bh);
      }
    } else if (t % TPS == 0 && t + 2 * TPS < T) {  // the tiles of stage t/TPS + 2
      stage_load<F16, NT>(cs, Sn, 0);
      cs.next(vs, bh);
      n_pre = 1;
      if (t + 2 * TPS + 1 < T) {
        stage_load<F16, NT>(cs, Sn, 1);
        cs.next(vs, bh);
        n_pre = 2;
      }
    }
    const int vi = ct.vi;
    const int n_valid = min(TILE, ct.n - ct.row0);
    if (seg_lse && vi != cur_view && cur_view >= 0 && ct.seg != cur_seg) {
      // the previous logical segment ended: its log-sum-exp per query row
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        const float ls = col_sum(st[qt].ls);
        const int r = r_wave + qt * 16 + i16;
        if (g4 == 0 && r < nq)
          seg_lse[(SPLIT ? (qbase + r) * sp.n + split : qbase + r) * nseg + cur_seg] =
              ls > 0.0f ? (st[qt].m + __log2f(ls)) * kLn2 : -INFINITY;
        st[qt].ls = 0.0f;
      }
    }
    cur_view = vi;
    cur_seg = ct.seg;
    ct.next(vs, bh);
    // past the last tile the next scores come from a stale buffer and are
    // never used
    tile_step<F16, TPS, decltype(pv)::value, QT>(t, lds, qop, st, sc, pp, pn, scale_log2,
                                                 n_valid, i16, g4);
    if (t % TPS == TPS - 1 || t == T - 1) {  // the stage's last tile
      const int t0 = t - t % TPS + 2 * TPS;  // first tile of the staged stage
      if (TPS == 1) {
        if (t0 < T) {
          stage_store<NT>(tile_buf<TPS>(lds, t0), Sc, 0);
          stage_store<NT>(tile_buf<TPS>(lds, t0), Sc, 1);
        }
      } else {  // Sc and Sn are the same set
        if (n_pre >= 1) stage_store<NT>(tile_buf<TPS>(lds, t0), Sc, 0);
        if (n_pre >= 2) stage_store<NT>(tile_buf<TPS>(lds, t0 + 1), Sc, 1);
      }
      n_pre = 0;
      __syncthreads();
    }
  };
  // with two tiles per stage both register-set roles are SA
  Stage& S1 = TPS == 1 ? SB : SA;
  iter(0, std::false_type{}, pb, pa, SA, S1);
  int t = 1;
  for (; t + 1 < T; t += 2) {
    iter(t, std::true_type{}, pa, pb, S1, SA);
    iter(t + 1, std::true_type{}, pb, pa, SA, S1);
  }
  // the last tile's O += V^T P
  if (t < T) {
    iter(t, std::true_type{}, pa, pb, S1, SA);
    tile_pv<F16, QT>(tile_buf<TPS>(lds, T - 1) + TILEB, pb, st, i16, g4);
  } else {
    tile_pv<F16, QT>(tile_buf<TPS>(lds, T - 1) + TILEB, pa, st, i16, g4);
  }
  return cur_view;
}

template <int W, int TPS, int QT, bool SPLIT>
__global__ __launch_bounds__(W * 64, W == 4 && QT == 2 ? 2 : 1) void prefill_mfma_kernel(Views vs, const uint16_t* __restrict__ q,
                                                              int Hq, int Hkv, int M, int nseg,
                                                              int n_qblocks, int n_work,
                                                              float scale_log2, float* __restrict__ o,
                                                              float* __restrict__ lse,
                                                              float* __restrict__ seg_lse,
                                                              Split sp,
                                                              const uint32_t* __restrict__ flags) {
  __shared__ __attribute__((aligned(16))) char lds[STAGES * TPS * SUBB];
  // XCD-aware work mapping: consecutive work items (the query blocks of one
  // head, which share its K/V rows) go to the same XCD
  const int per_xcd = (n_work + 7) / 8;
  const int work = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (work >= n_work) return;
  // the query blocks of one key split of one head are consecutive
  const int qb = work % n_qblocks, hs = work / n_qblocks;
  const int split = SPLIT ? hs % sp.n : 0, bh = SPLIT ? hs / sp.n : hs;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i16 = lane & 15, g4 = lane >> 4;
  const int G = Hq / Hkv, nq = G * M, b = bh / Hkv, hkv = bh % Hkv;
  const int64_t qbase = ((int64_t)b * Hq + hkv * G) * M;  // first query row of the head
  const int r_wave = qb * qrows<W, QT>() + wave * QT * 16;  // first row of the wave

  u4 qop[QT][4];
  QState st[QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const int r = r_wave + t * 16 + i16;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      qop[t][k] = r < nq ? *reinterpret_cast<const u4*>(q + (qbase + r) * D + k * 32 + g4 * 8)
                         : u4{0, 0, 0, 0};
    st[t].m = -INFINITY;
    st[t].l = 0.0f;
    st[t].ls = 0.0f;
#pragma unroll
    for (int d = 0; d < 8; ++d) st[t].acc[d] = f4{0.f, 0.f, 0.f, 0.f};
  }

  // segments without rows never see a tile: their log-sum-exp stays -inf
  if (seg_lse && g4 == 0) {
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      const int r = r_wave + t * 16 + i16;
      if (r < nq)
        for (int a = 0; a < nseg; ++a)
          seg_lse[(SPLIT ? (qbase + r) * sp.n + split : qbase + r) * nseg + a] = -INFINITY;
    }
  }
  // did any workgroup of the preparation meet a V value outside fp16's range
  // (scalar loads: the flags as a vector register cost the tile loop 3 %)
  uint32_t unsafe_v = 0;
#pragma unroll
  for (int i = 0; i < kPrepBlocks / 4; ++i) unsafe_v |= flags[i];
  const bool f16 = unsafe_v == 0;
  const int cur_view =
      f16 ? tile_loop<true, W, TPS, QT, SPLIT>(vs, sp, split, bh, lds, qop, st, scale_log2, r_wave,
                                               nq, qbase, nseg, seg_lse, i16, g4)
          : tile_loop<false, W, TPS, QT, SPLIT>(vs, sp, split, bh, lds, qop, st, scale_log2, r_wave,
                                                nq, qbase, nseg, seg_lse, i16, g4);
  // outputs
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    const int r = r_wave + qt * 16 + i16;
    const float l = col_sum(st[qt].l);
    const float ls = col_sum(st[qt].ls);
    if (r < nq) {
      const int64_t rec = SPLIT ? (qbase + r) * sp.n + split : qbase + r;
      const float inv = SPLIT ? 1.0f : 1.0f / l;
      float* orow = (SPLIT ? sp.o : o) + rec * D;
#pragma unroll
      for (int d = 0; d < 8; ++d) *reinterpret_cast<f4*>(orow + d * 16 + g4 * 4) = st[qt].acc[d] * inv;
      if (g4 == 0) {
        if (SPLIT) *reinterpret_cast<f2*>(sp.ml + rec * 2) = f2{st[qt].m, l};
        else if (lse) lse[rec] = (st[qt].m + __log2f(l)) * kLn2;
        if (seg_lse && cur_view >= 0)
          seg_lse[rec * nseg + vs.v[cur_view].seg] =
              ls > 0.0f ? (st[qt].m + __log2f(ls)) * kLn2 : -INFINITY;
      }
    }
  }
}

// One wave per query row: its n records merged into O (each lane two dims),
// lse and the per-segment lse.  Eight records are loaded at a time, all before
// any is used; a record's m is at least the first tile's maximum, so it is
// finite.
__global__ __launch_bounds__(256) void split_merge_kernel(int Q, int n, int nseg, Split sp,
                                                          float* __restrict__ o,
                                                          float* __restrict__ lse,
                                                          float* __restrict__ seg_lse) {
  const int64_t qi = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (qi >= Q) return;
  const int lane = threadIdx.x & 63;
  const float* ml = sp.ml + qi * n * 2;
  const float* po = sp.o + qi * n * D + 2 * lane;
  float M = -INFINITY, l = 0.0f;
  f2 acc = f2{0.0f, 0.0f};
  for (int s0 = 0; s0 < n; s0 += 8) {
    f2 a[8], x[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int s = min(s0 + r, n - 1);
      a[r] = *reinterpret_cast<const f2*>(ml + 2 * s);
      x[r] = *reinterpret_cast<const f2*>(po + (int64_t)s * D);
    }
    float mx = M;
#pragma unroll
    for (int r = 0; r < 8; ++r) mx = fmaxf(mx, a[r][0]);
    const float c = __builtin_amdgcn_exp2f(M - mx);
    l *= c;
    acc *= c;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const float w = s0 + r < n ? __builtin_amdgcn_exp2f(a[r][0] - mx) : 0.0f;
      l = fmaf(w, a[r][1], l);
      acc[0] = fmaf(w, x[r][0], acc[0]);
      acc[1] = fmaf(w, x[r][1], acc[1]);
    }
    M = mx;
  }
  *reinterpret_cast<f2*>(o + qi * D + 2 * lane) = acc * (1.0f / l);
  if (lse && lane == 0) lse[qi] = (float)(((double)M + (double)log2f(l)) * kLn2d);
  if (seg_lse && lane < nseg) {
    const float* ps = sp.seg + qi * n * nseg + lane;
    float m = -INFINITY, t = 0.0f;
    for (int s = 0; s < n; ++s) m = fmaxf(m, ps[s * nseg]);
    if (m != -INFINITY)
      for (int s = 0; s < n; ++s) t += expf(ps[s * nseg] - m);
    seg_lse[qi * nseg + lane] = m == -INFINITY ? m : m + logf(t);
  }
}

// 8 channels (column chunk c8) of row r of head bh of a packed segment:
// round_to_bf16(fmaf(code, scale, min)), the 8 codes in one 16-, 32- or
// 64-bit load, the key scales and minima in 16-byte loads, one value group
// (groups are at least 8 channels)
__device__ inline void dequant8(const KSeg& s, int bh, int r, int c8, u4& ko, u4& vo) {
  int bits;
  int64_t off;
  if (!head_codes(s, bh, D, bits, off) || (off & 15)) {
    const uint32_t nan2 = 0x7FC07FC0u;
    ko = u4{nan2, nan2, nan2, nan2};
    vo = ko;
    return;
  }
  const int rb = D * bits / 8, lgG = __builtin_ctz((unsigned)s.group);
  const int64_t cb = off + (int64_t)r * rb + c8 * bits;  // 8 channels = bits bytes
  uint64_t wk, wv;
  if (bits == 4) {
    wk = *reinterpret_cast<const uint32_t*>(s.codes_k + cb);
    wv = *reinterpret_cast<const uint32_t*>(s.codes_v + cb);
  } else if (bits == 2) {
    wk = *reinterpret_cast<const uint16_t*>(s.codes_k + cb);
    wv = *reinterpret_cast<const uint16_t*>(s.codes_v + cb);
  } else {
    wk = *reinterpret_cast<const uint64_t*>(s.codes_k + cb);
    wv = *reinterpret_cast<const uint64_t*>(s.codes_v + cb);
  }
  const int mask = (1 << bits) - 1;
  const int64_t kg = ((int64_t)bh * s.kgroups + (r >> lgG)) * D + c8 * 8;
  const f4 sk0 = *reinterpret_cast<const f4*>(s.scale_k + kg);
  const f4 sk1 = *reinterpret_cast<const f4*>(s.scale_k + kg + 4);
  const f4 mk0 = *reinterpret_cast<const f4*>(s.min_k + kg);
  const f4 mk1 = *reinterpret_cast<const f4*>(s.min_k + kg + 4);
  const float sk[8] = {sk0[0], sk0[1], sk0[2], sk0[3], sk1[0], sk1[1], sk1[2], sk1[3]};
  const float mk[8] = {mk0[0], mk0[1], mk0[2], mk0[3], mk1[0], mk1[1], mk1[2], mk1[3]};
  const int64_t vi = ((int64_t)bh * s.cap_full + r) * (D >> lgG) + ((c8 * 8) >> lgG);
  const float sv = s.scale_v[vi], mv = s.min_v[vi];
  uint32_t kw[4], vw[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int c0 = 2 * j, c1 = 2 * j + 1;
    const float k0 = fmaf((float)((wk >> (c0 * bits)) & mask), sk[c0], mk[c0]);
    const float k1 = fmaf((float)((wk >> (c1 * bits)) & mask), sk[c1], mk[c1]);
    const float v0 = fmaf((float)((wv >> (c0 * bits)) & mask), sv, mv);
    const float v1 = fmaf((float)((wv >> (c1 * bits)) & mask), sv, mv);
    kw[j] = bf2(k0, k1);
    vw[j] = bf2(v0, v1);
  }
  ko = u4{kw[0], kw[1], kw[2], kw[3]};
  vo = u4{vw[0], vw[1], vw[2], vw[3]};
}

// Preparation of a call in one launch: for every view, either the dequantised
// rows of a packed segment (bf16 K and V, fp16 V) or the fp16 copy of a dense
// view's V rows (round to nearest even).  A workgroup that meets a V value
// with no fp16 counterpart says so in its own flag byte, which the attention
// kernel reads, so no flag has to be cleared by a launch before this one.
// (A clearing kernel, a dequantisation and one conversion per dense view were
// four launches of 2 to 8 us each for a prompt of 203 rows over 6144; this one
// takes 8 us.  Two items per thread and pass: 11 us.)
struct PrepView {
  const uint16_t* src;  // dense: V rows of (b, h_kv) 0; packed: NULL
  uint16_t *kd, *vd;    // packed: dequantised rows
  uint16_t* vh;
  int64_t bh_stride;    // dense: elements between heads of src
  int n, seg;           // rows per head, segment (packed)
};
struct Prep {
  PrepView v[kMaxViews];
  int n, BH;
};

__global__ __launch_bounds__(kPrepThreads) void prepare_kernel(KSegs segs, Prep p,
                                                               uint8_t* __restrict__ flags) {
  bool over = false;
  for (int i = 0; i < p.n; ++i) {
    const PrepView& w = p.v[i];
    const int64_t items = (int64_t)p.BH * w.n * (D / 8);
    for (int64_t e = (int64_t)blockIdx.x * kPrepThreads + threadIdx.x; e < items;
         e += (int64_t)kPrepBlocks * kPrepThreads) {
      const uint32_t rr = (uint32_t)(e / (D / 8));  // fewer than 2^32 rows fit any memory
      const int c8 = (int)(e % (D / 8));
      const uint32_t bh = rr / (uint32_t)w.n, r = rr % (uint32_t)w.n;
      const int64_t oi = (int64_t)rr * D + c8 * 8;
      u4 vo;
      if (w.src) {
        vo = *reinterpret_cast<const u4*>(w.src + bh * w.bh_stride + (int64_t)r * D + c8 * 8);
      } else {
        u4 ko;
        dequant8(segs.s[w.seg], (int)bh, (int)r, c8, ko, vo);
        *reinterpret_cast<u4*>(w.kd + oi) = ko;
        *reinterpret_cast<u4*>(w.vd + oi) = vo;
      }
      *reinterpret_cast<u4*>(w.vh + oi) =
          u4{bf2_to_h2(vo[0]), bf2_to_h2(vo[1]), bf2_to_h2(vo[2]), bf2_to_h2(vo[3])};
      over = over || bf2_over_f16(vo[0]) || bf2_over_f16(vo[1]) || bf2_over_f16(vo[2]) ||
             bf2_over_f16(vo[3]);
    }
  }
  const int any = __syncthreads_or(over);
  if (threadIdx.x == 0) flags[blockIdx.x] = any != 0;
}

}  // namespace

bool prefill_mfma_eligible(const uc_shape& sh, const KSegs& segs, int q_dt, int M) {
  if (sh.D != D || q_dt != UC_BF16) return false;
  if ((sh.Hq / sh.Hkv) * M <= 16) return false;  // the decode kernel's range
  for (int i = 0; i < segs.n; ++i)
    if (segs.s[i].dtype != UC_BF16) return false;
  return true;
}

// Key splits of a call: none when its query blocks fill half of the resident
// workgroups (two per CU of the four-wave layout), else as many as fill them,
// each of at least kSplitTiles key tiles.  The count never falls as rows are
// added.  Measured, 203 query rows of 28 heads on 4 KV heads over 6144 rows (48
// query blocks), attention kernel alone: 148 us unsplit, 45 with 5 splits, 42
// with 8, 38 with 10 (the rule), 42 with 16.  Grids that already fill the chip
// lose: 1792 query blocks (3.5 rounds) 760 us unsplit, 1133 with 16.  Calls
// over fewer than 32 tiles are not split: a tile takes about 0.77 us, the merge
// and its records about 8 us, and calls of 24 and 30 us became 6 and 5 % slower.
constexpr int kSplitTiles = 8, kMinTiles = 32, kMaxSplits = 16;

static int64_t narrow_blocks(const uc_shape& sh, int M) {
  const int64_t nq = (int64_t)(sh.Hq / sh.Hkv) * M;
  return (nq + qrows<4, 2>() - 1) / qrows<4, 2>() * sh.B * sh.Hkv;
}

static int prefill_splits(const uc_shape& sh, int tiles, int M) {
  if (tiles < kMinTiles) return 1;
  const int64_t blocks = narrow_blocks(sh, M);
  const int64_t n = std::min<int64_t>({2 * device_cus() / blocks, tiles / kSplitTiles, kMaxSplits});
  return (int)std::max<int64_t>(n, 1);
}

static size_t split_bytes(const uc_shape& sh, int M, int n_segs) {  // of one split
  return (size_t)sh.B * sh.Hq * M * (D + 2 + n_segs) * sizeof(float);
}

static size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }

// Workspace: the preparation's flags (one byte per workgroup), then bf16 K
// and V plus fp16 V of every packed segment's whole row groups, and the fp16
// V copy of every dense view (dense segments, residual tails); then the
// records of the key splits.  A call runs with the first part alone
// (unsplit); the size reported to callers holds the records too.
size_t prefill_mfma_min_workspace(const uc_shape& sh, const KSegs& segs) {
  const size_t BH = (size_t)sh.B * sh.Hkv;
  size_t bytes = kPrepBlocks;
  for (int i = 0; i < segs.n; ++i) {
    const KSeg& s = segs.s[i];
    if (s.kind == UC_SEG_PACKED) {
      bytes += round256(BH * s.n_full * D * 2 * 3);
      bytes += round256(BH * s.tail_len * D * 2);
    } else {
      bytes += round256(BH * s.n_rows * D * 2);
    }
  }
  return bytes;
}

size_t prefill_mfma_workspace(const uc_shape& sh, const KSegs& segs, int M) {
  // tiles: every view rounds up, so one more than a segment's rows give
  // bounds it, and the bound grows with the rows
  int64_t tiles = 0;
  for (int i = 0; i < segs.n; ++i) tiles += segs.s[i].n_rows / TILE + 2;
  const int n = prefill_splits(sh, (int)std::min<int64_t>(tiles, INT32_MAX), M);
  return prefill_mfma_min_workspace(sh, segs) + (n > 1 ? round256(n * split_bytes(sh, M, segs.n)) : 0);
}

static_assert(sizeof(Views) <= kPrefillViewBytes, "prepared views do not fit their slot");

// Preparation of a call: the range flags, the dequantised rows of every
// packed segment and the fp16 V copies, all in ws; the views the attention
// kernel walks go to views_out (kPrefillViewBytes).  The result depends only
// on the segments' contents and ws, so calls over unchanged segments can
// reuse it (execution plans).
hipError_t launch_prefill_prepare(const uc_shape& sh, const KSegs& segs, void* ws, hipStream_t st,
                                  void* views_out) {
  const int BH = sh.B * sh.Hkv;
  Views vs{};
  Prep pr{};
  pr.BH = BH;
  char* wp = (char*)ws + kPrepBlocks;
  auto take = [&](size_t bytes) {
    char* p = wp;
    wp += round256(bytes);
    return (uint16_t*)p;
  };
  // views without rows are left out (their tiles would be empty)
  auto add = [&](const View& v, uint16_t* kd, uint16_t* vd) {
    if (v.n == 0) return;
    pr.v[vs.n] = PrepView{kd ? nullptr : v.v, kd, vd, (uint16_t*)v.vh, v.bh_stride, v.n, v.seg};
    vs.v[vs.n++] = v;
    vs.tiles += (v.n + TILE - 1) / TILE;
  };
  for (int i = 0; i < segs.n; ++i) {
    const KSeg& s = segs.s[i];
    if (s.kind == UC_SEG_DENSE) {
      add(View{(const uint16_t*)s.k, (const uint16_t*)s.v, take((size_t)BH * s.n_rows * D * 2),
               (int64_t)s.row_stride * D, s.n_rows, i}, nullptr, nullptr);
      continue;
    }
    const size_t head = (size_t)BH * s.n_full * D;
    uint16_t* kd = take(head * 2 * 3);
    add(View{kd, kd + head, kd + 2 * head, (int64_t)s.n_full * D, s.n_full, i}, kd, kd + head);
    uint16_t* th = take((size_t)BH * s.tail_len * D * 2);
    add(View{(const uint16_t*)s.tail_k, (const uint16_t*)s.tail_v, th, (int64_t)s.tail_stride * D,
             s.tail_len, i}, nullptr, nullptr);
  }
  pr.n = vs.n;
  hipLaunchKernelGGL(prepare_kernel, dim3(kPrepBlocks), dim3(kPrepThreads), 0, st, segs, pr,
                     (uint8_t*)ws);
  memcpy(views_out, &vs, sizeof vs);
  return hipGetLastError();
}

// The attention kernel over prepared views (launch_prefill_prepare on ws, which
// is only read here).  The records of key splits take rec_bytes at rec: without
// room for two splits there are none.
hipError_t launch_prefill_run(const uc_shape& sh, int n_segs, const void* views, const void* q,
                              int M, float sm_scale, float* o, float* lse, float* seg_lse,
                              const void* ws, void* rec, size_t rec_bytes, hipStream_t st) {
  Views vs;
  memcpy(&vs, views, sizeof vs);
  const int BH = sh.B * sh.Hkv;
  const uint32_t* flags = (const uint32_t*)ws;
  hipError_t e;
  const int nq = (sh.Hq / sh.Hkv) * M;
  // the 8-wave layout (one workgroup per CU) when its grid fills every round
  // or runs many rounds; otherwise the 4-wave one (two per CU), whose last
  // round leaves fewer CUs idle
  const int cus = device_cus();
  const int n8 = (nq + qrows<8, 2>() - 1) / qrows<8, 2>() * BH;
  const bool wide = n8 % cus == 0 || n8 >= 8 * cus;
  const int qr = wide ? qrows<8, 2>() : qrows<4, 2>();
  const int n_qblocks = (nq + qr - 1) / qr;
  Split sp{1, vs.tiles, nullptr, nullptr, nullptr};
  if (!wide) {
    const size_t room = rec_bytes / split_bytes(sh, M, n_segs);
    const int n = (int)std::min<size_t>(prefill_splits(sh, vs.tiles, M), room);
    if (n > 1) {
      sp.per = (vs.tiles + n - 1) / n;
      sp.n = (vs.tiles + sp.per - 1) / sp.per;
      const int64_t recs = (int64_t)sh.B * sh.Hq * M * sp.n;
      sp.o = (float*)rec;
      sp.ml = sp.o + recs * D;
      sp.seg = sp.ml + recs * 2;
    }
  }
  const int n_work = n_qblocks * BH * sp.n;
  const int grid = (n_work + 7) / 8 * 8;
  const float sl2 = sm_scale * kLog2e;
  const uint16_t* qp = (const uint16_t*)q;
  float* seg = sp.n > 1 && seg_lse ? sp.seg : seg_lse;
  if ((e = kernel_timer_begin(st)) != hipSuccess) return e;
  auto go = [&](auto kernel, int waves) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(waves * 64), 0, st, vs, qp, sh.Hq, sh.Hkv, M, n_segs,
                       n_qblocks, n_work, sl2, o, lse, seg, sp, flags);
  };
  if (wide) go(prefill_mfma_kernel<8, 2, 2, false>, 8);
  else if (sp.n == 1) go(prefill_mfma_kernel<4, 1, 2, false>, 4);
  else go(prefill_mfma_kernel<4, 1, 2, true>, 4);
  e = hipGetLastError();
  if (e == hipSuccess) e = kernel_timer_end(st);
  if (e != hipSuccess || sp.n == 1) return e;
  const int Q = sh.B * sh.Hq * M;
  hipLaunchKernelGGL(split_merge_kernel, dim3((Q + 3) / 4), dim3(256), 0, st, Q, sp.n, n_segs, sp, o,
                     lse, seg_lse);
  return hipGetLastError();
}

hipError_t launch_prefill_mfma(const uc_shape& sh, const KSegs& segs, const void* q, int M,
                               float sm_scale, float* o, float* lse, float* seg_lse, void* ws,
                               size_t ws_bytes, hipStream_t st) {
  alignas(16) char views[kPrefillViewBytes];
  const hipError_t e = launch_prefill_prepare(sh, segs, ws, st, views);
  if (e != hipSuccess) return e;
  const size_t min = prefill_mfma_min_workspace(sh, segs);
  return launch_prefill_run(sh, segs.n, views, q, M, sm_scale, o, lse, seg_lse, ws, (char*)ws + min,
                            ws_bytes - min, st);
}

}  // namespace uc
