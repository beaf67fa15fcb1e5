// score_mfma.hip -- attention-guided importance scores on the CDNA4 matrix
// cores (Sec. 3.2, Eq. 1 and App. E, "Batched GQA token selection": the
// attention probability each cached token receives from the observation
// queries, summed over the query heads that share its KV head).
//
// For one KV head the observation block is the G*W query rows of its query
// heads (row g*W + w is head h_kv*G + g, position w; these rows are
// contiguous in q).  Softmax normalises each query row over every key of
// every segment, so the scores take two passes over the keys:
//   pass 1  per (key chunk, query block of <= 256 rows, b*h_kv): running
//           reference and sum of exp2 per query row over the chunk's keys, one
//           (m, l) record per (row, chunk); launch_score_norm merges the
//           records into the row normalisers (M, 1/l).
//   pass 2  per (key chunk, b*h_kv): p = exp2(s - M) / l for every query row,
//           summed over the rows per key (column sums), for the query blocks
//           of a group; the per-key sums are written as the scores and
//           their total is the chunk's probability mass (Eq. 1 bracket).
// Both passes compute S^T = K Q^T with v_mfma_f32_16x16x32_bf16: a wave
// takes pairs of 32-key tiles of the chunk (keys straight from HBM into the
// A-operand layout; packed rows decoded in registers to their stored bf16
// values) and runs each pair against every 16-row query tile of the block,
// whose B operands it reads from the block staged in LDS.  The next pair is
// loaded while the current one is computed (but for packed rows in pass 2,
// whose registers would spill).  Logits are in base 2 (q.k times
// scale*log2(e)).
// Row normalisers: a record is (m, l), l the sum of exp2(s - m), with m a
// reference that is at most kLazy below the row's maximum; the records of a
// row merge to (M, 1/l) and a probability is exp2(s - M) * (1/l), so no
// log-sum-exp is rounded to binary32 on the way (its rounding, and that of
// the change of base, was the largest error of the scores: 5.5e-7 to 1e-6
// against 64 bits on 64k rows with heavy-tailed keys).
// Column sums: a lane sums its key's probabilities over the query tiles in
// fp32, the 16 query columns of a tile are added across lanes, and the
// query blocks are accumulated in fp64 in LDS; chunk masses are fp64.
// Bound: the vector ALU.  Per 16 logits a lane spends 16 v_exp_f32 (two issue
// slots each), 16 v_fma for the argument, 16 adds and, in pass 1, about 25
// instructions of row bookkeeping, beside 16 matrix instructions.  One MI355X,
// passes 1 and 2: 16 x 65536 keys x 4 heads, 224 rows 369 and 352 us before,
// 353 and 291 now; 2 x 9216 keys x 4 heads, 28672 rows 741 and 1002, 741 and 648 now.
#include <algorithm>

#include "mfma_util.h"
#include "uc_common.h"

namespace uc {
namespace {

using namespace mf;

constexpr int WAVES = 4;
constexpr int TPW = 2;                   // key tiles per wave and step
constexpr int SUB = WAVES * TPW * TILE;  // 256 keys per step (K held in registers, the next step's in flight)
constexpr int CHUNK = 4 * SUB;           // keys per workgroup
constexpr int QB = 256;                  // query rows per block (16 tiles)
constexpr int QT = QB / 16;
constexpr int QROW = D * 2 + 16;         // bytes of one staged query row (16 B padding)
constexpr float kLazy = 8.0f;            // a row's reference may trail its maximum by this (base 2)

// A wave's key tiles of a step as A operands: k[i][blk*4 + t] = row (tile i)
// blk*16 + i16, dims t*32 + g4*8 .. +7.  Rows past the descriptor's end read
// as zeros.
struct KTiles {
  u4 k[TPW][8];
};

__device__ inline void k_issue(__amdgpu_buffer_rsrc_t rk, int row0, int lane, u4 (&k)[8]) {
  const int i16 = lane & 15, g4 = lane >> 4;
  const int ko = (row0 + i16) * ROWB + g4 * 16;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    k[t] = bload(rk, ko + t * 64);
    k[4 + t] = bload(rk, ko + 16 * ROWB + t * 64);
  }
}

// Where one (b, h_kv)'s key rows of a segment come from: dense rows, or
// (packed) code rows 0 .. n_full-1 decoded in registers and residual-tail
// rows n_full .. read as stored.  n_full is a multiple of the group G >= 32,
// so a 32-row tile is all codes or all tail, and a code tile lies inside one
// key group (one scale and minimum per channel).
struct KSrc {
  __amdgpu_buffer_rsrc_t rk;   // dense rows, or the tail rows of a packed segment
  __amdgpu_buffer_rsrc_t rc;   // packed: this head's code rows
  const float* sk;             // packed: this head's key scales [groups, D]
  const float* mk;             // packed: this head's key minima
  int n_full, bits, G;         // n_full = 0 for dense segments
  bool bad;                    // packed head whose device-side layout is invalid
};

__device__ inline KSrc k_source(const KSeg& ks, int bh, int r1) {
  KSrc src{};
  if (ks.kind == UC_SEG_DENSE) {
    const int64_t base = (int64_t)bh * ks.row_stride * D;
    src.rk = rsrc((const uint16_t*)ks.k + base, (uint32_t)r1 * ROWB);
    return src;
  }
  src.n_full = ks.n_full;
  src.G = ks.group;
  const int64_t tb = (int64_t)bh * ks.tail_stride * D;
  src.rk = rsrc((const uint16_t*)ks.tail_k + tb, (uint32_t)max(0, r1 - ks.n_full) * ROWB);
  int bits;
  int64_t off;
  src.bad = !head_codes(ks, bh, D, bits, off) || (off & 15);
  src.bits = bits;
  const uint32_t rb = (uint32_t)(D * bits / 8);
  src.rc = rsrc(ks.codes_k + (src.bad ? 0 : off), src.bad ? 0u : (uint32_t)ks.n_full * rb);
  src.sk = ks.scale_k + (int64_t)bh * ks.kgroups * D;
  src.mk = ks.min_k + (int64_t)bh * ks.kgroups * D;
  return src;
}

// 8 channels of one code word (BITS per channel, least significant first)
// as bf16 A-operand bits: round_to_bf16(fmaf(code, scale, min)), the stored
// value of each code
template <int BITS>
__device__ inline u4 k_decode8(uint64_t w, const float (&sc)[8], const float (&mn)[8]) {
  constexpr uint32_t mask = (1u << BITS) - 1;
  uint32_t o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float a = fmaf((float)(uint32_t)((w >> (2 * j * BITS)) & mask), sc[2 * j], mn[2 * j]);
    const float b = fmaf((float)(uint32_t)((w >> ((2 * j + 1) * BITS)) & mask), sc[2 * j + 1],
                         mn[2 * j + 1]);
    o[j] = bf2(a, b);
  }
  return u4{o[0], o[1], o[2], o[3]};
}

// channels c0 .. c0+7 of code rows ra and ra + 16 (one key group: shared
// scales and minima)
template <int BITS>
__device__ inline void k_decode_pair(const KSrc& src, int ra, int c0, u4& ka, u4& kb) {
  const int rb = D * BITS / 8;
  uint64_t wa, wb;
  if (BITS == 4) {
    wa = bload32(src.rc, ra * rb + c0 / 2);
    wb = bload32(src.rc, (ra + 16) * rb + c0 / 2);
  } else if (BITS == 2) {
    wa = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(src.rc, ra * rb + c0 / 4, 0, 0);
    wb = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(src.rc, (ra + 16) * rb + c0 / 4, 0, 0);
  } else {
    wa = __builtin_bit_cast(uint64_t, __builtin_amdgcn_raw_buffer_load_b64(src.rc, ra * rb + c0, 0, 0));
    wb = __builtin_bit_cast(uint64_t,
                            __builtin_amdgcn_raw_buffer_load_b64(src.rc, (ra + 16) * rb + c0, 0, 0));
  }
  const int64_t g = (int64_t)(ra / src.G) * D + c0;
  const f4 s0 = *reinterpret_cast<const f4*>(src.sk + g), s1 = *reinterpret_cast<const f4*>(src.sk + g + 4);
  const f4 m0 = *reinterpret_cast<const f4*>(src.mk + g), m1 = *reinterpret_cast<const f4*>(src.mk + g + 4);
  const float sc[8] = {s0[0], s0[1], s0[2], s0[3], s1[0], s1[1], s1[2], s1[3]};
  const float mn[8] = {m0[0], m0[1], m0[2], m0[3], m1[0], m1[1], m1[2], m1[3]};
  ka = k_decode8<BITS>(wa, sc, mn);
  kb = k_decode8<BITS>(wb, sc, mn);
}

// a wave's 32-row key tile at row0 as A operands (see KTiles); without
// PACKED every segment of the call is dense
template <bool PACKED>
__device__ inline void k_load(const KSrc& src, int row0, int lane, u4 (&k)[8]) {
  if (!PACKED || row0 >= src.n_full) {  // dense rows, or a packed segment's tail
    k_issue(src.rk, row0 - src.n_full, lane, k);
    return;
  }
  const int i16 = lane & 15, g4 = lane >> 4;
  if (src.bad) {
    const uint32_t nan2 = 0x7FC07FC0u;
#pragma unroll
    for (int t = 0; t < 8; ++t) k[t] = u4{nan2, nan2, nan2, nan2};
    return;
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int c0 = t * 32 + g4 * 8;
    if (src.bits == 4) k_decode_pair<4>(src, row0 + i16, c0, k[t], k[4 + t]);
    else if (src.bits == 2) k_decode_pair<2>(src, row0 + i16, c0, k[t], k[4 + t]);
    else k_decode_pair<8>(src, row0 + i16, c0, k[t], k[4 + t]);
  }
}

// the wave's key tiles of a step, from row0 on
template <bool PACKED>
__device__ inline void k_step(const KSrc& src, int row0, int lane, KTiles& K) {
#pragma unroll
  for (int i = 0; i < TPW; ++i) k_load<PACKED>(src, row0 + i * TILE, lane, K.k[i]);
}

// B operands (Q^T) of query tile qt, four 32-dim steps, from the staged block
__device__ inline void q_tile(const char* qs, int qt, int lane, u4 (&qb)[4]) {
  const int i16 = lane & 15, g4 = lane >> 4;
  const char* qrow = qs + (qt * 16 + i16) * QROW + g4 * 16;
#pragma unroll
  for (int t = 0; t < 4; ++t) qb[t] = *reinterpret_cast<const u4*>(qrow + t * 64);
}

// stage query rows [q0, q0 + QB) of the head's observation block into LDS (past
// nq the last row again: what a key gives it, infinite or not, it gives a real
// row too, so a row of weight 0 adds no NaN that was not there); row g*W + w of the block is window row w of the
// group's query head g, which starts ld rows after head g - 1
__device__ inline void stage_q(char* qs, const uint16_t* qh, int q0, int nq, int W, int ld) {
  // half of a thread's chunks in flight at once: one memory latency per half,
  // where a load and its store in turn took sixteen
  constexpr int kThreads = 64 * WAVES, kEach = QB * (D / 8) / kThreads, kBatch = kEach / 2;
  static_assert(kThreads % (D / 8) == 0 && kBatch * 2 * kThreads == QB * (D / 8), "whole batches");
  const int c = threadIdx.x % (D / 8);
#pragma unroll
  for (int e0 = 0; e0 < kEach; e0 += kBatch) {
    u4 v[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int r = ((int)threadIdx.x + (e0 + j) * kThreads) / (D / 8);
      const int at = min(q0 + r, nq - 1);
      int64_t row = at;
      if (ld != W) {
        const int g = at / W;
        row = (int64_t)g * ld + (at - g * W);
      }
      v[j] = *reinterpret_cast<const u4*>(qh + row * D + c * 8);
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int r = ((int)threadIdx.x + (e0 + j) * kThreads) / (D / 8);
      *reinterpret_cast<u4*>(qs + r * QROW + c * 16) = v[j];
    }
  }
}

// chunk c of the plan -> segment and row range
__device__ inline int chunk_rows(const ChunkPlan& p, const KSegs& segs, int c, int& r0, int& r1) {
  int si = 0;
  while (si + 1 < segs.n && c >= p.first[si + 1]) ++si;
  r0 = (c - p.first[si]) * p.rows[si];
  r1 = min(r0 + p.rows[si], segs.s[si].n_rows);
  return si;
}

// sum over the four key-row lanes (g4) of a query column, in all four
__device__ inline float sum_g4(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(t[0]) + __uint_as_float(t[1]);
}

// The logits S^T of a wave's two key tiles against one query tile: s[i][h] =
// keys h*16 .. h*16 + 15 of tile i, of which lane (i16, g4) holds keys
// g4*4 + j of query column i16.
typedef f4 Pair[TPW][2];
static_assert(TPW == 2 && TILE == 32, "the tile loops are written out for 64 keys");

__device__ inline float pick(const Pair& s, int n) { return s[n >> 3][n >> 2 & 1][n & 3]; }

// One half of the loops below: the logits of one query tile on the matrix
// cores, and between them, one step of each kind per slot, the exponentials of
// the tile before: slot n forms argument n, takes exponential n - 1 and adds
// probability n - 2, so nothing waits for the instruction before it.  The
// order is fixed by the scheduling barriers: left alone, the compiler puts the
// matrix instructions together and the LDS reads next to their use, and the
// two units took turns (680 cycles per 16 logits and SIMD, against 430 measured
// for the same instructions side by side).
template <class Arg, class Add>
__device__ inline void s_pair(const KTiles& K, const u4 (&qb)[4], Pair& s, Arg arg, Add add) {
  float x[16];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int n = 0; n < 18; ++n) {
    if (n < 16) {
      const int t = n >> 2, i = n >> 1 & 1, h = n & 1;
      s[i][h] = mfma(K.k[i][h * 4 + t], qb[t], t == 0 ? f4{0.f, 0.f, 0.f, 0.f} : s[i][h]);
      x[n] = arg(n);
    }
    if (n >= 1 && n <= 16) x[n - 1] = __builtin_amdgcn_exp2f(x[n - 1]);
    if (n >= 2) add(n - 2, x[n - 2]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// the logits alone
__device__ inline void s_pair(const KTiles& K, const u4 (&qb)[4], Pair& s) {
#pragma unroll
  for (int n = 0; n < 16; ++n) {
    const int t = n >> 2, i = n >> 1 & 1, h = n & 1;
    s[i][h] = mfma(K.k[i][h * 4 + t], qb[t], t == 0 ? f4{0.f, 0.f, 0.f, 0.f} : s[i][h]);
  }
}

// Pass 1, one half: the row state (m, l) of query column i16 takes the 16 keys
// of each of its four lanes in s, while the logits of query tile q go to
// `next`.  m is re-referenced only when some row of the tile has a logit more
// than kLazy above it (every v_exp_f32 argument is at most kLazy, up to 256
// times 1024 terms), which is rare after a chunk's first step: the merge of
// maxima across lanes and the rescaling took a sixth of the loop when every
// tile did them.  A row with no valid key yet keeps m = -inf and l = 0.
template <bool MASK>
__device__ inline void lse_half(const KTiles& K, const u4 (&q)[4], Pair& next, Pair& s, int row0,
                                int r1, int g4, float scale_log2, float* rm, float m, float* rl,
                                float l) {
  if (MASK) {
#pragma unroll
    for (int n = 0; n < 16; ++n)
      if (row0 + (n >> 2) * 16 + g4 * 4 + (n & 3) >= r1) s[n >> 3][n >> 2 & 1][n & 3] = -INFINITY;
  }
  // maximum of the raw logits, NaN if there is one (the scale is positive);
  // v_maximum3 takes them as they are, where fmaxf first quiets each operand
  float mx = pick(s, 0);
#pragma unroll
  for (int n = 1; n < 15; n += 2)
    mx = __builtin_elementwise_maximum(__builtin_elementwise_maximum(mx, pick(s, n)), pick(s, n + 1));
  mx = __builtin_elementwise_maximum(mx, pick(s, 15));
  if (__any(!(mx * scale_log2 <= m + kLazy))) {
    float top = -INFINITY;  // the largest that is not a NaN
#pragma unroll
    for (int n = 0; n < 16; ++n) top = fmaxf(top, pick(s, n));
    top = fmaxf(top, __shfl_xor(top, 16, 64));
    top = fmaxf(top, __shfl_xor(top, 32, 64));
    const float mn = fmaxf(m, top * scale_log2);
    l = m == -INFINITY ? l : l * __builtin_amdgcn_exp2f(m - mn);
    m = mn;
    *rm = m;
  }
  const float ref = m == -INFINITY ? 0.0f : m;
  float e[4];
  s_pair(K, q, next, [&](int n) { return fmaf(pick(s, n), scale_log2, -ref); },
         [&](int n, float p) { e[n & 3] = n < 4 ? p : e[n & 3] + p; });
  *rl = l + sum_g4((e[0] + e[1]) + (e[2] + e[3]));
}

// One step of pass 1 for one wave.  The loop keeps the matrix cores and the
// vector ALUs busy together: while the exponentials of one query tile run, the
// logits of the next are computed, in two sets of registers taken in turn, and
// the operands and row states of the tile after are read from LDS.  An odd last
// tile is joined by the one after it (staged as repeated rows, never read).  rm /
// rl hold the wave's (m, l) per query row; the four lanes of a query column
// agree and all store them.
template <bool MASK>
__device__ inline void lse_step(const KTiles& K, const char* qs, float* rm, float* rl, int nqt,
                                int row0, int r1, int lane, float scale_log2) {
  const int i16 = lane & 15, g4 = lane >> 4;
  const int last = QT - 1;
  u4 qa[4], qb[4];
  Pair sa, sb;
  q_tile(qs, 0, lane, qa);
  q_tile(qs, 1, lane, qb);
  rm += i16;
  rl += i16;
  float ma = rm[0], la = rl[0], mb = rm[16], lb = rl[16];
  s_pair(K, qa, sa);
  for (int t = 0; t < nqt; t += 2) {
    const int t2 = min(t + 2, last), t3 = min(t + 3, last);  // the last round's tiles are unused
    q_tile(qs, t2, lane, qa);
    float m = ma, l = la;
    ma = rm[t2 * 16];
    la = rl[t2 * 16];
    lse_half<MASK>(K, qb, sb, sa, row0, r1, g4, scale_log2, rm + t * 16, m, rl + t * 16, l);
    q_tile(qs, t3, lane, qb);
    m = mb;
    l = lb;
    mb = rm[t3 * 16];
    lb = rl[t3 * 16];
    lse_half<MASK>(K, qa, sa, sb, row0, r1, g4, scale_log2, rm + t * 16 + 16, m, rl + t * 16 + 16, l);
  }
}

// One step of pass 2 for one wave, pipelined like pass 1: probabilities added
// to the lanes' column sums (those below 2^-126 of the row's reference flush to
// zero).  Rows past r1 read as zeros; their sums land in column slots nobody
// reads.
__device__ inline void col_step(const KTiles& K, const char* qs, const f2* ls, int nqt, int lane,
                                float scale_log2, float (&cs)[16]) {
  const int i16 = lane & 15;
  const int last = QT - 1;
  u4 qa[4], qb[4];
  Pair sa, sb;
  q_tile(qs, 0, lane, qa);
  q_tile(qs, 1, lane, qb);
  ls += i16;
  f2 ra = ls[0], rb = ls[16];
  s_pair(K, qa, sa);
  for (int t = 0; t < nqt; t += 2) {
    const int t2 = min(t + 2, last), t3 = min(t + 3, last);  // the last round's tiles are unused
    q_tile(qs, t2, lane, qa);
    f2 r = ra;
    ra = ls[t2 * 16];
    s_pair(K, qb, sb, [&](int n) { return fmaf(pick(sa, n), scale_log2, -r[0]); },
           [&](int n, float p) { cs[n] = fmaf(p, r[1], cs[n]); });
    q_tile(qs, t3, lane, qb);
    r = rb;
    rb = ls[t3 * 16];
    s_pair(K, qa, sa, [&](int n) { return fmaf(pick(sb, n), scale_log2, -r[0]); },
           [&](int n, float p) { cs[n] = fmaf(p, r[1], cs[n]); });
  }
}

template <int CTRL>
__device__ inline float dpp(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), CTRL, 0xF, 0xF, true));
}

// One halving of the sum over the 16 lanes of a row: a lane keeps the upper
// (hi) or lower N/2 values and adds its partner's share of them.
template <int CTRL, int N>
__device__ inline void halve(float (&v)[16], bool hi) {
#pragma unroll
  for (int j = 0; j < N / 2; ++j) {
    const float keep = hi ? v[j + N / 2] : v[j], give = hi ? v[j] : v[j + N / 2];
    v[j] = keep + dpp<CTRL>(give);
  }
}

// Sums over the 16 lanes of a row, value i16 of the 16 in lane i16: partners
// are i16 ^ 15, ^ 7, ^ 3 and ^ 1 (row mirror, half mirror, quad permutations),
// 15 adds instead of 64 and one result to store per lane instead of 16.
__device__ inline float column_sum(float (&v)[16], int i16) {
  halve<0x140, 16>(v, i16 & 8);
  halve<0x141, 8>(v, i16 & 4);
  halve<0x1B, 4>(v, i16 & 2);
  halve<0xB1, 2>(v, i16 & 1);
  return v[0];
}

// ---------------------------------------------------------------- pass 1
// grid (chunks, query blocks, b*h_kv); one (m, l) record per (row, chunk)
template <bool PACKED>
__global__ __launch_bounds__(256, 2) void score_lse_kernel(KSegs segs, ChunkPlan plan,
                                                           const uint16_t* __restrict__ q, int Hq,
                                                           int Hkv, int W, float scale_log2,
                                                           float* __restrict__ partial) {
  __shared__ __attribute__((aligned(16))) char qs[QB * QROW];
  __shared__ float red_m[WAVES][QB], red_l[WAVES][QB];
  const int c = blockIdx.x, qb = blockIdx.y, bh = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int G = Hq / Hkv, nq = G * W, b = bh / Hkv, hkv = bh % Hkv;
  int r0, r1;
  const int si = chunk_rows(plan, segs, c, r0, r1);
  const KSeg& ks = segs.s[si];
  const uint16_t* qh = q + ((int64_t)b * Hq + hkv * G) * W * D;
  const int q0 = qb * QB;
  const int nqt = min(QT, (nq - q0 + 15) / 16);
  // the first keys are on their way while the queries are staged
  const KSrc src = k_source(ks, bh, r1);
  const int w0 = wave * TPW * TILE;
  KTiles K, next;
  k_step<PACKED>(src, r0 + w0, lane, next);
  stage_q(qs, qh, q0, nq, W, W);
  for (int e = threadIdx.x; e < WAVES * QB; e += 64 * WAVES) {
    red_m[e / QB][e % QB] = -INFINITY;
    red_l[e / QB][e % QB] = 0.0f;
  }
  __syncthreads();

  // the wave's tiles of a step: rows sc + wave*TPW*TILE on
  for (int sc = r0; sc < r1; sc += SUB) {
    K = next;
    if (sc + SUB < r1) k_step<PACKED>(src, sc + SUB + w0, lane, next);
    if (sc + w0 + TPW * TILE <= r1)
      lse_step<false>(K, qs, red_m[wave], red_l[wave], nqt, sc + w0, r1, lane, scale_log2);
    else
      lse_step<true>(K, qs, red_m[wave], red_l[wave], nqt, sc + w0, r1, lane, scale_log2);
  }
  __syncthreads();
  const int C = plan.n_chunks;
  for (int r = threadIdx.x; r < nqt * 16; r += blockDim.x) {
    if (q0 + r >= nq) continue;
    float mm = -INFINITY;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) mm = fmaxf(mm, red_m[w][r]);
    float ll = 0.0f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w)
      if (red_m[w][r] != -INFINITY) ll += red_l[w][r] * exp2f(red_m[w][r] - mm);
    const int64_t qi = ((int64_t)b * Hq + hkv * G) * W + q0 + r;  // global query row
    partial[(qi * C + c) * 2] = mm;
    partial[(qi * C + c) * 2 + 1] = ll;
  }
}

// ---------------------------------------------------------------- pass 2
struct ScoreOut {
  float* p[kMaxSeg];
};

// grid (chunks, query-block groups, b*h_kv): the query blocks
// [s*qbs, (s+1)*qbs) of the head.  With one group the scores and chunk mass
// are written directly; with several, each group's column sums (double) go
// to colpart and score_col_reduce_kernel adds them in group order.
template <bool PACKED>
__global__ __launch_bounds__(256, 2) void score_col_kernel(KSegs segs, ChunkPlan plan,
                                                           const uint16_t* __restrict__ q, int Hq,
                                                           int Hkv, int W, int q_ld,
                                                           float scale_log2,
                                                           const f2* __restrict__ norm,
                                                           ScoreOut out,
                                                           double* __restrict__ mass_partial,
                                                           int qbs, double* __restrict__ colpart) {
  __shared__ __attribute__((aligned(16))) char qs[QB * QROW];
  __shared__ f2 ls[QB];
  __shared__ double colsum[CHUNK];
  __shared__ double red[WAVES];
  // the first pass walks heads and chunks in grid order, so this one walks
  // them backwards: the keys it reads first are those the first pass read
  // last, which the last-level cache may still hold
  const int c = gridDim.x - 1 - blockIdx.x, sg = blockIdx.y, bh = gridDim.z - 1 - blockIdx.z;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i16 = lane & 15, g4 = lane >> 4;
  const int G = Hq / Hkv, nq = G * W, b = bh / Hkv, hkv = bh % Hkv;
  int r0, r1;
  const int si = chunk_rows(plan, segs, c, r0, r1);
  const KSeg& ks = segs.s[si];
  const uint16_t* qh = q + ((int64_t)b * Hq + hkv * G) * q_ld * D;
  const f2* lh = norm + ((int64_t)b * Hq + hkv * G) * W;
  for (int e = threadIdx.x; e < CHUNK; e += blockDim.x) colsum[e] = 0.0;

  const KSrc src = k_source(ks, bh, r1);
  const int q_end = min(nq, (sg + 1) * qbs * QB);
  const int w0 = wave * TPW * TILE;
  KTiles K, next;
  for (int q0 = sg * qbs * QB; q0 < q_end; q0 += QB) {
    const int nqt = min(QT, (nq - q0 + 15) / 16);
    if (!PACKED) k_step<PACKED>(src, r0 + w0, lane, next);
    __syncthreads();  // the previous block's readers are done
    stage_q(qs, qh, q0, nq, W, q_ld);
    for (int r = threadIdx.x; r < QB; r += blockDim.x)
      ls[r] = q0 + r < nq ? lh[q0 + r] : f2{INFINITY, 0.0f};  // padded rows: p = 0
    __syncthreads();
    for (int sc = r0; sc < r1; sc += SUB) {
      if (PACKED) {
        // decoded where they are used: holding the next step's tiles beside
        // these spilled 36 registers (10240 keys of which 4096 in 4 bits,
        // 28672 rows, both passes: 1693 us so, 1656 us without)
        k_step<PACKED>(src, sc + w0, lane, K);
      } else {
        K = next;
        if (sc + SUB < r1) k_step<PACKED>(src, sc + SUB + w0, lane, next);
      }
      float cs[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) cs[j] = 0.0f;
      col_step(K, qs, ls, nqt, lane, scale_log2, cs);
      // value i16 of a lane's 16: tile i16/8, its upper or lower 16 keys, key g4*4 + i16%4
      const float v = column_sum(cs, i16);
      colsum[sc - r0 + w0 + (i16 >> 3) * TILE + (i16 >> 2 & 1) * 16 + g4 * 4 + (i16 & 3)] += (double)v;
    }
  }
  __syncthreads();
  if (colpart) {  // one group of several: its column sums, reduced later
    double* cp = colpart + (((int64_t)sg * gridDim.z + bh) * plan.n_chunks + c) * CHUNK;
    for (int e = threadIdx.x; e < CHUNK; e += blockDim.x) cp[e] = colsum[e];
    return;
  }
  // scores (rows past r1 were masked by never being written) and the
  // chunk's mass (fixed-order reduction: deterministic)
  float* sp = out.p[si];
  double part = 0.0;
  for (int e = threadIdx.x; e < CHUNK; e += blockDim.x) {
    if (r0 + e < r1) {
      if (sp) sp[(int64_t)bh * ks.n_rows + r0 + e] = (float)colsum[e];
      part += colsum[e];
    }
  }
  part = wave_sum_d(part);
  if (lane == 0) red[wave] = part;
  __syncthreads();
  if (threadIdx.x == 0 && mass_partial)
    mass_partial[(int64_t)bh * plan.n_chunks + c] = red[0] + red[1] + red[2] + red[3];
}

// grid (chunks, b*h_kv): the groups' column sums added in group order, then
// the scores and the chunk's mass as the single-group kernel writes them
__global__ __launch_bounds__(256) void score_col_reduce_kernel(KSegs segs, ChunkPlan plan,
                                                               int n_groups,
                                                               const double* __restrict__ colpart,
                                                               ScoreOut out,
                                                               double* __restrict__ mass_partial) {
  __shared__ double red[4];
  const int c = blockIdx.x, bh = blockIdx.y, BH = gridDim.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int r0, r1;
  const int si = chunk_rows(plan, segs, c, r0, r1);
  const KSeg& ks = segs.s[si];
  float* sp = out.p[si];
  double part = 0.0;
  for (int e = threadIdx.x; e < CHUNK; e += blockDim.x) {
    if (r0 + e >= r1) continue;
    double v = 0.0;
    for (int g = 0; g < n_groups; ++g)
      v += colpart[(((int64_t)g * BH + bh) * plan.n_chunks + c) * CHUNK + e];
    if (sp) sp[(int64_t)bh * ks.n_rows + r0 + e] = (float)v;
    part += v;
  }
  part = wave_sum_d(part);
  if (lane == 0) red[wave] = part;
  __syncthreads();
  if (threadIdx.x == 0 && mass_partial)
    mass_partial[(int64_t)bh * plan.n_chunks + c] = red[0] + red[1] + red[2] + red[3];
}

}  // namespace

bool score_mfma_eligible(const uc_shape& sh, const KSegs& segs, int q_dt) {
  if (sh.D != D || q_dt != UC_BF16) return false;
  for (int i = 0; i < segs.n; ++i) {
    if (segs.s[i].dtype != UC_BF16) return false;
    // packed: key groups of >= 32 rows, so a 32-row tile shares one scale set
    if (segs.s[i].kind == UC_SEG_PACKED && segs.s[i].group < TILE) return false;
  }
  return true;
}

int score_mfma_chunk_rows() { return CHUNK; }

// a packed segment with code rows among the plan's chunks (the plan may
// leave segments out)
static bool has_packed(const KSegs& segs, const ChunkPlan& plan) {
  for (int i = 0; i < segs.n; ++i)
    if (segs.s[i].kind == UC_SEG_PACKED && segs.s[i].n_full > 0 && plan.first[i + 1] > plan.first[i])
      return true;
  return false;
}

int score_mfma_qblocks(int nq) { return (nq + QB - 1) / QB; }

// chunk sums that the groups of the column pass may leave to be added, for
// `base` chunk-heads (grows with base)
int64_t score_mfma_col_slots(int64_t base) { return 1024 + base; }

// Query-block groups of the column pass.  A workgroup takes ceil(query blocks /
// groups) of them and the chip holds two workgroups per CU, so the pass lasts
// as many times that as rounds of workgroups are needed: the count with the
// least of it, and of those the smallest (fewer partial sums to add).  72
// chunk-heads of 112 blocks ran as 8 groups, 576 workgroups and two rounds of
// 14 blocks; as 7 they are one round of 16.
static int score_col_groups(const uc_shape& sh, const ChunkPlan& plan, int W) {
  const int qblocks = score_mfma_qblocks((sh.Hq / sh.Hkv) * W);
  const int64_t base = (int64_t)plan.n_chunks * sh.B * sh.Hkv, slots = 2 * device_cus();
  const int64_t most = std::min<int64_t>(qblocks, score_mfma_col_slots(base) / base);
  int best = 1;
  int64_t least = INT64_MAX;
  for (int g = 1; g <= most; ++g) {
    const int64_t cost = (base * g + slots - 1) / slots * ((qblocks + g - 1) / g);
    if (cost < least) {
      least = cost;
      best = g;
    }
  }
  return best;
}

hipError_t launch_score_lse_mfma(const uc_shape& sh, const KSegs& segs, const ChunkPlan& plan,
                                 const void* q, int W, float sm_scale, float* partial,
                                 hipStream_t st) {
  const int nq = (sh.Hq / sh.Hkv) * W;
  dim3 grid(plan.n_chunks, score_mfma_qblocks(nq), sh.B * sh.Hkv);
  if (has_packed(segs, plan))
    hipLaunchKernelGGL(score_lse_kernel<true>, grid, dim3(256), 0, st, segs, plan,
                       (const uint16_t*)q, sh.Hq, sh.Hkv, W, sm_scale * kLog2e, partial);
  else
    hipLaunchKernelGGL(score_lse_kernel<false>, grid, dim3(256), 0, st, segs, plan,
                       (const uint16_t*)q, sh.Hq, sh.Hkv, W, sm_scale * kLog2e, partial);
  return hipGetLastError();
}

hipError_t launch_score_col_mfma(const uc_shape& sh, const KSegs& segs, const ChunkPlan& plan,
                                 const void* q, int W, int q_ld, float sm_scale, const float* norm,
                                 float* const* scores, double* mass_partial, double* colpart,
                                 hipStream_t st) {
  ScoreOut so{};
  for (int i = 0; i < segs.n; ++i) so.p[i] = scores ? scores[i] : nullptr;
  const int groups = score_col_groups(sh, plan, W);
  const int qblocks = score_mfma_qblocks((sh.Hq / sh.Hkv) * W);
  const int qbs = (qblocks + groups - 1) / groups;
  const int n_groups = (qblocks + qbs - 1) / qbs;
  dim3 grid(plan.n_chunks, n_groups, sh.B * sh.Hkv);
  if (has_packed(segs, plan))
    hipLaunchKernelGGL(score_col_kernel<true>, grid, dim3(256), 0, st, segs, plan,
                       (const uint16_t*)q, sh.Hq, sh.Hkv, W, q_ld, sm_scale * kLog2e, (const f2*)norm, so,
                       mass_partial, qbs, n_groups > 1 ? colpart : nullptr);
  else
    hipLaunchKernelGGL(score_col_kernel<false>, grid, dim3(256), 0, st, segs, plan,
                       (const uint16_t*)q, sh.Hq, sh.Hkv, W, q_ld, sm_scale * kLog2e, (const f2*)norm, so,
                       mass_partial, qbs, n_groups > 1 ? colpart : nullptr);
  if (n_groups > 1)
    hipLaunchKernelGGL(score_col_reduce_kernel, dim3(plan.n_chunks, sh.B * sh.Hkv), dim3(256), 0,
                       st, segs, plan, n_groups, (const double*)colpart, so, mass_partial);
  return hipGetLastError();
}

}  // namespace uc
