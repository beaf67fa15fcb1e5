// attend_wide.hip -- attention and importance scores in binary32 or better on the
// matrix cores, for every input outside the bf16 kernels: fp32 / fp16 rows or
// queries, head dim 64, 8-bit codes, row groups below 32, any mixture of
// element types (App. E, "Attention over heterogeneous cache segments" and
// "Batched GQA token selection").
//
// Rows and queries are widened exactly; the logits are v_mfma_f64_16x16x4_f64
// products rounded to binary32, the value products v_mfma_f32_16x16x4_f32.  A
// wave takes 16-row tiles; nothing is staged in LDS, because the contraction may
// run over the head dims and the keys in any order as long as both operands
// agree on it:
//   S^T = K Q^T   step t contracts dims g4*(D/4) + t (g4 = lane/16), so a lane
//                 reads D/4 consecutive dims of key row lane%16;
//   O^T += V^T P  step j contracts keys g4 + 4*j, which is exactly where the
//                 binary64 S^T result leaves them, so the probabilities are the B
//                 operand as they stand; output row i of dim tile t stands for
//                 dim i*(D/16) + t, so a lane reads D/16 consecutive dims of
//                 value row g4 + 4*j.
// Each loop holds the raw rows (or codes and value scales) of the next tile
// in flight while it computes the current one.
//
// Bound: these calls are short, and a wave-per-row kernel on the vector ALUs
// spent six dependent cross-lane sums on every row.  Measured on one MI355X, one
// decode step, kernel times: 4 requests, 28 query heads on 4 KV heads, head dim
// 128, fp16, 577 dense rows and 4096 8-bit rows 165.8 us before, 22.6 now (and
// the merge of their records 4.7 and 4.6); fp32, head dim 64, 4 query heads on
// one KV head, 371 rows 31.6 us before, 5.2 now (merge 4.6 and 1.8).
#include "uc_common.h"

namespace uc {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef double d4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));

constexpr int WAVES = 4;
constexpr int ROWS = 16;         // rows per tile, query rows per block
constexpr float kLazy = 8.0f;    // base-2 headroom before the reference maximum is raised

__device__ inline f4 mfma4(float a, float b, const f4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// 8 stored 16-bit elements -> binary32
template <int DT>
__device__ inline void widen8(const u4& w, float* x) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (DT == UC_BF16) {
      x[2 * i] = __uint_as_float(w[i] << 16);
      x[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    } else {
      x[2 * i] = f16_to_f32((uint16_t)w[i]);
      x[2 * i + 1] = f16_to_f32((uint16_t)(w[i] >> 16));
    }
  }
}

template <int DT>
constexpr int elem() { return DT == UC_F32 ? 4 : 2; }

// N consecutive elements as stored; N * elem is a multiple of 8 bytes
template <int DT, int N>
struct RawRun {
  static constexpr int B = N * elem<DT>();
  static constexpr int NW = (B + 15) / 16;
  u4 w[NW];
  // p need not be aligned (query rows carry no alignment requirement on this
  // path; the memory system takes any address)
  __device__ inline void load(const void* p) {
    if constexpr (B % 16) {
      u2 h;
      __builtin_memcpy(&h, p, 8);
      w[0] = u4{h[0], h[1], 0, 0};
    } else {
      __builtin_memcpy(w, p, B);
    }
  }
  __device__ inline void widen(float* x) const {
    if constexpr (DT == UC_F32) {
#pragma unroll
      for (int i = 0; i < N; ++i) x[i] = __uint_as_float(w[i / 4][i % 4]);
    } else if constexpr (N < 8) {
      float y[8];
      widen8<DT>(w[0], y);
#pragma unroll
      for (int i = 0; i < N; ++i) x[i] = y[i];
    } else {
#pragma unroll
      for (int i = 0; i < N / 8; ++i) widen8<DT>(w[i], x + 8 * i);
    }
  }
};

// n elements rounded to the segment's element type (dt is uniform)
template <int N>
__device__ inline void round_all(float* x, int dt) {
  if (dt == UC_BF16) {
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = bf16_to_f32(f32_to_bf16_bits(x[i]));
  } else if (dt == UC_F16) {
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = f16_to_f32(f32_to_f16_bits(x[i]));
  }
}

// softmax state of the lane's query column and its O^T accumulators
template <int D>
struct State {
  float m, l;
  f4 acc[D / 16];
};

// The tile's logits: s[j] = <q, k> for key row g4 + 4*j of the tile and query
// column lane%16, in binary64 and rounded once: in binary32 their rounding was
// the largest error of a pass (3.3e-7 against 64 bits for a wave-wide sum on
// the vector ALUs, 3.4e-7 to 3.8e-7 for short chains of binary32 matrix
// products, 2.1e-7 so; 43 fp16 rows over 4085).  These products take twice the
// time of binary32 ones (28 -> 32 us for the fp16 step above).
template <int D>
__device__ inline f4 tile_scores(const float (&kf)[D / 4], const float (&qf)[D / 4]) {
  d4 a = d4{0., 0., 0., 0.}, b = a;
#pragma unroll
  for (int t = 0; t < D / 4; t += 2) {
    a = __builtin_amdgcn_mfma_f64_16x16x4f64((double)kf[t], (double)qf[t], a, 0, 0, 0);
    b = __builtin_amdgcn_mfma_f64_16x16x4f64((double)kf[t + 1], (double)qf[t + 1], b, 0, 0, 0);
  }
  a += b;
  return f4{(float)a[0], (float)a[1], (float)a[2], (float)a[3]};
}

// Softmax of a tile whose first `live` rows count (lazy reference maximum, as
// in the decode kernel), then O^T += V^T P.
template <int D, bool WANT_O>
__device__ inline void tile_softmax(State<D>& st, const f4& s, float scale_log2, int live,
                                    float (&vf)[4][D / 16], int g4) {
  float p[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) p[j] = g4 + 4 * j < live ? s[j] : -INFINITY;
  // the scale is positive: the maximum of the raw logits gives the maximum
  float mx = fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3])) * scale_log2;
  if (__builtin_amdgcn_ballot_w64(mx > st.m + kLazy)) {
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mn = fmaxf(st.m, mx);
    const float alpha = __builtin_amdgcn_exp2f(st.m - mn);
    st.l *= alpha;
    if (WANT_O) {
#pragma unroll
      for (int t = 0; t < D / 16; ++t) st.acc[t] *= alpha;
    }
    st.m = mn;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) p[j] = __builtin_amdgcn_exp2f(fmaf(p[j], scale_log2, -st.m));
  st.l += (p[0] + p[1]) + (p[2] + p[3]);
  if (WANT_O) {
    if (live < ROWS) {  // rows past the end repeat the last one, with p = 0: 0 * inf must not reach the sums
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (g4 + 4 * j >= live) {
#pragma unroll
          for (int t = 0; t < D / 16; ++t) vf[j][t] = 0.0f;
        }
    }
    // the tile's product on its own, then one addition: sums of 16 rows and
    // of a few tiles round less than one running sum
    f4 pv[D / 16];
#pragma unroll
    for (int t = 0; t < D / 16; ++t) pv[t] = mfma4(vf[0][t], p[0], f4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
    for (int j = 1; j < 4; ++j)
#pragma unroll
      for (int t = 0; t < D / 16; ++t) pv[t] = mfma4(vf[j][t], p[j], pv[t]);
#pragma unroll
    for (int t = 0; t < D / 16; ++t) st.acc[t] += pv[t];
  }
}

// ---------------------------------------------------------------- row sources
// A source loads the raw bytes of one tile (rows row0 .. row0 + 15 of
// [0, n), rows past the end replaced by the last one) and widens them.

template <int D, int DT, bool WANT_O>
struct DenseSrc {
  const char* k;
  const char* v;  // one head's rows
  struct Raw {
    RawRun<DT, D / 4> k;
    RawRun<DT, D / 16> v[4];
  };
  __device__ inline void load(int row0, int n, int lane, Raw& r) const {
    constexpr int64_t RB = (int64_t)D * elem<DT>();
    const int i16 = lane & 15, g4 = lane >> 4;
    r.k.load(k + min(row0 + i16, n - 1) * RB + g4 * (RB / 4));
    if (WANT_O) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        r.v[j].load(v + min(row0 + g4 + 4 * j, n - 1) * RB + i16 * (RB / 16));
    }
  }
  __device__ inline void keys(const Raw& r, int, int, int, float (&kf)[D / 4]) const {
    r.k.widen(kf);
  }
  __device__ inline void values(const Raw& r, int, float (&vf)[4][D / 16]) const {
#pragma unroll
    for (int j = 0; j < 4; ++j) r.v[j].widen(vf[j]);
  }
};

// Packed rows [0, n_full) of one head.  The codes of a lane's D/4 key channels
// are D*BITS/32 bytes, those of its D/16 value channels D*BITS/128 bytes; the
// value channels lie in one group (groups are at least 8 channels).
template <int D, int BITS, bool WANT_O>
struct PackedSrc {
  const uint8_t* ck;
  const uint8_t* cv;
  const float* sk;
  const float* mk;
  const float* sv;
  const float* mv;
  int lgG, dt;
  static constexpr int KB = D * BITS / 32, VB = D * BITS / 128;
  struct Raw {
    u4 k[(KB + 15) / 16];
    u2 v[4];
    float sv[4], mv[4];
  };
  template <int BYTES, int NW>
  __device__ static inline void bytes(const uint8_t* p, uint32_t (&w)[NW]) {
    w[0] = 0;
    __builtin_memcpy(w, p, BYTES);
  }
  __device__ inline void load(int row0, int n, int lane, Raw& r) const {
    constexpr int RB = D * BITS / 8;
    const int i16 = lane & 15, g4 = lane >> 4;
    uint32_t w[(KB + 3) / 4];
    bytes<KB>(ck + (int64_t)min(row0 + i16, n - 1) * RB + g4 * KB, w);
#pragma unroll
    for (int i = 0; i < (KB + 3) / 4; ++i) r.k[i / 4][i % 4] = w[i];
    if (WANT_O) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = min(row0 + g4 + 4 * j, n - 1);
        uint32_t x[(VB + 3) / 4];
        bytes<VB>(cv + (int64_t)row * RB + i16 * VB, x);
        r.v[j][0] = x[0];
        if constexpr (VB > 4) r.v[j][1] = x[1];
        const int64_t vi = (int64_t)row * (D >> lgG) + ((i16 * (D / 16)) >> lgG);
        r.sv[j] = sv[vi];
        r.mv[j] = mv[vi];
      }
    }
  }
  __device__ inline void keys(const Raw& r, int row0, int n, int lane, float (&kf)[D / 4]) const {
    const int i16 = lane & 15, g4 = lane >> 4;
    const int64_t g = (int64_t)(min(row0 + i16, n - 1) >> lgG) * D + g4 * (D / 4);
#pragma unroll
    for (int i = 0; i < D / 4; i += 4) {
      const f4 s = *reinterpret_cast<const f4*>(sk + g + i), m = *reinterpret_cast<const f4*>(mk + g + i);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int bit = (i + e) * BITS;
        const uint32_t c = (r.k[bit / 128][bit / 32 % 4] >> (bit % 32)) & ((1u << BITS) - 1);
        kf[i + e] = fmaf((float)c, s[e], m[e]);
      }
    }
    round_all<D / 4>(kf, dt);
  }
  __device__ inline void values(const Raw& r, int, float (&vf)[4][D / 16]) const {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int e = 0; e < D / 16; ++e) {
        const int bit = e * BITS;
        const uint32_t c = (r.v[j][bit / 32] >> (bit % 32)) & ((1u << BITS) - 1);
        vf[j][e] = fmaf((float)c, r.sv[j], r.mv[j]);
      }
      round_all<D / 16>(vf[j], dt);
    }
  }
};

// Rows [r0, r1) of a source, of which [0, n) exist (r1 <= n): the wave takes
// tiles wave, wave + WAVES, ...
template <int D, bool WANT_O, class Src>
__device__ inline void walk(State<D>& st, const Src& src, int r0, int r1, int wave, int lane,
                            const float (&qf)[D / 4], float scale_log2) {
  const int g4 = lane >> 4;
  int row = r0 + wave * ROWS;
  if (row >= r1) return;
  typename Src::Raw cur, nxt;
  src.load(row, r1, lane, cur);
  for (; row < r1; row += WAVES * ROWS) {
    // past the end the last row is read again and never used
    src.load(min(row + WAVES * ROWS, r1 - 1), r1, lane, nxt);
    float kf[D / 4], vf[4][D / 16];
    src.keys(cur, row, r1, lane, kf);
    const f4 s = tile_scores<D>(kf, qf);
    if (WANT_O) src.values(cur, lane, vf);
    tile_softmax<D, WANT_O>(st, s, scale_log2, r1 - row, vf, g4);
    cur = nxt;
  }
}

template <int D, bool WANT_O>
__device__ inline void walk_dense(State<D>& st, const void* k, const void* v, int dt, int64_t row,
                                  int r0, int r1, int wave, int lane, const float (&qf)[D / 4],
                                  float scale_log2) {
  if (r1 <= r0) return;
  const int64_t off = row * D * dtype_bytes(dt);
  const char* kb = (const char*)k + off;
  const char* vb = (const char*)v + off;
  if (dt == UC_F32)
    walk<D, WANT_O>(st, DenseSrc<D, UC_F32, WANT_O>{kb, vb}, r0, r1, wave, lane, qf, scale_log2);
  else if (dt == UC_F16)
    walk<D, WANT_O>(st, DenseSrc<D, UC_F16, WANT_O>{kb, vb}, r0, r1, wave, lane, qf, scale_log2);
  else
    walk<D, WANT_O>(st, DenseSrc<D, UC_BF16, WANT_O>{kb, vb}, r0, r1, wave, lane, qf, scale_log2);
}

// rows [r0, r1) of segment s for head bh; false if the head's device-side
// layout is invalid
template <int D, bool WANT_O>
__device__ inline bool walk_segment(State<D>& st, const KSeg& s, int bh, int r0, int r1, int wave,
                                    int lane, const float (&qf)[D / 4], float scale_log2) {
  if (s.kind == UC_SEG_DENSE) {
    walk_dense<D, WANT_O>(st, s.k, s.v, s.dtype, (int64_t)bh * s.row_stride, r0, r1, wave, lane,
                          qf, scale_log2);
    return true;
  }
  int bits = 0;
  int64_t off = 0;
  if (!head_codes(s, bh, D, bits, off)) return false;
  const int p1 = min(r1, s.n_full);
  if (p1 > r0) {
    const int lgG = __builtin_ctz((unsigned)s.group);
    const int64_t ko = (int64_t)bh * s.kgroups * D, vo = (int64_t)bh * s.cap_full * (D >> lgG);
    auto go = [&](auto src) {
      src.ck = s.codes_k + off;
      src.cv = s.codes_v + off;
      src.sk = s.scale_k + ko;
      src.mk = s.min_k + ko;
      src.sv = s.scale_v + vo;
      src.mv = s.min_v + vo;
      src.lgG = lgG;
      src.dt = s.dtype;
      walk<D, WANT_O>(st, src, r0, p1, wave, lane, qf, scale_log2);
    };
    if (bits == 4) go(PackedSrc<D, 4, WANT_O>{});
    else if (bits == 8) go(PackedSrc<D, 8, WANT_O>{});
    else go(PackedSrc<D, 2, WANT_O>{});
  }
  const int t0 = max(r0, s.n_full);
  walk_dense<D, WANT_O>(st, s.tail_k, s.tail_v, s.dtype, (int64_t)bh * s.tail_stride,
                        t0 - s.n_full, r1 - s.n_full, wave, lane, qf, scale_log2);
  return true;
}

// D/4 consecutive dims (from g4*(D/4)) of query row `row`, widened; zeros
// when the row does not exist
template <int D>
__device__ inline void load_query(const void* q, int q_dt, int64_t row, int g4, bool live,
                                  float (&qf)[D / 4]) {
#pragma unroll
  for (int i = 0; i < D / 4; ++i) qf[i] = 0.0f;
  if (!live) return;
  const char* p = (const char*)q + (row * D + g4 * (D / 4)) * dtype_bytes(q_dt);
  if (q_dt == UC_F32) {
    RawRun<UC_F32, D / 4> r;
    r.load(p);
    r.widen(qf);
  } else {
    RawRun<UC_F16, D / 4> r;  // the bytes of either 16-bit type
    r.load(p);
    if (q_dt == UC_F16) {
      r.widen(qf);
    } else {
      RawRun<UC_BF16, D / 4> b;
      __builtin_memcpy(&b, &r, sizeof b);
      b.widen(qf);
    }
  }
}

__device__ inline int chunk_segment(const ChunkPlan& plan, int nseg, int c) {
  int si = 0;
  while (si + 1 < nseg && c >= plan.first[si + 1]) ++si;
  return si;
}

// grid (chunks, blocks of 16 query rows of one KV head, b*h_kv): one partial
// record (m, l[, o]) per query row and chunk, base-2 units
template <int D, bool WANT_O>
__global__ __launch_bounds__(256, 2) void attend_wide_kernel(KSegs segs, ChunkPlan plan,
                                                             const void* __restrict__ q, int q_dt,
                                                             int Hq, int Hkv, int M,
                                                             float scale_log2,
                                                             float* __restrict__ partial) {
  constexpr int PS = WANT_O ? D + 2 : 2;
  __shared__ float red_m[WAVES][ROWS], red_l[WAVES][ROWS];
  __shared__ float red_o[WANT_O ? WAVES : 1][ROWS][WANT_O ? D + 4 : 1];
  const int c = blockIdx.x, bh = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i16 = lane & 15, g4 = lane >> 4;
  const int nq = Hq / Hkv * M, q0 = blockIdx.y * ROWS;
  const int64_t qbase = (int64_t)bh * nq;  // the head's query rows are consecutive
  const int si = chunk_segment(plan, segs.n, c);
  const KSeg& s = segs.s[si];
  const int r0 = (c - plan.first[si]) * plan.rows[si];
  const int r1 = min(r0 + plan.rows[si], s.n_rows);

  float qf[D / 4];
  load_query<D>(q, q_dt, qbase + q0 + i16, g4, q0 + i16 < nq, qf);
  State<D> st;
  st.m = -INFINITY;
  st.l = 0.0f;
#pragma unroll
  for (int t = 0; t < D / 16; ++t) st.acc[t] = f4{0.f, 0.f, 0.f, 0.f};
  const bool ok = walk_segment<D, WANT_O>(st, s, bh, r0, r1, wave, lane, qf, scale_log2);

  // merge the four waves' states; the four lanes of a query column hold
  // parts of its row sum
  st.l += __shfl_xor(st.l, 16, 64);
  st.l += __shfl_xor(st.l, 32, 64);
  if (g4 == 0) {
    red_m[wave][i16] = st.m;
    red_l[wave][i16] = st.l;
  }
  if (WANT_O) {
    // acc[t][j] is dim (g4*4 + j)*(D/16) + t of query column i16
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int t = 0; t < D / 16; t += 4)
        *reinterpret_cast<f4*>(&red_o[wave][i16][(g4 * 4 + j) * (D / 16) + t]) =
            f4{st.acc[t][j], st.acc[t + 1][j], st.acc[t + 2][j], st.acc[t + 3][j]};
  }
  __syncthreads();
  const int C = plan.n_chunks;
  const int rows = min(ROWS, nq - q0);
  for (int e = threadIdx.x; e < rows * PS; e += blockDim.x) {
    const int r = e / PS, f = e % PS;
    float mw[WAVES], M_ = -INFINITY;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      mw[w] = red_m[w][r];
      M_ = fmaxf(M_, mw[w]);
    }
    float val = M_;
    if (f > 0) {
      val = 0.0f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        const float wt = mw[w] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(mw[w] - M_);
        val += wt * (f == 1 ? red_l[w][r] : red_o[WANT_O ? w : 0][r][WANT_O ? f - 2 : 0]);
      }
    }
    if (!ok) val = f == 1 ? __builtin_nanf("") : 0.0f;
    partial[((qbase + q0 + r) * C + c) * PS + f] = val;
  }
}

// ---------------------------------------------------------------- merge
// Records of one query row -> o (and lse): NW waves per row, each lane owning
// D/64 dims.  A wave loads eight records at a time, every load issued before
// any is used; with four waves a row's records are dealt round-robin and the
// waves' states merged through LDS.  An empty record (m = -inf, the other
// fields undefined) is dropped by selects.
template <int D, int NW>
__global__ __launch_bounds__(256) void record_merge_kernel(int Q, int C,
                                                           const float* __restrict__ partial,
                                                           float* __restrict__ o,
                                                           float* __restrict__ lse) {
  constexpr int PER = D / 64, RPB = 4 / NW;  // dims per lane, query rows per workgroup
  constexpr int ps = D + 2;
  __shared__ float rm[4], rl[4], ro[4][D];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int qi = blockIdx.x * RPB + (NW == 1 ? wave : 0);
  if (NW == 1 && qi >= Q) return;
  const int w0 = NW == 1 ? 0 : wave;
  const float* P = partial + (int64_t)qi * C * ps;
  float M = -INFINITY, l = 0.0f, acc[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) acc[i] = 0.0f;
  for (int c0 = w0; c0 < C; c0 += 8 * NW) {
    f2 ml[8];
    float oc[8][PER];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const float* p = P + (int64_t)min(c0 + r * NW, C - 1) * ps;
      ml[r] = *reinterpret_cast<const f2*>(p);
#pragma unroll
      for (int i = 0; i < PER; ++i) oc[r][i] = p[2 + PER * lane + i];
    }
    float mx = M;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      if (c0 + r * NW >= C) ml[r][0] = -INFINITY;
      mx = fmaxf(mx, ml[r][0]);
    }
    const float a = M == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(M - mx);
    l *= a;
#pragma unroll
    for (int i = 0; i < PER; ++i) acc[i] *= a;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const bool live = ml[r][0] != -INFINITY;
      const float b = live ? __builtin_amdgcn_exp2f(ml[r][0] - mx) : 0.0f;
      l = fmaf(b, live ? ml[r][1] : 0.0f, l);
#pragma unroll
      for (int i = 0; i < PER; ++i) acc[i] = fmaf(b, live ? oc[r][i] : 0.0f, acc[i]);
    }
    M = mx;
  }
  if (NW > 1) {
    if (lane == 0) {
      rm[wave] = M;
      rl[wave] = l;
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) ro[wave][PER * lane + i] = acc[i];
    __syncthreads();
    if (wave > 0) return;
    M = fmaxf(fmaxf(rm[0], rm[1]), fmaxf(rm[2], rm[3]));
    l = 0.0f;
#pragma unroll
    for (int i = 0; i < PER; ++i) acc[i] = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float b = rm[w] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(rm[w] - M);
      l = fmaf(b, rl[w], l);
#pragma unroll
      for (int i = 0; i < PER; ++i) acc[i] = fmaf(b, ro[w][PER * lane + i], acc[i]);
    }
  }
  const float inv = 1.0f / l;
#pragma unroll
  for (int i = 0; i < PER; ++i) o[(int64_t)qi * D + PER * lane + i] = acc[i] * inv;
  if (lse && lane == 0) lse[qi] = (float)(((double)M + (double)log2f(l)) * kLn2d);
}

// ---------------------------------------------------------------- scores
struct ScorePtrs {
  float* p[kMaxSeg];
};

// Importance scores, second pass.  grid (chunks of 64 keys, b*h_kv): a wave
// holds one 16-key tile and runs it against every query row of the head, 64
// rows staged in LDS at a time.  S = Q K^T leaves a lane four query rows
// (g4 + 4*j) of its key (lane%16), so the sum over queries runs in the lane,
// in double, and the four lanes of a key are added at the end.
template <int D>
__global__ __launch_bounds__(256, 2) void score_wide_kernel(KSegs segs, ChunkPlan plan,
                                                            const void* __restrict__ q, int q_dt,
                                                            int Hq, int Hkv, int W, int q_ld,
                                                            float scale_log2,
                                                            const f2* __restrict__ norm,
                                                            ScorePtrs scores,
                                                            double* __restrict__ mass_partial) {
  constexpr int QB = 64, QS = D + 4;  // query rows per round, floats per staged row
  __shared__ __attribute__((aligned(16))) float qs[QB * QS];
  __shared__ __attribute__((aligned(16))) f2 ls[QB];
  __shared__ double red[WAVES];
  const int c = blockIdx.x, bh = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i16 = lane & 15, g4 = lane >> 4;
  const int G = Hq / Hkv, nq = G * W;
  const int si = chunk_segment(plan, segs.n, c);
  const KSeg& s = segs.s[si];
  const int r0 = (c - plan.first[si]) * plan.rows[si];
  const int r1 = min(r0 + plan.rows[si], s.n_rows);
  const int row0 = r0 + wave * ROWS, row = row0 + i16;
  const int rr = min(row, r1 - 1);  // lanes past the end repeat the last key

  float kf[D / 4];
  bool ok = true;
  auto dense = [&](const void* k, int64_t at) {
    const char* p = (const char*)k + (at * D + g4 * (D / 4)) * dtype_bytes(s.dtype);
    if (s.dtype == UC_F32) {
      RawRun<UC_F32, D / 4> x;
      x.load(p);
      x.widen(kf);
    } else if (s.dtype == UC_F16) {
      RawRun<UC_F16, D / 4> x;
      x.load(p);
      x.widen(kf);
    } else {
      RawRun<UC_BF16, D / 4> x;
      x.load(p);
      x.widen(kf);
    }
  };
  if (s.kind == UC_SEG_DENSE) {
    dense(s.k, (int64_t)bh * s.row_stride + rr);
  } else {
    int bits = 0;
    int64_t off = 0;
    ok = head_codes(s, bh, D, bits, off);
    if (!ok) {
#pragma unroll
      for (int i = 0; i < D / 4; ++i) kf[i] = 0.0f;
    } else if (rr >= s.n_full) {
      dense(s.tail_k, (int64_t)bh * s.tail_stride + rr - s.n_full);
    } else {
      const uint8_t* ck = s.codes_k + off + (int64_t)rr * (D * bits / 8) + g4 * (D * bits / 32);
      const int64_t g = ((int64_t)bh * s.kgroups + rr / s.group) * D + g4 * (D / 4);
      const int mask = (1 << bits) - 1;
#pragma unroll
      for (int i = 0; i < D / 4; ++i) {
        const int code = (ck[i * bits / 8] >> (i * bits % 8)) & mask;
        kf[i] = fmaf((float)code, s.scale_k[g + i], s.min_k[g + i]);
      }
      round_all<D / 4>(kf, s.dtype);
    }
  }

  double acc = 0.0;
  for (int q0 = 0; q0 < nq; q0 += QB) {
    __syncthreads();
    const int n = min(QB, nq - q0), tiles = (n + ROWS - 1) / ROWS;
    for (int e = threadIdx.x; e < tiles * ROWS * 4; e += blockDim.x) {
      const int j = e >> 2, part = e & 3;
      // rows past the last repeat it: what a key gives them it gives a real row
      // too, so that with weight 0 they add no NaN
      const int at = q0 + min(j, n - 1);
      const int g = at / W, w = at - g * W;
      float x[D / 4];
      load_query<D>(q, q_dt, (int64_t)(bh * G + g) * q_ld + w, part, true, x);
#pragma unroll
      for (int i = 0; i < D / 4; i += 4)
        *reinterpret_cast<f4*>(&qs[j * QS + part * (D / 4) + i]) = f4{x[i], x[i + 1], x[i + 2], x[i + 3]};
    }
    // rows past the window: p = exp2(-inf) = 0, times 0
    if (threadIdx.x < QB)
      ls[threadIdx.x] = (int)threadIdx.x < n ? norm[(int64_t)bh * nq + q0 + threadIdx.x] : f2{INFINITY, 0.0f};
    __syncthreads();
    for (int t = 0; t < tiles; ++t) {
      float qf[D / 4];
#pragma unroll
      for (int i = 0; i < D / 4; i += 4) {
        const f4 x = *reinterpret_cast<const f4*>(&qs[(t * ROWS + i16) * QS + g4 * (D / 4) + i]);
        qf[i] = x[0];
        qf[i + 1] = x[1];
        qf[i + 2] = x[2];
        qf[i + 3] = x[3];
      }
      const f4 sv = tile_scores<D>(qf, kf);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f2 row = ls[t * ROWS + g4 + 4 * j];
        acc = fma((double)exp2f(fmaf(sv[j], scale_log2, -row[0])), (double)row[1], acc);
      }
    }
  }
  acc += __shfl_xor(acc, 16, 64);
  acc += __shfl_xor(acc, 32, 64);
  if (!ok) acc = __builtin_nan("");
  const bool mine = g4 == 0 && row < r1;
  if (mine && scores.p[si]) scores.p[si][(int64_t)bh * s.n_rows + row] = (float)acc;
  // chunk mass (fixed-order reduction: deterministic)
  const double part = wave_sum_d(mine ? acc : 0.0);
  if (lane == 0) red[wave] = part;
  __syncthreads();
  if (threadIdx.x == 0 && mass_partial)
    mass_partial[(int64_t)bh * plan.n_chunks + c] = red[0] + red[1] + red[2] + red[3];
}

}  // namespace

hipError_t launch_attend_wide(const uc_shape& sh, const KSegs& segs, const ChunkPlan& plan,
                              const void* q, int q_dt, int M, float sm_scale, float* partial,
                              bool want_o, hipStream_t st) {
  const int nq = sh.Hq / sh.Hkv * M;
  const dim3 grid(plan.n_chunks, (nq + ROWS - 1) / ROWS, sh.B * sh.Hkv);
  const float sl2 = sm_scale * kLog2e;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(64 * WAVES), 0, st, segs, plan, q, q_dt, sh.Hq, sh.Hkv, M,
                       sl2, partial);
  };
  if (sh.D == 64) want_o ? go(attend_wide_kernel<64, true>) : go(attend_wide_kernel<64, false>);
  else want_o ? go(attend_wide_kernel<128, true>) : go(attend_wide_kernel<128, false>);
  return hipGetLastError();
}

// o (and lse) of records that share one softmax.  Four waves per row when one
// wave would take its records in more than one pass of eight.
hipError_t launch_record_merge(int D, int Q, int C, const float* partial, float* o, float* lse,
                               hipStream_t st) {
  auto go = [&](auto kernel, int rows) {
    hipLaunchKernelGGL(kernel, dim3((Q + rows - 1) / rows), dim3(256), 0, st, Q, C, partial, o, lse);
  };
  const bool wide = C > 8;
  if (D == 64) wide ? go(record_merge_kernel<64, 4>, 1) : go(record_merge_kernel<64, 1>, 4);
  else wide ? go(record_merge_kernel<128, 4>, 1) : go(record_merge_kernel<128, 1>, 4);
  return hipGetLastError();
}

int score_wide_chunk_rows() { return WAVES * ROWS; }

hipError_t launch_score_wide(const uc_shape& sh, const KSegs& segs, const ChunkPlan& plan,
                             const void* q, int q_dt, int W, int q_ld, float sm_scale,
                             const float* norm, float* const* scores, double* mass_partial,
                             hipStream_t st) {
  ScorePtrs sp{};
  for (int i = 0; i < segs.n; ++i) sp.p[i] = scores ? scores[i] : nullptr;
  const dim3 grid(plan.n_chunks, sh.B * sh.Hkv);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(64 * WAVES), 0, st, segs, plan, q, q_dt, sh.Hq, sh.Hkv, W,
                       q_ld, sm_scale * kLog2e, (const f2*)norm, sp, mass_partial);
  };
  sh.D == 64 ? go(score_wide_kernel<64>) : go(score_wide_kernel<128>);
  return hipGetLastError();
}

}  // namespace uc
