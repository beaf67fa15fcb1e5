// quantize.hip -- group-wise asymmetric min/max quantization of one segment
// into packed low-bit codes, float scales/minima and a residual tail
// (App. E, "Physical, type-aware KV storage").
//
//   keys:   one channel over G consecutive rows     (per-channel groups)
//   values: G consecutive channels of one row       (per-token groups)
//   mn = min, mx = max, s = (mx - mn) / (2^b - 1)
//   code = s > 0 ? clamp(rint((x - mn) / s), 0, 2^b - 1) : 0
// All in IEEE binary32 with correctly rounded division and no contraction, so
// codes and scales are reproducible bit for bit.
//
// Layout of the output (see unicache.h): row r of a head's codes occupies
// D*b/8 bytes; channel c sits in byte c*b/8 at bit (c % (8/b))*b.  A lane holds
// 8 consecutive channels of a row (one or two 16-byte loads: rows are 16-byte
// aligned, head dims 64 or 128, groups of at least 8) and writes their 8 codes
// as one 16-, 32- or 64-bit store.
#pragma clang fp contract(off)

#include "uc_common.h"

namespace uc {
namespace {

__device__ inline int quant_code(float x, float mn, float s, int qmax) {
  if (!(s > 0.0f)) return 0;
  float t = __fdiv_rn(x - mn, s);
  int c = (int)rintf(t);
  return min(max(c, 0), qmax);
}

// Eight elements of a row as loaded (16-byte aligned).
template <int DT>
struct Raw8 {
  uint4 w[DT == UC_F32 ? 2 : 1];
  __device__ inline void load(const void* p, int64_t e) {
    const uint4* q = reinterpret_cast<const uint4*>(static_cast<const char*>(p) + e * (DT == UC_F32 ? 4 : 2));
    w[0] = q[0];
    if constexpr (DT == UC_F32) w[1] = q[1];
  }
  __device__ inline void widen(float (&x)[8]) const {
    if constexpr (DT == UC_F32) {
      const uint32_t u[8] = {w[0].x, w[0].y, w[0].z, w[0].w, w[1].x, w[1].y, w[1].z, w[1].w};
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = __uint_as_float(u[j]);
    } else {
      const uint32_t u[4] = {w[0].x, w[0].y, w[0].z, w[0].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint16_t lo = (uint16_t)(u[j] & 0xFFFFu), hi = (uint16_t)(u[j] >> 16);
        x[2 * j] = DT == UC_BF16 ? bf16_to_f32(lo) : f16_to_f32(lo);
        x[2 * j + 1] = DT == UC_BF16 ? bf16_to_f32(hi) : f16_to_f32(hi);
      }
    }
  }
};

// Scale of a group from its range, and the scale's reciprocal, without the
// general division: correctly rounded like it where this returns true, which
// is for ranges clear of underflow and overflow and for 0 (one value in the
// group: scale, reciprocal and every code are 0).  Quotient and reciprocal come
// from fused multiply-add corrections (Markstein 1990).  Checked over all
// mantissas: range / (2^b - 1) is right after one correction; the reciprocal,
// from any start within 2 units in the last place (v_rcp_f32 has 1), is right
// after two steps except for a mantissa of all ones, which is left to the
// caller.  Nine issue slots, where two general divisions took about thirty.
__device__ inline bool plain_scale(float range, int b, float& s, float& r) {
  const float qmax = (float)((1 << b) - 1);
  const float c = b == 2 ? 1.0f / 3.0f : b == 4 ? 1.0f / 15.0f : 1.0f / 255.0f;
  s = range * c;
  s = __builtin_fmaf(__builtin_fmaf(-s, qmax, range), c, s);
  r = __builtin_amdgcn_rcpf(s);
  r = __builtin_fmaf(__builtin_fmaf(-s, r, 1.0f), r, r);
  r = __builtin_fmaf(__builtin_fmaf(-s, r, 1.0f), r, r);
  if (!(s > 0.0f)) r = 0.0f;
  return range == 0.0f || (range >= 0x1p-70f && range <= 0x1p80f &&
                           (__float_as_uint(s) & 0x7FFFFFu) != 0x7FFFFFu);
}

// rint of the correctly rounded quotient d / s, from r = 1 / s correctly rounded:
// two residual corrections by fused multiply-add, of which the first leaves a
// faithful and the second the correctly rounded quotient (Markstein 1990).  s
// and r are plain_scale's (r = 0 for s = 0).  Five instructions where the general
// division takes about twelve, several of them at a quarter of the rate.
__device__ inline uint32_t quotient_code(float d, float s, float r, float qmax) {
  float q = d * r;
  q = __builtin_fmaf(__builtin_fmaf(-q, s, d), r, q);
  q = __builtin_fmaf(__builtin_fmaf(-q, s, d), r, q);
  return (uint32_t)__builtin_amdgcn_fmed3f(rintf(q), 0.0f, qmax);
}

// the B-bit codes of 8 consecutive channels (channel e at bit B*e) stored at p
template <int B>
__device__ inline void put_codes8(uint8_t* p, const uint32_t (&code)[8]) {
  if constexpr (B == 8) {
    uint2 w{0, 0};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      w.x |= code[e] << (8 * e);
      w.y |= code[4 + e] << (8 * e);
    }
    *reinterpret_cast<uint2*>(p) = w;
  } else {
    uint32_t w = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) w |= code[e] << (B * e);
    if constexpr (B == 4) *reinterpret_cast<uint32_t*>(p) = w;
    else *reinterpret_cast<uint16_t*>(p) = (uint16_t)w;
  }
}

template <int B>
__device__ inline void codes8(uint8_t* p, const float (&x)[8], const float (&mn)[8],
                              const float (&s)[8], const float (&r)[8], bool plain) {
  uint32_t code[8];
  if (plain) {
#pragma unroll
    for (int e = 0; e < 8; ++e) code[e] = quotient_code(x[e] - mn[e], s[e], r[e], (float)((1 << B) - 1));
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) code[e] = (uint32_t)quant_code(x[e], mn[e], s[e], (1 << B) - 1);
  }
  put_codes8<B>(p, code);
}

// minimum and maximum that give NaN if either is NaN: v_minimum3 / v_maximum3
// take two more values per instruction as they are, where fminf first quiets
// each operand.  A NaN found so sends the caller to fminf and fmaxf, which
// drop it.
__device__ inline float low(float a, float b) { return __builtin_elementwise_minimum(a, b); }
__device__ inline float high(float a, float b) { return __builtin_elementwise_maximum(a, b); }

template <int CTRL>
__device__ inline float dpp_move(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), CTRL, 0xF, 0xF, true));
}

// minimum and maximum over neighbouring lanes: pairs, quads, eights, sixteens
template <int CTRL>
__device__ inline void range_step(float& mn, float& mx) {
  mn = fminf(mn, dpp_move<CTRL>(mn));
  mx = fmaxf(mx, dpp_move<CTRL>(mx));
}

constexpr int kVRows = 4;  // value rows per lane

// Values, group G >= 8: a group is G/8 neighbouring lanes of one row; its
// min and max combine across lanes.  A block takes kVRows * 256/(D/8) rows.
template <int DT, int D>
__device__ inline void quantize_v_block(const KSeg& seg, const void* __restrict__ v, int N, int blk,
                                        int bh) {
  constexpr int cpr = D / 8, RB = 256 / cpr;  // lanes per row, rows per pass
  const int c8 = threadIdx.x % cpr, r0 = blk * (RB * kVRows) + threadIdx.x / cpr;
  const int G = seg.group, lpg = G / 8;
  int b;
  int64_t off;
  const bool ok = head_codes(seg, bh, D, b, off) && !(off & 15);
  Raw8<DT> raw[kVRows];
#pragma unroll
  for (int i = 0; i < kVRows; ++i) {
    const int r = min(r0 + i * RB, seg.n_full - 1);  // rows past the end repeat the last
    raw[i].load(v, ((int64_t)bh * N + r) * D + c8 * 8);
  }
  uint8_t* codes = const_cast<uint8_t*>(seg.codes_v) + (ok ? off : 0) + c8 * b;
#pragma unroll
  for (int i = 0; i < kVRows; ++i) {
    const int r = r0 + i * RB;
    float x[8];
    raw[i].widen(x);
    float mn = low(low(x[0], x[1]), x[2]), mx = high(high(x[0], x[1]), x[2]);
    mn = low(low(mn, x[3]), x[4]);
    mx = high(high(mx, x[3]), x[4]);
    mn = low(low(low(mn, x[5]), x[6]), x[7]);
    mx = high(high(high(mx, x[5]), x[6]), x[7]);
    if (__any(mn != mn)) {
      mn = mx = x[0];
#pragma unroll
      for (int e = 1; e < 8; ++e) {
        mn = fminf(mn, x[e]);
        mx = fmaxf(mx, x[e]);
      }
    }
    if (lpg > 1) range_step<0xB1>(mn, mx);   // lane ^ 1
    if (lpg > 2) range_step<0x4E>(mn, mx);   // lane ^ 2
    if (lpg > 4) range_step<0x141>(mn, mx);  // the other quad of eight
    if (lpg > 8) range_step<0x140>(mn, mx);  // the other eight of sixteen
    float s, rs;
    const bool plain = __all(plain_scale(mx - mn, b, s, rs));
    if (!plain) s = __fdiv_rn(mx - mn, (float)((1 << b) - 1));
    if (!ok) s = __builtin_nanf("");
    const bool live = r < seg.n_full;
    if (live && c8 % lpg == 0) {
      const int64_t mi = ((int64_t)bh * seg.cap_full + r) * (D / G) + c8 / lpg;
      const_cast<float*>(seg.scale_v)[mi] = s;
      const_cast<float*>(seg.min_v)[mi] = mn;
    }
    if (!ok) continue;
    float mn8[8], s8[8], r8[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      mn8[e] = mn;
      s8[e] = s;
      r8[e] = rs;
    }
    if (!live) continue;
    uint8_t* p = codes + (int64_t)r * (D * b / 8);
    if (b == 4) codes8<4>(p, x, mn8, s8, r8, plain);
    else if (b == 2) codes8<2>(p, x, mn8, s8, r8, plain);
    else codes8<8>(p, x, mn8, s8, r8, plain);
  }
}

// LDS of a key block: minima and maxima of the lanes that share 8 channels,
// then the channels' minimum, scale and reciprocal.
struct KeyLds {
  float lo[32 * 64], hi[32 * 64];  // [256/(D/8)][D]
  float mn[128], s[128], rs[128];
  int plain;
};

// Keys: one block of 256 lanes per (row group, bh); a lane holds 8 channels
// of rows rr, rr + RB, ... of the group (RB = 256/(D/8) rows per pass, at
// most 8 rows per lane since G <= D).  Bound by the vector ALU: the lanes'
// minima and maxima meet in LDS, where one lane per channel reduces them and
// forms the scale; done by every lane for its 8 channels, with cross-lane
// steps, this took half of the block's instructions at G = 64.
template <int DT, int D>
__device__ inline void quantize_k_block(const KSeg& seg, const void* __restrict__ k, int N, int g,
                                        int bh, KeyLds& sh) {
  constexpr int cpr = D / 8, RB = 256 / cpr, RL = D / RB;
  static_assert(RB * D == 32 * 64, "the lanes' minima and maxima fill the array");
  const int c8 = threadIdx.x % cpr, rr = threadIdx.x / cpr;
  const int G = seg.group;
  int b;
  int64_t off;
  float* scale = const_cast<float*>(seg.scale_k) + ((int64_t)bh * seg.kgroups + g) * D;
  float* mnp = const_cast<float*>(seg.min_k) + ((int64_t)bh * seg.kgroups + g) * D;
  if (!head_codes(seg, bh, D, b, off) || (off & 15)) {  // uniform over the block
    if (threadIdx.x < D) scale[threadIdx.x] = __builtin_nanf("");
    return;
  }
  const int64_t base = ((int64_t)bh * N + (int64_t)g * G) * D + c8 * 8;
  Raw8<DT> raw[RL];
#pragma unroll
  for (int i = 0; i < RL; ++i)
    if (rr + i * RB < G) raw[i].load(k, base + (int64_t)(rr + i * RB) * D);
  if (threadIdx.x == 0) sh.plain = 1;
  float mn[8], mx[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    mn[e] = INFINITY;
    mx[e] = -INFINITY;
  }
#pragma unroll
  for (int i = 0; i < RL; ++i)
    if (rr + i * RB < G) {
      float x[8];
      raw[i].widen(x);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        mn[e] = low(mn[e], x[e]);
        mx[e] = high(mx[e], x[e]);
      }
    }
  bool nan = false;
#pragma unroll
  for (int e = 0; e < 8; ++e) nan |= mn[e] != mn[e];
  if (__any(nan)) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      mn[e] = INFINITY;
      mx[e] = -INFINITY;
    }
#pragma unroll
    for (int i = 0; i < RL; ++i)
      if (rr + i * RB < G) {
        float x[8];
        raw[i].widen(x);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          mn[e] = fminf(mn[e], x[e]);
          mx[e] = fmaxf(mx[e], x[e]);
        }
      }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    sh.lo[rr * D + c8 * 8 + e] = mn[e];
    sh.hi[rr * D + c8 * 8 + e] = mx[e];
  }
  __syncthreads();
  if (threadIdx.x < D) {
    const int c = threadIdx.x;
    // no NaN here any more; rows of lanes past the group hold the infinities
    float a = sh.lo[c], z = sh.hi[c];
#pragma unroll
    for (int r = 1; r < RB; ++r) {
      a = low(a, sh.lo[r * D + c]);
      z = high(z, sh.hi[r * D + c]);
    }
    // a channel of NaNs alone: float rows have always left NaN here
    if (DT == UC_F32 && a > z) a = z = __builtin_nanf("");
    float s, r;
    if (!plain_scale(z - a, b, s, r)) {
      s = __fdiv_rn(z - a, (float)((1 << b) - 1));
      sh.plain = 0;
    }
    sh.mn[c] = a;
    sh.s[c] = s;
    sh.rs[c] = r;
    scale[c] = s;
    mnp[c] = a;
  }
  __syncthreads();
  const bool plain = sh.plain != 0;
  float s[8], rs[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    mn[e] = sh.mn[c8 * 8 + e];
    s[e] = sh.s[c8 * 8 + e];
    rs[e] = sh.rs[c8 * 8 + e];
  }
  const int row_bytes = D * b / 8;
  uint8_t* codes = const_cast<uint8_t*>(seg.codes_k) + off + (int64_t)g * G * row_bytes + c8 * b;
#pragma unroll
  for (int i = 0; i < RL; ++i) {
    const int r = rr + i * RB;
    if (r < G) {
      float x[8];
      raw[i].widen(x);
      uint8_t* p = codes + (int64_t)r * row_bytes;
      if (b == 4) codes8<4>(p, x, mn, s, rs, plain);
      else if (b == 2) codes8<2>(p, x, mn, s, rs, plain);
      else codes8<8>(p, x, mn, s, rs, plain);
    }
  }
}

// grid (key groups + value blocks, b*h_kv): both halves of a segment in one
// launch, so that neither waits for the other's last blocks and a small
// segment pays for one launch.  64 heads of 4096 bf16 rows (176 MB): 60 us, of
// the vector ALU more than of memory, against 49 + 41 us in two launches; one
// head of 256 fp32 rows 5 us against 17 + 4.5.
template <int DT, int D>
__global__ __launch_bounds__(256) void quantize_vec_kernel(KSeg seg, const void* __restrict__ k,
                                                           const void* __restrict__ v, int N,
                                                           int k_blocks) {
  __shared__ __attribute__((aligned(16))) KeyLds sh;
  const int x = blockIdx.x;
  if (x < k_blocks) quantize_k_block<DT, D>(seg, k, N, x, blockIdx.y, sh);
  else quantize_v_block<DT, D>(seg, v, N, x - k_blocks, blockIdx.y);
}

// Residual tail: rows n_full..N-1 copied unchanged (16 bytes per lane).
__global__ void copy_tail_kernel(KSeg seg, const void* __restrict__ k, const void* __restrict__ v,
                                 int N, int row_bytes) {
  const int bh = blockIdx.y;
  const int64_t tail_bytes = (int64_t)seg.tail_len * row_bytes;
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 16;
  if (i >= tail_bytes) return;
  const int64_t src = ((int64_t)bh * N + seg.n_full) * row_bytes + i;
  const int64_t dst = (int64_t)bh * seg.tail_stride * row_bytes + i;
  *reinterpret_cast<uint4*>((char*)seg.tail_k + dst) =
      *reinterpret_cast<const uint4*>((const char*)k + src);
  *reinterpret_cast<uint4*>((char*)seg.tail_v + dst) =
      *reinterpret_cast<const uint4*>((const char*)v + src);
}

// Dequantisation of a whole packed segment into dense rows of its dtype:
// one thread per (row, channel) element of one (b, h_kv) (blockIdx.y);
// rows < n_full decode their code, tail rows are copied.
__global__ void dequantize_kernel(KSeg s, void* __restrict__ kout, void* __restrict__ vout,
                                  int D) {
  const int bh = blockIdx.y;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int N = s.n_rows;
  if (e >= (int64_t)N * D) return;
  const int r = (int)(e / D), c = (int)(e % D);
  const int64_t o = (int64_t)bh * N * D + e;
  float xk, xv;
  if (r >= s.n_full) {
    const int64_t t = ((int64_t)bh * s.tail_stride + (r - s.n_full)) * D + c;
    xk = load_elem(s.tail_k, s.dtype, t);
    xv = load_elem(s.tail_v, s.dtype, t);
  } else {
    int b;
    int64_t off;
    if (!head_codes(s, bh, D, b, off)) {
      xk = xv = __builtin_nanf("");
    } else {
      const int G = s.group, ngv = D / G;
      const int64_t byte = off + (int64_t)r * (D * b / 8) + c * b / 8;
      const int shift = (c % (8 / b)) * b, mask = (1 << b) - 1;
      const int ck = (s.codes_k[byte] >> shift) & mask;
      const int cv = (s.codes_v[byte] >> shift) & mask;
      const int64_t ki = ((int64_t)bh * s.kgroups + r / G) * D + c;
      const int64_t vi = ((int64_t)bh * s.cap_full + r) * ngv + c / G;
      xk = round_to(__builtin_fmaf((float)ck, s.scale_k[ki], s.min_k[ki]), s.dtype);
      xv = round_to(__builtin_fmaf((float)cv, s.scale_v[vi], s.min_v[vi]), s.dtype);
    }
  }
  if (s.dtype == UC_F32) {
    static_cast<float*>(kout)[o] = xk;
    static_cast<float*>(vout)[o] = xv;
  } else if (s.dtype == UC_BF16) {
    static_cast<uint16_t*>(kout)[o] = f32_to_bf16_bits(xk);
    static_cast<uint16_t*>(vout)[o] = f32_to_bf16_bits(xv);
  } else {
    static_cast<uint16_t*>(kout)[o] = f32_to_f16_bits(xk);
    static_cast<uint16_t*>(vout)[o] = f32_to_f16_bits(xv);
  }
}

// Streaming append: rows j0 .. j0+n-1 of each head's new rows (n_new per
// head) go to tail rows pos .. pos+n-1 (16 bytes per lane).
__global__ void stream_copy_kernel(const char* __restrict__ knew, const char* __restrict__ vnew,
                                   int n_new, int j0, int n, char* tk, char* tv, int tail_stride,
                                   int pos, int row_bytes) {
  const int bh = blockIdx.y;
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 16;
  if (i >= (int64_t)n * row_bytes) return;
  const int64_t src = ((int64_t)bh * n_new + j0) * row_bytes + i;
  const int64_t dst = ((int64_t)bh * tail_stride + pos) * row_bytes + i;
  *reinterpret_cast<uint4*>(tk + dst) = *reinterpret_cast<const uint4*>(knew + src);
  *reinterpret_cast<uint4*>(tv + dst) = *reinterpret_cast<const uint4*>(vnew + src);
}

}  // namespace

// Rows enter the tail; whenever it holds G rows they are quantised in place
// as the next row group of the codes and scales (a view of the segment whose
// storage starts at that group; the strides stay the segment's) and the tail
// empties.
hipError_t launch_stream_append(const uc_shape& sh, const KSeg& seg, const void* knew,
                                const void* vnew, int n_new, hipStream_t st) {
  const int G = seg.group, D = sh.D, BH = sh.B * sh.Hkv;
  const int row_bytes = D * dtype_bytes(seg.dtype), code_row = D * seg.bits / 8;
  int n_full = seg.n_full, tail = seg.tail_len;
  for (int j = 0; j < n_new;) {
    const int take = min(G - tail, n_new - j);
    const int64_t lanes = (int64_t)take * row_bytes / 16;
    hipLaunchKernelGGL(stream_copy_kernel, dim3((unsigned)((lanes + 255) / 256), BH), dim3(256), 0,
                       st, (const char*)knew, (const char*)vnew, n_new, j, take,
                       (char*)seg.tail_k, (char*)seg.tail_v, seg.tail_stride, tail, row_bytes);
    j += take;
    tail += take;
    if (tail == G) {
      KSeg v = seg;
      v.n_rows = v.n_full = G;
      v.tail_len = 0;
      v.codes_k = seg.codes_k + (int64_t)n_full * code_row;
      v.codes_v = seg.codes_v + (int64_t)n_full * code_row;
      v.codes_bytes = seg.codes_bytes - (uint64_t)n_full * code_row;
      v.scale_k = seg.scale_k + (int64_t)(n_full / G) * D;
      v.min_k = seg.min_k + (int64_t)(n_full / G) * D;
      v.scale_v = seg.scale_v + (int64_t)n_full * (D / G);
      v.min_v = seg.min_v + (int64_t)n_full * (D / G);
      hipError_t e = launch_quantize(sh, seg.tail_k, seg.tail_v, seg.dtype, G, v, st);
      if (e != hipSuccess) return e;
      n_full += G;
      tail = 0;
    }
  }
  return hipGetLastError();
}

hipError_t launch_dequantize(const uc_shape& sh, const KSeg& seg, void* kout, void* vout,
                             hipStream_t st) {
  const int64_t n = (int64_t)seg.n_rows * sh.D;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(dequantize_kernel, dim3((unsigned)((n + 255) / 256), sh.B * sh.Hkv),
                     dim3(256), 0, st, seg, kout, vout, sh.D);
  return hipGetLastError();
}

hipError_t launch_quantize(const uc_shape& sh, const void* k, const void* v, int dt, int N,
                           const KSeg& out, hipStream_t st) {
  const int BH = sh.B * sh.Hkv, D = sh.D;
  if (out.n_full > 0) {
    const int groups = out.n_full / out.group;
    const int rows = kVRows * 256 / (D / 8);
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(groups + (out.n_full + rows - 1) / rows, BH), dim3(256), 0,
                         st, out, k, v, N, groups);
    };
    if (dt == UC_F32) D == 64 ? go(quantize_vec_kernel<UC_F32, 64>) : go(quantize_vec_kernel<UC_F32, 128>);
    else if (dt == UC_F16) D == 64 ? go(quantize_vec_kernel<UC_F16, 64>) : go(quantize_vec_kernel<UC_F16, 128>);
    else D == 64 ? go(quantize_vec_kernel<UC_BF16, 64>) : go(quantize_vec_kernel<UC_BF16, 128>);
  }
  if (out.tail_len > 0) {
    const int row_bytes = D * dtype_bytes(dt);
    const int64_t lanes = ((int64_t)out.tail_len * row_bytes + 15) / 16;
    hipLaunchKernelGGL(copy_tail_kernel, dim3((unsigned)((lanes + 255) / 256), BH), dim3(256), 0,
                       st, out, k, v, N, row_bytes);
  }
  return hipGetLastError();
}

}  // namespace uc
