// HIP kernels of the SIR filter step for gfx950 (CDNA4, wave64).
//
// One step of Algorithm 1 (Section 2) is three to five launches on one
// stream, with every decision taken on the device (so the same sequence
// serves every step, and a HIP graph of it can be replayed):
//   k_step         gather parent + propagate (Section 6.1) + patch likelihood
//                  (Eqs. 3-4, Section 5.5) + per-block normalisation record
//   k_merge        merge of the block records per chunk
//   k_merge_final  fixed-order merge of the chunks: the normaliser, ESS, MMSE
//                  estimate, resampling decision and uniform; commits or rolls
//                  back the step; the fixed-point CDF prefixes of the chunks
//                  (k_merge_one: both, up to 262,144 particles)
//   k_anc          systematic resampling: one wave per segment of 1024
//                  particles, each particle's run of output slots from the
//                  segment's CDF
//   k_fill         the slots of heavy segments queued by k_anc (concentrated
//                  weights), in chunks of tiles (k_anc_all: both, up to 1024
//                  segments, with helper waves instead of a queue)
//   (or k_rna: RNA of Section 3, one wave or workgroup per group of particles;
//                  k_arna_* for ARNA; k_rpa_* after the ancestors for RPA)
#include "ppf_internal.hpp"

#include <array>
#include <cfloat>
#include <climits>
#include <cmath>
#include <cstddef>
#include <mutex>
#include <tuple>
#include <utility>

namespace ppf {
namespace {

// ------------------------------------------------------------ Philox4x32-10
// Counter-based generator of Salmon et al. (SC'11): ten rounds of two 32-bit
// multiplications whose high halves are xored with the other counter words
// and a Weyl-sequence round key.
__device__ __forceinline__ uint4 philox(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    // one 32 x 32 -> 64-bit product gives both halves; each three-way xor
    // is one v_bitop3 (truth table 0x96 = a ^ b ^ c)
    const uint64_t p0 = (uint64_t)0xD2511F53u * c.x;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
    c = make_uint4(__builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c.y, k0, 0x96), (uint32_t)p1,
                   __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c.w, k1, 0x96), (uint32_t)p0);
  }
  return c;
}

__device__ __forceinline__ uint4 draw(const Model& m, uint32_t index, uint32_t k,
                                      uint32_t purpose, uint32_t block) {
  return philox(make_uint4(index, k, (purpose << 24) | block, m.track), m.key0, m.key1);
}

// Uniforms from the top 24 bits: [0, 1) and (0, 1], exact in fp32.
__device__ __forceinline__ float u24_open_hi(uint32_t a) { return (float)(a >> 8) * 0x1p-24f; }
__device__ __forceinline__ double u53(uint32_t a, uint32_t b) {
  return ((double)a * 2097152.0 + (double)(b >> 11)) * 0x1p-53;
}

// The five normals of a particle come from one Philox block: three radius
// fields of 24 bits and three angle fields of 18 bits, laid end to end from
// bit 0 of word x as radius 0, angle 0, radius 1, angle 1, radius 2, angle 2
// (126 of the 128 bits). A radius field r is the uniform (r + 1) / 2^24 in
// (0, 1] and an angle field a the uniform a / 2^18 in [0, 1), both exact in
// fp32.
struct NormalFields {
  uint32_t r0, a0, r1, a1, r2, a2;
};
__device__ __forceinline__ NormalFields normal_fields(uint4 w) {
  NormalFields f;
  f.r0 = w.x & 0xFFFFFFu;                                           // bits 0-23
  f.a0 = __builtin_amdgcn_alignbit(w.y, w.x, 24) & 0x3FFFFu;        // bits 24-41
  f.r1 = __builtin_amdgcn_alignbit(w.z, w.y, 10) & 0xFFFFFFu;       // bits 42-65
  f.a1 = __builtin_amdgcn_ubfe(w.z, 2, 18);                         // bits 66-83
  f.r2 = __builtin_amdgcn_alignbit(w.w, w.z, 20) & 0xFFFFFFu;       // bits 84-107
  f.a2 = __builtin_amdgcn_ubfe(w.w, 12, 18);                        // bits 108-125
  return f;
}

// Box-Muller in fp32 from a radius field r and an angle field a. The radius
// sqrt(-2 ln u), u in (0, 1], uses the hardware log2 and square root
// (measured over all 2^24 uniforms: at most 1.9 ulp for ln u, 0.9 ulp for
// the root). The angle 2 pi t, t in [0, 1), is reduced exactly: x = 4 t,
// q = rint(x), r = x - q in [-1/2, 1/2], and sin, cos(2 pi t) are
// sin, cos(pi/2 r) rotated by the quadrant q, from the Taylor series in r to
// degree 9 and 10 (truncation below 2e-9; measured at most 8.8e-8 absolute
// with fp32 rounding).
__device__ __forceinline__ float bm_radius(uint32_t r) {
  // -2 ln u = -(2 ln 2) log2 u
  return __builtin_amdgcn_sqrtf(-0x1.62e430p+0f *
                                __builtin_amdgcn_logf((float)(r + 1u) * 0x1p-24f));
}

__device__ __forceinline__ float sin_halfpi(float r, float r2) {
  float p = 0x1.507834p-13f;   //  (pi/2)^9 / 9!
  p = fmaf(p, r2, -0x1.32d2ccp-8f);  // -(pi/2)^7 / 7!
  p = fmaf(p, r2, 0x1.466bc6p-4f);   //  (pi/2)^5 / 5!
  p = fmaf(p, r2, -0x1.4abbcep-1f);  // -(pi/2)^3 / 3!
  p = fmaf(p, r2, 0x1.921fb6p+0f);   //   pi/2
  return p * r;
}

__device__ __forceinline__ float cos_halfpi(float r2) {
  float p = -0x1.a6d1f2p-16f;        // -(pi/2)^10 / 10!
  p = fmaf(p, r2, 0x1.e1f506p-11f);  //  (pi/2)^8 / 8!
  p = fmaf(p, r2, -0x1.55d3c8p-6f);  // -(pi/2)^6 / 6!
  p = fmaf(p, r2, 0x1.03c1f0p-2f);   //  (pi/2)^4 / 4!
  p = fmaf(p, r2, -0x1.3bd3ccp+0f);  // -(pi/2)^2 / 2!
  return fmaf(p, r2, 1.0f);
}

// v, negated when bit 1 of the quadrant q is set.
__device__ __forceinline__ float with_sign_of_bit1(float v, int q) {
  return __uint_as_float(__float_as_uint(v) ^ (((uint32_t)q << 30) & 0x80000000u));
}

__device__ __forceinline__ void box_muller(uint32_t rf, uint32_t af, float& z0, float& z1) {
  const float rad = bm_radius(rf);
  const float x = (float)af * 0x1p-16f;  // 4 t, exact
  const float q = rintf(x);
  const float r = x - q, r2 = r * r;
  const float sn = sin_halfpi(r, r2), cs = cos_halfpi(r2);
  const int qi = (int)q;
  const float ss = (qi & 1) ? cs : sn, cc = (qi & 1) ? sn : cs;
  z0 = rad * with_sign_of_bit1(cc, qi + 1);
  z1 = rad * with_sign_of_bit1(ss, qi);
}

// The cosine branch alone.
__device__ __forceinline__ float box_muller_cos(uint32_t rf, uint32_t af) {
  const float rad = bm_radius(rf);
  const float x = (float)af * 0x1p-16f;
  const float q = rintf(x);
  const float r = x - q, r2 = r * r;
  const int qi = (int)q;
  const float cc = (qi & 1) ? sin_halfpi(r, r2) : cos_halfpi(r2);
  return rad * with_sign_of_bit1(cc, qi + 1);
}

__device__ __forceinline__ void box_muller64(uint32_t r, uint32_t a, double& z0, double& z1) {
  const double rad = sqrt(-2.0 * log(((double)r + 1.0) * 0x1p-24));
  double s, c;
  sincospi((double)a * 0x1p-17, &s, &c);  // 2 t
  z0 = rad * c;
  z1 = rad * s;
}

// x as an integer, saturated to the int range (NaN reads as 0).
__device__ __forceinline__ int cvt_sat_i32(double x) {
  int r;
  asm("v_cvt_i32_f64 %0, %1" : "=v"(r) : "v"(x));
  return r;
}

// A constant kept in scalar registers: the compiler otherwise moves it into a
// vector register pair before each fused multiply-add that overwrites it.
__device__ __forceinline__ double sconst(double c) {
  asm("" : "+s"(c));
  return c;
}

// e^x for finite x: Cody-Waite reduction x = k ln2 + r with ln 2 split into
// a 32-bit head (k * head exact) and a tail, |r| <= ln2 / 2, and the Taylor
// polynomial of degree 11 (truncation below 7e-15 relative); the result is
// scaled by 2^k (0 below the subnormal range, inf above the finite one).
__device__ __forceinline__ double exp_fast(double x) {
  const double k = rint(x * 0x1.71547652b82fep+0);  // x / ln 2
  double r = fma(-k, 0x1.62e42fee00000p-1, x);
  r = fma(-k, 0x1.a39ef35793c76p-33, r);
  double p = 0x1.ae64567f544e4p-26;     // 1/11!
  p = fma(p, r, 0x1.27e4fb7789f5cp-22);  // 1/10!
  p = fma(p, r, 0x1.71de3a556c734p-19);  // 1/9!
  p = fma(p, r, 0x1.a01a01a01a01ap-16);  // 1/8!
  p = fma(p, r, 0x1.a01a01a01a01ap-13);  // 1/7!
  p = fma(p, r, 0x1.6c16c16c16c17p-10);  // 1/6!
  p = fma(p, r, 0x1.1111111111111p-7);   // 1/5!
  p = fma(p, r, 0x1.5555555555555p-5);   // 1/4!
  p = fma(p, r, 0x1.5555555555555p-3);   // 1/3!
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  return ldexp(p, cvt_sat_i32(k));
}

// ------------------------------------------------------ wave64 primitives
// Cross-lane moves use DPP within rows of 16 lanes: row shifts (row_shr:k;
// lanes whose source falls outside the row read 0 and are masked off by the
// callers) for scans, row rotations (row_ror:k) for reductions, and either
// v_readlane for the four row results or row broadcasts that carry them into
// the last row. Every helper must be called with all 64 lanes active.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}

template <int CTRL>
__device__ __forceinline__ int dpp(int v) {
  return (int)dpp32<CTRL>((uint32_t)v);
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return dpp32<CTRL>(v);
}
template <int CTRL>
__device__ __forceinline__ uint64_t dpp(uint64_t v) {
  return (uint64_t)dpp32<CTRL>((uint32_t)v) | ((uint64_t)dpp32<CTRL>((uint32_t)(v >> 32)) << 32);
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  return __longlong_as_double((long long)dpp<CTRL>((uint64_t)__double_as_longlong(v)));
}
template <int K, class T>
__device__ __forceinline__ T shr(T v) {
  return dpp<0x110 + K>(v);
}
template <int K, class T>
__device__ __forceinline__ T ror(T v) {
  return dpp<0x120 + K>(v);
}

__device__ __forceinline__ int readlane(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
// The wave's index within its workgroup, as a wave-uniform (scalar) value.
__device__ __forceinline__ int wave_index() {
  return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
}
__device__ __forceinline__ uint64_t readlane(uint64_t v, int l) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ double readlane(double v, int l) {
  return __longlong_as_double((long long)readlane((uint64_t)__double_as_longlong(v), l));
}

struct OpAdd {
  template <class T>
  __device__ __forceinline__ T operator()(T a, T b) const { return a + b; }
};
struct OpMax {
  __device__ __forceinline__ double operator()(double a, double b) const { return fmax(a, b); }
  __device__ __forceinline__ uint64_t operator()(uint64_t a, uint64_t b) const {
    return a > b ? a : b;
  }
  __device__ __forceinline__ int operator()(int a, int b) const { return a > b ? a : b; }
};
struct OpMin {
  __device__ __forceinline__ int operator()(int a, int b) const { return a < b ? a : b; }
};
// Inclusive scan within each row of 16 lanes (r = lane & 15).
template <class T, class Op>
__device__ __forceinline__ T row_scan(T v, int r, Op op) {
  T t = shr<1>(v);
  if (r >= 1) v = op(v, t);
  t = shr<2>(v);
  if (r >= 2) v = op(v, t);
  t = shr<4>(v);
  if (r >= 4) v = op(v, t);
  t = shr<8>(v);
  if (r >= 8) v = op(v, t);
  return v;
}

// Reduction within each row of 16 lanes; every lane receives its row's
// result, combined in an order fixed for each lane.
template <class T, class Op>
__device__ __forceinline__ T row_allreduce(T v, Op op) {
  v = op(v, ror<1>(v));
  v = op(v, ror<2>(v));
  v = op(v, ror<4>(v));
  v = op(v, ror<8>(v));
  return v;
}

// Reduction over the wave, in a fixed order (result uniform).
template <class T, class Op>
__device__ __forceinline__ T wave_reduce(T v, int lane, Op op) {
  (void)lane;
  v = row_allreduce(v, op);
  return op(op(readlane(v, 0), readlane(v, 16)), op(readlane(v, 32), readlane(v, 48)));
}

// Row broadcasts: CTRL 0x142 (row_bcast:15) hands lane 15 of each row to the
// whole next row, CTRL 0x143 (row_bcast:31) hands lane 31 to rows 2 and 3.
// Only the rows in the mask ROWS receive; the others read `id`.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t bcast32(uint32_t v, uint32_t id) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)id, (int)v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ int bcast(int v, int id) {
  return (int)bcast32<CTRL, ROWS>((uint32_t)v, (uint32_t)id);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double bcast(double v, double id) {
  const uint64_t x = (uint64_t)__double_as_longlong(v), z = (uint64_t)__double_as_longlong(id);
  const uint64_t r = (uint64_t)bcast32<CTRL, ROWS>((uint32_t)x, (uint32_t)z) |
                     ((uint64_t)bcast32<CTRL, ROWS>((uint32_t)(x >> 32), (uint32_t)(z >> 32))
                      << 32);
  return __longlong_as_double((long long)r);
}

// Combines each odd row's result with the even row before it: after a
// row_allreduce, rows 1 and 3 hold op(row 0, row 1) and op(row 2, row 3).
template <class T, class Op>
__device__ __forceinline__ T pair_rows(T v, Op op, T id) {
  return op(v, bcast<0x142, 0xa>(v, id));
}

// Reduction over the wave whose result is exact in lane 63 only (no
// v_readlane): rows paired by row_bcast:15, then the pairs by row_bcast:31.
// id is the identity of op.
template <class T, class Op>
__device__ __forceinline__ T wave_reduce_last(T v, Op op, T id) {
  v = pair_rows(row_allreduce(v, op), op, id);
  return op(v, bcast<0x143, 0xc>(v, id));
}

// Order-preserving integer key of a float that is not NaN: a < b exactly
// when key(a) < key(b) (-0 sorts just below +0), and key + 1 is the key of
// the next float up.
__device__ __forceinline__ int ord_key(float f) {
  const int x = __float_as_int(f);
  return x ^ ((x >> 31) & 0x7fffffff);
}
__device__ __forceinline__ float ord_val(int k) {
  return __int_as_float(k ^ ((k >> 31) & 0x7fffffff));
}
// Key of the smallest float >= x (x not NaN).
__device__ __forceinline__ int ord_key_up(double x) {
  const float f = (float)x;
  return ord_key(f) + ((double)f < x ? 1 : 0);
}

// Inclusive scan over the wave, in a fixed order.
template <class T, class Op>
__device__ __forceinline__ T wave_scan(T v, int lane, Op op) {
  v = row_scan(v, lane & 15, op);
  const T r0 = readlane(v, 15), r1 = readlane(v, 31), r2 = readlane(v, 47);
  const int row = lane >> 4;
  if (row == 1)
    v = op(r0, v);
  else if (row == 2)
    v = op(op(r0, r1), v);
  else if (row == 3)
    v = op(op(op(r0, r1), r2), v);
  return v;
}

// Exclusive prefix sum of exact unsigned integers over a 256-thread
// workgroup; *total receives the sum of all.
__device__ __forceinline__ uint64_t block_excl_sum(uint64_t v, uint64_t* sh, uint64_t* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint64_t inc = wave_scan(v, lane, OpAdd());
  if (lane == 63) sh[w] = inc;
  __syncthreads();
  uint64_t before = 0;
  for (int j = 0; j < w; ++j) before += sh[j];
  *total = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  return before + inc - v;
}

// ------------------------------------------------------------ k_init
// The Morton key of the top 16 bits of two words: x's bits at the even
// positions, y's at the odd ones (each spread by doubling its bit distance).
__device__ __forceinline__ uint32_t spread16(uint32_t v) {
  v &= 0xffffu;
  v = (v | (v << 8)) & 0x00ff00ffu;
  v = (v | (v << 4)) & 0x0f0f0f0fu;
  v = (v | (v << 2)) & 0x33333333u;
  return (v | (v << 1)) & 0x55555555u;
}
__device__ __forceinline__ uint32_t zorder_key(uint32_t wx, uint32_t wy) {
  return spread16(wx >> 16) | (spread16(wy >> 16) << 1);
}
__device__ __forceinline__ void init_state(const Model& m, int64_t i, float* xs);
// Algorithm 1 initialisation, k = 0. The state is computed in fp64 and
// rounded once to fp32.
__device__ __forceinline__ void init_body(const Model& m, const Buffers& b, int64_t blk) {
  const int64_t i = blk * kBlock + threadIdx.x;
  if (i == 0) {
    Ctrl* c = b.ctrl;
    c->k = 0;
    c->cur = 0;
    c->mode = kModeInit;
    c->resampled = 0;
    c->rolled_back = 0;
    c->do_resample = 0;
    c->heavy_count = 0;
    c->m = c->log_sum = c->ess = c->delta = c->cum = 0.0;
    for (int d = 0; d < 5; ++d) c->mean[d] = 0.0;
    c->u = 0.0;
    c->total = 0;
    for (int d = 0; d < kNGrad; ++d) c->grad_cum[d] = c->grad_last[d] = 0.0;
    c->ring_key = 0;
    c->delta_ref = -INFINITY;
    c->lost = 0;
    c->arna_tracking = 0;
    c->arna_moved = 0;
  }
  if (i >= m.n) return;
  if (m.grad)
    for (int d = 0; d < kNTan; ++d) b.T0[(int64_t)d * m.n + i] = 0.0f;
  if (m.init_kind == 3) {
    // Z order: the sort key of draw i; k_init_place writes the states
    const uint4 r0 = draw(m, (uint32_t)i, 0u, kInit, 0u);
    b.zkey0[i] = zorder_key(r0.x, r0.y);
    return;
  }
  float xs[5];
  init_state(m, i, xs);
#pragma unroll
  for (int d = 0; d < 5; ++d) b.X0[(int64_t)d * m.n + i] = xs[d];
}

// The initial state of draw i (kinds 0-2; kind 3 draws as kind 0).
__device__ __forceinline__ void init_state(const Model& m, int64_t i, float* xs) {
  const uint4 r0 = draw(m, (uint32_t)i, 0u, kInit, 0u);
  const uint4 r1 = draw(m, (uint32_t)i, 0u, kInit, 1u);
  double x[5];
  if (m.init_kind == 1) {  // Gaussian
    double z[5], unused;
    const NormalFields nf = normal_fields(r0);
    box_muller64(nf.r0, nf.a0, z[0], z[1]);
    box_muller64(nf.r1, nf.a1, z[2], z[3]);
    box_muller64(nf.r2, nf.a2, z[4], unused);
#pragma unroll
    for (int d = 0; d < 5; ++d) x[d] = (double)m.init_a[d] + (double)m.init_b[d] * z[d];
  } else {
    const uint32_t w[5] = {r0.x, r0.y, r0.z, r0.w, r1.x};
    double f[5];
#pragma unroll
    for (int d = 0; d < 5; ++d) f[d] = (double)u24_open_hi(w[d]);
    if (m.init_kind == 2) {  // stratified over (x, y) in Z order
      const int t = m.strat_t;
      const uint64_t cell = ((uint64_t)i << t) / (uint64_t)m.n;
      uint32_t cx = 0, cy = 0;
      int bx = 0, by = 0;
      for (int j = 0; j < t; ++j) {
        const uint32_t bit = (uint32_t)(cell >> j) & 1u;
        if ((j & 1) == 0)
          cx |= bit << bx++;
        else
          cy |= bit << by++;
      }
      const double fx = ((double)cx + (double)u24_open_hi(r0.x)) / ldexp(1.0, (t + 1) / 2);
      const double fy = ((double)cy + (double)u24_open_hi(r0.y)) / ldexp(1.0, t / 2);
      f[0] = fx;
      f[1] = fy;
      f[2] = (double)u24_open_hi(r0.z);
      f[3] = (double)u24_open_hi(r0.w);
      f[4] = (double)u24_open_hi(r1.x);
    }
#pragma unroll
    for (int d = 0; d < 5; ++d)
      x[d] = (double)m.init_a[d] + ((double)m.init_b[d] - (double)m.init_a[d]) * f[d];
  }
#pragma unroll
  for (int d = 0; d < 5; ++d) xs[d] = (float)x[d];
}

__global__ __launch_bounds__(256) void k_init(Model m, Buffers b) { init_body(m, b, blockIdx.x); }

// Z-ordered init: position p takes draw zval0[p] (the keys sorted, stably).
__global__ __launch_bounds__(256) void k_init_place(Model m, Buffers b) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= m.n) return;
  float xs[5];
  init_state(m, (int64_t)b.zval0[p], xs);
#pragma unroll
  for (int d = 0; d < 5; ++d) b.X0[(int64_t)d * m.n + p] = xs[d];
}

// ------------------------------------------------------------ k_step
// Parent, carried log weight and propagated state of particle i.
struct Prop {
  float x, y, vx, vy, I;
};

// The particle's log weight before the new observation: its stored weight
// carried over (no resampling this step), its group's weight after RNA, a
// caller-set weight, or -log N after systematic resampling. Kept out of
// propagate so that kernels compute it only where the likelihood is added,
// instead of holding it across the patch sums.
// amv: the slots exchanged by the last ARNA resampling (the control block's).
__device__ __forceinline__ double prior_lw(const Model& m, const Buffers& b, int cur, int mode,
                                           double delta, int amv, int64_t i) {
  if (mode == kModeNone) {
    const float* Ein = cur ? b.E1 : b.E0;
    const double* Rin = cur ? b.R1 : b.R0;
    return log((double)Ein[i]) + Rin[(i / kBlock) * kRec] - delta;
  }
  if (mode == kModeRna) {
    const int64_t g = i / m.group;
    const int64_t l = i - g * m.group;
    const int64_t src = (l >= m.group - m.moved) ? (g + m.G - 1) % m.G : g;
    return b.lwg[src];
  }
  if (mode == kModeArna) {
    const int64_t g = i / m.group;
    const int64_t l = i - g * m.group;
    return (l >= m.group - amv) ? b.lwt[g] : b.lwg[g];
  }
  if (mode == kModeSet) return b.lw64[i];
  return -m.log_n;
}

// Addresses of a block's particles: a wave-uniform base and the thread's index in
// the block, so that an access needs no 64-bit vector arithmetic.
//
// Particle base + t of a block; zo (5 normals) and po (the parent) are optional
// outputs for the tangents.
__device__ __forceinline__ Prop propagate(const Model& m, const Buffers& b, int cur, int mode,
                                          int64_t base, uint32_t t, uint32_t k,
                                          float* zo = nullptr, int64_t* po = nullptr) {
  const float* Xin = cur ? b.X1 : b.X0;
  const uint32_t i = (uint32_t)base + t;  // particle indices are below 2^31
  // Loaded whatever the mode, so that it does not wait for the control block's word:
  // control block, ancestor and parent were three dependent loads at a wave's start
  // (100 K particles, linear-Gaussian step 5.4 -> 5.0 us; 1 M, 9 x 9 patch 26.3 -> 25.3;
  // 38 M, 13 x 13 patch 948 -> 942 a launch).
  const uint32_t a = (uint32_t)(b.anc + base)[t];
  const uint32_t p = (mode == kModeSys || mode == kModeRna || mode == kModeArna) ? a : i;
  const int64_t n = m.n;
  float px, py, pvx, pvy, pI;
  if (n <= (int64_t)1 << 30) {  // uniform: byte offsets of 32 bits
    auto at = [&](int d) {
      return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(Xin + d * n) + 4u * p);
    };
    px = at(0);
    py = at(1);
    pvx = at(2);
    pvy = at(3);
    pI = at(4);
  } else {
    px = Xin[p];
    py = Xin[n + p];
    pvx = Xin[2 * n + p];
    pvy = Xin[3 * n + p];
    pI = Xin[4 * n + p];
    // (keeps the compiler from folding the two ways into this one)
    asm volatile("" : "+v"(px), "+v"(py), "+v"(pvx), "+v"(pvy), "+v"(pI));
  }
  const NormalFields nf = normal_fields(draw(m, i, k, kPropagate, 0u));
  float z0, z1, z2, z3;
  box_muller(nf.r0, nf.a0, z0, z1);
  box_muller(nf.r1, nf.a1, z2, z3);
  const float z4 = box_muller_cos(nf.r2, nf.a2);
  if (zo) {
    zo[0] = z0;
    zo[1] = z1;
    zo[2] = z2;
    zo[3] = z3;
    zo[4] = z4;
  }
  if (po) *po = (int64_t)p;
  Prop o;
  // near-constant velocity, unit frame interval; in fp32 with one fused
  // multiply-add per component, the small velocity and noise terms first,
  // so a position is within half an ulp (plus the rounding of that small
  // sum) of the exact value
  o.x = px + fmaf(m.q[0], z0, pvx);
  o.y = py + fmaf(m.q[1], z1, pvy);
  o.vx = fmaf(m.q[2], z2, pvx);
  o.vy = fmaf(m.q[3], z3, pvy);
  o.I = fmaf(m.q[4], z4, pI);
  return o;
}

// The new states stream past the caches (non-temporal stores): the next
// step gathers them through the ancestors long after, and left in the
// caches as dirty lines their write-back would compete with the weight
// stream of the resampling pass that follows.
__device__ __forceinline__ void store_state(const Model& m, const Buffers& b, int cur,
                                            int64_t base, uint32_t t, const Prop& o) {
  float* Xout = (cur ? b.X0 : b.X1) + base;
  const int64_t n = m.n;
  __builtin_nontemporal_store(o.x, Xout + t);
  __builtin_nontemporal_store(o.y, Xout + n + t);
  __builtin_nontemporal_store(o.vx, Xout + 2 * n + t);
  __builtin_nontemporal_store(o.vy, Xout + 3 * n + t);
  __builtin_nontemporal_store(o.I, Xout + 4 * n + t);
}

// Fixed-point weight of a particle whose weight relative to its block
// maximum is e in [0, 1]: round(e 2^44), an exact integer held in a double
// (e 2^44 is an exact exponent shift below 2^52; rint rounds it once, half
// to even).
__device__ __forceinline__ double item_weight(double e) {
  static_assert(kItemScale == 0x1p44, "the scale is applied as an exponent shift");
  return rint(ldexp(e, 44));
}

// e^x for x <= 0 rounded to fp32 (0 below -104, where e^x is under half the
// least fp32 subnormal). Cody-Waite reduction x = k ln 2 + r with one fp64
// constant (|k| <= 150 keeps its error below 2^-47) and the Taylor polynomial
// of degree 9 on |r| <= ln 2 / 2 (truncation below 2^-36 relative): the fp64
// value is far closer to e^x than the fp32 rounding step.
__device__ __forceinline__ float exp_neg_f32(double x) {
  const double k = rint(x * 0x1.71547652b82fep+0);
  const double r = fma(-k, 0x1.62e42fefa39efp-1, x);
  double p = fma(sconst(0x1.71de3a556c734p-19), r,  // 1/9!
                 sconst(0x1.a01a01a01a01ap-16));    // 1/8!
  p = fma(p, r, sconst(0x1.a01a01a01a01ap-13));     // 1/7!
  p = fma(p, r, sconst(0x1.6c16c16c16c17p-10));     // 1/6!
  p = fma(p, r, sconst(0x1.1111111111111p-7));      // 1/5!
  p = fma(p, r, sconst(0x1.5555555555555p-5));      // 1/4!
  p = fma(p, r, sconst(0x1.5555555555555p-3));      // 1/3!
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  const float v = (float)ldexp(p, cvt_sat_i32(k));
  return x < -104.0 ? 0.0f : v;
}

// The block's normalisation record (see kRec) and the stored weights
// E = exp(l - m_b) in fp32. red: 7 x 256 doubles of LDS that no thread reads
// once it has reached this call (it may alias the caller's image tile); dsh
// and ksh: 4 doubles and 4 ints of LDS scratch.
// Returns e = E (0 for an inactive or non-finite particle).
//
// The shift m_b is any value at or above every finite l of the block and
// close to their maximum (the record carries it, so the normalisation does
// not depend on which): the maximum of the l rounded up to fp32, taken as
// order-preserving integer keys so that each DPP step is one v_max_i32, and
// within one fp32 ulp of the largest l. Where that ulp exceeds 1/8 (block
// maxima of magnitude 2^20 and above) the exact fp64 maximum is taken instead.
__device__ __forceinline__ double finish_block(const Buffers& b, int cur, int64_t blk,
                                               bool active, double l, const Prop& o, double* red,
                                               double* dsh, int* ksh) {
  // lane tests compare t with wave-uniform values, so no lane index stays live
  const int t = threadIdx.x, w = wave_index(), t0 = 64 * w;
  const bool bad = active && (isnan(l) || l == INFINITY);
  const bool ok = active && !bad;
  const int wk = wave_reduce_last(ok ? ord_key_up(l) : ord_key(-INFINITY), OpMax(), INT_MIN);
  if (t == t0 + 63) ksh[w] = wk;
  __syncthreads();
  const float mf = ord_val(max(max(ksh[0], ksh[1]), max(ksh[2], ksh[3])));
  double mb = (double)mf;
  if (mf != -INFINITY && !(fabsf(mf) < 0x1p20f)) {  // uniform across the workgroup
    const double wm = wave_reduce_last(ok ? l : -INFINITY, OpMax(), (double)-INFINITY);
    if (t == t0 + 63) dsh[w] = wm;
    __syncthreads();
    mb = fmax(fmax(dsh[0], dsh[1]), fmax(dsh[2], dsh[3]));
  }
  double e = 0.0;
  if (active) {
    float Ef = 0.0f;
    if (bad) {
      Ef = NAN;
    } else if (l != -INFINITY) {  // then m_b >= l > -inf
      Ef = exp_neg_f32(l - mb);
      e = (double)Ef;
    }
    float* Eout = (cur ? b.E0 : b.E1) + blk * kBlock;
    Eout[(uint32_t)t] = Ef;
  }
  const double wi = item_weight(e);
  // after the barrier above every thread is past its reads of the LDS that
  // red may alias
  red[t] = wi;
  red[256 + t] = bad ? NAN : e * e;
  red[512 + t] = e * (double)o.x;
  red[768 + t] = e * (double)o.y;
  red[1024 + t] = e * (double)o.vx;
  red[1280 + t] = e * (double)o.vy;
  red[1536 + t] = e * (double)o.I;
  __syncthreads();
  double s = 0.0;
  if (t < 224) {  // value t >> 5, eight consecutive entries (t & 31) * 8 ...
    const double* p = red + (t >> 5) * 256 + (t & 31) * 8;
    s = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
  }
  // value 2w in row 1 of wave w, value 2w + 1 in row 3
  s = pair_rows(row_allreduce(s, OpAdd()), OpAdd(), 0.0);
  double* R = (cur ? b.R0 : b.R1) + blk * kRec;
  if (t == t0 + 16) R[1 + 2 * w] = s;
  if (t == t0 + 48 && 2 * w + 1 < 7) R[2 + 2 * w] = s;
  if (t == 0) R[0] = mb;
  return e;
}

// LDS of one step workgroup: two copies of the tile of D = Z - b, each in
// one half of the first TILE doubles of `tile` (the first 7 x 256 of them
// double as the record exchange), then SQ doubles for the table of row sums of
// D^2; a workgroup whose box does not fit twice keeps one tile in all of it.
// And the reduction scratch. Kernels that run several patch sizes declare it
// once. The table has an entry per tile row and centre column, fewer than a
// copy has pixels: TILE / 2 doubles hold it (gradient mode keeps two tables in
// kSqCap), which lets six and seven workgroups share a CU where 1536 doubles
// let five and six.
template <int TILE, int SQ = TILE / 2>
struct StepLds {
  static_assert(TILE >= 7 * kBlock, "the tile doubles as the record exchange buffer");
  __align__(16) double tile[TILE + SQ];
  double dsh[4];
  int ish[16];
  int ksh[4];
};

// Patch sums of one particle over P rows of an LDS tile of D = Z - b (0
// outside the frame) with row stride tw, every row starting on 16 bytes:
//   X   += sum_dy g_y(dy) sum_dx D g_x(dx)    (Gaussian-weighted residual sum)
//   G2y += g_y^2
//   sd2 += sum D^2, from the table of row sums hrow (stride hs) when TAB,
//          else pixel by pixel.
// g_y is advanced by the exact recurrence g(d+1) = g(d) gstep(d) exp(f/s^2).
// gx[0] is 1, so each row's sum starts at its first pixel (an fma with a zero
// addend would cost an add, to turn -0 into +0; D = Z - b is never -0 here).
template <int P, bool TAB>
__device__ __forceinline__ void patch_lds(const double* __restrict__ p0, int tw,
                                          const double* __restrict__ hrow, int hs,
                                          const double (&gx)[P], double gy, double by,
                                          const double* gstep, double& X, double& G2y,
                                          double& sd2) {
#pragma unroll
  for (int dy = 0; dy < P; ++dy) {
    const double* row = static_cast<const double*>(__builtin_assume_aligned(p0 + dy * tw, 16));
    double rd = row[0];
    if (!TAB) sd2 = fma(rd, rd, sd2);
#pragma unroll
    for (int dx = 1; dx < P; ++dx) {
      const double d = row[dx];
      rd = fma(d, gx[dx], rd);
      if (!TAB) sd2 = fma(d, d, sd2);
    }
    if (TAB) sd2 += hrow[dy * hs];
    X = fma(gy, rd, X);
    G2y = fma(gy, gy, G2y);
    gy *= gstep[dy] * by;
  }
}

// The same sums, pixel by pixel in the same order, from a tile kept once
// (row stride tw, no alignment): D as doubles, or the pixels themselves as
// floats, the background subtracted here (pixels outside the frame are staged
// as the background, so their D is 0 either way).
template <int P, class T>
__device__ __forceinline__ void patch_single(const T* __restrict__ p0, int tw, double bsub,
                                             const double (&gx)[P], double gy, double by,
                                             const double* gstep, double& X, double& G2y,
                                             double& sd2) {
#pragma unroll 1
  for (int dy = 0; dy < P; ++dy) {
    const T* row = p0 + dy * tw;
    double rd = 0.0;
#pragma unroll
    for (int dx = 0; dx < P; ++dx) {
      double d;
      if constexpr (sizeof(T) == sizeof(double))
        d = row[dx];
      else
        d = (double)row[dx] - bsub;
      rd = dx == 0 ? d : fma(d, gx[dx], rd);
      sd2 = fma(d, d, sd2);
    }
    X = fma(gy, rd, X);
    G2y = fma(gy, gy, G2y);
    gy *= gstep[dy] * by;
  }
}

// The same sums read straight from the frame (waves whose patches fit no LDS
// tile); pixels outside the frame read as the background.
//
// A check and a branch per pixel make each load wait for the one before it, and
// then more waves on a CU (as the LDS up to 13 x 13 allows since their table takes
// half the tile) only make the frame's lines push each other out of the cache: 2^22
// particles spread over 90 x 90 pixels, 5 x 5 patches 201 us with five workgroups on
// a CU and 221 with six, 9 x 9 472 and 521. So a row's pixels (C of them at a time,
// as many as take no register more than the rest of the step) are loaded together,
// from one 32-bit offset: 124 and 204 us. A wave with a patch over a border, below
// 13 x 13, loads the frame's nearest column for the pixels beyond it and takes 0 for
// them, and skips the columns and the rows that lie outside for all its patches:
// 2^21 particles around the centre of a 512 x 512 frame, 200 pixels to a standard
// deviation, 5 x 5 155 -> 75 us, 9 x 9 434 -> 183, 11 x 11 636 -> 246. Wider patches
// there keep the check per pixel: 13 x 13 in the six-wave shape would spill, and a
// dense cloud on a border, most of whose pixels the check saves, takes 855 us with
// 25 x 25 patches and took 966 with the columns clamped.
template <int P>
__device__ __forceinline__ void patch_global(const float* __restrict__ obs, int u0, int v0,
                                             int W, int H, double bsub, const double (&gx)[P],
                                             double gy, double by, const double* gstep,
                                             double& X, double& G2y, double& sd2) {
  constexpr int C = P <= 7 ? P : P == 11 ? 6 : 5;
  const bool inside = u0 >= 0 && v0 >= 0 && u0 <= W - P && v0 <= H - P;
  if ((int64_t)W * H <= (int64_t)1 << 30) {  // byte offsets of 32 bits
    const char* const base = reinterpret_cast<const char*>(obs);
    uint32_t at = 4u * ((uint32_t)v0 * (uint32_t)W);  // modulo 2^32 above the frame
    if (__ballot(!inside) == 0) {
      at += 4u * (uint32_t)u0;
#pragma unroll 1
      for (int dy = 0; dy < P; ++dy) {
        double rd = 0.0;
#pragma unroll
        for (int d0 = 0; d0 < P; d0 += C) {
          float z[C];
#pragma unroll
          for (int dx = d0; dx < min(d0 + C, P); ++dx)
            z[dx - d0] = *reinterpret_cast<const float*>(base + 4 * dx + at);
#pragma unroll
          for (int dx = d0; dx < min(d0 + C, P); ++dx) {
            const double d = (double)z[dx - d0] - bsub;
            rd = dx == 0 ? d : fma(d, gx[dx], rd);
            sd2 = fma(d, d, sd2);
          }
          if (C < P) __builtin_amdgcn_sched_barrier(0);  // z's registers are the next ones'
        }
        X = fma(gy, rd, X);
        G2y = fma(gy, gy, G2y);
        gy *= gstep[dy] * by;
        at += 4u * (uint32_t)W;
      }
      return;
    }
    if constexpr (P < kFusedMaxP) {
      uint32_t some = 0;  // bit d0 / C: a patch of the wave has one of these columns inside
#pragma unroll
      for (int d0 = 0; d0 < P; d0 += C)
        if (__ballot(u0 + min(d0 + C, P) > 0 && u0 + d0 < W) != 0) some |= 1u << (d0 / C);
#pragma unroll 1
      for (int dy = 0; dy < P; ++dy) {
        double rd = 0.0;
        if ((unsigned)(v0 + dy) < (unsigned)H && u0 > -P && u0 < W) {
#pragma unroll
          for (int d0 = 0; d0 < P; d0 += C) {
            if (!(some >> (d0 / C) & 1)) continue;  // uniform in the wave
            float z[C];
#pragma unroll
            for (int dx = d0; dx < min(d0 + C, P); ++dx)
              z[dx - d0] = *reinterpret_cast<const float*>(
                  base + (at + 4u * (uint32_t)min(max(u0 + dx, 0), W - 1)));
#pragma unroll
            for (int dx = d0; dx < min(d0 + C, P); ++dx) {
              const double d =
                  (unsigned)(u0 + dx) < (unsigned)W ? (double)z[dx - d0] - bsub : 0.0;
              rd = fma(d, gx[dx], rd);  // (gx[0] = 1)
              sd2 = fma(d, d, sd2);
            }
            if (C < P) __builtin_amdgcn_sched_barrier(0);
          }
        }
        X = fma(gy, rd, X);
        G2y = fma(gy, gy, G2y);
        gy *= gstep[dy] * by;
        at += 4u * (uint32_t)W;
      }
      return;
    }
  }
#pragma unroll 1
  for (int dy = 0; dy < P; ++dy) {
    const int v = v0 + dy;
    const bool row_in = (unsigned)v < (unsigned)H;
    const float* row = obs + (int64_t)(row_in ? v : 0) * W;
    double rd = 0.0;
#pragma unroll
    for (int dx = 0; dx < P; ++dx) {
      const int u = u0 + dx;
      const double d = (row_in && (unsigned)u < (unsigned)W) ? (double)row[u] - bsub : 0.0;
      rd = dx == 0 ? d : fma(d, gx[dx], rd);
      sd2 = fma(d, d, sd2);
    }
    X = fma(gy, rd, X);
    G2y = fma(gy, gy, G2y);
    gy *= gstep[dy] * by;
  }
}

// Gradient mode: moments of one particle's patch. With D = Z - b (0 outside
// the frame), the Gaussian factors g = g_x g_y and the integer offsets
// a = dx - h, c = dy - h of a pixel from the patch centre:
//   X0 = sum D g,  X1 = sum D g a,  X2 = sum D g a^2,
//   Y1 = sum D g c,  Y2 = sum D g c^2,
//   B0, B1, B2 = sum_dy g_y^2 c^{0,1,2},  SD = sum D,
//   Gin = sum of g_y over the rows inside the frame,
//   sd2 = sum D^2 (from the row-sum table when TAB).
// X0, B0 and sd2 are accumulated in the same order as patch_lds, so the log
// weights equal those of the plain step.
struct Moments {
  double X0, X1, X2, Y1, Y2, B0, B1, B2, SD, Gin, sd2;
};

template <int P>
__device__ __forceinline__ void moments_row(const double (&d)[P], const double (&gx)[P], int dy,
                                            double gy, bool row_in, bool pix_sq, bool pix_sum,
                                            Moments& mo) {
  constexpr int h = (P - 1) / 2;
  // u = D g_x along the row. s0 = sum u (the plain step's order), and the
  // running sums of running sums s1 = sum_j u_j m_j, s2 = sum_j u_j m_j
  // (m_j + 1) / 2 with m_j = P - j give the moments in a = j - h = c0 - m_j
  // (c0 = h + 1) without a product per pixel:
  //   sum u a = c0 s0 - s1,   sum u a^2 = c0^2 s0 - 2 c0 s1 + 2 s2 - s1.
  // (gx[0] = 1: the sums start at the first pixel, as in patch_lds)
  double s0 = d[0], s1 = s0, s2 = s0, sd = d[0];
  if (pix_sq) mo.sd2 = fma(d[0], d[0], mo.sd2);
#pragma unroll
  for (int dx = 1; dx < P; ++dx) {
    s0 = fma(d[dx], gx[dx], s0);
    s1 += s0;
    s2 += s1;
    if (pix_sum) sd += d[dx];
    if (pix_sq) mo.sd2 = fma(d[dx], d[dx], mo.sd2);
  }
  constexpr double c0 = (double)(h + 1);
  const double r1 = fma(c0, s0, -s1);
  const double r2 = fma(c0 * c0, s0, fma(-2.0 * c0, s1, 2.0 * s2 - s1));
  const double c = (double)(dy - h);
  mo.X0 = fma(gy, s0, mo.X0);
  mo.X1 = fma(gy, r1, mo.X1);
  mo.X2 = fma(gy, r2, mo.X2);
  const double gr = gy * s0;
  mo.Y1 = fma(gr, c, mo.Y1);
  mo.Y2 = fma(gr, c * c, mo.Y2);
  mo.B0 = fma(gy, gy, mo.B0);
  const double g2 = gy * gy;
  mo.B1 = fma(g2, c, mo.B1);
  mo.B2 = fma(g2, c * c, mo.B2);
  if (pix_sum) mo.SD += sd;
  if (row_in) mo.Gin += gy;
}

// Rows from the LDS tile (TAB: sum D^2 of each row from the row-sum table
// hrow; SUMTAB: sum D from hsum as well) or from the frame; v0 is the frame
// row of the patch's first row.
template <int P, bool TAB, bool SUMTAB, bool GLOBAL>
__device__ __forceinline__ void patch_moments(const double* __restrict__ p0, int tw,
                                              const double* __restrict__ hrow,
                                              const double* __restrict__ hsum, int hs,
                                              const float* __restrict__ obs, int u0, double bsub,
                                              int W, int H, int64_t v0,
                                              const double (&gx)[P], double gy, double by,
                                              const double* gstep, Moments& mo) {
#pragma unroll 1
  for (int dy = 0; dy < P; ++dy) {
    const int64_t v = v0 + dy;
    const bool row_in = v >= 0 && v < H;
    double d[P];
    if (GLOBAL) {
      const float* row = obs + (row_in ? v : 0) * (int64_t)W;
#pragma unroll
      for (int dx = 0; dx < P; ++dx) {
        const int u = u0 + dx;
        d[dx] = (row_in && (unsigned)u < (unsigned)W) ? (double)row[u] - bsub : 0.0;
      }
    } else {
      const double* row =
          static_cast<const double*>(__builtin_assume_aligned(p0 + dy * tw, 16));
#pragma unroll
      for (int dx = 0; dx < P; ++dx) d[dx] = row[dx];
    }
    moments_row<P>(d, gx, dy, gy, row_in, !TAB, !SUMTAB, mo);
    if (TAB) mo.sd2 += hrow[dy * hs];
    if (SUMTAB) mo.SD += hsum[dy * hs];
    gy *= gstep[dy] * by;
  }
}

// Propagation and log weight of one particle per thread (Eq. 4 with the spot
// of Eq. 3 on the P x P patch). The residual sum is expanded as
//   sum (D - I g)^2 = sum D^2 - 2 I sum D g + I^2 sum g^2,   D = Z - b,
// (D = 0 for pixels outside the frame) with sum g^2 = (sum g_x^2)(sum g_y^2);
// everything in fp64. The workgroup stages D over the bounding box of its
// patches in LDS as fp64 (the conversion is paid once per pixel, not once per
// particle and pixel) and, when small enough, a table of the P-pixel row sums
// of D^2 at every patch-centre column, so a particle adds P table entries
// instead of squaring P^2 pixels.
// Five barriers per workgroup: the box, the tile, the table, the block
// maximum, and the record exchange.
template <int P, bool GRAD = false, int TILE = kTileCap>
__device__ __forceinline__ void step_spot(const Model& m, const Buffers& b,
                                          const float* __restrict__ obs, int64_t blk,
                                          StepLds<TILE, GRAD ? kSqCap : TILE / 2>& L) {
  constexpr int h = (P - 1) / 2;
  constexpr int kSq = GRAD ? kSqCap : TILE / 2;  // doubles of the table
  double* const tile = L.tile;
  double* const sq = L.tile + TILE;
  double* const dsh = L.dsh;
  int* const ish = L.ish;
  const Ctrl* cp = b.ctrl;
  const int cur = cp->cur, mode = cp->mode, amv = cp->arna_moved;
  const double cdelta = cp->delta;
  const uint32_t k = (uint32_t)(cp->k + 1);
  const int t = threadIdx.x, w = wave_index();
  const int64_t base = blk * kBlock;
  const int rem = (int)min((int64_t)kBlock, m.n - base);  // the block's particles
  const bool active = t < rem;
  // Lanes past the last particle (the tail of the last workgroup) repeat the
  // work of particle n - 1, which lies in the same workgroup, and store
  // nothing: every lane runs the same instructions on valid data.
  const int ta = min(t, rem - 1);

  Prop o;
  float tg[kNTan];  // gradient mode: the particle's new tangents
  if constexpr (GRAD) {
    float z[5];
    int64_t p;
    o = propagate(m, b, cur, mode, base, ta, k, z, &p);
    // tangents along the ancestral line (see kNTan): dx'/dq_x = dx/dq_x +
    // z_x, dx'/dq_vx = dx/dq_vx + dvx/dq_vx (the parent's), and alike
    const float* Tin = cur ? b.T1 : b.T0;
    float* Tout = cur ? b.T0 : b.T1;
    float tp[kNTan];
#pragma unroll
    for (int d = 0; d < kNTan; ++d) tp[d] = Tin[(int64_t)d * m.n + p];
    tg[0] = (float)((double)tp[0] + (double)z[0]);
    tg[1] = (float)((double)tp[1] + (double)z[1]);
    tg[2] = (float)((double)tp[2] + (double)z[2]);
    tg[3] = (float)((double)tp[3] + (double)tp[2]);
    tg[4] = (float)((double)tp[4] + (double)z[3]);
    tg[5] = (float)((double)tp[5] + (double)tp[4]);
    tg[6] = (float)((double)tp[6] + (double)z[4]);
    if (active)  // streamed like the states
#pragma unroll
      for (int d = 0; d < kNTan; ++d)
        __builtin_nontemporal_store(tg[d], Tout + (int64_t)d * m.n + base + (uint32_t)t);
  } else {
    o = propagate(m, b, cur, mode, base, ta, k);
  }
  if (active) store_state(m, b, cur, base, t, o);
  // patch centre: pixel nearest to (x, y); the offset f is exact in fp64
  const double rx = floor((double)o.x + 0.5);
  const double ry = floor((double)o.y + 0.5);
  const double fx = (double)o.x - rx;
  const double fy = (double)o.y - ry;
  // addresses only: far-away centres are clamped to [-P, W + P] x [-P, H + P]
  // (cx_max, cy_max: on the host, as W + P may pass the largest int),
  // where the whole patch already lies outside the frame (its pixels read as
  // background); a NaN centre reads as 0 (its weight is NaN: the step is rolled
  // back)
  const int cx = min(max(cvt_sat_i32(rx), -P), m.cx_max);
  const int cy = min(max(cvt_sat_i32(ry), -P), m.cy_max);
  // The 1-D Gaussian factors of Eq. 3 at the patch's pixel offsets. Only
  // their products g_x g_y enter the likelihood, so g_x is taken relative to
  // its first value, which moves into the first g_y: three exps per particle
  // (the host keeps both first values above e^-350, so the product stays
  // normal).
  double gx[P];
  gx[0] = 1.0;
  const double bx = exp_fast(fx * m.is2);
#pragma unroll
  for (int d = 0; d + 1 < P; ++d) gx[d + 1] = gx[d] * (m.gstep[d] * bx);
  double G2x = 0.0;
#pragma unroll
  for (int d = 0; d < P; ++d) G2x = fma(gx[d], gx[d], G2x);
  const double ax = (double)h + fx, ay = (double)h + fy;
  const double gy0 = exp_fast(-(ax * ax + ay * ay) * m.inv2s2);
  const double by = exp_fast(fy * m.is2);
  // Bounding box of the workgroup's patch centres (the tail lanes repeat
  // particle n - 1, whose centre is in the box anyway): four reductions whose
  // every step is one instruction with its lane move.
  {
    const int x0 = wave_reduce_last(cx, OpMin(), INT_MAX), x1 = wave_reduce_last(cx, OpMax(), INT_MIN);
    const int y0 = wave_reduce_last(cy, OpMin(), INT_MAX), y1 = wave_reduce_last(cy, OpMax(), INT_MIN);
    if (t == 64 * w + 63) {
      ish[w] = x0;
      ish[4 + w] = x1;
      ish[8 + w] = y0;
      ish[12 + w] = y1;
    }
  }
  __syncthreads();
  // the box as scalars: everything that follows from it (sizes, strides, the
  // choice of path) is then scalar work, off the vector units that bound the
  // kernel
  const int mnx = __builtin_amdgcn_readfirstlane(min(min(ish[0], ish[1]), min(ish[2], ish[3])));
  const int mxx = __builtin_amdgcn_readfirstlane(max(max(ish[4], ish[5]), max(ish[6], ish[7])));
  const int mny = __builtin_amdgcn_readfirstlane(min(min(ish[8], ish[9]), min(ish[10], ish[11])));
  const int mxy = __builtin_amdgcn_readfirstlane(max(max(ish[12], ish[13]), max(ish[14], ish[15])));
  // The tile is staged twice, copy B shifted one column left of copy A, each
  // in half of the LDS block with an even row stride: a patch row starting
  // at an even column is read from A, one starting at an odd column from B,
  // so every row starts on 16 bytes and is read with 128-bit LDS loads.
  // 128-bit reads meet the banks in 16-byte granules, 16 granules to a bank
  // row; copy B starts 8 granules after the half, so that the patch rows of
  // two neighbouring centres (one in each copy) fall 8 granules apart.
  constexpr int kCopy = TILE / 2;  // doubles per half
  constexpr int kOffB = 16;        // copy B's start within its half, in doubles
  static_assert(kCopy % 2 == 0, "copies must keep 16-byte alignment");
  const int64_t tw64 = (int64_t)mxx - mnx + P, th64 = (int64_t)mxy - mny + P;
  const int64_t ts2min = (tw64 + 1) >> 1;  // row stride in pairs of doubles
  const bool use_lds = 2 * ts2min * th64 <= kCopy - kOffB;  // uniform across the workgroup
  const int tw = (int)tw64, th = (int)th64;
  const int tx0 = mnx - h, ty0 = mny - h;
  const int64_t acx = (int64_t)mxx - mnx + 1;
  const int64_t nH = th64 * acx;
  const bool use_tab = use_lds && nH <= kSq;  // (the plain step's always fits)
  // gradient mode also tables the row sums of D, in the upper half, when both
  // fit (the D^2 table is used exactly when the plain step uses it, so the log
  // weights stay the plain step's)
  constexpr int kTab = kSqCap / 2;
  const bool use_sum = GRAD && use_lds && nH <= kTab;
  // Row stride ts = 2 ts2, with ts2 padded to ceil(acx / 2) (mod 16): the
  // granule where a patch row of the centre (cx, cy) starts is then
  // (cy - mny) ceil(acx / 2) + (cx - mnx) / 2 (+ 8 in copy B) (mod 16), so
  // lanes at distinct centres of a small box meet distinct granules (this
  // layout measured a fifth of the bank-conflict cycles of 8-granule rules).
  int ts2 = (int)ts2min;
  {
    const int padh = ((int)(((acx + 1) >> 1) & 15) - (ts2 & 15)) & 15;
    if ((int64_t)2 * (ts2 + padh) * th <= kCopy - kOffB) ts2 += padh;
  }
  const int ts = 2 * ts2;
  if (use_lds) {
    // one pass over the tile's pixels (row r = e / tw from the hardware
    // reciprocal, corrected by one step: e < 2^11 and the reciprocal is
    // within 1 ulp, so the estimate is off by at most 1)
    const int nt = tw * th;
    const float rcpw = __builtin_amdgcn_rcpf((float)tw);
    for (int e = t; e < nt; e += 256) {
      int r = (int)((float)e * rcpw);
      if (r * tw > e) --r;
      else if ((r + 1) * tw <= e) ++r;
      const int c = e - r * tw, v = ty0 + r, u = tx0 + c;
      const double dv = ((unsigned)v < (unsigned)m.H && (unsigned)u < (unsigned)m.W)
                            ? (double)obs[(int64_t)v * m.W + u] - m.b
                            : 0.0;
      tile[r * ts + c] = dv;
      if (c > 0) tile[kCopy + kOffB + r * ts + c - 1] = dv;
    }
  }
  // A box too large for two copies and the table is kept once, in all of the
  // workgroup's LDS, as doubles or (twice the pixels) as floats; where even
  // that is too small (a workgroup whose particles form clusters, as at a jump
  // of the Z order), each wave keeps its own box in a quarter of it, and a
  // wave whose box still does not fit reads the frame. The sums are taken in
  // the frame path's order, so the choice moves no bit. Over a border of the frame
  // a box is staged only whole, and only if its particles fill it: where they do
  // not, the waves' own boxes are small, so that the loads of each meet few lines,
  // and those of patches outside the frame are left out. The waves' boxes together
  // have to cover the workgroup's twice (four times in a box that is filled): 3.2
  // million particles around the middle column of a 96 x 512 frame, 60 pixels to a
  // standard deviation, with every box staged and with this rule 11 x 11 patches 116
  // and 79 us, 15 x 15 151 and 141; 2^21 particles that fill 44 x 44 pixels on a
  // corner, staged and from the frame, 11 x 11 102 and 130 us. Inside, 2^20 particles
  // in four clusters to a workgroup, staged and from the frame, in a box that fits
  // 25 x 25 169 and 237 us, wave by wave 111 and 237. Patches up to 3 x 3 are not
  // staged, nor 5 x 5, nor 7 x 7 where the box lies in the frame: staging takes more
  // loads than reading their pixels (2^22 particles spread over 68 x 68 pixels, staged
  // and from the frame: a step 1 x 1 138 and 85 us, 3 x 3 149 and 98, 5 x 5 157 and
  // 121, 7 x 7 170 and 141, 9 x 9 187 and 189). Gradient mode keeps the two choices: a
  // third cost its kernel 2 % (registers) on clouds that never need it.
  constexpr int kAll = TILE + kSq;
  enum { kFrame, kFloat, kDouble };
  int single = kFrame;  // uniform in a wave
  int sx0 = tx0, sy0 = ty0, sw = 0, sbase = 0;
  const bool inside = tx0 >= 0 && ty0 >= 0 && mxx < m.W - h && mxy < m.H - h;
  bool stage = P >= 9 && inside;  // uniform in the workgroup
  if (!GRAD && !use_lds && P >= 7 && !inside && tw64 * th64 <= 2 * kAll) {
    int own = 0;  // pixels of the waves' boxes
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int x0 = __builtin_amdgcn_readfirstlane(ish[i]);
      const int x1 = __builtin_amdgcn_readfirstlane(ish[4 + i]);
      const int y0 = __builtin_amdgcn_readfirstlane(ish[8 + i]);
      const int y1 = __builtin_amdgcn_readfirstlane(ish[12 + i]);
      own += (x1 - x0 + P) * (y1 - y0 + P);
    }
    stage = own >= 2 * tw * th;
  }
  if (!GRAD && !use_lds && stage) {
    int64_t bw = tw64, bh = th64, cap = kAll;
    int e0 = t, step = 256;
    if (bw * bh > 2 * (int64_t)kAll) {  // uniform in the workgroup
      const int x0 = __builtin_amdgcn_readfirstlane(ish[w]);
      const int x1 = __builtin_amdgcn_readfirstlane(ish[4 + w]);
      const int y0 = __builtin_amdgcn_readfirstlane(ish[8 + w]);
      const int y1 = __builtin_amdgcn_readfirstlane(ish[12 + w]);
      bw = (int64_t)x1 - x0 + P;
      bh = (int64_t)y1 - y0 + P;
      cap = kAll / 4;
      sbase = w * (kAll / 4);
      sx0 = x0 - h;
      sy0 = y0 - h;
      e0 = t & 63;
      step = 64;
    }
    const int64_t np = bw * bh;
    single = np <= cap ? kDouble : np <= 2 * cap ? kFloat : kFrame;
    if (single != kFrame) {
      sw = (int)bw;
      const int nt = (int)np;
      const float rcpw = __builtin_amdgcn_rcpf((float)sw);
      float* const ftile = reinterpret_cast<float*>(tile + sbase);
      for (int e = e0; e < nt; e += step) {
        int r = (int)((float)e * rcpw);
        if (r * sw > e) --r;
        else if ((r + 1) * sw <= e) ++r;
        const int v = sy0 + r, u = sx0 + (e - r * sw);
        const float z = ((unsigned)v < (unsigned)m.H && (unsigned)u < (unsigned)m.W)
                            ? obs[(int64_t)v * m.W + u]
                            : (float)m.b;
        if (single == kDouble)
          tile[sbase + e] = (double)z - m.b;
        else
          ftile[e] = z;
      }
    }
  }
  __syncthreads();
  if (use_tab) {
    // sq[r * acx + c] = sum_dx (Z[r][c + dx] - b)^2 over the tile's rows r and
    // the centres' columns c (gradient mode: sq[kTab + r * acx + c] = sum_dx
    // (Z[r][c + dx] - b), both in the per-pixel order)
    const int ax = (int)acx, nh = (int)nH;
    const float rcp = __builtin_amdgcn_rcpf((float)ax);
    for (int e = t; e < nh; e += 256) {
      int r = (int)((float)e * rcp);
      if (r * ax > e) --r;
      else if ((r + 1) * ax <= e) ++r;
      const double* src = tile + r * ts + (e - r * ax);
      double sacc = 0.0, dsum = 0.0;
#pragma unroll
      for (int dx = 0; dx < P; ++dx) {
        sacc = fma(src[dx], src[dx], sacc);
        if (GRAD) dsum += src[dx];
      }
      sq[e] = sacc;
      if (GRAD && use_sum) sq[kTab + e] = dsum;
    }
  }
  __syncthreads();

  // every lane's patch lies in the tile (the tail lanes' is particle
  // n - 1's); finish_block ignores the tail lanes' l
  double l;
  double gth[GRAD ? kNGrad : 1] = {};
  // the particle's first patch row in copy A (even first column) or B (odd)
  const int col0 = cx - h - tx0;
  const double* p0 =
      tile + ((cy - h - ty0) * ts + (col0 & ~1) + ((col0 & 1) ? kCopy + kOffB : 0));
  if constexpr (GRAD) {
    Moments mo{};
    // frame row of the patch's first row; centres far outside are clamped,
    // as for the addresses (every row of such a patch is outside the frame)
    const int64_t v0 = (int64_t)fmin(fmax(ry, -(double)P - 1.0), (double)m.H + P + 1.0) - h;
    // table index of the centre (below nH where a table is used)
    const int at = use_tab ? (cy - mny) * (int)acx + (cx - mnx) : 0;
    if (use_sum) {
      patch_moments<P, true, true, false>(p0, ts, sq + at, sq + kTab + at, (int)acx, obs, 0,
                                          m.b, m.W, m.H, v0, gx, gy0, by, m.gstep, mo);
    } else if (use_tab) {
      patch_moments<P, true, false, false>(p0, ts, sq + at, sq, (int)acx, obs, 0, m.b, m.W,
                                           m.H, v0, gx, gy0, by, m.gstep, mo);
    } else if (use_lds) {
      patch_moments<P, false, false, false>(p0, ts, sq, sq, 0, obs, 0, m.b, m.W, m.H, v0, gx,
                                            gy0, by, m.gstep, mo);
    } else {
      patch_moments<P, false, false, true>(p0, 0, sq, sq, 0, obs, cx - h, m.b, m.W, m.H, v0, gx,
                                           gy0, by, m.gstep, mo);
    }
    const double I = (double)o.I;
    const double ssq = mo.sd2 - 2.0 * I * mo.X0 + I * I * (G2x * mo.B0);
    l = prior_lw(m, b, cur, mode, cdelta, amv, base + ta) - ssq * m.inv2sig2 - m.lognorm_obs;
    // 1-D moments of g_x^2 and the in-frame sum of g_x (true centre rx)
    double A1 = 0.0, A2 = 0.0, Gin_x = 0.0;
#pragma unroll
    for (int dx = 0; dx < P; ++dx) {
      const double g2 = gx[dx] * gx[dx];
      A1 = fma(g2, (double)(dx - h), A1);
      A2 = fma(g2, (double)((dx - h) * (dx - h)), A2);
      const double u = rx + (double)(dx - h);
      if (u >= 0.0 && u < (double)m.W) Gin_x += gx[dx];
    }
    const double A0 = G2x, B0 = mo.B0;
    // moments in the offsets from the particle, e = a - f
    const double ex1 = mo.X1 - fx * mo.X0;
    const double ex2 = mo.X2 - 2.0 * fx * mo.X1 + fx * fx * mo.X0;
    const double ey1 = mo.Y1 - fy * mo.X0;
    const double ey2 = mo.Y2 - 2.0 * fy * mo.Y1 + fy * fy * mo.X0;
    const double gx1 = A1 - fx * A0, gx2 = A2 - 2.0 * fx * A1 + fx * fx * A0;
    const double gy1 = mo.B1 - fy * B0, gy2 = mo.B2 - 2.0 * fy * mo.B1 + fy * fy * B0;
    const double isg2 = 2.0 * m.inv2sig2, is2 = 2.0 * m.inv2s2;
    const double lI = (mo.X0 - I * A0 * B0) * isg2;
    const double lx = I * isg2 * is2 * (ex1 - I * B0 * gx1);
    const double ly = I * isg2 * is2 * (ey1 - I * A0 * gy1);
    const double ls = I * isg2 * is2 / m.s_psf * (ex2 + ey2 - I * (B0 * gx2 + A0 * gy2));
    const double lb = isg2 * (mo.SD - I * Gin_x * mo.Gin);
    const double lsig = ssq / (m.sig * m.sig * m.sig) - (double)(P * P) / m.sig;
    gth[0] = ls;
    gth[1] = lb;
    gth[2] = lsig;
    gth[3] = lx * (double)tg[0];
    gth[4] = ly * (double)tg[1];
    gth[5] = lx * (double)tg[3];
    gth[6] = ly * (double)tg[5];
    gth[7] = lI * (double)tg[6];
    gth[8] = lI;
  } else {
    double X = 0.0, G2y = 0.0, sd2 = 0.0;
    if (use_tab) {
      // the table index is below nH <= kSq: 32-bit arithmetic
      patch_lds<P, true>(p0, ts, sq + ((cy - mny) * (int)acx + (cx - mnx)), (int)acx, gx, gy0,
                         by, m.gstep, X, G2y, sd2);
    } else if (use_lds) {
      patch_lds<P, false>(p0, ts, sq, 0, gx, gy0, by, m.gstep, X, G2y, sd2);
    } else if (single != kFrame) {
      const int at = (cy - h - sy0) * sw + (cx - h - sx0);  // in the wave's own box
      if (single == kDouble)
        patch_single<P>(tile + sbase + at, sw, m.b, gx, gy0, by, m.gstep, X, G2y, sd2);
      else
        patch_single<P>(reinterpret_cast<const float*>(tile + sbase) + at, sw, m.b, gx, gy0, by,
                        m.gstep, X, G2y, sd2);
    } else {
      patch_global<P>(obs, cx - h, cy - h, m.W, m.H, m.b, gx, gy0, by, m.gstep, X, G2y, sd2);
    }
    const double I = (double)o.I;
    const double ssq = sd2 - 2.0 * I * X + I * I * (G2x * G2y);
    l = prior_lw(m, b, cur, mode, cdelta, amv, base + ta) - ssq * m.inv2sig2 - m.lognorm_obs;
  }
  // the MMSE sums convert the state anew: kept in doubles since the patch's centre was
  // taken, it would be the registers that the widest fused patch lacks
  if constexpr (P == kFusedMaxP && !GRAD) asm("" : "+v"(o.x), "+v"(o.y));
  const double e = finish_block(b, cur, blk, active, l, o, tile, dsh, L.ksh);
  if constexpr (GRAD) {
    // the block's sum_i E_i d l_i / d theta, weighted like the MMSE sums and
    // reduced the same way: derivatives 0-7 through the tile, 8 through the
    // table's space, eight consecutive entries per thread, then rows
    static_assert(kNGrad == 9 && TILE >= 8 * kBlock && kSqCap >= kBlock,
                  "eight derivatives fill the tile, the ninth goes to the table");
    double v[kNGrad];
#pragma unroll
    for (int d = 0; d < kNGrad; ++d) v[d] = (e > 0.0) ? e * gth[d] : 0.0;
    __syncthreads();  // every thread is past finish_block's reads of the tile
#pragma unroll
    for (int d = 0; d < 8; ++d) tile[d * kBlock + t] = v[d];
    sq[t] = v[8];
    __syncthreads();
    const double* p = tile + (t >> 5) * kBlock + (t & 31) * 8;
    double s = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
    s = pair_rows(row_allreduce(s, OpAdd()), OpAdd(), 0.0);
    double* RGb = b.RG + blk * kNGrad;
    // derivative 2w in row 1 of wave w, 2w + 1 in row 3
    if (t == 64 * w + 16) RGb[2 * w] = s;
    if (t == 64 * w + 48) RGb[2 * w + 1] = s;
    if (w == 0) {  // uniform: the first wave sums derivative 8
      double s8 = 0.0;
      if (t < 32) {
        const double* q = sq + t * 8;
        s8 = ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7]));
      }
      s8 = pair_rows(row_allreduce(s8, OpAdd()), OpAdd(), 0.0);
      if (t == 16) RGb[8] = s8;
    }
  }
}

// Patches up to 13 x 13 come in two workgroup shapes: five waves per SIMD, or
// six with a smaller tile; wider patches keep the compiler's default budget.
template <int P, int S>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kShapeWaves[S])))
void k_step_spot(Model m, Buffers b, const float* __restrict__ obs) {
  __shared__ StepLds<kShapeTile[S]> L;
  step_spot<P, false, kShapeTile[S]>(m, b, obs, blockIdx.x, L);
}

template <int P>
__global__ __launch_bounds__(256) void k_step_spot_wide(Model m, Buffers b,
                                                        const float* __restrict__ obs) {
  __shared__ StepLds<kTileCap> L;
  step_spot<P>(m, b, obs, blockIdx.x, L);
}

// Gradient mode (derivatives of log p^ alongside the step).
template <int P>
__global__ __launch_bounds__(256) void k_step_spot_grad(Model m, Buffers b,
                                                        const float* __restrict__ obs) {
  __shared__ StepLds<kTileCap, kSqCap> L;
  step_spot<P, true>(m, b, obs, blockIdx.x, L);
}

// Linear-Gaussian observation of (x, y, I0): three fp32 values on the device.
__global__ __launch_bounds__(256) void k_step_lg(Model m, Buffers b,
                                                 const float* __restrict__ obs) {
  __shared__ double red[7 * 256];
  __shared__ double dsh[4];
  __shared__ int ksh[4];
  const Ctrl* cp = b.ctrl;
  const int cur = cp->cur, mode = cp->mode, amv = cp->arna_moved;
  const double cdelta = cp->delta;
  const uint32_t k = (uint32_t)(cp->k + 1);
  const int64_t base = (int64_t)blockIdx.x * kBlock, i = base + threadIdx.x;
  const bool active = i < m.n;
  Prop o{};
  double l = -INFINITY;
  if (active) {
    o = propagate(m, b, cur, mode, base, threadIdx.x, k);
    store_state(m, b, cur, base, threadIdx.x, o);
    const double ex = (double)obs[0] - (double)o.x, ey = (double)obs[1] - (double)o.y,
                 eI = (double)obs[2] - (double)o.I;
    l = prior_lw(m, b, cur, mode, cdelta, amv, i) - ex * ex * m.lg_inv2r2[0] - ey * ey * m.lg_inv2r2[1] - eI * eI * m.lg_inv2r2[2] -
        m.lg_norm;
  }
  finish_block(b, cur, blockIdx.x, active, l, o, red, dsh, ksh);
}

// Records of caller-supplied absolute fp32 log weights (standalone
// resampling): the same layout, with weights e = exp(x - m) in fp64 and zero
// state sums. One wave per block, four consecutive weights per lane: the block
// maximum is a fp32 maximum of the fp32 inputs (exact), the fixed-point weights
// sum exactly in any order, and no barrier waits. The kernel is bound by issue,
// most of it the exps; with one weight per lane its fp64 maximum, two barriers
// and LDS sums took 57 us for 16.8 M weights, against 30.5 us.
__global__ __launch_bounds__(256) void k_records(Model m, Buffers b,
                                                 const float* __restrict__ logw) {
  const int lane = threadIdx.x & 63;
  const int64_t blk = (int64_t)blockIdx.x * 4 + wave_index();
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    // the standalone scratch starts uninitialised: clear the counters and
    // flags the following kernels of this call rely on
    Ctrl* c = b.ctrl;
    c->heavy_count = 0;
    c->do_resample = 0;
    c->total = 0;
    c->cur = 0;
    c->k = 0;
  }
  if (blk >= b.nb) return;  // whole waves; no barrier follows
  const int64_t i = blk * kBlock + 4 * lane;
  float x[4];
  if (i + 4 <= m.n && (reinterpret_cast<uintptr_t>(logw) & 15) == 0) {
    const float4 v = *reinterpret_cast<const float4*>(logw + i);
    x[0] = v.x;
    x[1] = v.y;
    x[2] = v.z;
    x[3] = v.w;
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = i + q < m.n ? logw[i + q] : -INFINITY;
  }
  bool bad = false;
  int key = ord_key(-INFINITY);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const bool bq = !(x[q] < INFINITY);  // NaN or +inf
    bad = bad || bq;
    key = bq ? key : max(key, ord_key(x[q]));
  }
  const float mf = ord_val(readlane(wave_reduce_last(key, OpMax(), INT_MIN), 63));
  const double mb = (double)mf;
  double sums[2] = {0.0, 0.0};  // fixed-point weights, sum e^2
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double e = x[q] > -INFINITY && x[q] < INFINITY ? exp((double)x[q] - mb) : 0.0;
    sums[0] += item_weight(e);
    sums[1] = fma(e, e, sums[1]);
  }
  if (bad) sums[1] = NAN;
#pragma unroll
  for (int k = 0; k < 2; ++k) sums[k] = wave_reduce_last(sums[k], OpAdd(), 0.0);
  // lane 63 holds the sums, every lane the maximum
  double* R = b.R0 + blk * kRec;
  if (lane == 63) {
    R[0] = mb;
    R[1] = sums[0];
    R[2] = sums[1];
  } else if (lane < 5) {
    R[3 + lane] = 0.0;
  }
}

// ------------------------------------------------------------- k_merge
// Two launches. Each workgroup of the first merges one chunk of block
// records relative to the chunk's maximum: the chunk record, and per block
// the exclusive prefix of the chunk's integer weights q_b = round(B_b
// exp(m_b - M_c)). One workgroup of the second merges the chunk records in a
// fixed order, takes the statistics of Algorithm 1 (normaliser, ESS, MMSE
// estimate), decides on resampling, commits or rolls back the step, and for
// systematic resampling writes each chunk's fixed-point CDF prefix. (The
// kernel boundary makes the chunk records visible to it: waiting for the
// last chunk inside one launch costs a device-scope release and acquire in
// every workgroup, which write back and invalidate that XCD's L2.)
//
// These launches are latency: kernel arguments, the control block, the
// records, then a chain of reductions and exps on a few waves, 3.5-5 us each.
// So a record is loaded from both buffers before the control block has told
// which one counts, a thread keeps its record in registers, and one wave holds
// up to 64 chunks and takes the scalar results in every lane (no broadcast, one
// division for the five means). With at most kOneMergeChunks chunks of 256
// records one launch does both, the chunks side by side in one workgroup and
// their records in LDS: 4096 particles 3.5 + 4.9 us in two launches, 5.5 us in
// one; 100,003 3.9 + 4.8 and 5.7 us; 262,144 with derivatives 5.4 + 6.8 and 9.1
// us (a gap between two launches is another 1 us or so).
struct MergeSh {
  double mx[4];
  uint64_t q[4];
  double sums[4 * 7];
  double grads[4 * kNGrad];
};

// Wave results combined over the four waves w of a 256-thread group (one wave
// alone when WAVES is 1: the absent ones would add zeros). Each sh is used
// once.
template <int WAVES, class T, class Op>
__device__ __forceinline__ T group_reduce(T v, T* sh, int w, Op op) {
  v = wave_reduce(v, 0, op);
  if (WAVES == 1) return v;
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  return op(op(sh[0], sh[1]), op(sh[2], sh[3]));
}
template <int WAVES, int K>
__device__ __forceinline__ void group_sum_n(double (&v)[K], double* sh, int w) {
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = wave_reduce_last(v[k], OpAdd(), 0.0);
  if (WAVES == 1) {
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = readlane(v[k], 63);
    return;
  }
  if ((threadIdx.x & 63) == 63) {
#pragma unroll
    for (int k = 0; k < K; ++k) sh[w * K + k] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = (sh[k] + sh[K + k]) + (sh[2 * K + k] + sh[3 * K + k]);
}
template <int WAVES>
__device__ __forceinline__ uint64_t group_excl_sum(uint64_t v, uint64_t* sh, int w,
                                                   uint64_t* total) {
  const int lane = threadIdx.x & 63;
  const uint64_t inc = wave_scan(v, lane, OpAdd());
  if (WAVES == 1) {
    *total = readlane(inc, 63);
    return inc - v;
  }
  if (lane == 63) sh[w] = inc;
  __syncthreads();
  uint64_t before = 0;
  for (int j = 0; j < w; ++j) before += sh[j];
  *total = sh[0] + sh[1] + sh[2] + sh[3];
  return before + inc - v;
}

// Merges chunk ch (records past the last chunk's end contribute nothing) with
// the 256 threads t of a group whose waves are w: the blocks' prefixes, and by
// thread 0 the chunk record and derivative record. ONE: a chunk is 256 records,
// one per thread.
template <bool ONE>
__device__ __forceinline__ void merge_chunk_body(const Model& m, const Buffers& b, int standalone,
                                                 int64_t ch, int t, int w, MergeSh& sh, double* cr,
                                                 double* crg) {
  const int64_t lo = ch * b.chunk, hi = min(b.nb, lo + b.chunk);
  const int per = ONE ? 1 : (int)(b.chunk / 256);
  const int64_t j0 = lo + (int64_t)t * per;
  constexpr int kPer = ONE ? 1 : kMergePer;  // records per thread at most

  double rec[kRec], rec1[kRec];  // ONE: the thread's record, from either buffer
  if (ONE) {
    const int64_t j = min(j0, b.nb - 1) * kRec;
#pragma unroll
    for (int d = 0; d < kRec; ++d) rec[d] = b.R0[j + d];
    if (!standalone)
#pragma unroll
      for (int d = 0; d < kRec; ++d) rec1[d] = b.R1[j + d];
  }
  const int which = standalone ? 0 : (b.ctrl->cur ^ 1);  // the records this step wrote
  const double* R = which ? b.R1 : b.R0;
  double mx = -INFINITY;
  if (ONE) {
    if (which)
#pragma unroll
      for (int d = 0; d < kRec; ++d) rec[d] = rec1[d];
    if (j0 < hi) mx = rec[0];
  } else {
    for (int q = 0; q < per; ++q) {
      const int64_t j = j0 + q;
      if (j < hi) mx = fmax(mx, R[j * kRec]);
    }
  }
  const double Mc = group_reduce<4>(mx, sh.mx, w, OpMax());
  uint64_t qs = 0, qj[kPer];
  double sums[6] = {};  // sum E^2, then sum E x
  double gs[kNGrad] = {};
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int64_t j = j0 + q;
    qj[q] = 0;
    if (q < per && j < hi) {
      const double* r = ONE ? rec : R + j * kRec;
      const double f = (r[0] == -INFINITY) ? 0.0 : exp(r[0] - Mc);
      qj[q] = (uint64_t)rint(r[1] * f);
      qs += qj[q];
      sums[0] += r[2] * (f * f);
#pragma unroll
      for (int d = 0; d < 5; ++d) sums[1 + d] += r[3 + d] * f;
      if (m.grad && f != 0.0)
#pragma unroll
        for (int d = 0; d < kNGrad; ++d) gs[d] += b.RG[j * kNGrad + d] * f;
    }
  }
  uint64_t qtot;
  uint64_t run = group_excl_sum<4>(qs, sh.q, w, &qtot);
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int64_t j = j0 + q;
    if (q < per && j < hi) {
      b.pfx[j] = run;
      run += qj[q];
    }
  }
  group_sum_n<4>(sums, sh.sums, w);
  if (t == 0) {
    cr[0] = Mc;
    cr[1] = __longlong_as_double((long long)qtot);
#pragma unroll
    for (int d = 0; d < 6; ++d) cr[2 + d] = sums[d];
  }
  if (m.grad) {
    group_sum_n<4, kNGrad>(gs, sh.grads, w);
    if (t == 0)
#pragma unroll
      for (int d = 0; d < kNGrad; ++d) crg[d] = gs[d];
  }
}

// With derivatives, by columns: lane d of a row of 16 takes sum d of kSums (sum E^2,
// sum E x, the derivatives) and the rows take the records in turn, so that a wave reads
// whole records and ends with two exchanges between its rows. A thread to a record
// needs six exchanges for each of the 15 sums, 270 fp64 steps a wave instead of 20, and
// its loads touch a line per lane: 262,144 particles in four chunks 10.8 -> 9.1 us.
// Without derivatives the wait for the factors costs more than that saves (two chunks
// 5.7 -> 6.1 us, and 7.5 with the columns of both buffers loaded ahead), so those keep
// a thread to a record.
constexpr int kSums = 6 + kNGrad;
static_assert(kSums <= 16 && kRec == 8, "a lane of a row per sum");
struct SumColumn {
  const double* p;  // the column's value in record 0
  int stride;
  bool grad;
  __device__ __forceinline__ SumColumn(const double* R, const double* RG, int d) {
    grad = d >= 6 && d < kSums;
    p = grad ? RG + (d - 6) : R + (d < 6 ? 2 + d : 0);  // (lanes past the sums: unused)
    stride = grad ? kNGrad : kRec;
  }
};

// Sum over the wave's four rows of 16 lanes, lane by lane.
__device__ __forceinline__ double sum_of_rows(double v) {
  typedef uint32_t U2 __attribute__((ext_vector_type(2)));
  auto pair = [](U2 lo, U2 hi) {
    auto d = [](uint32_t l, uint32_t h) {
      return __longlong_as_double((long long)(((uint64_t)h << 32) | l));
    };
    return d(lo.x, hi.x) + d(lo.y, hi.y);
  };
  uint64_t x = (uint64_t)__double_as_longlong(v);
  uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32);
  v = pair(__builtin_amdgcn_permlane16_swap(lo, lo, false, false),
           __builtin_amdgcn_permlane16_swap(hi, hi, false, false));
  x = (uint64_t)__double_as_longlong(v);
  lo = (uint32_t)x;
  hi = (uint32_t)(x >> 32);
  return pair(__builtin_amdgcn_permlane32_swap(lo, lo, false, false),
              __builtin_amdgcn_permlane32_swap(hi, hi, false, false));
}

// The same for a chunk of 256 records with derivatives, by columns. fac: LDS for the
// records' factors, part: for its waves' sums.
__device__ __forceinline__ void merge_chunk_deriv(const Model& m, const Buffers& b, int ch,
                                                  int t, int w, MergeSh& sh, double* fac,
                                                  double* part, double* cr, double* crg) {
  const int64_t lo = ch * 256, hi = min(b.nb, lo + 256), j = lo + t;
  const int64_t jr = min(j, b.nb - 1) * kRec;
  double rm = b.R0[jr], rq = b.R0[jr + 1];  // the thread's record, from either buffer
  const double rm1 = b.R1[jr], rq1 = b.R1[jr + 1];
  const int which = b.ctrl->cur ^ 1;  // the records this step wrote
  const double* R = which ? b.R1 : b.R0;
  const int d = t & 15, row = t >> 4;
  const SumColumn col(R, b.RG, d);
  double x[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) x[q] = col.p[min(lo + q * 16 + row, hi - 1) * col.stride];
  if (which) {
    rm = rm1;
    rq = rq1;
  }
  const double Mc = group_reduce<4>(j < hi ? rm : -INFINITY, sh.mx, w, OpMax());
  const double f = (j < hi && rm != -INFINITY) ? exp(rm - Mc) : 0.0;
  const uint64_t qj = j < hi ? (uint64_t)rint(rq * f) : 0;
  fac[t] = f;
  uint64_t qtot;
  const uint64_t run = group_excl_sum<4>(qj, sh.q, w, &qtot);  // (its barrier covers fac)
  if (j < hi) b.pfx[j] = run;
  double acc = 0.0;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const double fe = fac[q * 16 + row];
    const double y = x[q] * (d == 0 ? fe * fe : fe);
    acc += (col.grad && fe == 0.0) ? 0.0 : y;
  }
  acc = sum_of_rows(acc);
  if ((t & 63) < 16) part[w * 16 + d] = acc;
  __syncthreads();
  if (t < 16) {
    const double v = (part[t] + part[16 + t]) + (part[32 + t] + part[48 + t]);
    if (t < 6) cr[2 + t] = v;
    if (col.grad) crg[t - 6] = v;
    if (t == 0) {
      cr[0] = Mc;
      cr[1] = __longlong_as_double((long long)qtot);
    }
  }
}

// By one workgroup of WAVES waves holding the chunks (at most 64 with one
// wave); CR, CRG: the chunk records, in global memory or in LDS. BYCOL: one wave and
// up to kOneMergeChunks chunks, their sums by columns; fac: LDS for their factors.
template <int WAVES, bool BYCOL = false>
__device__ __forceinline__ void merge_final_body(const Model& m, const Buffers& b, int standalone,
                                                 double u_given, const double* CR,
                                                 const double* CRG, MergeSh& sh,
                                                 double* fac = nullptr) {
  __shared__ uint64_t ush[4];
  Ctrl* c = b.ctrl;
  const int t = threadIdx.x, w = WAVES == 1 ? 0 : wave_index();
  const int64_t nch = b.nch;
  const int per2 = WAVES == 1 ? 1 : (int)((nch + 255) / 256);
  const int64_t c0 = (int64_t)t * per2;
  // the control block's old values, loaded with the records (every thread is
  // past these loads at the barriers or reductions before the stores below)
  const int64_t k = (standalone ? 0 : c->k) + 1;
  const int cur = standalone ? 0 : c->cur;
  const double cum = c->cum, delta_ref = c->delta_ref;
  const int rolled = c->rolled_back;
  const int gl = min(max(t - 16, 0), kNGrad - 1);  // threads 16..24: a derivative each
  const double gcum = m.grad ? c->grad_cum[gl] : 0.0;
  double r1[kRec];  // per2 == 1: the thread's chunk record
  const bool one = per2 == 1;
  if (one) {
    const double* r = CR + min(c0, nch - 1) * kRec;
#pragma unroll
    for (int d = 0; d < kRec; ++d) r1[d] = r[d];
  }
  auto field = [&](int64_t cc, int d) { return one ? r1[d] : CR[cc * kRec + d]; };
  double mx2 = -INFINITY;
  for (int q = 0; q < per2; ++q) {
    const int64_t cc = c0 + q;
    if (cc < nch) mx2 = fmax(mx2, field(cc, 0));
  }
  const double M = group_reduce<WAVES>(mx2, sh.mx, w, OpMax());
  double tot7[7] = {};  // S, sum E^2, sum E x
  double G[kNGrad] = {};
  for (int q = 0; q < per2; ++q) {
    const int64_t cc = c0 + q;
    if (cc < nch) {
      const double mc = field(cc, 0);
      const double f = (mc == -INFINITY) ? 0.0 : exp(mc - M);
      const uint64_t Q = (uint64_t)__double_as_longlong(field(cc, 1));
      tot7[0] += (double)Q * f;
      if (BYCOL) {
        fac[t] = (mc == -INFINITY) ? -1.0 : f;  // (-1: no weight, whatever the derivatives)
        continue;
      }
      tot7[1] += field(cc, 2) * (f * f);
#pragma unroll
      for (int d = 0; d < 5; ++d) tot7[2 + d] += field(cc, 3 + d) * f;
      if (m.grad && mc != -INFINITY)
#pragma unroll
        for (int d = 0; d < kNGrad; ++d) G[d] += CRG[cc * kNGrad + d] * f;
    }
  }
  if (BYCOL) {
    double s1[1] = {tot7[0]};
    group_sum_n<1>(s1, nullptr, w);
    tot7[0] = s1[0];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
    static_assert(kOneMergeChunks == 4, "a chunk per row");
    const SumColumn col(CR, CRG, t & 15);
    const int cc = t >> 4;
    double acc = 0.0;
    if (cc < nch) {
      const double f = fac[cc], g = fmax(f, 0.0);
      const double y = col.p[cc * col.stride] * ((t & 15) == 0 ? g * g : g);
      acc = (col.grad && f < 0.0) ? 0.0 : y;
    }
    acc = sum_of_rows(acc);
#pragma unroll
    for (int d = 0; d < 6; ++d) tot7[1 + d] = readlane(acc, d);
#pragma unroll
    for (int d = 0; d < kNGrad; ++d) G[d] = readlane(acc, 6 + d);
  } else {
    group_sum_n<WAVES>(tot7, sh.sums, w);
    if (m.grad) group_sum_n<WAVES, kNGrad>(G, sh.grads, w);
  }
  const double S = tot7[0] * (1.0 / kItemScale), S2 = tot7[1];

  // every thread takes the step's scalars
  bool ok = isfinite(M) && isfinite(S) && S > 0.0 && isfinite(S2);
#pragma unroll
  for (int d = 0; d < 5; ++d) ok = ok && isfinite(tot7[2 + d]);
#pragma unroll
  for (int d = 0; d < kNGrad; ++d) ok = ok && isfinite(G[d]);
  const double logS = log(S);
  const double delta = ok ? M + logS : 0.0;
  const double ess = S * S / S2;
  const bool res = standalone ? ok : ok && ess < m.thr;
  if (standalone) {
    if (t == 0) {
      c->cur = 0;
      c->delta = delta;
      c->u = u_given;
      c->do_resample = ok ? 1 : 0;
      c->k = 0;
      c->heavy_count = 0;
    }
  } else if (ok) {
    if (t < 64) {
      // threads 1..5 a mean, threads 16..24 a derivative: one division
      double e = tot7[2];
#pragma unroll
      for (int d = 1; d < 5; ++d) e = t == 1 + d ? tot7[2 + d] : e;
      if (m.grad)
#pragma unroll
        for (int d = 0; d < kNGrad; ++d) e = t == 16 + d ? G[d] : e;
      e /= S;
      if (t >= 1 && t < 6) c->mean[t - 1] = e;
      if (m.grad && t >= 16 && t < 16 + kNGrad) {
        c->grad_last[t - 16] = e;
        c->grad_cum[t - 16] = gcum + e;
      }
      const uint4 rr = draw(m, 0u, (uint32_t)k, kResample, 0u);
      if (t == 0) {
        c->k = k;
        c->cur = cur ^ 1;
        c->m = M;
        c->log_sum = logS;
        c->ess = ess;
        c->delta = delta;
        c->cum = cum + delta;
        c->resampled = res ? 1 : 0;
        c->do_resample = res ? 1 : 0;
        c->mode = res ? (m.arna ? kModeArna : (m.group > 0 ? kModeRna : kModeSys)) : kModeNone;
        c->heavy_count = 0;
        c->u = u53(rr.x, rr.y);
        if (m.arna) {
          // the object is lost when this increment falls well below that of
          // the last frame that tracked it; each loss keys a new ring order
          const bool lost = delta < delta_ref - m.arna_drop;
          if (lost)
            c->ring_key = k;
          else
            c->delta_ref = delta;
          c->lost = lost ? 1 : 0;
          c->arna_tracking = 0;  // counted by k_arna_local
          c->arna_moved = 0;     // set by k_arna_exchange
        }
      }
    }
  } else if (t == 0) {
    c->rolled_back = rolled + 1;
    c->do_resample = 0;
    c->heavy_count = 0;
  }
  if (!res || (!standalone && m.group > 0)) return;  // uniform
  // chunk prefixes of the fixed-point CDF (2^62 = total weight)
  auto weight = [&](int64_t cc, double* phi) {
    const double mc = field(cc, 0);
    *phi = (mc == -INFINITY) ? 0.0 : exp(mc - delta) * kItemToCdf;
    return (uint64_t)rint((double)(uint64_t)__double_as_longlong(field(cc, 1)) * *phi);
  };
  uint64_t wsum = 0, wq = 0;
  double phi = 0.0;
  for (int q = 0; q < per2; ++q)
    if (c0 + q < nch) wsum += (wq = weight(c0 + q, &phi));
  uint64_t tot;
  uint64_t pre = group_excl_sum<WAVES>(wsum, ush, w, &tot);
  for (int q = 0; q < per2; ++q) {
    const int64_t cc = c0 + q;
    if (cc < nch) {
      if (!one) wq = weight(cc, &phi);
      b.cpre[cc].P = pre;
      b.cpre[cc].phi = phi;
      pre += wq;
    }
  }
  if (t == 0) c->total = tot;
}

__device__ __forceinline__ void merge_chunk(const Model& m, const Buffers& b, int standalone,
                                            int64_t ch) {
  __shared__ MergeSh sh;
  double* cr = b.CR + ch * kRec;
  double* crg = b.CRG + ch * kNGrad;
  const int t = threadIdx.x, w = wave_index();
  if (b.chunk == 256)
    merge_chunk_body<true>(m, b, standalone, ch, t, w, sh, cr, crg);
  else
    merge_chunk_body<false>(m, b, standalone, ch, t, w, sh, cr, crg);
}

template <int WAVES>
__device__ __forceinline__ void merge_final(const Model& m, const Buffers& b, int standalone,
                                            double u_given) {
  __shared__ MergeSh sh;
  merge_final_body<WAVES>(m, b, standalone, u_given, b.CR, b.CRG, sh);
}

__global__ __launch_bounds__(256) void k_merge(Model m, Buffers b, int standalone) {
  merge_chunk(m, b, standalone, blockIdx.x);
}

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_merge_final(Model m, Buffers b, int standalone,
                                                            double u_given) {
  merge_final<WAVES>(m, b, standalone, u_given);
}

// Both, for at most kOneMergeChunks chunks of 256 records: 256 threads to a
// chunk, then the first wave (the others would only take issue slots from it).
// GRAD: the filter has derivatives.
template <bool GRAD>
__device__ __forceinline__ void merge_one(const Model& m, const Buffers& b, int standalone,
                                          double u_given) {
  __shared__ MergeSh sh[kOneMergeChunks];
  __shared__ double cr[kOneMergeChunks * kRec], crg[kOneMergeChunks * kNGrad];
  const int sub = wave_index() >> 2, t = threadIdx.x & 255, w = wave_index() & 3;
  if constexpr (GRAD) {
    __shared__ double fac[256 * kOneMergeChunks], part[64 * kOneMergeChunks];
    merge_chunk_deriv(m, b, sub, t, w, sh[sub], fac + 256 * sub, part + 64 * sub,
                      cr + sub * kRec, crg + sub * kNGrad);
    __syncthreads();
    if (wave_index() != 0) return;
    merge_final_body<1, true>(m, b, standalone, u_given, cr, crg, sh[0], fac);
  } else {
    merge_chunk_body<true>(m, b, standalone, sub, t, w, sh[sub], cr + sub * kRec,
                           crg + sub * kNGrad);
    __syncthreads();
    if (wave_index() != 0) return;
    merge_final_body<1>(m, b, standalone, u_given, cr, crg, sh[0]);
  }
}
template <bool GRAD>
__global__ __launch_bounds__(256 * kOneMergeChunks) void k_merge_one(Model m, Buffers b,
                                                                     int standalone,
                                                                     double u_given) {
  merge_one<GRAD>(m, b, standalone, u_given);
}

// --------------------------------------------------- systematic resampling
// Slot s of N takes the particle j whose CDF interval [C_{j-1}, C_j) holds
// (s + u) / N (Algorithm 1's resampling step with one uniform u), so
// particle j owns the slots [bound(C_{j-1}), bound(C_j)) with bound(C) the
// number of slots below C. Block starts of the CDF are exact 2^62 fixed-point
// integers (so the partition of the slots over segments does not depend on
// summation order); inside a segment the CDF is a running maximum in fp64,
// so particles of zero weight own no slots, and the segment's last particle
// of positive weight takes the segment's remaining slots.

// The CDF at a block start from its block prefix and its chunk's record.
__device__ __forceinline__ double block_cdf(const ChunkPre& cp, uint64_t pfx) {
  return (double)(cp.P + (uint64_t)rint((double)pfx * cp.phi)) * (1.0 / kCdfScale);
}

// Number of slots s in [0, n) with (s + u) / n < C: ceil(C n - u), clamped.
// Monotone in C (the fma rounds once), so bounds taken at non-decreasing CDF
// values never overlap.
__device__ __forceinline__ int slot_bound(double C, double u, double nd, int n) {
  const double x = ceil(fma(C, nd, -u));
  return x <= 0.0 ? 0 : (x >= nd ? n : (int)x);
}

// Systematic resampling runs one wavefront per segment of kSegItems
// particles (kPerThread consecutive per lane, so the 256 particles of a
// block are one row of 16 lanes): every scan and maximum of the segment is
// a DPP operation within the wave and no barrier waits for other waves, so
// each wave streams its weights and ancestors at its own pace. Four blocks
// per wave spread the wave's fixed work (block records, the factor's exp,
// the scans) over 1024 particles.
constexpr int kWave = 64;
constexpr int kPerThread = kSegItems / kWave;  // particles, and slots of a tile, per lane
static_assert(kPerThread == 16 && kSlotTile == kSegItems && kSegBlocks == 4 &&
                  kBlock == 16 * kPerThread,
              "a segment is four blocks of one row each, sixteen particles and slots per lane");
// A tile's slot e lives at word slot_word(e) of the LDS tile, four spare
// words after every sixteen, so that each lane reads its slots with four
// 128-bit loads 80 bytes from its neighbour's (sixteen lanes then cover the
// 64 banks once); the lane-contiguous accesses (slots 4 lane + q of a
// block) meet at most two lanes on a bank.
constexpr int kTileWords = kSlotTile / kPerThread * (kPerThread + 4);
__device__ __forceinline__ int slot_word(int e) { return e + ((e >> 4) << 2); }

// Inclusive maximum scan over the wave of values >= 0 (each DPP step folds
// into one v_max_i32: row shifts, whose lanes outside the row read 0, then
// the row broadcasts into rows 1, 3 and into rows 2, 3). exclusive_of()
// shifts an inclusive scan one lane up (lane 0 reads 0).
__device__ __forceinline__ int wave_max_scan(int v) {
  v = max(v, (int)dpp32<0x111>((uint32_t)v));
  v = max(v, (int)dpp32<0x112>((uint32_t)v));
  v = max(v, (int)dpp32<0x114>((uint32_t)v));
  v = max(v, (int)dpp32<0x118>((uint32_t)v));
  v = max(v, bcast<0x142, 0xa>(v, 0));
  return max(v, bcast<0x143, 0xc>(v, 0));
}
__device__ __forceinline__ int exclusive_of(int inclusive) {
  return (int)dpp32<0x138>((uint32_t)inclusive);  // wave_shr:1
}

// Inclusive sum of exact integers held in doubles over the lanes of one
// block, one row of 16 lanes. Lanes whose source is outside the row read 0,
// the identity.
__device__ __forceinline__ double block_scan_add(double v) {
  v += shr<1>(v);
  v += shr<2>(v);
  v += shr<4>(v);
  v += shr<8>(v);
  return v;
}

// The resampling of one segment by one wave: the segment's slot range from
// its block starts, the particles' CDF from their fixed-point weights, every
// particle's run of slots, and the slots' particles, written tile by tile.
// Slot bounds are monotone in the CDF, so the running maximum that keeps
// runs from overlapping is taken over the integer bounds. LOG: the weights
// are caller log weights (standalone resampling), else the filter's stored
// E.
//
// k_anc runs each segment whose slots span at most kCoopTiles tiles; a
// heavier segment (concentrated weights) queues its tiles in chunks of
// kChunkTiles for k_fill, whose waves each recompute the segment's runs and
// write one chunk, so that heavy segments spread over many waves. (k_anc_all
// has helper waves in the same launch find the heavy segments themselves.)
// HEAVY: what a heavy segment's own wave does, queue it or leave it to them.
// queued: called for the tiles [tile_lo, tile_hi) of a heavy segment.
// One segment's loads, raw: its lanes' weights and its block records. Every
// lane loads (indices clamped into the arrays, values masked at use), so no
// load sits in a divergent branch that would consume it at once.
// The weights arrive lane-contiguous: x[4 h + q] is particle h kBlock +
// 4 lane + q of the segment (each load instruction reads one contiguous
// kWave x 16 bytes); anc_segment hands each lane its own kPerThread
// consecutive particles through the LDS tile.
typedef int V4i __attribute__((ext_vector_type(4)));  // for the nontemporal stores

struct SegIn {
  float x[kPerThread];
  uint64_t pfx;      // the block prefix of the lane's block b0 + lane / 16 (clamped)
  ChunkPre cp;       // its chunk's prefix and factor
  double mbt;        // its record maximum
  uint64_t pfx_end;  // the block prefix of block b0 + nbs, the first after the segment (clamped)
  ChunkPre cp_end;   // its chunk's
};

__device__ __forceinline__ SegIn load_seg(const Model& m, const Buffers& b, const float* E,
                                          const double* rec, bool log_src, int64_t seg) {
  SegIn in;
  const int lane = threadIdx.x;
  const int64_t b0 = seg * kSegBlocks;
  const int nbs = (int)min((int64_t)kSegBlocks, b.nb - b0);
  const int64_t bl = min(b0 + (lane >> 4), b.nb - 1);
  const int64_t be = min(b0 + nbs, b.nb - 1);
  // chunk = 256 per with per <= 8 and blk < 2^23: 32-bit quotients
  const uint32_t cb = (uint32_t)(b.chunk >> 8);
  in.cp = b.cpre[(uint32_t)(bl >> 8) / cb];
  in.pfx = b.pfx[bl];
  in.mbt = rec[bl * kRec];
  in.cp_end = b.cpre[(uint32_t)(be >> 8) / cb];
  in.pfx_end = b.pfx[be];
  const int64_t ib0 = b0 * kBlock;
  const int64_t ib1 = min(m.n, (b0 + nbs) * kBlock);
  if (ib1 - ib0 == kSegItems && (reinterpret_cast<uintptr_t>(E) & 15) == 0) {
    // a whole segment (uniform)
    const float4* v = reinterpret_cast<const float4*>(E + ib0);
#pragma unroll
    for (int h = 0; h < kSegBlocks; ++h) {
      const float4 f = v[h * (kBlock / 4) + lane];
      in.x[4 * h] = f.x;
      in.x[4 * h + 1] = f.y;
      in.x[4 * h + 2] = f.z;
      in.x[4 * h + 3] = f.w;
    }
  } else {
    // the ragged end: weight 0 past the last particle
#pragma unroll
    for (int h = 0; h < kSegBlocks; ++h)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t j = ib0 + h * kBlock + 4 * lane + q;
        const float v = E[min(j, ib1 - 1)];
        in.x[4 * h + q] = (j < ib1) ? v : (log_src ? -INFINITY : 0.0f);
      }
  }
  return in;
}

// The control block's values a resampling pass reads.
struct ResIn {
  int do_res;
  double delta, u;
};

enum Heavy { kQueue, kLeave };

template <bool LOG, Heavy HEAVY = kQueue>
__device__ __forceinline__ void anc_segment(const Model& m, const Buffers& b, const ResIn& ci,
                                            int64_t seg, const SegIn& in, bool queued,
                                            int tile_lo, int tile_hi) {
  __shared__ __align__(16) int A[kTileWords];
  Ctrl* c = b.ctrl;
  const int lane = threadIdx.x;
  const int lb = lane >> 4;  // this lane's block within the segment
  const int64_t b0 = seg * kSegBlocks;
  const int nbs = (int)min((int64_t)kSegBlocks, b.nb - b0);
  const int64_t ib0 = b0 * kBlock;
  const int64_t j0 = ib0 + kPerThread * (int64_t)lane;
  const double delta = ci.delta, u = ci.u;
  // the CDF at this lane's block start and at the block after the segment
  // (blocks past the data read as its end), and the block's factor from
  // integer weights to the CDF
  const bool in_seg = lb < nbs;
  const double Pblk = in_seg ? block_cdf(in.cp, in.pfx) : 1.0;
  const double Pend = b0 + nbs < b.nb ? block_cdf(in.cp_end, in.pfx_end) : 1.0;
  const double f =
      (in_seg && in.mbt != -INFINITY) ? exp(in.mbt - delta) * (1.0 / kItemScale) : 0.0;
  const int n = (int)m.n;
  const double nd = (double)m.n;
  const int fs = seg == 0 ? 0 : slot_bound(readlane(Pblk, 0), u, nd, n);
  const int fe = seg + 1 >= b.nseg ? n : slot_bound(Pend, u, nd, n);
  if (fe <= fs) return;  // uniform: no slot falls in this segment
  const int T0 = fs & ~3;  // tiles start on 16 bytes of anc
  const int ntiles = (fe - T0 + kSlotTile - 1) / kSlotTile;
  if (!queued && ntiles > kCoopTiles) {
    if (HEAVY == kLeave) return;
    // a heavy segment: its tiles go to k_fill in chunks
    const int chunks = (ntiles + kChunkTiles - 1) / kChunkTiles;
    int base = 0;
    if (lane == 0) base = atomicAdd(&c->heavy_count, chunks);
    base = readlane(base, 0);
    for (int q = lane; q < chunks; q += kWave)
      if (base >= 0 && (int64_t)base + q < b.hq_cap)  // the queue's size rules out overflow
        b.hq[base + q] = TileRun{(int32_t)seg, q * kChunkTiles,
                                 min(ntiles, (q + 1) * kChunkTiles), 0};
    return;
  }

  // each lane's kPerThread consecutive particles from the lane-contiguous
  // loads, through the tile (the tile is free: every earlier call on this
  // workgroup ended with its slots cleared and a barrier); the words a lane
  // reads stay until it clears them before the first tile
  float4* const Af = reinterpret_cast<float4*>(A);
  float4* const minef = Af + (slot_word(kPerThread * lane) >> 2);
#pragma unroll
  for (int h = 0; h < kSegBlocks; ++h)
    Af[slot_word(h * kBlock + 4 * lane) >> 2] =
        make_float4(in.x[4 * h], in.x[4 * h + 1], in.x[4 * h + 2], in.x[4 * h + 3]);
  __syncthreads();
  // a particle's fixed-point weight
  auto weight = [&](float xq) {
    if (LOG)  // particles past the data hold -inf
      return item_weight(xq == -INFINITY ? 0.0 : exp((double)xq - in.mbt));
    return item_weight((double)xq);
  };
  double kl[kPerThread];
  double tsum = 0.0;
#pragma unroll
  for (int r = 0; r < kPerThread / 4; ++r) {
    const float4 v = minef[r];
    const float xr[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int c4 = 0; c4 < 4; ++c4) {
      tsum += weight(xr[c4]);
      kl[4 * r + c4] = tsum;
    }
  }
  // prefix of the block's integer weights before this lane's particles
  // (exact: integers < 2^53)
  const double texcl = block_scan_add(tsum) - tsum;
  // each particle's slot bound at its CDF value C = Pblk + K f, with K the
  // block's integer weights up to and including the particle (exact):
  // ceil(C n - u) = ceil(K (n f) + (Pblk n - u)), one fma, at most fe.
  // Rounding may move a bound by one where C n - u is within a few ulps of
  // an integer; the running maximum below keeps the runs disjoint and
  // ordered regardless. Bounds are non-decreasing in K and equal K give
  // equal bounds in every lane of the block, so a particle of zero weight
  // after a positive one repeats its predecessor's bound and gets an empty
  // run. A block's leading particles of zero weight (K = 0) get 0, below
  // every bound: the previous block's CDF is computed apart and may round
  // lower than this block's start.
  const double fn = f * nd;
  const double gb = fma(Pblk, nd, -u);
  const int p0 = (int)j0;  // particle indices are below n < 2^31
  int rb[kPerThread];
#pragma unroll
  for (int q = 0; q < kPerThread; ++q) {
    const double K = texcl + kl[q];
    // |C n - u| stays far inside the int range (C in [0, 1], n < 2^31)
    rb[q] = K > 0.0 ? min((int)ceil(fma(K, fn, gb)), fe) : 0;
  }
  // the largest bound before the lane (bounds are non-decreasing in a lane)
  const int h0 = max(fs, exclusive_of(wave_max_scan(rb[kPerThread - 1])));
  // The segment's last particle of positive weight ends its runs at fe
  // (those after it have zero weight and empty runs), so every slot has an
  // owner whatever the rounding of the last bounds. Slots after its run's
  // end already take its mark; only if its own run came out empty (its
  // bound rounded to its predecessor's, below fe) does it need a mark, at
  // the start of its extended run: xmb / xmp, uniform, from a replay of that
  // lane's runs (rare: that lane's last bound then fell short of fe).
  int xmb = -1, xmp = 0;
  {
    const uint64_t pos_lanes = __builtin_amdgcn_ballot_w64(tsum > 0.0);
    const int L = 63 - __builtin_clzll(pos_lanes | 1ull);
    if (pos_lanes != 0 && readlane(rb[kPerThread - 1], L) < fe) {
      const double tl = readlane(texcl, L), fnl = readlane(fn, L), gbl = readlane(gb, L);
      const double mL = LOG ? readlane(in.mbt, L) : 0.0;  // lane L's block maximum
      const float* xl = reinterpret_cast<const float*>(A) + slot_word(kPerThread * L);
      int pv = readlane(h0, L), lastq = -1, pstart = 0;
      bool empty = false;
      double kk = 0.0;
#pragma nounroll
      for (int q = 0; q < kPerThread; ++q) {
        const float xq = xl[q];
        const double wq = LOG ? item_weight(xq == -INFINITY ? 0.0 : exp((double)xq - mL))
                              : item_weight((double)xq);
        kk += wq;
        const double K = tl + kk;
        const int rbq = K > 0.0 ? min((int)ceil(fma(K, fnl, gbl)), fe) : 0;
        const int e = max(pv, rbq);
        if (wq > 0.0) {
          lastq = q;
          pstart = pv;
          empty = !(e > pv);
        }
        pv = e;
      }
      if (lastq >= 0 && empty && pstart < fe) {
        const int r = pstart - T0;
        xmb = 4 * r + (r & ~15);
        xmp = p0 - kPerThread * lane + kPerThread * L + lastq;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < kPerThread / 4; ++r) minef[r] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  // particle kPerThread lane + q owns [e_{q-1}, e_q), e_q = max(e_{q-1},
  // rb[q]), e_{-1} = h0. Each non-empty run marks its first slot with the
  // particle; a slot's particle is then the largest mark at or before it.
  // mb: the LDS byte offset of the mark in tile coordinates from T0 (tile j:
  // subtract j kTileWords 4), 4 slot_word(e) = 4 e + (e & ~15), or -1.
  int mb[kPerThread];
  int prev = h0;
#pragma unroll
  for (int q = 0; q < kPerThread; ++q) {
    const int e = max(prev, rb[q]);
    const int r = prev - T0;
    mb[q] = e > prev ? 4 * r + (r & ~15) : -1;
    prev = e;
  }
  static_assert(kPerThread == 16, "4 slot_word(e) = 4 e + (e & ~15) for four spare words per sixteen");
  int32_t* anc = m.rpa ? b.asys : b.anc;  // RPA routes the systematic result afterwards
  const bool vec = (reinterpret_cast<uintptr_t>(anc) & 15) == 0;
  const int jt0 = queued ? tile_lo : 0, jt1 = queued ? min(tile_hi, ntiles) : ntiles;
  // the tiles before this call's first: the largest mark among them
  int carry = 0;
  if (jt0 > 0) {
    const int lim = jt0 * kTileWords * 4;  // marks at earlier bytes precede the first tile
#pragma unroll
    for (int q = 0; q < kPerThread; ++q)
      if (mb[q] >= 0 && mb[q] < lim) carry = p0 + q;  // the largest such (mb increases with q)
    carry = readlane(wave_reduce_last(carry, OpMax(), 0), 63);
    if (xmb >= 0 && xmb < lim) carry = xmp;  // the segment's last particle of positive weight
  }
  uint4* A4 = reinterpret_cast<uint4*>(A);
  uint4* mine = A4 + (slot_word(kPerThread * lane) >> 2);
  char* const Ab = reinterpret_cast<char*>(A);
  for (int j = jt0; j < jt1; ++j) {
    const int c0 = T0 + j * kSlotTile, wbase = j * kTileWords * 4;
    __syncthreads();  // one wave: orders the LDS accesses of the lanes
#pragma unroll
    for (int q = 0; q < kPerThread; ++q) {
      const int eb = mb[q] - wbase;
      if ((unsigned)eb < (unsigned)(kTileWords * 4)) *reinterpret_cast<int*>(Ab + eb) = p0 + q;
    }
    if (lane == 0 && (unsigned)(xmb - wbase) < (unsigned)(kTileWords * 4))
      *reinterpret_cast<int*>(Ab + (xmb - wbase)) = xmp;
    __syncthreads();
    // this lane's slots, their running maximum (particles increase with
    // slots), then the maximum over the lanes before it; 0 (the cleared
    // tile, and DPP's fill) is below every mark that precedes a slot from fs
    // on.
    int v[kPerThread];
#pragma unroll
    for (int r = 0; r < kPerThread / 4; ++r) {
      const uint4 a = mine[r];
      v[4 * r] = (int)a.x;
      v[4 * r + 1] = (int)a.y;
      v[4 * r + 2] = (int)a.z;
      v[4 * r + 3] = (int)a.w;
    }
#pragma unroll
    for (int q = 1; q < kPerThread; ++q) v[q] = max(v[q], v[q - 1]);
    const int winc = wave_max_scan(v[kPerThread - 1]);
    const int before = max(carry, exclusive_of(winc));
    carry = max(carry, readlane(winc, 63));
    // the slots' particles back into the tile, then out lane-contiguous
    // (slots 4 lane + q of each block-sized quarter of the tile), streamed
    // past the caches; a lane clears the words it reads for the next tile
#pragma unroll
    for (int r = 0; r < kPerThread / 4; ++r)
      mine[r] = make_uint4((uint32_t)max(before, v[4 * r]), (uint32_t)max(before, v[4 * r + 1]),
                           (uint32_t)max(before, v[4 * r + 2]), (uint32_t)max(before, v[4 * r + 3]));
    __syncthreads();
#pragma unroll
    for (int h = 0; h < kSegBlocks; ++h) {
      uint4* src = A4 + (slot_word(h * kBlock + 4 * lane) >> 2);
      const uint4 a = *src;
      *src = make_uint4(0u, 0u, 0u, 0u);
      const int s0 = c0 + h * kBlock + 4 * lane;
      int32_t* out = anc + s0;
      if (vec && s0 >= fs && s0 + 4 <= fe) {
        __builtin_nontemporal_store(V4i{(int)a.x, (int)a.y, (int)a.z, (int)a.w},
                                    reinterpret_cast<V4i*>(out));
      } else {
        const int w4[4] = {(int)a.x, (int)a.y, (int)a.z, (int)a.w};
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (s0 + q >= fs && s0 + q < fe) out[q] = w4[q];
      }
    }
  }
}

__device__ __forceinline__ ResIn res_in(const Ctrl* c) {
  ResIn ci;
  ci.do_res = c->do_resample;
  ci.delta = c->delta;
  ci.u = c->u;
  return ci;
}

// One wave per segment.
template <bool LOG, Heavy HEAVY = kQueue>
__device__ __forceinline__ void anc_seg(const Model& m, const Buffers& b, const WeightSrc& ws,
                                        int64_t seg) {
  const Ctrl* c = b.ctrl;
  const ResIn ci = res_in(c);
  if (!ci.do_res || seg >= b.nseg) return;
  const bool second = ws.use_cur && c->cur;
  const SegIn in = load_seg(m, b, second ? ws.E1 : ws.E0, second ? ws.rec1 : ws.rec0, LOG, seg);
  anc_segment<LOG, HEAVY>(m, b, ci, seg, in, false, 0, 0);
}

// Helper wave `id` of `count`: finds the heavy segments from the segments' slot
// ranges (kHelpPerLane segments per lane, the bounds that anc_segment takes) and
// writes the chunks id, id + count, ... of their tiles.
template <bool LOG>
__device__ __forceinline__ void anc_help(const Model& m, const Buffers& b, const WeightSrc& ws,
                                         int id, int count) {
  const Ctrl* c = b.ctrl;
  const ResIn ci = res_in(c);
  if (!ci.do_res) return;
  const int lane = threadIdx.x, n = (int)m.n;
  const int nseg = (int)b.nseg, per = (nseg + kWave - 1) / kWave;
  const uint32_t cb = (uint32_t)(b.chunk >> 8);
  const double nd = (double)m.n;
  // the slots where the lane's segments, and the one after them, start
  int at[kHelpPerLane + 1];
#pragma unroll
  for (int q = 0; q <= kHelpPerLane; ++q) {
    at[q] = n;
    if (q <= per) {  // uniform
      const int seg = lane * per + q;
      const int64_t blk = (int64_t)min(seg, nseg - 1) * kSegBlocks;
      const double C = block_cdf(b.cpre[(uint32_t)(blk >> 8) / cb], b.pfx[blk]);
      at[q] = seg == 0 ? 0 : seg >= nseg ? n : slot_bound(C, ci.u, nd, n);
    }
  }
  int chunks[kHelpPerLane], tiles[kHelpPerLane];
  int mine = 0;
#pragma unroll
  for (int q = 0; q < kHelpPerLane; ++q) {
    tiles[q] = q < per && at[q + 1] > at[q]
                   ? (at[q + 1] - (at[q] & ~3) + kSlotTile - 1) / kSlotTile
                   : 0;
    chunks[q] = tiles[q] > kCoopTiles ? (tiles[q] + kChunkTiles - 1) / kChunkTiles : 0;
    mine += chunks[q];
  }
  const int incl = wave_scan(mine, lane, OpAdd());
  const int total = readlane(incl, 63);
  const bool second = ws.use_cur && c->cur;
  for (int j = id; j < total; j += count) {  // uniform
    const int owner = __popcll(__ballot(incl <= j));  // the first lane whose chunks reach past j
    int first = readlane(incl - mine, owner), seg = 0, lo = 0, hi = 0;
#pragma unroll
    for (int q = 0; q < kHelpPerLane; ++q) {
      const int k = readlane(chunks[q], owner);
      if (j >= first && j < first + k) {
        seg = owner * per + q;
        lo = (j - first) * kChunkTiles;
        hi = min(readlane(tiles[q], owner), lo + kChunkTiles);
      }
      first += k;
    }
    const SegIn in = load_seg(m, b, second ? ws.E1 : ws.E0, second ? ws.rec1 : ws.rec0, LOG, seg);
    anc_segment<LOG, kLeave>(m, b, ci, seg, in, true, lo, hi);
    __syncthreads();  // the next chunk clears the tile again
  }
}

// The whole pass in one launch, for up to kWave kHelpPerLane segments: a wave
// per segment, then helper waves for the heavy ones, which find them while the
// others work. With no heavy segment (most steps) that takes no longer than the
// segments themselves; k_fill's launch for an empty queue costs 2-4 us and a gap.
// Beyond, the helpers' look over all segments outlasts a launch: with 64 segments to
// a lane 1.2 M particles take 18.9 us, and 11.7 in two launches; 2^21 31.6 and 12.7.
// The chunks of the lightest heavy segment, which spans at least kCoopTiles kSlotTile - 2
// slots, times as many segments: the most chunks there can be.
static_assert(kHelpWaves >= (kCoopTiles + kChunkTiles) / kChunkTiles *
                                (kWave * kHelpPerLane * kSegItems / (kCoopTiles * kSlotTile - 2)),
              "a helper wave per chunk");
template <bool LOG>
__global__ __launch_bounds__(kWave) void k_anc_all(Model m, Buffers b, WeightSrc ws) {
  const int nseg = (int)b.nseg, j = (int)blockIdx.x;
  if (j < nseg)
    anc_seg<LOG, kLeave>(m, b, ws, j);
  else
    anc_help<LOG>(m, b, ws, j - nseg, (int)gridDim.x - nseg);
}

__global__ __launch_bounds__(kWave) void k_anc(Model m, Buffers b, WeightSrc ws) {
  anc_seg<false>(m, b, ws, blockIdx.x);
}

// The same on caller log weights (standalone resampling).
__global__ __launch_bounds__(kWave) void k_anc_log(Model m, Buffers b, WeightSrc ws) {
  anc_seg<true>(m, b, ws, blockIdx.x);
}

// The tile chunks of heavy segments queued by k_anc: each wave takes queue
// entries in turn.
// Queue entry q of one filter: its chunk of tiles, then a barrier (the next
// entry clears the tile again).
template <bool LOG>
__device__ __forceinline__ void fill_entry(const Model& m, const Buffers& b, const WeightSrc& ws,
                                           const ResIn& ci, int64_t q) {
  const TileRun r = b.hq[q];
  if (r.seg < 0 || (int64_t)r.seg >= b.nseg || r.tile_lo < 0 || r.tile_hi <= r.tile_lo)
    return;  // uniform across the wave
  const bool second = ws.use_cur && b.ctrl->cur;
  const SegIn in = load_seg(m, b, second ? ws.E1 : ws.E0, second ? ws.rec1 : ws.rec0, LOG, r.seg);
  anc_segment<LOG>(m, b, ci, r.seg, in, true, r.tile_lo, r.tile_hi);
  __syncthreads();
}

template <bool LOG>
__device__ __forceinline__ void fill_body(const Model& m, const Buffers& b, const WeightSrc& ws,
                                          int64_t q0, int64_t qstep) {
  const ResIn ci = res_in(b.ctrl);
  if (!ci.do_res) return;
  const int64_t nh = min((int64_t)b.ctrl->heavy_count, b.hq_cap);
  for (int64_t q = q0; q < nh; q += qstep) fill_entry<LOG>(m, b, ws, ci, q);
}

__global__ __launch_bounds__(kWave) void k_fill(Model m, Buffers b, WeightSrc ws) {
  fill_body<false>(m, b, ws, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(kWave) void k_fill_log(Model m, Buffers b, WeightSrc ws) {
  fill_body<true>(m, b, ws, blockIdx.x, gridDim.x);
}

// ------------------------------------------------------------------- RNA
// Orders the LDS accesses of one wave's lanes (they are served in order; this
// keeps the compiler from moving them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// A group's resampling (Section 3) by WAVES waves, four consecutive particles
// and slots per lane: one wave for groups up to kWaveGroup particles, so that no
// barrier waits, a block's factor is one exp for four particles and the scans
// are a quarter; four waves for larger groups. The kernel is bound by issue
// (divisions, exps, searches): 4096 groups of 256 took 13.2 us with one particle
// per lane and a search per slot, 300 groups of 1000 10.3 us with loads that
// waited for each other.
constexpr int kWaveGroup = 256;
template <int WAVES>
struct GroupLds {
  static constexpr int kTeams = 4 / WAVES;  // groups per workgroup
  __align__(16) uint64_t C[kTeams][256 * WAVES];  // a group's local CDF, 2^60 fixed point
  double dsum[4];
  uint64_t wsum[4];
};

// The share W of group gg's ng particles (E relative to its block maximum, or
// absolute fp32 log weights) and, by local systematic resampling with the
// uniform u, the particles a[0..3] (indices in the group) of this lane's slots 4
// tl + i: the first j with C_j > (l + u) / ng (the identity when the group has
// no weight). team: the group's place in the workgroup; tl: thread in the group.
template <int WAVES>
__device__ __forceinline__ double group_resample(const WeightSrc& ws, const float* E,
                                                 const double* rec, double lognorm, int64_t gg,
                                                 int ng, double inv_ng, double u,
                                                 GroupLds<WAVES>& L, int team, int tl,
                                                 int (&a)[4]) {
  const int lane = threadIdx.x & 63, w = wave_index();
  uint64_t* const C = L.C[team];
  const int64_t base = gg * ng, idx = base + 4 * tl;
  const int64_t last = base + ng - 1;
  const int here = max(0, min(4, ng - 4 * tl));  // this lane's particles
  float x[4];
  if (here == 4 && (reinterpret_cast<uintptr_t>(E + idx) & 15) == 0) {
    const float4 v = *reinterpret_cast<const float4*>(E + idx);
    x[0] = v.x;
    x[1] = v.y;
    x[2] = v.z;
    x[3] = v.w;
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = E[min(idx + j, last)];
  }
  double wl[4];
  if (ws.log_src) {
#pragma unroll
    for (int j = 0; j < 4; ++j) wl[j] = j < here ? exp((double)x[j] - lognorm) : 0.0;
  } else {
    // the four lie in one block of records, or in two
    const int64_t b0 = min(idx, last) / kBlock, b3 = min(idx + 3, last) / kBlock;
    const double m0 = rec[b0 * kRec], m3 = rec[b3 * kRec];
    const double f0 = exp(m0 - lognorm);
    double f3 = f0;
    if (__ballot(b0 != b3)) f3 = exp(m3 - lognorm);  // uniform
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool second = min(idx + j, last) / kBlock != b0;
      const double mb = second ? m3 : m0, f = second ? f3 : f0;
      wl[j] = j >= here || mb == -INFINITY ? 0.0 : (double)x[j] * f;
    }
  }
  double W = wave_reduce(((wl[0] + wl[1]) + wl[2]) + wl[3], lane, OpAdd());
  if (WAVES > 1) {
    if (lane == 0) L.dsum[w] = W;
    __syncthreads();
    W = (L.dsum[0] + L.dsum[1]) + (L.dsum[2] + L.dsum[3]);
  }
  uint64_t v[4], run = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    run += (W > 0.0) ? __double2ull_rn(wl[j] / W * 0x1p60) : 0ull;
    v[j] = run;
  }
  uint64_t before = wave_scan(run, lane, OpAdd()) - run;
  if (WAVES > 1) {
    if (lane == 63) L.wsum[w] = before + run;
    __syncthreads();
    for (int j = 0; j < w; ++j) before += L.wsum[j];
  }
  // (entries from ng on repeat the total; no search reads them)
#pragma unroll
  for (int j = 0; j < 4; ++j) C[4 * tl + j] = before + v[j];
  if (WAVES > 1)
    __syncthreads();
  else
    wave_sync();
  // the first slot by binary search, the others from their predecessor's: the
  // same particle, the next, or a search beyond
  int lo = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int l = 4 * tl + i;
    const uint64_t us = (uint64_t)(((double)min(l, ng - 1) + u) * inv_ng * 0x1p60);
    int hi = ng - 1;
    if (i > 0) {
      if (lo < hi && !(C[lo] > us)) ++lo;
      if (lo >= hi || C[lo] > us) hi = lo;
    }
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (C[mid] > us)
        hi = mid;
      else
        lo = mid + 1;
    }
    a[i] = W > 0.0 ? lo : l;
  }
  return W;
}

// RNA of one group: its local resampling, the last `moved` slots of which go to
// the same slots of group g+1 on the ring (so group g's come from g-1, and no
// workgroup needs another's result), and its slot weight W_g / n.
template <int WAVES>
__device__ __forceinline__ void rna_body(const Model& m, const Buffers& b, const WeightSrc& ws,
                                         const double* __restrict__ u_dev, int64_t block) {
  __shared__ GroupLds<WAVES> L;
  const Ctrl* c = b.ctrl;
  if (!c->do_resample) return;
  const int team = WAVES == 1 ? wave_index() : 0;
  const int64_t g = block * (4 / WAVES) + team;
  const int64_t G = m.G;
  if (g >= G) return;  // whole waves, of groups of one wave (no barriers)
  const int tl = (int)threadIdx.x - (WAVES == 1 ? 64 * team : 0);
  const bool second = ws.use_cur && c->cur;
  const int ng = m.group;
  double u;
  if (u_dev) {
    u = u_dev[g];
  } else {
    const uint4 rr = draw(m, (uint32_t)g, (uint32_t)c->k, kRna, 0u);
    u = u53(rr.x, rr.y);
  }
  int a[4];
  const double W = group_resample<WAVES>(ws, second ? ws.E1 : ws.E0, second ? ws.rec1 : ws.rec0,
                                         c->delta, g, ng, m.inv_group, u, L, team, tl, a);
  const int64_t mine = g * ng, next = (g + 1 == G ? 0 : g + 1) * (int64_t)ng;
  const int stay = ng - m.moved;  // slots from here on go to the next group
  const int l = 4 * tl;
  int32_t* out = b.anc + (l < stay ? mine : next) + l;
  if (l + 4 <= ng && (l + 4 <= stay || l >= stay) &&
      (reinterpret_cast<uintptr_t>(out) & 15) == 0) {
    const int p = (int)mine;
    *reinterpret_cast<int4*>(out) = make_int4(p + a[0], p + a[1], p + a[2], p + a[3]);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (l + i < ng) b.anc[(l + i < stay ? mine : next) + l + i] = (int32_t)(mine + a[i]);
  }
  if (tl == 0) b.lwg[g] = log(W / (double)ng);
}

template <int WAVES>
__global__ __launch_bounds__(256) void k_rna(Model m, Buffers b, WeightSrc ws,
                                             const double* __restrict__ u_dev) {
  rna_body<WAVES>(m, b, ws, u_dev, blockIdx.x);
}

// ------------------------------------------------------------------ ARNA
// Adaptive RNA (Section 6.4 names its rules; the reading): RNA's local
// resampling per group; G_t groups track (share W_g >= theta / G); mu =
// mu_min + floor((mu_max - mu_min) (G - G_t) / G) slots move per group, from
// its predecessor on a ring of the groups whose order is redrawn whenever the
// object is lost (k_merge_final keys it by the frame of the loss).

// One round value of the ring's Feistel network: the low `half` bits of word
// 0 of the Philox block with counter (R, key, RING << 24 | r, track).
__device__ __forceinline__ uint32_t ring_f(const Model& m, uint32_t key, uint32_t r, uint32_t R,
                                           uint32_t mask) {
  return draw(m, R, key, kRing, r).x & mask;
}

// Eight Feistel rounds (L, R) -> (R, L xor F_r(R)) on the two halves of x,
// and their inverse: a keyed permutation of [0, 2^(2 half)).
__device__ __forceinline__ uint32_t ring_fwd(const Model& m, uint32_t key, int half, uint32_t x) {
  const uint32_t mask = (1u << half) - 1u;
  uint32_t L = x >> half, R = x & mask;
  for (uint32_t r = 0; r < 8; ++r) {
    const uint32_t nl = R;
    R = L ^ ring_f(m, key, r, R, mask);
    L = nl;
  }
  return (L << half) | R;
}
__device__ __forceinline__ uint32_t ring_back(const Model& m, uint32_t key, int half, uint32_t x) {
  const uint32_t mask = (1u << half) - 1u;
  uint32_t L = x >> half, R = x & mask;
  for (int r = 7; r >= 0; --r) {
    const uint32_t pl = R ^ ring_f(m, key, (uint32_t)r, L, mask);
    R = L;
    L = pl;
  }
  return (L << half) | R;
}

// The ring predecessor of group g among G groups under ring key `key`: the
// ring order is the permutation of [0, 2^b) (b the smallest even width with
// 2^b >= G) restricted to [0, G) by cycle walking; g's ring position comes
// from walking the inverse, its predecessor's group from walking forward.
// Key 0: the index ring (g - 1 mod G).
__device__ int64_t ring_pred(const Model& m, uint32_t key, int64_t G, int64_t g) {
  if (key == 0 || G < 2) return (g + G - 1) % G;
  int b = 2;
  while (((int64_t)1 << b) < G) b += 2;
  const int half = b / 2;
  uint32_t x = (uint32_t)g;
  do {
    x = ring_back(m, key, half, x);
  } while ((int64_t)x >= G);
  uint32_t y = (uint32_t)(((int64_t)x + G - 1) % G);
  do {
    y = ring_fwd(m, key, half, y);
  } while ((int64_t)y >= G);
  return (int64_t)y;
}

// W_g, the local systematic resampling (global indices into aloc), and the
// tracking count.
template <int WAVES>
__device__ __forceinline__ void arna_local_body(const Model& m, const Buffers& b, int64_t block) {
  __shared__ GroupLds<WAVES> L;
  Ctrl* c = b.ctrl;
  if (!c->do_resample) return;
  const int team = WAVES == 1 ? wave_index() : 0;
  const int64_t g = block * (4 / WAVES) + team;
  if (g >= m.G) return;
  const int tl = (int)threadIdx.x - (WAVES == 1 ? 64 * team : 0);
  const int cur = c->cur;
  const WeightSrc ws{b.E0, b.E1, b.R0, b.R1, 1, 0};
  const int ng = m.group;
  const uint4 rr = draw(m, (uint32_t)g, (uint32_t)c->k, kRna, 0u);
  int a[4];
  const double W = group_resample<WAVES>(ws, cur ? b.E1 : b.E0, cur ? b.R1 : b.R0, c->delta, g, ng,
                                         m.inv_group, u53(rr.x, rr.y), L, team, tl, a);
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (4 * tl + i < ng) b.aloc[g * ng + 4 * tl + i] = (int32_t)(g * ng + a[i]);
  if (tl == 0) {
    b.Wg[g] = W;
    if (W >= m.arna_share) atomicAdd(&c->arna_tracking, 1);
  }
}

// One workgroup per group: the exchange along the ring and the slot weights.
__device__ __forceinline__ void arna_exchange_body(const Model& m, const Buffers& b, int64_t g) {
  __shared__ int64_t sh_pred;
  Ctrl* c = b.ctrl;
  if (!c->do_resample) return;
  const int64_t G = m.G;
  const int ng = m.group;
  const int64_t mu =
      m.arna_mu_min + ((int64_t)(m.moved - m.arna_mu_min) * (G - c->arna_tracking)) / G;
  if (threadIdx.x == 0) sh_pred = ring_pred(m, (uint32_t)c->ring_key, G, g);
  __syncthreads();
  const int64_t pred = sh_pred;
  for (int l = threadIdx.x; l < ng; l += 256) {
    const int64_t src = (l >= ng - mu) ? pred : g;
    b.anc[g * ng + l] = b.aloc[src * ng + l];
  }
  if (threadIdx.x == 0) {
    b.lwg[g] = log(b.Wg[g] / (double)ng);
    b.lwt[g] = log(b.Wg[pred] / (double)ng);
    if (g == 0) c->arna_moved = (int32_t)mu;
  }
}

template <int WAVES>
__global__ __launch_bounds__(256) void k_arna_local(Model m, Buffers b) {
  arna_local_body<WAVES>(m, b, blockIdx.x);
}

__global__ __launch_bounds__(256) void k_arna_exchange(Model m, Buffers b) {
  arna_exchange_body(m, b, blockIdx.x);
}

// ------------------------------------------------------------------- RPA
// Resampling with proportional allocation (Section 3) over groups of n
// particles: group g's offspring are its share of the global systematic
// resampling (the slots whose ancestor lies in the group; the systematic
// ancestors are non-decreasing, so they form one range, found by binary
// search); a group keeps its first min(N_g, n) offspring, and the DLB
// schedule of Section 4 routes the surplus of the senders (N_g > n) into the
// free slots of the receivers (N_g < n). Greedy matching is the overlap of
// the senders' surplus intervals and the receivers' deficit intervals laid
// end to end in schedule order (group order for GS, by size descending for
// SGS): a routed particle is named by its place in that stream.

// First index of the non-decreasing a[0..n) with a[i] >= v.
__device__ __forceinline__ int64_t lower_bound_i32(const int32_t* a, int64_t n, int64_t v) {
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)a[mid] < v) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ int64_t rpa_count(const Buffers& b, int64_t g) {
  return b.rfirst[g + 1] - b.rfirst[g];
}

// The groups' offspring ranges, by a look at every slot: where the ancestors'
// group changes, the groups after the last slot's up to this one start here. One
// pass over 4 N bytes; a search per group is a chain of log2 N loads, 10 us for
// 4096 groups of 2^20 particles against 4.7 us, and the better one once N
// outgrows the caches (38 M: 19 us, against 30 us for the bytes alone).
__global__ __launch_bounds__(256) void k_rpa_bounds(Model m, Buffers b) {
  const Ctrl* c = b.ctrl;
  if (!c->do_resample) return;
  const int64_t N = m.n;
  const int64_t t0 = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x);
  const uint32_t n = (uint32_t)m.rpa_group;
  const int lane = threadIdx.x & 63;
  int prev = t0 > 0 ? (int)((uint32_t)b.asys[min(t0, N) - 1] / n) : -1;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    // past the last slot: a boundary to "group G", once
    const int64_t t = min(t0 + i, N);
    const int g = t < N ? (int)((uint32_t)b.asys[t] / n) : m.rpa_G;
    if (g > prev && t0 + i <= N) b.rfirst[g] = t;
    // the empty groups between are written by the whole wave
    uint64_t gaps = __ballot(g > prev + 1 && t0 + i <= N);
    while (gaps) {  // uniform
      const int l = __builtin_ctzll(gaps);
      gaps &= gaps - 1;
      const int g0 = readlane(prev, l) + 1, g1 = readlane(g, l);
      const int64_t first = (int64_t)readlane((uint64_t)t, l);
      for (int x = g0 + lane; x < g1; x += 64) b.rfirst[x] = first;
    }
    prev = g;
  }
}

// The same by one binary search per group boundary.
__global__ __launch_bounds__(256) void k_rpa_first(Model m, Buffers b) {
  const Ctrl* c = b.ctrl;
  if (!c->do_resample) return;
  const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t N = m.n, G = m.rpa_G;
  if (g <= G) b.rfirst[g] = g == G ? N : lower_bound_i32(b.asys, N, g * (int64_t)m.rpa_group);
}

// The whole plan for up to kRankGroups groups: group g's base in the stream is
// the sum of the values before it in its side's order, taken over all groups by
// 16 lanes (the values in LDS). G^2 compares: 10.6 us for 4096 groups, where the
// radix sort and the scans of the lists were 16 launches and 80 us. Sorted greedy, a
// step of 2^20 particles: 66 us with 4096 groups, 77 with 8192, and 121 with 8256 by
// sorting. The greedy lists need no sort, only the scans' three launches (a step with
// groups of 256, by counting and by scans: 2048 groups 50 and 56 us, 4096 64 and 66, 4608
// 71 and 67, 8192 98 and 85; with groups of 4 40 and 46, 43 and 46, 45 and 46, 53 and 47).
template <bool SORTED>
__global__ __launch_bounds__(256) void k_rpa_rank(Model m, Buffers b) {
  const Ctrl* c = b.ctrl;
  if (!c->do_resample) return;
  // the groups' first slots (below 2^31), then their offspring less their
  // slots, 0 past the groups
  __shared__ __align__(16) int v[kRankGroups + 4];
  const int G = m.rpa_G, n = m.rpa_group, t = threadIdx.x, r = t & 15;
  const int* first = reinterpret_cast<const int*>(b.rfirst);  // their low words
  for (int j0 = t; j0 <= G; j0 += 2048) {  // eight loads at a time
    int x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = first[2 * min(j0 + 256 * u, G)];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (j0 + 256 * u <= G) v[j0 + 256 * u] = x[u];
  }
  __syncthreads();
  // the differences, 1024 groups at a time from below (each round reads what
  // later rounds have not written yet), zeros up to a multiple of 64 groups
  const int G64 = (G + 63) & ~63;
  for (int j0 = 0; j0 < G64; j0 += 1024) {
    const int j = j0 + 4 * t;
    int f[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) f[i] = v[min(j + i, G)];
    __syncthreads();
    if (j < G64) {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[j + i] = j + i < G ? f[i + 1] - f[i] - n : 0;
    }
    __syncthreads();
  }
  const int g = min((int)blockIdx.x * 16 + (t >> 4), G - 1);
  const int vg = v[g], neg = vg > 0 ? 0 : -1;
  const int wg = (vg ^ neg) - neg;  // the group's surplus or deficit
  // GS: before g when the group is; SGS: when its value is larger, or equal and
  // the group is. (Values of the other side, and past the groups, are not
  // positive here.)
  int pre = 0;
#pragma unroll 4
  for (int j = 4 * r; j < G; j += 64) {
    const int4 q = *reinterpret_cast<const int4*>(v + j);
    const int w4[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int w = (w4[i] ^ neg) - neg, lower = j + i < g ? 1 : 0;
      if (SORTED)
        pre += w & -(int)(w + lower > wg);
      else
        pre += max(w, 0) & -lower;
    }
  }
  pre = row_allreduce(pre, OpAdd());
  if (r == 0 && (int)blockIdx.x * 16 + (t >> 4) < G && wg > 0) {
    if (vg > 0)
      b.rscum[g] = pre;
    else
      b.rdbase[g] = pre;
  }
}

// Surplus (side 0) or deficit (side 1) of group g; 0 when it is not a
// sender (receiver).
__device__ __forceinline__ uint64_t rpa_value(const Buffers& b, int64_t n, int64_t g, int side) {
  const int64_t cg = rpa_count(b, g);
  const int64_t v = side == 0 ? cg - n : n - cg;
  return v > 0 ? (uint64_t)v : 0;
}

// ------------------------------------------------------------ radix sort
// Stable least-significant-digit sort of (uint32 key, int32 value) pairs,
// eight bits per pass, in tiles of T * R pairs (T threads, R rounds; wave w
// holds the pairs [64 R w, 64 R (w + 1)) of its tile, 64 per round). A pass:
// the digit's count per tile (k_radix_hist), each digit's row of tile counts
// turned into exclusive prefixes (k_radix_rowscan, one workgroup per digit),
// then k_radix_scatter: every pair's rank among its tile's pairs of the same
// digit in input order, the pairs put in that order in LDS, and written from
// there to digit start + tile prefix + rank, so that a digit's pairs of a tile
// leave as one run. `gate`, when given, skips the pass on steps that do not
// resample.
//
// The scatter is bound by its writes: a tile's run of one digit is T R / 256
// pairs long on average. Over 38 M pairs (608 MB a pass) it takes 156 us in
// tiles of 4096, 192 us in tiles of 2048 and 243-261 us in tiles of 8192 (LDS
// for one workgroup per CU); written straight from tiles of 1024, 16 bytes to a
// run, it took 911 us. Three forms, by the number of pairs (radix_sort):
// - up to kSortFold, tiles of 4096 by 1024 threads whose counts the scatter adds up
//   itself: two launches a pass. A schedule waits for its launches: 32 list entries
//   76 us, and 102 in the next form; 304,000 114 and 118; 2^19 119 and 125. (Where the
//   stream is full anyway the next form's kernels are the shorter ones, in RPA's step
//   76 us against 73 with 32,768 entries and 86 against 77 with 262,144.) The rows to
//   add up grow with the square of the tiles: 1.6 M entries 257 us, and 207.
// - up to kSortLarge, tiles of 1024 by 256 threads, so that enough workgroups run, and
//   a launch of its own for the rows: 2^20 entries 139 us, and 154 in the next form.
// - from there on tiles of 4096 by 256 threads and the same three launches: the
//   Z-ordered initialisation of 2^22 particles 156 us, and 184 in tiles of 1024, of 2^23
//   254 and 320 (of 2^21 the two are equal, 119 and 121).

// The tile of a workgroup: consecutive tiles, whose runs of a digit are
// neighbours in the output, go to workgroups of one XCD (workgroups are dealt
// to the eight in turn), so that a cache line two tiles share is completed in
// that XCD's L2.
__device__ __forceinline__ int xcd_tile(int ntiles) {
  const int x = blockIdx.x & 7, q = ntiles >> 3, r = ntiles & 7;
  return x * q + min(x, r) + (int)(blockIdx.x >> 3);
}

// The lanes of this wave whose pair (in) has the digit d.
__device__ __forceinline__ uint64_t digit_peers(uint32_t d, bool in) {
  uint64_t peers = __ballot(in);
#pragma unroll
  for (int bit = 0; bit < 8; ++bit) {
    const bool set = (d >> bit) & 1u;
    const uint64_t bb = __ballot(set);
    peers &= set ? bb : ~bb;
  }
  return peers;
}

// Adds the digit of every lane's pair to the counts h. A wave whose pairs all
// hold one digit (the high digits of small values) adds once: 64 atomics on
// one address would go one after another.
__device__ __forceinline__ void count_digit(uint32_t* h, uint32_t d, bool in) {
  const uint64_t all = __ballot(in);
  if (!all) return;  // uniform
  const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, __builtin_ctzll(all));
  if (__ballot(in && d == d0) == all) {
    if ((threadIdx.x & 63) == 0) atomicAdd(&h[d0], (uint32_t)__popcll(all));
  } else if (in) {
    atomicAdd(&h[d], 1u);
  }
}

// FOLD: few tiles; their counts stay a row per tile and every workgroup of the
// scatter adds up the rows itself, instead of a launch of its own for it.
template <int T, int R, bool FOLD>
__global__ __launch_bounds__(T) void k_radix_hist(const uint32_t* __restrict__ key, int64_t count,
                                                  int shift, uint32_t* __restrict__ hist,
                                                  int32_t ntiles, const Ctrl* gate) {
  if (gate && !gate->do_resample) return;
  __shared__ uint32_t h[256];
  const int t = threadIdx.x;
  if (t < 256) h[t] = 0;
  const int tile = xcd_tile(ntiles);
  const int64_t base = (int64_t)tile * (T * R);
  uint32_t k[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t j = base + r * T + t;
    k[r] = key[min(j, count - 1)];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) count_digit(h, (k[r] >> shift) & 255u, base + r * T + t < count);
  __syncthreads();
  if (t < 256) hist[FOLD ? (int64_t)tile * 256 + t : (int64_t)t * ntiles + tile] = h[t];
}

__global__ __launch_bounds__(256) void k_radix_rowscan(uint32_t* __restrict__ hist, int32_t ntiles,
                                                       uint32_t* __restrict__ rowtot,
                                                       const Ctrl* gate) {
  if (gate && !gate->do_resample) return;
  __shared__ uint64_t sh[4];
  uint32_t* row = hist + (int64_t)blockIdx.x * ntiles;
  uint64_t carry = 0;
  for (int32_t i0 = 0; i0 < ntiles; i0 += 1024) {
    const int32_t i = i0 + 4 * (int32_t)threadIdx.x;
    uint32_t v[4];
    uint64_t s = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[q] = i + q < ntiles ? row[i + q] : 0;
      s += v[q];
    }
    uint64_t tot;
    uint64_t ex = carry + block_excl_sum(s, sh, &tot);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (i + q < ntiles) row[i + q] = (uint32_t)ex;
      ex += v[q];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) rowtot[blockIdx.x] = (uint32_t)carry;
}

// vin null: the values are the pairs' positions. kout null: the keys are not
// needed any more.
template <int T, int R, bool FOLD>
__global__ __launch_bounds__(T) void k_radix_scatter(
    const uint32_t* __restrict__ kin, const int32_t* __restrict__ vin, uint32_t* __restrict__ kout,
    int32_t* __restrict__ vout, int64_t count, int shift, const uint32_t* __restrict__ hist,
    const uint32_t* __restrict__ rowtot, int32_t ntiles, const Ctrl* gate) {
  static_assert(T % 256 == 0, "the first 256 threads take a digit each");
  if (gate && !gate->do_resample) return;
  constexpr int kWaves = T / 64, kTile = T * R;
  __shared__ uint32_t skey[kTile];
  __shared__ int32_t sval[kTile];
  __shared__ volatile uint32_t wcnt[kWaves][256];  // pairs per wave and digit, then their prefix
  __shared__ uint32_t lstart[256];  // each digit's first position in the tile's order
  __shared__ uint32_t gbase[256];   // its first output position, less lstart
  __shared__ uint32_t sh[2][4];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int tile = xcd_tile(ntiles);
  const int64_t tb = (int64_t)tile * kTile;
  const int cnt = (int)min((int64_t)kTile, count - tb);
  const int l0 = 64 * R * w + lane;
  uint32_t key[R];
  int32_t val[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t j = tb + min(l0 + 64 * r, cnt - 1);
    key[r] = kin[j];
    val[r] = vin ? vin[j] : (int32_t)j;
  }
  // the digit's pairs in all tiles, and in the tiles before this one
  uint32_t dtot = 0, before = 0;
  constexpr int kParts = T / 256;  // FOLD: threads that share a digit's rows
  if (FOLD) {
    static_assert(!FOLD || 2 * T <= kTile, "the partial sums go through skey");
    for (int i0 = t >> 8; i0 < ntiles; i0 += 16 * kParts) {
      uint32_t c[16];
#pragma unroll
      for (int i = 0; i < 16; ++i)
        c[i] = hist[(int64_t)min(i0 + i * kParts, ntiles - 1) * 256 + (t & 255)];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        dtot += i0 + i * kParts < ntiles ? c[i] : 0;
        before += i0 + i * kParts < tile ? c[i] : 0;
      }
    }
    skey[t] = dtot;
    skey[T + t] = before;
  } else if (t < 256) {
    dtot = rowtot[t];
    before = hist[(int64_t)t * ntiles + tile];
  }
#pragma unroll
  for (int q = 0; q < 256 / 64; ++q) wcnt[0][q * T + t] = 0;
  __syncthreads();
  uint32_t pos[R];  // rank among the wave's pairs of the same digit
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool in = l0 + 64 * r < cnt;
    const uint32_t d = (key[r] >> shift) & 255u;
    const uint64_t peers = digit_peers(d, in);
    const uint32_t rank = (uint32_t)__popcll(peers & ((1ull << lane) - 1ull));
    const uint32_t old = wcnt[w][d];
    // (a wave's LDS accesses are served in order: every lane has read the
    // count before the digit's first lane raises it)
    __builtin_amdgcn_wave_barrier();
    if (in && rank == 0) wcnt[w][d] = old + (uint32_t)__popcll(peers);
    __builtin_amdgcn_wave_barrier();
    pos[r] = old + rank;
  }
  __syncthreads();
  uint32_t tcnt = 0, li = 0, gi = 0;
  if (t < 256) {  // whole waves
    if (FOLD) {
      dtot = before = 0;
#pragma unroll
      for (int q = 0; q < kParts; ++q) {
        dtot += skey[q * 256 + t];
        before += skey[T + q * 256 + t];
      }
    }
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww) {
      const uint32_t c = wcnt[ww][t];
      wcnt[ww][t] = tcnt;
      tcnt += c;
    }
    li = (uint32_t)wave_scan((int)tcnt, lane, OpAdd());
    gi = (uint32_t)wave_scan((int)dtot, lane, OpAdd());
    if (lane == 63) {
      sh[0][w] = li;
      sh[1][w] = gi;
    }
  }
  __syncthreads();
  if (t < 256) {
    uint32_t l = li - tcnt, g = gi - dtot + before;
    for (int ww = 0; ww < w; ++ww) {
      l += sh[0][ww];
      g += sh[1][ww];
    }
    lstart[t] = l;
    gbase[t] = g - l;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (l0 + 64 * r < cnt) {
      const uint32_t d = (key[r] >> shift) & 255u;
      const uint32_t p = lstart[d] + wcnt[w][d] + pos[r];
      skey[p] = key[r];
      sval[p] = val[r];
    }
  }
  __syncthreads();
#pragma unroll 4
  for (int p = t; p < cnt; p += T) {
    const uint32_t k = skey[p];
    const uint32_t o = gbase[(k >> shift) & 255u] + (uint32_t)p;
    if (kout) kout[o] = k;
    vout[o] = sval[p];
  }
}

// SGS: the sort keys of the 2G list entries, senders (side 0) then
// receivers (side 1), each side by value descending; absent entries (value
// 0) sort last in their side, ties (stable) by group.
__global__ __launch_bounds__(256) void k_rpa_keys(Model m, Buffers b) {
  const Ctrl* c = b.ctrl;
  if (!c->do_resample) return;
  const int64_t G = m.rpa_G;
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= 2 * G) return;
  const int side = j >= G ? 1 : 0;
  const int64_t g = j - side * G;
  // values are below N < 2^31
  const uint64_t v = rpa_value(b, m.rpa_group, g, side);
  b.rkey0[j] = ((uint32_t)side << 31) | (v > 0 ? (uint32_t)(0x7fffffffu - (uint32_t)v) : 0x7fffffffu);
  b.rval0[j] = (int32_t)g;
}

// Group at position k of one side's list: group order (GS) or the sorted
// order (SGS: the sort's result is back in the ping buffers).
__device__ __forceinline__ int64_t rpa_at(const Model& m, const Buffers& b, int side, int64_t k) {
  return m.dlb == 1 ? (int64_t)b.rval0[side * (int64_t)m.rpa_G + k] : k;
}

// The plan: over each side's list in schedule order, the exclusive prefix of
// the values, in three launches: per tile of kSortTile positions the sum
// (k_rpa_plan_tiles), their exclusive prefixes over the tiles
// (k_rpa_plan_scan, one workgroup per side), then each position's prefix
// (k_rpa_plan_apply): the surplus before each sender, each receiver's first
// surplus particle.
__global__ __launch_bounds__(256) void k_rpa_plan_tiles(Model m, Buffers b) {
  __shared__ uint64_t sh[4];
  const Ctrl* c = b.ctrl;
  if (!c->do_resample) return;
  const int side = blockIdx.y;
  const int64_t G = m.rpa_G, n = m.rpa_group;
  const int64_t nt2 = (G + kSortTile - 1) / kSortTile;
  const int64_t k0 = (int64_t)blockIdx.x * kSortTile + 4 * threadIdx.x;
  uint64_t sv = 0;
  for (int i = 0; i < 4; ++i) {
    const int64_t k = k0 + i;
    if (k < G) sv += rpa_value(b, n, rpa_at(m, b, side, k), side);
  }
  uint64_t tv;
  block_excl_sum(sv, sh, &tv);
  if (threadIdx.x == 0) b.rtsum[side * nt2 + blockIdx.x] = tv;
}

__global__ __launch_bounds__(256) void k_rpa_plan_scan(Model m, Buffers b) {
  __shared__ uint64_t sh[4];
  const Ctrl* c = b.ctrl;
  if (!c->do_resample) return;
  const int side = blockIdx.x;
  const int64_t G = m.rpa_G;
  const int64_t nt2 = (G + kSortTile - 1) / kSortTile;
  uint64_t* ts = b.rtsum + side * nt2;
  uint64_t cv = 0;
  for (int64_t i0 = 0; i0 < nt2; i0 += 256) {
    const int64_t i = i0 + threadIdx.x;
    const uint64_t v = i < nt2 ? ts[i] : 0;
    uint64_t tv;
    const uint64_t ev = block_excl_sum(v, sh, &tv);
    if (i < nt2) ts[i] = cv + ev;
    cv += tv;
  }
}

__global__ __launch_bounds__(256) void k_rpa_plan_apply(Model m, Buffers b) {
  __shared__ uint64_t sh[4];
  const Ctrl* c = b.ctrl;
  if (!c->do_resample) return;
  const int side = blockIdx.y;
  const int64_t G = m.rpa_G, n = m.rpa_group;
  const int64_t nt2 = (G + kSortTile - 1) / kSortTile;
  const int64_t k0 = (int64_t)blockIdx.x * kSortTile + 4 * threadIdx.x;
  int64_t g[4];
  uint64_t v[4];
  uint64_t sv = 0;
  for (int i = 0; i < 4; ++i) {
    const int64_t k = k0 + i;
    g[i] = k < G ? rpa_at(m, b, side, k) : 0;
    v[i] = k < G ? rpa_value(b, n, g[i], side) : 0;
    sv += v[i];
  }
  uint64_t tv;
  uint64_t pv = block_excl_sum(sv, sh, &tv) + b.rtsum[side * nt2 + blockIdx.x];
  for (int i = 0; i < 4; ++i) {
    if (v[i] > 0) {
      if (side == 0)
        b.rscum[g[i]] = (int64_t)pv;
      else
        b.rdbase[g[i]] = (int64_t)pv;
      pv += v[i];
    }
  }
}

// The surplus stream: the q-th surplus offspring in schedule order is
// offspring n + j of the sender g with q = (surplus of the senders before g) +
// j. Each thread takes four consecutive
// systematic slots t: slot t is offspring t - first(g) of the group g that
// holds its ancestor (every load is issued before any store).
__global__ __launch_bounds__(256) void k_rpa_stream(Model m, Buffers b) {
  const Ctrl* c = b.ctrl;
  if (!c->do_resample) return;
  const int64_t t0 = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x);
  const int64_t N = m.n;
  if (t0 >= N) return;
  const int64_t n = m.rpa_group;
  const int32_t* __restrict__ asys = b.asys;
  int32_t a[4];
  if (t0 + 4 <= N && (reinterpret_cast<uintptr_t>(asys + t0) & 15) == 0) {
    const int4 v = *reinterpret_cast<const int4*>(asys + t0);
    a[0] = v.x;
    a[1] = v.y;
    a[2] = v.z;
    a[3] = v.w;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = asys[min(t0 + i, N - 1)];
  }
  int64_t q[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    // ancestors are below N < 2^31: a 32-bit quotient
    const int64_t g = (int64_t)((uint32_t)a[i] / (uint32_t)n);
    const int64_t j = t0 + i - b.rfirst[g] - n;
    q[i] = (t0 + i < N && j >= 0) ? b.rscum[g] + j : -1;  // -1: kept by its group
  }
  int32_t* __restrict__ out = b.rstream;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (q[i] >= 0 && q[i] < N) out[q[i]] = a[i];  // a balanced plan has q < N
}

// Four consecutive output slots per thread: each takes its group's own
// offspring first, then the surplus stream from the receiver's first
// surplus particle (every load is issued before any store).
__global__ __launch_bounds__(256) void k_rpa_route(Model m, Buffers b) {
  const Ctrl* c = b.ctrl;
  if (!c->do_resample) return;
  const int64_t s0 = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x);
  const int64_t N = m.n;
  if (s0 >= N) return;
  const int64_t n = m.rpa_group;
  const int32_t* __restrict__ asys = b.asys;
  const int32_t* __restrict__ stream = b.rstream;
  int32_t v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t s = min(s0 + i, N - 1);
    const int64_t g = (int64_t)((uint32_t)s / (uint32_t)n);
    const int64_t p = s - g * n;
    const int64_t f0 = b.rfirst[g];
    const int64_t keep = min(b.rfirst[g + 1] - f0, n);
    const int64_t q = min(max(b.rdbase[g] + (p - keep), (int64_t)0), N - 1);
    // (both indices stay in [0, N) whichever way the choice goes; a balanced
    // plan never clamps q)
    v[i] = p < keep ? asys[min(f0 + p, N - 1)] : stream[q];
  }
  int32_t* __restrict__ out = b.anc;
  if (s0 + 4 <= N && (reinterpret_cast<uintptr_t>(out + s0) & 15) == 0) {
    *reinterpret_cast<int4*>(out + s0) = make_int4(v[0], v[1], v[2], v[3]);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (s0 + i < N) out[s0 + i] = v[i];
  }
}

// ------------------------------------------------ standalone DLB schedules
// The DLB schedules of Section 4 for any number of groups. The lists: the
// 2G entries (senders, then receivers) radix-sorted by key, where GS keys a
// present entry by its group and SGS / LGS by the complement of its value
// (descending, ties in group order); absent entries sort last in their side.
__global__ __launch_bounds__(256) void k_dlb_keys(int32_t kind, const int32_t* __restrict__ counts,
                                                  int32_t G, int32_t n, uint32_t* __restrict__ key,
                                                  int32_t* __restrict__ val,
                                                  int32_t* __restrict__ nsr) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j < 2) nsr[j] = 0;
  if (j >= 2 * (int64_t)G) return;
  const int side = j >= G ? 1 : 0;
  const int64_t g = j - side * (int64_t)G;
  const int64_t v = side == 0 ? (int64_t)counts[g] - n : (int64_t)n - counts[g];
  // values and groups are below 2^31
  const uint32_t low = v <= 0 ? 0x7fffffffu
                              : (kind == 0 ? (uint32_t)g : 0x7fffffffu - (uint32_t)min(v, (int64_t)0x7ffffffe));
  key[j] = ((uint32_t)side << 31) | low;
  val[j] = (int32_t)g;
}

// The lists' prefixes, per side, and later the senders' entries': the tiles' sums
// in one launch with whatever makes the values, the prefixes in the next, where
// each workgroup adds up the tiles before its own
// (kScanFold of them at most; beyond, k_scan_top does it once). With the lists'
// sort in eight launches instead of twelve, a schedule of 152,000 groups takes 14
// launches and 94 us of kernels against 27 and 122 us.

// The sum of the tile sums before `tile` (its prefix already, when `scanned`).
__device__ __forceinline__ uint64_t tiles_before(const uint64_t* __restrict__ tsum, int64_t tile,
                                                 bool scanned, uint64_t* sh) {
  if (scanned) return tsum[tile];
  uint64_t s = 0, total;
  for (int64_t i = threadIdx.x; i < tile; i += 256) s += tsum[i];
  block_excl_sum(s, sh, &total);
  return total;
}

__global__ __launch_bounds__(256) void k_scan_top(uint64_t* __restrict__ tsum, int64_t ntiles) {
  __shared__ uint64_t sh[4];
  tsum += blockIdx.x * ntiles;
  uint64_t carry = 0;
  for (int64_t i0 = 0; i0 < ntiles; i0 += 256) {
    const int64_t i = i0 + threadIdx.x;
    const uint64_t v = i < ntiles ? tsum[i] : 0;
    uint64_t t;
    const uint64_t ex = block_excl_sum(v, sh, &t);
    if (i < ntiles) tsum[i] = carry + ex;
    carry += t;
  }
}

// Exclusive prefixes of tile `tile`'s 256 PER values into out, by the last tile
// the total into out[len].
template <int PER>
__device__ __forceinline__ void scan_tile(const uint64_t* __restrict__ in, int64_t len,
                                          const uint64_t* __restrict__ tsum, int64_t tile,
                                          bool scanned, uint64_t* __restrict__ out) {
  __shared__ uint64_t sh[4], sh2[4];
  const int64_t k0 = (tile * 256 + threadIdx.x) * PER;
  uint64_t v[PER], s = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    v[i] = k0 + i < len ? in[k0 + i] : 0;
    s += v[i];
  }
  const uint64_t base = tiles_before(tsum, tile, scanned, sh2);
  uint64_t tot;
  uint64_t p = base + block_excl_sum(s, sh, &tot);
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (k0 + i < len) out[k0 + i] = p;
    p += v[i];
  }
  if (threadIdx.x == 0 && (tile + 1) * 256 * PER >= len) out[len] = base + tot;
}

// The surplus (side 0) or deficit (side 1) at each list position, 0 past the
// present entries, with their tile sums; the present entries come first, so the
// last one marks their number (none: k_dlb_keys has left 0).
__global__ __launch_bounds__(256) void k_dlb_values(const int32_t* __restrict__ counts, int32_t G,
                                                    int32_t n, const int32_t* __restrict__ val,
                                                    uint64_t* __restrict__ vals,
                                                    uint64_t* __restrict__ tsum,
                                                    int32_t* __restrict__ nsr) {
  __shared__ uint64_t sh[4];
  const int side = blockIdx.y;
  const int64_t k0 = (int64_t)blockIdx.x * kSortTile + 4 * threadIdx.x;
  const int32_t* lv = val + side * (int64_t)G;
  int64_t c[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) c[i] = lv[min(k0 + i, (int64_t)G - 1)];
#pragma unroll
  for (int i = 0; i < 5; ++i) c[i] = counts[c[i]];
  uint64_t v[5], s = 0;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const int64_t d = side == 0 ? c[i] - n : n - c[i];
    v[i] = k0 + i < G && d > 0 ? (uint64_t)d : 0;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (k0 + i < G) vals[side * (int64_t)G + k0 + i] = v[i];
    if (v[i] > 0 && v[i + 1] == 0) nsr[side] = (int32_t)(k0 + i + 1);
    s += v[i];
  }
  uint64_t tot;
  block_excl_sum(s, sh, &tot);
  if (threadIdx.x == 0) tsum[side * (int64_t)gridDim.x + blockIdx.x] = tot;
}

__global__ __launch_bounds__(256) void k_dlb_prefix(const uint64_t* __restrict__ vals, int32_t G,
                                                    const uint64_t* __restrict__ tsum,
                                                    int32_t scanned, uint64_t* __restrict__ cs,
                                                    uint64_t* __restrict__ cd) {
  const int side = blockIdx.y;
  scan_tile<kSortTile / 256>(vals + side * (int64_t)G, G, tsum + side * (int64_t)gridDim.x, blockIdx.x,
            scanned != 0, side ? cd : cs);
}

__global__ __launch_bounds__(256) void k_dlb_entry_prefix(const uint64_t* __restrict__ cnt,
                                                          int32_t G,
                                                          const uint64_t* __restrict__ tsum,
                                                          int32_t scanned,
                                                          uint64_t* __restrict__ E) {
  scan_tile<1>(cnt, G, tsum, blockIdx.x, scanned != 0, E);
}

// The last j in [lo, hi] with a[j] <= v, a non-decreasing and a[lo] <= v: by one
// lane, or by the whole wave 64 ways at a time (v uniform).
__device__ __forceinline__ int64_t last_le(const uint64_t* a, int64_t lo, int64_t hi,
                                           uint64_t v) {
  while (lo < hi) {
    const int64_t mid = (lo + hi + 1) >> 1;
    if (a[mid] <= v) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}
// The same by steps that double from lo, for a j that is near it.
__device__ __forceinline__ int64_t last_le_near(const uint64_t* a, int64_t lo, int64_t hi,
                                                uint64_t v) {
  int64_t step = 1;
  while (lo + step <= hi && a[lo + step] <= v) {
    lo += step;
    step *= 2;
  }
  return last_le(a, lo, min(hi, lo + step - 1), v);
}
__device__ __forceinline__ int64_t wave_last_le(const uint64_t* __restrict__ a, int64_t lo,
                                                int64_t hi, uint64_t v) {
  const int lane = threadIdx.x & 63;
  while (lo < hi) {  // uniform
    const int64_t step = (hi - lo + 63) / 64, p = lo + (lane + 1) * step;
    const bool le = p <= hi && a[min(p, hi)] <= v;
    lo += __popcll(__ballot(le)) * step;
    hi = min(hi, lo + step - 1);
  }
  return lo;
}

// GS / SGS: the greedy walk of the two lists (Alg. 2, with filled receivers
// skipped) pairs sender i with every receiver whose deficit interval
// [cd_j, cd_j + de_j) overlaps its surplus interval [cs_i, cs_i + su_i),
// both laid end to end in list order and cut at T = min(total surplus,
// total deficit). Per sender: its first receiver and its number of entries;
// per workgroup's 256 senders their sum. A workgroup's senders meet a short range
// of receivers, which one wave finds 64 ways at a time before each sender searches
// it (a search of the whole list by every thread is a chain of 17 loads).
__global__ __launch_bounds__(256) void k_dlb_count(const uint64_t* __restrict__ cs,
                                                   const uint64_t* __restrict__ cd,
                                                   const int32_t* __restrict__ nsr, int32_t G,
                                                   int32_t* __restrict__ jlo,
                                                   uint64_t* __restrict__ cnt,
                                                   uint64_t* __restrict__ tsum) {
  __shared__ uint64_t sh[4];
  __shared__ int64_t range[2];
  const int64_t i0 = (int64_t)blockIdx.x * 256, i = i0 + threadIdx.x;
  const int64_t ns = nsr[0], nr = nsr[1];
  const uint64_t T = min(cs[ns], cd[nr]);
  const int64_t i1 = min(i0 + 256, ns);  // the workgroup's present senders end here
  const uint64_t c0 = cs[min(i, ns)], c1 = min(cs[min(i + 1, ns)], T);
  if (i0 < i1 && nr > 0 && wave_index() < 2) {  // uniform
    const uint64_t v = wave_index() == 0 ? cs[i0] : min(cs[i1], T) - 1;
    const int64_t r = cs[i0] < T ? wave_last_le(cd, 0, nr - 1, v) : 0;
    if ((threadIdx.x & 63) == 0) range[wave_index()] = r;
  }
  __syncthreads();
  uint64_t n_e = 0;
  if (i < ns && c0 < T) {
    // last j with d[j] <= cs[i], then last j with d[j] < min(cs[i + 1], T),
    // which is near it
    const int64_t lo = last_le(cd, range[0], range[1], c0);
    const int64_t hi = last_le_near(cd, lo, range[1], c1 - 1);
    jlo[i] = (int32_t)lo;
    n_e = (uint64_t)(hi - lo + 1);
  }
  if (i < G) cnt[i] = n_e;
  uint64_t tot;
  block_excl_sum(n_e, sh, &tot);
  if (threadIdx.x == 0) tsum[blockIdx.x] = tot;
}

// Entry e: GS / SGS its sender (the last with entry prefix <= e) and
// receiver, the overlap of their intervals; LGS the e-th sender with the e-th
// receiver and the smaller of their values (Alg. 4, the count recorded before
// it is zeroed). Thread 0 writes the number of entries, or -1 past cap.
__global__ __launch_bounds__(256) void k_dlb_entries(int32_t kind, const int32_t* __restrict__ val,
                                                     const uint64_t* __restrict__ vals,
                                                     const uint64_t* __restrict__ cs,
                                                     const uint64_t* __restrict__ cd,
                                                     const int32_t* __restrict__ nsr, int32_t G,
                                                     const int32_t* __restrict__ jlo,
                                                     const uint64_t* __restrict__ E,
                                                     int32_t* __restrict__ sched, int32_t cap,
                                                     int32_t* __restrict__ n_entries) {
  __shared__ int64_t range[2];
  const int64_t e0 = (int64_t)blockIdx.x * 256, e = e0 + threadIdx.x;
  const int64_t ns = nsr[0], nr = nsr[1];
  const int64_t M = kind == 2 ? min(ns, nr) : (int64_t)E[G];
  if (e == 0) *n_entries = M <= cap ? (int32_t)M : -1;
  if (e0 >= M || M > cap) return;  // uniform; nothing is written past the capacity
  if (kind != 2 && wave_index() < 2) {
    // the senders of the workgroup's first and last entries
    const int64_t r =
        wave_last_le(E, 0, ns - 1, (uint64_t)(wave_index() == 0 ? e0 : min(e0 + 255, M - 1)));
    if ((threadIdx.x & 63) == 0) range[wave_index()] = r;
  }
  __syncthreads();
  if (e >= M) return;
  int64_t i, j;
  uint64_t amount;
  if (kind == 2) {
    i = e;
    j = e;
    amount = min(vals[i], vals[G + j]);
  } else {
    i = last_le(E, range[0], range[1], (uint64_t)e);
    j = jlo[i] + (e - (int64_t)E[i]);
    const uint64_t* d = cd;
    const uint64_t T = min(cs[ns], d[nr]);
    amount = min(min(cs[i + 1], d[j + 1]), T) - max(cs[i], d[j]);
  }
  sched[3 * e] = val[i];
  sched[3 * e + 1] = val[G + j];
  sched[3 * e + 2] = (int32_t)amount;
}

// --------------------------------------------------------------- batches
// Independent filters (tracks) advance together: each launch covers every
// track, one workgroup per work item (track, index of the track's block,
// chunk, segment or group) from a list built on the host, with the track's
// model and buffers read from device arrays.

// A pointer that was read from memory, as one to global memory (which it is):
// the compiler otherwise has to use flat accesses, which also occupy the LDS path
// and wait on its counter (256 tracks, 11.7 M particles: the fused step 287 -> 264 us,
// the wide one 59.9 -> 56.1).
template <class T>
__device__ __forceinline__ T* as_global(T* p) {
  return (T*)(__attribute__((address_space(1))) T*)reinterpret_cast<uintptr_t>(p);
}
__device__ __forceinline__ Buffers track_buffers(const Buffers& s) {
  Buffers b = s;
  b.ctrl = as_global(s.ctrl);
  b.X0 = as_global(s.X0);
  b.X1 = as_global(s.X1);
  b.E0 = as_global(s.E0);
  b.E1 = as_global(s.E1);
  b.R0 = as_global(s.R0);
  b.R1 = as_global(s.R1);
  b.pfx = as_global(s.pfx);
  b.CR = as_global(s.CR);
  b.cpre = as_global(s.cpre);
  b.anc = as_global(s.anc);
  b.lw64 = as_global(s.lw64);
  b.lwg = as_global(s.lwg);
  b.hq = as_global(s.hq);
  return b;
}

__device__ __forceinline__ WeightSrc own_weights(const Buffers& b) {
  WeightSrc w{};
  w.E0 = b.E0;
  w.E1 = b.E1;
  w.rec0 = b.R0;
  w.rec1 = b.R1;
  w.use_cur = 1;
  w.log_src = 0;
  return w;
}

__global__ __launch_bounds__(256) void k_init_batch(const Model* __restrict__ ms,
                                                    const Buffers* __restrict__ bs,
                                                    const BatchItem* __restrict__ items) {
  const BatchItem it = items[blockIdx.x];
  init_body(ms[it.track], track_buffers(bs[it.track]), it.idx);
}

template <int P>
__global__ __launch_bounds__(256) void k_step_batch_wide(const Model* __restrict__ ms,
                                                         const Buffers* __restrict__ bs,
                                                         const BatchItem* __restrict__ items,
                                                         const float* __restrict__ obs) {
  __shared__ StepLds<kTileCap> L;
  const BatchItem it = items[blockIdx.x];
  step_spot<P>(ms[it.track], track_buffers(bs[it.track]), obs, it.idx, L);
}

// Every patch size up to kFusedMaxP in one launch of workgroup shape S: each
// workgroup takes its item's patch size (uniform across the workgroup) and
// shares one LDS block.
template <int S>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kShapeWaves[S])))
void k_step_batch_fused(const Model* __restrict__ ms, const Buffers* __restrict__ bs,
                        const BatchItem* __restrict__ items, const float* __restrict__ obs) {
  constexpr int T = kShapeTile[S];
  __shared__ StepLds<T> L;
  const BatchItem it = items[blockIdx.x];
  const Model& m = ms[it.track];
  const Buffers b = track_buffers(bs[it.track]);
  switch (m.P) {
    case 1: step_spot<1, false, T>(m, b, obs, it.idx, L); break;
    case 3: step_spot<3, false, T>(m, b, obs, it.idx, L); break;
    case 5: step_spot<5, false, T>(m, b, obs, it.idx, L); break;
    case 7: step_spot<7, false, T>(m, b, obs, it.idx, L); break;
    case 9: step_spot<9, false, T>(m, b, obs, it.idx, L); break;
    case 11: step_spot<11, false, T>(m, b, obs, it.idx, L); break;
    case 13: step_spot<13, false, T>(m, b, obs, it.idx, L); break;
    default: break;  // the host puts only these sizes in a fused launch
  }
}
static_assert(kFusedMaxP == 13, "k_step_batch_fused handles the odd patch sizes up to 13");

__global__ __launch_bounds__(256) void k_merge_batch(const Model* __restrict__ ms,
                                                     const Buffers* __restrict__ bs,
                                                     const BatchItem* __restrict__ items) {
  const BatchItem it = items[blockIdx.x];
  merge_chunk(ms[it.track], track_buffers(bs[it.track]), 0, it.idx);
}

// One workgroup per track. (256 tracks of 46 K particles: 8.8 us, and 5.2 + 5.9 and the
// gap between them in two launches.)
__global__ __launch_bounds__(256 * kOneMergeChunks) void k_merge_one_batch(
    const Model* __restrict__ ms, const Buffers* __restrict__ bs) {
  const Buffers b = track_buffers(bs[blockIdx.x]);
  // The workgroup has waves for the track with the most chunks: this one's idle waves
  // end here (whole waves, which the barriers of the merge then do not wait for) instead
  // of merging nothing beside those of other tracks. 2000 tracks of one chunk and one
  // of four: 37 -> 20 us, and 26 in two launches.
  if ((wave_index() >> 2) >= b.nch) return;
  merge_one<false>(ms[blockIdx.x], b, 0, 0.0);
}
__global__ __launch_bounds__(256) void k_merge_final_batch(const Model* __restrict__ ms,
                                                           const Buffers* __restrict__ bs) {
  merge_final<4>(ms[blockIdx.x], track_buffers(bs[blockIdx.x]), 0, 0.0);
}

__global__ __launch_bounds__(kWave) void k_anc_batch(const Model* __restrict__ ms,
                                                   const Buffers* __restrict__ bs,
                                                   const BatchItem* __restrict__ items) {
  const BatchItem it = items[blockIdx.x];
  const Buffers b = track_buffers(bs[it.track]);
  anc_seg<false>(ms[it.track], b, own_weights(b), it.idx);
}

// The queued chunks of all the tracks in `tracks` as one list, track after
// track (a track that did not resample this step has none). Wave w takes the
// list entries w, w + gridDim.x, ..., so a track whose weights collapsed gets
// as many waves as its chunks need. The tracks are counted kFillTracks at a
// time, their loads issued together.
constexpr int kFillTracks = 4 * kWave;
__global__ __launch_bounds__(kWave) void k_fill_batch(const Model* __restrict__ ms,
                                                    const Buffers* __restrict__ bs,
                                                    const int32_t* __restrict__ tracks,
                                                    int32_t n_tracks) {
  const int lane = threadIdx.x;
  const int64_t G = gridDim.x;
  int64_t base = 0;  // list entries of the tracks before this pass's
  for (int32_t j0 = 0; j0 < n_tracks; j0 += kFillTracks) {
    int32_t tr[4];
    int cnt[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int32_t j = j0 + u * kWave + lane;
      tr[u] = j < n_tracks ? tracks[j] : -1;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      cnt[u] = 0;
      if (tr[u] >= 0) {
        const Buffers& b = bs[tr[u]];
        const Ctrl* c = as_global(b.ctrl);
        if (c->do_resample) cnt[u] = (int)max((int64_t)0, min((int64_t)c->heavy_count, b.hq_cap));
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int incl = wave_scan(cnt[u], lane, OpAdd());
      const int tot = readlane(incl, 63);
      // the first list entry at or after base that is this wave's
      int64_t off = ((int64_t)blockIdx.x - base % G) % G;
      if (off < 0) off += G;
      for (int64_t q = base + off; q < base + tot; q += G) {
        const int r = (int)(q - base);
        // the lane whose entries [incl - cnt, incl) hold r: the lanes below
        // it are those whose entries end at or before r
        const int owner = __popcll(__ballot(incl <= r));
        const int32_t t_own = readlane(tr[u], owner);
        const int first = readlane(incl - cnt[u], owner);
        const Buffers b = track_buffers(bs[t_own]);
        fill_entry<false>(ms[t_own], b, own_weights(b), res_in(b.ctrl), r - first);
      }
      base += tot;
    }
  }
}

__global__ __launch_bounds__(256) void k_rna_batch(const Model* __restrict__ ms,
                                                   const Buffers* __restrict__ bs,
                                                   const BatchItem* __restrict__ items) {
  const BatchItem it = items[blockIdx.x];
  const Buffers b = track_buffers(bs[it.track]);
  // (a work item per group, whatever its size: one group to a workgroup)
  rna_body<4>(ms[it.track], b, own_weights(b), nullptr, it.idx);
}

// ------------------------------------------------------------- utilities
__global__ __launch_bounds__(256) void k_gather(Model m, Buffers b, float* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m.n) return;
  const Ctrl* c = b.ctrl;
  const float* X = c->cur ? b.X1 : b.X0;
  const int mode = c->mode;
  const int64_t p = (mode == kModeSys || mode == kModeRna || mode == kModeArna) ? b.anc[i] : i;
#pragma unroll
  for (int d = 0; d < 5; ++d) out[d * m.n + i] = X[d * m.n + p];
}

// Normalised log weights of the last committed step into lw64.
__global__ __launch_bounds__(256) void k_logw(Model m, Buffers b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m.n) return;
  const Ctrl* c = b.ctrl;
  const int mode = c->mode;
  if (mode == kModeSet) return;
  if (mode == kModeInit) {
    b.lw64[i] = -m.log_n;
    return;
  }
  const float* E = c->cur ? b.E1 : b.E0;
  const double* R = c->cur ? b.R1 : b.R0;
  b.lw64[i] = log((double)E[i]) + R[(i / kBlock) * kRec] - c->delta;
}

__global__ void k_set_mode(Ctrl* c, int32_t mode) { c->mode = mode; }

// Control block blockIdx.x, eight bytes per thread, to pinned host memory; with
// `clear` its roll-back report is zeroed (by the thread that has read it).
static_assert(sizeof(Ctrl) % 8 == 0 && sizeof(Ctrl) / 8 <= kWave &&
                  offsetof(Ctrl, rolled_back) % 8 == 4,
              "one word per thread, the report in the upper half of one");
__global__ __launch_bounds__(kWave) void k_report(Ctrl* c, int32_t clear, Ctrl* out) {
  constexpr int kWords = (int)(sizeof(Ctrl) / 8);
  const int t = threadIdx.x;
  if (t >= kWords) return;
  const uint64_t v = reinterpret_cast<const uint64_t*>(c + blockIdx.x)[t];
  reinterpret_cast<uint64_t*>(out + blockIdx.x)[t] = v;
  if (clear && t == (int)(offsetof(Ctrl, rolled_back) / 8) && (v >> 32) != 0)
    c[blockIdx.x].rolled_back = 0;
}

__global__ __launch_bounds__(256) void k_philox(uint32_t k0, uint32_t k1,
                                                const uint4* __restrict__ ctr,
                                                uint4* __restrict__ out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = philox(ctr[i], k0, k1);
}

// ---------------------------------------------------------------- launches
// Every kernel goes out through launch_k: onto the stream, or, while a
// StepGraph records on the calling thread, into its graph.
thread_local StepGraph* t_rec = nullptr;

template <class... T>
struct ArgTuple final : StepGraph::Args {
  std::tuple<T...> v;
  template <class... A>
  explicit ArgTuple(A&&... a) : v(std::forward<A>(a)...) {}
};

template <class Tup, size_t... I>
std::array<void*, sizeof...(I)> arg_ptrs(Tup& t, std::index_sequence<I...>) {
  return {{static_cast<void*>(&std::get<I>(t))...}};
}

template <class T>
void note_frame(T&, const float*, std::vector<const float**>*) {}
void note_frame(const float*& p, const float* frame, std::vector<const float**>* out) {
  if (p == frame) out->push_back(&p);
}

template <class... P, class... A>
hipError_t launch_k(void (*k)(P...), dim3 grid, dim3 block, hipStream_t s, A&&... a) {
  static_assert(sizeof...(P) == sizeof...(A), "kernel argument count");
  constexpr auto idx = std::index_sequence_for<P...>{};
  if (!t_rec) {
    std::tuple<P...> v(std::forward<A>(a)...);
    std::array<void*, sizeof...(P)> argv = arg_ptrs(v, idx);
    return hipLaunchKernel(reinterpret_cast<const void*>(k), grid, block, argv.data(), 0, s);
  }
  auto pack = std::make_unique<ArgTuple<P...>>(std::forward<A>(a)...);
  const std::array<void*, sizeof...(P)> argv = arg_ptrs(pack->v, idx);
  std::vector<const float**> slots;
  std::apply([&](auto&... x) { (note_frame(x, t_rec->frame(), &slots), ...); }, pack->v);
  return t_rec->add(reinterpret_cast<const void*>(k), grid, block, std::move(pack),
                    std::vector<void*>(argv.begin(), argv.end()), std::move(slots));
}

template <int P>
hipError_t launch_spot(const Model& m, const Buffers& b, const float* obs, hipStream_t s) {
  const dim3 grid((unsigned)b.nb), block(kBlock);
  if (m.grad) return launch_k(k_step_spot_grad<P>, grid, block, s, m, b, obs);
  if constexpr (P <= kFusedMaxP) {
    if (m.shape == 1) return launch_k(k_step_spot<P, 1>, grid, block, s, m, b, obs);
    return launch_k(k_step_spot<P, 0>, grid, block, s, m, b, obs);
  } else {
    return launch_k(k_step_spot_wide<P>, grid, block, s, m, b, obs);
  }
}

inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

template <int P>
hipError_t launch_spot_batch(const Model* ms, const Buffers* bs, const BatchItem* items,
                             int64_t n_items, const float* obs, hipStream_t s) {
  return launch_k(k_step_batch_wide<P>, dim3((unsigned)n_items), dim3(kBlock), s, ms, bs, items,
                  obs);
}

}  // namespace

StepGraph::~StepGraph() {
  if (t_rec == this) t_rec = nullptr;
  if (exec_) (void)hipGraphExecDestroy(exec_);
  if (graph_) (void)hipGraphDestroy(graph_);
}

hipError_t StepGraph::begin(const float* frame) {
  if (t_rec || graph_) return hipErrorInvalidValue;  // one recording per graph and thread
  const hipError_t e = hipGraphCreate(&graph_, 0);
  if (e != hipSuccess) return e;
  frame_ = frame;
  t_rec = this;
  return hipSuccess;
}

void StepGraph::stop() {
  if (t_rec == this) t_rec = nullptr;
}

hipError_t StepGraph::instantiate() {
  if (t_rec == this || nodes_.empty()) return hipErrorInvalidValue;
  return hipGraphInstantiate(&exec_, graph_, nullptr, nullptr, 0);
}

hipError_t StepGraph::add(const void* fn, dim3 grid, dim3 block, std::unique_ptr<Args> args,
                          std::vector<void*> argv, std::vector<const float**> frame_slots) {
  Node n;
  n.args = std::move(args);
  n.argv = std::move(argv);
  n.frame_slots = std::move(frame_slots);
  n.params.func = const_cast<void*>(fn);
  n.params.gridDim = grid;
  n.params.blockDim = block;
  n.params.sharedMemBytes = 0;
  n.params.kernelParams = n.argv.data();  // moving the vector keeps its storage
  n.params.extra = nullptr;
  const hipGraphNode_t* deps = deps_.empty() ? nullptr : deps_.data();
  const hipError_t e = hipGraphAddKernelNode(&n.node, graph_, deps, deps_.size(), &n.params);
  if (e != hipSuccess) return e;
  if (in_group_) {
    group_.push_back(n.node);
    open_blocks_ += (int64_t)grid.x * grid.y * grid.z;
  } else {
    deps_.assign(1, n.node);
  }
  nodes_.push_back(std::move(n));
  return hipSuccess;
}

void StepGraph::group_begin() {
  in_group_ = true;
  group_.clear();
  open_blocks_ = 0;
}

void StepGraph::group_end() {
  in_group_ = false;
  if (!group_.empty()) deps_ = group_;
  if (group_.size() > group_launches_) {
    group_launches_ = group_.size();
    group_blocks_ = open_blocks_;
  }
  group_.clear();
}

void launch_group_begin() {
  if (t_rec) t_rec->group_begin();
}

void launch_group_end() {
  if (t_rec) t_rec->group_end();
}

hipError_t StepGraph::set_frame(const float* frame) {
  if (!exec_) return hipErrorInvalidValue;
  if (frame == frame_) return hipSuccess;
  for (Node& n : nodes_) {
    if (n.frame_slots.empty()) continue;
    for (const float** slot : n.frame_slots) *slot = frame;
    const hipError_t e = hipGraphExecKernelNodeSetParams(exec_, n.node, &n.params);
    if (e != hipSuccess) return e;
  }
  frame_ = frame;
  return hipSuccess;
}

// Scratch of the allocation-free standalone resampler: every device that
// runs it holds one copy until the process ends. Host code must not use the
// array's name as a device address (on the host it names a stand-in): the
// device address comes from hipGetSymbolAddress, per device.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t static_scratch(void** ptr, size_t* bytes) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    // with this device current: its own copy of the array
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p || reinterpret_cast<uintptr_t>(p) % 256 != 0) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  *bytes = kStaticScratchBytes;
  return hipSuccess;
}

namespace {
// The sort of `count` pairs in tiles of T * R: four passes, ping -> pong on
// even ones and back on odd ones, so the result lands in ping (v0; the last
// pass leaves the keys unwritten). positions: the values start as the pairs'
// positions instead of v0.
template <int T, int R, bool FOLD>
hipError_t radix_sort_tiles(uint32_t* k0, uint32_t* k1, int32_t* v0, int32_t* v1, uint32_t* hist,
                            uint32_t* row, int64_t count, bool positions, const Ctrl* gate,
                            hipStream_t s) {
  static_assert(T * R >= kSortTile, "the digit counts hold 256 per kSortTile pairs");
  const int32_t nt = (int32_t)((count + T * R - 1) / (T * R));
  hipError_t e = hipSuccess;
  for (int pass = 0; pass < 4 && e == hipSuccess; ++pass) {
    const uint32_t* kin = pass & 1 ? k1 : k0;
    const int32_t* vin = pass & 1 ? v1 : (pass == 0 && positions ? nullptr : v0);
    uint32_t* kout = pass == 3 ? nullptr : (pass & 1 ? k0 : k1);
    int32_t* vout = pass & 1 ? v0 : v1;
    e = launch_k(k_radix_hist<T, R, FOLD>, dim3((unsigned)nt), dim3(T), s, kin, count, 8 * pass,
                 hist, nt, gate);
    if (e == hipSuccess && !FOLD)
      e = launch_k(k_radix_rowscan, dim3(256), dim3(256), s, hist, nt, row, gate);
    if (e == hipSuccess)
      e = launch_k(k_radix_scatter<T, R, FOLD>, dim3((unsigned)nt), dim3(T), s, kin, vin, kout,
                   vout, count, 8 * pass, (const uint32_t*)hist, (const uint32_t*)row, nt, gate);
  }
  return e;
}

hipError_t radix_sort(uint32_t* k0, uint32_t* k1, int32_t* v0, int32_t* v1, uint32_t* hist,
                      uint32_t* row, int64_t count, bool positions, const Ctrl* gate,
                      hipStream_t s) {
  if (count >= kSortLarge)
    return radix_sort_tiles<256, 16, false>(k0, k1, v0, v1, hist, row, count, positions, gate, s);
  if (count > kSortFold)
    return radix_sort_tiles<256, 4, false>(k0, k1, v0, v1, hist, row, count, positions, gate, s);
  return radix_sort_tiles<1024, 4, true>(k0, k1, v0, v1, hist, row, count, positions, gate, s);
}
}  // namespace

hipError_t launch_init(const Model& m, const Buffers& b, hipStream_t s) {
  hipError_t e = launch_k(k_init, dim3(grid_for(m.n, 256)), dim3(256), s, m, b);
  if (e != hipSuccess || m.init_kind != 3) return e;
  // Z order: sort the keys with their draw indices (stable), then place
  e = radix_sort(b.zkey0, b.zkey1, b.zval0, b.zval1, b.zhist, b.zrow, m.n, true, nullptr, s);
  if (e == hipSuccess) e = launch_k(k_init_place, dim3(grid_for(m.n, 256)), dim3(256), s, m, b);
  return e;
}

hipError_t launch_step(const Model& m, const Buffers& b, const float* obs, hipStream_t s) {
  if (m.obs == 1) {
    return launch_k(k_step_lg, dim3((unsigned)b.nb), dim3(kBlock), s, m, b, obs);
  }
  switch (m.P) {
    case 1: return launch_spot<1>(m, b, obs, s);
    case 3: return launch_spot<3>(m, b, obs, s);
    case 5: return launch_spot<5>(m, b, obs, s);
    case 7: return launch_spot<7>(m, b, obs, s);
    case 9: return launch_spot<9>(m, b, obs, s);
    case 11: return launch_spot<11>(m, b, obs, s);
    case 13: return launch_spot<13>(m, b, obs, s);
    case 15: return launch_spot<15>(m, b, obs, s);
    case 17: return launch_spot<17>(m, b, obs, s);
    case 19: return launch_spot<19>(m, b, obs, s);
    case 21: return launch_spot<21>(m, b, obs, s);
    case 23: return launch_spot<23>(m, b, obs, s);
    case 25: return launch_spot<25>(m, b, obs, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_init_batch(const Model* ms, const Buffers* bs, const BatchItem* items,
                             int64_t n_items, hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  return launch_k(k_init_batch, dim3((unsigned)n_items), dim3(kBlock), s, ms, bs, items);
}

hipError_t launch_step_batch_fused(int shape, const Model* ms, const Buffers* bs,
                                   const BatchItem* items, int64_t n_items, const float* obs,
                                   hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  const dim3 grid((unsigned)n_items), block(kBlock);
  if (shape == 1) return launch_k(k_step_batch_fused<1>, grid, block, s, ms, bs, items, obs);
  return launch_k(k_step_batch_fused<0>, grid, block, s, ms, bs, items, obs);
}

hipError_t launch_step_batch(int P, const Model* ms, const Buffers* bs, const BatchItem* items,
                             int64_t n_items, const float* obs, hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  switch (P) {
    case 15: return launch_spot_batch<15>(ms, bs, items, n_items, obs, s);
    case 17: return launch_spot_batch<17>(ms, bs, items, n_items, obs, s);
    case 19: return launch_spot_batch<19>(ms, bs, items, n_items, obs, s);
    case 21: return launch_spot_batch<21>(ms, bs, items, n_items, obs, s);
    case 23: return launch_spot_batch<23>(ms, bs, items, n_items, obs, s);
    case 25: return launch_spot_batch<25>(ms, bs, items, n_items, obs, s);
    default: return hipErrorInvalidValue;  // sizes up to kFusedMaxP go to the fused launch
  }
}

hipError_t launch_merge_batch(const Model* ms, const Buffers* bs, const BatchItem* items,
                              int64_t n_items, int32_t n_tracks, int64_t most, hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  if (most <= kOneMergeChunks)
    return launch_k(k_merge_one_batch, dim3((unsigned)n_tracks), dim3(256 * (unsigned)most), s, ms,
                    bs);
  const hipError_t e = launch_k(k_merge_batch, dim3((unsigned)n_items), dim3(256), s, ms, bs,
                                items);
  if (e != hipSuccess) return e;
  return launch_k(k_merge_final_batch, dim3((unsigned)n_tracks), dim3(256), s, ms, bs);
}

hipError_t launch_anc_batch(const Model* ms, const Buffers* bs, const BatchItem* items,
                            int64_t n_items, hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  return launch_k(k_anc_batch, dim3((unsigned)n_items), dim3(kWave), s, ms, bs, items);
}

hipError_t launch_fill_batch(const Model* ms, const Buffers* bs, const int32_t* tracks,
                             int32_t n_tracks, hipStream_t s) {
  if (n_tracks <= 0) return hipSuccess;
  return launch_k(k_fill_batch, dim3(kFillGridBatch), dim3(kWave), s, ms, bs, tracks, n_tracks);
}

hipError_t launch_rna_batch(const Model* ms, const Buffers* bs, const BatchItem* items,
                            int64_t n_items, hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  return launch_k(k_rna_batch, dim3((unsigned)n_items), dim3(256), s, ms, bs, items);
}

hipError_t launch_arna(const Model& m, const Buffers& b, hipStream_t s) {
  const hipError_t e =
      m.group <= kWaveGroup
          ? launch_k(k_arna_local<1>, dim3(grid_for(m.G, 4)), dim3(256), s, m, b)
          : launch_k(k_arna_local<4>, dim3((unsigned)m.G), dim3(256), s, m, b);
  if (e != hipSuccess) return e;
  return launch_k(k_arna_exchange, dim3((unsigned)m.G), dim3(256), s, m, b);
}

hipError_t launch_rpa(const Model& m, const Buffers& b, hipStream_t s) {
  const int64_t G = m.rpa_G;
  // (N + 1 entries: the last slot's successor closes the last group)
  hipError_t e = m.n <= kRpaScanN
                     ? launch_k(k_rpa_bounds, dim3(grid_for(m.n / 4 + 1, 256)), dim3(256), s, m, b)
                     : launch_k(k_rpa_first, dim3(grid_for(G + 1, 256)), dim3(256), s, m, b);
  if (G <= (m.dlb == 1 ? kRankGroups : kRankGreedy)) {
    if (e == hipSuccess)
      e = launch_k(m.dlb == 1 ? k_rpa_rank<true> : k_rpa_rank<false>, dim3(grid_for(G, 16)),
                   dim3(256), s, m, b);
  } else {
    if (e == hipSuccess && m.dlb == 1) {
      const int64_t cnt = 2 * G;
      e = launch_k(k_rpa_keys, dim3(grid_for(cnt, 256)), dim3(256), s, m, b);
      if (e == hipSuccess)
        e = radix_sort(b.rkey0, b.rkey1, b.rval0, b.rval1, b.rhist, b.rrow, cnt, false, b.ctrl, s);
    }
    const unsigned nt2 = (unsigned)((G + kSortTile - 1) / kSortTile);
    if (e == hipSuccess) e = launch_k(k_rpa_plan_tiles, dim3(nt2, 2), dim3(256), s, m, b);
    if (e == hipSuccess) e = launch_k(k_rpa_plan_scan, dim3(2), dim3(256), s, m, b);
    if (e == hipSuccess) e = launch_k(k_rpa_plan_apply, dim3(nt2, 2), dim3(256), s, m, b);
  }
  const int64_t quads = (m.n + 3) / 4;
  if (e == hipSuccess) e = launch_k(k_rpa_stream, dim3(grid_for(quads, 256)), dim3(256), s, m, b);
  if (e == hipSuccess) e = launch_k(k_rpa_route, dim3(grid_for(quads, 256)), dim3(256), s, m, b);
  return e;
}

namespace {
// Scratch of a standalone DLB schedule of G groups, carved from `base` (the
// pointers stay null when it is null); returns its size in bytes.
struct DlbScratch {
  uint32_t* key0;
  uint32_t* key1;
  int32_t* val0;
  int32_t* val1;
  uint32_t* hist;
  uint32_t* row;
  uint64_t* vals;  // list values, 2G
  uint64_t* cs;    // senders' prefixes, G + 1
  uint64_t* cd;    // receivers' prefixes, G + 1
  uint64_t* cnt;   // entries per sender, G
  uint64_t* E;     // their prefixes, G + 1
  int32_t* jlo;    // each sender's first receiver, G
  uint64_t* tsum;  // tile sums: 2 per 1024 list positions, or 1 per 256 senders
  int32_t* nsr;    // present entries per side, 2
};

size_t dlb_carve(int32_t G, char* base, DlbScratch* d) {
  const size_t L = 2 * (size_t)G, nt = (L + kSortTile - 1) / kSortTile;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* q = base ? base + off : nullptr;
    off += (bytes + 255) & ~(size_t)255;
    return q;
  };
  d->key0 = reinterpret_cast<uint32_t*>(take(L * 4));
  d->key1 = reinterpret_cast<uint32_t*>(take(L * 4));
  d->val0 = reinterpret_cast<int32_t*>(take(L * 4));
  d->val1 = reinterpret_cast<int32_t*>(take(L * 4));
  d->hist = reinterpret_cast<uint32_t*>(take(256 * nt * 4));
  d->row = reinterpret_cast<uint32_t*>(take(256 * 4));
  d->vals = reinterpret_cast<uint64_t*>(take(L * 8));
  d->cs = reinterpret_cast<uint64_t*>(take(((size_t)G + 1) * 8));
  d->cd = reinterpret_cast<uint64_t*>(take(((size_t)G + 1) * 8));
  d->cnt = reinterpret_cast<uint64_t*>(take((size_t)G * 8));
  d->E = reinterpret_cast<uint64_t*>(take(((size_t)G + 1) * 8));
  d->jlo = reinterpret_cast<int32_t*>(take((size_t)G * 4));
  d->tsum = reinterpret_cast<uint64_t*>(take(((size_t)G / 256 + 2) * 8));
  d->nsr = reinterpret_cast<int32_t*>(take(2 * 4));
  return off;
}

}  // namespace

size_t dlb_scratch_bytes(int32_t G) {
  DlbScratch d;
  return dlb_carve(G, nullptr, &d);
}

hipError_t launch_dlb_schedule(int32_t kind, const int32_t* counts, int32_t G, int32_t n,
                               int32_t* sched, int32_t cap, int32_t* n_entries, void* scratch,
                               hipStream_t s) {
  const int64_t L = 2 * (int64_t)G;
  DlbScratch d;
  dlb_carve(G, static_cast<char*>(scratch), &d);
  const unsigned nt = (unsigned)(((int64_t)G + kSortTile - 1) / kSortTile);
  const int32_t scanned = nt > kScanFold ? 1 : 0;
  hipError_t e = launch_k(k_dlb_keys, dim3(grid_for(L, 256)), dim3(256), s, kind, counts, G, n,
                          d.key0, d.val0, d.nsr);
  if (e == hipSuccess)
    e = radix_sort(d.key0, d.key1, d.val0, d.val1, d.hist, d.row, L, false, nullptr, s);
  if (e == hipSuccess)
    e = launch_k(k_dlb_values, dim3(nt, 2), dim3(256), s, counts, G, n, (const int32_t*)d.val0,
                 d.vals, d.tsum, d.nsr);
  if (e == hipSuccess && scanned)
    e = launch_k(k_scan_top, dim3(2), dim3(256), s, d.tsum, (int64_t)nt);
  if (e == hipSuccess)
    e = launch_k(k_dlb_prefix, dim3(nt, 2), dim3(256), s, (const uint64_t*)d.vals, G,
                 (const uint64_t*)d.tsum, scanned, d.cs, d.cd);
  if (kind != 2) {
    const unsigned nw = grid_for(G, 256);
    const int32_t scanned_e = nw > kScanFold ? 1 : 0;
    if (e == hipSuccess)
      e = launch_k(k_dlb_count, dim3(nw), dim3(256), s, (const uint64_t*)d.cs,
                   (const uint64_t*)d.cd, (const int32_t*)d.nsr, G, d.jlo, d.cnt, d.tsum);
    if (e == hipSuccess && scanned_e)
      e = launch_k(k_scan_top, dim3(1), dim3(256), s, d.tsum, (int64_t)nw);
    if (e == hipSuccess)
      e = launch_k(k_dlb_entry_prefix, dim3(nw), dim3(256), s, (const uint64_t*)d.cnt, G,
                   (const uint64_t*)d.tsum, scanned_e, d.E);
  }
  if (e == hipSuccess)
    e = launch_k(k_dlb_entries, dim3(grid_for(L, 256)), dim3(256), s, kind,
                 (const int32_t*)d.val0, (const uint64_t*)d.vals, (const uint64_t*)d.cs,
                 (const uint64_t*)d.cd, (const int32_t*)d.nsr, G, (const int32_t*)d.jlo,
                 (const uint64_t*)d.E, sched, cap, n_entries);
  return e;
}

hipError_t launch_merge(const Model& m, const Buffers& b, int standalone, double u_given,
                        hipStream_t s) {
  if (b.nch <= kOneMergeChunks && b.chunk == 256)
    return launch_k(m.grad ? k_merge_one<true> : k_merge_one<false>, dim3(1),
                    dim3(256 * (unsigned)b.nch), s, m, b, standalone, u_given);
  const hipError_t e = launch_k(k_merge, dim3((unsigned)b.nch), dim3(256), s, m, b, standalone);
  if (e != hipSuccess) return e;
  if (b.nch <= 64) return launch_k(k_merge_final<1>, dim3(1), dim3(64), s, m, b, standalone, u_given);
  return launch_k(k_merge_final<4>, dim3(1), dim3(256), s, m, b, standalone, u_given);
}

hipError_t launch_anc(const Model& m, const Buffers& b, const WeightSrc& w, hipStream_t s) {
  if (b.nseg <= kWave * kHelpPerLane) {
    const dim3 grid((unsigned)(b.nseg + (b.hq_cap < kHelpWaves ? b.hq_cap : kHelpWaves)));
    if (w.log_src) return launch_k(k_anc_all<true>, grid, dim3(kWave), s, m, b, w);
    return launch_k(k_anc_all<false>, grid, dim3(kWave), s, m, b, w);
  }
  const dim3 fill((unsigned)(b.hq_cap < kFillGrid ? b.hq_cap : kFillGrid));
  const dim3 segs((unsigned)b.nseg);
  hipError_t e = w.log_src ? launch_k(k_anc_log, segs, dim3(kWave), s, m, b, w)
                           : launch_k(k_anc, segs, dim3(kWave), s, m, b, w);
  if (e != hipSuccess) return e;
  return w.log_src ? launch_k(k_fill_log, fill, dim3(kWave), s, m, b, w)
                   : launch_k(k_fill, fill, dim3(kWave), s, m, b, w);
}

hipError_t launch_rna(const Model& m, const Buffers& b, const WeightSrc& w, const double* u_dev,
                      hipStream_t s) {
  if (m.group <= kWaveGroup)
    return launch_k(k_rna<1>, dim3(grid_for(m.G, 4)), dim3(256), s, m, b, w, u_dev);
  return launch_k(k_rna<4>, dim3((unsigned)m.G), dim3(256), s, m, b, w, u_dev);
}

hipError_t launch_gather(const Model& m, const Buffers& b, float* out, hipStream_t s) {
  return launch_k(k_gather, dim3(grid_for(m.n, 256)), dim3(256), s, m, b, out);
}

hipError_t launch_logw(const Model& m, const Buffers& b, hipStream_t s) {
  return launch_k(k_logw, dim3(grid_for(m.n, 256)), dim3(256), s, m, b);
}

hipError_t launch_set_mode(const Buffers& b, int32_t mode, hipStream_t s) {
  return launch_k(k_set_mode, dim3(1), dim3(1), s, b.ctrl, mode);
}

hipError_t launch_report(Ctrl* c, int32_t count, bool clear, Ctrl* out, hipStream_t s) {
  return launch_k(k_report, dim3((unsigned)count), dim3(kWave), s, c, (int32_t)clear, out);
}

hipError_t launch_records(const Model& m, const Buffers& b, const float* logw, hipStream_t s) {
  return launch_k(k_records, dim3(grid_for(b.nb, 4)), dim3(256), s, m, b, logw);
}

hipError_t launch_philox(uint64_t seed, const uint32_t* ctr, uint32_t* out, int64_t n,
                         hipStream_t s) {
  if (n == 0) return hipSuccess;
  return launch_k(k_philox, dim3(grid_for(n, 256)), dim3(256), s, (uint32_t)seed,
                  (uint32_t)(seed >> 32), reinterpret_cast<const uint4*>(ctr),
                  reinterpret_cast<uint4*>(out), n);
}

}  // namespace ppf
