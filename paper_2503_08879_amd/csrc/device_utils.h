// Device helpers for the gfx950 kernels: wave64 DPP reductions, typed 16-byte
// loads, block scans.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sagekv {

constexpr int kWave = 64;

enum : int { DT_BF16 = 0, DT_F32 = 1 };

// ---- element traits --------------------------------------------------------------------
template <int DT>
struct Elem;
template <>
struct Elem<DT_BF16> {
  static constexpr int bytes = 2;
};
template <>
struct Elem<DT_F32> {
  static constexpr int bytes = 4;
};

__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }

// The 16 bytes of one lane, eight bf16 values, as fp32 values.
__device__ __forceinline__ void unpack16(const uint4& a, float* f) {
  f[0] = bf16_lo(a.x); f[1] = bf16_hi(a.x); f[2] = bf16_lo(a.y); f[3] = bf16_hi(a.y);
  f[4] = bf16_lo(a.z); f[5] = bf16_hi(a.z); f[6] = bf16_lo(a.w); f[7] = bf16_hi(a.w);
}

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

__device__ __forceinline__ uint4 ld16(const void* p) { return *reinterpret_cast<const uint4*>(p); }
// Streaming 16-byte load (data read once: do not keep it in the caches).
__device__ __forceinline__ uint4 ld16_stream(const void* p) {
  const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st16(void* p, const uint4& v) { *reinterpret_cast<uint4*>(p) = v; }
__device__ __forceinline__ void st16_stream(void* p, const uint4& v) {
  __builtin_nontemporal_store(u32x4_t{v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4_t*>(p));
}

// ---- cross-lane sums -----------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// Sum over aligned groups of LANES consecutive lanes; every lane of the group gets the total.
template <int LANES>
__device__ __forceinline__ float group_sum(float v) {
  static_assert(LANES == 16 || LANES == 64, "");
  v += dpp_f32<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_f32<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_f32<0x141>(v);  // row_half_mirror
  v += dpp_f32<0x140>(v);  // row_mirror
  if (LANES >= 64) {
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
  }
  return v;
}

// The same sum for doubles, the moves on the two halves (shuffles through LDS: two per step and value, and a decode
// step over an fp32 cache needs a sum per token and head).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xF, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// The value of the lane 16 further (lane ^ 16): v_permlane16_swap exchanges the odd 16-lane rows of its first operand with
// the even rows of its second, so with both equal the first result holds rows 0 0 2 2 and the second rows 1 1 3 3.
// (Through an LDS shuffle an fp32 step over 8 rows x 4 heads x 512 tokens of head_dim 128 took 22.3 us, 4 rows x 7 heads
// 33.9; so 20.6 and 30.2.)
__device__ __forceinline__ double swap16_f64(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
  const bool odd = (threadIdx.x & 16) != 0;
  const uint32_t l = odd ? lo[0] : lo[1], h = odd ? hi[0] : hi[1];
  return __builtin_bit_cast(double, ((uint64_t)h << 32) | l);
}
// v of this lane + v of lane ^ 16, lane ^ 32
__device__ __forceinline__ float swap16_sum(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap32_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap16_max(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float swap32_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <int LANES>
__device__ __forceinline__ double group_sum_f64(double v) {
  static_assert(LANES == 16 || LANES == 32 || LANES == 64, "");
  v += dpp_f64<0xB1>(v);
  v += dpp_f64<0x4E>(v);
  v += dpp_f64<0x141>(v);
  v += dpp_f64<0x140>(v);
  if (LANES >= 32) v += swap16_f64(v);
  if (LANES >= 64) v += __shfl_xor(v, 32);
  return v;
}

__device__ __forceinline__ double swap32_sum_f64(double v) {  // v + v of lane ^ 32
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
  return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) + __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
}
// Four values summed over aligned groups of eight lanes; lane s of a group (`sl`) gets the total of value s % 4.  N = 1, 2: of the first value,
// of the first two in turn.
template <int N>
__device__ __forceinline__ double eight_lane_sums(double (&a)[4], int sl) {
  if constexpr (N <= 2) {
    double v = a[0] + dpp_f64<0x141>(a[0]);  // row_half_mirror
    if (N == 2) {
      const double w = a[1] + dpp_f64<0x141>(a[1]);
      v = (sl & 1 ? w : v) + dpp_f64<0xB1>(sl & 1 ? v : w);  // quad_perm [1,0,3,2]
    } else {
      v += dpp_f64<0xB1>(v);
    }
    return v + dpp_f64<0x4E>(v);  // quad_perm [2,3,0,1]
  }
  double z[2];
#pragma unroll
  for (int h = 0; h < 4; ++h) a[h] += dpp_f64<0x141>(a[h]);  // row_half_mirror
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const double lo = a[h], hi = a[h + 2];
    z[h] = (sl & 2 ? hi : lo) + dpp_f64<0x4E>(sl & 2 ? lo : hi);  // quad_perm [2,3,0,1]: from the lane that keeps the other two
  }
  const double lo = z[0], hi = z[1];
  return (sl & 1 ? hi : lo) + dpp_f64<0xB1>(sl & 1 ? lo : hi);  // quad_perm [1,0,3,2]
}

// Maximum over aligned groups of 16 lanes, in every lane of the group.
__device__ __forceinline__ float group16_max(float v) {
  v = fmaxf(v, dpp_f32<0xB1>(v));   // quad_perm [1,0,3,2]
  v = fmaxf(v, dpp_f32<0x4E>(v));   // quad_perm [2,3,0,1]
  v = fmaxf(v, dpp_f32<0x141>(v));  // row_half_mirror
  v = fmaxf(v, dpp_f32<0x140>(v));  // row_mirror
  return v;
}

// DPP moves within a wave, for scans and reductions of ints: a step costs a few cycles, a shuffle through LDS about
// fifty nanoseconds, and the single-workgroup kernels are chains of such steps.  Lanes the move has no source for get `fill`.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_i32(int fill, int v) {
  return __builtin_amdgcn_update_dpp(fill, v, CTRL, ROW_MASK, 0xF, false);
}
// inclusive prefix sum over the wave
__device__ __forceinline__ int wave_scan_incl(int v) {
  v += dpp_i32<0x111, 0xF>(0, v);  // row_shr:1
  v += dpp_i32<0x112, 0xF>(0, v);  // row_shr:2
  v += dpp_i32<0x114, 0xF>(0, v);  // row_shr:4
  v += dpp_i32<0x118, 0xF>(0, v);  // row_shr:8
  v += dpp_i32<0x142, 0xA>(0, v);  // row_bcast:15 into rows 1 and 3
  v += dpp_i32<0x143, 0xC>(0, v);  // row_bcast:31 into rows 2 and 3
  return v;
}
// maximum over the wave, in every lane (wave-uniform)
__device__ __forceinline__ int wave_max_i(int v) {
  constexpr int lo = -0x7FFFFFFF - 1;
  auto mx = [](int a, int b) { return a > b ? a : b; };
  v = mx(v, dpp_i32<0x111, 0xF>(lo, v));
  v = mx(v, dpp_i32<0x112, 0xF>(lo, v));
  v = mx(v, dpp_i32<0x114, 0xF>(lo, v));
  v = mx(v, dpp_i32<0x118, 0xF>(lo, v));
  v = mx(v, dpp_i32<0x142, 0xA>(lo, v));
  v = mx(v, dpp_i32<0x143, 0xC>(lo, v));
  return __builtin_amdgcn_readlane(v, 63);
}

// exp(x) * inv for x <= 0-ish and a normal `inv` in [2^-62, 1] (a softmax weight: inv = 1/Z), via the
// hardware exp2 with the rounding error of x*log2(e) folded back in (relative error a few 1e-7 where
// the result is a normal number).  The hardware exp2 returns 0 for every result under 2^-126, whereas
// the product is wanted correctly rounded all the way down through the denormal range (scores are
// RANKED, and fp32 keeps denormals): an argument more than 64 octaves down is raised by 64 octaves
// before exp2 (exact: the sum has a finer ulp than the argument) and the factor is lowered by 2^-64
// instead, so the final multiply rounds into the denormal range like any fp32 product.  Results
// under 2^-190 * inv come out as 0, which is also their nearest fp32 value.
__device__ __forceinline__ float exp_times(float x, float inv) {
  const float l2e_hi = 1.44269502162933349609375f;  // float(log2 e)
  const float l2e_lo = 1.92596299112661746e-8f;     // log2 e - l2e_hi
  const float t = x * l2e_hi;
  float e = fmaf(x, l2e_hi, -t);
  e = fmaf(x, l2e_lo, e);
  const bool far = t < -64.f;
  float r = __builtin_amdgcn_exp2f(far ? t + 64.f : t);
  r = fmaf(r, e * 0.693147182464599609375f, r);
  return r * (far ? inv * 0x1p-64f : inv);
}

// Absolute slack that goes with the relative band around a coarse k-th score: below 2^-126 an fp32
// score is a multiple of 2^-149, each head's term is rounded to that grid, and up to 64 heads add up.
constexpr float kDenormSlack = 0x1p-142f;

__device__ __forceinline__ float exp_fast(float x) { return __builtin_amdgcn_exp2f(x * 1.44269502162933349609375f); }

// Which terms of a head's softmax sum need an fp64 exponent.  An fp32 logit of magnitude |l| carries an
// absolute error of about eps = 1.2e-7 |l| (rms, measured: a head with 40-95 % of its mass on one token
// of logit 36 had its Z off by 2-3e-6), its exponential the same relative error.  Terms of weight w_i
// (share of Z) with independent errors put Z off by eps * sqrt(sum w_i^2) <= eps * sqrt(theta) if every
// term of weight >= theta is exact; theta = (1e-7 / eps)^2 keeps that at 1e-7, a third of what could
// move two group-sum scores past the 1e-6 that a kept set may differ by.  M, Z: the head's (estimated)
// maximum logit and sum of exp(l - M); returns the logit whose term has weight theta (+inf: no term
// qualifies).  The terms above it are few by construction: at most 1 / theta = 1.4 M^2 per head.
__host__ __device__ inline float heavy_logit_threshold(float M, float Z) {
  if (!(Z > 0.f) || !(M == M)) return INFINITY;
  const float mag = fabsf(M) > 4.f ? fabsf(M) : 4.f;
  const float r = 1e-7f / (1.2e-7f * mag);
  return M + logf(r * r * Z);
}

// ---- reductions over a workgroup of 16 waves ------------------------------------------------------
// The kernels that give a row to one workgroup are chains of these, and every instruction of a chain costs 4 cycles per wave of
// the SIMD, 7 ns with four: so the sixteen waves' parts are read by one LDS load, lane l taking wave l % 16's, and
// combined by DPP moves within rows of 16 lanes, in every wave alike, instead of sixteen loads and a second barrier.
template <int CTRL>
__device__ __forceinline__ int dpp_rot_i32(int v) {  // a permutation within rows of 16 lanes: every lane has a source
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <bool MAX>
__device__ __forceinline__ float combine(float a, float b) {
  return MAX ? fmaxf(a, b) : a + b;
}
// Over the lanes of a row of 16 whose numbers are equal modulo GQ (1, 2 or 4); every lane gets its own residue's result.
template <bool MAX, int GQ>
__device__ __forceinline__ float row_combine(float v) {
  v = combine<MAX>(v, dpp_f32<0x128>(v));               // row_ror:8
  v = combine<MAX>(v, dpp_f32<0x124>(v));               // row_ror:4
  if (GQ <= 2) v = combine<MAX>(v, dpp_f32<0x122>(v));  // row_ror:2
  if (GQ == 1) v = combine<MAX>(v, dpp_f32<0x121>(v));  // row_ror:1
  return v;
}
// The same over the whole wave.
template <bool MAX, int GQ>
__device__ __forceinline__ float wave_combine(float v) {
  v = row_combine<MAX, GQ>(v);
  return MAX ? swap32_max(swap16_max(v)) : swap32_sum(swap16_sum(v));
}

// ---- block-wide inclusive scan of one int per thread (1024 threads) ------------------------------
// `wave_tot` is 16 ints of shared memory that no thread reads any more from an earlier use (a barrier has come after that).
// Returns the inclusive prefix; *total gets the block sum.  One barrier.
__device__ __forceinline__ int block_scan_incl(int v, int* wave_tot, int* total) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int x = wave_scan_incl(v);
  if (lane == 63) wave_tot[w] = x;
  __syncthreads();
  int t = wave_tot[lane & 15];
  t += dpp_i32<0x111, 0xF>(0, t);  // row_shr: inclusive prefix over the 16 waves
  t += dpp_i32<0x112, 0xF>(0, t);
  t += dpp_i32<0x114, 0xF>(0, t);
  t += dpp_i32<0x118, 0xF>(0, t);
  *total = __builtin_amdgcn_readlane(t, 15);
  return x + (w > 0 ? __builtin_amdgcn_readlane(t, w - 1) : 0);
}

}  // namespace sagekv
