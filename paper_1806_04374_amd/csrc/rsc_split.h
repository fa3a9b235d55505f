// FP32 products on the BF16 matrix cores: both factors are split into three BF16 parts,
//   x = hi + mid + lo  (exact for a 24-bit significand),
// and the six products down to 2^-16 of the largest are accumulated in FP32,
//   hi hi, hi mid, mid hi, hi lo, lo hi, mid mid.
// The operand's parts are rounded (mid at most 2^-8 of it, lo 2^-17), the data's truncated (2^-7 and
// 2^-15), so the three dropped products add up to at most 2^-22 of |a||x| (2^-26.5 on average).  Six
// v_mfma_f32_32x32x16_bf16 take 192 cycles per 16 terms, eight v_mfma_f32_32x32x2f32 512, and the result
// is closer to the 64-bit one: at 15x15 the projection's relative error is 0.8e-7 against 2.3e-7 (a
// chain of 89 FP32 roundings).
//
// Operand layout of one 16-term step: lane l supplies terms 8 (l / 32) + i, i = 0..7, of row
// (or column) l % 32.
#pragma once

#include <hip/hip_runtime.h>

#include "rsc_device.h"
#include "rsc_lp.h"

namespace rsc {

// Eight values of a lane, split by truncation (hi never overflows, and the remainders are exact),
// each part packed into one operand register set.
__device__ __forceinline__ void split3(const float (&v)[8], uint4& hi, uint4& mid, uint4& lo) {
  unsigned h[8], m[8], l[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    h[i] = __float_as_uint(v[i]) & 0xffff0000u;
    const float r = v[i] - __uint_as_float(h[i]);
    m[i] = __float_as_uint(r) & 0xffff0000u;
    l[i] = __float_as_uint(r - __uint_as_float(m[i]));
  }
  // the high halves of two words in one register
  auto pack = [](unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); };
  hi = uint4{pack(h[0], h[1]), pack(h[2], h[3]), pack(h[4], h[5]), pack(h[6], h[7])};
  mid = uint4{pack(m[0], m[1]), pack(m[2], m[3]), pack(m[4], m[5]), pack(m[6], m[7])};
  lo = uint4{pack(l[0], l[1]), pack(l[2], l[3]), pack(l[4], l[5]), pack(l[6], l[7])};
}

// The parts hold every bit of a value only if its last part is a normal number: values below about
// 2^-110 lose low bits, and an infinite one leaves NaN remainders.  So each column (patch) of a
// chunk keeps its largest magnitude, and a chunk is done in plain FP32 where a column's is
// infinite, or so small that what its values lose (2^-126 at most) is more than 2^-26 of it.
__device__ __forceinline__ float largest(const float (&v)[8], float m) {
#pragma unroll
  for (int i = 0; i < 8; ++i) m = fmaxf(m, fabsf(v[i]));
  return m;
}
__device__ __forceinline__ bool needs_fp32(float largest) {
  return largest == __builtin_inff() || (largest > 0.f && largest < 0x1p-100f);
}

// Sum over NS steps of a[step] (three parts) times the operand in LDS, xb: [3][NS][64].  The five
// small products of every step are added first and the large ones last, so that the sum is
// rounded at its full size only NS times.  The next step's reads are issued before the current
// one's products; left alone the compiler reads all steps ahead into registers.
template <int NS>
__device__ __forceinline__ f32x16 contract_split3(const uint4 (&a)[NS][3], const uint4* __restrict__ xb, int lane) {
  auto v = [](const uint4& w) { return __builtin_bit_cast(bf16x8, w); };
  using P = Lp<RSC_BF16>;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  uint4 x[2][3];
#pragma unroll
  for (int q = 0; q < 3; ++q) x[0][q] = xb[q * NS * 64 + lane];
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    uint4 (&c)[3] = x[j % 2];
    uint4 (&n)[3] = x[(j + 1) % 2];
    if (j + 1 < NS) {
#pragma unroll
      for (int q = 0; q < 3; ++q) n[q] = xb[(q * NS + j + 1) * 64 + lane];
    } else {
      n[0] = xb[lane];
    }
    __builtin_amdgcn_sched_barrier(0);
    acc = P::mfma(v(a[j][1]), v(c[1]), acc);
    acc = P::mfma(v(a[j][2]), v(c[0]), acc);
    acc = P::mfma(v(a[j][0]), v(c[2]), acc);
    acc = P::mfma(v(a[j][1]), v(c[0]), acc);
    acc = P::mfma(v(a[j][0]), v(c[1]), acc);
    __builtin_amdgcn_sched_barrier(0);
  }
  uint4 h[2];
  h[0] = x[NS % 2][0];
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    if (j + 1 < NS) h[(j + 1) % 2] = xb[(j + 1) * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
    acc = P::mfma(v(a[j][0]), v(h[j % 2]), acc);
    __builtin_amdgcn_sched_barrier(0);
  }
  return acc;
}

// The lane's 16 rows of one column (32 x 32 result, rows 8 (v / 4) + 4 u + v % 4 from row0) to
// dst[row], rows below n: four 16-byte stores, which need no alignment and leave whole lines in
// L2 once the block's waves have written their rows.
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ void store_column(float* __restrict__ dst, const f32x16& acc, int row0, int u, int n) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int r = row0 + 8 * g + 4 * u;
    if (r + 3 < n) {
      *reinterpret_cast<v4f_any*>(dst + r) = v4f_any{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (r + i < n) dst[r + i] = acc[4 * g + i];
    }
  }
}

}  // namespace rsc
