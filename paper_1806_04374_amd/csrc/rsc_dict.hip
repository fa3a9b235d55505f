// The tables that depend on the dictionary, built on the device from its rows: the row tables
// of the encoders, their stage-1 operands and the per-pair harmonic inner products.
//
// One thread per table entry; the pair table (M^2 (2T+1) FP64 sums of S or 2S products) is
// nearly all of the work.  On the host it took 0.6 ms of a 15x15 upload at M = 100, against
// 0.02 ms here, and the upload shrinks from the tables (3 MB at M = 128) to the rows (54 KB).
// Sums run in the same order and without contraction, so every entry has the value that a
// plain host loop gives it.
#include <hip/hip_runtime.h>

#include "rsc_internal.h"
#include "rsc_screen.h"

namespace rsc {
namespace {

__device__ __forceinline__ uint16_t bf16_bits(float f) {
  const uint32_t v = __float_as_uint(f);   // finite: dictionary entries are checked
  return uint16_t((v + 0x7fffu + ((v >> 16) & 1u)) >> 16);
}

__device__ __forceinline__ uint16_t f16_bits(float f) { return __builtin_bit_cast(uint16_t, _Float16(f)); }

__global__ __launch_bounds__(256) void dict_tables_kernel(DictBuild p) {
#pragma clang fp contract(off)
  const int M = p.M, B = p.B, T = p.T, HQ = 2 * T + 1;
  const int64_t stride = int64_t(gridDim.x) * 256, i0 = int64_t(blockIdx.x) * 256 + threadIdx.x;
  auto D = [&](int m, int c) { return m < M ? p.rows[size_t(m) * B + c] : 0.f; };
  // <a, b> per harmonic: sum_s a_s b_s at k = 0, sum_s conj(a_s) b_s as (Re, Im) for k >= 1
  for (int64_t i = i0; i < int64_t(M) * M * (T + 1); i += stride) {
    const int k = int(i % (T + 1)), ab = int(i / (T + 1)), a = ab / M, b = ab - a * M;
    const int base = p.kbase[k], nk = p.sk[k];
    const float* ra = p.rows + size_t(a) * B + base;
    const float* rb = p.rows + size_t(b) * B + base;
    const size_t o = size_t(ab) * HQ;
    if (k == 0) {
      double h0 = 0.0;
      for (int s = 0; s < nk; ++s) h0 += double(ra[s]) * double(rb[s]);
      p.gramH64[o] = h0;
      p.gramH[o] = float(h0);
    } else {
      double re = 0.0, im = 0.0;
      for (int s = 0; s < nk; ++s) {
        const double ar = ra[s], ai = ra[nk + s], br = rb[s], bi = rb[nk + s];
        re += ar * br + ai * bi;
        im += ar * bi - ai * br;
      }
      p.gramH64[o + 2 * k - 1] = re;
      p.gramH64[o + 2 * k] = im;
      p.gramH[o + 2 * k - 1] = float(re);
      p.gramH[o + 2 * k] = float(im);
    }
  }
  // squared norms: the harmonics' own products, rounded and then added in FP32, which is what the
  // pair table gives an atom with itself
  for (int64_t m = i0; m < M; m += stride) {
    float n2 = 0.f;
    for (int k = 0; k <= T; ++k) {
      double h = 0.0;
      const float* r = p.rows + size_t(m) * B + p.kbase[k];
      const int nk = p.sk[k];
      for (int s = 0; s < nk; ++s) {
        const double a = r[s], b = k ? r[nk + s] : 0.0;
        h += a * a + b * b;
      }
      n2 = n2 + float(h);
    }
    p.norm2[m] = n2;
  }
  // rows padded with zero atoms, and i times them: per harmonic k >= 1 the (Re, Im) slots hold
  // (-Im d, Re d), zero at harmonic 0
  for (int64_t i = i0; i < int64_t(p.nrows) * B; i += stride) {
    const int m = int(i / B), c = int(i - int64_t(m) * B);
    p.hat[i] = D(m, c);
    if (p.hatI) {
      int k = 0;
      while (k < T && c >= p.kbase[k + 1]) ++k;
      const int nk = p.sk[k];
      p.hatI[i] = k == 0 ? 0.f : c - p.kbase[k] < nk ? -D(m, c + nk) : D(m, c - nk);
    }
  }
  // rows of the screened encoder: harmonic 0 padded to an even count, then (Re, Im) pairs
  if (p.pairs) {
    const int row = screen_row(B, p.sk[0]), s0 = p.sk[0] + p.sk[0] % 2;
    for (int64_t i = i0; i < int64_t(p.nrows) * row; i += stride) {
      const int m = int(i / row), e = int(i - int64_t(m) * row);
      float v = 0.f;
      if (e < s0) {
        if (e < p.sk[0]) v = D(m, e);
      } else if (e - s0 + p.sk[0] < B) {
        const int c = e - s0 + p.sk[0];        // the packed coordinate at this place
        int k = 1;
        while (k < T && c >= p.kbase[k + 1]) ++k;
        const int rem = c - p.kbase[k];
        v = D(m, p.kbase[k] + (rem % 2) * p.sk[k] + rem / 2);
      }
      p.pairs[i] = v;
    }
  }
  // 32x32 FP32 tiles, stage-1 operand: row 8i + j (j < 4) gives Re C_k of atom 16g + 4i + j and
  // row 8i + 4 + j its Im C_k, so that the accumulator register of an atom holds its Re C_k
  // in the low half-wave and its Im C_k in the high one; the two contraction lanes of a
  // step are (Re, Im) of one profile (k >= 1) or two consecutive profiles (k = 0, where
  // the Im rows are zero)
  if (p.dictA) {
    const int S = p.sk[0], K0 = (S + 1) / 2, NKS = K0 + T * S;
    for (int64_t i = i0; i < int64_t(p.nrows / 16) * NKS * 64; i += stride) {
      const int l = int(i % 64), ks = int(i / 64 % NKS), g = int(i / 64 / NKS);
      const int row = l % 32, hh = l / 32, m = 16 * g + 4 * (row / 8) + row % 4;
      const bool im_row = (row / 4) % 2 == 1;
      float v = 0.f;
      if (ks < K0) {
        const int s = 2 * ks + hh;
        if (!im_row && s < S) v = D(m, s);
      } else {
        const int q = ks - K0, k = 1 + q / S, s = q % S, base = p.kbase[k];
        const float re = D(m, base + s), im = D(m, base + S + s);
        v = im_row ? (hh == 0 ? -im : re) : (hh == 0 ? re : im);
      }
      p.dictA[i] = v;
    }
  }
  // screen, stage-1 operand (rsc_screen.h): lane l gives row l % 32 = (row pair 4(row/8) +
  // row%4, Re/Im = (row/4)%2) and contraction slots 8(l/32)..+7 of step j: the residual's
  // harmonic-j block, then (two operands) its harmonic-(j + 8) block, Re parts (k = 0: even
  // profiles) in the low half-wave, Im parts (k = 0: odd profiles) in the high one.  Row pair
  // v is atom v % AG of the group at harmonic j + 8 (v / AG).
  if (p.lpA) {
    const int AG = screen_group_atoms(T), NJ = screen_steps(T), NG = (M + AG - 1) / AG;
    for (int64_t i = i0; i < int64_t(NG) * NJ * 64 * 8; i += stride) {
      const int slot = int(i % 8), l = int(i / 8 % 64), j = int(i / 512 % NJ), g = int(i / 512 / NJ);
      const int row = l % 32, hh = l / 32, v = 4 * (row / 8) + row % 4, part = (row / 4) % 2;
      const int m = AG * g + v % AG, k = j + 8 * (v / AG);
      float val = 0.f;
      if (k <= T) {
        const int first = k == j ? 0 : (j == 0 ? (p.sk[0] + 1) / 2 : p.sk[j]);
        const int base = p.kbase[k], nk = p.sk[k], n = k == 0 ? (nk + 1) / 2 : nk, s = slot - first;
        if (s >= 0 && s < n) {
          if (k == 0) {
            if (part == 0 && 2 * s + hh < nk) val = D(m, 2 * s + hh);
          } else {
            const float re = D(m, base + s), im = D(m, base + nk + s);
            val = part == 0 ? (hh == 0 ? re : im) : (hh == 0 ? -im : re);
          }
        }
      }
      p.lpA[i] = p.bf16 ? bf16_bits(val) : f16_bits(val);
    }
  }
}

}  // namespace

int launch_dict_tables(const DictBuild& p, void* stream) {
  const int64_t work = int64_t(p.M) * p.M * (p.T + 1);
  const int64_t blocks = (work + 255) / 256;
  hipLaunchKernelGGL(dict_tables_kernel, dim3(unsigned(blocks < 1 ? 1 : blocks > 1024 ? 1024 : blocks)), dim3(256), 0,
                     reinterpret_cast<hipStream_t>(stream), p);
  return int(hipGetLastError());
}

}  // namespace rsc
