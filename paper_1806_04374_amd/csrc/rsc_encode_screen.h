// Rotational OMP with a 16-bit screen and FP32 selection (Fig. 2 with rotations replaced by
// steering: Sec. II-C, eq. (8); Sec. II-E step 3).
//
// Each wave owns 32 patches (MFMA columns).  Per pursuit step:
//   screen, v_mfma_f32_32x32x16_{f16,bf16}: stage 1 forms C_k = sum_s conj(d_{m,s,k}) x_{s,k}
//     of a group of atoms (rsc_screen.h), stage 2 the angle DFT per atom and 32 angles.  Only
//     the largest |score| of each atom over its angles is kept, and from it which atoms are
//     candidates: those within 8.5u ||r|| of the largest one (u: unit roundoff of the format).
//     Per harmonic k, rounding the atom and the residual moves C_k by at most (2u + u^2)
//     sum_s |d_{k,s}| |x_{k,s}| (complex magnitudes), and rounding the stage-2 operand C_k and
//     (cos, -sin) moves the term cos Re C_k - sin Im C_k by at most (2u + u^2) |C_k|
//     (Cauchy-Schwarz on the 2-vectors).  Summed over k with unit-norm atoms (Cauchy-Schwarz
//     again), a 16-bit score is within (2u + u^2)(1 + (1 + u)^2) ||r|| = 4.02u ||r|| (BF16;
//     less for FP16) of the exact one; FP32 accumulation adds below 1e-3 of that.  So the
//     atom with the exact maximum lies within twice that (8.05u ||r||) of the largest 16-bit
//     maximum, and the window keeps it.  FP16 residuals are first scaled by a power of two to
//     a norm in [0.5, 1), which keeps every coordinate that matters out of the subnormal
//     range; a residual too small for its norm to be exact to a few percent takes every atom.
//   selection in FP32: every candidate's scores are formed in FP32 (C_k from the packed
//     dictionary, the angle DFT on v_mfma_f32_32x32x2f32), and the atom and angle of the
//     largest one win; equal maxima go to the smaller atom, then the smaller angle.  The
//     screen only leaves out atoms that cannot win, so the selection is the one that FP32
//     scores of every atom give.
//   BF16 filter: a BF16 window holds several atoms per step, and a wave loops over its patches'
//     largest candidate count.  So the atom with the largest 16-bit maximum is scored first, and
//     of the others only those are kept whose 16-bit maximum reaches its FP32 maximum minus the
//     error bound (4.02u ||r||, taken as 4.25u): the atom with the largest FP32 maximum E has a
//     16-bit maximum of at least E - 4.02u ||r||, and E is at least the first one's.  The 16-bit
//     maxima are kept for this as FP16 fractions of ||r|| in private memory, which is read only
//     for candidates, with a margin of 2^-10 for their rounding.  FP16's window holds about one
//     atom, and the bookkeeping would cost more than it saves.
//   least squares and residual update in FP32 (ls_step), as in the FP32 encoders.
//
// FP32 handles (FULL) get the codes of the full form that they would run without a screen, bit for
// bit, so that no patch depends on which form coded it.  v_mfma_f32_32x32x2f32 and _16x16x4f32 add
// their terms one after the other, each rounded as an fmaf (checked over 384,000 results with
// exponents up to 2^100 apart), so the full form's sums can be formed here:
//   second pass: C_k and the residual norms summed as the full form's lanes hold the coordinates
//     (W = 2: the 32x32 tile; W = 4, the 16x16 tile: even and odd profiles apart), the angle DFT with its
//     parity split.  All candidates are scored like this, so the winner's angle and correlation are
//     the full form's, and with ls_step's sums so are the coefficients and the residual.
//   first pass, which chooses the atom: C_k as one chain over (Re, Im) of one profile after the
//     other, the order of the stage-1 instructions in both tiles.  Where the two largest maxima are
//     further apart than the rounding of both passes (tie_window) both choose the same atom; otherwise
//     the patch's candidates are scored once more in this order.  Of random patches about one step
//     in a thousand needs that; where atoms coincide every step does, and pays for one more scoring of
//     its candidates: with every atom twice in the dictionary 10^6 11x11 patches (M = 64, K = 4) take 1.50
//     ms against 1.07 with distinct atoms and 3.39 in the full form.  A dictionary whose atoms all
//     agree to 1e-6 leaves the screen nothing to leave out (9.5 ms).  (Rounds of one loop in place of
//     a second copy of the scoring code are 1 to 6% slower.)
//
// What bounds it: vector issue.  A wave's maxima over 64 angles cost 16 three-way maxima per
// atom for 32 patches, and the 16-bit products take as many cycles on the matrix cores, so
// two waves per SIMD hide one behind the other as far as registers allow: the least-squares
// state waits in LDS while the screen runs, which is what brings the kernel to 256 registers.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "rsc_device.h"
#include "rsc_internal.h"
#include "rsc_launch.h"
#include "rsc_lp.h"
#include "rsc_screen.h"

namespace rsc {
namespace screen {

struct ScreenParams {
  const float* xhat;
  int64_t P;
  int K, M, R;
  const uint4* dictA;      // stage-1 operand [NG][NJ][64] x 8 16-bit values
  const float* pairs;      // [>= NG AG][screen_row] dictionary rows (rsc_screen.h)
  const float* dictHat;    // [>= M][B] (the FP64 re-solve)
  const uint4* dft16;      // stage-2 operand [OPS][RT][64] x 8 16-bit values
  const float* dft32;      // FP32 angle DFT [FT][NQ][64]
  const float* cs;         // [2][NQ][R]
  const float* gramH;      // [M][M][2T+1]
  const float* norm2;      // [M] squared norms of the atoms
  const double* gramH64;   // [M][M][2T+1]
  const double* cs64;      // [2][NQ][R]
  int32_t* atom;
  int32_t* angle;
  float* coef;
  float* resid2;
  unsigned long long* stats;   // [4], see rsc_precision_stats
  float cond_max;              // least squares in FP64 beyond this bound (ls_update)
  bool count;                  // whether candidates are counted (16-bit handles)
  int32_t* label;              // not null: no codes; each patch keeps the smaller of sse and its squared
  float* sse;                  // residual norm, and class cls with it where that is the smaller (class 0
  int cls;                     // always), as classify_min_kernel
};

// The least-squares state of the wave's 32 patches in LDS: float4 q of patch col at
// mem[q * 32 + col].  Both half-waves hold the same values; the low one writes.
template <int KMAX>
struct StateIo {
  static constexpr int N4 = screen_state_f4(KMAX), NF = KMAX * (KMAX - 1) / 2 + 3 * KMAX;
  template <class F>
  __device__ __forceinline__ static void each(PursuitState<KMAX>& st, LsState<KMAX>& ls, F f) {
    int n = 0;
#pragma unroll
    for (int i = 0; i < KMAX; ++i)
#pragma unroll
      for (int j = 0; j < i; ++j) f(n++, st.L[i][j]);
#pragma unroll
    for (int i = 0; i < KMAX; ++i) f(n++, ls.Ld[i]);
#pragma unroll
    for (int i = 0; i < KMAX; ++i) f(n++, st.bv[i]);
#pragma unroll
    for (int i = 0; i < KMAX; ++i) f(n++, st.cf[i]);
  }
  __device__ __forceinline__ static void save(float4* mem, int lane, PursuitState<KMAX>& st, LsState<KMAX>& ls) {
    float v[4 * N4];
    zero(v);
    each(st, ls, [&](int n, float& x) { v[n] = x; });
    // selections as 16-bit words: atom << 6 | angle (M <= 128, R <= 64), -1 for an empty slot
#pragma unroll
    for (int i = 0; i < KMAX; i += 2) {
      const int a = st.selm[i] < 0 ? -1 : st.selm[i] << 6 | st.selr[i];
      const int b = i + 1 >= KMAX || st.selm[i + 1 < KMAX ? i + 1 : i] < 0
                        ? -1 : st.selm[i + 1 < KMAX ? i + 1 : i] << 6 | st.selr[i + 1 < KMAX ? i + 1 : i];
      v[NF + i / 2] = __int_as_float((a & 0xffff) | b << 16);
    }
    if (lane < 32) {
#pragma unroll
      for (int q = 0; q < N4; ++q) mem[q * 32 + lane] = float4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
    }
  }
  __device__ __forceinline__ static void load(const float4* mem, int col, PursuitState<KMAX>& st, LsState<KMAX>& ls) {
    float v[4 * N4];
#pragma unroll
    for (int q = 0; q < N4; ++q) {
      const float4 w = mem[q * 32 + col];
      v[4 * q] = w.x;
      v[4 * q + 1] = w.y;
      v[4 * q + 2] = w.z;
      v[4 * q + 3] = w.w;
    }
    each(st, ls, [&](int n, float& x) { x = v[n]; });
#pragma unroll
    for (int i = 0; i < KMAX; ++i) {
      const int w = __float_as_int(v[NF + i / 2]), z = i % 2 ? w >> 16 : w << 16 >> 16;
      st.selm[i] = z >> 6;
      st.selr[i] = z < 0 ? -1 : z & 63;
    }
  }
};

// Orders the low half-wave's LDS writes before the whole wave's reads: neither the compiler (which
// sees a conditional store and a load of one thread) nor the hardware moves one past the other.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// A dictionary row (rsc_screen.h) goes through registers in batches of whole harmonics of up to
// kRowPairs pairs, the next batch's LDS reads issued before the current one is used.  Left to
// itself the compiler waits for every read or two, and the reads' latency, not their number,
// was most of a step outside the screen.
constexpr int kRowPairs = 16;
template <class L>
struct RowBatches {
  __host__ __device__ static constexpr int next(int k) {     // first harmonic of the batch after k's
    int n = L::Sk(k), q = k + 1;
    while (q <= L::T && n + L::Sk(q) <= kRowPairs) n += L::Sk(q++);
    return q;
  }
  __host__ __device__ static constexpr int first(int b) {    // first harmonic of batch b
    int k = 1;
    for (int i = 0; i < b && k <= L::T; ++i) k = next(k);
    return k;
  }
  __host__ __device__ static constexpr int count() {
    int b = 0;
    for (int k = 1; k <= L::T; k = next(k)) ++b;
    return b;
  }
  // index of harmonic k's first pair within the row's pairs, and the floats before the pairs
  __host__ __device__ static constexpr int pair0(int k) { return (L::base(k) - L::Sk(0)) / 2; }
  static constexpr int S0 = 2 * L::J0;
  // f(k, i, x, y) for every profile i of every harmonic k >= 1, g(k) after each harmonic.  (x, y):
  // the pair (Re, Im), one 8-byte read; with OWN the part that the lane's half-wave holds (u = 0:
  // Re, 1: Im) and the other one
  template <bool OWN, class F, class G>
  __device__ __forceinline__ static void each(const float* __restrict__ row, int u, F f, G g) {
    const float *px = row + S0 + (OWN ? u : 0), *py = row + S0 + (OWN ? 1 - u : 1);
    float x[2][kRowPairs], y[2][kRowPairs];
    auto fetch = [&](auto B1) {
      constexpr int b = decltype(B1)::value, lo = pair0(first(b)), hi = pair0(first(b + 1) <= L::T ? first(b + 1) : L::T + 1);
#pragma unroll
      for (int i = lo; i < hi; ++i) {
        if constexpr (OWN) {
          x[b % 2][i - lo] = px[2 * i];
          y[b % 2][i - lo] = py[2 * i];
        } else {
          const float2 d = reinterpret_cast<const float2*>(px)[i];
          x[b % 2][i - lo] = d.x;
          y[b % 2][i - lo] = d.y;
        }
      }
    };
    fetch(std::integral_constant<int, 0>{});
    static_for<count()>([&](auto B1) {
      constexpr int b = decltype(B1)::value, k0 = first(b), k1 = b + 1 < count() ? first(b + 1) : L::T + 1;
      if constexpr (b + 1 < count()) fetch(std::integral_constant<int, b + 1>{});
      __builtin_amdgcn_sched_barrier(0);
      static_for<k1 - k0>([&](auto K1) {
        constexpr int k = k0 + decltype(K1)::value;
        static_for<L::Sk(k)>([&](auto I) {
          constexpr int i = decltype(I)::value, j = pair0(k) - pair0(k0) + i;
          f(std::integral_constant<int, k>{}, std::integral_constant<int, i>{}, x[b % 2][j], y[b % 2][j]);
        });
        g(std::integral_constant<int, k>{});
      });
      __builtin_amdgcn_sched_barrier(0);
    });
  }
};

// C_k = sum_s conj(d_{m,s,k}) x_{s,k} of the atom in `row` for this lane's patch: op[k] = Re C_k in
// the low half-wave and Im C_k in the high one, on a row of pairs.  Each half-wave multiplies its
// residual coordinates (Re parts low, Im parts high) with both parts of the atom, and one swap per
// harmonic adds the halves' sums: the order of atom_operand.  W = 4: even and odd profiles are
// summed apart, the order of atom_products4.
template <class L, int W>
__device__ __forceinline__ void row_operand(const float* __restrict__ row, int u, const float (&res)[L::NKS],
                                            float (&op)[L::NQ]) {
  float d0[L::J0];
#pragma unroll
  for (int j = 0; j < L::J0; ++j) d0[j] = row[2 * j + u];
  constexpr int NC = W / 2;                          // chains per sum
  float pr[NC][L::NQ], pi[NC][L::NQ];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    zero(pr[c]);
    zero(pi[c]);
  }
  RowBatches<L>::template each<false>(row, u, [&](auto K1, auto I, float re, float im) {
    constexpr int k = decltype(K1)::value, j = L::joff(k) + decltype(I)::value, c = decltype(I)::value % NC;
    pr[c][k] = fmaf(re, res[j], pr[c][k]);
    pi[c][k] = fmaf(im, res[j], pi[c][k]);
  }, [&](auto K1) {
    // low (Re x): Re += dRe x, Im -= dIm x; high (Im x): Re += dIm x, Im += dRe x
    constexpr int k = decltype(K1)::value;
#pragma unroll
    for (int c = 0; c < NC && c < L::Sk(k); ++c) {
      float x = u ? pi[c][k] : pr[c][k], y = u ? pr[c][k] : -pi[c][k];
      swap32(x, y);
      op[k] = c == 0 ? x + y : op[k] + (x + y);
    }
  });
#pragma unroll
  for (int c = 0; c < NC && c < L::J0; ++c) {
    float x = 0.f, y = 0.f;
#pragma unroll
    for (int j = c; j < L::J0; j += NC) x = fmaf(d0[j], res[j], x);
    swap32(x, y);
    op[0] = c == 0 ? x + y : op[0] + (x + y);
  }
}

// The same C_k in the order of the full form's first pass: one chain over the profiles, each
// profile's product with Re x before the one with Im x (harmonic 0: one chain over the profiles).
template <class L>
__device__ __forceinline__ void chain_operand(const float* __restrict__ row, int u, const float (&res)[L::NKS],
                                              float (&op)[L::NQ]) {
  zero(op);
#pragma unroll
  for (int j = 0; j < L::J0; ++j) {
    float x = res[j], y = res[j];
    swap32(x, y);                                    // profiles 2j and 2j + 1, in both half-waves
    op[0] = fmaf(row[2 * j + 1], y, fmaf(row[2 * j], x, op[0]));
  }
  op[0] = u ? 0.f : op[0];
  RowBatches<L>::template each<true>(row, u, [&](auto K1, auto I, float own, float oth) {
    constexpr int k = decltype(K1)::value, j = L::joff(k) + decltype(I)::value;
    float x = res[j], y = res[j];
    swap32(x, y);                                    // Re x and Im x
    // Re C: dRe Re x, then dIm Im x; Im C: -dIm Re x, then dRe Im x
    op[k] = fmaf(oth, y, fmaf(u ? -own : own, x, op[k]));
  }, [](auto) {});
}

// acc += alpha S_r d for the atom in `row` on this lane's coordinates; cs: (cos, sin) of this
// angle per harmonic.  Re' = c Re + s Im, Im' = c Im - s Re: the product with the other part of a
// pair is added first and the one with the lane's own part last, as in steer_axpy, so that the
// residual is rounded as there (Re first in both half-waves saves the half-waves' own addresses
// and nothing measurable: 0 to 1% of an encode; reading the pairs whole and selecting the parts
// costs 1 to 3%).
template <class L>
__device__ __forceinline__ void row_axpy(float (&acc)[L::NKS], float alpha, const float* __restrict__ row,
                                         const float2* __restrict__ cs, int u) {
  float d0[L::J0];
#pragma unroll
  for (int j = 0; j < L::J0; ++j) d0[j] = row[2 * j + u];
  float2 w[L::NQ];
#pragma unroll
  for (int k = 1; k < L::NQ; ++k) w[k] = cs[k];
  float c = 0.f, s = 0.f;
  RowBatches<L>::template each<true>(row, u, [&](auto K1, auto I, float own, float oth) {
    constexpr int k = decltype(K1)::value, i = decltype(I)::value, j = L::joff(k) + i;
    if constexpr (i == 0) {
      c = alpha * w[k].x;
      s = (u ? -alpha : alpha) * w[k].y;
    }
    acc[j] = fmaf(own, c, fmaf(oth, s, acc[j]));
  }, [](auto) {});
#pragma unroll
  for (int j = 0; j < L::J0; ++j) acc[j] = fmaf(alpha, d0[j], acc[j]);
}

// The least-squares step of ls_update (same formulas and thresholds) with what it indexes by
// slot at run time kept in the wave's LDS, `mem`: one copy of the code steers every selected
// column, instead of one per slot, and the half-waves share the pair products (slot 2i + u).
template <class L, int KMAX, int W>
__device__ __forceinline__ bool ls_step(PursuitState<KMAX>& st, LsState<KMAX>& ls, int it, int ms, int rs, float cval,
                                        const float* pairs, int row, const float2* cs, const LsTables& tb,
                                        const float* norm2, const float* hat, int64_t p, int u, int col, float* mem,
                                        float (&res)[L::NKS]) {
  constexpr int T = L::T, HQ = 2 * T + 1, AS = screen_angle_stride(T);
  const int M = tb.M, R = tb.R;
  const float dd = norm2[ms];
  int* sel = reinterpret_cast<int*>(mem) + col;      // [KMAX] x 32: atom << 6 | angle of slot i
  float* val = mem + KMAX * 32 + col;                // [KMAX] x 32: pair product, then coefficient change
  bool dup = false;
#pragma unroll
  for (int i = 0; i < KMAX; ++i) {
    dup = dup || (i < it && st.selm[i] == ms && st.selr[i] == rs);
    const int z = st.selm[i] < 0 ? 0 : st.selm[i] << 6 | st.selr[i];
    if (u == 0) sel[i * 32] = i == it ? ms << 6 | rs : z;
  }
  const bool upd = st.active && !dup;
  wave_lds_order();
  // <column i, new column> for i < it
  for (int i0 = 0; i0 < it; i0 += 2) {
    const int i = i0 + u < it ? i0 + u : i0;
    const int z = sel[i * 32], a = z >> 6;
    int dr = (z & 63) - rs;
    dr += dr < 0 ? R : 0;
    const float* h = tb.gramH + (size_t(a) * M + ms) * HQ;
    float hv[HQ];
#pragma unroll
    for (int k = 0; k < HQ; ++k) hv[k] = h[k];
    const float2* w = cs + dr * AS;
    float g = hv[0];
#pragma unroll
    for (int k = 1; k <= T; ++k) g += w[k].x * hv[2 * k - 1] - w[k].y * hv[2 * k];
    val[i * 32] = g;
  }
  wave_lds_order();
  float gcol[KMAX];
  float bx = cval;
#pragma unroll
  for (int i = 0; i < KMAX; ++i) {
    gcol[i] = i < it ? val[i * 32] : 0.f;
    bx += gcol[i] * st.cf[i];
  }
  float w[KMAX];
  float l2 = dd;
#pragma unroll
  for (int i = 0; i < KMAX; ++i) {
    float s = gcol[i];
#pragma unroll
    for (int j = 0; j < i; ++j) s -= st.L[i][j] * w[j];
    w[i] = i < it ? s * ls.Ld[i] : 0.f;
    l2 -= w[i] * w[i];
  }
  // new row of L^{-1}: [-(L^{-T} w)^T, 1] / l, so ||L^{-1}||_F^2 grows by (|L^{-T} w|^2 + 1) / l^2
  float z[KMAX];
  float zz = 0.f;
#pragma unroll
  for (int i = KMAX - 1; i >= 0; --i) {
    float s = w[i];
#pragma unroll
    for (int j = i + 1; j < KMAX; ++j) s -= (j < it ? st.L[j][i] : 0.f) * z[j];
    z[i] = i < it ? s * ls.Ld[i] : 0.f;
    zz += z[i] * z[i];
  }
  const float Fn = ls.condF + (zz + 1.f) / fmaxf(l2, 1e-30f);
  const bool ok32 = !ls.fp64 && l2 > 1e-6f * dd && float(it + 1) * Fn <= tb.cond_max;
  const bool up32 = upd && ok32;
  const bool go64 = upd && !ok32;
#pragma unroll
  for (int r = 0; r < KMAX; ++r) {
    const bool here = up32 && r == it;
#pragma unroll
    for (int i = 0; i < r; ++i) st.L[r][i] = here ? w[i] : st.L[r][i];
    ls.Ld[r] = here ? rsqrtf(l2) : ls.Ld[r];
    st.bv[r] = here ? bx : st.bv[r];
    st.selm[r] = here ? ms : st.selm[r];
    st.selr[r] = here ? rs : st.selr[r];
  }
  float y[KMAX], an[KMAX];
#pragma unroll
  for (int i = 0; i < KMAX; ++i) {
    float s = st.bv[i];
#pragma unroll
    for (int j = 0; j < i; ++j) s -= st.L[i][j] * y[j];
    y[i] = i <= it ? s * ls.Ld[i] : 0.f;
  }
#pragma unroll
  for (int i = KMAX - 1; i >= 0; --i) {
    float s = y[i];
#pragma unroll
    for (int j = i + 1; j < KMAX; ++j) s -= st.L[j][i] * an[j];
    an[i] = i <= it ? s * ls.Ld[i] : 0.f;
  }
  if (__any(up32)) {
    wave_lds_order();                                // the pair products have been read
#pragma unroll
    for (int i = 0; i < KMAX; ++i)
      if (u == 0) val[i * 32] = up32 && i <= it ? st.cf[i] - an[i] : 0.f;
    wave_lds_order();
#pragma unroll 1
    for (int i = 0; i <= it; ++i) {
      const int zi = sel[i * 32];
      row_axpy<L>(res, val[i * 32], pairs + (zi >> 6) * row, cs + (zi & 63) * AS, u);
    }
  }
#pragma unroll
  for (int i = 0; i < KMAX; ++i) st.cf[i] = (up32 && i <= it) ? an[i] : st.cf[i];
  ls.condF = up32 ? Fn : ls.condF;
  bool ok64 = false;
  if (__any(go64)) ok64 = ls_solve64<L, KMAX, W>(st, it, ms, rs, go64, hat, tb, p, u, res);
  ls.fp64 = ls.fp64 || ok64;
  st.nsel = (up32 || ok64) ? it + 1 : st.nsel;
  st.active = up32 || ok64;
  return go64;
}

// A patch's coordinates x [B] into the registers of its two lanes (W = 2): register j of
// harmonic k >= 1 reads the Re part in the low half-wave and the Im part, Sk(k) further on, in
// the high one, so each harmonic costs one address and constant offsets.  A padding register
// of harmonic 0 reads the value that follows, harmonic 1's first, and is set to 0.
template <class L>
__device__ __forceinline__ void load_hat(const float* __restrict__ x, int u, bool valid, float (&res)[L::NKS]) {
  static_assert(L::W == 2 && L::T >= 1, "two half-waves per patch");
#pragma unroll
  for (int j = 0; j < L::J0; ++j) res[j] = x[2 * j + u];
  static_for<L::T>([&](auto K1) {
    constexpr int k = decltype(K1)::value + 1;
    const float* xk = x + (u ? L::Sk(k) : 0);
#pragma unroll
    for (int i = 0; i < L::Sk(k); ++i) res[L::joff(k) + i] = xk[L::base(k) + i];
  });
  if (L::Sk(0) % 2 == 1) res[L::J0 - 1] = u ? 0.f : res[L::J0 - 1];
#pragma unroll
  for (int j = 0; j < L::NKS; ++j) res[j] = valid ? res[j] : 0.f;
}

// Bytes of the tables that a block keeps in LDS, rounded up to 16.
__host__ __device__ constexpr size_t screen_table_bytes(int NG, int NJ, int NQ, int rows, int row, int R, int FT) {
  return size_t(NG) * NJ * 1024 + ((sizeof(float) * (size_t(rows) * row + 2 * size_t(NQ | 1) * R + size_t(FT) * NQ * 64) + 15) & ~size_t(15));
}

// How far, in units of ||r||, the largest maximum of one pass can lie below the other pass's and still
// win there: twice what the passes can differ by in one score.  With u = 2^-24 and a_k = sum_s |d_s|
// |r_s| over harmonic k, the parts of C_k are rounded at most 2S times in the first pass and S + 2 times
// in the second, each by u a_k, and the angle DFT rounds each |C_k| <= a_k at most T + 3 times with
// the parity split and 2T + 2 without, in either pass.  The a_k add up to at most ||d|| ||r||, and
// |cos| + |sin| to sqrt(2).  (4u more for the norm and higher orders: 84u at 11x11, 109u at 15x15.)
constexpr float tie_window(int S, int T, bool split) {
  return (2 * (1.4143f * (3 * S + 2) + 2 * (split ? T + 3 : 2 * T + 2)) + 4) * 0x1p-24f;
}

// RT: 32-angle tiles of the screen (ceil(R / 32)).  SPLIT: the FP32 scores use the radix-2
// angle split (even R, R/2 <= 32 rows: E from even harmonics, O from odd ones, score(r) = E + O
// and score(r + R/2) = E - O); otherwise RT tiles of the direct angle DFT.  W, FULL: the order of
// the FP32 sums (above).
template <class C, int KMAX, int PREC, int RT, bool SPLIT, int W, bool FULL>
__global__ __launch_bounds__(512, 2) void encode_screen_kernel(ScreenParams prm) {
  using L = LayoutBase<C, 2>;
  using P = Lp<PREC>;
  using V8 = typename P::V8;
  constexpr int NKS = L::NKS, NQ = L::NQ, B = L::B, J0 = L::J0, T = L::T;
  constexpr int OPS = screen_ops(T), AG = screen_group_atoms(T), NJ = screen_steps(T), HA = AG / 2;
  constexpr int FT = SPLIT ? 1 : RT;
  static_assert(NQ <= 16, "two stage-2 operands hold 16 harmonics");
  extern __shared__ uint4 lds4[];
  const int R = prm.R, M = prm.M, K = prm.K, NG = (M + AG - 1) / AG, rows = NG * AG;
  const V8* sA = reinterpret_cast<const V8*>(lds4);             // [NG][NJ][64]
  constexpr int RB = screen_row(B, L::Sk(0)), AS = screen_angle_stride(T);
  float* sHat = reinterpret_cast<float*>(lds4 + NG * NJ * 64);  // [rows][RB]
  float2* sCs = reinterpret_cast<float2*>(sHat + rows * RB);    // [R][AS] (cos, sin)
  float* sF = reinterpret_cast<float*>(sCs + AS * R);           // [FT][NQ][64]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = int(blockDim.x) >> 6;
  float4* sState = reinterpret_cast<float4*>(reinterpret_cast<char*>(lds4) + screen_table_bytes(NG, NJ, NQ, rows, RB, R, FT)) +
                   wave * (StateIo<KMAX>::N4 * 32);
  {
    const int nA = NG * NJ * 64, nH = rows * RB, nC = NQ * R, nF = FT * NQ * 64;
    for (int i = threadIdx.x; i < nA; i += blockDim.x) lds4[i] = prm.dictA[i];
    for (int i = threadIdx.x; i < nH; i += blockDim.x) sHat[i] = prm.pairs[i];
    for (int i = threadIdx.x; i < nC; i += blockDim.x) {
      const int r = i / NQ, k = i - r * NQ;
      sCs[r * AS + k] = float2{prm.cs[k * R + r], prm.cs[(NQ + k) * R + r]};
    }
    for (int i = threadIdx.x; i < nF; i += blockDim.x) sF[i] = prm.dft32[i];
  }
  __syncthreads();

  const int col = lane & 31, u = lane >> 5;
  V8 F16[OPS][RT];
#pragma unroll
  for (int o = 0; o < OPS; ++o)
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const uint4 w = prm.dft16[(o * RT + t) * 64 + lane];
      __builtin_memcpy(&F16[o][t], &w, sizeof(w));
    }
  const LsTables tb{prm.gramH, prm.gramH64, prm.cs64, prm.xhat, M, R, prm.cond_max};
  constexpr float wfac = 8.5f * P::unit;
  constexpr bool kFilter = PREC == RSC_BF16;
  constexpr float efac = 4.25f * P::unit + 0x1p-10f;
  static_assert(!kFilter || HA == 8, "the filter keeps 8 maxima per lane and group");
  constexpr float ktie = tie_window(L::S, T, SPLIT);
  static_assert(!kFilter || !FULL, "the full form's atoms are compared in increasing order");
  uint4 vmax[kFilter ? 8 : 1];   // [groups] 8 FP16 fractions: this lane's maxima of the step
  unsigned n_sel = 0, n_cand = 0, n_fp64 = 0, max_cand = 0;

  // tiles go to the blocks first and then to their waves, so that a launch of few tiles
  // spreads over the CUs
  const int64_t nwt = (prm.P + 31) / 32;
  for (int64_t wt = int64_t(blockIdx.x) + int64_t(gridDim.x) * wave; wt < nwt; wt += int64_t(gridDim.x) * nw) {
    const int64_t p = wt * 32 + col;
    const bool valid = p < prm.P;
    float res[NKS];
    load_hat<L>(prm.xhat + (valid ? p : prm.P - 1) * B, u, valid, res);
    const float nx2 = norm2<L, W>(res);
    PursuitState<KMAX> st;
    init_state(st, valid);
    LsState<KMAX> ls;
    init_ls(ls);

    for (int it = 0; it < K; ++it) {
      const float n2 = norm2<L, W>(res);
      st.active = st.active && (n2 > kTau2 * nx2);
      if (!__any(st.active)) break;
      StateIo<KMAX>::save(sState, lane, st, ls);
      wave_lds_order();

      // ---------------- 16-bit residual operand, one per stage-1 step (FP16: the residual
      // scaled by 2^-e, ||r|| = f 2^e with f in [0.5, 1); the scores and the window are
      // compared in the scaled units)
      const float rn = sqrtf(n2);
      int ex = 0;
      if (PREC == RSC_FP16) (void)frexpf(rn, &ex);
      const float sc = PREC == RSC_FP16 ? ldexpf(1.f, -ex) : 1.f;
      V8 r16[NJ];
      static_for<NJ>([&](auto J) {
        constexpr int k = decltype(J)::value;
        constexpr int c0 = k == 0 ? J0 : L::Sk(k);
        constexpr int k2 = k + 8 < NQ ? k + 8 : 0, c1 = k + 8 < NQ ? L::Sk(k2) : 0;
        static_assert(c0 + c1 <= 8, "a step's profiles must fit one half-wave's 8 slots");
        float v[8];
        zero(v);
#pragma unroll
        for (int i = 0; i < c0; ++i) v[i] = sc * res[L::joff(k) + i];
#pragma unroll
        for (int i = 0; i < c1; ++i) v[c0 + i] = sc * res[L::joff(k2) + i];
        r16[k] = pack8<P>(v);
      });
      // below 1e-30 the squared norm is itself inexact: every atom is then a candidate
      const float wnd = n2 > 1e-30f ? wfac * rn * sc : 1e30f;

      // ---------------- 16-bit scores: per-atom maxima and the candidate mask
      float vh = -1.f;          // running maximum over this half-wave's atoms
      int va = 0;               // its atom (the first one on equal maxima; with the filter)
      const float invn = rn > 0.f ? 1.f / (rn * sc) : 0.f;
      uint64_t mask = 0;        // bit i: atom 2i + u is a candidate
      for (int g = 0; g < NG; ++g) {
        asm volatile("" ::: "memory");
        const V8* Ag = sA + g * NJ * 64 + lane;
        // stage 1 by pairs of steps; each pair is rounded at once into one 32-bit register
        // (two 16-bit slots) of every row pair's stage-2 operand
        u32x4 opk[16];
        f32x16 zro;
#pragma unroll
        for (int i = 0; i < 16; ++i) zro[i] = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int k0 = 2 * j, k1 = 2 * j + 1;
          if (k0 >= NJ) {
#pragma unroll
            for (int a = 0; a < 16; ++a) opk[a][j] = 0u;
            continue;
          }
          const f32x16 a0 = P::mfma(Ag[k0 * 64], r16[k0], zro);
          const f32x16 a1 = k1 < NJ ? P::mfma(Ag[(k1 < NJ ? k1 : k0) * 64], r16[k1 < NJ ? k1 : k0], zro) : zro;
#pragma unroll
          for (int a = 0; a < 16; ++a) opk[a][j] = pack2<P>(a0[a], a1[a]);
          // with one angle tile the scheduler would keep all eight accumulators (128 registers)
          if (RT == 1) __builtin_amdgcn_sched_barrier(0);
        }
        const int ab = AG * g;
        // stage 2 by (atom, angle tile) units, one unit in flight: the next unit's
        // products are issued before the current one's reduction
        auto issue = [&](int q) {
          const int a = q / RT, t = q % RT;
          f32x16 s = P::mfma(F16[0][t], __builtin_bit_cast(V8, opk[a]), zro);
          if constexpr (OPS == 2) s = P::mfma(F16[OPS - 1][t], __builtin_bit_cast(V8, opk[(a + 8) % 16]), s);
          return s;
        };
        float vs[HA];         // slot i: maximum of atom ab + 2i + u over its angles
        f32x16 cur = issue(0);
        float part = 0.f, mprev = 0.f;
#pragma unroll
        for (int q = 0; q < AG * RT; ++q) {
          const int a = q / RT, t = q % RT;
          f32x16 nxt;
          if (q + 1 < AG * RT) nxt = issue(q + 1);
          if (t == 0) part = 0.f;
#pragma unroll
          for (int i = 0; i < 16; i += 2) part = fmaxf(fmaxf(part, fabsf(cur[i])), fabsf(cur[i + 1]));
          if (t == RT - 1) {
            if (a % 2 == 0) {
              mprev = part;
            } else {
              // atoms a-1 and a completed across the half-waves: atom ab + a - 1 in
              // the low half-wave, ab + a in the high one (non-negative floats as integers)
              float m0 = mprev, m1 = part;
              swap32(m0, m1);
              vs[a / 2] = __uint_as_float(max(__float_as_uint(m0), __float_as_uint(m1)));
            }
          }
          if (q + 1 < AG * RT) cur = nxt;
        }
        if (ab + AG > M) {
#pragma unroll
          for (int i = 0; i < HA; ++i) vs[i] = ab + 2 * i + u < M ? vs[i] : -1.f;
        }
        // candidates of this group against the running maximum; a rise of the maximum
        // by more than the window drops every earlier candidate
        float gm = vs[0];
#pragma unroll
        for (int i = 1; i < HA; ++i) gm = fmaxf(gm, vs[i]);
        const float nvh = fmaxf(vh, gm), thr = nvh - wnd;
        mask = vh < thr ? uint64_t(0) : mask;
        const float thr0 = fmaxf(thr, 0.f);
        unsigned gb = 0;
#pragma unroll
        for (int i = 0; i < HA; ++i) gb |= vs[i] >= thr0 ? (1u << i) : 0u;
        mask |= uint64_t(gb) << (HA * g);
        if constexpr (kFilter) {
          int gi = HA - 1;
#pragma unroll
          for (int i = HA - 1; i >= 0; --i) gi = vs[i] == gm ? i : gi;
          va = gm > vh ? ab + 2 * gi + u : va;
          _Float16 hv[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) hv[i] = _Float16(vs[i < HA ? i : 0] * invn);
          __builtin_memcpy(&vmax[g], hv, sizeof(uint4));
        }
        vh = nvh;
      }
      const float vo = other_half(vh, u);
      if (!(vh >= fmaxf(vh, vo) - wnd) || !st.active) mask = 0;
      // with the filter: the atom of the largest 16-bit maximum (the low half-wave's on equal
      // maxima) goes first
      const int vao = kFilter ? other_half(va, u) : 0;
      const int m1 = (u == 0 ? vh >= vo : vo < vh) ? va : vao;
      const bool has1 = st.active && fmaxf(vh, vo) >= 0.f;
      if (kFilter && has1 && (m1 & 1) == u) mask &= ~(uint64_t(1) << (m1 >> 1));

      // ---------------- FP32 scores of the candidates, in increasing atom order (after the first)
      float best = -1.f, second = -1.f;   // the largest and the second largest of the atoms' maxima
      int bm = 0;
      unsigned nc = 0;
      f32x16 E[FT], O;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        O[i] = 0.f;
#pragma unroll
        for (int t = 0; t < FT; ++t) E[t][i] = 0.f;
      }
      // the atom's scores over all angles from its C_k, and the largest of them
      auto scores = [&](const float (&op32)[NQ], f32x16 (&e)[FT], f32x16& o) {
#pragma unroll
        for (int i = 0; i < 16; ++i) o[i] = 0.f;
#pragma unroll
        for (int t = 0; t < FT; ++t) {
#pragma unroll
          for (int i = 0; i < 16; ++i) e[t][i] = 0.f;
#pragma unroll
          for (int q = 0; q < NQ; ++q) {
            if (SPLIT && q % 2 == 1) o = mfma32(sF[q * 64 + lane], op32[q], o);
            else e[t] = mfma32(sF[(t * NQ + q) * 64 + lane], op32[q], e[t]);
          }
        }
        float cm = 0.f;
#pragma unroll
        for (int t = 0; t < FT; ++t)
#pragma unroll
          for (int i = 0; i < 16; ++i) cm = fmaxf(cm, SPLIT ? fabsf(e[t][i]) + fabsf(o[i]) : fabsf(e[t][i]));
        return max_halves_nonneg(cm);
      };
      // takes the patch's smallest candidate out of its lanes' masks; false if there is none
      auto next = [&](uint64_t& left, int& m) {
        const int mine = left ? 2 * int(__builtin_ctzll(left)) + u : 0x7fffffff;
        m = min(mine, other_half(mine, u));
        const bool has = m != 0x7fffffff;
        if (has && mine == m) left &= left - 1;
        return has;
      };
      const uint64_t cand = mask;
      for (int pass = 0;; ++pass) {
        int m = m1;
        const bool has = kFilter && pass == 0 ? has1 : next(mask, m);
        if (!__any(has)) break;
        nc += has ? 1 : 0;
        const int mc = has ? m : 0;
        float op32[NQ];
        row_operand<L, W>(sHat + mc * RB, u, res, op32);
        f32x16 e[FT], o;
        const float cm = scores(op32, e, o);
        // equal maxima go to the smaller atom (without the filter the atoms come in order)
        const bool gt = has && (cm > best || (kFilter && cm == best && mc < bm));
        if (FULL) second = has ? __builtin_amdgcn_fmed3f(best, cm, second) : second;   // second <= best
        best = gt ? cm : best;
        bm = gt ? mc : bm;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
#pragma unroll
          for (int t = 0; t < FT; ++t) E[t][i] = gt ? e[t][i] : E[t][i];
          if (SPLIT) O[i] = gt ? o[i] : O[i];
        }
        if (kFilter && pass == 0) {
          const float thrn = has ? best / rn - efac : -2.f;
          uint64_t mm = mask, keep = 0;
          while (mm) {
            const int i = int(__builtin_ctzll(mm));
            mm &= mm - 1;
            _Float16 hv[8];
            const uint4 w = vmax[i >> 3];
            __builtin_memcpy(hv, &w, sizeof(w));
            if (float(hv[i & 7]) >= thrn) keep |= uint64_t(1) << i;
          }
          mask = keep;
        }
      }
      // ---------------- where atoms tie, the one that the full form's first pass chooses (below a
      // squared norm of 1e-30, where products underflow, every second candidate counts as a tie)
      if constexpr (FULL) {
        const bool tie = st.active && second >= (n2 > 1e-30f ? fmaxf(best - ktie * rn, 0.f) : 0.f);
        if (__any(tie)) {
          uint64_t left = tie ? cand : 0;
          float b1 = -1.f, op32[NQ];
          int a1 = bm, m;
          f32x16 e[FT], o;
          for (;;) {
            const bool has = next(left, m);
            if (!__any(has)) break;
            const int mc = has ? m : 0;
            chain_operand<L>(sHat + mc * RB, u, res, op32);
            const float cm = scores(op32, e, o);
            const bool gt = has && cm > b1;
            b1 = gt ? cm : b1;
            a1 = gt ? mc : a1;
          }
          const bool swap = a1 != bm;
          if (__any(swap)) {
            row_operand<L, W>(sHat + a1 * RB, u, res, op32);
            const float cm = scores(op32, e, o);
            best = swap ? cm : best;
            bm = a1;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
#pragma unroll
              for (int t = 0; t < FT; ++t) E[t][i] = swap ? e[t][i] : E[t][i];
              if (SPLIT) O[i] = swap ? o[i] : O[i];
            }
          }
        }
      }
      // ---------------- angle of the best atom: the smallest angle index whose |score| is its
      // maximum.  max(|E| + |O|) is bit for bit the largest rounded |E + O| or |E - O|, so the
      // scores are compared with it for equality; rows past the valid angles score 0 and come
      // last.  The rows ascend with the register in each half-wave: searched from the last.
      // rc: 32 (half of the angles or tile) + 8 (i / 4) + i % 4, a constant of the instruction
      int rc = -1;
      float cval = 0.f;
#pragma unroll
      for (int t = SPLIT ? 1 : FT - 1; t >= 0; --t)
#pragma unroll
        for (int i = 15; i >= 0; --i) {
          const float s = !SPLIT ? E[t % FT][i] : t == 0 ? E[0][i] + O[i] : E[0][i] - O[i];
          const bool eq = fabsf(s) == best;
          rc = eq ? 32 * t + 8 * (i / 4) + i % 4 : rc;
          cval = eq ? s : cval;
        }
      int rs = rc < 0 ? 0x7fffffff : SPLIT ? (rc & 31) + 4 * u + (rc >> 5) * (R / 2) : rc + 4 * u;
      {
        const float ov = other_half(cval, u);
        const int oc = other_half(rs, u);
        cval = oc < rs ? ov : cval;
        rs = oc < rs ? oc : rs;
        rs = rs < R ? rs : R - 1;
      }
      // ---------------- least squares
      wave_lds_order();
      StateIo<KMAX>::load(sState, col, st, ls);
      wave_lds_order();
      n_sel += nc > 0 ? 1 : 0;
      n_cand += nc;
      max_cand = nc > max_cand ? nc : max_cand;
      n_fp64 += ls_step<L, KMAX, W>(st, ls, it, bm, rs, cval, sHat, RB, sCs, tb, prm.norm2, prm.dictHat, p, u, col,
                                 reinterpret_cast<float*>(sState), res) ? 1 : 0;
    }
    const float rn2 = norm2<L, W>(res);
    if (prm.label) {
      if (valid && u == 0 && (prm.cls == 0 || rn2 < prm.sse[p])) {
        prm.sse[p] = rn2;
        prm.label[p] = prm.cls;
      }
    } else if (valid && u == 0) {
#pragma unroll
      for (int i = 0; i < KMAX; ++i) {
        if (i < K) {
          const bool s = i < st.nsel;
          prm.atom[p * K + i] = s ? st.selm[i] : -1;
          prm.angle[p * K + i] = s ? st.selr[i] : -1;
          prm.coef[p * K + i] = s ? st.cf[i] : 0.f;
        }
      }
      if (prm.resid2) prm.resid2[p] = rn2;
    }
  }
  // totals of the counters: over the wave (both half-waves hold them), then over the block in
  // LDS, then one set of atomics per block (one per wave, 2,048 on one line, kept the memory
  // system busy past the work of a small launch)
#pragma unroll
  for (int off = 16; off >= 1; off >>= 1) {
    n_sel += __shfl_xor(n_sel, off);
    n_cand += __shfl_xor(n_cand, off);
    n_fp64 += __shfl_xor(n_fp64, off);
    const unsigned o = __shfl_xor(max_cand, off);
    max_cand = o > max_cand ? o : max_cand;
  }
  __syncthreads();                                   // the tables are no longer read
  unsigned* tot = reinterpret_cast<unsigned*>(lds4);
  if (threadIdx.x < 4) tot[threadIdx.x] = 0u;
  __syncthreads();
  if (lane == 0 && n_sel + n_fp64 > 0) {
    atomicAdd(tot + 0, n_sel);
    atomicAdd(tot + 1, n_cand);
    atomicMax(tot + 2, max_cand);
    atomicAdd(tot + 3, n_fp64);
  }
  __syncthreads();
  if (threadIdx.x == 0 && prm.stats) {
    if (prm.count && tot[0]) {
      atomicAdd(prm.stats + 0, (unsigned long long)tot[0]);
      atomicAdd(prm.stats + 1, (unsigned long long)tot[1]);
      atomicMax(prm.stats + 2, (unsigned long long)tot[2]);
    }
    if (tot[3]) atomicAdd(prm.stats + 3, (unsigned long long)tot[3]);
  }
}

// One launch: 8 waves per block where the tables and their states fit a CU's LDS, else 4.
template <class C, int KMAX, int PREC, int RT, bool SPLIT, int W, bool FULL>
int launch(const DeviceTables& t, const ScreenParams& prm, hipStream_t st) {
  const int nw = screen_waves(t, KMAX);
  if (nw == 0) return int(hipErrorInvalidValue);
  const size_t lds = screen_lds_bytes(t, KMAX, nw);
  auto kern = encode_screen_kernel<C, KMAX, PREC, RT, SPLIT, W, FULL>;
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (e != hipSuccess) return int(e);
  }
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 64 * nw, lds) != hipSuccess || per_cu < 1) per_cu = 1;
  if (t.enc_bpc > 0) per_cu = max(1, min(per_cu, t.enc_bpc * 4 / nw));
  const int64_t tiles = (prm.P + 31) / 32, cap = int64_t(num_cus()) * per_cu;
  hipLaunchKernelGGL(kern, dim3(unsigned(tiles < cap ? tiles : cap)), dim3(64 * nw), lds, st, prm);
  return int(hipGetLastError());
}

// 16-bit handles: the split for even R > 32, the order of sums of the 32x32 tile.
template <class C, int KMAX, int PREC>
int launch_lp(const DeviceTables& t, const ScreenParams& prm, hipStream_t st) {
  if (t.R <= 32) return launch<C, KMAX, PREC, 1, false, 2, false>(t, prm, st);
  if (t.lpSplit) return launch<C, KMAX, PREC, 2, true, 2, false>(t, prm, st);
  return launch<C, KMAX, PREC, 2, false, 2, false>(t, prm, st);
}

// FP32 handles in the order of the 16x16 tile: the split for every even R.
template <class C, int KMAX>
int launch_full16(const DeviceTables& t, const ScreenParams& prm, hipStream_t st) {
  if (t.lpSplit) {
    if (t.R <= 32) return launch<C, KMAX, RSC_FP16, 1, true, 4, true>(t, prm, st);
    return launch<C, KMAX, RSC_FP16, 2, true, 4, true>(t, prm, st);
  }
  if constexpr (std::is_same_v<C, AnnularCounts11>) {
    return int(hipErrorInvalidValue);                // even R only
  } else {
    if (t.R <= 32) return launch<C, KMAX, RSC_FP16, 1, false, 4, true>(t, prm, st);
    return launch<C, KMAX, RSC_FP16, 2, false, 4, true>(t, prm, st);
  }
}

}  // namespace screen
}  // namespace rsc
