// Pixels of coded or synthetic patches: x_p = Phi sum_j w_j S(theta_j) d_{m_j} (+ noise),
// the map back to pixels of Sec. II-E step 4 with the steering of eq. (6)/(8).
//
//  * reconstruct_kernel (grid angles, the layouts the pursuit is compiled for at 11x11 and
//    15x15): the hat rows of 32 patches are formed in LDS and mapped to pixels on FP32 MFMA.
//  * synth_kernel (continuous angles, other patch sizes): one block per 8 patches builds the
//    hat vectors in LDS, then every pixel is a dot product with a row of Phi.
#include <hip/hip_runtime.h>

#include "rsc_device.h"
#include "rsc_internal.h"
#include "rsc_launch.h"

namespace rsc {
namespace {

struct SynthParams {
  const int32_t* atom;
  const int32_t* angle_idx;   // grid angles (reconstruction), or null
  const float* theta;         // continuous angles (synthesis), or null
  const float* weight;
  const float* noise;
  float* out;
  int64_t P;
  int J, M, R, S, T, B, NN;
  const float* dictHat;       // [.][B]
  const float* cs;            // [2][T+1][R]
  const float* phiPad;        // [NN][B]
  const int* steerTab;        // annular basis: (k << 16) | (partner offset + 32768) per
                              // coordinate; null for the (S, T) grid
};

constexpr int kSynthPB = 8;

__global__ __launch_bounds__(128) void synth_kernel(SynthParams p) {
  extern __shared__ float hat[];  // [kSynthPB][B]
  const int B = p.B, S = p.S;
  const int64_t p0 = int64_t(blockIdx.x) * kSynthPB;
  for (int e = threadIdx.x; e < kSynthPB * B; e += blockDim.x) {
    const int pl = e / B, c = e % B;
    const int64_t pp = p0 + pl;
    float acc = 0.f;
    if (pp < p.P) {
      for (int j = 0; j < p.J; ++j) {
        const int m = p.atom[pp * p.J + j];
        if (m < 0 || m >= p.M) continue;
        int r = 0;
        if (p.angle_idx) {
          r = p.angle_idx[pp * p.J + j];
          if (r < 0 || r >= p.R) continue;
        }
        const float w = p.weight[pp * p.J + j];
        const float* d = p.dictHat + int64_t(m) * B;
        float v;
        if (p.steerTab) {
          // ragged layout: harmonic k and the offset of the Re/Im partner from the table
          const int e2 = p.steerTab[c], k = e2 >> 16, off = (e2 & 0xffff) - 32768;
          if (k == 0) {
            v = d[c];
          } else {
            float co, sn;
            if (p.angle_idx) {
              co = p.cs[k * p.R + r];
              sn = p.cs[(p.T + 1 + k) * p.R + r];
            } else {
              sincosf(float(k) * p.theta[pp * p.J + j], &sn, &co);
            }
            const float own = d[c], partner = d[c + off];
            v = off > 0 ? (own * co + partner * sn) : (own * co - partner * sn);
          }
        } else if (c < S) {
          v = d[c];
        } else {
          const int q = c - S, k = 1 + q / (2 * S), rem = q % (2 * S), s = rem % S;
          const bool im_part = rem >= S;
          const int base = S + 2 * S * (k - 1);
          float co, sn;
          if (p.angle_idx) {
            co = p.cs[k * p.R + r];
            sn = p.cs[(p.T + 1 + k) * p.R + r];
          } else {
            sincosf(float(k) * p.theta[pp * p.J + j], &sn, &co);
          }
          const float re = d[base + s], im = d[base + S + s];
          v = im_part ? (im * co - re * sn) : (re * co + im * sn);
        }
        acc += w * v;
      }
    }
    hat[pl * B + c] = acc;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < kSynthPB * p.NN; e += blockDim.x) {
    const int pl = e / p.NN, q = e % p.NN;
    const int64_t pp = p0 + pl;
    if (pp >= p.P) continue;
    float acc = 0.f;
    const float* ph = p.phiPad + int64_t(q) * B;
    for (int b = 0; b < B; ++b) acc += ph[b] * hat[pl * B + b];
    if (p.noise) acc += p.noise[pp * p.NN + q];
    p.out[pp * p.NN + q] = acc;
  }
}

// Codes to pixels (N*N = NNC pixels, B = BB coordinates, NP = (Re, Im) pairs and harmonic-0
// coordinates per patch).  A block of 4 waves takes 32 patches at a time:
//   codes   each (patch, slot) entry becomes (row offset, angle offset, weight) in LDS, weight 0
//           for an empty slot (the next chunk's entries are loaded meanwhile);
//   hat     one thread per (patch, pair): sum_j w_j S_{r_j} d_{m_j}.  Neighbouring lanes take
//           neighbouring pairs of one patch, so a row is read in one piece from L1 / L2 (the
//           dictionary is 14 to 54 KB), KU slots' reads in flight at a time, and the entry is an
//           LDS broadcast;
//   pixels  rows = output pixels (tiles of 32; wave w owns TPW of them, its rows of Phi in
//           registers), columns = patches, contraction over coordinates (v_mfma_f32_32x32x2f32);
//           they leave through an LDS tile as coalesced 16-byte stores.
// Bound by the pixels' matrix products (4 x 28 of 64 cycles per 32 patches at 11x11 are 0.09 ms
// per 10^6 patches), the vector work of the hat rows and the three barriers of a chunk, which
// five blocks per CU overlap; the 532 MB of codes and pixels take 0.105 ms.  10^6 11x11
// patches with 4 slots take 0.24 ms, against 2.81 ms with synth_kernel.
constexpr int kRecP = 32;

struct ReconParams {
  const int32_t* atom;
  const int32_t* angle;
  const float* coef;
  float* out;
  int64_t P;
  int K, M, R, NQ;
  const float* dictHat;   // [>= M][B]
  const float* cs;        // [2][NQ][R]
  const int* pairTab;     // [NP]: Re coordinate | Im coordinate << 8 | harmonic << 16
  const float* synA;      // [tiles][(B + 1) / 2][64]
  bool vec_out;
};

template <int NNC, int BB, int NP, int TPW, int KU>
__global__ __launch_bounds__(256, TPW == 1 ? 5 : 2) void reconstruct_kernel(ReconParams prm) {
  typedef float v4f __attribute__((ext_vector_type(4)));
  constexpr int KB = (BB + 1) / 2, IT = (kRecP * NP + 255) / 256, EPT = kRecP * 16 / 256;   // K <= 16: at most two entries a thread
  static_assert((kRecP * NNC) % 4 == 0 && 4 * TPW * 32 >= NNC, "whole float4s, tiles cover the pixels");
  __shared__ v4f st4[kRecP * NNC / 4];           // [32 patches][NNC]
  __shared__ float xs[kRecP * BB];               // [32][BB]
  extern __shared__ int4 code[];                 // [32][KP], then [R][NQ] (cos, sin)
  float* st = reinterpret_cast<float*>(st4);
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, col = lane & 31, u = lane >> 5;
  const int K = prm.K, R = prm.R, NQ = prm.NQ, NE = kRecP * K, KP = (K + KU - 1) / KU * KU;
  float2* sCs = reinterpret_cast<float2*>(code + kRecP * KP);
  for (int i = t; i < kRecP * KP; i += 256) code[i] = int4{0, 0, 0, 0};   // slots past K stay empty
  float a[TPW][KB];
#pragma unroll
  for (int i = 0; i < TPW; ++i)
#pragma unroll
    for (int j = 0; j < KB; ++j) a[i][j] = prm.synA[((w * TPW + i) * KB + j) * 64 + lane];
  for (int i = t; i < R * NQ; i += 256) {
    const int r = i / NQ, k = i - r * NQ;
    sCs[i] = float2{prm.cs[k * R + r], prm.cs[(NQ + k) * R + r]};
  }
  // this thread's (patch, pair) items: the same in every chunk
  int ipl[IT], ipr[IT];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int e = t + 256 * i;
    ipl[i] = e < kRecP * NP ? e / NP : 0;
    ipr[i] = prm.pairTab[e < kRecP * NP ? e - ipl[i] * NP : 0];
  }
  const int64_t nchunk = (prm.P + kRecP - 1) / kRecP, total = prm.P * K;
  int na[EPT], nr[EPT];
  float nc[EPT];
  auto fetch = [&](int64_t c) {
#pragma unroll
    for (int v = 0; v < EPT; ++v) {
      const int e = t + 256 * v;
      const int64_t g = c * NE + e;
      const bool in = e < NE && g < total;       // past the last patch: an empty slot
      na[v] = in ? prm.atom[g] : -1;
      nr[v] = in ? prm.angle[g] : 0;
      nc[v] = in ? prm.coef[g] : 0.f;
    }
  };
  int64_t c = blockIdx.x;
  fetch(c);
  const float* mine = xs + col * BB + u;
  __syncthreads();   // the cleared slots
  for (; c < nchunk; c += gridDim.x) {
    // (every wave is past the previous chunk's products: the barrier before its stores)
#pragma unroll
    for (int v = 0; v < EPT; ++v) {
      const int e = t + 256 * v;
      const bool use = unsigned(na[v]) < unsigned(prm.M) && unsigned(nr[v]) < unsigned(R);
      const int pl = e / K;
      if (e < NE)
        code[pl * KP + e - pl * K] = int4{use ? na[v] * BB : 0, use ? nr[v] * NQ : 0, use ? __float_as_int(nc[v]) : 0, 0};
    }
    __syncthreads();
    if (c + gridDim.x < nchunk) fetch(c + gridDim.x);
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      // an item past the last one repeats item 0 of its chunk, with the same result
      const int pl = ipl[i], ire = ipr[i] & 255, iim = (ipr[i] >> 8) & 255, k = ipr[i] >> 16;
      float re = 0.f, im = 0.f;
      for (int j0 = 0; j0 < KP; j0 += KU) {
        int4 z[KU];
        float dr[KU], di[KU];
#pragma unroll
        for (int j = 0; j < KU; ++j) z[j] = code[pl * KP + j0 + j];
#pragma unroll
        for (int j = 0; j < KU; ++j) {
          dr[j] = prm.dictHat[z[j].x + ire];
          di[j] = prm.dictHat[z[j].x + iim];
        }
#pragma unroll
        for (int j = 0; j < KU; ++j) {
          const float wgt = __int_as_float(z[j].z);  // an empty slot: weight 0, row 0
          const float2 cs = sCs[z[j].y + k];         // (1, 0) at harmonic 0
          re += wgt * (dr[j] * cs.x + di[j] * cs.y);
          im += wgt * (di[j] * cs.x - dr[j] * cs.y);
        }
      }
      xs[pl * BB + ire] = re;
      if (k) xs[pl * BB + iim] = im;
    }
    __syncthreads();
    f32x16 acc[TPW];
#pragma unroll
    for (int i = 0; i < TPW; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      const float b = 2 * j + u < BB ? mine[2 * j] : 0.f;   // odd B: the last slot is padding
#pragma unroll
      for (int i = 0; i < TPW; ++i) acc[i] = mfma32(a[i][j], b, acc[i]);
    }
#pragma unroll
    for (int i = 0; i < TPW; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int q = 32 * (w * TPW + i) + 8 * (r / 4) + 4 * u + (r % 4);
        if (q < NNC) st[col * NNC + q] = acc[i][r];
      }
    __syncthreads();
    const int64_t left = prm.P - c * kRecP;
    float* dst = prm.out + c * kRecP * NNC;
    if (prm.vec_out && left >= kRecP) {
      for (int i = t; i < kRecP * NNC / 4; i += 256) __builtin_nontemporal_store(st4[i], reinterpret_cast<v4f*>(dst) + i);
    } else {
      const int n = (left < kRecP ? int(left) : kRecP) * NNC;
      for (int i = t; i < n; i += 256) dst[i] = st[i];
    }
  }
}

}  // namespace

int launch_reconstruct(const DeviceTables& t, const int32_t* atom, const int32_t* angle, const float* coef, int64_t P,
                       int K, float* out, void* stream) {
  if (P <= 0) return 0;
  const int NN = t.N * t.N;
  const ReconParams prm{atom, angle, coef, out, P, K, t.M, t.R, t.T + 1, t.dictHat, t.cs, t.pairTab, t.synA,
                        (reinterpret_cast<uintptr_t>(out) & 15) == 0};
  // slots go by 1 or 2 at a time; 4 at a time took more registers and measured slower
  // (0.31 against 0.28 ms at 10^6 11x11 patches, K = 4)
  const int ku = K <= 1 ? 1 : 2, kp = (K + ku - 1) / ku * ku;
  const size_t lds = sizeof(int4) * size_t(kRecP) * kp + sizeof(float2) * size_t(t.R) * (t.T + 1);
  auto go = [&](auto k1, auto k2) {
    auto kern = ku == 1 ? k1 : k2;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 256, lds) != hipSuccess || per_cu < 1) per_cu = 1;
    const int64_t chunks = (P + kRecP - 1) / kRecP, cap = int64_t(num_cus()) * per_cu;
    hipLaunchKernelGGL(kern, dim3(unsigned(chunks < cap ? chunks : cap)), dim3(256), lds,
                       reinterpret_cast<hipStream_t>(stream), prm);
    return int(hipGetLastError());
  };
  // the layouts the pursuit is compiled for, at their own patch sizes
  if (K <= 16 && t.synA && t.pairTab) {
    if (NN == 121 && t.B == 55) return go(reconstruct_kernel<121, 55, 30, 1, 1>, reconstruct_kernel<121, 55, 30, 1, 2>);
    if (NN == 225 && t.B == 105) return go(reconstruct_kernel<225, 105, 56, 2, 1>, reconstruct_kernel<225, 105, 56, 2, 2>);
    if (NN == 121 && t.B == 81 && t.geo == kGeoAnnular11) return go(reconstruct_kernel<121, 81, 43, 1, 1>, reconstruct_kernel<121, 81, 43, 1, 2>);
    if (NN == 225 && t.B == 153 && t.geo == kGeoAnnular15) return go(reconstruct_kernel<225, 153, 80, 2, 1>, reconstruct_kernel<225, 153, 80, 2, 2>);
  }
  return launch_synthesize(t, atom, angle, nullptr, coef, P, K, nullptr, out, stream);
}

int launch_synthesize(const DeviceTables& t, const int32_t* atom, const int32_t* angle_idx,
                      const float* theta, const float* weight, int64_t P, int J, const float* noise,
                      float* out, void* stream) {
  if (P <= 0) return 0;
  SynthParams p{atom, angle_idx, theta, weight, noise, out, P, J, t.M, t.R, t.S, t.T, t.B,
                t.N * t.N, t.dictHat, t.cs, t.phiPad, t.geo == kGeoGrid ? nullptr : t.steerTab};
  const int64_t blocks = (P + kSynthPB - 1) / kSynthPB;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(synth_kernel, dim3(unsigned(blocks)), dim3(128), sizeof(float) * kSynthPB * t.B,
                     st, p);
  return int(hipGetLastError());
}

}  // namespace rsc
