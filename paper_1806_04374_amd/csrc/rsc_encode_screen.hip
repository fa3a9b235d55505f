// The screened encoder: which handles it serves, its LDS, and the dispatch over layouts; with
// the instances on the paper's annular basis at N = 11.
#include "rsc_encode_screen.h"

namespace rsc {

int screen_grid11_fp16(const DeviceTables& t, int tile, const screen::ScreenParams& prm, void* stream);
int screen_grid15_fp16(const DeviceTables& t, const screen::ScreenParams& prm, void* stream);
int screen_grid_bf16(const DeviceTables& t, const screen::ScreenParams& prm, void* stream);

namespace {

int kmax_of(const DeviceTables& t, int K) {
  if (t.scrPrec == RSC_BF16) return t.T == 5 ? (K <= 4 ? 4 : 8) : (K <= 6 ? 6 : 8);
  if (K <= 4) return K <= 2 ? 2 : 4;
  return K <= 6 ? 6 : 8;
}

size_t table_bytes(const DeviceTables& t) {
  const int ag = screen_group_atoms(t.T), ng = (t.M + ag - 1) / ag;
  const int ft = t.R <= 32 || t.lpSplit ? 1 : 2;
  return screen::screen_table_bytes(ng, screen_steps(t.T), t.T + 1, ng * ag, screen_row(t.B, t.sk[0]), t.R, ft);
}

}  // namespace

bool screen_supported(int geo, int S, int T, int M, int R) {
  if (M < 1 || M > 128 || R < 1 || R > 64) return false;
  return geo == kGeoGrid ? encode_supported(S, T) : geo == kGeoAnnular11;
}

size_t screen_lds_bytes(const DeviceTables& t, int kmax, int waves) {
  return table_bytes(t) + size_t(waves) * screen_state_f4(kmax) * 32 * 16;
}

int screen_waves(const DeviceTables& t, int kmax) {
  for (int nw = 8; nw >= 4; nw -= 4)
    if (screen_lds_bytes(t, kmax, nw) <= 160 * 1024) return nw;
  return 0;
}

bool screen_usable(const DeviceTables& t, int K) {
  if (t.geo != kGeoGrid && K > kAnnularMaxK) return false;   // no instance has that many slots
  return t.scrPrec != RSC_FP32 && screen_waves(t, kmax_of(t, K)) > 0;
}

double screen_mfma_flops_per_patch(const DeviceTables& t, int K) {
  // per step and 32 patches: the stage-1 and stage-2 32x32x16 instructions of every group
  const int ag = screen_group_atoms(t.T), ops = screen_ops(t.T), ng = (t.M + ag - 1) / ag, rt = t.R <= 32 ? 1 : 2;
  const double per_instr = 2.0 * 32 * 32 * 16;
  return double(K) * ng * (screen_steps(t.T) + double(ag) * rt * ops) * per_instr / 32.0;
}

int launch_encode_screen(const DeviceTables& t, int tile, const float* xhat, int64_t P, int K, int32_t* atom,
                         int32_t* angle, float* coef, float* resid2, void* stream, ClassOut cls) {
  if (P <= 0) return 0;
  const screen::ScreenParams prm{xhat, P, K, t.M, t.R,
                                 reinterpret_cast<const uint4*>(t.lpA), t.dictPairs, t.dictHat,
                                 reinterpret_cast<const uint4*>(t.lpF16), t.lpF32, t.cs, t.gramH, t.norm2, t.gramH64, t.cs64,
                                 atom, angle, coef, resid2, t.lpStats,
                                 t.prec == RSC_FP32 ? kCondMaxFp32 : kCondMax16, t.prec != RSC_FP32,
                                 cls.label, cls.sse, cls.c};
  if (t.geo == kGeoAnnular11) {
    const hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (K <= 2) return screen::launch_full16<AnnularCounts11, 2>(t, prm, st);
    return screen::launch_full16<AnnularCounts11, 4>(t, prm, st);
  }
  if (t.scrPrec == RSC_BF16) return screen_grid_bf16(t, prm, stream);
  if (t.scrPrec != RSC_FP16) return int(hipErrorInvalidValue);
  return t.T == 5 ? screen_grid11_fp16(t, tile, prm, stream) : screen_grid15_fp16(t, prm, stream);
}

}  // namespace rsc
