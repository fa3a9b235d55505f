// The screened encoder (rsc_encode_screen.h) on the 11x11 grid of profiles, FP16 screen.
#include "rsc_encode_screen.h"

namespace rsc {

int screen_grid11_fp16(const DeviceTables& t, const screen::ScreenParams& prm, void* stream) {
  const hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  using C = UniformCounts<5, 5>;
  if (prm.K <= 2) return screen::launch_angles<C, 2, RSC_FP16>(t, prm, st);
  if (prm.K <= 4) return screen::launch_angles<C, 4, RSC_FP16>(t, prm, st);
  if (prm.K <= 6) return screen::launch_angles<C, 6, RSC_FP16>(t, prm, st);
  return screen::launch_angles<C, 8, RSC_FP16>(t, prm, st);
}

}  // namespace rsc
