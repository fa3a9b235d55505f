// The screened encoder (rsc_encode_screen.h) on the 15x15 grid of profiles, FP16 screen.
#include "rsc_encode_screen.h"

namespace rsc {

int screen_grid15_fp16(const DeviceTables& t, const screen::ScreenParams& prm, void* stream) {
  const hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  using C = UniformCounts<7, 7>;
  if (t.prec == RSC_FP16) {
    if (prm.K <= 2) return screen::launch_lp<C, 2, RSC_FP16>(t, prm, st);
    if (prm.K <= 4) return screen::launch_lp<C, 4, RSC_FP16>(t, prm, st);
    if (prm.K <= 6) return screen::launch_lp<C, 6, RSC_FP16>(t, prm, st);
    return screen::launch_lp<C, 8, RSC_FP16>(t, prm, st);
  }
  if (prm.K <= 2) return screen::launch_full16<C, 2>(t, prm, st);
  if (prm.K <= 4) return screen::launch_full16<C, 4>(t, prm, st);
  if (prm.K <= 6) return screen::launch_full16<C, 6>(t, prm, st);
  return screen::launch_full16<C, 8>(t, prm, st);
}

}  // namespace rsc
