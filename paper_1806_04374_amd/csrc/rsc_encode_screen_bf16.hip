// The screened encoder (rsc_encode_screen.h) of BF16 handles: both grids of profiles.
#include "rsc_encode_screen.h"

namespace rsc {

int screen_grid_bf16(const DeviceTables& t, const screen::ScreenParams& prm, void* stream) {
  const hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (t.T == 5) {
    if (prm.K <= 4) return screen::launch_lp<UniformCounts<5, 5>, 4, RSC_BF16>(t, prm, st);
    return screen::launch_lp<UniformCounts<5, 5>, 8, RSC_BF16>(t, prm, st);
  }
  if (prm.K <= 6) return screen::launch_lp<UniformCounts<7, 7>, 6, RSC_BF16>(t, prm, st);
  return screen::launch_lp<UniformCounts<7, 7>, 8, RSC_BF16>(t, prm, st);
}

}  // namespace rsc
