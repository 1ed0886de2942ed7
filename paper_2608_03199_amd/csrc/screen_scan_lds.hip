// screen_scan_lds.hip -- the screened scan for rows of 129 to 1,024
// dimensions (see screen_tile.h): the tile's queries stay in LDS.
#include "screen_tile.h"

namespace sieve {

// Two work-groups of four waves per CU, so that one streams while the other
// ends its tile; tiles of 128 queries of more than 512 dimensions need a CU's
// LDS for one (of eight waves).
template <int NC>
static hipError_t launch_nc(const ScreenArgs& a, int32_t grid, hipStream_t s) {
  if (a.tile_q <= 64) return launch_screen_k<NC, false, 4, 256, 2>(a, grid, s);
  if constexpr (NC <= 8)
    return launch_screen_k<NC, false, 8, 256, 2>(a, grid, s);
  else
    return launch_screen_k<NC, false, 8, 512, 1>(a, grid, s);
}

hipError_t launch_screen_scan_lds(int nc, const ScreenArgs& a, int32_t grid, hipStream_t s) {
  switch (nc) {
    case 3: return launch_nc<3>(a, grid, s);
    case 4: return launch_nc<4>(a, grid, s);
    case 6: return launch_nc<6>(a, grid, s);
    case 8: return launch_nc<8>(a, grid, s);
    case 12: return launch_nc<12>(a, grid, s);
    case 16: return launch_nc<16>(a, grid, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sieve
