// screen_scan_lds.hip -- the screened scan for rows of 129 to 1,024
// dimensions (see screen_tile.h): the tile's queries stay in LDS.
#include "screen_tile.h"

namespace sieve {

hipError_t launch_screen_scan_lds(int nc, const ScreenArgs& a, int32_t grid, hipStream_t s) {
  switch (nc) {
    case 3: return launch_screen_k<3, false, 8, 512, 1>(a, grid, s);
    case 4: return launch_screen_k<4, false, 8, 512, 1>(a, grid, s);
    case 6: return launch_screen_k<6, false, 8, 512, 1>(a, grid, s);
    case 8: return launch_screen_k<8, false, 8, 512, 1>(a, grid, s);
    case 12: return launch_screen_k<12, false, 8, 512, 1>(a, grid, s);
    case 16: return launch_screen_k<16, false, 8, 512, 1>(a, grid, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sieve
