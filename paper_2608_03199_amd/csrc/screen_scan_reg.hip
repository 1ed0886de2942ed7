// screen_scan_reg.hip -- the screened scan for rows of at most 128 dimensions
// (see screen_tile.h): the tile's query fragments stay in registers.
#include "screen_tile.h"

namespace sieve {

// Dense rounds: tiles of up to 128 queries, two work-groups per CU; sparse
// rounds: up to 64 queries, as many.
hipError_t launch_screen_scan_reg(int nc, const ScreenArgs& a, int32_t grid, hipStream_t s) {
  const bool dense = a.tile_q > 64;
  if (nc == 1)
    return dense ? launch_screen_k<1, true, 8, 256, 2>(a, grid, s)
                 : launch_screen_k<1, true, 4, 256, 2>(a, grid, s);
  if (nc == 2)
    return dense ? launch_screen_k<2, true, 8, 256, 2>(a, grid, s)
                 : launch_screen_k<2, true, 4, 256, 2>(a, grid, s);
  return hipErrorInvalidValue;
}

}  // namespace sieve
