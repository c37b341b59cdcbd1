// The products + output-transform kernel with two pairs per lane (sfc_pair16.hpp) for 257 to 512 input
// channels: its own translation unit so that the instantiations compile beside the others.
#include "sfc_pair16.hpp"

namespace sfc {

hipError_t launch_pair16_wide(int out, const Geometry& g, const void* V, const FilterViews& f, float x_scale,
                              float inv_y, void* y, hipStream_t s, bool prepare) {
  switch (g.Cp / 64) {
    case 5: return launch_pair16_kc<5>(out, g, V, f, x_scale, inv_y, y, s, prepare);
    case 6: return launch_pair16_kc<6>(out, g, V, f, x_scale, inv_y, y, s, prepare);
    case 7: return launch_pair16_kc<7>(out, g, V, f, x_scale, inv_y, y, s, prepare);
    case 8: return launch_pair16_kc<8>(out, g, V, f, x_scale, inv_y, y, s, prepare);
  }
  return hipErrorNotSupported;
}

}  // namespace sfc
