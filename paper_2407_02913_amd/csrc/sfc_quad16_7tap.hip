// The products + output-transform kernel with 16 filters per wave (sfc_quad16.hpp) for
// SFC-6(4x4,7x7) (184 points): its own translation unit so that the instantiations compile beside
// those of the other forms.
#include "sfc_quad16.hpp"

namespace sfc {

constexpr int kAlg7Tap = 8;  // SFC_ALG_4X4_7X7_P184

template <int KC, int OUT>
static hipError_t launch_quad16_7tap_impl(const Geometry& g, const void* V, const FilterViews& f,
                                          float x_scale, float inv_y, void* y, hipStream_t s,
                                          bool prepare) {
  constexpr int NW = kQuad16Waves;
  auto kernel = quad16_kernel<kAlg7Tap, KC, OUT, 0, NW>;
  constexpr unsigned lds_bytes = quad16_lds_layout<KC, NW, OUT>(2);
  static_assert(lds_bytes <= 80u * 1024u, "two workgroups per compute unit");
  if (prepare) return raise_lds_limit(reinterpret_cast<const void*>(kernel));
  const int fgroups = quad16_filter_count(g) / 16;
  const dim3 grid((unsigned)((g.Tp / 16) * (fgroups / NW)));
  hipLaunchKernelGGL(kernel, grid, dim3(NW * 64), lds_bytes, s, (const int8_t*)V,
                     (const int8_t*)f.U_single, f.dequant_single, x_scale, inv_y, y, g, fgroups);
  return hipGetLastError();
}

hipError_t launch_quad16_7tap(int out, const Geometry& g, const void* V, const FilterViews& f,
                              float x_scale, float inv_y, void* y, hipStream_t s, bool prepare) {
  switch (g.Cp / 64) {
    case 1: return out == 2 ? launch_quad16_7tap_impl<1, 2>(g, V, f, x_scale, inv_y, y, s, prepare)
                            : launch_quad16_7tap_impl<1, 0>(g, V, f, x_scale, inv_y, y, s, prepare);
    case 2: return out == 2 ? launch_quad16_7tap_impl<2, 2>(g, V, f, x_scale, inv_y, y, s, prepare)
                            : launch_quad16_7tap_impl<2, 0>(g, V, f, x_scale, inv_y, y, s, prepare);
    case 3: return out == 2 ? launch_quad16_7tap_impl<3, 2>(g, V, f, x_scale, inv_y, y, s, prepare)
                            : launch_quad16_7tap_impl<3, 0>(g, V, f, x_scale, inv_y, y, s, prepare);
    case 4: return out == 2 ? launch_quad16_7tap_impl<4, 2>(g, V, f, x_scale, inv_y, y, s, prepare)
                            : launch_quad16_7tap_impl<4, 0>(g, V, f, x_scale, inv_y, y, s, prepare);
  }
  return hipErrorNotSupported;
}

}  // namespace sfc
