// Launch side of the products + output-transform kernel with two pairs per lane (sfc_pair16.hpp):
// limits, the regrouping of the filter operand and the dispatch.  More than 256 input channels are
// instantiated in sfc_pair16_wide.hip.
#include "sfc_pair16.hpp"

namespace sfc {

hipError_t launch_pair16_wide(int out, const Geometry& g, const void* V, const FilterViews& f, float x_scale,
                              float inv_y, void* y, hipStream_t s, bool prepare);

bool pair16_supported(const Geometry& g) {
  if (g.alg != kAlg5Tap) return false;
  const int kc = g.Cp / 64;
  if (kc > 8) return false;
  const long long filters = pair16_filter_count(g);
  const long long ybytes = 4ll * g.N * g.Cout * g.H * g.W, vbytes = (long long)g.P * g.Tp * g.Cp;
  const long long lim = 1ll << 31;
  return ybytes < lim && vbytes < lim && filters * g.P * g.Cp < lim;
}

int pair16_filter_count(const Geometry& g) {
  const int per_wg = 8 * pair16_waves(g);
  return (g.Cout + per_wg - 1) / per_wg * per_wg;
}

// Filter operand from the canonical U[p][k][c]: block (group of 8 filters fg, pair of positions jp,
// channel chunk kc) is one KiB; lane l holds the 16 channels 64*kc + 16*(l/16).. of point pt[2 jp + r%2]
// for filter 8*fg + 4*((r%4)/2) + r/4, r = l%16.  Filters beyond Kp are zero.
__global__ __launch_bounds__(64) void repack_filter8_kernel(const int8_t* __restrict__ U, int8_t* __restrict__ U8,
                                                            Geometry g) {
  constexpr int JP = AlgTraits<kAlg5Tap>::P / 2;
  constexpr Order<kAlg5Tap> order{};
  const int KC = g.Cp >> 6;
  const int fg = blockIdx.x / (JP * KC), rem = blockIdx.x - fg * (JP * KC);
  const int jp = rem / KC, kc = rem - jp * KC;
  const int l = threadIdx.x, r = l & 15, kseg = l >> 4;
  const int p = order.pt[2 * jp + (r & 1)];
  const int k = 8 * fg + 4 * ((r & 3) >> 1) + (r >> 2);
  v4i val = {0, 0, 0, 0};
  if (k < g.Kp) val = *(const v4i*)(U + ((size_t)p * g.Kp + k) * g.Cp + 64 * kc + 16 * kseg);
  *(v4i*)(U8 + ((size_t)blockIdx.x * 64 + l) * 16) = val;
}

hipError_t launch_repack_filter8(const Geometry& g, int filters, const void* U, void* U8, hipStream_t s) {
  if (g.alg != kAlg5Tap) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((filters / 8) * (g.P / 2) * (g.Cp / 64)));
  hipLaunchKernelGGL(repack_filter8_kernel, grid, dim3(64), 0, s, (const int8_t*)U, (int8_t*)U8, g);
  return hipGetLastError();
}

hipError_t launch_pair16(int out, const Geometry& g, const void* V, const FilterViews& f, float x_scale, float inv_y,
                         void* y, hipStream_t s, bool prepare) {
  if (!pair16_supported(g) || out == 1) return hipErrorNotSupported;
  switch (g.Cp / 64) {
    case 1: return launch_pair16_kc<1>(out, g, V, f, x_scale, inv_y, y, s, prepare);
    case 2: return launch_pair16_kc<2>(out, g, V, f, x_scale, inv_y, y, s, prepare);
    case 3: return launch_pair16_kc<3>(out, g, V, f, x_scale, inv_y, y, s, prepare);
    case 4: return launch_pair16_kc<4>(out, g, V, f, x_scale, inv_y, y, s, prepare);
  }
  return launch_pair16_wide(out, g, V, f, x_scale, inv_y, y, s, prepare);
}

}  // namespace sfc
