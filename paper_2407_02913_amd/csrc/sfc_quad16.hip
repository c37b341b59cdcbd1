// Launch side of the SFC-4 products + output-transform kernel (sfc_quad16.hpp): limits, the
// regrouping of the filter operand and the dispatch over channel chunks and output type.
#include "sfc_quad16.hpp"

namespace sfc {

hipError_t launch_quad16_7tap(int out, const Geometry& g, const void* V, const FilterViews& f,
                              float x_scale, float inv_y, void* y, hipStream_t s, bool prepare);

// Layers whose workgroups leave compute units idle, so that one workgroup's chain is the
// duration, on maps of two tile columns and odd width (7x7): a wave stores its 16 filters one
// element at a time, every instruction on pieces of many short rows, where a wave of the
// one-pair-per-lane kernel stores four.  7x7 filters, 64 to 64 channels on 7x7 maps, batch 64: 33.0 us
// here, 27.8 there (kernels 22.6 and 17.4); over 100 layers of at least 16 tiles and 64 filters 1.06 times
// its time here (0.98 to 1.20).  With fewer tiles or filters (0.9), on wider maps (9x13 0.95 to
// 1), and with several channel chunks from 128 tiles on (0.97), it is level or behind.
static bool quad16_stores_bound(const Geometry& g) {
  return g.W % 2 == 1 && g.tw == 2 && g.Cout >= 64 && g.T >= 16 && (g.Cp == 64 || g.T < 128) &&
         (long long)(g.Tp / 16) * ((g.Cout + 63) / 64) < 128;
}

// SFC-4 with 46 points and three to eight channel chunks: whether the layer has enough workgroups of 16 tiles x
// 64 filters.  A workgroup is one chain, 14 to 30 us with its input transform whatever the layer's size; below the line three kernels
// (three, five to seven chunks), the one-pair-per-lane kernel (four) or the split of the channels (eight)
// are ahead.  us here over us there from 187 layers, workgroups: ratio,
//   3   24: 1.02-1.2, 32: 0.97, 48: 0.90-1.0, 80: 0.84, 126: 0.83, 516: 0.79, 1200: 0.61
//   4   39-48: 0.87, 62-98: 0.89-0.98, 125-150: 0.82-0.92, 152-200: 0.77-0.91
//   5   80-108: 0.98-1.07, 124: 0.98-1.0, 147-216: 0.79-0.98, 1143: 0.71
//   6   104-144: 1.05-1.1, 160: 1.0, 174-233: 0.91, 304: 1.03, 378-672: 0.75-0.85
//   7   133-172: 0.98-1.03, 205-225: 0.71-0.88, 264: 1.0, 396-602: 0.66-0.86
//   8   66-158: 1.15-1.23, 180: 0.88, 212-384: 0.75-0.91, 512-576: 0.71-0.77
// Two tile columns and odd width (7x7): the stores of quad16_stores_bound; 56: 1.1, 128: 1.07-1.18, 189: 1.09, 232: 0.97,
// 368: 0.91.  From six chunks on no less than 5/8 of the filters must exist (16, 24, 40 and 72 of 64 or 128: 0.83 to 1.2,
// 1.0 in the middle).
static bool quad16_workgroups_enough(const Geometry& g) {
  constexpr int kLines[9] = {0, 0, 0, 40, 48, 140, 165, 200, 180};
  const int kc = g.Cp / 64;
  const int groups = (g.Cout + 63) / 64;
  if (kc >= 6 && g.Cout * 8ll < groups * 64ll * 5) return false;
  const int line = kLines[kc] + (g.W % 2 == 1 && g.tw == 2 ? 120 : 0);
  return (long long)(g.Tp / 16) * groups >= line;
}

// a wave takes 256 (tile, filter) pairs
static bool one_wave_per_simd(const Geometry& g) { return (long long)(g.Tp / 16) * ((g.Cout + 15) / 16) >= 1024; }

bool quad16_supported(const Geometry& g) {
  if (g.alg != 4 && g.alg != 5 && g.alg != 8) return false;
  const int kc = g.Cp / 64;
  // Up to four channel chunks (three with 184 points), with 46 points eight.
  if (kc > (g.alg == 4 ? 8 : 4) || (kc == 3 && g.alg == 5)) return false;
  // With fewer than one wave per SIMD of the chip the
  // one-pair-per-lane kernel, whose waves take 64, fills it better.  With 184 points its fourfold
  // matrix work and operand reads outweigh that on most layers (7x7 filters, layer: 16 channels
  // on one 32x32 map 30.3 us against 26.3 here, 128 channels on one 28x28 map 35.2 against 32.1,
  // 256 channels on 14x14 maps at batch 32 67.3 against 59.5), not where quad16_stores_bound.
  if (g.alg == 4 && kc >= 3) {
    if (!quad16_workgroups_enough(g)) return false;
  } else if (g.alg < 6 && !one_wave_per_simd(g)) {
    return false;
  }
  if (g.alg == 8 && quad16_stores_bound(g)) return false;
  const long long fgroups = quad16_filter_count(g) / 16;
  const long long ybytes = 4ll * g.N * g.Cout * g.H * g.W;
  const long long vbytes = (long long)g.P * g.Tp * g.Cp;
  const long long ubytes = fgroups * 16 * ((g.P + 3) / 4 * 4) * g.Cp;
  const long long lim = 1ll << 31;
  return ybytes < lim && vbytes < lim && ubytes < lim;
}

// filters covered by the regrouped operand: Cout rounded up to whole workgroups
int quad16_filter_count(const Geometry& g) {
  const int per_wg = 16 * kQuad16Waves;
  return (g.Cout + per_wg - 1) / per_wg * per_wg;
}

// Filter operand from the canonical U[p][k][c]: block (filter group fg, position j, channel
// chunk kc) is one KiB; lane l holds the 16 channels 64*kc + 16*(l/16).. of point pt[j] for
// filter 16*fg + 4*(r%4) + r/4, r = l%16 (row r of the MFMA operand).  Filters beyond Kp and
// positions without a point are zero.
template <int ALG>
__global__ __launch_bounds__(64) void repack_filter16_kernel(const int8_t* __restrict__ U,
                                                             int8_t* __restrict__ U16, Geometry g) {
  constexpr int PP = Order<ALG>::PP;
  constexpr Order<ALG> order{};
  const int KC = g.Cp >> 6;
  const int fg = blockIdx.x / (PP * KC), rem = blockIdx.x - fg * (PP * KC);
  const int j = rem / KC, kc = rem - j * KC;
  const int l = threadIdx.x;
  const int r = l & 15, kseg = l >> 4;
  const int p = order.pt[j];
  const int k = 16 * fg + 4 * (r & 3) + (r >> 2);
  v4i val = {0, 0, 0, 0};
  if (k < g.Kp && p >= 0) val = *(const v4i*)(U + ((size_t)p * g.Kp + k) * g.Cp + 64 * kc + 16 * kseg);
  *(v4i*)(U16 + ((size_t)blockIdx.x * 64 + l) * 16) = val;
}

hipError_t launch_repack_filter16(const Geometry& g, int filters, const void* U, void* U16,
                                  hipStream_t s) {
  const dim3 grid((unsigned)((filters / 16) * ((g.P + 3) / 4 * 4) * (g.Cp / 64)));
  switch (g.alg) {
    case 2: hipLaunchKernelGGL(repack_filter16_kernel<2>, grid, dim3(64), 0, s, (const int8_t*)U, (int8_t*)U16, g); break;
    case 3: hipLaunchKernelGGL(repack_filter16_kernel<3>, grid, dim3(64), 0, s, (const int8_t*)U, (int8_t*)U16, g); break;
    case 4: hipLaunchKernelGGL(repack_filter16_kernel<4>, grid, dim3(64), 0, s, (const int8_t*)U, (int8_t*)U16, g); break;
    case 5: hipLaunchKernelGGL(repack_filter16_kernel<5>, grid, dim3(64), 0, s, (const int8_t*)U, (int8_t*)U16, g); break;
    case 8: hipLaunchKernelGGL(repack_filter16_kernel<8>, grid, dim3(64), 0, s, (const int8_t*)U, (int8_t*)U16, g); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int ALG, int KC, int OUT, int EV>
static hipError_t launch_quad16_impl(const Geometry& g, const void* V, const FilterViews& f,
                                     float x_scale, float inv_y, void* y, hipStream_t s,
                                     bool prepare) {
  constexpr int NW = kQuad16Waves;
  auto kernel = quad16_kernel<ALG, KC, OUT, EV, NW>;
  constexpr unsigned lds_bytes = quad16_lds_layout<KC, NW, OUT>(2);
  static_assert(lds_bytes <= 160u * 1024u, "V buffers and staging exceed the LDS of a compute unit");
  if (prepare) return raise_lds_limit(reinterpret_cast<const void*>(kernel));
  const int fgroups = quad16_filter_count(g) / 16;
  const dim3 grid((unsigned)((g.Tp / 16) * (fgroups / NW)));
  hipLaunchKernelGGL(kernel, grid, dim3(NW * 64), lds_bytes, s, (const int8_t*)V,
                     (const int8_t*)f.U_single, f.dequant_single, x_scale, inv_y, y, g, fgroups);
  return hipGetLastError();
}

template <int ALG, int KC>
static hipError_t launch_quad16_kc(int out, const Geometry& g, const void* V, const FilterViews& f,
                                   float x_scale, float inv_y, void* y, hipStream_t s, bool prepare) {
  // elements per store: a tile row of four outputs never crosses the end of an image row when
  // 4 divides W; else pairs (W even) or single elements
  if (g.W % 4 == 0)
    return out == 2 ? launch_quad16_impl<ALG, KC, 2, 4>(g, V, f, x_scale, inv_y, y, s, prepare)
                    : launch_quad16_impl<ALG, KC, 0, 4>(g, V, f, x_scale, inv_y, y, s, prepare);
  if (g.W % 2 == 0)
    return out == 2 ? launch_quad16_impl<ALG, KC, 2, 2>(g, V, f, x_scale, inv_y, y, s, prepare)
                    : launch_quad16_impl<ALG, KC, 0, 2>(g, V, f, x_scale, inv_y, y, s, prepare);
  return out == 2 ? launch_quad16_impl<ALG, KC, 2, 1>(g, V, f, x_scale, inv_y, y, s, prepare)
                  : launch_quad16_impl<ALG, KC, 0, 1>(g, V, f, x_scale, inv_y, y, s, prepare);
}

// (the store's width chosen in the kernel)
template <int ALG, int KC>
static hipError_t launch_quad16_any_width(int out, const Geometry& g, const void* V, const FilterViews& f,
                                          float x_scale, float inv_y, void* y, hipStream_t s, bool prepare) {
  return out == 2 ? launch_quad16_impl<ALG, KC, 2, 0>(g, V, f, x_scale, inv_y, y, s, prepare)
                  : launch_quad16_impl<ALG, KC, 0, 0>(g, V, f, x_scale, inv_y, y, s, prepare);
}

template <int ALG>
static hipError_t launch_quad16_alg(int out, const Geometry& g, const void* V, const FilterViews& f,
                                    float x_scale, float inv_y, void* y, hipStream_t s, bool prepare) {
  switch (g.Cp / 64) {
    case 1: return launch_quad16_kc<ALG, 1>(out, g, V, f, x_scale, inv_y, y, s, prepare);
    case 2: return launch_quad16_kc<ALG, 2>(out, g, V, f, x_scale, inv_y, y, s, prepare);
    case 4: return launch_quad16_kc<ALG, 4>(out, g, V, f, x_scale, inv_y, y, s, prepare);
  }
  if constexpr (ALG == 4) {
    switch (g.Cp / 64) {
      case 3: return launch_quad16_any_width<ALG, 3>(out, g, V, f, x_scale, inv_y, y, s, prepare);
      case 5: return launch_quad16_any_width<ALG, 5>(out, g, V, f, x_scale, inv_y, y, s, prepare);
      case 6: return launch_quad16_any_width<ALG, 6>(out, g, V, f, x_scale, inv_y, y, s, prepare);
      case 7: return launch_quad16_any_width<ALG, 7>(out, g, V, f, x_scale, inv_y, y, s, prepare);
      case 8: return launch_quad16_any_width<ALG, 8>(out, g, V, f, x_scale, inv_y, y, s, prepare);
    }
  }
  return hipErrorNotSupported;
}

hipError_t launch_quad16(int out, const Geometry& g, const void* V, const FilterViews& f,
                         float x_scale, float inv_y, void* y, hipStream_t s, bool prepare) {
  if (!quad16_supported(g) || out == 1) return hipErrorNotSupported;
  // int8 outputs at a tie of their rounding: the staged path, the one-pair-per-lane kernel and the split of the
  // channels scale twice (store_pairs), this kernel up to two chunks once.  From three chunks on it scales twice,
  // so that a layer's bytes are the same on either side of the lines above; but for four chunks and a wave for
  // every SIMD, layers that no other kernel takes (1 * (x_scale inv_y): the product again).
  if (out == 2 && g.alg == 4 && g.Cp == 256 && one_wave_per_simd(g)) {
    inv_y *= x_scale;
    x_scale = 1.0f;
  }
  switch (g.alg) {
    case 4: return launch_quad16_alg<4>(out, g, V, f, x_scale, inv_y, y, s, prepare);
    case 5: return launch_quad16_alg<5>(out, g, V, f, x_scale, inv_y, y, s, prepare);
    case 8: return launch_quad16_7tap(out, g, V, f, x_scale, inv_y, y, s, prepare);
  }
  return hipErrorNotSupported;
}

}  // namespace sfc
