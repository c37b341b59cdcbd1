// Exact mode on the matrix cores (gfx950): transform-domain operands kept as 16-bit integers,
// sums as 32-bit ones, so that the result equals direct convolution bit for bit.
//
//   input_rows_kernel            V = B^T x B            (sfc_input_rows.hip; NCHW int8 -> int16 [P][Tp][Cp])
//   product_gemm_i16_kernel      M_p = V_p . U_p^T      (int16 operands as pairs of int8 ones)
//   output_exact_kernel          y = A^T M A / kDen, corrections, NCHW store
//
// M is kept as in requantized mode, in blocks of 16 tiles x 4 filters (sfc_gemm.hip).  The
// three kernels move V (2 bytes a value) and M (4) to memory and back and are bound by that.
// 64 channels on 56x56 maps, batch 32, 6x6 tiles (V 36 MB, M 72 MB, y 26 MB): 12.1 + 17.9 +
// 25.1 us (3.5, 6.1 and 3.9 TB/s); with the transforms and products on the vector ALU, one
// thread per (tile, channel), sum and (tile, filter), 31 + 133 + 47 us.
#include "sfc_device.hpp"
#include "sfc_internal.hpp"
#include "sfc_mfma_input.hpp"
#include "sfc_points.hpp"
#include "sfc_store.hpp"
#include "sfc_tile_input.hpp"

namespace sfc {

// ---------------------------------------------------------------------------------------
// Products.  A 16-bit operand is v = 256 h + l with l its low byte taken as a signed one and
// h = (v - l) / 256, |h| <= 25 for the transforms of this library (49 * 128 at the all-taps point
// of a 7x7 filter); a sum of products is then
// 65536 S(hh) + 256 S(hl + lh) + S(ll), three int32 accumulators and four int8 MFMA 16x16x64,
// exact (|S(ll)| <= 2^14 Cin; the combination is taken modulo 2^32 like everything behind it).
// A workgroup of four waves owns 64 filters x 64 tiles of one point, each wave 32 x 32; per
// 64-channel chunk it stages the two bytes of 64 rows of U and of V in LDS through registers,
// split on the way, the next chunk's loads in flight.
// ---------------------------------------------------------------------------------------
constexpr int kExactBlock = 64;  // filters and tiles per workgroup
constexpr int kExactPitch = 80;  // LDS bytes per operand row (64 + padding: conflict-free reads)

// low bytes, and high bytes after the low byte's sign has been carried into them, of the eight
// 16-bit values of d
__device__ __forceinline__ void split_i16(v4i d, v2i& lo, v2i& hi) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const unsigned d0 = (unsigned)d[2 * i], d1 = (unsigned)d[2 * i + 1];
    lo[i] = (int)__builtin_amdgcn_perm(d1, d0, 0x06040200u);
    typedef short v2s __attribute__((ext_vector_type(2)));
    const v2s half = {128, 128};
    const unsigned e0 = __builtin_bit_cast(unsigned, __builtin_bit_cast(v2s, d0) + half);
    const unsigned e1 = __builtin_bit_cast(unsigned, __builtin_bit_cast(v2s, d1) + half);
    hi[i] = (int)__builtin_amdgcn_perm(e1, e0, 0x07050301u);
  }
}

__global__ __launch_bounds__(256) void product_gemm_i16_kernel(const int16_t* __restrict__ V,
                                                               const int16_t* __restrict__ U,
                                                               int32_t* __restrict__ M, Geometry g,
                                                               int nbt, int nbf) {
  constexpr int BL = kExactBlock, PITCH = kExactPitch, PLANE = BL * PITCH;
  __shared__ __align__(16) unsigned char lds[2 * 4 * PLANE];  // [buffer][U low, U high, V low, V high]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int pos = xcd_contiguous(blockIdx.x, gridDim.x);
  const int per_point = nbt * nbf;
  const int p = pos / per_point, rem = pos - p * per_point;
  const int bt = rem / nbf, bf = rem - bt * nbf;
  const int KC = g.Cp >> 6;
  // loader: piece q = tid + 256 i is eight channels (16 bytes) of operand row q / 8; rows past
  // the tensor repeat its last one (their sums are not stored)
  const int16_t *usrc[2], *vsrc[2];
  unsigned ldst[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int q = (int)threadIdx.x + 256 * i, row = q >> 3, seg = q & 7;
    const int k = min(bf * BL + row, g.Kp - 1), t = min(bt * BL + row, g.Tp - 1);
    usrc[i] = U + ((size_t)p * g.Kp + k) * g.Cp + 8 * seg;
    vsrc[i] = V + ((size_t)p * g.Tp + t) * g.Cp + 8 * seg;
    ldst[i] = (unsigned)(row * PITCH + 8 * seg);
  }
  v4i ureg[2], vreg[2];
  auto load_regs = [&](int kc) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      ureg[i] = *(const v4i*)(usrc[i] + 64 * kc);
      vreg[i] = *(const v4i*)(vsrc[i] + 64 * kc);
    }
  };
  auto store_lds = [&](int buf) {
    unsigned char* b = lds + buf * (4 * PLANE);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      v2i lo, hi;
      split_i16(ureg[i], lo, hi);
      *(v2i*)(b + ldst[i]) = lo;
      *(v2i*)(b + PLANE + ldst[i]) = hi;
      split_i16(vreg[i], lo, hi);
      *(v2i*)(b + 2 * PLANE + ldst[i]) = lo;
      *(v2i*)(b + 3 * PLANE + ldst[i]) = hi;
    }
  };
  v4i ll[2][2], mid[2][2], hh[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) ll[i][j] = mid[i][j] = hh[i][j] = v4i{0, 0, 0, 0};
  const unsigned a_lane = (unsigned)((wm * 32 + (lane & 15)) * PITCH + (lane >> 4) * 16);
  const unsigned b_lane = 2u * PLANE + (unsigned)((wn * 32 + (lane & 15)) * PITCH + (lane >> 4) * 16);
  load_regs(0);
  store_lds(0);
  __syncthreads();
  for (int kc = 0; kc < KC; ++kc) {
    const unsigned char* b = lds + (kc & 1) * (4 * PLANE);
    if (kc + 1 < KC) load_regs(kc + 1);
    v4i al[2], ah[2], bl[2], bh[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      al[i] = *(const v4i*)(b + a_lane + i * 16 * PITCH);
      ah[i] = *(const v4i*)(b + a_lane + PLANE + i * 16 * PITCH);
      bl[i] = *(const v4i*)(b + b_lane + i * 16 * PITCH);
      bh[i] = *(const v4i*)(b + b_lane + PLANE + i * 16 * PITCH);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        ll[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al[i], bl[j], ll[i][j], 0, 0, 0);
        mid[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al[i], bh[j], mid[i][j], 0, 0, 0);
        hh[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ah[i], bh[j], hh[i][j], 0, 0, 0);
        mid[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ah[i], bl[j], mid[i][j], 0, 0, 0);
      }
    if (kc + 1 < KC) store_lds((kc + 1) & 1);
    __syncthreads();
  }
  // lane: filter quad lane / 16 of block i, tile lane % 16 of block j: 16 contiguous bytes of M
  const int kquads = g.Kp >> 2;
  int32_t* mp = M + (size_t)p * g.Tp * g.Kp;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int tb = bt * (BL / 16) + wn * 2 + j;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int kq = bf * (BL / 4) + wm * 8 + i * 4 + (lane >> 4);
      if (tb * 16 < g.Tp && kq < kquads) {
        v4i m;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          m[e] = (int)(((unsigned)hh[i][j][e] << 16) + ((unsigned)mid[i][j][e] << 8) + (unsigned)ll[i][j][e]);
        *(v4i*)(mp + ((size_t)tb * kquads + kq) * 64 + (lane & 15) * 4) = m;
      }
    }
  }
}

hipError_t launch_product_exact(const Geometry& g, const void* V, const void* U, int32_t* M, hipStream_t s) {
  const int nbt = (g.Tp + kExactBlock - 1) / kExactBlock, nbf = (g.Kp + kExactBlock - 1) / kExactBlock;
  const long long total = (long long)g.P * nbt * nbf;
  if (total > 0x7fffffffll) return hipErrorNotSupported;
  hipLaunchKernelGGL(product_gemm_i16_kernel, dim3((unsigned)total), dim3(256), 0, s, (const int16_t*)V,
                     (const int16_t*)U, M, g, nbt, nbf);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Output transform: the arrangement of output_sums_kernel (sfc_gemm.hip; lane = one pair, a
// ring of loads of M ahead, streaming transform, rows out through LDS) on unsigned integers:
// everything modulo 2^32, the division by kDen exact (a shift, and a multiplication by the
// inverse of 9 modulo 2^32 for the SFC-6 forms).
// ---------------------------------------------------------------------------------------
template <int ALG>
constexpr int exact_waves() { return AlgTraits<ALG>::NC <= 8 ? 8 : 4; }

template <int ALG, bool VEC2>
__global__ __launch_bounds__(exact_waves<ALG>() * 64) void output_exact_kernel(
    const int32_t* __restrict__ M, const float* __restrict__ wscale, float x_scale, int sums_out,
    void* __restrict__ y, Geometry g) {
  using Tr = AlgTraits<ALG>;
  constexpr int P = Tr::P, Mo = Tr::M, NC = Tr::NC, NW = exact_waves<ALG>(), D = NC <= 8 ? 16 : 24;
  constexpr Order<ALG> order{};
  __shared__ __align__(16) float stage_all[NW * 64 * Mo];
  __shared__ int tile_tab[48];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // workgroup -> (tile block, group of 4 NW filters), the filter group fastest
  const int kgroups = (g.Cout + 4 * NW - 1) / (4 * NW);
  const int pos = xcd_contiguous(blockIdx.x, gridDim.x);
  const int tb = pos / kgroups, kq = (pos - tb * kgroups) * NW + wave;
  const int kcol = kq * 4 + (lane >> 4);
  if (threadIdx.x < 16) {
    const int tl = threadIdx.x, t = tb * 16 + tl;
    const int per = g.th * g.tw;
    const int n = t / per, rem = t - n * per;
    const int ti = rem / g.tw, tj = rem - ti * g.tw;
    write_tile_entry<Mo>(tile_tab, tl, t < g.T, n, ti, tj, g.Cout, g.H, g.W);
  }
  __syncthreads();
  const unsigned mplane = (unsigned)g.Tp * (unsigned)g.Kp * 4u;
  const __amdgpu_buffer_rsrc_t mres =
      __builtin_amdgcn_make_buffer_rsrc((void*)M, 0, (int)(mplane * (unsigned)P), kBufferFlags);
  const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc(
      y, 0, (int)(4u * (unsigned)(g.N * g.Cout) * (unsigned)(g.H * g.W)), kBufferFlags);
  // filters beyond the padded count read nothing (zeros) and store nothing
  const bool kvalid = kcol < g.Kp;
  const unsigned m_lane =
      kvalid ? (unsigned)((tb * (g.Kp >> 2) + kq) * 64 + (lane & 15) * 4 + (lane >> 4)) * 4u : 0x80000000u;
  const float scale = x_scale * (kvalid ? wscale[kcol] : 0.0f);
  unsigned ring[D];
  auto load_point = [&](int j) {
    ring[j % D] = (unsigned)__builtin_amdgcn_raw_buffer_load_b32(mres, m_lane, (unsigned)order.pt[j] * mplane, 0);
  };
#pragma unroll
  for (int j = 0; j < D && j < P; ++j) load_point(j);
  int j = 0;  // folds to a constant after unrolling
  auto next = [&]() -> unsigned {
    unsigned v = ring[j % D];
    asm volatile("" : "+v"(v));  // the slot is free from here on
    if (j + D < P) load_point(j + D);
    ++j;
    return v;
  };
  unsigned z[NC][Mo];
  stream_vertical<ALG, unsigned>(next, z);
  store_pairs_as<ALG, 0, VEC2>(
      z, stage_all + wave * (64 * Mo), tile_tab, lane, kq,
      [=](unsigned v) {
        int acc;  // v / kDen, exact
        if constexpr (Tr::kDen == 16) acc = (int)v >> 4;
        else acc = (int)((unsigned)((int)v >> 2) * 0x38E38E39u);
        return sums_out ? __int_as_float(acc) : (float)acc * scale;
      },
      1.0f, yres, g.Cout, g.H, g.W);
}

template <int ALG>
static hipError_t launch_output_exact_alg(bool sums_out, const Geometry& g, const int32_t* M,
                                          const float* wscale, float x_scale, void* y, hipStream_t s) {
  constexpr int NW = exact_waves<ALG>();
  const dim3 grid((unsigned)(g.Tp / 16) * (unsigned)((g.Cout + 4 * NW - 1) / (4 * NW)));
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(NW * 64), 0, s, M, wscale, x_scale, sums_out ? 1 : 0, y, g);
    return hipGetLastError();
  };
  if constexpr (AlgTraits<ALG>::M % 2 == 0) {
    if (g.W % 2 == 0) return launch(output_exact_kernel<ALG, true>);
  }
  return launch(output_exact_kernel<ALG, false>);
}

// Where the kernel above is ahead of the one-thread-per-pair one (output_transform_kernel,
// sfc_kernels.hip), which asks for all sums of a pair at once and has few idle threads where
// there are few filters.  A wave here keeps a ring of sums in flight: 14.4 us of a lone workgroup
// with 88 points against 6.0 there.  The lines are in full waves of pairs, from 2158 layers (with
// the better kernel each time 0.89 of the time with this one alone); us of a layer here against
// there, waves: difference,
//   64 filters and more, even widths (two outputs per store)   88 points 400: +0.5, 800: -0.5, 1152: -7;
//       132 4: -0.3, 64: -1.2, 1024: -11; 46 392: +0.6, 512: -0.2, 1024: -1.8; 184 (5x5 filters)
//       18: +1.4, 50: -1.5, 800: -6; 184 (7x7) 128: +0.8, 196: -0.8, 1024: -5
//   odd widths   88 points 1024: +5.0, 1536: -7.7; 132 16: +0.5, 64: -0.1, 1024: -3.1; 46 512: +0.9, 768: +0.3,
//       1024: -0.5; 184 (5x5) 512: +3.3, 768: -2.5; 184 (7x7) 512: +1.9, 768: -0.5
//   16 to 63, where that kernel reads M in longer pieces   88 points 800: +3.8, 3200: -12; 132 576: +0.6,
//       2048: -13; 46 512: +2.4, 1568: -0.8; 184 (5x5) 2000: +8, 3200: -16; 184 (7x7) 1568: +1.9, 6272: -24
//   9 to 15   88 points 1200: +2, 2814: -2; 132 1800: +1, 3072: -4; 46 2520: +1, 5514: -3; 184 +0.6 to +53
//   8 and less   that kernel (8 filters, 46 points, 6272: +7; 184 points +74)
bool output_exact_ahead(const Geometry& g) {
  constexpr int kNever = 1 << 30;
  constexpr int kWaves[5][4] = {  // [alg / 2][9 to 15 filters; 16 to 63; more, even; more, odd width]
      {2560, 1025, 768, 1200}, {2560, 768, 0, 48}, {4096, 1024, 512, 768},
      {kNever, 2560, 48, 640}, {kNever, 4096, 160, 640}};
  const long long pairs = (long long)g.T * ((g.Cout + 3) / 4 * 4);
  return g.Cout > 8 && pairs >= 64ll * kWaves[g.alg >> 1][g.Cout < 16 ? 0 : g.Cout < 64 ? 1 : 2 + g.W % 2];
}

hipError_t launch_output_exact(bool sums_out, const Geometry& g, const int32_t* M, const float* wscale,
                               float x_scale, void* y, hipStream_t s) {
  const long long mbytes = 4ll * g.P * g.Tp * g.Kp, ybytes = 4ll * g.N * g.Cout * g.H * g.W;
  if (mbytes >= (1ll << 31) || ybytes >= (1ll << 31)) return hipErrorNotSupported;  // 32-bit offsets
  if (!output_exact_ahead(g)) return hipErrorNotSupported;
  switch (g.alg) {
    case 0: return launch_output_exact_alg<0>(sums_out, g, M, wscale, x_scale, y, s);
    case 1: return launch_output_exact_alg<1>(sums_out, g, M, wscale, x_scale, y, s);
    case 2: return launch_output_exact_alg<2>(sums_out, g, M, wscale, x_scale, y, s);
    case 3: return launch_output_exact_alg<3>(sums_out, g, M, wscale, x_scale, y, s);
    case 4: return launch_output_exact_alg<4>(sums_out, g, M, wscale, x_scale, y, s);
    case 5: return launch_output_exact_alg<5>(sums_out, g, M, wscale, x_scale, y, s);
    case 6: return launch_output_exact_alg<6>(sums_out, g, M, wscale, x_scale, y, s);
    case 7: return launch_output_exact_alg<7>(sums_out, g, M, wscale, x_scale, y, s);
    case 8: return launch_output_exact_alg<8>(sums_out, g, M, wscale, x_scale, y, s);
    case 9: return launch_output_exact_alg<9>(sums_out, g, M, wscale, x_scale, y, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace sfc
