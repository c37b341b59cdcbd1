// Transform-domain products + output transform in one kernel for SFC-6(6x6,5x5) with 184 points
// (gfx950): a wave owns 16 tiles x 8 filters, two (tile, filter) pairs per lane.
//
// The int8 MFMA 16x16x64 gives lane l the four results D[4(l/16) + i][l%16], i = 0..3.  The A operand
// holds TWO points, one after the other in processing order, for 8 filters: row r = point r%2, filter
// f0 + 4((r%4)/2) + r/4.  With V of the first point as operand B elements 0 and 2 are the lane's own
// products, with V of the second 1 and 3: filters f0 + l/16 and f0 + 4 + l/16 of tile l%16.  The 36
// outputs of a pair are all that is kept from one product to the next (stream_outputs), 72 registers
// a lane; four pairs to a lane (sfc_quad16.hpp) do not fit.
//
// What bounds it: the issue of vector instructions and a barrier for every four points.  Against
// one pair per lane (sfc_fused_quad.hpp) the matrix instructions, reads of V and filter-operand bytes
// of a product are half, and the matrix instructions of one position run under the arithmetic of the
// one before, where all waves of a workgroup read V, multiplied and added at the same time.  128 channels
// on 28x28 maps, batch 64: 64.0 -> 31.5 us (layer 78.7 -> 44.9); over 80 layers of the range of the 5x5
// filters the layer takes 0.79 of the time (0.56 to 1.0; with 512 channels and eight waves, 0.79 to 1.08).  With one pair per lane neither deeper rings of V
// (1, 2, 4 groups) nor of the filter operand (2, 4, 8 blocks) had changed the 64 us.
#pragma once
#include "sfc_device.hpp"
#include "sfc_internal.hpp"
#include "sfc_lane_values.hpp"
#include "sfc_points.hpp"
#include "sfc_store.hpp"
#include "sfc_stream_outputs.hpp"

namespace sfc {

namespace pair16 {

// keeps a value that stays until a later product from being put off (stream_outputs)
struct SettleF2 {
  __device__ __forceinline__ void operator()(f2& v) const { asm volatile("" : "+v"(v.v[0]), "+v"(v.v[1])); }
};

// a piece (tile, 16 channels) of an operand block of V lies at tile*64 + 16*(segment ^ this): the 16-byte
// reads of the 64 lanes fall into different banks
__device__ __forceinline__ int v_swizzle(int tile) { return (4 - (tile >> 2)) & 3; }

}  // namespace pair16

constexpr int kAlg5Tap = 6;  // SFC_ALG_6X6_5X5_P184
// groups of four points of V in LDS, and on the way to it in registers
constexpr int pair16_vbufs(int kc) { return kc <= 4 ? 3 : 2; }
constexpr int pair16_vregs(int kc) { return kc <= 2 ? 2 : 1; }

// LDS: the V buffers, which the waves' staging blocks of the store (64 x 6 floats) take over once
// the last products are done, then the tile table.
template <int KC, int NW>
constexpr unsigned pair16_tab_off() {
  constexpr unsigned vbytes = (unsigned)pair16_vbufs(KC) * 4u * 16u * 64u * KC, stage = NW * 64u * 6u * 4u;
  return vbytes > stage ? vbytes : stage;
}

template <int KC, int OUT, int NW>
__global__ __launch_bounds__(NW * 64, 2) void pair16_kernel(
    const int8_t* __restrict__ V, const int8_t* __restrict__ U8, const float* __restrict__ dq8, float x_scale,
    float inv_y, void* __restrict__ y, Geometry g, int fgroups) {
  using namespace pair16;
  constexpr int ALG = kAlg5Tap;
  using Tr = AlgTraits<ALG>;
  constexpr int P = Tr::P, M = Tr::M, PG = P / 4;
  static_assert(P % 4 == 0, "whole groups of four points");
  constexpr int CP = KC * 64;
  constexpr int GROUP_BYTES = 4 * 16 * CP, CHUNKS = GROUP_BYTES / 16, NT = NW * 64;
  constexpr int NL = (CHUNKS + NT - 1) / NT;  // 16-byte pieces of a group per thread
  constexpr int VB = pair16_vbufs(KC), VR = pair16_vregs(KC);
  constexpr Order<ALG> order{};
  extern __shared__ __align__(16) unsigned char lds[];
  unsigned char* vbuf = lds;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int* tile_tab = (int*)(lds + pair16_tab_off<KC, NW>());

  // workgroup -> (tile block, group of 8 NW filters), the filter group fastest: the workgroups an
  // XCD runs side by side share tile blocks
  const int wgroups = fgroups / NW;
  const int pos = xcd_contiguous(blockIdx.x, gridDim.x);
  const int tb = pos / wgroups, kb = pos - tb * wgroups;
  const int t0 = tb * 16;
  const int fg = kb * NW + wave;  // this wave's group of 8 filters

  if (threadIdx.x < 16) {
    const int tl = threadIdx.x, t = t0 + tl;
    const int per = g.th * g.tw;
    const int n = t / per, rem = t - n * per;
    const int ti = rem / g.tw, tj = rem - ti * g.tw;
    write_tile_entry<M>(tile_tab, tl, t < g.T, n, ti, tj, g.Cout, g.H, g.W);
  }

  const unsigned vplane = (unsigned)g.Tp * (unsigned)CP;
  const __amdgpu_buffer_rsrc_t vres =
      __builtin_amdgcn_make_buffer_rsrc((void*)V, 0, (int)(vplane * (unsigned)P), kBufferFlags);
  const __amdgpu_buffer_rsrc_t ures = __builtin_amdgcn_make_buffer_rsrc(
      (void*)U8, 0, (int)((unsigned)fgroups * (unsigned)(P * CP * 8)), kBufferFlags);
  const __amdgpu_buffer_rsrc_t dres = __builtin_amdgcn_make_buffer_rsrc(
      (void*)dq8, 0, (int)((unsigned)fgroups * (unsigned)(P * 32)), kBufferFlags);
  constexpr unsigned esz = OUT == 2 ? 1u : 4u;
  const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc(
      y, 0, (int)(esz * (unsigned)(g.N * g.Cout) * (unsigned)(g.H * g.W)), kBufferFlags);

  // ---- V: piece q = tid + NT*i of a group is 16 bytes of (point r, tile, channels), r = q / (64*KC)
  // uniform over the wave; offsets of the positions lie 64 to a register, a piece takes the one of
  // its point by its lane number ---------------------------------------------------------------
  unsigned gsrc[NL], ldst[NL];
  int rsel[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int q = (int)threadIdx.x + NT * i;
    const int r = (wave * 64 + NT * i) / (64 * KC);
    const int rem = q - r * (64 * KC);
    const int tile = rem / (4 * KC), ch = rem - tile * (4 * KC);
    rsel[i] = r < 4 ? r : -1;
    gsrc[i] = (unsigned)(t0 + tile) * (unsigned)CP + (unsigned)ch * 16u;
    ldst[i] = (unsigned)(((r * KC + (ch >> 2)) * 16 + tile) * 64 + ((ch & 3) ^ v_swizzle(tile)) * 16);
  }
  unsigned vofs[(P + 63) / 64];
#pragma unroll
  for (int m = 0; m < (P + 63) / 64; ++m) vofs[m] = (unsigned)order.pt[min(64 * m + lane, P - 1)] * vplane;
  v4i lreg[VR][NL];
  auto load_regs = [&](int pg) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const unsigned off =
          (unsigned)__builtin_amdgcn_readlane((int)vofs[pg >> 4], ((4 * pg) & 63) + max(rsel[i], 0));
      if (NL * NT == CHUNKS || rsel[i] >= 0)
        lreg[pg % VR][i] = __builtin_amdgcn_raw_buffer_load_b128(vres, gsrc[i], off, 0);
    }
  };
  auto store_lds = [&](int pg) {
#pragma unroll
    for (int i = 0; i < NL; ++i)
      if (NL * NT == CHUNKS || rsel[i] >= 0) *(v4i*)(vbuf + (pg % VB) * GROUP_BYTES + ldst[i]) = lreg[pg % VR][i];
  };
#pragma unroll
  for (int pg = 0; pg < VR; ++pg) load_regs(pg);

  // ---- filter operand, one block per two positions and channel chunk, eight blocks ahead; factors
  // of 16 positions per instruction (lane (quarter, n) those of position 16 m + n for its quarter) ----
  constexpr int STEPS = P / 2 * KC, AHEAD = 8, NDB = (P + 15) / 16, DR = 2;
  const unsigned a_lane = (unsigned)lane * 16u, a_wave = (unsigned)fg * (unsigned)(P / 2 * KC * 1024);
  const unsigned d_lane = (unsigned)(lane & 15) * 32u + (unsigned)(lane >> 4) * 8u, d_wave = (unsigned)fg * (unsigned)(P * 32);
  v4i aop[STEPS];  // (every index is a constant: a block lives from its load to its products)
  v2f dblk[DR];
  auto load_a = [&](int s) {
    aop[s] = __builtin_amdgcn_raw_buffer_load_b128(ures, a_lane, a_wave + (unsigned)s * 1024u, 0);
  };
  auto load_d = [&](int m) {  // (the last block reaches past the wave's table: never used)
    dblk[m % DR] = __builtin_bit_cast(v2f, __builtin_amdgcn_raw_buffer_load_b64(dres, d_lane, d_wave + (unsigned)m * 512u, 0));
  };
#pragma unroll
  for (int m = 0; m < DR; ++m) load_d(m);
#pragma unroll
  for (int s = 0; s < AHEAD; ++s) load_a(s);
  store_lds(0);
  load_regs(VR);
  __syncthreads();
  // the products of group pg are issued: bring in group pg + 1
  auto sync = [&](int pg) {
    if (pg + 1 < PG) store_lds(pg + 1);
    if (pg + 1 + VR < PG) load_regs(pg + 1 + VR);
    __syncthreads();
  };

  const unsigned char* blane = vbuf + (lane & 15) * 64 + ((lane >> 4) ^ v_swizzle(lane & 15)) * 16;
  // Up to two chunks V is read a position ahead of the matrix instructions that take it.
  constexpr bool PREB = KC <= 2;
  constexpr int NB = PREB ? KC : 1;
  v4i breg[NB];
  auto read_b = [&](int jj) {
    const unsigned char* bsrc = blane + ((jj >> 2) % VB) * GROUP_BYTES + (jj & 3) * (KC * 1024);
#pragma unroll
    for (int kc = 0; kc < NB; ++kc) breg[kc] = *(const v4i*)(bsrc + kc * 1024);
  };
  auto products = [&](auto position) __attribute__((always_inline)) -> v4i {
    constexpr int jj = decltype(position)::value;
    v4i acc = {0, 0, 0, 0};
    const unsigned char* bsrc = blane + ((jj >> 2) % VB) * GROUP_BYTES + (jj & 3) * (KC * 1024);
    static_for<KC>([&](auto kcc) __attribute__((always_inline)) {
      constexpr int kc = decltype(kcc)::value, s = jj / 2 * KC + kc;
      v4i b;
      if constexpr (PREB) b = breg[kc];
      else b = *(const v4i*)(bsrc + kc * 1024);
      acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(aop[s], b, acc, 0, 0, 0);
      if constexpr (jj % 2 == 1 && s + AHEAD < STEPS) load_a(s + AHEAD);
    });
    return acc;
  };
  if constexpr (PREB) read_b(0);
  v4i acc_cur = products(std::integral_constant<int, 0>{});
  if constexpr (PREB) read_b(1);
  // Call j issues the matrix instructions of position j + 1 and then converts the sums of position j.
  auto next = [&](auto position) __attribute__((always_inline)) -> f2 {
    constexpr int j = decltype(position)::value;
    v4i acc_new = acc_cur;
    if constexpr (PREB) {
      if constexpr (j + 1 < P) acc_new = products(std::integral_constant<int, j + 1>{});
      if (j + 2 < P) {
        if (((j + 2) & 3) == 0) sync((j + 2) / 4 - 1);
        read_b(j + 2);
      }
    } else if constexpr (j + 1 < P) {
      if (((j + 1) & 3) == 0) sync((j + 1) / 4 - 1);
      acc_new = products(std::integral_constant<int, j + 1>{});
    }
    __builtin_amdgcn_sched_barrier(0);  // the matrix instructions go first
    f2 v;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      float t = (float)acc_cur[2 * e + (j & 1)] * row_lane<j & 15>(dblk[(j >> 4) % DR][e]);
      asm volatile("" : "+v"(t));  // the accumulator is not kept alive
      v.v[e] = t;
    }
    if constexpr ((j & 15) == 15 && (j >> 4) + DR < NDB) load_d((j >> 4) + DR);
    acc_cur = acc_new;
    __builtin_amdgcn_sched_barrier(0);
    return v;
  };
  f2 out[M][M];
  stream_outputs<ALG, f2>(next, SettleF2{}, out);
  __syncthreads();  // the staging blocks take the place of the V buffers
  float* stage = (float*)lds + wave * (64 * M);
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    float z[M][M];
#pragma unroll
    for (int a = 0; a < M; ++a)
#pragma unroll
      for (int b = 0; b < M; ++b) z[a][b] = out[a][b].v[e];
    if (g.W % 2 == 0) store_pairs<kOutputColumns + M, OUT, true>(z, stage, tile_tab, lane, 2 * fg + e, x_scale, inv_y, yres, g.Cout, g.H, g.W);
    else store_pairs<kOutputColumns + M, OUT, false>(z, stage, tile_tab, lane, 2 * fg + e, x_scale, inv_y, yres, g.Cout, g.H, g.W);
  }
}

// ---------------------------------------------------------------------------------------

// Waves of a workgroup, eight filters each.  Up to 128 workgroups of eight waves, half of the compute units have none: four
// waves then, twice the workgroups.  us with four over us with eight, explicit fused path, layers of one, two, four and
// eight chunks: up to 128 workgroups 0.85-0.90, 0.82-0.92, 0.74-0.86, 0.85-0.94 (at 128 with 512 filters 1.1), against
// one pair per lane 0.64 to 0.97, where eight waves took up to 1.02, 0.91, 0.99 and 1.08; above 160 0.9-1.05, 0.92-1.28,
// 0.93-1.56, 0.95-1.74.  Four as well where eight would leave half of them without a filter, or reach past the 32-bit
// offsets into the filter operand.
inline int pair16_waves(const Geometry& g) {
  const int groups = (g.Cout + 63) / 64;
  if (g.Cout <= 32 || (long long)(g.Tp / 16) * groups <= 128) return 4;
  return (long long)groups * 64 * g.P * g.Cp < (1ll << 31) ? 8 : 4;
}

template <int KC, int OUT, int NW>
inline hipError_t launch_pair16_impl(const Geometry& g, const void* V, const FilterViews& f, float x_scale,
                                     float inv_y, void* y, hipStream_t s, bool prepare) {
  auto kernel = pair16_kernel<KC, OUT, NW>;
  constexpr unsigned lds_bytes = pair16_tab_off<KC, NW>() + 256u;
  static_assert(lds_bytes <= 160u * 1024u, "V buffers exceed the LDS of a compute unit");
  if (prepare) return raise_lds_limit(reinterpret_cast<const void*>(kernel));
  const int fgroups = pair16_filter_count(g) / 8;
  const dim3 grid((unsigned)((g.Tp / 16) * (fgroups / NW)));
  hipLaunchKernelGGL(kernel, grid, dim3(NW * 64), lds_bytes, s, (const int8_t*)V, (const int8_t*)f.U_single,
                     f.dequant_single, x_scale, inv_y, y, g, fgroups);
  return hipGetLastError();
}

template <int KC>
inline hipError_t launch_pair16_kc(int out, const Geometry& g, const void* V, const FilterViews& f, float x_scale,
                                   float inv_y, void* y, hipStream_t s, bool prepare) {
  if (pair16_waves(g) == 8)
    return out == 2 ? launch_pair16_impl<KC, 2, 8>(g, V, f, x_scale, inv_y, y, s, prepare)
                    : launch_pair16_impl<KC, 0, 8>(g, V, f, x_scale, inv_y, y, s, prepare);
  return out == 2 ? launch_pair16_impl<KC, 2, 4>(g, V, f, x_scale, inv_y, y, s, prepare)
                  : launch_pair16_impl<KC, 0, 4>(g, V, f, x_scale, inv_y, y, s, prepare);
}

}  // namespace sfc
