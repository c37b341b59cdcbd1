// The whole hot path of the SFC-4(4x4,3x3) forms in one kernel for layers with up to 128 input
// channels (gfx950): input-tile transform, transform-domain products and output transform
// without V or M ever leaving the compute unit.
//
// A workgroup owns a rectangle of up to 16 tiles (S strips x tlw tile columns, or whole small
// images; sfc_tile_input.hpp), all input channels (one or two chunks of 64) and 64 filters per
// chunk.  A wave takes a group of 16 channels up to V and a group of 16 filters from V on:
//  1. Stage: the six input rows of every strip go to LDS with dword loads, lanes running along
//     the row, padding halo zero-filled.  No barrier: the wave's patches are in the channels it
//     staged itself.
//  2. Input transform (sfc_mfma_input.hpp), V[position][chunk][tile][channel] (1 KiB per (position,
//     chunk) = one MFMA operand) over the staging area.  LDS holds 32 positions; the others stay
//     packed in registers and take the place of the first ones when those have been multiplied.
//  3. Products + output transform: four (tile, filter) pairs per lane (sfc_quad16.hpp): V from LDS,
//     filter operand and dequantization factors from global memory (asked for before V is
//     written), the 16 outputs of a pair kept (stream_outputs4).
//  4. Store: the wave's 16 x 16 x 16 outputs go through its LDS block (over V, once every
//     wave is done with it) and out as whole tile rows, four image rows of 16 tiles per filter
//     and instruction.
//
// What bounds it: a workgroup is a chain of phases, each at the latency of something else (memory,
// instruction issue at 5 clocks a wave, the 64 bytes a clock at which the filter operand, 188 KB for
// 64 channels, comes to a compute unit), and no unit is busy for more than two thirds of the
// time; so what counts is the number of workgroups side by side and the length of the chain.
// 34 KB of LDS and 128 registers let four workgroups of one chunk (two of two chunks, 67 KB) share
// a compute unit; with all 46 positions in LDS, 24 partial outputs a pair and 150 registers it were
// three (one).  us per layer before and after: 64 channels on 56x56 maps, batch 64, int8 21.0 ->
// 19.3, float32 25.1 -> 20.8; on 224x224 maps, batch 32, int8 151 -> 142; 128 channels on 28x28 maps,
// batch 128, int8 34.5 -> 26.1, 112x112 maps, batch 16, 63.8 -> 51.3.  With 49 points, which need more
// registers (single16_waves), three (one) instead of two (one): 25.1 -> 22.9, 26.9 -> 24.4; 175 -> 146;
// 37.0 -> 32.9, 68.9 -> 64.6.
// Layers of few workgroups: single16_few.
#include <cstring>

#include "sfc_device.hpp"
#include "sfc_internal.hpp"
#include "sfc_mfma_input.hpp"
#include "sfc_points.hpp"
#include "sfc_quad16.hpp"
#include "sfc_tile_input.hpp"

namespace sfc {

// waves per group of 16 filters
__host__ __device__ constexpr int single16_halves(int kc, bool few) { return few && kc == 1 ? 2 : 1; }
// LDS of a wave behind the products: its outputs on their way out (16 filters in int8, eight in
// float32), and with two waves per filter group first the partial outputs it hands over
__host__ __device__ constexpr unsigned single16_wave_bytes(int nh, int out) {
  return out != 2 ? 8192u : nh == 1 ? 4096u : (unsigned)kQuad16HalfBytes;
}
// V in LDS: a ring of 32 positions, the ones behind them stay in registers as packed bytes until
// the first have been multiplied; with two waves per filter group all of them
__host__ __device__ constexpr int single16_ring(int nh, int pp) { return nh == 1 ? 32 : pp; }

// Waves per SIMD that the registers are cut for.  49 points take 30 to 50 registers more than 46 (the
// complex column group leaves three products a row, 52 positions of V one block more): cut for four waves
// they spilled 86 to 115.  One chunk fits three workgroups to a compute unit, 168 registers, or one of
// eight waves (FEW); two chunks one, as more than 128 registers leave two waves.
__host__ __device__ constexpr int single16_waves(int alg, int kc, bool few) {
  return alg == 5 ? (kc == 1 && !few ? 3 : 2) : few && kc == 2 ? 2 : 4;
}

// Filter-operand blocks ahead (quad16_stream) with 128 registers: as many as the partial outputs of
// the moment leave room for.  (A constant 4: 64 channels on 56x56 maps, batch 32, float32 13.5 us a
// layer against 13.3; 8 to 10 ahead until position 32 spilled, 14.4.)  Two chunks put 6 to 10 values in
// scratch however few blocks are ahead: two from the start, the others, outputs, where the late V is
// written, each stored and loaded once in some 12000 instructions; with 256 registers there are none, and
// 128 channels on 28x28 maps, batch 128, int8, took 30.1 us against 26.1.
template <int KC>
struct Single16Ahead {
  static constexpr int at(int s) { return KC == 1 ? (s < 25 ? 8 : s < 32 ? 6 : 4) : (s < 36 ? 4 : s < 50 ? 6 : s < 64 ? 4 : 3); }
};
// (49 points, one chunk: 6; 8 spilled 8 to 10 registers)
template <int ALG, int KC, bool FEW>
using Single16Blocks = std::conditional_t<(ALG == 5 && KC == 1), ConstantAhead<6>,
                                          std::conditional_t<(ALG == 5 || FEW), ConstantAhead<16>, Single16Ahead<KC>>>;

struct Single16Plan {
  TileRect tr;
  int fgroups;         // groups of 16 filters in all; a workgroup takes one per wave
  unsigned row_bytes;  // rectangle: LDS bytes of a staged row (tile columns + 2 dwords)
  unsigned cs;         // LDS bytes of a channel: six rows and a dword, or a channel plane of an image
  unsigned chunk_in;   // LDS bytes of one staged 64-channel chunk
  unsigned tab_off;    // LDS byte offset of the tile table
  unsigned lds_bytes;
  int few;             // single16_few
  // reciprocals (16 fractional bits, exact for tile slots) of the tile columns of a strip, or of the
  // tiles of an image and its tile columns
  unsigned per_row, per_image;
};

// Stages the six rows of every strip for the NCH channels from c0 on: `dst` is their LDS block
// of strip 0.  One instruction covers four rows x 16 dwords of a channel (RG = 2 of them a strip),
// or, where a row has at most ten dwords, all six rows (RG = 1); lanes past the last dword or row
// repeat it (the same bytes to the same place), lanes outside the image get an offset outside the
// buffer, for which the load returns zero.  NB: strips in flight together.  TAIL: rows that are not whole dwords; a dword that straddles the end of a row keeps
// its valid bytes, one that would reach past the tensor is fetched byte by byte.  Channels beyond
// Cin re-read the last one (their filter operand is zero).
template <int ALG, int NCH, int RG, int NB, bool TAIL>
__device__ __forceinline__ void stage_channels(const int8_t* __restrict__ x, unsigned char* dst,
                                                 const Geometry& g, const Single16Plan& sp, int strip0,
                                                 int tj0, int c0, int lane) {
  constexpr int M = AlgTraits<ALG>::M, NI = AlgTraits<ALG>::NI, PAD = AlgTraits<ALG>::PAD;
  static_assert(NI == 6, "row groups");
  constexpr unsigned kOutOfRange = 0x80000000u;
  const int W = g.W, H = g.H, HW = H * W;
  const unsigned xbytes = (unsigned)(g.N * g.Cin) * (unsigned)HW;
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc((void*)x, 0, (int)xbytes, kBufferFlags);
  const int lrow = RG == 1 ? lane / 10 : lane >> 4;
  const int dcol = min(RG == 1 ? lane - 10 * lrow : lane & 15, sp.tr.tlw + 1);
  const int col = M * tj0 - 4 + 4 * dcol;  // image column of the lane's dword
  const int nvalid = col < 0 ? 0 : min(4, max(0, W - col));
  const unsigned bmask = nvalid >= 4 ? 0xffffffffu : ((1u << (8 * nvalid)) - 1u);
  int row[RG];
  unsigned laddr[RG];
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    row[rg] = min(4 * rg + lrow, NI - 1);
    laddr[rg] = (unsigned)row[rg] * sp.row_bytes + 4u * (unsigned)dcol;
  }
  for (int s0 = 0; s0 < sp.tr.S; s0 += NB) {
    unsigned vals[NB][RG][NCH];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int strip = strip0 + s0 + b;
      const bool live = s0 + b < sp.tr.S && strip < g.strips;
      const int n = strip_image(sp.tr, strip);
      const int hlo = M * (strip - n * g.th) - PAD;
      const int base = (n * g.Cin * H + hlo) * W;
#pragma unroll
      for (int rg = 0; rg < RG; ++rg) {
        const bool ok = live && nvalid > 0 && (unsigned)(hlo + row[rg]) < (unsigned)H;
        const unsigned voff = ok ? (unsigned)(base + row[rg] * W + col) : kOutOfRange;
#pragma unroll
        for (int ci = 0; ci < NCH; ++ci) {
          const int c = min(c0 + ci, g.Cin - 1);
          const unsigned plane = (unsigned)c * (unsigned)HW;
          unsigned v = __builtin_amdgcn_raw_buffer_load_b32(xres, voff, plane, 0);
          if constexpr (TAIL) {
            v &= bmask;
            if (n == g.N - 1 && c == g.Cin - 1) {  // (maps of one or two samples are whole images)
              if (ok && voff + plane + 4u > xbytes) {
                v = 0;
                for (int bb = 0; bb < nvalid; ++bb)
                  v |= (unsigned)__builtin_amdgcn_raw_buffer_load_b8(xres, voff + bb, plane, 0) << (8 * bb);
              }
            }
          }
          vals[b][rg][ci] = v;
        }
      }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b)
      if (s0 + b < sp.tr.S) {
        unsigned char* d = dst + (unsigned)(s0 + b) * 64u * sp.cs;
#pragma unroll
        for (int rg = 0; rg < RG; ++rg)
#pragma unroll
          for (int ci = 0; ci < NCH; ++ci) *(unsigned*)(d + (unsigned)ci * sp.cs + laddr[rg]) = vals[b][rg][ci];
      }
  }
}

// The same for whole images: the planes of NCH channels of the workgroup's images, as they lie in
// memory (stage_images of sfc_tile_input.hpp for one wave's channels).
template <int NCH>
__device__ __forceinline__ void stage_planes(const int8_t* __restrict__ x, unsigned char* dst, const Geometry& g,
                                               const Single16Plan& sp, int bx, int c0, int lane) {
  const int HW = g.H * g.W;
  const unsigned xbytes = (unsigned)(g.N * g.Cin) * (unsigned)HW;
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc((void*)x, 0, (int)xbytes, kBufferFlags);
  const int dpc = (HW + 3) >> 2;  // dwords per plane
  int lpc = 64 / NCH;             // lanes per plane: an instruction covers at most the NCH planes
  while (lpc < dpc && lpc < 64) lpc <<= 1;
  const int cpi = 64 / lpc;               // planes per instruction
  const int ipp = (dpc + 63) >> 6;        // instructions per plane (1 unless dpc > 64)
  const int per_image = (NCH / cpi) * ipp;
  const int total = sp.tr.ipw * per_image;
  const int sub = lane / lpc, dw_lane = lane - sub * lpc;
  constexpr int BATCH = 16;  // loads in flight before the first LDS write
  for (int k0 = 0; k0 < total; k0 += BATCH) {
    unsigned vals[BATCH];
    int to[BATCH];
#pragma unroll
    for (int kk = 0; kk < BATCH; ++kk) {
      const int k = k0 + kk;
      const int slot = k / per_image, rem = k - slot * per_image;
      const int cgrp = rem / ipp, piece = rem - cgrp * ipp;
      const int c = cgrp * cpi + sub, dw = piece * 64 + dw_lane;
      const int n = bx * sp.tr.ipw + slot;
      const bool ok = k < total && n < g.N && dw < dpc;
      const unsigned off = (unsigned)((n * g.Cin + min(c0 + c, g.Cin - 1)) * HW + 4 * dw);
      unsigned v = 0;
      if (ok) {
        if (off + 4u <= xbytes) {
          v = __builtin_amdgcn_raw_buffer_load_b32(xres, off, 0, 0);
        } else {
          for (unsigned bb = 0; off + bb < xbytes; ++bb)
            v |= (unsigned)__builtin_amdgcn_raw_buffer_load_b8(xres, off + bb, 0, 0) << (8 * bb);
        }
      }
      vals[kk] = v;
      to[kk] = ok ? (int)((unsigned)(slot * 64 + c) * sp.cs) + 4 * dw : -1;
    }
#pragma unroll
    for (int kk = 0; kk < BATCH; ++kk)
      if (to[kk] >= 0) *(unsigned*)(dst + to[kk]) = vals[kk];
  }
}

// FEW: for layers of few workgroups, whose duration is one workgroup's chain (single16_few).  One
// chunk: two waves to a group of 16 filters, and of 16 channels.  Two chunks: 256 registers and the
// filter operand further ahead, one workgroup to a compute unit instead of two.
template <int ALG, int KC, int OUT, int EV, bool FEW>
__global__ __launch_bounds__(single16_halves(KC, FEW) * KC * 256, single16_waves(ALG, KC, FEW)) void single16_kernel(
    const int8_t* __restrict__ x, const int8_t* __restrict__ U16, const float* __restrict__ dq16,
    const unsigned char* __restrict__ intab, float x_scale, float inv_y, void* __restrict__ y,
    Geometry g, Single16Plan sp) {
  using Tr = AlgTraits<ALG>;
  constexpr int M = Tr::M;
  constexpr int PP = Order<ALG>::PP;
  constexpr int NH = single16_halves(KC, FEW);
  constexpr int NG = 4 * KC;  // groups of 16 filters of a workgroup, and of 16 channels
  constexpr int RING = single16_ring(NH, PP);
  // bytes of V per position: KC operand blocks of 1 KiB and 16 bytes that put the 16 positions
  // a wave writes at once into different LDS banks
  constexpr int VS = KC * 1024 + 16;
  extern __shared__ __align__(16) unsigned char lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = NH == 1 ? 0 : wave / NG, group = wave - half * NG;
  const TileRect& tr = sp.tr;
  const int bx = xcd_contiguous(blockIdx.x, gridDim.x);
  int* tile_tab = (int*)(lds + sp.tab_off);
  MfmaInput<ALG> mi;
  mi.load(intab, lane);  // (used behind the staging)

  // ---- 1. stage: the waves of a group of 16 channels their own, so that with one wave nothing waits
  // for other waves -------------------------------------------------------------------------
  const int kc = group >> 2, cg = group & 3, c0 = 16 * group;
  // (16: plane patches are read from up to 4 bytes early)
  unsigned char* in = lds + 16 + kc * sp.chunk_in + 16 * cg * sp.cs;
  const bool channels = c0 < g.Cin;  // groups of channels that do not exist: any V will do
  if (channels) {
    constexpr int NCH = 16 / NH;
    unsigned char* dst = in + half * NCH * sp.cs;
    const int cs = c0 + half * NCH;
    if (tr.whole) {
      stage_planes<NCH>(x, dst, g, sp, bx, cs, lane);
    } else {
      const int chunk = bx % tr.chunks, strip0 = (bx / tr.chunks) * tr.S, tj0 = chunk * tr.tlw;
      if (g.W % 4 != 0) stage_channels<ALG, NCH, 2, 1, true>(x, dst, g, sp, strip0, tj0, cs, lane);
      else if (tr.tlw <= 8) stage_channels<ALG, NCH, 1, 2, false>(x, dst, g, sp, strip0, tj0, cs, lane);
      else stage_channels<ALG, NCH, 2, 1, false>(x, dst, g, sp, strip0, tj0, cs, lane);
    }
  }
  if (threadIdx.x < 16) {
    const TileCoord tc = tile_coord(g, tr, bx, threadIdx.x);
    write_tile_entry<M>(tile_tab, threadIdx.x, tc.live, tc.n, tc.ti, tc.tj, g.Cout, g.H, g.W);
  }
  if constexpr (NH > 1) __syncthreads();
  else wave_lds_order();  // a patch was staged by other lanes of its wave

  // ---- 2. input transform (sfc_mfma_input.hpp) --------------------------------------------
  // A patch is (tile, group of 16 channels); the waves of a group take every NH-th tile.  All
  // patches are transformed, rounded and packed in registers before the first byte of V is
  // written, because V lies over the staged rows.
  constexpr int NPB = MfmaInput<ALG>::NPB;
  constexpr int NQ = 16 / NH;  // tile slots of a wave
  unsigned packed[NQ][NPB];
  if (channels) {
    // Lane l: LDS bytes from the wave's first channel to the patch of tile slot l (to its first row and
    // dword, or to its image), slots beyond the last tile repeat it; whole images: image row and
    // column of the patch's first sample, 16 bits each.
    const int tl = min(lane & 15, tr.ntiles - 1);
    int patch, origin = 0;
    if (tr.whole) {
      const int img = (int)(((unsigned)tl * sp.per_image) >> 16), rem = tl - img * (g.th * g.tw);
      const int ti = (int)(((unsigned)rem * sp.per_row) >> 16), tj = rem - ti * g.tw;
      patch = img * 64 * (int)sp.cs;
      origin = (M * ti - Tr::PAD) * 65536 + ((M * tj - Tr::PAD) & 0xffff);
    } else {
      const int s = (int)(((unsigned)tl * sp.per_row) >> 16);
      patch = s * 64 * (int)sp.cs + 4 * (tl - s * tr.tlw);
    }
    // Software pipeline: the LDS reads of patch q + 2 and the matrix instructions of patch
    // q + 1 are issued before patch q is rounded, so neither latency is waited for.  (An empty
    // tile slot repeats the last tile: its bytes are not written.)
    auto run = [&](auto whole_images) __attribute__((always_inline)) {
      constexpr bool kWhole = decltype(whole_images)::value;
      // lane = (channel, patch rows 2 rp and 2 rp + 1); the patch starts at byte 3 of its first dword
      const int rp = min(lane >> 4, 2);
      const unsigned char* lane_in = in + (unsigned)(lane & 15) * sp.cs + (unsigned)(2 * rp) * sp.row_bytes;
      auto fetch = [&](int q) __attribute__((always_inline)) -> v4i {  // q folds to a constant
        const int off = __builtin_amdgcn_readlane(patch, NH * q + half);
        if constexpr (kWhole) {
          const int at = __builtin_amdgcn_readlane(origin, NH * q + half);
          return MfmaInput<ALG>::operand_plane(in + off, (int)sp.cs, 0, at >> 16, (int)(short)at, g.H, g.W, lane);
        } else {
          v4i a;
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            const unsigned* src = (const unsigned*)(lane_in + off + (unsigned)r * sp.row_bytes);
            const unsigned d0 = src[0], d1 = src[1], d2 = src[2];
            a[2 * r] = (int)__builtin_amdgcn_alignbyte(d1, d0, 3);
            a[2 * r + 1] = (int)__builtin_amdgcn_alignbyte(d2, d1, 3);
          }
          return a;
        }
      };
      v4i d_cur[NPB], d_nxt[NPB];
      v4i a_nxt = fetch(0);
      mi.sums(a_nxt, d_cur);
      a_nxt = fetch(1);
      // (one exit behind the last tile: the values under way are not merged again)
      auto step = [&](auto&& self, auto qc) __attribute__((always_inline)) -> void {
        constexpr int q = decltype(qc)::value;
        if (NH * q < tr.ntiles) {
          if (q + 1 < NQ) mi.sums(a_nxt, d_nxt);
          if (q + 2 < NQ) a_nxt = fetch(q + 2);
          __builtin_amdgcn_sched_barrier(0);  // reads and matrix instructions go first
          mi.round(d_cur, g.qmax, packed[q]);
          // (made here and not where V is written, with its halves kept until then)
#pragma unroll
          for (int m = 0; m < NPB; ++m) asm volatile("" : "+v"(packed[q][m]));
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int m = 0; m < NPB; ++m) d_cur[m] = d_nxt[m];
          if constexpr (q + 1 < NQ) self(self, std::integral_constant<int, q + 1>{});
        }
      };
      step(step, std::integral_constant<int, 0>{});
    };
    if (tr.whole) run(std::true_type{});
    else run(std::false_type{});
  }
  // V of positions 16 m .. 16 m + 15 (an empty tile slot keeps stale bytes: they only reach
  // products of that slot, which are never stored)
  auto write_v = [&](int m) __attribute__((always_inline)) {
    const int pos = 16 * m + (lane & 15);
    unsigned char* dst = lds + (pos % RING) * VS + kc * 1024 + half * 64 + 16 * cg + 4 * (lane >> 4);
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      if (channels && NH * q + half < tr.ntiles && (16 * m + 16 <= PP || pos < PP))
        *(unsigned*)(dst + NH * q * 64) = packed[q][m];
  };
  auto ready = [&]() __attribute__((always_inline)) {
    __syncthreads();  // every patch has been read: the staging area becomes V
#pragma unroll
    for (int m = 0; m < NPB && 16 * m < RING; ++m) write_v(m);
    __syncthreads();
  };

  // ---- 3. products + output transform, 4. store ------------------------------------------
  const __amdgpu_buffer_rsrc_t ures = __builtin_amdgcn_make_buffer_rsrc(
      (void*)U16, 0, (int)((unsigned)sp.fgroups * (unsigned)(PP * KC * 1024)), kBufferFlags);
  const __amdgpu_buffer_rsrc_t dres = __builtin_amdgcn_make_buffer_rsrc(
      (void*)dq16, 0, (int)((unsigned)sp.fgroups * (unsigned)(PP * 64)), kBufferFlags);
  constexpr unsigned esz = OUT == 2 ? 1u : 4u;
  const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc(
      y, 0, (int)(esz * (unsigned)(g.N * g.Cout) * (unsigned)(g.H * g.W)), kBufferFlags);
  // groups beyond the last one read zeros (offsets outside the operand) and store nothing
  const int fg = blockIdx.y * NG + group;
  const unsigned a_wave = (unsigned)fg * (unsigned)(PP * KC * 1024), d_wave = (unsigned)fg * (unsigned)(PP * 64);
  // (EV = 0: the width of a store is chosen here, the kernel is not compiled once for each)
  auto store_ev = [&](auto&& store) __attribute__((always_inline)) {
    if constexpr (EV != 0) store(std::integral_constant<int, EV>{});
    else if (g.W % 4 == 0) store(std::integral_constant<int, 4>{});
    else if (g.W % 2 == 0) store(std::integral_constant<int, 2>{});
    else store(std::integral_constant<int, 1>{});
  };
  if constexpr (NH == 1) {
    f4 out[M][M];
    constexpr int kLate = (PP - RING) / 4;  // groups of four positions behind the ring's
    quad16_stream<ALG, KC, RING / 4, VS, Single16Blocks<ALG, KC, FEW>>(
        lds, lane, ures, a_wave, dres, d_wave, ready,
        [&](int pg) __attribute__((always_inline)) {
          if (pg == kLate - 1) {  // every wave has read the positions whose place the late ones take
            __syncthreads();
#pragma unroll
            for (int m = RING / 16; m < NPB; ++m) write_v(m);
          }
          if (pg == RING / 4 - 1) __syncthreads();
        },
        [&](auto& next) __attribute__((always_inline)) { stream_outputs4<ALG, f4>(next, SettleF4{}, out); });
    __syncthreads();  // the staging blocks take the place of V
    unsigned char* stage = lds + wave * single16_wave_bytes(NH, OUT);
    constexpr int NP = OUT == 2 ? 4 : 2;  // (float32: eight filters at a time)
#pragma unroll
    for (int i0 = 0; i0 < 4; i0 += NP)
      store_ev([&](auto ev) __attribute__((always_inline)) {
        quad16_store<kOutputColumns + M, OUT, decltype(ev)::value, NP>(out, stage, tile_tab, lane, fg * 4 + i0, x_scale,
                                                                       inv_y, yres, g, i0);
      });
  } else {
    unsigned char* mine = lds + wave * single16_wave_bytes(NH, OUT);
    unsigned char* theirs = lds + (half == 0 ? wave + NG : wave - NG) * single16_wave_bytes(NH, OUT);
    auto finish = [&](auto which) __attribute__((always_inline)) {
      constexpr int HALF = decltype(which)::value;
      f4 zz[6][4];
      quad16_half<ALG, KC, PP / 4, VS, HALF, ConstantAhead<8>>(
          lds, lane, ures, a_wave, dres, d_wave, ready, [](int) {}, [] { __syncthreads(); }, mine, theirs, zz);
      // (the other wave's block is this wave's alone once it has been read)
      store_ev([&](auto ev) __attribute__((always_inline)) {
        quad16_store<ALG, OUT, decltype(ev)::value, 2>(zz, theirs, tile_tab, lane, fg * 4 + 2 * HALF, x_scale, inv_y, yres, g);
      });
    };
    if (half == 0) finish(std::integral_constant<int, 0>{});
    else finish(std::integral_constant<int, 1>{});
  }
}

// Coefficients of the input transform by processing position, from the add networks: the
// image of every unit patch under fwd_input (rows, then columns) and for_each_point.
template <int ALG>
static void fill_input_table(const float* inv_sx, unsigned char* tab) {
  using Tr = AlgTraits<ALG>;
  constexpr int NI = Tr::NI, NC = Tr::NC;
  constexpr Order<ALG> order{};
  float* inv_pos = reinterpret_cast<float*>(tab);
  signed char* coeff = reinterpret_cast<signed char*>(tab) + kInputTabRows * 4;
  std::memset(tab, 0, kInputTabBytes);
  for (int p = 0; p < Tr::P; ++p) inv_pos[order.pos[p]] = inv_sx[p];
  int* point = reinterpret_cast<int*>(tab + kInputTabPoints);
  for (int j = 0; j < kInputTabRows; ++j) point[j] = j < Order<ALG>::PP ? order.pt[j] : -1;
  for (int i = 0; i < NI; ++i)
    for (int j = 0; j < NI; ++j) {
      int half[NI][NC], comp[NC][NC];
      for (int r = 0; r < NI; ++r) {
        int row[NI] = {};
        if (r == i) row[j] = 1;
        fwd_input<NI, NC>(row, half[r]);
      }
      for (int b = 0; b < NC; ++b) {
        int colv[NI], cc[NC];
        for (int r = 0; r < NI; ++r) colv[r] = half[r][b];
        fwd_input<NI, NC>(colv, cc);
        for (int a = 0; a < NC; ++a) comp[a][b] = cc[a];
      }
      for_each_point<ALG>(comp, [&](int p, int v) { coeff[order.pos[p] * 64 + 8 * i + j] = (signed char)v; });
    }
}

// The same for the row form (sfc_input_rows.hip): k = 16 i + j.
template <int ALG>
static void fill_rows_table(const float* inv_sx, unsigned char* tab) {
  using Tr = AlgTraits<ALG>;
  constexpr int NI = Tr::NI, NC = Tr::NC;
  constexpr Order<ALG> order{};
  static_assert(NI <= 12 && Order<ALG>::PP <= kRowsTabRows, "three steps of four rows, table rows");
  std::memset(tab, 0, kRowsTabBytes);
  float* inv_pos = reinterpret_cast<float*>(tab);
  int* point = reinterpret_cast<int*>(tab + kRowsTabPoint);
  signed char* coeff = reinterpret_cast<signed char*>(tab) + kRowsTabCoeff;
  for (int p = 0; p < Tr::P; ++p) inv_pos[order.pos[p]] = inv_sx[p];
  for (int j = 0; j < kRowsTabRows; ++j) point[j] = j < Order<ALG>::PP ? order.pt[j] : -1;
  for (int i = 0; i < NI; ++i)
    for (int j = 0; j < NI; ++j) {
      int half[NI][NC], comp[NC][NC];
      for (int r = 0; r < NI; ++r) {
        int row[NI] = {};
        if (r == i) row[j] = 1;
        fwd_input<NI, NC>(row, half[r]);
      }
      for (int b = 0; b < NC; ++b) {
        int colv[NI], cc[NC];
        for (int r = 0; r < NI; ++r) colv[r] = half[r][b];
        fwd_input<NI, NC>(colv, cc);
        for (int a = 0; a < NC; ++a) comp[a][b] = cc[a];
      }
      for_each_point<ALG>(comp, [&](int p, int v) { coeff[order.pos[p] * 192 + 16 * i + j] = (signed char)v; });
    }
}

void build_rows_table(int alg, const float* inv_sx, unsigned char* tab) {
  switch (alg) {
    case 0: fill_rows_table<0>(inv_sx, tab); break;
    case 1: fill_rows_table<1>(inv_sx, tab); break;
    case 2: fill_rows_table<2>(inv_sx, tab); break;
    case 3: fill_rows_table<3>(inv_sx, tab); break;
    case 4: fill_rows_table<4>(inv_sx, tab); break;
    case 5: fill_rows_table<5>(inv_sx, tab); break;
    case 6: fill_rows_table<6>(inv_sx, tab); break;
    case 7: fill_rows_table<7>(inv_sx, tab); break;
    case 8: fill_rows_table<8>(inv_sx, tab); break;
    case 9: fill_rows_table<9>(inv_sx, tab); break;
    default: std::memset(tab, 0, kRowsTabBytes);
  }
}

void build_input_table(int alg, const float* inv_sx, unsigned char* tab) {
  if (alg == 4) fill_input_table<4>(inv_sx, tab);
  else if (alg == 5) fill_input_table<5>(inv_sx, tab);
  else std::memset(tab, 0, kInputTabBytes);
}

// LDS of a rectangle's staged rows for 64 channels
static unsigned single16_stage_bytes(const TileRect& tr) {
  return (unsigned)tr.S * 64u * (6u * 4u * (unsigned)(tr.tlw + 2) + 4u);
}

// Few workgroups (the kernel's FEW): one chunk while all of them are resident with eight waves each
// (int8, 64 channels on 56x56 maps, 16 / 32 / 40 / 64 images, 224 / 448 / 560 / 896 workgroups: 8.9 /
// 12.0 / 16.8 / 21.4 us a layer against 10.2 / 13.2 / 15.8 / 19.6 with four), with 49 points, in whose
// registers two such workgroups do not share a compute unit, while every one has its own (2 / 16 / 32
// images, 28 / 224 / 448 workgroups: 9.2 / 9.5 / 17.0 against 10.8 / 11.1 / 14.4); two chunks likewise (46
// points, 128 channels on 28x28 maps, 32 / 64 / 80 / 128 images, 112 / 224 / 280 / 448 workgroups: 15.7 /
// 16.2 / 29.8 / 30.1 us against 16.3 / 17.3 / 24.8 / 26.2 with 128 registers; 49 points have one form).
static bool single16_few(const Geometry& g, long long workgroups) {
  if (g.alg == 5 && g.Cp > 64) return false;
  return workgroups <= (g.alg == 4 && g.Cp == 64 ? 512 : 256);
}

static bool make_single16_plan(const Geometry& g, int out, Single16Plan* sp) {
  if ((g.alg != 4 && g.alg != 5) || (g.Cp != 64 && g.Cp != 128)) return false;
  const int kc = g.Cp / 64;
  const unsigned pp = (unsigned)((g.P + 3) / 4 * 4);
  const unsigned lds_max = 160u * 1024u - 256u;
  TileRect& tr = sp->tr;
  if (!make_tile_rect(g, (lds_max - 16u) / (unsigned)kc, &tr)) return false;
  sp->row_bytes = tr.whole ? 0u : 4u * (unsigned)(tr.tlw + 2);
  sp->cs = tr.whole ? (unsigned)tr.cs : 6u * sp->row_bytes + 4u;  // (an odd number of dwords)
  sp->chunk_in = tr.whole ? tile_rect_stage_bytes(g, tr) : single16_stage_bytes(tr);
  auto reciprocal = [](int d) { return (unsigned)((65536 + d - 1) / d); };
  sp->per_row = reciprocal(tr.whole ? g.tw : tr.tlw);
  sp->per_image = reciprocal(g.th * g.tw);
  sp->fgroups = (g.Cout + 15) / 16;
  const long long wgs = (long long)tile_rect_groups(g, tr) * ((sp->fgroups + 4 * kc - 1) / (4 * kc));
  sp->few = single16_few(g, wgs) ? 1 : 0;
  const int nh = single16_halves(kc, sp->few != 0);
  const unsigned vbytes = (unsigned)single16_ring(nh, (int)pp) * ((unsigned)kc * 1024u + 16u);
  const unsigned sbytes = (unsigned)(4 * kc * nh) * single16_wave_bytes(nh, out);
  // (8: the last patch rows of a plane are read up to 8 bytes past it)
  unsigned top = 16u + sp->chunk_in * (unsigned)kc + 8u;
  if (vbytes > top) top = vbytes;
  if (sbytes > top) top = sbytes;
  sp->tab_off = (top + 15u) & ~15u;
  sp->lds_bytes = sp->tab_off + 256u;
  const long long xb = (long long)g.N * g.Cin * g.H * g.W;
  const long long yb = 4ll * g.N * g.Cout * g.H * g.W;
  const long long ub = (long long)sp->fgroups * 16 * pp * g.Cp;
  const long long lim = 1ll << 31;
  return sp->lds_bytes <= 160u * 1024u && xb < lim && yb < lim && ub < lim;
}

bool single16_supported(const Geometry& g) {
  Single16Plan sp;
  return make_single16_plan(g, 0, &sp);
}

bool single16_few_workgroups(const Geometry& g) {
  Single16Plan sp;
  return make_single16_plan(g, 0, &sp) && sp.few;
}

template <int ALG, int KC, int OUT, int EV, bool FEW>
static hipError_t launch_single16_impl(const Geometry& g, const Single16Plan& sp, const int8_t* x,
                                       const FilterViews& f, float x_scale, float inv_y, void* y,
                                       hipStream_t s, bool prepare) {
  auto kernel = single16_kernel<ALG, KC, OUT, EV, FEW>;
  if (prepare) return raise_lds_limit(reinterpret_cast<const void*>(kernel));
  const dim3 grid(tile_rect_groups(g, sp.tr), (unsigned)((sp.fgroups + 4 * KC - 1) / (4 * KC)));
  hipLaunchKernelGGL(kernel, grid, dim3(single16_halves(KC, FEW) * KC * 256), sp.lds_bytes, s, x, (const int8_t*)f.U_single,
                     f.dequant_single, f.input_tab, x_scale, inv_y, y, g, sp);
  return hipGetLastError();
}

template <int ALG, int KC, int OUT>
static hipError_t launch_single16_out(const Geometry& g, const Single16Plan& sp, const int8_t* x,
                                      const FilterViews& f, float x_scale, float inv_y, void* y,
                                      hipStream_t s, bool prepare) {
  if constexpr (ALG == 4 || KC == 1) {
    if (sp.few) return launch_single16_impl<ALG, KC, OUT, 0, true>(g, sp, x, f, x_scale, inv_y, y, s, prepare);
  }
  if (g.W % 4 == 0) return launch_single16_impl<ALG, KC, OUT, 4, false>(g, sp, x, f, x_scale, inv_y, y, s, prepare);
  if (g.W % 2 == 0) return launch_single16_impl<ALG, KC, OUT, 2, false>(g, sp, x, f, x_scale, inv_y, y, s, prepare);
  return launch_single16_impl<ALG, KC, OUT, 1, false>(g, sp, x, f, x_scale, inv_y, y, s, prepare);
}

template <int ALG, int KC>
static hipError_t launch_single16_kc(int out, const Geometry& g, const Single16Plan& sp,
                                     const int8_t* x, const FilterViews& f, float x_scale,
                                     float inv_y, void* y, hipStream_t s, bool prepare) {
  return out == 2 ? launch_single16_out<ALG, KC, 2>(g, sp, x, f, x_scale, inv_y, y, s, prepare)
                  : launch_single16_out<ALG, KC, 0>(g, sp, x, f, x_scale, inv_y, y, s, prepare);
}

hipError_t launch_single16(int out, const Geometry& g, const int8_t* x, const FilterViews& f,
                           float x_scale, float inv_y, void* y, hipStream_t s, bool prepare) {
  Single16Plan sp;
  if (out == 1 || !make_single16_plan(g, out, &sp)) return hipErrorNotSupported;
  if (g.alg == 4)
    return g.Cp == 64 ? launch_single16_kc<4, 1>(out, g, sp, x, f, x_scale, inv_y, y, s, prepare)
                      : launch_single16_kc<4, 2>(out, g, sp, x, f, x_scale, inv_y, y, s, prepare);
  return g.Cp == 64 ? launch_single16_kc<5, 1>(out, g, sp, x, f, x_scale, inv_y, y, s, prepare)
                    : launch_single16_kc<5, 2>(out, g, sp, x, f, x_scale, inv_y, y, s, prepare);
}

}  // namespace sfc
