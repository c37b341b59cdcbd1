// Transform-domain products + output transform with no surplus matrix work (gfx950), for the
// SFC-4(4x4,3x3) forms and SFC-6(4x4,7x7) with 184 points: a wave owns 16 tiles x 16 filters,
// four (tile, filter) pairs per lane.
//
// The int8 MFMA 16x16x64 gives lane l the four results D[4(l/16) + i][l%16], i = 0..3.  With
// the A operand holding ONE point for 16 filters (row r = filter f0 + 4(r%4) + r/4) and the B
// operand V of the same point for 16 tiles, every accumulator element is a wanted product:
// lane l gets, for tile l%16, the filters f0 + 4i + l/16 -- filter l/16 of the four filter
// quads f0/4 + i.  The 16 outputs of a pair are all that is kept from one product to the next
// (sfc_stream_outputs.hpp), so four pairs fit a lane's registers and the streaming output transform
// runs on four-element vectors.  Per product that is a quarter of the matrix instructions, LDS reads of V and
// filter-operand bytes of the one-pair-per-lane form (sfc_fused_quad.hpp), which spends three
// of four accumulator elements on mixed points.
#pragma once
#include <type_traits>

#include "sfc_device.hpp"
#include "sfc_internal.hpp"
#include "sfc_lane_values.hpp"
#include "sfc_points.hpp"
#include "sfc_stream_outputs.hpp"
#include "sfc_store.hpp"

namespace sfc {

// waves per workgroup of the fused kernel = groups of 16 filters per workgroup
constexpr int kQuad16Waves = 4;

// V buffers of the fused kernel (groups of four points in LDS) and groups in flight in
// registers behind them, by channel chunks: the load of a group is issued kVRegs groups
// before its products
// (seven chunks: two buffers, 56 KB, leave room for a second workgroup on the compute unit)
constexpr int quad16_vbufs(int kc) { return kc >= 7 ? 2 : 3; }
// (four chunks: three groups ahead, 256 channels on 14x14 maps at batch 128 38.2 us per layer
// against 39.8 with one; eight chunks leave no registers for more than one)
constexpr int quad16_vregs(int kc) { return kc >= 8 ? 1 : kc == 4 ? 3 : 2; }

// filter-operand blocks asked for ahead (SFC-4), where three and five chunks leave registers for more (209 and
// 228 of them): 184 to 136 channels, seven 31x45 maps, 25.7 us with eight, 25.3; 320 to 192 on 31 20x20 maps 25.8
// and 25.1; 0.97 to 1.01 of the time over 14 such layers.  Fourteen at four chunks: level (0.99 to 1.006)
constexpr int quad16_ahead(int kc) { return kc == 3 ? 16 : kc == 5 ? 12 : 8; }

// the int8 outputs take two scales (quad16_store's TWO; launch_quad16 says which two)
constexpr bool quad16_two_scales(int alg, int kc) { return alg == 4 && kc >= 3; }

// LDS of the products + output kernel: the V buffers, which the per-wave store staging
// blocks (16 filters x 16 tiles x 16 outputs, float32 or int8) take over once the last
// products are done, then the tile table.
template <int KC, int NW, int OUT>
constexpr unsigned quad16_lds_layout(int what) {
  constexpr unsigned vbytes = (unsigned)quad16_vbufs(KC) * 4u * 16u * 64u * KC;
  constexpr unsigned stage = NW * 4096u * (OUT == 2 ? 1u : 4u);
  constexpr unsigned tab_off = vbytes > stage ? vbytes : stage;
  return what == 0 ? 0u : what == 1 ? tab_off : tab_off + 256u;
}

// Between LDS accesses of different lanes of one wave.  The hardware completes them in order; the
// compiler follows one lane at a time and may swap a write and a read that it can tell apart for
// that lane.  Emits nothing.  (A wave barrier holds back the arithmetic too: at the head of quad16_store
// it made the float32 form of single16_kernel with two waves to a filter group spill 32 registers.)
__device__ __forceinline__ void wave_lds_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local"); }

// Filter-operand blocks that are on the way or held when block s is multiplied, s included.
template <int N>
struct ConstantAhead {
  static constexpr int at(int) { return N; }
};

// The products and the output transform of one wave: 16 tiles (V in LDS, groups of four
// points in a ring of buffers kept filled by `sync`) x 16 filters (operand and dequantization
// factors from global memory, a ring of loads ahead).
//   vbuf, VB      ring of VB buffers of 4 x KC blocks of 1 KiB ([point][chunk][tile][64 channels]);
//                 group pg lives in buffer pg % VB
//   ures, a_wave  filter operand: block (position j, chunk kc) at a_wave + (j*KC + kc) KiB,
//                 16 bytes per lane
//   dres, d_wave  dequantization factors: 16 floats per position at d_wave + 64 j, lane
//                 quarter l/16 takes four.  They are loaded once, 16 positions per
//                 instruction (lane (quarter, n) fetches those of position 16 m + n), and a
//                 product takes its factors from lane n of its quarter by a row broadcast: a
//                 load per position and wave instead kept the compute unit's vector-memory
//                 path busy with 64-byte pieces.
//   sync(pg)      called when the wave has read the last V of group pg (or issued its last
//                 products): returns once group pg + 1 is in place; it may overwrite the
//                 buffers of the groups before pg
// Software pipeline: call j issues the matrix instructions of position j + 1 and then converts
// the sums of position j, so the matrix pipe works under the vector arithmetic of the output
// transform.
//   ready()       called once, when the first loads from memory are under way and before V is read
//   Ahead         filter-operand blocks asked for by position: constant, or fewer while more partial
//                 outputs are kept
//   J0, J1        the positions asked for
//   consume(next) takes the products of the lane's four pairs (f4 element i: filter quad i) in
//                 processing order, next(integral_constant<int, j>) being position j
template <int ALG, int KC, int VB, int PS = KC * 1024, typename Ahead = ConstantAhead<8>, int J0 = 0,
          int J1 = Order<ALG>::PP, typename Ready, typename Sync, typename Consume>
__device__ __forceinline__ void quad16_stream(const unsigned char* vbuf, int lane,
                                              __amdgpu_buffer_rsrc_t ures, unsigned a_wave,
                                              __amdgpu_buffer_rsrc_t dres, unsigned d_wave,
                                              Ready&& ready, Sync&& sync, Consume&& consume) {
  constexpr int GROUP_BYTES = 4 * PS;      // PS: bytes from one position's V to the next
  constexpr int STEP0 = J0 * KC, STEPS = J1 * KC;  // filter-operand blocks of the wave
  constexpr int ND0 = J0 / 16, NDB = (J1 + 15) / 16;  // blocks of 16 positions' factors
  constexpr int DR = NDB - ND0 > 4 ? 2 : NDB - ND0;   // ... held at a time
  const unsigned a_lane = (unsigned)lane * 16u;
  const unsigned d_lane = (unsigned)(lane & 15) * 64u + (unsigned)(lane >> 4) * 16u;
  v4i aop[STEPS];  // (every index is a constant: a block lives from its load to its products)
  v4f dblk[DR];
  auto load_a = [&](int s) {
    aop[s] = __builtin_amdgcn_raw_buffer_load_b128(ures, a_lane, a_wave + (unsigned)s * 1024u, 0);
  };
  // blocks asked for by the time block s is multiplied: no fewer than before
  auto asked = [](int s) constexpr {
    int n = 0;
    for (int i = STEP0; i <= s; ++i) {
      int m = i + Ahead::at(i);
      if (m > STEPS) m = STEPS;
      if (m > n) n = m;
    }
    return n;
  };
  auto load_d = [&](int m) {  // (a last block may reach past the wave's table: never used)
    dblk[m % DR] = __builtin_bit_cast(
        v4f, __builtin_amdgcn_raw_buffer_load_b128(dres, d_lane, d_wave + (unsigned)m * 1024u, 0));
  };
#pragma unroll
  for (int m = ND0; m < ND0 + DR; ++m) load_d(m);
#pragma unroll
  for (int s = STEP0; s < asked(STEP0); ++s) load_a(s);
  ready();
  const unsigned char* blane = vbuf + (lane & 15) * 64 + (lane >> 4) * 16;
  // V of position jj for the lane's tile: KC reads of 16 bytes.  Up to two chunks they are
  // issued a call ahead of the matrix instructions that take them (PREB); with more the
  // chain of matrix instructions is long enough to read them as it goes.
  constexpr bool PREB = KC <= 2;
  constexpr int NB = PREB ? KC : 1;
  v4i breg[NB];
  auto read_b = [&](int jj) {
    const unsigned char* bsrc = blane + ((jj >> 2) % VB) * GROUP_BYTES + (jj & 3) * PS;
#pragma unroll
    for (int kc = 0; kc < NB; ++kc) breg[kc] = *(const v4i*)(bsrc + kc * 1024);
  };
  // the sums of position jj: KC chained matrix instructions
  auto products = [&](auto position) __attribute__((always_inline)) -> v4i {
    constexpr int jj = decltype(position)::value;
    v4i acc = {0, 0, 0, 0};
    const unsigned char* bsrc = blane + ((jj >> 2) % VB) * GROUP_BYTES + (jj & 3) * PS;
    static_for<KC>([&](auto kcc) __attribute__((always_inline)) {
      constexpr int kc = decltype(kcc)::value, s = jj * KC + kc;
      v4i b;
      if constexpr (PREB) b = breg[kc];
      else b = *(const v4i*)(bsrc + kc * 1024);
      acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(aop[s], b, acc, 0, 0, 0);
      constexpr int from = asked(s), to = s + 1 < STEPS ? asked(s + 1) : from;
      static_for<to - from>([&](auto n) __attribute__((always_inline)) { load_a(from + decltype(n)::value); });
    });
    return acc;
  };
  if constexpr (PREB) read_b(J0);
  v4i acc_cur = products(std::integral_constant<int, J0>{});
  if constexpr (PREB) read_b(J0 + 1);
  // (the streaming output transform asks for the products in order and names the position)
  auto next = [&](auto position) __attribute__((always_inline)) -> f4 {
    constexpr int j = decltype(position)::value;
    v4i acc_new = acc_cur;
    if constexpr (PREB) {
      if constexpr (j + 1 < J1) acc_new = products(std::integral_constant<int, j + 1>{});
      if (j + 2 < J1) {
        if (((j + 2) & 3) == 0) sync((j + 2) / 4 - 1);
        read_b(j + 2);
      }
    } else if constexpr (j + 1 < J1) {
      if (((j + 1) & 3) == 0) sync((j + 1) / 4 - 1);
      acc_new = products(std::integral_constant<int, j + 1>{});
    }
    __builtin_amdgcn_sched_barrier(0);  // the matrix instructions go first
    f4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float t = (float)acc_cur[i] * row_lane<j & 15>(dblk[(j >> 4) % DR][i]);
      // the scaled products are materialized here, the accumulator is not kept alive
      asm volatile("" : "+v"(t));
      v.v[i] = t;
    }
    if constexpr ((j & 15) == 15 && (j >> 4) + DR < NDB) load_d((j >> 4) + DR);
    acc_cur = acc_new;
    __builtin_amdgcn_sched_barrier(0);
    return v;
  };
  // positions P .. PP-1 hold no point: their filter operand is zero, their products unused
  consume(next);
}

// keeps the compiler from putting additions off and the products in registers instead
// (stream_outputs)
struct SettleF4 {
  __device__ __forceinline__ void operator()(f4& v) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(v.v[i]));
  }
};

// Two waves for one block of 16 tiles x 16 filters (SFC-4), cut by horizontal class: wave HALF = 0
// takes the complex column group and column 0 (components 2, 3, 0), HALF = 1 columns 1, 4 and 5.
// Together they do the work of one wave, each with half of its chain and half of its partial outputs
// (12 values of four pairs instead of 24).
template <int ALG, int HALF>
struct Quad16Half {
  static constexpr int kCut = complex4_positions<ALG>() + 7;
  static constexpr int J0 = HALF == 0 ? 0 : kCut, J1 = HALF == 0 ? kCut : AlgTraits<ALG>::P;
  static constexpr int comp(int i) { return HALF == 0 ? (i < 2 ? 2 + i : 0) : (i == 0 ? 1 : 3 + i); }
};
constexpr int kQuad16HalfBytes = 6 * 1024;  // what a wave hands to the other one

// The products of one half, its partial outputs exchanged: leaves z of the pairs 2 HALF, 2 HALF + 1
// (as elements 0 and 1) with all their components.  give, take: LDS blocks of kQuad16HalfBytes that
// this wave writes and the other one reads, and the other way round; meet() is called twice, all V
// read before the first and every block written before the second.
template <int ALG, int KC, int VB, int PS, int HALF, typename Ahead, typename Ready, typename Sync, typename Meet>
__device__ __forceinline__ void quad16_half(const unsigned char* vbuf, int lane, __amdgpu_buffer_rsrc_t ures,
                                            unsigned a_wave, __amdgpu_buffer_rsrc_t dres, unsigned d_wave,
                                            Ready&& ready, Sync&& sync, Meet&& meet, unsigned char* give,
                                            const unsigned char* take, f4 (&zz)[6][4]) {
  using Mine = Quad16Half<ALG, HALF>;
  using Other = Quad16Half<ALG, 1 - HALF>;
  Vertical4<f4> v[3];
  quad16_stream<ALG, KC, VB, PS, Ahead, Mine::J0, Mine::J1>(
      vbuf, lane, ures, a_wave, dres, d_wave, ready, sync, [&](auto& next) __attribute__((always_inline)) {
        SettleF4 settle;
        if constexpr (HALF == 0) {
          stream_complex4<ALG, f4>(next, settle, v[0], v[1]);
          stream_real4<ALG, 0, f4>(next, settle, v[2]);
        } else {
          stream_real4<ALG, 1, f4>(next, settle, v[0]);
          stream_real4<ALG, 2, f4>(next, settle, v[1]);
          stream_real4<ALG, 3, f4>(next, settle, v[2]);
        }
      });
  meet();
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int e = 2 * (1 - HALF) + i;
      *(v4f*)(give + ((c * 2 + i) * 64 + lane) * 16) =
          v4f{v[c].v[0].v[e], v[c].v[1].v[e], v[c].v[2].v[e], v[c].v[3].v[e]};
#pragma unroll
      for (int o = 0; o < 4; ++o) zz[Mine::comp(c)][o].v[i] = v[c].v[o].v[2 * HALF + i];
    }
  meet();
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const v4f t = *(const v4f*)(take + ((c * 2 + i) * 64 + lane) * 16);
#pragma unroll
      for (int o = 0; o < 4; ++o) zz[Other::comp(c)][o].v[i] = t[o];
    }
}

// y of the wave's 16 tiles x 16 filters from z (pair i of lane l: tile l%16, filter
// 4*(kq0 + i) + l/16).  Every lane finishes its 4 x 4 x 4 outputs (inverse along the horizontal
// axis, activation scale; OUT = 2: ReLU and rounding to the next layer's int8) and stages them
// in the wave's block as [filter 16][tile 16][row 4][4 outputs]; then lane l takes row l/16 of
// tile l%16 for one filter after the other, so that a store instruction writes, for one
// filter, four image rows of 16 neighbouring tiles: consecutive lanes hold consecutive
// pieces of an image row.  A piece outside the image gets an offset outside the buffer and is
// dropped by the bounds check; filters beyond Cout end the loop.
// NP, i0: pairs i0 .. i0 + NP - 1 of z alone, filters from 4 kq0 on (a block of 4 NP filters).
// EV: elements per store instruction, 4 when W is a multiple of 4 (a tile row never crosses
// the end of an image row), else 2 (W even) or 1.
// TWO (OUT = 2): an output takes x_scale and then inv_y, each with a rounding of its own, as
// store_pairs does; else their product.  The two round a tie of the int8 output differently.
template <int ALG, int OUT, int EV, int NP = 4, bool TWO = false>
__device__ __forceinline__ void quad16_store(const f4 (&z)[AlgTraits<ALG>::NC][AlgTraits<ALG>::M],
                                             unsigned char* stage, const int* tile_tab, int lane,
                                             int kq0, float x_scale, float inv_y,
                                             __amdgpu_buffer_rsrc_t yres, const Geometry& g, int i0 = 0) {
  constexpr int NC = AlgTraits<ALG>::NC, M = AlgTraits<ALG>::M;
  static_assert(M == 4, "tiles of 4 x 4 outputs");
  constexpr unsigned esz = OUT == 2 ? 1u : 4u;
  constexpr unsigned kOutOfRange = 0x80000000u;
  constexpr float kMagic = 12582912.0f;
  const int tl = lane & 15, q = lane >> 4;
  const float act = x_scale * inv_y;  // int8 output: activation scale over output scale
  // this lane's piece: row q of tile tl (asked for here, waited for behind the transform)
  const int tile_off = tile_tab[tl], tile_rows = tile_tab[16 + tl], tile_cols = tile_tab[32 + tl];
  wave_lds_order();  // (the block may have been read a moment ago: a store of other pairs, a hand-over)
  // float32 staging: 16-byte slots, slot (tile, row) of a filter moved round by tile/4 so
  // that the 16 lanes of a quarter wave fall into different banks, writing and reading
  auto slot = [](int tile, int row) { return tile * 4 + ((row + (tile >> 2)) & 3); };
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    float zi[NC][M];
#pragma unroll
    for (int b = 0; b < NC; ++b)
#pragma unroll
      for (int o = 0; o < M; ++o) zi[b][o] = z[b][o].v[i0 + i];
    const int f = 4 * i + q;
#pragma unroll
    for (int o1 = 0; o1 < M; ++o1) {
      float out[M];
      stream_row<ALG, float>(zi, o1, out);
      if constexpr (OUT == 2) {
        unsigned b[M];
#pragma unroll
        for (int o2 = 0; o2 < M; ++o2) {
          // next layer's activation: ReLU, round half to even, clamp to [0, 127]
          float t = TWO ? __fmaf_rn(out[o2] * x_scale, inv_y, kMagic) : __fmaf_rn(out[o2], act, kMagic);
          t = __builtin_amdgcn_fmed3f(t, kMagic, kMagic + 127.0f);
          b[o2] = __float_as_uint(t);
        }
        // the low bytes of the four outputs -> one dword
        const unsigned word = __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u) | __builtin_amdgcn_perm(b[3], b[2], 0x04000c0cu);
        // (rows moved round by the quarter: the four quarters of the wave write different banks)
        *(unsigned*)(stage + ((f * 16 + tl) * 4 + ((o1 + q) & 3)) * 4) = word;
      } else {
        *(v4f*)(stage + (f * 64 + slot(tl, o1)) * 16) =
            v4f{out[0] * x_scale, out[1] * x_scale, out[2] * x_scale, out[3] * x_scale};
      }
    }
  }
  wave_lds_order();
  const int HW = g.H * g.W;
  const int cols = q < tile_rows ? tile_cols : 0;
  const unsigned base = esz * (unsigned)(tile_off + q * g.W);  // filter 0
  // byte offsets of the lane's store pieces (filter 0; outside the buffer: dropped); a filter's
  // plane is the scalar offset of the store
  constexpr int NE = EV == 4 ? 1 : EV == 2 ? 2 : 4;
  unsigned piece[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) piece[e] = cols > EV * e ? base + esz * (unsigned)(EV * e) : kOutOfRange;
  const bool stream = g.W >= 48;  // whole long rows per workgroup: past the L2
  const int nk = min(4 * NP, g.Cout - 4 * kq0);  // filters of the wave that exist
  auto put = [&](auto policy, auto full) {
  constexpr int kPolicy = decltype(policy)::value ? kStreamStore : 0;
  constexpr int KB = OUT == 2 ? 4 * NP : 4;  // filters read from the block before the first is stored
#pragma unroll
  for (int k0 = 0; k0 < 4 * NP; k0 += KB) {
    unsigned word[OUT == 2 ? KB : 1];
    v4f quad[OUT == 2 ? 1 : KB];
#pragma unroll
    for (int kk = 0; kk < KB; ++kk) {
      const int k = k0 + kk;
      if constexpr (OUT == 2) word[kk] = *(const unsigned*)(stage + ((k * 16 + tl) * 4 + ((q + k) & 3)) * 4);
      else quad[kk] = *(const v4f*)(stage + (k * 64 + slot(tl, q)) * 16);
    }
#pragma unroll
    for (int kk = 0; kk < KB; ++kk) {
      const int k = k0 + kk;
      if (!decltype(full)::value && k >= nk) break;
      const unsigned plane = esz * (unsigned)(4 * kq0 + k) * (unsigned)HW;
      if constexpr (OUT == 2) {
        const unsigned w = word[kk];
        if constexpr (EV == 4) {
          __builtin_amdgcn_raw_buffer_store_b32(w, yres, piece[0], plane, kPolicy);
        } else if constexpr (EV == 2) {
          __builtin_amdgcn_raw_buffer_store_b16((unsigned short)w, yres, piece[0], plane, 0);
          __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(w >> 16), yres, piece[1], plane, 0);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            __builtin_amdgcn_raw_buffer_store_b8((unsigned char)(w >> (8 * e)), yres, piece[e], plane, 0);
        }
      } else {
        const v4f v = quad[kk];
        if constexpr (EV == 4) {
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, v), yres, piece[0], plane, kPolicy);
        } else if constexpr (EV == 2) {
          __builtin_amdgcn_raw_buffer_store_b64(v2f{v[0], v[1]}, yres, piece[0], plane, 0);
          __builtin_amdgcn_raw_buffer_store_b64(v2f{v[2], v[3]}, yres, piece[1], plane, 0);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[e]), yres, piece[e], plane, 0);
        }
      }
    }
  }
  };
  auto run = [&](auto policy) {
    if (nk >= 4 * NP) put(policy, std::true_type{});
    else if (nk > 0) put(policy, std::false_type{});
  };
  if (EV == 4 && stream) run(std::true_type{});
  else run(std::false_type{});
}

// Products + output transform with V from the input-transform kernel (fused path).  A
// workgroup of NW waves owns 16 consecutive tiles and 16*NW filters; per group of four points
// it copies 4 x 16 x Cin bytes of V from memory into one of two LDS buffers (already in
// operand order) while the previous group is multiplied, one barrier per group.
template <int ALG, int KC, int OUT, int EV, int NW>
__global__ __launch_bounds__(NW * 64, 2) void quad16_kernel(
    const int8_t* __restrict__ V, const int8_t* __restrict__ U16, const float* __restrict__ dq16,
    float x_scale, float inv_y, void* __restrict__ y, Geometry g, int fgroups) {
  using Tr = AlgTraits<ALG>;
  constexpr int P = Tr::P, M = Tr::M;
  constexpr int PP = Order<ALG>::PP, PG = PP / 4;
  constexpr int CP = KC * 64;
  constexpr int GROUP_BYTES = 4 * 16 * CP;
  constexpr int CHUNKS = GROUP_BYTES / 16;
  constexpr int NT = NW * 64;
  constexpr int NL = CHUNKS / NT;
  static_assert(NL * NT == CHUNKS, "every thread loads the same number of pieces of a group");
  constexpr Order<ALG> order{};
  extern __shared__ __align__(16) unsigned char lds[];
  unsigned char* vbuf = lds;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  unsigned char* stage = lds + wave * (4096 * (OUT == 2 ? 1 : 4));
  int* tile_tab = (int*)(lds + quad16_lds_layout<KC, NW, OUT>(1));

  // workgroup -> (tile block, group of NW*16 filters): the workgroups an XCD runs side by
  // side share tile blocks (filter group fastest), so V is fetched into its L2 once
  const int wgroups = fgroups / NW;  // filter groups of a workgroup's size
  const int pos = xcd_contiguous(blockIdx.x, gridDim.x);
  const int tb = pos / wgroups, kb = pos - tb * wgroups;
  const int t0 = tb * 16;
  const int fg = kb * NW + wave;  // this wave's group of 16 filters

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
      (void*)U16, 0, (int)((unsigned)fgroups * (unsigned)(PP * CP * 16)), kBufferFlags);
  const __amdgpu_buffer_rsrc_t dres = __builtin_amdgcn_make_buffer_rsrc(
      (void*)dq16, 0, (int)((unsigned)fgroups * (unsigned)(PP * 64)), kBufferFlags);
  constexpr unsigned esz = OUT == 2 ? 1u : 4u;
  const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc(
      y, 0, (int)(esz * (unsigned)(g.N * g.Cout) * (unsigned)(g.H * g.W)), kBufferFlags);

  // loader: piece q = tid + NT*i of a group is 16 bytes of (point r, tile, channels) with
  // r = q / (64*KC) uniform per wave; it lands in block r*KC + kc at [tile][16*kseg..]
  unsigned gsrc[NL], ldst[NL];
  int rsel[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int q = (int)threadIdx.x + NT * i;
    const int r = (wave * 64 + NT * i) / (64 * KC);  // uniform over the wave
    const int rem = q - r * (64 * KC);
    const int tile = rem / (4 * KC), ch = rem - tile * (4 * KC);
    rsel[i] = r;
    gsrc[i] = (unsigned)(t0 + tile) * (unsigned)CP + (unsigned)ch * 16u;
    ldst[i] = (unsigned)(((r * KC + (ch >> 2)) * 16 + tile) * 64 + (ch & 3) * 16);
  }
  // Group pg is loaded into register set pg % VR when group pg - VR has been handed to LDS,
  // and handed to LDS buffer pg % VB when the products of group pg - 1 have been issued; the
  // barrier after that also tells that every wave is done with group pg - 2, whose buffer
  // group pg + 1 will take (VB >= 2; with VB = 3 the store may run a group earlier).
  constexpr int VB = quad16_vbufs(KC), VR = quad16_vregs(KC);
  v4i lreg[VR][NL];
  // V offset of a piece's point.  With as many waves as channel chunks (256 channels) piece i of
  // every thread is point i of the group, a constant.  Else the offsets of the positions lie 64
  // to a register and a piece takes the one of its point by its lane number.  (Selected among
  // four constants, the loads of every group became branches with a copy of the load each, four
  // to a piece: 516 loads and 400 branches in the code at 128 channels and 184 points, 1067 and
  // 900 at 256.  256 channels on 14x14 maps, batch 128, layer: 38.4 us selected, 38.7 by lane,
  // 38.3 constant; the 13-layer stack at batch 64 363.9, 356.2, 355.5; over 84 layers of 129 to
  // 256 channels the constant takes 0.992 of the time of the selection, 0.93 to 1.03.)
  constexpr bool kPieceIsPoint = NT == 64 * KC;
  unsigned vofs[(PP + 63) / 64];
#pragma unroll
  for (int m = 0; m < (PP + 63) / 64; ++m) vofs[m] = (unsigned)max(order.pt[min(64 * m + lane, PP - 1)], 0) * vplane;
  auto load_regs = [&](int pg) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      unsigned off;
      if constexpr (kPieceIsPoint) off = (unsigned)max(order.pt[4 * pg + i], 0) * vplane;
      else off = (unsigned)__builtin_amdgcn_readlane((int)vofs[pg >> 4], ((4 * pg) & 63) + rsel[i]);
      lreg[pg % VR][i] = __builtin_amdgcn_raw_buffer_load_b128(vres, gsrc[i], off, 0);
    }
  };
  auto store_lds = [&](int pg) {
#pragma unroll
    for (int i = 0; i < NL; ++i) *(v4i*)(vbuf + (pg % VB) * GROUP_BYTES + ldst[i]) = lreg[pg % VR][i];
  };
#pragma unroll
  for (int pg = 0; pg < VR && pg < PG; ++pg) load_regs(pg);
  store_lds(0);
  if (VR < PG) load_regs(VR);
  __syncthreads();

  auto sync = [&](int pg) {  // the products of group pg are issued: bring in group pg + 1
    if (pg + 1 < PG) store_lds(pg + 1);
    if (pg + 1 + VR < PG) load_regs(pg + 1 + VR);
    __syncthreads();
  };
  const unsigned a_wave = (unsigned)fg * (unsigned)(PP * KC * 1024), d_wave = (unsigned)fg * (unsigned)(PP * 64);
  static_assert(M == 4, "tiles of 4 x 4 outputs");
  constexpr int COLS = kOutputColumns + M;
  f4 out[M][M];
  using Ahead = ConstantAhead<Tr::kFamily == 4 ? quad16_ahead(KC) : 8>;
  quad16_stream<ALG, KC, VB, KC * 1024, Ahead>(vbuf, lane, ures, a_wave, dres, d_wave, [] {}, sync,
                             [&](auto& next) __attribute__((always_inline)) {
                               if constexpr (Tr::kFamily == 4) stream_outputs4<ALG, f4>(next, SettleF4{}, out);
                               else stream_outputs<ALG, f4>(next, SettleF4{}, out);
                             });
  __syncthreads();  // the staging blocks take the place of the V buffers
  constexpr bool TWO = quad16_two_scales(ALG, KC);
  if constexpr (EV != 0) {
    quad16_store<COLS, OUT, EV, 4, TWO>(out, stage, tile_tab, lane, fg * 4, x_scale, inv_y, yres, g);
  } else {  // (the width of a store is chosen here, the products are not compiled once for each)
    if (g.W % 4 == 0) quad16_store<COLS, OUT, 4, 4, TWO>(out, stage, tile_tab, lane, fg * 4, x_scale, inv_y, yres, g);
    else if (g.W % 2 == 0) quad16_store<COLS, OUT, 2, 4, TWO>(out, stage, tile_tab, lane, fg * 4, x_scale, inv_y, yres, g);
    else quad16_store<COLS, OUT, 1, 4, TWO>(out, stage, tile_tab, lane, fg * 4, x_scale, inv_y, yres, g);
  }
}

}  // namespace sfc
