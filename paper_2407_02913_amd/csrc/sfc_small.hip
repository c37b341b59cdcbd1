// SFC-4(4x4,3x3), Hermitian form, on small layers (gfx950): kernels built for the time of ONE
// workgroup, where a layer has fewer workgroups of the throughput kernels than the chip has
// compute units and its duration is a single chain of load, transform, multiply, store.  (An
// empty kernel takes 2.4 us of a stream of launches.)
//
// What such a chain costs in the throughput kernels (four waves per workgroup, one per SIMD: 64
// channels, one image of 56x56, 11.4 us) is instruction issue: a wave alone on its SIMD issues
// a vector instruction every 8 clocks, two or more waves share it at one every 4.  Here 16
// waves share the workgroup's phases, and a layer is cut into more workgroups.
//
//   single_small_kernel   whole path, up to 128 input channels
//   product_small_kernel  products + output transform from V, 256 and 512 input channels
//
// The first cuts the 46 positions of the processing order by horizontal class into seven parts
// of at most seven: the four real columns (positions 18..45), and of the complex column group the
// points kept from the nested form against real rows 0, 1 (6..11) and 5, 6 (12..17) and the
// Hermitian ones (0..5).  Every part leaves four partial outputs per (tile, filter) pair.
#include "sfc_device.hpp"
#include "sfc_internal.hpp"
#include "sfc_mfma_input.hpp"
#include "sfc_points.hpp"
#include "sfc_quad16.hpp"
#include "sfc_store.hpp"
#include "sfc_tile_input.hpp"

namespace sfc {

constexpr int kSmallWaves = 16;
constexpr int kSmallPatches = 4 * kSmallWaves;  // 16-channel patches of a workgroup at most
constexpr int kSmallAlg = 4;    // SFC_ALG_4X4_P46
constexpr int kParts = 7;
constexpr int kPartSlots = 7;  // positions of the largest part

__host__ __device__ constexpr int part_first(int part) { return part < 4 ? 18 + 7 * part : part == 6 ? 0 : 6 * (part - 3); }
__host__ __device__ constexpr int part_count(int part) { return part < 4 ? 7 : 6; }

// The products m[0..6] of one part -> four values: the vertical outputs of a real column (parts
// 0..3); of the two component columns of the complex group, the sum and difference of components
// 0 and 1 (part 4), four times components 4 and 5 (part 5), twice components 2 and 3 (part 6).
template <typename T>
__device__ __forceinline__ void part_outputs(int part, const T (&m)[kPartSlots], T (&z)[4]) {
  if (part < 4) {
    T cc[6];
    collapse4_rows(m, cc);
    inv4_outputs(cc, z);
  } else if (part < 6) {
    // rows a0 + a1, a1, a0 of two components
    const T a0 = m[2] - m[1], b0 = m[0] - m[2] - m[1];
    const T a1 = m[5] - m[4], b1 = m[3] - m[5] - m[4];
    if (part == 4) {
      z[0] = a0 + a1;
      z[1] = a0 - a1;
      z[2] = b0 + b1;
      z[3] = b0 - b1;
    } else {
      z[0] = T(4.0f) * a0;
      z[1] = T(4.0f) * a1;
      z[2] = T(4.0f) * b0;
      z[3] = T(4.0f) * b1;
    }
  } else {
    const T uo0 = m[0] - m[1], uo1 = m[2] - m[0] - m[1];
    const T vo0 = m[3] - m[4], vo1 = m[5] - m[3] - m[4];
    z[0] = uo0 + vo0;
    z[1] = uo1 + vo1;
    z[2] = uo1 - vo1;
    z[3] = vo0 - uo0;
  }
}

// Rows O0 .. O0 + ROWS - 1 of y of one pair per lane (tile lane % 16, filter kcol) from its
// vertical outputs z: row by row, 16 bytes (four with int8 output) per lane, tiles next to each
// other in lanes next to each other.  EV: elements per store, as in quad16_store.
template <int OUT, int EV, int O0, int ROWS>
__device__ __forceinline__ void store_pair_rows(const float (&z)[6][4], const int* tile_tab, int lane, int kcol,
                                                float x_scale, float inv_y, __amdgpu_buffer_rsrc_t yres,
                                                const Geometry& g) {
  constexpr unsigned esz = OUT == 2 ? 1u : 4u;
  constexpr unsigned kOutOfRange = 0x80000000u;
  constexpr float kMagic = 12582912.0f;
  const int tl = lane & 15;
  const int rows = kcol < g.Cout ? tile_tab[16 + tl] : 0, cols = tile_tab[32 + tl];
  const unsigned base = esz * (unsigned)(tile_tab[tl] + kcol * (g.H * g.W));
  const float act = x_scale * inv_y;
#pragma unroll
  for (int o1 = O0; o1 < O0 + ROWS; ++o1) {
    float out[4];
    stream_row<kSmallAlg, float>(z, o1, out);
    const unsigned off = base + esz * (unsigned)(o1 * g.W);
    const int ncol = o1 < rows ? cols : 0;
    if constexpr (OUT == 2) {
      unsigned b[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        // next layer's activation: ReLU, round half to even, clamp to [0, 127]
        float t = __fmaf_rn(out[e], act, kMagic);
        b[e] = __float_as_uint(__builtin_amdgcn_fmed3f(t, kMagic, kMagic + 127.0f));
      }
      const unsigned word = __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u) | __builtin_amdgcn_perm(b[3], b[2], 0x04000c0cu);
      if constexpr (EV == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(word, yres, ncol > 0 ? off : kOutOfRange, 0, 0);
      } else if constexpr (EV == 2) {
        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)word, yres, ncol > 0 ? off : kOutOfRange, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(word >> 16), yres, ncol > 2 ? off + 2u : kOutOfRange, 0, 0);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          __builtin_amdgcn_raw_buffer_store_b8((unsigned char)(word >> (8 * e)), yres,
                                               ncol > e ? off + (unsigned)e : kOutOfRange, 0, 0);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) out[e] *= x_scale;
      if constexpr (EV == 4) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, v4f{out[0], out[1], out[2], out[3]}), yres,
                                               ncol > 0 ? off : kOutOfRange, 0, 0);
      } else if constexpr (EV == 2) {
        __builtin_amdgcn_raw_buffer_store_b64(v2f{out[0], out[1]}, yres, ncol > 0 ? off : kOutOfRange, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b64(v2f{out[2], out[3]}, yres, ncol > 2 ? off + 8u : kOutOfRange, 0, 0);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(out[e]), yres,
                                                ncol > e ? off + 4u * (unsigned)e : kOutOfRange, 0, 0);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// Whole path in one kernel, up to 128 input channels.  The phases of single16_kernel
// (sfc_single16.hip): stage the input rows, transform on the matrix cores, V in LDS as MFMA
// operands, products; patches are dealt to 16 waves, only groups of 16 channels that exist are
// transformed (the filter operand of the others is zero), and the products of a group of 16
// filters go to seven waves, one per part, which exchange their partial outputs through LDS.
// Everything that does not depend on x (coefficients, the whole filter operand of a wave's part,
// factors) is requested before the staging.  A workgroup takes up to 16, 8, 4 or 2 tiles and one
// or two groups of 16 filters (make_small_plan).
// ---------------------------------------------------------------------------------------
struct SmallPlan {
  TileRect tr;
  int fgroups;        // groups of 16 filters in all
  int fper;           // ... per workgroup
  int cgroups;        // groups of 16 input channels
  unsigned chunk_in;  // LDS bytes of one staged 64-channel chunk
  unsigned tab_off;   // LDS byte offset of the tile table
  unsigned lds_bytes;
  double cost;
};

template <int KC, int OUT, int EV>
__global__ __launch_bounds__(kSmallWaves * 64) void single_small_kernel(
    const int8_t* __restrict__ x, const int8_t* __restrict__ U16, const float* __restrict__ dq16,
    const unsigned char* __restrict__ intab, float x_scale, float inv_y, void* __restrict__ y, Geometry g,
    SmallPlan sp) {
  constexpr int ALG = kSmallAlg, NW = kSmallWaves;
  using Tr = AlgTraits<ALG>;
  constexpr int M = Tr::M, PAD = Tr::PAD, PP = Order<ALG>::PP;
  constexpr int CS = stage_channel_bytes(Tr::NI);
  constexpr int VS = KC * 1024 + 16;  // bytes of V per position (sfc_single16.hip)
  constexpr int STEPS = kPartSlots * KC;  // filter operand blocks of a part
  extern __shared__ __align__(16) unsigned char lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const TileRect& tr = sp.tr;
  const int bx = blockIdx.x;
  int* tile_tab = (int*)(lds + sp.tab_off);
  if (threadIdx.x < 16) {
    const int tl = threadIdx.x;
    const TileCoord tc = tile_coord(g, tr, bx, tl);
    write_tile_entry<M>(tile_tab, tl, tc.live, tc.n, tc.ti, tc.tj, g.Cout, g.H, g.W);
    if (!tr.whole) {
      const int t = min(tl, tr.ntiles - 1), s = t / tr.tlw, tj0 = (bx % tr.chunks) * tr.tlw;
      const int halo = M * tj0 - PAD - ((M * tj0) & ~3) + 4;  // LDS byte of the rectangle's first patch column
      tile_tab[48 + tl] = s * 64 * CS + halo + M * (t - s * tr.tlw);
    }
  }
  // ---- this wave's filter group and part
  const int gi = wave >> 3, part = min(wave & 7, kParts - 1);
  const int fg = blockIdx.y * sp.fper + gi;
  const bool multiplies = gi < sp.fper && (wave & 7) < kParts;
  const int j0 = part_first(part);
  const __amdgpu_buffer_rsrc_t ures = __builtin_amdgcn_make_buffer_rsrc(
      (void*)U16, 0, (int)((unsigned)sp.fgroups * (unsigned)(PP * KC * 1024)), kBufferFlags);
  const __amdgpu_buffer_rsrc_t dres = __builtin_amdgcn_make_buffer_rsrc(
      (void*)dq16, 0, (int)((unsigned)sp.fgroups * (unsigned)(PP * 64)), kBufferFlags);
  const unsigned a_wave = (unsigned)(fg * PP + j0) * (unsigned)(KC * 1024);
  MfmaInput<ALG> mi;
  mi.load(intab, lane);
  v4i a[STEPS];
  auto load_a = [&](int s) {  // (the last position of a part of six is not used)
    a[s] = __builtin_amdgcn_raw_buffer_load_b128(ures, (unsigned)lane * 16u, a_wave + (unsigned)s * 1024u, 0);
  };
  v4f dq = {0.0f, 0.0f, 0.0f, 0.0f};
  if (multiplies) {
    // lane (quarter q, n): factors of position j0 + n for the filters 4 i + q
    dq = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(
                                     dres, (unsigned)(lane & 15) * 64u + (unsigned)(lane >> 4) * 16u,
                                     (unsigned)(fg * PP + j0) * 64u, 0));
#pragma unroll
    for (int s = 0; s < kPartSlots; ++s) load_a(s);
  }
  // ---- stage: with two chunks half of the waves take each
  {
    constexpr int NS = NW / KC;
    const int kc = KC == 1 ? 0 : wave / NS;
    stage_input<ALG, NS>(x, lds + 16 + kc * sp.chunk_in, g, tr, bx, 64 * kc, wave - kc * NS, lane);
  }
  if (multiplies) {  // (the rest of the operand: not before the staging's registers are free)
#pragma unroll
    for (int s = kPartSlots; s < STEPS; ++s) load_a(s);
  }
  __syncthreads();

  // ---- input transform: patch id = tile * cgroups + channel group, dealt to the waves; all
  // patches rounded and packed in registers before V goes over the staged rows
  {
    constexpr int NPB = MfmaInput<ALG>::NPB, NQ = 4;  // patches of a wave at most (kSmallPatches)
    const int npatch = tr.ntiles * sp.cgroups;
    unsigned packed[NQ][NPB];
    auto fetch = [&](int q) __attribute__((always_inline)) -> v4i {
      const int id = min(wave + NW * q, npatch - 1);
      const int tile = id / sp.cgroups, cg = id - tile * sp.cgroups;
      const unsigned char* in = lds + 16 + (cg >> 2) * sp.chunk_in;
      if (tr.whole) {
        const int tpi = g.th * g.tw;
        const int slot = tile / tpi, rem = tile - slot * tpi;
        const int ti = rem / g.tw, tj = rem - ti * g.tw;
        return MfmaInput<ALG>::operand_plane(in + slot * 64 * tr.cs, tr.cs, 16 * (cg & 3), M * ti - PAD,
                                             M * tj - PAD, g.H, g.W, lane);
      }
      return MfmaInput<ALG>::template operand_rect<CS>(in, 16 * (cg & 3),
                                                       __builtin_amdgcn_readfirstlane(tile_tab[48 + tile]), lane);
    };
    v4i a_cur = fetch(0);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      if (wave + NW * q < npatch) {
        v4i d[NPB];
        mi.sums(a_cur, d);
        if (q + 1 < NQ) a_cur = fetch(q + 1);
        mi.round(d, g.qmax, packed[q]);
      }
    }
    __syncthreads();  // every patch has been read: the staging area becomes V
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int id = wave + NW * q;
      if (id < npatch) {
        const int tile = id / sp.cgroups, cg = id - tile * sp.cgroups;
        unsigned char* dst = lds + (cg >> 2) * 1024 + tile * 64 + 16 * (cg & 3) + 4 * (lane >> 4);
#pragma unroll
        for (int m = 0; m < NPB; ++m) {
          const int pos = 16 * m + (lane & 15);
          if (pos < PP) *(unsigned*)(dst + pos * VS) = packed[q][m];
        }
      }
    }
  }
  __syncthreads();

  // ---- products of the wave's part, its partial outputs
  f4 z[4];
  if (multiplies) {
    const unsigned char* bsrc = lds + j0 * VS + (lane & 15) * 64 + (lane >> 4) * 16;
    f4 m[kPartSlots];
    static_for<kPartSlots>([&](auto jc) __attribute__((always_inline)) {
      constexpr int jj = decltype(jc)::value;
      v4i acc = {0, 0, 0, 0};
#pragma unroll
      for (int kc = 0; kc < KC; ++kc)  // (the seventh of a part of six is not used)
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[jj * KC + kc], *(const v4i*)(bsrc + jj * VS + kc * 1024), acc, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) m[jj].v[i] = (float)acc[i] * row_lane<jj>(dq[i]);
    });
    part_outputs(part, m, z);
  }
  __syncthreads();  // V has been read: the partial outputs take its place
  unsigned char* zx = lds + gi * (kParts * 4096) + lane * 16;  // [group][part][pair][lane] x 16 bytes
  if (multiplies) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *(v4f*)(zx + (part * 4 + i) * 1024) = v4f{z[0].v[i], z[1].v[i], z[2].v[i], z[3].v[i]};
  }
  __syncthreads();
  if (gi >= sp.fper) return;
  // wave (group, i, h) finishes rows 2 h and 2 h + 1 of the pairs of filter quad i
  const int i = wave & 3;
  v4f r[kParts];
#pragma unroll
  for (int p = 0; p < kParts; ++p) r[p] = *(const v4f*)(zx + (p * 4 + i) * 1024);
  float zz[6][4];
#pragma unroll
  for (int o = 0; o < 4; ++o) {
    zz[0][o] = r[0][o];
    zz[1][o] = r[1][o];
    zz[4][o] = r[2][o];
    zz[5][o] = r[3][o];
  }
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    zz[2 + b][0] = r[4][2 * b] + r[5][2 * b] - r[6][2 * b];
    zz[2 + b][1] = r[4][2 * b + 1] + r[6][2 * b + 1];
    zz[2 + b][2] = r[4][2 * b] + r[6][2 * b];
    zz[2 + b][3] = r[4][2 * b + 1] + r[5][2 * b + 1] - r[6][2 * b + 1];
  }
  constexpr unsigned esz = OUT == 2 ? 1u : 4u;
  const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc(
      y, 0, (int)(esz * (unsigned)(g.N * g.Cout) * (unsigned)(g.H * g.W)), kBufferFlags);
  const int kcol = fg * 16 + 4 * i + (lane >> 4);
  if ((wave & 4) == 0) store_pair_rows<OUT, EV, 0, 2>(zz, tile_tab, lane, kcol, x_scale, inv_y, yres, g);
  else store_pair_rows<OUT, EV, 2, 2>(zz, tile_tab, lane, kcol, x_scale, inv_y, yres, g);
}

// Tiles and filter groups of a workgroup: of the combinations whose workgroups all run at once
// (one per compute unit) the one with the least estimated time in us, less what all of them
// share.  The estimate is a fit to 2514 timings, every combination of 688 layers (16 to 128
// channels, 16 to 256 filters, maps from 5x5 to 224x224, 200x16 and 6x61, one image to the most that
// the kernel takes): 16-channel patches, a second filter group, workgroups (each fetches the
// filter operand of its groups), and the staging of whole images or strips, byte by byte where
// rows are not whole dwords.  The picked combination takes 1.004 times as long as the best one (at most
// 1.14); without the staging in the estimate, fitted to 56x56 and 28x28 maps, it was 1.036 (at most
// 1.68; 31x45 maps, 16 channels, ten images: 12.6 us against 8.5 with four tiles).
static bool make_small_plan(const Geometry& g, SmallPlan* best) {
  if (g.alg != kSmallAlg || g.Cp > 128) return false;
  const long long lim = 1ll << 31;
  if ((long long)g.N * g.Cin * g.H * g.W >= lim || 4ll * g.N * g.Cout * g.H * g.W >= lim) return false;
  const unsigned kc = (unsigned)(g.Cp / 64), lds_max = 160u * 1024u - 512u;
  bool found = false;
  for (int tiles = 16; tiles >= 2; tiles /= 2) {
    SmallPlan sp;
    if (!make_tile_rect(g, (lds_max - 16u) / kc, &sp.tr, tiles)) continue;
    sp.fgroups = (g.Cout + 15) / 16;
    sp.cgroups = (g.Cin + 15) / 16;
    if (sp.tr.ntiles * sp.cgroups > kSmallPatches) continue;
    sp.chunk_in = tile_rect_stage_bytes(g, sp.tr);
    for (sp.fper = 1; sp.fper <= 2; ++sp.fper) {
      if (sp.fper > sp.fgroups) break;
      unsigned top = 16u + sp.chunk_in * kc;
      const unsigned vbytes = 48u * (kc * 1024u + 16u), zbytes = (unsigned)(sp.fper * kParts) * 4096u;
      if (vbytes > top) top = vbytes;
      if (zbytes > top) top = zbytes;
      sp.tab_off = (top + 8u + 15u) & ~15u;
      sp.lds_bytes = sp.tab_off + 256u;
      if (sp.lds_bytes > lds_max) continue;
      const long long wgs = (long long)tile_rect_groups(g, sp.tr) * ((sp.fgroups + sp.fper - 1) / sp.fper);
      if (wgs > 256) continue;
      const bool dwords = g.W % 4 == 0;
      sp.cost = 0.045 * sp.tr.ntiles * sp.cgroups + (1.0 + 0.5 * kc) * (sp.fper - 1) + 0.006 * (double)wgs +
                (sp.tr.whole ? 3.5 + kc * (dwords ? 0.3 : 0.55) * sp.tr.ipw
                             : kc * (0.6 * sp.tr.S + (dwords ? 0.0 : 2.0)));
      if (!found || sp.cost < best->cost - 1e-9) {
        *best = sp;
        found = true;
      }
    }
  }
  return found;
}

// Where its workgroups fit the chip in one round, the kernel is ahead of single16_kernel (us per
// layer: 64 channels on 56x56 maps, 1 / 4 / 8 images, 6.9 / 7.6 / 8.8 against 9.7 / 10.0 / 9.9; 128
// channels on 28x28 maps 7.2 / 8.8 / 10.6 against 17.1 / 17.5 / 17.6; 0.28 to 0.96 of its time, 0.58 on
// average, over 547 layers of 16 to 128 channels on maps from 7x7 to 224x224, 200x16 and 6x61, up to
// the most images that fit); in two rounds it is behind (12 images: 16.0 against 10.2 and 19.6
// against 17.7).
bool single_small_supported(const Geometry& g) {
  SmallPlan sp;
  return make_small_plan(g, &sp);
}

template <int KC, int OUT>
static hipError_t launch_small_impl(const Geometry& g, const SmallPlan& sp, const int8_t* x, const FilterViews& f,
                                    float x_scale, float inv_y, void* y, hipStream_t s, bool prepare) {
  const dim3 grid(tile_rect_groups(g, sp.tr), (unsigned)((sp.fgroups + sp.fper - 1) / sp.fper));
  auto launch = [&](auto kernel) {
    if (prepare) return raise_lds_limit(reinterpret_cast<const void*>(kernel));
    hipLaunchKernelGGL(kernel, grid, dim3(kSmallWaves * 64), sp.lds_bytes, s, x, (const int8_t*)f.U_single,
                       f.dequant_single, f.input_tab, x_scale, inv_y, y, g, sp);
    return hipGetLastError();
  };
  return g.W % 4 == 0   ? launch(single_small_kernel<KC, OUT, 4>)
         : g.W % 2 == 0 ? launch(single_small_kernel<KC, OUT, 2>)
                        : launch(single_small_kernel<KC, OUT, 1>);
}

hipError_t launch_single_small(int out, const Geometry& g, const int8_t* x, const FilterViews& f, float x_scale,
                               float inv_y, void* y, hipStream_t s, bool prepare) {
  SmallPlan sp;
  if (out == 1 || !make_small_plan(g, &sp)) return hipErrorNotSupported;
  if (g.Cp == 64)
    return out == 2 ? launch_small_impl<1, 2>(g, sp, x, f, x_scale, inv_y, y, s, prepare)
                    : launch_small_impl<1, 0>(g, sp, x, f, x_scale, inv_y, y, s, prepare);
  return out == 2 ? launch_small_impl<2, 2>(g, sp, x, f, x_scale, inv_y, y, s, prepare)
                  : launch_small_impl<2, 0>(g, sp, x, f, x_scale, inv_y, y, s, prepare);
}

// ---------------------------------------------------------------------------------------
// Products + output transform from V, 256 and 512 input channels.  A workgroup takes 16 tiles
// and one quad of four filters; a wave one 64-channel chunk and a run of positions: operand A
// is the quad layout (four points x four filters, sfc_fused_quad.hpp; three of four results
// per instruction are mixed points, the matrix pipe has nothing else to do), V is read
// straight into operands.  Every load of a wave is in flight before its first product, no
// ring, no barrier: one round trip to memory.  The sums of the chunks meet in LDS, are scaled
// there by all waves, and four waves take the 46 products of every pair through the output
// transform, one output row each.
// ---------------------------------------------------------------------------------------
constexpr int small_product_pitch() { return 52; }  // floats per pair: 48 positions + 4 against bank conflicts

// (four waves per SIMD and 128 registers: at eight the loads would not all be in flight)
template <int KC, int OUT, int EV>
__global__ __launch_bounds__(kSmallWaves * 64) __attribute__((amdgpu_waves_per_eu(4, 4))) void product_small_kernel(
    const int8_t* __restrict__ V, const int8_t* __restrict__ Uf, const float* __restrict__ dqf, float x_scale,
    float inv_y, void* __restrict__ y, Geometry g, int kquads, int tiles) {
  constexpr int ALG = kSmallAlg, NW = kSmallWaves;
  constexpr int P = AlgTraits<ALG>::P, PP = Order<ALG>::PP, PG = PP / 4;
  constexpr int CP = KC * 64;
  constexpr int RUNS = NW / KC;   // runs of positions: 4 with four chunks, 2 with eight
  constexpr int GPR = PG / RUNS;  // groups of four positions per run
  static_assert(RUNS * KC == NW && GPR * RUNS == PG, "whole runs");
  constexpr int PITCH = small_product_pitch();
  constexpr Order<ALG> order{};
  __shared__ int part_sum[KC][PP][64];  // [chunk][position][pair]
  __shared__ __align__(16) float prod[64 * PITCH];
  __shared__ int tile_tab[48];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kq = blockIdx.x % kquads, tb = blockIdx.x / kquads;
  const int t0 = tb * tiles;  // (slots from `tiles` on stay empty)
  if (threadIdx.x < 16) {
    const int tl = threadIdx.x, t = t0 + tl;
    const int per = g.th * g.tw;
    const int n = t / per, rem = t - n * per;
    const int ti = rem / g.tw, tj = rem - ti * g.tw;
    write_tile_entry<AlgTraits<ALG>::M>(tile_tab, tl, tl < tiles && t < g.T, n, ti, tj, g.Cout, g.H, g.W);
  }
  const int kc = wave % KC, run = wave / KC;
  const unsigned vplane = (unsigned)g.Tp * (unsigned)CP;
  const __amdgpu_buffer_rsrc_t vres =
      __builtin_amdgcn_make_buffer_rsrc((void*)V, 0, (int)(vplane * (unsigned)P), kBufferFlags);
  const __amdgpu_buffer_rsrc_t ures = __builtin_amdgcn_make_buffer_rsrc(
      (void*)Uf, 0, (int)((unsigned)kquads * (unsigned)(PP * CP * 4)), kBufferFlags);
  v4i a[GPR], b[GPR][4];
#pragma unroll
  for (int i = 0; i < GPR; ++i)
    a[i] = __builtin_amdgcn_raw_buffer_load_b128(
        ures, (unsigned)lane * 16u, (unsigned)((kq * PG + run * GPR + i) * KC + kc) * 1024u, 0);
  // (tiles past the last one read nothing)
  const int t = t0 + (lane & 15);
  const unsigned v_lane =
      (lane & 15) < tiles && t < g.T ? (unsigned)t * (unsigned)CP + (unsigned)(64 * kc + 16 * (lane >> 4)) : 0x80000000u;
#pragma unroll
  for (int i = 0; i < GPR; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      // the position is one of RUNS compile-time values chosen by the run
      int p = 0;
#pragma unroll
      for (int u = 0; u < RUNS; ++u)
        if (u == run) p = max(order.pt[4 * (u * GPR + i) + r], 0);
      b[i][r] = __builtin_amdgcn_raw_buffer_load_b128(vres, v_lane, (unsigned)p * vplane, 0);
    }
  // factors of this wave's three positions for the lane's filter
  float d[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) d[i] = dqf[(size_t)(4 * kq + (lane >> 4)) * PP + 3 * wave + i];
  __builtin_amdgcn_sched_barrier(0);  // every load before the first product
#pragma unroll
  for (int i = 0; i < GPR; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const v4i acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b[i][r], v4i{0, 0, 0, 0}, 0, 0, 0);
      part_sum[kc][4 * (run * GPR + i) + r][lane] = acc[r];
    }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    int sum = 0;
#pragma unroll
    for (int c = 0; c < KC; ++c) sum += part_sum[c][3 * wave + i][lane];
    prod[lane * PITCH + 3 * wave + i] = (float)sum * d[i];
  }
  __syncthreads();
  if (wave >= 4) return;
  // wave w finishes row w of every pair (the parts of the transform that other rows need fall away)
  v4f pr[PG];
#pragma unroll
  for (int i = 0; i < PG; ++i) pr[i] = *(const v4f*)(prod + lane * PITCH + 4 * i);
  float z[6][4];
  stream_vertical<ALG, float>(
      [&](auto position) __attribute__((always_inline)) -> float {
        constexpr int j = decltype(position)::value;
        return pr[j >> 2][j & 3];
      },
      z);
  constexpr unsigned esz = OUT == 2 ? 1u : 4u;
  const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc(
      y, 0, (int)(esz * (unsigned)(g.N * g.Cout) * (unsigned)(g.H * g.W)), kBufferFlags);
  const int kcol = 4 * kq + (lane >> 4);
  if (wave == 0) store_pair_rows<OUT, EV, 0, 1>(z, tile_tab, lane, kcol, x_scale, inv_y, yres, g);
  else if (wave == 1) store_pair_rows<OUT, EV, 1, 1>(z, tile_tab, lane, kcol, x_scale, inv_y, yres, g);
  else if (wave == 2) store_pair_rows<OUT, EV, 2, 1>(z, tile_tab, lane, kcol, x_scale, inv_y, yres, g);
  else store_pair_rows<OUT, EV, 3, 1>(z, tile_tab, lane, kcol, x_scale, inv_y, yres, g);
}

int product_small_filter_count(const Geometry& g) { return (g.Cout + 3) / 4 * 4; }

// While the workgroups fit the chip in one round (us per layer, input transform included: 256
// channels on 14x14 maps, 1 / 4 images, 9.3 / 12.4 against 20.2 / 21.6 with the kernels for larger
// layers, 512 channels on 7x7 maps, 1 / 4 / 8 images, 12.3 / 14.1 / 18.0 against 22.2; in two rounds
// level or behind: 6 images 20.7 against 21.8, 12 images 31.2 against 22.2).  Every filter quad reads
// all of V, consecutive quads on different XCDs, so where V is not small next to an L2 the line
// comes earlier (512 channels on 7x7 maps, 32 / 96 / 128 images, 128 / 32 / 32 filters: 22.2 / 22.2 /
// 27.9 us against 20.5 / 19.7 / 23.5).  Time against the other kernels over 560 layers of 4 to 512
// filters: 256 channels, V to 4 MB 0.47 to 0.95, else up to 160 workgroups 0.73 to 1.04, above 0.95
// to 1.11; 512 channels, V to 2 MB 0.50 to 0.97, else up to 128 workgroups 0.65 to 1.04, above 0.92 to
// 1.22.
bool product_small_supported(const Geometry& g) {
  if (g.alg != kSmallAlg || (g.Cp != 256 && g.Cp != 512)) return false;
  const long long wgs = (long long)(g.Tp / 16) * (product_small_filter_count(g) / 4);
  const long long vbytes = (long long)g.P * g.Tp * g.Cp;
  const bool v_small = vbytes <= (g.Cp == 256 ? 4ll : 2ll) << 20;
  return wgs <= (v_small ? 256 : g.Cp == 256 ? 160 : 128) && 4ll * g.N * g.Cout * g.H * g.W < (1ll << 31);
}

template <int KC, int OUT>
static hipError_t launch_product_small_impl(const Geometry& g, const void* V, const FilterViews& f, float x_scale,
                                            float inv_y, void* y, hipStream_t s) {
  // 16 tiles per workgroup, or 8 or 4 while the chip has compute units to spare: a workgroup
  // then reads that much less of V
  const int kquads = product_small_filter_count(g) / 4;
  int tiles = 16;
  while (tiles > 4 && (long long)((g.T + tiles / 2 - 1) / (tiles / 2)) * kquads <= 256) tiles /= 2;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((g.T + tiles - 1) / tiles * kquads)), dim3(kSmallWaves * 64), 0, s,
                       (const int8_t*)V, (const int8_t*)f.U_single, f.dequant_single, x_scale, inv_y, y, g, kquads,
                       tiles);
    return hipGetLastError();
  };
  return g.W % 4 == 0   ? launch(product_small_kernel<KC, OUT, 4>)
         : g.W % 2 == 0 ? launch(product_small_kernel<KC, OUT, 2>)
                        : launch(product_small_kernel<KC, OUT, 1>);
}

hipError_t launch_product_small(int out, const Geometry& g, const void* V, const FilterViews& f, float x_scale,
                                float inv_y, void* y, hipStream_t s) {
  if (out == 1 || !product_small_supported(g)) return hipErrorNotSupported;
  if (g.Cp == 256)
    return out == 2 ? launch_product_small_impl<4, 2>(g, V, f, x_scale, inv_y, y, s)
                    : launch_product_small_impl<4, 0>(g, V, f, x_scale, inv_y, y, s);
  return out == 2 ? launch_product_small_impl<8, 2>(g, V, f, x_scale, inv_y, y, s)
                  : launch_product_small_impl<8, 0>(g, V, f, x_scale, inv_y, y, s);
}

}  // namespace sfc
