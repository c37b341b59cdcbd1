// Input-tile transform V = B^T x B in row form on the matrix cores (gfx950): requantized mode
// outside small feature maps (rounded to int8, [P][Tp][Cp]) and exact mode (kept as int16).
//
// A workgroup stages the input rows of a rectangle of tiles (S strips x tlw tile columns) for 64
// channels in LDS.  A patch row is up to 16 bytes, k = 16 i + j, so the sums of 16 channels at 16
// positions take two or three int8 matrix instructions of 64 k-bytes (sfc_mfma_input.hpp).  A WAVE
// OWNS POSITIONS, not tiles: one to four blocks of 16, whose coefficients stay in its registers
// while it walks over the tiles and their four groups of 16 channels.  The bytes of a tile are turned
// round in LDS of the wave's own and written with 16-byte lanes, 64 (int16: 128) contiguous bytes
// per (position, tile).
//
// What bounds it: instruction issue (7x7 filters, 128 channels on 28x28 maps, batch 64: 25.7 k of some 69 k
// clocks of every SIMD are vector instructions, 15 of 20 the rounding of four values, 14.6 k matrix
// instructions) and, while V is larger than the caches, its way to memory.  With a wave to a tile every
// wave read the whole coefficient table (36 KB at 184 positions) and its rounding waited for the matrix
// instructions just before it.  Staged rows are as long as the rectangle needs (64 bytes each before): 20 to 40 KB
// to a workgroup of four waves, three or four of which share a compute unit; one of twelve waves, 64 to 86 KB, with 7x7 tiles.  A
// wave's tiles all start at the same byte of a dword, so the coefficients are shifted once instead of every patch
// row.  us before and after, V 74, 37 and (int16) 36 MB: 7x7 filters on that layer 39.5 -> 28.8, 5x5 filters 21.2 -> 19.3,
// exact mode, 64 channels on 56x56 maps, batch 32, 13.8 -> 13.6.  Two, three and six position groups for 184 points instead
// of four: 35.0, 30.4 and 34.5 us for the first layer.
// The SFC-4 forms had a wave to a tile, 64-byte rows staged whatever the width (a byte at a time where 4 does
// not divide it) and V collected in LDS: 192 to 64 channels on 107 35x35 maps, three kernels, 349 -> 137 us, 350 to
// 40 on 256 53x25 maps 613 -> 485, 256 to 256 on 16 56x56 maps 56.3 -> 54.4; over 60 layers of more than 128 channels with
// 350 to 650 tiles 0.48 to 1.04 of the time, 0.93 in the middle.
#include <algorithm>

#include "sfc_device.hpp"
#include "sfc_internal.hpp"
#include "sfc_mfma_input.hpp"
#include "sfc_points.hpp"
#include "sfc_tile_input.hpp"

namespace sfc {

template <int ALG, bool EXACT>
struct RowsForm {
  using Tr = AlgTraits<ALG>;
  static constexpr int NPB = (Order<ALG>::PP + 15) / 16;  // blocks of 16 positions
  // Position groups.  More of them, fewer blocks and registers to a wave and more waves to a workgroup; a last group that
  // is not full works for nothing.  The kernel's time over 16 layers, geometric mean: 100 points with four groups
  // 0.87 of that with two (int8 and int16), 88 points with three 0.95 in int8 (int16 0.94, but 12.6 for 11.8 us
  // where V of 64 channels on 56x56 maps, batch 32, is written), 196 points in int16 with five and (4x4 tiles) seven
  // 0.94 and 0.89 of that with four; in int8 1.04 and 0.97, 0.8 to 1.2.  52 positions with two 0.93, four 1.0;
  // 48 with two 1.02; 184 points with five and six 1.04 to 1.19.
  static constexpr int PG = NPB <= 3 ? 1 : NPB <= 4 ? 2 : NPB <= 6 ? (EXACT ? 2 : 3) : NPB <= 7 ? 4 : NPB <= 9 ? 3
                            : NPB <= 12 || !EXACT ? 4 : Tr::M == 6 ? 5 : 7;
  static constexpr int BPW = (NPB + PG - 1) / PG;                           // blocks of a wave
  // tile groups: tile columns j, j + TG, ... of a rectangle, whose patches start at the same byte of a
  // dword (tile edges 4, 6, 7: every, every second, every fourth column)
  static constexpr int kPeriod = Tr::M % 4 == 0 ? 1 : Tr::M % 2 == 0 ? 2 : 4;
  static constexpr int TG = kPeriod * PG >= 4 ? kPeriod : 4 / PG;
  static constexpr int NW = PG * TG;
  static constexpr int KST = (Tr::NI + 3) / 4;        // matrix steps that carry patch rows
  static constexpr int kRowBytes = EXACT ? 144 : 80;  // LDS bytes per position in a wave's block (data and padding)
  static constexpr int kBlockBytes = 16 * BPW * kRowBytes;
  static_assert(16 * NPB <= kRowsTabRows && Tr::NI <= 12, "table rows, three steps of four patch rows");
  static_assert(TG % kPeriod == 0, "one byte offset to a wave");
};

struct RowsPlan {
  TileRect tr;
  int ndw;             // dwords of a staged row
  unsigned rcp_ndw;    // ceil(2^16 / ndw): exact quotients below 16 rows
  unsigned cs;         // LDS bytes from one channel's rows to the next
  unsigned blk_off;    // LDS byte offset of the waves' blocks
  unsigned lds_bytes;
};

// Stages the rows of every strip of the rectangle, channels c0 .. c0 + 63, zero outside the
// image: lane = (row, dword) pairs of a channel running along the rows, the same for all channels.
// Lanes outside the image get an offset outside the buffer, for which the load returns zero.
// TAIL: rows that are not whole dwords; a dword that straddles the end of a row keeps its valid
// bytes, one that would reach past the tensor is fetched byte by byte.  Channels beyond Cin re-read
// the last one (their filter operand is zero).
template <int ALG, int NW, bool TAIL>
__device__ __forceinline__ void stage_rows(const int8_t* __restrict__ x, unsigned char* lds, const Geometry& g,
                                           const RowsPlan& rp, int strip0, int tj0, int c0, int wave, int lane) {
  constexpr int M = AlgTraits<ALG>::M, NI = AlgTraits<ALG>::NI, PAD = AlgTraits<ALG>::PAD;
  constexpr unsigned kOutOfRange = 0x80000000u;
  constexpr int CPW = (64 + NW - 1) / NW;  // channels of a wave: wave, wave + NW, ...
  const int W = g.W, H = g.H;
  const unsigned xbytes = (unsigned)(g.N * g.Cin) * (unsigned)(H * W);
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc((void*)x, 0, (int)xbytes, kBufferFlags);
  const int colbase = ((M * tj0) & ~3) - 4;
  const int pairs = NI * rp.ndw, pieces = (pairs + 63) >> 6, total = rp.tr.S * pieces;
  // (two pieces' loads in flight before the first LDS write)
  int s = 0, i0 = 0;
  for (int k0 = 0; k0 < total; k0 += 2) {
    unsigned vals[2][CPW];
    int to[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const int strip = strip0 + s;
      const int n = strip_image(rp.tr, strip);
      const int hlo = M * (strip - n * g.th) - PAD;
      const int idx = i0 + lane;
      const int row = (int)(((unsigned)idx * rp.rcp_ndw) >> 16), dcol = idx - row * rp.ndw;
      const int col = colbase + 4 * dcol;
      const int nvalid = col < 0 ? 0 : min(4, max(0, W - col));
      const unsigned bmask = nvalid >= 4 ? 0xffffffffu : ((1u << (8 * nvalid)) - 1u);
      const bool mine = k0 + kk < total && idx < pairs;
      const bool ok = mine && strip < g.strips && nvalid > 0 && (unsigned)(hlo + row) < (unsigned)H;
      const unsigned voff = ok ? (unsigned)((n * g.Cin * H + hlo + row) * W + col) : kOutOfRange;
      to[kk] = mine ? (int)((unsigned)(s * 64 + wave) * rp.cs) + 4 * idx : -1;
#pragma unroll
      for (int ci = 0; ci < CPW; ++ci) {
        const int c = min(c0 + min(wave + NW * ci, 63), g.Cin - 1);
        const unsigned plane = (unsigned)c * (unsigned)(H * W);
        unsigned v = __builtin_amdgcn_raw_buffer_load_b32(xres, voff, plane, 0);
        if constexpr (TAIL) {
          v &= bmask;
          // (a plane in front of the last one too: maps of one or two samples)
          if (xbytes - (unsigned)(n * g.Cin) * (unsigned)(H * W) - plane < (unsigned)(H * W) + 3u) {
            if (ok && voff + plane + 4u > xbytes) {
              v = 0;
              for (int bb = 0; bb < nvalid; ++bb)
                v |= (unsigned)__builtin_amdgcn_raw_buffer_load_b8(xres, voff + bb, plane, 0) << (8 * bb);
            }
          }
        }
        vals[kk][ci] = v;
      }
      i0 += 64;
      if (i0 >= pairs) {
        i0 = 0;
        ++s;
      }
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
      if (to[kk] >= 0) {
#pragma unroll
        for (int ci = 0; ci < CPW; ++ci)
          if (wave + NW * ci < 64) *(unsigned*)(lds + to[kk] + (unsigned)(NW * ci) * rp.cs) = vals[kk][ci];
      }
  }
}

template <int ALG, bool EXACT>
__global__ __launch_bounds__((RowsForm<ALG, EXACT>::NW * 64), 4) void input_rows_kernel(
    const int8_t* __restrict__ x, void* __restrict__ Vout, const unsigned char* __restrict__ tab, Geometry g,
    RowsPlan rp) {
  using Tr = AlgTraits<ALG>;
  using Form = RowsForm<ALG, EXACT>;
  constexpr int NW = Form::NW, BPW = Form::BPW, KST = Form::KST, NI = Tr::NI, RB = Form::kRowBytes;
  extern __shared__ __align__(16) unsigned char lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const TileRect& tr = rp.tr;
  // Position = (rectangle, 64-channel group), the channel group varying fastest, contiguous on an
  // XCD: neighbours share halo rows, and the halves of a line of V are written next to each other.
  const int cgn = g.Cp >> 6;
  const int pos = xcd_contiguous(blockIdx.x, gridDim.x);
  const int bx = pos / cgn;
  const int c0 = (pos - bx * cgn) * 64;
  const int strip0 = (bx / tr.chunks) * tr.S, tj0 = (bx % tr.chunks) * tr.tlw;

  const int pgrp = wave % Form::PG, tgrp = wave / Form::PG;
  const int live_strips = min(tr.S, g.strips - strip0), live_cols = min(tr.tlw, g.tw - tj0);
  // first byte of the wave's patches within an aligned dword of a staged row
  const int o0 = ((Tr::M * tj0) & 3) - Tr::PAD + 4 + Tr::M * tgrp;
  const int sh = o0 & 3;

  // The wave's blocks (those past the last repeat table rows and store nothing).  A lane reads whole
  // dwords of a patch row, so the coefficients are moved up by the patch's first byte instead.
  const float* inv_pos = (const float*)tab;
  const int* point = (const int*)(tab + kRowsTabPoint);
  const unsigned char* ctab = tab + kRowsTabCoeff;
  constexpr int ESZ = EXACT ? 2 : 1;
  constexpr int SPB = EXACT ? 2 : 1;  // stores per block: 8 or 16 positions each
  constexpr int LPP = EXACT ? 8 : 4;  // lanes per position
  const size_t vplane = (size_t)g.Tp * (size_t)g.Cp;
  const __amdgpu_buffer_rsrc_t vres = __builtin_amdgcn_make_buffer_rsrc(
      Vout, 0, EXACT ? 0 : (int)((unsigned)vplane * (unsigned)Tr::P), kBufferFlags);
  v4i coeff[BPW][KST];
  float inv[BPW];
  unsigned vofs[BPW];              // int8: byte offset in V, outside it for positions without a point
  unsigned char* vdst[BPW][SPB];   // int16 (V may be larger than 32-bit offsets reach): null without a point
#pragma unroll
  for (int b = 0; b < BPW; ++b) {
    const int m = pgrp * BPW + b;
    const int p = 16 * min(m, Form::NPB - 1) + (lane & 15);
    inv[b] = inv_pos[p];
#pragma unroll
    for (int st = 0; st < KST; ++st) {
      const v4i c = *(const v4i*)(ctab + p * 192 + 64 * st + 16 * (lane >> 4));
      unsigned below = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        coeff[b][st][i] = sh == 0 ? c[i] : (int)__builtin_amdgcn_alignbyte((unsigned)c[i], below, 4u - (unsigned)sh);
        below = (unsigned)c[i];
      }
    }
#pragma unroll
    for (int h = 0; h < SPB; ++h) {
      const int pt = m < Form::NPB ? point[16 * m + (16 / SPB) * h + lane / LPP] : -1;
      const size_t at = ((size_t)max(pt, 0) * vplane + c0) * ESZ + 16 * (lane % LPP);
      if constexpr (EXACT) vdst[b][h] = pt >= 0 ? (unsigned char*)Vout + at : nullptr;
      else vofs[b] = pt >= 0 ? (unsigned)at : 0x80000000u;
    }
  }

  if ((g.W & 3) == 0) stage_rows<ALG, NW, false>(x, lds, g, rp, strip0, tj0, c0, wave, lane);
  else stage_rows<ALG, NW, true>(x, lds, g, rp, strip0, tj0, c0, wave, lane);
  __syncthreads();
  const int my_cols = (live_cols - tgrp + Form::TG - 1) / Form::TG;
  if (my_cols <= 0) return;  // (no workgroup barrier after this point)

  // operand A of a (tile, group of 16 channels): lane = (channel lane % 16, patch row 4 st + lane / 16),
  // 16 bytes (rows past the patch repeat the last one, bytes outside it belong to its neighbours: both
  // meet zero coefficients)
  unsigned lrow[KST];
#pragma unroll
  for (int st = 0; st < KST; ++st)
    lrow[st] = (unsigned)(lane & 15) * rp.cs + 4u * (unsigned)(min(4 * st + (lane >> 4), NI - 1) * rp.ndw);
  auto fetch = [&](const unsigned char* in, v4i (&a)[KST]) __attribute__((always_inline)) {
#pragma unroll
    for (int st = 0; st < KST; ++st) {
      const int* src = (const int*)(in + lrow[st]);
#pragma unroll
      for (int i = 0; i < 4; ++i) a[st][i] = src[i];
    }
  };
  auto sums = [&](const v4i (&a)[KST], v4i (&d)[BPW]) __attribute__((always_inline)) {
#pragma unroll
    for (int st = 0; st < KST; ++st)
#pragma unroll
      for (int b = 0; b < BPW; ++b)
        d[b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[st], coeff[b][st], st == 0 ? v4i{0, 0, 0, 0} : d[b], 0, 0, 0);
  };
  unsigned char* blk = lds + rp.blk_off + wave * Form::kBlockBytes;
  unsigned char* put_at = blk + (lane & 15) * RB + (EXACT ? 8 : 4) * (lane >> 4);
  const unsigned char* get_at = blk + (lane / LPP) * RB + 16 * (lane % LPP);
  constexpr float kMagic = 12582912.0f;
  const float lo = kMagic - g.qmax, hi = kMagic + g.qmax;
  // channels 16 cg + 4 (lane / 16) .. + 3 of position lane % 16 of every block
  auto put = [&](const v4i (&d)[BPW], int cg) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < BPW; ++b) {
      if constexpr (EXACT) {
        v2i w;
        w[0] = (int)__builtin_amdgcn_perm((unsigned)d[b][1], (unsigned)d[b][0], 0x05040100u);
        w[1] = (int)__builtin_amdgcn_perm((unsigned)d[b][3], (unsigned)d[b][2], 0x05040100u);
        *(v2i*)(put_at + b * 16 * RB + 32 * cg) = w;
      } else {
        unsigned q[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float v = __fmaf_rn((float)d[b][i], inv[b], kMagic);
          v = __builtin_amdgcn_fmed3f(v, lo, hi);
          q[i] = __float_as_uint(v);
        }
        *(unsigned*)(put_at + b * 16 * RB + 16 * cg) =
            __builtin_amdgcn_perm(q[1], q[0], 0x0c0c0400u) | __builtin_amdgcn_perm(q[3], q[2], 0x04000c0cu);
      }
    }
  };
  auto lds_order = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local"); };

  // Software pipeline over (tile, channel group) q: operand of q + 2 and matrix instructions of q + 1
  // before the rounding of q.
  const int ntiles = live_strips * my_cols;
  const unsigned gstep = 16u * rp.cs;
  const unsigned char* in = lds + (unsigned)(o0 & ~3);  // of the tile whose operand is fetched next
  int s = 0, col = 0;
  v4i a[2][KST], d[2][BPW];
  fetch(in, a[0]);
  fetch(in + gstep, a[1]);
  sums(a[0], d[0]);
  unsigned trow = (unsigned)(strip0 * g.tw + tj0 + tgrp);  // the tile's row of V
  for (int i = 0; i < ntiles; ++i) {
    unsigned tnext = trow;
#pragma unroll
    for (int cg = 0; cg < 4; ++cg) {
      if (cg == 2) {  // on to the next tile (past the last one: it is read again)
        if (col + 1 < my_cols) {
          ++col;
          in += Form::TG * Tr::M;
          tnext = trow + Form::TG;
        } else if (s + 1 < live_strips) {
          in += 64u * rp.cs - (unsigned)(col * (Form::TG * Tr::M));
          tnext = trow + (unsigned)(g.tw - Form::TG * col);
          col = 0;
          ++s;
        }
      }
      fetch(in + (unsigned)((cg + 2) & 3) * gstep, a[cg & 1]);
      sums(a[(cg + 1) & 1], d[(cg + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
      put(d[cg & 1], cg);
    }
    lds_order();
    v4i w[BPW][SPB];
#pragma unroll
    for (int b = 0; b < BPW; ++b)
#pragma unroll
      for (int h = 0; h < SPB; ++h) w[b][h] = *(const v4i*)(get_at + (b * 16 + (16 / SPB) * h) * RB);
    if constexpr (EXACT) {
      const size_t toff = (size_t)trow * (size_t)g.Cp * ESZ;
#pragma unroll
      for (int b = 0; b < BPW; ++b)
#pragma unroll
        for (int h = 0; h < SPB; ++h)
          if (vdst[b][h]) *(v4i*)(vdst[b][h] + toff) = w[b][h];
    } else {
#pragma unroll
      for (int b = 0; b < BPW; ++b)
        __builtin_amdgcn_raw_buffer_store_b128(w[b][0], vres, vofs[b], trow * (unsigned)g.Cp, 0);
    }
    lds_order();
    trow = tnext;
  }
}

// ---------------------------------------------------------------------------------------

// The rectangle of a workgroup.  What a layer takes goes by rounds: compute units times the workgroups that share
// one are served at a time, and a workgroup costs its staging and so many tiles.  Of rectangles of up to eight,
// four, two and one tiles, as many strips as fit in 40, 80 or 160 KB of LDS, the one with the least of
//   6 rounds + tiles of a compute unit
// is taken.  Rounds: workgroups of a compute unit over those that share it, no less than one; as whole numbers 64
// channels on 160 24x24 maps, 5x5 filters, layer, 33.1 -> 34.5 us.  At a tie more tiles (four, where a wave takes
// every tile of its workgroup), then less LDS.  Workgroups of four waves keep to 40 KB (or one strip): a compute
// unit holds four of those and three of 54 KB, 4x4 tiles, 7x7 filters, 512 channels on sixty 16x15 maps 40.8 -> 48.7 us.
// The kernel alone against one wave to a tile, geometric mean over 16 layers of every algorithm, int8 and int16
// (320): 0.87; eight tiles, else four, two, one until there are 512 workgroups: 1.00 (272 that had a plan).  Of the
// fixed choices the rule misses the best by 1 % in the mean.  Left behind, layers with many tiles: 7x7 tiles in
// int8, 64 channels on 56x56 maps, batch 32, 10.0 -> 11.6 us (sixteen 29x31 maps of 70 channels 12.6 -> 9.6), 196
// points of the 5x5 filters in int16 22.5 -> 27.4.
template <int ALG, bool EXACT>
static bool make_rows_plan(const Geometry& g, RowsPlan* rp) {
  using Form = RowsForm<ALG, EXACT>;
  constexpr int M = AlgTraits<ALG>::M, NI = AlgTraits<ALG>::NI, PAD = AlgTraits<ALG>::PAD, R = AlgTraits<ALG>::R;
  const long long xb = (long long)g.N * g.Cin * g.H * g.W, vb = (long long)g.P * g.Tp * g.Cp;
  if (xb >= (1ll << 31) || (!EXACT && vb >= (1ll << 31))) return false;  // 32-bit offsets
  if ((long long)g.strips * g.th >= (1ll << 32)) return false;  // strip_image's reciprocal
  constexpr unsigned kBlocks = (unsigned)Form::NW * (unsigned)Form::kBlockBytes, kLds = 160u * 1024u;
  constexpr unsigned kMost = Form::NW > 4 ? kLds : kLds / 4;
  constexpr int kUnits = 256, kWaves = 16;  // compute units, waves that share one (128 registers)
  RowsPlan c{};
  c.tr.th_magic = ((1ull << 32) + (unsigned long long)g.th - 1) / (unsigned long long)g.th;
  double best = -1;
  // (4x4 tiles, 46 points: a wave owns every position of its tile columns, with fewer than four tiles some waves
  // would have none)
  constexpr int kLeast = Form::PG == 1 ? Form::TG : 1;
  for (int tiles = 8; tiles >= kLeast; tiles >>= 1) {
    c.tr.chunks = (g.tw + tiles - 1) / tiles;
    c.tr.tlw = (g.tw + c.tr.chunks - 1) / c.tr.chunks;
    const int h = (c.tr.chunks > 1 && (M * c.tr.tlw) % 4 != 0 ? 2 + M % 2 : 0) + 4 - PAD;
    // An odd number of dwords from row to row and four times an odd one from channel to channel: the
    // 16 channels x 4 rows that an instruction reads lie in different banks.
    c.ndw = (h + M * c.tr.tlw + R - 1 + 3) / 4 | 1;
    c.rcp_ndw = (65536u + (unsigned)c.ndw - 1u) / (unsigned)c.ndw;
    c.cs = 16u * ((unsigned)(NI * c.ndw + 3) / 4u | 1u);
    auto bytes = [&](int S) { return (((unsigned)S * 64u * c.cs + 32u + 15u) & ~15u) + kBlocks; };
    const int strips = std::max(1, std::min(tiles / c.tr.tlw, g.strips));
    c.tr.S = 0;
    for (unsigned most = kLds / 4; most <= kMost && c.tr.S < strips; most *= 2) {
      c.tr.S = strips;
      while (c.tr.S > 1 && bytes(c.tr.S) > most) --c.tr.S;
      c.tr.ntiles = c.tr.S * c.tr.tlw;
      c.lds_bytes = bytes(c.tr.S);
      c.blk_off = c.lds_bytes - kBlocks;
      if (c.lds_bytes > kLds) continue;
      const long long of_unit = ((long long)tile_rect_groups(g, c.tr) * (g.Cp / 64) + kUnits - 1) / kUnits;
      const int shared = std::max(1, std::min((int)(kLds / c.lds_bytes), kWaves / Form::NW));
      const double cost = 6.0 * std::max(1.0, (double)of_unit / shared) + (double)(of_unit * c.tr.ntiles);
      if (best < 0 || cost < best || (cost == best && Form::TG == 1 && tiles == 4)) {
        best = cost;
        *rp = c;
      }
    }
  }
  return best >= 0;
}

template <int ALG, bool EXACT>
static hipError_t launch_rows_alg(const Geometry& g, const int8_t* x, void* V, const unsigned char* tab,
                                  hipStream_t s, bool prepare) {
  RowsPlan rp{};
  if (!make_rows_plan<ALG, EXACT>(g, &rp)) return hipErrorNotSupported;
  auto kernel = input_rows_kernel<ALG, EXACT>;
  if (prepare) return raise_lds_limit(reinterpret_cast<const void*>(kernel));
  const dim3 grid(tile_rect_groups(g, rp.tr) * (unsigned)(g.Cp / 64));
  hipLaunchKernelGGL(kernel, grid, dim3(RowsForm<ALG, EXACT>::NW * 64), rp.lds_bytes, s, x, V, tab, g, rp);
  return hipGetLastError();
}

bool input_rows_supported(const Geometry& g, bool exact) {
  RowsPlan rp{};
  auto plan = [&](auto alg) {
    constexpr int ALG = decltype(alg)::value;
    return exact ? make_rows_plan<ALG, true>(g, &rp) : make_rows_plan<ALG, false>(g, &rp);
  };
  switch (g.alg) {
    case 0: return plan(std::integral_constant<int, 0>{});
    case 1: return plan(std::integral_constant<int, 1>{});
    case 2: return plan(std::integral_constant<int, 2>{});
    case 3: return plan(std::integral_constant<int, 3>{});
    case 4: return plan(std::integral_constant<int, 4>{});
    case 5: return plan(std::integral_constant<int, 5>{});
    case 6: return plan(std::integral_constant<int, 6>{});
    case 7: return plan(std::integral_constant<int, 7>{});
    case 8: return plan(std::integral_constant<int, 8>{});
    case 9: return plan(std::integral_constant<int, 9>{});
  }
  return false;
}

hipError_t launch_input_rows(const Geometry& g, const int8_t* x, void* V, const unsigned char* tab, hipStream_t s,
                             bool prepare) {
  switch (g.alg) {
    case 0: return launch_rows_alg<0, false>(g, x, V, tab, s, prepare);
    case 1: return launch_rows_alg<1, false>(g, x, V, tab, s, prepare);
    case 2: return launch_rows_alg<2, false>(g, x, V, tab, s, prepare);
    case 3: return launch_rows_alg<3, false>(g, x, V, tab, s, prepare);
    case 4: return launch_rows_alg<4, false>(g, x, V, tab, s, prepare);
    case 5: return launch_rows_alg<5, false>(g, x, V, tab, s, prepare);
    case 6: return launch_rows_alg<6, false>(g, x, V, tab, s, prepare);
    case 7: return launch_rows_alg<7, false>(g, x, V, tab, s, prepare);
    case 8: return launch_rows_alg<8, false>(g, x, V, tab, s, prepare);
    case 9: return launch_rows_alg<9, false>(g, x, V, tab, s, prepare);
  }
  return hipErrorNotSupported;
}

hipError_t launch_input_exact(const Geometry& g, const int8_t* x, void* V, const unsigned char* tab, hipStream_t s,
                              bool prepare) {
  switch (g.alg) {
    case 0: return launch_rows_alg<0, true>(g, x, V, tab, s, prepare);
    case 1: return launch_rows_alg<1, true>(g, x, V, tab, s, prepare);
    case 2: return launch_rows_alg<2, true>(g, x, V, tab, s, prepare);
    case 3: return launch_rows_alg<3, true>(g, x, V, tab, s, prepare);
    case 4: return launch_rows_alg<4, true>(g, x, V, tab, s, prepare);
    case 5: return launch_rows_alg<5, true>(g, x, V, tab, s, prepare);
    case 6: return launch_rows_alg<6, true>(g, x, V, tab, s, prepare);
    case 7: return launch_rows_alg<7, true>(g, x, V, tab, s, prepare);
    case 8: return launch_rows_alg<8, true>(g, x, V, tab, s, prepare);
    case 9: return launch_rows_alg<9, true>(g, x, V, tab, s, prepare);
  }
  return hipErrorInvalidValue;
}

}  // namespace sfc
