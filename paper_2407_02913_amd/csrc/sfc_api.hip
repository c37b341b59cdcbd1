// C ABI of the SFC library: plans, argument checks, buffer layout, stage sequencing.
// Every numeric step runs in the kernels; this file only validates, lays out buffers and
// launches.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "../../include/sfc.h"
#include "sfc_internal.hpp"
#include "sfc_mfma_input.hpp"

using sfc::FilterViews;
using sfc::Geometry;

// The filter operand as a product kernel reads it, and its dequantization factors.
struct Regrouped {
  sfc::Kernel kernel;  // which kernel, and with it the layout of both
  int filters;         // filters covered by the operand (0: none)
  int dq_filters;      // ... by the factors (0: none)
  size_t off_dq, off_U;
};

struct sfc_plan_s {
  sfc_conv_desc d;
  Geometry g;
  int esz;  // bytes per transform-domain operand: 2 exact, 1 requantized
  // filter buffer layout (byte offsets)
  size_t off_U, off_dequant, off_inv_sw, off_inv_sx, off_wscale, off_input_tab, off_tables_end, filter_bytes;
  // workspace layout
  size_t off_V, off_M, workspace_bytes;
  std::vector<float> sx, sw;  // [P], [P][Cout]
  bool scales_set;
  std::vector<float> staging;  // host image of the float tables of the filter buffer
  void* filter_dev;
  bool filter_ready;
  Regrouped op;     // of the plan's path (staged: the factors alone)
  // The library's choice of the staged path for a layer that the fused path takes: the kernel of the latter
  // (kStaged: no such choice).  Where V and M exceed the static workspace, a call from there runs the products in
  // passes of so many filters, or (0) that kernel, whose operand the plan then holds as well.
  Regrouped fused;
  int static_pass;
  float inv_y;  // 1 / output scale (SFC_OUT_I8_RELU), 0: not set
};

// Workspace of sfc_conv2d_nchw_static: part of the code object, one copy per GPU.  In host
// code this name is only a handle for hipGetSymbolAddress; the device address it yields is
// what kernels and copies get.
static __device__ __align__(256) unsigned char scratch[SFC_STATIC_WORKSPACE_BYTES];

namespace {

// Device address of `scratch` on the current device, looked up once per device; nullptr if
// the runtime refuses.
void* static_workspace() {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return nullptr;
    }
    addr[dev] = p;
  }
  return addr[dev];
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

FilterViews views(const sfc_plan_s* p, const Regrouped& op, void* filter_dev) {
  char* b = static_cast<char*>(filter_dev);
  FilterViews f;
  f.U = b + p->off_U;
  f.dequant = reinterpret_cast<float*>(b + p->off_dequant);
  f.inv_sw = reinterpret_cast<float*>(b + p->off_inv_sw);
  f.inv_sx = reinterpret_cast<float*>(b + p->off_inv_sx);
  f.wscale = reinterpret_cast<float*>(b + p->off_wscale);
  f.input_tab = reinterpret_cast<unsigned char*>(b + p->off_input_tab);
  f.dequant_single = reinterpret_cast<float*>(b + op.off_dq);
  f.U_single = b + op.off_U;
  return f;
}

// filters covered by a kernel's regrouped operand
int regrouped_filters(sfc::Kernel kernel, const Geometry& g) {
  switch (kernel) {
    case sfc::Kernel::kStaged: return 0;
    case sfc::Kernel::kFusedQuad: return sfc::quad_filter_count(g);
    case sfc::Kernel::kQuad16: return sfc::quad16_filter_count(g);
    case sfc::Kernel::kPair16: return sfc::pair16_filter_count(g);
    case sfc::Kernel::kSplitK: return sfc::splitk_filter_count(g);
    case sfc::Kernel::kProductSmall: return sfc::product_small_filter_count(g);
    case sfc::Kernel::kSingleConv: return (g.Cout + 63) / 64 * 64;
    case sfc::Kernel::kSingle16:
    case sfc::Kernel::kSingle16K:
    case sfc::Kernel::kSingleSmall: return g.Kp;
  }
  return 0;
}

// The factors of a kernel from those of the points, dequant[p][k].  pt: canonical points by processing position.
void regroup_factors(sfc::Kernel kernel, const Geometry& g, const std::vector<int>& pt, const float* dequant, float* dqs) {
  const int pp = (int)pt.size();
  if (sfc::groups_of_16(kernel)) {
    // [group of 16 filters][processing position][lane quarter q][i]: filter 16*fg + 4*i + q
    for (int k = 0; k < g.Cout; ++k) {
      const int fg = k >> 4, i = (k & 15) >> 2, q = k & 3;
      for (int j = 0; j < pp; ++j)
        dqs[((size_t)fg * pp + j) * 16 + 4 * q + i] = pt[j] < 0 ? 0.0f : dequant[(size_t)pt[j] * g.Kp + k];
    }
  } else if (kernel == sfc::Kernel::kPair16) {
    // [group of 8 filters][processing position][lane quarter q][i]: filter 8*fg + 4*i + q
    for (int k = 0; k < g.Cout; ++k)
      for (int j = 0; j < pp; ++j)
        dqs[((size_t)(k >> 3) * pp + j) * 8 + 2 * (k & 3) + ((k & 7) >> 2)] = dequant[(size_t)pt[j] * g.Kp + k];
  } else {
    // [filter][processing position]; filters beyond Cout stay zero
    for (int k = 0; k < g.Cout; ++k)
      for (int j = 0; j < pp; ++j)
        dqs[(size_t)k * pp + j] = pt[j] < 0 ? 0.0f : dequant[(size_t)pt[j] * g.Kp + k];
  }
}

hipError_t launch_repack(const Regrouped& op, const Geometry& g, const FilterViews& f, hipStream_t s) {
  if (op.filters == 0) return hipSuccess;
  if (op.kernel == sfc::Kernel::kPair16) return sfc::launch_repack_filter8(g, op.filters, f.U, f.U_single, s);
  return sfc::groups_of_16(op.kernel) ? sfc::launch_repack_filter16(g, op.filters, f.U, f.U_single, s)
                                      : sfc::launch_repack_filter(g, op.filters, f.U, f.U_single, s);
}

bool alg_is_7x7(int alg) { return alg == SFC_ALG_7X7_P132 || alg == SFC_ALG_7X7_P144; }

// Tile grid and padded extents of a description whose algorithm is fixed.  False when the
// tile count leaves the 32-bit range the kernels index with.
bool make_geometry(const sfc_conv_desc& d, Geometry* out) {
  Geometry g;
  g.N = d.N; g.Cin = d.Cin; g.Cout = d.Cout; g.H = d.H; g.W = d.W;
  g.alg = d.alg;
  const int mt = sfc::alg_tile(d.alg);
  g.th = (d.H + mt - 1) / mt;
  g.tw = (d.W + mt - 1) / mt;
  const int64_t strips = (int64_t)d.N * g.th;
  const int64_t T = strips * g.tw;
  if (T > (1ll << 30)) return false;
  g.strips = (int)strips;
  g.T = (int)T;
  g.Tp = (int)((T + 15) / 16 * 16);
  g.Cp = (d.Cin + 63) / 64 * 64;
  g.Kp = (d.Cout + 15) / 16 * 16;
  g.P = sfc::alg_points(d.alg);
  g.qmax = (float)((1 << ((d.transform_bits ? d.transform_bits : 8) - 1)) - 1);
  *out = g;
  return true;
}

// Workspace of the sums of nf filters.  (The output transform reads three-byte sums as dwords: a byte past the last.)
size_t sums_bytes(const Geometry& g, int nf, int bytes) {
  return align_up((size_t)g.P * g.Tp * nf * bytes + (bytes == 3 ? 1 : 0), 256);
}

// SFC_ALG_AUTO (3x3 filters), from per-layer timings of the ResNet shapes on one MI355X.
// Requantized mode: SFC-4's 4x4 tiles -- 46 points per tile keep two or three workgroups on a
// compute unit and the filter operand small, which outweighs even the ragged tiles of 14x14
// and 7x7 maps (256 channels at 14x14: 28.9 us against 47.5 us for 7x7 tiles at batch 64,
// 49.1 against 55.8 at batch 128; 512 channels at 7x7, batch 64: 31.2 against 38.9) -- except
// on 7x7 maps, which one 7x7 tile covers exactly, once the layer has at least 96 K (tile,
// filter) pairs: then the 31 % of surplus outputs of the ragged 4x4 tiles cost more than the
// larger point set (512 channels at 7x7, batch 256: 53.8 us with 7x7 tiles against 68.0).
// Exact mode: 6x6 tiles, the form Sec. 4 and the 3.68x figure are about.
int choose_alg(const sfc_conv_desc& d) {
  if (d.mode == SFC_MODE_EXACT) return SFC_ALG_6X6_P88;
  if (d.H == 7 && d.W == 7) {
    const int64_t pairs = (int64_t)d.N * (d.H / 7) * (d.W / 7) * d.Cout;
    // (with 512 and more channels the 7x7 tiles go through the staged path, which is ahead
    // from batch 128 on: 512 channels, 30.9 against 42.4 us with 4x4 tiles; batch 64: 28.1
    // against 25.0)
    if (pairs >= (d.Cin >= 512 ? 56 : 96) * 1024) return SFC_ALG_7X7_P132;
  }
  return SFC_ALG_4X4_P46;
}

// Staged path from the static workspace, where V and M together exceed it: filters of a pass over products and
// output transform, V and the pass's sums within the workspace; 0: the fused kernel instead.  A pass takes some 20 us
// whatever its filters, the fused kernel 30 to 40, 50 to 60 and 90 to 100 with two, four and eight chunks.  Passes against
// the fused kernel, 5x5 and 7x7 filters: eight chunks two 0.58-0.64, three 0.79-0.89, four 1.0-1.1; four chunks two
// 0.96-1.13, three 1.4-1.5; two chunks two 1.4-1.7.  (Equal passes: 256 filters as 128 and 128 57.3 us, as 144 and 112,
// three blocks of 128 in the product, 61.8.)
int static_pass_filters(const Geometry& g) {
  const size_t v = align_up((size_t)g.P * g.Tp * g.Cp, 256);
  int nf = g.Kp;
  while (nf > 0 && v + sums_bytes(g, nf, sfc::m_sum_bytes(g)) > SFC_STATIC_WORKSPACE_BYTES) nf -= 16;
  const int most = g.Cp >= 512 ? 3 : 1;
  if (nf * most < g.Kp) return 0;
  const int passes = (g.Kp + nf - 1) / nf;
  return ((g.Kp + passes - 1) / passes + 15) / 16 * 16;
}

// The 5x5- and 7x7-filter forms with 184 points: whether three kernels are ahead of the fused path.  A
// workgroup there is one chain of 184 positions, as many matrix instructions to each as there are
// chunks of 64 channels, whatever the layer's size (5x5 filters: 23 to 88 us, 7x7: 21 to 87); the three kernels of a small layer
// take 20 to 30 us and grow with M.  The lines are in workgroups of 16 tiles x 64 filters, by channel
// chunks, from 920 layers on both paths; us staged against fused there, workgroups: ratio of staged,
//   5x5   1 chunk  16: 0.79, 32: 0.93-1.02, 54: 1.0, 72: 1.3; 32 filters and less 8: 1.0, 19: 1.1;  2  17: 0.95, 38: 0.85, 76: 1.15;
//         3  54: 0.75, 76: 0.95, 120: 1.0-1.16, 168: 1.35;  4  69: 0.71, 92: 0.83-1.03, 120: 1.03, 140: 1.3;
//         5  96: 0.81, 118: 0.94, 165: 1.27;  6  56: 0.49, 119: 0.90;  7  92: 0.88;  8  56: 0.43, 112: 0.69, 181: 0.91
//   7x7   1 chunk  10: 0.81-0.89, 16: 0.96, 25: 1.05;  2  30: 0.83, 50: 0.89, 72: 1.16;  4  64: 0.64, 84: 0.85,
//         100: 1.03, 136: 1.24;  8 (one pair per lane)  64: 0.45, 124: 0.86, 174: 0.72
// The 5x5 side of the lines was measured with eight waves to a workgroup of pair16_kernel.  With four, up to 128
// workgroups, it takes 0.74 to 0.94 of that and the two meet at 4, 14, 68 and 100 workgroups with one, two, four and
// eight chunks (460 layers); between there and its line a layer takes up to 1.4 times as long as it could.
// One chunk was behind its time with one pair per lane there, so maps of more than one tile have that line (64 to 64
// channels, 24x24 maps, staged / fused / one pair per lane: eight 22.1 / 20.4 / 25.2, sixteen 25.3 / 20.8 / 25.6,
// 24 28.9 / 21.6 / 25.8, 32 31.1 / 22.0 / 26.2; 128 filters, two 20.2 / 20.5 / 29.4, four 22.1 / 20.7 / 29.2).
bool staged_ahead(const Geometry& g) {
  constexpr int kLines[2][8] = {{36, 64, 92, 104, 130, 140, 150, 170}, {18, 60, 80, 100, 0, 0, 0, 200}};
  constexpr int kFewFilters[8] = {8, 30, 75, 85, 130, 150, 200, 300};  // 5x5, up to 32 filters
  const int kc = g.Cp / 64;
  if ((g.alg != SFC_ALG_6X6_5X5_P184 && g.alg != SFC_ALG_4X4_7X7_P184) || kc > 8) return false;
  const long long workgroups = (long long)(g.Tp / 16) * ((g.Cout + 63) / 64);
  if (g.alg == SFC_ALG_4X4_7X7_P184) return workgroups < kLines[1][kc - 1];
  if (g.Cout <= 32) return workgroups < kFewFilters[kc - 1];
  return workgroups < (kc == 1 && g.th * g.tw > 1 ? 5 : kLines[0][kc - 1]);
}

// SFC_PATH_AUTO: one kernel where the layer allows it, else input transform + fused
// product/output kernel, else the staged path (exact mode, channel counts the fused
// kernel does not take).  *instead: the staged path of a layer that the fused path would take.
int choose_path(const sfc_conv_desc& d, const Geometry& g, bool* instead) {
  if (d.mode != SFC_MODE_REQUANT_I8) return SFC_PATH_STAGED;
  // (with more than 128 channels the single-kernel path repeats the input transform for
  // every 64 filters and is slower than two kernels: 51 against 30 us for 256 channels on
  // 14x14 maps at batch 64; it stays available on request)
  if (g.Cp <= 128 && sfc::single_supported(g)) return SFC_PATH_SINGLE;
  // 7x7 tiles on 7x7 maps with 512 and more channels: the fused kernel would stream its
  // operands from L2 eight times over; the products as batched GEMMs through HBM are faster
  // (64.0 against 77.0 us at batch 256)
  const bool gemm = alg_is_7x7(d.alg) && d.H < 14 && d.Cin >= 512;
  if (gemm) return SFC_PATH_STAGED;
  if (sfc::fused_quad_supported(g)) {
    *instead = staged_ahead(g);
    return *instead ? SFC_PATH_STAGED : SFC_PATH_FUSED;
  }
  // chunk counts that the fused path does not take on request: its 184-point kernels do, and quad16_kernel
  // with 46 points (192 channels on 56x56 maps, batch 32: 161 us with three kernels, 75 there)
  if ((sfc::pair16_supported(g) || sfc::quad16_supported(g)) && !staged_ahead(g)) return SFC_PATH_FUSED;
  return SFC_PATH_STAGED;
}

}  // namespace

extern "C" {

const char* sfc_status_string(sfc_status s) {
  switch (s) {
    case SFC_OK: return "ok";
    case SFC_EINVAL: return "invalid argument";
    case SFC_EUNSUPPORTED: return "unsupported configuration";
    case SFC_ENOMEM: return "host allocation failed";
    case SFC_ENOTREADY: return "scales or filter not set";
    case SFC_EHIP: return "HIP runtime or launch failure";
    case SFC_EWORKSPACE: return "device buffer smaller than the plan needs";
  }
  return "unknown status";
}

sfc_status sfc_plan(const sfc_conv_desc* desc, sfc_plan_t** out) {
  if (!desc || !out) return SFC_EINVAL;
  *out = nullptr;
  sfc_conv_desc d = *desc;
  if (d.N <= 0 || d.Cin <= 0 || d.Cout <= 0 || d.H <= 0 || d.W <= 0) return SFC_EINVAL;
  if (d.alg < SFC_ALG_AUTO || d.alg > SFC_ALG_4X4_7X7_P196) return SFC_EINVAL;
  if (d.mode != SFC_MODE_EXACT && d.mode != SFC_MODE_REQUANT_I8) return SFC_EINVAL;
  if (d.out != SFC_OUT_F32 && d.out != SFC_OUT_I32 && d.out != SFC_OUT_I8_RELU) return SFC_EINVAL;
  if (d.path < SFC_PATH_AUTO || d.path > SFC_PATH_SINGLE) return SFC_EINVAL;
  if ((d.flags & ~SFC_FLAG_EXACT_WIDE) != 0) return SFC_EINVAL;
  if (d.per_channel_wscale != 0 && d.per_channel_wscale != 1) return SFC_EINVAL;
  if (d.transform_bits != 0 && (d.transform_bits < 2 || d.transform_bits > 8)) return SFC_EINVAL;
  if (d.transform_bits != 0 && d.mode != SFC_MODE_REQUANT_I8) return SFC_EUNSUPPORTED;
  if (d.out == SFC_OUT_I32 && d.mode != SFC_MODE_EXACT) return SFC_EUNSUPPORTED;
  if (d.out == SFC_OUT_I8_RELU && d.mode != SFC_MODE_REQUANT_I8) return SFC_EUNSUPPORTED;
  if (d.path > SFC_PATH_STAGED && d.mode != SFC_MODE_REQUANT_I8) return SFC_EUNSUPPORTED;
  // Cout: one workgroup row per filter (filter transform, abs-max) must fit a launch grid
  if (d.W > 1024 || d.H > (1 << 20) || d.Cin > (1 << 16) || d.Cout > 65520)
    return SFC_EUNSUPPORTED;
  if (d.alg == SFC_ALG_AUTO) d.alg = choose_alg(d);
  if (d.mode == SFC_MODE_EXACT && !(d.flags & SFC_FLAG_EXACT_WIDE) &&
      d.Cin > (d.alg >= SFC_ALG_4X4_7X7_P184 ? 74 : d.alg >= SFC_ALG_6X6_5X5_P184 ? 145 : 404))
    return SFC_EUNSUPPORTED;

  Geometry g;
  if (!make_geometry(d, &g)) return SFC_EUNSUPPORTED;
  bool instead = false;
  if (d.path == SFC_PATH_AUTO) d.path = choose_path(d, g, &instead);
  else if (d.path == SFC_PATH_FUSED && !sfc::fused_quad_supported(g)) return SFC_EUNSUPPORTED;
  if (d.path == SFC_PATH_SINGLE && !sfc::single_supported(g)) return SFC_EUNSUPPORTED;

  sfc_plan_s* p = new (std::nothrow) sfc_plan_s();
  if (!p) return SFC_ENOMEM;
  p->d = d;
  p->g = g;
  p->esz = d.mode == SFC_MODE_EXACT ? 2 : 1;
  const size_t PK = (size_t)g.P * g.Kp;
  size_t off = 0;
  p->off_U = off;        off = align_up(off + PK * g.Cp * p->esz, 256);
  p->off_dequant = off;  off = align_up(off + PK * sizeof(float), 256);
  p->off_inv_sw = off;   off = align_up(off + PK * sizeof(float), 256);
  p->off_inv_sx = off;   off = align_up(off + g.P * sizeof(float), 256);
  p->off_wscale = off;   off = align_up(off + g.Kp * sizeof(float), 256);
  p->off_input_tab = off;
  if (d.mode == SFC_MODE_REQUANT_I8 && (d.alg == SFC_ALG_4X4_P46 || d.alg == SFC_ALG_4X4_P49))
    off = align_up(off + sfc::kInputTabBytes, 256);
  if (d.mode == SFC_MODE_REQUANT_I8 && sfc::image_input_supported(g))
    off = align_up(off + sfc::image_table_bytes(g), 256);
  if (d.mode == SFC_MODE_REQUANT_I8 && d.path != SFC_PATH_SINGLE && sfc::rows_table_offset(g) != ~0u)
    off = align_up(off + sfc::kRowsTabBytes, 256);
  if (d.mode == SFC_MODE_EXACT) off = align_up(off + sfc::kRowsTabBytes, 256);  // every algorithm
  p->op.kernel = sfc::choose_kernel(d.path, g);
  p->fused.kernel = instead ? sfc::choose_kernel(SFC_PATH_FUSED, g) : sfc::Kernel::kStaged;
  const size_t m_bytes = d.path != SFC_PATH_STAGED ? 0 : sums_bytes(g, g.Kp, instead ? sfc::m_sum_bytes(g) : 4);
  const size_t v_bytes = align_up((size_t)g.P * g.Tp * g.Cp * p->esz, 256);
  // calibration scratch (abs-max tables)
  const size_t calib = align_up((size_t)g.P * (size_t)(g.Cout > 1 ? g.Cout : 1) * 4, 256);
  const bool exceeds_static = instead && std::max(v_bytes + m_bytes, calib) > SFC_STATIC_WORKSPACE_BYTES;
  p->static_pass = exceeds_static ? static_pass_filters(g) : 0;
  p->op.filters = p->op.dq_filters = regrouped_filters(p->op.kernel, g);
  // the staged output transform reads the same [filter][position] table as fused_quad_kernel
  if (d.path == SFC_PATH_STAGED && d.mode == SFC_MODE_REQUANT_I8) p->op.dq_filters = g.Kp;
  p->fused.filters = p->fused.dq_filters =
      exceeds_static && p->static_pass == 0 && v_bytes <= SFC_STATIC_WORKSPACE_BYTES ? regrouped_filters(p->fused.kernel, g) : 0;
  // the kernels take the points in groups of four: positions up to a multiple of 4
  const size_t pp = (size_t)(g.P + 3) / 4 * 4;
  for (Regrouped* op : {&p->op, &p->fused}) {
    op->off_dq = off;
    off = align_up(off + (size_t)op->dq_filters * pp * sizeof(float), 256);
  }
  p->off_tables_end = off;
  for (Regrouped* op : {&p->op, &p->fused}) {
    op->off_U = off;
    off = align_up(off + (size_t)op->filters * pp * g.Cp, 256);
  }
  p->filter_bytes = off;
  off = 0;
  p->off_V = off;
  // the single-kernel path keeps V on chip; its workspace only serves calibration
  if (d.path != SFC_PATH_SINGLE) off += v_bytes;
  p->off_M = off;
  off += m_bytes;
  p->workspace_bytes = std::max(off, calib);
  p->scales_set = false;
  p->filter_dev = nullptr;
  p->filter_ready = false;
  p->inv_y = 0.0f;
  *out = p;
  return SFC_OK;
}

void sfc_plan_destroy(sfc_plan_t* plan) { delete plan; }

sfc_status sfc_plan_choice(const sfc_plan_t* plan, int32_t* alg, int32_t* path) {
  if (!plan) return SFC_EINVAL;
  if (alg) *alg = plan->d.alg;
  if (path) *path = plan->d.path;
  return SFC_OK;
}

sfc_status sfc_plan_sizes(const sfc_plan_t* plan, size_t* filter_bytes, size_t* workspace_bytes,
                          int32_t* P, int64_t* tiles) {
  if (!plan) return SFC_EINVAL;
  if (filter_bytes) *filter_bytes = plan->filter_bytes;
  if (workspace_bytes) *workspace_bytes = plan->workspace_bytes;
  if (P) *P = plan->g.P;
  if (tiles) *tiles = plan->g.T;
  return SFC_OK;
}

sfc_status sfc_set_point_scales(sfc_plan_t* plan, const float* sx_host, const float* sw_host) {
  if (!plan || !sx_host || !sw_host) return SFC_EINVAL;
  if (plan->d.mode != SFC_MODE_REQUANT_I8) return SFC_EUNSUPPORTED;
  const int P = plan->g.P, K = plan->g.Cout;
  auto ok = [](float s) {
    if (!(s > 0.0f) || !std::isfinite(s)) return false;
    const float inv = 1.0f / s;
    return std::isfinite(inv) && inv > 0.0f;
  };
  for (int p = 0; p < P; ++p)
    if (!ok(sx_host[p])) return SFC_EINVAL;
  for (size_t i = 0; i < (size_t)P * K; ++i)
    if (!ok(sw_host[i])) return SFC_EINVAL;
  try {
    plan->sx.assign(sx_host, sx_host + P);
    plan->sw.assign(sw_host, sw_host + (size_t)P * K);
  } catch (...) {
    return SFC_ENOMEM;
  }
  plan->scales_set = true;
  plan->filter_ready = false;
  return SFC_OK;
}

sfc_status sfc_group_scales(const sfc_plan_t* plan, int32_t act_granularity,
                            int32_t filter_granularity, float* sx_host, float* sw_host) {
  if (!plan || !sx_host || !sw_host) return SFC_EINVAL;
  if (act_granularity != SFC_ACT_PER_TENSOR && act_granularity != SFC_ACT_PER_POINT)
    return SFC_EINVAL;
  if (filter_granularity < SFC_FILTER_PER_CHANNEL || filter_granularity > SFC_FILTER_PER_CHANNEL_POINT)
    return SFC_EINVAL;
  const int P = plan->g.P, K = plan->g.Cout;
  if (act_granularity == SFC_ACT_PER_TENSOR) {
    float m = sx_host[0];
    for (int p = 1; p < P; ++p) m = sx_host[p] > m ? sx_host[p] : m;
    for (int p = 0; p < P; ++p) sx_host[p] = m;
  }
  if (filter_granularity == SFC_FILTER_PER_CHANNEL) {
    for (int k = 0; k < K; ++k) {
      float m = sw_host[k];
      for (int p = 1; p < P; ++p) m = sw_host[(size_t)p * K + k] > m ? sw_host[(size_t)p * K + k] : m;
      for (int p = 0; p < P; ++p) sw_host[(size_t)p * K + k] = m;
    }
  } else if (filter_granularity == SFC_FILTER_PER_POINT) {
    for (int p = 0; p < P; ++p) {
      float* row = sw_host + (size_t)p * K;
      float m = row[0];
      for (int k = 1; k < K; ++k) m = row[k] > m ? row[k] : m;
      for (int k = 0; k < K; ++k) row[k] = m;
    }
  }
  return SFC_OK;
}

sfc_status sfc_set_output_scale(sfc_plan_t* plan, float y_scale) {
  if (!plan) return SFC_EINVAL;
  if (plan->d.out != SFC_OUT_I8_RELU) return SFC_EUNSUPPORTED;
  if (!(y_scale > 0.0f) || !std::isfinite(y_scale)) return SFC_EINVAL;
  const float inv = 1.0f / y_scale;
  if (!std::isfinite(inv) || !(inv > 0.0f)) return SFC_EINVAL;
  plan->inv_y = inv;
  return SFC_OK;
}

sfc_status sfc_transform_filter(sfc_plan_t* plan, const int8_t* w_dev, const float* wscale_host,
                                void* filter_dev, size_t filter_bytes, void* stream) {
  if (!plan || !w_dev || !wscale_host || !filter_dev) return SFC_EINVAL;
  if (!aligned16(w_dev) || !aligned16(filter_dev)) return SFC_EINVAL;
  if (filter_bytes < plan->filter_bytes) return SFC_EWORKSPACE;
  const Geometry& g = plan->g;
  const bool requant = plan->d.mode == SFC_MODE_REQUANT_I8;
  if (requant && !plan->scales_set) return SFC_ENOTREADY;
  for (int k = 0; k < (plan->d.per_channel_wscale ? g.Cout : 1); ++k)
    if (!(wscale_host[k] > 0.0f) || !std::isfinite(wscale_host[k])) return SFC_EINVAL;

  // host image of the float tables: [dequant | inv_sw | inv_sx | wscale | input | factors], contiguous
  const size_t table_bytes = plan->off_tables_end - plan->off_dequant;
  try {
    plan->staging.assign(table_bytes / sizeof(float), 0.0f);
  } catch (...) {
    return SFC_ENOMEM;
  }
  auto table = [&](size_t off) { return plan->staging.data() + (off - plan->off_dequant) / sizeof(float); };
  float* dequant = table(plan->off_dequant);
  float* inv_sw = table(plan->off_inv_sw);
  float* inv_sx = table(plan->off_inv_sx);
  float* wscale = table(plan->off_wscale);
  for (int k = 0; k < g.Kp; ++k)
    wscale[k] = k < g.Cout ? wscale_host[plan->d.per_channel_wscale ? k : 0] : 0.0f;
  // the output transform yields den * y
  const double den = (g.alg == SFC_ALG_4X4_P46 || g.alg == SFC_ALG_4X4_P49) ? 16.0 : 36.0;
  for (int p = 0; p < g.P; ++p) {
    inv_sx[p] = requant ? 1.0f / plan->sx[p] : 1.0f;
    for (int k = 0; k < g.Kp; ++k) {
      float dq = 0.0f, inv = 1.0f;
      if (requant && k < g.Cout) {
        const float sw = plan->sw[(size_t)p * g.Cout + k];
        inv = 1.0f / sw;
        dq = (float)((double)plan->sx[p] * (double)sw * (double)wscale[k] / den);
      }
      dequant[(size_t)p * g.Kp + k] = dq;
      inv_sw[(size_t)p * g.Kp + k] = inv;
    }
  }
  if (plan->op.off_dq > plan->off_input_tab) {
    unsigned char* tab = reinterpret_cast<unsigned char*>(table(plan->off_input_tab));
    if (!requant) {
      sfc::build_rows_table(g.alg, inv_sx, tab);
    } else {
      if (g.alg == SFC_ALG_4X4_P46 || g.alg == SFC_ALG_4X4_P49) sfc::build_input_table(g.alg, inv_sx, tab);
      if (sfc::image_input_supported(g))
        sfc::build_image_input_table(g, inv_sx, tab + sfc::image_table_offset(g));
      if (plan->d.path != SFC_PATH_SINGLE && sfc::rows_table_offset(g) != ~0u)
        sfc::build_rows_table(g.alg, inv_sx, tab + sfc::rows_table_offset(g));
    }
  }
  if (plan->op.dq_filters > 0) {
    std::vector<int> pt((g.P + 3) / 4 * 4, -1);
    sfc::single_point_order(plan->d.alg, pt.data());
    for (const Regrouped* op : {&plan->op, &plan->fused})
      if (op->dq_filters > 0) regroup_factors(op->kernel, g, pt, dequant, table(op->off_dq));
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  // the kernels of this plan's path that need more than the default 64 KB of dynamic LDS
  if (requant && sfc::prepare_kernels(plan->d.path, plan->d.out, g) != hipSuccess) return SFC_EHIP;
  if (plan->fused.filters > 0 && sfc::prepare_kernels(SFC_PATH_FUSED, plan->d.out, g) != hipSuccess) return SFC_EHIP;
  if (!requant) {  // (a layer beyond its limits takes the generic kernel)
    const hipError_t e = sfc::launch_input_exact(g, nullptr, nullptr, nullptr, nullptr, true);
    if (e != hipSuccess && e != hipErrorNotSupported) return SFC_EHIP;
  }
  if (hipMemcpyAsync(static_cast<char*>(filter_dev) + plan->off_dequant, plan->staging.data(),
                     table_bytes, hipMemcpyHostToDevice, s) != hipSuccess)
    return SFC_EHIP;
  if (sfc::launch_filter_transform(plan->d.mode, g, w_dev, views(plan, plan->op, filter_dev), s) != hipSuccess)
    return SFC_EHIP;
  for (const Regrouped* op : {&plan->op, &plan->fused})
    if (launch_repack(*op, g, views(plan, *op, filter_dev), s) != hipSuccess) return SFC_EHIP;
  plan->filter_dev = filter_dev;
  plan->filter_ready = true;
  return SFC_OK;
}

// sfc_conv2d_stages.  statically: sfc_conv2d_nchw_static with a plan whose workspace exceeds the static one, in
// passes or with the fused kernel (all stages).
static sfc_status run_stages(const sfc_plan_t* plan, const int8_t* x_dev, float x_scale, void* y_dev,
                             void* workspace_dev, void* stream, int32_t stage_mask, size_t workspace_bytes,
                             bool statically) {
  if (!plan || !x_dev || !y_dev || !workspace_dev) return SFC_EINVAL;
  if (!aligned16(x_dev) || !aligned16(y_dev) || !aligned16(workspace_dev)) return SFC_EINVAL;
  if (!(x_scale > 0.0f) || !std::isfinite(x_scale)) return SFC_EINVAL;
  if (stage_mask <= 0 || stage_mask > SFC_STAGE_ALL) return SFC_EINVAL;
  if (!statically && workspace_bytes < plan->workspace_bytes) return SFC_EWORKSPACE;
  if (!plan->filter_ready) return SFC_ENOTREADY;
  if (plan->d.out == SFC_OUT_I8_RELU && plan->inv_y == 0.0f) return SFC_ENOTREADY;
  const Regrouped& op = statically && plan->static_pass == 0 ? plan->fused : plan->op;
  const bool fused = plan->d.path == SFC_PATH_FUSED || &op == &plan->fused;
  if (plan->d.path == SFC_PATH_SINGLE) {
    if (stage_mask != SFC_STAGE_ALL) return SFC_EINVAL;  // one kernel: no stage runs alone
    const FilterViews f = views(plan, op, plan->filter_dev);
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e;
    switch (op.kernel) {
      case sfc::Kernel::kSingleSmall:
        e = sfc::launch_single_small(plan->d.out, plan->g, x_dev, f, x_scale, plan->inv_y, y_dev, s);
        break;
      case sfc::Kernel::kSingle16:
        e = sfc::launch_single16(plan->d.out, plan->g, x_dev, f, x_scale, plan->inv_y, y_dev, s);
        break;
      case sfc::Kernel::kSingle16K:
        e = sfc::launch_single16k(plan->d.out, plan->g, x_dev, f, x_scale, plan->inv_y, y_dev, s);
        break;
      default: e = sfc::launch_single_conv(plan->d.out, plan->g, x_dev, f, x_scale, plan->inv_y, y_dev, s);
    }
    if (e != hipSuccess) return SFC_EHIP;
    return SFC_OK;
  }
  const int tail = stage_mask & (SFC_STAGE_PRODUCT | SFC_STAGE_OUTPUT);
  if (fused && tail != 0 && tail != (SFC_STAGE_PRODUCT | SFC_STAGE_OUTPUT)) return SFC_EINVAL;
  const Geometry& g = plan->g;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const FilterViews f = views(plan, op, plan->filter_dev);
  char* ws = static_cast<char*>(workspace_dev);
  void* V = ws + plan->off_V;
  if (stage_mask & SFC_STAGE_INPUT) {
    if (sfc::launch_input_transform(plan->d.mode, g, x_dev, V, f.inv_sx, f.input_tab, s) !=
        hipSuccess)
      return SFC_EHIP;
  }
  if (fused) {
    if (!tail) return SFC_OK;
    hipError_t e;
    switch (op.kernel) {
      case sfc::Kernel::kProductSmall:
        e = sfc::launch_product_small(plan->d.out, g, V, f, x_scale, plan->inv_y, y_dev, s);
        break;
      case sfc::Kernel::kSplitK:
        e = sfc::launch_splitk(plan->d.out, g, V, f, x_scale, plan->inv_y, y_dev, s);
        break;
      case sfc::Kernel::kQuad16:
        e = sfc::launch_quad16(plan->d.out, g, V, f, x_scale, plan->inv_y, y_dev, s);
        break;
      case sfc::Kernel::kPair16:
        e = sfc::launch_pair16(plan->d.out, g, V, f, x_scale, plan->inv_y, y_dev, s);
        break;
      default: e = sfc::launch_fused_quad(plan->d.out, g, V, f, x_scale, plan->inv_y, y_dev, s);
    }
    if (e != hipSuccess) return SFC_EHIP;
    return SFC_OK;
  }
  int32_t* M = reinterpret_cast<int32_t*>(ws + plan->off_M);
  if (plan->fused.kernel != sfc::Kernel::kStaged) {
    // int8 ties as the fused kernel of the layer rounds them (launch_quad16's product of the two scales), and its
    // order of the float32 additions
    const bool once = plan->fused.kernel == sfc::Kernel::kQuad16;
    const float xs = once && plan->d.out == SFC_OUT_I8_RELU ? 1.0f : x_scale;
    const float inv_y = once ? plan->inv_y * x_scale : plan->inv_y;
    const int pass = statically ? plan->static_pass : g.Kp;
    for (int f0 = 0; f0 < g.Cout; f0 += pass) {
      if ((stage_mask & SFC_STAGE_PRODUCT) && sfc::launch_product_gemm_i8(g, V, f.U, M, s, f0, pass) != hipSuccess)
        return SFC_EHIP;
      if ((stage_mask & SFC_STAGE_OUTPUT) &&
          sfc::launch_output_sums(plan->d.out, g, M, f, xs, inv_y, y_dev, s, false, f0, pass,
                                  plan->fused.kernel != sfc::Kernel::kFusedQuad) != hipSuccess)
        return SFC_EHIP;
    }
    return SFC_OK;
  }
  if (stage_mask & SFC_STAGE_PRODUCT) {
    if (sfc::launch_product(plan->d.mode, g, V, f.U, M, s) != hipSuccess) return SFC_EHIP;
  }
  if (stage_mask & SFC_STAGE_OUTPUT) {
    if (sfc::launch_output_transform(plan->d.mode, plan->d.out, g, M, f, x_scale,
                                     plan->inv_y, y_dev, s) != hipSuccess)
      return SFC_EHIP;
  }
  return SFC_OK;
}

sfc_status sfc_conv2d_stages(const sfc_plan_t* plan, const int8_t* x_dev, float x_scale,
                             void* y_dev, void* workspace_dev, size_t workspace_bytes, void* stream,
                             int32_t stage_mask) {
  return run_stages(plan, x_dev, x_scale, y_dev, workspace_dev, stream, stage_mask, workspace_bytes, false);
}

sfc_status sfc_conv2d_nchw(const sfc_plan_t* plan, const int8_t* x_dev, float x_scale, void* y_dev,
                           void* workspace_dev, size_t workspace_bytes, void* stream) {
  return sfc_conv2d_stages(plan, x_dev, x_scale, y_dev, workspace_dev, workspace_bytes, stream,
                           SFC_STAGE_ALL);
}

sfc_status sfc_conv2d_nchw_static(const sfc_plan_t* plan, const int8_t* x_dev, float x_scale,
                                  void* y_dev, void* stream) {
  if (!plan) return SFC_EINVAL;
  const bool exceeds = plan->workspace_bytes > SFC_STATIC_WORKSPACE_BYTES;
  if (exceeds && plan->static_pass == 0 && plan->fused.filters == 0) return SFC_EWORKSPACE;
  void* ws = static_workspace();
  if (!ws) return SFC_EHIP;
  return run_stages(plan, x_dev, x_scale, y_dev, ws, stream, SFC_STAGE_ALL, SFC_STATIC_WORKSPACE_BYTES, exceeds);
}

sfc_status sfc_tap_info(const sfc_plan_t* plan, const void* workspace_dev, int32_t which,
                        const void** ptr, int32_t* elem_bytes, int64_t dims[5],
                        int64_t strides[5]) {
  if (!plan || !ptr || !elem_bytes || !dims || !strides) return SFC_EINVAL;
  const Geometry& g = plan->g;
  const char* ws = static_cast<const char*>(workspace_dev);
  switch (which) {
    case 0:
      if (!workspace_dev) return SFC_EINVAL;
      if (plan->d.path == SFC_PATH_SINGLE) return SFC_EUNSUPPORTED;
      *ptr = ws + plan->off_V;
      *elem_bytes = plan->esz;
      dims[0] = g.P; dims[1] = g.Tp; dims[2] = 1; dims[3] = g.Cp; dims[4] = 1;
      strides[0] = (int64_t)g.Tp * g.Cp; strides[1] = g.Cp; strides[2] = 0; strides[3] = 1;
      strides[4] = 0;
      return SFC_OK;
    case 1:
      if (!plan->filter_ready) return SFC_ENOTREADY;
      *ptr = static_cast<const char*>(plan->filter_dev) + plan->off_U;
      *elem_bytes = plan->esz;
      dims[0] = g.P; dims[1] = g.Kp; dims[2] = 1; dims[3] = g.Cp; dims[4] = 1;
      strides[0] = (int64_t)g.Kp * g.Cp; strides[1] = g.Cp; strides[2] = 0; strides[3] = 1;
      strides[4] = 0;
      return SFC_OK;
    case 2:
      if (!workspace_dev) return SFC_EINVAL;
      if (plan->d.path != SFC_PATH_STAGED) return SFC_EUNSUPPORTED;
      *ptr = ws + plan->off_M;
      *elem_bytes = plan->d.mode == SFC_MODE_REQUANT_I8 ? sfc::m_sum_bytes(g) : 4;
      dims[0] = g.P;
      strides[0] = (int64_t)g.Tp * g.Kp;
      // [P][tile block][filter quad][16 tiles][4 filters]
      dims[1] = g.Tp / 16; dims[2] = 16; dims[3] = g.Kp / 4; dims[4] = 4;
      strides[1] = (int64_t)g.Kp * 16; strides[2] = 4; strides[3] = 64; strides[4] = 1;
      return SFC_OK;
    default:
      return SFC_EINVAL;
  }
}

sfc_status sfc_stream_copy(void* dst_dev, const void* src_dev, size_t bytes, void* stream) {
  if (!dst_dev || !src_dev) return SFC_EINVAL;
  if (!aligned16(dst_dev) || !aligned16(src_dev) || (bytes & 15u) != 0) return SFC_EINVAL;
  if (sfc::launch_stream_copy(dst_dev, src_dev, bytes, static_cast<hipStream_t>(stream)) !=
      hipSuccess)
    return SFC_EHIP;
  return SFC_OK;
}

static sfc_status maxima_to_scales(const int32_t* dev, size_t count, float qmax, hipStream_t s,
                                   float* out) {
  std::vector<int32_t> host;
  try {
    host.resize(count);
  } catch (...) {
    return SFC_ENOMEM;
  }
  if (hipMemcpyAsync(host.data(), dev, count * sizeof(int32_t), hipMemcpyDeviceToHost, s) !=
      hipSuccess)
    return SFC_EHIP;
  if (hipStreamSynchronize(s) != hipSuccess) return SFC_EHIP;
  for (size_t i = 0; i < count; ++i)
    out[i] = host[i] == 0 ? 1.0f : (float)host[i] / qmax;
  return SFC_OK;
}

sfc_status sfc_calibrate_act_scales(const sfc_plan_t* plan, const int8_t* x_dev, int32_t n_images,
                                    void* workspace_dev, size_t workspace_bytes, void* stream,
                                    float* sx_host_out) {
  if (!plan || !x_dev || !workspace_dev || !sx_host_out) return SFC_EINVAL;
  if (!aligned16(x_dev) || !aligned16(workspace_dev)) return SFC_EINVAL;
  if (n_images <= 0 || n_images > plan->g.N) return SFC_EINVAL;
  if (workspace_bytes < plan->workspace_bytes) return SFC_EWORKSPACE;
  Geometry g = plan->g;
  g.N = n_images;
  g.strips = n_images * g.th;
  g.T = g.strips * g.tw;
  g.Tp = (g.T + 15) / 16 * 16;
  hipStream_t s = static_cast<hipStream_t>(stream);
  int32_t* maxima = static_cast<int32_t*>(workspace_dev);
  if (sfc::launch_act_absmax(g, x_dev, maxima, s) != hipSuccess) return SFC_EHIP;
  return maxima_to_scales(maxima, g.P, g.qmax, s, sx_host_out);
}

sfc_status sfc_calibrate_filter_scales(const sfc_plan_t* plan, const int8_t* w_dev,
                                       void* workspace_dev, size_t workspace_bytes, void* stream,
                                       float* sw_host_out) {
  if (!plan || !w_dev || !workspace_dev || !sw_host_out) return SFC_EINVAL;
  if (!aligned16(w_dev) || !aligned16(workspace_dev)) return SFC_EINVAL;
  if (workspace_bytes < plan->workspace_bytes) return SFC_EWORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  int32_t* maxima = static_cast<int32_t*>(workspace_dev);
  if (sfc::launch_filter_absmax(plan->g, w_dev, maxima, s) != hipSuccess)
    return SFC_EHIP;
  return maxima_to_scales(maxima, (size_t)plan->g.P * plan->g.Cout, plan->g.qmax, s, sw_host_out);
}

}  // extern "C"
