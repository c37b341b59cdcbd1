// Which kernels the library picks: reads layers "path alg N Cin Cout H W" (path and alg as in
// include/sfc.h) and prints the name of the product kernel of each, for the exact mode of the
// layer which output transform is ahead, the form of single16_kernel that it would take, and the kernels of its
// input transform, requantized and exact.  Linked against the built library, whose own rules it asks.
#include <cstdio>

#include "../../paper_2407_02913_amd/csrc/sfc_internal.hpp"
#include "../../paper_2407_02913_amd/csrc/sfc_points.hpp"

int main() {
  static const char* const kNames[] = {"staged",      "fused_quad", "quad16",     "splitk",      "product_small",
                                       "single_conv", "single16",   "single16k", "single_small", "pair16"};
  static const char* const kInputs[] = {"image", "waves", "rows", "generic"};
  int path;
  sfc::Geometry g{};
  while (std::scanf("%d %d %d %d %d %d %d", &path, &g.alg, &g.N, &g.Cin, &g.Cout, &g.H, &g.W) == 7) {
    const int m = sfc::alg_tile(g.alg);
    g.th = (g.H + m - 1) / m;
    g.tw = (g.W + m - 1) / m;
    g.strips = g.N * g.th;
    g.T = g.strips * g.tw;
    g.Tp = (g.T + 15) / 16 * 16;
    g.Cp = (g.Cin + 63) / 64 * 64;
    g.Kp = (g.Cout + 15) / 16 * 16;
    g.P = sfc::alg_points(g.alg);
    g.qmax = 127.0f;
    std::printf("%s %s %s %s %s\n", kNames[(int)sfc::choose_kernel(path, g)], sfc::output_exact_ahead(g) ? "waves" : "threads",
                sfc::single16_few_workgroups(g) ? "few" : "many", kInputs[(int)sfc::choose_input_kernel(false, g)],
                kInputs[(int)sfc::choose_input_kernel(true, g)]);
  }
  return 0;
}
