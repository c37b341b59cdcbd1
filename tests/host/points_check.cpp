// Host-side dump of the linear maps realized by the kernels' add networks
// (sfc_points.hpp), so that a CPU test can compare them with the oracle's
// matrices.  Prints, for every ALG (0: 6x6/88, 1: 6x6/100, 2: 7x7/132, 3: 7x7/144,
// 4: 4x4/46, 5: 4x4/49, 6: 6x6 with 5x5 filter/184, 7: the same/196, 8: 4x4 with 7x7
// filter/184, 9: the same/196):
//   B <alg> <p> <NI*NI ints>   input transform row p  (impulse responses)
//   G <alg> <p> <R*R ints>     filter transform row p
//   A <alg> <p> <M*M ints>     output transform row p (times 36; times 16 for 4x4)
//   S <alg> <p> <M*M ints>     the same row through the streaming form of the fused kernels
//                              (products fed in processing order, stream_vertical + stream_row)
//   O <alg> <p> <M*M ints>     4, 5, 6, 8: the same through stream_outputs4 and stream_outputs, which
//                              keep the outputs
//   F <alg> <0> <2 ints>       4, 5: outputs of both streaming forms, of all that were compared, whose
//                              float32 sums are not those of collapse4_rows and inv4_outputs bit for bit
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

#include "../../paper_2407_02913_amd/csrc/sfc_points.hpp"
#include "../../paper_2407_02913_amd/csrc/sfc_stream_outputs.hpp"

using namespace sfc;

// SFC-4: the outputs of products m (canonical order) from collapse4_rows and inv4_outputs alone, the
// vertical axis first, as the kernels for small layers add them.
template <int ALG>
void rounded_outputs4(const std::vector<float>& m, float (&y)[4][4]) {
  constexpr bool kHermitian = AlgTraits<ALG>::kHermitian;
  auto at = [&](int r1, int r2) { return m[kHermitian ? kept_index4(r1, r2) : 7 * r1 + r2]; };
  float z[6][4], c0[6], c1[6];
  for (int j = 0; j < 4; ++j) {
    float col[7], cc[6];
    for (int r1 = 0; r1 < 7; ++r1) col[r1] = at(r1, real_row4(j));
    collapse4_rows(col, cc);
    inv4_outputs(cc, z[real_comp4(j)]);
  }
  float h0[7] = {}, h1[7] = {};
  for (int r1 = 0; r1 < 7; ++r1)
    if (!kHermitian || !row4_is_complex(r1)) {
      h0[r1] = at(r1, 4) - at(r1, 3);
      h1[r1] = at(r1, 2) - at(r1, 4) - at(r1, 3);
    }
  collapse4_rows(h0, c0);
  collapse4_rows(h1, c1);
  if (kHermitian) {
    const float* b = &m[AlgTraits<ALG>::P - 6];
    const float uo0 = b[0] - b[1], uo1 = b[2] - b[0] - b[1];
    const float vo0 = b[3] - b[4], vo1 = b[5] - b[3] - b[4];
    c0[2] = 0.5f * (uo0 + vo0);
    c0[3] = 0.5f * (uo1 + vo1);
    c1[2] = 0.5f * (uo1 - vo1);
    c1[3] = 0.5f * (vo0 - uo0);
  }
  inv4_outputs(c0, z[2]);
  inv4_outputs(c1, z[3]);
  for (int o1 = 0; o1 < 4; ++o1) {
    float zc[6];
    for (int b = 0; b < 6; ++b) zc[b] = z[b][o1];
    inv4_outputs(zc, y[o1]);
  }
}

template <int ALG>
void compare_rounding() {
  constexpr Order<ALG> order{};
  std::mt19937 gen(7);
  std::uniform_real_distribution<float> uniform(-1.0f, 1.0f);
  int differ = 0, compared = 0;
  for (int trial = 0; trial < 500; ++trial) {
    std::vector<float> m(AlgTraits<ALG>::P);
    for (float& v : m) v = std::ldexp(uniform(gen), (int)(gen() % 8));
    float want[4][4], z[6][4], columns[4][4];
    rounded_outputs4<ALG>(m, want);
    int j = 0;
    auto next = [&]() -> float { return m[order.pt[j++]]; };
    stream_vertical<ALG, float>(next, z);
    j = 0;
    stream_outputs4<ALG, float>(next, [](float&) {}, columns);
    for (int o1 = 0; o1 < 4; ++o1) {
      float out[4], kept[4];
      stream_row<ALG, float>(z, o1, out);
      stream_row<kOutputColumns + 4, float>(columns, o1, kept);
      for (int o2 = 0; o2 < 4; ++o2) {
        differ += std::memcmp(&out[o2], &want[o1][o2], 4) != 0;
        differ += std::memcmp(&kept[o2], &want[o1][o2], 4) != 0;
        compared += 2;
      }
    }
  }
  std::printf("F %d 0 %d %d\n", ALG, differ, compared);
}

template <int ALG>
void dump() {
  using Tr = AlgTraits<ALG>;
  constexpr int P = Tr::P, NI = Tr::NI, NC = Tr::NC, M = Tr::M, R = Tr::R;
  std::vector<std::vector<int>> B(P, std::vector<int>(NI * NI)), G(P, std::vector<int>(R * R)),
      A(P, std::vector<int>(M * M));
  for (int i = 0; i < NI; ++i)
    for (int j = 0; j < NI; ++j) {
      int x[NI][NI] = {};
      x[i][j] = 1;
      int half[NI][NC], comp[NC][NC];
      for (int r = 0; r < NI; ++r) fwd_input<NI, NC>(x[r], half[r]);
      for (int b = 0; b < NC; ++b) {
        int col[NI], cc[NC];
        for (int r = 0; r < NI; ++r) col[r] = half[r][b];
        fwd_input<NI, NC>(col, cc);
        for (int a = 0; a < NC; ++a) comp[a][b] = cc[a];
      }
      for_each_point<ALG>(comp, [&](int p, int v) { B[p][i * NI + j] = v; });
    }
  for (int i = 0; i < R; ++i)
    for (int j = 0; j < R; ++j) {
      int f[R][R] = {};
      f[i][j] = 1;
      int half[R][NC], comp[NC][NC];
      for (int r = 0; r < R; ++r) fwd_filter<R, NC>(f[r], half[r]);
      for (int b = 0; b < NC; ++b) {
        int col[R], cc[NC];
        for (int r = 0; r < R; ++r) col[r] = half[r][b];
        fwd_filter<R, NC>(col, cc);
        for (int a = 0; a < NC; ++a) comp[a][b] = cc[a];
      }
      for_each_point<ALG>(comp, [&](int p, int v) { G[p][i * R + j] = v; });
    }
  for (int q = 0; q < P; ++q) {
    float out[M][M];
    output_transform<ALG, float>([&](int p) { return p == q ? 3.0f : 0.0f; }, out);
    for (int o = 0; o < M * M; ++o) A[q][o] = (int)std::lround(out[o / M][o % M] / 3.0f);
  }
  constexpr Order<ALG> order{};
  for (int q = 0; q < P; ++q) {
    int j = 0;
    auto next = [&]() -> float { return order.pt[j++] == q ? 3.0f : 0.0f; };
    float z[NC][M];
    stream_vertical<ALG, float>(next, z);
    std::printf("S %d %d", ALG, q);
    for (int o1 = 0; o1 < M; ++o1) {
      float out[M];
      stream_row<ALG, float>(z, o1, out);
      for (int o2 = 0; o2 < M; ++o2) std::printf(" %d", (int)std::lround(out[o2] / 3.0f));
    }
    std::printf("\n");
    if (q == 0 && j != P) std::printf("S %d -1 %d\n", ALG, j);  // must consume exactly P products
  }
  if constexpr (ALG == 6 || ALG == 8 || Tr::kFamily == 4) {
    for (int q = 0; q < P; ++q) {
      int j = 0;
      auto next = [&]() -> float { return order.pt[j++] == q ? 3.0f : 0.0f; };
      float y[M][M];
      if constexpr (Tr::kFamily == 4) stream_outputs4<ALG, float>(next, [](float&) {}, y);
      else stream_outputs<ALG, float>(next, [](float&) {}, y);
      std::printf("O %d %d", ALG, q);
      for (int o1 = 0; o1 < M; ++o1) {
        float out[M];
        stream_row<kOutputColumns + M, float>(y, o1, out);
        for (int o2 = 0; o2 < M; ++o2) std::printf(" %d", (int)std::lround(out[o2] / 3.0f));
      }
      std::printf("\n");
      if (q == 0 && j != P) std::printf("O %d -1 %d\n", ALG, j);
    }
  }
  for (int j = P; j < Order<ALG>::PP; ++j)
    if (order.pt[j] != -1) std::printf("S %d -2 %d\n", ALG, j);
  for (int p = 0; p < P; ++p) {
    std::printf("B %d %d", ALG, p);
    for (int v : B[p]) std::printf(" %d", v);
    std::printf("\nG %d %d", ALG, p);
    for (int v : G[p]) std::printf(" %d", v);
    std::printf("\nA %d %d", ALG, p);
    for (int v : A[p]) std::printf(" %d", v);
    std::printf("\n");
  }
}

int main() {
  dump<0>();
  dump<1>();
  dump<2>();
  dump<3>();
  dump<4>();
  dump<5>();
  dump<6>();
  dump<7>();
  dump<8>();
  dump<9>();
  compare_rounding<4>();
  compare_rounding<5>();
  return 0;
}
