// Streaming output transform that keeps the outputs themselves (SFC-6(4x4,7x7) and SFC-6(6x6,5x5),
// 184 points; SFC-4).
//
// stream_vertical (sfc_points.hpp) leaves NC x M values per pair for the inverse along the
// horizontal axis; with the 12 components of this form that is 48 registers a pair.  Here a
// component is added to the M output columns as soon as its vertical outputs exist: 16
// registers a pair, with as many additions, which is what lets a lane own four pairs
// (sfc_quad16.hpp).  (The 36 outputs of a 6x6 tile do not leave a lane the registers for four:
// SFC-6(6x6,5x5) spilled 55 this way; a lane owns two, sfc_pair16.hip.)
#pragma once
#include "sfc_points.hpp"

namespace sfc {

// "Algorithm" kOutputColumns + M of the store functions, which take a pair as z[b][o1] and
// ask stream_row for an output row: here z[o2][o1] are the outputs, column by column.
constexpr int kOutputColumns = 100;
template <>
struct AlgTraits<kOutputColumns + 4> {
  static constexpr int NC = 4, M = 4;
};
template <>
SFC_HD void stream_row<kOutputColumns + 4, float>(const float (&z)[4][4], int o1, float (&out)[4]) {
#pragma unroll
  for (int o = 0; o < 4; ++o) out[o] = z[o][o1];
}
template <>
struct AlgTraits<kOutputColumns + 6> {
  static constexpr int NC = 6, M = 6;
};
template <>
SFC_HD void stream_row<kOutputColumns + 6, float>(const float (&z)[6][6], int o1, float (&out)[6]) {
#pragma unroll
  for (int o = 0; o < 6; ++o) out[o] = z[o][o1];
}

// The inverse along one axis (inv_outputs of 12 components), one component after the other.
// Outputs, e and d as in inv_outputs: e0 - d0, e1 - d1, e2 - d2, e0 + d0 with four of them, with six
// e1 + d1, e2 + d2 and then these four.

// components 0 and 5 (d0, d1, d2 take component 5 as -, +, -)
template <int M, typename T>
SFC_HD void start_outputs(const T& c0, const T& c5, T (&v)[M]) {
  const T s = c0 + c5, d = c0 - c5;
#pragma unroll
  for (int o = 0; o < M; ++o) v[o] = o % 2 == 0 ? s : d;
}
// components 1 and 2 (G = 0: d) or 3 and 4 (G = 1: e)
template <int G, int M, typename T>
SFC_HD void add_complex(const T& a, const T& b, T (&v)[M]) {
  T w0, w1, w2;
  if constexpr (G == 0) {
    w0 = a - b;
    w1 = -a - b - b;
    w2 = -a - a - b;
  } else {
    w0 = -a - b - b;
    w1 = b - a;
    w2 = a + a + b;
  }
  static_assert(M == 4 || M == 6, "outputs of SFC-6(4x4,7x7) and SFC-6(6x6,5x5)");
  constexpr int F = M - 4;  // the first of the last four
  if constexpr (M == 6) {
    v[0] = v[0] + w1;
    v[1] = v[1] + w2;
  }
  v[F] = G == 0 ? v[F] - w0 : v[F] + w0;
  v[F + 1] = G == 0 ? v[F + 1] - w1 : v[F + 1] + w1;
  v[F + 2] = G == 0 ? v[F + 2] - w2 : v[F + 2] + w2;
  v[F + 3] = v[F + 3] + w0;
}
// the output that correction component B (6 ... 11) is added to, six times
template <int B, int M>
SFC_HD constexpr int corrected_output() {
  return (B == 6 || B == 8) ? 0 : B == 7 ? 1 : B == 10 ? M - 2 : M - 1;
}

// hermitian_collapse behind its subtractions
template <typename T>
SFC_HD void hermitian_components(const T& uo0, const T& uo1, const T& vo0, const T& vo1, T& o00, T& o10,
                                 T& o01, T& o11) {
  const T du = uo1 - vo1, dv = vo0 - uo0;
  o01 = Third<T>::apply(du + du - dv);
  o11 = Third<T>::apply(dv + dv - du);
  o00 = uo0 + o11;
  o10 = vo1 + o01;
}

// Consumes the products in processing order (as stream_vertical does) and leaves
// y[o2][o1] = 36 times output (o1, o2).  settle(v) is called on every value that stays until a
// later product: it keeps the compiler from putting the additions off and the products in
// registers instead (quad16_kernel at 64 / 128 / 256 channels: 188 / 214 / 253 vector registers,
// 196 / 218 / 253 without it, none spilled).
template <int ALG, typename T, typename F, typename Settle>
SFC_HD void stream_outputs(F&& next, Settle&& settle, T (&y)[AlgTraits<ALG>::M][AlgTraits<ALG>::M]) {
  using Tr = AlgTraits<ALG>;
  static_assert(Tr::NC == 12 && Tr::kHermitian, "the forms with 184 points");
  constexpr int NR = Tr::NR, NREAL = Tr::NREAL, M = Tr::M;
  auto settle_all = [&](T (&v)[M]) {
#pragma unroll
    for (int o = 0; o < M; ++o) settle(v[o]);
  };
  T dc[M];  // column component 0
  static_for<NREAL>([&](auto jc) {
    constexpr int j = decltype(jc)::value, b = real_comp(j), J0 = NR * j;
    T v[M];
    {
      const T r0 = take_product<J0>(next), r1 = take_product<J0 + 1>(next),
              r2 = take_product<J0 + 2>(next), r3 = take_product<J0 + 3>(next);
      T c1 = r1 - r2, c2 = r3 - r1;
      settle(c1);
      settle(c2);
      const T r4 = take_product<J0 + 4>(next), r5 = take_product<J0 + 5>(next),
              r6 = take_product<J0 + 6>(next);
      T c3 = r4 - r5, c4 = r6 - r4;
      settle(c3);
      settle(c4);
      start_outputs(r0, take_product<J0 + 7>(next), v);
      add_complex<0>(c1, c2, v);
      add_complex<1>(c3, c4, v);
      settle_all(v);
    }
    static_for<NREAL - 2>([&](auto rc) {
      constexpr int i = decltype(rc)::value;
      T& o = v[corrected_output<6 + i, M>()];
      o = o + T(6) * take_product<J0 + 8 + i>(next);
      settle(o);
    });
#pragma unroll
    for (int o = 0; o < M; ++o) {
      if constexpr (b == 0) {
        dc[o] = v[o];
      } else if constexpr (b == 5) {
        T col[M];
        start_outputs(dc[o], v[o], col);
#pragma unroll
        for (int c = 0; c < M; ++c) y[c][o] = col[c];
      } else {
        T& out = y[corrected_output<b, M>()][o];
        out = out + T(6) * v[o];
        settle(out);
      }
    }
  });
  constexpr int GSZ = 3 * NREAL + 12;
  static_for<2>([&](auto gc) {
    constexpr int g2 = decltype(gc)::value;
    constexpr int J0 = NREAL * NR + g2 * GSZ;
    T v0[M], v1[M];
    T dc0, dc1;
    static_for<NREAL>([&](auto jc) {
      constexpr int j = decltype(jc)::value, a = real_comp(j);
      const T m0 = take_product<J0 + 3 * j>(next), m1 = take_product<J0 + 3 * j + 1>(next),
              m2 = take_product<J0 + 3 * j + 2>(next);
      const T c0 = m0 - m1, c1 = m2 - m0;
      if constexpr (a == 0) {
        dc0 = c0;
        dc1 = c1;
        settle(dc0);
        settle(dc1);
      } else if constexpr (a == 5) {
        start_outputs(dc0, c0, v0);
        start_outputs(dc1, c1, v1);
      } else {
        constexpr int o = corrected_output<a, M>();
        v0[o] = v0[o] + T(6) * c0;
        v1[o] = v1[o] + T(6) * c1;
        settle(v0[o]);
        settle(v1[o]);
      }
    });
    static_for<2>([&](auto g1c) {
      constexpr int g1 = decltype(g1c)::value;
      constexpr int J1 = J0 + 3 * NREAL + 6 * g1;
      const T m0 = take_product<J1>(next), m1 = take_product<J1 + 1>(next),
              m2 = take_product<J1 + 2>(next);
      T uo0 = m0 - m1, uo1 = m2 - m0;
      settle(uo0);
      settle(uo1);
      const T m3 = take_product<J1 + 3>(next), m4 = take_product<J1 + 4>(next),
              m5 = take_product<J1 + 5>(next);
      T c00, c10, c01, c11;
      hermitian_components(uo0, uo1, m3 - m4, m5 - m3, c00, c10, c01, c11);
      add_complex<g1>(c00, c10, v0);
      add_complex<g1>(c01, c11, v1);
      settle_all(v0);
      settle_all(v1);
    });
#pragma unroll
    for (int o = 0; o < M; ++o) {
      T col[M];
#pragma unroll
      for (int c = 0; c < M; ++c) col[c] = y[c][o];
      add_complex<g2>(v0[o], v1[o], col);
#pragma unroll
      for (int c = 0; c < M; ++c) {
        y[c][o] = col[c];
        settle(y[c][o]);
      }
    }
  });
}

// The same for SFC-4: y[o2][o1] = 16 times output (o1, o2).  The complex column group comes first, so
// at most 21 values of a pair are kept at any time (8 of the group, 4 of column 0, column 1 on the
// way; from then on the 16 outputs and one column) where stream_vertical ends with 24.
template <int ALG, typename T, typename F, typename Settle>
SFC_HD void stream_outputs4(F&& next, Settle&& settle, T (&y)[4][4]) {
  static_assert(AlgTraits<ALG>::kFamily == 4, "SFC-4");
  Vertical4<T> va, vb, v0;
  stream_complex4<ALG, T>(next, settle, va, vb);
  stream_real4<ALG, 0, T>(next, settle, v0);
  {
    Vertical4<T> v1;
    stream_real4<ALG, 1, T>(next, settle, v1);
#pragma unroll
    for (int o1 = 0; o1 < 4; ++o1) {
      Vertical4<T> row;  // the same inverse along the row
      row.v[0] = v0.v[o1] + v1.v[o1];
      row.v[1] = v0.v[o1] - v1.v[o1];
      row.complex(va.v[o1] + va.v[o1], vb.v[o1] + vb.v[o1]);
#pragma unroll
      for (int o2 = 0; o2 < 4; ++o2) {
        y[o2][o1] = row.v[o2];
        settle(y[o2][o1]);
      }
    }
  }
  static_for<2>([&](auto jc) {
    constexpr int j = decltype(jc)::value;
    Vertical4<T> v;
    stream_real4<ALG, 2 + j, T>(next, settle, v);
#pragma unroll
    for (int o1 = 0; o1 < 4; ++o1) {
      T& o = y[j == 0 ? 0 : 3][o1];
      o = o + T(4) * v.v[o1];
      settle(o);
    }
  });
}

}  // namespace sfc
