// Rounding of the column transforms on the CPU: the relative L2 error of a column's round trip (forward
// transform, unit phases, inverse, aperture rows) against double precision, of the split transforms
// (csrc/col_fft.hpp) and of the staged ones (csrc/fft.hpp), both as the kernels compute them; and of the
// staged transforms of 64 and 96 points against other radices.  Also the split of 800-point halves
// phase by phase: its forward transform against the DFT, its LDS slots and their banks.
// Prints "name ratio" lines (split over staged; plan over other radices) and "forward800 error".
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstdio>
#include <random>
#include <set>
#include <vector>

#include "col_fft.hpp"

using namespace dpx;
typedef std::complex<double> cd;
typedef std::vector<float2> Column;

static double forward800 = 0.0;
static int failures = 0;

// one Stockham stage of radix R after stages of total size ns (tw: its twiddles, (r - 1) ns + k)
template <int R, bool INV, bool HALF>
void stage(Column& x, int& ns, const float2* tw) {
  const int M = static_cast<int>(x.size());
  Column y(M);
  for (int j = 0; j < M / R; ++j) {
    const int k = j % ns;
    float2 v[R];
    for (int r = 0; r < R; ++r) v[r] = x[j + r * (M / R)];
    if (ns > 1)
      for (int r = 1; r < R; ++r) v[r] = INV ? cmulc(v[r], tw[(r - 1) * ns + k]) : cmul(v[r], tw[(r - 1) * ns + k]);
    DFT<R, INV, HALF && R % 2 == 0>::run(v);
    for (int r = 0; r < R; ++r) y[(j / ns) * ns * R + k + r * ns] = v[r];
  }
  x = y;
  ns *= R;
}

// the staged transform with the radices of the length's plan
template <int M, bool INV, bool HALF>
void staged(Column& x) {
  Column tw;
  twiddle_table_host<M, 0>(tw);
  int ns = 1;
  static_for<0, Radix<M, 0>::NST>([&](auto st) {
    constexpr int ST = decltype(st)::value;
    stage<Radix<M, 0>::R[ST], INV, HALF && ST == 0>(x, ns, tw.data() + twiddle_offset<M, 0>(ST));
  });
}

// and with given ones
template <bool INV, bool HALF, int R>
void given_stage(Column& x, int& ns) {
  Column tw((R - 1) * ns);
  for (int r = 1; r < R; ++r)
    for (int k = 0; k < ns; ++k) tw[(r - 1) * ns + k] = unit_root(UnitRoots(static_cast<int>(x.size())), r * k, ns * R);
  if (ns == 1) stage<R, INV, HALF>(x, ns, tw.data());
  else stage<R, INV, false>(x, ns, tw.data());
}
template <bool INV, bool HALF, int... R>
void given(Column& x) {
  int ns = 1;
  (given_stage<INV, HALF, R>(x, ns), ...);
}

// phases of 800-point halves: h by h, rows to frequencies, the phases, back to the rows
template <int M, int PAD, typename F>
Column split_halves_of_800(const Column& x, const Column& tab, F&& product) {
  using G = ColSplit800<M, PAD>;
  constexpr int R1 = G::R1, R2 = G::R2, LEN = G::LEN;
  Column acc(LEN);
  for (int h = 0; h < 2; ++h) {
    Column lds(G::REG);
    for (int j = 0; j < R2; ++j) {
      float2 v[R1];
      for (int r = 0; r < R1; ++r) v[r] = x[j + R2 * r];
      if (h) dft_odd<R1>(v);
      else DFT<R1, false, false>::run(v);
      for (int k = 0; k < R1; ++k) lds[G::slot(k, j)] = v[k];
    }
    for (int k1 = 0; k1 < R1; ++k1) {
      float2 f[R2], p[R2 / 2];
      for (int i = 0; i < R2; ++i) f[i] = lds[G::slot(k1, i)];
      for (int e = 0; e < R2 / 2; ++e) p[e] = tab[(e * G::NH + h) * 32 + k1];
      dft_fused<R2, false>(f, p);
      for (int k2 = 0; k2 < R2; ++k2) f[k2] = product(2 * (k1 + R1 * k2) + h, f[k2]);
      DFT<R2, true, false>::run(f);
      for (int i = 0; i < R2; ++i) lds[G::slot(k1, i)] = f[i];
    }
    for (int j = 0; j < R2; ++j) {
      float2 y[R1];
      for (int k = 0; k < R1; ++k) y[k] = lds[G::slot(k, j)];
      for (int k = 1; k < R1; ++k) y[k] = cmulc(y[k], tab[G::OFF_C + (k - 1) * 32 + j]);
      DFT<R1, true, false>::run(y);
      for (int r = 0; r < R1; ++r) {
        const float2 w = tab[G::OFF_W + j + R2 * r];
        float2& a = acc[j + R2 * r];
        a = h ? make_float2(fmaf(w.y, y[r].y, fmaf(w.x, y[r].x, a.x)), fmaf(-w.y, y[r].x, fmaf(w.x, y[r].y, a.y))) : y[r];
      }
    }
  }
  return acc;
}

template <int M, int PAD, typename F>
Column split_halves_of_512(const Column& x, const Column& tab, F&& product) {
  using G = ColSplit3<M, PAD>;
  constexpr int NH = G::NH;
  Column acc(G::LEN);
  for (int h = 0; h < NH; ++h) {
    Column lds(G::REG);
    for (int j = 0; j < 64; ++j) {
      float2 v[8];
      for (int r = 0; r < 8; ++r) v[r] = x[j + 64 * r];
      if (h) dft_odd<8>(v);
      else DFT<8, false, false>::run(v);
      for (int k = 0; k < 8; ++k) lds[G::slot(k, j)] = v[k];
    }
    auto lanes = [&](auto body) {  // every lane reads before any writes
      Column out(lds);
      for (int l = 0; l < 64; ++l) body(l & 7, l >> 3, l, out);
      lds = out;
    };
    lanes([&](int k1, int j1, int, Column& out) {
      float2 f[8];
      for (int i = 0; i < 8; ++i) f[i] = lds[G::slot(k1, j1 + 8 * i)];
      dft8_table<false>(f, tab.data() + h * 8 + k1, NH * 8);
      for (int i = 0; i < 8; ++i) out[G::slot(k1, j1 + 8 * i)] = f[i];
    });
    lanes([&](int k1, int m, int lane, Column& out) {
      float2 f[8];
      for (int i = 0; i < 8; ++i) f[i] = lds[G::slot(k1, i + 8 * m)];
      dft8_table<false>(f, tab.data() + G::OFF_B2 + h * 64 + lane, NH * 64);
      for (int q = 0; q < 8; ++q) f[q] = product(NH * (lane + 64 * q) + h, f[q]);
      DFT<8, true, false>::run(f);
      for (int i = 0; i < 8; ++i) out[G::slot(k1, i + 8 * m)] = f[i];
    });
    lanes([&](int k1, int j1, int, Column& out) {
      float2 f[8];
      for (int i = 0; i < 8; ++i) f[i] = lds[G::slot(k1, j1 + 8 * i)];
      dft8_table<true>(f, tab.data() + G::OFF_R + j1, 8);
      for (int i = 0; i < 8; ++i) out[G::slot(k1, j1 + 8 * i)] = f[i];
    });
    for (int j = 0; j < 64; ++j) {
      float2 y[8];
      for (int k = 0; k < 8; ++k) y[k] = lds[G::slot(k, j)];
      dft8_table<true>(y, tab.data() + G::OFF_C + j, 64);
      for (int r = 0; r < 8; ++r) {
        float2& a = acc[j + 64 * r];
        if (h == 0) {
          a = y[r];
        } else {
          const float2 w = tab[G::OFF_W + j + 64 * r];
          a = make_float2(fmaf(w.y, y[r].y, fmaf(w.x, y[r].x, a.x)), fmaf(-w.y, y[r].x, fmaf(w.x, y[r].y, a.y)));
        }
      }
    }
  }
  return acc;
}

template <int M, int PAD, typename F>
Column split_in_two(const Column& x, const Column& tab, F&& product) {
  using G = ColSplit<M, PAD>;
  constexpr int NH = G::NH, R1 = G::R1, R2 = G::R2;
  Column out(G::LEN), lds[2] = {Column(G::region(16)), Column(G::region(16))};
  for (int h = 0; h < NH; ++h) {
    for (int j = 0; j < R2; ++j) {
      float2 v[R1];
      for (int r = 0; r < R1; ++r) v[r] = x[j + R2 * r];
      if (h) col_rows_forward<M, PAD, true>(v);
      else col_rows_forward<M, PAD, false>(v);
      for (int k = 0; k < R1; ++k) lds[h][G::slot(k, j)] = v[k];
    }
    for (int k1 = 0; k1 < R1; ++k1) {
      float2 f[R2];
      for (int j = 0; j < R2; ++j) f[j] = lds[h][G::slot(k1, j)];
      col_freq_forward<M, PAD>(f, tab.data(), h, k1);
      for (int k2 = 0; k2 < R2; ++k2) f[k2] = product(NH * (k1 + R1 * k2) + h, f[k2]);
      col_freq_inverse<M, PAD>(f);
      for (int j = 0; j < R2; ++j) lds[h][G::slot(k1, j)] = f[j];
    }
  }
  for (int j = 0; j < R2; ++j) {
    if constexpr (NH == 2) {
      for (int parity = 0; parity < 2; ++parity) {
        float2 y[G::RC];
        col_rows_inverse2<M, PAD>(y, tab.data(), j, parity, [&](int h, int k) { return lds[h][G::slot(k, j)]; });
        for (int r = 0; r < G::RC; ++r) out[j + R2 * (2 * r + parity)] = y[r];
      }
    } else {
      float2 y[R1];
      for (int k = 0; k < R1; ++k) y[k] = lds[0][G::slot(k, j)];
      col_rows_inverse<M, PAD>(y, tab.data(), j);
      for (int r = 0; r < R1; ++r) out[j + R2 * r] = y[r];
    }
  }
  return out;
}

template <int M, int PAD, typename F>
Column split(const Column& x, F&& product) {
  Column tab;
  if constexpr (ColSplit800<M, PAD>::BUILT) {
    col800_table_host<M, PAD>(tab);
    return split_halves_of_800<M, PAD>(x, tab, product);
  } else if constexpr (ColSplit3<M, PAD>::BUILT) {
    col3_table_host<M, PAD>(tab);
    return split_halves_of_512<M, PAD>(x, tab, product);
  } else {
    col_table_host<M, PAD>(tab);
    return split_in_two<M, PAD>(x, tab, product);
  }
}

struct Trip {  // a random column, random phases over M^2, and its exact round trip
  Column x, h;
  std::vector<cd> spectrum, rows;
  double norm = 0.0;
  Trip(int M, int len, int seed) : x(len), h(M), spectrum(M), rows(len) {
    std::mt19937 g(100 * M + len + 7919 * seed);
    std::normal_distribution<float> nd;
    std::uniform_real_distribution<double> ud;
    for (auto& v : x) v = make_float2(nd(g), nd(g));
    for (auto& v : h) {
      const double a = 2.0 * M_PI * ud(g);
      v = make_float2(static_cast<float>(std::cos(a) / M / M), static_cast<float>(std::sin(a) / M / M));
    }
    std::vector<cd> root(M);
    for (int k = 0; k < M; ++k) root[k] = std::polar(1.0, -2.0 * M_PI * k / M);
    for (int k = 0; k < M; ++k)
      for (int n = 0; n < len; ++n) spectrum[k] += cd(x[n].x, x[n].y) * root[static_cast<long long>(n) * k % M];
    for (int n = 0; n < len; ++n) {
      for (int k = 0; k < M; ++k)
        rows[n] += spectrum[k] * cd(h[k].x, h[k].y) * std::conj(root[static_cast<long long>(n) * k % M]);
      norm += std::norm(rows[n]);
    }
  }
  double error(const Column& y) const {
    double e = 0.0;
    for (size_t n = 0; n < rows.size(); ++n) e += std::norm(cd(y[n].x, y[n].y) - rows[n]);
    return std::sqrt(e / norm);
  }
  template <typename Forward, typename Inverse>
  double padded_error(Forward&& forward, Inverse&& inverse) const {
    Column y(h.size(), make_float2(0.f, 0.f));
    std::copy(x.begin(), x.end(), y.begin());
    forward(y);
    for (size_t k = 0; k < h.size(); ++k) y[k] = cmul(y[k], h[k]);
    inverse(y);
    return error(y);
  }
};

template <int M, int PAD>
double staged_error(const Trip& t) {
  return t.padded_error([](Column& y) { staged<M, false, PAD == 2>(y); }, [](Column& y) { staged<M, true, false>(y); });
}

template <int M, int PAD>
void compare(int seeds) {
  double a = 0.0, b = 0.0;
  for (int s = 0; s < seeds; ++s) {
    const Trip t(M, M / PAD, s);
    a += staged_error<M, PAD>(t);
    b += t.error(split<M, PAD>(t.x, [&](int k, float2 v) { return cmul(v, t.h[k]); }));
  }
  std::printf("split%dpad%d %.5f\n", M, PAD, b / a);
}

template <int M, int PAD, int... R>
void compare_plan(int seeds) {
  double a = 0.0, b = 0.0;
  for (int s = 0; s < seeds; ++s) {
    const Trip t(M, M / PAD, s);
    a += t.padded_error([](Column& y) { given<false, PAD == 2, R...>(y); }, [](Column& y) { given<true, false, R...>(y); });
    b += staged_error<M, PAD>(t);
  }
  std::printf("plan%dpad%d %.5f\n", M, PAD, b / a);
}

void check800() {
  using G = ColSplit800<1600, 2>;
  std::set<int> used;
  for (int k1 = 0; k1 < G::R1; ++k1)
    for (int j = 0; j < G::R2; ++j)
      if (G::slot(k1, j) < 0 || G::slot(k1, j) >= G::REG || !used.insert(G::slot(k1, j)).second) ++failures;
  // 16 lanes of one LDS cycle: eight columns and two j in the row phases, k1 in the frequencies
  for (int j = 0; j + 1 < G::R2; j += 2) {
    std::set<int> banks;
    for (int l = 0; l < 16; ++l) banks.insert((l % 8 * G::REG + G::slot(0, j + l / 8)) % 16);
    if (banks.size() < 16) ++failures;
  }
  std::set<int> banks;
  for (int l = 0; l < 16; ++l) banks.insert(G::slot(l, 0) % 16);
  if (banks.size() < 16) ++failures;
  const Trip t(1600, 800, 0);
  double e = 0.0, ref = 0.0;
  split<1600, 2>(t.x, [&](int k, float2 v) {
    e += std::norm(cd(v.x, v.y) - t.spectrum[k]);
    ref += std::norm(t.spectrum[k]);
    return v;
  });
  forward800 = std::sqrt(e / ref);
}

int main() {
  check800();
  compare<64, 2>(900), compare<96, 2>(700), compare<128, 2>(500), compare<192, 2>(300), compare<256, 2>(200);
  compare<384, 2>(120), compare<512, 2>(80), compare<1024, 2>(24), compare<1600, 2>(12);
  compare<64, 1>(900), compare<96, 1>(700), compare<128, 1>(500), compare<192, 1>(300), compare<256, 1>(200);
  compare<384, 1>(120), compare<512, 1>(80);
  compare_plan<64, 2, 16, 4>(900), compare_plan<64, 1, 16, 4>(900);
  compare_plan<96, 2, 3, 8, 4>(700), compare_plan<96, 1, 3, 8, 4>(700);
  std::printf("forward800 %.9g\n", forward800);
  return failures ? 1 : 0;
}
