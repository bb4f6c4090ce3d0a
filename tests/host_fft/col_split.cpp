// Checks the column transforms of every length (csrc/col_fft.hpp) on the CPU: the two phases of
// the forward transform against the DFT in double precision, forward and inverse back to the
// rows, the LDS slots (distinct, inside their region) and the bank spread of both access patterns
// for tiles of 16 columns.  Prints the worst relative errors and, on failure, a line per fault.
#include <algorithm>
#include <complex>
#include <cstdio>
#include <random>
#include <set>
#include <vector>

#include "col_fft.hpp"

using namespace dpx;
typedef std::complex<double> cd;

static int failures = 0;
static double worst_fwd = 0.0, worst_back = 0.0;

template <int M, int PAD>
void check() {
  using G = ColSplit<M, PAD>;
  constexpr int NH = G::NH, R1 = G::R1, R2 = G::R2, LEN = G::LEN;
  std::vector<float2> tab;
  col_table_host<M, PAD>(tab);
  std::mt19937 g(M + PAD);
  std::normal_distribution<float> nd;
  std::vector<float2> x(LEN);
  for (auto& v : x) v = make_float2(nd(g), nd(g));
  // slots
  std::set<int> used;
  for (int k1 = 0; k1 < R1; ++k1)
    for (int j = 0; j < R2; ++j) {
      const int s = G::slot(k1, j);
      if (s < 0 || s >= G::region(16) || s >= G::region(8) || !used.insert(s).second) {
        std::printf("M=%d pad %d: slot (%d, %d)\n", M, PAD, k1, j);
        ++failures;
      }
    }
  // 16 lanes of one LDS cycle: rows phase (column fast, then j), frequency phase (k1 fast, then column)
  for (int j = 0; j < R2; ++j) {
    std::set<int> banks;
    for (int c = 0; c < 16; ++c) banks.insert((c * G::region(16) + G::slot(0, j)) % 16);
    if (banks.size() < 16) { std::printf("M=%d pad %d: rows phase has bank conflicts\n", M, PAD); ++failures; break; }
  }
  if (pow2(R1)) {
    std::set<int> banks;
    for (int l = 0; l < 16; ++l) banks.insert((l / R1 * G::region(16) + G::slot(l % R1, 0)) % 16);
    if (banks.size() < 16) { std::printf("M=%d pad %d: frequency phase has bank conflicts\n", M, PAD); ++failures; }
  }
  std::vector<std::vector<float2>> lds(NH, std::vector<float2>(G::region(16)));
  for (int h = 0; h < NH; ++h)
    for (int j = 0; j < R2; ++j) {
      float2 v[R1];
      for (int r = 0; r < R1; ++r) v[r] = x[j + R2 * r];
      if (h) col_rows_forward<M, PAD, true>(v);
      else col_rows_forward<M, PAD, false>(v);
      for (int k1 = 0; k1 < R1; ++k1) lds[h][G::slot(k1, j)] = v[k1];
    }
  double err = 0.0, ref = 0.0;
  for (int h = 0; h < NH; ++h)
    for (int k1 = 0; k1 < R1; ++k1) {
      float2 v[R2];
      for (int j = 0; j < R2; ++j) v[j] = lds[h][G::slot(k1, j)];
      col_freq_forward<M, PAD>(v, tab.data(), h, k1);
      for (int k2 = 0; k2 < R2; ++k2) {
        const long long K = NH * (k1 + R1 * k2) + h;
        cd s = 0.0;
        for (int n = 0; n < LEN; ++n) s += cd(x[n].x, x[n].y) * std::polar(1.0, -2.0 * M_PI * double((n * K) % M) / M);
        err += std::norm(s - cd(v[k2].x, v[k2].y));
        ref += std::norm(s);
        v[k2] = make_float2(v[k2].x / M, v[k2].y / M);
      }
      col_freq_inverse<M, PAD>(v);
      for (int j = 0; j < R2; ++j) lds[h][G::slot(k1, j)] = v[j];
    }
  worst_fwd = std::max(worst_fwd, std::sqrt(err / ref));
  err = ref = 0.0;
  auto add = [&](int n, float2 y) {
    err += std::norm(cd(y.x, y.y) - cd(x[n].x, x[n].y));
    ref += std::norm(cd(x[n].x, x[n].y));
  };
  for (int j = 0; j < R2; ++j) {
    if constexpr (NH == 2) {
      for (int parity = 0; parity < 2; ++parity) {
        float2 y[G::RC];
        col_rows_inverse2<M, PAD>(y, tab.data(), j, parity, [&](int h, int k1) { return lds[h][G::slot(k1, j)]; });
        for (int r = 0; r < G::RC; ++r) add(j + R2 * (2 * r + parity), y[r]);
      }
    } else {
      float2 y[R1];
      for (int k1 = 0; k1 < R1; ++k1) y[k1] = lds[0][G::slot(k1, j)];
      col_rows_inverse<M, PAD>(y, tab.data(), j);
      for (int r = 0; r < R1; ++r) add(j + R2 * r, y[r]);
    }
  }
  worst_back = std::max(worst_back, std::sqrt(err / ref));
  std::fprintf(stderr, "M=%d pad %d: back %.3g\n", M, PAD, std::sqrt(err / ref));
}

// the same for halves of 512 points, whose B is 8 x 8 with an exchange of its own
template <int M, int PAD>
void check3() {
  using G = ColSplit3<M, PAD>;
  constexpr int NH = G::NH, LEN = G::LEN;
  std::vector<float2> tab;
  col3_table_host<M, PAD>(tab);
  std::mt19937 g(M + PAD);
  std::normal_distribution<float> nd;
  std::vector<float2> x(LEN), acc(LEN);
  for (auto& v : x) v = make_float2(nd(g), nd(g));
  std::set<int> used;
  for (int k1 = 0; k1 < 8; ++k1)
    for (int j = 0; j < 64; ++j)
      if (G::slot(k1, j) >= G::REG || !used.insert(G::slot(k1, j)).second) {
        std::printf("M=%d pad %d: slot (%d, %d)\n", M, PAD, k1, j);
        ++failures;
      }
  std::set<int> rows, b1, b2;  // 16 lanes: eight columns and two j; eight k1 and two j1 (m)
  for (int l = 0; l < 16; ++l) {
    rows.insert((l % 8 * G::REG + G::slot(0, l / 8)) % 16);
    b1.insert(G::slot(l % 8, l / 8) % 16);
    b2.insert(G::slot(l % 8, 8 * (l / 8)) % 16);
  }
  if (rows.size() < 16 || b1.size() < 16 || b2.size() < 16) {
    std::printf("M=%d pad %d: bank conflicts\n", M, PAD);
    ++failures;
  }
  double err = 0.0, ref = 0.0;
  for (int h = 0; h < NH; ++h) {
    std::vector<float2> lds(G::REG);
    for (int j = 0; j < 64; ++j) {
      float2 v[8];
      for (int r = 0; r < 8; ++r) v[r] = x[j + 64 * r];
      if (h) dft_odd<8>(v);
      else DFT<8, false, false>::run(v);
      for (int k = 0; k < 8; ++k) lds[G::slot(k, j)] = v[k];
    }
    auto step = [&](auto body) {  // every lane reads all before any writes, as wave_sync orders it
      std::vector<float2> out(lds);
      for (int lane = 0; lane < 64; ++lane) body(lane & 7, lane >> 3, lane, out);
      lds = out;
    };
    step([&](int k1, int j1, int, std::vector<float2>& out) {
      float2 f[8];
      for (int i = 0; i < 8; ++i) f[i] = lds[G::slot(k1, j1 + 8 * i)];
      dft8_table<false>(f, tab.data() + h * 8 + k1, NH * 8);
      for (int i = 0; i < 8; ++i) out[G::slot(k1, j1 + 8 * i)] = f[i];
    });
    step([&](int k1, int m, int lane, std::vector<float2>& out) {
      float2 f[8];
      for (int i = 0; i < 8; ++i) f[i] = lds[G::slot(k1, i + 8 * m)];
      dft8_table<false>(f, tab.data() + G::OFF_B2 + h * 64 + lane, NH * 64);
      for (int q = 0; q < 8; ++q) {
        const long long K = NH * (lane + 64 * q) + h;
        cd s = 0.0;
        for (int n = 0; n < LEN; ++n) s += cd(x[n].x, x[n].y) * std::polar(1.0, -2.0 * M_PI * double((n * K) % M) / M);
        err += std::norm(s - cd(f[q].x, f[q].y));
        ref += std::norm(s);
        f[q] = make_float2(f[q].x / M, f[q].y / M);
      }
      DFT<8, true, false>::run(f);
      for (int i = 0; i < 8; ++i) out[G::slot(k1, i + 8 * m)] = f[i];
    });
    step([&](int k1, int j1, int, std::vector<float2>& out) {
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
        if (h == 0) acc[j + 64 * r] = y[r];
        else acc[j + 64 * r] = cadd(acc[j + 64 * r], cmulc(y[r], tab[G::OFF_W + j + 64 * r]));
      }
    }
  }
  worst_fwd = std::max(worst_fwd, std::sqrt(err / ref));
  err = ref = 0.0;
  for (int n = 0; n < LEN; ++n) {
    err += std::norm(cd(acc[n].x, acc[n].y) - cd(x[n].x, x[n].y));
    ref += std::norm(cd(x[n].x, x[n].y));
  }
  worst_back = std::max(worst_back, std::sqrt(err / ref));
  std::fprintf(stderr, "M=%d pad %d: back %.3g\n", M, PAD, std::sqrt(err / ref));
}

int main() {
  check3<1024, 2>(); check3<512, 1>();
  check<64, 2>(); check<96, 2>(); check<128, 2>(); check<192, 2>(); check<256, 2>(); check<384, 2>(); check<512, 2>();
  check<64, 1>(); check<96, 1>(); check<128, 1>(); check<192, 1>(); check<256, 1>(); check<384, 1>();
  std::printf("%.9g %.9g\n", worst_fwd, worst_back);
  return failures ? 1 : 0;
}
