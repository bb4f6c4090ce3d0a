// Column transforms of the propagation: forward transform of the N aperture rows of a column,
// product with the transfer function, inverse transform back to the aperture rows.
//
// A zero-padded column (M = 2 N) is two transforms of N points, one for the even and one for
// the odd frequencies: with K = 2 k + h,
//   X[2 k + h] = sum_n (x[n] w_M^(n h)) w_N^(n k),       w_L = exp(-2 pi i / L),
// and the N aperture rows of the inverse are the sum over h of the two inverse transforms, the
// odd one turned by w_M^(-n).  A periodic column (pad 1) is the even one alone.  So NH = pad
// halves of LEN = M / pad points each.
//
// LEN = R1 R2 is split once: n = j + R2 r, k = k1 + R1 k2, and
//   A: a[j][k1] = sum_r x[j + R2 r] w_(NH R1)^(r K1)          K1 = NH k1 + h
//   B: X[k1][k2] = sum_j a[j][k1] (w_M^K1)^j w_R2^(j k2)       then H, then
//      b[k1][j] = sum_k2 X[k1][k2] w_R2^(-j k2)
//   C: y[j + R2 r] = sum_h w_M^(-(j + R2 r) h) sum_k1 b[k1][j] (w_LEN^(-j))^k1 w_R1^(-r k1)
// A thread of A and C owns (column, j) with its rows j + R2 r in registers, loaded from and
// stored to the plane directly (neighbouring threads take neighbouring columns, so a row
// segment of the tile is one contiguous access); a thread of B owns (column, k1) with all k2 in
// registers.  Between them lies one exchange through LDS each way, and B writes back to the
// slots it read.  Against the staged form (tile through LDS, then a full-length transform per
// column with one exchange between every two radix stages) this drops the staging round trip and
// all but one exchange per transform: the column passes were bound by vector instructions at
// 88 % issue with the LDS port 70 % busy and the waits between them.
//
// Twiddles multiply the inputs of B and C as powers base^r of one lane constant.  For a power of
// two they go into the butterflies (Linzer and Feig's fused form): with tau = c (1 + i t),
//   e +- tau o = e +- c ((o.re - t o.im) + i (o.im + t o.re)),
// six fused multiply-adds for a radix-2 butterfly with its twiddle against eight operations, and
// R / 2 pairs (c, t) instead of R - 1 twiddles.  Its rounding error is that of the product form:
// the inner sum is rounded relative to |tau o| / c, and scaled by c.  Where cos vanishes exactly
// c is 2^-30 and t = -+2^30, which leaves 2^-30 |o| of the vanishing component.
#pragma once

#include "fft.hpp"

namespace dpx {

// Splits of the built transform lengths.  R1 is the radix of A and C (registers of a row
// thread), R2 that of B.  R1 lanes of B are consecutive lanes of one wavefront (GP = R1 rounded
// up to a power of two) so that H can be shared with the mirrored rows across lanes.  S1 is the
// slot distance of neighbouring k1 and REG (per column and half) that of neighbouring columns:
// with 16 lanes per LDS cycle over 32 banks for 8-byte accesses, S1 odd (R1 = 16) or 2 mod 4
// (R1 = 8) with REG odd puts the 16 lanes of both access patterns on distinct banks.
template <int LEN> struct Split { static constexpr int R1 = 0, R2 = 0, S1 = 0, REG = 0; };
template <> struct Split<32>  { static constexpr int R1 = 8,  R2 = 4,  S1 = 6,  REG = 49; };
template <> struct Split<48>  { static constexpr int R1 = 6,  R2 = 8,  S1 = 10, REG = 61; };
template <> struct Split<64>  { static constexpr int R1 = 8,  R2 = 8,  S1 = 10, REG = 81; };
template <> struct Split<96>  { static constexpr int R1 = 8,  R2 = 12, S1 = 14, REG = 113; };
template <> struct Split<128> { static constexpr int R1 = 8,  R2 = 16, S1 = 18, REG = 145; };
template <> struct Split<192> { static constexpr int R1 = 16, R2 = 12, S1 = 13, REG = 209; };
template <> struct Split<256> { static constexpr int R1 = 16, R2 = 16, S1 = 17, REG = 273; };
template <> struct Split<384> { static constexpr int R1 = 16, R2 = 24, S1 = 25, REG = 401; };

constexpr bool pow2(int n) { return n > 0 && (n & (n - 1)) == 0; }
constexpr int pow2_at_least(int n) { int p = 1; while (p < n) p *= 2; return p; }

// twiddle entries of a radix-R transform whose inputs carry base^r: pairs (c, t) of the R / 2
// distinct butterfly twiddles of a power of two, else the R - 1 powers themselves
constexpr int input_twiddles(int R) { return pow2(R) ? R / 2 : R - 1; }
// pair of butterfly k (k < S / 4) of the level that joins transforms of S / 2 points
constexpr int pair_index(int S, int k) { return S == 2 ? 0 : S / 4 + k; }

template <int M, int PAD>
struct ColSplit {
  static constexpr int LEN = M / PAD, NH = PAD;
  static constexpr int R1 = Split<LEN>::R1, R2 = Split<LEN>::R2;
  static constexpr bool BUILT = R1 > 0;
  static constexpr int L = R2;                      // row threads of a column and half
  static constexpr int GP = pow2_at_least(R1 > 0 ? R1 : 1);  // lanes of a column and half in B
  static constexpr int RC = NH == 2 ? R1 / 2 : R1;  // radix of C: with two halves two threads
                                                    // share a (column, j), the rows r of one parity each
  static constexpr int NB = BUILT ? input_twiddles(R2) : 0;
  static constexpr int NC = BUILT ? input_twiddles(RC) : 0;
  // table: B [NB][NH][R1], C [NC][NH][L] (second index: row parity), with two halves also the
  // first level of C, w_LEN^(j R1 / 2), [L] and w_M^n, [LEN]
  static constexpr int OFF_C = NB * NH * R1;
  static constexpr int OFF_0 = OFF_C + NC * NH * L;
  static constexpr int OFF_W = OFF_0 + (NH == 2 ? L : 0);
  static constexpr int COUNT = OFF_W + (NH == 2 ? LEN : 0);
  // LDS slot of (k1, j) inside a column's region
  static __host__ __device__ constexpr int slot(int k1, int j) { return k1 * Split<LEN>::S1 + j; }
  // region of a column and half for tiles of TX columns
  static constexpr int region(int TX) { return Split<LEN>::REG + (TX == 8 ? 1 : 0); }
  // tiles of 8 columns where the threads of a half fill whole wavefronts
  static constexpr bool NARROW = (8 * L) % 64 == 0 && (8 * GP) % 64 == 0;
  static constexpr int threads(int TX) { return NH * TX * (L > GP ? L : GP); }
};

// LEN = 512 (1024 zero-padded points, or 512 periodic ones) would need 32 registers of data in one
// of two phases, or leave half of the lanes idle there.  Its B is a transform of 64 points on eight lanes,
// 8 x 8 with an exchange of its own inside the wavefront: LEN = 8 . (8 . 8).  With j = j1 + 8 i and
// k2 = m + 8 q,
//   B1: c[k1][j1][m] = sum_i a[j1 + 8 i][k1] (w_M^(8 K1))^i w_8^(i m)
//   B2: X[k1][m + 8 q] = sum_j1 c[k1][j1][m] (w_M^(K1 + 8 NH m))^j1 w_8^(j1 q)
// and back, X -> (over q) -> (over m, twiddled by w_64^(-j1)) -> b[k1][j1 + 8 i].  A lane of B is k1 + 8 j1
// or k1 + 8 m, so the frequency of (lane, q) is NH (lane + 64 q) + h.  Eight registers of data per
// lane: the halves follow each other on the same threads, with the rows and the even half's result
// kept in registers, and every exchange goes back to slots that only its own lane or wavefront uses.
template <int M, int PAD>
struct ColSplit3 {
  static constexpr int LEN = M / PAD, NH = PAD;
  static constexpr bool BUILT = LEN == 512;
  static constexpr int L = 64;  // row threads of a column, lanes of B
  // table: B1 [4][NH][8], B2 [4][NH][64], back [4][8], C [4][64], with two halves w_M^n [LEN]
  static constexpr int OFF_B2 = 4 * NH * 8;
  static constexpr int OFF_R = OFF_B2 + 4 * NH * 64;
  static constexpr int OFF_C = OFF_R + 4 * 8;
  static constexpr int OFF_W = OFF_C + 4 * 64;
  static constexpr int COUNT = OFF_W + (NH == 2 ? LEN : 0);
  // Slots: k1 is 74 apart (2 mod 8: eight k1 and two neighbouring j cover the 16 bank pairs), j padded
  // by one after every eight (neighbouring m of B2 fall on odd distances), columns 594 apart
  // (2 mod 16, for eight columns and two j).
  static constexpr int REG = 594;
  static __host__ __device__ constexpr int slot(int k1, int j) { return k1 * 74 + j + (j >> 3); }
};

// LEN = 800 (1600 zero-padded points) = 25 . 32: A and C on 32 threads per column with 25 rows each,
// B on 25 of 32 lanes with 32 values each, so two columns per wavefront.  The halves follow each other
// as in ColSplit3, one exchange each way, and every slot is read back by the thread that owns it.  The
// tables (21 KB) are read through the caches: the three blocks that share a CU leave no LDS for them.
template <int M, int PAD>
struct ColSplit800 {
  static constexpr int LEN = M / PAD, NH = PAD;
  static constexpr bool BUILT = LEN == 800 && PAD == 2;
  static constexpr int R1 = 25, R2 = 32, L = 32, GP = 32;
  // table: B [16][NH][32] (25 used), C [24][32], w_M^n [LEN]
  static constexpr int OFF_C = 16 * NH * 32;
  static constexpr int OFF_W = OFF_C + 24 * 32;
  static constexpr int COUNT = OFF_W + LEN;
  // k1 33 slots apart (odd), columns 826 (2 mod 8, for eight columns and two j)
  static constexpr int REG = 826;
  static __host__ __device__ constexpr int slot(int k1, int j) { return k1 * 33 + j; }
};

// the pair (c, t) of exp(-2 pi i k / M) = c (1 + i t)
inline float2 fused_pair(const UnitRoots& u, int k) {
  if (4 * k == u.length() || 4 * k == 3 * u.length()) {
    const float s = 4 * k == u.length() ? -1.f : 1.f;
    return make_float2(9.31322574615478515625e-10f, s * 1073741824.f);
  }
  // t over the rounded c: the sine c t that the butterfly forms is then off by t's own rounding alone
  const float c = static_cast<float>(u.cos(k));
  return make_float2(c, static_cast<float>(-u.sin(k) / c));
}
// entry e of the input twiddles of radix R with base exp(-2 pi i num / den)
inline float2 input_twiddle(const UnitRoots& u, int R, int e, long long num, long long den) {
  if (!pow2(R)) return unit_root(u, (e + 1) * num, den);
  int S = 2;
  while (S < R && pair_index(2 * S, 0) <= e) S *= 2;
  const int k = e - pair_index(S, 0);
  // base^(R / S) w_S^k
  return fused_pair(u, (u.index(num * (R / S), den) + u.index(k, S)) % u.length());
}

template <int M, int PAD>
inline void col_table_host(std::vector<float2>& out, const UnitRoots& u = UnitRoots(M)) {
  using G = ColSplit<M, PAD>;
  out.assign(G::COUNT > 0 ? G::COUNT : 1, make_float2(1.f, 0.f));
  if constexpr (G::BUILT) {
    for (int e = 0; e < G::NB; ++e)
      for (int h = 0; h < G::NH; ++h)
        for (int k1 = 0; k1 < G::R1; ++k1)
          out[(e * G::NH + h) * G::R1 + k1] = input_twiddle(u, G::R2, e, G::NH * k1 + h, M);
    for (int e = 0; e < G::NC; ++e)
      for (int p = 0; p < G::NH; ++p)
        for (int j = 0; j < G::L; ++j)  // w_LEN^j, turned by w_R1 for the odd rows
          out[G::OFF_C + (e * G::NH + p) * G::L + j] =
              input_twiddle(u, G::RC, e, j + p * (G::LEN / G::R1), G::LEN);
    if constexpr (G::NH == 2) {
      for (int j = 0; j < G::L; ++j)
        out[G::OFF_0 + j] = unit_root(u, static_cast<long long>(j) * (G::R1 / 2), G::LEN);
      for (int n = 0; n < G::LEN; ++n) out[G::OFF_W + n] = unit_root(u, n, M);
    }
  }
}

template <int M, int PAD>
inline void col3_table_host(std::vector<float2>& out, const UnitRoots& u = UnitRoots(M)) {
  using G = ColSplit3<M, PAD>;
  out.assign(G::COUNT, make_float2(1.f, 0.f));
  for (int e = 0; e < 4; ++e) {
    for (int h = 0; h < G::NH; ++h) {
      for (int k1 = 0; k1 < 8; ++k1) out[(e * G::NH + h) * 8 + k1] = input_twiddle(u, 8, e, 8 * (G::NH * k1 + h), M);
      for (int l = 0; l < 64; ++l)  // l = k1 + 8 m
        out[G::OFF_B2 + (e * G::NH + h) * 64 + l] = input_twiddle(u, 8, e, G::NH * l + h, M);
    }
    for (int j = 0; j < 8; ++j) out[G::OFF_R + e * 8 + j] = input_twiddle(u, 8, e, j, 64);
    for (int j = 0; j < 64; ++j) out[G::OFF_C + e * 64 + j] = input_twiddle(u, 8, e, j, G::LEN);
  }
  if constexpr (G::NH == 2)
    for (int n = 0; n < G::LEN; ++n) out[G::OFF_W + n] = unit_root(u, n, M);
}

template <int M, int PAD>
inline void col800_table_host(std::vector<float2>& out, const UnitRoots& u = UnitRoots(M)) {
  using G = ColSplit800<M, PAD>;
  out.assign(G::COUNT, make_float2(1.f, 0.f));
  for (int e = 0; e < 16; ++e)
    for (int h = 0; h < G::NH; ++h)
      for (int k1 = 0; k1 < G::R1; ++k1) out[(e * G::NH + h) * 32 + k1] = input_twiddle(u, 32, e, G::NH * k1 + h, M);
  for (int e = 0; e < 24; ++e)
    for (int j = 0; j < 32; ++j) out[G::OFF_C + e * 32 + j] = input_twiddle(u, 25, e, j, G::LEN);
  for (int n = 0; n < G::LEN; ++n) out[G::OFF_W + n] = unit_root(u, n, M);
}

// ------------------------------------------------------------------------------------------
// Register transforms
// ------------------------------------------------------------------------------------------
// e +- tau o for tau = c (1 + i t)
__device__ __forceinline__ void fused_butterfly(float2 e, float2 o, float c, float t, float2& lo, float2& hi) {
  const float u = fmaf(-t, o.y, o.x), v = fmaf(t, o.x, o.y);
  lo = make_float2(fmaf(c, u, e.x), fmaf(c, v, e.y));
  hi = make_float2(fmaf(-c, u, e.x), fmaf(-c, v, e.y));
}
// the same for tau turned by another quarter (-i forward, +i inverse)
template <bool INV>
__device__ __forceinline__ void fused_butterfly_quarter(float2 e, float2 o, float c, float t, float2& lo, float2& hi) {
  const float u = fmaf(-t, o.y, o.x), v = fmaf(t, o.x, o.y);
  const float cq = INV ? -c : c;  // -i (u + i v) = v - i u
  lo = make_float2(fmaf(cq, v, e.x), fmaf(-cq, u, e.y));
  hi = make_float2(fmaf(-cq, v, e.x), fmaf(cq, u, e.y));
}

// the last level of dft_fused: v from the transforms of its even and odd inputs, p its own pairs
template <int R, bool INV>
__device__ __forceinline__ void dft_fused_join(const float2* e, const float2* o, const float2* p, float2* v) {
#pragma unroll
  for (int k = 0; k < (R > 2 ? R / 4 : 1); ++k) {
    const float2 q = p[k];
    const float t = INV ? -q.y : q.y;
    fused_butterfly(e[k], o[k], q.x, t, v[k], v[k + R / 2]);
    if constexpr (R > 2)
      fused_butterfly_quarter<INV>(e[k + R / 4], o[k + R / 4], q.x, t, v[k + R / 4], v[k + 3 * R / 4]);
  }
}

// R-point transform (a power of two) of v[r] base^r, natural order in and out; p: the R / 2 pairs
// of base (of its conjugate's conjugate: INV negates t)
template <int R, bool INV>
__device__ __forceinline__ void dft_fused(float2* v, const float2* p) {
  if constexpr (R > 1) {
    float2 e[R / 2], o[R / 2];
#pragma unroll
    for (int i = 0; i < R / 2; ++i) {
      e[i] = v[2 * i];
      o[i] = v[2 * i + 1];
    }
    dft_fused<R / 2, INV>(e, p);
    dft_fused<R / 2, INV>(o, p);
    dft_fused_join<R, INV>(e, o, p + pair_index(R, 0), v);
  }
}

// R-point transform of v[r] base^r: fused for a power of two, else products and the plain one
template <int R, bool INV>
__device__ __forceinline__ void dft_input_twiddled(float2* v, const float2* p) {
  if constexpr (pow2(R)) {
    dft_fused<R, INV>(v, p);
  } else {
#pragma unroll
    for (int r = 1; r < R; ++r) v[r] = INV ? cmulc(v[r], p[r - 1]) : cmul(v[r], p[r - 1]);
    DFT<R, INV, false>::run(v);
  }
}

// Forward transform to the odd multiples of half a bin: sum_r v[r] w_(2R)^(r (2 k + 1)).  Even R joins
// the transforms of the even and odd inputs; for R = 3 the odd multiples are a permutation of the plain
// transform with the sign of v[1] turned, w_6^(2 k + 1) = -w_3^-(2 k + 1).
template <int R>
__device__ __forceinline__ void dft_odd(float2* v) {
  if constexpr (R == 2) {
    const float2 a = v[0], b = mul_negi(v[1]);
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else if constexpr (R == 3) {
    v[1] = make_float2(-v[1].x, -v[1].y);
    DFT<3, false, false>::run(v);
    const float2 x0 = v[2], x1 = v[0];
    v[2] = v[1];
    v[0] = x0;
    v[1] = x1;
  } else if constexpr (pow2(R) || R == 6) {
    float2 e[R / 2], o[R / 2];
#pragma unroll
    for (int i = 0; i < R / 2; ++i) {
      e[i] = v[2 * i];
      o[i] = v[2 * i + 1];
    }
    dft_odd<R / 2>(e);
    dft_odd<R / 2>(o);
    // the factor w_(2R)^(2 k + 1); of a power of two the upper half of them is the lower half turned by a
    // quarter, of 6 the one in the middle is a quarter itself
    static_for<0, R == 6 ? 3 : R / 4>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      if constexpr (R == 6 && k == 1) {
        const float2 b = mul_negi(o[k]);
        v[k] = cadd(e[k], b);
        v[k + R / 2] = csub(e[k], b);
      } else {
        constexpr float c = static_cast<float>(cos2pi(2 * k + 1, 2 * R));
        constexpr float t = static_cast<float>(-sin2pi(2 * k + 1, 2 * R) / c);
        fused_butterfly(e[k], o[k], c, t, v[k], v[k + R / 2]);
        if constexpr (R != 6)
          fused_butterfly_quarter<false>(e[k + R / 4], o[k + R / 4], c, t, v[k + R / 4], v[k + 3 * R / 4]);
      }
    });
  } else {
    static_for<1, R>([&](auto rc) {
      constexpr int r = decltype(rc)::value;
      v[r] = twc<2 * R, r, false>(v[r]);
    });
    DFT<R, false, false>::run(v);
  }
}

// keeps the compiler from moving instructions across (a no-op for the hardware and the host)
__device__ __forceinline__ void schedule_fence() {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_sched_barrier(0);
#endif
}

// ------------------------------------------------------------------------------------------
// The phases
// ------------------------------------------------------------------------------------------
// A: rows of one (column, j), half H1 (0 even, 1 odd frequencies)
template <int M, int PAD, bool ODD>
__device__ __forceinline__ void col_rows_forward(float2* v) {
  if constexpr (ODD) dft_odd<ColSplit<M, PAD>::R1>(v);
  else DFT<ColSplit<M, PAD>::R1, false, false>::run(v);
}

// C with one half: the rows of (column, j) from b[k1]
template <int M, int PAD>
__device__ __forceinline__ void col_rows_inverse(float2* v, const float2* __restrict__ tab, int j) {
  using G = ColSplit<M, PAD>;
  static_assert(G::NH == 1, "one half");
  float2 p[G::NC];
#pragma unroll
  for (int e = 0; e < G::NC; ++e) p[e] = tab[G::OFF_C + e * G::L + j];
  dft_input_twiddled<G::R1, true>(v, p);
}

// C with two halves: the rows r = 2 r' + parity of (column, j), from the even and the odd half's
// b[k1] (b(h, k1) reads one of them).  y[r'] holds row j + R2 (2 r' + parity).
template <int M, int PAD, typename B>
__device__ __forceinline__ void col_rows_inverse2(float2* y, const float2* __restrict__ tab,
                                                  int j, int parity, B&& b) {
  using G = ColSplit<M, PAD>;
  static_assert(G::NH == 2, "two halves");
  const float2 z = tab[G::OFF_0 + j];
  const float sg = parity ? -1.f : 1.f;
  const float zr = sg * z.x, zi = -sg * z.y;  // +- the conjugate of w_LEN^(j R1 / 2)
  float2 p[G::NC];
#pragma unroll
  for (int e = 0; e < G::NC; ++e) p[e] = tab[G::OFF_C + (e * 2 + parity) * G::L + j];
  float2 odd[G::RC];
#pragma unroll
  for (int k = 0; k < G::RC; ++k) {
    const float2 a = b(1, k), c = b(1, k + G::RC);
    odd[k] = make_float2(fmaf(-zi, c.y, fmaf(zr, c.x, a.x)), fmaf(zi, c.x, fmaf(zr, c.y, a.y)));
  }
  dft_input_twiddled<G::RC, true>(odd, p);
  schedule_fence();  // the even half's reads stay behind, or both halves' inputs are live at once
#pragma unroll
  for (int k = 0; k < G::RC; ++k) {
    const float2 a = b(0, k), c = b(0, k + G::RC);
    y[k] = make_float2(fmaf(-zi, c.y, fmaf(zr, c.x, a.x)), fmaf(zi, c.x, fmaf(zr, c.y, a.y)));
  }
  dft_input_twiddled<G::RC, true>(y, p);
#pragma unroll
  for (int k = 0; k < G::RC; ++k) {  // the odd half turned by the conjugate of w_M^n
    const float2 w = tab[G::OFF_W + j + G::L * (2 * k + parity)];
    y[k] = make_float2(fmaf(w.y, odd[k].y, fmaf(w.x, odd[k].x, y[k].x)),
                       fmaf(-w.y, odd[k].x, fmaf(w.x, odd[k].y, y[k].y)));
  }
}

// B without the transfer function: forward and inverse transforms over j of one (column, k1)
template <int M, int PAD>
__device__ __forceinline__ void col_freq_forward(float2* v, const float2* __restrict__ tab, int h, int k1) {
  using G = ColSplit<M, PAD>;
  float2 p[G::NB];
#pragma unroll
  for (int e = 0; e < G::NB; ++e) p[e] = tab[(e * G::NH + h) * G::R1 + k1];
  dft_input_twiddled<G::R2, false>(v, p);
}
template <int M, int PAD>
__device__ __forceinline__ void col_freq_inverse(float2* v) {
  DFT<ColSplit<M, PAD>::R2, true, false>::run(v);
}

// The four pairs of an eight-point transform with twiddled inputs, `step` table entries apart
template <bool INV>
__device__ __forceinline__ void dft8_table(float2* v, const float2* __restrict__ tab, int step) {
  float2 p[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) p[e] = tab[e * step];
  dft_fused<8, INV>(v, p);
}

}  // namespace dpx
