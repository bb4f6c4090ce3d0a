// Launchers of the propagation passes for one transform length M = DPX_M: row passes (every
// mode, single-design and grouped), column passes (every variant and transfer-function
// source, single-design and grouped, and the matrix-core form) and the transfer table.  The
// build compiles this file once per supported length, so the kernel templates of the
// different lengths are instantiated in parallel translation units.
#include <cmath>

#include "pass_kernels.hpp"

#ifndef DPX_M
#error "compile with -DDPX_M=<transform length>"
#endif

#define DPX_PASTE2(a, b) a##b
#define DPX_PASTE(a, b) DPX_PASTE2(a, b)
#define DPX_NAME(f) DPX_PASTE(f, DPX_M)

namespace dpx {
namespace {

constexpr int M = DPX_M;

unsigned group_grid(const GroupArgs& g) { return static_cast<unsigned>(g.block0[g.ntasks]); }

// runs f with the radix plan as a compile-time constant (plans beyond 0 exist for some lengths)
template <typename F>
hipError_t with_plan(int plan, F&& f) {
  if constexpr (radix_plans(M) > 1) {
    if (plan == 1) return f(std::integral_constant<int, 1>{});
    if (plan == 2) return f(std::integral_constant<int, 2>{});
  }
  if (plan == 0) return f(std::integral_constant<int, 0>{});
  return hipErrorInvalidValue;
}

template <int PAD, int V>
hipError_t row_mode(int mode, bool small, const RowArgs& a, dim3 grid, hipStream_t s) {
  if constexpr (M == 1600 && PAD == 2 && V == 0) {
    if (mode == ROW_FWD_MID || mode == ROW_ADJ_MID) {
      if (mode == ROW_FWD_MID)
        row_kernel_w3<M, PAD, ROW_FWD_MID><<<grid, row_block_threads<M, PAD, ROW_FWD_MID>(), 0, s>>>(a);
      else
        row_kernel_w3<M, PAD, ROW_ADJ_MID><<<grid, row_block_threads<M, PAD, ROW_ADJ_MID>(), 0, s>>>(a);
      return hipGetLastError();
    }
  }
  const auto go = [&](auto sc) -> hipError_t {
    constexpr bool SM = decltype(sc)::value;
    switch (mode) {
#define DPX_ROW(MD) \
  case MD: row_kernel<M, PAD, MD, V, SM><<<grid, row_block_threads<M, PAD, MD, SM>(), 0, s>>>(a); break;
      DPX_ROW(ROW_FWD_FIRST)
      DPX_ROW(ROW_FWD_MID)
      DPX_ROW(ROW_FWD_LAST)
      DPX_ROW(ROW_ADJ_SEED)
      DPX_ROW(ROW_ADJ_MID)
      DPX_ROW(ROW_ADJ_LAST)
      DPX_ROW(ROW_ADJ_LAST_U)
#undef DPX_ROW
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  };
  if (small) {
    if constexpr (Geo<M>::WAVE_LOCAL) return go(std::true_type{});
    else return hipErrorInvalidValue;
  }
  return go(std::false_type{});
}

template <int PAD>
hipError_t row_group_mode(int mode, const GroupArgs& g, hipStream_t s) {
  switch (mode) {
#define DPX_ROW(MD) \
  case MD: row_group_kernel<M, PAD, MD><<<group_grid(g), row_block_threads<M, PAD, MD>(), 0, s>>>(g); break;
    DPX_ROW(ROW_FWD_FIRST)
    DPX_ROW(ROW_FWD_MID)
    DPX_ROW(ROW_FWD_LAST)
    DPX_ROW(ROW_ADJ_SEED)
    DPX_ROW(ROW_ADJ_MID)
    DPX_ROW(ROW_ADJ_LAST)
    DPX_ROW(ROW_ADJ_LAST_U)
#undef DPX_ROW
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// H source of a launch: the table when the arguments carry one, the per-element evaluation
// with the translation ramp for a translated gap, else the variant's evaluation
int h_mode(int variant, bool table, bool shifted = false, bool band = false) {
  return table ? kHTable : band ? kHBand : shifted ? kHShift : (variant >= 2 ? kHMirror : kHEval);
}

// every aperture row in and out (the row-range tests compile away)
bool full_rows(const ColArgs& a) { return a.in_lo == 0 && a.out_lo == 0 && a.in_hi == a.n && a.out_hi == a.n; }

template <int PAD, int TX, int HM, int V>
hipError_t col_launch(bool conj, const ColArgs& a, int w_count, hipStream_t s) {
  constexpr int THREADS = ColShape<M, PAD, TX, V>::THREADS;
  dim3 grid(M / TX, (w_count + a.col_wpb - 1) / a.col_wpb);
  const bool full = full_rows(a);
  if constexpr (ColShape<M, PAD, TX, V>::SPLIT800) {
    if (grid.x * grid.y <= 256) {  // see col800_few_kernel
      if (conj) {
        if (full) col800_few_kernel<M, PAD, true, HM, true><<<grid, 512, 0, s>>>(a);
        else col800_few_kernel<M, PAD, true, HM, false><<<grid, 512, 0, s>>>(a);
      } else {
        if (full) col800_few_kernel<M, PAD, false, HM, true><<<grid, 512, 0, s>>>(a);
        else col800_few_kernel<M, PAD, false, HM, false><<<grid, 512, 0, s>>>(a);
      }
      return hipGetLastError();
    }
  }
  if (conj) {
    if (full) col_kernel<M, PAD, true, TX, HM, true, V><<<grid, THREADS, 0, s>>>(a);
    else col_kernel<M, PAD, true, TX, HM, false, V><<<grid, THREADS, 0, s>>>(a);
  } else {
    if (full) col_kernel<M, PAD, false, TX, HM, true, V><<<grid, THREADS, 0, s>>>(a);
    else col_kernel<M, PAD, false, TX, HM, false, V><<<grid, THREADS, 0, s>>>(a);
  }
  return hipGetLastError();
}

// tile widths of the transform variants: 8 / 16 columns (16 / 16 where 8 columns would not fill
// whole wavefronts, 8 / 8 for halves of 512 points), or 4 / 8 when a transform spans wavefronts (blocks stay within 1024 threads)
template <int PAD, int V>
constexpr int tile_narrow() {
  if (ColShape<M, PAD, 8, V>::SPLIT3 || ColShape<M, PAD, 8, V>::SPLIT800) return 8;
  if (ColShape<M, PAD, 16, V>::SPLIT) return ColSplit<M, PAD>::NARROW ? 8 : 16;
  return !Geo<M>::WAVE_LOCAL ? 4 : 8 * Geo<M>::P >= 64 ? 8 : 16;
}
template <int PAD, int V>
constexpr int tile_wide() {
  if (ColShape<M, PAD, 8, V>::SPLIT3 || ColShape<M, PAD, 8, V>::SPLIT800) return 8;
  return ColShape<M, PAD, 16, V>::SPLIT || Geo<M>::WAVE_LOCAL ? 16 : 8;
}
constexpr bool wide_variant(int variant) { return variant == 1 || variant == 3; }

// H sources of each radix plan: plan 0 has them all; the other plans only the evaluated and
// mirrored transfer functions of the untranslated, full-spectrum gap (the plan layer refuses
// the rest)
template <int PAD, int TX, int V>
hipError_t col_launch_h(int hm, bool conj, const ColArgs& a, int w_count, hipStream_t s) {
  if constexpr (V == 0) {
    if (hm == kHTable) return col_launch<PAD, TX, kHTable, V>(conj, a, w_count, s);
    if (hm == kHBand) return col_launch<PAD, TX, kHBand, V>(conj, a, w_count, s);
    if (hm == kHShift) return col_launch<PAD, TX, kHShift, V>(conj, a, w_count, s);
  } else {
    if (hm == kHTable || hm == kHBand || hm == kHShift) return hipErrorInvalidValue;
  }
  if constexpr (V == 0 && ColSplit800<M, PAD>::BUILT) {
    // whichever variant: the lanes of a column share a wavefront, and the mirrored form gives the bits
    // of the evaluated one (128 wavelengths: 1080 against 1215 us)
    return col_launch<PAD, TX, kHMirror, V>(conj, a, w_count, s);
  } else if constexpr (Geo<M>::WAVE_LOCAL) {
    if (hm == kHMirror) return col_launch<PAD, TX, kHMirror, V>(conj, a, w_count, s);
    return col_launch<PAD, TX, kHEval, V>(conj, a, w_count, s);
  } else {
    // the mirrored form exchanges H across the lanes of one wavefront
    if (hm == kHMirror) return hipErrorInvalidValue;
    return col_launch<PAD, TX, kHEval, V>(conj, a, w_count, s);
  }
}

template <int PAD>
hipError_t col_variant(int variant, int plan, bool conj, const ColArgs& args, int w_count, hipStream_t s) {
  const bool shifted = args.sx != 0.0 || args.sy != 0.0;
  const ColArgs& a = args;
  const int hm = h_mode(variant, a.htab != nullptr, shifted, a.band_limited != 0);
  return with_plan(plan, [&](auto vc) -> hipError_t {
    constexpr int V = decltype(vc)::value;
    if (!wide_variant(variant)) return col_launch_h<PAD, tile_narrow<PAD, V>(), V>(hm, conj, a, w_count, s);
    return col_launch_h<PAD, tile_wide<PAD, V>(), V>(hm, conj, a, w_count, s);
  });
}

template <int PAD>
hipError_t colgemm_launch(bool conj, const ColArgs& a, int w_count, hipStream_t s) {
  if constexpr (M <= 512 && M % 16 == 0 && (M / PAD) % 16 == 0) {
    ColArgs one = a;
    one.col_wpb = 1;
    dim3 grid(M / kGemmTile, w_count);
    if (conj)
      colgemm_kernel<M, PAD, true><<<grid, gemm_threads(M), 0, s>>>(one, a.dft);
    else
      colgemm_kernel<M, PAD, false><<<grid, gemm_threads(M), 0, s>>>(one, a.dft);
    return hipGetLastError();
  } else {
    return hipErrorInvalidValue;
  }
}

template <int PAD, int TX, int HM>
hipError_t col_group_tx(bool conj, bool full, const GroupArgs& g, hipStream_t s) {
  constexpr int THREADS = ColShape<M, PAD, TX, 0>::THREADS;
  if (conj) {
    if (full) col_group_kernel<M, PAD, true, TX, HM, true><<<group_grid(g), THREADS, 0, s>>>(g);
    else col_group_kernel<M, PAD, true, TX, HM, false><<<group_grid(g), THREADS, 0, s>>>(g);
  } else {
    if (full) col_group_kernel<M, PAD, false, TX, HM, true><<<group_grid(g), THREADS, 0, s>>>(g);
    else col_group_kernel<M, PAD, false, TX, HM, false><<<group_grid(g), THREADS, 0, s>>>(g);
  }
  return hipGetLastError();
}

template <int PAD, int TX>
hipError_t col_group_h(int hm, bool conj, bool full, const GroupArgs& g, hipStream_t s) {
  if (hm == kHTable) return col_group_tx<PAD, TX, kHTable>(conj, full, g, s);
  if constexpr (ColSplit800<M, PAD>::BUILT) {
    return col_group_tx<PAD, TX, kHMirror>(conj, full, g, s);
  } else if constexpr (Geo<M>::WAVE_LOCAL) {
    if (hm == kHMirror) return col_group_tx<PAD, TX, kHMirror>(conj, full, g, s);
    return col_group_tx<PAD, TX, kHEval>(conj, full, g, s);
  } else {
    if (hm == kHMirror) return hipErrorInvalidValue;
    return col_group_tx<PAD, TX, kHEval>(conj, full, g, s);
  }
}

template <int PAD>
hipError_t col_group_variant(int variant, bool table, bool conj, bool full, const GroupArgs& g, hipStream_t s) {
  const int hm = h_mode(variant, table);
  if (!wide_variant(variant)) return col_group_h<PAD, tile_narrow<PAD, 0>()>(hm, conj, full, g, s);
  return col_group_h<PAD, tile_wide<PAD, 0>()>(hm, conj, full, g, s);
}

}  // namespace

hipError_t DPX_NAME(launch_row_)(int pad, int mode, int plan, bool small, const RowArgs& a, int n_row_blocks, int n_w_blocks,
                                 hipStream_t s) {
  const dim3 grid(n_row_blocks, n_w_blocks);
  return with_plan(plan, [&](auto vc) -> hipError_t {
    constexpr int V = decltype(vc)::value;
    if (pad == 2) return row_mode<2, V>(mode, small, a, grid, s);
    if (pad == 1) return row_mode<1, V>(mode, small, a, grid, s);
    return hipErrorInvalidValue;
  });
}

hipError_t DPX_NAME(launch_row_group_)(int pad, int mode, const GroupArgs& g, hipStream_t s) {
  if (pad == 2) return row_group_mode<2>(mode, g, s);
  if (pad == 1) return row_group_mode<1>(mode, g, s);
  return hipErrorInvalidValue;
}

hipError_t DPX_NAME(launch_col_)(int pad, bool conj, int variant, int plan, const ColArgs& a, int w_count,
                                 hipStream_t s) {
  if (variant == 4) {
    if (a.sx != 0.0 || a.sy != 0.0) return hipErrorInvalidValue;  // matrix-core form: no translation
    if (pad == 2) return colgemm_launch<2>(conj, a, w_count, s);
    if (pad == 1) return colgemm_launch<1>(conj, a, w_count, s);
    return hipErrorInvalidValue;
  }
  if (pad == 2) return col_variant<2>(variant, plan, conj, a, w_count, s);
  if (pad == 1) return col_variant<1>(variant, plan, conj, a, w_count, s);
  return hipErrorInvalidValue;
}

void DPX_NAME(twiddle_table_)(int plan, const UnitRoots& u, std::vector<float2>& out) {
  out.clear();
  (void)with_plan(plan, [&](auto vc) -> hipError_t {
    twiddle_table_host<M, decltype(vc)::value>(out, u);
    return hipSuccess;
  });
}

void DPX_NAME(col_table_)(int pad, const UnitRoots& u, std::vector<float2>& out) {
  const auto build = [&](auto padc) {
    constexpr int PD = decltype(padc)::value;
    if constexpr (ColSplit800<M, PD>::BUILT) col800_table_host<M, PD>(out, u);
    else if constexpr (ColSplit3<M, PD>::BUILT) col3_table_host<M, PD>(out, u);
    else col_table_host<M, PD>(out, u);
  };
  if (pad == 2) build(std::integral_constant<int, 2>{});
  else build(std::integral_constant<int, 1>{});
}

bool DPX_NAME(col_split_)(int pad) {
  return pad == 2 ? ColSplit<M, 2>::BUILT || ColSplit3<M, 2>::BUILT || ColSplit800<M, 2>::BUILT : ColSplit<M, 1>::BUILT || ColSplit3<M, 1>::BUILT;
}

int DPX_NAME(col_tile_width_)(int pad, int variant) {
  if (pad == 2) return wide_variant(variant) ? tile_wide<2, 0>() : tile_narrow<2, 0>();
  return wide_variant(variant) ? tile_wide<1, 0>() : tile_narrow<1, 0>();
}

hipError_t DPX_NAME(launch_col_group_)(int pad, bool conj, int variant, bool table, bool full, const GroupArgs& g,
                                       hipStream_t s) {
  if (pad == 2) return col_group_variant<2>(variant, table, conj, full, g, s);
  if (pad == 1) return col_group_variant<1>(variant, table, conj, full, g, s);
  return hipErrorInvalidValue;
}

bool DPX_NAME(lds_supported_)(int pad) {
  return pad == 2 ? LdsGeo<M, 2>::FITS && M <= 128 : pad == 1 ? LdsGeo<M, 1>::FITS && M <= 128 : false;
}

hipError_t DPX_NAME(launch_lds_)(int pad, bool adjoint, const LdsArgs& a, hipStream_t s) {
  if constexpr (M <= 128) {
    auto go = [&](auto padc) -> hipError_t {
      constexpr int PD = decltype(padc)::value;
      if constexpr (LdsGeo<M, PD>::FITS) {
        if (adjoint && a.w_per_block > 1)
          lds_adjoint_kernel<M, PD, true><<<(a.W + a.w_per_block - 1) / a.w_per_block, kLdsThreads, 0, s>>>(a);
        else if (adjoint)
          lds_adjoint_kernel<M, PD, false><<<a.W, kLdsThreads, 0, s>>>(a);
        else
          lds_forward_kernel<M, PD><<<a.W, kLdsThreads, 0, s>>>(a);
        return hipGetLastError();
      } else {
        return hipErrorInvalidValue;
      }
    };
    if (pad == 2) return go(std::integral_constant<int, 2>{});
    if (pad == 1) return go(std::integral_constant<int, 1>{});
  }
  return hipErrorInvalidValue;
}

hipError_t DPX_NAME(launch_transfer_table_)(const WlConst* wl, int W, double zrev, float2* out, hipStream_t s) {
  const dim3 grid(M / 2 + 1, W);
  transfer_table_kernel<M><<<grid, 256, 0, s>>>(wl, zrev, out);
  return hipGetLastError();
}

}  // namespace dpx
