// Device code of the propagation passes for gfx950: row pass, column pass (transform and
// matrix-core forms), transfer-function table.  Included by the per-transform-length
// translation units (dpx_pass.hip), which instantiate the kernels of one length each.
//
// One propagation over a gap (Section 4, Eq. 4/5 via the angular spectrum) is split in two
// passes over a [N rows][M columns] complex plane per wavelength ("spec"):
//   row pass    : transform along x (the N non-zero rows of the zero-padded plane only)
//   column pass : transform along y, multiply by the transfer function, inverse along y,
//                 keep the N aperture rows
// and the next row pass starts with the inverse transform along x.  Zero padding is placed
// at the high end of each axis instead of centring it: a circular convolution commutes with
// shifts, so cropping the same corner returns the same N x N field.
#pragma once

#include <hip/hip_runtime.h>

#include "col_fft.hpp"
#include "dpx_internal.hpp"
#include "fft.hpp"
#include "phase.hpp"

namespace dpx {

// Word 3 of a raw buffer resource on gfx9: 32-bit data format, no stride or swizzle.
constexpr int kBufferRsrcWord3 = 0x00020000;

// One 8-byte load through a buffer resource: byte offset = voff (per lane) + soff (scalar).
__device__ __forceinline__ float2 buffer_load_c64(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
  const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
  return make_float2(__uint_as_float(v[0]), __uint_as_float(v[1]));
}

// One 8-byte store, the same way.
__device__ __forceinline__ void buffer_store_c64(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, float2 v) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 u = {__float_as_uint(v.x), __float_as_uint(v.y)};
  __builtin_amdgcn_raw_buffer_store_b64(u, r, voff, soff, 0);
}

// Reads an object that no kernel of the launch writes through the constant address space: scalar
// loads where the pointer is uniform (a plain load is a vector load as soon as the kernel stores
// anything, since the compiler cannot rule out an overlap).
template <typename T>
__device__ __forceinline__ T load_uniform(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "whole dwords");
  typedef const unsigned __attribute__((address_space(4)))* words;
  unsigned v[sizeof(T) / 4];
  const words q = (words) reinterpret_cast<uintptr_t>(p);
#pragma unroll
  for (unsigned i = 0; i < sizeof(T) / 4; ++i) v[i] = q[i];
  T out;
  __builtin_memcpy(&out, v, sizeof(T));
  return out;
}

// The lane's first row index, opaque to the optimiser: the per-element row terms of the
// transfer function (ky, ky^2, their conversions to FP64) are the same for every wavelength, and
// left visible the compiler keeps all E of them live across the wavelength loop, which spills.
// Derived from this value they are recomputed per wavelength (a few integer operations).
__device__ __forceinline__ int opaque_lane_row(int j0) {
  asm volatile("" : "+v"(j0));
  return j0;
}

// One spectrum row as the row passes read and write it: lane j0 holds columns j0 + P t.  The
// accesses go through a buffer resource over the wavelength's plane, and a lane whose column
// lies outside the disc takes an offset beyond the plane, so its load returns zero and its store
// is dropped without memory traffic and without a branch.  Bound by HBM: on the 1600-point glass
// design (28 % of the columns evanescent on average over 400-750 nm) the planes' traffic falls by
// as much; where every column propagates the select per access is hidden by the memory time.
template <int M, int PAD>
struct SpectrumRow {
  static constexpr int E = Geo<M>::E, P = Geo<M>::P;
  __amdgpu_buffer_rsrc_t rs;
  unsigned voff;  // byte offset of (row y, column j0)
  int j0, radius;

  // plane: uniform over the block; y and j0 per lane; radius: the wavelength's, or M (every column)
  __device__ __forceinline__ SpectrumRow(float2* plane, int y, int j0_, int radius_) : j0(j0_), radius(radius_) {
    const uint64_t base = reinterpret_cast<uint64_t>(plane);
    const uint64_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(base)));
    const uint64_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(base >> 32)));
    rs = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>((hi << 32) | lo), 0, M / PAD * M * 8,
                                           kBufferRsrcWord3);
    voff = static_cast<unsigned>((y * M + j0) * 8);
  }
  // The lane's offset in register t if its column is below `below` or at least `from`, else one past
  // every plane (j: j0, opaque, so that the offsets of the loads are not held for the stores).
  __device__ __forceinline__ unsigned offset(int t, int j, int below, int from) const {
    // a register's columns lie on one side of M / 2 where P divides it, the register in the middle
    // holds both sides otherwise
    bool in;
    if (P * (t + 1) <= M / 2) in = j < below - P * t;
    else if (P * t >= M / 2) in = j >= from - P * t;
    else in = j < below - P * t || j >= from - P * t;
    return in ? voff : 0x80000000u;
  }
  __device__ __forceinline__ void load(float2 (&reg)[E]) const {
    const int j = opaque_lane_row(j0);
#pragma unroll
    for (int t = 0; t < E; ++t) reg[t] = buffer_load_c64(rs, offset(t, j, radius + 1, M - radius), P * t * 8);
  }
  // stores end on whole 128-byte lines, or the memory pays for part of one at both ends of the gap
  // (first pass of 1024 wavelengths of 512 points: 209 us with ends at the disc, 183 without a gap)
  __device__ __forceinline__ void store(const float2 (&reg)[E]) const {
    const int j = opaque_lane_row(j0);
    const int below = (radius + 16) & ~15, from = M - ((radius + 15) & ~15);
#pragma unroll
    for (int t = 0; t < E; ++t) buffer_store_c64(rs, offset(t, j, below, from), P * t * 8, reg[t]);
  }
};

// Eq. 1 with the +j reading: t = exp(-ca h) exp(+i 2 pi rt h); phase argument in double.
__device__ __forceinline__ float2 transmission(float h, const WlConst& c) {
  asm volatile("" : "+v"(h));  // the FP64 height stays per wavelength (as in opaque_lane_row)
  const double hd = static_cast<double>(h);
  float2 t = cis_turns(c.rt * hd);
  if (c.ca != 0.0) {
    const float a = expf(-static_cast<float>(c.ca * hd));
    t.x *= a;
    t.y *= a;
  }
  return t;
}

template <int M, int PAD, int MODE, bool SMALL = false>
constexpr int row_block_threads() { return row_threads_for(M, Geo<M>::P, PAD, MODE, SMALL); }

// ------------------------------------------------------------------------------------------
// Row pass.  A block owns G = 256 / P consecutive rows (one transform group per row) and
// loops over a run of wavelengths, so the row's heights stay in registers.
// ------------------------------------------------------------------------------------------
// Block (bx, by) of a row pass: rows row_lo + bx G .. + G - 1, wavelength block by.
// lds_all: G exchange regions; tw: room for the twiddle table (both in LDS).
template <int M, int PAD, int MODE, int V = 0, bool SMALL = false>
__device__ __forceinline__ void row_body(const RowArgs& a, int bx, int by, float2* lds_all, float2* tw) {
  constexpr int kRowThreads = row_block_threads<M, PAD, MODE, SMALL>();
  constexpr int E = Geo<M>::E;
  constexpr int P = Geo<M>::P;
  constexpr int G = kRowThreads / P;
  constexpr int EN = E / PAD;  // registers that hold x < N
  constexpr bool HALF = (PAD == 2);
  constexpr int RG = Geo<M>::ROW_REGION;

  const int N = M / PAD;
  const int g = threadIdx.x / P;
  const int j0 = threadIdx.x % P;
  float2* lds = lds_all + g * RG;
  const int y_raw = a.row_lo + bx * G + g;
  const bool active = y_raw < a.row_hi;
  const int y = active ? y_raw : a.row_lo;
  const size_t nn = static_cast<size_t>(N) * N;
  // the lane's part of row y of wavelength w's plane
  auto spectrum = [&](int w, const WlConst& c) {
    return SpectrumRow<M, PAD>(a.spec + static_cast<size_t>(w - a.w_begin) * N * M, y, j0,
                               a.all_columns ? M : c.radius);
  };

  const int wb = a.w_begin + by * a.w_per_block;
  const int we = min(wb + a.w_per_block, a.w_begin + a.w_count);
  // A wavelength's row loads depend on its constants: they are scalar loads (load_uniform), read one
  // wavelength ahead, so that no wait for them comes on top of the rows'.  The twiddle table is requested
  // first, the first row behind it and before the table goes to LDS, every later row right behind the
  // stores of the one before.  (Loads return in order: with the row requested before the table, the
  // block's barrier waited for every wavefront's row.  Eight wavelengths of three unpadded 1024 x 1024
  // layers, forward: 231 -> 213 us, one of 512 x 512 padded 58 -> 55.5; no difference at thousands.)
  constexpr int TABLE = (twiddle_count<M, V>() + kRowThreads - 1) / kRowThreads;
  float2 table[TABLE];
#pragma unroll
  for (int k = 0; k < TABLE; ++k) {
    const int i = threadIdx.x + k * kRowThreads;
    if (i < twiddle_count<M, V>()) table[k] = a.tw[i];
  }
  WlConst c = load_uniform(a.wl + wb);
  auto constants_after = [&](int w) { return load_uniform(a.wl + min(w + 1, we - 1)); };
  auto stage_table = [&]() {
#pragma unroll
    for (int k = 0; k < TABLE; ++k) {
      const int i = threadIdx.x + k * kRowThreads;
      if (i < twiddle_count<M, V>()) tw[i] = table[k];
    }
    __syncthreads();
  };

  float hreg[EN];
  if constexpr (MODE == ROW_FWD_FIRST || MODE == ROW_FWD_MID || MODE == ROW_ADJ_MID ||
                MODE == ROW_ADJ_LAST || MODE == ROW_ADJ_LAST_U) {
    const bool read_h = MODE != ROW_FWD_FIRST || !a.no_layer;
#pragma unroll
    for (int t = 0; t < EN; ++t) hreg[t] = read_h ? a.h[static_cast<size_t>(y) * N + j0 + P * t] : 0.f;
  }

  if constexpr (MODE == ROW_FWD_FIRST) {
    float2 uin[EN];
#pragma unroll
    for (int t = 0; t < EN; ++t)
      uin[t] = a.u_in ? a.u_in[static_cast<size_t>(y) * N + j0 + P * t] : make_float2(1.f, 0.f);
    stage_table();
    for (int w = wb; w < we; ++w) {
      const int wc = w - a.w_begin;
      float2 reg[E];
      const WlConst next = constants_after(w);
      if (a.no_layer) {
#pragma unroll
        for (int t = 0; t < EN; ++t) reg[t] = uin[t];
      } else {
#pragma unroll
        for (int t = 0; t < EN; ++t) reg[t] = cmul(uin[t], transmission(hreg[t], c));
      }
      if (a.store_ckpt && !a.ckpt_first && active) {
        float2* ck = a.ckpt + (static_cast<size_t>(a.layer - a.ckpt_first) * a.ckpt_w_stride + wc) * nn +
                     static_cast<size_t>(y) * N;
#pragma unroll
        for (int t = 0; t < EN; ++t) ck[j0 + P * t] = reg[t];
      }
      fft<M, false, HALF, V, XPad<M>::ROWS>(reg, lds, j0, tw);
      if (active) spectrum(w, c).store(reg);
      c = next;
    }
  } else if constexpr (MODE == ROW_FWD_MID) {
    float2 reg[E];
    spectrum(wb, c).load(reg);
    stage_table();
    for (int w = wb; w < we; ++w) {
      const int wc = w - a.w_begin;
      const WlConst next = constants_after(w);
      fft<M, true, false, V, XPad<M>::ROWS>(reg, lds, j0, tw);
#pragma unroll
      for (int t = 0; t < EN; ++t) reg[t] = cmul(reg[t], transmission(hreg[t], c));
      if (a.store_ckpt && active) {
        float2* ck = a.ckpt + (static_cast<size_t>(a.layer - a.ckpt_first) * a.ckpt_w_stride + wc) * nn +
                     static_cast<size_t>(y) * N;
#pragma unroll
        for (int t = 0; t < EN; ++t) ck[j0 + P * t] = reg[t];
      }
      fft<M, false, HALF, V, XPad<M>::ROWS>(reg, lds, j0, tw);
      if (active) spectrum(w, c).store(reg);
      c = next;
      if (w + 1 < we) spectrum(w + 1, c).load(reg);
    }
  } else if constexpr (MODE == ROW_FWD_LAST) {
    const int F = a.fov;
    const int x0 = (N - F) / 2;
    float2 reg[E];
    spectrum(wb, c).load(reg);
    stage_table();
    for (int w = wb; w < we; ++w) {
      const int wc = w - a.w_begin;
      const WlConst next = constants_after(w);
      fft<M, true, false, V, XPad<M>::ROWS>(reg, lds, j0, tw);
      if (active) {
        float2* dst = a.ofov + static_cast<size_t>(wc) * F * F + static_cast<size_t>(y - x0) * F;
#pragma unroll
        for (int t = 0; t < EN; ++t) {
          const int x = j0 + P * t;
          if (x >= x0 && x < x0 + F) dst[x - x0] = reg[t];
        }
      }
      // The intensities too, where the block holds whole bins (G a multiple of the bin side): a
      // launch less (2.5 us of the 26 of the smallest forward).  Rows meet in the exchange regions.
      if (a.intensity) {
        const int b = a.bin, T = F / b;
        float* img = a.intensity + static_cast<size_t>(w) * T * T;
        if (b == 1) {
          if (active) {
#pragma unroll
            for (int t = 0; t < EN; ++t) {
              const int x = j0 + P * t;
              if (x >= x0 && x < x0 + F) img[(y - x0) * T + x - x0] = bin_sum(&reg[t], 1, 1);
            }
          }
        } else {
#pragma unroll
          for (int t = 0; t < EN; ++t) lds[j0 + P * t] = reg[t];
          __syncthreads();
          for (int i = threadIdx.x; i < G / b * T; i += kRowThreads) {
            const int ty = bx * (G / b) + i / T, tx = i % T;
            if (ty < T) img[ty * T + tx] = bin_sum(lds_all + (i / T * b) * RG + x0 + tx * b, RG, b);
          }
          __syncthreads();
        }
      }
      c = next;
      if (w + 1 < we) spectrum(w + 1, c).load(reg);
    }
  } else if constexpr (MODE == ROW_ADJ_SEED) {
    const int F = a.fov, b = a.bin, T = F / b;
    const int x0 = (N - F) / 2;
    stage_table();
    for (int w = wb; w < we; ++w) {
      const int wc = w - a.w_begin;
      const WlConst next = constants_after(w);
      const float2* o = a.ofov + static_cast<size_t>(wc) * F * F + static_cast<size_t>(y - x0) * F;
      const float* d = a.dl_di + static_cast<size_t>(w) * T * T + static_cast<size_t>((y - x0) / b) * T;
      float2 reg[E];
#pragma unroll
      for (int t = 0; t < EN; ++t) {
        const int x = j0 + P * t;
        if (x >= x0 && x < x0 + F) {
          const float s = 2.0f * kAdjointScale * d[(x - x0) / b];
          reg[t] = cscale(o[x - x0], s);
        } else {
          reg[t] = make_float2(0.f, 0.f);
        }
      }
      fft<M, false, HALF, V, XPad<M>::ROWS>(reg, lds, j0, tw);
      if (active) spectrum(w, c).store(reg);
      c = next;
    }
  } else {  // ROW_ADJ_MID, ROW_ADJ_LAST, ROW_ADJ_LAST_U
    // ROW_ADJ_LAST_U: the input field meets the first layer directly, so the field after the
    // first transmission is u_in t_0(h); the pass rebuilds it from the input and the heights
    // with the same operations as the first forward pass (so the same bits) instead of
    // reading back a stored copy.  u_in is read where it is used, not held in registers.
    constexpr bool REBUILD = (MODE == ROW_ADJ_LAST_U);
    const float2* urow = (REBUILD && a.u_in) ? a.u_in + static_cast<size_t>(y) * N : nullptr;
    float acc[EN];
#pragma unroll
    for (int t = 0; t < EN; ++t) acc[t] = 0.f;
    float2 reg[E];
    spectrum(wb, c).load(reg);
    stage_table();
    for (int w = wb; w < we; ++w) {
      const int wc = w - a.w_begin;
      const WlConst next = constants_after(w);
      const float2* ck = REBUILD ? nullptr
                                 : a.ckpt + (static_cast<size_t>(a.layer - a.ckpt_first) * a.ckpt_w_stride + wc) * nn +
                                       static_cast<size_t>(y) * N;
      fft<M, true, false, V, XPad<M>::ROWS>(reg, lds, j0, tw);
      const float ct = c.ct;
      const float ca = static_cast<float>(c.ca) / kAdjointScale;
#pragma unroll
      for (int t = 0; t < EN; ++t) {
        const float2 gv = reg[t];
        float2 v;
        if constexpr (REBUILD) {
          const float2 u = urow ? urow[j0 + P * t] : make_float2(1.f, 0.f);
          v = cmul(u, transmission(hreg[t], c));
        } else {
          v = ck[j0 + P * t];
        }
        // conj(g) v; acc += -ct Im - ca Re
        const float re = fmaf(gv.x, v.x, gv.y * v.y);
        const float im = fmaf(gv.x, v.y, -(gv.y * v.x));
        acc[t] = fmaf(-ct, im, fmaf(-ca, re, acc[t]));
        if constexpr (MODE == ROW_ADJ_MID) reg[t] = cmulc(gv, transmission(hreg[t], c));
      }
      if constexpr (MODE == ROW_ADJ_MID) {
        fft<M, false, HALF, V, XPad<M>::ROWS>(reg, lds, j0, tw);
        if (active) spectrum(w, c).store(reg);
      }
      c = next;
      if (w + 1 < we) spectrum(w + 1, c).load(reg);
    }
    if (active) {
      float* dst = a.dh_part +
                   (static_cast<size_t>(a.chunk_base + by) * a.layers + a.layer) * nn +
                   static_cast<size_t>(y) * N;
      if (a.accumulate) {
#pragma unroll
        for (int t = 0; t < EN; ++t) dst[j0 + P * t] += acc[t];
      } else {
#pragma unroll
        for (int t = 0; t < EN; ++t) dst[j0 + P * t] = acc[t];
      }
    }
  }
}

template <int M, int PAD, int MODE, int V = 0, bool SMALL = false>
__global__ void __launch_bounds__((row_block_threads<M, PAD, MODE, SMALL>())) row_kernel(RowArgs a) {
  __shared__ float2 lds_all[row_block_threads<M, PAD, MODE, SMALL>() / Geo<M>::P * Geo<M>::ROW_REGION];
  __shared__ float2 tw[twiddle_count<M, V>()];
  row_body<M, PAD, MODE, V, SMALL>(a, blockIdx.x, blockIdx.y, lds_all, tw);
}

// The same pass with at least three wavefronts per SIMD (a cap of 168 registers): the forward
// middle pass at transform 1600 fits it without spilling, and three of its 240-thread blocks
// then share a CU instead of two.
template <int M, int PAD, int MODE>
__global__ void __launch_bounds__((row_block_threads<M, PAD, MODE>())) __attribute__((amdgpu_waves_per_eu(3)))
row_kernel_w3(RowArgs a) {
  __shared__ float2 lds_all[row_block_threads<M, PAD, MODE>() / Geo<M>::P * Geo<M>::ROW_REGION];
  __shared__ float2 tw[twiddle_count<M>()];
  row_body<M, PAD, MODE>(a, blockIdx.x, blockIdx.y, lds_all, tw);
}

// One launch of a row pass for several designs of the same transform length and mode: each
// block finds its design's task, patches the per-call buffers into the design's arguments
// and runs the same body as the single-design kernel.
template <int M, int PAD, int MODE>
__global__ void __launch_bounds__((row_block_threads<M, PAD, MODE>())) row_group_kernel(GroupArgs g) {
  __shared__ float2 lds_all[row_block_threads<M, PAD, MODE>() / Geo<M>::P * Geo<M>::ROW_REGION];
  __shared__ float2 tw[twiddle_count<M>()];
  const int ti = group_task(g, blockIdx.x);
  const RowTask t = load_uniform(static_cast<const RowTask*>(g.tasks) + ti);
  const int local = static_cast<int>(blockIdx.x) - g.block0[ti];
  if (local >= t.nblocks) return;  // alignment padding between tasks
  RowArgs a = t.a;
  a.h = g.call.h ? g.call.h + t.h_off : nullptr;
  a.u_in = g.call.u_in ? g.call.u_in + t.u_off : nullptr;
  a.dl_di = g.call.dl_di ? g.call.dl_di + t.img_off : nullptr;
  if constexpr (MODE == ROW_FWD_LAST) a.intensity = t.bins ? g.call.intensity + t.img_off : nullptr;
  row_body<M, PAD, MODE>(a, local % t.gx, local / t.gx, lds_all, tw);
}

// H(kx, ky) / M^2 with the conjugate for the adjoint; 0 outside the propagating disc.  zrev is
// the phase in revolutions per unit of sqrt(q); outside the disc q is replaced by the smallest
// normal double (one maximum instead of two selects) and the result by 0.
template <int M, bool CONJ>
__device__ __forceinline__ float2 transfer(double zrev, double base, int ky) {
  const int kys = ky < M / 2 ? ky : ky - M;
  const double q = base - static_cast<double>(kys * kys);
  const float2 hh = cis_turns_hw<M * M>(zrev * sqrt_pos(fmax(q, kMinNormalF64)));
  return q > 0.0 ? (CONJ ? conjf2(hh) : hh) : make_float2(0.f, 0.f);
}

// ------------------------------------------------------------------------------------------
// Column pass.  A block owns TX adjacent columns of one wavelength's plane: it stages the
// [rows][TX] tile through LDS (coalesced 8*TX-byte row segments), each transform group
// then runs forward FFT -> transfer function -> inverse FFT on its column in registers, and
// the kept rows go back through the same LDS tile.
// ------------------------------------------------------------------------------------------
// Where a column pass takes the transfer function from: evaluated for every element, evaluated
// for the rows ky <= M/2 and shared with the mirrored rows across lanes, or read from the
// plan's table; a translated gap evaluates every element with its translation ramp folded into
// the phase; the band-limited spectrum evaluates every element inside the band.
constexpr int kHEval = 0, kHMirror = 1, kHTable = 2, kHShift = 3, kHBand = 4;

// XCD-aware order of a column pass's blocks.  Consecutive blocks go to the eight XCDs in turn,
// so blocks L and L + 8 of every run of 16 share an XCD and its L2; they take neighbouring
// column tiles of the same wavelength block, so the two halves of each 128-byte row segment
// meet in one L2 instead of being fetched twice.  Blocks are numbered L = bx + gx by from a
// multiple of 16 in launch order; with an even tile count gx a pair never straddles two
// wavelength blocks; a tail of fewer than 16 blocks keeps its order.
__device__ __forceinline__ void col_block_item(int L, int total, int gx, int& bx, int& by) {
  int item = L;
  if ((gx & 1) == 0 && L < (total & ~15)) {
    const int r = L & 15;
    item = (L & ~15) + ((r & 7) << 1) + (r >> 3);
  }
  bx = item % gx;
  by = item / gx;
}

// Drops the wavelengths at both ends of [wb, we) for which every column of the tile at kx0 lies
// outside the propagating disc: such columns are never read back (SpectrumRow), so a block with
// nothing else ends at once.  A wavelength between two others is transformed all the same; what
// it leaves in columns outside its disc is not read.
template <int M, int TX>
__device__ __forceinline__ void trim_evanescent(const ColArgs& a, int kx0, int& wb, int& we) {
  const int k = kx0 < M / 2 ? kx0 : M - (kx0 + TX - 1);  // the tile's smallest |kx|
  while (wb < we && k > load_uniform(&a.wl[a.w_begin + wb].radius)) ++wb;
  while (wb < we && k > load_uniform(&a.wl[a.w_begin + we - 1].radius)) --we;
}

// Block (bx, by) of a column pass: column tile bx, wavelength block by.
template <int M, int PAD, bool CONJ, int TX, int HM, bool FULL, int V = 0>
__device__ __forceinline__ void col_body(const ColArgs& a, int bx, int by, float2* tile, float2* tw) {
  constexpr int E = Geo<M>::E;
  constexpr int P = Geo<M>::P;
  constexpr int NT = TX * P;
  constexpr int LD = Geo<M>::COL_REGION;  // one column's staging rows / exchange region
  constexpr int EN = E / PAD;
  constexpr bool HALF = (PAD == 2);
  static_assert(NT / TX == P, "staging rows per pass");

  const int N = M / PAD;
  const int kx0 = bx * TX;
  const int cc = threadIdx.x % TX;
  const int yy = threadIdx.x / TX;
  const int g = threadIdx.x / P;
  const int j0 = threadIdx.x % P;
  float2* lds = tile + g * LD;
  const int kx = kx0 + g;
  const int kxs = kx < M / 2 ? kx : kx - M;
  // staged rows of tile column c start SKEW (c / 2) slots into its region (bank spread of the
  // staging with block-padded regions); the transforms' exchanges use the region from slot 0
  constexpr int SKEW = XPad<M>::SKEW;
  float2* lds_in = lds + SKEW * (g >> 1);
  float2* stg = tile + cc * LD + SKEW * (cc >> 1);

  // The block runs a.col_wpb wavelengths.  With zero padding the staged rows of the next one
  // are loaded into registers while the current one is transformed, so their latency is
  // hidden; without it those registers would not fit next to the full-length transform (nor
  // next to the band-limited source's per-element band tests) and the rows go straight to LDS.
  // Row k of a lane is one buffer load at the lane's 32-bit byte offset plus the scalar offset
  // k P M 8, so no per-row address stays live.
  constexpr bool PREFETCH = HALF && HM != kHBand;
  int wb = by * a.col_wpb;
  int we = min(wb + a.col_wpb, a.w_count);
  trim_evanescent<M, TX>(a, kx0, wb, we);
  if (wb >= we) return;
  const unsigned voff = static_cast<unsigned>((((FULL ? 0 : a.in_lo) + yy) * M + kx0 + cc) * 8);
  // The plane's base address is the same in every lane; reading it through readfirstlane
  // keeps the descriptor in scalar registers (a descriptor left in vector registers makes
  // the compiler wrap every load in a loop over the distinct descriptors of the wavefront).
  auto plane = [&](int w) {
    const uint64_t base = reinterpret_cast<uint64_t>(a.spec + static_cast<size_t>(w) * N * M);
    const uint64_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(base)));
    const uint64_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(base >> 32)));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>((hi << 32) | lo), 0, N * M * 8,
                                             kBufferRsrcWord3);
  };
  // FULL: the pass reads and keeps every aperture row (all passes but the first adjoint and
  // the last forward one), so the row-range tests drop out.
  const int in_lo = FULL ? 0 : a.in_lo, in_hi = FULL ? N : a.in_hi;
  const int out_lo = FULL ? 0 : a.out_lo, out_hi = FULL ? N : a.out_hi;
  float2 pre[PREFETCH ? EN : 1];
  auto fetch = [&](int w) {
    const auto rs = plane(w);
#pragma unroll
    for (int k = 0; k < EN; ++k) {
      const int y = in_lo + yy + k * P;
      pre[PREFETCH ? k : 0] = (y < in_hi) ? buffer_load_c64(rs, voff, k * P * M * 8) : make_float2(0.f, 0.f);
      if constexpr (!PREFETCH) {
        if (y < in_hi) stg[y] = pre[0];
      }
    }
  };
  auto stage = [&]() {
#pragma unroll
    for (int k = 0; k < EN; ++k) {
      const int y = in_lo + yy + k * P;
      if (y < in_hi) stg[y] = pre[k];
    }
  };
  // With every row in and out, the tile elements a thread stages for the next wavelength are
  // exactly those it copies out for the current one, so the staging follows the copy-out
  // without a barrier between them.
  constexpr bool STAGE_AFTER_STORE = FULL && PREFETCH;
  if constexpr (PREFETCH) fetch(wb);
  stage_twiddles<M, V>(tw, a.tw, threadIdx.x, NT);
  if constexpr (STAGE_AFTER_STORE) stage();

  // the twiddles of one stage stay in registers for the block's wavelengths (fewer LDS reads;
  // loaded after the first barrier, which also orders the table's staging) where the transfer
  // function leaves room for them: the evaluated, table and translated sources would spill
  constexpr bool TREG = (HM == kHMirror || HM == kHBand);
  float2 treg[RegTwiddles<M, V>::N];
  for (int w = wb; w < we; ++w) {
    if constexpr (!STAGE_AFTER_STORE) {
      if constexpr (PREFETCH) stage();
      else fetch(w);
    }
    __syncthreads();
    if (TREG && w == wb) load_register_twiddles<M, V>(treg, tw, j0);
    if constexpr (PREFETCH) {
      if (w + 1 < we) fetch(w + 1);
    }

    const WlConst c = load_uniform(a.wl + a.w_begin + w);
    float2 reg[E];
#pragma unroll
    for (int t = 0; t < EN; ++t) {
      const int y = j0 + P * t;
      reg[t] = (y >= in_lo && y < in_hi) ? lds_in[y] : make_float2(0.f, 0.f);
    }
    group_sync<M>();
    fft_sel<M, false, HALF, V, TREG>(reg, lds, j0, tw, treg);

    // transfer function H = exp(+i 2 pi z sqrt(q)) / M^2 on the propagating disc, else 0:
    // read from the plan's table of H(|kx|, |ky|) when there is one, else evaluated here.
    const double base = c.q0 - static_cast<double>(kxs * kxs);
    auto H = [&](int ky) { return transfer<M, CONJ>(a.zrev, base, ky); };
    if constexpr (HM == kHEval) {
      // the product is selected, not H: outside the disc the element becomes +0 and the compiler
      // branches the evaluation over runs of rows that lie wholly outside (a wavefront's rows are
      // consecutive ky), which at long wavelengths on a fine pitch are most of the plane
      const int jv = opaque_lane_row(j0);
#pragma unroll
      for (int t = 0; t < E; ++t) {
        const int ky = jv + P * t;
        const int kys = ky < M / 2 ? ky : ky - M;
        const double q = base - static_cast<double>(kys * kys);
        const float2 hh = cis_turns_hw<M * M>(a.zrev * sqrt_pos(fmax(q, kMinNormalF64)));
        reg[t] = q > 0.0 ? cmul(reg[t], CONJ ? conjf2(hh) : hh) : make_float2(0.f, 0.f);
      }
    } else if constexpr (HM == kHBand) {
      // band-limited angular spectrum: H = 0 where |kx| or |ky| exceeds the band limit
      // sqrt(q0 / (4 zrev^2 + 1)) (in frequency indices), beyond which the sampled phase aliases
      const double lim = c.q0 / (4.0 * a.zrev * a.zrev + 1.0);
      const bool col_in = static_cast<double>(kxs * kxs) <= lim;
      const int jv = opaque_lane_row(j0);
#pragma unroll
      for (int t = 0; t < E; ++t) {
        const int ky = jv + P * t;
        const int kys = ky < M / 2 ? ky : ky - M;
        const bool in = col_in && static_cast<double>(kys * kys) <= lim;
        reg[t] = in ? cmul(reg[t], H(ky)) : make_float2(0.f, 0.f);
      }
    } else if constexpr (HM == kHTable) {
      // table row of |kx|: every lane reads its E values (rows ky and M - ky share an entry)
      constexpr int HS = M / 2 + 1;
      const float2* hrow = a.htab + (static_cast<size_t>(a.w_begin + w) * HS + (kxs < 0 ? -kxs : kxs)) * HS;
      float2 hv[E];
#pragma unroll
      for (int t = 0; t < E; ++t) {
        const int ky = j0 + P * t;
        hv[t] = hrow[ky <= M / 2 ? ky : M - ky];
      }
#pragma unroll
      for (int t = 0; t < E; ++t) reg[t] = cmul(reg[t], CONJ ? conjf2(hv[t]) : hv[t]);
    } else if constexpr (HM == kHShift) {
      // translated gap: H times the ramp exp(-i 2 pi (kx sx + ky sy)) (signed indices) is one
      // phase per element, z sqrt(q) - kx sx - ky sy in revolutions, reduced in FP64 like H's
      // own; conjugated for the adjoint.  Per element, so no lane holds ramp state and the
      // next wavelength's rows still fit in registers.
      const double px = static_cast<double>(kxs) * a.sx;
      const int jv = opaque_lane_row(j0);
#pragma unroll
      for (int t = 0; t < E; ++t) {
        const int ky = jv + P * t;
        const int kys = ky < M / 2 ? ky : ky - M;
        const double q = base - static_cast<double>(kys * kys);
        const double ph = a.zrev * sqrt_pos(fmax(q, kMinNormalF64)) - fma(static_cast<double>(kys), a.sy, px);
        const float2 hh = cis_turns_hw<M * M>(ph);
        reg[t] = q > 0.0 ? cmul(reg[t], CONJ ? conjf2(hh) : hh) : make_float2(0.f, 0.f);
      }
    } else if constexpr (HM == kHMirror) {
      // H depends on ky^2 only: lane j0 holds ky = j0 + P t, and for t >= E/2 the row M - ky
      // is register E-1-t of lane P - j0 (lane 0 mirrors onto its own register E - t), so
      // each lane evaluates E/2 + 1 rows and fetches the others across lanes.  Streamed so
      // that only two evaluations are live at a time: step u applies row u and the mirrored
      // row E-1-u (whose value lane 0 takes from its own evaluation u+1).
      constexpr int EH = E / 2;
      const int lane = threadIdx.x & 63;
      const int src = ((lane - j0) + ((P - j0) & (P - 1))) << 2;
      float2 cur = H(j0);
#pragma unroll
      for (int u = 0; u < EH; ++u) {
        const float2 nxt = H(j0 + P * (u + 1));
        reg[u] = cmul(reg[u], cur);
        float2 m;
        m.x = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(cur.x)));
        m.y = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(cur.y)));
        if (j0 == 0) m = nxt;
        reg[E - 1 - u] = cmul(reg[E - 1 - u], m);
        cur = nxt;
      }
    }
    fft_sel<M, true, false, V, TREG>(reg, lds, j0, tw, treg);
    group_sync<M>();
#pragma unroll
    for (int t = 0; t < EN; ++t) {
      const int y = j0 + P * t;
      if (y >= out_lo && y < out_hi) lds_in[y] = reg[t];
    }
    __syncthreads();
    float2* sp = a.spec + static_cast<size_t>(w) * N * M + kx0 + cc;
    if constexpr (FULL) {
#pragma unroll
      for (int k = 0; k < EN; ++k) sp[static_cast<size_t>(yy + k * P) * M] = stg[yy + k * P];
    } else {
      for (int y = out_lo + yy; y < out_hi; y += P) sp[static_cast<size_t>(y) * M] = stg[y];
    }
    if constexpr (STAGE_AFTER_STORE) {
      if (w + 1 < we) stage();
    } else {
      __syncthreads();  // the next wavelength's staging overwrites the tile
    }
  }
}

// Transfer function of the split column transforms on v[k2], k2 = 0 .. R2 - 1, of lane k1 < R1 of a
// column and half h: element k2 is frequency ky = NH (k1 + R1 k2) + h.  HC: the half where it is known at
// compile time (a body of its own per half), else -1.
template <int M, int PAD, bool CONJ, int HM, int HC, int R1, int R2>
__device__ __forceinline__ void apply_transfer(float2* v, const ColArgs& a, const WlConst& c, int w, int kx, int half,
                                               int k1) {
  const int h = HC >= 0 ? HC : half;
  constexpr int NH = PAD;
  const int kxs = kx < M / 2 ? kx : kx - M;
  const double base = c.q0 - static_cast<double>(kxs * kxs);
  const int row0 = opaque_lane_row(NH * k1 + h);  // frequency of k2 = 0 (see opaque_lane_row)
  auto ky_of = [&](int k2) { return row0 + NH * R1 * k2; };
  if constexpr (HM == kHMirror) {
    // H depends on ky^2 only: frequency M - ky of (k1, k2) belongs to k1' = R1 - k1 - h (mod R1) at
    // k2' = R2 - 1 - k2, or at R2 - k2 on the lane k1 = 0 of the even half, which mirrors onto
    // itself.  So a lane evaluates the lower half of its frequencies (that one lane one more) and
    // takes the upper half from its partner.
    const int partner = h ? R1 - 1 - k1 : (k1 ? R1 - k1 : 0);
    const int src = ((static_cast<int>(threadIdx.x) & 63) - k1 + partner) << 2;
    const bool self = h == 0 && k1 == 0;
    float2 cur = transfer<M, CONJ>(a.zrev, base, ky_of(0));
#pragma unroll
    for (int u = 0; u < R2 / 2; ++u) {
      float2 nxt = cur;  // the odd half needs no value past the lower half
      if (u + 1 < R2 / 2 || HC != 1) nxt = transfer<M, CONJ>(a.zrev, base, ky_of(u + 1));
      v[u] = cmul(v[u], cur);
      float2 m;
      m.x = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(cur.x)));
      m.y = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(cur.y)));
      if (self) m = nxt;
      v[R2 - 1 - u] = cmul(v[R2 - 1 - u], m);
      cur = nxt;
    }
    static_assert(R2 % 2 == 0, "mirrored pairs");
  } else if constexpr (HM == kHTable) {
    constexpr int HS = M / 2 + 1;
    const float2* hrow = a.htab + (static_cast<size_t>(a.w_begin + w) * HS + (kxs < 0 ? -kxs : kxs)) * HS;
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2) {
      const int ky = ky_of(k2);
      const float2 hh = hrow[ky <= M / 2 ? ky : M - ky];
      v[k2] = cmul(v[k2], CONJ ? conjf2(hh) : hh);
    }
  } else {
    // per element (evaluated, translated or band-limited); the product is selected, not H, so that
    // the compiler branches the evaluation over runs of frequencies outside the disc or band
    const double px = HM == kHShift ? static_cast<double>(kxs) * a.sx : 0.0;
    const double lim = HM == kHBand ? c.q0 / (4.0 * a.zrev * a.zrev + 1.0) : 0.0;
    const bool col_in = HM != kHBand || static_cast<double>(kxs * kxs) <= lim;
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2) {
      const int ky = ky_of(k2);
      const int kys = ky < M / 2 ? ky : ky - M;
      if constexpr (HM == kHBand) {
        const bool in = col_in && static_cast<double>(kys * kys) <= lim;
        v[k2] = in ? cmul(v[k2], transfer<M, CONJ>(a.zrev, base, ky)) : make_float2(0.f, 0.f);
      } else {
        const double q = base - static_cast<double>(kys * kys);
        double ph = a.zrev * sqrt_pos(fmax(q, kMinNormalF64));
        // translated gap: H times the ramp exp(-i 2 pi (kx sx + ky sy)) is one phase, reduced in
        // FP64 like H's own; conjugated for the adjoint
        if constexpr (HM == kHShift) ph -= fma(static_cast<double>(kys), a.sy, px);
        const float2 hh = cis_turns_hw<M * M>(ph);
        v[k2] = q > 0.0 ? cmul(v[k2], CONJ ? conjf2(hh) : hh) : make_float2(0.f, 0.f);
      }
    }
  }
}

// Block (bx, by) of a column pass with split transforms (col_fft.hpp): column tile bx, wavelength
// block by.  The halves run on different wavefronts.  Three block barriers per wavelength: after
// the writes of A, after those of B, and before the next wavelength's A overwrites what C read.
template <int M, int PAD, bool CONJ, int TX, int HM, bool FULL>
__device__ __forceinline__ void col_split_body(const ColArgs& a, int bx, int by, float2* tile, float2* tab) {
  using G = ColSplit<M, PAD>;
  constexpr int N = M / PAD;
  constexpr int NT = G::threads(TX), R1 = G::R1, R2 = G::R2, L = G::L, GP = G::GP, REG = G::region(TX);
  constexpr int HALF_A = TX * L, HALF_B = TX * GP;  // threads of one half in A and C, and in B
  static_assert(HALF_A % 64 == 0 || G::NH == 1, "the half is the same over a wavefront");
  const int tid = threadIdx.x;
  const int kx0 = bx * TX;
  int wb = by * a.col_wpb;
  int we = min(wb + a.col_wpb, a.w_count);
  trim_evanescent<M, TX>(a, kx0, wb, we);
  if (wb >= we) return;

  // A and C: column cc, rows j + L r; ha: the half in A, the row parity in C
  const bool rows = tid < G::NH * HALF_A;
  const int ha = G::NH == 2 ? __builtin_amdgcn_readfirstlane(tid / HALF_A) : 0;
  const int cc = tid % TX, j = (tid / TX) % L;
  float2* const own = tile + (static_cast<size_t>(ha) * TX + cc) * REG;
  // B: column cb, k1 of half hb
  const int k1 = tid % GP, cb = (tid / GP) % TX;
  const int hb = HALF_B % 64 == 0 ? __builtin_amdgcn_readfirstlane(tid / HALF_B) : tid / HALF_B;
  const bool freq = k1 < R1 && hb < G::NH;
  float2* const freq_slots = tile + (static_cast<size_t>(hb < G::NH ? hb : 0) * TX + cb) * REG + G::slot(k1, 0);

  auto plane = [&](int w) {
    const uint64_t base = reinterpret_cast<uint64_t>(a.spec + static_cast<size_t>(w) * N * M);
    const uint64_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(base)));
    const uint64_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(base >> 32)));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>((hi << 32) | lo), 0, N * M * 8,
                                             kBufferRsrcWord3);
  };
  const unsigned voff = static_cast<unsigned>((j * M + kx0 + cc) * 8);
  constexpr unsigned kNowhere = 0x80000000u;  // beyond every plane: loads give zero, stores drop
  // The rows of the first wavelength are requested before the table is staged, those of a later one
  // when B of the one before is done, so that they arrive during its C.
  float2 v[R1];
  auto fetch = [&](int w) {
    if (!rows) return;
    const auto rs = plane(w);
    const int jv = opaque_lane_row(j);
#pragma unroll
    for (int r = 0; r < R1; ++r) {
      const int y = jv + L * r;
      const unsigned off = (FULL || (y >= a.in_lo && y < a.in_hi)) ? voff : kNowhere;
      v[r] = buffer_load_c64(rs, off, L * r * M * 8);
    }
  };
  fetch(wb);
  for (int i = tid; i < G::COUNT; i += NT) tab[i] = a.tw[i];
  for (int w = wb; w < we; ++w) {
    if (rows) {
      if (G::NH == 2 && ha) col_rows_forward<M, PAD, true>(v);
      else col_rows_forward<M, PAD, false>(v);
    }
    if (w > wb) __syncthreads();  // C of the wavelength before has read the slots
    if (rows) {
#pragma unroll
      for (int k = 0; k < R1; ++k) own[G::slot(k, j)] = v[k];
    }
    __syncthreads();
    const WlConst c = load_uniform(a.wl + a.w_begin + w);
    auto frequencies = [&](auto hc, int h) {
      constexpr int HC = decltype(hc)::value;
      float2 f[R2];
#pragma unroll
      for (int i = 0; i < R2; ++i) f[i] = freq_slots[i];
      col_freq_forward<M, PAD>(f, tab, h, k1);
      apply_transfer<M, PAD, CONJ, HM, HC, R1, R2>(f, a, c, w, kx0 + cb, h, k1);
      col_freq_inverse<M, PAD>(f);
#pragma unroll
      for (int i = 0; i < R2; ++i) freq_slots[i] = f[i];
    };
    // A body per half saves the odd one an evaluation of H; worth it for the longest split only (512
    // points, 1024 wavelengths: 604 against 620 us), shorter ones lose more to the longer code
    // (256 points 171 against 152 us, 192 points, 2048 wavelengths, 224 against 183 us).
    constexpr bool BOTH = G::NH == 2 && G::LEN >= 256;
    if (freq) {
      if constexpr (BOTH) {
        if (hb) frequencies(std::integral_constant<int, 1>{}, 1);
        else frequencies(std::integral_constant<int, 0>{}, 0);
      } else {
        frequencies(std::integral_constant<int, G::NH == 2 ? -1 : 0>{}, hb);
      }
    }
    // v starts anew here: where no rows follow, its old values would otherwise stay live through B
#pragma unroll
    for (int r = 0; r < R1; ++r) asm volatile("" : "=v"(v[r].x), "=v"(v[r].y));
    if (w + 1 < we) fetch(w + 1);
    __syncthreads();
    if (rows) {
      const auto rs = plane(w);
      const int jv = opaque_lane_row(j);
      if constexpr (G::NH == 2) {
        float2 y[G::RC];
        col_rows_inverse2<M, PAD>(y, tab, j, ha, [&](int h, int k) {
          return tile[(static_cast<size_t>(h) * TX + cc) * REG + G::slot(k, j)];
        });
#pragma unroll
        for (int r = 0; r < G::RC; ++r) {
          const int row = jv + L * (2 * r + ha);
          const unsigned off = (FULL || (row >= a.out_lo && row < a.out_hi)) ? voff : kNowhere;
          buffer_store_c64(rs, off, L * (2 * r + ha) * M * 8, y[r]);
        }
      } else {
        float2 y[R1];
#pragma unroll
        for (int k = 0; k < R1; ++k) y[k] = own[G::slot(k, j)];
        col_rows_inverse<M, PAD>(y, tab, j);
#pragma unroll
        for (int r = 0; r < R1; ++r) {
          const int row = jv + L * r;
          const unsigned off = (FULL || (row >= a.out_lo && row < a.out_hi)) ? voff : kNowhere;
          buffer_store_c64(rs, off, L * r * M * 8, y[r]);
        }
      }
    }
  }
}

// The same for halves of 512 points (ColSplit3): eight columns, one wavefront per column in B, the
// halves one after the other, one wavelength per block.  Two block barriers per half, none between a
// half's C and the next A, since a row thread's slots are its own.  Bound by vector issue: at four cycles
// each and the 1.8 to 1.9 GHz that they leave the chip, the 1197 vector instructions per wavefront take the
// whole launch (VALU busy 111 %, 88 % in the staged form).  Three blocks of eight wavefronts share a CU;
// 1024 points, 1024 wavelengths: 2418 us per pass against 2858 for the staged form with its two blocks
// (with one, two and four wavelengths per block and the next one's rows prefetched 2463, 2483, 2517).
template <int M, int PAD, bool CONJ, int HM, bool FULL>
__device__ __forceinline__ void col_split3_body(const ColArgs& a, int bx, int by, float2* tile, float2* tab) {
  using G = ColSplit3<M, PAD>;
  constexpr int N = M / PAD, TX = 8, NT = TX * G::L, NH = G::NH;
  const int tid = threadIdx.x;
  const int kx0 = bx * TX;
  const int w = by;
  const WlConst c = load_uniform(a.wl + a.w_begin + w);
  if ((kx0 < M / 2 ? kx0 : M - (kx0 + TX - 1)) > c.radius) return;  // as trim_evanescent

  // A and C: thread of column t % 8, row t / 8 + 64 r; B: lane of column t / 64.  The addresses are
  // formed where they are used (opaque_lane_row), or they alone would take ten of the 80 registers
  // that six wavefronts per SIMD leave.
  auto own_slots = [&](int t) { return tile + t % TX * G::REG + G::slot(0, 0) + t / TX + (t / TX >> 3); };
  constexpr int S1 = G::slot(1, 0), S8 = G::slot(0, 8);

  const uint64_t base = reinterpret_cast<uint64_t>(a.spec + static_cast<size_t>(w) * N * M);
  const uint64_t base_lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(base)));
  const uint64_t base_hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(base >> 32)));
  const auto rs = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>((base_hi << 32) | base_lo), 0, N * M * 8,
                                                    kBufferRsrcWord3);
  constexpr unsigned kNowhere = 0x80000000u;  // beyond every plane: loads give zero, stores drop
  float2 x[8], acc[8];
  {
    const int t = opaque_lane_row(tid), j = t / TX;
    const unsigned voff = static_cast<unsigned>((j * M + kx0 + t % TX) * 8);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int y = j + 64 * r;
      const unsigned off = (FULL || (y >= a.in_lo && y < a.in_hi)) ? voff : kNowhere;
      x[r] = buffer_load_c64(rs, off, 64 * r * M * 8);
    }
  }
  for (int i = tid; i < G::COUNT; i += NT) tab[i] = a.tw[i];
  static_for<0, NH>([&](auto hc) {
    constexpr int h = decltype(hc)::value;
    {
      float2 v[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) v[r] = x[r];
      if constexpr (h == 1) dft_odd<8>(v);
      else DFT<8, false, false>::run(v);
      float2* const own = own_slots(opaque_lane_row(tid));
#pragma unroll
      for (int k = 0; k < 8; ++k) own[k * S1] = v[k];
    }
    __syncthreads();
    {
      float2 f[8];
      const int t = opaque_lane_row(tid), lane = t & 63, k1 = t & 7, l8 = lane >> 3;
      float2* const freq = tile + (t >> 6) * G::REG + k1 * S1;
      float2* const fixed = freq + l8;       // (k1, l8 + 8 i): B1 and its inverse
      float2* const run = freq + l8 * S8;    // (k1, i + 8 l8): B2
#pragma unroll
      for (int i = 0; i < 8; ++i) f[i] = fixed[i * S8];
      dft8_table<false>(f, tab + h * 8 + k1, NH * 8);
#pragma unroll
      for (int i = 0; i < 8; ++i) fixed[i * S8] = f[i];
      wave_sync();
#pragma unroll
      for (int i = 0; i < 8; ++i) f[i] = run[i];
      dft8_table<false>(f, tab + G::OFF_B2 + h * 64 + lane, NH * 64);
      apply_transfer<M, PAD, CONJ, HM, h, 64, 8>(f, a, c, w, kx0 + (t >> 6), h, lane);
      DFT<8, true, false>::run(f);
#pragma unroll
      for (int i = 0; i < 8; ++i) run[i] = f[i];
      wave_sync();
#pragma unroll
      for (int i = 0; i < 8; ++i) f[i] = fixed[i * S8];
      dft8_table<true>(f, tab + G::OFF_R + l8, 8);
#pragma unroll
      for (int i = 0; i < 8; ++i) fixed[i * S8] = f[i];
    }
    __syncthreads();
    {
      float2 y[8];
      const int t = opaque_lane_row(tid), j = t / TX;
      const float2* const own = own_slots(t);
#pragma unroll
      for (int k = 0; k < 8; ++k) y[k] = own[k * S1];
      dft8_table<true>(y, tab + G::OFF_C + j, 64);
      if constexpr (h == 0) {
#pragma unroll
        for (int r = 0; r < 8; ++r) acc[r] = y[r];
      } else {  // the odd half turned by the conjugate of w_M^n
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          const float2 q = tab[G::OFF_W + j + 64 * r];
          acc[r] = make_float2(fmaf(q.y, y[r].y, fmaf(q.x, y[r].x, acc[r].x)),
                               fmaf(-q.y, y[r].x, fmaf(q.x, y[r].y, acc[r].y)));
        }
      }
    }
  });
  const int t = opaque_lane_row(tid), jv = t / TX;
  const unsigned voff = static_cast<unsigned>((jv * M + kx0 + t % TX) * 8);
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int row = jv + 64 * r;
    const unsigned off = (FULL || (row >= a.out_lo && row < a.out_hi)) ? voff : kNowhere;
    buffer_store_c64(rs, off, 64 * r * M * 8, acc[r]);
  }
}

// Frequencies of half h of a tile of halves of 800 points: the second phase, H and its inverse in place
template <int M, int PAD, bool CONJ, int HM, int h>
__device__ __forceinline__ void col800_freq(const ColArgs& a, const WlConst& c, int w, int kx0, float2* tile, int tid) {
  using G = ColSplit800<M, PAD>;
  constexpr int R1 = G::R1, R2 = G::R2;
  const int t = opaque_lane_row(tid), k1 = t % 32, cb = t / 32;
  if (k1 < R1) {
    float2* const freq = tile + cb * G::REG + G::slot(k1, 0);
    const float2* const tab = a.tw + h * 32 + k1;
    float2 f[R2];
    {
      float2 p[R2 / 4], even[R2 / 2], odd[R2 / 2];
#pragma unroll
      for (int e = 0; e < R2 / 4; ++e) p[e] = tab[e * G::NH * 32];
#pragma unroll
      for (int i = 0; i < R2; ++i) (i % 2 ? odd : even)[i / 2] = freq[i];
      dft_fused<R2 / 2, false>(even, p);
      dft_fused<R2 / 2, false>(odd, p);
      schedule_fence();  // the last level's factors take the registers of the others
#pragma unroll
      for (int k = 0; k < R2 / 4; ++k) p[k] = tab[(R2 / 4 + k) * G::NH * 32];
      dft_fused_join<R2, false>(even, odd, p, f);
    }
    apply_transfer<M, PAD, CONJ, HM, h, R1, R2>(f, a, c, w, kx0 + cb, h, k1);
    DFT<R2, true, false>::run(f);
#pragma unroll
    for (int i = 0; i < R2; ++i) freq[i] = f[i];
  }
}

// The last phase: row j's 25 values of one half from the tile
template <int M, int PAD>
__device__ __forceinline__ void col800_rows(const ColArgs& a, const float2* own, int j, float2* y) {
  using G = ColSplit800<M, PAD>;
  constexpr int R1 = G::R1;
#pragma unroll
  for (int k = 0; k < R1; ++k) y[k] = own[G::slot(k, 0)];
#pragma unroll
  for (int k = 1; k < R1; ++k) y[k] = cmulc(y[k], a.tw[G::OFF_C + (k - 1) * 32 + j]);
  schedule_fence();  // the factors of the odd half wait until the transform has let go of its own
  DFT<R1, true, false>::run(y);
  schedule_fence();
}

// The same for halves of 800 points (ColSplit800): eight columns on 256 threads.  Bound by vector issue and
// by the registers: 25 inputs, 25 sums and 32 frequencies per lane hold it to 12 wavefronts per CU, where
// the staged form ran 10 on twice the points; they issue in 93 % of the cycles (111 % with the 24
// wavefronts of the 512-point halves) and wait for 30 % of their time.  128 wavelengths of the glass
// design's discs, us per pass: staged, every frequency evaluated 1535; this form with two blocks per CU
// 1215, with the mirrored transfer function 1080, with three blocks 1012.
template <int M, int PAD, bool CONJ, int HM, bool FULL>
__device__ __forceinline__ void col_split800_body(const ColArgs& a, int bx, int by, float2* tile) {
  using G = ColSplit800<M, PAD>;
  constexpr int N = M / PAD, TX = 8, R1 = G::R1, R2 = G::R2, L = G::L;
  const int tid = threadIdx.x;
  const int kx0 = bx * TX;
  const int w = by;
  const WlConst c = load_uniform(a.wl + a.w_begin + w);
  if ((kx0 < M / 2 ? kx0 : M - (kx0 + TX - 1)) > c.radius) return;  // as trim_evanescent

  const uint64_t base = reinterpret_cast<uint64_t>(a.spec + static_cast<size_t>(w) * N * M);
  const uint64_t base_lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(base)));
  const uint64_t base_hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(base >> 32)));
  const auto rs = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>((base_hi << 32) | base_lo), 0, N * M * 8,
                                                    kBufferRsrcWord3);
  constexpr unsigned kNowhere = 0x80000000u;  // beyond every plane: loads give zero, stores drop
  float2 x[R1], acc[R1];
  {
    const int t = opaque_lane_row(tid), j = t / TX;
    const unsigned voff = static_cast<unsigned>((j * M + kx0 + t % TX) * 8);
#pragma unroll
    for (int r = 0; r < R1; ++r) {
      const int y = j + L * r;
      const unsigned off = (FULL || (y >= a.in_lo && y < a.in_hi)) ? voff : kNowhere;
      x[r] = buffer_load_c64(rs, off, L * r * M * 8);
    }
  }
  static_for<0, 2>([&](auto hc) {
    constexpr int h = decltype(hc)::value;
    {
      float2 v[R1];
#pragma unroll
      for (int r = 0; r < R1; ++r) v[r] = x[r];
      if constexpr (h == 1) dft_odd<R1>(v);
      else DFT<R1, false, false>::run(v);
      const int t = opaque_lane_row(tid);
      float2* const own = tile + t % TX * G::REG + t / TX;
#pragma unroll
      for (int k = 0; k < R1; ++k) own[G::slot(k, 0)] = v[k];
    }
    __syncthreads();
    col800_freq<M, PAD, CONJ, HM, h>(a, c, w, kx0, tile, tid);
    __syncthreads();
    {
      float2 y[R1];
      const int t = opaque_lane_row(tid), j = t / TX;
      col800_rows<M, PAD>(a, tile + t % TX * G::REG + j, j, y);
      if constexpr (h == 0) {
#pragma unroll
        for (int r = 0; r < R1; ++r) acc[r] = y[r];
      } else {  // the odd half turned by the conjugate of w_M^n
#pragma unroll
        for (int r = 0; r < R1; ++r) {
          const float2 q = a.tw[G::OFF_W + j + L * r];
          acc[r] = make_float2(fmaf(q.y, y[r].y, fmaf(q.x, y[r].x, acc[r].x)),
                               fmaf(-q.y, y[r].x, fmaf(q.x, y[r].y, acc[r].y)));
        }
      }
    }
  });
  const int t = opaque_lane_row(tid), jv = t / TX;
  const unsigned voff = static_cast<unsigned>((jv * M + kx0 + t % TX) * 8);
#pragma unroll
  for (int r = 0; r < R1; ++r) {
    const int row = jv + L * r;
    const unsigned off = (FULL || (row >= a.out_lo && row < a.out_hi)) ? voff : kNowhere;
    buffer_store_c64(rs, off, L * r * M * 8, acc[r]);
  }
}

// Launches of at most a block per CU: the halves on different wavefronts, which halves the chain that
// such a launch waits for; the sums are the same.  One wavelength, forward of two layers: 85.7 us with
// the halves in turn, 77.6 here (78.4 staged); from two wavelengths on the other form is faster.
template <int M, int PAD, bool CONJ, int HM, bool FULL>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) col800_few_kernel(ColArgs a) {
  using G = ColSplit800<M, PAD>;
  constexpr int N = M / PAD, TX = 8, R1 = G::R1, L = G::L, CUT = R1 / 2 + 1;
  __shared__ float2 tiles[G::NH * TX * G::REG];
  int bx, w;
  col_block_item(static_cast<int>(blockIdx.x + gridDim.x * blockIdx.y), static_cast<int>(gridDim.x * gridDim.y),
                 static_cast<int>(gridDim.x), bx, w);
  const int tid = threadIdx.x % 256, half = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / 256);
  const int kx0 = bx * TX, j = tid / TX;
  const WlConst c = load_uniform(a.wl + a.w_begin + w);
  if ((kx0 < M / 2 ? kx0 : M - (kx0 + TX - 1)) > c.radius) return;  // as trim_evanescent
  float2* const spec = a.spec + static_cast<size_t>(w) * N * M + kx0 + tid % TX;
  float2* const tile = tiles + half * TX * G::REG;
  float2* const own = tile + tid % TX * G::REG + j;  // slots of this thread alone in the row phases
  float2 v[R1];
#pragma unroll
  for (int r = 0; r < R1; ++r) {
    const int y = j + L * r;
    v[r] = (FULL || (y >= a.in_lo && y < a.in_hi)) ? spec[static_cast<size_t>(y) * M] : make_float2(0.f, 0.f);
  }
  if (half) dft_odd<R1>(v);
  else DFT<R1, false, false>::run(v);
#pragma unroll
  for (int k = 0; k < R1; ++k) own[G::slot(k, 0)] = v[k];
  __syncthreads();
  if (half) col800_freq<M, PAD, CONJ, HM, 1>(a, c, w, kx0, tile, tid);
  else col800_freq<M, PAD, CONJ, HM, 0>(a, c, w, kx0, tile, tid);
  __syncthreads();
  col800_rows<M, PAD>(a, own, j, v);
  // the even half's threads finish the first CUT rows, the odd half's the others
#pragma unroll
  for (int r = 0; r < R1; ++r)
    if ((r < CUT) == (half == 1)) own[G::slot(r, 0)] = v[r];
  __syncthreads();
  const float2* const other = tiles + (1 - half) * TX * G::REG + tid % TX * G::REG + j;
#pragma unroll
  for (int r = 0; r < R1; ++r) {
    const int row = j + L * r;
    if ((r < CUT) == (half == 1)) continue;
    const float2 o = other[G::slot(r, 0)], q = a.tw[G::OFF_W + row];
    const float2 even = half ? o : v[r], odd = half ? v[r] : o;
    if (FULL || (row >= a.out_lo && row < a.out_hi))
      spec[static_cast<size_t>(row) * M] = make_float2(fmaf(q.y, odd.y, fmaf(q.x, odd.x, even.x)),
                                                       fmaf(-q.y, odd.x, fmaf(q.x, odd.y, even.y)));
  }
}

// Shape of the column kernels: the split transforms where the length has them (radix plan 0),
// else the staged form.
template <int M, int PAD, int TX, int V>
struct ColShape {
  static constexpr bool SPLIT800 = V == 0 && ColSplit800<M, PAD>::BUILT;  // TX = 8
  static constexpr bool SPLIT3 = V == 0 && ColSplit3<M, PAD>::BUILT;      // TX = 8
  static constexpr bool SPLIT = V == 0 && ColSplit<M, PAD>::BUILT;
  static constexpr int THREADS = SPLIT800  ? TX * ColSplit800<M, PAD>::L
                                 : SPLIT3 ? TX * ColSplit3<M, PAD>::L
                                 : SPLIT  ? ColSplit<M, PAD>::threads(TX)
                                          : TX * Geo<M>::P;
  static constexpr int SLOTS = SPLIT800  ? TX * ColSplit800<M, PAD>::REG
                               : SPLIT3 ? TX * ColSplit3<M, PAD>::REG
                               : SPLIT  ? PAD * TX * ColSplit<M, PAD>::region(TX)
                                        : TX * Geo<M>::COL_REGION;
  static constexpr int TABLE = SPLIT800  ? 1
                               : SPLIT3 ? ColSplit3<M, PAD>::COUNT
                               : SPLIT  ? ColSplit<M, PAD>::COUNT
                                        : twiddle_count<M, V>();
  // wavefronts per SIMD the registers are held to: three blocks of eight wavefronts per CU for the
  // halves of 512 points; three of four for those of 800, two where each frequency evaluates a
  // transfer function of its own (60 bytes of spills at three mirrored, 480 unmirrored); else four
  static constexpr int waves(int hm) { return SPLIT800 ? (hm == kHMirror || hm == kHTable ? 3 : 2) : SPLIT3 ? 6 : 4; }
};

template <int M, int PAD, bool CONJ, int TX, int HM, bool FULL, int V>
__device__ __forceinline__ void col_any_body(const ColArgs& a, int bx, int by, float2* tile, float2* tw) {
  if constexpr (ColShape<M, PAD, TX, V>::SPLIT800) col_split800_body<M, PAD, CONJ, HM, FULL>(a, bx, by, tile);
  else if constexpr (ColShape<M, PAD, TX, V>::SPLIT3) col_split3_body<M, PAD, CONJ, HM, FULL>(a, bx, by, tile, tw);
  else if constexpr (ColShape<M, PAD, TX, V>::SPLIT) col_split_body<M, PAD, CONJ, TX, HM, FULL>(a, bx, by, tile, tw);
  else col_body<M, PAD, CONJ, TX, HM, FULL, V>(a, bx, by, tile, tw);
}

template <int M, int PAD, bool CONJ, int TX, int HM, bool FULL, int V = 0>
__global__ void __launch_bounds__((ColShape<M, PAD, TX, V>::THREADS)) __attribute__((amdgpu_waves_per_eu((ColShape<M, PAD, TX, V>::waves(HM)))))
col_kernel(ColArgs a) {
  __shared__ float2 tile[ColShape<M, PAD, TX, V>::SLOTS];
  __shared__ float2 tw[ColShape<M, PAD, TX, V>::TABLE];
  int bx, by;
  col_block_item(static_cast<int>(blockIdx.x + gridDim.x * blockIdx.y), static_cast<int>(gridDim.x * gridDim.y),
                 static_cast<int>(gridDim.x), bx, by);
  col_any_body<M, PAD, CONJ, TX, HM, FULL, V>(a, bx, by, tile, tw);
}

// One launch of a column pass for several designs of the same transform length (see
// row_group_kernel); every task starts at a multiple of 16 blocks.
template <int M, int PAD, bool CONJ, int TX, int HM, bool FULL>
__global__ void __launch_bounds__((ColShape<M, PAD, TX, 0>::THREADS)) __attribute__((amdgpu_waves_per_eu((ColShape<M, PAD, TX, 0>::waves(HM)))))
col_group_kernel(GroupArgs g) {
  __shared__ float2 tile[ColShape<M, PAD, TX, 0>::SLOTS];
  __shared__ float2 tw[ColShape<M, PAD, TX, 0>::TABLE];
  const int ti = group_task(g, blockIdx.x);
  const ColTask t = load_uniform(static_cast<const ColTask*>(g.tasks) + ti);
  const int local = static_cast<int>(blockIdx.x) - g.block0[ti];
  if (local >= t.nblocks) return;
  const ColArgs a = t.a;
  int bx, by;
  col_block_item(local, t.nblocks, t.gx, bx, by);
  col_any_body<M, PAD, CONJ, TX, HM, FULL, 0>(a, bx, by, tile, tw);
}

// H / M^2 of one gap for every wavelength on the quarter plane |kx|, |ky| <= M/2 (H depends on
// kx^2 + ky^2 only); block (|kx|, w), threads over |ky|.
template <int M>
__global__ void __launch_bounds__(256) transfer_table_kernel(const WlConst* __restrict__ wl, double zrev,
                                                             float2* __restrict__ out) {
  constexpr int HS = M / 2 + 1;
  const int kx = blockIdx.x;
  const int w = blockIdx.y;
  const double base = wl[w].q0 - static_cast<double>(kx * kx);
  float2* row = out + (static_cast<size_t>(w) * HS + kx) * HS;
  for (int ky = threadIdx.x; ky < HS; ky += blockDim.x) row[ky] = transfer<M, false>(zrev, base, ky);
}

// ------------------------------------------------------------------------------------------
// Column pass as two complex matrix products on the FP32 matrix cores (v_mfma_f32_16x16x4_f32):
//   Z = F S            F[ky][y] = exp(-2 pi i ky y / M)  (M x N, shared by every wavelength)
//   Z <- H . Z / M^2   (transfer function on the fly, as in the transform kernels)
//   Out = F^H Z        (N x M, keeps the aperture rows)
// for a tile of 16 columns of one wavelength.  S and Z live in LDS as separate real and
// imaginary planes; the DFT matrix is read from a table built on the host in double
// precision: FT[y][ky] (step 1, lanes read 16 consecutive ky) and F[ky][y] (step 3).
// Operand layout of the 16x16x4 instruction: lane l holds A[l%16][l/16], B[l/16][l%16] and
// D[4(l/16)+r][l%16], r = 0..3.
// ------------------------------------------------------------------------------------------
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kGemmTile = 16;
// threads per block: the LDS tiles of long transforms allow one block per CU, so those get
// eight wavefronts to keep two per SIMD
constexpr int gemm_threads(int M) { return M >= 256 ? 512 : 256; }

template <int M, int PAD, bool CONJ>
__global__ void __launch_bounds__(gemm_threads(M)) colgemm_kernel(ColArgs a, const float2* __restrict__ dft) {
  constexpr int N = M / PAD;
  constexpr int TN = kGemmTile;
  constexpr int kGemmThreads = gemm_threads(M);
  constexpr int WAVES = kGemmThreads / 64;
  __shared__ float sr[N * TN], si[N * TN];
  __shared__ float zr[M * TN], zi[M * TN];
  const float2* __restrict__ FT = dft;           // [N][M]
  const float2* __restrict__ F = dft + M * N;    // [M][N]

  const int kx0 = blockIdx.x * TN;
  float2* spec = a.spec + static_cast<size_t>(blockIdx.y) * N * M;
  const WlConst c = a.wl[a.w_begin + blockIdx.y];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;

  // stage rows [in_lo, in_hi) of the 16 columns (zeros elsewhere)
  for (int i = tid; i < N * TN; i += kGemmThreads) {
    const int y = i / TN, cc = i % TN;
    float2 v = make_float2(0.f, 0.f);
    if (y >= a.in_lo && y < a.in_hi) v = spec[static_cast<size_t>(y) * M + kx0 + cc];
    sr[i] = v.x;
    si[i] = v.y;
  }
  __syncthreads();

  // step 1: Z = F S, K = N.  A wave takes its row tiles of ky two at a time, so four
  // accumulator chains are in flight on the matrix core and the S operand is read once per
  // k step for both.
  {
    const int kx = kx0 + lr;
    const int kxs = kx < M / 2 ? kx : kx - M;
    const double base = c.q0 - static_cast<double>(kxs * kxs);
    for (int t0 = wave; t0 < M / 16; t0 += 2 * WAVES) {
      const int t1 = t0 + WAVES;
      const bool two = t1 < M / 16;
      v4f re0 = {0.f, 0.f, 0.f, 0.f}, im0 = re0, re1 = re0, im1 = re0;
#pragma unroll 4
      for (int k0 = 0; k0 < N; k0 += 4) {
        const float br = sr[(k0 + lk) * TN + lr], bi = si[(k0 + lk) * TN + lr];
        const float2 f0 = FT[(k0 + lk) * M + t0 * 16 + lr];
        re0 = __builtin_amdgcn_mfma_f32_16x16x4f32(f0.x, br, re0, 0, 0, 0);
        re0 = __builtin_amdgcn_mfma_f32_16x16x4f32(-f0.y, bi, re0, 0, 0, 0);
        im0 = __builtin_amdgcn_mfma_f32_16x16x4f32(f0.x, bi, im0, 0, 0, 0);
        im0 = __builtin_amdgcn_mfma_f32_16x16x4f32(f0.y, br, im0, 0, 0, 0);
        if (two) {
          const float2 f1 = FT[(k0 + lk) * M + t1 * 16 + lr];
          re1 = __builtin_amdgcn_mfma_f32_16x16x4f32(f1.x, br, re1, 0, 0, 0);
          re1 = __builtin_amdgcn_mfma_f32_16x16x4f32(-f1.y, bi, re1, 0, 0, 0);
          im1 = __builtin_amdgcn_mfma_f32_16x16x4f32(f1.x, bi, im1, 0, 0, 0);
          im1 = __builtin_amdgcn_mfma_f32_16x16x4f32(f1.y, br, im1, 0, 0, 0);
        }
      }
      // H at (kx0 + lr, ky0 + 4 lk + r)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int ky = t0 * 16 + 4 * lk + r;
        float2 z = cmul(make_float2(re0[r], im0[r]), transfer<M, CONJ>(a.zrev, base, ky));
        zr[ky * TN + lr] = z.x;
        zi[ky * TN + lr] = z.y;
        if (two) {
          ky = t1 * 16 + 4 * lk + r;
          z = cmul(make_float2(re1[r], im1[r]), transfer<M, CONJ>(a.zrev, base, ky));
          zr[ky * TN + lr] = z.x;
          zi[ky * TN + lr] = z.y;
        }
      }
    }
  }
  __syncthreads();

  // step 3: Out = F^H Z for the kept rows, K = M, two row tiles of y at a time
  for (int t0 = wave; t0 < N / 16; t0 += 2 * WAVES) {
    const int t1 = t0 + WAVES;
    const bool use0 = t0 * 16 < a.out_hi && t0 * 16 + 16 > a.out_lo;
    const bool use1 = t1 < N / 16 && t1 * 16 < a.out_hi && t1 * 16 + 16 > a.out_lo;
    if (!use0 && !use1) continue;
    v4f re0 = {0.f, 0.f, 0.f, 0.f}, im0 = re0, re1 = re0, im1 = re0;
#pragma unroll 4
    for (int k0 = 0; k0 < M; k0 += 4) {
      const float br = zr[(k0 + lk) * TN + lr], bi = zi[(k0 + lk) * TN + lr];
      // A[y][ky] = conj(F[ky][y]): lane (lr, lk) needs y = y0 + lr, ky = k0 + lk
      if (use0) {
        const float2 f0 = F[(k0 + lk) * N + t0 * 16 + lr];
        re0 = __builtin_amdgcn_mfma_f32_16x16x4f32(f0.x, br, re0, 0, 0, 0);
        re0 = __builtin_amdgcn_mfma_f32_16x16x4f32(f0.y, bi, re0, 0, 0, 0);
        im0 = __builtin_amdgcn_mfma_f32_16x16x4f32(f0.x, bi, im0, 0, 0, 0);
        im0 = __builtin_amdgcn_mfma_f32_16x16x4f32(-f0.y, br, im0, 0, 0, 0);
      }
      if (use1) {
        const float2 f1 = F[(k0 + lk) * N + t1 * 16 + lr];
        re1 = __builtin_amdgcn_mfma_f32_16x16x4f32(f1.x, br, re1, 0, 0, 0);
        re1 = __builtin_amdgcn_mfma_f32_16x16x4f32(f1.y, bi, re1, 0, 0, 0);
        im1 = __builtin_amdgcn_mfma_f32_16x16x4f32(f1.x, bi, im1, 0, 0, 0);
        im1 = __builtin_amdgcn_mfma_f32_16x16x4f32(-f1.y, br, im1, 0, 0, 0);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int y = t0 * 16 + 4 * lk + r;
      if (use0 && y >= a.out_lo && y < a.out_hi)
        spec[static_cast<size_t>(y) * M + kx0 + lr] = make_float2(re0[r], im0[r]);
      y = t1 * 16 + 4 * lk + r;
      if (use1 && y >= a.out_lo && y < a.out_hi)
        spec[static_cast<size_t>(y) * M + kx0 + lr] = make_float2(re1[r], im1[r]);
    }
  }
}

// ------------------------------------------------------------------------------------------
// LDS-resident path for short transforms.  A block owns one wavelength (the adjoint: the wavelengths of
// one gradient slot, in turn).  Its N aperture rows live in LDS with a row stride equal to a row
// transform's exchange region, so every row transforms in place; the columns run the split transforms in
// place too (lds_columns).  Every step is the one the multi-kernel path takes (same transforms,
// transmission, transfer function, products, and the same order of the gradient sums), so the results
// are the same bits.
// ------------------------------------------------------------------------------------------
template <int M, int PAD>
struct LdsGeo {
  static constexpr int N = M / PAD;
  static constexpr int P = Geo<M>::P;
  static constexpr int RS = Geo<M>::ROW_REGION;               // row stride of the plane
  static constexpr int RB = kLdsThreads / P;                  // rows transformed at once
  static constexpr int TABLE = ColSplit<M, PAD>::COUNT > 0 ? ColSplit<M, PAD>::COUNT : 1;
  static constexpr long long LDS_BYTES =
      8LL * (static_cast<long long>(N) * RS + twiddle_count<M>() + TABLE);
  static constexpr bool FITS = ColSplit<M, PAD>::BUILT && LDS_BYTES <= 160 * 1024 && (PAD == 2 || M <= 96);
};

// forward rows of one layer: FIRST = input field times t_0, else inverse row transform of the
// plane row, crop, times t_layer; checkpoint; zero-padded forward row transform in place
template <int M, int PAD, bool FIRST>
__device__ __forceinline__ void lds_rows_forward(const LdsArgs& a, const WlConst& c, int w, int layer,
                                                 float2* plane, const float2* tw) {
  using G = LdsGeo<M, PAD>;
  constexpr int E = Geo<M>::E, P = G::P, N = G::N, EN = E / PAD;
  constexpr bool HALF = (PAD == 2);
  const int g = threadIdx.x / P, j0 = threadIdx.x % P;
  const size_t nn = static_cast<size_t>(N) * N;
  for (int y = g; y < N; y += G::RB) {
    float2* row = plane + y * G::RS;
    const float* hrow = a.h + (static_cast<size_t>(layer) * N + y) * N;
    float2 reg[E];
    if constexpr (FIRST) {
#pragma unroll
      for (int t = 0; t < EN; ++t) {
        const float2 u = a.u_in ? a.u_in[static_cast<size_t>(y) * N + j0 + P * t] : make_float2(1.f, 0.f);
        reg[t] = cmul(u, transmission(hrow[j0 + P * t], c));
      }
    } else {
#pragma unroll
      for (int t = 0; t < E; ++t) reg[t] = row[j0 + P * t];
      fft<M, true, false>(reg, row, j0, tw);
#pragma unroll
      for (int t = 0; t < EN; ++t) reg[t] = cmul(reg[t], transmission(hrow[j0 + P * t], c));
    }
    float2* ck = a.ckpt + (static_cast<size_t>(layer) * a.W + w) * nn + static_cast<size_t>(y) * N;
#pragma unroll
    for (int t = 0; t < EN; ++t) ck[j0 + P * t] = reg[t];
    fft<M, false, HALF>(reg, row, j0, tw);
#pragma unroll
    for (int t = 0; t < E; ++t) row[j0 + P * t] = reg[t];
  }
}

// column transforms of one gap: rows [in_lo, in_hi) in, H or conj(H), rows [0, N) back.  The same
// phases as the column kernels' (col_split_body), in place: a column's GL consecutive lanes lie in
// one wavefront, slot (k1, j) is plane row j + R2 k1, which is the row thread's own, and the halves
// follow each other.
template <int M, int PAD, bool CONJ>
__device__ __forceinline__ void lds_columns(const WlConst& c, const ColArgs& ca, int in_lo, int in_hi,
                                            float2* plane, const float2* tab, int tid) {
  using G = LdsGeo<M, PAD>;
  using S = ColSplit<M, PAD>;
  constexpr int R1 = S::R1, R2 = S::R2, L = S::L, RS = G::RS;
  constexpr int GL = pow2_at_least(L > S::GP ? L : S::GP);
  constexpr int CB = kLdsThreads / GL;
  const int lane = tid % GL;
  for (int kx = tid / GL; kx < M; kx += CB) {
    float2* col = plane + kx;
    const bool rows = lane < L, freq = lane < R1;
    float2 x[R1], b[S::NH][R1];
    if (rows) {
#pragma unroll
      for (int r = 0; r < R1; ++r) {
        const int y = lane + L * r;
        x[r] = (y >= in_lo && y < in_hi) ? col[y * RS] : make_float2(0.f, 0.f);
      }
    }
    static_for<0, S::NH>([&](auto hc) {
      constexpr int h = decltype(hc)::value;
      if (rows) {
        float2 v[R1];
#pragma unroll
        for (int r = 0; r < R1; ++r) v[r] = x[r];
        col_rows_forward<M, PAD, h == 1>(v);
#pragma unroll
        for (int k = 0; k < R1; ++k) col[(lane + L * k) * RS] = v[k];
      }
      wave_sync();
      if (freq) {
        float2 v[R2];
#pragma unroll
        for (int i = 0; i < R2; ++i) v[i] = col[(i + L * lane) * RS];
        col_freq_forward<M, PAD>(v, tab, h, lane);
        apply_transfer<M, PAD, CONJ, kHEval, h, R1, R2>(v, ca, c, 0, kx, h, lane);
        col_freq_inverse<M, PAD>(v);
#pragma unroll
        for (int i = 0; i < R2; ++i) col[(i + L * lane) * RS] = v[i];
      }
      wave_sync();
      if (rows) {
#pragma unroll
        for (int k = 0; k < R1; ++k) b[h][k] = col[(lane + L * k) * RS];
      }
      wave_sync();
    });
    if (rows) {
      if constexpr (S::NH == 2) {
#pragma unroll
        for (int parity = 0; parity < 2; ++parity) {
          float2 y[S::RC];
          col_rows_inverse2<M, PAD>(y, tab, lane, parity, [&](int h, int k) { return b[h][k]; });
#pragma unroll
          for (int r = 0; r < S::RC; ++r) col[(lane + L * (2 * r + parity)) * RS] = y[r];
        }
      } else {
        col_rows_inverse<M, PAD>(b[0], tab, lane);
#pragma unroll
        for (int r = 0; r < R1; ++r) col[(lane + L * r) * RS] = b[0][r];
      }
    }
  }
}

template <int M, int PAD>
__global__ void __launch_bounds__(kLdsThreads) lds_forward_kernel(LdsArgs a) {
  using G = LdsGeo<M, PAD>;
  constexpr int E = Geo<M>::E, P = G::P, N = G::N, EN = E / PAD;
  __shared__ float2 plane[N * G::RS];
  __shared__ float2 tw[twiddle_count<M>()];
  __shared__ float2 tab[G::TABLE];
  stage_twiddles<M>(tw, a.tw, threadIdx.x, kLdsThreads);
  for (int i = threadIdx.x; i < G::TABLE; i += kLdsThreads) tab[i] = a.col_tab[i];
  __syncthreads();
  ColArgs gap{};  // what the transfer function of a column needs
  const int w = blockIdx.x;
  const WlConst c = a.wl[w];
  lds_rows_forward<M, PAD, true>(a, c, w, 0, plane, tw);
  __syncthreads();
  for (int l = 0; l < a.K; ++l) {
    gap.zrev = a.zrev[l];
    lds_columns<M, PAD, false>(c, gap, 0, N, plane, tab, threadIdx.x);
    __syncthreads();
    if (l + 1 < a.K) {
      lds_rows_forward<M, PAD, false>(a, c, w, l + 1, plane, tw);
      __syncthreads();
    }
  }
  // last inverse row transforms on the window rows: output field, and its intensity in bins (the
  // window rows go back in place of their spectra)
  const int F = a.fov, x0 = (N - F) / 2, T = F / a.bin;
  const int g = threadIdx.x / P, j0 = threadIdx.x % P;
  for (int y = x0 + g; y < x0 + F; y += G::RB) {
    float2* row = plane + y * G::RS;
    float2 reg[E];
#pragma unroll
    for (int t = 0; t < E; ++t) reg[t] = row[j0 + P * t];
    fft<M, true, false>(reg, row, j0, tw);
    float2* dst = a.ofov + static_cast<size_t>(w) * F * F + static_cast<size_t>(y - x0) * F;
#pragma unroll
    for (int t = 0; t < EN; ++t) {
      const int x = j0 + P * t;
      if (x >= x0 && x < x0 + F) {
        dst[x - x0] = reg[t];
        row[x] = reg[t];
      }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < T * T; i += kLdsThreads)
    a.intensity[static_cast<size_t>(w) * T * T + i] =
        bin_sum(plane + (x0 + i / T * a.bin) * G::RS + x0 + i % T * a.bin, G::RS, a.bin);
}

// RUNS: a gradient slot holds several wavelengths, which a block takes in turn and adds in the order of
// the row passes (else w_per_block is 1).  Four wavefronts per SIMD where the LDS has room for two blocks.
template <int M, int PAD, bool RUNS>
__global__ void __launch_bounds__(kLdsThreads)
__attribute__((amdgpu_waves_per_eu(2 * LdsGeo<M, PAD>::LDS_BYTES <= 160 * 1024 ? 4 : 2)))
lds_adjoint_kernel(LdsArgs a) {
  using G = LdsGeo<M, PAD>;
  constexpr int E = Geo<M>::E, P = G::P, N = G::N, EN = E / PAD;
  constexpr bool HALF = (PAD == 2);
  __shared__ float2 plane[N * G::RS];
  __shared__ float2 tw[twiddle_count<M>()];
  __shared__ float2 tab[G::TABLE];
  stage_twiddles<M>(tw, a.tw, threadIdx.x, kLdsThreads);
  for (int i = threadIdx.x; i < G::TABLE; i += kLdsThreads) tab[i] = a.col_tab[i];
  __syncthreads();
  ColArgs gap{};  // what the transfer function of a column needs
  const int F = a.fov, b = a.bin, T = F / b, x0 = (N - F) / 2;
  const size_t nn = static_cast<size_t>(N) * N;
  const int wb = blockIdx.x * (RUNS ? a.w_per_block : 1), we = RUNS ? min(wb + a.w_per_block, a.W) : wb + 1;
  int w = wb;
  do {
    // opaque per wavelength (as in opaque_lane_row): what is the same for each of them would otherwise
    // stay live across the loop (128 points: 166 registers against 116)
    const int tid = RUNS ? opaque_lane_row(threadIdx.x) & (kLdsThreads - 1) : threadIdx.x;
    const int g = tid / P, j0 = tid % P;
    const WlConst c = a.wl[w];
    // seed 2 (dL/dI) o on the window rows, forward row transform
    for (int y = x0 + g; y < x0 + F; y += G::RB) {
      float2* row = plane + y * G::RS;
      const float2* o = a.ofov + static_cast<size_t>(w) * F * F + static_cast<size_t>(y - x0) * F;
      const float* d = a.dl_di + static_cast<size_t>(w) * T * T + static_cast<size_t>((y - x0) / b) * T;
      float2 reg[E];
#pragma unroll
      for (int t = 0; t < EN; ++t) {
        const int x = j0 + P * t;
        if (x >= x0 && x < x0 + F) {
          const float s = 2.0f * kAdjointScale * d[(x - x0) / b];
          reg[t] = cscale(o[x - x0], s);
        } else {
          reg[t] = make_float2(0.f, 0.f);
        }
      }
      fft<M, false, HALF>(reg, row, j0, tw);
#pragma unroll
      for (int t = 0; t < E; ++t) row[j0 + P * t] = reg[t];
    }
    __syncthreads();
    const float ct = c.ct, ca = static_cast<float>(c.ca) / kAdjointScale;
    for (int l = a.K - 1; l >= 0; --l) {
      gap.zrev = a.zrev[l];
      lds_columns<M, PAD, true>(c, gap, l == a.K - 1 ? x0 : 0, l == a.K - 1 ? x0 + F : N, plane, tab, tid);
      __syncthreads();
      for (int y = g; y < N; y += G::RB) {
        float2* row = plane + y * G::RS;
        const float* hrow = a.h + (static_cast<size_t>(l) * N + y) * N;
        const float2* ck = a.ckpt + (static_cast<size_t>(l) * a.W + w) * nn + static_cast<size_t>(y) * N;
        float* dst = a.dh_part + (static_cast<size_t>(blockIdx.x) * a.K + l) * nn + static_cast<size_t>(y) * N;
        float2 reg[E];
#pragma unroll
        for (int t = 0; t < E; ++t) reg[t] = row[j0 + P * t];
        fft<M, true, false>(reg, row, j0, tw);
#pragma unroll
        for (int t = 0; t < EN; ++t) {
          const float2 gv = reg[t];
          const float2 v = ck[j0 + P * t];
          // conj(g) v; acc += -ct Im - ca Re
          const float re = fmaf(gv.x, v.x, gv.y * v.y);
          const float im = fmaf(gv.x, v.y, -(gv.y * v.x));
          dst[j0 + P * t] = fmaf(-ct, im, fmaf(-ca, re, RUNS && w > wb ? dst[j0 + P * t] : 0.f));
          if (l > 0) reg[t] = cmulc(gv, transmission(hrow[j0 + P * t], c));
        }
        if (l > 0) {
          fft<M, false, HALF>(reg, row, j0, tw);
#pragma unroll
          for (int t = 0; t < E; ++t) row[j0 + P * t] = reg[t];
        }
      }
      __syncthreads();
    }
  } while (RUNS && ++w < we);
}

}  // namespace dpx
