// HIP kernels for gfx950 that do not depend on the transform length (intensity binning, loss,
// gradient reduction), host-side tables (stage twiddles, DFT matrices), and the dispatch of
// the per-length pass launchers (dpx_pass.hip, one translation unit per length).
#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "dpx_internal.hpp"
#include "fft.hpp"

namespace dpx {

// ------------------------------------------------------------------------------------------
// Small kernels
// ------------------------------------------------------------------------------------------

__global__ void bin_intensity_kernel(const float2* __restrict__ ofov, float* __restrict__ out,
                                     int w_count, int fov, int bin) {
  bin_intensity_body(ofov, out, w_count, fov, bin, static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x);
}

// grouped: task = one design's window fields -> its intensities in the packed output
__global__ void bin_group_kernel(GroupArgs g, float* __restrict__ out) {
  const int ti = group_task(g, blockIdx.x);
  const BinTask& t = static_cast<const BinTask*>(g.tasks)[ti];
  const int local = static_cast<int>(blockIdx.x) - g.block0[ti];
  bin_intensity_body(t.ofov, out + t.img_off, t.w_count, t.fov, t.bin,
                     static_cast<size_t>(local) * blockDim.x + threadIdx.x);
}

constexpr int kLossThreads = 256;
constexpr int kLossThreadsLarge = 1024;  // large_image
constexpr int kLossCache = 16;           // most pixels a thread keeps in registers

// v plus its neighbour's value under the DPP control CTRL (0 where there is none)
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_neighbour(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(b), CTRL, ROWS, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(b >> 32), CTRL, ROWS, 0xf, true);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}

// Lane 63 ends with the combination of the wavefront's 64 values, in a fixed order: rows of 16 by
// shifts, then the rows' last lanes broadcast into the rows behind.  For sums, and maxima of
// non-negative values (missing neighbours count as zero).
template <typename Op>
__device__ __forceinline__ double wave_combine(double v, Op op) {
  v = op(v, dpp_neighbour<0x111, 0xf>(v));  // row_shr 1, 2, 4, 8
  v = op(v, dpp_neighbour<0x112, 0xf>(v));
  v = op(v, dpp_neighbour<0x114, 0xf>(v));
  v = op(v, dpp_neighbour<0x118, 0xf>(v));
  v = op(v, dpp_neighbour<0x142, 0xa>(v));  // row_bcast 15 into rows 1 and 3
  v = op(v, dpp_neighbour<0x143, 0xc>(v));  // row_bcast 31 into rows 2 and 3
  return v;
}

// Combination over the block, in every thread; sh: THREADS / 64 doubles of this call's own.
template <int THREADS, typename Op>
__device__ __forceinline__ void block_combine_begin(double v, double* sh, Op op) {
  v = wave_combine(v, op);
  if ((threadIdx.x & 63) == 63) sh[threadIdx.x >> 6] = v;
}
template <int THREADS, typename Op>
__device__ __forceinline__ double block_combine_end(const double* sh, Op op) {
  double r = sh[0];
#pragma unroll
  for (int k = 1; k < THREADS / 64; ++k) r = op(r, sh[k]);
  return r;
}
struct Plus {
  __device__ __forceinline__ double operator()(double a, double b) const { return a + b; }
};
struct Max {
  __device__ __forceinline__ double operator()(double a, double b) const { return fmax(a, b); }
};

// The pixels of one wavelength's image and target, walked several times: from CACHE registers where a
// thread has no more of them, else (CACHE = 0) from memory.
template <int THREADS, int CACHE>
struct Pixels {
  const float* __restrict__ I;
  const float* __restrict__ tau;
  int P;
  float iv[CACHE > 0 ? CACHE : 1], tv[CACHE > 0 ? CACHE : 1];
  __device__ __forceinline__ Pixels(const float* I_, const float* tau_, int P_) : I(I_), tau(tau_), P(P_) {
    if constexpr (CACHE > 0) {
#pragma unroll
      for (int k = 0; k < CACHE; ++k) {
        const int p = threadIdx.x + k * THREADS;
        iv[k] = p < P ? I[p] : 0.f;
        tv[k] = p < P ? tau[p] : 0.f;
      }
    }
  }
  template <typename F>
  __device__ __forceinline__ void each(F&& f) const {
    if constexpr (CACHE > 0) {
#pragma unroll
      for (int k = 0; k < CACHE; ++k)
        if (threadIdx.x + k * THREADS < P) f(static_cast<int>(threadIdx.x + k * THREADS), iv[k], tv[k]);
    } else {
#pragma unroll 4
      for (int p = threadIdx.x; p < P; p += THREADS) f(p, I[p], tau[p]);
    }
  }
};

// One block per wavelength w: sums in double in a fixed order (bitwise reproducible).  Bound by
// latency: each image is read once into registers and the two rounds of sums cost one block barrier
// each (a tree of barriers and three walks over memory took 7 us at 6 images of 32 x 32 and 27 us
// at 1024 of 64 x 64).
template <int THREADS, int CACHE>
__device__ __forceinline__ void loss_image(const float* __restrict__ Iw, const float* __restrict__ tw,
                                           float* __restrict__ gw, double* __restrict__ out, int W, int P, double* sh) {
  constexpr int WAVES = THREADS / 64;
  const Pixels<THREADS, CACHE> px(Iw, tw, P);
  double si = 0.0, st = 0.0;
  px.each([&](int, float i, float t) {
    si += i;
    st += t;
  });
  block_combine_begin<THREADS>(si, sh, Plus{});
  block_combine_begin<THREADS>(st, sh + WAVES, Plus{});
  __syncthreads();
  const double S = block_combine_end<THREADS>(sh, Plus{}), St = block_combine_end<THREADS>(sh + WAVES, Plus{});
  const double rS = S > 0.0 ? 1.0 / S : 0.0;
  const double rSt = St > 0.0 ? 1.0 / St : 0.0;
  double sd2 = 0.0, sdi = 0.0;
  px.each([&](int, float i, float t) {
    const double ih = i * rS;
    const double d = ih - t * rSt;
    sd2 += d * d;
    sdi += d * ih;
  });
  block_combine_begin<THREADS>(sd2, sh + 2 * WAVES, Plus{});
  block_combine_begin<THREADS>(sdi, sh + 3 * WAVES, Plus{});
  __syncthreads();
  const double D2 = block_combine_end<THREADS>(sh + 2 * WAVES, Plus{});
  const double inner = block_combine_end<THREADS>(sh + 3 * WAVES, Plus{});
  if (threadIdx.x == 0) *out = D2 / P;
  if (gw) {
    const double k = 2.0 * rS / (static_cast<double>(W) * P);
    px.each([&](int p, float i, float t) {
      const double d = i * rS - t * rSt;
      gw[p] = static_cast<float>(k * (d - inner));
    });
  }
}

template <int THREADS>
__device__ __forceinline__ void loss_body(const float* __restrict__ I, const float* __restrict__ tau,
                                          float* __restrict__ dl_di, double* __restrict__ per_wl,
                                          int W, int T, int w, double* sh) {
  const int P = T * T;
  const size_t o = static_cast<size_t>(w) * P;
  float* gw = dl_di ? dl_di + o : nullptr;
  if constexpr (THREADS == kLossThreads) {
    // short walks over few pixels: 4096 images of 16 x 16 take 10 us with the loss of one pixel per
    // thread, 18.7 where each thread steps over fifteen that are not there
    if (P <= THREADS) return loss_image<THREADS, 1>(I + o, tau + o, gw, per_wl + w, W, P, sh);
    if (P <= 4 * THREADS) return loss_image<THREADS, 4>(I + o, tau + o, gw, per_wl + w, W, P, sh);
  }
  if (P <= kLossCache * THREADS) loss_image<THREADS, kLossCache>(I + o, tau + o, gw, per_wl + w, W, P, sh);
  else loss_image<THREADS, 0>(I + o, tau + o, gw, per_wl + w, W, P, sh);
}

template <int THREADS>
__device__ __forceinline__ void loss_sum_body(const double* __restrict__ per_wl, double* __restrict__ loss,
                                              int W, double* sh) {
  double s = 0.0;
#pragma unroll 4
  for (int w = threadIdx.x; w < W; w += THREADS) s += per_wl[w];
  block_combine_begin<THREADS>(s, sh, Plus{});
  __syncthreads();
  if (threadIdx.x == 0) *loss = block_combine_end<THREADS>(sh, Plus{}) / W;
}

// arrived: null, or the design's count of finished blocks; then the block that finishes last also
// sums the wavelengths' losses, which saves the launch that would.  The count wraps to zero by itself
// after W blocks, so that calls which overlap on several streams leave it at zero too: every call
// adds W to a count modulo W.
template <int THREADS>
__global__ void __launch_bounds__(THREADS)
loss_kernel(const float* __restrict__ I, const float* __restrict__ tau, float* __restrict__ dl_di,
            double* __restrict__ per_wl, int W, int T, unsigned* __restrict__ arrived, double* __restrict__ loss) {
  __shared__ double sh[4 * (THREADS / 64)];
  __shared__ bool last;
  loss_body<THREADS>(I, tau, dl_di, per_wl, W, T, blockIdx.x, sh);
  if (!arrived) return;
  if (threadIdx.x == 0) {
    __threadfence();  // per_wl[w] before the count, for the block on another XCD that reads it
    last = atomicInc(arrived, static_cast<unsigned>(W) - 1u) == static_cast<unsigned>(W) - 1u;
  }
  __syncthreads();
  if (!last) return;
  __threadfence();
  loss_sum_body<THREADS>(per_wl, loss, W, sh);
}

// grouped: task = one design, one block per wavelength of every design; the designs of a launch have
// images of one size class, since the order of the sums goes with the block's size
template <int THREADS>
__global__ void __launch_bounds__(THREADS)
loss_group_kernel(GroupArgs g, const float* __restrict__ I, const float* __restrict__ tau,
                  float* __restrict__ dl_di) {
  __shared__ double sh[4 * (THREADS / 64)];
  const int ti = group_task(g, blockIdx.x);
  const LossTask& t = static_cast<const LossTask*>(g.tasks)[ti];
  const int w = static_cast<int>(blockIdx.x) - g.block0[ti];
  loss_body<THREADS>(I + t.img_off, tau + t.img_off, dl_di ? dl_di + t.img_off : nullptr, t.per_wl, t.W, t.T, w, sh);
}

__global__ void __launch_bounds__(kLossThreads)
loss_sum_kernel(const double* __restrict__ per_wl, double* __restrict__ loss, int W) {
  __shared__ double sh[kLossThreads / 64];
  loss_sum_body<kLossThreads>(per_wl, loss, W, sh);
}

// grouped: block i = design i of the plan (tasks in design order)
__global__ void __launch_bounds__(kLossThreads)
loss_sum_group_kernel(const LossTask* __restrict__ tasks, double* __restrict__ loss) {
  __shared__ double sh[kLossThreads / 64];
  const LossTask& t = tasks[blockIdx.x];
  loss_sum_body<kLossThreads>(t.per_wl, loss + blockIdx.x, t.W, sh);
}

// Fixed device array for the per-wavelength loss partials of dpx_loss_static (callers that cannot
// allocate): every GPU the library runs on holds one copy until the process ends.  Host code
// never passes the array's name to a kernel (in host code it is a stand-in, not a device
// address); static_loss_scratch() returns the device address, looked up once per device.
static __device__ __align__(256) double scratch[kStaticLossMaxWl];

constexpr int kMaxScratchDevices = 64;

hipError_t static_loss_scratch(double** out) {
  static std::mutex mu;
  static void* ptr[kMaxScratchDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    ptr[dev] = p;
  }
  *out = static_cast<double*>(ptr[dev]);
  return hipSuccess;
}

// Sum of the gradient slots in double, in an order fixed by the sizes alone.  Bound by the slots'
// traffic (128 MB for 2048 slots of a two-layer 64 x 64 design) and, where one thread walks all
// slots of an element, by one load latency per slot: that form took 794 us at 4096 wavelengths of a
// three-layer 64 x 64 design and 64 us (2.6 TB/s) at 128 slots of five 256 x 256 layers.  So a
// block of 256 threads takes LANES x 4 elements with 256 / LANES groups of threads, each summing
// every (256 / LANES)-th slot with 16-byte loads, four in flight; the groups' sums are added in
// order.
template <int LANES>
__device__ __forceinline__ void dh_reduce_body(const float* __restrict__ part, float* __restrict__ dh, int nslots,
                                               int64_t per, int64_t block, double* sh) {
  constexpr int G = kGroupThreads / LANES;
  const int g = threadIdx.x / LANES, l = threadIdx.x % LANES;
  const int64_t first = block * (LANES * 4);
  const int64_t i = first + l * 4;  // per is a multiple of four (K N N with N even)
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  if (i < per) {
    int c = g;
    for (; c + 3 * G < nslots; c += 4 * G) {
      float4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const float4*>(part + (c + u * G) * per + i);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        s[0] += v[u].x;
        s[1] += v[u].y;
        s[2] += v[u].z;
        s[3] += v[u].w;
      }
    }
    for (; c < nslots; c += G) {
      const float4 v = *reinterpret_cast<const float4*>(part + c * per + i);
      s[0] += v.x;
      s[1] += v.y;
      s[2] += v.z;
      s[3] += v.w;
    }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) sh[g * (LANES * 4) + l * 4 + u] = s[u];
  __syncthreads();
  const int e = threadIdx.x;
  if (e < LANES * 4 && first + e < per) {
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < G; ++k) t += sh[k * (LANES * 4) + e];
    dh[first + e] = static_cast<float>(t);
  }
}

// 16 groups of 16 threads where 64-thread groups would leave most CUs without a block and there
// are slots enough to share, else 4 groups of 64
constexpr int kDhNarrow = 16, kDhWide = 64;
static int dh_lanes(int64_t per, int nslots) {
  return per < 512LL * kDhWide * 4 && nslots >= 4 * (kGroupThreads / kDhNarrow) ? kDhNarrow : kDhWide;
}
int dh_blocks(int64_t per, int nslots) {
  const int lanes = dh_lanes(per, nslots);
  return static_cast<int>((per + lanes * 4 - 1) / (lanes * 4));
}

template <int LANES>
__global__ void __launch_bounds__(kGroupThreads)
dh_reduce_kernel(const float* __restrict__ part, float* __restrict__ dh, int nslots, int64_t per) {
  __shared__ double sh[kGroupThreads * 4];
  dh_reduce_body<LANES>(part, dh, nslots, per, blockIdx.x, sh);
}

// grouped: task = one design's gradient slots -> its dL/dh in the packed output
__global__ void __launch_bounds__(kGroupThreads) dh_group_kernel(GroupArgs g, float* __restrict__ dl_dh) {
  __shared__ double sh[kGroupThreads * 4];
  const int ti = group_task(g, blockIdx.x);
  const DhTask& t = static_cast<const DhTask*>(g.tasks)[ti];
  const int64_t local = static_cast<int>(blockIdx.x) - g.block0[ti];
  if (t.lanes == kDhNarrow) dh_reduce_body<kDhNarrow>(t.part, dl_dh + t.h_off, t.nslots, t.per, local, sh);
  else dh_reduce_body<kDhWide>(t.part, dl_dh + t.h_off, t.nslots, t.per, local, sh);
}
DhTask dh_task(const float* part, int64_t h_off, int64_t per, int nslots) {
  return {part, h_off, per, nslots, dh_lanes(per, nslots)};
}

// ------------------------------------------------------------------------------------------
// Training support (Section 4: Adam with the optimizer library's defaults; heights bounded to
// [0, h_max] through a sigmoid of an unconstrained variable)
// ------------------------------------------------------------------------------------------
// One Adam step on theta with h = h_max sigmoid(theta):
//   g = dL/dh * h_max s (1 - s),  m = b1 m + (1 - b1) g,  v = b2 v + (1 - b2) g^2,
//   theta -= lr (m c1) / (sqrt(v c2) + eps)  with c1 = 1 / (1 - b1^t), c2 = 1 / (1 - b2^t),
// then h = h_max sigmoid(theta).  Arithmetic in single precision; 1 - b1, 1 - b2 and the bias
// corrections come from the host, formed in double.
// Phase bit depth: the nearest of the levels k step, k = 0 .. kmax (ties to even), the level
// index decided in single precision as rint(h scale), clamped to the end levels.
__global__ void quantize_kernel(const float* h, float* out, int64_t n, float scale, float step, float kmax) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float k = fminf(fmaxf(rintf(h[i] * scale), 0.0f), kmax);
  out[i] = k * step;
}

__global__ void adam_sigmoid_kernel(float* __restrict__ theta, float* __restrict__ h, const float* __restrict__ dl_dh,
                                    float* __restrict__ m, float* __restrict__ v, int64_t n, AdamArgs a) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float th = theta[i];
  // s (1 - s) = e / (1 + e)^2 with e = exp(-|theta|): even in theta, no cancellation near
  // s = 1 and no overflow for large |theta|.
  const float e = expf(-fabsf(th));
  const float ope = 1.0f + e;
  const float g = dl_dh[i] * (a.h_max * (e / (ope * ope)));
  const float mi = fmaf(a.b1, m[i], a.omb1 * g);
  const float vi = fmaf(a.b2, v[i], a.omb2 * (g * g));
  m[i] = mi;
  v[i] = vi;
  const float t2 = th - a.lr * (mi * a.c1) / (sqrtf(vi * a.c2) + a.eps);
  theta[i] = t2;
  h[i] = a.h_max / (1.0f + expf(-t2));
}

// Per-wavelength PSNR of the intensity image against its target, both normalised to unit sum
// (as in the loss): 10 log10(max_p tau^2 / mean_p (I - tau)^2), in double; one block per
// wavelength of one design ([W][T][T] images, out [W]).
template <int THREADS, int CACHE>
__device__ __forceinline__ void psnr_image(const float* __restrict__ Iw, const float* __restrict__ tw,
                                           double* __restrict__ out, int P, double* sh) {
  constexpr int WAVES = THREADS / 64;
  const Pixels<THREADS, CACHE> px(Iw, tw, P);
  double si = 0.0, st = 0.0, mx = 0.0;
  px.each([&](int, float i, float t) {
    si += i;
    st += t;
    mx = fmax(mx, static_cast<double>(t));
  });
  block_combine_begin<THREADS>(si, sh, Plus{});
  block_combine_begin<THREADS>(st, sh + WAVES, Plus{});
  block_combine_begin<THREADS>(mx, sh + 2 * WAVES, Max{});
  __syncthreads();
  const double S = block_combine_end<THREADS>(sh, Plus{}), St = block_combine_end<THREADS>(sh + WAVES, Plus{});
  const double tmax = block_combine_end<THREADS>(sh + 2 * WAVES, Max{});
  const double rS = S > 0.0 ? 1.0 / S : 0.0;
  const double rSt = St > 0.0 ? 1.0 / St : 0.0;
  double sd2 = 0.0;
  px.each([&](int, float i, float t) {
    const double d = i * rS - t * rSt;
    sd2 += d * d;
  });
  block_combine_begin<THREADS>(sd2, sh + 3 * WAVES, Plus{});
  __syncthreads();
  if (threadIdx.x == 0) {
    const double mse = block_combine_end<THREADS>(sh + 3 * WAVES, Plus{}) / P;
    const double peak = tmax * rSt;
    *out = (mse > 0.0) ? 10.0 * log10(peak * peak / mse) : INFINITY;
  }
}

template <int THREADS>
__global__ void __launch_bounds__(THREADS)
psnr_kernel(const float* __restrict__ I, const float* __restrict__ tau, double* __restrict__ out, int T) {
  __shared__ double sh[4 * (THREADS / 64)];
  const int P = T * T;
  const size_t o = static_cast<size_t>(blockIdx.x) * P;
  if (P <= kLossCache * THREADS) psnr_image<THREADS, kLossCache>(I + o, tau + o, out + blockIdx.x, P, sh);
  else psnr_image<THREADS, 0>(I + o, tau + o, out + blockIdx.x, P, sh);
}

__global__ void fill_zero_kernel(float* p, int64_t n) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

// Counts the NaN and infinite values of x (grid-stride); one integer atomic per lane that
// found any, so the count is exact and independent of the launch shape.
template <typename T>
__global__ void __launch_bounds__(256) count_nonfinite_kernel(const T* __restrict__ x, int64_t n,
                                                              unsigned* __restrict__ count) {
  unsigned c = 0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    c += isfinite(x[i]) ? 0u : 1u;
  if (c) atomicAdd(count, c);
}


// ------------------------------------------------------------------------------------------
// Host-side tables and sizes
// ------------------------------------------------------------------------------------------
void build_dft_table(int M, int pad, std::vector<float2>& out) {
  const int N = M / pad;
  out.assign(static_cast<size_t>(2) * M * N, make_float2(0.f, 0.f));
  for (int ky = 0; ky < M; ++ky)
    for (int y = 0; y < N; ++y) {
      const long long m = (static_cast<long long>(ky) * y) % M;
      const double ang = 6.283185307179586476925286766559 * static_cast<double>(m) / M;
      const float2 v = make_float2(static_cast<float>(std::cos(ang)), static_cast<float>(-std::sin(ang)));
      out[static_cast<size_t>(y) * M + ky] = v;              // FT[y][ky]
      out[static_cast<size_t>(M) * N + static_cast<size_t>(ky) * N + y] = v;  // F[ky][y]
    }
}

void build_twiddle_table(int M, int plan, const UnitRoots& u, std::vector<float2>& out) {
  switch (M) {
#define DPX_CASE(m) case m: twiddle_table_##m(plan, u, out); return;
    DPX_FOR_EACH_M(DPX_CASE)
#undef DPX_CASE
    default:
      out.clear();
  }
}
int radix_plan_count(int M) { return fft_size_supported(M) ? radix_plans(M) : 0; }
template <int m, int v>
static void radix_name(char* buf, size_t cap) {
  int n = 0;
  for (int st = 0; st < Radix<m, v>::NST; ++st)
    n += snprintf(buf + n, cap - n, st ? "x%d" : "%d", Radix<m, v>::R[st]);
}
// "16x16x4": the radices of plan `plan` of length M (empty for an unknown pair)
const char* radix_plan_name(int M, int plan) {
  static thread_local char buf[32];
  buf[0] = 0;
  if (plan < 0 || plan >= radix_plan_count(M)) return buf;
  switch (M) {
#define DPX_CASE(m) \
  case m:           \
    if (plan == 0) radix_name<m, 0>(buf, sizeof(buf)); \
    break;
    DPX_FOR_EACH_M(DPX_CASE)
#undef DPX_CASE
    default: break;
  }
  if (M == 512 && plan == 1) radix_name<512, 1>(buf, sizeof(buf));
  if (M == 512 && plan == 2) radix_name<512, 2>(buf, sizeof(buf));
  if (M == 1024 && plan == 1) radix_name<1024, 1>(buf, sizeof(buf));
  if (M == 1024 && plan == 2) radix_name<1024, 2>(buf, sizeof(buf));
  return buf;
}

bool fft_size_supported(int M) {
  switch (M) {
#define DPX_CASE(m) case m:
    DPX_FOR_EACH_M(DPX_CASE)
#undef DPX_CASE
    return true;
    default:
      return false;
  }
}

int row_lanes_per_transform(int M) {
  switch (M) {
#define DPX_CASE(m) case m: return Geo<m>::P;
    DPX_FOR_EACH_M(DPX_CASE)
#undef DPX_CASE
    default:
      return 0;
  }
}

int row_rows_per_block(int M, int pad, int mode, bool small) {
  const int P = row_lanes_per_transform(M);
  if (P == 0) return 0;
  return row_threads_for(M, P, pad, mode, small) / P;
}

// Fewer blocks than the chip has CUs: the rows of 128-thread blocks spread over up to four times as
// many.  Measured, forward of three layers, us: one wavelength of 96 x 96 39 -> 34, 192 x 192 51 -> 43,
// 256 x 256 48 -> 42, 512 x 512 63 -> 59; eight of 192 x 192 60 -> 54; from 256 blocks on both forms
// take the same time and the larger blocks stage the twiddles for more rows.  Unpadded rows of 1024 points
// take their other form (row_threads_for) where theirs would put a second block on CUs: forward of three
// layers, us, in blocks of 256 and 512 threads: one wavelength 82 and 84, two 100 and 88, three 114 and 115,
// six 191 and 196.
bool row_blocks_small(int M, int pad, int mode, int rows, int n_w) {
  const int P = row_lanes_per_transform(M);
  if (P == 0 || P > 64 || 64 % P) return false;
  const int per = row_rows_per_block(M, pad, mode);
  const int64_t blocks = static_cast<int64_t>((rows + per - 1) / per) * n_w;
  return pad == 1 && M >= 1024 ? blocks > 256 && blocks <= 512 : blocks < 256;
}

namespace {
// the lanes of one transform lie in one wavefront (else its LDS exchanges take block barriers,
// tiles are 4 or 8 columns wide and H has no cross-lane mirrored form)
bool wave_local(int M) {
  const int P = row_lanes_per_transform(M);
  return P > 0 && P <= 64 && 64 % P == 0;
}
}  // namespace

// Column-pass variants (0-3 give the same results bit for bit; 4 differs by rounding):
//   0: 8-column tiles, 1: 16-column tiles, 2: 8-column tiles + mirrored H rows,
//   3: 16-column tiles + mirrored H rows, 4: DFT as complex matrix products on the matrix
//   cores (transform lengths up to 512).
// Tiles must be whole wavefronts: with fewer than 8 lanes per transform, 8-column tiles
// fall back to 16 columns.
const char* const kColVariantNames[kColVariants] = {"tile8", "tile16", "tile8+mirror",
                                                    "tile16+mirror", "dft-gemm-mfma"};

// built-in choice when no variant is forced and no autotuning is asked for: the mirrored forms
// where transforms stay in one wavefront; at 1600 unpadded the wide tile (8 columns, 10 waves per CU
// in one block) beats the narrow one, which the registers hold to one 5-wave block per CU.  The split
// transforms take 16 columns, so that a row segment is a whole 128-byte line (512 points, 1024
// wavelengths: column and next row pass 1165 against 1174 us, 256 points 700 against 780), except
// where the wide block is short of registers (384 points without padding: 96 against 66 us) or the
// launch would leave CUs empty.
int default_col_variant(int M, int pad, int wavelengths) {
  if (!wave_local(M)) return 1;
  if (!col_split(M, pad)) return M >= 512 ? 2 : 3;
  return (M / pad >= 384 || static_cast<int64_t>(wavelengths) * (M / 16) < 512) ? 2 : 3;
}

bool col_variant_supported(int M, int pad, int variant) {
  if (variant < 0 || variant >= kColVariants) return false;
  if (variant == 4) return M <= 512 && M % 16 == 0 && (M / pad) % 16 == 0;
  if (!wave_local(M)) return variant <= 1;
  return true;
}

int col_tile_width(int M, int pad, int variant) {
  switch (M) {
#define DPX_CASE(m) case m: return col_tile_width_##m(pad, variant);
    DPX_FOR_EACH_M(DPX_CASE)
#undef DPX_CASE
    default:
      return 16;
  }
}

bool col_split(int M, int pad) {
  switch (M) {
#define DPX_CASE(m) case m: return col_split_##m(pad);
    DPX_FOR_EACH_M(DPX_CASE)
#undef DPX_CASE
    default:
      return false;
  }
}

void build_col_table(int M, int pad, const UnitRoots& u, std::vector<float2>& out) {
  switch (M) {
#define DPX_CASE(m) case m: col_table_##m(pad, u, out); return;
    DPX_FOR_EACH_M(DPX_CASE)
#undef DPX_CASE
    default:
      out.clear();
  }
}


// ------------------------------------------------------------------------------------------
// Dispatch to the per-length launchers
// ------------------------------------------------------------------------------------------
hipError_t launch_row(int M, int pad, int mode, int plan, bool small, const RowArgs& a, int n_row_blocks, int n_w_blocks,
                      hipStream_t s) {
  switch (M) {
#define DPX_CASE(m) case m: return launch_row_##m(pad, mode, plan, small, a, n_row_blocks, n_w_blocks, s);
    DPX_FOR_EACH_M(DPX_CASE)
#undef DPX_CASE
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_row_group(int M, int pad, int mode, const GroupArgs& g, hipStream_t s) {
  if (g.ntasks < 1 || g.ntasks > kMaxGroupTasks) return hipErrorInvalidValue;
  switch (M) {
#define DPX_CASE(m) case m: return launch_row_group_##m(pad, mode, g, s);
    DPX_FOR_EACH_M(DPX_CASE)
#undef DPX_CASE
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_col(int M, int pad, bool conj, int variant, int plan, const ColArgs& a, int w_count,
                      hipStream_t s) {
  if (!col_variant_supported(M, pad, variant)) return hipErrorInvalidValue;
  switch (M) {
#define DPX_CASE(m) case m: return launch_col_##m(pad, conj, variant, plan, a, w_count, s);
    DPX_FOR_EACH_M(DPX_CASE)
#undef DPX_CASE
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_col_group(int M, int pad, bool conj, int variant, bool table, bool full, const GroupArgs& g,
                            hipStream_t s) {
  if (g.ntasks < 1 || g.ntasks > kMaxGroupTasks || variant < 0 || variant > 3) return hipErrorInvalidValue;
  switch (M) {
#define DPX_CASE(m) case m: return launch_col_group_##m(pad, conj, variant, table, full, g, s);
    DPX_FOR_EACH_M(DPX_CASE)
#undef DPX_CASE
    default:
      return hipErrorInvalidValue;
  }
}

bool lds_path_supported(int M, int pad) {
  switch (M) {
#define DPX_CASE(m) case m: return lds_supported_##m(pad);
    DPX_FOR_EACH_M(DPX_CASE)
#undef DPX_CASE
    default:
      return false;
  }
}

// A wavelength on one CU costs no launches and no plane traffic between the passes, but takes the CU's
// own time for all of it, so the passes win where a few wavelengths leave the other CUs idle (128
// and 96 points) and, for the short transforms whose planes stay in the last-level cache, where
// there are thousands.  Measured, one forward, loss and gradient of two layers, passes against
// LDS-resident, us: 64 points 44 / 30 (1 wavelength), 86 / 51 (512), 177 / 163 (2048), 276 / 304 (4096);
// 96 points 54 / 64 (32), 59 / 64 (64), 67 / 66 (96), 134 / 104 (512), 201 / 190 (1024), 346 / 362 (2048);
// 128 points 60 / 68 (32), 66 / 69 (64), 92 / 72 (128), 122 / 80 (256), 980 / 758 (4096); 64 points
// without padding 41 / 36 (1), 84 / 53 (256), 443 / 435 (4096), 96 without padding 53 / 110 (1),
// 126 / 137 (256).
bool lds_path_preferred(int M, int pad, int wavelengths) {
  if (pad == 1) return M == 64;
  if (M == 64) return wavelengths <= 2048;
  if (M == 96) return wavelengths >= 96 && wavelengths <= 1024;
  return M == 128 && wavelengths >= 64;
}

hipError_t launch_lds(int M, int pad, bool adjoint, const LdsArgs& a, hipStream_t s) {
  switch (M) {
#define DPX_CASE(m) case m: return launch_lds_##m(pad, adjoint, a, s);
    DPX_FOR_EACH_M(DPX_CASE)
#undef DPX_CASE
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_transfer_table(int M, const WlConst* wl, int W, double zrev, float2* out, hipStream_t s) {
  switch (M) {
#define DPX_CASE(m) case m: return launch_transfer_table_##m(wl, W, zrev, out, s);
    DPX_FOR_EACH_M(DPX_CASE)
#undef DPX_CASE
    default:
      return hipErrorInvalidValue;
  }
}

// ------------------------------------------------------------------------------------------
// Small kernels: launchers
// ------------------------------------------------------------------------------------------
hipError_t launch_bin_intensity(const float2* ofov, float* out, int w_count, int fov, int bin,
                                hipStream_t s) {
  const int T = fov / bin;
  const size_t total = static_cast<size_t>(w_count) * T * T;
  const int th = 256;
  bin_intensity_kernel<<<static_cast<unsigned>((total + th - 1) / th), th, 0, s>>>(ofov, out, w_count,
                                                                                 fov, bin);
  return hipGetLastError();
}

hipError_t launch_loss(const float* I, const float* tau, float* dl_di, double* per_wl, int W, int T,
                       unsigned* arrived, double* loss, hipStream_t s) {
  if (large_image(T))
    loss_kernel<kLossThreadsLarge><<<W, kLossThreadsLarge, 0, s>>>(I, tau, dl_di, per_wl, W, T, arrived, loss);
  else
    loss_kernel<kLossThreads><<<W, kLossThreads, 0, s>>>(I, tau, dl_di, per_wl, W, T, arrived, loss);
  return hipGetLastError();
}

hipError_t launch_loss_sum(const double* per_wl, double* loss, int W, hipStream_t s) {
  loss_sum_kernel<<<1, kLossThreads, 0, s>>>(per_wl, loss, W);
  return hipGetLastError();
}

hipError_t launch_dh_reduce(const float* part, float* dh, int nslots, int64_t per, hipStream_t s) {
  const unsigned blocks = static_cast<unsigned>(dh_blocks(per, nslots));
  if (dh_lanes(per, nslots) == kDhNarrow)
    dh_reduce_kernel<kDhNarrow><<<blocks, kGroupThreads, 0, s>>>(part, dh, nslots, per);
  else
    dh_reduce_kernel<kDhWide><<<blocks, kGroupThreads, 0, s>>>(part, dh, nslots, per);
  return hipGetLastError();
}

static unsigned group_grid(const GroupArgs& g) { return static_cast<unsigned>(g.block0[g.ntasks]); }

hipError_t launch_bin_group(const GroupArgs& g, float* out, hipStream_t s) {
  if (g.ntasks < 1 || g.ntasks > kMaxGroupTasks) return hipErrorInvalidValue;
  bin_group_kernel<<<group_grid(g), kGroupThreads, 0, s>>>(g, out);
  return hipGetLastError();
}

hipError_t launch_loss_group(const GroupArgs& g, bool large, const float* I, const float* tau, float* dl_di,
                             hipStream_t s) {
  if (g.ntasks < 1 || g.ntasks > kMaxGroupTasks) return hipErrorInvalidValue;
  if (large) loss_group_kernel<kLossThreadsLarge><<<group_grid(g), kLossThreadsLarge, 0, s>>>(g, I, tau, dl_di);
  else loss_group_kernel<kLossThreads><<<group_grid(g), kLossThreads, 0, s>>>(g, I, tau, dl_di);
  return hipGetLastError();
}

hipError_t launch_loss_sum_group(const LossTask* tasks, int ntasks, double* loss, hipStream_t s) {
  if (ntasks < 1) return hipErrorInvalidValue;
  loss_sum_group_kernel<<<ntasks, kLossThreads, 0, s>>>(tasks, loss);
  return hipGetLastError();
}

hipError_t launch_dh_group(const GroupArgs& g, float* dl_dh, hipStream_t s) {
  if (g.ntasks < 1 || g.ntasks > kMaxGroupTasks) return hipErrorInvalidValue;
  dh_group_kernel<<<group_grid(g), kGroupThreads, 0, s>>>(g, dl_dh);
  return hipGetLastError();
}

hipError_t launch_quantize(const float* h, float* out, int64_t n, float scale, float step, float kmax,
                           hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int th = 256;
  quantize_kernel<<<static_cast<unsigned>((n + th - 1) / th), th, 0, s>>>(h, out, n, scale, step, kmax);
  return hipGetLastError();
}

hipError_t launch_adam_sigmoid(float* theta, float* h, const float* dl_dh, float* m, float* v, int64_t n,
                               const AdamArgs& a, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int th = 256;
  adam_sigmoid_kernel<<<static_cast<unsigned>((n + th - 1) / th), th, 0, s>>>(theta, h, dl_dh, m, v, n, a);
  return hipGetLastError();
}

hipError_t launch_psnr(const float* I, const float* tau, double* out, int W, int T, hipStream_t s) {
  if (W <= 0) return hipSuccess;
  if (large_image(T)) psnr_kernel<kLossThreadsLarge><<<W, kLossThreadsLarge, 0, s>>>(I, tau, out, T);
  else psnr_kernel<kLossThreads><<<W, kLossThreads, 0, s>>>(I, tau, out, T);
  return hipGetLastError();
}

hipError_t launch_fill_zero(float* p, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int th = 256;
  fill_zero_kernel<<<static_cast<unsigned>((n + th - 1) / th), th, 0, s>>>(p, n);
  return hipGetLastError();
}

template <typename T>
hipError_t count_nonfinite(const T* x, int64_t n, unsigned* count, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int th = 256;
  const int64_t blocks = std::min<int64_t>((n + th - 1) / th, 4096);
  count_nonfinite_kernel<T><<<static_cast<unsigned>(blocks), th, 0, s>>>(x, n, count);
  return hipGetLastError();
}
hipError_t launch_count_nonfinite(const float* x, int64_t n, unsigned* count, hipStream_t s) {
  return count_nonfinite(x, n, count, s);
}
hipError_t launch_count_nonfinite(const double* x, int64_t n, unsigned* count, hipStream_t s) {
  return count_nonfinite(x, n, count, s);
}

}  // namespace dpx
