// Delay-rate fringe search over stacked sub-integrations (the search behind
// the paper's first-fringe result, section 2): a zero-padded FFT over the
// channels of every (sub-integration, subband, baseline) row, then per chunk
// of delay columns of every (subband, baseline) map a zero-padded FFT over
// sub-integrations and the chunk's windowed peak, then per map the parabolic
// refinement of its best peak.
#include <math.h>

#include <atomic>

#include "xc_fft.h"
#include "xc_launch.h"
#include "xc_runtime.h"

namespace xc {

// Delay transform: rows q = (t, map) of vis [T][n_maps][n_chan], each
// zero-padded to D, into F [n_maps][T][D].  A workgroup runs kDelayIters
// groups of G rows (T threads a row, as in the F stage's FFT), with the
// twiddles in LDS tables filled once: the full per-pass tables up to D = 2048,
// the split ones above (less LDS, more resident workgroups).
constexpr int kDelayIters = 4;

template <int D>
struct RowGeom {
  static constexpr int T = FftPlan<D>::T;
  static constexpr int E = FftPlan<D>::E;
  static constexpr int G = T >= 256 ? 1 : 256 / T;
  static constexpr int WG = T * G;
  static constexpr bool split = D >= 4096;
  static constexpr int tw_entries = split ? tw_split_entries<D>() : tw_lds_entries<D>();
  static constexpr size_t lds_bytes =
      ((size_t)G * lds_words<D>() + (size_t)tw_entries) * sizeof(float2);
};

// A map's best peak while its chunks run: the upper half of the key is |G|^2
// (its bits order like the value), the lower the complement of the bin index, so
// the largest key is the largest value, of the smallest index on a tie.  It sits
// in the map's entry of the result until the refinement writes that.
__device__ inline unsigned long long* peak_key(xc_fringe_peak* p) {
  return reinterpret_cast<unsigned long long*>(p);
}

template <int D, bool HALF>
__global__ void __launch_bounds__(RowGeom<D>::WG)
    k_fringe_delay(const float2* __restrict__ vis, float2* __restrict__ F,
                   const float2* __restrict__ tw, xc_fringe_peak* __restrict__ peaks, int n_sub,
                   int n_maps, int n_chan) {
  using Gm = RowGeom<D>;
  constexpr int T = Gm::T, E = Gm::E, G = Gm::G;
  extern __shared__ float2 lds_all[];
  float2* tab = lds_all + G * lds_words<D>();
  if constexpr (Gm::split)
    tw_split_fill<D>(tab, tw, threadIdx.x, blockDim.x);
  else
    tw_lds_fill<D>(tab, tw, threadIdx.x, blockDim.x);
  const int g = threadIdx.x / T, t = threadIdx.x % T;
  const long n_rows = (long)n_sub * n_maps;
  // no peak found yet
  for (int m = blockIdx.x * blockDim.x + threadIdx.x; m < n_maps; m += gridDim.x * blockDim.x)
    *peak_key(peaks + m) = 0ull;
  // a row's samples n = t + e T; HALF: the upper half are the padding's zeros,
  // which leaves registers to load the next row while this one is transformed
  constexpr int EL = HALF ? E / 2 : E;
  float2 nx[EL];
  auto load = [&](int it) {
    const long q = ((long)blockIdx.x * kDelayIters + it) * G + g;
    const float2* x = vis + q * n_chan;
#pragma unroll
    for (int e = 0; e < EL; ++e) {
      const int n = t + e * T;
      nx[e] = q < n_rows && n < n_chan ? x[n] : make_float2(0.f, 0.f);
    }
  };
  if constexpr (HALF) load(0);
#pragma unroll 1
  for (int it = 0; it < kDelayIters; ++it) {
    if constexpr (!HALF) load(it);
    __syncthreads();   // tables written / the previous group's exchange done
    const long q = ((long)blockIdx.x * kDelayIters + it) * G + g;
    const bool live = q < n_rows;   // (rows past the end transform zeros and store nothing)
    float2 v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = e < EL ? nx[e < EL ? e : 0] : make_float2(0.f, 0.f);
    if constexpr (HALF)
      if (it + 1 < kDelayIters) load(it + 1);
    if constexpr (Gm::split)
      fft_forward<D>(v, lds_all + g * lds_words<D>(), TwSplit<D>{tab}, t);
    else
      fft_forward<D>(v, lds_all + g * lds_words<D>(), TwLds<D>{tab}, t);
    if (!live) continue;
    const int m = (int)(q % n_maps), ts = (int)(q / n_maps);
    float2* out = F + ((size_t)m * n_sub + ts) * D;
    constexpr int B = E / 16;
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) out[t + b * T + r * (D / 16)] = v[b + r * B];
  }
}

// Rate transform and peak: one workgroup (256 threads) per chunk of columns of a
// (subband, baseline) map.  Each round takes GC delay columns; a column's
// R-point transform over sub-integrations (zero-padded from n_sub) runs on
// TR = R/16 threads of 16 values (the LDS Stockham FFT) for R >= 32, or in one
// thread's registers for R <= 16.  Thread (tl, c) = threadIdx tl GC + c, so a
// wave's loads of one sub-integration row are consecutive columns.
// A whole map per workgroup takes 180 us however few maps there are (R = 128,
// 2048 delays), and 1680 maps would be 2.2 rounds of the GPU; in chunks, 64 maps
// of 64 sub-integrations and 1024 channels take 85 us a call instead of 232, 960
// of 200 sub-integrations (R = 512) 355 instead of 870.  At four waves per SIMD
// and with a round's columns interleaved in LDS (ColIdx: half of the LDS cycles
// were bank conflicts) the kernel takes 409 us for 1680 maps (736 before),
// 4.3 TB/s of F; the delay kernel before it streams at a copy's rate (557 us,
// 4.8 TB/s).
constexpr int kFringeThreads = 256;

template <int R>
struct RateGeom {
  static constexpr bool fft = R >= 32;
  static constexpr int TR = fft ? R / 16 : 1;       // threads per column
  static constexpr int E = fft ? 16 : R;            // values per thread
  static constexpr int GC = kFringeThreads / TR;    // columns per round
  // up to 256 points the columns of a round lie interleaved in LDS
  static constexpr bool col = GC >= 16;
  static constexpr int words = !fft ? 0 : col ? R * GC + (GC < 32 ? R : 0) : GC * lds_words<R>();
  static constexpr size_t lds_bytes =
      fft ? ((size_t)words + (size_t)tw_lds_entries<R>()) * sizeof(float2) : 0;
};

template <int R>
__device__ inline void small_dft(float2 (&v)[R]) {
  if constexpr (R > 1) Dft<R>::run(v);
}

// signed bin: [-n/2, n/2) for even n; a one-point axis has the single bin 0
__device__ inline int signed_bin(int b, int n) { return b >= (n + 1) / 2 ? b - n : b; }

// |G|^2 ordering with the tie rule: larger value first, then smaller index.
__device__ inline bool better(float a, int ia, float b, int ib) {
  return a > b || (a == b && ia < ib);
}

// G[r, d] by direct summation over sub-integrations (the refinement's
// neighbours), in their order, twiddles exp(-2 pi i m / R) from the global table
__device__ inline float2 rate_point(const float2* __restrict__ Fm, const float2* __restrict__ tw,
                                    int n_sub, int R, int D, int r, int d) {
  float2 acc = make_float2(0.f, 0.f);
#pragma unroll 8
  for (int ts = 0; ts < n_sub; ++ts) {
    const float2 f = Fm[(size_t)ts * D + d];
    const float2 w = tw[(size_t)((ts * r) & (R - 1)) * (kTwiddleN / R)];
    acc.x = fmaf(f.x, w.x, fmaf(-f.y, w.y, acc.x));
    acc.y = fmaf(f.x, w.y, fmaf(f.y, w.x, acc.y));
  }
  return acc;
}

__device__ inline float parabola_off(float am, float a0, float ap) {
  const float den = am - 2.f * a0 + ap;
  return den == 0.f ? 0.f : (am - ap) / (2.f * den);
}

template <int R, bool HALF>
__global__ void __launch_bounds__(kFringeThreads, 4)
    k_fringe_rate(const float2* __restrict__ F, const float2* __restrict__ tw,
                  xc_fringe_peak* __restrict__ peaks, float2* __restrict__ map, int n_sub, int D,
                  int cols, int delay_win, int rate_win) {
  using Rg = RateGeom<R>;
  constexpr int TR = Rg::TR, E = Rg::E, GC = Rg::GC;
  extern __shared__ float2 sh[];
  const int map_id = blockIdx.x;
  const float2* Fm = F + (size_t)map_id * n_sub * D;
  float2* tab = sh + Rg::words;
  if constexpr (Rg::fft) tw_lds_fill<R>(tab, tw, threadIdx.x, blockDim.x);
  const int c = threadIdx.x % GC, tl = threadIdx.x / GC;
  float bv = -1.f;
  int bi = 0x7fffffff;
  // a column's sub-integrations ts = tl + e TR; HALF: the upper half are zeros,
  // which leaves registers to load the next round while this one is transformed
  constexpr int EL = HALF ? E / 2 : E;
  float2 nx[EL];
  auto load = [&](int d) {
#pragma unroll
    for (int e = 0; e < EL; ++e) {
      const int ts = tl + e * TR;
      nx[e] = ts < n_sub ? Fm[(size_t)ts * D + d] : make_float2(0.f, 0.f);
    }
  };
  auto search = [&](float2 (&v)[E], int d) {
    if constexpr (Rg::fft) {
      __syncthreads();   // tables written / the previous round's exchange done
      if constexpr (Rg::col)
        fft_forward<R, ColIdx<GC>>(v, sh + c, TwLds<R>{tab}, tl);
      else
        fft_forward<R>(v, sh + c * lds_words<R>(), TwLds<R>{tab}, tl);
    } else {
      small_dft<R>(v);
    }
    // v[j] = G[tl + j R/16, d] (FFT), G[j, d] (registers); r grows with j
    auto rate_of = [&](int j) { return Rg::fft ? tl + j * (R / 16) : j; };
    if (map) {
#pragma unroll
      for (int j = 0; j < E; ++j) map[((size_t)map_id * R + rate_of(j)) * D + d] = v[j];
    }
    // the round's largest |G|^2; only where it reaches the thread's best so far
    // (seldom, after a few rounds) its index, the first j on ties: the smallest r D + d
    float a2[E];
    const int ds = signed_bin(d, D);
    const bool d_in = delay_win <= 0 || (ds <= delay_win && ds >= -delay_win);
    float m = -1.f;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      a2[j] = v[j].x * v[j].x + v[j].y * v[j].y;
      if (rate_win > 0) {
        const int rs = signed_bin(rate_of(j), R);
        if (rs > rate_win || rs < -rate_win) a2[j] = -1.f;
      }
      m = fmaxf(m, a2[j]);
    }
    if (d_in && m >= fmaxf(bv, 0.f)) {
      int mj = 0;
#pragma unroll
      for (int j = E - 1; j >= 0; --j) mj = a2[j] == m ? j : mj;
      const int idx = rate_of(mj) * D + d;
      if (better(m, idx, bv, bi)) {
        bv = m;
        bi = idx;
      }
    }
  };
  // cols is a multiple of GC and divides D: every round is full
  const int d_end = ((int)blockIdx.y + 1) * cols;
  int d = (int)blockIdx.y * cols + c;
  if constexpr (HALF) load(d);
#pragma unroll 1
  for (; d < d_end; d += GC) {
    if constexpr (!HALF) load(d);
    float2 v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = e < EL ? nx[e < EL ? e : 0] : make_float2(0.f, 0.f);
    if constexpr (HALF)
      if (d + GC < d_end) load(d + GC);
    search(v, d);
  }
  // (a thread without a candidate: every value outside the window or not a number)
  unsigned long long key =
      bv >= 0.f ? (unsigned long long)__float_as_uint(bv) << 32 | (0xffffffffu - (unsigned)bi) : 0ull;
  for (int w = 32; w > 0; w >>= 1) {
    const unsigned long long o = __shfl_xor(key, w);
    key = o > key ? o : key;
  }
  if ((threadIdx.x & 63) == 0 && key) atomicMax(peak_key(peaks + map_id), key);
}

// The best peak's value and its four cyclic neighbours, recomputed from memory
// (a thread each), and the parabolic refinement: kRefineMaps maps a workgroup.
constexpr int kRefineMaps = 12;

__global__ void __launch_bounds__(64)
    k_fringe_refine(const float2* __restrict__ F, const float2* __restrict__ tw,
                    xc_fringe_peak* __restrict__ peaks, int n_maps, int n_sub, int R, int D,
                    int n_chan, double dnu, double t_int) {
  __shared__ float2 pts[5 * kRefineMaps];
  const int m = threadIdx.x / 5, k = threadIdx.x - 5 * m;
  const int map_id = blockIdx.x * kRefineMaps + m;
  const bool live = m < kRefineMaps && map_id < n_maps;
  int pr = 0, pd = 0;
  if (live) {
    const float2* Fm = F + (size_t)map_id * n_sub * D;
    const unsigned long long key = *peak_key(peaks + map_id);
    // (no candidate at all: bin 0, whose values the result then reports)
    const unsigned pi = key ? 0xffffffffu - (unsigned)key : 0u;
    pr = (int)(pi / (unsigned)D);
    pd = (int)(pi - (unsigned)pr * D);
    const int rr = k == 3 ? (pr + R - 1) % R : k == 4 ? (pr + 1) % R : pr;
    const int dd = k == 1 ? (pd + D - 1) % D : k == 2 ? (pd + 1) % D : pd;
    pts[threadIdx.x] = rate_point(Fm, tw, n_sub, R, D, rr, dd);
  }
  __syncthreads();
  if (live && k == 0) {
    const float2* z = pts + 5 * m;
    auto mag = [](float2 z) { return sqrtf(z.x * z.x + z.y * z.y); };
    const float a0 = mag(z[0]);
    const float od = parabola_off(mag(z[1]), a0, mag(z[2]));
    const float orr = parabola_off(mag(z[3]), a0, mag(z[4]));
    const int ds = signed_bin(pd, D), rs = signed_bin(pr, R);
    xc_fringe_peak p;
    p.delay_bin = ds;
    p.rate_bin = rs;
    p.amp = a0 / ((float)n_chan * (float)n_sub);
    p.phase = atan2f(z[0].y, z[0].x);
    p.delay_off = od;
    p.rate_off = orr;
    p.delay_s = ((double)ds + (double)od) / ((double)D * dnu);
    p.rate_hz = ((double)rs + (double)orr) / ((double)R * t_int);
    peaks[map_id] = p;
  }
}

// One attribute call per kernel and device (LDS above 64 KB).
template <class K>
static hipError_t allow_lds(K kernel, size_t bytes, std::atomic<bool> (&done)[64]) {
  if (bytes <= 65536) return hipSuccess;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (done[dev].load()) return hipSuccess;
  e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)bytes);
  if (e == hipSuccess) done[dev].store(true);
  return e;
}

template <int D, bool HALF>
static hipError_t launch_delay_h(const xc_fringe_setup* fs, const float2* vis, float2* F,
                                 const float2* tw, xc_fringe_peak* peaks, hipStream_t s) {
  using Gm = RowGeom<D>;
  static std::atomic<bool> done[64];
  hipError_t e = allow_lds(k_fringe_delay<D, HALF>, Gm::lds_bytes, done);
  if (e != hipSuccess) return e;
  const long n_maps = (long)fs->n_subbands * fs->n_baselines, rows = fs->n_subints * n_maps;
  const long per_wg = (long)Gm::G * kDelayIters;
  hipLaunchKernelGGL((k_fringe_delay<D, HALF>), dim3((unsigned)((rows + per_wg - 1) / per_wg)),
                     dim3(Gm::WG), Gm::lds_bytes, s, vis, F, tw, peaks, fs->n_subints,
                     (int)n_maps, fs->n_chan);
  return hipGetLastError();
}

template <int D>
static hipError_t launch_delay_d(const xc_fringe_setup* fs, const float2* vis, float2* F,
                                 const float2* tw, xc_fringe_peak* peaks, hipStream_t s) {
  return fs->n_chan <= D / 2 ? launch_delay_h<D, true>(fs, vis, F, tw, peaks, s)
                             : launch_delay_h<D, false>(fs, vis, F, tw, peaks, s);
}

template <int R, bool HALF>
static hipError_t launch_rate_h(const xc_fringe_setup* fs, const float2* F, const float2* tw,
                                xc_fringe_peak* peaks, float2* map, hipStream_t s) {
  static std::atomic<bool> done[64];
  hipError_t e = allow_lds(k_fringe_rate<R, HALF>, RateGeom<R>::lds_bytes, done);
  if (e != hipSuccess) return e;
  // Chunks of columns (powers of two of rounds): down to two rounds a workgroup
  // until the maps' workgroups fill the GPU some ten times
  const long maps = (long)fs->n_subbands * fs->n_baselines;
  int cols = fs->delay_len;
  while (cols > 2 * RateGeom<R>::GC && maps * (fs->delay_len / cols) < 8192) cols /= 2;
  hipLaunchKernelGGL((k_fringe_rate<R, HALF>), dim3((unsigned)maps, fs->delay_len / cols),
                     dim3(kFringeThreads), RateGeom<R>::lds_bytes, s, F, tw, peaks, map,
                     fs->n_subints, fs->delay_len, cols, fs->delay_win, fs->rate_win);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_fringe_refine, dim3((unsigned)((maps + kRefineMaps - 1) / kRefineMaps)),
                     dim3(64), 0, s, F, tw, peaks, (int)maps, fs->n_subints, R, fs->delay_len,
                     fs->n_chan, fs->chan_width_hz, fs->t_int_s);
  return hipGetLastError();
}

template <int R>
static hipError_t launch_rate_r(const xc_fringe_setup* fs, const float2* F, const float2* tw,
                                xc_fringe_peak* peaks, float2* map, hipStream_t s) {
  if constexpr (R >= 2)
    if (fs->n_subints <= R / 2) return launch_rate_h<R, true>(fs, F, tw, peaks, map, s);
  return launch_rate_h<R, false>(fs, F, tw, peaks, map, s);
}

hipError_t launch_fringe(const xc_fringe_setup* fs, const float2* vis, float2* F,
                         const float2* tw, xc_fringe_peak* peaks, float2* map, hipStream_t s) {
  hipError_t e;
  switch (fs->delay_len) {
#define XC_DCASE(DD) \
  case DD: e = launch_delay_d<DD>(fs, vis, F, tw, peaks, s); break;
    XC_DCASE(256) XC_DCASE(512) XC_DCASE(1024) XC_DCASE(2048) XC_DCASE(4096) XC_DCASE(8192)
    XC_DCASE(16384)
#undef XC_DCASE
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  switch (fs->rate_len) {
#define XC_RCASE(RR) \
  case RR: return launch_rate_r<RR>(fs, F, tw, peaks, map, s);
    XC_RCASE(1) XC_RCASE(2) XC_RCASE(4) XC_RCASE(8) XC_RCASE(16) XC_RCASE(32) XC_RCASE(64)
    XC_RCASE(128) XC_RCASE(256) XC_RCASE(512) XC_RCASE(1024)
#undef XC_RCASE
    default: return hipErrorInvalidValue;
  }
}

}  // namespace xc

using namespace xc;

namespace {

bool is_pow2(long x) { return x > 0 && (x & (x - 1)) == 0; }

int fringe_validate(xc_ctx* c, const xc_fringe_setup* fs) {
  if (!fs) return fail(c, XC_E_INVAL, "fringe setup is NULL");
  if (fs->n_subints < 1 || fs->n_subints > 256)
    return fail(c, XC_E_INVAL, "n_subints=%d outside 1..256", fs->n_subints);
  if (fs->n_subbands < 1 || fs->n_baselines < 1 || fs->n_chan < 1)
    return fail(c, XC_E_INVAL, "empty fringe search");
  if (!is_pow2(fs->delay_len) || fs->delay_len < 256 || fs->delay_len > 16384 ||
      fs->delay_len < fs->n_chan)
    return fail(c, XC_E_INVAL, "delay_len=%d: power of two in 256..16384 and >= n_chan",
                fs->delay_len);
  if (!is_pow2(fs->rate_len) || fs->rate_len < fs->n_subints || fs->rate_len > 1024)
    return fail(c, XC_E_INVAL, "rate_len=%d: power of two in n_subints..1024", fs->rate_len);
  if (fs->delay_win < 0 || fs->rate_win < 0) return fail(c, XC_E_INVAL, "negative window");
  if (!(fs->chan_width_hz > 0.0) || !(fs->t_int_s > 0.0))
    return fail(c, XC_E_INVAL, "chan_width_hz and t_int_s must be > 0");
  if ((long)fs->n_subbands * fs->n_baselines > 0x7fffffffL)
    return fail(c, XC_E_INVAL, "too many maps");
  return XC_OK;
}

size_t fringe_bytes(const xc_fringe_setup* fs) {
  return align_up((size_t)fs->n_subbands * fs->n_baselines * fs->n_subints * fs->delay_len *
                   sizeof(float2));
}

}  // namespace

extern "C" {

size_t xc_fringe_workspace_bytes(const xc_fringe_setup* fs) {
  if (fringe_validate(nullptr, fs) != XC_OK) return 0;
  return fringe_bytes(fs);
}

int xc_fringe_search(xc_ctx* c, const xc_fringe_setup* fs, const void* vis, void* peaks,
                     void* map, void* workspace, size_t ws_bytes, void* stream_) {
  if (!c) return XC_E_INVAL;
  int rc = fringe_validate(c, fs);
  if (rc != XC_OK) return rc;
  if (!vis || !peaks) return fail(c, XC_E_INVAL, "fringe search: vis or peaks is NULL");
  const size_t need = fringe_bytes(fs);
  if (!workspace || ws_bytes < need)
    return fail(c, XC_E_NOMEM, "workspace %zu bytes < %zu needed", ws_bytes, need);
  hipError_t e = hipSetDevice(c->device);
  if (e != hipSuccess) return hip_fail(c, e, "hipSetDevice");
  hipStream_t stream = (hipStream_t)stream_;
  e = timed(c, XC_K_FRINGE, stream, [&] {
    return launch_fringe(fs, static_cast<const float2*>(vis), static_cast<float2*>(workspace),
                         c->d_tw, static_cast<xc_fringe_peak*>(peaks),
                         static_cast<float2*>(map), stream);
  });
  return e == hipSuccess ? XC_OK : hip_fail(c, e, "fringe search");
}

}  // extern "C"
