// Small kernels: recording ingest (A0), delay/phase model per frame and
// station-pair weights (A1), weight clearing, finalise (A8) and the unpack test tap.
#include <string.h>

#include "xc_launch.h"

namespace xc {

__global__ void k_ingest(const uint32_t* __restrict__ words, int64_t n_frames,
                         uint8_t* __restrict__ ok) {
  const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (f < n_frames) ok[f] = words[f * kFrameWords] == kSync ? 1 : 0;
}

hipError_t launch_ingest(const uint32_t* words, int64_t n_frames, uint8_t* frame_ok,
                         hipStream_t s) {
  if (n_frames <= 0) return hipSuccess;
  const int b = 256;
  const int64_t g = (n_frames + b - 1) / b;
  hipLaunchKernelGGL(k_ingest, dim3((unsigned)g), dim3(b), 0, s, words, n_frames, frame_ok);
  return hipGetLastError();
}

__global__ void k_zero(unsigned long long* __restrict__ p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

hipError_t launch_zero(unsigned long long* p, size_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  size_t g = (n + 255) / 256;
  if (g > 65536) g = 65536;
  hipLaunchKernelGGL(k_zero, dim3((unsigned)g), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

// Write n words of a descriptor, which come in the launch's own arguments, and
// clear nw weights.  No staging buffer lies between the call and its launch, so
// nothing is waited for or reused, and a graph that records the launch records
// the descriptor with it.  A chunk and the other arguments stay below 4 KB; most
// descriptors are one or two chunks.
template <int W>
struct DescChunk {
  uint32_t w[W];
};

template <int W>
__global__ void __launch_bounds__(W)
    k_desc(const DescChunk<W> c, uint32_t* __restrict__ dst, int n,
           unsigned long long* __restrict__ wst, int nw) {
  const int i = threadIdx.x;
  if (i < n) dst[i] = c.w[i];
  for (int k = i; k < nw; k += W) wst[k] = 0;
}

template <int W>
static hipError_t launch_desc_chunk(const uint32_t* src, uint32_t* dst, int n,
                                    unsigned long long* wst, int nw, hipStream_t s) {
  DescChunk<W> c;
  memcpy(c.w, src, n * sizeof(uint32_t));
  hipLaunchKernelGGL(k_desc<W>, dim3(1), dim3(W), 0, s, c, dst, n, wst, nw);
  return hipGetLastError();
}

hipError_t launch_desc(const void* host, void* dst, size_t bytes, unsigned long long* wst, int nw,
                       hipStream_t s) {
  // the host copies the arguments twice, so calls of up to three stations (whose
  // time is the host's) pass 768 bytes: 32.5 us a call, 32.7 with 1 KB (32.9 with a
  // pinned buffer, which has to be kept and waited for)
  constexpr int kSmall = 192, kLarge = 896;
  const uint32_t* h = static_cast<const uint32_t*>(host);
  uint32_t* d = static_cast<uint32_t*>(dst);
  hipError_t e = hipSuccess;
  for (int n = (int)(bytes / sizeof(uint32_t)); n > 0 && e == hipSuccess; nw = 0) {
    const int k = n < kLarge ? n : kLarge;
    e = k <= kSmall ? launch_desc_chunk<kSmall>(h, d, k, wst, nw, s)
                    : launch_desc_chunk<kLarge>(h, d, k, wst, nw, s);
    h += k;
    d += k;
    n -= k;
  }
  return e;
}

// Delay record (subband 0 only) and phase record of frame fl of a block
// starting at frame f0, station s, subband sb; the frame's validity for
// subband 0.
__device__ inline bool delay_phase_records(const DevJob& J, int s, int sb, int64_t f0, int fl,
                                           int nf, DelayRec* __restrict__ drec,
                                           PhaseRec* __restrict__ prec) {
  const DevStation& S = J.st[s];
  const int64_t f = f0 + fl;
  const int64_t num = J.sub_start + f * (int64_t)J.N + (int64_t)(J.N / 2);
  const double t = (double)num / J.fs;
  // one thread per (frame, station, subband): each writes its subband's phase
  // record, the subband-0 thread also the frame's delay record
  prec[((size_t)s * J.n_subbands + sb) * nf + fl] = frame_phase(S, J, sb, t);
  if (sb != 0) return false;
  DelayRec r;
  frame_delay(S, J, f, &r.n_int, &r.d);
  r.base = J.sub_start + f * (int64_t)J.N + r.n_int - S.first_sample;
  const int64_t n_samples = S.n_frames_m5b * (int64_t)J.spf;
  bool ok = r.base >= 0 && r.base + J.N <= n_samples;
  if (ok) {
    // the recording frames of the window: the caller's mask, else their sync
    // words (four loads at a time)
    const int64_t a = r.base / J.spf, b = (r.base + J.N - 1) / J.spf;
    int bad = 0;
    if (S.frame_ok) {
      for (int64_t m = a; m <= b; ++m) bad |= S.frame_ok[m] == 0;
    } else {
      for (int64_t m = a; m <= b; m += 4) {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = S.words[(m + i < b ? m + i : b) * kFrameWords];
#pragma unroll
        for (int i = 0; i < 4; ++i) bad |= w[i] != kSync;
      }
    }
    ok = bad == 0;
  }
  r.valid = ok ? 1 : 0;
  double d1, d2;
  poly_derivs(S.delay_poly, S.poly_deg, t, d1, d2);
  r.rate = (float)d1;
  drec[(size_t)s * nf + fl] = r;
  return ok;
}

// One workgroup: 64-frame chunks (a frame a lane) of every station (a wave each)
// for one subband, as many chunks as its 16 waves have room for.  For subband 0
// the stations' validity masks then meet in LDS and each station pair's count of
// common valid frames is added to its total (wst, integers: exact in any order),
// so that no second launch reads the records back; the chunks of a workgroup
// add once (31250 frames of two stations: one add a chunk made 11.9 us of it).
constexpr int kDelayFrames = 64;
constexpr int kDelayWaves = 16;
__host__ __device__ inline int delay_chunks(int n_stations) {   // of a workgroup
  return n_stations < kDelayWaves ? kDelayWaves / n_stations : 1;
}

__device__ __forceinline__ void delays_chunk(const DevJob& J, int64_t f0, int block, int sb, int nf,
                                             DelayRec* __restrict__ drec,
                                             PhaseRec* __restrict__ prec,
                                             unsigned long long* __restrict__ wst) {
  __shared__ unsigned long long mask[kMaxStations];   // [chunk][station]
  const int S = J.n_stations, chunks = delay_chunks(S);
  const int lane = threadIdx.x & 63, waves = blockDim.x >> 6;
  for (int w = threadIdx.x >> 6; w < S * chunks; w += waves) {
    const int c = w / S, fl = (block * chunks + c) * kDelayFrames + lane;
    const bool ok = fl < nf && delay_phase_records(J, w - c * S, sb, f0, fl, nf, drec, prec);
    const unsigned long long m = __ballot(ok);
    if (lane == 0) mask[w] = m;
  }
  if (sb != 0 || !wst) return;
  __syncthreads();
  for (int p = threadIdx.x; p < S * S; p += blockDim.x) {
    const int i = p / S, j = p - i * S;
    if (j < i) continue;
    int n = 0;
    for (int c = 0; c < chunks; ++c) n += __popcll(mask[c * S + i] & mask[c * S + j]);
    if (n) atomicAdd(&wst[p], (unsigned long long)n);
  }
}

__global__ void __launch_bounds__(64 * kDelayWaves)
    k_delays(const DevJob* __restrict__ job, int64_t f0, int nf, DelayRec* __restrict__ drec,
             PhaseRec* __restrict__ prec, unsigned* __restrict__ ctr,
             unsigned long long* __restrict__ wst) {
  if (ctr && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
    ctr[0] = 0u;   // the F stage's task counter
    ctr[1] = 0u;   // the drift-correction pass's
  }
  delays_chunk(*job, f0, blockIdx.x, blockIdx.y, nf, drec, prec, wst);
}

hipError_t launch_delays(const DevJob* job, int n_stations, int n_subbands, int64_t f0, int nf,
                         DelayRec* drec, PhaseRec* prec, unsigned* ctr, unsigned long long* wst,
                         hipStream_t s) {
  const int chunks = delay_chunks(n_stations), frames = chunks * kDelayFrames;
  const dim3 grid((nf + frames - 1) / frames, n_subbands);
  const int waves = n_stations < kDelayWaves ? n_stations * chunks : kDelayWaves;
  hipLaunchKernelGGL(k_delays, grid, dim3(64 * waves), 0, s, job, f0, nf, drec, prec, ctr, wst);
  return hipGetLastError();
}

int delays_fused_blocks(int nf, int n_stations, int n_subbands) {
  const int frames = delay_chunks(n_stations) * kDelayFrames;
  return (nf + frames - 1) / frames * n_subbands;
}

// k_delays over the blocks of a fused round: workgroup -> (item, frame chunk,
// subband).
__global__ void __launch_bounds__(64 * kDelayWaves)
    k_delays_fused(const FusedItem* __restrict__ items, int n_items, unsigned* __restrict__ ctr) {
  const int it = fused_find(items, n_items, (int)blockIdx.x,
                            [](const FusedItem& I) { return I.dblk0; });
  const FusedItem& I = items[it];
  if (ctr && blockIdx.x == 0 && threadIdx.x == 0) {
    ctr[0] = 0u;
    ctr[1] = 0u;
  }
  const int frames = delay_chunks(I.jd.n_stations) * kDelayFrames;
  const int nfb = (I.nf + frames - 1) / frames;
  const int local = (int)blockIdx.x - I.dblk0;
  delays_chunk(I.jd, I.f0, local % nfb, local / nfb, I.nf, I.drec, I.prec, I.wst);
}

hipError_t launch_delays_fused(const FusedItem* items, int n_items, int n_blocks, unsigned* ctr,
                               hipStream_t s) {
  if (n_blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_delays_fused, dim3(n_blocks), dim3(64 * kDelayWaves), 0, s, items,
                     n_items, ctr);
  return hipGetLastError();
}

// Element e of a job's output: the sum of its n_slots FP64 slots over the
// weight of its station pair (W = 0 -> 0); the k = 0 element also writes W.
__device__ inline void finalise_elem(const double2* __restrict__ vacc, int n_slots,
                                     size_t slot_stride, const unsigned long long* __restrict__ wst, int S,
                                     int P, int M, float2* __restrict__ vis,
                                     float* __restrict__ weight, int nbl, int n_chan, size_t e) {
  const size_t row = e / n_chan;          // sb * nbl + bl
  const int k = (int)(e - row * n_chan);
  const int bl = (int)(row % nbl);
  int i = 0, rem = bl;                    // bl -> (i, j), row-major upper triangle
  while (rem >= M - i) {
    rem -= M - i;
    ++i;
  }
  const int j = i + rem;
  const double w = (double)wst[(i / P) * S + (j / P)];
  double2 a = vacc[e];
  // fixed slot order; the loads of eight slots are issued together, of 32 while
  // there are that many (a job of few channels and baselines can have over a hundred)
  int q = 1;
  for (; q + 32 <= n_slots; q += 32) {
    double2 b[32];
#pragma unroll
    for (int u = 0; u < 32; ++u) b[u] = vacc[e + (size_t)(q + u) * slot_stride];
#pragma unroll
    for (int u = 0; u < 32; ++u) {
      a.x += b[u].x;
      a.y += b[u].y;
    }
  }
  for (; q + 8 <= n_slots; q += 8) {
    double2 b[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) b[u] = vacc[e + (size_t)(q + u) * slot_stride];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      a.x += b[u].x;
      a.y += b[u].y;
    }
  }
  for (; q < n_slots; ++q) {
    const double2 b = vacc[e + (size_t)q * slot_stride];
    a.x += b.x;
    a.y += b.y;
  }
  vis[e] = w > 0.0 ? make_float2((float)(a.x / w), (float)(a.y / w)) : make_float2(0.f, 0.f);
  if (k == 0) weight[row] = (float)w;
}

__global__ void k_finalise(const double2* __restrict__ vacc, int n_slots, size_t slot_stride,
                           const unsigned long long* __restrict__ wst, int S, int P, int M,
                           float2* __restrict__ vis, float* __restrict__ weight, int nbl,
                           int n_chan, size_t total) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  finalise_elem(vacc, n_slots, slot_stride, wst, S, P, M, vis, weight, nbl, n_chan, e);
}

constexpr int kFinaliseThreads = 256;

int finalise_fused_blocks(int n_subbands, int M, int n_chan) {
  const size_t total = (size_t)n_subbands * (M * (M + 1) / 2) * n_chan;
  return (int)((total + kFinaliseThreads - 1) / kFinaliseThreads);
}

// k_finalise over the jobs of a fused batch: workgroup -> (job, element chunk).
__global__ void __launch_bounds__(kFinaliseThreads)
    k_finalise_fused(const FusedOut* __restrict__ outs, int n_outs) {
  int lo = 0, hi = n_outs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (outs[mid].blk0 <= (int)blockIdx.x)
      lo = mid;
    else
      hi = mid - 1;
  }
  const FusedOut& O = outs[lo];
  const size_t total = (size_t)O.n_sb * O.nbl * O.n_chan;
  const size_t e = (size_t)((int)blockIdx.x - O.blk0) * kFinaliseThreads + threadIdx.x;
  if (e >= total) return;
  finalise_elem(O.vacc, O.n_slots, O.slot_stride, O.wst, O.S, O.P, O.M, O.vis, O.weight, O.nbl,
                O.n_chan, e);
}

hipError_t launch_finalise_fused(const FusedOut* outs, int n_outs, int n_blocks, hipStream_t s) {
  if (n_blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_finalise_fused, dim3(n_blocks), dim3(kFinaliseThreads), 0, s, outs,
                     n_outs);
  return hipGetLastError();
}

hipError_t launch_finalise(const double2* vacc, int n_slots, size_t slot_stride,
                           const unsigned long long* wst, int n_stations, int n_pols, float2* vis,
                           float* weight, int n_subbands, int M, int n_chan, hipStream_t s) {
  const int nbl = M * (M + 1) / 2;
  const size_t total = (size_t)n_subbands * nbl * n_chan;
  const size_t g = (total + 255) / 256;
  hipLaunchKernelGGL(k_finalise, dim3((unsigned)g), dim3(256), 0, s, vacc, n_slots, slot_stride,
                     wst, n_stations, n_pols, M, vis, weight, nbl, n_chan, total);
  return hipGetLastError();
}

// Unpack tap: the same addressing the F stage uses, one thread per sample.
__global__ void k_debug_unpack(const DevJob* __restrict__ job, const DelayRec* __restrict__ drec,
                               int nf, int station, int input, int fl, float* __restrict__ out) {
  const DevJob& J = *job;
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= J.N) return;
  const DelayRec r = drec[(size_t)station * nf + fl];
  if (!r.valid) {
    out[n] = 0.f;
    return;
  }
  const FrameCursor c = make_cursor(J, r.base);
  const uint32_t w = *sample_word(J, J.st[station].words, c, n);
  out[n] = level_of((w >> (sample_shift(J, c, n) + 2 * J.stream_map[input])) & 3u);
}

hipError_t launch_debug_unpack(const DevJob* job, const DelayRec* drec, int nf, int station,
                               int input, int fl, float* out, int N, hipStream_t s) {
  hipLaunchKernelGGL(k_debug_unpack, dim3((N + 255) / 256), dim3(256), 0, s, job, drec, nf,
                     station, input, fl, out);
  return hipGetLastError();
}

}  // namespace xc
