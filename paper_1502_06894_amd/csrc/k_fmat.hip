// F stage on the matrix cores (A2-A5): the first radix-16 pass of every
// transform, with the 2-bit levels as one operand and the fringe rotation in
// the other, then one to three vector passes.
//
// Sample n = t + T e of a frame (T = N / 16, e < 16; t = t' + L j, L = T / J)
// is t + T (e - 8) about the frame centre, so with the fringe phase
// phi0 + phi1 x + phi2 x^2 of the sample x its rotation is
//   exp(2 pi i (phi0 + phi1 t + phi2 t^2)) exp(2 pi i (e - 8) T (phi1 + 2 phi2 t))
//   exp(2 pi i phi2 T^2 (e - 8)^2).
// With t replaced by its mean T / 2 in the middle factor, the pass over e is a
// product with one matrix per (station, subband, group of frames) for all t
// and all pols:
//   U[k1][t] = sum_e A[k1][e] q[t + T e],
//   A[k1][e] = exp(2 pi i ((e - 8) a1 + (e - 8)^2 a2 - e k1 / 16)),
// q the real levels.  What the replacement leaves out is 2 phi2 (t - T/2) T
// (e - 8); the host takes this path only where that stays below 3e-8 turns
// (fstage_matrix_ok), the size of an FP32 phase's rounding.  The other phases
// are products of per-lane phasors: with k = k1 + 16 k2 + R kr (R = 16 J), t'
// being one lane's column,
//   P_j[k1] = z_j(t') exp(2 pi i k1 ((d - t') / N - j / R))   before the DFT over j,
//   K2[k2]  = exp(2 pi i 16 k2 (d - t') / N)                  after it,
// where d is the fractional delay (the output bins' factor exp(2 pi i k d / N)
// is split over k1, k2 and kr).
//
// The product runs on FP16 MFMA 32x32x16 with A as two FP16 terms and the
// levels as exact signs (see kScaleX): an FP32 MFMA would take the vector
// units' own multipliers (measured: 64 cycles for 16 samples a lane, nothing
// else issued meanwhile, 31.5 ms for the F stage of a ten-station 4 s scan
// against 28.5 for the vector kernel), the FP16 one an eighth of that.
//
// A wave owns four 32-column tiles (32 complex values a lane): eight frames at
// N = 256, four at 512, two at 1024, one at 2048, and 2 / 4 / 8 waves share a
// frame at 4096 / 8192 / 16384.  Up to N = 2048 the one remaining pass over t'
// is a 16- or 32-point DFT in a lane, so a frame takes one exchange, through the
// wave's own LDS rows and without a barrier (the vector kernel: two or three).
// Above, lane = the row k1 + 16 k2: both remaining passes address LDS without
// conflicts.  Four waves share a matrix; it is formed once per subband.
//
// At N = 32768 the first radix is 32 (T = N / 32, e < 32), in two passes of 16 k1
// over the same codes: a pass's exchange fits LDS, and its stores are whole
// 128-byte lines.  (Folding the frame's halves into two 16384-point transforms,
// as the vector kernel does, writes every second channel: 16 384 channels of 12
// stations 1332 us a call against 1124.)
//
// Bound by vector issue, at the clock that the chip holds (1.75-1.9 GHz here,
// 1.93-2.0 in the vector kernel): 39 VALU instructions per station-sample at
// N = 2048 (vector kernel: 44 dual-pol, 58 single-pol), LDS cycles 0.36x.
// Whole calls of 8 x 4 inputs, 2^24 samples each: N = 512 dual-pol 1.48 ->
// 1.03 ms, 2048 1.29 -> 1.05, 8192 1.50 -> 1.24, 16384 1.69 -> 1.23,
// 32768 2.00 -> 1.32; the ten-station
// 4 s scan (N = 2048): F 28.5 -> 26.6 ms.  Its spectra are 2-4e-7 of their RMS
// from the oracle's (vector kernel: 0.5-2e-6).
// The gain shrinks where the vector kernel loads a station's words once for more
// than four inputs.  Whole calls against the vector kernel's, 2^24 to 2^26 samples
// an input: N = 256 0.94-1.01 up to four inputs a station, 0.98-1.06 single-pol and
// 1.01-1.10 dual-pol above; 4096 0.95-1.02, dual-pol above eight inputs 1.03-1.04;
// other lengths 0.70-0.96.  It stays the default there for its accuracy: visibilities
// 1.6e-7 from 64 bits at N = 256 (vector 1.3e-6), 4.0e-7 at 4096 (1.0e-6).
#include <atomic>

#include "xc_fft.h"
#include "xc_launch.h"
#include "xc_spec.h"

namespace xc {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// Shape of an N-point frame's transform; MATS matrices (the drift pass: two).
template <int N, int MATS = 1>
struct MGeom {
  // first radix: 16, or 32 at N = 32768, half of whose outputs k1 a pass (two
  // passes over the same codes; a pass's 16-channel runs are whole lines)
  static constexpr int RAD = N > 16384 ? 32 : 16;
  static constexpr int HH = RAD / 16;                       // passes
  static constexpr int KG = RAD / 8;                        // MFMA steps over the samples e
  static constexpr int T = N / RAD;                         // columns of a frame
  static constexpr int CPF = T < 32 ? T : 32;               // ... in one tile
  static constexpr int FPT = 32 / CPF;                      // frames per tile
  static constexpr int J = T / CPF < 4 ? T / CPF : 4;       // tiles of a frame in a wave
  static constexpr int NF = 4 / J;                          // frames per lane
  static constexpr int FPW = FPT * NF;                      // frames per wave
  static constexpr int WPF = T / (CPF * J);                 // waves per frame
  static constexpr int R = RAD * J;                         // radix of pass 1 with the DFT over j
  static constexpr int L = N / R;                           // points left
  static constexpr int ROWS = WPF > 1 ? 16 * J : FPW * R;       // LDS rows of a wave (frame)
  static constexpr int RS = L + 2;                          // row stride: 8-byte reads, no conflicts
  static constexpr int WAVES = WPF > 4 ? WPF : 4;           // waves per workgroup
  static constexpr int UNITS = WAVES / WPF;                 // waves or groups of WPF, with own rows
  static constexpr int FPG = UNITS * FPW;                   // frames per workgroup
  static constexpr int WG = 64 * WAVES;
  // WPF > 1: L = KB x KA, pass 2 of radix KB over tb (t' = ta + KA tb), pass 3 of radix KA
  static constexpr int KA = L >= 256 ? 16 : 8;
  static constexpr int KB = L / KA;
  static constexpr int unit_f = ROWS * RS;                  // floats of a unit's rows
  static constexpr int fd_n = WPF > 1 ? 16 : FPW * (ROWS > 64 ? 8 : 16);   // a wave's bin phasors
  // LDS: the matrix (4 KB; 8 for radix 32), the units' rows, the waves' phasors
  static constexpr size_t lo_off = (size_t)KG * 1024;       // its lower terms
  static constexpr size_t rows_off = 2 * lo_off * MATS;
  static_assert(WAVES >= RAD / 4, "a wave forms four columns of the matrix");
  static constexpr size_t fd_off = rows_off + (size_t)UNITS * unit_f * sizeof(float);
  // WPF > 1: pass-2 twiddles exp(-2 pi i ta kb / L), [ta][kb] (LDS broadcasts: as scalar
  // operands they overflow the SGPRs, whose spills are vector instructions)
  static constexpr size_t tw_off = fd_off + (size_t)WAVES * fd_n * sizeof(float2);
  static constexpr size_t lds_bytes = tw_off + (WPF > 1 ? (size_t)L * sizeof(float2) : 0);
  // waves per SIMD asked of the compiler: four (128 registers) leave the short transforms,
  // with several frames a lane, spilling: 256-point jobs 1.16 of their F stage's time
  // at two; 2048 and 16384 points 0.99 and 0.85
  // (the drift pass, with twice the accumulators: two at every length; asked for three
  // it spills, 256- and 512-point drift jobs 1.07 and 1.12 of their time, 16384 1.10)
  static constexpr int EU = N <= 1024 || MATS > 1 ? 2 : 4;
};

// x - round(x) as float: |result| <= 1/2 (half the rounding error of [0, 1))
__device__ inline float frac_c(double x) { return (float)(x - rint(x)); }
__device__ inline float2 phasor_c(double x) { return phasor_turns(frac_c(x)); }

// LDS written by other lanes of the same wave: DS operations of a wave stay in
// order, so only the compiler has to keep them so.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The levels as signs: with x, y = +-1 for the upper and lower code bit (offset
// binary 0 .. 3) the level is 2.16795 x + 1.16795 y (3.3359 = their sum, 1 their
// difference), so q A is a product of FP16 signs, exact, with two multiples of
// A, each split into two FP16 terms.  Of the product's 24 bits a quarter of the
// entries lose the last one: 4.8e-8 of the entries' RMS, where one FP32 rounding is
// 2.8e-8.  (A third term would hold the bit for half as many MFMAs again; with this
// pass's fewer rounded steps the spectra are closer to 64 bits than the vector
// kernel's all the same, see the top.)  kScaleA keeps the lower terms out of FP16's
// subnormals; a set bit becomes a negative sign, hence the minus.
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2 __attribute__((ext_vector_type(2)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
constexpr float kScaleA = 4096.0f;
constexpr float kScaleX = (float)(-4096.0 * ((double)3.3359f + 1.0) / 2.0);
constexpr float kScaleY = (float)(-4096.0 * ((double)3.3359f - 1.0) / 2.0);
__device__ inline uint32_t code_signs(uint32_t x, uint32_t one) {   // both halves' signs, as +-1
  return (x & 0x80008000u) | one;
}

// x = hi + lo, or one bit less than x.  The product and the upper term are each made
// once: fused into the conversion, the product would round to another upper
// term than the one subtracted, an FP16 ulp off, for some of the values.
__device__ inline half2 split_f16(float x) {
  __asm__ volatile("" : "+v"(x));
  _Float16 h = (_Float16)x;
  __asm__ volatile("" : "+v"(h));
  return half2{h, (_Float16)(x - (float)h)};
}

typedef const __attribute__((address_space(1))) unsigned char* GlobalBytes;

// exp(-2 pi i j / R), j < 4
template <int R>
__device__ inline float2 tw_const(int j) {
  constexpr float c[7] = {1.f, 0.99879545620517241f, 0.99518472667219693f, 0.98917650996478101f,
                          0.98078528040323043f, 0.f, 0.95694033573220882f};
  constexpr float s[7] = {0.f, 0.049067674327418015f, 0.098017140329560604f, 0.14673047445536175f,
                          0.19509032201612828f, 0.f, 0.29028467725446233f};
  const int q = j * (128 / R);   // (j < J, which is 1, 2, 4, 4 at R = 16, 32, 64, 128: q <= 6)
  return make_float2(c[q], -s[q]);
}

// exp(2 pi i (d - t) / N), |d| <= 1/2, N >= 256: the table's entry for t turned by a small angle
template <int N>
__device__ inline float2 bin_step(double d, int t, const float2* __restrict__ tw) {
  const float a = (float)d * (float)(6.283185307179586476925 / N), a2 = a * a;   // |a| <= 0.0123
  const float2 w = tw[t * (kTwiddleN / N)];
  const float cm = a2 * fmaf(a2, 1.f / 24.f, -0.5f), si = a * fmaf(a2, -1.f / 6.f, 1.f);
  return make_float2(fmaf(w.x, cm, fmaf(-w.y, si, w.x)), fmaf(w.y, cm, fmaf(w.x, si, w.y)));
}

// Keeps the compiler from moving work on these values across this point
// (interleaved transforms would hold both's temporaries in registers).
template <int K>
__device__ inline void pin(float2 (&v)[K]) {
#pragma unroll
  for (int i = 0; i < K; i += 4)
    __asm__ volatile("" : "+v"(v[i].x), "+v"(v[i].y), "+v"(v[i + 1].x), "+v"(v[i + 1].y),
                          "+v"(v[i + 2].x), "+v"(v[i + 2].y), "+v"(v[i + 3].x), "+v"(v[i + 3].y));
}

// 16 of 32 DFT outputs (m < 16) of x[2 i] = a[i], x[2 i + 1] = b[i], in a.
__device__ inline void dft32_half(float2 (&a)[16], float2 (&b)[16]) {
  constexpr float c[16] = {1.f, 0.98078528040323043f, 0.92387953251128674f, 0.83146961230254524f,
                           0.70710678118654757f, 0.55557023301960218f, 0.38268343236508978f,
                           0.19509032201612828f, 0.f, -0.19509032201612828f, -0.38268343236508978f,
                           -0.55557023301960218f, -0.70710678118654757f, -0.83146961230254524f,
                           -0.92387953251128674f, -0.98078528040323043f};
  constexpr float s[16] = {0.f, 0.19509032201612828f, 0.38268343236508978f, 0.55557023301960218f,
                           0.70710678118654757f, 0.83146961230254524f, 0.92387953251128674f,
                           0.98078528040323043f, 1.f, 0.98078528040323043f, 0.92387953251128674f,
                           0.83146961230254524f, 0.70710678118654757f, 0.55557023301960218f,
                           0.38268343236508978f, 0.19509032201612828f};
  Dft<16>::run(a);
  pin(a);   // one half's temporaries at a time
  pin(b);
  Dft<16>::run(b);
  pin(b);
#pragma unroll
  for (int m = 0; m < 16; ++m)
    a[m] = m == 0   ? cadd(a[0], b[0])
           : m == 8 ? cadd(a[8], mul_mi(b[8]))
                    : make_float2(fmaf(b[m].x, c[m], fmaf(b[m].y, s[m], a[m].x)),
                                  fmaf(b[m].y, c[m], fmaf(-b[m].x, s[m], a[m].y)));
}

constexpr int kMatInputs = 4;   // inputs of a task

// What the kernel writes besides the spectrum types: the delay-drift correction,
// run after the regular pass on the stations that ask for it.  The window is
// weighted by the ramp n - N / 2 = t + T (e - RAD / 2), so the first pass is t times
// the regular product plus T times one with the matrix weighted by e - RAD / 2,
// and the stored spectrum Y becomes (1 - rho) Y + (2 pi i rho k / N) Yr.
// The vector kernel's drift pass likewise transforms twice, from single phasors.
// Jobs of 5 stations (one corrected), 2 subbands, 2 polarisations and 2^23 samples
// an input, whole, with the vector kernel's drift pass and with this one: 256 points 476 -> 445 us, 512 453 -> 419, 1024 443 -> 405, 2048 443 -> 408,
// 8192 521 -> 508, 16384 605 -> 520 (4096: matrix_rate_ok).
constexpr int kOutRate = 3;

__device__ __forceinline__ void add_drift(float2* p, float2 yr, float rho, float k_over_n) {
  const float2 old = *p;
  const float a = 6.28318530717958648f * rho * k_over_n;
  *p = make_float2((1.0f - rho) * old.x - a * yr.y, (1.0f - rho) * old.y + a * yr.x);
}

// One task: station s, frames fg .. fg + FPG - 1 (this wave: f0 ..), inputs
// in_lo .. in_hi - 1 (at most kMatInputs; input = subband, pol).  wave: its
// number in the workgroup, w: its place in its frame (0 for N <= 2048).
template <int N, int OUT>
__device__ __forceinline__ void fmat_task(const DevJob& Jb, const DelayRec* __restrict__ drec,
                                          const PhaseRec* __restrict__ prec,
                                          void* __restrict__ spec,
                                          const int8_t* __restrict__ scale_exp, int nf, int s,
                                          int fg, int f0, int in_lo, int in_hi, int wave, int w,
                                          unsigned char* lds, float* rows, float2* fdt,
                                          const float2* __restrict__ tw) {
  constexpr bool RATE = OUT == kOutRate, F32 = RATE || OUT == kOutF32;
  using G = MGeom<N, RATE ? 2 : 1>;
  constexpr int RAD = G::RAD, KG = G::KG;
  constexpr int T = G::T, J = G::J, NF = G::NF, L = G::L, RS = G::RS, R = G::R, WPF = G::WPF;
  constexpr int RPL = WPF > 1 ? 1 : G::ROWS / 64;   // rows per lane after the exchange
  constexpr int NB = WPF > 1 ? 32 / G::KA : 1;      // WPF > 1: last-pass butterflies per lane
  const int P = Jb.n_pols, M = Jb.M, n_chan = Jb.n_chan, n_sb = Jb.n_subbands;
  const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
  const int tp = (WPF > 1 ? 32 * w : 0) + (c & (G::CPF - 1));   // this lane's column t'
  uint32_t one = 0x3C003C00u;          // (1, 1) in FP16, kept in a register: and-or is one instruction
  __asm__ volatile("" : "+v"(one));

  // The lane's samples e = 2 i + h of its four tiles: their codes, packed per
  // input (i < 8: tiles 0, 1 and 2, 3, then i >= 8; sample i of tile q: bits
  // 8 (q & 1) + 2 (i % 8 >> 1) of half i & 1), and the frames' phasors
  uint32_t code[kMatInputs][KG] = {};
  float2 W1[NF], K2[NF][J];
  float on[NF];                        // the levels' scale, or 0 for an invalid frame
  GlobalBytes wb[NF];                  // the windows' first recording frames
  uint32_t pb[NF];                     // ... and the lanes' first payload bytes there
  int sh0[NF];
  const int spw = Jb.spw_log2, spf = Jb.spf;
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    const int fl = f0 + i * G::FPT + (G::FPT > 1 ? c / G::CPF : 0);
    DelayRec r;
    r.valid = 0;
    r.d = 0.0;
    r.base = 0;
    if (fl < nf) r = drec[(size_t)s * nf + fl];
    on[i] = r.valid ? 1.0f / kScaleA : 0.0f;
    W1[i] = bin_step<N>(r.d, tp, tw);
#pragma unroll
    for (int k = 1; k < J; ++k) K2[i][k] = phasor_c((double)(RAD * k) * ((r.d - (double)tp) / N));
    // recording frame of the window start and the offset inside it
    int64_t fm = (int64_t)((double)r.base * (1.0 / (double)spf));
    int64_t in = r.base - fm * spf;
    if (in < 0) {
      in += spf;
      --fm;
    } else if (in >= spf) {
      in -= spf;
      ++fm;
    }
    wb[i] = (GlobalBytes)(Jb.st[s].words + fm * kFrameWords + kHeaderWords);
    const int ip = (int)in + tp + T * h;
    pb[i] = ((uint32_t)ip >> spw) * 4;
    sh0[i] = 2 * (ip & ((1 << spw) - 1)) * Jb.C;
  }
  const int n_in = in_hi - in_lo;
#pragma unroll
  for (int eb = 0; eb < RAD / 16; ++eb) {
    uint32_t wv[4][8];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
      for (int e = 0; e < 8; ++e) wv[q][e] = 0u;
      if (on[q / J] != 0.f) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          // payload byte of the window (T and L are whole numbers of words), and
          // 16 header bytes more per recording frame passed: x / 10000 =
          // floor(x 429497 / 2^32) for multiples of 4 below 2^19
          const uint32_t b =
              pb[q / J] + (uint32_t)(((L * (q % J) + 2 * T * (8 * eb + e)) >> spw) * 4);
          __builtin_assume(b < (1u << 19));
          const uint32_t k = (uint32_t)(((uint64_t)b * 429497u) >> 32);
          wv[q][e] =
              *(const __attribute__((address_space(1))) uint32_t*)(wb[q / J] + (b + 16 * k));
        }
      }
    }
#pragma unroll
    for (int k = 0; k < kMatInputs; ++k)
      if (k < n_in) {
        const int map2 = 2 * Jb.stream_map[in_lo + k];
#pragma unroll
        for (int m = 0; m < 32; ++m) {
          // two bits in at the top: 16 times, so the first ends at the bottom
          const int q = 2 * (m >> 4) + ((m >> 2) & 1), e = 2 * (m & 3) + ((m >> 3) & 1);
          uint32_t& cw = code[k][2 * eb + (m >> 4)];
          cw = __builtin_amdgcn_alignbit(wv[q][e] >> (sh0[q / J] + map2), cw, 2);
        }
      }
  }

  // fractional-delay phasors of the kept output bins' last digit, exp(2 pi i kr d / L):
  // N <= 2048 of each frame (kr = m), above of the wave's kr = kb + KB ka; one per lane
  if constexpr (WPF == 1) {
    constexpr int K = 16 / RPL;
    if (lane < G::FPW * K) {
      const int fl = min(f0 + lane / K, nf - 1);
      fdt[lane] = phasor_c((double)(lane % K) * (drec[(size_t)s * nf + fl].d * (1.0 / L)));
    }
  } else if (lane < 16) {
    const int i = lane / (G::KA / 2), ka = lane % (G::KA / 2), fl = min(f0, nf - 1);
    const int kb = 2 * w + (i & 1) + (G::KB / 2) * (i >> 1);
    fdt[lane] = phasor_c((double)(kb + G::KB * ka) * (drec[(size_t)s * nf + fl].d * (1.0 / L)));
  }

#pragma unroll 1
  for (int sb = in_lo / P; sb * P < in_hi; ++sb) {
    const int p_lo = max(in_lo - sb * P, 0), p_hi = min(in_hi - sb * P, P);
    const PhaseRec* ph = prec + ((size_t)s * n_sb + sb) * nf;
#pragma unroll 1
    for (int hh = 0; hh < G::HH; ++hh) {
      __syncthreads();   // the previous matrix has been read
      if (wave < RAD / 4) {
        // the matrix: wave p forms the columns e = 2 i + h of i = 2 p, 2 p + 1
        const PhaseRec pa = ph[fg];
        const double phi1 =
            G::FPG > 1 ? 0.5 * (pa.phi1 + ph[min(fg + G::FPG - 1, nf - 1)].phi1) : pa.phi1;
        double a1 = (double)T * (phi1 + pa.phi2 * (double)T);
        a1 -= rint(a1);
        const double a2 = pa.phi2 * (double)T * (double)T;
        // matrix row of this lane: register i of the product holds rows 8 (i / 4) +
        // 4 h + i % 4, which are given k1 = 8 h + i / 2 and re / im = i % 2
        const int row_k1 = 16 * hh + 8 * ((c >> 2) & 1) + 2 * (c >> 3) + ((c >> 1) & 1);
        const double row_im = (c & 1) ? 0.25 : 0.0;    // sin x = cos(x - 1/4 turn)
        unsigned char* o = lds + (wave >> 1) * 1024 + lane * 16 + (wave & 1) * 8;
        float a[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int e = 2 * (2 * wave + i) + h;
          const double ee = (double)(e - RAD / 2);
          const double off = (double)((e * row_k1) & (RAD - 1)) * (1.0 / RAD) + row_im;
          a[i] = __builtin_amdgcn_cosf(frac_c(fma(ee, fma(ee, a2, a1), -off)));
        }
#pragma unroll
        for (int m = 0; m < (RATE ? 2 : 1); ++m) {
          half4 hi, lo;                                // upper code bit of both, lower of both
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            // (the drift pass's second matrix: the samples' ramp e - RAD / 2, over RAD / 2)
            const float b =
                m == 0 ? a[i] : a[i] * ((float)(2 * (2 * wave + i) + h - RAD / 2) * (2.f / RAD));
            const half2 x = split_f16(b * kScaleX), y = split_f16(b * kScaleY);
            hi[i] = x[0];
            hi[i + 2] = y[0];
            lo[i] = x[1];
            lo[i + 2] = y[1];
          }
          *reinterpret_cast<half4*>(o + 2 * m * G::lo_off) = hi;
          *reinterpret_cast<half4*>(o + (2 * m + 1) * G::lo_off) = lo;
        }
      }
      float2 z[NF], S[NF];
#pragma unroll
      for (int i = 0; i < NF; ++i) {
        const int fl = min(f0 + i * G::FPT + (G::FPT > 1 ? c / G::CPF : 0), nf - 1);
        const PhaseRec pr = ph[fl];
        const double x = (double)tp, d = drec[(size_t)s * nf + fl].d;
        const double k0 = (double)(16 * hh + 8 * h);   // k1 of the lane's first row
        z[i] = phasor_c(fma(fma(pr.phi2, x, pr.phi1), x, pr.phi0) + k0 * ((d - x) / N));
        z[i].x *= on[i];
        z[i].y *= on[i];
        // step of j: t grows by L, for k1 = k0
        if constexpr (J > 1)
          S[i] = phasor_c((double)L * (pr.phi1 + 4.0 * pr.phi2 * (double)L) - k0 / R);
      }
      __syncthreads();
#pragma unroll 1
      for (int p = p_lo; p < p_hi; ++p) {
        const int k_in = sb * P + p - in_lo;
        uint32_t cd[KG];
#pragma unroll
        for (int i = 0; i < KG; ++i) {
          cd[i] = code[0][i];
#pragma unroll
          for (int k = 1; k < kMatInputs; ++k) cd[i] = k_in == k ? code[k][i] : cd[i];
        }
        float2 v[4][8];
#pragma unroll
        for (int i = 0; i < NF; ++i) {
          float2 zj = z[i];
#pragma unroll
          for (int j = 0; j < J; ++j) {
            f32x16 acc = {}, acc2 = {};
#pragma unroll
            for (int g = 0; g < KG; ++g) {
              uint4 b;
              {
                const uint32_t cw = cd[2 * (g >> 1) + ((i * J + j) >> 1)];
                const int pos = 8 * ((i * J + j) & 1) + 4 * (g & 1);
                b.x = code_signs(cw << (14 - pos), one);
                b.y = code_signs(cw << (15 - pos), one);
                b.z = code_signs(pos == 12 ? cw : cw << (12 - pos), one);
                b.w = code_signs(cw << (13 - pos), one);
              }
              const half8 B = __builtin_bit_cast(half8, b);
              const half8* am = reinterpret_cast<const half8*>(lds) + g * 64 + lane;
              acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(am[64 * KG], B, acc, 0, 0, 0);
              acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(am[0], B, acc, 0, 0, 0);
              if constexpr (RATE) {
                acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(am[192 * KG], B, acc2, 0, 0, 0);
                acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(am[128 * KG], B, acc2, 0, 0, 0);
              }
            }
            if constexpr (RATE) {
              // sample n - N / 2 = t + T (e - RAD / 2)
              const float t = (float)(tp + L * j);
#pragma unroll
              for (int k = 0; k < 16; ++k) acc[k] = fmaf(t, acc[k], (float)(N / 2) * acc2[k]);
            }
            // P[k] = zj Wj^k
            float2 Wa = W1[i];
            __asm__ volatile("" : "+v"(Wa.x), "+v"(Wa.y), "+v"(zj.x), "+v"(zj.y));   // (per tile)
            if (j > 0) Wa = cmul(Wa, tw_const<R>(j));
            const float2 Wb = cmul(Wa, Wa);
            float2 pa = zj, pb = cmul(zj, Wa);
#pragma unroll
            for (int k = 0; k < 8; k += 2) {
              v[i * J + j][k] = cmul(make_float2(acc[2 * k], acc[2 * k + 1]), pa);
              v[i * J + j][k + 1] = cmul(make_float2(acc[2 * k + 2], acc[2 * k + 3]), pb);
              if (k < 6) {
                pa = cmul(pa, Wb);
                pb = cmul(pb, Wb);
              }
            }
            if (j + 1 < J) zj = cmul(zj, S[i]);
            __builtin_amdgcn_sched_barrier(0);   // one tile's operands in registers at a time
          }
          // DFT over j and its twiddles; row (frame, k1 + 16 k2), column t'
          if constexpr (J > 1) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              float2 u[J];
#pragma unroll
              for (int j = 0; j < J; ++j) u[j] = v[i * J + j][k];
              Dft<J>::run(u);
#pragma unroll
              for (int j = 0; j < J; ++j) v[i * J + j][k] = j == 0 ? u[0] : cmul(u[j], K2[i][j]);
            }
          }
        }
        const int m_in = s * P + p;
        // exchanges: rows of real, then of imaginary parts (half the LDS of complex rows)
        float* o = rows + ((G::FPT > 1 ? c / G::CPF : 0) * R + 8 * h) * RS + tp;
        constexpr int IS = G::FPT * R * RS;     // a tile's (frame's) rows
        auto put = [&](auto part) {
#pragma unroll
          for (int i = 0; i < NF; ++i)
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
              for (int k = 0; k < 8; ++k) o[i * IS + (k + 16 * j) * RS] = part(v[i * J + j][k]);
        };
        auto re = [](float2 x) { return x.x; };
        auto im = [](float2 x) { return x.y; };
        if constexpr (WPF == 1) {
          float xr[RPL][L];
          put(re);
          wave_sync();
#pragma unroll
          for (int q = 0; q < RPL; ++q)
#pragma unroll
            for (int i = 0; i < L / 2; ++i) {
              const float2 y = reinterpret_cast<const float2*>(rows + (lane + 64 * q) * RS)[i];
              xr[q][2 * i] = y.x;
              xr[q][2 * i + 1] = y.y;
            }
          wave_sync();
          put(im);
          wave_sync();
#pragma unroll
          for (int q = 0; q < RPL; ++q) {
            const int rho = lane + 64 * q;
            const float2* x = reinterpret_cast<const float2*>(rows + rho * RS);
            float2 a[16], b[16];
            constexpr int K = 16 / RPL;     // kept outputs of the row
#pragma unroll
            for (int i = 0; i < L / 2; ++i) {
              const float2 y = x[i];
              if constexpr (L == 32) {
                a[i] = make_float2(xr[q][2 * i], y.x);
                b[i] = make_float2(xr[q][2 * i + 1], y.y);
              } else {
                a[2 * i] = make_float2(xr[q][2 * i], y.x);
                a[2 * i + 1] = make_float2(xr[q][2 * i + 1], y.y);
              }
            }
            if constexpr (L == 32) {
              dft32_half(a, b);
            } else {
              pin(a);
              Dft<16>::run(a);
              pin(a);
            }
            const int fl = f0 + rho / R, kap = rho & (R - 1);
            const float2* fdl = fdt + rho / R * K;
            if (fl < nf) {
              // bin kap + R m (low precision: channel-blocked, lp_index)
              const size_t row = F32 ? ((size_t)(sb * nf + fl) * M + m_in) * n_chan + kap
                                                : (size_t)(sb * nf + fl) * M * n_chan +
                                                      (m_in + (kap >> 4) * M) * 16 + (kap & 15);
              uint2 ex[2];
              if constexpr (!F32) {
                // bin kap + R m: exponent byte m / (N / 16 / R) of the word at its remainder
                const uint2* exw = reinterpret_cast<const uint2*>(
                    scale_exp + ((size_t)sb * M + m_in) * n_chan);
                ex[0] = exw[kap];
                ex[1] = L == 32 ? exw[kap + R] : ex[0];
              }
              const float rho = RATE ? drec[(size_t)s * nf + fl].rate : 0.f;
#pragma unroll
              for (int m = 0; m < K; ++m) {
                const float2 y = cmul(a[m], fdl[m]);
                if constexpr (RATE) {
                  add_drift(static_cast<float2*>(spec) + row + R * m, y, rho,
                            (float)(kap + R * m) / (float)N);
                } else if constexpr (OUT == kOutF32) {
                  put_spec<OUT>(spec, row + R * m, y, 0);
                } else {
                  const int byte = L == 32 ? m >> 1 : m;
                  const uint2 e2 = ex[L == 32 ? m & 1 : 0];
                  const uint32_t ew = byte < 4 ? e2.x : e2.y;
                  put_spec<OUT>(spec, row + R * M * m, y, (int)(ew << (24 - 8 * (byte & 3))) >> 24);
                }
              }
            }
          }
          wave_sync();   // the next input writes the rows
        } else {
          constexpr int KA = G::KA, KB = G::KB, TAW = KA / WPF;
          const float2* tab = reinterpret_cast<const float2*>(lds + G::tw_off) + TAW * w * KB;
          // lane = row k1 + 16 k2; this wave's columns ta = TAW w + a, all tb
          float2 y2[TAW][KB];
          const float2* x = reinterpret_cast<const float2*>(rows + lane * RS + TAW * w);
          put(re);   // (the rows are free: every wave is past its last reads)
          __syncthreads();
#pragma unroll
          for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int a = 0; a < TAW; a += 2) {
              const float2 y = x[(KA * b + a) / 2];
              y2[a][b].x = y.x;
              y2[a + 1][b].x = y.y;
            }
          __syncthreads();
          put(im);
          __syncthreads();
#pragma unroll
          for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int a = 0; a < TAW; a += 2) {
              const float2 y = x[(KA * b + a) / 2];
              y2[a][b].y = y.x;
              y2[a + 1][b].y = y.y;
            }
#pragma unroll
          for (int a = 0; a < TAW; ++a) {
            pin(y2[a]);
            Dft<KB>::run(y2[a]);
            pin(y2[a]);
#pragma unroll
            for (int b = 1; b < KB; ++b) y2[a][b] = cmul(y2[a][b], tab[a * KB + b]);
          }
          // second exchange [ta][kb][row]: this wave's kb, all ta
          float* o2 = rows + TAW * w * KB * 64 + lane;
          const float* x2 = rows + lane;
          float2 u[NB][KA];
          __syncthreads();
#pragma unroll
          for (int a = 0; a < TAW; ++a)
#pragma unroll
            for (int b = 0; b < KB; ++b) o2[(a * KB + b) * 64] = y2[a][b].x;
          __syncthreads();
#pragma unroll
          for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int a = 0; a < KA; ++a)
              u[i][a].x = x2[(a * KB + 2 * w + (i & 1) + (KB / 2) * (i >> 1)) * 64];
          __syncthreads();
#pragma unroll
          for (int a = 0; a < TAW; ++a)
#pragma unroll
            for (int b = 0; b < KB; ++b) o2[(a * KB + b) * 64] = y2[a][b].y;
          __syncthreads();
#pragma unroll
          for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int a = 0; a < KA; ++a)
              u[i][a].y = x2[(a * KB + 2 * w + (i & 1) + (KB / 2) * (i >> 1)) * 64];
          __syncthreads();   // the next input writes the rows
          if (f0 < nf) {
            const size_t row = F32 ? ((size_t)(sb * nf + f0) * M + m_in) * n_chan + 16 * hh +
                                                    RAD * (lane >> 4) + (lane & 15)
                                              : (size_t)(sb * nf + f0) * M * n_chan +
                                                    (m_in + (lane >> 4) * M) * 16 + (lane & 15);
            uint2 ex[2];
            if constexpr (!F32) {
              // bin lane + 64 kr, kr = kb + KB ka: byte kr / (N / 1024) of the word at the remainder
              const uint2* exw =
                  reinterpret_cast<const uint2*>(scale_exp + ((size_t)sb * M + m_in) * n_chan);
#pragma unroll
              for (int i = 0; i < 2; ++i) ex[i] = exw[lane + 64 * ((2 * w + i) & (N / 1024 - 1))];
            }
            const float rho = RATE ? drec[(size_t)s * nf + f0].rate : 0.f;
#pragma unroll
            for (int i = 0; i < NB; ++i) {
              const int kb = 2 * w + (i & 1) + (KB / 2) * (i >> 1);
              pin(u[i]);
              Dft<KA>::run(u[i]);
              pin(u[i]);
#pragma unroll
              for (int a = 0; a < KA / 2; ++a) {
                const float2 y = cmul(u[i][a], fdt[i * (KA / 2) + a]);
                const int kr = kb + KB * a;
                if constexpr (RATE) {
                  add_drift(static_cast<float2*>(spec) + row + R * kr, y, rho,
                            (float)(lane + R * kr) / (float)N);
                } else if constexpr (OUT == kOutF32) {
                  put_spec<OUT>(spec, row + R * kr, y, 0);
                } else {
                  const int byte = kr / (N / 1024);
                  const uint32_t ew = byte < 4 ? ex[i & 1].x : ex[i & 1].y;
                  put_spec<OUT>(spec, row + 64 * M * kr, y,
                                (int)(ew << (24 - 8 * (byte & 3))) >> 24);
                }
              }
            }
          }
        }
      }
    }
  }
}

// The pass-2 twiddles (the first subband's barrier comes before their use).
template <class G>
__device__ __forceinline__ void fmat_tab(unsigned char* lds, const float2* __restrict__ tw) {
  if constexpr (G::WPF > 1) {
    float2* tab = reinterpret_cast<float2*>(lds + G::tw_off);
    for (int i = threadIdx.x; i < G::L; i += G::WG)
      tab[i] = tw[(i / G::KB) * (i % G::KB) * (kTwiddleN / G::L)];
  }
}

// Tasks (station, group of FPG frames, group of ipt inputs), the last
// fastest; a workgroup takes every n-th.  Tasks of full input groups cost the
// same, so they are not fetched from a counter.  Where the number of groups
// divides that of the workgroups, a workgroup would meet the same group of inputs
// in every round, and with a smaller last group (five or six inputs: 4 + 1, 4 + 2)
// half of the workgroups would wait for the others; so the groups turn by one
// each round.  (A frame group's tasks lie in one round then.)  Whole calls, before ->
// with it: 7 stations of 6 inputs, 2^25 samples each, N = 4096 3757 -> 3167 us,
// 16384 4119 -> 3494; 8 stations of 5 inputs, 2^26, N = 2048 5873 -> 5403, 4096
// 6799 -> 6079 (the vector kernel's 6166); equal groups +-0.7 %.
// The drift pass (kOutRate) takes the stations that ask for it, in order.
template <int N, int OUT>
__global__ void __attribute__((amdgpu_flat_work_group_size(1, MGeom<N, OUT == kOutRate ? 2 : 1>::WG),
                               amdgpu_waves_per_eu(MGeom<N, OUT == kOutRate ? 2 : 1>::EU)))
    k_fmat(const DevJob* __restrict__ job, const DelayRec* __restrict__ drec,
           const PhaseRec* __restrict__ prec, const float2* __restrict__ tw,
           void* __restrict__ spec, const int8_t* __restrict__ scale_exp, int nf, int ipt) {
  constexpr bool RATE = OUT == kOutRate;
  using G = MGeom<N, RATE ? 2 : 1>;
  extern __shared__ __attribute__((aligned(16))) unsigned char fmat_lds[];
  const DevJob& J = *job;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int unit = wave / G::WPF;
  float* rows = reinterpret_cast<float*>(fmat_lds + G::rows_off) + unit * G::unit_f;
  float2* fdt = reinterpret_cast<float2*>(fmat_lds + G::fd_off) + wave * G::fd_n;
  fmat_tab<G>(fmat_lds, tw);
  const int n_in = J.n_inputs;
  const int n_ig = (n_in + ipt - 1) / ipt, per_station = (nf + G::FPG - 1) / G::FPG * n_ig;
  int n_stations = J.n_stations;
  if constexpr (RATE) {
    n_stations = 0;
    for (int i = 0; i < J.n_stations; ++i) n_stations += J.st[i].rate_correct ? 1 : 0;
  }
  const int n_tasks = per_station * n_stations;
  const bool turn = gridDim.x % n_ig == 0;
  int shift = 0;
#pragma unroll 1
  for (int task = blockIdx.x; task < n_tasks; task += gridDim.x) {
    int s = task / per_station;
    const int rem = task - s * per_station;
    const int grp = rem / n_ig;
    int ig = rem - grp * n_ig + shift;
    if (ig >= n_ig) ig -= n_ig;
    const int in = ig * ipt;
    if (turn && ++shift == n_ig) shift = 0;
    if constexpr (RATE) {
      int k = s;   // the s-th station that asks for it
      s = -1;
      do {
        ++s;
        k -= J.st[s].rate_correct ? 1 : 0;
      } while (k >= 0);
    }
    fmat_task<N, OUT>(J, drec, prec, spec, scale_exp, nf, s, grp * G::FPG,
                      grp * G::FPG + unit * G::FPW, in, min(in + ipt, n_in), wave, wave % G::WPF,
                      fmat_lds, rows, fdt, tw);
  }
}

// The same tasks over the blocks of many jobs of one FFT length.  A job's tasks begin
// anywhere in a round, so its input groups cannot turn there; where the last one of
// more than kMatInputs inputs is smaller, they come one after the other for each
// station instead (short jobs of fewer inputs in several groups: 0.3 % slower so).  24 jobs of 6
// inputs, 2^20 samples each, as one batch: N = 256 1465 -> 1412 us, 1024 1367 -> 1338,
// 4096 1517 -> 1490, 16384 1812 -> 1776.
template <int N>
__global__ void __attribute__((amdgpu_flat_work_group_size(1, MGeom<N>::WG),
                               amdgpu_waves_per_eu(MGeom<N>::EU)))
    k_fmat_fused(const FusedItem* __restrict__ items_g, int n_items, int n_tasks,
                 const float2* __restrict__ tw) {
  using G = MGeom<N>;
  extern __shared__ __attribute__((aligned(16))) unsigned char fmat_lds[];
  fmat_tab<G>(fmat_lds, tw);
  const FusedItemsK items = fused_const(items_g);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int unit = wave / G::WPF;
  float* rows = reinterpret_cast<float*>(fmat_lds + G::rows_off) + unit * G::unit_f;
  float2* fdt = reinterpret_cast<float2*>(fmat_lds + G::fd_off) + wave * G::fd_n;
#pragma unroll 1
  for (int task = blockIdx.x; task < n_tasks; task += gridDim.x) {
    int lo = 0, hi = n_items - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (items[mid].task0 <= task)
        lo = mid;
      else
        hi = mid - 1;
    }
    const DevJob& J = *(const DevJob*)&items[lo].jd;
    const int nf = items[lo].nf, n_in = J.n_inputs, ipt = items[lo].ipt;
    const int n_ig = (n_in + ipt - 1) / ipt, n_grp = (nf + G::FPG - 1) / G::FPG;
    const int local = task - items[lo].task0;
    const int s = local / (n_grp * n_ig), rem = local - s * n_grp * n_ig;
    const bool outer = n_in > kMatInputs && n_ig * ipt != n_in;
    const int q = rem / (outer ? n_grp : n_ig), r = rem - q * (outer ? n_grp : n_ig);
    const int grp = outer ? r : q, in = (outer ? q : r) * ipt;
    fmat_task<N, kOutF32>(J, items[lo].drec, items[lo].prec, items[lo].spec, nullptr, nf, s,
                          grp * G::FPG, grp * G::FPG + unit * G::FPW, in, min(in + ipt, n_in),
                          wave, wave % G::WPF, fmat_lds, rows, fdt, tw);
  }
}

// Workgroups of a kernel that fill the GPU (per device; set once, callers on
// several host threads may race to set the same value).
template <class K>
hipError_t resident_groups(K kernel, int wg, size_t lds, std::atomic<int> (&cache)[64], int& res) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  res = cache[dev].load();
  if (res) return hipSuccess;
  e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  int per_cu = 0, n_cu = 0;
  if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, wg, lds);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  res = (per_cu > 0 ? per_cu : 1) * (n_cu > 0 ? n_cu : 1);
  cache[dev].store(res);
  return hipSuccess;
}

template <int N, int OUT>
hipError_t launch_fmat_no(const DevJob* job, int n_stations, int n_subbands, int n_pols,
                          const DelayRec* drec, const PhaseRec* prec, const float2* tw, void* spec,
                          const int8_t* scale_exp, int nf, hipStream_t s) {
  using G = MGeom<N, OUT == kOutRate ? 2 : 1>;
  static std::atomic<int> cache[64];
  int res = 0;
  hipError_t e = resident_groups(k_fmat<N, OUT>, G::WG, G::lds_bytes, cache, res);
  if (e != hipSuccess) return e;
  const int ipt = fmat_inputs_per_task(N, n_stations, n_subbands, n_pols, nf);
  const int tasks = fmat_tasks(N, n_stations, n_subbands * n_pols, nf, ipt);
  if (tasks <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_fmat<N, OUT>), dim3(tasks < res ? tasks : res), dim3(G::WG), G::lds_bytes,
                     s, job, drec, prec, tw, spec, scale_exp, nf, ipt);
  return hipGetLastError();
}

template <int N>
hipError_t launch_fmat_n(const DevJob* job, int n_stations, int n_subbands, int n_pols,
                         const DelayRec* drec, const PhaseRec* prec, const float2* tw, void* spec,
                         const int8_t* scale_exp, int nf, int out, hipStream_t s) {
  if constexpr (N > 256)   // (matrix_out_ok)
    if (out == kOutF16)
      return launch_fmat_no<N, kOutF16>(job, n_stations, n_subbands, n_pols, drec, prec, tw, spec,
                                        scale_exp, nf, s);
  if constexpr (matrix_rate_ok(N))
    if (out == kOutRate)
      return launch_fmat_no<N, kOutRate>(job, n_stations, n_subbands, n_pols, drec, prec, tw, spec,
                                         nullptr, nf, s);
  if (out != kOutF32) return hipErrorInvalidValue;
  return launch_fmat_no<N, kOutF32>(job, n_stations, n_subbands, n_pols, drec, prec, tw, spec, scale_exp,
                                    nf, s);
}

template <int N>
hipError_t launch_fmat_fused_n(const FusedItem* items, int n_items, int n_tasks, const float2* tw,
                               hipStream_t s) {
  using G = MGeom<N>;
  static std::atomic<int> cache[64];
  int res = 0;
  hipError_t e = resident_groups(k_fmat_fused<N>, G::WG, G::lds_bytes, cache, res);
  if (e != hipSuccess) return e;
  if (n_tasks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fmat_fused<N>, dim3(n_tasks < res ? n_tasks : res), dim3(G::WG), G::lds_bytes,
                     s, items, n_items, n_tasks, tw);
  return hipGetLastError();
}

}  // namespace

int fmat_frames_per_task(int N) { return N >= 8192 ? 1 : 8192 / N; }

static_assert(MGeom<256>::FPG == 32 && MGeom<2048>::FPG == 4 && MGeom<4096>::FPG == 2 &&
                  MGeom<8192>::FPG == 1 && MGeom<16384>::FPG == 1,
              "fmat_frames_per_task mirrors MGeom");

int fmat_inputs_per_task(int N, int n_stations, int n_subbands, int n_pols, int nf) {
  // A task's words and phasors are set up once for its inputs, at about 0.3 of an
  // input's time (32 stations x 4 inputs of 8192 points: 7.0 ms at four inputs a
  // task, 8.5 at one); few tasks leave the last round of the resident workgroups
  // half empty.  The split of the subbands (down to single pols where all tasks fit
  // one round) that takes the least time, the fewest tasks on a tie.  Planned with
  // 1024 workgroups, the number from 2048 to 8192 points (four waves per SIMD); up to
  // 1024 points 768 are resident, and 512 of eight waves from 16384.
  const int F = fmat_frames_per_task(N);
  const long base = (long)n_stations * ((nf + F - 1) / F);
  int best = 1;
  double best_t = 0.0;
  for (int n = (n_subbands * n_pols + kMatInputs - 1) / kMatInputs; n <= n_subbands; ++n) {
    const int spt = (n_subbands + n - 1) / n;
    if (spt * n_pols > kMatInputs) continue;
    const long rounds = (base * n + 1023) / 1024;
    const double t = (double)rounds * ((double)n_subbands * n_pols / n + 0.3);
    if (best_t == 0.0 || t < 0.97 * best_t) {
      best_t = t;
      best = spt * n_pols;
    }
  }
  return base * n_subbands * n_pols <= 1024 ? 1 : best;
}

int fmat_tasks(int N, int n_stations, int n_inputs, int nf, int ipt) {
  const int F = fmat_frames_per_task(N);
  return n_stations * ((nf + F - 1) / F) * ((n_inputs + ipt - 1) / ipt);
}

hipError_t launch_fmat(int N, const DevJob* job, int n_stations, int n_subbands, int n_pols,
                       const DelayRec* drec, const PhaseRec* prec, const float2* tw, void* spec,
                       const int8_t* scale_exp, int nf, int out, hipStream_t s) {
  switch (N) {
#define XC_MCASE(NN)                                                                          \
  case NN:                                                                                    \
    return launch_fmat_n<NN>(job, n_stations, n_subbands, n_pols, drec, prec, tw, spec, scale_exp, nf, \
                             out, s);
    XC_MCASE(256) XC_MCASE(512) XC_MCASE(1024) XC_MCASE(2048) XC_MCASE(4096) XC_MCASE(8192)
    XC_MCASE(16384)
#undef XC_MCASE
    case 32768:
      if (out != kOutF32) return hipErrorInvalidValue;
      return launch_fmat_no<32768, kOutF32>(job, n_stations, n_subbands, n_pols, drec, prec, tw,
                                            spec, nullptr, nf, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_fmat_rate(int N, const DevJob* job, int n_flagged, int n_subbands, int n_pols,
                            const DelayRec* drec, const PhaseRec* prec, const float2* tw,
                            void* spec, int nf, hipStream_t s) {
  return launch_fmat(N, job, n_flagged, n_subbands, n_pols, drec, prec, tw, spec, nullptr, nf,
                     kOutRate, s);
}

hipError_t launch_fmat_fused(int N, const FusedItem* items, int n_items, int n_tasks,
                             const float2* tw, hipStream_t s) {
  switch (N) {
#define XC_MCASE(NN) \
  case NN: return launch_fmat_fused_n<NN>(items, n_items, n_tasks, tw, s);
    XC_MCASE(256) XC_MCASE(512) XC_MCASE(1024) XC_MCASE(2048) XC_MCASE(4096) XC_MCASE(8192)
    XC_MCASE(16384)
#undef XC_MCASE
    default: return hipErrorInvalidValue;
  }
}

}  // namespace xc
