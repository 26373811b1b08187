// HIP kernels of the F-statistic search path for gfx950.
//
// Per sky position (amortised over the spindown loop, Sect. 2):
//   k_sky_setup     direction, amplitude-modulation coefficients, n.r_0, the
//                   averages A, B, C and the 2F coefficients
//   k_sky_demod     a(t), b(t), Roemer delay, phase demodulation -> za, zb
//   (fstat_sky.hpp) 2x band-limited upsampling and the natural cubic spline through
//                   the upsampled series, evaluated at the detector positions of the
//                   barycentric grid
//   k_decimate      the resampled series at 5/8 of the rate
// Per (sky, spindown) template (the hot loop):
//   k_tmpl_pass_a   spindown chirp fused into the load, column DFTs of the
//                   four-step FFT, inter-pass twiddle
//   k_tmpl_pass_b   row DFTs, 2F for both amplitude series, threshold and
//                   stream compaction (or a store of the 2F spectrum)
//
// An nfft = P*Q point FFT is done in two passes over a P x Q view
// (j = j1 + P j2, k = Q k1 + k2):
//   pass A: for each column j1, Q-point DFT over j2, times W_nfft^(j1 k2),
//           stored transposed as T[k2][j1];
//   pass B: for each row k2, P-point DFT over j1 -> X[Q k1 + k2].
// Each workgroup handles TW adjacent columns (pass A) or rows (pass B) of both
// amplitude series, so global loads and stores move TW contiguous elements.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fstat_fft.hpp"

namespace fstat {

constexpr int NT = 256;  // threads per workgroup (4 wavefronts)

// Earth rotation rate: 2 pi / sidereal day (86164.0905 s).
__host__ __device__ constexpr double sidereal_rate() { return 6.283185307179586476925 / 86164.0905; }

struct SkyParams {
  double nx, ny, nz;           // unit vector towards the source
  double nr0;                  // n . r_0
  double cx0, sx0;             // cos, sin of x_0 = alpha - phi_r
  double ka[5];                // a = ka0 cos2x + ka1 sin2x + ka2 cos x + ka3 sin x + ka4
  double kb[4];                // b = kb0 cos2x + kb1 sin2x + kb2 cos x + kb3 sin x
  double A, B, C;              // <a^2>, <b^2>, <ab>
  double cfa, cfb, cfab;       // 2F = cfa |Fa|^2 + cfb |Fb|^2 + cfab Re(Fa Fb*)
  double pad;
};

struct SegConst {
  int n;            // samples
  int nfft;         // L
  double dt, f_off, sigma2;
  double phi_r;
  double s2g, c2g, sl, cl, s2l, c2l;   // sin, cos of 2 gamma, lat, 2 lat
  double mid;       // phase of the segment's middle sample, (n - 1) / 2 sidereal_rate() dt
  double dir[4];    // |mean over the samples of exp(i m x)|, signed, m = 1 .. 4
  const double* x;  // n
  const double* r;  // 3 n, component-major
};

// Candidate entry as written by the threshold stage; score: bits of the vetting score, not a
// number until there is one.
struct CandEntry {
  int32_t search, segment, sky, fdot_idx, bin, score;
  double twoF;
};
constexpr int32_t NO_SCORE = 0x7fc00000;

// ------------------------------------------------------------------ sky stage
// <p q> over the samples of two antenna functions p_0 cos 2x + p_1 sin 2x + p_2 cos x +
// p_3 sin x + p_4, from the means c[m] + i s[m] of exp(i m x) (index m = 1 .. 4).
__device__ __forceinline__ double antenna_mean(const double* p, const double* q, const double* c, const double* s) {
  return 0.5 * (p[0] * q[0] * (1.0 + c[4]) + p[1] * q[1] * (1.0 - c[4]) + p[2] * q[2] * (1.0 + c[2]) +
                p[3] * q[3] * (1.0 - c[2]) + (p[0] * q[1] + p[1] * q[0]) * s[4] +
                (p[0] * q[2] + p[2] * q[0]) * (c[3] + c[1]) + (p[0] * q[3] + p[3] * q[0]) * (s[3] - s[1]) +
                (p[1] * q[2] + p[2] * q[1]) * (s[3] + s[1]) + (p[1] * q[3] + p[3] * q[1]) * (c[1] - c[3]) +
                (p[2] * q[3] + p[3] * q[2]) * s[2]) +
         (p[0] * q[4] + p[4] * q[0]) * c[2] + (p[1] * q[4] + p[4] * q[1]) * s[2] +
         (p[2] * q[4] + p[4] * q[2]) * c[1] + (p[3] * q[4] + p[4] * q[3]) * s[1] + p[4] * q[4];
}

// Direction, antenna coefficients, n.r_0, and the averages A, B, C with the 2F coefficients.
// a and b are trigonometric polynomials of the sidereal phase x_j = x_0 - rate t_j, so their
// averages over the samples are sums of geometric series: no pass over the samples.
__global__ void k_sky_setup(const double* __restrict__ alpha, const double* __restrict__ delta,
                            int sky0, int nsky, SegConst sc, int full_form, SkyParams* __restrict__ sp) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nsky) return;
  const double al = alpha[sky0 + i], de = delta[sky0 + i];
  double sa, ca, sd, cd;
  sincos(al, &sa, &ca);
  sincos(de, &sd, &cd);
  SkyParams p;
  p.nx = cd * ca;
  p.ny = cd * sa;
  p.nz = sd;
  p.nr0 = p.nx * sc.r[0] + p.ny * sc.r[sc.n] + p.nz * sc.r[2 * sc.n];
  const double x0 = al - sc.phi_r;
  sincos(x0, &p.sx0, &p.cx0);
  const double s2d = 2.0 * sd * cd, c2d = cd * cd - sd * sd;
  p.ka[0] = sc.s2g * (3.0 - sc.c2l) * (3.0 - c2d) / 16.0;
  p.ka[1] = -sc.c2g * sc.sl * (3.0 - c2d) / 4.0;
  p.ka[2] = sc.s2g * sc.s2l * s2d / 4.0;
  p.ka[3] = -sc.c2g * sc.cl * s2d / 2.0;
  p.ka[4] = 0.75 * sc.s2g * sc.cl * sc.cl * cd * cd;
  p.kb[0] = sc.c2g * sc.sl * sd;
  p.kb[1] = sc.s2g * (3.0 - sc.c2l) * sd / 4.0;
  p.kb[2] = sc.c2g * sc.cl * cd;
  p.kb[3] = sc.s2g * sc.s2l * cd / 2.0;
  // mean of exp(i m x) = exp(i m (x_0 - mid)) dir[m - 1]
  double c[5], s[5];
  c[0] = 1.0;
  s[0] = 0.0;
  double cm, sm;
  sincos(x0 - sc.mid, &sm, &cm);
#pragma unroll
  for (int m = 1; m <= 4; ++m) {
    c[m] = c[m - 1] * cm - s[m - 1] * sm;
    s[m] = s[m - 1] * cm + c[m - 1] * sm;
  }
#pragma unroll
  for (int m = 1; m <= 4; ++m) {
    c[m] *= sc.dir[m - 1];
    s[m] *= sc.dir[m - 1];
  }
  const double kb[5] = {p.kb[0], p.kb[1], p.kb[2], p.kb[3], 0.0};
  p.A = antenna_mean(p.ka, p.ka, c, s);
  p.B = antenna_mean(kb, kb, c, s);
  p.C = antenna_mean(p.ka, kb, c, s);
  const double norm = 2.0 / ((double)sc.n * sc.sigma2);
  if (full_form) {
    const double D = p.A * p.B - p.C * p.C;
    p.cfa = norm * p.B / D;
    p.cfb = norm * p.A / D;
    p.cfab = -2.0 * norm * p.C / D;
  } else {
    p.cfa = norm / p.A;
    p.cfb = norm / p.B;
    p.cfab = 0.0;
  }
  p.pad = 0.0;
  sp[i] = p;
}

// Demodulation: za = x a e^{-i psi}, zb = x b e^{-i psi}, psi = 2 pi f_off D (reduced mod 2 pi
// in FP64), as pairs [j][a|b], sky i at z + i ldz.  A thread takes sample j of SKIES sky
// positions (those of blockIdx.y): the data and the sidereal rotation of the sample are
// read and formed once for them (one sky position a thread, with the antenna sums reduced
// here: 14 us per 8 sky positions at N = 86164).
constexpr int DEMOD_SKIES = 4;
template <typename T>
__global__ void __launch_bounds__(NT) k_sky_demod(SegConst sc, const SkyParams* __restrict__ sp, int nsky,
                                                  cx_pair<T>* __restrict__ z, long ldz) {
  const int j = blockIdx.x * NT + threadIdx.x;
  if (j >= sc.n) return;
  const int i0 = blockIdx.y * DEMOD_SKIES, i1 = min(i0 + DEMOD_SKIES, nsky);
  const double x = sc.x[j], rx = sc.r[j], ry = sc.r[sc.n + j], rz = sc.r[2 * sc.n + j];
  double st, ct;
  sincos(sidereal_rate() * ((double)j * sc.dt), &st, &ct);
  for (int i = i0; i < i1; ++i) {
    const SkyParams& p = sp[i];
    // x_j = x_0 - rate t_j
    const double cx_ = p.cx0 * ct + p.sx0 * st, sx = p.sx0 * ct - p.cx0 * st;
    const double c2x = cx_ * cx_ - sx * sx, s2x = 2.0 * sx * cx_;
    const double a = p.ka[0] * c2x + p.ka[1] * s2x + p.ka[2] * cx_ + p.ka[3] * sx + p.ka[4];
    const double b = p.kb[0] * c2x + p.kb[1] * s2x + p.kb[2] * cx_ + p.kb[3] * sx;
    const double d = p.nx * rx + p.ny * ry + p.nz * rz - p.nr0;
    double cyc = sc.f_off * d;
    cyc -= floor(cyc);
    T s, c;
    if constexpr (sizeof(T) == 8) {
      sincospi(2.0 * cyc, &s, &c);
    } else {
      sincospif((float)(2.0 * cyc), &s, &c);
    }
    const double xa = x * a, xb = x * b;
    z[i * ldz + j] = cx_pair<T>{mk<T>((T)xa * c, -(T)xa * s), mk<T>((T)xb * c, -(T)xb * s)};
  }
}

// Map a linear workgroup id to (tile, item) so that each XCD (workgroups are
// dealt round-robin over 8 XCDs) keeps a fixed subset of tiles for all items.
__device__ __forceinline__ void xcd_tile_item(int b, int ntiles, int& tile, int& item) {
  if ((ntiles & 7) == 0) {
    const int per = ntiles >> 3;
    const int xcd = b & 7, r = b >> 3;
    tile = xcd * per + (r % per);
    item = r / per;
  } else {
    tile = b % ntiles;
    item = b / ntiles;
  }
}

// ------------------------------------------------------------- template stage
struct TmplArgs {
  int n, P, Q, L;       // samples; template FFT L = P * Q
  float ibw;            // interbinning weight (second pass with interbinning only)
  int nfdot;            // spindowns per sky
  int t0;               // first template of this launch (within the sky batch)
  int sky0;             // global index of the batch's first sky
  double dt;
  const double* fdot;   // device list (explicit spindowns), or NULL on a lattice grid
  long ldzt;            // stride between series in zt
  // lattice grid (fdot NULL): template (sky, index) has spindown integer s = s_lo + index
  const double* w_freq; // per sky: w0 component of the sky vectors' combination
  const double* w_spin; // per sky: w1 component
  double m10, m11;      // w0 and w1 components of the spindown row
  double bins_per_rad;  // nfft / (2 pi)
  int s_lo, nfft;
  int nblk;             // first pass: tiles of the launch (its grid may be smaller and walk them)
  // which of two launched paths does the work: one of them returns at once (NULL: no choice)
  const int* route;
  int route_want;
  float ibpr, ibpi;     // interbinning of decimated transforms: exp(2 pi i dec_m0 / L)
};

// Lattice arithmetic shared by the kernels and the host's candidate records, with
// contraction off so that both round every product and sum the same way.
// s row + sky: a component of the grid point s M1 + (n M2 + m M3).
__host__ __device__ inline double lattice_w(int s, double row, double sky) {
#pragma clang fp contract(off)
  return (double)s * row + sky;
}

// Shift u, in bins of the nfft grid, of a template's frequencies above the Fourier bins:
// the fraction of w0 nfft / (2 pi) above the integer below it, where a value within 1e-6
// below an integer counts as that integer (u in [-1e-6, 1 - 1e-6)).
__host__ __device__ inline double lattice_shift_bins(double w0, double bins_per_rad) {
#pragma clang fp contract(off)
  const double x = w0 * bins_per_rad;
  return x - floor(x + 1e-6);
}

// Spindown chirp of one template in cycles, (c2 j + c1) j at resampled sample j:
// c2 = fdot dt^2 / 2 for an explicit spindown; on a lattice c2 = w1 / (2 pi) and
// c1 = u / nfft, the shift that puts the grid's frequencies on the transform's bins.
__device__ __forceinline__ void template_chirp(const TmplArgs& ta, int skyl, int sidx, double& c2, double& c1) {
  if (ta.fdot) {
    c2 = 0.5 * ta.fdot[sidx] * ta.dt * ta.dt;
    c1 = 0.0;
  } else {
    const int sky = ta.sky0 + skyl, s = ta.s_lo + sidx;
    c2 = lattice_w(s, ta.m11, ta.w_spin[sky]) * (0.5 / M_PI);
    c1 = lattice_shift_bins(lattice_w(s, ta.m10, ta.w_freq[sky]), ta.bins_per_rad) / (double)ta.nfft;
  }
}

// ------------------------------------------------------------- decimated series
// The searched bins [0, L/2) are half of a template transform's band, so the transform can
// run at 5/8 of the sampling rate: the resampled series is filtered once per sky position
// to the frequencies a template needs (its band, plus a margin for the spindown chirp's
// sweep) and sampled every 8/5 samples, and each template transforms 5 L / 8 points
// instead of L, with the same bins k / L at the same indices k.  The filter is a
// Kaiser-windowed sinc, centred on a quarter of the sampling rate: gain 1 within 0.25 + 0.006
// cycles per sample of the centre and 0 beyond 0.375 - 0.006, to 4e-8 (FP32) or 4e-15 (FP64),
// so that nothing folds into the searched bins.  Output m = 5 q + p (p < 5) is the filtered
// series at sample t = 8 (q - Q0) + 8 p / 5; the transform's bins so carry the phase
// exp(-2 pi i k 5 Q0 / L'), which |Fa|, |Fb| and Fa Fb* do not see.
constexpr int DEC_UP = 5, DEC_DOWN = 8;
template <typename T>
struct DecFilter;
template <>
struct DecFilter<float> {
  static constexpr int HALF = 44, Q0 = 6;   // half-width in samples
  static constexpr double BETA = 15.5;      // Kaiser parameter
};
template <>
struct DecFilter<double> {
  static constexpr int HALF = 92, Q0 = 12;
  static constexpr double BETA = 32.0;
};
template <typename T>
__host__ __device__ constexpr int dec_m0() { return DEC_UP * DecFilter<T>::Q0; }
// inputs of five outputs: 8 q' - HALF .. 8 q' + HALF + 7
template <typename T>
__host__ __device__ constexpr int dec_taps() { return 2 * DecFilter<T>::HALF + DEC_DOWN; }
template <typename T>
constexpr bool dec_ok() { return dec_taps<T>() % 8 == 0 && DecFilter<T>::Q0 * DEC_DOWN >= DecFilter<T>::HALF; }
static_assert(dec_ok<float>() && dec_ok<double>(), "filter geometry");
constexpr double DEC_SWEEP = 0.005;             // largest chirp sweep (cycles per sample) the margin takes
constexpr int DEC_NT = 128;                     // groups of five outputs per workgroup

// samples of the decimated series of n samples (whole groups of five)
template <typename T>
inline long dec_samples(long n) {
  return DEC_UP * (DecFilter<T>::Q0 + (n - 1 + DecFilter<T>::HALF) / DEC_DOWN + 1);
}

// Sky blockIdx.y, both series interleaved [m][a|b]; h[i][p] = filter value of input
// 8 (q - Q0) - HALF + i in output p.  A thread forms one group of five outputs of one
// series (wavefronts 0, 1: series a, 2, 3: b): 96 staged inputs and 480 taps in single
// precision, 192 and 960 in double, sums in double precision (as fast as single on this chip
// without packed single precision), so that the decimated series carries one rounding.  The
// taps are uniform (scalar loads); the centre frequency's rotation of the inputs, (-i)^i, only
// swaps and negates parts, and that of the outputs is a constant per p.  LDS index e sits at
// e + e / 8: lanes read eight inputs apart, and the padding spreads them over the banks.
template <typename T>
__global__ void __launch_bounds__(2 * DEC_NT) k_decimate(const cx_pair<T>* __restrict__ zt, long ldzt, int n,
                                                         cx<T>* __restrict__ zd, long ldzd, int nq,
                                                         const double* __restrict__ h) {
  constexpr int TAPS = dec_taps<T>(), NIN = DEC_DOWN * DEC_NT + TAPS - DEC_DOWN;
  __shared__ cx<T> sz[2][NIN + NIN / 8 + 1];
  const int s = threadIdx.x / DEC_NT, tid = threadIdx.x % DEC_NT;
  const int q0 = blockIdx.x * DEC_NT;
  const cx<T>* z = reinterpret_cast<const cx<T>*>(zt + (long)blockIdx.y * ldzt) + s;
  const int j0 = DEC_DOWN * (q0 - DecFilter<T>::Q0) - DecFilter<T>::HALF;
  for (int e = tid; e < NIN; e += DEC_NT) {
    const int j = j0 + e;
    sz[s][e + e / 8] = j >= 0 && j < n ? z[2 * j] : mk<T>(0, 0);
  }
  __syncthreads();
  const int q = q0 + tid;
  if (q >= nq) return;
  cx<double> acc[DEC_UP];
#pragma unroll
  for (int p = 0; p < DEC_UP; ++p) acc[p] = mk<double>(0.0, 0.0);
  const cx<T>* in = sz[s] + 9 * tid;
  for (int g = 0; g < TAPS / 8; ++g) {
    // eight inputs' taps at once: left to itself, the compiler waits for five at a time (16
    // sky positions of 86164 samples: 36 us, like this 28)
    double hc[8 * DEC_UP];
#pragma unroll
    for (int i = 0; i < 8 * DEC_UP; ++i) hc[i] = h[8 * g * DEC_UP + i];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const cx<T> v = in[9 * g + i];
      const double re = (double)v.re, im = (double)v.im;
      const cx<double> x = i % 4 == 0   ? mk<double>(re, im)
                           : i % 4 == 1 ? mk<double>(im, -re)
                           : i % 4 == 2 ? mk<double>(-re, -im)
                                        : mk<double>(-im, re);
#pragma unroll
      for (int p = 0; p < DEC_UP; ++p) {
        const double c = hc[i * DEC_UP + p];
        acc[p] = mk<double>(fma(c, x.re, acc[p].re), fma(c, x.im, acc[p].im));
      }
    }
  }
  // exp(2 pi i 0.25 t) with t = 8 p / 5 (whole turns left out): cos, sin of 2 pi 2 p / 5
  constexpr double c1 = 0.30901699437494742410, s1 = 0.95105651629515357212;   // 2 pi / 5
  constexpr double c2 = -0.80901699437494742410, s2 = 0.58778525229247312917;  // 4 pi / 5
  const cx<double> rot[DEC_UP] = {mk<double>(1.0, 0.0), mk<double>(c2, s2), mk<double>(c1, -s1), mk<double>(c1, s1),
                                  mk<double>(c2, -s2)};
  cx<T>* out = zd + (long)blockIdx.y * 2 * ldzd + 2 * (long)DEC_UP * q + s;
#pragma unroll
  for (int p = 0; p < DEC_UP; ++p) {
    const cx<double> a = cmul(acc[p], rot[p]);
    out[2 * p] = mk<T>((T)a.re, (T)a.im);
  }
}

// Whether the decimated series serves every template of a call: *route = 1 when no chirp
// sweeps more than DEC_SWEEP cycles per sample over the n samples (a value that is not a
// number fails), else 0.  One workgroup, once per call and segment: the lists are on the
// device and the call does not wait for them.
__global__ void __launch_bounds__(1024) k_route(const double* __restrict__ fdot, int nfdot, double dt,
                                                const double* __restrict__ w_spin, int nsky, int s_lo, double m11,
                                                int n, int* __restrict__ route) {
  const double per = fdot ? dt * dt * (double)n : (double)n / M_PI;   // sweep per unit of fdot, w1
  int bad = 0;
  const int count = fdot ? nfdot : nsky;
  for (int i = threadIdx.x; i < count; i += 1024) {
    if (fdot) {
      bad |= !(fabs(fdot[i]) * per <= DEC_SWEEP);
    } else {
      bad |= !(fabs(lattice_w(s_lo, m11, w_spin[i])) * per <= DEC_SWEEP);
      bad |= !(fabs(lattice_w(s_lo + nfdot - 1, m11, w_spin[i])) * per <= DEC_SWEEP);
    }
  }
  bad = __syncthreads_or(bad);
  if (threadIdx.x == 0) *route = bad ? 0 : 1;
}

// Where pass B puts its results.
struct OutArgs {
  int k_min, k_max;
  double threshold;
  const int* search_next;        // device: searches begun so far (this one included)
  int segment;
  CandEntry* cand;               // candidate buffer
  unsigned long long* count;     // crossings found so far (may exceed capacity)
  long long capacity;
  void* spectrum;                // [sky][fdot][k - k_min], T
};

// Start of a search: advance the device-side search index.
__global__ void k_begin_search(int* search_next) {
  if (threadIdx.x == 0 && blockIdx.x == 0) search_next[0] += 1;
}

// Exclusive prefix sum of one int per thread over a workgroup of NTH threads;
// returns the thread's offset and writes the total to *total (all threads).
template <int NTH>
__device__ __forceinline__ int block_exclusive_scan_n(int v, int* total) {
  __shared__ int wsum[NTH / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int k = 0; k < NTH / 64; ++k) {
    const int ws = wsum[k];
    if (k < w) before += ws;
    all += ws;
  }
  *total = all;
  return before + x - v;
}

// ------------------------------------------------------------ lattice sky loop
struct LatSkyArgs {
  double r2x, r2y, r3x, r3y;   // sky components (w2, w3) of rows 2 and 3
  double r2f, r2s, r3f, r3s;   // their w0 and w1 components
  double w;                    // W = 2 pi f_ref (1 AU / c)
  double ce, se;               // cos, sin of the obliquity
  double hemi;                 // +1 or -1
  int n_lo, m_lo, mspan;       // box origin and its extent in m
  long long total, capacity;   // box points; output capacity
  double *alpha, *delta, *w_freq, *w_spin;
  int* nm;
  long long* count;
};

// Sky loop of the lattice grid: every (n, m) of the box whose point (w2, w3) lies on the
// sky's disk, numbered in (n, m) order and written at its number.  One workgroup walks
// the box 256 points at a time (a workgroup scan numbers the points of each step), so
// the order needs no device-wide synchronisation.  The on-sky test and the w components
// are rounded as plain IEEE products and sums (no contraction).
__global__ __launch_bounds__(256) void k_lattice_sky(LatSkyArgs a) {
  long long base = 0;
  for (long long i0 = 0; i0 < a.total; i0 += 256) {
    const long long i = i0 + threadIdx.x;
    int on = 0, n = 0, m = 0;
    double xe = 0.0, ye = 0.0, r2 = 0.0;
    if (i < a.total) {
      n = a.n_lo + (int)(i / a.mspan);
      m = a.m_lo + (int)(i % a.mspan);
      {
#pragma clang fp contract(off)
        const double w2 = (double)n * a.r2x + (double)m * a.r3x;
        const double w3 = (double)n * a.r2y + (double)m * a.r3y;
        xe = w2 / a.w;
        ye = w3 / a.w;
        r2 = xe * xe + ye * ye;
      }
      on = r2 <= 1.0 ? 1 : 0;
    }
    int total = 0;
    const long long k = base + block_exclusive_scan_n<256>(on, &total);
    if (on && k < a.capacity) {
      double ze, wf, ws;
      {
#pragma clang fp contract(off)
        ze = a.hemi * sqrt(1.0 - r2);
        wf = (double)n * a.r2f + (double)m * a.r3f;
        ws = (double)n * a.r2s + (double)m * a.r3s;
      }
      // ecliptic to equatorial axes: rotation by the obliquity about the x axis
      const double x = xe;
      const double y = a.ce * ye - a.se * ze;
      const double z = a.se * ye + a.ce * ze;
      double al = atan2(y, x);
      if (al < 0.0) al += 2.0 * M_PI;
      a.alpha[k] = al;
      a.delta[k] = asin(fmin(1.0, fmax(-1.0, z)));
      a.w_freq[k] = wf;
      a.w_spin[k] = ws;
      if (a.nm) {
        a.nm[2 * k] = n;
        a.nm[2 * k + 1] = m;
      }
    }
    base += total;
    __syncthreads();   // the scan's LDS is reused by the next step
  }
  if (threadIdx.x == 0) *a.count = base;
}

}  // namespace fstat
