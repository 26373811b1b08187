// Per-sky kernels after the demodulation: the 2x band-limited upsampling (two transforms of
// M = nfft / 2 = P Q points) and the spline onto the barycentric grid.  Both amplitude
// series travel as pairs [sample][a|b], so that one position is one 16-byte access (32 in
// double precision) and eight neighbouring columns fill a 128-byte line.
//
//   k_sky_cols (forward)  columns j1 + P j2 of the demodulated series: Q-point DFTs over j2,
//                         times W_M^(j1 k2), to T[k2][j1];
//   k_sky_rows            rows T[k2][.] in place: P-point DFT over j1 (the spectrum
//                         X[Q k1 + k2]), the half-sample shift, the inverse P-point DFT
//                         over k1, times W_M^(-k2 n2): the forward transform's second pass
//                         and the inverse one's first, which work on the same rows;
//   k_sky_cols (inverse)  columns T[.][n2]: inverse Q-point DFTs over k2, the odd samples
//                         o[P n1 + n2] of the upsampled series (the even ones are the
//                         series itself).
// Bound by the memory traffic of the three passes (11 MB per sky position at M = 2^17,
// single precision); four passes that moved 32-byte row segments per series took 6.9 us a
// sky position in batches of 16.
#pragma once

#include "fstat_tmpl.hpp"

namespace fstat {

template <typename T>
__device__ __forceinline__ cx_pair<T> pmul(cx_pair<T> v, cx<T> w) {
  return cx_pair<T>{cmul(v.a, w), cmul(v.b, w)};
}

// Columns per workgroup: 2048 positions, at least a 128-byte line of a row; one radix-8
// butterfly of both series per thread and stage.
template <typename T, int LEN>
__host__ __device__ constexpr int sky_tw() {
  return 2048 / LEN > 128 / (int)sizeof(cx_pair<T>) ? 2048 / LEN : 128 / (int)sizeof(cx_pair<T>);
}
template <typename T, int LEN>
__host__ __device__ constexpr int sky_nt() { return LEN * sky_tw<T, LEN>() / 8; }

// One butterfly's inputs of the stage at stride NS, twiddled and transformed: p points at
// index j, inputs STEP pairs apart.
template <typename T, int LEN, int NS, int STEP, bool INV>
__device__ __forceinline__ void sky_stage_load(cx_pair<T>* v, const cx_pair<T>* p, int j,
                                               const cx<T>* __restrict__ twst) {
  constexpr int R = stage_radix<LEN, NS>();
  cx<T> a[R], b[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const cx_pair<T> x = p[r * STEP];
    a[r] = x.a;
    b[r] = x.b;
    if constexpr (NS > 1) {
      if (r > 0) {
        const cx<T> w = stage_tw<T, NS, R, INV>(twst, j % NS, r);
        a[r] = cmul(a[r], w);
        b[r] = cmul(b[r], w);
      }
    }
  }
  dftr<T, R, INV>(a);
  dftr<T, R, INV>(b);
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] = cx_pair<T>{a[r], b[r]};
}

template <typename T, int LEN, int NS, bool INV>
__device__ __forceinline__ void sky_cols_middle(cx_pair<T>* lds, const cx<T>* __restrict__ twst) {
  constexpr int R = stage_radix<LEN, NS>(), TW = sky_tw<T, LEN>(), NT_ = sky_nt<T, LEN>();
  if constexpr (NS * R < LEN) {
    constexpr int NB = LEN / R, PER = TW * NB / NT_;
    cx_pair<T> v[PER][R];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int b = (int)threadIdx.x + i * NT_;
      sky_stage_load<T, LEN, NS, NB * TW, INV>(v[i], lds + b, b / TW, twst);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int b = (int)threadIdx.x + i * NT_, c = b % TW, j = b / TW;
      cx_pair<T>* p = lds + ((j / NS) * NS * R + j % NS) * TW + c;
#pragma unroll
      for (int r = 0; r < R; ++r) p[r * NS * TW] = v[i][r];
    }
    __syncthreads();
    sky_cols_middle<T, LEN, NS * R, INV>(lds, twst);
  }
}

// LEN-point DFTs of columns c = 0 .. P - 1 of sky blockIdx.x / tiles, elements (i, c) at
// in[i P + c] and out[i P + c] (strides ld_in, ld_out pairs a sky).  Forward: elements from
// nvalid on read as zero, outputs times W_M^(c i).  Inverse: outputs times `scale`, those
// from nkeep on left out.
template <typename T, int LEN, bool INV>
__global__ void __launch_bounds__((sky_nt<T, LEN>()))
    k_sky_cols(const cx_pair<T>* __restrict__ in, long ld_in, int nvalid, cx_pair<T>* __restrict__ out, long ld_out,
               int nkeep, int P, T scale, const cx<T>* __restrict__ twst, const cx<T>* __restrict__ twlo,
               const cx<T>* __restrict__ twhi) {
  constexpr int TW = sky_tw<T, LEN>(), NT_ = sky_nt<T, LEN>(), NB = LEN / 8;
  __shared__ cx_pair<T> lds[LEN * TW];
  int tile, item;
  xcd_tile_item(blockIdx.x, P / TW, tile, item);
  const cx_pair<T>* src = in + (long)item * ld_in;
  {
    const int c = (int)threadIdx.x % TW, j = (int)threadIdx.x / TW;
    cx<T> a[8], b[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int e = (j + NB * r) * P + tile * TW + c;
      a[r] = b[r] = mk<T>(0, 0);
      if (INV || e < nvalid) {
        const cx_pair<T> x = src[e];
        a[r] = x.a;
        b[r] = x.b;
      }
    }
    dft8<T, INV>(a);
    dft8<T, INV>(b);
    cx_pair<T>* p = lds + 8 * j * TW + c;
#pragma unroll
    for (int r = 0; r < 8; ++r) p[r * TW] = cx_pair<T>{a[r], b[r]};
  }
  __syncthreads();
  sky_cols_middle<T, LEN, 8, INV>(lds, twst);
  constexpr int NSL = last_ns<LEN, 1>(), RL = stage_radix<LEN, NSL>(), NBL = LEN / RL, PER = TW * NBL / NT_;
  cx_pair<T>* dst = out + (long)item * ld_out;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int b = (int)threadIdx.x + i * NT_, j = b / TW, c = tile * TW + b % TW;
    cx_pair<T> v[RL];
    sky_stage_load<T, LEN, NSL, NBL * TW, INV>(v, lds + b, j, twst);
    if constexpr (INV) {
#pragma unroll
      for (int r = 0; r < RL; ++r) {
        const int e = (j + NSL * r) * P + c;
        if (e < nkeep) dst[e] = cx_pair<T>{cscale(v[r].a, scale), cscale(v[r].b, scale)};
      }
    } else {
#pragma unroll
      for (int r = 0; r < RL; ++r)
        dst[(j + NSL * r) * P + c] = pmul(v[r], twiddle_L<T, false>(twlo, twhi, c * (j + NSL * r)));
    }
  }
}

// The stages after the first of a row of P points, up to the last, whose outputs stay with
// the thread: output s of thread g is index g + G s.  row: the row's LDS, index i at i + i/8.
template <typename T, int P, int NS, bool INV>
__device__ __forceinline__ void sky_row_stages(cx_pair<T> (&v)[8], cx_pair<T>* row, int g,
                                               const cx<T>* __restrict__ twst) {
  constexpr int G = groups_per_col<P>(), R = stage_radix<P, NS>(), NB = P / R, PB = NB / G;
  static_assert(NB % 8 == 0, "constant offsets need NB a multiple of 8");
  cx_pair<T> u[PB][R];
#pragma unroll
  for (int b = 0; b < PB; ++b) {
    const int j = g + G * b;
    sky_stage_load<T, P, NS, NB + NB / 8, INV>(u[b], row + phys(j), j, twst);
  }
  if constexpr (NS * R < P) {
    stage_sync<rows_in_wave<P>()>();
#pragma unroll
    for (int b = 0; b < PB; ++b) {
      const int j = g + G * b;
      cx_pair<T>* p = row + phys((j / NS) * NS * R + j % NS);
#pragma unroll
      for (int r = 0; r < R; ++r) p[r * NS + (r * NS) / 8] = u[b][r];
    }
    stage_sync<rows_in_wave<P>()>();
    sky_row_stages<T, P, NS * R, INV>(v, row, g, twst);
  } else {
#pragma unroll
    for (int b = 0; b < PB; ++b)
#pragma unroll
      for (int r = 0; r < R; ++r) v[b + (NS / G) * r] = u[b][r];
  }
}

// First stage (radix 8) of a row whose inputs g + G s the thread holds, into LDS.
template <typename T, int P, bool INV>
__device__ __forceinline__ void sky_row_first(const cx_pair<T> (&v)[8], cx_pair<T>* row, int g) {
  cx<T> a[8], b[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    a[s] = v[s].a;
    b[s] = v[s].b;
  }
  dft8<T, INV>(a);
  dft8<T, INV>(b);
  stage_sync<rows_in_wave<P>()>();
#pragma unroll
  for (int s = 0; s < 8; ++s) row[9 * g + s] = cx_pair<T>{a[s], b[s]};
  stage_sync<rows_in_wave<P>()>();
}

// shlo, shhi: twiddle tables of 2 M points.
template <typename T, int P>
__global__ void __launch_bounds__(NT) k_sky_rows(cx_pair<T>* __restrict__ t, int Q, const cx<T>* __restrict__ twst,
                                                 const cx<T>* __restrict__ twlo, const cx<T>* __restrict__ twhi,
                                                 const cx<T>* __restrict__ shlo, const cx<T>* __restrict__ shhi) {
  constexpr int G = groups_per_col<P>(), RPW = NT / G;
  __shared__ cx_pair<T> lds[RPW * (P + P / 8)];
  const int g = threadIdx.x % G, sub = threadIdx.x / G;
  const int R = blockIdx.x * RPW + sub, sky = R / Q, k2 = R - sky * Q;
  cx_pair<T>* row = t + ((long)sky * Q + k2) * P;
  cx_pair<T>* col = lds + sub * (P + P / 8);
  cx_pair<T> v[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) v[s] = row[g + G * s];
  sky_row_first<T, P, false>(v, col, g);
  sky_row_stages<T, P, 8, false>(v, col, g, twst);
  // spectrum bins k = Q (g + G s) + k2 times exp(i pi k_s / M), k_s = k below M/2 (s < 4) and
  // k - M from there on
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const cx<T> w = twiddle_L<T, true>(shlo, shhi, Q * (g + G * s) + k2);
    v[s] = pmul(v[s], s < 4 ? w : mk<T>(-w.re, -w.im));
  }
  stage_sync<rows_in_wave<P>()>();   // the last forward stage has read the row
  sky_row_first<T, P, true>(v, col, g);
  sky_row_stages<T, P, 8, true>(v, col, g, twst);
  // every factor from the tables: as powers of a step (seven multiplications in a row) they
  // made the upsampled series 25% less accurate
#pragma unroll
  for (int s = 0; s < 8; ++s) row[g + G * s] = pmul(v[s], twiddle_L<T, true>(twlo, twhi, k2 * (g + G * s)));
}

// ----------------------------------------------------------------- resampling
// Sample q of the 2x upsampled series (0 <= q < L): the even samples are the series z itself
// (zero from n on), the odd samples the series o half a sample later.
template <typename T>
__device__ __forceinline__ cx_pair<T> upsampled(const cx_pair<T>* __restrict__ z, const cx_pair<T>* __restrict__ o,
                                                int q, int n) {
  const int h = q >> 1;
  if (q & 1) return o[h];
  return h < n ? z[h] : cx_pair<T>{mk<T>(0, 0), mk<T>(0, 0)};
}

// The same for any q within L of the series' ends, continued oddly about its first and last
// samples, as a natural spline continues.
template <typename T>
__device__ __forceinline__ cx_pair<T> upsampled_odd(const cx_pair<T>* __restrict__ z,
                                                    const cx_pair<T>* __restrict__ o, int q, int n, int L) {
  const int end = q < 0 ? 0 : L - 1;
  const int m = q < 0 ? -q : q >= L ? 2 * (L - 1) - q : q;
  cx_pair<T> v = upsampled(z, o, m, n);
  if (m != q) {
    const cx_pair<T> e = upsampled(z, o, end, n);
    v.a = mk<T>((T)2 * e.a.re - v.a.re, (T)2 * e.a.im - v.a.im);
    v.b = mk<T>((T)2 * e.b.re - v.b.re, (T)2 * e.b.im - v.b.im);
  }
  return v;
}

// Pairs in[0, n) apart: either plane may be NULL (stage-by-stage checks).
template <typename T>
__global__ void __launch_bounds__(NT) k_unpair(const cx_pair<T>* __restrict__ in, int n, cx<T>* __restrict__ a,
                                               cx<T>* __restrict__ b) {
  const int j = blockIdx.x * NT + threadIdx.x;
  if (j >= n) return;
  if (a) a[j] = in[j].a;
  if (b) b[j] = in[j].b;
}
// The upsampled series of both, odd samples h of a and b at oa[step h], ob[step h].
template <typename T>
__global__ void __launch_bounds__(NT) k_upsampled(const cx_pair<T>* __restrict__ z, const cx<T>* __restrict__ oa,
                                                  const cx<T>* __restrict__ ob, int step, int n, int L,
                                                  cx<T>* __restrict__ a, cx<T>* __restrict__ b) {
  const int q = blockIdx.x * NT + threadIdx.x, h = q >> 1;
  if (q >= L) return;
  cx_pair<T> v = {mk<T>(0, 0), mk<T>(0, 0)};
  if (q & 1) v = cx_pair<T>{oa[(long)step * h], ob[(long)step * h]};
  else if (h < n) v = z[h];
  if (a) a[q] = v.a;
  if (b) b[q] = v.b;
}

// Cubic B-spline through four coefficients at t in [0, 1] between the middle two (wt: its
// weights).
template <typename T>
__device__ __forceinline__ void bspline_weights(T t, T (&wt)[4]) {
  const T w = (T)1 - t, s = (T)1 / (T)6;
  wt[0] = s * (w * w * w);
  wt[1] = s * ((T)4 - t * t * ((T)6 - (T)3 * t));
  wt[2] = s * ((T)4 - w * w * ((T)6 - (T)3 * w));
  wt[3] = s * (t * t * t);
}

// Natural cubic spline through the upsampled series u[0..L) (unit spacing), evaluated at
// 2 s_j with s_j = j - D_j/dt; zero where s_j is outside [0, n-1].  In B-spline form: the
// coefficients solve (c_{p-1} + 4 c_p + c_{p+1}) / 6 = u_p, and natural ends are u continued
// oddly about its end points.  The inverse of (1, 4, 1) is z^|k| / (2 sqrt 3),
// z = sqrt 3 - 2, so
//   c_p = sqrt 3 (y+_p + y-_p - u_p),  y+_p = u_p + z y+_{p-1},  y-_p = u_p + z y-_{p+1}.
// A thread runs both recursions over SPL_C neighbouring knots, from SPL_W knots before and
// after them (|z|^16 = 7e-10, |z|^32 = 5e-19): per knot six LDS reads and 24 multiply-adds
// for both series in single precision.  The coefficients replace the knots in LDS.  (With
// the spline's moments beside the knots, twice the LDS, 40 us per 16 sky positions at
// N = 86164; a 33-tap filter for the moments, 33 LDS reads per knot, 70.)
constexpr double SPL_Z = -0.26794919243112270647;
template <typename T>
__host__ __device__ constexpr int spl_w() { return sizeof(T) == 8 ? 32 : 16; }
template <typename T>
__host__ __device__ constexpr int spl_c() { return sizeof(T) == 8 ? 4 : 8; }
constexpr int SPL_NT = 128;
template <typename T>
__host__ __device__ constexpr int spl_knots() { return SPL_NT * spl_c<T>(); }
// outputs of a workgroup: their knots, two each and slack for the delay's slope, fit
template <typename T>
__host__ __device__ constexpr int spl_out() { return spl_knots<T>() / 2 - 12; }

template <typename T>
__global__ void __launch_bounds__(SPL_NT) k_spline(SegConst sc, const SkyParams* __restrict__ sp,
                                                   const cx_pair<T>* __restrict__ z, long ldz,
                                                   const cx_pair<T>* __restrict__ o, long ldo,
                                                   cx_pair<T>* __restrict__ zt, long ldzt) {
  constexpr int W = spl_w<T>(), C = spl_c<T>(), KN = spl_knots<T>(), NOUT = spl_out<T>();
  constexpr int PER = (NOUT + SPL_NT - 1) / SPL_NT, NU = KN + 2 * W;
  constexpr T Z = (T)SPL_Z, ONE = (T)1 / ((T)1 - (T)SPL_Z), ROOT3 = (T)1.7320508075688772935;
  __shared__ cx_pair<T> su[NU + NU / C + 1];   // knot p0 - W + e at e + e / C
  __shared__ int sminmax[2];
  const int i = blockIdx.y, tid = threadIdx.x;
  const int L = sc.nfft, n = sc.n;
  const double nx = sp[i].nx, ny = sp[i].ny, nz = sp[i].nz, nr0 = sp[i].nr0;
  const int j0 = blockIdx.x * NOUT;
  int kn[PER];   // knot of each output, -1: outside the data
  T tf[PER];
  int mn = 0x7fffffff, mx = -1;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int jo = tid + SPL_NT * e, j = j0 + jo;
    kn[e] = -1;
    tf[e] = 0;
    if (jo < NOUT && j < n) {
      const double d = nx * sc.r[j] + ny * sc.r[n + j] + nz * sc.r[2 * n + j] - nr0;
      const double s = (double)j - d / sc.dt;
      if (s >= 0.0 && s <= (double)(n - 1)) {
        const double pos = 2.0 * s;
        kn[e] = min(max((int)floor(pos), 0), L - 2);
        tf[e] = (T)(pos - (double)kn[e]);
        mn = min(mn, kn[e]);
        mx = max(mx, kn[e]);
      }
    }
  }
  if (tid == 0) {
    sminmax[0] = 0x7fffffff;
    sminmax[1] = -1;
  }
  __syncthreads();
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    mn = min(mn, __shfl_xor(mn, off, 64));
    mx = max(mx, __shfl_xor(mx, off, 64));
  }
  if ((tid & 63) == 0) {
    atomicMin(&sminmax[0], mn);
    atomicMax(&sminmax[1], mx);
  }
  __syncthreads();
  // coefficients of knots p0 = first - 1 .. last + 2
  const int p0 = sminmax[0] - 1, pmax = sminmax[1];
  const int knots = pmax < 0 ? 0 : pmax + 3 - p0;
  const cx_pair<T>* zs = z + (long)i * ldz;
  const cx_pair<T>* os = o + (long)i * ldo;
  cx_pair<T>* out = zt + (long)i * ldzt;
  const bool staged = pmax >= 0 && knots <= KN;
  if (staged) {
    const int stage = (knots + C - 1) / C * C + 2 * W;   // whole chunks of knots and both warm-ups
    for (int e = tid; e < stage; e += SPL_NT) su[e + e / C] = upsampled_odd(zs, os, p0 - W + e, n, L);
    __syncthreads();
    T y[C][4];
    if (tid * C < knots) {
      // knots p0 + C tid .. + C - 1 are staged entries C tid + W ..
      auto u = [&](int e) { return su[C * tid + e + (C * tid + e) / C]; };
      cx_pair<T> v = u(0);
      T s[4] = {v.a.re * ONE, v.a.im * ONE, v.b.re * ONE, v.b.im * ONE};
#pragma unroll
      for (int e = 1; e < W + C; ++e) {
        v = u(e);
        s[0] = fma(Z, s[0], v.a.re);
        s[1] = fma(Z, s[1], v.a.im);
        s[2] = fma(Z, s[2], v.b.re);
        s[3] = fma(Z, s[3], v.b.im);
        if (e >= W) {
#pragma unroll
          for (int k = 0; k < 4; ++k) y[e - W][k] = s[k];
        }
      }
      v = u(2 * W + C - 1);
      s[0] = v.a.re * ONE;
      s[1] = v.a.im * ONE;
      s[2] = v.b.re * ONE;
      s[3] = v.b.im * ONE;
#pragma unroll
      for (int e = 2 * W + C - 2; e >= W; --e) {
        v = u(e);
        if (e < W + C) {
          // y+ + y- - u = y+ + z y-_{p+1}
#pragma unroll
          for (int k = 0; k < 4; ++k) y[e - W][k] = ROOT3 * fma(Z, s[k], y[e - W][k]);
        }
        s[0] = fma(Z, s[0], v.a.re);
        s[1] = fma(Z, s[1], v.a.im);
        s[2] = fma(Z, s[2], v.b.re);
        s[3] = fma(Z, s[3], v.b.im);
      }
    }
    __syncthreads();
    if (tid * C < knots) {
#pragma unroll
      for (int e = 0; e < C; ++e)
        su[(C + 1) * tid + e] = cx_pair<T>{mk<T>(y[e][0], y[e][1]), mk<T>(y[e][2], y[e][3])};
    }
    __syncthreads();
  }
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int jo = tid + SPL_NT * e, j = j0 + jo;
    if (jo >= NOUT || j >= n) continue;
    cx_pair<T> r = {mk<T>(0, 0), mk<T>(0, 0)};
    if (kn[e] >= 0) {
      T wt[4];
      bspline_weights(tf[e], wt);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int q = kn[e] - 1 + k;
        cx_pair<T> c;
        if (staged) {
          const int x = q - p0;
          c = su[x + x / C];
        } else {
          // knots too far apart for the tile (irregular delays): from global memory
          T w = 1;
          c = upsampled_odd(zs, os, q, n, L);
          for (int m = 1; m <= W; ++m) {
            w *= Z;
            const cx_pair<T> lo = upsampled_odd(zs, os, q - m, n, L), hi = upsampled_odd(zs, os, q + m, n, L);
            c.a = mk<T>(fma(w, lo.a.re + hi.a.re, c.a.re), fma(w, lo.a.im + hi.a.im, c.a.im));
            c.b = mk<T>(fma(w, lo.b.re + hi.b.re, c.b.re), fma(w, lo.b.im + hi.b.im, c.b.im));
          }
          c = cx_pair<T>{cscale(c.a, ROOT3), cscale(c.b, ROOT3)};
        }
        r.a = mk<T>(fma(wt[k], c.a.re, r.a.re), fma(wt[k], c.a.im, r.a.im));
        r.b = mk<T>(fma(wt[k], c.b.re, r.b.re), fma(wt[k], c.b.im, r.b.im));
      }
    }
    out[j] = r;
  }
}

// samples of the odd series the spline of n samples reads: knots up to 2 (n - 1) + 2, the
// rest of their chunk and the warm-up
template <typename T>
inline int spline_keep(int n, int M) { return std::min(M, n + (spl_c<T>() + spl_w<T>()) / 2 + 3); }

}  // namespace fstat
