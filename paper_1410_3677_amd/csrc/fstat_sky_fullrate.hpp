// The upsampling and spline of full-rate calls in mixed precision (single-precision series):
// every call of a plan with a vetting network attached, and the small calls of other plans
// whose templates are not decimated, spectra of single templates above all.  The network
// scores 2F windows of both, and its three layers of BF16 roundings turn another rounding of
// 2F's last place into up to 2e-3 of a score; so that a captured window and the same window
// read from a spectrum (of a plan with a vetter, or a small one of any plan) stay equal, and
// what they were bit for bit, these calls share the transforms (four passes, one series per
// LDS column) and the spline (by its moments, a 33-tap filter) that fstat_sky.hpp replaces
// with faster ones of another rounding everywhere else.  A large spectrum of a plan without a
// vetter is decimated, and agrees to rounding.
#pragma once

#include "fstat_sky.hpp"

namespace fstat {
namespace full {

// One Stockham stage over NC columns of LEN points (column stride STRIDE),
// radix R, NS = product of the previous radices.  tw1024[m] = exp(-2 pi i m/1024).
template <typename T, int LEN, int NC, int NT, int STRIDE, int R, int NS, bool INV>
__device__ __forceinline__ void stockham_stage(cx<T>* lds, const cx<T>* __restrict__ tw1024) {
  constexpr int NB = LEN / R;           // butterflies per column
  constexpr int TOT = NC * NB;
  constexpr int PER = (TOT + NT - 1) / NT;
  constexpr int TWSTEP = 1024 / (NS * R);
  const int tid = threadIdx.x;
  cx<T> v[PER][R];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int b = tid + i * NT;
    if ((TOT % NT == 0) || b < TOT) {
      const int c = b / NB, j = b % NB;
      const cx<T>* col = lds + c * STRIDE;
      const int k = j % NS;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        cx<T> x = col[j + r * NB];
        if (NS > 1 && r > 0) {
          cx<T> w = tw1024[k * r * TWSTEP];
          if (INV) w.im = -w.im;
          x = cmul(x, w);
        }
        v[i][r] = x;
      }
      dftr<T, R, INV>(v[i]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int b = tid + i * NT;
    if ((TOT % NT == 0) || b < TOT) {
      const int c = b / NB, j = b % NB;
      cx<T>* col = lds + c * STRIDE;
      const int k = j % NS;
      const int base = (j / NS) * NS * R + k;
#pragma unroll
      for (int r = 0; r < R; ++r) col[base + r * NS] = v[i][r];
    }
  }
  __syncthreads();
}

template <typename T, int LEN, int NC, int NT, int STRIDE, bool INV, int NS>
__device__ __forceinline__ void lds_fft_from(cx<T>* lds, const cx<T>* __restrict__ tw1024) {
  if constexpr (NS < LEN) {
    constexpr int REM = LEN / NS;
    constexpr int R = REM >= 8 ? 8 : REM;
    stockham_stage<T, LEN, NC, NT, STRIDE, R, NS, INV>(lds, tw1024);
    lds_fft_from<T, LEN, NC, NT, STRIDE, INV, NS * R>(lds, tw1024);
  }
}

// In-place DFT (unnormalised; forward sign -i, INV sign +i) of NC LDS columns.
// Callers must __syncthreads() after filling LDS; the routine ends with a barrier.
template <typename T, int LEN, int NC, int NT, int STRIDE, bool INV>
__device__ __forceinline__ void lds_fft(cx<T>* lds, const cx<T>* __restrict__ tw1024) {
  static_assert(LEN >= 2 && LEN <= 1024 && (LEN & (LEN - 1)) == 0, "LEN must be a power of two <= 1024");
  lds_fft_from<T, LEN, NC, NT, STRIDE, INV, 1>(lds, tw1024);
}

// Column stride of an LDS tile: LEN plus one element breaks power-of-two strides.
template <int LEN>
constexpr int lds_stride() { return LEN + 1; }

// Workgroup tile width: columns per workgroup so that both series fit in 64 KiB of LDS.
template <typename T, int LEN>
constexpr int tile_width() {
  constexpr int tw = (64 * 1024) / (2 * (int)sizeof(cx<T>) * (LEN + 1));
  constexpr int p2 = tw >= 16 ? 16 : tw >= 8 ? 8 : tw >= 4 ? 4 : tw >= 2 ? 2 : 1;
  return p2;
}

enum SrcKind { SRC_PLAIN = 0, SRC_HALFSHIFT = 1 };

// Pass A of an L = P*Q FFT (DFT length Q along j2), two series per item.
//   SRC_PLAIN:     x_s[j] = series s of pair in[item * ld_in + j] for j < nvalid, else 0
//   SRC_HALFSHIFT: x_s[k] = Z[k] exp(i pi k_s / L), k_s = k for k < L/2, k - L otherwise
//                  (Z = in, the spectrum of a series of L samples; shlo, shhi: the
//                  twiddle tables of length 2L).  The inverse transform of x is the
//                  series half a sample later, the odd samples of its band-limited 2x
//                  upsampling with the Nyquist term on the negative side.
// Output T_s[k2 * P + j1] at out + (2 item + s) * L.
template <typename T, int Q, bool INV, int SRC>
__global__ void __launch_bounds__(NT) k_fft_pass_a(const cx<T>* __restrict__ in, long ld_in, int nvalid,
                                                   cx<T>* __restrict__ out, int P, int L,
                                                   const cx<T>* __restrict__ tw1024,
                                                   const cx<T>* __restrict__ twlo, const cx<T>* __restrict__ twhi,
                                                   const cx<T>* __restrict__ shlo, const cx<T>* __restrict__ shhi) {
  constexpr int TW = tile_width<T, Q>();
  constexpr int ST = lds_stride<Q>();
  __shared__ cx<T> lds[2 * TW * ST];
  int tile, item;
  xcd_tile_item(blockIdx.x, P / TW, tile, item);
  const int j10 = tile * TW;
  for (int e = threadIdx.x; e < 2 * TW * Q; e += NT) {
    const int s = e / (TW * Q), rem = e % (TW * Q);
    const int j2 = rem / TW, c = rem % TW;
    const int j = j10 + c + P * j2;
    cx<T> v = mk<T>(0, 0);
    const cx<T>* src = in + (2 * item + s) * ld_in;
    if (SRC == SRC_PLAIN) {
      if (j < nvalid) v = in[2 * (item * ld_in + j) + s];
    } else {
      cx<T> w = twiddle_L<T, true>(shlo, shhi, j);
      if (j >= (L >> 1)) w = mk<T>(-w.re, -w.im);
      v = cmul(src[j], w);
    }
    lds[(s * TW + c) * ST + j2] = v;
  }
  __syncthreads();
  lds_fft<T, Q, 2 * TW, NT, ST, INV>(lds, tw1024);
  for (int e = threadIdx.x; e < 2 * TW * Q; e += NT) {
    const int s = e / (TW * Q), rem = e % (TW * Q);
    const int k2 = rem / TW, c = rem % TW;
    const int j1 = j10 + c;
    cx<T> v = cmul(lds[(s * TW + c) * ST + k2], twiddle_L<T, INV>(twlo, twhi, j1 * k2));
    out[(long)(2 * item + s) * L + (long)k2 * P + j1] = v;
  }
}

// Pass B of an L = P*Q FFT (DFT length P along j1) with natural-order output:
// X_s[Q k1 + k2] * scale at out + (2 item + s) * ld_out.
template <typename T, int P, bool INV>
__global__ void __launch_bounds__(NT) k_fft_pass_b(const cx<T>* __restrict__ in, cx<T>* __restrict__ out,
                                                   long ld_out, int Q, int L, T scale,
                                                   const cx<T>* __restrict__ tw1024) {
  constexpr int TW = tile_width<T, P>();
  constexpr int ST = lds_stride<P>();
  __shared__ cx<T> lds[2 * TW * ST];
  int tile, item;
  xcd_tile_item(blockIdx.x, Q / TW, tile, item);
  const int k20 = tile * TW;
  for (int e = threadIdx.x; e < 2 * TW * P; e += NT) {
    const int s = e / (TW * P), rem = e % (TW * P);
    const int c = rem / P, j1 = rem % P;
    lds[(s * TW + c) * ST + j1] = in[(long)(2 * item + s) * L + (long)(k20 + c) * P + j1];
  }
  __syncthreads();
  lds_fft<T, P, 2 * TW, NT, ST, INV>(lds, tw1024);
  for (int e = threadIdx.x; e < 2 * TW * P; e += NT) {
    const int s = e / (TW * P), rem = e % (TW * P);
    const int k1 = rem / TW, c = rem % TW;
    out[(long)(2 * item + s) * ld_out + (long)Q * k1 + k20 + c] = cscale(lds[(s * TW + c) * ST + k1], scale);
  }
}

// Natural cubic spline through the upsampled series u[0..L) (unit spacing),
// evaluated at 2 s_j with s_j = j - D_j/dt; zero where s_j is outside [0, n-1].
// Spline moments: m_0 = m_{L-1} = 0, m_{p-1} + 4 m_p + m_{p+1} = d_p = 6 (u_{p+1} - 2u_p + u_{p-1}).
// They are computed as m_p = sum_q G(p, q) d_q with the Green's function of the
// (1, 4, 1) operator, g(k) = z^|k| / (2 sqrt 3), z = sqrt 3 - 2, and odd images at
// both ends: G(p, q) = g(p-q) - g(p+q) - g(2(L-1)-p-q), truncated at |k| <= KT
// (|z|^KT below the working precision).
template <typename T, int KT>
__device__ __forceinline__ cx<T> spline_moment(int p, int L, const cx<T>* d, int dlo, const T* g,
                                               const T* __restrict__ gg) {
  // d[q - dlo] = d_q for q in [max(1, p - KT), min(L - 2, p + KT)]
  if (p <= 0 || p >= L - 1) return mk<T>(0, 0);
  if (p > KT && p < L - 1 - KT) {
    // interior knot: no image terms, the symmetric 2 KT + 1 taps with the weights read as
    // uniform values (gg: the same table in global memory)
    const cx<T>* c = d + (p - dlo);
    cx<T> acc = mk<T>(gg[0] * c[0].re, gg[0] * c[0].im);
#pragma unroll
    for (int k = 1; k <= KT; ++k) {
      const cx<T> a = c[-k], b = c[k];
      acc = mk<T>(acc.re + gg[k] * (a.re + b.re), acc.im + gg[k] * (a.im + b.im));
    }
    return acc;
  }
  cx<T> acc = mk<T>(0, 0);
  const int q0 = max(1, p - KT), q1 = min(L - 2, p + KT);
  for (int q = q0; q <= q1; ++q) {
    const int dpq = p > q ? p - q : q - p;
    T w = g[dpq];
    if (p + q <= KT) w -= g[p + q];
    const int far = 2 * (L - 1) - p - q;
    if (far <= KT) w -= g[far];
    const cx<T> dq = d[q - dlo];
    acc = mk<T>(acc.re + w * dq.re, acc.im + w * dq.im);
  }
  return acc;
}

// Sample q of the 2x upsampled series: the even samples from the pairs of z (zero from n
// on), the odd samples from the plane o.
template <typename T>
__device__ __forceinline__ cx<T> upsampled(const cx<T>* __restrict__ z, const cx<T>* __restrict__ o, int q, int n) {
  const int h = q >> 1;
  if (q & 1) return o[h];
  return h < n ? z[2 * h] : mk<T>(0, 0);
}

template <typename T>
__device__ __forceinline__ cx<T> spline_eval(cx<T> u0, cx<T> u1, cx<T> m0, cx<T> m1, T t) {
  const T w = (T)1 - t;
  const T c0 = (w * w * w - w) / (T)6, c1 = (t * t * t - t) / (T)6;
  return mk<T>(w * u0.re + t * u1.re + c0 * m0.re + c1 * m1.re,
               w * u0.im + t * u1.im + c0 * m0.im + c1 * m1.im);
}

// u of sky i, series s at u + (2 i + s) * L; output zt + (2 i + s) * ldzt.
// One workgroup covers NT outputs j; their knot range [pmin, pmax + 1] is staged in
// LDS together with the curvature sources d_q within KT of it.
template <typename T, int KT>
__global__ void __launch_bounds__(NT) k_spline(SegConst sc, const SkyParams* __restrict__ sp,
                                               const cx<T>* __restrict__ z, const cx<T>* __restrict__ o, long ldz,
                                               cx_pair<T>* __restrict__ zt, long ldzt, const T* __restrict__ gtab) {
  constexpr int CAP = 2 * NT + 64;              // knots held for one tile
  constexpr int DCAP = CAP + 2 * KT + 2;        // curvature sources held
  __shared__ cx<T> su[2][DCAP + 2];
  __shared__ cx<T> sd[2][DCAP];
  __shared__ cx<T> sm[2][CAP + 1];
  __shared__ T sg[KT + 1];
  __shared__ int sminmax[2];
  const int i = blockIdx.y;
  const int L = sc.nfft, n = sc.n;
  const SkyParams& p = sp[i];
  const int j = blockIdx.x * NT + threadIdx.x;
  bool valid = false;
  int kn = 0;
  T tf = 0;
  if (j < n) {
    const double d = p.nx * sc.r[j] + p.ny * sc.r[n + j] + p.nz * sc.r[2 * n + j] - p.nr0;
    const double s = (double)j - d / sc.dt;
    valid = (s >= 0.0) && (s <= (double)(n - 1));
    if (valid) {
      const double pos = 2.0 * s;
      kn = (int)floor(pos);
      kn = min(max(kn, 0), L - 2);
      tf = (T)(pos - (double)kn);
    }
  }
  if (threadIdx.x <= KT) sg[threadIdx.x] = gtab[threadIdx.x];
  if (threadIdx.x == 0) {
    sminmax[0] = 0x7fffffff;
    sminmax[1] = -1;
  }
  __syncthreads();
  {
    // the tile's knot range: a wavefront reduction, then one LDS atomic per wavefront
    int mn = valid ? kn : 0x7fffffff, mx = valid ? kn : -1;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      mn = min(mn, __shfl_xor(mn, off, 64));
      mx = max(mx, __shfl_xor(mx, off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
      atomicMin(&sminmax[0], mn);
      atomicMax(&sminmax[1], mx);
    }
  }
  __syncthreads();
  const int pmin = sminmax[0], pmax = sminmax[1];
  if (pmax < 0) {  // no valid output in this tile
    if (j < n) {
      zt[i * ldzt + j] = cx_pair<T>{mk<T>(0, 0), mk<T>(0, 0)};
    }
    return;
  }
  const cx<T>* za = z + 2 * (long)i * ldz;   // pairs: series b one element after a
  const cx<T>* zb = za + 1;
  const cx<T>* oa = o + (long)(2 * i) * ldz;
  const cx<T>* ob = o + (long)(2 * i + 1) * ldz;
  if (pmax + 1 - pmin + 1 <= CAP) {
    // knots needed for moments [pmin, pmax+1]: sources q in [pmin-KT, pmax+1+KT], each uses u[q-1..q+1]
    const int dlo = max(1, pmin - KT), dhi = min(L - 2, pmax + 1 + KT);
    const int ulo = dlo - 1, uhi = dhi + 1;
    for (int q = ulo + threadIdx.x; q <= uhi; q += NT) {
      su[0][q - ulo] = upsampled(za, oa, q, n);
      su[1][q - ulo] = upsampled(zb, ob, q, n);
    }
    __syncthreads();
    for (int q = dlo + threadIdx.x; q <= dhi; q += NT) {
      for (int s = 0; s < 2; ++s) {
        const cx<T> a = su[s][q - 1 - ulo], b = su[s][q - ulo], c = su[s][q + 1 - ulo];
        sd[s][q - dlo] = mk<T>((T)6 * (c.re - (T)2 * b.re + a.re), (T)6 * (c.im - (T)2 * b.im + a.im));
      }
    }
    __syncthreads();
    for (int q = pmin + threadIdx.x; q <= pmax + 1; q += NT) {
      sm[0][q - pmin] = spline_moment<T, KT>(q, L, sd[0], dlo, sg, gtab);
      sm[1][q - pmin] = spline_moment<T, KT>(q, L, sd[1], dlo, sg, gtab);
    }
    __syncthreads();
    if (j < n) {
      cx<T> va = mk<T>(0, 0), vb = mk<T>(0, 0);
      if (valid) {
        // pmin >= ulo + 1 and pmax + 1 <= uhi, so both knots are staged
        va = spline_eval(su[0][kn - ulo], su[0][kn + 1 - ulo], sm[0][kn - pmin], sm[0][kn + 1 - pmin], tf);
        vb = spline_eval(su[1][kn - ulo], su[1][kn + 1 - ulo], sm[1][kn - pmin], sm[1][kn + 1 - pmin], tf);
      }
      zt[i * ldzt + j] = cx_pair<T>{va, vb};
    }
  } else {
    // wide knot range (irregular delays): every thread works from global memory
    if (j < n) {
      cx<T> out[2] = {mk<T>(0, 0), mk<T>(0, 0)};
      if (valid) {
        for (int s = 0; s < 2; ++s) {
          const cx<T>* zs = s ? zb : za;
          const cx<T>* os = s ? ob : oa;
          auto us = [&](int q) { return upsampled(zs, os, q, n); };
          cx<T> m01[2];
          for (int h = 0; h < 2; ++h) {
            const int pp = kn + h;
            cx<T> acc = mk<T>(0, 0);
            if (pp > 0 && pp < L - 1) {
              const int q0 = max(1, pp - KT), q1 = min(L - 2, pp + KT);
              for (int q = q0; q <= q1; ++q) {
                const cx<T> a = us(q - 1), b = us(q), c = us(q + 1);
                const cx<T> dq = mk<T>((T)6 * (c.re - (T)2 * b.re + a.re), (T)6 * (c.im - (T)2 * b.im + a.im));
                const int dpq = pp > q ? pp - q : q - pp;
                T w = sg[dpq];
                if (pp + q <= KT) w -= sg[pp + q];
                const int far = 2 * (L - 1) - pp - q;
                if (far <= KT) w -= sg[far];
                acc = mk<T>(acc.re + w * dq.re, acc.im + w * dq.im);
              }
            }
            m01[h] = acc;
          }
          out[s] = spline_eval(us(kn), us(kn + 1), m01[0], m01[1], tf);
        }
      }
      zt[i * ldzt + j] = cx_pair<T>{out[0], out[1]};
    }
  }
}

}  // namespace full
}  // namespace fstat
