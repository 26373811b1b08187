// Training step of the vetting network: forward, backward and Adam.
//
// One workgroup takes a patch through its convolutions with the activations in LDS (no
// im2col matrices: a matrix-core operand of tap t is a row of the tile t positions on), the
// dense head is one kernel over 16 patches, and every kernel leaves its share of the
// gradient sums as partial sums that one reduction adds in a fixed order.
//
//   k_train_conv_fwd   input, three convolutions -> BF16 activations a1, a2, x = a3
//   k_gemm_nt_lds      z4 = x W4^T, split along K (fstat_vet.hpp)
//   k_train_head       z4 -> a4 -> z5 -> logit, loss terms; back to dz5, dz4
//   k_train_dense_bwd  dW4 = dz4^T x and dW5 = dz5^T a4; dz3 = (dz4 W4) [a3 > 0]
//   k_train_conv_bwd   per patch: dz2, dz1; its share of dW1, db1
//   k_train_dw_conv    dW3 and dW2 in parts of the positions
//   k_train_reduce     the parts and the head's columns added up
//   k_vet_update       Adam and the BF16 copies of the weights
//
// Every sum has a fixed order that depends on the number of patches alone: matrix-core steps
// of 16 with the bias added last, parts of the positions one after the other, trees over the
// positions.  It is the order of the im2col products and serial column sums that these
// kernels replace, bit for bit: Adam's first steps turn the last bit of a gradient into
// activations that round the other way.
// 256 patches: 740 us with 55 launches, which moved about 600 MB (half of it im2col matrices);
// 79 us here, with about 120 MB in eight launches.  Now bound by latency: one workgroup per
// CU or fewer in each launch, 5 to 14 us each.
#pragma once

#include "fstat_vet.hpp"

namespace fstat {
namespace vet {

constexpr int TR_LD = 36;              // BF16 per LDS row of 32 channels (8-byte aligned rows)
constexpr int TR_ROWS = L + 6;         // a patch's positions and three rows of zeros either side
constexpr int TF_ELEMS = KW * 2 * 2 * 64 * 4;   // weight fragments of one convolution

// Fragments of a convolution's weights for 16 x 16 x 16 steps: [tap t][half h of the inner
// channels][block nb of the outer ones][lane][4], inner channel 16 h + 4 (lane / 16) + i,
// outer channel 16 nb + lane % 16.
__device__ __forceinline__ int frag16(int t, int inner, int outer) {
  return (((t * 2 + (inner >> 4)) * 2 + (outer >> 4)) * 64 + ((inner & 15) >> 2) * 16 + (outer & 15)) * 4 + (inner & 3);
}

__device__ __forceinline__ v4f mfma16(v4s a, v4s b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// Transposing LDS read: each group of 16 lanes reads a block of 4 rows and 16 columns of
// 16-bit values (lane r of the group points at row r / 4, columns 4 (r % 4) ..) and lane r
// receives column r of the four rows: a matrix-core operand whose K index runs along rows.
typedef __attribute__((address_space(3))) v4s lds_v4s;
__device__ __forceinline__ v4s read_tr(const uint16_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)p);
}
// K = 32 operand from rows k0 .. k0 + 31 (row stride ld) and columns c0 .. c0 + 15: lane l
// holds column l % 16, rows k0 + 8 (l / 16) + j.
__device__ __forceinline__ v8s read_tr32(const uint16_t* base, int ld, int k0, int c0, int lane) {
  const uint16_t* p = base + (k0 + 8 * (lane >> 4) + ((lane & 15) >> 2)) * ld + c0 + 4 * (lane & 3);
  const v4s lo = read_tr(p), hi = read_tr(p + 4 * ld);
  return v8s{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
}

// A lane's fragments of a convolution's weights, in registers: read before the tiles are ready,
// as at one wavefront per SIMD nothing else hides their way from L2.
struct ConvWeights {
  v4s w[KW * 2][2];
  __device__ __forceinline__ void load(const uint16_t* __restrict__ frag, int lane) {
    const v4s* f = reinterpret_cast<const v4s*>(frag) + lane;
#pragma unroll
    for (int e = 0; e < KW * 2; ++e) {
      w[e][0] = f[(2 * e) * 64];
      w[e][1] = f[(2 * e + 1) * 64];
    }
  }
};

// One wavefront's share of a convolution from the tile `in` (position p at row p + 3): sums
// over taps t and channels of w times the row r0 + step t, for its 64 positions r0 ..
// r0 + 63 (rows) and all 32 outer channels.  acc[m][nb]: lane l holds outer channels
// 16 nb + 4 (l / 16) + i of position 16 m + l % 16.
__device__ __forceinline__ void conv_rows(const uint16_t* in, const ConvWeights& cw, int r0, int step, int lane,
                                          v4f (&acc)[4][2]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) acc[m][0] = acc[m][1] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < KW; ++t)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const v4s x = *reinterpret_cast<const v4s*>(in + (r0 + 16 * m + (lane & 15) + step * t) * TR_LD + 16 * h +
                                                    4 * (lane >> 4));
        acc[m][0] = mfma16(cw.w[2 * t + h][0], x, acc[m][0]);
        acc[m][1] = mfma16(cw.w[2 * t + h][1], x, acc[m][1]);
      }
}

__device__ __forceinline__ void zero_halo(uint16_t* buf, int tid) {
  if (tid < 6 * 8) {
    const int r = tid >> 3, row = r < 3 ? r : TR_ROWS - 6 + r;
    *reinterpret_cast<uint2*>(buf + row * TR_LD + 4 * (tid & 7)) = make_uint2(0u, 0u);
  }
}
// the patch's BF16 rows from HBM into the tile
__device__ __forceinline__ void load_rows(uint16_t* buf, const uint16_t* __restrict__ src, int tid) {
  for (int i = tid; i < L * C / 4; i += 256)
    *reinterpret_cast<uint2*>(buf + (3 + (i >> 3)) * TR_LD + 4 * (i & 7)) = reinterpret_cast<const uint2*>(src)[i];
}

// Forward convolutions of patch blockIdx.x.
__global__ void __launch_bounds__(256) k_train_conv_fwd(const float* __restrict__ patches,
                                                        const float* __restrict__ theta,
                                                        const uint16_t* __restrict__ f2,
                                                        const uint16_t* __restrict__ f3, float* __restrict__ u,
                                                        uint16_t* __restrict__ a1, uint16_t* __restrict__ a2,
                                                        uint16_t* __restrict__ a3) {
  __shared__ __align__(16) uint16_t b1[TR_ROWS * TR_LD], b2[TR_ROWS * TR_LD];
  __shared__ float su[L + 6];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const long s = blockIdx.x;
  ConvWeights w2, w3;
  w2.load(f2, lane);
  w3.load(f3, lane);
  const float uv = vet_u(patches[s * L + tid]);
  u[s * L + tid] = uv;
  su[3 + tid] = uv;
  if (tid < 3) su[tid] = su[L + 3 + tid] = 0.f;
  zero_halo(b1, tid);
  zero_halo(b2, tid);
  __syncthreads();
  {
    // first convolution: position tid, all channels (uniform weights)
    float x[KW];
#pragma unroll
    for (int t = 0; t < KW; ++t) x[t] = su[tid + t];
    uint2* o = reinterpret_cast<uint2*>(a1 + (s * L + tid) * C);
#pragma unroll
    for (int c = 0; c < C; c += 4) {
      v4f z;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float v = theta[O_B1 + c + i];
#pragma unroll
        for (int t = 0; t < KW; ++t) v += theta[O_W1 + (c + i) * KW + t] * x[t];
        z[i] = v;
      }
      const uint2 r = relu_bf16_tile(z);
      *reinterpret_cast<uint2*>(b1 + (3 + tid) * TR_LD + c) = r;
      o[c / 4] = r;
    }
  }
  __syncthreads();
  auto layer = [&](const uint16_t* in, const ConvWeights& cw, long bias, uint16_t* keep, uint16_t* out) {
    v4f acc[4][2];
    conv_rows(in, cw, 64 * w, 1, lane, acc);
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      const int c = 16 * nb + 4 * (lane >> 4);
      const v4f b = {theta[bias + c], theta[bias + c + 1], theta[bias + c + 2], theta[bias + c + 3]};
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int p = 64 * w + 16 * m + (lane & 15);
        const uint2 r = relu_bf16_tile(acc[m][nb] + b);
        if (keep) *reinterpret_cast<uint2*>(keep + (3 + p) * TR_LD + c) = r;
        *reinterpret_cast<uint2*>(out + (s * L + p) * C + c) = r;
      }
    }
  };
  layer(b1, w2, O_B2, b2, a2);
  __syncthreads();
  layer(b2, w3, O_B3, nullptr, a3);
}

// ---- dense head
// Per 16 patches: z4 from its split-K partial sums, bias, ReLU, BF16 (a4); z5 = a4 W5^T,
// bias, ReLU (a5); logit and loss term; dz5 = dlogit w6 [z5 > 0]; dz4 = (dz5 W5) [z4 > 0],
// both in FP32 (for the bias gradients) and BF16 (for the products).
constexpr int HP = 16, HA_LD = H + 4;
// FP32 values of a batch that the sums over patches need
struct HeadOut {
  float *a5, *dz5, *dz4, *dlogit, *term;
};
// 1024 threads for the 32 partial sums of each z4 value: at 256 patches there are only 16
// workgroups, and what a CU has in flight bounds them.  The products take the first eight
// wavefronts, 16 outputs each, with their parts of W5 read ahead.
constexpr int HEAD_NT = 1024;
__global__ void __launch_bounds__(HEAD_NT) k_train_head(const float* __restrict__ z4p, int splits, long count, int n,
                                                        const float* __restrict__ theta,
                                                        const uint16_t* __restrict__ w5b, const float* __restrict__ y,
                                                        uint16_t* __restrict__ a4b, uint16_t* __restrict__ dz5b,
                                                        uint16_t* __restrict__ dz4b, HeadOut out) {
  __shared__ __align__(16) uint16_t sa4[HP * HA_LD], sd5[HP * HA_LD];
  __shared__ float sa5[HP][H + 1], sd[HP], s6[H];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int r0 = blockIdx.x * HP;
  const int q4 = 4 * (lane >> 4), r16 = lane & 15, o = 16 * w + r16;
  const bool prod = w < H / 16;
  v4s wf[H / 16], wb[H / 16];
  float b5 = 0.f, w6 = 0.f;
  if (prod) {
#pragma unroll
    for (int k = 0; k < H / 16; ++k) {
      wf[k] = *reinterpret_cast<const v4s*>(w5b + (long)o * H + 16 * k + q4);
#pragma unroll
      for (int i = 0; i < 4; ++i) wb[k][i] = (short)w5b[(16 * k + q4 + i) * H + o];
    }
    b5 = theta[O_B5 + o];
    w6 = theta[O_W6 + o];
    if (lane < 16) s6[o] = w6;
  }
#pragma unroll
  for (int e = 0; e < HP * H / HEAD_NT; ++e) {
    const int i = tid + HEAD_NT * e, p = i / H, k = i % H, row = r0 + p;
    float acc = 0.f;
    if (row < n) {
      const float* z = z4p + (long)row * H + k;
      if (splits == 32) {
        float v[32];
#pragma unroll
        for (int q = 0; q < 32; ++q) v[q] = z[q * count];
#pragma unroll
        for (int q = 0; q < 32; ++q) acc += v[q];
      } else {
        for (int q = 0; q < splits; ++q) acc += z[q * count];
      }
      acc += theta[O_B4 + k];
    }
    const uint16_t a = f2bf(acc > 0.f ? acc : 0.f);
    sa4[p * HA_LD + k] = a;
    if (row < n) a4b[(long)row * H + k] = a;
  }
  __syncthreads();
  // z5: patches 4 (l / 16) + i, outputs 16 w + l % 16
  v4f z5 = {0.f, 0.f, 0.f, 0.f};
  if (prod) {
#pragma unroll
    for (int k = 0; k < H / 16; ++k)
      z5 = mfma16(*reinterpret_cast<const v4s*>(sa4 + r16 * HA_LD + 16 * k + q4), wf[k], z5);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      z5[i] += b5;
      const float a = z5[i] > 0.f ? z5[i] : 0.f;
      sa5[q4 + i][o] = a;
      if (r0 + q4 + i < n) out.a5[(long)(r0 + q4 + i) * H + o] = a;
    }
  }
  __syncthreads();
  if (tid < HP) {
    float l = theta[O_B6], d = 0.f;
#pragma unroll 16
    for (int j = 0; j < H; ++j) l += s6[j] * sa5[tid][j];
    if (r0 + tid < n) {
      const float yy = y[r0 + tid], sig = 1.f / (1.f + expf(-l));
      d = (sig - yy) / (float)n;
      out.dlogit[r0 + tid] = d;
      out.term[r0 + tid] = fmaxf(l, 0.f) - l * yy + log1pf(expf(-fabsf(l)));
    }
    sd[tid] = d;
  }
  __syncthreads();
  if (prod) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int p = q4 + i;
      const float g = z5[i] > 0.f ? sd[p] * w6 : 0.f;
      const uint16_t gb = f2bf(g);
      sd5[p * HA_LD + o] = gb;
      if (r0 + p < n) {
        dz5b[(long)(r0 + p) * H + o] = gb;
        out.dz5[(long)(r0 + p) * H + o] = g;
      }
    }
  }
  __syncthreads();
  if (prod) {
    v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < H / 16; ++k)
      acc = mfma16(*reinterpret_cast<const v4s*>(sd5 + r16 * HA_LD + 16 * k + q4), wb[k], acc);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int p = q4 + i;
      const float g = (short)sa4[p * HA_LD + o] > 0 ? acc[i] : 0.f;
      if (r0 + p < n) {
        dz4b[(long)(r0 + p) * H + o] = f2bf(g);
        out.dz4[(long)(r0 + p) * H + o] = g;
      }
    }
  }
}

// ---- dense layers, backward
// Weight gradients: dW[j][c] = sum_s a[s][j] x[s][c] over n patches: 128 x 64 of dW4 (a = dz4, x of 8192 columns)
// per workgroup, then dW5 (a = dz5, x = a4) in `split5` parts of `chunk5` patches, to `part5`
// if there is more than one.  Stages of 32 patches in LDS
// as they lie in memory; both operands by transposing reads.
constexpr int DW_ALD = H + 8, DW_XLD = 64 + 8, DW_TILES = X / 64;
struct DwDense {
  const uint16_t *dz4b, *x, *dz5b, *a4b;
  int n, split5, chunk5;
  float *grad, *grad_out, *part5;   // grad_out: the caller's copy, or null
};
__device__ __forceinline__ void dense_weights(const DwDense& d, int block, uint16_t* lds) {
  uint16_t *sa = lds, *sx = lds + 32 * DW_ALD;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const bool last = block >= DW_TILES;
  const uint16_t* a = last ? d.dz5b : d.dz4b;
  const uint16_t* xs = last ? d.a4b : d.x;
  const int tile = last ? (block - DW_TILES) & 1 : block, z = last ? (block - DW_TILES) >> 1 : 0;
  const int cols = last ? H : X, c0 = tile * 64;
  const int beg = last ? z * d.chunk5 : 0, end = last ? min(d.n, beg + d.chunk5) : d.n;
  const long base = last ? O_W5 : O_W4;
  const bool parts = last && d.split5 > 1;
  float* out = parts ? d.part5 + (long)z * H * H : d.grad + base;
  float* copy = parts || !d.grad_out ? nullptr : d.grad_out + base;
  uint4 ra[2], rx;
  // a: rows of 16 16-byte groups, two per thread; x: rows of 8, one per thread
  auto gload = [&](int s0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int e = tid + 256 * i, s = s0 + (e >> 4);
      ra[i] = make_uint4(0u, 0u, 0u, 0u);
      if (s < end) ra[i] = *reinterpret_cast<const uint4*>(a + (long)s * H + 8 * (e & 15));
    }
    const int s = s0 + (tid >> 3);
    rx = make_uint4(0u, 0u, 0u, 0u);
    if (s < end) rx = *reinterpret_cast<const uint4*>(xs + (long)s * cols + c0 + 8 * (tid & 7));
  };
  v4f acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  gload(beg);
  for (int s0 = beg; s0 < end; s0 += 32) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int e = tid + 256 * i;
      *reinterpret_cast<uint4*>(sa + (e >> 4) * DW_ALD + 8 * (e & 15)) = ra[i];
    }
    *reinterpret_cast<uint4*>(sx + (tid >> 3) * DW_XLD + 8 * (tid & 7)) = rx;
    __syncthreads();
    if (s0 + 32 < end) gload(s0 + 32);
    v8s fa[2], fx[4];
#pragma unroll
    for (int i = 0; i < 2; ++i) fa[i] = read_tr32(sa, DW_ALD, 0, 32 * w + 16 * i, lane);
#pragma unroll
    for (int j = 0; j < 4; ++j) fx[j] = read_tr32(sx, DW_XLD, 0, 16 * j, lane);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = mfma32(fa[i], fx[j], acc[i][j]);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const long e = (long)(32 * w + 16 * i + 4 * (lane >> 4) + k) * cols + c0 + 16 * j + (lane & 15);
        out[e] = acc[i][j][k];
        if (copy) copy[e] = acc[i][j][k];
      }
}

// Gradient of the flattened activations: dz3[s][c] = (sum_j dz4[s][j] W4[j][c]) [a3 > 0] for 64 patches and 64 columns (two
// positions), products transposed (lane: four columns of one patch); sums over each 16 patches
// to sums[s / 16][c] for the bias gradient.
constexpr int DX_LD = 64 + 8, DX_FLD = 64 + 4;
constexpr int DENSE_LDS = H * DX_LD * 2 + 64 * DX_FLD * 4;
static_assert((32 * DW_ALD + 32 * DW_XLD) * 2 <= DENSE_LDS, "both uses fit");
// The weight gradients' workgroups come first: theirs is the longer chain.
__global__ void __launch_bounds__(256) k_train_dense_bwd(DwDense dw, int ndw, const uint16_t* __restrict__ w4b,
                                                         uint16_t* __restrict__ dz3, float* __restrict__ sums) {
  __shared__ __align__(16) unsigned char lds[DENSE_LDS];
  if ((int)blockIdx.x < ndw) {
    dense_weights(dw, blockIdx.x, reinterpret_cast<uint16_t*>(lds));
    return;
  }
  const uint16_t *dz4b = dw.dz4b, *a3 = dw.x;
  const int n = dw.n, tile = (blockIdx.x - ndw) % DW_TILES, rows = (blockIdx.x - ndw) / DW_TILES;
  uint16_t* sw = reinterpret_cast<uint16_t*>(lds);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  float* sf = reinterpret_cast<float*>(lds + H * DX_LD * 2) + w * 16 * DX_FLD;
  const int c0 = tile * 64, s = rows * 64 + 16 * w + (lane & 15);
  for (int e = tid; e < H * 8; e += 256)
    *reinterpret_cast<uint4*>(sw + (e >> 3) * DX_LD + 8 * (e & 7)) =
        *reinterpret_cast<const uint4*>(w4b + (long)(e >> 3) * X + c0 + 8 * (e & 7));
  const bool in = s < n;
  v4s g[H / 16];
#pragma unroll
  for (int k = 0; k < H / 16; ++k) {
    g[k] = v4s{0, 0, 0, 0};
    if (in) g[k] = *reinterpret_cast<const v4s*>(dz4b + (long)s * H + 16 * k + 4 * (lane >> 4));
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < H / 16; ++k)
      acc = mfma16(read_tr(sw + (16 * k + (lane >> 2)) * DX_LD + 16 * b + 4 * (lane & 3)), g[k], acc);
    const int c = c0 + 16 * b + 4 * (lane >> 4);
    v4f d = {0.f, 0.f, 0.f, 0.f};
    if (in) {
      const v4s a = *reinterpret_cast<const v4s*>(a3 + (long)s * X + c);
#pragma unroll
      for (int i = 0; i < 4; ++i) d[i] = a[i] > 0 ? acc[i] : 0.f;
      *reinterpret_cast<uint2*>(dz3 + (long)s * X + c) = make_uint2(bf16_pair(d[0], d[1]), bf16_pair(d[2], d[3]));
    }
    *reinterpret_cast<v4f*>(&sf[(lane & 15) * DX_FLD + 16 * b + 4 * (lane >> 4)]) = d;
  }
  __syncthreads();
  if (rows * 64 + 16 * w < n) {
    float v = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) v += sf[k * DX_FLD + lane];
    sums[(long)(rows * 4 + w) * X + c0 + lane] = v;
  }
}

// ---- convolution gradients
// Patch blockIdx.x: da2 from dz3, masked (dz2, FP32 and BF16), da1 from that, masked; the
// patch's sums of dW1 and db1 to part1[patch][c][8], position after position: thread
// (c = tid % 32, tap or bias k = tid / 32).
constexpr int G_LD = L + 4, P1 = C * (KW + 1);
static_assert(C * G_LD * 4 <= 2 * TR_ROWS * TR_LD * 2, "dz1 fits over the two tiles");
__global__ void __launch_bounds__(256) k_train_conv_bwd(const float* __restrict__ u, const uint16_t* __restrict__ a1,
                                                        const uint16_t* __restrict__ a2,
                                                        const uint16_t* __restrict__ dz3,
                                                        const uint16_t* __restrict__ g3,
                                                        const uint16_t* __restrict__ g2, uint16_t* __restrict__ dz2b,
                                                        float* __restrict__ dz2, float* __restrict__ part1) {
  __shared__ __align__(16) uint16_t tiles[2 * TR_ROWS * TR_LD];
  __shared__ float su[L + 8];
  uint16_t *bd = tiles, *be = tiles + TR_ROWS * TR_LD;
  float* g1 = reinterpret_cast<float*>(tiles);   // dz1[c][position], once the tiles are done with
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r16 = lane & 15;
  const long s = blockIdx.x;
  ConvWeights w3, w2;
  w3.load(g3, lane);
  w2.load(g2, lane);
  load_rows(bd, dz3 + s * X, tid);
  zero_halo(bd, tid);
  zero_halo(be, tid);
  su[3 + tid] = u[s * L + tid];
  if (tid < 3) su[tid] = su[L + 3 + tid] = 0.f;
  // element of the lane's outputs m, nb: four channels of a position
  auto at = [&](int m, int nb) { return s * X + (64 * w + 16 * m + r16) * C + 16 * nb + 4 * (lane >> 4); };
  v4s k2[4][2], k1[4][2];
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      k2[m][nb] = *reinterpret_cast<const v4s*>(a2 + at(m, nb));
      k1[m][nb] = *reinterpret_cast<const v4s*>(a1 + at(m, nb));
    }
  __syncthreads();
  v4f acc[4][2];
  // da2[p] takes dz3[p - (t - 3)]: row p + 6 - t
  conv_rows(bd, w3, 64 * w + 6, -1, lane, acc);
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      v4f d;
#pragma unroll
      for (int i = 0; i < 4; ++i) d[i] = k2[m][nb][i] > 0 ? acc[m][nb][i] : 0.f;
      const uint2 h = make_uint2(bf16_pair(d[0], d[1]), bf16_pair(d[2], d[3]));
      *reinterpret_cast<uint2*>(be + (3 + 64 * w + 16 * m + r16) * TR_LD + 16 * nb + 4 * (lane >> 4)) = h;
      *reinterpret_cast<uint2*>(dz2b + at(m, nb)) = h;
      *reinterpret_cast<v4f*>(dz2 + at(m, nb)) = d;
    }
  __syncthreads();
  conv_rows(be, w2, 64 * w + 6, -1, lane, acc);
  __syncthreads();   // the tiles have been read
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        g1[(16 * nb + 4 * (lane >> 4) + i) * G_LD + 64 * w + 16 * m + r16] = k1[m][nb][i] > 0 ? acc[m][nb][i] : 0.f;
  __syncthreads();
  const int c = tid & 31, k = tid >> 5;
  float sum = 0.f;
#pragma unroll 8
  for (int p = 0; p < L; p += 4) {
    const v4f g = *reinterpret_cast<const v4f*>(g1 + c * G_LD + p);
#pragma unroll
    for (int i = 0; i < 4; ++i) sum += g[i] * (k < KW ? su[p + i + k] : 1.f);
  }
  part1[s * P1 + c * (KW + 1) + k] = sum;
}

// ---- weight gradients of the convolutions, sums for their biases
// Sum over positions p of act[p + t - 3][ci] d[p][co] in parts of `kchunk` positions (a multiple
// of 16) of the batch: workgroup (part, layer, taps 0..3 or 4..6), wavefront (half of ci, half
// of co), to part[layer][part][t 32 + ci][co].  Both operands are read transposed from
// patches staged as they lie in memory, the next patch's loads in flight meanwhile.
// The workgroups behind those add layer 2's bias gradient over each 16 patches, patch after
// patch, as k_train_dense_bwd did layer 3's: sums2[chunk][p][c].
constexpr int CP_W = KC * C;
__global__ void __launch_bounds__(256) k_train_dw_conv(const uint16_t* __restrict__ a1, const uint16_t* __restrict__ a2,
                                                       const uint16_t* __restrict__ dz2b,
                                                       const uint16_t* __restrict__ dz3b,
                                                       const float* __restrict__ dz2, int n, int splits,
                                                       int kchunk, float* __restrict__ part,
                                                       float* __restrict__ sums2) {
  __shared__ __align__(16) uint16_t ba[TR_ROWS * TR_LD], bd[TR_ROWS * TR_LD];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  int b = blockIdx.x;
  if (b >= 4 * splits) {
    b -= 4 * splits;
    const int chunk = b >> 3, e = 256 * (b & 7) + tid;   // float4 e of the chunk's 8192 values
    const v4f* src = reinterpret_cast<const v4f*>(dz2 + (long)chunk * 16 * X) + e;
    const int rows = min(16, n - 16 * chunk);
    v4f v[16], sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = src[min(r, rows - 1) * (X / 4)];
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (r < rows) sum += v[r];
    reinterpret_cast<v4f*>(sums2 + (long)chunk * X)[e] = sum;
    return;
  }
  const int z = b >> 2, layer = (b >> 1) & 1, t0 = 4 * (b & 1), ci = 16 * (w & 1), co = 16 * (w >> 1);
  const uint16_t *act = layer ? a2 : a1, *dz = layer ? dz3b : dz2b;
  const long beg = (long)z * kchunk, end = min((long)n * L, beg + kchunk);
  zero_halo(ba, tid);
  uint4 ra[4], rd[4];
  auto gload = [&](long s) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ra[i] = reinterpret_cast<const uint4*>(act + s * X)[tid + 256 * i];
      rd[i] = reinterpret_cast<const uint4*>(dz + s * X)[tid + 256 * i];
    }
  };
  v4f acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = v4f{0.f, 0.f, 0.f, 0.f};
  const int tr = lane >> 2, tc = 4 * (lane & 3);
  if (beg < end) gload(beg / L);
  for (long s = beg / L; s * L < end; ++s) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = tid + 256 * i, o = (3 + (e >> 2)) * TR_LD + 8 * (e & 3);
      *reinterpret_cast<uint2*>(ba + o) = make_uint2(ra[i].x, ra[i].y);
      *reinterpret_cast<uint2*>(ba + o + 4) = make_uint2(ra[i].z, ra[i].w);
      *reinterpret_cast<uint2*>(bd + o) = make_uint2(rd[i].x, rd[i].y);
      *reinterpret_cast<uint2*>(bd + o + 4) = make_uint2(rd[i].z, rd[i].w);
    }
    __syncthreads();
    if ((s + 1) * L < end) gload(s + 1);
    const int p0 = (int)(max(beg, s * L) - s * L), p1 = (int)(min(end, (s + 1) * L) - s * L);
    int p = p0;
    for (; p + 64 <= p1; p += 64) {
      // four steps' operands on their way before the first product (17 us for the launch at 256
      // patches with each step's reads before its products, 12 like this)
      v4s fd[4], fa[4][4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        fd[q] = read_tr(bd + (p + 16 * q + 3 + tr) * TR_LD + co + tc);
#pragma unroll
        for (int t = 0; t < 4; ++t)
          fa[q][t] = read_tr(ba + (p + 16 * q + min(t0 + t, KW - 1) + tr) * TR_LD + ci + tc);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = mfma16(fa[q][t], fd[q], acc[t]);
    }
    for (; p < p1; p += 16) {
      const v4s fd = read_tr(bd + (p + 3 + tr) * TR_LD + co + tc);
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (t0 + t < KW) acc[t] = mfma16(read_tr(ba + (p + t0 + t + tr) * TR_LD + ci + tc), fd, acc[t]);
    }
  }
  float* out = part + ((long)layer * splits + z) * CP_W;
#pragma unroll
  for (int t = 0; t < 4; ++t)
    if (t0 + t < KW)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        out[((t0 + t) * C + ci + 4 * (lane >> 4) + i) * C + co + (lane & 15)] = acc[t][i];
}

// ---- the parts added up
// Workgroups by what they add: 32 columns of the parts of the convolutions' weights, of the
// first convolution's patches or, if split, of dW5's parts, row after row; four columns of
// db2 or db3, a tree over the positions (pairs 128 apart, 64, ..) per 16 patches, those row
// after row; dW6, db6 and the loss, eight interleaved sums; 16 columns of db4 or db5, 256
// interleaved sums and their tree.
struct ReduceArgs {
  const float *conv, *part1, *sums2, *sums3, *part5;
  HeadOut head;
  int n, splits, split5;
};
constexpr int RD_CONV = 2 * CP_W / 32, RD_P1 = P1 / 32, RD_BIAS = 2 * C / 4, RD_W6 = H / 32 + 1, RD_DB = 2 * H / 16,
              RD_W5 = H * H / 32;
constexpr int RD_ROWS = 256;
__device__ __forceinline__ v4f tree64(v4f v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] += __shfl_down(v[i], o, 64);
  return v;
}
// sum over rows, in order, of column tid % 32 of src (row stride `stride`); valid for tid < 32
__device__ __forceinline__ float column_sum(const float* __restrict__ src, long stride, int rows, int tid,
                                            float (*buf)[33]) {
  float sum = 0.f;
  const int c = tid & 31;
  for (int r0 = 0; r0 < rows; r0 += RD_ROWS) {
    const int m = min(RD_ROWS, rows - r0);
    __syncthreads();
    if (m > 32) {
#pragma unroll
      for (int i = 0; i < RD_ROWS / 8; ++i) {
        const int r = (tid >> 5) + 8 * i;
        if (r < m) buf[r][c] = src[(r0 + r) * stride + c];
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = (tid >> 5) + 8 * i;
        if (r < m) buf[r][c] = src[(r0 + r) * stride + c];
      }
    }
    __syncthreads();
    if (tid < 32) {
#pragma unroll 16
      for (int r = 0; r < m; ++r) sum += buf[r][c];
    }
  }
  return sum;
}
__global__ void __launch_bounds__(256) k_train_reduce(ReduceArgs a, float* __restrict__ grad,
                                                      float* __restrict__ grad_out, float* __restrict__ loss,
                                                      float* __restrict__ loss_out) {
  __shared__ float buf[RD_ROWS][33];
  const int tid = threadIdx.x, n = a.n;
  auto put = [&](long e, float v) {
    grad[e] = v;
    if (grad_out) grad_out[e] = v;
  };
  int b = blockIdx.x;
  if (b < RD_DB) {
    // db5, then db4: wavefront of four columns, lane the rows lane, + 64, + 128, + 192 modulo 256
    const int lane = tid & 63, col = 4 * (4 * b + (tid >> 6)), c = col % H;
    const float* src = col < H ? a.head.dz5 : a.head.dz4;
    v4f total = {0.f, 0.f, 0.f, 0.f};
    for (int r0 = 0; r0 < n; r0 += 4096) {
      v4f v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = v4f{0.f, 0.f, 0.f, 0.f};
      const int r1 = min(n, r0 + 4096);
#pragma unroll 4
      for (int r = r0 + lane; r < r1; r += 256)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (r + 64 * q < r1) v[q] += *reinterpret_cast<const v4f*>(src + (long)(r + 64 * q) * H + c);
      total += tree64((v[0] + v[2]) + (v[1] + v[3]));
    }
    if (lane == 0)
#pragma unroll
      for (int i = 0; i < 4; ++i) put((col < H ? O_B5 : O_B4) + c + i, total[i]);
    return;
  }
  b -= RD_DB;
  if (b < RD_W6) {
    const int c = tid & 31, k = tid >> 5;
    float acc = 0.f;
    if (b < H / 32) {
#pragma unroll 16
      for (int s = k; s < n; s += 8) acc += a.head.dlogit[s] * a.head.a5[(long)s * H + 32 * b + c];
    } else if (c < 2) {
      const float* src = c ? a.head.term : a.head.dlogit;
#pragma unroll 16
      for (int s = k; s < n; s += 8) acc += src[s];
    }
    buf[k][c] = acc;
    __syncthreads();
    if (k != 0) return;
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) sum += buf[q][c];
    if (b < H / 32) {
      put(O_W6 + 32 * b + c, sum);
    } else if (c == 0) {
      put(O_B6, sum);
    } else if (c == 1) {
      *loss = sum / (float)n;
      if (loss_out) *loss_out = sum / (float)n;
    }
    return;
  }
  b -= RD_W6;
  if (b < RD_BIAS) {
    const int chunks = (n + 15) / 16, layer = b >= C / 4, c = 4 * (b % (C / 4));
    const int lane = tid & 63, w = tid >> 6;
    const float* src = (layer ? a.sums3 : a.sums2) + lane * C + c;
    float sum = 0.f;
    for (int k0 = 0; k0 < chunks; k0 += 32) {
      const int m = min(32, chunks - k0);
      __syncthreads();
#pragma unroll 4
      for (int k = w; k < m; k += 4) {
        const float* q = src + (long)(k0 + k) * X;
        v4f v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const v4f*>(q + 64 * i * C);
        const v4f t = tree64((v[0] + v[2]) + (v[1] + v[3]));
        if (lane == 0)
#pragma unroll
          for (int i = 0; i < 4; ++i) buf[k][i] = t[i];
      }
      __syncthreads();
      if (tid < 4)
        for (int k = 0; k < m; ++k) sum += buf[k][tid];
    }
    if (tid < 4) put((layer ? O_B3 : O_B2) + c + tid, sum);
    return;
  }
  b -= RD_BIAS;
  if (b < RD_P1) {
    const float v = column_sum(a.part1 + 32 * b, P1, n, tid, buf);
    const int e = 32 * b + tid, c = e / (KW + 1), t = e % (KW + 1);
    if (tid < 32) put(t == KW ? O_B1 + c : O_W1 + c * KW + t, v);
    return;
  }
  b -= RD_P1;
  if (b < RD_CONV) {
    const int layer = b >= RD_CONV / 2, e0 = 32 * (b - layer * (RD_CONV / 2));
    const float v = column_sum(a.conv + (long)layer * a.splits * CP_W + e0, CP_W, a.splits, tid, buf);
    const int ci = (e0 / C) % C, t = e0 / (C * C);
    if (tid < C) put((layer ? O_W3 : O_W2) + (tid * C + ci) * KW + t, v);
    return;
  }
  b -= RD_CONV;
  const float v = column_sum(a.part5 + 32 * b, H * H, a.split5, tid, buf);
  if (tid < 32) put(O_W5 + 32 * b + tid, v);
}

// ---- update
// STEP: one Adam step on the FP32 master vector (bias-corrected step size precomputed on the
// host); then the BF16 copies of the matrices: w4, w5 as they are, the convolutions as
// fragments for scoring (wq: [t][nb][lane][8]) and training (f forward, g backward).
struct WeightCopies {
  uint16_t *w4b, *w5b, *wq2, *wq3, *f2, *f3, *g2, *g3;
};
template <bool STEP>
__global__ void __launch_bounds__(256) k_vet_update(float* __restrict__ theta, const float* __restrict__ g,
                                                    float* __restrict__ m1, float* __restrict__ m2, WeightCopies wc,
                                                    float step, float b1, float b2, float eps) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= N_PARAMS) return;
  float v = theta[i];
  if constexpr (STEP) {
    const float gi = g[i];
    const float a = b1 * m1[i] + (1.f - b1) * gi;
    const float b = b2 * m2[i] + (1.f - b2) * gi * gi;
    m1[i] = a;
    m2[i] = b;
    v -= step * a / (sqrtf(b) + eps);
    theta[i] = v;
  }
  const uint16_t h = f2bf(v);
  if (i >= O_W4 && i < O_B4) {
    wc.w4b[i - O_W4] = h;
  } else if (i >= O_W5 && i < O_B5) {
    wc.w5b[i - O_W5] = h;
  } else {
    const bool second = i >= O_W2 && i < O_B2, third = i >= O_W3 && i < O_B3;
    if (second || third) {
      const int r = (int)(i - (second ? O_W2 : O_W3)), co = r / (C * KW), ci = (r / KW) % C, t = r % KW;
      (second ? wc.wq2 : wc.wq3)[((t * 2 + (co >> 4)) * 64 + (ci >> 3) * 16 + (co & 15)) * 8 + (ci & 7)] = h;
      (second ? wc.f2 : wc.f3)[frag16(t, ci, co)] = h;
      (second ? wc.g2 : wc.g3)[frag16(t, co, ci)] = h;
    }
  }
}

}  // namespace vet
}  // namespace fstat
