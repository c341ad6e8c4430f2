// Learned initialisation of inserted Gaussians: a small MLP (32 -> 64 -> 64
// -> 7, GELU) on BF16 MFMA with FP32 accumulation (its neighbour features:
// near.hip).
//
// Parameters: one FP32 vector of 6727 master weights, W1 [32][64], b1 [64],
// W2 [64][64], b2 [64], W3 [64][7], b3 [7] (z = x W + b).  Weights, the
// features and each hidden activation are rounded to BF16 (nearest, ties to
// even) where they enter a product; biases, pre-activations and GELU are
// FP32.  Backward: every gradient entering a product is rounded to BF16,
// bias gradients are not, and the rounding of weights and activations
// passes gradients unchanged.
//
// MFMA: v_mfma_f32_16x16x16_bf16 (one wave computes a 16x16 FP32 tile);
// lane l holds A[l % 16][4 (l / 16) + i], B[4 (l / 16) + i][l % 16] and
// D[4 (l / 16) + i][l % 16] for i = 0..3.  Every operand is kept with its
// contraction axis contiguous, so a lane's four values are one 8-byte LDS
// access or come straight from memory.

#include <math.h>

#include "gs_internal.h"

namespace gs {
namespace {

typedef short s4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int kIn = 32, kHid = 64, kOut = 7, kOutPad = 16;
constexpr int kOffW1 = 0, kOffB1 = kOffW1 + kIn * kHid;
constexpr int kOffW2 = kOffB1 + kHid, kOffB2 = kOffW2 + kHid * kHid;
constexpr int kOffW3 = kOffB2 + kHid, kOffB3 = kOffW3 + kHid * kOut;
constexpr int kParams = kOffB3 + kOut;
static_assert(kParams == 6727, "parameter count");

__device__ __forceinline__ unsigned short to_bf16(float f) {
  unsigned u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}

__device__ __forceinline__ float gelu(float z) {
  return 0.5f * z * (1.f + erff(z * 0.70710678118654752f));
}

__device__ __forceinline__ float gelu_grad(float z) {
  return 0.5f * (1.f + erff(z * 0.70710678118654752f)) +
         z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

__device__ __forceinline__ f4v mfma(s4v a, s4v b, f4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

constexpr int kLd = 72;   // LDS row stride of 64 values (16-byte rows, spread banks)

// Four consecutive values from p: one 16-byte load where the arrays allow it.
__device__ __forceinline__ float4 load4(const float* p, bool aligned) {
  if (aligned) return *(const float4*)p;
  return make_float4(p[0], p[1], p[2], p[3]);
}

__device__ __forceinline__ s4v pack(float4 f) {
  return s4v{(short)to_bf16(f.x), (short)to_bf16(f.y), (short)to_bf16(f.z),
             (short)to_bf16(f.w)};
}

__device__ __forceinline__ s4v lds4(const unsigned short* p) {
  return *(const s4v*)p;
}

// B operand of rows kb .. of a row-major [K][ldb] weight matrix, column c.
__device__ __forceinline__ s4v weight_frag(const float* w, int ldb, int k, int c) {
  return pack(make_float4(w[k * ldb + c], w[(k + 1) * ldb + c],
                          w[(k + 2) * ldb + c], w[(k + 3) * ldb + c]));
}

// (v - mean) / deviation per component, correctly rounded like the separate
// operations it stands for.
__device__ __forceinline__ float4 normalised(float4 v, float4 mu, float4 sd) {
  return make_float4((v.x - mu.x) / sd.x, (v.y - mu.y) / sd.y,
                     (v.z - mu.z) / sd.z, (v.w - mu.w) / sd.w);
}

// A workgroup of four waves takes 16 rows at a time through all three
// layers; wave v computes the columns 16 v .. of both hidden layers, so its
// weights (6 operands, and the 4 of the last layer) stay in registers, read
// once per workgroup.  The hidden activations meet in LDS.  What bounds it is
// latency (weights, rows, three dependent layers): 864 rows 4.6 us, 8,192
// rows 6.7 us; with 64 rows per workgroup, weights staged in LDS and two-byte
// operand reads 16.4 us (14 workgroups) and 21.2 us.
// NORM: the features are normalised as they are read, and with `denorm` the
// outputs are brought back as they are written (a prediction: four launches
// of 3.2 us each less), or the gradient vector g and the loss are cleared for
// the rest of a training step.
template <bool NORM>
__global__ __launch_bounds__(256) void k_mlp_fwd(const float* w, const float* x,
                                                 int M, float* y, float* cache,
                                                 bool aligned, MlpNorm nm,
                                                 bool denorm, float* g,
                                                 double* loss) {
  __shared__ __align__(16) unsigned short h1[16 * kLd], h2[16 * kLd];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int m = lane & 15, q = 4 * (lane >> 4);
  const int c = 16 * wv + m;   // this lane's hidden column
  s4v w1[2], w2[4], w3[4];
#pragma unroll
  for (int i = 0; i < 2; ++i) w1[i] = weight_frag(w + kOffW1, kHid, 16 * i + q, c);
#pragma unroll
  for (int i = 0; i < 4; ++i) w2[i] = weight_frag(w + kOffW2, kHid, 16 * i + q, c);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    w3[i] = weight_frag(w + kOffW3, kOut, 16 * i + q, min(m, kOut - 1));
    if (m >= kOut) w3[i] = s4v{0, 0, 0, 0};
  }
  const float b1 = w[kOffB1 + c], b2 = w[kOffB2 + c];
  const float b3 = m < kOut ? w[kOffB3 + m] : 0.f;
  float4 mu[2], sd[2];
  float out_mu = 0.f, out_sd = 1.f;
  if (NORM) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      mu[i] = load4(nm.x_mu + 16 * i + q, false);
      sd[i] = load4(nm.x_sd + 16 * i + q, false);
    }
    if (denorm && m < kOut) {
      out_mu = nm.y_mu[m];
      out_sd = nm.y_sd[m];
    }
    if (g)
      for (int i = blockIdx.x * 256 + threadIdx.x; i < kParams; i += gridDim.x * 256)
        g[i] = 0.f;
    if (loss && blockIdx.x == 0 && threadIdx.x == 0) *loss = 0.0;
  }
  const int blocks = (M + 15) / 16;
  for (int b = blockIdx.x, t = 0; b < blocks; b += gridDim.x, ++t) {
    const int row0 = 16 * b;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    const float* xr = x + (size_t)min(row0 + m, M - 1) * kIn + q;
    float4 xa = load4(xr, aligned), xb = load4(xr + 16, aligned);
    if (NORM) {
      xa = normalised(xa, mu[0], sd[0]);
      xb = normalised(xb, mu[1], sd[1]);
    }
    if (row0 + m >= M) xa = xb = zero;
    f4v z = {0.f, 0.f, 0.f, 0.f};
    z = mfma(pack(xa), w1[0], z);
    z = mfma(pack(xb), w1[1], z);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = q + i;
      const float v = z[i] + b1;
      if (cache && row0 + r < M) cache[(size_t)(row0 + r) * 128 + c] = v;
      h1[r * kLd + c] = to_bf16(gelu(v));
    }
    __syncthreads();
    z = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) z = mfma(lds4(h1 + m * kLd + 16 * i + q), w2[i], z);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = q + i;
      const float v = z[i] + b2;
      if (cache && row0 + r < M) cache[(size_t)(row0 + r) * 128 + 64 + c] = v;
      h2[r * kLd + c] = to_bf16(gelu(v));
    }
    __syncthreads();
    if (wv != (t & 3)) continue;   // the waves take the last layer in turn
    z = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) z = mfma(lds4(h2 + m * kLd + 16 * i + q), w3[i], z);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (m < kOut && row0 + q + i < M) {
        float v = z[i] + b3;
        if (NORM && denorm) v = __fadd_rn(__fmul_rn(v, out_sd), out_mu);
        y[(size_t)(row0 + q + i) * kOut + m] = v;
      }
  }
}

// A workgroup of 16 waves takes 64 rows at a time, wave v the 16 rows and 16
// columns of block (v / 4, v % 4) of both hidden layers, and keeps its sums
// of the weight gradients in registers (one 16x16 block of dW2 per wave, one
// of dW1 or dW3 in most) until its rows are done: one atomic per weight and
// workgroup.  The activations and gradients go to LDS transposed, so that
// the rows, the contraction axis of the weight gradients, are contiguous; a
// lane's four results are four such rows.  What bounds it at 8,192 rows is
// latency: the loads, the error function and exponential of a lane's values
// one after another (hence few values per lane: four waves with 16 rows and
// all 64 columns each spent 7.7 us there, 23.8 us in all against 19.2), and
// the atomics on 6,727 shared addresses (2,000 rows, 32 workgroups, 11 us).
// Four waves, 64 rows per workgroup, two-byte operand reads and an LDS
// atomic per bias term took 41.5 us.
struct MlpBwdShared {
  unsigned short h1[kHid * kLd], h2[kHid * kLd];     // [column][row]
  unsigned short d1[kHid * kLd], d2[kHid * kLd];     // [column][row]
  unsigned short x[kIn * kLd], dy[kOutPad * kLd];    // [column][row]
  unsigned short r2[64 * kLd];                       // dZ2 [row][column]
  float db[2 * kHid + kOutPad];
};
constexpr int kBwdThreads = 1024;

template <bool NORM>
__global__ __launch_bounds__(kBwdThreads) void k_mlp_bwd(
    const float* w, const float* x, const float* cache, const float* dy, int M,
    float* dw, bool aligned, MlpNorm nm) {
  __shared__ __align__(16) MlpBwdShared S;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int m = lane & 15, q = 4 * (lane >> 4);
  const int r0 = 16 * (wv >> 2), c0 = 16 * (wv & 3), c = c0 + m;
  // W3^T and W2^T operands: B[k][n] = W[n][k], column c of both products.
  s4v w3, w2[4];
  {
    const float* w3r = w + kOffW3 + c * kOut;
    float f[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = q + i < kOut ? w3r[min(q + i, kOut - 1)] : 0.f;
    w3 = pack(make_float4(f[0], f[1], f[2], f[3]));
#pragma unroll
    for (int i = 0; i < 4; ++i)
      w2[i] = pack(load4(w + kOffW2 + c * kHid + 16 * i + q, aligned));
  }
  if (tid < 2 * kHid + kOutPad) S.db[tid] = 0.f;
  const f4v zero4 = {0.f, 0.f, 0.f, 0.f};
  f4v g13 = zero4, g2 = zero4;   // dW1 (waves 0-7) or dW3 (waves 8-11), dW2
  float b1 = 0.f, b2 = 0.f, b3[4] = {0.f, 0.f, 0.f, 0.f};
  const int blocks = (M + 63) / 64;
  for (int b = blockIdx.x; b < blocks; b += gridDim.x) {
    const int row0 = 64 * b;
    // All loads first.  Pre-activations in the layout of the products'
    // results: rows r0 + q + i, column c.
    float z1[4], z2[4], xv[2], dv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = row0 + r0 + q + i;
      const float* cr = cache + (size_t)min(r, M - 1) * 128 + c;
      z2[i] = r < M ? cr[64] : 0.f;
      z1[i] = r < M ? cr[0] : 0.f;
      // dY row r0 + m, columns q + i.
      const int rd = row0 + r0 + m;
      dv[i] = rd < M && q + i < kOut ? dy[(size_t)rd * kOut + q + i] : 0.f;
    }
    const int xc = tid & 31, xr = 2 * (tid >> 5);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      xv[i] = 0.f;
      if (row0 + xr + i < M) {
        xv[i] = x[(size_t)(row0 + xr + i) * kIn + xc];
        if (NORM) xv[i] = (xv[i] - nm.x_mu[xc]) / nm.x_sd[xc];
      }
    }
    __syncthreads();   // the previous rows' products are done
    *(uint32_t*)(S.x + xc * kLd + xr) =
        (uint32_t)to_bf16(xv[0]) | ((uint32_t)to_bf16(xv[1]) << 16);
    const s4v da = pack(make_float4(dv[0], dv[1], dv[2], dv[3]));
    if (c0 == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        S.dy[(q + i) * kLd + r0 + m] = (unsigned short)da[i];
        b3[i] += dv[i];
      }
    }
    // dZ2 = (dY W3^T) * gelu'(Z2).
    {
      const f4v acc = mfma(da, w3, zero4);
      float h[4], d[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        h[i] = gelu(z2[i]);
        d[i] = acc[i] * gelu_grad(z2[i]);
        b2 += d[i];
        S.r2[(r0 + q + i) * kLd + c] = to_bf16(d[i]);
      }
      *(s4v*)(S.h2 + c * kLd + r0 + q) = pack(make_float4(h[0], h[1], h[2], h[3]));
      *(s4v*)(S.d2 + c * kLd + r0 + q) = pack(make_float4(d[0], d[1], d[2], d[3]));
    }
    float h[4], s[4];   // while the others finish dZ2
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      h[i] = gelu(z1[i]);
      s[i] = gelu_grad(z1[i]);
    }
    __syncthreads();
    // dZ1 = (dZ2 W2^T) * gelu'(Z1).
    f4v acc = zero4;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      acc = mfma(lds4(S.r2 + (r0 + m) * kLd + 16 * i + q), w2[i], acc);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[i] = acc[i] * s[i];
      b1 += s[i];
    }
    *(s4v*)(S.h1 + c * kLd + r0 + q) = pack(make_float4(h[0], h[1], h[2], h[3]));
    *(s4v*)(S.d1 + c * kLd + r0 + q) = pack(make_float4(s[0], s[1], s[2], s[3]));
    __syncthreads();
    // Weight gradients over the 64 rows: block (r0, c0) of dW2; of dW1 in
    // waves 0-7; rows 16 (v - 8) .. of dW3 in waves 8-11.
#pragma unroll
    for (int k = 0; k < 64; k += 16) {
      g2 = mfma(lds4(S.h1 + (r0 + m) * kLd + k + q), lds4(S.d2 + c * kLd + k + q), g2);
      if (wv < 8)
        g13 = mfma(lds4(S.x + (r0 + m) * kLd + k + q), lds4(S.d1 + c * kLd + k + q), g13);
      else if (wv < 12)
        g13 = mfma(lds4(S.h2 + (16 * (wv - 8) + m) * kLd + k + q),
                   lds4(S.dy + m * kLd + k + q), g13);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    atomicAdd(&dw[kOffW2 + (r0 + q + i) * kHid + c], g2[i]);
    if (wv < 8)
      atomicAdd(&dw[kOffW1 + (r0 + q + i) * kHid + c], g13[i]);
    else if (wv < 12 && m < kOut)
      atomicAdd(&dw[kOffW3 + (16 * (wv - 8) + q + i) * kOut + m], g13[i]);
  }
  // Bias gradients (unrounded): over the lanes that share a column, then the
  // waves.
  b1 += __shfl_xor(b1, 16, 64);
  b2 += __shfl_xor(b2, 16, 64);
  b1 += __shfl_xor(b1, 32, 64);
  b2 += __shfl_xor(b2, 32, 64);
  if (lane < 16) {
    atomicAdd(&S.db[c], b1);
    atomicAdd(&S.db[kHid + c], b2);
  }
  if (c0 == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {   // column q + i
      float t = b3[i];
      for (int off = 8; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
      if (m == 0) atomicAdd(&S.db[2 * kHid + q + i], t);
    }
  }
  __syncthreads();
  if (tid < kHid) {
    atomicAdd(&dw[kOffB1 + tid], S.db[tid]);
  } else if (tid < 2 * kHid) {
    atomicAdd(&dw[kOffB2 + tid - kHid], S.db[tid]);
  } else if (tid < 2 * kHid + kOut) {
    atomicAdd(&dw[kOffB3 + tid - 2 * kHid], S.db[tid]);
  }
}

template <bool NORM>
__global__ __launch_bounds__(256) void k_mlp_mse(const float* y, const float* t,
                                                 int n, float scale, float* dy,
                                                 double* loss, MlpNorm nm) {
  __shared__ double part[4];
  double s = 0.0;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    const int c = i % kOut;
    const float d = y[i] - (NORM ? (t[i] - nm.y_mu[c]) / nm.y_sd[c] : t[i]);
    dy[i] = scale * d;
    s += (double)d * (double)d;
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0 && loss)
    atomicAdd(loss, (part[0] + part[1] + part[2] + part[3]) / (double)n);
}

__global__ __launch_bounds__(256) void k_mlp_adam(float* w, const float* g,
                                                  float* m, float* v, float lr,
                                                  float b1, float b2, float eps,
                                                  float c1, float c2) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= kParams) return;
  const float gr = g[i];
  const float mm = b1 * m[i] + (1.f - b1) * gr;
  const float vv = b2 * v[i] + (1.f - b2) * gr * gr;
  m[i] = mm;
  v[i] = vv;
  w[i] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
}

// Workgroups of the backward: more share the rows of large batches, and each
// adds its 6,727 sums to the same addresses (65,536 rows: 64 workgroups 88
// us, 128 54 us, 256 45 us; 30,000 rows: 45, 30, 32 us).
constexpr int kBwdBlocks = 256;

}  // namespace

hipError_t launch_mlp_fwd(const float* w, const float* x, int M, float* y,
                          float* cache, hipStream_t st) {
  if (M > 0)
    hipLaunchKernelGGL(k_mlp_fwd<false>, dim3(min((M + 15) / 16, 1024)),
                       dim3(256), 0, st, w, x, M, y, cache,
                       ((uintptr_t)x & 15) == 0, MlpNorm{}, false, nullptr,
                       nullptr);
  return hipGetLastError();
}

hipError_t launch_mlp_predict(const float* w, const float* x, int M,
                              const MlpNorm& nm, float* y, hipStream_t st) {
  if (M > 0)
    hipLaunchKernelGGL(k_mlp_fwd<true>, dim3(min((M + 15) / 16, 1024)),
                       dim3(256), 0, st, w, x, M, y, nullptr,
                       ((uintptr_t)x & 15) == 0, nm, true, nullptr, nullptr);
  return hipGetLastError();
}

// One training step (M > 0).  scratch: [M][128] pre-activations, [M][7]
// outputs, [M][7] their gradient.  Four launches; features and targets are
// normalised where they are read (8,192 rows: 66 us with four launches for
// that and two to clear, bound by issuing them).
hipError_t launch_mlp_train(float* w, const float* x, const float* t, int M,
                            const MlpNorm& nm, float* scratch, double* loss,
                            float* g, float* m, float* v, float lr, float b1,
                            float b2, float eps, int step, hipStream_t st) {
  float* cache = scratch;
  float* y = cache + (size_t)M * 128;
  float* dy = y + (size_t)M * kOut;
  hipLaunchKernelGGL(k_mlp_fwd<true>, dim3(min((M + 15) / 16, 1024)), dim3(256),
                     0, st, w, x, M, y, cache, ((uintptr_t)x & 15) == 0, nm,
                     false, g, loss);
  const int n = M * kOut;
  hipLaunchKernelGGL(k_mlp_mse<true>, dim3(min((n + 255) / 256, 120)),
                     dim3(256), 0, st, y, t, n, 2.f / (float)n, dy, loss, nm);
  hipLaunchKernelGGL(k_mlp_bwd<true>, dim3(min((M + 63) / 64, kBwdBlocks)),
                     dim3(kBwdThreads), 0, st, w, x, cache, dy, M, g,
                     ((uintptr_t)w & 15) == 0, nm);
  return launch_mlp_adam(w, g, m, v, lr, b1, b2, eps, step, st);
}

hipError_t launch_mlp_bwd(const float* w, const float* x, const float* cache,
                          const float* dy, int M, float* dw, hipStream_t st) {
  if (M > 0)
    hipLaunchKernelGGL(k_mlp_bwd<false>, dim3(min((M + 63) / 64, kBwdBlocks)),
                       dim3(kBwdThreads), 0, st, w, x, cache, dy, M, dw,
                       ((uintptr_t)w & 15) == 0, MlpNorm{});
  return hipGetLastError();
}

hipError_t launch_mlp_mse(const float* y, const float* t, int M, float* dy,
                          double* loss, hipStream_t st) {
  const int n = M * kOut;
  if (n <= 0) return hipSuccess;
  int blocks = (n + 255) / 256;
  if (blocks > 120) blocks = 120;
  hipLaunchKernelGGL(k_mlp_mse<false>, dim3(blocks), dim3(256), 0, st, y, t, n,
                     2.f / (float)n, dy, loss, MlpNorm{});
  return hipGetLastError();
}

hipError_t launch_mlp_adam(float* w, const float* g, float* m, float* v,
                           float lr, float b1, float b2, float eps, int step,
                           hipStream_t st) {
  const float c1 = (float)(1.0 - pow((double)b1, step));
  const float c2 = (float)(1.0 - pow((double)b2, step));
  hipLaunchKernelGGL(k_mlp_adam, dim3((kParams + 255) / 256), dim3(256), 0, st,
                     w, g, m, v, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

}  // namespace gs
