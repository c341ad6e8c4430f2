// Structural-similarity term of the colour loss (Eq. 10) and its gradient.
//
// Per channel and pixel: window sums over an 11 x 11 Gaussian window
// (sigma 1.5, normalised, zero padding outside the image) of x, y, x^2, y^2
// and x y give mu_x, mu_y, var_x, var_y and cov; SSIM = A1 A2 / (B1 B2) with
// A1 = 2 mu_x mu_y + C1, A2 = 2 cov + C2, B1 = mu_x^2 + mu_y^2 + C1,
// B2 = var_x + var_y + C2 (C1 = 0.01^2, C2 = 0.03^2).  The loss adds
// lam * sum over views of (1 - mean SSIM over 3HW).
//
// The gradient is a second window sum: with D1, D2, D3 the per-pixel
// derivatives of the term with respect to mu_x, the sum of x^2 (which equals
// that of y^2) and the sum of x y, zero outside the image, and the window
// symmetric, dL/dx(p) += D1(p) + 2 x(p) D2(p) + y(p) D3(p) over the windowed
// maps.
//
// One pass (k_ssim): a workgroup walks down a strip of columns, four rows per
// step.  Both window sums run vertically first, then horizontally.
//   Vertical, one thread per column: four output rows of a map are a 4 x 14
// band of weights times 14 input rows; the 4x4x1 matrix instruction (16
// blocks of 4 rows x 4 columns, so that a lane's own column is its operand
// and its result) adds one input row to four output rows, 14 instructions
// where vector FMAs take 44, beside the vector unit.
//   Horizontal, one thread per four columns of a row, which the threads
// exchange through LDS: 14 reads serve 44 taps.
// The images are read once (10 rows and columns of overlap around a strip),
// the gradient is written once; the statistics need only four maps (x, y,
// (x - y)^2, x y):
//   B1 = A1 + (mu_x - mu_y)^2,  B2 = A2 + var(x - y),
// so that where the images resemble one another the rounding of A1 and A2 is
// that of B1 and B2 and leaves the quotients (a sum of x^2 + y^2 in the third
// map's place is one rounding of twice the size and does not: the gradient of
// a rendering close to its target was 1.2 times as far off).
//
// Bound by the horizontal sums: 308 FMAs per four pixels in a row plus the
// pointwise terms, about 500 vector instructions, at two waves per SIMD (240
// registers for the two sets of 28 open sums; at three the sums spill, 2
// times slower), which issue 0.47 of what the vector units take, with the
// matrix units busy 0.15 of the time: the chain of a step between its three
// barriers is not covered by one other wave.  Two sets of LDS buffers instead of three, with a barrier
// more per step, was 3 % slower.  In place of a statistics and a gradient
// kernel with the derivative maps in memory between them: ten 680 x 1200 views
// 284 us (was 405; 9.8 MB per plane in and out), one 41 (92), ten 480 x 640
// 103 (161), one 251 x 377 16.8 (21.2).  Small inputs keep those two kernels
// (ssim_tiles.hip, use_tiles).

#include <float.h>
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "gs_internal.h"

namespace gs {
namespace {

typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int kR = 5;                   // window radius
constexpr int kTaps = 2 * kR + 1;
constexpr int kRows = 4;                // rows per step
constexpr int kSpan = kTaps + kRows - 1;   // inputs of four outputs (14)
constexpr int kLag = 6;                 // steps from a row's load to its output
constexpr float kC1 = 0.01f * 0.01f, kC2 = 0.03f * 0.03f;
constexpr float kBig = 1e37f;           // its reciprocal is a normal number

struct SsimArgs {
  float w[kR + 1];      // normalised 1D window, taps 0 .. 5 (symmetric)
  const float* x;       // rendered [V][3][H][W]
  const float* y;       // target
  float* dL;            // [V][3][H][W], accumulated
  double* loss;
  double* ssim;         // [V] mean SSIM, accumulated (may be null)
  int V, H, W;
  int strip, rows;      // output columns and rows of a workgroup
  float lam;
  // L1 term fused in (l1 != 0): lam_l1 mean |x - y| is added to the loss and
  // the squared errors to sqerr, and dL is WRITTEN as lam_l1 sign(x - y) /
  // (3HW) + the SSIM gradient instead of added to.
  int l1;
  int aligned;         // rows of 16-byte aligned groups of four pixels
  float l1_scale;      // lam_l1 / (3HW)
  double l1_lam_inv;   // lam_l1 / (3HW) in FP64
  double* sqerr;       // [V], may be null
};

// Vertical window sums of N maps, four rows at a time.  Group g holds the
// output rows 4 g .. 4 g + 3 and takes the input rows 4 g .. 4 g + 13 (input
// row n is output row n - 5).  Step s first adds two of its four input rows
// to group s - 3, which is then finished, and afterwards all four to the
// groups s - 2, s - 1 and s, the last in the registers of the finished one.
// S: the step modulo 3, so that the groups' registers are constants of the
// unrolled loop.  band: lane 4 k + i holds tap k - i, the weight of input row
// k of a group for its output row i; the instruction broadcasts block k.
// It multiplies every input row by every weight, and 0 times infinity or NaN
// would reach output rows whose window does not hold that input.  Rows that
// are not finite are therefore added as zeros and the windows that hold them
// are set to NaN, what their statistics come to in any case.  Of the four
// maps of the statistics the squares alone may run over, where they still
// come to an SSIM of 0: these are added as zeros too, and their map's windows
// set to infinity.
template <int N>
struct VerticalSums {
  f4v acc[N][3];
  static constexpr int kSquares = N == 4 ? 2 : -1;   // the statistics' map
  unsigned bad;   // bit b: the input row 3 - b (of this step) is not finite,
                  // bit 16 + b: only its squares are not
  // check: not finite where one of v is not.
  __device__ __forceinline__ void screen(float check, float (&v)[kRows][N]) {
    bad = (bad << kRows) & 0xfff0fff0u;
    if (!__any(!(fabsf(check) <= FLT_MAX))) return;
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
      bool finite = true, square = true;
#pragma unroll
      for (int m = 0; m < N; ++m) {
        const bool f = fabsf(v[j][m]) <= FLT_MAX;
        if (m == kSquares) square = f;
        else finite = finite && f;
      }
      bad |= (finite ? square ? 0u : 0x10000u : 1u) << (kRows - 1 - j);
#pragma unroll
      for (int m = 0; m < N; ++m)
        v[j][m] = finite && (m != kSquares || square) ? v[j][m] : 0.f;
    }
  }
  // Output row i of the finished group takes the input rows i - 12 .. i - 2.
  template <int S>
  __device__ __forceinline__ void mark() {
    if (!__any(bad)) return;
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
      const unsigned rows = 0x7ffu << (5 - i);
      acc[0][S][i] = bad & rows ? NAN : acc[0][S][i];
      if (kSquares >= 0)
        acc[max(kSquares, 0)][S][i] =
            bad & (rows << 16) ? INFINITY : acc[max(kSquares, 0)][S][i];
    }
  }
  template <int G, int K>
  __device__ __forceinline__ void row(float band, const float (&v)[N]) {
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const f4v c = K == 0 ? f4v{0.f, 0.f, 0.f, 0.f} : acc[m][G];
      acc[m][G] = __builtin_amdgcn_mfma_f32_4x4x1f32(band, v[m], c, 4, K, 0);
    }
  }
  // Group s - 3, in the registers acc[..][S].
  template <int S>
  __device__ __forceinline__ void finish(float band, const float (&v)[kRows][N]) {
    row<S, 12>(band, v[0]);
    row<S, 13>(band, v[1]);
    mark<S>();
  }
  template <int S>
  __device__ __forceinline__ void add(float band, const float (&v)[kRows][N]) {
    constexpr int P = (S + 2) % 3, Q = (S + 1) % 3;   // groups s - 1, s - 2
    row<Q, 8>(band, v[0]);
    row<P, 4>(band, v[0]);
    row<S, 0>(band, v[0]);
    row<Q, 9>(band, v[1]);
    row<P, 5>(band, v[1]);
    row<S, 1>(band, v[1]);
    row<Q, 10>(band, v[2]);
    row<P, 6>(band, v[2]);
    row<S, 2>(band, v[2]);
    row<Q, 11>(band, v[3]);
    row<P, 7>(band, v[3]);
    row<S, 3>(band, v[3]);
  }
};

// Four exchanged rows.  Column c (of the workgroup, from -8 on) at word c + 8
// with one spare word after every fourth: the four-column reads of eight
// lanes then fall in distinct banks.
template <int NT>
struct Exchange {
  static constexpr int kWords = (NT + 16) * 5 / 4;
  float4 v[kRows][kWords];
  __device__ __forceinline__ static int at(int c) { return c + 8 + ((c + 8) >> 2); }
  // Horizontal window sums of the columns 4 cg - 2 .. 4 cg + 1 of a row.
  template <int N>
  __device__ __forceinline__ void sums(int row, int cg, const float* w,
                                       float (&out)[kRows][N]) const {
    // kChunk inputs are read ahead of those in use (the scheduler would read
    // all fourteen first, 56 registers).
    constexpr int kChunk = 3;
    const float4* p = &v[row][5 * cg];
    float4 next[kChunk];
#pragma unroll
    for (int q = 0; q < kChunk; ++q) next[q] = p[1 + q + ((1 + q) >> 2)];
#pragma unroll
    for (int j0 = 0; j0 < kSpan; j0 += kChunk) {
      float4 h[kChunk];
#pragma unroll
      for (int q = 0; q < kChunk; ++q) h[q] = next[q];
#pragma unroll
      for (int q = 0; q < kChunk; ++q) {
        const int j = j0 + kChunk + q;
        if (j < kSpan) next[q] = p[1 + j + ((1 + j) >> 2)];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < kChunk; ++q) {
        const int j = j0 + q;
        if (j >= kSpan) continue;
        const float in[4] = {h[q].x, h[q].y, h[q].z, h[q].w};
#pragma unroll
        for (int o = 0; o < 4; ++o) {
          if (j < o || j - o >= kTaps) continue;
#pragma unroll
          for (int m = 0; m < N; ++m)
            out[o][m] = j == o ? w[0] * in[m]
                               : fmaf(w[min(j - o, 2 * kR - j + o)], in[m], out[o][m]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
};

// Sums over the workgroup in FP64, in thread 0.
template <int N>
__device__ inline void block_sums(double (&v)[N], double (*part)[N]) {
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] += __shfl_down(v[k], off, 64);
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int k = 0; k < N; ++k) part[threadIdx.x >> 6][k] = v[k];
  __syncthreads();
  if (threadIdx.x == 0)
    for (int i = 1; i < (int)blockDim.x / 64; ++i)
#pragma unroll
      for (int k = 0; k < N; ++k) v[k] += part[i][k];
}

template <int NT>
struct StripShared {
  Exchange<NT> stat, d, der;
  double part[NT / 64][3];
};

// What a thread keeps over the steps: as the thread of column u, and as the
// row thread of four pixels from column uo on of every step's row `row`.
struct StripState {
  VerticalSums<4> stat;
  VerticalSums<3> der;
  float x[kRows], y[kRows];   // column u: the next four rows
  unsigned in, out;      // row thread: bit o for a pixel of the image, the strip
  float ss, ls;
  double ssum, l1sum, sqsum;
};

// The image rows v0 - 10 + 4 s .. of column u (0 outside the image).
__device__ __forceinline__ void load_rows(const SsimArgs& a, const float* X,
                                          const float* Y, int v0, int s, int u,
                                          StripState& st) {
  const unsigned uc = (unsigned)min(max(u, 0), a.W - 1);
  const bool col_in = u >= 0 && u < a.W;
#pragma unroll
  for (int j = 0; j < kRows; ++j) {
    const int v = v0 - 2 * kR + kRows * s + j;   // uniform
    const size_t o = (size_t)min(max(v, 0), a.H - 1) * a.W;
    const bool in = col_in && v >= 0 && v < a.H;
    const float x = (X + o)[uc], y = (Y + o)[uc];
    st.x[j] = in ? x : 0.f;
    st.y[j] = in ? y : 0.f;
  }
}

// a b + c d with both products rounded, so that identical images come to 0.
__device__ __forceinline__ float two_products(float a, float b, float c, float d) {
#pragma clang fp contract(off)
  return a * b + c * d;
}

// Step s (S: modulo 3): four image rows in, four rows of statistics (s - 3),
// of derivative sums (s - 6) and of the gradient out.  PHASE 0, steps 0-2:
// no statistics yet; 1, steps 3-5: no gradient yet; 2: all.
template <int NT, int S, int PHASE>
__device__ __forceinline__ void strip_step(const SsimArgs& a, const float* X,
                                           const float* Y, float* G, int u0,
                                           int u1, int v0, int v1, int s,
                                           float band, float scale,
                                           StripShared<NT>& sh, StripState& st) {
  const int tid = threadIdx.x;
  const int row = tid / (NT / 4), cg = tid % (NT / 4);
  const int c0 = 4 * cg - 2;            // first column of the row thread
  const int uo = u0 - 2 * kR + c0;      // its image column
  // Vertical sums of the statistics.
  {
    float v[kRows][4];
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
      v[j][0] = st.x[j];
      v[j][1] = st.y[j];
      const float e = st.x[j] - st.y[j];
      v[j][2] = e * e;
      v[j][3] = st.x[j] * st.y[j];
    }
    float check = 0.f;
#pragma unroll
    for (int j = 0; j < kRows; ++j) check += v[j][2] + v[j][3];
    load_rows(a, X, Y, v0, s + 1, u0 - 2 * kR + tid, st);
    st.stat.screen(check, v);
    if constexpr (PHASE >= 1) {
      st.stat.template finish<S>(band, v);
#pragma unroll
      for (int i = 0; i < kRows; ++i)
        sh.stat.v[i][Exchange<NT>::at(tid)] =
            make_float4(st.stat.acc[0][S][i], st.stat.acc[1][S][i],
                        st.stat.acc[2][S][i], st.stat.acc[3][S][i]);
    }
    __builtin_amdgcn_sched_barrier(0);
    st.stat.template add<S>(band, v);
  }
  if constexpr (PHASE == 0) return;
  __syncthreads();
  // Horizontal sums, SSIM and its derivatives.
  {
    float m[kRows][4];
    sh.stat.template sums<4>(row, cg, a.w, m);
    const int vs = v0 - kR + kRows * (s - 3) + row;
    const float row_scale = vs >= 0 && vs < a.H ? scale : 0.f;
    float rs = 0.f;
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      const float mx = m[o][0], my = m[o][1], mxy = mx * my;
      const float dm = mx - my, d1 = dm * dm;
      const float A1 = fmaf(2.f, mxy, kC1);
      const float A2 = fmaf(2.f, m[o][3] - mxy, kC2);
      // Bounded, so that its reciprocal is not 0 where the squares overflow.
      const float d2 = fminf(fmaf(-dm, dm, m[o][2]), kBig);
      // Reciprocals are enough here (the term is compared at 1e-5 / 1e-3).
      const float iB1 = __builtin_amdgcn_rcpf(A1 + d1);
      const float iB2 = __builtin_amdgcn_rcpf(A2 + d2);
      // q1 = A1 / B1 and q2 = A2 / B2; f1 and f2 what they lack of 1.
      const float q1 = A1 * iB1, f1 = d1 * iB1, f2 = d2 * iB2, q2 = 1.f - f2;
      rs += (st.out >> o) & 1 ? q1 * (A2 * iB2) : 0.f;
      // dS/dmu_x = 2 (q1 (dm - mx f2) / B2 + q2 (mx f1 - dm) / B1),
      // dS/dm_xx = -q1 q2 / B2, dS/dm_xy = 2 q1 / B2.
      const float q = (st.in >> o) & 1 ? row_scale : 0.f, qq = q + q;
      const float qB2 = q1 * iB2;
      float4 d;
      d.x = qq * fmaf(qB2, fmaf(-mx, f2, dm), (iB1 * q2) * fmaf(mx, f1, -dm));
      d.y = (-q * qB2) * q2;
      d.z = qq * qB2;
      d.w = 0.f;
      sh.d.v[row][Exchange<NT>::at(c0 + o)] = d;
    }
    st.ss += vs >= v0 && vs < v1 ? rs : 0.f;
  }
  __syncthreads();
  // Vertical sums of the derivatives (their step s - 3, the same modulo 3).
  {
    float v[kRows][3];
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
      const float4 d = sh.d.v[j][Exchange<NT>::at(tid)];
      v[j][0] = d.x;
      v[j][1] = d.y;
      v[j][2] = d.z;
    }
    float check = 0.f;
#pragma unroll
    for (int j = 0; j < kRows; ++j) check += (v[j][0] + v[j][1]) + v[j][2];
    st.der.screen(check, v);
    if constexpr (PHASE == 2) {
      st.der.template finish<S>(band, v);
#pragma unroll
      for (int i = 0; i < kRows; ++i)
        sh.der.v[i][Exchange<NT>::at(tid)] =
            make_float4(st.der.acc[0][S][i], st.der.acc[1][S][i],
                        st.der.acc[2][S][i], 0.f);
    }
    __builtin_amdgcn_sched_barrier(0);
    st.der.template add<S>(band, v);
  }
  if constexpr (PHASE < 2) return;
  // The gradient's four pixels of this row thread.
  const int vo = v0 + kRows * (s - kLag) + row;
  const bool any = vo < v1 && uo + 3 >= u0 && uo < u1;
  float x[4] = {0.f, 0.f, 0.f, 0.f}, y[4] = {0.f, 0.f, 0.f, 0.f};
  float g[4] = {0.f, 0.f, 0.f, 0.f};
  const size_t po = (size_t)(vo * (long long)a.W + uo);
  if (any && a.aligned) {   // all four pixels are the strip's
    const float4 fx = *(const float4*)(X + po), fy = *(const float4*)(Y + po);
    x[0] = fx.x; x[1] = fx.y; x[2] = fx.z; x[3] = fx.w;
    y[0] = fy.x; y[1] = fy.y; y[2] = fy.z; y[3] = fy.w;
    if (!a.l1) {
      const float4 fg = *(const float4*)(G + po);
      g[0] = fg.x; g[1] = fg.y; g[2] = fg.z; g[3] = fg.w;
    }
  } else if (any) {
#pragma unroll
    for (int o = 0; o < 4; ++o)
      if (uo + o >= u0 && uo + o < u1) {
        x[o] = X[po + o];
        y[o] = Y[po + o];
        if (!a.l1) g[o] = G[po + o];
      }
  }
  __syncthreads();
  float m[kRows][3];
  sh.der.template sums<3>(row, cg, a.w, m);
  if (!any) return;
#pragma unroll
  for (int o = 0; o < 4; ++o) {
    if (a.l1) {   // pixels outside the strip hold x = y: nothing to add
      const float e = x[o] - y[o];
      g[o] = e > 0.f ? a.l1_scale : (e < 0.f ? -a.l1_scale : 0.f);
      st.ls += fabsf(e);
      st.sqsum += (double)e * (double)e;
    }
    g[o] = g[o] + (m[o][0] + two_products(2.f * x[o], m[o][1], y[o], m[o][2]));
  }
  if (a.aligned) {
    *(float4*)(G + po) = make_float4(g[0], g[1], g[2], g[3]);
  } else {
#pragma unroll
    for (int o = 0; o < 4; ++o)
      if (uo + o >= u0 && uo + o < u1) G[po + o] = g[o];
  }
}

template <int NT>
__global__ __launch_bounds__(NT)
void k_ssim(SsimArgs a) {
  __shared__ StripShared<NT> sh;
  const int tid = threadIdx.x, lane = tid & 63;
  const int plane = blockIdx.z;                 // view * 3 + channel
  const size_t HW = (size_t)a.H * a.W;
  const float* X = a.x + (size_t)plane * HW;
  const float* Y = a.y + (size_t)plane * HW;
  float* G = a.dL + (size_t)plane * HW;
  const int u0 = blockIdx.x * a.strip, v0 = blockIdx.y * a.rows;
  const int u1 = min(a.W, u0 + a.strip), v1 = min(a.H, v0 + a.rows);
  float band = 0.f;
#pragma unroll
  for (int t = 0; t < kTaps; ++t)
    if ((lane >> 2) - (lane & 3) == t) band = a.w[min(t, 2 * kR - t)];
  const float n_inv = 1.f / (3.f * (float)HW);
  const float scale = -a.lam * n_inv;
  StripState st;
  st.ssum = st.l1sum = st.sqsum = 0.0;
  st.stat.bad = st.der.bad = 0u;
#pragma unroll
  for (int g = 0; g < 3; ++g) {
#pragma unroll
    for (int m = 0; m < 4; ++m) st.stat.acc[m][g] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < 3; ++m) st.der.acc[m][g] = f4v{0.f, 0.f, 0.f, 0.f};
  }
  st.in = st.out = 0u;
#pragma unroll
  for (int o = 0; o < 4; ++o) {
    const int u = u0 - 2 * kR - 2 + 4 * (tid % (NT / 4)) + o;
    st.in |= (u >= 0 && u < a.W ? 1u : 0u) << o;
    st.out |= (u >= u0 && u < u1 ? 1u : 0u) << o;
  }
  load_rows(a, X, Y, v0, 0, u0 - 2 * kR + tid, st);
  const int steps = (v1 - v0 + kRows - 1) / kRows + kLag;
  st.ss = st.ls = 0.f;
  auto step = [&](auto S, auto P, int s) {
    strip_step<NT, decltype(S)::value, decltype(P)::value>(
        a, X, Y, G, u0, u1, v0, v1, s, band, scale, sh, st);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  step(I0{}, I0{}, 0);
  step(I1{}, I0{}, 1);
  step(I2{}, I0{}, 2);
  step(I0{}, I1{}, 3);
  step(I1{}, I1{}, 4);
  step(I2{}, I1{}, 5);
  for (int s = kLag; s < steps; s += 3) {
    step(I0{}, I2{}, s);
    if (s + 1 < steps) step(I1{}, I2{}, s + 1);
    if (s + 2 < steps) step(I2{}, I2{}, s + 2);
    st.ssum += (double)st.ss;
    st.l1sum += (double)st.ls;
    st.ss = st.ls = 0.f;
  }
  double sum[3] = {st.ssum, st.l1sum, st.sqsum};
  block_sums(sum, sh.part);
  if (tid == 0) {
    const int k = plane / 3;
    atomicAdd(a.loss, -(double)a.lam * sum[0] * (double)n_inv + sum[1] * a.l1_lam_inv);
    if (a.l1 && a.sqerr) atomicAdd(&a.sqerr[k], sum[2]);
    if (a.ssim) atomicAdd(&a.ssim[k], sum[0] * (double)n_inv);
    if (plane == 0 && blockIdx.x == 0 && blockIdx.y == 0)
      atomicAdd(a.loss, (double)a.lam * a.V);
  }
}

// How the planes are split: threads of a workgroup (20 columns more than it
// writes), the rows that it writes, and about how long the pass takes.
struct Split {
  int nt, strips, rows;
  double us;
};

// The split of the least cost, in steps of a workgroup.  A workgroup takes
// five steps' time to its first output and one per four rows from there.  A
// SIMD holds two waves (registers) and a step of two takes 1.3 times as long
// as a step of one (a 680 x 1200 view by 256 threads: 252 workgroups of 52 rows
// take 49 us, 396 of 32 rows 44 us).
// Workgroups add their sums to the same addresses, 10 ns each where they end
// together (a 251 x 377 view: 567 workgroups of 64 threads with eight steps'
// time, 22.4 us; 432 with nine, 22.4 us), less where there are many.
Split split_planes(int planes, int H, int W) {
  const int groups = (H + kRows - 1) / kRows;
  Split best{};
  double least = 0.0;
  for (int nt = 64; nt <= 256; nt *= 2) {
    const int strips = (W + nt - 4 * kR - 1) / (nt - 4 * kR);
    const long long columns = (long long)strips * planes;
    const long long filled = 1024 / (nt / 64);   // workgroups: a wave per SIMD
    for (int r = 1; r <= 16; ++r) {
      const long long parts = std::max(filled * r / columns, 1LL);
      const int g = (int)((groups + parts - 1) / parts);
      const long long n = columns * ((groups + g - 1) / g);
      const long long waves = (n + filled - 1) / filled;
      const double rounds = waves / 2 * 1.3 + waves % 2;
      const double cost = rounds * (g + kLag - 1) + 0.002 * n;
      if (!best.nt || cost < least) {
        best = {nt, strips, kRows * g, 8.1 + 2.6 * rounds * (g + 1) + 0.0076 * n};
        least = cost;
      }
    }
  }
  return best;
}

}  // namespace

hipError_t launch_loss_colour(const float* rgb, const float* target, int V,
                              int H, int W, float lam_l1, float lam,
                              int fuse_l1, float* dL, double* loss,
                              double* sqerr, double* ssim, float* scratch,
                              hipStream_t st);

hipError_t launch_loss_ssim(const float* rgb, const float* target, int V,
                            int H, int W, float lam, float* dL, double* loss,
                            double* ssim, float* scratch, hipStream_t st) {
  return launch_loss_colour(rgb, target, V, H, W, 0.f, lam, 0, dL, loss,
                            nullptr, ssim, scratch, st);
}

// Whether the two kernels over 64 x 16 tiles are the faster form: few tiles,
// where the seven dependent steps of a strip, 1.6 us each, and the adds of the
// strips' sums to one address are the time; narrow images for longer, since
// each strip computes 20 columns more than it writes.  Tiles / strips us: ten
// 64 x 35 (90 tiles) 12.5 / 15.9, five 128 x 70 (150) 13.7 / 15.8, one 256 x
// 204 (156) 13.9 / 15.9, three 256 x 204 (468) 21.3 / 22.8; ten 100 x 80 (300)
// 18.1 / 20.6; one 377 x 251 (288) 21.2 / 17.0, eight 256 x 204 (1,248) 38 / 33.
// Past 600 tiles widths that fill their strips badly (45-64, 109-128 or
// 237-256 columns) are still faster in tiles; up to where depends on what the
// planes split into, so the two times are estimated (within 15 % of 350 sizes
// up to 3,000 tiles with one tile per workgroup).  Seven 256 x 140 (756 tiles)
// 26.4 / 29.7, five 237 x 189 (720) 26.2 / 29.8, 51 64 x 64 (612) 22.7 / 32.1,
// 433 64 x 16 (1,299) 37.9 / 46.4; ten 236 x 129 (1,080) 34.9 / 23.3.
static bool use_tiles(int V, int H, int W) {
  const long long plane = (long long)((W + 63) / 64) * ((H + 15) / 16);
  const long long tiles = 3 * V * plane;
  if (tiles <= 600) return tiles <= 256 || W <= 256;
  return plane <= 64 && tiles <= 3000 &&
         10.7 + 0.0208 * tiles < split_planes(3 * V, H, W).us;
}

hipError_t launch_loss_colour(const float* rgb, const float* target, int V,
                              int H, int W, float lam_l1, float lam,
                              int fuse_l1, float* dL, double* loss,
                              double* sqerr, double* ssim, float* scratch,
                              hipStream_t st) {
  if (use_tiles(V, H, W))
    return launch_ssim_tiles(rgb, target, V, H, W, lam_l1, lam, fuse_l1, dL,
                             loss, sqerr, ssim, scratch, st);
  SsimArgs a;
  {
    double g[2 * kR + 1], sum = 0.0;
    for (int i = 0; i < 2 * kR + 1; ++i) {
      const double d = i - kR;
      g[i] = exp(-d * d / (2.0 * 1.5 * 1.5));
      sum += g[i];
    }
    for (int i = 0; i <= kR; ++i) a.w[i] = (float)(g[i] / sum);
  }
  a.x = rgb; a.y = target; a.dL = dL; a.loss = loss;
  a.ssim = ssim; a.V = V; a.H = H; a.W = W; a.lam = lam;
  const size_t per = (size_t)3 * H * W;
  a.l1 = fuse_l1;
  a.l1_scale = (float)((double)lam_l1 / (double)per);
  a.l1_lam_inv = (double)lam_l1 / (double)per;
  a.sqerr = sqerr;
  // Workgroups read pixels whose gradients others write: a gradient written
  // over one of the images goes by way of the scratch.
  const size_t bytes = per * V * sizeof(float);
  auto over = [&](const float* p) {
    const uintptr_t i = (uintptr_t)p, g = (uintptr_t)dL;
    return i < g + bytes && g < i + bytes;
  };
  if (dL != scratch && (over(rgb) || over(target))) {
    if (hipError_t e = hipMemcpyAsync(scratch, dL, bytes, hipMemcpyDeviceToDevice, st)) return e;
    if (hipError_t e = launch_loss_colour(rgb, target, V, H, W, lam_l1, lam, fuse_l1,
                                          scratch, loss, sqerr, ssim, scratch, st))
      return e;
    return hipMemcpyAsync(dL, scratch, bytes, hipMemcpyDeviceToDevice, st);
  }
  a.aligned = (W & 3) == 0 &&
              (((uintptr_t)rgb | (uintptr_t)target | (uintptr_t)dL) & 15) == 0;
  const Split split = split_planes(3 * V, H, W);
  a.strip = ((W + split.strips - 1) / split.strips + 3) & ~3;
  a.rows = split.rows;
  const dim3 grid(split.strips, (H + a.rows - 1) / a.rows, V * 3);
  switch (split.nt) {
    case 64: hipLaunchKernelGGL(k_ssim<64>, grid, dim3(64), 0, st, a); break;
    case 128: hipLaunchKernelGGL(k_ssim<128>, grid, dim3(128), 0, st, a); break;
    default: hipLaunchKernelGGL(k_ssim<256>, grid, dim3(256), 0, st, a); break;
  }
  return hipGetLastError();
}

}  // namespace gs
