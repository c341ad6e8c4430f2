// Nearest existing Gaussians of insertion candidates: the nearest squared
// distance of the distance test (Eq. 7) and the 8 nearest neighbours of the
// learned initialisation's features, both exact (FP64 distances of the FP32
// means, formed in one order, ties to the lower index).
//
// Almost every mean is ruled out without its FP64 distances.  The candidates
// of a patch (3 x 3 pixels at one depth) lie within rho of the patch's
// middle, a few millimetres to centimetres, so with U an upper bound on the
// distance from the middle to its nearest (or eighth nearest) mean, a mean
// farther than U + 2 rho from the middle is nobody's neighbour.  Squared
// distances of 16 means to 16 middles are one FP32 matrix instruction,
//   |m|^2 - 2 m.x + |x|^2 = (m, |m|^2) . (-2 x, 1) + |x|^2,
// whose rounding stays below 2^-20 (|m|^2 + |x|^2); scaling both squares by
// 1 + 2^-19 or 1 - 2^-19 turns it into an upper or a lower bound.  Squares
// too large for that (or NaN) rule nothing out.
// m and x are taken from the camera's centre, so that the bounds are as tight
// far from the world's origin (their differences' rounding, 2^-24 of each,
// moves a squared distance by 2^-22 of the squares at most; 300k means 1 km
// out, all of them in reach of every patch from the origin: 249 us for the
// distance test and 6.1 ms for the neighbours' pass, now 28 and 51).
//
// Every pair in FP64 on the vector units took 113 us (distance test) and 320
// us (neighbours) for 96 patches against 300k means; now 16 us, and 35 us in
// three launches.  The matrix instructions of both passes take about 3 us of
// it; what bounds the kernels is the latency of one slice: load, bound,
// barrier, bound, a few exact distances.

#include <math.h>

#include "gs_internal.h"

namespace gs {
namespace {

typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int kWaves = 16, kThreads = 64 * kWaves;
constexpr int kPatches = 16;   // patches per workgroup (matrix columns)
// Groups of 64 means in flight per wave: 5 take a slice of 300k means in one
// go; with 3, 4, 6 or 8 the searches of 50k to 1M means are within 3 % (20,
// at 70 registers more, leaves half the waves: 37 us against 16).
constexpr int kAhead = 5;
constexpr float kUp = 1.f + 0x1p-19f, kDown = 1.f - 0x1p-19f;
constexpr float kTiny = 1e-30f;   // covers squares that underflow
constexpr float kHuge = 1e37f;    // squares below it cannot overflow the sum

struct NearArgs {
  const float* mean;   // [3][cap]
  const float* rgb;    // [3][cap]
  const int32_t* n_dev;
  int cap;
  const gs_camera* cam;
  int W, H;
  const float* kf_rgb;
  const float* pts;
  int n_pts, per;                // per: candidates per patch, 1 or 9
  unsigned long long* d2bits;    // distance test
  float* feats;                  // neighbours: [C][32], scratch before
  int32_t* knn_idx;              // [C][8] or null
  float* knn_dist;               // [C][8] or null
};

// Candidate pix of a patch: pixel (u, v), inverse depth d.
struct Candidate {
  int u, v;
  float d;
};
__device__ inline Candidate candidate(const NearArgs& a, int patch, int i) {
  const int pix = a.per == 1 ? 4 : i;
  return Candidate{(int)a.pts[3 * patch] + pix % 3 - 1,
                   (int)a.pts[3 * patch + 1] + pix / 3 - 1,
                   a.pts[3 * patch + 2]};
}

// Back-projection (Eq. 6), FP64; z = 0 for an inverse depth that is not
// positive.
__device__ inline void back_project(const gs_camera& cam, const Candidate& c,
                                    double* X) {
  const double z = c.d > 0.f ? 1.0 / (double)c.d : 0.0;
  const double xc[3] = {((double)c.u - (double)cam.cx) / (double)cam.fx * z,
                        ((double)c.v - (double)cam.cy) / (double)cam.fy * z,
                        z};
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < 3; ++j)
      s += (double)cam.R[3 * j + i] * (xc[j] - (double)cam.t[j]);
    X[i] = s;
  }
}

__device__ inline double dist2(const double* X, float mx, float my, float mz) {
  const double e0 = X[0] - (double)mx;
  const double e1 = X[1] - (double)my;
  const double e2 = X[2] - (double)mz;
  return (e0 * e0 + e1 * e1) + e2 * e2;
}

// The means [begin, end) of one of the launch's slices of the live map.
__device__ inline void slice_of(int n, int slices, int s, int& begin, int& end) {
  const int len = ((n + slices - 1) / slices + 15) & ~15;
  begin = (int)min((long long)n, (long long)s * len);
  end = min(n, begin + len);
}

// Where coordinates are taken from: the camera's centre -R^T t (any point
// near it would do).
struct Origin {
  float x, y, z;
};
__device__ inline Origin origin(const gs_camera& cam) {
  float o[3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
    o[i] = fmaf(-cam.R[i], cam.t[0], fmaf(-cam.R[3 + i], cam.t[1], -cam.R[6 + i] * cam.t[2]));
  return Origin{o[0], o[1], o[2]};
}

// Matrix operands of one lane: row (mean) and column (patch) l % 16,
// component l / 16.
struct Middle {
  float b;   // -2 x of the lane's component, 1 for the fourth
  f4v c;     // |x|^2 of the lane's column, scaled
};
__device__ inline Middle middle(const float (*mid)[3], const Origin& o,
                                float scale, float eps) {
  const int lane = threadIdx.x & 63, p = lane & 15, k = lane >> 4;
  const float x = mid[p][0] - o.x, y = mid[p][1] - o.y, z = mid[p][2] - o.z;
  Middle m;
  m.b = k == 0 ? -2.f * x : k == 1 ? -2.f * y : k == 2 ? -2.f * z : 1.f;
  const float x2 = ((x * x + y * y) + z * z) * scale + eps;
  m.c = f4v{x2, x2, x2, x2};
  return m;
}

// One mean per lane of each of the wave's groups of 64, kAhead groups from
// g0 on.
struct Batch {
  float x[kAhead], y[kAhead], z[kAhead];
};
__device__ __forceinline__ void load_batch(const NearArgs& a, int begin,
                                           int end, int g0, Batch& b) {
#pragma unroll
  for (int u = 0; u < kAhead; ++u) {
    const int g = min(begin + 64 * (g0 + u * kWaves) + ((int)threadIdx.x & 63), end - 1);
    b.x[u] = a.mean[g];
    b.y[u] = a.mean[(size_t)a.cap + g];
    b.z[u] = a.mean[2 * (size_t)a.cap + g];
  }
}

// Lanes 16 r + i of register q to lanes 16 q + i of register r: four swaps of
// register halves and rows.
__device__ __forceinline__ void transpose_rows(float (&v)[4]) {
  auto swap32 = [](float& p, float& q) {
    const auto t = __builtin_amdgcn_permlane32_swap(
        __float_as_uint(p), __float_as_uint(q), false, false);
    p = __uint_as_float(t[0]);
    q = __uint_as_float(t[1]);
  };
  auto swap16 = [](float& p, float& q) {
    const auto t = __builtin_amdgcn_permlane16_swap(
        __float_as_uint(p), __float_as_uint(q), false, false);
    p = __uint_as_float(t[0]);
    q = __uint_as_float(t[1]);
  };
  swap32(v[0], v[2]);
  swap32(v[1], v[3]);
  swap16(v[0], v[1]);
  swap16(v[2], v[3]);
}

// f(first mean, bounds) for the wave's means of [begin, end), 16 at a time:
// lane l gets the bounds of means first + 4 (l / 16) + r, r = 0..3, to middle
// l % 16 (+inf past the end; wild where a square of the 64 is not below
// kHuge).  first: the wave's first batch, loaded by the
// caller as early as it can (a slice of up to 5,120 means needs no other).
template <typename F>
__device__ __forceinline__ void each_bound(const NearArgs& a, int begin,
                                           int end, const Middle& m,
                                           const Origin& o, float scale,
                                           float wild,
                                           const Batch& first, F&& f) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int groups = (end - begin + 63) >> 6;
  Batch b = first;
  for (int g0 = wave; g0 < groups; g0 += kWaves * kAhead) {
    if (g0 != wave) load_batch(a, begin, end, g0, b);
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int at = begin + 64 * (g0 + u * kWaves);
      if (at >= end) break;   // uniform over the wave
      const bool in = at + lane < end;
      const float x = b.x[u] - o.x, y = b.y[u] - o.y, z = b.z[u] - o.z;
      const float m2 = (x * x + y * y) + z * z;
      const bool any_wild = __builtin_amdgcn_ballot_w64(in && !(m2 < kHuge)) != 0;
      float v[4] = {in ? x : 0.f, in ? y : 0.f, in ? z : 0.f,
                    in ? m2 * scale : INFINITY};
      transpose_rows(v);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        f4v d = __builtin_amdgcn_mfma_f32_16x16x4f32(v[q], m.b, m.c, 0, 0, 0);
        if (any_wild) d = f4v{wild, wild, wild, wild};
        f(at + 16 * q, d);
      }
    }
  }
}

__device__ inline float min4(f4v v) {
  return fminf(fminf(v[0], v[1]), fminf(v[2], v[3]));
}

// Smallest upper bound over the slice for each of the workgroup's 16
// middles, in every thread that passes tid < 16 (column tid).
__device__ inline float slice_min(const NearArgs& a, int begin, int end,
                                  const float (*mid)[3], const Origin& o,
                                  const Batch& first, float (*part)[kPatches]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const Middle m = middle(mid, o, kUp, kTiny);
  float best = INFINITY;
  each_bound(a, begin, end, m, o, kUp, INFINITY, first,
             [&](int, f4v d) { best = fminf(best, min4(d)); });
  best = fminf(best, __shfl_xor(best, 16, 64));
  best = fminf(best, __shfl_xor(best, 32, 64));
  if (lane < 16) part[wave][lane] = best;
  __syncthreads();
  float r = INFINITY;
  if (threadIdx.x < 16)
    for (int w = 0; w < kWaves; ++w) r = fminf(r, part[w][threadIdx.x]);
  return fmaxf(r, 0.f);
}

// (sqrt(u2) + 2 rho)^2, rounded up; everything for a middle whose own square
// is not below kHuge.
__device__ inline float reach2(float u2, double rho, const float* mid,
                               const Origin& o) {
  const float x = mid[0] - o.x, y = mid[1] - o.y, z = mid[2] - o.z;
  if (!((x * x + y * y) + z * z < kHuge)) return INFINITY;
  const double r = sqrt((double)u2) + 2.0 * rho;
  return (float)(r * r * (1.0 + 1e-6)) * (1.f + 0x1p-22f) + kTiny;
}

// ---- The distance test ------------------------------------------------------

// One slice of the map against 16 patches: the slice's own nearest bound sets
// the reach, so every workgroup finds its slice's exact minima, which meet in
// d2bits (FP64 bits order like the values).  The means within reach are
// listed first and then measured by all threads, one (mean, candidate) each;
// lanes that measured what they found, one after another, took 8 to 19 us
// of a workgroup's time.
constexpr int kWithin = 1024;

__global__ __launch_bounds__(kThreads) void k_nearest(NearArgs a) {
  __shared__ double X[kPatches][9][3];
  __shared__ unsigned long long best[kPatches][9], rho2[kPatches];
  __shared__ int tested[kPatches];
  __shared__ float mid[kPatches][3];
  __shared__ float part[kWaves][kPatches];
  __shared__ float reach[kPatches];
  __shared__ uint32_t within[kWithin];   // patch << 28 | mean - begin (2^28: eight slices)
  __shared__ int n_within;
  const int tid = threadIdx.x, lane = tid & 63;
  const int p0 = blockIdx.y * kPatches;
  int begin, end;
  slice_of(min(*a.n_dev, a.cap), gridDim.x, blockIdx.x, begin, end);
  if (begin >= end) return;   // uniform over the workgroup
  if (tid == 0) n_within = 0;
  Batch first;
  load_batch(a, begin, end, tid >> 6, first);
  const Origin o = origin(*a.cam);
  const int cp = tid / a.per, ci = tid - cp * a.per;
  bool live = false;
  if (cp < kPatches) {
    best[cp][ci] = ~0ull;
    if (p0 + cp < a.n_pts) {
      const Candidate c = candidate(a, p0 + cp, ci);
      back_project(*a.cam, c, X[cp][ci]);
      live = c.u >= 0 && c.u < a.W && c.v >= 0 && c.v < a.H && c.d > 0.f;
      if (live) best[cp][ci] = (unsigned long long)__double_as_longlong(INFINITY);
    } else {
      X[cp][ci][0] = X[cp][ci][1] = X[cp][ci][2] = 0.0;
    }
  }
  __syncthreads();
  const int mi = a.per == 1 ? 0 : 4;
  if (tid < kPatches) {
    for (int i = 0; i < 3; ++i) mid[tid][i] = (float)X[tid][mi][i];
    rho2[tid] = 0ull;
    tested[tid] = 0;
  }
  __syncthreads();
  if (live) {
    atomicMax(&rho2[cp], (unsigned long long)__double_as_longlong(
                             dist2(X[cp][ci], mid[cp][0], mid[cp][1], mid[cp][2])));
    tested[cp] = 1;
  }
  // A quarter of the slice bounds its nearest mean well enough: the means
  // within reach are few either way.
  const float u2 = slice_min(a, begin, begin + (end - begin + 3) / 4, mid, o,
                             first, part);
  if (tid < kPatches)
    reach[tid] = tested[tid]
                     ? reach2(u2, sqrt(__longlong_as_double((long long)rho2[tid])),
                              mid[tid], o)
                     : -INFINITY;
  __syncthreads();
  const int p = lane & 15;
  const float r = reach[p];
  auto exact = [&](int pp, int i, int g) {
    if (best[pp][i] == ~0ull) return;   // not tested
    const double d2 = dist2(X[pp][i], a.mean[g], a.mean[(size_t)a.cap + g],
                            a.mean[2 * (size_t)a.cap + g]);
    if (d2 == d2)
      atomicMin(&best[pp][i], (unsigned long long)__double_as_longlong(d2));
  };
  each_bound(a, begin, end, middle(mid, o, kDown, -kTiny), o, kDown, -INFINITY,
             first,
             [&](int first_mean, f4v d) {
    if (__builtin_amdgcn_ballot_w64(!(min4(d) > r)) == 0) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int g = first_mean + 4 * (lane >> 4) + q;
      if (d[q] > r || g >= end) continue;
      const int at = atomicAdd(&n_within, 1);
      if (at < kWithin) {
        within[at] = ((uint32_t)p << 28) | (uint32_t)(g - begin);
      } else {
        for (int i = 0; i < a.per; ++i) exact(p, i, g);
      }
    }
  });
  __syncthreads();
  const int jobs = min(n_within, kWithin) * a.per;
  for (int j = tid; j < jobs; j += kThreads) {
    const int e = j / a.per;
    const uint32_t w = within[e];
    exact((int)(w >> 28), j - e * a.per, begin + (int)(w & 0xfffffffu));
  }
  __syncthreads();
  if (live) atomicMin(&a.d2bits[(p0 + cp) * a.per + ci], best[cp][ci]);
}

// ---- The 8 nearest ----------------------------------------------------------
//
// Three launches over the feature rows as scratch (32 words per candidate,
// written last): k_knn_bound leaves each slice's smallest upper bound per
// patch; the eighth smallest of them bounds the eighth nearest mean (the
// slices are disjoint); k_knn_list appends the means within reach to the
// patch's list; k_knn_select takes the 8 nearest of the list per candidate
// and writes the features.  Where a list runs over (reach holds more means
// than the rows have words: patches far away in small images), the patch's
// workgroup gathers the means within reach again into a larger list in LDS,
// and beyond that each candidate walks the map.

__host__ __device__ inline int knn_slices(int per) { return per == 1 ? 16 : 64; }
__host__ __device__ inline int knn_words(int per) { return 32 * per; }
__host__ __device__ inline int knn_list(int per) {
  return knn_words(per) - knn_slices(per) - 1;   // behind the count
}

// The middle of a patch and its rho (both in every lane), by one wave.
__device__ inline double patch_middle(const NearArgs& a, int patch,
                                      float* mid) {
  const int lane = threadIdx.x & 63, mi = a.per == 1 ? 0 : 4;
  double X[3];
  back_project(*a.cam, candidate(a, patch, min(lane, a.per - 1)), X);
#pragma unroll
  for (int i = 0; i < 3; ++i)
    mid[i] = __uint_as_float(
        __builtin_amdgcn_readlane(__float_as_uint((float)X[i]), mi));
  double rho = dist2(X, mid[0], mid[1], mid[2]);
  // Lanes past the candidates repeat the last one, so the maximum is taken
  // over the whole wave.
  for (int off = 32; off > 0; off >>= 1) rho = fmax(rho, __shfl_xor(rho, off, 64));
  return sqrt(rho);
}

// The eighth smallest of the lanes' values >= 0 (as bit patterns), +inf when
// there are not eight: the largest t with fewer than eight lanes below it.
__device__ inline float wave_eighth(float x) {
  const uint32_t v = __float_as_uint(x);
  uint32_t t = 0;
  for (int bit = 30; bit >= 0; --bit) {
    const uint32_t c = t | (1u << bit);
    if (__popcll(__builtin_amdgcn_ballot_w64(v < c)) < 8) t = c;
  }
  return t >= 0x7f800000u ? INFINITY : __uint_as_float(t);
}

// The reach of one patch from its slices' bounds, by one wave (every lane).
__device__ inline float knn_reach(const NearArgs& a, int patch, double rho,
                                  const float* mid, const Origin& o) {
  const int lane = threadIdx.x & 63;
  const float* w = a.feats + (size_t)patch * knn_words(a.per);
  return reach2(wave_eighth(lane < knn_slices(a.per) ? w[lane] : INFINITY), rho,
                mid, o);
}

__global__ __launch_bounds__(kThreads) void k_knn_bound(NearArgs a) {
  __shared__ float mid[kPatches][3];
  __shared__ float part[kWaves][kPatches];
  const int tid = threadIdx.x, p0 = blockIdx.y * kPatches;
  int begin, end;
  slice_of(min(*a.n_dev, a.cap), gridDim.x, blockIdx.x, begin, end);
  Batch first{};
  if (begin < end) load_batch(a, begin, end, tid >> 6, first);
  const Origin o = origin(*a.cam);
  if (tid < kPatches) {
    double X[3] = {0.0, 0.0, 0.0};
    if (p0 + tid < a.n_pts)
      back_project(*a.cam, candidate(a, p0 + tid, a.per == 1 ? 0 : 4), X);
    for (int i = 0; i < 3; ++i) mid[tid][i] = (float)X[i];
  }
  __syncthreads();
  const float u2 =
      begin < end ? slice_min(a, begin, end, mid, o, first, part) : INFINITY;
  if (tid < kPatches && p0 + tid < a.n_pts) {
    uint32_t* w = (uint32_t*)a.feats + (size_t)(p0 + tid) * knn_words(a.per);
    w[blockIdx.x] = __float_as_uint(u2);
    if (blockIdx.x == 0) w[knn_slices(a.per)] = 0u;
  }
}

__global__ __launch_bounds__(kThreads) void k_knn_list(NearArgs a) {
  __shared__ float mid[kPatches][3];
  __shared__ float reach[kPatches];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int p0 = blockIdx.y * kPatches;
  int begin, end;
  slice_of(min(*a.n_dev, a.cap), gridDim.x, blockIdx.x, begin, end);
  if (begin >= end) return;   // uniform over the workgroup
  static_assert(kWaves == kPatches, "one wave per patch");
  Batch first;
  load_batch(a, begin, end, wave, first);
  const Origin o = origin(*a.cam);
  {
    float x[3] = {0.f, 0.f, 0.f}, r = -INFINITY;
    if (p0 + wave < a.n_pts) {
      const double rho = patch_middle(a, p0 + wave, x);
      r = knn_reach(a, p0 + wave, rho, x, o);
    }
    if (lane == 0) {
      for (int i = 0; i < 3; ++i) mid[wave][i] = x[i];
      reach[wave] = r;
    }
  }
  __syncthreads();
  const int p = lane & 15;
  const float r = reach[p];
  uint32_t* w = (uint32_t*)a.feats +
                (size_t)min(p0 + p, a.n_pts - 1) * knn_words(a.per) + knn_slices(a.per);
  const int room = knn_list(a.per);
  each_bound(a, begin, end, middle(mid, o, kDown, -kTiny), o, kDown, -INFINITY,
             first,
             [&](int first_mean, f4v d) {
    if (__builtin_amdgcn_ballot_w64(!(min4(d) > r)) == 0) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int g = first_mean + 4 * (lane >> 4) + q;
      if (d[q] > r || g >= end || p0 + p >= a.n_pts) continue;
      const uint32_t at = atomicAdd(w, 1u);
      if (at < (uint32_t)room) w[1 + at] = (uint32_t)g;
    }
  });
}

struct Nb {
  double d2;
  int idx;
};

__device__ __forceinline__ bool nb_less(const Nb& a, const Nb& b) {
  return a.d2 < b.d2 || (a.d2 == b.d2 && (unsigned)a.idx < (unsigned)b.idx);
}

// Sorted insertion as a chain of compare-swaps (no dynamic index, so the
// list stays in registers).
__device__ __forceinline__ void nb_insert(Nb (&best)[8], Nb x) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const bool lt = nb_less(x, best[j]);
    const double td = best[j].d2;
    const int ti = best[j].idx;
    best[j].d2 = lt ? x.d2 : td;
    best[j].idx = lt ? x.idx : ti;
    x.d2 = lt ? td : x.d2;
    x.idx = lt ? ti : x.idx;
  }
}

__device__ __forceinline__ void nb_cswap(Nb& lo, Nb& hi) {
  const bool sw = nb_less(hi, lo);
  const double d = lo.d2;
  const int i = lo.idx;
  lo.d2 = sw ? hi.d2 : d;
  lo.idx = sw ? hi.idx : i;
  hi.d2 = sw ? d : hi.d2;
  hi.idx = sw ? i : hi.idx;
}

// 64-bit value of lane (lane ^ m).
__device__ __forceinline__ unsigned long long xor_lane64(unsigned long long v, int m) {
  const int src = ((int)__lane_id() ^ m) << 2;
  const unsigned lo = __builtin_amdgcn_ds_bpermute(src, (int)v);
  const unsigned hi = __builtin_amdgcn_ds_bpermute(src, (int)(v >> 32));
  return ((unsigned long long)hi << 32) | lo;
}

// The 8 smallest over the wave of the lanes' sorted lists, in every lane.
// (Elementwise minima of one ascending and one descending list are the lower
// half of their union and form a bitonic sequence; three half-cleaner
// stages sort it.)
__device__ __forceinline__ void nb_wave_merge(Nb (&best)[8]) {
  for (int m = 1; m < 64; m <<= 1) {
    Nb o[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      o[j].d2 = __longlong_as_double(
          (long long)xor_lane64((unsigned long long)__double_as_longlong(best[j].d2), m));
      o[j].idx = __builtin_amdgcn_ds_bpermute(((int)__lane_id() ^ m) << 2, best[j].idx);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const bool tb = nb_less(o[7 - j], best[j]);
      best[j].d2 = tb ? o[7 - j].d2 : best[j].d2;
      best[j].idx = tb ? o[7 - j].idx : best[j].idx;
    }
#pragma unroll
    for (int s = 4; s >= 1; s >>= 1)
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if ((j & s) == 0) nb_cswap(best[j], best[j + s]);
  }
}

constexpr int kMaxList = 4096;

// One workgroup per patch, one wave per candidate (with one candidate, the
// other waves only help to gather).  Up to 64 means (the usual case, or what
// a longer list is cut to): lane l holds mean l, and its place is the number
// of smaller ones.  Else (many equal distances, or the whole map) every lane
// keeps the 8 nearest of its share and the lists are merged across the wave.
__global__ __launch_bounds__(576) void k_knn_select(NearArgs a) {
  __shared__ uint32_t list[kMaxList];
  __shared__ uint32_t gathered;
  // Per candidate and neighbour: log-distance, weight, weighted colour.
  __shared__ double term[9][5][8];
  __shared__ uint32_t cutlist[9][64];
  const int tid = threadIdx.x, lane = tid & 63, ci = tid >> 6;
  const int patch = blockIdx.x;
  const uint32_t* w = (const uint32_t*)a.feats + (size_t)patch * knn_words(a.per);
  // The list's words are loaded with the count, whatever it says.
  const int room = knn_list(a.per);
  const uint32_t word = tid < room ? w[knn_slices(a.per) + 1 + tid] : 0u;
  uint32_t cnt = w[knn_slices(a.per)];
  if (cnt <= (uint32_t)room) {   // uniform over the workgroup
    if (tid < (int)cnt) list[tid] = word;
  } else {
    float mid[3];
    const double rho = patch_middle(a, patch, mid);
    const float r = knn_reach(a, patch, rho, mid, origin(*a.cam));
    if (tid == 0) gathered = 0u;
    __syncthreads();
    const int n = min(*a.n_dev, a.cap);
    for (int g0 = tid; g0 < n; g0 += 8 * blockDim.x) {
      float e[8][3];
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int i = 0; i < 3; ++i)
          e[u][i] = a.mean[(size_t)i * a.cap + min(g0 + u * (int)blockDim.x, n - 1)] - mid[i];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int g = g0 + u * (int)blockDim.x;
        const float d2 = (e[u][0] * e[u][0] + e[u][1] * e[u][1]) + e[u][2] * e[u][2];
        if (g >= n || d2 * kDown - kTiny > r) continue;
        const uint32_t at = atomicAdd(&gathered, 1u);
        if (at < kMaxList) list[at] = (uint32_t)g;
      }
    }
    __syncthreads();
    cnt = gathered;
  }
  __syncthreads();   // the scratch is read, the list complete
  if (ci >= a.per) return;   // no barrier below
  const Candidate c = candidate(a, patch, ci);
  double X[3];
  back_project(*a.cam, c, X);
  auto exact = [&](int g) {
    return dist2(X, a.mean[g], a.mean[(size_t)a.cap + g], a.mean[2 * (size_t)a.cap + g]);
  };
  // Neighbour j of the candidate, found by some lane: its terms of the
  // features go to slot j.
  auto neighbour = [&](int j, double d2, int g, const float* rgb) {
    const double dist = fmax(sqrt(d2), 1e-6);
    const double wgt = 1.0 / dist;
    term[ci][0][j] = log(dist);
    term[ci][1][j] = wgt;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) term[ci][2 + ch][j] = wgt * (double)rgb[ch];
    if (a.knn_idx) a.knn_idx[((size_t)patch * a.per + ci) * 8 + j] = g;
    if (a.knn_dist)
      a.knn_dist[((size_t)patch * a.per + ci) * 8 + j] = (float)sqrt(d2);
  };
  auto colour = [&](int g, float* rgb) {
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) rgb[ch] = a.rgb[(size_t)ch * a.cap + g];
  };
  // More than 64: those beyond the eighth smallest of the lanes' nearest are
  // nobody's, the others take the list's place (per wave).
  int m = (int)cnt;
  const uint32_t* from = list;
  if (cnt > 64 && cnt <= kMaxList) {
    double near = INFINITY;
    for (int i = lane; i < (int)cnt; i += 64) near = fmin(near, exact((int)list[i]));
    const double cut = (double)wave_eighth(__double2float_ru(near));
    m = 0;
    for (int i0 = 0; i0 < (int)cnt; i0 += 64) {
      const int i = i0 + lane;
      const bool in = i < (int)cnt && exact((int)list[min(i, (int)cnt - 1)]) <= cut;
      const uint64_t who = __builtin_amdgcn_ballot_w64(in);
      const int at = m + (int)__builtin_amdgcn_mbcnt_hi(
                             (uint32_t)(who >> 32),
                             __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0));
      if (in && at < 64) cutlist[ci][at] = list[i];
      m += __popcll(who);
    }
    from = cutlist[ci];
    wave_sync();
  }
  int found;
  if (m <= 64) {
    Nb b{INFINITY, -1};
    float rgb[3] = {0.f, 0.f, 0.f};
    if (lane < m) {
      b.idx = (int)from[lane];
      colour(b.idx, rgb);
      b.d2 = exact(b.idx);
      if (!(b.d2 == b.d2)) b = Nb{INFINITY, -1};   // NaN: nobody's neighbour
    }
    int rank = 0;
    for (int j = 0; j < m; ++j) {
      const unsigned long long k = (unsigned long long)__double_as_longlong(b.d2);
      Nb o;
      o.d2 = __longlong_as_double((long long)(
          ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(k >> 32), j) << 32) |
          (uint32_t)__builtin_amdgcn_readlane((int)k, j)));
      o.idx = __builtin_amdgcn_readlane(b.idx, j);
      rank += nb_less(o, b);
    }
    const bool mine = b.idx >= 0 && rank < 8;
    if (mine) neighbour(rank, b.d2, b.idx, rgb);
    found = __popcll(__builtin_amdgcn_ballot_w64(mine));
  } else {
    Nb best[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) best[j] = Nb{INFINITY, -1};
    const bool walk = cnt > kMaxList;
    const int n = walk ? min(*a.n_dev, a.cap) : (int)cnt;
    for (int i = lane; i < n; i += 64) {
      const int g = walk ? i : (int)list[i];
      const double d2 = exact(g);
      if (d2 <= best[7].d2) nb_insert(best, Nb{d2, g});
    }
    nb_wave_merge(best);
    Nb b = best[0];   // lane j takes neighbour j
#pragma unroll
    for (int j = 1; j < 8; ++j)
      if (lane == j) b = best[j];
    const bool mine = lane < 8 && b.idx >= 0;
    if (mine) {
      float rgb[3];
      colour(b.idx, rgb);
      neighbour(lane, b.d2, b.idx, rgb);
    }
    found = __popcll(__builtin_amdgcn_ballot_w64(mine));
  }
  wave_sync();   // the wave's terms are in LDS
  const int cc = patch * a.per + ci;
  float* f = a.feats + (size_t)cc * 32;
  if (lane < 27) {
    const int q = lane / 3, ch = lane % 3;
    const int uu = c.u + q % 3 - 1, vv = c.v + q / 3 - 1;
    f[lane] = (uu >= 0 && uu < a.W && vv >= 0 && vv < a.H)
                  ? a.kf_rgb[((size_t)ch * a.H + vv) * a.W + uu] : 0.f;
  } else if (lane == 27) {
    f[27] = c.d;
  } else if (lane < 32) {
    // Mean log-distance, weighted mean colour: sums in neighbour order.
    const int q = lane == 28 ? 0 : lane - 27;   // 28: log, 29..31: colour
    double s = 0.0, sw = 0.0;
    for (int j = 0; j < found; ++j) {
      s += term[ci][q][j];
      sw += term[ci][1][j];
    }
    f[lane] = !found ? 0.f : (float)(lane == 28 ? s / found : s / sw);
  } else if (lane < 40 && lane - 32 >= found) {   // neighbours past the live count
    if (a.knn_idx) a.knn_idx[(size_t)cc * 8 + lane - 32] = -1;
    if (a.knn_dist) a.knn_dist[(size_t)cc * 8 + lane - 32] = 0.f;
  }
}

// Slices x groups of 16 patches: one workgroup per CU (their registers allow
// no second), so that no second round of workgroups follows the first; at
// least eight slices.
dim3 one_round(int n_pts) {
  const int groups = (n_pts + kPatches - 1) / kPatches;
  return dim3(max(8, min(64, 256 / groups)), groups);
}

}  // namespace

hipError_t launch_nearest(const gs_params* p, const gs_camera* cam, int W,
                          int H, const float* pts, int n_pts, int centre_only,
                          unsigned long long* d2bits, hipStream_t st) {
  NearArgs a{};
  a.mean = p->mean; a.n_dev = p->n_dev; a.cap = p->capacity; a.cam = cam;
  a.W = W; a.H = H; a.pts = pts; a.n_pts = n_pts;
  a.per = centre_only ? 1 : 9; a.d2bits = d2bits;
  if (n_pts > 0 && a.cap > 0)
    hipLaunchKernelGGL(k_nearest, one_round(n_pts), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_knn_features(const gs_params* p, const gs_camera* cam, int W,
                               int H, const float* kf_rgb, const float* pts,
                               int n_pts, int centre_only, float* feats,
                               int32_t* knn_idx, float* knn_dist,
                               hipStream_t st) {
  NearArgs a{};
  a.mean = p->mean; a.rgb = p->rgb; a.n_dev = p->n_dev; a.cap = p->capacity;
  a.cam = cam; a.W = W; a.H = H; a.kf_rgb = kf_rgb; a.pts = pts;
  a.n_pts = n_pts; a.per = centre_only ? 1 : 9; a.feats = feats;
  a.knn_idx = knn_idx; a.knn_dist = knn_dist;
  if (n_pts <= 0) return hipGetLastError();
  hipLaunchKernelGGL(k_knn_bound,
                     dim3(knn_slices(a.per), (n_pts + kPatches - 1) / kPatches),
                     dim3(kThreads), 0, st, a);
  hipLaunchKernelGGL(k_knn_list, one_round(n_pts), dim3(kThreads), 0, st, a);
  hipLaunchKernelGGL(k_knn_select, dim3(n_pts), dim3(a.per == 1 ? 512 : 576), 0, st, a);
  return hipGetLastError();
}

}  // namespace gs
