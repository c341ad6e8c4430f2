// Backward of the compositing (exact derivative of Eq. 3 with the forward's
// decisions), per screen tile.
//
// One workgroup per (view, tile), the same pixel ownership as the forward.
// Only per-pixel state is kept from the forward (T_final and n_last); the
// list is walked back to front from the tile's largest n_last, and each
// admitted entry's transmittance is recovered as T_i = T_{i+1} / (1 - a_i).
// The colour accumulated behind entry i, dotted with g = dL/dC, follows
// S_{i-1} = a_i (c_i . g) + (1 - a_i) S_i, so
//   dL/dc_i     = a_i T_i g
//   dL/da_i     = T_i (c_i . g - S_i) - T_final (bg . g) / (1 - a_i)
//   dL/dpi_i    = a_i dL/da_i                 (a = o exp(pi), unclamped)
//   dL/do_i     = G_i dL/da_i = (dL/dpi_i) / o   (summed per entry, then / o)
// with pi = -(A dx^2 + C dy^2) / 2 - B dx dy.  A thread's pixels share dx,
// so per entry it needs only the moments sum(dL/dpi), sum(dL/dpi dy) and
// sum(dL/dpi dy^2) over its strip; the rows of a strip are consecutive
// (dy_p = dy_0 - p), so these follow from sums weighted by the constants p
// and p^2.  Nine per-lane sums per entry (the three moments, the first one
// times dx and dx^2, the second times dx, and the colour gradient) are
// reduced over each 16-lane row with DPP (a transposed reduction that packs
// four quantities into one register), merged across rows and waves by LDS
// adds, and turned into the mean, conic and opacity gradients once per
// entry and workgroup, which adds them to global memory (kSpreadBlocks says
// where).

#include "raster_common.h"
#include "tails.h"

namespace gs {
namespace {

struct BwdArgs {
  RasterArgs r;
  const float* dL;
  const float* Tfin;
  const int32_t* nlast;
  float* grad2d;   // [V][5][cap]
  float* gop;      // [cap]
  float* grgb;     // [3][cap] (caller's gradient rows, accumulated), or
                   // [V][3][cap] per view (view-dependent colour)
  size_t grgb_vstride;   // 0, or 3 cap for per-view colour gradients
  // Per-Gaussian accumulators (not null: used in place of the above):
  // gview [V][cap][8], gsum [cap][4]; view-dependent colour goes to gview.
  double* gview;
  double* gsum;
  int view_colour;
  // L1 photometric term fused in (target not null): dL/dC is formed per
  // pixel from the forward's image instead of read from dL.
  const float* rgb;
  const float* target;
  float l1_scale;        // lambda / (3HW), the gradient's magnitude
  double l1_lam_inv;     // lambda / (3HW) in FP64, for the loss
  double* tile_loss;     // [tiles][2]: this tile's loss and squared error
  // Workgroups past the tiles' (tile_blocks) run the planar regulariser.
  int tile_blocks;
  PlanarJob planar;
  // Workgroups of k_spread's row past spread_blocks sum the fused L1 losses.
  int spread_blocks;
  L1ReduceJob l1;
};

// Sign of r times scale (sign(0) = 0): the L1 term's gradient.
__device__ __forceinline__ float l1_grad(float r, float scale) {
  return r > 0.f ? scale : (r < 0.f ? -scale : 0.f);
}

// x plus the DPP-permuted y.  Lanes whose source lies outside their row read
// 0; the reductions below only keep lanes whose source is inside the row.
template <int CTRL>
__device__ __forceinline__ float add_dpp(float x, float y) {
  const int t = __builtin_amdgcn_update_dpp(0, __float_as_int(y), CTRL, 0xf,
                                            0xf, true);
  return x + __int_as_float(t);
}

// a + b over the two halves of the wave: returns, in lanes 0-31, a's lanes
// l + (l + 32) and, in lanes 32-63, b's (v_permlane32_swap exchanges the
// upper half of its first operand with the lower half of its second).
__device__ __forceinline__ float fold32(float a, float b) {
  const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(a),
                                                  __float_as_uint(b), false,
                                                  false);
  return __uint_as_float(t[0]) + __uint_as_float(t[1]);
}

// The same over adjacent rows: rows 0 and 2 receive a's rows r + (r + 1)
// and rows 1 and 3 b's (v_permlane16_swap exchanges the odd rows of its
// first operand with the even rows of its second).
__device__ __forceinline__ float fold16(float a, float b) {
  const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(a),
                                                  __float_as_uint(b), false,
                                                  false);
  return __uint_as_float(t[0]) + __uint_as_float(t[1]);
}

// Sums over the wave of the nine values S0, dx S0, dx^2 S0, S1, dx S1, S2, r,
// g and b.  A transposed reduction: lanes 16 apart share their image column
// and so dx, hence the six values are folded over the four rows of lanes
// first, two or four to a register, and only their column sums are multiplied
// by dx.  That leaves four registers, A with S0, S2, S1, r in the rows 0-3, dx
// A, dx^2 A and B with g in the rows 0 and 1 and b in 2 and 3 (not folded
// further: the LDS adds join them).  Shift-8 and shift-4 exchanges that write
// only some banks (bank_mask: no select) merge the four into one, a quad of
// lanes per register in the order A, dx^2 A, dx A, B, and two exchanges
// within the quad finish the sums: every lane of a quad holds its total
// (nine_slot says which one).  DPP adds need two wait states after the VALU
// write of what they read.  Runs in converged control flow with every lane
// active.  Against sums of all nine per lane and two LDS adds (some forty
// instructions per entry and wave, beside about 25 per pixel): 10 views
// 1200x680, tile 32, 728 -> 688 us; one view, tile 16, 138 -> 128 us.
__device__ __forceinline__ float wave_sum9(float S0, float S1, float S2,
                                           float d_r, float d_g, float d_b,
                                           float dx) {
  const float A = fold16(fold32(S0, S1), fold32(S2, d_r));
  const float B = fold32(d_g, d_b);
  const float A1 = dx * A, A2 = dx * A1;
  float x, y, z;
  asm volatile(
      "s_nop 1\n\t"
      "v_add_f32_dpp %[x], %[A], %[A] row_shl:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %[x], %[A1], %[A1] row_shr:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %[y], %[A2], %[A2] row_shl:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %[y], %[B], %[B] row_shr:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %[z], %[x], %[x] row_shl:4 row_mask:0xf bank_mask:0x5\n\t"
      "s_nop 0\n\t"
      "v_add_f32_dpp %[z], %[y], %[y] row_shr:4 row_mask:0xf bank_mask:0xa\n\t"
      "s_nop 1\n\t"
      "v_add_f32_dpp %[z], %[z], %[z] quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\t"
      "v_add_f32_dpp %[z], %[z], %[z] quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
      : [x] "=&v"(x), [y] "=&v"(y), [z] "=&v"(z)
      : [A] "v"(A), [A1] "v"(A1), [A2] "v"(A2), [B] "v"(B));
  return z;
}

// The slot of the nine (in the order above) that a lane adds its wave_sum9
// to, -1 for none: the first lane of each quad that holds one.
__device__ __forceinline__ int nine_slot(int lane) {
  if (lane & 3) return -1;
  const int row = lane >> 4;
  switch ((lane >> 2) & 3) {
    case 0: return row == 0 ? 0 : row == 1 ? 5 : row == 2 ? 3 : 6;   // A
    case 1: return row == 0 ? 2 : -1;                                // dx^2 A
    case 2: return row == 0 ? 1 : row == 2 ? 4 : -1;                 // dx A
    default: return row < 2 ? 7 : 8;                                 // B
  }
}

// Sum over the lane's 16-lane row, in every lane of the row.
__device__ __forceinline__ float row_sum(float x) {
  x = add_dpp<0xb1>(x, x);   // quad_perm [1,0,3,2]
  x = add_dpp<0x4e>(x, x);   // quad_perm [2,3,0,1]
  x = add_dpp<0x141>(x, x);  // row_half_mirror
  x = add_dpp<0x140>(x, x);  // row_mirror
  return x;
}

__device__ __forceinline__ int wave_max(int x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x = max(x, __shfl_xor(x, off, 64));
  return x;
}

__device__ __forceinline__ int wave_min(int x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x = min(x, __shfl_xor(x, off, 64));
  return x;
}

template <int PPT>
struct BwdPix {
  float T[PPT], g0[PPT], g1[PPT], g2[PPT], Tb[PPT], Sg[PPT], vf[PPT];
  int last[PPT];
};

// Per-lane sums of one entry over the thread's strip: S0, S1, S2 are the
// moments sum(dL/dpi dy^k), k = 0, 1, 2.
struct EntrySums {
  float S0, S1, S2, d_r, d_g, d_b;
  bool hit;
};

// The backward of one entry over the thread's strip, back to front: T is
// recovered as T_{i+1} / (1 - alpha_i) (a pair that is not admitted takes
// alpha 0: 1 / (1 - 0) is exactly 1, so T, the weight and the running colour
// sum come out unchanged without a select each).  inb[p]: the pixel lies in
// the entry's render box and before its n_last (all true on the fast path).
// CLAMP: some entry of the batch has opacity above alpha_max, so alpha is
// clamped and a clamped pair passes no shape or opacity gradient; batches
// without such an entry (nearly all) run the version without the clamp.
// BG: a non-zero background, whose term enters dL/dalpha.  With the weight
// w = alpha T_i, dL/dpi = alpha dL/dalpha is w (c.g - S) without a
// background.  The moments are formed from P0 = sum(dL/dpi),
// P1 = sum(p dL/dpi) and P2 = sum(p^2 dL/dpi) over the strip's rows p:
// with dy_p = dy_0 - p, S1 = dy_0 P0 - P1 and
// S2 = dy_0^2 P0 - 2 dy_0 P1 + P2 = dy_0 (S1 - P1) + P2.
template <bool CLAMP, bool BG, int PPT>
__device__ __forceinline__ EntrySums entry_bwd(BwdPix<PPT>& px,
                                               const Column& col, float py,
                                               float C2, float cr, float cgc,
                                               float cbc, float amin,
                                               float amax, const bool* inb) {
  EntrySums r;
  r.hit = false;
  r.d_r = r.d_g = r.d_b = 0.f;
  float P0 = 0.f, P1 = 0.f, P2 = 0.f, dy0 = 0.f;
#pragma unroll
  for (int p = 0; p < PPT; ++p) {
    float dy;
    const float e2 = exponent2(col, py, C2, px.vf[p], dy);
    if (p == 0) dy0 = dy;
    const float oG = alpha2(e2);
    const float al = CLAMP ? fminf(amax, oG) : oG;
    const bool ok = inb[p] && al >= amin;
    r.hit |= ok;
    const float alo = ok ? al : 0.f;
    const float rom = __builtin_amdgcn_rcpf(1.f - alo);
    const float Ti = px.T[p] * rom;                 // T_i
    px.T[p] = Ti;
    const float w = alo * Ti;
    r.d_r = fmaf(w, px.g0[p], r.d_r);
    r.d_g = fmaf(w, px.g1[p], r.d_g);
    r.d_b = fmaf(w, px.g2[p], r.d_b);
    const float cgp = fmaf(cr, px.g0[p], fmaf(cgc, px.g1[p], cbc * px.g2[p]));
    const float diff = cgp - px.Sg[p];
    px.Sg[p] = fmaf(alo, diff, px.Sg[p]);
    float dpw = BG ? alo * fmaf(Ti, diff, -(px.Tb[p] * rom)) : w * diff;
    if (CLAMP) dpw = oG > amax ? 0.f : dpw;
    if (p == 0) {
      P0 = dpw;
    } else {
      P0 += dpw;
      P1 = p == 1 ? dpw : fmaf((float)p, dpw, P1);
      P2 = p == 1 ? dpw : fmaf((float)(p * p), dpw, P2);
    }
  }
  r.S0 = P0;
  r.S1 = fmaf(dy0, P0, -P1);
  r.S2 = fmaf(dy0, r.S1 - P1, P2);
  return r;
}

// Staged entry j for one wave; fast: the wave's fast-path bit and the entry
// lies before every pixel's n_last.
template <bool CLAMP, bool BG, int TILE, int NT>
__device__ __forceinline__ void walk_entry(
    BwdPix<PixLayout<TILE, NT>::PPT>& px, const Entry* ent, float (*acc)[9],
    int j, int pos, bool fast, int u, int v0, float uf, float amin,
    float amax, int slot) {
  constexpr int PPT = PixLayout<TILE, NT>::PPT;
  const float4 ea = ent[j].a;
  const float4 eb = ent[j].b;
  const float ecb = ent[j].c.x;
  const Column col = column(ea, eb.y, uf);
  // Only the box / position masks differ between the fast and the general
  // path, chosen in scalar registers, so the pixels' running state is
  // updated by one common body.
  bool inb[PPT];
  if (fast) {
#pragma unroll
    for (int p = 0; p < PPT; ++p) inb[p] = true;
  } else {
    const int4 box = ent[j].box;
    const bool in_u = u >= box.x && u <= box.y;
    const int rlo = box.z - v0, rhi = box.w - v0;
#pragma unroll
    for (int p = 0; p < PPT; ++p)
      inb[p] = in_u && rlo <= p && p <= rhi && pos < px.last[p];
  }
  const EntrySums es = entry_bwd<CLAMP, BG>(px, col, ea.y, eb.x, eb.z, eb.w,
                                            ecb, amin, amax, inb);
  if (__builtin_amdgcn_ballot_w64(es.hit) != 0) {
    // The wave totals, added into the entry's LDS slots in one instruction;
    // the other waves of the tile meet there.
    const float x = wave_sum9(es.S0, es.S1, es.S2, es.d_r, es.d_g, es.d_b,
                              col.dx);
    if (slot >= 0) atomicAdd(&acc[j][slot], x);
  }
}

// The entries [0, jn) of the staged batch, back to front, for one wave: the
// set bits of its eval mask below jn, highest first.
template <bool CLAMP, bool BG, int TILE, int BATCH, int NT>
__device__ __forceinline__ void walk_batch(
    BwdPix<PixLayout<TILE, NT>::PPT>& px, const Entry* ent,
    const WaveMasks<BATCH, NT>& masks, float (*acc)[9], int jn, int lo,
    int wave, int wfirst, int u, int v0, float uf, float amin, float amax,
    int slot) {
  for (int k = (jn - 1) >> 5; k >= 0; --k) {
    uint32_t e = __builtin_amdgcn_readfirstlane(masks.eval[wave][k]);
    const uint32_t f = __builtin_amdgcn_readfirstlane(masks.fast[wave][k]);
    const int top = jn - 32 * k;   // entries of this word below jn
    if (top < 32) e &= (1u << top) - 1u;
    while (e) {
      const int b = 31 - __builtin_clz(e);
      e &= ~(1u << b);
      const int j = 32 * k + b;
      const int pos = lo + j;
      walk_entry<CLAMP, BG, TILE, NT>(px, ent, acc, j, pos,
                                      ((f >> b) & 1) && pos < wfirst, u, v0,
                                      uf, amin, amax, slot);
    }
  }
}

// Adds the staged entries' gradients, from the nine sums of each, to global
// memory.  Called by the NT threads of the workgroup after a barrier.
template <int NT>
__device__ __forceinline__ void flush(const BwdArgs& a, float (*acc)[9],
                                      const Entry* ent, const float* eop,
                                      const uint32_t* gid, int cnt, int k,
                                      int tid) {
  const RasterArgs& r = a.r;
  float* gk = a.grad2d + (size_t)k * 5 * r.cap;
  float* gc = a.grgb + (size_t)k * a.grgb_vstride;
  // Per entry: the mean, conic and opacity gradients from the nine sums
  // (A, B, C the unscaled conic, o the opacity), then one atomic each:
  // straight into the planar gradients, or back into the entry's LDS slot
  // for the per-Gaussian accumulators.
  for (int jj = tid; jj < cnt; jj += NT) {
    const float* ac = acc[jj];
    const float s0 = ac[0], xs0 = ac[1], x2s0 = ac[2], s1 = ac[3];
    const float xs1 = ac[4], s2 = ac[5];
    const float4 ec = ent[jj].c;
    const float A = ec.y, B = ec.z, C = ec.w;
    float val[9];
    val[0] = -fmaf(A, xs0, B * s1);   // dL/dpx
    val[1] = -fmaf(C, s1, B * xs0);   // dL/dpy
    val[2] = -0.5f * x2s0;            // dL/dA
    val[3] = -xs1;                    // dL/dB
    val[4] = -0.5f * s2;              // dL/dC
    val[5] = s0 / eop[jj];            // dL/do
    val[6] = ac[6];
    val[7] = ac[7];
    val[8] = ac[8];
    if (a.gview) {
      float* out = acc[jj];
#pragma unroll
      for (int q = 0; q < 5; ++q) out[q] = val[q];
      out[5] = val[6]; out[6] = val[7]; out[7] = val[8]; out[8] = val[5];
      continue;
    }
    const uint32_t g = gid[jj];
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      if (val[q] == 0.f) continue;
      if (q < 5) atomicAdd(&gk[(size_t)q * r.cap + g], val[q]);
      else if (q == 5) atomicAdd(&a.gop[g], val[q]);
      else atomicAdd(&gc[(size_t)(q - 6) * r.cap + g], val[q]);
    }
  }
  if (a.gview) {
    // Nine consecutive lanes per entry: its adds fall in one 64-byte and
    // one 32-byte piece, two requests to the memory side instead of nine.
    __syncthreads();
    double* gv = a.gview + (size_t)k * 8 * r.cap;
    const float* flat = &acc[0][0];
    for (int i = tid; i < cnt * 9; i += NT) {
      const float val = flat[i];
      if (val == 0.f) continue;
      const int jj = i / 9, q = i - 9 * jj;
      const size_t g = gid[jj];
      const bool view = q < 5 || (q < 8 && a.view_colour);
      atomicAdd(view ? gv + 8 * g + q : a.gsum + 4 * g + (q - 5), (double)val);
    }
  }
}

// The per-pixel work is predicated like the forward's: every lane evaluates
// its pixels for each entry and the admit decision selects what is
// accumulated.  A wave starts its backward walk at the largest n_last of its
// own pixels, skips entries no pixel of its footprint can admit and takes
// the fast path (its fast mask bit, and the entry before every pixel's
// n_last) when it can; the choice is uniform over the wave, made in scalar
// registers.
template <int TILE, int BATCH, int NT, bool BG>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(BG ? 1 : 5))) void k_render_bwd(BwdArgs a) {
  using Lay = PixLayout<TILE, NT>;
  constexpr int PPT = Lay::PPT;
  __shared__ Entry ent[BATCH];
  __shared__ float acc[BATCH][9];
  __shared__ uint32_t gid[BATCH];
  __shared__ float eop[BATCH];   // opacity per staged entry
  __shared__ int smax;
  __shared__ double psh[NT / 64];
  if ((int)blockIdx.x >= a.tile_blocks) {   // dispatched last: the tail
    planar_part(a.planar, (int)blockIdx.x - a.tile_blocks,
                (int)gridDim.x - a.tile_blocks, psh);
    return;
  }
  const RasterArgs& r = a.r;
  const int t = (int)r.order[blockIdx.x];
  const int tpv = r.Tx * r.Ty;
  const int k = t / tpv;
  const int rem = t - k * tpv;
  const int ty = rem / r.Tx, tx = rem - ty * r.Tx;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  long long s, e;
  tile_range(r, t, s, e);
  const size_t HW = (size_t)r.H * r.W;

  int cu, cv0;
  Lay::of(tid, cu, cv0);
  const int u = tx * TILE + cu;
  const int v0 = ty * TILE + cv0;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  __shared__ WaveMasks<BATCH, NT> masks;
  const float uf = pinned((float)u);
  const float amax = r.alpha_max, amin = r.alpha_min;
  const int slot = nine_slot(lane);
  BwdPix<PPT> px;
  int mylast = 0, myfirst = 0x7fffffff;
  float l1_abs = 0.f;
  double l1_sq = 0.0;
#pragma unroll
  for (int p = 0; p < PPT; ++p) {
    const int v = v0 + p;
    px.last[p] = 0;
    px.vf[p] = pinned((float)v);
    // Pixels outside the image keep T = 0 and a zero gradient: every term
    // they could add is zero.
    px.T[p] = 0.f; px.g0[p] = px.g1[p] = px.g2[p] = 0.f; px.Tb[p] = 0.f;
    px.Sg[p] = 0.f;
    if (u < r.W && v < r.H) {
      const size_t pix = (size_t)v * r.W + u;
      px.T[p] = a.Tfin[(size_t)k * HW + pix];
      px.last[p] = a.nlast[(size_t)k * HW + pix];
      if (a.target) {
        float gg[3];
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
          const size_t i = ((size_t)k * 3 + ch) * HW + pix;
          const float d = a.rgb[i] - a.target[i];
          l1_abs += fabsf(d);
          l1_sq += (double)d * (double)d;
          gg[ch] = l1_grad(d, a.l1_scale);
        }
        px.g0[p] = gg[0]; px.g1[p] = gg[1]; px.g2[p] = gg[2];
      } else {
        px.g0[p] = a.dL[((size_t)k * 3 + 0) * HW + pix];
        px.g1[p] = a.dL[((size_t)k * 3 + 1) * HW + pix];
        px.g2[p] = a.dL[((size_t)k * 3 + 2) * HW + pix];
      }
      px.Tb[p] = px.T[p] * (r.bg0 * px.g0[p] + r.bg1 * px.g1[p] + r.bg2 * px.g2[p]);
      mylast = max(mylast, px.last[p]);
      myfirst = min(myfirst, px.last[p]);
    }
  }
  // The tile's share of the fused L1 loss: wave sums, then one plain store
  // per workgroup (a second kernel sums the tiles: FP64 atomics on one
  // address would serialise).
  __shared__ double lpart[2][NT / 64];
  if (a.target) {
    double la = l1_abs, lq = l1_sq;
    for (int off = 32; off > 0; off >>= 1) {
      la += __shfl_down(la, off, 64);
      lq += __shfl_down(lq, off, 64);
    }
    if (lane == 0) {
      lpart[0][wave] = la;
      lpart[1][wave] = lq;
    }
  }
  if (tid == 0) smax = 0;
  __syncthreads();
  atomicMax(&smax, mylast);
  const int wlast = __builtin_amdgcn_readfirstlane(wave_max(mylast));
  // Entries before every pixel's n_last: no per-pixel position test.
  const int wfirst = __builtin_amdgcn_readfirstlane(wave_min(myfirst));
  __syncthreads();
  if (a.target && tid == 0) {
    double la = 0.0, lq = 0.0;
    for (int w = 0; w < NT / 64; ++w) {
      la += lpart[0][w];
      lq += lpart[1][w];
    }
    a.tile_loss[2 * (size_t)t] = la * a.l1_lam_inv;
    a.tile_loss[2 * (size_t)t + 1] = lq;
  }
  const int maxlast = (int)min((long long)smax, e - s);
  const Record* rv = r.rec + (size_t)k * r.cap;
  const int2* rbv = r.rbox + (size_t)k * r.cap;
  for (int hi = maxlast; hi > 0; hi -= BATCH) {
    const int lo = max(0, hi - BATCH);
    const int cnt = hi - lo;
    __syncthreads();   // the previous batch is flushed
    int clampable = 0;
#pragma unroll
    for (int i0 = 0; i0 < BATCH; i0 += NT) {
      const int i = i0 + tid;
      int bits = 0;
      if (i < cnt) {
        const uint32_t g = r.vals[s + lo + i];
        gid[i] = g;
        const Record R = rv[g];
        eop[i] = R.q1.y;
        const int4 box = unpack_box(rbv[g]);
        stage(ent[i], R, box, r.lop[g]);
        bits = wave_bits<TILE, NT>(R, box, tx * TILE, ty * TILE, r.W, r.H,
                                   amin, amax, r.ellipse_test);
        clampable |= R.q1.y > amax;
      }
      publish_masks(masks, i0, bits, wave, lane);
    }
    for (int i = tid; i < cnt * 9; i += NT) (&acc[0][0])[i] = 0.f;
    const int jn = min(cnt, wlast - lo);
    if (__syncthreads_or(clampable)) {
      walk_batch<true, BG, TILE, BATCH, NT>(px, ent, masks, acc, jn, lo, wave,
                                            wfirst, u, v0, uf, amin, amax,
                                            slot);
    } else {
      walk_batch<false, BG, TILE, BATCH, NT>(px, ent, masks, acc, jn, lo, wave,
                                             wfirst, u, v0, uf, amin, amax,
                                             slot);
    }
    __syncthreads();
    flush<NT>(a, acc, ent, eop, gid, cnt, k, tid);
  }
}

// Sums over each 16-lane row of eight per-lane values: lane l of the row
// receives the total of q[l >> 1] in the order 0, 4, 2, 6, 1, 5, 3, 7 (bit 3
// of l picks the value's bit 0, bit 2 its bit 1, bit 1 its bit 2).  A
// transposed reduction: each exchange merges two registers into one (see
// wave_sum9 for bank_mask and the waits).
__device__ __forceinline__ float merge8(float a, float b) {
  float x;
  asm("s_nop 1\n\t"
      "v_add_f32_dpp %[x], %[a], %[a] row_shl:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %[x], %[b], %[b] row_shr:8 row_mask:0xf bank_mask:0xc\n\ts_nop 1"
      : [x] "=&v"(x)
      : [a] "v"(a), [b] "v"(b));
  return x;
}

__device__ __forceinline__ float merge4(float a, float b) {
  float x;
  asm("s_nop 1\n\t"
      "v_add_f32_dpp %[x], %[a], %[a] row_shl:4 row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %[x], %[b], %[b] row_shr:4 row_mask:0xf bank_mask:0xa\n\ts_nop 1"
      : [x] "=&v"(x)
      : [a] "v"(a), [b] "v"(b));
  return x;
}

__device__ __forceinline__ float row_sum8(const float (&q)[8], int lane) {
  const float a = merge4(merge8(q[0], q[1]), merge8(q[2], q[3]));
  const float b = merge4(merge8(q[4], q[5]), merge8(q[6], q[7]));
  const float a2 = add_dpp<0x4e>(a, a), b2 = add_dpp<0x4e>(b, b);
  const float x = lane & 2 ? b2 : a2;
  return add_dpp<0xb1>(x, x);
}

// The split shape (k_render_fwd_split): lane 16 r + p of a wave holds pixel p
// and takes the entries n - 1 - 4 i - r of the wave's list.  A step evaluates
// alpha, 1 / (1 - alpha) and the colour term of its own entry, hands them to
// all rows, and every row runs the pixel's T and running colour sum through
// the four entries in order, picking up the values that its own entry needs;
// the nine sums are reduced within the row and added to the entry's LDS slot.
template <int TILE, bool BG>
__global__ __launch_bounds__(BlockLayout::kThreads)
void k_render_bwd_split(BwdArgs a) {
  constexpr int kBatch = BlockLayout::kBatch, NT = BlockLayout::kThreads;
  __shared__ Entry ent[kBatch];
  __shared__ float acc[kBatch][9];
  __shared__ uint32_t gid[kBatch];
  __shared__ float eop[kBatch];
  __shared__ BlockLists lists;
  __shared__ int wmax[4];
  __shared__ double psh[NT / 64], lpart[2][NT / 64];
  if ((int)blockIdx.x >= a.tile_blocks) {   // dispatched last: the tail
    planar_part(a.planar, (int)blockIdx.x - a.tile_blocks,
                (int)gridDim.x - a.tile_blocks, psh);
    return;
  }
  const RasterArgs& r = a.r;
  constexpr int kParts = tile_parts(TILE), kAcross = TILE / BlockLayout::kSide;
  const int t = (int)r.order[blockIdx.x / kParts];
  const int part = blockIdx.x % kParts;
  const int tpv = r.Tx * r.Ty;
  const int k = t / tpv;
  const int rem = t - k * tpv;
  const int ty = rem / r.Tx, tx = rem - ty * r.Tx;
  const int tid = threadIdx.x, lane = tid & 63, row = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  long long s, e;
  tile_range(r, t, s, e);
  const size_t HW = (size_t)r.H * r.W;
  const int bu = tx * TILE + (part % kAcross) * BlockLayout::kSide;
  const int bv = ty * TILE + (part / kAcross) * BlockLayout::kSide;
  int wu, wv;
  BlockLayout::wave_origin(wave, wu, wv);
  BlockPixel px;
  px.u = bu + wu + (lane & 3);
  px.v = bv + wv + ((lane >> 2) & 3);
  px.uf = pinned((float)px.u);
  px.vf = pinned((float)px.v);
  const float amin = r.alpha_min;
  // Pixels outside the image keep T = 0 and a zero gradient: every term they
  // could add is zero.
  float T = 0.f, g0 = 0.f, g1 = 0.f, g2 = 0.f, Sg = 0.f;
  int last = 0;
  float l1_abs = 0.f;
  double l1_sq = 0.0;
  if (px.u < r.W && px.v < r.H) {
    const size_t pix = (size_t)px.v * r.W + px.u;
    T = a.Tfin[(size_t)k * HW + pix];
    last = a.nlast[(size_t)k * HW + pix];
    const size_t i0 = (size_t)k * 3 * HW + pix;
    if (a.target) {
      float d[3];
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) {
        d[ch] = a.rgb[i0 + ch * HW] - a.target[i0 + ch * HW];
        if (row == 0) {   // one row adds the pixel's loss
          l1_abs += fabsf(d[ch]);
          l1_sq += (double)d[ch] * (double)d[ch];
        }
      }
      g0 = l1_grad(d[0], a.l1_scale);
      g1 = l1_grad(d[1], a.l1_scale);
      g2 = l1_grad(d[2], a.l1_scale);
    } else {
      g0 = a.dL[i0];
      g1 = a.dL[i0 + HW];
      g2 = a.dL[i0 + 2 * HW];
    }
  }
  const float Tb = T * (r.bg0 * g0 + r.bg1 * g1 + r.bg2 * g2);
  if (a.target) {
    double la = l1_abs, lq = l1_sq;
    for (int off = 8; off > 0; off >>= 1) {
      la += __shfl_down(la, off, 64);
      lq += __shfl_down(lq, off, 64);
    }
    if (lane == 0) {
      lpart[0][wave] = la;
      lpart[1][wave] = lq;
    }
  }
  const int wlast = __builtin_amdgcn_readfirstlane(wave_max(last));
  if (lane == 0) wmax[wave] = wlast;
  __syncthreads();
  if (a.target && tid == 0) {
    double* out = a.tile_loss + 2 * ((size_t)t * kParts + part);
    out[0] = ((lpart[0][0] + lpart[0][1]) + (lpart[0][2] + lpart[0][3])) * a.l1_lam_inv;
    out[1] = (lpart[1][0] + lpart[1][1]) + (lpart[1][2] + lpart[1][3]);
  }
  const int maxlast = (int)min((long long)max(max(wmax[0], wmax[1]), max(wmax[2], wmax[3])),
                               e - s);
  const Record* rv = r.rec + (size_t)k * r.cap;
  const int2* rbv = r.rbox + (size_t)k * r.cap;
  // The value that the lane's row sum holds, and the slot that it adds it to
  // (lane 1: the ninth sum).
  const int slot = (lane & 15) == 1 ? 8
                   : ((lane >> 3) & 1) | ((lane >> 2) & 1) << 1 | ((lane >> 1) & 1) << 2;
  const bool adds = (lane & 1) == 0 || (lane & 15) == 1;
  for (int hi = maxlast; hi > 0; hi -= kBatch) {
    const int lo = max(0, hi - kBatch);
    const int cnt = hi - lo;
    __syncthreads();   // the previous batch is flushed
    int m = 0, clampable = 0;
    if (tid < cnt) {
      const uint32_t g = r.vals[s + lo + tid];
      gid[tid] = g;
      const Record R = rv[g];
      eop[tid] = R.q1.y;
      const int4 box = unpack_box(rbv[g]);
      stage(ent[tid], R, box, r.lop[g]);
      m = wave_mask<BlockLayout, 4>(R, box, bu, bv, amin, r.ellipse_test);
      clampable = R.q1.y > r.alpha_max;
    }
    lists.publish(m, wave, lane);
    for (int i = tid; i < cnt * 9; i += NT) (&acc[0][0])[i] = 0.f;
    const float amax = __syncthreads_or(clampable) ? r.alpha_max : INFINITY;
    const int n = lists.gather(min(cnt, wlast - lo), wave, lane);
    const uint16_t* list = lists.list[wave];
    auto at = [&](int i) { return (int)list[max(n - 1 - 4 * i - row, 0)]; };
    const int steps = (n + 3) >> 2;
    if (steps > 0) {
      int j = at(0), jn = at(1);
      BlockWords w;
      w.load(ent[j]);
#pragma unroll 2
      for (int i = 0; i < steps; ++i) {
        BlockWords wn;
        wn.load(ent[jn]);
        const int jnn = at(i + 2);
        float dx, dy;
        int out;
        const float oG = block_alpha(w, px, dx, dy, out);
        const float al = fminf(amax, oG);
        // Past the list's start the first entry stands again: not admitted.
        out |= (last - 1 - lo - j) | (n - 1 - 4 * i - row);
        const float alo = out >= 0 ? (al >= amin ? al : 0.f) : 0.f;
        const float rom = __builtin_amdgcn_rcpf(1.f - alo);
        const float cg = fmaf(w.b.z, g0, fmaf(w.b.w, g1, w.cb * g2));
        const Rows xa = all_rows(alo), xr = all_rows(rom), xc = all_rows(cg);
        float Town = 0.f, Sown = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          T *= xr.v[q];
          Town = q == 0 ? T : row == q ? T : Town;
          Sown = q == 0 ? Sg : row == q ? Sg : Sown;
          Sg = fmaf(xa.v[q], xc.v[q] - Sg, Sg);
        }
        const float wt = alo * Town, diff = cg - Sown;
        float dpw = BG ? alo * fmaf(Town, diff, -(Tb * rom)) : wt * diff;
        dpw = oG > amax ? 0.f : dpw;
        const float xs0 = dx * dpw, s1 = dy * dpw;
        const float q8[8] = {dpw, xs0, dx * xs0, s1, dx * s1, dy * s1, wt * g0, wt * g1};
        const float x = row_sum8(q8, lane);
        const float z = row_sum(wt * g2);
        // Nothing is added for an entry that no pixel of the row admits.
        const uint64_t hit = __builtin_amdgcn_ballot_w64(alo > 0.f);
        const bool any = ((uint32_t)(hit >> (16 * row)) & 0xffffu) != 0;
        if (any && adds) atomicAdd(&acc[j][slot], (lane & 15) == 1 ? z : x);
        w = wn;
        j = jn;
        jn = jnn;
      }
    }
    __syncthreads();
    flush<NT>(a, acc, ent, eop, gid, cnt, k, tid);
  }
}

// The per-Gaussian accumulators added to the planar gradients and cleared:
// grid (Gaussians / 256, views); one more column where the fused L1 term's
// losses are to be summed, which saves a launch of 4 us.
__global__ __launch_bounds__(256) void k_spread(BwdArgs a) {
  __shared__ double part[4];
  if ((int)blockIdx.x >= a.spread_blocks) {
    if (blockIdx.y == 0) l1_reduce_part(a.l1, part);
    return;
  }
  const int g = blockIdx.x * 256 + threadIdx.x, k = blockIdx.y;
  const size_t cap = a.r.cap;
  if (g >= a.r.cap) return;
  double2* p = (double2*)a.gview + (k * cap + g) * 4;
  const double2 zero = make_double2(0.0, 0.0);
  const double2 v0 = p[0], v1 = p[1], v2 = p[2], v3 = p[3];
  const double v[8] = {v0.x, v0.y, v1.x, v1.y, v2.x, v2.y, v3.x, v3.y};
  bool any = false;
  float* gk = a.grad2d + k * 5 * cap + g;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    if (v[q] == 0.0) continue;
    any = true;
    float* out = q < 5 ? gk + q * cap
                       : a.grgb + k * a.grgb_vstride + (q - 5) * cap + g;
    *out += (float)v[q];
  }
  if (any) p[0] = p[1] = p[2] = p[3] = zero;
  if (k != 0) return;
  double2* s = (double2*)a.gsum + 2 * (size_t)g;
  const double2 s0 = s[0], s1 = s[1];
  const double t[4] = {s0.x, s0.y, s1.x, s1.y};
  any = false;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (t[q] == 0.0) continue;
    any = true;
    float* out = q < 3 ? a.grgb + q * cap + g : a.gop + g;
    *out += (float)t[q];
  }
  if (any) s[0] = s[1] = zero;
}

// Sum of the tiles' fused L1 losses into *loss and of each view's squared
// errors into sqerr[view], in a fixed order (l1_reduce_part).
__global__ __launch_bounds__(1024) void k_l1_reduce(L1ReduceJob j) {
  __shared__ double part[16];
  l1_reduce_part(j, part);
}

// Where the gradients go.  Straight into the planar rows, each entry of a
// tile costs nine adds on nine lines, and a pass with many (tile, entry)
// pairs is bound by them (about 55 G adds/s reach the memory side): 5.0 M
// keys (10 views 640x480, tile 16) take 0.82 ms, of which 0.37 ms remain
// with the adds left out; tile 32 has a third of the keys, 0.351 against
// 0.344 ms.  Through the per-Gaussian accumulators the same pass takes 0.41
// ms.  The window graph's projection backward reads the accumulators; the
// entry points publish planar rows, so there a pass over the accumulators
// follows (9 us at 300k Gaussians and one view), which pays at tiles below
// 32 (1200x680, tile 16: 0.28 -> 0.164 ms with the pass; tile 32: 0.123 ms
// either way) from this many tiles on.  Whole backward us, planar rows
// against accumulators: 300 tiles of 16 48 / 52, 475 78 / 64, 690 106 / 82,
// 1,200 123 / 107; 690 tiles of 8 49 / 46.  In blocks it pays from about 450
// of them (320 25 / 27, 720 39 / 33, 1,200 67 / 47), but the accumulators are
// taken for all: four times as many FP32 adds per tile into a planar row
// would double the rounding of the case below.  The accumulators are FP64: a Gaussian next to the camera
// sums thousands of tiles' parts that mostly cancel, and FP32 adds in
// whatever order they arrive left its gradient 1.4e-6 to 4.6e-6 off from run
// to run (now 4.0e-7 on the same input, every run).
constexpr int kSpreadBlocks = 450;

struct BwdLauncher {
  const BwdArgs& a;
  int blocks;
  bool bg;
  hipStream_t st;
  template <int T, int B, int N>
  void go() const {
    if (bg)
      hipLaunchKernelGGL((k_render_bwd<T, B, N, true>), dim3(blocks), dim3(N),
                         0, st, a);
    else
      hipLaunchKernelGGL((k_render_bwd<T, B, N, false>), dim3(blocks),
                         dim3(N), 0, st, a);
  }
  void split(int tile) const {
    const dim3 grid(blocks), nt(BlockLayout::kThreads);
    if (tile == 8 && bg) hipLaunchKernelGGL((k_render_bwd_split<8, true>), grid, nt, 0, st, a);
    else if (tile == 8) hipLaunchKernelGGL((k_render_bwd_split<8, false>), grid, nt, 0, st, a);
    else if (bg) hipLaunchKernelGGL((k_render_bwd_split<16, true>), grid, nt, 0, st, a);
    else hipLaunchKernelGGL((k_render_bwd_split<16, false>), grid, nt, 0, st, a);
  }
};

}  // namespace

hipError_t launch_render_bwd(gs_workspace* ws, const gs_settings* s,
                             const float* dL, const float* T,
                             const int32_t* nlast, float* grad_rgb,
                             int per_view_colour, const L1Fused* l1,
                             hipStream_t st, const PlanarJob* planar,
                             bool window) {
  BwdArgs a;
  a.r = make_raster_args(ws, s);
  a.dL = dL; a.Tfin = T; a.nlast = nlast;
  a.rgb = nullptr; a.target = nullptr; a.l1_scale = 0.f; a.l1_lam_inv = 0.0;
  a.tile_loss = ws->tile_loss;
  if (l1) {
    const size_t per = (size_t)3 * ws->geo.height * ws->geo.width;
    a.rgb = l1->rgb; a.target = l1->target;
    a.l1_scale = (float)((double)l1->lambda / (double)per);
    a.l1_lam_inv = (double)l1->lambda / (double)per;
  }
  a.grad2d = ws->grad2d; a.gop = ws->gop;
  a.grgb = per_view_colour ? ws->gcol : grad_rgb;
  a.grgb_vstride = per_view_colour ? (size_t)3 * ws->geo.capacity : 0;
  a.view_colour = per_view_colour;
  const int tiles = ws->geo.n_views * ws->tiles_x * ws->tiles_y;
  const bool split = split_shape(ws, s, true);
  a.tile_blocks = split ? tiles * tile_parts(ws->geo.tile) : tiles;
  const bool spread =
      !window && ws->geo.tile < 32 && (split || tiles >= kSpreadBlocks);
  const bool acc = window || spread;
  a.gview = acc ? ws->gview : nullptr; a.gsum = acc ? ws->gsum : nullptr;
  a.planar = planar ? *planar : PlanarJob{};
  a.spread_blocks = 0;
  a.l1 = L1ReduceJob{};
  if (tiles <= 0) {
    if (planar) {
      const hipError_t e = launch_planar_job(*planar, st);
      if (e != hipSuccess) return e;
    }
  } else {
    // The regulariser's workgroups (a grid stride over the Gaussians, as
    // many as its own launch would have) follow the tiles'.
    const RasterShape shape = raster_shape(ws, s);
    const int nt = split ? BlockLayout::kThreads : shape.threads;
    const int pb = planar ? min(256, (planar->cap + nt - 1) / nt) : 0;
    const bool bg = s->bg[0] != 0.f || s->bg[1] != 0.f || s->bg[2] != 0.f;
    const BwdLauncher launcher{a, a.tile_blocks + pb, bg, st};
    if (split) launcher.split(shape.tile);
    else dispatch_shape(shape, launcher);
    if (spread && ws->geo.capacity > 0) {
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      const bool sum = l1 && !l1->defer_reduce;
      a.spread_blocks = (ws->geo.capacity + 255) / 256;
      if (sum) a.l1 = l1_reduce_job(ws, s, l1->loss, l1->sqerr);
      hipLaunchKernelGGL(k_spread, dim3(a.spread_blocks + sum, ws->geo.n_views),
                         dim3(256), 0, st, a);
      if (sum) return hipGetLastError();
    }
  }
  if (l1 && !l1->defer_reduce) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_l1_reduce(ws, s, l1->loss, l1->sqerr, st);
  }
  return hipGetLastError();
}

L1ReduceJob l1_reduce_job(const gs_workspace* ws, const gs_settings* s,
                          double* loss, double* sqerr) {
  const int parts = split_shape(ws, s, true) ? tile_parts(ws->geo.tile) : 1;
  return L1ReduceJob{(const double2*)ws->tile_loss, ws->geo.n_views,
                     ws->tiles_x * ws->tiles_y * parts, loss, sqerr};
}

hipError_t launch_l1_reduce(const gs_workspace* ws, const gs_settings* s,
                            double* loss, double* sqerr, hipStream_t st) {
  hipLaunchKernelGGL(k_l1_reduce, dim3(1), dim3(1024), 0, st,
                     l1_reduce_job(ws, s, loss, sqerr));
  return hipGetLastError();
}

}  // namespace gs
