// Student-training kernels: loss seeds, the tangent pass along the force
// residual, the reverse sweep through the descriptor and the embedding net,
// weight-gradient reductions and Adam.
//
// Notation (per pair p of centre i): s = sw(r)/r, rhat = d/r,
// R~ = (s, s rhat) (Sec. II-B), G = emb(s; t_j, t_i) with G' = dG/ds,
// T_i = (1/sel) sum_p R~_p (x) G_p, D_i = T^T T[:, :axis] (Sec. II-B DP-SE
// descriptor).  A dot marks the derivative along the displacement field
// Delta (d-dot_p = Delta_j - Delta_i), a bar the adjoint of
// Psi = sum_i (a e_i - e-dot_i).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "dpa1_internal.h"
#include "train_internal.h"

namespace dpa1 {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Order of one wavefront's LDS accesses (the hardware keeps them in order).
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------- seeds

__global__ __launch_bounds__(256) void k_tr_seed(const double *__restrict__ F,
                                                 const double *__restrict__ Flab, int n, float cf,
                                                 float4 *__restrict__ delta,
                                                 double *__restrict__ sq_part) {
  __shared__ double red[256];
  const int k = blockIdx.x * 256 + threadIdx.x;
  double sq = 0.0;
  if (k < n) {
    const double dx = F[3 * k] - Flab[3 * k];
    const double dy = F[3 * k + 1] - Flab[3 * k + 1];
    const double dz = F[3 * k + 2] - Flab[3 * k + 2];
    sq = dx * dx + dy * dy + dz * dz;
    delta[k] = make_float4((float)(cf * dx), (float)(cf * dy), (float)(cf * dz), 0.f);
  }
  red[threadIdx.x] = sq;
  __syncthreads();
  for (int h = 128; h >= 1; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) sq_part[blockIdx.x] = red[0];
}

__global__ void k_tr_energy_seed(const double *__restrict__ E, const double *__restrict__ Elab,
                                 double ca, double cl, float *__restrict__ a,
                                 double *__restrict__ le) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    const double d = E[0] - Elab[0];
    a[0] = (float)(ca * d);
    le[0] = cl * d * d;
  }
}

// ------------------------------------------------------- per-pair helpers

struct PairTangent {
  float s, sdot;
  float Rt[4], Rd[4];  // R~ and its derivative along Delta
};

// Geometry record -> R~, its tangent and s-dot (ds/dr = dsw/r - s/r).
__device__ __forceinline__ PairTangent pair_tangent(const float4 g0, const float4 g1,
                                                    const float4 di, const float4 dj) {
  PairTangent t;
  const float s = g0.x, rx = g0.y, ry = g0.z, rz = g0.w, r = g1.y, dsw = g1.z;
  const float ddx = dj.x - di.x, ddy = dj.y - di.y, ddz = dj.z - di.z;
  // (written as the fused operations they are, so that every kernel gets the
  // same bits)
  const float rdot = fmaf(rz, ddz, fmaf(ry, ddy, rx * ddx));
  const float inv_r = 1.0f / r;
  const float sdot = (dsw - s) * inv_r * rdot;
  const float ux = fmaf(-rx, rdot, ddx) * inv_r, uy = fmaf(-ry, rdot, ddy) * inv_r,
              uz = fmaf(-rz, rdot, ddz) * inv_r;
  t.s = s;
  t.sdot = sdot;
  t.Rt[0] = s;
  t.Rt[1] = s * rx;
  t.Rt[2] = s * ry;
  t.Rt[3] = s * rz;
  t.Rd[0] = sdot;
  t.Rd[1] = fmaf(rx, sdot, s * ux);
  t.Rd[2] = fmaf(ry, sdot, s * uy);
  t.Rd[3] = fmaf(rz, sdot, s * uz);
  return t;
}

// ------------------------------------------------ embedding net on 16 pairs
//
// The per-pair embedding passes run on the FP32 matrix cores, a wavefront
// taking tiles of 16 pairs of its centre.  v_mfma_f32_16x16x4_f32 is, bit for
// bit, a chain of fused multiply-adds over its four depths in order (checked on
// the hardware over 1.5 M results), so a product over ascending depth started
// from the bias gives the bits of the scalar loop z = fma(w[k], h[k], z), at
// twice the vector unit's rate and without a scalar weight load per use.  With
// weights as the row operand a lane receives, for pair r = lane % 16, outputs
// 16 t + 4 g + {0..3} (g = lane / 16) of tile t; as the column operand of the
// next product it has to hold depth 4 c + g in step c, which a turn through
// wave-private LDS arranges (rows of 68 or 36 floats: no bank conflicts).
// Weights sit in LDS in the order of the steps: 64 lanes' values side by side.
//
// One lane per pair with scalar weights left a third of the lanes idle (84
// neighbours in two chunks of 64) and, at 256 registers and more, one wavefront
// per SIMD.  Per frame at 15,668 atoms: tangents 753 -> 251 us, adjoints
// 1304 + 325 (a second kernel for the first two layers) -> 1058 us; at 192 atoms
// 58 -> 26 and 85 + 18 -> 43 us.

constexpr int kTrWaves = 12;             // wavefronts of a workgroup, three per SIMD
constexpr int kTrRow = 68;               // LDS row of 64 values
constexpr int kTrRow2 = 36;              // LDS row of 32 values
constexpr int kTrTile = 16 * kTrRow;     // floats of a 16 x 64 tile
// operand order in LDS: W2 [2 tiles][4 steps], W3 [4][8], and for the reverse
// W3^T [2][16] and W2^T with the residual's unit rows [16]
constexpr int kTrW2 = 2 * 4 * 64, kTrW3 = 4 * 8 * 64, kTrW3r = 2 * 16 * 64, kTrW2r = 16 * 64;

__device__ __forceinline__ floatx4 mfma4(float a, float b, const floatx4 &c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ void stage_forward_weights(const TrainPairArgs &a, float *w2, float *w3) {
  for (int e = threadIdx.x; e < kTrW2; e += 64 * kTrWaves) {
    const int l = e & 63, c = (e >> 6) & 3, t = e >> 8;
    w2[e] = a.W2t[(16 * t + (l & 15)) * kTrN1 + 4 * c + (l >> 4)];
  }
  for (int e = threadIdx.x; e < kTrW3; e += 64 * kTrWaves) {
    const int l = e & 63, c = (e >> 6) & 7, t = e >> 9;
    w3[e] = a.W3t[(16 * t + (l & 15)) * kTrN2 + 4 * c + (l >> 4)];
  }
}

// One tile's first two layers.  h1, h1d: outputs 4 g + v; h2, h2d, t2, zd2
// (second layer's tanh and derivative sum): outputs 16 t + 4 g + v.
struct TileL12 {
  floatx4 h1, h1d;
  floatx4 h2[2], h2d[2], t2[2], zd2[2];
};

// First layer h1 = tanh(table[t_j][t_i] + ws s), h1' = (1 - h1^2) ws; second
// (doubling residual) h2 = tanh(W2^T h1 + b2) + [h1, h1] and
// h2' = (1 - t^2) W2^T h1' + [h1', h1'].
__device__ __forceinline__ void tile_l12(const TrainPairArgs &a, const float *w2, const float *tab,
                                         float s, int lane, int g, TileL12 &o) {
  const floatx4 tv = *(const floatx4 *)(tab + 4 * g), wv = *(const floatx4 *)(a.ws + 4 * g);
  float tb[4], wb[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    tb[c] = tab[4 * c + g];
    wb[c] = a.ws[4 * c + g];
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const float t = tanh_fast(fmaf(wv[v], s, tv[v]));
    o.h1[v] = t;
    o.h1d[v] = (1.0f - t * t) * wv[v];
  }
  floatx4 z[2], zd[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    z[t] = *(const floatx4 *)(a.b2 + 16 * t + 4 * g);
    zd[t] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float t = tanh_fast(fmaf(wb[c], s, tb[c]));
    const float td = (1.0f - t * t) * wb[c];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float w = w2[(q * 4 + c) * 64 + lane];
      z[q] = mfma4(w, t, z[q]);
      zd[q] = mfma4(w, td, zd[q]);
    }
  }
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float t = tanh_fast(z[q][v]);
      o.t2[q][v] = t;
      o.zd2[q][v] = zd[q][v];
      o.h2[q][v] = t + o.h1[v];
      o.h2d[q][v] = (1.0f - t * t) * zd[q][v] + o.h1d[v];
    }
}

// Third layer's sums z3 = W3^T h2 + b3 and W3^T h2' of one tile; buf: 2 x 16
// rows of kTrRow2.
__device__ __forceinline__ void tile_l3(const TrainPairArgs &a, const float *w3, float *buf,
                                        int lane, int r, int g, const TileL12 &x, floatx4 (&z)[4],
                                        floatx4 (&zd)[4]) {
  float *b2 = buf + 16 * kTrRow2;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    *(floatx4 *)(buf + r * kTrRow2 + 16 * q + 4 * g) = x.h2[q];
    *(floatx4 *)(b2 + r * kTrRow2 + 16 * q + 4 * g) = x.h2d[q];
  }
  wave_fence();
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    z[t] = *(const floatx4 *)(a.b3 + 16 * t + 4 * g);
    zd[t] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const float h = buf[r * kTrRow2 + 4 * c + g], hd = b2[r * kTrRow2 + 4 * c + g];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float w = w3[(t * 8 + c) * 64 + lane];
      z[t] = mfma4(w, h, z[t]);
      zd[t] = mfma4(w, hd, zd[t]);
    }
  }
  wave_fence();
}

// ------------------------------------------------------------ tangent pass

// One wavefront per centre.  Per tile of 16 pairs: G, G' (embedding forward and
// its s-derivative, lanes over pairs and features) and the coefficients of
// T-dot[c][m] = (1/sel) sum_p (R~-dot_p[c] G_p[m] + R~_p[c] s-dot_p G'_p[m]);
// lanes over m then accumulate T-dot pair by pair and at the end form
// D-dot[m][a] = sum_c (T-dot[c][m] T[c][a] + T[c][m] T-dot[c][a]).
constexpr int kTrTanWave = 2 * kTrTile + 16 * 8;  // G rows, G' rows, coefficients
constexpr size_t kTrTanLds = sizeof(float) * (kTrW2 + kTrW3 + kTrWaves * kTrTanWave);

__global__ __launch_bounds__(64 * kTrWaves, 3) void k_tr_tangent(TrainPairArgs a,
                                                                 const float4 *__restrict__ delta,
                                                                 float *__restrict__ Td,
                                                                 float *__restrict__ Xd, int ldD) {
  extern __shared__ float4 smem[];
  float *w2 = (float *)smem, *w3 = w2 + kTrW2;
  stage_forward_weights(a, w2, w3);
  __syncthreads();
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  float *sG = w3 + kTrW3 + w * kTrTanWave, *sGp = sG + kTrTile, *sC = sGp + kTrTile;
  for (int i = w * (int)gridDim.x + blockIdx.x; i < a.nloc; i += kTrWaves * gridDim.x) {
    const int n = a.nnei[i];
    const int off = a.pair_off[i];
    const int ti = a.types[i];
    const float4 di = delta[i];
    float tacc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int p0 = 0; p0 < n; p0 += 16) {
      const int pc = p0 + r < n ? p0 + r : 0;  // (rows past n: the first pair's, unused)
      const float4 *gp = (const float4 *)(a.geom + (size_t)(off + pc) * kGeom);
      const float4 g0 = gp[0], g1 = gp[1];
      const int j = a.nlist[(size_t)i * a.sel + pc];
      const int tj = a.types[j];
      const float4 dj = delta[j];
      const PairTangent pt = pair_tangent(g0, g1, di, dj);
      TileL12 x;
      tile_l12(a, w2, a.table + (size_t)(tj * a.ntypes + ti) * kTrN1, pt.s, lane, g, x);
      floatx4 z[4], zd[4];
      tile_l3(a, w3, sG, lane, r, g, x, z, zd);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        floatx4 gv, gd;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float th = tanh_fast(z[t][v]);
          gv[v] = th + x.h2[t & 1][v];
          gd[v] = (1.0f - th * th) * zd[t][v] + x.h2d[t & 1][v];
        }
        *(floatx4 *)(sG + r * kTrRow + 16 * t + 4 * g) = gv;
        *(floatx4 *)(sGp + r * kTrRow + 16 * t + 4 * g) = gd;
      }
      if (g == 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          sC[r * 8 + c] = pt.Rd[c] * a.inv_sel;
          sC[r * 8 + 4 + c] = pt.Rt[c] * pt.sdot * a.inv_sel;
        }
      }
      wave_fence();
      const int cnt = min(16, n - p0);
      for (int pp = 0; pp < cnt; ++pp) {
        const float gv = sG[pp * kTrRow + lane], gd = sGp[pp * kTrRow + lane];
#pragma unroll
        for (int c = 0; c < 4; ++c)
          tacc[c] = fmaf(sC[pp * 8 + c], gv, fmaf(sC[pp * 8 + 4 + c], gd, tacc[c]));
      }
      wave_fence();
    }
    // D-dot from T-dot and T (lane = m)
    float tv[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      tv[c] = a.T[((size_t)i * 4 + c) * kTrN3 + lane];
      sG[c * 64 + lane] = tv[c];
      sG[256 + c * 64 + lane] = tacc[c];
      Td[((size_t)i * 4 + c) * kTrN3 + lane] = tacc[c];
    }
    wave_fence();
    float *xp = Xd + (size_t)i * ldD + (size_t)lane * a.axis;
    for (int ax = 0; ax < a.axis; ++ax) {
      float v = 0.f;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        v = fmaf(tacc[c], sG[c * 64 + ax], fmaf(tv[c], sG[256 + c * 64 + ax], v));
      xp[ax] = v;
    }
    wave_fence();
  }
}

// ------------------------------------------------------------ fitting steps

// Top fitting layer (identity residual): y2 = t2 + y1, y2-dot = g2 z2-dot + y1-dot,
// seeds y2-bar = a w, y2-dot-bar = -w.  Writes z2-bar (rows [0, nloc)),
// z2-dot-bar (rows [nloc, 2 nloc)) and a y2 - y2-dot (for w_out).
__global__ void k_tr_fit_top(const float *__restrict__ t2, const float *__restrict__ y2,
                             const float *__restrict__ yd1, const float *__restrict__ zd2,
                             const float *__restrict__ w_out, const float *__restrict__ a,
                             int nloc, int H, int ld, float *__restrict__ zb2,
                             float *__restrict__ wo_rows) {
  const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= (size_t)nloc * ld) return;
  const int o = (int)(k % ld);
  const float av = a[0];
  if (o >= H) {
    zb2[k] = 0.f;
    zb2[k + (size_t)nloc * ld] = 0.f;
    wo_rows[k] = 0.f;
    return;
  }
  const float t = t2[k], g = 1.0f - t * t, w = w_out[o], zd = zd2[k];
  const float yd2 = fmaf(g, zd, yd1[k]);
  zb2[k] = g * (av * w + 2.0f * t * zd * w);
  zb2[k + (size_t)nloc * ld] = -g * w;
  wo_rows[k] = av * y2[k] - yd2;
}

// First fitting layer (tanh, no residual): from y1-bar = yb1 + a w and
// y1-dot-bar = yb1' - w (the residual seeds of the top layer).
__global__ void k_tr_fit_l0(const float *__restrict__ t1, const float *__restrict__ zd1,
                            const float *__restrict__ yb1, const float *__restrict__ w_out,
                            const float *__restrict__ a, int nloc, int H, int ld,
                            float *__restrict__ zb1) {
  const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= (size_t)nloc * ld) return;
  const int o = (int)(k % ld);
  if (o >= H) {
    zb1[k] = 0.f;
    zb1[k + (size_t)nloc * ld] = 0.f;
    return;
  }
  const float w = w_out[o];
  const float t = t1[k], g = 1.0f - t * t;
  const float ybar = yb1[k] + a[0] * w;
  const float ydbar = yb1[k + (size_t)nloc * ld] - w;
  const float gbar = zd1[k] * ydbar;
  zb1[k] = g * (ybar - 2.0f * t * gbar);
  zb1[k + (size_t)nloc * ld] = g * ydbar;
}

// ------------------------------------------------------------- pair reverse

// Element of feature 0 of pair row q in a weight-gradient operand of nf
// features: blocks of 16 rows, feature by feature inside a block.  A tile's
// stores then fall into one or two blocks of contiguous memory; one row per
// feature over all pairs (320 streams a tile, 64 bytes at a time) bound the
// writer: 1372 us a frame at 15,668 atoms, this order 1058 us.
__device__ __forceinline__ unsigned tr_row(unsigned q, int nf) {
  return (q >> 4) * (unsigned)(16 * nf) + (q & 15u);
}

// One wavefront per centre.  Lanes over m form T-bar and T-dot-bar from D-bar
// and D-dot-bar (reverse of D = T^T T<, D-dot = T-dot^T T< + T^T T-dot<); per
// tile of 16 pairs follow G-bar = (1/sel)(R~ T-bar + R~-dot T-dot-bar) and
// G'-bar = (1/sel) s-dot R~ T-dot-bar, and the reverse of the embedding net and
// of its s-derivative down to the first layer, writing the rows of the weight
// gradients.  Every sum is a matrix-core chain in the order of its scalar form:
// the terms of G-bar alternate R~-dot T-dot-bar and R~ T-bar over c, the [h2, h2]
// and [h1, h1] residuals enter where the loop over outputs adds them (the
// latter as unit-weight depths between the outputs' own).
constexpr int kTrRevWave = 2 * 64 * 16 + 2 * 4 * 64;  // D-bar, D-dot-bar, T, T-dot; tiles
static_assert(kTrRevWave >= 2 * kTrTile, "two 16 x 64 tiles share the space");
constexpr size_t kTrRevLds =
    sizeof(float) * (kTrW2 + kTrW3 + kTrW3r + kTrW2r + kTrWaves * kTrRevWave);

__global__ __launch_bounds__(64 * kTrWaves, 3) void k_tr_pair_rev(
    TrainPairArgs a, const float4 *__restrict__ delta, const float *__restrict__ Td,
    const float *__restrict__ Db, int ldD, size_t Pcap, float *__restrict__ X3,
    float *__restrict__ Z3, float *__restrict__ X2, float *__restrict__ Z2,
    float *__restrict__ Z1, float *__restrict__ WS1, int *__restrict__ grp) {
  extern __shared__ float4 smem[];
  float *w2 = (float *)smem, *w3 = w2 + kTrW2, *w3r = w3 + kTrW3, *w2r = w3r + kTrW3r;
  stage_forward_weights(a, w2, w3);
  for (int e = threadIdx.x; e < kTrW3r; e += 64 * kTrWaves) {
    const int l = e & 63, c = (e >> 6) & 15, t = e >> 10;
    w3r[e] = a.W3t[(4 * c + (l >> 4)) * kTrN2 + 16 * t + (l & 15)];
  }
  for (int e = threadIdx.x; e < kTrW2r; e += 64 * kTrWaves) {
    // depth 4 c + g: output o = 2 c + g / 2, its weight (g even) or the residual
    const int l = e & 63, c = e >> 6, q = l >> 4, o = 2 * c + (q >> 1), k = l & 15;
    w2r[e] = (q & 1) ? (k == o % kTrN1 ? 1.f : 0.f) : a.W2t[o * kTrN1 + k];
  }
  __syncthreads();
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  float *sDb = w2r + kTrW2r + w * kTrRevWave, *sDdb = sDb + 64 * 16;
  float *sT = sDdb + 64 * 16, *sTd = sT + 4 * 64;
  float *ta = sDb, *tb_ = ta + kTrTile;  // the tiles' turns through LDS
  const int ax = a.axis;
  const unsigned pc32 = (unsigned)Pcap;
  const floatx4 wsv = *(const floatx4 *)(a.ws + 4 * g);
  for (int i = w * (int)gridDim.x + blockIdx.x; i < a.nloc; i += kTrWaves * gridDim.x) {
    const int n = a.nnei[i];
    const int off = a.pair_off[i];
    const int ti = a.types[i];
    const float4 di = delta[i];
    // --- T-bar, T-dot-bar (lane = m)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      sT[c * 64 + lane] = a.T[((size_t)i * 4 + c) * kTrN3 + lane];
      sTd[c * 64 + lane] = Td[((size_t)i * 4 + c) * kTrN3 + lane];
    }
    for (int b = 0; b < ax; ++b) {
      sDb[lane * 16 + b] = Db[(size_t)i * ldD + (size_t)lane * ax + b];
      sDdb[lane * 16 + b] = Db[(size_t)(a.nloc + i) * ldD + (size_t)lane * ax + b];
    }
    wave_fence();
    float tb[4] = {0.f, 0.f, 0.f, 0.f}, tdb[4] = {0.f, 0.f, 0.f, 0.f};
    for (int b = 0; b < ax; ++b) {
      const float db = sDb[lane * 16 + b], ddb = sDdb[lane * 16 + b];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        tb[c] = fmaf(db, sT[c * 64 + b], fmaf(ddb, sTd[c * 64 + b], tb[c]));
        tdb[c] = fmaf(ddb, sT[c * 64 + b], tdb[c]);
      }
    }
    if (lane < ax) {
#pragma unroll 4
      for (int mp = 0; mp < kTrN3; ++mp) {
        const float db = sDb[mp * 16 + lane], ddb = sDdb[mp * 16 + lane];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          tb[c] = fmaf(db, sT[c * 64 + mp], fmaf(ddb, sTd[c * 64 + mp], tb[c]));
          tdb[c] = fmaf(ddb, sT[c * 64 + mp], tdb[c]);
        }
      }
    }
    wave_fence();
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      sT[c * 64 + lane] = tb[c] * a.inv_sel;   // T-bar, T-dot-bar
      sTd[c * 64 + lane] = tdb[c] * a.inv_sel;
    }
    wave_fence();
    // row operands of G-bar (depths T-dot-bar_c, T-bar_c in turn) and G'-bar
    float ag[4][2], agd[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int c = 2 * h + (g >> 1);
        ag[t][h] = ((g & 1) ? sT : sTd)[c * 64 + 16 * t + r];
      }
      agd[t] = sTd[g * 64 + 16 * t + r];
    }
    wave_fence();
    // --- pairs
    for (int p0 = 0; p0 < n; p0 += 16) {
      const bool valid = p0 + r < n;
      const int pc = valid ? p0 + r : 0;
      const float4 *gp = (const float4 *)(a.geom + (size_t)(off + pc) * kGeom);
      const float4 g0 = gp[0], g1 = gp[1];
      const int j = a.nlist[(size_t)i * a.sel + pc];
      const int tj = a.types[j];
      const float4 dj = delta[j];
      const PairTangent pt = pair_tangent(g0, g1, di, dj);
      const unsigned q = (unsigned)(off + pc);
      // this lane's places in the operands (tr_row), from output 4 g on
      float *x3 = X3 + tr_row(q, kTrN2) + 64 * g, *z3 = Z3 + tr_row(q, kTrN3) + 64 * g;
      float *x2 = X2 + tr_row(q, kTrN1) + 64 * g, *z2 = Z2 + tr_row(q, kTrN2) + 64 * g;
      TileL12 x;
      tile_l12(a, w2, a.table + (size_t)(tj * a.ntypes + ti) * kTrN1, pt.s, lane, g, x);
      if (valid) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          x2[16 * v] = x.h1[v];
          x2[16 * v + pc32 * kTrN1] = x.h1d[v];
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            x3[16 * (16 * t + v)] = x.h2[t][v];
            x3[16 * (16 * t + v) + pc32 * kTrN2] = x.h2d[t][v];
          }
      }
      floatx4 z[4], zd[4];
      tile_l3(a, w3, ta, lane, r, g, x, z, zd);
      // G-bar, G'-bar of the tile's outputs
      float bg[2], bgd;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float lo = (g & 1) ? pt.Rt[2 * h] : pt.Rd[2 * h];
        const float hi = (g & 1) ? pt.Rt[2 * h + 1] : pt.Rd[2 * h + 1];
        bg[h] = (g & 2) ? hi : lo;
      }
      bgd = (g & 2) ? ((g & 1) ? pt.Rt[3] : pt.Rt[2]) : ((g & 1) ? pt.Rt[1] : pt.Rt[0]);
      const floatx4 zero = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const floatx4 Gb = mfma4(ag[t][1], bg[1], mfma4(ag[t][0], bg[0], zero));
        const floatx4 Gd = mfma4(agd[t], bgd, zero);
        floatx4 zb, zbd;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float Gdb = Gd[v] * pt.sdot;
          const float th = tanh_fast(z[t][v]), gg = 1.0f - th * th;
          zbd[v] = gg * Gdb;
          zb[v] = gg * (Gb[v] - 2.0f * th * zd[t][v] * Gdb);
        }
        *(floatx4 *)(ta + r * kTrRow + 16 * t + 4 * g) = zb;
        *(floatx4 *)(tb_ + r * kTrRow + 16 * t + 4 * g) = zbd;
        if (valid) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            z3[16 * (16 * t + v)] = zb[v];
            z3[16 * (16 * t + v) + pc32 * kTrN3] = zbd[v];
          }
        }
      }
      wave_fence();
      // h2-bar, h2'-bar: W3 z3-bar, then the [h2, h2] residual (G-bar[k] and
      // G-bar[k + 32] both feed h2[k])
      floatx4 hb[2], hbd[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) hb[t] = hbd[t] = zero;
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        const float b0 = ta[r * kTrRow + 4 * c + g], b1 = tb_[r * kTrRow + 4 * c + g];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const float wv = w3r[(t * 16 + c) * 64 + lane];
          hb[t] = mfma4(wv, b0, hb[t]);
          hbd[t] = mfma4(wv, b1, hbd[t]);
        }
      }
      wave_fence();
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        floatx4 gb = zero, gdb = zero;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          gb = mfma4(ag[t + 2 * hh][0], bg[0], gb);
          gb = mfma4(ag[t + 2 * hh][1], bg[1], gb);
          gdb = mfma4(agd[t + 2 * hh], bgd, gdb);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          hb[t][v] += gb[v];
          hbd[t][v] = fmaf(gdb[v], pt.sdot, hbd[t][v]);
        }
      }
      // second layer in reverse: rows of outputs and their residual gradients
      // in turn
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        floatx4 zb, zbd;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float th = x.t2[t][v], gg = 1.0f - th * th;
          zbd[v] = gg * hbd[t][v];
          zb[v] = gg * (hb[t][v] - 2.0f * th * x.zd2[t][v] * hbd[t][v]);
        }
        float *pa = ta + r * kTrRow + 2 * (16 * t + 4 * g);
        float *pb = tb_ + r * kTrRow + 2 * (16 * t + 4 * g);
        *(floatx4 *)pa = floatx4{zb[0], hb[t][0], zb[1], hb[t][1]};
        *(floatx4 *)(pa + 4) = floatx4{zb[2], hb[t][2], zb[3], hb[t][3]};
        *(floatx4 *)pb = floatx4{zbd[0], hbd[t][0], zbd[1], hbd[t][1]};
        *(floatx4 *)(pb + 4) = floatx4{zbd[2], hbd[t][2], zbd[3], hbd[t][3]};
        if (valid) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            z2[16 * (16 * t + v)] = zb[v];
            z2[16 * (16 * t + v) + pc32 * kTrN2] = zbd[v];
          }
        }
      }
      wave_fence();
      floatx4 hb1 = zero, hb1d = zero;
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        const float wv = w2r[c * 64 + lane];
        hb1 = mfma4(wv, ta[r * kTrRow + 4 * c + g], hb1);
        hb1d = mfma4(wv, tb_[r * kTrRow + 4 * c + g], hb1d);
      }
      wave_fence();
      // first layer: h1' = (1 - h1^2) ws
      if (valid) {
        float *z1 = Z1 + tr_row(q, kTrN1) + 64 * g, *ws1 = WS1 + tr_row(q, kTrN1) + 64 * g;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float gg = 1.0f - x.h1[v] * x.h1[v];
          const float gbar = wsv[v] * hb1d[v];
          const float zb = gg * (hb1[v] - 2.0f * x.h1[v] * gbar);
          z1[16 * v] = zb;
          ws1[16 * v] = fmaf(pt.s, zb, gg * hb1d[v]);
        }
        if (g == 0) grp[q] = tj * a.ntypes + ti;
      }
    }
  }
}

// ------------------------------------------------------- weight gradients

// part[blk][kin_pad][nout_pad] = sum over the block's rows of X^T Z for both
// segments.  Block = 4 waves over one 16KT x 16NT output tile group; each
// wave takes every 4th group of rows, the four waves are summed in LDS.
// ONEHOT: the X operand is not read but generated, X[r][k] = (group[r] == k)
// (group == nullptr: X[r][k] = (k == 0)), so the product sums Z by group.
template <int KT, int NT, bool BF, bool ONEHOT>
__global__ __launch_bounds__(256) void k_wgrad(const float *__restrict__ X1,
                                               const float *__restrict__ X2, int ldx,
                                               const float *__restrict__ Z1,
                                               const float *__restrict__ Z2, int ldz, int kin,
                                               int nout, const int *__restrict__ rows_dev,
                                               int rows_max, int rows_per_block,
                                               const int32_t *__restrict__ group,
                                               float *__restrict__ part, int kin_pad,
                                               int nout_pad) {
  __shared__ float red[4][KT * NT * 256];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int rows = rows_dev ? min(rows_dev[0], rows_max) : rows_max;
  const int r0 = blockIdx.x * rows_per_block;
  const int r1 = min(rows, r0 + rows_per_block);
  const int k0 = blockIdx.y * 16 * KT, n0 = blockIdx.z * 16 * NT;
  floatx4 acc[KT][NT];
#pragma unroll
  for (int kt = 0; kt < KT; ++kt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[kt][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int col = lane & 15, quad = lane >> 4;
  constexpr int RG = BF ? 32 : 4;  // rows per matrix-core step
  const int nseg = (ONEHOT || X2 == nullptr) ? 1 : 2;
  for (int seg = 0; seg < nseg; ++seg) {
    const float *X = seg ? X2 : X1;
    const float *Z = seg ? Z2 : Z1;
    for (int rg = r0 + w * RG; rg < r1; rg += 4 * RG) {
      if constexpr (!BF) {
        const int r = rg + quad;
        const bool rv = r < r1;
        const size_t rr = (size_t)(rv ? r : r0);
        float xv[KT], zv[NT];
        if constexpr (ONEHOT) {
          const int gr = group ? group[rr] : 0;
#pragma unroll
          for (int kt = 0; kt < KT; ++kt) xv[kt] = (rv && gr == k0 + 16 * kt + col) ? 1.f : 0.f;
        } else {
#pragma unroll
          for (int kt = 0; kt < KT; ++kt) {
            const int c = k0 + 16 * kt + col;
            const float v = X[rr * ldx + (c < kin ? c : 0)];
            xv[kt] = (rv && c < kin) ? v : 0.f;
          }
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const int c = n0 + 16 * nt + col;
          const float v = Z[rr * ldz + (c < nout ? c : 0)];
          zv[nt] = (rv && c < nout) ? v : 0.f;
        }
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            acc[kt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[kt], zv[nt], acc[kt][nt], 0, 0, 0);
      } else {
        // 32 rows per 16x16x32 step: lane slots u < 4 hold rows rg + 4q + u,
        // slots 4 + u rows rg + 16 + 4q + u (the same rows on both operands)
        static_assert(!ONEHOT, "group sums use FP32 operands");
        floatx8 xv[KT], zv[NT];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int r = rg + 16 * (u >> 2) + 4 * quad + (u & 3);
          const bool rv = r < r1;
          const size_t rr = (size_t)(rv ? r : r0);
#pragma unroll
          for (int kt = 0; kt < KT; ++kt) {
            const int c = k0 + 16 * kt + col;
            const float v = X[rr * ldx + (c < kin ? c : 0)];
            xv[kt][u] = (rv && c < kin) ? v : 0.f;
          }
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            const int c = n0 + 16 * nt + col;
            const float v = Z[rr * ldz + (c < nout ? c : 0)];
            zv[nt][u] = (rv && c < nout) ? v : 0.f;
          }
        }
        bf16x8 xb[KT], zb[NT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) xb[kt] = __builtin_convertvector(xv[kt], bf16x8);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) zb[nt] = __builtin_convertvector(zv[nt], bf16x8);
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            acc[kt][nt] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(xb[kt], zb[nt], acc[kt][nt], 0, 0, 0);
      }
    }
  }
  // D[i][j]: register v of lane l holds i = 4 (l / 16) + v, j = l % 16
#pragma unroll
  for (int kt = 0; kt < KT; ++kt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[w][((kt * NT + nt) * 4 + v) * 64 + lane] = acc[kt][nt][v];
  __syncthreads();
  for (int e = threadIdx.x; e < KT * NT * 256; e += 256) {
    const float sum = ((red[0][e] + red[1][e]) + red[2][e]) + red[3][e];
    const int l = e & 63, v = (e >> 6) & 3, tile = e >> 8;
    const int kt = tile / NT, nt = tile % NT;
    const int ki = k0 + 16 * kt + 4 * (l >> 4) + v, nj = n0 + 16 * nt + (l & 15);
    if (ki < kin_pad && nj < nout_pad)
      part[((size_t)blockIdx.x * kin_pad + ki) * nout_pad + nj] = sum;
  }
}

// Variant for the pair operands: Xt of kin features, Zt of nout features, each
// in blocks of 16 rows, feature by feature inside a block (tr_row); segment 2
// (if seg2 > 0, a multiple of 16) starts at row seg2.  Lane (c, q) of a 16-row
// step reads rows 4q..4q+3 of feature c as one float4 (16 features' rows side by
// side), which is the k-slice layout of the BF16 product; the FP32 product
// takes the four components as four 16x16x4 steps.
__device__ __forceinline__ size_t fm_row(size_t row, int nf) {
  return (row >> 4) * (size_t)(16 * nf) + (row & 15);
}

template <int KT, int NT, bool BF, bool ONEHOT>
__global__ __launch_bounds__(256) void k_wgrad_fm(const float *__restrict__ Xt,
                                                  const float *__restrict__ Zt, size_t seg2,
                                                  int kin, int nout,
                                                  const int *__restrict__ rows_dev, int rows_max,
                                                  int rows_per_block,
                                                  const int32_t *__restrict__ group,
                                                  float *__restrict__ part, int kin_pad,
                                                  int nout_pad) {
  __shared__ float red[4][KT * NT * 256];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int rows = rows_dev ? min(rows_dev[0], rows_max) : rows_max;
  const int r0 = blockIdx.x * rows_per_block;
  const int r1 = min(rows, r0 + rows_per_block);
  const int k0 = blockIdx.y * 16 * KT, n0 = blockIdx.z * 16 * NT;
  floatx4 acc[KT][NT];
#pragma unroll
  for (int kt = 0; kt < KT; ++kt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[kt][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int col = lane & 15, quad = lane >> 4;
  const int nseg = (ONEHOT || seg2 == 0) ? 1 : 2;
  for (int seg = 0; seg < nseg; ++seg) {
    const size_t base = seg ? seg2 : 0;
    if constexpr (BF) {
      // BF16: 32 rows per gfx950 16x16x32 step; lane slots 0..3 hold rows
      // rg + 4q + 0..3 and slots 4..7 rows rg + 16 + 4q + 0..3, on both
      // operands.  A second half that starts past r1 re-reads the first
      // half's rows (masked to zero).
      static_assert(!ONEHOT, "group sums use FP32 operands");
      for (int rg = r0 + w * 32; rg < r1; rg += 128) {
        const int rq0 = rg + 4 * quad, rq1 = rq0 + 16;
        const int rq1a = rq1 < r1 ? rq1 : rq0;
        bool rv[8];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          rv[j] = rq0 + j < r1;
          rv[4 + j] = rq1 + j < r1;
        }
        floatx8 xv[KT], zv[NT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
          const int c = k0 + 16 * kt + col;
          const float *xp = Xt + 16 * (c < kin ? c : 0);
          const floatx4 v0 = *(const floatx4 *)(xp + fm_row(base + rq0, kin)),
                        v1 = *(const floatx4 *)(xp + fm_row(base + rq1a, kin));
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            xv[kt][j] = (rv[j] && c < kin) ? v0[j] : 0.f;
            xv[kt][4 + j] = (rv[4 + j] && c < kin) ? v1[j] : 0.f;
          }
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const int c = n0 + 16 * nt + col;
          const float *zp = Zt + 16 * (c < nout ? c : 0);
          const floatx4 v0 = *(const floatx4 *)(zp + fm_row(base + rq0, nout)),
                        v1 = *(const floatx4 *)(zp + fm_row(base + rq1a, nout));
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            zv[nt][j] = (rv[j] && c < nout) ? v0[j] : 0.f;
            zv[nt][4 + j] = (rv[4 + j] && c < nout) ? v1[j] : 0.f;
          }
        }
        bf16x8 xb[KT], zb[NT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) xb[kt] = __builtin_convertvector(xv[kt], bf16x8);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) zb[nt] = __builtin_convertvector(zv[nt], bf16x8);
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            acc[kt][nt] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(xb[kt], zb[nt], acc[kt][nt], 0, 0, 0);
      }
      continue;
    }
    for (int rg = r0 + w * 16; rg < r1; rg += 64) {
      const int rq = rg + 4 * quad;
      bool rv[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) rv[j] = rq + j < r1;
      floatx4 xv[KT], zv[NT];
      if constexpr (ONEHOT) {
        const int4 gq = group ? *(const int4 *)(group + rq) : make_int4(0, 0, 0, 0);
        const int gg[4] = {gq.x, gq.y, gq.z, gq.w};
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
          for (int j = 0; j < 4; ++j) xv[kt][j] = (rv[j] && gg[j] == k0 + 16 * kt + col) ? 1.f : 0.f;
      } else {
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
          const int c = k0 + 16 * kt + col;
          const floatx4 v =
              *(const floatx4 *)(Xt + fm_row(base + rq, kin) + 16 * (c < kin ? c : 0));
#pragma unroll
          for (int j = 0; j < 4; ++j) xv[kt][j] = (rv[j] && c < kin) ? v[j] : 0.f;
        }
      }
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int c = n0 + 16 * nt + col;
        const floatx4 v =
            *(const floatx4 *)(Zt + fm_row(base + rq, nout) + 16 * (c < nout ? c : 0));
#pragma unroll
        for (int j = 0; j < 4; ++j) zv[nt][j] = (rv[j] && c < nout) ? v[j] : 0.f;
      }
      {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
              acc[kt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[kt][j], zv[nt][j],
                                                                  acc[kt][nt], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int kt = 0; kt < KT; ++kt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[w][((kt * NT + nt) * 4 + v) * 64 + lane] = acc[kt][nt][v];
  __syncthreads();
  for (int e = threadIdx.x; e < KT * NT * 256; e += 256) {
    const float sum = ((red[0][e] + red[1][e]) + red[2][e]) + red[3][e];
    const int l = e & 63, v = (e >> 6) & 3, tile = e >> 8;
    const int kt = tile / NT, nt = tile % NT;
    const int ki = k0 + 16 * kt + 4 * (l >> 4) + v, nj = n0 + 16 * nt + (l & 15);
    if (ki < kin_pad && nj < nout_pad)
      part[((size_t)blockIdx.x * kin_pad + ki) * nout_pad + nj] = sum;
  }
}

// acc[k][n] += sum_b part[b][k][n] in a fixed order: thread (slice, e) sums
// the blocks b = slice (mod 16) of output e in FP64, then the 16 slices are
// added in slice order.
__global__ __launch_bounds__(256) void k_reduce_parts(const float *__restrict__ part, int nblk,
                                                      int kin_pad, int nout_pad, int kin,
                                                      int nout, double *__restrict__ acc) {
  __shared__ double red[16][16];
  const int el = threadIdx.x & 15, sl = threadIdx.x >> 4;
  const int e = blockIdx.x * 16 + el;
  const bool ok = e < kin * nout;
  const int k = ok ? e / nout : 0, n = ok ? e % nout : 0;
  double s = 0.0;
  for (int b = sl; b < nblk; b += 16) s += (double)part[((size_t)b * kin_pad + k) * nout_pad + n];
  red[sl][el] = s;
  __syncthreads();
  if (sl == 0 && ok) {
    double t = 0.0;
    for (int q = 0; q < 16; ++q) t += red[q][el];
    acc[e] += t;
  }
}

// --------------------------------------------------------------------- Adam

__global__ void k_adam(float *__restrict__ theta, float *__restrict__ m, float *__restrict__ v,
                       const double *__restrict__ g, int n, float lr, float b1, float b2,
                       float eps, float bc1, float bc2) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const float gk = (float)g[k];
  const float mk = b1 * m[k] + (1.0f - b1) * gk;
  const float vk = b2 * v[k] + (1.0f - b2) * gk * gk;
  m[k] = mk;
  v[k] = vk;
  theta[k] -= lr * (mk / bc1) / (sqrtf(vk / bc2) + eps);
}

__global__ void k_fill_f64(double *p, size_t n) {
  const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) p[k] = 0.0;
}

__global__ __launch_bounds__(256) void k_force_error(const double *__restrict__ a,
                                                     const double *__restrict__ b, int n,
                                                     double *__restrict__ part) {
  __shared__ double ss[256], mx[256];
  double sq = 0.0, m = 0.0;
  for (int k = blockIdx.x * 256 + threadIdx.x; k < 3 * n; k += gridDim.x * 256) {
    const double d = a[k] - b[k];
    sq += d * d;
    m = fmax(m, fabs(d));
  }
  ss[threadIdx.x] = sq;
  mx[threadIdx.x] = m;
  __syncthreads();
  for (int h = 128; h >= 1; h >>= 1) {
    if ((int)threadIdx.x < h) {
      ss[threadIdx.x] += ss[threadIdx.x + h];
      mx[threadIdx.x] = fmax(mx[threadIdx.x], mx[threadIdx.x + h]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = ss[0];
    part[2 * blockIdx.x + 1] = mx[0];
  }
}

inline unsigned nblk(size_t n, int b) { return (unsigned)((n + b - 1) / b); }

template <int KT, int NT, bool ONEHOT>
void wgrad_t(const float *X1, const float *X2, int ldx, const float *Z1, const float *Z2, int ldz,
             int kin, int nout, const int *rows_dev, int rows_max, int bf16,
             const int32_t *group, float *part, size_t part_cap, double *acc, hipStream_t s) {
  const int kin_pad = (kin + 15) / 16 * 16, nout_pad = (nout + 15) / 16 * 16;
  const int gy = (kin + 16 * KT - 1) / (16 * KT), gz = (nout + 16 * NT - 1) / (16 * NT);
  const size_t per = (size_t)kin_pad * nout_pad;
  // about two row blocks per compute unit, each a multiple of 64 rows
  int rpb = std::max(1024, (rows_max + 511) / 512);
  rpb = (rpb + 63) / 64 * 64;
  while ((size_t)((rows_max + rpb - 1) / rpb) * per > part_cap) rpb *= 2;
  const int gx = std::max(1, (rows_max + rpb - 1) / rpb);
  const dim3 grid(gx, gy, gz);
  if (bf16 && !ONEHOT)
    hipLaunchKernelGGL((k_wgrad<KT, NT, true, false>), grid, dim3(256), 0, s, X1, X2, ldx, Z1, Z2,
                       ldz, kin, nout, rows_dev, rows_max, rpb, group, part, kin_pad, nout_pad);
  else
    hipLaunchKernelGGL((k_wgrad<KT, NT, false, ONEHOT>), grid, dim3(256), 0, s, X1, X2, ldx, Z1,
                       Z2, ldz, kin, nout, rows_dev, rows_max, rpb, group, part, kin_pad,
                       nout_pad);
  hipLaunchKernelGGL(k_reduce_parts, dim3(nblk((size_t)kin * nout, 16)), dim3(256), 0, s, part,
                     gx, kin_pad, nout_pad, kin, nout, acc);
}

template <int KT, int NT, bool ONEHOT>
void wgrad_fm_t(const float *Xt, const float *Zt, size_t seg2, int kin, int nout,
                const int *rows_dev, int rows_max, int bf16, const int32_t *group, float *part,
                size_t part_cap, double *acc, hipStream_t s) {
  const int kin_pad = (kin + 15) / 16 * 16, nout_pad = (nout + 15) / 16 * 16;
  const int gy = (kin + 16 * KT - 1) / (16 * KT), gz = (nout + 16 * NT - 1) / (16 * NT);
  const size_t per = (size_t)kin_pad * nout_pad;
  // row blocks of a multiple of 64 rows, about four per compute unit
  int rpb = std::max(512, (rows_max + 1023) / 1024);
  rpb = (rpb + 63) / 64 * 64;
  while ((size_t)((rows_max + rpb - 1) / rpb) * per > part_cap) rpb *= 2;
  const int gx = std::max(1, (rows_max + rpb - 1) / rpb);
  const dim3 grid(gx, gy, gz);
  if (bf16 && !ONEHOT)
    hipLaunchKernelGGL((k_wgrad_fm<KT, NT, true, false>), grid, dim3(256), 0, s, Xt, Zt,
                       seg2, kin, nout, rows_dev, rows_max, rpb, group, part, kin_pad, nout_pad);
  else
    hipLaunchKernelGGL((k_wgrad_fm<KT, NT, false, ONEHOT>), grid, dim3(256), 0, s, Xt, Zt,
                       seg2, kin, nout, rows_dev, rows_max, rpb, group, part, kin_pad, nout_pad);
  hipLaunchKernelGGL(k_reduce_parts, dim3(nblk((size_t)kin * nout, 16)), dim3(256), 0, s, part,
                     gx, kin_pad, nout_pad, kin, nout, acc);
}

}  // namespace

int tr_seed_blocks(int n) { return (int)nblk(std::max(n, 1), 256); }

void launch_tr_seed(const double *F, const double *Flab, int n, float cf, float4 *delta,
                    double *sq_part, hipStream_t s) {
  hipLaunchKernelGGL(k_tr_seed, dim3(tr_seed_blocks(n)), dim3(256), 0, s, F, Flab, n, cf, delta,
                     sq_part);
}

void launch_tr_energy_seed(const double *E, const double *Elab, double ca, double cl, float *a,
                           double *le, hipStream_t s) {
  hipLaunchKernelGGL(k_tr_energy_seed, dim3(1), dim3(64), 0, s, E, Elab, ca, cl, a, le);
}

namespace {

// Persistent grid of a per-centre kernel of kTrWaves wavefronts: one workgroup
// per CU (by LDS and registers), its dynamic LDS limit raised at the first
// launch on a device.
template <class K, class... A>
hipError_t launch_per_centre(K kernel, size_t lds, int (&ready)[64], int nloc, hipStream_t s,
                             A... args) {
  int dev = 0, cus = 256;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess)
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess && (dev < 0 || dev >= 64 || !ready[dev])) {
    e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds);
    if (e == hipSuccess && dev >= 0 && dev < 64) ready[dev] = 1;
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3(std::min(nloc, cus)), dim3(64 * kTrWaves), lds, s, args...);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_tr_tangent(const TrainPairArgs &a, const float4 *delta, float *Td, float *Xd,
                             int ldD, hipStream_t s) {
  if (a.nloc <= 0) return hipSuccess;
  static int ready[64];
  return launch_per_centre(k_tr_tangent, kTrTanLds, ready, a.nloc, s, a, delta, Td, Xd, ldD);
}

void launch_tr_fit_top(const float *t2, const float *y2, const float *yd1, const float *zd2,
                       const float *w_out, const float *a, int nloc, int H, int ld, float *zb2,
                       float *wo_rows, hipStream_t s) {
  const size_t n = (size_t)nloc * ld;
  if (!n) return;
  hipLaunchKernelGGL(k_tr_fit_top, dim3(nblk(n, 256)), dim3(256), 0, s, t2, y2, yd1, zd2, w_out,
                     a, nloc, H, ld, zb2, wo_rows);
}

void launch_tr_fit_l0(const float *t1, const float *zd1, const float *yb1, const float *w_out,
                      const float *a, int nloc, int H, int ld, float *zb1, hipStream_t s) {
  const size_t n = (size_t)nloc * ld;
  if (!n) return;
  hipLaunchKernelGGL(k_tr_fit_l0, dim3(nblk(n, 256)), dim3(256), 0, s, t1, zd1, yb1, w_out, a,
                     nloc, H, ld, zb1);
}

hipError_t launch_tr_pair_rev(const TrainPairArgs &a, const float4 *delta, const float *Td,
                              const float *Db, int ldD, size_t Pcap, float *X3,
                              float *Z3, float *X2, float *Z2, float *Z1, float *WS1, int *grp,
                              hipStream_t s) {
  if (a.nloc <= 0) return hipSuccess;
  static int ready[64];
  return launch_per_centre(k_tr_pair_rev, kTrRevLds, ready, a.nloc, s, a, delta, Td, Db, ldD, Pcap,
                           X3, Z3, X2, Z2, Z1, WS1, grp);
}

void tr_wgrad(const float *X1, const float *X2, int ldx, const float *Z1, const float *Z2, int ldz,
              int kin, int nout, const int *rows_dev, int rows_max, int bf16, float *part,
              size_t part_cap, double *acc, hipStream_t s) {
  if (rows_max <= 0) return;
  if (kin <= 16 && nout <= 32)
    wgrad_t<1, 2, false>(X1, X2, ldx, Z1, Z2, ldz, kin, nout, rows_dev, rows_max, bf16, nullptr,
                         part, part_cap, acc, s);
  else if (kin <= 32 && nout <= 64)
    wgrad_t<2, 4, false>(X1, X2, ldx, Z1, Z2, ldz, kin, nout, rows_dev, rows_max, bf16, nullptr,
                         part, part_cap, acc, s);
  else
    wgrad_t<4, 4, false>(X1, X2, ldx, Z1, Z2, ldz, kin, nout, rows_dev, rows_max, bf16, nullptr,
                         part, part_cap, acc, s);
}

void tr_wgrad_fm(const float *Xt, const float *Zt, size_t seg2, int kin, int nout,
                 const int *rows_dev, int rows_max, int bf16, float *part, size_t part_cap,
                 double *acc, hipStream_t s) {
  if (rows_max <= 0) return;
  if (kin <= 16 && nout <= 32)
    wgrad_fm_t<1, 2, false>(Xt, Zt, seg2, kin, nout, rows_dev, rows_max, bf16, nullptr,
                            part, part_cap, acc, s);
  else
    wgrad_fm_t<2, 4, false>(Xt, Zt, seg2, kin, nout, rows_dev, rows_max, bf16, nullptr,
                            part, part_cap, acc, s);
}

void tr_colsum_fm(const float *Zt, int ncol, const int *rows_dev, int rows_max,
                  const int32_t *group, int ngroups, float *part, size_t part_cap, double *acc,
                  hipStream_t s) {
  if (rows_max <= 0) return;
  if (ngroups <= 16)
    wgrad_fm_t<1, 4, true>(nullptr, Zt, 0, ngroups, ncol, rows_dev, rows_max, 0, group, part,
                           part_cap, acc, s);
  else
    wgrad_fm_t<4, 4, true>(nullptr, Zt, 0, ngroups, ncol, rows_dev, rows_max, 0, group, part,
                           part_cap, acc, s);
}

void tr_colsum(const float *Z, int ldz, int ncol, const int *rows_dev, int rows_max,
               const int32_t *group, int ngroups, float *part, size_t part_cap, double *acc,
               hipStream_t s) {
  if (rows_max <= 0) return;
  if (ngroups <= 16)
    wgrad_t<1, 4, true>(nullptr, nullptr, 0, Z, nullptr, ldz, ngroups, ncol, rows_dev, rows_max,
                        0, group, part, part_cap, acc, s);
  else
    wgrad_t<4, 4, true>(nullptr, nullptr, 0, Z, nullptr, ldz, ngroups, ncol, rows_dev, rows_max,
                        0, group, part, part_cap, acc, s);
}

void launch_adam(float *theta, float *m, float *v, const double *g, int n, float lr, float b1,
                 float b2, float eps, float bc1, float bc2, hipStream_t s) {
  hipLaunchKernelGGL(k_adam, dim3(nblk(n, 256)), dim3(256), 0, s, theta, m, v, g, n, lr, b1, b2,
                     eps, bc1, bc2);
}

int force_error_blocks(int n) { return (int)std::min<unsigned>(256, nblk(3 * (size_t)std::max(n, 1), 256)); }

void launch_force_error(const double *a, const double *b, int n, double *part, hipStream_t s) {
  hipLaunchKernelGGL(k_force_error, dim3(force_error_blocks(n)), dim3(256), 0, s, a, b, n, part);
}

void launch_fill_f64(double *p, size_t n, hipStream_t s) {
  if (n) hipLaunchKernelGGL(k_fill_f64, dim3(nblk(n, 256)), dim3(256), 0, s, p, n);
}

}  // namespace dpa1
