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
// bit, a chain of fused multiply-adds over its four depths in order (the
// gradients kept the bits that scalar loops had given them), so a product over
// ascending depth started from the bias gives the bits of the scalar loop
// z = fma(w[k], h[k], z), at twice the vector unit's rate and without a scalar
// weight load per use.  With weights as the row operand a lane receives, for pair
// r = lane % 16, outputs 16 t + 4 g + {0..3} (g = lane / 16) of tile t; as the
// column operand of the next product it has to hold depth 4 c + g in step c,
// which a turn through wave-private LDS arranges (rows of 68 or 36 floats: no
// bank conflicts).  Weights sit in LDS in the order of the steps: 64 lanes'
// values side by side.
//
// One lane per pair with scalar weights left a third of the lanes idle (84
// neighbours in two chunks of 64) and, at 256 registers and more, one wavefront
// per SIMD.  Per frame at 15,668 atoms: tangents 753 -> 248 us, adjoints
// 1304 + 325 (a second kernel for the first two layers) -> 616 us; at 192 atoms
// 58 -> 26 and 85 + 18 -> 40 us.  The adjoints write 1.7 GB of weight-gradient
// operands (330 us at the rate of a large copy), one row per pair: with one row
// per feature (320 streams, 64 bytes at a time) they took 1372 us.

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
      const size_t q = (size_t)(off + p0);  // the tile's first operand row
      const int row1 = r * kTrN1 + 4 * g, row2 = r * kTrN2 + 4 * g, row3 = r * kTrN3 + 4 * g;
      TileL12 x;
      tile_l12(a, w2, a.table + (size_t)(tj * a.ntypes + ti) * kTrN1, pt.s, lane, g, x);
      if (valid) {
        float *x2 = X2 + q * kTrN1, *x3 = X3 + q * kTrN2;
        *(floatx4 *)(x2 + row1) = x.h1;
        *(floatx4 *)(x2 + Pcap * kTrN1 + row1) = x.h1d;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          *(floatx4 *)(x3 + row2 + 16 * t) = x.h2[t];
          *(floatx4 *)(x3 + Pcap * kTrN2 + row2 + 16 * t) = x.h2d[t];
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
          float *z3 = Z3 + q * kTrN3 + 16 * t;
          *(floatx4 *)(z3 + row3) = zb;
          *(floatx4 *)(z3 + Pcap * kTrN3 + row3) = zbd;
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
          float *z2 = Z2 + q * kTrN2 + 16 * t;
          *(floatx4 *)(z2 + row2) = zb;
          *(floatx4 *)(z2 + Pcap * kTrN2 + row2) = zbd;
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
        floatx4 z1, ws1;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float gg = 1.0f - x.h1[v] * x.h1[v];
          const float gbar = wsv[v] * hb1d[v];
          z1[v] = gg * (hb1[v] - 2.0f * x.h1[v] * gbar);
          ws1[v] = fmaf(pt.s, z1[v], gg * hb1d[v]);
        }
        *(floatx4 *)(Z1 + q * kTrN1 + row1) = z1;
        *(floatx4 *)(WS1 + q * kTrN1 + row1) = ws1;
        if (g == 0) grp[q + r] = tj * a.ntypes + ti;
      }
    }
  }
}

// ------------------------------------------------------- weight gradients

// acc[k][n] += sum over rows of X[r][k] Z[r][n], for all the products of a
// frame in one launch: blocks of rows of every product first, their partials
// summed in FP64 by a second.  A product's own launch left the chip idle: a
// dozen products of 4 to 45 us each at 192 atoms, and the two of the fitting net
// (240 x 240 and smaller, 16 blocks of rows) waited for one 4-byte load per value
// in turn, 266 us each at 15,668 atoms.  All products and sums of a frame: 390 ->
// 25 us at 192 atoms (FP32), 1430 -> 460 us at 15,668 (BF16), where 2.2 GB of
// operands are read (440 us at the rate of a large copy).
//
// A workgroup takes one block of rows and one 16 KT x 16 NT tile of outputs; its
// four wavefronts share the rows, and their sums are added in LDS.  Lane (col,
// quad) holds the outputs KT col .. KT col + KT - 1 (NT col .. for Z), so a row
// of an operand tile is one contiguous load over 16 lanes; all loads of a step
// are issued before its products (FP32: those of the next step).
//
// One step is 64 rows of the workgroup on FP32 operands: four matrix-core steps
// j of the four rows of a wavefront's quads, 4 w + 16 j + quad, or for the pair
// operands (pair_rows) 16 w + 4 quad + j.  On BF16 operands it is 128 rows, 32 a
// wavefront, lane slots u < 4 rows 4 quad + u and slots 4 + u rows
// 16 + 4 quad + u on both sides.  Rows past the block's last one count as zero.
//
// ONEHOT: the X operand is not read but generated, X[r][k] = (group[r] == k)
// (group == nullptr: X[r][k] = (k == 0)), so the product sums Z by group; always
// on FP32 operands.
constexpr int kWgTile = 257;  // a 16 x 16 tile of the shared sums, off the bank period
constexpr int kWgRed = 4 * 8 * kWgTile;

template <int N> struct FloatVec { typedef float __attribute__((ext_vector_type(N))) type; };
template <> struct FloatVec<1> { typedef float type; };

template <int N>
__device__ __forceinline__ void load_cols(const float *p, float (&v)[N]) {
  const typename FloatVec<N>::type x = *(const typename FloatVec<N>::type *)p;
  if constexpr (N == 1) {
    v[0] = x;
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = x[i];
  }
}

template <int KT, int NT, bool BF, bool ONEHOT>
__device__ __forceinline__ void wgrad_tile(const TrWgradJob &J, int bx, int by, int bz,
                                           float *part, float *red) {
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int rows = J.rows_dev ? min(J.rows_dev[0], J.rows_max) : J.rows_max;
  const int r0 = bx * J.rpb, r1 = min(rows, r0 + J.rpb);
  const int k0 = by * 16 * KT, n0 = bz * 16 * NT;
  const int col = lane & 15, quad = lane >> 4;
  const int kc = k0 + KT * col, nc = n0 + NT * col;  // this lane's first outputs
  const int xo = kc < J.kin ? kc : 0, zo = nc < J.nout ? nc : 0;
  floatx4 acc[KT][NT];
#pragma unroll
  for (int kt = 0; kt < KT; ++kt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[kt][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int nseg = (ONEHOT || J.X2 == nullptr) ? 1 : 2;
  for (int seg = 0; seg < nseg; ++seg) {
    const float *X = (seg ? J.X2 : J.X1) + xo;
    const float *Z = (seg ? J.Z2 : J.Z1) + zo;
    if constexpr (BF) {
      static_assert(!ONEHOT, "group sums use FP32 operands");
      for (int rg = r0 + 32 * w; rg < r1; rg += 128) {
        float xv[8][KT], zv[8][NT];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const size_t r = (size_t)min(rg + 16 * (u >> 2) + 4 * quad + (u & 3), r1 - 1);
          load_cols<KT>(X + r * J.ldx, xv[u]);
          load_cols<NT>(Z + r * J.ldz, zv[u]);
        }
        bf16x8 xb[KT], zb[NT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
          floatx8 f;
#pragma unroll
          for (int u = 0; u < 8; ++u)
            f[u] = (rg + 16 * (u >> 2) + 4 * quad + (u & 3) < r1 && kc + kt < J.kin) ? xv[u][kt]
                                                                                    : 0.f;
          xb[kt] = __builtin_convertvector(f, bf16x8);
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          floatx8 f;
#pragma unroll
          for (int u = 0; u < 8; ++u)
            f[u] = (rg + 16 * (u >> 2) + 4 * quad + (u & 3) < r1 && nc + nt < J.nout) ? zv[u][nt]
                                                                                     : 0.f;
          zb[nt] = __builtin_convertvector(f, bf16x8);
        }
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            acc[kt][nt] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(xb[kt], zb[nt], acc[kt][nt], 0, 0, 0);
      }
    } else {
      // the rows of the next step are on their way during the products of this one
      const int lr = J.pair_rows ? 16 * w + 4 * quad : 4 * w + quad, lj = J.pair_rows ? 1 : 16;
      float xv[2][4][KT], zv[2][4][NT];
      int gr[2][4];
      auto fetch = [&](int rg, int b) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const size_t r = (size_t)min(rg + lr + lj * j, r1 - 1);
          if constexpr (ONEHOT)
            gr[b][j] = J.group ? J.group[r] : 0;
          else
            load_cols<KT>(X + r * J.ldx, xv[b][j]);
          load_cols<NT>(Z + r * J.ldz, zv[b][j]);
        }
      };
      auto step = [&](int rg, int b) {
        fetch(rg + 64, 1 - b);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool rv = rg + lr + lj * j < r1;
          float zj[NT];
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) zj[nt] = rv && nc + nt < J.nout ? zv[b][j][nt] : 0.f;
#pragma unroll
          for (int kt = 0; kt < KT; ++kt) {
            float xj;
            if constexpr (ONEHOT)
              xj = rv && gr[b][j] == kc + kt ? 1.f : 0.f;
            else
              xj = rv && kc + kt < J.kin ? xv[b][j][kt] : 0.f;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
              acc[kt][nt] =
                  __builtin_amdgcn_mfma_f32_16x16x4f32(xj, zj[nt], acc[kt][nt], 0, 0, 0);
          }
        }
      };
      if (r0 < r1) fetch(r0, 0);
      for (int rg = r0; rg < r1; rg += 128) {
        step(rg, 0);
        if (rg + 64 < r1) step(rg + 64, 1);
      }
    }
  }
  // D[i][j]: register v of lane l holds i = 4 (l / 16) + v, j = l % 16
  constexpr int kWave = KT * NT * kWgTile;
  static_assert(4 * kWave <= kWgRed, "shared sums");
#pragma unroll
  for (int kt = 0; kt < KT; ++kt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        red[w * kWave + (kt * NT + nt) * kWgTile + v * 64 + lane] = acc[kt][nt][v];
  __syncthreads();
  const int nout_pad = (J.nout + 15) / 16 * 16;
  for (int e = threadIdx.x; e < KT * NT * 256; e += 256) {
    const int nl = e % (16 * NT), kl = e / (16 * NT);
    const int ki = k0 + kl, nj = n0 + nl, i = kl / KT;
    if (ki >= J.kin || nj >= nout_pad) continue;
    const float *q =
        red + ((kl % KT) * NT + nl % NT) * kWgTile + (i & 3) * 64 + 16 * (i >> 2) + nl / NT;
    part[J.part + ((size_t)bx * J.kin + ki) * nout_pad + nj] =
        ((q[0] + q[kWave]) + q[2 * kWave]) + q[3 * kWave];
  }
}

template <bool BF>
__global__ __launch_bounds__(256) void k_wgrads(TrWgrads B, float *__restrict__ part) {
  __shared__ float red[kWgRed];
  int n = 0;
  while (n + B.job[n].members < B.n && (int)blockIdx.x >= B.job[n + B.job[n].members].blk0)
    n += B.job[n].members;
  const int l = blockIdx.x - B.job[n].blk0, m = 8 * B.job[n].members;
  const int b = l / m * 8 + l % 8;
  const TrWgradJob &J = B.job[n + l % m / 8];
  if (b >= J.gx * J.gy * J.gz) return;
  const int bx = b % J.gx, by = b / J.gx % J.gy, bz = b / (J.gx * J.gy);
  switch (J.tile) {
    case kWgX1: wgrad_tile<1, 2, BF, false>(J, bx, by, bz, part, red); break;
    case kWgX2: wgrad_tile<2, 4, BF, false>(J, bx, by, bz, part, red); break;
    case kWgSum: wgrad_tile<1, 4, false, true>(J, bx, by, bz, part, red); break;
    default: wgrad_tile<4, 1, false, true>(J, bx, by, bz, part, red); break;
  }
}

// acc[k][n] += sum_b part[b][k][n] in a fixed order: thread (slice, e) sums
// the blocks b = slice (mod 16) of output e in FP64, then the 16 slices are
// added in slice order.
__global__ __launch_bounds__(256) void k_wgrad_sums(TrWgrads B, const float *__restrict__ part) {
  __shared__ double red[16][16];
  int q = 0;
  while (q + 1 < B.n && (int)blockIdx.x >= B.job[q + 1].sum0) ++q;
  const TrWgradJob &J = B.job[q];
  const int nout_pad = (J.nout + 15) / 16 * 16;
  const int el = threadIdx.x & 15, sl = threadIdx.x >> 4;
  const int e = ((int)blockIdx.x - J.sum0) * 16 + el;
  const bool ok = e < J.kin * J.nout;
  const int k = ok ? e / J.nout : 0, n = ok ? e % J.nout : 0;
  const float *p = part + J.part + (size_t)k * nout_pad + n;
  double s = 0.0;
#pragma unroll 8
  for (int b = sl; b < J.gx; b += 16) s += (double)p[(size_t)b * J.kin * nout_pad];
  red[sl][el] = s;
  __syncthreads();
  if (sl == 0 && ok) {
    double t = 0.0;
    for (int i = 0; i < 16; ++i) t += red[i][el];
    J.acc[e] += t;
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

void TrWgrads::add(const float *X1, const float *X2, int ldx, const float *Z1, const float *Z2,
                   int ldz, int kin, int nout, const int *rows_dev, int rows_max,
                   bool pair_rows, const int32_t *group, bool onehot, double *acc) {
  if (rows_max <= 0) return;
  TrWgradJob &J = job[n++];
  J = TrWgradJob{X1, X2, Z1, Z2, group, rows_dev, acc, ldx, ldz, kin, nout, rows_max, pair_rows};
  J.tile = onehot ? (kin <= 16 ? kWgSum : kWgSumWide) : (kin <= 16 && nout <= 32 ? kWgX1 : kWgX2);
  const int tk = J.tile == kWgX2 ? 32 : J.tile == kWgSumWide ? 64 : 16;
  const int tn = J.tile == kWgX1 ? 32 : J.tile == kWgSumWide ? 16 : 64;
  J.gy = (kin + tk - 1) / tk;
  J.gz = (nout + tn - 1) / tn;
  // blocks of rows, a multiple of 64: about four per compute unit of the pairs',
  // two of the atoms'.  They fix the order of the sums.
  const size_t per = (size_t)((kin + 15) / 16 * 16) * ((nout + 15) / 16 * 16);
  J.rpb = pair_rows ? std::max(512, (rows_max + 1023) / 1024)
                    : std::max(1024, (rows_max + 511) / 512);
  J.rpb = (J.rpb + 63) / 64 * 64;
  while ((size_t)((rows_max + J.rpb - 1) / J.rpb) * per > kTrPartMax) J.rpb *= 2;
  J.gx = std::max(1, (rows_max + J.rpb - 1) / J.rpb);
}

void TrWgrads::product(const float *X1, const float *X2, int ldx, const float *Z1,
                       const float *Z2, int ldz, int kin, int nout, const int *rows_dev,
                       int rows_max, bool pair_rows, double *acc) {
  add(X1, X2, ldx, Z1, Z2, ldz, kin, nout, rows_dev, rows_max, pair_rows, nullptr, false, acc);
}

void TrWgrads::colsum(const float *Z, int ldz, int ncol, const int *rows_dev, int rows_max,
                      bool pair_rows, const int32_t *group, int ngroups, double *acc) {
  add(nullptr, nullptr, 0, Z, nullptr, ldz, ngroups, ncol, rows_dev, rows_max, pair_rows, group,
      true, acc);
}

void TrWgrads::plan() {
  size_t floats = 0;
  int blk = 0, sum = 0;
  for (int k = 0, m = 1; k < n; ++k) {
    TrWgradJob &J = job[k];
    if (--m == 0) {  // a new group
      auto count = [](const TrWgradJob &j) { return j.gx * j.gy * j.gz; };
      while (k + m + 1 < n && J.pair_rows && job[k + m + 1].pair_rows &&
             count(job[k + m + 1]) == count(J))
        ++m;
      J.members = ++m;
      J.blk0 = blk;
      blk += J.members * ((count(J) + 7) / 8 * 8);
    }
    J.sum0 = sum;
    J.part = floats;
    sum += (int)nblk((size_t)J.kin * J.nout, 16);
    floats += (size_t)J.gx * J.kin * ((J.nout + 15) / 16 * 16);
  }
  blocks = blk;
  sums = sum;
}

size_t TrWgrads::room() const {
  // the count of row blocks rises and falls with the rows, below these bounds
  size_t floats = 0;
  for (int k = 0; k < n; ++k) {
    const TrWgradJob &J = job[k];
    const size_t least = J.pair_rows ? 512 : 1024, most = J.pair_rows ? 1024 : 512;
    floats += std::min((J.rows_max + least - 1) / least, most) * J.kin *
              ((J.nout + 15) / 16 * 16);
  }
  return floats;
}

hipError_t launch_tr_wgrads(const TrWgrads &b, int bf16, float *part, hipStream_t s) {
  if (b.n <= 0) return hipSuccess;
  for (int k = 0; k < b.n; ++k)  // the rows are read as vectors
    if (b.job[k].ldx % 4 || b.job[k].ldz % 4) return hipErrorInvalidValue;
  if (bf16)
    hipLaunchKernelGGL((k_wgrads<true>), dim3(b.blocks), dim3(256), 0, s, b, part);
  else
    hipLaunchKernelGGL((k_wgrads<false>), dim3(b.blocks), dim3(256), 0, s, b, part);
  hipLaunchKernelGGL(k_wgrad_sums, dim3(b.sums), dim3(256), 0, s, b, part);
  return hipGetLastError();
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
