// Per-centre kernels of DPA-1: the gated neighbour self-attention core and
// the descriptor contraction, forward and input-gradient backward.
//
// DPA-1 refines the embedding matrix G of each centre with gated
// self-attention blocks that act only within that centre's neighbour set
// and whose gate carries the angular term R R^T (Sec. II-B, DPA-1); the
// descriptor is D = G^T R~ R~^T G_< (Sec. II-B, DP-SE).  With the per-pair
// switch w = sw(r) and unit vectors rhat the attention of one centre is
//   lam_qk = q_q . k_k / sqrt(d)
//   L_qk   = (lam_qk + S) w_q w_k - S
//   P_qk   = exp(L_qk) / (sum_k' exp(L_qk') + (sel - n) exp(-S))
//   A_qk   = P_qk w_q w_k (rhat_q . rhat_k)
//   o_q    = sum_k A_qk v_k
// The shift S, the w_q w_k factors and the (sel - n) exp(-S) term make the
// energy continuous when a neighbour crosses the cutoff (sw -> 0 turns its
// logit into -S, the value the padding term stands for).
//
// Layout: one wavefront per 16-neighbour tile of a centre (n <= 128 -> at most 8
// tiles), one centre or several to a workgroup.  Products run on the FP32 matrix
// cores in the FP32 forward, on two-term f16 operands (split.h) in its adjoint,
// and on BF16 operands in BF16 mode.  Logit tiles are computed transposed,
// S^T = K Q^T, so that lane l holds keys 4*(l/16)+{0..3} of query l%16: that
// register layout is exactly the B operand of the next product (A V, dS K, ...),
// so probabilities never leave registers in the forward pass.
#include <cfloat>
#include <mutex>

#include "attn_classes.h"
#include "dpa1_internal.h"
#include "ln_res.h"
#include "split.h"

namespace dpa1 {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
constexpr int kMaxTiles = 8;     // 128 neighbours
constexpr int kQKV = 3;          // q, k, v blocks in one row of the projection output

__device__ __forceinline__ floatx4 mfma4(float a, float b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// BF16 precision mode (template flag BF): gfx950's v_mfma_f32_16x16x32_bf16
// contracts two 16-deep chunks (two feature chunks, or two 16-neighbour
// tiles) at once.  Each lane's eight operand slots hold its four
// consecutive k values of the first chunk, then those of the second, on
// both operands alike (the values the FP32 path feeds to four 16x16x4 steps
// per chunk), which equals two 16x16x16 steps.  Operands are rounded to BF16
// in registers, accumulation is FP32.  Every class has an even number of
// tiles, so tiles always pair.
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ bf16x4 to_bf16(const floatx4 &v) {
  return __builtin_convertvector(v, bf16x4);
}
__device__ __forceinline__ bf16x8 to_bf16x8(const floatx4 &lo, const floatx4 &hi) {
  return __builtin_shufflevector(to_bf16(lo), to_bf16(hi), 0, 1, 2, 3, 4, 5, 6, 7);
}
__device__ __forceinline__ floatx4 mfma_bf16x2(const bf16x8 &a, const bf16x8 &b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// exp x = 2^(x log2 e) on the hardware v_exp_f32: two operations instead of
// the library expf's range reduction.  Its arguments here are logits minus
// their row maximum (<= 0); the relative error, about |x| ulps, is below the
// FP32 rounding of what follows.  The forward and both adjoint kernels use
// it alike, so the adjoint recomputes the forward's probabilities exactly.
__device__ __forceinline__ float exp_hw(float x) {
  return __builtin_amdgcn_exp2f(x * 1.44269504088896341f);
}

__device__ __forceinline__ float sum_groups(float v) {  // over lanes sharing lane%16
  v += __shfl_xor(v, 16);
  v += __shfl_xor(v, 32);
  return v;
}
__device__ __forceinline__ float max_groups(float v) {
  v = fmaxf(v, __shfl_xor(v, 16));
  v = fmaxf(v, __shfl_xor(v, 32));
  return v;
}

// The value of a partner lane within the 16 lanes of a group, on the vector
// ALU (data-parallel primitives): i ^ 8 (rotation by 8), i ^ 7 (mirror of 8
// lanes), i ^ 3 (mirror of 4), i ^ 1.  In this order the four exchanges reach
// all 16 lanes, and each keeps the lane bits above its own.
constexpr int kDppXor8 = 0x128, kDppXor7 = 0x141, kDppXor3 = 0x1B, kDppXor1 = 0xB1;
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float sum16(float v) {  // over the 16 lanes of a group
  v += dpp<kDppXor8>(v);
  v += dpp<kDppXor7>(v);
  v += dpp<kDppXor3>(v);
  v += dpp<kDppXor1>(v);
  return v;
}

// Pair tensors (QKV, the attention output o, dO, dQKV) are stored FP32, or
// BF16 in BF16 mode (SB), where they are only ever BF16 matrix-core operands
// (the one elementwise use, D_q = dO . o, then sees the rounded values).
// Offsets are in elements of the storage type.
template <bool SB>
__device__ __forceinline__ const float *pt_at(const float *base, size_t e) {
  if constexpr (SB) return (const float *)((const __bf16 *)base + e);
  else return base + e;
}
template <bool SB>
__device__ __forceinline__ float *pt_at(float *base, size_t e) {
  if constexpr (SB) return (float *)((__bf16 *)base + e);
  else return base + e;
}
template <bool SB>
__device__ __forceinline__ floatx4 ldp4(const float *p, int e) {
  if constexpr (SB)
    return __builtin_convertvector(*(const bf16x4 *)((const __bf16 *)p + e), floatx4);
  else
    return *(const floatx4 *)(p + e);
}
template <bool SB>
__device__ __forceinline__ void stp4(float *p, int e, const floatx4 &v) {
  if constexpr (SB)
    *(bf16x4 *)((__bf16 *)p + e) = __builtin_convertvector(v, bf16x4);
  else
    *(floatx4 *)(p + e) = v;
}

// Load one 16x128 row tile (columns col..col+127) as the MFMA B operand:
// lane holds row r, features 16c + 4g + {0..3}.  Rows past n read row 0 of
// the centre (finite values; every use of such a row is masked), so no load
// waits on a select.
template <bool SB>
__device__ __forceinline__ void load_rows(const float *__restrict__ rows, int col, int ld,
                                          int base, int n, int row, int g, floatx4 (&v)[8]) {
  const float *rb = pt_at<SB>(rows, (size_t)base * ld + col);
  const int off = (row < n ? row : 0) * ld + 4 * g;
#pragma unroll
  for (int c = 0; c < 8; ++c) v[c] = ldp4<SB>(rb, off + 16 * c);
}

// Row stride of the row-major LDS tiles: 128 features + 4 (with it, eight
// consecutive lanes reading 16 bytes each from eight consecutive rows touch
// 32 distinct banks).
constexpr int kLDR = 132;

// Stage rows [base, base + n) x 128 features of src (row stride ld) into LDS
// row-major, X[row][kLDR]; rows n..NPAD-1 are zero.  Products whose A operand
// runs along the features (Q K^T, dO V^T) read it with one 16-byte LDS load
// per lane per four MFMA steps.
// The loads and the LDS writes are separate steps so that a kernel issues
// every global load of a phase before it waits for any (a load whose value is
// consumed at once, or a branch that overwrites it, serialises the latencies).
// Rows past n read row 0 and are written as zeros (a select at the write).
template <int NPAD, bool SB>
__device__ __forceinline__ void stage_rows_load(const float *__restrict__ src, int col, int ld,
                                                int base, int n, int tid, float4 (&v)[8]) {
  constexpr int THREADS = NPAD / 16 * 64;
  static_assert(NPAD * 32 / THREADS == 8, "eight float4 per thread");
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    const int idx = tid + it * THREADS;
    const int row = idx >> 5, c4 = idx & 31;
    const int rr = row < n ? row : 0;
    const floatx4 x = ldp4<SB>(pt_at<SB>(src, (size_t)(base + rr) * ld + col + 4 * c4), 0);
    v[it] = make_float4(x[0], x[1], x[2], x[3]);
  }
}
template <int NPAD>
__device__ __forceinline__ void stage_rows_store(float *X, int tid, int n, const float4 (&v)[8]) {
  constexpr int THREADS = NPAD / 16 * 64;
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    const int idx = tid + it * THREADS;
    const int row = idx >> 5, c4 = idx & 31;
    const bool ok = row < n;
    *(float4 *)(X + row * kLDR + 4 * c4) =
        make_float4(ok ? v[it].x : 0.f, ok ? v[it].y : 0.f, ok ? v[it].z : 0.f, ok ? v[it].w : 0.f);
  }
}

// Stage rows [base, base + n) x 128 features of src into LDS transposed,
// XT[f][k] with row stride NPAD + 4; rows n..NPAD-1 are zero.  Products that
// contract over neighbours read it with one 16-byte LDS load per lane per
// four MFMA steps.  Wave w stages rows 16w..16w+15; in each step lane l takes
// row 16w + l%16 and feature quad 4 it + l/16, so the four scalar LDS writes
// of one float4 hit 64 distinct banks.
// The load half and the LDS half are separate so that a kernel can issue the
// loads one phase early (while the previous phase computes) and write LDS
// after the barrier that frees the buffer.
template <int NPAD, bool SB>
__device__ __forceinline__ void stage_t_load(const float *__restrict__ src, int col, int ld,
                                             int base, int n, int tid, float4 (&v)[8]) {
  const int row = (tid >> 6) * 16 + (tid & 15);
  const int cq = (tid >> 4) & 3;
  const int rr = row < n ? row : 0;
  const float *sp = pt_at<SB>(src, (size_t)(base + rr) * ld + col + 4 * cq);
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    const floatx4 x = ldp4<SB>(sp, 16 * it);
    v[it] = make_float4(x[0], x[1], x[2], x[3]);
  }
}
// rows past n (loaded from row 0) are written as zeros
template <int NPAD>
__device__ __forceinline__ void stage_t_store(float *XT, int tid, int n, const float4 (&v)[8]) {
  constexpr int LDT = NPAD + 4;
  const int row = (tid >> 6) * 16 + (tid & 15);
  const int cq = (tid >> 4) & 3;
  const bool ok = row < n;
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    float *d = XT + (16 * it + 4 * cq) * LDT + row;
    d[0] = ok ? v[it].x : 0.f;
    d[LDT] = ok ? v[it].y : 0.f;
    d[2 * LDT] = ok ? v[it].z : 0.f;
    d[3 * LDT] = ok ? v[it].w : 0.f;
  }
}

// Gate record of neighbour t = tid (rhat, sw; zeros past n), for kg[NPAD]:
// one unconditional load per thread (threads past NPAD read slot 0), written
// by gate_store.  lo is the FP32 remainder of the switch value (sw - hi in
// FP64), so that hi + lo carries sw to the logits with FP64 accuracy.
__device__ __forceinline__ float4 gate_load(const float *__restrict__ geom, int base, int n,
                                            int tid, float &lo) {
  const int t = tid < n ? tid : 0;
  const float4 *gp = (const float4 *)(geom + (size_t)(base + t) * kGeom);
  const float4 a = gp[0], b = gp[1];  // s, rx, ry, rz | sw, r, dsw, sw remainder
  lo = b.w;
  return make_float4(a.y, a.z, a.w, b.x);
}
// kw[NPAD]: the switch value of each neighbour in FP64 (zero past n), or null.
template <int NPAD>
__device__ __forceinline__ void gate_store(float4 *kg, double *kw, int tid, int n,
                                           const float4 &v, float lo) {
  const bool ok = tid < n;
  if (tid < NPAD) {
    kg[tid] = make_float4(ok ? v.x : 0.f, ok ? v.y : 0.f, ok ? v.z : 0.f, ok ? v.w : 0.f);
    if (kw) kw[tid] = ok ? (double)v.w + (double)lo : 0.0;
  }
}

// Scaled logit L = (lam + S) w_q w_k - S of the FP32 path, with the switch
// values and the shift in FP64 and one rounding at the end.  The logit's
// sensitivity to each switch value is lam + S (about S = 20), so with FP32
// switch values and FP32 arithmetic here the logit carries an absolute error
// of a few 1e-6; at the rare centres where a pair of opposite neighbours
// attend strongly to each other the forces amplify that by ~1e4 (measured on
// the oracle's formula evaluated in FP32).  The products and every other
// elementwise step stay FP32; the BF16 mode keeps FP32 logits.
__device__ __forceinline__ float logit64(float lam, double wq, double wk, float shift) {
  const double s = (double)shift;
  return (float)fma((double)lam + s, wq * wk, -s);
}

// acc[ft] += XT^T-tile x bt : contraction over the 16 rows of tile 'tile',
// XT in LDS (feature-major), bt a 16x16 B operand held in registers.
// Output lane layout: own row r, features 16 ft + 4 g + v.
template <int NPAD>
__device__ __forceinline__ void accum_lds(const float *XT, int tile, int r, int g,
                                          const floatx4 &bt, floatx4 (&acc)[8]) {
  constexpr int LDT = NPAD + 4;
#pragma unroll
  for (int h = 0; h < 2; ++h) {  // two halves of the features: 16 operand registers
    floatx4 x[4];
#pragma unroll
    for (int f = 0; f < 4; ++f)
      x[f] = *(const floatx4 *)(XT + ((4 * h + f) * 16 + r) * LDT + tile * 16 + 4 * g);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int f = 0; f < 4; ++f) acc[4 * h + f] = mfma4(x[f][t], bt[t], acc[4 * h + f]);
  }
}
// BF16: tiles 'tile' and 'tile' + 1 in one 16x16x32 step, B operands bt0, bt1.
template <int NPAD>
__device__ __forceinline__ void accum_lds2(const float *XT, int tile, int r, int g,
                                           const floatx4 &bt0, const floatx4 &bt1,
                                           floatx4 (&acc)[8]) {
  constexpr int LDT = NPAD + 4;
  const bf16x8 btb = to_bf16x8(bt0, bt1);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    floatx4 x0[4], x1[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const float *xp = XT + ((4 * h + f) * 16 + r) * LDT + tile * 16 + 4 * g;
      x0[f] = *(const floatx4 *)xp;
      x1[f] = *(const floatx4 *)(xp + 16);
    }
#pragma unroll
    for (int f = 0; f < 4; ++f)
      acc[4 * h + f] = mfma_bf16x2(to_bf16x8(x0[f], x1[f]), btb, acc[4 * h + f]);
  }
}

// The same contraction with the rows in row-major LDS (X[row][kLDR]): the A
// operand is read with scalar LDS loads, four rows per lane group.  Row tiles 'tile' and 'tile' + 1 in one 16x16x32 step.
__device__ __forceinline__ void accum_rows2(const float *X, int tile, int r, int g,
                                            const floatx4 &bt0, const floatx4 &bt1,
                                            floatx4 (&acc)[8]) {
  const float *xb = X + (tile * 16 + 4 * g) * kLDR + r;
  const bf16x8 btb = to_bf16x8(bt0, bt1);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    floatx4 x0[4], x1[4];
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        x0[f][t] = xb[t * kLDR + (4 * h + f) * 16];
        x1[f][t] = xb[(16 + t) * kLDR + (4 * h + f) * 16];
      }
#pragma unroll
    for (int f = 0; f < 4; ++f)
      acc[4 * h + f] = mfma_bf16x2(to_bf16x8(x0[f], x1[f]), btb, acc[4 * h + f]);
  }
}

// st[kt] (lane: own row r, tile rows 4g + v) = X-rows of tile kt times the
// wave's own 16 rows b, contracted over the 128 features; X row-major in LDS.
template <int NT, bool BF>
__device__ __forceinline__ void qk_lds(const float *X, int r, int g, const floatx4 (&b)[8],
                                       floatx4 (&st)[NT]) {
#pragma unroll
  for (int kt = 0; kt < NT; ++kt) st[kt] = floatx4{0.f, 0.f, 0.f, 0.f};
  const float *xb = X + r * kLDR + 4 * g;
  // one feature chunk at a time (LDS latency is covered by the other
  // wavefronts on the SIMD); the fence keeps the compiler from hoisting the
  // loads of later chunks, which would hold many more registers
  if constexpr (BF) {
    // feature chunks 2h and 2h + 1 in one 16x16x32 step
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      floatx4 a0[NT], a1[NT];
#pragma unroll
      for (int kt = 0; kt < NT; ++kt) {
        a0[kt] = *(const floatx4 *)(xb + kt * 16 * kLDR + 32 * h);
        a1[kt] = *(const floatx4 *)(xb + kt * 16 * kLDR + 32 * h + 16);
      }
      __builtin_amdgcn_sched_barrier(0);
      const bf16x8 bb = to_bf16x8(b[2 * h], b[2 * h + 1]);
#pragma unroll
      for (int kt = 0; kt < NT; ++kt) st[kt] = mfma_bf16x2(to_bf16x8(a0[kt], a1[kt]), bb, st[kt]);
    }
    return;
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    floatx4 a[NT];
#pragma unroll
    for (int kt = 0; kt < NT; ++kt) a[kt] = *(const floatx4 *)(xb + kt * 16 * kLDR + 16 * c);
    __builtin_amdgcn_sched_barrier(0);
    {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int kt = 0; kt < NT; ++kt) st[kt] = mfma4(a[kt][t], b[c][t], st[kt]);
    }
  }
}

// The thread index, opaque to the optimiser.  Taken afresh in every
// iteration of the per-centre loops so that per-lane addresses are
// recomputed there instead of being hoisted out of the loop and held in
// registers for its whole duration (which made the large classes spill).
__device__ __forceinline__ int fresh_tid() {
  int t = (int)threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Barrier of the wavefronts that work on one centre: the workgroup's barrier
// when it has one centre (C = 1), else an arrival count in LDS, one per centre,
// so that the centres of a workgroup do not wait for each other's phases.  All
// of a workgroup's wavefronts are resident and those of a centre pass the same
// barriers, so a count is always reached.  The constructor is for every
// thread of the workgroup.
template <int C, int WAVES>
struct CentreBarrier {
  unsigned *count;
  unsigned arrived = 0;
  __device__ __forceinline__ CentreBarrier(unsigned *counts, int part) : count(counts + part) {
    if constexpr (C > 1) {
      if (threadIdx.x < C) counts[threadIdx.x] = 0;
      __syncthreads();
    }
  }
  __device__ __forceinline__ void operator()() {
    if constexpr (C == 1) {
      __syncthreads();
    } else {
      arrived += WAVES;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      if ((threadIdx.x & 63) == 0)
        __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(
                 count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) < arrived)
        __builtin_amdgcn_s_sleep(1);
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
  }
};

// Floats of the staging buffer: NPAD rows x kLDR or 128 features x (NPAD + 4).
template <int NPAD>
constexpr int stage_floats() {
  return NPAD * kLDR > 128 * (NPAD + 4) ? NPAD * kLDR : 128 * (NPAD + 4);
}

// --------------------------------------------------------------------- forward
//
// Centres are processed by a persistent grid: block b takes the centres
// b, b + gridDim.x, ... of its class list (every centre of a class costs the
// same padded work, so the static split is balanced).  One wavefront per
// 16-query tile.  K is staged row-major in LDS for Q K^T, then V transposed
// for A V; global memory is touched only by the staging steps, the wave's
// own query rows and the outputs.  The scaled dot products lam = q.k/sqrt(d)
// (row stride kLamLd, all NPAD key columns of every query row) and the
// softmax statistics (m, 1/Z) of every query are stored for the adjoint,
// which then does not recompute Q K^T.  The FP32 forward issues the next
// centre's staging loads while it finishes the current one, so that the HBM
// latency of a centre's operands overlaps the previous centre's products.

constexpr int kLamLd = kAttnLamLd;
constexpr int kOpCols = kAttnOpCols;   // output columns of the fused projection
constexpr int kOpTiles = kOpCols / 16;

// OP: the output projection and its layer norm are applied here
// (W_O^T, 7 column tiles, staged in LDS once per workgroup; the epilogue is
// the one the projection GEMM uses), so the attention output o goes to
// memory only where the two-kernel adjoint of the 128 class reads it.
// LDS of one centre: kg, kw, buf.
template <int NPAD>
constexpr size_t fwd_centre_lds() {
  return (sizeof(float4) + sizeof(double)) * NPAD + sizeof(float) * stage_floats<NPAD>();
}

// With the projection a workgroup holds several centres (fwd_centres), each
// with its own buffer and barriers, around the one W_O^T: two of the 96 class
// put three wavefronts on every SIMD, where a workgroup of six leaves two SIMDs
// with half the others' MFMAs and a second one does not fit (160 KB of LDS, and
// six wavefronts of more than 128 registers cannot share a CU with another
// six: each workgroup starts on the first SIMD).  Per layer at 15,668 centres
// of 84 neighbours: FP32 1.69 -> 1.36 ms, BF16 0.78 -> 0.70 ms.
// Above 105 features W_O^T and two centres of the 96 class no longer fit, and
// a workgroup takes one centre (C = 1) in every class.
template <int NPAD>
constexpr int fwd_centres() { return NPAD > 96 ? 1 : (NPAD == 32 ? 4 : 2); }
constexpr int kFwdMaxCols = 105;

template <int NPAD, bool BF, bool OP, int C>
__global__ __launch_bounds__(C * NPAD / 16 * 64, OP ? (C == 2 && NPAD == 96 ? 3 : 2) : BF ? (NPAD <= 64 ? 4 : (NPAD <= 96 ? 3 : 2)) : 2) void k_attn_fwd(
    const float *__restrict__ qkv, const float *__restrict__ geom,
    const int *__restrict__ pair_off, const int *__restrict__ nnei,
    const int *__restrict__ clist, const int *__restrict__ ccount, int sel, float shift,
    float *__restrict__ out, float *__restrict__ lam, float2 *__restrict__ fstat,
    AttnOut op) {
  constexpr int NT = NPAD / 16;
  constexpr bool STORE_O = !OP || (BF && NPAD > 96);
  extern __shared__ float4 smem[];
  __shared__ unsigned bar[C];
  const int part = C == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / (NT * 64));
  float4 *kg = smem + part * (int)(fwd_centre_lds<NPAD>() / sizeof(float4));
  double *kw = (double *)(kg + NPAD);    // [NPAD] switch values in FP64
  float *buf = (float *)(kw + NPAD);     // K rows, then V^T
  // OP: W_O^T [op.Nreal][kLDR], then bias, gamma, beta [3][kOpCols]
  float *wo = (float *)(smem + C * (int)(fwd_centre_lds<NPAD>() / sizeof(float4)));
  float *cso = wo + op.Nreal * kLDR;
  const int ld = kQKV * 128;
  const float inv_sqrt_d = 0.08838834764831845f;  // 1/sqrt(128)
  const int cnt = *ccount;
  if ((int)blockIdx.x >= cnt) return;  // no centre for the whole workgroup
  if constexpr (OP) {
    for (int idx = threadIdx.x; idx < op.Nreal * 32; idx += blockDim.x) {
      const int row = idx >> 5, c4 = idx & 31;
      *(float4 *)(wo + row * kLDR + 4 * c4) = *(const float4 *)(op.Wt_o + row * 128 + 4 * c4);
    }
    for (int idx = threadIdx.x; idx < 3 * kOpCols; idx += blockDim.x) {
      const int k = idx / kOpCols, n = idx % kOpCols;
      cso[idx] = (k == 0 ? op.bias : (k == 1 ? op.gamma : op.beta))[n];
    }
    __syncthreads();
  }
  CentreBarrier<C, NT> barrier(bar, part);
  // the centres of part p are those of the list's positions first, first +
  // step, ...: with fewer centres than workgroups each has a CU to itself
  const int step = (int)gridDim.x * C;
  const int first = (int)blockIdx.x + part * (int)gridDim.x;
  if (first >= cnt) return;
  // FP32: the staging loads of a centre (and, with one centre to a workgroup,
  // its own query rows) are issued during the A V phase of the previous one
  // (BF16 holds more registers per tile and loads per centre); after the last
  // centre they are its own again, since under a branch the old values would
  // stay live through the whole loop
  constexpr bool PREF = !BF, PREFQ = PREF && C == 1;
  float4 sv[8];
  floatx4 qv[8];
  float4 gv;
  float gl = 0.f;
  int n_nx = 0, base_nx = 0;
  auto fetch = [&](int at, int tid) {
    const int i = clist[min(at, cnt - 1)];
    n_nx = nnei[i];
    base_nx = pair_off[i];
    stage_rows_load<NPAD, BF>(qkv, 128, ld, base_nx, n_nx, tid, sv);  // K
    gv = gate_load(geom, base_nx, n_nx, tid, gl);
    if constexpr (PREFQ || !PREF)
      load_rows<BF>(qkv, 0, ld, base_nx, n_nx, (tid >> 6) * 16 + (tid & 15), (tid & 63) >> 4, qv);
  };
  if (PREF) fetch(first, fresh_tid() - part * NT * 64);
  for (int it = first; it < cnt; it += step) {
    const int tid = fresh_tid() - part * NT * 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int r = lane & 15, g = lane >> 4;
    if constexpr (!PREF) fetch(it, tid);
    const int n = n_nx;
    const int base = base_nx;
    const int ntile = (n + 15) >> 4;
    const int q = wave * 16 + r;
    const bool qok = q < n;
    if constexpr (PREF && !PREFQ) load_rows<BF>(qkv, 0, ld, base, n, q, g, qv);
    stage_rows_store<NPAD>(buf, tid, n, sv);
    gate_store<NPAD>(kg, kw, tid, n, gv, gl);
    barrier();
    float4 vpre[8];  // V, read while Q K^T and the softmax run
    stage_t_load<NPAD, BF>(qkv, 256, ld, base, n, tid, vpre);

    floatx4 st[NT];
    float invz = 0.f;
    if (wave < ntile) {
      qk_lds<NT, BF>(buf, r, g, qv, st);
#pragma unroll
      for (int kt = 0; kt < NT; ++kt) st[kt] *= inv_sqrt_d;
      if (qok) {
        float *lp = lam + (size_t)(base + q) * kLamLd + 4 * g;
#pragma unroll
        for (int kt = 0; kt < NT; ++kt) *(floatx4 *)(lp + 16 * kt) = st[kt];
      }
      const float wq = qok ? kg[q].w : 0.f;
      const double wqd = qok ? kw[q] : 0.0;
      float mx = -FLT_MAX;
#pragma unroll
      for (int kt = 0; kt < NT; ++kt) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int k = kt * 16 + 4 * g + v;
          float l = BF ? (st[kt][v] + shift) * wq * kg[k].w - shift
                       : logit64(st[kt][v], wqd, kw[k], shift);
          l = k < n ? l : -INFINITY;
          st[kt][v] = l;
          mx = fmaxf(mx, l);
        }
      }
      const float m = fmaxf(max_groups(mx), -shift);
      float z = 0.f;
#pragma unroll
      for (int kt = 0; kt < NT; ++kt) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float e = exp_hw(st[kt][v] - m);
          st[kt][v] = e;
          z += e;
        }
      }
      z = sum_groups(z) + (float)(sel - n) * exp_hw(-shift - m);
      invz = 1.0f / z;
      if (g == 0 && qok) fstat[base + q] = make_float2(m, invz);
    }
    barrier();
    stage_t_store<NPAD>(buf, tid, n, vpre);  // V^T
    barrier();
    if constexpr (PREFQ) fetch(it + step, tid);

    if (wave < ntile) {
      const float4 gq = kg[q];
      const float wq = qok ? gq.w : 0.f;
      floatx4 oacc[8];
      floatx4 atp;  // BF16: probabilities of the even tile of a pair
#pragma unroll
      for (int ft = 0; ft < 8; ++ft) oacc[ft] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kt = 0; kt < NT; ++kt) {
        floatx4 at;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float4 gk = kg[kt * 16 + 4 * g + v];
          const float c = gq.x * gk.x + gq.y * gk.y + gq.z * gk.z;
          at[v] = st[kt][v] * invz * wq * gk.w * c;
        }
        if constexpr (BF) {  // tiles taken in pairs
          if (kt % 2 == 0) atp = at;
          else accum_lds2<NPAD>(buf, kt - 1, r, g, atp, at, oacc);
        } else {
          accum_lds<NPAD>(buf, kt, r, g, at, oacc);
        }
      }
      if (STORE_O && qok) {
        float *opp = pt_at<BF>(out, (size_t)(base + q) * 128 + 4 * g);
#pragma unroll
        for (int ft = 0; ft < 8; ++ft) stp4<BF>(opp, 16 * ft, oacc[ft]);
      }
      if constexpr (OP) {
        // y = o W_O in the projection GEMM's order (feature chunk, step,
        // column tile), then G_out = G_in + gamma LN(y + b) + beta
        const size_t rb = (size_t)(base + (qok ? q : 0)) * kOpCols;
        floatx4 gi[kOpTiles];
#pragma unroll
        for (int nt = 0; nt < kOpTiles; ++nt) gi[nt] = *(const floatx4 *)(op.gin + rb + 16 * nt + 4 * g);
        floatx4 y[kOpTiles];
#pragma unroll
        for (int nt = 0; nt < kOpTiles; ++nt) y[nt] = floatx4{0.f, 0.f, 0.f, 0.f};
        // columns past Nreal (96 < Nreal, so of the last tile) read its last
        // row; the epilogue zeroes them
        const float *wl = wo + r * kLDR + 4 * g;
        const float *wlast = wo + min((kOpTiles - 1) * 16 + r, op.Nreal - 1) * kLDR + 4 * g;
        const auto w_at = [&](int nt, int k) {
          return *(const floatx4 *)((nt < kOpTiles - 1 ? wl + nt * 16 * kLDR : wlast) + k);
        };
        if constexpr (BF) {
          // feature chunks 2h and 2h + 1 in one 16x16x32 step
#pragma unroll
          for (int h = 0; h < 4; ++h) {
            const bf16x8 ob = to_bf16x8(oacc[2 * h], oacc[2 * h + 1]);
            bf16x8 w[kOpTiles];
#pragma unroll
            for (int nt = 0; nt < kOpTiles; ++nt)
              w[nt] = to_bf16x8(w_at(nt, 32 * h),
                                w_at(nt, 32 * h + 16));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int nt = 0; nt < kOpTiles; ++nt) y[nt] = mfma_bf16x2(w[nt], ob, y[nt]);
          }
        } else {
#pragma unroll
          for (int c = 0; c < 8; ++c) {
            floatx4 w[kOpTiles];
#pragma unroll
            for (int nt = 0; nt < kOpTiles; ++nt)
              w[nt] = w_at(nt, 16 * c);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
              for (int nt = 0; nt < kOpTiles; ++nt) y[nt] = mfma4(w[nt][t], oacc[c][t], y[nt]);
          }
        }
        // three wavefronts to a SIMD leave registers for the loads only now
        if constexpr (PREF && !PREFQ) fetch(it + step, tid);
        lnres::apply_tile<kOpTiles>(y, gi, g, kOpTiles, op.Nreal, op.eps, cso, kOpCols, qok,
                                    base + q, rb, op.gout, op.xhat, op.rstd);
      }
    } else if constexpr (PREF && !PREFQ) {
      fetch(it + step, tid);
    }
    barrier();  // LDS is restaged for the next centre
  }
}

// -------------------------------------------------------------------- backward
//
// Given dO, with H = w_q w_k c_qk (c = rhat_q . rhat_k):
//   dA = dO V^T ; dV = A^T dO ; dP = dA H ; dH = dA P
//   D_q = sum_k P dP = dO_q . o_q ; dL = P (dP - D_q)
//   dS = dL w_q w_k / sqrt(d) ; dQ = dS K ; dK = dS^T Q
//   X = dL (lam + S) + dH c  -> dw_q += sum_k X w_k, dw_k += sum_q X w_q
//   Y = dH w_q w_k           -> drhat_q += sum_k Y rhat_k, drhat_k += sum_q Y rhat_q
// FP32 takes one kernel for every class (k_attn_bwd_s), BF16 one for the classes
// of up to 96 neighbours (k_attn_bwd_f) and two for the 128 class; all read lam
// and (m, 1/Z) stored by the forward.  The two:
// k_attn_bwd_q (wave = query tile): dA^T from V staged row-major, then dS,
// dQ (K^T staged) and the query-side sums; it writes dA in the layout of lam
// (row = query, n columns), (m, 1/Z, D_q) and the query-side sums per pair.
// k_attn_bwd_k (wave = key tile): reads dA key-major the way it reads lam
// (one column of the centre's rows per lane) instead of forming it a second
// time with a matrix product, forms dV from dO staged row-major, then dK
// (Q^T staged) and the key-side sums; it adds both sides into dE/dsw and
// dE/drhat.

__global__ __launch_bounds__(512, 2) void k_attn_bwd_q(
    const float *__restrict__ qkv, const float *__restrict__ o, const float *__restrict__ dO,
    const float *__restrict__ geom, const int *__restrict__ pair_off,
    const int *__restrict__ nnei, const int *__restrict__ clist, const int *__restrict__ ccount,
    int sel, float shift, const float *__restrict__ lam, const float2 *__restrict__ fstat,
    float *__restrict__ dqkv, float4 *__restrict__ astat, float4 *__restrict__ qside,
    float *__restrict__ dA) {
  constexpr int NPAD = 128, NT = NPAD / 16;
  extern __shared__ float4 smem[];
  float4 *kg = smem;                     // [NPAD] rhat, sw
  float *buf = (float *)(kg + NPAD);     // V rows, then K^T
  const int ld = kQKV * 128;
  const float inv_sqrt_d = 0.08838834764831845f;
  const int cnt = *ccount;
  for (int it = blockIdx.x; it < cnt; it += gridDim.x) {
    const int tid = fresh_tid();
    const int wave = tid >> 6;
    const int lane = tid & 63;
    const int r = lane & 15, g = lane >> 4;
    const int i = clist[it];
    const int n = nnei[i];
    const int base = pair_off[i];
    const int ntile = (n + 15) >> 4;
    const int q = wave * 16 + r;
    const bool qok = q < n;
    float4 sv[8];
    stage_rows_load<NPAD, true>(qkv, 256, ld, base, n, tid, sv);  // V
    float gl;
    const float4 gv = gate_load(geom, base, n, tid, gl);
    floatx4 dov[8], ov[8];
    load_rows<true>(dO, 0, 128, base, n, q, g, dov);
    load_rows<true>(o, 0, 128, base, n, q, g, ov);
    stage_rows_store<NPAD>(buf, tid, n, sv);
    gate_store<NPAD>(kg, nullptr, tid, n, gv, gl);
    __syncthreads();
    float dq = 0.f;
    if (wave < ntile) {
#pragma unroll
      for (int c = 0; c < 8; ++c)
        dq += dov[c][0] * ov[c][0] + dov[c][1] * ov[c][1] + dov[c][2] * ov[c][2] +
              dov[c][3] * ov[c][3];
      dq = sum_groups(dq);
    }
    float4 kpre[8];  // K, read while dA^T is formed
    stage_t_load<NPAD, true>(qkv, 128, ld, base, n, tid, kpre);

    floatx4 da[NT];
    if (wave < ntile) {
      qk_lds<NT, true>(buf, r, g, dov, da);  // dA^T tiles: lane (query r, keys 4g + v)
      if (qok) {  // dA row of this query, for the key-tile kernel
        float *dp = dA + (size_t)(base + q) * kLamLd + 4 * g;
#pragma unroll
        for (int kt = 0; kt < NT; ++kt) *(floatx4 *)(dp + 16 * kt) = da[kt];
      }
    }
    __syncthreads();
    stage_t_store<NPAD>(buf, tid, n, kpre);  // K^T
    __syncthreads();

    if (wave < ntile) {
      const int qr = qok ? q : 0;
      const float4 gq = kg[q];
      const float wq = qok ? gq.w : 0.f;
      const float2 fs = fstat[base + qr];
      const float m = fs.x, invz = fs.y;
      if (g == 0 && qok) astat[base + q] = make_float4(m, invz, dq, 0.f);
      // lam of this query row, read one key tile ahead of its use
      const float *lp = lam + (size_t)(base + qr) * kLamLd + 4 * g;
      floatx4 dqacc[8];
      floatx4 dsp;  // dS of the even tile of a pair
#pragma unroll
      for (int ft = 0; ft < 8; ++ft) dqacc[ft] = floatx4{0.f, 0.f, 0.f, 0.f};
      float dwq = 0.f, drqx = 0.f, drqy = 0.f, drqz = 0.f;
      floatx4 lcur = *(const floatx4 *)lp, lnxt;
#pragma unroll
      for (int kt = 0; kt < NT; ++kt) {
        if (kt + 1 < NT) lnxt = *(const floatx4 *)(lp + 16 * (kt + 1));
        floatx4 ds;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int k = kt * 16 + 4 * g + v;
          const bool ok = qok && k < n;
          const float4 gk = kg[k];
          const float c = gq.x * gk.x + gq.y * gk.y + gq.z * gk.z;
          const float ww = wq * gk.w;
          const float lm = ok ? lcur[v] : 0.f;
          const float l = (lm + shift) * ww - shift;
          const float p = ok ? exp_hw(l - m) * invz : 0.f;
          const float h = ww * c;
          const float dH = da[kt][v] * p;
          const float dL = p * (da[kt][v] * h - dq);
          ds[v] = dL * ww * inv_sqrt_d;
          const float X = dL * (lm + shift) + dH * c;
          const float Y = dH * ww;
          dwq += X * gk.w;
          drqx += Y * gk.x;
          drqy += Y * gk.y;
          drqz += Y * gk.z;
        }
        // tiles taken in pairs
        if (kt % 2 == 0) dsp = ds;
        else accum_lds2<NPAD>(buf, kt - 1, r, g, dsp, ds, dqacc);
        lcur = lnxt;
      }
      dwq = sum_groups(dwq);
      drqx = sum_groups(drqx);
      drqy = sum_groups(drqy);
      drqz = sum_groups(drqz);
      if (g == 0 && qok) qside[base + q] = make_float4(dwq, drqx, drqy, drqz);
      if (qok) {
        float *dp = pt_at<true>(dqkv, (size_t)(base + q) * ld + 4 * g);
#pragma unroll
        for (int ft = 0; ft < 8; ++ft) stp4<true>(dp, 16 * ft, dqacc[ft]);
      }
    }
    __syncthreads();  // LDS is restaged for the next centre
  }
}

__global__ __launch_bounds__(512, 2) void k_attn_bwd_k(
    const float *__restrict__ qkv, const float *__restrict__ dO,
    const float *__restrict__ geom, const int *__restrict__ pair_off,
    const int *__restrict__ nnei, const int *__restrict__ clist, const int *__restrict__ ccount,
    float shift, const float *__restrict__ lam, const float *__restrict__ dA,
    float *__restrict__ dqkv, const float4 *__restrict__ astat,
    const float4 *__restrict__ qsbuf, float *__restrict__ gw, float *__restrict__ gr,
    int accumulate) {
  constexpr int NPAD = 128, NT = NPAD / 16;
  extern __shared__ float4 smem[];
  float4 *kg = smem;                     // [NPAD] rhat, sw
  float4 *stats = kg + NPAD;             // [NPAD] m, 1/Z, D_q of each query
  float *buf = (float *)(stats + NPAD);  // dO rows, then Q^T
  const int ld = kQKV * 128;
  const float inv_sqrt_d = 0.08838834764831845f;
  const int cnt = *ccount;
  for (int it = blockIdx.x; it < cnt; it += gridDim.x) {
    const int tid = fresh_tid();
    const int wave = tid >> 6;
    const int lane = tid & 63;
    const int r = lane & 15, g = lane >> 4;
    const int i = clist[it];
    const int n = nnei[i];
    const int base = pair_off[i];
    float4 sv[8];
    stage_rows_load<NPAD, true>(dO, 0, 128, base, n, tid, sv);  // dO
    float gl;
    const float4 gv = gate_load(geom, base, n, tid, gl);
    const float4 av = astat[base + (tid < n ? tid : 0)];
    const int ntile = (n + 15) >> 4;
    const int kk = wave * 16 + r;
    const bool kok = kk < n;
    stage_rows_store<NPAD>(buf, tid, n, sv);
    gate_store<NPAD>(kg, nullptr, tid, n, gv, gl);
    if (tid < NPAD) stats[tid] = tid < n ? av : make_float4(0.f, 1.f, 0.f, 0.f);
    __syncthreads();

    // ---------------- phase 1: dV, dS and the key-side sums
    floatx4 ds[NT];
    float dwk = 0.f, drkx = 0.f, drky = 0.f, drkz = 0.f;
    if (wave < ntile) {
      const float4 gk = kg[kk];
      const float wk = kok ? gk.w : 0.f;
      // lam and dA of this key against the queries of one tile (lane: key r,
      // queries 4g + v), read one query tile ahead
      const size_t col = (size_t)base * kLamLd + (kok ? kk : 0);
      const float *lc = lam + col, *dc = dA + col;
      auto lam_tile = [&](int qt, float (&lv)[4], float (&dv)[4]) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int qq = qt * 16 + 4 * g + v;
          const size_t off = (size_t)(qq < n ? qq : 0) * kLamLd;
          lv[v] = lc[off];
          dv[v] = dc[off];
        }
      };
      float lcur[4], lnxt[4], dcur[4], dnxt[4];
      lam_tile(0, lcur, dcur);
      floatx4 dvacc[8];
      floatx4 atp;  // A^T of the even tile of a pair
#pragma unroll
      for (int ft = 0; ft < 8; ++ft) dvacc[ft] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int qt = 0; qt < NT; ++qt) {
        ds[qt] = floatx4{0.f, 0.f, 0.f, 0.f};
        if (qt >= ntile) {
          // an unpaired last tile meets a zero partner
          if (qt % 2 == 1 && qt - 1 < ntile)
            accum_rows2(buf, qt - 1, r, g, atp, floatx4{0.f, 0.f, 0.f, 0.f}, dvacc);
          continue;
        }
        if (qt + 1 < NT) lam_tile(qt + 1, lnxt, dnxt);
        floatx4 at;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int qq = qt * 16 + 4 * g + v;
          const bool ok = kok && qq < n;
          const float4 sq = stats[qq];
          const float4 gq = kg[qq];
          const float c = gq.x * gk.x + gq.y * gk.y + gq.z * gk.z;
          const float ww = gq.w * wk;
          const float lm = ok ? lcur[v] : 0.f;
          const float l = (lm + shift) * ww - shift;
          const float p = ok ? exp_hw(l - sq.x) * sq.y : 0.f;
          const float h = ww * c;
          const float dav = ok ? dcur[v] : 0.f;
          const float dH = dav * p;
          const float dL = p * (dav * h - sq.z);
          at[v] = p * h;
          ds[qt][v] = dL * ww * inv_sqrt_d;
          const float X = dL * (lm + shift) + dH * c;
          const float Y = dH * ww;
          dwk += X * gq.w;
          drkx += Y * gq.x;
          drky += Y * gq.y;
          drkz += Y * gq.z;
        }
        // dV = A^T dO, tiles taken in pairs
        if (qt % 2 == 0) atp = at;
        else accum_rows2(buf, qt - 1, r, g, atp, at, dvacc);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          lcur[v] = lnxt[v];
          dcur[v] = dnxt[v];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (kok) {
        float *dp = pt_at<true>(dqkv, (size_t)(base + kk) * ld + 256 + 4 * g);
#pragma unroll
        for (int ft = 0; ft < 8; ++ft) stp4<true>(dp, 16 * ft, dvacc[ft]);
      }
      dwk = sum_groups(dwk);
      drkx = sum_groups(drkx);
      drky = sum_groups(drky);
      drkz = sum_groups(drkz);
    }
    __syncthreads();
    // Q rows of phase 2 (loaded only now: fewer registers in phase 1)
    float4 qpre[8];
    stage_t_load<NPAD, true>(qkv, 0, ld, base, n, tid, qpre);
    stage_t_store<NPAD>(buf, tid, n, qpre);  // Q^T
    __syncthreads();

    // ---------------- phase 2: dK = dS^T Q
    if (wave < ntile) {
      floatx4 dkacc[8];
#pragma unroll
      for (int ft = 0; ft < 8; ++ft) dkacc[ft] = floatx4{0.f, 0.f, 0.f, 0.f};
      // tiles in pairs; ds of tiles at or past ntile is zero
#pragma unroll
      for (int qt = 0; qt < NT; qt += 2)
        if (qt < ntile) accum_lds2<NPAD>(buf, qt, r, g, ds[qt], ds[qt + 1], dkacc);
      if (kok) {
        float *dp = pt_at<true>(dqkv, (size_t)(base + kk) * ld + 128 + 4 * g);
#pragma unroll
        for (int ft = 0; ft < 8; ++ft) stp4<true>(dp, 16 * ft, dkacc[ft]);
        if (g == 0) {
          const float4 qs = qsbuf[base + kk];
          const size_t p = (size_t)(base + kk);
          const float tw = qs.x + dwk, tx = qs.y + drkx, ty = qs.z + drky, tz = qs.w + drkz;
          if (accumulate) {
            gw[p] += tw;
            gr[4 * p + 0] += tx;
            gr[4 * p + 1] += ty;
            gr[4 * p + 2] += tz;
          } else {
            gw[p] = tw;
            gr[4 * p + 0] = tx;
            gr[4 * p + 1] = ty;
            gr[4 * p + 2] = tz;
            gr[4 * p + 3] = 0.f;
          }
        }
      }
    }
    __syncthreads();  // LDS is restaged for the next centre
  }
}

// ------------------------------------------------------------ fused adjoint
//
// BF16 classes of up to 96 neighbours: the wavefronts of a centre run both
// halves of the adjoint.  Phase Q (wavefront = query tile) forms dA^T, the
// softmax adjoint, dS and dQ as the query-tile kernel does and leaves
// A = P H and dS of the centre in LDS ([query][key], rounded to BF16 as the
// products take them), with the query-side sums and the key-side sums reduced
// over its 16 queries; phase K (wavefront = key tile) forms dV = A^T dO and
// dK = dS^T Q from them.  Against the two-kernel form the centre's logits and
// gate records are read once, and dA and the per-pair statistics never go to
// memory.  dQ, dK and dV are accumulated in the same order as there; only
// the key-side sums are added in another order.
//
// LDS holds every operand in BF16, row-major: V, K, dO and Q rows in turn, each
// stored by the wavefront that owns the row, and A and dS.  Where a product
// contracts over rows, gfx950's transposing LDS read (ds_read_b64_tr_b16) brings
// four rows of one column per lane, so nothing is stored transposed.  That is
// 78 KB for the 96 class instead of 142 KB in FP32, and two centres to a CU, in
// one workgroup of 12 wavefronts (k_attn_bwd_s says why) instead of one of six.
// The sums over a query tile's 16 lanes run on the vector ALU.  15,668 centres of
// the 96 class: 1.20 -> 0.88 ms a layer, 3 GB of pair rows and logits (0.6 ms at
// the rate of a large copy); a second read of the logits instead of the second
// exponential 0.94 ms.
template <int NPAD>
constexpr int bwdf_centres() { return 12 / (NPAD / 16); }
constexpr int kLDB = 144;  // row of 128 features: 72 dwords, 8 mod 64 banks
template <int NPAD>
constexpr int fused_ld() { return NPAD + 8; }

template <int NPAD>
constexpr size_t bwdf_centre_lds() {
  return sizeof(float4) * NPAD * (2 + NPAD / 16)  // kg, qside, key-side sums per query tile
         + 2 * NPAD * (kLDB + 2 * fused_ld<NPAD>());
}
template <int NPAD>
size_t bwdf_lds() {
  return bwdf_centres<NPAD>() * bwdf_centre_lds<NPAD>();
}

// One 16-row tile of a BF16 pair tensor as load_rows gives it, kept in BF16.
__device__ __forceinline__ void load_rows_b(const float *rows, int col, int ld, int base, int n,
                                            int row, int g, bf16x4 (&v)[8]) {
  const __bf16 *rb = (const __bf16 *)rows + (size_t)base * ld + col;
  const int off = (row < n ? row : 0) * ld + 4 * g;
#pragma unroll
  for (int c = 0; c < 8; ++c) v[c] = *(const bf16x4 *)(rb + off + 16 * c);
}
// The lane's own row into X[row][kLDB]; rows past n as zeros.
__device__ __forceinline__ void store_rows_b(__bf16 *X, int row, bool ok, int g,
                                             const bf16x4 (&v)[8]) {
  const bf16x4 zero = to_bf16(floatx4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
  for (int c = 0; c < 8; ++c) *(bf16x4 *)(X + row * kLDB + 16 * c + 4 * g) = ok ? v[c] : zero;
}
__device__ __forceinline__ bf16x8 pair_b(const bf16x4 &lo, const bf16x4 &hi) {
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
// Rows 4g .. 4g + 3 of column r of a 16 x 16 tile: each lane names four columns
// of one row (row 4g + r / 4, columns 4 (r % 4)), p = tr_at(tile).
__device__ __forceinline__ int tr_at(int ld, int r, int g) {
  return (4 * g + (r >> 2)) * ld + 4 * (r & 3);
}
__device__ __forceinline__ bf16x4 tr_read(const __bf16 *p) {
  typedef short shortx4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) shortx4 *lds_ptr;
  return __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)p));
}
// acc[ft] += contraction over the rows of tiles 'tile' and 'tile' + 1 of X (xt at
// tr_at of X), B operand bt.  Output lane layout: own row r, features 16 ft + 4 g + v.
__device__ __forceinline__ void accum_tr(const __bf16 *xt, int tile, const bf16x8 &bt,
                                         floatx4 (&acc)[8]) {
  const __bf16 *x = xt + tile * 16 * kLDB;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    bf16x4 x0[4], x1[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      x0[f] = tr_read(x + (4 * h + f) * 16);
      x1[f] = tr_read(x + 16 * kLDB + (4 * h + f) * 16);
    }
#pragma unroll
    for (int f = 0; f < 4; ++f)
      acc[4 * h + f] = mfma_bf16x2(pair_b(x0[f], x1[f]), bt, acc[4 * h + f]);
  }
}

// The value of lane i ^ S of the 16 lanes of a group, on the vector ALU: a
// rotation by 8, a permutation of quads, and for 4 a shift up for the even quads
// and one down for the odd ones.  MIRROR: of lane i ^ (2 S - 1) below 8, one
// operation each; any lane across bit S does for a sum, in another order.
template <int S, bool MIRROR>
__device__ __forceinline__ float partner16(float x) {
  if constexpr (S == 4 && !MIRROR) {
    const int v = __builtin_bit_cast(int, x);
    const int lo = __builtin_amdgcn_update_dpp(0, v, 0x104, 0xf, 0x5, false);
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(lo, v, 0x114, 0xf, 0xa, false));
  } else {
    constexpr int kXor2 = MIRROR ? kDppXor3 : 0x4E;
    return dpp<S == 8 ? kDppXor8 : S == 4 ? kDppXor7 : S == 2 ? kXor2 : kDppXor1>(x);
  }
}

// Sum of 16 per-lane values over the 16 lanes of a lane group (those that
// share lane / 16): after four halving steps lane r of the group holds the
// total of value r (30 exchanges instead of 64).  Both halves are exchanged
// and the lane keeps one sum: a select between two array elements would be
// turned into an indexed access and push the array out of registers.  On the
// vector ALU, not through LDS: they were 180 of a wavefront's 480 LDS
// operations in the BF16 adjoint (0.98 -> 0.94 ms a layer), which keeps the
// order it had there; the FP32 one takes the cheaper mirrors.
template <int S, bool MIRROR>
__device__ __forceinline__ void halve16(float (&v)[16], int r) {
  const bool up = (r & S) != 0;
#pragma unroll
  for (int j = 0; j < S; ++j) {
    const float lo = v[j] + partner16<S, MIRROR>(v[j]);
    const float hi = v[j + S] + partner16<S, MIRROR>(v[j + S]);
    v[j] = up ? hi : lo;
  }
}
template <bool MIRROR>
__device__ __forceinline__ float reduce16(float (&v)[16], int r) {
  halve16<8, MIRROR>(v, r);
  halve16<4, MIRROR>(v, r);
  halve16<2, MIRROR>(v, r);
  halve16<1, MIRROR>(v, r);
  return v[0];
}

// Lane indices that the optimiser cannot connect with those of an earlier
// phase, so that no address is kept in registers from one to the next.
#define FRESH_LANES                                    \
  int lane_ = lane;                                    \
  asm volatile("" : "+v"(lane_));                      \
  const int r = lane_ & 15, g = lane_ >> 4;            \
  const int kk = wave * 16 + r;                        \
  const bool kok = kk < n;                             \
  (void)kok;

template <int NPAD>
__global__ __launch_bounds__(768, 3) void k_attn_bwd_f(
    const float *__restrict__ qkv, const float *__restrict__ dO,
    const float *__restrict__ geom, const int *__restrict__ pair_off,
    const int *__restrict__ nnei, const int *__restrict__ clist, const int *__restrict__ ccount,
    float shift, const float *__restrict__ lam, const float2 *__restrict__ fstat,
    float *__restrict__ dqkv, float *__restrict__ gw, float *__restrict__ gr, int accumulate) {
  constexpr int NT = NPAD / 16;
  constexpr int C = bwdf_centres<NPAD>();
  constexpr int LDF = fused_ld<NPAD>();
  extern __shared__ float4 smem[];
  __shared__ unsigned bar[C];  // arrivals at the barriers of each centre
  const int part = __builtin_amdgcn_readfirstlane((int)threadIdx.x / (NT * 64));
  float4 *kg = smem + part * (bwdf_centre_lds<NPAD>() / sizeof(float4));  // [NPAD] rhat, sw
  float4 *qside = kg + NPAD;               // [NPAD] query-side sums of each neighbour
  float4 *ksum = qside + NPAD;             // [NT][NPAD] key-side sums, per query tile
  __bf16 *buf = (__bf16 *)(ksum + NT * NPAD);  // V, K, dO, Q rows in turn
  __bf16 *As = buf + NPAD * kLDB;          // [NPAD][LDF] A = P H
  __bf16 *Ds = As + NPAD * LDF;            // [NPAD][LDF] dS
  const int ld = kQKV * 128;
  const float inv_sqrt_d = 0.08838834764831845f;
  const int cnt = *ccount;
  // the V and dO rows and gate records of a centre are loaded during the dK
  // product of the previous one
  bf16x4 vrow[8], dov[8];
  float4 gv;
  float gl = 0.f;
  int n_nx = 0, base_nx = 0;
  auto fetch = [&](int at, int tid) {  // (past the last centre: that one again)
    const int i = clist[min(at, cnt - 1)];
    n_nx = __builtin_amdgcn_readfirstlane(nnei[i]);
    base_nx = __builtin_amdgcn_readfirstlane(pair_off[i]);
    const int row = (tid >> 6) * 16 + (tid & 15), g = (tid & 63) >> 4;
    load_rows_b(qkv, 256, ld, base_nx, n_nx, row, g, vrow);
    load_rows_b(dO, 0, 128, base_nx, n_nx, row, g, dov);
    gv = gate_load(geom, base_nx, n_nx, tid, gl);
  };
  // part p takes the centres p grids further on: with fewer centres than
  // workgroups every centre has a CU to itself
  const int step = (int)gridDim.x * C;
  const int first = (int)blockIdx.x + part * (int)gridDim.x;
  CentreBarrier<C, NT> barrier(bar, part);
  if (first >= cnt) return;  // one centre's wavefronts, no shared barrier follows
  fetch(first, fresh_tid() - part * NT * 64);
  for (int it = first; it < cnt; it += step) {
    const int tid = fresh_tid() - part * NT * 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int n = n_nx;
    const int base = base_nx;
    const int ntile = (n + 15) >> 4;
    bf16x4 krow[8];  // K, read while dA^T is formed
    {
      FRESH_LANES
      store_rows_b(buf, kk, kok, g, vrow);
      gate_store<NPAD>(kg, nullptr, tid, n, gv, gl);
      load_rows_b(qkv, 128, ld, base, n, kk, g, krow);
    }
    barrier();

    // ---------------- phase Q: dA^T, dS, dQ, A and dS to LDS, both sides' sums
    floatx4 da[NT];  // lane: query r, keys 4g + v
    if (wave < ntile) {
      FRESH_LANES
#pragma unroll
      for (int kt = 0; kt < NT; ++kt) da[kt] = floatx4{0.f, 0.f, 0.f, 0.f};
      const __bf16 *xb = buf + r * kLDB + 4 * g;
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        bf16x4 a0[NT], a1[NT];
#pragma unroll
        for (int kt = 0; kt < NT; ++kt) {
          a0[kt] = *(const bf16x4 *)(xb + kt * 16 * kLDB + 32 * h);
          a1[kt] = *(const bf16x4 *)(xb + kt * 16 * kLDB + 32 * h + 16);
        }
        __builtin_amdgcn_sched_barrier(0);
        const bf16x8 bb = pair_b(dov[2 * h], dov[2 * h + 1]);
#pragma unroll
        for (int kt = 0; kt < NT; ++kt) da[kt] = mfma_bf16x2(pair_b(a0[kt], a1[kt]), bb, da[kt]);
      }
    }
    barrier();
    {
      FRESH_LANES
      store_rows_b(buf, kk, kok, g, krow);
    }
    barrier();
    if (wave < ntile) {
      FRESH_LANES
      const int q = kk;
      const bool qok = kok;
      const int qr = qok ? q : 0;
      const float4 gq = kg[q];
      const float wq = qok ? gq.w : 0.f;
      const float2 fs = fstat[base + qr];
      const float m = fs.x, invz = fs.y;
      const float *lp = lam + (size_t)(base + qr) * kLamLd + 4 * g;
      // pass 1: probabilities P of the query's row, and D_q = sum_k P H dA
      // (= dO . o, without o)
      float dq = 0.f;
      floatx4 lk[NT];  // lam of the query's row; P is formed again in pass 2
#pragma unroll
      for (int kt = 0; kt < NT; ++kt) lk[kt] = *(const floatx4 *)(lp + 16 * kt);
#pragma unroll
      for (int kt = 0; kt < NT; ++kt) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int k = kt * 16 + 4 * g + v;
          const bool ok = qok && k < n;
          const float4 gk = kg[k];
          const float c = gq.x * gk.x + gq.y * gk.y + gq.z * gk.z;
          const float lm = ok ? lk[kt][v] : 0.f;
          const float l = (lm + shift) * (wq * gk.w) - shift;
          const float p = ok ? exp_hw(l - m) * invz : 0.f;
          dq += p * (wq * gk.w * c) * da[kt][v];
          lk[kt][v] = lm;
        }
        asm volatile("" : "+v"(dq));  // summed here, not after the last tile
      }
      dq = sum_groups(dq);
      // pass 2 reads the gates again: with indices that the optimiser
      // knows, it would keep pass 1's values (a hundred registers) instead
      int g2 = g;
      asm volatile("" : "+v"(g2));
      floatx4 dqacc[8];
#pragma unroll
      for (int ft = 0; ft < 8; ++ft) dqacc[ft] = floatx4{0.f, 0.f, 0.f, 0.f};
      float dwq = 0.f, drqx = 0.f, drqy = 0.f, drqz = 0.f;
      const __bf16 *xt = buf + tr_at(kLDB, r, g);
      bf16x4 dsp;  // dS of the even tile of a pair
      // pass 2: the softmax adjoint
#pragma unroll
      for (int kt = 0; kt < NT; ++kt) {
        floatx4 ds, at;
        float ks[16];  // key-side terms: X w_q, Y rhat_q (x, y, z) for the four keys
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int k = kt * 16 + 4 * g2 + v;
          const float4 gk = kg[k];
          const float c = gq.x * gk.x + gq.y * gk.y + gq.z * gk.z;
          const float ww = wq * gk.w;
          const float lm = lk[kt][v];
          const float l = (lm + shift) * (wq * gk.w) - shift;
          const float p = qok && k < n ? exp_hw(l - m) * invz : 0.f;
          const float h = ww * c;
          const float dH = da[kt][v] * p;
          const float dL = p * (da[kt][v] * h - dq);
          ds[v] = dL * ww * inv_sqrt_d;
          at[v] = p * h;
          const float X = fmaf(dH, c, dL * (lm + shift));
          const float Y = dH * ww;
          dwq += X * gk.w;
          drqx += Y * gk.x;
          drqy += Y * gk.y;
          drqz += Y * gk.z;
          ks[v] = X * wq;
          ks[4 + v] = Y * gq.x;
          ks[8 + v] = Y * gq.y;
          ks[12 + v] = Y * gq.z;
        }
        const bf16x4 dsb = to_bf16(ds);
        *(bf16x4 *)(As + q * LDF + kt * 16 + 4 * g) = to_bf16(at);
        *(bf16x4 *)(Ds + q * LDF + kt * 16 + 4 * g) = dsb;
        // lane r now holds the wavefront's total of term r / 4 for key
        // 4g + r % 4 of this tile
        const float kt_sum = reduce16<false>(ks, r);
        ((float *)ksum)[(wave * NPAD + kt * 16 + 4 * g + (r & 3)) * 4 + (r >> 2)] = kt_sum;
        // dQ = dS K, tiles taken in pairs
        if (kt % 2 == 0) dsp = dsb;
        else accum_tr(xt, kt - 1, pair_b(dsp, dsb), dqacc);
      }
      dwq = sum_groups(dwq);
      drqx = sum_groups(drqx);
      drqy = sum_groups(drqy);
      drqz = sum_groups(drqz);
      if (g == 0 && qok) qside[q] = make_float4(dwq, drqx, drqy, drqz);
      if (qok) {
        float *dp = pt_at<true>(dqkv, (size_t)(base + q) * ld + 4 * g);
#pragma unroll
        for (int ft = 0; ft < 8; ++ft) stp4<true>(dp, 16 * ft, dqacc[ft]);
      }
    }
    barrier();
    bf16x4 qrow[8];  // Q, read while dV is formed
    {
      FRESH_LANES
      store_rows_b(buf, kk, kok, g, dov);
      load_rows_b(qkv, 0, ld, base, n, kk, g, qrow);
    }
    barrier();

    // ---------------- phase K: dV = A^T dO, dK = dS^T Q, key-side sums
    const bf16x4 zero = to_bf16(floatx4{0.f, 0.f, 0.f, 0.f});
    if (wave < ntile) {
      FRESH_LANES
      floatx4 dvacc[8];
#pragma unroll
      for (int ft = 0; ft < 8; ++ft) dvacc[ft] = floatx4{0.f, 0.f, 0.f, 0.f};
      const __bf16 *at = As + tr_at(LDF, r, g) + wave * 16;  // lane: key r, queries 4g + v
      const __bf16 *xt = buf + tr_at(kLDB, r, g);
      // tiles in pairs; A of query tiles at or past ntile (not written for this
      // centre) is zero
#pragma unroll
      for (int qt = 0; qt < NT; qt += 2) {
        if (qt >= ntile) continue;
        const bf16x4 a0 = tr_read(at + qt * 16 * LDF), a1 = tr_read(at + (qt + 1) * 16 * LDF);
        accum_tr(xt, qt, pair_b(a0, qt + 1 < ntile ? a1 : zero), dvacc);
      }
      if (kok) {
        float *dp = pt_at<true>(dqkv, (size_t)(base + kk) * ld + 256 + 4 * g);
#pragma unroll
        for (int ft = 0; ft < 8; ++ft) stp4<true>(dp, 16 * ft, dvacc[ft]);
      }
    }
    barrier();
    {
      FRESH_LANES
      store_rows_b(buf, kk, kok, g, qrow);
    }
    barrier();
    fetch(it + step, fresh_tid() - part * NT * 64);
    if (wave < ntile) {
      FRESH_LANES
      floatx4 dkacc[8];
#pragma unroll
      for (int ft = 0; ft < 8; ++ft) dkacc[ft] = floatx4{0.f, 0.f, 0.f, 0.f};
      const __bf16 *dt = Ds + tr_at(LDF, r, g) + wave * 16;
      const __bf16 *xt = buf + tr_at(kLDB, r, g);
#pragma unroll
      for (int qt = 0; qt < NT; qt += 2) {
        if (qt >= ntile) continue;
        const bf16x4 d0 = tr_read(dt + qt * 16 * LDF), d1 = tr_read(dt + (qt + 1) * 16 * LDF);
        accum_tr(xt, qt, pair_b(d0, qt + 1 < ntile ? d1 : zero), dkacc);
      }
      if (kok) {
        float *dp = pt_at<true>(dqkv, (size_t)(base + kk) * ld + 128 + 4 * g);
#pragma unroll
        for (int ft = 0; ft < 8; ++ft) stp4<true>(dp, 16 * ft, dkacc[ft]);
        if (g == 0) {
          float4 t = qside[kk];
          for (int w = 0; w < ntile; ++w) {
            const float4 kv = ksum[w * NPAD + kk];
            t.x += kv.x;
            t.y += kv.y;
            t.z += kv.z;
            t.w += kv.w;
          }
          const size_t p = (size_t)(base + kk);
          if (accumulate) {
            gw[p] += t.x;
            gr[4 * p + 0] += t.y;
            gr[4 * p + 1] += t.z;
            gr[4 * p + 2] += t.w;
          } else {
            gw[p] = t.x;
            gr[4 * p + 0] = t.y;
            gr[4 * p + 1] = t.z;
            gr[4 * p + 2] = t.w;
            gr[4 * p + 3] = 0.f;
          }
        }
      }
    }
    barrier();  // LDS is restaged for the next centre
  }
}

// ---------------------------------------------------- adjoint, split operands
//
// The FP32 adjoint of a centre on two-term f16 operands (split.h), two centres of
// the 96 class to a workgroup and one of the others.  Wavefront = tile of 16 keys: with its own V rows as the
// MFMA's column operand and dO in LDS, dA comes out as lane (key r, queries
// 4g + v), which is the column operand of dV = A^T dO and dK = dS^T Q as it
// stands; only dS goes through LDS, for dQ = dS K (wavefront = tile of 16
// queries).  dO is staged once for both dA and dV, V not at all, and A never
// leaves registers.  The sums over keys (D_q = sum_k A dA, and the query-side
// switch and direction gradients) are reduced over a wavefront's 16 keys by
// lane exchanges and over wavefronts through LDS in a fixed order.
//
// Rows staged in LDS carry their own power-of-two scale; where rows are
// contracted over, the scale is folded into the other operand, whose row then
// takes a scale of its own.
//
// LDS holds, one after the other, dO rows, Q rows, and dS beside the K rows in
// two halves of 64 features: 80 KB for the 96 class, so that a CU holds two
// centres.  They share one workgroup of 12 wavefronts, three on every SIMD: two
// workgroups of six would each put two wavefronts on the first SIMDs, four
// there in all, which their registers do not allow (measured: the second
// waits).  The two centres have barriers of their own (with the workgroup's
// barrier they wait for each other's phases: 1.62 ms against 1.41).
//
// Per layer at 15,668 centres of 84 neighbours: FP32 MFMAs with A and dS in LDS
// (141 KB, one centre per CU) 2.30 ms, this 1.43 ms for 5.3 GB, three quarters
// of what a plain copy reaches; at 3,800 centres of 107 neighbours (the
// 128 class, one centre of eight wavefronts per CU) 0.84 ms in two FP32
// kernels, 0.56 ms here.
template <int NPAD>
constexpr int split_ds_ld() { return NPAD + 4; }
constexpr int kLDH = 68;  // row stride of half the features: 64 + 4

template <int NPAD>
constexpr int split_main_floats() {
  constexpr int rows = NPAD * kLDR, halves = NPAD * (split_ds_ld<NPAD>() + kLDH);
  return rows > halves ? rows : halves;
}
// Centres of a workgroup: two of the 96 class (12 wavefronts, three per SIMD).
template <int NPAD>
constexpr int bwds_centres() { return NPAD == 96 ? 2 : 1; }
template <int NPAD>
constexpr int bwds_threads() { return bwds_centres<NPAD>() * NPAD / 16 * 64; }
template <int NPAD>
constexpr size_t bwds_lds() {
  constexpr int W = NPAD / 16;
  return bwds_centres<NPAD>() *
         (sizeof(float4) * NPAD * (1 + W)               // kg, query-side sums per key tile
          + (sizeof(double) + sizeof(float2)) * NPAD    // kw, softmax statistics
          // row scales, D_q per key tile (then the key-side sums) and whole
          + sizeof(float) * NPAD * (2 + (W > 4 ? W : 4))
          + sizeof(float) * split_main_floats<NPAD>());
}

// One 16-row tile as load_rows gives it, from a wave-uniform base with 32-bit
// offsets.
__device__ __forceinline__ void load_own(const float *rows, int ld, int row, int n, int g,
                                         floatx4 (&v)[8]) {
  const unsigned off = (unsigned)((row < n ? row : 0) * ld + 4 * g);
#pragma unroll
  for (int c = 0; c < 8; ++c) v[c] = *(const floatx4 *)(rows + off + 16 * c);
}

// Own rows, scaled and packed; rows that do not exist become zeros.
__device__ __forceinline__ float pack_rows(const floatx4 (&v)[8], bool ok, split::packx4 (&p)[8]) {
  float m = 0.f;
#pragma unroll
  for (int c = 0; c < 8; ++c) m = split::max_abs(m, v[c]);
  const split::Scale sc = split::scale_of(split::row_max(m));
  const split::packx4 z = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const split::packx4 x = split::pack(v[c] * sc.up);
    p[c] = ok ? x : z;
  }
  return sc.down;
}

// The column operand of a contraction over neighbours: b[kt][v] times the row
// scales of the other operand, with one scale for the whole column; returns
// its inverse.
template <int NT>
__device__ __forceinline__ float pack_column(const floatx4 (&b)[NT], const float *scl, int g,
                                             split::packx4 (&p)[NT]) {
  floatx4 x[NT];
  float m = 0.f;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    x[t] = b[t] * *(const floatx4 *)(scl + 16 * t + 4 * g);
    m = split::max_abs(m, x[t]);
  }
  const split::Scale sc = split::scale_of(split::row_max(m));
#pragma unroll
  for (int t = 0; t < NT; ++t) p[t] = split::pack(x[t] * sc.up);
  return sc.down;
}

// acc[f] = sum over the rows of X of X^T b for NF feature tiles f
// (X packed, row-major, row stride LD, first feature at X): lane own row r,
// features 16 f + 4 g + v.  Operands are read for four tiles at a time.
template <int NT, int NF, int LD>
__device__ __forceinline__ void contract_rows(const float *X, int r, int g,
                                              const split::packx4 (&b)[NT],
                                              floatx4 (&acc)[NF]) {
#pragma unroll
  for (int f = 0; f < NF; ++f) acc[f] = floatx4{0.f, 0.f, 0.f, 0.f};
  const uint32_t *xb = (const uint32_t *)X + 4 * g * LD + r;
#pragma unroll
  for (int qt = 0; qt < NT; ++qt) {
    const split::halfx8 lo = split::dup_lo(b[qt]), hi = split::dup_hi(b[qt]);
#pragma unroll
    for (int h = 0; h < NF; h += 4) {
      split::packx4 x[4];
#pragma unroll
      for (int f = 0; f < 4; ++f)
#pragma unroll
        for (int t = 0; t < 4; ++t) x[f][t] = xb[(16 * qt + t) * LD + 16 * (h + f)];
#pragma unroll
      for (int f = 0; f < 4; ++f) acc[h + f] = split::mfma(x[f], lo, acc[h + f]);
#pragma unroll
      for (int f = 0; f < 4; ++f) acc[h + f] = split::mfma(x[f], hi, acc[h + f]);
    }
    __builtin_amdgcn_sched_barrier(0);  // one tile's operands live at a time
  }
}
template <int NF>
__device__ __forceinline__ void store_rows(float *out, bool ok, const floatx4 (&acc)[NF],
                                           float down) {
  if (ok) {
#pragma unroll
    for (int f = 0; f < NF; ++f) *(floatx4 *)(out + 16 * f) = acc[f] * down;
  }
}

template <int NPAD>
__global__ __launch_bounds__(bwds_threads<NPAD>(), NPAD <= 96 ? 3 : 2) void k_attn_bwd_s(
    const float *__restrict__ qkv, const float *__restrict__ dO,
    const float *__restrict__ geom, const int *__restrict__ pair_off,
    const int *__restrict__ nnei, const int *__restrict__ clist, const int *__restrict__ ccount,
    float shift, const float *__restrict__ lam, const float2 *__restrict__ fstat,
    float *__restrict__ dqkv, float *__restrict__ gw, float *__restrict__ gr, int accumulate) {
  constexpr int NT = NPAD / 16;
  constexpr int LDD = split_ds_ld<NPAD>();
  constexpr int C = bwds_centres<NPAD>();
  extern __shared__ float4 smem[];
  __shared__ unsigned bar[C];  // arrivals at the barriers of each centre
  const int part = C == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / (NT * 64));
  float4 *kg = smem + part * (bwds_lds<NPAD>() / C / sizeof(float4));  // [NPAD] rhat, sw
  float4 *qsum = kg + NPAD;                         // [NT][NPAD] query-side sums per key tile
  double *kw = (double *)(qsum + NT * NPAD);        // [NPAD] switch values in FP64
  float2 *stats = (float2 *)(kw + NPAD);            // [NPAD] m, 1/Z
  float *scl = (float *)(stats + NPAD);             // [NPAD] inverse scales of the staged rows
  float *dqs = scl + NPAD;                          // [NT][NPAD] D_q per key tile
  float4 *kside = (float4 *)dqs;                    // [NPAD] key-side sums, in its place
  float *dqt = dqs + (NT > 4 ? NT : 4) * NPAD;      // [NPAD] D_q
  float *buf = dqt + NPAD;                          // dO rows, Q rows
  float *Ds = buf;                                  // [NPAD][LDD] dS, beside
  float *kh = buf + NPAD * LDD;                     // [NPAD][kLDH] half the features of K
  const int ld = kQKV * 128;
  const float inv_sqrt_d = 0.08838834764831845f;
  const int cnt = *ccount;
  // dO and V rows and the gate record of a centre are loaded during the last
  // product of the previous one
  floatx4 rows[8], vrows[8];
  float4 gv;
  float2 fs;
  float gl = 0.f;
  int n_nx = 0, base_nx = 0;
  auto fetch = [&](int at, int tid) {  // (past the last centre: that one again)
    const int i = clist[min(at, cnt - 1)];
    n_nx = __builtin_amdgcn_readfirstlane(nnei[i]);
    base_nx = __builtin_amdgcn_readfirstlane(pair_off[i]);
    const int row = (tid >> 6) * 16 + (tid & 15), g = (tid & 63) >> 4;
    load_own(dO + (size_t)base_nx * 128, 128, row, n_nx, g, rows);
    load_own(qkv + (size_t)base_nx * ld + 256, ld, row, n_nx, g, vrows);
    gv = gate_load(geom, base_nx, n_nx, tid, gl);
    fs = fstat[base_nx + (tid < n_nx ? tid : 0)];
  };
  // part 1 takes the centres one grid further on: with fewer centres than
  // workgroups every centre has a CU to itself
  const int step = (int)gridDim.x * C;
  const int first = (int)blockIdx.x + part * (int)gridDim.x;
  CentreBarrier<C, NT> barrier(bar, part);
  if (first >= cnt) return;  // one centre's wavefronts, no shared barrier follows
  fetch(first, fresh_tid() - part * NT * 64);
  for (int it = first; it < cnt; it += step) {
    const int tid = fresh_tid() - part * NT * 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int r = lane & 15, g = lane >> 4;
    const int n = n_nx;
    const int base = base_nx;
    const float *qb = qkv + (size_t)base * ld;
    const int kk = wave * 16 + r;  // own row: key, and query of the last product
    const bool kok = kk < n;
    float *db = dqkv + (size_t)base * ld;
    split::packx4 own[8];
    {
      const float down = pack_rows(rows, kok, own);
      if (g == 0) scl[kk] = down;
#pragma unroll
      for (int c = 0; c < 8; ++c) *(split::packx4 *)(buf + kk * kLDR + 16 * c + 4 * g) = own[c];
    }
    gate_store<NPAD>(kg, kw, tid, n, gv, gl);
    if (tid < NPAD) stats[tid] = fs;
    // logits of this key against the queries of every tile
    const float *lc = lam + (size_t)base * kLamLd;
    auto lam_tile = [&](int qt, int kk, int g) {
      floatx4 l;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int q = qt * 16 + 4 * g + v;
        l[v] = lc[(unsigned)((q < n ? q : 0) * kLamLd + (kk < n ? kk : 0))];
      }
      return l;
    };
    floatx4 lm[NT];
#pragma unroll
    for (int qt = 0; qt < NT; ++qt) lm[qt] = lam_tile(qt, kk, g);
    const float iv = pack_rows(vrows, true, own);
    barrier();

    // ---------------- dA, P, D_q
    floatx4 da[NT], pk[NT];
    {
#pragma unroll
      for (int qt = 0; qt < NT; ++qt) da[qt] = floatx4{0.f, 0.f, 0.f, 0.f};
      const float *xb = buf + r * kLDR + 4 * g;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        split::packx4 x[NT];
#pragma unroll
        for (int qt = 0; qt < NT; ++qt)
          x[qt] = *(const split::packx4 *)(xb + qt * 16 * kLDR + 16 * c);
        __builtin_amdgcn_sched_barrier(0);
        const split::halfx8 lo = split::dup_lo(own[c]), hi = split::dup_hi(own[c]);
#pragma unroll
        for (int qt = 0; qt < NT; ++qt) da[qt] = split::mfma(x[qt], lo, da[qt]);
#pragma unroll
        for (int qt = 0; qt < NT; ++qt) da[qt] = split::mfma(x[qt], hi, da[qt]);
      }
      const float4 gk = kg[kk];
      const double wkd = kok ? kw[kk] : 0.0;
#pragma unroll
      for (int qt = 0; qt < NT; ++qt) {
        const floatx4 sq = *(const floatx4 *)(scl + qt * 16 + 4 * g);
        floatx4 part;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int q = qt * 16 + 4 * g + v;
          const bool ok = kok && q < n;
          const float4 gq = kg[q];
          const float2 sm = stats[q];
          const float c = gq.x * gk.x + gq.y * gk.y + gq.z * gk.z;
          const float l = logit64(ok ? lm[qt][v] : 0.f, kw[q], wkd, shift);
          const float p = ok ? exp_hw(l - sm.x) * sm.y : 0.f;
          const float d = ok ? da[qt][v] * iv * sq[v] : 0.f;
          da[qt][v] = d;
          pk[qt][v] = p;
          part[v] = sum16(p * (gq.w * gk.w * c) * d);
        }
        if (r == 0) *(floatx4 *)(dqs + wave * NPAD + qt * 16 + 4 * g) = part;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    barrier();
    if (tid < NPAD) {
      float t = 0.f;
#pragma unroll
      for (int w = 0; w < NT; ++w) t += dqs[w * NPAD + tid];
      dqt[tid] = t;
    }
    barrier();

    // ---------------- softmax adjoint: A^T in pk, dS^T in da; both sides' sums.
    // The logits come from L2 a second time, one tile ahead: kept since the
    // first pass they would push the 96 class past its 168 registers, and a
    // spilled register's reload waits for every load and store before it.
    {
      FRESH_LANES
      float dwk = 0.f, drx = 0.f, dry = 0.f, drz = 0.f;  // key-side sums
      const float4 gk = kg[kk];
      const float wk = kok ? gk.w : 0.f;
      floatx4 lcur = lam_tile(0, kk, g);
#pragma unroll
      for (int qt = 0; qt < NT; ++qt) {
        const floatx4 lnxt = lam_tile(qt + 1 < NT ? qt + 1 : qt, kk, g);
        const floatx4 dq = *(const floatx4 *)(dqt + qt * 16 + 4 * g);
        float qs[16];  // query-side terms X w_k, Y rhat_k of the four queries
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int q = qt * 16 + 4 * g + v;
          const bool ok = kok && q < n;
          const float4 gq = kg[q];
          const float c = gq.x * gk.x + gq.y * gk.y + gq.z * gk.z;
          const float ww = gq.w * wk;
          const float p = pk[qt][v];
          const float h = ww * c;
          const float dH = da[qt][v] * p;
          const float dL = ok ? p * (da[qt][v] * h - dq[v]) : 0.f;
          const float X = dL * ((ok ? lcur[v] : 0.f) + shift) + dH * c;
          const float Y = dH * ww;
          pk[qt][v] = p * h;
          da[qt][v] = dL * ww * inv_sqrt_d;
          dwk += X * gq.w;
          drx += Y * gq.x;
          dry += Y * gq.y;
          drz += Y * gq.z;
          qs[v] = X * wk;
          qs[4 + v] = Y * gk.x;
          qs[8 + v] = Y * gk.y;
          qs[12 + v] = Y * gk.z;
        }
        // lane r now holds the tile's total of term r / 4 for query 4g + r % 4
        const float t = reduce16<true>(qs, r);
        ((float *)qsum)[(wave * NPAD + qt * 16 + 4 * g + (r & 3)) * 4 + (r >> 2)] = t;
        lcur = lnxt;
        __builtin_amdgcn_sched_barrier(0);
      }
      dwk = sum_groups(dwk);
      drx = sum_groups(drx);
      dry = sum_groups(dry);
      drz = sum_groups(drz);
      // (every wavefront is past the D_q sums)
      if (g == 0) kside[kk] = make_float4(dwk, drx, dry, drz);
      // dV = A^T dO
      split::packx4 bp[NT];
      const float down = pack_column<NT>(pk, scl, g, bp);
      floatx4 acc[8];
      contract_rows<NT, 8, kLDR>(buf, r, g, bp, acc);
      // Q on its way to LDS, ahead of the stores (a wait for loads waits for
      // every store issued before them)
      load_own(qb, ld, kk, n, g, rows);
      store_rows(db + (unsigned)(kk * ld + 4 * g) + 256, kok, acc, down);
    }
    barrier();

    // ---------------- dK = dS^T Q
    {
      FRESH_LANES
      const float down = pack_rows(rows, kok, own);
      if (g == 0) scl[kk] = down;
#pragma unroll
      for (int c = 0; c < 8; ++c) *(split::packx4 *)(buf + kk * kLDR + 16 * c + 4 * g) = own[c];
    }
    {
      FRESH_LANES
      load_own(qb + 128, ld, kk, n, g, rows);  // K
    }
    barrier();
    {
      FRESH_LANES
      split::packx4 bp[NT];
      const float down = pack_column<NT>(da, scl, g, bp);
      floatx4 acc[8];
      contract_rows<NT, 8, kLDR>(buf, r, g, bp, acc);
      store_rows(db + (unsigned)(kk * ld + 4 * g) + 128, kok, acc, down);
    }
    barrier();

    // ---------------- dQ = dS K, 64 features at a time
    {
      FRESH_LANES
      const float down = pack_rows(rows, kok, own);
      if (g == 0) scl[kk] = down;
#pragma unroll
      for (int c = 0; c < 4; ++c) *(split::packx4 *)(kh + kk * kLDH + 16 * c + 4 * g) = own[c];
    }
    {
#pragma unroll
      for (int qt = 0; qt < NT; ++qt)
#pragma unroll
        for (int v = 0; v < 4; ++v) Ds[(qt * 16 + 4 * g + v) * LDD + kk] = da[qt][v];
    }
    barrier();
    split::packx4 bp[NT];
    float down = 0.f;
    float gw0 = 0.f;  // the other layers' share of dE/dsw, dE/drhat
    float4 gr0 = make_float4(0.f, 0.f, 0.f, 0.f);
    {
      FRESH_LANES
      if (accumulate) {
        gw0 = gw[base + (kok ? kk : 0)];
        gr0 = *(const float4 *)(gr + 4 * (size_t)(base + (kok ? kk : 0)));
      }
      floatx4 x[NT];
#pragma unroll
      for (int kt = 0; kt < NT; ++kt)
        x[kt] = *(const floatx4 *)(Ds + kk * LDD + kt * 16 + 4 * g);
      down = pack_column<NT>(x, scl, g, bp);
      floatx4 acc[4];
      contract_rows<NT, 4, kLDH>(kh, r, g, bp, acc);
      store_rows(db + (unsigned)(kk * ld + 4 * g), kok, acc, down);
    }
    barrier();
#pragma unroll
    for (int c = 0; c < 4; ++c) *(split::packx4 *)(kh + kk * kLDH + 16 * c + 4 * g) = own[4 + c];
    // unconditional, also after the last centre: under a branch the old rows
    // would stay live to the end of the loop
    fetch(it + step, tid);
    barrier();
    {
      FRESH_LANES
      // (the operand's duplicates are formed again rather than kept)
#pragma unroll
      for (int kt = 0; kt < NT; ++kt) asm volatile("" : "+v"(bp[kt]));
      floatx4 acc[4];
      contract_rows<NT, 4, kLDH>(kh, r, g, bp, acc);
      store_rows(db + (unsigned)(kk * ld + 4 * g) + 64, kok, acc, down);
      if (kok && g == 0) {
        float4 t = kside[kk];
#pragma unroll
        for (int w = 0; w < NT; ++w) {
          const float4 q = qsum[w * NPAD + kk];
          t.x += q.x;
          t.y += q.y;
          t.z += q.z;
          t.w += q.w;
        }
        gw[base + kk] = gw0 + t.x;
        *(float4 *)(gr + 4 * (size_t)(base + kk)) = make_float4(gr0.x + t.y, gr0.y + t.z, gr0.z + t.w, 0.f);
      }
    }
    barrier();  // LDS is restaged for the next centre
  }
}

// Class lists: centre i with n = nnei[i] > 0 belongs to class (n - 1) / 32
// (counted in ccount[4 + class]) and is listed in the smallest class of the
// active set (bit c of `active`) that holds n neighbours; the host keeps the
// top class active, so every centre is listed.  A class that is not active
// is not launched: the host deactivates classes that were empty in an
// earlier step, and a centre that falls into one after all is computed by
// the next larger active class (more padding, the same result: in BF16 the
// host keeps the largest class of the fused adjoint active, so the fallback
// never changes the kind of adjoint).  Positions
// are taken with one atomic per wavefront and class, so the order inside a
// list varies from run to run; every centre is computed on its own, so
// results do not depend on it.
__global__ void k_attn_classes(const int *__restrict__ nnei, int nloc, int active,
                               int *__restrict__ ccount, int *__restrict__ clist) {
  attn_class_lists(blockIdx.x * blockDim.x + threadIdx.x, nnei, nloc, active, ccount, clist);
}

// ------------------------------------------------------------------ descriptor

// T[c][m] = (1/sel) sum_j R~_j[c] G_j[m];  D[m][a] = sum_c T[c][m] T[c][a].
__global__ __launch_bounds__(128) void k_desc_fwd(const float *__restrict__ geom,
                                                  const float *__restrict__ G, int ldg,
                                                  const int *__restrict__ pair_off,
                                                  const int *__restrict__ nnei, int sel, int M,
                                                  int axis, float *__restrict__ T,
                                                  float *__restrict__ dmat, int ldd) {
  __shared__ float Ts[4][128];
  const int i = blockIdx.x;
  const int n = nnei[i];
  const int base = pair_off[i];
  const int m = threadIdx.x;
  float t0 = 0.f, t1 = 0.f, t2 = 0.f, t3 = 0.f;
  if (m < M) {
#pragma unroll 4
    for (int j = 0; j < n; ++j) {
      const float *gp = geom + (size_t)(base + j) * kGeom;
      const float s = gp[G_S];
      const float gm = G[(size_t)(base + j) * ldg + m];
      t0 += s * gm;
      t1 += s * gp[G_RX] * gm;
      t2 += s * gp[G_RY] * gm;
      t3 += s * gp[G_RZ] * gm;
    }
    const float inv = 1.0f / (float)sel;
    t0 *= inv;
    t1 *= inv;
    t2 *= inv;
    t3 *= inv;
    float *tp = T + (size_t)i * 4 * M;
    tp[m] = t0;
    tp[M + m] = t1;
    tp[2 * M + m] = t2;
    tp[3 * M + m] = t3;
  }
  Ts[0][m] = t0;
  Ts[1][m] = t1;
  Ts[2][m] = t2;
  Ts[3][m] = t3;
  __syncthreads();
  if (m < M) {
    float *dp = dmat + (size_t)i * ldd + (size_t)m * axis;
    for (int a = 0; a < axis; ++a)
      dp[a] = t0 * Ts[0][a] + t1 * Ts[1][a] + t2 * Ts[2][a] + t3 * Ts[3][a];
  }
  // zero the row padding of the descriptor matrix
  for (int c = M * axis + m; c < ldd; c += blockDim.x) dmat[(size_t)i * ldd + c] = 0.f;
}

// dT[c][m] = sum_a dD[m][a] T[c][a] + [m < axis] sum_m' dD[m'][m] T[c][m'];
// per pair: dG_j = (1/sel) R~_j dT, dR~_j = (1/sel) dT G_j, then the
// layer-norm backward of the last attention layer (ln_mode 0), the tanh
// backward of the last embedding layer (ln_mode 1), or dG only (ln_mode 2).
// Sixteen lanes share a pair (lane li holds features li + 16k), so the row
// reductions take four cross-lane steps and four pairs run per wavefront.
// KF features per lane (16 lanes x KF >= ldg); LN_MODE as ln_mode below, fixed
// at compile time so that operands a mode does not use are never loaded.
template <int KF, int LN_MODE>
__global__ __launch_bounds__(256) void k_desc_bwd(
    const float *__restrict__ geom, const float *__restrict__ G, int ldg,
    const float *__restrict__ T, const float *__restrict__ dD, int ldd,
    const int *__restrict__ pair_off, const int *__restrict__ nnei, int sel, int M, int axis,
    const float *__restrict__ gamma, const float *__restrict__ xhat,
    const float *__restrict__ rstd, const float *__restrict__ temb, float *__restrict__ dG,
    float *__restrict__ dnext, float *__restrict__ dRt) {
  constexpr int ln_mode = LN_MODE;
  __shared__ float Ts[4][128];
  __shared__ float dTs[4][128];
  __shared__ float part[16][16][4];
  __shared__ float gam[128];  // gamma of the layer norm (ln_mode 0), zeros past M
  const int i = blockIdx.x;
  const int n = nnei[i];
  const int base = pair_off[i];
  const int tid = threadIdx.x;
  if (tid < 128) {
    for (int c = 0; c < 4; ++c) Ts[c][tid] = tid < M ? T[(size_t)i * 4 * M + c * M + tid] : 0.f;
    gam[tid] = (ln_mode == 0 && tid < M) ? gamma[tid] : 0.f;
  }
  __syncthreads();
  const float *dr = dD + (size_t)i * ldd;
  // second term, spread over all threads: a = tid % 16, rows m' = tid/16 + 16k
  {
    const int aa = tid & 15, pp = tid >> 4;
    float q0 = 0.f, q1 = 0.f, q2 = 0.f, q3 = 0.f;
    if (aa < axis) {
      for (int mm = pp; mm < M; mm += 16) {
        const float x = dr[mm * axis + aa];
        q0 += x * Ts[0][mm];
        q1 += x * Ts[1][mm];
        q2 += x * Ts[2][mm];
        q3 += x * Ts[3][mm];
      }
    }
    part[pp][aa][0] = q0;
    part[pp][aa][1] = q1;
    part[pp][aa][2] = q2;
    part[pp][aa][3] = q3;
  }
  __syncthreads();
  const float inv = 1.0f / (float)sel;
  if (tid < 128) {
    float d0 = 0.f, d1 = 0.f, d2 = 0.f, d3 = 0.f;
    if (tid < M) {
      for (int a = 0; a < axis; ++a) {
        const float x = dr[tid * axis + a];
        d0 += x * Ts[0][a];
        d1 += x * Ts[1][a];
        d2 += x * Ts[2][a];
        d3 += x * Ts[3][a];
      }
      if (tid < axis && tid < 16) {
        for (int pp = 0; pp < 16; ++pp) {
          d0 += part[pp][tid][0];
          d1 += part[pp][tid][1];
          d2 += part[pp][tid][2];
          d3 += part[pp][tid][3];
        }
      }
    }
    dTs[0][tid] = d0 * inv;
    dTs[1][tid] = d1 * inv;
    dTs[2][tid] = d2 * inv;
    dTs[3][tid] = d3 * inv;
  }
  __syncthreads();
  const int grp = tid >> 4, li = tid & 15;
  const float invm = 1.0f / (float)M;
  // Every global load of a pair is issued before any of its values is used
  // and is unconditional: feature indices are clamped to the row (columns
  // past M hold zeros).
  for (int j = grp; j < n; j += 16) {
    const size_t p = (size_t)(base + j);
    const float4 gq = *(const float4 *)(geom + p * kGeom);  // s, rx, ry, rz
    float gm[KF], xv[KF], tv[KF];
#pragma unroll
    for (int k = 0; k < KF; ++k) {
      const int m = li + 16 * k;
      const int mc = m < ldg ? m : 0;
      gm[k] = G[p * ldg + mc];
      xv[k] = ln_mode == 0 ? xhat[p * ldg + mc] : 0.f;
      tv[k] = ln_mode == 1 ? temb[p * ldg + mc] : 0.f;
    }
    const float rs = ln_mode == 0 ? rstd[p] : 0.f;
    const float R0 = gq.x, R1 = gq.x * gq.y, R2 = gq.x * gq.z, R3 = gq.x * gq.w;
    float dg[KF];
    float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f, s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int k = 0; k < KF; ++k) {
      const int m = li + 16 * k;
      const int mc = m < 128 ? m : 0;
      const bool in = m < M;
      const float v = R0 * dTs[0][mc] + R1 * dTs[1][mc] + R2 * dTs[2][mc] + R3 * dTs[3][mc];
      const float gmv = in ? gm[k] : 0.f;
      dg[k] = in ? v : 0.f;
      a0 += gmv * dTs[0][mc];
      a1 += gmv * dTs[1][mc];
      a2 += gmv * dTs[2][mc];
      a3 += gmv * dTs[3][mc];
      const float dx = gam[mc] * dg[k];
      s1 += dx;
      s2 += in ? dx * xv[k] : 0.f;
    }
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) {
      a0 += __shfl_xor(a0, off);
      a1 += __shfl_xor(a1, off);
      a2 += __shfl_xor(a2, off);
      a3 += __shfl_xor(a3, off);
      s1 += __shfl_xor(s1, off);
      s2 += __shfl_xor(s2, off);
    }
#pragma unroll
    for (int k = 0; k < KF; ++k) {
      const int m = li + 16 * k;
      if (m < ldg) {
        const int mc = m < 128 ? m : 0;
        const float ln = rs * (gam[mc] * dg[k] - s1 * invm - xv[k] * s2 * invm);
        const float th = dg[k] * (1.0f - tv[k] * tv[k]);
        const float nx = m < M ? (ln_mode == 0 ? ln : th) : 0.f;
        dG[p * ldg + m] = dg[k];
        if (ln_mode != 2) dnext[p * ldg + m] = nx;
      }
    }
    if (li == 0) *(float4 *)(dRt + 4 * p) = make_float4(a0, a1, a2, a3);
  }
}

// The descriptor adjoint fused with the adjoint of the last attention
// layer's output projection (Sec. II-B, DPA-1).  Per centre dT is formed as
// in k_desc_bwd; then each wavefront takes 16-neighbour tiles and forms, per
// pair, the residual-path gradient dG = R~ dT / sel, dR~ = dT G / sel, the
// layer-norm adjoint d(acc) of the pre-norm projection output, and finally
// dO = d(acc) W_O^T on the matrix cores with W_O^T resident in LDS.  d(acc)
// is produced in registers already in the operand layout of that product
// (lane l: pair l % 16, features 16 c + 4 (l / 16) + {0..3}), so it never
// reaches memory.  Blocks walk over centres (persistent grid), so W_O^T is
// staged once per workgroup.
//
// Shape: ldg = 112 (seven 16-feature chunks) and 96 < M <= 100, so the last
// chunk holds M - 96 real features: lane group g carries feature 96 + g of
// it, in one matrix-core step of depth four (FP32) or in the first operand
// slot of the last chunk pair (BF16).
constexpr int kDoN = 128;            // attention width: rows of W_O^T, columns of dO
constexpr int kDoK = 112;            // padded feature width of G
constexpr int kDoLdw = kDoK + 4;     // LDS row stride of W_O^T
constexpr int kDoDs = 17;            // LDS row stride of a centre's dD (axis <= 16)
constexpr int kDoLds = kDoN * kDoLdw + 4 * 128 * 2 + 16 * 16 * 4 + 128 + 1712;  // floats

struct DescOprojArgs {
  const float *geom, *G, *T, *dD;
  const int *pair_off, *nnei;
  int nloc, sel, M, axis, ldd;
  const float *gamma, *xhat, *rstd;
  const float *Wt;  // [kDoN][kDoK]: W_O^T of the last attention layer
  float *dG, *dRt;
  float *dO;        // [pairs][kDoN]: FP32, or BF16 (rounded to nearest even) when BF
};

template <bool BF>
__global__ __launch_bounds__(256, 2) void k_desc_oproj_bwd(DescOprojArgs a) {
  extern __shared__ float sm[];
  float *wsm = sm;                        // [kDoN][kDoLdw]
  float *Ts = wsm + kDoN * kDoLdw;        // [4][128]
  float *dTs = Ts + 4 * 128;              // [4][128]
  float *part = dTs + 4 * 128;            // [16][16][4]
  float *gam = part + 16 * 16 * 4;        // [128], zeros past M
  float *dDs = gam + 128;                 // [M][kDoDs]: the centre's dD
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int M = a.M, axis = a.axis;
  for (int idx = tid; idx < kDoN * (kDoK / 4); idx += 256) {
    const int n = idx / (kDoK / 4), c4 = idx % (kDoK / 4);
    *(float4 *)(wsm + n * kDoLdw + 4 * c4) = *(const float4 *)(a.Wt + (size_t)n * kDoK + 4 * c4);
  }
  if (tid < 128) gam[tid] = tid < M ? a.gamma[tid] : 0.f;
  const float inv = 1.0f / (float)a.sel;
  const float invm = 1.0f / (float)M;
  const int f6 = 96 + g;                  // this lane's feature of the last chunk
  const bool in6 = f6 < M;
  // A centre's dD row (ldd <= 512 float4) and T column tid arrive in
  // registers one centre ahead (issued while the current centre's tiles run)
  // and are then staged in LDS.
  const int nq = a.ldd >> 2;
  float4 dq[2];
  float tq[4];
  auto fetch = [&](int i) {
    const float4 *src = (const float4 *)(a.dD + (size_t)i * a.ldd);
    dq[0] = src[tid < nq ? tid : 0];
    dq[1] = src[tid + 256 < nq ? tid + 256 : 0];
    const float *tp = a.T + (size_t)i * 4 * M + (tid < M ? tid : 0);
#pragma unroll
    for (int c = 0; c < 4; ++c) tq[c] = tp[c * M];
  };
  // One tile's pair rows (rows past n read the centre's first pair).  A
  // wavefront issues its first tile of a centre before the centre's dT is
  // formed and each next tile while the current one is on the matrix cores.
  floatx4 gv[6], xv[6];
  float g6, x6, rs;
  float4 gq;
  auto load_tile = [&](int t, int base, int n) {
    const int j = 16 * t + r;
    const size_t p = (size_t)base + (j < n ? j : 0);
    gq = *(const float4 *)(a.geom + p * kGeom);  // s, rx, ry, rz
    rs = a.rstd[p];
    const float *gp = a.G + p * kDoK + 4 * g;
    const float *xp = a.xhat + p * kDoK + 4 * g;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      gv[c] = *(const floatx4 *)(gp + 16 * c);
      xv[c] = *(const floatx4 *)(xp + 16 * c);
    }
    g6 = a.G[p * kDoK + f6];
    x6 = a.xhat[p * kDoK + f6];
  };
  if (blockIdx.x < a.nloc) fetch(blockIdx.x);
  for (int i = blockIdx.x; i < a.nloc; i += gridDim.x) {
    const int n = a.nnei[i];
    const int base = a.pair_off[i];
    const int ntile = (n + 15) >> 4;
    if (wave < ntile) load_tile(wave, base, n);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int q = tid + 256 * k;
      if (q < nq) {
        const float v4[4] = {dq[k].x, dq[k].y, dq[k].z, dq[k].w};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int e = 4 * q + v, m = e / axis;
          if (m < M) dDs[m * kDoDs + (e - m * axis)] = v4[v];
        }
      }
    }
    if (tid < 128)
#pragma unroll
      for (int c = 0; c < 4; ++c) Ts[c * 128 + tid] = tid < M ? tq[c] : 0.f;
    __syncthreads();  // also: every wavefront is done with the previous centre's dTs
    if (i + (int)gridDim.x < a.nloc) fetch(i + gridDim.x);
    {
      const int aa = tid & 15, pp = tid >> 4;
      float q0 = 0.f, q1 = 0.f, q2 = 0.f, q3 = 0.f;
      if (aa < axis) {
        for (int mm = pp; mm < M; mm += 16) {
          const float x = dDs[mm * kDoDs + aa];
          q0 += x * Ts[0 * 128 + mm];
          q1 += x * Ts[1 * 128 + mm];
          q2 += x * Ts[2 * 128 + mm];
          q3 += x * Ts[3 * 128 + mm];
        }
      }
      *(float4 *)(part + (pp * 16 + aa) * 4) = make_float4(q0, q1, q2, q3);
    }
    __syncthreads();
    if (tid < 128) {
      float d0 = 0.f, d1 = 0.f, d2 = 0.f, d3 = 0.f;
      if (tid < M) {
        for (int c = 0; c < axis; ++c) {
          const float x = dDs[tid * kDoDs + c];
          d0 += x * Ts[0 * 128 + c];
          d1 += x * Ts[1 * 128 + c];
          d2 += x * Ts[2 * 128 + c];
          d3 += x * Ts[3 * 128 + c];
        }
        if (tid < axis && tid < 16) {
          for (int pp = 0; pp < 16; ++pp) {
            const float4 q = *(const float4 *)(part + (pp * 16 + tid) * 4);
            d0 += q.x;
            d1 += q.y;
            d2 += q.z;
            d3 += q.w;
          }
        }
      }
      dTs[0 * 128 + tid] = d0 * inv;
      dTs[1 * 128 + tid] = d1 * inv;
      dTs[2 * 128 + tid] = d2 * inv;
      dTs[3 * 128 + tid] = d3 * inv;
    }
    __syncthreads();
    for (int t = wave; t < ntile; t += 4) {
      const int j = 16 * t + r;
      const bool ok = j < n;
      const size_t p = (size_t)base + (ok ? j : 0);
      const float R0 = gq.x, R1 = gq.x * gq.y, R2 = gq.x * gq.z, R3 = gq.x * gq.w;
      floatx4 dy[6];
      float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f, s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        const int f = 16 * c + 4 * g;
        const floatx4 t0 = *(const floatx4 *)(dTs + 0 * 128 + f);
        const floatx4 t1 = *(const floatx4 *)(dTs + 1 * 128 + f);
        const floatx4 t2 = *(const floatx4 *)(dTs + 2 * 128 + f);
        const floatx4 t3 = *(const floatx4 *)(dTs + 3 * 128 + f);
        const floatx4 gm = *(const floatx4 *)(gam + f);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          dy[c][v] = R0 * t0[v] + R1 * t1[v] + R2 * t2[v] + R3 * t3[v];
          a0 += gv[c][v] * t0[v];
          a1 += gv[c][v] * t1[v];
          a2 += gv[c][v] * t2[v];
          a3 += gv[c][v] * t3[v];
          const float dx = gm[v] * dy[c][v];
          s1 += dx;
          s2 += dx * xv[c][v];
        }
      }
      float dy6;
      {
        const float t0 = dTs[0 * 128 + f6], t1 = dTs[1 * 128 + f6];
        const float t2 = dTs[2 * 128 + f6], t3 = dTs[3 * 128 + f6];
        const float gmv = in6 ? g6 : 0.f;
        dy6 = in6 ? R0 * t0 + R1 * t1 + R2 * t2 + R3 * t3 : 0.f;
        a0 += gmv * t0;
        a1 += gmv * t1;
        a2 += gmv * t2;
        a3 += gmv * t3;
        const float dx = gam[f6] * dy6;
        s1 += dx;
        s2 += in6 ? dx * x6 : 0.f;
      }
      a0 = sum_groups(a0);
      a1 = sum_groups(a1);
      a2 = sum_groups(a2);
      a3 = sum_groups(a3);
      s1 = sum_groups(s1);
      s2 = sum_groups(s2);
      if (ok) {
        float *dgp = a.dG + p * kDoK;
#pragma unroll
        for (int c = 0; c < 6; ++c) *(floatx4 *)(dgp + 16 * c + 4 * g) = dy[c];
        dgp[f6] = dy6;
        if (g > 0) *(floatx4 *)(dgp + 96 + 4 * g) = floatx4{0.f, 0.f, 0.f, 0.f};  // 100..111
        if (g == 0) *(float4 *)(a.dRt + 4 * p) = make_float4(a0, a1, a2, a3);
      }
      // layer-norm adjoint, in place of dy
      const float m1 = s1 * invm, m2 = s2 * invm;
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        const floatx4 gm = *(const floatx4 *)(gam + 16 * c + 4 * g);
#pragma unroll
        for (int v = 0; v < 4; ++v) dy[c][v] = rs * (gm[v] * dy[c][v] - m1 - xv[c][v] * m2);
      }
      const float x6a = in6 ? rs * (gam[f6] * dy6 - m1 - x6 * m2) : 0.f;
      if (t + 4 < ntile) load_tile(t + 4, base, n);
      floatx4 acc[8];
#pragma unroll
      for (int nt = 0; nt < 8; ++nt) acc[nt] = floatx4{0.f, 0.f, 0.f, 0.f};
      // the weight offsets are laundered per tile so that the compiler does
      // not hoist all of W_O^T into registers across tiles
      int woff = r * kDoLdw + 4 * g, w6off = r * kDoLdw + f6;
      asm volatile("" : "+v"(woff), "+v"(w6off));
      const float *wl = wsm + woff;
      if constexpr (BF) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const bf16x8 xb = to_bf16x8(dy[2 * q], dy[2 * q + 1]);
#pragma unroll
          for (int nt = 0; nt < 8; ++nt) {
            const floatx4 w0 = *(const floatx4 *)(wl + nt * 16 * kDoLdw + 32 * q);
            const floatx4 w1 = *(const floatx4 *)(wl + nt * 16 * kDoLdw + 32 * q + 16);
            acc[nt] = mfma_bf16x2(to_bf16x8(w0, w1), xb, acc[nt]);
          }
        }
        const floatx4 z = floatx4{0.f, 0.f, 0.f, 0.f};
        const bf16x8 xb = to_bf16x8(floatx4{x6a, 0.f, 0.f, 0.f}, z);
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) {
          const float w6 = wsm[w6off + nt * 16 * kDoLdw];
          acc[nt] = mfma_bf16x2(to_bf16x8(floatx4{w6, 0.f, 0.f, 0.f}, z), xb, acc[nt]);
        }
      } else {
#pragma unroll
        for (int c = 0; c < 6; ++c) {
          floatx4 w[8];
#pragma unroll
          for (int nt = 0; nt < 8; ++nt) w[nt] = *(const floatx4 *)(wl + nt * 16 * kDoLdw + 16 * c);
#pragma unroll
          for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int nt = 0; nt < 8; ++nt) acc[nt] = mfma4(w[nt][v], dy[c][v], acc[nt]);
        }
#pragma unroll
        for (int nt = 0; nt < 8; ++nt)
          acc[nt] = mfma4(wsm[w6off + nt * 16 * kDoLdw], x6a, acc[nt]);
      }
      if (ok) {
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) {
          const size_t o = p * kDoN + nt * 16 + 4 * g;
          if constexpr (BF)
            *(bf16x4 *)((__bf16 *)a.dO + o) = to_bf16(acc[nt]);
          else
            *(floatx4 *)(a.dO + o) = acc[nt];
        }
      }
    }
  }
}

// Centres are grouped by neighbour count into classes of 32, 64, 96 and 128
// slots; each class runs a kernel sized for it, over its own centre list, so
// the common case does not pay for the largest LDS size and an empty class
// costs one wave of exiting blocks.
// LDS of C centres, and of the projection to `cols` features (0: none).
template <int NPAD>
size_t fwd_lds(int C, int cols) {
  return C * fwd_centre_lds<NPAD>() +
         (cols ? sizeof(float) * (cols * kLDR + 3 * kOpCols) : 0);
}
template <int NPAD>
size_t bwdq_lds() {
  return sizeof(float4) * NPAD + sizeof(float) * stage_floats<NPAD>();
}
template <int NPAD>
size_t bwdk_lds() {
  return sizeof(float4) * 2 * NPAD + sizeof(float) * stage_floats<NPAD>();
}

// Persistent grid sizes: resident blocks per CU times CUs, per device.
constexpr int kMaxDevices = 64;
// kinds: FP32 forward, adjoint, forward with the projection on one centre; BF16
// forward, query-tile and key-tile adjoint, forward with the projection on one
// centre; FP32 forward with the projection; BF16 fused adjoint, forward with the
// projection
int g_grid[kMaxDevices][10][4];

int g_desc_grid[kMaxDevices][2];  // fused descriptor / projection adjoint: FP32, BF16

// The persistent grid, also of a class that held no centres in a recent step: the
// step may hold thousands after all (on 32 workgroups a step of 15,668 centres
// took 62 ms instead of 11), and an empty launch of it takes what one of 32
// workgroups takes (6.0 us with events around it).
int grid_for(int kind, int cls) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) dev = 0;
  return g_grid[dev][kind][cls] > 0 ? g_grid[dev][kind][cls] : 1024;
}

template <class K>
hipError_t occupancy_grid(K kernel, int threads, size_t lds, int cus, int *out) {
  int nb = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, threads, lds);
  if (e != hipSuccess) return e;
  *out = (nb > 0 ? nb : 1) * cus;
  return hipSuccess;
}

template <int NPAD, bool BF>
hipError_t prepare_class(int dev, int cus, int cls, int cols) {
  const int th = NPAD / 16 * 64;
  const auto prepare = [&](auto kernel, int threads, size_t lds, int kind) {
    int &grid = g_grid[dev][kind][cls];
    if (grid > 0) return hipSuccess;
    const hipError_t r =
        lds > 65536 ? hipFuncSetAttribute((const void *)kernel,
                                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)
                    : hipSuccess;
    return r == hipSuccess ? occupancy_grid(kernel, threads, lds, cus, &grid) : r;
  };
  constexpr int C = fwd_centres<NPAD>();
  hipError_t e;
  if (cols == 0)
    e = prepare(k_attn_fwd<NPAD, BF, false, 1>, th, fwd_lds<NPAD>(1, 0), BF ? 3 : 0);
  else if (cols <= kFwdMaxCols)
    e = prepare(k_attn_fwd<NPAD, BF, true, C>, C * th, fwd_lds<NPAD>(C, kFwdMaxCols), BF ? 9 : 7);
  else
    e = prepare(k_attn_fwd<NPAD, BF, true, 1>, th, fwd_lds<NPAD>(1, kOpCols), BF ? 6 : 2);
  if constexpr (!BF) {
    if (e == hipSuccess)
      e = prepare(k_attn_bwd_s<NPAD>, bwds_threads<NPAD>(), bwds_lds<NPAD>(), 1);
  } else if constexpr (NPAD <= 96) {
    if (e == hipSuccess) e = prepare(k_attn_bwd_f<NPAD>, 768, bwdf_lds<NPAD>(), 8);
  } else {
    if (e == hipSuccess) e = prepare(k_attn_bwd_q, th, bwdq_lds<NPAD>(), 4);
    if (e == hipSuccess) e = prepare(k_attn_bwd_k, th, bwdk_lds<NPAD>(), 5);
  }
  return e;
}

template <bool BF>
hipError_t prepare_classes(int dev, int cus, int classes, int cols) {
  hipError_t e = prepare_class<32, BF>(dev, cus, 0, cols);
  if (e == hipSuccess && classes > 1) e = prepare_class<64, BF>(dev, cus, 1, cols);
  if (e == hipSuccess && classes > 2) e = prepare_class<96, BF>(dev, cus, 2, cols);
  if (e == hipSuccess && classes > 3) e = prepare_class<128, BF>(dev, cus, 3, cols);
  int &grid = g_desc_grid[dev][BF ? 1 : 0];
  const int lds = (int)(sizeof(float) * kDoLds);
  if (e == hipSuccess && grid <= 0) {
    e = hipFuncSetAttribute((const void *)k_desc_oproj_bwd<BF>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e == hipSuccess) e = occupancy_grid(k_desc_oproj_bwd<BF>, 256, lds, cus, &grid);
  }
  return e;
}

}  // namespace

int attn_class_count(int sel) { return sel <= 32 ? 1 : sel <= 64 ? 2 : sel <= 96 ? 3 : 4; }
int attn_class_npad(int cls) { return 32 * (cls + 1); }

hipError_t attn_prepare(int sel, int cols, int bf16) {
  static std::mutex lock;  // models are created in any thread
  const std::lock_guard<std::mutex> guard(lock);
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const int classes = attn_class_count(sel);
  return bf16 ? prepare_classes<true>(dev, cus, classes, cols)
              : prepare_classes<false>(dev, cus, classes, cols);
}

void launch_attn_classes(const int *nnei, int nloc, int active, int *ccount, int *clist,
                         hipStream_t s) {
  if (nloc <= 0) return;
  hipLaunchKernelGGL(k_attn_classes, dim3((nloc + 255) / 256), dim3(256), 0, s, nnei, nloc,
                     active, ccount, clist);
}

// class (compile-time NP) and precision (compile-time BFV) dispatch
#define ATTN_CLASS_SWITCH1(cls, ...)                           \
  switch (cls) {                                               \
    case 0: { constexpr int NP = 32; __VA_ARGS__; } break;     \
    case 1: { constexpr int NP = 64; __VA_ARGS__; } break;     \
    case 2: { constexpr int NP = 96; __VA_ARGS__; } break;     \
    default: { constexpr int NP = 128; __VA_ARGS__; } break;   \
  }
#define ATTN_CLASS_SWITCH(cls, ...)                            \
  if (a.bf16) {                                                \
    constexpr bool BFV = true;                                 \
    ATTN_CLASS_SWITCH1(cls, __VA_ARGS__)                       \
  } else {                                                     \
    constexpr bool BFV = false;                                \
    ATTN_CLASS_SWITCH1(cls, __VA_ARGS__)                       \
  }

void launch_attn_fwd_class(int cls, const AttnArgs &a, const float *qkv, float *out, float *lam,
                           float *fstat, const AttnOut *op, hipStream_t s) {
  if (a.nloc <= 0) return;
  const int *cl = a.clist + (size_t)cls * a.nloc, *cc = a.ccount + cls;
  if (op && op->Nreal <= kFwdMaxCols) {
    const dim3 grid(grid_for(a.bf16 ? 9 : 7, cls));
    ATTN_CLASS_SWITCH(cls, {
      constexpr int C = fwd_centres<NP>();
      hipLaunchKernelGGL((k_attn_fwd<NP, BFV, true, C>), grid, dim3(C * NP / 16 * 64),
                         fwd_lds<NP>(C, op->Nreal), s, qkv, a.geom, a.pair_off, a.nnei, cl, cc,
                         a.sel, a.shift, out, lam, (float2 *)fstat, *op);
    });
  } else if (op) {
    const dim3 grid(grid_for(a.bf16 ? 6 : 2, cls));
    ATTN_CLASS_SWITCH(cls, hipLaunchKernelGGL((k_attn_fwd<NP, BFV, true, 1>), grid,
                                              dim3(NP / 16 * 64), fwd_lds<NP>(1, op->Nreal), s,
                                              qkv, a.geom, a.pair_off, a.nnei, cl, cc, a.sel,
                                              a.shift, out, lam, (float2 *)fstat, *op));
  } else {
    const dim3 grid(grid_for(a.bf16 ? 3 : 0, cls));
    ATTN_CLASS_SWITCH(cls, hipLaunchKernelGGL((k_attn_fwd<NP, BFV, false, 1>), grid,
                                              dim3(NP / 16 * 64), fwd_lds<NP>(1, 0), s, qkv,
                                              a.geom, a.pair_off, a.nnei, cl, cc, a.sel, a.shift,
                                              out, lam, (float2 *)fstat, AttnOut{}));
  }
}

bool attn_bwd_fused(const AttnArgs &a, int cls) { return !a.bf16 || cls <= 2; }

void launch_attn_bwd_fused_class(int cls, const AttnArgs &a, const float *qkv, const float *dO,
                                 const float *lam, const float *fstat, float *dqkv, float *gw,
                                 float *gr, int accumulate, hipStream_t s) {
  if (a.nloc <= 0 || !attn_bwd_fused(a, cls)) return;
  const int *cl = a.clist + (size_t)cls * a.nloc, *cc = a.ccount + cls;
  const dim3 grid(grid_for(a.bf16 ? 8 : 1, cls));
  ATTN_CLASS_SWITCH(cls, {
    if constexpr (!BFV)
      hipLaunchKernelGGL(k_attn_bwd_s<NP>, grid, dim3(bwds_threads<NP>()), bwds_lds<NP>(), s, qkv, dO,
                         a.geom, a.pair_off, a.nnei, cl, cc, a.shift, lam, (const float2 *)fstat,
                         dqkv, gw, gr, accumulate);
    else if constexpr (NP <= 96)
      hipLaunchKernelGGL(k_attn_bwd_f<NP>, grid, dim3(768), bwdf_lds<NP>(), s, qkv, dO, a.geom,
                         a.pair_off, a.nnei, cl, cc, a.shift, lam, (const float2 *)fstat, dqkv, gw,
                         gr, accumulate);
  });
}

void launch_attn_bwd_q(const AttnArgs &a, const float *qkv, const float *o, const float *dO,
                       const float *lam, const float *fstat, float *dqkv, float *astat,
                       float *qside, float *dA, hipStream_t s) {
  if (a.nloc <= 0) return;
  hipLaunchKernelGGL(k_attn_bwd_q, dim3(grid_for(4, 3)), dim3(512), bwdq_lds<128>(),
                     s, qkv, o, dO, a.geom, a.pair_off, a.nnei, a.clist + 3 * (size_t)a.nloc,
                     a.ccount + 3, a.sel, a.shift, lam, (const float2 *)fstat, dqkv,
                     (float4 *)astat, (float4 *)qside, dA);
}

void launch_attn_bwd_k(const AttnArgs &a, const float *qkv, const float *dO, const float *lam,
                       const float *dA, float *dqkv, const float *astat, const float *qside,
                       float *gw, float *gr, int accumulate, hipStream_t s) {
  if (a.nloc <= 0) return;
  hipLaunchKernelGGL(k_attn_bwd_k, dim3(grid_for(5, 3)), dim3(512), bwdk_lds<128>(),
                     s, qkv, dO, a.geom, a.pair_off, a.nnei, a.clist + 3 * (size_t)a.nloc,
                     a.ccount + 3, a.shift, lam, dA, dqkv, (const float4 *)astat,
                     (const float4 *)qside, gw, gr, accumulate);
}

void launch_desc_fwd(const float *geom, const float *G, int ldg, const int *pair_off,
                     const int *nnei, int nloc, int sel, int M, int axis, float *T, float *dmat,
                     hipStream_t s) {
  if (nloc <= 0) return;
  const int ldd = pad16(M * axis);
  // one lane per feature: a single wavefront when M <= 64
  const int threads = M <= 64 ? 64 : 128;
  hipLaunchKernelGGL(k_desc_fwd, dim3(nloc), dim3(threads), 0, s, geom, G, ldg, pair_off, nnei,
                     sel, M, axis, T, dmat, ldd);
}

void launch_desc_bwd(const float *geom, const float *G, int ldg, const float *T,
                     const float *dD, const int *pair_off, const int *nnei, int nloc, int sel,
                     int M, int axis, int ln_mode, const float *gamma, const float *xhat,
                     const float *rstd, const float *t_emb, float *dG, float *dnext,
                     float *dRt, hipStream_t s) {
  if (nloc <= 0) return;
  const int ldd = pad16(M * axis);
#define DESC_BWD(KF, MODE)                                                                  \
  hipLaunchKernelGGL((k_desc_bwd<KF, MODE>), dim3(nloc), dim3(256), 0, s, geom, G, ldg, T, dD, \
                     ldd, pair_off, nnei, sel, M, axis, gamma, xhat, rstd, t_emb, dG, dnext,   \
                     dRt)
  if (ldg <= 64) {
    if (ln_mode == 0)
      DESC_BWD(4, 0);
    else if (ln_mode == 1)
      DESC_BWD(4, 1);
    else
      DESC_BWD(4, 2);
  } else {
    if (ln_mode == 0)
      DESC_BWD(8, 0);
    else if (ln_mode == 1)
      DESC_BWD(8, 1);
    else
      DESC_BWD(8, 2);
  }
#undef DESC_BWD
}

bool desc_oproj_fusable(int ldg, int M, int axis, int D) {
  return ldg == kDoK && M > 96 && M <= 100 && axis >= 1 && axis <= 16 && D == kDoN;
}

void launch_desc_oproj_bwd(const float *geom, const float *G, const float *T, const float *dD,
                           const int *pair_off, const int *nnei, int nloc, int sel, int M,
                           int axis, const float *gamma, const float *xhat, const float *rstd,
                           const float *Wt, float *dG, float *dRt, float *dO, int bf16,
                           hipStream_t s) {
  if (nloc <= 0) return;
  const DescOprojArgs a{geom, G,     T,         dD,   pair_off, nnei, nloc, sel,
                        M,    axis,  pad16(M * axis), gamma, xhat, rstd, Wt,  dG,
                        dRt,  dO};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) dev = 0;
  int grid = g_desc_grid[dev][bf16 ? 1 : 0];
  if (grid <= 0) grid = 512;
  if (grid > nloc) grid = nloc;
  const size_t lds = sizeof(float) * kDoLds;
  if (bf16)
    hipLaunchKernelGGL(k_desc_oproj_bwd<true>, dim3(grid), dim3(256), lds, s, a);
  else
    hipLaunchKernelGGL(k_desc_oproj_bwd<false>, dim3(grid), dim3(256), lds, s, a);
}

}  // namespace dpa1
