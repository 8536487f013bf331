// Neighbour search and per-pair geometry for DPA-1 inference on gfx950.
//
// Full neighbour lists within the cutoff (Sec. II-A: cutoff lists make the
// cost O(N); Sec. II-C: a DP descriptor needs the full list of every centre).
// A cell grid with edge >= rcut bins the atoms; one workgroup per cell
// stages the candidates of the 27 surrounding cells in LDS, and one
// wavefront per centre tests them in FP64 and compacts hits with a ballot.  Lists are sorted by atom index so that every later stage
// sees a deterministic neighbour order.
//
// Pair vectors follow one fixed FP64 recipe, with contraction disabled so
// the result does not depend on FMA formation:
//   d = x_j - x_i;  with a box d -= L * rint(d / L);
//   r2 = (dx*dx + dy*dy) + dz*dz;  neighbour iff r2 < rcut*rcut.
#include <algorithm>
#include <climits>

#include "attn_classes.h"
#include "dpa1_internal.h"

namespace dpa1 {

namespace {

constexpr int kWave = 64;
constexpr int kListCap = 128;      // == DP_MAX_SEL

__device__ __forceinline__ void pair_vec(const double *__restrict__ x, int i, int j,
                                         const CellGrid &g, double d[3]) {
#pragma clang fp contract(off)
  for (int c = 0; c < 3; ++c) {
    double v = x[3 * j + c] - x[3 * i + c];
    if (g.periodic) v = v - g.L[c] * rint(v / g.L[c]);
    d[c] = v;
  }
}

__device__ __forceinline__ double norm2(const double d[3]) {
#pragma clang fp contract(off)
  return (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2];
}

__device__ __forceinline__ int cell_coord(double x, int c, const CellGrid &g) {
  double u;
  if (g.periodic) {
    double w = x - g.L[c] * floor(x / g.L[c]);
    u = w * g.inv_edge[c];
  } else {
    u = (x - g.lo[c]) * g.inv_edge[c];
  }
  int k = (int)floor(u);
  k = k < 0 ? 0 : k;
  k = k >= g.nc[c] ? g.nc[c] - 1 : k;
  return k;
}

// Flags out-of-range types and writes a clamped copy that every later kernel
// indexes tables with, so a bad input can never address outside them.
__global__ void k_check_types(const int32_t *__restrict__ types, int nall, int ntypes,
                              DevFlags *flags, int32_t *__restrict__ safe) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nall) return;
  int t = types[k];
  if (t < 0 || t >= ntypes) {
    atomicMin(&flags->bad_type_atom, k);
    t = t < 0 ? 0 : ntypes - 1;
  }
  safe[k] = t;
}

__global__ void k_cell_bin(const double *__restrict__ x, int nall, CellGrid g,
                           int *__restrict__ atom_cell, int *__restrict__ cell_count) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nall) return;
  int cx = cell_coord(x[3 * k + 0], 0, g);
  int cy = cell_coord(x[3 * k + 1], 1, g);
  int cz = cell_coord(x[3 * k + 2], 2, g);
  int c = (cz * g.nc[1] + cy) * g.nc[0] + cx;
  atom_cell[k] = c;
  atomicAdd(&cell_count[c], 1);
}

// Exclusive prefix of s over the 1024 threads of the block (one barrier; wtot is
// free again after the next one), and the total.
__device__ __forceinline__ int block_prefix(int s, int *wtot, int &total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int inc = s;  // inclusive within the wavefront
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int y = __shfl_up(inc, off);
    if (lane >= off) inc += y;
  }
  if (lane == 63) wtot[wave] = inc;
  __syncthreads();
  int before = 0;
  total = 0;
  for (int w = 0; w < 16; ++w) {
    if (w < wave) before += wtot[w];
    total += wtot[w];
  }
  return before + inc - s;
}

// The binning of a small system in one block: flags, safe types, cell starts and
// cell members.  Five launches of a few microseconds of work each cost 4.7 us
// apiece on the stream (24 us); one block takes 5 us at 192 atoms and 13 to 15
// us at 4000 to 8000.  The order of a cell's atoms is left to the atomics here as
// there; the neighbour lists are sorted.
__global__ __launch_bounds__(1024) void k_bin_small(
    const double *__restrict__ x, const int32_t *__restrict__ types, int nall, int ntypes,
    CellGrid g, int ncell, DevFlags *flags, int *__restrict__ ccount, int32_t *__restrict__ safe,
    int *__restrict__ cell_start, int *__restrict__ cell_atoms) {
  constexpr int U = kBinAtoms / 1024, V = kBinCells / 1024;
  __shared__ int cnt[kBinCells];
  __shared__ int wtot[16];
  __shared__ int bad;
  const int t = threadIdx.x;
#pragma unroll
  for (int v = 0; v < V; ++v) cnt[t + 1024 * v] = 0;
  if (t == 0) bad = INT_MAX;
  if (t < 8) ccount[t] = 0;
  __syncthreads();
  int cell[U], pos[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int k = t + 1024 * u;
    cell[u] = -1;
    if (k >= nall) continue;
    int ty = types[k];
    if (ty < 0 || ty >= ntypes) {
      atomicMin(&bad, k);
      ty = ty < 0 ? 0 : ntypes - 1;
    }
    safe[k] = ty;
    const int cx = cell_coord(x[3 * k + 0], 0, g), cy = cell_coord(x[3 * k + 1], 1, g),
              cz = cell_coord(x[3 * k + 2], 2, g);
    cell[u] = (cz * g.nc[1] + cy) * g.nc[0] + cx;
    pos[u] = atomicAdd(&cnt[cell[u]], 1);
  }
  __syncthreads();
  int c[V], s = 0, total;
#pragma unroll
  for (int v = 0; v < V; ++v) {
    c[v] = cnt[V * t + v];
    s += c[v];
  }
  int run = block_prefix(s, wtot, total);
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int q = V * t + v;
    cnt[q] = run;  // this thread's own counters: read above, by no one else
    if (q < ncell) cell_start[q] = run;
    run += c[v];
  }
  if (t == 0) {
    cell_start[ncell] = total;
    flags->overflow_atom = INT_MAX;
    flags->overflow_count = 0;
    flags->bad_type_atom = bad;
    flags->pair_overflow = 0;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (cell[u] >= 0) cell_atoms[cnt[cell[u]] + pos[u]] = t + 1024 * u;
}

// Single-block exclusive scan: out[0..n) exclusive prefix sums, out[n] total.
// Thread t owns the contiguous chunk [t per, (t + 1) per), per a multiple of four,
// read and written as int4 (in and out are aligned to 16 bytes; 4-byte accesses a
// chunk apart, 64 lines to a load, took 25 us instead of 10 for 15,668 centres),
// four loads at a time.
// Returns the total, to every thread.
__device__ __forceinline__ int4 load_upto(const int *in, int k, int e) {
  if (k + 4 <= e) return *(const int4 *)(in + k);
  return make_int4(k < e ? in[k] : 0, k + 1 < e ? in[k + 1] : 0, k + 2 < e ? in[k + 2] : 0, 0);
}

__device__ __forceinline__ int block_scan(const int *in, int n, int *out, int *wtot) {
  const int t = threadIdx.x;
  const int per = ((n + 1023) / 1024 + 3) & ~3;
  const int b = t * per;
  const int e = min(b + per, n);
  int s = 0;
  for (int k0 = b; k0 < e; k0 += 16) {
    int4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = load_upto(in, k0 + 4 * u, e);
#pragma unroll
    for (int u = 0; u < 4; ++u) s += (v[u].x + v[u].y) + (v[u].z + v[u].w);
  }
  int total, run = block_prefix(s, wtot, total);  // exclusive prefix of this chunk
  for (int k0 = b; k0 < e; k0 += 16) {
    int4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = load_upto(in, k0 + 4 * u, e);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = k0 + 4 * u;
      const int4 o = make_int4(run, run + v[u].x, run + v[u].x + v[u].y,
                               run + v[u].x + v[u].y + v[u].z);
      if (k + 4 <= e) {
        *(int4 *)(out + k) = o;
      } else {
        if (k < e) out[k] = o.x;
        if (k + 1 < e) out[k + 1] = o.y;
        if (k + 2 < e) out[k + 2] = o.z;
      }
      run = o.w + v[u].w;
    }
  }
  if (t == 0) out[n] = total;
  return total;
}

__global__ __launch_bounds__(1024) void k_scan(const int *__restrict__ in, int n,
                                               int *__restrict__ out) {
  __shared__ int wtot[16];
  block_scan(in, n, out, wtot);
}

// Pair offsets from the neighbour counts, and in the same block what hangs on
// them: the capacity check of the pair arena (a step with more neighbour pairs
// than cap records its count and gets no pair work at all: every neighbour
// count, locals and ghosts, and every pair offset set to 0, so no kernel indexes
// past the arena; the workspace grows at the next call), and with clist the
// attention class lists (attn_classes.h).
__global__ __launch_bounds__(1024) void k_pair_scan(int *nnei, int nloc, int nall, long cap,
                                                    int *pair_off, DevFlags *flags, int active,
                                                    int *ccount, int *clist) {
  __shared__ int wtot[16];
  __shared__ int cc[8];
  if (threadIdx.x < 8) cc[threadIdx.x] = 0;
  const int total = block_scan(nnei, nloc, pair_off, wtot);
  if ((long)total > cap) {
    __syncthreads();  // every offset is written before any is cleared
    if (threadIdx.x == 0) flags->pair_overflow = total;
    for (int k = threadIdx.x; k < nall; k += 1024) nnei[k] = 0;
    for (int k = threadIdx.x; k <= nloc; k += 1024) pair_off[k] = 0;
    __syncthreads();
  }
  if (!clist) return;
  for (int i0 = 0; i0 < nloc; i0 += 1024)
    attn_class_lists(i0 + threadIdx.x, nnei, nloc, active, cc, clist);
  __syncthreads();
  if (threadIdx.x < 8) ccount[threadIdx.x] = cc[threadIdx.x];
}

__global__ void k_cell_fill(const int *__restrict__ atom_cell, int nall,
                            const int *__restrict__ cell_start, int *__restrict__ cell_fill,
                            int *__restrict__ cell_atoms) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nall) return;
  int c = atom_cell[k];
  int pos = atomicAdd(&cell_fill[c], 1);
  cell_atoms[cell_start[c] + pos] = k;
}

// The k-th (k < 3) distinct neighbour cell of c along one dimension, or -1.
__device__ __forceinline__ int neighbour_cell(const CellGrid &g, int dim, int c, int k) {
  const int nc = g.nc[dim];
  if (g.periodic) return nc >= 3 ? (c + nc + k - 1) % nc : k < nc ? k : -1;
  const int q = c + k - 1;
  return q >= 0 && q < nc ? q : -1;
}

// One workgroup per cell.  Every atom of a cell has the same 27 neighbour
// cells, so the workgroup stages their candidates (atom index and FP64
// coordinates) in LDS once and each wavefront then tests its centres (one
// at a time) against the staged tile, 64 candidates per pass.  Local
// centres collect every atom within rcut; ghost centres collect local atoms
// only (they are needed by the force gather, never as energy centres).  A
// neighbourhood with more candidates than the tile holds is scanned from
// global memory instead (same ranges, same test).  Where there are few cells, up
// to four workgroups share the centres of one.
//
// Latency and FP64 work bound it, not memory: the ranges of the 27 cells are
// read by 27 lanes at once (one lane in turn waited for 18 loads and more), the
// periodic test multiplies by 1 / L (divisions only within 1e-6 of the cutoff),
// and the sort compares four entries per LDS read.  192 atoms 18 -> 10 us, 4095
// 60 -> 23, a domain of 980 and 7000 ghosts 56 -> 38, 15,668 atoms 77 -> 51.
constexpr int kCellWaves = 8;      // wavefronts per cell workgroup
constexpr int kTileCap = 1536;     // staged candidates (about 2.5x the protein density)
constexpr int kMaxRanges = 27;

// The pair test on FP64 coordinates: the recipe of pair_vec and norm2.
__device__ __forceinline__ bool within(double xi0, double xi1, double xi2, double xj0, double xj1,
                                       double xj2, const CellGrid &g, double rc2) {
#pragma clang fp contract(off)
  double d0 = xj0 - xi0, d1 = xj1 - xi1, d2 = xj2 - xi2;
  if (g.periodic) {
    d0 = d0 - g.L[0] * rint(d0 / g.L[0]);
    d1 = d1 - g.L[1] * rint(d1 / g.L[1]);
    d2 = d2 - g.L[2] * rint(d2 / g.L[2]);
  }
  return (d0 * d0 + d1 * d1) + d2 * d2 < rc2;
}

// The same decision without the divisions: d / L only picks the image, and a
// rounding that picked the other one has |d| = L / 2 either way; r2 is then off
// by parts in 1e9 at most, and the exact test decides within 1e-6 of the cutoff
// (and on NaN).
__device__ __forceinline__ bool within_fast(double xi0, double xi1, double xi2, double xj0,
                                            double xj1, double xj2, const CellGrid &g,
                                            const double (&inv)[3], double rc2) {
  if (!g.periodic) return within(xi0, xi1, xi2, xj0, xj1, xj2, g, rc2);
  double d0 = xj0 - xi0, d1 = xj1 - xi1, d2 = xj2 - xi2;
  d0 -= g.L[0] * rint(d0 * inv[0]);
  d1 -= g.L[1] * rint(d1 * inv[1]);
  d2 -= g.L[2] * rint(d2 * inv[2]);
  const double r2 = (d0 * d0 + d1 * d1) + d2 * d2;
  if (r2 > rc2 * (1.0 + 1e-6)) return false;
  if (r2 < rc2 * (1.0 - 1e-6)) return true;
  return within(xi0, xi1, xi2, xj0, xj1, xj2, g, rc2);
}

__global__ __launch_bounds__(kWave *kCellWaves) void k_nlist(
    const double *__restrict__ x, int nloc, CellGrid g, double rc2, int sel,
    const int *__restrict__ cell_start, const int *__restrict__ cell_atoms,
    int *__restrict__ nlist, int *__restrict__ nnei, DevFlags *flags) {
  __shared__ int tj[kTileCap];
  __shared__ double tx[kTileCap], ty[kTileCap], tz[kTileCap];
  __shared__ __attribute__((aligned(16))) int list[kCellWaves][kListCap + 4];
  __shared__ int rb[32], roff[32];  // ranges of cell_atoms, their places in the tile
  const int cell = blockIdx.x;
  const int a0 = cell_start[cell], a1 = cell_start[cell + 1];
  if (a0 == a1) return;  // empty cell: the whole workgroup leaves
  const int wave = threadIdx.x / kWave;
  const int lane = threadIdx.x % kWave;
  if (threadIdx.x < 32) {
    const int k = (int)threadIdx.x;
    const int ox = neighbour_cell(g, 0, cell % g.nc[0], k % 3);
    const int oy = neighbour_cell(g, 1, (cell / g.nc[0]) % g.nc[1], k / 3 % 3);
    const int oz = neighbour_cell(g, 2, cell / (g.nc[0] * g.nc[1]), k / 9 % 3);
    const bool ok = k < kMaxRanges && ox >= 0 && oy >= 0 && oz >= 0;
    const int c = ok ? (oz * g.nc[1] + oy) * g.nc[0] + ox : cell;
    const int beg = cell_start[c], n = ok ? cell_start[c + 1] - beg : 0;
    int inc = n;
#pragma unroll
    for (int off = 1; off < 32; off <<= 1) {
      const int y = __shfl_up(inc, off);
      if (k >= off) inc += y;
    }
    rb[k] = beg;
    roff[k] = inc - n;  // roff[27] and later: the total
  }
  __syncthreads();
  constexpr int R = kMaxRanges;
  const int T = roff[R];
  const bool staged = T <= kTileCap;
  if (staged) {
    for (int t = threadIdx.x; t < T; t += blockDim.x) {
      int q = 0;  // the last range that starts at or before t (empty ones end there too)
#pragma unroll
      for (int h = 16; h >= 1; h >>= 1)
        if (q + h < R && roff[q + h] <= t) q += h;
      const int j = cell_atoms[rb[q] + (t - roff[q])];
      tj[t] = j;
      tx[t] = x[3 * j + 0];
      ty[t] = x[3 * j + 1];
      tz[t] = x[3 * j + 2];
    }
  }
  __syncthreads();
  const double inv[3] = {1.0 / g.L[0], 1.0 / g.L[1], 1.0 / g.L[2]};
  for (int ai = a0 + (int)blockIdx.y * kCellWaves + wave; ai < a1;
       ai += kCellWaves * (int)gridDim.y) {
    const int k = cell_atoms[ai];
    const bool ghost = k >= nloc;
    const double xk0 = x[3 * k + 0], xk1 = x[3 * k + 1], xk2 = x[3 * k + 2];
    int count = 0;
    auto keep = [&](bool hit, int j) {
      const unsigned long long m = __ballot(hit);
      const int pos = count + __popcll(m & ((1ull << lane) - 1ull));
      if (hit && pos < kListCap) list[wave][pos] = j;
      count += __popcll(m);
    };
    if (staged) {
      for (int base = 0; base < T; base += kWave) {
        const int t = base + lane;
        bool hit = false;
        int j = -1;
        if (t < T) {
          j = tj[t];
          if (j != k && (!ghost || j < nloc))
            hit = within_fast(xk0, xk1, xk2, tx[t], ty[t], tz[t], g, inv, rc2);
        }
        keep(hit, j);
      }
    } else {
      for (int q = 0; q < R; ++q) {
        const int beg = rb[q], end = rb[q] + (roff[q + 1] - roff[q]);
        for (int base = beg; base < end; base += kWave) {
          const int idx = base + lane;
          bool hit = false;
          int j = -1;
          if (idx < end) {
            j = cell_atoms[idx];
            if (j != k && (!ghost || j < nloc))
              hit = within_fast(xk0, xk1, xk2, x[3 * j + 0], x[3 * j + 1], x[3 * j + 2], g, inv,
                                rc2);
          }
          keep(hit, j);
        }
      }
    }
    const int n = count < sel ? count : sel;
    if (count > sel) {
      if (lane == 0) {
        int old = atomicMin(&flags->overflow_atom, k);
        if (old > k) atomicExch(&flags->overflow_count, count);
      }
    }
    // rank sort of the (distinct) indices
    int vals[2], ranks[2];
    for (int h = 0; h < 2; ++h) {
      const int p = lane + h * kWave;
      vals[h] = p < n ? list[wave][p] : INT_MAX;
      ranks[h] = 0;
    }
    if (lane < 4) list[wave][n + lane] = INT_MAX;  // rounds the list up
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (int q = 0; q < n; q += 4) {
      const int4 v = *(const int4 *)&list[wave][q];
      ranks[0] += (v.x < vals[0]) + (v.y < vals[0]) + (v.z < vals[0]) + (v.w < vals[0]);
      ranks[1] += (v.x < vals[1]) + (v.y < vals[1]) + (v.z < vals[1]) + (v.w < vals[1]);
    }
    int *row = nlist + (size_t)k * sel;
    for (int h = 0; h < 2; ++h) {
      const int p = lane + h * kWave;
      if (p < n) row[ranks[h]] = vals[h];
      else if (p < sel) row[p] = -1;
    }
    if (lane == 0) nnei[k] = n;
    __builtin_amdgcn_wave_barrier();  // the wave's list is rewritten by its next centre
  }
}

// One thread per (centre, slot).  Geometry in FP64, stored as FP32.
// One wavefront per centre: lane l handles slots l, l + 64 of the centre's
// list, so the pair records (contiguous per centre) are written by
// consecutive lanes, and each lane writes its h1 row with 16-byte stores.
// The type-pair table and ws are staged in LDS once per block (when they
// fit), so no global load sits inside the per-element loop.
constexpr int kEnvWaves = 4;
constexpr int kEnvTable = 8192;  // floats of type table staged in LDS

__global__ __launch_bounds__(kEnvWaves * 64) void k_env_embed1(
    const double *__restrict__ x, const int32_t *__restrict__ types, CellGrid g, int nloc,
    int sel, double rcut, double rs, const int *__restrict__ nlist, const int *__restrict__ nnei,
    const int *__restrict__ pair_off, const float *__restrict__ type_table,
    const float *__restrict__ ws, int ntypes, int n1, int ld1, float *__restrict__ geom,
    float *__restrict__ h1) {
  __shared__ float tab_s[kEnvTable];
  __shared__ float ws_s[128];
  const int tsize = ntypes * ntypes * ld1;
  const bool staged = tsize <= kEnvTable && ld1 <= 128;
  if (staged) {
    for (int k = threadIdx.x; k < tsize; k += blockDim.x) tab_s[k] = type_table[k];
    for (int k = threadIdx.x; k < ld1; k += blockDim.x) ws_s[k] = ws[k];
  }
  __syncthreads();
  const float *tab = staged ? tab_s : type_table;
  const float *wsv = staged ? ws_s : ws;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = blockIdx.x * kEnvWaves + wave;
  if (i >= nloc) return;
  const int n = nnei[i];
  const int base = pair_off[i];
  const int ti = types[i];
  const double inv = 1.0 / (rcut - rs);
  for (int sl = lane; sl < n; sl += 64) {
    const int j = nlist[(size_t)i * sel + sl];
    const int tj = types[j];
    const int p = base + sl;
    double d[3];
    pair_vec(x, i, j, g, d);
    const double r = sqrt(norm2(d));
    // sw = u^3 (-6u^2 + 15u - 10) + 1 on [rs, rcut); dsw/dr = -30 u^2 (u - 1)^2 / (rcut - rs)
    const double u = (r - rs) * inv;
    const double swm = u * u * u * (-6.0 * u * u + 15.0 * u - 10.0) + 1.0;
    const double dswm = -30.0 * u * u * (u - 1.0) * (u - 1.0) * inv;
    const double sw = r < rs ? 1.0 : (r < rcut ? swm : 0.0);
    const double dsw = (r < rs || r >= rcut) ? 0.0 : dswm;
    const double sv = sw / r;
    float4 *gp = (float4 *)(geom + (size_t)p * kGeom);
    gp[0] = make_float4((float)sv, (float)(d[0] / r), (float)(d[1] / r), (float)(d[2] / r));
    // slot 7: FP32 remainder of sw (the FP32 attention logits take hi + lo in FP64)
    gp[1] = make_float4((float)sw, (float)r, (float)dsw, (float)(sw - (double)(float)sw));
    const float s32 = (float)sv;
    const float *tt = tab + ((size_t)tj * ntypes + ti) * ld1;
    float4 *hp = (float4 *)(h1 + (size_t)p * ld1);
    for (int o = 0; o < ld1; o += 4) {
      float4 v;
      v.x = o + 0 < n1 ? tanh_fast(tt[o + 0] + wsv[o + 0] * s32) : 0.0f;
      v.y = o + 1 < n1 ? tanh_fast(tt[o + 1] + wsv[o + 1] * s32) : 0.0f;
      v.z = o + 2 < n1 ? tanh_fast(tt[o + 2] + wsv[o + 2] * s32) : 0.0f;
      v.w = o + 3 < n1 ? tanh_fast(tt[o + 3] + wsv[o + 3] * s32) : 0.0f;
      hp[o >> 2] = v;
    }
  }
}

}  // namespace

static inline unsigned nblk(long n, int b) { return (unsigned)((n + b - 1) / b); }

void launch_check_types(const int32_t *types, int nall, int ntypes, DevFlags *flags,
                        int32_t *safe, hipStream_t s) {
  if (nall <= 0) return;
  hipLaunchKernelGGL(k_check_types, dim3(nblk(nall, 256)), dim3(256), 0, s, types, nall, ntypes,
                     flags, safe);
}

void launch_cell_bin(const double *coords, int nall, CellGrid grid, int *atom_cell,
                     int *cell_count, hipStream_t s) {
  if (nall <= 0) return;
  hipLaunchKernelGGL(k_cell_bin, dim3(nblk(nall, 256)), dim3(256), 0, s, coords, nall, grid,
                     atom_cell, cell_count);
}

void launch_scan(const int *in, int n, int *out_excl, hipStream_t s) {
  hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, s, in, n, out_excl);
}

void launch_bin_small(const double *coords, const int32_t *types, int nall, int ntypes,
                      CellGrid grid, DevFlags *flags, int *ccount, int32_t *safe,
                      int *cell_start, int *cell_atoms, hipStream_t s) {
  hipLaunchKernelGGL(k_bin_small, dim3(1), dim3(1024), 0, s, coords, types, nall, ntypes, grid,
                     grid.ncell, flags, ccount, safe, cell_start, cell_atoms);
}

void launch_pair_scan(int *nnei, int nloc, int nall, long cap, int *pair_off, DevFlags *flags,
                      int active, int *ccount, int *clist, hipStream_t s) {
  hipLaunchKernelGGL(k_pair_scan, dim3(1), dim3(1024), 0, s, nnei, nloc, nall, cap, pair_off,
                     flags, active, ccount, clist);
}

void launch_cell_fill(const int *atom_cell, int nall, const int *cell_start, int *cell_fill,
                      int *cell_atoms, hipStream_t s) {
  if (nall <= 0) return;
  hipLaunchKernelGGL(k_cell_fill, dim3(nblk(nall, 256)), dim3(256), 0, s, atom_cell, nall,
                     cell_start, cell_fill, cell_atoms);
}

void launch_nlist(const double *coords, int nloc, int nall, CellGrid grid, double rcut, int sel,
                  const int *cell_start, const int *cell_atoms, int *nlist, int *nnei,
                  DevFlags *flags, hipStream_t s) {
  if (nall <= 0) return;
  const int ncell = grid.nc[0] * grid.nc[1] * grid.nc[2];
  // Workgroups of a cell: as many as run at once on 256 CUs, three to each by LDS,
  // and four at most (a cell of 22 atoms leaves each then fewer than its eight
  // wavefronts take at once).  More than run at once stage tiles for nothing.  At
  // 0.1 atoms per cubic A with 1, 2, 3, 4 workgroups: 64 cells 23.4, 17.0, 15.3,
  // 12.3 us; 216 cells 26.0, 20.0, 18.6, 20.2; 343 cells 30.7, 24.7, 26.1, 26.8;
  // 512 cells 31.1, 32.9, 33.6, 34.7.
  const int parts = std::max(1, std::min(4, 768 / ncell));
  hipLaunchKernelGGL(k_nlist, dim3(ncell, parts), dim3(kWave * kCellWaves), 0, s, coords, nloc, grid,
                     rcut * rcut, sel, cell_start, cell_atoms, nlist, nnei, flags);
}

void launch_env_embed1(const double *coords, const int32_t *types, CellGrid grid, int nloc,
                       int sel, double rcut, double rcut_smth, const int *nlist, const int *nnei,
                       const int *pair_off, const float *type_table, const float *ws, int ntypes,
                       int n1, int ld1, float *geom, float *h1, hipStream_t s) {
  if (nloc <= 0) return;
  hipLaunchKernelGGL(k_env_embed1, dim3(nblk(nloc, kEnvWaves)), dim3(kEnvWaves * 64), 0, s, coords,
                     types, grid, nloc, sel, rcut, rcut_smth, nlist, nnei, pair_off, type_table,
                     ws, ntypes, n1, ld1, geom, h1);
}

}  // namespace dpa1
