// gfx950 kernels of the observables measured on a configuration between
// sweeps: the hexatic order parameter Psi (eq. Psi, Sec. 2) with cutoff or
// Delaunay neighbours, and the pair histogram of the pressure route
// (eq. pressure, Sec. 2).  All three look at the disks within a radius of a
// few sigma of every disk, so they sort the disks into a grid of their own
// whose cells are about that wide (the simulation cells hold hundreds of
// disks: scanning the 3 x 3 of them around a disk tested 2300 disks for the 6
// to 50 that count).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "ec_internal.h"

namespace ec {
namespace {

// ---------------------------------------------------------------------------
// The observables' grid: G x G cells of side L / G over the box, the disks of
// a cell contiguous in obs_pos / obs_id, obs_range[cell] = (first, end).  The
// order of the cells' ranges and of the disks in a cell is left to the atomics;
// every result below is a sum of integers (counts, fixed-point terms) or a
// minimum, so it does not depend on it.
// ---------------------------------------------------------------------------
struct Grid {
  int32_t G;    // cells per side; 1: all disks in one cell
  double inv;   // G / L
};

__device__ __forceinline__ int grid_axis(double v, const Grid& g) {
  const int k = (int)(v * g.inv);
  return k < 0 ? 0 : (k > g.G - 1 ? g.G - 1 : k);
}

__global__ void __launch_bounds__(256) k_grid_clear(const Dev* __restrict__ ds, int ncell) {
  const Dev& d = ds[blockIdx.y];
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i < ncell) d.obs_count[i] = 0;
  if (i < kObsCounters) d.obs_ctr[i] = 0;
  if (i < 2) d.status->psi_err[i] = 0;
}

__global__ void __launch_bounds__(256) k_grid_count(const Dev* __restrict__ ds, Grid g) {
  const Dev& d = ds[blockIdx.y];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.n) return;
  const int c = grid_axis(d.y[i], g) * g.G + grid_axis(d.x[i], g);
  atomicAdd(&d.obs_count[c], 1);
}

// Ranges of 1024 cells per workgroup: a prefix sum of their counts, and one
// atomic that takes that many places of the sorted arrays.  (A prefix sum over
// all cells in order would need two more launches and gain nothing: only the
// cells of one row need to be near each other.)
__global__ void __launch_bounds__(256) k_grid_ranges(const Dev* __restrict__ ds, int ncell) {
  const Dev& d = ds[blockIdx.y];
  __shared__ int32_t wsum[4], base_sh;
  const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
  const int i0 = (int)blockIdx.x * 1024 + 4 * t;
  int c[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) c[k] = i0 + k < ncell ? d.obs_count[i0 + k] : 0;
  const int tot = c[0] + c[1] + c[2] + c[3];
  int x = tot;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  if (t == 0) base_sh = atomicAdd(&d.obs_ctr[OBS_CURSOR], wsum[0] + wsum[1] + wsum[2] + wsum[3]);
  __syncthreads();
  int at = base_sh + x - tot;
  for (int w = 0; w < wave; ++w) at += wsum[w];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (i0 + k < ncell) d.obs_range[i0 + k] = make_int2(at, at + c[k]);
    at += c[k];
  }
}

// Each disk takes a place of its cell's range, counting the cell's count down.
__global__ void __launch_bounds__(256) k_grid_scatter(const Dev* __restrict__ ds, Grid g) {
  const Dev& d = ds[blockIdx.y];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.n) return;
  const double2 p = make_double2(d.x[i], d.y[i]);
  const int c = grid_axis(p.y, g) * g.G + grid_axis(p.x, g);
  const int at = d.obs_range[c].x + atomicSub(&d.obs_count[c], 1) - 1;
  d.obs_pos[at] = p;
  d.obs_id[at] = (int32_t)i;
}

// Ranges of the 3 x 3 cells around a position (the one cell of a 1 x 1 grid,
// and empty ranges beside it).  The three cells of a row that lie one behind
// the other in the sorted arrays (all but those at the box edge or at the end
// of a workgroup's 1024 cells) become one range: three short loops fewer per
// row, and lanes whose cells differ in size wait less for each other.
__device__ __forceinline__ void grid_block(const Dev& d, const Grid& g, double2 p, int2 (&r)[9]) {
  const int cx = grid_axis(p.x, g), cy = grid_axis(p.y, g);
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    int nx = cx + k % 3 - 1, ny = cy + k / 3 - 1;
    nx += nx < 0 ? g.G : (nx >= g.G ? -g.G : 0);
    ny += ny < 0 ? g.G : (ny >= g.G ? -g.G : 0);
    r[k] = (g.G > 1 || k == 4) ? d.obs_range[ny * g.G + nx] : make_int2(0, 0);
  }
#pragma unroll
  for (int k = 0; k < 9; k += 3) {
    const bool joined = r[k].y == r[k + 1].x && r[k + 1].y == r[k + 2].x;
    if (joined) r[k].y = r[k + 2].y;
    if (joined) r[k + 1] = r[k + 2] = make_int2(0, 0);
  }
}

// Offset to a disk by the minimum image.
__device__ __forceinline__ double2 offset_to(double2 q, double2 p, double L, double half_L) {
  double dx = q.x - p.x, dy = q.y - p.y;
  if (dx < -half_L) dx += L; else if (dx >= half_L) dx -= L;
  if (dy < -half_L) dy += L; else if (dy >= half_L) dy -= L;
  return make_double2(dx, dy);
}

// exp(6 i phi) of a bond as ((dx + i dy)^2 / r^2)^3, in units of 2^-52
// (|term| <= 1): integer sums do not depend on the order of the disks.
__device__ __forceinline__ void bond6(double dx, double dy, double r2, long long& fre, long long& fim) {
  const double u = (dx * dx - dy * dy) / r2, v = (2.0 * dx * dy) / r2;
  fre += __double2ll_rn((u * (u * u - 3.0 * v * v)) * 0x1p52);
  fim += __double2ll_rn((v * (3.0 * u * u - v * v)) * 0x1p52);
}

// Psi_k of the disk at sorted place i from its fixed-point sum.
__device__ __forceinline__ void store_psi(const Dev& d, int id, long long fre, long long fim, int nb) {
  double re = 0.0, im = 0.0;
  if (nb > 0) {
    re = ((double)fre * 0x1p-52) / (double)nb;
    im = ((double)fim * 0x1p-52) / (double)nb;
  }
  d.psi[id] = make_double2(re, im);
  d.psi_nb[id] = nb;
}

// ---------------------------------------------------------------------------
// Hexatic order parameter (Sec. 2, eq. Psi) with cutoff neighbours.  One
// thread per disk in sorted order (the lanes of a wave then read the same
// cells) tests the disks of 3 x 3 grid cells of side >= r_cut, of which about a
// third are neighbours whatever r_cut is, and takes a neighbour's bond term at
// once.  (With the terms put aside in LDS, eight to a lane, a lane whose eight
// are full makes the wave wait for it alone: 0.74 against 0.31 ms for 65k disks
// at eta 0.05 and r_cut 31.7, and nothing gained at short range: 72 against 74
// us for 1.2M disks at eta 0.72 and r_cut 1.4.)  Bound by instruction issue
// (about 20 B per disk are read and written); the grid before it 55 us; 6.3 ms
// as a scan of the simulation cells of 290 disks.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_psi6(const Dev* __restrict__ ds, Grid g, double rc2) {
  const Dev& d = ds[blockIdx.y];
  const int t = (int)threadIdx.x;
  const int64_t i = (int64_t)blockIdx.x * 256 + t;
  if (i >= d.n) return;
  const double2 p = d.obs_pos[i];
  const double L = d.L, half_L = d.half_L;
  int2 r[9];
  grid_block(d, g, p, r);
  long long fre = 0, fim = 0;
  int nb = 0;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    double2 next = p;
    if (r[k].x < r[k].y) next = d.obs_pos[r[k].x];
    for (int j = r[k].x; j < r[k].y; ++j) {
      const double2 o = offset_to(next, p, L, half_L);
      next = d.obs_pos[j + 1 < r[k].y ? j + 1 : j];  // in flight while this one is tested
      const double r2 = o.x * o.x + o.y * o.y;
      if (j != i && r2 < rc2) {
        bond6(o.x, o.y, r2, fre, fim);
        nb += 1;
      }
    }
  }
  store_psi(d, d.obs_id[i], fre, fim, nb);
}

// Sums of Psi_k and of the neighbour counts in disk order: per block of 256
// disks by a fixed tree, then one block adds the block sums in order, so that
// results repeat bit for bit.
__global__ void __launch_bounds__(256) k_psi6_sum(const Dev* __restrict__ ds) {
  const Dev& d = ds[blockIdx.y];
  __shared__ double sh[3][256];
  const int t = threadIdx.x;
  const int64_t k = (int64_t)blockIdx.x * 256 + t;
  const double2 v = k < d.n ? d.psi[k] : make_double2(0.0, 0.0);
  sh[0][t] = v.x;
  sh[1][t] = v.y;
  sh[2][t] = k < d.n ? (double)d.psi_nb[k] : 0.0;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (t < off) {
      sh[0][t] = sh[0][t] + sh[0][t + off];
      sh[1][t] = sh[1][t] + sh[1][t + off];
      sh[2][t] = sh[2][t] + sh[2][t + off];
    }
    __syncthreads();
  }
  if (t == 0) {
    d.psi_part[3 * blockIdx.x] = sh[0][0];
    d.psi_part[3 * blockIdx.x + 1] = sh[1][0];
    d.psi_part[3 * blockIdx.x + 2] = sh[2][0];
  }
}

__global__ void __launch_bounds__(1024) k_psi6_final(const Dev* __restrict__ ds, int nblocks) {
  const Dev& d = ds[blockIdx.y];
  __shared__ double sh[3][1024];
  const int t = threadIdx.x;
  double a = 0.0, b = 0.0, c = 0.0;
  for (int i = t; i < nblocks; i += 1024) {
    a = a + d.psi_part[3 * i];
    b = b + d.psi_part[3 * i + 1];
    c = c + d.psi_part[3 * i + 2];
  }
  sh[0][t] = a;
  sh[1][t] = b;
  sh[2][t] = c;
  __syncthreads();
  for (int off = 512; off > 0; off >>= 1) {
    if (t < off) {
      sh[0][t] = sh[0][t] + sh[0][t + off];
      sh[1][t] = sh[1][t] + sh[1][t + off];
      sh[2][t] = sh[2][t] + sh[2][t + off];
    }
    __syncthreads();
  }
  if (t == 0) {
    const double n = (double)d.n;
    d.status->psi_red[0] = sh[0][0] / n;
    d.status->psi_red[1] = sh[1][0] / n;
    d.status->psi_red[2] = sh[2][0] / n;
  }
}

// ---------------------------------------------------------------------------
// Hexatic order parameter with Delaunay neighbours (eq. Psi, Sec. 2, as the
// paper defines it).  Disk l is a Delaunay neighbour of k iff the bisector of
// k and l keeps a segment of k's Voronoi cell.  With k at the origin and the
// candidates r_m, the cell is {p : p.r_m <= |r_m|^2 / 2 for all m}; on the
// bisector of l, p = r_l / 2 + t e with e = (-r_ly, r_lx), each other m bounds
// t from one side, and l is a neighbour iff the largest lower bound stays
// below the smallest upper bound (a one-dimensional linear program).
// With the disks within a radius R as candidates the answer is exact when
// every vertex of the cell found lies within R / 2 of k: no disk farther than
// R can cut such a cell.
//
// Two passes.  k_delaunay_near takes R = r_near, a little below the distance of
// the third shell (about 12 candidates), 16 lanes per disk; where its cell is
// not certified within r_near / 2 the disk goes on a list.  k_delaunay_far takes
// R = r_search (about 50 candidates at the default of four mean spacings), one
// wavefront per disk, for the listed disks; a disk not certified there either,
// or with more than kMaxCand candidates, is counted in psi_err and the host
// reports it.  The cost of a disk grows with the square of its candidates, and
// in a dense system few disks are listed.  Bound by instruction issue: 0.50 ms
// for 1.2M disks at eta 0.72, against 12.3 ms with every disk's candidates
// within r_search, taken from the simulation cells.
// ---------------------------------------------------------------------------
constexpr int kMaxCand = 128;
constexpr int kNearCand = 32;   // candidates of the first pass; more: to the list
constexpr int kNearLanes = 16;  // lanes per disk there

__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

template <int LANES>
__device__ __forceinline__ long long lanes_sum_i64(long long v) {
  for (int off = LANES / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Candidate j of the list: does its bisector keep a segment of the cell, is
// that segment within the certified radius, and its bond term.
__device__ __forceinline__ void delaunay_edge(const double2* cand, int ncand, int j, double vmax2,
                                              bool& edge, bool& outside, long long& fre,
                                              long long& fim) {
  const double2 rl = cand[j];
  const double ex = -rl.y, ey = rl.x;
  double lo = -INFINITY, hi = INFINITY;
  for (int q = 0; q < ncand; ++q) {
    if (q == j) continue;
    const double2 rm = cand[q];
    const double den = ex * rm.x + ey * rm.y;
    const double rhs = 0.5 * (rm.x * (rm.x - rl.x) + rm.y * (rm.y - rl.y));
    const double t = rhs / den;  // one division for both sides; not used where den is 0
    if (den > 0.0) hi = fmin(hi, t);
    else if (den < 0.0) lo = fmax(lo, t);
    else if (rhs < 0.0) lo = INFINITY;  // parallel and in front: no segment
  }
  edge = lo < hi;
  outside = false;
  fre = fim = 0;
  if (edge) {
    const double ax = 0.5 * rl.x + lo * ex, ay = 0.5 * rl.y + lo * ey;
    const double bx = 0.5 * rl.x + hi * ex, by = 0.5 * rl.y + hi * ey;
    outside = !(ax * ax + ay * ay <= vmax2) || !(bx * bx + by * by <= vmax2);
    bond6(rl.x, rl.y, rl.x * rl.x + rl.y * rl.y, fre, fim);
  }
}

// First pass: four disks per wavefront.  Groups of a wave whose lists differ
// in length wait for the longest; 16 lanes hold the 12 candidates of a dense
// system in one round.
__global__ void __launch_bounds__(256) k_delaunay_near(const Dev* __restrict__ ds, Grid g, double rn2,
                                                       double vmax2) {
  const Dev& d = ds[blockIdx.y];
  __shared__ double2 cand_sh[256 / kNearLanes][kNearCand];
  const int t = (int)threadIdx.x, gl = t & (kNearLanes - 1), shift = t & 48;
  double2* const cand = cand_sh[t / kNearLanes];
  const int64_t i = (int64_t)blockIdx.x * (256 / kNearLanes) + t / kNearLanes;
  const bool live = i < d.n;  // the groups of a wave stay together for its shuffles
  const double2 p = d.obs_pos[live ? i : 0];
  const double L = d.L, half_L = d.half_L;
  int2 r[9];
  grid_block(d, g, p, r);
  int ncand = 0;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const int end = live ? r[k].y : r[k].x;
    for (int j0 = r[k].x; __builtin_amdgcn_ballot_w64(j0 < end) != 0; j0 += kNearLanes) {
      const int j = j0 + gl;
      bool keep = false;
      double2 o = make_double2(0.0, 0.0);
      if (j < end && j != i) {
        o = offset_to(d.obs_pos[j], p, L, half_L);
        keep = o.x * o.x + o.y * o.y < rn2;
      }
      const uint32_t m = (uint32_t)(__builtin_amdgcn_ballot_w64(keep) >> shift) & 0xFFFFu;
      if (keep) {
        const int slot = ncand + __popc(m & ((1u << gl) - 1u));
        if (slot < kNearCand) cand[slot] = o;
      }
      ncand += __popc(m);
    }
  }
  wave_fence();
  const bool fits = ncand <= kNearCand;
  bool outside = false;
  long long fre = 0, fim = 0;
  int nb = 0;
  for (int j = gl; fits && j < ncand; j += kNearLanes) {
    bool e, o;
    long long br, bi;
    delaunay_edge(cand, ncand, j, vmax2, e, o, br, bi);
    outside |= o;
    nb += e ? 1 : 0;
    fre += br;
    fim += bi;
  }
  fre = lanes_sum_i64<kNearLanes>(fre);
  fim = lanes_sum_i64<kNearLanes>(fim);
  for (int off = kNearLanes / 2; off > 0; off >>= 1) nb += __shfl_xor(nb, off, 64);
  outside = ((__builtin_amdgcn_ballot_w64(outside) >> shift) & 0xFFFFull) != 0;
  if (live && gl == 0) {
    if (fits && !outside && nb >= 3)
      store_psi(d, d.obs_id[i], fre, fim, nb);
    else
      d.obs_list[atomicAdd(&d.obs_ctr[OBS_LISTED], 1)] = (int32_t)i;
  }
}

// Second pass: the listed disks (all = 0) or every disk, one wavefront each;
// the cells within `span` of the disk's own on both axes hold every disk
// within the search radius.
__global__ void __launch_bounds__(256) k_delaunay_far(const Dev* __restrict__ ds, Grid g, int span,
                                                      int all, double rs2, double vmax2) {
  const Dev& d = ds[blockIdx.y];
  __shared__ double2 cand_sh[4][kMaxCand];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  double2* const cand = cand_sh[wave];
  const double L = d.L, half_L = d.half_L;
  const int across = 2 * span + 1 < g.G ? 2 * span + 1 : g.G;  // cells per axis, each once
  const int64_t total = all ? d.n : (int64_t)d.obs_ctr[OBS_LISTED];
  for (int64_t a = (int64_t)blockIdx.x * 4 + wave; a < total; a += (int64_t)gridDim.x * 4) {
    const int64_t i = all ? a : (int64_t)d.obs_list[a];
    wave_fence();  // the previous disk's candidate reads before this disk's writes
    const double2 p = d.obs_pos[i];
    const int cx = grid_axis(p.x, g), cy = grid_axis(p.y, g);
    int ncand = 0;
    for (int oy = 0; oy < across; ++oy) {
      const int ny = (cy - across / 2 + oy + g.G) % g.G;
      for (int ox = 0; ox < across; ++ox) {
        const int nx = (cx - across / 2 + ox + g.G) % g.G;
        const int2 r = d.obs_range[ny * g.G + nx];
        for (int j0 = r.x; j0 < r.y; j0 += 64) {
          const int j = j0 + lane;
          bool keep = false;
          double2 o = make_double2(0.0, 0.0);
          if (j < r.y && j != i) {
            o = offset_to(d.obs_pos[j], p, L, half_L);
            keep = o.x * o.x + o.y * o.y < rs2;
          }
          const uint64_t m = __builtin_amdgcn_ballot_w64(keep);
          if (keep) {
            const int slot = ncand + (int)__builtin_amdgcn_mbcnt_hi(
                                         (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            if (slot < kMaxCand) cand[slot] = o;
          }
          ncand += __popcll(m);
        }
      }
    }
    wave_fence();
    long long fre = 0, fim = 0;
    int nb = 0;
    if (ncand > kMaxCand) {
      if (lane == 0) atomicAdd(&d.status->psi_err[1], 1ull);
    } else {
      bool e0 = false, e1 = false, o0 = false, o1 = false;
      long long r1 = 0, i1 = 0;
      if (lane < ncand) delaunay_edge(cand, ncand, lane, vmax2, e0, o0, fre, fim);
      if (lane + 64 < ncand) delaunay_edge(cand, ncand, lane + 64, vmax2, e1, o1, r1, i1);
      if (__builtin_amdgcn_ballot_w64(o0 || o1) != 0 && lane == 0) atomicAdd(&d.status->psi_err[0], 1ull);
      nb = __popcll(__builtin_amdgcn_ballot_w64(e0)) + __popcll(__builtin_amdgcn_ballot_w64(e1));
      fre = lanes_sum_i64<64>(fre + r1);
      fim = lanes_sum_i64<64>(fim + i1);
    }
    if (lane == 0) store_psi(d, d.obs_id[i], fre, fim, nb);
  }
}

// ---------------------------------------------------------------------------
// Pair histogram for the pressure route of eq. (pressure), Sec. 2: one thread
// per disk in sorted order tests the disks of 3 x 3 grid cells of side >=
// r_max, minimum image, bin = floor((sqrt(dx*dx + dy*dy) - sigma) / delta).
// A pair counts twice (it is ordered) and is looked at once, from the disk of
// the lower sorted place; |offset| is the same number from either disk.  Counts
// go to a histogram per workgroup in LDS, then to the global one (integers:
// exact and independent of order); the workgroups go over the disks in strides,
// since each adds all its bins to the global counts at the end (how many there
// are: histogram_groups).  Pairs closer than sigma are counted apart.  35 us for
// 303k disks in random order (r_max 1.5, 500 bins), the grid before it 41 us;
// 12.2 ms as a scan of the simulation cells.  (As in k_psi6 nothing is put aside:
// 16k disks at eta 0.7, r_max 33.9, 2.6 ms against 10.3 ms.)
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_gr(const Dev* __restrict__ ds, Grid g, double r_max, double delta,
                                            int n_bins) {
  const Dev& d = ds[blockIdx.y];
  __shared__ unsigned int hist[kMaxGrBins + 1];
  const int t = (int)threadIdx.x;
  for (int i = t; i <= n_bins; i += 256) hist[i] = 0;
  __syncthreads();
  const double L = d.L, half_L = d.half_L, r2max = r_max * r_max, sigma = d.sigma;
  for (int64_t i = (int64_t)blockIdx.x * 256 + t; i < d.n; i += (int64_t)gridDim.x * 256) {
    const double2 p = d.obs_pos[i];
    int2 r[9];
    grid_block(d, g, p, r);
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const int first = r[k].x > i ? r[k].x : (int)i + 1;
      double2 next = p;
      if (first < r[k].y) next = d.obs_pos[first];
      for (int j = first; j < r[k].y; ++j) {
        const double2 o = offset_to(next, p, L, half_L);
        next = d.obs_pos[j + 1 < r[k].y ? j + 1 : j];  // in flight while this one is tested
        const double d2 = o.x * o.x + o.y * o.y;
        if (d2 < r2max) {
          const double dist = sqrt(d2);
          const double b = floor((dist - sigma) / delta);
          if (dist < sigma) atomicAdd(&hist[n_bins], 2u);
          else if (b < (double)n_bins) atomicAdd(&hist[(int)b], 2u);
        }
      }
    }
  }
  __syncthreads();
  for (int i = t; i <= n_bins; i += 256)
    if (hist[i]) atomicAdd(&d.gr_counts[i], (unsigned long long)hist[i]);
}

// ---------------------------------------------------------------------------
// Overlap check (debug): one thread per disk counts the disks j > i closer
// than sigma (1 - 1e-12), minimum image, among the 3 x 3 cells of the
// sweep's grid around its own (a pair closer than sigma < cell side lies in
// neighbouring cells; disks stay in their cells during a sweep), or among all
// disks for one periodic cell.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void report_overlap(const Dev& d, int64_t i, int64_t j, int64_t sweep) {
  if (atomicAdd(d.ovl, 1ull) == 0ull) {
    d.ovl[1] = (unsigned long long)i;
    d.ovl[2] = (unsigned long long)j;
    d.ovl[3] = (unsigned long long)sweep;
  }
  atomicOr(d.err, ERR_OVERLAP);
}

__global__ void __launch_bounds__(256) k_check_overlap(const Dev* __restrict__ ds) {
  const Dev& d = ds[blockIdx.y];
  if (!d.check_overlap) return;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.n) return;
  const double L = d.L, half = d.half_L;
  const double thr = d.sigma * (1.0 - 1e-12), thr2 = thr * thr;
  const double xi = d.x[i], yi = d.y[i];
  const int64_t sweep = *d.sweep_ctr;
  auto test = [&](int64_t j) {
    if (j <= i) return;
    double dx = d.x[j] - xi, dy = d.y[j] - yi;
    if (dx < -half) dx += L; else if (dx >= half) dx -= L;
    if (dy < -half) dy += L; else if (dy >= half) dy -= L;
    if (dx * dx + dy * dy < thr2) report_overlap(d, i, j, sweep);
  };
  if (d.C == 1) {
    for (int64_t j = i + 1; j < d.n; ++j) test(j);
    return;
  }
  const int c = d.cell_of[i];
  if (d.stripes) {  // the sweep's lists are stripes; a pair closer than sigma lies in neighbouring ones
    for (int side = -1; side <= 1; ++side) {
      const int nk = (c + side + d.C) % d.C;
      if (side == 1 && nk == (c - 1 + d.C) % d.C) continue;  // two stripes only
      for (int t = d.cell_start[nk]; t < d.cell_start[nk + 1]; ++t) test(d.cell_ids[t]);
    }
    return;
  }
  const int cx = c % d.C, cy = c / d.C;
  for (int nb = 0; nb < 9; ++nb) {
    const int ncx = (cx + nb % 3 - 1 + d.C) % d.C, ncy = (cy + nb / 3 - 1 + d.C) % d.C;
    const int nc = ncy * d.C + ncx;
    for (int t = d.cell_start[nc]; t < d.cell_start[nc + 1]; ++t) test(d.cell_ids[t]);
  }
}

}  // namespace

namespace {

// Grid for pairs within r: cells at least r wide (by 1e-9, far above the
// rounding of a position's cell), no more cells than disks, and at least 3 per
// side, where the 3 x 3 cells around a disk are nine different ones; else one.
Grid grid_for(const LaunchShape& sh, double r) {
  Grid g;
  const double by_radius = floor(sh.box / (r * (1.0 + 1e-9))), by_disks = floor(sqrt((double)sh.max_n));
  const double side = by_radius < by_disks ? by_radius : by_disks;
  g.G = side >= 3.0 ? (int32_t)side : 1;
  g.inv = (double)g.G / sh.box;
  return g;
}

hipError_t launch_grid(const Dev* ds, const LaunchShape& sh, const Grid& g, hipStream_t st) {
  const unsigned nblk = (unsigned)((sh.max_n + 255) / 256);
  const int ncell = g.G * g.G;
  hipLaunchKernelGGL(k_grid_clear, dim3((unsigned)((ncell + 255) / 256), 1), dim3(256), 0, st, ds, ncell);
  hipLaunchKernelGGL(k_grid_count, dim3(nblk, 1), dim3(256), 0, st, ds, g);
  hipLaunchKernelGGL(k_grid_ranges, dim3((unsigned)((ncell + 1023) / 1024), 1), dim3(256), 0, st, ds, ncell);
  hipLaunchKernelGGL(k_grid_scatter, dim3(nblk, 1), dim3(256), 0, st, ds, g);
  return hipGetLastError();
}

hipError_t launch_psi6_sums(const Dev* ds, const LaunchShape& sh, hipStream_t st) {
  const unsigned nblk = (unsigned)((sh.max_n + 255) / 256);
  hipLaunchKernelGGL(k_psi6_sum, dim3(nblk, 1), dim3(256), 0, st, ds);
  hipLaunchKernelGGL(k_psi6_final, dim3(1, 1), dim3(1024), 0, st, ds, (int)nblk);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_psi6(const Dev* ds, const LaunchShape& sh, double r_cut, hipStream_t st) {
  const unsigned nblk = (unsigned)((sh.max_n + 255) / 256);
  const Grid g = grid_for(sh, r_cut);
  hipError_t e = launch_grid(ds, sh, g, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_psi6, dim3(nblk, 1), dim3(256), 0, st, ds, g, r_cut * r_cut);
  return launch_psi6_sums(ds, sh, st);
}

hipError_t launch_psi6_delaunay(const Dev* ds, const LaunchShape& sh, double r_search, hipStream_t st) {
  // The first pass looks within two mean spacings (in a triangular lattice the
  // first two shells, at 1.07 and 1.86, and certifies vertices up to 1.0; they
  // lie at 0.62).  It is taken where its radius is below the search radius and
  // where no disk can have more than kMaxCand others within the search radius
  // (Oler's bound for a disc), which only the second pass would notice.
  const double near = 2.0 * sh.box / sqrt((double)sh.max_n), u = r_search / sh.sigma;
  const bool two = near < r_search && 3.6276 * u * u + 3.1416 * u + 1.0 <= (double)kMaxCand;
  // Where all disks take the wide search, the grid is as wide as that: 9 cells
  // instead of 25 or more of the first pass's width with four disks each for a
  // wavefront to test (1M disks, eta 0.1, r_search 6: 2.3 against 4.0 ms).
  const Grid g = grid_for(sh, two ? near : r_search);
  hipError_t e = launch_grid(ds, sh, g, st);
  if (e != hipSuccess) return e;
  if (two)
    hipLaunchKernelGGL(k_delaunay_near, dim3((unsigned)((sh.max_n + 15) / 16), 1), dim3(256), 0, st, ds, g,
                       near * near, 0.25 * near * near * (1.0 - 1e-9));
  const int span = g.G == 1 ? 0 : (int)fmin(ceil(r_search * g.inv * (1.0 + 1e-9)), (double)g.G);
  const int64_t blocks = (sh.max_n + 3) / 4;
  hipLaunchKernelGGL(k_delaunay_far, dim3((unsigned)(two && blocks > 1024 ? 1024 : (blocks > 8192 ? 8192 : blocks)), 1),
                     dim3(256), 0, st, ds, g, span, two ? 0 : 1, r_search * r_search,
                     0.25 * r_search * r_search);
  return launch_psi6_sums(ds, sh, st);
}

hipError_t launch_gr(const Dev* ds, const LaunchShape& sh, double r_max, double delta, int n_bins,
                     hipStream_t st) {
  const Grid g = grid_for(sh, r_max);
  hipError_t e = launch_grid(ds, sh, g, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_gr, dim3((unsigned)histogram_groups(sh.max_n, r_max / sh.sigma), 1), dim3(256), 0, st, ds, g,
                     r_max, delta, n_bins);
  return hipGetLastError();
}

hipError_t launch_check_overlap(const Dev* ds, const LaunchShape& sh, hipStream_t st) {
  if (!sh.check_overlap) return hipSuccess;
  const unsigned nblk = (unsigned)((sh.max_n + 255) / 256);
  hipLaunchKernelGGL(k_check_overlap, dim3(nblk, (unsigned)sh.n_sys), dim3(256), 0, st, ds);
  return hipGetLastError();
}

}  // namespace ec
