// gfx950 kernels of the parallel event-chain (PEC) sweep for 2D hard disks.
//
// Method: Kampmann, Boltz, Kierfeld, "Parallelized event chain algorithm for
// dense hard sphere and polymer systems" -- event chains Sec. 3.2, the
// parallel sweep Sec. 3.4 (steps 1-7), boundary reflection Fig. 1 (right),
// starts with replacement Fig. 2.
//
// Mapping to CDNA4: one wavefront (64 lanes) per active simulation cell.  A
// cell's own disks and its frozen neighbours (centres within sigma outside
// the cell) are staged in LDS in a grid of square bins of side b <
// sigma/sqrt(2); such a bin holds at most one centre of a configuration
// without overlaps, so one slot per bin suffices and a cell takes about 18 KB
// (eight cells, two wavefronts per SIMD, per CU).  One event search reads an
// 8 x 8 window of bins around the moving disk, one slot per lane, computes
// the contact distance of every slot in FP64, and takes a wave-wide minimum
// of the key (distance, disk id).  A geometric guard proves that no disk
// outside the window can be hit first; when it cannot (long free flights),
// the search is repeated over all slots of the cell.  The event found is
// therefore exactly the minimum over all candidate disks, in the same
// arithmetic as a plain serial search.
//
// Arithmetic contract (shared in writing with the CPU reference, no code
// shared): FP64 with no contraction (-ffp-contract=off) and explicit fma();
// correctly rounded sqrt and division; Philox4x64-10 streams keyed by
// (seed, kind) with counters (sweep, cell | system << 32, chain, block).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "ec_internal.h"

namespace ec {
namespace {

// ---------------------------------------------------------------------------
// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11)
// ---------------------------------------------------------------------------
constexpr uint64_t kM0 = 0xD2E7470EE14C6C93ull;
constexpr uint64_t kM1 = 0xCA5A826395121157ull;
constexpr uint64_t kW0 = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kW1 = 0xBB67AE8584CAA73Bull;

enum : uint64_t { kKindSweep = 1, kKindStart = 2, kKindDir = 3, kKindShuffle = 4 };

struct Block4 {
  uint64_t v0, v1, v2, v3;
};

__device__ __forceinline__ Block4 philox(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3,
                                         uint64_t k0, uint64_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) { k0 += kW0; k1 += kW1; }
    uint64_t hi0 = __umul64hi(kM0, c0), lo0 = kM0 * c0;
    uint64_t hi1 = __umul64hi(kM1, c2), lo1 = kM1 * c2;
    uint64_t n0 = hi1 ^ c1 ^ k0;
    uint64_t n2 = hi0 ^ c3 ^ k1;
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
  }
  return Block4{c0, c1, c2, c3};
}

// Words 0..3 of counter block 0, then block 1, ...
struct Stream {
  uint64_t k0, k1, c0, c1, c2, blk;
  Block4 b;
  int pos;
  __device__ Stream(uint64_t seed, uint64_t kind, uint64_t a, uint64_t bb, uint64_t c)
      : k0(seed), k1(kind), c0(a), c1(bb), c2(c), blk(0), b{0, 0, 0, 0}, pos(4) {}
  __device__ uint64_t next() {
    if (pos == 4) {
      b = philox(c0, c1, c2, blk, k0, k1);
      blk += 1;
      pos = 0;
    }
    uint64_t w = (pos == 0) ? b.v0 : (pos == 1) ? b.v1 : (pos == 2) ? b.v2 : b.v3;
    pos += 1;
    return w;
  }
};

// Loads and stores of global memory through a record's pointers.  A pointer
// that was itself loaded is generic to the compiler, and a generic (flat)
// access counts as an LDS access too: every LDS wait after it also waits for
// memory, 1 to 2 us.
#define EC_GLOBAL(T) __attribute__((address_space(1))) T
template <class T>
__device__ __forceinline__ T gload(const T* p) {
  return *(const EC_GLOBAL(T)*)p;
}
__device__ __forceinline__ double2 gload(const double2* p) {
  typedef double pair_t __attribute__((ext_vector_type(2)));
  const pair_t v = *(const EC_GLOBAL(pair_t)*)p;
  return make_double2(v.x, v.y);
}
template <class T>
__device__ __forceinline__ void gstore(T* p, T v) {
  *(EC_GLOBAL(T)*)p = v;
}

__device__ __forceinline__ double u01(uint64_t w) { return (double)(w >> 11) * 0x1.0p-53; }

// Lemire's multiply-shift with rejection: exactly uniform on [0, n).
__device__ uint64_t draw_index(Stream& st, uint64_t n) {
  uint64_t x = st.next();
  uint64_t hi = __umul64hi(x, n), lo = x * n;
  if (lo < n) {
    uint64_t t = (0ull - n) % n;
    while (lo < t) {
      x = st.next();
      hi = __umul64hi(x, n);
      lo = x * n;
    }
  }
  return hi;
}

__device__ __forceinline__ uint64_t cell_key(const Dev& d, int cell) {
  return (uint64_t)(uint32_t)cell | ((uint64_t)d.system << 32);
}

// Direction of chain k of a cell in a sweep.
__device__ void chain_direction(const Dev& d, int64_t sweep, int cell, int64_t k, double& dx,
                                double& dy) {
  if (d.dir_mode == 2) { dx = 1.0; dy = 0.0; return; }          // +x only
  if (d.dir_mode == 0) {                                         // +x / +y alternating
    if ((k & 1) == 0) { dx = 1.0; dy = 0.0; } else { dx = 0.0; dy = 1.0; }
    return;
  }
  // isotropic: uniform in the unit disk by rejection, then normalised
  Stream st(d.seed, kKindDir, (uint64_t)sweep, cell_key(d, cell), (uint64_t)k);
  double vx, vy, r2;
  for (;;) {
    vx = 2.0 * u01(st.next()) - 1.0;
    vy = 2.0 * u01(st.next()) - 1.0;
    r2 = fma(vx, vx, vy * vy);
    if (r2 < 1.0 && r2 >= 0x1p-40) break;
  }
  double r = sqrt(r2);
  dx = vx / r;
  dy = vy / r;
}

// ---------------------------------------------------------------------------
// Wave-level helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ unsigned umin_(unsigned a, unsigned b) { return a < b ? a : b; }

// Minimum of a 32-bit value over the 64 lanes as a scalar: DPP steps within
// rows of 16, then the row broadcasts of lane 15 into rows 1 and 3 and of
// lane 31 into rows 2 and 3, which leave the minimum in lane 63.
__device__ __forceinline__ unsigned wave_min_u32(unsigned v) {
  v = umin_(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true));
  v = umin_(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true));
  v = umin_(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true));
  v = umin_(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, true));
  // (rows outside a broadcast's mask take the identity, so that each step is
  // one instruction; only rows 1 and 3, then row 3, are read afterwards)
  v = umin_(v, (unsigned)__builtin_amdgcn_update_dpp(-1, (int)v, 0x142, 0xA, 0xF, false));
  v = umin_(v, (unsigned)__builtin_amdgcn_update_dpp(-1, (int)v, 0x143, 0xC, 0xF, false));
  return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int lane) {
  uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
  uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ double readlane_f64(double v, int lane) {
  return __longlong_as_double((long long)readlane_u64((uint64_t)__double_as_longlong(v), lane));
}
__device__ __forceinline__ int readlane_i32(int v, int lane) {
  return __builtin_amdgcn_readlane(v, lane);
}
// Make a value that is equal in all lanes visibly wave-uniform, so that the
// branches on it are scalar branches.  The event dispatch below relies on
// this: compiled as a divergent if/else chain on a vector register, one of
// its arms (the y-wall reflection) lost its direction update.
__device__ __forceinline__ int uniform_i32(int v) { return __builtin_amdgcn_readfirstlane(v); }
// Lane `lane` of a, b, c replaced by the wave-uniform values va, vb, vc
// (v_writelane, lane select in M0: no compare and no change of the execution
// mask)
__device__ __forceinline__ void writelane3(uint32_t& a, uint32_t& b, uint32_t& c, uint32_t va,
                                           uint32_t vb, uint32_t vc, int lane) {
  asm("v_writelane_b32 %0, %3, m0\n\t"
      "v_writelane_b32 %1, %4, m0\n\t"
      "v_writelane_b32 %2, %5, m0"
      : "+v"(a), "+v"(b), "+v"(c)
      : "s"(uniform_i32((int)va)), "s"(uniform_i32((int)vb)), "s"(uniform_i32((int)vc)),
        "{m0}"(lane));
}

// Lane holding the smallest key (s, id) among lanes with valid = true, where
// s >= 0 so that its bit pattern orders like its value.  -1 if none.
__device__ __forceinline__ int wave_argmin(double s, uint32_t id, bool valid) {
  uint64_t sb = (uint64_t)__double_as_longlong(s);
  unsigned hi = valid ? (unsigned)(sb >> 32) : 0xFFFFFFFFu;
  unsigned m = wave_min_u32(hi);
  if (m == 0xFFFFFFFFu) return -1;
  uint64_t mask = __ballot(valid && hi == m);
  int wl = __ffsll((unsigned long long)mask) - 1;
  mask &= mask - 1;
  if (mask) {  // equal high words: resolve on the full key
    uint64_t bs = readlane_u64(sb, wl);
    uint32_t bi = (uint32_t)readlane_i32((int)id, wl);
    while (mask) {
      int l = __ffsll((unsigned long long)mask) - 1;
      mask &= mask - 1;
      uint64_t ls = readlane_u64(sb, l);
      uint32_t li = (uint32_t)readlane_i32((int)id, l);
      if (ls < bs || (ls == bs && li < bi)) { bs = ls; bi = li; wl = l; }
    }
  }
  return wl;
}

// The argmin in two steps: argmin_key is the lane's key (the high word of s
// on valid lanes, all ones elsewhere); its wave minimum m is all ones exactly
// when no lane is valid, since a valid lane's high word (a non-negative
// distance) never is.  Given m below all ones, argmin_lane returns the lane.
__device__ __forceinline__ unsigned argmin_key(double s, bool valid) {
  return valid ? (unsigned)((uint64_t)__double_as_longlong(s) >> 32) : 0xFFFFFFFFu;
}
__device__ __forceinline__ int argmin_lane(double s, uint32_t id, unsigned hi, unsigned m) {
  const uint64_t sb = (uint64_t)__double_as_longlong(s);
  uint64_t mask = __builtin_amdgcn_ballot_w64(hi == m);  // not empty: some lane holds m
  int wl = __builtin_ctzll(mask);
  if (__builtin_expect(mask != (1ull << wl), 0)) {  // equal high words: resolve on the full key
    mask &= mask - 1;
    uint64_t bs = readlane_u64(sb, wl);
    uint32_t bi = (uint32_t)readlane_i32((int)id, wl);
    while (mask) {
      const int l = __ffsll((unsigned long long)mask) - 1;
      mask &= mask - 1;
      const uint64_t ls = readlane_u64(sb, l);
      const uint32_t li = (uint32_t)readlane_i32((int)id, l);
      if (ls < bs || (ls == bs && li < bi)) { bs = ls; bi = li; wl = l; }
    }
  }
  return wl;
}
__device__ __forceinline__ int wave_argmin_all(double s, uint32_t id, bool valid) {
  const unsigned hi = argmin_key(s, valid);
  const unsigned m = wave_min_u32(hi);
  if (m == 0xFFFFFFFFu) return -1;
  return argmin_lane(s, id, hi, m);
}

// Event digest (a test device, not part of the method).  Event i of a cell's
// phase has the record r = bits(s) ^ id*K1 ^ kind<<56; the cell digest is the
// XOR over i of mix(r ^ i*K2), mix being the splitmix64 finaliser (Steele,
// Lea, Flood, OOPSLA 2014).  The XOR lets a wave hash 64 events at once.
constexpr uint64_t kDigestK1 = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kDigestK2 = 0xD6E8FEB86659FD93ull;

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__device__ __forceinline__ uint64_t digest_term(int kind, uint64_t gid, double s, uint64_t i) {
  const uint64_t r = (uint64_t)__double_as_longlong(s) ^ (gid * kDigestK1) ^ ((uint64_t)kind << 56);
  return mix64(r ^ (i * kDigestK2));
}

// XOR of a 32-bit value over the 64 lanes, left in every lane.
__device__ __forceinline__ unsigned wave_xor_all(unsigned v) {
  v ^= (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);
  v ^= (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);
  v ^= (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true);
  v ^= (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, true);
  const auto r16 = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = (unsigned)r16[0] ^ (unsigned)r16[1];
  const auto r32 = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return (unsigned)r32[0] ^ (unsigned)r32[1];
}

// Event records of a simulation cell, held one per lane (lane k: record of
// event first + k, in three 32-bit registers): the step's bits and (kind ^ 1)
// << 29 | id, where a lift (kind 1) names its disk by the index into the cell's
// id-ordered list own_gid (a lift's word is then its disk's meta word), or by
// its id where there is no list.  XOR over the wave of the digest terms of the
// first `count`; lifts counts the lifts among them.
__device__ __forceinline__ uint64_t digest_records(uint32_t rec_lo, uint32_t rec_hi, uint32_t rec_tag,
                                                   int lane, int count, uint64_t first,
                                                   const int32_t* own_gid, uint32_t& lifts) {
  uint64_t t = 0;
  bool is_lift = false;
  if (lane < count) {
    is_lift = (rec_tag >> 29) == 0;
    uint32_t id = rec_tag & 0x1FFFFFFFu;
    if (is_lift && own_gid) id = (uint32_t)own_gid[id];
    t = digest_term((int)(rec_tag >> 29) ^ 1, id,
                    __longlong_as_double((long long)(((uint64_t)rec_hi << 32) | rec_lo)), first + (uint64_t)lane);
  }
  lifts = (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(is_lift));
  const uint32_t lo = (uint32_t)uniform_i32((int)wave_xor_all((uint32_t)t));
  const uint32_t hi = (uint32_t)uniform_i32((int)wave_xor_all((uint32_t)(t >> 32)));
  return ((uint64_t)hi << 32) | lo;
}

enum { EV_LIFT = 1, EV_FROZEN = 2, EV_WALL_X = 3, EV_WALL_Y = 4, EV_PSEUDO = 5, EV_END = 6 };

// Contact distance of a disk moving along unit d towards a disk at offset r:
// s = a - sqrt(sigma^2 - c^2) with a = r.d, c = r x d, for a > 0 and
// sigma^2 - c^2 > 0; negative values (touching disks) become 0.
// Correctly rounded square root of x in [2^-767, 2^1000] (Markstein's
// method: the hardware reciprocal square root estimate, one Newton step on
// (g, h) = (x y, y/2), then two corrections with the exact residual x - g^2
// from a fused multiply-add; P. Markstein, IBM J. Res. Dev. 34 (1990) 111).
// The general sqrt() adds range scaling and special-value selects; the
// contact term's argument sigma^2 - c^2, where positive, is at least about
// 2^-106 sigma^2, and sigma is limited to [2^-300, 2^300], so x stays in range.
__device__ __forceinline__ double sqrt_contact(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y;
  double h = 0.5 * y;
  const double r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  double dd = fma(-g, g, x);
  g = fma(dd, h, g);
  dd = fma(-g, g, x);
  return fma(dd, h, g);
}

__device__ __forceinline__ bool contact(double rx, double ry, double dx, double dy, double sig2,
                                        double& s) {
  double a = fma(rx, dx, ry * dy);
  double c = fma(rx, dy, -(ry * dx));
  double disc = fma(-c, c, sig2);
  // computed in every lane and selected (no branch): where disc <= 0 the
  // root is NaN or infinite and the lane is not a candidate
  const bool ok = a > 0.0 && disc > 0.0;
  const double t = a - sqrt_contact(disc);
  s = ok ? ((t < 0.0) ? 0.0 : t) : s;
  return ok;
}

// Shifted-frame coordinate in [0, L] and cell-local coordinate.
__device__ __forceinline__ double shifted(double p, double shift, double L) {
  double t = p - shift;
  if (t < 0.0) t += L;
  return t;
}
__device__ __forceinline__ double local_coord(double p, double shift, double origin, double L,
                                              double half_L) {
  double v = shifted(p, shift, L) - origin;
  if (v < -half_L) v += L;
  else if (v >= half_L) v -= L;
  return v;
}

// ---------------------------------------------------------------------------
// Start lattice
// ---------------------------------------------------------------------------
__global__ void k_lattice(const Dev* __restrict__ ds, int64_t k, double a) {
  const Dev& d = ds[blockIdx.y];
  int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= d.n) return;
  int64_t j = id / k, i = id % k;
  d.x[id] = ((double)i + ((j & 1) ? 0.75 : 0.25)) * a;
  d.y[id] = ((double)j + 0.5) * a;
}

// ---------------------------------------------------------------------------
// Rebin: sweep draws, cell of every disk, counting sort by cell
// ---------------------------------------------------------------------------
// Permutation number idx in [0, 24) decoded in the factorial base: the
// colour of phase q lands in bits 2q, 2q+1 of the result.  The colours not
// yet taken are kept in order as 2-bit fields of `avail`.
__device__ int32_t decode_perm(uint64_t idx) {
  uint32_t avail = 0 | (1u << 2) | (2u << 4) | (3u << 6);
  const uint32_t fact[4] = {6, 2, 1, 1};
  int32_t out = 0;
  uint32_t r = (uint32_t)idx;
#pragma unroll
  for (int pos = 0; pos < 4; ++pos) {
    const uint32_t q = r / fact[pos];
    r = r % fact[pos];
    out |= (int32_t)(((avail >> (2 * q)) & 3u) << (2 * pos));
    // drop field q: the fields above it move down by one
    const uint32_t low = avail & ((1u << (2 * q)) - 1u);
    avail = low | ((avail >> (2 * q + 2)) << (2 * q));
  }
  return out;
}

// The first kernel of a sweep: its number (the counter holds that of the last
// sweep, -1 before the first), its draws, cleared counts.
__global__ void k_prep(const Dev* __restrict__ ds) {
  const Dev& d = ds[blockIdx.y];
  const int nreg = kRegions * d.C * d.C;
  for (int c = threadIdx.x; c < nreg; c += blockDim.x) {
    d.reg_count[c] = 0;
  }
  if (threadIdx.x == 0) {
    const int64_t sweep = *d.sweep_ctr + 1;
    *d.sweep_ctr = sweep;
    Stream st(d.seed, kKindSweep, (uint64_t)sweep, (uint64_t)d.system, 0);
    SweepDraws dr;
    if (d.stripes) {
      // stripes: shift across them, and which of the two colours goes first
      dr.sx = u01(st.next()) * d.w;
      dr.sy = 0.0;
      dr.perm = (int32_t)draw_index(st, 2);
    } else {
      dr.sx = u01(st.next()) * d.w;
      dr.sy = u01(st.next()) * d.w;
      dr.perm = decode_perm(draw_index(st, 24));
    }
    dr.pad = 0;
    *d.draws = dr;
    d.digest_ring[sweep % kDigestRing] = 0;
    *d.queue = 0;  // ticket counter of the one-launch sweep
  }
}

__device__ __forceinline__ int cell_of_pos(const Dev& d, double px, double py, double sx,
                                           double sy) {
  int cx = (int)floor(shifted(px, sx, d.L) / d.w);
  int cy = (int)floor(shifted(py, sy, d.L) / d.w);
  if (cx > d.C - 1) cx = d.C - 1;
  if (cy > d.C - 1) cy = d.C - 1;
  return cy * d.C + cx;
}

// Region of a cell-local coordinate along one axis: 0 within the strip at the
// cell's low wall, 2 within the strip at its high wall, 1 between.
__device__ __forceinline__ int strip_of(double v, double w, double strip) {
  return v < strip ? 0 : (v >= w - strip ? 2 : 1);
}

// Lanes of the wave whose key equals this lane's (among the lanes that run).
__device__ __forceinline__ uint64_t lanes_of_key(int key) {
  uint64_t todo = __builtin_amdgcn_ballot_w64(true), mine = 0;
  while (todo) {
    const int lk = __builtin_amdgcn_readlane(key, (int)__builtin_ctzll(todo));
    const uint64_t same = __builtin_amdgcn_ballot_w64(key == lk);
    if (key == lk) mine = same;
    todo &= ~same;
  }
  return mine;
}

// Cell and region of every disk, the counts, and each disk's place in its
// (cell, region): one atomic per distinct (cell, region) of the wavefront
// (consecutive ids are mostly neighbours in space, so a wave's disks fall into a
// few), all of them at once, so that a wave waits for one trip to memory.  The
// place is kept for k_scatter (in the array of the shuffled lists, which are
// made after it); the order inside a region is free: staging sorts a cell's ids.
__global__ void k_count(const Dev* __restrict__ ds) {
  const Dev& d = ds[blockIdx.y];
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.n) return;
  SweepDraws dr = *d.draws;
  int c, r = 0;  // cell and region (stripes and one periodic cell: region 0)
  if (d.stripes) {
    // stripe index from the coordinate across the stripes: horizontal stripes
    // (across = y) on even sweeps, vertical ones (across = x) on odd sweeps
    const double across = (*d.sweep_ctr & 1) ? d.x[i] : d.y[i];
    c = (int)floor(shifted(across, dr.sx, d.L) / d.w);
    if (c > d.C - 1) c = d.C - 1;
  } else {
    c = cell_of_pos(d, d.x[i], d.y[i], dr.sx, dr.sy);
    if (d.C > 1) {
      // the disk's region in its cell, from its cell-local coordinates (the
      // wall strips are what neighbouring cells stage as their frozen band)
      const int cx = c % d.C, cy = c / d.C;
      const double vx = shifted(d.x[i], dr.sx, d.L) - (double)cx * d.w;
      const double vy = shifted(d.y[i], dr.sy, d.L) - (double)cy * d.w;
      r = 3 * strip_of(vy, d.w, d.strip) + strip_of(vx, d.w, d.strip);
    }
  }
  d.cell_of[i] = c;
  d.reg_of[i] = (uint8_t)r;
  const int key = kRegions * c + r;
  const uint64_t mine = lanes_of_key(key);
  const int lane = (int)(threadIdx.x & 63), leader = (int)__builtin_ctzll(mine);
  int base = 0;
  if (lane == leader) base = atomicAdd(&d.reg_count[key], (int)__builtin_popcountll(mine));
  base = __shfl(base, leader, 64);
  d.shuffle[i] = base + (int)__builtin_popcountll(mine & ((1ull << lane) - 1));
}

// Exclusive prefix sum of the (cell, region) counts, one workgroup of 1024
// threads; a cell's start is that of its first region.  The counts are
// taken in tiles of 4,096, four consecutive counts per thread in one 16-byte
// access (the count and start arrays are 256-byte aligned), summed in the
// thread, then over the wave and over the 16 waves; the next tile's counts
// are loaded while the current one is summed.
__global__ void __launch_bounds__(1024) k_scan(const Dev* __restrict__ ds) {
  const Dev& d = ds[blockIdx.y];
  constexpr int kTile = 4096;
  __shared__ int32_t wsum[16];
  const int ncell = d.C * d.C;
  const int nreg = kRegions * ncell;
  const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
  const int32_t* __restrict__ cnt = d.reg_count;
  int32_t* __restrict__ start = d.reg_start;
  auto load = [&](int base) __attribute__((always_inline)) {
    const int i0 = base + 4 * t;
    int4 v;
    if (i0 + 3 < nreg) {
      v = *(const int4*)(cnt + i0);
    } else {
      v.x = (i0 < nreg) ? cnt[i0] : 0;
      v.y = (i0 + 1 < nreg) ? cnt[i0 + 1] : 0;
      v.z = (i0 + 2 < nreg) ? cnt[i0 + 2] : 0;
      v.w = 0;
    }
    return v;
  };
  int4 v = load(0);
  int carry = 0;
  for (int base = 0; base < nreg; base += kTile) {
    const int4 cur = v;
    if (base + kTile < nreg) v = load(base + kTile);  // the next tile, in flight meanwhile
    const int tot = cur.x + cur.y + cur.z + cur.w;
    // inclusive sum of the thread totals over the wave
    int x = tot;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int y = __shfl_up(x, off, 64);
      if (lane >= off) x += y;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    int woff = 0, tile_total = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      const int sw = wsum[w];
      woff += (w < wave) ? sw : 0;
      tile_total += sw;
    }
    const int e0 = carry + woff + (x - tot);
    const int4 out = make_int4(e0, e0 + cur.x, e0 + cur.x + cur.y, e0 + cur.x + cur.y + cur.z);
    const int i0 = base + 4 * t;
    if (i0 + 3 < nreg) {
      *(int4*)(start + i0) = out;
    } else {
      if (i0 < nreg) start[i0] = out.x;
      if (i0 + 1 < nreg) start[i0 + 1] = out.y;
      if (i0 + 2 < nreg) start[i0 + 2] = out.z;
    }
    // the cell starts: the one multiple of kRegions among the four, if any
    const int r0 = i0 % kRegions;
    const int k = (r0 == 0) ? 0 : kRegions - r0;
    if (k < 4 && i0 + k < nreg) {
      const int sv = (k == 0) ? out.x : ((k == 1) ? out.y : ((k == 2) ? out.z : out.w));
      d.cell_start[(i0 + k) / kRegions] = sv;
    }
    carry += tile_total;
    __syncthreads();  // every thread has read wsum before the next tile writes it
  }
  if (t == 0) {
    start[nreg] = carry;
    d.cell_start[ncell] = carry;
  }
}

__global__ void k_scatter(const Dev* __restrict__ ds) {
  const Dev& d = ds[blockIdx.y];
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.n) return;
  const int k = kRegions * d.cell_of[i] + (int)d.reg_of[i];
  d.cell_ids[d.reg_start[k] + d.shuffle[i]] = (int32_t)i;
}

// ---------------------------------------------------------------------------
// Chain draws of a sweep (Sec. 3.4 step 5): one thread per chain computes the
// start index, drawn with replacement among the cell's n_c disks, and the
// isotropic direction.  Rejection loops are capped (kMaxDrawTries).
// ---------------------------------------------------------------------------
__device__ __forceinline__ int64_t chains_of(const Dev& d, int n_c) {
  if (n_c <= 0) return 0;
  return d.chains_per_cell > 0 ? d.chains_per_cell : n_c;
}
__device__ __forceinline__ int64_t chain_base(const Dev& d, int cell) {
  return d.chains_per_cell > 0 ? (int64_t)cell * d.chains_per_cell : (int64_t)gload(d.cell_start + cell);
}

__device__ bool draw_index_capped(Stream& st, uint64_t n, uint64_t& out) {
  uint64_t x = st.next();
  uint64_t hi = __umul64hi(x, n), lo = x * n;
  if (lo < n) {
    uint64_t t = (0ull - n) % n;
    int tries = 0;
    while (lo < t) {
      if (++tries > kMaxDrawTries) return false;
      x = st.next();
      hi = __umul64hi(x, n);
      lo = x * n;
    }
  }
  out = hi;
  return true;
}

__device__ bool iso_direction_capped(const Dev& d, int64_t sweep, int cell, int64_t k, double& dx,
                                     double& dy) {
  Stream st(d.seed, kKindDir, (uint64_t)sweep, cell_key(d, cell), (uint64_t)k);
  for (int tries = 0; tries < kMaxDrawTries; ++tries) {
    double vx = 2.0 * u01(st.next()) - 1.0;
    double vy = 2.0 * u01(st.next()) - 1.0;
    double r2 = fma(vx, vx, vy * vy);
    if (r2 < 1.0 && r2 >= 0x1p-40) {
      double r = sqrt(r2);
      dx = vx / r;
      dy = vy / r;
      return true;
    }
  }
  dx = 1.0;
  dy = 0.0;
  return false;
}

// Cell whose range [cell_start[c], cell_start[c+1]) holds chain slot i.
__device__ __forceinline__ int cell_of_slot(const Dev& d, int64_t i) {
  int lo = 0, hi = d.C * d.C - 1;
  while (lo < hi) {  // largest c with cell_start[c] <= i
    int mid = (lo + hi + 1) >> 1;
    if ((int64_t)d.cell_start[mid] <= i) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__global__ void k_draws(const Dev* __restrict__ ds) {
  const Dev& d = ds[blockIdx.y];
  const int64_t sweep = *d.sweep_ctr;
  const int64_t total = d.chains_per_cell > 0 ? (int64_t)d.C * d.C * d.chains_per_cell : d.n;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  int cell;
  int64_t k;
  if (d.chains_per_cell > 0) {
    cell = (int)(i / d.chains_per_cell);
    k = i % d.chains_per_cell;
  } else {
    cell = cell_of_slot(d, i);
    k = i - d.cell_start[cell];
  }
  int n_c = d.cell_start[cell + 1] - d.cell_start[cell];
  double dx, dy;
  bool ok = iso_direction_capped(d, sweep, cell, k, dx, dy);
  d.chain_dir[i] = make_double2(dx, dy);
  int32_t start = 0;
  if (n_c > 0 && d.start_mode == 0) {
    Stream st(d.seed, kKindStart, (uint64_t)sweep, cell_key(d, cell), (uint64_t)k);
    uint64_t v = 0;
    if (!draw_index_capped(st, (uint64_t)n_c, v)) ok = false;
    start = (int32_t)v;
  }
  if (d.start_mode == 0) d.chain_start[i] = start;
  if (!ok) atomicOr(d.err, ERR_DRAW_CAP);
}

// Distinct-start negative control: one thread per cell shuffles [0, n_c)
// (Fisher-Yates) and chain k starts at list[k mod n_c].
__global__ void k_shuffle(const Dev* __restrict__ ds) {
  const Dev& d = ds[blockIdx.y];
  if (d.start_mode != 1) return;
  const int64_t sweep = *d.sweep_ctr;
  int cell = blockIdx.x * blockDim.x + threadIdx.x;
  if (cell >= d.C * d.C) return;
  int s0 = d.cell_start[cell];
  int n_c = d.cell_start[cell + 1] - s0;
  if (n_c <= 0) return;
  int32_t* list = d.shuffle + s0;
  for (int i = 0; i < n_c; ++i) list[i] = i;
  Stream st(d.seed, kKindShuffle, (uint64_t)sweep, cell_key(d, cell), 0);
  bool ok = true;
  for (int i = 0; i + 1 < n_c; ++i) {
    uint64_t v = 0;
    if (!draw_index_capped(st, (uint64_t)(n_c - i), v)) ok = false;
    int j = i + (int)v;
    int t = list[i]; list[i] = list[j]; list[j] = t;
  }
  int64_t n_m = chains_of(d, n_c);
  int64_t base = chain_base(d, cell);
  for (int64_t k = 0; k < n_m; ++k) d.chain_start[base + k] = list[k % n_c];
  if (!ok) atomicOr(d.err, ERR_DRAW_CAP);
}

// ---------------------------------------------------------------------------
// Walled simulation cells: one wavefront per active cell of colour perm[q]
// ---------------------------------------------------------------------------
// Meta word of a slot: an own disk's index into the cell's id-ordered list,
// or a frozen disk's id with the top bit set; all ones while staging finds
// the slot empty.
constexpr uint32_t kFrozenBit = 0x80000000u;
constexpr uint32_t kEmptySlot = 0xFFFFFFFFu;

// Lane of the smallest key (s, id) among the window's candidates, given the
// wave minimum mn of their high words hi (as argmin_lane); the ids are taken
// only on the rare path of equal high words: a frozen disk's from its meta
// word, an own disk's from the cell's id list.
__device__ __forceinline__ int argmin_lane_slots(double s, uint32_t m, const int32_t* own_gid,
                                                 unsigned hi, unsigned mn) {
  const uint64_t sb = (uint64_t)__double_as_longlong(s);
  uint64_t mask = __builtin_amdgcn_ballot_w64(hi == mn);  // not empty: some lane holds mn
  int wl = __builtin_ctzll(mask);
  if (__builtin_expect(mask != (1ull << wl), 0)) {  // equal high words: resolve on the full key
    uint32_t id = 0;
    if (hi == mn) id = (m & kFrozenBit) ? (m & ~kFrozenBit) : (uint32_t)own_gid[m];
    mask &= mask - 1;
    uint64_t bs = readlane_u64(sb, wl);
    uint32_t bi = (uint32_t)readlane_i32((int)id, wl);
    while (mask) {
      const int l = __ffsll((unsigned long long)mask) - 1;
      mask &= mask - 1;
      const uint64_t ls = readlane_u64(sb, l);
      const uint32_t li = (uint32_t)readlane_i32((int)id, l);
      if (ls < bs || (ls == bs && li < bi)) { bs = ls; bi = li; wl = l; }
    }
  }
  return wl;
}

__device__ __forceinline__ int32_t load_err(const Dev& d) {
  return __hip_atomic_load((const EC_GLOBAL(int32_t)*)d.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------
// The plain lifts and reflections of a chain, written out
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)p;
}

// A plain lift: the nearest disk in the window is not frozen and is hit within
// the remaining length, the window vouches for the move, and the moved centre
// stays inside the cell by eps on both axes, so neither wall comes first (with
// the wall distance (wall - v) / d rounded as the full decision rounds it, a
// centre that stops eps short of the wall leaves the wall farther by far more
// than the rounding); the centre may change bin.  This is exactly the full
// decision finding such a lift.  A plain reflection is the same with a frozen
// disk.  The loop runs both (the rejection variant: lifts only) until the event
// found is another one, or two distances agree to their high words (left to the
// general path with nothing changed), or n_ring reaches the limit.
//
// Every lane tests its own disk, with the winner's own values, between the
// steps of the wave minimum, whose results must wait two issue slots each.  The
// lanes that hold the minimum (one, or the loop is left) become the execution
// mask: the winner stores the moved centre itself, and a lane read is then a
// first-lane read, without the lane's index.  What the next window's address
// does not need stands behind its reads.  A reflection is computed in the
// winner's lane, beside the loop, and comes back into it.
// Written out by hand because the compiler has no form for that mask, puts the
// loop's exits through flags, and places what can wait before the reads.
// Registers are fixed: halves of a pair cannot be named otherwise.  Wait states
// kept: 2 from a vector write to its use by a DPP step, or of a scalar or vcc to
// a vector use; 1 to a lane read, or from a root or reciprocal estimate to its
// use.  Everything read from LDS has arrived where the code is left.  Every
// output is written before the last input has been read, so all are early
// clobbers: without that an input that dies here may be given v96, v97 or v120.
//
// Costs found by doubling single instructions and by adding idle ones (a
// wavefront alone on its SIMD): vector and scalar instructions 4 cycles, an LDS
// store 22 to 34 (by its width, whatever the lanes), an LDS read 8 to 15, a
// branch 10 where it is not taken and about 25 where it is, and a scalar
// instruction waits about 16 cycles for any vector instruction that wrote a
// scalar register just before, its own operand or not.  So words go to the other
// lanes by lane reads and records by lane writes, not through LDS; and the lane
// reads stand together, with vector work or the LDS store between them and the
// next scalar instruction (the contact sum and term stand where they do for that
// alone: 1M disks 72.4 -> 67.1 ms a sweep).
// Measured, ms a sweep: 1M disks 67.1 and 65k disks 60.0, against 84.7 and 72.8
// with what the winner has to tell sent through LDS and reflections left to the
// general path, and about 97 and 84 with the loop compiled from C++.
#define EC_W(x) x "\n\t"
// g = sqrt(x), correctly rounded, as sqrt_contact; h, r scratch
#define EC_SQRT(x, g, h, r)                                                                    \
  EC_W("v_rsq_f64_e32 " h ", " x) EC_W("s_nop 0")                                              \
  EC_W("v_mul_f64 " g ", " x ", " h) EC_W("v_mul_f64 " h ", " h ", 0.5")                       \
  EC_W("v_fma_f64 " r ", -" h ", " g ", 0.5") EC_W("v_fmac_f64_e32 " g ", " g ", " r)          \
  EC_W("v_fmac_f64_e32 " h ", " h ", " r) EC_W("v_fma_f64 " r ", -" g ", " g ", " x)           \
  EC_W("v_fmac_f64_e64 " g ", " r ", " h) EC_W("v_fma_f64 " r ", -" g ", " g ", " x)           \
  EC_W("v_fmac_f64_e64 " g ", " r ", " h)
// (qx, qy) = (x, y) / d, as div_pair; r, e scratch (qy may be x)
#define EC_DIV_PAIR(x, y, d, qx, qy, r, e)                                                     \
  EC_W("v_rcp_f64_e32 " r ", " d) EC_W("s_nop 0")                                              \
  EC_W("v_fma_f64 " e ", -" d ", " r ", 1.0") EC_W("v_fmac_f64_e64 " r ", " r ", " e)          \
  EC_W("v_fma_f64 " e ", -" d ", " r ", 1.0") EC_W("v_fmac_f64_e64 " r ", " r ", " e)          \
  EC_W("v_mul_f64 " qx ", " x ", " r) EC_W("v_fma_f64 " e ", -" d ", " qx ", " x)              \
  EC_W("v_fmac_f64_e64 " qx ", " e ", " r)                                                     \
  EC_W("v_mul_f64 " qy ", " y ", " r) EC_W("v_fma_f64 " e ", -" d ", " qy ", " y)              \
  EC_W("v_fmac_f64_e64 " qy ", " e ", " r)
// window of the mover in slot a_slot, whose lanes' slots are in v69: its reads
#define EC_READ_SLOTS                                                                          \
  EC_W("v_lshl_add_u32 v125, v69, 4, %[pos]")                                                  \
  EC_W("v_lshl_add_u32 v126, v69, 2, %[meta]")                                                 \
  EC_W("ds_read_b128 v[64:67], v125")                                                          \
  EC_W("ds_read_b32 v98, v126")                                                                \
  EC_W("v_lshl_add_u32 v125, %[a_slot], 4, %[pos]")                                            \
  EC_W("ds_read_b128 v[70:73], v125")
// walled cells: rows clamped to the grid
#define EC_READ_WINDOW                                                                         \
  EC_W("s_mul_hi_u32 %[t], %[a_slot], %[inv_g32]")                                             \
  EC_W("s_add_i32 %[u], %[t], %[offy]")                                                        \
  EC_W("s_or_b32 %[expect], %[a_slot], 0x80000000")                                            \
  EC_W("s_min_i32 %[u], %[u], %[top]")                                                         \
  EC_W("s_max_i32 %[u], %[u], -2")                                                             \
  EC_W("s_sub_i32 %[u], %[u], %[t]")                                                           \
  EC_W("s_mul_i32 %[u], %[u], %[gridb]")                                                       \
  EC_W("s_add_i32 %[u], %[u], %[a_slot]")                                                      \
  EC_W("v_add_u32_e32 v69, %[u], %[woff]")                                                     \
  EC_READ_SLOTS
// the moved centre changes bin, to one that is empty (a bin holds one centre):
// the old slot is emptied, and the disk's meta word and slot index move
#define EC_CHANGE_BIN                                                                          \
  EC_W("v_mov_b32_e32 v116, 0")                                                                \
  EC_W("v_mov_b32_e32 v117, 0x7ff80000")                                                       \
  EC_W("v_mov_b32_e32 v118, 0")                                                                \
  EC_W("v_mov_b32_e32 v119, 0x7ff80000")                                                       \
  EC_W("v_lshl_add_u32 v125, %[a_slot], 4, %[pos]")                                            \
  EC_W("ds_write_b128 v125, v[116:119]")                                                       \
  EC_W("v_lshl_add_u32 v125, v123, 2, %[meta]")                                                \
  EC_W("v_mov_b32_e32 v126, %[a_lidx]")                                                        \
  EC_W("ds_write_b32 v125, v126")                                                              \
  EC_W("v_lshl_add_u32 v125, %[a_lidx], 1, %[own_loc]")                                        \
  EC_W("ds_write_b16 v125, v123")
// one event; K numbers its labels, BACK is what stands at its end
#define EC_EVENT(K, IMAGE, TERM_IMAGE, WINDOW, LOG, STEP, BACK)                                                   \
  EC_W("s_waitcnt lgkmcnt(0)")                                                                 \
  /* contact distance */                                                                       \
  EC_W("v_add_f64 v[108:109], v[66:67], -v[72:73]")                                            \
  EC_W("v_add_f64 v[110:111], v[64:65], -v[70:71]")                                            \
  IMAGE                                                                                        \
  EC_W("v_mul_f64 v[112:113], v[108:109], -v[80:81]")                                          \
  EC_W("v_mul_f64 v[114:115], v[82:83], v[108:109]")                                           \
  EC_W("v_fmac_f64_e32 v[112:113], v[110:111], v[82:83]")                                      \
  EC_W("v_fmac_f64_e32 v[114:115], v[110:111], v[80:81]")                                      \
  EC_W("v_fma_f64 v[116:117], -v[112:113], v[112:113], %[sig2]")                               \
  EC_W("v_rsq_f64_e64 v[118:119], v[116:117]")                                                 \
  EC_W("v_min_f64 v[112:113], v[114:115], v[116:117]")                                         \
  EC_W("v_mul_f64 v[108:109], v[116:117], v[118:119]")                                         \
  EC_W("v_mul_f64 v[118:119], v[118:119], 0.5")                                                \
  EC_W("v_cmp_lt_f64_e64 vcc, 0, v[112:113]")                                                  \
  EC_W("v_fma_f64 v[110:111], -v[118:119], v[108:109], 0.5")                                   \
  EC_W("v_fmac_f64_e32 v[108:109], v[108:109], v[110:111]")                                    \
  EC_W("v_fmac_f64_e32 v[118:119], v[118:119], v[110:111]")                                    \
  EC_W("v_fma_f64 v[110:111], -v[108:109], v[108:109], v[116:117]")                            \
  EC_W("v_fmac_f64_e64 v[108:109], v[110:111], v[118:119]")                                    \
  EC_W("v_fma_f64 v[110:111], -v[108:109], v[108:109], v[116:117]")                            \
  EC_W("v_fmac_f64_e64 v[108:109], v[110:111], v[118:119]")                                    \
  EC_W("v_add_f64 v[96:97], v[114:115], -v[108:109]")                                          \
  EC_W("v_max_f64 v[96:97], v[96:97], 0")                                                      \
  EC_W("v_cndmask_b32_e64 v120, -1, v97, vcc")                                                 \
  /* moved centre, its slot, tests, wave minimum */                                            \
  EC_W("v_fma_f64 v[104:105], v[96:97], v[80:81], v[70:71]")                                   \
  EC_W("v_fma_f64 v[106:107], v[96:97], v[82:83], v[72:73]")                                   \
  EC_W("v_min_u32_dpp v121, v120, v120 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf")        \
  EC_W("v_add_f64 v[108:109], v[104:105], -%[mid]")                                            \
  EC_W("v_add_f64 v[110:111], v[106:107], -%[mid]")                                            \
  EC_W("v_min_u32_dpp v121, v121, v121 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf")        \
  EC_W("v_max_f64 v[108:109], |v[108:109]|, |v[110:111]|")                                     \
  EC_W("v_mul_f64 v[112:113], v[106:107], %[inv_b]")                                           \
  EC_W("v_min_u32_dpp v121, v121, v121 row_half_mirror row_mask:0xf bank_mask:0xf")            \
  EC_W("v_mul_f64 v[114:115], v[104:105], %[inv_b]")                                           \
  EC_W("v_cvt_i32_f64_e64 v112, v[112:113]")                                                   \
  EC_W("v_min_u32_dpp v121, v121, v121 row_mirror row_mask:0xf bank_mask:0xf")                 \
  EC_W("v_cvt_i32_f64_e64 v114, v[114:115]")                                                   \
  EC_W("v_add_f64 v[108:109], v[108:109], -%[inner]")                                          \
  EC_W("v_min_u32_dpp v121, v121, v121 row_bcast:15 row_mask:0xa bank_mask:0xf")               \
  EC_W("v_mad_u32_u24 v123, v112, %[gridb], v114")                                             \
  EC_W("v_add_f64 v[100:101], v[96:97], s[90:91]")                                             \
  EC_W("v_min_u32_dpp v121, v121, v121 row_bcast:31 row_mask:0xc bank_mask:0xf")               \
  EC_W("v_add_f64 v[110:111], v[96:97], -v[84:85]")                                            \
  EC_W("v_readlane_b32 %[kmin], v121, 63")                                                     \
  EC_W("v_and_b32_e64 v122, v101, v109")                                                       \
  EC_W("v_bitop3_b32 v122, v122, v111, v98 bitop3:0x40") /* a & b & ~c */                      \
  EC_W("v_cmp_eq_u32_e64 %[mask], %[kmin], v120")                                              \
  EC_W("v_bfi_b32 v122, %[low31], v123, v122")                                                 \
  /* the contact term */                                                                       \
  EC_W("v_add_f64 v[78:79], v[78:79], s[92:93]")                                               \
  EC_W("v_add_f64 v[112:113], v[64:65], -v[104:105]")                                          \
  EC_W("v_add_f64 v[114:115], v[66:67], -v[106:107]")                                          \
  EC_W("s_mov_b64 exec, %[mask]")                                                              \
  EC_W("v_readfirstlane_b32 %[t], v122")                                                       \
  EC_W("v_lshl_add_u32 v124, v123, 4, %[pos]")                                                 \
  TERM_IMAGE                                                                                   \
  EC_W("v_mul_f64 v[102:103], v[82:83], v[114:115]")                                           \
  EC_W("v_fmac_f64_e64 v[102:103], v[112:113], v[80:81]")                                      \
  EC_W("s_bcnt1_i32_b64 %[u], %[mask]")                                                        \
  EC_W("s_add_i32 %[u], %[u], -1")                                                             \
  EC_W("s_xor_b32 %[t], %[t], %[expect]")                                                      \
  EC_W("s_or_b32 %[u], %[u], %[t]")                                                            \
  EC_W("s_cbranch_scc1 3" K "f")                                                               \
  EC_W("4" K ":")                                                                              \
  EC_W("v_readfirstlane_b32 %[a_lidx], v98")                                                   \
  LOG                                                                                          \
  EC_W("v_readfirstlane_b32 %[a_slot], v69")                                                   \
  EC_W("v_readfirstlane_b32 %[slo], v96")                                                      \
  EC_W("v_readfirstlane_b32 %[shi], v97")                                                      \
  EC_W("v_readfirstlane_b32 s92, v102")                                                        \
  EC_W("v_readfirstlane_b32 s93, v103")                                                        \
  EC_W("v_readfirstlane_b32 s90, v100")                                                        \
  EC_W("v_readfirstlane_b32 s91, v101")                                                        \
  EC_W("ds_write_b128 v124, v[104:107]")                                                       \
  EC_W("s_mov_b64 exec, -1")                                                                   \
  STEP                                                                                         \
  WINDOW                                                                                       \
  /* (the disk of a lift is not frozen: its meta word is its own index) */                     \
  EC_W("v_writelane_b32 v94, %[slo], m0")                                                      \
  EC_W("v_writelane_b32 v95, %[shi], m0")                                                      \
  EC_W("v_writelane_b32 v99, %[a_lidx], m0")                                                   \
  EC_W("s_add_i32 m0, m0, 1")                                                                  \
  BACK
// beside the loop: ties, bin changes, reflections
#define EC_ASIDE(K, FROZEN)                                                                    \
  EC_W("3" K ":")                                                                              \
  EC_W("s_bcnt1_i32_b64 %[u], %[mask]")                                                        \
  EC_W("s_xor_b32 %[t], %[t], %[expect]")                                                      \
  EC_W("s_cmp_lg_u32 %[u], 1")                                                                 \
  EC_W("s_cbranch_scc1 2f")                                                                    \
  EC_W("s_cmp_ge_i32 %[t], 0")                                                                 \
  EC_W("s_cbranch_scc1 " FROZEN)                                                               \
  EC_CHANGE_BIN                                                                                \
  EC_W("s_branch 4" K "b")
#define EC_REFLECTION                                                                          \
  EC_W("6:")                                                                                   \
  /* plain but for the frozen bit? */                                                          \
  EC_W("v_bitop3_b32 v122, v101, v109, v111 bitop3:0x80") /* a & b & c */                      \
  EC_W("v_and_b32_e32 v122, v122, v98")                                                        \
  EC_W("s_nop 0")                                                                              \
  EC_W("v_readfirstlane_b32 %[t], v122")                                                       \
  EC_W("v_readfirstlane_b32 %[next], v123")                                                    \
  EC_W("s_cmp_ge_i32 %[t], 0")                                                                 \
  EC_W("s_cbranch_scc1 2f")                                                                    \
  EC_W("v_readfirstlane_b32 s90, v100")                                                        \
  EC_W("v_readfirstlane_b32 s91, v101")                                                        \
  EC_W("v_readfirstlane_b32 %[slo], v96")                                                      \
  EC_W("v_readfirstlane_b32 %[shi], v97")                                                      \
  EC_W("v_readfirstlane_b32 s92, v102")                                                        \
  EC_W("v_readfirstlane_b32 s93, v103")                                                        \
  /* the normal n = r / |r| of r (v112, v114) */                                               \
  EC_W("v_mul_f64 v[108:109], v[114:115], v[114:115]")                                         \
  EC_W("v_fmac_f64_e32 v[108:109], v[112:113], v[112:113]")                                    \
  EC_W("s_cmp_eq_u32 %[next], %[a_slot]")                                                      \
  EC_W("s_cbranch_scc1 8f")                                                                    \
  EC_CHANGE_BIN                                                                                \
  EC_W("8:")                                                                                   \
  EC_W("ds_write_b128 v124, v[104:107]")                                                       \
  EC_SQRT("v[108:109]", "v[110:111]", "v[116:117]", "v[118:119]")                              \
  EC_DIV_PAIR("v[112:113]", "v[114:115]", "v[110:111]", "v[108:109]", "v[112:113]",            \
              "v[116:117]", "v[118:119]")                                                      \
  /* u = d - 2 (d.n) n, and the new direction u / |u| */                                       \
  EC_W("v_mul_f64 v[114:115], v[82:83], v[112:113]")                                           \
  EC_W("v_fmac_f64_e32 v[114:115], v[80:81], v[108:109]")                                      \
  EC_W("v_mul_f64 v[114:115], v[114:115], -2.0")                                               \
  EC_W("v_fma_f64 v[110:111], v[114:115], v[108:109], v[80:81]")                               \
  EC_W("v_fma_f64 v[116:117], v[114:115], v[112:113], v[82:83]")                               \
  EC_W("v_mul_f64 v[118:119], v[116:117], v[116:117]")                                         \
  EC_W("v_fmac_f64_e32 v[118:119], v[110:111], v[110:111]")                                    \
  EC_SQRT("v[118:119]", "v[108:109]", "v[112:113]", "v[114:115]")                              \
  EC_DIV_PAIR("v[110:111]", "v[116:117]", "v[108:109]", "v[118:119]", "v[110:111]",            \
              "v[112:113]", "v[114:115]")                                                      \
  /* the guard of the new direction, and all of it to every lane */                            \
  EC_W("v_max_f64 v[108:109], |v[118:119]|, |v[110:111]|")                                     \
  EC_W("v_rcp_f64_e32 v[112:113], v[108:109]")                                                 \
  EC_W("v_readfirstlane_b32 s94, v118")                                                        \
  EC_W("v_readfirstlane_b32 s95, v119")                                                        \
  EC_W("v_mul_f64 v[112:113], v[112:113], %[reach]")                                           \
  EC_W("v_readfirstlane_b32 s96, v110")                                                        \
  EC_W("v_readfirstlane_b32 s97, v111")                                                        \
  EC_W("v_readfirstlane_b32 s98, v112")                                                        \
  EC_W("v_readfirstlane_b32 s99, v113")                                                        \
  EC_W("v_readfirstlane_b32 %[t], v98")                                                        \
  EC_W("s_mov_b64 exec, -1")                                                                   \
  EC_W("s_ashr_i32 %[offx], s95, 31")                                                          \
  EC_W("s_ashr_i32 %[offy], s97, 31")                                                          \
  EC_W("s_mul_i32 %[offx], %[offx], 3")                                                        \
  EC_W("s_mul_i32 %[offy], %[offy], 3")                                                        \
  EC_W("s_add_i32 %[offx], %[offx], -2")                                                       \
  EC_W("s_add_i32 %[offy], %[offy], -2")                                                       \
  EC_W("v_mov_b64_e32 v[80:81], s[94:95]")                                                     \
  EC_W("v_mov_b64_e32 v[82:83], s[96:97]")                                                     \
  EC_W("v_mov_b64_e32 v[84:85], s[98:99]")                                                     \
  EC_W("v_add_u32_e32 %[woff], %[offx], %[loff]")                                              \
  /* its record, kind 2: (2 ^ 1) << 29 | id */                                                 \
  EC_W("s_and_b32 %[t], %[t], 0x1fffffff")                                                     \
  EC_W("s_or_b32 %[t], %[t], 0x60000000")                                                      \
  EC_W("v_writelane_b32 v94, %[slo], m0")                                                      \
  EC_W("v_writelane_b32 v95, %[shi], m0")                                                      \
  EC_W("v_writelane_b32 v99, %[t], m0")                                                        \
  EC_W("s_add_i32 %[n_frozen], %[n_frozen], 1")                                                \
  /* the same disk goes on */                                                                  \
  EC_W("s_mov_b32 %[a_slot], %[next]")                                                         \
  EC_READ_WINDOW                                                                               \
  EC_W("s_add_i32 m0, m0, 1")                                                                  \
  EC_W("s_sub_i32 %[t], m0, %[limit]")                                                         \
  EC_W("s_cmp_eq_u32 %[t], 0")                                                                 \
  EC_W("s_cbranch_scc1 5f")                                                                    \
  EC_W("s_and_b32 %[t], %[t], 3")                                                              \
  EC_W("s_cmp_eq_u32 %[t], 0")                                                                 \
  EC_W("s_cbranch_scc1 1b")                                                                    \
  EC_W("s_cmp_eq_u32 %[t], 1")                                                                 \
  EC_W("s_cbranch_scc1 12b")                                                                   \
  EC_W("s_cmp_eq_u32 %[t], 2")                                                                 \
  EC_W("s_cbranch_scc1 13b")                                                                   \
  EC_W("s_branch 14b")
// the way out: at the limit (5), or with an event that is another one (2)
#define EC_LEAVE                                                                               \
  EC_W("5:")                                                                                   \
  EC_W("s_mov_b32 %[full], 1")                                                                 \
  EC_W("s_waitcnt lgkmcnt(0)")                                                                 \
  EC_W("v_add_f64 v[78:79], v[78:79], s[92:93]")                                               \
  EC_W("s_branch 9f")                                                                          \
  EC_W("2:")                                                                                   \
  EC_W("s_mov_b64 exec, -1")                                                                   \
  EC_W("s_mov_b32 %[full], 0")                                                                 \
  EC_W("s_waitcnt lgkmcnt(0)")                                                                 \
  EC_W("9:")                                                                                   \
  "s_nop 4"
// Four copies of the event, of which only the last looks at the limit and takes
// a branch: the loop is entered at the copy from which the limit is reached at the
// end of the last.
// The code is laid out so that no 8-byte instruction crosses an 8-byte boundary:
// in a run of such instructions each costs a cycle more where they do.  So 4-byte
// instructions come in pairs, single ones in their 8-byte encoding (_e64), and
// the loop starts 4 bytes past a 32-byte boundary.
#define EC_ENTER                                                                               \
  EC_W("s_or_b32 %[expect], %[a_slot], 0x80000000")                                            \
  EC_W("s_sub_i32 %[t], m0, %[limit]")                                                         \
  EC_W("s_and_b32 %[t], %[t], 3")                                                              \
  EC_W("s_cmp_eq_u32 %[t], 1")                                                                 \
  EC_W("s_cbranch_scc1 12f")                                                                   \
  EC_W("s_cmp_eq_u32 %[t], 2")                                                                 \
  EC_W("s_cbranch_scc1 13f")                                                                   \
  EC_W("s_cmp_eq_u32 %[t], 3")                                                                 \
  EC_W("s_cbranch_scc1 14f")                                                                   \
  EC_W(".p2align 5")                                                                           \
  EC_W("s_nop 0")                                                                              \
  EC_W("1:")
#define EC_BACK                                                                                \
  EC_W("s_cmp_lg_u32 m0, %[limit]")                                                            \
  EC_W("s_cbranch_scc1 1b")                                                                    \
  EC_W("s_branch 5f")
#define EC_FOUR(IMAGE, TERM_IMAGE, WINDOW, LOG, STEP, FROZEN)                                  \
  EC_ENTER                                                                                     \
  EC_EVENT("1", IMAGE, TERM_IMAGE, WINDOW, LOG, STEP, EC_W("12:"))                             \
  EC_EVENT("2", IMAGE, TERM_IMAGE, WINDOW, LOG, STEP, EC_W("13:"))                             \
  EC_EVENT("3", IMAGE, TERM_IMAGE, WINDOW, LOG, STEP, EC_W("14:"))                             \
  EC_EVENT("4", IMAGE, TERM_IMAGE, WINDOW, LOG, STEP, EC_BACK)                                 \
  EC_ASIDE("1", FROZEN)                                                                        \
  EC_ASIDE("2", FROZEN)                                                                        \
  EC_ASIDE("3", FROZEN)                                                                        \
  EC_ASIDE("4", FROZEN)
#define EC_LOOP(LOG, STEP, FROZEN, REFLECTION, UNDO)                                           \
  asm volatile(                                                                                \
      EC_FOUR(, , EC_READ_WINDOW, LOG, STEP, FROZEN)                                           \
      REFLECTION                                                                               \
      EC_LEAVE                                                                                 \
      : "+&{v[64:65]}"(p.x), "+&{v[66:67]}"(p.y), "+&{v69}"(widx), "+&{v[70:71]}"(ax),         \
        "+&{v[72:73]}"(ay), "+&{s[90:91]}"(nrem), "+&{s[92:93]}"(dacc), "+&{v[78:79]}"(sum),   \
        "+&{v[80:81]}"(dx), "+&{v[82:83]}"(dy), "+&{v[84:85]}"(guard), "+&{v94}"(rec_lo),      \
        "+&{v95}"(rec_hi), "+&{v98}"(m), "+&{v99}"(rec_tag), "=&{v[96:97]}"(s), "=&{v120}"(key), \
        [kmin] "=&s"(key_min), [full] "=&s"(full), [a_slot] "+&s"(a_slot),                     \
        [a_lidx] "+&s"(a_lidx), "+&{m0}"(n_ring), [offx] "+&s"(offx), [offy] "+&s"(offy),      \
        [n_frozen] "+&s"(n_frozen), [woff] "+&v"(woff), [mask] "=&s"(a_mask), [t] "=&s"(a_t),  \
        [u] "=&s"(a_u), [next] "=&s"(a_next), [slo] "=&s"(a_slo), [shi] "=&s"(a_shi),          \
        [expect] "=&s"(a_expect) UNDO                                                          \
      : [pos] "v"(pos_at), [meta] "v"(meta_at), [own_loc] "v"(own_loc_at), [loff] "v"(loff),   \
        [mid] "s"(mid), [inner] "s"(inner), [sig2] "s"(s_sig2), [inv_b] "s"(s_inv_b),          \
        [reach] "s"(s_reach), [gridb] "s"(s_gridb), [inv_g32] "s"(s_inv_g32),                  \
        [top] "s"(s_top), [limit] "s"(limit), [low31] "s"(0x7FFFFFFF)                          \
      : "vcc", "scc", "memory", "s94", "s95", "s96", "s97", "s98", "s99", "v100",              \
        "v101", "v102", "v103", "v104", "v105", "v106", "v107", "v108", "v109", "v110",        \
        "v111", "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119", "v121",        \
        "v122", "v123", "v124", "v125", "v126", "v127")
// The rejection variant's undo log of a plain lift: slots before and after, old
// position; then the next entry's addresses.
#define EC_UNDO_LOG                                                                            \
  EC_W("v_mov_b32_e32 v126, %[a_slot]")                                                        \
  EC_W("v_mov_b32_e32 v127, v123")                                                             \
  EC_W("ds_write_b64 %[uslot], v[126:127]")                                                    \
  EC_W("ds_write_b128 %[upos], v[70:73]")
#define EC_UNDO_STEP                                                                           \
  EC_W("v_add_u32_e32 %[uslot], 8, %[uslot]")                                                  \
  EC_W("v_add_u32_e32 %[upos], 16, %[upos]")
#define EC_UNDO_OPERANDS , [uslot] "+&v"(uslot_at), [upos] "+&v"(upos_at)

// One periodic cell: the window wraps around the box (an index i in [-nb, 2 nb)
// is brought into [0, nb) as the least of i and i + nb, then of i and i - nb,
// unsigned), and offsets take the nearest image.  The image number is the
// nearest integer to v / L, which is the one the definition's comparisons with
// L / 2 give but for |v| within rounding of L / 2; a disk that far away is
// never a plain lift's (its distance is above the guard, which stays 1e-9 below
// the free-flight cap L / 2 - sigma).  v - n L is then one rounding of v - L,
// v or v + L, as there.  A lift across the box edge is not plain (the moved
// centre's test against the walls of a cell is one against the box here).
// 256 disks: 28.8 -> 13.9 ms a sweep against the loop compiled from C++.
#define EC_READ_PERIODIC                                                                       \
  EC_W("s_mul_hi_u32 %[t], %[a_slot], %[inv_g32]")                                             \
  EC_W("s_mul_i32 %[u], %[t], %[gridb]")                                                       \
  EC_W("s_or_b32 %[expect], %[a_slot], 0x80000000")                                            \
  EC_W("s_sub_i32 %[u], %[a_slot], %[u]")                                                      \
  EC_W("s_add_i32 %[u], %[u], %[offx]")                                                        \
  EC_W("s_add_i32 %[t], %[t], %[offy]")                                                        \
  EC_W("v_add_u32_e32 v125, %[u], %[lx]")                                                      \
  EC_W("v_add_u32_e32 v126, %[t], %[ly]")                                                      \
  EC_W("v_add_u32_e32 v127, %[gridb], v125")                                                   \
  EC_W("v_add_u32_e32 v69, %[gridb], v126")                                                    \
  EC_W("v_min_u32_e32 v125, v125, v127")                                                       \
  EC_W("v_min_u32_e32 v126, v126, v69")                                                        \
  EC_W("v_subrev_u32_e32 v127, %[gridb], v125")                                                \
  EC_W("v_subrev_u32_e32 v69, %[gridb], v126")                                                 \
  EC_W("v_min_u32_e32 v125, v125, v127")                                                       \
  EC_W("v_min_u32_e64 v126, v126, v69")                                                        \
  EC_W("v_mad_u32_u24 v69, v126, %[gridb], v125")                                              \
  EC_READ_SLOTS
#define EC_NEAREST_IMAGE                                                                       \
  EC_W("v_mul_f64 v[86:87], v[108:109], %[inv_L]")                                             \
  EC_W("v_mul_f64 v[88:89], v[110:111], %[inv_L]")                                             \
  EC_W("v_rndne_f64_e32 v[86:87], v[86:87]")                                                   \
  EC_W("v_rndne_f64_e32 v[88:89], v[88:89]")                                                   \
  EC_W("v_fma_f64 v[108:109], -v[86:87], %[L], v[108:109]")                                    \
  EC_W("v_fma_f64 v[110:111], -v[88:89], %[L], v[110:111]")
#define EC_TERM_IMAGE                                                                          \
  EC_W("v_fma_f64 v[112:113], -v[88:89], %[L], v[112:113]")                                    \
  EC_W("v_fma_f64 v[114:115], -v[86:87], %[L], v[114:115]")
#define EC_LOOP_PERIODIC                                                                       \
  asm volatile(                                                                                \
      EC_FOUR(EC_NEAREST_IMAGE, EC_TERM_IMAGE, EC_READ_PERIODIC, , , "2f")                     \
      EC_LEAVE                                                                                 \
      : "+&{v[64:65]}"(p.x), "+&{v[66:67]}"(p.y), "+&{v69}"(wsl), "+&{v[70:71]}"(ax),          \
        "+&{v[72:73]}"(ay), "+&{s[90:91]}"(nrem), "+&{s[92:93]}"(dacc), "+&{v[78:79]}"(acc),   \
        "+&{v94}"(rec_lo), "+&{v95}"(rec_hi), "+&{v98}"(m), "+&{v99}"(rec_tag), "=&{v[96:97]}"(s), \
        "=&{v120}"(key), [kmin] "=&s"(key_min), [full] "=&s"(full), [a_slot] "+&s"(a_slot),    \
        [a_lidx] "+&s"(a), "+&{m0}"(n_ring), [mask] "=&s"(a_mask), [t] "=&s"(a_t),             \
        [u] "=&s"(a_u), [next] "=&s"(a_next), [slo] "=&s"(a_slo), [shi] "=&s"(a_shi),          \
        [expect] "=&s"(a_expect)                                                               \
      : "{v[80:81]}"(dx), "{v[82:83]}"(dy), "{v[84:85]}"(guard), [pos] "v"(pos_at),            \
        [meta] "v"(meta_at), [own_loc] "v"(slot_of_at), [lx] "v"(lx), [ly] "v"(ly),            \
        [L] "s"(s_L), [inv_L] "s"(s_inv_L), [mid] "s"(s_mid), [inner] "s"(s_inner),            \
        [sig2] "s"(s_sig2), [inv_b] "s"(s_inv_b), [gridb] "s"(s_nb), [inv_g32] "s"(s_inv_n32), \
        [offx] "s"(offx), [offy] "s"(offy), [limit] "s"(kDigestBatch), [low31] "s"(0x7FFFFFFF) \
      : "vcc", "scc", "memory", "v86", "v87", "v88", "v89", "v100", "v101", "v102", "v103",    \
        "v104", "v105", "v106", "v107", "v108", "v109", "v110", "v111", "v112", "v113",        \
        "v114", "v115", "v116", "v117", "v118", "v119", "v121", "v122", "v123", "v124",        \
        "v125", "v126", "v127")

// Both components of (x, y) / den: the compiler's own FP64 division sequence
// (reciprocal estimate, two Newton steps, quotient, one correction with the
// exact residual), with the reciprocal formed once and without the range
// scaling and special-value fix-up, which do nothing for a denominator between
// 2^-300 and 2^301 and numerators that are 0 or above 2^-960: the same
// quotients.
__device__ __forceinline__ void div_pair(double x, double y, double den, double& qx, double& qy) {
  double r = __builtin_amdgcn_rcp(den);
  r = fma(r, fma(-den, r, 1.0), r);
  r = fma(r, fma(-den, r, 1.0), r);
  qx = x * r;
  qx = fma(fma(-den, qx, x), r, qx);
  qy = y * r;
  qy = fma(fma(-den, qy, y), r, qy);
}

__device__ __forceinline__ int hi_word(double v) {
  return (int)((uint64_t)__double_as_longlong(v) >> 32);
}

// One active cell of colour phase q (Sec. 3.4, steps 3-6): stage the own
// disks and the frozen band into LDS, run the cell's chains, write back.  One
// wavefront; base is its LDS region.  Returns early, with d.err set, when a
// capacity check fails.  REJ 1: a chain that reaches a wall or a frozen disk
// is rejected and undone (the rejection variant of Sec. 3.4); each lift is
// logged for the undo.
//
// What bounds it: a cell's events are one serial chain, and a wavefront alone
// on its SIMD issues one instruction per 4 to 5 cycles whatever its kind.  Four
// things cost more: a scalar instruction that reads what a vector one has just
// written (about 15 cycles of waiting), a branch (10 cycles not taken, 25
// taken), the FP64 reciprocal square root (16) and the LDS round trip (60 for
// the reads, 90 behind a store).  So plain lifts (above) make their tests in
// vector registers as sign bits that are ANDed into one word and read once.
template <int REJ>
__device__ __forceinline__ void phase_cell(const Dev& d, const int64_t sweep, const SweepDraws& dr,
                                           const int q, const int blk, unsigned char* const base,
                                           const int lane) {
  const int half = d.C >> 1;
  const int colour = (dr.perm >> (2 * (q & 3))) & 3;
  const int cx = 2 * (blk % half) + (colour & 1);
  const int cy = 2 * (blk / half) + (colour >> 1);
  const int cell = cy * d.C + cx;
  const double ox = (double)cx * d.w, oy = (double)cy * d.w;
  const double L = d.L, half_L = d.half_L, w = d.w, sigma = d.sigma, sig2 = d.sig2;
  const int gridb = d.gridb, nb = d.nb;
  const int nslots = gridb * gridb;  // one slot per bin
  // Slots are counted from that of the first own bin (bin (0, 0) of nb x nb;
  // the frozen band's bins are -2, -1, nb and nb + 1): slot = by * gridb + bx.
  const int qoff = 2 * gridb + 2;
  // row of an own slot: floor(slot / gridb) as (slot * m) >> 32 with m =
  // ceil(2^32 / gridb), exact for 0 <= slot < gridb^2 <= 100^2
  const uint32_t inv_g32 = 0xFFFFFFFFu / (uint32_t)gridb + 1u;

  const CellLds lay = cell_lds_layout(gridb, d.cap_own, REJ == 1);
  double2* const pos_all = (double2*)(base + lay.off_pos);
  uint32_t* const meta_all = (uint32_t*)(base + lay.off_meta);
  double2* const pos = pos_all + kSlotPad + qoff;
  uint32_t* const meta = meta_all + kSlotPad + qoff;
  int32_t* own_gid = (int32_t*)(base + lay.off_own_gid);
  uint16_t* own_loc = (uint16_t*)(base + lay.off_own_loc);
  // the id staging buffer of the rank sort lies in the position slots, which
  // are filled only after the sort
  int32_t* tmp = (int32_t*)(base + lay.off_pos);
  // REJ 1 only: per logged lift the old position, then (slot before, slot after)
  double2* undo_pos = (double2*)(base + lay.off_undo);
  int2* undo_slot = (int2*)(undo_pos + kUndoCap);

  // ---- stage ---------------------------------------------------------------
  // Lists of disks to read, one per lane, so that their bounds come in one trip
  // to memory: lanes 0-11 the frozen band, lane 12 the cell's own list.  The
  // band is the centres of the 8 neighbouring cells within sigma of this cell.
  // Only a neighbour's regions that face this cell are read (its wall strips
  // are wider than sigma, so they hold every such centre): the strip along the
  // shared wall of an edge neighbour, the corner region of a diagonal one.  A
  // region row is one range of the list, a region column three.
  int s0 = 0, s1 = 0;
  if (lane < 13) {
    // neighbour at (cx + ox_, cy + oy_), region row ry; lanes 0-2 below, 3-5
    // above, 6-8 the three rows to the left, 9-11 to the right
    const int k3 = lane % 3;
    const int ox_ = lane < 6 ? k3 - 1 : (lane < 9 ? -1 : 1), oy_ = lane < 3 ? -1 : (lane < 6 ? 1 : 0);
    const int ry = lane < 3 ? 2 : (lane < 6 ? 0 : k3);
    const int rx0 = ox_ < 0 ? 2 : 0, rx1 = ox_ > 0 ? 0 : 2;
    const int nc = ((cy + oy_ + d.C) % d.C) * d.C + (cx + ox_ + d.C) % d.C;
    const int k0 = kRegions * nc + 3 * ry;
    s0 = gload(lane == 12 ? d.cell_start + cell : d.reg_start + k0 + rx0);
    s1 = gload(lane == 12 ? d.cell_start + cell + 1 : d.reg_start + k0 + rx1 + 1);
  }
  if (__builtin_amdgcn_ballot_w64(s0 < 0 || s1 < s0 || s1 - s0 > d.cap_own || (int64_t)s1 > d.n) != 0) {
    if (lane == 0) atomicOr(d.err, ERR_OWN_CAP);
    return;
  }
  const int start = readlane_i32(s0, 12), n_own = readlane_i32(s1, 12) - start;
  // own disks, sorted by id: each lane counts the smaller ids of its own
  for (int i = lane; i < ((n_own + 3) & ~3); i += 64)
    tmp[i] = i < n_own ? gload(d.cell_ids + start + i) : 0x7FFFFFFF;
  wave_sync();
  for (int i = lane; i < n_own; i += 64) {
    int v = tmp[i];
    int r = 0;
    for (int j = 0; j < n_own; j += 4) {
      const int4 t4 = *(const int4*)(tmp + j);
      r += (t4.x < v ? 1 : 0) + (t4.y < v ? 1 : 0) + (t4.z < v ? 1 : 0) + (t4.w < v ? 1 : 0);
    }
    own_gid[r] = v;
  }
  wave_sync();
  const double2 nan2 = make_double2(__builtin_nan(""), __builtin_nan(""));
  for (int s = lane; s < nslots + 2 * kSlotPad; s += 64) {
    pos_all[s] = nan2;
    meta_all[s] = kEmptySlot;
  }
  wave_sync();

  // own disks into bins 0..nb-1: a bin's diagonal is below sigma, so it holds
  // at most one centre of a configuration without overlaps (a second one is
  // reported as a capacity error)
  for (int k = lane; k < n_own; k += 64) {
    int g = own_gid[k];
    double vx = local_coord(gload(d.x + g), dr.sx, ox, L, half_L);
    double vy = local_coord(gload(d.y + g), dr.sy, oy, L, half_L);
    int bx = (int)floor(vx * d.inv_b), by = (int)floor(vy * d.inv_b);
    bx = bx < 0 ? 0 : (bx > nb - 1 ? nb - 1 : bx);
    by = by < 0 ? 0 : (by > nb - 1 ? nb - 1 : by);
    const int s = by * gridb + bx;
    if (atomicCAS(&meta[s], kEmptySlot, (uint32_t)k) != kEmptySlot) {
      atomicOr(d.err, ERR_BIN_CAP);
      continue;
    }
    pos[s] = make_double2(vx, vy);
    own_loc[k] = (uint16_t)s;
  }
  // frozen disks, in the two outer rings of bins: the twelve lists read as one
  {
    int upto = lane < 12 ? s1 - s0 : 0;  // disks of this lane's list and those before
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
      const int before = __shfl_up(upto, off, 16);
      if ((lane & 15) >= off) upto += before;
    }
    const int n_band = readlane_i32(upto, 11);
    for (int i = lane; i < n_band; i += 64) {
      int at = readlane_i32(s0, 0) + i;
#pragma unroll
      for (int r = 1; r < 12; ++r) {
        const int first = readlane_i32(upto, r - 1);
        at = i >= first ? readlane_i32(s0, r) + (i - first) : at;
      }
      int g = gload(d.cell_ids + at);
      double vx = local_coord(gload(d.x + g), dr.sx, ox, L, half_L);
      double vy = local_coord(gload(d.y + g), dr.sy, oy, L, half_L);
      if (vx >= -sigma && vx <= w + sigma && vy >= -sigma && vy <= w + sigma) {
        int bx = (int)floor(vx * d.inv_b), by = (int)floor(vy * d.inv_b);
        bx = bx < -2 ? -2 : (bx > nb + 1 ? nb + 1 : bx);
        by = by < -2 ? -2 : (by > nb + 1 ? nb + 1 : by);
        const int s = by * gridb + bx;
        if (atomicCAS(&meta[s], kEmptySlot, (uint32_t)g | kFrozenBit) != kEmptySlot) {
          atomicOr(d.err, ERR_BIN_CAP);
          continue;
        }
        pos[s] = make_double2(vx, vy);
      }
    }
  }
  wave_sync();
  if (load_err(d) != 0) return;  // a capacity check failed somewhere: do not run chains

  // ---- chains --------------------------------------------------------------
  const int64_t n_m = chains_of(d, n_own);
  const int64_t cbase = chain_base(d, cell);
  double acc = gload(d.acc_delta + cell);
  uint32_t n_lift = 0, n_frozen = 0, n_wall = 0;
  uint64_t h = 0;
  int n_ring = 0;            // event records held in the lanes (lane k: record k)
  uint64_t ring_first = 0;    // digest index of record 0
  uint32_t rec_lo = 0, rec_hi = 0, rec_tag = 0;
  // LDS addresses of the plain-lift loop
  const uint32_t pos_at = lds_address(pos), meta_at = lds_address(meta), own_loc_at = lds_address(own_loc);
  // lane = lx + 8 ly: one bin of an 8 x 8 window per lane, a window row in 8
  // neighbouring lanes
  const int loff = (lane >> 3) * gridb + (lane & 7);  // this lane's slot inside a window
  const double inv_b = d.inv_b;
  // A window of 8 x 8 bins reaches 2 bins behind the moving disk's bin and 5
  // ahead of it along each axis.  With sigma/2 < b < sigma/sqrt(2), the 2b
  // behind cover sigma, and a move of length t keeps its sigma-neighbourhood
  // inside the window whenever t * max(|dx|, |dy|) <= 5b - sigma - eps: then no
  // disk outside the window can be hit first, and the event found in the window
  // is exact.  Rows are clamped to the grid (nothing is staged beyond it).
  // Columns are not: a window across the left or right edge reads the end of
  // the row before or the start of the row after, which are slots of the same
  // cell (or, before the first and after the last slot, kSlotPad empty ones);
  // more disks tested change no minimum.
  const double eps = 1e-9 * sigma;
  const double reach = 5.0 * d.b - sigma - eps;
  // a plain lift keeps the moved centre in [eps, w - eps] on both axes, that is
  // |v - mid| < inner (see there)
  // (the loop's scalar operands, read as such)
  const double mid = readlane_f64(0.5 * w, 0), inner = readlane_f64(0.5 * w - eps, 0);
  const double s_sig2 = readlane_f64(sig2, 0), s_inv_b = readlane_f64(inv_b, 0);
  const double s_reach = readlane_f64(reach * (1.0 - 0x1p-20), 0);
  const int s_gridb = uniform_i32(gridb), s_inv_g32 = uniform_i32((int)inv_g32), s_top = uniform_i32(nb - 6);
  const int use_window = uniform_i32(d.search == 0 ? 1 : 0);
  const uint64_t wall_x_id = (uint64_t)d.n, wall_y_id = (uint64_t)d.n + 1, end_id = (uint64_t)d.n + 3;
  int aborted = 0;
  int stop = 0;  // nonzero once a poll sees the device error word set

  // draws of chain 0; later, those of chain k + 1 and the device error word
  // are loaded while chain k runs (their latency is then hidden)
  int32_t nxt_start = n_m > 0 ? gload(d.chain_start + cbase) : 0;
  double2 nxt_dir = n_m > 0 ? gload(d.chain_dir + cbase) : make_double2(1.0, 0.0);
  int32_t nxt_err = load_err(d);
  for (int64_t k = 0; k < n_m && aborted == 0; ++k) {
    int j = uniform_i32(nxt_start);
    if (j < 0 || j >= n_own) j = 0;  // guarded: the draw kernel writes indices below n_own
    double dx = nxt_dir.x, dy = nxt_dir.y;
    stop = uniform_i32(nxt_err);
    if (k + 1 < n_m) {
      nxt_start = gload(d.chain_start + cbase + k + 1);
      nxt_dir = gload(d.chain_dir + cbase + k + 1);
    }
    nxt_err = load_err(d);
    // per direction: the window's origin relative to the mover's bin, and the
    // longest move it vouches for, reach / max(|dx|, |dy|) from the hardware's
    // reciprocal (good to about 2^-24), made smaller by 2^-20: only ever a guard
    double dsafe;
    int offx, offy;
#define EC_SET_DIRECTION()                                                          \
    do {                                                                            \
      const double lead_ = fmax(fabs(dx), fabs(dy));                                \
      dsafe = use_window ? s_reach * __builtin_amdgcn_rcp(lead_) : -1.0;            \
      offx = uniform_i32(dx < 0.0 ? -5 : -2);                                       \
      offy = uniform_i32(dy < 0.0 ? -5 : -2);                                       \
    } while (0)
    // the 8 x 8 window of the mover in slot a_slot: this lane's slot, its
    // position and meta word, and the mover's position
#define EC_WINDOW()                                                                 \
    do {                                                                            \
      const int by_ = (int)__umulhi((uint32_t)a_slot, inv_g32);                     \
      const int wy_ = max(min(by_ + offy, nb - 6), -2);                             \
      widx = (a_slot + offx + (wy_ - by_) * gridb) + loff;                          \
      p = pos[widx];                                                                \
      m = meta[widx];                                                               \
      const double2 ap_ = pos[a_slot];                                              \
      ax = ap_.x;                                                                   \
      ay = ap_.y;                                                                   \
    } while (0)
    const int slot_j = (int)own_loc[j];  // read while the direction is set
    EC_SET_DIRECTION();
    int a_slot = uniform_i32(slot_j);
    int a_lidx = j;
    double ax, ay;
    double nrem = -d.ell;  // minus the chain length left
    // event cap and abort polling, both at the digest flush (every 64 events
    // of the cell): the error word loaded at the previous flush (or chain
    // start) is read, the next load is issued, and the chain's event count,
    // ring_first - ev0 at a flush, is held against the cap (so a chain makes
    // at most kMaxEventsPerChain + 63 events)
    const uint64_t ev0 = ring_first + (uint64_t)n_ring;
    int capped = 0;
#define EC_POLL()                                                                   \
    do {                                                                            \
      stop |= uniform_i32(nxt_err);                                                 \
      nxt_err = load_err(d);                                                        \
      capped = (ring_first - ev0 >= (uint64_t)kMaxEventsPerChain) ? 1 : 0;          \
    } while (0)
#define EC_FLUSH()                                                                  \
    do {                                                                            \
      uint32_t lifts_;                                                              \
      h ^= digest_records(rec_lo, rec_hi, rec_tag, lane, kDigestBatch, ring_first, own_gid, lifts_); \
      if (REJ == 0) n_lift += lifts_;                                               \
      ring_first += kDigestBatch;                                                   \
      n_ring = 0;                                                                   \
      EC_POLL();                                                                    \
    } while (0)
    // REJ 1: the chain's undo log, contact sum and lifts (counted once accepted)
    int n_undo = 0;
    double chain_acc = 0.0;
    uint32_t chain_lifts = 0;
    int widx;
    double2 p;
    uint32_t m;
    EC_WINDOW();
    int ended = 0;  // the chain length is used up

    while (ended == 0 && stop == 0 && capped == 0) {
      // contact distance of the disk in this lane's window slot, its high word
      // (all ones: no contact) and the wave minimum of those
      double s;
      uint32_t key, key_min;
      // plain lifts and reflections, up to the next digest of 64 records (none
      // where no window is to vouch for a move: every event is then the exact
      // search's, below)
      s = 0.0;
      key = key_min = 0xFFFFFFFFu;
      while (use_window != 0) {
        const int before = n_ring;
        double sum = REJ == 1 ? chain_acc : acc, dacc = 0.0;
        int limit = kDigestBatch, full, a_t, a_u, a_next, a_slo, a_shi, a_expect, woff = loff + offx;
        uint64_t a_mask;
        nrem = readlane_f64(nrem, 0);
        a_slot = uniform_i32(a_slot);
        a_lidx = uniform_i32(a_lidx);
        n_ring = uniform_i32(n_ring);
        n_frozen = (uint32_t)uniform_i32((int)n_frozen);
        offx = uniform_i32(offx);
        offy = uniform_i32(offy);
        if (REJ == 1) {
          // the log's end is a limit too; with a full log no lift is plain
          // (whose move would be the general path's error)
          double guard = n_undo == kUndoCap ? -1.0 : dsafe;
          if (n_undo < kUndoCap) limit = min(limit, n_ring + kUndoCap - n_undo);
          limit = uniform_i32(limit);
          uint32_t upos_at = lds_address(undo_pos + n_undo), uslot_at = lds_address(undo_slot + n_undo);
          EC_LOOP(EC_UNDO_LOG, EC_UNDO_STEP, "2f", "", EC_UNDO_OPERANDS);
          chain_acc = sum;
          n_undo += n_ring - before;
          chain_lifts += (uint32_t)(n_ring - before);
        } else {
          double& guard = dsafe;
          EC_LOOP("", "", "6f", EC_REFLECTION, );
          acc = sum;
        }
        if (full == 0) break;
        if (n_ring == kDigestBatch) {
          EC_FLUSH();
          if (stop != 0 || capped != 0) break;
        }
      }
      if (stop != 0 || capped != 0) continue;  // leaves the event loop

      // ---- the chain end: every disk of the window is farther than the length
      // left (by the high word of its distance), and the move by that length is
      // one the window vouches for and ends eps inside the cell (as for plain
      // lifts)
      const double rem = -nrem;
      {
        const double ex = fma(rem, dx, ax), ey = fma(rem, dy, ay);
        const double wall = fmax(fabs(ex - mid), fabs(ey - mid)) - inner;
        const int calm = hi_word(rem - dsafe) & hi_word(wall) & (int)(key_min > (uint32_t)hi_word(rem) ? 0x80000000 : 0);
        if (uniform_i32(calm) < 0) {
          const int es = uniform_i32((int)(ey * inv_b) * gridb + (int)(ex * inv_b));
          const uint64_t sb = (uint64_t)__double_as_longlong(rem);
          writelane3(rec_lo, rec_hi, rec_tag, (uint32_t)sb, (uint32_t)(sb >> 32),
                     ((uint32_t)(EV_END ^ 1) << 29) | (uint32_t)end_id, n_ring);
          if (es != a_slot) {  // to a bin that is empty
            pos[a_slot] = nan2;
            meta[es] = (uint32_t)a_lidx;
            own_loc[a_lidx] = (uint16_t)es;
          }
          pos[es] = make_double2(ex, ey);
          if (REJ == 1) {  // accepted: its contact sum and lifts count
            acc = acc + chain_acc;
            n_lift += chain_lifts;
          }
          ended = 1;
          __builtin_amdgcn_wave_barrier();
          if (__builtin_expect(++n_ring == kDigestBatch, 0)) EC_FLUSH();
          continue;
        }
      }
      // ---- any other event.  The nearest disk of the window:
      double best_s = INFINITY, wpx = 0.0, wpy = 0.0;  // (a disk can be hit exactly when best_s is finite)
      uint32_t wm = kFrozenBit;
      int w_slot = 0;
      if (key_min != 0xFFFFFFFFu) {
        const int win = argmin_lane_slots(s, m, own_gid, key, key_min);
        best_s = readlane_f64(s, win);
        wm = (uint32_t)readlane_i32((int)m, win);
        wpx = readlane_f64(p.x, win);
        wpy = readlane_f64(p.y, win);
        w_slot = readlane_i32(widx, win);
      }
      // Where the move to the nearest disk, or by the length left if that is
      // shorter, is one the window vouches for and ends eps inside the cell, it
      // is the event (as for plain lifts): a contact or the chain end.
      double step = fmin(best_s, rem);
      double nax = fma(step, dx, ax), nay = fma(step, dy, ay);
      int kind = best_s < rem ? ((wm & kFrozenBit) ? EV_FROZEN : EV_LIFT) : EV_END;
      {
        const double wall = fmax(fabs(nax - mid), fabs(nay - mid)) - inner;
        kind |= hi_word(step - dsafe) & hi_word(wall) & (int)0x80000000;
      }
      kind = uniform_i32(kind);
      if (__builtin_expect(kind >= 0, 0)) {
        // The full decision: distances to the walls of the cell ahead, (wall -
        // v) / d as a product with 1/d, clamped at 0; first the nearest disk,
        // then the x and the y wall, where strictly nearer.
        const double idx = (dx != 0.0) ? 1.0 / dx : 1.0, idy = (dy != 0.0) ? 1.0 / dy : 1.0;
        const double wallx = (dx > 0.0) ? w : ((dx < 0.0) ? 0.0 : INFINITY);
        const double wally = (dy > 0.0) ? w : ((dy < 0.0) ? 0.0 : INFINITY);
        double tx = (wallx - ax) * idx;
        tx = (tx < 0.0) ? 0.0 : tx;
        double ty = (wally - ay) * idy;
        ty = (ty < 0.0) ? 0.0 : ty;
#define EC_DECIDE()                                                                 \
        do {                                                                        \
          double e_ = best_s;                                                       \
          kind = (wm & kFrozenBit) ? EV_FROZEN : EV_LIFT;                           \
          if (tx < e_) { e_ = tx; kind = EV_WALL_X; }                               \
          if (ty < e_) { e_ = ty; kind = EV_WALL_Y; }                               \
          if (!(e_ < rem)) kind = EV_END;                                           \
          kind = uniform_i32(kind);                                                 \
          step = fmin(e_, rem);                                                     \
        } while (0)
        EC_DECIDE();
        if (__builtin_expect(uniform_i32(step <= dsafe ? 1 : 0) == 0, 0)) {
          // the window cannot vouch for this event: exact search over every slot
          double ls = INFINITY;
          uint32_t lid = 0xFFFFFFFFu;
          int lslot = 0;
          bool found = false;
          for (int i = lane; i < nslots; i += 64) {
            const int sl = i - qoff;
            const double2 q2 = pos[sl];
            double s2;
            if (contact(q2.x - ax, q2.y - ay, dx, dy, sig2, s2)) {
              const uint32_t m2 = meta[sl];
              const uint32_t i2 = (m2 & kFrozenBit) ? (m2 & ~kFrozenBit) : (uint32_t)own_gid[m2];
              if (s2 < ls || (s2 == ls && i2 < lid)) { ls = s2; lid = i2; lslot = sl; found = true; }
            }
          }
          const int fl = wave_argmin_all(ls, lid, found);
          best_s = INFINITY;
          wm = kFrozenBit;
          if (fl >= 0) {
            best_s = readlane_f64(ls, fl);
            w_slot = readlane_i32(lslot, fl);
            wm = (uint32_t)uniform_i32((int)meta[w_slot]);
            // read into scalar registers here, so no load is left in flight
            // where this rare path rejoins the event path
            const double2 q2 = pos[w_slot];
            wpx = readlane_f64(q2.x, 0);
            wpy = readlane_f64(q2.y, 0);
          }
          EC_DECIDE();
        }
#undef EC_DECIDE
        nax = fma(step, dx, ax);
        nay = fma(step, dy, ay);
      }
      kind &= 7;
      // bin of the moved centre, which lies in [0, w] up to rounding: truncation
      // gives 0..nb-1, and nb on the far wall
      const int ns = uniform_i32(min((int)(nay * inv_b), nb - 1) * gridb + min((int)(nax * inv_b), nb - 1));
      // REJ 1: a wall or a frozen disk rejects the chain
      const bool rejected = REJ == 1 && kind != EV_END && kind != EV_LIFT;
      {
        // event record for the digest, kept by lane n_ring
        const uint32_t eid = kind == EV_END ? (uint32_t)end_id
                             : (kind == EV_WALL_X ? (uint32_t)wall_x_id
                                                  : (kind == EV_WALL_Y ? (uint32_t)wall_y_id
                                                                       : (wm & ~kFrozenBit)));
        const uint64_t sb = (uint64_t)__double_as_longlong(step);
        writelane3(rec_lo, rec_hi, rec_tag, (uint32_t)sb, (uint32_t)(sb >> 32),
                   ((uint32_t)(kind ^ 1) << 29) | eid, n_ring);
      }
      if (REJ == 1 && kind == EV_LIFT && n_undo == kUndoCap) {
        // a full log stops the sweep with an error
        if (lane == 0) atomicOr(d.err, ERR_UNDO_CAP);
        stop = 1;
      }
      if (rejected) {
        // undo every logged lift, latest first: each disk goes back to the
        // slot it left (a slot vacated in between was refilled only by moves
        // that are undone before it) and to its old position
        if (lane == 0) {
          bool lost = false;  // the slot to leave is empty already: another disk's undo left it
          for (int u = n_undo - 1; u >= 0; --u) {
            const int2 sl = undo_slot[u];
            const double2 old = undo_pos[u];
            lost |= __builtin_isnan(pos[sl.y].x);
            if (sl.y != sl.x) {
              const uint32_t mv = meta[sl.y];
              pos[sl.y] = nan2;
              meta[sl.x] = mv;
              own_loc[(int)mv] = (uint16_t)sl.x;
            }
            pos[sl.x] = old;
          }
          if (lost) atomicOr(d.err, ERR_BIN_CAP);
        }
        n_undo = 0;
        if (kind == EV_FROZEN) n_frozen += 1;
        else n_wall += 1;
      } else {
        // store the moved disk (all lanes the same); move it to another bin if
        // it crossed a bin edge
        const int from = a_slot;
        if (ns != a_slot) {
          if (__builtin_expect(!__builtin_isnan(readlane_f64(pos[ns].x, 0)), 0)) {
            if (lane == 0) atomicOr(d.err, ERR_BIN_CAP);
          } else {
            pos[a_slot] = nan2;
            meta[ns] = (uint32_t)a_lidx;
            own_loc[a_lidx] = (uint16_t)ns;
            a_slot = ns;
          }
        }
        pos[a_slot] = make_double2(nax, nay);
        if (REJ == 1 && kind == EV_LIFT && stop == 0) {
          undo_pos[n_undo] = make_double2(ax, ay);
          undo_slot[n_undo] = make_int2(from, a_slot);
          n_undo += 1;
        }
      }
      __builtin_amdgcn_wave_barrier();
      if (__builtin_expect(++n_ring == kDigestBatch, 0)) EC_FLUSH();
      if (rejected) {
        ended = 1;
      } else if (kind == EV_LIFT) {
        // straight chain: the hit disk goes on in the same direction
        const double dacc = fma(wpx - nax, dx, (wpy - nay) * dy);
        if (REJ == 1) {
          chain_acc = chain_acc + dacc;
          chain_lifts += 1;
        } else {
          acc = acc + dacc;
        }
        nrem = nrem + step;
        a_slot = w_slot;
        a_lidx = (int)wm;
      } else if (kind == EV_END) {
        ended = 1;
        if (REJ == 1) {  // accepted: its contact sum and lifts count
          acc = acc + chain_acc;
          n_lift += chain_lifts;
        }
      } else {
        nrem = nrem + step;
        if (__builtin_expect(kind == EV_FROZEN, 1)) {
          // mirror the direction about the contact normal (both square roots
          // are correctly rounded; their arguments, about sigma^2 and 1, lie in
          // the range of sqrt_contact)
          const double rx = wpx - nax, ry = wpy - nay;
          acc = acc + fma(rx, dx, ry * dy);
          n_frozen += 1;
          double nx, ny;
          div_pair(rx, ry, sqrt_contact(fma(rx, rx, ry * ry)), nx, ny);
          const double tt = -2.0 * fma(dx, nx, dy * ny);
          const double ux = fma(tt, nx, dx), uy = fma(tt, ny, dy);
          div_pair(ux, uy, sqrt_contact(fma(ux, ux, uy * uy)), dx, dy);
          EC_SET_DIRECTION();
        } else {
          // a wall: reverse the normal component of the direction
          n_wall += 1;
          if (kind == EV_WALL_X) {
            dx = -dx;
            offx = -7 - offx;
          } else {
            dy = -dy;
            offy = -7 - offy;
          }
        }
      }
      // window of the next event (the stores above are seen: LDS operations
      // of one wave complete in order)
      EC_WINDOW();
    }
#undef EC_POLL
#undef EC_FLUSH
    if (ended == 0) {
      // stopped by another wave's error, or this chain reached the event cap
      if (stop == 0 && lane == 0) {
        atomicOr(d.err, ERR_EVENT_CAP);
        if (atomicAdd(d.err + 1, 1) == 0) {
          double* g = d.dbg;
          g[0] = (double)cell; g[1] = (double)k; g[2] = (double)sweep; g[3] = (double)q;
          g[4] = ax; g[5] = ay; g[6] = dx; g[7] = dy; g[8] = -nrem; g[9] = (double)a_slot;
          g[10] = (double)own_gid[a_lidx]; g[11] = (double)n_own;
        }
      }
      aborted = 1;
    }
#undef EC_WINDOW
#undef EC_SET_DIRECTION
  }

  // ---- does every disk have its slot? --------------------------------------
  // The written-out loop and the short way to the chain end store into the bin
  // of the moved centre without looking whether it is empty.  It is, unless
  // disks overlapped.  One look per disk and sweep here, where one per event
  // would cost a trip to LDS and a branch each.  (An undo looks for itself: it
  // can give a lost disk back under another's name.)  If not, the cell is left
  // as it was before the phase.
  wave_sync();
  {
    bool lost = false;
    for (int k = lane; k < n_own; k += 64) {
      const int at = (int)own_loc[k];
      lost |= !slot_kept(meta[at], (uint32_t)k, pos[at].x);
    }
    if (__builtin_amdgcn_ballot_w64(lost) != 0) {
      if (lane == 0) atomicOr(d.err, ERR_BIN_CAP);
      return;
    }
  }

  // ---- write back: old position + local displacement, wrapped --------------
  uint32_t last_lifts;
  h ^= digest_records(rec_lo, rec_hi, rec_tag, lane, n_ring, ring_first, own_gid, last_lifts);
  if (REJ == 0) n_lift += last_lifts;
  // The cell's id list is sorted again by the regions of the moved disks:
  // the neighbours of later colour phases stage their frozen band from the
  // regions that face them.  The list keeps its range [start, start + n_own)
  // (disks stay in their cell), and the region starts are rewritten; both
  // are published with the positions.  LDS: the meta words are free now and
  // hold the 9 region counts and the 9 fill cursors; own_loc takes each
  // disk's region once its slot has been read.
  uint32_t* const rcnt = meta_all;
  if (lane < 2 * kRegions) rcnt[lane] = 0u;
  wave_sync();
  for (int k = lane; k < n_own; k += 64) {
    int g = own_gid[k];
    double2 v = pos[(int)own_loc[k]];
    double px = gload(d.x + g), py = gload(d.y + g);
    double v0x = local_coord(px, dr.sx, ox, L, half_L);
    double v0y = local_coord(py, dr.sy, oy, L, half_L);
    double nx = px + (v.x - v0x);
    double ny = py + (v.y - v0y);
    if (nx < 0.0) nx += L; else if (nx >= L) nx -= L;
    if (ny < 0.0) ny += L; else if (ny >= L) ny -= L;
    gstore(d.x + g, nx);
    gstore(d.y + g, ny);
    // (from the cell-local position, which differs from the one a neighbour
    // computes from (nx, ny) by a few ulps of L, far inside the strip margin)
    const int r = 3 * strip_of(v.y, w, d.strip) + strip_of(v.x, w, d.strip);
    own_loc[k] = (uint16_t)r;
    atomicAdd(&rcnt[r], 1u);
  }
  wave_sync();
  if (lane == 0) {
    uint32_t run = (uint32_t)start;
    for (int r = 0; r < kRegions; ++r) {
      gstore(d.reg_start + kRegions * cell + r, (int32_t)run);
      rcnt[kRegions + r] = run;
      run += rcnt[r];
    }
  }
  wave_sync();
  for (int k = lane; k < n_own; k += 64) {
    const uint32_t at = atomicAdd(&rcnt[kRegions + (int)own_loc[k]], 1u);
    gstore(d.cell_ids + at, own_gid[k]);
  }
  if (lane == 0) {
    gstore(d.acc_delta + cell, acc);
    EC_GLOBAL(unsigned long long)* c = (EC_GLOBAL(unsigned long long)*)(d.acc_cnt + (size_t)cell * CNT_NCOL);
    c[CNT_LIFTS] += n_lift;
    c[CNT_FROZEN] += n_frozen;
    c[CNT_WALLS] += n_wall;
    c[CNT_CHAINS] += (uint64_t)n_m;
    gstore(d.cell_digest + cell, (unsigned long long)h);
    atomicAdd(&d.digest_ring[sweep % kDigestRing], h * (2ull * (uint64_t)cell + 1ull));
  }
}

// Colour phase q of a sweep: one launch per phase, one wavefront per active
// cell; the launch boundary separates the phases.
template <int REJ>
__global__ void __launch_bounds__(256) k_phase(const Dev* __restrict__ ds, int q) {
  const Dev& d = ds[blockIdx.y];
  const int64_t sweep = *d.sweep_ctr;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int half = d.C >> 1;
  const int blk = blockIdx.x * d.cells_per_block + wave;
  if (blk >= half * half) return;  // the whole wave leaves; no workgroup barrier follows
  const SweepDraws dr = *d.draws;
  phase_cell<REJ>(d, sweep, dr, q, blk, lds_raw + (size_t)wave * d.lds_per_cell, lane);
}

// All four colour phases of a sweep in one launch.  The phases order only
// neighbouring cells: a cell of phase q reads the disks of its eight
// neighbours (frozen band) and writes its own, so it must follow the
// neighbours of earlier phases and precede those of later ones, while cells
// farther apart share nothing.  Each wavefront takes tickets from a counter
// in phase order (ticket = q * C^2/4 + block), waits until the neighbours of
// earlier phases have published this sweep's epoch, runs the cell and
// publishes its own epoch.  Every cell then reads exactly the positions the
// phase-by-phase schedule gives it, so the results are identical; a cell no
// longer waits for the slowest cell of the previous phase anywhere in the
// system.
//
// Progress: a wave waits only for cells with smaller tickets, which were
// taken by waves already running, so by induction over tickets every wait
// ends.  Every wait is also bounded by d.dep_wait_ticks (100 MHz clock) and
// abandoned when any wave has set d.err: on either, the wave sets or sees the
// error and leaves, and the sweep reports it.
template <int REJ>
__global__ void __launch_bounds__(256) k_sweep_cells(const Dev* __restrict__ ds) {
  const Dev& d = ds[blockIdx.y];
  const int64_t sweep = *d.sweep_ctr;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  unsigned char* const base = lds_raw + (size_t)wave * d.lds_per_cell;
  const SweepDraws dr = *d.draws;
  const int half = d.C >> 1;
  const int per_phase = half * half;
  // as many workers as one phase has cells (a batch launches for its largest system)
  if (blockIdx.x * d.cells_per_block + wave >= per_phase) return;
  const int64_t epoch = sweep + 1;
  // phase of each colour, two bits per colour
  int phase_of = 0;
  for (int q = 0; q < 4; ++q) phase_of |= q << (2 * ((dr.perm >> (2 * q)) & 3));

  for (;;) {
    int t = 0;
    if (lane == 0) t = atomicAdd(d.queue, 1);
    t = __builtin_amdgcn_readfirstlane(t);
    if (t >= 4 * per_phase) break;
    const int q = t / per_phase;
    const int blk = t - q * per_phase;
    const int colour = (dr.perm >> (2 * q)) & 3;
    const int cx = 2 * (blk % half) + (colour & 1);
    const int cy = 2 * (blk / half) + (colour >> 1);
    if (q > 0) {
      // lanes 0-7 watch the eight neighbours; those of earlier phases count
      bool need = false;
      int nc = 0;
      if (lane < 8) {
        const int k = lane < 4 ? lane : lane + 1;  // the 3 x 3 block without its centre
        const int ncx = (cx + (k % 3) - 1 + d.C) % d.C;
        const int ncy = (cy + (k / 3) - 1 + d.C) % d.C;
        nc = ncy * d.C + ncx;
        need = ((phase_of >> (2 * ((ncx & 1) | ((ncy & 1) << 1)))) & 3) < q;
      }
      const uint64_t t0 = wall_clock64();
      bool ok = true;
      for (;;) {
        // the limit is tested first, so a limit of 0 fails every wait
        if (wall_clock64() - t0 >= (uint64_t)d.dep_wait_ticks) {
          if (lane == 0) atomicOr(d.err, ERR_DEP_WAIT);
          ok = false;
          break;
        }
        const bool ready =
            !need || __hip_atomic_load(d.cell_done + nc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == epoch;
        if (__builtin_amdgcn_ballot_w64(!ready) == 0) break;
        if (__builtin_amdgcn_readfirstlane(load_err(d)) != 0) {
          ok = false;
          break;
        }
        __builtin_amdgcn_s_sleep(4);
      }
      if (!ok) break;
      // the neighbours' write-backs are visible to the staging loads below
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    phase_cell<REJ>(d, sweep, dr, q, blk, base, lane);
    // this cell's write-back before its flag
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    if (lane == 0)
      __hip_atomic_store(d.cell_done + (cy * d.C + cx), epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(load_err(d)) != 0) break;
    wave_sync();  // LDS reads of this cell before the next cell's staging writes
  }
}

// ---------------------------------------------------------------------------
// Batched sweep with a ready queue: one launch runs every cell of every
// system of a batch.  A cell is ready once its earlier-phase neighbours in its
// own system are done (the only order the colour phases impose, Sec. 3.4 step
// 4); ready cells are appended to a queue, and persistent wavefronts take
// them in order, so no wavefront holds a slot while it waits for a
// neighbour, and no system waits for the slowest cell of another.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int cell_phase(int phase_of, int C, int cell) {
  const int cx = cell % C, cy = cell / C;
  return (phase_of >> (2 * ((cx & 1) | ((cy & 1) << 1)))) & 3;
}
__device__ __forceinline__ int phase_map(int perm) {  // phase of each colour, two bits per colour
  int phase_of = 0;
  for (int q = 0; q < 4; ++q) phase_of |= q << (2 * ((perm >> (2 * q)) & 3));
  return phase_of;
}

__device__ __forceinline__ void queue_push(const ReadyQueue& rq, int32_t epoch, int64_t task) {
  const int r = atomicAdd(rq.hdr + QH_RESERVE, 1);
  rq.tasks[r] = task;
  // the task word before its flag
  __hip_atomic_store(rq.flags + r, epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// New sweep: counters cleared, epoch advanced (one thread).
__global__ void k_queue_reset(ReadyQueue rq) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    rq.hdr[QH_READ] = 0;
    rq.hdr[QH_RESERVE] = 0;
    rq.hdr[QH_EPOCH] += 1;
    rq.hdr[QH_ABORT] = 0;
  }
}

// Count every cell's earlier-phase neighbours; cells with none (the first
// phase) are ready at once.  One thread per cell, grid y = system, in the order
// of the work in one of its cells: a sweep is four cells deep, so those of the
// densest systems are the ones to start with.
__global__ void k_queue_prep(const Dev* __restrict__ ds, ReadyQueue rq) {
  const int sys = rq.order[blockIdx.y];
  const Dev& d = ds[sys];
  const int ncell = d.C * d.C;
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncell) return;
  const int phase_of = phase_map(d.draws->perm);
  const int q = cell_phase(phase_of, d.C, c);
  const int cx = c % d.C, cy = c / d.C;
  int n = 0;
  for (int k = 0; k < 9; ++k) {
    if (k == 4) continue;
    const int nc = ((cy + k / 3 - 1 + d.C) % d.C) * d.C + (cx + k % 3 - 1 + d.C) % d.C;
    n += cell_phase(phase_of, d.C, nc) < q ? 1 : 0;
  }
  const int g = rq.base[sys] + c;
  rq.dep[g] = n;
  if (n == 0) queue_push(rq, rq.hdr[QH_EPOCH], ((int64_t)sys << 32) | (uint32_t)c);
}

// Persistent wavefronts: take the next queue slot, wait until it is
// published, run that cell, then count it off at its later-phase neighbours
// and append those that become ready.  Every slot below the cell total is
// published eventually: if every wave waited, every published cell would be
// done, and the not-done cell of smallest phase would have all its
// earlier-phase neighbours done, hence be published -- a contradiction.  Each
// wait is also bounded (the first system's dep_wait_ticks) and given up once
// any wave has flagged an abort.
template <int REJ>
__global__ void __launch_bounds__(256) k_queue_cells(const Dev* __restrict__ ds, ReadyQueue rq,
                                                     int lds_stride) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  // the waves of a workgroup take cells of any system: regions of the largest size
  unsigned char* const base = lds_raw + (size_t)wave * lds_stride;
  const int32_t epoch = __hip_atomic_load(rq.hdr + QH_EPOCH, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint64_t limit = (uint64_t)ds[0].dep_wait_ticks;
  for (;;) {
    int t = 0;
    if (lane == 0) t = atomicAdd(rq.hdr + QH_READ, 1);
    t = __builtin_amdgcn_readfirstlane(t);
    if (t >= rq.total) break;
    const uint64_t t0 = wall_clock64();
    bool ok = true;
    for (;;) {
      int f = 0, ab = 0;
      if (lane == 0) {
        f = __hip_atomic_load(rq.flags + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ab = __hip_atomic_load(rq.hdr + QH_ABORT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      f = __builtin_amdgcn_readfirstlane(f);
      ab = __builtin_amdgcn_readfirstlane(ab);
      if (f == epoch) break;
      if (ab != 0) { ok = false; break; }
      if (wall_clock64() - t0 >= limit) {
        if (lane == 0) {
          atomicOr(ds[0].err, ERR_DEP_WAIT);
          atomicExch(rq.hdr + QH_ABORT, 1);
        }
        ok = false;
        break;
      }
      __builtin_amdgcn_s_sleep(4);
    }
    if (!ok) break;
    // the slot, and the write-backs of the cell's earlier-phase neighbours,
    // are visible to the loads below
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    const int64_t task = rq.tasks[t];
    // (read as scalars, so that the record is read by scalar loads)
    const int sys = uniform_i32((int)(task >> 32)), cell = uniform_i32((int)(uint32_t)task);
    const Dev& d = ds[sys];
    const int64_t sweep = *d.sweep_ctr;
    const SweepDraws dr = *d.draws;
    const int phase_of = phase_map(dr.perm);
    const int q = cell_phase(phase_of, d.C, cell);
    const int cx = cell % d.C, cy = cell / d.C;
    const int blk = (cy >> 1) * (d.C >> 1) + (cx >> 1);
    // Waves that share a SIMD: the one whose cell holds more work issues first,
    // since a sweep ends with the fourth of a densest system's cells and each of
    // them runs at a third of its speed beside two waves of equal priority.
    // (16 systems of 4.6e3 to 2.6e5 disks, eta 0.30 to 0.71: 39.7 ms per sweep
    // without, 35.3 to 36.9 with it; the order of the queue alone gives 0.5 ms.)
    const int priority = uniform_i32(d.wave_priority);
    if (priority == 1) __builtin_amdgcn_s_setprio(1);
    if (priority == 2) __builtin_amdgcn_s_setprio(2);
    if (priority == 3) __builtin_amdgcn_s_setprio(3);
    phase_cell<REJ>(d, sweep, dr, q, blk, base, lane);
    __builtin_amdgcn_s_setprio(0);
    if (__builtin_amdgcn_readfirstlane(load_err(d)) != 0) {
      if (lane == 0) atomicExch(rq.hdr + QH_ABORT, 1);
      break;
    }
    // this cell's write-back before its neighbours count it off
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    if (lane < 8) {
      const int k = lane < 4 ? lane : lane + 1;  // the 3 x 3 block without its centre
      const int nc = ((cy + k / 3 - 1 + d.C) % d.C) * d.C + (cx + k % 3 - 1 + d.C) % d.C;
      if (cell_phase(phase_of, d.C, nc) > q) {
        const int g = rq.base[sys] + nc;
        const int left = __hip_atomic_fetch_add(rq.dep + g, -1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if (left == 1) queue_push(rq, epoch, ((int64_t)sys << 32) | (uint32_t)nc);
      }
    }
    wave_sync();  // LDS reads of this cell before the next cell's staging writes
  }
}

// After the launch: if a wave gave up (an error in some system, or a wait
// limit), mark every system of the batch, since their sweeps are unfinished.
__global__ void k_queue_check(const Dev* __restrict__ ds, ReadyQueue rq) {
  const Dev& d = ds[blockIdx.y];
  if (threadIdx.x == 0 && rq.hdr[QH_ABORT] != 0) atomicOr(d.err, ERR_ABANDONED);
}

// ---------------------------------------------------------------------------
// Striped decomposition with rejection (Sec. 3.4, Fig. 3 "stripes"; Sec. 4):
// C stripes of width w span the box; on even sweeps they are horizontal and
// chains run along x, on odd sweeps vertical with chains along y, each chain
// with a random sign (a chain and its reverse are proposed alike, and a chain
// is rejected exactly when its reverse is).  Colour phase q runs every stripe
// k with (k & 1) == first ^ q, one wavefront each; a chain that hits a disk
// of a neighbouring stripe is rejected and undone.
// The search is a brute-force minimum over the stripe's disks and the frozen
// disks of its two neighbours within sigma of it (nearest image along the
// stripe, flights capped at L/2 - sigma as in one periodic box).
// ---------------------------------------------------------------------------
template <int DUMMY>
__global__ void __launch_bounds__(64) k_stripe_phase(const Dev* __restrict__ ds, int q) {
  const Dev& d = ds[blockIdx.y];
  const int64_t sweep = *d.sweep_ctr;
  const SweepDraws dr = *d.draws;
  const int k = 2 * (int)blockIdx.x + ((dr.perm ^ q) & 1);
  if (k >= d.C) return;  // the whole wave leaves
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int lane = threadIdx.x;
  const int cap_own = d.stripe_cap_own, cap_fr = d.stripe_cap_frozen, cap_undo = d.stripe_undo;
  double* own_a = (double*)lds_raw;
  double* own_v = own_a + cap_own;
  double* fr_a = own_v + cap_own;
  double* fr_v = fr_a + cap_fr;
  double* undo_a = fr_v + cap_fr;
  int32_t* own_gid = (int32_t*)(undo_a + cap_undo);
  int32_t* tmp = own_gid + cap_own;
  int32_t* fr_gid = tmp + cap_own;
  int32_t* undo_i = fr_gid + cap_fr;
  int32_t* n_fr_sh = undo_i + cap_undo;

  double* const along = (sweep & 1) ? d.y : d.x;
  const double* const across = (sweep & 1) ? d.x : d.y;
  const double L = d.L, half_L = d.half_L, sigma = d.sigma, sig2 = d.sig2, cap = d.cap;
  const double origin = (double)k * d.w;

  // ---- stage: own disks in id order, frozen disks of the two neighbours
  const int start = d.cell_start[k];
  const int n_own = d.cell_start[k + 1] - start;
  if (n_own < 0 || n_own > cap_own) {
    if (lane == 0) atomicOr(d.err, ERR_OWN_CAP);
    return;
  }
  for (int i = lane; i < n_own; i += 64) tmp[i] = d.cell_ids[start + i];
  if (lane == 0) *n_fr_sh = 0;
  wave_sync();
  for (int i = lane; i < n_own; i += 64) {
    const int v = tmp[i];
    int r = 0;
    for (int j = 0; j < n_own; ++j) r += (tmp[j] < v) ? 1 : 0;
    own_gid[r] = v;
  }
  wave_sync();
  for (int i = lane; i < n_own; i += 64) {
    const int g = own_gid[i];
    own_a[i] = along[g];
    own_v[i] = local_coord(across[g], dr.sx, origin, L, half_L);
  }
  for (int side = -1; side <= 1; side += 2) {
    const int nk = (k + side + d.C) % d.C;
    const int s0 = d.cell_start[nk], s1 = d.cell_start[nk + 1];
    for (int t = s0 + lane; t < s1; t += 64) {
      const int g = d.cell_ids[t];
      const double v = local_coord(across[g], dr.sx, origin, L, half_L);
      if (v >= -sigma && v <= d.w + sigma) {
        const int slot = atomicAdd(n_fr_sh, 1);
        if (slot < cap_fr) {
          fr_a[slot] = along[g];
          fr_v[slot] = v;
          fr_gid[slot] = g;
        } else {
          atomicOr(d.err, ERR_OWN_CAP);
        }
      }
    }
  }
  wave_sync();
  const int n_fr = min(*n_fr_sh, cap_fr);
  if (__builtin_amdgcn_readfirstlane(load_err(d)) != 0) return;

  // ---- chains
  const int64_t n_m = chains_of(d, n_own);
  const int64_t cbase = chain_base(d, k);
  double acc = d.acc_delta[k];
  uint64_t n_lift = 0, n_frozen = 0, n_pseudo = 0, h = 0, n_ev = 0;
  bool stop = false;
  for (int64_t c = 0; c < n_m && !stop; ++c) {
    int a = uniform_i32(d.chain_start[cbase + c]);
    if (a < 0 || a >= n_own) a = 0;  // guarded: the draw kernel writes indices below n_own
    // the chain's sign: the top bit of the first word of its direction stream
    Stream ss(d.seed, kKindDir, (uint64_t)sweep, cell_key(d, k), (uint64_t)c);
    const bool neg = (ss.next() >> 63) != 0;
    double rem = d.ell, chain_acc = 0.0;
    uint64_t chain_lifts = 0;
    int n_undo = 0;
    int64_t events = 0;
    for (;;) {
      if (++events > kMaxEventsPerChain || (events % kAbortPollEvents) == 0) {
        if (events > kMaxEventsPerChain) {
          if (lane == 0) atomicOr(d.err, ERR_EVENT_CAP);
          stop = true;
          break;
        }
        if (uniform_i32(load_err(d)) != 0) { stop = true; break; }
      }
      const double aa = own_a[a], av = own_v[a];
      double ls = INFINITY;
      uint32_t lid = 0xFFFFFFFFu;
      int lj = -1;  // own index, or cap_own + frozen index
      for (int j = lane; j < n_own + n_fr; j += 64) {
        if (j == a) continue;
        const bool own = j < n_own;
        const int f = j - n_own;
        double ra = (own ? own_a[j] : fr_a[f]) - aa;
        if (ra < -half_L) ra += L; else if (ra >= half_L) ra -= L;
        if (neg) ra = -ra;
        const double rv = (own ? own_v[j] : fr_v[f]) - av;
        const double disc = fma(-rv, rv, sig2);
        if (ra > 0.0 && disc > 0.0) {
          double s = ra - sqrt(disc);
          if (s < 0.0) s = 0.0;
          const uint32_t gid = (uint32_t)(own ? own_gid[j] : fr_gid[f]);
          if (s < ls || (s == ls && gid < lid)) { ls = s; lid = gid; lj = j; }
        }
      }
      const int wl = wave_argmin(ls, lid, lj >= 0);
      double best_s = INFINITY;
      int bj = -1;
      uint32_t bgid = 0;
      if (wl >= 0) {
        best_s = readlane_f64(ls, wl);
        bj = readlane_i32(lj, wl);
        bgid = (uint32_t)readlane_i32((int)lid, wl);
      }
      const double lim = best_s < rem ? best_s : rem;
      if (lim > cap) {
        // a free flight beyond the nearest-image range: moved in pieces
        h ^= digest_term(EV_PSEUDO, (uint64_t)d.n + 2, cap, n_ev++);
        if (n_undo == cap_undo) {
          if (lane == 0) atomicOr(d.err, ERR_UNDO_CAP);
          stop = true;
          break;
        }
        if (lane == 0) { undo_i[n_undo] = a; undo_a[n_undo] = aa; }
        n_undo += 1;
        double na = neg ? aa - cap : aa + cap;
        if (na >= L) na -= L; else if (na < 0.0) na += L;
        if (lane == 0) own_a[a] = na;
        wave_sync();
        rem = rem - cap;
        n_pseudo += 1;
        continue;
      }
      if (!(best_s < rem)) {
        h ^= digest_term(EV_END, (uint64_t)d.n + 3, rem, n_ev++);
        double na = neg ? aa - rem : aa + rem;
        if (na >= L) na -= L; else if (na < 0.0) na += L;
        if (lane == 0) own_a[a] = na;
        wave_sync();
        acc = acc + chain_acc;  // accepted
        n_lift += chain_lifts;
        break;
      }
      const bool frozen = bj >= n_own;
      h ^= digest_term(frozen ? EV_FROZEN : EV_LIFT, bgid, best_s, n_ev++);
      if (n_undo == cap_undo) {
        if (lane == 0) atomicOr(d.err, ERR_UNDO_CAP);
        stop = true;
        break;
      }
      if (lane == 0) { undo_i[n_undo] = a; undo_a[n_undo] = aa; }
      n_undo += 1;
      double na = neg ? aa - best_s : aa + best_s;
      if (na >= L) na -= L; else if (na < 0.0) na += L;
      if (lane == 0) own_a[a] = na;
      wave_sync();
      rem = rem - best_s;
      if (frozen) {
        // a disk of a neighbouring stripe: the chain is rejected and undone
        n_frozen += 1;
        if (lane == 0)
          for (int u = n_undo - 1; u >= 0; --u) own_a[undo_i[u]] = undo_a[u];
        wave_sync();
        break;
      }
      double r = own_a[bj] - na;
      if (r < -half_L) r += L; else if (r >= half_L) r -= L;
      chain_acc = chain_acc + (neg ? -r : r);
      chain_lifts += 1;
      a = bj;
    }
  }
  wave_sync();
  for (int i = lane; i < n_own; i += 64) along[own_gid[i]] = own_a[i];
  if (lane == 0) {
    d.acc_delta[k] = acc;
    unsigned long long* cn = d.acc_cnt + (size_t)k * CNT_NCOL;
    cn[CNT_LIFTS] += n_lift;
    cn[CNT_FROZEN] += n_frozen;
    cn[CNT_CHAINS] += (uint64_t)n_m;
    cn[CNT_PSEUDO] += n_pseudo;
    d.cell_digest[k] = h;
    atomicAdd(&d.digest_ring[sweep % kDigestRing], h * (2ull * (uint64_t)k + 1ull));
  }
}

// ---------------------------------------------------------------------------
// One periodic cell (C = 1): all N disks in LDS, brute-force search with the
// minimum image; flights longer than L/2 - sigma are split (free-flight cap).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(64) k_periodic(const Dev* __restrict__ ds) {
  const Dev& d = ds[blockIdx.y];
  const int64_t sweep = *d.sweep_ctr + 1;  // (no k_prep before it)
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int lane = threadIdx.x;
  const int n = (int)d.n;
  double* px = (double*)lds_raw;
  double* py = px + n;
  int32_t* tmp = (int32_t*)(py + n);
  const double L = d.L, half_L = d.half_L, sig2 = d.sig2, cap = d.cap;
  for (int i = lane; i < n; i += 64) { px[i] = d.x[i]; py[i] = d.y[i]; }
  int64_t n_m = d.chains_per_cell > 0 ? d.chains_per_cell : n;
  if (d.start_mode == 1) {
    wave_sync();
    if (lane == 0) {
      for (int i = 0; i < n; ++i) tmp[i] = i;
      Stream st(d.seed, kKindShuffle, (uint64_t)sweep, cell_key(d, 0), 0);
      for (int i = 0; i + 1 < n; ++i) {
        int j = i + (int)draw_index(st, (uint64_t)(n - i));
        int t = tmp[i]; tmp[i] = tmp[j]; tmp[j] = t;
      }
    }
  }
  wave_sync();
  double acc = d.acc_delta[0];
  uint64_t n_lift = 0, n_pseudo = 0, h = 0, n_ev = 0;

  for (int64_t k = 0; k < n_m; ++k) {
    int a;
    if (d.start_mode == 1) {
      a = tmp[k % n];
    } else {
      Stream st(d.seed, kKindStart, (uint64_t)sweep, cell_key(d, 0), (uint64_t)k);
      a = (int)draw_index(st, (uint64_t)n);
    }
    double dx, dy;
    chain_direction(d, sweep, 0, k, dx, dy);
    double rem = d.ell;
    double ax = px[a], ay = py[a];
    int64_t n_events = 0;
    for (;;) {
      if (++n_events > kMaxEventsPerChain) {
        if (lane == 0) atomicOr(d.err, ERR_EVENT_CAP);
        break;
      }
      double ls = INFINITY;
      int lj = -1;
      for (int j = lane; j < n; j += 64) {
        if (j == a) continue;
        double rx = px[j] - ax, ry = py[j] - ay;
        if (rx < -half_L) rx += L; else if (rx >= half_L) rx -= L;
        if (ry < -half_L) ry += L; else if (ry >= half_L) ry -= L;
        double s;
        if (contact(rx, ry, dx, dy, sig2, s)) {
          if (s < ls) { ls = s; lj = j; }  // j rises with the loop: lowest id kept on ties
        }
      }
      int wl = wave_argmin(ls, (uint32_t)lj, lj >= 0);
      double best_s = INFINITY;
      int bj = -1;
      if (wl >= 0) { best_s = readlane_f64(ls, wl); bj = readlane_i32(lj, wl); }
      double lim = best_s < rem ? best_s : rem;
      double step;
      int kind;
      if (lim > cap) {
        step = cap; kind = EV_PSEUDO;
        h ^= digest_term(EV_PSEUDO, (uint64_t)d.n + 2, cap, n_ev++);
      } else if (!(best_s < rem)) {
        step = rem; kind = EV_END;
        h ^= digest_term(EV_END, (uint64_t)d.n + 3, rem, n_ev++);
      } else {
        step = best_s; kind = EV_LIFT;
        h ^= digest_term(EV_LIFT, (uint64_t)bj, best_s, n_ev++);
      }
      ax = fma(step, dx, ax);
      ay = fma(step, dy, ay);
      if (ax >= L) ax -= L; else if (ax < 0.0) ax += L;
      if (ay >= L) ay -= L; else if (ay < 0.0) ay += L;
      if (lane == 0) { px[a] = ax; py[a] = ay; }
      wave_sync();
      if (kind == EV_END) break;
      if (kind == EV_PSEUDO) { rem = rem - cap; n_pseudo += 1; continue; }
      rem = rem - best_s;
      double rx = px[bj] - ax, ry = py[bj] - ay;
      if (rx < -half_L) rx += L; else if (rx >= half_L) rx -= L;
      if (ry < -half_L) ry += L; else if (ry >= half_L) ry -= L;
      acc = acc + fma(rx, dx, ry * dy);
      n_lift += 1;
      a = bj;
      ax = px[a];
      ay = py[a];
    }
  }
  wave_sync();
  for (int i = lane; i < n; i += 64) { d.x[i] = px[i]; d.y[i] = py[i]; }
  if (lane == 0) {
    d.acc_delta[0] = acc;
    d.acc_cnt[CNT_LIFTS] += n_lift;
    d.acc_cnt[CNT_CHAINS] += (uint64_t)n_m;
    d.acc_cnt[CNT_PSEUDO] += n_pseudo;
    d.digest_ring[sweep % kDigestRing] = h;
    d.cell_digest[0] = h;
    *d.sweep_ctr = sweep;
  }
}

// ---------------------------------------------------------------------------
// Tallies
// ---------------------------------------------------------------------------
// Totals over the cells, one workgroup: the contact sum in index order (a sum
// of doubles is defined by its order), the counters in any.  The tiles of the
// contact sums come through LDS while the one before is added up by a single
// wavefront, whose lanes all make the same additions of values broadcast from
// LDS.  Bound by that chain of additions: 4,096 cells in 41 us, 256 in 7 us
// (640 and 40 us with the loads in the chain).
__global__ void __launch_bounds__(1024) k_reduce(const Dev* __restrict__ ds) {
  const Dev& d = ds[blockIdx.y];
  constexpr int kTile = 2048;
  __shared__ double tile[2][kTile];
  __shared__ unsigned long long total[CNT_NCOL];
  const int t = (int)threadIdx.x, ncell = d.C * d.C;
  if (t < CNT_NCOL) total[t] = 0;
  unsigned long long c[CNT_NCOL] = {0, 0, 0, 0, 0};
  for (int i = t; i < ncell; i += 1024)
    for (int k = 0; k < CNT_NCOL; ++k) c[k] += d.acc_cnt[(size_t)i * CNT_NCOL + k];
  // (past the end: zeros, which change no sum that starts from 0)
  auto load = [&](int i) { return i < ncell ? d.acc_delta[i] : 0.0; };
  double a0 = load(t), a1 = load(t + 1024), s = 0.0;
  for (int base = 0, b = 0; base < ncell; base += kTile, b ^= 1) {
    tile[b][t] = a0;
    tile[b][t + 1024] = a1;
    __syncthreads();  // (a wave is at most one tile ahead of the one that adds: two buffers)
    if (base + kTile < ncell) {
      a0 = load(base + kTile + t);
      a1 = load(base + kTile + t + 1024);
    }
    if (t < 64) {
      const int n = min(ncell - base, kTile);
#pragma unroll 8
      for (int j = 0; j < n; ++j) s = s + tile[b][j];
    }
  }
  for (int k = 0; k < CNT_NCOL; ++k) {
    for (int off = 32; off > 0; off >>= 1) c[k] += __shfl_xor(c[k], off, 64);
    if ((t & 63) == 0) atomicAdd(&total[k], c[k]);
  }
  __syncthreads();
  if (t == 0) {
    d.status->red[0] = s;
    for (int k = 0; k < CNT_NCOL; ++k) d.status->red[1 + k] = __longlong_as_double((long long)total[k]);
  }
}

__global__ void k_zero_tallies(const Dev* __restrict__ ds) {
  const Dev& d = ds[blockIdx.y];
  int ncell = d.C * d.C;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < ncell; i += gridDim.x * blockDim.x) {
    d.acc_delta[i] = 0.0;
    for (int k = 0; k < CNT_NCOL; ++k) d.acc_cnt[(size_t)i * CNT_NCOL + k] = 0;
  }
}

// ---------------------------------------------------------------------------
// One periodic cell (C = 1) with a bin grid: the same events as k_periodic,
// found in an 8 x 8-bin window around the moving disk as in the walled cells.
// Bins of side b = L / pbins < 0.7 sigma hold one disk each (a slot: FP64
// position, NaN when empty, and the disk's id); the window wraps around the
// box, and each lane forms its disk's offset with the minimum image exactly
// as k_periodic does, so the contact distances are the same numbers.  The
// window reaches 2 bins behind the moving disk and 5 ahead along each axis,
// so a move of length t with t max(|dx|, |dy|) <= 5b - sigma - eps keeps its
// sigma-neighbourhood inside it; the host takes this kernel only where that
// reach is below the free-flight cap L/2 - sigma, so a window event is never
// a pseudo event.  Every other event (a longer flight, the chain end, the
// cap) is decided as in k_periodic, over every slot when the window cannot
// vouch.  Plain lifts (the nearest disk in the window hit within the
// remaining length, the cap and the window's reach) run in an inner loop, as
// in the walled cells.  Event records are kept in the lanes and hashed 64 at
// a time; the lifts are counted from them.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(64) k_periodic_bins(const Dev* __restrict__ ds) {
  const Dev& d = ds[blockIdx.y];
  const int64_t sweep = *d.sweep_ctr + 1;  // (no k_prep before it)
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int lane = threadIdx.x;
  const int n = (int)d.n;
  const int nb = d.pbins;
  const PeriodicLds lay = periodic_lds_layout(nb, n);
  double2* const pos = (double2*)(lds_raw + lay.off_pos);
  uint32_t* const meta = (uint32_t*)(lds_raw + lay.off_meta);
  uint16_t* const slot_of = (uint16_t*)(lds_raw + lay.off_slot_of);
  int32_t* const tmp = (int32_t*)(lds_raw + lay.off_tmp);
  double2* const sink = (double2*)(lds_raw + lay.off_sink) + lane;
  uint32_t* const sink32 = (uint32_t*)sink;
  const int nslots = nb * nb;
  const double L = d.L, half_L = d.half_L, sig2 = d.sig2, cap = d.cap, sigma = d.sigma;
  const double b = L / (double)nb, inv_b = 1.0 / b;
  const double2 nan2 = make_double2(__builtin_nan(""), __builtin_nan(""));
  // row of a slot: floor(slot / nb) as (slot * m) >> 32 with m = ceil(2^32 /
  // nb), exact for slot < nb^2 <= 100^2
  const uint32_t inv_n32 = 0xFFFFFFFFu / (uint32_t)nb + 1u;
  // the minimum image of an offset, as k_periodic forms it (v + L below
  // -L/2, v - L from L/2 on), written as selects so that no lane branches
  auto min_image = [&](double v) __attribute__((always_inline)) {
    const double vp = v + L, vm = v - L;
    return v < -half_L ? vp : (v >= half_L ? vm : v);
  };
  auto bin_of = [&](double v) __attribute__((always_inline)) {
    int k = (int)(v * inv_b);
    return k > nb - 1 ? nb - 1 : (k < 0 ? 0 : k);
  };

  for (int sl = lane; sl < nslots; sl += 64) {
    pos[sl] = nan2;
    meta[sl] = kEmptySlot;
  }
  wave_sync();
  for (int i = lane; i < n; i += 64) {
    const double x = d.x[i], y = d.y[i];
    const int sl = bin_of(y) * nb + bin_of(x);
    if (atomicCAS(&meta[sl], kEmptySlot, (uint32_t)i) != kEmptySlot) {
      atomicOr(d.err, ERR_BIN_CAP);
      continue;
    }
    pos[sl] = make_double2(x, y);
    slot_of[i] = (uint16_t)sl;
  }
  const int64_t n_m = d.chains_per_cell > 0 ? d.chains_per_cell : n;
  if (d.start_mode == 1) {
    wave_sync();
    if (lane == 0) {
      for (int i = 0; i < n; ++i) tmp[i] = i;
      Stream st(d.seed, kKindShuffle, (uint64_t)sweep, cell_key(d, 0), 0);
      for (int i = 0; i + 1 < n; ++i) {
        int j = i + (int)draw_index(st, (uint64_t)(n - i));
        int t = tmp[i]; tmp[i] = tmp[j]; tmp[j] = t;
      }
    }
  }
  wave_sync();
  if (load_err(d) != 0) {  // two disks in one bin: an overlap
    if (lane == 0) *d.sweep_ctr = sweep;
    return;
  }

  double acc = d.acc_delta[0];
  uint64_t n_lift = 0, n_pseudo = 0, h = 0;
  int n_ring = 0;           // event records held in the lanes (lane k: record k)
  uint64_t ring_first = 0;  // event index of record 0
  uint32_t rec_lo = 0, rec_hi = 0, rec_tag = 0;
  const int lx = lane & 7, ly = lane >> 3;
  const double eps = 1e-9 * sigma;
  const double reach = 5.0 * b - sigma - eps;
  const uint32_t pseudo_id = (uint32_t)d.n + 2, end_id = (uint32_t)d.n + 3;
  // the loop's scalar operands, and its LDS addresses
  const double s_L = readlane_f64(L, 0), s_inv_L = readlane_f64(1.0 / L, 0), s_mid = readlane_f64(half_L, 0),
               s_inner = readlane_f64(half_L * (1.0 - 1e-12), 0), s_sig2 = readlane_f64(sig2, 0),
               s_inv_b = readlane_f64(inv_b, 0);
  const int s_nb = uniform_i32(nb), s_inv_n32 = uniform_i32((int)inv_n32);
  const uint32_t pos_at = lds_address(pos), meta_at = lds_address(meta), slot_of_at = lds_address(slot_of);
  // the records are hashed 64 at a time; lifts are counted from the records
  auto flush = [&](int count) __attribute__((always_inline)) {
    uint32_t lifts;
    h ^= digest_records(rec_lo, rec_hi, rec_tag, lane, count, ring_first, nullptr, lifts);
    n_lift += lifts;
    ring_first += (uint64_t)count;
    n_ring = 0;
  };
  // a coordinate moved across the box edge comes back from the other side
  // (both candidates formed first, so that no lane branches)
  auto wrap_box = [&](double v) __attribute__((always_inline)) {
    const double vm = v - L, vp = v + L;
    return v >= L ? vm : (v < 0.0 ? vp : v);
  };

  for (int64_t k = 0; k < n_m; ++k) {
    int a;
    if (d.start_mode == 1) {
      a = tmp[k % n];
    } else {
      Stream st(d.seed, kKindStart, (uint64_t)sweep, cell_key(d, 0), (uint64_t)k);
      a = (int)draw_index(st, (uint64_t)n);
    }
    // every lane draws the same values; read them as one (scalar) value so
    // that every decision below is a uniform branch
    a = uniform_i32(a);
    double dx, dy;
    chain_direction(d, sweep, 0, k, dx, dy);
    dx = readlane_f64(dx, 0);
    dy = readlane_f64(dy, 0);
    // reach / max(|dx|, |dy|) from the reciprocals (a 0 component has a factor 1)
    const double rx_ = dx != 0.0 ? 1.0 / dx : 1.0, ry_ = dy != 0.0 ? 1.0 / dy : 1.0;
    const double dsafe = reach * fmin(fabs(rx_), fabs(ry_));
    const double guard = fmin(dsafe, cap * (1.0 - 1e-9));  // below the flight cap: a plain lift is no pseudo event
    const int offx = uniform_i32(dx < 0.0 ? -5 : -2), offy = uniform_i32(dy < 0.0 ? -5 : -2);  // window origin
    // this lane's slot in the 8 x 8-bin window around the bin of `slot`,
    // wrapped around the box
    auto window_slot = [&](int slot) __attribute__((always_inline)) {
      const int by = (int)__umulhi((uint32_t)slot, inv_n32);
      const int bx = slot - by * nb;
      int wx = bx + offx + lx, wy = by + offy + ly;
      wx += wx < 0 ? nb : 0;
      wx -= wx >= nb ? nb : 0;
      wy += wy < 0 ? nb : 0;
      wy -= wy >= nb ? nb : 0;
      return wy * nb + wx;
    };
    double nrem = -d.ell;  // minus the chain length left
    int a_slot = uniform_i32((int)slot_of[a]);
    double ax = pos[a_slot].x, ay = pos[a_slot].y;
    // the event cap is held at the digest flushes: ring_first - ev0 is the
    // chain's event count there, so a chain makes at most
    // kMaxEventsPerChain + 63 events before it stops with the error
    const uint64_t ev0 = ring_first + (uint64_t)n_ring;
    int capped = 0;
    int wsl = window_slot(a_slot);
    double2 p = pos[wsl];
    uint32_t m = meta[wsl];
    for (;;) {
      // Plain lifts, up to the next 64 records: the nearest disk in the window
      // is hit within the remaining length and within the reach the window
      // vouches for (below the flight cap), and the moved centre stays off the
      // box edge.  That is exactly the full decision below finding a lift;
      // every other event (no disk in the window, the chain end, a pseudo
      // event, a flight the window cannot vouch for, a move across the edge) is
      // left to it, with nothing changed.
      for (;;) {
        double dacc = 0.0, s;
        uint32_t key, key_min;
        int full, a_t, a_u, a_next, a_slo, a_shi, a_expect;
        uint64_t a_mask;
        nrem = readlane_f64(nrem, 0);
        a = uniform_i32(a);
        a_slot = uniform_i32(a_slot);
        n_ring = uniform_i32(n_ring);
        EC_LOOP_PERIODIC;
        (void)s; (void)key; (void)key_min;
        if (full == 0) break;
        flush(kDigestBatch);
        capped = (ring_first - ev0 >= (uint64_t)kMaxEventsPerChain) ? 1 : 0;
        if (capped != 0) break;
      }
      if (capped != 0) {
        if (lane == 0) atomicOr(d.err, ERR_EVENT_CAP);
        break;
      }
      // the full decision, on the window already read
      const double rem = -nrem;
      const double rx = min_image(p.x - ax), ry = min_image(p.y - ay);
      double s = 0.0;
      const bool valid = contact(rx, ry, dx, dy, sig2, s);  // the mover's own slot: no contact
      const unsigned key = argmin_key(s, valid);
      const unsigned key_min = wave_min_u32(key);
      double best_s = INFINITY, wpx = 0.0, wpy = 0.0;
      int bj = -1, bslot = -1;
      if (key_min != 0xFFFFFFFFu) {
        const int wl = argmin_lane(s, m, key, key_min);
        best_s = readlane_f64(s, wl);
        bj = readlane_i32((int)m, wl);
        bslot = readlane_i32(wsl, wl);
        wpx = readlane_f64(p.x, wl);
        wpy = readlane_f64(p.y, wl);
      }
      if (uniform_i32(best_s <= dsafe ? 0 : 1) != 0) {
        // the window cannot vouch: the nearest contact over every slot
        double ls = INFINITY;
        uint32_t lid = 0xFFFFFFFFu;
        int lsl = -1;
        for (int sl = lane; sl < nslots; sl += 64) {
          const double2 q = pos[sl];
          const double qx = min_image(q.x - ax), qy = min_image(q.y - ay);
          double s2;
          if (contact(qx, qy, dx, dy, sig2, s2)) {
            const uint32_t i2 = meta[sl];
            if (s2 < ls || (s2 == ls && i2 < lid)) { ls = s2; lid = i2; lsl = sl; }
          }
        }
        const int fl = wave_argmin_all(ls, lid, lsl >= 0);
        best_s = INFINITY;
        bj = -1;
        if (fl >= 0) {
          best_s = readlane_f64(ls, fl);
          bj = readlane_i32((int)lid, fl);
          bslot = readlane_i32(lsl, fl);
          const double2 q = pos[bslot];
          wpx = readlane_f64(q.x, 0);
          wpy = readlane_f64(q.y, 0);
        }
      }
      // the event, in the order k_periodic decides it (one scalar value)
      const double lim = best_s < rem ? best_s : rem;
      const int kind = uniform_i32(lim > cap ? EV_PSEUDO : (!(best_s < rem) ? EV_END : EV_LIFT));
      const double step = kind == EV_PSEUDO ? cap : (kind == EV_END ? rem : best_s);
      {
        const uint32_t id = kind == EV_PSEUDO ? pseudo_id : (kind == EV_END ? end_id : (uint32_t)bj);
        const uint64_t sb = (uint64_t)__double_as_longlong(step);
        writelane3(rec_lo, rec_hi, rec_tag, (uint32_t)sb, (uint32_t)(sb >> 32),
                   ((uint32_t)(kind ^ 1) << 29) | id, n_ring);
      }
      const double nax = wrap_box(fma(step, dx, ax)), nay = wrap_box(fma(step, dy, ay));
      // store the moved disk (lane 0) and move it to another bin if it crossed
      // one (lane 0 empties the old slot, lane 1 fills the new one, which is
      // empty: a bin holds one centre)
      const int ns = uniform_i32(bin_of(nay) * nb + bin_of(nax));
      {
        double2* const dst = (lane == 0) ? pos + a_slot : sink;
        *dst = make_double2(nax, nay);
      }
      if (ns != a_slot) {
        double2* const dst = (lane == 0) ? pos + a_slot : ((lane == 1) ? pos + ns : sink);
        *dst = (lane == 0) ? nan2 : make_double2(nax, nay);
        uint32_t* const dm = (lane == 0) ? meta + a_slot : ((lane == 1) ? meta + ns : sink32);
        *dm = (lane == 0) ? kEmptySlot : (uint32_t)a;
        if (lane == 0) slot_of[a] = (uint16_t)ns;
        a_slot = ns;
      }
      wave_sync();
      if (++n_ring == kDigestBatch) {
        flush(kDigestBatch);
        capped = (ring_first - ev0 >= (uint64_t)kMaxEventsPerChain) ? 1 : 0;
      }
      if (kind == EV_END) break;
      if (kind == EV_PSEUDO) {
        nrem = nrem + cap;
        n_pseudo += 1;
        ax = nax;
        ay = nay;
      } else {
        nrem = nrem + best_s;
        const double tx = min_image(wpx - nax), ty = min_image(wpy - nay);
        acc = acc + fma(tx, dx, ty * dy);
        a = bj;
        a_slot = bslot;
        ax = wpx;
        ay = wpy;
      }
      if (capped != 0) {
        if (lane == 0) atomicOr(d.err, ERR_EVENT_CAP);
        break;
      }
      wsl = window_slot(a_slot);
      p = pos[wsl];
      m = meta[wsl];
    }
  }
  wave_sync();
  flush(n_ring);
  for (int i = lane; i < n; i += 64) {
    const double2 v = pos[(int)slot_of[i]];
    d.x[i] = v.x;
    d.y[i] = v.y;
  }
  if (lane == 0) {
    d.acc_delta[0] = acc;
    d.acc_cnt[CNT_LIFTS] += n_lift;
    d.acc_cnt[CNT_CHAINS] += (uint64_t)n_m;
    d.acc_cnt[CNT_PSEUDO] += n_pseudo;
    d.digest_ring[sweep % kDigestRing] = h;
    d.cell_digest[0] = h;
    *d.sweep_ctr = sweep;
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// Grid x-extents are the maxima over the systems of a launch (gridDim.y =
// systems); blocks beyond a system's own extent leave at once.
// ---------------------------------------------------------------------------
hipError_t launch_lattice(const Dev* ds, int64_t n, int64_t k, double a, hipStream_t st) {
  int64_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(k_lattice, dim3((unsigned)blocks), dim3(256), 0, st, ds, k, a);
  return hipGetLastError();
}

hipError_t launch_zero_tallies(const Dev* ds, int32_t n_cells, hipStream_t st) {
  int blocks = (n_cells + 255) / 256;
  hipLaunchKernelGGL(k_zero_tallies, dim3(blocks), dim3(256), 0, st, ds);
  return hipGetLastError();
}

hipError_t set_phase_lds_limit(int bytes) {
  const void* fns[8] = {(const void*)k_phase<0>,       (const void*)k_phase<1>,
                        (const void*)k_sweep_cells<0>, (const void*)k_sweep_cells<1>,
                        (const void*)k_queue_cells<0>, (const void*)k_queue_cells<1>,
                        (const void*)k_stripe_phase<0>, (const void*)k_periodic_bins};
  for (const void* f : fns) {
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t ready_queue_workers(int lds_per_cell, int cpb, int reject, int* workers) {
  const void* f = reject ? (const void*)k_queue_cells<1> : (const void*)k_queue_cells<0>;
  int per_cu = 0, dev = 0, cus = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, 64 * cpb,
                                                              (size_t)cpb * lds_per_cell);
  if (e == hipSuccess) e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  *workers = (per_cu > 0 ? per_cu : 1) * (cus > 0 ? cus : 1) * cpb;
  return hipSuccess;
}

hipError_t launch_reduce(const Dev* ds, hipStream_t st) {
  hipLaunchKernelGGL(k_reduce, dim3(1), dim3(1024), 0, st, ds);
  return hipGetLastError();
}

hipError_t launch_sweep(const Dev* ds, const LaunchShape& sh, hipStream_t st,
                        const PhaseEvents* ev) {
  const unsigned ns = (unsigned)sh.n_sys;
  if (sh.periodic) {
    if (ev) (void)hipEventRecord(ev->begin[0], st);
    if (sh.pbins > 0) {
      const size_t lds = (size_t)periodic_lds_layout(sh.pbins, (int)sh.max_n).bytes;
      hipLaunchKernelGGL(k_periodic_bins, dim3(1, ns), dim3(64), lds, st, ds);
    } else {
      const size_t lds = (size_t)sh.max_n * 16 + (size_t)sh.max_n * 4;
      hipLaunchKernelGGL(k_periodic, dim3(1, ns), dim3(64), lds, st, ds);
    }
    if (ev) (void)hipEventRecord(ev->end[0], st);
    hipError_t e = launch_check_overlap(ds, sh, st);
    if (e != hipSuccess) return e;
    return hipGetLastError();
  }
  const unsigned nblk = (unsigned)((sh.max_n + 255) / 256);
  hipLaunchKernelGGL(k_prep, dim3(1, ns), dim3(1024), 0, st, ds);
  if (ev) (void)hipEventRecord(ev->rebin[0], st);
  hipLaunchKernelGGL(k_count, dim3(nblk, ns), dim3(256), 0, st, ds);
  if (ev) (void)hipEventRecord(ev->rebin[1], st);
  hipLaunchKernelGGL(k_scan, dim3(1, ns), dim3(1024), 0, st, ds);
  if (ev) (void)hipEventRecord(ev->rebin[2], st);
  hipLaunchKernelGGL(k_scatter, dim3(nblk, ns), dim3(256), 0, st, ds);
  if (ev) (void)hipEventRecord(ev->rebin[3], st);
  hipLaunchKernelGGL(k_draws, dim3((unsigned)((sh.max_chains + 255) / 256), ns), dim3(256), 0, st,
                     ds);
  if (sh.any_distinct)
    hipLaunchKernelGGL(k_shuffle, dim3((unsigned)((sh.max_cells + 63) / 64), ns), dim3(64), 0, st,
                       ds);
  if (sh.stripes) {
    // two colour phases of C/2 stripes each, one wavefront per stripe
    const unsigned sgrid = (unsigned)((sh.max_cells_side + 1) / 2);
    for (int q = 0; q < 2; ++q) {
      if (ev) (void)hipEventRecord(ev->begin[q], st);
      hipLaunchKernelGGL(k_stripe_phase<0>, dim3(sgrid, ns), dim3(64), (size_t)sh.max_lds_per_cell, st,
                         ds, q);
      if (ev) (void)hipEventRecord(ev->end[q], st);
    }
    hipError_t e = launch_check_overlap(ds, sh, st);
    if (e != hipSuccess) return e;
    return hipGetLastError();
  }
  const int cpb = sh.cpb;
  const unsigned grid = (unsigned)((sh.max_active + cpb - 1) / cpb);
  const size_t lds = (size_t)cpb * sh.max_lds_per_cell;
  if (sh.ready_queue) {
    const ReadyQueue& rq = sh.queue;
    hipLaunchKernelGGL(k_queue_reset, dim3(1), dim3(64), 0, st, rq);
    hipLaunchKernelGGL(k_queue_prep, dim3((unsigned)((sh.max_cells + 255) / 256), ns), dim3(256), 0,
                       st, ds, rq);
    const unsigned qgrid = (unsigned)((rq.workers + cpb - 1) / cpb);
    if (ev) (void)hipEventRecord(ev->begin[0], st);
    if (sh.reject)
      hipLaunchKernelGGL((k_queue_cells<1>), dim3(qgrid), dim3(64 * cpb), lds, st, ds, rq,
                         sh.max_lds_per_cell);
    else
      hipLaunchKernelGGL((k_queue_cells<0>), dim3(qgrid), dim3(64 * cpb), lds, st, ds, rq,
                         sh.max_lds_per_cell);
    if (ev) (void)hipEventRecord(ev->end[0], st);
    hipLaunchKernelGGL(k_queue_check, dim3(1, ns), dim3(64), 0, st, ds, rq);
    hipError_t e = launch_check_overlap(ds, sh, st);
    if (e != hipSuccess) return e;
    return hipGetLastError();
  }
  if (sh.one_launch) {
    // as many wavefronts as one phase has cells; each takes cells of all phases
    if (ev) (void)hipEventRecord(ev->begin[0], st);
    if (sh.reject)
      hipLaunchKernelGGL((k_sweep_cells<1>), dim3(grid, ns), dim3(64 * cpb), lds, st, ds);
    else
      hipLaunchKernelGGL((k_sweep_cells<0>), dim3(grid, ns), dim3(64 * cpb), lds, st, ds);
    if (ev) (void)hipEventRecord(ev->end[0], st);
    hipError_t e = launch_check_overlap(ds, sh, st);
    if (e != hipSuccess) return e;
    return hipGetLastError();
  }
  for (int q = 0; q < 4; ++q) {
    if (ev) (void)hipEventRecord(ev->begin[q], st);
    if (sh.reject)
      hipLaunchKernelGGL((k_phase<1>), dim3(grid, ns), dim3(64 * cpb), lds, st, ds, q);
    else
      hipLaunchKernelGGL((k_phase<0>), dim3(grid, ns), dim3(64 * cpb), lds, st, ds, q);
    if (ev) (void)hipEventRecord(ev->end[q], st);
  }
  hipError_t e = launch_check_overlap(ds, sh, st);
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

}  // namespace ec
