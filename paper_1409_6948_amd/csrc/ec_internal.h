// Internal interface between the C ABI (ec_api.cpp) and the gfx950 kernels
// (ec_kernels.hip).  Not installed; not part of the ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ec {

// Per-sweep draws written by the prep kernel (shift of the cell grid and the
// order of the four colours, Sec. 3.4 steps 1 and 3).
struct SweepDraws {
  double sx, sy;
  int32_t perm;  // colour of phase q in bits 2q, 2q+1
  int32_t pad;
};

// Column order of the per-cell counters.
enum { CNT_LIFTS = 0, CNT_FROZEN = 1, CNT_WALLS = 2, CNT_CHAINS = 3, CNT_PSEUDO = 4, CNT_NCOL = 5 };

// Device error bits.  Any nonzero value also tells every running wave to stop.
enum {
  ERR_OWN_CAP = 1,     // a cell (own or neighbour) holds more disks than the packing bound
  ERR_BIN_CAP = 2,     // two centres in one LDS bin: disks overlap
  ERR_EVENT_CAP = 4,   // a chain exceeded kMaxEventsPerChain events
  ERR_DRAW_CAP = 8,    // a rejection draw exceeded kMaxDrawTries attempts
  ERR_DEP_WAIT = 16,   // a cell waited longer than dep_wait_ticks for a neighbour of an earlier phase
  ERR_UNDO_CAP = 32,   // rejection variant: a chain made more lifts than the undo log holds
  ERR_OVERLAP = 64,    // overlap check (debug flag): two disks closer than sigma after a sweep
  ERR_ABANDONED = 128  // ready-queue batch sweep: left unfinished after another system's error
};

// Ready queue of the batched sweep (one launch runs every cell of every
// system of a batch): header words, then per cell of the batch a task slot,
// its publication flag, and the count of earlier-phase neighbours not yet
// done.  Laid out by the batch in its workspace.
struct ReadyQueue {
  int32_t* hdr;        // [0] tasks claimed, [1] tasks reserved, [2] sweep epoch, [3] abort
  int64_t* tasks;      // [total] system << 32 | cell, in the order cells became ready
  int32_t* flags;      // [total] epoch of the sweep that published the slot
  int32_t* dep;        // [total] earlier-phase neighbours still running or waiting
  const int32_t* base; // [n_sys + 1] first queue index of each system's cells
  const int32_t* order; // [n_sys] systems by the work of one of their cells, most first
  int32_t total;       // cells of all systems
  int32_t workers;     // wavefronts of the persistent launch
};
enum { QH_READ = 0, QH_RESERVE = 1, QH_EPOCH = 2, QH_ABORT = 3 };

// Events allowed in one chain before the sweep gives up with ERR_EVENT_CAP.
// Only degenerate input (a closed ring of touching disks, a disk pinned
// between two antipodal frozen contacts) comes near it; every wave then
// leaves its loops and the host reports the error.
constexpr int64_t kMaxEventsPerChain = int64_t(1) << 20;
// Events between two polls of the device error word.
constexpr int64_t kAbortPollEvents = 1024;
static_assert(kMaxEventsPerChain % kAbortPollEvents == 0, "the event cap is tested at polls");
// Attempts of one rejection draw (acceptance 0.785 for directions, > 1 - 2^-50
// for indices); reaching the cap sets ERR_DRAW_CAP.
constexpr int kMaxDrawTries = 256;
// Doubles in the debug snapshot written by the first wave that trips a cap.
constexpr int kDebugWords = 16;

constexpr int kDigestRing = 1024;
// Workgroups of the pair histogram over n disks, r_max in units of sigma: 1024 (each
// adds all its bins to the global counts at the end), or as many as 256 disks each
// need, but so many that no 32-bit bin of a workgroup can overflow.  A pair adds 2,
// in the workgroup of one of its disks, and at most (2 pi / sqrt 3) u^2 + pi u other
// disks lie within u diameters of one (Oler's bound for a disc).
__host__ __device__ inline int64_t histogram_groups(int64_t n, double r_max) {
  const int64_t blocks = (n + 255) / 256;
  const double per_block = 256.0 * 2.0 * (3.6276 * r_max * r_max + 3.1416 * r_max);
  const int64_t most = per_block < 4294967295.0 ? (int64_t)(4294967295.0 / per_block) : 1;  // blocks of one workgroup
  const int64_t least = (blocks + most - 1) / most, wanted = blocks < 1024 ? blocks : 1024;
  return least > wanted ? least : wanted;
}
// Counters of the observables' grid: places of the sorted arrays taken, disks
// on the Delaunay list.
enum { OBS_CURSOR = 0, OBS_LISTED = 1, kObsCounters = 2 };
// Bins of the pair histogram (pressure route).
constexpr int kMaxGrBins = 1024;
// Events hashed together, one per lane, by the walled-cell kernel's digest
// (event ids then fit in 29 bits: N < 2^29 - 3).
constexpr int kDigestBatch = 64;
// regions of a cell: 3 x 3, r = 3 * ry + rx with rx, ry in {0: first strip,
// 1: middle, 2: last strip}
constexpr int kRegions = 9;
// Rejection variant: lifts of one chain that can be undone (LDS log entries).
constexpr int kUndoCap = 256;

// What the host reads back after a call, in one copy.
struct Status {
  int32_t err[2];                // device error word; number of chains that tripped a cap
  double dbg[kDebugWords];       // state of the first wave that tripped a cap
  unsigned long long ovl[4];     // overlap check: pairs found, first pair (i, j), its sweep
  double red[8];                 // reduced tallies (contact sum, then the counters as bits)
  double psi_red[3];             // Psi (re, im) and the mean neighbour count
  unsigned long long psi_err[2]; // disks whose Voronoi cell was not certified; candidate overflows
};

// Everything a kernel needs: device pointers into the caller's workspace and
// the derived constants.  Kernels read it from device memory.
struct Dev {
  double* x;                        // [N] positions, disk-id order
  double* y;
  int32_t* reg_count;               // [9*C*C] disks per (cell, region)
  int32_t* cell_start;              // [C*C+1] exclusive prefix sum over cells
  int32_t* reg_start;               // [9*C*C+1] exclusive prefix sum over (cell, region)
  int32_t* cell_of;                 // [N]
  uint8_t* reg_of;                  // [N] region of the disk in its cell (see k_count)
  int32_t* cell_ids;                // [N] ids grouped by cell, by region inside a cell
  double* acc_delta;                // [C*C]
  unsigned long long* acc_cnt;      // [C*C*CNT_NCOL]
  unsigned long long* digest_ring;  // [kDigestRing]
  unsigned long long* cell_digest;  // [C*C] digest of each cell in the last sweep it ran
  SweepDraws* draws;                // [1]
  int32_t* err;                     // (status->err)
  Status* status;                   // [1] what the host reads after a call
  int32_t* chain_start;             // [max chains per sweep] start index within its cell
  double2* chain_dir;               // [max chains per sweep] direction of each chain
  int32_t* shuffle;                 // [N] rebin: places in the (cell, region) lists; then per-cell
                                    // shuffled lists (distinct-start mode)
  double* dbg;                      // (status->dbg)
  int64_t* sweep_ctr;               // [1] number of the current or last sweep, -1 before the first
  double2* psi;                     // [N] per-disk hexatic order Psi_k (re, im)
  double* psi_part;                 // [3 * ceil(N/256)] per-block sums (re, im, neighbours)
  int32_t* psi_nb;                  // [N] neighbour count of each disk
  double2* obs_pos;                 // [N] observables: positions grouped by the cells of their grid
  int32_t* obs_id;                  // [N] ids in that order
  int32_t* obs_list;                // [N] sorted places whose Delaunay neighbours need the wide search
  int32_t* obs_count;               // [N] disks per grid cell (never more cells than disks)
  int2* obs_range;                  // [N] sorted range of each grid cell
  int32_t* obs_ctr;                 // [kObsCounters]
  unsigned long long* gr_counts;    // [kMaxGrBins + 1] pair counts per bin, then pairs < sigma
  int32_t* queue;                   // [1] ticket counter of the one-launch sweep
  int64_t* cell_done;               // [C*C] last sweep + 1 whose write-back the cell has published
  unsigned long long* ovl;          // (status->ovl)

  int64_t n;
  double sigma, sig2, ell, L, half_L, w, cap, b, inv_b;
  // width of the wall strips that split a cell into 3 x 3 regions: sigma plus
  // a margin far above the rounding of cell-local coordinates, so every disk a
  // neighbour stages as frozen lies in the strips that face it
  double strip;
  int32_t C, nb, gridb, cap_own, chains_per_cell, dir_mode, start_mode;
  int32_t pbins;  // one periodic cell: bins per side of its bin grid, 0 = brute-force search
  int32_t lds_per_cell, cells_per_block;
  int32_t search;                   // 0: 8x8-bin window with guard; 1: scan of every slot
  int64_t dep_wait_ticks;           // one-launch sweep: limit of one wait, 100 MHz clock ticks
  int32_t reject;                   // 1: a chain reaching a wall or a frozen disk is undone
  int32_t check_overlap;            // 1: every sweep ends with a check of all neighbour pairs
  int32_t stripes;                  // 1: striped decomposition, C stripes of width w, rejection
  int32_t stripe_cap_own, stripe_cap_frozen, stripe_undo;  // LDS capacities of one stripe
  int32_t wave_priority;            // ready queue: issue priority of a wave with one of its cells, 0..3
  uint64_t seed;
  uint32_t system;
};

// LDS layout of one simulation cell in the walled-cell kernel: a grid of
// gridb x gridb square bins of side b < sigma/sqrt(2), one slot each (FP64
// position, 32-bit meta word: own index, or frozen id | top bit), with
// kSlotPad empty slots before the first and after the last (a window's columns
// are not clamped to the grid); the cell's id-ordered list and the 16-bit slot
// of each own disk (at most 100^2 slots).
constexpr int kSlotPad = 3;
struct CellLds {
  int32_t off_pos, off_meta, off_own_gid, off_own_loc, off_undo, bytes;
};

// reject: an undo log of kUndoCap entries (slots and old position, 32 B each).
__host__ __device__ inline CellLds cell_lds_layout(int gridb, int cap_own, bool reject) {
  CellLds l;
  int slots = gridb * gridb + 2 * kSlotPad;
  int o = 0;
  l.off_pos = o;      o += 16 * slots;
  l.off_meta = o;     o += 4 * slots;
  o = (o + 15) & ~15;
  l.off_own_gid = o;  o += 4 * cap_own;
  l.off_own_loc = o;  o += 2 * cap_own;
  o = (o + 15) & ~15;
  l.off_undo = o;     o += reject ? 32 * kUndoCap : 0;
  l.bytes = (o + 15) & ~15;
  return l;
}

// A walled cell's disk k still has its slot: the slot that own_loc names for it
// names it (its meta word) and holds a centre (x is a coordinate; NaN where
// empty).  Stores of a moved centre go unchecked to the bin it lies in; where
// that held another disk (possible only if disks overlap), no later move leaves
// every disk of the cell with its slot, since the disks are then more than the
// slots that hold a centre.  An undo can, but one of its moves then starts from
// a slot that is empty.
__host__ __device__ inline bool slot_kept(uint32_t meta_word, uint32_t k, double x) {
  return meta_word == k && x == x;
}

// LDS of the binned periodic cell: pbins x pbins slots (FP64 position, 32-bit
// disk id), the slot of every disk (16 bits each; the field has 4 n bytes), the
// shuffled start list, one sink slot per lane.
struct PeriodicLds {
  int32_t off_pos, off_meta, off_slot_of, off_tmp, off_sink, bytes;
};
__host__ __device__ inline PeriodicLds periodic_lds_layout(int pbins, int n) {
  PeriodicLds l;
  const int slots = pbins * pbins;
  int o = 0;
  l.off_pos = o;      o += 16 * slots;
  l.off_meta = o;     o += 4 * slots;
  l.off_slot_of = o;  o += 4 * n;
  l.off_tmp = o;      o += 4 * n;
  o = (o + 15) & ~15;
  l.off_sink = o;     o += 16 * 64;
  l.bytes = o;
  return l;
}

// LDS of one stripe in the striped-decomposition kernel: own disks (position
// along and across the stripe, id, and a staging word), frozen disks
// (along, across, id), and the undo log (disk, old position along).
__host__ __device__ inline int stripe_lds_bytes(int cap_own, int cap_frozen, int undo) {
  return 24 * cap_own + 20 * cap_frozen + 16 * undo + 64;
}

// Largest N the one-periodic-cell kernel keeps in LDS.
constexpr int64_t kPeriodicMaxN = 2048;

// Extents of one launch over n_sys systems whose Dev records are in device
// memory (ds[0..n_sys)): maxima over the systems, and the shared schedule.
struct LaunchShape {
  int32_t n_sys;
  bool periodic;            // one periodic cell (single system only)
  bool any_distinct;        // some system uses the distinct-start control
  bool one_launch;          // all four phases in one launch (k_sweep_cells), else one per phase
  bool ready_queue;         // a batch: every cell of every system in one launch fed by a ready queue
  ReadyQueue queue;         // (ready_queue only)
  bool reject;              // rejection at the cell boundary (same for all)
  bool check_overlap;       // some system checks for overlaps after every sweep
  bool stripes;             // striped decomposition (same for all)
  double box, sigma;        // box side and disk diameter (observables: a system alone)
  int64_t max_n;            // disks
  int64_t max_chains;       // chains per sweep
  int32_t max_cells;        // C * C
  int32_t max_cells_side;   // C (stripes: the number of stripes)
  int32_t pbins;            // one periodic cell: bins per side (0: brute-force kernel)
  int32_t max_active;       // C * C / 4
  int32_t cpb;              // simulation cells per workgroup (same for all)
  int32_t max_lds_per_cell; // bytes
};

// Optional HIP events recorded around every phase launch (begin[q], end[q]);
// the one-launch sweep and the periodic cell use begin[0], end[0] only.
// rebin[0..1] bracket the count kernel, rebin[2..3] the scatter kernel
// (walled cells).
struct PhaseEvents {
  hipEvent_t begin[4], end[4];
  hipEvent_t rebin[4];
};

hipError_t launch_lattice(const Dev* ds, int64_t n, int64_t k, double a, hipStream_t st);
// One sweep of every system in ds: the sweep counters advance, rebin, draws,
// four colour phases (or the periodic kernel).  Kernels only (no memset or
// copy), so the sequence can be captured in a HIP graph and replayed.
hipError_t launch_sweep(const Dev* ds, const LaunchShape& sh, hipStream_t st,
                        const PhaseEvents* ev = nullptr);
hipError_t launch_reduce(const Dev* ds, hipStream_t st);
// Allow the phase kernel up to `bytes` of dynamic LDS per workgroup.
hipError_t set_phase_lds_limit(int bytes);
// Wavefronts per workgroup of the ready queue, from the wavefronts that fit on the
// device with one each and with four (0: four do not fit).  Four land on the four
// SIMDs of a CU, while workgroups of one are spread unevenly and stay so for the
// whole sweep: 16 systems of 64 disks per cell (12 KB of LDS, 12 wavefronts per CU
// either way) 34.0 against 35.8 ms per sweep, 64 systems of 160 (33 KB, 4 either
// way) 57.3 against 60.3.  But four are never worth a wavefront that fits no more:
// 64 systems of 96 disks per cell (21 KB, 4 per CU against 7) 57.9 against 42.2, of
// 128 (27 KB, 4 against 6) 57.1 against 46.3; rejected short chains of 96 (29 KB, 4
// against 5) 5.6 against 4.8.
inline int queue_cells_per_block(int one, int four) { return four >= one ? 4 : 1; }
// Wavefronts of the ready-queue launch that fit on the device at once with
// this much LDS per cell and cells per workgroup (resident workgroups per CU
// times CUs times cells per workgroup).
hipError_t ready_queue_workers(int lds_per_cell, int cpb, int reject, int* workers);
hipError_t launch_zero_tallies(const Dev* ds, int32_t n_cells, hipStream_t st);
// Hexatic order parameter of one system (cutoff neighbours within r_cut):
// the observables' grid, per-disk Psi_k, and a fixed-order reduction into
// psi_red.
hipError_t launch_psi6(const Dev* ds, const LaunchShape& sh, double r_cut, hipStream_t st);
// Psi with Delaunay neighbours: candidates within r_search, Voronoi cells
// certified within r_search / 2.
hipError_t launch_psi6_delaunay(const Dev* ds, const LaunchShape& sh, double r_search, hipStream_t st);
// Add the current configuration's ordered-pair counts (bins of width delta =
// (r_max - sigma)/n_bins from sigma) to gr_counts.
hipError_t launch_gr(const Dev* ds, const LaunchShape& sh, double r_max, double delta, int n_bins,
                     hipStream_t st);
// Allocation-free sweeps (ec_sweep_static): bytes of the library's static
// device buffer (one per GPU) and the largest system it holds.
constexpr size_t kStaticScratchBytes = size_t(10) << 20;
constexpr int64_t kStaticMaxDisks = int64_t(1) << 18;
// Address of this GPU's static buffer (looked up once per device).
hipError_t static_scratch(void** ptr);
// Clear [base, base + bytes) with a kernel, then store rec at dst and the
// sweep counter before the first sweep in rec.sweep_ctr.
hipError_t launch_static_setup(const Dev& rec, Dev* dst, unsigned char* base, size_t bytes,
                               int64_t first_sweep, hipStream_t st);
// Digests of sweeps first .. first + n - 1 and the device error word into
// caller device buffers (either may be null).
hipError_t launch_static_copy_out(const Dev* ds, int64_t first, int64_t n,
                                  unsigned long long* digests, int32_t* err, hipStream_t st);

// Debug check after a sweep: every pair of disks in neighbouring cells of the
// sweep's grid (all pairs for one periodic cell) closer than sigma (1 - 1e-12)
// is counted in ovl and sets ERR_OVERLAP.  Systems without check_overlap skip it.
hipError_t launch_check_overlap(const Dev* ds, const LaunchShape& sh, hipStream_t st);

}  // namespace ec
