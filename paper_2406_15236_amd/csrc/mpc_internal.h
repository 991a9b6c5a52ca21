// mpc_internal.h -- layouts shared by the host planner and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mpc {

constexpr int kThreads = 256;               // threads per workgroup (4 wave64)
constexpr int kCollideThreads = 64;         // collide workgroup: one wave64
constexpr int kTileCap = 256;               // particles held in LDS per tile pass
constexpr int kTileMaxCells = 32;           // cells per collide tile (< kCollideThreads)
constexpr int kObsPass = 256;               // particles per pass of the observables' order
constexpr int kObsSums = 128;               // sums left of the observables' partial sums
constexpr int kObsList = 320;               // particles of an obs tile listed in LDS
constexpr uint32_t kObsRows = 2048;         // most blocks of the order-free sums
constexpr uint32_t kObsFew = 32;            // rows that the host adds itself
constexpr int kObsBad = 60;                 // their anchor after a term that is not finite
constexpr int kScanItems = 16;              // cells per thread in the scan kernels
constexpr int kScanBlock = kThreads * kScanItems;
constexpr int kPartBlock = kThreads * 4;    // particles per block of per-particle kernels
constexpr int kMaxRuns = 32;                // most runs in a tile's table (more go to chains)
constexpr int kGroups = 27;                 // next-step tiles of a pass: 3 per row, 9 rows
constexpr int kTileBlock = kThreads * 4;    // tiles per block of the tile prefix
constexpr uint32_t kTileOne = 16384;        // most tiles with a prefix in one launch
constexpr uint32_t kTileDirect = 2048;      // most tiles with a prefix inside the collide
constexpr uint32_t kMinDrawBlock = 64, kMaxDrawBlock = 1024;  // cells per block of the draws
constexpr int kDrawList = 256;              // cells listed for repeated draws at a time
constexpr uint32_t kNeverAccepted = 1024;   // more particles than a cell can hold
constexpr uint32_t kNoSlot = 0xffffffffu;

// Random-stream tags (counter word 3); counter = {draw, id, step, tag}.
enum : uint32_t { kTagShift = 1, kTagAxis = 2, kTagThermo = 3, kTagPhantom = 4,
                  kTagInitPos = 5, kTagInitVel = 6 };

// Sticky error bits in Ctrl::err.
enum : uint32_t { kErrKey = 1u, kErrCellOverflow = 2u, kErrFixRange = 4u,
                 kErrDraws = 8u };

enum : int { kFormF64 = 0, kFormF32 = 1, kFormSplit = 2 };

// Split form packs the unshifted cell as x | y << 11 | z << 22.
constexpr uint32_t kSplitXBits = 11, kSplitYBits = 11, kSplitZBits = 10;

struct BoxDev {
  int32_t L[3];        // cells per axis (walls: L[2] = H)
  int32_t nlz;         // z layers in key space: L[2], or H + 2 with walls
  uint32_t pbase, np;  // particle range in the flattened index space
  uint32_t cbase, nc;  // cell range in the flattened key space
  uint32_t key_lo, key_hi;
  uint32_t walls, mbs;
  double Ld[3];        // L as double
  float Lf[3];         // L as float
  double h;            // time step
  float hf;
  float pad0;
  double ca, sa, omc;  // cos(alpha), sin(alpha), 1 - cos(alpha)
  double kT, mass, density, sd;  // sd = sqrt(kT / m)
  double gh[3];        // g * h
  uint32_t grav;
  uint32_t wcbase;     // walls: first index of this box's cells of the two
                       // wall-cut layers (2 L0 L1 per box) in a flat index space
  uint32_t slip;       // walls: specular reflection, no phantoms
  float uwf;           // uw as float
  double uw;           // no-slip walls: x velocity of the wall at z = H (cells per
                       // unit time); the wall at z = 0 moves with -uw
  uint32_t le;         // periodic z with Lees-Edwards shear
  float leuf;          // leu as float
  double leu;          // Lees-Edwards: x velocity of the image above the box
  uint32_t tbase;      // first tile (key order)
  uint32_t T, ntx;     // cells per tile, tiles per row
  uint32_t pad1;
};

struct BoxStep {       // per box and step, made a step ahead by the side work
  double s[3], sn[3];  // lattice shifts of t and t + 1
  double d1, d2;       // Lees-Edwards offsets at the end of step t and t + 1
  int32_t w[2];        // first row (y, z) of the window of next-step rows
};

struct Tile {          // one collide work item: cells [c0, c0 + nc) of box `box`
  uint32_t c0;         // first global cell key
  uint32_t tid;        // index in key order (run lists, counters, output positions)
  uint16_t nc;
  uint16_t box;
  uint32_t x0, y0, z0; // coordinates of the first cell in its box (z0: key layer)
};

struct PBlock {        // one block of a per-particle kernel
  uint32_t box;
  uint32_t p0;         // first global particle index
};

struct Ctrl {          // device-resident step state, read by every kernel
  uint64_t step;       // step index t of the next step
  uint32_t cur;        // which state buffer holds the current state (flips every step)
  uint32_t tri;        // which set of tile counters belongs to it (of three, in turn)
  uint32_t err;        // sticky error bits
  int32_t reorder;     // R
  uint32_t pad[2];
};

struct Run {           // consecutive slots of the state that belong to one tile
  uint32_t start, count;
};

struct Attempt {        // of a cell's gamma draw
  double z;
  uint16_t least;      // smallest particle count that accepts it
  uint16_t next;       // the cell's next attempt in the segment; 0: none
  uint32_t pad;
};

// Attempts that a draw block of b cells can list: 0.028 b on average.
__host__ __device__ constexpr uint32_t later_seg(uint32_t b) { return b / 4 + 48; }

struct PhantomSums {   // phantom particles of an occupied wall-cut cell
  double v[3];         // sum of their velocities
  double v2;           // sum of |v|^2
  double n;            // their number
  double pad;
};

template <int NV>
struct ObsRow {        // order-free sums of a block of particles (see k_obs_exact)
  long long d[NV][3];  // digits of 40 bits, lowest first
  int32_t anchor[NV];  // bin of the top digit: its unit is 2^(40 anchor - 1023)
};
struct Vec3 {
  double v[3];
};
struct ObsTotal {      // one sum of a box
  uint64_t lo[3];      // digits as 128-bit integers
  int64_t hi[3];
  int32_t anchor, pad;
};
template <int NV>
struct ObsResult {     // sums of a box as copied to the host
  uint32_t rows;       // rows to add; 0: totals
  ObsTotal total[NV];
  ObsRow<NV> row[kObsFew];
};

// Particle records, one per storage slot (array of structures): the collide
// gathers a particle with one or two 16-byte loads per 16 bytes of record, so
// that a run of consecutive slots is one contiguous span of memory instead of
// one span per component.  Positions and velocities are in cell units.
struct alignas(16) RecF64 {
  double x[3];
  double v[3];
};
struct alignas(8) RecF32 {
  float x[3];
  float v[3];
};
struct alignas(16) RecSplit {
  uint32_t cell;  // x | y << 11 | z << 22
  float o[3];     // offsets inside the cell, [0, 1)
  float v[3];
  uint32_t id;    // logical index of the particle in this slot
};
static_assert(sizeof(RecF64) == 48 && sizeof(RecF32) == 24 && sizeof(RecSplit) == 32,
              "record sizes");
constexpr size_t rec_bytes(int form) {
  return form == kFormF64 ? sizeof(RecF64) : (form == kFormF32 ? sizeof(RecF32) : sizeof(RecSplit));
}

// One state buffer.  Every step writes the state into the other buffer, tile
// by tile of the current step in key order, and inside the particles of one
// tile pass grouped by their tile of the next step (so that the next step
// gathers contiguous runs).  The logical index of slot i (its index in the
// caller's order, renumbered to the (cell, index) order on reorder steps) is
// id[i * id_stride]: an array of its own for FP64 and FP32 (stride 1), the id
// word of the record for the split form (stride 8).
struct StatePtrs {
  void* rec;
  uint32_t* id;
  uint32_t id_stride;
};

struct Dev {           // device pointers carved from the workspace
  StatePtrs S[2];
  // binning export (shares its memory with the run lists below)
  uint32_t* key;       // cell key per particle (storage order)
  uint16_t* rank;      // rank of the particle among those counted for its key
  uint32_t* perm;      // position in (cell, any order) -> stored slot
  uint32_t* hist;      // particles per cell
  uint32_t* offset;    // exclusive prefix, ncell + 1
  uint32_t* scan_blk;  // per scan-block totals
  // run lists of the tiles, one set per state buffer
  unsigned long long* tcnt[3];  // particles << 32 | runs; sets in turn (Ctrl::tri)
  Run* runs[2];        // maxr per tile
  uint32_t* rhead[2];  // maxr chain heads per tile (tiles with more runs)
  uint32_t* rnext[2];  // next slot of a chain, per slot; in a sort every
                       // particle's tile and rank there
  uint32_t* toff;      // first output slot of each tile
  uint32_t* tblk;      // particles per block of tiles
  uint32_t maxr, ntile;
  // what a step reads besides the particles, one set per state buffer
  BoxStep* bstep[2];
  Ctrl* ctrl;
  BoxDev* boxes;
  Tile* tiles;
  PBlock* pblocks;
  double* partials;    // per-block observable partial sums
  double* obs;         // kObsSums rows of their sums: high parts [4], low parts [4];
                       // or four ObsTotal and kObsRows rows (ObsRow<4>) of the
                       // order-free sums
  double4* draws[2];      // per cell: rotation axis, z of attempt 0 of the gamma draw
  // thermostat: per cell, the least count that accepts attempt 0 and the first
  // of its later attempts << 16 in the block's segment of later_seg(drawb) attempts
  uint32_t* least[2];
  Attempt* later[2];
  uint32_t drawb;      // cells per block of the draws
  PhantomSums* phs[2];  // walls only: phantom sums of wall-cut cells
  uint32_t ntot;       // particles over all boxes (bound of every particle index)
};

struct Side {          // side work of a collide (see k_collide)
  uint32_t nbox, ctot, wcells;
  int round32;
  uint32_t blocks;     // workgroups that do nothing else
  uint32_t period;     // every so many groups of 8 workgroups one of them
  uint32_t direct;     // every wavefront sums the tiles before its own
};

struct Launch {
  int form;
  int round_phantoms;      // split form: phantom velocities rounded to FP32
  int walls, mbs, amc;     // feature flags (identical for all boxes)
  int fixed;               // fixed-point cell sums
  int le;                  // some box has Lees-Edwards shear
  uint32_t nbox;
  uint64_t ntot, ctot;     // particles, cells over all boxes
  uint32_t ntiles, npblocks, nscan;
  uint32_t collide_grid;
  uint32_t resident;       // collide workgroups that fit the chip at once
  uint32_t wcells;         // walls: cells of the wall-cut layers over all boxes
  int xcd_remap;
  uint32_t seq;            // number of the step in its launch sequence (see Ctrl)
  hipStream_t stream;
};

// Launchers (mpc_kernels.hip).
hipError_t launch_zero_u32(uint32_t* p, uint64_t n, hipStream_t s);
hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t value, hipStream_t s);
hipError_t launch_binning(const Dev& d, const Launch& l, const StatePtrs& S, uint64_t t);
hipError_t launch_sort(const Dev& d, const Launch& l, uint32_t from, uint32_t to, int caller);
hipError_t launch_prefix(const Dev& d, const Launch& l);
hipError_t launch_advance(const Dev& d, const Launch& l, uint32_t n);
hipError_t launch_collide(const Dev& d, const Launch& l);
hipError_t launch_set_ctrl(const Dev& d, const Launch& l, uint64_t step, uint32_t cur,
                           int32_t reorder, int clear_err);
hipError_t launch_init_state(const Dev& d, const Launch& l, uint64_t seed);
// observables of particle blocks [pb0, pb0 + npb) of state buffer cur; order:
// slots in the order of the sums (null: slot order)
hipError_t launch_obs_order(const Dev& d, const Launch& l, uint32_t box, uint32_t nrows,
                            uint32_t l0, uint32_t cur, uint32_t To, uint32_t* order);
hipError_t launch_obs_pass1(const Dev& d, const Launch& l, uint32_t pb0, uint32_t npb, uint32_t cur,
                            const uint32_t* order);
// NV sums (4: momentum and energy; 1: relative energy, vmean) of a box
template <int NV>
hipError_t launch_obs_exact(const Dev& d, const Launch& l, uint32_t box, uint32_t np, uint32_t cur,
                            const Vec3& vmean, ObsResult<NV>* out);
hipError_t launch_obs_sums(const Dev& d, const Launch& l, uint32_t pb0, uint32_t npb);
hipError_t launch_remove_mean(const Dev& d, const Launch& l, const double* vmean_dev);
// sel: box-local logical indices, overwritten; keys: 2 (mask + 1) entries of a
// hash table, or null and inv: np entries; out: [6][m] FP64
hipError_t launch_gather_particles(const Dev& d, const Launch& l, const StatePtrs& S,
                                  uint32_t* inv, uint32_t* keys, uint32_t mask, uint32_t pbase,
                                  uint32_t np, uint32_t* sel, uint32_t m, double* out);
// FP64 arrays x[3][m], v[3][m] on the device <-> records of particles i0 ..
// i0 + m - 1 of a box; in: checked if bad is given, else packed
hipError_t launch_state_in(const Dev& d, const Launch& l, const StatePtrs& S, uint32_t box,
                           uint32_t i0, const double* x, const double* v, uint32_t m, double a,
                           uint32_t* bad);
hipError_t launch_state_out(const Launch& l, const StatePtrs& S, uint32_t pbase, uint32_t np,
                            uint32_t i0, double* x, double* v, uint32_t m, double a,
                            uint32_t* bad);
// box 0, FP64 form: caller's device arrays (physical units) <-> state buffer cur
hipError_t launch_load_f64(const Dev& d, const Launch& l, const double* x, const double* v,
                           uint32_t n, double a, uint32_t cur);
hipError_t launch_store_f64(const Dev& d, const Launch& l, double* x, double* v, uint32_t n,
                            double a, uint32_t cur);
hipError_t launch_canon_perm(const Dev& d, const Launch& l, const StatePtrs& ids);
hipError_t collide_occupancy(const Launch& l, int* blocks_per_cu);  // flags of l only

}  // namespace mpc
