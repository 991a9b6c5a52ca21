// mpc_capi.cpp -- host side of the C ABI declared in include/mpc.h: parameter
// validation, workspace planning, tile tables, step sequencing (direct launches
// or replayed hipGraphs of several steps), state transfer, observables.
#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include <algorithm>
#include <cstdio>
#include <mutex>
#include <string>
#include <vector>

#include "mpc.h"
#include "mpc_internal.h"
#include "sample_table.h"

using namespace mpc;

namespace {

constexpr uint64_t kMaxIndex = 0x7fffffffull;  // particle and cell indices stay below 2^31
constexpr int64_t kStateChunk = int64_t(1) << 22;  // particles per host staging chunk
constexpr size_t kKeepStage = (size_t)64 << 20;    // largest device staging a handle keeps
constexpr size_t kMaxStage = (size_t)1 << 30;      // and largest of one call
constexpr size_t kSmallCopy = (size_t)256 << 10;   // a state read back in one copy
constexpr size_t kOwnExport = (size_t)1 << 20;     // largest binning export with memory of its own
constexpr int kMinTileCells = 4;
constexpr int32_t kMaxGraphSteps = 1000;  // steps captured in one graph
static_assert(MPC_MAX_CELL_PARTICLES == kTileCap, "the ABI's cell limit is one collide pass");

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct BoxPlan {
  uint64_t n, ncell;
  int nlz;
};

// Cells per tile.  The mean particle count of a tile is at most 84 % of the
// capacity of one collide pass, so that about one tile in 400 at 10 particles
// per cell needs a second pass.  With fewer than 2048 such tiles in all boxes
// (`rows`: their rows of cells), shorter ones down to 80 particles put more
// wavefronts to work: 24^3 with the thermostat 25.9 us a step with tiles of 8
// cells, 27.2 with 12, 29.9 with 20 (and 29.7 with 4); 41 x 33 x 27 35.1 with
// 14, 43.2 with 21; 64^3 (4096 rows) 109 with 16, 127 with 11.  The tiles of a
// row are of about equal length: 75^3 158 us with 19, 182 with 21.
int auto_tile_cells(double density, int l0, uint64_t rows) {
  const double target = 0.84 * kTileCap / density;
  const int most = (int)std::max(1.0, std::min<double>(kTileMaxCells, floor(target)));
  const int least = (int)std::max(1.0, std::min<double>(most, ceil(80.0 / density)));
  const int want = (int)std::min<uint64_t>((2048 + rows - 1) / rows, (uint64_t)(l0 / least));
  const int per_row = std::max((l0 + most - 1) / most, want);
  return (l0 + per_row - 1) / per_row;
}

// Runs that the table of a tile holds, of at most kMaxRuns: three rows of three
// tiles in three layers send it one run each, and a tile of few particles has
// no more runs than particles, so a table for the mean number of particles and
// three standard deviations is enough (a fuller tile goes to chains).  Tables of
// 32 runs had taken 768 bytes for every tile, eight times what else a thin
// sparse box needs.
uint64_t tile_runs(double density, int tile_cells) {
  const double mean = density * tile_cells;
  return (uint64_t)std::max(1.0, std::min<double>(kMaxRuns, ceil(mean + 3.0 * sqrt(mean))));
}

struct Plan {
  std::vector<BoxPlan> box;
  uint64_t ntot = 0, ctot = 0, cpad = 0;
  uint32_t nscan = 0;
  uint64_t max_tiles = 0, npblocks = 0;
  uint64_t rows = 0;      // rows of cells in all boxes
  uint32_t drawb = 0;     // cells per draw block
  size_t off_shared = 0, shared = 0;  // run lists and binning export
  bool own_export = false;            // the export does not take the run lists' memory
  uint64_t run_pool = 0;  // runs of all tiles' tables per state buffer
  size_t charge = 0;      // bytes the static scratch is checked against
  size_t rec = 0;  // bytes per particle record
  bool split = false;
  // byte offsets in the workspace: records of the two state buffers and, for
  // FP64 and FP32, their logical-index arrays (the split record holds its id)
  size_t off_rec[2] = {}, off_id[2] = {};
  size_t off_rank = 0, off_phs[2] = {}, off_least[2] = {}, off_later[2] = {}, off_bstep[2] = {};
  size_t off_tcnt[3] = {}, off_runs[2] = {}, off_rhead[2] = {}, off_rnext[2] = {}, off_toff = 0,
         off_tblk = 0;
  size_t off_key = 0, off_perm = 0, off_hist = 0, off_offset = 0, off_scan = 0, off_ctrl = 0,
         off_boxes = 0, off_tiles = 0, off_pblocks = 0, off_partials = 0, off_vmean = 0,
         off_draws[2] = {}, off_obs = 0;
  size_t total = 0;
};

int validate(const mpc_params* p, int32_t nbox, std::string* why) {
  if (!p || nbox < 1 || nbox > MPC_MAX_BOXES) {
    *why = "need 1..MPC_MAX_BOXES boxes";
    return MPC_EINVAL;
  }
  for (int32_t b = 0; b < nbox; ++b) {
    const mpc_params& q = p[b];
    char msg[160];
    auto bad = [&](const char* what) {
      snprintf(msg, sizeof msg, "box %d: %s", b, what);
      *why = msg;
      return MPC_EINVAL;
    };
    if (q.form < MPC_FP64 || q.form > MPC_SPLIT32) return bad("unknown form");
    if (q.flags & ~(uint32_t)(MPC_MBS | MPC_WALLS_Z | MPC_SLIP | MPC_AMC | MPC_FIXED_SUMS))
      return bad("unknown flags");
    if ((q.flags & MPC_SLIP) && !(q.flags & MPC_WALLS_Z)) return bad("MPC_SLIP needs MPC_WALLS_Z");
    if (!isfinite(q.wall_u)) return bad("wall_u must be finite");
    if (q.wall_u != 0.0 && (!(q.flags & MPC_WALLS_Z) || (q.flags & MPC_SLIP)))
      return bad("wall_u needs no-slip walls (MPC_WALLS_Z without MPC_SLIP)");
    if (!isfinite(q.le_u)) return bad("le_u must be finite");
    if (q.le_u != 0.0 && (q.flags & MPC_WALLS_Z))
      return bad("le_u (Lees-Edwards) needs a periodic box (no MPC_WALLS_Z)");
    if ((q.flags & MPC_AMC) && (q.flags & MPC_WALLS_Z) && !(q.flags & MPC_SLIP))
      return bad("MPC_AMC is defined for periodic boxes and slip walls (MPC_SLIP)");
    if (q.form != p[0].form || q.flags != p[0].flags || q.reorder_every != p[0].reorder_every)
      return bad("form, flags and reorder_every must be equal for all boxes");
    if (q.reorder_every < 0) return bad("reorder_every < 0");
    for (int k = 0; k < 3; ++k)
      if (q.L[k] < 1) return bad("L must be >= 1");
    if (!(q.a > 0.0) || !isfinite(q.a)) return bad("a must be > 0");
    if (!(q.density > 0.0) || !isfinite(q.density)) return bad("density must be > 0");
    if (!(q.dt > 0.0) || !isfinite(q.dt)) return bad("dt must be > 0");
    if (!isfinite(q.alpha)) return bad("alpha must be finite");
    if (!(q.kT > 0.0) || !isfinite(q.kT)) return bad("kT must be > 0");
    if (!(q.mass > 0.0) || !isfinite(q.mass)) return bad("mass must be > 0");
    for (int k = 0; k < 3; ++k)
      if (!isfinite(q.g[k])) return bad("g must be finite");
    if (q.form == MPC_SPLIT32) {
      const int zmax = (q.flags & MPC_WALLS_Z) ? 1023 : 1024;
      if (q.L[0] > 2048 || q.L[1] > 2048 || q.L[2] > zmax) {
        snprintf(msg, sizeof msg, "box %d: split form needs L0, L1 <= 2048, L2 <= %d", b, zmax);
        *why = msg;
        return MPC_ERANGE;
      }
    }
  }
  return MPC_OK;
}

// What a call of the allocation-free entry point is charged against the limit
// of its scratch: state and ids 56 B per particle and buffer, 10 B per
// particle and 8 B per cell for binning, 32 B of draws per cell, tables.  The
// limit is part of the interface, so it does not follow the workspace layout.
size_t scratch_charge(const mpc_params* p, const Plan& P) {
  size_t off = 0;
  auto take = [&](size_t bytes) { off = align256(off + bytes); };
  const size_t nbox = P.box.size();
  uint64_t tiles = 0;
  for (size_t b = 0; b < nbox; ++b)
    tiles += (uint64_t)p[b].L[1] * P.box[b].nlz * ((p[b].L[0] + kMinTileCells - 1) / kMinTileCells);
  for (int k = 0; k < 2; ++k) {
    take(P.rec * P.ntot);
    if (!P.split) take(4 * P.ntot);
  }
  take(4 * P.ntot);
  take(4 * P.ntot);
  take(2 * P.ntot);
  take(4 * P.cpad);
  take(4 * (P.cpad + 1));
  take(4 * (size_t)P.nscan);
  take(32);
  take(280 * nbox);
  take(20 * tiles);
  take(8 * P.npblocks);
  take(32 * P.npblocks);
  take(24 * nbox);
  take(32 * P.cpad);
  if (p[0].flags & MPC_WALLS_Z) take(48 * P.cpad);
  return off;
}

int make_plan(const mpc_params* p, int32_t nbox, Plan& P, std::string* why) {
  int rc = validate(p, nbox, why);
  if (rc) return rc;
  P.box.resize(nbox);
  uint64_t tiles = 0, maxr = 1;
  for (int32_t b = 0; b < nbox; ++b)
    P.rows += (uint64_t)p[b].L[1] * ((uint64_t)p[b].L[2] + ((p[b].flags & MPC_WALLS_Z) ? 2 : 0));
  for (int32_t b = 0; b < nbox; ++b) {
    const mpc_params& q = p[b];
    const bool walls = q.flags & MPC_WALLS_Z;
    const double vol = (double)q.L[0] * q.L[1] * q.L[2];
    const double nd = llround(q.density * vol);
    const int nlz = walls ? q.L[2] + 2 : q.L[2];
    const double cd = (double)q.L[0] * q.L[1] * nlz;
    if (nd < 1.0) {
      *why = "box with no particles";
      return MPC_EINVAL;
    }
    if (nd > (double)kMaxIndex || cd > (double)kMaxIndex) {
      *why = "particles or cells of a box >= 2^31";
      return MPC_ERANGE;
    }
    P.box[b].n = (uint64_t)nd;
    P.box[b].ncell = (uint64_t)cd;
    P.box[b].nlz = nlz;
    P.ntot += P.box[b].n;
    P.ctot += P.box[b].ncell;
    const uint64_t rows = (uint64_t)q.L[1] * nlz;
    const int ta = auto_tile_cells(q.density, q.L[0], P.rows);
    const uint64_t auto_tiles = rows * ((q.L[0] + ta - 1) / ta);
    P.max_tiles += std::max(auto_tiles, rows * ((q.L[0] + kMinTileCells - 1) / kMinTileCells));
    tiles += auto_tiles;
    maxr = std::max(maxr, tile_runs(q.density, ta));  // one length for all boxes
    P.npblocks += (P.box[b].n + kPartBlock - 1) / kPartBlock;
  }
  P.nscan = (uint32_t)((P.ctot + kScanBlock - 1) / kScanBlock);
  P.cpad = (uint64_t)P.nscan * kScanBlock;
  if (P.ntot > kMaxIndex || P.cpad + 1 > kMaxIndex) {
    *why = "total particles or cells >= 2^31";
    return MPC_ERANGE;
  }
  const int form = p[0].form;
  P.split = form == MPC_SPLIT32;
  P.rec = form == MPC_FP64 ? sizeof(RecF64) : (form == MPC_FP32 ? sizeof(RecF32) : sizeof(RecSplit));
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align256(off + bytes);
    return o;
  };
  for (int s = 0; s < 2; ++s) {
    P.off_rec[s] = take(P.rec * P.ntot);
    P.off_id[s] = P.split ? 0 : take(4 * P.ntot);
  }
  // the binning export and the run lists of the tiles share their memory: the
  // export is formed from the last step's input when it is asked for, and the
  // next step then sorts the state by tile again.  That sort is most of a step of
  // a small box (3^3: 60 us), whose export has its own memory
  const size_t shared0 = off;
  P.off_key = take(4 * P.ntot);
  P.off_perm = take(4 * P.ntot);
  P.off_rank = take(2 * P.ntot);
  P.off_hist = take(4 * P.cpad);
  P.off_offset = take(4 * (P.cpad + 1));
  P.off_scan = take(4 * (size_t)P.nscan);
  const size_t shared1 = off;
  P.own_export = shared1 - shared0 <= kOwnExport;
  if (!P.own_export) off = shared0;
  // a tiling with more tiles than the automatic one has shorter run tables,
  // of at least one run a tile
  P.run_pool = std::max<uint64_t>(tiles * maxr, P.max_tiles);
  for (int k = 0; k < 3; ++k) P.off_tcnt[k] = take(8 * P.max_tiles);
  for (int k = 0; k < 2; ++k) {
    P.off_runs[k] = take(sizeof(Run) * P.run_pool);
    P.off_rhead[k] = take(4 * P.run_pool);
    P.off_rnext[k] = take(4 * P.ntot);
  }
  P.off_tblk = take(4 * (P.max_tiles / kTileBlock + 1));
  off = std::max(off, shared1);
  P.off_shared = shared0;
  P.shared = off - shared0;
  P.off_toff = take(4 * P.max_tiles);
  P.off_ctrl = take(sizeof(Ctrl));
  P.off_boxes = take(sizeof(BoxDev) * nbox);
  P.off_tiles = take(sizeof(Tile) * P.max_tiles);
  P.off_pblocks = take(sizeof(PBlock) * P.npblocks);
  P.off_partials = take(sizeof(double) * 4 * P.npblocks);
  P.off_vmean = take(sizeof(double) * 3 * nbox);
  P.off_obs = take(std::max<size_t>(sizeof(double) * 8 * kObsSums,
                                    4 * sizeof(ObsTotal) + sizeof(ObsRow<4>) *
                                        std::min<uint64_t>(kObsRows, P.npblocks)));
  // draw blocks of one wavefront each: about 1024 of them if the box is small,
  // so that they run beside each other, else as long as their lists allow
  P.drawb = (uint32_t)std::min<uint64_t>(
      kMaxDrawBlock, std::max<uint64_t>(kMinDrawBlock, (P.ctot + 65535) / 65536 * 64));
  const uint64_t ndraw = (P.ctot + P.drawb - 1) / P.drawb;
  for (int k = 0; k < 2; ++k) {
    P.off_bstep[k] = take(sizeof(BoxStep) * nbox);
    P.off_draws[k] = take(sizeof(double4) * P.cpad);
    if (p[0].flags & MPC_MBS) {
      P.off_least[k] = take(4 * P.cpad);
      P.off_later[k] = take(sizeof(Attempt) * later_seg(P.drawb) * ndraw);
    }
    if (p[0].flags & MPC_WALLS_Z) P.off_phs[k] = take(sizeof(PhantomSums) * P.cpad);
  }
  P.charge = scratch_charge(p, P);
  P.total = off;
  return MPC_OK;
}

// Device scratch of the allocation-free entry point: the whole workspace of
// one call lives here.  Each device holds its own copy from module load to
// process end; host code reaches it only through the address that
// hipGetSymbolAddress returns for the current device.
constexpr size_t kScratchLimit = (size_t)256 << 20;  // see scratch_charge
// The workspace of a call within the limit: at most 2.7 times its charge, in a
// box of rows of one cell with 0.1 particles per cell, where the cells' draws (64
// bytes, 82 with the thermostat) and the tiles' tables (52 bytes and 24 a run)
// dominate.
constexpr size_t kScratchBytes = (size_t)704 << 20;
static __device__ __align__(256) uint8_t scratch[kScratchBytes];
constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
void* scratch_ptr[kMaxDevices] = {};

int scratch_of_current_device(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return MPC_EHIP;
  std::lock_guard<std::mutex> lock(scratch_mu);
  if (!scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr)
      return MPC_EHIP;
    scratch_ptr[dev] = ptr;
  }
  *out = scratch_ptr[dev];
  return MPC_OK;
}

struct Neumaier {
  double s = 0.0, c = 0.0;
  void add(double x) {
    const double t = s + x;
    if (fabs(s) >= fabs(x)) {
      c += (s - t) + x;
    } else {
      c += (x - t) + s;
    }
    s = t;
  }
  double val() const { return s + c; }
};

}  // namespace

// Order of the slots of a box: the caller's; the output of a step of this
// tiling; neither (runs to be appended in any order, tiles of another tiling).
enum : char { kSlotsCaller, kSlotsStep, kSlotsOther };

struct mpc_sim {
  std::vector<mpc_params> params;
  Plan plan;
  std::vector<BoxDev> boxes;
  std::vector<Tile> tiles;
  std::vector<PBlock> pblocks;
  std::vector<uint32_t> box_pb0;  // first pblock of each box, nbox + 1 entries
  Dev dev{};
  Launch L{};
  int form = 0;
  int32_t R = 0;
  uint64_t step = 0;
  uint32_t cur = 0;
  bool keys_valid = false;
  bool have_binning = false;
  bool binning_ready = false;  // the binning export holds the last step's binning
  std::vector<char> slots;     // per box: what its slots' order is (kSlots*)
  bool use_graph = true;
  int32_t graph_steps = 1;         // steps per replay of the chunk graph
  bool graph_ready = false;
  hipGraphExec_t gexec = nullptr;  // graph_chunk() steps
  hipStream_t capture_stream = nullptr;
  int tile_override = 0, grid_override = 0, yblock = 8;
  int order = 0;  // tile order: 0 = row by row inside a block of rows, 1 = x-segment major
  int num_cu = 256, occupancy = 4;
  double* vmean = nullptr;
  char* ws = nullptr;
  int device = 0;         // of the workspace (and the stream)
  char* stage = nullptr;  // device staging of set_state and get_state, kept up to kKeepStage
  size_t stage_bytes = 0;
  std::string err;
};

namespace {

int hip_fail(mpc_sim* s, hipError_t e, const char* where) {
  if (e == hipSuccess) return MPC_OK;
  if (s) {
    s->err = std::string(where) + ": " + hipGetErrorString(e);
  }
  return MPC_EHIP;
}
#define HIPCHK(s, expr)                                  \
  do {                                                   \
    hipError_t _e = (expr);                              \
    if (_e != hipSuccess) return hip_fail((s), _e, #expr); \
  } while (0)

// Tiles are runs of at most T consecutive cells inside one row (fixed y and z),
// so a tile's particles land in three tiles of nine rows of the next step
// (others are handled one by one).  Tiles are numbered in key order, which is
// the order of their particles in memory, and listed (processed) so
// that the persistent grid, which hands each XCD a contiguous part of the list,
// keeps cells that exchange particles on one XCD at the same time: each XCD
// gets a slab of z planes, walked in blocks of `yblock` rows with z inside a
// block (order 0: each row's tiles in turn; order 1: one x segment of all
// rows of the block, then the next), so the rows a tile reads from are in
// flight together.
void build_tiles(mpc_sim* s) {
  s->tiles.clear();
  const uint64_t yb = (uint64_t)std::max(1, s->yblock);
  uint32_t tbase = 0;
  for (BoxDev& B : s->boxes) {
    B.T = (uint32_t)(s->tile_override ? s->tile_override
                                      : auto_tile_cells(B.density, B.L[0], s->plan.rows));
    B.ntx = ((uint32_t)B.L[0] + B.T - 1) / B.T;
    B.tbase = tbase;
    tbase += (uint32_t)B.nlz * (uint32_t)B.L[1] * B.ntx;
  }
  s->tiles.reserve(tbase);  // once: growing it box by box copied all tiles so far
  for (size_t b = 0; b < s->boxes.size(); ++b) {
    const BoxDev& B = s->boxes[b];
    const int T = (int)B.T;
    const uint64_t L0 = (uint64_t)B.L[0], L1 = (uint64_t)B.L[1], nz = (uint64_t)B.nlz;
    const uint64_t ntx = B.ntx;
    auto add = [&](uint64_t cz, uint64_t cy, uint64_t tx) {
      const uint64_t row = cz * L1 + cy, cx = tx * (uint64_t)T;
      Tile t;
      t.c0 = B.cbase + (uint32_t)(row * L0 + cx);
      t.tid = B.tbase + (uint32_t)(row * ntx + tx);
      t.nc = (uint16_t)std::min<uint64_t>((uint64_t)T, L0 - cx);
      t.box = (uint16_t)b;
      t.x0 = (uint32_t)cx;
      t.y0 = (uint32_t)cy;
      t.z0 = (uint32_t)cz;
      s->tiles.push_back(t);
    };
    for (uint64_t slab = 0; slab < 8; ++slab) {
      const uint64_t z0 = (slab * nz + 7) / 8, z1 = ((slab + 1) * nz + 7) / 8;  // cz * 8 / nz == slab
      for (uint64_t y0 = 0; y0 < L1; y0 += yb) {
        const uint64_t y1 = std::min(L1, y0 + yb);
        // order 0: the rows of a block one after the other; order 1: the same
        // x segment of every row of the block, then the next segment
        for (uint64_t seg = 0; seg < (s->order == 0 ? 1 : ntx); ++seg)
          for (uint64_t cz = z0; cz < z1; ++cz)
            for (uint64_t cy = y0; cy < y1; ++cy) {
              if (s->order == 0) {
                for (uint64_t tx = 0; tx < ntx; ++tx) add(cz, cy, tx);
              } else {
                add(cz, cy, seg);
              }
            }
      }
    }
  }
  s->L.ntiles = (uint32_t)s->tiles.size();
  s->dev.ntile = s->L.ntiles;
  s->dev.maxr = (uint32_t)std::min<uint64_t>(kMaxRuns, s->plan.run_pool / s->tiles.size());
  s->keys_valid = false;  // the run lists belong to a tiling, and so do the steps' outputs
  s->slots.resize(s->boxes.size(), kSlotsCaller);
  for (char& o : s->slots)
    if (o == kSlotsStep) o = kSlotsOther;
  // default grid: about four tiles per wavefront.  Short-lived wavefronts keep
  // the tiles in flight close together in the list, so that the gathered runs
  // are still in L2 (collide of 384^3 FP64 16.7 ms with 12288 wavefronts of 230
  // tiles, 15.0 with 12 tiles each, 14.5 with two to six; 256^3 4.79, 4.50 and
  // 4.4; split with the thermostat 3.58, 3.46 and 3.50); one tile each leaves
  // nothing to fetch ahead (256^3 with the thermostat 5.2 against 4.6 ms)
  const uint32_t full = (uint32_t)(s->num_cu * std::max(1, s->occupancy));
  uint32_t g = s->grid_override ? (uint32_t)s->grid_override
                                : std::max(4 * full, (s->L.ntiles / 4 + 7) / 8 * 8);
  s->L.resident = full;
  // one launch takes 2^32 threads, side work included
  g = std::max<uint32_t>(1, std::min<uint32_t>(std::min<uint32_t>(g, s->L.ntiles), 1u << 25));
  s->L.collide_grid = g;
}

int upload_tables(mpc_sim* s) {
  HIPCHK(s, hipMemcpyAsync(s->dev.tiles, s->tiles.data(), sizeof(Tile) * s->tiles.size(),
                           hipMemcpyHostToDevice, s->L.stream));
  HIPCHK(s, hipMemcpyAsync(s->dev.boxes, s->boxes.data(), sizeof(BoxDev) * s->boxes.size(),
                           hipMemcpyHostToDevice, s->L.stream));
  HIPCHK(s, hipStreamSynchronize(s->L.stream));
  return MPC_OK;
}

int read_ctrl(mpc_sim* s, Ctrl* c) {
  HIPCHK(s, hipMemcpyAsync(c, s->dev.ctrl, sizeof(Ctrl), hipMemcpyDeviceToHost, s->L.stream));
  HIPCHK(s, hipStreamSynchronize(s->L.stream));
  return MPC_OK;
}

int check_sticky(mpc_sim* s) {
  Ctrl c;
  int rc = read_ctrl(s, &c);
  if (rc) return rc;
  if (c.err & kErrKey) {
    s->err = "a particle left the box or is not finite";
    return MPC_ESTATE;
  }
  if (c.err & kErrCellOverflow) {
    s->err = "a collision cell held more than MPC_MAX_CELL_PARTICLES (256) particles; "
             "it was streamed but not collided";
    return MPC_ERANGE;
  }
  if (c.err & kErrDraws) {
    s->err = "the list of repeated thermostat draws of a block of cells is full";
    return MPC_ERANGE;
  }
  if (c.err & kErrFixRange) {
    s->err = "a fixed-point summand was outside |x| < 2^37 (cell units)";
    return MPC_ERANGE;
  }
  return MPC_OK;
}

// The launches of n steps on `st`.
hipError_t enqueue_steps(mpc_sim* s, hipStream_t st, int64_t n) {
  Launch l = s->L;
  l.stream = st;
  for (l.seq = 0; l.seq < (uint32_t)n; ++l.seq) {
    hipError_t e = launch_prefix(s->dev, l);
    if (e == hipSuccess) e = launch_collide(s->dev, l);
    if (e != hipSuccess) return e;
  }
  return launch_advance(s->dev, l, (uint32_t)n);
}

// A state set from outside (or a binning export, which takes the memory of
// the run lists): sort by tile of the next step into the other buffer.
int ensure_keys(mpc_sim* s) {
  if (s->keys_valid) return MPC_OK;
  HIPCHK(s, launch_set_ctrl(s->dev, s->L, s->step, s->cur ^ 1u, s->R, 0));
  const bool caller = std::count(s->slots.begin(), s->slots.end(), (char)kSlotsCaller) ==
                      (int64_t)s->slots.size();
  HIPCHK(s, launch_sort(s->dev, s->L, s->cur, s->cur ^ 1u, caller));
  s->cur ^= 1u;
  s->slots.assign(s->boxes.size(), kSlotsOther);
  s->keys_valid = true;
  s->binning_ready = false;
  return MPC_OK;
}

void advance_mirror(mpc_sim* s, int64_t n) {
  s->cur ^= (uint32_t)(n & 1);
  s->step += (uint64_t)n;
}

int drop_graph(mpc_sim* s) {
  if (s->gexec) {
    HIPCHK(s, hipGraphExecDestroy(s->gexec));
    s->gexec = nullptr;
  }
  s->graph_ready = false;
  return MPC_OK;
}

// Steps per graph.  Without a wish of the caller 16: graphs of 2 steps take 13.5
// us a step at 16^3, of 8 11.0, of 16 and single launches 10.6, of 50 10.3 (24^3
// with the thermostat 18.2, 15.7, 15.3 and 15.0), and a graph spares the host.
int64_t graph_chunk(const mpc_sim* s) { return s->graph_steps > 1 ? s->graph_steps : 16; }

// One executable graph of `steps` consecutive steps (every step reads the
// step counter and the state buffer index from device memory, so one graph
// serves every replay).
int capture_steps(mpc_sim* s, int64_t steps, hipGraphExec_t* out) {
  if (!s->capture_stream) HIPCHK(s, hipStreamCreateWithFlags(&s->capture_stream, hipStreamNonBlocking));
  hipGraph_t g = nullptr;
  HIPCHK(s, hipStreamBeginCapture(s->capture_stream, hipStreamCaptureModeThreadLocal));
  hipError_t e = enqueue_steps(s, s->capture_stream, steps);
  hipError_t e2 = hipStreamEndCapture(s->capture_stream, &g);
  if (e != hipSuccess) {
    if (g) (void)hipGraphDestroy(g);
    return hip_fail(s, e, "capture step");
  }
  if (e2 != hipSuccess) return hip_fail(s, e2, "hipStreamEndCapture");
  e = hipGraphInstantiate(out, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (e != hipSuccess) return hip_fail(s, e, "hipGraphInstantiate");
  return MPC_OK;
}

int capture_graph(mpc_sim* s) {
  if (s->graph_ready) return MPC_OK;
  const int rc = capture_steps(s, graph_chunk(s), &s->gexec);
  if (rc) return rc;
  s->graph_ready = true;
  return MPC_OK;
}

template <typename T>
int copy_d2h(mpc_sim* s, const void* src_base, uint64_t elem0, std::vector<T>& dst) {
  HIPCHK(s, hipMemcpyAsync(dst.data(), (const T*)src_base + elem0, sizeof(T) * dst.size(),
                           hipMemcpyDeviceToHost, s->L.stream));
  return MPC_OK;
}

// Logical indices of slots p0 .. p0 + out.size() - 1 of state buffer S: a copy
// of the id array, or of the records a chunk at a time (ids inside records).
int read_ids(mpc_sim* s, const StatePtrs& S, uint64_t p0, std::vector<uint32_t>& out) {
  const uint64_t n = out.size();
  if (S.id_stride == 1) {
    HIPCHK(s, hipMemcpyAsync(out.data(), S.id + p0, sizeof(uint32_t) * n, hipMemcpyDeviceToHost,
                             s->L.stream));
    HIPCHK(s, hipStreamSynchronize(s->L.stream));
    return MPC_OK;
  }
  const uint64_t st = S.id_stride;
  const uint64_t w = (uint64_t)(S.id - (const uint32_t*)S.rec);  // id word inside a record
  const uint64_t chunk = std::min<uint64_t>(n, (uint64_t)kStateChunk);
  std::vector<uint32_t> buf((size_t)(chunk * st));
  for (uint64_t i0 = 0; i0 < n; i0 += chunk) {
    const uint64_t m = std::min(chunk, n - i0);
    HIPCHK(s, hipMemcpyAsync(buf.data(), (const uint32_t*)S.rec + (p0 + i0) * st,
                             sizeof(uint32_t) * m * st, hipMemcpyDeviceToHost, s->L.stream));
    HIPCHK(s, hipStreamSynchronize(s->L.stream));
    for (uint64_t i = 0; i < m; ++i) out[i0 + i] = buf[i * st + w];
  }
  return MPC_OK;
}

// Makes the handle's device the current one for a call that allocates: the
// caller's current device may be another.
struct OnDevice {
  int before = -1;
  explicit OnDevice(const mpc_sim* s) {
    int now = -1;
    if (hipGetDevice(&now) == hipSuccess && now != s->device && hipSetDevice(s->device) == hipSuccess)
      before = now;
  }
  ~OnDevice() {
    if (before >= 0) (void)hipSetDevice(before);
  }
};

// Device staging for up to n particles (48 bytes each) and a flag before them.
// Small ones stay with the handle; without device memory the run lists' part
// of the workspace serves, and the next step sorts the state again.
struct Stage {
  mpc_sim* s = nullptr;
  char* own = nullptr;
  uint32_t* flag = nullptr;
  double* data = nullptr;
  int64_t cap = 0;  // particles
  ~Stage() {
    if (own) (void)hipFree(own);
  }
};
void get_stage(mpc_sim* s, int64_t n, Stage* st) {
  st->s = s;
  const size_t want = std::min<size_t>(kMaxStage, 256 + 48 * (size_t)n);
  char* p = nullptr;
  size_t bytes = want;
  if (want <= s->stage_bytes) {
    p = s->stage;
    bytes = s->stage_bytes;
  } else if (hipMalloc((void**)&p, want) == hipSuccess) {
    if (want <= kKeepStage) {
      if (s->stage) (void)hipFree(s->stage);
      s->stage = p;
      s->stage_bytes = want;
    } else {
      st->own = p;
    }
  } else {
    (void)hipGetLastError();
    p = s->ws + s->plan.off_shared;
    bytes = s->plan.shared;
    s->keys_valid = false;
    s->binning_ready = false;
  }
  st->flag = (uint32_t*)p;
  st->data = (double*)(p + 256);
  st->cap = (int64_t)((bytes - 256) / 48);
}

// Rows k of host arrays x[3][n], v[3][n], particles i0 .. i0 + m - 1 <-> the
// staged arrays x[3][m], v[3][m].
int stage_copy(mpc_sim* s, double* dx, double* dv, const double* x, const double* v, int64_t n,
               int64_t i0, int64_t m, bool in) {
  for (int a = 0; a < 2; ++a) {
    double* d = a ? dv : dx;
    double* h = const_cast<double*>(a ? v : x);
    const int rows = m == n ? 1 : 3;  // whole arrays are contiguous
    for (int k = 0; k < rows; ++k) {
      double* dk = d + (size_t)k * m;
      double* hk = h + (size_t)k * n + i0;
      const size_t bytes = sizeof(double) * (size_t)m * (rows == 1 ? 3 : 1);
      HIPCHK(s, in ? hipMemcpyAsync(dk, hk, bytes, hipMemcpyHostToDevice, s->L.stream)
                   : hipMemcpyAsync(hk, dk, bytes, hipMemcpyDeviceToHost, s->L.stream));
    }
  }
  return MPC_OK;
}

// Cells per tile of the order of the observables' sums: a mean of 95 % of its
// passes' capacity.
uint32_t obs_tile_cells(double density) {
  const double target = 0.95 * kObsPass / density;
  return (uint32_t)std::max<double>(kMinTileCells, std::min<double>(kTileMaxCells, floor(target)));
}

// Momentum and energy from the partial sums of particle blocks [pb0, pb0 +
// npb), compensated.  Of many blocks the device first makes kObsSums sums of
// twice the precision each (copied and added here, the 553 000 blocks of a
// 384^3 box had taken 4 ms per pass).
int sum_partials(mpc_sim* s, uint32_t pb0, uint32_t npb, double (&sum)[4]) {
  const bool many = npb > 1024;
  const size_t rows = many ? kObsSums : npb, width = many ? 8 : 4;
  std::vector<double> part(rows * width);
  if (many) HIPCHK(s, launch_obs_sums(s->dev, s->L, pb0, npb));
  HIPCHK(s, hipMemcpyAsync(part.data(), many ? s->dev.obs : s->dev.partials + 4 * (size_t)pb0,
                           sizeof(double) * part.size(), hipMemcpyDeviceToHost, s->L.stream));
  HIPCHK(s, hipStreamSynchronize(s->L.stream));
  for (int k = 0; k < 4; ++k) {
    Neumaier a;
    for (size_t q = 0; q < rows; ++q) {
      a.add(part[q * width + k]);
      if (many) a.add(part[q * width + 4 + k]);
    }
    sum[k] = a.val();
  }
  return MPC_OK;
}

// A sum's digits under bin `anchor`, rounded once.
double exact_value(__int128 (&d)[3], int anchor) {
  if (anchor < 0) return 0.0;
  if (anchor >= kObsBad) return NAN;
  // carries: d[2] 2^80 + low, 0 <= low < 2^80, in units of 2^(40 anchor - 1103)
  constexpr __int128 kMask = ((__int128)1 << 40) - 1;
  d[1] += d[0] >> 40;
  d[2] += d[1] >> 40;
  unsigned __int128 low = (unsigned __int128)((d[1] & kMask) << 40 | (d[0] & kMask));
  __int128 high = d[2];
  const bool neg = high < 0;
  if (neg) {
    high = -high - (low != 0 ? 1 : 0);
    if (low != 0) low = ((unsigned __int128)1 << 80) - low;
  }
  // |high| < 2^73: 55 bits and more with a sticky one decide the rounding
  double x;
  if (high == 0) {
    x = ldexp((double)low, 40 * anchor - 1103);
  } else {
    const unsigned __int128 rest = low & (((unsigned __int128)1 << 26) - 1);
    x = ldexp((double)((unsigned __int128)high << 54 | low >> 26 | (rest != 0 ? 1u : 0u)),
              40 * anchor - 1103 + 26);
  }
  return neg ? -x : x;
}

// Momentum and energy (NV = 4) or relative energy (NV = 1) of a box in sums that do
// not depend on the order of its slots.
template <int NV>
int sum_exact(mpc_sim* s, int32_t box, const Vec3& vmean, double* sum) {
  ObsResult<NV> r;
  HIPCHK(s, launch_obs_exact(s->dev, s->L, (uint32_t)box, s->boxes[box].np, s->cur, vmean, &r));
  HIPCHK(s, hipStreamSynchronize(s->L.stream));
  for (int k = 0; k < NV; ++k) {
    __int128 d[3] = {0, 0, 0};
    int top = -1;
    if (!r.rows) {
      top = r.total[k].anchor;
      for (int j = 0; j < 3; ++j) d[j] = (__int128)r.total[k].hi[j] << 64 | r.total[k].lo[j];
    }
    for (uint32_t q = 0; q < r.rows; ++q) top = std::max(top, r.row[q].anchor[k]);
    for (uint32_t q = 0; q < r.rows; ++q) {
      const int by = top - r.row[q].anchor[k];
      for (int j = 0; j + by < 3; ++j) d[j] += r.row[q].d[k][j + by];
    }
    sum[k] = exact_value(d, top);
  }
  return MPC_OK;
}

// Whether FP64 momentum and energy of a step's slots are added in the order of
// the cells: tiles of at least 16 particles on average, as all but thin sparse
// boxes have (1 x 1000 x 1000 at 0.5 per cell: 0.68 ms in order, 0.10 free of
// it), and no more of them than one launch takes (2^32 threads).
bool obs_ordered(const mpc_sim* s, const BoxDev& B) {
  const uint64_t l0 = (uint64_t)B.L[0], to = obs_tile_cells(B.density);
  const uint64_t tiles = (uint64_t)B.L[1] * (uint64_t)B.nlz * ((l0 + to - 1) / to);
  return s->form == MPC_FP64 && B.density * (double)std::min(to, l0) >= 16.0 &&
         tiles < ((uint64_t)1 << 32) / 64;
}

// Momentum P[3], kinetic energy E and relative kinetic energy K of one box.
int obs_box(mpc_sim* s, int32_t box, double* P, double* E, double* K) {
  const BoxDev& B = s->boxes[box];
  const uint32_t pb0 = s->box_pb0[box], npb = s->box_pb0[box + 1] - pb0;
  // The slots of a step depend on the order in which runs were appended.  FP64
  // momentum and energy are added in an order of the particles' cells then (a
  // total momentum is a sum of rounding errors, of which every digit depends on
  // that order), all other sums are free of the order.
  const char slots = s->slots[box];
  double sum[4];
  int rc;
  if (slots == kSlotsCaller || (slots == kSlotsStep && obs_ordered(s, B))) {
    uint32_t* order = nullptr;
    if (slots == kSlotsStep) {
      // the chains of the buffer that the next step writes are free until then
      order = s->dev.rnext[s->cur ^ 1u];
      s->binning_ready = false;
      HIPCHK(s, launch_obs_order(s->dev, s->L, (uint32_t)box, (uint32_t)B.L[1] * (uint32_t)B.nlz,
                                 (uint32_t)B.L[0], s->cur, obs_tile_cells(B.density), order));
    }
    HIPCHK(s, launch_obs_pass1(s->dev, s->L, pb0, npb, s->cur, order));
    rc = sum_partials(s, pb0, npb, sum);
  } else {
    rc = sum_exact<4>(s, box, Vec3{}, sum);
  }
  if (rc) return rc;
  const double M = (double)B.np * B.mass;
  Vec3 vm;
  for (int k = 0; k < 3; ++k) {
    P[k] = sum[k];
    vm.v[k] = P[k] / M;
  }
  *E = sum[3];
  return sum_exact<1>(s, box, vm, K);
}

}  // namespace

extern "C" {

const char* mpc_strerror(int code) {
  switch (code) {
    case MPC_OK: return "ok";
    case MPC_EINVAL: return "invalid argument";
    case MPC_ENOSPACE: return "workspace too small";
    case MPC_ERANGE: return "size out of range";
    case MPC_EHIP: return "HIP runtime error";
    case MPC_ESTATE: return "invalid particle state";
    default: return "unknown error";
  }
}

const char* mpc_last_error(mpc_sim* s) { return s ? s->err.c_str() : ""; }

int mpc_workspace_bytes(const mpc_params* p, int32_t nbox, size_t* bytes) {
  if (!bytes) return MPC_EINVAL;
  Plan P;
  std::string why;
  const int rc = make_plan(p, nbox, P, &why);
  if (rc) return rc;
  *bytes = P.total;
  return MPC_OK;
}

int mpc_create(const mpc_params* p, int32_t nbox, void* workspace, size_t bytes,
               void* hip_stream, mpc_sim** out) {
  if (!out) return MPC_EINVAL;
  *out = nullptr;
  mpc_sim* s = new mpc_sim();
  std::string why;
  int rc = make_plan(p, nbox, s->plan, &why);
  if (rc) {
    delete s;
    return rc;
  }
  if (!workspace || bytes < s->plan.total || ((uintptr_t)workspace & 255)) {
    delete s;
    return workspace && bytes >= s->plan.total ? MPC_EINVAL : MPC_ENOSPACE;
  }
  s->params.assign(p, p + nbox);
  s->form = p[0].form;
  s->R = p[0].reorder_every;
  const Plan& P = s->plan;
  char* ws = s->ws = (char*)workspace;
  for (int b = 0; b < 2; ++b) {
    s->dev.S[b].rec = ws + P.off_rec[b];
    s->dev.S[b].id = P.split ? &((RecSplit*)(ws + P.off_rec[b]))->id : (uint32_t*)(ws + P.off_id[b]);
    s->dev.S[b].id_stride = P.split ? (uint32_t)(sizeof(RecSplit) / 4) : 1u;
  }
  s->dev.key = (uint32_t*)(ws + P.off_key);
  s->dev.perm = (uint32_t*)(ws + P.off_perm);
  s->dev.rank = (uint16_t*)(ws + P.off_rank);
  s->dev.hist = (uint32_t*)(ws + P.off_hist);
  s->dev.offset = (uint32_t*)(ws + P.off_offset);
  s->dev.scan_blk = (uint32_t*)(ws + P.off_scan);
  for (int k = 0; k < 3; ++k) s->dev.tcnt[k] = (unsigned long long*)(ws + P.off_tcnt[k]);
  for (int k = 0; k < 2; ++k) {
    s->dev.runs[k] = (Run*)(ws + P.off_runs[k]);
    s->dev.rhead[k] = (uint32_t*)(ws + P.off_rhead[k]);
    s->dev.rnext[k] = (uint32_t*)(ws + P.off_rnext[k]);
  }
  s->dev.toff = (uint32_t*)(ws + P.off_toff);
  s->dev.tblk = (uint32_t*)(ws + P.off_tblk);
  s->dev.ctrl = (Ctrl*)(ws + P.off_ctrl);
  s->dev.boxes = (BoxDev*)(ws + P.off_boxes);
  s->dev.tiles = (Tile*)(ws + P.off_tiles);
  s->dev.pblocks = (PBlock*)(ws + P.off_pblocks);
  s->dev.partials = (double*)(ws + P.off_partials);
  s->dev.obs = (double*)(ws + P.off_obs);
  s->dev.ntot = (uint32_t)P.ntot;
  s->vmean = (double*)(ws + P.off_vmean);
  s->dev.drawb = P.drawb;
  for (int k = 0; k < 2; ++k) {
    s->dev.bstep[k] = (BoxStep*)(ws + P.off_bstep[k]);
    s->dev.draws[k] = (double4*)(ws + P.off_draws[k]);
    s->dev.least[k] = (p[0].flags & MPC_MBS) ? (uint32_t*)(ws + P.off_least[k]) : nullptr;
    s->dev.later[k] = (p[0].flags & MPC_MBS) ? (Attempt*)(ws + P.off_later[k]) : nullptr;
    s->dev.phs[k] = (p[0].flags & MPC_WALLS_Z) ? (PhantomSums*)(ws + P.off_phs[k]) : nullptr;
  }

  // boxes
  uint64_t pb = 0, cb = 0, wcb = 0;
  s->box_pb0.push_back(0);
  for (int32_t b = 0; b < nbox; ++b) {
    const mpc_params& q = p[b];
    BoxDev B{};
    for (int k = 0; k < 3; ++k) {
      B.L[k] = q.L[k];
      B.Ld[k] = (double)q.L[k];
      B.Lf[k] = (float)q.L[k];
    }
    B.nlz = P.box[b].nlz;
    B.pbase = (uint32_t)pb;
    B.np = (uint32_t)P.box[b].n;
    B.cbase = (uint32_t)cb;
    B.nc = (uint32_t)P.box[b].ncell;
    B.key_lo = (uint32_t)(q.seed & 0xffffffffu);
    B.key_hi = (uint32_t)(q.seed >> 32);
    B.walls = (q.flags & MPC_WALLS_Z) ? 1u : 0u;
    B.mbs = (q.flags & MPC_MBS) ? 1u : 0u;
    // internal units: lengths in cells, so velocities / a, energies / a^2
    B.h = q.dt;
    B.hf = (float)q.dt;
    B.ca = cos(q.alpha);
    B.sa = sin(q.alpha);
    B.omc = 1.0 - B.ca;
    B.kT = q.kT / (q.a * q.a);
    B.mass = q.mass;
    B.density = q.density;
    B.sd = sqrt(B.kT / q.mass);
    B.grav = (q.g[0] != 0.0 || q.g[1] != 0.0 || q.g[2] != 0.0) ? 1u : 0u;
    B.wcbase = (uint32_t)wcb;
    if (B.walls) wcb += 2ull * (uint64_t)q.L[0] * (uint64_t)q.L[1];
    for (int k = 0; k < 3; ++k) B.gh[k] = (q.g[k] / q.a) * q.dt;
    B.slip = (B.walls && (q.flags & MPC_SLIP)) ? 1u : 0u;
    B.uw = q.wall_u / q.a;
    B.uwf = (float)B.uw;
    B.le = (!B.walls && q.le_u != 0.0) ? 1u : 0u;
    if (B.le) s->L.le = 1;
    B.leu = q.le_u / q.a;
    B.leuf = (float)B.leu;
    s->boxes.push_back(B);
    for (uint64_t p0 = 0; p0 < P.box[b].n; p0 += kPartBlock)
      s->pblocks.push_back(PBlock{(uint32_t)b, (uint32_t)(pb + p0)});
    s->box_pb0.push_back((uint32_t)s->pblocks.size());
    pb += P.box[b].n;
    cb += P.box[b].ncell;
  }

  s->L.form = s->form;
  s->L.round_phantoms = s->form == MPC_SPLIT32 ? 1 : 0;
  s->L.wcells = (uint32_t)wcb;
  s->L.walls = (p[0].flags & MPC_WALLS_Z) ? 1 : 0;
  s->L.mbs = (p[0].flags & MPC_MBS) ? 1 : 0;
  s->L.amc = (p[0].flags & MPC_AMC) ? 1 : 0;
  s->L.fixed = (p[0].flags & MPC_FIXED_SUMS) ? 1 : 0;
  s->L.nbox = (uint32_t)nbox;
  s->L.ntot = P.ntot;
  s->L.ctot = P.ctot;
  s->L.nscan = P.nscan;
  s->L.npblocks = (uint32_t)s->pblocks.size();
  s->L.stream = (hipStream_t)hip_stream;
  s->L.xcd_remap = 1;

  int dev = 0;
  hipDeviceProp_t prop;
  hipPointerAttribute_t attr;
  if (hipGetDevice(&dev) == hipSuccess) s->device = dev;
  if (hipPointerGetAttributes(&attr, workspace) == hipSuccess) {
    s->device = attr.device;
  } else {
    (void)hipGetLastError();  // static scratch: of the current device
  }
  if (hipGetDeviceProperties(&prop, s->device) == hipSuccess)
    s->num_cu = prop.multiProcessorCount;
  s->occupancy = 2;
  if (collide_occupancy(s->L, &s->occupancy) != hipSuccess ||
      s->occupancy < 1)
    s->occupancy = 1;
  build_tiles(s);

  auto fail = [&](int code) {
    delete s;
    return code;
  };
  if ((rc = upload_tables(s))) return fail(rc);
  if (hipMemcpyAsync(s->dev.pblocks, s->pblocks.data(), sizeof(PBlock) * s->pblocks.size(),
                     hipMemcpyHostToDevice, s->L.stream) != hipSuccess ||
      launch_set_ctrl(s->dev, s->L, 0, 0, s->R, 1) != hipSuccess ||
      hipStreamSynchronize(s->L.stream) != hipSuccess)
    return fail(MPC_EHIP);
  *out = s;
  return MPC_OK;
}

int mpc_destroy(mpc_sim* s) {
  if (!s) return MPC_EINVAL;
  (void)hipStreamSynchronize(s->L.stream);
  drop_graph(s);
  if (s->capture_stream) (void)hipStreamDestroy(s->capture_stream);
  if (s->stage) (void)hipFree(s->stage);
  delete s;
  return MPC_OK;
}

int mpc_set_graph(mpc_sim* s, int32_t enable) {
  if (!s || enable < 0 || enable > kMaxGraphSteps) return MPC_EINVAL;
  if (enable >= 1 && enable != s->graph_steps) {
    HIPCHK(s, hipStreamSynchronize(s->L.stream));
    int rc = drop_graph(s);
    if (rc) return rc;
    s->graph_steps = enable;
  }
  s->use_graph = enable != 0;
  return MPC_OK;
}

int mpc_set_tiling(mpc_sim* s, int32_t tile_cells, int32_t grid, int32_t yblock,
                   int32_t order) {
  if (!s) return MPC_EINVAL;
  if (tile_cells != 0 && (tile_cells < kMinTileCells || tile_cells > kTileMaxCells))
    return MPC_EINVAL;
  if (grid < 0 || yblock < 0 || yblock > 4096 || order < 0 || order > 1) return MPC_EINVAL;
  HIPCHK(s, hipStreamSynchronize(s->L.stream));
  s->tile_override = tile_cells;
  s->grid_override = grid;
  s->yblock = yblock ? yblock : 8;
  s->order = order;
  build_tiles(s);
  int rc = drop_graph(s);
  if (rc) return rc;
  return upload_tables(s);
}

int mpc_get_tiling(mpc_sim* s, int32_t* tile_cells, int32_t* grid, int32_t* yblock,
                   int32_t* order, int64_t* ntiles) {
  if (!s) return MPC_EINVAL;
  if (tile_cells) *tile_cells = s->tile_override;
  if (grid) *grid = (int32_t)s->L.collide_grid;
  if (yblock) *yblock = s->yblock;
  if (order) *order = s->order;
  if (ntiles) *ntiles = (int64_t)s->L.ntiles;
  return MPC_OK;
}

int mpc_step(mpc_sim* s, int64_t nsteps) {
  if (!s || nsteps < 0) return MPC_EINVAL;
  if (nsteps == 0) return MPC_OK;
  int rc = ensure_keys(s);
  if (rc) return rc;
  int64_t k = 0;
  const int64_t chunk = graph_chunk(s);
  if (s->use_graph && nsteps >= chunk) {
    if ((rc = capture_graph(s))) return rc;
    for (; k + chunk <= nsteps; k += chunk) HIPCHK(s, hipGraphLaunch(s->gexec, s->L.stream));
  }
  while (k < nsteps) {
    const int64_t n = std::min<int64_t>(nsteps - k, kMaxGraphSteps);
    HIPCHK(s, enqueue_steps(s, s->L.stream, n));
    k += n;
  }
  advance_mirror(s, nsteps);
  s->have_binning = true;
  s->binning_ready = false;
  s->slots.assign(s->boxes.size(), kSlotsStep);
  return MPC_OK;
}

int mpc_step_profiled(mpc_sim* s, int64_t nsteps, mpc_kernel_times* acc) {
  if (!s || nsteps < 0 || !acc) return MPC_EINVAL;
  if (nsteps == 0) return MPC_OK;
  hipStream_t st = s->L.stream;
  std::vector<hipEvent_t> ev;
  auto mark = [&]() -> hipError_t {
    hipEvent_t e;
    hipError_t r = hipEventCreate(&e);
    if (r != hipSuccess) return r;
    ev.push_back(e);
    return hipEventRecord(e, st);
  };
  int kinds_prologue = 0;
  HIPCHK(s, mark());
  if (!s->keys_valid) {
    int rc = ensure_keys(s);
    if (rc) return rc;
    HIPCHK(s, mark());
    kinds_prologue = 1;
  }
  Launch l = s->L;
  for (int64_t k = 0; k < nsteps; ++k) {
    l.seq = (uint32_t)(k % kMaxGraphSteps);
    HIPCHK(s, launch_prefix(s->dev, l));
    HIPCHK(s, mark());
    HIPCHK(s, launch_collide(s->dev, l));
    if (k + 1 == nsteps || l.seq + 1 == (uint32_t)kMaxGraphSteps)
      HIPCHK(s, launch_advance(s->dev, l, l.seq + 1));
    HIPCHK(s, mark());
  }
  HIPCHK(s, hipStreamSynchronize(st));
  size_t e = 0;
  auto span = [&]() {
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, ev[e], ev[e + 1]);
    ++e;
    return (double)ms;
  };
  if (kinds_prologue) {
    acc->prologue_ms += span();
    acc->prologue_launches += 1;
  }
  for (int64_t k = 0; k < nsteps; ++k) {
    acc->scan_ms += span();
    acc->collide_ms += span();
    acc->scan_launches += 1;
    acc->collide_launches += 1;
  }
  for (hipEvent_t x : ev) (void)hipEventDestroy(x);
  advance_mirror(s, nsteps);
  s->have_binning = true;
  s->binning_ready = false;
  s->slots.assign(s->boxes.size(), kSlotsStep);
  return MPC_OK;
}

int mpc_sync(mpc_sim* s) {
  if (!s) return MPC_EINVAL;
  HIPCHK(s, hipStreamSynchronize(s->L.stream));
  return check_sticky(s);
}

int mpc_box_info(mpc_sim* s, int32_t box, int64_t* n, int64_t* ncell) {
  if (!s || box < 0 || box >= (int32_t)s->boxes.size()) return MPC_EINVAL;
  if (n) *n = (int64_t)s->boxes[box].np;
  if (ncell) *ncell = (int64_t)s->boxes[box].nc;
  return MPC_OK;
}

int mpc_get_step(mpc_sim* s, uint64_t* step) {
  if (!s || !step) return MPC_EINVAL;
  *step = s->step;
  return MPC_OK;
}

int mpc_set_step(mpc_sim* s, uint64_t step) {
  if (!s) return MPC_EINVAL;
  s->step = step;
  s->keys_valid = false;
  s->have_binning = false;
  s->binning_ready = false;
  HIPCHK(s, launch_set_ctrl(s->dev, s->L, s->step, s->cur, s->R, 0));
  HIPCHK(s, hipStreamSynchronize(s->L.stream));
  return MPC_OK;
}

int mpc_init_state(mpc_sim* s, uint64_t init_seed) {
  if (!s) return MPC_EINVAL;
  HIPCHK(s, launch_set_ctrl(s->dev, s->L, s->step, s->cur, s->R, 1));
  HIPCHK(s, launch_init_state(s->dev, s->L, init_seed));
  // mean of each box
  const size_t nbox = s->boxes.size();
  const size_t npb = s->pblocks.size();
  std::vector<double> part(4 * npb);
  HIPCHK(s, launch_obs_pass1(s->dev, s->L, 0, (uint32_t)npb, s->cur, nullptr));
  HIPCHK(s, hipMemcpyAsync(part.data(), s->dev.partials, sizeof(double) * 4 * npb,
                           hipMemcpyDeviceToHost, s->L.stream));
  HIPCHK(s, hipStreamSynchronize(s->L.stream));
  std::vector<double> vm(3 * nbox);
  for (size_t b = 0; b < nbox; ++b) {
    Neumaier a[3];
    for (uint32_t q = s->box_pb0[b]; q < s->box_pb0[b + 1]; ++q)
      for (int k = 0; k < 3; ++k) a[k].add(part[4 * q + k]);
    const double M = (double)s->boxes[b].np * s->boxes[b].mass;
    for (int k = 0; k < 3; ++k) vm[3 * b + k] = a[k].val() / M;
  }
  HIPCHK(s, hipMemcpyAsync(s->vmean, vm.data(), sizeof(double) * 3 * nbox, hipMemcpyHostToDevice,
                           s->L.stream));
  HIPCHK(s, launch_remove_mean(s->dev, s->L, s->vmean));
  HIPCHK(s, hipStreamSynchronize(s->L.stream));
  s->keys_valid = false;
  s->have_binning = false;
  s->binning_ready = false;
  s->slots.assign(s->boxes.size(), kSlotsCaller);
  return MPC_OK;
}

int mpc_set_state(mpc_sim* s, int32_t box, const double* x, const double* v, int64_t n) {
  if (!s || box < 0 || box >= (int32_t)s->boxes.size() || !x || !v) return MPC_EINVAL;
  const BoxDev& B = s->boxes[box];
  if (n != (int64_t)B.np) {
    s->err = "n differs from the box's particle count";
    return MPC_EINVAL;
  }
  const double a = s->params[box].a;
  const OnDevice on(s);
  HIPCHK(s, hipStreamSynchronize(s->L.stream));
  Stage st;
  get_stage(s, n, &st);
  const int64_t chunk = std::min(n, st.cap);
  if (chunk < 1) return hip_fail(s, hipErrorOutOfMemory, "staging");
  HIPCHK(s, launch_zero_u32(st.flag, 1, s->L.stream));
  // everything is checked before anything is changed: one chunk stays on the
  // device in between, several are copied twice
  for (int pass = 0; pass < 2; ++pass) {
    for (int64_t i0 = 0; i0 < n; i0 += chunk) {
      const int64_t m = std::min(chunk, n - i0);
      double* dx = st.data;
      double* dv = st.data + 3 * m;
      int rc;
      if ((pass == 0 || chunk < n) && (rc = stage_copy(s, dx, dv, x, v, n, i0, m, true))) return rc;
      HIPCHK(s, launch_state_in(s->dev, s->L, s->dev.S[s->cur], (uint32_t)box, (uint32_t)i0, dx, dv,
                                (uint32_t)m, a, pass == 0 ? st.flag : nullptr));
    }
    if (pass == 0) {
      uint32_t bad = 0;
      HIPCHK(s, hipMemcpyAsync(&bad, st.flag, sizeof bad, hipMemcpyDeviceToHost, s->L.stream));
      HIPCHK(s, hipStreamSynchronize(s->L.stream));
      if (bad) {
        s->err = "position outside the box or non-finite velocity";
        return MPC_EINVAL;
      }
    }
  }
  HIPCHK(s, launch_set_ctrl(s->dev, s->L, s->step, s->cur, s->R, 1));
  HIPCHK(s, hipStreamSynchronize(s->L.stream));
  s->keys_valid = false;
  s->have_binning = false;
  s->binning_ready = false;
  s->slots[box] = kSlotsCaller;
  return MPC_OK;
}

int mpc_get_state(mpc_sim* s, int32_t box, double* x, double* v, int64_t n) {
  if (!s || box < 0 || box >= (int32_t)s->boxes.size() || !x || !v) return MPC_EINVAL;
  const BoxDev& B = s->boxes[box];
  if (n != (int64_t)B.np) return MPC_EINVAL;
  int rc = mpc_sync(s);
  if (rc) return rc;
  const double a = s->params[box].a;
  const OnDevice on(s);
  Stage st;
  get_stage(s, n, &st);
  const int64_t chunk = std::min(n, st.cap);
  if (chunk < 1) return hip_fail(s, hipErrorOutOfMemory, "staging");
  for (int64_t i0 = 0; i0 < n; i0 += chunk) {
    const int64_t m = std::min(chunk, n - i0);
    double* dx = st.data;
    double* dv = st.data + 3 * m;
    HIPCHK(s, launch_state_out(s->L, s->dev.S[s->cur], B.pbase, B.np, (uint32_t)i0, dx, dv,
                               (uint32_t)m, a, st.flag));
    uint32_t bad = 0;
    const size_t arr = sizeof(double) * 3 * (size_t)m;
    if (m == n && 2 * arr <= kSmallCopy) {  // flag and arrays lie one after the other
      std::vector<char> all(256 + 2 * arr);
      HIPCHK(s, hipMemcpyAsync(all.data(), st.flag, all.size(), hipMemcpyDeviceToHost, s->L.stream));
      HIPCHK(s, hipStreamSynchronize(s->L.stream));
      memcpy(&bad, all.data(), sizeof bad);
      memcpy(x, all.data() + 256, arr);
      memcpy(v, all.data() + 256 + arr, arr);
    } else {
      if ((rc = stage_copy(s, dx, dv, x, v, n, i0, m, false))) return rc;
      HIPCHK(s, hipMemcpyAsync(&bad, st.flag, sizeof bad, hipMemcpyDeviceToHost, s->L.stream));
      HIPCHK(s, hipStreamSynchronize(s->L.stream));
    }
    if (bad) {
      s->err = "logical particle indices are not a permutation";
      return MPC_ESTATE;
    }
  }
  return MPC_OK;
}

int mpc_get_particles(mpc_sim* s, int32_t box, const int64_t* idx, int64_t m, double* x,
                      double* v) {
  if (!s || box < 0 || box >= (int32_t)s->boxes.size() || m < 0) return MPC_EINVAL;
  if (m > 0 && (!idx || !x || !v)) return MPC_EINVAL;
  const BoxDev& B = s->boxes[box];
  if (m > (int64_t)kMaxIndex) {
    s->err = "more than 2^31 - 1 particles requested";
    return MPC_EINVAL;
  }
  std::vector<uint32_t> lidx((size_t)m);
  for (int64_t k = 0; k < m; ++k) {
    if (idx[k] < 0 || idx[k] >= (int64_t)B.np) {
      s->err = "particle index outside the box";
      return MPC_EINVAL;
    }
    lidx[k] = (uint32_t)idx[k];
  }
  int rc = mpc_sync(s);
  if (rc || m == 0) return rc;
  const OnDevice on(s);
  const StatePtrs& S = s->dev.S[s->cur];
  // one allocation: the sample's states, indices, and the table that finds
  // their slots (see k_sample_find)
  const uint32_t mask = sample_table_mask((uint64_t)m, B.np);
  const size_t o_sel = align256(sizeof(double) * 6 * (size_t)m);
  const size_t o_tab = o_sel + align256(sizeof(uint32_t) * (size_t)m);
  const size_t n_tab = mask ? 2 * ((size_t)mask + 1) : (size_t)B.np;
  char* dbuf = nullptr;
  std::vector<double> out(6 * (size_t)m);
  hipError_t e = hipSuccess;
  const char* where = "";
  do {
    where = "hipMalloc (sample)";
    if ((e = hipMalloc(&dbuf, o_tab + sizeof(uint32_t) * n_tab)) != hipSuccess) break;
    double* dout = (double*)dbuf;
    uint32_t* dl = (uint32_t*)(dbuf + o_sel);
    uint32_t* tab = (uint32_t*)(dbuf + o_tab);
    where = "copy of the sample indices";
    if ((e = hipMemcpyAsync(dl, lidx.data(), sizeof(uint32_t) * (size_t)m,
                            hipMemcpyHostToDevice, s->L.stream)) != hipSuccess)
      break;
    where = "gather kernels";
    if ((e = launch_gather_particles(s->dev, s->L, S, mask ? nullptr : tab, mask ? tab : nullptr,
                                     mask, B.pbase, B.np, dl, (uint32_t)m, dout)) != hipSuccess)
      break;
    where = "copy of the sample";
    if ((e = hipMemcpyAsync(out.data(), dout, sizeof(double) * 6 * (size_t)m,
                            hipMemcpyDeviceToHost, s->L.stream)) != hipSuccess)
      break;
    where = "hipStreamSynchronize";
    e = hipStreamSynchronize(s->L.stream);
  } while (false);
  if (dbuf) (void)hipFree(dbuf);
  if (e != hipSuccess) return hip_fail(s, e, where);
  const double a = s->params[box].a;
  for (int64_t k = 0; k < m; ++k) {
    if (isnan(out[k])) {
      s->err = "logical particle indices are not a permutation";
      return MPC_ESTATE;
    }
    for (int c = 0; c < 3; ++c) {
      x[c * m + k] = out[(size_t)c * m + k] * a;
      v[c * m + k] = out[(size_t)(3 + c) * m + k] * a;
    }
  }
  return MPC_OK;
}

int mpc_observables(mpc_sim* s, int32_t box, mpc_obs* out) {
  if (!s || !out || box < 0 || box >= (int32_t)s->boxes.size()) return MPC_EINVAL;
  int rc = mpc_sync(s);
  if (rc) return rc;
  double P[3], E, K;
  if ((rc = obs_box(s, box, P, &E, &K))) return rc;
  const BoxDev& B = s->boxes[box];
  const double a = s->params[box].a;
  out->step = s->step;
  out->n = B.np;
  for (int k = 0; k < 3; ++k) out->P[k] = P[k] * a;
  out->E = E * a * a;
  out->T = B.np > 1 ? K / (3.0 * (double)(B.np - 1)) * a * a : 0.0;
  out->mass_total = (double)B.np * B.mass;
  if (!isfinite(out->E) || !isfinite(out->P[0]) || !isfinite(out->P[1]) || !isfinite(out->P[2])) {
    s->err = "non-finite observables";
    return MPC_ESTATE;
  }
  return MPC_OK;
}

int mpc_get_binning(mpc_sim* s, int32_t box, uint32_t* key, uint32_t* perm, uint32_t* offset) {
  if (!s || box < 0 || box >= (int32_t)s->boxes.size()) return MPC_EINVAL;
  if (!s->have_binning) {
    s->err = "no step since the state was set";
    return MPC_EINVAL;
  }
  int rc = mpc_sync(s);
  if (rc) return rc;
  // the last step read the buffer that is not current; its ids give the
  // logical order before that step
  const StatePtrs& Sin = s->dev.S[s->cur ^ 1u];
  if (!s->binning_ready) {
    // the export takes the memory of the run lists
    if (!s->plan.own_export) s->keys_valid = false;
    HIPCHK(s, launch_binning(s->dev, s->L, Sin, s->step - 1));
    HIPCHK(s, launch_canon_perm(s->dev, s->L, Sin));
    s->binning_ready = true;
  }
  const BoxDev& B = s->boxes[box];
  std::vector<uint32_t> off(B.nc + 1), pm(B.np), lid(B.np);
  if ((rc = copy_d2h(s, s->dev.offset, B.cbase, off))) return rc;
  if ((rc = copy_d2h(s, s->dev.perm, B.pbase, pm))) return rc;
  HIPCHK(s, hipStreamSynchronize(s->L.stream));
  if ((rc = read_ids(s, Sin, B.pbase, lid))) return rc;
  const uint32_t o0 = off[0];
  for (auto& o : off) o -= o0;
  for (auto& q : pm) {
    if (q < B.pbase || q - B.pbase >= B.np) {
      s->err = "permutation entry outside the box";
      return MPC_ESTATE;
    }
    q = lid[q - B.pbase] - B.pbase;
    if (q >= B.np) {
      s->err = "logical particle index outside the box";
      return MPC_ESTATE;
    }
  }
  if (offset) memcpy(offset, off.data(), sizeof(uint32_t) * off.size());
  if (perm) memcpy(perm, pm.data(), sizeof(uint32_t) * pm.size());
  if (key) {
    for (uint32_t c = 0; c < B.nc; ++c)
      for (uint32_t j = off[c]; j < off[c + 1]; ++j) key[pm[j]] = c;
  }
  return MPC_OK;
}

int mpc_autotune(mpc_sim* s, int32_t trial_steps, int32_t* tile_cells, int32_t* grid) {
  if (!s || trial_steps < 1 || trial_steps > 1000) return MPC_EINVAL;
  int rc = mpc_sync(s);
  if (rc) return rc;
  const OnDevice on(s);
  const Plan& P = s->plan;
  hipStream_t st = s->L.stream;
  const uint64_t step0 = s->step;
  const uint32_t cur0 = s->cur;
  std::vector<char> slots0 = s->slots;
  for (char& o : slots0)
    if (o == kSlotsStep) o = kSlotsOther;
  const int T0 = s->tile_override, g0 = s->grid_override, y0 = s->yblock, o0 = s->order;
  // the arrays of the current state buffer, backed up on the device (or in
  // host memory if the device has no room) and restored before every trial
  std::vector<std::pair<void*, size_t>> arrs;
  const StatePtrs& S = s->dev.S[cur0];
  arrs.push_back({S.rec, P.rec * P.ntot});
  if (!P.split) arrs.push_back({S.id, 4 * P.ntot});
  size_t total = 0;
  for (auto& a : arrs) total += align256(a.second);
  void* backup = nullptr;
  bool on_host = false;
  if (hipMalloc(&backup, total) != hipSuccess) {
    (void)hipGetLastError();
    backup = nullptr;
    if (hipHostMalloc(&backup, total, hipHostMallocDefault) != hipSuccess) {
      s->err = "autotune: no memory for the state backup";
      return MPC_EHIP;
    }
    on_host = true;
  }
  auto copy_all = [&](bool save) -> hipError_t {
    size_t o = 0;
    for (auto& a : arrs) {
      char* bk = (char*)backup + o;
      hipError_t e = save ? hipMemcpyAsync(bk, a.first, a.second, hipMemcpyDefault, st)
                          : hipMemcpyAsync(a.first, bk, a.second, hipMemcpyDefault, st);
      if (e != hipSuccess) return e;
      o += align256(a.second);
    }
    return hipStreamSynchronize(st);
  };
  auto release = [&]() {
    if (on_host) {
      (void)hipHostFree(backup);
    } else {
      (void)hipFree(backup);
    }
  };
  auto restore = [&]() -> int {
    hipError_t e = copy_all(false);
    if (e != hipSuccess) return hip_fail(s, e, "autotune restore");
    s->cur = cur0;
    s->step = step0;
    s->keys_valid = false;
    s->have_binning = false;
    s->binning_ready = false;
    s->slots = slots0;
    HIPCHK(s, launch_set_ctrl(s->dev, s->L, step0, cur0, s->R, 1));
    return MPC_OK;
  };
  hipError_t e0 = copy_all(true);
  if (e0 != hipSuccess) {
    release();
    return hip_fail(s, e0, "autotune backup");
  }
  // one trial: set the tiling, one untimed step (binning prologue), then
  // trial_steps timed steps; returns the fastest step in milliseconds (the
  // minimum is robust to a step slowed by other work on the device)
  std::vector<hipEvent_t> ev((size_t)trial_steps + 1, nullptr);
  auto trial = [&](int T, int g, int yb, int ord, double* ms) -> int {
    int r = mpc_set_tiling(s, T, g, yb, ord);
    if (r) return r;
    if ((r = restore())) return r;
    if ((r = ensure_keys(s))) return r;
    HIPCHK(s, enqueue_steps(s, st, 1));
    advance_mirror(s, 1);
    HIPCHK(s, hipEventRecord(ev[0], st));
    for (int32_t k = 0; k < trial_steps; ++k) {
      HIPCHK(s, enqueue_steps(s, st, 1));
      HIPCHK(s, hipEventRecord(ev[(size_t)k + 1], st));
    }
    HIPCHK(s, hipEventSynchronize(ev[(size_t)trial_steps]));
    advance_mirror(s, trial_steps);
    double m = 1e300;
    for (int32_t k = 0; k < trial_steps; ++k) {
      float f = 0.f;
      HIPCHK(s, hipEventElapsedTime(&f, ev[(size_t)k], ev[(size_t)k + 1]));
      m = std::min(m, (double)f);
    }
    *ms = m;
    return check_sticky(s);
  };
  rc = MPC_OK;
  for (hipEvent_t& x : ev)
    if (!rc && hipEventCreate(&x) != hipSuccess) rc = MPC_EHIP;
  int bestT = T0, bestG = g0, bestY = y0, bestO = o0;
  double best = 1e300;
  // coordinate search: tile size, then the persistent grid, then the row block
  const int Ts[] = {0, 8, 12, 16, 20, 22, 24, 28, 32};
  // grids: the default (0) and multiples of the resident workgroups
  const int full = s->num_cu * std::max(1, s->occupancy);
  const int gs[] = {0, 2 * full, 4 * full, 16 * full, 32 * full, 64 * full};
  const int ys[] = {8, 4, 16};
  for (int T : Ts) {
    double ms;
    if (rc || (rc = trial(T, 0, 8, 0, &ms))) break;
    if (ms < best) best = ms, bestT = T, bestG = 0, bestY = 8, bestO = 0;
  }
  for (int g : gs) {
    double ms;
    if (rc || g == 0) continue;
    if ((rc = trial(bestT, (g + 7) / 8 * 8, bestY, 0, &ms))) break;
    if (ms < best) best = ms, bestG = (g + 7) / 8 * 8;
  }
  for (int yb : ys) {
    double ms;
    if (rc || yb == 8) continue;
    if ((rc = trial(bestT, bestG, yb, 0, &ms))) break;
    if (ms < best) best = ms, bestY = yb;
  }
  // then the x-segment-major order with each row block
  for (int yb : ys) {
    double ms;
    if (rc) break;
    if ((rc = trial(bestT, bestG, yb, 1, &ms))) break;
    if (ms < best) best = ms, bestY = yb, bestO = 1;
  }
  for (hipEvent_t x : ev)
    if (x) (void)hipEventDestroy(x);
  const std::string why = s->err;
  int rc2 = mpc_set_tiling(s, rc ? T0 : bestT, rc ? g0 : bestG, rc ? y0 : bestY, rc ? o0 : bestO);
  int rc3 = restore();
  release();
  if (rc) {
    s->err = "autotune: " + why;
    return rc;
  }
  if (rc2) return rc2;
  if (rc3) return rc3;
  if (tile_cells) *tile_cells = bestT;
  if (grid) *grid = (int32_t)s->L.collide_grid;
  return MPC_OK;
}

int mpc_run_noalloc(const mpc_params* p, double* x, double* v, int64_t n, uint64_t step,
                    int64_t nsteps, void* hip_stream) {
  if (!p || !x || !v || n < 1 || nsteps < 0) return MPC_EINVAL;
  if (p->form != MPC_FP64) return MPC_EINVAL;
  Plan P;
  std::string why;
  int rc = make_plan(p, 1, P, &why);
  if (rc) return rc;
  if ((uint64_t)n != P.box[0].n) return MPC_EINVAL;
  if (P.charge > kScratchLimit || P.total > kScratchBytes) return MPC_ERANGE;
  void* ws = nullptr;
  if ((rc = scratch_of_current_device(&ws))) return rc;
  mpc_sim* s = nullptr;
  if ((rc = mpc_create(p, 1, ws, kScratchBytes, hip_stream, &s))) return rc;
  auto done = [&](int code) {
    (void)mpc_destroy(s);
    return code;
  };
  s->use_graph = false;  // kernel by kernel: graph instantiation may allocate
  const double a = p->a;
  if (launch_load_f64(s->dev, s->L, x, v, (uint32_t)n, a, 0) != hipSuccess)
    return done(MPC_EHIP);
  if ((rc = check_sticky(s))) return done(rc == MPC_ESTATE ? MPC_EINVAL : rc);
  if ((rc = mpc_set_step(s, step))) return done(rc);
  if ((rc = mpc_step(s, nsteps))) return done(rc);
  if ((rc = check_sticky(s))) return done(rc);
  if (launch_store_f64(s->dev, s->L, x, v, (uint32_t)n, a, s->cur) != hipSuccess ||
      hipStreamSynchronize(s->L.stream) != hipSuccess)
    return done(MPC_EHIP);
  return done(MPC_OK);
}

}  // extern "C"
