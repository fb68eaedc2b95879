// Batched PCG engine: data layout shared by the kernels and the host driver.
//
// Every solve -- one map or many -- runs on an Engine: the maps' work vectors
// are concatenated (each map contiguous, row-major, at a 64-element aligned
// offset), and every kernel walks a device-resident list of active tiles
// (grid-stride, fixed grid), so one launch serves all maps of a phase and maps
// that have stopped cost nothing once the host compacts the list.
//
// Reductions: each tile writes its FP64 partial sums to its own slot; a
// finisher (a kernel of one block per map, or fused into the tile kernel,
// in the block that completes the map) sums the map's slots in a fixed
// order and advances that map's PCG state.  No grid-wide fences, so results
// are deterministic and nothing serialises across the chip's L2s.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <vector>

namespace lpu {

constexpr int kTW = 128;  // stencil tile width (columns): two per lane of one wave
constexpr int kTH = 16;   // default stencil tile height (rows), four to a wave
constexpr int kDT = 64;   // DCT output tile (64 x 64)
constexpr int kEngineGrid = 16384;  // default cap on the blocks of the grid-stride tile kernels
constexpr int kDctGrid = 2048;     // default cap on the blocks of a DCT stage
constexpr int kArriveGroup = 32;   // tiles per first-level arrival counter of the fused finishers
constexpr int kArriveStride = 64;  // ints from one arrival counter to the next (a 256-byte line each)
constexpr int kEoParts = 4;        // partials of r^T s of an even/odd DCT tile, one per quarter
constexpr int kNumSlots = 4;       // partial-sum slots
constexpr int kListHead = 16;      // ints of counts[] ahead of the active-map list
// polls of one wait of the sweeps: about a second, where a wait on a running predecessor
// takes microseconds
constexpr int kSweepPolls = 1 << 20;
constexpr int kSweepLostAt = 8;    // word of wctl where the address of Engine::lost lies

// DCT tables of one size n as seen by the FP32 FMA kernel.
struct DctTabDev {
  const float* c32;
  const float* ct32;
  const double* lam;
};

// One tile of the MFMA DCT stages for one stage parity (rows of X are the map's
// rows for parity 0, its columns for parity 1), with everything a block reads to
// start the tile, so a tile costs one record load instead of a chain of descriptor
// loads.
struct EoTile {
  long long off;          // element offset of the map
  const uint16_t* tf[3];  // forward tables of the contracted side (EO, or the dense C with
                          // padded rows): fp16, bf16 hi, bf16 lo
  const uint16_t* ti[3];  // inverse tables (EOt, or C^T): fp16, bf16 hi, bf16 lo
  const double* lam_m;    // eigenvalues along M and along N (even/odd in 16 bits: split order)
  const double* lam_n;
  const double* c64;      // C and C^T of the contracted side
  const double* ct64;
  int m, R, K, r0, c0;    // map, rows and contraction length at this parity, tile origin
  int local, ndt, gbd;    // tile index within the map, the map's tile count, arrival group base
  float lmin;             // smallest nonzero eigenvalue of the map's Laplacian
  int side;               // tile side (MapDesc::dtr)
};

struct MapDesc {
  int M, N;
  int th;                     // stencil tile height (rows)
  int tiles_x, ntiles, tile0;  // stencil tiles
  int ndt, dtile0;             // DCT tiles (same count in every stage)
  int dparts;                  // partials of r^T s per DCT tile: kEoParts (even/odd MFMA) or 1
  int dtr;                     // side of a DCT tile: 128 (even/odd MFMA), 64 or 32
  int gb, gbd;                 // first arrival-group counter of the stencil / DCT tiles
  int use_iso;                 // zero the preconditioner output on isolated pixels
  long long off;               // element offset of this map in the work vectors
  long long edge0;             // first entry of this map in the sweeps' edge buffer
  const double* psi;           // caller's wrapped phase
  const float* mask;           // caller's quality mask or null
  double* phi;                 // caller's solution (FP64)
  const DctTabDev* tabM;
  const DctTabDev* tabN;
};

// PCG state of one map (written only by finisher kernels and by the host).
struct MapState {
  double delta_new, delta_old, delta0;
  double alpha, beta;
  double alpha_p;              // x[xi] lacks alpha_p d[l & 1] (added by the next SpMV)
  double dq, rr, bb, rs;
  double thr_rr, thr_delta, tol2, eps2;
  double rr_chk;               // true residual at the last stagnation checkpoint
  long long l_chk, chk_gap;    // its iteration; least iterations between compared checkpoints
  long long l, l_max, period, nfinish;
  long long brk_at;            // > 0: report iteration brk_at's d^T A d as a breakdown (testing hook)
  int state, rule, replaced, stall;  // stall: 1 = stop when the true residual stagnates
  int xi, pad_;                // x[xi] holds the iterate (up to the pending term)
  float amax[4];
};

// What an engine's buffers hold at most.  A smaller map can need more of one of them
// than a larger one (DCT tiles, edge values), so they are kept one by one.
struct EngineCaps {
  long long px = 0;     // pixels
  long long vec = 0;    // bytes of a vector of the working precision
  long long edges = 0;  // entries of wedge
  int tiles = 0, dtiles = 0, maps = 0, strips = 0;
  bool cover(const EngineCaps& o) const {
    return px >= o.px && vec >= o.vec && edges >= o.edges && tiles >= o.tiles && dtiles >= o.dtiles &&
           maps >= o.maps && strips >= o.strips;
  }
  EngineCaps with(const EngineCaps& o) const {
    return {std::max(px, o.px), std::max(vec, o.vec), std::max(edges, o.edges), std::max(tiles, o.tiles),
            std::max(dtiles, o.dtiles), std::max(maps, o.maps), std::max(strips, o.strips)};
  }
};

struct Engine {
  EngineCaps caps;
  int n_maps = 0;
  int total_tiles = 0, total_dtiles = 0;
  int total_strips = 0;      // 64-row strips of the natural-order sweeps
  int act_strips = 0;        // those of the active maps
  int th = kTH;              // stencil tile height (rows)
  int grid = kEngineGrid;    // cap on the blocks of the stencil tile kernels
  int dct_grid = kDctGrid;   // cap on the blocks of a DCT stage (multiple of 8)
  std::vector<MapDesc> hdesc;
  MapDesc* desc = nullptr;
  MapState* ms = nullptr;
  MapState* hms = nullptr;   // pinned mirror
  int* dtile_map = nullptr;  // global DCT tile -> map
  int* act = nullptr;        // active stencil tiles, (tile, map) pairs
  int* dact = nullptr;       // active DCT tiles: XCD-ordered lists of narrow tiles for the
                             // two stage parities, then of wide tiles (see driver)
  long long dlist_cap = 0;   // capacity of each of the four DCT lists
  int dct_trows = kDT;       // 128 when the even/odd MFMA kernels serve the maps, else 64
  bool dct_tile64 = false;   // a map takes FP64 or dense MFMA DCT tiles of 64 x 64
  int* mact = nullptr;       // active maps (sweep kernels)
  int* slist = nullptr;      // (map, strip) pairs of the active maps' strips, strip by strip
  bool no_wait = false;      // sweeps: give up every wait at its first poll (tests)
  int* lost = nullptr;       // sweeps: pinned word, set when a wait was given up
  unsigned int* wctl = nullptr;        // sweeps: ticket, workgroups done, launches so far
  unsigned long long* wedge = nullptr; // sweeps: tagged last rows of the strips
  int* fcnt = nullptr;       // per-map arrival counters of the fused finishers (zero between launches)
  int* gcnt = nullptr;       // per-group arrival counters (groups of kArriveGroup tiles of one map)
  double* gsum = nullptr;    // group sums of the fused finishers: 2 rows of gstride
  long long gstride = 0;
  EoTile* eot = nullptr;     // tile records of the MFMA DCT stages, [parity][global DCT tile]
  int* counts = nullptr;     // [0] active tiles, [1] DCT list (even stages), [2] active
                             // maps, [3] DCT list (odd stages), [4] active strips, [5] and
                             // [7] the wide-tile lists; kListHead ints, followed in the same
                             // allocation by mact, slist, act and dact
  int* hlist = nullptr;      // pinned staging for counts and the lists, same layout
  // FP64 arrays
  double* dx = nullptr;
  double* dy = nullptr;
  double* phi_prev = nullptr;
  double* r64 = nullptr;
  // T arrays (elem bytes per pixel)
  void* U = nullptr;
  void* V = nullptr;
  void* aux = nullptr;
  void* x[2] = {nullptr, nullptr};
  void* d[2] = {nullptr, nullptr};
  void* r = nullptr;
  void* s = nullptr;
  void* q = nullptr;
  void* b = nullptr;
  void* t1 = nullptr;
  void* t2 = nullptr;
  unsigned char* iso = nullptr;  // isolated-pixel flags
  double* P = nullptr;           // partials: kNumSlots x pstride
  long long pstride = 0;
};

}  // namespace lpu
