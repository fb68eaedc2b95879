// Batched kernels of the phase-unwrapping PCG (gfx950).
//
// Stencil tiles are 128 columns x 16 rows, one block each: lane l owns
// columns j0 + l and j0 + 64 + l (two coalesced 64-wide rows per load), a
// wave takes four of the rows with the operand's rows above and below them in
// registers, and horizontal neighbours come from lane shuffles (plus one halo
// column at each side, loaded by lanes 0 and 63).  Each tile writes its FP64
// partial sums to its own slot; finisher kernels reduce per map.
//
// The operator is Eq. (7):
//   (A x)_{i,j} = (U_{i,j-1} + U_{i,j} + V_{i-1,j} + V_{i,j}) x_{i,j}
//               - U_{i,j} x_{i,j+1} - U_{i,j-1} x_{i,j-1}
//               - V_{i,j} x_{i+1,j} - V_{i-1,j} x_{i-1,j},
// out-of-grid terms zero (U is 0 on the last column, V on the last row).

#include <type_traits>

#include "lpu_internal.h"
#include "lpu_device.h"
#include "lpu_finish.h"

namespace lpu {

// ---------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------
template <typename T>
struct R2 {
  T a, b;  // columns j0 + lane, j0 + 64 + lane
};

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// Lane moves on the VALU instead of the LDS crossbar: DPP whole-wave shifts
// by one lane (wave_shr:1 = 0x138: lane l receives lane l-1; wave_shl:1 =
// 0x130: lane l receives lane l+1; the lane with no source receives 0 and is
// overwritten by the caller) and readlane broadcasts.
template <int CTRL>
__device__ __forceinline__ int dpp32(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __builtin_bit_cast(float, dpp32<CTRL>(__builtin_bit_cast(int, v)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = dpp32<CTRL>((int)(b & 0xffffffffLL)), hi = dpp32<CTRL>((int)(b >> 32));
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ float bcast(float v, int src) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), src));
}
__device__ __forceinline__ double bcast(double v, int src) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffLL), src);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), src);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}
template <typename T>
__device__ __forceinline__ T shup(T v) { return dpp_move<0x138>(v); }
template <typename T>
__device__ __forceinline__ T shdn(T v) { return dpp_move<0x130>(v); }
template <typename T>
__device__ __forceinline__ T shfrom(T v, int src) { return bcast(v, src); }

// Blocks of the tile kernels have one wave per kRW rows of a tile (the update
// per kRWUpdate), at most kMaxTileWaves (tile_threads).
constexpr int kMaxTileWaves = 8, kMaxTileThreads = 64 * kMaxTileWaves;

struct TileRef {
  int g, m;  // stencil tile of the engine and its map
};

// the tile sums keep one order over the rows (TileSum)
template <typename T>
constexpr bool kOrdered = sizeof(T) == 8;

struct TilePos {
  int m, i0, j0, M, N, rows;
  int local, ntiles, gb;  // position among the map's tiles, for the fused finishers
  long long off;
};

__device__ __forceinline__ TilePos tile_pos(const MapDesc* __restrict__ desc,
                                            const TileRef& ref) {
  TilePos t;
  t.m = ref.m;
  const MapDesc& d = desc[t.m];
  const int lt = ref.g - d.tile0;
  const int ty = lt / d.tiles_x;
  t.local = lt;
  t.ntiles = d.ntiles;
  t.gb = d.gb;
  t.rows = d.th;
  t.i0 = ty * d.th;
  t.j0 = (lt - ty * d.tiles_x) * kTW;
  t.M = d.M;
  t.N = d.N;
  t.off = d.off;
  return t;
}

// left/right neighbours of a row pair: lane shuffles, and the halo values
// h0 (column j0 - 1) and h1 (column j0 + 128)
template <typename T>
__device__ __forceinline__ void neighbours(const R2<T>& v, T h0, T h1, R2<T>& w, R2<T>& e) {
  const int l = lane_id();
  const T up_a = shup(v.a), up_b = shup(v.b);
  const T dn_a = shdn(v.a), dn_b = shdn(v.b);
  const T a63 = shfrom(v.a, 63), b0 = shfrom(v.b, 0);
  w.a = l > 0 ? up_a : h0;   // column j0 - 1 for lane 0
  w.b = l > 0 ? up_b : a63;  // column j0 + 63 for lane 0
  e.a = l < 63 ? dn_a : b0;  // column j0 + 64 for lane 63
  e.b = l < 63 ? dn_b : h1;  // column j0 + 128 for lane 63
}

// a(i, j), or zero outside the grid; the load goes through a clamped index, so
// it always executes (no lane-divergent branch around it).
template <typename T>
__device__ __forceinline__ T ldz(const T* __restrict__ a, int i, int j, int M, int N) {
  const bool ok = (unsigned)i < (unsigned)M && (unsigned)j < (unsigned)N;
  const int ic = min(max(i, 0), M - 1), jc = min(max(j, 0), N - 1);
  const T v = a[(size_t)ic * N + jc];
  return ok ? v : T(0);
}

__device__ __forceinline__ float fused(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fused(double a, double b, double c) { return __builtin_fma(a, b, c); }

template <typename T>
__device__ __forceinline__ T stencil5(T uw, T uc, T vn, T vc, T xc, T xw, T xe, T xn, T xs) {
  return (uw + uc + vn + vc) * xc - uc * xe - uw * xw - vc * xs - vn * xn;
}

// Rows of a tile go to the block's waves kRW at a time: wave w takes rows
// kRW w, kRW (w + waves), ... .  The wave index is made uniform, so row
// offsets stay in scalar registers.
//
// A map of up to a million pixels has too few tiles to hide memory latency by
// their number (1024^2: 512 tiles on 256 CUs), so a tile's time is what bounds
// its kernels, and with all rows of a tile in flight at once it is one round
// trip instead of the 16 rows of a single wave that marched down the tile two
// rows ahead of its arithmetic.  Measured per SpMV / update launch, one wave
// per tile against four rows per wave (update eight): 64^2 FP64 12.7 / 7.2
// against 8.1 / 6.7 us, 720x960 FP64 Jacobi 18.7 / 18.1 against 16.8 / 10.8,
// 1024^2 FP32 19.5 / 14.5 against 13.2 / 9.2 (with the arrival counters on
// lines of their own, see Arrival), 4096^2 FP32 110 / 50 against 109 / 49,
// where HBM is the bound (537 MB and 201 MB a launch).  The rows above and below
// a wave's own come from the caches.  Two rows per wave: 2 to 4 % faster up to
// 720x960, 6 to 20 % slower from 2048^2 on.  The update has no halo and takes
// eight rows a wave, so that enough loads are in flight at every size (4096^2
// with four: 60 us).
constexpr int kRW = 4;
constexpr int kRWUpdate = 8;

__device__ __forceinline__ int wave_id() {
  return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}
__device__ __forceinline__ int wave_count() { return (int)(blockDim.x >> 6); }

// The addends x y of one pixel's sums.
template <typename T, int NS>
struct Terms {
  T x[NS], y[NS];
};
template <typename T>
struct Terms<T, 0> {};

// Sums over a tile of products of values of type T.
//
// ORDERED (the FP64 path): lane l adds its columns' terms row by row, column
// j0 + l before j0 + 64 + l, and a tree adds the lanes, whatever the number of
// waves the rows are spread over: the lanes' running sums pass from wave to
// wave through LDS in row order.  FP64 solves of some thousand weakly
// preconditioned iterations end at iterates that depend on the order of these
// sums in the eighth digit, so the order is kept free of the launch's shape.
// It costs 0.1 to 0.4 us of a kernel.
// Otherwise (the FP32 path, whose scalars are rounded to FP32): every wave
// adds its own rows, a tree its lanes, and the waves are added in order.
template <typename T, int NS, bool ORDERED>
struct TileSum {
  double* lds;  // NS * 64 doubles
  double sum[NS > 0 ? NS : 1];  // after finish(): valid in thread 0

  __device__ __forceinline__ explicit TileSum(double* smem) : lds(smem) {
#pragma unroll
    for (int n = 0; n < NS; ++n) sum[n] = 0.0;
  }
  // a pixel's terms: added here, or kept in its place of the wave's rows
  __device__ __forceinline__ void put(Terms<T, NS>& place, const Terms<T, NS>& t) {
    if constexpr (ORDERED) place = t;
    else accumulate(t);
  }
  // the kept terms of this wave's next G rows (zero where there is no pixel);
  // every wave of the block calls it equally often, `first` the first time
  template <int G>
  __device__ __forceinline__ void add(bool first, const Terms<T, NS> (&ta)[G],
                                      const Terms<T, NS> (&tb)[G]) {
    if constexpr (NS > 0 && ORDERED) {
      const int l = lane_id(), w = wave_id(), nw = wave_count();
      for (int k = 0; k < nw; ++k) {
        if (w == k) {
          if (!first || k > 0)
#pragma unroll
            for (int n = 0; n < NS; ++n) sum[n] = lds[64 * n + l];
#pragma unroll
          for (int c = 0; c < G; ++c) {
            accumulate(ta[c]);
            accumulate(tb[c]);
          }
#pragma unroll
          for (int n = 0; n < NS; ++n) lds[64 * n + l] = sum[n];
        }
        __syncthreads();
      }
    }
  }
  __device__ __forceinline__ void accumulate(const Terms<T, NS>& t) {
    if constexpr (NS > 0)
#pragma unroll
      for (int n = 0; n < NS; ++n) sum[n] = fma((double)t.x[n], (double)t.y[n], sum[n]);
  }
  __device__ __forceinline__ void finish() {
    if constexpr (NS > 0 && !ORDERED) {
      block_sum<NS>(sum, lds);
    } else if constexpr (NS > 0) {
      if (wave_id() == 0)
#pragma unroll
        for (int n = 0; n < NS; ++n) sum[n] = tree64(lds[64 * n + lane_id()]);
    }
  }
};

// Stencil over the tile's rows of this wave: for every interior pixel
// epi(i, row, j, x_ij, (A x)_ij, raw_ij, own_ij), row = i N, which returns the
// pixel's terms of the sums in ts.  The operand x is
// formed as make(load(row, j), i, j) (make_north in the first column group of
// the row above the tile) and is zero outside the grid; own(row, j)
// loads what only the pixel itself needs.  load and own must only load: every
// load of kRW rows (and of the operand rows above and below them) is issued
// through clamped coordinates before the first value is used, so a wave pays
// one memory round trip per kRW rows.
template <typename T, int NS, bool OR, typename Ld, typename Mk, typename Mn, typename Ow, typename E>
__device__ __forceinline__ void stencil_tile(const TilePos& tp, TileSum<T, NS, OR>& ts,
                                             const T* __restrict__ U, const T* __restrict__ V,
                                             Ld load, Mk make, Mn make_north, Ow own, E epi) {
  const int M = tp.M, N = tp.N, j0 = tp.j0, l = lane_id();
  const int ca = j0 + l, cb = j0 + 64 + l;
  const bool oka = ca < N, okb = cb < N;
  const unsigned ja = min(ca, N - 1), jb = min(cb, N - 1);
  // The halo columns of the wave's rows come in one load: lane 2 c + side holds
  // row c's column j0 - 1 (side 0) or j0 + 128 (side 1).
  static_assert(kRW <= 32, "two lanes a row");
  const int hj = (l & 1) ? j0 + kTW : j0 - 1;
  const bool okh = (unsigned)hj < (unsigned)N;
  const unsigned jh = min(max(hj, 0), N - 1);
  const int i_end = min(tp.i0 + tp.rows, M);
  using Raw = decltype(load(size_t(0), 0u));
  using Own = decltype(own(size_t(0), 0u));
  // ordered sums need the same number of turns in every wave; otherwise a wave
  // without rows leaves at once (4096^2 FP32 SpMV 109 against 114 us)
  const int wrow = wave_id() * kRW, step = wave_count() * kRW, lead = OR ? wrow : 0;
  for (int i0 = tp.i0 + wrow; i0 - lead < i_end; i0 += step) {
    Terms<T, NS> ta[kRW] = {}, tb[kRW] = {};
    Raw ra[kRW + 2], rb[kRW + 2];  // operand rows i0 - 1 .. i0 + kRW
    Own oa[kRW], ob[kRW];
    R2<T> u[kRW], v[kRW + 1];  // V rows i0 - 1 .. i0 + kRW - 1
    const int ih = i0 + (l >> 1) % kRW;
    const size_t hrow = (size_t)min(ih, M - 1) * N;
    const Raw rh = load(hrow, jh);
    const T uh = U[hrow + jh];
#pragma unroll
    for (int c = 0; c < kRW + 2; ++c) {
      const size_t row = (size_t)min(max(i0 - 1 + c, 0), M - 1) * N;
      ra[c] = load(row, ja);
      rb[c] = load(row, jb);
      if (c <= kRW) {
        v[c].a = V[row + ja];
        v[c].b = V[row + jb];
      }
      if (c > 0 && c <= kRW) {
        u[c - 1].a = U[row + ja];
        u[c - 1].b = U[row + jb];
        oa[c - 1] = own(row, ja);
        ob[c - 1] = own(row, jb);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    auto operand = [&](const Raw& r, int i, int j, bool okc) {
      return okc && (unsigned)i < (unsigned)M ? make(r, i, j) : T(0);
    };
    R2<T> xm{operand(ra[0], i0 - 1, ca, oka), operand(rb[0], i0 - 1, cb, okb)};
    if constexpr (!std::is_same_v<Mk, Mn>) {
      if (i0 == tp.i0) xm.a = oka && i0 > 0 ? make_north(ra[0], i0 - 1, ca) : T(0);
    }
    R2<T> xc{operand(ra[1], i0, ca, oka), operand(rb[1], i0, cb, okb)};
    const T xh = operand(rh, ih, hj, okh);
    const T uw0 = j0 > 0 ? uh : T(0);  // the couplings to column j0 - 1
    if (i0 == 0) v[0].a = v[0].b = T(0);
#pragma unroll
    for (int c = 0; c < kRW; ++c) {
      const int i = i0 + c;
      if (i >= i_end) break;  // uniform over the wave
      const R2<T> xp{operand(ra[c + 2], i + 1, ca, oka), operand(rb[c + 2], i + 1, cb, okb)};
      R2<T> xw, xe, uw, ue;
      neighbours(xc, shfrom(xh, 2 * c), shfrom(xh, 2 * c + 1), xw, xe);
      neighbours(u[c], shfrom(uw0, 2 * c), T(0), uw, ue);
      const T qa = stencil5<T>(uw.a, u[c].a, v[c].a, v[c + 1].a, xc.a, xw.a, xe.a, xm.a, xp.a);
      const T qb = stencil5<T>(uw.b, u[c].b, v[c].b, v[c + 1].b, xc.b, xw.b, xe.b, xm.b, xp.b);
      const size_t row = (size_t)i * N;
      if (oka) ts.put(ta[c], epi(i, row, ja, xc.a, qa, ra[c + 1], oa[c]));
      if (okb) ts.put(tb[c], epi(i, row, jb, xc.b, qb, rb[c + 1], ob[c]));
      xm = xc;
      xc = xp;
    }
    ts.template add<kRW>(i0 == tp.i0 + wrow, ta, tb);
  }
  ts.finish();
}

template <typename T, int NS, bool OR, typename Ld, typename Mk, typename Ow, typename E>
__device__ __forceinline__ void stencil_tile(const TilePos& tp, TileSum<T, NS, OR>& ts,
                                             const T* __restrict__ U, const T* __restrict__ V,
                                             Ld load, Mk make, Ow own, E epi) {
  stencil_tile<T>(tp, ts, U, V, load, make, make, own, epi);
}

// Elementwise walk over the tile's pixels.
template <typename E>
__device__ __forceinline__ void march_points(const TilePos& tp, E epi) {
  const int l = lane_id();
  const int kend = min(tp.rows, tp.M - tp.i0);
  for (int k = wave_id(); k < kend; k += wave_count()) {
    const int i = tp.i0 + k;
    const int ca = tp.j0 + l, cb = tp.j0 + 64 + l;
    if (ca < tp.N) epi(i, ca);
    if (cb < tp.N) epi(i, cb);
  }
}

// Elementwise walk in groups of G rows: load(i, j) issues every load of one
// pixel (the walk passes in-grid coordinates, clamped for lanes and rows past
// the map, whose results are dropped), store(i, j, v) computes and stores
// (and returns the pixel's terms of the sums in ts).
// All loads of a group are issued before its first store: loads and stores
// share one wait counter, so a load issued after a store would also wait for
// the store, a memory round trip per pixel row.
template <int G, typename T, int NS, bool OR, typename L, typename S>
__device__ __forceinline__ void march_points_grouped(const TilePos& tp, TileSum<T, NS, OR>& ts, L load,
                                                     S store) {
  const int l = lane_id();
  const int kend = min(tp.rows, tp.M - tp.i0);
  const int ca = tp.j0 + l, cb = tp.j0 + 64 + l;
  const int ja = min(ca, tp.N - 1), jb = min(cb, tp.N - 1);
  using Val = decltype(load(0, 0));
  const int wrow = wave_id() * G, lead = OR ? wrow : 0;  // as in stencil_tile
  for (int k0 = wrow; k0 - lead < kend; k0 += wave_count() * G) {
    Terms<T, NS> ta[G] = {}, tb[G] = {};
    Val v[G][2];
#pragma unroll
    for (int c = 0; c < G; ++c) {
      const int i = min(tp.i0 + k0 + c, tp.M - 1);
      v[c][0] = load(i, ja);
      v[c][1] = load(i, jb);
    }
#pragma unroll
    for (int c = 0; c < G; ++c) {
      if (k0 + c >= kend) break;  // uniform over the wave
      const int i = tp.i0 + k0 + c;
      if (ca < tp.N) ts.put(ta[c], store(i, ca, v[c][0]));
      if (cb < tp.N) ts.put(tb[c], store(i, cb, v[c][1]));
    }
    ts.template add<G>(k0 == wrow, ta, tb);
  }
  ts.finish();
}
template <int G, typename L, typename S>
__device__ __forceinline__ void march_points_grouped(const TilePos& tp, L load, S store) {
  TileSum<float, 0, false> none(nullptr);
  march_points_grouped<G>(tp, none, load, [&](int i, int j, const auto& v) {
    store(i, j, v);
    return Terms<float, 0>{};
  });
}

template <typename T>
__device__ __forceinline__ T* vec(void* base, long long off) {
  return reinterpret_cast<T*>(base) + off;
}
template <typename T>
__device__ __forceinline__ const T* cvec(const void* base, long long off) {
  return reinterpret_cast<const T*>(base) + off;
}

// Kernel arguments shared by the tile kernels.
struct EArgs {
  const MapDesc* desc;
  MapState* ms;
  const int* act;  // (tile, map) pairs
  int act_cap;     // its capacity in pairs
  const int* counts;
  double* P;
  long long pstride;
  void *U, *V, *aux, *x0, *x1, *d0, *d1, *r, *s, *q, *b;
  double *dx, *dy, *phi_prev, *r64;
  const unsigned char* iso;
  int *fcnt, *gcnt;  // arrival counters of the finisher fused into the tile kernel
  double* gsum;      // its group sums (rows of gstride)
  long long gstride;
  int fuse_pw;  // -1: no fused finisher; else its pointwise-preconditioner flag
  int expect;   // two-colour preconditioner: state of the maps it applies to
  int fin_mode;  // two-colour preconditioner: FinishMode of its fused finisher (0: none)
};

__device__ __forceinline__ Arrival arrival(const EArgs& A) {
  return Arrival{A.fcnt, A.gcnt, A.gsum, A.gstride, A.P, A.pstride};
}

__device__ __forceinline__ TileRef tile_ref(const EArgs& A, int t) {
  return TileRef{A.act[2 * (size_t)t], A.act[2 * (size_t)t + 1]};
}

// Grid-stride walk over the active tiles.  The block's first list entry is
// requested together with the list's length (through an index clamped to
// the list's capacity; it is used only when the block has a tile), and the
// entry names the tile's map, so the map's descriptor and state are the
// second memory round trip of a block and its pixels the third.
#define TILE_LOOP(A)                                                          \
  const int n_act_ = (A).counts[0];                                           \
  const TileRef first_ = tile_ref(A, min((int)blockIdx.x, max((A).act_cap - 1, 0))); \
  __asm__ volatile("" ::"s"(n_act_), "s"(first_.g), "s"(first_.m)); /* loads issued here */ \
  for (int t_ = blockIdx.x; t_ < n_act_; t_ += gridDim.x)
#define TILE_REF(A) (t_ == (int)blockIdx.x ? first_ : tile_ref(A, t_))

// ---------------------------------------------------------------------------
// Set-up kernels: wrapped differences, weights, Jacobi diagonal, isolation
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wrap_w(double x) {
#pragma clang fp contract(off)
  const double k = ceil((x - kPi) / kTwoPi);
  return x - kTwoPi * k;
}

// zero_phi: also set the caller's phi to 0 (the start value when the caller
// does not supply one)
__global__ void __launch_bounds__(kMaxTileThreads) k_e_wrapdiff(EArgs A, int zero_phi) {
  TILE_LOOP(A) {
    const TileRef ref = TILE_REF(A);
    const TilePos tp = tile_pos(A.desc, ref);
    const double* psi = A.desc[tp.m].psi;
    double* phi = A.desc[tp.m].phi;
    double* dx = A.dx + tp.off;
    double* dy = A.dy + tp.off;
    struct Px {
      double c, e, s;
    };
    march_points_grouped<4>(
        tp,
        [&](int i, int j) {
          // neighbours outside the grid read the pixel itself (never used)
          const size_t p = (size_t)i * tp.N + j;
          Px x;
          x.c = psi[p];
          x.e = psi[j < tp.N - 1 ? p + 1 : p];
          x.s = psi[i < tp.M - 1 ? p + tp.N : p];
          return x;
        },
        [&](int i, int j, const Px& x) {
          const size_t p = (size_t)i * tp.N + j;
          dx[p] = (j < tp.N - 1) ? wrap_w(x.e - x.c) : 0.0;
          dy[p] = (i < tp.M - 1) ? wrap_w(x.s - x.c) : 0.0;
          if (zero_phi) phi[p] = 0.0;
        });
  }
}

// Input check of every map in one launch: *bad |= 1 when psi holds a
// non-finite value or the mask one outside [0, 1].
__global__ void __launch_bounds__(kMaxTileThreads) k_e_check(EArgs A, unsigned int* bad) {
  unsigned int b = 0;
  TILE_LOOP(A) {
    const TileRef ref = TILE_REF(A);
    const TilePos tp = tile_pos(A.desc, ref);
    const double* psi = A.desc[tp.m].psi;
    const float* mask = A.desc[tp.m].mask;
    march_points(tp, [&](int i, int j) {
      const size_t p = (size_t)i * tp.N + j;
      if (!isfinite(psi[p])) b = 1;
      if (mask && !(isfinite(mask[p]) && mask[p] >= 0.0f && mask[p] <= 1.0f)) b = 1;
    });
  }
  if (b) atomicOr(bad, 1u);
}

__device__ __forceinline__ double abs_pow(double r, double e) {
  if (e == 2.0) return r * r;
  if (e == 1.0) return fabs(r);
  if (e == 0.0) return 1.0;
  return pow(fabs(r), e);
}

// U, V of Eq. (6) from phi (FP64), stored as T; also the Jacobi inverse
// diagonal needs U, V of neighbours, so it is a separate pass.
template <typename T>
__global__ void __launch_bounds__(kMaxTileThreads) k_e_weights(EArgs A, double e, double tau) {
  TILE_LOOP(A) {
    const TileRef ref = TILE_REF(A);
    const TilePos tp = tile_pos(A.desc, ref);
    const MapDesc& d = A.desc[tp.m];
    const double* phi = d.phi;
    const float* mask = d.mask;
    const double* dx = A.dx + tp.off;
    const double* dy = A.dy + tp.off;
    T* U = vec<T>(A.U, tp.off);
    T* V = vec<T>(A.V, tp.off);
    struct Px {
      double c, e, s, dx, dy;
      float mc, me, ms;
    };
    march_points_grouped<2>(
        tp,
        [&](int i, int j) {
          // neighbours outside the grid read the pixel itself (never used)
          const size_t p = (size_t)i * tp.N + j;
          const size_t pe = j < tp.N - 1 ? p + 1 : p, ps = i < tp.M - 1 ? p + tp.N : p;
          Px x;
          x.c = phi[p];
          x.e = phi[pe];
          x.s = phi[ps];
          x.dx = dx[p];
          x.dy = dy[p];
          x.mc = mask ? mask[p] : 1.0f;
          x.me = mask ? mask[pe] : 1.0f;
          x.ms = mask ? mask[ps] : 1.0f;
          return x;
        },
        [&](int i, int j, const Px& x) {
          const size_t p = (size_t)i * tp.N + j;
          double u = 0.0, v = 0.0;
          if (j < tp.N - 1) {
            const double r = x.e - x.c - x.dx;
            const double w = mask ? (double)fminf(x.mc, x.me) : 1.0;
            u = w * (tau / (abs_pow(r, e) + tau));
          }
          if (i < tp.M - 1) {
            const double r = x.s - x.c - x.dy;
            const double w = mask ? (double)fminf(x.mc, x.ms) : 1.0;
            v = w * (tau / (abs_pow(r, e) + tau));
          }
          U[p] = (T)u;
          V[p] = (T)v;
        });
  }
}

// Jacobi inverse diagonal (0 on isolated pixels) and isolation flags.
template <typename T>
__global__ void __launch_bounds__(kMaxTileThreads) k_e_diag(EArgs A, int want_inv) {
  TILE_LOOP(A) {
    const TileRef ref = TILE_REF(A);
    const TilePos tp = tile_pos(A.desc, ref);
    const T* U = cvec<T>(A.U, tp.off);
    const T* V = cvec<T>(A.V, tp.off);
    T* inv = vec<T>(A.aux, tp.off);
    unsigned char* iso = const_cast<unsigned char*>(A.iso) + tp.off;
    march_points(tp, [&](int i, int j) {
      const size_t p = (size_t)i * tp.N + j;
      const T dg = ldz(U, i, j - 1, tp.M, tp.N) + U[p] + ldz(V, i - 1, j, tp.M, tp.N) + V[p];
      if (want_inv) inv[p] = dg > T(0) ? T(1) / dg : T(0);
      iso[p] = dg == T(0) ? 1 : 0;
    });
  }
}

// ---------------------------------------------------------------------------
// b = D^T W Delta and r64 = b - A phi (FP64; r formed as D^T W (Delta - D phi)).
// mode 0: b as T and as FP64 in r64 (phi unused); mode 1: r64 and (T) r64 into b;
// mode 2: r64 only.  Partials: slot 0 = r.r (mode 0: b.b), slot 1 = b.b.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(kMaxTileThreads) k_e_rhs(EArgs A, int mode) {
  __shared__ double red[2 * 64];
  TILE_LOOP(A) {
    const TileRef ref = TILE_REF(A);
    const TilePos tp = tile_pos(A.desc, ref);
    const MapDesc& d = A.desc[tp.m];
    const T* U = cvec<T>(A.U, tp.off);
    const T* V = cvec<T>(A.V, tp.off);
    const double* dx = A.dx + tp.off;
    const double* dy = A.dy + tp.off;
    const double* phi = d.phi;
    T* bT = vec<T>(A.b, tp.off);
    double* r64 = A.r64 + tp.off;
    const int M = tp.M, N = tp.N;
    const bool usephi = mode != 0;
    TileSum<double, 2, kOrdered<T>> ts(red);  // r.r, b.b
    struct Px {
      double pc, pe, pw, pn, ps, dxc, dxw, dyc, dyn;
      T uc, uw, vc, vn;
    };
    march_points_grouped<2>(
        tp, ts,
        [&](int i, int j) {
          // neighbours outside the grid read the pixel itself (never used)
          const size_t p = (size_t)i * N + j;
          const size_t pe = j < N - 1 ? p + 1 : p, pw = j > 0 ? p - 1 : p;
          const size_t pn = i > 0 ? p - N : p, ps = i < M - 1 ? p + N : p;
          Px x;
          x.pc = usephi ? phi[p] : 0.0;
          x.pe = usephi ? phi[pe] : 0.0;
          x.pw = usephi ? phi[pw] : 0.0;
          x.pn = usephi ? phi[pn] : 0.0;
          x.ps = usephi ? phi[ps] : 0.0;
          x.dxc = dx[p];
          x.dxw = dx[pw];
          x.dyc = dy[p];
          x.dyn = dy[pn];
          x.uc = U[p];
          x.uw = U[pw];
          x.vc = V[p];
          x.vn = V[pn];
          return x;
        },
        [&](int i, int j, const Px& x) {
          const size_t p = (size_t)i * N + j;
          double hx = 0.0, hy = 0.0, bx = 0.0, by = 0.0, hxw = 0.0, hyn = 0.0, bxw = 0.0, byn = 0.0;
          if (j < N - 1) {
            const double u = (double)x.uc;
            bx = u * x.dxc;
            hx = usephi ? u * (x.dxc - (x.pe - x.pc)) : bx;
          }
          if (i < M - 1) {
            const double v = (double)x.vc;
            by = v * x.dyc;
            hy = usephi ? v * (x.dyc - (x.ps - x.pc)) : by;
          }
          if (j > 0) {
            const double u = (double)x.uw;
            bxw = u * x.dxw;
            hxw = usephi ? u * (x.dxw - (x.pc - x.pw)) : bxw;
          }
          if (i > 0) {
            const double v = (double)x.vn;
            byn = v * x.dyn;
            hyn = usephi ? v * (x.dyn - (x.pc - x.pn)) : byn;
          }
          const double b = bxw + byn - bx - by;
          const double r = hxw + hyn - hx - hy;
          if (mode == 0) bT[p] = (T)b;
          if (mode == 1) bT[p] = (T)r;
          r64[p] = mode == 0 ? b : r;
          return Terms<double, 2>{{r, b}, {r, b}};
        });
    if (threadIdx.x == 0) {
      A.P[0 * A.pstride + ref.g] = ts.sum[0];
      A.P[1 * A.pstride + ref.g] = ts.sum[1];
    }
  }
}

// ---------------------------------------------------------------------------
// Small per-tile passes used by the outer loop
// ---------------------------------------------------------------------------
// op 0: phi_prev = phi; op 1: x0 = phi (T); op 2: x0 = 0;
// op 3: phi += x_final (x[xi] plus a pending step); op 4: partials of
// ||phi - phi_prev||^2 (slot 0) and ||phi_prev||^2 (slot 1);
// op 5: phi = x_final (FP64 path).
template <typename T>
__global__ void __launch_bounds__(kMaxTileThreads) k_e_pass(EArgs A, int op) {
  __shared__ double red[2 * 64];
  TILE_LOOP(A) {
    const TileRef ref = TILE_REF(A);
    const TilePos tp = tile_pos(A.desc, ref);
    double* phi = A.desc[tp.m].phi;
    double* pp = A.phi_prev + tp.off;
    const MapState& ms = A.ms[tp.m];
    const long long l = ms.l;
    T* x0 = vec<T>(A.x0, tp.off);
    // the final iterate: x[xi] plus the pending step alpha_p d[l & 1]
    const T* xf = cvec<T>(ms.xi ? A.x1 : A.x0, tp.off);
    const T* dp = cvec<T>((l & 1) ? A.d1 : A.d0, tp.off);
    const T ap = (T)ms.alpha_p;
    const bool pend = ms.alpha_p != 0.0;
    TileSum<double, 2, kOrdered<T>> ts(red);  // op 4
    struct Px {
      double a, b;  // phi (ops 0, 1, 3, 4), phi_prev (op 4)
      T x, dd;      // final iterate and pending direction (ops 3, 5)
    };
    march_points_grouped<4>(
        tp, ts,
        [&](int i, int j) {
          const size_t p = (size_t)i * tp.N + j;
          Px v{0.0, 0.0, T(0), T(0)};
          if (op == 0 || op == 1 || op == 3 || op == 4) v.a = phi[p];
          if (op == 4) v.b = pp[p];
          if (op == 3 || op == 5) {
            v.x = xf[p];
            if (pend) v.dd = dp[p];
          }
          return v;
        },
        [&](int i, int j, const Px& v) {
          const size_t p = (size_t)i * tp.N + j;
          Terms<double, 2> t{{0.0, 0.0}, {0.0, 0.0}};
          switch (op) {
            case 0: pp[p] = v.a; break;
            case 1: x0[p] = (T)v.a; break;
            case 2: x0[p] = T(0); break;
            case 3: phi[p] = v.a + (double)(pend ? v.x + ap * v.dd : v.x); break;
            case 4: {
              const double dd = v.a - v.b;
              t = Terms<double, 2>{{dd, v.b}, {dd, v.b}};
            } break;
            case 5: phi[p] = (double)(pend ? v.x + ap * v.dd : v.x); break;
          }
          return t;
        });
    if (op == 4 && threadIdx.x == 0) {
      A.P[0 * A.pstride + ref.g] = ts.sum[0];
      A.P[1 * A.pstride + ref.g] = ts.sum[1];
    }
  }
}

// ---------------------------------------------------------------------------
// PCG tile kernels
// ---------------------------------------------------------------------------
// init: r = b - A x0, d_old(parity 0) = 0, pointwise s; partials r.r, r.s, b.b
// confirm (CONF = 1): r = b - A x (current parity), pointwise s; partials r.r, r.s
template <typename T, int PC, int CONF>
__global__ void __launch_bounds__(kMaxTileThreads) k_e_resid(EArgs A) {
  __shared__ double red[3 * 64];
  TILE_LOOP(A) {
    const TileRef ref = TILE_REF(A);
    const TilePos tp = tile_pos(A.desc, ref);
    const MapState& st = A.ms[tp.m];
    if (st.state != (CONF ? kConfirm : kRun)) continue;
    const long long l = st.l;
    const T* U = cvec<T>(A.U, tp.off);
    const T* V = cvec<T>(A.V, tp.off);
    const T* aux = cvec<T>(A.aux, tp.off);
    const T* b = cvec<T>(A.b, tp.off);
    // the iterate: x0 (init), or x[xi] plus the pending step alpha_p d[l & 1]
    const T* x = cvec<T>(CONF && st.xi ? A.x1 : A.x0, tp.off);
    const T* dp = cvec<T>((l & 1) ? A.d1 : A.d0, tp.off);
    const T ap = CONF ? (T)st.alpha_p : T(0);
    const bool pend = CONF && st.alpha_p != 0.0;
    T* r = vec<T>(A.r, tp.off);
    T* d0 = vec<T>(A.d0, tp.off);
    TileSum<T, 3, kOrdered<T>> ts(red);  // r.r, r.s, b.b
    struct Op {
      T x, d;
    };
    struct Own {
      T b, w;
    };
    stencil_tile<T>(
        tp, ts, U, V, [&](size_t row, unsigned j) { return Op{x[row + j], pend ? dp[row + j] : T(0)}; },
        [&](const Op& v, int, int) { return pend ? v.x + ap * v.d : v.x; },
        [&](size_t row, unsigned j) {
          return Own{b[row + j], PC == kPcJacobi ? aux[row + j] : T(1)};
        },
        [&](int, size_t row, unsigned j, T, T ax, const Op&, const Own& o) {
          const T rv = o.b - ax;
          r[row + j] = rv;
          if (!CONF) d0[row + j] = T(0);
          const T sv = PC == kPcJacobi ? rv * o.w : rv;
          return Terms<T, 3>{{rv, rv, o.b}, {rv, sv, o.b}};
        });
    if (threadIdx.x == 0) {
      A.P[0 * A.pstride + ref.g] = ts.sum[0];
      A.P[1 * A.pstride + ref.g] = ts.sum[1];
      A.P[2 * A.pstride + ref.g] = ts.sum[2];
    }
  }
}

// Non-temporal accesses for data whose next use is a later iteration (the
// iterate, the new direction) or that is dead after this read (q in the
// update): they leave the caches to what the next kernel reads.
template <typename T>
__device__ __forceinline__ T ld_stream(const T* p) { return __builtin_nontemporal_load(p); }
template <typename T>
__device__ __forceinline__ void st_stream(T* p, T v) { __builtin_nontemporal_store(v, p); }

// spmv: d_new = s + beta d_old; q = A d_new; partial d^T q.  Also adds the
// previous iteration's step to the iterate, x += alpha_p d_old (the update
// leaves it here: x is first needed again by a replacement or at the end, and
// this kernel reads d_old anyway, so the step costs one read and one write of
// x instead of two reads, a write and a second read of d in the update).
template <typename T, int PC>
__global__ void __launch_bounds__(kMaxTileThreads) k_e_spmv(EArgs A) {
  __shared__ double lsum[1 * 64];
  __shared__ double fred[3 * kMaxTileWaves];
  __shared__ int fflag;
  TILE_LOOP(A) {
    const TileRef ref = TILE_REF(A);
    const TilePos tp = tile_pos(A.desc, ref);
    const MapState& st = A.ms[tp.m];
    const int state = st.state, xi = st.xi;
    const long long l = st.l;
    const double beta64 = st.beta, ap64 = st.alpha_p;
    // requested together, with the descriptor
    __asm__ volatile("" ::"s"(state), "s"(xi), "s"(l), "s"(beta64), "s"(ap64));
    if (state != kRun) continue;
    const T beta = (T)beta64;
    const T ap = (T)ap64;
    const bool pend = ap64 != 0.0;
    T* x = vec<T>(xi ? A.x1 : A.x0, tp.off);
    const T* U = cvec<T>(A.U, tp.off);
    const T* V = cvec<T>(A.V, tp.off);
    const T* aux = cvec<T>(A.aux, tp.off);
    const T* src = cvec<T>(PC == kPcNone || PC == kPcJacobi ? A.r : A.s, tp.off);
    const T* dold = cvec<T>((l & 1) ? A.d1 : A.d0, tp.off);
    T* dnew = vec<T>((l & 1) ? A.d0 : A.d1, tp.off);
    T* q = vec<T>(A.q, tp.off);
    TileSum<T, 1, kOrdered<T>> ts(lsum);  // d_new^T q
    struct Op {
      T s, w, d;  // s (or r), inverse diagonal, d_old
    };
    stencil_tile<T>(
        tp, ts, U, V,
        [&](size_t row, unsigned j) {
          return Op{src[row + j], PC == kPcJacobi ? aux[row + j] : T(1), dold[row + j]};
        },
        // Jacobi: s w + beta d rounds beta d first, except in the left half of the
        // row above the tile, where q is formed with a d that differs from the one
        // its own tile stores in the last bit.  One rounding everywhere would be as
        // good, but solves keep the bits they have always had (a mixed one of a
        // thousand iterations moves by 1e-4 with one such rounding)
        [&](const Op& v, int, int) {
          return PC == kPcJacobi ? fused(v.s, v.w, beta * v.d) : fused(beta, v.d, v.s);
        },
        [&](const Op& v, int, int) {
          return fused(beta, v.d, PC == kPcJacobi ? v.s * v.w : v.s);
        },
        [&](size_t row, unsigned j) { return ld_stream(x + row + j); },
        [&](int, size_t row, unsigned j, T dv, T qv, const Op& v, T xv) {
          st_stream(dnew + row + j, dv);
          q[row + j] = qv;
          if (pend) st_stream(x + row + j, xv + ap * v.d);
          return Terms<T, 1>{{dv}, {qv}};
        });
    if (threadIdx.x == 0) store_partial(A.P + 0 * A.pstride + ref.g, ts.sum[0]);
    if (A.fuse_pw >= 0) {
      const int sl[1] = {0};
      fused_finish<kFinAlpha, 1, 64>(arrival(A), sl, ref.g - tp.local, tp.local, tp.ntiles, tp.gb, A.desc,
                                 A.ms, tp.m, kFinishNone, A.fuse_pw, &fflag, fred);
    }
  }
}

// update: r -= alpha q (the step alpha d is added to x by the next SpMV), or,
// when l is a multiple of the replacement period, x_new = x + alpha d into
// the other x buffer and r = b - A x_new; pointwise s; partials r.r, r.s
template <typename T, int PC>
__global__ void __launch_bounds__(kMaxTileThreads) k_e_update(EArgs A) {
  __shared__ double lsum[2 * 64];
  __shared__ double fred[3 * kMaxTileWaves];
  __shared__ int fflag;
  TILE_LOOP(A) {
    const TileRef ref = TILE_REF(A);
    const TilePos tp = tile_pos(A.desc, ref);
    const MapState& st = A.ms[tp.m];
    const int state = st.state, xi = st.xi;
    const long long l = st.l, period = st.period;
    const double alpha64 = st.alpha;
    // requested together, with the descriptor
    __asm__ volatile("" ::"s"(state), "s"(xi), "s"(l), "s"(period), "s"(alpha64));
    if (state != kRun) continue;
    const T alpha = (T)alpha64;
    const bool replace = divides(period, l);
    const T* U = cvec<T>(A.U, tp.off);
    const T* V = cvec<T>(A.V, tp.off);
    const T* aux = cvec<T>(A.aux, tp.off);
    const T* b = cvec<T>(A.b, tp.off);
    const T* q = cvec<T>(A.q, tp.off);
    T* r = vec<T>(A.r, tp.off);
    TileSum<T, 2, kOrdered<T>> ts(lsum);  // r.r, r.s
    if (replace) {
      const T* xold = cvec<T>(xi ? A.x1 : A.x0, tp.off);
      T* xnew = vec<T>(xi ? A.x0 : A.x1, tp.off);
      const T* d = cvec<T>((l & 1) ? A.d0 : A.d1, tp.off);
      struct Op {
        T x, d;
      };
      struct Own {
        T b, w;
      };
      stencil_tile<T>(
          tp, ts, U, V, [&](size_t row, unsigned j) { return Op{xold[row + j], d[row + j]}; },
          [&](const Op& v, int, int) { return v.x + alpha * v.d; },
          [&](size_t row, unsigned j) {
            return Own{b[row + j], PC == kPcJacobi ? aux[row + j] : T(1)};
          },
          [&](int, size_t row, unsigned j, T xv, T ax, const Op&, const Own& o) {
            const T rv = o.b - ax;
            xnew[row + j] = xv;
            r[row + j] = rv;
            const T sv = PC == kPcJacobi ? rv * o.w : rv;
            return Terms<T, 2>{{rv, rv}, {rv, sv}};
          });
    } else {
      struct Px {
        T r, q, w;
      };
      march_points_grouped<kRWUpdate>(
          tp, ts,
          [&](int i, int j) {
            const size_t row = (size_t)i * tp.N;
            return Px{r[row + (unsigned)j], ld_stream(q + row + (unsigned)j),
                      PC == kPcJacobi ? aux[row + (unsigned)j] : T(1)};
          },
          [&](int i, int j, const Px& v) {
            const T rn = v.r - alpha * v.q;
            r[(size_t)i * tp.N + (unsigned)j] = rn;
            const T sv = PC == kPcJacobi ? rn * v.w : rn;
            return Terms<T, 2>{{rn, rn}, {rn, sv}};
          });
    }
    if (threadIdx.x == 0) {
      store_partial(A.P + 0 * A.pstride + ref.g, ts.sum[0]);
      store_partial(A.P + 1 * A.pstride + ref.g, ts.sum[1]);
    }
    if (A.fuse_pw >= 0) {
      const int sl[2] = {0, 1};
      fused_finish<kFinUpdate, 2, 64>(arrival(A), sl, ref.g - tp.local, tp.local, tp.ntiles, tp.gb, A.desc,
                                  A.ms, tp.m, kFinishNone, A.fuse_pw, &fflag, fred);
    }
  }
}

// ---------------------------------------------------------------------------
// Two-colour ILU(0) = IC(0) and SSOR of Eq. (7)'s matrix (a GPU-parallel
// change of M; the paper's sweeps use the natural order).  Pixel (i, j) is
// "even" when i + j is even.  With the even pixels ordered first the matrix is
// [[D_e, -B], [-B^T, D_o]]: no two pixels of one colour are coupled, so the
// no-fill factorisation keeps the even diagonal as pivots and gives the odd
// pivots p_o = a_oo - sum over even neighbours e of a_oe^2 / a_ee (SSOR: every
// pivot a / omega).  M = (P + L) P^-1 (P + L^T) (over 2 - omega for SSOR) is
// applied in two passes, c = 2 - omega for SSOR and 1 otherwise:
//   odd pixels:  s_o = c (r_o + sum_e w_oe r_e / p_e) / p_o   (forward solve)
//   even pixels: s_e = (c r_e + sum_o w_eo s_o) / p_e         (backward solve)
// Each pass is a stencil pass of Eq. (7) with an operand that is zero on the
// pixels it writes, so the neighbour sum is -(A x) there; the first pass only
// writes odd pixels and the second only even ones, and each reads s only on
// the colour it does not write.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(kMaxTileThreads) k_e_tc_pivots(EArgs A, int ssor, double omega) {
  TILE_LOOP(A) {
    const TileRef ref = TILE_REF(A);
    const TilePos tp = tile_pos(A.desc, ref);
    const T* U = cvec<T>(A.U, tp.off);
    const T* V = cvec<T>(A.V, tp.off);
    T* piv = vec<T>(A.aux, tp.off);
    unsigned char* iso = const_cast<unsigned char*>(A.iso) + tp.off;
    const int M = tp.M, N = tp.N;
    auto diag = [&](int i, int j) {
      return ldz(U, i, j - 1, M, N) + ldz(U, i, j, M, N) + ldz(V, i - 1, j, M, N) + ldz(V, i, j, M, N);
    };
    march_points(tp, [&](int i, int j) {
      const size_t p = (size_t)i * N + j;
      const T d = diag(i, j);
      iso[p] = d == T(0) ? 1 : 0;
      T q = d;
      if (d == T(0)) {
        q = T(1);  // isolated pixel: identity row, output forced to zero
      } else if (ssor) {
        q = d / (T)omega;
      } else if ((i + j) & 1) {
        // couplings to the four (even) neighbours and their diagonals
        const T w[4] = {ldz(U, i, j - 1, M, N), ldz(U, i, j, M, N), ldz(V, i - 1, j, M, N),
                        ldz(V, i, j, M, N)};
        const int ni[4] = {i, i, i - 1, i + 1}, nj[4] = {j - 1, j + 1, j, j};
        T sub = T(0);
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (w[k] != T(0)) sub += w[k] * w[k] / diag(ni[k], nj[k]);
        q = d - sub;
        if (q < T(1e-4) * d) q = d;  // the pivot floor of the natural-order factorisation
      }
      piv[p] = q;
    });
  }
}

template <typename T, int PASS>
__global__ void __launch_bounds__(kMaxTileThreads) k_e_twocolor(EArgs A, T c) {
  __shared__ double lsum[64];
  __shared__ double fred[3 * kMaxTileWaves];
  __shared__ int fflag;
  TILE_LOOP(A) {
    const TileRef ref = TILE_REF(A);
    const TilePos tp = tile_pos(A.desc, ref);
    if (A.ms[tp.m].state != A.expect) continue;
    const T* U = cvec<T>(A.U, tp.off);
    const T* V = cvec<T>(A.V, tp.off);
    const T* piv = cvec<T>(A.aux, tp.off);
    const T* r = cvec<T>(A.r, tp.off);
    T* s = vec<T>(A.s, tp.off);
    const unsigned char* iso = A.iso + tp.off;
    TileSum<T, PASS, kOrdered<T>> ts(lsum);  // r^T s (pass 1)
    struct Op {
      T v, p;  // pass 0: r and the pivot; pass 1: s
    };
    struct Own {
      T r, p;  // pass 1
      unsigned char iso;
    };
    auto even = [](int i, int j) { return ((i + j) & 1) == 0; };
    stencil_tile<T>(
        tp, ts, U, V,
        [&](size_t row, unsigned j) {
          return Op{PASS == 0 ? r[row + j] : s[row + j], PASS == 0 ? piv[row + j] : T(1)};
        },
        [&](const Op& v, int i, int j) {
          if (PASS == 0) return even(i, j) ? v.v / v.p : T(0);
          return even(i, j) ? T(0) : v.v;
        },
        [&](size_t row, unsigned j) {
          return Own{PASS == 1 ? r[row + j] : T(0), PASS == 1 ? piv[row + j] : T(1), iso[row + j]};
        },
        [&](int i, size_t row, unsigned j, T xv, T ax, const Op& v, const Own& o) {
          if constexpr (PASS == 0) {
            if (!even(i, j)) s[row + j] = o.iso ? T(0) : c * (v.v - ax) / v.p;
            return Terms<T, 0>{};
          } else {
            T sv = xv;
            if (even(i, j)) {
              sv = o.iso ? T(0) : (c * o.r - ax) / o.p;
              s[row + j] = sv;
            }
            return Terms<T, 1>{{o.r}, {sv}};
          }
        });
    if constexpr (PASS == 1) {
      if (threadIdx.x == 0) store_partial(A.P + 1 * A.pstride + ref.g, ts.sum[0]);
      if (A.fin_mode) {
          const int sl[1] = {1};
        fused_finish<kFinTailS, 1, 64>(arrival(A), sl, ref.g - tp.local, tp.local, tp.ntiles, tp.gb, A.desc,
                                   A.ms, tp.m, A.fin_mode, 0, &fflag, fred);
      }
    }
  }
}

// y = A x for the step entry point (x in A.s, y in A.q)
template <typename T>
__global__ void __launch_bounds__(kMaxTileThreads) k_e_apply(EArgs A) {
  TILE_LOOP(A) {
    const TileRef ref = TILE_REF(A);
    const TilePos tp = tile_pos(A.desc, ref);
    const T* U = cvec<T>(A.U, tp.off);
    const T* V = cvec<T>(A.V, tp.off);
    const T* x = cvec<T>(A.s, tp.off);
    T* y = vec<T>(A.q, tp.off);
    TileSum<T, 0, false> ts(nullptr);
    stencil_tile<T>(
        tp, ts, U, V, [&](size_t row, unsigned j) { return x[row + j]; }, [](T v, int, int) { return v; },
        [](size_t, unsigned) { return 0; },
        [&](int, size_t row, unsigned j, T, T ax, T, int) {
          y[row + j] = ax;
          return Terms<T, 0>{};
        });
  }
}

// ---------------------------------------------------------------------------
// Finisher: one block per map, fixed-order sums of the map's partials, then
// the map's PCG state advances.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_e_finish(const MapDesc* __restrict__ desc, MapState* ms,
                                                  const double* __restrict__ P, long long pstride,
                                                  int op, int expect, int mode, int pointwise) {
  __shared__ double red[3 * 4];
  const int m = blockIdx.x;
  if (expect >= 0 && ms[m].state != expect) return;
  const FinSrc src{P, pstride, nullptr, 0, (int)blockDim.x};
  finish_map<false>(desc, ms, src, m, op, mode, pointwise, red);
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
// Grid of the tile kernels: the next power of two >= the active tiles, capped
// (blocks stride over the list, so any grid is correct; few distinct shapes
// keep captured graphs reusable as the active set shrinks).
int egrid(const Engine& e, int ntiles) {
  int g = 1;
  while (g < ntiles && g < e.grid) g <<= 1;
  return std::max(1, std::min(g, e.grid));
}

static int tile_threads(const Engine& e, int rows = kRW) {
  return 64 * std::min((e.th + rows - 1) / rows, kMaxTileWaves);
}

EArgs make_args(const Engine& e) {
  EArgs a;
  a.desc = e.desc;
  a.ms = e.ms;
  a.act = e.act;
  a.act_cap = (int)e.caps.tiles;
  a.counts = e.counts;
  a.P = e.P;
  a.pstride = e.pstride;
  a.U = e.U;
  a.V = e.V;
  a.aux = e.aux;
  a.x0 = e.x[0];
  a.x1 = e.x[1];
  a.d0 = e.d[0];
  a.d1 = e.d[1];
  a.r = e.r;
  a.s = e.s;
  a.q = e.q;
  a.b = e.b;
  a.dx = e.dx;
  a.dy = e.dy;
  a.phi_prev = e.phi_prev;
  a.r64 = e.r64;
  a.iso = e.iso;
  a.fcnt = e.fcnt;
  a.gcnt = e.gcnt;
  a.gsum = e.gsum;
  a.gstride = e.gstride;
  a.fuse_pw = -1;
  a.expect = kRun;
  a.fin_mode = 0;
  return a;
}

void e_wrapdiff(hipStream_t st, const Engine& e, int ntiles, bool zero_phi) {
  hipLaunchKernelGGL(k_e_wrapdiff, dim3(egrid(e, ntiles)), dim3(tile_threads(e)), 0, st, make_args(e),
                     zero_phi ? 1 : 0);
}

void e_check(hipStream_t st, const Engine& e, int ntiles, unsigned int* bad) {
  hipLaunchKernelGGL(k_e_check, dim3(egrid(e, ntiles)), dim3(tile_threads(e)), 0, st, make_args(e), bad);
}

template <typename T>
void e_weights(hipStream_t st, const Engine& e, int ntiles, double p, double tau) {
  hipLaunchKernelGGL(k_e_weights<T>, dim3(egrid(e, ntiles)), dim3(tile_threads(e)), 0, st, make_args(e),
                     2.0 - p, tau);
}

template <typename T>
void e_diag(hipStream_t st, const Engine& e, int ntiles, bool inv) {
  hipLaunchKernelGGL(k_e_diag<T>, dim3(egrid(e, ntiles)), dim3(tile_threads(e)), 0, st, make_args(e),
                     inv ? 1 : 0);
}

template <typename T>
void e_rhs(hipStream_t st, const Engine& e, int ntiles, int mode) {
  hipLaunchKernelGGL(k_e_rhs<T>, dim3(egrid(e, ntiles)), dim3(tile_threads(e)), 0, st, make_args(e), mode);
}

template <typename T>
void e_pass(hipStream_t st, const Engine& e, int ntiles, int op) {
  hipLaunchKernelGGL(k_e_pass<T>, dim3(egrid(e, ntiles)), dim3(tile_threads(e)), 0, st, make_args(e), op);
}

template <typename T, int PC>
static void e_resid_pc(hipStream_t st, const Engine& e, int ntiles, bool confirm) {
  if (confirm)
    hipLaunchKernelGGL((k_e_resid<T, PC, 1>), dim3(egrid(e, ntiles)), dim3(tile_threads(e)), 0, st,
                       make_args(e));
  else
    hipLaunchKernelGGL((k_e_resid<T, PC, 0>), dim3(egrid(e, ntiles)), dim3(tile_threads(e)), 0, st,
                       make_args(e));
}

template <typename T>
void e_resid(hipStream_t st, const Engine& e, int ntiles, int pc, bool confirm) {
  if (pc == kPcJacobi) e_resid_pc<T, kPcJacobi>(st, e, ntiles, confirm);
  else e_resid_pc<T, kPcNone>(st, e, ntiles, confirm);
}

template <typename T, int PC>
static void e_spmv_pc(hipStream_t st, const Engine& e, int gr, int fuse_pw) {
  EArgs a = make_args(e);
  a.fuse_pw = fuse_pw;
  hipLaunchKernelGGL((k_e_spmv<T, PC>), dim3(gr), dim3(tile_threads(e)), 0, st, a);
}

// fused: the launch also runs the per-map finisher of its partials (alpha
// after the SpMV, the update's stop tests and pointwise beta after the update)
template <typename T>
void e_spmv(hipStream_t st, const Engine& e, int ntiles, int pc, bool fused) {
  const int gr = egrid(e, ntiles);
  const int pw = pc == kPcNone || pc == kPcJacobi ? 1 : 0;
  const int f = fused ? pw : -1;
  if (pc == kPcNone) e_spmv_pc<T, kPcNone>(st, e, gr, f);
  else if (pc == kPcJacobi) e_spmv_pc<T, kPcJacobi>(st, e, gr, f);
  else e_spmv_pc<T, kPcDct>(st, e, gr, f);
}

template <typename T, int PC>
static void e_update_pc(hipStream_t st, const Engine& e, int gr, int fuse_pw) {
  EArgs a = make_args(e);
  a.fuse_pw = fuse_pw;
  hipLaunchKernelGGL((k_e_update<T, PC>), dim3(gr), dim3(tile_threads(e, kRWUpdate)), 0, st, a);
}

template <typename T>
void e_update(hipStream_t st, const Engine& e, int ntiles, int pc, bool fused) {
  const int gr = egrid(e, ntiles);
  const int pw = pc == kPcNone || pc == kPcJacobi ? 1 : 0;
  const int f = fused ? pw : -1;
  if (pc == kPcJacobi) e_update_pc<T, kPcJacobi>(st, e, gr, f);
  else e_update_pc<T, kPcNone>(st, e, gr, f);
}

template <typename T>
void e_tc_pivots(hipStream_t st, const Engine& e, int ntiles, bool ssor, double omega) {
  hipLaunchKernelGGL(k_e_tc_pivots<T>, dim3(egrid(e, ntiles)), dim3(tile_threads(e)), 0, st, make_args(e),
                     ssor ? 1 : 0, omega);
}

template <typename T, int PASS>
static void e_twocolor_pass(hipStream_t st, const Engine& e, int gr, const EArgs& a, T c) {
  hipLaunchKernelGGL((k_e_twocolor<T, PASS>), dim3(gr), dim3(tile_threads(e)), 0, st, a, c);
}

// s = M^-1 r of the two-colour preconditioner for the maps in state `expect`;
// fin_mode != 0 runs the per-map finisher of r^T s at the end of the second pass
template <typename T>
void e_twocolor(hipStream_t st, const Engine& e, int ntiles, int expect, bool ssor, double omega,
                int fin_mode) {
  const int gr = egrid(e, ntiles);
  EArgs a = make_args(e);
  a.expect = expect;
  const T c = ssor ? (T)(2.0 - omega) : T(1);
  e_twocolor_pass<T, 0>(st, e, gr, a, c);
  a.fin_mode = fin_mode;
  e_twocolor_pass<T, 1>(st, e, gr, a, c);
}

template <typename T>
void e_apply(hipStream_t st, const Engine& e, int ntiles) {
  hipLaunchKernelGGL(k_e_apply<T>, dim3(egrid(e, ntiles)), dim3(tile_threads(e)), 0, st, make_args(e));
}

void e_finish(hipStream_t st, const Engine& e, int op, int expect, int mode, bool pointwise) {
  hipLaunchKernelGGL(k_e_finish, dim3(e.n_maps), dim3(256), 0, st, e.desc, e.ms, e.P, e.pstride,
                     op, expect, mode, pointwise ? 1 : 0);
}

#define LPU_INST_E(T)                                                                   \
  template void e_weights<T>(hipStream_t, const Engine&, int, double, double);         \
  template void e_diag<T>(hipStream_t, const Engine&, int, bool);                      \
  template void e_rhs<T>(hipStream_t, const Engine&, int, int);                        \
  template void e_pass<T>(hipStream_t, const Engine&, int, int);                       \
  template void e_resid<T>(hipStream_t, const Engine&, int, int, bool);                \
  template void e_spmv<T>(hipStream_t, const Engine&, int, int, bool);                       \
  template void e_update<T>(hipStream_t, const Engine&, int, int, bool);                     \
  template void e_apply<T>(hipStream_t, const Engine&, int);                            \
  template void e_tc_pivots<T>(hipStream_t, const Engine&, int, bool, double);         \
  template void e_twocolor<T>(hipStream_t, const Engine&, int, int, bool, double, int);
LPU_INST_E(float)
LPU_INST_E(double)

}  // namespace lpu
