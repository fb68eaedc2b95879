// Natural-order ILU(0) = IC(0) and SSOR preconditioners (Section 2.1's list,
// items 3-5) across the whole device.
//
// With P the pivots and L the strict lower part of A (entries -U west, -V
// north), M = (P + L) P^{-1} (P + L^T) (times 1/(2 - omega) for SSOR, where
// P = D/omega), so s = M^{-1} r is
//   forward : y_ij = (r_ij + V_{i-1,j} y_{i-1,j} + U_{i,j-1} y_{i,j-1}) / p_ij
//   backward: z_ij = y_ij + (U_ij z_{i,j+1} + V_ij z_{i+1,j}) / p_ij,  s = c z
// (c = 2 - omega for SSOR, 1 otherwise), and the ILU(0) pivots are
//   p_ij = a_ij - U_{i,j-1}^2 / p_{i,j-1} - V_{i-1,j}^2 / p_{i-1,j}
// (a_ij the diagonal of A; below 1e-4 a_ij the pivot falls back to a_ij; an
// isolated pixel, a_ij = 0, gets 1).  The factorisation stores 1 / p_ij, once
// per outer step, so the solves multiply.
//
// Each value depends on its west and north neighbours (east and south for the
// backward solve, which is the forward recurrence on the map rotated by 180
// degrees), so a solve is a chain of M + N - 1 dependent pixels and its time
// is that chain's: the map is cut into strips of 64 rows, one workgroup each,
// and a strip is swept from left to right by ONE wave, lane l on row l, in
// steps: at step k lane l computes column k - l.  The north neighbour is lane
// l - 1's value of the previous step (a DPP lane shift), the west one the
// lane's own.  Everything else is kept off that wave:
//  * four loader waves, each with a quarter of the rows, bring the operands of a
//    chunk of steps at a time from memory, three to five chunks ahead, and write
//    them into an LDS ring indexed by step, so the sweeping wave reads 64
//    consecutive entries at an immediate offset, eight steps ahead of their use;
//  * two storer waves take its results from LDS back to rows in memory (the
//    backward ones form s and the partial of r^T s as they pass);
//  * the strip's last row goes to the strip below as it is made: every value
//    is published with a tag, the launch's epoch, in the same 8-byte word (two
//    words for a double), so the one wave that waits for it in the next
//    strip's workgroup polls the data itself and needs no flag or fence.
// The eight waves meet at one barrier per chunk.  Strips run concurrently,
// each some 150 to 200 steps behind the one above it.
//
// What one workgroup can bring from memory sets the pace (a compute unit gets
// about 50 GB/s of misses), so nothing is fetched twice: a chunk is 16 steps, and
// a row's share of it is one aligned run of 16 elements, the one whose first
// element is due within the chunk's steps: a 128-byte line of doubles, or half a
// line of floats (the other half follows from the caches a chunk later).  At 16
// bytes per lane an instruction brings 8 rows (floats: 16).
//
// Progress: workgroups take strips from a ticket counter, in an order in which
// a strip's predecessor always has the smaller ticket, so the strip a
// workgroup waits for is finished or held by a workgroup that already runs,
// whatever the number of resident workgroups.  The wait is bounded all the
// same; a strip whose wait runs out goes on with NaN, which ends that map's
// solve as a breakdown, and says so in a word that the calls that wait for the
// device read (WArgs::ctl).
//
// Measured (960 x 1280 FP64; 840 x 1120 FP32): a forward solve 143 and 105 us,
// a backward one 148 and 112 us, the pivots 286 and 213 us, where one launch
// per anti-diagonal of 64 x 64 tiles took 34 x 14.7 us and 31 x 13.4 us for a
// solve and 1290 and 1020 us for the pivots.  A chunk of 16 steps takes 0.5 us
// (FP32) to 0.75 us (FP64), nearly all of it the sweeping wave's (76 and 105
// cycles a step forward; leaving out any one of its LDS reads, its writes or the
// lane shift saves 3 to 7 %), and a strip starts 5 to 6 us after the one above
// it: 80 steps it must wait (64 of skew and the chunk), two chunks of
// look-ahead, and the trip of the last row's values through memory.

#include <type_traits>

#include "lpu_internal.h"
#include "lpu_device.h"
#include "lpu_finish.h"

namespace lpu {

constexpr int kWT = 64;                 // rows of a strip (lanes of the sweeping wave)
constexpr int kWLoad = 4, kWStore = 2;  // loader and storer waves
constexpr int kWThreads = 64 * (2 + kWLoad + kWStore);
constexpr int kWRing = 4;    // chunks of operands in LDS: in use, next, and the two a write spans
constexpr int kWOut = 3;     // chunks of results: in work, and the two a store spans
constexpr int kWAhead = 8;   // steps between reading a step's operands and using them
constexpr int kWHeld = 3;    // chunks a loader or storer wave holds in registers
constexpr int kWPitch = kWT + 1;  // LDS entries per step (an element's row + 1 is a valid entry)
constexpr int kWMaxGrid = 512;

// flags of a launch: SSOR's scale 2 - omega; give up every wait at its first poll (tests)
enum : int { kWSsor = 1, kWNoWait = 2 };

enum SweepMode : int { kWPivots = 0, kWForward = 1, kWBackward = 2 };

struct WArgs {
  const MapDesc* desc;
  MapState* ms;
  const int* slist;   // (map, strip) pairs of the active maps, predecessors first
  const int* mact;
  const int* counts;
  double* P;
  long long pstride;
  const void *U, *V, *piv, *r;
  void *s, *y;
  unsigned int* ctl;         // ticket, workgroups done, launches so far; from kSweepLostAt on the
                             // address of the host word to set when a wait is given up, or null
  unsigned long long* edge;  // tagged last rows of the strips
  int *fcnt, *gcnt;          // arrival counters of the fused finisher
  double* gsum;
  long long gstride;
  int expect;    // state of the maps to work on (-1: every active map)
  int fin_mode;  // backward: FinishMode of the fused finisher of r^T s (0: none)
  int recip;     // pivots: store 1 / p (what the solves read) instead of p
  double omega;
  int flags;     // kWSsor, kWNoWait
};

// DPP whole-wave shift with a fill: lane l receives lane l-1's v, lane 0 keeps
// its own value of fill.
__device__ __forceinline__ int wshr_fill(int fill, int v) {
  return __builtin_amdgcn_update_dpp(fill, v, 0x138, 0xF, 0xF, false);
}
__device__ __forceinline__ float from_prev_lane(float fill, float v) {
  return __builtin_bit_cast(float, wshr_fill(__builtin_bit_cast(int, fill), __builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double from_prev_lane(double fill, double v) {
  const long long f = __builtin_bit_cast(long long, fill), b = __builtin_bit_cast(long long, v);
  const int lo = wshr_fill((int)(f & 0xffffffffLL), (int)(b & 0xffffffffLL));
  const int hi = wshr_fill((int)(f >> 32), (int)(b >> 32));
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ double wf_wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Quotients of the pivot recurrence.  Both a pivot's quotients (by the pivot
// to its west and by the one to its north) divide by a value some lane formed
// one step earlier, so that lane forms its reciprocal once, and the shift
// brings it along with the pivot.  rcp_full: 1 / b (the hardware's estimate and two
// Newton steps).  quot: a / b as the division operator rounds it.
//  * float: the product in double, whose error of 2^-51 cannot reach across a rounding
//    boundary of a normal 24-bit quotient (2^-49 away at least).  A subnormal quotient
//    is too small to count: its diagonal is at least the coupling, and a coupling
//    whose square is not 0 is above 2^-75.
//  * double: the steps by which the operator itself is carried out here (product with
//    the reciprocal, then q + r (a - b q): Markstein, IBM J. Res. Dev. 34, 1990), but
//    without its scaling, so as long as nothing leaves the normal range.  Couplings of
//    Eq. (6) are at most 1.  With every coupling 0 or in 2^-300 .. 2^300 a pivot lies
//    between kPivotFloor times the least and four times the largest, and squares,
//    quotients, reciprocals and residuals are normal numbers.  A strip that meets
//    another coupling, or a pivot above it outside that range, divides by the operator
//    from there on (840 x 1120: 313 us for the pivots where the reciprocals take 260).
__device__ __forceinline__ double rcp_full(double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = __builtin_fma(__builtin_fma(-b, r, 1.0), r, r);
  return __builtin_fma(__builtin_fma(-b, r, 1.0), r, r);
}
__device__ __forceinline__ float quot(float a, float, double r) { return (float)((double)a * r); }
__device__ __forceinline__ double quot(double a, double b, double r) {
  const double q = a * r;
  return __builtin_fma(__builtin_fma(-b, q, a), r, q);
}

// Whether every value seen is 0 or a double within 2^-300 .. 2^300 (SLACK: 2^-(300 +
// SLACK) .. 2^(300 + SLACK)), from the high words: the least and the largest.
struct PlainRange {
  unsigned int least = 0x3ff00000u, most = 0x3ff00000u;
  __device__ __forceinline__ void see(double x) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const unsigned int h = b == 0 ? 0x3ff00000u : (unsigned int)(b >> 32);
    least = min(least, h);
    most = max(most, h);  // (a negative value or a NaN is large)
  }
  template <int SLACK = 0>
  __device__ __forceinline__ bool holds() const {
    return least >= (1023u - 300u - SLACK) << 20 && most < (1023u + 300u + SLACK) << 20;
  }
};

// A value of a strip's last row with its launch's tag: one 8-byte word for a
// float, two (low and high half) for a double.  Words are single agent-coherent
// accesses, so a word whose tag matches holds its value.
__device__ __forceinline__ void edge_put(unsigned long long* p, unsigned int tag, float v) {
  const unsigned long long w = ((unsigned long long)tag << 32) | __builtin_bit_cast(unsigned int, v);
  __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void edge_put(unsigned long long* p, unsigned int tag, double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v), t = (unsigned long long)tag << 32;
  __hip_atomic_store(p, t | (b & 0xffffffffULL), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(p + 1, t | (b >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The words of one value as read, and the value once every tag matches.
template <typename T>
struct Edge {
  unsigned long long w[sizeof(T) / 4];
  __device__ __forceinline__ void read(const unsigned long long* p) {
#pragma unroll
    for (int k = 0; k < (int)sizeof(T) / 4; ++k)
      w[k] = __hip_atomic_load(p + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ bool ready(unsigned int tag) const {
    bool ok = true;
#pragma unroll
    for (int k = 0; k < (int)sizeof(T) / 4; ++k) ok = ok && (unsigned int)(w[k] >> 32) == tag;
    return ok;
  }
  __device__ __forceinline__ T value() const {
    if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, (unsigned int)w[0]);
    else return __builtin_bit_cast(T, (w[1] << 32) | (w[0] & 0xffffffffULL));
  }
};

template <typename T>
struct alignas(2 * sizeof(T)) Pair {
  T a, b;
};

// The lane, opaque: what a role derives from it is formed in that role, not
// ahead of the branch to it for every role at once.
__device__ __forceinline__ int wf_lane() {
  int l = threadIdx.x & 63;
  __asm__ volatile("" : "+v"(l));
  return l;
}

// A wave-uniform value read from memory, in scalar registers.
__device__ __forceinline__ long long wf_uniform(long long v) {
  const unsigned int lo = __builtin_amdgcn_readfirstlane((int)(v & 0xffffffffLL));
  return ((long long)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) | lo;
}

// Every wave of the workgroup, at whatever place in its own role's loop.
__device__ __forceinline__ void wf_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Sizes per element type: C steps of a chunk, V elements of 16 bytes, L lanes
// for a row's share of a chunk, H rows per instruction (a group), GL and GS
// groups per loader and storer wave, R steps of the operand ring.
template <typename T>
struct WSize {
  static constexpr int C = 16, V = 16 / sizeof(T), L = C / V, H = 64 / L;
  static constexpr int GL = kWT / H / kWLoad, GS = kWT / H / kWStore, R = kWRing * C;
};
template <typename T>
using wvec = T __attribute__((ext_vector_type(16 / sizeof(T)), aligned(sizeof(T))));

// The elements of chunk q that a lane of a loader or storer wave handles: in
// group g of its G, the 16 bytes (l mod L) of row H (g0 + g) + l / L's run of C
// elements.  Along the sweep
// the run starts at column q C + dl - row, i.e. at step q C + dl with
// dl = 0 .. C - 1 such that it is aligned in memory.  at[g]: offset of
// the lane's 16 bytes at q = 0 from the strip's base; it moves C per chunk
// with the sweep.  Rows past the map take row 0's place (and are dropped).
template <typename T, bool REV, int G>
struct WLanes {
  int dl[G];
  unsigned int at[G];
  int lr, sub;  // row of group 0, first element within the run

  __device__ __forceinline__ WLanes(int l, int g0, int rows, int N, long long base) {
    constexpr int C = WSize<T>::C, V = WSize<T>::V, L = WSize<T>::L, H = WSize<T>::H;
    lr = H * g0 + l / L;
    sub = l % L * V;
    // element index (mod C) of the strip's first pixel along the sweep
    const int e0 = (int)((REV ? base + (long long)kWT * N - 1 : base) & (C - 1));
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int r = H * g + lr, row = r < rows ? r : 0;
      dl[g] = (REV ? row + e0 - row * N + 1 : row - e0 - row * N) & (C - 1);
      at[g] = REV ? (unsigned int)((kWT - row) * N + row - dl[g] - sub - V)
                  : (unsigned int)(row * N - row + dl[g] + sub);
    }
  }
  __device__ __forceinline__ int row(int g) const { return WSize<T>::H * g + lr; }
  // step (counted from chunk q's first) and column of the lane's element e
  __device__ __forceinline__ int step(int g, int e) const { return dl[g] + sub + e; }
  __device__ __forceinline__ int col(int q, int g, int e) const {
    return q * WSize<T>::C + step(g, e) - row(g);
  }
  // Keeps what the accessors derive from being held in registers across the
  // whole sweep (it is cheaper to form again per chunk than to spill).
  __device__ __forceinline__ void fresh() { __asm__ volatile("" : "+v"(lr), "+v"(sub)); }
  // element e of a vector in memory order
  static __device__ __forceinline__ int mem(int e) { return REV ? WSize<T>::V - 1 - e : e; }
};

// Whether every lane's 16 bytes of chunk q lie in the map's array (they may
// reach into neighbouring rows): all but chunk -1 of the first strip and the
// last few chunks of the last strip (or strips, on maps a few pixels wide).
// wf_last: the last such chunk.
template <typename T>
__device__ __forceinline__ int wf_last(int strip, int rows, int M, int N) {
  constexpr int C = WSize<T>::C;
  const long long room = (long long)(M - strip * kWT - rows + 1) * N + (rows - 1) - 2 * C;
  return room < 0 ? -2 : (int)min(room / C, (long long)1 << 20);
}

// Whether every element of chunk q and its east neighbour lie in the map's
// strip.
template <typename T>
__device__ __forceinline__ bool wf_inner(int q, int rows, int N) {
  constexpr int C = WSize<T>::C;
  return rows == kWT && q * C >= kWT - 1 && (q + 2) * C < N;
}

// ---------------------------------------------------------------------------
// The pivots, the forward solve (P + L) y = r or the backward solve
// (P + L^T) z = P y with s = c z and the strips' partials of r^T s.
//   Operands of a step, as two pairs per lane:
//     pivots   {U, V}, {U_west, V_north}
//     forward  {r, 1 / p}, {U_west, V_north}
//     backward {y, 1 / p}, {U, V}
// (a loader writes an element's U as its row's west coupling of the next step
// and its V as the next row's north coupling of that step).  Off the map they are 0 (1 / p:
// 1), which keeps every value there from reaching a pixel of the map, so the
// sweeping wave has no conditions.
// ---------------------------------------------------------------------------
template <typename T, int MODE>
__global__ void __launch_bounds__(kWThreads, sizeof(T) == 8 ? 2 : 4) k_wf_sweep(WArgs a) {
  using W = WSize<T>;
  constexpr int C = W::C, V16 = W::V, kGL = W::GL, kGS = W::GS;
  __shared__ Pair<T> pa[W::R][kWPitch], pb[W::R][kWPitch];
  __shared__ T yo[kWOut * C][kWPitch];  // results
  __shared__ T yb[W::R];                // the row above the strip
  __shared__ double yr[MODE == kWPivots ? W::R : 1];  // pivots: its reciprocals
  __shared__ double red[kWThreads / 64 * 3];
  __shared__ int sh_ticket, fflag;
  __shared__ int sh_divide;  // kWatch: the strip met a value outside PlainRange
  constexpr T kOff = MODE == kWPivots ? T(1) : T(0);  // value off the map
  constexpr bool kRev = MODE == kWBackward;           // the sweep runs from the map's last pixel
  constexpr bool kWatch = MODE == kWPivots && sizeof(T) == 8;  // see quot
  constexpr int kWords = sizeof(T) / 4;               // words of an edge entry
  const int tid = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_strips = a.counts[4];
  const unsigned int tag = a.ctl[2] + 1u;
  const bool one_each = (int)gridDim.x >= n_strips;
  for (;;) {
    if (tid == 0) {
      if (kWatch) sh_divide = 0;
      sh_ticket = (int)__hip_atomic_fetch_add(a.ctl, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    const int tk = __builtin_amdgcn_readfirstlane(sh_ticket);
    if (tk >= n_strips) break;
    const int m = __builtin_amdgcn_readfirstlane(a.slist[2 * tk]);
    const int strip = __builtin_amdgcn_readfirstlane(a.slist[2 * tk + 1]);
    const MapDesc& d = a.desc[m];
    const int M = __builtin_amdgcn_readfirstlane(d.M), N = __builtin_amdgcn_readfirstlane(d.N);
    const int state = a.ms[m].state;
    if (a.expect < 0 || state == a.expect) {
      const int n_map = (M + kWT - 1) / kWT;  // strips of this map
      const int rows = min(kWT, M - strip * kWT);
      const int nc = (N + kWT - 1 + C - 1) / C;
      // the strip's base: offsets are row * N + column (backward: counted from
      // the first pixel of the strip's 64 rows in memory; the base may lie
      // before the map, no accessed element does)
      const long long base =
          wf_uniform(d.off) + (kRev ? (long long)(M - (strip + 1) * kWT) : (long long)strip * kWT) * N;
      const int q_last = wf_last<T>(strip, rows, M, N);
      auto in_array = [&](int q) { return (q >= 0 || strip > 0) && q <= q_last; };
      unsigned long long* edge = a.edge + wf_uniform(d.edge0) + (size_t)strip * N * 2;
      double part = 0.0;

      // Roles: wave 0 sweeps, waves 1..3 and 5 load, wave 4 polls (it shares
      // wave 0's SIMD and has the least to issue), waves 6 and 7 store.  At
      // iteration n chunk n is swept, chunk n + 2 written to LDS (its lines
      // reach into chunk n + 3's steps) and the lines that end in chunk n - 1
      // stored.
      // The second wave of a SIMD (5 to 7) would fall behind the first, which is
      // the older one, and a chunk waits for the last wave: with priority over
      // the first the solves take 3 to 6 % less (840 x 1120 FP64 SSOR apply 318
      // against 300 us, FP32 270 / 257).
      if (wv >= 5) __builtin_amdgcn_s_setprio(1);
      if (wv == 0) {
        const int l = wf_lane();
        wf_barrier();
        __builtin_amdgcn_s_setprio(3);
        T own = kOff;
        Pair<T> oa[kWAhead], ob[kWAhead];
        T of[kWAhead];
        double rown = 1.0, orf[kWAhead];  // pivots: 1 / own, and of the row above
#pragma unroll
        for (int u = 0; u < kWAhead; ++u) {
          oa[u] = pa[u][l], ob[u] = pb[u][l], of[u] = yb[u];
          if (MODE == kWPivots) orf[u] = yr[u];
        }
        int b = 0, ob3 = 0;
        auto chunk = [&](auto divide) {
          const int bn = (b + C) & (W::R - 1);
#pragma unroll
          for (int u = 0; u < C; ++u) {
            const int k = u % kWAhead;
            const T up = from_prev_lane(of[k], own);  // lane 0: the row above the strip
            T v;
            if (MODE == kWPivots) {
              const T uw = ob[k].a, vn = ob[k].b;
              const T av = uw + oa[k].a + vn + oa[k].b;
              v = av;
              T qw, qn;
              if constexpr (decltype(divide)::value) {
                qw = uw * uw / own;
                qn = vn * vn / up;
              } else {
                const double rup = from_prev_lane(orf[k], rown);
                qw = quot(uw * uw, own, rown);
                qn = quot(vn * vn, up, rup);
              }
              v = uw != T(0) ? v - qw : v;
              v = vn != T(0) ? v - qn : v;
              if (v < (T)kPivotFloor * av) v = av;
              if (av == T(0)) v = T(1);
              rown = rcp_full((double)v);
            } else if (MODE == kWForward) {
              v = fma_t(ob[k].a, own, fma_t(ob[k].b, up, oa[k].a)) * oa[k].b;
            } else {
              v = fma_t(fma_t(ob[k].a, own, ob[k].b * up), oa[k].b, oa[k].a);
            }
            yo[ob3 + u][l] = v;
            own = v;
            const int f = (u + kWAhead) % C, fb = u + kWAhead < C ? b : bn;
            oa[k] = pa[fb + f][l];
            ob[k] = pb[fb + f][l];
            of[k] = yb[fb + f];
            if (MODE == kWPivots) orf[k] = yr[fb + f];
          }
          b = bn;
          ob3 = ob3 == (kWOut - 1) * C ? 0 : ob3 + C;
        };
        // a value outside the range is seen two chunks before its use; the flag is
        // read a chunk ahead, and stays up to the strip's end
        int n = 0, divide = kWatch ? __builtin_amdgcn_readfirstlane(sh_divide) : 0;
        for (; n < nc && !divide; ++n) {
          const int next = kWatch ? sh_divide : 0;
          if (kWatch) __asm__ volatile("" ::: "memory");
          chunk(std::false_type{});
          if (kWatch) divide = __builtin_amdgcn_readfirstlane(next);
          wf_barrier();
        }
        for (; kWatch && n < nc; ++n) {
          chunk(std::true_type{});
          wf_barrier();
        }
        __builtin_amdgcn_s_setprio(0);
        wf_barrier();
        wf_barrier();
      } else if (wv < 4 || wv == 5) {
        const int l = wf_lane();
        // raw operands of a chunk, held from the load to the write
        struct Held {
          wvec<T> f[4][kGL];
        };
        Held h0{}, h1{}, h2{};
        const T* U = reinterpret_cast<const T*>(a.U) + base;
        const T* V = reinterpret_cast<const T*>(a.V) + base;
        const T* P = reinterpret_cast<const T*>(a.piv) + base;
        const T* R = reinterpret_cast<const T*>(kRev ? a.y : a.r) + base;
        WLanes<T, kRev, kGL> ln(l, (wv == 5 ? 3 : wv - 1) * kGL, rows, N, base);
        // (past the last chunk the last one is loaded again: every iteration
        // issues as many loads, or the wait for a chunk's would have to cover
        // the chunks requested after it as well)
        auto load = [&](auto fast, int q, Held& h) {
          q = min(q, nc - 1);
          ln.fresh();
          const long long qo = kRev ? -(long long)q * C : (long long)q * C;
          if (decltype(fast)::value || in_array(q)) {
#pragma unroll
            for (int g = 0; g < kGL; ++g) {
              h.f[2][g] = *reinterpret_cast<const wvec<T>*>(U + qo + ln.at[g]);
              h.f[3][g] = *reinterpret_cast<const wvec<T>*>(V + qo + ln.at[g]);
              if (MODE != kWPivots) {
                h.f[0][g] = *reinterpret_cast<const wvec<T>*>(R + qo + ln.at[g]);
                h.f[1][g] = *reinterpret_cast<const wvec<T>*>(P + qo + ln.at[g]);
              }
            }
            return;
          }
#pragma unroll
          for (int g = 0; g < kGL; ++g) {
#pragma unroll
            for (int e = 0; e < V16; ++e) {
              const int row = ln.row(g), c = ln.col(q, g, e), x = ln.mem(e);
              const bool ok = row < rows && (unsigned)c < (unsigned)N;
              // row 0 column 0 of the strip for the elements off the map
              const int rw = ok ? row : 0, cl = ok ? c : 0;
              const unsigned int o = kRev ? (kWT - 1 - rw) * N + (N - 1 - cl) : rw * N + cl;
              h.f[2][g][x] = U[o];
              h.f[3][g][x] = V[o];
              if (MODE != kWPivots) {
                h.f[0][g][x] = R[o];
                h.f[1][g][x] = P[o];
              }
            }
          }
        };
        auto stash = [&](int q, const Held& h) {
          if (q >= nc) return;
          ln.fresh();
          const bool inner = wf_inner<T>(q, rows, N);
          PlainRange seen;
#pragma unroll
          for (int g = 0; g < kGL; ++g) {
#pragma unroll
            for (int e = 0; e < V16; ++e) {
              const int row = ln.row(g), c = ln.col(q, g, e), x = ln.mem(e);
              const int at = (q * C + ln.step(g, e)) & (W::R - 1);
              T u = h.f[2][g][x], v = h.f[3][g][x], w = u;
              Pair<T> p;
              if (MODE != kWPivots) p = {h.f[0][g][x], h.f[1][g][x]};
              if (!inner) {
                const bool ok = row < rows && (unsigned)c < (unsigned)N;
                u = ok ? u : T(0);
                v = ok ? v : T(0);
                w = c < N - 1 ? u : T(0);
                p = {ok ? p.a : T(0), ok ? p.b : T(1)};
              }
              if (kWatch) seen.see(u), seen.see(v);
              if (kRev) {
                pa[at][row] = p;
                pb[at][row] = {u, v};
              } else {
                pa[at][row] = MODE == kWPivots ? Pair<T>{u, v} : p;
                const int next = (at + 1) & (W::R - 1);
                pb[next][row].a = w;
                pb[next][row + 1].b = v;
              }
            }
          }
          if (kWatch && !seen.holds()) sh_divide = 1;
        };
        // lines of chunk -1 reach into chunk 0's steps
        const std::false_type any{};
        load(any, -1, h0);
        load(any, 0, h1);
        load(any, 1, h2);
        stash(-1, h0);
        load(any, 2, h0);
        stash(0, h1);
        load(any, 3, h1);
        stash(1, h2);
        load(any, 4, h2);
        wf_barrier();
        int n = 0;
        auto iteration = [&](auto fast, Held& h) {
          stash(n + 2, h);
          load(fast, n + 2 + kWHeld, h);
          wf_barrier();
          return n++ < nc + 1;
        };
        // with no other form of load in the loop, the wait for a chunk leaves
        // the two requested after it in flight
        const std::true_type fast{};
        const int n_fast = q_last >= nc - 1 ? nc + 2 : q_last - (2 + kWHeld) + 1;
        while (n + kWHeld <= n_fast) {
          iteration(fast, h0);
          iteration(fast, h1);
          iteration(fast, h2);
        }
        while (n <= nc + 1 && iteration(any, h0) && iteration(any, h1) && iteration(any, h2)) {
        }
      } else if (wv == 4) {
        const int l = wf_lane();
        // the strip above's last row: its values, and the couplings to it.  A
        // chunk's are requested an iteration before they are looked at (a
        // round trip), and asked for again until they are there.
        const unsigned long long* above = edge - (size_t)N * 2;
        const T* Va = reinterpret_cast<const T*>(a.V) + base - N;
        bool lost = false;
        const int k0 = (a.flags & kWNoWait) ? kSweepPolls : 0;
        Edge<T> ew;
        T vn = T(0);
        // the column of this lane in chunk q, or a valid one (whose values are
        // not used) for lanes without any
        auto column = [&](int q) { return min(q * C + min(l, C - 1), N - 1); };
        auto request = [&](int q) {
          if (strip == 0) return;
          ew.read(above + (size_t)column(q) * kWords);
          if (!kRev) vn = Va[column(q)];
        };
        auto take = [&](int q) {
          const int c = q * C + l;
          const bool mine = strip > 0 && l < C && c < N;
          T v = kOff;
          if (strip > 0) {
            bool need = mine;
            for (int k = k0;; ++k) {
              if (need && ew.ready(tag)) v = ew.value(), need = false;
              if (__builtin_amdgcn_ballot_w64(need) == 0) break;
              if (lost || k >= kSweepPolls) {
                if (need) v = T(__builtin_nanf(""));
                lost = true;
                break;
              }
              ew.read(above + (size_t)column(q) * kWords);
            }
          }
          if (l < C) {
            yb[c & (W::R - 1)] = v;
            if (MODE == kWPivots) yr[c & (W::R - 1)] = rcp_full((double)v);
            if (kWatch && mine) {
              PlainRange seen, above;
              seen.see(vn);
              above.see(v);
              if (!seen.holds() || !above.template holds<16>()) sh_divide = 1;
            }
            if (!kRev) pb[c & (W::R - 1)][0].b = mine ? vn : T(0);
          }
        };
        request(0);
        take(0);
        request(1);
        take(1);
        request(2);
        wf_barrier();
        for (int n = 0; n <= nc + 1; ++n) {
          if (n + 2 < nc) {
            take(n + 2);
            request(n + 3);
          }
          wf_barrier();
        }
        if (lost) {
          int* const word = *reinterpret_cast<int* const*>(a.ctl + kSweepLostAt);
          if (word) __hip_atomic_store(word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
      } else {
        const int l = wf_lane(), st = wv - 6;
        struct Held {
          wvec<T> r[kGS];
        };
        Held h0{}, h1{}, h2{};  // backward: r of the lines to store next
        const T* R = reinterpret_cast<const T*>(a.r) + base;
        T* out = reinterpret_cast<T*>(MODE == kWPivots ? const_cast<void*>(a.piv)
                                                       : (kRev ? a.s : a.y)) + base;
        const T scale = (a.flags & kWSsor) ? (T)(2.0 - a.omega) : T(1);
        WLanes<T, kRev, kGS> ln(l, st * kGS, rows, N, base);
        auto load_r = [&](auto fast, int q, Held& h) {
          if (!kRev) return;
          q = min(q, nc - 1);  // every iteration issues as many loads
          ln.fresh();
          const long long qo = -(long long)q * C;
          if (decltype(fast)::value || in_array(q)) {
#pragma unroll
            for (int g = 0; g < kGS; ++g)
              h.r[g] = *reinterpret_cast<const wvec<T>*>(R + qo + ln.at[g]);
            return;
          }
#pragma unroll
          for (int g = 0; g < kGS; ++g) {
#pragma unroll
            for (int e = 0; e < V16; ++e) {
              const int row = ln.row(g), c = ln.col(q, g, e);
              const bool ok = row < rows && (unsigned)c < (unsigned)N;
              const int rw = ok ? row : 0, cl = ok ? c : 0;
              h.r[g][ln.mem(e)] = R[(unsigned int)((kWT - 1 - rw) * N + (N - 1 - cl))];
            }
          }
        };
        auto store = [&](int q, const Held& h) {
          ln.fresh();
          const long long qo = kRev ? -(long long)q * C : (long long)q * C;
          const bool inner = wf_inner<T>(q, rows, N);
          const int first = (q + kWOut) % kWOut * C;  // ring place of chunk q's first step
          wvec<T> w[kGS];  // all reads before the first store
#pragma unroll
          for (int g = 0; g < kGS; ++g) {
#pragma unroll
            for (int e = 0; e < V16; ++e) {
              int at = first + ln.step(g, e);
              at -= at >= kWOut * C ? kWOut * C : 0;
              w[g][ln.mem(e)] = yo[at][ln.row(g)];
            }
          }
#pragma unroll
          for (int g = 0; g < kGS; ++g) {
            if (MODE == kWPivots && a.recip) w[g] = T(1) / w[g];
            if (kRev) w[g] *= scale;
          }
          if (inner) {
#pragma unroll
            for (int g = 0; g < kGS; ++g) {
              *reinterpret_cast<wvec<T>*>(out + qo + ln.at[g]) = w[g];
              if (kRev)
#pragma unroll
                for (int e = 0; e < V16; ++e) part += (double)h.r[g][ln.mem(e)] * (double)w[g][ln.mem(e)];
            }
            return;
          }
#pragma unroll
          for (int g = 0; g < kGS; ++g) {
#pragma unroll
            for (int e = 0; e < V16; ++e) {
              const int row = ln.row(g), c = ln.col(q, g, e);
              if (row < rows && (unsigned)c < (unsigned)N) {
                out[(unsigned int)(kRev ? (kWT - 1 - row) * N + (N - 1 - c) : row * N + c)] =
                    w[g][ln.mem(e)];
                if (kRev) part += (double)h.r[g][ln.mem(e)] * (double)w[g][ln.mem(e)];
              }
            }
          }
        };
        const std::false_type any{};
        load_r(any, -1, h0);
        load_r(any, 0, h1);
        load_r(any, 1, h2);
        wf_barrier();  // the preamble's
        wf_barrier();  // iteration 0: nothing swept yet
        int n = 1;
        auto iteration = [&](auto fast, Held& h) {
          // chunk n - 1 is swept: its last row first, then the lines that end in it
          if (st == 0 && n - 1 < nc && strip + 1 < n_map && l < C) {
            const int c = (n - 1) * C + l - (kWT - 1);
            if ((unsigned)c < (unsigned)N)
              edge_put(edge + (size_t)c * kWords, tag, yo[(n - 1) % kWOut * C + l][kWT - 1]);
          }
          store(n - 2, h);
          load_r(fast, n - 2 + kWHeld, h);
          wf_barrier();
          return n++ < nc + 1;
        };
        const std::true_type fast{};
        const int n_fast = q_last >= nc - 1 ? nc + 2 : q_last + 2 - kWHeld + 1;
        while (n + kWHeld <= n_fast) {
          iteration(fast, h0);
          iteration(fast, h1);
          iteration(fast, h2);
        }
        while (n <= nc + 1 && iteration(any, h0) && iteration(any, h1) && iteration(any, h2)) {
        }
      }
      if (kRev) {
        part = wf_wave_sum(part);
        if ((tid & 63) == 0) red[wv] = part;
        __syncthreads();
        if (tid == 0) {
          double tot = 0.0;
#pragma unroll
          for (int k = 0; k < kWStore; ++k) tot += red[6 + k];
          store_partial(a.P + 1 * a.pstride + d.dtile0 + strip, tot);
        }
        if (a.fin_mode) {
          const int sl[1] = {1};
          __syncthreads();  // red is the finisher's scratch next
          fused_finish<kFinTailW, 1>(Arrival{a.fcnt, a.gcnt, a.gsum, a.gstride, a.P, a.pstride}, sl,
                                     d.dtile0, strip, n_map, d.gbd, a.desc, a.ms, m, a.fin_mode, 0,
                                     &fflag, red);
        }
      }
    }
    if (one_each) break;
    __syncthreads();  // the ticket has been read by every wave
  }
  // the last workgroup to leave rearms the counters and ends the epoch (every
  // workgroup read it before it left)
  if (tid == 0 && __hip_atomic_fetch_add(a.ctl + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                      gridDim.x - 1) {
    __hip_atomic_store(a.ctl, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(a.ctl + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(a.ctl + 2, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// SSOR "pivots" D / omega are pointwise (stored as 1 / p like the ILU ones):
// every active map, grid-stride.
template <typename T>
__global__ void __launch_bounds__(256) k_wf_ssor_diag(WArgs a) {
  if ((int)blockIdx.y >= a.counts[2]) return;
  const int m = a.mact[blockIdx.y];
  const MapDesc& d = a.desc[m];
  const T* U = reinterpret_cast<const T*>(a.U) + d.off;
  const T* V = reinterpret_cast<const T*>(a.V) + d.off;
  T* piv = reinterpret_cast<T*>(const_cast<void*>(a.piv)) + d.off;
  const int M = d.M, N = d.N;
  for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < (long long)M * N;
       p += (long long)gridDim.x * blockDim.x) {
    const int i = (int)(p / N), j = (int)(p % N);
    const T dg = (j > 0 ? U[p - 1] : T(0)) + U[p] + (i > 0 ? V[p - N] : T(0)) + V[p];
    piv[p] = T(1) / (dg == T(0) ? T(1) : dg / (T)a.omega);
  }
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
static WArgs make_wargs(const Engine& e, int expect, bool ssor, double omega, const void* r,
                        void* s, void* y) {
  WArgs a;
  a.desc = e.desc;
  a.ms = e.ms;
  a.slist = e.slist;
  a.mact = e.mact;
  a.counts = e.counts;
  a.P = e.P;
  a.pstride = e.pstride;
  a.U = e.U;
  a.V = e.V;
  a.piv = e.aux;
  a.r = r;
  a.s = s;
  a.y = y;
  a.ctl = e.wctl;
  a.edge = e.wedge;
  a.fcnt = e.fcnt;
  a.gcnt = e.gcnt;
  a.gsum = e.gsum;
  a.gstride = e.gstride;
  a.expect = expect;
  a.fin_mode = 0;
  a.recip = 1;
  a.omega = omega;
  a.flags = (ssor ? kWSsor : 0) | (e.no_wait ? kWNoWait : 0);
  return a;
}

// Strips of a map and entries of its edge buffer.
int wf_strips(int M) { return (M + kWT - 1) / kWT; }

// Grid of a sweep: the next power of two >= the active strips (few distinct
// shapes keep captured graphs reusable), capped: workgroups take further
// strips by ticket.
int wf_grid(const Engine& e) {
  int g = 1;
  while (g < e.act_strips && g < kWMaxGrid) g <<= 1;
  return g;
}

template <typename T>
void e_pivots(hipStream_t st, const Engine& e, int nmaps, bool ssor, double omega, bool recip) {
  WArgs a = make_wargs(e, -1, ssor, omega, nullptr, nullptr, nullptr);
  a.recip = recip ? 1 : 0;
  if (ssor) {
    hipLaunchKernelGGL(k_wf_ssor_diag<T>, dim3(64, std::max(1, nmaps)), dim3(256), 0, st, a);
    return;
  }
  hipLaunchKernelGGL((k_wf_sweep<T, kWPivots>), dim3(wf_grid(e)), dim3(kWThreads), 0, st, a);
}

// s = M^-1 r for the maps in state `expect`; fin_mode != 0 runs the per-map
// finisher of r^T s in the workgroup that completes the map
template <typename T>
void e_sweep(hipStream_t st, const Engine& e, int expect, bool ssor, double omega, const void* r,
             void* s, void* y, int fin_mode) {
  WArgs a = make_wargs(e, expect, ssor, omega, r, s, y);
  const dim3 g(wf_grid(e));
  hipLaunchKernelGGL((k_wf_sweep<T, kWForward>), g, dim3(kWThreads), 0, st, a);
  a.fin_mode = fin_mode;
  hipLaunchKernelGGL((k_wf_sweep<T, kWBackward>), g, dim3(kWThreads), 0, st, a);
}

template void e_pivots<float>(hipStream_t, const Engine&, int, bool, double, bool);
template void e_pivots<double>(hipStream_t, const Engine&, int, bool, double, bool);
template void e_sweep<float>(hipStream_t, const Engine&, int, bool, double, const void*, void*, void*,
                             int);
template void e_sweep<double>(hipStream_t, const Engine&, int, bool, double, const void*, void*,
                              void*, int);

}  // namespace lpu
