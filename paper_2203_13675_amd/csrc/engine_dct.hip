// Batched DCT Poisson preconditioner: grouped contractions over all active maps.
//
// DCT (s = L0^+ r, L0 the unit-weight Neumann Laplacian):
//   s = C_M^T [ (C_M r C_N^T) ./ Lambda ] C_N,
//   C_n[k][j] = s_k cos(pi k (2j+1) / (2n)), Lambda_kl = (2 - 2cos(pi k/M)) + (2 - 2cos(pi l/N)),
//   zero mode dropped.  Four stages of Out^T = X B^T (rows of X transformed by
//   the basis in B, result stored transposed):
//     stage 0: X = r  (M x N), B = C_N   -> t1 (N x M)
//     stage 1: X = t1 (N x M), B = C_M   -> t2 (M x N), t2 ./= Lambda
//     stage 2: X = t2 (M x N), B = C_N^T -> t1 (N x M)
//     stage 3: X = t1 (N x M), B = C_M^T -> s  (M x N), zero on isolated pixels,
//              FP64 partial of r^T s per tile.
// Every map contributes ceil(M/t) ceil(N/t) output tiles to every stage, t its
// tile side (MapDesc::dtr).

#include <type_traits>

#include "lpu_internal.h"
#include "lpu_device.h"
#include "lpu_finish.h"

namespace lpu {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

struct DArgs {
  const MapDesc* desc;
  MapState* ms;
  const int* dtile_map;
  const int* dact;
  const int* counts;
  double* P;
  long long pstride;
  const void* X;
  void* Out;
  const void* rvec;
  const unsigned char* iso;
  int stage, expect;
  int cidx;   // counts[] slot holding the length of `dact`
  int dact_cap;  // entries of `dact` (its capacity)
  int *fcnt, *gcnt;  // arrival counters of the fused finisher
  double* gsum;      // its group sums (rows of gstride)
  long long gstride;
  const EoTile* eot;  // tile records: [stage parity][global DCT tile]
  long long eot_cap;
  int fin_mode;  // last stage of the MFMA kernels: 0, or the FinishMode of the
                 // fused finisher (the map's r^T s, beta and stop tests)
};

struct DTile {
  int m, R, K, r0, c0;
  long long off;
  const DctTabDev* tab;
  bool ok;
};

__device__ __forceinline__ DTile dtile(const DArgs& a, int g) {
  DTile t;
  t.m = a.dtile_map[g];
  const MapDesc& d = a.desc[t.m];
  t.ok = a.ms[t.m].state == a.expect;
  const bool rows_m = (a.stage & 1) == 0;
  t.R = rows_m ? d.M : d.N;
  t.K = rows_m ? d.N : d.M;
  const int tiles_r = (t.R + d.dtr - 1) / d.dtr;
  const int local = g - d.dtile0;
  t.r0 = (local % tiles_r) * d.dtr;
  t.c0 = (local / tiles_r) * d.dtr;
  t.off = d.off;
  t.tab = rows_m ? d.tabN : d.tabM;
  return t;
}

__device__ __forceinline__ float fp16_scale(float amax) {
  if (!(amax > 0.0f) || !isfinite(amax)) return 1.0f;
  int e;
  frexpf(amax, &e);
  return ldexpf(1.0f, 14 - e);
}

// ---------------------------------------------------------------------------
// Even/odd MFMA stage (mixed path, both sides multiples of 128).
//
// The basis satisfies C[k][n-1-j] = (-1)^k C[k][j].  With h = n/2 and the
// spectrum kept in split order (even k first):
//   forward  X_even = E (x_a + x_b),  X_odd = O (x_a - x_b),
//            x_a = x[0..h), x_b = x[n-1 .. h] (mirrored), E, O the h x h
//            even/odd rows of C restricted to j < h;
//   inverse  u = E^T X_even, v = O^T X_odd;  x[j] = u_j + v_j,
//            x[n-1-j] = u_j - v_j  (j < h).
// Both halve the multiply-adds of the dense transform.
//
// A block owns 128 rows of X and 64 output columns c0 .. c0+63 of the half
// range [0, h), in two halves computed side by side from the same loads:
//   forward: half 0 = even outputs c (A = x_a + x_b), half 1 = odd outputs
//            h + c (A = x_a - x_b);
//   inverse: half 0 = u (spectrum columns [0, h)), half 1 = v (columns
//            [h, n)), combined at the end into outputs c and n-1-c.
// Wave w computes rows 64 (w & 1) .. +63 of half w >> 1 as 4 x 4 MFMA tiles
// of 16 x 16 (64 accumulator registers).  Each K step stages both halves of A
// and of the table slice in LDS, A converted on the way to bf16 hi/lo (or
// scaled fp16).  LDS rows are KS 16-bit values without padding; the 16-byte
// chunk q of row r sits at q ^ swz(r), which keeps both the staging writes and
// the fragment reads free of bank conflicts (rows of 4 chunks: 8 rows read in
// one LDS cycle land in 8 distinct bank quads; rows of 8 chunks: likewise for 8
// or 16 rows).
//
// What bounds it: a block's steps.  Small launches wait for memory, so the
// operands of two steps are held in registers on top of the two buffers in
// LDS (one barrier a step), and tiles are a quarter as large; large ones share
// their time between matrix cores, LDS and the L1 fill (28 to 35 us each of
// a 4096^2 fp16 stage's 81 to 105), so the tile is as wide as the registers
// allow, which leaves room for one step in registers only (two: 5 to 10 %
// slower), and the 16-bit matrices are laid out for whole lines (eo_at: 427
// against 385 us for the four stages; half-line requests had the L1 wait half
// of its cycles).  KS = 64 with one buffer: 465.  Four stages, one launch, us,
// against the kernel before (KS = 64, one buffer, one step ahead, row-major, 128
// rows for every launch): 1024^2 fp16 36 / 65, bf16 split 64 / 115, 2048^2 fp16
// 96 / 117, 4096^2 fp16 385 / 489.
// ---------------------------------------------------------------------------
template <int NC>
__device__ __forceinline__ int swz(int r) {
  return NC == 4 ? (((r >> 1) ^ (r >> 2)) & 3) : ((r ^ (r >> 3)) & 7);
}
// offset (16-bit elements) of element 8q + e of LDS row r (rows of NC chunks)
template <int NC>
__device__ __forceinline__ int lds_at(int r, int q) { return r * (8 * NC) + ((q ^ swz<NC>(r)) << 3); }

typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));

// The 16-bit matrices of these stages (tables, and the scaled-fp16 values
// between the stages) lie in blocks of 16 rows by 32 columns, row by row in
// each, so that one load of a wave, 16 rows of a K step, is 1 KB on end.
// Offset of (row, col) in a matrix of K columns, from a row that starts a block.
template <typename I>
__device__ __forceinline__ I eo_at(I row, I col, I K) {
  return (row & ~I(15)) * K + (col >> 5) * 512 + (row & 15) * 32 + (col & 31);
}

// Tile shapes: the tile above (NI = NJ = 4: 4 x 4 MFMA tiles a wave); NJ = 8
// (scaled fp16 only), "wide": two such tiles side by side, 128 output pairs,
// from the same staged rows of X; NI = NJ = 2, "fine": a quarter of the tile,
// 64 rows and 32 output pairs, four blocks to a list entry.  A wide tile is
// named by its left narrow tile; where the map has no right partner (h an odd
// multiple of 64) it stages its own table rows twice and stores the left half
// only.  Per output the MFMAs run over the same K chunks in the same order in
// every shape, and stage 3 writes one partial of r^T s per quarter tile, summed
// in one order whatever the shape, so the results are identical.
template <int SPLIT, int INV, int IN16, int OUT16, int NI, int NJ>
__global__ void __launch_bounds__(256, 2) k_e_dct_eo(DArgs a) {
  static_assert((NI == 4 && NJ == 4) || (NI == 2 && NJ == 2) ||
                    (NI == 4 && NJ == 8 && !SPLIT), "wide tiles: scaled fp16");
  constexpr bool FINE = NI == 2;
  constexpr int NP = SPLIT ? 2 : 1;                // hi (+ lo) planes
  constexpr int KS = FINE ? 64 : 32;                      // K step
  constexpr int NBUF = SPLIT ? 1 : 2;
  constexpr int DEPTH = NJ == 8 || (SPLIT && !FINE) ? 1 : 2;
  constexpr int NC = KS / 8;                       // 16-byte chunks per LDS row
  constexpr int TR = 32 * NI;                      // rows of X
  constexpr int kBW = 16 * NJ;                     // table rows per half (output pairs)
  constexpr int kA = TR * KS, kB = kBW * KS;       // elements of one A / B half-plane
  constexpr int kBuf = NP * 2 * (kA + kB);         // elements of one step's operands
  constexpr int JR = NJ < 4 ? NJ : 4;              // column groups per round of the inverse's exchange
  constexpr int kXchg = INV ? 2 * 2 * NI * JR * 64 * 16 : 0;  // its bytes
  constexpr int kSmem = NBUF * kBuf * 2 > kXchg ? NBUF * kBuf * 2 : kXchg;
  constexpr int VPT = IN16 ? 8 : 4;                // X staging: values per thread and load
  constexpr int TPR = KS / VPT;                    // X staging: threads per row
  constexpr int XP = TR * TPR / 256;               // X staging passes (rows xr + XP-stride)
  constexpr int SEGS = 256 / NC;                   // table staging: segments per pass
  constexpr int TP = NP * 2 * kBW / SEGS;          // table staging passes
  static_assert(XP >= 1 && TP >= 1, "a pass of the block covers at most one step");
  static_assert(kBW % SEGS == 0, "a pass stages rows of one half and plane");
  __shared__ __attribute__((aligned(16))) unsigned char smem[kSmem];
  __shared__ double red[4 * NJ];
  __shared__ double fred[3 * 4];
  __shared__ int fflag;
  const int nact = a.counts[a.cidx];
  // list position and quarter of a block's k-th tile: the four quarters of a
  // list entry go to blocks 8 apart, so to the XCD of the entry
  auto pos_of = [](int b) { return FINE ? (b >> 5) * 8 + (b & 7) : b; };
  // the block's first list entry is requested with the list's length
  const int g_first = a.dact[min(pos_of((int)blockIdx.x), max(a.dact_cap - 1, 0))];
  __asm__ volatile("" ::"s"(nact), "s"(g_first));  // both loads issued before the loop test
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int wr = (w & 1) * 16 * NI, hf = w >> 1;
  const int lr = lane & 15, kq = lane >> 4;        // MFMA operand map: row lr, k chunk kq
  const int xr = tid / TPR, xk = (tid % TPR) * VPT;  // X staging: rows xr + (256/TPR) p, k xk ..
  static_assert(!(SPLIT && (IN16 || OUT16)), "the bf16 split keeps FP32 intermediates");
  const int bseg = tid / NC, bq = tid % NC;         // table staging: segment, 16-byte chunk
  for (int t_ = blockIdx.x; FINE ? (t_ >> 5) * 8 < nact : t_ < nact; t_ += gridDim.x) {
    const int pos = pos_of(t_), quarter = FINE ? (t_ >> 3) & 3 : 0;
    if (FINE && pos >= nact) continue;
    const int g = t_ == (int)blockIdx.x ? g_first : a.dact[pos];
    if (g < 0) continue;  // padding slot of the XCD-ordered list
    // the tile's record (one load); its first K steps are fetched before the
    // map's state is read, so the two round trips overlap
    const EoTile& tt = a.eot[(size_t)(a.stage & 1) * a.eot_cap + g];
    const int R = tt.R, n = tt.K, h = n >> 1, tm = tt.m;
    const int c0 = tt.c0 + 32 * (quarter >> 1), r0 = tt.r0 + 64 * (quarter & 1);
    const long long toff = tt.off;
    const int t_local = tt.local, t_ndt = tt.ndt, t_gbd = tt.gbd;
    const float t_lmin = tt.lmin;
    // wide tiles: does the right partner exist (uniform over the block)?
    const bool full = NJ != 8 || c0 + 128 <= h;
    const double* t_lam_m = tt.lam_m;
    const double* t_lam_n = tt.lam_n;
    const float* X = reinterpret_cast<const float*>(a.X) + toff;
    const uint16_t* X16 = reinterpret_cast<const uint16_t*>(a.X) + toff;
    float* Out = reinterpret_cast<float*>(a.Out) + toff;
    uint16_t* Out16 = reinterpret_cast<uint16_t*>(a.Out) + toff;
    const uint16_t* T0 = INV ? (SPLIT ? tt.ti[1] : tt.ti[0]) : (SPLIT ? tt.tf[1] : tt.tf[0]);
    const uint16_t* T1 = INV ? tt.ti[2] : tt.tf[2];
    float xs = 1.0f, inv_xs = 1.0f, os = 1.0f;
    // register staging of one K step
    struct Held {
      float4 sa[IN16 ? 1 : XP], sb[IN16 ? 1 : XP];
      u16x8 ha[IN16 ? XP : 1], hb[IN16 ? XP : 1];
      u16x8 sT[TP];
    };
    // a load's address is a uniform base, which moves with the step, and a
    // 32-bit offset of the lane, which does not
    unsigned xa[XP], xb[XP], to[TP];
#pragma unroll
    for (int p = 0; p < XP; ++p) {
      const unsigned row = xr + (256 / TPR) * p;
      const unsigned kb = INV ? xk : KS - VPT - xk;  // forward: from the top, mirrored
      xa[p] = IN16 ? eo_at<unsigned>(row, xk, n) : row * (unsigned)n + xk;
      xb[p] = IN16 ? eo_at<unsigned>(row, kb, n) : row * (unsigned)n + kb;
    }
#pragma unroll
    for (int p = 0; p < TP; ++p) {
      // a wide tile without its partner stages its own rows twice (the
      // extra outputs are computed but never stored)
      const int s = p * SEGS + bseg, row = full ? s % kBW : s % 64;
      to[p] = eo_at<unsigned>(row, 8 * bq, INV ? n : h);
    }
    auto fetch = [&](Held& v, int k0) {
      const size_t rb = (size_t)r0 * n, kb = INV ? h + k0 : n - KS - k0;
#pragma unroll
      for (int p = 0; p < XP; ++p) {
        if (IN16) {
          v.ha[p] = *reinterpret_cast<const u16x8*>(X16 + rb + 16 * (size_t)k0 + xa[p]);
          v.hb[p] = *reinterpret_cast<const u16x8*>(X16 + rb + 16 * kb + xb[p]);
        } else {
          v.sa[p] = *reinterpret_cast<const float4*>(X + rb + k0 + xa[p]);
          v.sb[p] = *reinterpret_cast<const float4*>(X + rb + kb + xb[p]);
        }
      }
#pragma unroll
      for (int p = 0; p < TP; ++p) {
        // segment ((half * NP) + plane) * kBW + row: half and plane by the pass
        const int half = p * SEGS / (kBW * NP), plane = (p * SEGS / kBW) % NP;
        const uint16_t* T = (plane ? T1 : T0) + 16 * (size_t)k0 +
                            (INV ? (size_t)c0 * n + (half ? 16 * (size_t)h : 0)
                                 : (size_t)((half ? h : 0) + c0) * h);
        v.sT[p] = *as_global(reinterpret_cast<const u16x8*>(T + to[p]));
      }
    };
    auto stash = [&](const Held& v, uint16_t* As) {  // As: [plane][half][TR x KS], then the table's
      uint16_t* Bs = As + NP * 2 * kA;               // [plane][half][kBW x KS]
      if constexpr (IN16) {
        // fp16 input already carries the stage's scale: the inverse copies
        // it, the forward folds x_a +- x_b in FP32 and rounds once more
#pragma unroll
        for (int p = 0; p < XP; ++p) {
          const int r = xr + (256 / TPR) * p;
          u16x8 v0 = v.ha[p], v1 = v.hb[p];
          if (!INV) {
            // whole-vector form: x_b reversed (it holds x[n-1-k] from the top),
            // sum and difference in FP32, one rounding back to fp16
            const f16x8 fa = __builtin_bit_cast(f16x8, v.ha[p]);
            const f16x8 fbr = __builtin_bit_cast(f16x8, v.hb[p]);
            const f16x8 fb = __builtin_shufflevector(fbr, fbr, 7, 6, 5, 4, 3, 2, 1, 0);
            const f32x8 a32 = __builtin_convertvector(fa, f32x8);
            const f32x8 b32 = __builtin_convertvector(fb, f32x8);
            v0 = __builtin_bit_cast(u16x8, __builtin_convertvector(a32 + b32, f16x8));
            v1 = __builtin_bit_cast(u16x8, __builtin_convertvector(a32 - b32, f16x8));
          }
          const int o = lds_at<NC>(r, xk >> 3);
          *reinterpret_cast<u16x8*>(As + 0 * kA + o) = v0;
          *reinterpret_cast<u16x8*>(As + 1 * kA + o) = v1;
        }
      } else {
#pragma unroll
        for (int p = 0; p < XP; ++p) {
          const int r = xr + (256 / TPR) * p;
          const float av[4] = {v.sa[p].x, v.sa[p].y, v.sa[p].z, v.sa[p].w};
          // forward: the b part is x mirrored, x[n-1-k] for k = k0 + xk .. +3
          const float bv[4] = {INV ? v.sb[p].x : v.sb[p].w, INV ? v.sb[p].y : v.sb[p].z,
                               INV ? v.sb[p].z : v.sb[p].y, INV ? v.sb[p].w : v.sb[p].x};
          u16x4 hv[2], lv[2];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float v0 = INV ? av[e] : av[e] + bv[e];
            const float v1 = INV ? bv[e] : av[e] - bv[e];
            if (SPLIT) {
              const __bf16 h0 = (__bf16)v0, h1 = (__bf16)v1;
              hv[0][e] = __builtin_bit_cast(uint16_t, h0);
              hv[1][e] = __builtin_bit_cast(uint16_t, h1);
              lv[0][e] = __builtin_bit_cast(uint16_t, (__bf16)(v0 - (float)h0));
              lv[1][e] = __builtin_bit_cast(uint16_t, (__bf16)(v1 - (float)h1));
            } else {
              hv[0][e] = __builtin_bit_cast(uint16_t, (_Float16)(v0 * xs));
              hv[1][e] = __builtin_bit_cast(uint16_t, (_Float16)(v1 * xs));
            }
          }
          const int o = lds_at<NC>(r, xk >> 3) + (xk & 4);
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            *reinterpret_cast<u16x4*>(As + (0 * 2 + half) * kA + o) = hv[half];
            if (SPLIT) *reinterpret_cast<u16x4*>(As + (1 * 2 + half) * kA + o) = lv[half];
          }
        }
      }
#pragma unroll
      for (int p = 0; p < TP; ++p) {
        const int half = p * SEGS / (kBW * NP), plane = (p * SEGS / kBW) % NP;
        const int row = (p * SEGS + bseg) % kBW;
        *reinterpret_cast<u16x8*>(Bs + (plane * 2 + half) * kB + lds_at<NC>(row, bq)) = v.sT[p];
      }
    };
    f32x4 acc[NI][NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto product = [&](const uint16_t* As) {
      const uint16_t* Bs = As + NP * 2 * kA;
      const uint16_t* Ah = As + (0 * 2 + hf) * kA;
      const uint16_t* Al = As + (1 * 2 + hf) * kA;
      const uint16_t* Bh = Bs + (0 * 2 + hf) * kB;
      const uint16_t* Bl = Bs + (1 * 2 + hf) * kB;
#pragma unroll
      for (int ks = 0; ks < KS / 32; ++ks) {
        const int q = 4 * ks + kq;
        // the smaller operand's fragments are held, the other's come one by one
        u16x8 ah[NI], al[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          ah[i] = *reinterpret_cast<const u16x8*>(Ah + lds_at<NC>(wr + 16 * i + lr, q));
          if (SPLIT) al[i] = *reinterpret_cast<const u16x8*>(Al + lds_at<NC>(wr + 16 * i + lr, q));
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const u16x8 bh = *reinterpret_cast<const u16x8*>(Bh + lds_at<NC>(16 * j + lr, q));
          u16x8 bl;
          if (SPLIT) bl = *reinterpret_cast<const u16x8*>(Bl + lds_at<NC>(16 * j + lr, q));
#pragma unroll
          for (int i = 0; i < NI; ++i) {
            if (SPLIT) {
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                  __builtin_bit_cast(bf16x8, ah[i]), __builtin_bit_cast(bf16x8, bh), acc[i][j], 0, 0, 0);
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                  __builtin_bit_cast(bf16x8, ah[i]), __builtin_bit_cast(bf16x8, bl), acc[i][j], 0, 0, 0);
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                  __builtin_bit_cast(bf16x8, al[i]), __builtin_bit_cast(bf16x8, bh), acc[i][j], 0, 0, 0);
            } else {
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                  __builtin_bit_cast(f16x8, ah[i]), __builtin_bit_cast(f16x8, bh), acc[i][j], 0, 0, 0);
            }
          }
        }
      }
    };
    const int nsteps = h / KS;
    // the map's state and the first steps' operands are requested together;
    // the compiler barriers keep that order (it would otherwise sink the
    // operand loads behind the state test's branch)
    const int m_state = a.ms[tm].state;
    const double m_rr = a.ms[tm].rr;
    const int t_iso = a.desc[tm].use_iso;
    __asm__ volatile("" ::: "memory");
    Held va, vb;
    fetch(va, 0);
    if (DEPTH > 1) fetch(vb, min(1, nsteps - 1) * KS);
    __asm__ volatile("" ::: "memory");
    if (m_state != a.expect) continue;  // uniform over the block
    const auto* lamMs = as_global(t_lam_m);
    const auto* lamNs = as_global(t_lam_n);
    // output index of column group j and first output row of row group i
    auto out_c = [&](int j) {
      const int c = c0 + 16 * j + lr;
      return INV ? (hf ? n - 1 - c : c) : (hf ? h : 0) + c;
    };
    auto out_rb = [&](int i) { return r0 + wr + 16 * i + 4 * kq; };
    // Which stages an instance can run: the forward instances with fp16 input
    // (or the split's, which serve both forward stages) run stage 1, the
    // inverse instances with an FP32 output run stage 3.
    constexpr bool kS1 = !INV && (SPLIT || IN16);
    constexpr bool kS3 = INV && !OUT16;
    const bool st1 = kS1 && a.stage == 1, st3 = kS3 && a.stage == 3;
    if (!SPLIT) {
      // Scaled fp16: power-of-two scales from bounds that hold before any
      // value exists.  The transforms are orthonormal, so every stage output
      // is bounded by the Frobenius norm of r (first forward stage; twice
      // that after the even/odd fold) or of S ./ Lambda <= ||r|| / lambda_min
      // (second forward stage and the first inverse stage).
      const float nr = (float)sqrt(m_rr) * 1.0000001f;
      const float b01 = 2.0f * nr, b23 = nr / t_lmin * 1.0000001f;
      xs = fp16_scale(a.stage <= 1 ? b01 : b23);
      inv_xs = 1.0f / xs;
      os = fp16_scale(a.stage == 0 ? b01 : b23);
    }
    uint16_t* cur = reinterpret_cast<uint16_t*>(smem);
    uint16_t* nxt = cur + (NBUF - 1) * kBuf;
    // Past the last step the last one is fetched again: with as many loads in
    // flight on every path, the wait for one step's leaves the later ones' alone.
    auto at = [&](int s) { return min(s, nsteps - 1) * KS; };
    if constexpr (NBUF == 2) {
      stash(va, cur);
      fetch(va, at(DEPTH));
      __syncthreads();
      // v: step s + 1's operands, replaced by those of step s + 1 + DEPTH
      auto step = [&](int s, Held& v) {
        stash(v, nxt);
        fetch(v, at(s + 1 + DEPTH));
        product(cur);
        __syncthreads();
        uint16_t* const c = cur;
        cur = nxt;
        nxt = c;
      };
      int s = 0;
      if constexpr (DEPTH > 1) {
        for (; s + 2 < nsteps; s += 2) {
          step(s, vb);
          step(s + 1, va);
        }
        if (s + 1 < nsteps) step(s, vb);
      } else {
        for (; s + 1 < nsteps; ++s) step(s, va);
      }
      product(cur);
    } else {
      auto step = [&](int s, Held& v) {
        stash(v, cur);
        __syncthreads();
        fetch(v, at(s + DEPTH));
        product(cur);
        __syncthreads();
      };
      int s = 0;
      if constexpr (DEPTH > 1) {
        for (; s + 1 < nsteps; s += 2) {
          step(s, va);
          step(s + 1, vb);
        }
        if (s < nsteps) step(s, va);
      } else {
        for (; s < nsteps; ++s) step(s, va);
      }
    }
    // epilogue: lane holds D[row 4*(lane/16) + e][col lane mod 16] of each 16x16 tile,
    // i.e. outputs (c, rb .. rb+3) with rb a multiple of 4.  Everything it
    // reads is loaded before its first store: loads and stores share one
    // counter, so a load issued after a store would wait for that store too,
    // one memory round trip per output tile (r and the isolated-pixel flags of
    // stage 3: one column group ahead).
    float lam_c[NJ], lam_r[NI][4];  // stage 1: eigenvalues along M and N (FP32)
    if (st1) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) lam_c[j] = (j < 4 || full) ? (float)lamMs[out_c(j)] : 0.0f;
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) lam_r[i][e] = (float)lamNs[out_rb(i) + e];
    }
    const float* rv = reinterpret_cast<const float*>(a.rvec) + toff;
    const unsigned char* iso = (a.iso && t_iso) ? a.iso + toff : nullptr;
    f32x4 r_cur[NI], r_nxt[NI];
    unsigned int z_cur[NI], z_nxt[NI];
    auto load_rz = [&](int j, f32x4 (&rr)[NI], unsigned int (&zz)[NI]) {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const size_t o = (size_t)out_c(j) * R + out_rb(i);
        rr[i] = *as_global(reinterpret_cast<const f32x4*>(rv + o));
        zz[i] = iso ? *as_global(reinterpret_cast<const unsigned int*>(iso + o)) : 0u;
      }
    };
    if (st3) load_rz(0, r_cur, z_cur);
    // stage 3: this wave's sums of r^T s over 32 rows by 32 output pairs each
    double part[NI / 2][NJ / 2];
#pragma unroll
    for (int i = 0; i < NI / 2; ++i)
#pragma unroll
      for (int j = 0; j < NJ / 2; ++j) part[i][j] = 0.0;
    auto emit = [&](int i, int j, const float (&y)[4]) {
      const int c = out_c(j), rb = out_rb(i);
      float v[4] = {y[0], y[1], y[2], y[3]};
      if (st1) {
        // spectrum ./ Lambda with the zero mode dropped; an FP32 reciprocal
        // (the preconditioner stays one fixed linear map)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float l = lam_c[j] + lam_r[i][e];
          v[e] = (c == 0 && rb + e == 0) ? 0.0f : v[e] * __builtin_amdgcn_rcpf(l);
        }
      }
      if (st3) {
        // zero on isolated pixels; FP64 partial of r^T s (four outputs at once)
        const unsigned int z = z_cur[i];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if ((z >> (8 * e)) & 0xffu) v[e] = 0.0f;
          part[i / 2][j / 2] = fma((double)r_cur[i][e], (double)v[e], part[i / 2][j / 2]);
        }
      }
      if (OUT16) {
        u16x4 hv;
#pragma unroll
        for (int e = 0; e < 4; ++e) hv[e] = __builtin_bit_cast(uint16_t, (_Float16)(v[e] * os));
        *reinterpret_cast<u16x4*>(Out16 + eo_at<size_t>(c, rb, R)) = hv;
      } else {
        *reinterpret_cast<float4*>(Out + (size_t)c * R + rb) = make_float4(v[0], v[1], v[2], v[3]);
      }
    };
    if (!INV) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if (j >= 4 && !full) continue;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          const float y[4] = {acc[i][j][0] * inv_xs, acc[i][j][1] * inv_xs, acc[i][j][2] * inv_xs,
                              acc[i][j][3] * inv_xs};
          emit(i, j, y);
        }
      }
    } else {
      // u (half 0) and v (half 1) of the same rows meet through LDS: the
      // waves of half 0 write u + v to output c, those of half 1 write
      // u - v to output n-1-c
      f32x4* xg = reinterpret_cast<f32x4*>(smem);  // [half][row group][NI JR tiles][64 lanes]
      const int oh = hf ^ 1;
      // one round per four column groups (wide tiles: two rounds, the
      // second only when the partner exists; uniform over the block)
#pragma unroll
      for (int jr = 0; jr < NJ / JR; ++jr) {
        if (jr > 0 && !full) break;
        __syncthreads();  // every wave is done reading the staged operands (or the last round)
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int jj = 0; jj < JR; ++jj)
            xg[((hf * 2 + (w & 1)) * NI * JR + i * JR + jj) * 64 + lane] = acc[i][JR * jr + jj];
        __syncthreads();
#pragma unroll
        for (int jj = 0; jj < JR; ++jj) {
          const int j = JR * jr + jj;
          if (st3 && j < NJ - 1) load_rz(j + 1, r_nxt, z_nxt);
#pragma unroll
          for (int i = 0; i < NI; ++i) {
            const f32x4 o = xg[((oh * 2 + (w & 1)) * NI * JR + i * JR + jj) * 64 + lane];  // the other half
            const float y[4] = {(hf ? o[0] - acc[i][j][0] : acc[i][j][0] + o[0]) * inv_xs,
                                (hf ? o[1] - acc[i][j][1] : acc[i][j][1] + o[1]) * inv_xs,
                                (hf ? o[2] - acc[i][j][2] : acc[i][j][2] + o[2]) * inv_xs,
                                (hf ? o[3] - acc[i][j][3] : acc[i][j][3] + o[3]) * inv_xs};
            emit(i, j, y);
          }
          if (st3 && j < NJ - 1) {
#pragma unroll
            for (int i = 0; i < NI; ++i) r_cur[i] = r_nxt[i], z_cur[i] = z_nxt[i];
          }
        }
      }
    }
    if (st3) {
      // one partial per quarter of the 128-row tile: its four sums (two row
      // groups of two halves) in order
      if constexpr (FINE) {
        double vv[1] = {part[0][0]};
        block_sum<1>(vv, red);
        if (tid == 0) store_partial(a.P + 1 * a.pstride + kEoParts * g + quarter, vv[0]);
      } else {
#pragma unroll
        for (int i = 0; i < NI / 2; ++i)
#pragma unroll
          for (int j = 0; j < NJ / 2; ++j) {
            const double v = tree64(part[i][j]);
            if (lane == 0) red[(2 * j + (w & 1)) * 4 + 2 * hf + i] = v;  // [quarter][half, row group]
          }
        __syncthreads();
        if (tid < (full ? NJ : 4)) {  // a wide tile's right half: the partner's quarters
          double v = 0.0;
#pragma unroll
          for (int k = 0; k < 4; ++k) v += red[4 * tid + k];
          store_partial(a.P + 1 * a.pstride + kEoParts * (g + (tid < 4 ? 0 : R / 128)) + (tid & 3), v);
        }
      }
      if (a.fin_mode) {
        const int sl[1] = {1};
        for (int k = 0; k < (NJ == 8 && full ? 2 : 1); ++k) {
          if (k > 0) __syncthreads();  // every wave has read fflag
          fused_finish<kFinTail, 1>(Arrival{a.fcnt, a.gcnt, a.gsum, a.gstride, a.P, a.pstride}, sl,
                                    kEoParts * (g - t_local),
                                    kEoParts * (t_local + k * (R / 128)) + quarter,
                                    kEoParts * t_ndt, t_gbd, a.desc, a.ms, tm, a.fin_mode, 0, &fflag,
                                    fred, FINE ? 1 : kEoParts);
        }
      }
    }
    __syncthreads();  // the next tile's first step may overwrite what slower waves still read
  }
}

// ---------------------------------------------------------------------------
// Dense MFMA stage (mixed path, any side lengths): a block (4 waves) owns
// TR x TR outputs, a wave a quarter of them as MFMA tiles of 16 x 16 x 32; lane
// l supplies row l mod 16 and the 8 values of chunk l / 16 of an operand.  K
// steps of 64 go through two LDS buffers, X converted once on the way (bf16 hi
// and lo, or scaled fp16), every operand requested three steps before its
// products; the tables' rows are padded with zeros to whole steps, so only X
// needs guards, in the last, partial step, which is requested ahead of the
// loop.  An output's products run over the K chunks in increasing order
// whatever the tile, hi hi, hi lo, lo hi in each.
//
// What bounds it at the sizes of one image is the latency of a tile's steps
// (the products of a step take some 100 cycles, the barrier and LDS around them
// three times that), so small maps take tiles of 32 x 32, four times as many as
// of 64 x 64, which re-read X and the tables half as often.  One PCG iteration
// (split bf16 / fp16) with tiles of 64 and of 32: 53 / 53 and 45 / 48 us at
// 64^2, 88 / 79 and 75 / 75 at 480 x 640, 110 / 97 and 106 / 101 at 720 x 960
// (180 tiles of 64), 176 / 144 and 209 / 185 at 1000 x 1500 (384), 436 / 305 and
// 662 / 485 at 2000^2.  kDenseWide lies just above 180 tiles, where the split
// still prefers 32 (by 4 %) and fp16 already 64 (by 4 %); nothing was measured
// between there and 384.  The side is the map's alone, so a full launch of many
// small maps takes 32 as well (48 maps of 480 x 640, split: 99 ms a call where
// the kernel before took 140).  The kernel it replaces
// (64 x 64, operands straight from memory, no step ahead, element by element
// where a side is not a multiple of 8) took 62 / 62, 145 / 133, 192 / 185,
// 887 / 632 and 824 / 679 us, and 353 / 267 at 509 x 733, now 83 / 84.
// ---------------------------------------------------------------------------
constexpr int kDenseWide = 192;

template <int SPLIT, int TR>
__device__ __forceinline__ void dct_dense_tile(const DArgs& a, const EoTile& t, bool use_iso, int g,
                                               float xs, float* amax_out, uint16_t* smem, double* red,
                                               float* fmx) {
  constexpr int NP = SPLIT ? 2 : 1, KS = 64, NT = TR / 32, XP = TR / 32;
  constexpr int kPlane = TR * KS, kBuf = 2 * NP * kPlane;  // 16-bit elements: X planes, table planes
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int lr = lane & 15, kq = lane >> 4;
  const int R = t.R, K = t.K, Kp = (K + KS - 1) / KS * KS;
  const float* X = reinterpret_cast<const float*>(a.X) + t.off;
  float* Out = reinterpret_cast<float*>(a.Out) + t.off;
  const bool fwd = a.stage < 2;
  const auto* Th = as_global(fwd ? t.tf[SPLIT ? 1 : 0] : t.ti[SPLIT ? 1 : 0]);
  const auto* Tl = as_global(fwd ? t.tf[2] : t.ti[2]);
  const int sr = tid >> 3, sq = tid & 7;  // staging: row of a pass, 16-byte chunk (8 values)
  // rows and columns past the map repeat the last one (their outputs are dropped)
  size_t xo[XP], to[XP];
#pragma unroll
  for (int p = 0; p < XP; ++p) {
    xo[p] = (size_t)min(t.r0 + sr + 32 * p, R - 1) * K + 8 * sq;
    to[p] = (size_t)min(t.c0 + sr + 32 * p, K - 1) * Kp + 8 * sq;
  }
  typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
  using gtab = const __attribute__((address_space(1))) u16x8*;
  struct Held {  // one K step's operands on the way to LDS
    f32x4u x0[XP], x1[XP];
    u16x8 th[XP], tl[XP];
  };
  auto fetch = [&](Held& v, int k0) {
#pragma unroll
    for (int p = 0; p < XP; ++p) {
      v.x0[p] = *reinterpret_cast<const f32x4u*>(X + xo[p] + k0);
      v.x1[p] = *reinterpret_cast<const f32x4u*>(X + xo[p] + k0 + 4);
      v.th[p] = *(gtab)(Th + to[p] + k0);
      if (SPLIT) v.tl[p] = *(gtab)(Tl + to[p] + k0);
    }
  };
  const int nf = K / KS, kt = nf * KS;
  const bool tail = kt < K;
  Held vt;
  auto fetch_tail = [&]() {
#pragma unroll
    for (int p = 0; p < XP; ++p) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int k = kt + 8 * sq + e;
        const float x = X[xo[p] - 8 * sq + min(k, K - 1)];
        if (e < 4) vt.x0[p][e & 3] = k < K ? x : 0.0f;
        else vt.x1[p][e & 3] = k < K ? x : 0.0f;
      }
      vt.th[p] = *(gtab)(Th + to[p] + min(kt, Kp - KS));
      if (SPLIT) vt.tl[p] = *(gtab)(Tl + to[p] + min(kt, Kp - KS));
    }
  };
  // buffer: X planes, then table planes, each [TR][KS], chunks swizzled
  auto stash = [&](const Held& v, uint16_t* buf) {
#pragma unroll
    for (int p = 0; p < XP; ++p) {
      const int o = lds_at<8>(sr + 32 * p, sq);
      const float xv[8] = {v.x0[p][0], v.x0[p][1], v.x0[p][2], v.x0[p][3],
                           v.x1[p][0], v.x1[p][1], v.x1[p][2], v.x1[p][3]};
      u16x8 h, l;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (SPLIT) {
          const __bf16 b = (__bf16)xv[e];
          h[e] = __builtin_bit_cast(uint16_t, b);
          l[e] = __builtin_bit_cast(uint16_t, (__bf16)(xv[e] - (float)b));
        } else {
          h[e] = __builtin_bit_cast(uint16_t, (_Float16)(xv[e] * xs));
        }
      }
      *reinterpret_cast<u16x8*>(buf + o) = h;
      *reinterpret_cast<u16x8*>(buf + NP * kPlane + o) = v.th[p];
      if (SPLIT) {
        *reinterpret_cast<u16x8*>(buf + kPlane + o) = l;
        *reinterpret_cast<u16x8*>(buf + NP * kPlane + kPlane + o) = v.tl[p];
      }
    }
  };
  const int wr = (w & 1) * (TR / 2), wc = (w >> 1) * (TR / 2);
  f32x4 acc[NT][NT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto product = [&](const uint16_t* buf, int chunks) {
    const uint16_t* A = buf;
    const uint16_t* B = buf + NP * kPlane;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      if (ks >= chunks) break;  // uniform: the last step may hold one chunk of 32
      const int q = 4 * ks + kq;
      u16x8 bh[NT], bl[NT];
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        bh[j] = *reinterpret_cast<const u16x8*>(B + lds_at<8>(wc + 16 * j + lr, q));
        if (SPLIT) bl[j] = *reinterpret_cast<const u16x8*>(B + kPlane + lds_at<8>(wc + 16 * j + lr, q));
      }
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        const u16x8 ah = *reinterpret_cast<const u16x8*>(A + lds_at<8>(wr + 16 * i + lr, q));
        u16x8 al;
        if (SPLIT) al = *reinterpret_cast<const u16x8*>(A + kPlane + lds_at<8>(wr + 16 * i + lr, q));
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          if (SPLIT) {
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, ah), __builtin_bit_cast(bf16x8, bh[j]), acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, ah), __builtin_bit_cast(bf16x8, bl[j]), acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, al), __builtin_bit_cast(bf16x8, bh[j]), acc[i][j], 0, 0, 0);
          } else {
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                __builtin_bit_cast(f16x8, ah), __builtin_bit_cast(f16x8, bh[j]), acc[i][j], 0, 0, 0);
          }
        }
      }
    }
  };
  uint16_t* cur = smem;
  uint16_t* nxt = smem + kBuf;
  auto swap = [&]() {
    uint16_t* const c = cur;
    cur = nxt;
    nxt = c;
  };
  // (past the last step the last one is fetched again: with as many loads in
  // flight on every path, the wait for one step's leaves the later ones' alone)
  Held va, vb;
  if (tail) fetch_tail();
  if (nf > 0) {
    fetch(va, 0);
    fetch(vb, min(1, nf - 1) * KS);
    stash(va, cur);
    fetch(va, min(2, nf - 1) * KS);
  } else {
    stash(vt, cur);
  }
  __syncthreads();
  auto step = [&](int s, Held& v) {
    stash(v, nxt);
    fetch(v, min(s + 3, nf - 1) * KS);
    product(cur, 2);
    __syncthreads();
    swap();
  };
  int s = 0;
  for (; s + 2 < nf; s += 2) {
    step(s, vb);
    step(s + 1, va);
  }
  if (s + 1 < nf) step(s, vb);
  if (nf > 0 && tail) {
    stash(vt, nxt);
    product(cur, 2);
    __syncthreads();
    swap();
  }
  product(cur, tail ? (K - kt + 31) / 32 : 2);
  // epilogue: lane holds D[row 4*(lane/16) + e][col lane mod 16] of each 16x16
  // tile; everything it reads is loaded before its first store
  const float inv_xs = SPLIT ? 1.0f : 1.0f / xs;
  const float* rv = reinterpret_cast<const float*>(a.rvec) + t.off;
  const unsigned char* iso = (a.iso && use_iso) ? a.iso + t.off : nullptr;
  float y[NT][NT][4];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) y[i][j][e] = acc[i][j][e] * inv_xs;
  auto row = [&](int i, int e) { return t.r0 + wr + 16 * i + 4 * kq + e; };
  auto col = [&](int j) { return t.c0 + wc + 16 * j + lr; };
  if (a.stage == 1) {
    const auto* lm = as_global(t.lam_m);
    const auto* ln = as_global(t.lam_n);
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int c = col(j), r = row(i, e);
          const double l = lm[min(c, K - 1)] + ln[min(r, R - 1)];
          y[i][j][e] = (c == 0 && r == 0) ? 0.0f : (float)((double)y[i][j][e] / l);
        }
  }
  double part = 0.0;
  if (a.stage == 3) {
    float rr[NT][NT][4];
    bool z[NT][NT][4];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool in = col(j) < K && row(i, e) < R;
          const size_t o = in ? (size_t)col(j) * R + row(i, e) : 0;
          rr[i][j][e] = in ? rv[o] : 0.0f;
          z[i][j][e] = iso && iso[o];
        }
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (z[i][j][e]) y[i][j][e] = 0.0f;
          part += (double)rr[i][j][e] * (double)y[i][j][e];
        }
  }
  float vmax = 0.0f;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int c = col(j);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int rb = row(i, 0);
      if (c >= K) continue;
      if (rb + 3 < R) {
        f32x4u v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = y[i][j][e];
        *reinterpret_cast<f32x4u*>(Out + (size_t)c * R + rb) = v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (rb + e < R) Out[(size_t)c * R + rb + e] = y[i][j][e];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (rb + e < R) vmax = fmaxf(vmax, fabsf(y[i][j][e]));
    }
  }
  if (!SPLIT && a.stage < 3) {
    // the next stage's scale: the largest output (an order-independent maximum)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) vmax = fmaxf(vmax, __shfl_down(vmax, off, 64));
    if (lane == 0) fmx[w] = vmax;
    __syncthreads();
    if (tid == 0) {
      vmax = fmaxf(fmaxf(fmx[0], fmx[1]), fmaxf(fmx[2], fmx[3]));
      // one address takes its atomics one at a time: only a block that raises
      // the value it finds there adds one
      if (vmax > __hip_atomic_load(amax_out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(reinterpret_cast<unsigned int*>(amax_out), __float_as_uint(vmax));
    }
  }
  if (a.stage == 3) {
    double vv[1] = {part};
    block_sum<1>(vv, red);
    if (tid == 0) store_partial(a.P + 1 * a.pstride + g, vv[0]);
  }
}

// TMAX: the larger of the tile sides in the launch (launches of small maps only
// take the instance for side 32, whose LDS and registers leave room for more
// blocks on a CU).
template <int SPLIT, int TMAX>
__global__ void __launch_bounds__(256, TMAX == 64 ? 2 : 4) k_e_dct_dense(DArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t smem[2 * 2 * (SPLIT ? 2 : 1) * TMAX * 64];
  __shared__ double red[4];
  __shared__ double fred[3 * 4];
  __shared__ float fmx[4];
  __shared__ int fflag;
  const int nact = a.counts[a.cidx];
  // the block's first list entry is requested with the list's length
  const int g_first = a.dact[min((int)blockIdx.x, max(a.dact_cap - 1, 0))];
  __asm__ volatile("" ::"s"(nact), "s"(g_first));  // both loads issued before the loop test
  for (int t_ = blockIdx.x; t_ < nact; t_ += gridDim.x) {
    const int g = t_ == (int)blockIdx.x ? g_first : a.dact[t_];
    if (g < 0) continue;  // padding slot of the XCD-ordered list
    const EoTile t = a.eot[(size_t)(a.stage & 1) * a.eot_cap + g];
    const bool use_iso = a.desc[t.m].use_iso != 0;
    MapState& st = a.ms[t.m];
    float xs = 1.0f;
    if (!SPLIT) xs = fp16_scale(a.stage == 0 ? (float)sqrt(st.rr) * 1.0000001f : st.amax[a.stage]);
    if (st.state != a.expect) continue;  // uniform over the block
    float* amax = a.stage < 3 ? &st.amax[a.stage + 1] : nullptr;
    if (TMAX == 64 && t.side == 64)
      dct_dense_tile<SPLIT, TMAX>(a, t, use_iso, g, xs, amax, smem, red, fmx);
    else
      dct_dense_tile<SPLIT, 32>(a, t, use_iso, g, xs, amax, smem, red, fmx);
    if (a.stage == 3 && a.fin_mode) {
      const int sl[1] = {1};
      fused_finish<kFinTail, 1>(Arrival{a.fcnt, a.gcnt, a.gsum, a.gstride, a.P, a.pstride}, sl,
                                g - t.local, t.local, t.ndt, t.gbd, a.desc, a.ms, t.m, a.fin_mode, 0,
                                &fflag, fred);
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// FP64 stage: even/odd split on the FP64 matrix cores, any side length.
//
// With h = ceil(n/2) and h2 = floor(n/2) the fold of the even/odd kernel above
// holds for every n (an odd n's middle element has no mirror and joins the
// even outputs only):
//   forward  X_2c = sum_{j<h} C[2c][j] a_j,  X_2c+1 = sum_{j<h2} C[2c+1][j] d_j,
//            a_j = x_j + x_{n-1-j}, d_j = x_j - x_{n-1-j}  (middle: a = x);
//   inverse  u_j = sum_{k<h} C[2k][j] X_2k,  v_j = sum_{k<h2} C[2k+1][j] X_2k+1,
//            x_j = u_j + v_j, x_{n-1-j} = u_j - v_j,
// half the multiply-adds of the plain product.  Spectra are kept in split
// order (even k first).  Both halves' table rows are rows of C (forward) and
// of C^T (inverse, even and odd entries side by side) as they are.
//
// A block (4 waves) owns TR rows of X and TR / 2 output pairs; wave w computes
// half w >> 1 of rows (TR / 2)(w & 1) .., as MFMA tiles of 16 x 16 x 4 with the
// table as the first operand, so that a lane's results lie along the rows and
// the transposed store is contiguous over 16 lanes.  K steps of 32 are folded
// on the way from registers to LDS (two buffers; rows of 34 doubles: the fragment reads, 16
// rows of 4 consecutive values, touch every bank equally often); the next step's
// loads are in flight during the current one's MFMAs.  The last, partial step
// has its own guarded loads, ahead of the loop, which has none.
//
// Which tile: 64 x 64 (K steps of 16, two blocks on a CU) halves the traffic
// per product of 32 x 32 (steps of 32, three blocks), which gives four times as
// many tiles.  One PCG iteration, the four stages the larger part of it, with
// tiles of 64 and of 32: 5.3 and 7.0 ms at 4096^2, 756 and 960 us at 2048^2,
// 179 and 193 at 1024^2, 290 and 307 at 1000 x 1500 (384 tiles), but 156 and
// 148 at 720 x 960 (180 tiles), 145 and 132 at 768^2, 134 and 113 at 509 x 733,
// 66 and 58 at 64^2: so maps of at least kF64Wide tiles of 64 x 64 take those.
// The choice is the map's alone: its results do not depend on its batch-mates.
// The plain FMA product it replaces took 18.3 ms, 2288, 656, 949, 548, 503, 557
// and 94 us.  Large maps run at 55 TFLOP/s of the 74 a large FP64 product
// reaches here; small ones are bound by the latency of one tile's steps.
// ---------------------------------------------------------------------------
constexpr int kF64Wide = 224;

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2u __attribute__((ext_vector_type(2), aligned(8)));

template <int INV, int TR>
__device__ __forceinline__ void dct_f64_tile(const DArgs& a, const EoTile& t, bool use_iso, int g,
                                             double* smem, double* red) {
  constexpr int TP = TR / 2;             // output pairs
  constexpr int KS = TR == 64 ? 16 : 32, P = KS + 2;  // K step, LDS row pitch
  constexpr int NI = TR / 32, NJ = TP / 16;  // 16-row and 16-pair tiles per wave
  constexpr int TPR = KS / 2, RP = 256 / TPR;  // staging: threads per row, rows per pass
  constexpr int XP = TR / RP, QP = TP / RP;    // staging passes
  constexpr int kBuf = 2 * (TR + TP) * P;  // doubles of one K step's operands
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int hf = w >> 1, wr = (w & 1) * (TR / 2), l16 = lane & 15, lq = lane >> 4;
  const int R = t.R, n = t.K, h = (n + 1) >> 1, h2 = n >> 1, r0 = t.r0, c0 = t.c0;
  const double* X = reinterpret_cast<const double*>(a.X) + t.off;
  double* Out = reinterpret_cast<double*>(a.Out) + t.off;
  const auto* T = as_global(INV ? t.ct64 : t.c64);
  const int sr = tid / TPR, sk = tid % TPR * 2;  // staging: row of a pass, first of two k
  // rows and pairs past the map repeat the last one (their results are dropped)
  size_t xo[XP];
  size_t to[QP], to1[QP];
#pragma unroll
  for (int p = 0; p < XP; ++p) xo[p] = (size_t)min(r0 + sr + RP * p, R - 1) * n;
#pragma unroll
  for (int p = 0; p < QP; ++p) {
    const int c = min(c0 + sr + RP * p, h - 1);
    to[p] = INV ? (size_t)c * n : (size_t)(2 * c) * n;
    to1[p] = (size_t)min(2 * c + 1, n - 1) * n;  // forward: the odd output's row
  }
  struct Held {  // one K step's operands on the way to LDS
    f64x2u xa[XP], xb[XP], ta[QP], tb[QP];
  };
  using gvec = const __attribute__((address_space(1))) f64x2u*;
  auto fetch = [&](Held& v, int k0) {
    const int k = k0 + sk;
#pragma unroll
    for (int p = 0; p < XP; ++p) {
      v.xa[p] = *reinterpret_cast<const f64x2u*>(X + xo[p] + k);
      v.xb[p] = *reinterpret_cast<const f64x2u*>(X + xo[p] + (INV ? h + k : n - 2 - k));
    }
#pragma unroll
    for (int p = 0; p < QP; ++p) {
      v.ta[p] = *(gvec)(INV ? T + to[p] + 2 * k : T + to[p] + k);
      v.tb[p] = *(gvec)(INV ? T + to[p] + 2 * k + 2 : T + to1[p] + k);
    }
  };
  // a buffer: X [half][TR][P], then the table [half][TP][P]
  auto put = [&](double* base, int rows, int half, int row, double v0, double v1) {
    double* q = base + (half * rows + row) * P + sk;
    q[0] = v0;
    q[1] = v1;
  };
  // one of the XP + QP pieces of a step's way into LDS
  auto stash = [&](const Held& v, double* Xs, int p) {
    double* Ts = Xs + 2 * TR * P;
    if (p < XP) {
      const int row = sr + RP * p;
      if (INV) {
        put(Xs, TR, 0, row, v.xa[p][0], v.xa[p][1]);
        put(Xs, TR, 1, row, v.xb[p][0], v.xb[p][1]);
      } else {
        put(Xs, TR, 0, row, v.xa[p][0] + v.xb[p][1], v.xa[p][1] + v.xb[p][0]);
        put(Xs, TR, 1, row, v.xa[p][0] - v.xb[p][1], v.xa[p][1] - v.xb[p][0]);
      }
    } else {
      const int q = p - XP, row = sr + RP * q;
      if (INV) {
        put(Ts, TP, 0, row, v.ta[q][0], v.tb[q][0]);
        put(Ts, TP, 1, row, v.ta[q][1], v.tb[q][1]);
      } else {
        put(Ts, TP, 0, row, v.ta[q][0], v.ta[q][1]);
        put(Ts, TP, 1, row, v.tb[q][0], v.tb[q][1]);
      }
    }
  };
  // the last, partial step (from k = nf * KS), requested with the first one:
  // X zero past its half's length, table indices clamped into the row (any
  // finite value does there)
  const int nf = h2 / KS, kt = nf * KS + sk;
  const bool tail = nf * KS < h;
  double ya[XP][2], yb[XP][2], ua[QP][2], ub[QP][2];
  auto fetch_tail = [&]() {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int k = kt + e;
#pragma unroll
      for (int p = 0; p < XP; ++p) {
        ya[p][e] = X[xo[p] + min(k, h - 1)];
        yb[p][e] = X[xo[p] + (INV ? min(h + k, n - 1) : max(n - 1 - k, 0))];
      }
#pragma unroll
      for (int p = 0; p < QP; ++p) {
        ua[p][e] = T[to[p] + min(INV ? 2 * k : k, n - 1)];
        ub[p][e] = INV ? T[to[p] + min(2 * k + 1, n - 1)] : T[to1[p] + min(k, n - 1)];
      }
    }
  };
  auto stash_tail = [&](double* Xs) {
    double* Ts = Xs + 2 * TR * P;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int k = kt + e;
#pragma unroll
      for (int p = 0; p < XP; ++p) {
        const int row = sr + RP * p;
        const double a0 = INV ? ya[p][e] : (k < h2 ? ya[p][e] + yb[p][e] : ya[p][e]);
        const double a1 = INV ? yb[p][e] : ya[p][e] - yb[p][e];
        Xs[(0 * TR + row) * P + sk + e] = k < h ? a0 : 0.0;
        Xs[(1 * TR + row) * P + sk + e] = k < h2 ? a1 : 0.0;
      }
#pragma unroll
      for (int p = 0; p < QP; ++p) {
        const int row = sr + RP * p;
        Ts[(0 * TP + row) * P + sk + e] = ua[p][e];
        Ts[(1 * TP + row) * P + sk + e] = ub[p][e];
      }
    }
  };
  f64x4 acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  // the products of one K step from buffer Xs; with NEXT, the next step's
  // pieces go to buffer Xn between them (a product occupies the matrix core
  // for 64 cycles, in which the wave can issue them)
  auto product = [&](const Held* next, const double* Xs, double* Xn) {
    const double* Xw = Xs + (hf * TR + wr + l16) * P + lq;
    const double* Tw = Xs + 2 * TR * P + (hf * TP + l16) * P + lq;
#pragma unroll
    for (int s = 0; s < KS; s += 4) {
      double xv[NI], tv[NJ];
#pragma unroll
      for (int i = 0; i < NI; ++i) xv[i] = Xw[16 * i * P + s];
#pragma unroll
      for (int j = 0; j < NJ; ++j) tv[j] = Tw[16 * j * P + s];
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(tv[j], xv[i], acc[i][j], 0, 0, 0);
      if (next && s / 4 < XP + QP) stash(*next, Xn, s / 4);
    }
  };
  // two buffers, one barrier per step; a step's operands are requested two
  // steps before its products
  double* cur = smem;
  double* nxt = smem + kBuf;
  Held va, vb;
  if (nf > 0) {
    // (past the last step the last one is fetched again: with as many loads in
    // flight on every path, the wait for one step's leaves the next one's alone)
    fetch_tail();
    fetch(va, 0);
    fetch(vb, min(1, nf - 1) * KS);
#pragma unroll
    for (int p = 0; p < XP + QP; ++p) stash(va, cur, p);
    fetch(va, min(2, nf - 1) * KS);
  } else {
    fetch_tail();
    stash_tail(cur);
  }
  __syncthreads();
  auto step = [&](int s, Held& v) {
    product(&v, cur, nxt);
    fetch(v, min(s + 3, nf - 1) * KS);
    __syncthreads();
    double* const c = cur;
    cur = nxt;
    nxt = c;
  };
  int s = 0;
  for (; s + 2 < nf; s += 2) {
    step(s, vb);
    step(s + 1, va);
  }
  if (s + 1 < nf) step(s, vb);
  if (nf > 0 && tail) {
    product(nullptr, cur, nullptr);
    stash_tail(nxt);
    __syncthreads();
    cur = nxt;
  }
  product(nullptr, cur, nullptr);
  // a lane holds outputs of row l16 (of each 16) at pairs lq + 4 e (of each 16)
  const double* rv = reinterpret_cast<const double*>(a.rvec) + t.off;
  const unsigned char* iso = (a.iso && use_iso) ? a.iso + t.off : nullptr;
  double y[NI][NJ][4];
  if (!INV) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) y[i][j][e] = acc[i][j][e];
  } else {
    // u (half 0) and v (half 1) of the same rows meet through LDS
    __syncthreads();
    double* xg = smem + w * (NI * NJ * 4 * 64) + lane;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) xg[((i * NJ + j) * 4 + e) * 64] = acc[i][j][e];
    __syncthreads();
    const double* og = smem + (w ^ 2) * (NI * NJ * 4 * 64) + lane;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double o = og[((i * NJ + j) * 4 + e) * 64];
          const int pair = c0 + 16 * j + lq + 4 * e;
          // the middle of an odd side: no v
          y[i][j][e] = hf ? o - acc[i][j][e] : (pair < h2 ? acc[i][j][e] + o : acc[i][j][e]);
        }
  }
  // output index of pair element (j, e), or -1; row of i
  auto out_c = [&](int j, int e) {
    const int pair = c0 + 16 * j + lq + 4 * e;
    if (pair >= (hf ? h2 : h)) return -1;
    return INV ? (hf ? n - 1 - pair : pair) : (hf ? h + pair : pair);
  };
  double part = 0.0;
  if (!INV && a.stage == 1) {
    // spectrum ./ Lambda, zero mode dropped; indices in split order
    const auto* lm = as_global(t.lam_m);
    const auto* ln = as_global(t.lam_n);
    const int hR = (R + 1) >> 1;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = min(r0 + wr + 16 * i + l16, R - 1);
      const double lr = ln[r < hR ? 2 * r : 2 * (r - hR) + 1];
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int k = min(2 * (c0 + 16 * j + lq + 4 * e) + hf, n - 1);
          y[i][j][e] = k == 0 && r == 0 ? 0.0 : y[i][j][e] / (lm[k] + lr);
        }
    }
  }
  if (INV && a.stage == 3) {
    // zero on isolated pixels; FP64 partial of r^T s
    double rr[NI][NJ][4];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int c = out_c(j, e), r = r0 + wr + 16 * i + l16;
          const bool in = c >= 0 && r < R;
          const size_t o = in ? (size_t)c * R + r : 0;
          rr[i][j][e] = in ? rv[o] : 0.0;
          if (iso && iso[o]) y[i][j][e] = 0.0;
        }
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) part += rr[i][j][e] * y[i][j][e];
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int r = r0 + wr + 16 * i + l16;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = out_c(j, e);
        if (c >= 0 && r < R) Out[(size_t)c * R + r] = y[i][j][e];
      }
  }
  if (INV && a.stage == 3) {
    double vv[1] = {part};
    block_sum<1>(vv, red);
    if (tid == 0) store_partial(a.P + 1 * a.pstride + g, vv[0]);
  }
}

// TMAX: the larger of the tile sides in the launch.  Launches of small maps
// only take the instance for side 32, whose LDS leaves room for three blocks on
// a CU (side 64: two).
template <int INV, int TMAX>
__global__ void __launch_bounds__(256, 2) k_e_dct_f64(DArgs a) {
  // two K steps' operands; the inverse's exchange fits in them
  __shared__ __attribute__((aligned(16))) double smem[TMAX == 64 ? 2 * 2 * 96 * 18 : 2 * 2 * 48 * 34];
  __shared__ double red[4];
  __shared__ double fred[3 * 4];
  __shared__ int fflag;
  const int nact = a.counts[a.cidx];
  // the block's first list entry is requested with the list's length
  const int g_first = a.dact[min((int)blockIdx.x, max(a.dact_cap - 1, 0))];
  __asm__ volatile("" ::"s"(nact), "s"(g_first));  // both loads issued before the loop test
  for (int t_ = blockIdx.x; t_ < nact; t_ += gridDim.x) {
    const int g = t_ == (int)blockIdx.x ? g_first : a.dact[t_];
    if (g < 0) continue;  // padding slot of the XCD-ordered list
    const EoTile t = a.eot[(size_t)(a.stage & 1) * a.eot_cap + g];
    const bool use_iso = a.desc[t.m].use_iso != 0;
    if (a.ms[t.m].state != a.expect) continue;  // uniform over the block
    if (TMAX == 64 && t.side == 64) dct_f64_tile<INV, TMAX>(a, t, use_iso, g, smem, red);
    else dct_f64_tile<INV, 32>(a, t, use_iso, g, smem, red);
    if (INV && a.stage == 3 && a.fin_mode) {
      const int sl[1] = {1};
      fused_finish<kFinTail, 1>(Arrival{a.fcnt, a.gcnt, a.gsum, a.gstride, a.P, a.pstride}, sl,
                                g - t.local, t.local, t.ndt, t.gbd, a.desc, a.ms, t.m, a.fin_mode, 0,
                                &fflag, fred);
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// FMA stage (FP32 option): 64 x 64 tile, 16 x 16 threads x 4 x 4.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_e_dct_fma(DArgs a) {
  using T = float;
  __shared__ T Xs[16][64 + 4];
  __shared__ T Bs[16][64 + 4];
  __shared__ double red[4];
  const int nact = a.counts[a.cidx];
  // the block's first list entry is requested with the list's length
  const int g_first = a.dact[min((int)blockIdx.x, max(a.dact_cap - 1, 0))];
  __asm__ volatile("" ::"s"(nact), "s"(g_first));  // both loads issued before the loop test
  const int tid = threadIdx.x, tr = tid % 16, tc = tid / 16;
  const int lrow = tid / 4, lk = (tid % 4) * 4;
  for (int t_ = blockIdx.x; t_ < nact; t_ += gridDim.x) {
    const int g = t_ == (int)blockIdx.x ? g_first : a.dact[t_];
    if (g < 0) continue;  // padding slot of the XCD-ordered list
    const DTile t = dtile(a, g);
    if (!t.ok) continue;
    const int R = t.R, K = t.K, r0 = t.r0, c0 = t.c0;
    const T* X = reinterpret_cast<const T*>(a.X) + t.off;
    T* Out = reinterpret_cast<T*>(a.Out) + t.off;
    const T* B;
    B = reinterpret_cast<const T*>(a.stage < 2 ? (const void*)t.tab->c32 : (const void*)t.tab->ct32);
    T acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = T(0);
    for (int k0 = 0; k0 < K; k0 += 16) {
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = k0 + lk + e, rr = r0 + lrow, cc = c0 + lrow;
        Xs[lk + e][lrow] = (rr < R && k < K) ? X[(size_t)rr * K + k] : T(0);
        Bs[lk + e][lrow] = (cc < K && k < K) ? as_global(B)[(size_t)cc * K + k] : T(0);
      }
      __syncthreads();
#pragma unroll
      for (int kk = 0; kk < 16; ++kk) {
        T xa[4], bb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) xa[i] = Xs[kk][4 * tr + i];
#pragma unroll
        for (int j = 0; j < 4; ++j) bb[j] = Bs[kk][4 * tc + j];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] += xa[i] * bb[j];
      }
    }
    const MapDesc& d = a.desc[t.m];
    const T* rv = reinterpret_cast<const T*>(a.rvec) + t.off;
    const unsigned char* iso = (a.iso && d.use_iso) ? a.iso + t.off : nullptr;
    double part = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = c0 + 4 * tc + j;
      if (c >= K) continue;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = r0 + 4 * tr + i;
        if (r >= R) continue;
        const size_t o = (size_t)c * R + r;
        T v = acc[i][j];
        if (a.stage == 1) v = (c == 0 && r == 0) ? T(0) : (T)((double)v / (as_global(d.tabM->lam)[c] + as_global(d.tabN->lam)[r]));
        if (a.stage == 3) {
          if (iso && iso[o]) v = T(0);
          part += (double)rv[o] * (double)v;
        }
        Out[o] = v;
      }
    }
    if (a.stage == 3) {
      double vv[1] = {part};
      block_sum<1>(vv, red);
      if (tid == 0) a.P[1 * a.pstride + g] = vv[0];
    }
    __syncthreads();
  }
}

// Tile side of the FP64 and the dense MFMA stages for an M x N map (a function
// of the map alone).
int dct_side(int M, int N, bool fp64) {
  const long long t = (long long)((M + 63) / 64) * ((N + 63) / 64);
  return t >= (fp64 ? kF64Wide : kDenseWide) ? 64 : 32;
}

// An upper bound of the DCT tiles of any one map of at most M x N, in every kind of
// stage: below the rule's line (kF64Wide tiles of 64 x 64, the higher one) a map has up
// to four tiles of 32 x 32 for each of 64 x 64, so a smaller map can have more tiles than
// a larger one.
int dct_tiles_most(int M, int N) {
  auto tiles = [&](int side) { return (long long)((M + side - 1) / side) * ((N + side - 1) / side); };
  static_assert(kF64Wide >= kDenseWide, "the higher line");
  return (int)std::max(tiles(64), std::min(tiles(32), 4LL * (kF64Wide - 1)));
}

// Tile shape of the even/odd stages (k_e_dct_eo): 0 fine, 1 narrow, 2 wide in
// the first three stages, 3 wide in all; elsewhere 1 if the instances that take
// tiles of 64 x 64 run, else 0.  It changes no result and is part of the
// captured graphs' key.
//
// Four stages, us, of fine / narrow / wide tiles, scaled fp16 (narrow list
// positions): 512^2 (16) 39 / 67 / 60, 1024^2 (64) 36 / 55 / 88, 1536^2 (144)
// 81 / 74 / 118, 2048^2 (256) 128 / 96 / 148, 2560^2 (400) 275 / 167 / 189,
// 3072^2 (576) 366 / 282 / 277, 4096^2 (1024) 832 / 507 / 386; bf16 split: 64 /
// 116, 169 / 171, 265 / 228 at 1024^2 to 2048^2.  The last stage, with its FP32
// output and reads of r, gains from wide tiles later: 70 / 82 us at 576
// positions, 122 / 109 at 1024.
constexpr int kFineMax = 128;
constexpr int kWideMin = 576;
constexpr int kWideLastMin = 1024;

int dct_shape_for(const Engine& e, int ndtiles, int kind) {
  if (kind < 4) return e.dct_tile64 ? 1 : 0;
  if (ndtiles < kFineMax) return 0;
  if (kind != 5 || ndtiles < kWideMin) return 1;
  return ndtiles < kWideLastMin ? 2 : 3;
}

// Grid of a DCT stage: the next power of two >= the list length (fine tiles: four
// blocks to an entry), capped; a multiple of 8, so list position q always runs on
// XCD q mod 8.
int dct_grid_for(const Engine& e, int ndtiles, int kind) {
  const long long blocks = kind >= 4 && dct_shape_for(e, ndtiles, kind) == 0 ? 4LL * ndtiles : ndtiles;
  const int cap = std::max(8, e.dct_grid / 8 * 8);
  int g = 8;
  while (g < blocks && g < cap) g <<= 1;
  return std::min(g, cap);
}

void e_dct_stage(hipStream_t st, const Engine& e, int ndtiles, int stage, int expect, int kind,
                 const void* X, void* Out, const void* rvec, int fin_mode) {
  const int shape = dct_shape_for(e, ndtiles, kind);
  const bool fine = kind >= 4 && shape == 0;
  const bool wide = kind >= 4 && (shape == 3 || (shape == 2 && stage < 3));
  const int grid = dct_grid_for(e, ndtiles, kind);
  DArgs a;
  a.fcnt = e.fcnt;
  a.gcnt = e.gcnt;
  a.gsum = e.gsum;
  a.gstride = e.gstride;
  a.eot = e.eot;
  a.eot_cap = e.caps.dtiles;
  // the finisher rides on the last stage of every kernel but the FP32 FMA one
  a.fin_mode = (stage == 3 && kind != 1) ? fin_mode : 0;
  a.desc = e.desc;
  a.ms = e.ms;
  a.dtile_map = e.dtile_map;
  // lists: narrow tiles of the two stage parities, then wide tiles
  a.dact = e.dact + ((wide ? 2 : 0) + (stage & 1)) * e.dlist_cap;
  a.dact_cap = (int)e.dlist_cap;
  a.cidx = (wide ? 4 : 0) + ((stage & 1) ? 3 : 1);
  a.counts = e.counts;
  a.P = e.P;
  a.pstride = e.pstride;
  a.X = X;
  a.Out = Out;
  a.rvec = rvec;
  a.iso = e.iso;
  a.stage = stage;
  a.expect = expect;
  // kind: 0 FP64 MFMA, 1 FP32 FMA, 2 split-bf16 MFMA, 3 scaled-fp16 MFMA;
  // +2 (kinds 4, 5): the even/odd MFMA kernels (every side a multiple of 128)
  // (FP64 and dense: the instance that takes tiles of 64 x 64 as well, if any map has them)
  if (kind == 0 && e.dct_tile64) {
    if (stage < 2) hipLaunchKernelGGL((k_e_dct_f64<0, 64>), dim3(grid), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_e_dct_f64<1, 64>), dim3(grid), dim3(256), 0, st, a);
  } else if (kind == 0) {
    if (stage < 2) hipLaunchKernelGGL((k_e_dct_f64<0, 32>), dim3(grid), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_e_dct_f64<1, 32>), dim3(grid), dim3(256), 0, st, a);
  }
  else if (kind == 1) hipLaunchKernelGGL(k_e_dct_fma, dim3(grid), dim3(256), 0, st, a);
  else if (kind == 2 && e.dct_tile64) hipLaunchKernelGGL((k_e_dct_dense<1, 64>), dim3(grid), dim3(256), 0, st, a);
  else if (kind == 2) hipLaunchKernelGGL((k_e_dct_dense<1, 32>), dim3(grid), dim3(256), 0, st, a);
  else if (kind == 3 && e.dct_tile64) hipLaunchKernelGGL((k_e_dct_dense<0, 64>), dim3(grid), dim3(256), 0, st, a);
  else if (kind == 3) hipLaunchKernelGGL((k_e_dct_dense<0, 32>), dim3(grid), dim3(256), 0, st, a);
  // scaled fp16 even/odd: intermediates between the stages are stored as
  // scaled fp16 (first stage reads FP32 r, last stage writes FP32 s)
  else if (kind == 4 && stage < 2) {
    if (fine) hipLaunchKernelGGL((k_e_dct_eo<1, 0, 0, 0, 2, 2>), dim3(grid), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_e_dct_eo<1, 0, 0, 0, 4, 4>), dim3(grid), dim3(256), 0, st, a);
  } else if (kind == 4) {
    if (fine) hipLaunchKernelGGL((k_e_dct_eo<1, 1, 0, 0, 2, 2>), dim3(grid), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_e_dct_eo<1, 1, 0, 0, 4, 4>), dim3(grid), dim3(256), 0, st, a);
  } else if (stage == 0) {
    if (fine) hipLaunchKernelGGL((k_e_dct_eo<0, 0, 0, 1, 2, 2>), dim3(grid), dim3(256), 0, st, a);
    else if (wide) hipLaunchKernelGGL((k_e_dct_eo<0, 0, 0, 1, 4, 8>), dim3(grid), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_e_dct_eo<0, 0, 0, 1, 4, 4>), dim3(grid), dim3(256), 0, st, a);
  } else if (stage == 1) {
    if (fine) hipLaunchKernelGGL((k_e_dct_eo<0, 0, 1, 1, 2, 2>), dim3(grid), dim3(256), 0, st, a);
    else if (wide) hipLaunchKernelGGL((k_e_dct_eo<0, 0, 1, 1, 4, 8>), dim3(grid), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_e_dct_eo<0, 0, 1, 1, 4, 4>), dim3(grid), dim3(256), 0, st, a);
  } else if (stage == 2) {
    if (fine) hipLaunchKernelGGL((k_e_dct_eo<0, 1, 1, 1, 2, 2>), dim3(grid), dim3(256), 0, st, a);
    else if (wide) hipLaunchKernelGGL((k_e_dct_eo<0, 1, 1, 1, 4, 8>), dim3(grid), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_e_dct_eo<0, 1, 1, 1, 4, 4>), dim3(grid), dim3(256), 0, st, a);
  } else {
    if (fine) hipLaunchKernelGGL((k_e_dct_eo<0, 1, 1, 0, 2, 2>), dim3(grid), dim3(256), 0, st, a);
    else if (wide) hipLaunchKernelGGL((k_e_dct_eo<0, 1, 1, 0, 4, 8>), dim3(grid), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_e_dct_eo<0, 1, 1, 0, 4, 4>), dim3(grid), dim3(256), 0, st, a);
  }
}

}  // namespace lpu
