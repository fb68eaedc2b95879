// DCT tables for the fast-Poisson preconditioner.
//
// C_n[k][j] = s_k cos(pi k (2j + 1) / (2n)), s_0 = sqrt(1/n), s_k = sqrt(2/n)
// (orthonormal DCT-II), its transpose, and the eigenvalues 2 - 2 cos(pi k / n)
// of the unit-weight 1-D Neumann Laplacian, stored in every arithmetic the
// contraction kernels use: FP64, FP32, a bf16 hi/lo split (hi = bf16(c), lo =
// bf16(c - hi)) and fp16.
//
// An n x n table holds only the 4n values sqrt(2/n) cos(pi m / (2n)), m = k (2j + 1)
// mod 4n: these are evaluated on the host in long double and the tables filled
// on the device, 48 bytes of stores per entry of C.  Evaluating and converting
// every entry on the host and copying the tables up took most of a first solve:
// 2.72 s of a 4096^2 one, now 92 ms (a repeated one 86), 178 ms at 1024^2, now
// 15.7 (13.4), 119 ms at 480 x 640, now 13.7 (13.5).

#include <algorithm>
#include <cmath>
#include <vector>

#include "lpu_internal.h"

namespace lpu {

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  const uint32_t lsb = (u >> 16) & 1u;
  u += 0x7FFFu + lsb;
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Position of (row, col) in a matrix of K columns kept in blocks of 16 rows by
// 32 columns (the layout the even/odd kernels read, eo_at).
__device__ __forceinline__ size_t block_at(size_t row, size_t col, size_t K) {
  return row / 16 * 16 * K + col / 32 * 512 + row % 16 * 32 + col % 32;
}

// C[k][j] from q[m] = sqrt(2/n) cos(pi m / (2n)), m < 4n.
__device__ __forceinline__ double entry(const double* __restrict__ q, double s0, int n, int k, int j) {
  return k == 0 ? s0 : q[(unsigned long long)k * (2ull * j + 1) % (4ull * n)];
}

// One 16-bit triple (bf16 hi and lo, fp16) of a value rounded to FP32 first:
// the barrier keeps the compiler from rounding the FP64 value to fp16 at once,
// which differs where the FP32 value lies halfway (one value at n = 4096).
__device__ __forceinline__ void put16(float v, uint16_t* hi, uint16_t* lo, uint16_t* h, size_t o) {
  __asm__ volatile("" : "+v"(v));
  const uint16_t b = f32_to_bf16_rne(v);
  hi[o] = b;
  lo[o] = f32_to_bf16_rne(v - bf16_to_f32(b));
  h[o] = __builtin_bit_cast(uint16_t, (_Float16)v);
}

// The dense tables, C (TR = 0) or C^T (TR = 1): element (row, col) of rows
// padded with zeros to np columns in the 16-bit ones.  One pass of stores, 24
// bytes an element: the memory's write rate bounds it.
template <int TR>
__global__ void __launch_bounds__(256) k_dct_dense_tables(const double* __restrict__ q, double s0,
                                                          int n, int np, double* c64, float* c32,
                                                          uint16_t* hi, uint16_t* lo, uint16_t* h) {
  const size_t total = (size_t)n * np;
  for (size_t o = blockIdx.x * (size_t)256 + threadIdx.x; o < total; o += gridDim.x * (size_t)256) {
    const int row = (int)(o / np), col = (int)(o % np);
    float v = 0.0f;
    if (col < n) {
      const double c = TR ? entry(q, s0, n, col, row) : entry(q, s0, n, row, col);
      v = (float)c;
      c64[(size_t)row * n + col] = c;
      c32[(size_t)row * n + col] = v;
    }
    put16(v, hi, lo, h, o);
  }
}

// The even/odd tables EO[c][j] and EOt[j][c], c < n in split order, j < n / 2, in
// blocks of 16 x 32: C[k][n-1-j] = (-1)^k C[k][j].
__global__ void __launch_bounds__(256) k_dct_eo_tables(const double* __restrict__ q, double s0, int n,
                                                       uint16_t* eh, uint16_t* el, uint16_t* e16,
                                                       uint16_t* th, uint16_t* tl, uint16_t* t16) {
  const int h = n / 2;
  const size_t total = (size_t)n * h;
  for (size_t o = blockIdx.x * (size_t)256 + threadIdx.x; o < total; o += gridDim.x * (size_t)256) {
    const int c = (int)(o / h), j = (int)(o % h);
    const float v = (float)entry(q, s0, n, c < h ? 2 * c : 2 * (c - h) + 1, j);
    put16(v, eh, el, e16, block_at(c, j, h));
    put16(v, th, tl, t16, block_at(j, c, n));
  }
}

static void free_tables(DctTables& t) {
  void* tp[] = {t.c64,   t.ct64,   t.c32,  t.ct32,   t.c_hi,   t.c_lo, t.ct_hi,    t.ct_lo, t.c_h,
                t.ct_h,  t.lam,    t.eo_hi, t.eo_lo, t.eo_h, t.eot_hi, t.eot_lo, t.eot_h, t.lam_split};
  for (void* p : tp)
    if (p) (void)hipFree(p);
}

const DctTables* get_dct_tables(lp_unwrap_ctx* ctx, int n, int* status) {
  for (auto& t : ctx->dct)
    if (t.n == n) {
      *status = LPU_OK;
      return &t;
    }
  const long double pi = 3.141592653589793238462643383279502884L;
  DctTables t;
  t.n = n;
  const size_t nn = (size_t)n * n;
  // rows of the dense 16-bit tables padded with zeros to whole K steps
  const size_t np = ((size_t)n + 63) / 64 * 64, nnp = (size_t)n * np;
  const bool eo = n % 128 == 0;
  const size_t nh = (size_t)n * (n / 2);
  std::vector<double> lam(n), ls(n), q(4 * (size_t)n);
  for (int k = 0; k < n; ++k) lam[k] = (double)(2.0L - 2.0L * std::cos(pi * k / n));
  for (int c = 0; eo && c < n; ++c) ls[c] = lam[c < n / 2 ? 2 * c : 2 * (c - n / 2) + 1];
  for (int m = 0; m < 4 * n; ++m)
    q[m] = (double)(std::sqrt(2.0L / n) * std::cos(pi * m / (2.0L * n)));
  const double s0 = (double)std::sqrt(1.0L / n);
  bool ok = true;
  double* dq = nullptr;
  auto get = [&](auto** dst, size_t count) {
    if (ok) ok = hipMalloc((void**)dst, count * sizeof(**dst)) == hipSuccess;
  };
  auto up = [&](double** dst, const std::vector<double>& src) {
    get(dst, src.size());
    if (ok) ok = hipMemcpy(*dst, src.data(), src.size() * 8, hipMemcpyHostToDevice) == hipSuccess;
  };
  get(&t.c64, nn);
  get(&t.ct64, nn);
  get(&t.c32, nn);
  get(&t.ct32, nn);
  for (uint16_t** p : {&t.c_hi, &t.c_lo, &t.ct_hi, &t.ct_lo, &t.c_h, &t.ct_h}) get(p, nnp);
  up(&t.lam, lam);
  up(&dq, q);
  if (eo) {
    for (uint16_t** p : {&t.eo_hi, &t.eo_lo, &t.eo_h, &t.eot_hi, &t.eot_lo, &t.eot_h}) get(p, nh);
    up(&t.lam_split, ls);
  }
  if (ok) {
    hipStream_t st = ctx->stream;
    const int grid = (int)std::min<size_t>(4096, (nnp + 255) / 256);
    hipLaunchKernelGGL(k_dct_dense_tables<0>, dim3(grid), dim3(256), 0, st, dq, s0, n, (int)np, t.c64,
                       t.c32, t.c_hi, t.c_lo, t.c_h);
    hipLaunchKernelGGL(k_dct_dense_tables<1>, dim3(grid), dim3(256), 0, st, dq, s0, n, (int)np, t.ct64,
                       t.ct32, t.ct_hi, t.ct_lo, t.ct_h);
    if (eo)
      hipLaunchKernelGGL(k_dct_eo_tables, dim3(grid), dim3(256), 0, st, dq, s0, n, t.eo_hi, t.eo_lo,
                         t.eo_h, t.eot_hi, t.eot_lo, t.eot_h);
    // complete before any other stream may use them, and before dq goes
    ok = hipStreamSynchronize(st) == hipSuccess;
  }
  if (dq) (void)hipFree(dq);
  if (!ok) {
    free_tables(t);
    *status = set_error(ctx, LPU_ERR_OOM, "DCT table allocation failed");
    return nullptr;
  }
  ctx->dct.push_back(t);
  *status = LPU_OK;
  return &ctx->dct.back();
}

void free_dct_tables(lp_unwrap_ctx* ctx) {
  for (auto& t : ctx->dct) free_tables(t);
  ctx->dct.clear();
  for (auto& p : ctx->dct_dev) (void)hipFree(p.second);
  ctx->dct_dev.clear();
}

}  // namespace lpu
