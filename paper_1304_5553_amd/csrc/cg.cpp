// Conjugate gradients on the five-point model problem: fused kernels and the
// native iteration loop (the paper lists a conjugate-gradient Krylov solver
// among the facilities shipped beside its kernels; section "Further
// Facilities").
//
// One iteration of the textbook method is
//   q = A p;  c1 = p . q;  alpha = c0 / c1;  r -= alpha q;  d0 = r . r;
//   x += alpha p;  p = r + (d0 / c0) p
// and takes two launches inside a run of iterations:
//   cgr  folds the partials of p . A p, updates r and sums r . r;
//   cgu  folds those, updates x and p, and sums p . A p of the new p.
// A p is recomputed from p where it is needed instead of being stored (p comes
// out of the caches), every kernel folds the previous one's block partials in
// its own prologue (no fold launches), and p alternates between two buffers,
// so that a tile can read its neighbours' old p while they write the new one.
// The first iteration's p . A p comes from cgp; the last one is finished by
// cgf, which needs no neighbours and so writes the caller's p.  Per unknown
// and iteration: 12 bytes for cgr (r, p read, r written), 20 for cgu (x, p, r
// read, x, p written).
//
// Bound: the chain of dependent launches for grids inside the caches (a kernel
// of 256^2 unknowns takes 4.4 us: partials, tile and their folds are dependent
// trips to memory), HBM above.  Six launches per iteration from four generated
// kernels, 52 bytes per unknown, took 37 us per iteration at 1024 x 768 (issued
// from Python; 21 us of GPU time) and 135 at 4096^2; now 12.4 and 98.5.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstring>

#include "internal.h"

using namespace hipmr;

namespace {

// Tiles are TX columns by TY rows (the shapes below).  Sums are kept in FP64, in
// an order fixed by the grid size alone, and the same in cgp and cgu.  The vectors
// and the scalars between kernels are float; what is computed from them in one
// kernel (A p, alpha, the updates) is rounded once, when it is stored.
const char* kCgCommon = R"HIP(
// sum over the block's 256 threads, in every thread
__device__ __forceinline__ double cg_block_sum(double v) {
  __shared__ double cg_lds[4];
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) cg_lds[threadIdx.x >> 6] = v;
  __syncthreads();
  return (cg_lds[0] + cg_lds[1]) + (cg_lds[2] + cg_lds[3]);
}
// the fold of at most 2048 block partials, in every thread; loaded first, so
// that the first tile's loads are in flight together with the partials'
struct cg_partials { double v[8]; };
__device__ __forceinline__ cg_partials cg_fold_load(const double* __restrict__ part, int g) {
  cg_partials s;
#pragma unroll
  for (int k = 0; k < 8; ++k) s.v[k] = (int)threadIdx.x + 256 * k < g ? part[threadIdx.x + 256 * k] : 0.0;
  return s;
}
__device__ __forceinline__ double cg_fold_sum(const cg_partials& s) {
  return cg_block_sum(((s.v[0] + s.v[1]) + (s.v[2] + s.v[3])) + ((s.v[4] + s.v[5]) + (s.v[6] + s.v[7])));
}
__device__ __forceinline__ double cg_fold(const double* __restrict__ part, int g) {
  return cg_fold_sum(cg_fold_load(part, g));
}

// Workgroups go round-robin to the 8 XCDs: renumbered so that each takes a
// contiguous run of tiles, whose shared rows then lie in its own L2.
__device__ __forceinline__ int cg_block() {
  const int x = blockIdx.x & 7, q = gridDim.x >> 3, r = gridDim.x & 7;
  return x * q + (x < r ? x : r) + (blockIdx.x >> 3);
}

)HIP";

// The kernels below that work on tiles are in a namespace per tile shape.  A
// thread has one column and, of a step of RPS rows over the tile, one row.
const char* kCgTile = R"HIP(
typedef @@IDX@@ cg_idx;                          // of rows and columns
constexpr int TX = @@TX@@, TY = @@TY@@, RPS = 256 / TX, ROWS = TY / RPS;

// rows [r0 - 1, r0 + TY + 1), columns [c0 - 1, c0 + TX + 1) of an nx by ny
// grid into dst (row length TX + 2), zero outside the grid
__device__ __forceinline__ void cg_load_tile(float* dst, const float* src, cg_idx nx, cg_idx ny, cg_idx r0, cg_idx c0) {
  constexpr int W = TX + 2, R = TY + 2;
  const int lane = threadIdx.x % TX, w = threadIdx.x / TX;
#pragma unroll
  for (int k = 0; k < (R + RPS - 1) / RPS; ++k) {
    const int j = w + RPS * k;
    const cg_idx gr = r0 - 1 + j, gc = c0 + lane;
    if (j < R) dst[j * W + 1 + lane] = gr >= 0 && gr < ny && gc < nx ? src[(long long)gr * nx + gc] : 0.0f;
  }
#pragma unroll
  for (int i = 0; i < (2 * R + 255) / 256; ++i) {
    const int j = (threadIdx.x >> 1) + 128 * i, k = threadIdx.x & 1 ? TX + 1 : 0;
    const cg_idx gr = r0 - 1 + j, gc = c0 - 1 + k;
    if (j < R) dst[j * W + k] = gr >= 0 && gr < ny && gc >= 0 && gc < nx ? src[(long long)gr * nx + gc] : 0.0f;
  }
}

// (A p) at position k of a tile with row length W: zero boundary values
template <int W>
__device__ __forceinline__ double cg_apply(const float* p, int k) {
  return 4.0 * (double)p[k] - ((double)p[k - 1] + (double)p[k + 1]) - ((double)p[k - W] + (double)p[k + W]);
}
)HIP";

// first p . A p of a run; after cgs also the fold of b . b
const char* kCgP = R"HIP(
extern "C" __global__ void __launch_bounds__(256)
@@KNAME@@(const float* __restrict__ p, cg_idx nx, cg_idx ny, int tx, int tiles, double* __restrict__ pq_part,
          const double* __restrict__ rr_part, int rr_g, float* __restrict__ c)
{
  constexpr int W = TX + 2;
  __shared__ float sp[(TY + 2) * W];
  const int lane = threadIdx.x % TX, w = threadIdx.x / TX, b = cg_block();
  double acc = 0.0;
  for (int t = b; t < tiles; t += gridDim.x) {
    const cg_idx r0 = (cg_idx)(t / tx) * TY, c0 = (cg_idx)(t % tx) * TX;
    __syncthreads();
    cg_load_tile(sp, p, nx, ny, r0, c0);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      const int at = (w * ROWS + k + 1) * W + lane + 1;
      if (r0 + w * ROWS + k < ny && c0 + lane < nx) acc += (double)sp[at] * cg_apply<W>(sp, at);
    }
  }
  acc = cg_block_sum(acc);
  if (threadIdx.x == 0) pq_part[b] = acc;
  if (rr_g && b == 0) {
    const double rr = cg_fold(rr_part, rr_g);
    if (threadIdx.x == 0) c[0] = (float)rr;
  }
}
)HIP";

// r -= alpha A p, r . r; stores q = A p too if asked to
const char* kCgR = R"HIP(
extern "C" __global__ void __launch_bounds__(256)
@@KNAME@@(const float* __restrict__ p, float* __restrict__ r, float* __restrict__ q, cg_idx nx, cg_idx ny, int tx,
          int tiles, const double* __restrict__ pq_part, int pq_g, double* __restrict__ rr_part, float* c)
{
  constexpr int W = TX + 2;
  __shared__ float sp[(TY + 2) * W];
  const int lane = threadIdx.x % TX, w = threadIdx.x / TX, b = cg_block();
  const cg_partials parts = cg_fold_load(pq_part, pq_g);
  const float c0v = c[0];
  float rv[ROWS];
  auto load = [&](int t) {
    const cg_idx r0 = (cg_idx)(t / tx) * TY, c0 = (cg_idx)(t % tx) * TX;
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      const cg_idx gr = r0 + w * ROWS + k, gc = c0 + lane;
      rv[k] = gr < ny && gc < nx ? r[(long long)gr * nx + gc] : 0.0f;
    }
    cg_load_tile(sp, p, nx, ny, r0, c0);
  };
  if (b < tiles) load(b);
  const float pq = (float)cg_fold_sum(parts);
  const double alpha = (double)c0v / (double)pq;
  if (b == 0 && threadIdx.x == 0) c[1] = pq;
  double acc = 0.0;
  for (int t = b; t < tiles; t += gridDim.x) {
    const cg_idx r0 = (cg_idx)(t / tx) * TY, c0 = (cg_idx)(t % tx) * TX;
    if (t != b) {
      __syncthreads();
      load(t);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      const cg_idx gr = r0 + w * ROWS + k, gc = c0 + lane;
      if (gr < ny && gc < nx) {
        const double qv = cg_apply<W>(sp, (w * ROWS + k + 1) * W + lane + 1);
        const float rn = (float)__builtin_fma(-alpha, qv, (double)rv[k]);
        acc += (double)rn * (double)rn;
        r[(long long)gr * nx + gc] = rn;
        if (q) q[(long long)gr * nx + gc] = (float)qv;
      }
    }
  }
  acc = cg_block_sum(acc);
  if (threadIdx.x == 0) rr_part[b] = acc;
}
)HIP";

// x += alpha p, p_out = r + beta p, and p_out . A p_out
const char* kCgU = R"HIP(
extern "C" __global__ void __launch_bounds__(256)
@@KNAME@@(const float* __restrict__ p, const float* __restrict__ r, float* __restrict__ x,
          float* __restrict__ p_out, cg_idx nx, cg_idx ny, int tx, int tiles, const double* __restrict__ rr_part,
          int rr_g, double* __restrict__ pq_part, const float* __restrict__ c, float* __restrict__ d)
{
  constexpr int W = TX + 2, R = TY + 2, K = (R + RPS - 1) / RPS, S = (2 * R + 255) / 256;
  __shared__ float sn[R * W];
  const int lane = threadIdx.x % TX, w = threadIdx.x / TX, b = cg_block();
  const cg_partials parts = cg_fold_load(rr_part, rr_g);
  const double c0v = c[0], c1v = c[1];
  // rows w, w + RPS, ... of the tile and the ring around it (zero outside the
  // grid); the ring's side columns two rows' worth per pair of threads and step
  float pv[K], rv[K], xv[K], ps[S], rs[S];
  const int sj = threadIdx.x >> 1, sk = threadIdx.x & 1 ? TX + 1 : 0;
  auto load = [&](int t) {
    const cg_idx r0 = (cg_idx)(t / tx) * TY, c0 = (cg_idx)(t % tx) * TX, gc = c0 + lane;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int j = w + RPS * k;
      const cg_idx gr = r0 - 1 + j;
      const bool in = j < R && gr >= 0 && gr < ny && gc < nx;
      const long long at = (long long)gr * nx + gc;
      pv[k] = in ? p[at] : 0.0f;
      rv[k] = in ? r[at] : 0.0f;
      xv[k] = in && j >= 1 && j <= TY ? x[at] : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < S; ++k) {
      const int j = sj + 128 * k;
      const cg_idx gr = r0 - 1 + j, gs = c0 - 1 + sk;
      const bool in = j < R && gr >= 0 && gr < ny && gs >= 0 && gs < nx;
      ps[k] = in ? p[(long long)gr * nx + gs] : 0.0f;
      rs[k] = in ? r[(long long)gr * nx + gs] : 0.0f;
    }
  };
  if (b < tiles) load(b);
  const float rr = (float)cg_fold_sum(parts);
  const double alpha = c0v / c1v, beta = (double)rr / c0v;
  if (b == 0 && threadIdx.x == 0) d[0] = rr;
  double acc = 0.0;
  for (int t = b; t < tiles; t += gridDim.x) {
    const cg_idx r0 = (cg_idx)(t / tx) * TY, c0 = (cg_idx)(t % tx) * TX, gc = c0 + lane;
    if (t != b) load(t);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int j = w + RPS * k;
      const cg_idx gr = r0 - 1 + j;
      if (j < R) {
        const float pn = (float)__builtin_fma(beta, (double)pv[k], (double)rv[k]);
        sn[j * W + lane + 1] = pn;
        if (j >= 1 && j <= TY && gr < ny && gc < nx) {
          const long long at = (long long)gr * nx + gc;
          p_out[at] = pn;
          x[at] = (float)__builtin_fma(alpha, (double)pv[k], (double)xv[k]);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < S; ++k)
      if (sj + 128 * k < R) sn[(sj + 128 * k) * W + sk] = (float)__builtin_fma(beta, (double)ps[k], (double)rs[k]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      const int at = (w * ROWS + k + 1) * W + lane + 1;
      if (r0 + w * ROWS + k < ny && gc < nx) acc += (double)sn[at] * cg_apply<W>(sn, at);
    }
  }
  acc = cg_block_sum(acc);
  if (threadIdx.x == 0) pq_part[b] = acc;
}
)HIP";

// the same update at the end of a run: no neighbours, p_out may be p
const char* kCgF = R"HIP(
extern "C" __global__ void __launch_bounds__(256)
@@KNAME@@(const float* p, const float* __restrict__ r, float* __restrict__ x, float* p_out, long long n,
          const double* __restrict__ rr_part, int rr_g, const float* __restrict__ c, float* __restrict__ d)
{
  const float rr = (float)cg_fold(rr_part, rr_g);
  const double alpha = (double)c[0] / (double)c[1], beta = (double)rr / (double)c[0];
  if (blockIdx.x == 0 && threadIdx.x == 0) d[0] = rr;
  for (long long i0 = (long long)blockIdx.x * 1024 + threadIdx.x; i0 < n; i0 += (long long)gridDim.x * 1024) {
    float pv[4], rv[4], xv[4];                       // every load before any store
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const long long i = i0 + 256 * k;
      if (i < n) { pv[k] = p[i]; rv[k] = r[i]; xv[k] = x[i]; }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const long long i = i0 + 256 * k;
      if (i < n) {
        x[i] = (float)__builtin_fma(alpha, (double)pv[k], (double)xv[k]);
        p_out[i] = (float)__builtin_fma(beta, (double)pv[k], (double)rv[k]);
      }
    }
  }
}
)HIP";

// x = 0, r = p = b, b . b
const char* kCgS = R"HIP(
extern "C" __global__ void __launch_bounds__(256)
@@KNAME@@(const float* b, float* x, float* r, float* p, long long n, double* __restrict__ rr_part)
{
  double acc = 0.0;
  for (long long i0 = (long long)blockIdx.x * 1024 + threadIdx.x; i0 < n; i0 += (long long)gridDim.x * 1024) {
    float v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = i0 + 256 * k < n ? b[i0 + 256 * k] : 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const long long i = i0 + 256 * k;
      if (i < n) {
        x[i] = 0.0f;
        r[i] = v[k];
        p[i] = v[k];
        acc += (double)v[k] * (double)v[k];
      }
    }
  }
  acc = cg_block_sum(acc);
  if (threadIdx.x == 0) rr_part[blockIdx.x] = acc;
}
)HIP";

// r . r of a start that no iteration follows
const char* kCgZ = R"HIP(
extern "C" __global__ void __launch_bounds__(256)
@@KNAME@@(const double* __restrict__ rr_part, int rr_g, float* __restrict__ c)
{
  const double rr = cg_fold(rr_part, rr_g);
  if (threadIdx.x == 0) c[0] = (float)rr;
}
)HIP";

enum { kP, kR, kU, kF, kS, kZ, kCgKernels };         // the first three work on tiles
const char* const kCgBodies[kCgKernels] = {kCgP, kCgR, kCgU, kCgF, kCgS, kCgZ};
const char* const kCgTags[kCgKernels] = {"cgp", "cgr", "cgu", "cgf", "cgs", "cgz"};
// (256 x 4 would suit flat grids better than 128 x 8, but crashes the compiler
// that comes with PyTorch's ROCm 7.0 libraries.)
struct CgShape {
    int tx, ty;
};
constexpr CgShape kCgShape[] = {{64, 8}, {64, 16}, {128, 8}, {16, 64}, {4, 256}, {1, 1024}};
constexpr int kCgShapes = sizeof(kCgShape) / sizeof(kCgShape[0]);
// Blocks of a kernel, and so the partials its successor folds in every block:
// eight per compute unit (at 4096^2, 98.5 us per iteration; 103 with 1536
// blocks, 114 with 1024, 126 with 768).
constexpr int kCgBlocks = 2048;
constexpr size_t kCgPartBytes = kCgBlocks * sizeof(double);
constexpr int64_t kCgMostUnknowns = (int64_t)1 << 48;

void replace_key(std::string& s, const std::string& key, const std::string& val) {
    for (size_t at; (at = s.find(key)) != std::string::npos;) s.replace(at, key.size(), val);
}

// The kernels of every grid size, built as one program and loaded together, so
// that a capture of any size finds them once a run of any size went before.
struct CgKernels {
    std::shared_ptr<CodeObject> of[kCgShapes][kCgKernels];
};
// (`wide`: grids with a side that 32-bit row and column numbers do not reach, a
// program of their own.)
hipmr_status cg_kernels(bool wide, const CgKernels** out) {
    static std::mutex mu;
    static CgKernels both[2];
    CgKernels& built = both[wide];
    std::lock_guard<std::mutex> lk(mu);
    if (!built.of[0][0]) {
        std::string text = kCgCommon;
        std::vector<std::string> symbols;
        const auto add = [&](std::string body, int which, const std::string& shape) {
            symbols.push_back(std::string("hipmr_") + kCgTags[which] + shape + "_" +
                              sha256_hex(body.data(), body.size()).substr(0, 8));
            replace_key(body, "@@KNAME@@", symbols.back());
            text += body;
        };
        for (const CgShape& sh : kCgShape) {
            const std::string name = "_" + std::to_string(sh.tx) + "x" + std::to_string(sh.ty) + (wide ? "w" : "");
            std::string tile = kCgTile;
            replace_key(tile, "@@TX@@", std::to_string(sh.tx));
            replace_key(tile, "@@TY@@", std::to_string(sh.ty));
            replace_key(tile, "@@IDX@@", wide ? "long long" : "int");
            text += "namespace cg" + name + " {\n" + tile;
            for (int k : {kP, kR, kU}) add(kCgBodies[k], k, name);
            text += "}\n";
        }
        for (int k : {kF, kS, kZ}) add(kCgBodies[k], k, "");
        hipmr_status st;
        const auto all = get_or_build(text, symbols, &st);
        if (all.empty()) return st;
        for (int s = kCgShapes - 1; s >= 0; --s)
            for (int k = kCgKernels - 1; k >= 0; --k)
                built.of[s][k] = k < 3 ? all[s * 3 + k] : all[kCgShapes * 3 + k - 3];
    }
    *out = &built;
    return HIPMR_OK;
}

long long cg_tiles(const CgShape& s, long long nx, long long ny) {
    return ((nx + s.tx - 1) / s.tx) * ((ny + s.ty - 1) / s.ty);
}

// Tiles of 64 x 8 while there are at most 1024 of them (more blocks for the
// latency of a small grid), else of 64 x 16 (a smaller ring, fewer partials).  Us
// per iteration with 8 / 16 rows: 256^2 8.6 / 9.4, 333 x 777 10.4 / 11.2,
// 1024 x 768 13.9 / 12.4, 2048^2 33.6 / 30.4, 4096^2 109 / 98.5.  Other shapes
// only where 64 x 16 would work for columns or rows that a narrow grid does not
// have: a third more elements, ring included, than the best shape.
int cg_shape(long long nx, long long ny) {
    if (cg_tiles(kCgShape[0], nx, ny) <= 1024) return 0;
    const auto work = [&](int k) { return cg_tiles(kCgShape[k], nx, ny) * ((kCgShape[k].tx + 2) * (kCgShape[k].ty + 2)); };
    int best = 1;
    for (int k = 2; k < kCgShapes; ++k)
        if (work(k) < work(best)) best = k;
    return work(best) * 4 < work(1) * 3 ? best : 1;
}

}  // namespace

namespace hipmr {

hipmr_status cg_selftest(int32_t* built) {
    for (bool wide : {false, true}) {
        const CgKernels* all;
        hipmr_status st = cg_kernels(wide, &all);
        if (st != HIPMR_OK) return st;
        *built += kCgShapes * 3 + 3;
    }
    return HIPMR_OK;
}

}  // namespace hipmr

extern "C" {

size_t hipmr_poisson_cg_workspace_bytes(int64_t nx, int64_t ny) {
    int64_t n;
    if (nx < 0 || ny < 0 || __builtin_mul_overflow(nx, ny, &n) || n > kCgMostUnknowns) return 0;
    return 2 * kCgPartBytes + (size_t)n * 4;
}

hipmr_status hipmr_poisson_cg(int64_t nx, int64_t ny, const void* b, int32_t iters, void* x, void* r,
                              void* p, void* q, void* s, int32_t parity, void* workspace,
                              size_t workspace_bytes, void* stream) {
    clear_error();
    int64_t n;
    if (nx < 0 || ny < 0 || __builtin_mul_overflow(nx, ny, &n) || n > kCgMostUnknowns)
        return fail(HIPMR_E_INVALID, "a grid side is negative, or the grid beyond any memory");
    if (nx == 0 || ny == 0) return HIPMR_OK;
    if (iters < 0 || (parity != 0 && parity != 1)) return fail(HIPMR_E_INVALID, "iters < 0 or parity not 0 / 1");
    if (!x || !r || !p || !q || !s) return fail(HIPMR_E_INVALID, "NULL array");
    if (!workspace || workspace_bytes < hipmr_poisson_cg_workspace_bytes(nx, ny))
        return fail(HIPMR_E_WORKSPACE, "workspace smaller than hipmr_poisson_cg_workspace_bytes()");
    if ((uintptr_t)workspace % 8) return fail(HIPMR_E_WORKSPACE, "workspace off its 8-byte alignment");
    for (const void* a : {b, (const void*)x, (const void*)r, (const void*)p, (const void*)q, (const void*)s})
        if ((uintptr_t)a % 4) return fail(HIPMR_E_INVALID, "array off its element alignment");
    if (ny == 1) std::swap(nx, ny);                  // the same unknowns and operator, one above the other
    const int shape = cg_shape(nx, ny);
    const long long tiles64 = cg_tiles(kCgShape[shape], nx, ny);
    if (tiles64 > INT32_MAX) return fail(HIPMR_E_UNSUPPORTED, "grid too large");
    const bool wide = std::max(nx, ny) > INT32_MAX / 2;
    const CgKernels* all;
    hipmr_status st = cg_kernels(wide, &all);
    if (st != HIPMR_OK) return st;
    static std::atomic<uint64_t> loaded_on[2];         // devices on which every shape's kernels are
    std::atomic<uint64_t>& loaded = loaded_on[wide];
    int dev = 0;
    void* fn[kCgKernels];
    if (hipGetDevice(&dev) == hipSuccess && dev < 64 && !(loaded.load() >> dev & 1) && !capturing_now()) {
        for (const auto& kernels : all->of)
            for (const auto& co : kernels)
                if ((st = get_function(*co, &fn[0])) != HIPMR_OK) return st;
        loaded.fetch_or(1ull << dev);
    }
    for (int k = 0; k < kCgKernels; ++k)
        if ((st = get_function(*all->of[shape][k], &fn[k])) != HIPMR_OK) return st;

    double* pq_part = (double*)workspace;
    double* rr_part = pq_part + kCgBlocks;
    float* spare = (float*)((char*)workspace + 2 * kCgPartBytes);     // the other buffer of p
    int nx32 = (int)nx, ny32 = (int)ny;
    void *inx = wide ? (void*)&nx : &nx32, *iny = wide ? (void*)&ny : &ny32;
    int tx = (int)((nx + kCgShape[shape].tx - 1) / kCgShape[shape].tx);
    int tiles = (int)tiles64;
    int g = std::min(tiles, kCgBlocks);
    int gf = (int)std::min<long long>((n + 1023) / 1024, kCgBlocks);   // four unknowns per thread and pass
    float* c = (float*)s + 2 * parity;
    float* d = (float*)s + 2 * (1 - parity);
    long long n_arg = n;
    if (b) {
        void* a[] = {&b, &x, &r, &p, &n_arg, &rr_part};
        st = launch(fn[kS], (unsigned)gf, 256, a, stream);
        if (st == HIPMR_OK && iters == 0) {
            void* z[] = {&rr_part, &gf, &c};
            st = launch(fn[kZ], 1, 256, z, stream);
        }
    }
    if (iters == 0 || st != HIPMR_OK) return st;
    float* pc = (float*)p;                           // the current p
    int rr_g = b ? gf : 0;
    {
        void* a[] = {&pc, inx, iny, &tx, &tiles, &pq_part, &rr_part, &rr_g, &c};
        st = launch(fn[kP], (unsigned)g, 256, a, stream);
    }
    for (int it = 0; it < iters && st == HIPMR_OK; ++it) {
        const bool last = it == iters - 1;
        float* qa = last ? (float*)q : nullptr;
        void* a[] = {&pc, &r, &qa, inx, iny, &tx, &tiles, &pq_part, &g, &rr_part, &c};
        st = launch(fn[kR], (unsigned)g, 256, a, stream);
        if (st != HIPMR_OK) break;
        if (last) {
            void* f[] = {&pc, &r, &x, &p, &n_arg, &rr_part, &g, &c, &d};
            st = launch(fn[kF], (unsigned)gf, 256, f, stream);
        } else {
            float* pn = pc == p ? spare : (float*)p;
            void* u[] = {&pc, &r, &x, &pn, inx, iny, &tx, &tiles, &rr_part, &g, &pq_part, &c, &d};
            st = launch(fn[kU], (unsigned)g, 256, u, stream);
            pc = pn;
        }
        std::swap(c, d);
    }
    return st;
}

}  // extern "C"
