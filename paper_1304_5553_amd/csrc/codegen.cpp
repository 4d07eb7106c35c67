// Code generation: HIP device templates for gfx950 and their rendering.
//
// The paper generates device code at run time by textual keyword replacement,
// optionally combined with preprocessor macros, and by templating when
// control flow is needed (section "Generating Code"); run-time specialisation
// bakes constants, types and trip counts into the source (section "The Cost
// of Flexibility"), and the user's expression lands inside the inner loop
// with no function-pointer indirection (section "High-Performance
// Abstractions").  Here the templates below carry @@KEY@@ markers that are
// replaced by the signature's types, the user's statement / map / reduce /
// neutral text and the launch constants (block size, vector chunks per
// thread, elements per chunk, index width).
//
// Kernel families (all wave64; LDS for the trees across a block's waves, a
// scan's hand-over and a segmented call's tile table):
//   ew, ews     grid-stride over VEC-element chunks, each thread with IPT chunks
//               of every accessed array in flight (16-byte loads and stores),
//               the statement run per element from registers; or one element
//               per step (any access pattern);
//   rs1, rs1s   the same loads; per-thread accumulators (one per in-flight
//               chunk) folded pairwise, a wave64 butterfly (cross-lane
//               shuffles) and an LDS tree across the block's waves: one partial
//               per block.  The last block folds the others' partials in the
//               same launch, exchanged as tagged 64-bit words (device-scope
//               atomic loads and stores; no read-modify-write), or
//   rs2         one block folds them in a launch of its own: the same bits;
//   csum, nrm1, nrm2 (csums, ...), csumf, nrm2f
//               the same for compensated sums and norms;
//   seg1, seg2, segplan
//               tiles of segments by a persistent kernel, their fold, the
//               table where it does not fit LDS;
//   sc1, scu + scd, scz + scl
//               prefix scans: one tile, totals and rescan, one pass (tiles
//               take tickets, publish totals and wait for earlier ones').
#include <algorithm>

#include "common.h"
#include "internal.h"

namespace hipmr {
namespace {

const char* kPrelude = R"HIP(
// ---- hipmr device prelude (gfx950) ----
#ifndef INFINITY
#define INFINITY __builtin_huge_valf()
#endif
#ifndef NAN
#define NAN __builtin_nanf("")
#endif
#ifndef HUGE_VALF
#define HUGE_VALF __builtin_huge_valf()
#endif
#ifndef HUGE_VAL
#define HUGE_VAL __builtin_huge_val()
#endif
#ifndef FLT_MAX
#define FLT_MAX 3.40282347e+38F
#endif
#ifndef FLT_MIN
#define FLT_MIN 1.17549435e-38F
#endif
#ifndef DBL_MAX
#define DBL_MAX 1.7976931348623157e+308
#endif
#ifndef INT_MAX
#define INT_MAX 2147483647
#endif
#ifndef INT_MIN
#define INT_MIN (-2147483647 - 1)
#endif
#ifndef UINT_MAX
#define UINT_MAX 4294967295U
#endif
#ifndef LLONG_MAX
#define LLONG_MAX 9223372036854775807LL
#endif
#ifndef LLONG_MIN
#define LLONG_MIN (-9223372036854775807LL - 1LL)
#endif

typedef unsigned int hipmr_u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int hipmr_u32x2 __attribute__((ext_vector_type(2)));

// Storage-only number formats: a read converts exactly to float, arithmetic
// happens in float, a store rounds to nearest even.
struct hipmr_bf16 {
  unsigned short bits;
  __device__ __forceinline__ operator float() const {
    return __uint_as_float((unsigned int)bits << 16);
  }
  __device__ __forceinline__ hipmr_bf16& operator=(float f) {
    unsigned int u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) {
      bits = (unsigned short)((u >> 16) | 0x40u);          // quiet NaN
    } else {
      u += 0x7fffu + ((u >> 16) & 1u);                      // round to nearest even
      bits = (unsigned short)(u >> 16);
    }
    return *this;
  }
  __device__ __forceinline__ hipmr_bf16& operator+=(float f) { return *this = (float)*this + f; }
  __device__ __forceinline__ hipmr_bf16& operator-=(float f) { return *this = (float)*this - f; }
  __device__ __forceinline__ hipmr_bf16& operator*=(float f) { return *this = (float)*this * f; }
  __device__ __forceinline__ hipmr_bf16& operator/=(float f) { return *this = (float)*this / f; }
};

struct hipmr_f16 {
  _Float16 h;
  __device__ __forceinline__ operator float() const { return (float)h; }
  __device__ __forceinline__ hipmr_f16& operator=(float f) { h = (_Float16)f; return *this; }
  __device__ __forceinline__ hipmr_f16& operator+=(float f) { return *this = (float)*this + f; }
  __device__ __forceinline__ hipmr_f16& operator-=(float f) { return *this = (float)*this - f; }
  __device__ __forceinline__ hipmr_f16& operator*=(float f) { return *this = (float)*this * f; }
  __device__ __forceinline__ hipmr_f16& operator/=(float f) { return *this = (float)*this / f; }
};

// OCP FP8 E4M3 ("fn"): gfx950's conversion instructions use the OCP encoding.
struct hipmr_fp8 {
  unsigned char bits;
  __device__ __forceinline__ operator float() const {
    return __builtin_amdgcn_cvt_f32_fp8((int)bits, 0);
  }
  __device__ __forceinline__ hipmr_fp8& operator=(float f) {
    const float c = (f != f) ? f : __builtin_fminf(__builtin_fmaxf(f, -448.0f), 448.0f);
    bits = (unsigned char)(__builtin_amdgcn_cvt_pk_fp8_f32(c, c, 0, false) & 0xff);
    return *this;
  }
  __device__ __forceinline__ hipmr_fp8& operator+=(float f) { return *this = (float)*this + f; }
  __device__ __forceinline__ hipmr_fp8& operator-=(float f) { return *this = (float)*this - f; }
  __device__ __forceinline__ hipmr_fp8& operator*=(float f) { return *this = (float)*this * f; }
  __device__ __forceinline__ hipmr_fp8& operator/=(float f) { return *this = (float)*this / f; }
};

// Complex values with float components (real, imaginary).
struct hipmr_c64 {
  float re, im;
  hipmr_c64() = default;
  __device__ __forceinline__ constexpr hipmr_c64(float r, float i) : re(r), im(i) {}
  __device__ __forceinline__ constexpr hipmr_c64(float r) : re(r), im(0.0f) {}
  __device__ __forceinline__ constexpr hipmr_c64(double r) : re((float)r), im(0.0f) {}
  __device__ __forceinline__ constexpr hipmr_c64(int r) : re((float)r), im(0.0f) {}
  __device__ __forceinline__ constexpr hipmr_c64(unsigned int r) : re((float)r), im(0.0f) {}
  __device__ __forceinline__ constexpr hipmr_c64(long long r) : re((float)r), im(0.0f) {}
  __device__ __forceinline__ hipmr_c64& operator+=(hipmr_c64 b) { re += b.re; im += b.im; return *this; }
  __device__ __forceinline__ hipmr_c64& operator-=(hipmr_c64 b) { re -= b.re; im -= b.im; return *this; }
  __device__ __forceinline__ hipmr_c64& operator*=(hipmr_c64 b) {
    const float r = re * b.re - im * b.im;
    im = re * b.im + im * b.re;
    re = r;
    return *this;
  }
};
__device__ __forceinline__ hipmr_c64 operator+(hipmr_c64 a, hipmr_c64 b) { return hipmr_c64(a.re + b.re, a.im + b.im); }
__device__ __forceinline__ hipmr_c64 operator-(hipmr_c64 a, hipmr_c64 b) { return hipmr_c64(a.re - b.re, a.im - b.im); }
__device__ __forceinline__ hipmr_c64 operator-(hipmr_c64 a) { return hipmr_c64(-a.re, -a.im); }
__device__ __forceinline__ hipmr_c64 operator+(hipmr_c64 a) { return a; }
__device__ __forceinline__ hipmr_c64 operator*(hipmr_c64 a, hipmr_c64 b) {
  return hipmr_c64(a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re);
}
__device__ __forceinline__ hipmr_c64 conj(hipmr_c64 z) { return hipmr_c64(z.re, -z.im); }
__device__ __forceinline__ float real(hipmr_c64 z) { return z.re; }
__device__ __forceinline__ float imag(hipmr_c64 z) { return z.im; }
__device__ __forceinline__ float abs(hipmr_c64 z) { return __builtin_sqrtf(z.re * z.re + z.im * z.im); }
__device__ __forceinline__ hipmr_c64 __shfl_xor(hipmr_c64 v, int m, int w) {
  return hipmr_c64(__shfl_xor(v.re, m, w), __shfl_xor(v.im, m, w));
}
__device__ __forceinline__ hipmr_c64 __shfl_up(hipmr_c64 v, unsigned int d, int w) {
  return hipmr_c64(__shfl_up(v.re, d, w), __shfl_up(v.im, d, w));
}
__device__ __forceinline__ hipmr_c64 __shfl(hipmr_c64 v, int l, int w) {
  return hipmr_c64(__shfl(v.re, l, w), __shfl(v.im, l, w));
}

// A vector chunk of N elements held in registers.
template <typename T, int N> struct hipmr_pack { T v[N]; };

template <int B> struct hipmr_word;
template <> struct hipmr_word<1> { typedef unsigned char t; };
template <> struct hipmr_word<2> { typedef unsigned short t; };
template <> struct hipmr_word<4> { typedef unsigned int t; };
template <> struct hipmr_word<8> { typedef hipmr_u32x2 t; };
template <> struct hipmr_word<16> { typedef hipmr_u32x4 t; };

// Loads / stores one chunk with the widest (<= 16-byte) accesses its size
// allows; NT selects streaming (non-temporal) accesses.
template <bool NT, typename T, int N>
__device__ __forceinline__ void hipmr_load(hipmr_pack<T, N>& p, const T* src) {
  constexpr int B = (int)sizeof(T) * N;
  constexpr int W = B >= 16 ? 16 : B;
  typedef typename hipmr_word<W>::t word;
  word tmp[B / W];
  const word* s = reinterpret_cast<const word*>(src);
#pragma unroll
  for (int k = 0; k < B / W; ++k) {
    if constexpr (NT) tmp[k] = __builtin_nontemporal_load(s + k);
    else tmp[k] = s[k];
  }
  __builtin_memcpy(&p, tmp, B);
}

// A read-only chunk of N FP8 values kept as 32-bit words: elements 2k and
// 2k + 1 decode together with the packed conversion instruction (one
// instruction per pair; the pair's two reads share it), no byte extraction.
typedef float hipmr_f32x2 __attribute__((ext_vector_type(2)));
template <int N> struct hipmr_fp8_words {
  unsigned int w[N / 4];
  __device__ __forceinline__ float operator[](int j) const {
    const int word = (int)w[j >> 2];
    const hipmr_f32x2 pair = (j & 2) ? __builtin_amdgcn_cvt_pk_f32_fp8(word, true)
                                     : __builtin_amdgcn_cvt_pk_f32_fp8(word, false);
    return (j & 1) ? pair.y : pair.x;
  }
};
template <int N> struct hipmr_pack_fp8ro { hipmr_fp8_words<N> v; };

template <bool NT, int N>
__device__ __forceinline__ void hipmr_load(hipmr_pack_fp8ro<N>& p, const hipmr_fp8* src) {
  hipmr_pack<hipmr_fp8, N> raw;
  hipmr_load<NT>(raw, src);
  __builtin_memcpy(&p, &raw, N);
}

// A chunk wider than 16 bytes leaves in several store instructions, each
// covering every other 16 bytes of the lanes' lines: streaming stores would
// write those half lines out unmerged, so wide chunks are stored temporally
// (the L2 merges them).
template <bool NT, typename T, int N>
__device__ __forceinline__ void hipmr_store(T* dst, const hipmr_pack<T, N>& p) {
  constexpr int B = (int)sizeof(T) * N;
  constexpr int W = B >= 16 ? 16 : B;
  typedef typename hipmr_word<W>::t word;
  word tmp[B / W];
  __builtin_memcpy(tmp, &p, B);
  word* d = reinterpret_cast<word*>(dst);
#pragma unroll
  for (int k = 0; k < B / W; ++k) {
    if constexpr (NT && B <= 16) __builtin_nontemporal_store(tmp[k], d + k);
    else d[k] = tmp[k];
  }
}
)HIP";

// Reduction helpers; rendered after hipmr_acc and hipmr_combine are defined.
const char* kReduceHelpers = R"HIP(
// wave64 butterfly then an LDS tree over the block's waves; the result is
// valid in thread 0.  The order of combination is fixed by the block size.
template <int B>
__device__ __forceinline__ hipmr_acc hipmr_block_reduce(hipmr_acc v, hipmr_acc neutral) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v = hipmr_combine(v, __shfl_xor(v, m, 64));
  if constexpr (B > 64) {
    // W waves (any count up to 16): lanes >= W of wave 0 hold the neutral
    // element and the butterfly spans the next power of two >= W
    constexpr int W = B / 64;
    constexpr int P = W <= 2 ? 2 : W <= 4 ? 4 : W <= 8 ? 8 : 16;
    __shared__ hipmr_acc hipmr_lds[W];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    if (l == 0) hipmr_lds[w] = v;
    __syncthreads();
    if (w == 0) {
      v = l < W ? hipmr_lds[l] : neutral;
#pragma unroll
      for (int m = P / 2; m >= 1; m >>= 1) v = hipmr_combine(v, __shfl_xor(v, m, 64));
    }
  }
  return v;
}

// pairwise fold of a thread's U accumulators into a[0]
template <int U>
__device__ __forceinline__ hipmr_acc hipmr_fold(hipmr_acc* a) {
#pragma unroll
  for (int s = 1; s < U; s *= 2) {
#pragma unroll
    for (int u = 0; u + s < U; u += 2 * s) a[u] = hipmr_combine(a[u], a[u + s]);
  }
  return a[0];
}
)HIP";

// The end of a reduction in one launch: every block publishes its partial, and
// the last one (by index) waits for the others' and folds them in the order of
// the separate fold kernel (rs2), so both give the same bits.  A partial is
// published as words of 16 data bits and a 48-bit tag that no other launch of
// the process carries, so the caller's workspace needs no clearing: a word is
// taken only with this launch's tag (a launch that may be replayed, with the
// same tag, folds in a launch of its own).  Device-scope accesses, no counter:
// counting 512 blocks in through one address costs more than the second launch.
// The wait is bounded (2^20 polls, about a second).  It can run out while the
// others still queue behind another stream's kernel, or where another call has
// overwritten the words; the last block then computes every share itself, in
// the same order, so the result is the same.
// Against a separate fold launch: a dot of 2 x 2^20 floats 8.5 -> 5.5 us per
// call, of 2 x 3.1 M 8.6 -> 6.6, a sum of 18.9 M 14.0 -> 12.8, of 157 M 92.4 ->
// 91.2 (HBM bound).
const char* kTagged = R"HIP(
// publishes block k's value (hipmr_put_tagged), and waits for it (get: false
// if it did not come); bit 63 of the launch's tag word asks for no wait
template <typename T>
__device__ __forceinline__ void hipmr_put_tagged(unsigned long long* part, int k, T v, unsigned long long tag) {
  constexpr int W = (int)sizeof(T) / 2;
  unsigned long long bits = 0;
  __builtin_memcpy(&bits, &v, sizeof(v));
#pragma unroll
  for (int j = 0; j < W; ++j)
    __hip_atomic_store(part + (long long)k * W + j, ((bits >> (16 * j)) & 0xffffull) | tag << 16,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ bool hipmr_get_tagged(const unsigned long long* part, int k, unsigned long long tag, T* v) {
  constexpr int W = (int)sizeof(T) / 2;
  const unsigned limit = tag >> 63 ? 1u : 1u << 20;
  unsigned long long bits;
  for (unsigned polls = 1;; ++polls) {
    bool here = true;
    bits = 0;
#pragma unroll
    for (int j = 0; j < W; ++j) {
      const unsigned long long w = __hip_atomic_load(part + (long long)k * W + j, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
      here = here && (w >> 16) == (tag & 0xffffffffffffull);
      bits |= (w & 0xffffull) << (16 * j);
    }
    if (here) break;
    if (polls >= limit) return false;
    __builtin_amdgcn_s_sleep(1);
  }
  __builtin_memcpy(v, &bits, sizeof(T));
  return true;
}
// whether any thread of the block says so (a barrier)
template <int B>
__device__ __forceinline__ bool hipmr_any(bool says) {
  __shared__ int hipmr_says[B / 64];
  const bool some = __ballot(says) != 0;
  if ((threadIdx.x & 63) == 0) hipmr_says[threadIdx.x >> 6] = some;
  __syncthreads();
  int any = 0;
#pragma unroll
  for (int w = 0; w < B / 64; ++w) any |= hipmr_says[w];
  return any != 0;
}
)HIP";

// hipmr_finish returns whether the block has to compute every share: a loop over
// the shares then follows it in the kernel (the templates named ...Share below:
// the body's order of combination, but one chunk at a time), each added by
// hipmr_add_share.  (The body itself in a loop cost registers, and the compiler
// then issued a compensated bfloat16 dot's loads one by one, 55 us against 40
// at 2^26; a copy of it doubled them, 13.0 us against 11.1 for twelve arrays of
// 2^22.)
const char* kRedFinish = R"HIP(
template <int B>
__device__ __forceinline__ bool hipmr_finish(hipmr_acc r, hipmr_acc neutral, unsigned long long* part,
                                             hipmr_acc* __restrict__ out, unsigned long long tag) {
  const int g = (int)gridDim.x;
  if (threadIdx.x == 0) hipmr_put_tagged(part, (int)blockIdx.x, r, tag);
  if ((int)blockIdx.x != g - 1) return false;
  hipmr_acc v = neutral;
  bool here = true;
  for (int k = threadIdx.x; here && k < g; k += B) {
    hipmr_acc p;
    here = hipmr_get_tagged(part, k, tag, &p);
    if (here) v = hipmr_combine(v, p);
  }
  if (hipmr_any<B>(!here)) return true;          // a barrier: the share's fold has been read
  v = hipmr_block_reduce<B>(v, neutral);
  if (threadIdx.x == 0) *out = v;
  return false;
}
template <int B>
__device__ __forceinline__ void hipmr_add_share(hipmr_acc& v, hipmr_acc r, hipmr_acc neutral,
                                                hipmr_acc* __restrict__ out, int b) {
  __shared__ hipmr_acc hipmr_share;
  if (threadIdx.x == 0) hipmr_share = r;
  __syncthreads();
  if ((int)threadIdx.x == b % B) v = hipmr_combine(v, hipmr_share);
  __syncthreads();
  if (b + 1 < (int)gridDim.x) return;
  v = hipmr_block_reduce<B>(v, neutral);
  if (threadIdx.x == 0) *out = v;
}
)HIP";

const char* kEwVector = R"HIP(
extern "C" __global__ void __launch_bounds__(@@BLOCK@@)
@@KNAME@@(@@PARAMS@@, long long hipmr_n, long long hipmr_head)
{
  typedef @@IDX@@ hipmr_idx;
  constexpr int HIPMR_B = @@BLOCK@@, HIPMR_U = @@IPT@@, HIPMR_V = @@VEC@@;
  constexpr bool HIPMR_NTL = @@NTL@@, HIPMR_NTS = @@NTS@@;
  const hipmr_idx n = (hipmr_idx)hipmr_n;
  // elements [0, head) precede the first aligned chunk; [t0, n) is the ragged tail
  const long long hipmr_h = hipmr_head < hipmr_n ? hipmr_head : hipmr_n;
  const long long hipmr_nc = (hipmr_n - hipmr_h) / HIPMR_V;
  const long long hipmr_t0 = hipmr_h + hipmr_nc * HIPMR_V;
  if (blockIdx.x == 0) {
    if ((long long)threadIdx.x < hipmr_h) {
      const hipmr_idx i = (hipmr_idx)threadIdx.x;
      { @@STMT@@; }
    }
    if ((long long)threadIdx.x < hipmr_n - hipmr_t0) {
      const hipmr_idx i = (hipmr_idx)(hipmr_t0 + threadIdx.x);
      { @@STMT@@; }
    }
  }
  const long long hipmr_step = (long long)gridDim.x * (HIPMR_B * HIPMR_U);
  long long hipmr_c0 = (long long)blockIdx.x * (HIPMR_B * HIPMR_U) + threadIdx.x;
  for (; hipmr_c0 + (HIPMR_U - 1) * HIPMR_B < hipmr_nc; hipmr_c0 += hipmr_step) {
    @@DECL_PACKS@@
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_off = hipmr_h + (hipmr_c0 + hipmr_u * HIPMR_B) * HIPMR_V;
      @@LOADS@@
    }
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_off = hipmr_h + (hipmr_c0 + hipmr_u * HIPMR_B) * HIPMR_V;
#pragma unroll
      for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
        const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
        { @@VSTMT@@; }
      }
      @@STORES@@
    }
  }
  if (hipmr_c0 < hipmr_nc) {
    @@DECL_PACKS@@
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_c = hipmr_c0 + hipmr_u * HIPMR_B;
      if (hipmr_c < hipmr_nc) {
        const long long hipmr_off = hipmr_h + hipmr_c * HIPMR_V;
        @@LOADS@@
      }
    }
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_c = hipmr_c0 + hipmr_u * HIPMR_B;
      if (hipmr_c < hipmr_nc) {
        const long long hipmr_off = hipmr_h + hipmr_c * HIPMR_V;
#pragma unroll
        for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
          const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
          { @@VSTMT@@; }
        }
        @@STORES@@
      }
    }
  }
}
)HIP";

// The vector elementwise kernel for statements with shifted reads
// name[i + E]: per chunk, each distinct shifted read is one unaligned load of
// V elements from name + off + E.  A chunk whose shifted loads would leave
// [0, n) (within |E| of either end) runs the statement one element at a time
// instead, with the statement's own guards.
const char* kShiftHelpers = R"HIP(
// 16 bytes at 4-byte alignment: one dwordx4 load (the memory system accepts
// dword-aligned multi-dword accesses); narrower element types go by memcpy
typedef unsigned int hipmr_u32x4u __attribute__((ext_vector_type(4), aligned(4)));

template <typename T, int N>
__device__ __forceinline__ void hipmr_loadu(hipmr_pack<T, N>& p, const T* src) {
  if constexpr (sizeof(p) % 16 == 0 && alignof(T) >= 4) {
    hipmr_u32x4u w[sizeof(p) / 16];
#pragma unroll
    for (int k = 0; k < (int)(sizeof(p) / 16); ++k) w[k] = reinterpret_cast<const hipmr_u32x4u*>(src)[k];
    __builtin_memcpy(&p, w, sizeof(p));
  } else {
    __builtin_memcpy(&p, src, sizeof(p));
  }
}

// XCD-aware order: workgroups go round-robin to the 8 XCDs, each with its own
// L2.  Renumbered, each XCD takes a contiguous run of chunks, so the
// neighbouring elements a shifted read reaches were loaded by the same XCD.
// the window start off + s clamped into [0, hi] (hi = n - V >= 0, 0 <= off <= hi),
// without forming off + s when it would leave that range (s may be huge)
__device__ __forceinline__ long long hipmr_clampv(long long off, long long s, long long hi) {
  return s < -off ? 0 : (s > hi - off ? hi : off + s);
}

__device__ __forceinline__ unsigned hipmr_xcd_block(unsigned b) {
  const unsigned x = b % 8u, q = gridDim.x / 8u, r = gridDim.x % 8u;
  return x * q + (x < r ? x : r) + b / 8u;
}
)HIP";

// Chunk loads at element alignment, for arrays whose chunks do not start on
// the written arrays' (or the other inputs') 16-byte boundary, such as the two
// views x[1:] and x[:-1] of one signal.  One dwordx4 load all the same: the
// memory system takes any byte address, and neighbouring lanes share the lines
// their chunks straddle, so a shifted stream runs within 2-5 % of an aligned one.
const char* kUnalignedHelpers = R"HIP(
template <bool NT, typename T, int N>
__device__ __forceinline__ void hipmr_load_any(hipmr_pack<T, N>& p, const T* src) {
  constexpr int B = (int)sizeof(T) * N;
  constexpr int W = B >= 16 ? 16 : B;
  typedef typename hipmr_word<W>::t hipmr_aligned_word;
  typedef hipmr_aligned_word word __attribute__((aligned(sizeof(T))));
  hipmr_aligned_word tmp[B / W];
  const word* s = reinterpret_cast<const word*>(src);
#pragma unroll
  for (int k = 0; k < B / W; ++k) {
    if constexpr (NT) tmp[k] = __builtin_nontemporal_load(s + k);
    else tmp[k] = s[k];
  }
  __builtin_memcpy(&p, tmp, B);
}
template <bool NT, int N>
__device__ __forceinline__ void hipmr_load_any(hipmr_pack_fp8ro<N>& p, const hipmr_fp8* src) {
  hipmr_pack<hipmr_fp8, N> raw;
  hipmr_load_any<NT>(raw, src);
  __builtin_memcpy(&p, &raw, N);
}
)HIP";

const char* kEwVectorShift = R"HIP(
extern "C" __global__ void __launch_bounds__(@@BLOCK@@)
@@KNAME@@(@@PARAMS@@, long long hipmr_n, long long hipmr_head)
{
  typedef @@IDX@@ hipmr_idx;
  constexpr int HIPMR_B = @@BLOCK@@, HIPMR_U = @@IPT@@, HIPMR_V = @@VEC@@;
  constexpr bool HIPMR_NTL = @@NTL@@, HIPMR_NTS = @@NTS@@;
  const hipmr_idx n = (hipmr_idx)hipmr_n;
  @@SHIFT_INIT@@
  const long long hipmr_h = hipmr_head < hipmr_n ? hipmr_head : hipmr_n;
  const long long hipmr_nc = (hipmr_n - hipmr_h) / HIPMR_V;
  const long long hipmr_t0 = hipmr_h + hipmr_nc * HIPMR_V;
  if (blockIdx.x == 0) {
    if ((long long)threadIdx.x < hipmr_h) {
      const hipmr_idx i = (hipmr_idx)threadIdx.x;
      { @@STMT@@; }
    }
    if ((long long)threadIdx.x < hipmr_n - hipmr_t0) {
      const hipmr_idx i = (hipmr_idx)(hipmr_t0 + threadIdx.x);
      { @@STMT@@; }
    }
  }
  const long long hipmr_step = (long long)gridDim.x * (HIPMR_B * HIPMR_U);
  for (long long hipmr_c0 = (long long)hipmr_xcd_block(blockIdx.x) * (HIPMR_B * HIPMR_U) + threadIdx.x;
       hipmr_c0 < hipmr_nc; hipmr_c0 += hipmr_step) {
    @@DECL_PACKS@@
    @@SHIFT_PACKS@@
    bool hipmr_vec[HIPMR_U];
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_c = hipmr_c0 + hipmr_u * HIPMR_B;
      const long long hipmr_off = hipmr_h + hipmr_c * HIPMR_V;
      hipmr_vec[hipmr_u] = hipmr_c < hipmr_nc && hipmr_smin >= -hipmr_off &&
                           hipmr_smax <= hipmr_n - HIPMR_V - hipmr_off;   // no overflow for any distance
      if (hipmr_vec[hipmr_u]) {
        @@LOADS@@
        @@SHIFT_LOADS@@
      }
    }
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_c = hipmr_c0 + hipmr_u * HIPMR_B;
      const long long hipmr_off = hipmr_h + hipmr_c * HIPMR_V;
      if (hipmr_vec[hipmr_u]) {
#pragma unroll
        for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
          const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
          { @@VSTMT@@; }
        }
        @@STORES@@
      } else if (hipmr_c < hipmr_nc) {
        for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
          const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
          { @@STMT@@; }
        }
      }
    }
  }
}
)HIP";

const char* kEwScalar = R"HIP(
extern "C" __global__ void __launch_bounds__(@@BLOCK@@)
@@KNAME@@(@@PARAMS@@, long long hipmr_n, long long hipmr_head)
{
  typedef @@IDX@@ hipmr_idx;
  const hipmr_idx n = (hipmr_idx)hipmr_n;
  const long long hipmr_step = (long long)gridDim.x * @@BLOCK@@;
#pragma unroll @@IPT@@
  for (long long hipmr_k = (long long)blockIdx.x * @@BLOCK@@ + threadIdx.x; hipmr_k < hipmr_n;
       hipmr_k += hipmr_step) {
    const hipmr_idx i = (hipmr_idx)hipmr_k;
    { @@STMT@@; }
  }
}
)HIP";

const char* kRedS1Vector = R"HIP(
extern "C" __global__ void __launch_bounds__(@@BLOCK@@)
@@KNAME@@(@@PARAMS@@, long long hipmr_n, long long hipmr_head,
          hipmr_acc* __restrict__ hipmr_partial@@FPARAMS@@)
{
  typedef @@IDX@@ hipmr_idx;
  constexpr int HIPMR_B = @@BLOCK@@, HIPMR_U = @@IPT@@, HIPMR_V = @@VEC@@;
  constexpr bool HIPMR_NTL = @@NTL@@, HIPMR_NTS = @@NTS@@;
  const hipmr_idx n = (hipmr_idx)hipmr_n;
  const hipmr_acc hipmr_neutral = (hipmr_acc)(@@NEUTRAL@@);
  @@SHARES@@
  hipmr_acc hipmr_a[HIPMR_U];
#pragma unroll
  for (int u = 0; u < HIPMR_U; ++u) hipmr_a[u] = hipmr_neutral;
  const long long hipmr_h = hipmr_head < hipmr_n ? hipmr_head : hipmr_n;
  const long long hipmr_nc = (hipmr_n - hipmr_h) / HIPMR_V;
  const long long hipmr_t0 = hipmr_h + hipmr_nc * HIPMR_V;
  if (hipmr_b == 0) {
    if ((long long)threadIdx.x < hipmr_h) {
      const hipmr_idx i = (hipmr_idx)threadIdx.x;
      hipmr_a[0] = hipmr_combine(hipmr_a[0], (hipmr_acc)(@@MAP@@));
    }
    if ((long long)threadIdx.x < hipmr_n - hipmr_t0) {
      const hipmr_idx i = (hipmr_idx)(hipmr_t0 + threadIdx.x);
      hipmr_a[0] = hipmr_combine(hipmr_a[0], (hipmr_acc)(@@MAP@@));
    }
  }
  const long long hipmr_step = (long long)gridDim.x * (HIPMR_B * HIPMR_U);
  long long hipmr_c0 = (long long)hipmr_b * (HIPMR_B * HIPMR_U) + threadIdx.x;
  for (; hipmr_c0 + (HIPMR_U - 1) * HIPMR_B < hipmr_nc; hipmr_c0 += hipmr_step) {
    @@DECL_PACKS@@
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_off = hipmr_h + (hipmr_c0 + hipmr_u * HIPMR_B) * HIPMR_V;
      @@LOADS@@
    }
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_off = hipmr_h + (hipmr_c0 + hipmr_u * HIPMR_B) * HIPMR_V;
#pragma unroll
      for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
        const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
        hipmr_a[hipmr_u] = hipmr_combine(hipmr_a[hipmr_u], (hipmr_acc)(@@VMAP@@));
      }
    }
  }
  if (hipmr_c0 < hipmr_nc) {
    @@DECL_PACKS@@
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_c = hipmr_c0 + hipmr_u * HIPMR_B;
      if (hipmr_c < hipmr_nc) {
        const long long hipmr_off = hipmr_h + hipmr_c * HIPMR_V;
        @@LOADS@@
      }
    }
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_c = hipmr_c0 + hipmr_u * HIPMR_B;
      if (hipmr_c < hipmr_nc) {
        const long long hipmr_off = hipmr_h + hipmr_c * HIPMR_V;
#pragma unroll
        for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
          const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
          hipmr_a[hipmr_u] = hipmr_combine(hipmr_a[hipmr_u], (hipmr_acc)(@@VMAP@@));
        }
      }
    }
  }
  hipmr_acc hipmr_r = hipmr_fold<HIPMR_U>(hipmr_a);
  hipmr_r = hipmr_block_reduce<HIPMR_B>(hipmr_r, hipmr_neutral);
  @@FINISH@@
}
)HIP";

const char* kRedS1Scalar = R"HIP(
extern "C" __global__ void __launch_bounds__(@@BLOCK@@)
@@KNAME@@(@@PARAMS@@, long long hipmr_n, long long hipmr_head,
          hipmr_acc* __restrict__ hipmr_partial@@FPARAMS@@)
{
  typedef @@IDX@@ hipmr_idx;
  const hipmr_idx n = (hipmr_idx)hipmr_n;
  const hipmr_acc hipmr_neutral = (hipmr_acc)(@@NEUTRAL@@);
  @@SHARES@@
  hipmr_acc hipmr_r = hipmr_neutral;
  const long long hipmr_step = (long long)gridDim.x * @@BLOCK@@;
#pragma unroll @@IPT@@
  for (long long hipmr_k = (long long)hipmr_b * @@BLOCK@@ + threadIdx.x; hipmr_k < hipmr_n;
       hipmr_k += hipmr_step) {
    const hipmr_idx i = (hipmr_idx)hipmr_k;
    hipmr_r = hipmr_combine(hipmr_r, (hipmr_acc)(@@MAP@@));
  }
  hipmr_r = hipmr_block_reduce<@@BLOCK@@>(hipmr_r, hipmr_neutral);
  @@FINISH@@
}
)HIP";

// Reduce stage 1 for maps with shifted reads: as kEwVectorShift, each
// distinct shifted read is one unaligned chunk load, chunks within the largest
// distance of either end are mapped one element at a time, and workgroups
// take XCD-contiguous runs of chunks.  Each lane folds its chunks in order
// into U accumulators; the partial of workgroup b lands in partial[b].
const char* kRedS1VectorShift = R"HIP(
extern "C" __global__ void __launch_bounds__(@@BLOCK@@)
@@KNAME@@(@@PARAMS@@, long long hipmr_n, long long hipmr_head,
          hipmr_acc* __restrict__ hipmr_partial@@FPARAMS@@)
{
  typedef @@IDX@@ hipmr_idx;
  constexpr int HIPMR_B = @@BLOCK@@, HIPMR_U = @@IPT@@, HIPMR_V = @@VEC@@;
  constexpr bool HIPMR_NTL = @@NTL@@, HIPMR_NTS = @@NTS@@;
  const hipmr_idx n = (hipmr_idx)hipmr_n;
  @@SHIFT_INIT@@
  const hipmr_acc hipmr_neutral = (hipmr_acc)(@@NEUTRAL@@);
  @@SHARES@@
  hipmr_acc hipmr_a[HIPMR_U];
#pragma unroll
  for (int u = 0; u < HIPMR_U; ++u) hipmr_a[u] = hipmr_neutral;
  const long long hipmr_h = hipmr_head < hipmr_n ? hipmr_head : hipmr_n;
  const long long hipmr_nc = (hipmr_n - hipmr_h) / HIPMR_V;
  const long long hipmr_t0 = hipmr_h + hipmr_nc * HIPMR_V;
  if (hipmr_b == 0) {
    if ((long long)threadIdx.x < hipmr_h) {
      const hipmr_idx i = (hipmr_idx)threadIdx.x;
      hipmr_a[0] = hipmr_combine(hipmr_a[0], (hipmr_acc)(@@MAP@@));
    }
    if ((long long)threadIdx.x < hipmr_n - hipmr_t0) {
      const hipmr_idx i = (hipmr_idx)(hipmr_t0 + threadIdx.x);
      hipmr_a[0] = hipmr_combine(hipmr_a[0], (hipmr_acc)(@@MAP@@));
    }
  }
  const long long hipmr_step = (long long)gridDim.x * (HIPMR_B * HIPMR_U);
  for (long long hipmr_c0 = (long long)hipmr_xcd_block(hipmr_b) * (HIPMR_B * HIPMR_U) + threadIdx.x;
       hipmr_c0 < hipmr_nc; hipmr_c0 += hipmr_step) {
    @@DECL_PACKS@@
    @@SHIFT_PACKS@@
    bool hipmr_vec[HIPMR_U];
    // every lane loads every chunk, from a clamped in-range window where its
    // chunk is past the end or within a shifted read's distance of an end
    // (those chunks are then evaluated element by element): no branch
    // separates the loads, so they all stay in flight together
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_c = hipmr_c0 + hipmr_u * HIPMR_B;
      const long long hipmr_off = hipmr_c < hipmr_nc ? hipmr_h + hipmr_c * HIPMR_V : hipmr_h;
      hipmr_vec[hipmr_u] = hipmr_c < hipmr_nc && hipmr_smin >= -hipmr_off &&
                           hipmr_smax <= hipmr_n - HIPMR_V - hipmr_off;   // no overflow for any distance
      @@LOADS@@
      @@SHIFT_LOADS@@
    }
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_c = hipmr_c0 + hipmr_u * HIPMR_B;
      const long long hipmr_off = hipmr_h + hipmr_c * HIPMR_V;
      if (hipmr_vec[hipmr_u]) {
#pragma unroll
        for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
          const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
          hipmr_a[hipmr_u] = hipmr_combine(hipmr_a[hipmr_u], (hipmr_acc)(@@VMAP@@));
        }
      } else if (hipmr_c < hipmr_nc) {
        for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
          const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
          hipmr_a[hipmr_u] = hipmr_combine(hipmr_a[hipmr_u], (hipmr_acc)(@@MAP@@));
        }
      }
    }
  }
  hipmr_acc hipmr_r = hipmr_fold<HIPMR_U>(hipmr_a);
  hipmr_r = hipmr_block_reduce<HIPMR_B>(hipmr_r, hipmr_neutral);
  @@FINISH@@
}
)HIP";

// Share hipmr_b of a reduction, one chunk at a time: accumulator u takes the
// chunks that the body's u takes, in the same order.
const char* kRedShare = R"HIP(
    hipmr_acc hipmr_c[HIPMR_U];
#pragma unroll
    for (int u = 0; u < HIPMR_U; ++u) hipmr_c[u] = hipmr_neutral;
    if (hipmr_b == 0) {
      if ((long long)threadIdx.x < hipmr_h) {
        const hipmr_idx i = (hipmr_idx)threadIdx.x;
        hipmr_c[0] = hipmr_combine(hipmr_c[0], (hipmr_acc)(@@MAP@@));
      }
      if ((long long)threadIdx.x < hipmr_n - hipmr_t0) {
        const hipmr_idx i = (hipmr_idx)(hipmr_t0 + threadIdx.x);
        hipmr_c[0] = hipmr_combine(hipmr_c[0], (hipmr_acc)(@@MAP@@));
      }
    }
    for (long long hipmr_at = (long long)@@SHARE_BLOCK@@ * (HIPMR_B * HIPMR_U) + threadIdx.x; hipmr_at < hipmr_nc;
         hipmr_at += hipmr_step) {
#pragma unroll
      for (int hipmr_w = 0; hipmr_w < HIPMR_U; ++hipmr_w) {
        if (hipmr_at + hipmr_w * HIPMR_B < hipmr_nc) {
          const long long hipmr_off = hipmr_h + (hipmr_at + hipmr_w * HIPMR_B) * HIPMR_V;
          constexpr int HIPMR_U = 1, hipmr_u = 0;
          @@DECL_PACKS@@
          @@SHARE_CHUNK@@
        }
      }
    }
    hipmr_acc hipmr_q = hipmr_fold<HIPMR_U>(hipmr_c);
    hipmr_q = hipmr_block_reduce<HIPMR_B>(hipmr_q, hipmr_neutral);
)HIP";
const char* kRedShareChunk = R"HIP(
          @@LOADS@@
#pragma unroll
          for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
            const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
            hipmr_c[hipmr_w] = hipmr_combine(hipmr_c[hipmr_w], (hipmr_acc)(@@VMAP@@));
          }
)HIP";
const char* kRedShareChunkShift = R"HIP(
          @@SHIFT_PACKS@@
          @@LOADS@@
          @@SHIFT_LOADS@@
          if (hipmr_smin >= -hipmr_off && hipmr_smax <= hipmr_n - HIPMR_V - hipmr_off) {
#pragma unroll
            for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
              const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
              hipmr_c[hipmr_w] = hipmr_combine(hipmr_c[hipmr_w], (hipmr_acc)(@@VMAP@@));
            }
          } else {
            for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
              const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
              hipmr_c[hipmr_w] = hipmr_combine(hipmr_c[hipmr_w], (hipmr_acc)(@@MAP@@));
            }
          }
)HIP";
const char* kRedShareScalar = R"HIP(
    hipmr_acc hipmr_q = hipmr_neutral;
    for (long long hipmr_at = (long long)hipmr_b * @@BLOCK@@ + threadIdx.x; hipmr_at < hipmr_n; hipmr_at += hipmr_step) {
      const hipmr_idx i = (hipmr_idx)hipmr_at;
      hipmr_q = hipmr_combine(hipmr_q, (hipmr_acc)(@@MAP@@));
    }
    hipmr_q = hipmr_block_reduce<@@BLOCK@@>(hipmr_q, hipmr_neutral);
)HIP";

const char* kRedS2 = R"HIP(
extern "C" __global__ void __launch_bounds__(@@BLOCK@@)
@@KNAME@@(const hipmr_acc* __restrict__ hipmr_partial, int hipmr_g,
          hipmr_acc* __restrict__ hipmr_out)
{
  const hipmr_acc hipmr_neutral = (hipmr_acc)(@@NEUTRAL@@);
  hipmr_acc hipmr_r = hipmr_neutral;
  for (int k = threadIdx.x; k < hipmr_g; k += @@BLOCK@@)
    hipmr_r = hipmr_combine(hipmr_r, hipmr_partial[k]);
  hipmr_r = hipmr_block_reduce<@@BLOCK@@>(hipmr_r, hipmr_neutral);
  if (threadIdx.x == 0) *hipmr_out = hipmr_r;
}
)HIP";


// Compensated FP32 accumulation (precision extension).  Error-free
// transformations must not be contracted into FMAs.
const char* kCompHelpers = R"HIP(
#pragma clang fp contract(off)
// (hi, lo): an unevaluated sum of two floats
struct hipmr_ff { float hi, lo; };
struct hipmr_dd { double hi, lo; };

// Kahan: s + (-c) carries the running sum; c holds the rounding lost so far.
// Once the sum is infinite (or NaN) the correction is dropped, so that an
// infinity is not turned into a NaN by inf - inf.
__device__ __forceinline__ void hipmr_kahan_add(float& s, float& c, float v) {
  const float y = v - c;
  const float t = s + y;
  c = __builtin_isfinite(t) ? (t - s) - y : 0.0f;
  s = t;
}

// Knuth's TwoSum: a + b = s + e exactly, no ordering assumption
__device__ __forceinline__ hipmr_ff hipmr_two_sum(float a, float b) {
  const float s = a + b;
  const float bb = s - a;
  return {s, __builtin_isfinite(s) ? (a - (s - bb)) + (b - bb) : 0.0f};
}
__device__ __forceinline__ hipmr_ff hipmr_ff_add(hipmr_ff x, hipmr_ff y) {
  const hipmr_ff s = hipmr_two_sum(x.hi, y.hi);
  return hipmr_two_sum(s.hi, s.lo + (x.lo + y.lo));
}
__device__ __forceinline__ hipmr_dd hipmr_two_sum_d(double a, double b) {
  const double s = a + b;
  const double bb = s - a;
  return {s, __builtin_isfinite(s) ? (a - (s - bb)) + (b - bb) : 0.0};
}
__device__ __forceinline__ hipmr_dd hipmr_dd_add(hipmr_dd x, hipmr_dd y) {
  const hipmr_dd s = hipmr_two_sum_d(x.hi, y.hi);
  return hipmr_two_sum_d(s.hi, s.lo + (x.lo + y.lo));
}

// Block maximum of non-negative values (NaN wins), valid in every thread.
template <int B>
__device__ __forceinline__ float hipmr_block_amax(float m) {
  __shared__ float hipmr_amax_lds[B / 64];
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) m = __builtin_elementwise_maximum(m, __shfl_xor(m, d, 64));
  if ((threadIdx.x & 63) == 0) hipmr_amax_lds[threadIdx.x >> 6] = m;
  __syncthreads();
  m = hipmr_amax_lds[0];
#pragma unroll
  for (int w = 1; w < B / 64; ++w) m = __builtin_elementwise_maximum(m, hipmr_amax_lds[w]);
  return m;
}

// The norm's power-of-two scale from its first pass: the max |map| over
// that pass's block partials (one per block of this grid: both passes use
// the same geometry).  Where that maximum is 0 or lies in [2^-40, 2^40] the
// first pass's own sums of unscaled squares stand (0 is returned): n < 2^47 such
// squares stay below 2^127.  Scaling by a power of two changes no bit of a
// square that is normal either way; a value below 2^-63, which the scale would
// have raised, has a subnormal square here and loses at most 2^-150, which is
// 2^-70 of the largest square: far below the sum's own rounding.  Else s = 2^-e, e the
// exponent of the max clamped to [-126, 126], so the largest scaled
// magnitude lies in [1, 2).  Every block computes it.
template <int B>
__device__ __forceinline__ float hipmr_norm_scale(const float* __restrict__ amax, int g) {
  float m = 0.0f;
  for (int k = threadIdx.x; k < g; k += B) m = __builtin_elementwise_maximum(m, amax[k]);
  m = hipmr_block_amax<B>(m);
  const bool stands = m == 0.0f || (m >= 0x1p-40f && m <= 0x1p40f);
  float s = 1.0f;
  if (m > 0.0f && !stands) {
    int e = (int)((__float_as_uint(m) >> 23) & 0xffu) - 127;
    e = e < -126 ? -126 : (e > 126 ? 126 : e);
    s = __uint_as_float((unsigned int)(127 - e) << 23);
  }
  return stands ? 0.0f : s;
}

// pairwise sum of one chunk's V terms (fixed tree); the chunk sum then
// enters the compensated accumulator
template <int V>
__device__ __forceinline__ float hipmr_chunk_sum(float* t) {
#pragma unroll
  for (int w = 1; w < V; w *= 2) {
#pragma unroll
    for (int j = 0; j + w < V; j += 2 * w) t[j] += t[j + w];
  }
  return t[0];
}

template <bool SQ, bool TRACK>
__device__ __forceinline__ float hipmr_term(float v, float scale, float& amax) {
  if constexpr (TRACK) amax = __builtin_elementwise_maximum(amax, __builtin_fabsf(v));
  if constexpr (SQ) {
    const float w = TRACK ? v : v * scale;
    return w * w;
  } else {
    return v;
  }
}

// pairwise combination of (hi, lo) pairs across the wave, then the block
template <int B, typename P, typename F>
__device__ __forceinline__ P hipmr_block_reduce_pair(P v, F add) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    P o;
    o.hi = __shfl_xor(v.hi, m, 64);
    o.lo = __shfl_xor(v.lo, m, 64);
    v = add(v, o);
  }
  if constexpr (B > 64) {
    constexpr int W = B / 64;
    constexpr int PW = W <= 2 ? 2 : W <= 4 ? 4 : W <= 8 ? 8 : 16;
    __shared__ P hipmr_lds_pair[W];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    if (l == 0) hipmr_lds_pair[w] = v;
    __syncthreads();
    if (w == 0) {
      if (l < W) v = hipmr_lds_pair[l];
      else { v.hi = 0; v.lo = 0; }
#pragma unroll
      for (int m = PW / 2; m >= 1; m >>= 1) {
        P o;
        o.hi = __shfl_xor(v.hi, m, 64);
        o.lo = __shfl_xor(v.lo, m, 64);
        v = add(v, o);
      }
    }
  }
  return v;
}

// The end of a sum or norm, by one block: the FP64 block partials folded
// (Neumaier per thread, double-double tree), times the per-tensor post scale;
// a norm is the root, over the data's scale.  The partials may be other
// blocks' of the same launch: they are read with device-scope loads.
struct hipmr_neumaier {
  double s, c;
  __device__ __forceinline__ void add(double v) {
    const double t = s + v;
    if (__builtin_isfinite(t)) c += fabs(s) >= fabs(v) ? (s - t) + v : (v - t) + s;
    s = t;
  }
};
template <int B, bool NORM>
__device__ __forceinline__ void hipmr_comp_end(hipmr_neumaier f, double post, double scale, double* __restrict__ out) {
  hipmr_dd r = hipmr_two_sum_d(f.s, f.c);
  r = hipmr_block_reduce_pair<B>(r, [](hipmr_dd a, hipmr_dd b) { return hipmr_dd_add(a, b); });
  if (threadIdx.x == 0) {
    const double total = __builtin_isfinite(r.hi) ? r.hi + r.lo : r.hi;
    if constexpr (NORM) *out = post * (sqrt(total) / scale);
    else *out = post * total;
  }
}
template <int B, bool NORM>
__device__ __forceinline__ void hipmr_comp_fold(const double* partial, int g, double post, double scale,
                                                double* __restrict__ out) {
  hipmr_neumaier f = {0.0, 0.0};
  for (int k = threadIdx.x; k < g; k += B)
    f.add(__builtin_bit_cast(double, __hip_atomic_load((const unsigned long long*)partial + k, __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT)));
  hipmr_comp_end<B, NORM>(f, post, scale, out);
}

// The end of a sum or norm in its own launch (partials by tag), as hipmr_finish
// and hipmr_add_share above.
template <int B, bool NORM>
__device__ __forceinline__ bool hipmr_comp_finish(double v, unsigned long long* part, double post, double scale,
                                                  unsigned long long tag, double* __restrict__ out) {
  const int g = (int)gridDim.x;
  if (threadIdx.x == 0) hipmr_put_tagged(part, (int)blockIdx.x, v, tag);
  if ((int)blockIdx.x != g - 1) return false;
  hipmr_neumaier f = {0.0, 0.0};
  bool here = true;
  for (int k = threadIdx.x; here && k < g; k += B) {
    double p;
    here = hipmr_get_tagged(part, k, tag, &p);
    if (here) f.add(p);
  }
  if (hipmr_any<B>(!here)) return true;
  hipmr_comp_end<B, NORM>(f, post, scale, out);
  return false;
}
template <int B, bool NORM>
__device__ __forceinline__ void hipmr_comp_add_share(hipmr_neumaier& f, double v, double post, double scale,
                                                     double* __restrict__ out, int b) {
  __shared__ double hipmr_share;
  if (threadIdx.x == 0) hipmr_share = v;
  __syncthreads();
  if ((int)threadIdx.x == b % B) f.add(hipmr_share);
  __syncthreads();
  if (b + 1 == (int)gridDim.x) hipmr_comp_end<B, NORM>(f, post, scale, out);
}
)HIP";

// Stage 1 of a compensated sum, or of the norm's sum of squares: its first
// pass (nrm1) sums the unscaled squares and keeps each block's max |map|, its
// second (nrm2) rescales and sums again only where those squares could have
// left the float range, its last block folding the partials (the words they
// travel in are cleared by the first pass, so their tag is a constant, also in
// a replay), and otherwise one block of it folds the first pass's
// partials.  Bound: HBM, one read (a pass for the maximum, always a second one
// for the sum and a fold launch took 81.6 us for 2^27 bfloat16 values, the sums
// beside the maximum 45.0, without the fold launch 43.4).
const char* kCompS1Vector = R"HIP(
extern "C" __global__ void __launch_bounds__(@@BLOCK@@)
@@KNAME@@(@@PARAMS@@, long long hipmr_n, long long hipmr_head,
          double* __restrict__ hipmr_partial, float* __restrict__ hipmr_scale_p,
          double hipmr_post, double* __restrict__ hipmr_out, unsigned long long hipmr_tag)
{
  typedef @@IDX@@ hipmr_idx;
  constexpr int HIPMR_B = @@BLOCK@@, HIPMR_U = @@IPT@@, HIPMR_V = @@VEC@@;
  constexpr bool HIPMR_NTL = @@NTL@@, HIPMR_NTS = @@NTS@@;
  constexpr bool HIPMR_SQ = @@SQUARE@@, HIPMR_RUNS = @@RUNS@@, HIPMR_SCALED = @@SCALED@@, HIPMR_TRACK = @@TRACK@@;
  const hipmr_idx n = (hipmr_idx)hipmr_n;
  float hipmr_sc = 1.0f, hipmr_m = 0.0f;
  if constexpr (HIPMR_SCALED) {
    hipmr_sc = hipmr_norm_scale<HIPMR_B>(hipmr_scale_p, (int)gridDim.x);
    if (!@@ONE@@ && blockIdx.x == 0 && threadIdx.x == 0) hipmr_scale_p[@@SCALE_AT@@] = hipmr_sc;   // for the fold
    if (hipmr_sc == 0.0f) {                     // the first pass's sums stand
      if (@@ONE@@ && blockIdx.x == 0)
        hipmr_comp_fold<HIPMR_B, true>(hipmr_partial, (int)gridDim.x, hipmr_post, 1.0, hipmr_out);
      return;
    }
  }
  @@SHARES@@
  float hipmr_s[HIPMR_U], hipmr_e[HIPMR_U];
#pragma unroll
  for (int u = 0; u < HIPMR_U; ++u) { hipmr_s[u] = 0.0f; hipmr_e[u] = 0.0f; }
  const long long hipmr_h = hipmr_head < hipmr_n ? hipmr_head : hipmr_n;
  const long long hipmr_nc = (hipmr_n - hipmr_h) / HIPMR_V;
  const long long hipmr_t0 = hipmr_h + hipmr_nc * HIPMR_V;
  if (hipmr_b == 0) {
    if ((long long)threadIdx.x < hipmr_h) {
      const hipmr_idx i = (hipmr_idx)threadIdx.x;
      hipmr_kahan_add(hipmr_s[0], hipmr_e[0], hipmr_term<HIPMR_SQ, HIPMR_TRACK>((float)(@@MAP@@), hipmr_sc, hipmr_m));
    }
    if ((long long)threadIdx.x < hipmr_n - hipmr_t0) {
      const hipmr_idx i = (hipmr_idx)(hipmr_t0 + threadIdx.x);
      hipmr_kahan_add(hipmr_s[0], hipmr_e[0], hipmr_term<HIPMR_SQ, HIPMR_TRACK>((float)(@@MAP@@), hipmr_sc, hipmr_m));
    }
  }
  const long long hipmr_step = (long long)gridDim.x * (HIPMR_B * HIPMR_U);
  long long hipmr_c0 = (long long)hipmr_b * (HIPMR_B * HIPMR_U) + threadIdx.x;
  for (; hipmr_c0 + (HIPMR_U - 1) * HIPMR_B < hipmr_nc; hipmr_c0 += hipmr_step) {
    @@DECL_PACKS@@
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_off = hipmr_h + (hipmr_c0 + hipmr_u * HIPMR_B) * HIPMR_V;
      @@LOADS@@
    }
    if constexpr (HIPMR_RUNS) {
      // every value is k * 2^-9 with |k| <= 229376: a float sum of at most
      // 64 of them is exact, so one compensated step per run suffices
      float hipmr_run = 0.0f;
#pragma unroll
      for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
        const long long hipmr_off = hipmr_h + (hipmr_c0 + hipmr_u * HIPMR_B) * HIPMR_V;
#pragma unroll
        for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
          const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
          hipmr_run += (float)(@@VMAP@@);
        }
      }
      hipmr_kahan_add(hipmr_s[0], hipmr_e[0], hipmr_run);
    } else {
#pragma unroll
      for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
        const long long hipmr_off = hipmr_h + (hipmr_c0 + hipmr_u * HIPMR_B) * HIPMR_V;
        float hipmr_t[HIPMR_V];
#pragma unroll
        for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
          const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
          hipmr_t[hipmr_j] = hipmr_term<HIPMR_SQ, HIPMR_TRACK>((float)(@@VMAP@@), hipmr_sc, hipmr_m);
        }
        hipmr_kahan_add(hipmr_s[hipmr_u], hipmr_e[hipmr_u], hipmr_chunk_sum<HIPMR_V>(hipmr_t));
      }
    }
  }
  if (hipmr_c0 < hipmr_nc) {
    @@DECL_PACKS@@
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_c = hipmr_c0 + hipmr_u * HIPMR_B;
      if (hipmr_c < hipmr_nc) {
        const long long hipmr_off = hipmr_h + hipmr_c * HIPMR_V;
        @@LOADS@@
      }
    }
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_c = hipmr_c0 + hipmr_u * HIPMR_B;
      if (hipmr_c < hipmr_nc) {
        const long long hipmr_off = hipmr_h + hipmr_c * HIPMR_V;
        float hipmr_t[HIPMR_V];
#pragma unroll
        for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
          const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
          hipmr_t[hipmr_j] = hipmr_term<HIPMR_SQ, HIPMR_TRACK>((float)(@@VMAP@@), hipmr_sc, hipmr_m);
        }
        hipmr_kahan_add(hipmr_s[hipmr_u], hipmr_e[hipmr_u], hipmr_chunk_sum<HIPMR_V>(hipmr_t));
      }
    }
  }
  hipmr_ff hipmr_r = {hipmr_s[0], -hipmr_e[0]};
#pragma unroll
  for (int u = 1; u < HIPMR_U; ++u) hipmr_r = hipmr_ff_add(hipmr_r, hipmr_ff{hipmr_s[u], -hipmr_e[u]});
  hipmr_r = hipmr_block_reduce_pair<HIPMR_B>(hipmr_r, [](hipmr_ff a, hipmr_ff b) { return hipmr_ff_add(a, b); });
  const double hipmr_v = __builtin_isfinite(hipmr_r.hi) ? (double)hipmr_r.hi + (double)hipmr_r.lo
                                                        : (double)hipmr_r.hi;
  unsigned long long* const hipmr_words = (unsigned long long*)hipmr_partial + (HIPMR_SCALED || HIPMR_TRACK ? @@WORDS_AT@@ : 0);
  @@FINISH@@
  if constexpr (HIPMR_TRACK) {
    hipmr_m = hipmr_block_amax<@@BLOCK@@>(hipmr_m);
    if (threadIdx.x == 0) hipmr_scale_p[blockIdx.x] = hipmr_m;
    if (threadIdx.x < 4 && gridDim.x <= @@WORDS_FOR@@) hipmr_words[blockIdx.x * 4 + threadIdx.x] = 0;
  }
}
)HIP";

const char* kCompS1Scalar = R"HIP(
extern "C" __global__ void __launch_bounds__(@@BLOCK@@)
@@KNAME@@(@@PARAMS@@, long long hipmr_n, long long hipmr_head,
          double* __restrict__ hipmr_partial, float* __restrict__ hipmr_scale_p,
          double hipmr_post, double* __restrict__ hipmr_out, unsigned long long hipmr_tag)
{
  typedef @@IDX@@ hipmr_idx;
  constexpr bool HIPMR_SQ = @@SQUARE@@, HIPMR_SCALED = @@SCALED@@, HIPMR_TRACK = @@TRACK@@;
  const hipmr_idx n = (hipmr_idx)hipmr_n;
  float hipmr_sc = 1.0f, hipmr_m = 0.0f;
  if constexpr (HIPMR_SCALED) {
    hipmr_sc = hipmr_norm_scale<@@BLOCK@@>(hipmr_scale_p, (int)gridDim.x);
    if (!@@ONE@@ && blockIdx.x == 0 && threadIdx.x == 0) hipmr_scale_p[@@SCALE_AT@@] = hipmr_sc;   // for the fold
    if (hipmr_sc == 0.0f) {                     // the first pass's sums stand
      if (@@ONE@@ && blockIdx.x == 0)
        hipmr_comp_fold<@@BLOCK@@, true>(hipmr_partial, (int)gridDim.x, hipmr_post, 1.0, hipmr_out);
      return;
    }
  }
  @@SHARES@@
  float hipmr_s = 0.0f, hipmr_cc = 0.0f;
  const long long hipmr_step = (long long)gridDim.x * @@BLOCK@@;
  for (long long hipmr_k = (long long)hipmr_b * @@BLOCK@@ + threadIdx.x; hipmr_k < hipmr_n;
       hipmr_k += hipmr_step) {
    const hipmr_idx i = (hipmr_idx)hipmr_k;
    hipmr_kahan_add(hipmr_s, hipmr_cc, hipmr_term<HIPMR_SQ, HIPMR_TRACK>((float)(@@MAP@@), hipmr_sc, hipmr_m));
  }
  hipmr_ff hipmr_r = {hipmr_s, -hipmr_cc};
  hipmr_r = hipmr_block_reduce_pair<@@BLOCK@@>(hipmr_r, [](hipmr_ff a, hipmr_ff b) { return hipmr_ff_add(a, b); });
  const double hipmr_v = __builtin_isfinite(hipmr_r.hi) ? (double)hipmr_r.hi + (double)hipmr_r.lo
                                                        : (double)hipmr_r.hi;
  unsigned long long* const hipmr_words = (unsigned long long*)hipmr_partial + (HIPMR_SCALED || HIPMR_TRACK ? @@WORDS_AT@@ : 0);
  @@FINISH@@
  if constexpr (HIPMR_TRACK) {
    hipmr_m = hipmr_block_amax<@@BLOCK@@>(hipmr_m);
    if (threadIdx.x == 0) hipmr_scale_p[blockIdx.x] = hipmr_m;
    if (threadIdx.x < 4 && gridDim.x <= @@WORDS_FOR@@) hipmr_words[blockIdx.x * 4 + threadIdx.x] = 0;
  }
}
)HIP";

// Share hipmr_b of a compensated sum or norm, one chunk at a time.
const char* kCompShare = R"HIP(
    float hipmr_c[HIPMR_U], hipmr_d[HIPMR_U];
#pragma unroll
    for (int u = 0; u < HIPMR_U; ++u) { hipmr_c[u] = 0.0f; hipmr_d[u] = 0.0f; }
    if (hipmr_b == 0) {
      if ((long long)threadIdx.x < hipmr_h) {
        const hipmr_idx i = (hipmr_idx)threadIdx.x;
        hipmr_kahan_add(hipmr_c[0], hipmr_d[0], hipmr_term<HIPMR_SQ, HIPMR_TRACK>((float)(@@MAP@@), hipmr_sc, hipmr_m));
      }
      if ((long long)threadIdx.x < hipmr_n - hipmr_t0) {
        const hipmr_idx i = (hipmr_idx)(hipmr_t0 + threadIdx.x);
        hipmr_kahan_add(hipmr_c[0], hipmr_d[0], hipmr_term<HIPMR_SQ, HIPMR_TRACK>((float)(@@MAP@@), hipmr_sc, hipmr_m));
      }
    }
    for (long long hipmr_at = (long long)hipmr_b * (HIPMR_B * HIPMR_U) + threadIdx.x; hipmr_at < hipmr_nc;
         hipmr_at += hipmr_step) {
      const bool hipmr_run_of_all = HIPMR_RUNS && hipmr_at + (HIPMR_U - 1) * HIPMR_B < hipmr_nc;
      float hipmr_run = 0.0f;
#pragma unroll
      for (int hipmr_w = 0; hipmr_w < HIPMR_U; ++hipmr_w) {
        if (hipmr_at + hipmr_w * HIPMR_B < hipmr_nc) {
          const long long hipmr_off = hipmr_h + (hipmr_at + hipmr_w * HIPMR_B) * HIPMR_V;
          constexpr int HIPMR_U = 1, hipmr_u = 0;
          @@DECL_PACKS@@
          @@LOADS@@
          float hipmr_t[HIPMR_V];
#pragma unroll
          for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
            const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
            const float hipmr_x = (float)(@@VMAP@@);
            if (hipmr_run_of_all) hipmr_run += hipmr_x;
            hipmr_t[hipmr_j] = hipmr_term<HIPMR_SQ, HIPMR_TRACK>(hipmr_x, hipmr_sc, hipmr_m);
          }
          if (!hipmr_run_of_all) hipmr_kahan_add(hipmr_c[hipmr_w], hipmr_d[hipmr_w], hipmr_chunk_sum<HIPMR_V>(hipmr_t));
        }
      }
      if (hipmr_run_of_all) hipmr_kahan_add(hipmr_c[0], hipmr_d[0], hipmr_run);
    }
    hipmr_ff hipmr_q = {hipmr_c[0], -hipmr_d[0]};
#pragma unroll
    for (int u = 1; u < HIPMR_U; ++u) hipmr_q = hipmr_ff_add(hipmr_q, hipmr_ff{hipmr_c[u], -hipmr_d[u]});
)HIP";
const char* kCompShareScalar = R"HIP(
    float hipmr_c = 0.0f, hipmr_d = 0.0f;
    for (long long hipmr_at = (long long)hipmr_b * @@BLOCK@@ + threadIdx.x; hipmr_at < hipmr_n; hipmr_at += hipmr_step) {
      const hipmr_idx i = (hipmr_idx)hipmr_at;
      hipmr_kahan_add(hipmr_c, hipmr_d, hipmr_term<HIPMR_SQ, HIPMR_TRACK>((float)(@@MAP@@), hipmr_sc, hipmr_m));
    }
    hipmr_ff hipmr_q = {hipmr_c, -hipmr_d};
)HIP";
const char* kCompShareEnd = R"HIP(
    hipmr_q = hipmr_block_reduce_pair<@@BLOCK@@>(hipmr_q, [](hipmr_ff a, hipmr_ff b) { return hipmr_ff_add(a, b); });
    const double hipmr_y = __builtin_isfinite(hipmr_q.hi) ? (double)hipmr_q.hi + (double)hipmr_q.lo : (double)hipmr_q.hi;
    hipmr_comp_add_share<@@BLOCK@@, HIPMR_SQ>(hipmr_f, hipmr_y, hipmr_post, (double)hipmr_sc, hipmr_out, hipmr_b);
)HIP";

// Final fold of a compensated sum or a norm in a launch of its own; after two
// passes the partials are the second's if there was a scale, else the first's.
const char* kCompS2 = R"HIP(
extern "C" __global__ void __launch_bounds__(@@BLOCK@@)
@@KNAME@@(const double* __restrict__ hipmr_partial, int hipmr_g, double hipmr_post,
          const float* __restrict__ hipmr_scale_p, double* __restrict__ hipmr_out)
{
  float hipmr_sc = 1.0f;
  if constexpr (@@SCALED@@) hipmr_sc = hipmr_scale_p[@@SCALE_AT@@];
  hipmr_comp_fold<@@BLOCK@@, @@NORM@@>(hipmr_partial, hipmr_g, hipmr_post, hipmr_sc == 0.0f ? 1.0 : (double)hipmr_sc,
                                       hipmr_out);
}
)HIP";



// ------------------------------------------------------------ batching
// Segments [off[s], off[s+1]) of the concatenated arrays are cut into tiles:
// tile 0 of a segment holds its unaligned head plus up to T body elements,
// later tiles T body elements each, where body elements start at the first
// index congruent to `head` modulo V (every accessed array is 16-byte aligned
// there) and T = 64 * V * IPT.  One wave reduces one tile.  The partition of
// a segment depends only on its bounds, V and IPT, never on other segments.
const char* kSegHelpers = R"HIP(
__device__ __forceinline__ void hipmr_seg_clamp(long long a0, long long b0, long long total,
                                                long long head, int V,
                                                long long& a, long long& b, long long& ab) {
  a = a0;
  b = b0;
  a = a < 0 ? 0 : (a > total ? total : a);
  b = b < a ? a : (b > total ? total : b);
  long long r = (head - a) % V;
  if (r < 0) r += V;
  ab = a + r < b ? a + r : b;
}
__device__ __forceinline__ int hipmr_seg_tiles(long long a, long long b, long long ab, long long T) {
  if (b == a) return 0;
  const long long t = (b - ab + T - 1) / T;
  return t < 1 ? 1 : (int)t;
}

// The tile table: tiles per segment and their exclusive prefix, by one block
// of B threads, in rounds of B * R segments: a thread takes R consecutive ones
// (all of a round's offsets are loaded before any is used), so a round costs
// one trip to memory, two barriers and one wave scan per R segments.  Every
// block of the tile kernel plans for itself, so the instructions count as well:
// a scan per 64 segments over coalesced loads took 46.4 us where this takes
// 41.1 (8191 segments of 2^24 floats, 256 threads x 8 blocks per compute unit),
// and 21.8 against 20.8 in the default geometry; R = 8 is level there and costs
// the planning launch 24.1 against 22.4.  Counts are
// summed in 64 bits and every entry is capped at the tile capacity of the
// workspace, so offsets that describe more tiles than it holds (overlapping
// segments) can never send a later kernel past it.  The table goes to `lds`
// and / or `glob` (either may be null); it is complete when this returns.
template <int B, int R>
__device__ void hipmr_seg_plan(const long long* __restrict__ off, int nseg, long long total,
                               long long head, int V, long long T, long long cap,
                               int* lds, int* __restrict__ glob) {
  __shared__ long long hipmr_wsum[B / 64];
  const auto hipmr_plus = [](long long p, long long q) { return p + q; };
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  long long carry = 0;                           // tiles of the earlier rounds, in every thread
  for (int base = 0; base < nseg; base += B * R) {
    const int s0 = base + (int)threadIdx.x * R;
    long long o[R + 1];
#pragma unroll
    for (int j = 0; j <= R; ++j) o[j] = s0 + j <= nseg ? off[s0 + j] : 0;
    long long t[R], sum = 0;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      t[j] = 0;
      if (s0 + j < nseg) {
        long long a, b, ab;
        hipmr_seg_clamp(o[j], o[j + 1], total, head, V, a, b, ab);
        t[j] = hipmr_seg_tiles(a, b, ab, T);
      }
      sum += t[j];
    }
    const long long incl = hipmr_dpp_scan(sum, 0LL, hipmr_plus);
    if (l == 63) hipmr_wsum[w] = incl;
    __syncthreads();
    const long long v = hipmr_dpp_scan(l < B / 64 ? hipmr_wsum[l] : 0LL, 0LL, hipmr_plus);
    long long run = carry + (w > 0 ? __shfl(v, w - 1, 64) : 0LL) + incl - sum;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (s0 + j < nseg) {
        const int e = (int)(run < cap ? run : cap);
        if (lds) lds[s0 + j] = e;
        if (glob) glob[s0 + j] = e;
      }
      run += t[j];
    }
    carry += __shfl(v, B / 64 - 1, 64);
    __syncthreads();                             // hipmr_wsum is written again; the table is read next
  }
  if (threadIdx.x == 0) {
    const int e = (int)(carry < cap ? carry : cap);
    if (lds) lds[nseg] = e;
    if (glob) glob[nseg] = e;
  }
  __syncthreads();
}
)HIP";

// Planner (for tables too large for LDS): the tile table in global memory,
// one block of 1024 threads.
const char* kSegPlan = R"HIP(
extern "C" __global__ void __launch_bounds__(1024)
@@KNAME@@(const long long* __restrict__ hipmr_off, int hipmr_nseg, long long hipmr_total,
          long long hipmr_head, int* __restrict__ hipmr_tile_start, long long hipmr_cap)
{
  hipmr_seg_plan<1024, 4>(hipmr_off, hipmr_nseg, hipmr_total, hipmr_head, @@VEC@@,
                       64LL * @@VEC@@ * @@IPT@@, hipmr_cap, nullptr, hipmr_tile_start);
}
)HIP";

// the fold of a wave's values, in lane order (stage 1)
const char* kSegFold = R"HIP(
__device__ __forceinline__ hipmr_acc hipmr_wave_total(hipmr_acc v, hipmr_acc e, int lane) {
  if constexpr (sizeof(hipmr_acc) == 4 || sizeof(hipmr_acc) == 8) {
    return hipmr_dpp_scan(v, e, [](hipmr_acc a, hipmr_acc b) { return hipmr_combine(a, b); });
  } else {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const hipmr_acc y = __shfl_up(v, d, 64);
      if (lane >= d) v = hipmr_combine(y, v);
    }
    return v;
  }
}
)HIP";

// Persistent stage 1: waves take tiles t = wave, wave + nwaves, ...  (With
// the table in LDS this is also the planner: no separate planning launch.)
// Per tile, every load is issued before any result is used: the head and
// tail elements, then the body chunks; the next tile's segment is found (in
// the table) and its offsets fetched while they are in flight.  The wave's
// fold is a DPP scan whose last lane holds the tile partial.
const char* kSegS1 = R"HIP(
extern "C" __global__ void __launch_bounds__(@@BLOCK@@)
@@KNAME@@(@@PARAMS@@, long long hipmr_total, long long hipmr_head,
          const long long* __restrict__ hipmr_offsets, int hipmr_nseg,
          int* __restrict__ hipmr_tile_start, hipmr_acc* __restrict__ hipmr_tpart,
          long long hipmr_cap)
{
  typedef @@IDX@@ hipmr_idx;
  constexpr int HIPMR_B = @@BLOCK@@, HIPMR_U = @@IPT@@, HIPMR_V = @@VEC@@, HIPMR_LDS_SEGS = @@LDS_SEGS@@;
  constexpr bool HIPMR_NTL = @@NTL@@, HIPMR_NTS = @@NTS@@;
  constexpr long long HIPMR_T = 64LL * HIPMR_V * HIPMR_U;
  const hipmr_idx n = (hipmr_idx)hipmr_total;
  const hipmr_acc hipmr_neutral = (hipmr_acc)(@@NEUTRAL@@);
  const int hipmr_lane = threadIdx.x & 63;
  // the tile-start table: a variant with LDS room computes it there in
  // every block (block 0 also writes it to global memory for the
  // per-segment fold); otherwise the planner has written it to global
  // memory.  (The host picks the LDS variant only when the table fits.)
  const int* hipmr_tab;
  if constexpr (HIPMR_LDS_SEGS > 0) {
    __shared__ int hipmr_ts_lds[HIPMR_LDS_SEGS + 1];
    if (hipmr_nseg > HIPMR_LDS_SEGS) return;
    constexpr int HIPMR_R = HIPMR_LDS_SEGS < HIPMR_B ? 1 : HIPMR_LDS_SEGS >= 4 * HIPMR_B ? 4 : (HIPMR_LDS_SEGS + 1) / HIPMR_B;
    hipmr_seg_plan<HIPMR_B, HIPMR_R>(hipmr_offsets, hipmr_nseg, hipmr_total, hipmr_head, HIPMR_V, HIPMR_T,
                            hipmr_cap, hipmr_ts_lds, blockIdx.x == 0 ? hipmr_tile_start : nullptr);
    hipmr_tab = hipmr_ts_lds;
  } else {
    hipmr_tab = hipmr_tile_start;
  }
  // the planner caps the table at the workspace's tile capacity; the cap is
  // applied here again so that no tile partial is written past it
  const int hipmr_total_tiles = hipmr_tab[hipmr_nseg] < hipmr_cap ? hipmr_tab[hipmr_nseg] : (int)hipmr_cap;
  const int hipmr_nwaves = gridDim.x * (HIPMR_B / 64);
  // segment of a tile: the last s with tile_start[s] <= tile (64-way ballot search)
  auto hipmr_find = [&](int hipmr_tile) -> int {
    int hipmr_lo = 0, hipmr_hi = hipmr_nseg - 1;
    while (hipmr_lo < hipmr_hi) {
      const int hipmr_step = (hipmr_hi - hipmr_lo + 64) / 64;
      const int hipmr_cand = hipmr_lo + hipmr_lane * hipmr_step;
      const bool hipmr_pred = hipmr_cand <= hipmr_hi && hipmr_tab[hipmr_cand] <= hipmr_tile;
      const unsigned long long hipmr_m = __ballot(hipmr_pred);
      const int hipmr_k = 63 - __builtin_clzll(hipmr_m);
      hipmr_lo = hipmr_lo + hipmr_k * hipmr_step;
      hipmr_hi = hipmr_lo + hipmr_step - 1 < hipmr_hi ? hipmr_lo + hipmr_step - 1 : hipmr_hi;
    }
    return hipmr_lo;
  };
  int hipmr_t = blockIdx.x * (HIPMR_B / 64) + (threadIdx.x >> 6);
  int hipmr_s = 0;
  long long hipmr_oa = 0, hipmr_ob = 0;
  if (hipmr_t < hipmr_total_tiles) {
    hipmr_s = hipmr_find(hipmr_t);
    hipmr_oa = hipmr_offsets[hipmr_s];
    hipmr_ob = hipmr_offsets[hipmr_s + 1];
  }
  for (; hipmr_t < hipmr_total_tiles; hipmr_t += hipmr_nwaves) {
    long long hipmr_sa, hipmr_sb, hipmr_sab;
    hipmr_seg_clamp(hipmr_oa, hipmr_ob, hipmr_total, hipmr_head, HIPMR_V, hipmr_sa, hipmr_sb, hipmr_sab);
    const long long hipmr_k = hipmr_t - hipmr_tab[hipmr_s];
    const long long hipmr_tstart = hipmr_k == 0 ? hipmr_sa : hipmr_sab + hipmr_k * HIPMR_T;
    const long long hipmr_hend = hipmr_k == 0 ? hipmr_sab : hipmr_tstart;
    const long long hipmr_te = hipmr_sab + (hipmr_k + 1) * HIPMR_T < hipmr_sb ? hipmr_sab + (hipmr_k + 1) * HIPMR_T : hipmr_sb;
    const long long hipmr_nch = hipmr_te > hipmr_hend ? (hipmr_te - hipmr_hend) / HIPMR_V : 0;
    const long long hipmr_tail = hipmr_hend + hipmr_nch * HIPMR_V;
    // the unaligned head (tile 0 only) and the ragged tail, one element per lane
    hipmr_acc hipmr_hv = hipmr_neutral, hipmr_tv = hipmr_neutral;
    const bool hipmr_in_head = hipmr_lane < hipmr_hend - hipmr_tstart;
    const bool hipmr_in_tail = hipmr_lane < hipmr_te - hipmr_tail;
    if (hipmr_in_head) {
      const hipmr_idx i = (hipmr_idx)(hipmr_tstart + hipmr_lane);
      hipmr_hv = (hipmr_acc)(@@MAP@@);
    }
    if (hipmr_in_tail) {
      const hipmr_idx i = (hipmr_idx)(hipmr_tail + hipmr_lane);
      hipmr_tv = (hipmr_acc)(@@MAP@@);
    }
    hipmr_acc hipmr_a[HIPMR_U];
#pragma unroll
    for (int u = 0; u < HIPMR_U; ++u) hipmr_a[u] = hipmr_neutral;
    @@DECL_PACKS@@
    const bool hipmr_full = hipmr_nch == 64LL * HIPMR_U;   // every lane has all U chunks
    if (hipmr_full) {
#pragma unroll
      for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
        const long long hipmr_off = hipmr_hend + (hipmr_lane + 64LL * hipmr_u) * HIPMR_V;
        @@LOADS@@
      }
    } else {
#pragma unroll
      for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
        const long long hipmr_c = hipmr_lane + 64 * hipmr_u;
        if (hipmr_c < hipmr_nch) {
          const long long hipmr_off = hipmr_hend + hipmr_c * HIPMR_V;
          @@LOADS@@
        }
      }
    }
    const int hipmr_tn = hipmr_t + hipmr_nwaves;
    if (hipmr_tn < hipmr_total_tiles) {
      hipmr_s = hipmr_find(hipmr_tn);
      hipmr_oa = hipmr_offsets[hipmr_s];
      hipmr_ob = hipmr_offsets[hipmr_s + 1];
    }
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_c = hipmr_lane + 64 * hipmr_u;
      if (hipmr_full || hipmr_c < hipmr_nch) {
        const long long hipmr_off = hipmr_hend + hipmr_c * HIPMR_V;
#pragma unroll
        for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
          const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
          hipmr_a[hipmr_u] = hipmr_combine(hipmr_a[hipmr_u], (hipmr_acc)(@@VMAP@@));
        }
      }
    }
    // the head joins on the left of the body it precedes (combined only
    // now, so that no wait for its load comes before the body's loads)
    if (hipmr_in_head) hipmr_a[0] = hipmr_combine(hipmr_hv, hipmr_a[0]);
    if (hipmr_in_tail) hipmr_a[HIPMR_U - 1] = hipmr_combine(hipmr_a[HIPMR_U - 1], hipmr_tv);
    hipmr_acc hipmr_r = hipmr_fold<HIPMR_U>(hipmr_a);
    hipmr_r = hipmr_wave_total(hipmr_r, hipmr_neutral, hipmr_lane);
    if (hipmr_lane == 63) hipmr_tpart[hipmr_t] = hipmr_r;
  }
}
)HIP";

// Stage 2: one wave per segment folds its tile partials in tile order.
const char* kSegS2 = R"HIP(
extern "C" __global__ void __launch_bounds__(@@BLOCK@@)
@@KNAME@@(const int* __restrict__ hipmr_tile_start, int hipmr_nseg,
          const hipmr_acc* __restrict__ hipmr_tpart, hipmr_acc* __restrict__ hipmr_out,
          long long hipmr_cap)
{
  const int s = blockIdx.x * (@@BLOCK@@ / 64) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (s >= hipmr_nseg) return;                  // whole waves only
  const hipmr_acc hipmr_neutral = (hipmr_acc)(@@NEUTRAL@@);
  hipmr_acc r = hipmr_neutral;
  const int t1 = hipmr_tile_start[s + 1] < hipmr_cap ? hipmr_tile_start[s + 1] : (int)hipmr_cap;
  // lane order t, t + 64, t + 128, ...; eight loads in flight per round
  for (int t = hipmr_tile_start[s] + lane; t < t1; t += 64 * 8) {
    hipmr_acc v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (t + 64 * k < t1) v[k] = hipmr_tpart[t + 64 * k];
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (t + 64 * k < t1) r = hipmr_combine(r, v[k]);
  }
  r = hipmr_block_reduce<64>(r, hipmr_neutral);
  if (lane == 0) hipmr_out[s] = r;
}
)HIP";

// Data-parallel-primitive (DPP) lane moves and the inclusive wave scan built
// from them (shared by the segmented and scan kernels).
const char* kDppHelpers = R"HIP(
// DPP lane moves on 32-bit halves: lanes whose source lies outside the
// pattern (or whose row is masked off) receive `fill`.
template <int CTRL, int ROWS, typename T>
__device__ __forceinline__ T hipmr_dpp(T v, T fill) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(
        __builtin_bit_cast(int, fill), __builtin_bit_cast(int, v), CTRL, ROWS, 0xf, false));
  } else {
    const unsigned long long a = __builtin_bit_cast(unsigned long long, v);
    const unsigned long long f = __builtin_bit_cast(unsigned long long, fill);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)f, (int)(unsigned)a, CTRL, ROWS, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)(f >> 32), (int)(unsigned)(a >> 32),
                                                              CTRL, ROWS, 0xf, false);
    return __builtin_bit_cast(T, ((unsigned long long)hi << 32) | lo);
  }
}

// inclusive scan across the wave of a 4- or 8-byte value under op (lane l
// receives v_0 op ... op v_l, the earlier lanes always on the left): shifts
// by 1, 2, 4, 8 inside each row of 16 lanes, then the totals of row 0 /
// rows 0-1 broadcast into the rows after them; e is op's neutral element
template <typename T, typename Op>
__device__ __forceinline__ T hipmr_dpp_scan(T v, T e, Op op) {
  v = op(hipmr_dpp<0x111, 0xf>(v, e), v);     // row_shr:1
  v = op(hipmr_dpp<0x112, 0xf>(v, e), v);     // row_shr:2
  v = op(hipmr_dpp<0x114, 0xf>(v, e), v);     // row_shr:4
  v = op(hipmr_dpp<0x118, 0xf>(v, e), v);     // row_shr:8
  v = op(hipmr_dpp<0x142, 0xa>(v, e), v);     // row_bcast:15 into rows 1, 3
  v = op(hipmr_dpp<0x143, 0xc>(v, e), v);     // row_bcast:31 into rows 2, 3
  return v;
}
)HIP";

// ------------------------------------------------------------ prefix scan
// The array is cut into tiles of B threads x U sub-tiles x V elements; wave w
// of a tile owns U consecutive sub-tiles of 64 V elements, lane l the V
// consecutive elements at V l of each.  A tile stays in registers between
// its load and its stores.  What the tile needs from outside is the fold of
// everything before it; MODE says where that comes from:
//   0  nothing precedes it (one tile in all);
//   1  (no outputs) the tile's total goes to partial[tile];
//   2  the tile folds partial[0 .. tile) of a MODE 1 launch itself;
//   3  one launch: tiles publish their totals and read their predecessors'.
// Every combination's order is a fixed function of n and the geometry in
// every mode (the tree below does not depend on which tile ran first).
// Bound: HBM, 8 bytes per element for float -> float (MODE 3).  A
// reduce-then-scan over wave ranges (four launches, input read twice) took
// 516 us at n = 2^28 float and 16.4 us per call at 100,003 int32 -> int64;
// MODE 3 takes 360 us (5.97 TB/s), MODE 1 + 2 10.4 us.
const char* kScanHelpers = R"HIP(
// inclusive scan across the wave (lane l receives v_0 (+) ... (+) v_l)
__device__ __forceinline__ hipmr_acc hipmr_wave_scan(hipmr_acc v, hipmr_acc e) {
  return hipmr_dpp_scan(v, e, [](hipmr_acc a, hipmr_acc b) { return hipmr_combine(a, b); });
}

// a 4- or 8-byte value as the low bits of a 64-bit word, and back
typedef unsigned long long hipmr_u64;
template <typename T> __device__ __forceinline__ hipmr_u64 hipmr_to_bits(T v) {
  if constexpr (sizeof(T) == 4) return __builtin_bit_cast(unsigned, v);
  else return __builtin_bit_cast(hipmr_u64, v);
}
template <typename T> __device__ __forceinline__ T hipmr_from_bits(hipmr_u64 b) {
  if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, (unsigned)b);
  else return __builtin_bit_cast(T, b);
}

// lane l's value (l the same in every lane), without an LDS round trip
__device__ __forceinline__ hipmr_acc hipmr_lane_value(hipmr_acc v, int l) {
  const hipmr_u64 a = hipmr_to_bits(v);
  hipmr_u64 r = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)a, l);
  if constexpr (sizeof(hipmr_acc) == 8)
    r |= (hipmr_u64)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)(a >> 32), l) << 32;
  return hipmr_from_bits<hipmr_acc>(r);
}

// Published totals (MODE 3).  A 4-byte total is one 64-bit word, value | 1 << 32
// (3 << 32: built on a total that never came); an 8-byte total two such words,
// so a single 64-bit load tells whether a word is there and what it holds, and
// no fence is needed.  Accesses are
// device-scope (the L2s of the eight dies are not coherent otherwise).  Word 0
// counts tickets, word 1 is set when a wait has been given up; words 2 and 3
// carry the fold of all before from one launch to the next where a workspace
// holds the totals of a part of the tiles at a time (the launches take turns),
// word 4 whether it is known.
constexpr int HIPMR_S = (int)sizeof(hipmr_acc) / 4, HIPMR_STATE0 = 16;

__device__ __forceinline__ hipmr_u64 hipmr_peek(const hipmr_u64* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void hipmr_publish(hipmr_u64* p, hipmr_acc v, bool lost) {
  const hipmr_u64 a = hipmr_to_bits(v), there = (lost ? 3ull : 1ull) << 32;
  __hip_atomic_store(p, there | (unsigned)a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if constexpr (HIPMR_S == 2)
    __hip_atomic_store(p + 1, there | (a >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
struct hipmr_slot { hipmr_u64 w0, w1; };
__device__ __forceinline__ hipmr_slot hipmr_first_look(const hipmr_u64* p, bool mine) {
  hipmr_slot s = {1ull << 32, 1ull << 32};
  if (mine) {
    s.w0 = hipmr_peek(p);
    if constexpr (HIPMR_S == 2) s.w1 = hipmr_peek(p + 1);
  }
  return s;
}
// The fold, in lane order, of the totals the lanes wait for (lanes with
// mine = false hold the neutral element); every lane receives it.  The waits
// end: a total is published by a tile with an earlier ticket, whose block is
// already running and itself waits for still earlier ones only.  So the limit
// (a number of polls, some seconds of them, or another wave's expiry) is
// reached only if something else writes the workspace while the scan runs, or
// if the call asked for no wait; `lost` then tells the tile and, through the
// totals built on it, all later ones that their sums are not known.
struct hipmr_wait { hipmr_u64* state; unsigned limit; bool lost; };
__device__ __forceinline__ hipmr_acc hipmr_await_fold(const hipmr_u64* p, bool mine, hipmr_slot s,
                                                      hipmr_acc e, hipmr_wait& wait) {
  unsigned polls = 0;
  while (__ballot(!((s.w0 >> 32) && (s.w1 >> 32)))) {
    if (++polls >= wait.limit || ((polls & 63u) == 0 && hipmr_peek(wait.state + 1))) {
      __hip_atomic_store(wait.state + 1, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      wait.lost = true;
      break;
    }
    __builtin_amdgcn_s_sleep(16);                    // 1024 clocks: fewer polls beside the ticket atomics
    if (!(s.w0 >> 32)) s.w0 = hipmr_peek(p);
    if constexpr (HIPMR_S == 2) { if (!(s.w1 >> 32)) s.w1 = hipmr_peek(p + 1); }
  }
  if (__ballot((s.w0 >> 33) || (s.w1 >> 33))) wait.lost = true;
  hipmr_acc v = e;
  if (mine) v = hipmr_from_bits<hipmr_acc>(HIPMR_S == 1 ? s.w0 & 0xffffffffull : (s.w1 << 32) | (s.w0 & 0xffffffffull));
  return hipmr_lane_value(hipmr_wave_scan(v, e), 63);
}

// The fold of every tile before `tile`, by one wave (MODE 3), after it has
// published the tile's own total.  Tiles form groups of 64 and groups of 64
// groups; the last tile of a group publishes the group's total, and the last
// of a supergroup that one's, so three short folds reach any distance:
// earlier tiles of the group, earlier groups of the supergroup, earlier
// supergroups (64 per round).
__device__ __forceinline__ hipmr_acc hipmr_before(int tile, int tiles, hipmr_acc own, hipmr_wait& wait,
                                                  hipmr_acc e, int lane) {
  hipmr_u64* const state = wait.state;
  const int g = tile >> 6, r = tile & 63, h = g >> 6, q = g & 63;
  hipmr_u64* const pt = state + HIPMR_STATE0;
  hipmr_u64* const pg = pt + (long long)tiles * HIPMR_S;
  hipmr_u64* const ph = pg + (long long)((tiles + 63) >> 6) * HIPMR_S;
  if (lane == 0) hipmr_publish(pt + (long long)tile * HIPMR_S, own, false);
  const hipmr_u64* const at = pt + ((long long)(tile - r) + lane) * HIPMR_S;
  const hipmr_u64* const ag = pg + ((long long)(g - q) + lane) * HIPMR_S;
  const hipmr_u64* ah = ph + (long long)lane * HIPMR_S;
  const hipmr_slot st = hipmr_first_look(at, lane < r);
  const hipmr_slot sg = hipmr_first_look(ag, lane < q);
  hipmr_slot sh = hipmr_first_look(ah, lane < h);
  const hipmr_acc ft = hipmr_await_fold(at, lane < r, st, e, wait);
  if (r == 63 && lane == 0) hipmr_publish(pg + (long long)g * HIPMR_S, hipmr_combine(ft, own), wait.lost);
  const hipmr_acc fg = hipmr_await_fold(ag, lane < q, sg, e, wait);
  if (r == 63 && q == 63 && lane == 0)
    hipmr_publish(ph + (long long)h * HIPMR_S, hipmr_combine(fg, hipmr_combine(ft, own)), wait.lost);
  hipmr_acc fh = hipmr_await_fold(ah, lane < h, sh, e, wait);
  for (int k = 64; k < h; k += 64) {
    ah += 64 * HIPMR_S;
    sh = hipmr_first_look(ah, lane < h - k);
    fh = hipmr_combine(fh, hipmr_await_fold(ah, lane < h - k, sh, e, wait));
  }
  return hipmr_combine(fh, hipmr_combine(fg, ft));
}

// what an output whose sum is not known holds: NaN where the type has one
template <typename T> __device__ __forceinline__ T hipmr_unknown() {
  if constexpr (__is_same(T, float)) return __builtin_nanf("");
  else if constexpr (__is_same(T, double)) return __builtin_nan("");
  else if constexpr (__is_same(T, hipmr_c64)) return T(__builtin_nanf(""), __builtin_nanf(""));
  else return T(0);
}
)HIP";

// Clears the ticket counter and the published totals of a MODE 3 launch (not
// what the launch before it handed on).
const char* kScanClear = R"HIP(
extern "C" __global__ void __launch_bounds__(256)
@@KNAME@@(unsigned long long* __restrict__ hipmr_state, int hipmr_words)
{
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k < hipmr_words && (k < 2 || k > 4)) hipmr_state[k] = 0ull;
}
)HIP";

const char* kScanTile = R"HIP(
extern "C" __global__ void __launch_bounds__(@@BLOCK@@)
@@KNAME@@(@@PARAMS@@, long long hipmr_n, long long hipmr_base, int hipmr_tiles,
          void* __restrict__ hipmr_state, hipmr_acc* __restrict__ hipmr_out, int hipmr_flags,
          unsigned* __restrict__ hipmr_gave_up)
{
  // bit 1: no wait; bits 2 and 3: a launch went before, one comes after; bit 4: its turn
  const bool hipmr_exclusive = hipmr_flags & 1;
  typedef @@IDX@@ hipmr_idx;
  constexpr int HIPMR_B = @@BLOCK@@, HIPMR_U = @@IPT@@, HIPMR_V = @@VEC@@, HIPMR_MODE = @@MODE@@;
  constexpr int HIPMR_W = HIPMR_B / 64;
  constexpr bool HIPMR_NTL = @@NTL@@, HIPMR_NTS = @@NTS@@;
  constexpr long long HIPMR_SUB = 64LL * HIPMR_V, HIPMR_TILE = HIPMR_SUB * HIPMR_U * HIPMR_W;
  const hipmr_idx n = (hipmr_idx)hipmr_n;
  const hipmr_acc hipmr_neutral = (hipmr_acc)(@@NEUTRAL@@);
  const int hipmr_lane = threadIdx.x & 63;
  const int hipmr_w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  int hipmr_tile = blockIdx.x;
  if constexpr (HIPMR_MODE == 3) {
    // tiles are taken in ticket order: a tile's predecessors are running or done
    __shared__ int hipmr_ticket;
    if (threadIdx.x == 0)
      hipmr_ticket = (int)__hip_atomic_fetch_add((unsigned*)hipmr_state, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    hipmr_tile = __builtin_amdgcn_readfirstlane(hipmr_ticket);
    if (hipmr_tile < 0) return;
  }
  if (hipmr_tile >= hipmr_tiles) return;
  // base may be negative (the first aligned chunk starts before element 0):
  // chunks that are not wholly inside [0, n) go element by element
  const long long hipmr_b0 = hipmr_base + (long long)hipmr_tile * HIPMR_TILE;
  const bool hipmr_whole = hipmr_b0 >= 0 && hipmr_b0 + HIPMR_TILE <= hipmr_n;
  const long long hipmr_l0 = hipmr_b0 + hipmr_w * (HIPMR_SUB * HIPMR_U) + (long long)hipmr_lane * HIPMR_V;
  hipmr_pack<hipmr_acc, HIPMR_V> hipmr_t[HIPMR_U];   // mapped values, then the lane's inclusive prefixes
  @@DECL_PACKS@@
  if (hipmr_whole) {
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_off = hipmr_l0 + hipmr_u * HIPMR_SUB;
      @@LOADS@@
    }
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_off = hipmr_l0 + hipmr_u * HIPMR_SUB;
#pragma unroll
      for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
        const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
        hipmr_t[hipmr_u].v[hipmr_j] = (hipmr_acc)(@@VMAPX@@);
      }
    }
  } else {
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_off = hipmr_l0 + hipmr_u * HIPMR_SUB;
      if (hipmr_off >= 0 && hipmr_off + HIPMR_V <= hipmr_n) {
        @@LOADS@@
      }
    }
#pragma unroll
    for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
      const long long hipmr_off = hipmr_l0 + hipmr_u * HIPMR_SUB;
      const bool hipmr_full = hipmr_off >= 0 && hipmr_off + HIPMR_V <= hipmr_n;
#pragma unroll
      for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
        hipmr_acc hipmr_m = hipmr_neutral;
        const hipmr_idx i = (hipmr_idx)(hipmr_off + hipmr_j);
        if (hipmr_full) hipmr_m = (hipmr_acc)(@@VMAPX@@);
        else if (hipmr_off + hipmr_j >= 0 && hipmr_off + hipmr_j < hipmr_n) hipmr_m = (hipmr_acc)(@@MAP@@);
        hipmr_t[hipmr_u].v[hipmr_j] = hipmr_m;
      }
    }
  }
  // MODE 2: this thread's run of the earlier tiles' totals, in order
  hipmr_acc hipmr_pp = hipmr_neutral;
  if constexpr (HIPMR_MODE == 2) {
    const hipmr_acc* const hipmr_partial = (const hipmr_acc*)hipmr_state;
    const int hipmr_run = (hipmr_tile + HIPMR_B - 1) / HIPMR_B;
    for (int k = threadIdx.x * hipmr_run; k < (int)(threadIdx.x + 1) * hipmr_run && k < hipmr_tile; ++k)
      hipmr_pp = hipmr_combine(hipmr_pp, hipmr_partial[k]);
    hipmr_pp = hipmr_wave_scan(hipmr_pp, hipmr_neutral);   // lane 63: the wave's runs
  }
  // inside the wave: lane prefixes, then each sub-tile's exclusive offset
  // (the sub-tiles' wave scans are independent; only their totals chain)
  hipmr_acc hipmr_q[HIPMR_U];
  hipmr_acc hipmr_carry = hipmr_neutral;
#pragma unroll
  for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
#pragma unroll
    for (int hipmr_j = 1; hipmr_j < HIPMR_V; ++hipmr_j)
      hipmr_t[hipmr_u].v[hipmr_j] = hipmr_combine(hipmr_t[hipmr_u].v[hipmr_j - 1], hipmr_t[hipmr_u].v[hipmr_j]);
    const hipmr_acc hipmr_x = hipmr_wave_scan(hipmr_t[hipmr_u].v[HIPMR_V - 1], hipmr_neutral);
    const hipmr_acc hipmr_up = hipmr_dpp<0x138, 0xf>(hipmr_x, hipmr_neutral);   // wave_shr:1
    const hipmr_acc hipmr_sum = hipmr_lane_value(hipmr_x, 63);
    hipmr_q[hipmr_u] = hipmr_u == 0 ? hipmr_up : hipmr_combine(hipmr_carry, hipmr_up);
    hipmr_carry = hipmr_u == 0 ? hipmr_sum : hipmr_combine(hipmr_carry, hipmr_sum);
  }
  // across the block's waves: every wave scans the wave totals itself
  __shared__ hipmr_acc hipmr_wt[HIPMR_W], hipmr_wp[HIPMR_W], hipmr_pre_lds;
  __shared__ bool hipmr_lost_lds;
  if (hipmr_lane == 63) {
    hipmr_wt[hipmr_w] = hipmr_carry;
    hipmr_wp[hipmr_w] = hipmr_pp;
  }
  __syncthreads();
  const hipmr_acc hipmr_ws = hipmr_wave_scan(hipmr_lane < HIPMR_W ? hipmr_wt[hipmr_lane] : hipmr_neutral, hipmr_neutral);
  if constexpr (HIPMR_MODE == 1) {
    if (threadIdx.x == HIPMR_W - 1) ((hipmr_acc*)hipmr_state)[hipmr_tile] = hipmr_ws;
    return;
  }
  hipmr_acc hipmr_pre = hipmr_neutral;               // the fold of every element before the tile
  if constexpr (HIPMR_MODE == 2)
    hipmr_pre = hipmr_lane_value(hipmr_wave_scan(hipmr_lane < HIPMR_W ? hipmr_wp[hipmr_lane] : hipmr_neutral,
                                                 hipmr_neutral), 63);
  if constexpr (HIPMR_MODE == 3) {
    if (hipmr_w == 0) {
      hipmr_wait hipmr_wt8 = {(hipmr_u64*)hipmr_state, hipmr_flags & 2 ? 1u : 1u << 22, false};
      const hipmr_acc hipmr_own = hipmr_lane_value(hipmr_ws, HIPMR_W - 1);
      hipmr_acc hipmr_b = hipmr_before(hipmr_tile, hipmr_tiles, hipmr_own, hipmr_wt8, hipmr_neutral, hipmr_lane);
      const int hipmr_turn = hipmr_flags >> 4 & 1;
      if (hipmr_flags & 4) {
        hipmr_b = hipmr_combine(hipmr_from_bits<hipmr_acc>(hipmr_wt8.state[3 - hipmr_turn]), hipmr_b);
        if (hipmr_wt8.state[4]) hipmr_wt8.lost = true;
      }
      if ((hipmr_flags & 8) && hipmr_tile == hipmr_tiles - 1 && hipmr_lane == 0) {
        hipmr_wt8.state[2 + hipmr_turn] = hipmr_to_bits(hipmr_combine(hipmr_b, hipmr_own));
        hipmr_wt8.state[4] = hipmr_wt8.lost;
      }
      if (hipmr_lane == 0) {
        hipmr_pre_lds = hipmr_b;
        hipmr_lost_lds = hipmr_wt8.lost;
      }
    }
    __syncthreads();
    hipmr_pre = hipmr_pre_lds;
    if (hipmr_lost_lds) {                            // said in the outputs and to the host
      if (threadIdx.x == 0 && hipmr_gave_up)
        __hip_atomic_store(hipmr_gave_up, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      for (int k = threadIdx.x; k < (int)HIPMR_TILE; k += HIPMR_B)
        if (hipmr_b0 + k >= 0 && hipmr_b0 + k < hipmr_n) hipmr_out[hipmr_b0 + k] = hipmr_unknown<hipmr_acc>();
      return;
    }
  }
  const hipmr_acc hipmr_wpre = hipmr_w == 0 ? hipmr_neutral : hipmr_lane_value(hipmr_ws, hipmr_w - 1);
#pragma unroll
  for (int hipmr_u = 0; hipmr_u < HIPMR_U; ++hipmr_u) {
    const long long hipmr_off = hipmr_l0 + hipmr_u * HIPMR_SUB;
    // the offsets inside the tile are combined first: one rounding at the
    // prefix's magnitude here, one per output
    const hipmr_acc hipmr_p = hipmr_combine(hipmr_pre, hipmr_combine(hipmr_wpre, hipmr_q[hipmr_u]));
    hipmr_pack<hipmr_acc, HIPMR_V> hipmr_o;
#pragma unroll
    for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j) {
      if (hipmr_exclusive) hipmr_o.v[hipmr_j] = hipmr_j == 0 ? hipmr_p : hipmr_combine(hipmr_p, hipmr_t[hipmr_u].v[hipmr_j > 0 ? hipmr_j - 1 : 0]);
      else hipmr_o.v[hipmr_j] = hipmr_combine(hipmr_p, hipmr_t[hipmr_u].v[hipmr_j]);
    }
    if (hipmr_whole || (hipmr_off >= 0 && hipmr_off + HIPMR_V <= hipmr_n)) {
      hipmr_store<HIPMR_NTS>(hipmr_out + hipmr_off, hipmr_o);
    } else {
#pragma unroll
      for (int hipmr_j = 0; hipmr_j < HIPMR_V; ++hipmr_j)
        if (hipmr_off + hipmr_j >= 0 && hipmr_off + hipmr_j < hipmr_n) hipmr_out[hipmr_off + hipmr_j] = hipmr_o.v[hipmr_j];
    }
  }
}
)HIP";

void replace_all(std::string& s, const std::string& key, const std::string& val) {
    size_t pos = 0;
    while ((pos = s.find(key, pos)) != std::string::npos) {
        s.replace(pos, key.size(), val);
        pos += val.size();
    }
}

// symbol tags of the scan modes (vector, one-element)
const char* const kScanTags[4][2] = {{"sc1", "sc1s"}, {"scu", "scus"}, {"scd", "scds"}, {"scl", "scls"}};

std::string combine_body(DType r, const KernelSpec& spec) {
    bool fp = r == DT_F32 || r == DT_F64;
    switch (canonical_combine(spec.combine)) {
        case Combine::Sum: return "a + b";
        case Combine::Max: return fp ? "__builtin_elementwise_maximum(a, b)" : "(a > b ? a : b)";
        case Combine::Min: return fp ? "__builtin_elementwise_minimum(a, b)" : "(a < b ? a : b)";
        default: return spec.combine;
    }
}

// What a kernel's source is made of: the helpers it needs, in order, and the
// kernel itself.
struct Source {
    std::vector<std::string> parts;
    std::string body, symbol;
};

Source render_parts(const Program& prog, const KernelSpec& spec) {
    const char* tmpl = nullptr;
    const char* tag = "";
    bool reduce = false;
    bool comp = false;       // compensated helpers
    const DType acc = prog.sig.result;
    switch (spec.kind) {
        case KernelKind::EwVector:
            tmpl = prog.info.shifts.empty() ? kEwVector : kEwVectorShift;
            tag = "ew";
            break;
        case KernelKind::EwScalar: tmpl = kEwScalar; tag = "ews"; break;
        case KernelKind::RedS1Vector:
            tmpl = prog.info.shifts.empty() ? kRedS1Vector : kRedS1VectorShift;
            tag = "rs1";
            reduce = true;
            break;
        case KernelKind::RedS1Scalar: tmpl = kRedS1Scalar; tag = "rs1s"; reduce = true; break;
        case KernelKind::RedS2: tmpl = kRedS2; tag = "rs2"; reduce = true; break;
        case KernelKind::CompS1Vector:
            tmpl = kCompS1Vector; tag = spec.track ? "nrm1" : spec.square ? "nrm2" : "csum"; comp = true; break;
        case KernelKind::CompS1Scalar:
            tmpl = kCompS1Scalar; tag = spec.track ? "nrm1s" : spec.square ? "nrm2s" : "csums"; comp = true; break;
        case KernelKind::CompS2: tmpl = kCompS2; tag = spec.norm ? "nrm2f" : "csumf"; comp = true; break;
        case KernelKind::SegPlan: tmpl = kSegPlan; tag = "segplan"; break;
        case KernelKind::SegS1: tmpl = kSegS1; tag = "seg1"; reduce = true; break;
        case KernelKind::SegS2: tmpl = kSegS2; tag = "seg2"; reduce = true; break;
        case KernelKind::ScanVector: tmpl = kScanTile; tag = kScanTags[spec.scan_mode][0]; reduce = true; break;
        case KernelKind::ScanScalar: tmpl = kScanTile; tag = kScanTags[spec.scan_mode][1]; reduce = true; break;
        case KernelKind::ScanClear: tmpl = kScanClear; tag = "scz"; break;
    }
    // the scalar scan reads its one-element chunks through the expression itself
    const bool scan_scalar = spec.kind == KernelKind::ScanScalar;
    const bool scan = spec.kind == KernelKind::ScanVector || scan_scalar;
    const bool seg = spec.kind == KernelKind::SegPlan || spec.kind == KernelKind::SegS1;
    std::string body = tmpl;

    // parameters in declaration order
    std::string params;
    for (size_t k = 0; k < prog.sig.args.size(); ++k) {
        const ArgDecl& a = prog.sig.args[k];
        if (k) params += ", ";
        if (a.pointer) {
            params += std::string(a.is_const ? "const " : "") + dtype_device_name(a.dtype) +
                      "* __restrict__ " + a.name;
        } else {
            params += std::string("const ") + dtype_device_name(a.dtype) + " " + a.name;
        }
    }
    if (params.empty()) params = "int hipmr_unused";

    std::string decl_packs, loads, stores;
    for (const ArgDecl& a : prog.sig.args) {
        if (!chunked(a)) continue;
        if (a.dtype == DT_FP8 && !a.written && spec.vec >= 4)
            decl_packs += "hipmr_pack_fp8ro<HIPMR_V> hipmr_p_" + a.name + "[HIPMR_U]; ";
        else
            decl_packs += std::string("hipmr_pack<") + dtype_device_name(a.dtype) + ", HIPMR_V> hipmr_p_" +
                          a.name + "[HIPMR_U]; ";
        if (!a.write_only)
            loads += std::string(spec.unaligned ? "hipmr_load_any" : "hipmr_load") + "<HIPMR_NTL>(hipmr_p_" + a.name + "[hipmr_u], " + a.name + " + hipmr_off); ";
        if (a.written)
            stores += "hipmr_store<HIPMR_NTS>(" + a.name + " + hipmr_off, hipmr_p_" + a.name + "[hipmr_u]); ";
    }

    // shifted reads (vector elementwise kernels): distances, packs and loads
    std::string shift_init, shift_packs, shift_loads;
    // (the other vector kernels read shifted elements directly, as written)
    const bool shifts = (spec.kind == KernelKind::EwVector || spec.kind == KernelKind::RedS1Vector) &&
                        !prog.info.shifts.empty();
    if (shifts) {
        std::string bounds = "long long hipmr_smin = 0, hipmr_smax = 0; ";
        for (size_t r = 0; r < prog.info.shifts.size(); ++r) {
            const ShiftRead& sr = prog.info.shifts[r];
            const ArgDecl& a = prog.sig.args[sr.arg];
            const std::string k = std::to_string(r);
            shift_init += "const long long hipmr_s" + k + " = (long long)" + sr.offset + "; ";
            bounds += "hipmr_smin = hipmr_s" + k + " < hipmr_smin ? hipmr_s" + k + " : hipmr_smin; ";
            bounds += "hipmr_smax = hipmr_s" + k + " > hipmr_smax ? hipmr_s" + k + " : hipmr_smax; ";
            shift_packs += std::string("hipmr_pack<") + dtype_device_name(a.dtype) + ", HIPMR_V> hipmr_q" + k +
                           "[HIPMR_U]; ";
            // the reduce kernel loads every chunk (clamped into the array);
            // the elementwise kernel loads only chunks it evaluates as vectors
            const std::string at = spec.kind == KernelKind::RedS1Vector
                                       ? "hipmr_clampv(hipmr_off, hipmr_s" + k + ", hipmr_n - HIPMR_V)"
                                       : "hipmr_off + hipmr_s" + k;
            shift_loads += "hipmr_loadu(hipmr_q" + k + "[hipmr_u], " + a.name + " + " + at + "); ";
        }
        shift_init += bounds;
    }

    std::string scalar_text = join_tokens(prog.toks);
    std::string vector_text = scan_scalar ? scalar_text
                                          : vectorize_accesses(prog.toks, prog.sig,
                                                               shifts ? prog.info.shifts : std::vector<ShiftRead>{});
    if (scan_scalar) {
        decl_packs.clear();
        loads.clear();
    }
    replace_all(body, "@@VMAPX@@", vector_text);
    replace_all(body, "@@MODE@@", std::to_string(spec.scan_mode));
    replace_all(body, "@@SHARES@@", "const unsigned hipmr_b = blockIdx.x;");
    std::string finish = std::string("if (threadIdx.x == 0) hipmr_partial[blockIdx.x] = ") +
                         (comp ? "hipmr_v;" : "hipmr_r;");
    if (spec.finish) {
        const bool vector = spec.kind == KernelKind::RedS1Vector || spec.kind == KernelKind::CompS1Vector;
        const std::string loop = "#pragma clang loop unroll(disable)\n"
                                 "  for (int hipmr_b = 0; hipmr_b < (int)gridDim.x; ++hipmr_b) {";
        if (comp) {
            finish = "if (!hipmr_comp_finish<@@BLOCK@@, HIPMR_SQ>(hipmr_v, hipmr_words, hipmr_post, (double)hipmr_sc, "
                     "hipmr_tag, hipmr_out)) return;\n  hipmr_neumaier hipmr_f = {0.0, 0.0};\n" + loop +
                     (vector ? kCompShare : kCompShareScalar) + kCompShareEnd + "  }";
        } else {
            finish = "if (!hipmr_finish<@@BLOCK@@>(hipmr_r, hipmr_neutral, (unsigned long long*)hipmr_partial, "
                     "hipmr_out, hipmr_tag)) return;\n  hipmr_acc hipmr_f = hipmr_neutral;\n" + loop +
                     (vector ? kRedShare : kRedShareScalar) +
                     "    hipmr_add_share<@@BLOCK@@>(hipmr_f, hipmr_q, hipmr_neutral, hipmr_out, hipmr_b);\n  }";
            replace_all(finish, "@@SHARE_CHUNK@@", shifts ? kRedShareChunkShift : kRedShareChunk);
            replace_all(finish, "@@SHARE_BLOCK@@", shifts ? "hipmr_xcd_block(hipmr_b)" : "hipmr_b");
        }
    }
    replace_all(body, "@@FINISH@@", finish);
    replace_all(body, "@@SHIFT_INIT@@", shift_init);
    replace_all(body, "@@SHIFT_PACKS@@", shift_packs);
    replace_all(body, "@@SHIFT_LOADS@@", shift_loads);
    replace_all(body, "@@ONE@@", spec.finish ? "true" : "false");
    replace_all(body, "@@FPARAMS@@",
                spec.finish ? ", hipmr_acc* __restrict__ hipmr_out, unsigned long long hipmr_tag" : "");
    replace_all(body, "@@PARAMS@@", params);
    replace_all(body, "@@DECL_PACKS@@", decl_packs);
    replace_all(body, "@@LOADS@@", loads);
    replace_all(body, "@@STORES@@", stores);
    replace_all(body, "@@STMT@@", scalar_text);
    replace_all(body, "@@VSTMT@@", vector_text);
    replace_all(body, "@@MAP@@", scalar_text);
    replace_all(body, "@@VMAP@@", vector_text);
    replace_all(body, "@@NEUTRAL@@", spec.neutral.empty() ? "0" : spec.neutral);
    replace_all(body, "@@SQUARE@@", spec.square ? "true" : "false");
    replace_all(body, "@@RUNS@@", spec.exact_runs ? "true" : "false");
    replace_all(body, "@@NORM@@", spec.norm ? "true" : "false");
    replace_all(body, "@@SCALED@@", spec.scaled ? "true" : "false");
    replace_all(body, "@@TRACK@@", spec.track ? "true" : "false");
    replace_all(body, "@@WORDS_AT@@", std::to_string(kNormWordsOffset / 8));
    replace_all(body, "@@SCALE_AT@@", std::to_string(kMaxPartials));
    replace_all(body, "@@WORDS_FOR@@", std::to_string(kNormWordsBlocks));
    replace_all(body, "@@LDS_SEGS@@", std::to_string(spec.lds_segs));
    replace_all(body, "@@IDX@@", spec.idx64 ? "long long" : "int");
    replace_all(body, "@@BLOCK@@", std::to_string(spec.block));
    replace_all(body, "@@IPT@@", std::to_string(spec.ipt));
    replace_all(body, "@@VEC@@", std::to_string(spec.vec));
    replace_all(body, "@@NTL@@", spec.nt_loads ? "true" : "false");
    replace_all(body, "@@NTS@@", spec.nt_stores ? "true" : "false");

    Source src;
    std::vector<std::string>& parts = src.parts;
    parts.push_back(kPrelude);
    if (reduce) {
        parts.push_back(std::string("typedef ") + dtype_device_name(acc) + " hipmr_acc;\n"
                        "__device__ __forceinline__ hipmr_acc hipmr_combine(hipmr_acc a, hipmr_acc b) "
                        "{ return (hipmr_acc)(" + combine_body(acc, spec) + "); }\n");
        parts.push_back(kReduceHelpers);
        if (spec.finish) parts.insert(parts.end(), {kTagged, kRedFinish});
    }
    if (comp) parts.insert(parts.end(), {kTagged, kCompHelpers});
    if (seg || scan) parts.push_back(kDppHelpers);
    if (seg) parts.push_back(kSegHelpers);
    if (spec.kind == KernelKind::SegS1) parts.push_back(kSegFold);
    if (scan) parts.push_back(kScanHelpers);
    if (shifts) parts.push_back(kShiftHelpers);
    if (spec.unaligned) parts.push_back(kUnalignedHelpers);
    // the symbol carries a hash of the whole source (prelude and helpers
    // included), so any change to the generated code renames the kernel
    std::string text;
    for (const std::string& p : parts) text += p;
    text += body;
    src.symbol = prog.name + "_" + tag + "_" + sha256_hex(text.data(), text.size()).substr(0, 8);
    replace_all(body, "@@KNAME@@", src.symbol);
    src.body = "// generated by hipmr: " + std::string(tag) + " kernel of \"" + prog.name + "\"\n" + body;
    return src;
}

}  // namespace

std::string render(const Program& prog, const std::vector<KernelSpec>& specs, std::vector<std::string>* symbols) {
    std::vector<std::string> parts;
    std::string bodies;
    symbols->clear();
    for (const KernelSpec& spec : specs) {
        Source s = render_parts(prog, spec);
        for (std::string& p : s.parts)       // a helper needs only helpers that every kernel with it names before it
            if (std::find(parts.begin(), parts.end(), p) == parts.end()) parts.push_back(std::move(p));
        symbols->push_back(s.symbol);
        bodies += s.body;
    }
    std::string text;
    for (const std::string& p : parts) text += p;
    return text + bodies;
}

const char* device_prelude() { return kPrelude; }

}  // namespace hipmr
