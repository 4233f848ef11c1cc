// Shared host/device helpers of the routed-LoRA library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/milora.h"

namespace milora {

// ---- host-side error plumbing -------------------------------------------------------------------
extern thread_local int g_last_hip_error;

inline int hip_fail(hipError_t e) {
  g_last_hip_error = (int)e;
  return MILORA_EHIP;
}

#define MILORA_HIP(call)                              \
  do {                                                \
    hipError_t e__ = (call);                          \
    if (e__ != hipSuccess) return milora::hip_fail(e__); \
  } while (0)

inline int check_launch() {
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? MILORA_OK : hip_fail(e);
}

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Input and output width of the linear at `site` (Sec. 3.1 of the paper).
inline void site_dims(int site, int d, int F, int* d1, int* d2) {
  *d1 = (site == 6) ? F : d;
  *d2 = (site == 4 || site == 5) ? F : d;
}

// ---- device-side scalar conversions -------------------------------------------------------------
typedef uint16_t bf16_t;  // raw bits

__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float((uint32_t)v << 16); }

// Round-to-nearest-even; NaN stays NaN: the chip's conversion of two values, whose bits are those of the rounding by integer
// arithmetic for all 2^32 inputs, in one instruction instead of fourteen (a wave issues one every four cycles or more, and a
// wave of the 256 x 256 tiles rounds 256 values per lane: seven linears of 32768 rows 11.68 -> 11.42 ms, of 777 rows 504 -> 488 us).
typedef __bf16 cvt_bf16x2 __attribute__((ext_vector_type(2)));
typedef float cvt_f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(cvt_f32x2{lo, hi}, cvt_bf16x2));
}
__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }

typedef float f32x4 __attribute__((ext_vector_type(4)));

// 16-byte stores of data another workgroup reads inside this launch: written through to the memory all XCDs
// share (a plain store may stay in the writer's L2 until the launch ends).  The two idle cycles behind the store
// belong to it: a store of more than eight bytes still reads its data registers for two cycles after it issues,
// the compiler keeps vector writes away from them only for stores it can see, and it reuses these registers at
// once (seen: the next store's address computed into them, and address bits arriving as partial sums).
__device__ __forceinline__ void st_through(f32x4* p, f32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
}
// Eight 16-byte loads that bypass the caches (data written by other workgroups in this launch, into memory that
// earlier levels and launches have used), complete when the function returns.
__device__ __forceinline__ void ld_through8(const f32x4* const (&q)[8], f32x4 (&v)[8]) {
  asm volatile(
      "global_load_dwordx4 %0, %8, off sc0 sc1\n\t"
      "global_load_dwordx4 %1, %9, off sc0 sc1\n\t"
      "global_load_dwordx4 %2, %10, off sc0 sc1\n\t"
      "global_load_dwordx4 %3, %11, off sc0 sc1\n\t"
      "global_load_dwordx4 %4, %12, off sc0 sc1\n\t"
      "global_load_dwordx4 %5, %13, off sc0 sc1\n\t"
      "global_load_dwordx4 %6, %14, off sc0 sc1\n\t"
      "global_load_dwordx4 %7, %15, off sc0 sc1\n\t"
      "s_waitcnt vmcnt(0)"
      : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
      : "v"(q[0]), "v"(q[1]), "v"(q[2]), "v"(q[3]), "v"(q[4]), "v"(q[5]), "v"(q[6]), "v"(q[7])
      : "memory");
}
// 16 bytes per lane from base + voff (global) to LDS at dst + lane * 16, asynchronously; counted by vmcnt.
// Written as assembly so that the compiler does not order its own LDS reads behind the copy.
__device__ __forceinline__ void copy_to_lds16(const void* base, uint32_t voff, uint32_t dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(dst), "v"(voff), "s"(base)
               : "memory");
}

template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int kDtype = MILORA_F32;
  __device__ static __forceinline__ float load(const float* p, size_t i) { return p[i]; }
  __device__ static __forceinline__ void store(float* p, size_t i, float v) { p[i] = v; }
};
template <> struct Elem<bf16_t> {
  static constexpr int kDtype = MILORA_BF16;
  __device__ static __forceinline__ float load(const bf16_t* p, size_t i) { return bf16_to_f32(p[i]); }
  __device__ static __forceinline__ void store(bf16_t* p, size_t i, float v) { p[i] = f32_to_bf16(v); }
};

inline size_t dtype_size(int dtype) { return dtype == MILORA_BF16 ? 2 : 4; }

__device__ __forceinline__ float silu(float g) { return g / (1.0f + __expf(-g)); }

// Device view of the per-tenant adapter tables of one layer.
struct AdapterView {
  const int32_t* rank;
  const void* const* A;
  const void* const* B;
  int n_tenants;
  int r_max;
};

inline AdapterView view_of(const milora_adapters* a) {
  return AdapterView{a->rank, a->A, a->B, a->n_tenants, a->r_max};
}

// Does a route byte select `site`?  0..6 name one site, 0x80 | mask a set of sites (bit m = site m), 255 none.
__host__ __device__ __forceinline__ bool route_has(uint8_t route, int site) {
  if (route < MILORA_NUM_SITES) return route == site;
  if (route == MILORA_ROUTE_NONE || !(route & 0x80)) return false;
  return ((route >> site) & 1) != 0;
}

// Rank of the LoRA term of request `b` at `site`, or 0 when the request carries none there
// (not routed to the site, or an id out of range).
__device__ __forceinline__ int routed_rank(const AdapterView& ad, const int32_t* tenant_id, const uint8_t* route,
                                           int b, int B, int site, int* tenant) {
  if (b < 0 || b >= B || !route_has(route[b], site)) return 0;
  int t = tenant_id[b];
  if (t < 0 || t >= ad.n_tenants) return 0;
  int r = ad.rank[t];
  if (r < 1 || r > ad.r_max) return 0;
  *tenant = t;
  return r;
}

// Optional per-launch event marks of the packed layer path (measurement only).
struct LaunchMarks {
  hipEvent_t* ev;
  int n;
  long long* trace = nullptr;  // device buffer for the kernels' own time stamps (tracing launch), or null
  int grid = 0, stages = 0;    // filled in by a tracing launch: workgroups and stages it ran
};

// The matrix-core LoRA shrink: few rows in blocks of 16 (rows of many tenants then meet in few workgroups), many in blocks
// of 64 (W^A is read less often); its reduction is cut into parts, one workgroup each, so that some 512 workgroups of
// eight waves are there and no wave is without a chunk.  The workspace holds one [M][r_max] fp32 array per part.
constexpr int kShrinkChunkK = 128;
constexpr int64_t kTileMaxRows = 4096;  // rows of one launch of the tile kernel
inline int shrink_parts(int64_t M, int d1) {
  const int64_t blocks = M <= kTileMaxRows ? (M + 15) / 16 : (M + 63) / 64;
  const int most = (d1 + 8 * kShrinkChunkK - 1) / (8 * kShrinkChunkK);
  int parts = 1;
  while (parts < 8 && parts * 2 <= most && blocks * parts * 2 <= 512) parts *= 2;
  return parts;
}

// The most rows x parts over all calls of up to M rows and d1 inputs (a call of more than one part has at most 512 blocks x parts).
inline size_t shrink_rows_bound(int64_t M, int d1) {
  const int most = (d1 + 8 * kShrinkChunkK - 1) / (8 * kShrinkChunkK);
  int parts = 1;
  while (parts < 8 && parts * 2 <= most) parts *= 2;
  const int64_t cut = M * parts, cap = 512 * (M <= kTileMaxRows ? 16 : 64);
  const int64_t n = parts > 1 && cut < cap ? cut : cap;
  return (size_t)(parts == 1 || n < M ? M : n);
}

// ---- internal entry points shared between translation units ------------------------------------
// LoRA shrink in fp32: for every row m whose request is routed to site `site + i`, i < sites, t[i][m][0..r) = X[m] . A.
// X has rows of ldx elements, t is [sites][M][r_max] floats; rows that carry no LoRA term are left untouched.
int launch_shrink(const void* X, int64_t ldx, int64_t M, int d1, int dtype, const int32_t* row_to_req, const AdapterView& ad,
                  int site, int sites, const int32_t* tenant_id, const uint8_t* route, int B, float* t, hipStream_t stream);

// Any-shape linear with the LoRA term added before the single rounding:
// Y[m] = X[m] W + bias + (X[m] A) B for routed rows.  W row-major [d2][d1]; t: scratch of [M][r_max] floats.
int launch_linear_generic(const void* X, int64_t M, int d1, int d2, int dtype, const int32_t* row_to_req,
                          const void* W, const void* bias, const AdapterView& ad, int site,
                          const int32_t* tenant_id, const uint8_t* route, int B, float* t, void* Y, hipStream_t stream);

// The same for up to kFewRows rows, with the glue of a layer's decode step in its store.
constexpr int kFewRows = 16;
constexpr int kFuseRank = 16;  // the largest rank that can be shrunk inside the launch
enum FewMode {
  kFewPlain,   // Y[i] = the linear at site[i], i < sites
  kFewResid,   // h = x_res + linear (fp32); Y[0] = h rounded, if given
  kFewGateUp,  // Y[0] = silu(linear at site[0]) * linear at site[1]
  kFewDown,    // Y[0] = h + linear
};
struct FewArgs {
  const void* X;  // M rows of ldx elements
  int64_t ldx;
  int M, d1, d2;
  const void* W[3];
  const void* bias;
  void* Y[3];     // rows of ldy elements
  int64_t ldy;
  int site[3];    // consecutive
  const int32_t* row_to_req;
  const int32_t* tenant_id;
  const uint8_t* route;
  int B;
  AdapterView ad;
  const void* x_res;
  float* h;
  const float* t;  // filled in by the launch
  int col0;        // first column of the launch, the same
};
// t: scratch of [sites][M][r_max] floats
int launch_few_rows(const FewArgs& args, int dtype, int sites, int mode, float* t, hipStream_t stream);

}  // namespace milora
