// Prompt-aware LoRA router of one layer (paper Sec. 3.3): pooler (Eq. 2 and the pooler list of Sec. 3.3:
// last token, average, max, self-attention of App. C), activation g (fixed functions or the rational form of
// Sec. 3.4), router linear and top-k selection (Eq. 3).  Last-token, average and max pooling run with the router
// in one kernel (one HBM pass over H, the finish inside the same launch); the self-attention pooler is one pass that leaves
// partial rows, and a launch that merges them and finishes the same way.
// Pooled state, activation and logits stay in fp32; every sum runs in a fixed order, so the
// same prompt always yields the same route.
#include <atomic>

#include "common.h"

namespace milora {

namespace {

constexpr int kMaxSplits = 128;  // token slices per request at most

typedef uint32_t raw_u32x4 __attribute__((ext_vector_type(4)));

template <typename T, int VEC> struct VecLoad;
template <> struct VecLoad<bf16_t, 8> {
  __device__ static __forceinline__ void load(const bf16_t* p, float* out) {
    uint4 v = *reinterpret_cast<const uint4*>(p);
    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      out[2 * i] = __uint_as_float(w[i] << 16);
      out[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  // the same for data that is read once (no cache line kept for it)
  __device__ static __forceinline__ void load_once(const bf16_t* p, float* out) {
    const raw_u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const raw_u32x4*>(p));
    uint32_t w[4] = {v[0], v[1], v[2], v[3]};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      out[2 * i] = __uint_as_float(w[i] << 16);
      out[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
};
template <> struct VecLoad<float, 4> {
  __device__ static __forceinline__ void load(const float* p, float* out) {
    float4 v = *reinterpret_cast<const float4*>(p);
    out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w;
  }
  __device__ static __forceinline__ void load_once(const float* p, float* out) {
    const raw_u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const raw_u32x4*>(p));
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = __uint_as_float(v[i]);
  }
};
template <typename T> struct VecLoad<T, 1> {
  __device__ static __forceinline__ void load(const T* p, float* out) { out[0] = Elem<T>::load(p, 0); }
  __device__ static __forceinline__ void load_once(const T* p, float* out) { out[0] = Elem<T>::load(p, 0); }
};

__device__ __forceinline__ bool span_ok(int64_t start, int64_t n, int64_t M_tok) {
  return n >= 1 && start >= 0 && start + n <= M_tok;
}

// Coefficients of the rational activation Ra(x) = (a_0 + a_1 x + ... + a_6 x^6) / (1 + |b_1 x + ... + b_5 x^5|)
// (Sec. 3.4); passed by value.
struct RationalCoef {
  float a[7];
  float b[5];
};

// g of four columns.  One function at a time for all four: a wave jumps once to the code it needs and runs straight through it.
__device__ __forceinline__ void activate4(float (&x)[4], int act, const RationalCoef& rc) {
  switch (act) {
    case MILORA_ACT_TANH:
#pragma unroll 1
      for (int i = 0; i < 4; ++i) {  // (one copy of the code: the values go round)
        const float t = tanhf(x[0]);
        x[0] = x[1]; x[1] = x[2]; x[2] = x[3]; x[3] = t;
      }
      break;
    case MILORA_ACT_RELU:
#pragma unroll
      for (int v = 0; v < 4; ++v) x[v] = x[v] > 0.f ? x[v] : 0.f;
      break;
    case MILORA_ACT_GELU:
#pragma unroll 1
      for (int i = 0; i < 4; ++i) {
        const float t = 0.5f * x[0] * (1.0f + erff(x[0] * 0.70710678118654752440f));
        x[0] = x[1]; x[1] = x[2]; x[2] = x[3]; x[3] = t;
      }
      break;
    case MILORA_ACT_RATIONAL:
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float num = rc.a[6], den = rc.b[4];
#pragma unroll
        for (int j = 5; j >= 0; --j) num = num * x[v] + rc.a[j];
#pragma unroll
        for (int j = 3; j >= 0; --j) den = den * x[v] + rc.b[j];
        x[v] = num / (1.0f + fabsf(den * x[v]));
      }
      break;
    default: break;
  }
}

// The top_k largest logits as a route byte, an exact tie going to the lower index.
__device__ __forceinline__ uint8_t select_route(const float (&logit)[MILORA_NUM_SITES], int top_k) {
  unsigned mask = 0;
  int last = 0;
#pragma unroll 1
  for (int q = 0; q < top_k; ++q) {
    int best = -1;
    float most = 0.f;
#pragma unroll
    for (int j = 0; j < MILORA_NUM_SITES; ++j)
      if (!((mask >> j) & 1) && (best < 0 || logit[j] > most)) {
        best = j;
        most = logit[j];
      }
    mask |= 1u << best;
    last = best;
  }
  return top_k == 1 ? (uint8_t)last : (uint8_t)(0x80u | mask);
}

// ---- last-token, average and max pooling with the router behind them: one kernel ---------------------------------
// A workgroup of 512 threads pools one slab of 32 * VEC columns over one slice of a request's valid tokens (32
// column lanes by 16 token lanes: half a wave covers 32 * VEC contiguous elements of one row).  Its first wave
// finishes: g and the slab's share of the seven logits, stored as four 16-byte units that each carry the call's
// 64-bit tag; the wave then loads the units of all the request's slabs and, if every tag is there, adds the
// shares in slab order and selects.  The wave whose units reach memory last sees all of them; a second wave that
// sees them too computes the same bytes.  Slices that cut a prompt (few, long prompts) hand their slab sums
// through memory the same way, behind one tagged flag per slice, and the wave that sees all flags adds them in
// slice order.  Every sum has a fixed order, so the same prompt always yields the same route, whichever wave
// finishes.  The workspace needs no preparation: a tag is unique to the call, and the finishing wave wipes the tags
// it has used (a recorded launch that is replayed meets wiped tags again).
// Data another workgroup reads inside the launch is stored through to memory and loaded past the caches (an
// L2 serves one XCD only); a store is acknowledged before anything that tells of it is read.  (A 16-byte store
// reads its data registers for two more cycles after it issues, and the compiler guards only stores it can see:
// the idle cycles are part of the statement.)
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void st_through(f32x4* p, f32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void st_through(u32x4* p, u32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void st_through(u32x2* p, u32x2 v) {
  asm volatile("global_store_dwordx2 %0, %1, off sc0 sc1" : : "v"(p), "v"(v) : "memory");
}
// Loads past the caches, complete when the function returns.
__device__ __forceinline__ u32x4 ld_through(const u32x4* p) {
  u32x4 v;
  asm volatile("global_load_dwordx4 %0, %1, off sc0 sc1\n\ts_waitcnt vmcnt(0)" : "=&v"(v) : "v"(p) : "memory");
  return v;
}
__device__ __forceinline__ u32x2 ld_through(const u32x2* p) {
  u32x2 v;
  asm volatile("global_load_dwordx2 %0, %1, off sc0 sc1\n\ts_waitcnt vmcnt(0)" : "=&v"(v) : "v"(p) : "memory");
  return v;
}
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
__device__ __forceinline__ void wait_all_mem() { __builtin_amdgcn_s_waitcnt(0); }

constexpr int kPoolThreads = 512;
constexpr int kColLanes = 32;
constexpr int kTokenLanes = kPoolThreads / kColLanes;

template <typename T> struct alignas(4 * sizeof(T)) Four { T v[4]; };

template <typename T>
struct PoolRouteArgs {
  const T* H;
  int64_t M_tok;
  int d;
  const int32_t* seq_start;
  const int32_t* seq_len;
  const int32_t* tenant_id;
  int T_tenants;
  const T* Wr;
  int pool, act, top_k;
  bool wr4;            // rows of Wr in aligned fours
  int S, C;            // token slices per request, column slabs
  uint32_t tag_lo, tag_hi;  // this call's tag, tag_lo != 0
  float* partial;      // [B][C][S][32 * VEC]
  u32x2* arrived;      // [B][C][S]: the tag once the slice's slab sums are in `partial`
  u32x4* share;        // [B][C][4]: {logit 2u, logit 2u + 1, tag} of the slab
  uint8_t* route_out;
  float* logits_out;
  RationalCoef coef;
};

// A request without a valid span or tenant.
template <typename T>
__device__ __forceinline__ void no_route(const PoolRouteArgs<T>& p, int b) {
  if (threadIdx.x == 0) p.route_out[b] = MILORA_ROUTE_NONE;
  if (p.logits_out && threadIdx.x < MILORA_NUM_SITES) p.logits_out[b * MILORA_NUM_SITES + threadIdx.x] = __uint_as_float(0x7fc00000u);
}

// Router weights of the four columns that lane f < FT finishes, zero past the row's end.
template <typename T, int FT>
__device__ __forceinline__ void load_router_weights(const PoolRouteArgs<T>& p, int ten, int f, int fcol, float (&wr)[MILORA_NUM_SITES][4]) {
#pragma unroll
  for (int j = 0; j < MILORA_NUM_SITES; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) wr[j][v] = 0.f;
  if (f >= FT || fcol >= p.d) return;
  const T* wt = p.Wr + (size_t)ten * MILORA_NUM_SITES * p.d + fcol;
  if (p.wr4) {  // rows of whole, aligned fours
#pragma unroll
    for (int j = 0; j < MILORA_NUM_SITES; ++j) {
      const Four<T> q = *reinterpret_cast<const Four<T>*>(wt + (size_t)j * p.d);
#pragma unroll
      for (int v = 0; v < 4; ++v) wr[j][v] = Elem<T>::load(q.v, v);
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < MILORA_NUM_SITES; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float w = Elem<T>::load(wt + (size_t)j * p.d, fcol + v < p.d ? v : 0);
      wr[j][v] = fcol + v < p.d ? w : 0.f;
    }
}

// Columns 4 f .. + 3 of the sixteen token lanes, added in a fixed tree.
template <int SW>
__device__ __forceinline__ f32x4 add_token_lanes(const float (&red)[kTokenLanes][SW], int f) {
  f32x4 r[kTokenLanes];
#pragma unroll
  for (int i = 0; i < kTokenLanes; ++i) r[i] = *reinterpret_cast<const f32x4*>(&red[i][4 * f]);
  return (((r[0] + r[1]) + (r[2] + r[3])) + ((r[4] + r[5]) + (r[6] + r[7]))) +
         (((r[8] + r[9]) + (r[10] + r[11])) + ((r[12] + r[13]) + (r[14] + r[15])));
}

// z = g(scale * h) of a lane's columns fcol .. fcol + 3 (where `on`) and what they add to the seven logits, summed over the wave: lane
// 8 j .. 8 j + 7 end with logit j.  Each of the first three steps halves what a lane holds: ten exchanges, not forty-two.
// (The end of a router's launch is a chain of round trips and of the code between them: with these ten, the activation as one jump for
// four columns, router weights in one load per row and the maximum apart from the sums, a call on 32 prompts of 256 tokens,
// d = 4096, went from 18.0 to 14.8 us, and to 14.3, 4.7 TB/s, with the choice below made between values.)
template <typename T>
__device__ __forceinline__ float wave_logits(const PoolRouteArgs<T>& p, bool on, int fcol, int lane, f32x4 h, float scale,
                                             const float (&wr)[MILORA_NUM_SITES][4]) {
  float z[4], lg[8];
#pragma unroll
  for (int v = 0; v < 4; ++v) z[v] = h[v] * scale;
  activate4(z, p.act, p.coef);
#pragma unroll
  for (int v = 0; v < 4; ++v) z[v] = on && fcol + v < p.d ? z[v] : 0.f;  // (nothing of what lies past the end, its weights are zeros)
#pragma unroll
  for (int j = 0; j < 8; ++j) lg[j] = 0.f;
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int j = 0; j < MILORA_NUM_SITES; ++j) lg[j] += z[v] * wr[j][v];
#pragma unroll
  for (int half = 4, off = 32; half >= 1; half >>= 1, off >>= 1)
#pragma unroll
    for (int i = 0; i < half; ++i) {
      const bool up = (lane & off) != 0;
      const float x0 = lg[i], x1 = lg[i + half];  // (values: a choice between elements becomes a search by index)
      const float give = up ? x0 : x1, keep = up ? x1 : x0;
      lg[i] = keep + __shfl_xor(give, off, 64);
    }
#pragma unroll
  for (int off = 4; off >= 1; off >>= 1) lg[0] += __shfl_xor(lg[0], off, 64);
  return lg[0];
}

// A slab's share of the seven logits is known (lanes 8 j ..: logit j): hand it over and, by the wave that finds every slab's share,
// select.  Called by one wave.
template <typename T>
__device__ __forceinline__ void finish_request(const PoolRouteArgs<T>& p, int b, int c, int lane, float share) {
  // (lane u: logits 2 u and 2 u + 1)
  float a0 = __shfl(share, (16 * lane) & 63, 64), a1 = __shfl(share, (16 * lane + 8) & 63, 64);
  if (p.C > 1) {
    // unit u of the slab: logits 2u and 2u + 1 with the tag.  Lane i takes units i, i + 64, ...: always unit i % 4,
    // of slabs i / 4, i / 4 + 16, ...; the sixteen running sums of a unit are then added across the lanes.
    u32x4* units = p.share + (size_t)b * p.C * 4;
    if (lane < 4) st_through(units + c * 4 + lane, u32x4{__float_as_uint(a0), __float_as_uint(a1), p.tag_lo, p.tag_hi});
    wait_all_mem();
    bool all = true;
    a0 = a1 = 0.f;
    for (int i = lane; i < 4 * p.C; i += 64) {
      const u32x4 g = ld_through(units + i);
      all = all && g[2] == p.tag_lo && g[3] == p.tag_hi;
      a0 += __uint_as_float(g[0]);
      a1 += __uint_as_float(g[1]);
    }
    if (__builtin_amdgcn_readfirstlane(__ballot(all) != ~0ull)) return;
    for (int i = lane; i < 4 * p.C; i += 64) st_through(units + i, u32x4{0u, 0u, 0u, 0u});
    for (int off = 4; off < 64; off <<= 1) {
      a0 += __shfl_xor(a0, off, 64);
      a1 += __shfl_xor(a1, off, 64);
    }
  }
  float logit[MILORA_NUM_SITES];
#pragma unroll
  for (int j = 0; j < MILORA_NUM_SITES; ++j) logit[j] = __shfl(j & 1 ? a1 : a0, j >> 1, 64);
  const float mine0 = __shfl(a0, lane >> 1, 64), mine1 = __shfl(a1, lane >> 1, 64);
  if (p.logits_out && lane < MILORA_NUM_SITES) p.logits_out[b * MILORA_NUM_SITES + lane] = lane & 1 ? mine1 : mine0;
  const uint8_t route = select_route(logit, p.top_k);
  if (lane == 0) p.route_out[b] = route;
}

template <typename T, int VEC, bool is_max>
__global__ void __launch_bounds__(kPoolThreads) pool_route_kernel(PoolRouteArgs<T> p) {
  constexpr int SW = kColLanes * VEC;  // columns of a slab
  constexpr int FT = SW / 4;           // lanes of the first wave that finish the slab, four columns each
  constexpr int TL = kTokenLanes;
  static_assert(FT <= 64 && TL == 16, "the finish is written for one wave and sixteen token lanes");
  __shared__ __align__(16) float red[TL][SW];
  const int c = blockIdx.x % p.C, s = blockIdx.x / p.C, b = blockIdx.y;
  const int cl = threadIdx.x % kColLanes, tl = threadIdx.x / kColLanes;
  const int d = p.d;
  int64_t start = p.seq_start[b], n = p.seq_len[b];
  const int ten = p.tenant_id[b];
  if (!span_ok(start, n, p.M_tok) || ten < 0 || ten >= p.T_tenants) {
    if (blockIdx.x == 0) no_route(p, b);
    return;
  }
  float scale = is_max ? 1.0f : 1.0f / (float)n;
  if (p.pool == MILORA_POOL_LAST) {  // the average over the last valid row alone
    start += n - 1;
    n = 1;
    scale = 1.0f;
  }
  const int64_t per = (n + p.S - 1) / p.S;
  const int64_t t0 = start + (int64_t)s * per;
  int64_t t1 = t0 + per;
  if (t1 > start + n) t1 = start + n;

  // ---- the finishing lanes ask for their router weights first: the values arrive while the rows stream
  const int f = threadIdx.x;
  const int fcol = c * SW + 4 * f;
  float wr[MILORA_NUM_SITES][4];
  load_router_weights<T, FT>(p, ten, f, fcol, wr);

  // ---- pool the slice: token lane tl takes rows t0 + tl, t0 + tl + 16, ...
  const int col = c * SW + cl * VEC;
  const float ident = is_max ? -INFINITY : 0.f;
  float acc[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) acc[v] = ident;
  if (col < d) {
    const T* q = p.H + col;
    int64_t t = t0 + tl;
    for (; t + 7 * TL < t1; t += 8 * TL) {
      float x[8][VEC];
#pragma unroll
      for (int u = 0; u < 8; ++u) VecLoad<T, VEC>::load_once(q + (size_t)(t + u * TL) * d, x[u]);
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        if (is_max)
          acc[v] = fmaxf(acc[v], fmaxf(fmaxf(fmaxf(x[0][v], x[1][v]), fmaxf(x[2][v], x[3][v])),
                                       fmaxf(fmaxf(x[4][v], x[5][v]), fmaxf(x[6][v], x[7][v]))));
        else
          acc[v] += ((x[0][v] + x[1][v]) + (x[2][v] + x[3][v])) + ((x[4][v] + x[5][v]) + (x[6][v] + x[7][v]));
      }
    }
    for (; t < t1; t += TL) {
      float x0[VEC];
      VecLoad<T, VEC>::load_once(q + (size_t)t * d, x0);
#pragma unroll
      for (int v = 0; v < VEC; ++v) acc[v] = is_max ? fmaxf(acc[v], x0[v]) : acc[v] + x0[v];
    }
  }
#pragma unroll
  for (int v = 0; v < VEC; ++v) red[tl][cl * VEC + v] = acc[v];
  __syncthreads();
  if (threadIdx.x >= 64) return;  // the first wave finishes
  const int lane = threadIdx.x;

  f32x4 h = {ident, ident, ident, ident};
  if (f < FT) {
    if (is_max) {
      f32x4 r[TL];
#pragma unroll
      for (int i = 0; i < TL; ++i) r[i] = *reinterpret_cast<const f32x4*>(&red[i][4 * f]);
#pragma unroll
      for (int v = 0; v < 4; ++v)
        h[v] = fmaxf(fmaxf(fmaxf(fmaxf(r[0][v], r[1][v]), fmaxf(r[2][v], r[3][v])),
                           fmaxf(fmaxf(r[4][v], r[5][v]), fmaxf(r[6][v], r[7][v]))),
                     fmaxf(fmaxf(fmaxf(r[8][v], r[9][v]), fmaxf(r[10][v], r[11][v])),
                           fmaxf(fmaxf(r[12][v], r[13][v]), fmaxf(r[14][v], r[15][v]))));
    } else {
      h = add_token_lanes<SW>(red, f);
    }
  }
  if (p.S > 1) {
    // slab sums of this slice to memory, then the flag; whoever then finds every slice's flag adds the slices up
    f32x4* mine = reinterpret_cast<f32x4*>(p.partial + (((size_t)b * p.C + c) * p.S + s) * SW);
    if (f < FT) st_through(mine + f, h);
    wait_all_mem();
    u32x2* flags = p.arrived + ((size_t)b * p.C + c) * p.S;
    if (lane == 0) st_through(flags + s, u32x2{p.tag_lo, p.tag_hi});
    wait_all_mem();
    bool all = true;
    for (int i = lane; i < p.S; i += 64) {
      const u32x2 g = ld_through(flags + i);
      all = all && g[0] == p.tag_lo && g[1] == p.tag_hi;
    }
    if (__builtin_amdgcn_readfirstlane(__ballot(all) != ~0ull)) return;
    // Two slices that store their flags at the same time both find every flag.  Only one may go on: the second would
    // store the slab's share again after the request's finishing wave has wiped the shares, and a replay of a
    // recorded launch (same tag) would take that left-over share for the new one.  The one that takes the flag of
    // slice 0 away goes on.
    {
      unsigned long long old = 0ull;
      if (lane == 0)
        old = __hip_atomic_exchange(reinterpret_cast<unsigned long long*>(flags), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint32_t old_lo = __builtin_amdgcn_readfirstlane((uint32_t)old), old_hi = __builtin_amdgcn_readfirstlane((uint32_t)(old >> 32));
      if (old_lo != p.tag_lo || old_hi != p.tag_hi) return;
    }
    for (int i = lane; i < p.S; i += 64) st_through(flags + i, u32x2{0u, 0u});
    if (f < FT) {
      const f32x4* base = reinterpret_cast<const f32x4*>(p.partial + ((size_t)b * p.C + c) * p.S * SW) + f;
      f32x4 tot = {ident, ident, ident, ident};
      for (int s0 = 0; s0 < p.S; s0 += 8) {
        const f32x4* q8[8];
        f32x4 x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) q8[u] = base + (size_t)(s0 + u < p.S ? s0 + u : p.S - 1) * FT;
        ld_through8(q8, x);
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (s0 + u >= p.S) x[u] = f32x4{ident, ident, ident, ident};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (is_max)
            tot[v] = fmaxf(tot[v], fmaxf(fmaxf(fmaxf(x[0][v], x[1][v]), fmaxf(x[2][v], x[3][v])),
                                         fmaxf(fmaxf(x[4][v], x[5][v]), fmaxf(x[6][v], x[7][v]))));
          else
            tot[v] += ((x[0][v] + x[1][v]) + (x[2][v] + x[3][v])) + ((x[4][v] + x[5][v]) + (x[6][v] + x[7][v]));
        }
      }
      h = tot;
    }
  }

  finish_request(p, b, c, lane, wave_logits(p, f < FT, fcol, lane, h, scale, wr));
}

// ---- self-attention pooling (App. C): u_t = H[t] . w_sa, a = softmax over the request's tokens, p = sum_t a_t H[t] ----
// One pass over H.  The valid tokens of all requests, one request after the other, are a line that is cut into equal
// pieces, one per workgroup, whatever the lengths.  A workgroup holds a row across its threads (16 bytes each, P of them) and
// takes R rows at a time: R scores (in-wave sums, then over the waves through LDS, one barrier), weights relative to the
// running maximum (a batch that raises it rescales what was gathered before), weighted sum out of the same registers,
// while the next R rows are on their way.  The part of a piece that lies in one request leaves a row of unnormalised sums
// and (maximum, sum of weights) in the workspace, at index piece + request; the finishing launch merges a request's rows.
// Bound: the read of H.  16 prompts of 1024 to 2048 tokens, d = 4096 (201 MB): 38.6 us = 5.2 TB/s and 8.2 us
// for the finishing launch, six dependent round trips (with slices of 16 tokens, each read twice, and one finishing workgroup
// per request: 65 and 72 us).
constexpr int kSelfAttnMaxD = 8192;
constexpr int kAttnMaxWaves = 16;

// VEC neighbouring elements as they lie in memory; read once.
template <typename T, int VEC> struct Piece;
template <> struct Piece<bf16_t, 8> {
  raw_u32x4 v;
  __device__ __forceinline__ void load(const bf16_t* p) { v = __builtin_nontemporal_load(reinterpret_cast<const raw_u32x4*>(p)); }
  __device__ __forceinline__ float get(int i) const { return __uint_as_float((i & 1) ? v[i >> 1] & 0xffff0000u : v[i >> 1] << 16); }
};
template <> struct Piece<float, 4> {
  raw_u32x4 v;
  __device__ __forceinline__ void load(const float* p) { v = __builtin_nontemporal_load(reinterpret_cast<const raw_u32x4*>(p)); }
  __device__ __forceinline__ float get(int i) const { return __uint_as_float(v[i]); }
};
template <typename T> struct Piece<T, 1> {
  T v;
  __device__ __forceinline__ void load(const T* p) { v = *p; }
  __device__ __forceinline__ float get(int) const { return Elem<T>::load(&v, 0); }
};

struct AttnParts {
  float* partial;  // [pieces + B][pitch]
  float2* ml;      // [pieces + B] maximum, sum of weights
  int2* span;      // [B] first row of the request in `partial`, rows
  int pitch;
};

__device__ __forceinline__ int64_t attn_tokens(const int32_t* seq_start, const int32_t* seq_len, const int32_t* tenant_id, int b,
                                               int64_t M_tok, int T_tenants) {
  const int64_t start = seq_start[b], n = seq_len[b];
  const int ten = tenant_id[b];
  const bool ok = (n >= 1) & (start >= 0) & (start + n <= M_tok) & ((uint32_t)ten < (uint32_t)T_tenants);  // (no branches: many are in flight)
  return ok ? n : 0;
}

template <typename T, int VEC, int P>
__global__ void __launch_bounds__(kAttnMaxWaves * 64) pool_selfattn_kernel(const T* __restrict__ H, int64_t M_tok, int d, int B,
                                                                          const int32_t* __restrict__ seq_start,
                                                                          const int32_t* __restrict__ seq_len,
                                                                          const int32_t* __restrict__ tenant_id, int T_tenants,
                                                                          const T* __restrict__ w_sa, AttnParts out) {
  constexpr int R = P == 1 ? 8 : P == 2 ? 4 : 2;  // rows of a batch: two batches of P * R pieces are in registers
  constexpr int Lanes = 64 / R;      // lanes that share a row's sum
  __shared__ float red[2][kAttnMaxWaves][R];
  __shared__ int64_t wave_sum[kAttnMaxWaves], s_base;
  __shared__ int s_lo, s_hi;
  const int tid = threadIdx.x, lane = tid & 63, n_threads = blockDim.x, nw = n_threads >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // ---- this workgroup's piece of the line, and the request of its first token: by sums over ever smaller runs of requests, one
  // run a thread (one pass for up to n_threads requests, three for 65535 and a single wave)
  const int g = blockIdx.x;
  int64_t per = 0, pos = 0, left = 0, base = 0;  // (base: tokens of the requests before lo)
  int lo = 0;
  for (int hi = B, run = 0; run != 1;) {
    run = (hi - lo + n_threads - 1) / n_threads;
    const int b0 = lo + tid * run, b1 = b0 + run < hi ? b0 + run : hi;
    int64_t mine = 0;
#pragma unroll 4
    for (int b = b0; b < b1; ++b) mine += attn_tokens(seq_start, seq_len, tenant_id, b, M_tok, T_tenants);
    int64_t incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int64_t o = __shfl_up(incl, off, 64);
      incl += lane >= off ? o : 0;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int64_t total = 0;
    incl += base;
    for (int i = 0; i < nw; ++i) {
      incl += i < wave ? wave_sum[i] : 0;
      total += wave_sum[i];
    }
    if (per == 0) {
      per = (total + gridDim.x - 1) / gridDim.x;
      if (per > R) per = (per + R - 1) / R * R;
      pos = (int64_t)g * per;
      if (pos >= total) return;
      left = total - pos < per ? total - pos : per;
    }
    if (pos >= incl - mine && pos < incl) {
      s_lo = b0;
      s_hi = b1;
      s_base = incl - mine;
    }
    __syncthreads();
    lo = __builtin_amdgcn_readfirstlane(s_lo);
    hi = __builtin_amdgcn_readfirstlane(s_hi);
    base = s_base;
  }
  int off = __builtin_amdgcn_readfirstlane((int)(pos - base));  // of the piece's first token in its request

  const int ncg = d / VEC;
  // The requests behind the first that take part are looked up 64 at a time: one that does not costs a 64th of a round trip.
  unsigned long long todo = 1;  // of requests lo ..
  for (int window = 1; left > 0; todo &= todo - 1, off = 0) {
    while (!todo) {
      lo += window;
      window = 64;
      const int b = lo + lane;
      todo = __ballot(b < B && attn_tokens(seq_start, seq_len, tenant_id, b < B ? b : B - 1, M_tok, T_tenants) > 0);
    }
    const int b = lo + __builtin_ctzll(todo);
    const int64_t n = seq_len[b];
    const uint32_t rows_n = __builtin_amdgcn_readfirstlane((int)(n - off < left ? n - off : left));
    const T* rows = H + ((size_t)seq_start[b] + off) * d;  // (the row may lie beyond 2^31)
    const T* q = w_sa + (size_t)tenant_id[b] * d;
    int col[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int c = p * n_threads + tid;
      col[p] = (c < ncg ? c : ncg - 1) * VEC;  // past the row's end: its last piece, of which nothing is taken
    }
    Piece<T, VEC> x[2][R][P];
    auto ask = [&](uint32_t t, Piece<T, VEC> (&v)[R][P]) __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint32_t row = t + r < rows_n ? t + r : rows_n - 1;  // past the end: the last row, with no weight
        const T* src = rows + (size_t)row * d;
#pragma unroll
        for (int p = 0; p < P; ++p) v[r][p].load(src + col[p]);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    ask(0, x[0]);
    float w[P][VEC], acc[P][VEC];
#pragma unroll
    for (int p = 0; p < P; ++p) {
      float v[VEC];
      VecLoad<T, VEC>::load(q + col[p], v);
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        w[p][e] = v[e];
        acc[p][e] = 0.f;
      }
    }
    float m_run = -INFINITY, l_run = 0.f;  // (l_run: of row lane % R of every batch)
    auto batch = [&](uint32_t t, int buf, Piece<T, VEC> (&v)[R][P]) __attribute__((always_inline)) {
      float u[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        u[r] = 0.f;
#pragma unroll
        for (int p = 0; p < P; ++p) {
          const float before = u[r];
#pragma unroll
          for (int e = 0; e < VEC; ++e) u[r] += v[r][p].get(e) * w[p][e];
          u[r] = p * n_threads + tid < ncg ? u[r] : before;  // (not a product with zero: the row's last piece may hold Inf)
        }
      }
      // sums over the lanes: every step halves the rows a lane holds, row lane / Lanes is left
#pragma unroll
      for (int h = R / 2, o = 32; h >= 1; h >>= 1, o >>= 1)
#pragma unroll
        for (int i = 0; i < h; ++i) {
          const bool up = (lane & o) != 0;
          const float x0 = u[i], x1 = u[i + h];  // (values: a choice between elements becomes a search by index)
          const float give = up ? x0 : x1, keep = up ? x1 : x0;
          u[i] = keep + __shfl_xor(give, o, 64);
        }
#pragma unroll
      for (int o = Lanes / 2; o >= 1; o >>= 1) u[0] += __shfl_xor(u[0], o, 64);
      if (lane % Lanes == 0) red[buf][wave][lane / Lanes] = u[0];
      __builtin_amdgcn_s_waitcnt(0xc07f);  // LDS only: the next rows stay on their way
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      float s = 0.f;
      for (int i = lane / R; i < nw; i += Lanes) s += red[buf][i][lane % R];
#pragma unroll
      for (int o = R; o < 64; o <<= 1) s += __shfl_xor(s, o, 64);
      if (t + lane % R >= rows_n) s = -INFINITY;
      float m_new = s;
#pragma unroll
      for (int o = 1; o < R; o <<= 1) m_new = fmaxf(m_new, __shfl_xor(m_new, o, 64));
      m_new = fmaxf(m_run, m_new);
      const float ref = m_new == -INFINITY ? 0.f : m_new;
      const float scale = expf(m_run - ref), pw = expf(s - ref);  // (first batch: scale 0)
      l_run = l_run * scale + pw;
      m_run = m_new;
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[p][e] *= scale;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        // (opaque: the floats of the scores are formed again rather than kept)
        if constexpr (VEC * sizeof(T) == 16)
#pragma unroll
          for (int p = 0; p < P; ++p) asm volatile("" : "+v"(v[r][p].v));
        const float a = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(pw), r));
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
          for (int e = 0; e < VEC; ++e) acc[p][e] += a * v[r][p].get(e);
      }
    };
    for (uint32_t t = 0; t < rows_n; t += 2 * R) {
      ask(t + R, x[1]);
      batch(t, 0, x[0]);
      if (t + R >= rows_n) break;
      ask(t + 2 * R, x[0]);
      batch(t + R, 1, x[1]);
    }
#pragma unroll
    for (int o = 1; o < R; o <<= 1) l_run += __shfl_xor(l_run, o, 64);
    const size_t idx = (size_t)g + b;
    float* const o = out.partial + idx * out.pitch;
#pragma unroll
    for (int p = 0; p < P; ++p)
      if (p * n_threads + tid < ncg)
#pragma unroll
        for (int e = 0; e < VEC; ++e) o[col[p] + e] = acc[p][e];
    if (tid == 0) {
      out.ml[idx] = float2{m_run, l_run};
      if (off == 0) out.span[b] = int2{(int)idx, (int)((pos + n - 1) / per) - g + 1};
    }
    pos += rows_n;
    left -= rows_n;
    __syncthreads();  // (the next request's first batch writes the buffer that the last one's may still be read from)
  }
}

// Finish of the self-attention pooler: a workgroup of 512 threads merges CL * 4 columns of a request's rows (each holds a
// sum weighted by exp(u - m_s): brought to the common maximum and normalised), 512 / CL rows side by side, eight of each on
// their way, and goes on as pool_route_kernel does.  The widest take four: there are few rows to merge then and many workgroups, of
// which a compute unit holds more so (calls of 1000 requests of 4 rows, d = 4096: 47.4 us with eight, 41.3 with four).
template <typename T, int CL>
__global__ void __launch_bounds__(kPoolThreads) selfattn_finish_kernel(PoolRouteArgs<T> p, AttnParts in) {
  constexpr int SW = CL * 4, TL = kPoolThreads / CL, kWaves = (CL + 63) / 64;  // waves that finish
  __shared__ __align__(16) float red[TL][SW];
  __shared__ float wave_lg[kWaves][64];
  const int c = blockIdx.x, b = blockIdx.y;
  const int cl = threadIdx.x % CL, tl = threadIdx.x / CL, lane = threadIdx.x & 63;
  const int2 sp = in.span[b];  // (asked for with the facts that say whether it means anything)
  const int64_t start = p.seq_start[b], n = p.seq_len[b];
  const int ten = p.tenant_id[b];
  if (!span_ok(start, n, p.M_tok) || ten < 0 || ten >= p.T_tenants) {
    if (c == 0) no_route(p, b);
    return;
  }
  // the first U * TL rows and their maxima before anything waits, the router weights behind them
  const float2* ml = in.ml + sp.x;
  const int col = c * SW + cl * 4 < in.pitch ? c * SW + cl * 4 : 0;  // (past the end: never used)
  const f32x4* rows = reinterpret_cast<const f32x4*>(in.partial + (size_t)sp.x * in.pitch + col);
  constexpr int U = CL == 512 ? 4 : 8;  // rows on their way
  f32x4 x[U];
  float m[U];
  auto ask = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * TL < sp.y ? i0 + u * TL : sp.y - 1;
      m[u] = ml[i].x;
      x[u] = rows[(size_t)i * (in.pitch / 4)];
    }
  };
  float2 own = float2{-INFINITY, 0.f};
  if (lane < sp.y) own = ml[lane];
  ask(tl);
  float wr[MILORA_NUM_SITES][4];
  load_router_weights<T, CL>(p, ten, threadIdx.x, c * SW + 4 * (int)threadIdx.x, wr);
  __builtin_amdgcn_sched_barrier(0);
  float mx = own.x;
  for (int i = lane + 64; i < sp.y; i += 64) mx = fmaxf(mx, ml[i].x);
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  const float ref = mx == -INFINITY ? 0.f : mx;
  float z = own.y * expf(own.x - ref);
  for (int i = lane + 64; i < sp.y; i += 64) z += ml[i].y * expf(ml[i].x - ref);
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) z += __shfl_xor(z, o, 64);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int i0 = tl; i0 < sp.y; i0 += U * TL) {
    if (i0 != tl) ask(i0);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + u * TL < sp.y) acc += expf(m[u] - ref) * x[u];
  }
  acc *= 1.0f / z;
  if constexpr (TL > 1) {
    *reinterpret_cast<f32x4*>(&red[tl][cl * 4]) = acc;
    __syncthreads();
    if (threadIdx.x < CL) {
      acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < TL; ++i) acc += *reinterpret_cast<const f32x4*>(&red[i][cl * 4]);
    }
  }
  float share = 0.f;
  if (threadIdx.x < kWaves * 64) share = wave_logits(p, threadIdx.x < CL, c * SW + 4 * (int)threadIdx.x, lane, acc, 1.0f, wr);
  if constexpr (kWaves > 1) {
    if (threadIdx.x < kWaves * 64) wave_lg[threadIdx.x >> 6][lane] = share;
    __syncthreads();
  }
  if (threadIdx.x >= 64) return;
  if constexpr (kWaves > 1) {
    share = wave_lg[0][lane];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) share += wave_lg[w][lane];
  }
  finish_request(p, b, c, lane, share);
}

// Workspace of the self-attention pooler.  Pieces of the line: two workgroups of up to eight waves per compute unit, one of
// more, four of up to four; as many as there are eights of rows in H, but one per request at least: requests may be shorter, or share
// their rows, so that the line is longer than H (d = 4096, 64 requests of one row each: 35.8 us with 8 pieces, 12.6 with 64; 64 over
// the same 16 rows: 182 us with 2, 13.9 with 64).
// Column lanes of a finishing workgroup: few rows to merge, wide slabs (many requests are then few workgroups, and a row that fits
// one of them needs no hand-over); more, narrow ones, so that all rows are on their way together.  Calls of 200 prompts of 16
// to 128 tokens, d = 4096 (4 rows each): 133 us with 32 lanes, 53 with 512; 32 of 256 (17 rows): 36 us with 32, 29 with 128; 16 of
// 1024 to 2048 (33 rows): the finishing launch 10.6 us with 32, 11.6 with 128 (all before its end got shorter: 40.5, 25.9 and 8.2 us
// at the widths taken).
struct AttnCarve {
  int pieces, lanes, C, pitch;
  size_t ml, span, share, total;  // byte offsets, and the size
};
AttnCarve carve_attn(int B, int d, int64_t M_tok, int waves) {
  AttnCarve a;
  const int64_t eights = (M_tok + 7) / 8, most = eights > B ? eights : B;
  a.pieces = waves <= 4 ? 1024 : waves <= 8 ? 512 : 256;
  if (a.pieces > most) a.pieces = (int)most;
  const int to_merge = a.pieces / B + 1;
  a.lanes = to_merge <= 8 ? 512 : to_merge <= 20 ? 128 : 32;
  a.C = (d + a.lanes * 4 - 1) / (a.lanes * 4);
  a.pitch = (d + 3) / 4 * 4;
  const size_t rows = (size_t)a.pieces + B;
  a.ml = align_up(rows * a.pitch * sizeof(float), 256);
  a.span = a.ml + align_up(rows * sizeof(float2), 256);
  a.share = a.span + align_up((size_t)B * sizeof(int2), 256);
  a.total = a.share + align_up((size_t)B * ((d + 127) / 128) * 4 * 16, 256);
  return a;
}

// Token slices per request of pool_route_kernel with C column slabs: one, unless the requests are so few that
// compute units would be left without work; none shorter than 64 rows.  (Slices of a fixed 256 rows, eight per
// 2048-token prompt, measured a third slower than two: every cut adds the hand-over through memory.)
int pick_slices(int B, int C, int64_t M_tok) {
  const int64_t avg = (M_tok + B - 1) / B;
  int64_t s = (512 + (int64_t)B * C - 1) / ((int64_t)B * C);
  if (s > (avg + 63) / 64) s = (avg + 63) / 64;
  if (s > kMaxSplits) s = kMaxSplits;
  if (s < 1) s = 1;
  return (int)s;
}

// Workspace of pool_route_kernel: slab sums of the slices, their flags, the slabs' logit shares.
struct PoolRouteCarve {
  int S, C;
  size_t partial, arrived, share, total;  // byte offsets, and the size
};
PoolRouteCarve carve_pool_route(int B, int d, int64_t M_tok, int slab_cols, bool last_only) {
  PoolRouteCarve c;
  c.C = (d + slab_cols - 1) / slab_cols;
  c.S = last_only ? 1 : pick_slices(B, c.C, M_tok);
  c.partial = 0;
  c.arrived = align_up((size_t)B * c.C * c.S * slab_cols * sizeof(float), 256);
  c.share = c.arrived + align_up((size_t)B * c.C * c.S * 8, 256);
  c.total = c.share + align_up((size_t)B * c.C * 4 * 16, 256);
  return c;
}

std::atomic<uint32_t> g_route_calls{0};

template <typename T>
void new_tag(PoolRouteArgs<T>& a) {
  a.tag_hi = ++g_route_calls;
  a.tag_lo = (a.tag_hi * 2654435761u ^ 0x9e3779b9u) | 1u;
}

template <typename T, int VEC>
int launch_pool_route(PoolRouteArgs<T> a, int B, int64_t M_tok, void* workspace, size_t workspace_bytes,
                      hipStream_t st) {
  const PoolRouteCarve cv = carve_pool_route(B, a.d, M_tok, kColLanes * VEC, a.pool == MILORA_POOL_LAST);
  if (!workspace || workspace_bytes < cv.total) return MILORA_EWORKSPACE;
  if ((size_t)cv.C * cv.S > 65535u * 32u) return MILORA_ERANGE;
  a.S = cv.S;
  a.C = cv.C;
  new_tag(a);
  a.partial = (float*)((char*)workspace + cv.partial);
  a.arrived = (u32x2*)((char*)workspace + cv.arrived);
  a.share = (u32x4*)((char*)workspace + cv.share);
  const dim3 grid(cv.C * cv.S, B);
  if (a.pool == MILORA_POOL_MAX) hipLaunchKernelGGL((pool_route_kernel<T, VEC, true>), grid, dim3(kPoolThreads), 0, st, a);
  else hipLaunchKernelGGL((pool_route_kernel<T, VEC, false>), grid, dim3(kPoolThreads), 0, st, a);
  return check_launch();
}

template <typename T, int VEC, int P>
int launch_attn(PoolRouteArgs<T> a, const T* w_sa, int B, void* workspace, hipStream_t st) {
  const int pieces_of_row = a.d / VEC, waves = (pieces_of_row + 64 * P - 1) / (64 * P);
  const AttnCarve cv = carve_attn(B, a.d, a.M_tok, waves);
  char* const ws = (char*)workspace;
  AttnParts parts{(float*)ws, (float2*)(ws + cv.ml), (int2*)(ws + cv.span), cv.pitch};
  hipLaunchKernelGGL((pool_selfattn_kernel<T, VEC, P>), dim3(cv.pieces), dim3(waves * 64), 0, st, a.H, a.M_tok, a.d, B, a.seq_start,
                     a.seq_len, a.tenant_id, a.T_tenants, w_sa, parts);
  int rc = check_launch();
  if (rc) return rc;
  a.C = cv.C;
  new_tag(a);
  a.share = (u32x4*)(ws + cv.share);
  const dim3 grid(cv.C, B);
  if (cv.lanes == 512) hipLaunchKernelGGL((selfattn_finish_kernel<T, 512>), grid, dim3(kPoolThreads), 0, st, a, parts);
  else if (cv.lanes == 128) hipLaunchKernelGGL((selfattn_finish_kernel<T, 128>), grid, dim3(kPoolThreads), 0, st, a, parts);
  else hipLaunchKernelGGL((selfattn_finish_kernel<T, 32>), grid, dim3(kPoolThreads), 0, st, a, parts);
  return check_launch();
}

}  // namespace

}  // namespace milora

using namespace milora;

extern "C" size_t milora_route_workspace_bytes(int B, int d, int64_t M_tok) {
  if (B < 1 || d < 1 || M_tok < 1) return 0;
  size_t need = 0;
  for (int waves : {4, 8, kAttnMaxWaves}) {  // of the self-attention pooler: a wave of it holds at most 512 columns, 1024 if there are 16
    const int most = waves < kAttnMaxWaves ? waves * 512 : d;
    const size_t n = carve_attn(B, d < most ? d : most, M_tok, waves).total;
    if (n > need) need = n;
  }
  for (int slab_cols : {32, 128, 256}) {  // the slab widths pool_route_kernel is built for
    const size_t n = carve_pool_route(B, d, M_tok, slab_cols, false).total;
    if (n > need) need = n;
  }
  return need;
}

namespace {

template <typename T>
int route_typed(const void* H, int64_t M_tok, int d, const int32_t* seq_start, const int32_t* seq_len,
                const int32_t* tenant_id, int B, int n_tenants, const void* Wr, int pool, int act, const void* w_sa,
                const RationalCoef& coef, int top_k, uint8_t* route_out, float* logits_out, void* workspace,
                size_t workspace_bytes, hipStream_t st) {
  constexpr int VEC = 16 / (int)sizeof(T);  // elements of a 16-byte load
  const bool vec = ((uintptr_t)H % 16) == 0 && d % VEC == 0;
  PoolRouteArgs<T> a;
  a.H = (const T*)H;
  a.M_tok = M_tok;
  a.d = d;
  a.seq_start = seq_start;
  a.seq_len = seq_len;
  a.tenant_id = tenant_id;
  a.T_tenants = n_tenants;
  a.Wr = (const T*)Wr;
  a.wr4 = d % 4 == 0 && (uintptr_t)Wr % (4 * sizeof(T)) == 0;
  a.pool = pool;
  a.act = act;
  a.top_k = top_k;
  a.route_out = route_out;
  a.logits_out = logits_out;
  a.coef = coef;
  if (pool == MILORA_POOL_SELFATTN) {
    if (workspace_bytes < milora_route_workspace_bytes(B, d, M_tok)) return MILORA_EWORKSPACE;
    const T* const w = (const T*)w_sa;
    if (vec && ((uintptr_t)w_sa % 16) == 0) {
      if constexpr (kSelfAttnMaxD > kAttnMaxWaves * 64 * VEC)  // more than one piece of a row per thread of the largest workgroup
        if (d > kAttnMaxWaves * 64 * VEC) return launch_attn<T, VEC, 2>(a, w, B, workspace, st);
      return launch_attn<T, VEC, 1>(a, w, B, workspace, st);
    }
    return d <= kAttnMaxWaves * 64 ? launch_attn<T, 1, 1>(a, w, B, workspace, st) : launch_attn<T, 1, 8>(a, w, B, workspace, st);
  }
  if (vec) return launch_pool_route<T, VEC>(a, B, M_tok, workspace, workspace_bytes, st);
  return launch_pool_route<T, 1>(a, B, M_tok, workspace, workspace_bytes, st);
}

}  // namespace

extern "C" int milora_route(const void* H, int64_t M_tok, int d, int dtype, const int32_t* seq_start,
                            const int32_t* seq_len, const int32_t* tenant_id, int B, int n_tenants, const void* Wr,
                            int pool, int act, const void* w_sa, const float* act_coef, int top_k,
                            uint8_t* route_out, float* logits_out, void* workspace, size_t workspace_bytes,
                            void* stream) {
  if (!H || !seq_start || !seq_len || !tenant_id || !Wr || !route_out) return MILORA_EINVAL;
  if (M_tok < 1 || d < 1 || B < 1 || n_tenants < 1) return MILORA_EINVAL;
  if (dtype != MILORA_BF16 && dtype != MILORA_F32) return MILORA_EINVAL;
  if (pool < MILORA_POOL_MEAN || pool > MILORA_POOL_SELFATTN) return MILORA_EINVAL;
  if (act < MILORA_ACT_IDENTITY || act > MILORA_ACT_RATIONAL) return MILORA_EINVAL;
  if (pool == MILORA_POOL_SELFATTN && !w_sa) return MILORA_EINVAL;
  if (act == MILORA_ACT_RATIONAL && !act_coef) return MILORA_EINVAL;
  if (top_k < 1 || top_k >= MILORA_NUM_SITES) return MILORA_EINVAL;
  if (B > 65535) return MILORA_ERANGE;
  if (pool == MILORA_POOL_SELFATTN && d > kSelfAttnMaxD) return MILORA_ERANGE;
  if (!workspace) return MILORA_EWORKSPACE;
  RationalCoef coef = {};
  if (act == MILORA_ACT_RATIONAL) {
    for (int j = 0; j < 7; ++j) coef.a[j] = act_coef[j];
    for (int j = 0; j < 5; ++j) coef.b[j] = act_coef[7 + j];
  }
  hipStream_t st = (hipStream_t)stream;
  if (dtype == MILORA_BF16)
    return route_typed<bf16_t>(H, M_tok, d, seq_start, seq_len, tenant_id, B, n_tenants, Wr, pool, act, w_sa, coef, top_k,
                               route_out, logits_out, workspace, workspace_bytes, st);
  return route_typed<float>(H, M_tok, d, seq_start, seq_len, tenant_id, B, n_tenants, Wr, pool, act, w_sa, coef, top_k,
                            route_out, logits_out, workspace, workspace_bytes, st);
}
