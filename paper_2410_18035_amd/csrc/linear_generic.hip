// Any-shape, any-dtype routed LoRA linear (paper Eq. 1 with the layer-level gate of Sec. 3.3): fp32 tensors, and bf16 ones
// of widths or alignments that the bf16 matrix-core kernels do not take.  All arithmetic is fp32, on the fp32 matrix
// instructions (157 TFLOP/s on the chip, twice the rate of vector FMA, each product and sum rounded as there).
//
// Operands are taken four consecutive k per lane (any element alignment; the row's last k one by one): instruction e of
// four multiplies element e of both sides, so the k of a block of 8 or 16 are taken in another order than memory's, the
// same one on both sides.  All sums run in a fixed order.
#include "common.h"

namespace milora {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint16_t u16x4_a2 __attribute__((ext_vector_type(4), aligned(2)));

__device__ __forceinline__ f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4_a4*>(p); }
__device__ __forceinline__ f32x4 load4(const bf16_t* p) {
  const u16x4_a2 v = *reinterpret_cast<const u16x4_a2*>(p);
  return f32x4{bf16_to_f32(v[0]), bf16_to_f32(v[1]), bf16_to_f32(v[2]), bf16_to_f32(v[3])};
}
// Elements k .. k + 3 of a row of K, zero past its end.
template <typename T>
__device__ __forceinline__ f32x4 load4_end(const T* row, int k, int K) {
  f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
  if (k + 4 <= K) v = load4(row + k);
  else
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (k + e < K) v[e] = Elem<T>::load(row, k + e);
  return v;
}
// Columns of one launch: a grid has to stay below 2^32 threads (512 for 16 columns in the few-row kernel).
constexpr int kLaunchCols = 1 << 26;

__device__ __forceinline__ int pow2_above(int r) {
  int p = 1;
  while (p < r) p <<= 1;
  return p;
}

// ---- LoRA shrink: t[m][c] = sum_k X[m][k] * A[k][c], c < r, one workgroup per (row, site) -------------------------
// Threads are laid out with the rank index fastest (coalesced reads of A's rows), eight rows of A per thread on their
// way; the k-lanes are summed through LDS in a fixed order.  Bound by the latency of those loads: 512 threads instead of
// 256 and eight loads in flight instead of one.
constexpr int kShrinkT = 512;
template <typename T>
__global__ void __launch_bounds__(kShrinkT) shrink_rows_kernel(const T* __restrict__ X, int64_t ldx, int64_t M, int d1,
                                                               const int32_t* __restrict__ row_to_req, AdapterView ad,
                                                               int site0, const int32_t* __restrict__ tenant_id,
                                                               const uint8_t* __restrict__ route, int B,
                                                               float* __restrict__ t) {
  __shared__ float red[kShrinkT];
  const int64_t m = blockIdx.x;
  const int site = site0 + blockIdx.y;
  const int64_t req = row_to_req ? (int64_t)row_to_req[m] : m;
  int tenant = 0;
  const int r = (req >= 0 && req < B) ? routed_rank(ad, tenant_id, route, (int)req, B, site, &tenant) : 0;
  if (r == 0) return;
  const T* A = (const T*)ad.A[tenant * MILORA_NUM_SITES + site];
  const int rpad = pow2_above(r);
  const int c = threadIdx.x & (rpad - 1), krow = threadIdx.x / rpad, rpp = kShrinkT / rpad;
  const T* x = X + (size_t)m * ldx;
  float acc = 0.f;
  if (c < r) {
    int k = krow;
    for (; k + 7 * rpp < d1; k += 8 * rpp) {
      float xv[8], av[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        xv[u] = Elem<T>::load(x, k + u * rpp);
        av[u] = Elem<T>::load(A, (size_t)(k + u * rpp) * r + c);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += xv[u] * av[u];
    }
    for (; k < d1; k += rpp) acc += Elem<T>::load(x, k) * Elem<T>::load(A, (size_t)k * r + c);
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  if (krow == 0 && c < r) {
    float s = 0.f;
    for (int j = 0; j < rpp; ++j) s += red[j * rpad + c];
    t[((size_t)blockIdx.y * M + m) * ad.r_max + c] = s;
  }
}

// ---- few rows: up to 16 --------------------------------------------------------------------------------------------
// A workgroup takes 16 columns of one linear (gate and up: of both) and the whole reduction, dealt to its waves in
// blocks of 16 k that go straight from global memory into matrix operands; the waves' sums meet in LDS.  Where rows, ranks
// and widths are small the shrinks are formed here too (FUSED, fuse_shrink), each wave over its share of k and one row after
// the other, again in every workgroup; else they come from shrink_rows_kernel.
// The layer's glue is part of the store: a decode step of a layer is four launches instead of eighteen.
// Bound: launches (about 2.4 us each with nothing in them), and the code a launch runs through, whose time goes with its
// bytes (4.6 KB 4.8 us, 7.7 KB 8.0 us): what a call does not need is compiled out, the shrinks of two sites are one loop, and
// four waves run through it where that is enough (few_waves: d = 256 22.3 -> 19.6 us).  A decode step of 4 rows through the 256 x 688 fp32 layer, rank 8: 284 us with eighteen launches,
// 22.3 us with four of eight waves and both expands in them, 19.6 us so.  Tried: base and adapter pointers asked for ahead of the
// look-ups (fewer dependent loads, more code: 26.9 against 24.3 us), 32-bit offsets with a path for whole trips (41.1 against 35.6 us at
// 16 rows, d = 504).
constexpr int kFewBlocks = 4;  // blocks of 16 k per wave on their way
constexpr int kFewNarrow = 256;  // no reduction longer than this on four waves

template <typename T>
__device__ __forceinline__ float round_to(float v) {
  T q;
  Elem<T>::store(&q, 0, v);
  return Elem<T>::load(&q, 0);
}

template <typename T, int MODE, int kFewW, bool FUSED>
__global__ void __launch_bounds__(kFewW * 64, 4) few_rows_kernel(const FewArgs g) {
  constexpr int NW = MODE == kFewGateUp ? 2 : 1;
  __shared__ float red[NW][kFewW][16][17];
  __shared__ float tpart[FUSED ? NW : 1][FUSED ? kFewW : 1][16][kFuseRank];
  __shared__ float ts[FUSED ? NW : 1][16][kFuseRank];
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int s0 = MODE == kFewGateUp ? 0 : blockIdx.y, n0 = g.col0 + blockIdx.x * 16;
  const int d1 = g.d1;

  // rank and tenant of row li at the workgroup's site, of its two sites in lanes 0 .. 15 and 16 .. 31 (route byte and tenant id are
  // asked for together)
  int rank = 0, ten = 0;
  {
    const int64_t req = li < g.M ? (g.row_to_req ? (int64_t)g.row_to_req[li] : li) : -1;
    const bool in = req >= 0 && req < g.B;
    const uint8_t rt = in ? g.route[req] : (uint8_t)MILORA_ROUTE_NONE;
    const int tn = in ? g.tenant_id[req] : -1;
    const bool known = tn >= 0 && tn < g.ad.n_tenants;
    const int r = known ? g.ad.rank[tn] : 0;
    if (known && lq < NW && route_has(rt, g.site[s0] + lq) && r >= 1 && r <= g.ad.r_max) {  // (sites of a workgroup are consecutive)
      rank = r;
      ten = tn;
    }
  }

  // ---- base linear ----
  const T* const xr = (const T*)g.X + (size_t)(li < g.M ? li : g.M - 1) * g.ldx;  // (rows past the end: results dropped)
  const int col = n0 + li < g.d2 ? n0 + li : g.d2 - 1;
  const T* wr[NW];
  f32x4 acc[NW];
#pragma unroll
  for (int j = 0; j < NW; ++j) {
    wr[j] = (const T*)g.W[s0 + j] + (size_t)col * d1;
    acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int full = d1 >> 4;
  for (int b0 = w; b0 < full; b0 += kFewW * kFewBlocks) {
    f32x4 xv[kFewBlocks], wv[NW][kFewBlocks];
#pragma unroll
    for (int u = 0; u < kFewBlocks; ++u) {
      const int b = b0 + u * kFewW < full ? b0 + u * kFewW : full - 1;
      xv[u] = load4(xr + b * 16 + lq * 4);
#pragma unroll
      for (int j = 0; j < NW; ++j) wv[j][u] = load4(wr[j] + b * 16 + lq * 4);
    }
#pragma unroll
    for (int u = 0; u < kFewBlocks; ++u)
      if (b0 + u * kFewW < full)
#pragma unroll
        for (int j = 0; j < NW; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[j][u][e], xv[u][e], acc[j], 0, 0, 0);
  }
  if (__builtin_expect(full * 16 < d1 && w == full % kFewW, 0)) {
    const f32x4 x = load4_end(xr, full * 16 + lq * 4, d1);
#pragma unroll
    for (int j = 0; j < NW; ++j) {
      const f32x4 v = load4_end(wr[j], full * 16 + lq * 4, d1);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[e], x[e], acc[j], 0, 0, 0);
    }
  }
  // (lane: row li, columns 4 lq .. + 3 of the 16)
#pragma unroll
  for (int j = 0; j < NW; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) red[j][w][li][lq * 4 + e] = acc[j][e];

  // ---- shrinks of the routed rows over this wave's share of k ----
  if constexpr (FUSED) {
    const int share = (d1 + kFewW - 1) / kFewW, k0 = w * share, k1 = k0 + share < d1 ? k0 + share : d1;
    for (unsigned long long left = __ballot(rank > 0); left; left &= left - 1) {
      const int at = __builtin_ctzll(left), m = at & 15, j = NW > 1 ? at >> 4 : 0;
      const int r = __builtin_amdgcn_readlane(rank, at), tn = __builtin_amdgcn_readlane(ten, at);
      const T* const A = (const T*)g.ad.A[tn * MILORA_NUM_SITES + g.site[s0] + j];
      const T* const x = (const T*)g.X + (size_t)m * g.ldx;
      const int rpad = pow2_above(r), c = lane & (rpad - 1), kpl = 64 / rpad;
      float sum = 0.f;
      for (int k = k0 + lane / rpad; __any(k < k1); k += 8 * kpl) {
        float xv[8], av[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int kk = k + u * kpl < k1 ? k + u * kpl : d1 - 1;
          xv[u] = Elem<T>::load(x, kk);
          av[u] = Elem<T>::load(A, (size_t)kk * r + (c < r ? c : 0));
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) sum += k + u * kpl < k1 ? xv[u] * av[u] : 0.f;
      }
      for (int off = rpad; off < 64; off <<= 1) sum += __shfl_xor(sum, off, 64);
      if (lane < r) tpart[j][w][m][lane] = sum;
    }
  }
  __syncthreads();
  const int m = tid >> 4, n = n0 + (tid & 15);  // threads 0 .. 255: one output each; their lanes' rows are 4 (tid / 64) ..
  int rm[NW], tm[NW];
#pragma unroll
  for (int j = 0; j < NW; ++j) {
    rm[j] = __shfl(rank, (m & 15) + 16 * j, 64);
    tm[j] = __shfl(ten, (m & 15) + 16 * j, 64);
  }
  if (FUSED && tid < 256) {
    const int c = tid & 15;
#pragma unroll
    for (int j = 0; j < NW; ++j) {
      float s = 0.f;
      if (c < rm[j])
        for (int k = 0; k < kFewW; ++k) s += tpart[j][k][m][c];
      ts[j][m][c] = s;  // (read by the same sixteen lanes)
    }
  }
  __syncthreads();
  if (tid >= 256 || m >= g.M || n >= g.d2) return;

  // ---- bias, LoRA expand, glue, one rounding ----
  float val[NW];
#pragma unroll
  for (int j = 0; j < NW; ++j) {
    float v = 0.f;
#pragma unroll
    for (int k = 0; k < kFewW; ++k) v += red[j][k][m][tid & 15];
    if (g.bias) v += Elem<T>::load((const T*)g.bias, n);
    if (rm[j] > 0) {
      const T* const Bm = (const T*)g.ad.B[tm[j] * MILORA_NUM_SITES + g.site[s0 + j]] + n;
      const float* const tg = FUSED ? nullptr : g.t + ((size_t)(s0 + j) * g.M + m) * g.ad.r_max;
      float delta = 0.f;
      for (int c0 = 0; c0 < rm[j]; c0 += 8) {
        float bv[8], tv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int c = c0 + u < rm[j] ? c0 + u : rm[j] - 1;
          bv[u] = Elem<T>::load(Bm, (size_t)c * g.d2);
          tv[u] = FUSED ? ts[j][m][c & (kFuseRank - 1)] : tg[c];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) delta += c0 + u < rm[j] ? tv[u] * bv[u] : 0.f;
      }
      v += delta;
    }
    val[j] = v;
  }
  if constexpr (MODE == kFewPlain) {
    Elem<T>::store((T*)g.Y[s0], (size_t)m * g.ldy + n, val[0]);
  } else if constexpr (MODE == kFewResid) {
    const size_t i = (size_t)m * g.d2 + n;
    const float h = Elem<T>::load((const T*)g.x_res, i) + round_to<T>(val[0]);
    g.h[i] = h;
    if (g.Y[0]) Elem<T>::store((T*)g.Y[0], i, h);
  } else if constexpr (MODE == kFewGateUp) {
    Elem<T>::store((T*)g.Y[0], (size_t)m * g.ldy + n, silu(round_to<T>(val[0])) * round_to<T>(val[1]));
  } else {
    const size_t i = (size_t)m * g.d2 + n;
    Elem<T>::store((T*)g.Y[0], i, g.h[i] + round_to<T>(val[0]));
  }
}

// ---- more rows ------------------------------------------------------------------------------------------------------
// A workgroup of eight waves computes a BM x BN tile: KQ groups of waves share a stage's k, the waves of a group the tile,
// 32 x 32 each (v_mfma_f32_32x32x2_f32).  Stages go through registers (four on their way) into one of two LDS buffers.
// WIDE (d1 >= 4): every load is four elements without a branch, a row's end read from its last four and shifted when it
// is stored (a branch around the loads makes the compiler wait for all of them at each store: 28.9 us a call of 300 rows on
// 1000 x 2730 without LoRA rows against 27.5 us).
// Bound: the matrix instructions (13.7 us of that call) and the chain of look-ups, t and W^B behind them (10 us where rows
// carry a LoRA term).  Seven fp32 linears of 300 rows, 1000 x 2730: 1757 us with vector FMA out of single-buffered tiles,
// 190 us here.  64 x 64 tiles where they are at least half the compute units, 32 x 32 with the reduction over eight waves
// below (300 rows on 1000 x 1000: 17.6 us).
template <int BM_, int BN_, int KW_>
struct GenCfg {
  static constexpr int BM = BM_, BN = BN_, KW = KW_;                 // KW: k of a stage per wave
  static constexpr int WM = BM / 32, WN = BN / 32, KQ = 8 / (WM * WN);
  static constexpr int SK = KQ * KW, Ld = SK + 4;                    // rows padded: 16 rows at one k hit all banks
  static constexpr int T = 512;
  static constexpr int Items = (BM + BN) * (SK / 4) / T;             // 16-byte pieces of a stage per thread
  static constexpr int BufFloats = (BM + BN) * Ld;
  static constexpr int LdR = BN + 4;
  static constexpr int Outs = BM * BN / T;                           // outputs per thread
  static constexpr int TsOff = KQ * BM * LdR;                        // after the sums: t of the rows, 32 ranks at a time
  static constexpr int LdsBytes = (2 * BufFloats > TsOff + BM * 32 ? 2 * BufFloats : TsOff + BM * 32) * 4;
  static_assert((BM + BN) * (SK / 4) % T == 0 && BM * BN % T == 0 && KW % 8 == 0 && 2 * LdsBytes <= 158 * 1024, "tile shape");
};
typedef GenCfg<32, 32, 16> GenSmall;
typedef GenCfg<64, 64, 32> GenLarge;
constexpr int kGenLargeTiles = 128;

template <typename T, class C, bool WIDE>
__global__ void __launch_bounds__(C::T, 4) linear_tile_kernel(const T* __restrict__ X, int64_t M, int d1, int d2, int col0,
                                                           const int32_t* __restrict__ row_to_req, const T* __restrict__ W,
                                                           const T* __restrict__ bias, AdapterView ad, int site,
                                                           const int32_t* __restrict__ tenant_id,
                                                           const uint8_t* __restrict__ route, int B,
                                                           const float* __restrict__ t, T* __restrict__ Y) {
  extern __shared__ __attribute__((aligned(16))) float buf[];
  __shared__ int s_rank[C::BM], s_ten[C::BM], s_most;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = w / (C::WM * C::WN), wm = w % (C::WM * C::WN) % C::WM, wn = w % (C::WM * C::WN) / C::WM;
  const int64_t m0 = (int64_t)blockIdx.y * C::BM;
  const int n0 = col0 + blockIdx.x * C::BN;

  const T* src[C::Items];
  const int kq = tid % (C::SK / 4) * 4;
  int dst[C::Items];
#pragma unroll
  for (int i = 0; i < C::Items; ++i) {
    const int row = tid / (C::SK / 4) + i * (C::T / (C::SK / 4));
    if (row < C::BM) {
      const int64_t m = m0 + row < M ? m0 + row : M - 1;  // past the edge: the last row again, its results are dropped
      src[i] = X + (size_t)m * d1;
    } else {
      const int n = n0 + row - C::BM < d2 ? n0 + row - C::BM : d2 - 1;
      src[i] = W + (size_t)n * d1;
    }
    dst[i] = row * C::Ld + kq;
  }
  const int stages = (d1 + C::SK - 1) / C::SK;
  constexpr int kSets = 4;
  f32x4 r[kSets][C::Items];
  auto load = [&](int st, f32x4 (&v)[C::Items]) __attribute__((always_inline)) {
    const int k = (st < stages ? st : stages - 1) * C::SK + kq;  // past the end: the last stage again, never stored
#pragma unroll
    for (int i = 0; i < C::Items; ++i) v[i] = WIDE ? load4(src[i] + (k < d1 - 4 ? k : d1 - 4)) : load4_end(src[i], k, d1);
    __builtin_amdgcn_sched_barrier(0);  // the sets in their order: the oldest can then be waited for alone
  };
  auto store = [&](int st, f32x4 (&r)[C::Items]) __attribute__((always_inline)) {
    const int shift = st * C::SK + kq - (d1 - 4);  // k by which a load past d1 - 4 was moved back
    if (WIDE && (st + 1) * C::SK > d1)
#pragma unroll
      for (int i = 0; i < C::Items; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float v = shift <= 0 ? r[i][e] : 0.f;
#pragma unroll
          for (int h = 1; e + h < 4; ++h) v = shift == h ? r[i][e + h] : v;
          r[i][e] = v;
        }
#pragma unroll
    for (int i = 0; i < C::Items; ++i) *reinterpret_cast<f32x4*>(buf + (st & 1) * C::BufFloats + dst[i]) = r[i];
  };
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  const int xo = (wm * 32 + l32) * C::Ld + q * C::KW + lh * 4, wo = (C::BM + wn * 32 + l32) * C::Ld + q * C::KW + lh * 4;
  auto compute = [&](int b) __attribute__((always_inline)) {
    const float* const s = buf + b * C::BufFloats;
#pragma unroll
    for (int k = 0; k < C::KW; k += 8) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(s + xo + k), v = *reinterpret_cast<const f32x4*>(s + wo + k);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(v[e], x[e], acc, 0, 0, 0);
    }
  };
#pragma unroll
  for (int j = 0; j < kSets; ++j) load(j, r[j]);
  if (tid == 0) s_most = 0;
  store(0, r[0]);
  load(kSets, r[0]);
  __syncthreads();
  if (tid < C::BM) {  // which rows carry a LoRA term
    const int64_t m = m0 + tid;
    int tenant = 0, r = 0;
    if (m < M) {
      const int64_t req = row_to_req ? (int64_t)row_to_req[m] : m;
      r = (req >= 0 && req < B) ? routed_rank(ad, tenant_id, route, (int)req, B, site, &tenant) : 0;
    }
    s_rank[tid] = r;
    s_ten[tid] = tenant;
    if (r) atomicMax(&s_most, r);
  }
  for (int s0 = 0; s0 < stages; s0 += kSets) {
#pragma unroll
    for (int j = 0; j < kSets; ++j) {
      const int st = s0 + j;
      if (st >= stages) break;
      compute(j & 1);
      if (st + 1 < stages) store(st + 1, r[(j + 1) % kSets]);
      load(st + 1 + kSets, r[(j + 1) % kSets]);
      __syncthreads();
    }
  }

  // the groups' sums meet in LDS (lane: row l % 32 of the 32 x 32 tile; registers 4 g .. + 3: columns 8 g + 4 (l / 32) ..)
#pragma unroll
  for (int g = 0; g < 4; ++g)
    *reinterpret_cast<f32x4*>(buf + (size_t)(q * C::BM + wm * 32 + l32) * C::LdR + wn * 32 + g * 8 + lh * 4) =
        f32x4{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
  __syncthreads();
  const int nc = tid % C::BN, r0 = tid / C::BN, n = n0 + nc;
  constexpr int kStep = C::T / C::BN;
  const int ns = n < d2 ? n : d2 - 1;
  const float bv = bias ? Elem<T>::load(bias, ns) : 0.f;
  float val[C::Outs];
#pragma unroll
  for (int i = 0; i < C::Outs; ++i) {
    float v = 0.f;
#pragma unroll
    for (int k = 0; k < C::KQ; ++k) v += buf[(size_t)(k * C::BM + r0 + i * kStep) * C::LdR + nc];
    val[i] = v + bv;
  }

  // LoRA expand, 32 ranks at a time; eight rows of W^B for all of a thread's outputs on their way together (one output after
  // the other, each waited for its own loads: 43.4 us a call of 300 rows on 1000 x 2730 against 37.8 us)
  const int most = s_most;
  float* const ts = buf + C::TsOff;
  if (most > 0) {
    const T* Bm[C::Outs];
    int last[C::Outs];
#pragma unroll
    for (int i = 0; i < C::Outs; ++i) {
      const int row = r0 + i * kStep;
      last[i] = s_rank[row] - 1;
      Bm[i] = last[i] >= 0 ? (const T*)ad.B[s_ten[row] * MILORA_NUM_SITES + site] + ns : nullptr;
    }
    for (int c0 = 0; c0 < most; c0 += 32) {
      for (int e = tid; e < C::BM * 32; e += C::T) {
        const int row = e >> 5, c = c0 + (e & 31);
        ts[e] = c < s_rank[row] ? t[(size_t)(m0 + row) * ad.r_max + c] : 0.f;
      }
      __syncthreads();
      for (int c1 = 0; c1 < 32 && c0 + c1 < most; c1 += 8) {
        float b[C::Outs][8];
#pragma unroll
        for (int i = 0; i < C::Outs; ++i)
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int c = c0 + c1 + u;
            b[i][u] = c <= last[i] ? Elem<T>::load(Bm[i], (size_t)c * d2) : 0.f;
          }
#pragma unroll
        for (int i = 0; i < C::Outs; ++i)
#pragma unroll
          for (int u = 0; u < 8; ++u) val[i] += ts[(r0 + i * kStep) * 32 + c1 + u] * b[i][u];
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int i = 0; i < C::Outs; ++i) {
    const int64_t m = m0 + r0 + i * kStep;
    if (m < M && n < d2) Elem<T>::store(Y, (size_t)m * d2 + n, val[i]);
  }
}

template <typename T, class C, bool WIDE>
int launch_tile(const void* X, int64_t M, int d1, int d2, const int32_t* row_to_req, const void* W, const void* bias,
                const AdapterView& ad, int site, const int32_t* tenant_id, const uint8_t* route, int B, const float* t, void* Y,
                hipStream_t stream) {
  static thread_local int lds_set_for = -1;
  int dev = 0;
  MILORA_HIP(hipGetDevice(&dev));
  if (lds_set_for != dev) {
    MILORA_HIP(hipFuncSetAttribute((const void*)linear_tile_kernel<T, C, WIDE>, hipFuncAttributeMaxDynamicSharedMemorySize, C::LdsBytes));
    lds_set_for = dev;
  }
  int rc = MILORA_OK;
  for (int64_t col0 = 0; col0 < d2 && !rc; col0 += kLaunchCols) {
    const int cols = d2 - col0 < kLaunchCols ? (int)(d2 - col0) : kLaunchCols;
    dim3 grid((unsigned)((cols + C::BN - 1) / C::BN), (unsigned)((M + C::BM - 1) / C::BM));
    hipLaunchKernelGGL((linear_tile_kernel<T, C, WIDE>), grid, dim3(C::T), C::LdsBytes, stream, (const T*)X, M, d1, d2, (int)col0,
                       row_to_req, (const T*)W, (const T*)bias, ad, site, tenant_id, route, B, t, (T*)Y);
    rc = check_launch();
  }
  return rc;
}

}  // namespace

int launch_shrink(const void* X, int64_t ldx, int64_t M, int d1, int dtype, const int32_t* row_to_req, const AdapterView& ad,
                  int site, int sites, const int32_t* tenant_id, const uint8_t* route, int B, float* t, hipStream_t stream) {
  if (dtype == MILORA_BF16)
    hipLaunchKernelGGL((shrink_rows_kernel<bf16_t>), dim3((unsigned)M, sites), dim3(kShrinkT), 0, stream, (const bf16_t*)X,
                       ldx, M, d1, row_to_req, ad, site, tenant_id, route, B, t);
  else
    hipLaunchKernelGGL((shrink_rows_kernel<float>), dim3((unsigned)M, sites), dim3(kShrinkT), 0, stream, (const float*)X, ldx,
                       M, d1, row_to_req, ad, site, tenant_id, route, B, t);
  return check_launch();
}

template <typename T, int W, bool FUSED>
static int launch_few_rows_t(FewArgs& g, int sites, int mode, hipStream_t st) {
  int rc = MILORA_OK;
  for (int64_t col0 = 0; col0 < g.d2 && !rc; col0 += kLaunchCols) {
    const int cols = g.d2 - col0 < kLaunchCols ? (int)(g.d2 - col0) : kLaunchCols;
    const dim3 grid((unsigned)((cols + 15) / 16), (unsigned)sites);
    g.col0 = (int)col0;
    switch (mode) {
      case kFewPlain: hipLaunchKernelGGL((few_rows_kernel<T, kFewPlain, W, FUSED>), grid, dim3(W * 64), 0, st, g); break;
      case kFewResid: hipLaunchKernelGGL((few_rows_kernel<T, kFewResid, W, FUSED>), grid, dim3(W * 64), 0, st, g); break;
      case kFewGateUp: hipLaunchKernelGGL((few_rows_kernel<T, kFewGateUp, W, FUSED>), dim3(grid.x), dim3(W * 64), 0, st, g); break;
      default: hipLaunchKernelGGL((few_rows_kernel<T, kFewDown, W, FUSED>), grid, dim3(W * 64), 0, st, g); break;
    }
    rc = check_launch();
  }
  return rc;
}

// Shrinks inside the launch spare one of its own (3 to 4 us) and cost every wave about 0.7 us per routed row and round trip, a trip
// taking d1 / 8 x rank in pieces of 64 lanes x 8 loads.  With every row routed the two meet at some 10 trips (fp32, 8 rows, 512 x
// 1376, rank 8: 11.3 us a call inside, 12.7 apart; 8 rows, 1000 x 2730: 16.6 and 13.2; 16 rows, 4100 x 11010, rank 16: 306 and
// 59).  In a layer's step a request has one of the seven sites, or a few: there it is some 45 trips of all rows (16 rows, d = 512,
// rank 8, 16 trips and 42 of the down projection: 40.2 and 45.3 us a step; d = 1000, rank 8, 31 and 85: 61.6 and 63.0; rank 16, 62 and
// 171: 80.6 and 70.0).
// (A trip is one of eight waves; four, where few_waves takes them, make one trip of a row's shrink as well.  The calls were made one
// by one from the host, where a second launch costs most; replayed from a graph the two meet sooner, fp32, 512 x 1359, rank 8: 4 rows
// 7.2 us inside and 7.2 apart, 8 rows 10.3 and 7.7, 16 rows 16.3 and 8.0.)
static int64_t shrink_work(int d1, int r_max) {  // of one row, in products
  int rpad = 1;
  while (rpad < r_max) rpad <<= 1;
  return (int64_t)d1 * rpad;
}
static constexpr int64_t shrink_trip(int waves) { return waves * 64 * 8; }

static bool fuse_shrink(int M, int d1, int r_max, bool layer) {
  if (r_max > kFuseRank) return false;
  const int64_t trip = shrink_trip(8), work = shrink_work(d1, r_max);
  return M * (work > trip ? work : trip) <= (layer ? 48 : 16) * trip;
}

// Waves of a launch with the shrinks inside.  Four where eight would each find two blocks of 16 k or fewer and where four form a
// row's shrink in one trip too: fp32, 1359 columns, all rows routed, d1 = 256: rank 8, 1, 8 and 16 rows 4.2, 8.8 and 14.3 us with four and
// 4.7, 10.2 and 16.1 with eight; d1 = 288: 4.6, 11.0, 18.3 and 4.7, 10.0, 16.2; rank 16, 343 columns, d1 = 200, 16 rows: 17.8 and
// 15.2.  Few rows of a layer's step, most of them without a term at a given site, take four up to any rank: d = 256, rank 16, 1 and
// 4 rows 16.9 and 21.4 us a step, 18.6 and 22.8 with eight; 16 rows with three sites each 55.6 and 52.0.
static int few_waves(int M, int d1, int r_max, bool layer) {
  return d1 <= kFewNarrow && (shrink_work(d1, r_max) <= shrink_trip(4) || (layer && M <= 4)) ? 4 : 8;
}

int launch_few_rows(const FewArgs& args, int dtype, int sites, int mode, float* t, hipStream_t st) {
  FewArgs g = args;
  g.t = nullptr;
  const bool layer = sites > 1 || mode != kFewPlain;
  if (!fuse_shrink(g.M, g.d1, g.ad.r_max, layer)) {
    const int rc = launch_shrink(g.X, g.ldx, g.M, g.d1, dtype, g.row_to_req, g.ad, g.site[0], sites, g.tenant_id, g.route, g.B, t, st);
    if (rc) return rc;
    g.t = t;
  }
  const bool bf = dtype == MILORA_BF16;
  if (g.t) return bf ? launch_few_rows_t<bf16_t, 8, false>(g, sites, mode, st) : launch_few_rows_t<float, 8, false>(g, sites, mode, st);
  if (few_waves(g.M, g.d1, g.ad.r_max, layer) == 4) return bf ? launch_few_rows_t<bf16_t, 4, true>(g, sites, mode, st) : launch_few_rows_t<float, 4, true>(g, sites, mode, st);
  return bf ? launch_few_rows_t<bf16_t, 8, true>(g, sites, mode, st) : launch_few_rows_t<float, 8, true>(g, sites, mode, st);
}

int launch_linear_generic(const void* X, int64_t M, int d1, int d2, int dtype, const int32_t* row_to_req,
                          const void* W, const void* bias, const AdapterView& ad, int site,
                          const int32_t* tenant_id, const uint8_t* route, int B, float* t, void* Y, hipStream_t stream) {
  if ((M + 63) / 64 > 65535) return MILORA_ERANGE;
  if (M <= kFewRows) {
    FewArgs g{};
    g.X = X; g.ldx = d1; g.M = (int)M; g.d1 = d1; g.d2 = d2;
    g.W[0] = W; g.bias = bias; g.Y[0] = Y; g.ldy = d2; g.site[0] = site;
    g.row_to_req = row_to_req; g.tenant_id = tenant_id; g.route = route; g.B = B; g.ad = ad;
    return launch_few_rows(g, dtype, 1, kFewPlain, t, stream);
  }
  const int rc = launch_shrink(X, d1, M, d1, dtype, row_to_req, ad, site, 1, tenant_id, route, B, t, stream);
  if (rc) return rc;
  const int64_t large = ((M + 63) / 64) * (int64_t)((d2 + 63) / 64);
#define MILORA_TILE(T, C, WIDE) \
  launch_tile<T, C, WIDE>(X, M, d1, d2, row_to_req, W, bias, ad, site, tenant_id, route, B, t, Y, stream)
  const bool bf = dtype == MILORA_BF16;
  if (d1 < 4) return bf ? MILORA_TILE(bf16_t, GenLarge, false) : MILORA_TILE(float, GenLarge, false);
  if (large >= kGenLargeTiles) return bf ? MILORA_TILE(bf16_t, GenLarge, true) : MILORA_TILE(float, GenLarge, true);
  return bf ? MILORA_TILE(bf16_t, GenSmall, true) : MILORA_TILE(float, GenSmall, true);
#undef MILORA_TILE
}

}  // namespace milora
