// Routed LoRA linears on bf16 for few to some thousand rows (paper Eq. 1 with the layer-level gate of Sec. 3.3), on
// row-major or packed base weights: Y = X W + bias + (X W^A) W^B for the rows whose request is routed to this site.
//
// One workgroup of eight waves computes a BM x BN tile of Y over one part of the reduction with the bf16 matrix cores
// (v_mfma_f32_32x32x16_bf16).  X rows and W come through LDS: whole 128-byte lines of 64 k (packed weights: their 1 KiB
// operand blocks as they lie) are copied straight from global memory (global_load_lds_dwordx4) into a ring of NS
// stages, NS - 1 of them on their way while one is multiplied, one barrier per stage.  The waves split a stage's 64 k
// among KQ groups of waves and the tile among the waves of a group: a wave then holds a large piece of the tile (few
// operand reads per matrix instruction) although eight waves share it.  The groups' sums meet in LDS at the end.
//
// Few rows leave few tiles: the reduction is then cut into S parts, one workgroup each, so that every compute unit
// streams weights.  A workgroup stores its partial tile (written through) and counts itself in; the one that comes last
// adds the parts in part order and finishes the tile.  Nobody waits for anybody, so any number of workgroups may
// be resident, and the sums do not depend on timing.  The shrink's launch zeroes the counters.
//
// The LoRA term of the routed rows (t = X W^A is computed beforehand, in fp32) enters in one of two ways.  ROWS: after the matrix
// work every thread adds t W^B of its own outputs in fp32, the ranks dealt to the parts; what one tenant's adapter holds, Inf and NaN
// too, reaches that tenant's rows only.  This serves packed weights and calls of fewer than 64 rows, where rows of many tenants
// meet.  Else as more stages of the matrix work: t split into two bf16 halves (hi + lo, about 17 bits of it) against
// W^B, the rows of other tenants entering as zeros (Inf and NaN of W^B are kept out and added for their own rows behind
// the stages).  Then bias, one rounding, 16-byte stores.
//
// Bound: few rows, the stream of the weights (a 4096 x 11008 linear at 45 rows: 23 us = 3.9 TB/s); from some hundred rows on
// the copies through the L2 (0.58 us per 128 x 128 x 64 stage and compute unit, 56 GB/s each).  The seven linears of the 7B
// layer: 45 rows 4940 us with the any-shape kernel, 158 us here; 777 rows 966 us with 256 x 256 tiles only, 472 us;
// packed weights, 96 rows, three sites a request: 495 us with the stream kernel of decode.hip, 250 us.
#include "shrink.h"
#include "tiles.h"

namespace milora {
namespace {

typedef uint32_t u32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));
typedef uint32_t u32x4_a2 __attribute__((ext_vector_type(4), aligned(2)));
typedef __attribute__((address_space(1))) const u32x4_a2 gu32x4_a2;
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kT = 512;        // threads: eight waves
constexpr int kCtlBytes = 4096;
constexpr int kMaxGroups = 256;  // groups of 8 ranks of the LoRA phase listed at a time
constexpr int kGroupM = 6;
constexpr int kCtlBad = 4;  // control word: W^B holds Inf or NaN
constexpr int kTs = MILORA_MAX_RANK + 4;  // t of a row in LDS

template <int BM_, int BN_, int KQ_, int WMC_, int WNC_, int NS_, int OCC_>
struct TileCfg {
  static constexpr int BM = BM_, BN = BN_, KQ = KQ_, WMC = WMC_, WNC = WNC_, NS = NS_, OCC = OCC_;
  static constexpr int TM = BM / WMC / 32, TN = BN / WNC / 32;  // 32 x 32 tiles of a wave
  static constexpr int KS = 4 / KQ;                             // 16-k sub-steps of a stage per wave
  static constexpr int CPW = (BM + BN) / 8 / 8;                 // copy instructions of a stage per wave (8 lines each)
  static constexpr int StageBytes = (BM + BN) * 128;
  static constexpr int Ld = BN + 4;                             // fp32 row of the sums in LDS, padded against bank conflicts
  static constexpr int Items = BM * BN / 8 / kT;                // pieces of 8 columns per thread at the end
  static constexpr int RedBytes = KQ * BM * Ld * 4;
  static constexpr int RingBytes = NS * StageBytes;
  static constexpr int LdsBytes = kCtlBytes + (RedBytes > RingBytes ? RedBytes : RingBytes);
  static_assert(BM * kTs * 4 <= LdsBytes - kCtlBytes, "t of the tile's rows");
  static_assert(KQ * WMC * WNC == 8 && (BM + BN) % 64 == 0 && BM * BN % (8 * kT) == 0, "tile shape");
  static_assert(CPW * (NS - 2) < 63 && LdsBytes * OCC <= 160 * 1024 && BM * 12 + kMaxGroups * 8 + 64 <= kCtlBytes, "resources");
};
typedef TileCfg<64, 64, 4, 2, 1, 4, 2> CfgSmall;
typedef TileCfg<128, 128, 2, 2, 2, 4, 1> CfgMid;

struct TParams {
  const bf16_t* X;
  const bf16_t* W;
  const bf16_t* bias;
  bf16_t* Y;
  const float* t;  // partial shrinks [part][M][r_max], to be added in part order
  size_t t_stride;
  int parts;
  const int32_t* row_to_req;
  const int32_t* tenant_id;
  const uint8_t* route;
  AdapterView ad;
  int64_t M;
  const int2* row_lora;  // [M], ROWS: tenant and rank of each row, from the shrink's look-ups (one load instead of a chain of four)
  int d1, d2, site, B;
  int tilesM, tilesN;
  int S, steps;    // parts of the reduction and stages (64 k) per part
  float* partial;  // [tile][part][BM * BN] partial tiles, in the order the finishing threads take them
  int* cnt;        // [tile] parts stored so far
};

// Which of the eight 16-byte pieces of its 128-byte LDS line holds k group kg of row r (mod 16): kg ^ swz(r).  Eight
// neighbouring rows get eight different pieces, and rows r and r + 8 differ too, so a 16-byte operand read of 16 rows at
// one k group touches every bank once.
__device__ __forceinline__ int swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

template <int N>
__device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0f70);
}

template <class C, bool PK, bool ROWS>
__global__ void __launch_bounds__(kT, 2 * C::OCC) tile_kernel(const TParams p) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  int* const row_ten = reinterpret_cast<int*>(lds);   // [BM] tenant of each row of the tile, -1: no LoRA term
  int* const row_rank = row_ten + C::BM;              // [BM]
  int* const row_group = row_rank + C::BM;            // [BM] first rank group of the row's run
  int2* const groups = reinterpret_cast<int2*>(row_group + C::BM);  // [kMaxGroups] tenant, first rank
  int* const ctl = reinterpret_cast<int*>(groups + kMaxGroups);     // 0: arrivals before this one, 1, 2: rows with a LoRA term, kCtlBad
  int* const row_c0 = row_rank;    // (ROWS) [BM] first rank of the row in this part
  int* const row_cnt = row_group;  // (ROWS) [BM] ranks of the row in this part
  unsigned char* const ring = lds + kCtlBytes;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

  // workgroup -> (part, column tile, row tile): workgroup ids go round-robin over the 8 XCDs; each XCD takes a contiguous
  // run of an order that walks kGroupM row tiles of one column tile before the next column tile, so that its L2
  // serves the re-reads of both operands (32 workgroups of an XCD then cover about 6 row tiles x 6 column tiles)
  const int total = p.tilesM * p.tilesN * p.S;
  const int per = (total + 7) >> 3;
  const int id = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (id >= total) return;
  const int tile = id % (p.tilesM * p.tilesN), part = id / (p.tilesM * p.tilesN);
  const int first = tile / (kGroupM * p.tilesN) * kGroupM;
  const int gsz = p.tilesM - first < kGroupM ? p.tilesM - first : kGroupM;
  const int in_group = tile % (kGroupM * p.tilesN);
  const int64_t m0 = (int64_t)(first + in_group % gsz) * C::BM;
  const int n0 = in_group / gsz * C::BN;

  const int KT = (p.d1 + 63) >> 6;
  const int kt0 = part * p.steps, n_steps = KT - kt0 < p.steps ? KT - kt0 : p.steps;

  // ---- copies: instruction i of a stage brings lines 8 i .. 8 i + 7 (X rows first, then W columns) ----
  const size_t row_bytes = (size_t)p.d1 * 2;
  const unsigned char* const xb = (const unsigned char*)p.X + (size_t)m0 * row_bytes;
  const unsigned char* const wb = (const unsigned char*)p.W + (PK ? (size_t)(n0 >> 4) * (p.d1 >> 5) * 1024 : (size_t)n0 * row_bytes);
  const int rows = p.M - m0 < C::BM ? (int)(p.M - m0) : C::BM;
  const int cols = p.d2 - n0 < C::BN ? p.d2 - n0 : C::BN;
  uint32_t voff[C::CPW];
  bool isw[C::CPW];
#pragma unroll
  for (int j = 0; j < C::CPW; ++j) {
    const int i = w * C::CPW + j;
    isw[j] = i >= C::BM / 8;
    const int line = isw[j] ? i - C::BM / 8 : i;
    const int rr = lane >> 3;
    if (PK && isw[j]) {
      int blk = line >> 1;
      blk = blk < (cols >> 4) ? blk : (cols >> 4) - 1;
      voff[j] = ((uint32_t)blk * (uint32_t)(p.d1 >> 5) + (uint32_t)(line & 1)) * 1024u + (uint32_t)lane * 16u;
    } else {
      int r = line * 8 + rr;
      const int lim = isw[j] ? cols : rows;
      r = r < lim ? r : lim - 1;  // past the edge: the last line again, its results are dropped
      voff[j] = (uint32_t)((uint32_t)r * (uint32_t)row_bytes) + (uint32_t)(((lane & 7) ^ swz(((line & 1) << 3) + rr)) << 4);
    }
  }
  const uint32_t ring0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)ring;
  auto issue = [&](int st, int slot) __attribute__((always_inline)) {
    const int kt = kt0 + (st < n_steps ? st : n_steps - 1);  // past the end: the last stage again, into a slot nobody reads
    const bool half = PK && (kt + 1) * 64 > p.d1;            // the last 32 k of a reduction that is no multiple of 64
#pragma unroll
    for (int j = 0; j < C::CPW; ++j) {
      const uint32_t dst = ring0 + slot * C::StageBytes + (w * C::CPW + j) * 1024;
      const unsigned char* b = isw[j] ? wb + (size_t)kt * (PK ? 2048 : 128) : xb + (size_t)kt * 128;
      uint32_t v = voff[j];
      if (half) {  // the k past the end are not multiplied: read valid memory in their place
        const int line = isw[j] ? w * C::CPW + j - C::BM / 8 : w * C::CPW + j;
        if (isw[j]) v -= (line & 1) ? 1024u : 0u;
        else v -= (((lane & 7) ^ swz(((line & 1) << 3) + (lane >> 3))) & 4) ? 64u : 0u;
      }
      copy_to_lds16(b, v, dst);
    }
  };

  // ---- this wave's part: k group q of the stage, rows wm, columns wn of the tile ----
  const int q = w / (C::WMC * C::WNC), sp = w % (C::WMC * C::WNC), wm = sp % C::WMC, wn = sp / C::WMC;
  const int l32 = lane & 31, lh = lane >> 5;
  f32x16 acc[C::TM][C::TN];
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  int xrd[C::KS], wrd[C::KS];
#pragma unroll
  for (int s = 0; s < C::KS; ++s) {
    const int ks = q * C::KS + s;
    const int sw = ((2 * ks + lh) ^ swz(l32 & 15)) << 4;
    xrd[s] = (wm * (C::BM / C::WMC) + l32) * 128 + sw;
    const int n = wn * (C::BN / C::WNC) + l32;
    wrd[s] = C::BM * 128 + (PK ? ((n >> 4) * 2 + (ks >> 1)) * 1024 + ((n & 15) + 16 * ((ks & 1) * 2 + lh)) * 16 : n * 128 + sw);
  }

  // one 16-k sub-step of the wave's part
  auto mma = [&](const unsigned char* sb, int xo, int wo) __attribute__((always_inline)) {
    bf16x8 a[C::TM], b[C::TN];
#pragma unroll
    for (int i = 0; i < C::TM; ++i) a[i] = *(const bf16x8*)(sb + xo + i * 4096);
#pragma unroll
    for (int j = 0; j < C::TN; ++j) b[j] = *(const bf16x8*)(sb + wo + j * 4096);
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
      for (int j = 0; j < C::TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
  };

#pragma unroll
  for (int s = 0; s < C::NS - 1; ++s) issue(s, s);
  // which rows carry a LoRA term (looked up while the first stages are on their way)
  const bool with_lora = part == p.S - 1;
  if ((ROWS || with_lora) && tid < C::BM) {
    if constexpr (ROWS) {
      const int2 ten_rank = tid < rows ? p.row_lora[m0 + tid] : int2{-1, 0};
      const int r = ten_rank.y;
      const int ng = (r + 7) >> 3, c0 = part * ng / p.S * 8, c1 = (part + 1) * ng / p.S * 8, cnt = (c1 < r ? c1 : r) - c0;
      row_ten[tid] = ten_rank.x;
      row_c0[tid] = c0;
      row_cnt[tid] = cnt > 0 ? cnt : 0;
      int most = cnt;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_xor(most, off, 64);
        most = o > most ? o : most;
      }
      if (lane == 0) ctl[1 + w] = most;
    } else {
      int tenant = -1, r = 0;
      if (tid < rows) {
        const int64_t m = m0 + tid;
        const int64_t req = p.row_to_req ? (int64_t)p.row_to_req[m] : m;
        r = (req >= 0 && req < p.B) ? routed_rank(p.ad, p.tenant_id, p.route, (int)req, p.B, p.site, &tenant) : 0;
      }
      row_ten[tid] = r ? tenant : -1;
      row_rank[tid] = r;
      const unsigned long long any = __ballot(r > 0);
      if (lane == 0) ctl[1 + w] = any != 0;
      if (tid == 0) ctl[kCtlBad] = 0;
    }
  }
  int slot = 0;
  for (int st = 0; st < n_steps; ++st) {
    wait_vm<C::CPW * (C::NS - 2)>();     // this wave's copies of stage st have landed
    __builtin_amdgcn_s_waitcnt(0xc07f);  // its operand reads of the stage before are done
    __builtin_amdgcn_s_barrier();        // the same for every wave
    asm volatile("" ::: "memory");
    issue(st + C::NS - 1, slot == 0 ? C::NS - 1 : slot - 1);
    const unsigned char* sb = ring + slot * C::StageBytes;
#pragma unroll
    for (int s = 0; s < C::KS; ++s) {
      if (PK && (kt0 + st) * 64 + (q * C::KS + s) * 16 >= p.d1) break;
      mma(sb, xrd[s], wrd[s]);
    }
    asm volatile("" ::: "memory");
    slot = slot + 1 == C::NS ? 0 : slot + 1;
  }
  wait_vm<0>();
  __syncthreads();

  // ---- LoRA term of the routed rows (by the workgroup of the last part): more stages of 64 k -----------------------
  // A stage takes four groups of 8 ranks, and as many stages as the ring holds are filled together (one round trip for t and
  // W^B instead of one per stage: 777 rows of 5 requests, ranks 8 to 64, 4096 x 4096: 47.8 -> 46.0 us a call).  t = X W^A (fp32)
  // enters as bf16 hi + lo, hi against the groups' rows of W^B in the first 32 k, lo against the same rows in the second.
  // Consecutive rows of one tenant are a run; a run's ranks get groups of their own, in which the other rows of the tile are
  // zero, so tenants share stages.
  bool lora = false;
  if (!ROWS && with_lora)
#pragma unroll
    for (int i = 0; i < C::BM / 64; ++i) lora = lora || ctl[1 + i];
  if (lora) {
    int n_groups = 0;
    for (int g0 = 0;; g0 += kMaxGroups) {
      if (w == 0) {  // list groups g0 .. g0 + kMaxGroups - 1
        int base = 0;
        for (int b0 = 0; b0 < C::BM; b0 += 64) {
          const int i = b0 + lane, ten = row_ten[i], prev = i > 0 ? row_ten[i - 1] : -1;
          const int ng = ten >= 0 && ten != prev ? (row_rank[i] + 7) >> 3 : 0;  // a run begins here
          int sum = ng;
#pragma unroll
          for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(sum, off, 64);
            sum += lane >= off ? o : 0;
          }
          // (the last run's first group: rows inside a run take it from its first row, which has the largest index so far)
          int first = ng ? base + sum - ng : -1;
          for (int k = 0; k < ng; ++k)
            if (first + k >= g0 && first + k < g0 + kMaxGroups) groups[first + k - g0] = int2{ten, k * 8};
#pragma unroll
          for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(first, off, 64);
            first = lane >= off && o > first ? o : first;
          }
          if (b0 > 0 && first < 0) first = row_group[b0 - 1];
          row_group[i] = first;
          base += __shfl(sum, 63, 64);
        }
        if (lane == 0) ctl[0] = base;
      }
      __syncthreads();
      n_groups = ctl[0];
      const int g1 = n_groups < g0 + kMaxGroups ? n_groups : g0 + kMaxGroups;
      // X side: a row's groups by kRowT threads; W side: (8 columns, group) by thread
      constexpr int kBatch = C::NS * 4, kRowT = kT / C::BM, kPieces = C::BN / 8;
      static_assert(kPieces * kBatch <= kT && kT % C::BM == 0, "one piece of W^B per thread");
      for (int s0 = g0; s0 < g1; s0 += kBatch) {
        int tb = tid;  // opaque: addresses formed from it stay inside the loop instead of being spilled in front of it
        asm volatile("" : "+v"(tb));
        const int xr = tb / kRowT;
        const int my_first = row_group[xr], my_rank = row_ten[xr] >= 0 ? row_rank[xr] : 0;
        const int wc = tb % kPieces * 8, wg = tb / kPieces;
        const bool tvec = (p.ad.r_max & 3) == 0;
        constexpr int kFly = C::OCC == 1 ? 4 : 2;  // parts in flight: registers of half a compute unit allow two
        auto ask_t = [&](int c0, int k0, f32x4 (&v)[2][kFly]) __attribute__((always_inline)) {  // parts k0 .. of ranks c0 .. c0 + 7 of row xr
          const float* tp = p.t + (size_t)(m0 + xr) * p.ad.r_max + c0;
#pragma unroll
          for (int k = 0; k < kFly; ++k)
#pragma unroll
            for (int h = 0; h < 2; ++h)
              v[h][k] = *reinterpret_cast<const f32x4*>(tp + (k0 + k < p.parts ? k0 + k : p.parts - 1) * p.t_stride + h * 4);
        };
        auto add_t = [&](int k0, const f32x4 (&v)[2][kFly], float (&tv)[8]) __attribute__((always_inline)) {
#pragma unroll
          for (int k = 0; k < kFly; ++k)
            if (k0 + k < p.parts)
#pragma unroll
              for (int e = 0; e < 8; ++e) tv[e] += v[e >> 2][k][e & 3];
        };
        auto load_t = [&](int c0, int k0, float (&tv)[8]) __attribute__((always_inline)) {  // the parts from k0 on
          if (tvec && c0 + 8 <= my_rank) {
            for (; k0 < p.parts; k0 += kFly) {
              f32x4 v[2][kFly];
              ask_t(c0, k0, v);
              add_t(k0, v, tv);
            }
          } else {
            const float* tp = p.t + (size_t)(m0 + xr) * p.ad.r_max + c0;
            for (int e = 0; e < 8; ++e)
              if (c0 + e < my_rank)
                for (int k = 0; k < p.parts; ++k) tv[e] += tp[k * p.t_stride + e];
          }
        };
        auto put_t = [&](int group, const float (&tv)[8]) __attribute__((always_inline)) {  // group of the batch
          u32x4 hi, lo;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const bf16_t h0 = f32_to_bf16(tv[2 * e]), h1 = f32_to_bf16(tv[2 * e + 1]);
            hi[e] = (uint32_t)h0 | ((uint32_t)h1 << 16);
            lo[e] = pack_bf16x2(tv[2 * e] - bf16_to_f32(h0), tv[2 * e + 1] - bf16_to_f32(h1));
          }
          unsigned char* const row = ring + (group >> 2) * C::StageBytes + xr * 128;
          *reinterpret_cast<u32x4*>(row + (((group & 3) ^ swz(xr & 15)) << 4)) = hi;
          *reinterpret_cast<u32x4*>(row + ((((group & 3) + 4) ^ swz(xr & 15)) << 4)) = lo;
        };
        const int stages = ((g1 - s0 < kBatch ? g1 - s0 : kBatch) + 3) >> 2;
        // this thread's groups of the row in this batch: k, k + kRowT, ... < k_end (counted from the row's first)
        const int off = s0 - my_first, end = g1 - my_first < off + kBatch ? g1 - my_first : off + kBatch;
        const int ng = (my_rank + 7) >> 3, k_end = end < ng ? end : ng;
        int k = (off > 0 ? off : 0) + tb % kRowT;
        const bool has = k < k_end;
        // One workgroup per compute unit: the first two groups of t and W^B on their way together, a round trip takes about 3 us
        // (777 rows on 4096 x 4096: 52.8 us a call one after the other, 51.9 so).  Two share its registers: W^B and t one after the other.
        float tv[C::OCC == 1 ? 2 : 1][8];
        f32x4 raw[2][2][kFly];
        bool whole[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          whole[j] = C::OCC == 1 && tvec && k + j * kRowT < k_end && (k + j * kRowT) * 8 + 8 <= my_rank;
          if (whole[j]) ask_t((k + j * kRowT) * 8, 0, raw[j]);
        }
        u32x4 a[8];
        const bool wput = wg < stages * 4;
        auto guard_w = [&]() __attribute__((always_inline)) {
          float bad[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) bad[e] = taint(bad[e], a[i][e]);
          if ((bad[0] + bad[1]) + (bad[2] + bad[3]) != 0.f) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
              for (int e = 0; e < 4; ++e) a[i][e] = finite2(a[i][e]);
            ctl[kCtlBad] = 1;
          }
        };
#pragma unroll
        for (int i = 0; i < 8; ++i) a[i] = u32x4{0u, 0u, 0u, 0u};
        if (wput && s0 + wg < g1 && wc < cols) {
          const int2 gr = groups[s0 + wg - g0];
          const int r = p.ad.rank[gr.x];
          gbf16* b = in_global(p.ad.B[gr.x * MILORA_NUM_SITES + p.site]) + n0 + wc;
          // (whole pieces of 8 columns, d2 % 16 == 0, at whatever alignment the adapter has: one load each)
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (gr.y + i < r) a[i] = *(gu32x4_a2*)(b + (size_t)(gr.y + i) * p.d2);
          if (C::OCC > 1) guard_w();
        }
        auto put_w = [&]() __attribute__((always_inline)) {
          if (C::OCC == 1) guard_w();
          u32x4 at[8];
          transpose8(a, at);
          unsigned char* const wst = ring + (wg >> 2) * C::StageBytes + C::BM * 128;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int n = wc + j;
            *reinterpret_cast<u32x4*>(wst + n * 128 + (((wg & 3) ^ swz(n & 15)) << 4)) = at[j];
            *reinterpret_cast<u32x4*>(wst + n * 128 + ((((wg & 3) + 4) ^ swz(n & 15)) << 4)) = at[j];
          }
        };
        if (C::OCC > 1 && wput) put_w();
        if (C::OCC > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < (C::OCC == 1 ? 2 : 1); ++j) {
#pragma unroll
          for (int e = 0; e < 8; ++e) tv[j][e] = 0.f;
          if (whole[j]) add_t(0, raw[j], tv[j]);
          if (k + j * kRowT < k_end) load_t((k + j * kRowT) * 8, whole[j] ? kFly : 0, tv[j]);
        }
        for (int e = tb; e < stages * C::BM * 8; e += kT)
          *reinterpret_cast<u32x4*>(ring + e / (C::BM * 8) * C::StageBytes + e % (C::BM * 8) * 16) = u32x4{0u, 0u, 0u, 0u};
        __syncthreads();
        if (has) put_t(k - off, tv[0]);
        if (C::OCC == 1 && k + kRowT < k_end) put_t(k + kRowT - off, tv[C::OCC == 1 ? 1 : 0]);
        for (k += kRowT * (C::OCC == 1 ? 2 : 1); k < k_end; k += kRowT) {
#pragma unroll
          for (int e = 0; e < 8; ++e) tv[0][e] = 0.f;
          load_t(k * 8, 0, tv[0]);
          put_t(k - off, tv[0]);
        }
        if (C::OCC == 1 && wput) put_w();
        __syncthreads();
        for (int st = 0; st < stages; ++st)
#pragma unroll
          for (int s = 0; s < C::KS; ++s) {
            const int ks = q * C::KS + s;
            const int n = wn * (C::BN / C::WNC) + l32;
            mma(ring + st * C::StageBytes, xrd[s], C::BM * 128 + n * 128 + (((2 * ks + lh) ^ swz(l32 & 15)) << 4));
          }
        __syncthreads();
      }
      if (g1 == n_groups) break;
    }
  }

  // ---- the groups' sums meet in LDS; a thread takes pieces of 8 columns: column piece cg, rows r0, r0 + kRowStep, ... ----
  // (of a 32 x 32 tile a lane holds row l % 32 and, in registers 4 g .. 4 g + 3, the columns 8 g + 4 (l / 32) .. + 3)
  float* const red = reinterpret_cast<float*>(ring);
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int m = wm * (C::BM / C::WMC) + i * 32 + l32, n = wn * (C::BN / C::WNC) + j * 32 + g * 8 + lh * 4;
        *reinterpret_cast<f32x4*>(red + ((size_t)q * C::BM + m) * C::Ld + n) =
            f32x4{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
      }
  constexpr int kGroups = C::BN / 8, kRowStep = kT / kGroups;
  const int cg = tid % kGroups, r0 = tid / kGroups;
  __syncthreads();
  f32x4 val[C::Items][2];
#pragma unroll
  for (int it = 0; it < C::Items; ++it)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float* e = red + (size_t)(r0 + it * kRowStep) * C::Ld + cg * 8 + h * 4;
      f32x4 v = *reinterpret_cast<const f32x4*>(e);
#pragma unroll
      for (int k = 1; k < C::KQ; ++k) v += *reinterpret_cast<const f32x4*>(e + (size_t)k * C::BM * C::Ld);
      val[it][h] = v;
    }

  // ---- ROWS: LoRA term of this part's ranks: t of the tile's rows through LDS (the shrink's parts added in part order), then
  // kU rows of W^B for all of a thread's rows on their way together.  Bound by the reads of W^B where every row has a tenant of
  // its own: 64 packed rows, rank 64, 4096 x 4096: 143 us a call with the term as matrix stages, 56 us so (37 since the shrink in
  // front has more workgroups).  A tile of one tenant reads its W^B again for each row: 300 rows of 4 tenants, rank 64, 4096 x
  // 11008: 77 -> 90 us.
  if constexpr (ROWS) {
    int most = ctl[1];
    if (C::BM > 64) most = ctl[2] > most ? ctl[2] : most;
    if (most > 0) {
      constexpr int kU = C::Items == 1 ? 16 : 8;
      float* const ts = reinterpret_cast<float*>(ring);  // [BM][kTs]: rows 16 bytes past a multiple of all banks
      gbf16* bp[C::Items];
      int cnt[C::Items], ranks = 0;
#pragma unroll
      for (int it = 0; it < C::Items; ++it) {
        cnt[it] = cg * 8 < cols ? row_cnt[r0 + it * kRowStep] : 0;
        const int row = r0 + it * kRowStep;
        bp[it] = in_global(p.W);  // (no rank: any valid 16 bytes)
        if (cnt[it] > 0) bp[it] = in_global(p.ad.B[row_ten[row] * MILORA_NUM_SITES + p.site]) + (size_t)row_c0[row] * p.d2 + n0 + cg * 8;
        ranks = cnt[it] > ranks ? cnt[it] : ranks;
      }
      __syncthreads();  // the sums are read
      const int pieces = (most + kU - 1) / kU * (kU / 4), total4 = C::BM * pieces;  // of four ranks, whole steps of kU
      for (int e = tid; e < total4; e += kT) {
        const int row = e / pieces, c = (e - row * pieces) * 4, left = row_cnt[row] - c;
        f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
        if (left > 0) {
          const float* const tp = p.t + (size_t)(m0 + row) * p.ad.r_max + row_c0[row] + c;
          if ((p.ad.r_max & 3) == 0) {
            for (int k0 = 0; k0 < p.parts; k0 += 4) {
              f32x4 x[4];
#pragma unroll
              for (int k = 0; k < 4; ++k)
                x[k] = *reinterpret_cast<const f32x4*>(tp + (k0 + k < p.parts ? k0 + k : p.parts - 1) * p.t_stride);
#pragma unroll
              for (int k = 0; k < 4; ++k)
                if (k0 + k < p.parts) v += x[k];
            }
#pragma unroll
            for (int i = 1; i < 4; ++i) v[i] = i < left ? v[i] : 0.f;  // (past the rank: never written)
          } else {
            for (int k = 0; k < p.parts; ++k)
#pragma unroll
              for (int i = 0; i < 4; ++i)
                if (i < left) v[i] += tp[k * p.t_stride + i];
          }
        }
        *reinterpret_cast<f32x4*>(ts + row * kTs + c) = v;
      }
      __syncthreads();
      for (int c0 = 0; __any(ranks > c0); c0 += kU) {
        u32x4 b[C::Items][kU];
#pragma unroll
        for (int it = 0; it < C::Items; ++it)
#pragma unroll
          for (int u = 0; u < kU; ++u) b[it][u] = *(gu32x4_a2*)(bp[it] + (size_t)(c0 + u < cnt[it] ? c0 + u : 0) * p.d2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int it = 0; it < C::Items; ++it)
#pragma unroll
          for (int u = 0; u < kU; ++u) {
            const float t = ts[(r0 + it * kRowStep) * kTs + c0 + u];
            const bool in = c0 + u < cnt[it];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const uint32_t x = in ? b[it][u][e] : 0u;
              val[it][e >> 1][2 * (e & 1)] += t * __uint_as_float(x << 16);
              val[it][e >> 1][2 * (e & 1) + 1] += t * __uint_as_float(x & 0xffff0000u);
            }
          }
      }
    }
  }

  // ---- what the stages could not take: products with the tenant's own Inf and NaN ----
  if (!ROWS && lora && ctl[kCtlBad] && cg * 8 < cols) {
#pragma unroll
    for (int it = 0; it < C::Items; ++it) {
      const int row = r0 + it * kRowStep, ten = row_ten[row], r = ten >= 0 ? row_rank[row] : 0;
      for (int c = 0; c < r; ++c) {
        const u32x4 b = *(gu32x4_a2*)(in_global(p.ad.B[ten * MILORA_NUM_SITES + p.site]) + (size_t)c * p.d2 + n0 + cg * 8);
        if (!(nonfinite2(b[0]) | nonfinite2(b[1]) | nonfinite2(b[2]) | nonfinite2(b[3]))) continue;
        float t = 0.f;
        for (int k = 0; k < p.parts; ++k) t += p.t[k * p.t_stride + (size_t)(m0 + row) * p.ad.r_max + c];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t bad = nonfinite2(b[e]);
          if (bad & 0x8000u) val[it][e >> 1][2 * (e & 1)] += t * __uint_as_float(b[e] << 16);
          if (bad & 0x80000000u) val[it][e >> 1][2 * (e & 1) + 1] += t * __uint_as_float(b[e] & 0xffff0000u);
        }
      }
    }
  }

  if (p.S > 1) {
    f32x4* const mine = reinterpret_cast<f32x4*>(p.partial) + ((size_t)tile * p.S + part) * (C::BM * C::BN / 4);
#pragma unroll
    for (int it = 0; it < C::Items; ++it)
#pragma unroll
      for (int h = 0; h < 2; ++h) st_through(mine + (it * kT + tid) * 2 + h, val[it][h]);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) ctl[0] = __hip_atomic_fetch_add(p.cnt + tile, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (ctl[0] != p.S - 1) return;
    if (tid == 0) __hip_atomic_store(p.cnt + tile, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // for the next slice of rows
    const f32x4* const all = reinterpret_cast<const f32x4*>(p.partial) + (size_t)tile * p.S * (C::BM * C::BN / 4);
    if constexpr (C::Items == 1) {
      for (int s0 = 0; s0 < p.S; s0 += 4) {
        f32x4 v[8];
        const f32x4* a[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int s = s0 + (u >> 1) < p.S ? s0 + (u >> 1) : p.S - 1;
          a[u] = all + (size_t)s * (C::BM * C::BN / 4) + tid * 2 + (u & 1);
        }
        ld_through8(a, v);
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (s0 + (u >> 1) < p.S) val[0][u & 1] = s0 + (u >> 1) == 0 ? v[u] : val[0][u & 1] + v[u];
      }
    } else {
      static_assert(C::Items % 4 == 0 || C::Items == 1, "eight loads at a time");
      for (int s = 0; s < p.S; ++s)
#pragma unroll
        for (int i0 = 0; i0 < C::Items; i0 += 4) {
          f32x4 v[8];
          const f32x4* a[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) a[u] = all + (size_t)s * (C::BM * C::BN / 4) + ((i0 + (u >> 1)) * kT + tid) * 2 + (u & 1);
          ld_through8(a, v);
#pragma unroll
          for (int u = 0; u < 8; ++u) val[i0 + (u >> 1)][u & 1] = s == 0 ? v[u] : val[i0 + (u >> 1)][u & 1] + v[u];
        }
    }
  }

  // ---- bias, one rounding, stores ----
  if (cg * 8 >= cols) return;
  const int n = n0 + cg * 8;
  float bv[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) bv[e] = p.bias ? bf16_to_f32(p.bias[n + e]) : 0.f;
#pragma unroll
  for (int it = 0; it < C::Items; ++it) {
    const int r = r0 + it * kRowStep;
    if (r >= rows) continue;
    u32x4_a8 o;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      o[e] = pack_bf16x2(val[it][e >> 1][2 * (e & 1)] + bv[2 * e], val[it][e >> 1][2 * (e & 1) + 1] + bv[2 * e + 1]);
    *reinterpret_cast<u32x4_a8*>(p.Y + (size_t)(m0 + r) * p.d2 + n) = o;
  }
}

template <class C, bool PK, bool ROWS>
int launch_tiles(const TParams& p, hipStream_t st) {
  static thread_local int lds_set_for = -1;
  int dev = 0;
  MILORA_HIP(hipGetDevice(&dev));
  if (lds_set_for != dev) {
    MILORA_HIP(hipFuncSetAttribute((const void*)tile_kernel<C, PK, ROWS>, hipFuncAttributeMaxDynamicSharedMemorySize, C::LdsBytes));
    lds_set_for = dev;
  }
  const int total = p.tilesM * p.tilesN * p.S;
  hipLaunchKernelGGL((tile_kernel<C, PK, ROWS>), dim3(8 * ((total + 7) / 8)), dim3(kT), C::LdsBytes, st, p);
  return check_launch();
}

}  // namespace

// Which tiles, and how many parts: the estimated time in 10 ns, fitted to launches of 16 .. 4096 rows on the seven linears
// of the 7B and 13B layers and a 1088 x 2624 one.  A compute unit takes 0.26 us per stage of 64 k for a 64 x 64 tile
// (two workgroups share it: half the rate each), 0.58 us for a 128 x 128 one and 1.2 .. 1.6 us (few .. all units busy:
// the L2 is shared) for a 256 x 256 one (600 rows on 5120 x 13824: 110 us a call, 133 with 128 x 128; 2048 on 4096 x 4096: 86 and 79);
// its 7.75 us a turn are what short reductions show.  The choice knows sizes only; it was timed with no row routed and with every row
// routed to one of two tenants of rank 32, 128 x 128 / 256 x 256 tiles: 3846 rows on 512 x 1040 18.6 / 20.6 and 31.5 / 34.2 us, 1406
// on 192 x 11008 25.8 / 28.0 and 45.5 / 47.8, 1805 on 192 x 7488 25.4 / 18.0 and 45.5 / 29.1; near a tie it gives away some percent:
// 3390 on 64 x 2048, which take 256 x 256, 13.6 / 13.8 and 25.1 / 26.1;
// workgroups beyond 256 wait for a second turn; a last turn of few is shorter than a whole one (256 x 256, 1700 rows on 4096 x 11008: 301
// workgroups, 2.6 us a step for both turns, 3.2 for two whole ones; of more than two turns of 128 x 128, 600 rows on 5120 x 13824: 540,
// 2.7 turns; below that, 300 rows on 4096 x 11008: 258, 70.2 us against 66.5 with 64 x 64; packed weights, for which there is no
// 256 x 256 kernel, keep the choice between 64 and 128 that was timed for them); cutting the reduction costs the
// partial tiles and the last workgroup's sums (M = 64 on 4096 x 4096: one part 25.0 us a call, two 19.8, four 16.4, six 22.2).
TilePlan plan_tiles(int64_t M, int d1, int d2, bool small, bool large) {
  const int KT = (d1 + 63) / 64;
  TilePlan best{};
  int64_t best_t = INT64_MAX;
  auto offer = [&](int shape, int side, int64_t per_step, int64_t per_tile, int S, int64_t split_cost) {
    const int64_t tm = (M + side - 1) / side, tn = (d2 + side - 1) / side, units = tm * tn * S;
    if (S > 1 && (units > kMaxSplitUnits || S > KT)) return;
    const int steps = (KT + S - 1) / S;
    const int64_t turn = per_step * steps + per_tile, rest = units % 256;
    int64_t t = (units + 255) / 256 * turn + (S > 1 ? split_cost : 0);
    if (rest && large && S == 1 && shape == kTiles128 && units > 512) t -= turn / 2 - turn * rest / 512;
    if (rest && shape == kTiles256) t -= 46 * (256 - rest) / 256 * steps;
    if (t >= best_t) return;
    best_t = t;
    best = TilePlan{shape, (int)tm, (int)tn, (KT + steps - 1) / steps, steps, 0};  // (no empty part)
    if (best.S > 1) best.partial_bytes = (size_t)(tm * tn) * best.S * side * side * sizeof(float);
  };
  if (small && M <= kTileMaxRows)
    for (int S = 1; S <= kMaxParts; ++S) {
      offer(kTiles64, 64, 26, 200, S, 400 + 70 * S);
      offer(kTiles128, 128, 58, 400, S, 250 + 220 * S);
    }
  if (large) offer(kTiles256, 256, 163, 775, 1, 0);
  return best;
}

// A plan's own need rises and falls with the sizes (4096 x 4096: 12.6 MB at 300 rows, 16.8 at 512, none at 777); what bounds
// every plan is the number of tiles, the parts of each and the units of a launch.
size_t partial_bytes_bound(int64_t M, int d1, int d2) {
  const int64_t KT = ((int64_t)d1 + 63) / 64, rows = M < kTileMaxRows ? M : kTileMaxRows;
  const int64_t parts = KT < kMaxParts ? KT : kMaxParts;
  if (parts < 2) return 0;
  size_t bytes = 0;
  for (int side = 64; side <= 128; side *= 2) {
    const int64_t units = ((rows + side - 1) / side) * (((int64_t)d2 + side - 1) / side) * parts;
    const size_t n = (size_t)(units < kMaxSplitUnits ? units : kMaxSplitUnits) * side * side * sizeof(float);
    bytes = n > bytes ? n : bytes;
  }
  return bytes;
}

bool tiles_supported(int64_t M, int d1, int d2, bool packed, const void* X, const void* W, const void* Y) {
  if (M < 1 || d2 % 16 != 0 || d1 % (packed ? 32 : 64) != 0) return false;
  const int64_t rows = M < kTileMaxRows ? M : kTileMaxRows;
  if (((rows + 63) / 64) * (((int64_t)d2 + 63) / 64) >= 1 << 22) return false;  // a grid has to stay below 2^32 threads
  if ((((uintptr_t)X | (uintptr_t)W) & 15) != 0 || ((uintptr_t)Y & 7) != 0) return false;
  return (uint64_t)d1 * 128u * 2u < (1ull << 31);  // byte offsets inside a tile's lines
}

int routed_linear_tiles(const bf16_t* X, int64_t M, int d1, int d2, const int32_t* row_to_req, const bf16_t* W, bool packed,
                        const int2* row_lora, const bf16_t* bias, const AdapterView& ad, int site, const int32_t* tenant_id, const uint8_t* route,
                        int B, const float* t, size_t t_stride, int parts, const TilePlan& pl, int* cnt, float* partial, bf16_t* Y, hipStream_t st) {
  TParams p;
  p.X = X; p.W = W; p.bias = bias; p.Y = Y; p.t = t; p.t_stride = t_stride; p.parts = parts;
  p.row_to_req = row_to_req; p.tenant_id = tenant_id; p.route = route; p.ad = ad; p.M = M; p.row_lora = row_lora; p.d1 = d1; p.d2 = d2;
  p.site = site; p.B = B; p.tilesM = pl.tilesM; p.tilesN = pl.tilesN; p.S = pl.S; p.steps = pl.steps;
  p.partial = partial; p.cnt = cnt;
  const bool mid = pl.shape == kTiles128;
  static_assert(kMaxSplitUnits <= kShrinkClear, "counters the shrink zeroes");
  if (packed) return mid ? launch_tiles<CfgMid, true, true>(p, st) : launch_tiles<CfgSmall, true, true>(p, st);
  if (row_lora) return mid ? launch_tiles<CfgMid, false, true>(p, st) : launch_tiles<CfgSmall, false, true>(p, st);
  return mid ? launch_tiles<CfgMid, false, false>(p, st) : launch_tiles<CfgSmall, false, false>(p, st);
}

}  // namespace milora
