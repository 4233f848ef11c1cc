// LoRA shrink on the matrix cores: t[m][0..r) = X[m] . W^A of the row's tenant, routed rows only (device code shared by
// the launches that need it).
//
// A workgroup takes 16 * RT rows and one part of the reduction; the part's chunks of 128 k are dealt to its NW waves,
// each works alone until their sums meet in LDS at the end.  W^A is [d1][r] (reduction index outermost), the matrix cores
// want 8 consecutive reduction indices per lane: a lane loads eight 16-byte pieces (8 ranks at 8 consecutive k), turns
// the 8 x 8 block with byte permutes and puts it into the wave's own LDS as [rank][k].  X rows come straight from
// global memory as operands.  Rows of several tenants are computed once per tenant and each row keeps its own tenant's
// result; where workgroups are few, the block's units (32 ranks of a tenant) are dealt to several of them: a unit is a chain
// of table, W^A and LDS round trips, about 3 us.  Needs d1 % 32 == 0.
#pragma once
#include "common.h"

namespace milora {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
// Adapter matrices are reached through pointer tables read at run time; telling the compiler that they lie in
// global memory keeps their loads off the counter the LDS reads wait on.
typedef __attribute__((address_space(1))) const bf16_t gbf16;
typedef __attribute__((address_space(1))) const u32x4 gu32x4;
__device__ __forceinline__ gbf16* in_global(const void* p) { return (gbf16*)p; }

constexpr int kShrinkClear = 512;
constexpr int kShrinkC = 32;                                    // ranks at a time
constexpr int kShrinkLd = kShrinkChunkK + 8;                    // LDS row of a rank, padded: 16 ranks at one k group hit all banks
constexpr int kShrinkWaveBytes = kShrinkC * kShrinkLd * 2;      // 8.5 KiB: the wave's chunk of W^A, at the end its sums

struct ShrinkArgs {
  const bf16_t* X;
  int64_t M, row_base;  // rows, and the index of the first one in the caller's matrix (requests of unmapped rows)
  int d1, site, B;
  const int32_t* row_to_req;
  const int32_t* tenant_id;
  const uint8_t* route;
  AdapterView ad;
  float* t;        // [part][M][r_max]
  size_t t_stride;
  int2* row_lora;  // INFO: [M] receives tenant and rank of each row (rank 0: no LoRA term), or null
  int* clear;      // INFO: [kShrinkClear] words of the launch behind this one that have to start from zero, or null
};

// Two by two bf16 of two words a (k) and b (k + 1): the pair of low halves, the pair of high halves.
__device__ __forceinline__ uint32_t lo_pair(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ uint32_t hi_pair(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// 8 x 8 block of bf16, a[i] = row i: out[j] = column j.
__device__ __forceinline__ void transpose8(const u32x4 (&a)[8], u32x4 (&out)[8]) {
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      out[2 * e][i] = lo_pair(a[2 * i][e], a[2 * i + 1][e]);
      out[2 * e + 1][i] = hi_pair(a[2 * i][e], a[2 * i + 1][e]);
    }
}

// Tenants whose rows share a matrix stage see each other's W^B times zero, and zero times Inf is NaN.  Inf and NaN therefore never
// enter a stage: a 1 of their sign goes in (for the tenant's own rows it stands beside the true product, which is not finite and
// is added behind the stages), and the workgroup remembers that it has to add.
// Bits 15 and 31: whether the low or high bf16 of the word is Inf or NaN.
__device__ __forceinline__ uint32_t nonfinite2(uint32_t w) { return ((w & 0x7f807f80u) + 0x00800080u) & 0x80008000u; }
__device__ __forceinline__ uint32_t finite2(uint32_t w) {
  const uint32_t bad = nonfinite2(w);
  if (bad & 0x8000u) w = (w & 0xffff8000u) | 0x3f80u;
  if (bad & 0x80000000u) w = (w & 0x8000ffffu) | 0x3f800000u;
  return w;
}
// `sum` plus zero times both bf16 of the word: NaN from the first Inf or NaN on, else as it was (one instruction per word; by bit
// tests, three: 4096 scattered rows of 64 tenants, rank 256, 4096 x 4096: 5.22 ms a call, 5.10 so).
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float taint(float sum, uint32_t w) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), __builtin_bit_cast(bf16x2, 0u), sum, false);
}
// Eight bf16 of a row that ends after `left` elements (zero past the end); 16-byte load where `vec` allows it.
__device__ __forceinline__ u32x4 load8(gbf16* p, int left, bool vec) {
  if (vec) return *(gu32x4*)p;
  u32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t lo = 2 * e < left ? (uint32_t)p[2 * e] : 0u;
    const uint32_t hi = 2 * e + 1 < left ? (uint32_t)p[2 * e + 1] : 0u;
    v[e] = lo | (hi << 16);
  }
  return v;
}

// STORE(float* p, float v) stores one element of t.  `smem`: NW * kShrinkWaveBytes, `row_ten`: 16 * RT ints (INFO: twice that).
template <int RT, int NW, bool INFO, class STORE>
__device__ __forceinline__ void shrink_block(const ShrinkArgs& g, int row_block, int part, int parts, int share, int shares,
                                             unsigned char* smem, int* row_ten, STORE store) {
  constexpr int kRows = RT * 16;
  static_assert(kRows * kShrinkC * 4 <= kShrinkWaveBytes, "sums of a wave");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t m0 = (int64_t)row_block * kRows;
  if (tid < kRows) {
    const int64_t m = m0 + tid;
    int ten = -1, r = 0;
    if (m < g.M) {
      const int64_t req = g.row_to_req ? (int64_t)g.row_to_req[m] : g.row_base + m;
      int tenant = 0;
      if (req >= 0 && req < g.B && (r = routed_rank(g.ad, g.tenant_id, g.route, (int)req, g.B, g.site, &tenant))) ten = tenant;
    }
    row_ten[tid] = ten;
    if (INFO) row_ten[kRows + tid] = r;
  }
  __syncthreads();
  const int my_ten = lane < kRows ? row_ten[lane] : -1;
  bf16_t* const At = reinterpret_cast<bf16_t*>(smem + wave * kShrinkWaveBytes);  // [rank][k]
  float* const sums = reinterpret_cast<float*>(smem + wave * kShrinkWaveBytes);  // [row][rank], after the last chunk
  const int chunks = (g.d1 + kShrinkChunkK - 1) / kShrinkChunkK;
  float* const t = g.t + (size_t)part * g.t_stride;
  const bf16_t* xp[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    int64_t m = m0 + rt * 16 + (lane & 15);
    m = m < g.M ? m : g.M - 1;
    xp[rt] = g.X + (size_t)m * g.d1 + (lane >> 4) * 8;
  }
  int last = -1, unit = 0;  // (unit % shares)
  for (;;) {
    int cur = my_ten > last ? my_ten : 0x7fffffff;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int o = __shfl_xor(cur, off, 64);
      cur = o < cur ? o : cur;
    }
    cur = __builtin_amdgcn_readfirstlane(cur);
    if (cur == 0x7fffffff) break;
    const unsigned long long mine = __ballot(my_ten == cur);
    const int r = g.ad.rank[cur];
    gbf16* A = in_global(g.ad.A[cur * MILORA_NUM_SITES + g.site]);
    const bool vec = (r & 7) == 0 && ((uintptr_t)A & 15) == 0;
    for (int cb = 0; cb < r; cb += kShrinkC) {
      const bool ours = unit == share;
      unit = unit + 1 == shares ? 0 : unit + 1;
      if (!ours) continue;
      const int rc = r - cb < kShrinkC ? r - cb : kShrinkC;
      const int groups = (rc + 7) >> 3, ntile = (rc + 15) >> 4;
      f32x4 acc[RT][2];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) acc[rt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
      // a lane's 8 x 8 block of the chunk: ranks cb + 8 cg .., k 8 oct .. (up to 4 x 16 blocks, one per lane)
      const int cg = lane % groups, oct = lane / groups;
      for (int ch = part * NW + wave; ch < chunks; ch += parts * NW) {
        const int k0 = ch * kShrinkChunkK;
        const int steps = g.d1 - k0 < kShrinkChunkK ? (g.d1 - k0) / 32 : kShrinkChunkK / 32;
        if (oct < kShrinkChunkK / 8) {
          u32x4 a[8], at[8];
          const int k = k0 + oct * 8 < g.d1 ? k0 + oct * 8 : g.d1 - 8;  // past the end: valid rows, not multiplied
#pragma unroll
          for (int i = 0; i < 8; ++i) a[i] = load8(A + (size_t)(k + i) * r + cb + cg * 8, rc - cg * 8, vec);
          transpose8(a, at);
#pragma unroll
          for (int j = 0; j < 8; ++j) *reinterpret_cast<u32x4*>(At + (cg * 8 + j) * kShrinkLd + oct * 8) = at[j];
        }
        bf16x8 xf[RT][kShrinkChunkK / 32];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int ks = 0; ks < kShrinkChunkK / 32; ++ks) xf[rt][ks] = *(const bf16x8*)(xp[rt] + k0 + (ks < steps ? ks : 0) * 32);
        __builtin_amdgcn_s_waitcnt(0xc07f);  // the wave's own LDS writes, read by its other lanes
        asm volatile("" ::: "memory");
#pragma unroll
        for (int ks = 0; ks < kShrinkChunkK / 32; ++ks)
          if (ks < steps)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
              if (nt < ntile) {
                const bf16x8 w = *reinterpret_cast<const bf16x8*>(At + (nt * 16 + (lane & 15)) * kShrinkLd + ks * 32 + (lane >> 4) * 8);
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                  if (RT == 1 || ((mine >> (16 * rt)) & 0xffff))
                    acc[rt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, xf[rt][ks], acc[rt][nt], 0, 0, 0);
              }
        __builtin_amdgcn_s_waitcnt(0xc07f);
        asm volatile("" ::: "memory");
      }
      // lane holds row lane % 16 of a row tile, ranks (lane / 16) * 4 .. + 3 of each 16-rank tile
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
          *reinterpret_cast<f32x4*>(sums + (rt * 16 + (lane & 15)) * kShrinkC + nt * 16 + (lane >> 4) * 4) = acc[rt][nt];
      __syncthreads();
      for (int e = tid; e < kRows * kShrinkC; e += NW * 64) {
        const int row = e / kShrinkC, c = e % kShrinkC;
        if (row_ten[row] == cur && c < rc) {
          float v = 0.f;
#pragma unroll
          for (int w = 0; w < NW; ++w) v += reinterpret_cast<const float*>(smem + w * kShrinkWaveBytes)[e];
          store(t + (size_t)(m0 + row) * g.ad.r_max + cb + c, v);
        }
      }
      __syncthreads();
    }
    last = cur;
  }
  if (INFO && g.row_lora && part == 0 && share == 0 && tid < kRows && m0 + tid < g.M)
    g.row_lora[m0 + tid] = int2{row_ten[tid], row_ten[kRows + tid]};
}

}  // namespace milora
