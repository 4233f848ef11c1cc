// Many-row (prefill) routed LoRA linear on row-major bf16 weights (paper Eq. 1 with the layer-level gate of
// Sec. 3.3): Y = X W^T + bias + (X W^A) W^B for the rows whose request is routed to this site.
//
// One workgroup of four waves computes a 256 x 256 tile of Y with the bf16 matrix cores
// (v_mfma_f32_32x32x16_bf16, fp32 accumulators, 128 x 128 per wave; a kernel of nothing but this instruction
// sustains 2.3-2.4 PFLOP/s on the chip, one of nothing but the 16x16x32 form 1.45-1.5).  X and W are both contiguous along the
// reduction index: 16-row x 64-k blocks of either are copied from global memory straight into LDS
// (global_load_lds_dwordx4, no registers; whole 128-byte lines per row), in a ring of five half steps of
// 32 KB, and read back as matrix-core operands with one conflict-free 16-byte LDS load per lane, pair of blocks
// and 16 k.  A step's operands are all in registers after a quarter of its matrix work; its ring slots are
// refilled from there on, so that nearly the whole LDS is data on its way (the copies are bound by latency:
// bytes in flight over about two microseconds).
// The LoRA term enters as extra k steps: t = X W^A (fp32, computed beforehand) split into two bf16 halves
// (hi + lo, about 17 of its 24 bits) against W^B of the tenant, masked to that tenant's rows; Inf and NaN of W^B are kept
// out of the stages and added to those rows at the end.
// Bias is added and the result rounded once at the store.
#include "shrink.h"

namespace milora {
namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));
typedef uint32_t u32x4_a2 __attribute__((ext_vector_type(4), aligned(2)));
typedef __attribute__((address_space(1))) const u32x4_a2 gu32x4_a2;
typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr int kTM = 256, kTN = 256, kTK = 64;
constexpr int kThreadsP = 256;
constexpr int kBlocksM = kTM / 16, kBlocksN = kTN / 16;
constexpr int kBlockBytes = 16 * kTK * 2;                 // 16 rows x 64 k: 2 KiB, a row is one 128-byte line
constexpr int kHalfBytes = (kBlocksM + kBlocksN) / 2 * kBlockBytes;  // 8 X blocks + 8 W blocks: 32 KiB
constexpr int kHalves = 5;                                // ring of half steps
constexpr int kLdsBytesP = kHalves * kHalfBytes;
constexpr int kAccTilesRows = 3;
constexpr int kOutPitch = 128 * 2 + 16;                   // a row of a wave's results on their way out, padded: 16 rows at one column hit all banks
static_assert(4 * 128 * kOutPitch <= kLdsBytesP, "results of the four waves");
// Where the sixteen copy instructions of a k step sit among its 64 matrix instructions: those of the first half
// after instructions 0, kCopyAStride, ..., those of the second half from instruction kCopyB0 on (16 or later: the
// slot they fill is read until then).
constexpr int kCopyAStride = 2, kCopyB0 = 16, kCopyBStride = 3;
static_assert(kCopyB0 >= 16 && 7 * kCopyAStride < kCopyB0 && kCopyB0 + 7 * kCopyBStride < 64, "copy positions");
constexpr int kGroupM = 4;  // consecutive workgroups of an XCD walk 4 row tiles of one column tile

struct PParams {
  const bf16_t* X;
  const bf16_t* W;
  const bf16_t* bias;
  bf16_t* Y;
  const float* t;     // `parts` partial shrinks [part][rows of the whole call][r_max], to be added in part order
  size_t t_stride;    // floats from one part to the next
  int parts;
  const int32_t* row_to_req;
  const int32_t* tenant_id;
  const uint8_t* route;
  AdapterView ad;
  int64_t M;         // rows of this launch
  int64_t row_base;  // index of its first row in the caller's matrix (requests of unmapped rows)
  int d1, d2, site, B;
  int tilesM, tilesN;
};

// Which of the eight 16-byte pieces of its 128-byte LDS line holds k group kg of row r (0..15) of a block:
// kg ^ swz(r).  Eight neighbouring rows get eight different pieces, and rows r and r + 8 (which lie 1 KiB apart, on
// the same banks) differ too, so a 16-byte operand read of 16 rows at one k group touches every bank once.
__device__ __forceinline__ int swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

template <int N>
__device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0f70);
}

__global__ void __launch_bounds__(kThreadsP, 1) prefill_kernel(PParams p) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wn = wave >> 1;

  // workgroup -> tile: workgroup ids go round-robin over the 8 XCDs; each XCD takes a contiguous run of the
  // tile order, which walks kGroupM row tiles per column tile so that the XCD's L2 serves the re-reads
  // (the 32 workgroups resident on an XCD then cover 4 row tiles x 8 column tiles)
  const int total = p.tilesM * p.tilesN;
  const int per = (total + 7) / 8;
  const int id = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (id >= total) return;
  const int gspan = kGroupM * p.tilesN;
  const int first = id / gspan * kGroupM;
  const int gsz = p.tilesM - first < kGroupM ? p.tilesM - first : kGroupM;
  const int in_group = id % gspan;
  const int64_t m0 = (int64_t)(first + in_group % gsz) * kTM;
  const int n0 = in_group / gsz * kTN;

  const int KT = p.d1 / kTK;
  const uint32_t lds0 = lds_addr(lds);

  // copies.  A k step of 64 is brought in two halves: half 0 = X rows 0..127 and W rows 0..127 of the tile,
  // half 1 = the other rows; a half is 8 + 8 blocks of 16 rows, a block two copy instructions of 8 rows each
  // (8 lanes take the 128-byte line of a row, so every request is for whole cache lines).  Waves 0,1 bring
  // the X blocks of a half (4 each), waves 2,3 the W blocks.  Which 16 bytes of the line a lane takes is
  // permuted by the row so that the operand reads below spread over all LDS banks.
  const bool is_w = wave >= 2;
  const unsigned char* src = is_w ? (const unsigned char*)p.W : (const unsigned char*)p.X;
  const int64_t row0 = is_w ? (int64_t)n0 : m0;
  const int64_t rlim = is_w ? (int64_t)p.d2 : p.M;
  uint32_t voff[2][8];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int rr = lane >> 3;
      int64_t r = row0 + (hh * 8 + (wave & 1) * 4 + (j >> 1)) * 16 + (j & 1) * 8 + rr;
      r = r < rlim ? r : rlim - 1;
      voff[hh][j] = (uint32_t)((uint64_t)r * (uint32_t)p.d1 * 2u + (uint32_t)((lane & 7) ^ swz((j & 1) * 8 + rr)) * 16u);
    }
  const uint32_t dst_in_half = (uint32_t)((is_w ? 8 : 0) + (wave & 1) * 4) * kBlockBytes;
  // half H = 2 * (k step) + hh lives in ring slot H % kHalves
  // copy j (0..7) of a half; a wave's eight copies of a half are spread between its matrix instructions: issued
  // back to back they would hold the wave at the issue of the memory instructions while the matrix cores idle
  auto issue_one = [&](int kt, int hh, int slot, int j) __attribute__((always_inline)) {
    const int kk = kt < KT ? kt : KT - 1;  // past the end: re-read the last step into a slot nobody reads
    const unsigned char* b = src + (size_t)kk * (kTK * 2);
    const uint32_t dst = lds0 + slot * kHalfBytes + dst_in_half;
    copy_to_lds16(b, voff[hh][j], dst + j * 1024);
  };
  auto issue = [&](int kt, int hh, int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 8; ++j) issue_one(kt, hh, slot, j);
  };

  // acc[i][j]: rows 32 i .. 32 i + 31 of the wave's X part against rows 32 j .. of its W part
  f32x16 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // operand read: lane l takes row l % 32 of a pair of 16-row blocks and the 16 bytes of k group 2 ks + l / 32
  // (ks = 0..3: the four 16-k sub-steps of a block's 64 k)
  const int rrow = lane & 31;
  int rd[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    rd[ks] = (rrow >> 4) * kBlockBytes + (rrow & 15) * 128 + (((2 * ks + (lane >> 5)) ^ swz(rrow & 15)) << 4);
  const unsigned char* wbase = lds + (kBlocksM / 2) * kBlockBytes;
  // One k step of 64 for the wave's 128 x 128 part: 64 matrix instructions, number q = 16 ks + 4 i + j.  The
  // operand reads come early: the sixteen of the first two sub-steps, then the other sixteen between the matrix
  // instructions of the first sub-step.  `mid` runs after instruction 15, once every wave of the workgroup has
  // its operands in registers: the step's two ring slots are free from there on.  copy(q) runs after instruction q.
  auto mma64 = [&](int slot_x, int slot_w, auto mid, auto copy) __attribute__((always_inline)) {
    const unsigned char* sa = lds + slot_x * kHalfBytes;
    const unsigned char* sb = wbase + slot_w * kHalfBytes;
    bf16x8 a[4][4], b[4][4];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int i = 0; i < 4; ++i) a[ks][i] = *(const bf16x8*)(sa + rd[ks] + i * 2 * kBlockBytes);
#pragma unroll
      for (int j = 0; j < 4; ++j) b[ks][j] = *(const bf16x8*)(sb + rd[ks] + j * 2 * kBlockBytes);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      acc[q >> 2][q & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[0][q & 3], a[0][q >> 2], acc[q >> 2][q & 3], 0, 0, 0);
      const int ks = 2 + (q >> 3), e = q & 3;
      if (q & 4) b[ks][e] = *(const bf16x8*)(sb + rd[ks] + e * 2 * kBlockBytes);
      else a[ks][e] = *(const bf16x8*)(sa + rd[ks] + e * 2 * kBlockBytes);
      copy(q);
      __builtin_amdgcn_sched_barrier(0);
    }
    mid();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 16; q < 64; ++q) {
      acc[(q >> 2) & 3][q & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[q >> 4][q & 3], a[q >> 4][(q >> 2) & 3],
                                                                         acc[(q >> 2) & 3][q & 3], 0, 0, 0);
      copy(q);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  issue(0, 0, 0);
  issue(0, 1, 1);
  issue(1, 0, 2);
  issue(1, 1, 3);
  // 12 of the 16 accumulator tiles in the accumulation registers, 4 in ordinary ones: with all 256 in the
  // accumulation file the compiler has no spare tile there and shuffles tiles between the files in the loop
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (i < kAccTilesRows) asm volatile("" : "+a"(acc[i][j]));
      else asm volatile("" : "+v"(acc[i][j]));
    }
  // The ring: halves 2 kt and 2 kt + 1 (this step) are read, the two of the next step are on their way, the
  // fifth slot takes the first half of the step after next at once and the second half goes into this step's
  // first slot as soon as every wave has taken its operands out: a copy has between one and three quarters and
  // two whole steps of matrix work to arrive.
  int h0 = 0;  // ring slot of half 0 of the current step
  for (int kt = 0; kt < KT; ++kt) {
    const int h1 = h0 + 1 >= kHalves ? h0 + 1 - kHalves : h0 + 1;
    const int h2 = h0 + 2 >= kHalves ? h0 + 2 - kHalves : h0 + 2;
    const int h4 = h0 + 4 >= kHalves ? h0 + 4 - kHalves : h0 + 4;
    wait_vm<16>();                  // all but the two halves issued last have landed: both halves of this step
    __builtin_amdgcn_s_barrier();   // for every wave
    asm volatile("" ::: "memory");
    mma64(
        wm ? h1 : h0, wn ? h1 : h0,
        [&]() __attribute__((always_inline)) {
          __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's operand reads have returned
          __builtin_amdgcn_s_barrier();        // and every other wave's
          asm volatile("" ::: "memory");
        },
        [&](int q) __attribute__((always_inline)) {
          // first half of the step after next into the free slot, second half into this step's first slot
          if (q < kCopyB0) {
            if (q % kCopyAStride == 0 && q / kCopyAStride < 8) issue_one(kt + 2, 0, h4, q / kCopyAStride);
          } else if ((q - kCopyB0) % kCopyBStride == 0 && (q - kCopyB0) / kCopyBStride < 8) {
            issue_one(kt + 2, 1, h0, (q - kCopyB0) / kCopyBStride);
          }
        });
    asm volatile("" ::: "memory");
    h0 = h2;
  }
  wait_vm<0>();
  __syncthreads();

  // ---- LoRA term of the routed rows as one more k step per 32 ranks, two of them filled together ------------
  // t = X W^A (fp32) goes in as bf16 hi + lo: hi in the first k half of a block, lo in the second, against the
  // same 32 rows of the tenant's W^B in both halves; rows of other tenants and unrouted rows enter as zeros.  Bound by the
  // instructions of filling a step: W^B in pieces of 8 ranks x 8 columns, 16-byte loads turned with byte permutes, t four ranks of
  // a row at a time straight into its two halves; and by the round trips to t, about 3 us each (32 loads of two bytes a thread,
  // t by way of LDS, one step at a time: a call of 777 rows on 4096 x 11008 with a tenant of rank 64 131 us, 120 so, 97 without).
  int* ctl = (int*)(lds + 4 * kHalfBytes);  // ring slots 0 .. 3 hold the operand blocks
  int* const row_ten = ctl + 16;            // tenant of each row of the tile, -1: no LoRA term
  int my_ten = -1;
  {
    const int64_t m = m0 + tid;
    if (m < p.M) {
      const int64_t req = p.row_to_req ? (int64_t)p.row_to_req[m] : p.row_base + m;
      int tenant = 0;
      const int r = (req >= 0 && req < p.B) ? routed_rank(p.ad, p.tenant_id, p.route, (int)req, p.B, p.site, &tenant) : 0;
      if (r) my_ten = tenant;
    }
  }
  row_ten[tid] = my_ten;
  if (tid == 0) ctl[1] = 0;  // set: W^B of some tenant of the tile holds Inf or NaN
  int last = -1;
  for (;;) {
    if (tid == 0) ctl[0] = 0x7fffffff;
    __syncthreads();
    int cand = my_ten > last ? my_ten : 0x7fffffff;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int o = __shfl_xor(cand, off, 64);
      cand = o < cand ? o : cand;
    }
    if (lane == 0) atomicMin(&ctl[0], cand);
    __syncthreads();
    const int cur = ctl[0];
    if (cur == 0x7fffffff) break;
    const int r = p.ad.rank[cur];
    gbf16* Bm = in_global(p.ad.B[cur * MILORA_NUM_SITES + p.site]);
    for (int c0 = 0; c0 < r; c0 += 64) {
      int tb = tid;  // opaque: addresses formed from it stay inside the loop instead of being spilled in front of it
      asm volatile("" : "+v"(tb));
      const int steps = r - c0 > 32 ? 2 : 1;
      // W side: ranks c0 + 8 gq .. + 7 of columns 8 pc .. + 7, asked for first, used last
      const int pc = tb & 31, gq = tb >> 5, cw = c0 + gq * 8;
      const bool wput = gq < steps * 4;
      u32x4 a[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) a[i] = u32x4{0u, 0u, 0u, 0u};
      if (wput && n0 + pc * 8 < p.d2) {
        gbf16* b = Bm + (size_t)cw * p.d2 + n0 + pc * 8;
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (cw + i < r) a[i] = *(gu32x4_a2*)(b + (size_t)i * p.d2);  // (whole pieces of 8 columns, d2 % 16 == 0, at any alignment)
      }
      // X side: eight lanes take 32 ranks of a row, the shrink's parts added in part order
      const int rq = tb & 7;
      for (int st = 0; st < steps; ++st) {
        const int cq = c0 + st * 32 + rq * 4;
        const bool vec = (p.ad.r_max & 3) == 0 && cq + 3 < p.ad.r_max;
#pragma unroll 1
        for (int i0 = 0; i0 < 8; i0 += 4) {
          f32x4 v[4];
          const float* q[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            const int64_t mr = m0 + (tb >> 3) + 32 * (i0 + i);
            q[i] = p.t + (size_t)(mr < p.M ? mr : p.M - 1) * p.ad.r_max + cq;
          }
          if (vec) {
            for (int k0 = 0; k0 < p.parts; k0 += 4) {  // four rows and four parts in flight
              f32x4 x[4][4];
#pragma unroll
              for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                  x[k][i] = *reinterpret_cast<const f32x4*>(q[i] + (k0 + k < p.parts ? k0 + k : p.parts - 1) * p.t_stride);
#pragma unroll
              for (int k = 0; k < 4; ++k)
                if (k0 + k < p.parts)
#pragma unroll
                  for (int i = 0; i < 4; ++i) v[i] += x[k][i];
            }
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
              for (int e = 0; e < 4; ++e)
                if (cq + e < p.ad.r_max)
                  for (int part = 0; part < p.parts; ++part) v[i][e] += q[i][part * p.t_stride + e];
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int row = (tb >> 3) + 32 * (i0 + i);
            const bool ours = row_ten[row] == cur;
            float tv[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) tv[e] = ours && cq + e < r ? v[i][e] : 0.f;
            u32x2 hi, lo;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              hi[h] = pack_bf16x2(tv[2 * h], tv[2 * h + 1]);
              lo[h] = pack_bf16x2(tv[2 * h] - __uint_as_float(hi[h] << 16), tv[2 * h + 1] - __uint_as_float(hi[h] & 0xffff0000u));
            }
            unsigned char* const x = lds + (2 * st + (row >> 7)) * kHalfBytes + ((row >> 4) & 7) * kBlockBytes + (row & 15) * 128 + (rq & 1) * 8;
            *(u32x2*)(x + (((rq >> 1) ^ swz(row & 15)) << 4)) = hi;
            *(u32x2*)(x + ((((rq >> 1) + 4) ^ swz(row & 15)) << 4)) = lo;
          }
        }
      }
      if (wput) {
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
          ctl[1] = 1;
        }
        u32x4 at[8];
        transpose8(a, at);
        // (columns 8 pc .. + 7: one half of a block of 16)
        unsigned char* const wst = lds + (2 * (gq >> 2) + (pc >> 4)) * kHalfBytes + (kBlocksM / 2 + ((pc >> 1) & 7)) * kBlockBytes;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int n = (pc & 1) * 8 + j;
          *(u32x4*)(wst + n * 128 + (((gq & 3) ^ swz(n)) << 4)) = at[j];
          *(u32x4*)(wst + n * 128 + ((((gq & 3) + 4) ^ swz(n)) << 4)) = at[j];
        }
      }
      __syncthreads();
      for (int st = 0; st < steps; ++st) mma64(2 * st + wm, 2 * st + wn, []() {}, [](int) {});
      __syncthreads();
    }
    last = cur;
  }

  // ---- bias, one rounding, store: of a 32 x 32 tile a lane holds row l % 32 and, in registers 4 g .. 4 g + 3, the
  // columns 8 g + 4 (l / 32) .. + 3.  By way of the wave's own LDS, so that a store writes whole lines (256 bytes of four rows instead
  // of 16 bytes of 32 rows, lines that had to be read before they could be written: seven linears of 32768 rows 11.43 -> 10.79 ms), and
  // past the L2's lines of X and W (10.80 -> 10.57 ms).  Also where results are small and read soon: us with all of them past the L2 /
  // those below 64 MB through it / 16 bytes of 32 rows a store, 777 rows of 4096 x 11008: up alone 84.5 / 85.3 / 93.7, up and the down
  // that reads it 182 / 170 / 184, gate, up, their product and down 262 / 263 / 285; the same with every row routed 102.0 / 103.5 /
  // 115.5, 204 / 205 / 223, 316 / 318 / 350; up of 1805 rows of 192 x 7488, every row routed, 30.7 / 33.6 / 45.9.
  const bool bad = ctl[1] != 0;
  __syncthreads();
  unsigned char* const mine = lds + wave * (128 * kOutPitch);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int c = j * 32 + g * 8 + (lane >> 5) * 4, n = n0 + wn * 128 + c;
      float bv[4] = {0.f, 0.f, 0.f, 0.f};
      if (p.bias && n < p.d2) {
#pragma unroll
        for (int e = 0; e < 4; ++e) bv[e] = bf16_to_f32(p.bias[n + e]);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        u32x2 v;
        v[0] = pack_bf16x2(acc[i][j][4 * g] + bv[0], acc[i][j][4 * g + 1] + bv[1]);
        v[1] = pack_bf16x2(acc[i][j][4 * g + 2] + bv[2], acc[i][j][4 * g + 3] + bv[3]);
        *(u32x2*)(mine + (i * 32 + (lane & 31)) * kOutPitch + c * 2) = v;
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0xc07f);  // the wave's own writes, read by its other lanes
  asm volatile("" ::: "memory");
  {
    const int n = n0 + wn * 128 + (lane & 15) * 8;
    const int64_t mw = m0 + wm * 128 + (lane >> 4);
    bf16_t* y = p.Y + (size_t)mw * p.d2 + n;
    const unsigned char* q = mine + (lane >> 4) * kOutPitch + (lane & 15) * 16;
    if (n < p.d2)
#pragma unroll 4
      for (int it = 0; it < 32; ++it) {
        if (mw + it * 4 < p.M) {
          const u32x4_a8 v = *(const u32x4*)(q + it * 4 * kOutPitch);
          __builtin_nontemporal_store(v, (u32x4_a8*)(y + (size_t)(it * 4) * p.d2));
        }
      }
  }

  // ---- what the stages could not take: products with the tenant's own Inf and NaN, onto the stored results (no finite part of
  // them matters any more)
  if (bad) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    for (int i = 0; i < 4; ++i) {
      const int64_t m = m0 + wm * 128 + i * 32 + (lane & 31);
      if (m >= p.M) continue;
      const int64_t req = p.row_to_req ? (int64_t)p.row_to_req[m] : p.row_base + m;
      int tenant = 0;
      const int r = (req >= 0 && req < p.B) ? routed_rank(p.ad, p.tenant_id, p.route, (int)req, p.B, p.site, &tenant) : 0;
      for (int c = 0; c < r; ++c) {
        gbf16* b = in_global(p.ad.B[tenant * MILORA_NUM_SITES + p.site]) + (size_t)c * p.d2;
        float t = 0.f;
        for (int k = 0; k < p.parts; ++k) t += p.t[k * p.t_stride + (size_t)m * p.ad.r_max + c];
        for (int q = 0; q < 64; ++q) {  // this lane's columns
          const int n = n0 + wn * 128 + (q >> 4) * 32 + ((q >> 2) & 3) * 8 + (lane >> 5) * 4 + (q & 3);
          if (n >= p.d2 || (b[n] & 0x7f80u) != 0x7f80u) continue;
          bf16_t* const y = p.Y + (size_t)m * p.d2 + n;
          *y = f32_to_bf16(bf16_to_f32(*y) + t * bf16_to_f32(b[n]));
        }
      }
    }
  }
}

template <int RT, bool INFO>
__global__ void __launch_bounds__(512, 4) shrink_tiles_kernel(const ShrinkArgs g) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[8 * kShrinkWaveBytes];
  __shared__ int row_ten[RT * 16 * (INFO ? 2 : 1)];
  shrink_block<RT, 8, INFO>(g, blockIdx.x, blockIdx.y, gridDim.y, blockIdx.z, gridDim.z, smem, row_ten,
                            [](float* p, float v) { *p = v; });
  static_assert(kShrinkClear == 512, "one word per thread");
  if (INFO && g.clear && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0) g.clear[threadIdx.x] = 0;
}

template <int RT>
void launch_shrink_block(const ShrinkArgs& g, dim3 grid, hipStream_t st) {
  if (g.row_lora || g.clear) hipLaunchKernelGGL((shrink_tiles_kernel<RT, true>), grid, dim3(512), 0, st, g);
  else hipLaunchKernelGGL((shrink_tiles_kernel<RT, false>), grid, dim3(512), 0, st, g);
}

}  // namespace

bool prefill_supported(int64_t M, int d1, int d2, const void* X, const void* W, const void* Y) {
  if (M < 64 || d1 % kTK != 0 || d2 % 16 != 0) return false;
  if ((((uintptr_t)X | (uintptr_t)W) & 15) != 0 || ((uintptr_t)Y & 7) != 0) return false;
  return (uint64_t)d2 * (uint64_t)d1 * 2u < (1ull << 32);  // 32-bit byte offsets inside W (X is cut into row slices)
}

int routed_linear_prefill(const bf16_t* X, int64_t M, int d1, int d2, const int32_t* row_to_req, const bf16_t* W,
                          const bf16_t* bias, const AdapterView& ad, int site, const int32_t* tenant_id,
                          const uint8_t* route, int B, const float* t, bf16_t* Y, hipStream_t stream) {
  static thread_local int lds_set_for = -1;
  int dev = 0;
  MILORA_HIP(hipGetDevice(&dev));
  if (lds_set_for != dev) {
    MILORA_HIP(hipFuncSetAttribute((const void*)prefill_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytesP));
    lds_set_for = dev;
  }
  // rows are independent: slices whose byte offsets inside X fit 32 bits and whose tile count fits a launch
  int64_t slice = (int64_t)(((1ull << 32) - 1) / ((uint64_t)d1 * 2u)) / kTM * kTM;
  const int tilesN = (d2 + kTN - 1) / kTN;
  const int64_t by_grid = (int64_t)((1 << 24) / tilesN) * kTM;
  if (slice > by_grid) slice = by_grid;
  if (slice < kTM) return MILORA_EUNSUPPORTED;
  for (int64_t r0 = 0; r0 < M; r0 += slice) {
    PParams p;
    p.M = M - r0 < slice ? M - r0 : slice;
    p.X = X + (size_t)r0 * d1;
    p.W = W;
    p.bias = bias;
    p.Y = Y + (size_t)r0 * d2;
    p.t = t + (size_t)r0 * ad.r_max;
    p.t_stride = (size_t)M * ad.r_max;
    p.parts = shrink_parts(M, d1);
    p.row_to_req = row_to_req ? row_to_req + r0 : nullptr;
    p.row_base = r0;
    p.tenant_id = tenant_id;
    p.route = route;
    p.ad = ad;
    p.d1 = d1;
    p.d2 = d2;
    p.site = site;
    p.B = B;
    p.tilesM = (int)((p.M + kTM - 1) / kTM);
    p.tilesN = tilesN;
    const int total = p.tilesM * p.tilesN;
    const int per = (total + 7) / 8;
    hipLaunchKernelGGL(prefill_kernel, dim3(8 * per), dim3(kThreadsP), kLdsBytesP, stream, p);
    const int rc = check_launch();
    if (rc) return rc;
  }
  return MILORA_OK;
}

// LoRA shrink of the rows the tile kernel serves (same conditions as prefill_supported): t receives
// shrink_parts(M, d1) partial results [part][M][r_max], to be added in part order, row_lora (or null) what the look-ups found of
// each row; `clear` (or null) is zeroed.
int launch_shrink_tiles(const bf16_t* X, int64_t M, int d1, const int32_t* row_to_req, const AdapterView& ad, int site,
                        const int32_t* tenant_id, const uint8_t* route, int B, float* t, int2* row_lora, int* clear, hipStream_t stream) {
  const int parts = shrink_parts(M, d1);
  const int64_t slice = (int64_t)1 << 28;  // rows per launch: 512 threads for 64 rows, a grid has to stay below 2^32 threads
  for (int64_t r0 = 0; r0 < M; r0 += slice) {
    ShrinkArgs g{X + (size_t)r0 * d1, M - r0 < slice ? M - r0 : slice, r0, d1, site, B, row_to_req ? row_to_req + r0 : nullptr,
                 tenant_id, route, ad, t + (size_t)r0 * ad.r_max, (size_t)M * ad.r_max, row_lora ? row_lora + r0 : nullptr, clear};
    if (M <= kTileMaxRows) {
      // Workgroups share the units of a block (32 ranks of a tenant each) while there can be units for them and all are resident
      // at once, two per compute unit.  64 packed rows of 64 tenants, rank 256, 4096 x 4096, a call: 189 us with four at
      // most, 87 so; 45 rows of one request have one unit a block, and no workgroup comes for nothing.
      const int64_t blocks = (g.M + 15) / 16;
      const int tenants = B < ad.n_tenants ? B : ad.n_tenants;
      const int units = (tenants < 16 ? tenants : 16) * ((ad.r_max + kShrinkC - 1) / kShrinkC);
      int shares = 1;
      while (shares < units && blocks * parts * shares * 2 <= 512) shares *= 2;
      launch_shrink_block<1>(g, dim3((unsigned)blocks, parts, shares), stream);
    }
    else
      launch_shrink_block<4>(g, dim3((unsigned)((g.M + 63) / 64), parts), stream);
    const int rc = check_launch();
    if (rc) return rc;
  }
  return MILORA_OK;
}

}  // namespace milora
