// Products of a few rows (at most 128 tokens) with the whole weight, read where it lies: in the shards, or for slices in
// DP mode in the caller's replica.
//   forward  Y[T x O]  = X . W       W N-contiguous: its rows are the reduction
//   dX       dX[T x I] = dY . W^T    W K-contiguous
// These are bound by the bytes of W.  With one row of tiles every weight is used by one workgroup once, so a staged
// copy would only add a write and a second read of W (and a launch per slice, each over a fraction of the columns): the
// gather happens in the loads instead, from the shards straight into LDS, one launch for the operator, and nothing is
// staged at all.  What counts is the bytes in flight: a workgroup owns BN output columns, its four waves take a quarter
// of the reduction each, and every wave streams its own K blocks through its own ring of LDS stages with no barrier
// until the four partial sums meet at the end, added in ascending order of k and rounded once.  The quarters end on
// multiples of 32 (dX: 64) whatever the K block of the tile, so the order of the sum depends on the reduction length alone:
// not on the tile (the number of tokens and of columns), the slicing, the place of a slice or where the weights lie.
//
// MFMA as in the other kernels (16 x 16 x 32, k ascending); rows beyond T arrive as zeros.
//
// Measured against slices gathered and multiplied one after another: 1 token 4096 -> 16384 (128 MiB of weights, k = 8)
// 314 -> 32 us, 4.2 TB/s; 33 tokens 8192 -> 32768 (512 MiB) 641 -> 99 us, 5.4 TB/s, where a plain copy moves 4.9 TB/s.
#pragma once
#include "gemm_dma.h"
#include "gemm_w4.h"

namespace osdp {
namespace {

constexpr int kSkinnyWaves = 4;

struct SkinnyParams {
  int32_t M, N, K;       // tokens, output columns, reduction length
  const uint16_t *A;     // X or dY
  int64_t lda;
  uint16_t *C;           // Y or dX
  int64_t ldc;
  WeightMap w;
  int32_t tiles_m;       // row tiles; more than one only where that spreads a small product over more CUs
  int32_t by_lane;       // some K block may lie in more than one array: lanes need the tables
};

// n / d for 0 <= n < 2^45 and a quotient below 2^22, exactly: what the division in 64 bits rounds away (2^-53 of the
// quotient) is less than the 1 / d that keeps a quotient from the next integer.  A fraction of an integer division's cost.
__device__ __forceinline__ int32_t quotient(int64_t n, int64_t d) {
  return static_cast<int32_t>(static_cast<double>(n) / static_cast<double>(d));
}

// The slice that holds row or column x (slice j is [floor(j len / k), floor((j + 1) len / k))), and where it begins.
// Only plans with slices in DP mode ask: k <= 64, and len < 2^22, so 32 bits hold every product.
__device__ __forceinline__ uint32_t slice_of(const WeightMap &w, uint32_t x, uint32_t len) {
  return ((x + 1) * static_cast<uint32_t>(w.k) - 1) / len;
}
__device__ __forceinline__ uint32_t slice_begin(const WeightMap &w, uint32_t j, uint32_t len) {
  return j * len / static_cast<uint32_t>(w.k);
}

// Element (r, c) of the weight matrix, for any lane by itself: 8 elements from a column that is a multiple of 8 on lie
// together.  The tables sit in LDS, where lanes may index them freely.
__device__ __forceinline__ const uint16_t *locate(const WeightMap &w, const uint16_t *const *shards, const uint16_t *const *dp,
                                                  uint32_t r, uint32_t c) {
  if (w.dp_mask) {
    const uint32_t len = static_cast<uint32_t>(w.rows ? w.I : w.lay.O), x = w.rows ? r : c, j = slice_of(w, x, len);
    if ((w.dp_mask >> j) & 1ull) {
      const int64_t d = x - slice_begin(w, j, len);
      return dp[j] + (w.rows ? d * w.ld_dp + c : r * w.ld_dp + d);
    }
  }
  const int64_t f = static_cast<int64_t>(r) * w.lay.O + c;
  const int64_t s = w.lay.rows_per_shard > 0 ? static_cast<int64_t>(r / static_cast<uint32_t>(w.lay.rows_per_shard)) : quotient(f, w.lay.L);
  return shards[s] + (f - s * w.lay.L);
}

// Where a wave's K blocks of the weight come from: as long as they lie in one array (one shard, or one slice's replica)
// they are boxes of one matrix, and only the base address moves.  Everything is common to the wave.
struct WeightRun {
  uint64_t base = 0;  // the block's first element
  uint32_t ld2 = 0;   // bytes from one of its rows to the next
  int32_t left = 0;   // blocks from this one on that lie in the same array

  // Looks the block of `rows` x `cols` elements at (r, c) up; the next blocks lie `step` further along the reduction, the
  // rows (kBKc: the columns).  left = 0: the block lies in more than one array, or in a replica whose row length is
  // beyond the loads' 32-bit offsets.
  template <bool kBKc>
  __device__ __forceinline__ void find(const WeightMap &w, int r, int c, int rows, int cols, int step) {
    const uint32_t along = static_cast<uint32_t>(kBKc ? cols : rows);
    uint32_t room = 0x7fffffff;  // elements along the reduction from the block's first one to the end of its array
    if (w.dp_mask) {
      const uint32_t len = static_cast<uint32_t>(w.rows ? w.I : w.lay.O);
      const uint32_t x = static_cast<uint32_t>(w.rows ? r : c), j = __builtin_amdgcn_readfirstlane(slice_of(w, x, len));
      const uint32_t end = __builtin_amdgcn_readfirstlane(slice_begin(w, j + 1, len));
      if ((w.rows != 0) != kBKc) room = end - x;  // (the slices cut the reduction)
      const bool inside = x + static_cast<uint32_t>(w.rows ? rows : cols) <= end;
      if ((w.dp_mask >> j) & 1ull) {
        const int64_t d = x - __builtin_amdgcn_readfirstlane(slice_begin(w, j, len));
        base = reinterpret_cast<uint64_t>(w.dp.p[j]) + static_cast<uint64_t>(w.rows ? d * w.ld_dp + c : r * w.ld_dp + d) * 2;
        ld2 = static_cast<uint32_t>(w.ld_dp) * 2;
        left = inside && w.ld_dp < (1 << 22) ? static_cast<int32_t>((room - along) / step) + 1 : 0;
        return;
      }
      if (!inside) {
        left = 0;
        return;
      }
    }
    const uint32_t per_shard = static_cast<uint32_t>(w.lay.rows_per_shard);
    int64_t first;  // the block's first element, in its shard
    uint32_t s;
    if (per_shard > 0) {
      s = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(r) / per_shard);
      const uint32_t row = r - s * per_shard, rows_left = per_shard - row;
      if (rows_left < static_cast<uint32_t>(rows)) {
        left = 0;
        return;
      }
      if (!kBKc && rows_left < room) room = rows_left;
      first = static_cast<int64_t>(row) * w.lay.O + c;
    } else {
      const int64_t f = static_cast<int64_t>(r) * w.lay.O + c;
      s = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(quotient(f, w.lay.L)));
      first = f - s * w.lay.L;
      const int64_t behind = w.lay.L - first;  // what of the shard follows from there
      int64_t fits;
      if (kBKc) fits = behind - static_cast<int64_t>(rows - 1) * w.lay.O;
      else fits = behind < cols ? 0 : quotient(behind - cols, w.lay.O) + 1;
      if (fits < room) room = fits < 0 ? 0 : static_cast<uint32_t>(fits);
    }
    base = reinterpret_cast<uint64_t>(w.shards.p[s]) + static_cast<uint64_t>(first) * 2;
    ld2 = static_cast<uint32_t>(w.lay.O) * 2;
    left = room >= along ? static_cast<int32_t>((room - along) / step) + 1 : 0;
  }
};

// A wave-level direct-to-LDS load from 64 addresses of their own.
__device__ __forceinline__ void dma16_from(const void *src, uint32_t dst) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane(dst);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(m0), "v"(src) : "memory");
}

// 16 bytes of zeros for the lanes of such a load that lie outside the matrix.
__device__ __constant__ const uint4 kZeros = {0u, 0u, 0u, 0u};

// One K block of an operand (BN of its rows or columns) in LDS, filled and read by one wave.
//   K-contiguous (X, dY; the weight in dX): [BN][BK], as DmaOperand.
//   N-contiguous (forward): [BK][BN] with the 32-byte pieces of a k-row permuted, so that the eight k-rows that the
//       lanes of one transposing-read phase touch (k .. k+3 and the same + 8) lie in eight different 32-byte bank
//       groups: rows of 256 bytes as DmaOperand does it, rows of 128 bytes by bits 1 and 3 of k.
template <bool kKC, int BN, int BK>
struct SkinnyOperand {
  using Kc = DmaOperand<true, BN, BK, 1>;
  static_assert(kKC || BN == 64 || BN == 128, "N-contiguous blocks are 64 or 128 columns wide");
  static constexpr int kElems = BN * BK, kLoads = kElems / 512;
  static constexpr int kVec = kKC ? BK / 8 : BN / 8;  // 16-byte pieces in a row of the block
  static constexpr int kRowsPerLoad = 64 / kVec;
  // the loads p of a wave use two permutations in turn, (p / kPermStep) & 1
  static constexpr int kPermStep = !kKC && BN == 128 ? 2 : 1;
  static __device__ __forceinline__ int swz(int k) {
    return BN == 128 ? ((k & 3) << 5) | (((k >> 3) & 1) << 4) : (((k >> 1) & 1) | (((k >> 3) & 1) << 1)) << 4;
  }
  // row of the block that this lane fetches in load 0, and the position in the row (elements) in load p
  static __device__ __forceinline__ int row(int lane) { return lane / kVec; }
  static __device__ __forceinline__ int pos(int lane, int p) {
    const int r = p * kRowsPerLoad + row(lane);
    return kKC ? ((lane % kVec) ^ Kc::swz_k(r)) * 8 : ((lane % kVec) * 8) ^ swz(r);
  }
  static __device__ __forceinline__ bf16x8 frag(const uint16_t *s, int n0, int kk, int lane) {
    if constexpr (kKC) {
      return Kc::frag(s, n0, kk, lane);
    } else {
      const int i = lane & 15, k = kk * 32 + (lane >> 4) * 8 + (i >> 2);
      const uint16_t *q = s + k * BN + ((n0 + (i & 3) * 4) ^ swz(k));
      typedef dma_s16x4 __attribute__((address_space(3))) * lds_s16x4;
      const dma_s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(q));
      const dma_s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(q + 4 * BN));
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  }
};

// block(): which workgroup of the product this is (asked for where it is used: in front of everything else it costs 0.3 us).
template <int BM, int BN, int BK, int kStages, bool kBKc, class Block>
__device__ __forceinline__ void skinny_tile(const SkinnyParams &p, Block &&block) {
  constexpr int MB = BM / 16, NB = BN / 16, KS = BK / 32;
  using OpA = SkinnyOperand<true, BM, BK>;
  using OpB = SkinnyOperand<kBKc, BN, BK>;
  constexpr int LA = OpA::kLoads, LB = OpB::kLoads, L = LA + LB;
  constexpr int kStageBytes = (OpA::kElems + OpB::kElems) * 2;
  static_assert((kStages - 1) * L < 64, "in-flight loads must fit the vmcnt counter");
  constexpr int kRedLd = BN + 4;  // fp32 row of a wave's partial sums (16 bytes of padding: rows start on different banks)
  static_assert(kStages * kStageBytes >= BM * kRedLd * 4, "the partial sums reuse the ring");
  extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];
  __shared__ const uint16_t *s_shards[OSDP_MAX_SHARDS], *s_dp[OSDP_MAX_SHARDS];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, q4 = lane >> 4;
  if (p.by_lane) {
    if (tid < OSDP_MAX_SHARDS) {
      s_shards[tid] = static_cast<const uint16_t *>(p.w.shards.p[tid]);
      s_dp[tid] = static_cast<const uint16_t *>(p.w.dp.p[tid]);
    }
    __syncthreads();
  }
  const int id = block(), tn = __builtin_amdgcn_readfirstlane(id / p.tiles_m);
  const int n0 = tn * BN, m0 = (id - tn * p.tiles_m) * BM;
  const int m_left = p.M - m0 < BM ? p.M - m0 : BM;

  // this wave's K blocks: a quarter of the reduction, in units of the largest K block of any tile
  constexpr int kUnit = kBKc ? 64 : 32;
  static_assert(kUnit % BK == 0, "the waves' ranges are whole K blocks");
  const int blocks = (p.K + BK - 1) / BK, per = ((p.K + kUnit - 1) / kUnit + kSkinnyWaves - 1) / kSkinnyWaves * (kUnit / BK);
  const int b0 = wave * per, b1 = b0 + per < blocks ? b0 + per : blocks;

  // byte offset of this lane in load 0 of a block with rows of ld2 bytes; `h`: which of the two permutations
  auto lane_offset = [&](auto op, int h, uint32_t ld2) {
    using Op = decltype(op);
    return static_cast<uint32_t>(Op::row(lane)) * ld2 + Op::pos(lane, h * Op::kPermStep) * 2;
  };
  uint64_t baseA = uniform64(reinterpret_cast<uint64_t>(p.A + static_cast<int64_t>(m0) * p.lda + static_cast<int64_t>(b0) * BK)) & 0xffffffffffffull;
  const uint32_t lda2 = static_cast<uint32_t>(p.lda) * 2, bytesA = static_cast<uint32_t>(m_left) * lda2;
  const uint32_t offA[2] = {lane_offset(OpA{}, 0, lda2), lane_offset(OpA{}, 1, lda2)};

  // The weight.  A block that lies in one array is fetched like any operand, and mostly the next one does too: plans with
  // slices in DP mode run at the rate of those without.  A block that reaches over the end of a shard or of a slice is
  // fetched lane by lane, which the address arithmetic bounds (128 tokens 4096 -> 16384, every slice in DP mode: dX and dW
  // 286 us with all blocks by lane, 104 us like this).  In dX the blocks hold the same rows all along: where a row lies in
  // one array, each lane finds its rows once (128 tokens 1024 -> 4096, 64 shards of 16 rows: dX and dW 51 -> 28 us).
  const int n_left = p.N - n0 < BN ? p.N - n0 : BN;
  WeightRun run;
  uint32_t offB[2] = {0, 0};
  bool by_row = false;
  const uint16_t *lane_row[kBKc ? LB : 1];
  auto issue_weight = [&](int b, uint32_t dst) {
    const int k0 = b * BK, k_left = b < b1 ? (p.K - k0 < BK ? p.K - k0 : BK) : 0;
    const int rows = kBKc ? n_left : k_left, cols = kBKc ? k_left : n_left;  // of the block that are in the matrix
    if (__builtin_expect(run.left == 0 && k_left > 0 && !by_row, 0)) {
      run.template find<kBKc>(p.w, kBKc ? n0 : k0, kBKc ? k0 : n0, rows, cols, BK);
      run.base = uniform64(run.base) & 0xffffffffffffull;
      run.left = __builtin_amdgcn_readfirstlane(run.left);
      run.ld2 = __builtin_amdgcn_readfirstlane(run.ld2);
      offB[0] = lane_offset(OpB{}, 0, run.ld2);
      offB[1] = lane_offset(OpB{}, 1, run.ld2);
      if (!kBKc) {
        if (OpB::pos(lane, 0) >= n_left) offB[0] = kOutOfRange;
        if (OpB::pos(lane, OpB::kPermStep) >= n_left) offB[1] = kOutOfRange;
      }
      if constexpr (kBKc) {
        if (run.left == 0 && p.w.lay.rows_per_shard > 0 && (p.w.dp_mask == 0 || p.w.rows)) {
          by_row = true;
          static_for<LB>([&](auto idx) {
            constexpr int i = decltype(idx)::value;
            const int row = i * OpB::kRowsPerLoad + OpB::row(lane);
            lane_row[i] = locate(p.w, s_shards, s_dp, n0 + (row < n_left ? row : n_left - 1), 0);
          });
        }
      }
    }
    if (__builtin_expect(run.left > 0 || k_left == 0, 1)) {
      const osdp_u32x4 rsrc = {static_cast<uint32_t>(run.base), static_cast<uint32_t>(run.base >> 32),
                               k_left == 0 ? 0 : rows * run.ld2, 0x00020000u};
      static_for<LB>([&](auto idx) {
        constexpr int i = decltype(idx)::value;
        uint32_t lane_off = offB[(i / OpB::kPermStep) & 1];
        if (kBKc && k_left < BK) lane_off = OpB::pos(lane, i) < k_left ? lane_off : kOutOfRange;
        dma16<i * 1024>(rsrc, lane_off + static_cast<uint32_t>(i * OpB::kRowsPerLoad) * run.ld2, dst);
      });
      run.base += kBKc ? BK * 2 : BK * run.ld2;
      run.left -= 1;
    } else if (kBKc && by_row) {
      static_for<LB>([&](auto idx) {
        constexpr int i = decltype(idx)::value;
        const int row = i * OpB::kRowsPerLoad + OpB::row(lane), pos = OpB::pos(lane, i);
        const void *src = &kZeros;
        if (row < rows && pos < cols) src = lane_row[kBKc ? i : 0] + k0 + pos;
        dma16_from(src, dst + i * 1024);
      });
    } else {
#pragma unroll 1
      for (int i = 0; i < LB; ++i) {
        const int row = i * OpB::kRowsPerLoad + OpB::row(lane), pos = OpB::pos(lane, i);
        const void *src = &kZeros;
        if (row < rows && pos < cols) src = locate(p.w, s_shards, s_dp, (kBKc ? n0 : k0) + row, (kBKc ? k0 : n0) + pos);
        dma16_from(src, dst + i * 1024);
      }
    }
  };
  const uint32_t ring = lds_address(smem) + wave * (kStages * kStageBytes);
  auto issue = [&](int b, int stage) {
    const uint32_t dst = ring + stage * kStageBytes;
    const int k_left = b < b1 ? p.K - b * BK : 0;
    const osdp_u32x4 rsrc = {static_cast<uint32_t>(baseA), static_cast<uint32_t>(baseA >> 32), bytesA, 0x00020000u};
    static_for<LA>([&](auto idx) {
      constexpr int i = decltype(idx)::value;
      uint32_t lane_off = offA[i & 1];
      if (k_left < BK) lane_off = OpA::pos(lane, i) < k_left ? lane_off : kOutOfRange;
      dma16<i * 1024>(rsrc, lane_off + static_cast<uint32_t>(i * OpA::kRowsPerLoad) * lda2, dst);
    });
    baseA += BK * 2;
    issue_weight(b, dst + OpA::kElems * 2);
  };

  f32x4 acc[MB][NB];
#pragma unroll
  for (int bm = 0; bm < MB; ++bm)
#pragma unroll
    for (int bn = 0; bn < NB; ++bn) acc[bm][bn] = f32x4{0.f, 0.f, 0.f, 0.f};

  // The loop starts kStages - 1 blocks early, only to put the first blocks in flight.
  int stage = 0, fill = 0;
#pragma unroll 1
  for (int b = b0 - (kStages - 1); b < b1; ++b) {
    // block b has landed, and the fragment reads of block b - 1 are done
    if (b >= b0) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((kStages - 2) * L) : "memory");
    issue(b + kStages - 1, fill);  // into the stage of block b - 1
    fill = fill + 1 == kStages ? 0 : fill + 1;
    if (b < b0) continue;
    const uint16_t *sA = smem + (wave * kStages + stage) * (kStageBytes / 2), *sB = sA + OpA::kElems;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      bf16x8 fa[MB], fb[NB];
#pragma unroll
      for (int bm = 0; bm < MB; ++bm) fa[bm] = OpA::frag(sA, bm * 16, kk, lane);
#pragma unroll
      for (int bn = 0; bn < NB; ++bn) fb[bn] = OpB::frag(sB, bn * 16, kk, lane);
#pragma unroll
      for (int bn = 0; bn < NB; ++bn)
#pragma unroll
        for (int bm = 0; bm < MB; ++bm) acc[bm][bn] = mma_16x16x32(fa[bm], fb[bn], acc[bm][bn]);
    }
    stage = stage + 1 == kStages ? 0 : stage + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the blocks beyond the last one too: the ring is used again)
  __syncthreads();
  float *red = reinterpret_cast<float *>(smem);
#pragma unroll
  for (int bm = 0; bm < MB; ++bm)
#pragma unroll
    for (int bn = 0; bn < NB; ++bn)
      *reinterpret_cast<f32x4 *>(red + (wave * BM + bm * 16 + l16) * kRedLd + bn * 16 + 4 * q4) = acc[bm][bn];
  __syncthreads();
  for (int i = tid; i < BM * BN / 4; i += kSkinnyWaves * 64) {
    const int m = i / (BN / 4), n = (i % (BN / 4)) * 4;
    if (m >= m_left || n >= n_left) continue;
    f32x4 c = *reinterpret_cast<const f32x4 *>(red + m * kRedLd + n);
#pragma unroll
    for (int w = 1; w < kSkinnyWaves; ++w) {
      const f32x4 d = *reinterpret_cast<const f32x4 *>(red + (w * BM + m) * kRedLd + n);
#pragma unroll
      for (int e = 0; e < 4; ++e) c[e] += d[e];
    }
    store_global8(p.C + static_cast<int64_t>(m0 + m) * p.ldc + n0 + n, uint2{pack_bf16x2(c[0], c[1]), pack_bf16x2(c[2], c[3])});
  }
}

template <int BM, int BN, int BK, int kStages, bool kBKc>
__global__ __launch_bounds__(kSkinnyWaves * 64, 1)
void gemm_skinny_kernel(SkinnyParams p) {
  skinny_tile<BM, BN, BK, kStages, kBKc>(p, [] { return logical_block(); });
}

// The backward of few tokens as one launch: workgroups [0, n_dx) are those of dX, the others 128 x 128 tiles of dW into the
// shards.  Neither needs the other, both are short, and a launch of its own is what the second one costs most (128 tokens
// 256 -> 1024: dW 6.0 and dX 6.5 us, and 3 to 4 us of host time each).
template <int BM, int BK, int kStages>
__global__ __launch_bounds__(kSkinnyWaves * 64, 1)
void few_token_backward_kernel(SkinnyParams dx, GemmParams dw, int n_dx, int tiles_m, int tiles_n) {
  const int id = blockIdx.x;
  if (id < n_dx) skinny_tile<BM, 64, BK, kStages, true>(dx, [&] { return id; });
  else gemm_w4_tile<4, 4, 4, false, false, static_cast<int>(Epilogue::kBf16ShardMajor), false, false>(dw, tiles_m, tiles_n, id - n_dx);
}

}  // namespace
}  // namespace osdp
