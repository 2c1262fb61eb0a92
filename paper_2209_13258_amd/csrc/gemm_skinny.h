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
// multiples of 64 whatever the K block of the tile, so the order of the sum depends on the reduction length alone: not on
// the tile (the number of tokens and of columns), the slicing, the place of a slice or where the weights lie.
//
// MFMA as in the other kernels (16 x 16 x 32, k ascending); rows beyond T arrive as zeros.
//
// Measured against slices gathered and multiplied one after another: 1 token 4096 -> 16384 (128 MiB of weights, k = 8)
// 314 -> 32 us, 4.2 TB/s; 33 tokens 8192 -> 32768 (512 MiB) 641 -> 99 us, 5.4 TB/s, where a plain copy moves 4.9 TB/s.
#pragma once
#include "gemm_dma.h"

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
  int32_t by_lane;       // some K block may reach over the end of a shard or of a slice (else the tables are not needed)
};

// Element (r, c) of the weight matrix, for any lane by itself: 8 elements from a column that is a multiple of 8 on lie
// together.  The tables sit in LDS, where lanes may index them freely.
__device__ __forceinline__ const uint16_t *locate(const WeightMap &w, const uint16_t *const *shards, const uint16_t *const *dp,
                                                  int64_t r, int64_t c) {
  if (w.dp_mask) {
    const int64_t len = w.rows ? w.I : w.lay.O, x = w.rows ? r : c;
    const int64_t j = ((x + 1) * w.k - 1) / len;  // the slice with floor(j len / k) <= x < floor((j + 1) len / k)
    if ((w.dp_mask >> j) & 1ull) {
      const int64_t first = j * len / w.k;
      return dp[j] + (w.rows ? (r - first) * w.ld_dp + c : r * w.ld_dp + (c - first));
    }
  }
  const int64_t f = r * w.lay.O + c;
  const int64_t s = w.lay.rows_per_shard > 0 ? static_cast<int64_t>(static_cast<uint32_t>(r) / static_cast<uint32_t>(w.lay.rows_per_shard))
                                             : f / w.lay.L;
  return shards[s] + (f - s * w.lay.L);
}

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

template <int BM, int BN, int BK, int kStages, bool kBKc>
__global__ __launch_bounds__(kSkinnyWaves * 64, 1)
void gemm_skinny_kernel(SkinnyParams p) {
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
  const int id = logical_block(), tn = __builtin_amdgcn_readfirstlane(id / p.tiles_m);
  const int n0 = tn * BN, m0 = (id - tn * p.tiles_m) * BM;
  const int m_left = p.M - m0 < BM ? p.M - m0 : BM;

  // this wave's K blocks: a quarter of the reduction in units of 64
  static_assert(64 % BK == 0, "the waves' ranges are whole K blocks");
  const int blocks = (p.K + BK - 1) / BK, per = ((p.K + 63) / 64 + kSkinnyWaves - 1) / kSkinnyWaves * (64 / BK);
  const int b0 = wave * per, b1 = b0 + per < blocks ? b0 + per : blocks;

  // byte offset of this lane in load 0 of a block with rows of ld2 bytes; `h`: which of the two permutations
  auto lane_offset = [&](auto op, int h, uint32_t ld2) {
    using Op = decltype(op);
    return static_cast<uint32_t>(Op::row(lane)) * ld2 + Op::pos(lane, h * Op::kPermStep) * 2;
  };
  uint64_t baseA = uniform64(reinterpret_cast<uint64_t>(p.A + static_cast<int64_t>(m0) * p.lda + static_cast<int64_t>(b0) * BK)) & 0xffffffffffffull;
  const uint32_t lda2 = static_cast<uint32_t>(p.lda) * 2, bytesA = static_cast<uint32_t>(m_left) * lda2;
  const uint32_t offA[2] = {lane_offset(OpA{}, 0, lda2), lane_offset(OpA{}, 1, lda2)};

  // The weight.  A block that lies in one shard is a matrix with a base address and the row length O, and is fetched
  // like any operand; one that reaches over the end of a shard, or of a matrix with slices in DP mode, is fetched lane
  // by lane.  `first` is the flat index of the block's first element, `shard_end` where its shard ends.
  const int64_t O = p.w.lay.O, L64 = p.w.lay.L;
  const uint32_t ld2 = static_cast<uint32_t>(O) * 2;
  const int n_left = p.N - n0 < BN ? p.N - n0 : BN;
  int64_t first = kBKc ? static_cast<int64_t>(n0) * O + static_cast<int64_t>(b0) * BK : static_cast<int64_t>(b0) * BK * O + n0;
  int shard = -1;  // (none yet: the first block finds its own)
  int64_t shard_end = 0;
  uint64_t shard_base = 0;
  uint32_t offB[2] = {lane_offset(OpB{}, 0, ld2), lane_offset(OpB{}, 1, ld2)};
  if (!kBKc) {
    if (OpB::pos(lane, 0) >= n_left) offB[0] = kOutOfRange;
    if (OpB::pos(lane, OpB::kPermStep) >= n_left) offB[1] = kOutOfRange;
  }
  auto issue_weight = [&](int b, uint32_t dst) {
    const int k0 = b * BK, k_left = b < b1 ? (p.K - k0 < BK ? p.K - k0 : BK) : 0;
    const int rows = kBKc ? n_left : k_left, cols = kBKc ? k_left : n_left;  // of the block that are in the matrix
    if (first >= shard_end && shard + 1 < p.w.lay.N) {
      do {
        ++shard;
        shard_end += L64;
      } while (first >= shard_end && shard + 1 < p.w.lay.N);
      shard_base = reinterpret_cast<uint64_t>(p.w.shards.p[shard]);
    }
    const int64_t last = first + static_cast<int64_t>(rows - 1) * O + cols;
    if (!p.by_lane || (p.w.dp_mask == 0 && last <= shard_end) || k_left == 0) {
      const uint64_t base = (shard_base + static_cast<uint64_t>(first - (shard_end - L64)) * 2) & 0xffffffffffffull;
      const osdp_u32x4 rsrc = {static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(base))),
                               static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(base >> 32))),
                               static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(k_left == 0 ? 0 : rows * ld2)), 0x00020000u};
      static_for<LB>([&](auto idx) {
        constexpr int i = decltype(idx)::value;
        uint32_t lane_off = offB[(i / OpB::kPermStep) & 1];
        if (kBKc && k_left < BK) lane_off = OpB::pos(lane, i) < k_left ? lane_off : kOutOfRange;
        dma16<i * 1024>(rsrc, lane_off + static_cast<uint32_t>(i * OpB::kRowsPerLoad) * ld2, dst);
      });
    } else {
#pragma unroll 1
      for (int i = 0; i < LB; ++i) {
        const int row = i * OpB::kRowsPerLoad + OpB::row(lane), pos = OpB::pos(lane, i);
        const void *src = &kZeros;
        if (row < rows && pos < cols)
          src = locate(p.w, s_shards, s_dp, static_cast<int64_t>(kBKc ? n0 : k0) + row, static_cast<int64_t>(kBKc ? k0 : n0) + pos);
        dma16_from(src, dst + i * 1024);
      }
    }
    first += kBKc ? BK : BK * O;
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

}  // namespace
}  // namespace osdp
