// Device-side pieces shared by the GEMM kernels of libosdp: parameter block, bf16 rounding,
// the workgroup -> tile map, accumulator load and the three epilogues.
#pragma once
#include <utility>

#include "osdp_internal.h"

namespace osdp {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// Compile-time integers as lambda arguments.
template <int v>
struct Int {
  static constexpr int value = v;
};
// f(Int<0>{}), f(Int<1>{}), ..., f(Int<N-1>{}): a loop whose index is a compile-time constant in every iteration, so
// that register arrays are never indexed at run time and nothing depends on the optimiser's unrolling.
template <class F, int... Is>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, Is...>) {
  (f(Int<Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
  static_for_impl(static_cast<F &&>(f), std::make_integer_sequence<int, N>{});
}

// One matrix-core step of every GEMM kernel here: a 16 x 16 block of C gains the product over 32 consecutive k.
// Lane l supplies 8 consecutive k (8 * (l / 16) ..) of row / column l % 16 of each operand.  The operands are
// passed swapped (the B fragment first), so that lane l ends up with C[m = l % 16][n = 4 * (l / 16) + 0..3]:
// runs of 4 consecutive output columns.  All kernels use this one instruction with k ascending, which is what
// makes their results bit-identical whatever the tile shape.
__device__ __forceinline__ f32x4 mma_16x16x32(bf16x8 a_rows, bf16x8 b_cols, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(b_cols, a_rows, c, 0, 0, 0);
}

// A slice gather that rides along with a GEMM launch (four-wave kernel only): the copy Ws[r, c] = W[r0 + r, c0 + c]
// of osdp_gather.hip, cut into one piece of 256 vectors per workgroup and K block and issued between the
// MFMAs (it saves the launch, not the memory time: the kernel is bound by the same memory pipe).  dst is the dense destination, total_vecs its size in 16-byte vectors (below 2^32).
struct GatherJob {
  ShardTable src;
  ShardLayout lay;
  uint32_t r0;
  uint32_t vecs_per_row;
  uint64_t c0;
  uint64_t total_vecs;
  uint4 *dst;
};

struct GemmParams {
  int32_t M, N, K;
  const uint16_t *A;
  int64_t lda;
  const uint16_t *B;
  int64_t ldb;
  const uint16_t *B2;  // second B segment: K-contiguous B, rows k >= k_split; N-contiguous B, columns n >= n_split
  int64_t ldb2;
  int32_t k_split;     // 0: none
  int32_t n_split;     // 0: none
  // B read from the weight shards instead of a staged slice (ldb = O; the shards are in `shards`): each holds seg_k rows
  // of an N-contiguous B (multiple of 64), or seg_n rows, which are columns of C, of a K-contiguous one.  0: not so.
  int32_t seg_k, seg_n;
  int32_t k_parts;     // > 1 (fp32 workspace epilogue with ldc = N, no second K segment): the grid is k_parts times the
                       // tiles, part s takes k in [s K / k_parts, (s + 1) K / k_parts) and writes plane s of C ([M x N] fp32 each)
  void *C;
  int64_t ldc;
  const float *acc_in;
  int64_t ld_acc;
  ShardLayout lay;
  int64_t c0;          // shard-major epilogue: column of the full matrix where C starts
  int64_t r0;          // shard-major epilogue: row of the full matrix where C starts
  ShardTable shards;
  GatherJob job;       // only read by kernels instantiated to carry one
};

// Two fp32 values rounded to bf16, nearest even, in one instruction (v_cvt_pk_bf16_f32): in integer arithmetic the same
// rounding takes about ten instructions a value, a third of what an epilogue used to execute.  The same bits for all 2^32
// inputs (NaN stays NaN, quiet, with the upper bits of its payload).
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  const bf16x2 v = {static_cast<__bf16>(lo), static_cast<__bf16>(hi)};
  return __builtin_bit_cast(uint32_t, v);
}

// Tile index of this workgroup.  Workgroups are dealt round-robin to the 8 XCDs, each with its
// own L2, so consecutive logical tile ids are first mapped onto one XCD; logical ids then walk
// the tile grid in column-major groups of kGroupM tile rows, which keeps the tiles that run
// together on an XCD inside a small patch of A row panels and B column panels (4 measured best of 2..16).
constexpr int kXcds = 8;
constexpr int kGroupM = 4;

// Logical id of this workgroup: the ids an XCD runs are consecutive.
__device__ __forceinline__ int logical_block() {
  const int nb = gridDim.x, bid = blockIdx.x;
  const int xcd = bid % kXcds, idx = bid / kXcds;
  const int base = nb / kXcds, rem = nb % kXcds;
  return xcd * base + (xcd < rem ? xcd : rem) + idx;
}

__device__ __forceinline__ void tile_of_pid(int pid, int tiles_m, int tiles_n, int *tm, int *tn) {
  const int per_group = kGroupM * tiles_n;
  const int group = pid / per_group, in_group = pid - group * per_group;
  const int first_m = group * kGroupM;
  const int gm = (tiles_m - first_m) < kGroupM ? (tiles_m - first_m) : kGroupM;
  // (the divisions run on the vector unit; what follows from the tile's place belongs in scalar registers)
  *tm = __builtin_amdgcn_readfirstlane(first_m + in_group % gm);
  *tn = __builtin_amdgcn_readfirstlane(in_group / gm);
}

// Columns [n0, n_end) of C that tile column tn covers.  With seg_n tiles do not reach over the end of a shard.
template <bool kBKc>
__device__ __forceinline__ void tile_columns(const GemmParams &p, int tn, int BN, int *n0, int *n_end) {
  *n0 = tn * BN;
  *n_end = p.N;
  if (kBKc && p.seg_n) {
    const int per = (p.seg_n + BN - 1) / BN, s = __builtin_amdgcn_readfirstlane(tn / per);
    *n0 = s * p.seg_n + (tn - s * per) * BN;
    *n_end = (s + 1) * p.seg_n;
  }
}

// Accumulator layout of one wave: acc[bm][bn][i] is C[m][n] with
//   m = m_base + 16*bm + l16,  n = n_base + 16*bn + 4*q + i        (l16 = lane % 16, q = lane / 16).
// Outside the matrix (n_end: the end of the tile's columns) the load repeats the last row / column group (the values are never stored) and the store does
// nothing; N is a multiple of 8 and n of 4, so the 4 columns are in or out together.
template <int MB, int NB>
__device__ __forceinline__ void load_acc_tile(const GemmParams &p, f32x4 (&acc)[MB][NB], int m_base, int n_base,
                                              int n_end, int l16, int q) {
#pragma unroll
  for (int bm = 0; bm < MB; ++bm)
#pragma unroll
    for (int bn = 0; bn < NB; ++bn) {
      const int m = m_base + bm * 16 + l16, n = n_base + bn * 16 + 4 * q;
      const float *src = p.acc_in + static_cast<int64_t>(m < p.M ? m : p.M - 1) * p.ld_acc + (n < n_end ? n : n_end - 4);
      const float4 c = *reinterpret_cast<const float4 *>(src);
      acc[bm][bn][0] = c.x;
      acc[bm][bn][1] = c.y;
      acc[bm][bn][2] = c.z;
      acc[bm][bn][3] = c.w;
    }
}

// Stores 4 consecutive columns of row m starting at column n according to the epilogue.
template <int kEpi>
__device__ __forceinline__ void store_acc4(const GemmParams &p, f32x4 c, int m, int n, uint16_t *const *s_tab) {
  if (kEpi == static_cast<int>(Epilogue::kF32Workspace)) {
    float4 o = {c[0], c[1], c[2], c[3]};
    *reinterpret_cast<float4 *>(static_cast<float *>(p.C) + static_cast<int64_t>(m) * p.ldc + n) = o;
    return;
  }
  uint2 o = {pack_bf16x2(c[0], c[1]), pack_bf16x2(c[2], c[3])};
  uint16_t *dst;
  if (kEpi == static_cast<int>(Epilogue::kBf16RowMajor)) {
    dst = static_cast<uint16_t *>(p.C) + static_cast<int64_t>(m) * p.ldc + n;
  } else {
    int s;
    int64_t off;
    const int row = m + static_cast<int>(p.r0);
    if (p.lay.rows_per_shard > 0) {
      s = row / p.lay.rows_per_shard;
      off = static_cast<int64_t>(row - s * p.lay.rows_per_shard) * p.lay.O + p.c0 + n;
    } else {
      const int64_t f = static_cast<int64_t>(row) * p.lay.O + p.c0 + n;
      s = static_cast<int>(f / p.lay.L);
      off = f - static_cast<int64_t>(s) * p.lay.L;
    }
    dst = s_tab[s] + off;
  }
  store_global8(dst, o);
}

// One wave's share of the result, 16 * MB x 16 * NB from row m_base and column n_base on; read(bm, bn) gives a block's
// accumulators (indices are compile-time).  Rows from p.M and columns from n_end on are left out.  plane_row: added to the
// row where the tile is stored (launches that run parts of the reduction), not to the bound.
//
// An epilogue is straight-line code that every wave runs once a tile, so its length is what it costs: fetched for the first
// time, it runs as fast as the instructions arrive.  One row block therefore takes one address, and everything else is an
// immediate offset; where a row lies in the shards is worked out once and then carried from row block to row block (the
// division, once per block of 16 x 16 in either layout, was what made the kernels 180 KB long).  bf16 results of two
// neighbouring blocks change lanes (v_permlane16_swap) so that a lane holds 8 columns: 16 bytes a store, 64 a row.
// 4096 x 4096 over K = 512 in 256 x 256 tiles, one to a CU, forward / dX / dW into shards: 28.4 / 28.0 / 51.5 us before,
// 23.8 / 22.8 / 34.9 now (dW with the gather it carries); 8192^3 in four rounds 768 / 776 / 819 and 765 / 764 / 765.
template <int MB, int NB, int kEpi, class Read>
__device__ __forceinline__ void store_tile(const GemmParams &p, Read &&read, int m_base, int n_base, int n_end,
                                           int plane_row, int l16, int q, uint16_t *const *s_tab) {
  const int m = m_base + l16;
  if constexpr (kEpi == static_cast<int>(Epilogue::kF32Workspace)) {
    float *dst = static_cast<float *>(p.C) + static_cast<int64_t>(plane_row + m) * p.ldc + n_base + 4 * q;
    static_for<MB>([&](auto bm_) {
      constexpr int bm = decltype(bm_)::value;
      const bool row = m + 16 * bm < p.M;
      static_for<NB>([&](auto bn_) {
        constexpr int bn = decltype(bn_)::value;
        if (row && n_base + 16 * bn + 4 * q < n_end) {
          const f32x4 c = read(Int<bm>{}, Int<bn>{});
          *reinterpret_cast<float4 *>(dst + 16 * bn) = float4{c[0], c[1], c[2], c[3]};
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      dst += static_cast<int64_t>(16) * p.ldc;
    });
    return;
  }
  constexpr bool kShards = kEpi == static_cast<int>(Epilogue::kBf16ShardMajor);
  // Blocks 2 i and 2 i + 1 side by side: lane group q has columns 8 * (q / 2) .. of block 2 i + (q & 1); a last block
  // without a neighbour keeps its four columns a lane.
  const int col = 16 * (q & 1) + 8 * (q >> 1), tail = 16 * (NB - 1) + 4 * q;
  uint16_t *dst = nullptr;   // where column n_base + col of the lane's row goes
  int64_t off = 0;           // shards: its offset in shard s
  int s = 0;
  if constexpr (kShards) {
    const int64_t row = m + p.r0, c = p.c0 + n_base + col;
    if (p.lay.rows_per_shard > 0) {
      s = static_cast<int>(static_cast<uint32_t>(row) / static_cast<uint32_t>(p.lay.rows_per_shard));
      off = (row - static_cast<int64_t>(s) * p.lay.rows_per_shard) * p.lay.O + c;
    } else {
      const uint64_t f = static_cast<uint64_t>(row * p.lay.O + c);
      s = static_cast<int>(f / static_cast<uint64_t>(p.lay.L));
      off = static_cast<int64_t>(f - static_cast<uint64_t>(s) * static_cast<uint64_t>(p.lay.L));
    }
  } else {
    dst = static_cast<uint16_t *>(p.C) + static_cast<int64_t>(m) * p.ldc + n_base + col;
  }
  static_for<MB>([&](auto bm_) {
    constexpr int bm = decltype(bm_)::value;
    const bool row = m + 16 * bm < p.M;  // (rows ascend: a lane outside stays outside, and its place is not looked up)
    if constexpr (kShards) {
      if (row) {
        while (off >= p.lay.L) {
          off -= p.lay.L;
          ++s;
        }
        dst = s_tab[s] + off;
      }
    }
    // columns `by` further on (of a general flat map they may lie in a later shard)
    auto place = [&](int by) {
      uint16_t *at = dst + by;
      if constexpr (kShards) {
        if (off + by >= p.lay.L) {
          int64_t o = off + by;
          int t = s;
          while (o >= p.lay.L) {
            o -= p.lay.L;
            ++t;
          }
          at = s_tab[t] + o;
        }
      }
      return at;
    };
    static_for<NB / 2>([&](auto i_) {
      constexpr int i = decltype(i_)::value;
      const f32x4 c = read(Int<bm>{}, Int<2 * i>{}), d = read(Int<bm>{}, Int<2 * i + 1>{});
      const auto lo = __builtin_amdgcn_permlane16_swap(pack_bf16x2(c[0], c[1]), pack_bf16x2(d[0], d[1]), false, false);
      const auto hi = __builtin_amdgcn_permlane16_swap(pack_bf16x2(c[2], c[3]), pack_bf16x2(d[2], d[3]), false, false);
      if (row && n_base + 32 * i + col < n_end) store_global16(place(32 * i), uint4{lo[0], hi[0], lo[1], hi[1]});
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (NB % 2) {
      const f32x4 c = read(Int<bm>{}, Int<NB - 1>{});
      if (row && n_base + tail < n_end)
        store_global8(place(tail - col), uint2{pack_bf16x2(c[0], c[1]), pack_bf16x2(c[2], c[3])});
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (kShards) off += static_cast<int64_t>(16) * p.lay.O;
    else dst += static_cast<int64_t>(16) * p.ldc;
  });
}

}  // namespace
}  // namespace osdp
