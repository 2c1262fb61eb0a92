// Eight-wave GEMM kernel of libosdp, and the operand layouts that the others share: tiles stream from global memory straight into LDS
// (global_load_lds_dwordx4, no staging registers), a ring of LDS stages keeps one or more K
// blocks in flight behind the MFMAs (v_mfma_f32_16x16x32_bf16), and operand fragments are
// double-buffered in registers.
//
// Any M, N >= 1 and K >= 1 (M, N multiples of 8 where the operand is MN-contiguous, K where it is K-contiguous: a
// 16-byte load is inside the matrix or outside it as a whole).  The edges cost the K loop nothing: operands are fetched
// with buffer loads, whose hardware range check delivers zeros for what lies outside, so a tile at the edge runs the
// same instructions as any other and only its stores are guarded (OperandSource below).  Measured against sending such
// shapes to the bounds-checked kernel: a layer of 2560 features over 3001 tokens, forward and backward, 7.39 -> 1.62 ms;
// slices of 640 and 160 columns over 8192 tokens 7.76 -> 4.01 ms; 500 tokens 2560 -> 10240 forward 562 -> 118 us.
// The K loop is uniform: it goes on asking for K blocks beyond the last one, which the range check turns into zeros
// that nobody reads.  Without the branches of a loop that stops asking it has a third fewer scalar instructions
// (dW of 4096 x 1024 over 8192 tokens 87 -> 81 us).
//
// LDS layouts.  A direct-to-LDS load of one wave deposits lane i's 16 bytes at base + 16*i, so a
// stage is a sequence of 1 KB chunks that cannot be padded; bank conflicts are avoided by
// permuting which 16 bytes of global memory each lane fetches (an XOR swizzle on the source side):
//   K-contiguous operand  [rows][BK]   : 16-byte chunk c of row r is stored at chunk c ^ f(r),
//       f(r) = (r >> 1) & 7 for BK = 64, 2 * ((r >> 3) & 1) for BK = 32, so that the 16 lanes a
//       ds_read_b128 serves per cycle fall into 16 different 16-byte bank groups.
//   MN-contiguous operand [BK][rows]   : 64-byte granule w of k-row k is stored at granule
//       w ^ (k & 3) and its 32-byte halves are swapped when bit 3 of k is set, so that the k-rows the
//       lane groups of one ds_read_b64_tr_b16 phase touch fall into different bank groups.
#pragma once
#include "gemm_common.h"

namespace osdp {
namespace {

typedef __attribute__((address_space(3))) void *lds_void_ptr;
typedef const __attribute__((address_space(1))) void *global_void_ptr;
typedef __attribute__((ext_vector_type(4))) short dma_s16x4;
typedef __attribute__((ext_vector_type(8))) short dma_s16x8;

// A 64-bit value that is the same in every lane, as the compiler can see.
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

// One wave-level direct-to-LDS load: the 16 bytes at offset lane_off of lane i in the raw buffer `rsrc` land at LDS byte
// address dst + kDstOff + 16*i (rsrc and dst are common to the wave; the LDS address travels in M0).  A lane whose
// offset is not below the buffer's record count reads nothing and deposits zeros.  Written as inline assembly on
// purpose: the compiler then does not know that LDS is written asynchronously and inserts no waits of its own in front
// of the fragment reads; the kernels order these loads themselves with wait_vmcnt + barrier.
template <int kDstOff>
__device__ __forceinline__ void dma16(osdp_u32x4 rsrc, uint32_t lane_off, uint32_t dst) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane(dst);
  asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(m0), "v"(lane_off),
               "s"(rsrc), "n"(kDstOff)
               : "memory", "scc");
}

__device__ __forceinline__ uint32_t lds_address(const void *p) {
  return static_cast<uint32_t>(reinterpret_cast<size_t>((lds_void_ptr)p));
}

// s_waitcnt vmcnt(n) alone (expcnt and lgkmcnt left at their maxima), gfx9 encoding.
template <int n>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(n >= 0 && n < 64, "vmcnt is a 6-bit counter");
  __builtin_amdgcn_s_waitcnt((n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14));
}

template <bool kKC, int kRows, int kBK, int kWaves>
struct DmaOperand {
  static constexpr int kElems = kRows * kBK;             // one stage
  static constexpr int kLoads = kElems / 512 / kWaves;   // wave-level loads (1 KB each) per wave per stage
  static_assert(kLoads >= 1 && kLoads * kWaves * 512 == kElems, "stage must divide into 1 KB chunks over the waves");
  static constexpr int CPR = kBK / 8, RPL = 64 / CPR;    // K-contiguous: 16-byte chunks per row, rows per load
  static constexpr int VPR = kRows / 8, KPL = 64 / VPR;  // MN-contiguous: 16-byte vectors per k-row, k-rows per load
  static_assert(kBK == 64 || kBK == 32, "BK is 32 or 64");
  static_assert(kKC || (kRows >= 128 && kRows <= 512), "MN-contiguous tiles are 128..512 wide");

  // A ds_read_b128 is served 16 lanes at a time, and not 16 consecutive ones: measured on the box, lane 0 shares
  // its cycle with lanes 1-3, 12-15 and 20-27 (within each half of the wave the two groups are the lanes with even
  // and with odd parity of lane bits 2, 3 and 4).  With lane = 16 * q + row the swizzles below put the 16 reads
  // of every such group into 16 different 16-byte bank groups.
  static __device__ __forceinline__ int swz_k(int row) { return CPR == 8 ? ((row >> 1) & 7) : (((row >> 3) & 1) << 1); }
  // MN-contiguous: element offset mn of k-row k is stored at mn ^ swz_mn(k): the 64-byte granule index is
  // XORed with k & 3 and the 32-byte half inside the granule with bit 3 of k, so that the 8 k-rows the two
  // lane groups of one transposing-read phase touch (k, k+1, k+2, k+3 and the same + 8) fall into 8 different
  // 32-byte bank groups.
  static __device__ __forceinline__ int swz_mn(int krow) { return ((krow & 3) << 5) | (((krow >> 3) & 1) << 4); }

  // Element offset, from the tile origin (mn = 0 of the tile, k = k0), of the 16 bytes this lane fetches in
  // its wave's load 0.  Load p of the wave adds p * load_stride(); the swizzle terms do not change with p
  // because a wave's loads are a multiple of 16 rows (16 k-rows) apart.
  static __device__ __forceinline__ int64_t lane_src(int wave, int lane, int64_t ld) {
    static_assert(kKC || (kWaves * KPL) % 16 == 0, "a wave's loads must be a multiple of 16 k-rows apart");
    if (kKC) {
      const int row = wave * RPL + lane / CPR;
      const int c = (lane % CPR) ^ swz_k(row);
      return static_cast<int64_t>(row) * ld + c * 8;
    } else {
      const int krow = wave * KPL + lane / VPR;
      const int pv = lane % VPR;
      return static_cast<int64_t>(krow) * ld + ((pv * 8) ^ swz_mn(krow));
    }
  }
  // Where in the tile and K block those 16 bytes lie: the k of a K-contiguous operand, the mn of the other kind.
  static __device__ __forceinline__ int lane_pos(int wave, int lane) {
    return kKC ? ((lane % CPR) ^ swz_k(wave * RPL + lane / CPR)) * 8 : ((lane % VPR) * 8) ^ swz_mn(wave * KPL + lane / VPR);
  }
  static __device__ __forceinline__ constexpr int load_rows(int p) { return p * kWaves * (kKC ? RPL : KPL); }
  // The 1 KB chunk of the stage that load p of a wave fills: first_chunk(wave) + chunk_step(p).
  static __device__ __forceinline__ constexpr int first_chunk(int wave) { return wave; }
  static __device__ __forceinline__ constexpr int chunk_step(int p) { return p * kWaves; }

  // Fragment of the 16-row block at mn0 for K step kk (32 wide): lane (l16, q) gets k = 32*kk + 8*q + 0..7 of
  // row mn0 + l16.
  static __device__ __forceinline__ bf16x8 frag(const uint16_t *s, int mn0, int kk, int lane) {
    if (kKC) {
      const int r = mn0 + (lane & 15);
      const int c = (kk * 4 + (lane >> 4)) ^ swz_k(r);
      return *reinterpret_cast<const bf16x8 *>(s + r * kBK + c * 8);
    } else {
      // ds_read_b64_tr_b16: within 16 lanes, lane s supplies 4 consecutive mn of k-row s / 4 and lane i
      // receives the 4 k of mn i; two reads, 4 k-rows apart, give the lane its 8 consecutive k
      const int i = lane & 15;
      const int krow = kk * 32 + (lane >> 4) * 8 + (i >> 2);
      const int mn = mn0 + (i & 3) * 4;
      const uint16_t *q = s + krow * kRows + (mn ^ swz_mn(krow));
      typedef dma_s16x4 __attribute__((address_space(3))) * lds_s16x4;
      const dma_s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(q));
      const dma_s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(q + 4 * kRows));
      const dma_s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      return __builtin_bit_cast(bf16x8, both);
    }
  }
};

// Where an operand's current K block comes from: a raw buffer that starts at the tile's first element in that block.
// `Op` says which 16 bytes a lane fetches (lane_src, lane_pos, and load_rows(p) for the rows between a wave's load 0
// and load p); everything outside the matrix is put out of the buffer's range:
//   K-contiguous operand : the buffer ends where row mn_left would begin; in a K block that the reduction does not
//       fill, the lanes whose k lies beyond it get an offset outside any range.
//   MN-contiguous operand: the buffer ends where k-row krem would begin; lanes whose column lies beyond mn_left get
//       the outside offset.
// The offsets of one block stay below 2^31 because the host admits leading dimensions below 2^22 only.
constexpr uint32_t kOutOfRange = 0x80000000u;

template <class Op, bool kKC, int kRows, int kBK>
struct OperandSource {
  uint64_t base;     // the raw buffer: base address and bytes in range (common to the wave)
  uint32_t bytes;
  uint32_t lane;     // byte offset of this lane in its wave's load 0
  uint32_t ld2;      // bytes from one row to the next

  // The block at `origin`, of a tile with mn_left rows / columns of the matrix from its first one on.  (kRows, the
  // tile's own, may be fewer than the LDS layout of Op holds: the surplus lanes fetch nothing.)
  __device__ __forceinline__ void begin(const uint16_t *origin, int64_t ld, int mn_left, int wave, int lane_id) {
    mn_left = mn_left < kRows ? mn_left : kRows;
    base = uniform64(reinterpret_cast<uint64_t>(origin)) & 0xffffffffffffull;
    ld2 = static_cast<uint32_t>(ld) * 2;
    bytes = kKC ? static_cast<uint32_t>(mn_left) * ld2 : kBK * ld2;
    lane = static_cast<uint32_t>(Op::lane_src(wave, lane_id, ld) * 2);
    if (!kKC) lane = Op::lane_pos(wave, lane_id) < mn_left ? lane : kOutOfRange;
  }
  // On to the next K block.
  __device__ __forceinline__ void next() { base += kKC ? kBK * 2 : ld2 * kBK; }
  // The current block holds k_left < kBK k only (0: nothing, now and in every later block).
  __device__ __forceinline__ void cut(int k_left, int wave, int lane_id) {
    if (kKC) lane = Op::lane_pos(wave, lane_id) < k_left ? lane : kOutOfRange;
    else bytes = static_cast<uint32_t>(k_left) * ld2;
  }
  // load p of the wave; dst: LDS address of the operand's stage plus the wave's first chunk
  template <int p>
  __device__ __forceinline__ void load(uint32_t dst) const {
    const osdp_u32x4 rsrc = {static_cast<uint32_t>(base), static_cast<uint32_t>(base >> 32), bytes, 0x00020000u};
    dma16<Op::chunk_step(p) * 1024>(rsrc, lane + static_cast<uint32_t>(Op::load_rows(p)) * ld2, dst);
  }
};

// Both operands of a tile, K block by K block.  Most blocks only move the two base addresses; at `stop` something else
// is due: B goes on in its next K segment (a second staged slice, or the next shard), the last block is cut short, or
// the blocks beyond the last one, which the kernels' uniform K loops still ask for, must deliver nothing.
template <class OpA, class OpB, bool kAK, bool kBKc, int BM, int BN, int kBK>
struct TileSource {
  OperandSource<OpA, kAK, BM, kBK> a;
  OperandSource<OpB, kBKc, BN, kBK> b;
  int32_t block, stop;          // the block the sources stand at; the next one at which something is due
  int32_t n0, n_end, nb;        // the tile's columns (n_end: where those it may store end); its K blocks
  int32_t segment, segment_end; // B's K segment; the block where the next one begins

  // Block 0 of the tile of rows m0 .. and tile column tn, reducing over k0 .. k0 + K (k0 > 0 only with one K segment).
  __device__ __forceinline__ void begin(const GemmParams &p, int m0, int tn, int64_t k0, int K, int wave, int lane) {
    tile_columns<kBKc>(p, tn, BN, &n0, &n_end);
    nb = (K + kBK - 1) / kBK;
    // B may come in two column segments (two staged slices): the tile lies in one of them
    const bool second = p.n_split && n0 >= p.n_split;
    const uint16_t *base = second ? p.B2 : p.B;
    const int64_t ldb = second ? p.ldb2 : p.ldb;
    int nB = second ? n0 - p.n_split : n0;
    if (kBKc && p.seg_n) {
      const int s = __builtin_amdgcn_readfirstlane(n0 / p.seg_n);
      base = static_cast<const uint16_t *>(p.shards.p[s]);
      nB = n0 - s * p.seg_n;
    }
    if (!kBKc && p.seg_k) base = static_cast<const uint16_t *>(p.shards.p[0]);
    a.begin(kAK ? p.A + static_cast<int64_t>(m0) * p.lda + k0 : p.A + m0 + k0 * p.lda, p.lda, p.M - m0, wave, lane);
    b.begin(kBKc ? base + static_cast<int64_t>(nB) * ldb + k0 : base + nB + k0 * ldb, ldb, n_end - n0, wave, lane);
    block = segment = 0;
    segment_end = kAK && p.k_split ? p.k_split / kBK : (kAK && !kBKc && p.seg_k ? p.seg_k / kBK : 0x7fffffff);
    due(p, K, wave, lane);
  }
  __device__ __forceinline__ void due(const GemmParams &p, int K, int wave, int lane) {
    if (kAK && block == segment_end) {
      ++segment;
      const bool shards = !kBKc && p.seg_k;
      if (block < nb) {
        const uint16_t *base = shards ? static_cast<const uint16_t *>(p.shards.p[segment]) : p.B2;
        const int64_t ldb = shards ? p.ldb : p.ldb2;
        b.begin(kBKc ? base + static_cast<int64_t>(n0) * ldb : base + n0, ldb, n_end - n0, wave, lane);
      }
      segment_end = shards ? segment_end + p.seg_k / kBK : 0x7fffffff;
    }
    const int left = K - block * kBK;
    if (left < kBK) {
      a.cut(left > 0 ? left : 0, wave, lane);
      b.cut(left > 0 ? left : 0, wave, lane);
    }
    const int tail = K / kBK;  // the first block that is not full: the cut one, or the first beyond the end
    stop = block < tail ? tail : (block < nb ? nb : 0x7fffffff);
    if (kAK && segment_end < stop) stop = segment_end;
  }
  // After the last load of a block: on to the next.
  __device__ __forceinline__ void next(const GemmParams &p, int K, int wave, int lane) {
    a.next();
    b.next();
    if (__builtin_expect(++block == stop, 0)) due(p, K, wave, lane);
  }
};

// Workgroups of one tile shape that fit a CU's 160 KB of LDS together (at most 2 are aimed for), and the waves
// per SIMD that this takes: the register budget the compiler is held to.
constexpr int dma_groups_per_cu(int BM, int BN, int BK, int kStages) {
  return (2 * (kStages * (BM + BN) * BK * 2 + OSDP_MAX_SHARDS * 8) <= 160 * 1024) ? 2 : 1;
}

template <int BM, int BN, int WM, int WN, int BK, int kStages, bool kAK, bool kBK, int kEpi, bool kAccIn>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64, dma_groups_per_cu(BM, BN, BK, kStages) * (BM / WM) * (BN / WN) / 4)
void gemm_dma_kernel(GemmParams p, int tiles_m, int tiles_n) {
  constexpr int kWaves = (BM / WM) * (BN / WN);
  constexpr int MB = WM / 16, NB = WN / 16, NH = NB / 2;  // 16 x 16 blocks of the wave tile; B blocks per half
  constexpr int KS = BK / 32;                              // K steps per block
  constexpr int U = 2 * KS;                                // micro-steps per block: (K step, half of the B blocks)
  static_assert(NB % 2 == 0, "the wave tile is split in two column halves");
  using OpA = DmaOperand<kAK, BM, BK, kWaves>;
  using OpB = DmaOperand<kBK, BN, BK, kWaves>;
  constexpr int kStageElems = OpA::kElems + OpB::kElems;
  static_assert(kStages >= 2 && kStages <= 4, "2 to 4 LDS stages");
  extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];
  __shared__ uint16_t *s_tab[OSDP_MAX_SHARDS];

  const int tid = threadIdx.x;
  if (kEpi == static_cast<int>(Epilogue::kBf16ShardMajor)) {
    if (tid < OSDP_MAX_SHARDS) s_tab[tid] = static_cast<uint16_t *>(p.shards.p[tid]);
  }
  // A launch split along K: the logical ids of one part are consecutive, each part runs its own range of k and
  // stores its own fp32 plane (the planes lie one below the other: ldc = N).
  int tm, tn;
  int pid = logical_block();
  int K = p.K, plane_row = 0;
  int64_t k0 = 0;
  if (p.k_parts > 1) {
    const int tiles = tiles_m * tiles_n, part = __builtin_amdgcn_readfirstlane(pid / tiles);
    pid -= part * tiles;
    K = __builtin_amdgcn_readfirstlane(p.K / p.k_parts);
    k0 = static_cast<int64_t>(part) * K;
    plane_row = part * p.M;
  }
  tile_of_pid(pid, tiles_m, tiles_n, &tm, &tn);
  const int m0 = tm * BM;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave / (BN / WN)) * WM, wn = (wave % (BN / WN)) * WN;
  const int l16 = lane & 15, q4 = lane >> 4;

  TileSource<OpA, OpB, kAK, kBK, BM, BN, BK> src;
  src.begin(p, m0, tn, k0, K, wave, lane);
  const int nk = src.nb, n0 = src.n0, n_end = src.n_end;

  f32x4 acc[MB][NB];
  if constexpr (!kAccIn) {
#pragma unroll
    for (int bm = 0; bm < MB; ++bm)
#pragma unroll
      for (int bn = 0; bn < NB; ++bn)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[bm][bn][i] = 0.f;
  }

  // ---- global -> LDS: the LA + LB wave-level loads of one K block, issued in shares ------------------
  constexpr int LA = OpA::kLoads, LB = OpB::kLoads, L = LA + LB;
  static_assert((kStages - 1) * L < 64, "in-flight loads must fit the vmcnt counter");
  // The workgroup barrier of block it sits after the MFMAs of its micro-step U-2 and block it+1 must have
  // landed there.  With two stages the loads of block it+1 can only start once the barrier of block it-1 has
  // freed their stage, so they are spread over the micro-steps before the barrier; with more stages the loads
  // of block it+kStages-1 are spread over all micro-steps.
  constexpr int kIssueSteps = (kStages == 2 && U > 1) ? U - 1 : U;
  const uint32_t lds_base = lds_address(smem);
  // loads [first, last) of the block that the sources stand at, into `stage`; first / last are compile-time
  auto issue_range = [&](int stage, int first, int last) {
    const uint32_t sa = lds_base + stage * (kStageElems * 2);
    const uint32_t sb = sa + OpA::kElems * 2;
    static_for<L>([&](auto idx) {
      constexpr int i = decltype(idx)::value;
      if (i < first || i >= last) return;
      if constexpr (i < LA) src.a.template load<i>(sa + OpA::first_chunk(wave) * 1024);
      else src.b.template load<i - LA>(sb + OpB::first_chunk(wave) * 1024);
    });
    if (last == L) src.next(p, K, wave, lane);  // block fully issued
  };

  // Prologue: K blocks 0 .. kStages-2 are put in flight, block 0 is awaited.
  // (Every block runs the same code: loads of blocks beyond the last one are issued too, and deliver zeros nobody uses.)
#pragma unroll
  for (int s = 0; s < kStages - 1; ++s) issue_range(s, 0, L);
  // The sum to go on from is asked for behind them, so that both are under way together.  (Loads return in order, so the
  // wait below also covers part of these; the compiler waits for the rest where the first MFMA reads them.)
  if constexpr (kAccIn) load_acc_tile<MB, NB>(p, acc, m0 + wm, n0 + wn, n_end, l16, q4);
  wait_vmcnt<(kStages - 2) * L>();
  __builtin_amdgcn_s_barrier();

  // Fragments in registers: the A blocks of two K steps (alternating), the B blocks of two micro-steps.
  bf16x8 fa[2][MB], fb[2][NH];
  auto read_a = [&](int stage, int kk, auto buf) {
    const uint16_t *cA = smem + stage * kStageElems;
#pragma unroll
    for (int bm = 0; bm < MB; ++bm) fa[decltype(buf)::value][bm] = OpA::frag(cA, wm + bm * 16, kk, lane);
  };
  auto read_b = [&](int stage, int kk, int half, auto buf) {
    const uint16_t *cB = smem + stage * kStageElems + OpA::kElems;
#pragma unroll
    for (int bn = 0; bn < NH; ++bn) fb[decltype(buf)::value][bn] = OpB::frag(cB, wn + (half * NH + bn) * 16, kk, lane);
  };
  auto mfmas = [&](auto abuf, auto bbuf, auto half) {
#pragma unroll
    for (int bn = 0; bn < NH; ++bn)
#pragma unroll
      for (int bm = 0; bm < MB; ++bm)
        acc[bm][decltype(half)::value * NH + bn] =
            mma_16x16x32(fa[decltype(abuf)::value][bm], fb[decltype(bbuf)::value][bn], acc[bm][decltype(half)::value * NH + bn]);
  };

  // Steady state, one K block `it` (stage cur) = U micro-steps.  In micro-step u = (K step kk, column half h):
  //   - the fragments of micro-step u+1 are read from LDS (the other half of the B blocks; the A blocks too when
  //     it starts a new K step) while the MB * NH MFMAs of micro-step u run;
  //   - a share of the loads of block it+kStages-1 goes out (stage nxt, freed by the previous barrier);
  //   - after the MFMAs of micro-step U-2 every fragment read of block it has been issued: block it+1 is awaited
  //     and the workgroup barrier taken there, so that the last micro-step's MFMAs cover the first fragment
  //     reads of block it+1.
  // `par` is the parity of the block's first K step: A fragments of K step kk sit in fa[(par + kk) & 1].
  // load_: whether loads go out (see the loop below).
  int cur = 0, nxt = kStages - 1;
  auto block = [&](auto par, auto load_) {
    constexpr int P = decltype(par)::value;
    constexpr bool kLoad = decltype(load_)::value != 0;
    const int next_stage = (cur + 1 == kStages) ? 0 : cur + 1;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kk = u >> 1, h = u & 1;
      // fragments of micro-step u+1 (its B half goes to fb[(u+1) & 1]; U is even, so the first micro-step of a
      // block always uses fb[0])
      if (u + 1 < U) {
        const int kk2 = (u + 1) >> 1, h2 = (u + 1) & 1;
        if (h2 == 0) {
          if (((P + kk2) & 1) == 0) read_a(cur, kk2, Int<0>{}); else read_a(cur, kk2, Int<1>{});
        }
        if (((u + 1) & 1) == 0) read_b(cur, kk2, h2, Int<0>{}); else read_b(cur, kk2, h2, Int<1>{});
      } else {
        if (((P + KS) & 1) == 0) read_a(next_stage, 0, Int<0>{}); else read_a(next_stage, 0, Int<1>{});
        read_b(next_stage, 0, 0, Int<0>{});
      }
      if (kLoad && u < kIssueSteps) issue_range(nxt, u * L / kIssueSteps, (u + 1) * L / kIssueSteps);
      __builtin_amdgcn_sched_barrier(0);
      if (((P + kk) & 1) == 0) {
        if (h == 0) mfmas(Int<0>{}, Int<0>{}, Int<0>{}); else mfmas(Int<0>{}, Int<1>{}, Int<1>{});
      } else {
        if (h == 0) mfmas(Int<1>{}, Int<0>{}, Int<0>{}); else mfmas(Int<1>{}, Int<1>{}, Int<1>{});
      }
      __builtin_amdgcn_sched_barrier(0);
      if (u == U - 2) {
        // loads issued after the last load of block it+1: the full blocks it+2 .. it+kStages-2 and the
        // shares of block it+kStages-1 issued so far in this block
        constexpr int kYounger = (kStages >= 3) ? (kStages - 3) * L + (U - 1) * L / kIssueSteps : 0;
        wait_vmcnt<kLoad ? kYounger : 0>();
        __builtin_amdgcn_s_waitcnt((15) | (7 << 4) | (0 << 8) | (3 << 14));  // lgkmcnt(0): this wave's LDS reads are done
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    cur = next_stage;
    nxt = (nxt + 1 == kStages) ? 0 : nxt + 1;
  };

  read_a(0, 0, Int<0>{});
  read_b(0, 0, 0, Int<0>{});
  // Launches that go on from a sum are short (a slice's worth of k) and many: blocks beyond the last one, which elsewhere are
  // asked for and deliver zeros, would be half as much as what counts, so these end with blocks that load nothing (the
  // backward of 8192 -> 2048 over 768 tokens in 16 slices: 204 us, with this and the sum asked for behind the first
  // blocks 198; 640 tokens 4096 -> 2048 128 and 125).  Over a long reduction the second loop costs what it saves.
  constexpr bool kShort = kAccIn && KS % 2 == 0;
  if constexpr (kShort) {
    const int ahead = nk - (kStages - 1);
    int it = 0;
    for (; it < ahead; ++it) block(Int<0>{}, Int<1>{});
    for (; it < nk; ++it) block(Int<0>{}, Int<0>{});
  } else if constexpr (KS % 2 == 0) {
    for (int it = 0; it < nk; ++it) block(Int<0>{}, Int<1>{});
  } else {  // an odd number of K steps per block: the A fragment buffers swap roles from block to block
    for (int it = 0; it < nk; it += 2) {
      block(Int<0>{}, Int<1>{});
      if (it + 1 < nk) block(Int<1>{}, Int<1>{});
    }
  }
  wait_vmcnt<0>();  // surplus loads must have landed before the workgroup gives its LDS back

  store_tile<MB, NB, kEpi>(p, [&](auto bm, auto bn) { return acc[decltype(bm)::value][decltype(bn)::value]; }, m0 + wm, n0 + wn,
                           n_end, plane_row, l16, q4, s_tab);
}

}  // namespace
}  // namespace osdp
