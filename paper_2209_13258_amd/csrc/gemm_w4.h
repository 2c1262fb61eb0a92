// Large-tile GEMM kernel of libosdp: a 256 x 256 output tile per workgroup of four waves, one wave per SIMD,
// each wave owning a 128 x 128 quarter whose 256 fp32 accumulator registers fill the AGPR half of the
// register file.  Against the eight-wave kernel (waves of 64 x 128) every byte read from LDS feeds a third
// more MFMAs (16 fragment reads per 64 MFMAs instead of 12 per 32).
//
// With one wave per SIMD nothing hides a wave's own stalls, so the K loop is one interleaved instruction
// stream: the 64 MFMAs of a K step of 32 carry, in their shadow, the fragment reads of the next K step and the
// global -> LDS loads of a K block further ahead.  LDS holds two K blocks of 64 (64 KB each: A 256 x 64, then
// B 256 x 64).  A wave-level load of a K-contiguous operand covers 128 contiguous bytes of each of 8 rows, whole
// cache lines: with K blocks of 32 the same bytes take twice the requests (64 bytes of each of 16 rows), and the
// stream from L2 into LDS, which on this chip takes about as long as the MFMAs themselves, slows down by 15 %
// (measured on 8192^3, everything else equal).  One workgroup barrier per K block, at the start of its second K
// step: there every wave holds that step's fragments in registers, so block b's slot is free for the loads of
// block b+2, and the loads of block b+1, issued during the previous block's second step, must have landed.
//
// Same MFMA sequence per output element as every other GEMM kernel of the library (K ascending in steps of 32,
// v_mfma_f32_16x16x32_bf16, the same lane -> k map), so the result bits are the same.
//
// Tiles of 32 * MB x 32 * NB, the large one (8 x 8) wherever its rounds are full.  Any M, N and K
// (k_split % 64 == 0, n_split a multiple of the tile's columns): edges are handled by the range check of the operand
// loads, which also lets blocks beyond the last one deliver nothing, and guarded stores (OperandSource in gemm_dma.h).
#pragma once
#include "gemm_common.h"
#include "gemm_dma.h"

namespace osdp {
namespace {

// The matrix-core step with its accumulator pinned to AGPRs and updated in place.  Written as inline assembly
// because the compiler, left to place 256 accumulator registers itself, keeps moving them between the two halves of
// the register file inside the K loop.  It then no longer sees an MFMA here, so the two hazards it would have
// covered are covered by hand in the kernel: VALU writes of the accumulators before the first step, and VALU reads
// after the last.  For the same reason the K loop below exists once, for every K block alike (no separate code for
// the last blocks): where two copies of it meet, the compiler copies accumulators from the registers one copy chose
// to those the other chose, with VALU moves it does not know to keep clear of the MFMAs.
__device__ __forceinline__ void mma_16x16x32_agpr(f32x4 &c, bf16x8 a_rows, bf16x8 b_cols) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(b_cols), "v"(a_rows));
}

// The four values of an accumulator block, read where this stands and nowhere else: read by the compiler's own
// copies they may move to the head of the epilogue, all 256 at once, into registers the K loop's fragments hold.
__device__ __forceinline__ f32x4 acc_read(const f32x4 &c) {
  float x0, x1, x2, x3;
  asm volatile("v_accvgpr_read_b32 %0, %4\n\tv_accvgpr_read_b32 %1, %5\n\tv_accvgpr_read_b32 %2, %6\n\tv_accvgpr_read_b32 %3, %7"
               : "=v"(x0), "=v"(x1), "=v"(x2), "=v"(x3) : "a"(c[0]), "a"(c[1]), "a"(c[2]), "a"(c[3]));
  return f32x4{x0, x1, x2, x3};
}

// What an epilogue takes of it: fp32 results are stored straight from the accumulators.
template <int kEpi>
__device__ __forceinline__ f32x4 acc_value(const f32x4 &c) {
  return kEpi == static_cast<int>(Epilogue::kF32Workspace) ? c : acc_read(c);
}

// One operand's share of a ring slot: 32 * kBlocks rows (or columns) x 64 k, filled by wave-level direct-to-LDS loads of
// 1 KB.  kBlocks: 16-row blocks of a wave tile, of a tile of 32 * kBlocks rows.  A K-contiguous operand takes as many rows as
// the tile has; the other kind, whose swizzle works on runs of 128, takes 128 or 256 columns, and the lanes of those beyond
// the tile are out of range.
template <bool kKC, int kBlocks>
struct W4Operand {
  static constexpr int kRows = kKC ? 32 * kBlocks : (kBlocks > 4 ? 256 : 128), kBK = 64, kWaves = 4;
  static constexpr int kElems = kRows * kBK;         // 32 KB for 256 rows
  static constexpr int kLoads = kElems / 2048;       // per wave and block
  using Base = DmaOperand<kKC, kKC ? 256 : kRows, kBK, kWaves>;
  static constexpr int kPerChunk = 512 / (kKC ? kBK : kRows);  // rows, or k-rows, that 1 KB holds
  // 1 KB chunk that load p of wave w fills.  K-contiguous: chunk c = rows 8c .. 8c+7.  MN-contiguous: chunk c = k-rows
  // 2c, 2c+1 (256 columns), with (c & 1) and ((c >> 2) & 1) fixed over a wave's loads (the source swizzle depends on them),
  // or k-rows 4c .. 4c+3 (128 columns), with (c >> 1) & 1 fixed.
  static __device__ __forceinline__ constexpr int chunk(int w, int p) {
    return kKC || kRows == 128 ? p * 4 + w : (w & 1) + 2 * (p & 1) + 4 * (w >> 1) + 8 * (p >> 1);
  }
  static __device__ __forceinline__ int64_t lane_src(int w, int lane, int64_t ld) {
    if (kKC) {
      const int row = chunk(w, 0) * kPerChunk + lane / Base::CPR;
      const int c = (lane % Base::CPR) ^ Base::swz_k(row);
      return static_cast<int64_t>(row) * ld + c * 8;
    } else {
      constexpr int kVecs = kRows / 8;
      const int krow = chunk(w, 0) * kPerChunk + lane / kVecs;
      return static_cast<int64_t>(krow) * ld + (((lane % kVecs) * 8) ^ Base::swz_mn(krow));
    }
  }
  static __device__ __forceinline__ int lane_pos(int w, int lane) {  // k (K-contiguous) or mn of those 16 bytes
    if (kKC) return ((lane % Base::CPR) ^ Base::swz_k(chunk(w, 0) * kPerChunk + lane / Base::CPR)) * 8;
    constexpr int kVecs = kRows / 8;
    return ((lane % kVecs) * 8) ^ Base::swz_mn(chunk(w, 0) * kPerChunk + lane / kVecs);
  }
  static __device__ __forceinline__ constexpr int first_chunk(int w) { return chunk(w, 0); }
  static __device__ __forceinline__ constexpr int chunk_step(int p) { return chunk(0, p) - chunk(0, 0); }
  static __device__ __forceinline__ constexpr int load_rows(int p) { return chunk_step(p) * kPerChunk; }
  static __device__ __forceinline__ bf16x8 frag(const uint16_t *slot, int mn0, int kk, int lane) { return Base::frag(slot, mn0, kk, lane); }
};

// Fragment read r of the MB + NB of a K step goes out behind MFMA r * w4_read_step, B's block 0 first, then all of A's, then
// the rest of B's: the order in which the next step's MFMAs ask for them.
constexpr int w4_read_step(int MB, int NB) { return 3 * (MB + NB) <= MB * NB + 1 ? 3 : (2 * (MB + NB) <= MB * NB - 4 ? 2 : 1); }
constexpr int w4_read_behind(int i, int MB, int NB) {
  const int step = w4_read_step(MB, NB), first = step > 1 ? 1 : 0;
  return i % step == first % step && i / step < MB + NB ? i / step : -1;
}

// Load l of the L per block goes out behind MFMA (l * N) / L + 2 of the N in a K step (or + 1 or 0, so that the last one has a
// place too); l, or -1, for a given MFMA.
constexpr int w4_load_behind(int i, int N, int L) {
  const int room = N - 1 - (L - 1) * N / L, late = room < 2 ? room : 2;
  for (int l = 0; l < L; ++l)
    if (l * N / L + late == i) return l;
  return -1;
}
// Every read and every load has its place.
constexpr bool w4_all_placed(int MB, int NB, int L) {
  int reads = 0, loads = 0;
  for (int i = 0; i < MB * NB; ++i) {
    reads += w4_read_behind(i, MB, NB) >= 0;
    loads += w4_load_behind(i, MB * NB, L) >= 0;
  }
  return reads == MB + NB && loads == L;
}

// kCopy: the launch also carries p.job, the gather of a slice that a later launch will read (the forward GEMM of
// slice j gathers slice j+1 into the other staging slot; a dW launch, which needs no weights, gathers the slices of
// the dX pass that follows it).  Every workgroup copies total_vecs / gridDim.x vectors, 256 per K block: one 16-byte
// load and one 16-byte store per lane and block, against that block's 16 KB of operand loads per wave; what the K blocks
// do not hold follows behind them, several pieces at a time.  A gather kernel of its own
// cannot run beside this kernel, whose four waves hold every register of their SIMDs: on a second stream it only takes
// turns with the tiles, and both get slower.  The carried copy is not free either (the kernel is bound by the memory pipe
// the copy shares: a 64 MiB slice adds 25 us to a 190 us launch, against 28 us as a launch of its own); it saves the
// launch, its gap and every cross-stream event.
template <int MB, int NB, int kSlots, bool kAK, bool kBKc, int kEpi, bool kAccIn, bool kCopy>
__device__ __forceinline__ void gemm_w4_tile(const GemmParams &p, int tiles_m, int tiles_n, int pid) {
  constexpr int WM = 16 * MB, WN = 16 * NB, BM = 2 * WM, BN = 2 * WN;
  using OpA = W4Operand<kAK, MB>;
  using OpB = W4Operand<kBKc, NB>;
  // The loads of block b + kAhead go out in block b's second step.  With two slots they fill the slot that every wave has
  // just read the last fragments of; with more, the one before it, and nobody waits for those reads.
  constexpr int kAhead = kSlots == 2 ? 2 : kSlots - 1;
  constexpr int kSlotElems = OpA::kElems + OpB::kElems;  // 64 KB
  constexpr int L = OpA::kLoads + OpB::kLoads;           // wave-level loads per wave and block (16 for 256 x 256)
  static_assert(w4_all_placed(MB, NB, L), "a K step must hold the next one's fragment reads and a block's loads");
  extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];
  uint16_t *const *s_tab = nullptr;
  if constexpr (kEpi == static_cast<int>(Epilogue::kBf16ShardMajor)) {
    __shared__ uint16_t *tab[OSDP_MAX_SHARDS];
    if (threadIdx.x < OSDP_MAX_SHARDS) tab[threadIdx.x] = static_cast<uint16_t *>(p.shards.p[threadIdx.x]);
    s_tab = tab;
  }
  const int tid = threadIdx.x;
  // ---- the carried gather: this workgroup's range of vectors, piece i = vectors first + 256 i + tid ----------
  // Lanes beyond the range's end inside its last piece copy the range's last vector again (the same bytes to the
  // same place); K blocks beyond the last piece issue nothing for the copy (one uniform test per hook), which is what
  // keeps a small slice cheap to carry through a long reduction.
  uint64_t copy_first = 0, copy_last = 0;
  uint32_t copy_pieces = 0;
  const uint16_t *const *g_tab = nullptr;
  if constexpr (kCopy) {
    __shared__ const uint16_t *gtab[OSDP_MAX_SHARDS];
    if (tid < OSDP_MAX_SHARDS) gtab[tid] = static_cast<const uint16_t *>(p.job.src.p[tid]);
    g_tab = gtab;  // read after the prologue's barrier
    const uint64_t per_wg = ((p.job.total_vecs + gridDim.x - 1) / gridDim.x + 255) & ~static_cast<uint64_t>(255);
    const uint64_t first = static_cast<uint64_t>(blockIdx.x) * per_wg;
    if (first < p.job.total_vecs) {
      const uint64_t end = first + per_wg < p.job.total_vecs ? first + per_wg : p.job.total_vecs;
      copy_first = first;
      copy_last = end - 1;
      copy_pieces = static_cast<uint32_t>((end - first + 255) / 256);
    }
  }
  // source address of this lane's vector of piece i
  auto copy_src = [&](uint32_t i, uint32_t *v_out) -> const uint4 * {
    uint64_t v = copy_first + static_cast<uint64_t>(i) * 256 + tid;
    v = v < copy_last ? v : copy_last;
    const uint32_t v32 = static_cast<uint32_t>(v);
    const uint32_t rd = v32 / p.job.vecs_per_row, cv = v32 - rd * p.job.vecs_per_row;
    const uint32_t r = p.job.r0 + rd;
    uint32_t s;
    uint64_t off;
    if (p.job.lay.rows_per_shard > 0) {
      s = r / static_cast<uint32_t>(p.job.lay.rows_per_shard);
      off = static_cast<uint64_t>(r - s * p.job.lay.rows_per_shard) * p.job.lay.O + p.job.c0 + cv * 8u;
    } else {
      const uint64_t f = static_cast<uint64_t>(r) * p.job.lay.O + p.job.c0 + cv * 8u;
      s = static_cast<uint32_t>(f / static_cast<uint64_t>(p.job.lay.L));
      off = f - static_cast<uint64_t>(s) * p.job.lay.L;
    }
    *v_out = v32;
    return reinterpret_cast<const uint4 *>(g_tab[s] + off);
  };
  uint4 copy_data = {0u, 0u, 0u, 0u};  // the piece in flight
  uint32_t copy_v = 0;                 // its destination vector
  uint32_t copy_i = 0;                 // its index
  const uint4 *copy_ptr = nullptr;     // source and destination vector of the piece after it
  uint32_t copy_next_v = 0;

  // A launch split along K: the logical ids of one part are consecutive (so an XCD's tiles still share panels),
  // each part runs its own range of k and stores its own fp32 plane.
  int tm, tn;
  int K = p.K;
  int64_t k0 = 0;    // first k of this workgroup's part
  int plane_row = 0;  // its plane starts at this row of C (the planes lie one below the other: ldc = N)
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
  const int wm = (wave >> 1) * WM, wn = (wave & 1) * WN;
  const int l16 = lane & 15, q4 = lane >> 4;

  TileSource<OpA, OpB, kAK, kBKc, BM, BN, 64> src;
  src.begin(p, m0, tn, k0, K, wave, lane);
  const int nb = src.nb, n0 = src.n0, n_end = src.n_end;

  f32x4 acc[MB][NB];
  if constexpr (!kAccIn) {
#pragma unroll
    for (int bm = 0; bm < MB; ++bm)
#pragma unroll
      for (int bn = 0; bn < NB; ++bn)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[bm][bn][i] = 0.f;
  }

  const uint32_t lds_base = lds_address(smem);
  const uint32_t dstA = lds_base + OpA::first_chunk(wave) * 1024;
  const uint32_t dstB = lds_base + OpA::kElems * 2 + OpB::first_chunk(wave) * 1024;

  // load i of the block that the sources stand at, into `slot`; after the last one they move on to the next block
  // (beyond the last block they deliver zeros that nobody uses)
  auto issue = [&](int slot, auto idx) {
    constexpr int i = decltype(idx)::value;
    if constexpr (i < OpA::kLoads) src.a.template load<i>(dstA + slot * (kSlotElems * 2));
    else src.b.template load<i - OpA::kLoads>(dstB + slot * (kSlotElems * 2));
    if constexpr (i == L - 1) src.next(p, K, wave, lane);
  };
  bf16x8 fa[2][MB], fb[2][NB];

  // prologue: the first blocks go in flight; block 0 is awaited and the fragments of its first K step read
  static_for<kAhead>([&](auto b) { static_for<L>([&](auto i) { issue(decltype(b)::value, i); }); });
  if constexpr (kAccIn) load_acc_tile<MB, NB>(p, acc, m0 + wm, n0 + wn, n_end, l16, q4);  // (the sum is asked for behind them)
  asm volatile("s_nop 7");  // accumulator writes (VALU) settle before the first MFMA reads them
  wait_vmcnt<(kAhead - 1) * L>();
  __builtin_amdgcn_s_barrier();
  if constexpr (kCopy) {  // piece 0 of the carried gather (the barrier has published the shard table)
    copy_ptr = copy_src(0, &copy_v);
    copy_data = load_global16(copy_ptr);
  }
  {
    const uint16_t *sA = smem, *sB = smem + OpA::kElems;
#pragma unroll
    for (int b = 0; b < MB; ++b) fa[0][b] = OpA::frag(sA, wm + b * 16, 0, lane);
#pragma unroll
    for (int b = 0; b < NB; ++b) fb[0][b] = OpB::frag(sB, wn + b * 16, 0, lane);
  }

  // 64 MFMAs of one K step out of fragment set P; in their shadow the 16 fragment reads of the next K step
  // (slot rs, K step rk) into the other set and, when kLoad, the 16 loads of the block two ahead into slot ls.
  auto kstep = [&](auto par, auto load_, const uint16_t *rs, int rk, int ls) {
    constexpr int P = decltype(par)::value, Q = P ^ 1;
    constexpr bool kLoad = decltype(load_)::value != 0;
    const uint16_t *nA = rs, *nB = rs + OpA::kElems;
    static_for<MB * NB>([&](auto idx) {
      constexpr int i = decltype(idx)::value, bn = i / MB, bm = i % MB;
      mma_16x16x32_agpr(acc[bm][bn], fa[P][bm], fb[P][bn]);
      if constexpr (w4_read_behind(i, MB, NB) >= 0) {
        constexpr int r = w4_read_behind(i, MB, NB);
        if constexpr (r == 0) fb[Q][0] = OpB::frag(nB, wn, rk, lane);
        else if constexpr (r <= MB) fa[Q][r - 1] = OpA::frag(nA, wm + (r - 1) * 16, rk, lane);
        else fb[Q][r - MB] = OpB::frag(nB, wn + (r - MB) * 16, rk, lane);
      }
      if constexpr (kLoad && w4_load_behind(i, MB * NB, L) >= 0) issue(ls, Int<w4_load_behind(i, MB * NB, L)>{});
      // carried gather: in the block's first K step the address of the next piece is worked out; in the second,
      // just behind the barrier where every load has landed, the piece in registers goes out and the next comes in
      // (all three behind one uniform test: once the range is copied the remaining K blocks issue nothing for it)
      if constexpr (kCopy && !kLoad && i == MB * NB * 5 / 8) {
        if (copy_i + 1 < copy_pieces) copy_ptr = copy_src(copy_i + 1, &copy_next_v);
      }
      if constexpr (kCopy && kLoad && i == 0) {
        if (copy_i < copy_pieces) store_global16(p.job.dst + copy_v, copy_data);
      }
      if constexpr (kCopy && kLoad && i == 1) {
        if (copy_i + 1 < copy_pieces) {
          copy_data = load_global16(copy_ptr);
          copy_v = copy_next_v;
        }
        ++copy_i;
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // Every block runs the same code: the last ones still issue their load instructions (with every lane out of
  // range) and the last still reads fragments nobody uses.
  int cur = 0, fill = kSlots == 2 ? 0 : kAhead;
  auto after = [](int slot) { return slot + 1 == kSlots ? 0 : slot + 1; };
  for (int b = 0; b < nb; ++b) {
    const uint16_t *sc = smem + cur * kSlotElems, *sn = smem + after(cur) * kSlotElems;
    // first K step; its shadow reads the second step's fragments of this block
    kstep(Int<0>{}, Int<0>{}, sc, 1, 0);
    // block b + 1 must be in LDS, and (two slots) block b fully in registers or consumed
    wait_vmcnt<(kAhead - 2) * L>();
    if constexpr (kSlots == 2) __builtin_amdgcn_s_waitcnt((15) | (7 << 4) | (0 << 8) | (3 << 14));  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    kstep(Int<1>{}, Int<1>{}, sn, 0, fill);
    cur = after(cur);
    fill = after(fill);
  }
  wait_vmcnt<0>();  // surplus loads must have landed before the workgroup gives its LDS back
  if constexpr (kCopy) {
    // The piece still in registers, and whatever the K loop was too short for.  Nothing else is under way here: eight pieces
    // share a round trip to memory (the fragments' registers are free).  Backward, us with one piece a round trip / eight / the
    // gathers as launches, weights from memory, 32 pieces: 4096 -> 16384, k = 8, over 640 tokens (10 K blocks) 355 / 314 / 318,
    // over 1100 (18) 418 / 399 / 395, over 1536 (24) 455 / 444 / 447; 4096 -> 4096, k = 2, over 640 77 / 67 / 69, and with the
    // weights in a cache 66 / 60 / 64.
    if (copy_i < copy_pieces) store_global16(p.job.dst + copy_v, copy_data);
    constexpr int kBatch = 8;
#pragma unroll 1
    for (uint32_t i = copy_i + 1; i < copy_pieces; i += kBatch) {
      uint4 data[kBatch];
      uint32_t v[kBatch];
#pragma unroll
      for (int e = 0; e < kBatch; ++e) {
        // (beyond the end the last piece again: the same bytes to the same place)
        const uint4 *src = copy_src(i + e < copy_pieces ? i + e : copy_pieces - 1, &v[e]);
        data[e] = load_global16(src);
      }
#pragma unroll
      for (int e = 0; e < kBatch; ++e) store_global16(p.job.dst + v[e], data[e]);
    }
  }

  asm volatile("s_nop 15");
  asm volatile("s_nop 15");
  store_tile<MB, NB, kEpi>(p, [&](auto bm, auto bn) { return acc_value<kEpi>(acc[decltype(bm)::value][decltype(bn)::value]); },
                           m0 + wm, n0 + wn, n_end, plane_row, l16, q4, s_tab);
}

template <bool kAK, bool kBKc, int kEpi, bool kAccIn, bool kCopy = false>
__global__ __launch_bounds__(256, 1)
void gemm_w4_kernel(GemmParams p, int tiles_m, int tiles_n) {
  gemm_w4_tile<8, 8, 2, kAK, kBKc, kEpi, kAccIn, kCopy>(p, tiles_m, tiles_n, logical_block());
}

// Tiles of fewer than 256 rows or columns: 32 * MB x 32 * NB.
template <int MB, int NB, bool kAK, bool kBKc, int kEpi, bool kAccIn, bool kCopy = false>
__global__ __launch_bounds__(256, 1)
void gemm_w4_small_kernel(GemmParams p, int tiles_m, int tiles_n) {
  gemm_w4_tile<MB, NB, 2, kAK, kBKc, kEpi, kAccIn, kCopy>(p, tiles_m, tiles_n, logical_block());
}

// Tiles of 160 columns for launches of at most one tile per CU (dX), with as many slots as fit.
template <int MB, int kSlots, bool kAK, bool kBKc, int kEpi, bool kAccIn>
__global__ __launch_bounds__(256, 1)
void gemm_w4_160_kernel(GemmParams p, int tiles_m, int tiles_n) {
  gemm_w4_tile<MB, 5, kSlots, kAK, kBKc, kEpi, kAccIn, false>(p, tiles_m, tiles_n, logical_block());
}

// Tiles of 128 x 128, two workgroups to a CU with two slots each, or one with four (launches of at most one tile per CU).
// Waves of 64 x 64.  Against eight waves of 32 x 64 (one workgroup to a CU) and a loop of micro-steps over half the B
// blocks (two) they read a third less out of LDS, or the same with fewer instructions.  What bounds them is the card's power
// (K = 8192, 512 tiles: 119 us on random data, 94 on zeros) and the bytes through LDS.  us before / now, forward, dW, dX:
// 2048 x 2048 over K = 8192 68.3 / 65.4, 73.1 / 72.1, 64.8 / 62.1; 2048 x 8192 over 4096 132 / 122, 135 / 132, 129 / 119; the
// prompt of 500 tokens 2560 -> 10240 35.8 / 33.8.  Tiles of 256 x 128 in waves of 128 x 64 lose to the eight-wave kernel's
// (4096 x 2048 over K = 4096: 62 against 57 us): with one wave to a SIMD and three slots nothing hides the barriers.
template <int kSlots, bool kAK, bool kBKc, int kEpi, bool kAccIn>
__global__ __launch_bounds__(256, kSlots == 2 ? 2 : 1)
void gemm_w4_128_kernel(GemmParams p, int tiles_m, int tiles_n) {
  gemm_w4_tile<4, 4, kSlots, kAK, kBKc, kEpi, kAccIn, false>(p, tiles_m, tiles_n, logical_block());
}

}  // namespace
}  // namespace osdp
