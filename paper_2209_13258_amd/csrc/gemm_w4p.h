// The four-wave 256 x 256 GEMM kernel of gemm_w4.h as a persistent kernel: one workgroup per CU walks through the
// tiles t = w, w + G, w + 2G, ... (G workgroups) and treats their K blocks as one stream.
//
// Why: with one workgroup per CU nothing overlaps a tile's start-up and wind-down with another tile's MFMAs.  A
// tile of the plain kernel pays about 10 us beyond its K loop (the workgroup's launch, the latency of its first two
// K blocks, the drain of its stores): 17 % of a tile with K = 2048, 9 % with K = 4096.  Here the loads run two K
// blocks ahead of the MFMAs across tile boundaries, so the first blocks of the next tile are in LDS before the last
// MFMA of the current one; between the two tiles stand only the stores of the finished tile and the reset of the
// accumulators.  (The stores of tile t are older than the loads of block 2 of tile t+1 in the wave's memory
// counter, which counts loads and stores together and in order: the wait for that block also waits for their
// acknowledgement.)
//
// Same tiles in the same order per XCD, same MFMA sequence per output element as every other GEMM kernel of the
// library: same bits.  Takes what the plain kernel takes except a carried gather: any M, N and K (n_split a multiple of the
// tile's columns, k_split % 64 == 0; per part, when the launch runs parts of the reduction).
#pragma once
#include "gemm_w4.h"

namespace osdp {
namespace {

// Starting a tile's accumulators inside the loop over tiles.  To the compiler an assignment (acc = 0, acc = loaded
// values) would be a new value that has to be merged with the one the K loop carries, and it merges 256 pinned
// registers through scratch memory.  So the reset is itself a matrix-core step on the same registers, c = 0 * 0 + 0,
// written like the K loop's own steps as an update in place ...
__device__ __forceinline__ void acc_clear(f32x4 &c, bf16x8 zero) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %1, 0" : "+a"(c) : "v"(zero));
}
// ... and initial values come from memory straight into the accumulator registers; the caller waits (vmcnt) before
// the first MFMA.
__device__ __forceinline__ void acc_load(f32x4 &c, const float *src) {
  asm volatile("global_load_dwordx4 %0, %1, off" : "+a"(c) : "v"(src) : "memory");
}

template <int MB, int NB, bool kAK, bool kBKc, int kEpi, bool kAccIn>
__device__ __forceinline__ void gemm_w4p_tiles(const GemmParams &p, int tiles_m, int tiles_n) {
  constexpr int WM = 16 * MB, WN = 16 * NB, BM = 2 * WM, BN = 2 * WN;
  using OpA = W4Operand<kAK, MB>;
  using OpB = W4Operand<kBKc, NB>;
  constexpr int kSlotElems = OpA::kElems + OpB::kElems;  // 64 KB
  constexpr int L = OpA::kLoads + OpB::kLoads;           // wave-level loads per wave and block (16 for 256 x 256)
  static_assert(w4_all_placed(MB, NB, L), "a K step must hold the next one's fragment reads and a block's loads");
  extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];
  uint16_t *const *s_tab = nullptr;
  if constexpr (kEpi == static_cast<int>(Epilogue::kBf16ShardMajor)) {
    __shared__ uint16_t *tab[OSDP_MAX_SHARDS];
    if (threadIdx.x < OSDP_MAX_SHARDS) tab[threadIdx.x] = static_cast<uint16_t *>(p.shards.p[threadIdx.x]);
    s_tab = tab;  // read after the prologue's barrier
  }
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave >> 1) * WM, wn = (wave & 1) * WN;
  const int l16 = lane & 15, q4 = lane >> 4;
  // A launch split along K: the tiles of part 0 come first, then those of part 1, ...; each part runs its own range
  // of k and stores its own fp32 plane (the planes lie one below the other in C).
  const int parts = p.k_parts > 1 ? p.k_parts : 1;
  const int part_tiles = tiles_m * tiles_n, tiles = part_tiles * parts, G = gridDim.x;
  const int first = logical_block();  // < tiles: the host launches at most one workgroup per tile
  const int part_k = __builtin_amdgcn_readfirstlane(p.K / parts);
  const int nb = (part_k + 63) / 64;
  const int my_tiles = __builtin_amdgcn_readfirstlane((tiles - first + G - 1) / G);

  // ---- the load side: tile `lt` and the sources of its next block ------------------------------------------
  int lt = first;
  TileSource<OpA, OpB, kAK, kBKc, BM, BN, 64> src;
  auto load_tile = [&](int t) {  // point the sources at block 0 of tile t
    int tm, tn;
    const int part = __builtin_amdgcn_readfirstlane(t / part_tiles);
    tile_of_pid(t - part * part_tiles, tiles_m, tiles_n, &tm, &tn);
    src.begin(p, tm * BM, tn, static_cast<int64_t>(part) * part_k, part_k, wave, lane);
  };
  auto block_issued = [&]() {  // after the last load of a block: on to the next block, of this tile or the next
    if (src.block + 1 == nb && lt + G < tiles) {
      lt += G;
      load_tile(lt);
    } else {
      src.next(p, part_k, wave, lane);
    }
  };

  const uint32_t lds_base = lds_address(smem);
  const uint32_t dstA = lds_base + OpA::first_chunk(wave) * 1024;
  const uint32_t dstB = lds_base + OpA::kElems * 2 + OpB::first_chunk(wave) * 1024;
  auto issue = [&](int slot, auto idx) {
    constexpr int i = decltype(idx)::value;
    if constexpr (i < OpA::kLoads) src.a.template load<i>(dstA + slot * (kSlotElems * 2));
    else src.b.template load<i - OpA::kLoads>(dstB + slot * (kSlotElems * 2));
  };

  // ---- the compute side: tile `ct`, its origin, its accumulators --------------------------------------------
  int ct = first, cb = 0, m0c = 0, n0c = 0, n_endc = 0, plane_row = 0;
  f32x4 acc[MB][NB];
#pragma unroll
  for (int bm = 0; bm < MB; ++bm)
#pragma unroll
    for (int bn = 0; bn < NB; ++bn)
      asm volatile("" : "=a"(acc[bm][bn]));  // (a value to the compiler, no instruction: begin_tile sets the registers)
  bf16x8 zero;
#pragma unroll
  for (int i = 0; i < 8; ++i) zero[i] = static_cast<__bf16>(0.0f);
  // Written once, here: an MFMA may not read a register in the two cycles after a VALU instruction wrote it, and the
  // compiler, which does not see the MFMAs inside the asm statements, would otherwise write these zeros anew right
  // in front of each use.
  asm volatile("s_nop 1" : "+v"(zero));
  auto begin_tile = [&](int t, int l16e, int q4e) {
    int tm, tn;
    const int part = __builtin_amdgcn_readfirstlane(t / part_tiles);
    tile_of_pid(t - part * part_tiles, tiles_m, tiles_n, &tm, &tn);
    m0c = tm * BM;
    tile_columns<kBKc>(p, tn, BN, &n0c, &n_endc);
    plane_row = part * p.M;  // (the part's plane starts at this row of C)
    static_for<MB * NB>([&](auto idx) {
      constexpr int i = decltype(idx)::value, bn = i / MB, bm = i % MB;  // the order of the K loop's steps
      if constexpr (kAccIn) {
        const int m = m0c + wm + bm * 16 + l16e, n = n0c + wn + bn * 16 + 4 * q4e;
        const float *src = p.acc_in + static_cast<int64_t>(m < p.M ? m : p.M - 1) * p.ld_acc + (n < n_endc ? n : n_endc - 4);
        acc_load(acc[bm][bn], src);
      } else {
        acc_clear(acc[bm][bn], zero);
      }
    });
    if constexpr (kAccIn) wait_vmcnt<0>();
  };

  // prologue: blocks 0 and 1 of the first tile go in flight; block 0 is awaited and its first fragments read
  load_tile(lt);
  static_for<L>([&](auto i) { issue(0, i); });
  block_issued();
  static_for<L>([&](auto i) { issue(1, i); });
  block_issued();
  begin_tile(ct, l16, q4);
  wait_vmcnt<L>();
  __builtin_amdgcn_s_barrier();
  bf16x8 fa[2][MB], fb[2][NB];
  {
    const uint16_t *sA = smem, *sB = smem + OpA::kElems;
#pragma unroll
    for (int b = 0; b < MB; ++b) fa[0][b] = OpA::frag(sA, wm + b * 16, 0, lane);
#pragma unroll
    for (int b = 0; b < NB; ++b) fb[0][b] = OpB::frag(sB, wn + b * 16, 0, lane);
  }

  // 64 MFMAs of one K step out of fragment set P; between them the 16 fragment reads of the next K step (slot rs,
  // K step rk) into the other set and, when kLoad, the 16 loads of the block two ahead into slot ls.
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
      if constexpr (kLoad && w4_load_behind(i, MB * NB, L) >= 0) {
        issue(ls, Int<w4_load_behind(i, MB * NB, L)>{});
        if constexpr (w4_load_behind(i, MB * NB, L) == L - 1) block_issued();
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // One loop over all K blocks of all tiles of this workgroup; every block runs the same code.  Loads beyond the
  // last block of the last tile are issued with every lane out of range, and the fragments read ahead at the very end
  // are nobody's.
  int cur = 0;
  const int total = my_tiles * nb;
  for (int g = 0; g < total; ++g) {
    const uint16_t *sc = smem + cur * kSlotElems, *sn = smem + (cur ^ 1) * kSlotElems;
    kstep(Int<0>{}, Int<0>{}, sc, 1, 0);
    // this block is now fully in registers or consumed, and the next one must be in LDS
    wait_vmcnt<0>();
    __builtin_amdgcn_s_waitcnt((15) | (7 << 4) | (0 << 8) | (3 << 14));  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    kstep(Int<1>{}, Int<1>{}, sn, 0, cur);
    cur ^= 1;
    if (++cb == nb) {  // the tile is complete: store it and start the next (its first blocks are in LDS or on their way)
      cb = 0;
      asm volatile("s_nop 15");
      asm volatile("s_nop 15");
      // The lane's coordinates pass through an empty asm so that every address of the epilogue is computed here:
      // computed ahead of the loop they would sit in registers that the K loop has no room for.
      int l16e = l16, q4e = q4;
      asm volatile("" : "+v"(l16e), "+v"(q4e));
      // (a block or two at a time, a scheduling fence after each: read all at once, the 256 values would push the K
      // loop's fragments out of their registers)
      store_tile<MB, NB, kEpi>(p, [&](auto bm, auto bn) { return acc_value<kEpi>(acc[decltype(bm)::value][decltype(bn)::value]); },
                               m0c + wm, n0c + wn, n_endc, plane_row, l16e, q4e, s_tab);
      ct += G;
      if (ct < tiles) begin_tile(ct, l16e, q4e);
      // The fragments read ahead for the next K step are read again here, so that none of them has to outlive the
      // epilogue: it needs their registers.
      {
        const uint16_t *sA = smem + cur * kSlotElems, *sB = sA + OpA::kElems;
#pragma unroll
        for (int b = 0; b < MB; ++b) fa[0][b] = OpA::frag(sA, wm + b * 16, 0, lane);
#pragma unroll
        for (int b = 0; b < NB; ++b) fb[0][b] = OpB::frag(sB, wn + b * 16, 0, lane);
      }
    }
  }
  wait_vmcnt<0>();  // surplus loads must have landed before the workgroup gives its LDS back
}

template <bool kAK, bool kBKc, int kEpi, bool kAccIn>
__global__ __launch_bounds__(256, 1)
void gemm_w4p_kernel(GemmParams p, int tiles_m, int tiles_n) {
  gemm_w4p_tiles<8, 8, kAK, kBKc, kEpi, kAccIn>(p, tiles_m, tiles_n);
}

// Tiles of fewer than 256 rows or columns: 32 * MB x 32 * NB.
template <int MB, int NB, bool kAK, bool kBKc, int kEpi, bool kAccIn>
__global__ __launch_bounds__(256, 1)
void gemm_w4p_small_kernel(GemmParams p, int tiles_m, int tiles_n) {
  gemm_w4p_tiles<MB, NB, kAK, kBKc, kEpi, kAccIn>(p, tiles_m, tiles_n);
}

}  // namespace
}  // namespace osdp
