// Slice GEMMs of the operator-split linear layer (arXiv 2209.13258, Section 3.3):
//   forward   Y[:, slice]  = X . Ws          A K-contiguous, B N-contiguous
//   dW        dW[:, slice] = X^T . dY_slice  A M-contiguous, B N-contiguous
//   dX        dX (+)= dY_slice . Ws^T        A K-contiguous, B K-contiguous
// bf16 operands, fp32 accumulation on the gfx950 matrix cores
// (v_mfma_f32_16x16x32_bf16), bf16 round-to-nearest-even outputs.
//
// Every kernel in this file but the few-token one (gemm_skinny.h) feeds each output element the same sequence of
// MFMA operations: K is walked in ascending blocks of 32, and inside a block
// logical k = 8*q + e sits in lane group q, element e of both operands.  Tile
// shape therefore never changes a result bit, which is what makes Y and dW of
// a split operator bit-identical to the unsplit ones.
#include "gemm_common.h"
#include "gemm_dma.h"
#include "gemm_skinny.h"
#include "gemm_w4.h"
#include "gemm_w4p.h"

namespace osdp {

namespace {

// ---------------------------------------------------------------------------
// Generic kernel: 128 x 128 x 32 tile, 4 waves of 64 x 64, single LDS buffer,
// every access bounds-checked.  Handles any M, N and any K that is a multiple
// of 8 (the tail of the last K block is zero-filled, which adds exact zeros);
// K = 0 is the empty sum: it stores zeros (or acc_in) and reads neither operand.  It runs empty sums, leading
// dimensions beyond the other kernels' 32-bit offsets, and whatever the tests compare with the other kernels.
// ---------------------------------------------------------------------------
constexpr int GBM = 128, GBN = 128, GBK = 32, GLDK = GBK + 8;

template <bool kKContig>
__device__ __forceinline__ void generic_load(const uint16_t *__restrict__ src, int64_t ld, int rows_lim,
                                             int row0, int k0, int K, uint4 (&v)[2]) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int id = tid + p * 256;
    int gr, gk;
    if (kKContig) {
      gr = row0 + (id >> 2);
      gk = k0 + (id & 3) * 8;
    } else {
      gk = k0 + (id >> 4);
      gr = row0 + (id & 15) * 8;
    }
    uint4 z = {0u, 0u, 0u, 0u};
    if (gr < rows_lim && gk < K) {
      const int64_t off = kKContig ? static_cast<int64_t>(gr) * ld + gk : static_cast<int64_t>(gk) * ld + gr;
      z = *reinterpret_cast<const uint4 *>(src + off);
    }
    v[p] = z;
  }
}

template <bool kKContig>
__device__ __forceinline__ void generic_store_lds(uint16_t (*S)[GLDK], const uint4 (&v)[2]) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int id = tid + p * 256;
    if (kKContig) {
      *reinterpret_cast<uint4 *>(&S[id >> 2][(id & 3) * 8]) = v[p];
    } else {
      const int kr = id >> 4, r = (id & 15) * 8;
      const uint32_t w[4] = {v[p].x, v[p].y, v[p].z, v[p].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        S[r + 2 * e][kr] = static_cast<uint16_t>(w[e] & 0xffffu);
        S[r + 2 * e + 1][kr] = static_cast<uint16_t>(w[e] >> 16);
      }
    }
  }
}

template <bool kAK, bool kBK, int kEpi, bool kAccIn>
__global__ __launch_bounds__(256) void gemm_generic_kernel(GemmParams p) {
  __shared__ __attribute__((aligned(16))) uint16_t As[GBM][GLDK];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[GBN][GLDK];
  __shared__ uint16_t *s_tab[OSDP_MAX_SHARDS];

  const int tid = threadIdx.x;
  if (kEpi == static_cast<int>(Epilogue::kBf16ShardMajor)) {
    if (tid < OSDP_MAX_SHARDS) s_tab[tid] = static_cast<uint16_t *>(p.shards.p[tid]);
    __syncthreads();  // with K = 0 the loop below, and its barriers, do not run
  }
  const int tiles_m = (p.M + GBM - 1) / GBM;
  // a launch split along K: part s of the grid takes its range of k and stores plane s (the planes lie one below the other)
  const int tiles = tiles_m * ((p.N + GBN - 1) / GBN);
  const int part = p.k_parts > 1 ? blockIdx.x / tiles : 0;
  const int bid = blockIdx.x - part * tiles;
  const int k_len = p.k_parts > 1 ? p.K / p.k_parts : p.K;
  const int k_begin = part * k_len, k_end = k_begin + k_len;
  const int plane_row = part * p.M;
  const int tm = bid % tiles_m, tn = bid / tiles_m;
  const int m0 = tm * GBM, n0 = tn * GBN;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  const int l16 = lane & 15, q = lane >> 4;

  // acc[bm][bn][i] is C[m0 + wm + 16*bm + l16][n0 + wn + 16*bn + 4*q + i]
  f32x4 acc[4][4];
#pragma unroll
  for (int bm = 0; bm < 4; ++bm)
#pragma unroll
    for (int bn = 0; bn < 4; ++bn) {
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[bm][bn][i] = 0.f;
      if (kAccIn) {
        const int m = m0 + wm + bm * 16 + l16, n = n0 + wn + bn * 16 + 4 * q;
        if (m < p.M && n < p.N) {
          const float4 c = *reinterpret_cast<const float4 *>(p.acc_in + static_cast<int64_t>(m) * p.ld_acc + n);
          acc[bm][bn][0] = c.x;
          acc[bm][bn][1] = c.y;
          acc[bm][bn][2] = c.z;
          acc[bm][bn][3] = c.w;
        }
      }
    }

  for (int k0 = k_begin; k0 < k_end; k0 += GBK) {
    uint4 va[2], vb[2];
    generic_load<kAK>(p.A, p.lda, p.M, m0, k0, k_end, va);
    if (p.k_split && k0 >= p.k_split)       // B's second segment, by k or by column (both on tile and block boundaries)
      generic_load<kBK>(p.B2, p.ldb2, p.N, n0, k0 - p.k_split, k_end - p.k_split, vb);
    else if (p.n_split && n0 >= p.n_split)
      generic_load<kBK>(p.B2, p.ldb2, p.N - p.n_split, n0 - p.n_split, k0, k_end, vb);
    else
      generic_load<kBK>(p.B, p.ldb, p.n_split ? p.n_split : p.N, n0, k0, p.k_split ? p.k_split : k_end, vb);
    __syncthreads();  // the previous block's LDS reads are done
    generic_store_lds<kAK>(As, va);
    generic_store_lds<kBK>(Bs, vb);
    __syncthreads();
    // one K step of 32 per block: lane (l16, q) holds k = k0 + 8*q + 0..7 of its row / column
    bf16x8 a[4], b[4];
#pragma unroll
    for (int bm = 0; bm < 4; ++bm) a[bm] = *reinterpret_cast<const bf16x8 *>(&As[wm + bm * 16 + l16][q * 8]);
#pragma unroll
    for (int bn = 0; bn < 4; ++bn) b[bn] = *reinterpret_cast<const bf16x8 *>(&Bs[wn + bn * 16 + l16][q * 8]);
#pragma unroll
    for (int bm = 0; bm < 4; ++bm)
#pragma unroll
      for (int bn = 0; bn < 4; ++bn) acc[bm][bn] = mma_16x16x32(a[bm], b[bn], acc[bm][bn]);
  }

#pragma unroll
  for (int bm = 0; bm < 4; ++bm)
#pragma unroll
    for (int bn = 0; bn < 4; ++bn) {
      const int m = m0 + wm + bm * 16 + l16, n = n0 + wn + bn * 16 + 4 * q;
      if (m >= p.M || n >= p.N) continue;  // N is a multiple of 8 and n of 4: the 4 columns are in or out together
      store_acc4<kEpi>(p, acc[bm][bn], plane_row + m, n, s_tab);
    }
}

template <bool kAK, bool kBK, int kEpi, bool kAccIn>
hipError_t launch_generic(const GemmParams &p, hipStream_t stream) {
  const int tiles = ((p.M + GBM - 1) / GBM) * ((p.N + GBN - 1) / GBN);
  const int parts = p.k_parts > 1 ? p.k_parts : 1;
  hipLaunchKernelGGL((gemm_generic_kernel<kAK, kBK, kEpi, kAccIn>), dim3(tiles * parts), dim3(256), 0, stream, p);
  return hipGetLastError();
}

// The kernels use more dynamic LDS than the default limit; the attribute is set once per kernel and device.
constexpr int kMaxDevices = 16;

template <class Kernel>
hipError_t allow_lds(Kernel kernel, size_t lds, bool (&configured)[kMaxDevices]) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  if (!configured[dev]) {  // a benign race sets the same attribute twice
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            static_cast<int>(lds));
    if (e != hipSuccess) return e;
    configured[dev] = true;
  }
  return hipSuccess;
}

int tile_columns_of(const GemmParams &p, int BN) {
  return p.seg_n ? p.N / p.seg_n * ((p.seg_n + BN - 1) / BN) : (p.N + BN - 1) / BN;
}

template <int BM, int BN, int WM, int WN, int BK, int kStages, bool kAK, bool kBK, int kEpi, bool kAccIn>
hipError_t launch_dma(const GemmParams &p, hipStream_t stream) {
  constexpr int kWaves = (BM / WM) * (BN / WN);
  constexpr size_t lds = static_cast<size_t>(kStages) * (BM + BN) * BK * sizeof(uint16_t);
  static_assert(lds + OSDP_MAX_SHARDS * 8 <= 160 * 1024, "tile does not fit the 160 KB of LDS");
  auto kernel = gemm_dma_kernel<BM, BN, WM, WN, BK, kStages, kAK, kBK, kEpi, kAccIn>;
  static bool configured[kMaxDevices] = {};
  hipError_t e = allow_lds(kernel, lds, configured);
  if (e != hipSuccess) return e;
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = tile_columns_of(p, BN);
  const int parts = p.k_parts > 1 ? p.k_parts : 1;
  hipLaunchKernelGGL(kernel, dim3(tiles_m * tiles_n * parts), dim3(kWaves * 64), lds, stream, p, tiles_m, tiles_n);
  return hipGetLastError();
}

// The four-wave kernel, two K blocks of 64 in LDS (128 KB): 256 x 256 tiles, or fewer rows or columns (32 per block).
template <int MB, int NB, bool kAK, bool kBK, int kEpi, bool kAccIn, bool kCopy>
hipError_t launch_w4(const GemmParams &p, hipStream_t stream) {
  constexpr size_t lds = 2 * (W4Operand<kAK, MB>::kElems + W4Operand<kBK, NB>::kElems) * sizeof(uint16_t);
  static_assert(lds + 2 * OSDP_MAX_SHARDS * 8 <= 160 * 1024, "tile does not fit the 160 KB of LDS");
  auto kernel = [] {
    if constexpr (MB == 8 && NB == 8) return gemm_w4_kernel<kAK, kBK, kEpi, kAccIn, kCopy>;
    else return gemm_w4_small_kernel<MB, NB, kAK, kBK, kEpi, kAccIn, kCopy>;
  }();
  static bool configured[kMaxDevices] = {};
  hipError_t e = allow_lds(kernel, lds, configured);
  if (e != hipSuccess) return e;
  const int tiles_m = (p.M + 32 * MB - 1) / (32 * MB), tiles_n = tile_columns_of(p, 32 * NB);
  const int parts = p.k_parts > 1 ? p.k_parts : 1;
  hipLaunchKernelGGL(kernel, dim3(tiles_m * tiles_n * parts), dim3(256), lds, stream, p, tiles_m, tiles_n);
  return hipGetLastError();
}

// The same with 128 x 128 tiles, 32 KB a slot.
template <int kSlots, bool kAK, bool kBK, int kEpi, bool kAccIn>
hipError_t launch_w4_128(const GemmParams &p, hipStream_t stream) {
  constexpr size_t lds = static_cast<size_t>(kSlots) * (W4Operand<kAK, 4>::kElems + W4Operand<kBK, 4>::kElems) * sizeof(uint16_t);
  static_assert((kSlots == 2 ? 2 : 1) * (lds + OSDP_MAX_SHARDS * 8) <= 160 * 1024, "tile does not fit the 160 KB of LDS");
  auto kernel = gemm_w4_128_kernel<kSlots, kAK, kBK, kEpi, kAccIn>;
  static bool configured[kMaxDevices] = {};
  hipError_t e = allow_lds(kernel, lds, configured);
  if (e != hipSuccess) return e;
  const int tiles_m = (p.M + 127) / 128, tiles_n = tile_columns_of(p, 128);
  const int parts = p.k_parts > 1 ? p.k_parts : 1;
  hipLaunchKernelGGL(kernel, dim3(tiles_m * tiles_n * parts), dim3(256), lds, stream, p, tiles_m, tiles_n);
  return hipGetLastError();
}

// The same with 160 columns and 128 or 64 rows.
template <int MB, bool kAK, bool kBK, int kEpi, bool kAccIn>
hipError_t launch_w4_160(const GemmParams &p, hipStream_t stream) {
  constexpr size_t slot = (W4Operand<kAK, MB>::kElems + W4Operand<kBK, 5>::kElems) * sizeof(uint16_t);
  constexpr int kSlots = 5 * slot <= 160 * 1024 ? 5 : (4 * slot <= 160 * 1024 ? 4 : 3);
  static_assert(kSlots * slot <= 160 * 1024 && kEpi != static_cast<int>(Epilogue::kBf16ShardMajor), "tile does not fit the 160 KB of LDS");
  auto kernel = gemm_w4_160_kernel<MB, kSlots, kAK, kBK, kEpi, kAccIn>;
  static bool configured[kMaxDevices] = {};
  hipError_t e = allow_lds(kernel, kSlots * slot, configured);
  if (e != hipSuccess) return e;
  const int tiles_m = (p.M + 32 * MB - 1) / (32 * MB), tiles_n = tile_columns_of(p, 160);
  const int parts = p.k_parts > 1 ? p.k_parts : 1;
  hipLaunchKernelGGL(kernel, dim3(tiles_m * tiles_n * parts), dim3(256), kSlots * slot, stream, p, tiles_m, tiles_n);
  return hipGetLastError();
}

// Adds up the fp32 planes of a launch that was split along K, plane 0 first, and stores the sum through the
// launch's own epilogue.  One thread per 4 consecutive columns.
template <int kEpi>
__global__ __launch_bounds__(256)
void combine_parts_kernel(GemmParams p, const float *parts, int n_parts) {
  uint16_t *const *s_tab = nullptr;
  if constexpr (kEpi == static_cast<int>(Epilogue::kBf16ShardMajor)) {
    __shared__ uint16_t *tab[OSDP_MAX_SHARDS];
    if (threadIdx.x < OSDP_MAX_SHARDS) tab[threadIdx.x] = static_cast<uint16_t *>(p.shards.p[threadIdx.x]);
    __syncthreads();
    s_tab = tab;
  }
  const int64_t plane = static_cast<int64_t>(p.M) * p.N;
  const int64_t v = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (v * 4 >= plane) return;
  const int per_row = p.N / 4;
  const int m = static_cast<int>(v / per_row), n = static_cast<int>(v - static_cast<int64_t>(m) * per_row) * 4;
  const float4 *src = reinterpret_cast<const float4 *>(parts) + v;
  float4 a = src[0];
  for (int s = 1; s < n_parts; ++s) {
    const float4 b = src[static_cast<int64_t>(s) * (plane / 4)];
    a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
  }
  const f32x4 c = {a.x, a.y, a.z, a.w};
  store_acc4<kEpi>(p, c, m, n, s_tab);
}

constexpr int kCUs = 256;

thread_local int64_t t_persistent_launches = 0;

// The persistent form of the four-wave kernel: one workgroup per CU walks through the tiles.
template <int MB, int NB, bool kAK, bool kBK, int kEpi, bool kAccIn>
hipError_t launch_w4p(const GemmParams &p, hipStream_t stream) {
  constexpr size_t lds = 2 * (W4Operand<kAK, MB>::kElems + W4Operand<kBK, NB>::kElems) * sizeof(uint16_t);
  auto kernel = [] {
    if constexpr (MB == 8 && NB == 8) return gemm_w4p_kernel<kAK, kBK, kEpi, kAccIn>;
    else return gemm_w4p_small_kernel<MB, NB, kAK, kBK, kEpi, kAccIn>;
  }();
  static bool configured[kMaxDevices] = {};
  hipError_t e = allow_lds(kernel, lds, configured);
  if (e != hipSuccess) return e;
  const int tiles_m = (p.M + 32 * MB - 1) / (32 * MB), tiles_n = tile_columns_of(p, 32 * NB);
  const int tiles = tiles_m * tiles_n * (p.k_parts > 1 ? p.k_parts : 1);
  hipLaunchKernelGGL(kernel, dim3(tiles < kCUs ? tiles : kCUs), dim3(256), lds, stream, p, tiles_m, tiles_n);
  t_persistent_launches += 1;
  return hipGetLastError();
}

constexpr int kShortK = 1024;
constexpr int kW4MinK = 129;  // 256 x 256 tiles: from three K blocks of 64 on the four-wave kernel (both sides at case 0 of launch_best)

// Estimated cost of covering M x N with BM x BN tiles on 256 CUs: tiles per CU times the tile's area, with a
// penalty for the lower MFMA efficiency of smaller tiles.  Tiles that run two to a CU were measured in pairs; a
// CU's odd last tile runs alone and slower, which is priced as one and a half tiles.  A launch of one to two tiles of
// 128 x 128 per CU lasts nearly as its number of tiles: what it waits for is the memory that the CUs share (K = 2560: 320
// tiles 38 us, 480 tiles 52 us).  Of tiles of 256 x 128 and 128 x 256 one and a quarter a CU last nearly as long as two
// (1.5 + 0.25 x; us against 256 x 256, one to a CU: 4096 x 2688 over K = 2688 73 and 72 against 65, dX 74 and 75 against 62;
// 2048 x 6144 over 6912 178 and 172 against 155; 768 x 14592 over 9984 305 and 274 against 239; dW of 2048 x 5632 over 16384
// tokens 392 and 421 against 374).  A tile that sticks out of the matrix costs what a full one does.
// lone > 0: the penalty of a launch of at most one tile per CU, which has the CU's whole LDS for its pipeline.
long tile_count(int M, int N, int BM, int BN) { return static_cast<long>((M + BM - 1) / BM) * ((N + BN - 1) / BN); }

double tile_cost(int M, int N, int BM, int BN, double penalty, int parts = 1, double lone = 0.0) {
  const long tiles = tile_count(M, N, BM, BN) * parts;
  const long per_cu = (tiles + kCUs - 1) / kCUs;
  const bool two_per_cu = BM * BN <= 256 * 128;
  if (two_per_cu && per_cu == 1 && lone > 0.0) return lone * BM * BN;
  const double x = static_cast<double>(tiles) / kCUs;
  const double units = (two_per_cu && per_cu == 2)  ? (BM * BN > 128 * 128 ? 1.5 + 0.25 * x : 0.4 + 0.8 * x)
                       : (two_per_cu && per_cu % 2) ? static_cast<double>(per_cu) + 0.5
                                                    : static_cast<double>(per_cu);
  return units * BM * BN * penalty;
}

// The direct-to-LDS kernels take every size; a second segment of B must start on a K block or a tile column.
bool fast_path(int K, int k_split, int n_split) {
  const bool generic = debug_options().gemm_generic.load(std::memory_order_relaxed) != 0;  // testing: the bounds-checked kernel
  return !generic && K > 0 && k_split % 64 == 0 && n_split % 128 == 0;
}

// Their lanes address an operand's tile with 32-bit byte offsets.
constexpr int64_t kMaxLd = 1 << 22;
bool fits_offsets(const GemmParams &p) { return p.lda < kMaxLd && p.ldb < kMaxLd && p.ldb2 < kMaxLd; }

// Tile shapes of the direct-to-LDS kernels and their measured cost per unit of tile area relative to 256 x 256, for
// the three operand layouts (forward, dW, dX).
struct TileShape {
  int bm, bn;
  double penalty[3];
  double lone[3];  // the same for a launch of at most one tile per CU
};
// 8192^3 on MI355X, forward / dW / dX in PFLOP/s: 256x256 on the four-wave kernel 1.47 / 1.45 / 1.48, on the eight-wave one 1.27 / 1.37 /
// 1.37; 256x128 (two workgroups per CU) 1.19 / 1.28 / 1.10; 128x256 (two per CU) 1.28 / 1.27 / 1.06; 128x128 (two per CU) 1.20 / 1.12 /
// 1.20.  The penalties are older than these kernels' short epilogues and than the four-wave kernel's 128x128 tiles: they were taken
// from 1.43 / 1.30 / 1.45 for 256x256 against 1.04 / 0.90 / 1.09, 1.19 / 1.02 / 1.06 and 1.03 / 1.05 / 1.03 (128x128 in eight waves), and
// fitted to launches of one and two tiles a CU.  From the rates above they would be 1.23 / 1.13 / 1.34, 1.15 / 1.14 / 1.39 and 1.23 / 1.30 / 1.23;
// with those below the choice was still within 6 % of the best tile in 183 of 192 launches (4096 rows, 512 to 12288 columns, K from
// 1024 to 10240).
// K block and LDS stages of the eight-wave kernels per layout, also measured: forward (transposing reads of B) runs
// best with K blocks of 64 in two stages, dW and dX on the 256x256 tile with K blocks of 32 in four stages.
// The smaller tiles are sized for two workgroups per CU.  A launch with no more tiles than CUs has one, and is
// then bound by the latency of its loads (1024x4096x8192 for dW on 128x128 tiles: 41 GB/s per CU with 48 KB in
// flight); it takes the CU's whole LDS for K blocks of 64 in three or four stages: the forward launch over two 256-column
// slices with K = 4096 64 -> 52 us.  The 128x128 tile runs on the four-wave kernel (gemm_w4_128_kernel).
// 224 x 256 and 256 x 160 run on the four-wave kernel alone, in the layouts where they were measured (0: not offered).  They fill
// rounds that whole tiles leave partly empty; the smaller the tile the more bytes from L2 each MFMA needs, which is
// what the penalties are (7 % more for 224 x 256, 30 % more for 256 x 160).  dW of 2560 x 5120 over 16384 tokens: 200
// tiles of 256 rows 412 us, 240 of 224 rows 382 us.  8192 x 1280 over K = 2560: 160 tiles of 256 columns 60 us, 256
// tiles of 160 columns 51 us (dX 48 us); where they only replace full rounds the narrow tiles lose (16384 x 2560 over
// K = 2560 in 4 rounds 240 us, against 196 us for two rounds of large tiles and a remainder).
// 128 x 160 and 64 x 160 are for dX launches of at most one tile per CU: narrow slices, and few rows.  Both operands keep whole rows of
// K blocks in LDS, so any number of rows and columns fits.  us in 128 x 128 tiles / in these: 8192 x 320 over K = 10240 71 / 64,
// 1000 x 5120 over 2560 38 / 29, 2048 x 1280 over 4096 31 / 28, 4096 x 128 over 2048 17 / 15.  (The forward, whose weight
// tile takes 256 columns of LDS for 160, loses: 8192 x 320 over 10240 86 / 95.)
// 256 x 160 from K = 768 on, one tile to a CU, against two tiles of 128 x 128 or fewer of 256 x 256, us: dX of 4096 x 2304 over 768 24.5 /
// 21.5, 4096 x 2560 over 768 25.0 / 21.1 and over 1024 29.5 / 24.5, 8192 x 1280 over 1024 29.5 / 24.5; forward of 4096 x 2304 over 768 26.6 /
// 23.4, 4096 x 2560 over 768 25.6 / 22.7, over 1024 30.2 / 25.8 and over 1536 39.0 / 33.9, 3001 x 3200 over 1024 29.6 / 25.2.
constexpr int kTileShapes = 8, kPricedShapes = 6;
// lone: K = 2560 to 10240 against 256 x 256 tiles of the same K, one to a CU.  In place of two 128 x 128 tiles a CU, one
// of 256 x 128 took 2048 x 4096 over K = 4096 from 76 to 65 us (dX 69 to 64), 3001 x 2560 over K = 2560 from 52 to 45.
constexpr TileShape kTiles[kTileShapes] = {{256, 256, {1.0, 1.0, 1.0}, {1.0, 1.0, 1.0}},
                                           {256, 128, {1.37, 1.40, 1.33}, {1.19, 1.15, 1.16}},
                                           {128, 256, {1.21, 1.23, 1.37}, {1.21, 1.20, 1.22}},
                                           {128, 128, {1.39, 1.20, 1.40}, {1.60, 1.55, 1.60}},
                                           {224, 256, {0.0, 1.06, 0.0}, {0.0, 1.06, 0.0}},
                                           {256, 160, {1.30, 0.0, 1.28}, {1.30, 0.0, 1.28}},
                                           {128, 160, {0.0, 0.0, 0.0}, {0.0, 0.0, 1.35}},
                                           {64, 160, {0.0, 0.0, 0.0}, {0.0, 0.0, 1.70}}};
// From which K 256 x 160 is launched, and from which it counts where slices are paired: how much workspace a call asks for hangs on
// that, and must not change with the kernels.
constexpr int kNarrowMinK = 768, kNarrowPricedK = 2048;

constexpr int layout_kind(bool a_kcontig, bool b_kcontig) { return (a_kcontig && !b_kcontig) ? 0 : (!a_kcontig ? 1 : 2); }

// Whether tile shape i serves a launch of the layout with K as the reduction of a workgroup: the four-wave kernel's own
// shapes from a K loop that pays for its start-up.
bool tile_offered(int i, int kind, int K, int narrow_k = kNarrowMinK) {
  if (i < 4) return true;
  if (i >= kPricedShapes) return kTiles[i].lone[kind] > 0.0 && debug_options().small_tile.load(std::memory_order_relaxed) != 0;
  return kTiles[i].penalty[kind] > 0.0 && K >= (kind == 1 ? kW4MinK : narrow_k) &&
         debug_options().four_wave.load(std::memory_order_relaxed) != 0 &&
         debug_options().small_tile.load(std::memory_order_relaxed) != 0;
}

// What a tile is chosen for, which decides the shapes and prices that count.
enum class TileUse {
  kLaunch,       // a launch, or a plan of launches, that starts from zero: all shapes
  kSumLaunch,    // a launch that starts from a sum in memory: no prices of lone tiles, whose first K blocks alone would have to
                 // cover that load (2048 x 4096 over K = 4096 and 8192 1 to 3 us slower than in pairs of 128 x 128)
  kSumPlan,      // a plan of such launches: see plan_launches
  kFirstShapes,  // the shapes that workspace sizes were first given for
};

// Cheapest tile for M x N; a column split must fall on a tile boundary.
// parts > 1: the launch has that many workgroups per tile (parts of the reduction); the cost is in tile passes over
// the whole reduction all the same, so the caller divides it by parts.
int best_tile(int M, int N, int K, int n_split, int kind, double *cost, int parts = 1, TileUse use = TileUse::kLaunch) {
  const bool lone = use != TileUse::kSumLaunch && debug_options().deep.load(std::memory_order_relaxed) != 0;
  const int shapes = lone && use == TileUse::kLaunch ? kTileShapes : kPricedShapes;
  int best = -1;
  double best_cost = 0.0;
  for (int i = 0; i < shapes; ++i) {
    if (i >= kPricedShapes && tile_count(M, N, kTiles[i].bm, kTiles[i].bn) * parts > kCUs) continue;  // lone tiles only
    if (n_split % kTiles[i].bn || !tile_offered(i, kind, K / parts, use == TileUse::kFirstShapes ? kNarrowPricedK : kNarrowMinK)) continue;
    const double c = tile_cost(M, N, kTiles[i].bm, kTiles[i].bn, kTiles[i].penalty[kind], parts, lone ? kTiles[i].lone[kind] : 0.0);
    if (best < 0 || c < best_cost) {
      best = i;
      best_cost = c;
    }
  }
  if (cost) *cost = best_cost;
  return best;
}

// ---- concatenating launches split along K ----------------------------------------------------------------------
// A slice of a wide operator applied to few tokens (4096 x 1024 x 32768) has few output tiles and a long reduction:
// most CUs get no 256 x 256 tile, and the 128 x 128 tiles that would occupy them run at 70 % of the large tile's
// rate.  The forward product of such an operator over column slices (and likewise dX over row slices) is therefore
// defined as the sum of kPartK-long parts of the reduction: the parts run side by side as one launch (grid = parts x tiles), each into its own fp32 plane, and a
// second kernel adds the planes, plane 0 first, and rounds to bf16.  The number of parts depends on the token count
// and the reduction length alone - never on the slice width, the tile shape or the kernel - so Y keeps the same bits
// for every k, as the unsplit operator (k = 1) runs the same parts.
// Measured on 4096 tokens, 32768 -> 8192, whole steps with parts of 16384 / 8192 / 4096 against none, in TFLOP/s:
// k = 8 two slots 1130 / 1122 / 1068 against 1082; k = 16 978 / 1017 / 981 against 987; k = 4 1181 / 1170 / 1107
// against 1187; k = 8 one slot 975 / 1020 / 979 against 986; k = 8 half slices 926 / 920 / 884 against 826.
constexpr int kPartK = 8192;          // length of a part
constexpr int kPartMaxTokens = 4096;  // more tokens than this fill the CUs with any slice width that is worth staging
constexpr int kMaxParts = 8;

int forward_k_parts(int64_t M, int64_t K) {
  if (debug_options().split_k.load(std::memory_order_relaxed) == 0) return 1;  // testing: one part always
  if (M <= 0 || M > kPartMaxTokens || K < 2 * kPartK) return 1;
  const int parts = static_cast<int>(std::min<int64_t>(K / kPartK, kMaxParts));
  return K % (static_cast<int64_t>(parts) * 64) ? 1 : parts;
}

// Estimated duration of the combining kernel: the planes read, the result written.
double combine_estimate_us(int64_t M, int64_t N, int parts) {
  return (4.0 * parts + 2.0) * static_cast<double>(M) * static_cast<double>(N) / 3.0e6 + 8.0;
}

// The four-wave kernel in the form that suits the number of tiles.
template <int MB, int NB, bool kAK, bool kBK, int kEpi, bool kAccIn>
hipError_t launch_four_wave(const GemmParams &p, hipStream_t stream, bool *carry) {
  const int parts = p.k_parts > 1 ? p.k_parts : 1;
  // More tiles than CUs: the persistent form overlaps each tile's start-up with its predecessor's end
  // (3-12 % per launch).  It takes no gather along: *carry stays as it is and the caller launches the
  // gather by itself, which measured better on every workload than keeping the plain kernel for its sake.
  const int pst = debug_options().persistent.load(std::memory_order_relaxed);  // testing: 0 never, 1 for any number of tiles
  if (pst != 0 && !(parts > 1 && (p.k_split || kAccIn)) && (pst == 1 || tile_count(p.M, p.N, 32 * MB, 32 * NB) * parts > kCUs))
    return launch_w4p<MB, NB, kAK, kBK, kEpi, kAccIn>(p, stream);
  if constexpr (!(kAK && kBK)) {  // dX launches read every staged slice there is: they never carry a gather
    if (*carry) {
      *carry = false;
      return launch_w4<MB, NB, kAK, kBK, kEpi, kAccIn, true>(p, stream);
    }
  }
  return launch_w4<MB, NB, kAK, kBK, kEpi, kAccIn, false>(p, stream);
}

// *carry: the launch has a gather to carry (GemmParams::job is filled in); cleared by the launch that takes it.
template <bool kAK, bool kBK, int kEpi, bool kAccIn>
hipError_t launch_best(const GemmParams &p, hipStream_t stream, bool *carry) {
  constexpr int kind = layout_kind(kAK, kBK);
  const int parts = p.k_parts > 1 ? p.k_parts : 1;  // parts of the reduction run as further tiles of the same launch
  if (fast_path(p.K, p.k_split, p.n_split) && fits_offsets(p)) {
    int best = best_tile(p.M, p.N, p.K, p.n_split, kind, nullptr, parts,
                         kAccIn ? TileUse::kSumLaunch : p.seg_n ? TileUse::kFirstShapes : TileUse::kLaunch);
    const int forced = debug_options().tile.load(std::memory_order_relaxed);  // testing: tile 0..3 where it fits the segments of B
    bool force = forced >= 0 && forced <= 3;
    if (force && p.n_split % kTiles[forced].bn == 0) best = forced;
    constexpr int small = kind == 1 ? 4 : 5;
    if (debug_options().small_tile.load(std::memory_order_relaxed) == 1 && p.n_split % kTiles[small].bn == 0 && p.K / parts >= kW4MinK) {
      best = small;  // testing
      force = true;
    }
    // A dX launch with a short reduction whose fp32 partial sum comes from or goes to memory is bound by that
    // traffic, and with only a round or two of large tiles every CU loads, computes and stores in step with the
    // others: two smaller workgroups per CU overlap one's loads and stores with the other's MFMAs (8192 x 4096 with
    // K = 256: 62 -> 54 us; with 8 rounds of large tiles, 4096 x 32768, the large tile stays 7 % ahead).
    if (kind == 2 && (kAccIn || kEpi == static_cast<int>(Epilogue::kF32Workspace)) && p.K <= kShortK && best == 0 &&
        tile_count(p.M, p.N, 256, 256) <= 2 * kCUs && !force)
      best = p.n_split % 256 == 0 ? 2 : 1;
    // A launch of at most one tile per CU cannot hide the latency of its loads behind a second workgroup: it gets
    // the whole LDS for a deeper pipeline instead (twice the bytes in flight).
    const bool deep = best > 0 && best < 4 && tile_count(p.M, p.N, kTiles[best].bm, kTiles[best].bn) * parts <= kCUs &&
                      debug_options().deep.load(std::memory_order_relaxed) != 0;  // testing: 0 keeps the shallow pipelines
    const int fw = debug_options().four_wave.load(std::memory_order_relaxed);  // testing: 0 never, 1 for any K
    switch (best) {
      case 0:
        // (The four-wave kernel takes any K; 256 x 256 tiles of the eight-wave kernel are left for at most two K blocks of 64, where
        // start-up is all there is and neither is ahead everywhere: us, eight / four waves, forward of 4096 x 4096 over K = 64 and 128
        // 13.2 / 13.8, 14.9 / 15.6, of 8192 x 16384 over 64 64 / 69, but 8192 x 8192 over 128 46 / 37; dX of those 13.1 / 13.5, 15.1 / 15.0,
        // 45 / 37; dW of 8192 x 16384 over 96 79 / 75.  dW ran on them
        // below 8192 tokens as long as the four-wave epilogue into shards took 32 us a tile and not 15; now, eight / four waves, 8192 x
        // 8192 over 4096 / 1024 / 256 tokens 417 / 378, 133 / 117, 59 / 50 us; 2560 x 10240 over 3001 and 1500 160 / 130, 83 / 74)
        if (fw != 0 && (fw == 1 || p.K / parts >= kW4MinK)) {
          return launch_four_wave<8, 8, kAK, kBK, kEpi, kAccIn>(p, stream, carry);
        }
        if (kind == 0) return launch_dma<256, 256, 64, 128, 64, 2, kAK, kBK, kEpi, kAccIn>(p, stream);
        return launch_dma<256, 256, 64, 128, 32, 4, kAK, kBK, kEpi, kAccIn>(p, stream);
      case 1:
        if (deep) return launch_dma<256, 128, 64, 64, 64, 3, kAK, kBK, kEpi, kAccIn>(p, stream);
        return launch_dma<256, 128, 64, 64, 32, 3, kAK, kBK, kEpi, kAccIn>(p, stream);
      case 2:
        if (deep) return launch_dma<128, 256, 64, 64, 64, 3, kAK, kBK, kEpi, kAccIn>(p, stream);
        return launch_dma<128, 256, 64, 64, 32, 3, kAK, kBK, kEpi, kAccIn>(p, stream);
      case 3:
        if (deep) return launch_w4_128<4, kAK, kBK, kEpi, kAccIn>(p, stream);
        return launch_w4_128<2, kAK, kBK, kEpi, kAccIn>(p, stream);
      case 4:
        if constexpr (kind == 1) return launch_four_wave<7, 8, kAK, kBK, kEpi, kAccIn>(p, stream, carry);
        break;
      case 5:
        if constexpr (kind != 1) return launch_four_wave<8, 5, kAK, kBK, kEpi, kAccIn>(p, stream, carry);
        break;
      case 6:
        if constexpr (kind == 2 && !kAccIn) return launch_w4_160<4, kAK, kBK, kEpi, kAccIn>(p, stream);
        break;
      case 7:
        if constexpr (kind == 2 && !kAccIn) return launch_w4_160<2, kAK, kBK, kEpi, kAccIn>(p, stream);
        break;
    }
  }
  if (p.k_split % GBK || p.n_split % GBN || p.seg_k || p.seg_n) return hipErrorInvalidValue;
  return launch_generic<kAK, kBK, kEpi, kAccIn>(p, stream);
}

// Columns [n0, n1) of a one-segment problem as a problem of its own.
template <bool kBK, int kEpi>
GemmParams column_range(const GemmParams &p, int n0, int n1) {
  GemmParams s = p;
  s.N = n1 - n0;
  s.B = kBK ? p.B + static_cast<int64_t>(n0) * p.ldb : p.B + n0;
  if (kEpi == static_cast<int>(Epilogue::kBf16ShardMajor)) s.c0 = p.c0 + n0;
  else if (kEpi == static_cast<int>(Epilogue::kF32Workspace)) s.C = static_cast<float *>(p.C) + n0;
  else s.C = static_cast<uint16_t *>(p.C) + n0;
  if (p.acc_in) s.acc_in = p.acc_in + n0;
  return s;
}

// Rows [m0, m1) likewise.
template <bool kAK, int kEpi>
GemmParams row_range(const GemmParams &p, int m0, int m1) {
  GemmParams s = p;
  s.M = m1 - m0;
  s.A = kAK ? p.A + static_cast<int64_t>(m0) * p.lda : p.A + m0;
  if (kEpi == static_cast<int>(Epilogue::kBf16ShardMajor)) s.r0 = p.r0 + m0;
  else if (kEpi == static_cast<int>(Epilogue::kF32Workspace)) s.C = static_cast<float *>(p.C) + static_cast<int64_t>(m0) * p.ldc;
  else s.C = static_cast<uint16_t *>(p.C) + static_cast<int64_t>(m0) * p.ldc;
  if (p.acc_in) s.acc_in = p.acc_in + static_cast<int64_t>(m0) * p.ld_acc;
  return s;
}

// A problem whose 256 x 256 tiles fill the CUs a whole number of times plus a little is run as two launches:
// the part that makes (nearly) whole rounds on the large tile, and the remainder on whatever tile suits it
// (usually a small one that spreads it over all CUs).  Tile shape never changes a result bit, so neither does this.
// Returns the modelled cost (tile-area units) of the best plan for a one-segment M x N x K problem of the given
// layout; axis = 1: columns [0, cut) and [cut, N) are launched separately; axis = 0: rows; axis = -1: one launch.
// acc_in: launches that start from a sum in memory.  They run no tile that is for lone launches only, and none is priced here: a
// remainder that looked as cheap as in 64 x 160 tiles ran in 128 x 128 (a dX pass of three slices, us priced so / priced as
// here: 10241 x 3136 over K = 512 224 / 199, 6131 x 3008 over 3264 385 / 363, 5652 x 2944 over 1024 184 / 170).  The shapes that both
// kinds of launches run keep their prices as lone tiles, although best_tile picks those launches without: with both alike 60
// dX passes are as fast within 0.4 %, and 39 forward passes 3 % slower, some by 15.
double plan_launches(int M, int N, int K, int kind, bool acc_in, int *axis, int *cut) {
  const TileUse use = acc_in ? TileUse::kSumPlan : TileUse::kLaunch;
  double whole = 0.0;
  *axis = -1;
  *cut = 0;
  best_tile(M, N, K, 0, kind, &whole, 1, use);
  // testing: split_launch = 0 keeps every problem in one launch, as does a forced tile shape
  if (debug_options().split_launch.load(std::memory_order_relaxed) == 0 ||
      debug_options().tile.load(std::memory_order_relaxed) >= 0)
    return whole;
  const int tm = (M + 255) / 256, tn = (N + 255) / 256;
  const double between = 1.0e7 / K;  // about 5 us from one launch to the next, in the cost's units of tile area
  double best = 0.95 * whole;        // only for a clear gain
  double rest = 0.0;
  // candidate cuts: for every number of rounds r, the most tile columns (rows) that r rounds of large tiles hold
  for (int r = 1; r <= 16; ++r) {
    const int cn = static_cast<int>(static_cast<long>(kCUs) * r / tm);
    if (cn <= 0) continue;
    if (cn >= tn) break;
    best_tile(M, N - cn * 256, K, 0, kind, &rest, 1, use);
    const double c = tile_cost(M, cn * 256, 256, 256, 1.0) + rest + between;
    if (c < best) { best = c; *axis = 1; *cut = cn * 256; }
  }
  for (int r = 1; r <= 16; ++r) {
    const int cm = static_cast<int>(static_cast<long>(kCUs) * r / tn);
    if (cm <= 0) continue;
    if (cm >= tm) break;
    best_tile(M - cm * 256, N, K, 0, kind, &rest, 1, use);
    const double c = tile_cost(cm * 256, N, 256, 256, 1.0) + rest + between;
    if (c < best) { best = c; *axis = 0; *cut = cm * 256; }
  }
  return *axis >= 0 ? best : whole;
}

template <bool kAK, bool kBK, int kEpi, bool kAccIn>
hipError_t launch_planned(const GemmParams &p, hipStream_t stream, bool *carry, float *planes, size_t planes_bytes) {
  // (forward launches of column slices, and the dX launches of row slices, which have the same shape of problem:
  // few tokens, a slice's worth of output columns, the whole uncut dimension as the reduction)
  if constexpr (kAK && !kAccIn && kEpi == static_cast<int>(Epilogue::kBf16RowMajor)) {
    // (a caller that passes no planes asks for the one-part product: the forward of row slices, whose launches
    // continue one accumulator chain instead)
    const int parts = (p.k_split || !planes) ? 1 : forward_k_parts(p.M, p.K);
    if (parts > 1) {
      if (planes_bytes < static_cast<size_t>(parts) * p.M * p.N * 4) return hipErrorInvalidValue;
      constexpr int kF32 = static_cast<int>(Epilogue::kF32Workspace);
      GemmParams s = p;
      s.k_parts = parts;
      s.C = planes;
      s.ldc = p.N;
      hipError_t e = launch_best<kAK, kBK, kF32, false>(s, stream, carry);
      if (e != hipSuccess) return e;
      const int64_t vecs = static_cast<int64_t>(p.M) * p.N / 4;
      hipLaunchKernelGGL((combine_parts_kernel<kEpi>), dim3(static_cast<unsigned>((vecs + 255) / 256)), dim3(256), 0, stream, p,
                         static_cast<const float *>(planes), parts);
      return hipGetLastError();
    }
  }
  if (!p.k_split && !p.n_split && !p.seg_k && !p.seg_n && fast_path(p.K, 0, 0) && fits_offsets(p)) {
    int axis, cut;
    plan_launches(p.M, p.N, p.K, layout_kind(kAK, kBK), kAccIn, &axis, &cut);
    if (axis == 1) {
      hipError_t e = launch_best<kAK, kBK, kEpi, kAccIn>(column_range<kBK, kEpi>(p, 0, cut), stream, carry);
      if (e != hipSuccess) return e;
      return launch_best<kAK, kBK, kEpi, kAccIn>(column_range<kBK, kEpi>(p, cut, p.N), stream, carry);
    }
    if (axis == 0) {
      hipError_t e = launch_best<kAK, kBK, kEpi, kAccIn>(row_range<kAK, kEpi>(p, 0, cut), stream, carry);
      if (e != hipSuccess) return e;
      return launch_best<kAK, kBK, kEpi, kAccIn>(row_range<kAK, kEpi>(p, cut, p.M), stream, carry);
    }
  }
  return launch_best<kAK, kBK, kEpi, kAccIn>(p, stream, carry);
}

}  // namespace

namespace {
bool shards_are_k_blocks(const ShardLayout &lay) { return lay.rows_per_shard > 0 && lay.rows_per_shard % 64 == 0; }
}  // namespace

bool gemm_reads_shards(int64_t T, int64_t ld_act, const ShardLayout &lay) {
  const DebugOptions &d = debug_options();
  const bool forced = d.gemm_generic.load(std::memory_order_relaxed) != 0 || d.tile.load(std::memory_order_relaxed) >= 0 ||
                      d.fwd_pair.load(std::memory_order_relaxed) >= 0 || d.fused_gather.load(std::memory_order_relaxed) >= 0 ||
                      d.poison_staging.load(std::memory_order_relaxed) != 0;  // (these ask for the staged schedule)
  return !forced && T <= kShardReadMaxTokens && shards_are_k_blocks(lay) && ld_act < kMaxLd && lay.O < kMaxLd;
}

int gemm_forward_parts(int64_t M, int64_t K) { return forward_k_parts(M, K); }

bool gemm_takes_two_segments(int64_t k_first, int64_t k_second) {
  return k_first > 0 && k_second > 0 && fast_path(static_cast<int>(k_first + k_second), static_cast<int>(k_first), 0);
}

bool gemm_takes_two_column_segments(int64_t n_first, int64_t n_second, int64_t K) {
  return n_first > 0 && n_second > 0 && fast_path(static_cast<int>(K), 0, static_cast<int>(n_first));
}

double gemm_estimate_us(int64_t M, int64_t N, int64_t K, bool forward_parts) {
  // one CU sustains about 5e6 flop per microsecond (1.3 PFLOP/s over 256 CUs) on 256 x 256 tiles
  // (one launch on its best tile: pricing the whole-rounds + remainder pair here instead was measured and made the
  // forward launch grouping of config 3 slightly worse)
  double cost = 0.0;
  if (M > 0 && fast_path(static_cast<int>(K), 0, 0)) {
    // (how slices are paired decides how much workspace a call asks for: it goes by the shapes that sizes were first given for)
    best_tile(static_cast<int>(M), static_cast<int>(N), static_cast<int>(K), 0, 0, &cost, 1, TileUse::kFirstShapes);
    const int parts = forward_parts ? forward_k_parts(M, K) : 1;
    if (parts > 1) {
      best_tile(static_cast<int>(M), static_cast<int>(N), static_cast<int>(K), 0, 0, &cost, parts, TileUse::kFirstShapes);
      return cost / parts * 2.0 * static_cast<double>(K) / 5.0e6 + combine_estimate_us(M, N, parts) + 6.0;
    }
    return cost * 2.0 * static_cast<double>(K) / 5.0e6 + 6.0;
  }
  const double tiles = static_cast<double>((M + GBM - 1) / GBM) * static_cast<double>((N + GBN - 1) / GBN);
  const double rounds = static_cast<double>(static_cast<long>((tiles + kCUs - 1) / kCUs));
  return rounds * GBM * GBN * 5.0 * 2.0 * static_cast<double>(K) / 5.0e6 + 6.0;  // the checked kernel is about 5x slower per tile
}

double gemm_planned_us(int64_t M, int64_t N, int64_t K, bool dx, bool acc_in) {
  if (M <= 0 || !fast_path(static_cast<int>(K), 0, 0)) return gemm_estimate_us(M, N, K);
  int axis, cut;
  const double cost = plan_launches(static_cast<int>(M), static_cast<int>(N), static_cast<int>(K), dx ? 2 : 0, acc_in, &axis, &cut);
  return cost * 2.0 * static_cast<double>(K) / 5.0e6 + 6.0;
}

int64_t gemm_persistent_launches() { return t_persistent_launches; }

size_t gemm_forward_parts_bytes(int64_t M, int64_t N, int64_t K) {
  const int parts = forward_k_parts(M, K);
  return parts > 1 && N > 0 ? static_cast<size_t>(parts) * static_cast<size_t>(M) * static_cast<size_t>(N) * 4 : 0;
}

hipError_t check_device() {
  static std::atomic<int8_t> verdict[kMaxDevices] = {};  // 0: not looked at, 1: fits, -1: does not
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  int8_t v = verdict[dev].load(std::memory_order_relaxed);
  if (v == 0) {
    int cus = 0, xcds = 0;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&xcds, hipDeviceAttributeNumberOfXccs, dev)) != hipSuccess) return e;
    v = (cus == kCUs && xcds == kXcds) ? 1 : -1;
    verdict[dev].store(v, std::memory_order_relaxed);
  }
  return v > 0 ? hipSuccess : hipErrorInvalidDevice;
}

namespace {
GemmParams gemm_params(const GemmProblem &q) {
  GemmParams p{};
  p.M = q.M; p.N = q.N; p.K = q.K;
  p.A = static_cast<const uint16_t *>(q.A); p.lda = q.lda;
  p.B = static_cast<const uint16_t *>(q.B); p.ldb = q.ldb;
  p.C = q.C; p.ldc = q.ldc;
  p.acc_in = q.acc_in; p.ld_acc = q.ld_acc;
  p.lay = q.layout; p.c0 = q.c0; p.r0 = q.r0; p.shards = q.shards;
  p.B2 = static_cast<const uint16_t *>(q.B2); p.ldb2 = q.ldb2;
  p.k_split = q.B2 ? q.k_split : 0; p.n_split = q.B2 ? q.n_split : 0;
  p.seg_k = q.b_kcontig ? 0 : q.b_shard_rows; p.seg_n = q.b_kcontig ? q.b_shard_rows : 0;
  return p;
}

hipError_t dispatch_gemm(const GemmProblem &q, hipStream_t stream, bool *carry) {
  GemmParams p = gemm_params(q);
  if (q.b_shard_rows && (!q.a_kcontig || q.acc_in || p.k_split || p.n_split || p.seg_k % 64)) return hipErrorInvalidValue;
  if (*carry) {
    const GatherRequest &g = *q.carry;
    const uint64_t total = static_cast<uint64_t>(g.rows) * (static_cast<uint64_t>(g.w) / 8);
    if (g.w % 8 || (total >> 32) || (reinterpret_cast<uintptr_t>(g.staging) & 15u)) return hipErrorInvalidValue;
    p.job.src = g.shards; p.job.lay = g.layout;
    p.job.r0 = static_cast<uint32_t>(g.r0); p.job.c0 = static_cast<uint64_t>(g.c0);
    p.job.vecs_per_row = static_cast<uint32_t>(g.w / 8); p.job.total_vecs = total;
    p.job.dst = static_cast<uint4 *>(g.staging);
  }
  if ((p.k_split || p.n_split) && !q.a_kcontig) return hipErrorInvalidValue;  // dW never takes a second segment
  if (p.k_split && p.n_split) return hipErrorInvalidValue;
  float *planes = static_cast<float *>(q.parts);
  const size_t planes_bytes = q.parts_bytes;
  constexpr int kRow = static_cast<int>(Epilogue::kBf16RowMajor), kShard = static_cast<int>(Epilogue::kBf16ShardMajor),
                kF32 = static_cast<int>(Epilogue::kF32Workspace);
  const bool acc = q.acc_in != nullptr;
  // The three GEMMs of the split linear layer, with the four accumulate forms for forward and dX, are the only combinations built.
  if (q.a_kcontig && !q.b_kcontig) {                                               // forward (accumulating when the reduction dimension is split)
    if (q.epilogue == Epilogue::kBf16RowMajor) return acc ? launch_planned<true, false, kRow, true>(p, stream, carry, planes, planes_bytes) : launch_planned<true, false, kRow, false>(p, stream, carry, planes, planes_bytes);
    if (q.epilogue == Epilogue::kF32Workspace) return acc ? launch_planned<true, false, kF32, true>(p, stream, carry, planes, planes_bytes) : launch_planned<true, false, kF32, false>(p, stream, carry, planes, planes_bytes);
  }
  if (!q.a_kcontig && !q.b_kcontig && !acc) {                                      // dW: into the shards, or (DP slice) a plain array
    if (q.epilogue == Epilogue::kBf16ShardMajor) return launch_planned<false, false, kShard, false>(p, stream, carry, planes, planes_bytes);
    if (q.epilogue == Epilogue::kBf16RowMajor) return launch_planned<false, false, kRow, false>(p, stream, carry, planes, planes_bytes);
  }
  if (q.a_kcontig && q.b_kcontig) {                                                // dX
    if (q.epilogue == Epilogue::kBf16RowMajor) return acc ? launch_planned<true, true, kRow, true>(p, stream, carry, planes, planes_bytes) : launch_planned<true, true, kRow, false>(p, stream, carry, planes, planes_bytes);
    if (q.epilogue == Epilogue::kF32Workspace) return acc ? launch_planned<true, true, kF32, true>(p, stream, carry, planes, planes_bytes) : launch_planned<true, true, kF32, false>(p, stream, carry, planes, planes_bytes);
  }
  return hipErrorInvalidValue;
}
}  // namespace

namespace {
// Whether some K block lies in more than one array: whole ones lie in one shard where shards are row blocks that the blocks
// (dX: the tiles) divide.
template <int BN, int BK, bool kBKc>
bool skinny_by_lane(const WeightMap &w) {
  return w.dp_mask != 0 || w.lay.rows_per_shard == 0 || w.lay.rows_per_shard % (kBKc ? BN : BK) != 0;
}

template <int BM, int BN, int BK, int kStages, bool kBKc>
hipError_t launch_skinny_as(SkinnyParams p, hipStream_t stream) {
  constexpr size_t lds = static_cast<size_t>(kSkinnyWaves) * kStages * (BM + BN) * BK * sizeof(uint16_t);
  static_assert(lds + 2 * OSDP_MAX_SHARDS * 8 <= 160 * 1024, "the rings do not fit the 160 KB of LDS");
  auto kernel = gemm_skinny_kernel<BM, BN, BK, kStages, kBKc>;
  static bool configured[kMaxDevices] = {};
  const hipError_t e = allow_lds(kernel, lds, configured);
  if (e != hipSuccess) return e;
  p.tiles_m = (p.M + BM - 1) / BM;
  p.by_lane = skinny_by_lane<BN, BK, kBKc>(p.w);
  hipLaunchKernelGGL(kernel, dim3(p.tiles_m * ((p.N + BN - 1) / BN)), dim3(kSkinnyWaves * 64), lds, stream, p);
  return hipGetLastError();
}
}  // namespace

bool skinny_takes(bool dx, int64_t T, int64_t ld_act, const ShardLayout &lay, int64_t I) {
  // (the switches that pick a kernel or a tile for the staged products keep those)
  const DebugOptions &d = debug_options();
  if (T <= 0 || T > kSkinnyMaxTokens || ld_act >= kMaxLd || I >= kMaxLd || lay.O >= kMaxLd ||
      d.gemm_generic.load(std::memory_order_relaxed) != 0 || d.tile.load(std::memory_order_relaxed) >= 0)
    return false;
  const int64_t N = dx ? I : lay.O, K = dx ? lay.O : I;
  return !(T > kSkinnyMaxWideTokens && N > kSkinnyMaxColumns && shards_are_k_blocks(lay) && forward_k_parts(T, K) == 1);
}

// Rows of a workgroup's tile.  Every workgroup streams (BM + 64) rows' worth of operands, and the launch lasts as long
// as its fullest CU: all tokens in one tile when the columns alone occupy the CUs (the weights are then read once),
// smaller tiles, which read them again from the L2, when that leaves CUs idle (128 tokens 256 -> 1024: forward 10.0 us
// in 16 tiles of 128 rows, 5.7 us in 128 tiles of 16; dX 15.5 against 5.0 us).
int skinny_rows(int64_t T, int64_t N, int cus = kCUs) {
  int best = 0;
  int64_t best_cost = 0;
  for (int bm : {16, 32, 48, 64, 128}) {
    const int64_t tiles = ((T + bm - 1) / bm) * ((N + 63) / 64);
    const int64_t cost = (tiles + cus - 1) / cus * (bm + 64);
    if (best == 0 || cost < best_cost) {
      best = bm;
      best_cost = cost;
    }
  }
  return best;
}

namespace {
SkinnyParams skinny_params(bool dx, const WeightMap &w, int64_t T, const void *act, int64_t ld_act, void *out, int64_t ld_out) {
  SkinnyParams p{};
  p.M = static_cast<int32_t>(T);
  p.N = static_cast<int32_t>(dx ? w.I : w.lay.O);
  p.K = static_cast<int32_t>(dx ? w.lay.O : w.I);
  p.A = static_cast<const uint16_t *>(act); p.lda = ld_act;
  p.C = static_cast<uint16_t *>(out); p.ldc = ld_out;
  p.w = w;
  return p;
}
}  // namespace

// As many LDS stages as fit; 128 columns to a workgroup where that still gives every CU one, else 64.
hipError_t launch_skinny(bool dx, const WeightMap &w, int64_t T, const void *act, int64_t ld_act, void *out, int64_t ld_out,
                         hipStream_t stream) {
  const SkinnyParams p = skinny_params(dx, w, T, act, ld_act, out, ld_out);
  const int bm = skinny_rows(T, p.N);
  if (dx) {
    if (bm == 16) return launch_skinny_as<16, 64, 64, 3, true>(p, stream);
    if (bm == 32) return launch_skinny_as<32, 64, 64, 3, true>(p, stream);
    if (bm <= 64) return launch_skinny_as<64, 64, 64, 2, true>(p, stream);
    return launch_skinny_as<128, 64, 32, 3, true>(p, stream);
  }
  if (p.N > 128 * (kCUs - 1) && T <= 64) {
    if (T <= 16) return launch_skinny_as<16, 128, 32, 4, false>(p, stream);
    if (T <= 32) return launch_skinny_as<32, 128, 32, 3, false>(p, stream);
    if (T <= 48) return launch_skinny_as<48, 128, 32, 3, false>(p, stream);
    return launch_skinny_as<64, 128, 32, 3, false>(p, stream);
  }
  if (bm == 16) return launch_skinny_as<16, 64, 32, 7, false>(p, stream);
  if (bm == 32) return launch_skinny_as<32, 64, 32, 6, false>(p, stream);
  if (bm == 48) return launch_skinny_as<48, 64, 32, 5, false>(p, stream);
  if (bm == 64) return launch_skinny_as<64, 64, 32, 4, false>(p, stream);
  return launch_skinny_as<128, 64, 32, 3, false>(p, stream);
}

namespace {
template <int BM, int BK, int kStages>
hipError_t launch_backward_as(SkinnyParams dx, const GemmParams &dw, hipStream_t stream) {
  constexpr size_t lds_dx = static_cast<size_t>(kSkinnyWaves) * kStages * (BM + 64) * BK * sizeof(uint16_t);
  constexpr size_t lds_dw = 4 * (W4Operand<false, 4>::kElems + W4Operand<false, 4>::kElems) * sizeof(uint16_t);
  constexpr size_t lds = lds_dx > lds_dw ? lds_dx : lds_dw;
  static_assert(lds + 3 * OSDP_MAX_SHARDS * 8 <= 160 * 1024, "the rings do not fit the 160 KB of LDS");
  auto kernel = few_token_backward_kernel<BM, BK, kStages>;
  static bool configured[kMaxDevices] = {};
  const hipError_t e = allow_lds(kernel, lds, configured);
  if (e != hipSuccess) return e;
  dx.tiles_m = (dx.M + BM - 1) / BM;
  dx.by_lane = skinny_by_lane<64, BK, true>(dx.w);
  const int n_dx = dx.tiles_m * ((dx.N + 63) / 64), tiles_m = (dw.M + 127) / 128, tiles_n = (dw.N + 127) / 128;
  hipLaunchKernelGGL(kernel, dim3(n_dx + tiles_m * tiles_n), dim3(256), lds, stream, dx, dw, n_dx, tiles_m, tiles_n);
  return hipGetLastError();
}
}  // namespace

namespace {
// Rows of a workgroup's tile of dX beside n_dw tiles of dW: for the CUs that these leave, or a quarter of all where they leave
// fewer.  us for tiles chosen for a quarter / a half / all of the CUs: 128 tokens 1024 -> 3072 12.2 / 13.5 / 13.5, 1024 -> 4096 14.2 /
// 15.2 / 15.2; 64 tokens 3072 -> 768 7.2 / 7.4 / 9.9; 128 tokens 2048 -> 2048 12.8 / 11.3 / 18.4; over 90 calls of 16 to 128 tokens
// (two launches: 1) 0.72 / 0.70 / 0.74.
int beside_rows(int64_t T, int64_t N, int64_t n_dw) { return skinny_rows(T, N, static_cast<int>(std::max<int64_t>(kCUs - n_dw, kCUs / 4))); }
}  // namespace

// us, two launches / one: 128 tokens 256 -> 1024 10.7 / 5.8, 1536 -> 1536 12.3 / 8.6, 2048 -> 2048 13.9 / 12.4, 512 -> 8192
// 24.7 / 19.5, 16 tokens 1024 -> 4096 16.5 / 11.9.  Two launches are kept for more than 64 tokens and so many in-features that tiles of dX
// with all rows make more than one round with those of dW: 128 tokens 4096 -> 1024 13.7 against 15.7 for one launch with such tiles (of 64
// rows, as one launch has now, 10.4; 8192 -> 512 13.5 and 12.5: the line could move).
bool few_token_backward_takes(const GemmProblem &dw, int64_t T) {
  const DebugOptions &d = debug_options();
  const GemmParams p = gemm_params(dw);
  int axis = -1, cut = 0;
  if (dw.epilogue != Epilogue::kBf16ShardMajor || !fast_path(p.K, 0, 0) || !fits_offsets(p) || tile_count(p.M, p.N, 128, 128) > kCUs ||
      d.deep.load(std::memory_order_relaxed) == 0 || d.small_tile.load(std::memory_order_relaxed) == 1 ||
      best_tile(p.M, p.N, p.K, 0, 1, nullptr) != 3)
    return false;
  plan_launches(p.M, p.N, p.K, 1, false, &axis, &cut);
  if (axis >= 0) return false;
  const int64_t n_dw = tile_count(p.M, p.N, 128, 128), bm = beside_rows(T, p.M, n_dw);
  return bm <= 64 || n_dw + (T + bm - 1) / bm * ((p.M + 63) / 64) <= kCUs;
}

hipError_t launch_few_token_backward(const GemmProblem &dw, const WeightMap &w, int64_t T, const void *dY, int64_t lddy, void *dX,
                                     int64_t lddx, hipStream_t stream) {
  const SkinnyParams p = skinny_params(true, w, T, dY, lddy, dX, lddx);
  const GemmParams g = gemm_params(dw);
  const int bm = beside_rows(T, p.N, tile_count(g.M, g.N, 128, 128));
  if (bm == 16) return launch_backward_as<16, 64, 3>(p, g, stream);
  if (bm == 32) return launch_backward_as<32, 64, 3>(p, g, stream);
  // (never 128 rows: their tile is the longest of the launch by far.  us as two launches / one with 128 rows / one with 64, 128
  // tokens: 3072 -> 1024 13.4 / 16.3 / 10.0, 2560 -> 1280 14.0 / 18.3 / 10.5)
  return launch_backward_as<64, 64, 2>(p, g, stream);
}

hipError_t launch_gemm(const GemmProblem &q, hipStream_t stream) {
  if (q.M < 0 || q.N < 0 || q.K < 0) return hipErrorInvalidValue;
  const GatherRequest *g = q.carry;
  const bool has_gather = g && g->rows > 0 && g->w > 0;
  if (has_gather && !q.carried) return hipErrorInvalidValue;  // the caller must learn whether the gather is still to do
  bool carry = has_gather;
  if (q.M > 0 && q.N > 0) {  // else nothing to write; K == 0 still writes the empty sum
    const hipError_t e = dispatch_gemm(q, stream, &carry);
    if (e != hipSuccess) return e;
  }
  if (q.carried) *q.carried = has_gather && !carry;
  return hipSuccess;
}

}  // namespace osdp
