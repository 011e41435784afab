// Learned projection of the kept rows (paper eq. bsca: W_v v_i and W_k k_j
// before their inner product; Def. B.3: h_v, h_k; the attention query W_Q v):
//
//   Y[r] = W x_r,   x_r the kept row r (given rows, or V[b][kept_idx[r]]),
//   W: [d_out][d] bf16, float32 sums on v_mfma_f32_32x32x16_bf16.
//
//   proj_pack_kernel : W repacked in the order the GEMM's waves read it (one
//                      1 KiB run per wave, step and k16 sub-step)
//   proj_gemm_kernel : work item = (96 kept rows, 256 output columns); the row
//                      tile arrives in a 4-slot LDS ring by direct global->LDS
//                      loads three 32-column steps ahead, rows gathered through
//                      kept_idx as they are loaded; each wave's weight fragments
//                      come straight from the packed copy into registers two
//                      steps ahead; 8 waves of 32 output columns x 96 rows
//   proj_wide_kernel : long contractions of many rows: 192 rows a work item,
//                      loads further ahead
//   proj_few_kernel  : few rows: work item = (96 kept rows, 32 output columns),
//                      the contraction split over the workgroup's waves
#include <algorithm>
#include <type_traits>

#include "skip_common.h"
#include "skip_internal.h"

namespace skip {

constexpr int kProjNT = 256;       // output columns per tile (8 waves x 32)
constexpr int kProjKS = 32;        // columns of d per step
constexpr int kProjThreads = 512;
// 96-row tiles (3072 kept rows make 32, so with 16 column tiles 512 items fill
// 256 CUs twice over)
constexpr int kProjMT = 96;
constexpr int kProjMB = kProjMT / 32;     // 32-row blocks per tile
constexpr int kProjRing = 4;
constexpr int kProjAhead = 3;
// 192-row tiles
constexpr int kWideRows = 192;
constexpr int kWideThreads = 256;
constexpr int kWideRing = 5;       // row tiles in LDS (the direct loads address 64 KiB)
constexpr int kWideAhead = 4;      // steps from the request of a row tile to its use
constexpr int kWideWD = 4;         // the same of weights
constexpr int kProjPackBlocks = 1024;

// Packed order: for column tile nt, wave w, step s, k16 sub-step kk and lane
// l, the 16 bytes W[256 nt + 32 w + l % 32][32 s + 8 (2 kk + l / 32) .. +7].
__global__ void __launch_bounds__(256)
proj_pack_kernel(const bf16_t* __restrict__ W, int d, int d_out, u32x4* __restrict__ Wp) {
  const size_t total = (size_t)d_out * d / 8;          // 16-byte units
  const int ksteps = d / kProjKS;
  for (size_t u = (size_t)blockIdx.x * blockDim.x + threadIdx.x; u < total;
       u += (size_t)gridDim.x * blockDim.x) {
    const int l = (int)(u % 64);
    size_t r = u / 64;
    const int kk = (int)(r % 2); r /= 2;
    const int s = (int)(r % ksteps); r /= ksteps;
    const int w = (int)(r % 8);
    const int nt = (int)(r / 8);
    const int j = nt * kProjNT + w * 32 + (l & 31);
    const int col = s * kProjKS + (2 * kk + (l >> 5)) * 8;
    Wp[u] = *reinterpret_cast<const u32x4*>(W + (size_t)j * d + col);
  }
}

// Row of `rows` that holds kept row r: itself, or V's row of its index.
template <bool IDX>
__device__ __forceinline__ size_t source_row(int r, const int32_t* __restrict__ kept_offsets,
                                             const int32_t* __restrict__ kept_idx, int B, int N,
                                             int M) {
  if (!IDX) return (size_t)r;
  // question of kept row r (kept_offsets ascending)
  int lo = 0, hi = B;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (clampi(kept_offsets[mid], 0, M) <= r) lo = mid;
    else hi = mid;
  }
  return (size_t)lo * N + clampi(kept_idx[r], 0, N - 1);
}

// Work items are dealt to XCDs in runs (the hardware sends workgroup id L to
// XCD L % 8): item = (L % 8) * per_xcd + L / 8, row tile fastest, so the
// items of one XCD share their weight tiles in its L2.
template <bool IDX, bool OUT_F32>
__global__ void __launch_bounds__(kProjThreads)
proj_gemm_kernel(const bf16_t* __restrict__ rows, const int32_t* __restrict__ kept_offsets,
                 const int32_t* __restrict__ kept_idx, int B, int N, int M, int d, int d_out,
                 const u32x4* __restrict__ Wp, void* __restrict__ Y, int n_items) {
  constexpr int A_ELEMS = kProjMT * kProjKS;          // 3072 (6 KiB)
  __shared__ __attribute__((aligned(1024))) bf16_t Ar[kProjRing * A_ELEMS];

  const int per_xcd = gridDim.x / 8;
  const int item = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (item >= n_items) return;
  const int MTL = (M + kProjMT - 1) / kProjMT;
  const int mt = item % MTL, nt = item / MTL;
  const int i0 = mt * kProjMT, j0 = nt * kProjNT;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ksteps = d / kProjKS;
  const int hh = lane >> 5, r32 = lane & 31;

  // this thread's 16 bytes of a row tile: row tid/4 of the tile, physical
  // chunk tid%4 holding logical chunk lc (XOR-swizzled by (row/2) % 4, so the
  // operand reads of 8 consecutive rows hit distinct banks)
  const int trow = tid >> 2;
  const int lc = (tid & 3) ^ ((trow >> 1) & 3);
  const size_t rid = source_row<IDX>(min(i0 + trow, M - 1), kept_offsets, kept_idx, B, N, M);
  const bf16_t* asrc = rows + rid * d + lc * 8;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const uint32_t ar_lds = lds_addr(Ar) + (uint32_t)(wave_s * 1024);
  // (waves past the tile's rows, 4 * kProjMT threads and up, copy nothing)
  const bool a_loader = tid < 4 * kProjMT;
  auto issue_a = [&](int s) {
    if (a_loader)
      lds_dma16(asrc + s * kProjKS, __builtin_amdgcn_readfirstlane(
                                     ar_lds + (uint32_t)((s % kProjRing) * A_ELEMS * 2)));
  };
  const u32x4* wsrc = Wp + ((size_t)(nt * 8 + wave) * ksteps) * 128 + lane;
  auto load_w = [&](int s, u32x4 (&w)[2]) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) w[kk] = wsrc[(size_t)s * 128 + kk * 64];
  };

  f32x16_t acc[kProjMB];
#pragma unroll
  for (int mb = 0; mb < kProjMB; ++mb)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[mb][v] = 0.f;

  int aoff[2][kProjMB];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk)
#pragma unroll
    for (int mb = 0; mb < kProjMB; ++mb) {
      const int row = mb * 32 + r32;
      aoff[kk][mb] = row * kProjKS + (((2 * kk + hh) ^ ((row >> 1) & 3)) << 3);
    }

  auto mma_step = [&](int s, const u32x4 (&w)[2]) {
    __builtin_amdgcn_sched_barrier(0);
    const bf16_t* At = Ar + (s % kProjRing) * A_ELEMS;
    u32x4 a[2][kProjMB];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int mb = 0; mb < kProjMB; ++mb) a[kk][mb] = *reinterpret_cast<const u32x4*>(At + aoff[kk][mb]);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int mb = 0; mb < kProjMB; ++mb) acc[mb] = mfma32_bf16(a[kk][mb], w[kk], acc[mb]);
    // half the operand reads ahead, then one MFMA per read
    constexpr int NR = 2 * kProjMB;          // operand reads (= MFMAs)
    __builtin_amdgcn_sched_group_barrier(0x100, NR / 2, 0);
#pragma unroll
    for (int i = 0; i < NR / 2; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, NR / 2, 0);
    __builtin_amdgcn_sched_barrier(0);
  };

#pragma unroll
  for (int a = 0; a < kProjAhead; ++a)
    if (a < ksteps) issue_a(a);
  u32x4 wA[2], wB[2];
  load_w(0, wA);
  load_w(min(1, ksteps - 1), wB);

  // Step s: wait for the row tile of step s (outstanding after the wait: the
  // tiles of steps s+1, s+2 while they exist, and the fragments of step s+1),
  // barrier (publishes it; the slot of step s-1 is free), load the tile of
  // step s+3, multiply step s, load the fragments of step s+2.
  auto step = [&](int s, u32x4 (&w)[2]) {
    if (s + 2 < ksteps) wait_vmcnt<4>();
    else if (s + 1 < ksteps) wait_vmcnt<3>();
    else wait_vmcnt<2>();
    barrier_nofence();
    if (s + kProjAhead < ksteps) issue_a(s + kProjAhead);
    mma_step(s, w);
    // unconditional (the last steps reload the final fragments): a
    // conditional load would make the compiler drain the queue before the
    // next use of w
    load_w(min(s + 2, ksteps - 1), w);
  };
  int s = 0;
  for (; s + 1 < ksteps; s += 2) {
    step(s, wA);
    step(s + 1, wB);
  }
  if (s < ksteps) step(s, wA);

  // Accumulator element v of block mb: row mb*32 + 8*(v/4) + 4*hh + v%4,
  // column j0 + 32*wave + r32.
  const int j = j0 + wave * 32 + r32;
#pragma unroll
  for (int mb = 0; mb < kProjMB; ++mb)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int row = i0 + mb * 32 + 8 * (v >> 2) + 4 * hh + (v & 3);
      if (row < M) {
        if (OUT_F32)
          static_cast<float*>(Y)[(size_t)row * d_out + j] = acc[mb][v];
        else
          static_cast<bf16_t*>(Y)[(size_t)row * d_out + j] = (bf16_t)f32_to_bf16(acc[mb][v]);
      }
    }
}

// Many rows of wide matrices (proj_wide_tiles): 192 rows x 256 columns a workgroup,
// four waves of 64 columns.  Beside the matrix cores the bytes a CU draws from
// the L2 and reads from LDS bound the GEMM: 28 KiB of rows and weights per
// 32-column step here, for twice the products of the tile above with its 22 KiB,
// and every wave reads the whole row tile.  Back-to-back calls with packed
// weights of 4096 x 4096: 3072 rows 101 -> 93 us, 12288 rows 401 -> 370.  Items as
// above.
//
// Few waves cover the latencies, so the loads run far ahead: row tiles are
// requested kWideAhead steps before their use and published one step early, so
// that the first operands of a step are read during the step before; weights
// are requested kWideWD steps ahead, each k16 sub-step's as soon as its
// products have read the registers (a wave waits for its loads in the order it
// issued them, and the compiler counts these but not the direct loads: its
// counted waits then only reach loads that are steps old).
template <bool IDX, bool OUT_F32>
__global__ void __launch_bounds__(kWideThreads, 1)
proj_wide_kernel(const bf16_t* __restrict__ rows, const int32_t* __restrict__ kept_offsets,
                 const int32_t* __restrict__ kept_idx, int B, int N, int M, int d, int d_out,
                 const u32x4* __restrict__ Wp, void* __restrict__ Y, int n_items) {
  constexpr int MB = kWideRows / 32, NB = 8 / (kWideThreads / 64);
  constexpr int WD = kWideWD, AH = kWideAhead;
  constexpr int MT = kWideRows;
  constexpr int A_ELEMS = MT * kProjKS;
  constexpr int WCH = 16 * MB * NB;                   // 16-byte chunks of a tile per wave
  constexpr int NI = (WCH + 63) / 64;                 // direct loads they take
  __shared__ __attribute__((aligned(1024))) bf16_t Ar[kWideRing * A_ELEMS];
  static_assert(sizeof(Ar) <= 65536, "direct loads address 64 KiB of LDS");

  const int per_xcd = gridDim.x / 8;
  const int item = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (item >= n_items) return;
  const int MTL = (M + MT - 1) / MT;
  const int mt = item % MTL, nt = item / MTL;
  const int i0 = mt * MT, j0 = nt * kProjNT;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ksteps = d / kProjKS;
  const int hh = lane >> 5, r32 = lane & 31;

  // the lane's 16-byte chunks of a row tile: chunk g is row g / 4, physical
  // chunk g % 4 holding logical chunk (g % 4) ^ (row / 2) % 4 (the operand
  // reads of 8 consecutive rows hit distinct banks)
  const bf16_t* asrc[NI];
#pragma unroll
  for (int q = 0; q < NI; ++q) {
    const int g = wave * WCH + min(q * 64 + lane, WCH - 1);
    const int trow = g >> 2;
    const int lc = (g & 3) ^ ((trow >> 1) & 3);
    const int r = min(i0 + trow, M - 1);
    const size_t rid = source_row<IDX>(r, kept_offsets, kept_idx, B, N, M);
    asrc[q] = rows + rid * d + lc * 8;
  }
  const uint32_t ar_lds = lds_addr(Ar) + (uint32_t)(wave * WCH * 16);
  auto issue_a = [&](int s) {
#pragma unroll
    for (int q = 0; q < NI; ++q)
      if (q * 64 + lane < WCH)
        lds_dma16(asrc[q] + s * kProjKS,
                  __builtin_amdgcn_readfirstlane(
                      ar_lds + ((uint32_t)s % kWideRing) * (A_ELEMS * 2) + q * 1024));
  };
  // weight fragments of this wave's 32-column blocks, [kk][nb] per step
  const u32x4* wsrc = Wp + ((size_t)(nt * 8 + wave * NB) * ksteps) * 128 + lane;
  const size_t wblk = (size_t)ksteps * 128;           // from one 32-column block to the next
  auto load_w = [&](int s, int kk, u32x4 (&w)[NB]) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) w[nb] = wsrc[nb * wblk + (size_t)s * 128 + kk * 64];
  };

  f32x16_t acc[NB][MB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[nb][mb][v] = 0.f;

  // operand offset of row block 0 (the swizzle repeats every 8 rows)
  int aoff[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk)
    aoff[kk] = r32 * kProjKS + (((2 * kk + hh) ^ ((r32 >> 1) & 3)) << 3);
  auto read_a = [&](int s, int kk, u32x4 (&a)[MB]) {
    const bf16_t* At = Ar + ((uint32_t)s % kWideRing) * A_ELEMS + aoff[kk];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      a[mb] = *reinterpret_cast<const u32x4*>(At + mb * 32 * kProjKS);
  };
  // products of one sub-step, one operand read of the next beside each of the
  // first of them
  auto multiply = [&](const u32x4 (&a)[MB], const u32x4 (&w)[NB]) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[nb][mb] = mfma32_bf16(a[mb], w[nb], acc[nb][mb]);
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, MB * NB - MB, 0);
    __builtin_amdgcn_sched_barrier(0);
  };

#pragma unroll
  for (int a = 0; a < AH; ++a)
    if (a < ksteps) issue_a(a);
  u32x4 w[WD][2][NB];
#pragma unroll
  for (int t = 0; t < WD; ++t)
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) load_w(min(t, ksteps - 1), kk, w[t][kk]);
  wait_vmcnt<0>();
  barrier_nofence();
  u32x4 f0[MB], f1[MB];
  read_a(0, 0, f0);

  // Step s: wait for this wave's part of the row tile of step s+1 (issued
  // after it: the weights of AH - 1 steps and, while they exist, the tiles of
  // steps s+2 .. s+AH-1), barrier (publishes that tile; the slot of step s-1
  // is free), request the tile of step s+AH, multiply step s and read the
  // first operands of step s+1 (past the last step: stale values that nothing
  // uses).  The tail steps (after the last whole group of WD; every tile is
  // requested by then) load nothing and wait for all.
  static_assert(AH >= WD && AH < kWideRing, "tail steps request no tile; a slot is free");
  constexpr int WQ = (AH - 1) * 2 * NB;
  auto step = [&](int s, u32x4 (&ws)[2][NB], auto tail) {
    constexpr bool TAIL = decltype(tail)::value;
    if (TAIL) wait_vmcnt<0>();
    else if (s + AH <= ksteps) wait_vmcnt<WQ + (AH - 2) * NI>();
    else wait_vmcnt<WQ>();
    barrier_nofence();
    if (!TAIL && s + AH < ksteps) issue_a(s + AH);
    __builtin_amdgcn_sched_barrier(0);
    read_a(s, 1, f1);
    multiply(f0, ws[0]);
    // unconditional (the last steps reload the final fragments): a
    // conditional load would make the compiler drain the queue before the
    // next use of w
    if (!TAIL) load_w(min(s + WD, ksteps - 1), 0, ws[0]);
    __builtin_amdgcn_sched_barrier(0);
    read_a(s + 1, 0, f0);
    multiply(f1, ws[1]);
    if (!TAIL) load_w(min(s + WD, ksteps - 1), 1, ws[1]);
    __builtin_amdgcn_sched_barrier(0);
  };
  int s = 0;
  for (; s + WD <= ksteps; s += WD) {
#pragma unroll
    for (int t = 0; t < WD; ++t) step(s + t, w[t], std::false_type{});
  }
#pragma unroll
  for (int t = 0; t < WD - 1; ++t)
    if (s + t < ksteps) step(s + t, w[t], std::true_type{});

  // Accumulator element v of block (nb, mb): row mb*32 + 8*(v/4) + 4*hh + v%4,
  // column j0 + 32*(wave*NB + nb) + r32.
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int j = j0 + (wave * NB + nb) * 32 + r32;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = i0 + mb * 32 + 8 * (v >> 2) + 4 * hh + (v & 3);
        if (row < M) {
          if (OUT_F32)
            static_cast<float*>(Y)[(size_t)row * d_out + j] = acc[nb][mb][v];
          else
            static_cast<bf16_t*>(Y)[(size_t)row * d_out + j] = (bf16_t)f32_to_bf16(acc[nb][mb][v]);
        }
      }
  }
}

// Few rows: the tiles above leave most CUs without work (160 keys x 4096
// columns make 32 of them), so a workgroup takes 96 rows x 32 columns and its
// eight waves split the contraction; their partial sums meet in LDS, added in
// wave order.  Operands come straight from memory into registers, four k16
// groups in flight while four are multiplied: bound by the lines a CU draws
// from the L2 (96 + 32 rows of d; a load touches 32 of them).  PACKED: W is
// the packed copy; otherwise W itself, which saves the packing pass (160 rows
// of 4096 x 4096, back to back: tiles after packing 60 us, this 36).
constexpr int kFewRows = 96;
constexpr int kFewMB = kFewRows / 32;
constexpr int kFewWaves = 8;
constexpr int kFewU = 4;           // k16 groups per batch of loads

template <bool PACKED, bool IDX, bool OUT_F32>
__global__ void __launch_bounds__(64 * kFewWaves, 2)
proj_few_kernel(const bf16_t* __restrict__ rows, const int32_t* __restrict__ kept_offsets,
                const int32_t* __restrict__ kept_idx, int B, int N, int M, int d, int d_out,
                const bf16_t* __restrict__ W, void* __restrict__ Y, int n_items) {
  __shared__ float red[kFewWaves][16][64];
  // (column tiles dealt to the XCDs in runs, row tile fastest)
  const int per_xcd = gridDim.x / 8;
  const int item = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (item >= n_items) return;
  const int MTL = (M + kFewRows - 1) / kFewRows;
  const int mt = item % MTL, ct = item / MTL;
  const int i0 = mt * kFewRows, j0 = ct * 32;
  const int lane = threadIdx.x & 63, hh = lane >> 5, r32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int G = d / 16;
  const int g0 = w * G / kFewWaves, g1 = (w + 1) * G / kFewWaves;   // the wave's groups
  const int gl = max(g1 - 1, 0);

  const bf16_t* ap[kFewMB];
#pragma unroll
  for (int mb = 0; mb < kFewMB; ++mb)
    ap[mb] = rows + source_row<IDX>(min(i0 + mb * 32 + r32, M - 1), kept_offsets, kept_idx, B,
                                    N, M) * d + hh * 8;
  // group g of W: 16 columns from its row, or one 1 KiB run of the packed copy
  const bf16_t* wp = PACKED ? W + ((size_t)ct * G * 64 + lane) * 8
                            : W + (size_t)(j0 + r32) * d + hh * 8;
  constexpr int WS = PACKED ? 512 : 16;                // elements from group to group
  struct Batch {
    u32x4 a[kFewU][kFewMB], w[kFewU];
  };
  // (a row's four groups, one cache line, back to back: with eight waves in
  // flight the L1 would not hold the lines until a later load)
  auto load = [&](Batch& x, int g) {
    size_t gg[kFewU];                                  // groups past the wave's are not multiplied
#pragma unroll
    for (int u = 0; u < kFewU; ++u) gg[u] = (size_t)min(g + u, gl);
#pragma unroll
    for (int u = 0; u < kFewU; ++u) x.w[u] = *reinterpret_cast<const u32x4*>(wp + gg[u] * WS);
#pragma unroll
    for (int mb = 0; mb < kFewMB; ++mb)
#pragma unroll
      for (int u = 0; u < kFewU; ++u)
        x.a[u][mb] = *reinterpret_cast<const u32x4*>(ap[mb] + gg[u] * 16);
  };
  f32x16_t acc[kFewMB];
#pragma unroll
  for (int mb = 0; mb < kFewMB; ++mb)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[mb][v] = 0.f;
  auto multiply = [&](const Batch& x, int g) {
#pragma unroll
    for (int u = 0; u < kFewU; ++u)
      if (g + u < g1)
#pragma unroll
        for (int mb = 0; mb < kFewMB; ++mb) acc[mb] = mfma32_bf16(x.a[u][mb], x.w[u], acc[mb]);
  };
  Batch x0, x1;
  load(x0, g0);
  for (int g = g0; g < g1; g += 2 * kFewU) {
    load(x1, g + kFewU);
    multiply(x0, g);
    load(x0, g + 2 * kFewU);
    multiply(x1, g + kFewU);
  }
  // Accumulator element v of block mb: row mb*32 + 8*(v/4) + 4*hh + v%4,
  // column j0 + r32; wave w adds elements 2 w and 2 w + 1.
#pragma unroll
  for (int mb = 0; mb < kFewMB; ++mb) {
    if (mb > 0) __syncthreads();                       // the block before is read
#pragma unroll
    for (int v = 0; v < 16; ++v) red[w][v][lane] = acc[mb][v];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int v = 2 * w + e;
      float sum = red[0][v][lane];
#pragma unroll
      for (int u = 1; u < kFewWaves; ++u) sum += red[u][v][lane];
      const int row = i0 + mb * 32 + 8 * (v >> 2) + 4 * hh + (v & 3);
      if (row < M) {
        if (OUT_F32)
          static_cast<float*>(Y)[(size_t)row * d_out + j0 + r32] = sum;
        else
          static_cast<bf16_t*>(Y)[(size_t)row * d_out + j0 + r32] = (bf16_t)f32_to_bf16(sum);
      }
    }
  }
}

size_t proj_scratch_bytes(int d, int d_out) {
  return ((size_t)d_out * d * sizeof(bf16_t) + 255) & ~(size_t)255;
}

hipError_t launch_proj_pack(int d, int d_out, const void* W, void* packed, hipStream_t s) {
  hipLaunchKernelGGL(proj_pack_kernel, dim3(kProjPackBlocks), dim3(256), 0, s,
                     (const bf16_t*)W, d, d_out, static_cast<u32x4*>(packed));
  return hipGetLastError();
}

constexpr long long kProjCUs = 256;

// At most one 96 x 32 item per CU, and a contraction long enough to split: its
// eight parts and their sum cost about 11.7 us of back-to-back calls whatever d
// is (one row 5.4, 40 rows 8.0), the 96-row tiles grow with d.  Packed weights,
// 160 rows x 1024 columns, this form against tiles: d = 512 11.8 us against 9.0,
// 768 11.8 against 11.4, 1024 11.8 against 13.9, 4096 0.66 of the tiles; 40 rows:
// d = 512 8.0 against 8.6; one row: d = 256 5.3 against 5.8.  At two rounds of
// items the tiles win (d = 4096: 1.2 times), and so they do on few columns of
// many rows (3072 rows x 256: 1.04 to 1.12).  The same line with and without packed
// weights: both calls give the same bits.
static bool few_fit(int M, int d_out) {
  return M <= 24 * kFewRows &&
         (long long)((M + kFewRows - 1) / kFewRows) * (d_out / 32) <= kProjCUs;
}
bool proj_few_rows(int M, int d, int d_out) {
  return d >= (M < 98 ? 240 + 8 * M : 1024) && few_fit(M, d_out);
}

// 192-row tiles, one per CU and round, where whole rounds cost at most an
// eighth more row blocks than 96-row tiles, two per CU (6680 rows of 2048 x
// 2048, 280 tiles in two rounds: 88 us against 74), and the contraction is long
// enough for loads that run four steps ahead: 192- over 96-row tiles, over the
// sizes of whole rounds, 0.85-0.97 from d = 3072 on, 0.95-1.01 at 2048, 0.98-1.06
// at 1536, 1.02-1.14 at 1024 and up to 2.1 at 64.
bool proj_wide_tiles(int M, int d, int d_out) {
  if (d < 2048) return false;
  const long long nt = d_out / kProjNT;
  const long long n96 = (M + 95) / 96 * nt, n192 = (M + 191) / 192 * nt;
  const long long rounds = (n192 + kProjCUs - 1) / kProjCUs;
  return rounds * kProjCUs * 2 * 8 <= n96 * 9;
}

template <bool PACKED>
static hipError_t launch_proj_few(const skip_problem_t& p, const bf16_t* rows,
                                  const int32_t* kept_offsets, const int32_t* kept_idx,
                                  const bf16_t* W, int d_out, void* Y, int out_f32,
                                  hipStream_t s) {
  const int M = p.total_kept;
  const int n_items = ((M + kFewRows - 1) / kFewRows) * (d_out / 32);
  auto go = [&](auto idx, auto f32) -> hipError_t {
    hipLaunchKernelGGL((proj_few_kernel<PACKED, decltype(idx)::value, decltype(f32)::value>),
                       dim3((n_items + 7) / 8 * 8), dim3(64 * kFewWaves), 0, s, rows,
                       kept_offsets, kept_idx, p.B, p.N, M, p.d, d_out, W, Y, n_items);
    return hipGetLastError();
  };
  using T = std::true_type;
  using F = std::false_type;
  if (kept_idx) return out_f32 ? go(T{}, T{}) : go(T{}, F{});
  return out_f32 ? go(F{}, T{}) : go(F{}, F{});
}

hipError_t launch_proj_gemm(const skip_problem_t& p, const void* rows, const int32_t* kept_offsets,
                            const int32_t* kept_idx, const void* packed, int d_out, void* Y,
                            int out_f32, hipStream_t s) {
  const int M = p.total_kept;
  if (M <= 0) return hipSuccess;
  const bf16_t* R = static_cast<const bf16_t*>(rows);
  if (proj_few_rows(M, p.d, d_out))
    return launch_proj_few<true>(p, R, kept_offsets, kept_idx, static_cast<const bf16_t*>(packed),
                                 d_out, Y, out_f32, s);
  const u32x4* Wc = static_cast<const u32x4*>(packed);
  const bool wide = proj_wide_tiles(M, p.d, d_out);
  const int rt = wide ? kWideRows : kProjMT;
  const int n_items = ((M + rt - 1) / rt) * (d_out / kProjNT);
  auto go = [&](auto idx, auto f32) -> hipError_t {
    constexpr bool IDX = decltype(idx)::value, F32 = decltype(f32)::value;
    const dim3 grid((n_items + 7) / 8 * 8);
    if (wide)
      hipLaunchKernelGGL((proj_wide_kernel<IDX, F32>), grid, dim3(kWideThreads), 0, s, R,
                         kept_offsets, kept_idx, p.B, p.N, M, p.d, d_out, Wc, Y, n_items);
    else
      hipLaunchKernelGGL((proj_gemm_kernel<IDX, F32>), grid, dim3(kProjThreads), 0, s, R,
                         kept_offsets, kept_idx, p.B, p.N, M, p.d, d_out, Wc, Y, n_items);
    return hipGetLastError();
  };
  using T = std::true_type;
  using F = std::false_type;
  if (kept_idx) return out_f32 ? go(T{}, T{}) : go(T{}, F{});
  return out_f32 ? go(F{}, T{}) : go(F{}, F{});
}

// Passage keys as bf16 rows for the projection: k~ = the bf16 rounding
// (through float, nearest even at both steps) of the pooled double key or of
// the caller's float key.
__global__ void __launch_bounds__(256)
keys_bf16_kernel(const double* __restrict__ kbar, const float* __restrict__ given, size_t n,
                 bf16_t* __restrict__ out) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x) {
    const float f = given ? given[i] : (float)kbar[i];
    out[i] = __builtin_bit_cast(bf16_t, (__bf16)f);
  }
}

hipError_t launch_keys_bf16(const double* kbar, const float* given, size_t n, void* out,
                            hipStream_t s) {
  if (n == 0) return hipSuccess;
  const size_t blocks = std::min<size_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(keys_bf16_kernel, dim3((unsigned)blocks), dim3(256), 0, s, kbar, given, n,
                     static_cast<bf16_t*>(out));
  return hipGetLastError();
}

// keys: passage keys, which no packed call has to agree with, take the split
// contraction at every d: W as it is and one launch instead of two (160 rows of
// 256 x 1024: calls one after another 15.4 us against 17.7, bound by their
// launches; captured 13.6 against 9.0).
hipError_t launch_project(const skip_problem_t& p, const void* rows, const int32_t* kept_offsets,
                          const int32_t* kept_idx, const void* W, int d_out, void* Y,
                          int out_f32, void* scratch, hipStream_t s, bool keys) {
  if (p.total_kept <= 0) return hipSuccess;
  if (keys ? few_fit(p.total_kept, d_out) : proj_few_rows(p.total_kept, p.d, d_out))
    return launch_proj_few<false>(p, static_cast<const bf16_t*>(rows), kept_offsets, kept_idx,
                                  static_cast<const bf16_t*>(W), d_out, Y, out_f32, s);
  hipError_t e = launch_proj_pack(p.d, d_out, W, scratch, s);
  if (e != hipSuccess) return e;
  return launch_proj_gemm(p, rows, kept_offsets, kept_idx, scratch, d_out, Y, out_f32, s);
}

}  // namespace skip
