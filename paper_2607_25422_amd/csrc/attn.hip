// Sparse cross-attention restricted to the bipartite graph (paper App. B.3,
// Def. B.3 attention rule; Alg. 1, fuse step).
//
// For kept row i of question b and head h, the logits run over every token of
// every passage adjacent to i (one 64-bit neighbour mask per row):
//   e_m = sm_scale * <Qh[i,h], Kh[m,h]>,  O = softmax(e) . Vh,  LSE = log sum exp e.
//
// bf16 path (MFMA): passage-major, only the graph's edges are computed (the
// kernel comment below); a device-built work list orders the items by cost.
//
// fp32 inputs and small bf16 problems: 16 rows per workgroup, token blocks
// split over its waves (at that kernel).
#include <algorithm>

#include "skip_common.h"
#include "skip_internal.h"
#include "skip_plan.h"

namespace skip {

typedef short s16x4_t __attribute__((ext_vector_type(4)));
template <int N>
struct IntC {                     // a compile-time count passed to a generic lambda
  static constexpr int value = N;
};
// f(IntC<0>), .., f(IntC<N-1>)
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(IntC<I>{});
    static_for<N, I + 1>(f);
  }
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Value of lane l ^ 32 (v_permlane32_swap: the two half-waves trade places).
__device__ __forceinline__ float swap_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x),
                                                  false, false);
  return __uint_as_float(__lane_id() < 32 ? r[1] : r[0]);
}

// Value of lane l ^ 16 (v_permlane16_swap: odd and even 16-lane rows trade).
__device__ __forceinline__ float swap16(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x),
                                                  false, false);
  return __uint_as_float((__lane_id() & 16) ? r[0] : r[1]);
}

// Transposing LDS read (ds_read_b64_tr_b16) at byte address lds + OFF: in
// each group of 16 lanes, lane j receives element j & 3 of the 8-byte pieces
// addressed by lanes (j >> 2) + 4e, e = 0..3.  Issued through inline
// assembly so that the constant offset sits in the instruction (the builtin
// takes a full address per read); the compiler does not track its
// completion, so the results pass through lds_wait_all before any use.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
template <int OFF>
__device__ __forceinline__ u32x2 ds_read_tr16_at(uint32_t lds) {
  static_assert(OFF >= 0 && OFF < 65536 && OFF % 8 == 0, "DS offset field");
  u32x2 r;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(lds), "i"(OFF));
  return r;
}

// Waits for every outstanding LDS read of the wave; the registers passed
// through it are the values after the wait (a true dependency for the
// compiler, so no use of them is scheduled above it).
template <int N>
__device__ __forceinline__ void lds_wait_all(u32x2 (&v)[N]) {
  static_assert(N == 16 || N == 8, "operand count");
  if constexpr (N == 16) {
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]),
                   "+v"(v[6]), "+v"(v[7]), "+v"(v[8]), "+v"(v[9]), "+v"(v[10]), "+v"(v[11]),
                   "+v"(v[12]), "+v"(v[13]), "+v"(v[14]), "+v"(v[15])
                 :
                 : "memory");
  } else {
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]),
                   "+v"(v[6]), "+v"(v[7])
                 :
                 : "memory");
  }
}

// ---------------------------------------------------------------------------
// bf16 path, passage-major.  Attention is computed only on the graph's edges:
// for each passage j, only the kept rows adjacent to j (Def. B.3: a row's
// softmax runs over the tokens of its neighbour passages, and no other pair
// is touched), so the work grows with the number of edges and a passage
// adjacent to none of an item's rows is never read.
//
// Work item = (question b, head h, chunk of <= kSpRows kept rows).  The item
// walks the passages with at least one adjacent row in the chunk, in
// ascending order, 32 tokens at a time.  K and V tiles of head h stream
// through two LDS rings of three tiles, one barrier per tile; two loader
// waves (one for K, one for V) keep four more tiles in flight in registers
// and write each into the ring when its slot frees.  For each passage the
// adjacent rows (a 192-bit row mask per passage) form blocks of 16 in row
// order; compute wave w takes blocks w and w + 6.  Per tile and block:
//   S^T (32 tokens x 16 rows) = K_tile . Q^T        v_mfma_f32_16x16x32_bf16
//   online softmax in fp32 (base 2); each weight p split into bf16 hi + lo
//   (hi = p truncated, lo = the rest rounded), so the PV product sees p to
//   about 2^-16 relative and the result does not depend on the output type,
//   O^T (d_h x 16 rows)     += V_tile^T . (P_hi + P_lo)^T
// Computing the transposed products keeps each query row in one lane column
// (row statistics need an exchange among the four lanes of that column) and
// makes the S^T accumulator the P^T operand; V^T comes from transposing LDS
// reads in the token order of that layout.  The queries of a block's rows
// sit in registers, loaded at the previous busy passage's last tile.  After
// a passage's last tile each block's partial (O, max, sum) is merged into
// the item's accumulators, fp32 in LDS for every row of the chunk, by
// log-sum-exp rescaling; one passage's blocks hold disjoint rows and
// passages merge in ascending order (a barrier at least between two), so the
// result is deterministic.  The item ends by writing O = acc / sum and LSE
// for every row of the chunk (0 and -inf for a row without neighbours).
constexpr int kSpTile = 32;               // tokens per K/V tile
constexpr int kSpStages = 3;              // K (and V) tiles resident in LDS
constexpr int kSpRegTiles = 4;            // K (and V) tiles in flight in loader registers
constexpr int kSpCompute = kSpRows / 32;  // compute waves (two 16-row blocks each)
constexpr int kSpWaves = kSpCompute + 2;  // + a K loader and a V loader
constexpr int kSpThreads = 64 * kSpWaves;
constexpr float kLazy = 8.f;              // log2 slack of the softmax reference maximum
static_assert(kSpRows <= 3 * 64, "row masks have three 64-bit words");

// Position of the n-th (from 0) set bit of x; n < popcount(x).
__device__ __forceinline__ int nth_bit64(uint64_t x, int n) {
  int pos = 0;
#pragma unroll
  for (int w = 32; w >= 1; w >>= 1) {
    const int c = __popcll(x & ((1ull << w) - 1ull));
    if (n >= c) {
      n -= c;
      x >>= w;
      pos += w;
    }
  }
  return pos;
}

// Work item record: {question, first kept row (global), first passage,
// head | rows << 8 | passages << 16}; question -1: no item.
template <int D>
__global__ void __launch_bounds__(kSpThreads)
attn_sparse_kernel(const bf16_t* __restrict__ qbase, const int32_t* __restrict__ kept_idx,
                   int N, int qstride, const bf16_t* __restrict__ Kh,
                   const bf16_t* __restrict__ Vh, const int32_t* __restrict__ passage_offsets,
                   const uint64_t* __restrict__ rowmask, const int4* __restrict__ items, int H,
                   int total_tokens, float scale_log2, void* __restrict__ O, int o_f32,
                   float* __restrict__ lse) {
  constexpr int NCH = D / 8;               // 16-byte chunks per token row
  constexpr int NC4 = D / 4;               // 4-float chunks per accumulator row
  constexpr int KB = D / 32;               // k-blocks of QK^T (32 features each)
  constexpr int DB = D / 16;               // 16-wide feature blocks of O
  // Tiles are token-major with padded rows: K rows of D + 8 elements put the
  // sixteen tokens of one S^T operand read on distinct banks, V rows of D +
  // 16 the sixteen tokens of one transposing read (two 8-byte pieces each);
  // every operand read is then a register base plus an immediate offset.
  constexpr int SK = D + 8, SV = D + 16;   // row strides (elements)
  constexpr int TK = kSpTile * SK, TV = kSpTile * SV;
  constexpr int NI = kSpTile * NCH / 64;   // 16-byte loads per lane per K (or V) tile
  __shared__ __attribute__((aligned(1024))) bf16_t Kbuf[kSpStages * TK];
  __shared__ __attribute__((aligned(1024))) bf16_t Vbuf[kSpStages * TV];
  __shared__ __attribute__((aligned(16))) float Oacc[kSpRows * D];
  __shared__ float m_acc[kSpRows], l_acc[kSpRows];
  __shared__ uint64_t rmask[3][kSpMaxP];   // rows 64w..64w+63 adjacent to each passage
  __shared__ int p_ts[kSpMaxP], p_te[kSpMaxP], p_cnt[kSpMaxP];
  __shared__ int32_t qsrc[kSpRows];        // visual-token index of each row (fused route)

  const int4 item = items[blockIdx.x];
  const int b = item.x;
  if (b < 0) return;
  const int row0 = item.y, p0 = item.z;
  const int h = item.w & 0xff;
  const int nrows = (item.w >> 8) & 0xff;
  const int P = (item.w >> 16) & 0xff;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform per wave

  // accumulators, passage ranges, row sources, row masks per passage
  const uint64_t pm = (P >= 64) ? ~0ull : ((1ull << P) - 1ull);
  const uint64_t mk = (tid < nrows) ? (rowmask[row0 + tid] & pm) : 0ull;
  const int src = (kept_idx && tid < nrows) ? kept_idx[row0 + tid] : 0;
  int ts = 0, te = 0;
  if (tid < P) range_of(passage_offsets, p0 + tid, total_tokens, ts, te);
  for (int i = tid; i < nrows * NC4; i += kSpThreads)
    reinterpret_cast<float4*>(Oacc)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  if (tid < nrows) {
    m_acc[tid] = -INFINITY;
    l_acc[tid] = 0.f;
    qsrc[tid] = clampi(src, 0, N - 1);
  }
  if (tid < P) {
    p_ts[tid] = ts;
    p_te[tid] = te;
  }
  if (wave < 3) {
    for (int j = 0; j < P; ++j) {
      const uint64_t bal = __ballot((mk >> j) & 1ull);
      if (lane == 0) rmask[wave][j] = bal;
    }
  }
  __syncthreads();
  if (tid < P) p_cnt[tid] = __popcll(rmask[0][tid]) + __popcll(rmask[1][tid]) +
                            __popcll(rmask[2][tid]);
  __syncthreads();
  // passages with at least one adjacent row of the chunk (and some tokens)
  const bool touched = lane < P && p_cnt[lane] > 0 && p_te[lane] > p_ts[lane];
  const uint64_t U = uniform64(__ballot(touched));

  // Tile cursor over (touched passage, 32-token block).
  struct Cursor {
    uint64_t rem;
    int j, t, ts, te;
  };
  auto advance = [&](Cursor& cu) -> bool {
    if (cu.j >= 0 && cu.t + kSpTile < cu.te) {
      cu.t += kSpTile;
      return true;
    }
    if (!cu.rem) return false;
    const int j = __builtin_ctzll(cu.rem);
    cu.rem &= cu.rem - 1ull;
    cu.j = j;
    cu.ts = __builtin_amdgcn_readfirstlane(p_ts[j]);
    cu.te = __builtin_amdgcn_readfirstlane(p_te[j]);
    cu.t = cu.ts;
    return true;
  };

  // One barrier per tile publishes it; the loads run two tiles ahead.
  int n_tiles = 0;
  for (uint64_t r = U; r; r &= r - 1ull) {
    const int j = __builtin_ctzll(r);
    n_tiles += (__builtin_amdgcn_readfirstlane(p_te[j]) - __builtin_amdgcn_readfirstlane(p_ts[j]) +
                kSpTile - 1) / kSpTile;
  }

  if (wave >= kSpCompute) {
    // ---- loader waves: the first streams K, the second V --------------------
    // (their LDS writes must land before each barrier; issuing ahead of the
    // compute waves' operand reads keeps them from queueing behind those)
    __builtin_amdgcn_s_setprio(3);
    const bool isV = wave == kSpCompute + 1;
    const bf16_t* gsrc = isV ? Vh : Kh;
    bf16_t* buf = isV ? Vbuf : Kbuf;
    const int S = isV ? SV : SK, T = isV ? TV : TK;
    // load q of a tile: lane l takes 16-byte chunk (q*64 + l) % NCH of token
    // row (q*64 + l) / NCH; byte offsets from the tile's first token
    uint32_t voff[NI];
#pragma unroll
    for (int q = 0; q < NI; ++q) {
      const int o = q * 64 + lane;
      voff[q] = (uint32_t)(((o / NCH) * H * D + (o % NCH) * 8) * 2);
    }
    const int lds_lane = (lane / NCH) * S + (lane % NCH) * 8;
    const bf16_t* hsrc = gsrc + (size_t)h * D;
    // Tiles travel through registers: global loads run kSpRegTiles tiles
    // ahead of the LDS ring (which holds the tile being consumed and the next
    // one), so the loads keep streaming while the compute waves merge or
    // start a passage.  Slot n % kSpRegTiles holds tile n.
    u32x4 rg[kSpRegTiles][NI];
    auto gload = [&](auto slot, int t, int te_) {
      const bf16_t* tbase = hsrc + (size_t)t * H * D;
      const int over_base = t - (te_ - 1);
#pragma unroll
      for (int q = 0; q < NI; ++q) {
        // rows past the passage's end read its last token (finite values,
        // masked in the softmax)
        const int row = (q * 64 + lane) / NCH;
        const uint32_t o = voff[q] - (uint32_t)(max(over_base + row, 0) * H * D * 2);
        rg[decltype(slot)::value][q] = *reinterpret_cast<const u32x4*>(
            reinterpret_cast<const char*>(tbase) + o);
      }
      // tiles issue in order (the wait counts assume it)
      asm volatile("" ::: "memory");
    };
    auto swrite = [&](auto slot, int n) {
      bf16_t* dst = buf + (n % kSpStages) * T + lds_lane;
#pragma unroll
      for (int q = 0; q < NI; ++q)
        *reinterpret_cast<u32x4*>(dst + q * (64 / NCH) * S) = rg[decltype(slot)::value][q];
    };
    // Every step issues one tile's loads, unconditionally (past the last
    // tile the cursor stays put and the last tile is read again), so that
    // the compiler's wait counts before each register slot's LDS write are
    // exact: the slot's loads are the oldest of the four in flight.
    Cursor ci{U, -1, 0, 0, 0};
    auto issue = [&](auto slot) {
      advance(ci);
      gload(slot, ci.t, ci.te);
    };
    static_assert(kSpRegTiles == 4 && kSpStages == 3, "slot arithmetic below");
    if (n_tiles > 0) {
      // prologue: loads of tiles 0 .. 3, tiles 0 and 1 into LDS, loads of
      // tiles 4 and 5
      issue(IntC<0>{});
      issue(IntC<1>{});
      issue(IntC<2>{});
      issue(IntC<3>{});
      swrite(IntC<0>{}, 0);
      issue(IntC<0>{});
      swrite(IntC<1>{}, 1);            // (a repeat of tile 0 if there is one tile)
      issue(IntC<1>{});
      // step i: after its barrier the LDS slot of tile i-1, which every wave
      // finished in step i-1, is free; tile i+2 goes there from register slot
      // (i+2) % 4, which then takes tile i+6
      auto step = [&](auto u, int i) {
        constexpr int sl = (decltype(u)::value + 2) % kSpRegTiles;
        if (i < n_tiles) {
          barrier_lds();                                         // tile i is published
          // (past the last tile a repeat, into a slot that is not read again)
          swrite(IntC<sl>{}, i + 2);
        }
        issue(IntC<sl>{});
      };
      // whole groups of four steps, one exit: the loads of every step are
      // unconditional, so each slot's wait count is the same on every path
      for (int i = 0; i < n_tiles; i += kSpRegTiles) {
        step(IntC<0>{}, i);
        step(IntC<1>{}, i + 1);
        step(IntC<2>{}, i + 2);
        step(IntC<3>{}, i + 3);
      }
    }
  } else {
    // ---- compute waves ------------------------------------------------------
    // Lane layout of every product (16 x 16 blocks): r16 = lane & 15 is the
    // lane's row within a block (the column of S^T, P^T and O^T); g = lane
    // >> 4 picks tokens 4g..4g+3 of each 16-token half of S^T, the k-slice
    // 8g..8g+7 of P^T (those same eight tokens, halves in order) and
    // features 16db + 4g..4g+3 of O^T.
    const int g = lane >> 4;
    const int r16 = lane & 15;
    // K (A of S^T): token r16 (+16), features 32kb + 8g .. +7
    const int koff = r16 * SK + 8 * g;
    // V^T (A of O^T) by transposing reads: lane (e = r16 >> 2, q = r16 & 3)
    // addresses token 4g + e (+16), features 16db + 4q .. +3; lane r16 then
    // holds feature 16db + r16 of tokens 4g .. 4g+3
    const uint32_t vlds = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)(
        Vbuf + (4 * g + (r16 >> 2)) * SV + 4 * (r16 & 3));
    // a negative scale is folded into the queries (bf16 sign flips), so the
    // logits are scaled by |scale| and their maximum is a plain maximum
    const uint32_t neg = (scale_log2 < 0.f) ? 0x80008000u : 0u;
    const float sc = fabsf(scale_log2);
    // Touched passages in which this wave has its first block (block `wave`)
    // and its second (block wave + kSpCompute).
    const uint64_t bmask = uniform64(
        __ballot(lane < P && ((U >> lane) & 1ull) && p_cnt[lane] > 16 * wave));
    const uint64_t bmask2 = uniform64(__ballot(
        lane < P && ((U >> lane) & 1ull) && p_cnt[lane] > 16 * (wave + kSpCompute)));
    // Queries of the blocks' rows go straight into qf.  For the wave's busy
    // passages in order: at the first tile of busy passage k the lookup of
    // busy passage k+1 starts and runs in phases, one per step: (1) the
    // passage's row masks, (2) this lane's rows (the n-th adjacent row, n =
    // 16 * block + r16) and their visual-token indices.  At passage k's last
    // tile, once its S^T products have read qf, the lookup is finished and
    // the loads of passage k+1's queries are issued into qf; they land while
    // that tile's softmax, PV product and merge run.  A lane past a block's
    // rows loads a placeholder row, whose scores land in a column that is
    // never merged.
    u32x4 qf[2][KB];
    int lk_j = -1, lk_phase = 2;       // passage being looked up; phases done (2: done)
    uint64_t lkw0 = 0, lkw1 = 0, lkw2 = 0;
    int lk_row[2] = {-1, -1}, lk_src[2] = {0, 0};   // result of the lookup
    int nx_row[2] = {-1, -1};          // rows of the queries in qf for the next passage
    auto nth_row = [&](int n) -> int {
      const int c0 = __popcll(lkw0), c1 = __popcll(lkw1), c2 = __popcll(lkw2);
      if (n >= c0 + c1 + c2) return -1;
      if (n < c0) return nth_bit64(lkw0, n);
      if (n < c0 + c1) return 64 + nth_bit64(lkw1, n - c0);
      return 128 + nth_bit64(lkw2, n - c0 - c1);
    };
    auto lookup_phase = [&]() {
      if (lk_phase == 0) {
        lkw0 = uniform64(rmask[0][lk_j]);
        lkw1 = uniform64(rmask[1][lk_j]);
        lkw2 = uniform64(rmask[2][lk_j]);
      } else {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          lk_row[k] = nth_row(16 * (wave + k * kSpCompute) + r16);
          lk_src[k] = kept_idx ? qsrc[lk_row[k] >= 0 ? lk_row[k] : 0] : 0;
        }
      }
      ++lk_phase;
    };
    auto start_lookup = [&](int j) {   // j < 0: nothing
      lk_j = j;
      lk_phase = j < 0 ? 2 : 0;
    };
    // qf <- the queries of the looked-up passage's rows (its second block
    // only where this wave has one)
    auto load_q = [&]() {
      if (lk_j < 0) return;
      while (lk_phase < 2) lookup_phase();
      const bool two_next = (bmask2 >> lk_j) & 1ull;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        if (k == 1 && !two_next) break;
        nx_row[k] = lk_row[k];
        const int rr = lk_row[k] >= 0 ? lk_row[k] : 0;
        const bf16_t* qrow = kept_idx
            ? qbase + ((size_t)b * N + lk_src[k]) * qstride + (size_t)h * D
            : qbase + (size_t)(row0 + rr) * qstride + (size_t)h * D;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
          qf[k][kb] = *reinterpret_cast<const u32x4*>(qrow + 32 * kb + 8 * g);
      }
    };
    start_lookup(bmask ? __builtin_ctzll(bmask) : -1);
    load_q();

    // per block: row of this lane's column, O^T partial, running maximum and
    // row sum of the weights (per lane until the merge)
    int acc_row[2] = {-1, -1};
    f32x4_t acc[2][DB];
    float m_run[2], l_run[2];

    // a block's partial into the item's accumulators
    auto merge = [&](auto kk) {
      constexpr int k = decltype(kk)::value;
      float l_tot = l_run[k] + swap16(l_run[k]);
      l_tot += swap_halves(l_tot);
      const int ri = acc_row[k];
      if (ri < 0) return;
      const float mo = m_acc[ri], lo = l_acc[ri];
      float4* orow = reinterpret_cast<float4*>(Oacc + ri * D);
      const float mn = fmaxf(mo, m_run[k]);
      const float a = __builtin_amdgcn_exp2f(mo - mn);    // 0 while the row is empty
      const float cb = __builtin_amdgcn_exp2f(m_run[k] - mn);
      float4 ov[DB];                    // features 16db + 4g .. +3
#pragma unroll
      for (int db = 0; db < DB; ++db) ov[db] = orow[(4 * db + g) ^ (ri & (NC4 - 1))];
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        float4 o = ov[db];
        o.x = fmaf(o.x, a, acc[k][db][0] * cb);
        o.y = fmaf(o.y, a, acc[k][db][1] * cb);
        o.z = fmaf(o.z, a, acc[k][db][2] * cb);
        o.w = fmaf(o.w, a, acc[k][db][3] * cb);
        orow[(4 * db + g) ^ (ri & (NC4 - 1))] = o;
      }
      if (g == 0) {
        m_acc[ri] = mn;
        l_acc[ri] = fmaf(lo, a, l_tot * cb);
      }
    };

    // One tile for block K0: S^T = K . Q^T (two 16-token halves), online
    // softmax of each row, O^T += V^T . P^T.  All of a phase's LDS reads are
    // issued before its products (the V reads before the softmax, which
    // hides them).  A wave with two blocks in the passage runs them one
    // after the other.
    auto tile = [&](auto k0, int stage, int t, int te_, bool first) {
      constexpr int K0 = decltype(k0)::value;
      constexpr int NBK = 1;
      if (first) {
#pragma unroll
        for (int k = 0; k < NBK; ++k) {
#pragma unroll
          for (int db = 0; db < DB; ++db) acc[K0 + k][db] = f32x4_t{0.f, 0.f, 0.f, 0.f};
          m_run[K0 + k] = -INFINITY;
          l_run[K0 + k] = 0.f;
        }
      }
      const bf16_t* Ks = Kbuf + stage * TK + koff;
      u32x4 ka[2][KB];
#pragma unroll
      for (int th = 0; th < 2; ++th)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
          ka[th][kb] = *reinterpret_cast<const u32x4*>(Ks + th * 16 * SK + 32 * kb);
      __builtin_amdgcn_sched_barrier(0);
      f32x4_t s[NBK][2];
#pragma unroll
      for (int k = 0; k < NBK; ++k)
#pragma unroll
        for (int th = 0; th < 2; ++th) {
          s[k][th] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int kb = 0; kb < KB; ++kb) s[k][th] = mfma16_bf16(ka[th][kb], qf[K0 + k][kb], s[k][th]);
        }
      __builtin_amdgcn_sched_barrier(0);
      // V reads (DB feature blocks x two 16-token halves) at constant offsets
      // from one address
      const uint32_t vaddr = vlds + (uint32_t)(stage * TV * 2);
      u32x2 vr[2 * DB];
      static_for<2 * DB>([&](auto c) {
        constexpr int th = decltype(c)::value & 1, db = decltype(c)::value >> 1;
        vr[2 * db + th] = ds_read_tr16_at<(th * 16 * SV + 16 * db) * 2>(vaddr);
      });
      __builtin_amdgcn_sched_barrier(0);
      // Online softmax of this lane's row: s[k][th][j] is token 16th + 4g + j
      // of the tile.  The weights are taken against a reference maximum m_run
      // that moves only when a tile's maximum exceeds it by more than 2^kLazy
      // (the weights then stay <= 2^kLazy and acc is rescaled only then, not
      // on every tile).
      u32x4 pb[NBK], pl[NBK];
#pragma unroll
      for (int k = 0; k < NBK; ++k) {
        if (t + kSpTile > te_) {
          const int rem = te_ - t - 4 * g;        // tokens 4g + j < rem are valid
#pragma unroll
          for (int th = 0; th < 2; ++th)
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (16 * th + j >= rem) s[k][th][j] = -INFINITY;
        }
        // this lane's 8 logits; the row maximum (over the four lanes of the
        // row) is needed only when some row's reference has to move, which
        // a lane can tell from its own logits
        const float lm = fmaxf(fmaxf(fmaxf(s[k][0][0], s[k][0][1]), fmaxf(s[k][0][2], s[k][0][3])),
                               fmaxf(fmaxf(s[k][1][0], s[k][1][1]), fmaxf(s[k][1][2], s[k][1][3])));
        float m_new = m_run[K0 + k];                        // -inf on a block's first tile
        if (__any(lm * sc > m_new + kLazy)) {
          float sm = fmaxf(lm, swap16(lm));
          sm = fmaxf(sm, swap_halves(sm));
          const float tmax = sm * sc;                       // the tile has a valid token
          if (tmax > m_new + kLazy) {
            // acc and the sum are 0 before a block's first tile: nothing to
            // rescale then
            const float alpha = m_new != -INFINITY ? __builtin_amdgcn_exp2f(m_new - tmax) : 1.f;
            m_new = tmax;
            l_run[K0 + k] *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db) acc[K0 + k][db] *= alpha;
          }
          m_run[K0 + k] = m_new;
        }
        // each weight p as a bf16 pair hi + lo: hi = p truncated to bf16 (its
        // top 16 bits, v_perm_b32 packs two), lo = the rest p - hi (exact)
        // rounded to bf16, so hi + lo is p to about 2^-16 relative
        uint32_t w[4], wl[4];
        float ls = 0.f;
#pragma unroll
        for (int th = 0; th < 2; ++th)
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(s[k][th][2 * q], sc, -m_new));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(s[k][th][2 * q + 1], sc, -m_new));
            ls += p0 + p1;
            const uint32_t b0 = __float_as_uint(p0), b1 = __float_as_uint(p1);
            w[2 * th + q] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);
            wl[2 * th + q] = pack2_bf16(p0 - __uint_as_float(b0 & 0xffff0000u),
                                        p1 - __uint_as_float(b1 & 0xffff0000u));
          }
        pb[k] = u32x4{w[0], w[1], w[2], w[3]};
        pl[k] = u32x4{wl[0], wl[1], wl[2], wl[3]};
        l_run[K0 + k] += ls;
      }
      __builtin_amdgcn_sched_barrier(0);
      // O^T += V^T . P^T
      lds_wait_all(vr);
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const u32x4 va = __builtin_shufflevector(vr[2 * db], vr[2 * db + 1], 0, 1, 2, 3);
#pragma unroll
        for (int k = 0; k < NBK; ++k) {
          acc[K0 + k][db] = mfma16_bf16(va, pb[k], acc[K0 + k][db]);
          acc[K0 + k][db] = mfma16_bf16(va, pl[k], acc[K0 + k][db]);
        }
      }
    };

    Cursor cc{U, -1, 0, 0, 0};
    for (int i = 0; i < n_tiles; ++i) {
      advance(cc);
      const bool busy = (bmask >> cc.j) & 1ull;
      const bool two = (bmask2 >> cc.j) & 1ull;
      const bool first = cc.t == cc.ts;
      const bool last = cc.t + kSpTile >= cc.te;   // the passage's last tile
      if (busy && first) {
        // this passage's queries are in qf (a negative scale's sign folded
        // in here); the lookup of the next busy passage starts
        acc_row[0] = nx_row[0];
        acc_row[1] = nx_row[1];
        if (neg) {
#pragma unroll
          for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) qf[k][kb] ^= neg;
        }
        const uint64_t rest = bmask & cc.rem;
        start_lookup(rest ? __builtin_ctzll(rest) : -1);
      } else if (lk_phase < 2) {
        lookup_phase();
      }
      // tile i has landed, and every wave's merges of the passage before (the
      // next passage's blocks hand rows to other waves)
      barrier_lds();
      if (!busy) continue;
      const int stage = i % kSpStages;
      tile(IntC<0>{}, stage, cc.t, cc.te, first);
      if (two) tile(IntC<1>{}, stage, cc.t, cc.te, first);
      if (last) {
        load_q();                      // the next busy passage's queries
        merge(IntC<0>{});
        if (two) merge(IntC<1>{});
      }
    }
  }
  __syncthreads();

  // O = acc / sum for every row of the chunk; LSE (natural log)
  const size_t obase = (size_t)row0 * H * D + (size_t)h * D;
  for (int e = tid; e < nrows * NC4; e += kSpThreads) {
    const int ri = e / NC4, q = e % NC4;
    const float4 v = reinterpret_cast<const float4*>(Oacc + ri * D)[q ^ (ri & (NC4 - 1))];
    const float l = l_acc[ri];
    const float inv = (l > 0.f) ? 1.f / l : 0.f;
    const size_t off = obase + (size_t)ri * H * D + q * 4;
    if (o_f32) {
      *reinterpret_cast<float4*>(static_cast<float*>(O) + off) =
          make_float4(v.x * inv, v.y * inv, v.z * inv, v.w * inv);
    } else {
      uint2 w;
      w.x = pack2_bf16(v.x * inv, v.y * inv);
      w.y = pack2_bf16(v.z * inv, v.w * inv);
      *reinterpret_cast<uint2*>(static_cast<bf16_t*>(O) + off) = w;
    }
  }
  if (lse && tid < nrows) {
    const float l = l_acc[tid];
    lse[(size_t)(row0 + tid) * H + h] = (l > 0.f) ? (m_acc[tid] + log2f(l)) * kLn2 : -INFINITY;
  }
}

// Standalone work-list launch (calls whose graph is given; the fused route
// builds the list in the edge-selection launch).
constexpr int kPlanThreads = 1024;

__global__ void __launch_bounds__(kPlanThreads)
attn_plan_kernel(const int32_t* __restrict__ kept_offsets,
                 const int32_t* __restrict__ query_passages,
                 const int32_t* __restrict__ passage_offsets, int B, int H, int total_kept,
                 int total_passages, int total_tokens, int k_max, int P_max, int n_ids,
                 int4* __restrict__ items) {
  __shared__ PlanLds L;
  __shared__ uint32_t scan_sh[kPlanThreads / 64 + 1];
  build_attention_plan(L, scan_sh, kept_offsets, query_passages, passage_offsets, B, H,
                       total_kept, total_passages, total_tokens, k_max, P_max, n_ids, items);
}

// ---------------------------------------------------------------------------
// Row-tile path (fp32 inputs, and small bf16 problems).  Workgroup =
// (question, head, 16 consecutive kept rows) of NW waves, which take the
// token blocks of the passages adjacent to at least one of the rows in turn
// (block i to wave i mod NW), each with its own (O, max, sum); they are
// merged in wave order through LDS at the end, so the loop has no barrier and
// no LDS access.  Per block:
//   S^T (tokens x 16 rows) = K . Q^T, a logit of a row not adjacent to the
//   passage at -inf, online softmax in base 2, O^T += V^T . P^T.
// Both products take their operands as loaded, in the order the lanes hold
// them: lane l (r16 = l % 16, g = l / 16) supplies the contraction slots of
// group g, and which feature (S) or token (O) a slot stands for is free as
// long as both operands agree.
template <typename T, int D> struct TileOps;

// float32: 16 tokens a block, v_mfma_f32_16x16x4_f32 (float32 products and
// sums).  S: slot g of product m of a 16-feature group is feature 4g + m (one
// float4 of the row).  O: slot g of product j is token 4g + j of the block,
// where S^T leaves that logit, and output row f of feature block e is feature
// 4f + e (one float4 of a token's 64 features).
template <int D> struct TileOps<float, D> {
  static constexpr int kTok = 16;      // tokens per block
  static constexpr int kS = 4;         // logits per lane and block
  static constexpr int NQ = D / 16, NH = D / 64;
  static constexpr int NA = D / 16;    // accumulator blocks (16 features x 16 rows)
  struct Q { f32x4_t x[NQ]; };
  struct KV { f32x4_t k[NQ], v[4 * NH]; };
  __device__ static void load_q(Q& q, const float* row, int g) {
#pragma unroll
    for (int i = 0; i < NQ; ++i) q.x[i] = *reinterpret_cast<const f32x4_t*>(row + 16 * i + 4 * g);
  }
  // token of logit i in the block
  __device__ static int token(int g, int i) { return 4 * g + i; }
  // head h's tokens t .. of a passage ending at te (past it: the last token,
  // masked in the softmax)
  __device__ static void load_kv(KV& x, const float* Kh, const float* Vh, int t, int te,
                                 size_t stride, int g, int r16) {
    const float* kr = Kh + (size_t)min(t + r16, te - 1) * stride + 4 * g;
#pragma unroll
    for (int i = 0; i < NQ; ++i) x.k[i] = *reinterpret_cast<const f32x4_t*>(kr + 16 * i);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float* vr = Vh + (size_t)min(t + 4 * g + j, te - 1) * stride + 4 * r16;
#pragma unroll
      for (int hf = 0; hf < NH; ++hf)
        x.v[NH * j + hf] = *reinterpret_cast<const f32x4_t*>(vr + 64 * hf);
    }
  }
  __device__ static void logits(float (&s)[kS], const Q& q, const KV& x) {
    f32x4_t a[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int i = 0; i < NQ; ++i)
#pragma unroll
      for (int m = 0; m < 4; ++m)
        a[i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.k[i][m], q.x[i][m], a[i & 1], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = a[0][i] + a[1][i];
  }
  __device__ static void weigh(f32x4_t (&acc)[NA], const KV& x, const float (&p)[kS]) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < NA; ++e)
        acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.v[NH * j + (e >> 2)][e & 3], p[j],
                                                      acc[e], 0, 0, 0);
  }
  // four consecutive features from element i of the accumulators: q-th piece
  // of the lane's 16 NH features, starting at feature first(g, q)
  static constexpr int kPieces = 4 * NH;
  __device__ static int first(int g, int q) { return 64 * (q >> 2) + 16 * g + 4 * (q & 3); }
  __device__ static f32x4_t piece(const f32x4_t (&acc)[NA], int q) {
    const int hf = q >> 2, i = q & 3;
    return f32x4_t{acc[4 * hf][i], acc[4 * hf + 1][i], acc[4 * hf + 2][i], acc[4 * hf + 3][i]};
  }
  __device__ static void set_piece(f32x4_t (&acc)[NA], int q, f32x4_t x) {
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[4 * (q >> 2) + u][q & 3] = x[u];
  }
  // the values of token(g, i) as zeros
  __device__ static void clear_v(KV& x, int i) {
#pragma unroll
    for (int hf = 0; hf < NH; ++hf) x.v[NH * i + hf] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
};

// bfloat16: 32 tokens a block, v_mfma_f32_16x16x32_bf16.  S as in the sparse
// kernel.  O: a lane loads E = D / 16 features of each of its eight tokens and
// pairs tokens into the slots' order (one v_perm_b32 per word), so output row
// f of feature block e is feature E f + e; the weights as bf16 pairs hi + lo.
template <int D> struct TileOps<bf16_t, D> {
  static constexpr int kTok = 32, kS = 8;
  static constexpr int KB = D / 32;
  static constexpr int NA = D / 16, E = D / 16;      // E: features per lane of a token
  typedef uint32_t vword __attribute__((ext_vector_type(E / 2)));
  struct Q { u32x4 x[KB]; };
  struct KV { u32x4 k[2][KB]; vword v[8]; };
  __device__ static void load_q(Q& q, const bf16_t* row, int g) {
#pragma unroll
    for (int i = 0; i < KB; ++i) q.x[i] = *reinterpret_cast<const u32x4*>(row + 32 * i + 8 * g);
  }
  __device__ static int token(int g, int i) { return 16 * (i >> 2) + 4 * g + (i & 3); }
  __device__ static void load_kv(KV& x, const bf16_t* Kh, const bf16_t* Vh, int t, int te,
                                 size_t stride, int g, int r16) {
#pragma unroll
    for (int th = 0; th < 2; ++th) {
      const bf16_t* kr = Kh + (size_t)min(t + 16 * th + r16, te - 1) * stride + 8 * g;
#pragma unroll
      for (int i = 0; i < KB; ++i) x.k[th][i] = *reinterpret_cast<const u32x4*>(kr + 32 * i);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
      x.v[i] = *reinterpret_cast<const vword*>(
          Vh + (size_t)min(t + token(g, i), te - 1) * stride + E * r16);
  }
  __device__ static void logits(float (&s)[kS], const Q& q, const KV& x) {
#pragma unroll
    for (int th = 0; th < 2; ++th) {
      f32x4_t a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < KB; ++i) a = mfma16_bf16(x.k[th][i], q.x[i], a);
#pragma unroll
      for (int i = 0; i < 4; ++i) s[4 * th + i] = a[i];
    }
  }
  __device__ static void weigh(f32x4_t (&acc)[NA], const KV& x, const float (&p)[kS]) {
    u32x4 hi, lo;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t b0 = __float_as_uint(p[2 * q]), b1 = __float_as_uint(p[2 * q + 1]);
      hi[q] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);
      lo[q] = pack2_bf16(p[2 * q] - __uint_as_float(b0 & 0xffff0000u),
                         p[2 * q + 1] - __uint_as_float(b1 & 0xffff0000u));
    }
#pragma unroll
    for (int e = 0; e < NA; ++e) {
      u32x4 a;                          // feature E f + e of the eight tokens
#pragma unroll
      for (int q = 0; q < 4; ++q)
        a[q] = __builtin_amdgcn_perm(x.v[2 * q + 1][e >> 1], x.v[2 * q][e >> 1],
                                     (e & 1) ? 0x07060302u : 0x05040100u);
      acc[e] = mfma16_bf16(a, hi, acc[e]);
      acc[e] = mfma16_bf16(a, lo, acc[e]);
    }
  }
  static constexpr int kPieces = E;
  __device__ static int first(int g, int q) { return 4 * E * g + 4 * q; }
  __device__ static f32x4_t piece(const f32x4_t (&acc)[NA], int q) {
    const int i = 4 * q / E, e = 4 * q % E;
    return f32x4_t{acc[e][i], acc[e + 1][i], acc[e + 2][i], acc[e + 3][i]};
  }
  __device__ static void set_piece(f32x4_t (&acc)[NA], int q, f32x4_t x) {
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[4 * q % E + u][4 * q / E] = x[u];
  }
  __device__ static void clear_v(KV& x, int i) { x.v[i] = vword(0u); }
};

// Bound by the waves' chains of loads, products and softmax: on 768 float32
// tiles of 640 tokens (8 questions of 96 rows, 16 heads of 64, 5 passages of
// 97-160) the matrix cores are busy 38 % of the cycles, the waves wait 28 % of
// theirs for loads and 57 % to issue, and two workgroups a CU make one and a half
// rounds of it; on 768 bf16 tiles the matrix cores are busy 6 %.  Rows not
// adjacent to a passage of their tile compute for nothing there, yet one wave per
// row and head on the vector units, edges only, took ten times as long: that
// batch 35.5 us (359); one question of 96 rows, 4 heads of 64, 4 passages of 64
// tokens 8.1 us (38.3).
constexpr int kTileRows = 16;
// Workgroups from which four waves each fill the chip; below, eight shorten
// the wave's chain (routes of 350 to 2304 workgroups: 134 us with four and
// 111 with eight at the low end, equal within 1.5 % at 768, 154 with eight
// and 140 with four at the high end).
constexpr long long kTileWide = 1024;
// bf16 problems of at most this many workgroups x d_h go by row tiles, larger
// ones to the sparse kernel, whose items of up to 192 rows read K and V once
// but leave most of the chip idle at few (question, head) pairs and walk the
// passages one tile of tokens after the other.  A tile computes every passage
// adjacent to one of its rows; with many passages and few edges that is more
// work, but the sparse kernel's items walk as many.  Graph and attention call,
// 16 heads of 64, 96 rows, tiles against sparse: 8 questions (768 workgroups),
// 5 passages of 128 tokens and degree 4 40 us against 47, 20 of 256 140 against
// 146, 64 of 128 175 against 259 (degree 1: 119 against 212); one question, 64
// of 512 191 against 627.  At 1536 workgroups routes take 75-230 us against
// 77-167.
// Long passages cost the tiles more, as each streams K and V again: past 256
// tokens 768 workgroups lose up to 14 % (20 of 1024 tokens, degree 2: 488 us
// against 421; 5 of 512 86 against 83), 576 break even (81-451 against 83-417)
// and 480 win from 14 % up (72-336 against 83-417), the same at half the
// workgroups of d_h = 128: hence kTileWorkLong.
constexpr long long kTileWork = 768 * 64;
constexpr long long kTileWorkLong = 512 * 64;
constexpr int kTileLong = 256;         // longest passage, in tokens, that kTileWork holds for

// Whether an element of x is infinite or not a number, from the bits: at least
// those of the infinity of its sign, as integers (opaque to the compiler: this
// file is compiled for values that are numbers).
template <int N>
__device__ __forceinline__ bool any_not_finite(const f32x4_t (&x)[N]) {
  int pos = 0;
  uint32_t neg = 0u;
#pragma unroll
  for (int e = 0; e < N; ++e)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t u = __float_as_uint(x[e][i]);
      asm("" : "+v"(u));
      pos = max(pos, (int)u);
      neg = max(neg, u);
    }
  return pos >= 0x7f800000 || neg >= 0xff800000u;
}

// Workgroups of a row of the grid: a dimension of a launch takes fewer than 2^32
// threads, 2^23 workgroups of 512.
constexpr int kTileGridX = 1 << 22;

template <typename T, int D, int NW>
__global__ void __launch_bounds__(64 * NW, 2)
attn_tile_kernel(const T* __restrict__ qbase, const int32_t* __restrict__ kept_idx, int N,
                 int qstride, const int32_t* __restrict__ kept_offsets,
                 const T* __restrict__ Kh, const T* __restrict__ Vh,
                 const int32_t* __restrict__ passage_offsets,
                 const int32_t* __restrict__ query_passages,
                 const uint64_t* __restrict__ rowmask, int H, int groups, int ygroups,
                 int tiles, int total_kept, int total_passages, int total_tokens, int k_max, int P_max,
                 float scale_log2, void* __restrict__ O, int o_f32, float* __restrict__ lse) {
  using Ops = TileOps<T, D>;
  constexpr int TB = Ops::kTok, NS = Ops::kS, NA = Ops::NA;
  constexpr int OS = D + 4;            // floats per row of a wave's partial (bank spread)
  __shared__ __align__(16) float po[NW][kTileRows][OS];
  __shared__ float pm[NW][kTileRows], pl[NW][kTileRows];
  // all row tiles of a (question, head) on one XCD (workgroup id L goes to
  // XCD L % 8), where they share its K and V in the L2; blockIdx.y: ygroups
  // (question, head) pairs each
  const int L = blockIdx.x, grp = blockIdx.y * ygroups + (L & 7) + 8 * ((L >> 3) / tiles);
  if (grp >= groups) return;
  const int b = grp / H, h = grp % H, r0 = ((L >> 3) % tiles) * kTileRows;
  int k0, k1, p0, p1;
  range_of(kept_offsets, b, total_kept, k0, k1);
  range_of(query_passages, b, total_passages, p0, p1);
  const int kq = min(k1 - k0, k_max);
  const int P = min(min(p1 - p0, P_max), 64);
  if (r0 >= kq) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, r16 = lane & 15;

  // this lane's row (a lane past the question's rows repeats its last one,
  // adjacent to nothing)
  const int r = min(r0 + r16, kq - 1);
  uint64_t mk = (r0 + r16 < kq) ? rowmask[k0 + r] : 0ull;
  if (P < 64) mk &= (1ull << P) - 1ull;
  typename Ops::Q qf;
  Ops::load_q(qf, kept_idx
      ? qbase + ((size_t)b * N + clampi(kept_idx[k0 + r], 0, N - 1)) * qstride + (size_t)h * D
      : qbase + (size_t)(k0 + r) * qstride + (size_t)h * D, g);
  uint64_t U = mk;                     // passages adjacent to some row of the tile
#pragma unroll
  for (int x = 1; x < 16; x <<= 1) U |= (uint64_t)__shfl_xor((unsigned long long)U, x, kWave);
  U = uniform64(U);

  // A block in flight: its K and V operands, passage and tokens t .. te - 1.
  struct Block {
    typename Ops::KV kv;
    int j, t, te;
  };
  // the wave's cursor: block nb of passage j (nbk blocks, tokens ts .. te - 1)
  uint64_t rem;
  int j = 0, ts = 0, te = 0, nb, nbk;
  auto load = [&](Block& x) -> bool {    // the next block of the wave, if any
    while (nb >= nbk) {
      if (!rem) return false;
      nb -= nbk;
      j = __builtin_ctzll(rem);
      rem &= rem - 1ull;
      range_of(passage_offsets, p0 + j, total_tokens, ts, te);
      ts = __builtin_amdgcn_readfirstlane(ts);
      te = __builtin_amdgcn_readfirstlane(te);
      nbk = (te - ts + TB - 1) / TB;
    }
    x.j = j;
    x.t = ts + TB * nb;
    x.te = te;
    nb += NW;
    Ops::load_kv(x.kv, Kh + (size_t)h * D, Vh + (size_t)h * D, x.t, te, (size_t)H * D, g, r16);
    return true;
  };

  // Rows not adjacent to a block's passage, and the tokens that pad its last
  // block, meet V with a weight of 0.  That adds nothing as long as V is
  // finite; if an accumulator ends infinite or not a number, the wave goes
  // over its blocks again, `careful`: the accumulators of a row not adjacent to
  // the passage are put back after the product, padding tokens count as zeros,
  // and the weights stay <= 1, so that a value reaches only the rows with an
  // edge to its passage and a sum overflows only where it must.
  f32x4_t acc[NA];
  float m_run, l_run;                    // l_run: this lane's share of the row's sum
  auto start = [&]() {
    rem = U;
    nb = wave;
    nbk = 0;
    m_run = -INFINITY;
    l_run = 0.f;
#pragma unroll
    for (int e = 0; e < NA; ++e) acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  };
  auto compute = [&](Block& x, auto careful_) {
    constexpr bool careful = decltype(careful_)::value != 0;
    float s[NS];
    Ops::logits(s, qf, x.kv);
    const bool adj = (mk >> x.j) & 1ull;
    float lm = -INFINITY;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      s[i] = (adj && x.t + Ops::token(g, i) < x.te) ? s[i] * scale_log2 : -INFINITY;
      lm = fmaxf(lm, s[i]);
    }
    // the reference maximum moves when a logit exceeds it by more than kLazy
    // (weights stay <= 2^kLazy), so most blocks need no exchange or rescale
    constexpr float slack = careful ? 0.f : kLazy;
    if (__any(lm > m_run + slack)) {
      float mx = fmaxf(lm, swap16(lm));
      mx = fmaxf(mx, swap_halves(mx));
      if (mx > m_run + slack) {
        const float alpha = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - mx);
        m_run = mx;
        l_run *= alpha;
#pragma unroll
        for (int e = 0; e < NA; ++e) acc[e] *= alpha;
      }
    }
    const float ref = m_run == -INFINITY ? 0.f : m_run;   // (no logit of the row yet: weights 0)
    float p[NS], ls = 0.f;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      p[i] = __builtin_amdgcn_exp2f(s[i] - ref);
      ls += p[i];
    }
    l_run += ls;
    if (careful) {
#pragma unroll
      for (int i = 0; i < NS; ++i)
        if (x.t + Ops::token(g, i) >= x.te) Ops::clear_v(x.kv, i);
#pragma unroll
      for (int q = 0; q < Ops::kPieces; ++q)
        *reinterpret_cast<f32x4_t*>(&po[wave][r16][Ops::first(g, q)]) = Ops::piece(acc, q);
    }
    Ops::weigh(acc, x.kv, p);
    if (careful && !adj)
#pragma unroll
      for (int q = 0; q < Ops::kPieces; ++q)
        Ops::set_piece(acc, q, *reinterpret_cast<f32x4_t*>(&po[wave][r16][Ops::first(g, q)]));
  };
  start();
  // two blocks in turn: one's loads are in flight while the other computes
  Block xa, xb;
  bool more = load(xa);
  while (more) {
    const bool second = load(xb);
    compute(xa, IntC<0>{});
    if (!second) break;
    more = load(xa);
    compute(xb, IntC<0>{});
  }
  if (__builtin_expect(__any(any_not_finite(acc)), 0)) {
    start();
    while (load(xa)) compute(xa, IntC<1>{});
  }

  // the waves' partials, merged in wave order
  float l_tot = l_run + swap16(l_run);
  l_tot += swap_halves(l_tot);
  if (g == 0) {
    pm[wave][r16] = m_run;
    pl[wave][r16] = l_tot;
  }
#pragma unroll
  for (int q = 0; q < Ops::kPieces; ++q)
    *reinterpret_cast<f32x4_t*>(&po[wave][r16][Ops::first(g, q)]) = Ops::piece(acc, q);
  __syncthreads();
  for (int u = threadIdx.x; u < kTileRows * (D / 4); u += 64 * NW) {
    const int ri = u / (D / 4), c = 4 * (u % (D / 4));
    if (r0 + ri >= kq) continue;
    float M = pm[0][ri];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, pm[w][ri]);
    const float ref = M == -INFINITY ? 0.f : M;
    f32x4_t o = {0.f, 0.f, 0.f, 0.f};
    float l = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float a = __builtin_amdgcn_exp2f(pm[w][ri] - ref);
      l = fmaf(pl[w][ri], a, l);
      o += *reinterpret_cast<const f32x4_t*>(&po[w][ri][c]) * a;
    }
    const float inv = (l > 0.f) ? 1.f / l : 0.f;
    const size_t row = (size_t)(k0 + r0 + ri);
    const size_t off = (row * H + h) * D + c;
    o *= inv;
    if (o_f32)
      *reinterpret_cast<f32x4_t*>(static_cast<float*>(O) + off) = o;
    else
      *reinterpret_cast<uint2*>(static_cast<bf16_t*>(O) + off) =
          make_uint2(pack2_bf16(o[0], o[1]), pack2_bf16(o[2], o[3]));
    if (lse && c == 0) lse[row * H + h] = (l > 0.f) ? (M + log2f(l)) * kLn2 : -INFINITY;
  }
}

// ---------------------------------------------------------------------------
// Whether the row-tile kernel runs (else the passage-major sparse kernel).
bool attn_by_tiles(const skip_problem_t& p) {
  if (p.dtype != SKIP_BF16) return true;
  return (long long)p.B * p.H * ((p.k_max + kTileRows - 1) / kTileRows) * p.d_h <=
         (p.L_max <= kTileLong ? kTileWork : kTileWorkLong);
}

long long attn_plan_ids(const skip_problem_t& p) {
  if (p.dtype != SKIP_BF16 || p.k_max <= 0 || p.B <= 0 || p.H <= 0) return 0;
  const long long runs = ((long long)p.B * p.H + 7) / 8;
  const long long nch = (p.k_max + kSpRows - 1) / kSpRows;
  return 8 * runs * nch;
}

hipError_t launch_attention_plan(const skip_problem_t& p, const int32_t* kept_offsets,
                                 const int32_t* query_passages,
                                 const int32_t* passage_offsets, int32_t* plan, hipStream_t s) {
  const long long n_ids = attn_plan_ids(p);
  if (n_ids == 0 || attn_by_tiles(p)) return hipSuccess;
  if (n_ids > INT32_MAX / 16 || (long long)p.B * p.H > INT32_MAX / 16)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(attn_plan_kernel, dim3(1), dim3(kPlanThreads), 0, s, kept_offsets,
                     query_passages, passage_offsets, p.B, p.H, p.total_kept,
                     p.total_passages, p.total_tokens, p.k_max, p.P_max, (int)n_ids,
                     reinterpret_cast<int4*>(plan));
  return hipGetLastError();
}

hipError_t launch_attention(const skip_problem_t& p, QuerySource q,
                            const int32_t* kept_offsets, const void* Kh, const void* Vh,
                            const int32_t* passage_offsets, const int32_t* query_passages,
                            const uint64_t* rowmask, const int32_t* plan, void* O, float* lse,
                            hipStream_t s) {
  if (p.k_max <= 0) return hipSuccess;
  const int qstride = p.d;
  if (!attn_by_tiles(p)) {
    const long long n_ids = attn_plan_ids(p);
    if (n_ids > INT32_MAX / 16 || (long long)p.B * p.H > INT32_MAX / 16)
      return hipErrorInvalidValue;
    const int4* items = reinterpret_cast<const int4*>(plan);
    const float sl2 = p.sm_scale * kLog2e;
#define SKIP_ATTN_SPARSE(DD)                                                                 \
  hipLaunchKernelGGL((attn_sparse_kernel<DD>), dim3((unsigned)n_ids), dim3(kSpThreads),     \
                     0, s, (const bf16_t*)q.base, q.kept_idx, q.N, qstride, (const bf16_t*)Kh, \
                     (const bf16_t*)Vh, passage_offsets, rowmask, items, p.H, p.total_tokens, \
                     sl2, O, p.o_f32, lse)
    if (p.d_h == 64) SKIP_ATTN_SPARSE(64);
    else SKIP_ATTN_SPARSE(128);
#undef SKIP_ATTN_SPARSE
  } else {
    const long long groups = (long long)p.B * p.H;
    if (groups > INT32_MAX - kTileGridX) return hipErrorInvalidValue;
    const int tiles = (p.k_max + kTileRows - 1) / kTileRows;
    const long long nwg = 8 * ((groups + 7) / 8) * tiles;
    // one row of the grid, as a rule
    const int ygroups = (int)std::min<long long>(8 * ((groups + 7) / 8),
                                                 std::max(8, kTileGridX / tiles / 8 * 8));
    const dim3 grid(ygroups * tiles, (unsigned)((groups + ygroups - 1) / ygroups));
#define SKIP_ATTN_TILE(T, DD, NW)                                                            \
  hipLaunchKernelGGL((attn_tile_kernel<T, DD, NW>), grid, dim3(64 * NW), 0, s,               \
                     (const T*)q.base, q.kept_idx, q.N, qstride, kept_offsets,               \
                     (const T*)Kh, (const T*)Vh, passage_offsets, query_passages, rowmask,   \
                     p.H, (int)groups, ygroups, tiles, p.total_kept, p.total_passages,       \
                     p.total_tokens, p.k_max, p.P_max, p.sm_scale * kLog2e, O,               \
                     p.dtype == SKIP_F32 || p.o_f32, lse)
    const bool wide = nwg >= kTileWide;
    if (p.dtype == SKIP_BF16) {
      if (p.d_h == 64) SKIP_ATTN_TILE(bf16_t, 64, 8);
      else SKIP_ATTN_TILE(bf16_t, 128, 8);
    } else if (p.d_h == 64) {
      if (wide) SKIP_ATTN_TILE(float, 64, 4);
      else SKIP_ATTN_TILE(float, 64, 8);
    } else {
      if (wide) SKIP_ATTN_TILE(float, 128, 4);
      else SKIP_ATTN_TILE(float, 128, 8);
    }
#undef SKIP_ATTN_TILE
  }
  return hipGetLastError();
}

}  // namespace skip
