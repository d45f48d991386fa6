// Device kernels of the fused projection + cross-entropy path.
//
//   forward : fwd_tiles_kernel  (logit tiles on MFMA, online max / sum-exp and target
//             gather per lane: Alg. 1 in tile form; one workgroup per row block x
//             vocabulary window: Section 3.2.1)
//             merge_rows_kernel (the merging epilogue of Section 3.2.1, lse = m + ln a,
//             per-row loss; its last block adds the blocks' sums in fixed order;
//             finalize_loss_kernel does that for flce_merge_partials)
//   backward: compact_targets_kernel (n_valid, range flag, the rows that count; up to 2048
//             rows the row preparation does its scan itself) and prep_rows_tiled_kernel /
//             prep_rows_kernel (the rows that count packed together, since ignored rows have a
//             zero row of G: pre-tiled, twice, for the tuned loop; as they are for fp32;
//             as they are and transposed for the generic loop)
//             pack_rows_kernel (the forward's pre-tiled copy of H for the tuned loop, where
//             it pays); transpose_pad_kernel (generic loop: the K-contiguous copy of W that the
//             dH contraction needs)
//             recompute_kernel (Alg. 2: z recomputed, g = p - onehot, staged once in a
//             fixed-size buffer; the generic loop also stages the transpose)
//             contract_kernel (Eq. 4 and Eq. 5 as output-stationary MFMA
//             contractions with a fixed chunk order; Gamma applied at the flush);
//             contract_pair_kernel (both in one launch, small problems)
//             splitk_reduce_kernel / splitk_reduce_pair_kernel (fixed-order sum of K slices
//             when a contraction launch would otherwise leave most CUs idle)
//   Alg. 3/4: the forward and the backward above with Gamma = 1, then scale_kernel
//   per row : merge_rows_kernel writes one loss per row (label smoothing: colsum_* and
//             mean_logit_kernel give mean_v Z_iv), recompute_kernel<.., PER_ROW> scales each
//             row of G by that row's upstream gradient
//   slices  : the same kernels on rows [v_begin, v_begin + V) of the vocabulary
//             (classify_target_in_slice); merge_rows_partial_kernel hands out (m, a, z_target)
#pragma once
#include <type_traits>

#include "mainloop_f32.h"
#include "mainloop_fast.h"
#include "tile_mma.h"

namespace flce {

// Byte offset of row block rb in a pre-tiled copy of a matrix with d columns: the block's ceil(d / 32) images of 16 KiB
// plus a skew, so that the blocks do not start a power of two apart (the workgroups resident at one time stream
// several dozen blocks side by side, and blocks exactly 2^k bytes apart land on the same DRAM banks).
#ifndef FLCE_PACK_SKEW
#define FLCE_PACK_SKEW 17408
#endif
__host__ __device__ __forceinline__ int64_t packed_block_offset(int rb, int d) {
  return (int64_t)rb * ((int64_t)((d + 31) / 32 * 32) * (TILE * 2) + FLCE_PACK_SKEW);
}
// The same for the transposed pre-tiled copy of a matrix with `rows` rows (a multiple of 256): byte offset of the
// block of column tile q (256 columns), which holds rows / 32 images.
__host__ __device__ __forceinline__ int64_t packed_cols_offset(int q, int rows) {
  return (int64_t)q * ((int64_t)rows * (TILE * 2) + FLCE_PACK_SKEW);
}

// Main-loop policies.  A kernel is written once against this interface:
//   THREADS, MIN_WAVES (launch bounds), TILE (output tile edge), LDS (dynamic LDS bytes), WM x WN (accumulator blocks per wavefront, 16 values of a
//   lane in one N column of ROWS rows each), Acc: a finished tile's accumulators, get(i, j, r) element r of block (i, j)
//   (i, j, r constants after unrolling), tile_m(i, r) / tile_n(j): its position inside the tile; inside its block it is row
//   (r / 4) QUAD + lane_row() + r % 4,
//   slot(): which of the SLOTS lanes that share an N column this lane is,
//   TRANSPOSING: can take an operand whose K index runs over memory rows (otherwise K-contiguous copies are made),
//   TUNED: the bf16 loop with its persistent launches, pre-tiled copies and blocked G.
template <int WM, int WN>
struct VectorAcc {        // of the loops that leave the accumulators to the compiler
  f32x16 v[WM][WN];
  __device__ __forceinline__ float get(int i, int j, int r) const { return v[i][j][r]; }
};
struct GenericLoop {      // bf16 where the tuned loop does not reach (address windows); 8 wavefronts 2 x 4
  static constexpr int TILE = flce::TILE, THREADS = flce::THREADS, WM = flce::WM, WN = flce::WN, LDS = LDS_BYTES;
  static constexpr bool TRANSPOSING = false, TUNED = false;
  static constexpr int MIN_WAVES = 1;
  static constexpr int ROWS = 32, QUAD = 8, SLOTS = 4;
  using Acc = VectorAcc<WM, WN>;
  static __device__ __forceinline__ int lane_row() { return (threadIdx.x & 32) >> 3; }
  static __device__ __forceinline__ int tile_m(int i, int r) { return flce::tile_m(i, r); }
  static __device__ __forceinline__ int tile_n(int j) { return flce::tile_n(j); }
  static __device__ __forceinline__ int slot() {
    return ((threadIdx.x >> 6) >> 2) * 2 + ((threadIdx.x & 63) >> 5);
  }
  // A sequence of tiles A[a_row0 ..][:] x B[b_row0 ..][:] over K = k_elems; start() names the next tile, run() computes
  // it and calls `released` when the next start() may come.  This loop has nothing to request ahead: start() only records the operands.
  template <bool BT>
  struct Stream {
    TileSrc As, Bs;
    int k_bytes;
    __device__ __forceinline__ void start(const bf16_t* A, int64_t lda_bytes, int a_row0, int a_rows, const bf16_t* B,
                                          const bf16_t*, int64_t ldb_bytes, int b_row0, int b_rows, int k_elems, char*) {
      As = TileSrc{reinterpret_cast<const char*>(A), lda_bytes, a_row0, a_rows};
      Bs = TileSrc{reinterpret_cast<const char*>(B), ldb_bytes, b_row0, b_rows};
      k_bytes = k_elems * (int)sizeof(bf16_t);
    }
    template <typename F>
    __device__ __forceinline__ void run(char* lds, Acc& acc, F released) {
      tile_mainloop(As, Bs, k_bytes, lds, acc.v);
      released();
    }
  };
  static __device__ __forceinline__ void run(const void* A, int64_t lda_bytes, int a_row0, int a_rows, const void* B,
                                             int64_t ldb_bytes, int b_row0, int b_rows, int k_bytes, char* lds,
                                             Acc& acc) {
    const TileSrc As{static_cast<const char*>(A), lda_bytes, a_row0, a_rows};
    const TileSrc Bs{static_cast<const char*>(B), ldb_bytes, b_row0, b_rows};
    tile_mainloop(As, Bs, k_bytes, lds, acc.v);
  }
};

template <int T>
struct F32Loop {          // fp32; T x T tiles, 4 wavefronts 2 x 2, two workgroups per CU
  static constexpr int TILE = T, THREADS = f32::THREADS, WM = T / 64, WN = T / 64, LDS = f32::lds_bytes<T>();
  static constexpr bool TRANSPOSING = true, TUNED = false;
  // wavefronts per SIMD that the compiler has to leave registers for: two workgroups of 128-row tiles need it told (64-row ones have
  // room anyway, and are 1 % faster with their sums in the accumulation registers)
  static constexpr int MIN_WAVES = T == 128 ? 2 : 1;
  static constexpr int ROWS = 32, QUAD = 8, SLOTS = 4;
  using Acc = VectorAcc<WM, WN>;
  static __device__ __forceinline__ int lane_row() { return (threadIdx.x & 32) >> 3; }
  static __device__ __forceinline__ int tile_m(int i, int r) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    return (wave >> 1) * (T / 2) + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
  }
  static __device__ __forceinline__ int tile_n(int j) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    return (wave & 1) * (T / 2) + j * 32 + (lane & 31);
  }
  static __device__ __forceinline__ int slot() { return fast::slot_of_lane(); }
  template <bool BT>
  struct Stream {         // as GenericLoop::Stream: the other resident workgroup covers a tile's first requests
    f32::Operand As, Bs;
    int k_elems;
    __device__ __forceinline__ void start(const float* A, int64_t lda_bytes, int a_row0, int a_rows, const float* B,
                                          const float*, int64_t ldb_bytes, int b_row0, int b_rows, int k, char*) {
      As = f32::Operand{reinterpret_cast<const char*>(A), lda_bytes, a_row0, a_rows, 0};
      Bs = f32::Operand{reinterpret_cast<const char*>(B), ldb_bytes, b_row0, b_rows, 0};
      k_elems = k;
    }
    template <typename F>
    __device__ __forceinline__ void run(char* lds, Acc& acc, F released) {
      f32::mainloop<T, f32::KC, f32::KC>(As, Bs, k_elems, lds, acc.v);
      released();
    }
  };
};

// The tuned bf16 loop; 4 wavefronts 2 x 2 of 32 B rows x 32 B columns, global -> LDS DMA.
// RAGGED: the hidden size is a multiple of 8 but not of 32 (the K extent of the forward and the recompute; the
// contractions' K extents are whole tiles, they always run with the plain form).
template <bool RAGGED, int B>
struct TunedLoop {
  static constexpr int TILE = 64 * B, THREADS = fast::THREADS, WM = B / 2, WN = 2 * B;
  static constexpr bool TRANSPOSING = true, TUNED = true;
  static constexpr int MIN_WAVES = 1;
  static constexpr int ROWS = 64, QUAD = 16, SLOTS = 8;
  using Acc = fast::Acc<2 * B, 2 * B>;
  // 256-row tiles: one workgroup per CU, 4 stages of 32 KiB; 128-row tiles: two, 5 stages of 16 KiB each
  static constexpr int PER_CU = B == 4 ? 1 : 2, STAGES = B == 4 ? fast::NS : 5, STAGE = B * 8192, LDS = STAGES * STAGE;
  template <int LA, int LB, bool RG = false> using Pipe = fast::Pipe<LA, LB, true, B, STAGES, RG, B>;
  // LDS that post-processing may use while the next tile's first K stages are being filled: the last stage
  static constexpr int FREE_LDS_OFFSET = (STAGES - 1) * STAGE;
  static __device__ __forceinline__ int lane_row() { return (threadIdx.x & 48) >> 2; }
  static __device__ __forceinline__ int tile_m(int i, int r) {
    const int wave = threadIdx.x >> 6;
    return (wave >> 1) * (B * 32) + i * ROWS + (r >> 2) * QUAD + lane_row() + (r & 3);
  }
  static __device__ __forceinline__ int tile_n(int j) {
    const int wave = threadIdx.x >> 6;
    return (wave & 1) * (B * 32) + j * 16 + (threadIdx.x & 15);
  }
  static __device__ __forceinline__ int slot() { return (threadIdx.x >> 7) * 4 + ((threadIdx.x & 63) >> 4); }
  // A sequence of tiles with the same B operand: start() requests the first K stages of a tile (all LDS stages must
  // be free: every wavefront is past the previous run()), run() computes it.  BP: B is also given pre-tiled (Bp:
  // per 256-row block and K step the 16 KiB image of its LDS tile, see pack_rows_kernel), and that copy is read.
  template <bool BP>
  struct Stream {
    Pipe<fast::KC, BP ? fast::PK : fast::KC, RAGGED> pipe;
    __device__ __forceinline__ void start(const bf16_t* A, int64_t lda_bytes, int a_row0, int a_rows, const bf16_t* Bm,
                                          const bf16_t* Bp, int64_t ldb_bytes, int b_row0, int b_rows, int k_elems,
                                          char* lds) {
      const fast::Operand As{reinterpret_cast<const char*>(A), lda_bytes, a_row0, a_rows, 0};
      if constexpr (BP) {
        // the block's images follow each other, one per K step, 64 bytes per row
        const fast::Operand Bs{reinterpret_cast<const char*>(Bp) + packed_block_offset(b_row0 / flce::TILE, k_elems) +
                                   b_row0 % flce::TILE * 64, 0, 0, 0, 0};
        pipe.start(As, Bs, k_elems, lds);
      } else {
        const fast::Operand Bs{reinterpret_cast<const char*>(Bm), ldb_bytes, b_row0, b_rows, 0};
        pipe.start(As, Bs, k_elems, lds);
      }
    }
    template <typename F>
    __device__ __forceinline__ void run(char* lds, Acc& acc, F released) { pipe.run(lds, released); }
  };
  // A wavefront's pieces of 16 rows x (32 B) columns of bf16 on their way through its slice of the free stage, rows of
  // ROW_BYTES in 16-byte chunks whose number is XOR-ed with mix(row), so that the 16 rows (x 2 neighbouring 8-byte halves)
  // one write cycle touches lie in different banks, and likewise the four rows x four neighbouring chunks of a read
  // cycle (blocks of G; output rows are read in the order of the places, and the store takes the chunks as they come).  Counted
  // bank conflicts, of the LDS's busy cycles: recompute 3 % at 8192 x 4096 x 128256, 12 % at 4096 x 768 x 50257, dW up to 2.5 %.
  // piece_slot: where a lane writes its 4 columns of quad rq of block i in row r; piece_chunk: where chunk c of row r is read.
  static constexpr int ROW_BYTES = 64 * B, CHUNKS = ROW_BYTES / 16, ROWS_PER_STORE = 64 / CHUNKS;
  static __device__ __forceinline__ int mix(int r) {
    return B == 4 ? ((r & 3) << 2 | r >> 2) : ((r >> 1 & 1) << 2 | r >> 2);
  }
  static __device__ __forceinline__ int piece_slot(int r, int i, int rq) {      // chunk i * 8 + rq * 2 + (lane / 32), half (lane / 16) % 2
    const int quarter = (threadIdx.x & 63) >> 4;
    return r * ROW_BYTES + (((i * 8 + rq * 2 + (quarter >> 1)) ^ mix(r)) << 4) + ((quarter & 1) << 3);
  }
  static __device__ __forceinline__ int piece_chunk(int r, int c) { return r * ROW_BYTES + ((c ^ mix(r)) << 4); }
};
template <bool RAGGED> struct FastLoop : TunedLoop<RAGGED, 4> { using Even = FastLoop<false>; };
template <bool RAGGED> struct SmallLoop : TunedLoop<RAGGED, 2> { using Even = SmallLoop<false>; };

#ifndef FLCE_FWD_GROUP
#define FLCE_FWD_GROUP 8     // row blocks per raster patch of the forward (x 32 / this many windows per XCD)
#endif
constexpr float LOG2E = 1.4426950408889634f;
constexpr float NEG_INF = -__builtin_inff();

// First 256 bytes of every workspace.
struct Header {
  int32_t status;      // 0 or FLCE_ERR_TARGET_RANGE
  int32_t pad0;
  int64_t n_valid;     // number of counted rows
  float loss_sum;      // un-normalised sum of per-row losses (forward only)
  uint32_t arrived;    // blocks of the window merge that have handed in their sums (forward only)
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Four consecutive elements of the storage type <-> four floats.
template <typename T> struct Pack4;
template <> struct Pack4<float> {
  static __device__ __forceinline__ void store(float* p, float a, float b, float c, float d) {
    *reinterpret_cast<f32x4*>(p) = f32x4{a, b, c, d};
  }
  static __device__ __forceinline__ void load(const float* p, float (&v)[4]) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(p);
    v[0] = x[0]; v[1] = x[1]; v[2] = x[2]; v[3] = x[3];
  }
  static __device__ __forceinline__ float one(float v) { return v; }
};
template <> struct Pack4<bf16_t> {
  static __device__ __forceinline__ void store(bf16_t* p, float a, float b, float c, float d) {
    uint2 v;
    v.x = f32x2_to_bf16x2_bits(a, b);
    v.y = f32x2_to_bf16x2_bits(c, d);
    *reinterpret_cast<uint2*>(p) = v;
  }
  static __device__ __forceinline__ void load(const bf16_t* p, float (&v)[4]) {
    const uint2 x = *reinterpret_cast<const uint2*>(p);
    v[0] = __uint_as_float(x.x << 16); v[1] = __uint_as_float(x.x & 0xFFFF0000u);
    v[2] = __uint_as_float(x.y << 16); v[3] = __uint_as_float(x.y & 0xFFFF0000u);
  }
  static __device__ __forceinline__ bf16_t one(float v) { return bf16_t{f32_to_bf16_bits(v)}; }
};


// Whether a row counts towards the loss: its target is not the ignore index and lies in
// [0, V_total); a target outside that range that is not the ignore index is reported through `oor`.
__device__ __forceinline__ bool target_counts(int64_t y, int64_t ignore_index, int64_t V_total, bool& oor) {
  oor = false;
  if (y == ignore_index) return false;
  if (y < 0 || y >= V_total) { oor = true; return false; }
  return true;
}

// A counted target as a column of the vocabulary slice [v_begin, v_begin + Vs) that a call works
// on: its column inside the slice, or `outside` when it lies in another slice; -1 for rows that do
// not count.  The whole vocabulary as the slice is v_begin = 0, Vs = V_total.
__device__ __forceinline__ int classify_target_in_slice(int64_t y, int64_t ignore_index, int64_t V_total,
                                                        int64_t v_begin, int Vs, int outside, bool& oor) {
  if (!target_counts(y, ignore_index, V_total, oor)) return -1;
  const int64_t c = y - v_begin;
  return (c >= 0 && c < (int64_t)Vs) ? (int)c : outside;
}

// Merge of safe-softmax partials (m_k, a_k) in slot order; slots with a == 0 are
// the identity.  Returns (M, A) with A relative to M.
template <int S>
__device__ __forceinline__ void merge_fixed(const float (&m)[S], const float (&a)[S], float& M, float& A) {
  M = NEG_INF;
#pragma unroll
  for (int s = 0; s < S; ++s) if (a[s] > 0.f) M = fmaxf(M, m[s]);
  A = 0.f;
#pragma unroll
  for (int s = 0; s < S; ++s) if (a[s] > 0.f) A += a[s] * fast_exp2((m[s] - M) * LOG2E);
}

// ------------------------------------------------------------------------------------
// Forward tiles.  A = W tile (M = vocabulary, inside a lane), B = H tile (N = tokens,
// across lanes): each lane streams the logits of its own token columns and keeps
// (m, a, z_target) in registers across the vocabulary tiles of its window.
// part = [3][n_win][npad] floats: m, a, z_target per (window, row).
// ------------------------------------------------------------------------------------
// HKR: the hidden states are also given pre-tiled (HT: pack_rows_kernel's copy, zero padded to whole row
// blocks), and the main loop reads that copy: every global -> LDS request is then 1 KiB of consecutive
// bytes, where the rows of H themselves give it 64 bytes at a time.
template <typename T, typename L, bool HKR>
__global__ __launch_bounds__(L::THREADS, L::MIN_WAVES) void fwd_tiles_kernel(
    const T* __restrict__ H, const T* __restrict__ HT, const T* __restrict__ W, const int64_t* __restrict__ y,
    int N, int d, int V, int64_t ignore_index, int64_t V_total, int64_t v_begin, int n_rb, int n_win, int n_vt,
    double vt_per_win, float* __restrict__ part, int64_t npad, int item_begin, Header* __restrict__ hdr) {
  extern __shared__ __align__(16) char lds[];
  if (blockIdx.x == 0 && threadIdx.x == 0) hdr->arrived = 0;   // for the merge that follows on the stream
  // One workgroup per item (row block x window); a launch covers the items item_begin .. item_begin + gridDim.x - 1
  // of the raster (the host launches at most one round of workgroups at a time: all of them start together, and the
  // workgroups of an XCD stay close enough to each other to share the operands of their raster patch in its L2).
  const int id = item_begin + xcd_contiguous_id(blockIdx.x, gridDim.x);
  int rb, win;
  grouped_raster(id, n_rb, n_win, FLCE_FWD_GROUP, rb, win);
  // The tiles of window `win`, spread evenly; vt_per_win = n_vt / n_win, so that no division is on the way to the first load
  // (two of 64 bits before; with the launch arguments in registers 334 x 320 x 2142 forward 14.4 -> 13.7 us, fp32
  // 256 x 256 x 4096 36.8 -> 35.4).  Both sides of a boundary come from the same expression, the last one is n_vt.
  const int vt_begin = __builtin_amdgcn_readfirstlane((int)(win * vt_per_win));
  const int vt_end = win + 1 < n_win ? __builtin_amdgcn_readfirstlane((int)((win + 1) * vt_per_win)) : n_vt;
  const int n0 = rb * L::TILE;
  const int64_t ld_bytes = (int64_t)d * sizeof(T);

  int64_t yj[L::WN];
  int tgt[L::WN];
  float m[L::WN], a[L::WN], zt[L::WN];
#pragma unroll
  for (int j = 0; j < L::WN; ++j) {
    yj[j] = y[min(n0 + L::tile_n(j), N - 1)];
    m[j] = NEG_INF; a[j] = 0.f; zt[j] = 0.f;
  }
  // Small tuned tiles look at the targets near the end of the first tile: a wait for them here comes before the first operands
  // are requested (334 x 320 x 2142, one tile per workgroup, 8.15 -> 7.8 us).  The others walk many tiles and have no
  // scalar registers for it.
  constexpr bool LATE = L::TUNED && L::TILE < TILE;
  auto classify = [&] {
#pragma unroll
    for (int j = 0; j < L::WN; ++j) {
      asm volatile("" : "+v"(yj[j]));
      bool oor;
      // W holds the V vocabulary rows [v_begin, v_begin + V) of V_total; a target in another slice matches no column
      tgt[j] = n0 + L::tile_n(j) < N ? classify_target_in_slice(yj[j], ignore_index, V_total, v_begin, V, -1, oor) : -1;
    }
  };

  if constexpr (!LATE) classify();
  typename L::Acc acc;
  // The tuned loop's first K stages of tile t+1 are requested before the softmax update of tile t (which touches
  // no memory), so the update hides their latency: it matters when the K loop is short (small d).
  typename L::template Stream<HKR> stream;
  if (vt_begin < vt_end) stream.start(W, ld_bytes, vt_begin * L::TILE, V, H, HT, ld_bytes, n0, N, d, lds);
  for (int vt = vt_begin; vt < vt_end; ++vt) {
    const int v0 = vt * L::TILE;
    stream.run(lds, acc, [&] {
      if constexpr (LATE) { if (vt == vt_begin) classify(); }
      if (vt + 1 < vt_end) stream.start(W, ld_bytes, v0 + L::TILE, V, H, HT, ld_bytes, n0, N, d, lds);
    });

    // Online update of (m, a) and the target gather, one accumulator block at a time
    // (16 logits of one token per lane).  All rows of a block belong to one wavefront, so
    // "entirely behind the vocabulary's end" and "straddles the end" are wave-uniform tests;
    // padded rows count as logits of -inf.
#pragma unroll
    for (int j = 0; j < L::WN; ++j) {
#pragma unroll
      for (int i = 0; i < L::WM; ++i) {
        const int blk0 = v0 + __builtin_amdgcn_readfirstlane(L::tile_m(i, 0) & ~(L::ROWS - 1));   // first row of the block
        if (blk0 >= V) continue;
        float z[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) z[r] = acc.get(i, j, r);
        // Row of register r inside its block: QUAD * (r / 4) + (r % 4), a constant, plus what the lane adds (the MFMA's
        // accumulator layout); comparisons are written against the constant.
        const int lrow = L::lane_row();
        if (blk0 + L::ROWS > V) {
          const int live = V - blk0 - lrow;                 // rows of this block below the vocabulary's end, for this lane
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if ((r >> 2) * L::QUAD + (r & 3) >= live) z[r] = NEG_INF;
        }
        float bmax = z[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) bmax = fmaxf(bmax, z[r]);
        const float mn = fmaxf(m[j], bmax);
        const float ms = (mn == NEG_INF) ? 0.f : mn;     // nothing but padding so far: keep exp arguments finite
        const float msl = -ms * LOG2E;                   // exp(z - ms) = 2^(z * log2e - ms * log2e): one fma per logit
        float sum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) sum += fast_exp2(fmaf(z[r], LOG2E, msl));
        a[j] = a[j] * fast_exp2((m[j] - ms) * LOG2E) + sum;
        m[j] = mn;

        const int rel = tgt[j] - blk0;                    // target row inside this block, if any
        const bool mine = (unsigned)rel < (unsigned)L::ROWS && tgt[j] >= 0;
        if (__ballot(mine) != 0ull) {
          const int rell = rel - lrow;
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (mine && (r >> 2) * L::QUAD + (r & 3) == rell) zt[j] = z[r];
        }
        // one block at a time in VGPRs
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // SLOTS lanes hold partial state of each token (2 M-wavefronts x the lanes of one that share a column):
  // merge them in fixed slot order through LDS (free after the main loop's last barrier).
  constexpr int S = L::SLOTS;
  float* sm = reinterpret_cast<float*>(lds);
  float* sa = sm + S * L::TILE;
  float* sz = sa + S * L::TILE;
  {
    const int slot = L::slot();
#pragma unroll
    for (int j = 0; j < L::WN; ++j) {
      const int tok = L::tile_n(j);
      sm[slot * L::TILE + tok] = m[j];
      sa[slot * L::TILE + tok] = a[j];
      sz[slot * L::TILE + tok] = zt[j];
    }
  }
  __syncthreads();
  if (threadIdx.x < L::TILE) {
    const int tok = threadIdx.x;
    float pm[S], pa[S];
    float z = 0.f;
#pragma unroll
    for (int s = 0; s < S; ++s) { pm[s] = sm[s * L::TILE + tok]; pa[s] = sa[s * L::TILE + tok]; z += sz[s * L::TILE + tok]; }
    float M, A;
    merge_fixed<S>(pm, pa, M, A);
    const int64_t o = (int64_t)win * npad + n0 + tok;
    part[o] = M;
    part[(int64_t)n_win * npad + o] = A;
    part[2 * (int64_t)n_win * npad + o] = z;
  }
}

// Sum over the 64 lanes of a wavefront in a fixed tree (every lane gets it).
template <typename V>
__device__ __forceinline__ V wave_sum(V v) {
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) v += __shfl_xor(v, s, 64);
  return v;
}

// The partials (m, a, z_target) of a row's `n_parts` windows or vocabulary slices, merged (part k of row n at
// pm[k * stride + n], likewise pa, pz).  A block has ROWS rows x GROUPS threads; group g takes a contiguous run of the
// parts, U of them at a time with all their loads in flight together (a part past the end re-reads the last one and is
// not used), and the groups' results are merged through LDS in group order: every sum has a fixed order.
// What bounds it is memory latency: the parts of one row lie in different memory rows, and where there are many parts
// there are few rows (row blocks x windows are a few rounds of workgroups): a thread per row took 45 us for 77 rows of 197 windows and
// 40 us for 500 rows of 128 windows, 16 threads per row with 16 loads each take 7.9 and 9.8 us (the loss included).
// Returns with the row's (M, A, z) valid in the threads of group 0.
template <int ROWS, int GROUPS, int U>
__device__ __forceinline__ void merge_parts(const float* __restrict__ pm, const float* __restrict__ pa,
                                            const float* __restrict__ pz, int n_parts, int64_t stride, int n, int N,
                                            float& M, float& A, float& z) {
  const int g = threadIdx.x / ROWS;
  const int per = (n_parts + GROUPS - 1) / GROUPS;
  const int w_end = min(n_parts, (g + 1) * per);
  M = NEG_INF; A = 0.f; z = 0.f;
  if (n < N) {
    for (int w0 = g * per; w0 < w_end; w0 += U) {
      float mw[U], aw[U], zw[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t o = (int64_t)min(w0 + u, w_end - 1) * stride + n;
        mw[u] = pm[o]; aw[u] = pa[o]; zw[u] = pz[o];
      }
      float Mn = M;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (w0 + u < w_end && aw[u] > 0.f) Mn = fmaxf(Mn, mw[u]);
      if (A > 0.f) A *= fast_exp2((M - Mn) * LOG2E);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (w0 + u < w_end) {
          if (aw[u] > 0.f) A += aw[u] * fast_exp2((mw[u] - Mn) * LOG2E);
          z += zw[u];
        }
      M = Mn;
    }
  }
  if constexpr (GROUPS > 1) {
    __shared__ float sm[GROUPS][ROWS], sa[GROUPS][ROWS], sz[GROUPS][ROWS];
    const int t = threadIdx.x % ROWS;
    sm[g][t] = M; sa[g][t] = A; sz[g][t] = z;
    __syncthreads();
    if (g == 0) {
      float gm[GROUPS], ga[GROUPS];
      z = 0.f;
#pragma unroll
      for (int k = 0; k < GROUPS; ++k) { gm[k] = sm[k][t]; ga[k] = sa[k][t]; z += sz[k][t]; }
      merge_fixed<GROUPS>(gm, ga, M, A);
    }
  }
}

// Where the reduced loss of a call goes.
struct LossOut {
  float* blk_loss; int* blk_cnt; int* blk_oor;      // one entry per block of the merge
  Header* hdr; float* loss; int mean;
  int32_t* status; int64_t* n_valid;                // the caller's own words, or null
};

// The call's loss, by one thread: normalisation, header.
__device__ __forceinline__ void write_loss(const LossOut& o, double total, int64_t nv, int any) {
  double loss = total;
  if (o.mean) loss = nv > 0 ? total / (double)nv : 0.0;
  o.hdr->status = any ? 4 : 0;
  o.hdr->pad0 = 0;
  o.hdr->n_valid = nv;
  o.hdr->loss_sum = (float)total;
  *o.loss = (float)loss;
  if (o.status) *o.status = any ? 4 : 0;
  if (o.n_valid) *o.n_valid = nv;
}

// The second half of the reduction, by one block: fixed-order fp64 sum of the per-block partials.
__device__ __forceinline__ void finalize_loss(const LossOut& o, int n_blk) {
  __shared__ double sl[16];
  __shared__ long long sc[16];
  __shared__ int so[16];
  double l = 0.0; long long c = 0; int bad = 0;
  for (int b = threadIdx.x; b < n_blk; b += blockDim.x) {
    // (written by other blocks of this launch when the merge calls this: read past this XCD's own caches)
    l += (double)__hip_atomic_load(o.blk_loss + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    c += __hip_atomic_load(o.blk_cnt + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bad |= __hip_atomic_load(o.blk_oor + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  l = wave_sum(l); c = wave_sum(c); bad = __ballot(bad != 0) != 0ull;
  const int wave = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
  if ((threadIdx.x & 63) == 0) { sl[wave] = l; sc[wave] = c; so[wave] = bad; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double total = 0.0; long long nv = 0; int any = 0;
    for (int w = 0; w < n_waves; ++w) { total += sl[w]; nv += sc[w]; any |= so[w]; }
    write_loss(o, total, nv, any);
  }
}

// lse = M + ln A, loss_i = lse - z_target for counted rows (optionally label-smoothed and written out
// per row); per-block sums in a fixed tree, and the call's loss from them: by the block that hands its sums in last
// (hdr->arrived, zeroed by the forward's tile kernel; whichever block that is, it adds all of them in block order), or,
// when `fused` is 0, by finalize_loss_kernel.  A chain of memory latencies: the targets are loaded beside the parts, and the sums go
// to the other blocks by stores that pass the XCD's caches themselves, waited for before the count, so that
// neither a write-back nor an invalidation of a cache stands between (one block, 40 rows of 238 windows: 7.8 -> 5.7 us; several blocks: level).  One launch instead of three (the sum and the copy of the header to the
// caller's words each took 4.7 us, nearly all of it the launch).
template <int ROWS, int GROUPS, int U>
__global__ __launch_bounds__(ROWS * GROUPS) void merge_rows_kernel(
    const float* __restrict__ pm, const float* __restrict__ pa, const float* __restrict__ pz, int n_parts,
    int64_t stride, const int64_t* __restrict__ y, int N, int64_t V_total, int64_t ignore_index,
    float* __restrict__ lse_out, LossOut o, int fused, float* __restrict__ loss_rows_out,
    const float* __restrict__ zbar, float eps) {
  constexpr int WAVES = ROWS / 64;     // of group 0
  __shared__ float sl[WAVES];
  __shared__ int sc[WAVES], so[WAVES], last;
  const int n = blockIdx.x * ROWS + threadIdx.x % ROWS;
  float M, A, z;
  int64_t target = 0;
  float mean_z = 0.f;
  if (threadIdx.x < ROWS && n < N) {
    target = y[n];
    if (zbar) mean_z = zbar[n];
  }
  merge_parts<ROWS, GROUPS, U>(pm, pa, pz, n_parts, stride, n, N, M, A, z);
  if (threadIdx.x < ROWS) {
    float loss = 0.f;
    bool counts = false, oor = false;
    if (n < N) {
      const float lse = M + logf(A);
      lse_out[n] = lse;
      counts = target_counts(target, ignore_index, V_total, oor);
      if (counts) {
        loss = lse - z;
        // label smoothing: the target distribution keeps 1 - eps on y_i and spreads eps evenly, so
        // the row's loss mixes in eps * (lse - mean_v Z_iv)
        if (zbar) loss = (1.f - eps) * loss + eps * (lse - mean_z);
      }
      if (loss_rows_out) loss_rows_out[n] = loss;
    }
    loss = wave_sum(loss);
    const int cnt = __popcll(__ballot(counts)), bad = __ballot(oor) != 0ull;
    if ((threadIdx.x & 63) == 0) { const int w = threadIdx.x >> 6; sl[w] = loss; sc[w] = cnt; so[w] = bad; }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float l = 0.f;
    int c = 0, bad = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) { l += sl[w]; c += sc[w]; bad |= so[w]; }
    last = 0;
    if (fused && gridDim.x == 1) {
      write_loss(o, l, c, bad);
    } else {
      __hip_atomic_store(o.blk_loss + blockIdx.x, l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(o.blk_cnt + blockIdx.x, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(o.blk_oor + blockIdx.x, bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (fused) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the three stores have reached the point the other XCDs read from
        last = __hip_atomic_fetch_add(&o.hdr->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
      }
    }
  }
  __syncthreads();
  if (last) finalize_loss(o, gridDim.x);
}

__global__ __launch_bounds__(256) void finalize_loss_kernel(LossOut o, int n_blk) { finalize_loss(o, n_blk); }

// 16 bytes of the storage type as floats.
template <typename T>
struct Vec16 {
  static constexpr int N = 16 / (int)sizeof(T);
  static __device__ __forceinline__ void load(const T* p, float (&v)[N]) {
    const u32x4 x = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (sizeof(T) == 2) { v[2 * e] = __uint_as_float(x[e] << 16); v[2 * e + 1] = __uint_as_float(x[e] & 0xFFFF0000u); }
      else v[e] = __uint_as_float(x[e]);
    }
  }
};

// mean_v Z_iv = H_i . (sum_v W_v) / V, for label smoothing: the column sums of W in two fixed-order
// steps (1024-row chunks, then the chunks in order), then one dot product per row.
// The first step is one read of W, bound by memory.  grid (ceil(V / 1024), ceil(d / columns)): a block takes 1024 rows x
// 16 lanes of 16 bytes (256 consecutive bytes of a row), 16 rows at a time, each thread with 16 loads in flight.  At
// V = 32000, d = 1024 (bf16) that is 256 blocks and 12 us; one block per chunk of rows, a thread walking all 1024
// of them, took 286 us.
template <typename T>
__global__ __launch_bounds__(256) void colsum_chunks_kernel(const T* __restrict__ W, int V, int d,
                                                            float* __restrict__ wpart) {
  constexpr int VEC = Vec16<T>::N, U = 16;
  __shared__ float sh[16][16 * VEC + 4];
  const int cl = threadIdx.x & 15, rl = threadIdx.x >> 4;
  const int m = (blockIdx.y * 16 + cl) * VEC;               // d is a multiple of 8: a lane is inside or outside
  const int r0 = blockIdx.x * 1024, r1 = min(V, r0 + 1024);
  float acc[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
  if (m < d) {
    int r = r0 + rl;
    for (; r + (U - 1) * 16 < r1; r += U * 16) {
      float v[U][VEC];
#pragma unroll
      for (int u = 0; u < U; ++u) Vec16<T>::load(W + (int64_t)(r + u * 16) * d + m, v[u]);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] += v[u][e];
    }
    for (; r < r1; r += 16) {
      float v[VEC];
      Vec16<T>::load(W + (int64_t)r * d + m, v);
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[e] += v[e];
    }
  }
#pragma unroll
  for (int e = 0; e < VEC; ++e) sh[rl][cl * VEC + e] = acc[e];
  __syncthreads();
  const int c = threadIdx.x, col = blockIdx.y * 16 * VEC + c;
  if (c < 16 * VEC && col < d) {
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) t += sh[k][c];
    wpart[(int64_t)blockIdx.x * d + col] = t;
  }
}

__global__ __launch_bounds__(64) void colsum_finish_kernel(const float* __restrict__ wpart, int n_chunks, int d,
                                                           float* __restrict__ wsum) {
  const int m = blockIdx.x * 64 + threadIdx.x;
  if (m >= d) return;
  float acc = 0.f;
#pragma unroll 16
  for (int c = 0; c < n_chunks; ++c) acc += wpart[(int64_t)c * d + m];
  wsum[m] = acc;
}

// One wavefront per row, four rows per block.
template <typename T>
__global__ __launch_bounds__(256) void mean_logit_kernel(const T* __restrict__ H, const float* __restrict__ wsum, int N,
                                                         int d, float inv_V, float* __restrict__ zbar) {
  constexpr int VEC = Vec16<T>::N;
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (n >= N) return;
  float acc = 0.f;
  for (int m = lane * VEC; m < d; m += 64 * VEC) {
    float v[VEC];
    Vec16<T>::load(H + (int64_t)n * d + m, v);
#pragma unroll
    for (int q = 0; q < VEC; q += 4) {
      const f32x4 w = *reinterpret_cast<const f32x4*>(wsum + m + q);
      acc += v[q] * w[0] + v[q + 1] * w[1] + v[q + 2] * w[2] + v[q + 3] * w[3];
    }
  }
  const float tot = wave_sum(acc);
  if (lane == 0) zbar[n] = tot * inv_V;
}

// The window merge of a call that covers one vocabulary slice: the slice's (m, a, z_target) per row,
// to be merged with the other slices' later (Section 3.2, "Model Parallelism": tensor parallelism).
template <int ROWS, int GROUPS, int U>
__global__ __launch_bounds__(ROWS * GROUPS) void merge_rows_partial_kernel(const float* __restrict__ part, int n_win,
                                                                          int64_t npad, int N,
                                                                          float* __restrict__ m_out,
                                                                          float* __restrict__ a_out,
                                                                          float* __restrict__ zt_out) {
  const int n = blockIdx.x * ROWS + threadIdx.x % ROWS;
  float M, A, z;
  merge_parts<ROWS, GROUPS, U>(part, part + (int64_t)n_win * npad, part + 2 * (int64_t)n_win * npad, n_win, npad, n, N,
                               M, A, z);
  if (threadIdx.x < ROWS && n < N) { m_out[n] = M; a_out[n] = A; zt_out[n] = z; }
}

// Backward's integer pass over the targets (exact): n_valid, the range flag, and the
// compaction map.  Rows that do not count have an all-zero row of G, so the three
// backward contractions run on the counted rows only, packed in ascending row order:
//   rowmap[c] = original row of compact row c   (c < n_valid),  -1 for c >= n_valid
//   tgt_c[c]  = its target's column in the vocabulary slice W holds (2^31 - 1, which matches no column,
//               when the target lies in another slice),           -1 for c >= n_valid
// One block; every wavefront owns a contiguous range of rows and walks it 64 consecutive rows at a time, 8 loads in
// flight; ballots count and place the rows that count, the counts of the 16 wavefronts give each range its first compact
// index.  Bound by load latency.  (Threads that walked contiguous rows of their own, one load at a time, made the step at
// 32768 x 128 x 4000 50 us longer and at 8192 x 256 x 8000 5 us.)
__global__ __launch_bounds__(1024) void compact_targets_kernel(const int64_t* __restrict__ y, int N, int V,
                                                               int64_t V_total, int64_t v_begin,
                                                               int64_t ignore_index, int npad,
                                                               int* __restrict__ rowmap, int* __restrict__ tgt_c,
                                                               Header* __restrict__ hdr) {
  constexpr int U = 8;
  __shared__ int sc[16], so[16];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int per = ((N + 1023) / 1024) * 64;            // rows of a wavefront's range: whole groups of 64
  const int64_t r0 = (int64_t)wave * per, r1 = min((int64_t)N, r0 + per);
  // the target of row r as classify_target_in_slice gives it, -1 past the range
  auto classify = [&](int64_t (&v)[U], int64_t r, int u, bool& oor) -> int {
    oor = false;
    if (r + u * 64 + lane >= r1) return -1;
    return classify_target_in_slice(v[u], ignore_index, V_total, v_begin, V, 0x7FFFFFFF, oor);
  };
  auto load = [&](int64_t (&v)[U], int64_t r) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (r + u * 64 < r1) v[u] = y[min(r + u * 64 + lane, (int64_t)N - 1)];
  };
  const bool once = per <= U * 64;                     // a range's targets stay in registers for the second pass
  int64_t v[U];
  int cnt = 0, bad = 0;
  for (int64_t r = r0; r < r1; r += U * 64) {
    load(v, r);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      bool oor;
      cnt += __popcll(__ballot(classify(v, r, u, oor) >= 0));
      bad |= __ballot(oor) != 0ull;
    }
  }
  if (lane == 0) { sc[wave] = cnt; so[wave] = bad; }
  __syncthreads();
  int pos = 0, total = 0, any = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) { if (w < wave) pos += sc[w]; total += sc[w]; any |= so[w]; }
  for (int64_t r = r0; r < r1; r += U * 64) {
    if (!once) load(v, r);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      bool oor;
      const int tg = classify(v, r, u, oor);
      const uint64_t m = __ballot(tg >= 0);
      if (tg >= 0) {
        const int at = pos + __popcll(m & ((1ull << lane) - 1));
        rowmap[at] = (int)(r + u * 64 + lane);
        tgt_c[at] = tg;
      }
      pos += __popcll(m);
    }
  }
  for (int cidx = total + t; cidx < npad; cidx += 1024) { rowmap[cidx] = -1; tgt_c[cidx] = -1; }
  if (t == 0) {
    hdr->status = any ? 4 : 0;
    hdr->pad0 = 0;
    hdr->n_valid = total;
    hdr->loss_sum = 0.f;
    hdr->arrived = 0;
  }
}

// The same scan inside a block of the row preparation (256 threads, N <= COMPACT_HERE rows): every block reads all targets
// (16 KiB at most, from the L2) and keeps what concerns its own ROWS compact rows c0 .. c0 + ROWS - 1, which saves the
// launch of compact_targets_kernel (4.5 us).  The blocks named by `owner` also store the map for the kernels that
// follow, one of them (`first`) the header.
constexpr int COMPACT_HERE = 2048;
struct CompactArgs {
  const int64_t* y; int N, V; int64_t V_total, v_begin, ignore_index;
  int* rowmap; int* tgt_c; Header* hdr;
};
template <int ROWS>
__device__ __forceinline__ void compact_here(const CompactArgs& a, int c0, bool owner, bool first, int (&row)[ROWS]) {
  constexpr int U = COMPACT_HERE / 256;
  __shared__ int cnt[U * 4], bad[U * 4], tgt[ROWS];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int64_t v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) v[u] = a.y[min(u * 256 + t, a.N - 1)];
  if (t < ROWS) { row[t] = -1; tgt[t] = -1; }
  int tg[U];
  uint64_t m[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    bool oor = false;
    tg[u] = u * 256 + t < a.N ? classify_target_in_slice(v[u], a.ignore_index, a.V_total, a.v_begin, a.V, 0x7FFFFFFF, oor) : -1;
    m[u] = __ballot(tg[u] >= 0);
    const bool any = __ballot(oor) != 0ull;
    if (lane == 0) { cnt[u * 4 + wave] = __popcll(m[u]); bad[u * 4 + wave] = any; }
  }
  __syncthreads();
  int pos = 0, total = 0, any = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    int mine = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) { if (w == wave) mine = total; total += cnt[u * 4 + w]; any |= bad[u * 4 + w]; }
    pos = mine + __popcll(m[u] & ((1ull << lane) - 1)) - c0;
    if (tg[u] >= 0 && pos >= 0 && pos < ROWS) { row[pos] = u * 256 + t; tgt[pos] = tg[u]; }
  }
  __syncthreads();
  if (owner && t < ROWS) { a.rowmap[c0 + t] = row[t]; a.tgt_c[c0 + t] = tgt[t]; }
  if (first && t == 0) {
    a.hdr->status = any ? 4 : 0;
    a.hdr->pad0 = 0;
    a.hdr->n_valid = total;
    a.hdr->loss_sum = 0.f;
    a.hdr->arrived = 0;
  }
}

// The backward's row preparation, one launch, 64 compact rows x 64 hidden positions per block:
//   Hc[c][:]  = H[rowmap[c]][:], zero for the padding rows behind the last counted row;
//   HcT[:][c] = the same transposed, when a main loop reads that copy (HcT != nullptr; ld_t elements per row);
//   lse_c[c], gam_c[c] = the row's log-sum-exp and (per-row variant) upstream gradient, 0 for padding rows;
//   dH[n][:]  = exactly +0 for every token n that does not count (the contractions write the counted rows only).
// U is an unsigned integer type of the element's width (pure data movement).
// SCAN: the blocks find their rows themselves (compact_here) instead of reading rowmap.
template <typename U, bool SCAN>
__global__ __launch_bounds__(256) void prep_rows_kernel(const U* __restrict__ H, int d, U* __restrict__ Hc,
                                                        U* __restrict__ HcT, int64_t ld_t,
                                                        const float* __restrict__ lse, float* __restrict__ lse_c,
                                                        const float* __restrict__ grad_rows, float* __restrict__ gam_c,
                                                        CompactArgs ca, U* __restrict__ dH) {
  __shared__ U tile[64][65];
  __shared__ int src_row[64];
  __shared__ int dead[64];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int rb = blockIdx.x * 64, cb = blockIdx.y * 64;
  if constexpr (SCAN) compact_here(ca, rb, blockIdx.y == 0, blockIdx.x == 0 && blockIdx.y == 0, src_row);
  if (threadIdx.x < 64) {
    const int r = rb + (int)threadIdx.x;               // a compact row, and also token r of the original order
    const int n = SCAN ? src_row[threadIdx.x] : ca.rowmap[r];
    src_row[threadIdx.x] = n;
    bool oor;
    dead[threadIdx.x] = (r < ca.N && !target_counts(ca.y[r], ca.ignore_index, ca.V_total, oor)) ? 1 : 0;
    if (blockIdx.y == 0) {
      lse_c[r] = (n >= 0) ? lse[n] : 0.f;
      if (grad_rows) gam_c[r] = (n >= 0) ? grad_rows[n] : 0.f;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int rr = ty + 4 * k, r = rb + rr, c = cb + tx;
    const int n = src_row[rr];
    U v = 0;
    if (c < d) {
      if (n >= 0) v = H[(int64_t)n * d + c];
      Hc[(int64_t)r * d + c] = v;
      if (dead[rr]) dH[(int64_t)r * d + c] = 0;
    }
    tile[rr][tx] = v;
  }
  if (HcT == nullptr) return;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int c = cb + ty + 4 * k, r = rb + tx;
    if (c < d) HcT[(int64_t)c * ld_t + r] = tile[tx][ty + 4 * k];
  }
}

// The pre-tiled copy of a row-major bf16 matrix X[rows][d] (d a multiple of 8) that the tuned main loop reads as
// its B operand: for every block of 256 rows and every K step of 32 elements, the 16 KiB image of that step's LDS
// tile, images of one row block following each other in K order:
//   P[(rb * d / 32 + kt) * 16 KiB + r * 64 + 16 * pos] = the 16 bytes X[rb * 256 + r][kt * 32 + 8 * (pos ^ chunk_swizzle(r)) ...]
// (the main loop's K-contiguous LDS tile, 256 rows of 64 bytes with its chunk swizzle), rows and columns past the end as zeros.
// pack_rows_store: one thread's part, the 64 bytes of row r of row block rb at K step kt.
__device__ __forceinline__ void pack_rows_store(const u32x4 (&chunk)[4], char* __restrict__ P, int rb, int kt, int d, int r) {
  u32x4* dst = reinterpret_cast<u32x4*>(P + packed_block_offset(rb, d) + (int64_t)kt * fast::OPER + r * 64);
  const int sw = fast::chunk_swizzle(r);
#pragma unroll
  for (int c = 0; c < 4; ++c) dst[c ^ sw] = chunk[c];
}

// grid (rows_pad / 64, ceil(d / 128)), 256 threads: thread t copies the 64 bytes of row 64 * blockIdx.x + t / 4 at
// K step 4 * blockIdx.y + t % 4, so that a wavefront reads 16 rows x 256 consecutive bytes and writes 1 KiB runs.
__global__ __launch_bounds__(256) void pack_rows_kernel(const char* __restrict__ X, int rows, int d,
                                                        char* __restrict__ P) {
  const int row = blockIdx.x * 64 + (threadIdx.x >> 2), kt = blockIdx.y * 4 + (threadIdx.x & 3);
  if (kt * fast::BK >= d) return;
  u32x4 chunk[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) chunk[c] = u32x4{0u, 0u, 0u, 0u};
  if (row < rows) {
    const u32x4* src = reinterpret_cast<const u32x4*>(X + ((int64_t)row * d + kt * fast::BK) * 2);
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (kt * fast::BK + c * 8 < d) chunk[c] = src[c];
  }
  pack_rows_store(chunk, P, row / TILE, kt, d, row % TILE);
}

// The backward's row preparation for the tuned loop, one launch; block (kt, q) handles the 32 compact rows of K step
// kt of the dW contraction and the 256 hidden columns of tile q (grid: rows_pad / 32 x ceil(d / 256), 256 threads):
//   HcP  = the counted rows of H, packed together (zero behind the last one), pre-tiled as pack_rows_kernel does: the
//          recompute's second operand (nullptr: not wanted);
//   HcTP = the same rows pre-tiled the other way round, for the dW contraction, whose K index runs over the rows: per
//          hidden tile q and K step kt the 16 KiB LDS image [256 hidden positions][32 rows] (chunk swizzle included),
//          the images of one q following each other, block q at packed_cols_offset(q, rows_pad); hidden positions
//          past d are zeros;
//   lse_c / gam_c gathered likewise; dH rows of tokens that do not count set to exactly +0.
// SCAN: the blocks find their rows themselves (compact_here) instead of reading rowmap.
template <bool SCAN>
__global__ __launch_bounds__(256) void prep_rows_tiled_kernel(const char* __restrict__ H, int d, int rows_pad,
                                                              char* __restrict__ HcP, char* __restrict__ HcTP,
                                                              const float* __restrict__ lse, float* __restrict__ lse_c,
                                                              const float* __restrict__ grad_rows,
                                                              float* __restrict__ gam_c, CompactArgs ca,
                                                              char* __restrict__ dH) {
  __shared__ __align__(16) uint16_t tile[32][TILE + 8];     // 528-byte rows: a column read touches every bank once
  const int kt = blockIdx.x, q = blockIdx.y;
  const int rr = threadIdx.x >> 3, g = threadIdx.x & 7;    // row of the K step, group of 32 hidden positions
  const int c = kt * 32 + rr;                               // compact row c, and also token c of the original order
  const int col0 = q * TILE + g * 32;
  int n;
  if constexpr (SCAN) {
    __shared__ int src_row[32];
    compact_here(ca, kt * 32, q == 0, kt == 0 && q == 0, src_row);
    n = src_row[rr];
  } else {
    n = ca.rowmap[c];
  }
  if (q == 0 && g == 0) {
    lse_c[c] = (n >= 0) ? lse[n] : 0.f;
    if (grad_rows) gam_c[c] = (n >= 0) ? grad_rows[n] : 0.f;
  }
  u32x4 chunk[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) chunk[i] = u32x4{0u, 0u, 0u, 0u};
  if (col0 < d) {                                           // d is a multiple of 8: a 16-byte chunk is inside or outside
    if (n >= 0) {
      const u32x4* src = reinterpret_cast<const u32x4*>(H + ((int64_t)n * d + col0) * 2);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (col0 + i * 8 < d) chunk[i] = src[i];
    }
    if (HcP) pack_rows_store(chunk, HcP, c / TILE, col0 / fast::BK, d, c % TILE);
    bool oor;
    if (c < ca.N && !target_counts(ca.y[c], ca.ignore_index, ca.V_total, oor)) {
      u32x4* z = reinterpret_cast<u32x4*>(dH + ((int64_t)c * d + col0) * 2);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (col0 + i * 8 < d) z[i] = u32x4{0u, 0u, 0u, 0u};
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4*>(&tile[rr][g * 32 + i * 8]) = chunk[i];
  __syncthreads();
  // thread m: the 32 rows' values at hidden position q * 256 + m, as the 64 bytes of row m of the image
  const int m = threadIdx.x, sw = fast::chunk_swizzle(m);
  u32x4* dst = reinterpret_cast<u32x4*>(HcTP + packed_cols_offset(q, rows_pad) + (int64_t)kt * fast::OPER + m * 64);
#pragma unroll
  for (int ch = 0; ch < 4; ++ch) {
    u32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      v[e] = (uint32_t)tile[ch * 8 + 2 * e][m] | ((uint32_t)tile[ch * 8 + 2 * e + 1][m] << 16);
    dst[ch ^ sw] = v;
  }
}

// dst[c][r] = src[r0 + r][c]  for c < cols, r < rows_pad; zero where r0 + r >= rows_total.
// U is an unsigned integer type of the element's width (pure data movement).
template <typename U>
__global__ __launch_bounds__(256) void transpose_pad_kernel(const U* __restrict__ src, int64_t ld_src, int rows_total,
                                                            int r0, int cols, U* __restrict__ dst, int64_t ld_dst,
                                                            int rows_pad) {
  __shared__ U tile[64][65];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int rb = blockIdx.x * 64, cb = blockIdx.y * 64;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int r = rb + ty + 4 * k, c = cb + tx;
    U v = 0;
    if (r < rows_pad && r0 + r < rows_total && c < cols) v = src[(int64_t)(r0 + r) * ld_src + c];
    tile[ty + 4 * k][tx] = v;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int c = cb + ty + 4 * k, r = rb + tx;
    if (c < cols && r < rows_pad) dst[(int64_t)c * ld_dst + r] = tile[tx][ty + 4 * k];
  }
}

// ------------------------------------------------------------------------------------
// Backward, step 1 (on the compacted rows): logit tile recomputed exactly as in the
// forward (the same products added up in the same order; fp32 on the same tile edge, see plan_base), then
//   g = exp(z - lse_row) - [v == y_row]            (unscaled; Gamma comes later)
// rounded to T and written to the staging tile
//   G [row - chunk_n0][vocab - chunk_v0]   (ldG  elements per row; with the tuned loop in blocks of 16 rows x 32
//                                           positions of 1 KiB, ldG = BYTES from one group of 16 rows to the next)
// and, for main loops that need K-contiguous operands, also transposed:
//   GT[vocab - chunk_v0][row - chunk_n0]   (ldGT elements per row)
// Padded vocabulary columns and the padding rows behind the last counted row are 0.
// Tiles that lie entirely behind the last counted row return at once; the
// contractions never read them.
// ------------------------------------------------------------------------------------
template <typename T>
struct RecomputeArgs {
  const T* Hc; const T* HcT; const T* W; const int* tgt_c; const float* lse_c; const Header* hdr;
  int npad, d, V, nt0, n_nt, vt0, n_vt;
  T* G; int64_t ldG; T* GT; int64_t ldGT;
  // per-row variant only: upstream gradient of each compact row, label-smoothing constants
  const float* gam_c; float onehot_weight; float uniform_part;   // 1 - eps, eps / V
};

// Per-row inputs of a recompute tile, one set per token column a lane owns.
template <typename L>
struct RowMeta {
  int tgt[L::WN];       // target column inside the slice, -1 for a padding row
  float lse[L::WN];
  float gam[L::WN];     // per-row variant only
};

// The recompute step.  With the tuned loop the launch has at most one round of workgroups (NUM_CU * L::PER_CU: 256 with
// 256-row tiles, 512 with 128-row ones) and workgroup b takes tiles b, b + gridDim.x, ... of the chunk; with the other loops
// it has one per tile.  With the tuned loop the first K stages of a workgroup's next tile (and that tile's per-row inputs) are
// requested before the current tile's G is formed and stored, so the latency of a tile's first operands hides behind
// the previous tile's post-processing: it matters when the K loop is short (small d).
// PER_ROW: g = Gamma_row * (p - (1 - eps) [v == y_row] - eps / V), the upstream gradient applied here because
// it differs from row to row (Alg. 2 with a per-position Gamma); otherwise g = p - [v == y_row] and the
// scalar Gamma is applied when the contractions write out.
template <typename T, typename L, bool HKR, bool PER_ROW = false>
__global__ __launch_bounds__(L::THREADS, L::MIN_WAVES) void recompute_kernel(RecomputeArgs<T> a) {
  extern __shared__ __align__(16) char lds[];
  const T* __restrict__ Hc = a.Hc; const T* __restrict__ HcT = a.HcT; const T* __restrict__ W = a.W;
  const int npad = a.npad, d = a.d, V = a.V;
  T* __restrict__ G = a.G; T* __restrict__ GT = a.GT; const int64_t ldG = a.ldG, ldGT = a.ldGT;
  // Only the row tiles that hold counted rows are rastered (their number is known on the device
  // alone), so the XCDs share the work evenly however many rows are ignored; workgroups beyond the
  // useful tiles of a launch sized for N rows leave at once.
  const int n_nt = max(0, min(a.n_nt, ((int)a.hdr->n_valid - a.nt0 * L::TILE + L::TILE - 1) / L::TILE));
  const int useful = n_nt * a.n_vt;
  int t = blockIdx.x;
  if (t >= useful) return;
  const int64_t ld_bytes = (int64_t)d * sizeof(T);
  auto place = [&](int tile, int& p, int& q) {     // row tile, vocabulary tile inside the chunk
    grouped_raster(xcd_contiguous_id(tile, useful), n_nt, a.n_vt, 8, p, q);
  };
  auto load_meta = [&](int n0, RowMeta<L>& m) {
#pragma unroll
    for (int j = 0; j < L::WN; ++j) {
      const int n = n0 + L::tile_n(j);
      m.tgt[j] = a.tgt_c[n];
      m.lse[j] = a.lse_c[n];
      if constexpr (PER_ROW) m.gam[j] = a.gam_c[n];
    }
  };
  // Marks the point where a tile's per-row inputs must have arrived: the compiler's wait for them lands here (it
  // cannot see the main loop's own requests, so a wait placed later would also wait for the next tile's operands).
  auto need_meta = [&](RowMeta<L>& m) {
#pragma unroll
    for (int j = 0; j < L::WN; ++j) {
      asm volatile("" : "+v"(m.tgt[j]), "+v"(m.lse[j]));
      if constexpr (PER_ROW) asm volatile("" : "+v"(m.gam[j]));
    }
  };
  typename L::template Stream<HKR> stream;
  int p, q;
  place(t, p, q);
  RowMeta<L> meta;
  if constexpr (L::TUNED) load_meta((a.nt0 + p) * L::TILE, meta);
  stream.start(W, ld_bytes, (a.vt0 + q) * L::TILE, V, Hc, HcT, ld_bytes, (a.nt0 + p) * L::TILE, npad, d, lds);
  typename L::Acc acc;
  for (;;) {
    const int t_next = t + gridDim.x;
    // (a main loop with nothing to request ahead gets one tile per workgroup)
    const bool more = L::TUNED && t_next < useful;
    int p_next = 0, q_next = 0;
    RowMeta<L> meta_next;
    stream.run(lds, acc, [&] {
      if constexpr (!L::TUNED) load_meta((a.nt0 + p) * L::TILE, meta);   // no registers to spare across that main loop
      need_meta(meta);
      if (more) {
        place(t_next, p_next, q_next);
        load_meta((a.nt0 + p_next) * L::TILE, meta_next);
        stream.start(W, ld_bytes, (a.vt0 + q_next) * L::TILE, V, Hc, HcT, ld_bytes, (a.nt0 + p_next) * L::TILE, npad, d, lds);
      }
    });

    const int v0 = (a.vt0 + q) * L::TILE;
    if constexpr (L::TUNED) {
      // Tuned loop.  A lane holds, of 16 token rows x (32 B) vocabulary positions per j, scattered 8-byte pieces of one
      // row; stored as they lie, every store instruction would touch 16 different memory rows in 32-byte pieces.  Each wavefront
      // therefore passes its piece (4 KiB of bf16 with 256-row tiles) through its own slice of the free LDS stage and
      // writes whole blocks of G, 1 KiB of consecutive bytes per instruction.
      static_assert(sizeof(T) == 2, "the tuned epilogue is laid out for bf16");
      constexpr int POS = L::WM * L::ROWS;                        // vocabulary positions of a piece
      const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
      char* stage = lds + L::FREE_LDS_OFFSET + wave * (16 * L::ROW_BYTES);
      const int wrow = lane & 15;                                 // writer: token row of the piece
      const int rrow = lane >> 2, rchunk = lane & 3;              // reader: row and 16-byte chunk inside a block
      const int vbase = v0 + (wave >> 1) * POS;                   // first vocabulary position of the piece
#pragma unroll
      for (int j = 0; j < L::WN; ++j) {
        const int tgt = meta.tgt[j];
        // exp(z - lse) = 2^(z * log2e - lse * log2e); a padding row (tgt < 0) gets lse = +inf here, so its p is
        // exactly 0, and no column equals its target: its row of G is 0 without a mask
        const float ll = tgt >= 0 ? -meta.lse[j] * LOG2E : NEG_INF;
        float gam = 1.f;
        if constexpr (PER_ROW) gam = tgt >= 0 ? meta.gam[j] : 0.f;
        const float unif = tgt >= 0 ? a.uniform_part : 0.f;
        // A whole column of blocks without a target of the wavefront and inside the vocabulary (almost all are: POS of V
        // positions) needs no tests (step of 4326 x 232 x 74697 1044 -> 1008 us, 1144 x 576 x 191782 1306 -> 1264,
        // 4096 x 768 x 50257 1198 -> 1178).
        if (vbase + POS <= V && __ballot((unsigned)(tgt - vbase) < (unsigned)POS) == 0ull) {
#pragma unroll
          for (int i = 0; i < L::WM; ++i) {
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
              float g[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                g[e] = fast_exp2(fmaf(acc.get(i, j, rq * 4 + e), LOG2E, ll));
                if constexpr (PER_ROW) g[e] = gam * (g[e] - unif);
              }
              uint2 packed;
              packed.x = f32x2_to_bf16x2_bits(g[0], g[1]);
              packed.y = f32x2_to_bf16x2_bits(g[2], g[3]);
              *reinterpret_cast<uint2*>(stage + L::piece_slot(wrow, i, rq)) = packed;
            }
            __builtin_amdgcn_sched_barrier(0);   // one accumulator block at a time in VGPRs
          }
        } else {
#pragma unroll
          for (int i = 0; i < L::WM; ++i) {
            const int blk0 = vbase + i * L::ROWS;                   // wave-uniform
            const bool whole = blk0 + L::ROWS <= V;
            // Does any token column of this wavefront have its target among the block's vocabulary positions?
            // Almost never, and then the one-hot term costs nothing: a wave-uniform branch.
            const bool hit = __ballot((unsigned)(tgt - blk0) < (unsigned)L::ROWS) != 0ull;
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
              const int vpos = blk0 + rq * L::QUAD + L::lane_row();   // first of this lane's 4 consecutive positions
              float g[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) g[e] = fast_exp2(fmaf(acc.get(i, j, rq * 4 + e), LOG2E, ll));
              if (hit) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                  if (vpos + e == tgt) g[e] -= PER_ROW ? a.onehot_weight : 1.f;
              }
              if constexpr (PER_ROW) {
#pragma unroll
                for (int e = 0; e < 4; ++e) g[e] = gam * (g[e] - unif);
              }
              if (!whole) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                  if (vpos + e >= V) g[e] = 0.f;
              }
              uint2 packed;
              packed.x = f32x2_to_bf16x2_bits(g[0], g[1]);
              packed.y = f32x2_to_bf16x2_bits(g[2], g[3]);
              *reinterpret_cast<uint2*>(stage + L::piece_slot(wrow, i, rq)) = packed;
            }
            __builtin_amdgcn_sched_barrier(0);   // one accumulator block at a time in VGPRs
          }
        }
        // the piece is complete in LDS (a wavefront's LDS operations complete in order): write it out, a block at a
        // time.  G is stored in blocks of 16 rows x 32 positions (1 KiB; the blocks of a row
        // group along the vocabulary, row groups ldG BYTES apart), so that both contractions fetch whole blocks.
        const int row0 = p * L::TILE + (wave & 1) * (L::WN * 16) + j * 16;          // a row group
        char* __restrict__ gdst = reinterpret_cast<char*>(G) + (int64_t)(row0 >> 4) * ldG +
                                  (int64_t)(q * (L::TILE / 32) + (wave >> 1) * (POS / 32)) * 1024 + lane * 16;
#pragma unroll
        for (int k = 0; k < POS / 32; ++k)
          *reinterpret_cast<u32x4*>(gdst + k * 1024) = *reinterpret_cast<const u32x4*>(stage + L::piece_chunk(rrow, k * 4 + rchunk));
      }
    } else {
    // Blocks in (i, j) order, i outermost: what depends on the vocabulary position only (the padding masks of a
    // block that straddles the vocabulary's end) is then shared by the four j of one i and dies with it.
#pragma unroll
    for (int i = 0; i < L::WM; ++i) {
      // All 32 vocabulary positions of a block belong to one wavefront: "behind the vocabulary's end" and
      // "straddles the end" are wave-uniform tests, and only a straddling block masks single elements.
      const int blk0 = v0 + __builtin_amdgcn_readfirstlane(L::tile_m(i, 0) & ~31);
      const bool whole = blk0 + 32 <= V;
#pragma unroll
      for (int j = 0; j < L::WN; ++j) {
        const int nl = p * L::TILE + L::tile_n(j);       // row inside the staging tile
        // this lane's first position in the row; block (i, rq) lies a constant 32 i + 8 rq further on
        T* __restrict__ grow = G + (int64_t)nl * ldG + q * L::TILE + L::tile_m(0, 0);
        const int tgt = meta.tgt[j];
        // exp(z - lse) = 2^(z * log2e - lse * log2e); a padding row (tgt < 0) gets lse = +inf here, so its p is
        // exactly 0, and no column equals its target: its row of G is 0 without a mask
        const float ll = tgt >= 0 ? -meta.lse[j] * LOG2E : NEG_INF;
        float gam = 1.f;
        if constexpr (PER_ROW) gam = tgt >= 0 ? meta.gam[j] : 0.f;
        const float unif = tgt >= 0 ? a.uniform_part : 0.f;
        // Does any token column of this wavefront have its target among the block's 32 vocabulary positions?
        // Almost never (32 of V positions), and then the one-hot term costs nothing: a wave-uniform branch.
        const bool hit = __ballot((unsigned)(tgt - blk0) < 32u) != 0ull;
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          const int mloc = L::tile_m(i, rq * 4);    // first of 4 consecutive vocabulary positions
          float g[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) g[e] = fast_exp2(fmaf(acc.get(i, j, rq * 4 + e), LOG2E, ll));
          if (hit) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (v0 + mloc + e == tgt) g[e] -= PER_ROW ? a.onehot_weight : 1.f;
          }
          if constexpr (PER_ROW) {
#pragma unroll
            for (int e = 0; e < 4; ++e) g[e] = gam * (g[e] - unif);
          }
          if (!whole) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (v0 + mloc + e >= V) g[e] = 0.f;
          }
          const int vl = q * L::TILE + mloc;
          Pack4<T>::store(grow + (i * 32 + rq * 8), g[0], g[1], g[2], g[3]);
          if constexpr (!L::TRANSPOSING) {
#pragma unroll
            for (int e = 0; e < 4; ++e) GT[(int64_t)(vl + e) * ldGT + nl] = Pack4<T>::one(g[e]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);   // one 32x32 block at a time in VGPRs
      }
    }
    }
    if (!more) break;
    need_meta(meta_next);
    t = t_next; p = p_next; q = q_next;
    meta = meta_next;
  }
}

// ------------------------------------------------------------------------------------
// Backward, step 2: out[n][m] (+)= sum_k A[m][k] * B[n][k]
//   dH: A = W^T chunk [d][Vc], B = G  [rows][Vc]   (contraction over the vocabulary chunk)
//   dW: A = Hc^T      [d][Nc], B = GT [vocab][Nc]  (contraction over the compact-row chunk)
// M = hidden index, so each lane owns 4 consecutive output elements of one row.
// Chunks are accumulated in fp32 in a fixed order: READ_ACC adds the running sum,
// WRITE_ACC stores it back, WRITE_OUT multiplies by Gamma and rounds to T.
// ROWS_COMPACT (dH): output rows are compact rows; tiles behind the last counted row
// return at once and row c is written to out[rowmap[c]].
// K_COMPACT (dW): the contraction runs over compact rows k_start .. k_start + k_elems and
// stops at the last counted row (rounded up to a whole K step of 32; that padding is zero.  Whole tiles
// cost up to 255 rows of K more: 350 counted rows x 4096 x 128256 1878 -> 1798 us per step, 331 x 3136 x 102294 1282 -> 1219).
// ------------------------------------------------------------------------------------
//
// OPS selects how the operands lie in memory:
//   OPS_KC    : A[m][k], B[n][k] both K-contiguous (the transposed copies W^T, Hc^T, GT)
//   OPS_DH_TR : A = W rows of the vocabulary chunk [k][m] (K over memory rows), B = G of the chunk, stored in blocks
//               of 16 rows x 32 positions (recompute_kernel; ldb = BYTES from one group of 16 rows to the next)
//   OPS_DW_TR : A = the transposed pre-tiled copy of Hc (prep_rows_tiled_kernel; lda = its padded row count, the
//               K steps of the row chunk start at image k_start / 32), B = the same blocked G, K over its rows
enum : int { READ_ACC = 1, WRITE_ACC = 2, WRITE_OUT = 4, ROWS_COMPACT = 8, K_COMPACT = 16 };
//   OPS_DH_F32 : fp32; A = W rows of the vocabulary chunk [k][m], B = G row-major [n][k]
//   OPS_DW_F32 : fp32; A = Hc rows of the row chunk [k][m], B = G row-major [k][n] (K over the rows of both)
enum : int { OPS_KC = 0, OPS_DH_TR = 1, OPS_DW_TR = 2, OPS_DH_F32 = 3, OPS_DW_F32 = 4 };

// Upstream gradient of the scalar loss: a device word if there is one, a host value otherwise.
struct GradLoss {
  float value; const float* word;
  __device__ __forceinline__ float get() const { return word ? *word : value; }
};

template <typename T>
struct ContractArgs {
  const T* A; int64_t lda; int a_krows, d;
  const T* B; int64_t ldb; int b_rows, k_elems, k_start, n_mt, n_nt;
  float* accbuf; int acc_row0;
  T* out; int out_row0, out_rows, flags;
  const Header* hdr; const int* rowmap; GradLoss grad_loss; int mean;
  // split-K (n_split > 1): the launch has n_split x tiles workgroups; slice z contracts K elements
  // [z * k_split, (z + 1) * k_split) and stores its fp32 tile into partial + z * partial_stride (indexed like
  // accbuf); splitk_reduce_kernel then adds the slices in slice order and does the READ/WRITE part of `flags`.
  int n_split, k_split; float* partial; int64_t partial_stride;
};

// With the tuned loop a launch has at most one round of workgroups (NUM_CU * L::PER_CU); workgroup b takes work items b, b + n_wg, ... (an
// item = one output tile of one K slice) and requests the first K stages of its next item before it writes out the
// current one, as the recompute step does.
// ONE: there are as many workgroups as items.
template <typename T, typename L, int OPS, bool ONE = false>
__device__ __forceinline__ void contract(const ContractArgs<T>& a, int wg, int n_wg, char* lds) {
  const T* __restrict__ A = a.A; const T* __restrict__ B = a.B;
  const int64_t lda = a.lda, ldb = a.ldb;
  const int d = a.d;
  T* __restrict__ out = a.out;
  const int nv = (int)a.hdr->n_valid;
  // With compacted output rows only the row tiles that hold counted rows are rastered, so the
  // XCDs share the work evenly; surplus workgroups of the launch leave at once.
  int n_nt = a.n_nt;
  if (a.flags & ROWS_COMPACT) n_nt = max(0, min(n_nt, (nv - a.out_row0 + L::TILE - 1) / L::TILE));
  const int tiles = n_nt * a.n_mt;
  const int n_split = max(1, a.n_split);
  const int total = tiles * n_split;
  int b = wg;
  if (b >= total) return;
  int k_all = a.k_elems;
  if (a.flags & K_COMPACT) k_all = max(0, min(k_all, (nv - a.k_start + 31) / 32 * 32));   // whole K steps
  float scale = a.grad_loss.get();
  if (a.mean) scale = nv > 0 ? scale / (float)nv : 0.f;

  // item -> K slice z, output-row tile p, hidden tile q; K range [k0, k0 + k_elems) of the slice
  auto place = [&](int item, int& z, int& p, int& q, int& k0, int& k_elems) {
    // (opaque per tile: the divisions' constants would be kept in scalar registers, which the tuned loop is short of)
    const int per_slice = fast::scalar(tiles), n_mt = fast::scalar(a.n_mt);
    z = item / per_slice;
    grouped_raster(xcd_contiguous_id(item - z * per_slice, per_slice), n_nt, n_mt, 8, p, q);
    k0 = 0; k_elems = k_all;
    if (a.n_split > 1) { k0 = z * a.k_split; k_elems = max(0, min(a.k_split, k_all - k0)); }
  };
  // output rows of the lane's token columns: the original row of a compact row, -1 = nothing to write
  auto load_rows = [&](int p, int (&orow)[L::WN]) {
#pragma unroll
    for (int j = 0; j < L::WN; ++j) {
      const int n = a.out_row0 + p * L::TILE + L::tile_n(j);
      orow[j] = -1;
      if (n < a.out_rows) orow[j] = (a.flags & ROWS_COMPACT) ? a.rowmap[n] : n;
    }
  };
  auto need_rows = [&](int (&orow)[L::WN]) {     // the compiler's wait for the loads above lands here
#pragma unroll
    for (int j = 0; j < L::WN; ++j) asm volatile("" : "+v"(orow[j]));
  };
  // Running sum / Gamma / rounding of one finished tile.
  auto flush = [&](const typename L::Acc& acc, int z, int p, int q, const int (&orow)[L::WN]) {
    int flags = a.flags;
    float* __restrict__ accbuf = a.accbuf;
    if (a.n_split > 1) {
      accbuf = a.partial + (int64_t)z * a.partial_stride;
      flags = (flags & ROWS_COMPACT) | WRITE_ACC;
    }
    // one column of blocks straight from the accumulator layout
    auto direct = [&](const typename L::Acc& acc, int j) {
      if (orow[j] < 0) return;
      const int n = a.out_row0 + p * L::TILE + L::tile_n(j);
      // this lane's first hidden position; quad (i, rq) lies a constant further on
      const int m0 = q * L::TILE + L::tile_m(0, 0);
      float* __restrict__ arow = accbuf + (int64_t)(n - a.acc_row0) * d + m0;
      T* __restrict__ orowp = out + (int64_t)orow[j] * d + m0;
#pragma unroll
      for (int i = 0; i < L::WM; ++i)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          const int c = i * L::ROWS + rq * L::QUAD;
          if (m0 + c >= d) continue;
          f32x4 v = {acc.get(i, j, rq * 4), acc.get(i, j, rq * 4 + 1), acc.get(i, j, rq * 4 + 2),
                     acc.get(i, j, rq * 4 + 3)};
          float* ap = arow + c;
          if (flags & READ_ACC) v += *reinterpret_cast<const f32x4*>(ap);
          if (flags & WRITE_ACC) *reinterpret_cast<f32x4*>(ap) = v;
          if (flags & WRITE_OUT) {
            // "+ 0.f" turns a -0 product into +0
            Pack4<T>::store(orowp + c, v[0] * scale + 0.f, v[1] * scale + 0.f, v[2] * scale + 0.f, v[3] * scale + 0.f);
          }
          if (rq == 3) __builtin_amdgcn_sched_barrier(0);   // one accumulator block at a time in VGPRs
        }
    };
    if constexpr (L::TUNED) {
      // The rounded output: in the accumulator layout a store instruction would touch 16 output rows with 32 bytes each.
      // As in the recompute step, each wavefront passes 16 rows x 256 bytes at a time through its slice of the free LDS
      // stage and writes whole 256-byte runs, 4 rows per instruction.
      // It matters where the K loop is short: dW at 500 tokens x 4096 x 128256 807 -> 750 us (the K loops alone take 479),
      // the step at 1000 x 2048 x 100000 1616 -> 1528 us; at 8192 tokens it changes nothing.  The fp32 sums gain nothing
      // from the detour (64 bytes per row as they lie) and go out directly.
      static_assert(sizeof(T) == 2, "laid out for bf16");
      constexpr int RPS = L::ROWS_PER_STORE;
      const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
      char* stage = lds + L::FREE_LDS_OFFSET + wave * (16 * L::ROW_BYTES);
      const int wrow = lane & 15;                                 // writer: output row of the piece
      const int rrow = lane / L::CHUNKS, rpos = lane % L::CHUNKS;   // reader: row within a store, place of a 16-byte chunk
      const int mw = q * L::TILE + (wave >> 1) * (L::WM * L::ROWS);   // first hidden position of the wavefront's columns
      // output row of piece row r: rows of dW follow each other, rows of dH go where the compact rows came from
      auto row_of = [&](int j, int r) -> int {
        if constexpr (OPS == OPS_DH_TR) return __shfl(orow[j], r, 64);
        const int n = a.out_row0 + p * L::TILE + (wave & 1) * (L::WN * 16) + j * 16 + r;
        return n < a.out_rows ? n : -1;
      };
      if (mw >= d) return;                                        // all of the wavefront's columns lie past the hidden size
#pragma unroll
      for (int j = 0; j < L::WN; ++j) {
        if (!(flags & (READ_ACC | WRITE_ACC))) {
          // Gamma applied, rounded, out ("+ 0.f" turns a -0 product into +0)
#pragma unroll
          for (int i = 0; i < L::WM; ++i)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
              float v[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = acc.get(i, j, rq * 4 + e) * scale + 0.f;
              uint2 packed;
              packed.x = f32x2_to_bf16x2_bits(v[0], v[1]);
              packed.y = f32x2_to_bf16x2_bits(v[2], v[3]);
              *reinterpret_cast<uint2*>(stage + L::piece_slot(wrow, i, rq)) = packed;
              if (rq == 3) __builtin_amdgcn_sched_barrier(0);     // one accumulator block at a time in VGPRs
            }
#pragma unroll
          for (int k = 0; k < 16 / RPS; ++k) {
            const int r = k * RPS + rrow, m = mw + (rpos ^ L::mix(r)) * 8;
            const u32x4 v = *reinterpret_cast<const u32x4*>(stage + r * L::ROW_BYTES + rpos * 16);
            const int row = row_of(j, r);
            if (row >= 0 && m < d) *reinterpret_cast<u32x4*>(out + (int64_t)row * d + m) = v;
          }
        } else {
          // fp32 running sums and K slices go out as they lie, 16 bytes per lane
          direct(acc, j);
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < L::WN; ++j) direct(acc, j);
    }
  };

  typename L::Acc acc;
  int z, p, q, k0, k_elems;
  place(b, z, p, q, k0, k_elems);
  int orow[L::WN];
  if constexpr (OPS == OPS_KC) {
    // one item per workgroup: this main loop has nothing to request ahead
    L::run(A + k0, lda * (int64_t)sizeof(T), q * L::TILE, d, B + k0, ldb * (int64_t)sizeof(T), p * L::TILE, a.b_rows,
           k_elems * (int)sizeof(T), lds, acc);
    load_rows(p, orow);
    flush(acc, z, p, q, orow);
  } else if constexpr (OPS == OPS_DH_F32 || OPS == OPS_DW_F32) {
    // likewise one item per workgroup: the other workgroup of the CU covers its start and its end
    const int width = min(L::TILE, d - q * L::TILE) * 4;
    const f32::Operand As{reinterpret_cast<const char*>(A + (int64_t)k0 * lda + q * L::TILE), lda * 4, 0, a.a_krows - k0, width};
    if constexpr (OPS == OPS_DH_F32) {
      const f32::Operand Bs{reinterpret_cast<const char*>(B + k0), ldb * 4, p * L::TILE, a.b_rows, 0};
      f32::mainloop<L::TILE, f32::KR, f32::KC>(As, Bs, k_elems, lds, acc.v);
    } else {
      const f32::Operand Bs{reinterpret_cast<const char*>(B + (int64_t)k0 * ldb + p * L::TILE), ldb * 4, 0, k_elems, L::TILE * 4};
      f32::mainloop<L::TILE, f32::KR, f32::KR>(As, Bs, k_elems, lds, acc.v);
    }
    load_rows(p, orow);
    flush(acc, z, p, q, orow);
  } else {
    typename L::template Pipe<OPS == OPS_DH_TR ? fast::KR : fast::PK, OPS == OPS_DH_TR ? fast::KB : fast::RB> pipe;
    auto start = [&](int p, int q, int k0, int k_elems) {
      if constexpr (OPS == OPS_DH_TR) {
        // A: K rows start at A (a_krows valid from there), window of the tile's hidden columns at q
        const int width = max(0, min(L::TILE, d - q * L::TILE)) * 2;
        const fast::Operand As{reinterpret_cast<const char*>(A + (int64_t)k0 * lda) + (int64_t)q * L::TILE * 2, lda * 2, 0,
                               a.a_krows - k0, width};
        // B: G blocked (ldb = bytes from one group of 16 rows to the next), rows p * TILE ..., K from position k0
        const fast::Operand Bs{reinterpret_cast<const char*>(B) + (int64_t)(p * (L::TILE / 16)) * ldb + (int64_t)(k0 / 32) * 1024,
                               ldb, 0, 0, 0};
        pipe.start(As, Bs, k_elems, lds);
      } else {
        // A: the images of hidden tile q, from K step (k_start + k0) / 32 on
        const fast::Operand As{reinterpret_cast<const char*>(A) + packed_cols_offset(q * L::TILE / flce::TILE, (int)lda) + q * L::TILE % flce::TILE * 64 +
                                   (int64_t)((a.k_start + k0) / fast::BK) * fast::OPER, 0, 0, 0, 0};
        // B: G blocked, K over its rows from row k0, the tile's vocabulary positions from p * TILE
        const fast::Operand Bs{reinterpret_cast<const char*>(B) + (int64_t)(k0 / 16) * ldb + (int64_t)(p * (L::TILE / 32)) * 1024,
                               ldb, 0, 0, 0};
        pipe.start(As, Bs, k_elems, lds);
      }
    };
    load_rows(p, orow);
    start(p, q, k0, k_elems);
    for (;;) {
      if constexpr (ONE) {
        pipe.run(lds, [&] { need_rows(orow); });
        flush(acc, z, p, q, orow);
        return;
      }
      const int b_next = b + n_wg;
      const bool more = b_next < total;
      int z_next = 0, p_next = 0, q_next = 0, k0_next = 0, k_next = 0;
      int orow_next[L::WN];
      pipe.run(lds, [&] {
        need_rows(orow);
        if (more) {
          place(b_next, z_next, p_next, q_next, k0_next, k_next);
          load_rows(p_next, orow_next);
          start(p_next, q_next, k0_next, k_next);
        }
      });
      flush(acc, z, p, q, orow);
      if (!more) break;
      need_rows(orow_next);
      b = b_next; z = z_next; p = p_next; q = q_next;
#pragma unroll
      for (int j = 0; j < L::WN; ++j) orow[j] = orow_next[j];
    }
  }
}

template <typename T, typename L, int OPS>
__global__ __launch_bounds__(L::THREADS, L::MIN_WAVES) void contract_kernel(ContractArgs<T> a) {
  extern __shared__ __align__(16) char lds[];
  contract<T, L, OPS>(a, blockIdx.x, gridDim.x, lds);
}

// dW and dH of one chunk side by side: the first wg_w workgroups take dW's items, the others dH's.  For problems whose
// output tiles fit the chip together, at most two rounds of them K slices included: `contractions` in plan_backward.
template <typename T, typename L, int OPS_W, int OPS_H>
__global__ __launch_bounds__(L::THREADS, L::MIN_WAVES) void contract_pair_kernel(ContractArgs<T> w, ContractArgs<T> h, int wg_w) {
  extern __shared__ __align__(16) char lds[];
  if ((int)blockIdx.x < wg_w) contract<T, L, OPS_W, true>(w, blockIdx.x, wg_w, lds);
  else contract<T, L, OPS_H, true>(h, (int)blockIdx.x - wg_w, (int)gridDim.x - wg_w, lds);
}

// Second half of a split-K contraction: one thread per four output elements; adds the K
// slices in slice order (fixed), then the running sum / Gamma / rounding exactly as the
// unsplit epilogue would.  Memory bound; the loads of eight slices are in flight together.
template <typename T>
__device__ __forceinline__ void splitk_reduce(const ContractArgs<T>& a, int launch_rows, int block) {
  const int d4 = a.d / 4;
  const int64_t i = (int64_t)block * 256 + threadIdx.x;
  const int row = (int)(i / d4), m = (int)(i - (int64_t)row * d4) * 4;
  const int n = a.out_row0 + row;
  if (row >= launch_rows || n >= a.out_rows) return;
  const int nv = (int)a.hdr->n_valid;
  int64_t orow = n;
  if (a.flags & ROWS_COMPACT) {
    if (n >= nv) return;
    orow = a.rowmap[n];
    if (orow < 0) return;
  }
  float scale = a.grad_loss.get();
  if (a.mean) scale = nv > 0 ? scale / (float)nv : 0.f;
  const int64_t off = (int64_t)(n - a.acc_row0) * a.d + m;
  f32x4 v = *reinterpret_cast<const f32x4*>(a.partial + off);
  constexpr int U = 8;
  for (int z0 = 1; z0 < a.n_split; z0 += U) {
    f32x4 t[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      t[u] = *reinterpret_cast<const f32x4*>(a.partial + (int64_t)min(z0 + u, a.n_split - 1) * a.partial_stride + off);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (z0 + u < a.n_split) v += t[u];
  }
  float* ap = a.accbuf + off;
  if (a.flags & READ_ACC) v += *reinterpret_cast<const f32x4*>(ap);
  if (a.flags & WRITE_ACC) *reinterpret_cast<f32x4*>(ap) = v;
  if (a.flags & WRITE_OUT)
    Pack4<T>::store(a.out + orow * a.d + m, v[0] * scale + 0.f, v[1] * scale + 0.f, v[2] * scale + 0.f,
                    v[3] * scale + 0.f);
}

template <typename T>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(ContractArgs<T> a, int launch_rows) {
  splitk_reduce(a, launch_rows, blockIdx.x);
}
// The slice sums of dW (the first blocks_w blocks) and dH in one launch.
template <typename T>
__global__ __launch_bounds__(256) void splitk_reduce_pair_kernel(ContractArgs<T> w, int rows_w, int blocks_w,
                                                                 ContractArgs<T> h, int rows_h) {
  if ((int)blockIdx.x < blocks_w) splitk_reduce(w, rows_w, blockIdx.x);
  else splitk_reduce(h, rows_h, (int)blockIdx.x - blocks_w);
}

// Alg. 4, scalar branch: out = Gamma * in, elementwise, Gamma from the header's n_valid.  Both gradients in one launch, one
// after the other in 8-byte or 16-byte groups of four; bound by memory.
template <typename T>
__global__ __launch_bounds__(256) void scale_kernel(const T* __restrict__ in_h, T* __restrict__ out_h, int64_t n4_h,
                                                    const T* __restrict__ in_w, T* __restrict__ out_w, int64_t n4_w,
                                                    const Header* __restrict__ hdr, float grad_loss, int mean) {
  const int nv = (int)hdr->n_valid;
  float scale = grad_loss;
  if (mean) scale = nv > 0 ? grad_loss / (float)nv : 0.f;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4_h + n4_w; i += (int64_t)gridDim.x * 256) {
    const bool h = i < n4_h;
    const T* in = h ? in_h + i * 4 : in_w + (i - n4_h) * 4;
    T* out = h ? out_h + i * 4 : out_w + (i - n4_h) * 4;
    float v[4];
    Pack4<T>::load(in, v);
    Pack4<T>::store(out, v[0] * scale + 0.f, v[1] * scale + 0.f, v[2] * scale + 0.f, v[3] * scale + 0.f);
  }
}

}  // namespace flce
