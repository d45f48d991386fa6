// bf16 main loop tuned for gfx950: 256 x 256 tile, 256 threads = 4 wavefronts (one per
// SIMD) arranged 2 x 2, each owning a 128 x 128 sub-tile (8 x 8 blocks of the
// 16x16x32 MFMA, 256 fp32 accumulators per lane); or, with 4 x 4 blocks per wavefront, a 128 x 128
// tile of which two workgroups fit on a CU, for problems with few tiles or a short K.
//
//   * The 16x16x32 MFMA and not the 32x32x16 one: the chip is power-limited under matrix load, and per flop the
//     16x16x32 one moves half the accumulator values.  From registers it sustains 2000 TFLOP/s where the other
//     sustains 1790 (same box, same data).
//   * Operand tiles go from global memory straight into LDS (buffer_load ... lds,
//     16 bytes per lane), four stages (128-row tiles: five) of 32 bf16 of K deep, so a tile is requested
//     two to three K steps before it is read.  Rows past the end of a tensor are
//     zero-filled by the buffer's range check.
//   * Each operand may be stored either way round in memory:
//       KC ("K contiguous"): 256 tile rows, each with its 32 K values adjacent (64 bytes).
//           LDS tile [256][64 B]; fragments are plain 128-bit LDS reads.
//       KR ("K rows"): the 32 K values of a tile row lie in 32 different memory rows, and
//           one memory row holds the 256 tile rows' values side by side (512 bytes).
//           LDS tile [32][512 B]; fragments come from the transposing LDS read
//           (ds_read_b64_tr_b16: 16 lanes hand in four K rows of 4 x 8 bytes and each
//           lane gets back 4 consecutive K values of one tile row).
//     This lets dH = G.W and dW = G^T.H read G, W and H where they are, with no
//     transposed copies.
//       PK ("packed"): the operand has been copied into the order of its LDS tiles beforehand:
//           per 256-row block and K step one 16 KiB image of the KC tile (swizzle included),
//           images of a block one after the other.  Every request is then 1 KiB of consecutive
//           bytes (KC: 16 pieces of 64 bytes) and the fragments are KC's.  Worth a copy for an
//           operand that is small and read many times (the hidden states in the forward and the
//           recompute: +2 % on the whole loop).
//   * LDS swizzles (applied on the global side, because the DMA writes LDS linearly):
//     KC: 16-byte chunk index ^ chunk_swizzle(row); KR: 64-byte chunk index ^ (k % 4), 32-byte half ^ (k / 8) % 2; RB:
//     32-byte half ^ (row / 8) % 2.  All spread what one LDS instruction touches in a cycle over all 64 banks.
//   * A wavefront holds the fragments of a whole K step twice: while the MFMAs of step kt run on one set, the other
//     is read from LDS for step kt + 1.  One barrier per K step, at its start: behind it every wavefront holds its
//     fragments of step kt and tile kt + 1 has landed.
//   * The instruction order inside a K step is pinned by hand (LDS reads and global
//     requests spread between consecutive MFMAs, fenced with scheduling barriers):
//     with one wavefront per SIMD a burst of other instructions stalls the MFMA
//     stream.  A wavefront issues an instruction every 7 to 8 cycles and an MFMA takes 16: one other instruction per MFMA is
//     free, two cost 5 cycles, three 12 (measured with scalar moves between MFMAs; LDS reads alike).
//
// Requires the K extent to be a multiple of 32 elements (of 8 in the RAGGED form) and offsets inside one tile's
// address window within 2^32 bytes (unsigned 32-bit buffer offsets); the generic loop in tile_mma.h covers everything else.
#pragma once
#include <type_traits>

#include "tile_mma.h"

namespace flce {
namespace fast {

constexpr int THREADS = 256;
constexpr int WM = 4, WN = 4;             // 32-row units of a wavefront's sub-tile
constexpr int BK = 32;                    // K elements per stage
constexpr int NS = 4;                     // stages
constexpr int OPER = TILE * BK * 2;       // 16 KiB per operand per stage (either layout)
constexpr int STAGE = 2 * OPER;
constexpr int LDS_BYTES = NS * STAGE;     // 128 KiB with 4 stages

enum : int { KC = 0, KR = 1, PK = 2, KB = 3, RB = 4 };
// KB and RB read a matrix that is stored in blocks of 16 rows x 32 columns (1 KiB, row-major inside), the blocks of a
// group of 16 rows one after the other along the columns and the row groups `ld_bytes` apart ("blocked"): both of its
// readers then fetch whole blocks, 1 KiB of consecutive bytes per request.
//   KB: K runs along the columns (32 columns = one block per 16 tile rows and K step); the LDS tile and the fragment
//       reads are KC's.  Operand: base = the block of the tile's first row and first K column, ld_bytes = bytes
//       from one row group to the next.
//   RB: K runs over the rows (two row groups per K step), the 256 tile rows are 256 consecutive columns (8 blocks);
//       the LDS tile holds the 16 blocks as they are, [2][8][16 rows][64 B], and the fragments come from the
//       transposing LDS read (rows of a block lie 64 bytes apart: every bank once without a swizzle).  Operand:
//       base = the block of the first K row and the tile's first column, ld_bytes as for KB.
// The chunk swizzle of the K-contiguous LDS tile, 0, 2, 3, 1 for row / 4 = 0 .. 3: one cycle of a 128-bit read serves lanes 0-3, 12-15, 20-27
// (or 4-11, 16-19, 28-31, and so in the upper half), i.e. of a fragment four groups of four rows with two different chunks.
__host__ __device__ __forceinline__ constexpr int chunk_swizzle(int row) {
  return ((row >> 3) & 1) | ((((row >> 2) ^ (row >> 3)) & 1) << 1);
}
constexpr bool kc_like(int layout) { return layout == KC || layout == PK || layout == KB; }

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// One operand of the contraction.
//   KC: base = first byte of row 0 of the tensor at the first K element; row0 = first tile
//       row; rows = valid rows of the tensor; width_bytes unused.
//   KR: base = first byte of K row 0 at the tile's first column; rows = valid K rows from
//       there; width_bytes = valid bytes of the tile's 512-byte column window (columns
//       beyond it may read as the next row's data: the caller masks what they produce).
struct Operand {
  const char* base;
  int64_t ld_bytes;
  int row0;
  int rows;
  int width_bytes;
};

// Global -> LDS requests are issued through inline assembly: as an intrinsic the compiler
// treats one as a store that may alias every later LDS read it cannot disambiguate (the
// transposing reads among them) and waits for vmcnt(0) before each, which serialises the
// pipeline.  Here the only consumers are separated from the DMA by the explicit vmcnt
// wait + barrier of the main loop.  M0 carries the LDS destination of the wavefront.  The descriptor may come fresh from
// vector instructions (readfirstlane), whose scalar results a memory instruction may read five wait states later: the compiler
// keeps that distance from its own instructions only, hence the s_nop 4 ahead of a group's first request.

__device__ __forceinline__ uint32_t lds_address(const char* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}

// Requests name memory as base + BIAS (3 KiB) below it + offset: request i has 1024 i in its instruction and BIAS - 1024 i in its
// per-lane offset, which is therefore never negative.
constexpr uint32_t BIAS = 3072;
template <int LAYOUT, int REQS>
__device__ __forceinline__ u32x4 make_rsrc(const Operand& s, int k_elems) {
  uint32_t n = 0;
  const char* b = s.base;
  if (LAYOUT == PK) {
    const int kt = (k_elems + BK - 1) / BK;   // images of 256 rows; a 128-row tile is one half of each
    if (kt > 0) n = (uint32_t)(kt - 1) * OPER + REQS * 4096;
  } else if (LAYOUT == KB) {         // a row group per request of the workgroup, the last one up to the end of the K extent
    n = (uint32_t)((4 * REQS - 1) * s.ld_bytes + (int64_t)(k_elems / BK) * 1024);
  } else if (LAYOUT == RB) {         // k_elems / 16 row groups, the tile's blocks of the last one
    if (k_elems > 0) n = (uint32_t)((int64_t)(k_elems / 16 - 1) * s.ld_bytes + 2 * REQS * 1024);
  } else if (LAYOUT == KC) {
    int vr = min(64 * REQS, s.rows - s.row0);
    if (vr > 0) n = (uint32_t)((int64_t)(vr - 1) * s.ld_bytes + k_elems * 2);
    b += (int64_t)s.row0 * s.ld_bytes;
  } else {
    const int kr = min(s.rows, k_elems);
    if (kr > 0 && s.width_bytes > 0) n = (uint32_t)((int64_t)(kr - 1) * s.ld_bytes + s.width_bytes);
  }
  // raw buffer descriptor: 48-bit base, stride 0, num_records in bytes, untyped 32-bit data format
  const uint64_t addr = (uint64_t)(uintptr_t)b - BIAS;
  u32x4 r = {(uint32_t)addr, (uint32_t)(addr >> 32) & 0xFFFFu, n ? n + BIAS : 0, 0x00020000u};
  r[0] = __builtin_amdgcn_readfirstlane(r[0]);
  r[1] = __builtin_amdgcn_readfirstlane(r[1]);
  r[2] = __builtin_amdgcn_readfirstlane(r[2]);
  return r;
}

// The accumulators of a wavefront's sub-tile, MA x NA blocks of 16 x 16, in the accumulation registers a0, a1, ... by number: block
// (mi, mj) is a[4 (mj MA + mi) .. + 3], element e of a lane is row 4 (lane / 16) + e of column lane % 16 of the block.  By number and not as
// variables: the compiler moved those between the branches of the main loop (252 moves per tile), and it cannot know how
// many wait states a move behind an MFMA in assembly needs.  It has no other use for these registers while a kernel's other
// values fit the vector registers (a test looks).  Every access is in (volatile, hence ordered) assembly; nothing may read a
// result before settle().
template <int MA, int NA>
struct Acc {
  static constexpr int REGS = MA * NA * 4;
  static __device__ __forceinline__ void claim() {      // counts the registers as the kernel's
    static_assert(REGS == 64 || REGS == 128 || REGS == 256, "the lists below");
    asm volatile("" ::: "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15",
                   "a16", "a17", "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31",
                   "a32", "a33", "a34", "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46", "a47",
                   "a48", "a49", "a50", "a51", "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61", "a62", "a63");
    if constexpr (REGS > 64)
      asm volatile("" ::: "a64", "a65", "a66", "a67", "a68", "a69", "a70", "a71", "a72", "a73", "a74", "a75", "a76", "a77", "a78", "a79",
                   "a80", "a81", "a82", "a83", "a84", "a85", "a86", "a87", "a88", "a89", "a90", "a91", "a92", "a93", "a94", "a95",
                   "a96", "a97", "a98", "a99", "a100", "a101", "a102", "a103", "a104", "a105", "a106", "a107", "a108", "a109", "a110", "a111",
                   "a112", "a113", "a114", "a115", "a116", "a117", "a118", "a119", "a120", "a121", "a122", "a123", "a124", "a125", "a126", "a127");
    if constexpr (REGS > 128)
      asm volatile("" ::: "a128", "a129", "a130", "a131", "a132", "a133", "a134", "a135", "a136", "a137", "a138", "a139", "a140", "a141", "a142", "a143",
                   "a144", "a145", "a146", "a147", "a148", "a149", "a150", "a151", "a152", "a153", "a154", "a155", "a156", "a157", "a158", "a159",
                   "a160", "a161", "a162", "a163", "a164", "a165", "a166", "a167", "a168", "a169", "a170", "a171", "a172", "a173", "a174", "a175",
                   "a176", "a177", "a178", "a179", "a180", "a181", "a182", "a183", "a184", "a185", "a186", "a187", "a188", "a189", "a190", "a191",
                   "a192", "a193", "a194", "a195", "a196", "a197", "a198", "a199", "a200", "a201", "a202", "a203", "a204", "a205", "a206", "a207",
                   "a208", "a209", "a210", "a211", "a212", "a213", "a214", "a215", "a216", "a217", "a218", "a219", "a220", "a221", "a222", "a223",
                   "a224", "a225", "a226", "a227", "a228", "a229", "a230", "a231", "a232", "a233", "a234", "a235", "a236", "a237", "a238", "a239",
                   "a240", "a241", "a242", "a243", "a244", "a245", "a246", "a247", "a248", "a249", "a250", "a251", "a252", "a253", "a254", "a255");
  }
  static __device__ __forceinline__ void clear() {
#pragma unroll
    for (int r = 0; r < REGS; ++r) asm volatile("v_accvgpr_write_b32 a[%0], 0" ::"i"(r));
    asm volatile("s_nop 7" ::: "memory");
  }
  // element 4 q + e of the 64 rows x 16 columns block (i, j): rows 64 i + 16 q + 4 (lane / 16) + e, column 16 j + lane % 16
  static __device__ __forceinline__ float get(int i, int j, int r) {     // constants after unrolling
    float v;
    asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(v) : "i"(4 * (j * MA + i * 4 + (r >> 2)) + (r & 3)));
    return v;
  }
  // the wait states between the last MFMA and the first plain read of its result (at most 11 for a 16x16x32)
  static __device__ __forceinline__ void settle() { asm volatile("s_nop 15" ::: "memory"); }
};

// a[r .. r + 3] (+)= a . b on the matrix cores; FIRST: from zero (the instruction takes the constant as its
// addend: no pass over the registers to clear them).
template <bool FIRST>
__device__ __forceinline__ void mfma(int r, bf16x8 a, bf16x8 b) {
  if constexpr (FIRST) asm volatile("v_mfma_f32_16x16x32_bf16 a[%0:%1], %2, %3, 0" ::"i"(r), "i"(r + 3), "v"(a), "v"(b));
  else asm volatile("v_mfma_f32_16x16x32_bf16 a[%0:%1], %2, %3, a[%0:%1]" ::"i"(r), "i"(r + 3), "v"(a), "v"(b));
}
// Four MFMAs of a column of blocks (a[r .. r + 15]) with the REQS global -> LDS requests of one operand between them, in one piece.
// M0 holds the LDS destination of request 0; request i goes 1024 i further on in LDS and, the instruction's offset counting for
// both, in memory.  (Setting M0 needs one instruction before its use.)  MASKED: the requests run under the execution mask `lanes`
// (all of the wavefront or none), which MFMAs ignore and nothing else may meet.
template <bool FIRST, int REQS, bool MASKED>
__device__ __forceinline__ void mfma_requests(int r, bf16x8 a0, bf16x8 a1, bf16x8 a2, bf16x8 a3, bf16x8 b, uint64_t lanes, u32x4 rsrc,
                                              const uint32_t (&v)[REQS], uint32_t soffset) {
#define FLCE_MFMA(c, a) "v_mfma_f32_16x16x32_bf16 a[%[" c "]:%[" c "e]], %[" a "], %[b], "
#define FLCE_REQ(k, offset) "\n\tbuffer_load_dwordx4 %[v" k "], %[r], %[s] offen" offset " lds\n\t"
#define FLCE_BODY(z0, z1, z2, z3, r2, r3)                                                                       \
  FLCE_MFMA("c0", "a0") z0 FLCE_REQ("0", "") FLCE_MFMA("c1", "a1") z1 FLCE_REQ("1", " offset:1024")             \
  FLCE_MFMA("c2", "a2") z2 r2 FLCE_MFMA("c3", "a3") z3 r3
#define FLCE_R2 FLCE_REQ("2", " offset:2048")
#define FLCE_R3 FLCE_REQ("3", " offset:3072")
#define FLCE_MASK(body) "s_mov_b64 exec, %[m]\n\t" body "s_mov_b64 exec, -1"
#define FLCE_SUM(c) "a[%[" c "]:%[" c "e]]"
#define FLCE_SUMS(r2, r3) FLCE_BODY(FLCE_SUM("c0"), FLCE_SUM("c1"), FLCE_SUM("c2"), FLCE_SUM("c3"), r2, r3)
#define FLCE_IN                                                                                                        \
  [c0] "i"(r), [c0e] "i"(r + 3), [c1] "i"(r + 4), [c1e] "i"(r + 7), [c2] "i"(r + 8), [c2e] "i"(r + 11), [c3] "i"(r + 12),           \
  [c3e] "i"(r + 15), [a0] "v"(a0), [a1] "v"(a1), [a2] "v"(a2), [a3] "v"(a3), [b] "v"(b), [r] "s"(rsrc), [s] "s"(soffset),     \
  [v0] "v"(v[0]), [v1] "v"(v[1])
#define FLCE_IN4 FLCE_IN, [v2] "v"(v[2]), [v3] "v"(v[3])
  static_assert(!FIRST || MASKED, "the first step is a masked one");
  if constexpr (REQS == 4) {
    if constexpr (FIRST) asm volatile(FLCE_MASK(FLCE_BODY("0", "0", "0", "0", FLCE_R2, FLCE_R3)) :: FLCE_IN4, [m] "s"(lanes) : "memory");
    else if constexpr (MASKED) asm volatile(FLCE_MASK(FLCE_SUMS(FLCE_R2, FLCE_R3)) :: FLCE_IN4, [m] "s"(lanes) : "memory");
    else asm volatile(FLCE_SUMS(FLCE_R2, FLCE_R3) :: FLCE_IN4 : "memory");
  } else {
    if constexpr (FIRST) asm volatile(FLCE_MASK(FLCE_BODY("0", "0", "0", "0\n\t", "\n\t", "")) :: FLCE_IN, [m] "s"(lanes) : "memory");
    else if constexpr (MASKED) asm volatile(FLCE_MASK(FLCE_SUMS("\n\t", "\n\t")) :: FLCE_IN, [m] "s"(lanes) : "memory");
    else asm volatile(FLCE_SUMS("\n\t", "") :: FLCE_IN : "memory");
  }
#undef FLCE_MFMA
#undef FLCE_REQ
#undef FLCE_BODY
#undef FLCE_R2
#undef FLCE_R3
#undef FLCE_MASK
#undef FLCE_SUM
#undef FLCE_SUMS
#undef FLCE_IN
#undef FLCE_IN4
}
__device__ __forceinline__ void set_m0(uint32_t lds_addr, uint32_t offset) {
  asm volatile("s_add_i32 m0, %0, %1" : : "s"(lds_addr), "s"(offset) : "m0", "scc");
}
__device__ __forceinline__ uint64_t lanes_if_less(int a, int b) {      // all lanes or none (a, b in scalar registers)
  uint64_t m;
  asm volatile("s_cmp_lt_i32 %1, %2\n\ts_cselect_b64 %0, -1, 0" : "=s"(m) : "s"(a), "s"(b) : "scc");
  return m;
}
// A value that is the same in every lane, in a scalar register.  (In assembly: the builtin is folded away for a value that the
// compiler keeps in a vector register all the same.  A vector register written right before needs one wait state.)
__device__ __forceinline__ int scalar(int x) {
  int m;
  asm volatile("s_nop 0\n\tv_readfirstlane_b32 %0, %1" : "=s"(m) : "v"(x));
  return m;
}

__device__ __forceinline__ int slot_of_lane() {      // fp32 loop: which of the 4 lanes sharing an N column this is
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  return (wave >> 1) * 2 + (lane >> 5);
}

// s_waitcnt with vmcnt <= N and lgkmcnt == 0 (all of this wavefront's LDS reads returned).
// gfx9 encoding: vmcnt in bits [3:0] and [15:14], expcnt [6:4], lgkmcnt [11:8].
template <int N>
__device__ __forceinline__ void wait_vm_and_lds() {
  constexpr int lo = N & 15, hi = (N >> 4) & 3;
  __builtin_amdgcn_s_waitcnt((hi << 14) | (0x0 << 8) | (0x7 << 4) | lo);
}

// Global -> LDS requests of one operand: REQS per wavefront per stage (4 for a 256-row tile, 2 for a 128-row one), 1 KiB each, written linearly into this wavefront's slice of the operand tile.
// RAGGED (K-contiguous layout): K need not be a multiple of a stage's 32 elements, only of 8; the 16-byte chunks of the
// last stage past the end of K are requested out of the descriptor's range and land as zeros.  (Such shapes ran on the
// generic loop, with transposed copies of H, W and G: 20597 x 168 x 179711 13.46 -> 9.25 ms per step, 3716 x 136 x 84702
// 1027 -> 713 us, 500 x 1000 x 30000 271 -> 207 us, same bits.)
template <int LAYOUT, int REQS = 4, bool RAGGED = false>
struct Loader {
  static_assert(REQS == 4 || REQS == 2, "256 or 128 tile rows");
  u32x4 rs;
  uint32_t v[REQS];       // per-lane byte offsets of the requests; unsigned: a window may reach 2^32 bytes
  uint32_t soff, k_step;  // scalar offset; KC: bytes of K per stage (scalar offset); KR: bytes of 32 K rows (added per lane)
  int end_kt;             // RAGGED: the last K tile if this lane's chunk of it lies past the end of K (every request
                          // of a lane takes the same chunk: request rows are a multiple of 16 apart), -1 otherwise
  __device__ __forceinline__ void init(const Operand& s, int k_elems, int tid) {
    rs = make_rsrc<LAYOUT, REQS>(s, k_elems);
    const int wave = tid >> 6, lane = tid & 63;
#pragma unroll
    for (int i = 0; i < REQS; ++i) {
      if (LAYOUT == PK) {
        v[i] = (uint32_t)(wave * (REQS * 1024) + i * 1024 + lane * 16);
      } else if (LAYOUT == KB) {     // request = row group wave * REQS + i of the tile: one block, KC's chunk order
        const int chunk = (lane & 3) ^ chunk_swizzle(lane >> 2);
        v[i] = (uint32_t)((wave * REQS + i) * s.ld_bytes) + (lane >> 2) * 64 + chunk * 16;
      } else if (LAYOUT == RB) {     // request = block (row group, column block) of the 2 x (2 REQS) of a K step; halves of rows 8.. swapped
        const int b = wave * REQS + i;
        v[i] = (uint32_t)(b / (2 * REQS) * s.ld_bytes) + b % (2 * REQS) * 1024 + ((lane * 16) ^ (lane >> 5 << 5));
      } else if (LAYOUT == KC) {
        const int row = wave * (16 * REQS) + i * 16 + (lane >> 2);
        const int chunk = (lane & 3) ^ chunk_swizzle(row);
        v[i] = (uint32_t)(row * s.ld_bytes) + chunk * 16;
      } else {
        constexpr int LANES = 8 * REQS;        // of 16 bytes per K row
        const int krow = wave * 8 + i * (64 / LANES) + lane / LANES;
        const int off = ((lane % LANES) * 16) ^ ((krow & 3) << 6) ^ ((krow >> 3 & 1) << 5);
        v[i] = (uint32_t)(krow * s.ld_bytes) + off;
      }
    }
#pragma unroll
    for (int i = 0; i < REQS; ++i) v[i] += BIAS - 1024 * i;
    soff = 0;
    if (LAYOUT == KC && RAGGED) {
      const int chunk = (lane & 3) ^ chunk_swizzle(lane >> 2);
      const int last_kt = (k_elems + BK - 1) / BK - 1;
      end_kt = last_kt * BK + chunk * 8 >= k_elems ? last_kt : -1;
    }
    k_step = LAYOUT == PK ? OPER : LAYOUT == KC ? BK * 2 : LAYOUT == KB ? 1024 : LAYOUT == RB ? (uint32_t)(2 * s.ld_bytes)
                                                                                      : (uint32_t)(BK * s.ld_bytes);
  }
  // The requests of a K tile: where they are for the tile that comes next, and on to the one behind it.
  // K advances in the scalar offset where it runs along the rows, and in the per-lane offsets, which the range check covers,
  // where it moves to other rows (and in the RAGGED form).
  static constexpr bool BY_LANE = !kc_like(LAYOUT) || RAGGED && LAYOUT == KC;
  __device__ __forceinline__ void ragged_end(int kt) {      // before the requests of K tile kt
    if (LAYOUT == KC && RAGGED) {
      if (kt == end_kt) {
#pragma unroll
        for (int i = 0; i < REQS; ++i) v[i] = 0xFFFFFFF0u - 1024 * i;
      }
    }
  }
  __device__ __forceinline__ void advance() {
    if (BY_LANE) {
#pragma unroll
      for (int i = 0; i < REQS; ++i) {
        v[i] += k_step;
        asm volatile("" : "+v"(v[i]));      // (opaque: one register each, not one per use and loop)
      }
    } else {
      soff += k_step;
      asm volatile("" : "+s"(soff));
    }
  }
  // all requests of the next K tile into `dst` (this wavefront's slice of the operand tile of some stage)
  __device__ __forceinline__ void issue_all(uint32_t dst, int kt) {
    ragged_end(kt);
    if constexpr (REQS == 4)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %5, %6 offen lds\n\t"
                   "buffer_load_dwordx4 %2, %5, %6 offen offset:1024 lds\n\t"
                   "buffer_load_dwordx4 %3, %5, %6 offen offset:2048 lds\n\t"
                   "buffer_load_dwordx4 %4, %5, %6 offen offset:3072 lds"
                   :: "s"(dst), "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "s"(rs), "s"(soff) : "memory", "m0");
    else
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %3, %4 offen lds\n\t"
                   "buffer_load_dwordx4 %2, %3, %4 offen offset:1024 lds"
                   :: "s"(dst), "v"(v[0]), "v"(v[1]), "s"(rs), "s"(soff) : "memory", "m0");
    advance();
  }
};

// Per-lane LDS byte offsets of the fragment reads of one operand; wsub = which half of the tile's rows this
// wavefront works on (2 BLOCKS blocks of 16 rows: 8 for a 256-row tile, 4 for a 128-row one).  A lane's fragment of a block is
// row lane % 16, K 8 (lane / 16) .. + 7.
template <int LAYOUT, int BLOCKS = 4>
struct FragAddr {
  static_assert(BLOCKS == 4 || BLOCKS == 2, "256 or 128 tile rows");
  static constexpr int N = 2 * BLOCKS;
  int o[N];   // KC: o[0]; KR: o[i] for the blocks; RB: o[0], o[1] for even and odd ones
  __device__ __forceinline__ void init(int wsub, int tid) {
    const int lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    if (kc_like(LAYOUT)) {
      o[0] = (wsub * 32 * BLOCKS + l16) * 64 + ((g ^ chunk_swizzle(l16)) << 4);
    } else {
      const int e = l16 >> 2, q = l16 & 3;
#pragma unroll
      for (int i = 0; i < (LAYOUT == RB ? 2 : N); ++i)
        o[i] = LAYOUT == RB ? (g >> 1) * (BLOCKS * 2048) + wsub * BLOCKS * 1024 + (8 * (g & 1) + e) * 64 + ((i ^ (g & 1)) << 5) + 8 * q
                            : (8 * g + e) * (128 * BLOCKS) + (((wsub * N + i) << 5) ^ (e << 6) ^ ((g & 1) << 5)) + 8 * q;
    }
  }
  static constexpr int READS = kc_like(LAYOUT) ? N : 2 * N;   // LDS reads per K step
  // on to another stage, in place (opaque: the compiler would keep a second set of sums)
  __device__ __forceinline__ void move(int bytes) {
#pragma unroll
    for (int i = 0; i < (kc_like(LAYOUT) ? 1 : LAYOUT == RB ? 2 : N); ++i) {
      o[i] += bytes;
      asm volatile("" : "+v"(o[i]));
    }
  }
};

template <int AM, int AN>
struct Frags {
  bf16x8 a[2 * AM], b[2 * AN];
};

// Read number t (0 .. READS-1) of the fragments of one operand.
template <int LAYOUT, int BLOCKS>
__device__ __forceinline__ void read_frag(bf16x8 (&f)[2 * BLOCKS], const FragAddr<LAYOUT, BLOCKS>& fa, const char* tile, int t) {
  if (kc_like(LAYOUT)) {
    f[t] = *reinterpret_cast<const bf16x8*>(tile + fa.o[0] + t * 16 * 64);
  } else {
    const int i = t >> 1, r = t & 1;
    // K rows 8 g + 4 r + (0..3): KR has them one tile row apart; RB has 16 rows per row group of the tile, 64 bytes apart,
    // two blocks of 16 rows side by side
    const char* at = LAYOUT == RB ? tile + fa.o[i & 1] + (i >> 1) * 1024 + r * 256 : tile + fa.o[i] + 4 * r * (128 * BLOCKS);
    const s16x4 h = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)at);
    const bf16x4 hb = __builtin_bit_cast(bf16x4, h);
    if (r == 0) { f[i][0] = hb[0]; f[i][1] = hb[1]; f[i][2] = hb[2]; f[i][3] = hb[3]; }
    else        { f[i][4] = hb[0]; f[i][5] = hb[1]; f[i][6] = hb[2]; f[i][7] = hb[3]; }
  }
}

// The contraction of one tile, split in two calls so that a kernel that works on several
// tiles can request the first stages of the next tile before it post-processes the
// accumulators of the current one:
//   start(A, B, k_elems, lds): requests K tiles 0 .. NSTAGES - 2 into the stages of the same numbers, which must be
//                              free (the last stage stays empty until run(): post-processing may use it);
//   run(lds, released):        acc = A_tile . B_tile^T over k_elems of K (a multiple of 32).  Before the MFMAs of the last
//                              K step all wavefronts have passed a barrier behind their last LDS read: `released` is called
//                              there and may call start() for the next tile.
//
// WITH_MFMA = false leaves the matrix instructions out (everything else, i.e. the global -> LDS requests, the LDS
// fragment reads, the waits and barriers, stays): only the measurement probe uses it, to time the data path alone.
//
// AM, AN = 32-row units of A and B per wavefront: 4 x 4 is the 256 x 256 tile above.  2 x 2 is a 128 x 128 tile (64
// accumulators per lane, two workgroups per CU) for problems with too few 256-row tiles; 2 x 4 serves the probe.
//
// RAGGED: K is a multiple of 8 elements, K-contiguous operands have it as their extent and a pre-tiled operand is padded
// with zeros to whole stages.
template <int LA, int LB, bool WITH_MFMA = true, int AM = WM, int NSTAGES = NS, bool RAGGED = false,
          int AN = WN>
struct Pipe {
  static constexpr int REQS_A = AM, REQS_B = AN;       // requests per wavefront per stage (1 KiB each)
  static constexpr int OPER_A = AM * 4096;             // bytes of the A tile of one stage
  static constexpr int STAGE_BYTES = OPER_A + AN * 4096;   // A tile, then B tile
  static constexpr int LDS_TOTAL = NSTAGES * STAGE_BYTES;
  static constexpr int LOADS = REQS_A + REQS_B;        // requests per wavefront per K tile
  static constexpr int MA = 2 * AM, NA = 2 * AN, NM = MA * NA;   // MFMAs per K step
  Loader<LA, REQS_A, RAGGED> la;
  Loader<LB, REQS_B, RAGGED> lb;
  FragAddr<LA, AM> fa;
  FragAddr<LB, AN> fb;
  int KT;
  uint32_t lds_a;              // LDS address of this wavefront's slice of the A tile of stage 0

  __device__ __forceinline__ void start(const Operand& A, const Operand& B, int k_elems, char* lds) {
    KT = RAGGED ? (k_elems + BK - 1) / BK : k_elems / BK;
    int tid = threadIdx.x;
    if (AM != AN) asm volatile("" : "+v"(tid));      // (the probe's half tile has no vector registers for what is derived from it)
    la.init(A, k_elems, tid);
    lb.init(B, k_elems, tid);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    fa.init(wave >> 1, tid);
    fb.init(wave & 1, tid);
    lds_a = lds_address(lds) + wave * (REQS_A * 1024);
    // Opaque to the optimiser: in a kernel that walks several tiles these are loop invariant, and everything
    // derived from them (a dozen comparisons of the K count, the LDS address of every request of every stage)
    // would be precomputed once and kept alive in scalar registers across the whole tile loop, which overflows them.
    asm volatile("" : "+s"(KT), "+s"(lds_a));
#pragma unroll
    for (int s = 0; s < NSTAGES - 1; ++s)
      if (s < KT) {
        la.issue_all(lds_a + s * STAGE_BYTES, s);
        lb.issue_all(b_slice(s * STAGE_BYTES, wave), s);
      }
  }

  // waits until at most min(tiles, MOST) whole K tiles of this wavefront's requests are outstanding
  template <int MOST>
  static __device__ __forceinline__ void wait_requests(int tiles) {
    if (MOST == 0 || tiles >= MOST) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(MOST * LOADS) : "memory");
    else if constexpr (MOST > 0) wait_requests<MOST - 1>(tiles);
  }

  using Sums = Acc<MA, NA>;
  // this wavefront's slice of the B tile of the stage at `stage`
  __device__ __forceinline__ uint32_t b_slice(uint32_t stage, int wave) const {
    return lds_a + stage + OPER_A + wave * ((REQS_B - REQS_A) * 1024);
  }

  template <typename F>
  __device__ __forceinline__ void run(char* lds, F released) {
    Sums::claim();
    static_assert(NSTAGES >= 3 && (NSTAGES - 2) * LOADS < 64, "the waits count at most 63 requests");
    constexpr int RA = FragAddr<LA, AM>::READS, RB = FragAddr<LB, AN>::READS, RT = RA + RB;
    const int n = scalar(KT);    // (`released` may set up the next tile)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Frags<AM, AN> f0, f1;        // of the even and the odd K steps

    // The MFMAs of K step kt on fragment set FM.  READ: between them the LDS reads of tile kt + 1 (stage at rd) into
    // fragment set FR.  LOAD: between them the global requests of tile kt + NSTAGES into the stage of tile kt (lst), which
    // every wavefront has in registers, 2: if there is such a tile.
    auto step = [&](auto first, auto read, auto load, const Frags<AM, AN>& FM, Frags<AM, AN>& FR, int kt, const char* rd, uint32_t lst) {
      constexpr bool FIRST = decltype(first)::value != 0, READ = decltype(read)::value != 0;
      constexpr int LOAD = decltype(load)::value;
      __builtin_amdgcn_sched_barrier(0);
      uint64_t lanes = ~0ull;
      // columns of four blocks, in patches of 4 x 4 blocks; two neighbours share an operand
      constexpr int COLS = NM / 4, COL_A = LOAD ? COLS / 4 : COLS, COL_B = LOAD ? COLS == 4 ? 3 : COLS * 5 / 8 : COLS;
      static_assert(!LOAD || (COL_A > 0 && COL_B > COL_A + 1 && COL_B < COLS), "a column before each request column sets M0");
      constexpr int SLOTS = (COLS - (LOAD ? 2 : 0)) * 4, READ_SLOTS = SLOTS - SLOTS / 8;      // of the MFMAs that have no request behind them
      static_assert(RT <= 4 * READ_SLOTS, "at most four reads behind an MFMA");
#pragma unroll
      for (int c = 0; c < COLS; ++c) {
        const int patch = c >> 2;
        const int mj = (patch / (MA / 4)) * 4 + (c & 3), m0 = (patch % (MA / 4)) * 4;
        const int r0 = 4 * (mj * MA + m0);
        if (WITH_MFMA && c == COL_A) {
          mfma_requests<FIRST, REQS_A, LOAD == 2>(r0, FM.a[m0], FM.a[m0 + 1], FM.a[m0 + 2], FM.a[m0 + 3], FM.b[mj], lanes, la.rs, la.v, la.soff);
          la.advance();
        } else if (WITH_MFMA && c == COL_B) {
          mfma_requests<FIRST, REQS_B, LOAD == 2>(r0, FM.a[m0], FM.a[m0 + 1], FM.a[m0 + 2], FM.a[m0 + 3], FM.b[mj], lanes, lb.rs, lb.v, lb.soff);
          lb.advance();
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int mi = m0 + (c & 1 ? 3 - u : u);
            if constexpr (WITH_MFMA) mfma<FIRST>(r0 + 4 * (mi - m0), FM.a[mi], FM.b[mj]);
            else asm volatile("" ::"v"(FM.a[mi]), "v"(FM.b[mj]));       // keep the fragment reads alive without arithmetic on them
            // the reads, spread evenly over the first seven eighths of the step: the last one's latency is covered by the rest
            const int slot = (c - (c > COL_A) - (c > COL_B)) * 4 + u, t0 = (slot * RT + READ_SLOTS - 1) / READ_SLOTS;
#pragma unroll
            for (int t = t0; t < t0 + 4; ++t)
              if (READ && t < RT && t * READ_SLOTS / RT == slot) {
                if (t < RA) read_frag<LA>(FR.a, fa, rd, t);
                else read_frag<LB>(FR.b, fb, rd + OPER_A, t - RA);
              }
            if (LOAD == 2 && c == 0 && u == 1) lanes = lanes_if_less(kt + NSTAGES, n);
            if (u == 2 && c + 1 == COL_A) { la.ragged_end(kt + NSTAGES); set_m0(lds_a, lst); }
            if (u == 2 && c + 1 == COL_B) { lb.ragged_end(kt + NSTAGES); set_m0(b_slice(0, wave), lst); }
            if constexpr (!WITH_MFMA) {
              if (u == 3 && c + 1 == COL_A && kt + NSTAGES < n) la.issue_all(lds_a + lst, kt + NSTAGES);
              if (u == 3 && c + 1 == COL_B && kt + NSTAGES < n) lb.issue_all(b_slice(lst, wave), kt + NSTAGES);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
      asm volatile("" ::: "memory");      // the reads stay above (left to itself the compiler sinks them behind a loop's exit)
    };
    constexpr std::integral_constant<int, 0> NO{};
    constexpr std::integral_constant<int, 1> YES{};
    constexpr std::integral_constant<int, 2> IF{};
    // Tile kt lies in stage kt % NSTAGES, fa and fb point at the stage that is read from next.  With four stages two steps go
    // through a half of the ring: even steps read one stage behind the half's first, odd ones from the first of the
    // other half, where fa and fb move to (half the moves: the 256-row loop has few instructions to spare).
    int half = 0, sc = 0;
    auto rd_of = [&](int odd) -> const char* {      // on top of fa, fb; `odd` = kt % 2
      return NSTAGES == 4 && !odd ? lds + STAGE_BYTES : lds;
    };
    auto lst_of = [&](int odd) -> int {             // the stage that a step requests into
      if constexpr (NSTAGES == 4) return odd ? 3 * STAGE_BYTES - half : half;
      return sc * STAGE_BYTES;
    };
    auto next = [&](int odd) {                      // before step kt: `odd` = kt % 2
      if constexpr (NSTAGES == 4) {
        if (!odd) return;
        half = 2 * STAGE_BYTES - half;
        const int by = half ? 2 * STAGE_BYTES : -2 * STAGE_BYTES;
        fa.move(by);
        fb.move(by);
      } else {
        sc = sc + 1 == NSTAGES ? 0 : sc + 1;
        const int by = sc + 1 == NSTAGES ? STAGE_BYTES - LDS_TOTAL : STAGE_BYTES;
        fa.move(by);
        fb.move(by);
      }
    };
    // What a step that reads waits for: tile kt + 1 has landed (only tiles kt + 2 .. kt + NSTAGES - 1 may be in flight), and
    // this wavefront holds its fragments of tile kt (lgkmcnt(0)): behind the barrier all of it goes for every wavefront.
    auto arrive = [&] {
      wait_vm_and_lds<(NSTAGES - 2) * LOADS>();
      __builtin_amdgcn_s_barrier();
    };
    auto arrive_late = [&](int kt) {                // the same near the end, where fewer tiles are in flight
      wait_vm_and_lds<63>();
      wait_requests<NSTAGES - 2>(n - kt - 2);
      __builtin_amdgcn_s_barrier();
    };
    if (n > 0) {
      // tile 0 has landed once only the other tiles requested by start() are in flight; behind the barrier the last stage is
      // free too (post-processing may have used it)
      wait_requests<NSTAGES - 2>(n - 1);
      __builtin_amdgcn_s_barrier();
      if (NSTAGES - 1 < n) {
        la.issue_all(lds_a + (NSTAGES - 1) * STAGE_BYTES, NSTAGES - 1);
        lb.issue_all(b_slice((NSTAGES - 1) * STAGE_BYTES, wave), NSTAGES - 1);
      }
      // in the order in which the MFMAs need them
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int t = h * RA / 2; t < (h + 1) * RA / 2; ++t) read_frag<LA>(f0.a, fa, lds, t);
#pragma unroll
        for (int t = h * RB / 2; t < (h + 1) * RB / 2; ++t) read_frag<LB>(f0.b, fb, lds + OPER_A, t);
      }
      if constexpr (NSTAGES != 4) {
        fa.move(STAGE_BYTES);
        fb.move(STAGE_BYTES);
      }
      asm volatile("" ::: "memory");
    }
    if (n > 1) {
      arrive_late(0);
      step(YES, YES, IF, f0, f1, 0, rd_of(0), lst_of(0));
      int kt = 1;
      for (; kt + 2 + NSTAGES <= n; kt += 2) {      // steps kt and kt + 1 have a tile to request
        next(1);
        arrive();
        step(NO, YES, YES, f1, f0, kt, rd_of(1), lst_of(1));
        next(0);
        arrive();
        step(NO, YES, YES, f0, f1, kt + 1, rd_of(0), lst_of(0));
      }
      // of the steps that are left, the last one apart, at most the first has a tile to request
      if (kt + 1 < n) {
        next(1);
        arrive_late(kt);
        step(NO, YES, IF, f1, f0, kt, rd_of(1), lst_of(1));
        for (++kt; kt + 1 < n; ++kt) {
          next(0);
          arrive_late(kt);
          step(NO, YES, NO, f0, f1, kt, rd_of(0), 0);
          if (++kt + 1 >= n) break;
          next(1);
          arrive_late(kt);
          step(NO, YES, NO, f1, f0, kt, rd_of(1), 0);
        }
      }
    } else {
      // one step or an empty K extent (no counted row, or a K slice past the end)
      Sums::clear();
    }
    // The last step: behind its barrier every fragment is in registers and all stages are free.
    wait_vm_and_lds<63>();
    __builtin_amdgcn_s_barrier();
    released();
    if (n > 0) {
      if (n & 1) step(NO, NO, NO, f0, f1, 0, nullptr, 0);
      else step(NO, NO, NO, f1, f0, 0, nullptr, 0);
    }
    Sums::settle();
  }
};

}  // namespace fast
}  // namespace flce
