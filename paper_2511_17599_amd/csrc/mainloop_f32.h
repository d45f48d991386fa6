// fp32 main loop for gfx950: T x T output tile (T = 128 or 64), 256 threads = 4 wavefronts arranged 2 x 2, each owning
// WB x WB = T / 64 blocks of a 32 x 32 MFMA, two workgroups per CU.
//
// The fp32 matrix instruction is 16 times slower than the bf16 one (256 flops per clock and CU).  128-row tiles therefore
// write each operand value as the exact sum of three bf16 numbers, x = h + m + l (8 bits of mantissa each), and add up the six
// products hh, hm, mh, mm, hl, lh in the bf16 instruction's fp32 accumulators; what is left out is below 2^-24 of a product.
// (The method: Henry, Tang and Heinecke, "Leveraging the bfloat16 artificial intelligence datatype for higher-precision
// computations", ARITH 2019.)
// Its sums round once per 16 products and part instead of once per 2 products, and the partial sums are kept
// short (sum_stages), so the error against 64 bits is no larger: dH and dW 4.0e-7 -> 1.7e-7 (1000 x 512 x 10007), 4.2e-7 ->
// 2.0e-7 and 4.1e-7 -> 1.8e-7 (4096 x 1024 x 8192), log-sum-exp level (its rounding to 32 bits dominates).  Forward and
// backward, us (both sides in turn): 1000 x 512 x 10007 116 + 340 -> 106 + 267, 4096 x 1024 x 32768 2030 + 6258 -> 1587 + 5425.  What
// bounds it: the vector work of taking the parts (52 instructions per eight values and block row) beside the 24 MFMAs of a K step of 16, of
// which two wavefronts per SIMD overlap about two thirds.  64-row tiles serve problems too small to fill the chip, where one
// wavefront per SIMD would do the two one after the other: they stay with the fp32 instruction (with parts 256 x 256 x 4096
// forward 37.0 -> 39.2 us).  A 256-row tile of K = 512 keeps a CU busy for 109 us and
// a problem of a few thousand rows by a few thousand vocabulary entries has fewer such tiles than the chip has CUs, hence
// the small tiles and the two resident workgroups that even out a ragged last round.
//
//   * Operand tiles go from global memory straight into LDS (buffer_load ... lds), 32 K elements per stage, NS stages;
//     each wavefront's part of a stage has a descriptor of its own, advanced with K, so that no operand size is out of a
//     32-bit offset's reach; rows and K elements past the end are zero-filled by the range check.
//   * Each operand may be stored either way round:
//       KC: T rows with their 32 K values adjacent, 128 bytes (K ends at a multiple of 4 elements; 16-byte chunks
//           past it are not read).  LDS [T][128 B], 16-byte chunk index ^ (row / 2) % 8: a 128-bit fragment read
//           touches every bank once.
//       KR: K runs over memory rows, T columns side by side.  LDS [32][4 T B], chunk index ^ 8 on K rows with bit 2
//           set: the two lane halves of a fragment read, four K rows apart, use different halves of the banks.
//     so that dH = G.W and dW = G^T.H read G, W and H where they are.
//   * K is taken in groups of 8: lane half h holds K = 8 g + 4 h + j, j = 0..3, for the group's four MFMAs (the order of
//     K inside a group is free as long as both operands agree), which makes a KC fragment one 128-bit read.
#pragma once
#include "mainloop_fast.h"

namespace flce {
namespace f32 {

constexpr int THREADS = 256;
constexpr int BK = 32;                                      // K elements per stage
// Stages whose products are added up before they are added to the tile's sum: a chain of that many and one of the rest instead
// of one of K, which the contractions (K = the vocabulary, the rows) would otherwise show.  Relative error of dH and dW against 64
// bits at 4096 x 1024 x 16384 with the fp32 instruction: about 3e-6 with one chain, 4.2e-7 and 4.1e-7 with 512 elements;
// with bf16 parts 2.8e-7 and 2.6e-7 with 512, 2.5e-7 and 1.8e-7 with 128, at the same speed.
template <bool SPLIT>
constexpr int sum_stages() { return SPLIT ? 4 : 16; }
enum : int { KC = 0, KR = 1 };

// One operand of the contraction.
//   KC: base = first byte of row 0 at the first K element; row0 = first tile row; rows = valid rows of the tensor.
//   KR: base = first byte of K row 0 at the tile's first column; rows = valid K rows; width_bytes = valid bytes of the
//       tile's columns (columns past it may read as the next row's data: the caller masks what they produce).
struct Operand {
  const char* base;
  int64_t ld_bytes;
  int row0, rows, width_bytes;
};

// This wavefront's requests of one operand: T / 32 of 1 KiB per stage, its quarter of the operand's LDS tile.
template <int T, int LAYOUT>
struct Loader {
  static constexpr int REQS = T / 32;
  static_assert(REQS == 4 || REQS == 2, "128 or 64 tile rows");
  const char* base;        // first row of the wavefront's quarter, K tile 0
  int64_t ld_bytes;
  int rows;                // valid rows of the quarter (KC), valid K rows from the quarter's first on (KR)
  int k_bytes, width_bytes;
  uint32_t v[REQS], chunk[REQS];
  __device__ __forceinline__ void init(const Operand& s, int k_elems) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    ld_bytes = s.ld_bytes; k_bytes = k_elems * 4; width_bytes = s.width_bytes;
    if (LAYOUT == KC) {
      const int r0 = wave * (T / 4);
      base = s.base + (int64_t)(s.row0 + r0) * s.ld_bytes;
      rows = max(0, min(s.rows - s.row0 - r0, T / 4));
#pragma unroll
      for (int i = 0; i < REQS; ++i) {
        const int row = i * 8 + (lane >> 3), c = (lane & 7) ^ (((r0 + row) >> 1) & 7);
        v[i] = (uint32_t)(row * s.ld_bytes) + c * 16;
        chunk[i] = c * 16;
      }
    } else {
      constexpr int CHUNKS = T / 4;                         // 16-byte chunks per K row
      const int r0 = wave * 8;
      base = s.base + (int64_t)r0 * s.ld_bytes;
      rows = min(s.rows, k_elems) - r0;
#pragma unroll
      for (int i = 0; i < REQS; ++i) {
        const int kr = i * (64 / CHUNKS) + lane / CHUNKS, c = (lane % CHUNKS) ^ ((((r0 + kr) >> 2) & 1) << 3);
        v[i] = (uint32_t)(kr * s.ld_bytes) + c * 16;
        chunk[i] = 0;
      }
    }
  }
  __device__ __forceinline__ void issue(char* tile, int kt) const {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t off = LAYOUT == KC ? (int64_t)kt * (BK * 4) : (int64_t)kt * BK * ld_bytes;
    uint32_t n = 0;                                         // bytes in reach of the quarter at this K tile
    if (LAYOUT == KC) {
      if (rows > 0) n = (uint32_t)((int64_t)(rows - 1) * ld_bytes + k_bytes - off);
    } else {
      const int kr = max(0, min(rows - kt * BK, 8));
      if (kr > 0) n = (uint32_t)((int64_t)(kr - 1) * ld_bytes + width_bytes);
    }
    const uint64_t addr = (uint64_t)(uintptr_t)(base + off);
    u32x4 r = {(uint32_t)addr, (uint32_t)(addr >> 32) & 0xFFFFu, n, 0x00020000u};
    r[0] = __builtin_amdgcn_readfirstlane(r[0]);
    r[1] = __builtin_amdgcn_readfirstlane(r[1]);
    r[2] = __builtin_amdgcn_readfirstlane(r[2]);
    uint32_t o[REQS];
#pragma unroll
    for (int i = 0; i < REQS; ++i) {
      o[i] = v[i];
      if (LAYOUT == KC) o[i] = kt * (BK * 4) + (int)chunk[i] < k_bytes ? o[i] : 0xFFFFFF00u;   // out of range: reads as zero
    }
    // One piece of assembly with the wait states that a descriptor made by vector instructions asks for (see mainloop_fast.h).
    const uint32_t dst = fast::lds_address(tile + wave * (T * 32));
    if constexpr (REQS == 4)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %5, 0 offen lds\n\t"
                   "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %5, 0 offen lds\n\t"
                   "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tbuffer_load_dwordx4 %3, %5, 0 offen lds\n\t"
                   "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tbuffer_load_dwordx4 %4, %5, 0 offen lds"
                   :: "s"(dst), "v"(o[0]), "v"(o[1]), "v"(o[2]), "v"(o[3]), "s"(r) : "memory", "m0", "scc");
    else
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %3, 0 offen lds\n\t"
                   "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, 0 offen lds"
                   :: "s"(dst), "v"(o[0]), "v"(o[1]), "s"(r) : "memory", "m0", "scc");
  }
};

// Fragments of one K group of 8: per 32-row block this lane's four K values.
template <int T, int LAYOUT>
__device__ __forceinline__ void read_frags(f32x4 (&f)[T / 64], const char* tile, int wsub, int g) {
  const int l32 = threadIdx.x & 31, half = (threadIdx.x >> 5) & 1;
#pragma unroll
  for (int i = 0; i < T / 64; ++i) {
    const int row = wsub * (T / 2) + i * 32 + l32;
    if (LAYOUT == KC) {
      f[i] = *reinterpret_cast<const f32x4*>(tile + row * 128 + (((2 * g + half) ^ ((l32 >> 1) & 7)) << 4));
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        f[i][j] = *reinterpret_cast<const float*>(tile + (8 * g + 4 * half + j) * (T * 4) + ((row * 4) ^ (half << 7)));
    }
  }
}

template <int T>
constexpr int stages() { return T == 128 ? 2 : 4; }         // 64 KiB of LDS either way: two workgroups per CU
template <int T>
constexpr int lds_bytes() { return stages<T>() * 2 * T * BK * 4; }

// Eight fp32 values times 2^PART_SHIFT as three bf16 each, exactly (8 bits of mantissa each, rounded to nearest).  Without the factor
// the third part of a value below 2^-109 falls under bf16's smallest normal number, 2^-126, and the parts lose bits: columns of
// H or W or upstream gradients of 1e-36 gave gradients off by 5e-4.  With it the smallest fp32 subnormal becomes 2^-109, and
// every value below 2^87 has its parts.  The factors leave a sum where it is added to the tile's; the multiplications cost 5 %
// (1000 x 512 x 10007 102 + 255 -> 108 + 271 us, 4096 x 1024 x 32768 1540 + 5180 -> 1633 + 5590).
constexpr int PART_SHIFT = 40;
constexpr float PART_FACTOR = (float)(1ll << PART_SHIFT), SUM_FACTOR = 1.f / PART_FACTOR / PART_FACTOR;
struct Split { bf16x8 h, m, l; };
__device__ __forceinline__ Split split(const f32x4& x0, const f32x4& x1, float factor) {
  union { bf16x8 v; uint32_t w[4]; } h, m, l;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const float a = factor * (p < 2 ? x0[2 * p] : x1[2 * p - 4]), b = factor * (p < 2 ? x0[2 * p + 1] : x1[2 * p - 3]);
    h.w[p] = f32x2_to_bf16x2_bits(a, b);
    const float ra = a - __uint_as_float(h.w[p] << 16), rb = b - __uint_as_float(h.w[p] & 0xFFFF0000u);
    m.w[p] = f32x2_to_bf16x2_bits(ra, rb);
    l.w[p] = f32x2_to_bf16x2_bits(ra - __uint_as_float(m.w[p] << 16), rb - __uint_as_float(m.w[p] & 0xFFFF0000u));
  }
  return Split{h.v, m.v, l.v};
}

// The bf16 instruction's sums round down (sums of either sign: -0.33 of sqrt(K) 2^-24 on average at K = 512, against 2.8 rms), which a
// log-sum-exp does not average out: every other block of A rows is multiplied negated, at no cost.  Error of the
// log-sum-exp, fp32 products / parts / parts with the sign: 4096 x 1024 x 8192 5.74 / 5.69 / 5.60e-8, 1000 x 512 x 10007 5.46 / 5.49 /
// 5.46e-8, 2048 x 1024 x 32768 5.33 / 5.36 / 5.28e-8.
__device__ __forceinline__ constexpr float block_sign(int i) { return i & 1 ? -1.f : 1.f; }

// acc = A_tile . B_tile^T over k_elems of K.  On return every wavefront has passed a barrier after its last LDS read.  `blocks`: bit
// (i, j) at i T / 64 + j, which blocks this wavefront multiplies (fp32 products; the others stay zero).
template <int T, int LA, int LB, bool SPLIT>
__device__ __forceinline__ void mainloop_as(const Operand& A, const Operand& B, int k_elems, char* lds,
                                         f32x16 (&acc)[T / 64][T / 64], uint32_t blocks = ~0u) {
  constexpr int W = T / 64, NS = stages<T>(), OPER = T * BK * 4, STAGE = 2 * OPER, LOADS = 2 * (T / 32);
#pragma unroll
  for (int i = 0; i < W; ++i)
#pragma unroll
    for (int j = 0; j < W; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  const int KT = (k_elems + BK - 1) / BK;
  Loader<T, LA> la;
  Loader<T, LB> lb;
  la.init(A, k_elems);
  lb.init(B, k_elems);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int s = 0; s < NS - 1 && s < KT; ++s) {
    la.issue(lds + s * STAGE, s);
    lb.issue(lds + s * STAGE + OPER, s);
  }
  for (int kb = 0; kb < KT; kb += sum_stages<SPLIT>()) {
    const int kb_end = min(KT, kb + sum_stages<SPLIT>());
    f32x16 part[W][W];
#pragma unroll
    for (int i = 0; i < W; ++i)
#pragma unroll
      for (int j = 0; j < W; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) part[i][j][r] = 0.f;
    for (int kt = kb; kt < kb_end; ++kt) {
      // tile kt has landed once only the requests of the later tiles are in flight; this wavefront's LDS reads of the
      // stage that is requested next (tile kt - 1's) have returned
      switch (min(NS - 2, KT - 1 - kt)) {
        case 0: fast::wait_vm_and_lds<0>(); break;
        case 1: fast::wait_vm_and_lds<LOADS>(); break;
        default: fast::wait_vm_and_lds<2 * LOADS>(); break;
      }
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      if (kt + NS - 1 < KT) {
        char* dst = lds + (kt + NS - 1) % NS * STAGE;
        la.issue(dst, kt + NS - 1);
        lb.issue(dst + OPER, kt + NS - 1);
      }
      const char* st = lds + kt % NS * STAGE;
      if constexpr (SPLIT) {
#pragma unroll
        for (int g = 0; g < BK / 8; g += 2) {
          f32x4 x[2][W];
          Split a[W], b[W];
          read_frags<T, LA>(x[0], st, wave >> 1, g);
          read_frags<T, LA>(x[1], st, wave >> 1, g + 1);
#pragma unroll
          for (int i = 0; i < W; ++i) a[i] = split(x[0][i], x[1][i], block_sign(i) * PART_FACTOR);
          read_frags<T, LB>(x[0], st + OPER, wave & 1, g);
          read_frags<T, LB>(x[1], st + OPER, wave & 1, g + 1);
#pragma unroll
          for (int j = 0; j < W; ++j) b[j] = split(x[0][j], x[1][j], PART_FACTOR);
          auto products = [&](auto pa, auto pb) {
#pragma unroll
            for (int i = 0; i < W; ++i)
#pragma unroll
              for (int j = 0; j < W; ++j) part[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i].*pa, b[j].*pb, part[i][j], 0, 0, 0);
          };
          products(&Split::l, &Split::h);
          products(&Split::h, &Split::l);
          products(&Split::m, &Split::m);
          products(&Split::m, &Split::h);
          products(&Split::h, &Split::m);
          products(&Split::h, &Split::h);
        }
      } else
#pragma unroll
      for (int g = 0; g < BK / 8; ++g) {
        f32x4 a[W], b[W];
        read_frags<T, LA>(a, st, wave >> 1, g);
        read_frags<T, LB>(b, st + OPER, wave & 1, g);
        if constexpr (W == 1) {
#pragma unroll
          for (int k = 0; k < 4; ++k) part[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[0][k], b[0][k], part[0][0], 0, 0, 0);
        } else {
#pragma unroll
          for (int i = 0; i < W; ++i)
#pragma unroll
            for (int j = 0; j < W; ++j)
              if (blocks >> (i * W + j) & 1) {
#pragma unroll
                for (int k = 0; k < 4; ++k) part[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][k], b[j][k], part[i][j], 0, 0, 0);
              }
        }
      }
      asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int i = 0; i < W; ++i)
#pragma unroll
      for (int j = 0; j < W; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = SPLIT ? fmaf(part[i][j][r], block_sign(i) * SUM_FACTOR, acc[i][j][r]) : acc[i][j][r] + part[i][j][r];
  }
  fast::wait_vm_and_lds<0>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int T, int LA, int LB>
__device__ __forceinline__ void mainloop(const Operand& A, const Operand& B, int k_elems, char* lds,
                                         f32x16 (&acc)[T / 64][T / 64]) {
  mainloop_as<T, LA, LB, T == 128>(A, B, k_elems, lds, acc);
  if constexpr (T == 128) {
    // An infinity, a NaN, a value from 2^87 or a sum from 2^47 on has no such parts or sums: what it is in comes out as NaN or
    // infinity.  The tile is then done again as it is, for those elements alone (and blocks of them): which method an element is computed by depends
    // on its own row and column, not on what shares the tile, so that the backward (which leaves out rows) repeats the forward's logits.
    // Such calls pay for both: 1000 x 512 x 10007 forward + backward 106 + 267 us, 123 + 390 with one infinity in W, 169 + 467 with a
    // row of NaN in H (fp32 products throughout: 116 + 340 either way; whole tiles again: 134 + 432 and 204 + 523).
    auto finite = [](float x) { return x * 0.f == 0.f; };
    uint32_t blocks = 0;      // of this wavefront that hold such an element
#pragma unroll
    for (int i = 0; i < T / 64; ++i)
#pragma unroll
      for (int j = 0; j < T / 64; ++j) {
        float bad = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) bad = fmaf(acc[i][j][r], 0.f, bad);
        blocks |= __ballot(!finite(bad)) ? 1u << (i * (T / 64) + j) : 0u;
      }
    if (__syncthreads_or(blocks)) {
      f32x16 whole[T / 64][T / 64];
      mainloop_as<T, LA, LB, false>(A, B, k_elems, lds, whole, blocks);
#pragma unroll
      for (int i = 0; i < T / 64; ++i)
#pragma unroll
        for (int j = 0; j < T / 64; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] = finite(acc[i][j][r]) ? acc[i][j][r] : whole[i][j][r];
    }
  }
}

}  // namespace f32
}  // namespace flce
