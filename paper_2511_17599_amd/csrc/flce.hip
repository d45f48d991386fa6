// C-ABI entry points of libflce (see include/flce.h): argument checks, the launch
// plan (windows, chunks, workspace layout) and the launch sequences.  Host code
// only; every step of the path runs in the kernels of kernels.h.
#include "../../include/flce.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <mutex>
#include <vector>

#include "kernels.h"
#include "probe.h"

// Workspace of flce_forward_static, the forward for callers that cannot allocate: a file-scope device array.
// Every GPU the library is loaded on holds its own copy, at its own address, until the process ends.  In host
// code this name is only a handle for hipGetSymbolAddress; kernels are given the address that call returns.
static __device__ __align__(256) unsigned char scratch[FLCE_STATIC_SCRATCH_BYTES];

namespace flce {
namespace {

constexpr int64_t ALIGN = 256;
constexpr int NUM_CU = 256;   // MI355X; the plan must not depend on a device query
// Most K slices of a contraction launch.  One output tile (256 rows, d <= 256) over a long vocabulary is where many help:
// 256 rows, d = 128, V = 82194 has 321 K tiles; with 8 slices (8 busy CUs)
// the whole step took 318 us, with 64 it takes 134 (200 x 1024 x 50257: 317 and 210).
constexpr int MAX_SPLIT = 64;
// Most bytes that a plan spends on the forward's copy of H at a ragged hidden size, and on the fp32 tiles of the K slices of
// one contraction launch (60000 random shapes up to 140000 x 8192 x 262144: five would take more, 617 MB at most).
constexpr int64_t BYTES_CAP = (int64_t)512 << 20;

int64_t align_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }
int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

int env_int(const char* name, int dflt, int lo, int hi) {
  const char* s = std::getenv(name);
  if (!s || !*s) return dflt;
  long v = std::strtol(s, nullptr, 10);
  if (v < lo) v = lo;
  if (v > hi) v = hi;
  return (int)v;
}

// The tuning knobs of the launch plan.  Read from the environment once, when the first call needs them, and
// fixed for the process from then on (flce_tuning_reload reads them again): a plan never changes between the
// sizing of a workspace and its use, and no call touches the environment afterwards.
struct Tuning {
  int windows, vc_tiles, nc_tiles, splitk_dh, splitk_dw, generic, tile;
};
std::mutex g_tuning_mu;
bool g_tuning_loaded = false;
Tuning g_tuning;

Tuning read_tuning_from_env() {
  Tuning t;
  t.windows = env_int("FLCE_WINDOWS", 0, 0, 1 << 16);
  t.vc_tiles = env_int("FLCE_VC_TILES", 0, 0, 4096);
  t.nc_tiles = env_int("FLCE_NC_TILES", 128, 1, 4096);
  t.splitk_dh = env_int("FLCE_SPLITK_DH", 0, 0, MAX_SPLIT);
  t.splitk_dw = env_int("FLCE_SPLITK_DW", 0, 0, MAX_SPLIT);
  t.generic = env_int("FLCE_GENERIC", 0, 0, 1);
  t.tile = env_int("FLCE_TILE", 0, 0, TILE);
  if (t.tile != TILE && t.tile != 128) t.tile = 0;
  return t;
}

Tuning tuning() {
  std::lock_guard<std::mutex> lk(g_tuning_mu);
  if (!g_tuning_loaded) { g_tuning = read_tuning_from_env(); g_tuning_loaded = true; }
  return g_tuning;
}

struct Plan {
  int64_t N, d, V;
  int esize;
  int n_rb, n_vt;          // 256-row tiles of tokens / vocabulary
  int tile, fwd_tile;      // output tile edge of the main loop, backward and forward (bf16: 256 or 128, fp32: 128 or 64)
  int64_t npad;
  // forward
  int n_win;
  int64_t off_part, off_blk_loss, off_blk_cnt, off_blk_oor, off_wpart, off_wsum, off_zbar, off_fHT, fwd_bytes;
  // backward
  int n_vch, n_nch;        // chunks along vocabulary / tokens
  int vc_tiles, nc_tiles;  // largest chunk, in tiles
  int64_t ld_v, ld_n;      // elements per row of the buffers whose rows run over a vocabulary / row chunk: the
                           // chunk's extent plus 64, so that rows never lie a power of two apart
  bool fast;               // tuned bf16 loop: W, Hc and G read in place by the contractions
  bool ragged;             // its form for hidden sizes that are no multiple of a K step's 32 elements
  bool hkr;                // forward / recompute read a pre-tiled copy of H (tuned loop, unless the caller rules the copy out)
  bool fwd_copy;           // the forward makes that copy (long enough for it to pay)
  int split_dh, split_dw;  // K slices of the dH / dW contraction launches (1 = unsplit)
  bool pair;               // dW and dH of the only chunk go out as one launch
  int64_t off_Hc, off_rowmap, off_tgt, off_lsec, off_gamc, off_HT, off_WT, off_G, off_GT, off_dHacc, off_dWacc, off_partial, off_partial_dh, bwd_bytes;
};

// A contraction launch of more than one round of workgroups whose last round would be mostly empty: the output-row
// tiles of that last round ("tail") are launched on their own with their K extent cut into `slices` slices (summed
// in slice order by splitk_reduce_kernel, like any split-K launch), so that the tail takes 1 / slices of a round.
// rows = 0: no tail (one round or less; more than four rounds, where the last one matters little and the partial
// sums would cost workspace for it; a last round that is more than half full; a launch that is split anyway).
struct TailSplit { int rows, slices; };
TailSplit tail_split(int64_t out_row_tiles, int64_t n_mt, int n_split, int64_t k_tiles) {
  if (n_split != 1) return {0, 1};
  const int64_t tiles = out_row_tiles * n_mt;
  if (tiles <= NUM_CU || tiles > 4 * NUM_CU) return {0, 1};
  const int64_t body_rows = tiles / NUM_CU * NUM_CU / n_mt;
  const int64_t rows = out_row_tiles - body_rows;
  if (rows <= 0 || body_rows <= 0) return {0, 1};
  // whole slices of at least two 256-element K tiles each, at most 8
  const int64_t slices = std::min<int64_t>(std::min<int64_t>(NUM_CU / (rows * n_mt), 8), k_tiles / 2);
  if (slices < 2) return {0, 1};
  return {(int)rows, (int)slices};
}

// The tuned bf16 loop needs every tile's address window within reach of a buffer descriptor: offsets and the record count are unsigned 32-bit, and
// the zero-filled overshoot of a last K stage (up to 32 rows, with the tile's columns and the bias of the offsets) must not wrap 2^32.
// The `generic` knob forces the generic loop everywhere.
bool window_ok(int64_t k_rows, int64_t ld_bytes) {
  return (k_rows + 32) * ld_bytes + TILE * 2 + fast::BIAS < ((int64_t)1 << 32);
}
bool fast_loop_ok(const Plan& p, const Tuning& tn) {
  if (p.esize != 2 || tn.generic) return false;
  const int64_t vc = (int64_t)p.vc_tiles * TILE, nc = (int64_t)p.nc_tiles * TILE;
  const int64_t ld_hw = p.d * 2, ld_g = p.ld_v * 2;
  return window_ok(257, ld_hw) && window_ok(257, ld_g) &&      // K-contiguous tiles
         window_ok(vc, ld_hw) && window_ok(nc, ld_hw) && window_ok(nc, ld_g);   // K over memory rows
}

// The least number of slices above n whose longest slice is shorter than with n.
int64_t next_slices(int64_t k_tiles, int64_t n) {
  const int64_t len = ceil_div(k_tiles, n);
  return len > 1 ? ceil_div(k_tiles, len - 1) : MAX_SPLIT + 1;
}
// Tiles of 128 in sequence on a CU; one alone is slower than half of two.
double small_waves(int64_t tiles) { return tiles <= NUM_CU ? 1.3 : 2.0 * (double)ceil_div(tiles, 2 * NUM_CU); }
// A pass over all logits with tiles of a given edge, in us (bf16; the rule that uses it is in plan_base).
double logits_us(const Plan& p, int tile, double ends256, double ends128) {
  const double steps = (double)ceil_div(p.d, 32);
  const int64_t tiles = ceil_div(p.N, tile) * ceil_div(p.V, tile);
  if (tile == TILE) return (double)ceil_div(tiles, NUM_CU) * (0.775 * steps + ends256);
  return small_waves(tiles) * (0.28 * steps + 0.12 * std::max(0.0, steps - 64.0) + ends128);
}

// The plan in three parts: what both directions need, the forward's and the backward's.  A call plans its own direction only:
// flce_workspace_bytes, mean of 150 random shapes on one core of the host, 2.4 us in either direction with everything planned
// and every number of K slices tried, 0.7 forward and 1.1 backward as it is (0.7 without any search of slices or windows).
bool plan_base(int64_t N, int64_t d, int64_t V, flce_dtype dt, const Tuning& tn, bool allow_h_copy, Plan& p) {
  if (N <= 0 || d <= 0 || V <= 0 || (d % 8) != 0) return false;
  if (N > 0x7FFFFF00ll || V > 0x7FFFFF00ll || d > (1 << 24)) return false;
  if (dt != FLCE_DTYPE_BF16 && dt != FLCE_DTYPE_F32) return false;
  p.N = N; p.d = d; p.V = V;
  p.esize = dt == FLCE_DTYPE_BF16 ? 2 : 4;
  p.n_rb = (int)ceil_div(N, TILE);
  p.n_vt = (int)ceil_div(V, TILE);
  p.npad = (int64_t)p.n_rb * TILE;

  // Backward staging: a fixed-size G tile of at most vc x nc 256-tiles.
  const int nc_max = tn.nc_tiles;
  // Automatic vocabulary chunk: 128 tiles; with few token rows the same staging bytes reach further along the
  // vocabulary (at most 128 x 32 tiles of G, 512 MiB in bf16, up to 512 vocabulary tiles), which saves whole
  // launches and the fp32 running sum of dH on short-sequence shapes.  Kept within a buffer descriptor's reach.
  int vc_max = tn.vc_tiles;
  if (vc_max == 0) {
    const int64_t nct = std::min<int64_t>(p.n_rb, nc_max);
    vc_max = (int)std::max<int64_t>(128, std::min<int64_t>(512, 4096 / nct));
    const int64_t reach = (((int64_t)1 << 32) / (d * p.esize) - 64) / TILE;
    if (vc_max > 128 && reach < vc_max) vc_max = (int)std::max<int64_t>(128, reach);
  }
  // Chunks of the full size plus a remainder, so that launches of full chunks come out in whole rounds of 256
  // workgroups (128 tiles times any even tile count); an even split only when the remainder would be a sliver.
  auto chunking = [](int tiles, int cmax, int& n_chunks, int& chunk) {
    n_chunks = (int)ceil_div(tiles, cmax);
    const int rem = tiles - (n_chunks - 1) * cmax;
    chunk = (n_chunks == 1 || rem * 4 >= cmax) ? std::min(tiles, cmax) : (int)ceil_div(tiles, n_chunks);
  };
  chunking(p.n_vt, vc_max, p.n_vch, p.vc_tiles);
  chunking(p.n_rb, nc_max, p.n_nch, p.nc_tiles);
  const int64_t vc_pad = (int64_t)p.vc_tiles * TILE, nc_pad = (int64_t)p.nc_tiles * TILE;
  p.ld_v = vc_pad + 64;
  p.ld_n = nc_pad + 64;
  p.fast = fast_loop_ok(p, tn);
  p.ragged = p.fast && d % 32 != 0;
  p.hkr = allow_h_copy && p.fast;

  p.tile = TILE;
  // fp32: 64-row tiles while there are too few 128-row ones to give every CU more than one.  One line for both directions: the
  // 128-row tiles compute with bf16 parts of the operands and the 64-row ones do not, and where the backward's logit is rounded
  // otherwise than the forward's, exp(logit - lse) - 1 of a confident row is their difference instead of zero (1024 x 512 x 4096,
  // target logits of 165: 2e-4, 5e-6 with the same tiles).  Forward with 64 and with 128, us: 1024 x 512 x 4096 (256 tiles of 128)
  // 61 / 70, 300 x 304 x 12000 (282) 43 / 49, 2000 x 1024 x 2400 (304) 131 / 125; backward 512 x 512 x 4096 (128) 88 / 84,
  // 1024 x 512 x 4096 150 / 114.
  if (dt == FLCE_DTYPE_F32) p.tile = ceil_div(N, 128) * ceil_div(V, 128) < 320 ? 64 : 128;
  p.fwd_tile = p.tile;
  // bf16: 256-row tiles are the faster loop (1.4 PFLOP/s against 0.8 with 128-row ones, which move twice the bytes per
  // flop), but one of them keeps a CU busy for K / 32 x 0.78 us + the work at its end, and where there are too few of them,
  // or K is short, the 128-row ones with two workgroups per CU are done earlier.  Times in us, fitted over 29 shapes from
  // 256 x 1024 x 2048 to 9588 x 128 x 16317; `ends` is what a tile costs beyond its K steps, and very long K loops of
  // several rounds fall back a little further (331 x 3136 x 102294).  Forward + backward with 256- and by this rule:
  // 614 x 2496 x 512 135 -> 65 us, 742 x 384 x 4845 79 / 52, 357 x 1408 x 10140 139 / 98, 4730 x 320 x 4151 137 / 106,
  // 5435 x 104 x 18745 263 / 203, 18786 x 128 x 76178 3074 / 2755; 59 random shapes 1.13x and 1.11x, at worst 0.99x.
  if (p.fast && (tn.tile ? tn.tile == 128 : logits_us(p, 128, 6.5, 0.9) < 0.95 * logits_us(p, TILE, 6.5, 0.9))) p.fwd_tile = 128;
  return true;
}

// wide: the caller has a workspace for the partials of more windows than cover the CUs.
void plan_forward(const Tuning& tn, bool wide, Plan& p) {
  const int64_t N = p.N, d = p.d, V = p.V;
  const bool f32 = p.esize == 4;
  const double steps = (double)ceil_div(d, 32);

  // Windows (Section 3.2.1): enough (row block, window) workgroups to cover the CUs.
  // At least 4, so that the 32 workgroups resident on one XCD are 8 row blocks x 4 windows and
  // share both operands through that XCD's L2 (one window would stream every H block from HBM).
  const int cover = (int)std::min<int64_t>(std::max<int64_t>(4, ceil_div(NUM_CU, p.n_rb)), p.n_vt);
  p.n_win = cover;
  int part_windows = cover;                 // what the partials are sized for
  if (tn.windows) {
    p.n_win = part_windows = std::min(tn.windows, p.n_vt);
  } else {
    // Among the window counts that fill up to 8 rounds of workgroups, the one with the least work in sequence.  bf16
    // (one workgroup per CU): rounds x (tiles of the longest window + `fill`, the start and end of an item, 8 us against
    // 24 ns per K element and tile).  fp32 (two per CU): a CU with two items takes them side by side at half the speed,
    // one alone leaves about a fifth of it unused.  One more than a round is what this avoids: 13 row blocks x 20 windows
    // were 260 items, the last 4 of them a launch as long as the first 256 (3300 x 2048 x 65536 forward: 1187 us, with 19
    // windows 743).  Callers without a workspace may have room for the partials of `cover` windows only (100 x 2112 x 22439
    // without one: 57 us with 88 windows, 36 with 176), and fp32 keeps to them too.
    const int64_t rb = ceil_div(N, p.fwd_tile), vt = ceil_div(V, p.fwd_tile);
    const double fill = 8.0 / (0.0242 * (double)d);
    const double tile_us = p.fwd_tile == TILE ? 0.775 * steps : 0.28 * steps + 0.9;
    auto cost = [&](int64_t win) {
      const int64_t items = rb * win, longest = ceil_div(vt, win);
      // the merge takes 16 threads x 16 windows at a time, 4 us each
      const double merge = f32 ? 0.0 : 4.0 * (double)(ceil_div(win, 256) - 1) / tile_us;
      if (p.fwd_tile == TILE) return (double)ceil_div(items, NUM_CU) * ((double)longest + fill) + merge;
      const double start = f32 ? 0.0 : 1.5 / (0.28 * steps + 0.9), alone = f32 ? 1.2 : 1.3;
      return (items <= NUM_CU ? alone : 2.0 * (double)ceil_div(items, 2 * NUM_CU)) * ((double)longest + start) + merge;
    };
    const int64_t most = wide && !f32 ? std::min<int64_t>(vt, std::max<int64_t>(cover, 8 * NUM_CU / rb)) : cover;
    double least = cost(p.n_win);
    int64_t last = p.n_win;
    for (int r = 1; r <= 8; ++r) {          // per number of rounds the most windows that fit, and of those as few as
      const int64_t fit = std::max<int64_t>(1, std::min<int64_t>(most, r * NUM_CU / rb));      // make the longest no longer
      const int64_t win = std::min(most, std::max<int64_t>(std::min<int64_t>(4, cover), ceil_div(vt, ceil_div(vt, fit))));
      if (win == last) continue;
      last = win;
      const double c = cost(win);
      if (c < 0.99 * least) { p.n_win = (int)win; least = c; }
    }
    part_windows = std::max(cover, p.n_win);
  }
  const int win = part_windows;
  int64_t o = ALIGN;                                  // header
  p.off_part = o;       o = align_up(o + 3ll * win * p.npad * 4, ALIGN);
  p.off_blk_loss = o;   o = align_up(o + (int64_t)p.n_rb * 4, ALIGN);
  p.off_blk_cnt = o;    o = align_up(o + (int64_t)p.n_rb * 4, ALIGN);
  p.off_blk_oor = o;    o = align_up(o + (int64_t)p.n_rb * 4, ALIGN);
  // label smoothing (per-row forward): column sums of W by 1024-row chunks, their sum, mean logit per row
  p.off_wpart = o;      o = align_up(o + ceil_div(V, 1024) * d * 4, ALIGN);
  p.off_wsum = o;       o = align_up(o + d * 4, ALIGN);
  p.off_zbar = o;       o = align_up(o + N * 4, ALIGN);
  p.off_fHT = o;        // sized below, once the loop flavour is known
  const int64_t fwd_fixed = o;

  // The copy takes a launch (5 us) and one pass over H (4 N d bytes at 4 TB/s), and saves the loop about 7 % (2 N d V flops
  // at 1.3 PFLOP/s): below this it costs more than it gives (585 x 384 x 20040 forward 27.9 us
  // with it, 25.7 without; 614 x 2496 x 512 step 159 / 152; 2048 x 1024 x 32000, just above the line, level).
  // Hidden sizes that are no multiple of 32 take it up to a bounded size only: without it such a forward runs in O(N + d)
  // words, and an evaluation sized by those has to fit whatever N and d (H read in place costs 6-20 %: 8192 x 4104 x 128256
  // 7.09 -> 8.49 ms, 32768 x 1048 x 131072 8.44 -> 9.89, 16384 x 520 x 60000 1.07 -> 1.14, below the bound; beyond it
  // 103047 x 7824 x 22916 takes 36.2 ms in 7 MB, 31.2 with the copy in 1.6 GB, 49.0 on the generic loop; same bits).
  const int64_t copy_bytes = align_up(packed_block_offset(p.n_rb, (int)d), ALIGN);
  p.fwd_copy = p.hkr && !(p.ragged && copy_bytes > BYTES_CAP) &&
               (double)N * (double)d * (double)V >= 4.6e10 + 9300.0 * (double)N * (double)d;
  p.fwd_bytes = fwd_fixed + (p.fwd_copy ? copy_bytes : 0);
}

void plan_backward(const Tuning& tn, Plan& p) {
  const int64_t N = p.N, d = p.d;
  const bool f32 = p.esize == 4;
  const int64_t vc_pad = (int64_t)p.vc_tiles * TILE, nc_pad = (int64_t)p.nc_tiles * TILE;
  int64_t o = ALIGN;
  // the counted rows of H: as they are (fp32, generic loop), or pre-tiled for the dW contraction (tuned loop)
  p.off_Hc = o;     o = align_up(o + (p.fast ? packed_cols_offset((int)ceil_div(d, TILE), (int)p.npad) : d * p.npad * p.esize), ALIGN);
  p.off_rowmap = o; o = align_up(o + p.npad * 4, ALIGN);
  p.off_tgt = o;    o = align_up(o + p.npad * 4, ALIGN);
  p.off_lsec = o;   o = align_up(o + p.npad * 4, ALIGN);
  p.off_gamc = o;   o = align_up(o + p.npad * 4, ALIGN);
  p.off_G = o;      o = align_up(o + nc_pad * p.ld_v * p.esize, ALIGN);
  // K-contiguous copies, only for the main loop that cannot read an operand across memory rows
  const bool copies = !f32 && !p.fast;
  p.off_HT = o;     if (copies) o = align_up(o + d * p.npad * p.esize, ALIGN);
                    else if (p.hkr) o = align_up(o + packed_block_offset(p.n_rb, (int)d), ALIGN);
  p.off_WT = o;     if (copies) o = align_up(o + d * p.ld_v * p.esize, ALIGN);
  p.off_GT = o;     if (copies) o = align_up(o + vc_pad * p.ld_n * p.esize, ALIGN);
  p.off_dHacc = o;  if (p.n_vch > 1) o = align_up(o + N * d * 4, ALIGN);
  p.off_dWacc = o;  if (p.n_nch > 1) o = align_up(o + vc_pad * d * 4, ALIGN);
  // Split-K for launches with too few output tiles to occupy the CUs (small N or small d): the K
  // extent is cut into slices whose fp32 tiles are summed in slice order by a second kernel.
  // The contractions of a full chunk with tiles of a given edge: K slices of each, whether both go out as one launch, and
  // the time in us.  A launch takes rounds of workgroups times (K tiles of a slice + `ends` for filling the pipeline and
  // writing the tile out), plus, for a split, the launch that adds the slices and the fp32 tiles written and read back.
  // A K tile (K elements = tile edge) takes 6.2 us in bf16 with 256-tiles and 1.12 with 128-tiles (two workgroups per
  // CU), and at fp32 (likewise two) 5.2 us per CU with 128-tiles, 0.85 with 64-tiles.
  struct Contractions { int split_dh, split_dw; bool pair; double us; };
  auto contractions = [&](int tile) {
    Contractions c{tn.splitk_dh, tn.splitk_dw, false, 0.0};
    const int64_t n_mt = ceil_div(d, tile), unit = TILE / tile;
    const bool small = !f32 && tile != TILE;
    const double k_us = small ? 1.12 : !f32 ? 6.2 : tile == 128 ? 5.2 : 0.85, ends = tile == 64 ? 3.5 : small ? 2.0 : 1.2,
                 tile_us = !f32 && !small ? 0.124 : tile == 64 ? 0.0085 : 0.034, launch = 5.0;
    auto rounds = [&](int64_t wgs) { return small ? small_waves(wgs) : (double)ceil_div(wgs, NUM_CU); };
    auto split_cost = [&](int64_t tiles, int64_t k_tiles, int sp) {
      return rounds(tiles * sp) * ((double)ceil_div(k_tiles, sp) + ends) * k_us +
             (sp > 1 ? launch + tile_us * (double)(tiles * sp) : 0.0);
    };
    auto auto_split = [&](int64_t tiles, int64_t k_tiles, int64_t out_rows) -> int {     // a split has to win by 5 %
      int best = 1;
      const int64_t most = std::min(std::min<int64_t>(MAX_SPLIT, BYTES_CAP / (out_rows * d * 4)), k_tiles);
      double least = 0.95 * split_cost(tiles, k_tiles, 1);
      // Of the numbers of slices with the same longest slice the first costs least, and no cut does better than all CUs
      // sharing the K tiles, the ends of every slice and its sums evenly.
      const double even = launch + (double)(tiles * k_tiles) * k_us / NUM_CU;
      for (int64_t sp = 2; sp <= most; sp = next_slices(k_tiles, sp)) {
        if (even + (double)(tiles * sp) * (k_us * ends / NUM_CU + tile_us) >= least) break;
        const double cost = split_cost(tiles, k_tiles, (int)sp);
        if (cost < least) { least = cost; best = (int)sp; }
      }
      return best;
    };
    const int64_t tiles_dh = p.nc_tiles * unit * n_mt, k_dh = p.vc_tiles * unit;
    const int64_t tiles_dw = p.vc_tiles * unit * n_mt, k_dw = p.nc_tiles * unit;
    if (c.split_dh == 0) c.split_dh = auto_split(tiles_dh, k_dh, nc_pad);
    if (c.split_dw == 0) c.split_dw = auto_split(tiles_dw, k_dw, vc_pad);
    c.split_dh = (int)std::min<int64_t>(c.split_dh, k_dh);
    c.split_dw = (int)std::min<int64_t>(c.split_dw, k_dw);
    c.us = split_cost(tiles_dh, k_dh, c.split_dh) + split_cost(tiles_dw, k_dw, c.split_dw) + launch;
    // One launch for both: K is cut so that no slice of either is longer than `len` K tiles and all of them together are
    // at most two rounds of workgroups; taken where that beats one launch after the other, and only while the uncut tiles
    // of both are resident together (742 x 384 x 4845 102 -> 82 us, 2048 x 512 x 8000 149 -> 126, fp32 849 x 216 x 1732
    // 89 -> 80, the row preparation without its own scan launch included).
    if (p.n_vch == 1 && p.n_nch == 1 && (p.fast || f32) && tn.splitk_dh == 0 && tn.splitk_dw == 0 &&
        tiles_dh + tiles_dw <= (tile != TILE ? 2 : 1) * NUM_CU) {
      double best = 0.97 * c.us;
      auto consider = [&](int64_t len) {              // false: too many slices, and more of them with any shorter `len`
        const int64_t sh = ceil_div(k_dh, len), sw = ceil_div(k_dw, len);
        const int64_t wgs = tiles_dh * sh + tiles_dw * sw;
        if (sh > MAX_SPLIT || sw > MAX_SPLIT || wgs > 2 * NUM_CU) return false;
        const double cost = rounds(wgs) * ((double)len + ends) * k_us + (sh > 1 || sw > 1 ? launch : 0.0) +
                            tile_us * (double)((sh > 1 ? tiles_dh * sh : 0) + (sw > 1 ? tiles_dw * sw : 0));
        if (cost < best) { best = c.us = cost; c.pair = true; c.split_dh = (int)sh; c.split_dw = (int)sw; }
        return true;
      };
      int64_t next_dh = 1, next_dw = 1;               // the slice lengths at which one of the two numbers of slices changes
      for (int64_t sp = 1; sp <= MAX_SPLIT; sp = std::min(next_dh, next_dw)) {
        if (sp == next_dh) next_dh = consider(ceil_div(k_dh, sp)) ? next_slices(k_dh, sp) : MAX_SPLIT + 1;
        if (sp == next_dw) next_dw = consider(ceil_div(k_dw, sp)) ? next_slices(k_dw, sp) : MAX_SPLIT + 1;
      }
    }
    return c;
  };
  Contractions con = contractions(p.tile);
  if (p.fast && tn.tile == 128) {
    p.tile = 128;
    con = contractions(128);
  } else if (p.fast && tn.tile == 0) {
    const double chunks = (double)p.n_vch * p.n_nch;
    const double recompute = logits_us(p, 128, 8.0, 1.6), big = 0.97 * (logits_us(p, TILE, 8.0, 1.6) + chunks * con.us);
    if (recompute < big) {
      const Contractions small = contractions(128);
      if (recompute + chunks * small.us < big) { p.tile = 128; con = small; }
    }
  }
  p.split_dh = con.split_dh; p.split_dw = con.split_dw; p.pair = con.pair;
  const int64_t n_mt = ceil_div(d, p.tile);
  p.off_partial = o;
  {
    const int64_t dh_bytes = p.split_dh > 1 ? align_up((int64_t)p.split_dh * nc_pad * d * 4, ALIGN) : 0;
    int64_t bytes = p.split_dw > 1 ? align_up((int64_t)p.split_dw * vc_pad * d * 4, ALIGN) : 0;
    // one after the other they share the buffer, side by side they do not
    p.off_partial_dh = p.pair ? o + bytes : o;
    bytes = p.pair ? bytes + dh_bytes : std::max(bytes, dh_bytes);
    if (p.fast && !p.pair && p.tile == TILE) {
      // tails of the launches that occur: full chunks and the last (shorter) chunk of either direction
      const int64_t v_last = p.n_vt - (int64_t)(p.n_vch - 1) * p.vc_tiles, n_last = p.n_rb - (int64_t)(p.n_nch - 1) * p.nc_tiles;
      for (const int64_t vt : {(int64_t)p.vc_tiles, v_last})
        for (const int64_t nt : {(int64_t)p.nc_tiles, n_last}) {
          const TailSplit tw = tail_split(vt, n_mt, p.split_dw, nt), th = tail_split(nt, n_mt, p.split_dh, vt);
          if (tw.rows) bytes = std::max(bytes, (int64_t)tw.slices * tw.rows * TILE * d * 4);
          if (th.rows) bytes = std::max(bytes, (int64_t)th.slices * th.rows * TILE * d * 4);
        }
    }
    o = align_up(o + bytes, ALIGN);
  }
  p.bwd_bytes = o;
}

enum : int { PLAN_FORWARD = 1, PLAN_BACKWARD = 2, PLAN_BOTH = 3 };   // 0: the shape's check only
// allow_h_copy: the caller has a workspace for the pre-tiled copy of H.
bool make_plan(int parts, int64_t N, int64_t d, int64_t V, flce_dtype dt, Plan& p, bool allow_h_copy = true, bool wide = true) {
  const Tuning tn = tuning();
  if (!plan_base(N, d, V, dt, tn, allow_h_copy, p)) return false;
  if (parts & PLAN_FORWARD) plan_forward(tn, wide, p);
  if (parts & PLAN_BACKWARD) plan_backward(tn, p);
  return true;
}

// Optional per-launch event timing (flce_profile_*).
struct ProfRec { int cls; hipEvent_t a, b; };
struct Prof {
  std::mutex mu;
  bool on = false;
  std::vector<hipEvent_t> pool;
  std::vector<ProfRec> recs;
  hipEvent_t get() {
    if (!pool.empty()) { hipEvent_t e = pool.back(); pool.pop_back(); return e; }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
  }
};
Prof g_prof;

struct ProfScope {
  hipStream_t st;
  hipEvent_t b = nullptr;
  ProfScope(int cls, hipStream_t s) : st(s) {
    if (!g_prof.on) return;
    std::lock_guard<std::mutex> lk(g_prof.mu);
    hipEvent_t a = g_prof.get();
    b = g_prof.get();
    if (!a || !b) { b = nullptr; return; }
    (void)hipEventRecord(a, st);
    g_prof.recs.push_back(ProfRec{cls, a, b});
  }
  ~ProfScope() { if (b) (void)hipEventRecord(b, st); }
};

template <typename K>
hipError_t allow_big_lds(K kernel, int bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

// The kernels of one (storage type, main loop) pair need the large dynamic LDS allowance; it is a property of
// the loaded code object on a device, so it is set once per device and pair, not per call.
constexpr int MAX_DEVICES = 64;

template <typename T, typename L>
hipError_t set_lds_allowances() {
  hipError_t e;
  if ((e = allow_big_lds(fwd_tiles_kernel<T, L, false>, L::LDS)) != hipSuccess) return e;
  if constexpr (L::TUNED) {
    if ((e = allow_big_lds(fwd_tiles_kernel<T, L, true>, L::LDS)) != hipSuccess) return e;
    if ((e = allow_big_lds(recompute_kernel<T, L, true>, L::LDS)) != hipSuccess) return e;
    if ((e = allow_big_lds(recompute_kernel<T, L, true, true>, L::LDS)) != hipSuccess) return e;
    if ((e = allow_big_lds(contract_kernel<T, typename L::Even, OPS_DH_TR>, L::LDS)) != hipSuccess) return e;
    if ((e = allow_big_lds(contract_kernel<T, typename L::Even, OPS_DW_TR>, L::LDS)) != hipSuccess) return e;
    if ((e = allow_big_lds(contract_pair_kernel<T, typename L::Even, OPS_DW_TR, OPS_DH_TR>, L::LDS)) != hipSuccess) return e;
  } else {
    if ((e = allow_big_lds(recompute_kernel<T, L, false>, L::LDS)) != hipSuccess) return e;
    if ((e = allow_big_lds(recompute_kernel<T, L, false, true>, L::LDS)) != hipSuccess) return e;
    if constexpr (L::TRANSPOSING) {
      if ((e = allow_big_lds(contract_kernel<T, L, OPS_DH_F32>, L::LDS)) != hipSuccess) return e;
      if ((e = allow_big_lds(contract_kernel<T, L, OPS_DW_F32>, L::LDS)) != hipSuccess) return e;
      if ((e = allow_big_lds(contract_pair_kernel<T, L, OPS_DW_F32, OPS_DH_F32>, L::LDS)) != hipSuccess) return e;
    } else {
      if ((e = allow_big_lds(contract_kernel<T, L, OPS_KC>, L::LDS)) != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

template <typename T, typename L>
hipError_t prepare_kernels() {
  static std::mutex mu;
  static bool done[MAX_DEVICES] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(mu);
  if (done[dev]) return hipSuccess;
  if ((e = set_lds_allowances<T, L>()) != hipSuccess) return e;
  done[dev] = true;
  return hipSuccess;
}

// W holds the p.V vocabulary rows [slice.v_begin, slice.v_begin + p.V) of slice.V_total.  With m_out set the
// call stops after the window merge and hands out the slice's (m, a, z_target) per row.
struct Slice { int64_t V_total, v_begin; };
// Per-row variant: the forward writes one loss per row (label-smoothed by eps), the backward takes one
// upstream gradient per row (device arrays of N floats).
struct PerRow { float* loss_rows_out; const float* grad_rows; float eps; };
// Device words of the caller that receive the range flag and the number of counted rows (either may be null).
struct StatusOut { int32_t* status; int64_t* n_valid; };

// The window merge.  While a row's parts fit one batch of loads, one thread merges them; otherwise 16 threads do where
// the block sums of 64-row blocks fit the arrays (they are padded to 64 entries, and many windows mean few row blocks),
// and 4 threads in 256-row blocks elsewhere.  `launch` gets the kernel's shape: rows, threads per row, loads in flight.
constexpr int MERGE_ONE_BATCH = 8;
template <int R, int G, int LOADS> struct MergeShape { static constexpr int ROWS = R, GROUPS = G, U = LOADS; };
template <typename F>
int merge_dispatch(int64_t N, int n_parts, F launch) {
  auto blocks = [&](auto shape) {
    const int n_blk = (int)ceil_div(N, decltype(shape)::ROWS);
    launch(shape, n_blk);
    return n_blk;
  };
  if (n_parts <= MERGE_ONE_BATCH) return blocks(MergeShape<256, 1, 8>{});
  if (ceil_div(N, 64) <= ALIGN / 4) return blocks(MergeShape<64, 16, 16>{});
  return blocks(MergeShape<256, 4, 16>{});
}
// Returns the number of blocks (entries of the block sums).
int launch_merge(const float* pm, const float* pa, const float* pz, int n_parts, int64_t stride, const int64_t* y, int N,
                 int64_t V_total, int64_t ignore_index, float* lse_out, const LossOut& o, bool fused,
                 float* loss_rows_out, const float* zbar, float eps, hipStream_t st) {
  return merge_dispatch(N, n_parts, [&](auto shape, int n_blk) {
    using S = decltype(shape);
    merge_rows_kernel<S::ROWS, S::GROUPS, S::U><<<n_blk, S::ROWS * S::GROUPS, 0, st>>>(
        pm, pa, pz, n_parts, stride, y, N, V_total, ignore_index, lse_out, o, fused, loss_rows_out, zbar, eps);
  });
}

template <typename T, typename U, typename L>
flce_status forward_t(const Plan& p, const void* H, const void* W, const int64_t* y, int64_t ignore_index,
                      int mean, float* loss_out, float* lse_out, char* ws, hipStream_t st, Slice slice,
                      float* m_out = nullptr, float* a_out = nullptr, float* zt_out = nullptr,
                      PerRow rows = PerRow{nullptr, nullptr, 0.f}, StatusOut so = StatusOut{nullptr, nullptr}) {
  if (prepare_kernels<T, L>() != hipSuccess) return FLCE_ERR_HIP;
  Header* hdr = reinterpret_cast<Header*>(ws);
  float* part = reinterpret_cast<float*>(ws + p.off_part);
  float* blk_loss = reinterpret_cast<float*>(ws + p.off_blk_loss);
  int* blk_cnt = reinterpret_cast<int*>(ws + p.off_blk_cnt);
  int* blk_oor = reinterpret_cast<int*>(ws + p.off_blk_oor);
  // One workgroup per item (row block x window).  With the tuned loop a launch takes at most one round of workgroups
  // (256 items, 512 of 128-row tiles; whole raster groups of 8 row blocks when the window count divides 32): a larger grid's later rounds
  // drift apart over the ~100 tiles of an item and stop sharing their operands in the L2 (measured at 512 row blocks:
  // 361 GB of fabric traffic per forward against 192 GB that the raster should need).
  const int n_rb = (int)ceil_div(p.N, L::TILE), n_vt = (int)ceil_div(p.V, L::TILE);
  const int items = n_rb * p.n_win;
  const int per_launch = [&] { if constexpr (L::TUNED) return NUM_CU * L::PER_CU; return items; }();
  bool hkr = false;
  if constexpr (L::TUNED) hkr = p.fwd_copy;
  T* HT = nullptr;
  if (hkr) {
    if constexpr (L::TUNED) {
      HT = reinterpret_cast<T*>(ws + p.off_fHT);
      // the pre-tiled copy of H, zero padded to whole row blocks: the forward's second operand
      ProfScope ps(FLCE_PROF_FWD_EPILOGUE, st);
      pack_rows_kernel<<<dim3((unsigned)(p.npad / 64), (unsigned)ceil_div(p.d, 128)), 256, 0, st>>>(
          static_cast<const char*>(H), (int)p.N, (int)p.d, reinterpret_cast<char*>(HT));
    }
  }
  {
    ProfScope ps(FLCE_PROF_FWD_TILES, st);
    for (int item0 = 0; item0 < items; item0 += per_launch) {
      const int grid = std::min(per_launch, items - item0);
      if (hkr) {
        if constexpr (L::TUNED)
          fwd_tiles_kernel<T, L, true><<<grid, L::THREADS, L::LDS, st>>>(
              static_cast<const T*>(H), HT, static_cast<const T*>(W), y, (int)p.N, (int)p.d, (int)p.V, ignore_index,
              slice.V_total, slice.v_begin, n_rb, p.n_win, n_vt, (double)n_vt / p.n_win, part, p.npad, item0, hdr);
      } else {
        fwd_tiles_kernel<T, L, false><<<grid, L::THREADS, L::LDS, st>>>(
            static_cast<const T*>(H), nullptr, static_cast<const T*>(W), y, (int)p.N, (int)p.d, (int)p.V, ignore_index,
            slice.V_total, slice.v_begin, n_rb, p.n_win, n_vt, (double)n_vt / p.n_win, part, p.npad, item0, hdr);
      }
    }
  }
  {
    ProfScope ps(FLCE_PROF_FWD_EPILOGUE, st);
    if (m_out) {
      merge_dispatch(p.N, p.n_win, [&](auto shape, int n_blk) {
        using S = decltype(shape);
        merge_rows_partial_kernel<S::ROWS, S::GROUPS, S::U><<<n_blk, S::ROWS * S::GROUPS, 0, st>>>(
            part, p.n_win, p.npad, (int)p.N, m_out, a_out, zt_out);
      });
    } else {
      const int64_t plane = (int64_t)p.n_win * p.npad;
      const float* zbar = nullptr;
      if (rows.loss_rows_out && rows.eps != 0.f) {
        float* wpart = reinterpret_cast<float*>(ws + p.off_wpart);
        float* wsum = reinterpret_cast<float*>(ws + p.off_wsum);
        float* zb = reinterpret_cast<float*>(ws + p.off_zbar);
        const int n_chunks = (int)ceil_div(p.V, 1024);
        colsum_chunks_kernel<T><<<dim3((unsigned)n_chunks, (unsigned)ceil_div(p.d, 16 * Vec16<T>::N)), 256, 0, st>>>(
            static_cast<const T*>(W), (int)p.V, (int)p.d, wpart);
        colsum_finish_kernel<<<(unsigned)ceil_div(p.d, 64), 64, 0, st>>>(wpart, n_chunks, (int)p.d, wsum);
        mean_logit_kernel<T><<<(unsigned)ceil_div(p.N, 4), 256, 0, st>>>(static_cast<const T*>(H), wsum, (int)p.N, (int)p.d,
                                                                         1.0f / (float)p.V, zb);
        zbar = zb;
      }
      // the per-row call has no scalar loss to hand out: the sum goes to a spare word of the header block
      float* scalar = loss_out ? loss_out : reinterpret_cast<float*>(ws + 64);
      launch_merge(part, part + plane, part + 2 * plane, p.n_win, p.npad, y, (int)p.N, slice.V_total, ignore_index, lse_out,
                   LossOut{blk_loss, blk_cnt, blk_oor, hdr, scalar, mean, so.status, so.n_valid}, /*fused=*/true,
                   rows.loss_rows_out, zbar, rows.eps, st);
    }
  }
  return hipGetLastError() == hipSuccess ? FLCE_OK : FLCE_ERR_HIP;
}

template <typename T, typename U, typename L>
flce_status backward_t(const Plan& p, const void* H, const void* W, const int64_t* y, const float* lse,
                       int64_t ignore_index, int mean, GradLoss grad_loss, void* dH, void* dW, char* ws,
                       hipStream_t st, Slice slice, PerRow rows = PerRow{nullptr, nullptr, 0.f}) {
  if (prepare_kernels<T, L>() != hipSuccess) return FLCE_ERR_HIP;
  if (L::TUNED && !p.hkr) return FLCE_ERR_UNSUPPORTED;   // (no caller plans a backward without the copies of H)
  const int N = (int)p.N, d = (int)p.d, V = (int)p.V;
  Header* hdr = reinterpret_cast<Header*>(ws);
  T* Hc = reinterpret_cast<T*>(ws + p.off_Hc);
  int* rowmap = reinterpret_cast<int*>(ws + p.off_rowmap);
  int* tgt_c = reinterpret_cast<int*>(ws + p.off_tgt);
  float* lse_c = reinterpret_cast<float*>(ws + p.off_lsec);
  float* gam_c = reinterpret_cast<float*>(ws + p.off_gamc);
  T* HT = reinterpret_cast<T*>(ws + p.off_HT);
  T* WT = reinterpret_cast<T*>(ws + p.off_WT);
  T* G = reinterpret_cast<T*>(ws + p.off_G);
  T* GT = reinterpret_cast<T*>(ws + p.off_GT);
  float* dHacc = reinterpret_cast<float*>(ws + p.off_dHacc);
  float* dWacc = reinterpret_cast<float*>(ws + p.off_dWacc);
  const int64_t vc_pad = (int64_t)p.vc_tiles * TILE, nc_pad = (int64_t)p.nc_tiles * TILE;
  const int n_mt = (int)ceil_div(d, L::TILE);
  // the plan counts 256-row tiles; this loop's tiles may be a half or a quarter of that
  constexpr int UNIT = TILE / L::TILE;
  const int all_vt = (int)ceil_div(p.V, L::TILE), all_nt = (int)ceil_div(p.N, L::TILE);
  const int npad = (int)p.npad;

  {
    ProfScope ps(FLCE_PROF_BWD_PREP, st);
    const CompactArgs ca{y, N, V, slice.V_total, slice.v_begin, ignore_index, rowmap, tgt_c, hdr};
    const bool scan = N <= COMPACT_HERE;
    if (!scan)
      compact_targets_kernel<<<1, 1024, 0, st>>>(y, N, V, slice.V_total, slice.v_begin, ignore_index, npad, rowmap, tgt_c,
                                                 hdr);
    // lse and Gamma per compact row, zero rows of dH, and the counted rows of H packed together: with the tuned loop
    // pre-tiled for the recompute (in HT's place) and pre-tiled the other way round for dW (in Hc's place); otherwise as
    // they are (Hc), and with the generic loop also transposed [d][npad] (the dW contraction's K-contiguous operand)
    if constexpr (L::TUNED) {
      const dim3 grid((unsigned)(p.npad / 32), (unsigned)ceil_div(d, TILE));
      auto prep = [&](auto kernel) {
        kernel<<<grid, 256, 0, st>>>(static_cast<const char*>(H), d, npad, reinterpret_cast<char*>(HT),
                                     reinterpret_cast<char*>(Hc), lse, lse_c, rows.grad_rows, gam_c, ca,
                                     static_cast<char*>(dH));
      };
      if (scan) prep(prep_rows_tiled_kernel<true>);
      else prep(prep_rows_tiled_kernel<false>);
    } else {
      const dim3 grid((unsigned)(p.npad / 64), (unsigned)ceil_div(d, 64));
      auto prep = [&](auto kernel) {
        kernel<<<grid, 256, 0, st>>>(static_cast<const U*>(H), d, reinterpret_cast<U*>(Hc),
                                     L::TRANSPOSING ? nullptr : reinterpret_cast<U*>(HT), p.npad, lse, lse_c,
                                     rows.grad_rows, gam_c, ca, static_cast<U*>(dH));
      };
      if (scan) prep(prep_rows_kernel<U, true>);
      else prep(prep_rows_kernel<U, false>);
    }
  }

  // With the tuned loop G is staged in blocks of 16 rows x 32 positions (1 KiB), the blocks of a row group one after
  // the other plus one block of skew, so that row groups do not lie a power of two apart; this fits the row-major
  // size the plan reserves (16 rows of ld_v = vc_pad + 64 elements are one block more per group).
  const int64_t g_group_bytes = (vc_pad / 32 + 1) * 1024;
  float* partial = reinterpret_cast<float*>(ws + p.off_partial);
  float* partial_dh = reinterpret_cast<float*>(ws + p.off_partial_dh);
  // K elements per split-K slice: whole tiles
  auto slice_len = [](int k_elems, int n_split) { return (int)ceil_div(ceil_div(k_elems, L::TILE), n_split) * L::TILE; };
  // argument blocks of the three steps of chunk (vc, nc); `Gb` is the staging buffer of that chunk
  auto chunk_vt = [&](int vc, int& vt0, int& n_vt) {
    vt0 = vc * p.vc_tiles * UNIT;
    n_vt = std::min(p.vc_tiles * UNIT, all_vt - vt0);
  };
  auto chunk_nt = [&](int nc, int& nt0, int& n_nt) {
    nt0 = nc * p.nc_tiles * UNIT;
    n_nt = std::min(p.nc_tiles * UNIT, all_nt - nt0);
  };
  auto recompute_args = [&](int vc, int nc, T* Gb) {
    int vt0, n_vt, nt0, n_nt;
    chunk_vt(vc, vt0, n_vt);
    chunk_nt(nc, nt0, n_nt);
    return RecomputeArgs<T>{Hc, HT, static_cast<const T*>(W), tgt_c, lse_c, hdr, npad, d, V, nt0, n_nt, vt0, n_vt,
                            Gb, L::TUNED ? g_group_bytes : p.ld_v, GT, p.ld_n, gam_c, 1.f - rows.eps,
                            rows.eps / (float)slice.V_total};
  };
  // dW[vocab chunk] += G^T . Hc[row chunk]   (contraction over the compact rows of the chunk)
  auto dw_args = [&](int vc, int nc, const T* Gb) {
    int vt0, n_vt, nt0, n_nt;
    chunk_vt(vc, vt0, n_vt);
    chunk_nt(nc, nt0, n_nt);
    int flags = K_COMPACT;
    if (nc > 0) flags |= READ_ACC;
    flags |= (nc + 1 < p.n_nch) ? WRITE_ACC : WRITE_OUT;
    if constexpr (L::TRANSPOSING && !L::TUNED)
      return ContractArgs<T>{Hc + (int64_t)nt0 * L::TILE * d, d, n_nt * L::TILE, d, Gb, p.ld_v, 0, n_nt * L::TILE,
                             nt0 * L::TILE, n_mt, n_vt, dWacc, vt0 * L::TILE, static_cast<T*>(dW), vt0 * L::TILE, V, flags,
                             hdr, rowmap, grad_loss, mean, p.split_dw, slice_len(n_nt * L::TILE, p.split_dw),
                             partial, vc_pad * d};
    else if constexpr (L::TUNED)
      return ContractArgs<T>{Hc, npad, 0, d, Gb, g_group_bytes, n_nt * L::TILE,
                             n_nt * L::TILE, nt0 * L::TILE, n_mt, n_vt, dWacc, vt0 * L::TILE, static_cast<T*>(dW), vt0 * L::TILE,
                             V, flags, hdr, rowmap, grad_loss, mean, p.split_dw,
                             slice_len(n_nt * L::TILE, p.split_dw), partial, vc_pad * d};
    else
      return ContractArgs<T>{HT + (int64_t)nt0 * L::TILE, p.npad, 0, d, GT, p.ld_n, n_vt * L::TILE, n_nt * L::TILE,
                             nt0 * L::TILE, n_mt, n_vt, dWacc, vt0 * L::TILE, static_cast<T*>(dW), vt0 * L::TILE, V, flags,
                             hdr, rowmap, grad_loss, mean, p.split_dw, slice_len(n_nt * L::TILE, p.split_dw), partial,
                             vc_pad * d};
  };
  // dH[row chunk] += G . W[vocab chunk]      (contraction over the vocabulary chunk)
  auto dh_args = [&](int vc, int nc, const T* Gb) {
    int vt0, n_vt, nt0, n_nt;
    chunk_vt(vc, vt0, n_vt);
    chunk_nt(nc, nt0, n_nt);
    // K: the chunk's vocabulary rows, the last tile's up to a whole K step (G is zero past the vocabulary's end)
    const int k_v = std::min(n_vt * L::TILE, (int)align_up((int64_t)V - (int64_t)vt0 * L::TILE, 32));
    int flags = ROWS_COMPACT;
    if (vc > 0) flags |= READ_ACC;
    flags |= (vc + 1 < p.n_vch) ? WRITE_ACC : WRITE_OUT;
    if constexpr (L::TRANSPOSING && !L::TUNED)
      return ContractArgs<T>{static_cast<const T*>(W) + (int64_t)vt0 * L::TILE * d, d, V - vt0 * L::TILE, d, Gb, p.ld_v,
                             n_nt * L::TILE, k_v, 0, n_mt, n_nt, dHacc, 0, static_cast<T*>(dH), nt0 * L::TILE,
                             npad, flags, hdr, rowmap, grad_loss, mean, p.split_dh, slice_len(k_v, p.split_dh),
                             partial_dh - (int64_t)nt0 * L::TILE * d, nc_pad * d};
    else if constexpr (L::TUNED)
      return ContractArgs<T>{static_cast<const T*>(W) + (int64_t)vt0 * L::TILE * d, d, V - vt0 * L::TILE, d, Gb, g_group_bytes,
                             n_nt * L::TILE, k_v, 0, n_mt, n_nt, dHacc, 0, static_cast<T*>(dH), nt0 * L::TILE, npad,
                             flags, hdr, rowmap, grad_loss, mean, p.split_dh, slice_len(k_v, p.split_dh),
                             partial_dh - (int64_t)nt0 * L::TILE * d, nc_pad * d};
    else
      return ContractArgs<T>{WT, p.ld_v, 0, d, Gb, p.ld_v, n_nt * L::TILE, k_v, 0, n_mt, n_nt, dHacc, 0,
                             static_cast<T*>(dH), nt0 * L::TILE, npad, flags, hdr, rowmap, grad_loss, mean, p.split_dh,
                             slice_len(k_v, p.split_dh), partial_dh - (int64_t)nt0 * L::TILE * d, nc_pad * d};
  };

  // One contraction (dW or dH) of a chunk: the launch, its split-K sum if it has one, and with the tuned loop a
  // separately launched, K-split tail when the last round of workgroups would be mostly empty (tail_split).
  auto contract = [&](const ContractArgs<T>& a, bool is_dw) {
    auto launch = [&](const ContractArgs<T>& x) {
      if constexpr (L::TUNED) {
        const int grid = std::min(x.n_nt * x.n_mt * x.n_split, NUM_CU * L::PER_CU);
        if (is_dw) contract_kernel<T, typename L::Even, OPS_DW_TR><<<grid, L::THREADS, L::LDS, st>>>(x);
        else contract_kernel<T, typename L::Even, OPS_DH_TR><<<grid, L::THREADS, L::LDS, st>>>(x);
      } else if constexpr (L::TRANSPOSING) {
        const int grid = x.n_nt * x.n_mt * x.n_split;
        if (is_dw) contract_kernel<T, L, OPS_DW_F32><<<grid, L::THREADS, L::LDS, st>>>(x);
        else contract_kernel<T, L, OPS_DH_F32><<<grid, L::THREADS, L::LDS, st>>>(x);
      } else {
        contract_kernel<T, L, OPS_KC><<<x.n_nt * x.n_mt * x.n_split, L::THREADS, L::LDS, st>>>(x);
      }
      if (x.n_split > 1)
        splitk_reduce_kernel<T><<<(unsigned)ceil_div((int64_t)x.n_nt * L::TILE * (d / 4), 256), 256, 0, st>>>(x, x.n_nt * L::TILE);
    };
    TailSplit ts{0, 1};
    if constexpr (L::TUNED && L::TILE == TILE) ts = tail_split(a.n_nt, a.n_mt, a.n_split, ceil_div(a.k_elems, L::TILE));
    if (!ts.rows) { launch(a); return; }
    ContractArgs<T> body = a, tail = a;
    body.n_nt = a.n_nt - ts.rows;
    const int64_t first = (int64_t)body.n_nt * L::TILE;     // the tail's first output row, relative to the launch's
    tail.n_nt = ts.rows;
    tail.out_row0 = a.out_row0 + (int)first;
    // G (blocked, ldb = bytes per group of 16 rows) is the B operand of both: its columns are dW's output rows (32
    // per block of 1 KiB), its rows are dH's
    const char* g = reinterpret_cast<const char*>(a.B);
    if (is_dw) { tail.B = reinterpret_cast<const T*>(g + first / 32 * 1024); }
    else { tail.B = reinterpret_cast<const T*>(g + first / 16 * a.ldb); tail.b_rows = a.b_rows - (int)first; }
    tail.n_split = ts.slices;
    tail.k_split = slice_len(a.k_elems, ts.slices);
    tail.partial = a.partial - first * a.d;                // indexed like accbuf: by output row from the launch's first
    tail.partial_stride = (int64_t)ts.rows * L::TILE * a.d;
    launch(body);
    launch(tail);
  };

  // dW and dH of the only chunk in one launch, and the slice sums of whichever is cut in another.
  auto contract_pair = [&](const ContractArgs<T>& w, const ContractArgs<T>& h) {
    const int wg_w = w.n_nt * w.n_mt * w.n_split, wg_h = h.n_nt * h.n_mt * h.n_split;
    if constexpr (L::TUNED)
      contract_pair_kernel<T, typename L::Even, OPS_DW_TR, OPS_DH_TR><<<wg_w + wg_h, L::THREADS, L::LDS, st>>>(w, h, wg_w);
    else if constexpr (L::TRANSPOSING)
      contract_pair_kernel<T, L, OPS_DW_F32, OPS_DH_F32><<<wg_w + wg_h, L::THREADS, L::LDS, st>>>(w, h, wg_w);
    auto blocks = [&](const ContractArgs<T>& x) {
      return x.n_split > 1 ? (int)ceil_div((int64_t)x.n_nt * L::TILE * (d / 4), 256) : 0;
    };
    const int bw = blocks(w), bh = blocks(h);
    if (bw + bh > 0)
      splitk_reduce_pair_kernel<T><<<bw + bh, 256, 0, st>>>(w, w.n_nt * L::TILE, bw, h, h.n_nt * L::TILE);
  };

  for (int vc = 0; vc < p.n_vch; ++vc) {
    int vt0, n_vt;
    chunk_vt(vc, vt0, n_vt);
    if constexpr (!L::TRANSPOSING) {
      // W^T chunk [d][ld_v]: K-contiguous operand of the dH contraction
      ProfScope ps(FLCE_PROF_BWD_PREP, st);
      transpose_pad_kernel<U><<<dim3((unsigned)(n_vt * L::TILE / 64), (unsigned)ceil_div(d, 64)), 256, 0, st>>>(
          static_cast<const U*>(W), d, V, vt0 * L::TILE, d, reinterpret_cast<U*>(WT), p.ld_v, n_vt * L::TILE);
    }
    for (int nc = 0; nc < p.n_nch; ++nc) {
      {
        const RecomputeArgs<T> rc = recompute_args(vc, nc, G);
        ProfScope ps(FLCE_PROF_RECOMPUTE, st);
        // at most as many workgroups as fit the chip: each walks its share of the chunk's tiles
        int grid = rc.n_nt * rc.n_vt;
        if constexpr (L::TUNED) grid = std::min(grid, NUM_CU * L::PER_CU);
        if constexpr (L::TUNED) {     // the tuned loop's backward always has the pre-tiled copies
          if (rows.grad_rows) recompute_kernel<T, L, true, true><<<grid, L::THREADS, L::LDS, st>>>(rc);
          else recompute_kernel<T, L, true><<<grid, L::THREADS, L::LDS, st>>>(rc);
        } else {
          if (rows.grad_rows) recompute_kernel<T, L, false, true><<<grid, L::THREADS, L::LDS, st>>>(rc);
          else recompute_kernel<T, L, false><<<grid, L::THREADS, L::LDS, st>>>(rc);
        }
      }
      if (p.pair) {
        ProfScope ps(FLCE_PROF_CONTRACT_DW, st);       // (both: one launch)
        contract_pair(dw_args(vc, nc, G), dh_args(vc, nc, G));
        continue;
      }
      {
        ProfScope ps(FLCE_PROF_CONTRACT_DW, st);
        contract(dw_args(vc, nc, G), true);
      }
      {
        ProfScope ps(FLCE_PROF_CONTRACT_DH, st);
        contract(dh_args(vc, nc, G), false);
      }
    }
  }
  return hipGetLastError() == hipSuccess ? FLCE_OK : FLCE_ERR_HIP;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

constexpr size_t STATIC_SCRATCH_BYTES = FLCE_STATIC_SCRATCH_BYTES;

std::mutex g_scratch_mu;
void* g_scratch_ptr[MAX_DEVICES] = {};

// Device address of `scratch` on the current device (looked up once per device), or nullptr.
hipError_t static_scratch(void** out) {
  *out = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(::scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace
}  // namespace flce

extern "C" {

const char* flce_version(void) { return "0.2.0"; }

void flce_tuning_reload(void) {
  std::lock_guard<std::mutex> lk(flce::g_tuning_mu);
  flce::g_tuning = flce::read_tuning_from_env();
  flce::g_tuning_loaded = true;
}

const char* flce_status_string(flce_status s) {
  switch (s) {
    case FLCE_OK: return "ok";
    case FLCE_ERR_BAD_ARG: return "bad argument";
    case FLCE_ERR_BAD_SHAPE: return "bad shape";
    case FLCE_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case FLCE_ERR_TARGET_RANGE: return "target outside [0, V)";
    case FLCE_ERR_UNSUPPORTED: return "unsupported";
    case FLCE_ERR_HIP: return "HIP runtime error";
  }
  return "unknown status";
}

int flce_plan_describe(int64_t N, int64_t d, int64_t V, flce_dtype dt, char* buf, size_t buf_bytes) {
  flce::Plan p;
  if (!buf || buf_bytes == 0 || !flce::make_plan(flce::PLAN_BOTH, N, d, V, dt, p)) return -1;
  // K-split tails of the contraction launches of a full chunk (output-row tiles x slices; 0x1 = none)
  const int64_t n_mt = (d + flce::TILE - 1) / flce::TILE;
  flce::TailSplit th{0, 1}, tw{0, 1};
  if (p.fast && !p.pair && p.tile == flce::TILE) {
    th = flce::tail_split(p.nc_tiles, n_mt, p.split_dh, p.vc_tiles);
    tw = flce::tail_split(p.vc_tiles, n_mt, p.split_dw, p.nc_tiles);
  }
  return std::snprintf(buf, buf_bytes,
                       "flce %s loop=%s h_copy=%d/%d windows=%d vocab_chunks=%dx%d row_chunks=%dx%d splitk_dH=%d splitk_dW=%d "
                       "tail_dH=%dx%d tail_dW=%dx%d pair=%d tiles=%d/%d staging_bytes=%lld fwd_ws=%lld bwd_ws=%lld",
                       flce_version(), p.fast ? "tuned" : "generic", p.fwd_copy ? 1 : 0, p.hkr ? 1 : 0, p.n_win, p.n_vch, p.vc_tiles, p.n_nch,
                       p.nc_tiles, p.split_dh, p.split_dw, th.rows, th.slices, tw.rows, tw.slices, p.pair ? 1 : 0, p.fwd_tile, p.tile,
                       (long long)((int64_t)p.nc_tiles * flce::TILE * p.ld_v * p.esize), (long long)p.fwd_bytes,
                       (long long)p.bwd_bytes);
}

size_t flce_workspace_bytes(int64_t N, int64_t d, int64_t V, flce_dtype dt, int for_backward) {
  flce::Plan p;
  if (!flce::make_plan(for_backward ? flce::PLAN_BACKWARD : flce::PLAN_FORWARD, N, d, V, dt, p)) return 0;
  return (size_t)(for_backward ? p.bwd_bytes : p.fwd_bytes);
}

static flce_status forward_impl(const void* H, const void* W, const int64_t* targets, int64_t N, int64_t d,
                                int64_t V, int64_t ignore_index, flce_reduction reduction, flce_dtype dt,
                                float* loss_out, float* lse_out, void* workspace, size_t workspace_bytes,
                                void* hip_stream, flce::Slice slice, float* m_out, float* a_out, float* zt_out,
                                flce::PerRow rows = flce::PerRow{nullptr, nullptr, 0.f}, bool allow_h_copy = true,
                                bool wide = true, flce::StatusOut so = flce::StatusOut{nullptr, nullptr}) {
  const bool partial = m_out || a_out || zt_out;
  if (!H || !W || !targets) return FLCE_ERR_BAD_ARG;
  if (partial ? (!m_out || !a_out || !zt_out) : ((!loss_out && !rows.loss_rows_out) || !lse_out))
    return FLCE_ERR_BAD_ARG;
  if (!(rows.eps >= 0.f && rows.eps < 1.f)) return FLCE_ERR_BAD_ARG;
  if (reduction != FLCE_REDUCE_MEAN && reduction != FLCE_REDUCE_SUM) return FLCE_ERR_BAD_ARG;
  if (dt != FLCE_DTYPE_BF16 && dt != FLCE_DTYPE_F32) return FLCE_ERR_BAD_ARG;
  flce::Plan p;
  if (!flce::make_plan(flce::PLAN_FORWARD, N, d, V, dt, p, allow_h_copy, wide)) return FLCE_ERR_BAD_SHAPE;
  if (slice.v_begin < 0 || slice.v_begin + V > slice.V_total) return FLCE_ERR_BAD_SHAPE;
  if (!flce::aligned16(H) || !flce::aligned16(W)) return FLCE_ERR_BAD_ARG;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) || workspace_bytes < (size_t)p.fwd_bytes)
    return FLCE_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const int mean = reduction == FLCE_REDUCE_MEAN;
  char* ws = static_cast<char*>(workspace);
  if (dt == FLCE_DTYPE_BF16) {
    if (p.ragged && p.fwd_tile == 128)
      return flce::forward_t<flce::bf16_t, uint16_t, flce::SmallLoop<true>>(p, H, W, targets, ignore_index, mean, loss_out, lse_out, ws, st, slice, m_out, a_out, zt_out, rows, so);
    if (p.ragged)
      return flce::forward_t<flce::bf16_t, uint16_t, flce::FastLoop<true>>(p, H, W, targets, ignore_index, mean, loss_out, lse_out, ws, st, slice, m_out, a_out, zt_out, rows, so);
    if (p.fast && p.fwd_tile == 128)
      return flce::forward_t<flce::bf16_t, uint16_t, flce::SmallLoop<false>>(p, H, W, targets, ignore_index, mean, loss_out, lse_out, ws, st, slice, m_out, a_out, zt_out, rows, so);
    if (p.fast)
      return flce::forward_t<flce::bf16_t, uint16_t, flce::FastLoop<false>>(p, H, W, targets, ignore_index, mean, loss_out, lse_out, ws, st, slice, m_out, a_out, zt_out, rows, so);
    return flce::forward_t<flce::bf16_t, uint16_t, flce::GenericLoop>(
        p, H, W, targets, ignore_index, mean, loss_out, lse_out, ws, st, slice, m_out, a_out, zt_out, rows, so);
  }
  if (p.fwd_tile == 64)
    return flce::forward_t<float, uint32_t, flce::F32Loop<64>>(p, H, W, targets, ignore_index, mean, loss_out, lse_out, ws, st, slice, m_out, a_out, zt_out, rows, so);
  return flce::forward_t<float, uint32_t, flce::F32Loop<128>>(p, H, W, targets, ignore_index, mean, loss_out, lse_out, ws, st, slice, m_out, a_out, zt_out, rows, so);
}

static flce_status backward_impl(const void* H, const void* W, const int64_t* targets, const float* lse, int64_t N,
                                 int64_t d, int64_t V, int64_t ignore_index, flce_reduction reduction, flce_dtype dt,
                                 flce::GradLoss grad_loss, void* dH_out, void* dW_out, void* workspace,
                                 size_t workspace_bytes, void* hip_stream, flce::Slice slice,
                                 flce::PerRow rows = flce::PerRow{nullptr, nullptr, 0.f}) {
  if (!H || !W || !targets || !lse || !dH_out || !dW_out) return FLCE_ERR_BAD_ARG;
  if (!(rows.eps >= 0.f && rows.eps < 1.f)) return FLCE_ERR_BAD_ARG;
  if (reduction != FLCE_REDUCE_MEAN && reduction != FLCE_REDUCE_SUM) return FLCE_ERR_BAD_ARG;
  if (dt != FLCE_DTYPE_BF16 && dt != FLCE_DTYPE_F32) return FLCE_ERR_BAD_ARG;
  flce::Plan p;
  if (!flce::make_plan(flce::PLAN_BACKWARD, N, d, V, dt, p)) return FLCE_ERR_BAD_SHAPE;
  if (slice.v_begin < 0 || slice.v_begin + V > slice.V_total) return FLCE_ERR_BAD_SHAPE;
  if (!flce::aligned16(H) || !flce::aligned16(W) || !flce::aligned16(dH_out) || !flce::aligned16(dW_out))
    return FLCE_ERR_BAD_ARG;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) || workspace_bytes < (size_t)p.bwd_bytes)
    return FLCE_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const int mean = reduction == FLCE_REDUCE_MEAN;
  char* ws = static_cast<char*>(workspace);
  if (dt == FLCE_DTYPE_BF16) {
    if (p.ragged && p.tile == 128)
      return flce::backward_t<flce::bf16_t, uint16_t, flce::SmallLoop<true>>(p, H, W, targets, lse, ignore_index, mean, grad_loss, dH_out, dW_out, ws, st, slice, rows);
    if (p.ragged)
      return flce::backward_t<flce::bf16_t, uint16_t, flce::FastLoop<true>>(p, H, W, targets, lse, ignore_index, mean, grad_loss, dH_out, dW_out, ws, st, slice, rows);
    if (p.fast && p.tile == 128)
      return flce::backward_t<flce::bf16_t, uint16_t, flce::SmallLoop<false>>(p, H, W, targets, lse, ignore_index, mean, grad_loss, dH_out, dW_out, ws, st, slice, rows);
    if (p.fast)
      return flce::backward_t<flce::bf16_t, uint16_t, flce::FastLoop<false>>(p, H, W, targets, lse, ignore_index, mean, grad_loss, dH_out, dW_out, ws, st, slice, rows);
    return flce::backward_t<flce::bf16_t, uint16_t, flce::GenericLoop>(
        p, H, W, targets, lse, ignore_index, mean, grad_loss, dH_out, dW_out, ws, st, slice, rows);
  }
  if (p.tile == 64)
    return flce::backward_t<float, uint32_t, flce::F32Loop<64>>(p, H, W, targets, lse, ignore_index, mean, grad_loss, dH_out, dW_out, ws, st, slice, rows);
  return flce::backward_t<float, uint32_t, flce::F32Loop<128>>(p, H, W, targets, lse, ignore_index, mean, grad_loss, dH_out, dW_out, ws, st, slice, rows);
}

flce_status flce_forward(const void* H, const void* W, const int64_t* targets, int64_t N, int64_t d, int64_t V,
                         int64_t ignore_index, flce_reduction reduction, flce_dtype dt, float* loss_out,
                         float* lse_out, void* workspace, size_t workspace_bytes, void* hip_stream) {
  return forward_impl(H, W, targets, N, d, V, ignore_index, reduction, dt, loss_out, lse_out, workspace,
                      workspace_bytes, hip_stream, flce::Slice{V, 0}, nullptr, nullptr, nullptr);
}

flce_status flce_backward(const void* H, const void* W, const int64_t* targets, const float* lse, int64_t N,
                          int64_t d, int64_t V, int64_t ignore_index, flce_reduction reduction, flce_dtype dt,
                          float grad_loss, void* dH_out, void* dW_out, void* workspace, size_t workspace_bytes,
                          void* hip_stream) {
  return backward_impl(H, W, targets, lse, N, d, V, ignore_index, reduction, dt, flce::GradLoss{grad_loss, nullptr}, dH_out,
                       dW_out, workspace, workspace_bytes, hip_stream, flce::Slice{V, 0});
}

flce_status flce_backward_device_grad(const void* H, const void* W, const int64_t* targets, const float* lse, int64_t N,
                                      int64_t d, int64_t V, int64_t ignore_index, flce_reduction reduction, flce_dtype dt,
                                      const float* grad_loss, void* dH_out, void* dW_out, void* workspace,
                                      size_t workspace_bytes, void* hip_stream) {
  if (!grad_loss) return FLCE_ERR_BAD_ARG;
  return backward_impl(H, W, targets, lse, N, d, V, ignore_index, reduction, dt, flce::GradLoss{0.f, grad_loss}, dH_out,
                       dW_out, workspace, workspace_bytes, hip_stream, flce::Slice{V, 0});
}

flce_status flce_forward_static(const void* H, const void* W, const int64_t* targets, int64_t N, int64_t d, int64_t V,
                                int64_t ignore_index, flce_reduction reduction, flce_dtype dt, float* loss_out,
                                float* lse_out, int32_t* status_out, int64_t* n_valid_out, void* hip_stream) {
  // The plan without the pre-tiled copy of H (its size grows with N*d): what is left of the forward
  // workspace is the per-window partials and per-block sums, O(N) words.
  if (!H || !W || !targets || !loss_out || !lse_out) return FLCE_ERR_BAD_ARG;
  if (reduction != FLCE_REDUCE_MEAN && reduction != FLCE_REDUCE_SUM) return FLCE_ERR_BAD_ARG;
  if (dt != FLCE_DTYPE_BF16 && dt != FLCE_DTYPE_F32) return FLCE_ERR_BAD_ARG;
  // More windows than cover the CUs are used where their partials fit too; what fits is decided without them.
  flce::Plan p;
  if (!flce::make_plan(flce::PLAN_FORWARD, N, d, V, dt, p, /*allow_h_copy=*/false, /*wide=*/false)) return FLCE_ERR_BAD_SHAPE;
  if ((size_t)p.fwd_bytes > flce::STATIC_SCRATCH_BYTES) return FLCE_ERR_WORKSPACE;
  flce::Plan w;
  const bool wide = flce::make_plan(flce::PLAN_FORWARD, N, d, V, dt, w, /*allow_h_copy=*/false, /*wide=*/true) &&
                    (size_t)w.fwd_bytes <= flce::STATIC_SCRATCH_BYTES;
  void* ws = nullptr;
  if (flce::static_scratch(&ws) != hipSuccess) return FLCE_ERR_HIP;
  return forward_impl(H, W, targets, N, d, V, ignore_index, reduction, dt, loss_out, lse_out, ws,
                      flce::STATIC_SCRATCH_BYTES, hip_stream, flce::Slice{V, 0}, nullptr, nullptr, nullptr,
                      flce::PerRow{nullptr, nullptr, 0.f}, /*allow_h_copy=*/false, wide,
                      flce::StatusOut{status_out, n_valid_out});
}

flce_status flce_forward_rows(const void* H, const void* W, const int64_t* targets, int64_t N, int64_t d, int64_t V,
                              int64_t ignore_index, float label_smoothing, flce_dtype dt, float* loss_rows_out,
                              float* lse_out, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!loss_rows_out) return FLCE_ERR_BAD_ARG;
  return forward_impl(H, W, targets, N, d, V, ignore_index, FLCE_REDUCE_SUM, dt, nullptr, lse_out, workspace,
                      workspace_bytes, hip_stream, flce::Slice{V, 0}, nullptr, nullptr, nullptr,
                      flce::PerRow{loss_rows_out, nullptr, label_smoothing});
}

flce_status flce_backward_rows(const void* H, const void* W, const int64_t* targets, const float* lse,
                               const float* grad_rows, int64_t N, int64_t d, int64_t V, int64_t ignore_index,
                               float label_smoothing, flce_dtype dt, void* dH_out, void* dW_out, void* workspace,
                               size_t workspace_bytes, void* hip_stream) {
  if (!grad_rows) return FLCE_ERR_BAD_ARG;
  return backward_impl(H, W, targets, lse, N, d, V, ignore_index, FLCE_REDUCE_SUM, dt, flce::GradLoss{1.0f, nullptr}, dH_out, dW_out,
                       workspace, workspace_bytes, hip_stream, flce::Slice{V, 0},
                       flce::PerRow{nullptr, grad_rows, label_smoothing});
}

flce_status flce_forward_partial(const void* H, const void* W_slice, const int64_t* targets, int64_t N, int64_t d,
                                 int64_t V_slice, int64_t v_begin, int64_t V_total, int64_t ignore_index,
                                 flce_dtype dt, float* m_out, float* a_out, float* zt_out, void* workspace,
                                 size_t workspace_bytes, void* hip_stream) {
  if (!m_out || !a_out || !zt_out) return FLCE_ERR_BAD_ARG;
  return forward_impl(H, W_slice, targets, N, d, V_slice, ignore_index, FLCE_REDUCE_SUM, dt, nullptr, nullptr,
                      workspace, workspace_bytes, hip_stream, flce::Slice{V_total, v_begin}, m_out, a_out, zt_out);
}

size_t flce_merge_workspace_bytes(int64_t N) {
  if (N <= 0 || N > 0x7FFFFF00ll) return 0;
  const int64_t n_rb = flce::ceil_div(N, flce::TILE);
  return (size_t)(flce::ALIGN + 3 * flce::align_up(n_rb * 4, flce::ALIGN));
}

flce_status flce_merge_partials(const float* m_parts, const float* a_parts, const float* zt_parts, int n_parts,
                                const int64_t* targets, int64_t N, int64_t V_total, int64_t ignore_index,
                                flce_reduction reduction, float* loss_out, float* lse_out, void* workspace,
                                size_t workspace_bytes, void* hip_stream) {
  if (!m_parts || !a_parts || !zt_parts || !targets || !loss_out || !lse_out || n_parts < 1) return FLCE_ERR_BAD_ARG;
  if (reduction != FLCE_REDUCE_MEAN && reduction != FLCE_REDUCE_SUM) return FLCE_ERR_BAD_ARG;
  const size_t need = flce_merge_workspace_bytes(N);
  if (need == 0 || V_total <= 0) return FLCE_ERR_BAD_SHAPE;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) || workspace_bytes < need)
    return FLCE_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  char* ws = static_cast<char*>(workspace);
  const int n_rb = (int)flce::ceil_div(N, flce::TILE);
  const int64_t blk = flce::align_up((int64_t)n_rb * 4, flce::ALIGN);
  flce::Header* hdr = reinterpret_cast<flce::Header*>(ws);
  float* blk_loss = reinterpret_cast<float*>(ws + flce::ALIGN);
  int* blk_cnt = reinterpret_cast<int*>(ws + flce::ALIGN + blk);
  int* blk_oor = reinterpret_cast<int*>(ws + flce::ALIGN + 2 * blk);
  flce::ProfScope ps(FLCE_PROF_FWD_EPILOGUE, st);
  // no tile kernel has run before this merge to zero the arrival count: the sum of several blocks is a launch of its own
  const flce::LossOut o{blk_loss, blk_cnt, blk_oor, hdr, loss_out, reduction == FLCE_REDUCE_MEAN, nullptr, nullptr};
  const int n_blk = flce::launch_merge(m_parts, a_parts, zt_parts, n_parts, N, targets, (int)N, V_total, ignore_index,
                                       lse_out, o, /*fused=*/false, nullptr, nullptr, 0.f, st);
  flce::finalize_loss_kernel<<<1, 256, 0, st>>>(o, n_blk);
  return hipGetLastError() == hipSuccess ? FLCE_OK : FLCE_ERR_HIP;
}

flce_status flce_backward_partial(const void* H, const void* W_slice, const int64_t* targets, const float* lse,
                                  int64_t N, int64_t d, int64_t V_slice, int64_t v_begin, int64_t V_total,
                                  int64_t ignore_index, flce_reduction reduction, flce_dtype dt, float grad_loss,
                                  void* dH_partial_out, void* dW_slice_out, void* workspace,
                                  size_t workspace_bytes, void* hip_stream) {
  return backward_impl(H, W_slice, targets, lse, N, d, V_slice, ignore_index, reduction, dt,
                       flce::GradLoss{grad_loss, nullptr}, dH_partial_out, dW_slice_out, workspace, workspace_bytes, hip_stream,
                       flce::Slice{V_total, v_begin});
}

flce_status flce_forward_with_grads(const void* H, const void* W, const int64_t* targets, int64_t N, int64_t d,
                                    int64_t V, int64_t ignore_index, flce_reduction reduction, flce_dtype dt,
                                    float* loss_out, float* lse_out, void* dH_partial, void* dW_partial,
                                    void* workspace, size_t workspace_bytes, void* hip_stream) {
  // Alg. 3 = Alg. 1 followed by the gradient sweep with the upstream gradient left out: the forward,
  // then the backward with Gamma = 1 (sum semantics, grad_loss 1), on the same stream and workspace.
  flce::Plan p;
  if (!flce::make_plan(flce::PLAN_BOTH, N, d, V, dt, p)) return FLCE_ERR_BAD_SHAPE;
  if (workspace_bytes < (size_t)std::max(p.fwd_bytes, p.bwd_bytes)) return FLCE_ERR_WORKSPACE;
  if (!dH_partial || !dW_partial) return FLCE_ERR_BAD_ARG;
  const flce_status st = flce_forward(H, W, targets, N, d, V, ignore_index, reduction, dt, loss_out, lse_out,
                                      workspace, workspace_bytes, hip_stream);
  if (st != FLCE_OK) return st;
  return flce_backward(H, W, targets, lse_out, N, d, V, ignore_index, FLCE_REDUCE_SUM, dt, 1.0f, dH_partial,
                       dW_partial, workspace, workspace_bytes, hip_stream);
}

flce_status flce_scale(const void* dH_partial, const void* dW_partial, int64_t N, int64_t d, int64_t V,
                       flce_reduction reduction, flce_dtype dt, float grad_loss, const void* workspace,
                       void* dH_out, void* dW_out, void* hip_stream) {
  if (!dH_partial || !dW_partial || !dH_out || !dW_out || !workspace) return FLCE_ERR_BAD_ARG;
  if (reduction != FLCE_REDUCE_MEAN && reduction != FLCE_REDUCE_SUM) return FLCE_ERR_BAD_ARG;
  flce::Plan p;
  if (!flce::make_plan(0, N, d, V, dt, p)) return FLCE_ERR_BAD_SHAPE;
  if (!flce::aligned16(dH_partial) || !flce::aligned16(dW_partial) || !flce::aligned16(dH_out) ||
      !flce::aligned16(dW_out))
    return FLCE_ERR_BAD_ARG;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const flce::Header* hdr = static_cast<const flce::Header*>(workspace);
  const int mean = reduction == FLCE_REDUCE_MEAN;
  auto run = [&](auto tag) {
    using T = decltype(tag);
    flce::ProfScope ps(FLCE_PROF_SCALE, st);
    const int64_t nh = N * d / 4, nw = V * d / 4;
    const unsigned grid = (unsigned)std::min<int64_t>(flce::ceil_div(nh + nw, 256), 16384);
    flce::scale_kernel<T><<<grid, 256, 0, st>>>(static_cast<const T*>(dH_partial), static_cast<T*>(dH_out), nh,
                                                static_cast<const T*>(dW_partial), static_cast<T*>(dW_out), nw, hdr,
                                                grad_loss, mean);
  };
  if (dt == FLCE_DTYPE_BF16) run(flce::bf16_t{});
  else run(float{});
  return hipGetLastError() == hipSuccess ? FLCE_OK : FLCE_ERR_HIP;
}

flce_status flce_last_device_status(const void* workspace, void* hip_stream, int64_t* n_valid_out) {
  if (!workspace) return FLCE_ERR_BAD_ARG;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  flce::Header h;
  if (hipStreamSynchronize(st) != hipSuccess) return FLCE_ERR_HIP;
  if (hipMemcpy(&h, workspace, sizeof(h), hipMemcpyDeviceToHost) != hipSuccess) return FLCE_ERR_HIP;
  if (n_valid_out) *n_valid_out = h.n_valid;
  return h.status == 0 ? FLCE_OK : FLCE_ERR_TARGET_RANGE;
}

flce_status flce_probe(int mode, const void* A, const void* B, const void* BT, int64_t a_rows, int64_t b_rows,
                       int64_t k_elems, int workgroups, int tiles_per_workgroup, float* sink, void* hip_stream) {
  if (!A || !B || !BT || !sink) return FLCE_ERR_BAD_ARG;
  if (mode < flce::PROBE_MFMA || mode > flce::PROBE_PAIR_PK_PK) return FLCE_ERR_BAD_ARG;
  if (a_rows <= 0 || b_rows <= 0 || (a_rows % flce::TILE) || (b_rows % flce::TILE) || k_elems < 32 || (k_elems % 32) ||
      workgroups <= 0 || tiles_per_workgroup <= 0)
    return FLCE_ERR_BAD_SHAPE;
  if (!flce::window_ok(257, k_elems * 2) || !flce::window_ok(k_elems, b_rows * 2)) return FLCE_ERR_BAD_SHAPE;
  if (!flce::aligned16(A) || !flce::aligned16(B) || !flce::aligned16(BT)) return FLCE_ERR_BAD_ARG;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const flce::ProbeArgs pa{static_cast<const flce::bf16_t*>(A), static_cast<const flce::bf16_t*>(B),
                           static_cast<const flce::bf16_t*>(BT), (int)a_rows, (int)b_rows, (int)k_elems,
                           tiles_per_workgroup, sink};
  auto launch = [&](auto kernel, int lds_bytes = flce::fast::LDS_BYTES) -> flce_status {
    if (flce::allow_big_lds(kernel, lds_bytes) != hipSuccess) return FLCE_ERR_HIP;
    kernel<<<workgroups, flce::fast::THREADS, lds_bytes, st>>>(pa);
    return hipGetLastError() == hipSuccess ? FLCE_OK : FLCE_ERR_HIP;
  };
  switch (mode) {
    case flce::PROBE_MFMA: return launch(flce::probe_kernel<flce::PROBE_MFMA>);
    case flce::PROBE_LOOP_KR: return launch(flce::probe_kernel<flce::PROBE_LOOP_KR>);
    case flce::PROBE_LOOP_KC: return launch(flce::probe_kernel<flce::PROBE_LOOP_KC>);
    case flce::PROBE_DATA_KR: return launch(flce::probe_kernel<flce::PROBE_DATA_KR>);
    case flce::PROBE_DATA_KC: return launch(flce::probe_kernel<flce::PROBE_DATA_KC>);
    case flce::PROBE_FREE_RUN: return launch(flce::probe_kernel<flce::PROBE_FREE_RUN>);
    case flce::PROBE_LOOP_KR_SOFTMAX: return launch(flce::probe_kernel<flce::PROBE_LOOP_KR_SOFTMAX>);
    case flce::PROBE_HALF_KR: return launch(flce::probe_half_kernel<false>, flce::PROBE_HALF_LDS);
    case flce::PROBE_HALF_KR_SOFTMAX: return launch(flce::probe_half_kernel<true>, flce::PROBE_HALF_LDS);
    case flce::PROBE_LOOP_KR_COLD: return launch(flce::probe_kernel<flce::PROBE_LOOP_KR_COLD>);
    case flce::PROBE_MFMA_16X16: return launch(flce::probe_mfma16_kernel<0>);
    case flce::PROBE_LOOP_PK: return launch(flce::probe_kernel<flce::PROBE_LOOP_PK>);
    case flce::PROBE_PAIR_KR_KR: return launch(flce::probe_pair_kernel<flce::fast::KR, flce::fast::KR>);
    case flce::PROBE_PAIR_PK_KR: return launch(flce::probe_pair_kernel<flce::fast::PK, flce::fast::KR>);
    case flce::PROBE_PAIR_KR_KC: return launch(flce::probe_pair_kernel<flce::fast::KR, flce::fast::KC>);
    case flce::PROBE_PAIR_KR_PK: return launch(flce::probe_pair_kernel<flce::fast::KR, flce::fast::PK>);
    case flce::PROBE_PAIR_PK_PK: return launch(flce::probe_pair_kernel<flce::fast::PK, flce::fast::PK>);
  }
  return FLCE_ERR_BAD_ARG;
}

flce_status flce_profile_enable(int on) {
  std::lock_guard<std::mutex> lk(flce::g_prof.mu);
  for (auto& r : flce::g_prof.recs) { flce::g_prof.pool.push_back(r.a); flce::g_prof.pool.push_back(r.b); }
  flce::g_prof.recs.clear();
  flce::g_prof.on = on != 0;
  return FLCE_OK;
}

flce_status flce_profile_collect(double* ms_by_class, int64_t* launches_by_class) {
  std::lock_guard<std::mutex> lk(flce::g_prof.mu);
  flce_status rc = FLCE_OK;
  for (auto& r : flce::g_prof.recs) {
    float ms = 0.f;
    if (hipEventSynchronize(r.b) != hipSuccess || hipEventElapsedTime(&ms, r.a, r.b) != hipSuccess) rc = FLCE_ERR_HIP;
    if (r.cls >= 0 && r.cls < FLCE_PROF_CLASSES) {
      if (ms_by_class) ms_by_class[r.cls] += (double)ms;
      if (launches_by_class) launches_by_class[r.cls] += 1;
    }
    flce::g_prof.pool.push_back(r.a);
    flce::g_prof.pool.push_back(r.b);
  }
  flce::g_prof.recs.clear();
  return rc;
}

}  // extern "C"
