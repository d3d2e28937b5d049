// Internal plan structure shared by the host plan code and the launchers.
//
// Every problem is held in "row form": a 2-D layer is an Hi x Wi plane on an
// Lh x Lw grid; a 1-D layer is a single row (Hi = 1, Lh = 1) of length Wi on a
// grid of length Lw.  With Lh = 1 the kept-row set is {u = 0} and the 2-D
// kernels reduce to the 1-D transform, so one set of kernels serves both.
#pragma once

#include <cmath>
#include <cstddef>
#include <cstdint>
#include <vector>

#include "../../include/blconv.h"

// Dynamic LDS of one weight-gradient slice (its inverse-DFT weights): with
// the kernel's static LDS (at most 16 KB) a block stays within 64 KB.
constexpr long kWgradSliceLds = 48 * 1024;

// Tiling of the per-bin contraction [M x K] . [K x N] (complex) over `bins`
// bins: tile height bm and width bn (32 or 64), the number of k-splits, whose
// partial tiles a separate pass sums in a fixed order, and the groups of waves
// that share a block's k range.
struct BlContractTiling {
  int bm, bn, splits, ks;
};
// Wave groups of a tile in a launch of `tiles` tiles with complex64 operands
// and more than one stage of 16 k: with no more tiles than compute units a
// SIMD would run one wave, whose stages (about 0.9 us each) are a serial chain
// (128 -> 32 channels, 45 to 84 bins: 8.9 us with one group, 7.6 with four; 256
// channels, 224 tiles: 16.5 and 15.5).  bfloat16 stages are short and memory
// bound: 5.4 us with one group, 5.9 with four.
inline int bl_contract_groups(int bm, int bn, long tiles, long stages, bool bf16) {
  return bf16 || tiles > 256 || stages < 2 ? 1 : bm == 64 && bn == 64 ? 2 : 4;
}
inline BlContractTiling bl_contract_tiling(long M, long N, long K, long bins, bool bf16) {
  // 64 x 64 tiles wherever both sides pass 32 (smaller ones load more per
  // product: 1.2 to 1.8 times the time on the workload layers), 32 where a
  // side would be mostly padding
  BlContractTiling t{M <= 32 ? 32 : 64, N <= 32 ? 32 : 64, 1, 1};
  const long tiles = bins * ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
  const long stages = (K + 15) / 16;
  t.ks = bl_contract_groups(t.bm, t.bn, tiles, stages, bf16);
  // a handful of tiles with long sums: the pass that adds the partial tiles
  // costs about 4 us, a stage nearly 1 us, one of 32 k with bfloat16 half that
  const long rounds = bf16 ? (K + 31) / 32 / 2 : stages / t.ks;
  while (t.splits < 16 && tiles * t.splits <= 128 && rounds / t.splits >= 16) t.splits *= 2;
  return t;
}

// Whether the contraction [M x K] . [K x N] over B bins (dgrad, wgrad: the
// input and the weight gradient's) runs on the vector ALUs (thin.hip).
inline bool bl_contract_thin(long M, long N, long K, long B, bool dgrad, bool wgrad) {
  // Against the tiled kernels, whose matrix tiles are mostly padding here but
  // whose loads are wide and whose sums run beside each other (us, thin / tiled,
  // at 14, 101 and 1001 bins unless said):
  //  - outer products (K = 1): 64 x 128 4.3 / 4.5 and 14.7 / 19.0.  K = 2: 32 x
  //    128 12.4 / 13.4 at 1001 bins; 2 x 256 x 256 of a gradient 160 / 135;
  if (K == 1 || (K == 2 && !wgrad)) return true;
  //  - one or two rows: 64 -> 64 3.9 / 5.7, 4.2 / 5.9, 6.7 / 11.0; two rows 81 ->
  //    100 4.9 / 8.5 at 51 bins, 17.1 / 25.9 at 1001, 256 -> 256 102 / 94 at 546.
  //    The input gradient's lanes walk rows of W one element apart in k: 4.1 /
  //    5.3, 4.4 / 5.7, then 13.6 / 9.9, and 256 -> 256 11.0 / 9.1, 215 / 116;
  if (M <= 2) return B * N * K <= (dgrad ? 500000 : 20000000);
  //  - one or two columns, a wave per row: 64 rows of 128 4.1 / 6.9, 4.1 / 7.3,
  //    15.7 / 16.1; 128 rows of 64 4.2 / 6.1 at 51 bins, 19.3 / 13.1 at 546.  The
  //    weight gradient's lanes read A one row apart: 128 rows of 64 4.1 / 6.4,
  //    6.7 / 6.4, 49.7 / 19.9;
  //  - three to eight columns while rows are few, the more the longer: 64 rows of
  //    64 4.2 / 5.7, 5.6 / 5.9, 31.9 / 9.7; 16 rows of 352 5.5 / 10.7, 7.0 / 11.0,
  //    30 / 34.
  // Three rows or products and more: tiled throughout (M = 8, 512 x 512 136 / 16
  // at 14 bins; M = 3, 64 x 64 11.9 / 6.1 at 51; K = 3, 64 x 64 4.4 / 4.5, 5.5 /
  // 5.1, 15.1 / 11.0).
  // (few columns with few rows or products would leave the lanes of k_thin_cols
  // idle: 6 x 2, 114 products, 36 bins 28.8)
  if (N > 8 || M <= 8 || K <= 8) return false;
  if (N <= 2) return B * M <= (wgrad ? 8192 : 32768);
  return B * M <= (64 * K > 8192 ? 64 * K : 8192);
}

struct bl_conv_plan_s {
  bl_conv_desc_t desc;
  int ndim;
  bool bf16;           // stored spectra X, W, DY as bfloat16 pairs (BL_DESC_BF16_SPECTRA)
  bool fused_fwd;      // forward through the fused small-map kernel where it applies
  int N, Cin, Cout;
  // row form
  int Hi, Wi;          // input plane
  int Kh, Kw;          // filter support
  int pt, pb, pl, pr;  // zero padding
  int Hp, Wp;          // padded input
  int Ho, Wo;          // output plane
  int Lh, Lw;          // FFT grid
  int Wh;              // half-plane width Lw/2 + 1
  int t, r_h, r_w;     // peeled layers and radii of the kept band
  int R, V;            // kept rows and kept columns
  long kept, total;
  double c_eff;
  std::vector<uint8_t> mask;  // [Lh][Wh]
  // workspace layout (bytes)
  int wg_chunks;        // bin slices of the weight-gradient inverse DFT
  int wg_bins;          // bins per slice (a multiple of 8)
  int wg_groups;        // groups of 256 threads per block summing parts of the bins (2 or 4), or 0
  BlContractTiling ct[3];  // contraction tiling: forward, grad-input, grad-weight
  // paired backward contraction (one launch for grad-input and grad-weight):
  // k-splits of grad-input, whose partial sums (in the contraction-partials
  // area) the inverse transform adds; 0: two launches
  int bp_s1;
  int bp_bm, bp_bn;  // the paired launch's tile shape
  // forward contraction split along k into partial spectra that the 2-D
  // output inverse adds (1: not split), for launches of few tiles
  int fwd_split, fwd_ks;  // (fwd_ks: wave groups per tile, as BlContractTiling::ks)
  size_t off_X, off_W, off_DY, off_T, off_DW, off_Part, off_CPart, ws_bytes;
  // device tables (operands of the matrix-product transforms, 1-D chirps and
  // filter spectra, weight-gradient inverse-DFT weights), made in a plan's first
  // call that needs them on each device; freed with the plan
  mutable void* tables;
};

// Frees a plan's device tables (null is a no-op).
void bl_plan_tables_free(void* tables);

// FFT row index of the r-th kept row: the top-left corner (u = 0..r_h) first,
// then the bottom-left corner (u = Lh - r_h .. Lh - 1).
inline int bl_kept_row(int r, int r_h, int Lh, int R) { return r <= r_h ? r : r + (Lh - R); }

// Number of kept rows for radius r on an axis of length L.
inline int bl_rows_for_radius(int r, int L) {
  return (L % 2 == 0 && r == L / 2) ? L : 2 * r + 1;
}
