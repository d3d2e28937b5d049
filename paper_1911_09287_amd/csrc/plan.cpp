// Host plan of the band-limited convolution: geometry, kept band, workspace.
// Pure host code; makes no HIP call, so plans can be built and inspected on a
// machine without a GPU.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>

#include "plan.hpp"

namespace {

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Kept count after peeling t L-shaped layers (Sec. 3.2.2, Fig. 2): rows with
// |s(u)| <= Lh/2 - t times columns v <= Lw/2 - t of the half plane.
long kept_after(int t, int Lh, int Lw, int ndim) {
  if (ndim == 1) return (long)(Lw / 2 + 1 - t);
  int r_h = Lh / 2 - t, r_w = Lw / 2 - t;
  return (long)bl_rows_for_radius(r_h, Lh) * (long)(r_w + 1);
}

}  // namespace

extern "C" bl_status_t bl_conv_plan_create(bl_conv_plan_t* out, const bl_conv_desc_t* d) {
  if (!out || !d) return BL_ERR_INVALID_ARG;
  *out = nullptr;
  if (d->ndim != 1 && d->ndim != 2) return BL_ERR_INVALID_ARG;
  if (d->N <= 0 || d->C_in <= 0 || d->C_out <= 0 || d->H <= 0 || d->K <= 0) return BL_ERR_INVALID_ARG;
  if (d->pad_lo[0] < 0 || d->pad_hi[0] < 0 || d->pad_lo[1] < 0 || d->pad_hi[1] < 0) return BL_ERR_INVALID_ARG;
  if (!(d->c >= 0.0 && d->c < 1.0)) return BL_ERR_INVALID_ARG;  // also rejects NaN
  if (d->fft_h < 0 || d->fft_w < 0) return BL_ERR_INVALID_ARG;
  if (d->flags & ~(BL_DESC_BF16_SPECTRA | BL_DESC_FUSED_FORWARD)) return BL_ERR_INVALID_ARG;
  if (d->ndim == 1 && (d->W != 1 || d->pad_lo[1] != 0 || d->pad_hi[1] != 0 || d->fft_w > 1))
    return BL_ERR_INVALID_ARG;
  if (d->ndim == 2 && d->W <= 0) return BL_ERR_INVALID_ARG;
  if (d->K > 8) return BL_ERR_UNSUPPORTED;

  bl_conv_plan_s* p = new (std::nothrow) bl_conv_plan_s();
  if (!p) return BL_ERR_OOM;
  p->desc = *d;
  p->ndim = d->ndim;
  p->bf16 = (d->flags & BL_DESC_BF16_SPECTRA) != 0;
  p->fused_fwd = (d->flags & BL_DESC_FUSED_FORWARD) != 0;
  p->N = d->N; p->Cin = d->C_in; p->Cout = d->C_out;
  if (d->ndim == 2) {
    p->Hi = d->H; p->Wi = d->W; p->Kh = d->K; p->Kw = d->K;
    p->pt = d->pad_lo[0]; p->pb = d->pad_hi[0]; p->pl = d->pad_lo[1]; p->pr = d->pad_hi[1];
  } else {
    p->Hi = 1; p->Wi = d->H; p->Kh = 1; p->Kw = d->K;
    p->pt = 0; p->pb = 0; p->pl = d->pad_lo[0]; p->pr = d->pad_hi[0];
  }
  p->Hp = p->Hi + p->pt + p->pb;
  p->Wp = p->Wi + p->pl + p->pr;
  p->Ho = p->Hp - p->Kh + 1;
  p->Wo = p->Wp - p->Kw + 1;
  if (p->Ho < 1 || p->Wo < 1) { delete p; return BL_ERR_INVALID_ARG; }
  if (d->ndim == 2) {
    p->Lh = d->fft_h ? d->fft_h : p->Hp;
    p->Lw = d->fft_w ? d->fft_w : p->Wp;
  } else {
    p->Lh = 1;
    p->Lw = d->fft_h ? d->fft_h : p->Wp;
  }
  if (p->Lh < p->Hp || p->Lw < p->Wp) { delete p; return BL_ERR_INVALID_ARG; }
  if (p->Lw > 4096 || p->Lh > 4096) { delete p; return BL_ERR_UNSUPPORTED; }
  p->Wh = p->Lw / 2 + 1;
  p->total = (long)p->Lh * (long)p->Wh;

  // Rate -> layers: the fewest t with kept(t) <= (1 - c) * total, in double.
  int t_max = (d->ndim == 1) ? p->Wh - 1 : std::min(p->Lh / 2, p->Lw / 2);
  const double budget = (1.0 - d->c) * (double)p->total;
  int t = t_max;
  for (int tt = 0; tt <= t_max; ++tt) {
    if ((double)kept_after(tt, p->Lh, p->Lw, d->ndim) <= budget) { t = tt; break; }
  }
  p->t = t;
  if (d->ndim == 1) {
    p->r_h = 0;
    p->r_w = p->Wh - 1 - t;
    p->R = 1;
  } else {
    p->r_h = p->Lh / 2 - t;
    p->r_w = p->Lw / 2 - t;
    p->R = bl_rows_for_radius(p->r_h, p->Lh);
  }
  p->V = p->r_w + 1;
  p->kept = (long)p->R * p->V;
  // every compute call must find a kernel for the shape, so that a call that
  // fails has enqueued nothing: the contraction takes at most 65535 kept bins,
  // and the direct transforms (the fallback of every faster one) hold a plane
  // in at most 160 KB of LDS
  {
    const size_t tw = (size_t)(p->Lh + p->Lw) * 8;
    const size_t fwd = tw + ((size_t)p->Hi * p->V + 1) * 8 + (size_t)p->Hi * p->Wi * 4;
    const size_t inv = tw + ((size_t)p->R * p->V + 1 + (size_t)p->Hi * p->V + 1) * 8;
    if (p->kept > 65535 || fwd > 160 * 1024 || inv > 160 * 1024) { delete p; return BL_ERR_UNSUPPORTED; }
  }
  p->c_eff = 1.0 - (double)p->kept / (double)p->total;

  p->mask.assign((size_t)p->total, 0);
  for (int r = 0; r < p->R; ++r) {
    int u = bl_kept_row(r, p->r_h, p->Lh, p->R);
    for (int v = 0; v < p->V; ++v) p->mask[(size_t)u * p->Wh + v] = 1;
  }

  const size_t cb = 8;                  // complex64
  const size_t sb = p->bf16 ? 4 : cb;  // a stored spectrum's element: complex64 or a bfloat16 pair
  const size_t B = (size_t)p->kept;
  size_t o = 0;
  p->off_X = o;  o = align_up(o + B * p->N * p->Cin * sb, 256);
  p->off_W = o;  o = align_up(o + B * p->Cin * p->Cout * sb, 256);
  p->off_DY = o; o = align_up(o + B * p->N * p->Cout * sb, 256);
  p->off_T = o;  o = align_up(o + B * p->N * (size_t)std::max(p->Cin, p->Cout) * cb, 256);
  p->off_DW = o; o = align_up(o + B * p->Cin * p->Cout * cb, 256);
  // contraction tiling of the three passes, and the paired backward launch:
  // one tile shape, the larger of the two passes' (64 x 64 measured best on
  // every workload layer: the pair runs 2 to 6 us faster than its two passes).
  // Its long tiles start first, so unequal sums need no split while the CUs
  // have short tiles to fill in behind them; where the CUs' average load (in
  // stages of 16 k) is less than 1.6 times the longest tile, grad-input is
  // split along k in up to 4, its partial spectra added by the 2-D inverse (the
  // 512-channel layer, 6 bins: 42.3 us unsplit, 38.5 split in 4; 15 bins: 66.7
  // unsplit, 68.9 in 4)
  {
    const long Bk = p->kept, N = p->N, Ci = p->Cin, Co = p->Cout;
    p->ct[0] = bl_contract_tiling(N, Co, Ci, Bk, p->bf16);
    p->ct[1] = bl_contract_tiling(N, Ci, Co, Bk, p->bf16);
    p->ct[2] = bl_contract_tiling(Ci, Co, N, Bk, p->bf16);
    p->bp_s1 = 1;
    p->bp_bm = std::max(p->ct[1].bm, p->ct[2].bm);
    p->bp_bn = std::max(p->ct[1].bn, p->ct[2].bn);
    const long bm = p->bp_bm, bn = p->bp_bn, st1 = (Co + 15) / 16, st2 = (N + 15) / 16;
    const long tiles1 = Bk * ((N + bm - 1) / bm) * ((Ci + bn - 1) / bn);
    const long tiles2 = Bk * ((Ci + bm - 1) / bm) * ((Co + bn - 1) / bn);
    const double load = (double)(tiles1 * st1 + tiles2 * st2) / 256.0;
    if (p->Lh > 1)
      while (p->bp_s1 < 4 && st1 % (2 * p->bp_s1) == 0 && st1 / p->bp_s1 >= 16 && 1.6 * st1 / p->bp_s1 > load) p->bp_s1 *= 2;
    // A tile of the pair is one wave group's; where the longest is a serial chain
    // well past the CUs' load, two launches whose groups share a tile's sum are
    // the faster (combined call with stored spectra, pair / apart, us: 18 images,
    // 17 -> 1000 channels, 6 bins 56.8 / 32.4; 4 images, 17 -> 496, 28 bins 33.7 /
    // 22.9; -> 304 24.7 / 19.9, 12 stages apart, within the bound; 64 images, 64 ->
    // 400, 76 bins 41.6 / 51.0).
    const long longest = std::max((st1 + p->bp_s1 - 1) / p->bp_s1, st2);
    const double apart = (double)st1 / p->ct[1].ks + (double)st2 / p->ct[2].ks;
    if (longest - apart > 13 && longest > 2 * load) p->bp_s1 = 0;
  }
  // forward contractions with long sums in at most two tiles per CU are split
  // along k where the 2-D inverse can add the partial spectra as it loads them
  // (512 channels, contraction and inverse, unsplit against split in 2: 24 bins
  // 47.4 and 41.5 us, 15 bins 34.0 and 30.0, 6 bins 29.4 and 19.5; with 256
  // channels, 28 bins, 20.4 and 21.7: sums of 16 stages stay whole)
  p->fwd_split = 1;
  {
    const BlContractTiling& t0 = p->ct[0];
    const long tiles0 = (long)p->kept * ((p->N + t0.bm - 1) / t0.bm) * ((p->Cout + t0.bn - 1) / t0.bn);
    const long st0 = (p->Cin + 15) / 16;
    if (p->Lh > 1)
      while (p->fwd_split < 4 && st0 % (2 * p->fwd_split) == 0 && st0 / p->fwd_split >= 32 &&
             tiles0 * p->fwd_split <= 512)
        p->fwd_split *= 2;
    // On the vector ALUs instead (forward pass with stored spectra, us, split
    // tiles / those):
    //  - one or two images: past one tile per CU, where a tile has one wave group
    //    (512 -> 256, 28 bins 16.3 / 12.5, 45 bins 31.4 / 18.9; two images, 768 ->
    //    512, 15 bins 19.4 / 27.5, 28 bins 40.6 / 28.6; 1024 -> 16, 45 bins 20.7 /
    //    25.2, 66 bins 31.7 / 24.0), but for sums of 2048 (-> 16, 120 bins 49.0 /
    //    57.7); and one image of fewer than 768 channels (512 -> 64, 6 bins 13.0 /
    //    11.5; 768 -> 256, 28 bins 20.1 / 25.0) onto more than 32 (512 -> 16, 28
    //    bins 12.8 / 15.0);
    //  - one or two output channels (128 images, 512 -> 1, 120 bins 31.1 / 15.8;
    //    2048 -> 2 65.1 / 59.3), three or four of few rows (1024 -> 4, 64 images,
    //    120 bins 36.4 / 25.9; 128 images, 120 bins 40.6 / 42.3, 231 bins 61.6 /
    //    76.1), five to eight of fewer (512 -> 8, 16 images, 45 bins 15.1 / 11.1; 64
    //    images, 6 bins 13.3 / 11.2, 45 bins 16.6 / 17.8; 2048 -> 8, 16 images, 6
    //    bins 17.6 / 20.5).
    if (bl_contract_thin(p->N, p->Cout, p->Cin, p->kept, false, false)) {
      const long rows = p->kept * p->N;
      const bool row = (tiles0 * p->fwd_split > 256 && p->Cin < 2048) || (p->N == 1 && p->Cin < 768 && p->Cout > 32);
      const bool col = p->Cout <= 2 || (p->Cout <= 4 && rows <= 8192) || (rows <= 1536 && p->Cin < 2048);
      if (p->N <= 2 ? row : col) p->fwd_split = 1;
    }
    p->fwd_ks = bl_contract_groups(t0.bm, t0.bn, tiles0 * p->fwd_split, st0 / p->fwd_split, p->bf16);
  }
  // partial sums of the weight-gradient inverse DFT over bin slices (filters of
  // up to 9 taps; larger ones take a matrix product): enough slices for ~1024
  // blocks of 256 (c, f) pairs, at least 16 bins per slice, whole batches of 8
  // bins, and a slice's weights [bins][taps] within kWgradSliceLds
  p->wg_bins = (int)p->kept;
  p->wg_chunks = 1;
  p->wg_groups = 0;
  p->off_Part = o;
  const long T = (long)p->Kh * p->Kw;
  if (T <= 9) {
    const long Q = (long)p->Cin * p->Cout;
    const long xblocks = (Q + 255) / 256;
    const long want = (1024 + xblocks - 1) / xblocks;
    long per = std::max<long>(16, (p->kept + want - 1) / want);
    per = std::min((per + 7) / 8 * 8, kWgradSliceLds / (T * 8) / 8 * 8);
    const long chunks = (p->kept + per - 1) / per;
    p->wg_bins = (int)per;
    p->wg_chunks = (int)chunks;
    // 128 to 511 tiles of 16 x 16 channel pairs: one pass over all bins with
    // 2 or 4 groups of 256 threads per tile (k_wgrad_tile), at least 2048
    // waves, the bins' weights and the groups' sums within 64 KB of LDS each.
    // With more tiles one group per tile would sum every bin in series; the
    // bin slices above split that work instead.
    const long tiles = (long)((p->Cin + 15) / 16) * ((p->Cout + 15) / 16);
    int ng = 2;
    while (ng < 4 && tiles * ng * 4 < 2048) ng *= 2;
    p->wg_groups = (tiles < 512 && tiles * ng * 4 >= 2048 && p->kept * T * 8 <= 64 * 1024) ? ng : 0;
    if (chunks > 1) o = align_up(o + (size_t)chunks * Q * T * sizeof(float), 256);
  }
  // split-k partial tiles of the contraction (largest of the three passes and
  // of the paired backward launch)
  {
    const long Bk = p->kept, N = p->N, Ci = p->Cin, Co = p->Cout;
    size_t need = 0;
    const long mn[3] = {N * Co, N * Ci, Ci * Co};
    for (int i = 0; i < 3; ++i)
      if (p->ct[i].splits > 1) need = std::max(need, (size_t)p->ct[i].splits * Bk * mn[i] * cb);
    if (p->fwd_split > 1) need = std::max(need, (size_t)p->fwd_split * Bk * mn[0] * cb);
    if (p->bp_s1 > 1) need = std::max(need, (size_t)p->bp_s1 * Bk * mn[1] * cb);
    p->off_CPart = o;
    o = align_up(o + need, 256);
  }
  p->ws_bytes = o;
  *out = p;
  return BL_OK;
}

extern "C" bl_status_t bl_conv_plan_destroy(bl_conv_plan_t p) {
  if (!p) return BL_ERR_INVALID_ARG;
  bl_plan_tables_free(p->tables);
  delete p;
  return BL_OK;
}

extern "C" bl_status_t bl_conv_plan_info(bl_conv_plan_t p, int* fft_h, int* fft_w, int* r_h, int* r_w,
                                         long* kept, long* total, double* c_eff) {
  if (!p) return BL_ERR_INVALID_ARG;
  if (fft_h) *fft_h = p->ndim == 1 ? p->Lw : p->Lh;
  if (fft_w) *fft_w = p->ndim == 1 ? 1 : p->Lw;
  if (r_h) *r_h = p->r_h;
  if (r_w) *r_w = p->r_w;
  if (kept) *kept = p->kept;
  if (total) *total = p->total;
  if (c_eff) *c_eff = p->c_eff;
  return BL_OK;
}

extern "C" bl_status_t bl_conv_plan_get_mask(bl_conv_plan_t p, unsigned char* m, size_t n) {
  if (!p || !m || n != (size_t)p->total) return BL_ERR_INVALID_ARG;
  std::memcpy(m, p->mask.data(), n);
  return BL_OK;
}

extern "C" bl_status_t bl_conv_plan_get_bins(bl_conv_plan_t p, int* u, int* v, size_t n) {
  if (!p || !u || !v || n != (size_t)p->kept) return BL_ERR_INVALID_ARG;
  size_t b = 0;
  for (int r = 0; r < p->R; ++r)
    for (int vv = 0; vv < p->V; ++vv, ++b) {
      u[b] = bl_kept_row(r, p->r_h, p->Lh, p->R);
      v[b] = vv;
    }
  return BL_OK;
}

extern "C" bl_status_t bl_conv_workspace_size(bl_conv_plan_t p, size_t* bytes) {
  if (!p || !bytes) return BL_ERR_INVALID_ARG;
  *bytes = p->ws_bytes;
  return BL_OK;
}

extern "C" bl_status_t bl_conv_workspace_layout(bl_conv_plan_t p, size_t* off_x, size_t* off_w, size_t* off_dy) {
  if (!p) return BL_ERR_INVALID_ARG;
  if (off_x) *off_x = p->off_X;
  if (off_w) *off_w = p->off_W;
  if (off_dy) *off_dy = p->off_DY;
  return BL_OK;
}

extern "C" const char* bl_status_string(bl_status_t s) {
  switch (s) {
    case BL_OK: return "ok";
    case BL_ERR_INVALID_ARG: return "invalid argument";
    case BL_ERR_UNSUPPORTED: return "unsupported configuration";
    case BL_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
    case BL_ERR_HIP: return "HIP error";
    case BL_ERR_OOM: return "out of host memory";
  }
  return "unknown status";
}
