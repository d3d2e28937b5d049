// Kept spectra of series and of small planes as matrix products (gfx950).
//
// A whole transform is linear in its plane's samples, so for series (any
// length) and planes of a few samples it is a product with a table of roots.
// Seen from the plane's centre, sample k and its mirror image n - 1 - k have
// opposite angles, so pairs' sums go through a table of cosines and their
// differences through one of sines, half the products of the plain sum:
//   forward  X[b] = e^{-i a(b)} (sum_k C[b][k] (x[k] + x[n-1-k]) - i sum_k S[b][k] (x[k] - x[n-1-k])),
//   inverse  y[k], y[n-1-k] = sum_b C[k][b] Re Y' -+ sum_b S[k][b] Im Y', Y'[b] = e^{i a(b)} Y[b],
// a(b) bin b's angle at the centre; the crop, the column weights h_v and the
// scale are in the inverse's tables.
// Series lengths of the FCN layers have large prime factors; a chirp-z FFT pads
// them to a power of two and pays for two transforms, and lengths past 700 had
// only the direct sum.  On the bf16 matrix cores (values split exactly into
// three bfloat16, split.hpp) the plain product is cheaper than either wherever
// its tiles are few enough; see the dispatch.
//
// Planes are the columns, so that bin rows are read and written in runs of 16
// planes; data operands come from HBM and are split once per two row tiles.
// What bounds it: vector instructions (fold, turn, split: 30 to 50 % of the
// SIMDs' cycles against 15 to 18 % of the products), and at one or two waves to
// a SIMD the waits for loads (30 to 40 % of the waves' time).
// Measured: 1250 samples from 628 bins, 1024 series 26.8 forward (0.35 of the
// rate of a large bf16 product), 27.4 inverse.
#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "split.hpp"

namespace blc {
namespace {

struct PgemmArgs {
  unsigned P;          // planes
  int kept, n;         // bins; samples per plane
  int rows, steps;     // table rows (forward: bins, inverse: sample pairs); steps of 32 of the other
  int ctiles;          // groups of planes (blocks along the planes)
  unsigned F;          // inverse of a filter bank of F filters: plane (c, f) = c F + f of the spectrum is plane f (P / F) + c of the samples; 0: the same
  unsigned nsplit;             // inverse: partial spectra to add
  unsigned long long pstride;  // complex values between two partial spectra
  const uintx4* tab;   // [row tile][step][cosine, sine][part][lane]
  // e^{i a(b)} of every bin's angle at the plane's centre, to a multiple of 32
  // bins; forward: each followed by what its rounding leaves
  const float2* phase;
};

// Index among the samples of spectrum plane p.
__device__ __forceinline__ size_t sample_plane(const PgemmArgs& g, unsigned p) {
  return g.F ? (size_t)(p % g.F) * (g.P / g.F) + p / g.F : (size_t)p;
}

// What a step's eight k of a plane are loaded from: forward eight sample pairs,
// inverse eight bins.  Those past the last (their table entries are zero)
// repeat the plane's own: what is not finite spreads to the whole plane anyway.
template <bool INV, bool PARTS>
__device__ __forceinline__ void load8(const void* in, const PgemmArgs& g, size_t p, int k0, float* x) {
  if constexpr (!INV) {
    const float* s = static_cast<const float*>(in) + p * g.n;
#pragma unroll
    for (int h = 0; h < 2; ++h) {  // (n >= 4: a quad that starts at a pair's first sample ends within the plane)
      const int k = min(k0 + 4 * h, g.n - 4);
      const floatx4u v = *reinterpret_cast<const floatx4u*>(s + k);
      const floatx4u w = *reinterpret_cast<const floatx4u*>(s + (g.n - 4 - k));
#pragma unroll
      for (int e = 0; e < 4; ++e) x[4 * h + e] = v[e], x[8 + 4 * h + e] = w[3 - e];
    }
  } else {
    const float2* s = static_cast<const float2*>(in) + p;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float2* q = s + (size_t)min(k0 + e, g.kept - 1) * g.P;
      float2 v = *q;
      if constexpr (PARTS)
        for (unsigned i = 1; i < g.nsplit; ++i) v = cadd(v, q[(size_t)i * g.pstride]);
      x[e] = v.x, x[8 + e] = v.y;
    }
  }
}

// The step's operands of the cosine and the sine product: sums and differences
// of the pairs, or the bins turned to the plane's centre.
template <bool INV>
__device__ __forceinline__ void fold8(const float2* phase, const float* x, Split8* b) {
  float u[8], v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    if constexpr (!INV) {
      u[e] = x[e] + x[8 + e], v[e] = x[e] - x[8 + e];
    } else {
      const float2 t = phase[e];
      u[e] = fmaf(x[e], t.x, -x[8 + e] * t.y), v[e] = fmaf(x[e], t.y, x[8 + e] * t.x);
    }
  }
  b[0] = split8(u), b[1] = split8(v);
}

// One wave: RM x 16 table rows (each a cosine and a sine product) by 16 planes.
// S: stored-spectrum element of the forward output.
template <bool INV, int RM, int KW, bool PARTS, typename S>
__global__ __launch_bounds__(256, 2) void k_pgemm(const void* __restrict__ in, void* __restrict__ out_, PgemmArgs g) {
  constexpr bool ST = KW == 1 && RM == 2;  // the waves share their table rows: staged through LDS, a step ahead
  __shared__ float red[KW > 1 ? (KW - 1) * RM * 512 : 1];
  __shared__ uintx4 stage[2][ST ? RM * 384 : 1];
  __shared__ uintx4 turns[2][16];  // a step's 32 phases
  const int lane = threadIdx.x & 63, g4 = lane >> 4, c16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), kw = KW > 1 ? wave : 0;
  const int ct = blockIdx.x % g.ctiles, rt = (blockIdx.x / g.ctiles) * RM;
  const unsigned col = (KW > 1 ? (unsigned)ct : (unsigned)ct * 4 + wave) * 16 + c16;
  const int rtiles = (g.rows + 15) / 16;
  const unsigned colc = min(col, g.P - 1);  // columns past the last repeat it, and are not stored
  const size_t p = INV ? (size_t)colc : sample_plane(g, colc);
  Acc16 d[RM][2];  // cosine and sine sums
#pragma unroll
  for (int r = 0; r < RM; ++r) d[r][0] = d[r][1] = Acc16{};
  // Loads return in order: a step's table is asked for before the planes' next
  // values, so that waiting for the one does not wait for the other.
  const int last = g.steps - 1;
  if constexpr (ST) {
    const uintx4* tp[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int i = threadIdx.x + 256 * j;
      tp[j] = g.tab + (size_t)min(rt + i / 384, rtiles - 1) * g.steps * 384 + i % 384;
    }
    uintx4 tv[3], pv{};
    auto fetch = [&](int s) {
#pragma unroll
      for (int j = 0; j < 3; ++j) tv[j] = tp[j][(size_t)s * 384];
      if (INV && threadIdx.x < 16) pv = reinterpret_cast<const uintx4*>(g.phase)[s * 16 + threadIdx.x];
    };
    auto put = [&](int w) {
#pragma unroll
      for (int j = 0; j < 3; ++j) stage[w][threadIdx.x + 256 * j] = tv[j];
      if (INV && threadIdx.x < 16) turns[w][threadIdx.x] = pv;
      __syncthreads();
    };
    float x[2][16];
    fetch(0);
#pragma unroll
    for (int w = 0; w < 2; ++w) load8<INV, PARTS>(in, g, p, 32 * min(w, last) + 8 * g4, x[w]);
    put(0);
    // A step of buffer w: its planes' values were loaded two steps ago, its table
    // a step ago.  Steps past the last load the last again.
    auto step = [&](int s, int w) {
      Split8 b[2];
      fetch(min(s + 1, last));
      __builtin_amdgcn_sched_barrier(0);
      fold8<INV>(reinterpret_cast<const float2*>(turns[w]) + 8 * g4, x[w], b);
      load8<INV, PARTS>(in, g, p, 32 * min(s + 2, last) + 8 * g4, x[w]);
#pragma unroll
      for (int r = 0; r < RM; ++r)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          uintx4 a[3];
#pragma unroll
          for (int q = 0; q < 3; ++q) a[q] = stage[w][((r * 2 + h) * 3 + q) * 64 + lane];
          mma16(a, b[h].p, d[r][h]);
        }
      put(w ^ 1);  // (last read a step ago, before the barrier in between)
    };
    for (int s = 0; s <= last; s += 2) {
      step(s, 0);
      if (s < last) step(s + 1, 1);
    }
  } else {
    float x[16];
    load8<INV, PARTS>(in, g, p, 32 * min(kw, last) + 8 * g4, x);
    for (int s = kw; s <= last; s += KW) {
      uintx4 a[RM][6];
      Split8 b[2];
#pragma unroll
      for (int r = 0; r < RM; ++r) {
        const uintx4* t = g.tab + ((size_t)min(rt + r, rtiles - 1) * g.steps + s) * 384 + lane;
#pragma unroll
        for (int q = 0; q < 6; ++q) a[r][q] = t[q * 64];
      }
      __builtin_amdgcn_sched_barrier(0);
      fold8<INV>(g.phase + 32 * s + 8 * g4, x, b);
      load8<INV, PARTS>(in, g, p, 32 * min(s + KW, last) + 8 * g4, x);  // the last round loads the last step again
#pragma unroll
      for (int r = 0; r < RM; ++r)
#pragma unroll
        for (int h = 0; h < 2; ++h) mma16(a[r] + 3 * h, b[h].p, d[r][h]);
    }
  }
  floatx4 w[INV ? 1 : RM][4];  // (asked for before the sums are put together)
  if constexpr (!INV) {
#pragma unroll
    for (int r = 0; r < RM; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        w[r][e] = reinterpret_cast<const floatx4*>(g.phase)[min(rt + r, rtiles - 1) * 16 + 4 * g4 + e];
  }
#pragma unroll
  for (int r = 0; r < RM; ++r)
#pragma unroll
    for (int h = 0; h < 2; ++h) d[r][h].hi += d[r][h].lo;
  if constexpr (KW > 1) {
    auto sums = [&](int q, auto f) {
#pragma unroll
      for (int r = 0; r < RM; ++r)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) f(red[((q * RM + r) * 2 + h) * 256 + e * 64 + lane], d[r][h].hi, e);
    };
    if (kw > 0) sums(kw - 1, [](float& m, floatx4& v, int e) { m = v[e]; });
    __syncthreads();
    if (kw > 0) return;
#pragma unroll
    for (int q = 0; q < KW - 1; ++q) sums(q, [](float& m, floatx4& v, int e) { v[e] += m; });
  }
  if (col >= g.P) return;
#pragma unroll
  for (int r = 0; r < RM; ++r) {
    const int row = (rt + r) * 16 + 4 * g4;
    const floatx4 u = d[r][0].hi, v = d[r][1].hi;
    if constexpr (!INV) {  // X = (sum of cosines + i (sum of negated sines)) e^{-i a(b)}
      // A bin's phase is one for all planes: energies summed over the planes would
      // be off by twice its magnitude's rounding, so what that leaves goes in too
      // (4608 planes of 5 x 5: 3.3e-8 -> 3.9e-9).
      S* o = static_cast<S*>(out_) + col;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const floatx4 t = w[r][e];
        const float x = fmaf(u[e], t[2], v[e] * t[3]), y = fmaf(v[e], t[2], -u[e] * t[3]);
        if (row + e < g.rows)
          spec_put(o, (size_t)(row + e) * g.P,
                   make_float2(fmaf(u[e], t[0], fmaf(v[e], t[1], x)), fmaf(v[e], t[0], fmaf(-u[e], t[1], y))));
      }
    } else {
      float* o = static_cast<float*>(out_) + sample_plane(g, col) * g.n;
      const floatx4 lo = u + v, hi = u - v;
      if (row + 4 <= g.rows) {
        *reinterpret_cast<floatx4u*>(o + row) = lo;
        *reinterpret_cast<floatx4u*>(o + (g.n - 4 - row)) = (floatx4){hi[3], hi[2], hi[1], hi[0]};
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (row + e < g.rows) o[row + e] = lo[e], o[g.n - 1 - row - e] = hi[e];
      }
    }
  }
}

struct TableGeom {
  int H, W, Lh, Lw, r_h, R, V;
  int kept, rows, steps, phases;
  int oi, oj;    // grid offset of the second set of phases (the first has none)
  double scale;  // inverse: 1 / (Lh Lw)
};

// The operands (split root tables) and, after them, the bins' phases for both
// of the plan's offsets, in double precision; one thread per (row tile, step,
// lane, k of eight): a thread for all eight k is a serial chain, 5.8 to 9.4 us.
template <bool INV>
__global__ __launch_bounds__(256) void k_pgemm_table(unsigned short* __restrict__ out, float2* __restrict__ phase,
                                                     TableGeom g, long n) {
  const long id = (long)blockIdx.x * 256 + threadIdx.x;
  if (id >= n) return;
  // e^{pi i (u i / Lh + w j / Lw)}, i and j of either sign (sides and samples up to 4096: products of 25 bits)
  auto root = [&](int b, int i, int j, double* re, double* im) {
    const int u = kept_row_d(b / g.V, g.r_h, g.Lh, g.R), w = b % g.V;
    sincospi((double)(u * i % (2 * g.Lh)) / g.Lh + (double)(w * j % (2 * g.Lw)) / g.Lw, im, re);
  };
  double re, im;
  if (id < g.phases)
    for (int set = 0; set < 2; ++set) {
      root((int)min(id, (long)g.kept - 1), (set ? 2 * g.oi : 0) + g.H - 1, (set ? 2 * g.oj : 0) + g.W - 1, &re, &im);
      const float2 hi = make_float2((float)re, (float)im);
      if constexpr (INV) {
        phase[set * g.phases + id] = hi;
      } else {
        phase[2 * (set * g.phases + id)] = hi;
        phase[2 * (set * g.phases + id) + 1] = make_float2((float)(re - hi.x), (float)(im - hi.y));
      }
    }
  const int e = (int)(id & 7), lane = (int)(id >> 3 & 63);
  const long ts = id >> 9;  // row tile * steps + step
  const int row = (int)(ts / g.steps) * 16 + (lane & 15), k = (int)(ts % g.steps) * 32 + 8 * (lane >> 4) + e;
  const int pairs = (g.H * g.W + 1) / 2, b = INV ? k : row, s = INV ? row : k;
  double v[2] = {0.0, 0.0};
  if (b < g.kept && s < pairs) {
    const int i = s / g.W, j = s - i * g.W;
    root(b, 2 * i - (g.H - 1), 2 * j - (g.W - 1), &re, &im);
    // (the middle sample of an odd count is its own partner)
    const double f = INV ? g.scale * (b % g.V == 0 || 2 * (b % g.V) == g.Lw ? 1.0 : 2.0) : 2 * s + 1 == g.H * g.W ? 0.5 : 1.0;
    v[0] = f * re, v[1] = -f * im;
  }
  for (int h = 0; h < 2; ++h) split3_store(v[h], out + ((ts * 2 + h) * 3 * 64 + lane) * 8 + e, 512);
}

// Row tiles and steps of a transform from or to n samples; tables up to 64 MB.
template <bool INV>
bool pgemm_sizes(const bl_conv_plan_s* p, long P, long n, PgemmArgs& g) {
  const long pairs = (n + 1) / 2, rows = INV ? pairs : p->kept, k = INV ? p->kept : pairs;
  const double units = (double)((rows + 15) / 16) * ((k + 31) / 32) * 6144.0;
  if (P >= 2147483647L || units > 64.0 * (1 << 20) || (!INV && n < 4)) return false;
  g.P = (unsigned)P, g.kept = (int)p->kept, g.n = (int)n, g.rows = (int)rows, g.steps = (int)((k + 31) / 32);
  return true;
}

// The operands depend on the samples' shape and the band, not on where the
// samples lie on the grid: inputs and outputs of one size share them, and the
// phases of the plan's two places (the input's, after the padding, and the
// output's) are kept beside them.
template <bool INV>
bl_status_t pgemm_table(const bl_conv_plan_s* p, int H, int W, int oi, int oj, PgemmArgs& g, hipStream_t s) {
  const bool place = oi != 0 || oj != 0;
  if (place && (oi != p->pt || oj != p->pl)) return BL_ERR_UNSUPPORTED;
  const std::vector<long> key{6, INV, p->Lh, p->Lw, p->r_h, p->V, H, W};
  const size_t units = (size_t)((g.rows + 15) / 16) * g.steps * 384;  // of 16 bytes
  const size_t phases = (size_t)(g.kept + 31) / 32 * 32;              // float2, after the operands
  const float2* tab;
  const bl_status_t st = plan_table_on_device(
      p, key, 2 * units + (INV ? 2 : 4) * phases,
      [&](float2* d) {
        const TableGeom t{H, W, p->Lh, p->Lw, p->r_h, p->R, p->V, g.kept, g.rows, g.steps, (int)phases, p->pt, p->pl,
                          1.0 / ((double)p->Lh * (double)p->Lw)};
        const long n = (long)(units / 6) * 8;
        hipLaunchKernelGGL((k_pgemm_table<INV>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                           reinterpret_cast<unsigned short*>(d), d + 2 * units, t, n);
      },
      &tab, s);
  g.tab = reinterpret_cast<const uintx4*>(tab);
  g.phase = tab + 2 * units + (place ? (INV ? 1 : 2) * phases : 0);
  return st;
}

template <bool INV, bool PARTS, typename S>
bl_status_t pgemm_launch(const bl_conv_plan_s* p, const void* in, void* out, PgemmArgs g, double bytes, double flops,
                         hipStream_t s) {
  const char* name = g.F ? "wgrad_idft"
                     : INV ? (p->Lh == 1 ? "spec_inv_1d" : "spec_inv_2d") : (p->Lh == 1 ? "spec_fwd_1d" : "spec_fwd_2d");
  const int rtiles = (g.rows + 15) / 16;
  auto go = [&](auto kern, int rm, int kw) {
    const int cols = 16 * (4 / kw);
    g.ctiles = (int)((g.P + cols - 1) / cols);
    const long blocks = (long)g.ctiles * ((rtiles + rm - 1) / rm);
    if (blocks >= 2147483647L) return BL_ERR_UNSUPPORTED;
    return timed_launch(name, bytes, flops, s, [&](hipEvent_t e0, hipEvent_t e1) {
      hipExtLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, s, e0, e1, 0, in, out, g);
    });
  };
  // Two row tiles to a wave with the table staged once their waves give every
  // SIMD one; below that a block's waves share a tile's k range, with one row
  // tile to a wave below a quarter.  Forward / inverse us of the three:
  // 270 samples, 138 bins, 8192 planes 14.8 / 13.5, 16.8 / 18.1, 20.7 / 22.0; 2048
  // planes 7.4 / 6.8, 6.7 / 6.4, 7.5 / 7.4; 256 planes 6.5 / 6.4, 4.2 / 4.2, 4.0 / 4.0.
  // 1250 samples, 628 bins, 2048 planes 39 / 39, 46 / 48, 63 / 67; 64 planes
  // 16 / 18, 9.6 / 9.0, 7.2 / 8.3.  (Two column groups to a wave: 18.2 / 15.9 and
  // 47 / 47 of the largest, its waves too few.)
  const long ctiles = (g.P + 15) / 16, waves = (rtiles + 1) / 2 * ctiles;
  if (rtiles > 1 && waves >= 1024) return go(k_pgemm<INV, 2, 1, PARTS, S>, 2, 1);
  if (rtiles > 1 && waves >= 256 && g.steps >= 4) return go(k_pgemm<INV, 2, 4, PARTS, S>, 2, 4);
  if (g.steps >= 2 && rtiles * ctiles < 2048) return go(k_pgemm<INV, 1, 4, PARTS, S>, 1, 4);
  return go(k_pgemm<INV, 1, 1, PARTS, S>, 1, 1);
}

}  // namespace

bl_status_t launch_pgemm_fwd(const bl_conv_plan_s* p, const float* in, void* out, long P, int Hin, int Win, int oi,
                             int oj, hipStream_t s) {
  const long n = (long)Hin * Win;
  PgemmArgs g{};
  if (!pgemm_sizes<false>(p, P, n, g)) return BL_ERR_UNSUPPORTED;
  const bl_status_t st = pgemm_table<false>(p, Hin, Win, oi, oj, g, s);
  if (st != BL_OK) return st == BL_ERR_OOM ? BL_ERR_UNSUPPORTED : st;
  const double bytes = (double)P * n * 4 + (double)P * p->kept * (p->bf16 ? 4 : 8);
  const double flops = (double)P * 2.5 * p->Lh * p->Lw * std::log2(std::max(2.0, (double)p->Lh * p->Lw));
  return p->bf16 ? pgemm_launch<false, false, unsigned>(p, in, out, g, bytes, flops, s)
                 : pgemm_launch<false, false, float2>(p, in, out, g, bytes, flops, s);
}

bl_status_t launch_pgemm_inv(const bl_conv_plan_s* p, const float2* in, float* out, long P, int OH, int OW, int ci,
                             int cj, hipStream_t s, int nsplit, size_t pstride, int filters) {
  const long n = (long)OH * OW;
  PgemmArgs g{};
  if (!pgemm_sizes<true>(p, P, n, g)) return BL_ERR_UNSUPPORTED;
  g.F = (unsigned)filters;
  g.nsplit = (unsigned)std::max(1, nsplit), g.pstride = pstride;
  const bl_status_t st = pgemm_table<true>(p, OH, OW, ci, cj, g, s);
  if (st != BL_OK) return st == BL_ERR_OOM ? BL_ERR_UNSUPPORTED : st;
  const double bytes = (double)P * n * 4 + (double)P * p->kept * 8 * g.nsplit;
  const double flops = filters ? 0.0 : (double)P * 2.5 * p->Lh * p->Lw * std::log2(std::max(2.0, (double)p->Lh * p->Lw));
  return g.nsplit > 1 ? pgemm_launch<true, true, float2>(p, in, out, g, bytes, flops, s)
                      : pgemm_launch<true, false, float2>(p, in, out, g, bytes, flops, s);
}

}  // namespace blc
