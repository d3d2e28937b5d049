// Kept spectra of series and of small planes as one matrix product (gfx950).
//
// A whole transform is linear in its plane's samples, so for series (any
// length) and planes of a few samples it is one product with a table of roots:
//   forward  X[b][re, im][p] = sum_k E[(b, re/im)][k] x[p][k], k over the samples,
//   inverse  y[p][j] = sum_k D[j][k] Y[k = (b, re/im)][p], the crop, the column
//            weights h_v and the scale in D.
// Series lengths of the FCN layers have large prime factors; a chirp-z FFT pads
// them to a power of two and pays for two transforms, and lengths past 700 had
// only the direct sum.  On the bf16 matrix cores (values split exactly into
// three bfloat16, split.hpp) the plain product is cheaper than either wherever
// its tiles are few enough; see the dispatch.
//
// One wave takes RM x 16 table rows and CN x 16 planes: planes are the columns,
// so that bin rows are read and written in runs of 16 planes.  Table operands
// come straight from L2 in the MFMA's layout (waves of a block share rows, so
// mostly from L1), data operands from HBM, split once per RM row tiles; no LDS
// and no barrier, except where KW waves share a tile's k range and add their
// sums in order.
#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "split.hpp"

namespace blc {
namespace {

struct PgemmArgs {
  unsigned P;          // planes
  int rows, K, steps;  // table rows, inner size, its steps of 32
  int n;               // samples per plane (forward: K; inverse: rows)
  int ctiles;          // groups of planes (blocks along the planes)
  unsigned F;          // filters: plane (c, f) = c F + f of the spectrum is plane f (P / F) + c of the samples; 0: the same
  unsigned nsplit;             // inverse: partial spectra to add
  unsigned long long pstride;  // complex values between two partial spectra
  const uintx4* tab;   // [row tile][step][part][lane]
};

// Index among the samples of spectrum plane p.
__device__ __forceinline__ size_t sample_plane(const PgemmArgs& g, unsigned p) {
  return g.F ? (size_t)(p % g.F) * (g.P / g.F) + p / g.F : (size_t)p;
}

// Eight k of a step for plane p: forward samples, inverse (bin, re/im) pairs.
// In the last step (tail) those past K repeat the plane's own: their table
// entries are zero, and what is not finite spreads to the whole plane anyway.
template <bool INV, bool PARTS>
__device__ __forceinline__ void load8(const void* in, const PgemmArgs& g, size_t p, int k0, bool tail, float* x) {
  if constexpr (!INV) {
    const float* s = static_cast<const float*>(in) + p * g.n;
    if (!tail || g.K % 4 == 0) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int k = k0 + 4 * h;
        const floatx4u v = *reinterpret_cast<const floatx4u*>(s + (tail ? min(k, g.K - 4) : k));
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * h + e] = v[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = s[min(k0 + e, g.K - 1)];
    }
  } else {
    const float2* s = static_cast<const float2*>(in) + p;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float2* q = s + (size_t)min((k0 >> 1) + e, (g.K >> 1) - 1) * g.P;
      float2 v = *q;
      if constexpr (PARTS)
        for (unsigned i = 1; i < g.nsplit; ++i) v = cadd(v, q[(size_t)i * g.pstride]);
      x[2 * e] = v.x, x[2 * e + 1] = v.y;
    }
  }
}

// S: stored-spectrum element of the forward output.
template <bool INV, int RM, int CN, int KW, bool PARTS, typename S>
__global__ __launch_bounds__(256, 2) void k_pgemm(const void* __restrict__ in, void* __restrict__ out_, PgemmArgs g) {
  constexpr int CW = 4 / KW;  // column groups of a block
  __shared__ float red[KW > 1 ? (KW - 1) * RM * CN * 256 : 1];
  const int lane = threadIdx.x & 63, g4 = lane >> 4, c16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), kw = wave / CW;
  const int ct = blockIdx.x % g.ctiles, rt = (blockIdx.x / g.ctiles) * RM;
  const unsigned c0 = ((unsigned)ct * CW + wave % CW) * (CN * 16);
  const int rtiles = (g.rows + 15) / 16;
  size_t p[CN];
#pragma unroll
  for (int c = 0; c < CN; ++c) {
    const unsigned q = min(c0 + 16 * c + c16, g.P - 1);  // columns past the last repeat it, and are not stored
    p[c] = INV ? q : sample_plane(g, q);
  }
  Acc16 d[RM][CN];
#pragma unroll
  for (int r = 0; r < RM; ++r)
#pragma unroll
    for (int c = 0; c < CN; ++c) d[r][c] = Acc16{};
  const uintx4* t[RM];
#pragma unroll
  for (int r = 0; r < RM; ++r) t[r] = g.tab + (size_t)min(rt + r, rtiles - 1) * g.steps * 192 + lane;
  float x[CN][8];
#pragma unroll
  for (int c = 0; c < CN; ++c) load8<INV, PARTS>(in, g, p[c], 32 * kw + 8 * g4, kw >= g.steps - 1, x[c]);
  for (int s = kw; s < g.steps; s += KW) {
    Split8 b[CN];
#pragma unroll
    for (int c = 0; c < CN; ++c) b[c] = split8(x[c]);
    const int next = min(s + KW, g.steps - 1);  // the last round loads its own step again
#pragma unroll
    for (int c = 0; c < CN; ++c) load8<INV, PARTS>(in, g, p[c], 32 * next + 8 * g4, next == g.steps - 1, x[c]);
#pragma unroll
    for (int r = 0; r < RM; ++r) {
      uintx4 a[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) a[q] = t[r][(s * 3 + q) * 64];
#pragma unroll
      for (int c = 0; c < CN; ++c) mma16(a, b[c].p, d[r][c]);
    }
  }
#pragma unroll
  for (int r = 0; r < RM; ++r)
#pragma unroll
    for (int c = 0; c < CN; ++c) d[r][c].hi += d[r][c].lo;
  if constexpr (KW > 1) {
    if (kw > 0) {
#pragma unroll
      for (int r = 0; r < RM; ++r)
#pragma unroll
        for (int c = 0; c < CN; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) red[(((kw - 1) * RM + r) * CN + c) * 256 + e * 64 + lane] = d[r][c].hi[e];
    }
    __syncthreads();
    if (kw > 0) return;
#pragma unroll
    for (int q = 0; q < KW - 1; ++q)
#pragma unroll
      for (int r = 0; r < RM; ++r)
#pragma unroll
        for (int c = 0; c < CN; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) d[r][c].hi[e] += red[((q * RM + r) * CN + c) * 256 + e * 64 + lane];
  }
#pragma unroll
  for (int r = 0; r < RM; ++r) {
    const int row = (rt + r) * 16 + 4 * g4;
#pragma unroll
    for (int c = 0; c < CN; ++c) {
      const unsigned col = c0 + 16 * c + c16;
      if (col >= g.P) continue;
      const floatx4 v = d[r][c].hi;
      if constexpr (!INV) {
        S* o = static_cast<S*>(out_) + col;
#pragma unroll
        for (int h = 0; h < 2; ++h)
          if (row + 2 * h < g.rows)
            spec_put(o, (size_t)((row >> 1) + h) * g.P, make_float2(v[2 * h], v[2 * h + 1]));
      } else {
        float* o = static_cast<float*>(out_) + sample_plane(g, col) * g.n + row;
        if (row + 4 <= g.rows) {
          *reinterpret_cast<floatx4u*>(o) = v;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (row + e < g.rows) o[e] = v[e];
        }
      }
    }
  }
}

struct TableGeom {
  int H, W, oi, oj, Lh, Lw, r_h, R, V;
  int rows, K, steps;
  double scale;  // inverse: 1 / (Lh Lw)
};

// Expands the roots e^{2 pi i m / Lh}, e^{2 pi i m / Lw} (double precision) into
// the split operands; one thread per (row tile, step, lane).
template <bool INV>
__global__ __launch_bounds__(256) void k_pgemm_table(const double2* __restrict__ rh, const double2* __restrict__ rw,
                                                     unsigned short* __restrict__ out, TableGeom g, long n) {
  const long id = (long)blockIdx.x * 256 + threadIdx.x;
  if (id >= n) return;
  const int lane = (int)(id & 63);
  const long ts = id >> 6;  // row tile * steps + step
  const int row = (int)(ts / g.steps) * 16 + (lane & 15), k0 = (int)(ts % g.steps) * 32 + 8 * (lane >> 4);
  for (int e = 0; e < 8; ++e) {
    const int k = k0 + e;
    double v = 0.0;
    if (row < g.rows && k < g.K) {
      const int bc = INV ? k : row, s = INV ? row : k;  // (bin, re/im) and sample
      const int b = bc >> 1, c = bc & 1, i = s / g.W, j = s - i * g.W;
      const int u = kept_row_d(b / g.V, g.r_h, g.Lh, g.R), w = b % g.V;
      const double2 a = rh[(long)u * (i + g.oi) % g.Lh], q = rw[(long)w * (j + g.oj) % g.Lw];
      v = c ? -(a.x * q.y + a.y * q.x) : a.x * q.x - a.y * q.y;
      if (INV) v *= g.scale * (w == 0 || 2 * w == g.Lw ? 1.0 : 2.0);
    }
    for (int p = 0; p < 3; ++p) {
      const unsigned f = __float_as_uint((float)v);
      const unsigned short h = (unsigned short)((f + 0x7FFFu + ((f >> 16) & 1u)) >> 16);
      out[((ts * 3 + p) * 64 + lane) * 8 + e] = h;
      v -= (double)__uint_as_float((unsigned)h << 16);
    }
  }
}

template <bool INV>
bl_status_t pgemm_table(const bl_conv_plan_s* p, int H, int W, int oi, int oj, int rows, int K, int steps,
                        const uintx4** out) {
  const std::vector<long> key{6, INV, p->Lh, p->Lw, p->r_h, p->V, H, W, oi, oj};
  const size_t units = (size_t)((rows + 15) / 16) * steps * 192;  // of 16 bytes
  const size_t roots = (size_t)p->Lh + p->Lw;                     // double2, after the table
  const float2* tab;
  const bl_status_t st = plan_table(
      p, key,
      [&](std::vector<float2>& h) {
        h.assign(2 * roots, make_float2(0.f, 0.f));
        double* r = reinterpret_cast<double*>(h.data());
        size_t at = 0;
        for (int L : {p->Lh, p->Lw})
          for (int k = 0; k < L; ++k) {
            const double a = 2.0 * 3.141592653589793238462643383279502884 * (double)k / (double)L;
            r[at++] = std::cos(a);
            r[at++] = std::sin(a);
          }
      },
      &tab, 2 * units,
      [&](const float2* d, float2* expanded) {
        const double2* rh = reinterpret_cast<const double2*>(d);
        const TableGeom g{H, W, oi, oj, p->Lh, p->Lw, p->r_h, p->R, p->V, rows, K, steps,
                          1.0 / ((double)p->Lh * (double)p->Lw)};
        const long n = (long)(units / 3);
        hipLaunchKernelGGL((k_pgemm_table<INV>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, 0, rh, rh + p->Lh,
                           reinterpret_cast<unsigned short*>(expanded), g, n);
      });
  *out = reinterpret_cast<const uintx4*>(tab);
  return st;
}

// Tables up to 64 MB.
bool table_fits(long rows, long K) { return (double)((rows + 15) / 16) * ((K + 31) / 32) * 3072.0 <= 64.0 * (1 << 20); }

template <bool INV, bool PARTS, typename S>
bl_status_t pgemm_launch(const bl_conv_plan_s* p, const void* in, void* out, PgemmArgs g, double bytes, double flops,
                         hipStream_t s) {
  const char* name = g.F ? (INV ? "wgrad_idft" : "spec_filt") : INV ? (p->Lh == 1 ? "spec_inv_1d" : "spec_inv_2d") : (p->Lh == 1 ? "spec_fwd_1d" : "spec_fwd_2d");
  const int rtiles = (g.rows + 15) / 16;
  auto go = [&](auto kern, int rm, int cn, int kw) {
    const int cols = cn * 16 * (4 / kw);
    g.ctiles = (int)((g.P + cols - 1) / cols);
    const long blocks = (long)g.ctiles * ((rtiles + rm - 1) / rm);
    if (blocks >= 2147483647L) return BL_ERR_UNSUPPORTED;
    return timed_launch(name, bytes, flops, s, [&](hipEvent_t e0, hipEvent_t e1) {
      hipExtLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, s, e0, e1, 0, in, out, g);
    });
  };
  auto waves = [&](int rm, int cn) { return (long)((rtiles + rm - 1) / rm) * ((g.P + 16 * cn - 1) / (16 * cn)); };
  if (waves(4, 2) >= 1024) return go(k_pgemm<INV, 4, 2, 1, PARTS, S>, 4, 2, 1);
  if (waves(4, 2) >= 192 && g.steps >= 8) return go(k_pgemm<INV, 4, 2, 4, PARTS, S>, 4, 2, 4);
  if (g.steps >= 4 && waves(2, 2) < 1024) return go(k_pgemm<INV, 2, 1, 4, PARTS, S>, 2, 1, 4);
  return go(k_pgemm<INV, 2, 1, 1, PARTS, S>, 2, 1, 1);
}

}  // namespace

bl_status_t launch_pgemm_fwd(const bl_conv_plan_s* p, const float* in, void* out, long P, int Hin, int Win, int oi,
                             int oj, hipStream_t s, int filters) {
  const long rows = 2 * p->kept, K = (long)Hin * Win;
  if (P >= 2147483647L || !table_fits(rows, K)) return BL_ERR_UNSUPPORTED;
  PgemmArgs g{};
  g.P = (unsigned)P, g.rows = (int)rows, g.K = (int)K, g.steps = (int)((K + 31) / 32), g.n = (int)K;
  g.F = (unsigned)filters;
  const bl_status_t st = pgemm_table<false>(p, Hin, Win, oi, oj, g.rows, g.K, g.steps, &g.tab);
  if (st != BL_OK) return st == BL_ERR_OOM ? BL_ERR_UNSUPPORTED : st;
  const double bytes = (double)P * K * 4 + (double)P * p->kept * (p->bf16 ? 4 : 8);
  const double flops = filters ? 0.0 : (double)P * 2.5 * p->Lh * p->Lw * std::log2(std::max(2.0, (double)p->Lh * p->Lw));
  return p->bf16 ? pgemm_launch<false, false, unsigned>(p, in, out, g, bytes, flops, s)
                 : pgemm_launch<false, false, float2>(p, in, out, g, bytes, flops, s);
}

bl_status_t launch_pgemm_inv(const bl_conv_plan_s* p, const float2* in, float* out, long P, int OH, int OW, int ci,
                             int cj, hipStream_t s, int nsplit, size_t pstride, int filters) {
  const long rows = (long)OH * OW, K = 2 * p->kept;
  if (P >= 2147483647L || !table_fits(rows, K)) return BL_ERR_UNSUPPORTED;
  PgemmArgs g{};
  g.P = (unsigned)P, g.rows = (int)rows, g.K = (int)K, g.steps = (int)((K + 31) / 32), g.n = (int)rows;
  g.F = (unsigned)filters;
  g.nsplit = (unsigned)std::max(1, nsplit), g.pstride = pstride;
  const bl_status_t st = pgemm_table<true>(p, OH, OW, ci, cj, g.rows, g.K, g.steps, &g.tab);
  if (st != BL_OK) return st == BL_ERR_OOM ? BL_ERR_UNSUPPORTED : st;
  const double bytes = (double)P * rows * 4 + (double)P * p->kept * 8 * g.nsplit;
  const double flops = filters ? 0.0 : (double)P * 2.5 * p->Lh * p->Lw * std::log2(std::max(2.0, (double)p->Lh * p->Lw));
  return g.nsplit > 1 ? pgemm_launch<true, true, float2>(p, in, out, g, bytes, flops, s)
                      : pgemm_launch<true, false, float2>(p, in, out, g, bytes, flops, s);
}

}  // namespace blc
