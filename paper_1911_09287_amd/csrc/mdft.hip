// 2-D kept spectra of any grid by matrix products on the matrix cores (gfx950).
//
// A kept spectrum is two small matrix products per plane: with the placed
// input x [H][W], T = x Ew (Ew the W x V roots of the kept columns, real times
// complex) and X = Eh T (the R kept rows); the inverse is the mirror image,
// Z = Eh^H Y over the kept rows, then y = Re(Z Ew^H) with the Hermitian column
// weights (c2r: imaginary parts of the DC and Nyquist columns are dropped by
// zero weights).  Only kept columns and rows are formed, and only the input's
// or output's window of the grid, so grid size and padding cost nothing else,
// and any size takes the same code: the products are padded to tiles of 16
// with zeros.  Rows u and -u share their cosines and sines: with P = C T and
// Q = S T over u = 0 .. r_h, X[+-u] = (Pre +- Qim, Pim -+ Qre), half the
// products; the inverse forms Y[u] +- Y[-u] first, likewise.
//
// fp32 values are split exactly into three bfloat16 (split.hpp), six products
// each; the root tables are split on the host from double precision.  Few
// accumulator roundings (6 per 32 terms, five of them in the small products'
// own accumulator) make the error about that of the FFT kernels.
//
// A block takes G planes.  Forward: rows of 16 (plane, input row) go from HBM
// into MFMA operands, T passes through LDS once as [v][plane][re, im][row], and
// the second product's columns (v, plane, re/im) leave as runs of G planes of
// a bin row; lane pairs hold re and im of one column and trade halves so that
// each stores 8 bytes, of row +u or -u.  Inverse: lane pairs load rows +u and
// -u, Z passes through LDS once as [plane][row][v, re/im], and the second
// product's results are 4 consecutive samples of an output row per lane.
// What bounds it: the HBM stream where planes are many (see the measurements at
// the dispatch), else the latency of its two load phases.
#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "split.hpp"

namespace blc {
namespace {

constexpr int kWaves = kThreads / 64;

struct MdftArgs {
  int H, W;           // forward: input plane; inverse: output window
  int r_h, R, V;      // kept band
  unsigned P;         // planes
  int lg;             // planes per block: 1 << lg
  unsigned VP;        // V P, values between two kept rows
  int S1, S2;         // LDS strides (floats): forward column, kept column; inverse row, plane
  int n1, n2, m2;     // tiles: see the kernels
  unsigned magic;     // ceil(2^32 / H) (H > 1): plane of a row of the block
  unsigned K;         // plane groups per 128-byte line (as the FFT kernels')
  unsigned nsplit;              // inverse: partial spectra to add
  unsigned long long pstride;   // complex values between two partial spectra
  const uintx4 *t1, *t2;        // root tables of the two products, as MFMA operands
};

// Value of the other lane of an even/odd lane pair (DPP quad permutation 1 0 3 2).
__device__ __forceinline__ float pair_swap(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, false));
}

// Plane group of a block: the K groups that fill a 128-byte line of a bin row
// go to blocks of one XCD, while blocks in flight cover one range of planes.
__device__ inline unsigned mdft_group(unsigned b, unsigned nb, unsigned K) {
  const unsigned set = 8u * K;
  if (K <= 1 || b >= nb / set * set) return b;
  const unsigned r = b % set;
  return b - r + (r % 8u) * K + r / 8u;
}

// Operand q of a table: [tile][k step][part][lane].
template <int KS>
__device__ __forceinline__ void table_frag(const uintx4* t, int tile, int ks, uintx4* f) {
#pragma unroll
  for (int p = 0; p < 3; ++p) f[p] = t[((tile * KS + ks) * 3 + p) * 64 + (threadIdx.x & 63)];
}

__device__ __forceinline__ int div_magic(int e, int d, unsigned magic) {
  return d == 1 ? e : (int)__umulhi((unsigned)e, magic);
}

// Forward transform of the planes of one block (id of nb).  KA, KB: steps of 32
// of the input width and height; S: stored-spectrum element.  t1: Ew [n1 tiles
// of (v, re/im)][KA]; t2: C and S of the rows u <= r_h, [2 m2 tiles][KB].
template <int KA, int KB, typename S>
__device__ __forceinline__ void mdft_fwd_block(const float* __restrict__ in, S* __restrict__ out, const MdftArgs& g,
                                               unsigned id, unsigned nb, float* sm) {
  constexpr int RT = KA == 1 ? 4 : 2;  // row tiles a wave holds at a time
  constexpr int CT = KB == 1 ? 4 : 2;  // column tiles
  const int lane = threadIdx.x & 63, g4 = lane >> 4, c16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned p0 = mdft_group(id, nb, g.K) << g.lg;
  if (p0 >= g.P) return;
  const int np = (int)min(1u << g.lg, g.P - p0);
  const int rows = np * g.H, tiles = (rows + 15) / 16;
  const float* src = in + (size_t)p0 * g.H * g.W;
  for (int t0 = wave * RT; t0 < tiles; t0 += kWaves * RT) {
    float x[RT][KA][8];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int row = (t0 + t) * 16 + c16;
      const float* xr = src + (row < rows ? row : 0) * g.W;
      // samples past the row repeat its own (their table entries are zero, and
      // what is not finite spreads to the whole plane anyway); rows past the
      // last are not stored
#pragma unroll
      for (int k = 0; k < KA; ++k) {
        const int j = 32 * k + 8 * g4;
        if (g.W >= 8 && g.W % 8 == 0) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const floatx4u v = *reinterpret_cast<const floatx4u*>(xr + min(j, g.W - 8) + 4 * h);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[t][k][4 * h + e] = v[e];
          }
        } else if (g.W % 4 == 0) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const floatx4u v = *reinterpret_cast<const floatx4u*>(xr + min(j + 4 * h, g.W - 4));
#pragma unroll
            for (int e = 0; e < 4; ++e) x[t][k][4 * h + e] = v[e];
          }
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) x[t][k][e] = xr[min(j + e, g.W - 1)];
        }
      }
    }
    Split8 a[RT][KA];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int k = 0; k < KA; ++k)
        if (t0 + t < tiles) a[t][k] = split8(x[t][k]);
    for (int n = 0; n < g.n1; ++n) {
      uintx4 b[KA][3];
#pragma unroll
      for (int k = 0; k < KA; ++k) table_frag<KA>(g.t1, n, k, b[k]);
      const int col = n * 16 + c16, v = col >> 1, c = col & 1;
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        if (t0 + t >= tiles) break;
        Acc16 d{};
#pragma unroll
        for (int k = 0; k < KA; ++k) mma16(a[t][k].p, b[k], d);
        const int row = (t0 + t) * 16 + 4 * g4;
        if (v < g.V && row < rows) {
          int p = div_magic(row, g.H, g.magic), i = row - p * g.H;
          float* o = sm + v * g.S2 + c * g.S1;
          if (g.H % 4 == 0) {  // the four rows are one plane's, and rows past the last are whole groups
            *reinterpret_cast<floatx4*>(o + 2 * p * g.S1 + i) = d.hi + d.lo;
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              if (row + r < rows) o[2 * p * g.S1 + i] = d.hi[r] + d.lo[r];
              if (++i == g.H) i = 0, ++p;
            }
          }
        }
      }
    }
  }
  __syncthreads();
  // columns (v, plane, re/im), planes G apart per v
  const int cols = (2 * g.V) << g.lg, ctiles = (cols + 15) / 16;
  const float sgn = (lane & 1) ? -1.f : 1.f;
  for (int t0 = wave * CT; t0 < ctiles; t0 += kWaves * CT) {
    Split8 b[CT][KB];
    S* dst[CT];
    bool live[CT];
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      const int col = (t0 + t) * 16 + c16, vp = col >> 1, v = vp >> g.lg, p = vp - (v << g.lg);
      live[t] = col < cols && p < np;
      dst[t] = out + (p0 + p) + (unsigned)v * g.P;
      if (t0 + t >= ctiles) break;
      // columns that are not live are not stored; rows past the plane repeat
      // its last ones (zero table entries), or are zeroed
      const float* tc = sm + (live[t] ? v * g.S2 + (2 * p + (col & 1)) * g.S1 : 0);
      const int last = (g.H - 1) & ~3;
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const int i = 32 * k + 8 * g4;
        float w[8];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const floatx4 q = *reinterpret_cast<const floatx4*>(tc + min(i + 4 * h, last));
#pragma unroll
          for (int e = 0; e < 4; ++e) w[4 * h + e] = q[e];
        }
        if (g.H % 4 != 0) {
#pragma unroll
          for (int e = 0; e < 8; ++e) w[e] = i + e < g.H ? w[e] : 0.f;
        }
        b[t][k] = split8(w);
      }
    }
    for (int m = 0; m < g.m2; ++m) {
      uintx4 ac[KB][3], as[KB][3];
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        table_frag<KB>(g.t2, m, k, ac[k]);
        table_frag<KB>(g.t2, g.m2 + m, k, as[k]);
      }
#pragma unroll
      for (int t = 0; t < CT; ++t) {
        if (t0 + t >= ctiles) break;
        Acc16 dc{}, ds{};
#pragma unroll
        for (int k = 0; k < KB; ++k) {
          mma16(ac[k], b[t][k].p, dc);
          mma16(as[k], b[t][k].p, ds);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int u = m * 16 + 4 * g4 + r;
          const float c = dc.hi[r] + dc.lo[r], o = pair_swap(ds.hi[r] + ds.lo[r]);
          const float plus = fmaf(sgn, o, c), minus = fmaf(-sgn, o, c);  // this part of X[u] and X[-u]
          const float other = pair_swap((lane & 1) ? plus : minus);
          const int slot = (lane & 1) ? g.R - u : u;
          const bool ok = (lane & 1) ? u >= 1 && slot > g.r_h : u <= g.r_h;
          if (live[t] && ok)
            spec_put(dst[t], (unsigned)slot * g.VP,
                     (lane & 1) ? make_float2(other, minus) : make_float2(plus, other));
        }
      }
    }
  }
}

template <int KA, int KB, typename S>
__global__ __launch_bounds__(kThreads) void k_mdft_fwd(const float* __restrict__ in, S* __restrict__ out, MdftArgs g) {
  extern __shared__ __align__(16) float smf[];
  mdft_fwd_block<KA, KB, S>(in, out, g, blockIdx.x, gridDim.x, smf);
}

// Inverse transform of the planes of one block (id of nb).  KA: steps of 32
// rows u <= r_h, KB: steps of 32 (v, re/im).  t1: C and S of the output rows,
// [2 n1 tiles][KA]; t2: weighted column roots of the output columns, [n2 tiles][KB].
template <int KA, int KB, bool PARTS>
__device__ __forceinline__ void mdft_inv_block(const float2* __restrict__ in, float* __restrict__ out,
                                               const MdftArgs& g, unsigned id, unsigned nb, float* sm) {
  constexpr int CT = 2;
  constexpr int RT = KB == 1 ? 4 : 2;
  const int lane = threadIdx.x & 63, g4 = lane >> 4, c16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned p0 = mdft_group(id, nb, g.K) << g.lg;
  if (p0 >= g.P) return;
  const int np = (int)min(1u << g.lg, g.P - p0);
  const bool odd = lane & 1;
  const int cols = (2 * g.V) << g.lg, ctiles = (cols + 15) / 16;
  for (int t0 = wave * CT; t0 < ctiles; t0 += kWaves * CT) {
    float2 y[CT][KA][8];
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      const int col = (t0 + t) * 16 + c16, vp = col >> 1, v = vp >> g.lg, p = vp - (v << g.lg);
      if (t0 + t >= ctiles) break;
      const bool live = col < cols && p < np;
      const float2* s = in + p0 + (live ? p + (unsigned)v * g.P : 0u);
#pragma unroll
      for (int k = 0; k < KA; ++k)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          // even lanes row +u, odd lanes row -u.  Rows past r_h repeat it (their
          // table entries are zero); -0 and the -u of a Nyquist row are zero.
          const int u = min(32 * k + 8 * g4 + e, g.r_h);
          const int slot = odd && u > 0 ? g.R - u : u;
          const float2* q = s + (unsigned)slot * g.VP;
          float2 z = *q;
          if constexpr (PARTS)
            for (unsigned i = 1; i < g.nsplit; ++i) z = cadd(z, q[(size_t)i * g.pstride]);
          const bool none = odd && (u == 0 || slot <= g.r_h);
          y[t][k][e] = none ? make_float2(0.f, 0.f) : z;
        }
    }
    Split8 bp[CT][KA], bm[CT][KA];
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int k = 0; k < KA; ++k) {
        if (t0 + t >= ctiles) break;
        float p[8], m[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float2 z = y[t][k][e];
          const float2 w = make_float2(pair_swap(z.x), pair_swap(z.y));
          // this column's part c of Y[u] + Y[-u], and of i (Y[u] - Y[-u]): the
          // real one takes -(Im Y[u] - Im Y[-u]), the imaginary one Re Y[u] - Re Y[-u]
          p[e] = (odd ? z.y : z.x) + (odd ? w.y : w.x);
          m[e] = (odd ? w.x : w.y) - (odd ? z.x : z.y);
        }
        bp[t][k] = split8(p);
        bm[t][k] = split8(m);
      }
    for (int n = 0; n < g.n1; ++n) {
      uintx4 ac[KA][3], as[KA][3];
#pragma unroll
      for (int k = 0; k < KA; ++k) {
        table_frag<KA>(g.t1, n, k, ac[k]);
        table_frag<KA>(g.t1, g.n1 + n, k, as[k]);
      }
#pragma unroll
      for (int t = 0; t < CT; ++t) {
        if (t0 + t >= ctiles) break;
        Acc16 d{};
#pragma unroll
        for (int k = 0; k < KA; ++k) {
          mma16(ac[k], bp[t][k].p, d);
          mma16(as[k], bm[t][k].p, d);
        }
        const int col = (t0 + t) * 16 + c16, vp = col >> 1, v = vp >> g.lg, p = vp - (v << g.lg);
        if (col < cols && p < np) {
          float* o = sm + p * g.S2 + 2 * v + (col & 1);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = n * 16 + 4 * g4 + r;
            if (i < g.H) o[i * g.S1] = d.hi[r] + d.lo[r];
          }
        }
      }
    }
  }
  __syncthreads();
  const int rows = np * g.H, tiles = (rows + 15) / 16;
  float* dst = out + (size_t)p0 * g.H * g.W;
  for (int t0 = wave * RT; t0 < tiles; t0 += kWaves * RT) {
    Split8 b[RT][KB];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int row = (t0 + t) * 16 + c16;
      const bool live = row < rows;
      const int p = live ? div_magic(row, g.H, g.magic) : 0, i = live ? row - p * g.H : 0;
      if (t0 + t >= tiles) break;
      const float* z = sm + p * g.S2 + i * g.S1;
      const int last = (2 * g.V - 1) & ~3;
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const int q = 32 * k + 8 * g4;
        float w[8];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const floatx4 f = *reinterpret_cast<const floatx4*>(z + min(q + 4 * h, last));
#pragma unroll
          for (int e = 0; e < 4; ++e) w[4 * h + e] = f[e];
        }
        if (g.V % 2 != 0) {
#pragma unroll
          for (int e = 0; e < 8; ++e) w[e] = q + e < 2 * g.V ? w[e] : 0.f;
        }
        b[t][k] = split8(w);
      }
    }
    for (int n = 0; n < g.n2; ++n) {
      uintx4 a[KB][3];
#pragma unroll
      for (int k = 0; k < KB; ++k) table_frag<KB>(g.t2, n, k, a[k]);
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        if (t0 + t >= tiles) break;
        Acc16 d{};
#pragma unroll
        for (int k = 0; k < KB; ++k) mma16(a[k], b[t][k].p, d);
        const int row = (t0 + t) * 16 + c16, j = n * 16 + 4 * g4;
        if (row < rows) {
          float* o = dst + (size_t)row * g.W + j;
          const floatx4 v = d.hi + d.lo;
          if (j + 4 <= g.W) {
            *reinterpret_cast<floatx4u*>(o) = v;
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (j + r < g.W) o[r] = v[r];
          }
        }
      }
    }
  }
}

template <int KA, int KB, bool PARTS>
__global__ __launch_bounds__(kThreads) void k_mdft_inv(const float2* __restrict__ in, float* __restrict__ out,
                                                       MdftArgs g) {
  extern __shared__ __align__(16) float smf[];
  mdft_inv_block<KA, KB, PARTS>(in, out, g, blockIdx.x, gridDim.x, smf);
}

// ---- tables and geometry ------------------------------------------------------
struct MdftTable {
  int H, W, oi, oj;  // samples and their place on the grid
  int Lh, Lw, r_h, V;
  int ka, kb;        // steps of 32 of the two products
  int n1, n2;        // row tiles of the two operands (both of the cosine and sine operand's sets)
  double scale;      // inverse: 1 / (Lh Lw)
};

// The root tables of the two products as MFMA operands [tile][k step][part]
// [lane][8], in double precision before the split; one thread per (tile, step,
// lane, k of eight).  Forward: Ew, then C and S of the kept rows; inverse: C and S of the
// output rows, then the weighted column roots.
template <bool INV>
__global__ __launch_bounds__(256) void k_mdft_table(unsigned short* __restrict__ out, MdftTable g) {
  const int id = blockIdx.x * 256 + threadIdx.x, e = id & 7, lane = id >> 3 & 63, first = g.n1 * g.ka;
  int ts = id >> 9;  // tile and step
  if (ts >= first + g.n2 * g.kb) return;
  out += (size_t)ts * 1536 + lane * 8 + e;
  const bool one = ts < first;
  if (!one) ts -= first;
  const int steps = one ? g.ka : g.kb, row = (ts / steps) * 16 + (lane & 15);
  const int k = (ts % steps) * 32 + 8 * (lane >> 4) + e;
  auto turn = [](int m, int L, bool sine) {  // cos or sin of 2 pi m / L
    double c, s;
    sincospi(2.0 * (m % L) / L, &s, &c);
    return sine ? s : c;
  };
  double v = 0.0;
  if (one == INV) {  // cosines and sines along the columns of the grid
    const int half = (one ? g.n1 : g.n2) / 2 * 16;  // the sines' first row
    const int r = row < half ? row : row - half, u = INV ? k : r, i = INV ? r : k;
    if (u <= g.r_h && i < g.H) v = turn(u * (i + g.oi), g.Lh, row >= half);
  } else if constexpr (!INV) {  // x[j] e^{-2 pi i w (j + oj) / Lw}
    const int w = row >> 1;
    if (w < g.V && k < g.W) v = (row & 1) ? -turn(w * (k + g.oj), g.Lw, true) : turn(w * (k + g.oj), g.Lw, false);
  } else {  // h_w Re((zr + i zi) e^{+2 pi i w (j + cj) / Lw})
    const int w = k >> 1;
    const bool real = w == 0 || 2 * w == g.Lw;
    if (row < g.W && w < g.V && !(real && (k & 1))) {
      const double t = turn(w * (row + g.oj), g.Lw, k & 1);
      v = g.scale * (real ? 1.0 : 2.0) * ((k & 1) ? -t : t);
    }
  }
  split3_store(v, out, 512);
}

template <bool INV>
bl_status_t mdft_table(const bl_conv_plan_s* p, const MdftTable& t, const float2** tab, hipStream_t s) {
  const std::vector<long> key{INV ? 5 : 4, p->Lh, p->Lw, p->r_h, p->V, t.H, t.W, t.oi, t.oj};
  const int n = t.n1 * t.ka + t.n2 * t.kb;  // of 3 KB
  return plan_table_on_device(
      p, key, (size_t)n * 384,
      [&](float2* d) {
        hipLaunchKernelGGL((k_mdft_table<INV>), dim3((unsigned)(2 * n)), dim3(256), 0, s,
                           reinterpret_cast<unsigned short*>(d), t);
      },
      tab, s);
}

int steps32(int n) { return (n + 31) / 32; }
int steps_of(int s) { return s <= 1 ? 1 : s == 2 ? 2 : s <= 4 ? 4 : 0; }  // as instantiated; 0: none
// a multiple of 4 floats, an odd number of 16-byte groups: the operands'
// 16-byte reads of 16 columns or rows then fall on all banks
int odd_groups(int n) { return ((n + 3) / 4 | 1) * 4; }

unsigned magic_of(unsigned d) { return d > 1 ? (unsigned)((0x100000000ull + d - 1) / d) : 0u; }

struct MdftSetup {
  MdftArgs g;
  int ka, kb;
  long blocks;
  size_t lds;
  double bytes, flops;
};

// Planes per block: about 256 rows, in LDS of at most 40 KB (80 KB where 8
// planes, a 64-byte run of a bin row, need that, 160 KB where one does).
template <class F>
int planes_for(int H, long P, F&& lds) {
  int G = 8;
  while (G < 64 && 2 * G * H <= 256) G *= 2;
  while (G > 8 && lds(G) > 40 * 1024) G /= 2;
  while (G > 1 && lds(G) > 80 * 1024) G /= 2;
  // few planes: fewer per block, while that fills more compute units
  while (G > 1 && (P + G - 1) / G < 256 && (P + G / 2 - 1) / (G / 2) <= 512) G /= 2;
  return G;
}

double fft_flops(const bl_conv_plan_s* p, long P, int H) {
  const double LH = p->Lh, LW = p->Lw;
  return (double)P * (H * 2.5 * LW * std::log2(std::max(2.0, LW)) + p->V * 5.0 * LH * std::log2(std::max(2.0, LH)));
}

bl_status_t mdft_fwd_setup(const bl_conv_plan_s* p, long P, int H, int W, int oi, int oj, MdftSetup& f,
                           hipStream_t s) {
  f.ka = steps_of(steps32(W)), f.kb = steps_of(steps32(H));
  if (!f.ka || !f.kb || (double)p->kept * P >= 2147483647.0) return BL_ERR_UNSUPPORTED;
  MdftArgs& g = f.g;
  g = MdftArgs{};
  g.H = H, g.W = W, g.r_h = p->r_h, g.R = p->R, g.V = p->V, g.P = (unsigned)P;
  g.S1 = odd_groups(H);
  auto v_stride = [&](int G) { return 2 * G * g.S1 + 8; };
  auto lds = [&](int G) { return (size_t)g.V * v_stride(G) * sizeof(float); };
  const int G = planes_for(H, P, lds);
  g.S2 = v_stride(G);
  f.lds = lds(G);
  if (f.lds > 160 * 1024) return BL_ERR_UNSUPPORTED;
  g.n1 = (2 * p->V + 15) / 16, g.m2 = (p->r_h + 16) / 16;
  g.magic = magic_of((unsigned)H);
  const int run = G * (p->bf16 ? 4 : 8);
  g.K = run < 64 ? (unsigned)(128 / run) : 1u;
  const float2* tab;
  const bl_status_t st = mdft_table<false>(
      p, MdftTable{H, W, oi, oj, p->Lh, p->Lw, p->r_h, p->V, f.ka, f.kb, g.n1, 2 * g.m2, 1.0}, &tab, s);
  if (st != BL_OK) return st == BL_ERR_OOM ? BL_ERR_UNSUPPORTED : st;  // the direct DFT needs no table
  g.t1 = reinterpret_cast<const uintx4*>(tab);
  g.t2 = g.t1 + (size_t)g.n1 * f.ka * 192;
  f.blocks = (P + G - 1) / G;
  while (1 << g.lg < G) ++g.lg;
  g.VP = (unsigned)(p->V * P);
  f.bytes = (double)P * H * W * 4 + (double)P * p->kept * (p->bf16 ? 4 : 8);
  f.flops = fft_flops(p, P, H);
  return BL_OK;
}

bl_status_t mdft_inv_setup(const bl_conv_plan_s* p, long P, int OH, int OW, int ci, int cj, int nsplit, size_t pstride,
                           MdftSetup& f, hipStream_t s) {
  f.ka = steps_of(steps32(p->r_h + 1)), f.kb = steps_of(steps32(2 * p->V));
  if (!f.ka || f.ka > 2 || !f.kb || (double)p->kept * P >= 2147483647.0) return BL_ERR_UNSUPPORTED;
  MdftArgs& g = f.g;
  g = MdftArgs{};
  g.H = OH, g.W = OW, g.r_h = p->r_h, g.R = p->R, g.V = p->V, g.P = (unsigned)P;
  g.nsplit = (unsigned)std::max(1, nsplit), g.pstride = pstride;
  g.S1 = odd_groups(2 * p->V);
  // planes 4 (mod 64) floats apart: with rows of an odd number of 16-byte
  // groups the first product's stores hit two lanes a bank at most
  g.S2 = (OH * g.S1 + 63) / 64 * 64 + 4;
  auto lds = [&](int G) { return (size_t)G * g.S2 * sizeof(float); };
  const int G = planes_for(OH, P, lds);
  f.lds = lds(G);
  if (f.lds > 160 * 1024) return BL_ERR_UNSUPPORTED;
  g.n1 = (OH + 15) / 16, g.n2 = (OW + 15) / 16;
  g.magic = magic_of((unsigned)OH);
  g.K = G * 8 < 128 ? (unsigned)(128 / (G * 8)) : 1u;
  const float2* tab;
  const bl_status_t st = mdft_table<true>(p, MdftTable{OH, OW, ci, cj, p->Lh, p->Lw, p->r_h, p->V, f.ka, f.kb, 2 * g.n1, g.n2,
                                                       1.0 / ((double)p->Lh * (double)p->Lw)}, &tab, s);
  if (st != BL_OK) return st == BL_ERR_OOM ? BL_ERR_UNSUPPORTED : st;  // the direct DFT needs no table
  g.t1 = reinterpret_cast<const uintx4*>(tab);
  g.t2 = g.t1 + (size_t)2 * g.n1 * f.ka * 192;
  f.blocks = (P + G - 1) / G;
  while (1 << g.lg < G) ++g.lg;
  g.VP = (unsigned)(p->V * P);
  f.bytes = (double)P * p->kept * 8 * g.nsplit + (double)P * OH * OW * 4;
  f.flops = fft_flops(p, P, OH);
  return BL_OK;
}

template <class K, class... A>
bl_status_t mdft_go(K kern, const char* name, long blocks, size_t lds, double bytes, double flops, hipStream_t s,
                    A... args) {
  if (lds > kMaxLds) {
    const bl_status_t at = lds_opt_in(reinterpret_cast<const void*>(kern), 160 * 1024);
    if (at != BL_OK) return at;
  }
  return timed_launch(name, bytes, flops, s, [&](hipEvent_t e0, hipEvent_t e1) {
    hipExtLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kThreads), lds, s, e0, e1, 0, args...);
  });
}

}  // namespace

bl_status_t launch_mdft_fwd(const bl_conv_plan_s* p, const float* in, void* out, long P, int Hin, int Win, int oi,
                            int oj, hipStream_t s) {
  MdftSetup f;
  const bl_status_t st = mdft_fwd_setup(p, P, Hin, Win, oi, oj, f, s);
  if (st != BL_OK) return st;
#define X(a, b)                                                                                                  \
  if (f.ka == a && f.kb == b)                                                                                    \
    return p->bf16 ? mdft_go(k_mdft_fwd<a, b, unsigned>, "spec_fwd_2d", f.blocks, f.lds, f.bytes, f.flops, s, in, \
                             static_cast<unsigned*>(out), f.g)                                                    \
                   : mdft_go(k_mdft_fwd<a, b, float2>, "spec_fwd_2d", f.blocks, f.lds, f.bytes, f.flops, s, in,   \
                             static_cast<float2*>(out), f.g);
  X(1, 1) X(1, 2) X(1, 4) X(2, 1) X(2, 2) X(2, 4) X(4, 1) X(4, 2) X(4, 4)
#undef X
  return BL_ERR_UNSUPPORTED;
}

bl_status_t launch_mdft_inv(const bl_conv_plan_s* p, const float2* in, float* out, long P, int OH, int OW, int ci,
                            int cj, hipStream_t s, int nsplit, size_t pstride) {
  MdftSetup f;
  const bl_status_t st = mdft_inv_setup(p, P, OH, OW, ci, cj, nsplit, pstride, f, s);
  if (st != BL_OK) return st;
#define X(a, b, parts)                                 \
  if (f.ka == a && f.kb == b && parts == (f.g.nsplit > 1)) \
    return mdft_go(k_mdft_inv<a, b, parts>, "spec_inv_2d", f.blocks, f.lds, f.bytes, f.flops, s, in, out, f.g);
  X(1, 1, false) X(1, 2, false) X(1, 4, false) X(2, 1, false) X(2, 2, false) X(2, 4, false)
  // (more than 32 row frequencies by 16 columns are at least 1088 bins: too many for a contraction to be split)
  X(1, 1, true) X(1, 2, true) X(1, 4, true) X(2, 1, true)
#undef X
  return BL_ERR_UNSUPPORTED;
}

}  // namespace blc
