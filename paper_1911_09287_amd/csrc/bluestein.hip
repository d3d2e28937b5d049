// 1-D kept spectra by Bluestein's chirp-z identity (gfx950).
//
// A length-L DFT evaluated only at n_out consecutive outputs from n_in
// consecutive inputs is a linear convolution with a chirp: with
// c[m] = exp(-i pi m^2 / L) and nk = (n^2 + k^2 - (k - n)^2) / 2,
//   sum_n a[n] exp(-2 pi i n k / L) = c[k] sum_n (a[n] c[n]) conj(c[k - n]).
// The convolution is done as a circular one over an FFT of 1024 >= n_in + n_out
// - 1 points, so no wrap-around reaches the kept outputs.  This serves any
// sequence length (the FCN layers of the time-series experiments use 519 =
// 3 * 173, 516 and 514 = 2 * 257 points, where a mixed-radix FFT would need 173-
// and 257-point stages); shorter and fewer series take a matrix product.
//
// Forward (real rows -> kept bins, Sec. 3.2.2: only v <= r_w is produced):
//   pre[j] = c[j + oj], filter[d] = conj(c[d - oj]), X[v] = c[v] * conv[v].
// Inverse (kept bins -> real rows, Hermitian weights h_v, crop offset cj):
//   pre[v] = h_v conj(c[v]), filter[d] = c[d + cj],
//   y[j] = Re(conj(c[j + cj]) * conv[j]) / L.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <new>
#include <vector>

#include "common.hpp"

namespace blc {
namespace {

// e^{-2 pi i k / 32}, k < 16.
constexpr float kW32c[16] = {1.0f, 0.98078528040323043f, 0.92387953251128674f, 0.83146961230254524f,
                             0.70710678118654757f, 0.55557023301960218f, 0.38268343236508984f, 0.19509032201612833f,
                             0.0f, -0.19509032201612819f, -0.38268343236508973f, -0.55557023301960196f,
                             -0.70710678118654746f, -0.83146961230254535f, -0.92387953251128674f,
                             -0.98078528040323043f};
constexpr float kW32s[16] = {0.0f, -0.19509032201612825f, -0.38268343236508978f, -0.55557023301960218f,
                             -0.70710678118654746f, -0.83146961230254524f, -0.92387953251128674f,
                             -0.98078528040323043f, -1.0f, -0.98078528040323043f, -0.92387953251128674f,
                             -0.83146961230254546f, -0.70710678118654757f, -0.55557023301960218f,
                             -0.38268343236508989f, -0.19509032201612861f};

// In-register R-point DFT (natural order in and out), radix-2 decimation in
// time, R <= 32.  A butterfly with a general twiddle w forms e + w o with four
// fused multiply-adds and takes the difference as 2 e - (e + w o), one more
// each (6 instructions instead of 4 for w o and 4 for the sum and difference).
template <int R>
struct RegFft {
  static __device__ __forceinline__ void run(float2* v) {
    float2 e[R / 2], o[R / 2];
#pragma unroll
    for (int k = 0; k < R / 2; ++k) {
      e[k] = v[2 * k];
      o[k] = v[2 * k + 1];
    }
    RegFft<R / 2>::run(e);
    RegFft<R / 2>::run(o);
#pragma unroll
    for (int k = 0; k < R / 2; ++k) {
      if (k == 0) {
        v[k] = cadd(e[k], o[k]);
        v[k + R / 2] = csub(e[k], o[k]);
      } else if (4 * k == R) {  // w = -i
        v[k] = make_float2(e[k].x + o[k].y, e[k].y - o[k].x);
        v[k + R / 2] = make_float2(e[k].x - o[k].y, e[k].y + o[k].x);
      } else {
        const float c = kW32c[k * (32 / R)], sn = kW32s[k * (32 / R)];
        const float2 x = make_float2(fmaf(o[k].x, c, fmaf(-o[k].y, sn, e[k].x)),
                                     fmaf(o[k].x, sn, fmaf(o[k].y, c, e[k].y)));
        v[k] = x;
        v[k + R / 2] = make_float2(fmaf(2.f, e[k].x, -x.x), fmaf(2.f, e[k].y, -x.y));
      }
    }
  }
};
template <>
struct RegFft<1> {
  static __device__ __forceinline__ void run(float2*) {}
};

struct BlueGeom {
  int n_in, n_out;     // inputs and outputs of the chirp convolution per FFT
  int L;               // DFT length
  int V;               // kept bins per series
  int off_in, off_out; // DFT index of input 0 and of output 0
  int nyq;             // Nyquist bin (L even) or -1
  long P;              // number of series
  float out_scale;     // extra output scale (inverse: 1 / L)
  const float2* tab;   // 1024-point kernel: [pre n_in][post n_out][F 1024][TW 1024]
};
// Modes: bit 0 = inverse (bins -> real rows), bit 1 = two series per FFT.
//   forward, single:  inputs x[0..Win), outputs X[0..V)
//   inverse, single:  inputs h_v Y[v], v < V; outputs y[0..OW)
//   forward, paired:  input x1 + i x2; outputs Z[k], k = -(V-1)..V-1, then
//                     X1 = (Z[k] + conj Z[-k]) / 2, X2 = (Z[k] - conj Z[-k]) / 2i
//                     (both spectra of real rows are conjugate-symmetric)
//   inverse, paired:  input the conjugate-symmetric extensions of Y1 and Y2
//                     over k = -(V-1)..V-1 as Y1 + i Y2 (real DC parts); the
//                     real and imaginary parts of the result are y1 and y2.
// S: stored-spectrum element of the forward modes' output (float2 or bfloat16 pairs)
// ---------------------------------------------------------------------------
// M = 1024 as 32 x 32 per half-wave: with n = l + 32 j and k' = k + 32 m,
//   X[k + 32 m] = sum_l w32^{lm} [w1024^{lk} sum_j x[l + 32 j] w32^{jk}],
// lane l of a half-wave runs the inner 32-point FFT over j in registers, the
// twiddled results cross lanes once through LDS (a 32 x 33 transpose), and
// lane k runs the outer 32-point FFT over l, ending with X[k + 32 m] in its
// registers.  That is exactly the layout the second FFT's inner pass needs
// (lane k holding element k + 32 m), so the pointwise product with the filter
// spectrum needs no extra transpose: each Bluestein job costs one LDS
// transpose per FFT instead of a pass per radix stage.
//
// Every wave runs its own jobs, with no block barrier once the tables are in
// LDS: half-wave q of the wave with grid-wide index p takes job 2 p + q, then
// job 2 (p + W) + q for W waves in the grid, and so on.  A wave's jobs are two
// consecutive series (four in the paired modes), and the waves of a block
// hold consecutive jobs, so the rows of a bin-major spectrum are read and
// written in runs of consecutive series that meet in the L2.  A wave loads its
// inputs (the next round's while it transforms the current one, when they fit
// in 32 registers per lane), transforms and stores, and the waves of a CU fall
// into different phases, overlapping memory traffic with arithmetic.
// Inputs and outputs that run along the series (real samples) move straight
// between HBM and registers; bin-major spectra pass through the wave's slot
// buffers in LDS, where the conjugate-symmetric pairs of the paired modes are
// formed or split.
// ---------------------------------------------------------------------------
constexpr int kWaves1k = 8;
// Slot stride (complex): the 32 x 33 transpose tile plus 4 elements.
constexpr int kXS = 32 * 33 + 4;

// Rows of input one lane loads per round (NR, a compile-time bound; loads past
// the data are clamped to its last row and their values unused):
//   MODE 0, 2: rows j of the series, element h + 32 j;
//   MODE 1, 3: bins k = lane / 2 + 32 t, t < NR.
// Floats per row: 1 (MODE 0), 2 (MODE 1, 2), 4 (MODE 3).  The next round is
// prefetched when NR rows take at most 32 floats.
template <int MODE>
constexpr int floats_per_row() {
  return MODE == 0 ? 1 : MODE == 3 ? 4 : 2;
}

template <int MODE, int NR, typename S = float2>
__global__ __launch_bounds__(64 * kWaves1k) void k_bluestein1k(const void* __restrict__ in_, void* __restrict__ out_,
                                                               BlueGeom a, int wpb) {
  constexpr int M = 1024;
  constexpr bool PACK = MODE >= 2;
  constexpr int FPR = floats_per_row<MODE>();
  constexpr bool PREF = NR * FPR <= 32;
  extern __shared__ float2 sm[];
  float2* bufs = sm;                          // 16 slots x kXS
  float2* pre = bufs + 2 * kWaves1k * kXS;    // n_in
  float2* post = pre + a.n_in;                // n_out
  float2* F = post + a.n_out;                 // spectrum of the chirp filter (M)
  float2* TW = F + M;                         // TW[32 k + h] = w1024^{h k}
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int q = lane >> 5, h = lane & 31;
  float2* xw = bufs + wave * 2 * kXS;  // the wave's two slot buffers
  float2* xb = xw + q * kXS;           // this half-wave's

  // the chirps, the filter's spectrum and the twiddles, built once per plan
  // in double precision on the host, are laid out in the table as in LDS
  // (all of a thread's table loads in flight together, and with the first
  // round's input loads: n_in + n_out <= M + 1)
  constexpr int NT = 64 * kWaves1k;
  constexpr int NTAB = (3 * M + 1 + NT - 1) / NT;
  const int ntab = a.n_in + a.n_out + 2 * M;
  float2 tv[NTAB];
#pragma unroll
  for (int u = 0; u < NTAB; ++u) tv[u] = a.tab[min(tid + NT * u, ntab - 1)];

  auto exchange = [&](float2* v) {
#pragma unroll
    for (int k = 0; k < 32; ++k) xb[k * 33 + h] = v[k];
    wave_sync();
#pragma unroll
    for (int l = 0; l < 32; ++l) v[l] = xb[h * 33 + l];
    wave_sync();
  };
  // inner FFT over j (input v[j] = element h + 32 j), twiddle, transpose, outer FFT:
  // leaves v[m] = element h + 32 m of the transform.
  auto fft1k = [&](float2* v) {
    RegFft<32>::run(v);
#pragma unroll
    for (int k = 1; k < 32; ++k) v[k] = cmul(v[k], TW[32 * k + h]);
    exchange(v);
    RegFft<32>::run(v);
  };

  // element indices fit in 32 bits (checked on the host)
  const float* xin = static_cast<const float*>(in_);
  const float2* yin = static_cast<const float2*>(in_);
  const unsigned P = (unsigned)a.P;
  const unsigned jobs = PACK ? (P + 1) / 2 : P;
  const unsigned pairs = (jobs + 1) / 2;  // rounds of the grid's waves: one job pair each
  // waves past the first wpb of a block only help with the tables
  const unsigned nw = gridDim.x * (unsigned)wpb;
  const unsigned p0 = wave < wpb ? blockIdx.x * (unsigned)wpb + wave : pairs;
  // series of the wave in round p: MODE 0/1: 2p + q; MODE 2/3: 4p .. 4p + 3
  float pf[PREF ? NR * FPR : 1];
  float2 v[32];
  auto load = [&](unsigned p, float* dst) {
    if constexpr (MODE == 0) {
      const unsigned s = min(2 * p + q, P - 1);
#pragma unroll
      for (int j = 0; j < NR; ++j) dst[j] = xin[s * (unsigned)a.n_in + min(h + 32 * j, a.n_in - 1)];
    } else if constexpr (MODE == 2) {
      const unsigned s1 = min(4 * p + 2 * q, P - 1), s2 = min(4 * p + 2 * q + 1, P - 1);
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        const int n = min(h + 32 * j, a.n_in - 1);
        dst[2 * j] = xin[s1 * (unsigned)a.n_in + n];
        dst[2 * j + 1] = xin[s2 * (unsigned)a.n_in + n];
      }
    } else if constexpr (MODE == 1) {
      const unsigned s = min(2 * p + (lane & 1), P - 1);
#pragma unroll
      for (int t = 0; t < NR; ++t) {
        const float2 y = yin[(unsigned)min((lane >> 1) + 32 * t, a.V - 1) * P + s];
        dst[2 * t] = y.x;
        dst[2 * t + 1] = y.y;
      }
    } else {
      const unsigned s1 = min(4 * p + 2 * (lane & 1), P - 1), s2 = min(4 * p + 2 * (lane & 1) + 1, P - 1);
#pragma unroll
      for (int t = 0; t < NR; ++t) {
        const unsigned k = (unsigned)min((lane >> 1) + 32 * t, a.V - 1);
        const float2 y1 = yin[k * P + s1], y2 = yin[k * P + s2];
        dst[4 * t] = y1.x;
        dst[4 * t + 1] = y1.y;
        dst[4 * t + 2] = y2.x;
        dst[4 * t + 3] = y2.y;
      }
    }
  };
  // loaded rows -> v (element h + 32 j of this half-wave's job), times the pre-chirp
  auto stage = [&](unsigned p, const float* src) {
    if constexpr (MODE == 0 || MODE == 2) {
      const bool two = MODE == 2 && 4 * p + 2 * q + 1 < P;
      const int jfull = a.n_in >> 5;  // rows complete for every lane (uniform branch)
      const bool tail = h < (a.n_in & 31);
#pragma unroll
      for (int j = 0; j < 32; ++j) {
        v[j] = make_float2(0.f, 0.f);
        if (j < NR && (j < jfull || (j == jfull && tail))) {
          const float2 z = MODE == 0 ? make_float2(src[j], 0.f) : make_float2(src[2 * j], two ? src[2 * j + 1] : 0.f);
          v[j] = cmul(z, pre[h + 32 * j]);
        }
      }
    } else {
      float2* dst = xw + (lane & 1) * kXS;
#pragma unroll
      for (int t = 0; t < NR; ++t) {
        const int k = (lane >> 1) + 32 * t;
        if (k < a.V) {
          if constexpr (MODE == 1) {
            dst[k] = cmul(make_float2(src[2 * t], src[2 * t + 1]), pre[k]);
          } else {
            // two Hermitian spectra packed into one series: Z[k] = Y1[k] + i Y2[k]
            // at index k + V - 1 for |k| < V, with Y[-k] = conj(Y[k])
            const bool two = 4 * p + 2 * (lane & 1) + 1 < P;
            const float2 y1 = make_float2(src[4 * t], src[4 * t + 1]);
            const float2 y2 = two ? make_float2(src[4 * t + 2], src[4 * t + 3]) : make_float2(0.f, 0.f);
            const int ip = a.V - 1 + k, im = a.V - 1 - k;
            if (k == 0) {
              dst[ip] = cmul(make_float2(y1.x, y2.x), pre[ip]);
            } else {
              dst[ip] = cmul(make_float2(y1.x - y2.y, y1.y + y2.x), pre[ip]);
              dst[im] = cmul(make_float2(y1.x + y2.y, y2.x - y1.y), pre[im]);
            }
          }
        }
      }
      wave_sync();
#pragma unroll
      for (int j = 0; j < 32; ++j) {
        const int n = h + 32 * j;
        v[j] = n < a.n_in ? xb[n] : make_float2(0.f, 0.f);
      }
      wave_sync();
    }
  };

  if constexpr (PREF) load(min(p0, pairs - 1), pf);  // clamped: no branch between these loads and the table's
  // (indices past the table are clamped like the loads: those threads store
  // the last entry's own value again, so the stores need no branch)
#pragma unroll
  for (int u = 0; u < NTAB; ++u) pre[min(tid + NT * u, ntab - 1)] = tv[u];
  __syncthreads();  // tables in LDS; no block barrier follows

  for (unsigned p = p0; p < pairs; p += nw) {
    if constexpr (PREF) {
      stage(p, pf);
      load(p + nw < pairs ? p + nw : p, pf);  // the last round reloads its own rows (cache hits)
    } else {
      float ld[NR * FPR];
      load(p, ld);
      stage(p, ld);
    }
    fft1k(v);
    // inverse FFT of (A * F) as conj(FFT(conj(A * F)))
#pragma unroll
    for (int m = 0; m < 32; ++m) v[m] = cconj(cmul(v[m], F[h + 32 * m]));
    fft1k(v);
    // v[m] -> output element i = h + 32 m: post[i] conj(v[m])
    // rows m < nfull are complete for every lane (a uniform branch); row
    // nfull is partial
    const int nfull = a.n_out >> 5;
    const bool tail = h < (a.n_out & 31);
    if constexpr (MODE == 1) {
      const unsigned s = 2 * p + q;
      if (s < P) {
        float* dst = static_cast<float*>(out_) + s * (unsigned)a.n_out + h;
#pragma unroll
        for (int m = 0; m < 32; ++m) {
          if (m < nfull || (m == nfull && tail)) dst[32 * m] = cmul(post[h + 32 * m], cconj(v[m])).x;
        }
      }
    } else if constexpr (MODE == 3) {
      const unsigned s1 = 4 * p + 2 * q;
      const bool two = s1 + 1 < P;
      float* d1 = static_cast<float*>(out_) + s1 * (unsigned)a.n_out + h;
      float* d2 = d1 + a.n_out;
      if (two) {
#pragma unroll
        for (int m = 0; m < 32; ++m) {
          if (m < nfull || (m == nfull && tail)) {
            const float2 r = cmul(post[h + 32 * m], cconj(v[m]));
            d1[32 * m] = r.x;
            d2[32 * m] = r.y;
          }
        }
      } else if (s1 < P) {  // a lone last series
#pragma unroll
        for (int m = 0; m < 32; ++m) {
          if (m < nfull || (m == nfull && tail)) d1[32 * m] = cmul(post[h + 32 * m], cconj(v[m])).x;
        }
      }
    } else {
#pragma unroll
      for (int m = 0; m < 32; ++m) {
        if (m < nfull || (m == nfull && tail)) xb[h + 32 * m] = cmul(post[h + 32 * m], cconj(v[m]));
      }
      wave_sync();
      S* X = static_cast<S*>(out_);
      if constexpr (MODE == 0) {
        // bins i of the wave's two series, two consecutive series per bin row
        const unsigned s = 2 * p + (lane & 1);
        const float2* src = xw + (lane & 1) * kXS;
        if (s < P) {
          for (int i = lane >> 1; i < a.n_out; i += 32) spec_put(X, (unsigned)i * P + s, src[i]);
        }
      } else {
        // Z[k] sits at index k + V - 1; the two series of a job split by
        // conjugate symmetry; four consecutive series per bin row
        const unsigned s = 4 * p + (lane & 3);
        const float2* src = xw + ((lane >> 1) & 1) * kXS + (a.V - 1);
        if (s < P) {
          for (int k = lane >> 2; k < a.V; k += 16) {
            const float2 zp = src[k], zm = cconj(src[-k]);
            spec_put(X, (unsigned)k * P + s, (lane & 1) ? make_float2(zp.y - zm.y, zm.x - zp.x) : cadd(zp, zm));
          }
        }
      }
      wave_sync();  // slot buffers free for the next round's transposes
    }
  }
}

// ---- tables of the 1024-point kernel, built on the host in double precision ----
// For one transform geometry: pre[n] (n < n_in), post[k] (k < n_out), the
// spectrum F of the chirp filter, and the twiddles TW[32 k + h] = w^{h k}, in
// that order, as the kernel lays them out in LDS.
void host_tables_1k(const BlueGeom& a, int mode, std::vector<float2>& out) {
  constexpr int M = 1024;
  const bool inv = mode & 1, pack = mode >= 2;
  const double pi = 3.141592653589793238462643383279502884;
  auto chirp = [&](long m, double& re, double& im) {  // e^{-i pi m^2 / L}, conjugated for the inverse
    const long mm = m < 0 ? -m : m;
    const long q = (mm * mm) % (2L * a.L);
    re = std::cos(pi * (double)q / a.L);
    im = -std::sin(pi * (double)q / a.L);
    if (inv) im = -im;
  };
  out.assign((size_t)a.n_in + a.n_out + 2 * M, make_float2(0.f, 0.f));
  double re, im;
  for (int k = 0; k < a.n_in; ++k) {
    chirp(k + a.off_in, re, im);
    const double w = (inv && !pack && k != 0 && k != a.nyq) ? 2.0 : 1.0;
    out[k] = make_float2((float)(w * re), (float)(w * im));
  }
  const double osc = (double)a.out_scale / M * (pack && !inv ? 0.5 : 1.0);
  for (int k = 0; k < a.n_out; ++k) {
    chirp(k + a.off_out, re, im);
    out[a.n_in + k] = make_float2((float)(osc * re), (float)(osc * im));
  }
  // filter b[m] = conj(c[d + off_out - off_in]) for lags d in (-n_in, n_out),
  // d = m or m - M; its M-point DFT by iterative radix-2 in double
  std::vector<double> br(M, 0.0), bi(M, 0.0);
  for (int m = 0; m < M; ++m) {
    const int d = m < a.n_out ? m : m - M;
    if (d >= -(a.n_in - 1)) {
      chirp((long)d + a.off_out - a.off_in, re, im);
      br[m] = re;
      bi[m] = -im;
    }
  }
  for (int i = 1, j = 0; i < M; ++i) {  // bit reversal
    int bit = M >> 1;
    for (; j & bit; bit >>= 1) j ^= bit;
    j ^= bit;
    if (i < j) std::swap(br[i], br[j]), std::swap(bi[i], bi[j]);
  }
  for (int len = 2; len <= M; len <<= 1) {
    for (int i = 0; i < M; i += len) {
      for (int k = 0; k < len / 2; ++k) {
        const double t = -2.0 * pi * k / len, wr = std::cos(t), wi = std::sin(t);
        const int u = i + k, v = i + k + len / 2;
        const double xr = br[v] * wr - bi[v] * wi, xi = br[v] * wi + bi[v] * wr;
        br[v] = br[u] - xr; bi[v] = bi[u] - xi;
        br[u] += xr; bi[u] += xi;
      }
    }
  }
  float2* F = out.data() + a.n_in + a.n_out;
  for (int m = 0; m < M; ++m) F[m] = make_float2((float)br[m], (float)bi[m]);
  float2* TW = F + M;
  for (int i = 0; i < M; ++i) {
    const int e = ((i >> 5) * (i & 31)) & (M - 1);
    TW[i] = make_float2((float)std::cos(2.0 * pi * e / M), (float)-std::sin(2.0 * pi * e / M));
  }
}

// Device copy of the tables for this geometry (built and uploaded on first use).
bl_status_t blue_tables(const bl_conv_plan_s* p, const BlueGeom& a, int mode, const float2** out, hipStream_t s) {
  const std::vector<long> key{1, mode, a.n_in, a.n_out, a.off_in, a.off_out, a.L, a.nyq, float_key(a.out_scale)};
  return plan_table(p, key, [&](std::vector<float2>& host) { host_tables_1k(a, mode, host); }, out, s);
}

template <int MODE, int NR, typename S>
bl_status_t launch_1k_nr(const BlueGeom& a, const void* in, void* out, const char* name, double bytes,
                         hipStream_t s) {
  constexpr int M = 1024;
  const size_t lds = (size_t)(2 * kWaves1k * kXS + a.n_in + a.n_out + 2 * M) * sizeof(float2);
  if (lds > 160 * 1024) return BL_ERR_UNSUPPORTED;
  const bl_status_t at = lds_opt_in(reinterpret_cast<const void*>(&k_bluestein1k<MODE, NR, S>), 160 * 1024);
  if (at != BL_OK) return at;
  const long jobs = (MODE >= 2) ? (a.P + 1) / 2 : a.P;
  const long pairs = (jobs + 1) / 2;  // one job per half-wave
  // one block per CU at most; when there is less than a full block of work
  // per CU, fewer waves per block, so that the SIMDs are shared by fewer waves
  const long cus = device_cus();
  const int wpb = (int)std::min<long>(kWaves1k, (pairs + cus - 1) / cus);
  const long blocks = std::min<long>(cus, (pairs + wpb - 1) / wpb);
  const double flops = (double)jobs * 2.0 * 5.0 * M * 10.0;
  return timed_launch(name, bytes, flops, s, [&](hipEvent_t e0, hipEvent_t e1) {
    hipExtLaunchKernelGGL((k_bluestein1k<MODE, NR, S>), dim3((unsigned)blocks), dim3(64 * kWaves1k), lds, s, e0, e1, 0,
                          in, out, a, wpb);
  });
}

// NR: rows of input per lane as instantiated (the smallest that covers the
// data); the kernel prefetches the next round when they fit in 32 floats.
template <int MODE, typename S>
bl_status_t launch_1k(const bl_conv_plan_s* p, const BlueGeom& a0, const void* in, void* out, const char* name,
                      double bytes, hipStream_t s) {
  // the kernel indexes its input and output with 32-bit element offsets
  const long rows = std::max<long>({(long)a0.n_in, (long)a0.n_out, 2L * a0.V});
  if (a0.P < 1 || a0.P * rows >= 2147483647L || a0.P * rows < 0) return BL_ERR_UNSUPPORTED;
  BlueGeom a = a0;
  const bl_status_t ts = blue_tables(p, a, MODE, &a.tab, s);
  if (ts != BL_OK) return ts;
  if constexpr (MODE == 0 || MODE == 2) {
    const int nr = (a.n_in + 31) / 32;
    if (nr <= 16) return launch_1k_nr<MODE, 16, S>(a, in, out, name, bytes, s);
    return launch_1k_nr<MODE, 32, S>(a, in, out, name, bytes, s);
  } else {
    const int nr = (a.V + 31) / 32;
    if (nr <= 4) return launch_1k_nr<MODE, 4, S>(a, in, out, name, bytes, s);
    if (nr <= 8) return launch_1k_nr<MODE, 8, S>(a, in, out, name, bytes, s);
    if (nr <= 16) return launch_1k_nr<MODE, 16, S>(a, in, out, name, bytes, s);
    if constexpr (MODE == 1) return launch_1k_nr<MODE, 32, S>(a, in, out, name, bytes, s);
    return BL_ERR_UNSUPPORTED;
  }
}

// The chirp convolution takes an FFT of 1024 points and no fewer (shorter ones
// are slower than one matrix product), and whether two series share one (when
// the conjugate-symmetric output or input range fits it as well).
bool takes_1k(int L, int V, long P, int other, bool* pack) {
  const int points = V + other - 1;
  if (2 * L > 64 * 64 || points <= 512 || points > 1024) return false;
  if ((long)V * other < 2048) return false;  // a few bins: left to the matrix product
  *pack = P >= 2 && 2 * (V - 1) < L && points + V - 1 <= 1024;
  return true;
}

bl_status_t launch_any(const bl_conv_plan_s* p, BlueGeom& a, bool inv, int other, const void* in, void* out,
                       const char* name, double bytes, hipStream_t s) {
  bool pack = false;
  if (!takes_1k(a.L, a.V, a.P, other, &pack)) return BL_ERR_UNSUPPORTED;
  if (!inv) {
    a.n_in = other;
    if (pack) {
      a.n_out = 2 * a.V - 1;
      a.off_out = -(a.V - 1);
      return p->bf16 ? launch_1k<2, unsigned>(p, a, in, out, name, bytes, s)
                     : launch_1k<2, float2>(p, a, in, out, name, bytes, s);
    }
    a.n_out = a.V;
    a.off_out = 0;
    return p->bf16 ? launch_1k<0, unsigned>(p, a, in, out, name, bytes, s)
                   : launch_1k<0, float2>(p, a, in, out, name, bytes, s);
  }
  a.n_out = other;
  if (pack) {
    a.n_in = 2 * a.V - 1;
    a.off_in = -(a.V - 1);
    return launch_1k<3, float2>(p, a, in, out, name, bytes, s);
  }
  a.n_in = a.V;
  a.off_in = 0;
  return launch_1k<1, float2>(p, a, in, out, name, bytes, s);
}

}  // namespace

bool bluestein_takes(const bl_conv_plan_s* p, long P, int other) {
  bool pack;
  return takes_1k(p->Lw, p->V, P, other, &pack);
}

bl_status_t launch_bluestein_fwd(const bl_conv_plan_s* p, const float* in, void* out, long P, int Win, int oj,
                                 hipStream_t s) {
  BlueGeom a{};
  a.L = p->Lw;
  a.V = p->V;
  a.off_in = oj;
  a.nyq = (p->Lw % 2 == 0) ? p->Lw / 2 : -1;
  a.P = P;
  a.out_scale = 1.0f;
  const double bytes = (double)P * Win * 4 + (double)P * p->V * (p->bf16 ? 4 : 8);
  return launch_any(p, a, false, Win, in, out, "spec_fwd_1d", bytes, s);
}

bl_status_t launch_bluestein_inv(const bl_conv_plan_s* p, const float2* in, float* out, long P, int OW, int cj,
                                 hipStream_t s) {
  BlueGeom a{};
  a.L = p->Lw;
  a.V = p->V;
  a.off_out = cj;
  a.nyq = (p->Lw % 2 == 0) ? p->Lw / 2 : -1;
  a.P = P;
  a.out_scale = 1.0f / (float)p->Lw;
  const double bytes = (double)P * p->V * 8 + (double)P * OW * 4;
  return launch_any(p, a, true, OW, in, out, "spec_inv_1d", bytes, s);
}

}  // namespace blc


