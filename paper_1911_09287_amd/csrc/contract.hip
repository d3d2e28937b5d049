// Per-kept-bin complex channel contraction on the bf16 matrix cores (gfx950).
//
// For each kept bin, O[m][n] = sum_k A[m][k] op(B[k][n]) with op = conj or
// identity: the Hadamard product of the spectra fused with the sum over a
// channel index (Sec. 3.3), as four real products of the operands' real and
// imaginary planes with fp32 accumulators for the result's.
//
// complex64 spectra are multiplied exactly enough on the bf16 units: a float
// is the sum of three bfloat16 (8 significant bits each: x1 = bf16(x),
// x2 = bf16(x - x1), x3 = x - x1 - x2, all differences exact), and the six
// products x_i y_j with i + j <= 4 leave out terms below 2^-26 |x y|.  Six
// v_mfma_f32_32x32x16_bf16 do the work of eight fp32 32x32x2 instructions of
// twice their length each, 2.7 times the fp32 rate.  x1 y1 has an accumulator
// of its own, rounded K / 8 times instead of the fp32 chain's K; the five small
// products share another.  (All in one: 4 % faster, as three blocks then fit a
// CU's registers, but up to 8 % more error in a weight gradient than the fp32
// instructions gave; apart, the error is 0.35 to 0.9 of theirs.)  bfloat16
// spectra take the one product x1 y1.
//
// Measured against the fp32 instructions, contractions of one training step,
// c = 0.5: 64 channels 46 -> 38 us, 128 46 -> 38, 256 62 -> 45, 512 53 -> 39;
// 1-D 128 -> 256 channels 86 -> 60; 64 channels on the 58-grid at c = 0
// 112 -> 73 (4.8 TB/s of its compulsory bytes).
//
// Block tile: BM rows x BN complex columns, one wave per 32 x 32 complex block.
// Stages of 16 complex k (32 with bfloat16 spectra) are double buffered in
// LDS: while a wave multiplies stage s it splits and stores its part of stage
// s + 1, whose loads were issued a stage ahead; the splitting's vector
// instructions issue between the MFMAs.  (A single
// buffer, with splitting and products in turn, ran the 512-channel layer's
// passes 1.5 times longer: the blocks of a CU fall into step and their phases
// add up.)  Every thread loads patches of one row x 4 k of both operands, so
// that the loop has no branches; addresses outside the matrix or the k range
// read zero through the buffer bounds check.  LDS holds
// [part][re, im][k half][row][8 k], the operand layout of the MFMA: its reads
// are 16 bytes and its stores 8 bytes a lane, both free of bank conflicts.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "split.hpp"

namespace blc {
namespace {

// Byte offsets inside one bin's matrices are below 2^31 (checked on the host);
// the per-bin bases are 64-bit.
struct CgemmArgs {
  int M, N, K;                   // complex sizes
  unsigned sAm, sAk, sBk, sBn;   // element strides (complex units); one of each pair is 1
  unsigned ldo;
  unsigned long long bA, bB, bO;  // per-bin strides
  unsigned long long split_stride;  // complex elements between the partial outputs of two k-splits
  int tiles_n, tiles;               // tiles per bin along n, and per bin in all
  int kper;                         // complex k per split (multiple of the stage depth)
};

constexpr unsigned kOutside = 0x80000000u;  // a byte offset past any bin's matrix: reads zero

// Geometry of a BM x BN tile.
template <int BM, int BN, bool BF16>
struct Tile {
  static constexpr int STEPS = BF16 ? 2 : 1;  // steps of 16 complex k per stage
  static constexpr int KB = 16 * STEPS;
  static constexpr int PARTS = BF16 ? 1 : 3;
  static constexpr int NB = (BM / 32) * (BN / 32);  // 32 x 32 blocks, one wave each
  static constexpr int NT = 64 * NB;
  static constexpr int PTA = 4 * BM / NT, PTB = 4 * BN / NT;  // patches of the operands per thread and step
  // 16-byte units: a k half of an operand plane (rows plus a pad of half the
  // banks), planes, steps, stage buffer
  static constexpr int GA = BM + 4, GB = BN + 4;
  static constexpr int PA = 2 * GA, PB = 2 * GB;
  static constexpr int SA = 2 * PARTS * PA, SB = 2 * PARTS * PB;
  static constexpr int units = STEPS * (SA + SB);
};

// One operand as a matrix [row][k] (rows: m of A, n of B).
struct Operand {
  __amdgpu_buffer_rsrc_t buf;
  unsigned s_row, s_k;  // element strides; one of them is 1
  int rows, row0;       // rows of the matrix, first row of the tile
};

// A patch of one row x 4 k of a step: raw words, [k] (complex64: 2 words per
// value).  Element e of quarter q is k = 2 q + 8 (e / 2) + e % 2 of the step
// (both operands in the same order), in k half q / 2.
template <bool BF16>
struct Patch {
  static constexpr int W = BF16 ? 1 : 2;
  unsigned w[4][W];
};

// Patch p of an operand of R rows.  Along k (KC) the four quarters of a row
// are on neighbouring threads (a quad reads 64 consecutive bytes of
// complex64), else eight threads are on neighbouring rows.  Either way 16
// threads' 8-byte stores cover all banks.
template <int R, bool KC>
__device__ __forceinline__ void patch_pos(int p, int& row, int& q) {
  if constexpr (KC) {
    q = p & 3;
    row = p >> 2;
  } else {
    constexpr int H = R == 64 ? 3 : 2;  // row bits above the lowest three
    q = ((p >> 3) & 1) | ((p >> (4 + H)) << 1);
    row = (p & 7) | (((p >> 4) & ((1 << H) - 1)) << 3);
  }
}

// VEC: two-element loads along k (KC; an even number of k).
template <int R, bool KC, bool BF16, bool VEC>
__device__ __forceinline__ void load_patch(const Operand& o, int p, int k0, int kend, Patch<BF16>& d) {
  constexpr unsigned ES = BF16 ? 4 : 8;
  int row, q;
  patch_pos<R, KC>(p, row, q);
  const int left = o.row0 + row < o.rows ? kend - k0 - 2 * q : 0;  // elements of k inside, from the patch's first
  const unsigned base = (unsigned)(o.row0 + row) * o.s_row * ES + (unsigned)(k0 + 2 * q) * o.s_k * ES;
#pragma unroll
  for (int e = 0; e < 4; e += KC && VEC ? 2 : 1) {
    const int dk = 8 * (e >> 1) + (e & 1);
    const unsigned off = dk < left ? base + (unsigned)dk * o.s_k * ES : kOutside;
    if constexpr (KC && VEC) {
      if constexpr (BF16) {
        const uintx2 v = __builtin_amdgcn_raw_buffer_load_b64(o.buf, off, 0, 0);
        d.w[e][0] = v.x, d.w[e + 1][0] = v.y;
      } else {
        const uintx4 v = __builtin_amdgcn_raw_buffer_load_b128(o.buf, off, 0, 0);
        d.w[e][0] = v.x, d.w[e][1] = v.y, d.w[e + 1][0] = v.z, d.w[e + 1][1] = v.w;
      }
    } else if constexpr (BF16) {
      d.w[e][0] = __builtin_amdgcn_raw_buffer_load_b32(o.buf, off, 0, 0);
    } else {
      const uintx2 v = __builtin_amdgcn_raw_buffer_load_b64(o.buf, off, 0, 0);
      d.w[e][0] = v.x, d.w[e][1] = v.y;
    }
  }
}

// Splits a patch and stores it: plane (part, re/im) at dst + (2 part + im) * plane.
template <int R, bool KC, bool BF16>
__device__ __forceinline__ void store_patch(int p, const Patch<BF16>& d, uintx4* dst, int plane) {
  int row, q;
  patch_pos<R, KC>(p, row, q);
  uintx2* o = reinterpret_cast<uintx2*>(dst + (q >> 1) * (R + 4) + row) + (q & 1);
  if constexpr (BF16) {
    uintx2 re, im;
#pragma unroll
    for (int k = 0; k < 2; ++k) {  // (re, im) words of k and k + 1 to (re, re) and (im, im)
      re[k] = __builtin_amdgcn_perm(d.w[2 * k + 1][0], d.w[2 * k][0], 0x05040100u);
      im[k] = __builtin_amdgcn_perm(d.w[2 * k + 1][0], d.w[2 * k][0], 0x07060302u);
    }
    o[0] = re;
    o[2 * plane] = im;
  } else {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      uintx2 p1, p2, p3;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        unsigned q1, q2, q3;
        split3(__uint_as_float(d.w[2 * k][c]), __uint_as_float(d.w[2 * k + 1][c]), q1, q2, q3);
        p1[k] = q1, p2[k] = q2, p3[k] = q3;
      }
      o[2 * c * plane] = p1;
      o[2 * (2 + c) * plane] = p2;
      o[2 * (4 + c) * plane] = p3;
    }
  }
}

// One output tile: tile id (bin-major over the launch's tiles) and k-split kz,
// with the two stage buffers in smem (2 x Tile::units 16-byte units per group).
// KS groups of waves share the tile: group g takes stages g, g + KS, ... through
// its own buffers, and the groups' sums are added through LDS in group order.
template <int BM, int BN, bool A_KC, bool B_KC, bool CONJ, bool BF16, bool VEC, int KS>
__device__ __forceinline__ void cgemm_tile(const void* __restrict__ A, const void* __restrict__ B,
                                           float2* __restrict__ O, const CgemmArgs& g, unsigned id, int kz,
                                           uintx4* smem) {
  using T = Tile<BM, BN, BF16>;
  constexpr int ES = BF16 ? 4 : 8, KB = T::KB;
  const int bin = id / g.tiles, tile = id - bin * g.tiles;
  const int kbeg = kz * g.kper, kend = min(g.K, kbeg + g.kper);
  const int tm = tile / g.tiles_n, tn = tile - tm * g.tiles_n;
  const int m0 = tm * BM, n0 = tn * BN;
  const int grp = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / T::NT);
  const int tid = threadIdx.x - grp * T::NT, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const char* Ab = static_cast<const char*>(A) + (unsigned long long)bin * g.bA * ES;
  const char* Bb = static_cast<const char*>(B) + (unsigned long long)bin * g.bB * ES;
  const Operand oa{__builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(Ab), 0, (int)(g.bA * ES), 0x00020000),
                   g.sAm, g.sAk, g.M, m0};
  const Operand ob{__builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(Bb), 0, (int)(g.bB * ES), 0x00020000),
                   g.sBn, g.sBk, g.N, n0};

  // this thread's patches of both operands
  struct Stage {
    Patch<BF16> a[T::STEPS][T::PTA], b[T::STEPS][T::PTB];
  };
  auto load = [&](int k0, Stage& x) {
#pragma unroll
    for (int t = 0; t < T::STEPS; ++t) {
#pragma unroll
      for (int q = 0; q < T::PTA; ++q) load_patch<BM, A_KC, BF16, VEC>(oa, tid + T::NT * q, k0 + 16 * t, kend, x.a[t][q]);
#pragma unroll
      for (int q = 0; q < T::PTB; ++q) load_patch<BN, B_KC, BF16, VEC>(ob, tid + T::NT * q, k0 + 16 * t, kend, x.b[t][q]);
    }
  };
  auto store = [&](const Stage& x, uintx4* buf) {
#pragma unroll
    for (int t = 0; t < T::STEPS; ++t) {
      uintx4* at = buf + t * (T::SA + T::SB);
#pragma unroll
      for (int q = 0; q < T::PTA; ++q) store_patch<BM, A_KC, BF16>(tid + T::NT * q, x.a[t][q], at, T::PA);
#pragma unroll
      for (int q = 0; q < T::PTB; ++q) store_patch<BN, B_KC, BF16>(tid + T::NT * q, x.b[t][q], at + T::SA, T::PB);
    }
  };

  const int wm = wave / (BN / 32) * 32, wn = wave % (BN / 32) * 32;  // the wave's block
  const int half = lane >> 5, col = lane & 31;
  const int a_at = half * T::GA + wm + col, b_at = T::SA + half * T::GB + wn + col;
  floatx16 re, im, lre, lim;  // the first parts' product, and the smaller ones'
#pragma unroll
  for (int v = 0; v < 16; ++v) re[v] = 0.f, im[v] = 0.f, lre[v] = 0.f, lim[v] = 0.f;
  auto mma = [](uintx4 a, uintx4 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                   0);
  };
  auto compute = [&](const uintx4* buf) {
#pragma unroll
    for (int t = 0; t < T::STEPS; ++t) {
      const uintx4* ap = buf + t * (T::SA + T::SB) + a_at;
      const uintx4* bp = buf + t * (T::SA + T::SB) + b_at;
      uintx4 a[T::PARTS][2], b[T::PARTS][2], nb[T::PARTS];
#pragma unroll
      for (int q = T::PARTS - 1; q >= 0; --q)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          a[q][c] = ap[(2 * q + c) * T::PA];
          b[q][c] = bp[(2 * q + c) * T::PB];
        }
#pragma unroll
      for (int q = 0; q < T::PARTS; ++q) nb[q] = b[q][1] ^ 0x80008000u;  // -B's imaginary part
#pragma unroll
      for (int sum = T::PARTS - 1; sum >= 0; --sum)
#pragma unroll
        for (int i = 0; i <= sum; ++i) {
          const int j = sum - i;
          floatx16 &r = sum ? lre : re, &m = sum ? lim : im;
          r = mma(a[i][0], b[j][0], r);
          m = mma(a[i][1], b[j][0], m);
          r = mma(a[i][1], CONJ ? b[j][1] : nb[j], r);
          m = mma(a[i][0], CONJ ? nb[j] : b[j][1], m);
        }
    }
  };

  // the group's stage s lies in buffer s % 2; stages past the end read zero.
  // All groups run the same number of rounds.
  constexpr int STEP = KS * KB;
  Stage next;
  uintx4 *buf0 = smem + grp * 2 * T::units, *buf1 = buf0 + T::units;
  const int kg = kbeg + grp * KB;
  load(kg, next);
  store(next, buf0);
  load(kg + STEP, next);
  __syncthreads();
  for (int k0 = kbeg; k0 < kend; k0 += 2 * STEP) {
    const int kk = k0 + grp * KB;
    compute(buf0);
    store(next, buf1);
    load(kk + 2 * STEP, next);
    __syncthreads();
    if (k0 + STEP >= kend) break;
    compute(buf1);
    store(next, buf0);
    load(kk + 3 * STEP, next);
    __syncthreads();
  }
  if constexpr (!BF16) {
#pragma unroll
    for (int v = 0; v < 16; ++v) re[v] += lre[v], im[v] += lim[v];
  }
  if constexpr (KS > 1) {
    // groups 1.. leave their sums in the stage buffers; group 0 adds them in order
    float* red = reinterpret_cast<float*>(smem) + wave * 2048 + lane;
    static_assert((KS - 1) * T::NB * 2048 <= KS * 2 * T::units * 4, "the groups' sums fit the stage buffers");
    if (grp > 0) {
      float* r = red + (grp - 1) * T::NB * 2048;
#pragma unroll
      for (int v = 0; v < 16; ++v) r[v * 64] = re[v], r[(16 + v) * 64] = im[v];
    }
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int q = 0; q < KS - 1; ++q) {
      const float* r = red + q * T::NB * 2048;
#pragma unroll
      for (int v = 0; v < 16; ++v) re[v] += r[v * 64], im[v] += r[(16 + v) * 64];
    }
  }

  // D of a 32 x 32 block: register v holds row 8 (v / 4) + 4 (lane / 32) + v % 4, column lane % 32;
  // a store outside the matrix is dropped by the buffer bounds check
  float2* Ob = O + (unsigned long long)kz * g.split_stride + (unsigned long long)bin * g.bO;
  const __amdgpu_buffer_rsrc_t oo = __builtin_amdgcn_make_buffer_rsrc(Ob, 0, (int)(g.bO * 8), 0x00020000);
  const int n = n0 + wn + col, m1 = m0 + wm + 4 * half;
  const unsigned at = ((unsigned)m1 * g.ldo + n) * 8;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int dm = 8 * (v >> 2) + (v & 3);
    const unsigned off = m1 + dm < g.M && n < g.N ? at + dm * g.ldo * 8 : kOutside;
    __builtin_amdgcn_raw_buffer_store_b64((uintx2){__float_as_uint(re[v]), __float_as_uint(im[v])}, oo, off, 0, 0);
  }
}

// XCD-aware numbering of a launch's nb blocks: the hardware deals blocks to
// the 8 XCDs in turn, so consecutive logical ids (tiles of one bin, which
// share operand rows) land on one XCD and its L2.
__device__ __forceinline__ unsigned xcd_block_id(unsigned raw, unsigned nb) {
  const unsigned x = raw % 8, full = nb / 8, rest = nb % 8;
  return x * full + min(x, rest) + raw / 8;
}

// Blocks: (tile, bin) pairs, then k-splits.  LDS: KS x 2 x Tile::units.
template <int BM, int BN, bool A_KC, bool B_KC, bool CONJ, bool BF16, bool VEC, int KS>
__global__ __launch_bounds__(KS * BM * BN / 16, 2) void k_cgemm(
    const void* __restrict__ A, const void* __restrict__ B, float2* __restrict__ O, CgemmArgs g, unsigned per_split) {
  extern __shared__ uintx4 smem[];
  const unsigned id = xcd_block_id(blockIdx.x, gridDim.x), kz = id / per_split;
  cgemm_tile<BM, BN, A_KC, B_KC, CONJ, BF16, VEC, KS>(A, B, O, g, id - kz * per_split, kz, smem);
}

// The grad-input and grad-weight contractions of a layer in one launch (both
// need only the stored spectra), one tile shape for both: every XCD takes an
// eighth of each pass's tiles, those of the pass with the longer sums first,
// so that short tiles fill the CUs behind the long ones.  t1, t2: tiles x bins
// of grad-input (DX = DY W; s1 k ranges, whose partial sums lie split_stride
// apart) and grad-weight (DW = X^T conj(DY)).
template <int BM, int BN, bool BF16>
__global__ __launch_bounds__(BM * BN / 16, 2) void k_cgemm_bwd(
    const void* __restrict__ A1, const void* __restrict__ B1, float2* __restrict__ O1, CgemmArgs g1,
    const void* __restrict__ A2, const void* __restrict__ B2, float2* __restrict__ O2, CgemmArgs g2, unsigned t1,
    unsigned s1, unsigned t2, int first) {
  __shared__ uintx4 smem[2 * Tile<BM, BN, BF16>::units];
  const unsigned n1 = t1 * s1, n2 = t2, c1 = (n1 + 7) / 8, c2 = (n2 + 7) / 8;  // tiles, and each XCD's share
  const unsigned x = blockIdx.x % 8, at = blockIdx.x / 8, lead = first == 1 ? c1 : c2;
  const bool one = (at < lead) == (first == 1);
  const unsigned id = x * (one ? c1 : c2) + (at < lead ? at : at - lead);
  if (id >= (one ? n1 : n2)) return;
  if (one) {
    cgemm_tile<BM, BN, true, true, false, BF16, true, 1>(A1, B1, O1, g1, id % t1, id / t1, smem);
  } else {
    cgemm_tile<BM, BN, false, false, true, BF16, true, 1>(A2, B2, O2, g2, id, 0, smem);
  }
}

// out[i] = sum over k-splits of part[s][i], in split order.  V: two complex
// values, or one where the partial spectra's odd length leaves every second
// one off a 16-byte address.
template <typename V>
__global__ __launch_bounds__(256) void k_split_reduce(const V* __restrict__ part, V* __restrict__ out,
                                                      unsigned long long n, int splits) {
  const unsigned long long i = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  V acc = part[i];
  for (int s = 1; s < splits; ++s) acc += part[(unsigned long long)s * n + i];
  out[i] = acc;
}

constexpr int kSplitUnit = 32;  // k ranges are whole multiples of this

// Operand geometry of one pass; false when a bin's matrices are too large for
// 31-bit byte offsets.  vec: the two-element loads along k (operands with k
// contiguous) are aligned.
bool tiled_args(const bl_conv_plan_s* p, Contract which, CgemmArgs& g, bool& vec) {
  g = CgemmArgs{};
  const unsigned long long B = p->kept, N = p->N, Ci = p->Cin, Co = p->Cout;
  switch (which) {
    case Contract::Forward:  // Y[n][f] = sum_c X[n][c] conj(W[c][f])
      g.M = (int)N; g.N = (int)Co; g.K = (int)Ci;
      g.sAm = (unsigned)Ci; g.sAk = 1; g.sBk = (unsigned)Co; g.sBn = 1; g.ldo = (unsigned)Co;
      g.bA = N * Ci; g.bB = Ci * Co; g.bO = N * Co;
      break;
    case Contract::GradInput:  // DX[n][c] = sum_f DY[n][f] W[c][f]
      g.M = (int)N; g.N = (int)Ci; g.K = (int)Co;
      g.sAm = (unsigned)Co; g.sAk = 1; g.sBk = 1; g.sBn = (unsigned)Co; g.ldo = (unsigned)Ci;
      g.bA = N * Co; g.bB = Ci * Co; g.bO = N * Ci;
      break;
    case Contract::GradWeight:  // DW[c][f] = sum_n X[n][c] conj(DY[n][f])
      g.M = (int)Ci; g.N = (int)Co; g.K = (int)N;
      g.sAm = 1; g.sAk = (unsigned)Ci; g.sBk = (unsigned)Co; g.sBn = 1; g.ldo = (unsigned)Co;
      g.bA = N * Ci; g.bB = N * Co; g.bO = Ci * Co;
      break;
  }
  vec = g.K % 2 == 0;  // then every row, and every bin, starts on an even element of the k-contiguous operands
  if (B > 65535) return false;
  const long most = std::max<long>({(long)g.M * g.K, (long)g.K * g.N, (long)g.M * g.N});
  return 8 * most < 2147483647L;
}

double pass_bytes(const bl_conv_plan_s* p, const CgemmArgs& g) {
  const double ob = p->bf16 ? 4.0 : 8.0;  // bytes per stored operand element
  return (double)p->kept * (ob * ((double)g.M * g.K + (double)g.K * g.N) + 8.0 * g.M * g.N);
}

// Tile counts of a pass on BM x BN tiles and `splits` k ranges of whole
// stages (partial outputs split_stride = bins x M x N apart); returns the
// number of k ranges that hold stages.
int split_k_tiles(CgemmArgs& g, int BM, int BN, int splits, unsigned long long bins) {
  g.tiles_n = (g.N + BN - 1) / BN;
  g.tiles = ((g.M + BM - 1) / BM) * g.tiles_n;
  g.kper = ((g.K + splits - 1) / splits + kSplitUnit - 1) / kSplitUnit * kSplitUnit;
  g.split_stride = bins * (unsigned long long)g.M * g.N;
  return (g.K + g.kper - 1) / g.kper;
}

}  // namespace

bl_status_t launch_contract_tiled(const bl_conv_plan_s* p, Contract which, const void* A, const void* Bm,
                                  float2* O, float2* part, hipStream_t s, int parts) {
  CgemmArgs g;
  bool vec;
  if (!tiled_args(p, which, g, vec)) return BL_ERR_UNSUPPORTED;
  const unsigned long long B = p->kept;
  BlContractTiling t = p->ct[which == Contract::Forward ? 0 : which == Contract::GradInput ? 1 : 2];
  if (parts > 1) t.ks = p->fwd_ks;
  const int BM = t.bm, BN = t.bn;
  const unsigned long long total = B * (unsigned long long)g.M * g.N;  // complex outputs
  // the reduction works on pairs of outputs
  const int want = parts > 0 ? parts : total % 2 == 0 ? t.splits : 1;
  const int splits = split_k_tiles(g, BM, BN, want, B);
  if (parts > 1 && splits != parts) return BL_ERR_UNSUPPORTED;
  float2* dst = splits > 1 ? part : O;
  const unsigned long long blocks = B * (unsigned long long)g.tiles * splits;
  if (blocks >= 2147483647ULL) return BL_ERR_UNSUPPORTED;
  const dim3 grid((unsigned)blocks);
  const unsigned per_split = (unsigned)(B * g.tiles);
  const double flops = 8.0 * B * g.M * g.N * g.K;
  const double bytes = pass_bytes(p, g);
  const char* name = which == Contract::Forward ? "contract_fwd"
                     : which == Contract::GradInput ? "contract_dgrad" : "contract_wgrad";
  bl_status_t st = BL_ERR_UNSUPPORTED;
  // the groups' buffers can pass 64 KB of LDS: allowed once per kernel and device
  auto go = [&](auto kern, int units, int ks) {
    const size_t lds = (size_t)ks * 2 * units * 16;
    if (lds > kMaxLds) {
      const bl_status_t at = lds_opt_in(reinterpret_cast<const void*>(kern), (int)lds);
      if (at != BL_OK) return at;
    }
    return timed_launch(name, bytes, flops, s, [&](hipEvent_t e0, hipEvent_t e1) {
      hipExtLaunchKernelGGL(kern, grid, dim3(ks * BM * BN / 16), lds, s, e0, e1, 0, A, Bm, dst, g, per_split);
    });
  };
#define BL_VEC(BMV, BNV, AK, BK, CJ, BF, KSV)                                                  \
  (vec ? go(k_cgemm<BMV, BNV, AK, BK, CJ, BF, true, KSV>, Tile<BMV, BNV, BF>::units, KSV)        \
       : go(k_cgemm<BMV, BNV, AK, BK, CJ, BF, !(AK || BK), KSV>, Tile<BMV, BNV, BF>::units, KSV))
#define BL_TYPES(BMV, BNV, AK, BK, CJ, KSV)                      \
  st = p->bf16    ? BL_VEC(BMV, BNV, AK, BK, CJ, true, 1)    \
       : t.ks > 1 ? BL_VEC(BMV, BNV, AK, BK, CJ, false, KSV) \
                  : BL_VEC(BMV, BNV, AK, BK, CJ, false, 1)
#define BL_SHAPES(AK, BK, CJ)                                     \
  if (BM == 64 && BN == 64) BL_TYPES(64, 64, AK, BK, CJ, 2);      \
  else if (BM == 64 && BN == 32) BL_TYPES(64, 32, AK, BK, CJ, 4); \
  else if (BM == 32 && BN == 64) BL_TYPES(32, 64, AK, BK, CJ, 4); \
  else if (BM == 32 && BN == 32) BL_TYPES(32, 32, AK, BK, CJ, 4);
  if (which == Contract::Forward) {
    BL_SHAPES(true, false, true)
  } else if (which == Contract::GradInput) {
    BL_SHAPES(true, true, false)
  } else {
    vec = true;  // no operand has k contiguous
    BL_SHAPES(false, false, true)
  }
#undef BL_SHAPES
#undef BL_TYPES
#undef BL_VEC
  if (st != BL_OK || splits == 1 || parts > 1) return st;
  return launch_split_reduce(part, O, total, splits, s);
}

bl_status_t launch_contract_bwd_pair(const bl_conv_plan_s* p, const void* DY, const void* W, float2* DX,
                                     const void* X, float2* DW, hipStream_t s) {
  // With two images one launch of mostly empty tiles takes less than two where
  // one is thin (3 x 16 channels, 480 bins 17.3 / 21.2 us of the combined call
  // with stored spectra, 1740 bins 28.0 / 28.8); with one image, where both are,
  // while bins and products are few: 16 x 16, 544 bins 20.2 / 21.0, 684 bins 23.5 /
  // 22.1, 1740 bins 30.5 / 26.3; 64 x 64, 544 bins 34.9 / 34.8, 1002 bins 47.2 /
  // 43.2; 128 x 128, 252 bins 36.9 / 37.7, 480 bins 56.5 / 50.3; 256 x 256, 91 bins
  // 44.1 / 51.0, 252 bins 92 / 78; 512 x 512, 51 bins 73.7 / 83.8, 91 bins 142 / 140.
  const long products = (long)p->kept * p->Cin * p->Cout;
  const bool few = p->N == 2 || (p->N == 1 && (p->kept <= 96 || (p->kept <= 640 && products <= 6000000)));
  if (!few && (contract_is_thin(p, Contract::GradInput) || contract_is_thin(p, Contract::GradWeight)))
    return BL_ERR_UNSUPPORTED;
  if (p->bp_s1 == 0) return BL_ERR_UNSUPPORTED;
  CgemmArgs g1, g2;
  bool v1, v2;
  if (!tiled_args(p, Contract::GradInput, g1, v1) || !tiled_args(p, Contract::GradWeight, g2, v2)) return BL_ERR_UNSUPPORTED;
  if (!v1) return BL_ERR_UNSUPPORTED;
  const int BM = p->bp_bm, BN = p->bp_bn;
  const unsigned long long B = p->kept;
  if (split_k_tiles(g1, BM, BN, p->bp_s1, B) != p->bp_s1 || split_k_tiles(g2, BM, BN, 1, B) != 1)
    return BL_ERR_UNSUPPORTED;
  const unsigned long long n1 = (unsigned long long)g1.tiles * B, n2 = (unsigned long long)g2.tiles * B;
  if (n1 * p->bp_s1 + n2 >= 2147483600ULL) return BL_ERR_UNSUPPORTED;
  const double flops = 8.0 * p->kept * ((double)g1.M * g1.N * g1.K + (double)g2.M * g2.N * g2.K);
  const double bytes = pass_bytes(p, g1) + pass_bytes(p, g2);
  const unsigned t1 = (unsigned)n1, s1 = (unsigned)p->bp_s1, t2 = (unsigned)n2;
  const dim3 grid(8 * ((t1 * s1 + 7) / 8 + (t2 + 7) / 8));
  const int first = g1.kper >= g2.kper ? 1 : 2;  // the pass with the longer sums
  bl_status_t st = BL_ERR_UNSUPPORTED;
  auto go = [&](auto kern) {
    return timed_launch("contract_bwd", bytes, flops, s, [&](hipEvent_t e0, hipEvent_t e1) {
      hipExtLaunchKernelGGL(kern, grid, dim3(BM * BN / 16), 0, s, e0, e1, 0, DY, W, DX, g1, X, DY, DW, g2, t1, s1, t2, first);
    });
  };
  if (BM == 64 && BN == 64) st = p->bf16 ? go(k_cgemm_bwd<64, 64, true>) : go(k_cgemm_bwd<64, 64, false>);
  else if (BM == 64 && BN == 32) st = p->bf16 ? go(k_cgemm_bwd<64, 32, true>) : go(k_cgemm_bwd<64, 32, false>);
  else if (BM == 32 && BN == 64) st = p->bf16 ? go(k_cgemm_bwd<32, 64, true>) : go(k_cgemm_bwd<32, 64, false>);
  else if (BM == 32 && BN == 32) st = p->bf16 ? go(k_cgemm_bwd<32, 32, true>) : go(k_cgemm_bwd<32, 32, false>);
  return st;
}

bl_status_t launch_split_reduce(const float2* part, float2* out, unsigned long long n, int splits, hipStream_t s) {
  return timed_launch("contract_reduce", 8.0 * n * (splits + 1), 0.0, s, [&](hipEvent_t e0, hipEvent_t e1) {
    auto go = [&](auto kern, auto* from, auto* to, unsigned long long m) {
      hipExtLaunchKernelGGL(kern, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, s, e0, e1, 0, from, to, m, splits);
    };
    if (n % 2 == 0)
      go(k_split_reduce<floatx4>, reinterpret_cast<const floatx4*>(part), reinterpret_cast<floatx4*>(out), n / 2);
    else
      go(k_split_reduce<floatx2>, reinterpret_cast<const floatx2*>(part), reinterpret_cast<floatx2*>(out), n);
  });
}

}  // namespace blc
