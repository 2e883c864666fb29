// bruteforce.hip -- exhaustive t-MAD (Definition 1) with MFMA matrix cores:
// the products a_i . b_j of every pair, top t by |c|, without ever storing
// the m x n product (the exact baseline of Sec. 5.3 computes C in blocks and
// keeps a priority queue; here the GEMM epilogue filters against a bound).
//
//   pass A  GEMM over every 64th row of A; the epilogue histograms the lower
//           bounds |c^| - margin(i,j) of the computed values and their upper
//           bounds (1024 monotone bins each; screening: the values, 2048).
//           The lower edge tau of the bin holding the t-th largest lower
//           bound is <= the t-th largest |c| over all pairs, and the count of
//           the upper bounds that may reach tau sizes pass B's list.
//   pass B  GEMM over all pairs; the epilogue appends every pair with
//           |c^| + margin(i,j) >= tau.  That set holds every pair of the
//           exact top t.
//   final   fp32 dot products of the survivors (the same kernel the sampled
//           path uses) and an exact top-t selection on them.
//
// margin(i,j) bounds |c^ - c_fp32| for the MFMA arithmetic: inputs rounded to
// bf16 / fp8-e4m3 (relative error u, plus an absolute underflow term for
// fp8 after a per-vector power-of-two scale), fp32 accumulation over d
// terms (gamma_d), and the error of the fp32 re-rank itself (standard dot
// product error analysis, Higham, "Accuracy and Stability of Numerical
// Algorithms", 2nd ed., Sec. 3.1).
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include "../../include/mad.h"
#include "bf_common.hpp"
#include "mad_common.hpp"
#include "plan.hpp"

namespace mad {

constexpr int kBM = 128, kBN = 128;  // workgroup tile
constexpr int kRowBytes = 128;       // bytes of one row slice in LDS
constexpr int kLdsStride = kRowBytes + 16;

// ---------------------------------------------------------------------------
// preparation: padded low-precision copies (row stride Kp elements), the
// per-vector scale (fp8: a power of two), L2 and L1 norms of the fp32
// vector and the absolute rounding floor eta (in the vector's own units)
// ---------------------------------------------------------------------------
template <int P>
__global__ __launch_bounds__(256) void k_prep(const float* X, int64_t rows,
                                              int64_t d, int64_t Kp,
                                              void* out, VecInfo* info) {
  const int lane = threadIdx.x & 63;
  const int64_t r = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (r >= rows) return;
  const float* x = X + r * d;
  double s2 = 0.0, s1 = 0.0;
  float mx = 0.0f;
  for (int64_t k = lane; k < d; k += 64) {
    const double v = x[k];
    s2 += v * v;
    s1 += fabs(v);
    mx = fmaxf(mx, fabsf(x[k]));
  }
  const VecInfo vi = vec_info<P>(wave_sum(s2), wave_sum(s1), wave_max(mx));
  const float scale = vec_scale<P>(vi);
  if (lane == 0) info[r] = vi;
  for (int64_t k = lane; k < Kp; k += 64) {
    const float v = k < d ? x[k] : 0.0f;
    if (P == kF32) ((float*)out)[r * Kp + k] = v;
    else if (P == kBF16) ((uint16_t*)out)[r * Kp + k] = to_bf16(v);
    else ((uint8_t*)out)[r * Kp + k] = to_fp8(v * scale);
  }
}

// ---------------------------------------------------------------------------
// the GEMM: a 128 x 128 tile per workgroup, 4 waves of 64 x 64, each wave
// 2 x 2 MFMA blocks of 32 x 32.  MFMA operand layout (32 x 32 x K): lane l
// supplies row (l mod 32) of A and column (l mod 32) of B for its k group
// (l / 32); accumulator register r of lane l is row 8(r/4) + 4(l/32) + r%4,
// column l mod 32 of the block.
// ---------------------------------------------------------------------------
// the MFMA operands of one K step: rows (l mod 32) of the wave's two
// 32-row blocks of A and of B, K group l / 32
template <int P> struct Frag;
template <> struct Frag<kF32> { typedef float T; T a[2], b[2]; };
template <> struct Frag<kBF16> { typedef bf8v T; T a[2], b[2]; };
template <> struct Frag<kFP8> { typedef i8v T; T a[2], b[2]; };

template <int P>
__device__ __forceinline__ void frag_load(const char* la, const char* lb,
                                          int koff_bytes, int lane,
                                          Frag<P>& f) {
  const int r = lane & 31, g = lane >> 5;
  using PT = PrecT<P>;
  constexpr int gb = PT::KS / 2 * PT::EB;  // bytes of one K group
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    typedef typename Frag<P>::T T;
    f.a[u] = *(const T*)(la + (u * 32 + r) * kLdsStride + koff_bytes +
                         g * gb);
    f.b[u] = *(const T*)(lb + (u * 32 + r) * kLdsStride + koff_bytes +
                         g * gb);
  }
}

// ZERO: the accumulators start from zero (the tile's first K step)
template <int P, bool ZERO = false>
__device__ __forceinline__ void frag_mma(const Frag<P>& f, f16v (&acc)[2][2],
                                         const int (&sa)[2],
                                         const int (&sb)[2]) {
  const f16v zero = {};
#pragma unroll
  for (int bi = 0; bi < 2; ++bi)
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
      const f16v c = ZERO ? zero : acc[bi][bj];
      if constexpr (P == kF32)
        acc[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x2f32(
            f.a[bi], f.b[bj], c, 0, 0, 0);
      else if constexpr (P == kBF16)
        acc[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            f.a[bi], f.b[bj], c, 0, 0, 0);
      else
        acc[bi][bj] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
            f.a[bi], f.b[bj], c, 0, 0, 0, sa[bi], 0, sb[bj]);
    }
}

// Tiles of 128 x 128 in bands of 8 row-tiles; within a band the column
// tiles advance.  Workgroups are dispatched to the 8 XCDs round robin, so
// virtual block v = (blockIdx mod 8) G/8 + blockIdx / 8 gives each XCD a
// contiguous run of G/8 tiles per sweep: a column tile (a slice of B) is
// read by one XCD per band instead of by all eight.  K runs in stages of
// 128-byte row slices through two LDS buffers: the next stage (or the next
// tile's first) is loaded into registers while the current one computes.
__device__ __forceinline__ void gemm_coords(int64_t tile, int64_t tiles_m,
                                            int64_t tiles_n, int64_t& i0,
                                            int64_t& j0) {
  const int64_t band = tile / (8 * tiles_n);
  const int64_t within = tile % (8 * tiles_n);
  const int64_t band_rows = tiles_m - band * 8 < 8 ? tiles_m - band * 8 : 8;
  i0 = (band * 8 + within % band_rows) * kBM;
  j0 = (within / band_rows) * kBN;
}

// (Each stage's loads go where the compiler puts them, after the stage before
// has issued its MFMAs: kept ahead of them they were slower at K = 512, 1.71
// to 1.77 s against 1.44 to 1.59 at 1e6 x 1e6 in bf16.)
// (fp8's pass A would take 268 registers, and a CU then one workgroup.)
template <int P, bool HIST>
__global__ __launch_bounds__(256, P == kFP8 ? 2 : 1) void k_gemm_topk(
    GemmArgs g) {
  using PT = PrecT<P>;
  __shared__ __attribute__((aligned(16))) char lds_a[2][kBM * kLdsStride];
  __shared__ __attribute__((aligned(16))) char lds_b[2][kBN * kLdsStride];
  __shared__ unsigned hist[HIST ? 2048 : 1];
  // the running bound is kept in the padding of a row: the 80 KB of the
  // others are half of a CU's LDS, and four bytes more would leave it one
  // workgroup (pass A at 1024 x 65,536 x 1024 in fp32: 1.60 ms, 2.09 then)
  unsigned* thr = (unsigned*)(lds_a[0] + kRowBytes);
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int wr = wv >> 1, wc = wv & 1;
  if (HIST) {
    for (int b = t; b < 2048; b += 256) hist[b] = 0;
    if (t == 0) *thr = 0u;
    __syncthreads();
  }
  const int64_t tiles_m = (g.m_rows + kBM - 1) / kBM;
  const int64_t tiles_n = (g.n + kBN - 1) / kBN;
  const int64_t ntiles = tiles_m * tiles_n;
  const int64_t row_bytes = g.Kp * PT::EB;
  const int64_t nst = row_bytes / kRowBytes;  // Kp EB is a multiple of 128
  const char* Ab = (const char*)g.A;
  const char* Bb = (const char*)g.B;
  const float tau = HIST ? 0.0f : __uint_as_float(*g.tau_bits);
  BoundBins bins{-1};
  if (HIST) bins = bound_bins(g.maxes, g.coarse);
  // |c| below `pre` is dropped at once: |c| + margin does not reach tau (pass
  // B; 1 - 2^-20 absorbs the roundings of the comparisons), or the bound that
  // g.target lower bounds counted so far lie above (pass A)
  const float mg_max = HIST ? margin_max(g) : g.mg_max;
  float pre = HIST ? -mg_max : fmaf(tau, 1.0f - 0x1p-20f, -mg_max);
  unsigned done = 0;
  const int64_t G = gridDim.x;  // a multiple of 8
  const int64_t v = (int64_t)(blockIdx.x & 7) * (G >> 3) + (blockIdx.x >> 3);
  // this thread's 4 x 16 bytes of each operand's stage: rows (t >> 3) +
  // 32 q, bytes (t & 7) 16 of the 128-byte slice
  const int seg = (t & 7) * 16;
// one 16-byte piece q of each operand's stage (rows (t >> 3) + 32 q), and
// its store to LDS; written out per q so that ra / rb stay in registers
#define MAD_BF_GLOAD1(Q, I0, J0, KB)                                         \
  {                                                                          \
    const int row = (t >> 3) + 32 * (Q);                                     \
    int64_t ia = (I0) + row;                                                 \
    ia = ia < g.m_rows ? ia : g.m_rows - 1;                                  \
    int64_t jb = (J0) + row;                                                 \
    jb = jb < g.n ? jb : g.n - 1;                                            \
    ra##Q = *(const uint4*)(Ab + ia * g.a_stride_rows * row_bytes + (KB) +   \
                            seg);                                            \
    rb##Q = *(const uint4*)(Bb + jb * row_bytes + (KB) + seg);               \
  }
#define MAD_BF_GLOAD(I0, J0, KB)                                             \
  MAD_BF_GLOAD1(0, I0, J0, KB) MAD_BF_GLOAD1(1, I0, J0, KB)                  \
  MAD_BF_GLOAD1(2, I0, J0, KB) MAD_BF_GLOAD1(3, I0, J0, KB)
#define MAD_BF_LSTORE1(Q, BUF)                                               \
  {                                                                          \
    const int row = (t >> 3) + 32 * (Q);                                     \
    *(uint4*)(lds_a[BUF] + row * kLdsStride + seg) = ra##Q;                  \
    *(uint4*)(lds_b[BUF] + row * kLdsStride + seg) = rb##Q;                  \
  }
#define MAD_BF_LSTORE(BUF)                                                   \
  MAD_BF_LSTORE1(0, BUF) MAD_BF_LSTORE1(1, BUF) MAD_BF_LSTORE1(2, BUF)       \
  MAD_BF_LSTORE1(3, BUF)
// full tiles (no row past the end): the 4 pieces of an operand are 32 rows
// apart, so one base pointer per tile serves every stage
#define MAD_BF_FULL(I0, J0) ((I0) + kBM <= g.m_rows && (J0) + kBN <= g.n)
#define MAD_BF_PA(I0) (Ab + ((I0) + trow) * g.a_stride_rows * row_bytes + seg)
#define MAD_BF_PB(J0) (Bb + ((J0) + trow) * row_bytes + seg)
#define MAD_BF_GLOADF(PA, PB, KB)                                            \
  {                                                                          \
    ra0 = *(const uint4*)((PA) + (KB));                                      \
    ra1 = *(const uint4*)((PA) + astep + (KB));                              \
    ra2 = *(const uint4*)((PA) + 2 * astep + (KB));                          \
    ra3 = *(const uint4*)((PA) + 3 * astep + (KB));                          \
    rb0 = *(const uint4*)((PB) + (KB));                                      \
    rb1 = *(const uint4*)((PB) + bstep + (KB));                              \
    rb2 = *(const uint4*)((PB) + 2 * bstep + (KB));                          \
    rb3 = *(const uint4*)((PB) + 3 * bstep + (KB));                          \
  }
  const int64_t trow = t >> 3;
  const int64_t astep = 32 * g.a_stride_rows * row_bytes;
  const int64_t bstep = 32 * row_bytes;
  uint4 ra0, ra1, ra2, ra3, rb0, rb1, rb2, rb3;
  int64_t tile = v;
  int64_t i0 = 0, j0 = 0;
  bool full = false;
  const char* pa = Ab;
  const char* pb = Bb;
  if (tile < ntiles) {
    gemm_coords(tile, tiles_m, tiles_n, i0, j0);
    full = MAD_BF_FULL(i0, j0);
    pa = MAD_BF_PA(i0);
    pb = MAD_BF_PB(j0);
    if (full) {
      MAD_BF_GLOADF(pa, pb, 0)
    } else {
      MAD_BF_GLOAD(i0, j0, 0)
    }
  }
  while (tile < ntiles) {
    const int64_t next = tile + G;
    int64_t ni0 = 0, nj0 = 0;
    if (next < ntiles) gemm_coords(next, tiles_m, tiles_n, ni0, nj0);
    const bool nfull = next < ntiles && MAD_BF_FULL(ni0, nj0);
    const char* npa = MAD_BF_PA(ni0);
    const char* npb = MAD_BF_PB(nj0);
    // fp8: the per-vector scales of the rows this lane feeds the MFMA
    int sa[2] = {127, 127}, sb[2] = {127, 127};
    if (P == kFP8) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        int64_t ia = i0 + wr * 64 + u * 32 + (lane & 31);
        ia = ia < g.m_rows ? ia : g.m_rows - 1;
        int64_t jb = j0 + wc * 64 + u * 32 + (lane & 31);
        jb = jb < g.n ? jb : g.n - 1;
        sa[u] = e8m0_of(g.ia[ia * g.a_stride_rows].inv_s);
        sb[u] = e8m0_of(g.ib[jb].inv_s);
      }
    }
    MAD_BF_LSTORE(0)
    __syncthreads();
    // the tile's first MFMAs start from a zero C operand (no per-tile
    // clearing of the 64 accumulators); a tile always has a stage (Kp >= 1)
    f16v acc[2][2];
    int cur = 0;
    for (int64_t st = 0; st < nst; ++st) {
      // the next stage, else the next tile's first, else (last tile) a
      // harmless reload of this tile's first: unconditional loads keep
      // ra / rb in registers
      const bool more = st + 1 < nst;
      const bool nx = !more && next < ntiles;
      const int64_t li0 = nx ? ni0 : i0;
      const int64_t lj0 = nx ? nj0 : j0;
      const int64_t lkb = more ? (st + 1) * kRowBytes : 0;
      if (nx ? nfull : full) {
        const char* lpa = nx ? npa : pa;
        const char* lpb = nx ? npb : pb;
        MAD_BF_GLOADF(lpa, lpb, lkb)
      } else {
        MAD_BF_GLOAD(li0, lj0, lkb)
      }
      const char* la = lds_a[cur] + (wr * 64) * kLdsStride;
      const char* lb = lds_b[cur] + (wc * 64) * kLdsStride;
      // the next K step's operands are read from LDS while the current
      // step's MFMAs run
      constexpr int nks = PT::KC / PT::KS;
      Frag<P> fr[2];
      frag_load<P>(la, lb, 0, lane, fr[0]);
#pragma unroll
      for (int ks = 0; ks < nks; ++ks) {
        if (ks + 1 < nks)
          frag_load<P>(la, lb, (ks + 1) * PT::KS * PT::EB, lane,
                       fr[(ks + 1) & 1]);
        if (ks == 0 && st == 0)
          frag_mma<P, true>(fr[0], acc, sa, sb);
        else
          frag_mma<P>(fr[ks & 1], acc, sa, sb);
      }
      if (more) {
        MAD_BF_LSTORE(cur ^ 1)
      }
      __syncthreads();
      cur ^= 1;
    }
    // epilogue: one max over the lane's 64 values first; the per-element
    // work below, with the exact margin, runs only in waves where some lane
    // reaches `pre`, which almost no pair does
    const int cl = lane & 31, rg = lane >> 5;
    float mx = 0.0f;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int bj = 0; bj < 2; ++bj)
#pragma unroll
        for (int e = 0; e < 16; ++e) mx = fmaxf(mx, fabsf(acc[bi][bj][e]));
    const bool any = mx >= pre;
    if (any) {
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
      const int64_t j = j0 + wc * 64 + bj * 32 + cl;
      const bool jok = j < g.n;
#pragma unroll
      for (int bi = 0; bi < 2; ++bi) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int64_t i = i0 + wr * 64 + bi * 32 + 8 * (e >> 2) + 4 * rg +
                            (e & 3);
          const float c = acc[bi][bj][e];
          // (pass A counts the others of the lane as well: they do no harm,
          // and a test of each takes longer)
          if (!HIST && !(fabsf(c) >= pre)) continue;
          if (!(jok && i < g.m_rows)) continue;
          const VecInfo va = g.ia[i * g.a_stride_rows];
          const VecInfo vb = g.ib[j];
          const float mg = g.screen ? 0.0f
                                    : pair_margin(g.kappa, g.onepu, g.d_f,
                                                  va, vb);
          if (HIST) {
            count_bounds(bins, c, mg, hist);
          } else if (fabsf(c) + mg >= tau) {
            const unsigned long long p = atomicAdd(g.ccount, 1ull);
            if ((int64_t)p < g.ccap) {
              g.ckey[p] = (uint64_t)(i * g.m_key) * (uint64_t)g.n + (uint64_t)j;
              g.cval[p] = c;
            }
          }
        }
      }
    }
    }
    // after 16, 64, 256, ... tiles while 16 or more are left: a raise takes
    // as long as the bound saves in five to ten tiles, and an early bound
    // saves little (pass A at 3125 x 2e5 x 512 in bf16, 76 tiles a workgroup:
    // 2.25 ms, 2.49 with raises after 1 and 4 too; at 1024 x 65,536 x 257,
    // eight tiles, 0.30 and 0.38)
    ++done;
    if (HIST && (done & (done - 1)) == 0 && (done & 0x55555550u) &&
        ntiles - tile > 16 * G)
      pre = raise_bound(g, bins, mg_max, hist, thr);
    tile = next;
    i0 = ni0;
    j0 = nj0;
    full = nfull;
    pa = npa;
    pb = npb;
  }
  if (HIST) {
    __syncthreads();
    for (int b = t; b < 2048; b += 256)
      if (hist[b]) atomicAdd(&g.hist[b], hist[b]);
  }
}
#undef MAD_BF_GLOAD1
#undef MAD_BF_GLOAD
#undef MAD_BF_FULL
#undef MAD_BF_PA
#undef MAD_BF_PB
#undef MAD_BF_GLOADF
#undef MAD_BF_LSTORE1
#undef MAD_BF_LSTORE

// maxima of n2, n1 and eta over the vectors of A (blockIdx.y 0, to mx[0..2])
// and of B (1, to mx[4..6]), as float bits
__global__ __launch_bounds__(1024) void k_vecinfo_max(const VecInfo* va,
                                                      int64_t m,
                                                      const VecInfo* vb,
                                                      int64_t n,
                                                      unsigned* mx) {
  __shared__ float red[3][16];
  const VecInfo* v = blockIdx.y ? vb : va;
  const int64_t rows = blockIdx.y ? n : m;
  float a = 0.0f, b = 0.0f, c = 0.0f;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < rows;
       r += stride) {
    a = fmaxf(a, v[r].n2);
    b = fmaxf(b, v[r].n1);
    c = fmaxf(c, v[r].eta);
  }
  a = wave_max(a);
  b = wave_max(b);
  c = wave_max(c);
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    red[0][wv] = a;
    red[1][wv] = b;
    red[2][wv] = c;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    float x = 0.0f;
    for (int w = 0; w < 16; ++w) x = fmaxf(x, red[threadIdx.x][w]);
    atomicMax(&mx[4 * blockIdx.y + threadIdx.x], __float_as_uint(x));
  }
}

// One wave over pass A's histogram: tau_bits = the lower edge of the bin
// holding the t-th largest lower bound, from the top (0 when fewer than t
// are positive), and est = the subset's pairs that pass B's filter will
// keep: those whose upper bound (screening: value) reaches that bin.  (One
// thread walking the 2048 bins took 54 us.)
__global__ __launch_bounds__(64) void k_bf_tau(GemmArgs g,
                                               unsigned* tau_bits,
                                               unsigned long long* est) {
  const int lane = threadIdx.x;
  const int64_t t = g.target;
  const BoundBins bins = bound_bins(g.maxes, g.coarse);
  // lane l: `per` bins from the top
  const int per = bins.count() / 64;
  const int hi = bins.count() - 1 - per * lane;
  unsigned long long sum = 0;
  for (int b = hi; b > hi - per; --b) sum += g.hist[b];
  const unsigned long long incl = wave_incl_scan(sum);
  const uint64_t reach = __ballot((int64_t)incl >= t);
  const int src = reach ? __builtin_ctzll(reach) : 63;
  int found = 0;
  if (reach && lane == src) {
    unsigned long long acc = incl - sum;
    found = hi;
    for (; found > hi - per + 1; --found) {
      acc += g.hist[found];
      if ((int64_t)acc >= t) break;
    }
  }
  found = __shfl(found, src, 64);
  const unsigned* up = bins.fine0 < 0 ? g.hist : g.hist + kUpperBins;
  unsigned long long in = 0;
  for (int b = hi; b > hi - per; --b) in += b >= found ? up[b] : 0u;
  in = wave_sum(in);
  if (lane == 0) {
    *tau_bits = bins.edge(found);
    *est = in;
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct BfWork {
  DeviceBuffer ac, bc, ia, ib, e8, misc, keys, vals, sel, selbuf, fin;
};

static BfWork g_bf;  // process-wide cache of the conversion workspace

static double gamma_d(int64_t d) {
  const double u = ldexp(1.0, -24);
  return d * u / (1.0 - d * u);
}

template <int P>
static void launch_gemm(const GemmArgs& a, bool hist, hipStream_t st) {
  // persistent workgroups, two per CU (LDS), a multiple of 8 (one share
  // per XCD); MAD_BF_GRID overrides the count (the result is the same)
  const int64_t tiles = ((a.m_rows + kBM - 1) / kBM) * ((a.n + kBN - 1) / kBN);
  int64_t grid = tiles < 256 * 2 ? (tiles + 7) / 8 * 8 : 256 * 2;
  if (const char* ev = getenv("MAD_BF_GRID")) {
    const int64_t gv = atoll(ev) / 8 * 8;
    if (gv >= 8) grid = gv;
  }
  if (grid < 8) grid = 8;

  if (hist)
    k_gemm_topk<P, true><<<(unsigned)grid, 256, 0, st>>>(a);
  else
    k_gemm_topk<P, false><<<(unsigned)grid, 256, 0, st>>>(a);
}

hipError_t lowp_prepare(const float* X, int64_t rows, int64_t d, int prec,
                        DeviceBuffer& data, DeviceBuffer& info, int64_t* Kp,
                        hipStream_t st) {
  const int KC = prec == kBF16 ? 64 : 128;
  const int EB = prec == kBF16 ? 2 : 1;
  if (prec != kBF16 && prec != kFP8) return hipErrorInvalidValue;
  const int64_t kp = (d + KC - 1) / KC * KC;
  hipError_t e;
  if ((e = dev_alloc(data, (size_t)rows * kp * EB)) != hipSuccess ||
      (e = dev_alloc(info, (size_t)rows * sizeof(VecInfo))) != hipSuccess)
    return e;
  const unsigned g = (unsigned)((rows + 3) / 4);
  if (prec == kBF16)
    k_prep<kBF16><<<g, 256, 0, st>>>(X, rows, d, kp, data.p,
                                      (VecInfo*)info.p);
  else
    k_prep<kFP8><<<g, 256, 0, st>>>(X, rows, d, kp, data.p,
                                     (VecInfo*)info.p);
  *Kp = kp;
  return hipGetLastError();
}

void lowp_consts(int prec, int64_t d, float* kappa, float* onepu) {
  const double u = prec == kF32 ? 0.0 : prec == kBF16 ? ldexp(1.0, -8)
                                                       : ldexp(1.0, -4);
  const double g = gamma_d(d);
  *kappa = (float)((2 * u + u * u + g * (1 + u) * (1 + u) + g) * (1 + 1e-5));
  *onepu = (float)((1 + u) * (1 + 1e-5));
}

hipError_t bruteforce_topk(const float* A, int64_t m, const float* B,
                           int64_t n, int64_t d, int prec, int64_t t,
                           int64_t cap_hint, void* out, int64_t* n_out,
                           BfStats* stats, hipStream_t st) {
  return bruteforce_run(A, m, B, n, d, prec, t, cap_hint, -1.0f, out, n_out,
                        nullptr, nullptr, stats, st);
}

hipError_t bruteforce_run(const float* A, int64_t m, const float* B,
                          int64_t n, int64_t d, int prec, int64_t t,
                          int64_t cap_hint, float tau_user, void* out,
                          int64_t* n_out, const uint64_t** cand_keys,
                          int64_t* cand_count, BfStats* stats,
                          hipStream_t st) {
  hipError_t e;
  int KC = prec == kF32 ? 32 : prec == kBF16 ? 64 : 128;
  int EB = prec == kF32 ? 4 : prec == kBF16 ? 2 : 1;
  const int64_t Kp = (d + KC - 1) / KC * KC;
  const bool panel = panel_steps(prec, d) > 0;
  const size_t abytes = panel ? (size_t)panel_bytes(prec, d, m)
                              : (size_t)m * Kp * EB;
  const size_t bbytes = panel ? (size_t)panel_bytes(prec, d, n)
                              : (size_t)n * Kp * EB;
  BfWork& w = g_bf;
  if ((e = dev_alloc(w.ac, abytes)) != hipSuccess) return e;
  if ((e = dev_alloc(w.bc, bbytes)) != hipSuccess) return e;
  // E8M0 scales of both sides' vectors (fp8 panels), padded rows too
  const int64_t mpad = (m + 127) / 128 * 128, npad = (n + 127) / 128 * 128;
  if (panel && prec == kFP8 &&
      (e = dev_alloc(w.e8, (size_t)(mpad + npad) * 4)) != hipSuccess)
    return e;
  int* ea8 = (int*)w.e8.p;
  int* eb8 = ea8 + mpad;
  if ((e = dev_alloc(w.ia, (size_t)m * sizeof(VecInfo))) != hipSuccess) return e;
  if ((e = dev_alloc(w.ib, (size_t)n * sizeof(VecInfo))) != hipSuccess) return e;
  if ((e = dev_alloc(w.misc, 2048 * 4 + 512)) != hipSuccess) return e;
  hipEvent_t ev[4];
  for (auto& x : ev) (void)hipEventCreate(&x);
  (void)hipEventRecord(ev[0], st);
  // conversion is part of every call (the inputs may change between calls)
  const unsigned ga = (unsigned)((m + 3) / 4), gb = (unsigned)((n + 3) / 4);
  if (panel) {
    if ((e = panel_prepare(A, m, d, prec, w.ac.p, (VecInfo*)w.ia.p, ea8,
                           st)) != hipSuccess ||
        (e = panel_prepare(B, n, d, prec, w.bc.p, (VecInfo*)w.ib.p, eb8,
                           st)) != hipSuccess)
      return e;
  } else if (prec == kF32) {
    k_prep<kF32><<<ga, 256, 0, st>>>(A, m, d, Kp, w.ac.p, (VecInfo*)w.ia.p);
    k_prep<kF32><<<gb, 256, 0, st>>>(B, n, d, Kp, w.bc.p, (VecInfo*)w.ib.p);
  } else if (prec == kBF16) {
    k_prep<kBF16><<<ga, 256, 0, st>>>(A, m, d, Kp, w.ac.p, (VecInfo*)w.ia.p);
    k_prep<kBF16><<<gb, 256, 0, st>>>(B, n, d, Kp, w.bc.p, (VecInfo*)w.ib.p);
  } else {
    k_prep<kFP8><<<ga, 256, 0, st>>>(A, m, d, Kp, w.ac.p, (VecInfo*)w.ia.p);
    k_prep<kFP8><<<gb, 256, 0, st>>>(B, n, d, Kp, w.bc.p, (VecInfo*)w.ib.p);
  }
  unsigned* hist = (unsigned*)w.misc.p;
  unsigned* tau_bits = hist + 2048;
  unsigned long long* ccount = (unsigned long long*)(hist + 2048 + 16);
  unsigned* maxes = hist + 2048 + 32;  // n2, n1, eta of A then of B
  unsigned long long* est = (unsigned long long*)(hist + 2048 + 48);
  if ((e = launch_fill_u64((uint64_t*)hist, 1024 + 8 + 8 + 8 + 8, 0ull,
                           st)) != hipSuccess)
    return e;
  k_vecinfo_max<<<dim3(64, 2), 1024, 0, st>>>(
      (const VecInfo*)w.ia.p, m, (const VecInfo*)w.ib.p, n, maxes);
  // margin factor: input rounding (2u + u^2) plus gamma_d for the MFMA
  // accumulation and gamma_d for the fp32 re-rank
  const double u = prec == kF32 ? 0.0 : prec == kBF16 ? ldexp(1.0, -8)
                                                       : ldexp(1.0, -4);
  const double g = gamma_d(d);
  GemmArgs a;
  a.A = w.ac.p;
  a.B = w.bc.p;
  a.ia = (const VecInfo*)w.ia.p;
  a.ib = (const VecInfo*)w.ib.p;
  a.n = n;
  a.Kp = Kp;
  a.kappa = (float)((2 * u + u * u + g * (1 + u) * (1 + u) + g) * (1 + 1e-5));
  a.onepu = (float)((1 + u) * (1 + 1e-5));
  a.d_f = (float)d;
  a.hist = hist;
  a.maxes = maxes;
  a.tau_bits = tau_bits;
  // screening (t_screen > 0, low precision): threshold and filter on the
  // computed value, keep the t_screen largest, re-rank those in fp32
  const bool screen = prec != kF32 && cap_hint > 0;
  a.screen = screen ? 1 : 0;
  a.coarse = a.screen;
  a.mg_max = 0.0f;
  // pass A over every stride-th row of A
  const int64_t stride = m >= 128 * 64 ? 64 : (m >= 128 * 8 ? 8 : 1);
  a.m_rows = (m + stride - 1) / stride;
  a.a_stride_rows = stride;
  a.m_key = stride;
  a.ckey = nullptr;
  a.ccap = 0;
  a.ccount = ccount;
  auto gemm = [&](bool hist_pass) -> hipError_t {
    if (panel) return launch_panel(a, prec, d, hist_pass, eb8, st);
    if (prec == kF32) launch_gemm<kF32>(a, hist_pass, st);
    else if (prec == kBF16) launch_gemm<kBF16>(a, hist_pass, st);
    else launch_gemm<kFP8>(a, hist_pass, st);
    return hipGetLastError();
  };
  // pass A's subset holds about 1/stride of the pairs
  a.target = screen ? (cap_hint + stride - 1) / stride : t;
  auto pass_a = [&]() -> hipError_t {
    const hipError_t r = gemm(true);
    if (r == hipSuccess) k_bf_tau<<<1, 64, 0, st>>>(a, tau_bits, est);
    return r;
  };
  if (tau_user >= 0.0f) {
    // a threshold given by the caller (a lower bound it knows for the t-th
    // largest |c|): pass B keeps every pair that may reach it
    uint32_t tb;
    memcpy(&tb, &tau_user, 4);
    if ((e = launch_fill_u64((uint64_t*)tau_bits, 1, (uint64_t)tb, st)) !=
        hipSuccess)
      return e;
  } else {
    if ((e = pass_a()) != hipSuccess) return e;
  }
  (void)hipEventRecord(ev[1], st);
  // the largest margin over all pairs, for pass B's pre-test, and pass A's
  // estimate of its survivors
  unsigned long long sub = 0;
  {
    unsigned mxb[50];  // tau, then (+32) the maxima, (+48) the estimate
    auto read = [&]() -> hipError_t {
      const hipError_t r = hipMemcpyAsync(mxb, tau_bits, sizeof mxb,
                                          hipMemcpyDeviceToHost, st);
      return r != hipSuccess ? r : hipStreamSynchronize(st);
    };
    if ((e = read()) != hipSuccess) return e;
    if (tau_user < 0.0f && !a.coarse && mxb[0] == 0) {
      // fewer than t bounds above the finer bins' range (200 octaves under
      // the largest possible |c|): the bins over all floats
      a.coarse = 1;
      if ((e = launch_fill_u64((uint64_t*)hist, 1024, 0ull, st)) !=
              hipSuccess ||
          (e = pass_a()) != hipSuccess || (e = read()) != hipSuccess)
        return e;
    }
    float f[8];
    memcpy(f, mxb + 32, sizeof f);
    memcpy(&sub, mxb + 48, 8);
    const double mgm = screen ? 0.0
                              : (double)a.kappa * f[0] * f[4] +
                                    (double)a.onepu * (f[2] * f[5] + f[6] * f[1]) +
                                    (double)a.d_f * f[2] * f[6];
    a.mg_max = (float)(mgm * (1.0 + 1e-5));
  }
  // pass B over all pairs
  int64_t cap = screen ? 4 * cap_hint : (cap_hint > 0 ? cap_hint : (1 << 20));
  if (cap < 16 * t) cap = 16 * t;
  // room for what pass A's subset (1 / stride of the rows) lets expect, a
  // quarter and four standard deviations over it: a list that overflows
  // costs the whole GEMM again (1e5 x 1e6 x 256 in bf16, t = 1000: 153.8
  // ms a call with two runs, 70.6 with one).  Above 2^26 pairs the estimate
  // is not followed: the first run counts the pairs exactly before that much
  // memory is taken.
  const double want = ((double)sub * 1.25 + 4.0 * sqrt((double)sub)) *
                          (double)stride + 1024.0;
  if (want > (double)cap && want <= (double)(int64_t(1) << 26))
    cap = (int64_t)want;
  // a longer list that the workspace holds already is used as it is
  const int64_t have = (int64_t)(w.keys.bytes / 8 < w.vals.bytes / 4
                                     ? w.keys.bytes / 8
                                     : w.vals.bytes / 4);
  if (cap < have) cap = have;
  a.m_rows = m;
  a.a_stride_rows = 1;
  a.m_key = 1;
  unsigned long long count = 0;
  for (int attempt = 0; attempt < 4; ++attempt) {
    if ((e = dev_alloc(w.keys, (size_t)cap * 8)) != hipSuccess) break;
    if ((e = dev_alloc(w.vals, (size_t)cap * 4)) != hipSuccess) break;
    a.ckey = (uint64_t*)w.keys.p;
    a.cval = (float*)w.vals.p;
    a.ccap = cap;
    if ((e = launch_fill_u64((uint64_t*)ccount, 1, 0ull, st)) != hipSuccess)
      break;
    if ((e = gemm(false)) != hipSuccess) break;
    if ((e = hipMemcpyAsync(&count, ccount, 8, hipMemcpyDeviceToHost, st)) !=
        hipSuccess) break;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) break;
    if ((int64_t)count <= cap) break;
    if (count > (1ull << 28)) {  // the bound filters nothing useful
      e = hipErrorOutOfMemory;
      break;
    }
    cap = (int64_t)(count + count / 4 + 1024);  // rerun with room for all
  }
  (void)hipEventRecord(ev[2], st);
  int64_t nre = (int64_t)count;
  const uint64_t* rkeys = (const uint64_t*)w.keys.p;
  if (cand_keys) *cand_keys = rkeys;
  if (cand_count) *cand_count = nre;
  if (e == hipSuccess && screen && nre > cap_hint) {
    // the t_screen survivors with the largest computed |c|
    if ((e = dev_alloc(w.sel, (size_t)cap_hint * 8)) == hipSuccess)
      e = launch_select_keys_by_absval(rkeys, (const float*)w.vals.p, nre,
                                       cap_hint, w.selbuf,
                                       (uint64_t*)w.sel.p, st);
    rkeys = (const uint64_t*)w.sel.p;
    nre = cap_hint;
  }
  if (e == hipSuccess && out) {
    // final: fp32 re-rank and the exact top t of the re-ranked pairs
    e = launch_rerank_topk(rkeys, nre, A, B, n, d, t < nre ? t : nre, w.fin,
                           out, n_out, nullptr, st);
  }
  (void)hipEventRecord(ev[3], st);
  if (e == hipSuccess) e = hipEventSynchronize(ev[3]);
  if (e == hipSuccess && stats) {
    float f;
    (void)hipEventElapsedTime(&f, ev[0], ev[1]);
    stats->ms_screen = f;
    (void)hipEventElapsedTime(&f, ev[1], ev[2]);
    stats->ms_filter = f;
    (void)hipEventElapsedTime(&f, ev[2], ev[3]);
    stats->ms_rerank = f;
    stats->candidates = (int64_t)count;
    unsigned tb = 0;
    (void)hipMemcpy(&tb, tau_bits, 4, hipMemcpyDeviceToHost);
    float tf;
    memcpy(&tf, &tb, 4);
    stats->tau = tf;
    stats->row_stride = stride;
    stats->reranked = nre;
  }
  for (auto& x : ev) (void)hipEventDestroy(x);
  return e;
}

}  // namespace mad
