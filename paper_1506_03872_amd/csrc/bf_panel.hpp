// bf_panel.hpp -- the brute force's GEMM for short vectors: each wave keeps
// its 64 (or 32) rows of A in registers for all of K and streams the columns
// of B through LDS.
//
// What bounds a GEMM of K <= 256 here is not the matrix cores but feeding
// them: with both operands of a 64 x 64 wave tile read from LDS, each MFMA
// (32 cycles) needs one 1 KB fragment, and four SIMDs then ask for all of
// the LDS's 128 bytes per cycle; bf16 and fp8 stood at 0.29 of peak.  With
// the rows of A in registers (K x 64 rows: 128 VGPRs at K = 256 in bf16) a
// fragment of B serves two MFMAs, so LDS reads take half its rate, and a
// stage is a whole column tile (32 to 128 columns, all of K): one barrier
// per 32 or more MFMAs of each wave.  fp32, whose MFMAs take 64 cycles per
// 256 bytes of operand, is not short of LDS; it gains from the finer padding
// of K (to 8 instead of 32), the conflict-free reads and the rarer barriers
// (65133 x 71567 x 150: 12.2 ms in LDS tiles, 10.4 here, 135 TFLOP/s).
//
// Both copies are stored in fragment order: the 1 KB that a wave's MFMA
// operand takes (32 vectors x one K step, 16 bytes per lane) is contiguous,
// lane by lane.  A column tile is then one contiguous run of memory, goes
// to LDS by direct 16-byte loads without passing registers, and is read
// back without bank conflicts at immediate offsets.
#pragma once

#include "bf_common.hpp"

namespace mad {

typedef int i4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));

// column blocks of 32 per tile: about 16 KB up to 8 steps, so that LDS (two
// buffers per workgroup) allows as many workgroups per CU as the registers
constexpr int panel_tile_blocks(int ns) {
  return ns <= 4 ? 4 : ns <= 16 ? 2 : 1;
}

// blocks of 32 rows per wave: two while the rows fit in 160 registers.  (fp32
// at 65,536 x 65,536, pass B with two and with one: 9.02 and 9.12 ms at 19
// steps, 9.41 and 9.61 at 20, 10.46 and 10.54 at 22, 11.53 and 11.47 at 24.
// 20 is the last step count that is built singly.)
constexpr int panel_row_blocks(int ns) { return ns <= 20 ? 2 : 1; }

// rows of A per workgroup (4 waves)
constexpr int panel_rows(int ns) { return 128 * panel_row_blocks(ns); }

// bytes [16 lane, 16 lane + 16) of dst (wave-uniform) from src (per lane)
__device__ __forceinline__ void lds_load16(const char* src, char* dst) {
  __builtin_amdgcn_global_load_lds(
      (const __attribute__((address_space(1))) void*)src,
      (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}

__device__ __forceinline__ void lds_load4(const int* src, int* dst) {
  __builtin_amdgcn_global_load_lds(
      (const __attribute__((address_space(1))) void*)src,
      (__attribute__((address_space(3))) void*)dst, 4, 0, 0);
}

// one MFMA operand per lane: step s of a block's fragments (two steps in fp8)
template <int P> struct PanelFrag { typedef bf8v T; };
template <> struct PanelFrag<kFP8> { typedef i8v T; };
template <> struct PanelFrag<kF32> { typedef f4v T; };

template <int P>
__device__ __forceinline__ typename PanelFrag<P>::T frag_at(const i4v* p,
                                                            int s) {
  if constexpr (P == kFP8) {
    const i4v x = p[2 * s * 64], y = p[(2 * s + 1) * 64];
    return __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7);
  } else {
    return __builtin_bit_cast(typename PanelFrag<P>::T, p[s * 64]);
  }
}

// c += a b over one step's coordinates (fp32: four MFMAs of two coordinates,
// one of each lane half)
template <int P>
__device__ __forceinline__ f16v panel_mma(const typename PanelFrag<P>::T& a,
                                          const typename PanelFrag<P>::T& b,
                                          f16v c, int sa, int sb) {
  if constexpr (P == kFP8) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0,
                                                           sa, 0, sb);
  } else if constexpr (P == kBF16) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], b[q], c, 0, 0, 0);
    return c;
  }
}

// NS: steps of 16 bytes per lane (bf16: 16 coordinates and one MFMA each;
// fp8: 32 coordinates, one MFMA per two steps; fp32: 8 coordinates, four
// MFMAs each).  HIST: pass A.
template <int P, int NS, bool HIST>
__global__ __launch_bounds__(256, 2) void k_gemm_panel(PanelArgs a) {
  constexpr int TB = panel_tile_blocks(NS);
  constexpr int RB = panel_row_blocks(NS);
  constexpr int NM = P == kFP8 ? NS / 2 : NS;  // operands per 32 vectors
  constexpr int kTile = TB * NS * 1024;        // bytes of a column tile
  __shared__ __attribute__((aligned(16))) char buf0[kTile];
  __shared__ __attribute__((aligned(16))) char buf1[kTile];
  __shared__ int sc0[P == kFP8 ? TB * 32 : 1];
  __shared__ int sc1[P == kFP8 ? TB * 32 : 1];
  __shared__ unsigned hist[HIST ? 2048 : 1];
  __shared__ unsigned thr_s;
  // survivors of each wave on their way to memory
  __shared__ uint64_t qkey[HIST ? 1 : 4][HIST ? 1 : 64];
  __shared__ float qval[HIST ? 1 : 4][HIST ? 1 : 64];
  const GemmArgs& g = a.g;
  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int rl = lane & 31, rg = lane >> 5;
  BoundBins bins{-1};
  if (HIST) {
    bins = bound_bins(g.maxes, g.coarse);
    for (int b = t; b < 2048; b += 256) hist[b] = 0;
    if (t == 0) thr_s = 0u;
    __syncthreads();
  }
  // |c| below `pre` is dropped at once: |c| + margin does not reach tau (pass
  // B; 1 - 2^-20 absorbs the roundings of the comparisons), or the bound
  // that g.target lower bounds counted so far lie above (pass A)
  const float tau = HIST ? 0.0f : __uint_as_float(*g.tau_bits);
  const float mg_max = HIST ? margin_max(g) : g.mg_max;
  float pre = HIST ? -mg_max : fmaf(tau, 1.0f - 0x1p-20f, -mg_max);
  // Work items (a row panel x a run of column tiles) in segment-major
  // order; each XCD takes a contiguous share, so that the workgroups of one
  // L2 stream the same columns at the same time.
  const int64_t G = gridDim.x >> 3;  // workgroups per XCD
  const int64_t xcd = blockIdx.x & 7;
  const int64_t lo = a.items * xcd / 8, hi = a.items * (xcd + 1) / 8;
  int64_t item = lo + (blockIdx.x >> 3);
  const char* Ab = (const char*)g.A;
  const char* Bb = (const char*)g.B;
  typedef typename PanelFrag<P>::T frag_t;
  frag_t fa[RB][NM];
  int sa[2] = {127, 127};
  int64_t i0 = 0, tile = 0, tend = 0;
  auto locate = [&](int64_t it) {
    const int64_t seg = it / a.panels;
    i0 = (it - seg * a.panels) * panel_rows(NS) + wv * (32 * RB);
    tile = seg * a.seg;
    tend = tile + a.seg < a.tiles_n ? tile + a.seg : a.tiles_n;
  };
  auto load_a = [&]() {
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      int64_t i = i0 + u * 32 + rl;
      i = (i < g.m_rows ? i : g.m_rows - 1) * g.a_stride_rows;
      const i4v* p = (const i4v*)(Ab + (i >> 5) * (NS * 1024)) + rg * 32 +
                     (i & 31);
#pragma unroll
      for (int s = 0; s < NM; ++s) fa[u][s] = frag_at<P>(p, s);
      if (P == kFP8) sa[u] = e8m0_of(g.ia[i].inv_s);
    }
    // the rows are waited for here (once per item), so that no wait for
    // them stands in the tile loop, where it would also wait for the next
    // tile's loads
    __builtin_amdgcn_s_waitcnt(0x0f70);
  };
  // the tile's 1 KB fragments, shared out over the four waves
  auto fetch = [&](int64_t tl, char* dst, int* sdst) {
    const char* src = Bb + tl * kTile + lane * 16;
#pragma unroll
    for (int q = 0; q < (TB * NS + 3) / 4; ++q) {
      const int f = q * 4 + wv;
      if ((TB * NS) % 4 == 0 || f < TB * NS)
        lds_load16(src + f * 1024, dst + f * 1024);
    }
    if (P == kFP8 && wv < TB / 2)
      lds_load4(a.sb + tl * (TB * 32) + wv * 64 + lane, sdst + wv * 64);
  };
  // Survivors wait in the wave's LDS queue until 64 are there, so that the
  // shared list's counter takes an atomic per 33 or more of them: one each
  // serialises at 12 ns a survivor (30,000 x 30,000 x 256 sparse columns in
  // bf16: 622 us, 388 with the queue).
  int qn = 0;
  auto flush = [&]() {
    if (qn == 0) return;
    unsigned long long at = 0;
    if (lane == 0) at = atomicAdd(g.ccount, (unsigned long long)qn);
    at = __shfl(at, 0, 64) + (unsigned)lane;
    if (lane < qn && (int64_t)at < g.ccap) {
      g.ckey[at] = qkey[wv][lane];
      g.cval[at] = qval[wv][lane];
    }
    qn = 0;
  };
  // the kept values of one block of the wave's rows x 32 columns
  auto emit = [&](const f16v (&acc)[RB], int64_t j) {
    const VecInfo vb = g.ib[j < g.n ? j : g.n - 1];
    // an opaque copy of the lane's first row: without it the 32 rows'
    // addresses are computed ahead of the tile loop and spill
    int row = 4 * rg;
    asm volatile("" : "+v"(row));
#pragma unroll
    for (int u = 0; u < RB; ++u)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float c = acc[u][e];
        bool keep = fabsf(c) >= pre;
        if (!__any(keep)) continue;
        const int64_t i = i0 + (u * 32 + 8 * (e >> 2) + (e & 3) + row);
        keep = keep && j < g.n && i < g.m_rows;
        float mg = 0.0f;
        if (keep && !g.screen)
          mg = pair_margin(g.kappa, g.onepu, g.d_f,
                           g.ia[i * g.a_stride_rows], vb);
        if (HIST) {
          if (keep) count_bounds(bins, c, mg, hist);
          continue;
        }
        keep = keep && fabsf(c) + mg >= tau;
        const uint64_t who = __ballot(keep);
        const int cnt = __popcll(who);
        if (cnt == 0) continue;
        if (qn + cnt > 64) flush();
        if (keep) {
          const int at = qn + __popcll(who & ((1ull << lane) - 1));
          qkey[wv][at] = (uint64_t)(i * g.m_key) * (uint64_t)g.n +
                         (uint64_t)j;
          qval[wv][at] = c;
        }
        qn += cnt;
      }
  };
  auto compute = [&](const char* buf, const int* sc, int64_t tl) {
    const f16v zero = {};
#pragma unroll 1
    for (int cb = 0; cb < TB; ++cb) {
      const i4v* fb = (const i4v*)(buf + cb * (NS * 1024)) + lane;
      int sb = 127;
      if (P == kFP8) sb = sc[cb * 32 + rl];
      f16v acc[RB];
      // kAhead operands are in flight ahead of the MFMAs that take them, in
      // the order written (the barriers keep it: left alone, the compiler
      // reads two fragments at a time into the same registers and waits
      // them out before each four MFMAs)
      constexpr int kAhead = P == kFP8 ? 2 : 4;
      frag_t b[kAhead];
#pragma unroll
      for (int s = 0; s < kAhead && s < NM; ++s) b[s] = frag_at<P>(fb, s);
#pragma unroll
      for (int s = 0; s < NM; ++s) {
        __builtin_amdgcn_sched_barrier(0);
        const frag_t x = b[s % kAhead];
#pragma unroll
        for (int u = 0; u < RB; ++u)
          acc[u] = panel_mma<P>(fa[u][s], x, s == 0 ? zero : acc[u], sa[u],
                                sb);
        if (s + kAhead < NM) b[s % kAhead] = frag_at<P>(fb, s + kAhead);
      }
      __builtin_amdgcn_sched_barrier(0);
      // one max of |c| over the lane's values; the per-value work runs only
      // in waves where a lane reaches `pre`
      float mx = 0.0f;
#pragma unroll
      for (int e = 0; e < 16; ++e)
#pragma unroll
        for (int u = 0; u < RB; ++u) mx = fmaxf(mx, fabsf(acc[u][e]));
      if (__any(mx >= pre)) {
        emit(acc, tl * (TB * 32) + cb * 32 + rl);
        // emit's loads end here, for the reason given in load_a
        __builtin_amdgcn_s_waitcnt(0x0f70);
      }
    }
  };
  if (item < hi) {
    locate(item);
    fetch(tile, buf0, sc0);
    load_a();
    unsigned done = 0;
    bool more = true;
    // one tile: wait for its loads, start the next tile's into the other
    // buffer (every wave has left that one at the barrier), compute
    auto step = [&](char* cur, int* icur, char* oth, int* ioth) {
      const int64_t tl = tile;
      int64_t nitem = item, ntile = tile + 1, ni0 = i0, nend = tend;
      if (ntile == tend) {
        nitem = item + G;
        if (nitem < hi) {
          const int64_t keep = i0;
          locate(nitem);
          ntile = tile;
          ni0 = i0;
          nend = tend;
          i0 = keep;
        } else {
          more = false;
        }
      }
      __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's loads
      __syncthreads();
      if (more) fetch(ntile, oth, ioth);
      compute(cur, icur, tl);
      ++done;
      if (HIST && (done & (done - 1)) == 0)
        pre = raise_bound(g, bins, mg_max, hist, &thr_s);
      if (more) {
        tile = ntile;
        tend = nend;
        i0 = ni0;
        if (nitem != item) {
          item = nitem;
          load_a();
        }
      }
    };
    while (true) {
      step(buf0, sc0, buf1, sc1);
      if (!more) break;
      step(buf1, sc1, buf0, sc0);
      if (!more) break;
    }
  }
  if (HIST) {
    __syncthreads();
    for (int b = t; b < 2048; b += 256)
      if (hist[b]) atomicAdd(&g.hist[b], hist[b]);
  } else {
    flush();
  }
}

// workgroups that a CU holds (registers and LDS)
template <int P, int NS, bool HIST>
unsigned panel_per_cu() {
  static const unsigned per_cu = [] {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &n, k_gemm_panel<P, NS, HIST>, 256, 0) != hipSuccess ||
        n < 1)
      n = 2;
    return (unsigned)n;
  }();
  return per_cu;
}

template <int P, int NS, bool HIST>
hipError_t launch_panel_one(PanelArgs a, int64_t grid, hipStream_t st) {
  const unsigned per_cu = panel_per_cu<P, NS, HIST>();
  if (grid <= 0) grid = 256 * (int64_t)per_cu;
  constexpr int TB = panel_tile_blocks(NS);
  constexpr int tn = TB * 32;
  a.tiles_n = (a.g.n + tn - 1) / tn;
  a.panels = (a.g.m_rows + panel_rows(NS) - 1) / panel_rows(NS);
  // Column tiles per item: the least of rounds x (tiles + the rows' load),
  // where a workgroup does its items one after another.  Loading the rows
  // takes about 2.5 us, a tile its MFMAs' cycles on the SIMDs it shares.
  // (Items of one tile, which the fewest rounds lose least by when each
  // workgroup has a dozen tiles, spend most of their time on the rows: pass
  // A at 1018 x 71567 x 150 in fp32 530 us, 258 by this rule.)  Up to 4096
  // columns: the workgroups of an XCD stream the same columns, 2 MB at K =
  // 256.
  constexpr int cycles =
      panel_row_blocks(NS) * TB *
      (P == kF32 ? NS * 4 * 64 : P == kFP8 ? NS / 2 * 64 : NS * 32);
  const double load = 2.5 / (cycles * (double)per_cu / 2200.0);
  double best = 0.0;
  a.seg = 1;
  for (int64_t seg = 1; seg <= 4096 / tn && seg <= a.tiles_n; ++seg) {
    const int64_t items = a.panels * ((a.tiles_n + seg - 1) / seg);
    const double cost =
        (double)((items + grid - 1) / grid) * ((double)seg + load);
    if (seg == 1 || cost < best) {
      best = cost;
      a.seg = seg;
    }
  }
  a.items = a.panels * ((a.tiles_n + a.seg - 1) / a.seg);
  k_gemm_panel<P, NS, HIST><<<(unsigned)grid, 256, 0, st>>>(a);
  return hipGetLastError();
}

template <int P, int NS>
hipError_t launch_panel_ns(const PanelArgs& a, bool hist, int64_t grid,
                           hipStream_t st) {
  return hist ? launch_panel_one<P, NS, true>(a, grid, st)
              : launch_panel_one<P, NS, false>(a, grid, st);
}

}  // namespace mad
