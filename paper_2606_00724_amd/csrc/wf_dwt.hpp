// The wavelet transform of key rows, shared by the skim tiles (coefficients
// into LDS) and the staged transform (coefficients to memory): Haar block
// sums, the Daubechies-2 banded and end filters, and the filter-bank cascade.
//
//  * Haar: the level-J approximation of block j is 2^{-J/2} times the sum of
//    its 2^J rows (the orthonormal pyramid collapses to a block sum), so a
//    wave streams rows with 16-byte loads, accumulates in fp32 registers and
//    finishes the block with cross-lane butterflies.
//  * Daubechies-2, J <= 7: one banded filter of the rows (below).
//  * Daubechies-2 past J = 7, and the staged transform that also returns
//    details: every lane owns two channels and runs the filter-bank cascade
//    along the sequence, level by level, with three samples of state per
//    level; the half-sample symmetric extension is applied per level at the
//    true end.
#pragma once

#include <mutex>
#include <vector>

#include "wf_device.hpp"
#include "wf_kernels.hpp"
#include "wf_launch.hpp"

namespace wf {

struct Taps {
  float g[4];
  float h[4];
  float inv_norm;  // 2^{-J/2}, for the Haar block sum
  double gd[4];    // the db2 low-pass taps
};

struct F2 {
  float x, y;
};

__device__ __forceinline__ F2 load_pair(const bf16_t* p) {
  uint32_t w = *reinterpret_cast<const uint32_t*>(p);
  return F2{bf16_lo(w), bf16_hi(w)};
}
__device__ __forceinline__ F2 load_pair(const float* p) {
  u32x2 w = *reinterpret_cast<const u32x2*>(p);
  return F2{__uint_as_float(w[0]), __uint_as_float(w[1])};
}

// ------------------------------------------------------------ cascade

// Filter-bank cascade over one stream of rows for one channel pair.  Level j
// (1..J) consumes samples y^{j-1}[i] in increasing i and, after every odd i,
// emits y^j[n] = sum_m g_m y^{j-1}[2n+m] (and the detail with h), with
// n = (i - (M-1)) / 2.  Samples pushed before the stream's first aligned
// coefficient produce emissions with smaller indices, which sinks ignore.
template <int M, int J, bool DET>
struct Cascade {
  F2 s1[J + 1], s2[J + 1], s3[J + 1];  // y[i-1], y[i-2], y[i-3] per level
  float g0, g1, g2, g3, h0, h1, h2, h3;
  long L;
  bool symmetric;

  __device__ void init(const Taps& t, long L_, bool sym) {
    g0 = t.g[0]; g1 = t.g[1]; g2 = t.g[2]; g3 = t.g[3];
    h0 = t.h[0]; h1 = t.h[1]; h2 = t.h[2]; h3 = t.h[3];
    L = L_;
    symmetric = sym;
#pragma unroll
    for (int j = 0; j <= J; ++j) {
      s1[j] = F2{0.f, 0.f};
      s2[j] = F2{0.f, 0.f};
      s3[j] = F2{0.f, 0.f};
    }
  }

  template <int j, class Sink>
  __device__ __forceinline__ void feed(long i, F2 v, Sink& sink) {
    if (i & 1) {
      long n;
      F2 a, d;
      if constexpr (M == 2) {
        n = (i - 1) >> 1;
        a.x = g0 * s1[j].x + g1 * v.x;
        a.y = g0 * s1[j].y + g1 * v.y;
        if constexpr (DET) {
          d.x = h0 * s1[j].x + h1 * v.x;
          d.y = h0 * s1[j].y + h1 * v.y;
        }
      } else {
        n = (i - 3) >> 1;
        a.x = g0 * s3[j].x + g1 * s2[j].x + g2 * s1[j].x + g3 * v.x;
        a.y = g0 * s3[j].y + g1 * s2[j].y + g2 * s1[j].y + g3 * v.y;
        if constexpr (DET) {
          d.x = h0 * s3[j].x + h1 * s2[j].x + h2 * s1[j].x + h3 * v.x;
          d.y = h0 * s3[j].y + h1 * s2[j].y + h2 * s1[j].y + h3 * v.y;
        }
      }
      if constexpr (DET) sink.detail(j, n, d);
      if constexpr (j < J) {
        push<j + 1>(n, a, sink);
      } else {
        sink.approx(n, a);
      }
    }
    s3[j] = s2[j];
    s2[j] = s1[j];
    s1[j] = v;
  }

  // Pushes y^{j-1}[i].  After the last sample of a level (i = N - 1) the
  // symmetric mode continues with y[N] = y[N-1] and y[N+1] = y[N-2]
  // (half-sample symmetric extension); a loop keeps one copy of the deeper
  // levels' code.
  template <int j, class Sink>
  __device__ __forceinline__ void push(long i, F2 v, Sink& sink) {
    int reps = 1;
    const F2 prev = s1[j];
    if constexpr (M == 4) {
      if (symmetric && i == (L >> (j - 1)) - 1) reps = 3;
    }
#pragma unroll 1
    for (int r = 0; r < reps; ++r) {
      const F2 x = (r == 2) ? prev : v;
      feed<j>(i + r, x, sink);
    }
  }
};

// Rows a stream reads past its own 2^J-aligned range: level-J coefficient n
// of a 4-tap bank depends on rows 2^J n .. 2^J n + 3 (2^J - 1), so the last
// owned coefficient needs 2^{J+1} - 2 extra rows; a 2-tap bank needs none.
__host__ __device__ constexpr long cascade_halo(int M, int J) {
  return M == 4 ? (2L << J) - 2 : 0;
}

// Row t of the sequence a tile transforms: the unit's key row t, or on a
// refinement scale of the recursion row t of the gathered kept blocks
// (parent [npar] ids of 2^shift rows each; ids are clamped into the unit).
struct RowsIdentity {
  __device__ __forceinline__ long operator()(long t) const { return t; }
};
struct RowsGathered {
  const int32_t* par;
  int shift;
  long last;
  __device__ __forceinline__ long operator()(long t) const {
    const long r = ((long)par[t >> shift] << shift) | (t & ((1L << shift) - 1));
    return min(max(r, 0L), last);
  }
};

// Streams rows [t0, t_stop) of one unit into the cascade (periodic extension
// reads row t mod L), 16 loads in flight per lane.
template <int M, int J, bool DET, typename T, class Sink, class RowMap = RowsIdentity>
__device__ void run_stream(Cascade<M, J, DET>& cas, const T* Kunit, int D,
                           int cp, long t0, long t_stop, long L, Sink& sink,
                           const RowMap& map = RowMap{}) {
  constexpr int U = 16;
  for (long t = t0; t < t_stop; t += U) {
    F2 v[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      long tt = t + k;
      if (tt < t_stop) {
        long row = tt < L ? tt : tt % L;
        v[k] = load_pair(Kunit + map(row) * D + 2 * cp);
      } else {
        v[k] = F2{0.f, 0.f};
      }
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      if (t + k < t_stop) cas.template push<1>(t + k, v[k], sink);
    }
  }
}

struct LdsSink {
  float* coef;  // tile base + 2 cp
  long nbase;   // coefficient index of tile row 0
  long n0, n1;  // rows owned by the stream
  int stride;
  __device__ __forceinline__ void approx(long n, F2 a) {
    if (n >= n0 && n < n1) {
      float* p = coef + (n - nbase) * stride;
      p[0] = a.x;
      p[1] = a.y;
    }
  }
  __device__ __forceinline__ void detail(int, long, F2) {}
};

// ------------------------------------------------------------ skim tiles

// Haar level-J approximation of tile rows [n0, n0 + ncoef) into LDS.
// Coefficient n covers tokens bid(n) 2^J .. bid(n) 2^J + 2^J - 1.  A wave
// sums groups of G = max(2^J, RPL) rows (RPL rows per 16-byte wave load):
// one coefficient per group, or RPL / 2^J of them reduced across lanes.
// LOADS = G / RPL loads per group (8 stands for 8 or more); small groups
// are taken 8 / LOADS at a time so that a lane always has 8 loads in flight.
// STREAM: the rows are read with the nt policy.
template <typename T, int D, int LOADS, bool STREAM, class BlockId>
__device__ void haar_sum_tile_groups(const T* Kunit, long n0, int ncoef, int J,
                                     float inv_norm, float* coef, const BlockId& bid) {
  constexpr int CPL = 16 / sizeof(T);  // channels per lane (16-byte load)
  constexpr int LPR = D / CPL;         // lanes per row
  constexpr int RPL = kWave / LPR;     // rows per wave load
  constexpr int STRIDE = D + kCoefPad;
  constexpr int NW = kBlock / kWave;
  constexpr int GPI = LOADS >= 8 ? 1 : 8 / LOADS;  // groups per iteration
  constexpr int LPI = LOADS >= 8 ? 8 : LOADS;      // loads per group and batch
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rsub = lane / LPR, csub = lane % LPR;
  const int blk = 1 << J;
  const int G = blk > RPL ? blk : RPL;
  const int cpg = G / blk;                // coefficients per group
  const int red = blk < RPL ? blk : RPL;  // rows reduced across lanes
  const long rows = (long)ncoef << J;     // tile rows, in coefficient order
  const int ngroups = (int)((rows + G - 1) / G);
  const int nloads = LOADS >= 8 ? G / RPL : 1;  // batches of LPI loads per group
  for (int gb = wave; gb < ngroups; gb += NW * GPI) {
    float acc[GPI][CPL];
#pragma unroll
    for (int gi = 0; gi < GPI; ++gi)
#pragma unroll
      for (int e = 0; e < CPL; ++e) acc[gi][e] = 0.f;
    for (int i0 = 0; i0 < nloads; i0 += LPI) {
      u32x4 v[GPI][LPI];
#pragma unroll
      for (int gi = 0; gi < GPI; ++gi)
#pragma unroll
        for (int li = 0; li < LPI; ++li) {
          const int grp = gb + gi * NW;
          const long r = (long)grp * G + rsub + (long)(i0 + li) * RPL;
          if (grp < ngroups && r < rows) {
            const long t = ((long)bid(n0 + (r >> J)) << J) + (r & (blk - 1));
            const u32x4* src = reinterpret_cast<const u32x4*>(Kunit + t * D + csub * CPL);
            v[gi][li] = STREAM ? __builtin_nontemporal_load(src) : *src;
          } else {
            v[gi][li] = u32x4{0u, 0u, 0u, 0u};
          }
        }
#pragma unroll
      for (int gi = 0; gi < GPI; ++gi)
#pragma unroll
        for (int li = 0; li < LPI; ++li) {
          if constexpr (sizeof(T) == 2) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              acc[gi][2 * e] += bf16_lo(v[gi][li][e]);
              acc[gi][2 * e + 1] += bf16_hi(v[gi][li][e]);
            }
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[gi][e] += __uint_as_float(v[gi][li][e]);
          }
        }
    }
#pragma unroll
    for (int gi = 0; gi < GPI; ++gi) {
      // the red rows of a coefficient sit LPR, 2 LPR, ... lanes apart (LDS
      // permutes: with many waves resident their latency hides, where the
      // VALU lane swaps would take issue slots)
#pragma unroll
      for (int sh = 1; sh < red; sh <<= 1) {
#pragma unroll
        for (int e = 0; e < CPL; ++e) acc[gi][e] += __shfl_xor(acc[gi][e], LPR * sh);
      }
      const int grp = gb + gi * NW;
      if (grp < ngroups && rsub % red == 0) {
        const int c = grp * cpg + rsub / blk;
        if (c < ncoef) {
          float* dst = coef + c * STRIDE + csub * CPL;
#pragma unroll
          for (int e = 0; e < CPL; ++e) dst[e] = acc[gi][e] * inv_norm;
        }
      }
    }
  }
}

template <typename T, int D, bool STREAM, class BlockId>
__device__ void haar_sum_tile(const T* Kunit, long n0, int ncoef, int J, float inv_norm,
                              float* coef, const BlockId& bid) {
  constexpr int RPL = kWave / (D / (16 / (int)sizeof(T)));
  const int blk = 1 << J;
  const int loads = (blk > RPL ? blk : RPL) / RPL;
  switch (loads) {
    case 1: haar_sum_tile_groups<T, D, 1, STREAM>(Kunit, n0, ncoef, J, inv_norm, coef, bid); break;
    case 2: haar_sum_tile_groups<T, D, 2, STREAM>(Kunit, n0, ncoef, J, inv_norm, coef, bid); break;
    case 4: haar_sum_tile_groups<T, D, 4, STREAM>(Kunit, n0, ncoef, J, inv_norm, coef, bid); break;
    default: haar_sum_tile_groups<T, D, 8, STREAM>(Kunit, n0, ncoef, J, inv_norm, coef, bid); break;
  }
}

// Cascade level-J approximation of tile rows [n0, n0 + ncoef) into LDS.
// The tile is split into one stream per half/whole wave.
template <int M, int J, typename T, int D, class RowMap>
__device__ void cascade_tile(const T* Kunit, long L, long n0, int ncoef,
                             int cpt, bool sym, const Taps& taps,
                             float* coef, const RowMap& map) {
  constexpr int LPS = D / 2;
  constexpr int SPW = kWave / LPS;
  constexpr int NSTREAM = (kBlock / kWave) * SPW;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int cp = lane % LPS;
  const int sid = wave * SPW + lane / LPS;
  const int cps = cpt / NSTREAM;
  const long s0 = n0 + (long)sid * cps;
  const long s1 = min(s0 + (long)cps, n0 + (long)ncoef);
  if (s0 >= s1) return;
  LdsSink sink;
  sink.coef = coef + 2 * cp;
  sink.nbase = n0;
  sink.n0 = s0;
  sink.n1 = s1;
  sink.stride = D + kCoefPad;
  Cascade<M, J, false> cas;
  cas.init(taps, L, sym);
  const long t0 = s0 << J;
  long t_stop = (s1 << J) + cascade_halo(M, J);
  if (sym || M == 2) t_stop = min(t_stop, L);
  run_stream<M, J, false, T>(cas, Kunit, D, cp, t0, t_stop, L, sink, map);
}

// ------------------------------------------------------------ banded filter

// Away from the end of the sequence the level-J approximation of a 4-tap
// bank is one banded filter: A_J[n] = sum_m f_J[m] y0[2^J n + m] with
// f_1 = g and f_{j+1}[s] = sum_k g_k f_j[s - 2^j k] (length 3 (2^J - 1) + 1).
// With the symmetric extension the per-level extensions do not compose, so
// the filter is exact only while 2^J n + 3 (2^J - 1) < L; the periodic
// extension composes (even lengths), with rows read modulo L.
__host__ __device__ constexpr int band_len(int J) { return 3 * ((1 << J) - 1) + 1; }

// Rows a 16-byte wave load covers and whether the banded fill applies: every
// load must lie inside one 2^J-row block.
template <typename T, int D, int J>
struct BandShape {
  static constexpr int CPL = 16 / (int)sizeof(T);  // channels per lane
  static constexpr int LPR = D / CPL;              // lanes per row
  static constexpr int RPI = kWave / LPR;          // rows per load
  static constexpr bool ok = (1 << J) >= RPI;
};

// f_J into taps[0 .. 3 2^J) (zero past its length), built in LDS by the
// whole workgroup from the 4 low-pass taps; tmp is scratch of as many R.
// R = double rounds every tap once.
template <int J, typename R>
__device__ void build_band_taps(const R (&g)[4], R* taps, R* tmp) {
  constexpr int N = 3 << J;
  R* cur = (J % 2 == 1) ? taps : tmp;  // f_1 lands where f_J ends up
  for (int i = threadIdx.x; i < N; i += kBlock) cur[i] = i < 4 ? g[i] : R(0);
  __syncthreads();
  for (int j = 1; j < J; ++j) {
    R* nxt = cur == taps ? tmp : taps;
    const int step = 1 << j;
    for (int i = threadIdx.x; i < N; i += kBlock) {
      R v = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int src = i - step * k;
        if (src >= 0) v += g[k] * cur[src];
      }
      nxt[i] = v;
    }
    __syncthreads();
    cur = nxt;
  }
}

// Sum of v over the lanes l ^ sh, sh = LPR .. 32 (the RPI rows of a load).
template <int LPR>
__device__ __forceinline__ float sum_rows(float v) {
  if constexpr (LPR <= 8)
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, false));
  if constexpr (LPR <= 16) v = add_xor16(v);
  v = add_xor32(v);
  return v;
}

// Level-J approximation of coefficients [c0, c1) by the banded filter, by
// the calling wave: it streams their rows once.  At block b a lane adds its
// row's contribution to coefficients b, b - 1, b - 2 (taps o, o + 2^J,
// o + 2^(J+1) at offset o in the block); when block b + 1 starts,
// coefficient b - 2 is complete, its RPI row lanes are summed and the lanes
// of row 0 call put(n, values) with their CPL channels.
// AHEAD takes batches of eight loads whatever the block's length and keeps
// the next one in flight while one is added up (56 more registers; in the
// skim tiles, four or eight waves a CU deep already, short blocks' batches
// of eight measured slower: db2 J = 2, 4K keys, 61.5 -> 65.3 us a call).
// STREAM: the rows are read with the nt policy.
template <typename T, int D, int J, bool AHEAD, bool STREAM, class RowMap, class Put>
__device__ __forceinline__ void band_run(const T* Kunit, long L, long c0, long c1, bool periodic,
                                         const float* taps, const RowMap& map, const Put& put) {
  using BS = BandShape<T, D, J>;
  constexpr int CPL = BS::CPL, LPR = BS::LPR, RPI = BS::RPI;
  constexpr int BLK = 1 << J;
  constexpr int GPB = BLK / RPI;  // loads per block
  constexpr int BATCH = !AHEAD && GPB < 8 ? GPB : 8;  // loads per batch
  constexpr int NBB = GPB > BATCH ? GPB / BATCH : 1;  // batches per block
  constexpr int BPB = GPB < BATCH ? BATCH / GPB : 1;  // blocks per batch
  static_assert(BS::ok, "a load must stay inside one block");
  const int lane = threadIdx.x & 63;
  const int rsub = lane / LPR, csub = lane % LPR;
  float a0[CPL], a1[CPL], a2[CPL];  // coefficients b, b - 1, b - 2
#pragma unroll
  for (int e = 0; e < CPL; ++e) a0[e] = a1[e] = a2[e] = 0.f;
  auto flush = [&](long n) {
    float r[CPL];
#pragma unroll
    for (int e = 0; e < CPL; ++e) r[e] = sum_rows<LPR>(a2[e]);
    if (rsub == 0 && n >= c0 && n < c1) put(n, r);
  };
  // batches over blocks c0 .. c1 + 1 (past them the rows are loaded, in
  // bounds, and their sums dropped)
  const int nbt = (int)((c1 + 2 - c0 + BPB - 1) / BPB) * NBB;
  auto load = [&](int bi, u32x4 (&v)[BATCH]) {
    const long r0 = c0 * BLK + (long)bi * (BATCH * RPI) + rsub;
#pragma unroll
    for (int gi = 0; gi < BATCH; ++gi) {
      const long r = r0 + gi * RPI;
      // past L: wrapped (periodic) or the last row with a zero tap
      const long row = r < L ? r : (periodic ? r % L : L - 1);
      const u32x4* src = reinterpret_cast<const u32x4*>(Kunit + map(row) * D + csub * CPL);
      v[gi] = STREAM ? __builtin_nontemporal_load(src) : *src;
    }
  };
  auto add = [&](int bi, const u32x4 (&v)[BATCH]) {
    const int g0 = NBB > 1 ? (bi % NBB) * BATCH : 0;
    // opaque past four loads a block, so that the taps are read from LDS in
    // every batch: up to 48 of them kept in registers cost occupancy
    int ro = rsub;
    if constexpr (GPB > 4) asm volatile("" : "+v"(ro));
    // AHEAD: a batch's rows of a block are summed by themselves and then
    // added to the coefficients, whose running sums so round a third as often
    float s0[CPL], s1[CPL], s2[CPL];
    float(&b0)[CPL] = AHEAD ? s0 : a0;
    float(&b1)[CPL] = AHEAD ? s1 : a1;
    float(&b2)[CPL] = AHEAD ? s2 : a2;
#pragma unroll
    for (int gi = 0; gi < BATCH; ++gi) {
      if (gi % GPB == 0) {
        if (g0 == 0 && (bi > 0 || gi > 0)) {  // a block starts
          flush(c0 + (NBB > 1 ? bi / NBB : bi * BPB + gi / GPB) - 3);
#pragma unroll
          for (int e = 0; e < CPL; ++e) {
            a2[e] = a1[e];
            a1[e] = a0[e];
            a0[e] = 0.f;
          }
        }
        if constexpr (AHEAD) {
#pragma unroll
          for (int e = 0; e < CPL; ++e) s0[e] = s1[e] = s2[e] = 0.f;
        }
      }
      const int o = (g0 + gi % GPB) * RPI + ro;
      const float t0 = taps[o], t1 = taps[o + BLK], t2 = taps[o + 2 * BLK];
      float x[CPL];
      if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          x[2 * e] = bf16_lo(v[gi][e]);
          x[2 * e + 1] = bf16_hi(v[gi][e]);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = __uint_as_float(v[gi][e]);
      }
#pragma unroll
      for (int e = 0; e < CPL; ++e) {
        b0[e] = fmaf(t0, x[e], b0[e]);
        b1[e] = fmaf(t1, x[e], b1[e]);
      }
      // the filter has 3 2^J - 2 taps: a block's last two rows do not reach
      // the coefficient two blocks back, whatever they hold
      const bool none = (gi % GPB == GPB - 1 || gi == BATCH - 1) && o >= BLK - 2;
#pragma unroll
      for (int e = 0; e < CPL; ++e) b2[e] = fmaf(t2, none ? 0.f : x[e], b2[e]);
      if (AHEAD && (gi % GPB == GPB - 1 || gi == BATCH - 1)) {
#pragma unroll
        for (int e = 0; e < CPL; ++e) {
          a0[e] += s0[e];
          a1[e] += s1[e];
          a2[e] += s2[e];
        }
      }
    }
  };
  if constexpr (AHEAD) {
    u32x4 va[BATCH], vb[BATCH];
    load(0, va);
    for (int bi = 0; bi < nbt; bi += 2) {
      if (bi + 1 < nbt) load(bi + 1, vb);
      add(bi, va);
      if (bi + 1 >= nbt) break;
      if (bi + 2 < nbt) load(bi + 2, va);
      add(bi + 1, vb);
    }
  } else {
    for (int bi = 0; bi < nbt; ++bi) {
      u32x4 v[BATCH];
      load(bi, v);
      add(bi, v);
    }
  }
  flush(c0 + (NBB > 1 ? nbt / NBB : nbt * BPB) - 3);
}

// Coefficients [n0, n0 + ncoef) ∩ [0, n_end) into the LDS tile by the banded
// filter; wave w takes a contiguous run of them.
template <typename T, int D, int J, class RowMap>
__device__ void band_tile(const T* Kunit, long L, long n0, int ncoef, long n_end,
                          bool periodic, const float* taps, float* coef, const RowMap& map) {
  constexpr int CPL = BandShape<T, D, J>::CPL, LPR = BandShape<T, D, J>::LPR;
  constexpr int STRIDE = D + kCoefPad;
  constexpr int NW = kBlock / kWave;
  const int wave = threadIdx.x >> 6, csub = threadIdx.x % LPR;
  const int per = (ncoef + NW - 1) / NW;
  const long c0 = n0 + (long)wave * per;
  const long c1 = min(min(c0 + (long)per, n0 + (long)ncoef), n_end);
  if (c0 >= c1) return;  // uniform per wave; no barrier follows inside
  band_run<T, D, J, false, false>(
      Kunit, L, c0, c1, periodic, taps, map, [&](long n, const float (&r)[CPL]) {
        float* dst = coef + (n - n0) * STRIDE + csub * CPL;
#pragma unroll
        for (int e = 0; e < CPL; e += 4)
          *reinterpret_cast<f32x4*>(dst + e) = f32x4{r[e], r[e + 1], r[e + 2], r[e + 3]};
      });
}

// The coefficients next to a symmetric end: coefficient nJ - 1 - m (m < 3)
// is sum_r E_m[r] y0[(nJ - 1 - m) 2^J + r], r < 2^J (m + 1).  The per-level
// extensions make E_m differ from f_J, but E_m depends only on m (lengths
// are multiples of 2^J), so the host builds the three filters once per J by
// pushing impulses through the extended cascade.  Filter m starts at
// 2^J m (m + 1) / 2.  A window of 3 2^J - 2 rows from coefficient nJ - 3 ends inside
// the sequence, so the skim tiles and the staged transform reach m < 2 only; the
// token skim's last three blocks take all three.  The banded path with edges covers
// J <= kBandMaxJ.
constexpr int kBandMaxJ = 7;
struct EdgeTaps {
  float e[6 << kBandMaxJ];
};

// Edge coefficient n by the calling wave; the lanes of row 0 call put(n,
// values) with their CPL channels.
template <typename T, int D, int J, class RowMap, class Put>
__device__ __forceinline__ void edge_coef(const T* Kunit, long n, long nJ, const float* edge,
                                          const RowMap& map, const Put& put) {
  using BS = BandShape<T, D, J>;
  constexpr int CPL = BS::CPL, LPR = BS::LPR, RPI = BS::RPI;
  constexpr int BLK = 1 << J;
  constexpr int BATCH = BLK / RPI < 8 ? BLK / RPI : 8;  // loads in flight together
  const int lane = threadIdx.x & 63;
  const int rsub = lane / LPR, csub = lane % LPR;
  const int m = (int)(nJ - 1 - n);
  const float* e = edge + BLK * (m * (m + 1) / 2);
  const int len = BLK * (m + 1);  // rows n 2^J .. L - 1
  float acc[CPL];
#pragma unroll
  for (int k = 0; k < CPL; ++k) acc[k] = 0.f;
  for (int r0 = 0; r0 < len; r0 += BATCH * RPI) {
    u32x4 v[BATCH];
#pragma unroll
    for (int i = 0; i < BATCH; ++i)
      v[i] = *reinterpret_cast<const u32x4*>(Kunit + map(n * BLK + r0 + i * RPI + rsub) * D +
                                             csub * CPL);
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const float t = e[r0 + i * RPI + rsub];
      if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          acc[2 * k] = fmaf(t, bf16_lo(v[i][k]), acc[2 * k]);
          acc[2 * k + 1] = fmaf(t, bf16_hi(v[i][k]), acc[2 * k + 1]);
        }
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] = fmaf(t, __uint_as_float(v[i][k]), acc[k]);
      }
    }
  }
#pragma unroll
  for (int k = 0; k < CPL; ++k) acc[k] = sum_rows<LPR>(acc[k]);
  if (rsub == 0) put(n, acc);
}

// ------------------------------------------------------------ host side

inline Taps make_taps(int wavelet, int J) {
  Taps t{};
  const double r2 = std::sqrt(2.0);
  if (wavelet == WF_HAAR) {
    t.g[0] = t.g[1] = (float)(1.0 / r2);
    t.h[0] = (float)(1.0 / r2);
    t.h[1] = (float)(-1.0 / r2);
  } else {
    const double r3 = std::sqrt(3.0), den = 4.0 * r2;
    const double g[4] = {(1 + r3) / den, (3 + r3) / den, (3 - r3) / den,
                         (1 - r3) / den};
    for (int m = 0; m < 4; ++m) {
      t.gd[m] = g[m];
      t.g[m] = (float)g[m];
      t.h[m] = (float)((m % 2 == 0 ? 1.0 : -1.0) * g[3 - m]);
    }
  }
  t.inv_norm = (float)std::pow(2.0, -0.5 * J);
  return t;
}

// The three symmetric-end filters of the level-J Daubechies-2 approximation
// (see EdgeTaps), in double, once per J: impulses at each of the last 3 2^J
// rows of a sequence of 6 2^J rows, through the cascade with the
// half-sample symmetric extension at every level.
inline const EdgeTaps& symmetric_edge_filters(int J) {
  static EdgeTaps table[kBandMaxJ + 1];
  static std::once_flag once[kBandMaxJ + 1];
  std::call_once(once[J], [J] {
    const double r2 = std::sqrt(2.0), r3 = std::sqrt(3.0), den = 4.0 * r2;
    const double g[4] = {(1 + r3) / den, (3 + r3) / den, (3 - r3) / den, (1 - r3) / den};
    const int blk = 1 << J, len = 6 * blk, nJ = 6;
    EdgeTaps& t = table[J];
    for (int i = 0; i < (6 << kBandMaxJ); ++i) t.e[i] = 0.f;
    for (int r = len - 3 * blk; r < len; ++r) {
      std::vector<double> y(len, 0.0);
      y[r] = 1.0;
      for (int j = 1; j <= J; ++j) {
        const int N = (int)y.size();
        std::vector<double> a(N / 2);
        for (int n = 0; n < N / 2; ++n) {
          double v = 0.0;
          for (int m = 0; m < 4; ++m) {
            const int i = 2 * n + m;
            v += g[m] * (i < N ? y[i] : y[2 * N - 1 - i]);
          }
          a[n] = v;
        }
        y.swap(a);
      }
      for (int m = 0; m < 3; ++m) {
        const int start = len - blk * (m + 1);  // first row of coefficient nJ - 1 - m
        if (r >= start) t.e[blk * (m * (m + 1) / 2) + (r - start)] = (float)y[nJ - 1 - m];
      }
    }
  });
  return table[J];
}

// Haar coefficient tile size at level J.
inline int haar_cpt(int J) { return std::min(kMaxCoefTile, std::max(16, 2048 >> J)); }

// The same for U units of nJ coefficients: halved, down to the 16 of one MFMA
// tile, while there is at most one tile per CU.  A tile's workgroup has 32 KiB
// of loads in flight, less than a CU needs, and none during its products: two
// fp32 units of 128 coefficients 11.0 -> 6.0 us, 16 bf16 units of 1024 23.8 ->
// 20.8, A_J of 32 units of 512 14.1 -> 12.1.  With more tiles than that to
// begin with (28 units of 512, J = 6) halving them costs 1.5 us, and four per
// CU cost the W kernel more slices to merge than the tiles save (8.0 -> 10.4).
inline int haar_cpt(int J, long U, long nJ) {
  int cpt = haar_cpt(J);
  while (cpt > 16 && U * ((nJ + cpt - 1) / cpt) <= device_cu_count()) cpt /= 2;
  return cpt;
}

}  // namespace wf
