// The skim: perception weights of the query block over the level-J
// approximation of the keys (eq. 7), their column sums W (eq. 8) and the
// top-S coarse regions (eq. 9).
//
// Layout: one unit = one (batch, head) pair; K is [U][L][D] with channels
// contiguous.  A tile's coefficients (wf_dwt.hpp) stay in LDS: the epilogue
// multiplies them with the query block on MFMA, then writes the logits and
// per-tile row max / row sum of exponentials.  A per-unit kernel merges the
// tiles' row statistics, forms W and selects.
#include <vector>

#include "wf_dwt.hpp"

namespace wf {

// In place, every fp32 coefficient row of the tile becomes [hi x D][lo x D]
// bf16 in the same bytes: hi = bf16(c), lo = bf16(c - hi) (round to nearest
// even), so |c - hi - lo| <= 2^-17 |c|.  The whole workgroup reads, then
// writes (the halves overlap other threads' sources); it ends with a barrier.
template <int D>
__device__ void split_tile_bf16(float* coef, int ncoef) {
  constexpr int STRIDE = D + kCoefPad;
  constexpr int GPR = D / 8;  // 8-channel groups per row
  constexpr int MAXI = kMaxCoefTile * GPR / kBlock;
  uint32_t hi[MAXI][4], lo[MAXI][4];
#pragma unroll
  for (int k = 0; k < MAXI; ++k) {
    const int it = threadIdx.x + k * kBlock, row = it / GPR, grp = it % GPR;
    if (row < ncoef) {
      const float* src = coef + row * STRIDE + 8 * grp;
      const f32x4 v0 = *reinterpret_cast<const f32x4*>(src);
      const f32x4 v1 = *reinterpret_cast<const f32x4*>(src + 4);
      const float v[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        hi[k][e] = pack_bf16x2(v[2 * e], v[2 * e + 1]);
        lo[k][e] = pack_bf16x2(v[2 * e] - bf16_lo(hi[k][e]), v[2 * e + 1] - bf16_hi(hi[k][e]));
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < MAXI; ++k) {
    const int it = threadIdx.x + k * kBlock, row = it / GPR, grp = it % GPR;
    if (row < ncoef) {
      unsigned char* dst = reinterpret_cast<unsigned char*>(coef + row * STRIDE);
      *reinterpret_cast<u32x4*>(dst + 16 * grp) = u32x4{hi[k][0], hi[k][1], hi[k][2], hi[k][3]};
      *reinterpret_cast<u32x4*>(dst + 2 * D + 16 * grp) = u32x4{lo[k][0], lo[k][1], lo[k][2], lo[k][3]};
    }
  }
  __syncthreads();
}

// logits[q][n0 + c] = scale * <Q_q, coef_c> for the tile, plus per-row max
// and sum of exp over the tile's columns.
template <typename T, int D>
__device__ void skim_epilogue(const SkimTileArgs& a, int u, int tile, long n0,
                              int ncoef, const float* coef) {
  constexpr int STRIDE = D + kCoefPad;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, col = lane & 15;
  const int nqb = (a.B + 15) / 16;
  const int ncb = (ncoef + 15) / 16;
  const T* Qunit = reinterpret_cast<const T*>(a.Q) + (long)u * a.B * D;
  for (int qb = wave; qb < nqb; qb += kBlock / kWave) {
    const int qrow = min(qb * 16 + col, a.B - 1);  // clamped query row
    f32x4 acc[kMaxCoefTile / 16];
    if constexpr (sizeof(T) == 2) {
      // bf16 queries are exact; the tile holds each coefficient row as
      // [hi x D][lo x D] bf16 (split_tile_bf16), so two bf16 products give
      // the fp32 dot product to within 2^-17 of each term.  A operand: query
      // row, channels 32 s + 8 g ..; B operand: the same channels of
      // coefficient 16 cb + col.
      u32x4 qa[D / 32];
#pragma unroll
      for (int s32 = 0; s32 < D / 32; ++s32)
        qa[s32] = *reinterpret_cast<const u32x4*>(Qunit + (long)qrow * D + 32 * s32 + 8 * g);
#pragma unroll
      for (int cb = 0; cb < kMaxCoefTile / 16; ++cb) {
        acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (cb < ncb) {
          const unsigned char* crow =
              reinterpret_cast<const unsigned char*>(coef + (cb * 16 + col) * STRIDE);
#pragma unroll
          for (int s32 = 0; s32 < D / 32; ++s32) {
            const u32x4 hi = *reinterpret_cast<const u32x4*>(crow + 2 * (32 * s32 + 8 * g));
            const u32x4 lo = *reinterpret_cast<const u32x4*>(crow + 2 * D + 2 * (32 * s32 + 8 * g));
            acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, qa[s32]), __builtin_bit_cast(bf16x8, hi), acc[cb], 0, 0, 0);
            acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, qa[s32]), __builtin_bit_cast(bf16x8, lo), acc[cb], 0, 0, 0);
          }
        }
      }
    } else {
      // A operand: query row, channels [g D/4, (g+1) D/4) (fp32 products)
      float qv[D / 4];
      const T* qsrc = Qunit + (long)qrow * D + g * (D / 4);
#pragma unroll
      for (int v = 0; v < D / 16; ++v) {
        f32x4 w = *reinterpret_cast<const f32x4*>(qsrc + 4 * v);
#pragma unroll
        for (int e = 0; e < 4; ++e) qv[4 * v + e] = w[e];
      }
#pragma unroll
      for (int cb = 0; cb < kMaxCoefTile / 16; ++cb) {
        acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (cb < ncb) {
          const float* crow = coef + (cb * 16 + col) * STRIDE + g * (D / 4);
#pragma unroll
          for (int s4 = 0; s4 < D / 16; ++s4) {
            f32x4 cv = *reinterpret_cast<const f32x4*>(crow + 4 * s4);
#pragma unroll
            for (int e = 0; e < 4; ++e)
              acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(qv[4 * s4 + e], cv[e], acc[cb], 0, 0, 0);
          }
        }
      }
    }
    // lane holds logit[q = 16 qb + 4 g + i][c = 16 cb + col]
    float m[4], z[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float mx = -INFINITY;
#pragma unroll
      for (int cb = 0; cb < kMaxCoefTile / 16; ++cb) {
        const int c = cb * 16 + col;
        const bool ok = cb < ncb && c < ncoef;
        const float v = ok ? acc[cb][i] * a.scale : -INFINITY;
        acc[cb][i] = v;
        mx = fmaxf(mx, v);
      }
      m[i] = wave_max16(mx);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float s = 0.f;
#pragma unroll
      for (int cb = 0; cb < kMaxCoefTile / 16; ++cb) {
        const int c = cb * 16 + col;
        if (cb < ncb && c < ncoef) s += __expf(acc[cb][i] - m[i]);
      }
      s = wave_sum16(s);
      z[i] = s;
    }
    float* lg = a.logits + (long)u * a.B * a.nJ + n0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int q = qb * 16 + 4 * g + i;
      if (q < a.B) {
#pragma unroll
        for (int cb = 0; cb < kMaxCoefTile / 16; ++cb) {
          const int c = cb * 16 + col;
          if (cb < ncb && c < ncoef) lg[(long)q * a.nJ + c] = acc[cb][i];
        }
      }
    }
    if (col == 0) {
      float* st = a.stats + ((long)u * a.ntiles + tile) * 2 * a.B;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int q = qb * 16 + 4 * g + i;
        if (q < a.B) {
          st[q] = m[i];
          st[a.B + q] = z[i];
        }
      }
    }
  }
}

// Waves per SIMD a skim tile instance is compiled for: the banded db2 tiles
// at J = 6, 7 (d = 128, bf16) take three without spills, and with four they
// spill 19 registers (64K keys, 128 query rows, J = 6: 149.4 us a call with
// four, 145.1 with three).
constexpr int skim_tile_waves(int src, int M, int J, int elem, int D) {
  return src == kCascade && M == 4 && elem == 2 && D == 128 && (J == 6 || J == 7) ? 3 : 1;
}

template <int SRC, int M, int J, typename T, int D>
__global__ __launch_bounds__(kBlock, skim_tile_waves(SRC, M, J, (int)sizeof(T), D)) void
skim_tile_kernel(SkimTileArgs a, Taps taps, EdgeTaps edge) {
  extern __shared__ float coef[];  // [cpt][D + kCoefPad], then the banded taps
  constexpr bool kBand = SRC == kCascade && M == 4 && BandShape<T, D, J>::ok && J <= kBandMaxJ;
  float* band = coef + a.cpt * (D + kCoefPad);  // [2][3 << J], then [6 << J] edge filters
  float* edge_lds = band + 2 * (3 << J);
  if constexpr (kBand) {
    for (int i = threadIdx.x; i < (6 << J); i += kBlock) edge_lds[i] = edge.e[i];
    build_band_taps<J>(taps.g, band, band + (3 << J));  // ends with a barrier
  }
  const int total = a.U * a.ntiles;
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int u = item / a.ntiles;
    const int tile = item % a.ntiles;
    const long n0 = (long)tile * a.cpt;
    const int ncoef = (int)min((long)a.cpt, (long)a.nJ - n0);
    if constexpr (SRC == kHaarSum || SRC == kHaarStream) {
      const T* Kunit = reinterpret_cast<const T*>(a.K) + (long)u * a.Ls * D;
      if (SRC == kHaarSum && a.parent) {
        // block ids are clamped into the unit: a bad id cannot leave K
        const int32_t* par = a.parent + (long)u * a.npar;
        const long last = ((long)a.L >> a.J) - 1;
        haar_sum_tile<T, D, false>(Kunit, n0, ncoef, a.J, taps.inv_norm, coef, [=](long n) {
          return min(max(2L * par[n >> 1] + (n & 1), 0L), last);
        });
      } else {
        haar_sum_tile<T, D, SRC == kHaarStream>(Kunit, n0, ncoef, a.J, taps.inv_norm, coef,
                                                [](long n) { return n; });
      }
    } else if constexpr (SRC == kCascade) {
      const T* Kunit = reinterpret_cast<const T*>(a.K) + (long)u * a.Ls * D;
      const bool sym = M == 4 && a.boundary == 0;
      // a.L rows: the filtered keys, or on a refinement scale of the
      // recursion the gathered kept blocks (eq. 11), read across their joins
      auto transform = [&](const auto& map) {
        if constexpr (kBand) {
          // interior coefficients by the banded filter, those whose window
          // reaches a symmetric end by the end filters (a wave each)
          const long nJf = (long)a.L >> J;
          const long n_end =
              sym ? (a.L >= band_len(J) ? min((a.L - band_len(J)) / (1L << J) + 1, nJf) : 0L) : nJf;
          band_tile<T, D, J>(Kunit, a.L, n0, ncoef, n_end, !sym, band, coef, map);
          // at most two edge coefficients: wave w takes the w-th of the tile
          const long n = max(n0, n_end) + (threadIdx.x >> 6);
          if (n < n0 + ncoef) {
            using BS = BandShape<T, D, J>;
            const int csub = threadIdx.x % BS::LPR;
            edge_coef<T, D, J>(Kunit, n, nJf, edge_lds, map,
                               [&](long c, const float (&r)[BS::CPL]) {
                                 float* dst = coef + (c - n0) * (D + kCoefPad) + csub * BS::CPL;
#pragma unroll
                                 for (int k = 0; k < BS::CPL; ++k) dst[k] = r[k];
                               });
          }
        } else {
          cascade_tile<M, J, T, D>(Kunit, a.L, n0, ncoef, a.cpt, sym, taps, coef, map);
        }
      };
      if (a.parent)
        transform(RowsGathered{a.parent + (long)u * a.npar, J + 1, a.Ls - 1});
      else
        transform(RowsIdentity{});
    } else {
      // the tile of A_J rows: every load issued before the first is waited
      // for (row indices clamped, stores guarded); with bf16 queries the
      // rows go straight to the [hi x D][lo x D] layout of split_tile_bf16
      const float* src = a.approx + ((long)u * a.nJ + n0) * D;
      constexpr int GPR = D / 8;  // 8-channel groups per row
      constexpr int MAXI = kMaxCoefTile * GPR / kBlock;
      f32x4 v0[MAXI], v1[MAXI];
#pragma unroll
      for (int k = 0; k < MAXI; ++k) {
        const int it = threadIdx.x + k * kBlock, row = min(it / GPR, ncoef - 1), grp = it % GPR;
        v0[k] = *reinterpret_cast<const f32x4*>(src + (long)row * D + 8 * grp);
        v1[k] = *reinterpret_cast<const f32x4*>(src + (long)row * D + 8 * grp + 4);
      }
#pragma unroll
      for (int k = 0; k < MAXI; ++k) {
        const int it = threadIdx.x + k * kBlock, row = it / GPR, grp = it % GPR;
        if (row >= ncoef) continue;
        if constexpr (sizeof(T) == 2) {
          const float v[8] = {v0[k][0], v0[k][1], v0[k][2], v0[k][3],
                              v1[k][0], v1[k][1], v1[k][2], v1[k][3]};
          uint32_t hi[4], lo[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            hi[e] = pack_bf16x2(v[2 * e], v[2 * e + 1]);
            lo[e] = pack_bf16x2(v[2 * e] - bf16_lo(hi[e]), v[2 * e + 1] - bf16_hi(hi[e]));
          }
          unsigned char* dst = reinterpret_cast<unsigned char*>(coef + row * (D + kCoefPad));
          *reinterpret_cast<u32x4*>(dst + 16 * grp) = u32x4{hi[0], hi[1], hi[2], hi[3]};
          *reinterpret_cast<u32x4*>(dst + 2 * D + 16 * grp) = u32x4{lo[0], lo[1], lo[2], lo[3]};
        } else {
          float* dst = coef + row * (D + kCoefPad) + 8 * grp;
          *reinterpret_cast<f32x4*>(dst) = v0[k];
          *reinterpret_cast<f32x4*>(dst + 4) = v1[k];
        }
      }
    }
    __syncthreads();
    if constexpr (sizeof(T) == 2 && SRC != kFromApprox) split_tile_bf16<D>(coef, ncoef);
    skim_epilogue<T, D>(a, u, tile, n0, ncoef, coef);
    __syncthreads();
  }
}

// W_j (eq. 8) of unit u for the columns 4 j4 .. 4 j4 + 3, j4 in [j4_lo,
// j4_hi) (nJ a multiple of 4), from the query-major logits and the row
// normalisers c_q = M_q log2(e) + log2(Z_q); also into wsh when given.
template <int NT>
__device__ void skim_w_columns(const SkimSelectArgs& a, int u, const float* row_c, int j4_lo,
                               int j4_hi, float* wsh) {
  const float* lg = a.logits + (long)u * a.B * a.nJ;
  float* W = a.W + (long)u * a.nJ;
  // four adjacent columns per thread, 16 query rows of loads in flight
  constexpr int QB = 16;
  for (int j4 = j4_lo + (int)threadIdx.x; j4 < j4_hi; j4 += NT) {
    float w[4] = {0.f, 0.f, 0.f, 0.f};
    for (int q0 = 0; q0 < a.B; q0 += QB) {
      float4 v[QB];
#pragma unroll
      for (int i = 0; i < QB; ++i)
        v[i] = q0 + i < a.B ? *reinterpret_cast<const float4*>(lg + (long)(q0 + i) * a.nJ + 4 * j4)
                            : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int i = 0; i < QB; ++i) {
        if (q0 + i < a.B) {
          const float c = row_c[q0 + i];
          w[0] += __builtin_amdgcn_exp2f(fmaf(v[i].x, kLog2e, -c));
          w[1] += __builtin_amdgcn_exp2f(fmaf(v[i].y, kLog2e, -c));
          w[2] += __builtin_amdgcn_exp2f(fmaf(v[i].z, kLog2e, -c));
          w[3] += __builtin_amdgcn_exp2f(fmaf(v[i].w, kLog2e, -c));
        }
      }
    }
    *reinterpret_cast<float4*>(W + 4 * j4) = make_float4(w[0], w[1], w[2], w[3]);
    if (wsh) {
#pragma unroll
      for (int e = 0; e < 4; ++e) wsh[4 * j4 + e] = w[e];
    }
  }
}

// Per query row of unit u: c_q = M_q log2(e) + log2(Z_q) of the coarse
// logits, from the tiles' (max, sum) slices, 64 rows at a time; thread
// (part, q) = (tid / 64, tid % 64) folds slices part, part + 4, ..., and the
// four parts meet in pm / pz.
__device__ void unit_row_norms(const SkimSelectArgs& a, int u, float* row_c, float (*pm)[64],
                               float (*pz)[64]) {
  const float* st = a.stats + (long)u * a.ntiles * 2 * a.B;
  for (int qc = 0; qc < a.B; qc += 64) {
    const int q = qc + (threadIdx.x & 63), pp = threadIdx.x >> 6;
    float m = -INFINITY, z = 0.f;
    if (q < a.B) {
      constexpr int BATCH = 8;
      for (int t0 = pp; t0 < a.ntiles; t0 += 4 * BATCH) {
        float tm[BATCH], tz[BATCH];
#pragma unroll
        for (int k = 0; k < BATCH; ++k) {
          const int t = t0 + 4 * k;
          tm[k] = t < a.ntiles ? st[(long)t * 2 * a.B + q] : -INFINITY;
          tz[k] = t < a.ntiles ? st[(long)t * 2 * a.B + a.B + q] : 0.f;
        }
#pragma unroll
        for (int k = 0; k < BATCH; ++k) pair_merge(m, z, tm[k], tz[k]);
      }
    }
    pm[pp][threadIdx.x & 63] = m;
    pz[pp][threadIdx.x & 63] = z;
    __syncthreads();
    if (threadIdx.x < 64 && q < a.B) {
      float mm = pm[0][threadIdx.x], zz = pz[0][threadIdx.x];
#pragma unroll
      for (int k = 1; k < 4; ++k) pair_merge(mm, zz, pm[k][threadIdx.x], pz[k][threadIdx.x]);
      row_c[q] = fmaf(mm, kLog2e, __log2f(zz));
    }
    __syncthreads();
  }
}

// W of a wide candidate set spread over `parts` workgroups per unit (the
// loads of one workgroup per unit would leave most CUs idle): every
// workgroup merges the unit's (max, sum) slices itself, then forms W for its
// share of the columns, four adjacent columns and every query row a thread.
__global__ __launch_bounds__(kBlock) void skim_weights_kernel(SkimSelectArgs a, int parts) {
  __shared__ float row_c[WF_MAX_Q_LEN];
  __shared__ float pm[4][64], pz[4][64];
  // a unit's parts on the XCD of the token skim that wrote its logits
  const int item = xcd_swizzle(blockIdx.x, gridDim.x);
  const int u = item / parts, part = item % parts;
  unit_row_norms(a, u, row_c, pm, pz);
  const int n4 = a.nJ / 4, per = (n4 + parts - 1) / parts;
  skim_w_columns<kBlock>(a, u, row_c, part * per, min(n4, (part + 1) * per), nullptr);
}

typedef float f32x4_dword __attribute__((ext_vector_type(4), aligned(4)));
// four floats at a 4-byte aligned address, one 16-byte load
__device__ __forceinline__ float4 load4(const float* p) {
  const f32x4_dword v = *reinterpret_cast<const f32x4_dword*>(p);
  return make_float4(v[0], v[1], v[2], v[3]);
}

// The same W for a narrower candidate set (a thousand or so columns a unit),
// where a thread per four columns leaves too few threads: thread (g, c) adds
// the terms of 64 / NQG query rows (and those 64 rows on) of four adjacent
// columns, the NQG groups' partial sums meet in LDS and are added in order of
// g.  The first batch of logits is loaded before the slices are merged, so
// that the two loads overlap.  The last group of a row may reach up to three
// floats into the next row, and past the last row into the statistics that
// follow the logits in the workspace; their sums are not stored.  NQG = 16 where a
// workgroup has at most 16 groups of columns, which would leave three quarters
// of the lanes of NQG = 4 idle (16 units of 128 rows, 1024 columns: 10.9 us
// with 4, 7.6 with 16; 28 units of 32 rows, 1000 columns: 11.2 and 6.0).
template <int NQG>
__global__ __launch_bounds__(kBlock) void skim_weights_rows_kernel(SkimSelectArgs a, int parts) {
  constexpr int QB = 64 / NQG;       // query rows of one batch
  constexpr int CPW = kBlock / NQG;  // four-column groups per step
  __shared__ float row_c[WF_MAX_Q_LEN];
  __shared__ float pm[4][64], pz[4][64];
  __shared__ float4 wpart[NQG][CPW];
  const int item = xcd_swizzle(blockIdx.x, gridDim.x);
  const int u = item / parts, part = item % parts;
  const int n4 = (a.nJ + 3) / 4, per = (n4 + parts - 1) / parts;
  const int j4_lo = part * per, j4_hi = min(n4, j4_lo + per);
  const int qg = threadIdx.x / CPW, cl = threadIdx.x % CPW;
  const float* lg = a.logits + (long)u * a.B * a.nJ;
  float4 v[QB];
  auto load = [&](int j4, int q0) {
#pragma unroll
    for (int i = 0; i < QB; ++i)
      v[i] = j4 < j4_hi && q0 + i < a.B
                 ? load4(lg + (long)(q0 + i) * a.nJ + 4 * j4)
                 : make_float4(0.f, 0.f, 0.f, 0.f);
  };
  load(j4_lo + cl, QB * qg);
  unit_row_norms(a, u, row_c, pm, pz);

  float* W = a.W + (long)u * a.nJ;
  for (int s0 = j4_lo; s0 < j4_hi; s0 += CPW) {
    const int j4 = s0 + cl;
    float w[4] = {0.f, 0.f, 0.f, 0.f};
    for (int q0 = QB * qg; q0 < a.B; q0 += QB * NQG) {
      if (s0 != j4_lo || q0 != QB * qg) load(j4, q0);  // the first batch is in
#pragma unroll
      for (int i = 0; i < QB; ++i) {
        if (q0 + i < a.B) {
          // exp(l - M) / Z = 2^(l log2(e) - c)
          const float c = row_c[q0 + i];
          w[0] += __builtin_amdgcn_exp2f(fmaf(v[i].x, kLog2e, -c));
          w[1] += __builtin_amdgcn_exp2f(fmaf(v[i].y, kLog2e, -c));
          w[2] += __builtin_amdgcn_exp2f(fmaf(v[i].z, kLog2e, -c));
          w[3] += __builtin_amdgcn_exp2f(fmaf(v[i].w, kLog2e, -c));
        }
      }
    }
    wpart[qg][cl] = make_float4(w[0], w[1], w[2], w[3]);
    __syncthreads();
    if (qg == 0 && j4 < j4_hi) {
      float4 t = wpart[0][cl];
#pragma unroll
      for (int g = 1; g < NQG; ++g) {
        const float4 o = wpart[g][cl];
        t.x += o.x;
        t.y += o.y;
        t.z += o.z;
        t.w += o.w;
      }
      if ((a.nJ & 3) == 0) {
        *reinterpret_cast<float4*>(W + 4 * j4) = t;
      } else {  // units' rows of W are not 16-byte aligned
        const float tw[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (4 * j4 + e < a.nJ) W[4 * j4 + e] = tw[e];
      }
    }
    __syncthreads();
  }
}

// One workgroup per unit: merge the tiles' row statistics and form W (eq. 8),
// unless w_ready, and select the top-S regions (eq. 9).
constexpr int kSelectBlock = 1024;

__global__ __launch_bounds__(kSelectBlock) void skim_select_kernel(SkimSelectArgs a,
                                                                   int w_in_lds, int w_ready) {
  constexpr int NT = kSelectBlock;
  __shared__ float row_c[WF_MAX_Q_LEN];  // per query: M log2(e) + log2(Z)
  __shared__ float pm[16][65], pz[16][65];
  __shared__ SelectShared<NT> sh;
  extern __shared__ float wsh[];
  // the unit on the XCD whose L2 took its W (or its logits)
  const int u = xcd_swizzle(blockIdx.x, gridDim.x);
  const float* st = a.stats + (long)u * a.ntiles * 2 * a.B;
  float* W = a.W + (long)u * a.nJ;
  // candidate n is block n, or on a refinement scale child n % 2 of kept
  // block parent[n / 2]; the last scale emits the two tokens of each block
  int32_t* out = a.seg + (long)u * (a.pairs ? 2 : 1) * a.S;
  auto put = [&](uint32_t pos, int32_t id) {
    if (a.pairs) {
      out[2 * pos] = 2 * id;
      out[2 * pos + 1] = 2 * id + 1;
    } else {
      out[pos] = id;
    }
  };
  if (w_ready && a.nJ <= 8 * NT) {
    // W from skim_weights_kernel, eight scores a thread read once into
    // registers; the parent ids wait in LDS (the select's first barrier
    // orders them before any emit; n_J = 2 npar floats of LDS were sized)
    const int32_t* pg = a.parent ? a.parent + (long)u * a.npar : nullptr;
    int32_t* par_sh = reinterpret_cast<int32_t*>(wsh);
    if (pg)
      for (int i = threadIdx.x; i < a.npar; i += NT) par_sh[i] = pg[i];
    block_select_topk_regs<NT, 8>(
        W, a.nJ, a.S, [&](uint32_t pos, int n) { put(pos, pg ? 2 * par_sh[n >> 1] + (n & 1) : n); },
        sh);
    return;
  }
  if (w_ready) {
    // W was formed by skim_weights_kernel
    if (w_in_lds)
      for (int j = threadIdx.x; j < a.nJ; j += NT) wsh[j] = W[j];
  } else {
    // merge the tiles' (max, sum of exp) pairs, 64 queries at a time: thread
    // (part, q) = (tid / 64, tid % 64) folds tiles part, part + 16, ...; the 16
    // pairs of a query meet in a 16-lane row and are merged by rotations
    for (int qc = 0; qc < a.B; qc += 64) {
      {
        const int q = qc + (threadIdx.x & 63), part = threadIdx.x >> 6;
        float m = -INFINITY, z = 0.f;
        if (q < a.B) {
          constexpr int BATCH = 8;
          for (int t0 = part; t0 < a.ntiles; t0 += 16 * BATCH) {
            float tm[BATCH], tz[BATCH];
#pragma unroll
            for (int k = 0; k < BATCH; ++k) {
              const int t = t0 + 16 * k;
              tm[k] = t < a.ntiles ? st[(long)t * 2 * a.B + q] : -INFINITY;
              tz[k] = t < a.ntiles ? st[(long)t * 2 * a.B + a.B + q] : 0.f;
            }
#pragma unroll
            for (int k = 0; k < BATCH; ++k) pair_merge(m, z, tm[k], tz[k]);
          }
        }
        pm[part][threadIdx.x & 63] = m;
        pz[part][threadIdx.x & 63] = z;
      }
      __syncthreads();
      {
        const int ql = threadIdx.x >> 4, part = threadIdx.x & 15;
        float m = pm[part][ql], z = pz[part][ql];
        row16_merge<8>(m, z);
        row16_merge<4>(m, z);
        row16_merge<2>(m, z);
        row16_merge<1>(m, z);
        // exp(l - M) / Z = 2^(l log2(e) - c)
        if (part == 0 && qc + ql < a.B) row_c[qc + ql] = fmaf(m, kLog2e, __log2f(z));
      }
      __syncthreads();
    }
    const float* lg = a.logits + (long)u * a.B * a.nJ;
    if ((a.nJ & 3) == 0) {
      skim_w_columns<NT>(a, u, row_c, 0, a.nJ / 4, w_in_lds ? wsh : nullptr);
    } else {
      constexpr int RB = 16;  // rows in flight per thread
      for (int j = threadIdx.x; j < a.nJ; j += NT) {
        float w = 0.f;
        for (int q0 = 0; q0 < a.B; q0 += RB) {
          float v[RB];
#pragma unroll
          for (int i = 0; i < RB; ++i) v[i] = q0 + i < a.B ? lg[(long)(q0 + i) * a.nJ + j] : 0.f;
#pragma unroll
          for (int i = 0; i < RB; ++i)
            if (q0 + i < a.B) w += __builtin_amdgcn_exp2f(fmaf(v[i], kLog2e, -row_c[q0 + i]));
        }
        W[j] = w;
        if (w_in_lds) wsh[j] = w;
      }
    }
  }
  __syncthreads();
  const int32_t* par = a.parent ? a.parent + (long)u * a.npar : nullptr;
  auto emit = [&](uint32_t pos, int n) { put(pos, par ? 2 * par[n >> 1] + (n & 1) : n); };
  // one instance per address space of the weights
  if (w_in_lds)
    block_select_topk<kSelectBlock>(wsh, a.nJ, a.S, emit, sh);
  else
    block_select_topk<kSelectBlock>(W, a.nJ, a.S, emit, sh);
}

// ------------------------------------------------------------ host side

void db2_token_taps(int J, Db2TokenTaps* out) {
  const double r2 = std::sqrt(2.0), r3 = std::sqrt(3.0), den = 4.0 * r2;
  const double g[4] = {(1 + r3) / den, (3 + r3) / den, (3 - r3) / den, (1 - r3) / den};
  // f_1 = g, f_{j+1}[s] = sum_k g_k f_j[s - 2^j k]
  std::vector<double> f(g, g + 4);
  for (int j = 1; j < J; ++j) {
    std::vector<double> nf(f.size() + 3 * ((size_t)1 << j), 0.0);
    for (size_t s = 0; s < nf.size(); ++s)
      for (int k = 0; k < 4; ++k) {
        const long i = (long)s - ((long)k << j);
        if (i >= 0 && i < (long)f.size()) nf[s] += g[k] * f[i];
      }
    f.swap(nf);
  }
  for (int i = 0; i < (3 << 6); ++i) out->band[i] = i < (int)f.size() ? (float)f[i] : 0.f;
  const EdgeTaps& e = symmetric_edge_filters(J);
  for (int i = 0; i < (6 << 6); ++i) out->edge[i] = e.e[i];
}

// coefficients per tile at scale b of the recursion
static int rec_cpt(const wf_params& p, int b) {
  return p.wavelet == WF_HAAR ? haar_cpt(b) : kMaxCoefTile;
}

SkimPlan plan_skim(const wf_params& p, bool fused, int fine) {
  SkimPlan k;
  const int J = p.levels;
  if (!fused) {
    k.source = kFromApprox;
    k.cpt = kMaxCoefTile;
  } else if (p.wavelet == WF_HAAR) {
    k.source = keys_stream(p) ? kHaarStream : kHaarSum;
    k.cpt = fine & kFineTiles ? haar_cpt(J, (long)p.batch * p.heads, (long)p.ctx_len >> J) : haar_cpt(J);
  } else {
    k.source = kCascade;
    k.cpt = kMaxCoefTile;  // 4 (d=128) or 8 (d=64) streams of 16 or 8
  }
  const long nJ = (long)p.ctx_len >> J;
  k.ntiles = (int)((nJ + k.cpt - 1) / k.cpt);
  k.lds_bytes = ((size_t)k.cpt * (p.head_dim + kCoefPad) +
                 (k.source == kCascade ? (size_t)12 << J : 0)) * sizeof(float);
  return k;
}

template <int SRC, int M, int J, typename T, int D>
static hipError_t skim_launch_one(const SkimTileArgs& a, const Taps& taps, const EdgeTaps& edge,
                                  size_t lds, hipStream_t s) {
  auto kern = skim_tile_kernel<SRC, M, J, T, D>;
  int per_cu = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &per_cu, reinterpret_cast<const void*>(kern), kBlock, lds);
  if (e != hipSuccess) return e;
  const long total = (long)a.U * a.ntiles;
  const long cap = (long)std::max(1, per_cu) * device_cu_count();
  dim3 grid((unsigned)std::min(total, cap));
  hipLaunchKernelGGL(kern, grid, dim3(kBlock), lds, s, a, taps, edge);
  return hipGetLastError();
}

template <typename T, int D>
static hipError_t skim_dispatch(int source, const SkimTileArgs& a, const Taps& taps,
                                const EdgeTaps& edge, size_t lds, hipStream_t s) {
  if (source == kHaarSum) return skim_launch_one<kHaarSum, 2, 1, T, D>(a, taps, edge, lds, s);
  if (source == kHaarStream)
    return skim_launch_one<kHaarStream, 2, 1, T, D>(a, taps, edge, lds, s);
  if (source == kFromApprox)
    return skim_launch_one<kFromApprox, 2, 1, T, D>(a, taps, edge, lds, s);
  switch (a.J) {
#define WF_SKIM_CASE(JJ) \
  case JJ:               \
    return skim_launch_one<kCascade, 4, JJ, T, D>(a, taps, edge, lds, s);
    WF_SKIM_CASE(1) WF_SKIM_CASE(2) WF_SKIM_CASE(3) WF_SKIM_CASE(4)
    WF_SKIM_CASE(5) WF_SKIM_CASE(6) WF_SKIM_CASE(7) WF_SKIM_CASE(8)
    WF_SKIM_CASE(9) WF_SKIM_CASE(10)
#undef WF_SKIM_CASE
    default:
      return hipErrorInvalidValue;
  }
}

static hipError_t skim_tiles_common(const wf_params& p, int source, int cpt, int J,
                                    long nJ, const int32_t* parent, int npar,
                                    const void* Q, const void* K, const float* approx,
                                    float* logits, float* stats, hipStream_t s) {
  SkimTileArgs a;
  a.K = K;
  a.approx = approx;
  a.Q = Q;
  a.logits = logits;
  a.stats = stats;
  a.parent = parent;
  a.npar = npar;
  a.U = p.batch * p.heads;
  // rows transformed: the filtered keys, or for the db2 filter on a
  // refinement scale of the recursion the gathered kept blocks of 2^(J+1)
  // rows each (Haar sums read the kept blocks' halves in place)
  a.L = parent && source == kCascade ? (int)((long)npar << (J + 1)) : (int)filtered_len(p);
  a.Ls = p.ctx_len;
  a.B = p.q_len;
  a.J = J;
  a.nJ = (int)nJ;
  a.cpt = cpt;
  a.ntiles = (int)((nJ + cpt - 1) / cpt);
  a.boundary = p.boundary;
  a.scale = effective_scale(p);
  // the coefficient tile, then (cascade source) the banded filter's taps
  // and the symmetric-end filters
  const size_t lds = ((size_t)cpt * (p.head_dim + kCoefPad) +
                      (source == kCascade ? (size_t)12 << J : 0)) *
                     sizeof(float);
  const Taps taps = make_taps(p.wavelet, J);
  static const EdgeTaps no_edge{};
  const EdgeTaps& edge = source == kCascade && p.wavelet == WF_DB2 &&
                                 p.boundary == WF_EXT_SYMMETRIC && J <= kBandMaxJ
                             ? symmetric_edge_filters(J)
                             : no_edge;
  if (p.dtype == WF_BF16)
    return p.head_dim == 128 ? skim_dispatch<bf16_t, 128>(source, a, taps, edge, lds, s)
                             : skim_dispatch<bf16_t, 64>(source, a, taps, edge, lds, s);
  return p.head_dim == 128 ? skim_dispatch<float, 128>(source, a, taps, edge, lds, s)
                           : skim_dispatch<float, 64>(source, a, taps, edge, lds, s);
}

hipError_t launch_skim_tiles(const wf_params& p, bool fused, const void* Q,
                             const void* K, const float* approx, float* logits,
                             float* stats, int fine, hipStream_t s) {
  const SkimPlan pl = plan_skim(p, fused, fine);
  return skim_tiles_common(p, pl.source, pl.cpt, p.levels, (long)p.ctx_len >> p.levels,
                           nullptr, 0, Q, K, approx, logits, stats, s);
}

// W of args `a` over as many workgroups as are resident at once, two per CU of
// NQG = 4, at most 1024 columns each (the staged skim of 96 units of 512 columns,
// 16 rows: 22.3 us with 576 workgroups, 18.9 with 480)
static void launch_weights_rows(const SkimSelectArgs& a, hipStream_t s) {
  const long n4 = (a.nJ + 3) / 4, wide = (a.nJ + 1023L) / 1024;
  if ((a.nJ & 3) == 0 && a.nJ >= 4096 &&
      a.U * wide >= (a.B < 64 ? 1L : 2L) * device_cu_count()) {
    // 1024 columns a workgroup fill the chip, and fewer than 64 rows would leave
    // some of the NQG groups idle (the staged skim of 256 units of 4096 columns,
    // 16 rows: 106.5 us, with a thread per four columns 96.9)
    hipLaunchKernelGGL(skim_weights_kernel, dim3((unsigned)(a.U * wide)), dim3(kBlock), 0, s, a,
                       (int)wide);
    return;
  }
  const int parts = (int)std::min(n4, std::max(wide, 2L * device_cu_count() / a.U));
  const dim3 grid((unsigned)(a.U * parts));
  if ((n4 + parts - 1) / parts <= 16)
    hipLaunchKernelGGL(skim_weights_rows_kernel<16>, grid, dim3(kBlock), 0, s, a, parts);
  else
    hipLaunchKernelGGL(skim_weights_rows_kernel<4>, grid, dim3(kBlock), 0, s, a, parts);
}

static hipError_t skim_select_common(const wf_params& p, bool two_stage, long nJ, int ntiles, int S,
                                     const int32_t* parent, int npar, int pairs,
                                     const float* logits, const float* stats, float* W,
                                     int32_t* out, hipStream_t s) {
  SkimSelectArgs a;
  a.logits = logits;
  a.stats = stats;
  a.W = W;
  a.seg = out;
  a.parent = parent;
  a.npar = npar;
  a.pairs = pairs;
  a.U = p.batch * p.heads;
  a.B = p.q_len;
  a.nJ = (int)nJ;
  a.ntiles = ntiles;
  a.S = S;
  const int in_lds = a.nJ <= kSelectLdsFloats ? 1 : 0;
  const size_t lds = in_lds ? (size_t)a.nJ * sizeof(float) : 0;
  if (lds > 32768) {  // with the static arrays, past the default 64 KiB
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(skim_select_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  // W over all CUs first: on the two-stage path where the call has the
  // coefficients to fill the chip with it (28 units of 1914: 24.2 us in one
  // kernel, 11.7 + 7.8 in two; 32 of 512: 14.5 and 7.1 + 6.4), on the
  // recursion's scales from 4096 candidates on (1024 columns a workgroup).
  // So few rows and columns that one workgroup per unit is done with W before a
  // second kernel starts stay in one kernel, where the units fit the CUs at once
  // (the staged skim of 64 units of 256 columns, 8 rows: 15.8 us, in two kernels
  // 17.3; 8 units of 8 rows: 15.9 and 15.6).
  const bool short_w = a.nJ <= 512 && (a.B == 1 || a.U >= 8 * a.B) && a.U <= device_cu_count();
  int w_ready = 0;
  if (two_stage && wide_weights(p) && !short_w) {
    w_ready = 1;
    launch_weights_rows(a, s);
  } else if (a.nJ >= 4096 && (a.nJ & 3) == 0) {
    w_ready = 1;
    const int parts = (a.nJ + 1023) / 1024;
    hipLaunchKernelGGL(skim_weights_kernel, dim3((unsigned)(a.U * parts)), dim3(kBlock), 0, s,
                       a, parts);
  }
  hipLaunchKernelGGL(skim_select_kernel, dim3((unsigned)a.U), dim3(kSelectBlock),
                     lds, s, a, in_lds, w_ready);
  return hipGetLastError();
}

hipError_t launch_select_w(const wf_params& p, long groups, const float* W, int32_t* seg,
                           hipStream_t s) {
  if (groups < 1 || !W || !seg) return hipErrorInvalidValue;
  SkimSelectArgs a{};
  a.W = const_cast<float*>(W);
  a.seg = seg;
  a.U = (int)groups;
  a.B = p.q_len;
  a.nJ = (int)((long)p.ctx_len >> p.levels);
  a.S = p.segments;
  const int in_lds = a.nJ <= kSelectLdsFloats ? 1 : 0;
  const size_t lds = in_lds ? (size_t)a.nJ * sizeof(float) : 0;
  if (lds > 32768) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(skim_select_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(skim_select_kernel, dim3((unsigned)a.U), dim3(kSelectBlock), lds, s, a,
                     in_lds, 1);
  return hipGetLastError();
}

hipError_t launch_skim_weights(const wf_params& p, int ntiles, const float* logits,
                               const float* stats, float* W, hipStream_t s) {
  SkimSelectArgs a{};
  a.logits = logits;
  a.stats = stats;
  a.W = W;
  a.U = p.batch * p.heads;
  a.B = p.q_len;
  a.nJ = (int)((long)p.ctx_len >> p.levels);
  a.ntiles = ntiles;
  if (!logits || !stats || !W || a.nJ == 0) return hipErrorInvalidValue;
  launch_weights_rows(a, s);
  return hipGetLastError();
}

hipError_t launch_skim_select(const wf_params& p, int ntiles,
                              const float* logits, const float* stats,
                              float* W, int32_t* seg, hipStream_t s) {
  return skim_select_common(p, true, (long)p.ctx_len >> p.levels, ntiles, p.segments, nullptr,
                            0, 0, logits, stats, W, seg, s);
}

RecPlan plan_recursion(const wf_params& p, const int32_t* counts) {
  RecPlan r{};
  long n = (long)p.ctx_len >> p.levels;
  for (int b = p.levels; b >= 1; --b) {
    const int cpt = rec_cpt(p, b);
    // with token logits the statistics come from the token skim's ranges
    const int ntiles =
        rec_token_path(p) && b <= 5
            ? plan_rec_token(p, b, b == p.levels ? filtered_len(p) : n << b, b != p.levels).R
            : (int)((n + cpt - 1) / cpt);
    r.max_n = std::max(r.max_n, n);
    r.max_tiles = std::max(r.max_tiles, ntiles);
    r.max_keep = std::max(r.max_keep, (long)counts[b - 1]);
    n = 2L * counts[b - 1];
  }
  return r;
}

hipError_t launch_rec_tiles(const wf_params& p, int b, long n, const int32_t* parent,
                            int npar, const void* Q, const void* K, float* logits,
                            float* stats, hipStream_t s) {
  return skim_tiles_common(p,
                           p.wavelet != WF_HAAR            ? kCascade
                           : parent == nullptr && keys_stream(p) ? kHaarStream
                                                           : kHaarSum,
                           rec_cpt(p, b), b, n,
                           parent, npar, Q, K, nullptr, logits, stats, s);
}

hipError_t launch_rec_select(const wf_params& p, int b, long n, int keep,
                             const int32_t* parent, int npar, const float* logits,
                             const float* stats, float* W, int32_t* out, hipStream_t s) {
  const int cpt = rec_cpt(p, b);
  const int ntiles = (int)((n + cpt - 1) / cpt);
  return skim_select_common(p, false, n, ntiles, keep, parent, npar, b == 1 ? 1 : 0, logits,
                            stats, W, out, s);
}
hipError_t launch_rec_select_slices(const wf_params& p, int b, long n, int keep,
                                    const int32_t* parent, int npar, int nslices,
                                    const float* logits, const float* stats, float* W,
                                    int32_t* out, hipStream_t s) {
  return skim_select_common(p, false, n, nslices, keep, parent, npar, b == 1 ? 1 : 0, logits,
                            stats, W, out, s);
}

hipError_t load_skim_kernels() {
  hipFuncAttributes fa;
  return hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(skim_select_kernel));
}

}  // namespace wf
