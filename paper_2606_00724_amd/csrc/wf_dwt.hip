// The staged transform wf_dwt_keys: the J-level DWT of the prompt keys along
// the sequence (eqs. 5-6), A_J alone or with the details of every level.
#include <type_traits>

#include "wf_dwt.hpp"

namespace wf {

struct GlobalSink {
  float* aout;     // approximation, unit base + 2 cp
  float* dout;     // details, unit base + 2 cp, nullable
  long n0, n1;     // level-J rows owned by the stream
  long L;
  int J, D;
  __device__ __forceinline__ void store2(float* p, F2 a) {
    *reinterpret_cast<float2*>(p) = make_float2(a.x, a.y);
  }
  __device__ __forceinline__ void approx(long n, F2 a) {
    if (n >= n0 && n < n1) store2(aout + n * D, a);
  }
  __device__ __forceinline__ void detail(int j, long n, F2 d) {
    const long lo = n0 << (J - j), hi = n1 << (J - j);
    if (dout && n >= lo && n < hi) {
      const long row = (L - (L >> (j - 1))) + n;  // D_1 rows come first
      store2(dout + row * D, d);
    }
  }
};

// ------------------------------------------------------------ staged DWT

template <int M, int J, typename T>
__global__ __launch_bounds__(kBlock) void dwt_kernel(DwtArgs a, Taps taps) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lps = a.D / 2;             // lanes per stream
  const int spw = kWave / lps;         // streams per wave
  const int cp = lane % lps;
  const int sid = wave * spw + lane / lps;
  const int u = blockIdx.x / a.ntiles;
  const int tile = blockIdx.x % a.ntiles;
  const long n0 = ((long)tile * a.streams + sid) * a.cps;
  if (u >= a.U || n0 >= a.nJ) return;  // no barrier in this kernel
  const long n1 = min(n0 + (long)a.cps, (long)a.nJ);
  const T* Kunit = reinterpret_cast<const T*>(a.K) + (long)u * a.Ls * a.D;
  GlobalSink sink;
  sink.aout = a.approx + (long)u * a.nJ * a.D + 2 * cp;
  sink.dout = a.details ? a.details + (long)u * (a.L - a.nJ) * a.D + 2 * cp
                        : nullptr;
  sink.n0 = n0;
  sink.n1 = n1;
  sink.L = a.L;
  sink.J = J;
  sink.D = a.D;
  Cascade<M, J, true> cas;
  const bool sym = (M == 4) && a.boundary == 0;
  cas.init(taps, a.L, sym);
  const long t0 = n0 << J;
  long t_stop = (n1 << J) + cascade_halo(M, J);
  if (sym || M == 2) t_stop = min(t_stop, (long)a.L);
  run_stream<M, J, true, T>(cas, Kunit, a.D, cp, t0, t_stop, a.L, sink);
}

// Haar A_J alone (no details): block sums of 2^J rows in coefficient tiles
// (the same tiles the skim builds), then copied to approx [U][nJ][D].
// Persistent grid over (unit, tile) items.
template <typename T, int D, bool STREAM>
__global__ __launch_bounds__(kBlock) void haar_approx_kernel(DwtArgs a, float inv_norm,
                                                             int cpt) {
  extern __shared__ float coef[];  // [cpt][D + kCoefPad]
  constexpr int STRIDE = D + kCoefPad;
  const int total = a.U * a.ntiles;
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int u = item / a.ntiles;
    const int tile = item % a.ntiles;
    const long n0 = (long)tile * cpt;
    const int ncoef = (int)min((long)cpt, (long)a.nJ - n0);
    const T* Kunit = reinterpret_cast<const T*>(a.K) + (long)u * a.Ls * D;
    haar_sum_tile<T, D, STREAM>(Kunit, n0, ncoef, a.J, inv_norm, coef,
                                [](long n) { return n; });
    __syncthreads();
    float* dst = a.approx + ((long)u * a.nJ + n0) * D;
    for (int v = threadIdx.x; v < ncoef * (D / 4); v += kBlock) {
      const int c = v / (D / 4), k = v % (D / 4);
      *reinterpret_cast<f32x4*>(dst + (long)c * D + 4 * k) =
          *reinterpret_cast<const f32x4*>(coef + c * STRIDE + 4 * k);
    }
    __syncthreads();
  }
}

// f_J in LDS, every tap rounded once; ends with a barrier.
template <int J>
__device__ __forceinline__ void band_taps_once(const Taps& t, float* band, double* tmp) {
  constexpr int N = 3 << J;
  build_band_taps<J>(t.gd, tmp, tmp + N);
  for (int i = threadIdx.x; i < N; i += kBlock) band[i] = (float)tmp[i];
  __syncthreads();
}

// Daubechies-2 A_J alone (no details, J <= kBandMaxJ): the banded filter and
// the symmetric-end filters, straight from registers to approx [U][nJ][D].
// Bound by the key stream; a wave takes `per` consecutive coefficients (two
// more blocks of rows are read for them), 8 to 16 loads in flight a lane,
// and with a symmetric end each unit's last workgroup has one wave per edge
// coefficient.  128K keys, 32 units, d = 128, bf16, J = 6: 1752 -> 208 us
// (5.3 TB/s, a device copy on the same card 5.2); 1.5K keys, 2 units, J = 2:
// 558 -> 5.0 us.  The serial cascade it replaces there waited for each of
// 2048 rows a stream in turn.  The error against a 64-bit transform is that
// of the cascade or less (J = 6: 9e-8 against 1.3e-7 relative).
template <typename T, int D, int J>
__global__ __launch_bounds__(kBlock, 2) void band_approx_kernel(DwtArgs a, Taps taps, EdgeTaps edge,
                                                             int per) {
  using BS = BandShape<T, D, J>;
  constexpr int CPL = BS::CPL, LPR = BS::LPR;
  __shared__ float band[3 << J];
  __shared__ float edge_lds[6 << J];
  __shared__ double tmp[6 << J];
  const int wave = threadIdx.x >> 6, csub = threadIdx.x % LPR;
  const bool sym = a.boundary == 0;
  const int item = xcd_swizzle(blockIdx.x, gridDim.x);
  const int u = item / a.ntiles, tile = item % a.ntiles;
  const T* Kunit = reinterpret_cast<const T*>(a.K) + (long)u * a.Ls * D;
  float* out = a.approx + (long)u * a.nJ * D + csub * CPL;
  auto put = [&](long n, const float (&r)[CPL]) {
#pragma unroll
    for (int e = 0; e < CPL; e += 4)
      *reinterpret_cast<f32x4*>(out + n * D + e) = f32x4{r[e], r[e + 1], r[e + 2], r[e + 3]};
  };
  // coefficients whose window ends inside the sequence
  const long n_end =
      sym ? (a.L >= band_len(J) ? min((a.L - band_len(J)) / (1L << J) + 1, (long)a.nJ) : 0L)
          : (long)a.nJ;
  if (sym && tile == a.ntiles - 1) {
    for (int i = threadIdx.x; i < (6 << J); i += kBlock) edge_lds[i] = edge.e[i];
    __syncthreads();
    const long n = n_end + wave;  // at most two
    if (n < a.nJ) edge_coef<T, D, J>(Kunit, n, a.nJ, edge_lds, RowsIdentity{}, put);
    return;
  }
  band_taps_once<J>(taps, band, tmp);
  const long c0 = ((long)tile * (kBlock / kWave) + wave) * per;
  const long c1 = min(c0 + per, n_end);
  if (c0 < c1)
    band_run<T, D, J, true, true>(Kunit, a.L, c0, c1, !sym, band, RowsIdentity{}, put);
}

// The same where a 16-byte wave load spans more than one block of 2^J rows
// (J = 1, and J = 2 of 64-channel bf16 rows): a row's lanes take one
// coefficient each time and read its 3 2^J - 2 rows (the neighbours' rows
// come from the cache).
template <typename T, int D, int J>
__global__ __launch_bounds__(kBlock) void short_band_approx_kernel(DwtArgs a, Taps taps,
                                                                   EdgeTaps edge) {
  constexpr int CPL = 16 / (int)sizeof(T), LPR = D / CPL, RPG = kBlock / LPR;
  constexpr int NT = 3 * (1 << J) - 2;  // taps of the banded filter
  __shared__ float band[3 << J];
  __shared__ float edge_lds[6 << J];
  __shared__ double tmp[6 << J];
  const bool sym = a.boundary == 0;
  for (int i = threadIdx.x; i < (6 << J); i += kBlock) edge_lds[i] = edge.e[i];
  band_taps_once<J>(taps, band, tmp);
  const int csub = threadIdx.x % LPR;
  const long total = (long)a.U * a.nJ;
  for (long c = (long)blockIdx.x * RPG + threadIdx.x / LPR; c < total;
       c += (long)gridDim.x * RPG) {
    const long u = c / a.nJ, n = c % a.nJ;
    const long r0 = n << J;
    // a window past a symmetric end: the end filter of the last rows
    const int m = (int)(a.nJ - 1 - n);
    const bool at_end = sym && r0 + NT > a.L;
    const float* f = at_end ? edge_lds + ((m * (m + 1) / 2) << J) : band;
    const int len = at_end ? (m + 1) << J : NT;
    const T* Kunit = reinterpret_cast<const T*>(a.K) + u * a.Ls * D + csub * CPL;
    u32x4 v[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const long r = r0 + k;
      const long row = r < a.L ? r : (sym ? a.L - 1L : r % a.L);
      v[k] = *reinterpret_cast<const u32x4*>(Kunit + row * D);
    }
    float acc[CPL];
#pragma unroll
    for (int e = 0; e < CPL; ++e) acc[e] = 0.f;
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      if (k < len) {
        const float t = f[k];
        if constexpr (sizeof(T) == 2) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            acc[2 * e] = fmaf(t, bf16_lo(v[k][e]), acc[2 * e]);
            acc[2 * e + 1] = fmaf(t, bf16_hi(v[k][e]), acc[2 * e + 1]);
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[e] = fmaf(t, __uint_as_float(v[k][e]), acc[e]);
        }
      }
    }
    float* dst = a.approx + c * D + csub * CPL;
#pragma unroll
    for (int e = 0; e < CPL; e += 4)
      *reinterpret_cast<f32x4*>(dst + e) =
          f32x4{acc[e], acc[e + 1], acc[e + 2], acc[e + 3]};
  }
}

// ------------------------------------------------------------ host side

template <int M, typename T>
static hipError_t dwt_dispatch(const DwtArgs& a, const Taps& taps, dim3 grid,
                               hipStream_t s) {
  switch (a.J) {
#define WF_DWT_CASE(JJ)                                                  \
  case JJ:                                                               \
    hipLaunchKernelGGL((dwt_kernel<M, JJ, T>), grid, dim3(kBlock), 0, s, \
                       a, taps);                                         \
    break;
    WF_DWT_CASE(1) WF_DWT_CASE(2) WF_DWT_CASE(3) WF_DWT_CASE(4)
    WF_DWT_CASE(5) WF_DWT_CASE(6) WF_DWT_CASE(7) WF_DWT_CASE(8)
    WF_DWT_CASE(9) WF_DWT_CASE(10)
#undef WF_DWT_CASE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// A_J of Daubechies-2 keys by the banded filter, J <= kBandMaxJ.
template <typename T, int D>
static hipError_t band_approx_launch(const wf_params& p, DwtArgs a, const Taps& taps,
                                     hipStream_t s) {
  static const EdgeTaps no_edge{};
  const bool sym = p.boundary == WF_EXT_SYMMETRIC;
  const EdgeTaps& edge = sym ? symmetric_edge_filters(a.J) : no_edge;
  auto run = [&](auto jc) -> hipError_t {
    constexpr int J = decltype(jc)::value;
    if constexpr (BandShape<T, D, J>::ok) {
      // coefficients per wave.  Blocks of 8 loads or more: two workgroups
      // fit a CU (their registers) and the pass costs rounds * (per + 2)
      // blocks of rows a wave (128K keys, J = 6: 208 us against 216 us at
      // 16 waves per CU; 51K, J = 5: 78 against 88).  Shorter blocks: 16
      // waves per CU (8K keys of 64 channels, J = 3: 25 us against 32)
      const long cus = device_cu_count();
      long per = std::max(4L, std::min(64L, ((long)a.U * a.nJ + 16 * cus - 1) / (16 * cus)));
      if ((1 << J) / BandShape<T, D, J>::RPI >= 8) {
        long best = 0;
        for (long c = 4; c <= 64; ++c) {
          const long wgs = a.U * ((a.nJ + 4 * c - 1) / (4 * c) + (sym ? 1 : 0));
          const long cost = (wgs + 2 * cus - 1) / (2 * cus) * (c + 2);
          if (best == 0 || cost < best) {
            best = cost;
            per = c;
          }
        }
      }
      const long wpw = per * (kBlock / kWave);
      a.ntiles = (int)((a.nJ + wpw - 1) / wpw) + (sym ? 1 : 0);
      hipLaunchKernelGGL((band_approx_kernel<T, D, J>), dim3((unsigned)(a.U * a.ntiles)),
                         dim3(kBlock), 0, s, a, taps, edge, (int)per);
    } else {
      constexpr int rpg = kBlock / (D / (16 / (int)sizeof(T)));
      const long want = ((long)a.U * a.nJ + rpg - 1) / rpg;
      const long blocks = std::min(want, 32L * device_cu_count());
      hipLaunchKernelGGL((short_band_approx_kernel<T, D, J>), dim3((unsigned)blocks),
                         dim3(kBlock), 0, s, a, taps, edge);
    }
    return hipGetLastError();
  };
  switch (a.J) {
    case 1: return run(std::integral_constant<int, 1>{});
    case 2: return run(std::integral_constant<int, 2>{});
    case 3: return run(std::integral_constant<int, 3>{});
    case 4: return run(std::integral_constant<int, 4>{});
    case 5: return run(std::integral_constant<int, 5>{});
    case 6: return run(std::integral_constant<int, 6>{});
    case 7: return run(std::integral_constant<int, 7>{});
    default: return hipErrorInvalidValue;
  }
}

DwtPlan plan_dwt(const wf_params& p) {
  DwtPlan d;
  const int spw = kWave / (p.head_dim / 2);
  d.streams = (kBlock / kWave) * spw;
  d.cps = std::max(1, 2048 >> p.levels);
  const long nJ = (long)p.ctx_len >> p.levels;
  const long per_tile = (long)d.streams * d.cps;
  d.ntiles = (int)((nJ + per_tile - 1) / per_tile);
  return d;
}

hipError_t launch_dwt(const wf_params& p, const void* K, float* approx,
                      float* details, hipStream_t s) {
  DwtPlan pl = plan_dwt(p);
  DwtArgs a;
  a.K = K;
  a.approx = approx;
  a.details = details;
  a.U = p.batch * p.heads;
  a.L = (int)filtered_len(p);
  a.Ls = p.ctx_len;
  a.D = p.head_dim;
  a.J = p.levels;
  a.nJ = p.ctx_len >> p.levels;
  a.cps = pl.cps;
  a.streams = pl.streams;
  a.ntiles = pl.ntiles;
  a.boundary = p.boundary;
  const Taps taps = make_taps(p.wavelet, p.levels);
  if (p.wavelet == WF_HAAR && !details) {
    // A_J is the scaled block sum: coefficient tiles at streaming rate
    const int cpt = haar_cpt(p.levels, a.U, a.nJ);
    a.ntiles = (int)((a.nJ + cpt - 1) / cpt);
    const size_t lds = (size_t)cpt * (p.head_dim + kCoefPad) * sizeof(float);
    auto run = [&](auto kern) -> hipError_t {
      int per_cu = 0;
      hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &per_cu, reinterpret_cast<const void*>(kern), kBlock, lds);
      if (e != hipSuccess) return e;
      const long total = (long)a.U * a.ntiles;
      const long cap = (long)std::max(1, per_cu) * device_cu_count();
      hipLaunchKernelGGL(kern, dim3((unsigned)std::min(total, cap)), dim3(kBlock), lds, s, a,
                         taps.inv_norm, cpt);
      return hipGetLastError();
    };
    auto of_type = [&](auto stream) -> hipError_t {
      constexpr bool S = decltype(stream)::value;
      if (p.dtype == WF_BF16)
        return p.head_dim == 128 ? run(haar_approx_kernel<bf16_t, 128, S>)
                                 : run(haar_approx_kernel<bf16_t, 64, S>);
      return p.head_dim == 128 ? run(haar_approx_kernel<float, 128, S>)
                               : run(haar_approx_kernel<float, 64, S>);
    };
    return keys_stream(p) ? of_type(std::true_type{}) : of_type(std::false_type{});
  }
  if (p.wavelet == WF_DB2 && !details && p.levels <= kBandMaxJ) {
    // A_J is one banded filter of the keys: every row read about once, where
    // the cascade below is a serial chain over 2048 rows a stream
    if (p.dtype == WF_BF16)
      return p.head_dim == 128 ? band_approx_launch<bf16_t, 128>(p, a, taps, s)
                               : band_approx_launch<bf16_t, 64>(p, a, taps, s);
    return p.head_dim == 128 ? band_approx_launch<float, 128>(p, a, taps, s)
                             : band_approx_launch<float, 64>(p, a, taps, s);
  }
  dim3 grid((unsigned)(a.U * a.ntiles));
  const bool haar = p.wavelet == WF_HAAR;
  if (p.dtype == WF_BF16)
    return haar ? dwt_dispatch<2, bf16_t>(a, taps, grid, s)
                : dwt_dispatch<4, bf16_t>(a, taps, grid, s);
  return haar ? dwt_dispatch<2, float>(a, taps, grid, s)
              : dwt_dispatch<4, float>(a, taps, grid, s);
}

hipError_t load_dwt_kernels() {
  hipFuncAttributes fa;
  return hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(haar_approx_kernel<bf16_t, 128, false>));
}

}  // namespace wf
