// Scan: the skim's regions mapped to token indices (eq. 10) and scored at
// token resolution with the same perception-weight procedure (eqs. 7-8 over
// the pool only, Section 3.2), then the top-k tokens (eq. 9) -> mu^0.
//
// The pool of a unit is S runs of 2^J consecutive rows.  It is split into
// ranges of whole chunks (PoolShape), one workgroup each.  The softmax over
// the pool needs every chunk's row maximum and normaliser before any weight
// can be formed, so the scan runs as two passes over the chunks:
//   pass 1 (stats):   logits of the chunk on MFMA, per-row max and
//                     sum of exp -> workspace;
//   pass 2 (weights): merge the unit's row statistics, recompute the same
//                     logits (bit-identical: same code and operands), and
//                     W'_p = sum_q exp(s_qp - M_q) / Z_q for the chunk.
// A per-unit select kernel then takes the top-k of W' (ties to the lower
// pool position, which is the lower token index because the regions are
// ascending) and emits token indices in ascending order.
#include "wf_device.hpp"
#include "wf_kernels.hpp"
#include "wf_launch.hpp"

namespace wf {

// Pool rows through an LDS ring filled by direct global->LDS loads.
// Row r of the chunk at p0 is pool position min(p0 + r, plast) (rows past
// the range repeat the last valid row and are masked).
template <typename T, int D>
struct PoolRowPtr {
  const T* Kunit;
  const int32_t* segs;  // LDS: region ids from s_lo on
  long p0, plast;
  long last;            // the unit's last row (region ids are clamped to it)
  int J, mask, s_lo;
  __device__ __forceinline__ const T* operator()(int r) const {
    // row numbers fit in 32 bits (ctx_len <= 2^30)
    const int p = (int)min(p0 + r, plast);
    const int t = (segs[(p >> J) - s_lo] << J) | (p & mask);
    return Kunit + (long)min(max(t, 0), (int)last) * D;
  }
};

// The pool rows of one chunk into a ring slot, as issue_chunk, but every
// row's region id is read from LDS before the first load is issued: an LDS
// read between two of the asm loads waits out its own latency each time.
template <int CR, int G, int NW, bool STREAM, typename T, int D>
__device__ __forceinline__ void issue_pool_chunk(uint32_t lds_base,
                                                 const PoolRowPtr<T, D>& rowptr) {
  constexpr int RPI = 64 / G;
  constexpr int IPW = CR * G / (64 * NW);
  static_assert(IPW * 64 * NW == CR * G, "chunk must fill whole instructions");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned char* g[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    const int r = (wave * IPW + i) * RPI + lane / G;
    const int k = (lane % G) ^ granule_swz<G>(r);
    g[i] = reinterpret_cast<const unsigned char*>(rowptr(r)) + 16 * k;
  }
#pragma unroll
  for (int i = 0; i < IPW; ++i)
    async_load16<STREAM>(g[i], __builtin_amdgcn_readfirstlane(lds_base + 1024u * (wave * IPW + i)));
}

// 8 waves: two per SIMD, so that one wave's MFMA, exp and LDS latencies
// overlap the other's work (with one wave per SIMD the ring kernel ran at
// well under the gather rate of its memory pattern).
constexpr int kPoolBlock = 512;
constexpr int kPoolWaves = kPoolBlock / kWave;

// One running (reference, sum of 2^(logit - reference)) pair, log2 units,
// absorbs another.
__device__ __forceinline__ void stat_absorb2(float& m, float& z, float m2, float z2) {
  const float mn = fmaxf(m, m2);
  if (mn == -INFINITY) return;
  z = (m > -INFINITY ? z * __builtin_amdgcn_exp2f(m - mn) : 0.f) +
      (m2 > -INFINITY ? z2 * __builtin_amdgcn_exp2f(m2 - mn) : 0.f);
  m = mn;
}

// How far (log2 units) a logit may pass the statistics pass's running
// reference before that is raised: sums of 2^16 per term stay far from the
// ends of the fp32 range.
constexpr float kRefSlack = 16.f;
// The reference before any logit: so low that the first finite logit raises it,
// and finite, so that a logit of -inf adds 2^-inf = 0 rather than a NaN.
constexpr float kNoRef = -3.4028234663852886e38f;

// The ring kernel's shape per element type.  bf16: chunks of 128 rows, 16 of
// them a wave, every query block in every wave.  fp32: 64 rows of twice the
// bytes, 16 of them a wave pair that shares the query blocks, so that eight
// waves still hide the products' latencies.
template <typename T>
struct PoolShape {
  static constexpr bool BF = sizeof(T) == 2;
  static constexpr int CR = BF ? 128 : 64;     // pool rows per chunk
  static constexpr int QW = BF ? 1 : 2;        // waves that share a row block's queries
  static constexpr int RW = kPoolWaves / QW;   // waves over the rows
  static constexpr int QPG = BF ? 4 : 2;       // query blocks a wave holds in registers
};

// 16 x 16 logits of one query block and one row block from their 16-byte
// granules: granule 4 s + g of each row in lane group g.
template <typename T>
__device__ __forceinline__ f32x4 granule_dot(u32x4 q, u32x4 k, f32x4 acc) {
  if constexpr (sizeof(T) == 2) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, q),
                                                   __builtin_bit_cast(bf16x8, k), acc, 0, 0, 0);
  } else {
    const f32x4 qf = __builtin_bit_cast(f32x4, q), kf = __builtin_bit_cast(f32x4, k);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(qf[e], kf[e], acc, 0, 0, 0);
    return acc;
  }
}

// SEL: the workgroup first takes the unit's top-S regions from W (eq. 9) itself,
// then queues its first pool chunks.  In the
// weights pass of the token-level path it forms the pool normalisers from
// the selected blocks' log-sum-exps while they load; in the statistics pass
// (the coefficient-tile path and the step from cached coefficients) the selection is all it adds, and the
// weights pass that follows reads the region ids the unit's first range
// wrote.
template <int WEIGHTS, typename T, int D, bool SEL = false>
__global__ __launch_bounds__(kPoolBlock) void scan_ring_kernel(ScanArgs a) {
  using Shape = PoolShape<T>;
  constexpr int NW = kPoolWaves;
  constexpr int CR = Shape::CR;
  constexpr int QW = Shape::QW, RW = Shape::RW;
  constexpr int ES = (int)sizeof(T), EPV = 16 / ES;  // element size, elements per granule
  constexpr int G = D / EPV;           // 16-byte granules per row
  constexpr int CHB = CR * ES * D;     // bytes per chunk buffer
  constexpr int IPW = CR * G / (64 * NW);
  constexpr int QSTR = D + EPV;
  constexpr int TBW = CR / 16 / RW;    // token blocks per wave
  static_assert(TBW >= 1 && TBW * 16 * RW == CR, "whole 16-row blocks per wave");
  constexpr int QPG = Shape::QPG;      // query blocks held in registers
  constexpr int S32 = G / 4;           // granules of a row per lane group
  // bf16 query rows are staged in LDS; fp32 ones, twice the bytes, are read
  // from memory by each group of query blocks
  constexpr bool QLDS = Shape::BF;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* ring = smem;                                            // [nbuf][CHB]
  T* Qs = reinterpret_cast<T*>(smem + (size_t)a.nbuf * CHB);            // QLDS: [B][QSTR]
  int32_t* segs = reinterpret_cast<int32_t*>(Qs + (QLDS ? (size_t)a.B * QSTR : 0));  // [seg_cap]
  float* red = reinterpret_cast<float*>(segs + a.seg_cap);
  const int nqb = (a.B + 15) / 16;
  float* part = red;                   // [nqb][RW][16][2]
  // weights: log2 of the pool's sum of exp, per query; fp32: the reference (log2
  // units), and 1 / sum apart, as one number of the two would round a large
  // reference to its last place, and every weight with it
  float* lse2 = red + nqb * RW * 32;
  float* zinv = lse2 + a.B;                               // fp32
  float* wsum = lse2 + (Shape::BF ? a.B : 2 * a.B);  // weights: W' of the range [QW][span]

  const int item = xcd_swizzle(blockIdx.x, gridDim.x);
  const int u = item / a.C, c = item % a.C;
  const long pb = (long)c * a.span;
  const long pe = min(pb + (long)a.span, (long)a.P);
  const int nch = (int)((pe - pb + CR - 1) / CR);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, col = lane & 15;
  // the wave's rows, its share of the query blocks
  const int rw = QW == 1 ? wave : wave % RW, wq = QW == 1 ? 0 : wave / RW;

  // SEL, at most 64 query rows: the query rows are loaded into registers
  // first and written to LDS after the selection, by when they have landed;
  // more rows go to LDS before it
  const T* Qunit = reinterpret_cast<const T*>(a.Q) + (long)u * a.B * D;
  constexpr int QVR = G;                                      // 16-byte vectors per row
  constexpr int QV = (64 * QVR + kPoolBlock - 1) / kPoolBlock;  // vectors per thread
  const int qtotal = a.B * QVR;
  u32x4 qpre[QV];
  // (the selecting weights pass has at most 64)
  const bool qheld = QLDS && SEL && (WEIGHTS || a.B <= 64);
  if (qheld) {
#pragma unroll
    for (int i = 0; i < QV; ++i) {
      const int v = min(i * kPoolBlock + (int)threadIdx.x, qtotal - 1);
      qpre[i] = *reinterpret_cast<const u32x4*>(Qunit + (long)(v / QVR) * D + (v % QVR) * EPV);
    }
  } else if constexpr (QLDS) {
    stage_rows_any<T, D, kPoolBlock>(Qs, a.B, [&](int r) { return Qunit + (long)r * D; });
  }

  // region ids of this range: the span's own, or with SEL all S of the unit
  const int s_lo = SEL ? 0 : (int)(pb >> a.J);
  const uint32_t ring_lds = lds_offset(ring);
  const int nbuf = a.nbuf;
  // the pool chunk at the row pointer's p0 into the ring slot at `slot`
  auto issue = [&](const PoolRowPtr<T, D>& rows, uint32_t slot) {
    if (WEIGHTS || a.stream)
      issue_pool_chunk<CR, G, NW, true>(slot, rows);
    else
      issue_pool_chunk<CR, G, NW, false>(slot, rows);
  };
  PoolRowPtr<T, D> rp;
  rp.Kunit = reinterpret_cast<const T*>(a.K) + (long)u * a.Ls * D;
  rp.segs = segs;
  rp.plast = pe - 1;
  rp.last = a.Ls - 1;
  rp.J = a.J;
  rp.mask = (1 << a.J) - 1;
  rp.s_lo = s_lo;
  if constexpr (SEL) {
    // top-S of W: the selection's histograms in the last ring slot, and
    // past the register select's reach W in the slots before it when it
    // fits (the ring is free until the first chunks are queued below)
    unsigned char* spare = ring + (size_t)(nbuf - 1) * CHB;
    auto& sh = *reinterpret_cast<SelectShared<kPoolBlock>*>(spare);
    float* Wl = reinterpret_cast<float*>(ring);
    const int sel = u / a.share;  // the unit's selection
    const float* Wg = a.W + (long)sel * a.nJ;
    int32_t* seg_out = c == 0 && u % a.share == 0 ? a.seg_out + (long)sel * a.S : nullptr;
    auto emit = [&](uint32_t pos, int j) {
      segs[pos] = j;
      if (seg_out) seg_out[pos] = j;
    };
    constexpr int EPT = 16;  // weights per thread held in registers
    if (a.nJ <= EPT * kPoolBlock) {
      block_select_topk_regs<kPoolBlock, EPT>(Wg, a.nJ, a.S, emit, sh);
    } else {
      if (a.w_in_lds) {
        for (int i = threadIdx.x; i < a.nJ; i += kPoolBlock) Wl[i] = Wg[i];
        __syncthreads();
        block_select_topk<kPoolBlock>(Wl, a.nJ, a.S, emit, sh);
      } else {
        block_select_topk<kPoolBlock>(Wg, a.nJ, a.S, emit, sh);
      }
    }
    __syncthreads();
    // the first chunks load while the normalisers are formed (the weights
    // pass reads the pool for the last time: streaming loads)
    for (int k = 0; k < nch && k < nbuf - 1; ++k) {
      rp.p0 = pb + (long)k * CR;
      issue(rp, ring_lds + (uint32_t)(k * CHB));
    }
    if constexpr (WEIGHTS) {
      // pool normalisers (M_q, Z_q) over the pool's tokens, from the selected
      // blocks' log-sum-exps: thread (part, q) folds blocks part, part +
      // parts, ...; the parts' pairs meet in the spare slot
      const int B = a.B;
      const int parts = min(kPoolBlock / B, 16);
      float* pm = reinterpret_cast<float*>(spare);  // [parts][B + 1]
      float* pz = pm + 16 * (B + 1);
      {
        const int q = threadIdx.x % B, part = threadIdx.x / B;
        const float* lse = a.blocks + (long)u * a.nJ * 2 * B + B;  // block j: at (2 j + 1) B
        if (part < parts) {
          float mx = -INFINITY, z = 0.f;
          constexpr int BATCH = 8;  // loads in flight together
          for (int s0 = part; s0 < a.S; s0 += BATCH * parts) {
            float v[BATCH];
  #pragma unroll
            for (int k = 0; k < BATCH; ++k) {
              const int s_ = s0 + parts * k;
              v[k] = s_ < a.S ? lse[(long)segs[s_] * 2 * B + q] : -INFINITY;
            }
  #pragma unroll
            for (int k = 0; k < BATCH; ++k) stat_absorb(mx, z, v[k], 1.f);
          }
          pm[part * (B + 1) + q] = mx;
          pz[part * (B + 1) + q] = z;
        }
      }
      __syncthreads();
      for (int q = threadIdx.x; q < B; q += kPoolBlock) {
        float mx = -INFINITY, z = 0.f;
        for (int k = 0; k < parts; ++k) stat_absorb(mx, z, pm[k * (B + 1) + q], pz[k * (B + 1) + q]);
        // exp(s - M) / Z = 2^(s log2(e) - (M log2(e) + log2(Z)))
        lse2[q] = fmaf(mx, kLog2e, __log2f(z));
      }
    }
  } else {
    const int ns = (int)((pe - 1) >> a.J) - s_lo + 1;
    const int32_t* useg = a.seg + (long)(u / a.share) * a.S;  // the unit's selection
    for (int i = threadIdx.x; i < ns; i += kPoolBlock) segs[i] = useg[s_lo + i];
  }
  if (qheld) {
#pragma unroll
    for (int i = 0; i < QV; ++i) {
      const int v = i * kPoolBlock + (int)threadIdx.x;
      if (v < qtotal) *reinterpret_cast<u32x4*>(Qs + (v / QVR) * QSTR + (v % QVR) * EPV) = qpre[i];
    }
  }
  if constexpr (WEIGHTS && !SEL) {
    const float* stt = a.stats + (long)u * a.Cs * 2 * a.B;
    for (int q = threadIdx.x; q < a.B; q += kPoolBlock) {
      float mx = -INFINITY, z = 0.f;
      constexpr int SB = 8;  // slices whose loads are in flight together
      for (int k0 = 0; k0 < a.Cs; k0 += SB) {
        float mk[SB], zk[SB];
#pragma unroll
        for (int k = 0; k < SB; ++k) {
          const bool ok = k0 + k < a.Cs;
          mk[k] = ok ? stt[(long)(k0 + k) * 2 * a.B + q] : -INFINITY;
          zk[k] = ok ? stt[(long)(k0 + k) * 2 * a.B + a.B + q] : 0.f;
        }
#pragma unroll
        for (int k = 0; k < SB; ++k) stat_absorb2(mx, z, mk[k], zk[k]);
      }
      if constexpr (Shape::BF) {
        lse2[q] = mx + __log2f(z);
      } else {
        lse2[q] = mx;
        zinv[q] = 1.f / z;
      }
    }
  }
  __syncthreads();  // every regular load above has been consumed

  const float s2 = a.scale * kLog2e;
  // LDS byte offsets of the lane's key operands: the same rows of every chunk
  int boff[TBW][S32];
#pragma unroll
  for (int k = 0; k < TBW; ++k)
#pragma unroll
    for (int s = 0; s < S32; ++s) boff[k][s] = granule_offset<G>((rw * TBW + k) * 16 + col, 4 * s + g);
  // query block j of a wave in group qg is block qg + j QW + wq
  for (int qg = 0; qg < nqb; qg += QPG * QW) {
    // an fp32 range that fits the ring is in it from the first group on
    // (160 query rows in three groups, 64 units of 128 positions: the staged
    // scan 48.3 -> 44.3 us)
    const bool held = !Shape::BF && qg > 0 && nch <= nbuf;
    // query operands of this group, in registers for the whole range
    u32x4 qreg[QPG][S32];
#pragma unroll
    for (int j = 0; j < QPG; ++j) {
      const int q = min((qg + j * QW + wq) * 16 + col, a.B - 1);
      const T* arow = QLDS ? Qs + q * QSTR : Qunit + (long)q * D;
#pragma unroll
      for (int s = 0; s < S32; ++s)
        qreg[j][s] = *reinterpret_cast<const u32x4*>(arow + EPV * (4 * s + g));
    }
    // rows from memory are consumed here, so that the compiler's own wait for
    // them is not inside the loop below
    if constexpr (!QLDS) {
#pragma unroll
      for (int j = 0; j < QPG; ++j)
#pragma unroll
        for (int s = 0; s < S32; ++s) asm volatile("" ::"v"(qreg[j][s]));
    }
    // weights: the log2-domain normalisers of the lane's query rows (rows
    // past B contribute 2^-inf = 0)
    float c2[QPG][4], ci[QPG][4];
#pragma unroll
    for (int j = 0; j < QPG; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int q = (qg + j * QW + wq) * 16 + 4 * g + i;
        c2[j][i] = WEIGHTS && q < a.B ? lse2[q] : INFINITY;
        if constexpr (WEIGHTS && !Shape::BF) ci[j][i] = q < a.B ? zinv[q] : 0.f;
      }
    // statistics: a lane's reference per query row (log2 units, within
    // kRefSlack of the largest logit it has seen) and its sum of
    // 2^(logit - reference)
    float sm[QPG][4], sz[QPG][4];
#pragma unroll
    for (int j = 0; j < QPG; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sm[j][i] = kNoRef;
        sz[j][i] = 0.f;
      }
    // ring of nbuf slots, nbuf - 1 chunks in flight ahead of the one consumed.
    // The weights pass reads each pool row for the last time with the
    // streaming (nt) policy: keeping the rows cached measured slower (the
    // attention that follows loads the selected keys with nt as well).
    for (int k = 0; k < nch && k < nbuf - 1 && !(SEL && qg == 0) && !held; ++k) {
      rp.p0 = pb + (long)k * CR;
      issue(rp, ring_lds + (uint32_t)(k * CHB));
    }
    for (int ch = 0; ch < nch; ++ch) {
      const long p0 = pb + (long)ch * CR;
      const int np = (int)min((long)CR, pe - p0);
      if (!held) {
        wait_vmcnt_chunks<IPW>(min(nch - 1 - ch, nbuf - 2));
        lds_barrier();  // chunk ch visible; everyone is past chunk ch - 1
      }
      if (ch + nbuf - 1 < nch && !held) {
        rp.p0 = pb + (long)(ch + nbuf - 1) * CR;
        issue(rp, ring_lds + (uint32_t)(((ch + nbuf - 1) % nbuf) * CHB));
      }
      const unsigned char* buf = ring + (ch % nbuf) * CHB;
#pragma unroll
      for (int k = 0; k < TBW; ++k) {
        const int row = (rw * TBW + k) * 16 + col;
        const bool ok = row < np;
        u32x4 bv[S32];
#pragma unroll
        for (int s = 0; s < S32; ++s) bv[s] = *reinterpret_cast<const u32x4*>(buf + boff[k][s]);
        f32x4 acc[QPG];
#pragma unroll
        for (int j = 0; j < QPG; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (Shape::BF) {
          // the query blocks' products interleaved: independent accumulators
          // (blocks past B use clamped query rows; their results are unused)
#pragma unroll
          for (int s = 0; s < S32; ++s)
#pragma unroll
            for (int j = 0; j < QPG; ++j) acc[j] = granule_dot<T>(qreg[j][s], bv[s], acc[j]);
        } else {
          // an fp32 block takes 4 S32 products of 32 cycles: blocks past B
          // are left out (32 fp32 units, 32 queries: the two passes 17.0 + 11.3 us, without 15.3 + 9.5)
#pragma unroll
          for (int j = 0; j < QPG; ++j) {
            if (qg + j * QW + wq >= nqb) break;  // uniform
#pragma unroll
            for (int s = 0; s < S32; ++s) acc[j] = granule_dot<T>(qreg[j][s], bv[s], acc[j]);
          }
        }
        // lane holds logit[q = 16 (qg + j QW + wq) + 4 g + i][p = p0 + row]
        float wk = 0.f;
        if constexpr (!WEIGHTS) {
          // The reference need not be the maximum: it is raised, and the sum
          // rescaled, only when some lane's logit passes it by more than
          // kRefSlack (in the first block, and then rarely), so a logit costs
          // one fma and one exp2.  Raising it at every new maximum, a branch
          // and two exponentials on most lanes' paths, took this pass 45.3 us
          // on 128 units of 4096 pool rows and 64 queries, and this 43.9.
          float t[QPG][4], top = -INFINITY;
#pragma unroll
          for (int j = 0; j < QPG; ++j) {
            if (qg + j * QW + wq >= nqb) break;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              t[j][i] = ok ? fmaf(acc[j][i], s2, -sm[j][i]) : -INFINITY;
              top = fmaxf(top, t[j][i]);
            }
          }
          if (__builtin_amdgcn_ballot_w64(top > kRefSlack) != 0) {
#pragma unroll
            for (int j = 0; j < QPG; ++j) {
              if (qg + j * QW + wq >= nqb) break;
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                if (t[j][i] > kRefSlack) {
                  const float v = acc[j][i] * s2;
                  sz[j][i] *= __builtin_amdgcn_exp2f(sm[j][i] - v);  // 0 at the first logit
                  sm[j][i] = v;
                  // (fp32: v's rounding; an infinite logit counts 1)
                  t[j][i] = !Shape::BF && v < INFINITY ? fmaf(acc[j][i], s2, -v) : 0.f;
                }
              }
            }
          }
#pragma unroll
          for (int j = 0; j < QPG; ++j) {
            if (qg + j * QW + wq >= nqb) break;
#pragma unroll
            for (int i = 0; i < 4; ++i) sz[j][i] += __builtin_amdgcn_exp2f(t[j][i]);
          }
        } else {
#pragma unroll
          for (int j = 0; j < QPG; ++j) {
            if (qg + j * QW + wq >= nqb) break;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float e = __builtin_amdgcn_exp2f(fmaf(acc[j][i], s2, -c2[j][i]));
              if constexpr (Shape::BF) wk += e;
              else wk = fmaf(e, ci[j][i], wk);
            }
          }
        }
        if constexpr (WEIGHTS) {
          wk = add_xor32(add_xor16(wk));
          // query groups add up in place: the same lane owns this position
          // in every group
          float* ws = wsum + wq * a.span + (p0 - pb) + row;
          if (g == 0 && ok) *ws = (qg == 0 ? 0.f : *ws) + wk;
        }
      }
    }
    if constexpr (!WEIGHTS) {
      // merge the 16 lanes of each row (their largest reference, then the sums
      // brought to it), then the waves, through LDS.  Rows no lane has seen
      // keep (kNoRef, 0).  (Pairwise merges of the lanes, four rounds of two
      // exponentials each: 24.4 us instead of 17.2 for 16 units of 128 query
      // rows, 43.9 instead of 40.2 for 128 units of 64.)
#pragma unroll
      for (int j = 0; j < QPG; ++j) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float m = wave_max16(sm[j][i]);
          const float z = wave_sum16(sz[j][i] * __builtin_amdgcn_exp2f(sm[j][i] - m));
          const int qb = qg + j * QW + wq;
          if (col == 0 && qb < nqb) {
            part[((qb * RW + rw) * 16 + 4 * g + i) * 2] = m;
            part[((qb * RW + rw) * 16 + 4 * g + i) * 2 + 1] = z;
          }
        }
      }
    }
    lds_barrier();  // the ring is idle; `part` / `wsum` complete
  }
  if constexpr (!WEIGHTS) {
    float* stt = a.stats + ((long)u * a.Cs + c) * 2 * a.B;
    for (int q = threadIdx.x; q < a.B; q += kPoolBlock) {
      const int qb = q >> 4, r = q & 15;
      float mx = -INFINITY, z = 0.f;
#pragma unroll
      for (int w = 0; w < RW; ++w)
        stat_absorb2(mx, z, part[((qb * RW + w) * 16 + r) * 2], part[((qb * RW + w) * 16 + r) * 2 + 1]);
      stt[q] = mx;
      stt[a.B + q] = z;
    }
  } else {
    float* dst = a.wpool + (long)u * a.P + pb;
    for (int i = threadIdx.x; i < (int)(pe - pb); i += kPoolBlock)
      dst[i] = QW == 1 ? wsum[i] : wsum[i] + wsum[a.span + i];
  }
}

constexpr int kScanSelectBlock = 1024;

__global__ __launch_bounds__(kScanSelectBlock) void scan_select_kernel(ScanSelectArgs a,
                                                                       int seg_in_lds) {
  __shared__ SelectShared<kScanSelectBlock> sh;
  extern __shared__ int32_t seg_sh[];
  const int u = blockIdx.x;
  const float* W = a.wpool + (long)u * a.P;
  // the unit's region ids, read by the emits (from LDS when they fit; the
  // selection's first barrier publishes them)
  const int32_t* seg = a.seg + (long)u * a.S;
  if (seg_in_lds) {
    for (int i = threadIdx.x; i < a.S; i += kScanSelectBlock) seg_sh[i] = seg[i];
    seg = seg_sh;
  }
  const int J = a.J;
  const int mask = (1 << J) - 1;
  int32_t* tok = a.tok + (long)u * a.keff;
  auto emit = [&](uint32_t pos, int p) { tok[pos] = (seg[p >> J] << J) | (p & mask); };
  // weights in registers, eight or 16 a thread (28 units of 13184: 25.7 us
  // from LDS, 16.0 here), else from memory
  if (a.P <= 8 * kScanSelectBlock)
    block_select_topk_regs<kScanSelectBlock, 8>(W, a.P, a.keff, emit, sh);
  else if (a.P <= 16 * kScanSelectBlock)
    block_select_topk_regs<kScanSelectBlock, 16>(W, a.P, a.keff, emit, sh);
  else
    block_select_topk<kScanSelectBlock>(W, a.P, a.keff, emit, sh);
}

// ------------------------------------------------------------ host side

// LDS a workgroup may use (gfx950: 160 KiB per CU), with a little margin.
constexpr size_t kLdsBudget = 160 * 1024 - 1024;

// Most fp32 ranges of a unit: those of 1 to 8 chunks of 128 positions, about
// 1024 in all (the coarse statistics), at most twice as many where fine.
static long most_fp32_ranges(long U, long P, int fine) {
  const long chunks = (P + 127) / 128;
  const long cpw = std::max(1L, std::min(8L, U * chunks / 1024));
  return (chunks + cpw - 1) / cpw * (fine & kFineSplits ? 2 : 1);
}

ScanPlan plan_scan(const wf_params& p, bool select, int fine) {
  ScanPlan s{};
  const long P = (long)p.segments << p.levels;
  const long U = (long)p.batch * p.heads;
  const bool bf = p.dtype == WF_BF16;
  const int es = bf ? 2 : 4;
  const int cr = bf ? PoolShape<bf16_t>::CR : PoolShape<float>::CR;
  const int qw = bf ? PoolShape<bf16_t>::QW : PoolShape<float>::QW;
  const long chunks = (P + cr - 1) / cr;
  const int nqb = (p.q_len + 15) / 16;
  const size_t chb = (size_t)cr * es * p.head_dim;
  const size_t queries = bf ? (size_t)p.q_len * (p.head_dim + 8) * 2 : 0;
  // LDS beside the ring of a workgroup with `span` positions and seg_cap
  // region ids: queries, ids, wave partials, the per-query normalisers, W'
  auto beside = [&](long span, long seg_cap) {
    return queries + (size_t)seg_cap * 4 +
           ((size_t)nqb * (kPoolWaves / qw) * 16 * 2 + (size_t)(bf ? 1 : 2) * p.q_len +
            (size_t)qw * span) *
               sizeof(float);
  };
  auto slots = [&](size_t other) {
    // three slots (two chunks in flight) measured slightly faster than four
    return (int)std::min<size_t>(3, (kLdsBudget - std::min(other, kLdsBudget)) / chb);
  };
  // one workgroup per CU, each streaming a long range through the ring (at
  // most 4096 positions; no longer than ceil(CUs / U) ranges make it where
  // W' of more would leave no room for two slots).  The same ranges whether
  // or not the scan selects: both forms share their statistics.
  const long most = std::min(chunks, std::max(1L, ((long)device_cu_count() + U - 1) / U));
  const long most_cpw = std::min((chunks + most - 1) / most, 4096L / cr);
  auto fits = [&](long c) { return slots(beside(c * cr, (c * cr >> p.levels) + 2)) >= 2; };
  const long C = bf ? ranges_per_unit(U, chunks, device_cu_count(), 4096L / cr)
                    : std::max((chunks * cr + 4095) / 4096,
                               fp32_ranges_per_unit(U, chunks, device_cu_count(),
                                                    most_fp32_ranges(U, P, fine),
                                                    p.head_dim == 64 ? 1 : 2));
  long cpw = (chunks + C - 1) / C;
  if (!fits(cpw) || !fits(most_cpw)) cpw = most_cpw;
  s.span = (int)(cpw * cr);
  s.chunks = (int)((P + s.span - 1) / s.span);
  // region ids in LDS: the span's, or all S when the scan selects them
  s.seg_cap = select ? p.segments : (s.span >> p.levels) + 2;
  const size_t other = beside(s.span, s.seg_cap);
  s.nbuf = slots(other);
  s.lds_bytes = s.nbuf * chb + other;
  if (s.nbuf < 2) s.nbuf = 0;  // rejected by the caller
  return s;
}

template <class Kernel>
static hipError_t launch_with_lds(Kernel kern, dim3 grid, int block, size_t lds, hipStream_t s,
                                  const ScanArgs& a) {
  if (lds > 65536) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, grid, dim3(block), lds, s, a);
  return hipGetLastError();
}

template <int WEIGHTS, typename T, int D>
static hipError_t scan_launch(const ScanArgs& a, size_t lds, hipStream_t s) {
  const dim3 grid((unsigned)(a.U * a.C));
  return launch_with_lds(scan_ring_kernel<WEIGHTS, T, D>, grid, kPoolBlock, lds, s, a);
}

// The two-pass scan takes fp32 query blocks up to the size whose rows, beside
// 128 pool rows, fit the LDS (169 rows of 128 channels): callers see the same
// limit whatever a kernel stages.
static bool fp32_rows_fit(const wf_params& p) {
  const size_t stride = (size_t)p.head_dim * 4 + 16, nqb = (size_t)(p.q_len + 15) / 16;
  return p.dtype == WF_BF16 ||
         (p.q_len + 128) * stride + (nqb * 128 + 2 * (size_t)p.q_len) * sizeof(float) <= 160 * 1024;
}

// Whether the statistics pass reads the pool with the streaming (nt) policy.
// The weights pass reads it again: a pool that fits the L2s (4 MiB per XCD) is
// kept there for it (8 MiB: 17.2 + 9.3 us for the two passes, streamed 17.6 +
// 10.3); a larger one only displaces itself and is found in the Infinity Cache
// either way (128 MiB: 40.2 + 24.4 us kept, 31.2 + 26.4 streamed).
static int scan_streams(const wf_params& p) {
  const size_t pool = ((size_t)p.batch * p.heads * p.segments << p.levels) * p.head_dim *
                      (p.dtype == WF_BF16 ? 2 : 4);
  return pool > (size_t)32 << 20 ? 1 : 0;
}

// the scan's arguments when its workgroups take the top-S regions from W
// themselves; false when the shape does not allow it
static bool scan_select_args(const wf_params& p, const void* Q, const void* K, const float* W,
                             int32_t* seg_out, int share, int fine, ScanArgs& a, ScanPlan& pl) {
  if (p.segments > kSelectLdsSegs || share < 1 ||
      (p.batch * p.heads) % share != 0)
    return false;
  pl = plan_scan(p, true, fine);
  if (pl.nbuf < 2) return false;
  a = ScanArgs{};
  a.Q = Q;
  a.K = K;
  a.W = W;
  a.share = share;
  a.seg_out = seg_out;
  a.U = p.batch * p.heads;
  a.L = (int)filtered_len(p);
  a.Ls = p.ctx_len;
  a.B = p.q_len;
  a.J = p.levels;
  a.S = p.segments;
  a.P = p.segments << p.levels;
  a.nJ = p.ctx_len >> p.levels;
  a.C = pl.chunks;
  a.span = pl.span;
  a.nbuf = pl.nbuf;
  a.seg_cap = pl.seg_cap;
  a.stream = scan_streams(p);
  a.scale = effective_scale(p);
  // W in the ring slots before the spare one when it fits there
  const size_t chb = p.dtype == WF_BF16 ? (size_t)PoolShape<bf16_t>::CR * 2 * p.head_dim
                                        : (size_t)PoolShape<float>::CR * 4 * p.head_dim;
  a.w_in_lds = (size_t)a.nJ * sizeof(float) <= (size_t)(pl.nbuf - 1) * chb ? 1 : 0;
  return true;
}

bool scan_can_select(const wf_params& p) {
  ScanArgs a;
  ScanPlan pl;
  return scan_select_args(p, nullptr, nullptr, nullptr, nullptr, 1, kFineSplits, a, pl) &&
         scan_select_args(p, nullptr, nullptr, nullptr, nullptr, 1, 0, a, pl);
}

hipError_t launch_scan_select_weights(const wf_params& p, const void* Q, const void* K,
                                      const float* W, const float* blocks, int32_t* seg_out,
                                      float* wpool, hipStream_t s, int share) {
  ScanArgs a;
  ScanPlan pl;
  // (the pool normalisers take a thread per query row, 64 rows at most)
  if (p.dtype != WF_BF16 || p.q_len > 64 || !scan_select_args(p, Q, K, W, seg_out, share, 0, a, pl))
    return hipErrorInvalidValue;
  a.blocks = blocks;
  a.wpool = wpool;
  a.Cs = 1;
  const dim3 grid((unsigned)(a.U * a.C));
  if (p.head_dim == 128)
    return launch_with_lds(scan_ring_kernel<1, bf16_t, 128, true>, grid, kPoolBlock, pl.lds_bytes, s, a);
  return launch_with_lds(scan_ring_kernel<1, bf16_t, 64, true>, grid, kPoolBlock, pl.lds_bytes, s, a);
}

hipError_t launch_scan_select_stats(const wf_params& p, const void* Q, const void* K,
                                    const float* W, int32_t* seg_out, float* stats,
                                    int fine, hipStream_t s) {
  ScanArgs a;
  ScanPlan pl;
  if (!fp32_rows_fit(p) || !scan_select_args(p, Q, K, W, seg_out, 1, fine, a, pl))
    return hipErrorInvalidValue;
  a.stats = stats;
  a.Cs = pl.chunks;
  const dim3 grid((unsigned)(a.U * a.C));
  auto kern = [&] {
    if (p.dtype == WF_BF16)
      return p.head_dim == 128 ? scan_ring_kernel<0, bf16_t, 128, true>
                               : scan_ring_kernel<0, bf16_t, 64, true>;
    return p.head_dim == 128 ? scan_ring_kernel<0, float, 128, true>
                             : scan_ring_kernel<0, float, 64, true>;
  }();
  return launch_with_lds(kern, grid, kPoolBlock, pl.lds_bytes, s, a);
}

hipError_t launch_scan_chunks(const wf_params& p, int weights, const void* Q,
                              const void* K, const int32_t* seg, float* stats,
                              float* wpool, int fine, hipStream_t s, int share) {
  if (share < 1 || (p.batch * p.heads) % share != 0 || !fp32_rows_fit(p))
    return hipErrorInvalidValue;
  const ScanPlan pl = plan_scan(p, false, fine);
  ScanArgs a;
  a.share = share;
  a.Q = Q;
  a.K = K;
  a.seg = seg;
  a.stats = stats;
  a.wpool = wpool;
  a.U = p.batch * p.heads;
  a.L = (int)filtered_len(p);
  a.Ls = p.ctx_len;
  a.B = p.q_len;
  a.J = p.levels;
  a.S = p.segments;
  a.P = p.segments << p.levels;
  a.C = pl.chunks;
  a.Cs = pl.chunks;
  a.span = pl.span;
  a.nbuf = pl.nbuf;
  a.seg_cap = pl.seg_cap;
  a.stream = scan_streams(p);
  a.scale = effective_scale(p);
  const bool bf = p.dtype == WF_BF16, d128 = p.head_dim == 128;
  if (weights) {
    if (bf) return d128 ? scan_launch<1, bf16_t, 128>(a, pl.lds_bytes, s)
                        : scan_launch<1, bf16_t, 64>(a, pl.lds_bytes, s);
    return d128 ? scan_launch<1, float, 128>(a, pl.lds_bytes, s)
                : scan_launch<1, float, 64>(a, pl.lds_bytes, s);
  }
  if (bf) return d128 ? scan_launch<0, bf16_t, 128>(a, pl.lds_bytes, s)
                      : scan_launch<0, bf16_t, 64>(a, pl.lds_bytes, s);
  return d128 ? scan_launch<0, float, 128>(a, pl.lds_bytes, s)
              : scan_launch<0, float, 64>(a, pl.lds_bytes, s);
}

hipError_t launch_scan_select(const wf_params& p, const float* wpool,
                              const int32_t* seg, int32_t* tok,
                              hipStream_t s) {
  ScanSelectArgs a;
  a.wpool = wpool;
  a.seg = seg;
  a.tok = tok;
  a.U = p.batch * p.heads;
  a.J = p.levels;
  a.S = p.segments;
  a.P = p.segments << p.levels;
  a.keff = wf_effective_budget(&p);
  const int seg_in_lds = a.S <= kSelectLdsSegs ? 1 : 0;
  const size_t lds = seg_in_lds ? (size_t)a.S * sizeof(int32_t) : 0;
  hipLaunchKernelGGL(scan_select_kernel, dim3((unsigned)a.U), dim3(kScanSelectBlock), lds, s, a,
                     seg_in_lds);
  return hipGetLastError();
}

hipError_t load_scan_kernels() {
  hipFuncAttributes fa;
  return hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(scan_select_kernel));
}

}  // namespace wf
