// Sparse cache and attention over it (Section 3.2, last paragraph; the
// cached-attention form of eq. 3, bidirectional: no mask).
//
// The cache rows of a unit are split into ranges of whole chunks, one
// workgroup each (split-KV); each workgroup writes its unnormalised partial
// output with the per-row max and sum of exp, and a combine kernel merges the
// splits.  In the fused path the rows are read in place: row r < k_eff is
// K[tok[r]] / V[tok[r]], the rest are the tail rows K_g / V_g.
//
// bf16: S^T = K Q^T runs on v_mfma_f32_16x16x32_bf16 over 32-row sub-blocks.
// The two 16-row MFMA tiles of a sub-block take rows 8(m/4) + m%4 and
// 8(m/4) + 4 + m%4, so that lane group g ends up holding the scores of rows
// 8g .. 8g+7 for query l%16 -- exactly the A operand of O = P V for the same
// instruction.  Online softmax (running max / sum per query row) spans the
// sub-blocks.  fp32 uses v_mfma_f32_16x16x4_f32 on 16-row sub-blocks.
#include "wf_device.hpp"
#include "wf_kernels.hpp"
#include "wf_launch.hpp"

namespace wf {

// Chunks of kRingRows cache rows (K and V) stream into an LDS ring through
// direct global->LDS loads; rows stay in their natural row-major form with
// swizzled 16-byte granules.  bf16: the PV B operand (8 consecutive rows of
// one channel per lane) comes from two ds_read_b64_tr_b16: in each 16-lane
// group, lane i points at row t0 + i/4, channels c0 + 4(i%4) .. +3, and
// receives rows t0 .. t0+3 of channel c0 + i.  fp32: it is four dword reads,
// whose 64 lanes (rows 4g + i, channels c0 + col) fall on 64 banks by the
// granule swizzle.
constexpr int kRingRows = 64;

typedef short v4i16 __attribute__((ext_vector_type(4)));

template <typename T, int D>
struct RingRowPtr {
  const T* base;
  const T* tail;
  const int32_t* toks;  // LDS: token ids of the selected rows from split_r0 on, or null
  long unit_rows;       // rows per unit in `base`
  long r0, rlast;       // absolute first row of the chunk, last valid row
  long split_r0;        // the row of toks[0]
  long Lf;              // rows Lf .. Lf + R - 1 of `base` follow the token list
  int u, nsel, G, R;
  __device__ __forceinline__ const T* operator()(int r) const {
    const long rr = min(r0 + r, rlast);
    if (toks) {
      // token ids are clamped into the unit: a bad id cannot leave K / V
      if (rr < nsel)
        return base + ((long)u * unit_rows +
                       min(max((long)toks[rr - split_r0], 0L), unit_rows - 1)) * D;
      if (rr < nsel + R) return base + ((long)u * unit_rows + Lf + (rr - nsel)) * D;
      return tail + ((long)u * G + (rr - nsel - R)) * D;
    }
    return base + ((long)u * unit_rows + rr) * D;
  }
};

// 8 waves, two per SIMD, so that one wave's MFMA, exp and LDS latencies
// overlap the other's work; with few query blocks each block's rows are
// split over two waves (bf16, 32-row products) or up to four (fp32, 16-row).
constexpr int kAttnRingBlock = 512;

// SEL (token-level path): the workgroup first takes the unit's top-nsel
// tokens of the scan weights itself (eq. 9 over the pool; ties to the lower
// pool position, which is the lower token) and keeps the ascending ids of
// its split; tok_out (nullable) receives them.
// BATCHES (fp32): the split holds more rows than ids fit the LDS and takes them a
// batch of tcap rows at a time (an instance of its own: the loop's registers cost
// the smallest calls 0.4 us of 8.2).
template <typename T, int D, bool SEL = false, bool BATCHES = false>
__global__ __launch_bounds__(kAttnRingBlock) void attn_ring_kernel(AttnArgs a) {
  constexpr bool BF = sizeof(T) == 2;
  constexpr int NW = kAttnRingBlock / kWave;
  constexpr int CR = kRingRows;
  constexpr int ES = (int)sizeof(T), EPV = 16 / ES;  // element size, elements per granule
  constexpr int G = D / EPV;
  constexpr int CHB = CR * ES * D;           // bytes of one K (or V) chunk
  constexpr int IPW = CR * G / (64 * NW);    // loads per wave per matrix
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* ring = smem;                                       // [nbuf][K, V]
  int32_t* toks = reinterpret_cast<int32_t*>(smem + (size_t)a.nbuf * 2 * CHB);

  const int item = xcd_swizzle(blockIdx.x, gridDim.x);
  const int u = item / a.NS, sp = item % a.NS;
  const long rb0 = (long)sp * a.rps;
  const long re0 = min(rb0 + (long)a.rps, (long)a.nrows);
  const int nch = (int)((re0 - rb0 + CR - 1) / CR);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, col = lane & 15;

  if constexpr (SEL) {
    // the selection's histograms, the unit's region ids and (when they fit)
    // its scan weights in the ring, which is free until the first chunk
    auto& sh = *reinterpret_cast<SelectShared<kAttnRingBlock>*>(ring);
    int32_t* segl = reinterpret_cast<int32_t*>(ring + sizeof(SelectShared<kAttnRingBlock>));
    float* Wl = reinterpret_cast<float*>(segl + a.S);
    const int sel = u / a.share;  // the unit's selection
    const float* Wg = a.wpool + (long)sel * a.P;
    for (int i = threadIdx.x; i < a.S; i += kAttnRingBlock) segl[i] = a.seg[(long)sel * a.S + i];
    const long hi = min(re0, (long)a.nsel);
    const int J = a.J, mask = (1 << J) - 1;
    int32_t* tout =
        a.tok_out && u % a.share == 0 ? a.tok_out + (long)sel * a.nsel : nullptr;
    auto emit = [&](uint32_t pos, int pp) {
      if ((long)pos >= rb0 && (long)pos < hi) {
        const int32_t t = (segl[pp >> J] << J) | (pp & mask);
        toks[pos - rb0] = t;
        if (tout) tout[pos] = t;
      }
    };
    // weights per thread held in registers: 16, or 32 past 8192 positions
    constexpr int EPT = 16;
    if (a.P <= EPT * kAttnRingBlock) {
      // (the selection's first barrier publishes the region ids)
      block_select_topk_regs<kAttnRingBlock, EPT>(Wg, a.P, a.nsel, emit, sh);
    } else if (a.P <= 2 * EPT * kAttnRingBlock) {
      block_select_topk_regs<kAttnRingBlock, 2 * EPT>(Wg, a.P, a.nsel, emit, sh);
    } else {
      if (a.w_in_lds) {
        for (int i = threadIdx.x; i < a.P; i += kAttnRingBlock) Wl[i] = Wg[i];
        __syncthreads();
        block_select_topk<kAttnRingBlock>(Wl, a.P, a.nsel, emit, sh);
      } else {
        __syncthreads();
        block_select_topk<kAttnRingBlock>(Wg, a.P, a.nsel, emit, sh);
      }
    }
  }
  // ids of the split's rows from r0 on (!SEL)
  auto stage_toks = [&](long r0) {
    const long hi = min(BATCHES ? min(re0, r0 + a.tcap) : re0, (long)a.nsel);
    for (long i = r0 + threadIdx.x; i < hi; i += kAttnRingBlock)
      toks[i - r0] = a.tok[(long)(u / a.share) * a.nsel + i];
  };
  if (!SEL && a.tok) stage_toks(rb0);
  __syncthreads();

  RingRowPtr<T, D> kp, vp;
  kp.base = reinterpret_cast<const T*>(a.K);
  vp.base = reinterpret_cast<const T*>(a.V);
  kp.tail = reinterpret_cast<const T*>(a.Kg);
  vp.tail = reinterpret_cast<const T*>(a.Vg);
  const bool indexed = SEL || a.tok != nullptr;
  kp.toks = vp.toks = indexed ? toks : nullptr;
  kp.unit_rows = vp.unit_rows = indexed ? (long)a.L : (long)a.nrows;
  kp.rlast = vp.rlast = re0 - 1;
  kp.split_r0 = vp.split_r0 = rb0;
  kp.u = vp.u = u;
  kp.nsel = vp.nsel = a.nsel;
  kp.G = vp.G = a.G;
  kp.R = vp.R = a.R;
  kp.Lf = vp.Lf = a.Lf;

  const int nqb = (a.B + 15) / 16;
  // row parts per query block (bf16: two or one)
  const int tsplit = !BF && 4 * nqb <= NW ? 4 : 2 * nqb <= NW ? 2 : 1;
  const int qpg = NW / tsplit;
  const int ngroups = (nqb + qpg - 1) / qpg;
  const int part = wave % tsplit;
  const int R = CR / tsplit;
  const T* Qunit = reinterpret_cast<const T*>(a.Q) + (long)u * a.B * D;
  float* po_base = a.part + ((long)u * a.NS + sp) * a.B * D;
  float* ps_base = a.pstat + ((long)u * a.NS + sp) * 2 * a.B;
  const uint32_t ring_lds = lds_offset(ring);
  const int nbuf = a.nbuf;
  const float c2 = a.scale * kLog2e;  // scores in log2 units

  // K and V rows of chunk c into the ring slot at `slot`.  A chunk whose
  // rows are all selected tokens (rows past the split repeat its last row)
  // takes one token id and one address per row for both loads; any other
  // chunk goes through the general row map.
  const T* kunit = kp.base + (long)u * kp.unit_rows * D;
  const T* vunit = vp.base + (long)u * vp.unit_rows * D;
  const int split_last = (int)(re0 - 1 - rb0);
  // (b0: the batch's first chunk)
  auto issue_kv = [&](int c, uint32_t slot, int b0) {
    const long r0 = rb0 + (long)c * CR;
    if (indexed && min(r0 + CR, re0) <= (long)a.nsel) {
      constexpr int RPI = 64 / G;
      // every token id is read from LDS before the first load is issued (an
      // LDS read between two asm loads waits out its own latency each time)
      long off[IPW];
#pragma unroll
      for (int i = 0; i < IPW; ++i) {
        const int r = (wave * IPW + i) * RPI + lane / G;
        const int k = (lane % G) ^ granule_swz<G>(r);
        // token ids are clamped into the unit: a bad id cannot leave K / V
        const int t = min(max(toks[min((int)(r0 - rb0) + r, split_last) - (BATCHES ? b0 * CR : 0)], 0), a.L - 1);
        off[i] = (long)t * D + EPV * k;
      }
#pragma unroll
      for (int i = 0; i < IPW; ++i) {
        const int inst = wave * IPW + i;
        async_load16<true>(kunit + off[i], __builtin_amdgcn_readfirstlane(slot + 1024u * inst));
        async_load16<true>(vunit + off[i], __builtin_amdgcn_readfirstlane(slot + CHB + 1024u * inst));
      }
    } else {
      kp.r0 = vp.r0 = r0;
      issue_chunk<CR, G, NW, true>(slot, kp);
      issue_chunk<CR, G, NW, true>(slot + CHB, vp);
    }
  };

  // LDS byte offsets of the lane's operands inside a 32-row block: the
  // granule swizzle depends only on the row mod 32 and every block starts at
  // a multiple of 32 rows, so one set serves all blocks
  // (fp32: inside a 16-row block, the first or second of 32 rows)
  constexpr int KS = G / 4;  // granules of a row per lane group
  int koff[KS], kyoff[KS], vlo[D / 16], vhi[D / 16];
  if constexpr (BF) {
    const int rx0 = 8 * (col >> 2) + (col & 3);  // QK rows rx0 and rx0 + 4
    const int t00 = 8 * g + (col >> 2);          // PV rows t00 and t00 + 4
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      koff[s] = granule_offset<G>(rx0, 4 * s + g);
      kyoff[s] = granule_offset<G>(rx0 + 4, 4 * s + g);
    }
#pragma unroll
    for (int cb = 0; cb < D / 16; ++cb) {
      const int gran = 2 * cb + ((col & 3) >> 1);
      const int byte = 8 * (col & 1);
      vlo[cb] = granule_offset<G>(t00, gran) + byte;
      vhi[cb] = granule_offset<G>(t00 + 4, gran) + byte;
    }
  }

  for (int grp = 0; grp < ngroups; ++grp) {
    const int qb = grp * qpg + wave / tsplit;
    const bool active = qb < nqb;
    const T* qrow = Qunit + (long)min(qb * 16 + col, a.B - 1) * D;
    u32x4 qreg[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s)
      qreg[s] = *reinterpret_cast<const u32x4*>(qrow + EPV * (4 * s + g));
    f32x4 O[D / 16];
#pragma unroll
    for (int cb = 0; cb < D / 16; ++cb) O[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;
    // consume the q operand before async loads are queued, so that the
    // compiler's own wait for it sits here and not inside the loop below
#pragma unroll
    for (int s = 0; s < KS; ++s) asm volatile("" ::"v"(qreg[s]));
    int next = 0;
    do {
    const int b0 = BATCHES ? next : 0;
    const int b1 = BATCHES ? min(nch, b0 + a.tcap / CR) : nch;
    if constexpr (BATCHES) {
      kp.split_r0 = vp.split_r0 = rb0 + (long)b0 * CR;
      stage_toks(kp.split_r0);  // (no chunk is in flight, every wave is past its issues)
      __syncthreads();
    }
    // ring of nbuf slots, nbuf - 1 chunks in flight ahead of the one consumed
    for (int k = b0; k < b1 && k - b0 < nbuf - 1; ++k)
      issue_kv(k, ring_lds + (uint32_t)((k - b0) * 2 * CHB), b0);
    for (int ch = b0; ch < b1; ++ch) {
      const int nr = (int)min((long)CR, re0 - (rb0 + (long)ch * CR));
      wait_vmcnt_chunks<2 * IPW>(min(b1 - 1 - ch, nbuf - 2));
      lds_barrier();  // chunk ch visible; everyone is past chunk ch - 1
      if (ch + nbuf - 1 < b1)
        issue_kv(ch + nbuf - 1, ring_lds + (uint32_t)(((ch + nbuf - 1 - b0) % nbuf) * 2 * CHB),
                 b0);
      const unsigned char* Kb = ring + ((ch - b0) % nbuf) * 2 * CHB;
      const unsigned char* Vb = Kb + CHB;
      if (active) {
        const int rb = part * R;
        const int re = min(rb + R, nr);
        if constexpr (!BF) {
          for (int sb = rb; sb < re; sb += 16) {
            const unsigned char* kblk = Kb + sb * (16 * G);
            const unsigned char* vblk = Vb + sb * (16 * G);
            const int h = sb & 16;  // the block's place in its 32 rows
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KS; ++s) {
              const f32x4 kv = *reinterpret_cast<const f32x4*>(
                  kblk + granule_offset<G>(h + col, 4 * s + g) - h * (16 * G));
              const f32x4 qv = __builtin_bit_cast(f32x4, qreg[s]);
#pragma unroll
              for (int e = 0; e < 4; ++e)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[e], qv[e], acc, 0, 0, 0);
            }
            // lane holds the scores of rows sb + 4g + i for query col; t: in log2
            // units, rows past the range -inf.  Only the reference is taken from
            // the rounded t: a weight's exponent is the unrounded product less the
            // reference, so that scores of thousands keep their differences.
            float t[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) t[i] = sb + 4 * g + i < re ? acc[i] * c2 : -INFINITY;
            const float mb =
                max_xor32(max_xor16(fmaxf(fmaxf(t[0], t[1]), fmaxf(t[2], t[3]))));
            const float m_new = fmaxf(m_run, mb);
            // (while every score so far is -inf, their weights are 2^-inf = 0)
            const float ref = m_new > -INFINITY ? m_new : 0.f;
            float pv[4], ps = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              pv[i] = sb + 4 * g + i < re ? __builtin_amdgcn_exp2f(fmaf(acc[i], c2, -ref)) : 0.f;
              ps += pv[i];
            }
            ps = add_xor32(add_xor16(ps));
            if (__builtin_amdgcn_ballot_w64(m_new != m_run) != 0) {
              const float alpha = __builtin_amdgcn_exp2f(m_run - ref);
              l_run = l_run * alpha + ps;
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const float ai = __shfl(alpha, 4 * g + i);
#pragma unroll
                for (int cb = 0; cb < D / 16; ++cb) O[cb][i] *= ai;
              }
            } else {
              l_run += ps;
            }
            // rows past the range repeat its last one: 0 there, as 0 times an
            // infinite value is NaN (every wave that reads the block does it)
            if (sb + 16 > re) {
              f32x4* pad = reinterpret_cast<f32x4*>(const_cast<unsigned char*>(vblk));
              for (int i = (re - sb) * G + lane; i < 16 * G; i += 64)
                pad[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
            // P is the A operand in place; V row 4g + i, channel 16 cb + col
#pragma unroll
            for (int i = 0; i < 4; ++i) {
#pragma unroll
              for (int cb = 0; cb < D / 16; ++cb) {
                const float vb = *reinterpret_cast<const float*>(
                    vblk + granule_offset<G>(h + 4 * g + i, 4 * cb + (col >> 2)) -
                    h * (16 * G) + 4 * (col & 3));
                O[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[i], vb, O[cb], 0, 0, 0);
              }
            }
            m_run = m_new;
          }
        } else for (int sb = rb; sb < re; sb += 32) {
          // every LDS operand of the block is read first: the V reads'
          // latency then overlaps the QK products and the softmax
          const unsigned char* kblk = Kb + sb * (16 * G);
          const uint32_t vblk = lds_offset(Vb) + (uint32_t)(sb * (16 * G));
          u32x4 kx[KS], ky[KS], vb[D / 16];
#pragma unroll
          for (int s = 0; s < D / 32; ++s) {
            kx[s] = *reinterpret_cast<const u32x4*>(kblk + koff[s]);
            ky[s] = *reinterpret_cast<const u32x4*>(kblk + kyoff[s]);
          }
#pragma unroll
          for (int cb = 0; cb < D / 16; ++cb) {
            const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) v4i16*)(size_t)(vblk + vlo[cb]));
            const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) v4i16*)(size_t)(vblk + vhi[cb]));
            const u32x2 l2 = __builtin_bit_cast(u32x2, lo);
            const u32x2 h2 = __builtin_bit_cast(u32x2, hi);
            vb[cb] = u32x4{l2[0], l2[1], h2[0], h2[1]};
          }
          f32x4 ax = {0.f, 0.f, 0.f, 0.f}, ay = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s = 0; s < D / 32; ++s) {
            ax = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, kx[s]), __builtin_bit_cast(bf16x8, qreg[s]), ax, 0, 0, 0);
            ay = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, ky[s]), __builtin_bit_cast(bf16x8, qreg[s]), ay, 0, 0, 0);
          }
          // lane holds the scores of rows sb + 8g + e (e < 8) for query col,
          // here in log2 units; rows past the range (only in a last partial
          // block) are -inf
          float t[8];
          const bool full = sb + 32 <= re;  // uniform
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            t[i] = ax[i] * c2;
            t[4 + i] = ay[i] * c2;
          }
          if (!full) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (sb + 8 * g + e >= re) t[e] = -INFINITY;
          }
          float mb = fmaxf(fmaxf(fmaxf(t[0], t[1]), fmaxf(t[2], t[3])),
                           fmaxf(fmaxf(t[4], t[5]), fmaxf(t[6], t[7])));
          mb = max_xor32(max_xor16(mb));
          const float m_new = fmaxf(m_run, mb);  // finite: row sb is in range
          float pv[8], ps = 0.f;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            pv[e] = __builtin_amdgcn_exp2f(t[e] - m_new);  // 2^-inf = 0
            ps += pv[e];
          }
          ps = add_xor32(add_xor16(ps));
          // rescale only when some row maximum grew: otherwise the factor
          // is exactly 1 and the update is the same without it
          if (__builtin_amdgcn_ballot_w64(m_new != m_run) != 0) {
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            l_run = l_run * alpha + ps;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float ai = __shfl(alpha, 4 * g + i);
#pragma unroll
              for (int cb = 0; cb < D / 16; ++cb) O[cb][i] *= ai;
            }
          } else {
            l_run += ps;
          }
          const u32x4 pp = {pack_bf16x2(pv[0], pv[1]), pack_bf16x2(pv[2], pv[3]),
                            pack_bf16x2(pv[4], pv[5]), pack_bf16x2(pv[6], pv[7])};
#pragma unroll
          for (int cb = 0; cb < D / 16; ++cb)
            O[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, pp), __builtin_bit_cast(bf16x8, vb[cb]), O[cb], 0, 0, 0);
          m_run = m_new;
        }
      }
    }
    lds_barrier();  // the ring is idle before it is refilled or reused
    next = b1;
    } while (BATCHES && next < nch);

    if (tsplit == 1) {
      if (active) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int q = qb * 16 + 4 * g + i;
          if (q < a.B) {
#pragma unroll
            for (int cb = 0; cb < D / 16; ++cb) po_base[(long)q * D + cb * 16 + col] = O[cb][i];
          }
        }
        const int q = qb * 16 + col;
        if (g == 0 && q < a.B) {
          ps_base[q] = m_run;
          ps_base[a.B + q] = l_run;
        }
      }
    } else {
      // one group; the tsplit waves of a query block merge their row parts
      // (the ring is idle: every wave passed the barrier after the loop)
      float* cO = reinterpret_cast<float*>(smem);  // [NW][16][D]
      float* cm = cO + NW * 16 * D;                 // [NW][16]
      float* cl = cm + NW * 16;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int cb = 0; cb < D / 16; ++cb)
          cO[(wave * 16 + 4 * g + i) * D + cb * 16 + col] = O[cb][i];
      }
      if (g == 0) {
        cm[wave * 16 + col] = m_run;
        cl[wave * 16 + col] = l_run;
      }
      lds_barrier();
      constexpr int MP = BF ? 2 : 4;  // most parts
      if (part == 0 && active) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int rr = 4 * g + i;
          const int q = qb * 16 + rr;
          float mp[MP], w[MP];
#pragma unroll
          for (int k = 0; k < MP; ++k)
            mp[k] = BF || k < tsplit ? cm[(wave + k) * 16 + rr] : -INFINITY;
          float M = mp[0];
#pragma unroll
          for (int k = 1; k < MP; ++k) M = fmaxf(M, mp[k]);
          float lsum = 0.f;
#pragma unroll
          for (int k = 0; k < MP; ++k) {
            w[k] = mp[k] > -INFINITY ? __builtin_amdgcn_exp2f(mp[k] - M) : 0.f;
            if (BF || k < tsplit) lsum += w[k] * cl[(wave + k) * 16 + rr];
          }
          if (q < a.B) {
#pragma unroll
            for (int cb = 0; cb < D / 16; ++cb) {
              float o[MP];
#pragma unroll
              for (int k = 0; k < MP; ++k)
                o[k] = BF || k < tsplit
                           ? w[k] * cO[((wave + k) * 16 + rr) * D + cb * 16 + col]
                           : 0.f;
              po_base[(long)q * D + cb * 16 + col] =
                  BF ? o[0] + o[1] : (o[0] + o[1]) + (o[MP - 2] + o[MP - 1]);
            }
            if (col == 0) {
              ps_base[q] = M;
              ps_base[a.B + q] = lsum;
            }
          }
        }
      }
    }
  }
}

// Merges the splits of each query row: O = sum_s 2^(M_s - M) O_s / sum_s
// 2^(M_s - M) l_s (M_s in log2 units).  A workgroup takes 2048 / D rows of one unit, a thread 8
// consecutive channels of one row (two 16-byte loads per split, one 16-byte
// store for bf16).
constexpr int kCombineBlock = 256;

template <typename T>
__device__ __forceinline__ void store8(T* dst, const float* v);
template <>
__device__ __forceinline__ void store8<bf16_t>(bf16_t* dst, const float* v) {
  *reinterpret_cast<u32x4*>(dst) = u32x4{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                         pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
}
template <>
__device__ __forceinline__ void store8<float>(float* dst, const float* v) {
  reinterpret_cast<float4*>(dst)[0] = float4{v[0], v[1], v[2], v[3]};
  reinterpret_cast<float4*>(dst)[1] = float4{v[4], v[5], v[6], v[7]};
}

// Output row q, channels c0 .. c0 + 7, of unit u merged from the unit's NS
// split partials.
template <typename T>
__device__ __forceinline__ void merge_splits(const AttnArgs& a, int u, int q, int c0, int D) {
  const float* ps = a.pstat + (long)u * a.NS * 2 * a.B;
  // splits in groups of SB whose loads are all in flight together; each
  // group is merged into the running (max, sum, output) in one step, so up
  // to SB splits the arithmetic is the plain max-then-sum
  constexpr int SB = 8;
  float M = -INFINITY, lsum = 0.f;
  float o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < a.NS; s0 += SB) {
    float ms[SB], zs[SB];
    float4 x[SB][2];
#pragma unroll
    for (int k = 0; k < SB; ++k) {
      const int s = s0 + k;
      if (s < a.NS) {
        ms[k] = ps[(long)s * 2 * a.B + q];
        zs[k] = ps[(long)s * 2 * a.B + a.B + q];
        const float4* src =
            reinterpret_cast<const float4*>(a.part + (((long)u * a.NS + s) * a.B + q) * D + c0);
        x[k][0] = src[0];
        x[k][1] = src[1];
      } else {
        ms[k] = -INFINITY;
        zs[k] = 0.f;
        x[k][0] = x[k][1] = float4{0.f, 0.f, 0.f, 0.f};
      }
    }
    float mn = M;
#pragma unroll
    for (int k = 0; k < SB; ++k) mn = fmaxf(mn, ms[k]);
    if (mn == -INFINITY) continue;
    const float r = M > -INFINITY ? __builtin_amdgcn_exp2f(M - mn) : 0.f;
    lsum *= r;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] *= r;
#pragma unroll
    for (int k = 0; k < SB; ++k) {
      const float w = ms[k] > -INFINITY ? __builtin_amdgcn_exp2f(ms[k] - mn) : 0.f;
      lsum += zs[k] * w;
      o[0] += w * x[k][0].x;
      o[1] += w * x[k][0].y;
      o[2] += w * x[k][0].z;
      o[3] += w * x[k][0].w;
      o[4] += w * x[k][1].x;
      o[5] += w * x[k][1].y;
      o[6] += w * x[k][1].z;
      o[7] += w * x[k][1].w;
    }
    M = mn;
  }
  const float inv = 1.f / lsum;
#pragma unroll
  for (int i = 0; i < 8; ++i) o[i] *= inv;
  store8<T>(reinterpret_cast<T*>(a.O) + ((long)u * a.B + q) * D + c0, o);
}

template <typename T>
__global__ __launch_bounds__(kCombineBlock) void attn_combine_kernel(AttnArgs a, int D) {
  const int tpr = D / 8;                  // threads per row
  const int rpb = kCombineBlock / tpr;    // rows per workgroup
  const int nqb = (a.B + rpb - 1) / rpb;
  // the unit on the XCD whose L2 took its partials from the attention
  const int item = xcd_swizzle(blockIdx.x, gridDim.x);
  const int u = item / nqb;
  const int q = (item % nqb) * rpb + threadIdx.x / tpr;
  const int c0 = (threadIdx.x % tpr) * 8;
  if (q >= a.B) return;  // no barrier follows
  merge_splits<T>(a, u, q, c0, D);
}

// Sparse cache rows: [K[tok]; Kg] and [V[tok]; Vg], 16 bytes per thread.
__global__ __launch_bounds__(kBlock) void gather_kernel(GatherArgs a) {
  const int vpr = a.D * a.elem / 16;
  const long rows = (long)a.keff + a.R + a.G;
  const long total = (long)a.U * rows * vpr;
  for (long v = (long)blockIdx.x * kBlock + threadIdx.x; v < total;
       v += (long)gridDim.x * kBlock) {
    const long ur = v / vpr;
    const int k = (int)(v % vpr);
    const int u = (int)(ur / rows);
    const long r = ur % rows;
    const unsigned char* ks;
    const unsigned char* vs;
    const long row_bytes = (long)a.D * a.elem;
    if (r < a.keff) {
      const long t = min(max((long)a.tok[(long)u * a.keff + r], 0L), (long)a.L - 1);
      ks = (const unsigned char*)a.K + ((long)u * a.L + t) * row_bytes;
      vs = (const unsigned char*)a.V + ((long)u * a.L + t) * row_bytes;
    } else if (r < a.keff + a.R) {
      ks = (const unsigned char*)a.K + ((long)u * a.L + a.Lf + (r - a.keff)) * row_bytes;
      vs = (const unsigned char*)a.V + ((long)u * a.L + a.Lf + (r - a.keff)) * row_bytes;
    } else {
      ks = (const unsigned char*)a.Kg + ((long)u * a.G + (r - a.keff - a.R)) * row_bytes;
      vs = (const unsigned char*)a.Vg + ((long)u * a.G + (r - a.keff - a.R)) * row_bytes;
    }
    const long dst = ur * row_bytes + (long)k * 16;
    *reinterpret_cast<u32x4*>((unsigned char*)a.Ks + dst) =
        *reinterpret_cast<const u32x4*>(ks + k * 16);
    *reinterpret_cast<u32x4*>((unsigned char*)a.Vs + dst) =
        *reinterpret_cast<const u32x4*>(vs + k * 16);
  }
}

// ------------------------------------------------------------ host side

// Token ids of a split in LDS at once (bf16 splits hold no more rows).
constexpr long kTokCap = 4096;

// Most fp32 splits of a unit: those of whole 128-row chunks, about 512 in all
// (the coarse partials), at most twice as many where fine.  (With a split every
// 4096 rows, as the ids alone would have it, 700 units of a few rows and a
// tail of 5000 took 1.9 times the workspace, and 500 units of 100K rows 25.)
static long most_fp32_splits(long U, long nrows, int fine) {
  const long chunks = std::max(1L, (nrows + 127) / 128);
  const long splits = std::min(chunks, std::max(1L, (512 + U - 1) / U));
  const long cps = (chunks + splits - 1) / splits;
  return (chunks + cps - 1) / cps * (fine & kFineSplits ? 2 : 1);
}

AttnPlan plan_attn(const wf_params& p, long nrows, int fine) {
  AttnPlan a{};
  const long U = (long)p.batch * p.heads;
  const int D = p.head_dim;
  const int es = p.dtype == WF_BF16 ? 2 : 4;
  // one workgroup per CU streaming its rows through the LDS ring
  const long chunks = std::max(1L, (nrows + kRingRows - 1) / kRingRows);
  // (bf16: at most 4096 rows)
  const long splits =
      p.dtype == WF_BF16
          ? ranges_per_unit(U, chunks, device_cu_count(), kTokCap / kRingRows)
          : fp32_ranges_per_unit(U, chunks, device_cu_count(), most_fp32_splits(U, nrows, fine),
                                 1);
  const long cps = (chunks + splits - 1) / splits;
  a.rps = (int)(cps * kRingRows);
  a.splits = (int)((nrows + a.rps - 1) / a.rps);
  a.tcap = (int)std::min((long)a.rps, kTokCap);
  const size_t stage = (size_t)2 * kRingRows * es * D;     // K + V chunk
  const size_t toks = (size_t)a.tcap * sizeof(int32_t);
  const size_t budget = 160 * 1024 - 1024;
  // three slots (two chunks in flight) measured slightly faster than four;
  // fp32 rows of 128 channels leave room for two.  fp32 rows of 64 channels
  // take two where there are more workgroups than CUs, so that two fit a CU
  // (400 units of 100 rows, 64 query rows: 30.3 -> 26.1 us)
  const bool two = p.dtype != WF_BF16 && D == 64 && U * a.splits > device_cu_count();
  a.nbuf = (int)std::min<size_t>(two ? 2 : 3, (budget - toks) / stage);
  if (a.nbuf < 2) a.nbuf = 0;  // rejected by the caller
  constexpr int nw = kAttnRingBlock / kWave;  // row-part merge: [nw][16][D] + 2 [nw][16]
  const size_t comb = (size_t)nw * 16 * D * 4 + (size_t)2 * nw * 16 * 4;
  a.lds_bytes = std::max((size_t)a.nbuf * stage, comb) + toks;
  return a;
}

long most_attn_splits(const wf_params& p, long nrows) {
  const long U = (long)p.batch * p.heads;
  if (p.dtype != WF_BF16)
    return std::min((nrows + 127) / 128, std::max(1L, (512 + U - 1) / U));
  const long chunks = (nrows + kRingRows - 1) / kRingRows;
  const long least = (chunks + kTokCap / kRingRows - 1) / (kTokCap / kRingRows);
  return std::min(chunks, std::max(least, std::max(1L, (device_cu_count() + U - 1) / U)));
}

template <typename T, int D, bool BATCHES = false>
static hipError_t attn_launch(const AttnArgs& a, size_t lds, hipStream_t s) {
  auto kern = attn_ring_kernel<T, D, false, BATCHES>;
  if (lds > 65536) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)(a.U * a.NS)), dim3(kAttnRingBlock), lds, s, a);
  return hipGetLastError();
}

static hipError_t launch_attn_batches(bool d128, const AttnArgs& a, size_t lds, hipStream_t s);

hipError_t launch_attn(const wf_params& p, const void* Q, const void* K,
                       const void* V, const int32_t* tok, int nsel,
                       const void* Kg, const void* Vg, int G, long nrows,
                       float* part, float* pstat, int fine, hipStream_t s, int share) {
  if (share < 1 || (p.batch * p.heads) % share != 0) return hipErrorInvalidValue;
  const AttnPlan pl = plan_attn(p, nrows, fine);
  AttnArgs a;
  a.share = share;
  a.Q = Q;
  a.K = K;
  a.V = V;
  a.tok = tok;
  a.Kg = Kg;
  a.Vg = Vg;
  a.part = part;
  a.pstat = pstat;
  a.O = nullptr;
  a.U = p.batch * p.heads;
  a.L = p.ctx_len;
  a.B = p.q_len;
  a.nsel = nsel;
  a.G = G;
  // indexed rows: the selection, then the always-kept remainder, then the tail
  a.Lf = filtered_len(p);
  a.R = tok ? (int)remainder_len(p) : 0;
  a.nrows = (int)nrows;
  a.NS = pl.splits;
  a.rps = pl.rps;
  a.tcap = pl.tcap;
  a.nbuf = pl.nbuf;
  a.scale = effective_scale(p);
  const bool d128 = p.head_dim == 128;
  if (p.dtype == WF_BF16)
    return d128 ? attn_launch<bf16_t, 128>(a, pl.lds_bytes, s)
                : attn_launch<bf16_t, 64>(a, pl.lds_bytes, s);
  if (tok && pl.rps > pl.tcap) return launch_attn_batches(d128, a, pl.lds_bytes, s);
  return d128 ? attn_launch<float, 128>(a, pl.lds_bytes, s)
              : attn_launch<float, 64>(a, pl.lds_bytes, s);
}

bool pool_on_chip(const wf_params& p) {
  return ((long)p.segments << p.levels) <= 2L * 16 * kAttnRingBlock;
}

bool attn_can_select(const wf_params& p, long nrows) {
  if (p.segments > kSelectLdsSegs || (p.dtype != WF_BF16 && !wide_weights(p))) return false;
  // (the coarse plan's splits are the longest, its ring is no deeper)
  const AttnPlan pl = plan_attn(p, nrows, 0);
  if (pl.nbuf < 2 || pl.rps > pl.tcap) return false;
  if (p.dtype != WF_BF16 && !pool_on_chip(p)) return false;
  const size_t ring = (size_t)pl.nbuf * 2 * kRingRows * (p.dtype == WF_BF16 ? 2 : 4) * p.head_dim;
  return sizeof(SelectShared<kAttnRingBlock>) + (size_t)p.segments * sizeof(int32_t) <= ring;
}

hipError_t launch_attn_select(const wf_params& p, const void* Q, const void* K, const void* V,
                              const float* wpool, const int32_t* seg, int32_t* tok_out,
                              const void* Kg, const void* Vg, long nrows, float* part,
                              float* pstat, int fine, hipStream_t s, int share) {
  if (!attn_can_select(p, nrows) || share < 1 || (p.batch * p.heads) % share != 0)
    return hipErrorInvalidValue;
  const AttnPlan pl = plan_attn(p, nrows, fine);
  AttnArgs a{};
  a.Q = Q;
  a.K = K;
  a.V = V;
  a.tok = nullptr;
  a.wpool = wpool;
  a.seg = seg;
  a.tok_out = tok_out;
  a.Kg = Kg;
  a.Vg = Vg;
  a.part = part;
  a.pstat = pstat;
  a.share = share;
  a.U = p.batch * p.heads;
  a.L = p.ctx_len;
  a.B = p.q_len;
  a.nsel = wf_effective_budget(&p);
  a.P = p.segments << p.levels;
  a.S = p.segments;
  a.J = p.levels;
  a.G = p.gen_len;
  a.Lf = filtered_len(p);
  a.R = (int)remainder_len(p);
  a.nrows = (int)nrows;
  a.NS = pl.splits;
  a.rps = pl.rps;
  a.tcap = pl.tcap;
  a.nbuf = pl.nbuf;
  a.scale = effective_scale(p);
  // the unit's scan weights in the ring beside the histograms and region
  // ids when they fit
  const size_t ring = (size_t)pl.nbuf * 2 * kRingRows * (p.dtype == WF_BF16 ? 2 : 4) * p.head_dim;
  const size_t fixed = sizeof(SelectShared<kAttnRingBlock>) + (size_t)a.S * sizeof(int32_t);
  a.w_in_lds = fixed + (size_t)a.P * sizeof(float) <= ring ? 1 : 0;
  auto kern = [&] {
    if (p.dtype == WF_BF16)
      return p.head_dim == 128 ? attn_ring_kernel<bf16_t, 128, true>
                               : attn_ring_kernel<bf16_t, 64, true>;
    return p.head_dim == 128 ? attn_ring_kernel<float, 128, true>
                             : attn_ring_kernel<float, 64, true>;
  }();
  if (pl.lds_bytes > 65536) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)pl.lds_bytes);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)(a.U * a.NS)), dim3(kAttnRingBlock), pl.lds_bytes, s, a);
  return hipGetLastError();
}

static hipError_t launch_attn_batches(bool d128, const AttnArgs& a, size_t lds, hipStream_t s) {
  return d128 ? attn_launch<float, 128, true>(a, lds, s) : attn_launch<float, 64, true>(a, lds, s);
}

hipError_t launch_attn_combine(const wf_params& p, long nrows,
                               const float* part, const float* pstat, void* O,
                               int fine, hipStream_t s) {
  AttnArgs a{};
  a.part = const_cast<float*>(part);
  a.pstat = const_cast<float*>(pstat);
  a.O = O;
  a.U = p.batch * p.heads;
  a.B = p.q_len;
  a.NS = plan_attn(p, nrows, fine).splits;
  const int rpb = kCombineBlock / (p.head_dim / 8);
  const dim3 grid((unsigned)(a.U * ((a.B + rpb - 1) / rpb)));
  if (p.dtype == WF_BF16)
    hipLaunchKernelGGL(attn_combine_kernel<bf16_t>, grid, dim3(kCombineBlock), 0, s, a,
                       p.head_dim);
  else
    hipLaunchKernelGGL(attn_combine_kernel<float>, grid, dim3(kCombineBlock), 0, s, a,
                       p.head_dim);
  return hipGetLastError();
}

hipError_t launch_gather(const wf_params& p, const void* K, const void* V,
                         const int32_t* tok, const void* Kg, const void* Vg,
                         void* Ks, void* Vs, hipStream_t s) {
  GatherArgs a;
  a.K = K;
  a.V = V;
  a.tok = tok;
  a.Kg = Kg;
  a.Vg = Vg;
  a.Ks = Ks;
  a.Vs = Vs;
  a.U = p.batch * p.heads;
  a.L = p.ctx_len;
  a.D = p.head_dim;
  a.keff = wf_effective_budget(&p);
  a.G = p.gen_len;
  a.Lf = filtered_len(p);
  a.R = (int)remainder_len(p);
  a.elem = p.dtype == WF_BF16 ? 2 : 4;
  const long total = (long)a.U * (a.keff + a.R + a.G) * (a.D * a.elem / 16);
  const long blocks = std::min((total + kBlock - 1) / kBlock,
                               (long)device_cu_count() * 16);
  hipLaunchKernelGGL(gather_kernel, dim3((unsigned)std::max(1L, blocks)),
                     dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t load_attn_kernels() {
  hipFuncAttributes fa;
  return hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(attn_ring_kernel<bf16_t, 128, true>));
}

}  // namespace wf
