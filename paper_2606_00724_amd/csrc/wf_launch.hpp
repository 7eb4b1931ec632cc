// Host-side plans and launchers of the WaveFilter kernels (used by the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "wavefilter.h"

namespace wf {

// Scores up to this many floats are staged in LDS by the select kernels.
constexpr int kSelectLdsFloats = 16384;
// region ids a select kernel keeps in LDS (more are read from global memory)
constexpr int kSelectLdsSegs = 8192;

struct DwtPlan {
  int streams;  // streams per workgroup
  int cps;      // coefficients per stream
  int ntiles;   // workgroups per unit
};

struct SkimPlan {
  int source;        // CoefSource
  int cpt;           // coefficients per tile
  int ntiles;        // tiles per unit
  size_t lds_bytes;  // dynamic LDS of the tile kernel
};

struct ScanPlan {
  int chunks;        // workgroups per unit
  int span;          // pool positions per workgroup
  int nbuf;          // LDS ring depth
  int seg_cap;       // region ids staged per workgroup
  size_t lds_bytes;  // dynamic LDS of the chunk kernels
};

struct AttnPlan {
  int splits;        // workgroups (row splits) per unit
  int rps;           // cache rows per split
  int tcap;          // token ids of a split in LDS at once
  int nbuf;          // LDS ring depth
  size_t lds_bytes;
};

struct FastPlan {
  int R;             // ranges (workgroups) per unit
  int span;          // tokens per range
  int nbuf;          // LDS ring depth
  int par_cap;       // parent ids staged per range (gathered rows), else 0
  size_t lds_bytes;
  bool held;         // block results kept in registers until the range's keys are read
};

// Workspace extents of the multi-scale recursion (maxima over its scales).
struct RecPlan {
  long max_n = 0;      // candidates of the widest scale
  int max_tiles = 0;   // coefficient tiles of the widest scale
  long max_keep = 0;   // kept blocks of the widest selection
};

float effective_scale(const wf_params& p);

// Filtered prompt rows: ctx_len rounded down to a multiple of 2^levels; the
// remaining ctx_len - filtered_len rows are always kept after the selection.
inline long filtered_len(const wf_params& p) {
  return ((long)p.ctx_len >> p.levels) << p.levels;
}
inline long remainder_len(const wf_params& p) { return (long)p.ctx_len - filtered_len(p); }
// Ranges each of U units' `chunks` chunks are split into, for a kernel of which
// `slots` workgroups are resident at once and a workgroup takes at most max_cpw
// chunks.  ceil(slots / U) ranges fill every slot, but where U does not divide
// the slots the workgroups past them run after the others, nearly alone: one
// range fewer then ends sooner, as fewer workgroups share the same bandwidth
// (about 0.7 of the CUs reach it) and the fixed part of a workgroup (its
// selection, its first loads: about six chunks) is paid once.  28 units of 61K
// keys, 32-token blocks: 216.8 us a call with 10 ranges a unit, 147.5 with 9; 100 units
// of 32K: 317.6 and 224.6.  Kernel by kernel over 34 to 700 units of 1K to 12K keys
// (648 calls), against ceil(slots / U) ranges: the scan's weights pass 0.93 of the
// time (at most 1.02), the attention 0.93 (1.04), the skims 0.93.  Never more ranges than ceil(slots / U) except for max_cpw.
//
// cu_slots: CUs, for workgroups that a CU rather than the memory bounds, two of
// which are resident per CU (the token skims of 64 channels): a CU that has one more
// than the others ends last (fixed part: four chunks).  Skim of 300 units of 6000
// keys, 8-token blocks: 77.3 us with one range a unit, 70.0 with two; 400 of 1734:
// 0.95 of two ranges' time with one.
inline long ranges_per_unit(long U, long chunks, long slots, long max_cpw, long cu_slots = 0) {
  const long up = std::min(chunks, std::max(1L, (slots + U - 1) / U));
  const long down = std::min(chunks, std::max(1L, slots / U));
  const long least = (chunks + max_cpw - 1) / max_cpw;
  auto cost = [&](long C) {
    const double cpw = (double)((chunks + C - 1) / C), fixed = 6.0;
    const long n = U * ((chunks + (long)cpw - 1) / (long)cpw), rest = n % slots;
    if (cu_slots) return (double)((n + cu_slots - 1) / cu_slots) * (cpw + 4.0);
    return (double)(n / slots) * (cpw + fixed) +
           (rest ? cpw * std::max(0.7, (double)rest / (double)slots) + fixed : 0.0);
  };
  const long C = std::max(least, cost(down) <= cost(up) ? down : up);
  return std::min(chunks, C);
}

// The same for the fp32 kernels, at most `most` ranges a unit.  A chunk takes an
// fp32 workgroup the same time however few CUs are busy (64 rows of 64 channels,
// 64 query rows: 3.7 us in the attention, 3.1 in the two scan passes, with 129
// workgroups as with 256; one query row 1.5), so a round of workgroups lasts as
// long as its longest, and more rounds of shorter ranges leave fewer CUs idle
// (staged attention, 64 query rows of 64 channels: 265 units of 500 rows 73.4 ->
// 53.4 us, 129 of 1000 68.0 -> 51.0; 128 channels, 129 of 4000: 413.9 -> 269.7).
// fixed: a workgroup's constant part, in chunks (measured over 1 to 600 units and
// 1 to 160 query rows: 1 in the attention and the scan of 64 channels, of which
// two workgroups fit a CU, 2 in the scan of 128).
inline long fp32_ranges_per_unit(long U, long chunks, long slots, long most, long fixed) {
  most = std::min(chunks, most);
  long best = 0, best_cost = 0, last = 0;
  for (long rounds = 1; rounds <= 4 && last < most; ++rounds) {
    const long C = std::min(most, std::max(1L, rounds * slots / U));  // as many as they take
    if (C == last) continue;
    last = C;
    const long cpw = (chunks + C - 1) / C, n = U * ((chunks + cpw - 1) / cpw);
    const long cost = (n + slots - 1) / slots * (cpw + fixed);
    if (best == 0 || cost < best_cost) {
      best = C;
      best_cost = cost;
    }
  }
  return best;
}

// Whether a call has the coefficients to fill the chip with a W kernel and
// selections in the kernels that consume them, whatever its keys, query rows
// and coefficient count.  16 units of 128 bf16 query rows: with 1024
// coefficients each a call takes 89.5 us instead of 107.5, with 128 64.4
// instead of 80.0; 32 fp32 units of 128 coefficients 63.8 instead of 70.0.
// The line is drawn at 1024 in all: calls below it (two fp32 units of 128
// coefficients would take 49.1 us instead of 54.2) keep the sequence of
// kernels that the timed entry points have always named for them.  The names draw
// this line, not the times.
inline bool wide_weights(const wf_params& p) {
  return (long)p.batch * p.heads * ((long)p.ctx_len >> p.levels) >= 1024;
}
int device_cu_count();
// Whether the Haar coefficient tiles read the keys with the streaming (nt)
// policy:
// keys past the Infinity Cache's 256 MiB displace what the kernels beside them
// reuse and find nothing of themselves there (A_J of 1 GiB of Haar keys: 235 us
// kept, 198 streamed); smaller ones may still be cached from the call or the
// copy before (64 MiB: 24.0 us kept, 25.8 streamed).  The choice is a template
// argument of the kernels: a run-time one, twice the load code, cost the
// smallest calls 0.7 us of instruction fetch.
inline bool keys_stream(const wf_params& p) {
  return (size_t)p.batch * p.heads * p.ctx_len * p.head_dim * (p.dtype == WF_BF16 ? 2 : 4) >
         (size_t)256 << 20;
}

// fine: the splits that are fastest, kFineTiles for the Haar tiles and kFineSplits
// for the fp32 scan ranges and attention splits.  Without them those are so coarse
// that their statistics and partials need no more workspace than whole
// 64-coefficient tiles and splits of whole 128-row chunks do: programs keep
// workspaces of that size, and the allocation-free call's scratch has to hold every
// call it held.  The caller of a plan and the launches that follow it pass the
// same value.
constexpr int kFineTiles = 1, kFineSplits = 2;
DwtPlan plan_dwt(const wf_params& p);
SkimPlan plan_skim(const wf_params& p, bool fused, int fine);
// select: the scan workgroups take the top-S regions themselves (all S
// region ids in LDS)
ScanPlan plan_scan(const wf_params& p, bool select, int fine);
AttnPlan plan_attn(const wf_params& p, long nrows, int fine);
// Most splits that the coarse plan of any row count up to nrows takes (fewer rows
// can take more splits: 9 chunks in 5 splits of two, 8 in 8 of one).
long most_attn_splits(const wf_params& p, long nrows);

// The fused path streams the keys once with token-level scores when the keys
// are bf16, the wavelet is Haar with 3..5 levels and the query block has at
// most 64 rows; the scan then needs only its weights pass.
bool fast_path(const wf_params& p);
// The Daubechies-2 form of that path (J = 6, at least 4 coefficients).
bool db2_token_path(const wf_params& p);
// f_J (J <= 6) and the symmetric-end filters, computed in double.
void db2_token_taps(int J, Db2TokenTaps* out);
FastPlan plan_fast(const wf_params& p);
hipError_t launch_token_skim(const wf_params& p, const void* Q, const void* K,
                             float* blocks, float* wstats, hipStream_t s);
// W (eq. 8) of every coarse block from the token skim's block rows, by
// weights_slices(p) workgroups per unit.
int weights_slices(const wf_params& p);
hipError_t launch_block_weights(const wf_params& p, const float* blocks,
                                const float* wstats, float* W, hipStream_t s);

hipError_t launch_dwt(const wf_params& p, const void* K, float* approx,
                      float* details, hipStream_t s);
hipError_t launch_skim_tiles(const wf_params& p, bool fused, const void* Q,
                             const void* K, const float* approx, float* logits,
                             float* stats, int fine, hipStream_t s);
// One scale b of the multi-scale recursion (Haar).  Tiles: the coarse
// logits of its n candidates (all 2^b-blocks when parent is null, else the
// two halves of each block in parent [U][npar]).  Select: the eq. 8 weights
// and the top `keep`, written to out as block ids (b > 1) or as the two
// tokens of each kept block (b = 1).
RecPlan plan_recursion(const wf_params& p, const int32_t* counts);
hipError_t launch_rec_tiles(const wf_params& p, int b, long n, const int32_t* parent,
                            int npar, const void* Q, const void* K, float* logits,
                            float* stats, hipStream_t s);
hipError_t launch_rec_select(const wf_params& p, int b, long n, int keep,
                             const int32_t* parent, int npar, const float* logits,
                             const float* stats, float* W, int32_t* out, hipStream_t s);
// A scale b <= 5 of the recursion from token logits (bf16 keys, Haar, at
// most 64 query rows): over all filtered keys when parent is null (b =
// levels), else over the gathered kept blocks parent [U][npar] of 2^(b+1)
// tokens.  Writes the same n coarse logits per query row as the tiles
// ([U][B][n]) and one (max, sum) slice per range; the select then merges
// plan_rec_token(..).R slices.
bool rec_token_path(const wf_params& p);
FastPlan plan_rec_token(const wf_params& p, int b, long rows, bool gather);
hipError_t launch_rec_token_skim(const wf_params& p, int b, long n, const int32_t* parent,
                                 int npar, const void* Q, const void* K, float* logits,
                                 float* stats, hipStream_t s);
hipError_t launch_rec_select_slices(const wf_params& p, int b, long n, int keep,
                                    const int32_t* parent, int npar, int nslices,
                                    const float* logits, const float* stats, float* W,
                                    int32_t* out, hipStream_t s);
hipError_t launch_skim_select(const wf_params& p, int ntiles,
                              const float* logits, const float* stats,
                              float* W, int32_t* seg, hipStream_t s);
// W [U][nJ] of the coarse logits [U][B][nJ] and their tiles' (max, sum)
// pairs, spread over enough workgroups per unit to fill the chip (no
// selection).
hipError_t launch_skim_weights(const wf_params& p, int ntiles, const float* logits,
                               const float* stats, float* W, hipStream_t s);
// stats: one (reference, sum) slice per scan workgroup, the reference in log2
// units, written by the statistics pass and read by the weights pass.
// share: units per selection (seg indexed by u / share).
hipError_t launch_scan_chunks(const wf_params& p, int weights, const void* Q,
                              const void* K, const int32_t* seg, float* stats,
                              float* wpool, int fine, hipStream_t s, int share = 1);
// Token-level path: the weights pass that first takes the unit's top-S
// regions of W itself (seg_out [U][S] receives them) and forms the pool
// normalisers from the selected blocks' log-sum-exps (blocks [U][nJ][2][B]).
// share: units per selection (W and seg_out indexed by u / share; 1 = per
// unit).
hipError_t launch_scan_select_weights(const wf_params& p, const void* Q, const void* K,
                                      const float* W, const float* blocks, int32_t* seg_out,
                                      float* wpool, hipStream_t s, int share = 1);
// Whether the scan's workgroups can take the top-S regions themselves (the region
// ids and the selection fit in LDS).
bool scan_can_select(const wf_params& p);
// The statistics pass that first takes the unit's top-S regions of W itself
// (seg_out [U][S] receives them, for the weights pass that follows) and
// writes one (max, sum) slice per workgroup into stats.
hipError_t launch_scan_select_stats(const wf_params& p, const void* Q, const void* K,
                                    const float* W, int32_t* seg_out, float* stats,
                                    int fine, hipStream_t s);
hipError_t launch_scan_select(const wf_params& p, const float* wpool,
                              const int32_t* seg, int32_t* tok,
                              hipStream_t s);
hipError_t launch_gather(const wf_params& p, const void* K, const void* V,
                         const int32_t* tok, const void* Kg, const void* Vg,
                         void* Ks, void* Vs, hipStream_t s);
// share: units per selection (tok indexed by u / share).
hipError_t launch_attn(const wf_params& p, const void* Q, const void* K,
                       const void* V, const int32_t* tok, int nsel,
                       const void* Kg, const void* Vg, int G, long nrows,
                       float* part, float* pstat, int fine, hipStream_t s, int share = 1);
// The top-S regions (eq. 9) of given weights W [groups][L >> J], one
// workgroup per group, into seg [groups][S].
hipError_t launch_select_w(const wf_params& p, long groups, const float* W, int32_t* seg,
                           hipStream_t s);
// Token-level path: the attention that first takes the unit's top-k_eff
// tokens of the scan weights wpool [U][S 2^J] itself (the pool of the
// regions seg [U][S]); tok_out [U][k_eff] (nullable) receives them.
bool attn_can_select(const wf_params& p, long nrows);
// Whether the selecting attention holds a unit's scan weights in registers (16384).
// Past that each of a unit's workgroups reads them from memory several times, and
// the general path with fp32 keys, more than 64 query rows or coefficients that
// are no multiple of four selects in a kernel of its own (5 units, 45412 of
// 120288 positions: 178.6 + 26.5 us apart, 225.1 in one).
bool pool_on_chip(const wf_params& p);
// share: units per selection (wpool, seg and tok_out indexed by u / share).
hipError_t launch_attn_select(const wf_params& p, const void* Q, const void* K, const void* V,
                              const float* wpool, const int32_t* seg, int32_t* tok_out,
                              const void* Kg, const void* Vg, long nrows, float* part,
                              float* pstat, int fine, hipStream_t s, int share = 1);
// out [groups][n] = sum over h < H of in [groups H + h][n], in order of h
// (the selection weights of a sequence's heads added up).
hipError_t launch_head_sum(const float* in, float* out, long n, int H, int groups,
                           hipStream_t s);
// Loads the code object of one translation unit onto the current device
// (each .hip file is its own code object; asking for a kernel's attributes
// loads it).
hipError_t load_fast_kernels();
hipError_t load_scan_kernels();
hipError_t load_attn_kernels();
hipError_t load_skim_kernels();
hipError_t load_dwt_kernels();
hipError_t launch_attn_combine(const wf_params& p, long nrows,
                               const float* part, const float* pstat, void* O,
                               int fine, hipStream_t s);

}  // namespace wf
