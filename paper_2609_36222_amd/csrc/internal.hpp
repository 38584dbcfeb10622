// Launchers of the BASE kernels, called by the C ABI layer (api.hip).
// Each enqueues on `st` and returns hipGetLastError() of its launch.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

namespace basek {

constexpr int MAX_K = 16;     // experts per token
constexpr int MAX_E = 256;    // experts per layer
constexpr int MAX_B = 1024;   // tokens per batch

// Events attached to the next kernel launch (per host thread): when set,
// launch_k hands them to the dispatch itself, which records `start` as the
// kernel begins and `stop` as it ends, then clears them.
struct KernelEvents {
  hipEvent_t start = nullptr, stop = nullptr;
};
KernelEvents &kernel_events();

template <typename F, typename... Args>
inline void launch_k(F kernel, dim3 grid, dim3 block, uint32_t shm, hipStream_t st,
                     Args... args) {
  KernelEvents &ev = kernel_events();
  if (ev.start || ev.stop) {
    hipExtLaunchKernelGGL(kernel, grid, block, shm, st, ev.start, ev.stop, 0, args...);
    ev.start = ev.stop = nullptr;
  } else {
    // the ordinary launch: the form a stream capture records as a graph node
    hipLaunchKernelGGL(kernel, grid, block, shm, st, args...);
  }
}

constexpr int N_XCD = 8;   // accelerator dies, one L2 each

// Token groups on dies.  The scoring launches keep a group of TOK_GROUP
// consecutive tokens on one die, g on die g % N_XCD, so that a token's
// logits are read where they were written (in that die's L2).  Workgroup b
// of such a launch runs on die b % N_XCD; with `per` workgroups per group it
// takes group g = b % N_XCD + N_XCD * (q / per) and share q % per of it (q =
// b / N_XCD).  The launch has xcd_grid(groups, per) workgroups; those past
// the last group have nothing to do.
constexpr int TOK_GROUP = 16;
__host__ __device__ inline int xcd_grid(int groups, int per) {
  return N_XCD * ((groups + N_XCD - 1) / N_XCD) * per;
}
__device__ inline void xcd_group(int b, int per, int &g, int &share) {
  const int q = b / N_XCD;
  g = b % N_XCD + N_XCD * (q / per);
  share = q % per;
}

constexpr int MAX_SHARED = 8;               // shared experts per layer
constexpr int MAX_SLOTS = MAX_E + MAX_SHARED;  // kept slots + shared slots

// Upper bound (host-known) of the FFN's 16-pair tiles for a batch over all
// kept slots and the ns shared slots (B pairs each).
inline int ffn_max_tiles(int B, int K, int budget, int ns) {
  return (B * K + 15) / 16 + budget + ns * ((B + 15) / 16);
}

// The grouped bf16 FFN (see "Grouped bf16 FFN" in ffn.hip).  A part is at
// most FFN_GU_PT (gate/up) or FFN_DN_PT (down) 16-pair tiles of one kept or
// shared slot; a unit of work is (part, row group), one per workgroup of
// FFN_WAVES wavefronts at a time, each wavefront owning 16-row tiles over the
// whole contraction with weights requested FFN_GU_DW (gate/up) or FFN_DN_DW
// (down) k-steps ahead and token fragments FFN_GU_DT steps (two k-steps each,
// one step further ahead than the weights) or FFN_DN_DT k-steps ahead (the
// deep down instance: one k-step further ahead than its weights).
constexpr int FFN_WAVES = 8;
constexpr int FFN_GU_DW = 8;
constexpr int FFN_GU_DT = FFN_GU_DW / 2 + 1;
constexpr int FFN_DN_DW = 2;
constexpr int FFN_DN_DT = 2;
// wavefronts per SIMD the down kernel's registers allow: three workgroups
// per CU, so that a die's down units mostly run in one round
constexpr int FFN_DN_WPE = 6;
// down with a long contraction (more than FFN_DN_LONG_KS k-steps of I): few
// units that each stream many k-steps, so more weights in flight per
// wavefront and one workgroup per CU
constexpr int FFN_DN_LONG_KS = 64;
constexpr int FFN_DN_DW_LONG = 8;
constexpr int FFN_DN_WPE_LONG = 2;
__host__ __device__ inline bool ffn_dn_long(int I) { return I / 32 > FFN_DN_LONG_KS; }
// down for launches with few kept slots (fewer than 4 per die, so that the
// compaction cuts each slot's row groups over the dies): fewer units, so
// four k-steps of weights in flight and two workgroups per CU
constexpr int FFN_DN_DW_MID = 4;
constexpr int FFN_DN_WPE_MID = 4;
// down's instance: 2 long contraction, 1 few slots (budget + shared ones),
// 0 otherwise
__host__ __device__ inline int ffn_dn_kind(int budget, int ns, int I) {
  return ffn_dn_long(I) ? 2 : (budget + ns < 4 * N_XCD ? 1 : 0);
}
constexpr int FFN_GU_PT = 6;
constexpr int FFN_DN_PT = 8;
// gate/up reads its token rows straight from the hidden states: entry i of
// gate/up unit k's row is the byte offset of the row of its part's pair i,
// tokoff[k * FFN_GU_TOK + i] = t * d * 2 (written for the part's pairs only)
constexpr int FFN_GU_TOK = FFN_GU_PT * 16;
constexpr uint32_t FFN_TOK_PAD = 0x80000000u;   // past every x: a buffer load returns zero
static_assert(FFN_GU_PT <= FFN_WAVES, "one token tile per gate/up wavefront");
static_assert((size_t)MAX_B * 16384 * 2 < FFN_TOK_PAD, "token row offsets below the pad mark");

// Small batches, at most FFN_SPLIT_B tokens (FFN_SPLIT_LONG_B when down's
// contraction is long): the fused layer makes its plan in one launch
// (k_plan_split) and the bf16 FFN takes its split kernels (see "Small batches"
// in ffn.hip), which need no unit tables.  A slot then holds at most four
// 16-pair tiles and the FFN is a weight stream.  Measured per layer against the
// unit kernels and two plan launches (us): Qwen3-shaped, ten kept experts, B = 1
// 60 -> 38, B = 16 65 -> 45, B = 48 67 -> 54; 32 kept, B = 64 95 -> 87;
// OLMoE-shaped B = 32 76 -> 63, B = 64 79 -> 71; row-major Qwen1.5-MoE-shaped B =
// 31 120 -> 103, B = 61 127 -> 115; Mixtral-shaped B = 32 295 -> 268.  Long
// contractions between 32 and 64 tokens gain and lose (Mixtral-shaped B = 64 295
// -> 300; the layer split against unit kernels, d = 512 to 4096: 36 and 48 tokens
// on 2 slots, I = 5504 and 4800, 1.27 and 1.20 times faster, 48 on 42, I = 2112,
// 1.02, 60 and 64 on 4, I = 4416 and 5952, 0.88).
constexpr int FFN_SPLIT_B = 64, FFN_SPLIT_LONG_B = 32;
__host__ __device__ inline bool ffn_small(int B, int I) {
  return B <= (ffn_dn_long(I) ? FFN_SPLIT_LONG_B : FFN_SPLIT_B);
}
// The split kernels read a slot's token rows four times as often as the unit
// kernels (a workgroup has two row-pair tiles, not eight), so what they lose
// grows with the pairs past a slot's first 16 and with the expert's size, and
// what they gain is mostly fixed, the launches' starts and steps.  The line is
// (pairs - 16 slots) d I = FFN_SPLIT_EXTRA; over 800 packed layers of B <= 64
// (20 MB to 1.4 GB of kept weights, split against unit kernels, the fused layer
// and base_moe_forward): every slot full, B = 64, 16 slots of d = 4096, I = 2048
// 223 and 222 us split, 196 and 173 with units; 10 slots of d = 2048, I = 2048
// 104 and 86 against 95 and 70; 4 slots of d = 2048, I = 1408 (below the line)
// 43 and 35 against 59 and 45.  Below the line the split kernels win by 1.2
// times in the mean, just below it the fused layer by a few per cent, with the
// plan launch it saves, and base_moe_forward, which saves none, loses up to 1.16
// times (8 slots of d = 4096, I = 1280, B = 60: 105 and 79 us split, 106 and 67
// with units); the two have to take the same kernels.  With at most 16 tokens no
// slot has more than one tile.  Row-major weights would keep the split
// kernels longer (8 of 217 layers past the line, by up to 1.17 times: the unit
// kernels read them 64 bytes at a time), but both layouts have to take the same
// sums.
constexpr int64_t FFN_SPLIT_EXTRA = 1800000000;
inline bool ffn_split(int B, int K, int d, int I, int budget, int ns) {
  if (!ffn_small(B, I)) return false;
  if (B <= 16) return true;
  const int kept = budget < B * K ? budget : B * K;
  const int64_t pairs = (int64_t)B * ((K < kept ? K : kept) + ns);
  return (pairs - 16 * (kept + ns)) * d * I <= FFN_SPLIT_EXTRA;
}

// Slot s of a small batch for the split kernels, one copy per die (written by
// the plan's workgroup on that die, so that the FFN's first loads hit that
// die's L2): expert u (u >= E: shared expert u - E), first pair and pair count
// (0: nothing kept).  Records 0 .. budget - 1 are the kept slots, budget + i
// shared expert i; the die's copy of the pair list's tokens lies beside it.
struct alignas(16) SpRec {
  int32_t u, p0, n, pad;
};

// A unit: expert u (u >= E: shared expert u - E), the part's first 16-pair
// tile, its tile count, its first pair in the compacted order and its pair
// count, and the unit's row group (gate/up: hdr.rp_gu row-pair tiles;
// down: hdr.rt_dn row tiles).
struct alignas(32) FfnUnit {
  int32_t u, tile0, nt, p0, n, rg, pad0, pad1;
};
// Die x's header, written by the compaction workgroup that ran on die x:
// gate/up's row group (rp_gu row-pair tiles), down's (rt_dn row tiles) and
// die x's runs of units, [gu0, gu1) of the gate/up table and [dn0, dn1) of
// the down table.
struct alignas(32) FfnHdr {
  int32_t rp_gu, gu0, gu1, dn0, dn1, rt_dn, pad1, pad2;
};

// Upper bound of the parts of a launch with at most pt tiles per part: the
// sum over slots of ceil(tiles / pt) is below tiles / pt + slots.
inline int ffn_parts_bound(int B, int K, int budget, int ns, int pt) {
  return ffn_max_tiles(B, K, budget, ns) / pt + budget + ns + 1;
}
// Upper bounds of the units: every part times its row groups (gate/up: at
// least FFN_WAVES / 2 row-pair tiles per group; down: at least 2 row tiles).
inline int ffn_units_bound_gu(int B, int K, int budget, int ns, int I) {
  return ffn_parts_bound(B, K, budget, ns, FFN_GU_PT) * ((I / 16 + FFN_WAVES / 2 - 1) / (FFN_WAVES / 2));
}
inline int ffn_units_bound_dn(int B, int K, int budget, int ns, int d) {
  return ffn_parts_bound(B, K, budget, ns, FFN_DN_PT) * ((d / 16 + 1) / 2);
}
// Workgroups of the FFN launches: a multiple of N_XCD, from the device's
// compute units -- gate/up one per CU (its registers allow no second), down
// FFN_DN_WPE / 2 (FFN_DN_WPE_MID / 2, FFN_DN_WPE_LONG / 2) per CU: a
// workgroup of FFN_WAVES wavefronts puts two on each SIMD.
__host__ __device__ inline unsigned ffn_cu_grid(int n_cu) { return (unsigned)(((n_cu + N_XCD - 1) / N_XCD) * N_XCD); }
__host__ __device__ inline unsigned ffn_gu_grid(int n_cu) { return ffn_cu_grid(n_cu); }
__host__ __device__ inline unsigned ffn_dn_grid(int n_cu, int kind) {
  const int wpe = kind == 2 ? FFN_DN_WPE_LONG : kind == 1 ? FFN_DN_WPE_MID : FFN_DN_WPE;
  return (unsigned)(wpe / 2) * ffn_cu_grid(n_cu);
}

// Few dot products: k_scores_small, which may also take the predictor's rows.
// With the predictor the line is B <= 64 or B E <= 64 * 128 (its comment in
// scores.hip has both sides).  Every expert's row against the tail's K routed
// ones, the layer over E = 8 to 256, d = 1024 to 16384, K = 1 to 16: up to 48
// tokens never slower, up to 1.13 times faster (E = 64, d = 16384, K = 8, B = 1
// 62.5 us in the tail, 55.5 here); from 49 to 64 still up to 1.07 times faster (E =
// 200, d = 8192, K = 16 93.8 and 87.6), but 2 to 8% slower at E = 128 and 256 with
// few routes (E = 256, d = 4096, B = 64, K = 1 53.3 and 56.6, K = 8 63.7 and 65.1).
// No product of E, d and K separates the two.
constexpr int SC_SMALL_B = 64, SC_SMALL_DOTS = 64 * 128;
inline bool scores_small(int B, int E) { return B <= SC_SMALL_B || B * E <= SC_SMALL_DOTS; }
// Without the predictor (base_route, the other rules, a gate alone with E = 0)
// the tiles win for bf16 tokens where a wavefront's ring has nothing to hide, d
// <= 512, and past 128 rows, both with more tokens than two wavefronts of a group
// take (base_route, us, tiled against small: E = 64, B = 16 d = 256 5.4 and 5.7, d
// = 1024 6.5 and 6.2, d = 4096 12.2 and 9.6; E = 64, B = 8, d = 512 5.8 and 5.2; E =
// 3, B = 13, d = 256 4.9 and 5.6; E = 135, B = 13, d = 1536 10.6 and 11.6; E = 160, B
// = 32 d = 512 8.9 and 9.8, d = 2048 12.4 and 12.3; E = 256, B = 8 d = 256 8.0 and
// 8.6, d = 2048 12.4 and 10.5; a gate alone, the staged call, B = 300 d = 256 26.3
// and 27.3, d = 4096 65.0 and 62.6).  fp32 tokens, twice the bytes to stage, never
// (E = 1, B = 64, d = 256 6.4 and 5.5; E = 256, B = 64 d = 256 10.4 and 9.7, d = 2048
// 24.7 and 13.3).
inline bool scores_small_router(bool bf16, int B, int E, int d) {
  const bool few = E <= 128, ring = d > 512;
  return scores_small(B, E) && (!bf16 || (B <= TOK_GROUP / 2 ? few || ring : few && ring));
}
// rows: n_router of Wr (logits, + beta), then the vector G when given (gdot);
// scores_small launches may also take the predictor's rows A [n_router]: the
// dot products of every expert (q [B][n_router]) and ||x||^2 (ss [B])
hipError_t launch_scores(bool bf16, const void *x, int B, int d, const float *Wr,
                         const float *beta, int n_router, const float *G, float *logits,
                         float *gdot, hipStream_t st, const float *A = nullptr,
                         float *q = nullptr, float *ss = nullptr);
// Selection rules (the values of BASE_SCORE_* in base.h): the per-pair
// score k_tail writes as the cost
constexpr int SCORE_BASE = 0, SCORE_TOP1 = 1, SCORE_WEIGHT = 2, SCORE_WEIGHT_SQ = 3,
              SCORE_STATIC = 4;
// mode bit 0: top-K + weights from logits; bit 1: per-pair scores of `rule`
// (SCORE_BASE: the predictor a_u . x / ||x|| from x (rows of d) and A)
// order / ex / den (optional, route mode): per token the experts in rank
// order [B][E] (bytes), exp(l - l_max) in rank order [B][E] and the router's
// softmax denominator S [B], for the fused layer's backfill
// q / ss (optional, SCORE_BASE): the predictor's dot products and ||x||^2 from
// launch_scores; x and A are then not read
hipError_t launch_tail(bool bf16, int B, int E, int K, int d, int norm_topk,
                       const float *logits, const void *x, const float *A, const float *bp,
                       int32_t *ids, float *w, float *cost, int mode, int rule,
                       hipStream_t st, uint8_t *order = nullptr, float *ex = nullptr,
                       float *den = nullptr, const float *q = nullptr,
                       const float *ss = nullptr);
// binary: rank by (score > 0) instead of the score (the top-1-union rule)
hipError_t launch_select(int B, int K, int E, const int32_t *ids,
                         const float *cost, int budget, bool binary, float *scores,
                         int32_t *counts, int32_t *sel_ids, int32_t *n_sel,
                         int32_t *slot_of, hipStream_t st);
// selection and backfill in one launch (same results as the two launches)
// (order / ex / den: k_tail's rank rows and denominators of the batch)
hipError_t launch_select_backfill(int B, int K, int E, const int32_t *ids, const float *cost,
                                  int budget, bool binary, int flags, const uint8_t *order,
                                  const float *ex, const float *den, float *scores,
                                  int32_t *counts, int32_t *sel_ids, int32_t *n_sel,
                                  int32_t *slot_of, int32_t *exec_ids, float *exec_gates,
                                  int n_cu, hipStream_t st);
// selection, backfill and compaction in one launch, for ffn_small batches
// (same results as the three); rec / sptok (bf16 layers, else null): the split
// kernels' records and token lists
hipError_t launch_plan_split(int B, int K, int E, int budget, int ns, bool binary, int flags,
                             const int32_t *ids, const float *cost, const uint8_t *order,
                             const float *ex, const float *den, const float *gdot,
                             float *scores, int32_t *counts, int32_t *sel_ids, int32_t *n_sel,
                             int32_t *slot_of, int32_t *exec_ids, float *exec_gates,
                             int32_t *offsets, int32_t *pair_tok, float *pair_gate,
                             int32_t *pair_of, SpRec *rec, int32_t *sptok, hipStream_t st);
hipError_t launch_backfill(int B, int E, int K, int norm_topk, int flags,
                           const float *logits, const int32_t *ids,
                           const int32_t *slot_of, const int32_t *n_sel,
                           int32_t *exec_ids, float *exec_gates,
                           hipStream_t st);
// ns shared slots follow the kept ones (expert E + i, every token, gate
// sigmoid(gdot[t]) or 1 when gdot is null).  With `tables` (bf16 layers)
// the same launch also writes the FFN's unit tables (units_gu, units_dn, of
// at most ffn_units_bound_gu / _dn rows), the per-die headers and gate/up's
// token row offsets (tokoff, FFN_GU_TOK per gate/up unit; d: the hidden
// size); n_cu: the device's compute units (the FFN launches' sizes follow
// from it).  Without tables, rec / sptok (may be null) as launch_plan_split.
hipError_t launch_compact(int B, int K, int E, int budget, int ns, const int32_t *exec_ids,
                          const float *exec_gates, const int32_t *slot_of,
                          const int32_t *n_sel, const float *gdot, int32_t *offsets,
                          int32_t *pair_tok, float *pair_gate,
                          int32_t *pair_of, const int32_t *sel_ids, bool tables, int d,
                          int I, uint32_t *tokoff, FfnHdr *hdr, FfnUnit *units_gu,
                          FfnUnit *units_dn, SpRec *rec, int32_t *sptok, int n_cu,
                          hipStream_t st);
hipError_t launch_pack(const void *w13, const void *w2, void *w13p, void *w2p,
                       int E, int d, int I, hipStream_t st);
// slots: at most this many kept slots (budget, or fewer where the kept set is
// known to come from this batch's routes)
// parts of expert u >= E read the shared experts' weights (w13s / w2s, u - E)
hipError_t launch_gateup(bool bf16, bool packed, const void *x, int B, int d,
                         int I, int E, int K, int budget, int slots, int ns, const void *w13,
                         const void *w13s,
                         const int32_t *sel_ids, const int32_t *n_sel,
                         const int32_t *offsets, const int32_t *pair_tok,
                         const FfnHdr *hdr, const FfnUnit *units, int n_cu,
                         const uint32_t *tokoff, const SpRec *rec, const int32_t *sptok, void *H,
                         hipStream_t st);   // rec: the split kernels, else the unit kernels
hipError_t launch_down(bool bf16, bool packed, int B, int d, int I, int E, int K,
                       int budget, int slots, int ns, const void *w2, const void *w2s,
                       const int32_t *sel_ids,
                       const int32_t *n_sel, const int32_t *offsets,
                       const FfnHdr *hdr, const FfnUnit *units, const SpRec *rec, int n_cu,
                       const float *pair_gate, const void *H, float *pairbuf, hipStream_t st);
// kc: columns of pair_of (K routed + the shared experts)
hipError_t launch_combine(bool bf16, int B, int d, int kc,
                          const int32_t *pair_of, const float *pairbuf,
                          const void *residual, void *y, hipStream_t st);

// Calibration statistics (per expert u): head[u] = (n, sum y, sum y^2, 0)
// fp64, sz[u][d] and q[u][d] fp64, G[u][d][d] fp32; each array 256-byte
// aligned in the caller's buffer, in this order.
struct CalibStats {
  double *head, *sz, *q;
  float *G;
};
inline size_t calib_up256(size_t v) { return (v + 255) & ~(size_t)255; }
inline size_t calib_stats_bytes(int E, int d) {
  return calib_up256((size_t)E * 4 * 8) + 2 * calib_up256((size_t)E * d * 8) +
         calib_up256((size_t)E * d * d * 4);
}
inline CalibStats calib_stats_at(void *base, int E, int d) {
  char *p = static_cast<char *>(base);
  CalibStats s;
  s.head = reinterpret_cast<double *>(p);
  p += calib_up256((size_t)E * 4 * 8);
  s.sz = reinterpret_cast<double *>(p);
  p += calib_up256((size_t)E * d * 8);
  s.q = reinterpret_cast<double *>(p);
  p += calib_up256((size_t)E * d * 8);
  s.G = reinterpret_cast<float *>(p);
  return s;
}
hipError_t launch_calib_zero(void *stats, size_t bytes, hipStream_t st);
hipError_t launch_calib_stats(const void *x, bool bf16, int B, int d, int E, int K,
                              const float *pairbuf, const int32_t *n_sel,
                              const int32_t *sel_ids, const int32_t *offsets,
                              const int32_t *pair_tok, double *inv, double *y, float *zbuf,
                              CalibStats st, hipStream_t s);

// internal flags bit of the backfill: unit gates (calibration runs the
// experts' own outputs)
constexpr int FLAG_UNIT_GATES = 4;

}  // namespace basek
