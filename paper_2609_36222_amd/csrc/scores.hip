// Router logits and the per-token tail of the scoring path (Sec. 3.1
// router; Sec. 3.4, eq. log_energy_predictor).
//
// k_scores  the router's dot products for a batch, as a tiled batch x rows
//           product: logit l[t][e] = x_t . W_r[e] + beta_e (and, with shared
//           experts gated by a vector, gdot[t] = x_t . g).
// k_scores_small  the same straight into registers, for few dot products; for
//           the fused layer's small batches also the predictor's dot products
//           with every expert and ||x||^2.
// k_tail    one workgroup per token: top-K by exact ranks, router weights,
//           then the score of each routed pair.  For the method's own rule
//           the pair's predicted removal cost w^2 exp(q / ||x|| + b_u), q =
//           a_u . x_t, from k_scores_small's dot products or else from ones
//           made here for the K routed experts only (App. "Custom GPU
//           Kernels": the token is normalised once and reused across its K
//           experts), wavefront w taking routes 2w and 2w + 1; the other
//           rules need only the routes.
//
// Fixed fp32 order of every dot product of length d: partial j (0..63) owns
// the elements 256m + 4j + r (r = 0..3) and accumulates them in ascending
// element order with single-rounding FMA from +0; the 64 partials are then
// joined by the halving tree "s[j] = s[j] + s[j + h], j < h" for h = 32 ..
// 1.  Lane j of a wavefront holds partial j.  A halving-tree level is a
// lane exchange over distance h, so the tree runs on lane shuffles (see
// tree16 and wave_tree_sum: any lane holding partial j^m of the same dot at
// each level gives the same sums).
#include "common.hpp"
#include "internal.hpp"

namespace basek {

constexpr int SC_T = 4;        // tokens per wavefront tile
constexpr int SC_R = 4;        // matrix rows per wavefront tile
constexpr int SC_WT = 4;       // wavefronts of a workgroup along tokens
constexpr int SC_WR = 2;       // wavefronts of a workgroup along rows
constexpr int SC_WAVES = SC_WT * SC_WR;
constexpr int SC_TB = SC_T * SC_WT;           // tokens per workgroup
constexpr int SC_RB = SC_R * SC_WR;           // rows per workgroup
constexpr int SC_CH = 256;                    // elements per chunk
constexpr int SC_PF = 2;                      // chunks requested ahead (register stages)
static_assert(SC_T * SC_R == 16, "tree16 joins 16 dot products");
static_assert(SC_TB == TOK_GROUP, "a workgroup's tokens are one group");

// Four consecutive elements of a token row as loaded (bf16 bits or fp32),
// widened only where used, so that holding a request does not wait for it.
template <typename XT> struct Raw4;
template <> struct Raw4<uint16_t> {
  u32x2 v;
  __device__ __forceinline__ void load(const uint16_t *p) { v = *reinterpret_cast<const u32x2 *>(p); }
  __device__ __forceinline__ float at(int r) const {
    const uint32_t h = (r < 2) ? v.x : v.y;
    return __uint_as_float((r & 1) ? (h & 0xFFFF0000u) : (h << 16));
  }
};
template <> struct Raw4<float> {
  float4 v;
  __device__ __forceinline__ void load(const float *p) { v = *reinterpret_cast<const float4 *>(p); }
  __device__ __forceinline__ float at(int r) const {
    return r == 0 ? v.x : r == 1 ? v.y : r == 2 ? v.z : v.w;
  }
};

template <typename XT> struct XPiece;
// 8 bf16 elements, widened to fp32 on their way into LDS
template <> struct XPiece<uint16_t> {
  static constexpr int ELEMS = 8;
  u32x4 v;
  __device__ __forceinline__ void load(const uint16_t *p) { v = *reinterpret_cast<const u32x4 *>(p); }
  __device__ __forceinline__ void put(float *dst) const {
    *reinterpret_cast<float4 *>(dst) =
        float4{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u),
               __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xFFFF0000u)};
    *reinterpret_cast<float4 *>(dst + 4) =
        float4{__uint_as_float(v.z << 16), __uint_as_float(v.z & 0xFFFF0000u),
               __uint_as_float(v.w << 16), __uint_as_float(v.w & 0xFFFF0000u)};
  }
};
template <> struct XPiece<float> {
  static constexpr int ELEMS = 4;
  float4 v;
  __device__ __forceinline__ void load(const float *p) { v = *reinterpret_cast<const float4 *>(p); }
  __device__ __forceinline__ void put(float *dst) const { *reinterpret_cast<float4 *>(dst) = v; }
};

// Staging of one 256-element chunk of the workgroup's SC_TB token rows and
// SC_RB matrix rows: XP token pieces and WP row pieces (16 bytes each) per
// thread.
template <typename XT>
struct ScStage {
  static constexpr int XE = XPiece<XT>::ELEMS;
  static constexpr int XB = SC_TB * SC_CH / XE;    // token pieces
  static constexpr int WB = SC_RB * SC_CH / 4;     // row pieces
  static constexpr int XP = XB / (SC_WAVES * WAVE), WP = WB / (SC_WAVES * WAVE);
  static_assert(XB % (SC_WAVES * WAVE) == 0 && WB % (SC_WAVES * WAVE) == 0,
                "staging pieces per thread");
  XPiece<XT> xv[XP];
  float4 wv[WP];
};

// rows r < n_router: W_r (logits, + beta); with G != nullptr one more row,
// the shared experts' gate vector (gdot).  A workgroup covers one token
// group (16 tokens) x 8 rows (4 x 2 wavefronts of 4 x 4), every row group of
// token group g on die g % N_XCD (xcd_group); each 256-element chunk of its
// rows is staged once in LDS (tokens widened to fp32), the next chunk's
// loads in flight meanwhile.  Grid xcd_grid(ceil(B / 16), ceil(rows / 8)).
template <typename XT>
__global__ __launch_bounds__(SC_WAVES * WAVE, 2)
void k_scores(const XT *__restrict__ x, int B, int d,
              const float *__restrict__ Wr, const float *__restrict__ beta,
              int n_router, const float *__restrict__ G, float *__restrict__ logits,
              float *__restrict__ gdot) {
  using St = ScStage<XT>;
  constexpr int XE = St::XE;
  __shared__ __attribute__((aligned(16))) float xs[2][SC_TB][SC_CH];
  __shared__ __attribute__((aligned(16))) float wsh[2][SC_RB][SC_CH];
  const int tid = threadIdx.x, lane = lane_id(), wv = wave_id();
  const int tw = wv % SC_WT, rw = wv / SC_WT;
  const int rows = n_router + (G ? 1 : 0);
  int tg, rg;
  xcd_group(blockIdx.x, (rows + SC_RB - 1) / SC_RB, tg, rg);
  if (tg * SC_TB >= B) return;
  const int tb0 = tg * SC_TB, rb0 = rg * SC_RB;

  // the thread's staging pieces: token row / matrix row and column
  const XT *xsrc[St::XP];
  const float *wsrc[St::WP];
  int xt[St::XP], xc[St::XP], wr[St::WP], wc[St::WP];
#pragma unroll
  for (int i = 0; i < St::XP; ++i) {
    const int c = tid + i * SC_WAVES * WAVE;
    xt[i] = c / (SC_CH / XE);
    xc[i] = (c % (SC_CH / XE)) * XE;
    xsrc[i] = x + (size_t)min(tb0 + xt[i], B - 1) * d + xc[i];
  }
#pragma unroll
  for (int i = 0; i < St::WP; ++i) {
    const int c = tid + i * SC_WAVES * WAVE;
    wr[i] = c / (SC_CH / 4);
    wc[i] = (c % (SC_CH / 4)) * 4;
    const int r = min(rb0 + wr[i], rows - 1);
    wsrc[i] = (r < n_router ? Wr + (size_t)r * d : G) + wc[i];
  }
  St st[SC_PF];
  auto fetch = [&](St &sg, int m) {
#pragma unroll
    for (int i = 0; i < St::XP; ++i) sg.xv[i].load(xsrc[i] + m);
#pragma unroll
    for (int i = 0; i < St::WP; ++i) sg.wv[i] = *reinterpret_cast<const float4 *>(wsrc[i] + m);
  };
  auto put = [&](const St &sg, int b) {
#pragma unroll
    for (int i = 0; i < St::XP; ++i) sg.xv[i].put(&xs[b][xt[i]][xc[i]]);
#pragma unroll
    for (int i = 0; i < St::WP; ++i) *reinterpret_cast<float4 *>(&wsh[b][wr[i]][wc[i]]) = sg.wv[i];
  };

  float acc[SC_T * SC_R];
#pragma unroll
  for (int i = 0; i < SC_T * SC_R; ++i) acc[i] = 0.0f;
  const int nch = d / SC_CH;
  // register stage q holds the chunks m = q (mod SC_PF); chunk m + 1 goes
  // to LDS while chunk m is used, chunk m + SC_PF is requested meanwhile
#pragma unroll
  for (int q = 0; q < SC_PF; ++q) {
    if (q < nch) fetch(st[q], q * SC_CH);
    __builtin_amdgcn_sched_barrier(0);
  }
  put(st[0], 0);
  lds_barrier();
  for (int m0 = 0; m0 < nch; m0 += SC_PF) {
#pragma unroll
    for (int q = 0; q < SC_PF; ++q) {
      const int m = m0 + q;
      if (m < nch) {
        const int buf = m & 1;
        // this lane's elements 4 lane .. 4 lane + 3 of the chunk
        float4 xv[SC_T], wv4[SC_R];
#pragma unroll
        for (int a = 0; a < SC_T; ++a)
          xv[a] = *reinterpret_cast<const float4 *>(&xs[buf][tw * SC_T + a][4 * lane]);
#pragma unroll
        for (int b = 0; b < SC_R; ++b)
          wv4[b] = *reinterpret_cast<const float4 *>(&wsh[buf][rw * SC_R + b][4 * lane]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
          for (int a = 0; a < SC_T; ++a) {
            const float xe = r == 0 ? xv[a].x : r == 1 ? xv[a].y : r == 2 ? xv[a].z : xv[a].w;
#pragma unroll
            for (int b = 0; b < SC_R; ++b) {
              const float we = r == 0 ? wv4[b].x : r == 1 ? wv4[b].y : r == 2 ? wv4[b].z : wv4[b].w;
              acc[a * SC_R + b] = __builtin_fmaf(xe, we, acc[a * SC_R + b]);
            }
          }
        }
        if (m + 1 < nch) {
          // buffer buf ^ 1 was last read for chunk m - 1, before the
          // previous barrier
          put(st[(q + 1) % SC_PF], buf ^ 1);
          lds_barrier();
        }
        __builtin_amdgcn_sched_barrier(0);
        if (m + SC_PF < nch) fetch(st[q], (m + SC_PF) * SC_CH);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // dot i of the tile (token a = i / SC_R, row b = i % SC_R) ends in the
  // lanes 4i .. 4i + 3
  const float v = tree16(acc);
  const int i = lane >> 2;
  const int t = tb0 + tw * SC_T + i / SC_R, r = rb0 + rw * SC_R + i % SC_R;
  if ((lane & 3) == 0 && t < B && r < rows) {
    if (r < n_router)
      logits[(size_t)t * n_router + r] = beta ? v + beta[r] : v;
    else
      gdot[t] = v;
  }
}

// Few dot products (scores_small, scores_small_router).  The tiled kernel's few
// workgroups (16 at B <= 16, on one die) walk their chunks behind LDS barriers;
// here a wavefront takes 4 tokens x 4 rows straight into registers, SS_GC chunks
// of 256 elements at a time with the next ones in flight, and nothing is shared,
// so the launch is a ring of loads (d = 2048: four stages, two of them in flight
// at once), 64 FMAs a chunk and a tree.  With the chip
// otherwise idle it also makes the predictor's dot products with every
// expert (A, q) and ||x||^2 (ss), which k_tail would otherwise start only once
// the routing is known.  Each dot product in the fixed order.  The extra rows
// go through the same ring (as a plain loop, one round trip a chunk, they were
// the launch's longest wavefronts: d = 4096, a staged layer with a gate, B = 16,
// 27.2 us, now 26.6; d = 16384 at B = 1 48.6 and 46.4, the fused layer 65.1 and
// 58.1).
// A workgroup is 4 wavefronts: 16 tokens (a token group) x 4 rows.  The router
// rows of token group g run on die g % N_XCD, where k_tail reads the logits;
// the predictor's and the extra rows (G; x itself) on the dies without a token
// group, or, past N_XCD / 2 groups, on the group's own: workgroup b on die b %
// N_XCD is number b / N_XCD there.
// Scores + tail, against the tiled kernel and the predictor in the tail (E =
// 128, d = 2048, us): B = 1 7.6 + 5.1 -> 4.8 + 4.0, B = 16 7.8 + 5.5 -> 5.7 + 4.0,
// B = 64 8.0 + 5.6 -> 7.6 + 4.0; E = 8, d = 4096, B = 16 13.3 + 4.8 -> 9.0 +
// 4.0.  The line, B <= 64 or B E <= 64 * 128: beyond, the unshared reads (48 KB a
// wavefront) catch up with what the tiles save (E = 128: layer at B = 80 66.4
// tiled, 67.7 here; B = 128 87.8, 87.2; B = 256 111, 115), below they gain (E =
// 64: B = 72 76.9 -> 73.8, B = 128 84.2 -> 81.4; E = 8, d = 4096: B = 128 299.7
// -> 293.6, B = 1000 1041 -> 1036); what it excepts:
// scores_small_router.  Four chunks at a time: equal, slower at d = 256.
constexpr int SS_GC = 2;

template <typename XT>
__global__ __launch_bounds__(4 * WAVE, 2)
void k_scores_small(const XT *__restrict__ x, int B, int d, const float *__restrict__ Wr,
                    const float *__restrict__ beta, int E, const float *__restrict__ A,
                    const float *__restrict__ G, int n_group, int n_other,
                    float *__restrict__ logits, float *__restrict__ q, float *__restrict__ ss,
                    float *__restrict__ gdot) {
  const int lane = lane_id(), w = wave_id_u();
  const int die = blockIdx.x % N_XCD, nb = blockIdx.x / N_XCD;
  const int rgs = (E + 3) / 4;   // row groups of 4
  const int per = n_other / n_group;   // a token group's others: predictor groups, one of extras
  int g, rg;
  bool router = die < n_group;
  if (n_group > N_XCD / 2) {
    const int q = nb / (rgs + per);
    g = die + N_XCD * q;
    rg = nb - q * (rgs + per);
    router = rg < rgs;
    if (!router) rg -= rgs;
  } else if (router) {
    g = die;
    rg = nb;
    if (rg >= rgs) return;
  } else {
    const int i = nb * (N_XCD - n_group) + die - n_group;
    if (i >= n_other) return;
    g = i / per;
    rg = i - g * per;
  }
  const int t0 = g * TOK_GROUP + 4 * w;
  if (t0 >= B) return;
  const bool extra = !router && (A == nullptr || rg >= rgs);
  const XT *xr[4];
  const float *wr[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) xr[a] = x + (size_t)min(t0 + a, B - 1) * d + 4 * lane;
#pragma unroll
  for (int b = 0; b < 4; ++b)
    wr[b] = extra ? (G ? G + 4 * lane : nullptr)
                  : (router ? Wr : A) + (size_t)min(4 * rg + b, E - 1) * d + 4 * lane;
  float acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
  // the rows' chunks through a ring of two stages of SS_GC chunks: load(s, c, m)
  // requests the matrix rows of the chunk at element m, use(s, c) adds it
  Raw4<XT> xv[2][SS_GC][4];
  float4 wv[2][SS_GC][4];
  auto stream = [&](auto load, auto use) {
    auto fetch = [&](int s, int m0) {
#pragma unroll
      for (int c = 0; c < SS_GC; ++c) {
        const int m = min(m0 + 256 * c, d - 256);   // past the end: not used
        load(s, c, m);
#pragma unroll
        for (int a = 0; a < 4; ++a) xv[s][c][a].load(xr[a] + m);
      }
    };
    auto add = [&](int s, int m0) {
#pragma unroll
      for (int c = 0; c < SS_GC; ++c) {
        if (m0 + 256 * c >= d) break;
        use(s, c);
      }
    };
    fetch(0, 0);
    for (int m0 = 0; m0 < d; m0 += 2 * SS_GC * 256) {
      fetch(1, m0 + SS_GC * 256);
      __builtin_amdgcn_sched_barrier(0);
      add(0, m0);
      __builtin_amdgcn_sched_barrier(0);
      if (m0 + 2 * SS_GC * 256 < d) fetch(0, m0 + 2 * SS_GC * 256);
      __builtin_amdgcn_sched_barrier(0);
      if (m0 + SS_GC * 256 < d) add(1, m0 + SS_GC * 256);
    }
  };
  // rows: 0 x itself (also where ss is not asked for: its FMAs hide behind the
  // loads), 1 G
  if (extra) {
    stream(
        [&](int s, int c, int m) {
          wv[s][c][0] = G ? *reinterpret_cast<const float4 *>(wr[0] + m) : float4{0.f, 0.f, 0.f, 0.f};
        },
        [&](int s, int c) {
          const float gv[4] = {wv[s][c][0].x, wv[s][c][0].y, wv[s][c][0].z, wv[s][c][0].w};
#pragma unroll
          for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float xe = xv[s][c][a].at(r);
              acc[4 * a] = __builtin_fmaf(xe, xe, acc[4 * a]);
              acc[4 * a + 1] = __builtin_fmaf(xe, gv[r], acc[4 * a + 1]);
            }
        });
  } else {
    stream(
        [&](int s, int c, int m) {
#pragma unroll
          for (int b = 0; b < 4; ++b) wv[s][c][b] = *reinterpret_cast<const float4 *>(wr[b] + m);
        },
        [&](int s, int c) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
              const float xe = xv[s][c][a].at(r);
#pragma unroll
              for (int b = 0; b < 4; ++b) {
                const float we = r == 0   ? wv[s][c][b].x
                                 : r == 1 ? wv[s][c][b].y
                                 : r == 2 ? wv[s][c][b].z
                                          : wv[s][c][b].w;
                acc[4 * a + b] = __builtin_fmaf(xe, we, acc[4 * a + b]);
              }
            }
        });
  }
  const float v = tree16(acc);   // dot i of (token i / 4, row i % 4) in lanes 4 i ..
  const int i = lane >> 2, t = t0 + (i >> 2), b = i & 3, r = 4 * rg + b;
  if ((lane & 3) != 0 || t >= B) return;
  if (extra) {
    if (b == 0 && ss) ss[t] = v;
    if (b == 1 && G) gdot[t] = v;
  } else if (r < E) {
    if (router)
      logits[(size_t)t * E + r] = beta ? v + beta[r] : v;
    else
      q[(size_t)t * E + r] = v;
  }
}

constexpr int TL_NI = MAX_E / WAVE;
constexpr int TL_RANK = 256;                  // lanes that rank the logits
constexpr int TL_MAXW = (MAX_K + 1) / 2 > TL_RANK / WAVE ? (MAX_K + 1) / 2 : TL_RANK / WAVE;

// Wavefronts of a k_tail workgroup: the TL_RANK ranking lanes, and with the
// method's predictor one wavefront per two routes.
__host__ __device__ inline int tail_waves(int K, bool pred) {
  const int wp = pred ? (K + 1) / 2 : 0;
  return wp > TL_RANK / WAVE ? wp : TL_RANK / WAVE;
}

// w^2 exp(q / ||x|| + b), ss = ||x||^2, in the fixed order.
__device__ __forceinline__ float pair_cost(float q, float ss, float b, float w) {
  float inv = 0.0f;
  if (ss > 0.0f) {
    const float rt = sqrtf(ss);
    inv = 1.0f / rt;
  }
  float s = q * inv;
  s = s + b;
  const float w2 = w * w;
  return w2 * base_exp(s);
}

// mode bit 0: route (top-K and weights from the logits into ids / w)
// mode bit 1: per-pair scores of the routed pairs (ids / w, read back when
//             bit 0 is off) under `rule`: SCORE_BASE w^2 exp(q / ||x|| + b_u)
//             with q = a_u . x_t and ||x_t||^2 in the fixed order, read (qd,
//             ssd: k_scores_small's) or computed here; SCORE_TOP1 1 for the
//             first route, else 0; SCORE_WEIGHT w; SCORE_WEIGHT_SQ w * w;
//             SCORE_STATIC (w * w) * exp(b_u)
// One workgroup of tail_waves(K, pred) wavefronts per token, token group g on
// die g % N_XCD as in k_scores (xcd_group).  Top-K in the
// order (logit desc, index asc) of rank_key: the token's keys go to LDS and
// the first TL_RANK lanes count, for every expert, the keys that rank before
// its own -- lane g counts for expert g % E2 over stretch g / E2 of the C
// equal stretches of the keys (E2 the power of two >= E, C = min(TL_RANK /
// E2, E2)); route k is the expert of rank k.  Every wavefront then takes the
// routes and weights from LDS; wavefront w computes the predictor of routes
// 2w and 2w + 1 (without qd).
// DENSE: the method's rule on k_scores_small's dot products (qd, ssd); an
// instance of its own: the others carried its registers and LDS for 0.1 to 0.2
// us of a base_route of 8 to 13.
template <typename XT, bool DENSE>
__global__ __launch_bounds__(TL_MAXW * WAVE)
void k_tail(int B, int E, int K, int d, int norm_topk, const float *__restrict__ logits,
            const XT *__restrict__ x, const float *__restrict__ A,
            const float *__restrict__ bp, int32_t *__restrict__ ids_io,
            float *__restrict__ w_io, float *__restrict__ cost, int mode, int rule,
            uint8_t *__restrict__ order, float *__restrict__ ex, float *__restrict__ den,
            const float *__restrict__ qd, const float *__restrict__ ssd) {
  __shared__ __attribute__((aligned(16))) uint64_t keys[MAX_E];
  __shared__ float lrow[MAX_E];
  __shared__ int part[TL_RANK];
  __shared__ int route[MAX_K];
  __shared__ float qrow[DENSE ? MAX_E : 1];
  const int tid = threadIdx.x, lane = lane_id(), w = wave_id_u();
  int tg, ti;
  xcd_group(blockIdx.x, TOK_GROUP, tg, ti);
  const int t = tg * TOK_GROUP + ti;   // on the die that wrote its logits
  if (t >= B) return;
  // the predictor's dot products: made here, or (qd, ssd) by k_scores_small
  const bool pred = !DENSE && (mode & 2) && rule == SCORE_BASE;
  // the logits row (clamped, no branches, so that the loads are in flight
  // together); the method's predictor's first pass of the token row is
  // requested once the routing's inputs have arrived (it does not depend on
  // the routing, which then runs while it is in flight)
  float lv[TL_NI];
  if ((mode & 1) && w == 0) {
#pragma unroll
    for (int i = 0; i < TL_NI; ++i) lv[i] = logits[(size_t)t * E + min(lane + WAVE * i, E - 1)];
  }
  float qv[TL_NI], ssv = 0.0f;
  if (DENSE && w == 0) {   // written on other dies: they arrive while the routing runs
#pragma unroll
    for (int i = 0; i < TL_NI; ++i) qv[i] = qd[(size_t)t * E + min(lane + WAVE * i, E - 1)];
    ssv = ssd[t];
  }
  constexpr int GC = 8;   // chunks of 256 elements per pass, loads issued together
  const XT *xr = x + (size_t)t * d + 4 * lane;
  Raw4<XT> xv[GC];
  auto prefetch_x = [&]() {
    if (pred && 2 * w < K) {
#pragma unroll
      for (int c = 0; c < GC; ++c) xv[c].load(xr + min(c * 256, d - 256));
    }
  };

  int my_id = 0;       // lane k < K: routed expert k
  float my_w = 0.0f;   // and its weight
  if (!(mode & 1)) {
    my_id = ids_io[(size_t)t * K + min(lane, K - 1)];
    my_w = w_io[(size_t)t * K + min(lane, K - 1)];
    prefetch_x();
  } else {
    int E2 = 1;
    while (E2 < E) E2 <<= 1;
    if (w == 0) {
#pragma unroll
      for (int i = 0; i < TL_NI; ++i) {
        const int e = lane + WAVE * i;
        if (e < E2) {
          keys[e] = e < E ? rank_key(lv[i], e) : 0;   // 0 ranks after every expert
          lrow[e] = lv[i];
        }
      }
    }
    prefetch_x();
    __syncthreads();
    const int C = min(TL_RANK / E2, E2), len = E2 / C;
    if (tid < C * E2) {
      const int i = tid & (E2 - 1), j0 = (tid / E2) * len;
      const uint64_t ku = keys[i];
      int r = 0;
      if (len < 16) {
        for (int j = j0; j < j0 + len; ++j) r += keys[j] > ku;
      } else {
        // 16 keys per step, their LDS reads issued together
        for (int j = j0; j < j0 + len; j += 16) {
          u32x4 o[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) o[q] = *reinterpret_cast<const u32x4 *>(&keys[j + 2 * q]);
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            r += (((uint64_t)o[q].y << 32 | o[q].x) > ku);
            r += (((uint64_t)o[q].w << 32 | o[q].z) > ku);
          }
        }
      }
      part[tid] = r;
    }
    __syncthreads();
    int my_rank = 0;   // thread tid < E: the rank of expert tid
    if (tid < E) {
      for (int c = 0; c < C; ++c) my_rank += part[c * E2 + tid];
      if (my_rank < K) route[my_rank] = tid;
    }
    __syncthreads();
    my_id = route[min(lane, K - 1)];
    const float lmax = lrow[route[0]];
    const float eps = base_exp(lrow[my_id] - lmax);
    float S;
    if (norm_topk) {
      S = 0.0f;
      for (int k = 0; k < K; ++k)
        S = S + __builtin_bit_cast(float, __builtin_amdgcn_readlane(__float_as_int(eps), k));
    } else {
      float pt = 0.0f;
#pragma unroll
      for (int i = 0; i < TL_NI; ++i)
        if (lane + WAVE * i < E) pt = pt + base_exp(lrow[lane + WAVE * i] - lmax);
      S = wave_tree_sum(pt);
    }
    my_w = eps / S;
    if (w == 0 && lane < K) {
      ids_io[(size_t)t * K + lane] = my_id;
      w_io[(size_t)t * K + lane] = my_w;
    }
    if (order) {
      // for the fused layer's backfill: the experts in rank order, their
      // exp(l - l_max) in rank order, and the router's denominator S
      if (tid < E) {
        order[(size_t)t * E + my_rank] = (uint8_t)tid;
        ex[(size_t)t * E + my_rank] = base_exp(lrow[tid] - lmax);
      }
      if (tid == 0) den[t] = S;
    }
  }
  if (!(mode & 2)) return;

  const int u = (lane < K && my_id >= 0 && my_id < E) ? my_id : 0;   // out-of-range ids read row 0
  if constexpr (DENSE) {   // the method's rule on k_scores_small's dot products
    if (w != 0) return;
#pragma unroll
    for (int i = 0; i < TL_NI; ++i)
      if (lane + WAVE * i < E) qrow[lane + WAVE * i] = qv[i];
    if (lane < K) cost[(size_t)t * K + lane] = pair_cost(qrow[u], ssv, bp[u], my_w);
    return;
  }
  if (!pred) {
    if (w == 0 && lane < K) {
      float c;
      if (rule == SCORE_TOP1) {
        c = lane == 0 ? 1.0f : 0.0f;
      } else if (rule == SCORE_WEIGHT) {
        c = my_w;
      } else if (rule == SCORE_WEIGHT_SQ) {
        c = my_w * my_w;
      } else {   // SCORE_STATIC
        const float w2 = my_w * my_w;
        c = w2 * base_exp(bp[u]);
      }
      cost[(size_t)t * K + lane] = c;
    }
    return;
  }

  // this wavefront's routes k0 = 2w, k1 = 2w + 1: ||x_t||^2, q0, q1 in the
  // fixed order
  const int k0 = 2 * w, k1 = 2 * w + 1;
  if (k0 >= K) return;
  const bool has1 = k1 < K;
  const int u0 = __builtin_amdgcn_readlane(u, k0);
  const int u1 = __builtin_amdgcn_readlane(u, has1 ? k1 : k0);
  const float b_my = (lane == k0 || lane == k1) ? bp[u] : 0.0f;
  const float *a0 = A + (size_t)u0 * d + 4 * lane;
  const float *a1 = A + (size_t)u1 * d + 4 * lane;
  float ss = 0.0f, q0 = 0.0f, q1 = 0.0f;
  for (int m0 = 0; m0 < d; m0 += GC * 256) {
    float av0[GC][4], av1[GC][4];
#pragma unroll
    for (int c = 0; c < GC; ++c) {
      const int m = min(m0 + c * 256, d - 256);
      if (m0 > 0) xv[c].load(xr + m);
      load4(a0 + m, av0[c]);
      if (has1) load4(a1 + m, av1[c]);
    }
#pragma unroll
    for (int c = 0; c < GC; ++c) {
      if (m0 + c * 256 < d) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float xe = xv[c].at(r);
          ss = __builtin_fmaf(xe, xe, ss);
          q0 = __builtin_fmaf(xe, av0[c][r], q0);
          if (has1) q1 = __builtin_fmaf(xe, av1[c][r], q1);
        }
      }
    }
  }
  ss = wave_tree_sum(ss);
  q0 = wave_tree_sum(q0);
  if (has1) q1 = wave_tree_sum(q1);
  if (lane == k0 || (has1 && lane == k1))
    cost[(size_t)t * K + lane] = pair_cost(lane == k0 ? q0 : q1, ss, b_my, my_w);
}

template <typename XT>
static void launch_scores_t(const XT *x, int B, int d, const float *Wr, const float *beta,
                            int n_router, const float *G, float *logits, float *gdot,
                            const float *A, float *q, float *ss, hipStream_t st) {
  if (A || scores_small_router(sizeof(XT) == 2, B, n_router, d)) {
    const int n_group = (B + TOK_GROUP - 1) / TOK_GROUP, rgs = (n_router + 3) / 4;
    const int n_other = n_group * ((A ? rgs : 0) + (A || G ? 1 : 0));
    int nb;   // workgroups per die
    if (n_group > N_XCD / 2) {
      nb = (n_group + N_XCD - 1) / N_XCD * (rgs + n_other / n_group);
    } else {
      const int dies = N_XCD - n_group, no = (n_other + dies - 1) / dies;
      nb = rgs > no ? rgs : no;
    }
    launch_k(k_scores_small<XT>, dim3(N_XCD * nb), dim3(4 * WAVE), 0, st, x, B,
             d, Wr, beta, n_router, A, G, n_group, n_other, logits, q, ss, gdot);
    return;
  }
  const int rows = n_router + (G ? 1 : 0);
  const dim3 grid(xcd_grid((B + SC_TB - 1) / SC_TB, (rows + SC_RB - 1) / SC_RB));
  launch_k(k_scores<XT>, grid, dim3(SC_WAVES * WAVE), 0, st, x, B, d, Wr, beta, n_router, G,
           logits, gdot);
}

hipError_t launch_scores(bool bf16, const void *x, int B, int d, const float *Wr,
                         const float *beta, int n_router, const float *G, float *logits,
                         float *gdot, hipStream_t st, const float *A, float *q, float *ss) {
  if (bf16)
    launch_scores_t((const uint16_t *)x, B, d, Wr, beta, n_router, G, logits, gdot, A, q, ss, st);
  else
    launch_scores_t((const float *)x, B, d, Wr, beta, n_router, G, logits, gdot, A, q, ss, st);
  return hipGetLastError();
}

hipError_t launch_tail(bool bf16, int B, int E, int K, int d, int norm_topk,
                       const float *logits, const void *x, const float *A, const float *bp,
                       int32_t *ids, float *w, float *cost, int mode, int rule,
                       hipStream_t st, uint8_t *order, float *ex, float *den, const float *q,
                       const float *ss) {
  const dim3 block(tail_waves(K, (mode & 2) && rule == SCORE_BASE && !q) * WAVE);
  const dim3 grid(xcd_grid((B + TOK_GROUP - 1) / TOK_GROUP, TOK_GROUP));
#define BASE_TL(XT, D)                                                                          \
  launch_k(k_tail<XT, D>, grid, block, 0, st, B, E, K, d, norm_topk, logits, (const XT *)x, A, \
           bp, ids, w, cost, mode, rule, order, ex, den, q, ss)
  if (bf16) {
    if (q) BASE_TL(uint16_t, true);
    else BASE_TL(uint16_t, false);
  } else {
    if (q) BASE_TL(float, true);
    else BASE_TL(float, false);
  }
#undef BASE_TL
  return hipGetLastError();
}

}  // namespace basek
