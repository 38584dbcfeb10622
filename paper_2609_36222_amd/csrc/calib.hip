// Streaming calibration statistics of the log-energy predictor (Sec. 3.4;
// App. A "Calibration Details"): for every routed pair (t, u) of a batch of
// calibration tokens, the target y = log(||E_u(z_t)||^2 + eps) and the
// input z_bar = z_t / ||z_t||, accumulated per expert into
//   n, sum y, sum y^2 (fp64), sum z_bar and sum z_bar y (fp64 vectors) and
//   the Gram matrix sum z_bar z_bar^T (fp32, as App. A keeps it).
// The expert outputs come from the layer's own FFN run with every routed
// expert kept and unit gates, so one batch costs one dense routed MoE pass.
//
// k_calib_norm     inv[t] = 1 / ||x_t|| (0 for x = 0), fp64, and the rows the
//                  Gram reads (plus a zero row): fp32 layers z_bar_t =
//                  fp32(x_t inv[t]), bf16 layers x_t times a power of two
// k_calib_pairs    y[p] = log(sum_c out_p[c]^2 + eps), fp64, one wavefront per pair
// k_calib_moments  per (kept slot, 128 columns): the fp64 sums, the pairs
//                  dealt to eight wavefronts
// k_calib_gram, k_calib_gram_bf16
//                  per (kept slot, 128 x 128 block of the upper triangle):
//                  G += sum_p z_i z_j on the matrix cores (fp32 sums over the
//                  slot's pairs, then one add), mirrored
// Every statistic has a single writer and a fixed summation order: the
// results are deterministic.
#include "common.hpp"
#include "internal.hpp"

namespace basek {

constexpr int CAL_THREADS = 256;
constexpr double CAL_EPS = 1e-12;

// A 16-byte load and store of the statistics; STREAM: past the caches' usual
// replacement (non-temporal).
template <bool STREAM>
__device__ __forceinline__ f32x4 load_g(const float *p) {
  if constexpr (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
  return *reinterpret_cast<const f32x4 *>(p);
}
template <bool STREAM>
__device__ __forceinline__ void store_g(float *p, f32x4 v) {
  if constexpr (STREAM)
    __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(p));
  else
    *reinterpret_cast<f32x4 *>(p) = v;
}
// Gram matrices larger than the 256 MB Infinity Cache are gone from it before
// the next batch reads them, and as they pass they push out the token rows:
// non-temporal then (OLMoE-shaped, 1.07 GB, two batches from zero 1610 -> 1517
// us; d = 1280, E = 48, 315 MB, one batch 247 -> 240).  Smaller ones are found
// there again (d = 1024, E = 32, 134 MB, two batches: 279 us, 292
// non-temporal).
constexpr size_t G_STREAM_BYTES = (size_t)256 << 20;

// Elements c, c + 1 of an activation row.
__device__ __forceinline__ double2 act2(const void *row, bool bf16, int c) {
  if (bf16) {
    const uint32_t v = *reinterpret_cast<const uint32_t *>((const uint16_t *)row + c);
    return {(double)__uint_as_float(v << 16), (double)__uint_as_float(v & 0xFFFF0000u)};
  }
  const float2 v = *reinterpret_cast<const float2 *>((const float *)row + c);
  return {(double)v.x, (double)v.y};
}

// Elements c .. c + 7 (exact widening).
__device__ __forceinline__ void load8(const void *row, bool bf16, int c, float (&v)[8]) {
  if (bf16) {
    const u32x4 r = *reinterpret_cast<const u32x4 *>((const uint16_t *)row + c);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(r[i] << 16);
      v[2 * i + 1] = __uint_as_float(r[i] & 0xFFFF0000u);
    }
  } else {
    float a[4], b[4];
    load4((const float *)row + c, a);
    load4((const float *)row + c + 4, b);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = a[i];
      v[4 + i] = b[i];
    }
  }
}

// Fixed-order fp64 sum over the wavefront (every lane gets it).
__device__ __forceinline__ double wave_sum64(double v) {
#pragma unroll
  for (int h = WAVE / 2; h >= 1; h >>= 1) v = v + __shfl_xor(v, h, WAVE);
  return v;
}

// What the Gram reads.  fp32 layers: rows z_bar_t = fp32(x_t inv[t]); bf16
// layers: bf16 rows xs_t = x_t 2^k (exact) with 1 <= ||xs_t|| < 2, and sc[t] =
// fp32(1 / ||xs_t||^2), so that z_i z_j = xs_i (xs_j sc) whatever the scale of
// x.  d elements a row, B + 1 rows; row B (and sc[B]) are zero.
struct GramRows {
  float *z;
  uint16_t *xs;
  float *sc;
};

// One wavefront per token (and one for the zero row).
__global__ __launch_bounds__(CAL_THREADS)
void k_calib_norm(const void *__restrict__ x, int bf16, int B, int d, double *__restrict__ inv,
                  GramRows gr) {
  const int t = blockIdx.x * (CAL_THREADS / WAVE) + threadIdx.x / WAVE, lane = lane_id();
  if (t > B) return;
  if (t == B) {
    const int words = bf16 ? d / 2 : d;
    uint32_t *z = (bf16 ? (uint32_t *)gr.xs : (uint32_t *)gr.z) + (size_t)B * words;
    for (int c = lane; c < words; c += WAVE) z[c] = 0u;
    if (bf16 && lane == 0) gr.sc[B] = 0.0f;
    return;
  }
  const size_t at = (size_t)t * d;
  const void *row = bf16 ? (const void *)((const uint16_t *)x + at) : (const void *)((const float *)x + at);
  // eight elements per lane and piece
  double s = 0.0;
#pragma unroll 4
  for (int c = 8 * lane; c < d; c += 8 * WAVE) {
    float v[8];
    load8(row, bf16, c, v);
#pragma unroll
    for (int i = 0; i < 8; ++i) s = fma((double)v[i], (double)v[i], s);
  }
  s = wave_sum64(s);
  const double iv = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
  if (lane == 0) inv[t] = iv;
  if (bf16) {
    int e = 0;
    if (s > 0.0) (void)frexp(sqrt(s), &e);   // ||x|| = m 2^e, 1/2 <= m < 1
    const int k = 1 - e;
    const double is = ldexp(iv, -k);
    if (lane == 0) gr.sc[t] = (float)(is * is);   // 1 / ||xs||^2 (0 for x = 0)
#pragma unroll 4
    for (int c = 8 * lane; c < d; c += 8 * WAVE) {
      float v[8];
      load8(row, true, c, v);
      u32x4 o;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        o[i] = (__float_as_uint(__builtin_ldexpf(v[2 * i], k)) >> 16) |
               (__float_as_uint(__builtin_ldexpf(v[2 * i + 1], k)) & 0xFFFF0000u);
      *reinterpret_cast<u32x4 *>(gr.xs + at + c) = o;
    }
  } else {
    for (int c = 8 * lane; c < d; c += 8 * WAVE) {
      float v[8];
      load8(row, false, c, v);
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = (float)((double)v[i] * iv);
      *reinterpret_cast<float4 *>(gr.z + at + c) = float4{v[0], v[1], v[2], v[3]};
      *reinterpret_cast<float4 *>(gr.z + at + c + 4) = float4{v[4], v[5], v[6], v[7]};
    }
  }
}

// pairs p < offsets[n_slots] (the routed pairs of the kept slots)
__global__ __launch_bounds__(CAL_THREADS)
void k_calib_pairs(const float *__restrict__ out, int d, const int32_t *__restrict__ offsets,
                   int n_slots, double *__restrict__ y) {
  const int p = blockIdx.x * (CAL_THREADS / WAVE) + threadIdx.x / WAVE, lane = lane_id();
  if (p >= offsets[n_slots]) return;
  const float *row = out + (size_t)p * d;
  double s = 0.0;
#pragma unroll 8
  for (int c = 4 * lane; c < d; c += 4 * WAVE) {
    const float4 v = *reinterpret_cast<const float4 *>(row + c);
    s = fma((double)v.x, (double)v.x, s);
    s = fma((double)v.y, (double)v.y, s);
    s = fma((double)v.z, (double)v.z, s);
    s = fma((double)v.w, (double)v.w, s);
  }
  s = wave_sum64(s);
  if (lane == 0) y[p] = log(s + CAL_EPS);
}

// One workgroup per (kept slot, 128 columns), two columns per lane.  The
// slot's pairs come in chunks whose token, 1 / ||x|| and target sit in LDS;
// wavefront w takes the pairs w, w + 8, ... of a chunk, eight token rows in
// flight, and the wavefronts' sums are added in order.  (One thread per
// column walking all pairs, each a chain of dependent loads, took 135 us per
// batch of 1024 OLMoE-shaped tokens, whose most popular expert sees nearly
// every token.)
constexpr int CM_WAVES = 8;
constexpr int CM_COLS = 2 * WAVE;
constexpr int CM_CHUNK = CM_WAVES * WAVE;
__global__ __launch_bounds__(CM_WAVES * WAVE)
void k_calib_moments(const void *__restrict__ x, int bf16, int d, const double *__restrict__ inv,
                     const int32_t *__restrict__ n_sel, const int32_t *__restrict__ sel_ids,
                     const int32_t *__restrict__ offsets, const int32_t *__restrict__ pair_tok,
                     const double *__restrict__ y, CalibStats st) {
  __shared__ int tok_s[CM_CHUNK];
  __shared__ double inv_s[CM_CHUNK], y_s[CM_CHUNK];
  __shared__ double2 red[2][CM_WAVES][WAVE];
  const int s = blockIdx.x;
  if (s >= *n_sel) return;
  const int u = sel_ids[s];
  const int p0 = offsets[s], p1 = offsets[s + 1];
  const int tid = threadIdx.x, w = tid / WAVE, lane = lane_id();
  const int j = blockIdx.y * CM_COLS + 2 * lane;
  double2 sz = {0.0, 0.0}, q = {0.0, 0.0};
  double sy = 0.0, syy = 0.0;   // (first column group) lane sums of this wavefront's targets
  for (int c0 = p0; c0 < p1; c0 += CM_CHUNK) {
    const int n = min(CM_CHUNK, p1 - c0);
    if (c0 > p0) __syncthreads();
    if (tid < n) {
      const int t = pair_tok[c0 + tid];
      tok_s[tid] = t;
      inv_s[tid] = inv[t];
      const double yv = y[c0 + tid];
      y_s[tid] = yv;
      sy = sy + yv;
      syy = fma(yv, yv, syy);
    }
    __syncthreads();
    constexpr int AHEAD = 8;
    for (int i0 = w; i0 < n; i0 += AHEAD * CM_WAVES) {
      double2 v[AHEAD];
#pragma unroll
      for (int a = 0; a < AHEAD; ++a) {
        const int i = min(i0 + a * CM_WAVES, n - 1);
        const size_t at = (size_t)tok_s[i] * d;
        v[a] = act2(bf16 ? (const void *)((const uint16_t *)x + at) : (const void *)((const float *)x + at),
                    bf16, j);
      }
#pragma unroll
      for (int a = 0; a < AHEAD; ++a) {
        const int i = i0 + a * CM_WAVES;
        if (i < n) {
          const double zx = v[a].x * inv_s[i], zy = v[a].y * inv_s[i];
          sz.x = sz.x + zx;
          sz.y = sz.y + zy;
          q.x = fma(zx, y_s[i], q.x);
          q.y = fma(zy, y_s[i], q.y);
        }
      }
    }
  }
  red[0][w][lane] = sz;
  red[1][w][lane] = q;
  __syncthreads();
  if (w < 2) {   // wavefront 0: sz, 1: q
    double2 r = red[w][0][lane];
    for (int i = 1; i < CM_WAVES; ++i) {
      r.x = r.x + red[w][i][lane].x;
      r.y = r.y + red[w][i][lane].y;
    }
    double *dst = (w == 0 ? st.sz : st.q) + (size_t)u * d + j;
    dst[0] += r.x;
    dst[1] += r.y;
  }
  if (blockIdx.y != 0) return;
  __syncthreads();
  sy = wave_sum64(sy);
  syy = wave_sum64(syy);
  if (lane == 0) red[0][w][0] = double2{sy, syy};
  __syncthreads();
  if (tid == 0) {
    double2 r = red[0][0][0];
    for (int i = 1; i < CM_WAVES; ++i) {
      r.x = r.x + red[0][i][0].x;
      r.y = r.y + red[0][i][0].y;
    }
    st.head[(size_t)u * 4 + 0] += (double)(p1 - p0);
    st.head[(size_t)u * 4 + 1] += r.x;
    st.head[(size_t)u * 4 + 2] += r.y;
  }
}

// fp32 layers: the Gram matrices on the matrix cores (v_mfma_f32_16x16x4_f32: fp32
// operands, products and sums).  A workgroup owns one 128 x 128 block (I, J),
// I <= J, of one kept slot's G_u, and each of its four wavefronts a 64 x 64
// quarter (rows rb.., columns cb..) as 4 x 4 instruction tiles.  Tile (a, b)
// takes rows rb + 4 i + a and columns cb + 4 j + b (i, j = 0..15), so that a
// lane's four A values (and four B values) are one 16-byte load: lane l
// supplies A[l % 16][l / 16] = z_p[rb + 4 (l % 16) + a] and B[l / 16][l % 16]
// = z_p[cb + 4 (l % 16) + b] with p = the step's first pair + l / 16, and
// holds C[4 (l / 16) + r][l % 16], r = 0..3, i.e. row rb + 16 (l / 16) + 4 r
// + a, column cb + 4 (l % 16) + b: for each (r, a) a 16-byte piece of a row.
// The contraction runs over the slot's pairs in order, four per step, in
// chunks of 64 pairs whose tokens the lanes hold (one each) and pass round
// by lane exchange; operands are requested three steps ahead; pairs past
// the slot's end read zbuf's zero row B.  The batch's sums start from zero
// and are added to G once.  Only blocks I <= J are computed: the new
// values of (I, J) are also written, transposed, to (J, I), so G_u stays
// exactly symmetric and the lower blocks are never read.  Workgroup b runs
// on die b mod 8 and the blocks of slot s go to die s mod 8, so that the
// slot's operand rows stay in one L2.  zbuf [B + 1][d] (fp32) holds the
// rows z_bar_t = fp32(x_t inv[t]) and a zero row (k_calib_norm).
constexpr int GM_TILE = 128;
constexpr int GM_WAVES = 4;
constexpr int GM_AHEAD = 3;   // steps of operands in flight (ring of 4)

__device__ __forceinline__ f32x4 mfma_f32_4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_bf16_32(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Rows cb + 4 m + b, columns rb + 16 kk + 4 r .. + 3 get v[r][0..3][b]: a
// quarter's mirror.  Stored as held, every lane of an instruction has a 64-byte
// segment of its own; so the lanes m % 4 first exchange pieces r, and four
// neighbours then store 64 contiguous bytes (two batches of 1024 OLMoE-shaped
// tokens from zero 1710 -> 1607 us).
template <int H>
__device__ __forceinline__ void swap_piece(f32x4 &lo, f32x4 &hi, bool odd) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float got = xor_lane<H>(odd ? lo[e] : hi[e]);
    lo[e] = odd ? got : lo[e];
    hi[e] = odd ? hi[e] : got;
  }
}
template <bool STREAM>
__device__ __forceinline__ void store_mirror(float *g, int d, int rb, int cb, int m, int kk,
                                             const f32x4 (&v)[4][4]) {
  const int q = m & 3;
  float *to = g + (size_t)(cb + 4 * (m - q)) * d + rb + 16 * kk + 4 * q;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    f32x4 t[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) t[r] = f32x4{v[r][0][b], v[r][1][b], v[r][2][b], v[r][3][b]};
    swap_piece<1>(t[0], t[1], q & 1);
    swap_piece<1>(t[2], t[3], q & 1);
    swap_piece<2>(t[0], t[2], q & 2);
    swap_piece<2>(t[1], t[3], q & 2);
    // t[i]: piece q of the row that lane m - q + i held
#pragma unroll
    for (int i = 0; i < 4; ++i) store_g<STREAM>(to + (size_t)(4 * i + b) * d, t[i]);
  }
}

__global__ __launch_bounds__(GM_WAVES * WAVE, 2)
void k_calib_gram(const float *__restrict__ zbuf, int B, int d, int n_blk, int slots_per_die,
                  const int32_t *__restrict__ n_sel, const int32_t *__restrict__ sel_ids,
                  const int32_t *__restrict__ offsets, const int32_t *__restrict__ pair_tok,
                  float *__restrict__ G) {
  const int x = blockIdx.x % N_XCD, i = blockIdx.x / N_XCD;
  const int s = x + N_XCD * (i / n_blk);
  int k = i % n_blk;
  if (i / n_blk >= slots_per_die || s >= *n_sel) return;
  const int p0 = offsets[s], p1 = offsets[s + 1];
  if (p1 <= p0) return;
  // block k of the upper triangle, row by row
  const int T = d / GM_TILE;
  int I = 0;
  while (k >= T - I) { k -= T - I; ++I; }
  const int J = I + k;
  const int lane = threadIdx.x % WAVE, w = threadIdx.x / WAVE;
  const int m = lane & 15, kk = lane >> 4;
  const int rb = I * GM_TILE + (w >> 1) * 64, cb = J * GM_TILE + (w & 1) * 64;
  float *g = G + (size_t)sel_ids[s] * d * d;

  auto toks = [&](int pc) { return pc + lane < p1 ? pair_tok[pc + lane] : B; };
  f32x4 ra[GM_AHEAD + 1], rbv[GM_AHEAD + 1];
  auto load = [&](int slot, int t) {
    const float *zr = zbuf + (size_t)t * d;
    ra[slot] = *(const f32x4 *)(zr + rb + 4 * m);
    rbv[slot] = *(const f32x4 *)(zr + cb + 4 * m);
  };
  int tcur = toks(p0), tnext = toks(p0 + WAVE);
#pragma unroll
  for (int q = 0; q < GM_AHEAD; ++q) load(q, __shfl(tcur, 4 * q + kk));
  // the block's old values (rows rb + 16 kk + 4 r + a, 16 bytes at cb + 4 m)
  f32x4 old[4][4];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int a = 0; a < 4; ++a)
      old[r][a] = *(const f32x4 *)(g + (size_t)(rb + 16 * kk + 4 * r + a) * d + cb + 4 * m);

  f32x4 acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int pc = p0; pc < p1; pc += WAVE) {
#pragma unroll
    for (int st = 0; st < WAVE / 4; ++st) {
      if (pc + 4 * st >= p1) break;
      const int ahead = st + GM_AHEAD;
      load(ahead % (GM_AHEAD + 1),
           ahead < WAVE / 4 ? __shfl(tcur, 4 * ahead + kk) : __shfl(tnext, 4 * (ahead - WAVE / 4) + kk));
      const f32x4 za = ra[st % (GM_AHEAD + 1)], zb = rbv[st % (GM_AHEAD + 1)];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = mfma_f32_4(za[a], zb[b], acc[a][b]);
    }
    tcur = tnext;
    tnext = toks(pc + 2 * WAVE);
  }

#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 v = old[r][a] + f32x4{acc[a][0][r], acc[a][1][r], acc[a][2][r], acc[a][3][r]};
      *(f32x4 *)(g + (size_t)(rb + 16 * kk + 4 * r + a) * d + cb + 4 * m) = v;
      old[r][a] = v;
    }
  if (I != J) store_mirror<false>(g, d, rb, cb, m, kk, old);
}

// bf16 layers: the same blocks, quarters and tiles, on the bf16 matrix
// instruction: z_i z_j = xs_i v_j (GramRows), v_j = fp32(xs_j sc) cut without
// loss into three bf16 values (8 significant bits each, by truncation), so
// that three v_mfma_f32_16x16x32_bf16 (exact products, fp32 sums) replace
// eight fp32 ones of a sixteenth of their rate.
// A step is 32 pairs: lane l loads, for the pairs 8 (l / 16) .. + 7, the
// columns 4 (l % 16) .. + 3 of each side (8 bytes of a token row), and turns
// the 8 x 4 values into one operand fragment (8 pairs of one column) per
// column with byte permutes; v is formed and cut in registers (three stored
// planes of v instead: 643 against 451 us, the row reads then bound it).
// G's old values are read after the contraction: held across it (as in the fp32
// kernel) they spill, 473 against 420 us per batch of 1024 OLMoE-shaped tokens
// (before the mirror's 64-byte stores and non-temporal access; without the
// contraction 313 then).  The fp32 kernel took 548; now 365 (1.6 GB of G moved,
// 4.4 TB/s), traced on a box whose other kernels ran up to a tenth longer.
// The two sides are not alike, so inside a diagonal 64 x 64 quarter the
// elements above the diagonal are kept and mirrored, and the quarter below
// the diagonal of a diagonal block is the mirror of the one above: G_u stays
// exactly symmetric.
__device__ __forceinline__ bf16x8 halves8(const u32x2 (&r)[8], int c) {
  u32x4 f;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    f[q] = __builtin_amdgcn_perm(r[2 * q + 1][c >> 1], r[2 * q][c >> 1],
                                 (c & 1) ? 0x07060302u : 0x05040100u);
  return __builtin_bit_cast(bf16x8, f);
}

template <bool STREAM>
__global__ __launch_bounds__(GM_WAVES * WAVE, 2)
void k_calib_gram_bf16(GramRows gr, int B, int d, int n_blk, int slots_per_die,
                       const int32_t *__restrict__ n_sel, const int32_t *__restrict__ sel_ids,
                       const int32_t *__restrict__ offsets, const int32_t *__restrict__ pair_tok,
                       float *__restrict__ G) {
  const int x = blockIdx.x % N_XCD, i = blockIdx.x / N_XCD;
  const int s = x + N_XCD * (i / n_blk);
  int k = i % n_blk;
  if (i / n_blk >= slots_per_die || s >= *n_sel) return;
  const int p0 = offsets[s], p1 = offsets[s + 1];
  if (p1 <= p0) return;
  const int T = d / GM_TILE;
  int I = 0;
  while (k >= T - I) { k -= T - I; ++I; }
  const int J = I + k;
  const int lane = threadIdx.x % WAVE, w = threadIdx.x / WAVE;
  const int m = lane & 15, kk = lane >> 4;
  const int rb = I * GM_TILE + (w >> 1) * 64, cb = J * GM_TILE + (w & 1) * 64;
  if (rb > cb) return;   // below the diagonal: the mirror of quarter 1
  float *g = G + (size_t)sel_ids[s] * d * d;

  // the tokens and scales of 64 pairs, one per lane (past the end: the zero row)
  auto toks = [&](int pc) { return pc + lane < p1 ? pair_tok[pc + lane] : B; };
  int tc = toks(p0), tn = toks(p0 + WAVE);
  float scl = gr.sc[tc];
  u32x2 ra[8], rv[8];
  auto load = [&](int tv, int half) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint16_t *row = gr.xs + (uint32_t)__shfl(tv, 32 * half + 8 * kk + e) * (uint32_t)d;
      ra[e] = *reinterpret_cast<const u32x2 *>(row + rb + 4 * m);
      rv[e] = *reinterpret_cast<const u32x2 *>(row + cb + 4 * m);
    }
  };
  load(tc, 0);
  f32x4 acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int pc = p0; pc < p1; pc += WAVE) {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (half == 1 && pc + 32 >= p1) break;
      float se[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) se[e] = __shfl(scl, 32 * half + 8 * kk + e);
      bf16x8 fa[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) fa[a] = halves8(ra, a);
      u32x2 cv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) cv[e] = rv[e];
      // the next step's rows (past the last pair: the zero row)
      if (half == 0) load(tc, 1);
      else load(tn, 0);
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        u32x4 fh, fm, fl;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float v[2], r1[2], r2[2];
#pragma unroll
          for (int z = 0; z < 2; ++z) {
            const uint32_t wd = cv[2 * q + z][b >> 1];
            v[z] = __uint_as_float((b & 1) ? (wd & 0xFFFF0000u) : (wd << 16)) * se[2 * q + z];
            r1[z] = v[z] - __uint_as_float(__float_as_uint(v[z]) & 0xFFFF0000u);
            r2[z] = r1[z] - __uint_as_float(__float_as_uint(r1[z]) & 0xFFFF0000u);
          }
          fh[q] = __builtin_amdgcn_perm(__float_as_uint(v[1]), __float_as_uint(v[0]), 0x07060302u);
          fm[q] = __builtin_amdgcn_perm(__float_as_uint(r1[1]), __float_as_uint(r1[0]), 0x07060302u);
          fl[q] = __builtin_amdgcn_perm(__float_as_uint(r2[1]), __float_as_uint(r2[0]), 0x07060302u);
        }
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          acc[a][b] = mfma_bf16_32(fa[a], __builtin_bit_cast(bf16x8, fl), acc[a][b]);
          acc[a][b] = mfma_bf16_32(fa[a], __builtin_bit_cast(bf16x8, fm), acc[a][b]);
          acc[a][b] = mfma_bf16_32(fa[a], __builtin_bit_cast(bf16x8, fh), acc[a][b]);
        }
      }
    }
    tc = tn;
    scl = gr.sc[tc];
    tn = toks(pc + 2 * WAVE);
  }

  // the block's old values (rows rb + 16 kk + 4 r + a, 16 bytes at cb + 4 m)
  f32x4 old[4][4];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int a = 0; a < 4; ++a)
      old[r][a] = load_g<STREAM>(g + (size_t)(rb + 16 * kk + 4 * r + a) * d + cb + 4 * m);

  if (rb == cb) {
    // a diagonal quarter: i <= j, mirrored
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int ii = 16 * kk + 4 * r + a, jj = 4 * m + b;
          if (ii > jj) continue;
          const float v = old[r][a][b] + acc[a][b][r];
          g[(size_t)(rb + ii) * d + cb + jj] = v;
          if (ii < jj) g[(size_t)(cb + jj) * d + rb + ii] = v;
        }
    return;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 v = old[r][a] + f32x4{acc[a][0][r], acc[a][1][r], acc[a][2][r], acc[a][3][r]};
      store_g<STREAM>(g + (size_t)(rb + 16 * kk + 4 * r + a) * d + cb + 4 * m, v);
      old[r][a] = v;
    }
  store_mirror<STREAM>(g, d, rb, cb, m, kk, old);
}

__global__ __launch_bounds__(CAL_THREADS)
void k_fill_zero(uint32_t *__restrict__ p, size_t n) {
  for (size_t i = blockIdx.x * (size_t)CAL_THREADS + threadIdx.x; i < n;
       i += (size_t)gridDim.x * CAL_THREADS)
    p[i] = 0u;
}

hipError_t launch_calib_zero(void *stats, size_t bytes, hipStream_t st) {
  const size_t n = bytes / 4;
  const size_t nb = (n + CAL_THREADS - 1) / CAL_THREADS;
  const unsigned blocks = (unsigned)(nb < 65536 ? nb : 65536);
  launch_k(k_fill_zero, dim3(blocks), dim3(CAL_THREADS), 0, st, (uint32_t *)stats, n);
  return hipGetLastError();
}

hipError_t launch_calib_stats(const void *x, bool bf16, int B, int d, int E, int K,
                              const float *pairbuf, const int32_t *n_sel,
                              const int32_t *sel_ids, const int32_t *offsets,
                              const int32_t *pair_tok, double *inv, double *y, float *zbuf,
                              CalibStats st, hipStream_t s) {
  constexpr int per = CAL_THREADS / WAVE;
  launch_k(k_calib_pairs, dim3((B * K + per - 1) / per), dim3(CAL_THREADS), 0, s,
           pairbuf, d, offsets, E, y);
  GramRows gr;
  gr.z = zbuf;
  gr.xs = reinterpret_cast<uint16_t *>(zbuf);
  gr.sc = reinterpret_cast<float *>(gr.xs + (size_t)(B + 1) * d);
  launch_k(k_calib_norm, dim3((B + per) / per), dim3(CAL_THREADS), 0, s, x, (int)bf16, B, d, inv,
           gr);
  launch_k(k_calib_moments, dim3(E, d / CM_COLS), dim3(CM_WAVES * WAVE), 0,
           s, x, (int)bf16, d, (const double *)inv, n_sel, sel_ids, offsets, pair_tok,
           (const double *)y, st);
  const int T = d / GM_TILE, n_blk = T * (T + 1) / 2;
  const int per_die = (E + N_XCD - 1) / N_XCD;
  const dim3 grid((unsigned)(N_XCD * per_die * n_blk));
  if (bf16)
    launch_k((size_t)E * d * d * 4 > G_STREAM_BYTES ? k_calib_gram_bf16<true> : k_calib_gram_bf16<false>,
             grid, dim3(GM_WAVES * WAVE), 0, s, gr, B, d, n_blk, per_die, n_sel, sel_ids, offsets,
             pair_tok, st.G);
  else
    launch_k(k_calib_gram, grid, dim3(GM_WAVES * WAVE), 0, s, (const float *)zbuf, B, d, n_blk,
             per_die, n_sel, sel_ids, offsets, pair_tok, st.G);
  return hipGetLastError();
}

}  // namespace basek
