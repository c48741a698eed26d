// Attention for launches that cover one in-block position t of every candidate (token-by-token generation).
// The MFMA kernel in its single-position mode stacks the n*g query rows of a (beam, kv head) against the prefix keys, which
// the n candidates share, and leaves partial results per run of key tiles (O un-normalised, running maximum m in the log2
// domain, weight sum l). Where the prefix leaves room on the chip its launch covers the candidates' own block keys 0..t as
// well, with one more partial result per row; this file merges, or merges and covers the block keys.
#include "common.h"

bool launch_attention_mfma_decode(const bf16_t* q, const bf16_t* kb, const bf16_t* vbT, const bf16_t* poolK,
                                  const bf16_t* poolV, const BatchGeom& g, const ModelDims& md, int Lp, const DecodeRuns& runs,
                                  float* part, size_t part_floats, bool with_block, const WeightsAhead& ahead, hipStream_t s);
bool decode_block_beside(const BatchGeom& g, const ModelDims& md, int Lp, const DecodeRuns& runs, size_t part_floats);

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

struct MergeArgs {
  const bf16_t* q;      // [C][Hq][HD]
  const bf16_t* kb;     // [C*Lk][Hkv][HD]
  const bf16_t* vbT;    // [C][Hkv][HD][Lp]
  const float* part_o;  // [beam*Hkv + kvh][split][n*g][HD]: the runs, then the block keys (not the long kernel)
  const float* part_m;
  const float* part_l;
  bf16_t* out;          // [C][Hq*HD]
  const int32_t* lens;
  int b0, len_override;
  int n, Hq, Hkv, Lk, Lp, t, run_tiles, n_splits, osum_off, rows_total, all_runs;
  float scale_log2e;
};

// One wavefront per (candidate, query head): HD / 4 lanes hold 16 bytes each of a partial output, 64 / (HD / 4) partial
// outputs at a time; lane s holds the statistics of run s, the lane after the runs those of the block keys. Bound by the latency of
// its loads, which are all requested at once; a single beam's do not even wait for its length, since it has all the runs
// unless its prefix has changed since the launch was captured.
template <int HD>
__global__ void __launch_bounds__(256) attention_decode_merge_kernel(MergeArgs a) {
  constexpr int LANES = HD / 4, GROUPS = 64 / LANES, NP = (DECODE_MAX_RUNS + 1 + GROUPS - 1) / GROUPS;
  static_assert(DECODE_MAX_RUNS < 64, "a lane per partial result");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + wave;                 // candidate * Hq + query head
  if (row >= a.rows_total) return;
  const int c = row / a.Hq, h = row - c * a.Hq;
  const int g = a.Hq / a.Hkv, kvh = h / g, j = h - kvh * g;
  const int b = c / a.n, i = c - b * a.n;
  const int P = a.len_override >= 0 ? a.len_override : a.lens[a.b0 + b];
  const size_t rows = (size_t)a.n * g;
  const size_t prow0 = ((size_t)b * a.Hkv + kvh) * (a.n_splits + 1) * rows + (size_t)i * g + j;   // + split*rows
  // runs of this beam: what others hold is whatever an earlier launch left there
  const int ns = min((((P + 63) >> 6) + a.run_tiles - 1) / a.run_tiles, a.n_splits);
  const int loaded = a.all_runs ? a.n_splits : ns;
  const int st = lane < loaded ? lane : a.n_splits;
  float m = a.part_m[prow0 + st * rows], l = a.part_l[prow0 + st * rows];
  const int grp = lane / LANES, col = lane % LANES;
  const float4* po = (const float4*)(a.part_o + prow0 * HD) + col;
  float4 v[NP];
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const int s = k * GROUPS + grp;
    if (k * GROUPS <= loaded) v[k] = po[(size_t)(s < loaded ? s : a.n_splits) * rows * LANES];
  }
  const bool valid = lane < ns || lane == loaded;
  m = valid ? m : -INFINITY;
  const float mx = wave_max(m);                          // finite: a position sees its own key
  const float w = __builtin_amdgcn_exp2f(m - mx);
  l = wave_sum(valid ? w * l : 0.f);
  float4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const int s = k * GROUPS + grp;
    if (k * GROUPS > loaded) break;
    const float ws = __shfl(w, s < 64 ? s : 63, 64);
    if (s < ns || s == loaded) {
      acc.x = fmaf(ws, v[k].x, acc.x);
      acc.y = fmaf(ws, v[k].y, acc.y);
      acc.z = fmaf(ws, v[k].z, acc.z);
      acc.w = fmaf(ws, v[k].w, acc.w);
    }
  }
#pragma unroll
  for (int o = LANES; o < 64; o <<= 1) {
    acc.x += __shfl_xor(acc.x, o, 64);
    acc.y += __shfl_xor(acc.y, o, 64);
    acc.z += __shfl_xor(acc.z, o, 64);
    acc.w += __shfl_xor(acc.w, o, 64);
  }
  const float inv = 1.0f / l;
  if (grp == 0)
    *(bf16x4*)(a.out + (size_t)row * HD + 4 * col) =
        bf16x4{(__bf16)(acc.x * inv), (__bf16)(acc.y * inv), (__bf16)(acc.z * inv), (__bf16)(acc.w * inv)};
}

// The merge where the prefix fills the chip by itself: it covers the block keys too.
// One workgroup of four wavefronts per (candidate, kv head, 16 of its query heads): the g query heads share the block
// keys and values, which are therefore read once, in whole cache lines, and multiplied by MFMA (heads are the 16
// columns). The kernel is a chain of short dependent phases on a few KB, bound by latency, so whatever does not depend
// on computed values (statistics and the first partial outputs of the runs, values) is requested before the scores.
// (One wavefront per (candidate, query head), each lane with a key row of its own, touched 64 cache lines with every
// load: 25.9 us at 256 candidates x 12 heads with 8 runs each; this form 8.1 us with up to 19 runs. At 16 x 12 the two take
// the same, 9.3 - 9.5 us on average over the 128 positions of a block, but this one with the 32 runs that the prefix kernel
// wants, 8.7 us instead of 10.7 with 16.)
template <int HD>
__global__ void __launch_bounds__(256) attention_decode_merge_block_kernel(MergeArgs a) {
  constexpr int KS = HD / 32;                   // MFMA K-steps of the scores
  constexpr int ND = HD / 64;                   // 16-dim tiles of the output per wavefront
  constexpr int NPG = 4, NPS = DECODE_MAX_RUNS / 4;   // partial outputs requested up front: 64-lane groups of 16-byte
                                                // columns, runs per wavefront
  constexpr int NVP = 4;                        // 32-key value steps requested up front
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int Lq = (a.Lp + 31) & ~31;             // keys of the weights, whole MFMA K-steps
  const int PS = Lq + 8;                        // row stride of the bf16 weights: 16-byte reads of 16 rows spread over the banks
  const int HS = a.Hq / a.Hkv < 16 ? a.Hq / a.Hkv : 16;            // head rows of the arrays
  float* sc = (float*)smem;                     // [HS][SS] scores
  bf16_t* pw = (bf16_t*)(sc + HS * (Lq + 4));   // [HS][PS] weights
  float* wm = (float*)(pw + HS * PS);           // [HS][n_splits] maxima, then weights, of the runs
  float* wl = wm + HS * a.n_splits;             // [HS][n_splits] weight sums
  float* inv = wl + HS * a.n_splits;            // [HS]
  float* osum = (float*)(smem + a.osum_off);    // [4][HS][HD] the wavefronts' sums of partial outputs
  const int SS = Lq + 1;

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int col = lane & 15, quad = lane >> 4;
  const int c = blockIdx.x, kvh = blockIdx.y, j0 = blockIdx.z * 16;
  const int g = a.Hq / a.Hkv, gh = g - j0 < 16 ? g - j0 : 16;      // query heads of this workgroup
  const int b = c / a.n, i = c - b * a.n, t = a.t;
  const int P = a.len_override >= 0 ? a.len_override : a.lens[a.b0 + b];
  const int hc = col < gh ? col : gh - 1;       // columns beyond the heads repeat the last one and are not stored

  bf16x8 qf[KS];
  const bf16_t* qr = a.q + ((size_t)c * a.Hq + (size_t)kvh * g + j0 + hc) * HD + 8 * quad;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qf[ks] = *(const bf16x8*)(qr + 32 * ks);
  const int nkt = (t + 16) >> 4;                // 16-key tiles that hold a visible key
  const bf16_t* kbase = a.kb + ((size_t)c * a.Lk * a.Hkv + kvh) * HD + 8 * quad;
  bf16x8 kf[KS];
  auto load_keys = [&](int kt) {
    const int key = 16 * kt + col;
    const bf16_t* kr = kbase + (size_t)(key <= t ? key : t) * a.Hkv * HD;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kf[ks] = *(const bf16x8*)(kr + 32 * ks);
  };
  if (wave < nkt) load_keys(wave);
  const int nvs = (t + 32) >> 5;                // 32-key steps that hold a visible key
  const bf16_t* vbase = a.vbT + (((size_t)c * a.Hkv + kvh) * HD + 16 * wave + col) * a.Lp;
  // values of keys 32 st + 8 quad .. + 7; those beyond t are whatever an earlier call left there and become 0
  auto load_vals = [&](int u, int st) {
    const int key = 32 * st + 8 * quad;
    return *(const bf16x8*)(vbase + (size_t)64 * u * a.Lp + (key < a.Lp ? key : 0));
  };
  auto visible_vals = [&](bf16x8 v, int st) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = 32 * st + 8 * quad + e <= t ? v[e] : (__bf16)0.f;
    return v;
  };
  bf16x8 vv[ND][NVP];
#pragma unroll
  for (int u = 0; u < ND; ++u)
#pragma unroll
    for (int st = 0; st < NVP; ++st) vv[u][st] = load_vals(u, st < nvs ? st : 0);
  const int ns = min((((P + 63) >> 6) + a.run_tiles - 1) / a.run_tiles, a.n_splits);   // runs of this beam
  const size_t rows = (size_t)a.n * g;
  const size_t prow0 = ((size_t)b * a.Hkv + kvh) * a.n_splits * rows + (size_t)i * g + j0;   // + split*rows + head
  for (int e = tid; e < gh * ns; e += 256) {
    const int s = e / gh, h = e - s * gh;
    wm[h * a.n_splits + s] = a.part_m[prow0 + s * rows + h];
    wl[h * a.n_splits + s] = a.part_l[prow0 + s * rows + h];
  }
  // partial outputs: wavefront w takes the runs w, w + 4, .., its lanes 16-byte columns of the heads' rows
  const int ncol = gh * (HD / 4);
  float4 po[NPG][NPS];
  auto load_parts = [&](int g0) {
#pragma unroll
    for (int u = 0; u < NPG; ++u) {
      if ((g0 + u) * 64 >= ncol) break;
      const int idx = (g0 + u) * 64 + lane;
      const float4* pb = (const float4*)(a.part_o + prow0 * HD) + (idx < ncol ? idx : ncol - 1);
#pragma unroll
      for (int k = 0; k < NPS; ++k)
        if (wave + 4 * k < ns) po[u][k] = pb[(size_t)(wave + 4 * k) * rows * (HD / 4)];
    }
  };
  load_parts(0);
  // scores of the block keys: lane holds keys 16 kt + 4 quad + e of head col
  for (int kt = wave; kt < nkt; kt += 4) {
    floatx4 s4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) s4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks], qf[ks], s4, 0, 0, 0);
    if (kt + 4 < nkt) load_keys(kt + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (col < gh) sc[col * SS + 16 * kt + 4 * quad + e] = s4[e] * a.scale_log2e;
  }
  __syncthreads();
  // softmax statistics: 16 lanes per head, all heads at a time
  const int h = tid >> 4, sub = tid & 15;
  if (h < gh) {
    float mx = -INFINITY;
    for (int k = sub; k <= t; k += 16) mx = fmaxf(mx, sc[h * SS + k]);
    for (int s = sub; s < ns; s += 16) mx = fmaxf(mx, wm[h * a.n_splits + s]);
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 16));
    mx = ceilf(mx);                             // finite (key t itself is always visible); an integer, so that
                                                // the bf16 rounding of the weights does not depend on the reference
    float l = 0.f;
    for (int k = sub; k < Lq; k += 16) {
      const float p = k <= t ? __builtin_amdgcn_exp2f(sc[h * SS + k] - mx) : 0.f;
      l += p;
      pw[h * PS + k] = (bf16_t)p;               // the weight that multiplies V is a bf16 operand
    }
    for (int s = sub; s < ns; s += 16) {
      const float w = __builtin_amdgcn_exp2f(wm[h * a.n_splits + s] - mx);
      l += w * wl[h * a.n_splits + s];
      wm[h * a.n_splits + s] = w;
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) l += __shfl_xor(l, o, 16);
    if (sub == 0) inv[h] = 1.0f / l;
  }
  __syncthreads();
  for (int g0 = 0; g0 * 64 < ncol; g0 += NPG) {
    if (g0) load_parts(g0);
#pragma unroll
    for (int u = 0; u < NPG; ++u) {
      const int idx = (g0 + u) * 64 + lane;
      if (idx >= ncol) break;
      const float* wr = wm + idx / (HD / 4) * a.n_splits + wave;
      float4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < NPS; ++k)
        if (wave + 4 * k < ns) {
          const float w = wr[4 * k];
          o.x = fmaf(w, po[u][k].x, o.x);
          o.y = fmaf(w, po[u][k].y, o.y);
          o.z = fmaf(w, po[u][k].z, o.z);
          o.w = fmaf(w, po[u][k].w, o.w);
        }
      ((float4*)osum)[wave * HS * (HD / 4) + idx] = o;
    }
  }
  __syncthreads();
  const float winv = inv[hc];
#pragma unroll
  for (int u = 0; u < ND; ++u) {
    // this lane's output dims: 16 (wave + 4 u) + 4 quad .. + 3 of head col
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float4 o = *(const float4*)(osum + ((size_t)w * HS + hc) * HD + 16 * wave + 64 * u + 4 * quad);
      acc[0] += o.x; acc[1] += o.y; acc[2] += o.z; acc[3] += o.w;
    }
    const bf16_t* pr = pw + hc * PS + 8 * quad;
#pragma unroll
    for (int st = 0; st < NVP; ++st)
      if (st < nvs) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(visible_vals(vv[u][st], st), *(const bf16x8*)(pr + 32 * st), acc, 0, 0, 0);
    for (int st = NVP; st < nvs; ++st)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(visible_vals(load_vals(u, st), st), *(const bf16x8*)(pr + 32 * st), acc, 0, 0, 0);
    if (col < gh) {
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (__bf16)(acc[e] * winv);
      *(bf16x4*)(a.out + ((size_t)c * a.Hq + (size_t)kvh * g + j0 + col) * HD + 16 * wave + 64 * u + 4 * quad) = o;
    }
  }
}

// The same for blocks whose scores do not fit the LDS above: one wavefront per (candidate, query head).
template <int HD>
__global__ void __launch_bounds__(64) attention_decode_merge_long_kernel(MergeArgs a) {
  extern __shared__ float sm[];                 // [HD] query, [Lp] block scores then weights, [n_splits] run weights
  float* qs = sm;
  float* sc = sm + HD;
  float* wrun = sc + a.Lp;
  const int c = blockIdx.x, h = blockIdx.y, lane = threadIdx.x, t = a.t;
  const int g = a.Hq / a.Hkv, kvh = h / g, j = h - kvh * g;
  const int b = c / a.n, i = c - b * a.n;
  const int P = a.len_override >= 0 ? a.len_override : a.lens[a.b0 + b];
  const int ns = min((((P + 63) >> 6) + a.run_tiles - 1) / a.run_tiles, a.n_splits);
  const size_t rows = (size_t)a.n * g;
  const size_t prow0 = ((size_t)b * a.Hkv + kvh) * a.n_splits * rows + (size_t)i * g + j;   // + split*rows

  const bf16_t* qr = a.q + ((size_t)c * a.Hq + h) * HD;
  for (int d = lane; d < HD; d += 64) qs[d] = (float)qr[d];
  __syncthreads();
  float mx = -INFINITY;
  for (int jk = lane; jk <= t; jk += 64) {
    const bf16_t* kr = a.kb + (((size_t)c * a.Lk + jk) * a.Hkv + kvh) * HD;
    float dot = 0.f;
#pragma unroll
    for (int i8 = 0; i8 < HD / 8; ++i8) {
      const bf16x8 kv = *(const bf16x8*)(kr + 8 * i8);
#pragma unroll
      for (int e = 0; e < 8; ++e) dot = fmaf(qs[8 * i8 + e], (float)kv[e], dot);
    }
    dot *= a.scale_log2e;
    sc[jk] = dot;
    mx = fmaxf(mx, dot);
  }
  for (int s = lane; s < ns; s += 64) mx = fmaxf(mx, a.part_m[prow0 + s * rows]);
  mx = ceilf(wave_max(mx));
  float l = 0.f;
  for (int jk = lane; jk <= t; jk += 64) {
    const float p = __builtin_amdgcn_exp2f(sc[jk] - mx);
    l += p;
    sc[jk] = (float)(bf16_t)p;
  }
  for (int s = lane; s < ns; s += 64) {
    const float w = __builtin_amdgcn_exp2f(a.part_m[prow0 + s * rows] - mx);
    wrun[s] = w;
    l += w * a.part_l[prow0 + s * rows];
  }
  l = wave_sum(l);
  __syncthreads();
  const float inv = 1.0f / l;
  for (int d = lane; d < HD; d += 64) {
    float acc = 0.f;
    for (int s = 0; s < ns; ++s) acc = fmaf(wrun[s], a.part_o[(prow0 + s * rows) * HD + d], acc);
    const bf16_t* vr = a.vbT + (((size_t)c * a.Hkv + kvh) * HD + d) * a.Lp;
    for (int k0 = 0; k0 <= t; k0 += 8) {
      const bf16x8 vv = *(const bf16x8*)(vr + k0);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc = fmaf(k0 + e <= t ? sc[k0 + e] : 0.f, k0 + e <= t ? (float)vv[e] : 0.f, acc);
    }
    a.out[((size_t)c * a.Hq + h) * HD + d] = (bf16_t)(acc * inv);
  }
}

// LDS of the merge that covers the block keys: scores, weights and statistics (*osum_off bytes), then the wavefronts' sums.
static size_t merge_block_lds(const ModelDims& md, int Lp, int n_splits, size_t* osum_off) {
  const int gq = md.Hq / md.Hkv, HS = gq < 16 ? gq : 16, Lq = (Lp + 31) & ~31;
  *osum_off = ((size_t)HS * (4 * (Lq + 4) + 2 * (Lq + 8) + 8 * n_splits + 4) + 15) & ~(size_t)15;
  return *osum_off + 4 * (size_t)HS * md.hd * 4;
}
// Which kernels cover the block keys: workgroups beside the prefix's (0), the merge (1), or the merge of one wavefront per
// row (2), where the block's scores exceed its LDS: 6 Lq + 8 n_splits + 16 hd + 36 bytes per head row, so with 16 rows of
// 128 and 32 runs (1) takes blocks of up to 288 tokens.
int decode_block_kernel(const BatchGeom& g, const ModelDims& md, int Lp, const DecodeRuns& runs, size_t part_floats) {
  size_t osum_off;
  if (decode_block_beside(g, md, Lp, runs, part_floats)) return 0;
  return merge_block_lds(md, Lp, runs.count, &osum_off) <= 64 * 1024 ? 1 : 2;
}

// Returns false when the shape is not taken (the caller then uses the plain kernel).
bool launch_attention_decode(const bf16_t* q, const bf16_t* kb, const bf16_t* vbT, const bf16_t* poolK,
                             const bf16_t* poolV, bf16_t* out, const BatchGeom& g, const ModelDims& md, int Lp,
                             const DecodeRuns& runs, float* part, size_t part_floats, const WeightsAhead& ahead, hipStream_t s) {
  const int kernel = decode_block_kernel(g, md, Lp, runs, part_floats);
  const bool with_block = kernel == 0;
  if (!launch_attention_mfma_decode(q, kb, vbT, poolK, poolV, g, md, Lp, runs, part, part_floats, with_block, ahead, s)) return false;
  const int n_splits = runs.count;
  const size_t rows_all = (size_t)g.B * md.Hkv * (n_splits + (with_block ? 1 : 0)) * g.n * (md.Hq / md.Hkv);
  MergeArgs a;
  a.q = q; a.kb = kb; a.vbT = vbT; a.out = out;
  a.part_o = part; a.part_m = part + rows_all * md.hd; a.part_l = a.part_m + rows_all;
  a.lens = g.lens; a.b0 = g.b0; a.len_override = g.len_override;
  a.n = g.n; a.Hq = md.Hq; a.Hkv = md.Hkv; a.Lk = g.Lk; a.Lp = Lp; a.t = g.t0; a.run_tiles = runs.tiles;
  a.n_splits = n_splits;
  a.rows_total = g.B * g.n * md.Hq;
  a.all_runs = g.B == 1;
  a.scale_log2e = 1.4426950408889634f / sqrtf((float)md.hd);
  if (with_block) {
    const dim3 grid((a.rows_total + 3) / 4);
    if (md.hd == 128) attention_decode_merge_kernel<128><<<grid, 256, 0, s>>>(a);
    else attention_decode_merge_kernel<64><<<grid, 256, 0, s>>>(a);
    return true;
  }
  size_t osum_off;
  const size_t lds = merge_block_lds(md, Lp, n_splits, &osum_off);
  a.osum_off = (int)osum_off;
  if (kernel == 1) {
    const dim3 grid(g.B * g.n, md.Hkv, (md.Hq / md.Hkv + 15) / 16);
    if (md.hd == 128) attention_decode_merge_block_kernel<128><<<grid, 256, lds, s>>>(a);
    else attention_decode_merge_block_kernel<64><<<grid, 256, lds, s>>>(a);
  } else {
    const dim3 grid(g.B * g.n, md.Hq);
    const size_t lds_long = (size_t)(md.hd + Lp + n_splits) * sizeof(float);
    if (md.hd == 128) attention_decode_merge_long_kernel<128><<<grid, 64, lds_long, s>>>(a);
    else attention_decode_merge_long_kernel<64><<<grid, 64, lds_long, s>>>(a);
  }
  return true;
}
