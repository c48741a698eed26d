// Shared-prefix paged attention on MFMA (bf16, head_dim 64 or 128, 16-token pages).
//
// Work decomposition. For one beam b, candidate i and kv head, the g = Hq/Hkv query heads of the
// L block tokens are stacked into L*g rows (row r = t*g + j: token t, query head kvh*g + j) that
// all read the same keys. A workgroup (4 wavefronts) owns 32*QT*4 of those rows, or 16*4 (Rows16), and walks over
// the keys in tiles of 64: first the beam's cached prefix (4 pages per tile), then the
// candidate's own block (causal). The n candidates of a beam run as neighbouring workgroups on the
// same XCD, so the prefix pages are fetched from HBM once and re-read from L2.
//
// Per tile (flash-attention recurrence, float state):
//   S^T[key, q] = K Q^T   (MFMA 32x32x16, A = keys from LDS, B = queries held in registers)
//   m' = max(m, max_key S), alpha = exp(m - m'), p = exp(S - m'), l = l*alpha + sum p
//   O^T[d, q] = O^T*alpha + V^T P^T   (A = V^T from LDS, B = p rounded to bf16)
// In the transposed orientation a lane owns one query column, so the max over keys is a reduction
// over the lane's own 32 accumulator values plus one exchange with the other half-wave, and the
// rescale by alpha is a per-lane scalar.
//
// The A-rows of the S^T product are fed with keys in the order pi(i) (the two middle groups of
// four swapped inside every 16) so that the eight accumulator values a lane holds for one MFMA
// K-step of the second product are eight CONSECUTIVE keys: with V stored transposed
// ([head_dim][16 tokens] per page) the matching A-operand is one 16-byte LDS read. In LDS the two 16-byte
// halves of a V^T row are swapped for rows with bit 3 set, so that 16 consecutive lanes (rows 32 bytes apart,
// same half) cover all 64 banks instead of every other 16-byte column.
#include "common.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

#define LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))
#define GLB_PTR(p) ((const __attribute__((address_space(1))) void*)(p))
// Tables that no kernel writes while this one runs, read by scalar loads. (Left to itself the compiler takes vector loads where it
// cannot rule out that the stores and loads to LDS before them change the table, and then waits for all of these.)
typedef const __attribute__((address_space(4))) int32_t* table_t;
constexpr float RESCALE_LOG2 = 8.f;             // how far weights may outgrow the reference exponent of their row (see the kernel)

struct AttnArgs {
  const bf16_t* q;      // [M][Hq][hd]
  const bf16_t* kb;     // [M][Hkv][hd] block keys
  const bf16_t* vbT;    // [B*n][Hkv][hd][g.vs] block values, transposed; columns below Lp are values or zeros
  const bf16_t* poolK;  // [pages][Hkv][16][hd]
  const bf16_t* poolV;  // [pages][Hkv][hd][16]
  bf16_t* out;          // [M][Hq*hd]
  BatchGeom g;
  int Hq, Hkv, Lp, q_tiles, total_wg, wg_per_xcd;
  float scale_log2e;
  // launches that cut the key list: n_splits runs of tiles per query tile, and every workgroup leaves an
  // un-normalised partial result for a second kernel to merge
  int n_splits;
  int last_first;       // one block of one beam (prefill): query tiles dealt to the XCDs from the last one down
  int run_tiles;        // single positions (generation): tiles of a run; a beam has as many runs as its length asks for
  int part_splits;      // single positions: partial results of a row, n_splits and, where the launch covers the block keys
  int block_wgs;        // too, one more for these, which the first block_wgs workgroups leave
  float* part_o;        // whole blocks: [b*Hkv + kvh][candidate][q_tile][split][128][HD]
                        // single positions: [b*Hkv + kvh][part_splits][n*g rows][HD]
  float* part_m;        // [..][128] running maximum (log2 domain), -inf if the run was empty
  float* part_l;        // [..][128] sum of weights relative to that maximum
  WeightsAhead ahead;   // touched by the workgroups with blockIdx.y > 0 (an id that costs no argument to know)
};

// The value of lane l and of lane l ^ 32 (v_permlane32_swap: the upper half of one copy trades places with the lower
// half of the other, no trip through the LDS crossbar), combined with max or +.
__device__ __forceinline__ float half_wave_max(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_wave_sum(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Where a key row keeps its 16-byte chunks, so that the rows of a fragment read (16 consecutive lanes) spread over all banks:
// 16 rows in a row, in some order, for 32 query rows a wavefront; rows 8 i + (0..3) or 8 i + (4..7), i = 0..3, for 16.
template <int HD, int ROWS>
__device__ __forceinline__ int k_swizzle(int row, int chunk) {
  if (ROWS == 16) return HD == 128 ? (chunk ^ ((row & 3) | ((row >> 1) & 12))) : (chunk ^ (((row >> 1) & 1) | ((row >> 2) & 6)));
  return HD == 128 ? (chunk ^ (row & 15)) : (chunk ^ ((row >> 1) & 7));
}

// Sixteen query rows of a wavefront, one per lane of each quarter wavefront: launches whose stacked rows do not fill wavefronts
// of 32. A tile takes such a wavefront half the exponentials and half the matrix time, and four of them cover 64 rows that
// would leave half of the workgroup's SIMDs to padding. Bound by the chain of one tile (LDS, scores, maximum, exponentials,
// values). (8 candidates x 32 tokens x 16 heads of 64 dims, 8 kv heads, 512 keys: 10.4 us with wavefronts of 32 rows, 9.1 so;
// single positions of 32 beams x 8 candidates x 12 heads of 128 dims, 2 kv heads, 1024 to 8192 keys: 47.4 and 43.0.)
// Quarter q holds keys 8 q .. 8 q + 7 of each 32: two score products, whose A-rows 4 q + e are keys 8 q + e and 8 q + 4 + e. The
// results are those of wavefronts of 32 rows to the bit: the same products in the same order of K, and the weights are added
// in the order in which a lane there holds them, keys 8 h + 16 i + (0..7) for i = 0..3 on one chain, h = 0 and 1.
template <int HD>
struct Rows16 {
  typedef float floatx4 __attribute__((ext_vector_type(4)));
  bf16x8 qf[HD / 32];                           // dims 32 ks + 8 q .. + 7
  floatx4 o[HD / 16];                           // dims 16 dt + 4 q + e
  float m, l;                                   // l: in the upper half of the wavefront

  __device__ __forceinline__ void clear() {
    m = -INFINITY;
    l = 0.f;
#pragma unroll
    for (int dt = 0; dt < HD / 16; ++dt) o[dt] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  static __device__ __forceinline__ float from_lower(float v) {
    return __uint_as_float(__builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false)[0]);
  }
  static __device__ __forceinline__ float from_upper(float v) {
    return __uint_as_float(__builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false)[1]);
  }
  // the value of lane l in the other quarter of its half: lane l ^ 16
  static __device__ __forceinline__ float quarter_max(float v) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  __device__ __forceinline__ float sum() const {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(l), __float_as_uint(l), false, false);
    return from_upper(__uint_as_float(r[0]) + __uint_as_float(r[1]));
  }

  // one tile of 64 keys; keys from `limit` on are masked if need_mask
  __device__ __forceinline__ void tile(const char* Ks, const char* Vs, bool need_mask, int key_base, int limit, float scale_log2e) {
    const int lane = threadIdx.x & 63, col = lane & 15, quad = lane >> 4;
    bf16x8 kf[4][HD / 32], vf[2][HD / 16];
#pragma unroll
    for (int ks = 0; ks < HD / 32; ++ks)
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int row = 32 * (p >> 1) + 8 * (col >> 2) + 4 * (p & 1) + (col & 3);
        kf[p][ks] = *(const bf16x8*)(Ks + row * HD * 2 + (k_swizzle<HD, 16>(row, ks * 4 + quad) << 4));
      }
    // the values are on their way while the scores become weights
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int dt = 0; dt < HD / 16; ++dt)
        vf[hf][dt] = *(const bf16x8*)(Vs + (hf * 2 + (quad >> 1)) * HD * 32 + (dt * 16 + col) * 32 + (((quad & 1) ^ (col >> 3)) << 4));
    floatx4 s[4];                               // [2 half tile + which four of the eight keys]
#pragma unroll
    for (int p = 0; p < 4; ++p) s[p] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < HD / 32; ++ks)
#pragma unroll
      for (int p = 0; p < 4; ++p) s[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[p][ks], qf[ks], s[p], 0, 0, 0);
    if (need_mask) {
#pragma unroll
      for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          s[p][e] = key_base + 32 * (p >> 1) + 8 * quad + 4 * (p & 1) + e < limit ? s[p][e] : -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int e = 0; e < 4; ++e) mx = fmaxf(mx, s[p][e]);
    mx = half_wave_max(quarter_max(mx));
    const float m_tile = mx * scale_log2e;      // the reference exponent as for 32 rows, below
    const bool move = m_tile > m + RESCALE_LOG2;
    if (__any(move)) {
      const float m_new = move ? ceilf(m_tile) : m;
      const float alpha = move ? __builtin_amdgcn_exp2f(m - m_new) : 1.f;
      l *= alpha;
#pragma unroll
      for (int dt = 0; dt < HD / 16; ++dt) o[dt] *= alpha;
      m = m_new;
    }
    const float m_use = m == -INFINITY ? 0.f : m;
    float p8[2][8];
    bf16x8 pf[2];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        p8[hf][e] = __builtin_amdgcn_exp2f(fmaf(s[2 * hf + (e >> 2)][e & 3], scale_log2e, -m_use));
        pf[hf][e] = (bf16_t)p8[hf][e];
      }
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int dt = 0; dt < HD / 16; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[hf][dt], pf[hf], o[dt], 0, 0, 0);
    // quarters 0 and 2 (1 and 3) in turn: what the other half adds meanwhile is dropped
    float sum = 0.f;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      if (hf) sum = from_upper(sum);
#pragma unroll
      for (int e = 0; e < 8; ++e) sum += p8[hf][e];
      sum = from_lower(sum);
#pragma unroll
      for (int e = 0; e < 8; ++e) sum += p8[hf][e];
    }
    l += sum;
  }
};

// MODE 1's block keys: one workgroup of four wavefronts per (candidate, kv head, 16 of its query heads), which share the
// block keys 0..t and values. The chain of short dependent phases on a few KB, bound by latency, is as long as that of a
// prefix workgroup, so these come first in the launch (10.2 us instead of 8.3 with the prefix workgroups in front).
constexpr int BLOCK_LDS = 32 * 1024;
__host__ __device__ constexpr int block_part_lds(int heads, int Lq) { return heads * (4 * (Lq + 4) + 2 * (Lq + 8)); }

template <int HD>
__device__ __forceinline__ void block_part(const AttnArgs& a, int id, char* smem) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  typedef float floatx4 __attribute__((ext_vector_type(4)));
  constexpr int KS = HD / 32;                   // MFMA K-steps of the scores
  constexpr int ND = HD / 64;                   // 16-dim tiles of the output per wavefront
  constexpr int NVP = 4;                        // 32-key value steps requested up front
  const BatchGeom& G = a.g;
  const int g = a.Hq / a.Hkv, groups = (g + 15) >> 4, t = G.t0;
  const int j0 = id % groups * 16, kvh = id / groups % a.Hkv, c = id / (groups * a.Hkv);
  const int gh = g - j0 < 16 ? g - j0 : 16;     // query heads of this workgroup
  const int Lq = (a.Lp + 31) & ~31;             // keys of the weights, whole MFMA K-steps
  const int SS = Lq + 4, PS = Lq + 8;           // row strides: reads of 16 rows spread over the banks
  const int HS = g < 16 ? g : 16;
  float* sc = (float*)smem;                     // [HS][SS] scores
  bf16_t* pw = (bf16_t*)(sc + HS * SS);         // [HS][PS] weights
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int col = lane & 15, quad = lane >> 4;
  const int b = c / G.n, i = c - b * G.n;
  const int hc = col < gh ? col : gh - 1;       // columns beyond the heads repeat the last one and are not stored

  bf16x8 qf[KS];
  const bf16_t* qr = a.q + ((size_t)c * a.Hq + (size_t)kvh * g + j0 + hc) * HD + 8 * quad;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qf[ks] = *(const bf16x8*)(qr + 32 * ks);
  const int nkt = (t + 16) >> 4;                // 16-key tiles that hold a visible key
  const bf16_t* kbase = a.kb + ((size_t)c * G.Lk * a.Hkv + kvh) * HD + 8 * quad;
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
  // scores of the block keys: lane holds keys 16 kt + 4 quad + e of head col
  for (int kt = wave; kt < nkt; kt += 4) {
    floatx4 s4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) s4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks], qf[ks], s4, 0, 0, 0);
    if (kt + 4 < nkt) load_keys(kt + 4);
    if (col < gh) *(floatx4*)(sc + col * SS + 16 * kt + 4 * quad) = s4 * a.scale_log2e;
  }
  __syncthreads();
  // rows of this workgroup in the partial results
  const size_t prow = (((size_t)b * a.Hkv + kvh) * a.part_splits + a.n_splits) * G.n * g + (size_t)i * g + j0;
  // softmax statistics: 16 lanes per head, all heads at a time
  const int h = tid >> 4, sub = tid & 15;
  if (h < gh) {
    float mx = -INFINITY;
    for (int k = sub; k <= t; k += 16) mx = fmaxf(mx, sc[h * SS + k]);
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
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) l += __shfl_xor(l, o, 16);
    if (sub == 0) { a.part_m[prow + h] = mx; a.part_l[prow + h] = l; }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < ND; ++u) {
    // this lane's output dims: 16 (wave + 4 u) + 4 quad .. + 3 of head col
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    const bf16_t* pr = pw + hc * PS + 8 * quad;
#pragma unroll
    for (int st = 0; st < NVP; ++st)
      if (st < nvs) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(visible_vals(vv[u][st], st), *(const bf16x8*)(pr + 32 * st), acc, 0, 0, 0);
    for (int st = NVP; st < nvs; ++st)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(visible_vals(load_vals(u, st), st), *(const bf16x8*)(pr + 32 * st), acc, 0, 0, 0);
    if (col < gh) *(floatx4*)(a.part_o + (prow + col) * HD + 16 * wave + 64 * u + 4 * quad) = acc;
  }
}

// The launches of a few hundred rows leave CUs and nearly all of HBM idle while their chain of softmaxes runs, and the projections
// behind them wait for weights: what these CUs touch meanwhile comes out of the Infinity Cache afterwards.
__device__ __forceinline__ void touch_weights(const WeightsAhead& a, char* smem) {
  const uint32_t all = gridDim.x * (gridDim.y - 1) * 256, first = (gridDim.x * (blockIdx.y - 1) + blockIdx.x) * 256 + threadIdx.x;
  char* dst = smem + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 256;
#pragma unroll
  for (int r = 0; r < 3; ++r)
    for (uint32_t i = first; i < a.lines[r]; i += all)
      __builtin_amdgcn_global_load_lds(GLB_PTR(a.at[r] + (size_t)i * 32), LDS_PTR(dst), 4, 0, 0);
  __builtin_amdgcn_s_waitcnt(0x0f70);                  // vmcnt(0)
}

// MODE 0: whole blocks, as described above. MODE 1: one position per candidate; the stacked rows of a
// (beam, kv head) are its n candidates x g query heads (row r = i*g + j), the workgroup covers only one run of
// run_tiles prefix tiles and writes (O un-normalised, m, l) instead of the output; the candidate's own block keys
// are covered by further workgroups (block_part), and a second kernel merges. Runs are equally long over all beams, so a launch whose beams differ in length has
// no long workgroups that the others wait for. MODE 2: whole blocks, but the tile list (prefix tiles, then block tiles) is cut
// into n_splits runs handled by different workgroups, for launches that would otherwise leave most CUs idle; a
// merge kernel combines the partial results.
// ROWS: query rows of a wavefront and query tile, 32 or (QT 1, MODE 0 and 1) 16.
template <int HD, int QT, int MODE, int ROWS>
__global__ void __launch_bounds__(256, QT == 1 ? 2 : 1) attention_mfma_kernel(AttnArgs a) {
  static_assert(ROWS == 32 || (ROWS == 16 && QT == 1), "16 rows");
  constexpr bool DEC = MODE == 1, SPLIT = MODE != 0;
  constexpr int KROW = HD * 2;              // bytes per key row
  constexpr int KCH = HD / 8;               // 16-byte chunks per key row
  constexpr int K_BYTES = 64 * KROW;        // 64 keys
  constexpr int V_BYTES = 4 * HD * 32;      // 4 pages of [HD][16]
  constexpr int STAGE = K_BYTES + V_BYTES;
  constexpr int NI = HD / 32;               // direct-to-LDS instructions per wave per operand; also d-tiles
  constexpr int KS = HD / 16;               // MFMA K-steps of the S^T product
  constexpr int BQ = 4 * ROWS * QT;
  extern __shared__ __attribute__((aligned(1024))) char smem[];

  if (blockIdx.y != 0) {
    touch_weights(a.ahead, smem);
    return;
  }
  // workgroup id -> logical index: each XCD (id % 8) takes a contiguous run of the (beam, kv head, candidate, tile)
  // list; single positions deal the (beam, kv head, run) list round, since beams of different lengths lie in a row, and
  // keep the query tiles of one entry together
  int logical = (blockIdx.x & 7) * a.wg_per_xcd + (blockIdx.x >> 3);
  if constexpr (DEC) {
    if ((int)blockIdx.x < a.block_wgs) {
      block_part<HD>(a, blockIdx.x, smem);
      return;
    }
    const int id = blockIdx.x - a.block_wgs;
    const int pass = (id >> 3) / a.q_tiles, qt = (id >> 3) - pass * a.q_tiles;
    logical = (pass * 8 + (id & 7)) * a.q_tiles + qt;
  }
  if ((DEC || !a.last_first) && logical >= a.total_wg) return;
  const BatchGeom& G = a.g;
  const int g = a.Hq / a.Hkv;
  int rem = logical;
  int split = 0;
  if (SPLIT && !DEC && !a.last_first) { split = rem % a.n_splits; rem /= a.n_splits; }
  int qt_idx = rem % a.q_tiles; rem /= a.q_tiles;
  if (DEC) { split = rem % a.n_splits; rem /= a.n_splits; }
  int cand = 0;
  if (!DEC) { cand = rem % G.n; rem /= G.n; }
  int kvh = rem % a.Hkv;
  int b = rem / a.Hkv;
  if (!DEC && a.last_first) {
    // A prompt: the keys of a query tile grow with its position; dealt round from the longest down, all XCDs finish
    // together (a contiguous run of tiles gave an XCD the short or the long ones)
    const int unit = blockIdx.x / a.Hkv;
    if ((int)blockIdx.x >= a.total_wg) return;
    b = 0;
    kvh = blockIdx.x - unit * a.Hkv;
    split = unit % a.n_splits;
    qt_idx = a.q_tiles - 1 - unit / a.n_splits;
  }

  // the wavefront index as a scalar: page ids, page bases and LDS destinations then live in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int lq = lane & (ROWS - 1), lh = lane / ROWS;
  const int P = G.len_override >= 0 ? G.len_override : ((table_t)G.lens)[G.b0 + b];
  const int L = G.L;
  const int cand_idx = b * G.n + cand;
  const size_t m_c0 = (size_t)cand_idx * L;                 // first row of this candidate
  const int rows_total = DEC ? G.n * g : L * g;
  const int r_wg0 = qt_idx * BQ;
  const table_t ptab = (table_t)G.page_table + (size_t)(G.b0 + b) * G.max_pages;

  // --- queries of this wavefront as B-operand fragments (column = query) ---
  int tq[QT];
  bf16x8 qf[QT][KS];
  Rows16<HD> r16;
#pragma unroll
  for (int u = 0; u < QT; ++u) {
    int r = r_wg0 + (wave * QT + u) * ROWS + lq;
    int rc = r < rows_total ? r : rows_total - 1;
    int t = rc / g, j = rc - t * g;                 // DEC: t is the candidate index within the beam
    tq[u] = t;
    const size_t qrow = DEC ? (size_t)b * G.n + t : m_c0 + t;
    const bf16_t* src = a.q + (qrow * a.Hq + (size_t)kvh * g + j) * HD;
    if constexpr (ROWS == 16) {
#pragma unroll
      for (int ks = 0; ks < HD / 32; ++ks) r16.qf[ks] = *(const bf16x8*)(src + ks * 32 + lh * 8);
    } else {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) qf[u][ks] = *(const bf16x8*)(src + ks * 16 + lh * 8);
    }
  }

  r16.clear();
  floatx16 o[QT][NI];
  float m_run[QT], l_run[QT];
#pragma unroll
  for (int u = 0; u < QT; ++u) {
    m_run[u] = -INFINITY;
    l_run[u] = 0.f;
#pragma unroll
    for (int dt = 0; dt < NI; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[u][dt][r] = 0.f;
  }

  const int n_ptiles = (P + 63) >> 6;
  const int n_pages = (P + 15) >> 4;
  int t_hi = (r_wg0 + BQ - 1) / g;
  t_hi = t_hi < L - 1 ? t_hi : L - 1;
  const int n_btiles = DEC ? 0 : ((r_wg0 < rows_total) ? (t_hi >> 6) + 1 : 0);
  // tiles [tile_lo, tile_lo + n_tiles) of the list (prefix tiles, then block tiles)
  const int n_list = n_ptiles + n_btiles;
  const int tile_lo = DEC ? split * a.run_tiles : SPLIT ? (int)((long)split * n_list / a.n_splits) : 0;
  // (the last run takes all that is left: a captured launch may be replayed on a prefix that has grown since)
  const int n_tiles = DEC     ? (split == a.n_splits - 1 || n_list - tile_lo < a.run_tiles ? n_list - tile_lo : a.run_tiles)
                      : SPLIT ? (int)((long)(split + 1) * n_list / a.n_splits) - tile_lo
                              : n_list;
  if (DEC && n_tiles <= 0) return;                     // a run beyond this beam's prefix: the merge does not read it

  // one wavefront stages one 16-key group (a page, or 16 block tokens) of the tile: K rows and V^T
  // physical page of this wavefront's 16-key group of a prefix tile (looked up one tile before it is staged, so
  // that the staging loads never wait for the table)
  auto page_of = [&](int tile) {
    int pg = tile * 4 + wave;
    pg = pg < n_pages ? pg : n_pages - 1;
    return tile < n_ptiles ? ptab[pg] : 0;
  };
  auto stage_tile = [&](int tile, int page_id, char* buf) {
    char* kdst = buf + wave * 16 * KROW;
    char* vdst = buf + K_BYTES + wave * HD * 32;
    if (tile < n_ptiles) {
      // scalar page base + a 32-bit lane offset that does not change from tile to tile
      size_t page = (size_t)__builtin_amdgcn_readfirstlane(page_id);
      const bf16_t* ksrc = a.poolK + (page * a.Hkv + kvh) * 16 * HD;
      const bf16_t* vsrc = a.poolV + (page * a.Hkv + kvh) * HD * 16;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        int qi = i * 64 + lane;
        int row = qi / KCH, slot = qi % KCH;
        int chunk = k_swizzle<HD, ROWS>(wave * 16 + row, slot);
        __builtin_amdgcn_global_load_lds(GLB_PTR(ksrc + (unsigned)(row * HD + chunk * 8)), LDS_PTR(kdst + i * 1024), 16, 0,
                                         0);
      }
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        int qi = i * 64 + lane;
        int d = qi >> 1, half = (qi & 1) ^ ((d >> 3) & 1);       // LDS chunk position qi&1 holds key half `half`
        __builtin_amdgcn_global_load_lds(GLB_PTR(vsrc + (unsigned)(d * 16 + half * 8)), LDS_PTR(vdst + i * 1024), 16, 0, 0);
      }
    } else {
      int key0 = (tile - n_ptiles) * 64 + wave * 16;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        int qi = i * 64 + lane;
        int row = qi / KCH, slot = qi % KCH;
        int chunk = k_swizzle<HD, ROWS>(wave * 16 + row, slot);
        int key = key0 + row;
        key = key < L ? key : L - 1;
        const bf16_t* src = a.kb + ((m_c0 + key) * a.Hkv + kvh) * HD + chunk * 8;
        __builtin_amdgcn_global_load_lds(GLB_PTR(src), LDS_PTR(kdst + i * 1024), 16, 0, 0);
      }
      const bf16_t* vsrc = a.vbT + ((size_t)cand_idx * a.Hkv + kvh) * HD * a.g.vs;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        int qi = i * 64 + lane;
        int d = qi >> 1, half = (qi & 1) ^ ((d >> 3) & 1);
        int key = key0 + half * 8;
        key = key < a.Lp ? key : a.Lp - 8;
        __builtin_amdgcn_global_load_lds(GLB_PTR(vsrc + (size_t)d * a.g.vs + key), LDS_PTR(vdst + i * 1024), 16, 0, 0);
      }
    }
  };

  int page_next = 0;
  if (n_tiles > 0) {
    stage_tile(tile_lo, page_of(tile_lo), smem);
    page_next = page_of(tile_lo + 1);
  }
  // pi(i): A-row i of the S^T product carries key pi(i) of the 32-key half tile
  const int pi_row = (lq & 16) | ((lq & 4) << 1) | ((lq & 8) >> 1) | (lq & 3);

  for (int it = 0; it < n_tiles; ++it) {
    const int tile = tile_lo + it;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (it + 1 < n_tiles) {
      stage_tile(tile + 1, page_next, smem + ((it + 1) & 1) * STAGE);
      page_next = page_of(tile + 2);                   // lands while this tile is being multiplied
    }
    if ((DEC || ROWS == 16) && r_wg0 + wave * QT * ROWS >= rows_total) continue;   // no rows of its own: this wavefront only stages
    const char* Ks = smem + (it & 1) * STAGE;
    const char* Vs = Ks + K_BYTES;
    const bool is_block = tile >= n_ptiles;
    const int key_base = is_block ? (tile - n_ptiles) * 64 : tile * 64;
    if constexpr (ROWS == 16) {
      r16.tile(Ks, Vs, is_block || key_base + 64 > P, key_base, is_block ? tq[0] + 1 : P, a.scale_log2e);
      continue;
    }

    // S^T for the two 32-key halves
    floatx16 s[QT][2];
#pragma unroll
    for (int u = 0; u < QT; ++u)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[u][hf][r] = 0.f;
    // K-step outer, key half inner: the two accumulator chains of a query tile alternate. The key fragments are
    // read KPF K-steps ahead of the MFMAs that use them, so that the LDS latency is hidden behind MFMAs.
    constexpr int KPF = 2;
    auto read_kf = [&](int ks, int hf) {
      int row = hf * 32 + pi_row;
      return *(const bf16x8*)(Ks + row * KROW + (k_swizzle<HD, ROWS>(row, ks * 2 + lh) << 4));
    };
    bf16x8 kf[KPF + 1][2];
#pragma unroll
    for (int ks = 0; ks < KPF; ++ks)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) kf[ks][hf] = read_kf(ks, hf);
    __builtin_amdgcn_sched_group_barrier(0x100, 2 * KPF, 0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ks + KPF < KS) {
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) kf[(ks + KPF) % (KPF + 1)][hf] = read_kf(ks + KPF, hf);
      }
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int u = 0; u < QT; ++u)
          s[u][hf] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks % (KPF + 1)][hf], qf[u][ks], s[u][hf], 0, 0, 0);
      if (ks + KPF < KS) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 2 * QT, 0);
    }

    // accumulator value r of half hf in this lane is key  key_base + hf*32 + 16*(r/8) + 8*lh + r%8
    bf16x8 pf[QT][4];
#pragma unroll
    for (int u = 0; u < QT; ++u) {
      const bool need_mask = is_block || (key_base + 64 > P);
      if (need_mask) {
        const int limit = is_block ? tq[u] + 1 : P;      // keys < limit are visible
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            int key = key_base + hf * 32 + 16 * (r >> 3) + 8 * lh + (r & 7);
            s[u][hf][r] = key < limit ? s[u][hf][r] : -INFINITY;
          }
      }
      float mx = -INFINITY;
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[u][hf][r]);
      mx = half_wave_max(mx);
      // Reference exponent of the row in the log2 domain (scores are scaled by scale*log2(e) > 0 inside the
      // exponent's FMA). It is always an INTEGER: the weights that multiply V are rounded to bf16, and that rounding
      // commutes with a power-of-two scale, so the rounded operand is the same whichever integer reference a tile
      // happens to see (a streaming evaluation and one that knows the global maximum round the same values). It
      // follows the row maximum lazily: the accumulators are rescaled only when the maximum has grown by more than
      // 2^RESCALE_LOG2 past the reference, so weights reach at most that factor (exact in float; O/l at the end
      // does not depend on the reference) and the 64 multiplications per lane become rare.
      const float m_tile = mx * a.scale_log2e;
      const bool move = m_tile > m_run[u] + RESCALE_LOG2;   // also the first visible key: -inf + 8 = -inf
      if (__any(move)) {
        const float m_new = move ? ceilf(m_tile) : m_run[u];
        const float alpha = move ? __builtin_amdgcn_exp2f(m_run[u] - m_new) : 1.f;   // exp2(-inf) = 0: nothing yet
        l_run[u] *= alpha;
#pragma unroll
        for (int dt = 0; dt < NI; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[u][dt][r] *= alpha;
        m_run[u] = m_new;
      }
      const float m_use = m_run[u] == -INFINITY ? 0.f : m_run[u];   // nothing visible yet: every p below is exp2(-inf) = 0
      float psum = 0.f;
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float p = __builtin_amdgcn_exp2f(fmaf(s[u][hf][r], a.scale_log2e, -m_use));
          psum += p;
          pf[u][hf * 2 + (r >> 3)][r & 7] = (bf16_t)p;
        }
      l_run[u] += psum;
    }

    // O^T += V^T P^T : K-step = one 16-key group (page) pg, this lane supplies keys 8*lh .. 8*lh+7 of it
    // (value fragments are read VPF MFMA steps ahead of their use, like the key fragments above)
    constexpr int VPF = 2, NST = 4 * NI;
    auto read_vf = [&](int st) {
      const int pg = st / NI, dt = st % NI;
      return *(const bf16x8*)(Vs + pg * HD * 32 + (dt * 32 + lq) * 32 + ((lh ^ ((lq >> 3) & 1)) << 4));
    };
    bf16x8 vf[VPF + 1];
#pragma unroll
    for (int st = 0; st < VPF; ++st) vf[st] = read_vf(st);
    __builtin_amdgcn_sched_group_barrier(0x100, VPF, 0);
#pragma unroll
    for (int st = 0; st < NST; ++st) {
      const int pg = st / NI, dt = st % NI;
      if (st + VPF < NST) vf[(st + VPF) % (VPF + 1)] = read_vf(st + VPF);
#pragma unroll
      for (int u = 0; u < QT; ++u)
        o[u][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[st % (VPF + 1)], pf[u][pg], o[u][dt], 0, 0, 0);
      if (st + VPF < NST) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, QT, 0);
    }
  }

  // normalise and store: lane = query column, accumulator value r of d-tile dt is d = dt*32 + 8*(r/4) + 4*lh + r%4
#pragma unroll
  for (int u = 0; u < QT; ++u) {
    int r = r_wg0 + (wave * QT + u) * ROWS + lq;
    if (ROWS == 16) m_run[u] = r16.m;
    float l = ROWS == 16 ? r16.sum() : half_wave_sum(l_run[u]);
    if (SPLIT) {
      if ((DEC || ROWS == 16) && r >= rows_total) continue;
      const size_t group = DEC ? (size_t)b * a.Hkv + kvh : ((size_t)b * a.Hkv + kvh) * G.n + cand;
      const size_t prow = DEC ? (group * a.part_splits + split) * rows_total + r
                              : ((group * a.q_tiles + qt_idx) * a.n_splits + split) * 128 + (wave * QT + u) * ROWS + lq;
      if (lh == 0) { a.part_m[prow] = m_run[u]; a.part_l[prow] = l; }
      float* dst = a.part_o + prow * HD;
      if constexpr (ROWS == 16) {
#pragma unroll
        for (int dt = 0; dt < HD / 16; ++dt) *(typename Rows16<HD>::floatx4*)(dst + 16 * dt + 4 * lh) = r16.o[dt];
        continue;
      }
#pragma unroll
      for (int dt = 0; dt < NI; ++dt)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          float4 v = {o[u][dt][r4 * 4], o[u][dt][r4 * 4 + 1], o[u][dt][r4 * 4 + 2], o[u][dt][r4 * 4 + 3]};
          *(float4*)(dst + dt * 32 + 8 * r4 + 4 * lh) = v;
        }
    } else if (r < rows_total) {
      int t = r / g, j = r - t * g;
      float inv = 1.0f / l;
      bf16_t* dst = a.out + ((m_c0 + t) * a.Hq + (size_t)kvh * g + j) * HD;
      if constexpr (ROWS == 16) {
#pragma unroll
        for (int dt = 0; dt < HD / 16; ++dt)
#pragma unroll
          for (int e = 0; e < 4; ++e) dst[16 * dt + 4 * lh + e] = (bf16_t)(r16.o[dt][e] * inv);
        continue;
      }
#pragma unroll
      for (int dt = 0; dt < NI; ++dt)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          int d = dt * 32 + 8 * r4 + 4 * lh;
#pragma unroll
          for (int e = 0; e < 4; ++e) dst[d + e] = (bf16_t)(o[u][dt][r4 * 4 + e] * inv);
        }
    }
  }
}

// Workgroups that touch weights, in units of the `own` that attend: at least wgs of them, beside workgroups that leave CUs without
// one only (32 beams x 8 candidates x 12 heads, 608: nothing gained). A single position, whose runs of keys are short, loses
// where the two share CUs, or where fewer touch (generation with d = 1536, attending + touching: 80 + 160 0.971 of the time, 128 + 128
// 0.971, 64 + 128 0.986; 160 + 160 1.012, 112 + 224 1.008, 96 + 96 1.014).
int ahead_groups(int own, int wgs, bool position) {
  const int more = (wgs + own - 1) / own;
  return own > 256 || (position && own * (1 + more) > 256) ? 0 : more;
}

template <int HD, int QT, int MODE = 0, int ROWS = 32>
static void launch_attn_variant(const AttnArgs& a, hipStream_t s) {
  constexpr int smem = 2 * (64 * HD * 2 + 4 * HD * 32);
  static_assert(smem >= BLOCK_LDS, "MODE 1's block keys");
  static bool configured = false;
  if (!configured) {
    (void)hipFuncSetAttribute((const void*)attention_mfma_kernel<HD, QT, MODE, ROWS>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    configured = true;
  }
  const int own = a.wg_per_xcd * 8 + a.block_wgs, more = ahead_groups(own, a.ahead.wgs, MODE == 1);
  attention_mfma_kernel<HD, QT, MODE, ROWS><<<dim3(own, 1 + more), 256, smem, s>>>(a);
}

// Merge of the partial results of a MODE 2 launch: HD / 4 lanes per (row, query head), each 16 bytes of it, with all of the
// (at most 8) partial results requested at once. Bound by the bytes of the partial results (one
// wavefront per row and head, 8 bytes a lane, one run after the other: 10.6 us for 96 tiles of 5 runs; 7.5 so).
template <int HD>
__global__ void __launch_bounds__(256) attention_split_merge_kernel(const float* __restrict__ part_o,
                                                                    const float* __restrict__ part_m,
                                                                    const float* __restrict__ part_l,
                                                                    bf16_t* __restrict__ out, int n, int L, int Hq, int Hkv,
                                                                    int q_tiles, int n_splits) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  constexpr int LANES = HD / 4, ROWS = 256 / LANES;
  const int g = Hq / Hkv, rows = L * g;                    // stacked rows of a (beam, kv head, candidate)
  const int r = blockIdx.x * ROWS + threadIdx.x / LANES, col = threadIdx.x % LANES;
  if (r >= rows) return;
  const size_t group = blockIdx.y;                         // (b*Hkv + kvh)*n + i
  const size_t bk = group / n, i = group - bk * n, b = bk / Hkv, kvh = bk - b * Hkv;
  const size_t prow0 = ((group * q_tiles + (r >> 7)) * n_splits) * 128 + (r & 127);   // + split*128
  float4 po[8];
  float m[8], pl[8], mx = -INFINITY;
#pragma unroll
  for (int s = 0; s < 8; ++s)
    if (s < n_splits) {
      m[s] = part_m[prow0 + (size_t)s * 128];
      pl[s] = part_l[prow0 + (size_t)s * 128];
      po[s] = ((const float4*)(part_o + (prow0 + (size_t)s * 128) * HD))[col];
    }
#pragma unroll
  for (int s = 0; s < 8; ++s)
    if (s < n_splits) mx = fmaxf(mx, m[s]);
  float l = 0.f;
  float4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < 8; ++s)
    if (s < n_splits) {
      const float w = __builtin_amdgcn_exp2f(m[s] - mx);   // 0 for a run that saw no visible key
      l = fmaf(w, pl[s], l);
      acc.x = fmaf(w, po[s].x, acc.x);
      acc.y = fmaf(w, po[s].y, acc.y);
      acc.z = fmaf(w, po[s].z, acc.z);
      acc.w = fmaf(w, po[s].w, acc.w);
    }
  const float inv = 1.0f / l;
  const int t = r / g, j = r - t * g;
  bf16_t* dst = out + (((b * n + i) * L + t) * Hq + kvh * g + j) * HD + 4 * col;
  *(bf16x4*)dst = bf16x4{(__bf16)(acc.x * inv), (__bf16)(acc.y * inv), (__bf16)(acc.z * inv), (__bf16)(acc.w * inv)};
}

// Returns false if the shape is not one this kernel takes (head_dim 64/128, 16-token pages).
// part: scratch of part_floats floats for launches whose key tiles are split over several workgroups (may be null).
bool launch_attention_mfma(const bf16_t* q, const bf16_t* kb, const bf16_t* vbT, const bf16_t* poolK,
                           const bf16_t* poolV, bf16_t* out, const BatchGeom& g, const ModelDims& md, int Lp,
                           int max_ctx, float* part, size_t part_floats, const WeightsAhead& ahead, hipStream_t s) {
  if ((md.hd != 64 && md.hd != 128) || g.page_tokens != 16 || Lp % 16 != 0) return false;
  AttnArgs a;
  a.ahead = ahead;
  a.q = q; a.kb = kb; a.vbT = vbT; a.poolK = poolK; a.poolV = poolV; a.out = out; a.g = g;
  a.Hq = md.Hq; a.Hkv = md.Hkv; a.Lp = Lp;
  a.last_first = g.B == 1 && g.n == 1;
  a.n_splits = 1; a.run_tiles = 0; a.part_splits = 0; a.block_wgs = 0; a.part_o = nullptr; a.part_m = nullptr; a.part_l = nullptr;
  a.scale_log2e = 1.4426950408889634f / sqrtf((float)md.hd);
  int rows = g.L * (md.Hq / md.Hkv);
  // 256-row workgroups only when they waste less padding than 128-row ones (the latter run two per CU)
  int t1 = (rows + 127) / 128, t2 = (rows + 255) / 256;
  bool big = t2 * 256 < t1 * 128;
  a.q_tiles = big ? t2 : t1;
  a.total_wg = g.B * md.Hkv * g.n * a.q_tiles;
  // Few workgroups and a long key list: cut the list into as many runs as still leave all workgroups resident at
  // once (two per CU; one more run would add a second, almost empty round), at least four tiles per run, at most
  // eight runs.
  int list_tiles = (max_ctx + 63) / 64 + (g.L + 63) / 64;
  int splits = 1;
  if (!big && part && a.total_wg < 384 && list_tiles >= 16 && ((uintptr_t)out & 7) == 0) {   // short lists: a second kernel costs more than it saves
    splits = 512 / a.total_wg;
    splits = splits > 8 ? 8 : splits;
    splits = splits > list_tiles / 4 ? list_tiles / 4 : splits;
    size_t per_split = (size_t)a.total_wg * 128 * (md.hd + 2);
    if (splits > 1 && (size_t)splits * per_split > part_floats) splits = (int)(part_floats / per_split);
    if (splits < 1) splits = 1;
  }
  if (splits > 1) {
    size_t rows_all = (size_t)a.total_wg * splits * 128;
    a.n_splits = splits;
    a.part_o = part; a.part_m = part + rows_all * md.hd; a.part_l = a.part_m + rows_all;
    a.total_wg *= splits;
    a.wg_per_xcd = (a.total_wg + 7) / 8;
    if (rows <= 64) {                                        // 64 rows, 1024 keys: 12.7 us with 32 a wavefront, 11.3 so; 4096: 21.9 and 19.2
      if (md.hd == 128) launch_attn_variant<128, 1, 2, 16>(a, s); else launch_attn_variant<64, 1, 2, 16>(a, s);
    } else {
      if (md.hd == 128) launch_attn_variant<128, 1, 2>(a, s); else launch_attn_variant<64, 1, 2>(a, s);
    }
    const int groups = g.B * md.Hkv * g.n;                   // fewer than 384
    if (md.hd == 128)
      attention_split_merge_kernel<128><<<dim3((rows + 7) / 8, groups), 256, 0, s>>>(
          a.part_o, a.part_m, a.part_l, out, g.n, g.L, md.Hq, md.Hkv, a.q_tiles, splits);
    else
      attention_split_merge_kernel<64><<<dim3((rows + 15) / 16, groups), 256, 0, s>>>(
          a.part_o, a.part_m, a.part_l, out, g.n, g.L, md.Hq, md.Hkv, a.q_tiles, splits);
    return true;
  }
  // At most 64 rows, or so few that each workgroup of 64 has a CU to itself: 16 rows a wavefront (64 rows, 2048 workgroups:
  // 61.0 us with 32, 43.7 so; 128, 192 and 224 rows, 256 workgroups of 64 or fewer: 11.2, 15.2, 15.9 and 9.5, 12.0, 12.9; 384,
  // 512 and 768 workgroups: 11.7, 12.0, 25.9 and 12.7, 12.8, 27.3, since the rows of a wavefront share its reads of the keys).
  const int t64 = (rows + 63) / 64;
  const long wgs64 = (long)g.B * md.Hkv * g.n * t64;
  if (t64 == 1 || wgs64 <= 256) {
    a.q_tiles = t64;
    a.total_wg = (int)wgs64;
    a.wg_per_xcd = (a.total_wg + 7) / 8;
    if (md.hd == 128) launch_attn_variant<128, 1, 0, 16>(a, s); else launch_attn_variant<64, 1, 0, 16>(a, s);
    return true;
  }
  a.wg_per_xcd = (a.total_wg + 7) / 8;
  if (md.hd == 128) { if (big) launch_attn_variant<128, 2>(a, s); else launch_attn_variant<128, 1>(a, s); }
  else { if (big) launch_attn_variant<64, 2>(a, s); else launch_attn_variant<64, 1>(a, s); }
  return true;
}

// How a single-position launch cuts prefixes of lens[0 .. B) tokens: the shortest run that keeps all workgroups resident
// (two per CU), and at most DECODE_MAX_RUNS partial results per row for the merge to read. units: workgroups per run of a
// beam; per_split: floats of the partial results of one run of every beam. (An equal number of runs for every beam, 8 at
// 32 beams of 1k-8k tokens: 35.5 us, the longest beam's workgroups last; runs of equal length, and no stores for the 80 of
// 128 rows that hold no query: 30.7.)
// Longer runs give fewer workgroups and fewer partial results, so the search is by bisection: where no run length meets
// the limits (more than 512 units) it would otherwise go through every length of the longest prefix and all beams.
DecodeRuns plan_decode_runs(const int32_t* lens, int B, int len_override, long units, size_t per_split, size_t part_floats) {
  auto tiles_of = [&](int b) { return ((len_override >= 0 ? len_override : lens[b]) + 63) / 64; };
  int max_tiles = 1;
  long sum_tiles = 0;
  for (int b = 0; b < B; ++b) {
    const int t = tiles_of(b);
    max_tiles = t > max_tiles ? t : max_tiles;
    sum_tiles += t;
  }
  auto fits = [&](int run) {
    if ((size_t)((max_tiles + run - 1) / run) * per_split > part_floats) return false;
    long wgs = 0;
    for (int b = 0; b < B; ++b) wgs += (tiles_of(b) + run - 1) / run;
    return wgs * units <= 512;
  };
  const long least = sum_tiles * units / 512;
  int lo = (max_tiles + DECODE_MAX_RUNS - 1) / DECODE_MAX_RUNS, hi = max_tiles;
  if (least > lo) lo = least < max_tiles ? (int)least : max_tiles;
  while (lo < hi) {
    const int mid = (lo + hi) / 2;
    if (fits(mid)) hi = mid;
    else lo = mid + 1;
  }
  return {lo, (max_tiles + lo - 1) / lo};
}
DecodeRuns plan_decode_runs(const BatchGeom& g, const ModelDims& md, const int32_t* lens_host, size_t part_floats) {
  const int rows = g.n * (md.Hq / md.Hkv);
  const size_t per_split = (size_t)g.B * md.Hkv * rows * (md.hd + 2);
  if (part_floats >= 2 * per_split) part_floats -= per_split;           // the block keys' partial result
  return plan_decode_runs(lens_host + g.b0, g.B, g.len_override, (long)md.Hkv * ((rows + 127) / 128), per_split, part_floats);
}

static int decode_block_wgs(const BatchGeom& g, const ModelDims& md) {
  return g.B * g.n * md.Hkv * ((md.Hq / md.Hkv + 15) / 16);
}
// Whether a single-position launch covers the block keys beside the prefix: where all its workgroups are resident
// at once, two per CU (16 x 12 heads, 4096 keys: 8.3 us + 4.7 for the merge, 8.0 + 7.1 with the block keys in the merge;
// 32 beams x 8 x 12, 1024 to 8192 keys: 35.3 + 8.2 and 31.0 + 8.0), the scores of the block fit the LDS and the partial
// results the scratch. The runs are planned before: where they take up to 512 workgroups by themselves, as a few beams of
// several thousand keys can, the block keys go to the merge, whether or not longer runs would have left room for them
// (not measured).
bool decode_block_beside(const BatchGeom& g, const ModelDims& md, int Lp, const DecodeRuns& runs, size_t part_floats) {
  const int gq = md.Hq / md.Hkv, rows = g.n * gq;
  const long prefix_wgs = (long)g.B * md.Hkv * runs.count * ((rows + 127) / 128);
  return prefix_wgs + decode_block_wgs(g, md) <= 512 && block_part_lds(gq < 16 ? gq : 16, (Lp + 31) & ~31) <= BLOCK_LDS &&
         (size_t)(runs.count + 1) * g.B * md.Hkv * rows * (md.hd + 2) <= part_floats;
}

// Partial results of a single-position launch (g.L == 1) per (beam, kv head, run of key tiles, row), in runs as
// plan_decode_runs gives them, and after the runs those of the block keys if with_block. part_floats: room in `part`
// (floats); returns false if the shape is not taken or the partials of the prefix would not fit.
bool launch_attention_mfma_decode(const bf16_t* q, const bf16_t* kb, const bf16_t* vbT, const bf16_t* poolK,
                                  const bf16_t* poolV, const BatchGeom& g, const ModelDims& md, int Lp, const DecodeRuns& runs,
                                  float* part, size_t part_floats, bool with_block, const WeightsAhead& ahead, hipStream_t s) {
  if ((md.hd != 64 && md.hd != 128) || g.page_tokens != 16 || g.L != 1 || runs.count < 1) return false;
  AttnArgs a;
  a.ahead = ahead;
  a.last_first = 0;
  a.q = q; a.kb = kb; a.vbT = vbT; a.poolK = poolK; a.poolV = poolV; a.out = nullptr; a.g = g;
  a.Hq = md.Hq; a.Hkv = md.Hkv; a.Lp = Lp;
  a.scale_log2e = 1.4426950408889634f / sqrtf((float)md.hd);
  const int rows = g.n * (md.Hq / md.Hkv);
  a.q_tiles = (rows + 127) / 128;
  a.run_tiles = runs.tiles;
  a.n_splits = runs.count;
  const size_t rows_one = (size_t)g.B * md.Hkv * rows;
  const int entries = g.B * md.Hkv * a.n_splits;
  a.total_wg = entries * a.q_tiles;
  a.wg_per_xcd = (entries + 7) / 8 * a.q_tiles;
  a.part_splits = a.n_splits + (with_block ? 1 : 0);
  const size_t rows_all = rows_one * a.part_splits;
  if (rows_all * (md.hd + 2) > part_floats) return false;
  a.part_o = part;
  a.part_m = part + rows_all * md.hd;
  a.part_l = a.part_m + rows_all;
  a.block_wgs = with_block ? decode_block_wgs(g, md) : 0;
  // 16 rows a wavefront where workgroups of 64 rows are no more than those of 128, or all resident at once all the same. The runs
  // and so the results stay. (48 rows of 32 beams: 47.4 us with 32, 43.0 so; 96 rows, 2 kv heads, 4096 keys: 12.9 and 11.7; 112
  // rows, 4 kv heads: 15.3 and 14.4.)
  const int t64 = (rows + 63) / 64;
  if (t64 == 1 || (long)entries * t64 + a.block_wgs <= 512) {
    a.q_tiles = t64;
    a.total_wg = entries * t64;
    a.wg_per_xcd = (entries + 7) / 8 * t64;
    if (md.hd == 128) launch_attn_variant<128, 1, 1, 16>(a, s); else launch_attn_variant<64, 1, 1, 16>(a, s);
  } else {
    if (md.hd == 128) launch_attn_variant<128, 1, 1>(a, s); else launch_attn_variant<64, 1, 1>(a, s);
  }
  return true;
}
