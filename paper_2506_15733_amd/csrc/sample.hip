// Ancestral sampling of one token per row (Alg. 1, Step I): y = min{k : c_k > u * c_V}, c_k the running sum of
// exp(z_v - max z) over vocabulary ids v <= k, i.e. the inverse distribution function of the full softmax in id
// order, read at a uniform u supplied by the caller. Two kernels. The first cuts the ids into 128 chunks and
// leaves, per (row, chunk), the chunk's maximum and its sum of exp(z - chunk max) in double. The second, one block
// per row, rescales the chunk sums to the row maximum, scans them in id order to find the chunk in which the
// running sum crosses the threshold, and repeats the same scan-and-locate inside that chunk over per-thread runs
// and finally over single ids. All sums run in id order; only the grouping of the additions differs from one
// long running sum.
#include "common.h"
#include <climits>

constexpr int SAMPLE_CHUNKS = 128;
constexpr int RUN_REGS = 8;                            // ids of a thread that are kept in registers: up to 262 144 ids
constexpr int RUN_ANY = 0;                             // longer runs: read id by id

// The row's next input: the embedding of its token and its row of the rotary table, which the pick leaves behind (a launch of
// its own takes 4.7 us a position). The angles depend on no token, so they are computed while the pick waits for its loads.
template <typename T>
struct NextInput {
  const T* E;
  float* x;
  float* cs;
  int d, n, hd, b0, len_override, t;
  bool quads;
  double base;
  const int32_t* lens;
};
template <typename T>
__device__ __forceinline__ void next_angles(const NextInput<T>& a, int m, int thread, int threads) {
  const int half = a.hd / 2, pos = (a.len_override >= 0 ? a.len_override : a.lens[a.b0 + m / a.n]) + a.t;
  for (int i = thread; i < half; i += threads) rope_row(a.cs, m, i, pos, half, a.hd, a.base);
}
template <typename T>
__device__ __forceinline__ void next_row(const NextInput<T>& a, size_t m, int id) {
  const T* row = a.E + (size_t)id * a.d;
  float* xo = a.x + m * a.d;
  if (a.quads)
    for (int c = 4 * threadIdx.x; c < a.d; c += 4 * blockDim.x) *(float4*)(xo + c) = load_quad<T>(row + c);
  else
    for (int c = threadIdx.x; c < a.d; c += blockDim.x) xo[c] = to_f32<T>(row[c]);
}

// Scan of one value per thread over 256 threads: a wavefront scans its 64 in registers, one barrier joins the four. Each
// thread takes what it needs from the four totals, in the order in which a running sum over the wavefronts adds them.
struct Scan {
  double incl, excl, total;
};
__device__ __forceinline__ Scan block_scan_256(double v, double* wave_total) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double other = __shfl_up(v, o, 64);
    if (lane >= o) v += other;
  }
  if (lane == 63) wave_total[wave] = v;
  __syncthreads();
  double upto = 0.0, before = 0.0;                     // the wavefronts up to this one, and without it
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if (w == wave) before = upto;
    upto += wave_total[w];
  }
  const double incl = v + before, left = __shfl_up(incl, 1, 64);
  return {incl, lane ? left : before, upto};
}

// Consecutive ids of one thread. In double, exp takes more time than the load: with the number of ids known to the compiler
// and ids beyond the chunk as -infinity, whose exp is an exact 0, it is straight code that holds the polynomial's
// coefficients in scalar registers (24 vector instructions an id; a branch at each id sets them up again, 45: 256 rows of
// 152k ids 70 us, 60 so).
template <int RUN>
__device__ __forceinline__ void load_run(const float* z, int k0, int k1, float* zr) {
#pragma unroll
  for (int j = 0; j < RUN; ++j) zr[j] = k0 + j < k1 ? z[k0 + j] : -INFINITY;
}

// RUN: ids per thread, (ids of a chunk + 255) / 256, up to RUN_REGS, or RUN_ANY
template <int RUN>
__global__ void __launch_bounds__(256) sample_chunks_kernel(const float* __restrict__ logits, int V, int limit,
                                                            float* __restrict__ cmax, double* __restrict__ csum) {
  __shared__ float wmax[4];
  __shared__ double wsum[4];
  const size_t row = blockIdx.x;
  const int chunk = blockIdx.y, tid = threadIdx.x;
  const int CH = (limit + SAMPLE_CHUNKS - 1) / SAMPLE_CHUNKS;
  const int c0 = chunk * CH, c1 = min(limit, c0 + CH);
  const float* z = logits + row * (size_t)V;
  const int run = RUN != RUN_ANY ? RUN : (CH + 255) / 256;
  const int k0 = c0 + tid * run, k1 = min(c1, k0 + run);
  // the thread's ids in registers, requested at once (one load after the other, twice: 256 rows of 152k ids 13
  // us more, 16 rows 1.1)
  float zr[RUN_REGS], mx = -INFINITY;
  if constexpr (RUN != RUN_ANY) {
    load_run<RUN>(z, k0, k1, zr);
#pragma unroll
    for (int j = 0; j < RUN; ++j) mx = fmaxf(mx, zr[j]);
  } else {
    for (int k = k0; k < k1; ++k) mx = fmaxf(mx, z[k]);
  }
  mx = wave_max(mx);
  if ((tid & 63) == 0) wmax[tid >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
  double sm = 0.0;
  if (mx > -INFINITY) {
    if constexpr (RUN != RUN_ANY) {
#pragma unroll
      for (int j = 0; j < RUN; ++j) sm += exp((double)zr[j] - (double)mx);
    } else {
      for (int k = k0; k < k1; ++k) sm += exp((double)z[k] - (double)mx);
    }
  }
  // thread order = id order: add the wavefront's lanes in order, then the four wavefronts
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    double other = __shfl_up(sm, o, 64);
    if ((tid & 63) >= o) sm += other;
  }
  if ((tid & 63) == 63) wsum[tid >> 6] = sm;
  __syncthreads();
  if (tid == 0) {
    cmax[row * SAMPLE_CHUNKS + chunk] = mx;
    csum[row * SAMPLE_CHUNKS + chunk] = ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
  }
}

// A chain of dependent steps on one workgroup per row: what it waits for is latency, so every load whose address is known
// is requested at the start (the sums and u behind a barrier each cost a trip to memory), and what one wavefront decides
// goes through the same barrier as the others' (five in all; with ten and the loads in between 9.9 us at 8 rows
// of 32k ids, 6.7 so; 11.0 and 8.6 at 256 of 152k).
template <typename T, int RUN>
__global__ void __launch_bounds__(256) sample_pick_kernel(const float* __restrict__ logits, int V, int limit,
                                                          const float* __restrict__ cmax,
                                                          const double* __restrict__ csum,
                                                          const double* __restrict__ u, int32_t* __restrict__ cand,
                                                          float* __restrict__ tok_logp, int L, int t, int* status,
                                                          NextInput<T> next) {
  __shared__ double chunk_total[4], run_total[4], over_before[4], last_before[4];
  __shared__ float wmax[4];
  __shared__ int over_at[4], last_at[4], picked[4];
  const size_t row = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* z = logits + row * (size_t)V;
  const int CH = (limit + SAMPLE_CHUNKS - 1) / SAMPLE_CHUNKS;

  const double uu = u[row * L + t];
  const float cm = tid < SAMPLE_CHUNKS ? cmax[row * SAMPLE_CHUNKS + tid] : -INFINITY;
  const double cs = tid < SAMPLE_CHUNKS ? csum[row * SAMPLE_CHUNKS + tid] : 0.0;
  float mx = wave_max(cm);
  if (lane == 0) wmax[wave] = mx;
  if (tid >= SAMPLE_CHUNKS) next_angles(next, (int)row, tid - SAMPLE_CHUNKS, 256 - SAMPLE_CHUNKS);
  __syncthreads();
  mx = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
  const double m = (double)mx;
  const double w = cm > -INFINITY ? cs * exp((double)cm - m) : 0.0;
  const Scan chunks = block_scan_256(w, chunk_total);
  const double total = chunks.total;
  const double thr = uu * total;
  const bool bad_u = !(uu >= 0.0 && uu < 1.0);
  const bool bad_z = !(total > 0.0) || !(total < INFINITY) || !(mx > -INFINITY);
  if (bad_u || bad_z) {
    if (tid == 0) {
      report_status(status, bad_u ? SPECS_ERANGE : SPECS_ENONFINITE);
      cand[row * L + t] = 0;
      tok_logp[row * L + t] = -INFINITY;
    }
    next_row(next, row, 0);
    return;
  }
  // First chunk OF POSITIVE WEIGHT whose inclusive sum exceeds the threshold; none (rounding) -> the last chunk of
  // positive weight that the sum grows in. The scan adds the same terms in a different grouping for every position, so
  // its values need not be monotone to the last bit: "first" is taken as a minimum over the threads that qualify, never
  // as "the one whose predecessor does not qualify", and growth alone is no sign of weight; both may hold for a chunk of
  // zero weight beyond the permitted ids. Every wavefront writes its own two before the barrier and all read them after
  // it, so that all take the same chunk. (As ballots: an LDS maximum over the 128 threads of the chunks makes the kernel
  // 1.2 us longer at 8 rows of 32k ids.)
  const unsigned long long over = __ballot(w > 0.0 && chunks.incl > thr);
  const unsigned long long grown = __ballot(w > 0.0 && (tid == 0 || chunks.incl > chunks.excl));
  const int first_over = over ? __ffsll(over) - 1 : 0, last_grown = grown ? 63 - __clzll(grown) : 0;
  if (lane == first_over) {
    over_at[wave] = over ? tid : INT_MAX;
    over_before[wave] = chunks.excl;
  }
  if (lane == last_grown) {
    last_at[wave] = grown ? tid : -1;
    last_before[wave] = chunks.excl;
  }
  __syncthreads();
  int chunk = 0;
  double before = 0.0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (last_at[i] >= 0) { chunk = last_at[i]; before = last_before[i]; }
#pragma unroll
  for (int i = 3; i >= 0; --i)
    if (over_at[i] != INT_MAX) { chunk = over_at[i]; before = over_before[i]; }
  // the same scan inside the chunk, over per-thread runs of ids
  const int c0 = chunk * CH, c1 = min(limit, c0 + CH);
  const int run = RUN != RUN_ANY ? RUN : (CH + 255) / 256;
  const int k0 = c0 + tid * run, k1 = min(c1, k0 + run);
  double mine = 0.0, wt[RUN_REGS];
  float zr[RUN_REGS];
  load_run<RUN>(z, k0, k1, zr);
  const double log_total = log(total);                 // while the loads are on their way
  if constexpr (RUN != RUN_ANY) {
#pragma unroll
    for (int j = 0; j < RUN; ++j) {
      wt[j] = exp((double)zr[j] - m);
      mine += wt[j];
    }
  } else {
    for (int k = k0; k < k1; ++k) mine += exp((double)z[k] - m);
  }
  const Scan runs = block_scan_256(mine, run_total);
  // the first run of each wavefront that crosses the threshold, as above, and the id in it; the first wavefront's counts
  const unsigned long long crosses = __ballot(mine > 0.0 && runs.incl + before > thr);
  if (lane == (crosses ? __ffsll(crosses) - 1 : 0)) {
    int pick = -1;
    if (crosses) {
      double c = runs.excl + before;
      int positive = -1;                               // the first id past the threshold, or the last one of positive weight
      if constexpr (RUN != RUN_ANY) {
#pragma unroll
        for (int j = 0; j < RUN; ++j)
          if (k0 + j < k1 && pick < 0) {
            c += wt[j];
            if (c > thr) pick = k0 + j;
            if (wt[j] > 0.0) positive = k0 + j;
          }
      } else {
        for (int k = k0; k < k1 && pick < 0; ++k) {
          const double w1 = exp((double)z[k] - m);
          c += w1;
          if (c > thr) pick = k;
          if (w1 > 0.0) positive = k;
        }
      }
      if (pick < 0) pick = positive;
    }
    picked[wave] = pick;
  }
  __syncthreads();
  int pick = -1;
#pragma unroll
  for (int i = 3; i >= 0; --i)
    if (picked[i] >= 0) pick = picked[i];
  if (pick < 0) {                                      // threshold not exceeded inside the chunk: its last id of positive weight
    for (int k = c1 - 1; k >= c0; --k)
      if (exp((double)z[k] - m) > 0.0) { pick = k; break; }
    if (pick < 0) pick = c0;
  }
  if (tid == 0) {
    cand[row * L + t] = pick;
    tok_logp[row * L + t] = (float)((double)z[pick] - m - log_total);
  }
  next_row(next, row, pick);
}

// Vocabularies of at most 4096 permitted ids: one block per row holds its logits in registers, four consecutive ids per
// thread, and makes the same choice with one scan (two kernels, the pick as it was then: 4.3 + 6.8 us at 16 rows of 512 ids; 8.3 so. With 32
// ids per thread for 32k ids the exponentials of a row, on one CU, take 38 us; the two kernels 3.9 + 6.7).
template <typename T>
__global__ void __launch_bounds__(1024) sample_row_kernel(const float* __restrict__ logits, int V, int limit,
                                                          const double* __restrict__ u, int32_t* __restrict__ cand,
                                                          float* __restrict__ tok_logp, int L, int t, int* status,
                                                          NextInput<T> next) {
  constexpr int RUN = 4;
  __shared__ float wmax[16];
  __shared__ double wtotal[16];
  __shared__ int first, last, sel;
  const int waves = blockDim.x >> 6;
  const size_t row = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, k0 = tid * RUN;
  const float* z = logits + row * (size_t)V;
  const double uu = u[row * L + t];
  float zr[RUN];
  float mx = -INFINITY;
#pragma unroll
  for (int k = 0; k < RUN; ++k) zr[k] = k0 + k < limit ? z[k0 + k] : -INFINITY;
#pragma unroll
  for (int k = 0; k < RUN; ++k) mx = fmaxf(mx, zr[k]);
  mx = wave_max(mx);
  if (lane == 0) wmax[wave] = mx;
  if (tid == 0) { first = INT_MAX; last = -1; }
  next_angles(next, (int)row, tid, blockDim.x);
  __syncthreads();
  for (int w = 0; w < waves; ++w) mx = fmaxf(mx, wmax[w]);
  const double m = (double)mx;
  double wt[RUN], mine = 0.0;
#pragma unroll
  for (int k = 0; k < RUN; ++k) {
    wt[k] = k0 + k < limit ? exp((double)zr[k] - m) : 0.0;
    mine += wt[k];
  }
  double incl = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double other = __shfl_up(incl, o, 64);
    if (lane >= o) incl += other;
  }
  if (lane == 63) wtotal[wave] = incl;
  const double up = __shfl_up(incl, 1, 64);
  __syncthreads();
  double before = 0.0, total = 0.0;
  for (int w = 0; w < waves; ++w) {
    if (w == wave) before = total;
    total += wtotal[w];
  }
  incl += before;
  const double thr = uu * total;
  const bool bad_u = !(uu >= 0.0 && uu < 1.0);
  const bool bad_z = !(total > 0.0) || !(total < INFINITY) || !(mx > -INFINITY);
  if (bad_u || bad_z) {
    if (tid == 0) {
      report_status(status, bad_u ? SPECS_ERANGE : SPECS_ENONFINITE);
      cand[row * L + t] = 0;
      tok_logp[row * L + t] = -INFINITY;
    }
    next_row(next, row, 0);
    return;
  }
  // the first run of positive weight that crosses the threshold; none (rounding): the last run of positive weight
  if (mine > 0.0) {
    if (incl > thr) atomicMin(&first, tid);
    atomicMax(&last, tid);
  }
  __syncthreads();
  if (tid == (first != INT_MAX ? first : last)) {
    double c = before + (lane ? up : 0.0);
    int pick = -1, positive = -1;
#pragma unroll
    for (int k = 0; k < RUN; ++k)
      if (k0 + k < limit) {
        c += wt[k];
        if (wt[k] > 0.0) positive = k0 + k;
        if (pick < 0 && first != INT_MAX && c > thr) pick = k0 + k;
      }
    if (pick < 0) pick = positive;
    sel = pick;
    cand[row * L + t] = pick;
    tok_logp[row * L + t] = (float)((double)z[pick] - m - log(total));
  }
  __syncthreads();
  next_row(next, row, sel);
}

size_t sample_scratch_bytes(int rows) { return (size_t)rows * SAMPLE_CHUNKS * (sizeof(double) + sizeof(float)); }

// scratch: sample_scratch_bytes(rows) bytes, 8-byte aligned
template <typename T>
void launch_sample_tokens(const float* logits, int rows, int V, int limit, const double* u, int32_t* cand,
                          float* tok_logp, int L, void* scratch, int* status, const T* E, float* x, int d, float* cs,
                          const BatchGeom& g, int hd, float base, hipStream_t s) {
  const NextInput<T> next = {E, x, cs, d, g.n, hd, g.b0, g.len_override, g.t0, embed_quads(E, x, d), (double)base, g.lens};
  if (limit <= 4096) {
    sample_row_kernel<T><<<rows, (limit + 255) / 256 * 64, 0, s>>>(logits, V, limit, u, cand, tok_logp, L, g.t0, status, next);
    return;
  }
  double* csum = (double*)scratch;
  float* cmax = (float*)(csum + (size_t)rows * SAMPLE_CHUNKS);
  const int run = ((limit + SAMPLE_CHUNKS - 1) / SAMPLE_CHUNKS + 255) / 256;
#define SAMPLE_RUN(R)                                                                                               \
  case R:                                                                                                           \
    sample_chunks_kernel<R><<<dim3(rows, SAMPLE_CHUNKS), 256, 0, s>>>(logits, V, limit, cmax, csum);                 \
    sample_pick_kernel<T, R><<<rows, 256, 0, s>>>(logits, V, limit, cmax, csum, u, cand, tok_logp, L, g.t0, status, \
                                                  next);                                                            \
    break;
  switch (run <= RUN_REGS ? run : RUN_ANY) {
    SAMPLE_RUN(1) SAMPLE_RUN(2) SAMPLE_RUN(3) SAMPLE_RUN(4) SAMPLE_RUN(5) SAMPLE_RUN(6) SAMPLE_RUN(7) SAMPLE_RUN(RUN_REGS)
    SAMPLE_RUN(RUN_ANY)
  }
#undef SAMPLE_RUN
}
template void launch_sample_tokens<float>(const float*, int, int, int, const double*, int32_t*, float*, int, void*, int*,
                                          const float*, float*, int, float*, const BatchGeom&, int, float, hipStream_t);
template void launch_sample_tokens<bf16_t>(const float*, int, int, int, const double*, int32_t*, float*, int, void*, int*,
                                           const bf16_t*, float*, int, float*, const BatchGeom&, int, float, hipStream_t);
