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

// Inclusive scan of 256 values, left in buf[256]: a wavefront scans its 64 in registers, one barrier joins the four.
// (Through LDS with two barriers per doubling: 10.6 us for the pick kernel at 16 rows of 152k ids, 9.5 so.)
__device__ __forceinline__ double block_scan_256(double v, double* buf, double* wave_total) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double other = __shfl_up(v, o, 64);
    if (lane >= o) v += other;
  }
  if (lane == 63) wave_total[wave] = v;
  __syncthreads();
  double before = 0.0;
  for (int w = 0; w < wave; ++w) before += wave_total[w];
  v += before;
  buf[tid] = v;
  __syncthreads();
  return v;
}

__global__ void __launch_bounds__(256) sample_chunks_kernel(const float* __restrict__ logits, int V, int limit,
                                                            float* __restrict__ cmax, double* __restrict__ csum) {
  __shared__ float wmax[4];
  __shared__ double wsum[4];
  const size_t row = blockIdx.x;
  const int chunk = blockIdx.y, tid = threadIdx.x;
  const int CH = (limit + SAMPLE_CHUNKS - 1) / SAMPLE_CHUNKS;
  const int c0 = chunk * CH, c1 = min(limit, c0 + CH);
  const float* z = logits + row * (size_t)V;
  const int run = (CH + 255) / 256;
  const int k0 = c0 + tid * run, k1 = min(c1, k0 + run);
  // the thread's ids in registers, requested at once (one load after the other, twice: 256 rows of 152k ids 82
  // us instead of 69, 16 rows 8.6 instead of 7.5)
  float zr[RUN_REGS], mx = -INFINITY;
  if (run <= RUN_REGS) {
#pragma unroll
    for (int j = 0; j < RUN_REGS; ++j) zr[j] = k0 + j < k1 ? z[k0 + j] : -INFINITY;
#pragma unroll
    for (int j = 0; j < RUN_REGS; ++j) mx = fmaxf(mx, zr[j]);
  } else {
    for (int k = k0; k < k1; ++k) mx = fmaxf(mx, z[k]);
  }
  mx = wave_max(mx);
  if ((tid & 63) == 0) wmax[tid >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
  double sm = 0.0;
  if (mx > -INFINITY) {
    if (run <= RUN_REGS) {
#pragma unroll
      for (int j = 0; j < RUN_REGS; ++j)
        if (j < run) sm += k0 + j < k1 ? exp((double)zr[j] - (double)mx) : 0.0;
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

template <typename T>
__global__ void __launch_bounds__(256) sample_pick_kernel(const float* __restrict__ logits, int V, int limit,
                                                          const float* __restrict__ cmax,
                                                          const double* __restrict__ csum,
                                                          const double* __restrict__ u, int32_t* __restrict__ cand,
                                                          float* __restrict__ tok_logp, int L, int t, int* status,
                                                          NextInput<T> next) {
  __shared__ double buf[256], wave_total[4];
  __shared__ float wmax[4];
  __shared__ int sel, over_at[4], last_at[4];
  const size_t row = blockIdx.x;
  const int tid = threadIdx.x, wave = tid >> 6;
  const float* z = logits + row * (size_t)V;
  const int CH = (limit + SAMPLE_CHUNKS - 1) / SAMPLE_CHUNKS;

  float mx = tid < SAMPLE_CHUNKS ? cmax[row * SAMPLE_CHUNKS + tid] : -INFINITY;
  mx = wave_max(mx);
  if ((tid & 63) == 0) wmax[wave] = mx;
  if (tid >= SAMPLE_CHUNKS) next_angles(next, (int)row, tid - SAMPLE_CHUNKS, 256 - SAMPLE_CHUNKS);
  __syncthreads();
  mx = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
  const double m = (double)mx;
  double w = 0.0;
  if (tid < SAMPLE_CHUNKS) {
    float cm = cmax[row * SAMPLE_CHUNKS + tid];
    if (cm > -INFINITY) w = csum[row * SAMPLE_CHUNKS + tid] * exp((double)cm - m);
  }
  double incl = block_scan_256(w, buf, wave_total);
  const double total = buf[255];
  const double uu = u[row * L + t];
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
  // 11.2 us at 8 rows of 32k ids.)
  const unsigned long long over = __ballot(w > 0.0 && incl > thr);
  const unsigned long long grown = __ballot(w > 0.0 && (tid == 0 || buf[tid] > buf[tid - 1]));
  if ((tid & 63) == 0) {
    over_at[wave] = over ? tid + __ffsll(over) - 1 : INT_MAX;
    last_at[wave] = grown ? tid + 63 - __clzll(grown) : 0;
  }
  __syncthreads();
  int chunk = min(min(over_at[0], over_at[1]), min(over_at[2], over_at[3]));
  if (chunk == INT_MAX) chunk = max(max(last_at[0], last_at[1]), max(last_at[2], last_at[3]));
  const double before = chunk ? buf[chunk - 1] : 0.0;
  __syncthreads();                                     // buf is reused below
  // the same scan inside the chunk, over per-thread runs of ids
  const int c0 = chunk * CH, c1 = min(limit, c0 + CH);
  const int run = (CH + 255) / 256;
  const int k0 = c0 + tid * run, k1 = min(c1, k0 + run);
  double mine = 0.0, wt[RUN_REGS];
  if (run <= RUN_REGS) {
    float zr[RUN_REGS];
#pragma unroll
    for (int j = 0; j < RUN_REGS; ++j) zr[j] = k0 + j < k1 ? z[k0 + j] : -INFINITY;
#pragma unroll
    for (int j = 0; j < RUN_REGS; ++j) {
      wt[j] = j < run && k0 + j < k1 ? exp((double)zr[j] - m) : 0.0;
      mine += wt[j];
    }
  } else {
    for (int k = k0; k < k1; ++k) mine += exp((double)z[k] - m);
  }
  incl = block_scan_256(mine, buf, wave_total) + before;
  const double excl = (tid ? buf[tid - 1] : 0.0) + before;
  __shared__ int first;
  if (tid == 0) { sel = -1; first = INT_MAX; }
  __syncthreads();
  if (mine > 0.0 && incl > thr) atomicMin(&first, tid);       // the first run that crosses the threshold, as above
  __syncthreads();
  if (tid == first) {
    double c = excl;
    int pick = -1, positive = -1;                      // the first id past the threshold; the last one of positive weight
    if (run <= RUN_REGS) {
#pragma unroll
      for (int j = 0; j < RUN_REGS; ++j)
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
    sel = pick < 0 ? positive : pick;
  }
  __syncthreads();
  int pick = sel;
  if (pick < 0) {                                      // threshold not exceeded inside the chunk: its last id of positive weight
    for (int k = c1 - 1; k >= c0; --k)
      if (exp((double)z[k] - m) > 0.0) { pick = k; break; }
    if (pick < 0) pick = c0;
  }
  if (tid == 0) {
    cand[row * L + t] = pick;
    tok_logp[row * L + t] = (float)((double)z[pick] - m - log(total));
  }
  next_row(next, row, pick);
}

// Vocabularies of at most 4096 permitted ids: one block per row holds its logits in registers, four consecutive ids per
// thread, and makes the same choice with one scan (two kernels: 4.3 + 6.8 us at 16 rows of 512 ids; 8.3 so. With 32
// ids per thread for 32k ids the exponentials of a row, on one CU, take 38 us; the two kernels 4.5 + 9.2).
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
  sample_chunks_kernel<<<dim3(rows, SAMPLE_CHUNKS), 256, 0, s>>>(logits, V, limit, cmax, csum);
  sample_pick_kernel<T><<<rows, 256, 0, s>>>(logits, V, limit, cmax, csum, u, cand, tok_logp, L, g.t0, status, next);
}
template void launch_sample_tokens<float>(const float*, int, int, int, const double*, int32_t*, float*, int, void*, int*,
                                          const float*, float*, int, float*, const BatchGeom&, int, float, hipStream_t);
template void launch_sample_tokens<bf16_t>(const float*, int, int, int, const double*, int32_t*, float*, int, void*, int*,
                                           const bf16_t*, float*, int, float*, const BatchGeom&, int, float, hipStream_t);
