// Straightforward shared-prefix attention: one wavefront per (row, query head). Serves the float
// configuration, head sizes the MFMA kernel does not take, and launches that cover one in-block position of every
// candidate (row m = candidate m / L at position t0 + m % L; its block keys are rows cand*Lk .. of kb). Three passes over the keys:
// scores into LDS (+ max), un-normalised weights 2^(s' - ceil(max s')) in the log2 domain (+ sum; the integer
// reference makes the bf16 rounding of the weights independent of which power of two they are scaled by), weighted
// sum of V.
// The key loop reads a key row in 16-byte pieces where alignment allows; the value loop deals the keys over the 64 / hd
// groups of lanes that the head dimension leaves and adds the groups' sums in order (16 lanes walking every key, one
// division and one page lookup each: 20 us for 16 rows of 4 heads on 100 to 230 keys).
#include "common.h"

// QUADS: hd % 4 == 0 and key rows aligned for load_quad. pt_shift: log2(page_tokens), negative if it is no power of two.
template <typename T, bool QUADS>
__global__ void __launch_bounds__(64) attention_simple_kernel(const T* __restrict__ q, const T* __restrict__ kb,
                                                              const T* __restrict__ vbT, const T* __restrict__ poolK,
                                                              const T* __restrict__ poolV, T* __restrict__ out,
                                                              BatchGeom g, int Hq, int Hkv, int hd, int pt_shift, float scale) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  float* qs = smem;                             // [hd] query staged in LDS as float
  float* sc = smem + hd;                        // [ctx + t + 1] scores, then weights
  int m = blockIdx.x, h = blockIdx.y, lane = threadIdx.x;
  int nL = g.n * g.L;
  int b = m / nL, t = g.t0 + m % g.L;               // in-block position of this row
  int ctx = g.len_override >= 0 ? g.len_override : g.lens[g.b0 + b];
  int kvh = h / (Hq / Hkv);
  int nkeys = ctx + t + 1;
  const T* qr = q + ((size_t)m * Hq + h) * hd;
  const int32_t* pt = g.page_table + (size_t)(g.b0 + b) * g.max_pages;
  for (int c = lane; c < hd; c += 64) qs[c] = to_f32<T>(qr[c]);
  __syncthreads();
  auto page_slot = [&](int j, int& slot) {
    const int p = pt_shift >= 0 ? j >> pt_shift : j / g.page_tokens;
    slot = j - p * g.page_tokens;
    return pt[p];
  };

  float mx = -INFINITY;
  for (int j = lane; j < nkeys; j += 64) {
    const T* kr;
    if (j < ctx) {
      int slot;
      const int page = page_slot(j, slot);
      kr = poolK + (((size_t)page * Hkv + kvh) * g.page_tokens + slot) * hd;
    } else {
      kr = kb + (((size_t)(m / g.L) * g.Lk + (j - ctx)) * Hkv + kvh) * hd;
    }
    float dot = 0.f;
    if (QUADS) {
#pragma unroll 4
      for (int c = 0; c < hd; c += 4) {
        const float4 kv = load_quad<T>(kr + c), qv = *(const float4*)(qs + c);
        dot = fmaf(qv.x, kv.x, dot);
        dot = fmaf(qv.y, kv.y, dot);
        dot = fmaf(qv.z, kv.z, dot);
        dot = fmaf(qv.w, kv.w, dot);
      }
    } else {
      for (int c = 0; c < hd; ++c) dot = fmaf(qs[c], to_f32<T>(kr[c]), dot);
    }
    dot *= scale;                                // scale = log2(e) / sqrt(hd): scores in the log2 domain
    sc[j] = dot;
    mx = fmaxf(mx, dot);
  }
  mx = ceilf(wave_max(mx));
  float sm = 0.f;
  for (int j = lane; j < nkeys; j += 64) {
    float p = exp2f(sc[j] - mx);
    sm += p;
    sc[j] = to_f32<T>(from_f32<T>(p));          // the weight that multiplies V is an operand: rounded to T
  }
  sm = wave_sum(sm);
  __syncthreads();
  float inv = 1.0f / sm;
  // values are stored transposed: pages [page][Hkv][hd][pt], block [cand][Hkv][hd][vs]
  size_t cand = (size_t)(m / g.L);
  auto weighted_sum = [&](int c, int first, int step) {
    float acc = 0.f;
    const T* vpool = poolV + ((size_t)kvh * hd + c) * g.page_tokens;
    const size_t page_stride = (size_t)Hkv * hd * g.page_tokens;
    int j = first;
#pragma unroll 8
    for (; j < ctx; j += step) {
      int slot;
      const int page = page_slot(j, slot);
      acc = fmaf(sc[j], to_f32<T>(vpool[page * page_stride + slot]), acc);
    }
    const T* vblk = vbT + ((cand * Hkv + kvh) * hd + c) * g.vs;
#pragma unroll 4
    for (; j < nkeys; j += step) acc = fmaf(sc[j], to_f32<T>(vblk[j - ctx]), acc);
    return acc;
  };
  T* dst = out + ((size_t)m * Hq + h) * hd;
  const int groups = 64 / hd;                   // lanes per head dimension
  if (groups > 1) {
    const int grp = lane / hd, c = lane - grp * hd;
    const float mine = grp < groups ? weighted_sum(c, grp, groups) : 0.f;
    float acc = mine;
    for (int k = 1; k < groups; ++k) acc += __shfl(mine, k * hd + c, 64);
    if (grp == 0) dst[c] = from_f32<T>(acc * inv);
  } else {
    for (int c = lane; c < hd; c += 64) dst[c] = from_f32<T>(weighted_sum(c, 0, 1) * inv);
  }
}

template <typename T>
void launch_attention_simple(const T* q, const T* kb, const T* vbT, const T* poolK, const T* poolV, T* out,
                             const BatchGeom& g, const ModelDims& md, int max_ctx, hipStream_t s) {
  const size_t lds = (size_t)(max_ctx + g.Lk + md.hd) * sizeof(float);
  const float scale = 1.4426950408889634f / sqrtf((float)md.hd);
  int shift = 0;
  while ((1 << shift) < g.page_tokens) ++shift;
  if ((1 << shift) != g.page_tokens) shift = -1;
  const bool quads = md.hd % 4 == 0 && (((uintptr_t)kb | (uintptr_t)poolK) & (4 * sizeof(T) - 1)) == 0;
#define GO(Q)                                                                                                          \
  (void)hipFuncSetAttribute((const void*)attention_simple_kernel<T, Q>, hipFuncAttributeMaxDynamicSharedMemorySize,    \
                            (int)lds);                                                                                 \
  attention_simple_kernel<T, Q><<<dim3(g.M, md.Hq), 64, lds, s>>>(q, kb, vbT, poolK, poolV, out, g, md.Hq, md.Hkv,     \
                                                                  md.hd, shift, scale)
  if (quads) { GO(true); } else { GO(false); }
#undef GO
}
template void launch_attention_simple<float>(const float*, const float*, const float*, const float*, const float*,
                                             float*, const BatchGeom&, const ModelDims&, int, hipStream_t);
template void launch_attention_simple<bf16_t>(const bf16_t*, const bf16_t*, const bf16_t*, const bf16_t*,
                                              const bf16_t*, bf16_t*, const BatchGeom&, const ModelDims&, int,
                                              hipStream_t);
