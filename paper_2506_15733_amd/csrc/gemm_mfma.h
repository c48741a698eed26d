// bf16 MFMA GEMM for gfx950: C[M,N] = A[M,K] * W[N,K]^T, float accumulation, K % 64 == 0.
//
// Block tiles of 256 or 128 rows x 256 columns, where two rows of wavefronts take turns at the matrix cores and at moving
// operands, or narrower ones with a ring of whole K-tiles for smaller products. All multiply with v_mfma_f32_16x16x32_bf16.
// Operand tiles go global -> LDS directly (16 bytes per lane, no register staging). LDS rows are 128 bytes (64 bf16); the
// 16-byte chunk c of row r is stored at chunk position c ^ ((r >> 1) & 7) so that the 16 rows a fragment read touches
// spread over all banks. Workgroup ids are dealt round-robin to the 8 XCDs by the hardware; the id -> tile map
// below keeps the M-tiles of one N-tile on one XCD, so a weight tile is fetched from HBM once
// and re-used out of that XCD's L2 by workgroups that walk through K in step.
//
// Epilogues: plain float store; residual add into the float stream; SwiGLU (gate/up columns
// interleaved in groups of 32 so that a lane holds gate and up of the same unit) with bf16
// output; QKV projection: rotary embedding, conversion and the layouts of attention; vocabulary head: per-row (max, sum exp)
// over the tile's 256 columns plus the logit of the row's target token, so that logits never reach memory.
#pragma once
#include "common.h"
#include <type_traits>

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

#define LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))
#define GLB_PTR(p) ((const __attribute__((address_space(1))) void*)(p))

enum MfmaEpilogue { ME_STORE = 0, ME_RESIDUAL = 1, ME_SWIGLU = 2, ME_LMHEAD = 3, ME_QKV_ROPE = 4 };

struct GemmArgs {
  const bf16_t* A;
  const bf16_t* W;
  int M, N, K;
  int m_tiles, n_tiles;
  float* C;              // ME_STORE / ME_RESIDUAL: [M, N]
  bf16_t* act;           // ME_SWIGLU: [M, N/2]
  const int32_t* tok;    // ME_LMHEAD: target token per row
  float* part_max;       // ME_LMHEAD: [M, part_tiles]
  float* part_sum;
  float* zt;             // ME_LMHEAD: [M]
  int ksplit;            // ME_STORE only: slices of K, slice s writes its partial product to C + s*M*N
  int rest_block, rest_m_tiles, rest_n_tiles;   // REST kernels: the first workgroup of the rest, its tiles
  int part_tiles;        // ME_LMHEAD: entries of a row in part_max and part_sum
  // ME_QKV_ROPE: the product is the QKV projection [M, (Hq + 2 Hkv) * hd]; the epilogue rotates the q and k heads
  // (pairs (i, i + hd/2), angles from the table cs[M][hd] = cos | sin) and writes bf16 q [M][Hq][hd], block keys
  // kblk[cand][Lk][Hkv][hd] and block values transposed per candidate vT[cand][Hkv][hd][Lp], where row m is in-block position
  // t0 + m % Lrows of candidate m / Lrows.
  const float* cs;
  bf16_t* q;
  bf16_t* kblk;
  bf16_t* vT;
  int Hq, Hkv, Lrows, Lk, Lp, t0;
};

// One direct-to-LDS load instruction: the workgroup's NW wavefronts write NW consecutive 1 KiB spans
// (8 rows of 128 bytes each) of an operand tile.
// SWAP56: LDS row r holds tile row r with bits 5 and 6 exchanged (see the ME_QKV_ROPE epilogue).
// SPANS: of the whole tile; where the wavefronts outnumber the last of them, some fetch the last one again.
template <int NW, int SPANS, bool SWAP56 = false>
__device__ __forceinline__ void load_span_async(const bf16_t* __restrict__ G, int row0, int rows_total, int K, int k0,
                                                char* lds_tile, int p, int wave) {
  const int lane = threadIdx.x & 63;
  int span = p * NW + wave;                  // 1 KiB of LDS = 8 rows, written by one wavefront
  if (SPANS % NW != 0) span = span < SPANS ? span : SPANS - 1;
  int q = span * 64 + lane;
  int row = q >> 3, slot = q & 7;
  int chunk = slot ^ ((row >> 1) & 7);
  int grow = row0 + (SWAP56 ? ((row & ~0x60) | ((row & 0x20) << 1) | ((row & 0x40) >> 1)) : row);
  grow = grow < rows_total ? grow : rows_total - 1;
  const bf16_t* src = G + (size_t)grow * K + k0 + chunk * 8;
  __builtin_amdgcn_global_load_lds(GLB_PTR(src), LDS_PTR(lds_tile + span * 1024), 16, 0, 0);
}

__device__ __forceinline__ bf16x8 lds_frag(const char* tile, int row, int chunk) {
  return *(const bf16x8*)(tile + row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4));
}

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
// the same of lane l and of lane l ^ 16 (v_permlane16_swap: odd rows of 16 lanes against even ones)
__device__ __forceinline__ float quarter_wave_max(float v) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float quarter_wave_sum(float v) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Workgroup -> (K slice, m_tile, n_tile): ids congruent mod 8 share an XCD. The tile list goes through bands of 32 N-tiles,
// in a band through blocks of 8 M-tiles, in a block through sub-bands of 4 N-tiles, so that 32 consecutive entries are
// 8 M-tiles x 4 N-tiles: an XCD that runs them at one time fetches every A panel into its L2 once per 4 users and
// every W tile once per 8 users. Every 256 entries the XCDs take 32 each: they then work on the same 8 A panels at the
// same time (with one contiguous eighth of the list each they drift apart in M: 16384 x 37888 x 3584 then takes 5 %
// longer). What is left, and all of a short list, is cut into eight equal runs. The list has no gaps: a grid padded to whole blocks leaves the
// shader engines of an XCD unevenly loaded (with 70 tiles of one M-tile all of them met on one engine of four and ran
// in two rounds: 48 us instead of 26 at 64 x 17920 x 1536).
struct TileAt { int kslice, m, n; };
__device__ __forceinline__ bool tile_of(int block, int m_tiles, int n_tiles, int ksplit, TileAt& at) {
  const int tiles = m_tiles * n_tiles, total = tiles * ksplit;
  const int xcd = block & 7, slot = block >> 3, dealt = total >> 8;
  int idx;
  if (slot < 32 * dealt) {
    idx = (slot >> 5) * 256 + xcd * 32 + (slot & 31);
  } else {
    const int rest = total - 256 * dealt, run = (rest + 7) >> 3, i = xcd * run + slot - 32 * dealt;
    if (i >= rest) return false;                         // slot - 32 * dealt < run by the size of the grid
    idx = 256 * dealt + i;
  }
  at.kslice = idx / tiles;
  idx -= at.kslice * tiles;
  const int band = idx / (32 * m_tiles);
  idx -= band * 32 * m_tiles;
  const int bw = n_tiles - 32 * band < 32 ? n_tiles - 32 * band : 32;
  const int mb = idx / (8 * bw);
  idx -= mb * 8 * bw;
  const int mh = m_tiles - 8 * mb < 8 ? m_tiles - 8 * mb : 8;
  at.m = 8 * mb + idx % mh;
  at.n = 32 * band + idx / mh;
  return true;
}
static int tile_grid(int total) { return 8 * (32 * (total / 256) + (total % 256 + 7) / 8); }

// ---- epilogues ----
// An accumulator [i][j] of a wavefront is a 16x16 tile of the TRANSPOSED product (the W fragment is the first MFMA operand):
// lane l holds columns 4 (l / 16) .. + 3 of row l % 16. The storing epilogues write them as one 16-byte (8-byte bf16) piece,
// and the vocabulary head reduces most of a row inside the lane. m, n: first row and column of the wavefront's part.
// part: ME_LMHEAD, the tile's entry in a row of part_max.
template <int BM, int BN, int NWM, int EPI, bool HD128, int TM>
__device__ __forceinline__ void epilogue(const GemmArgs& a, floatx4 (&acc)[TM][4], int m0, int n0, int wm, int wn, int kslice, int part,
                                         char* smem) {
  constexpr int NWN = BN / 64, NW = NWM * NWN, TN = 4;
  const int lane = threadIdx.x & 63, r16 = lane & 15, quad = lane >> 4;
  const int m = m0 + wm * 16 * TM, n = n0 + wn * 64;
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  // one decision for the workgroup: a tile inside the matrix stores without per-piece bounds checks
  const bool inside = m0 + BM <= a.M && n0 + BN <= a.N;
  if constexpr (EPI == ME_STORE || EPI == ME_RESIDUAL) {
    float* __restrict__ Cs = a.C + (size_t)kslice * a.M * a.N;
    // PIECES: 16 bytes at a time, aligned and wholly inside a row or outside. (Where a check per piece chooses between 16 bytes
    // and elements, the compiler splits the pieces to share a tail: 256 x 131072 x 1536 152 us instead of 134.)
    auto emit = [&](auto pieces, auto checked) {
      constexpr bool PIECES = decltype(pieces)::value, CHECK = decltype(checked)::value;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = m + i * 16 + r16;
        if (CHECK && row >= a.M) continue;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int col = n + j * 16 + 4 * quad;
          float* dst = Cs + (size_t)row * a.N + col;
          if constexpr (PIECES) {
            if (CHECK && col >= a.N) continue;
            floatx4 v = acc[i][j];
            if (EPI == ME_RESIDUAL) v += *(const floatx4*)dst;
            *(floatx4*)dst = v;
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (col + e < a.N) {
                if (EPI == ME_RESIDUAL) dst[e] += acc[i][j][e];
                else dst[e] = acc[i][j][e];
              }
          }
        }
      }
    };
    if ((a.N & 3) != 0 || ((uintptr_t)a.C & 15) != 0) emit(std::false_type{}, std::true_type{});
    else if (inside) emit(std::true_type{}, std::false_type{});
    else emit(std::true_type{}, std::true_type{});
  } else if constexpr (EPI == ME_SWIGLU) {
    const int F = a.N >> 1;                            // a multiple of 32: whole 4-unit pieces
    auto emit = [&](auto checked) {
      constexpr bool CHECK = decltype(checked)::value;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = m + i * 16 + r16;
#pragma unroll
        for (int j = 0; j < TN / 2; ++j) {             // columns 0..31 of the part are gates, 32..63 the same units' ups
          const int unit = (n >> 1) + j * 16 + 4 * quad;
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float gt = acc[i][j][e], u = acc[i][j + TN / 2][e];
            // v_rcp_f32 (1 ulp) instead of an IEEE division: the quotient is rounded to bf16 right away, and the
            // division's scale/fix-up sequence alone was ten instructions per value
            o[e] = (__bf16)(gt * __builtin_amdgcn_rcpf(1.0f + __expf(-gt)) * u);
          }
          if (!CHECK || (row < a.M && unit < F)) *(bf16x4*)(a.act + (size_t)row * F + unit) = o;
        }
      }
    };
    if (inside) emit(std::false_type{});
    else emit(std::true_type{});
  } else if constexpr (EPI == ME_QKV_ROPE) {
    // columns 0..31 of the part: 32 pairs' first elements, 32..63 their second ones
    constexpr int HDIM = HD128 ? 128 : 64, HALF = HDIM / 2;
    const int head = HD128 ? (n >> 7) : (n >> 6), wq = HD128 ? (n >> 6) & 1 : 0;
    const int i_base = wq * 32 + 4 * quad;                               // + 16 j + e: index of the pair inside the head
    if (head < a.Hq + 2 * a.Hkv) {
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = m + i * 16 + r16;
        const int cand = row / a.Lrows, t = a.t0 + row - cand * a.Lrows;
        if (head < a.Hq + a.Hkv) {
          if (row >= a.M) continue;
          const float* cs = a.cs + (size_t)row * HDIM;
          bf16_t* dst = head < a.Hq ? a.q + ((size_t)row * a.Hq + head) * HDIM
                                    : a.kblk + (((size_t)cand * a.Lk + t) * a.Hkv + (head - a.Hq)) * HDIM;
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int i0 = i_base + 16 * j;
            const float4 cn = *(const float4*)(cs + i0), sn = *(const float4*)(cs + HALF + i0);
            const float c4[4] = {cn.x, cn.y, cn.z, cn.w}, s4[4] = {sn.x, sn.y, sn.z, sn.w};
            bf16x4 y1, y2;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float2 y = rotate_pair(acc[i][j][e], acc[i][2 + j][e], c4[e], s4[e]);
              y1[e] = (__bf16)y.x;
              y2[e] = (__bf16)y.y;
            }
            *(bf16x4*)(dst + i0) = y1;
            *(bf16x4*)(dst + HALF + i0) = y2;
          }
        } else {
          // values: not rotated, stored transposed; 16 lanes write 16 consecutive positions
          bf16_t* head_v = a.vT + (size_t)(head - a.Hq - a.Hkv) * HDIM * a.Lp;
          const size_t cand_v = (size_t)a.Hkv * HDIM * a.Lp;
          if (row < a.M) {
            bf16_t* dst = head_v + cand * cand_v + t;
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const int d = i_base + 16 * j + e;
                dst[(size_t)d * a.Lp] = (__bf16)acc[i][j][e];
                dst[(size_t)(HALF + d) * a.Lp] = (__bf16)acc[i][2 + j][e];
              }
          }
          // The positions that pad a candidate's block to whole 16s: the wavefront that holds its last row clears them, a
          // lane per column (the lanes of that row on their own took 32 stores a position).
          unsigned ends = (unsigned)(__ballot(row < a.M && t == a.Lk - 1 && a.Lp > a.Lk) & 0xffff);
          while (ends) {
            const int of = __builtin_amdgcn_readlane(cand, __builtin_ctz(ends));
            ends &= ends - 1;
            const int d = HD128 ? wq * 32 + (lane & 31) + (lane >> 5) * HALF : lane;
            bf16_t* pad = head_v + of * cand_v + (size_t)d * a.Lp;
            for (int k = a.Lk; k < a.Lp; ++k) pad[k] = (__bf16)0.f;
          }
        }
      }
    }
  } else {  // ME_LMHEAD
    __syncthreads();                                   // every wavefront is done with the operand tiles
    float* red_max = (float*)smem;                     // [BM][NWN]
    float* red_sum = red_max + BM * NWN;
    // A lane owns, of row r16 of each of its TM row tiles, the 16 columns with (column / 4) % 4 == quad: maximum and sum of
    // exponentials run over the lane's own registers, two exchanges join the four lanes of a row, and the row's target column
    // is looked for among the same registers.
    const bool ragged = n0 + BN > a.N;                 // only the last N-tile has columns beyond the matrix
    const int cbase = n + 4 * quad;                    // column of element (j, e): cbase + 16 j + e
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int lr = wm * 16 * TM + i * 16 + r16, row = m0 + lr;
      const int target = row < a.M ? a.tok[row] : -1;
      float mx = -INFINITY;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (ragged && cbase + 16 * j + e >= a.N) acc[i][j][e] = -INFINITY;
          mx = fmaxf(mx, acc[i][j][e]);
        }
      mx = half_wave_max(quarter_wave_max(mx));
      const int d = target - cbase;                    // the target's offset among this lane's columns
      float sm = 0.f, zt = 0.f;
      bool hit = false;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float v = acc[i][j][e];
          sm += mx == -INFINITY ? 0.f : __expf(v - mx);
          const bool here = d == 16 * j + e;
          zt = here ? v : zt;
          hit |= here;
        }
      sm = half_wave_sum(quarter_wave_sum(sm));
      if (hit) a.zt[row] = zt;
      if (quad == 0) {
        red_max[lr * NWN + wn] = mx;
        red_sum[lr * NWN + wn] = sm;
      }
    }
    __syncthreads();
    for (int lr = threadIdx.x; lr < BM; lr += 64 * NW) {
      int row = m0 + lr;
      if (row < a.M) {
        float mx = -INFINITY;
#pragma unroll
        for (int w = 0; w < NWN; ++w) mx = fmaxf(mx, red_max[lr * NWN + w]);
        float sm = 0.f;
#pragma unroll
        for (int w = 0; w < NWN; ++w)
          if (red_max[lr * NWN + w] > -INFINITY) sm += red_sum[lr * NWN + w] * expf(red_max[lr * NWN + w] - mx);
        a.part_max[(size_t)row * a.part_tiles + part] = mx;
        a.part_sum[(size_t)row * a.part_tiles + part] = sm;
      }
    }
  }
}

// Rotary pairs are columns (i, i + hd/2) of a head. With head_dim 64 a wavefront's 64 columns are one head, the first 32 of
// them one half of its pairs. With head_dim 128 a head spans two wavefronts, so the W tile is loaded with rows 32..63 and
// 64..95 of every 128 exchanged: wavefront (head, wq) then holds columns wq*32 .. +31 of the first half in its first 32
// columns and the same columns of the second half in the others. (A tile of 64 columns is loaded from its whole head's rows.)
__device__ __forceinline__ constexpr int swap56(int row) { return (row & ~0x60) | ((row & 0x20) << 1) | ((row & 0x40) >> 1); }

// K-tiles [kt0, kt0 + KT) of K slice kslice
__device__ __forceinline__ void slice_tiles(const GemmArgs& a, int kslice, int& kt0, int& KT) {
  kt0 = (int)((long)kslice * (a.K / 64) / a.ksplit);
  KT = (int)((long)(kslice + 1) * (a.K / 64) / a.ksplit) - kt0;
}

// Barriers of a workgroup, in which no instruction moves across. LANDED_AND_MEET: own LDS reads are done before it (their
// place may be overwritten after it), and own loads but the newest n have landed. The compiler is told of the wait, as it
// would otherwise wait for these reads, and all later ones with them, where they are used.
#define MEET()                            \
  __builtin_amdgcn_sched_barrier(0);      \
  asm volatile("s_barrier" ::: "memory"); \
  __builtin_amdgcn_sched_barrier(0)
#define LANDED_AND_MEET(n)                                          \
  asm volatile("" ::: "memory");                                    \
  __builtin_amdgcn_sched_barrier(0);                                \
  __builtin_amdgcn_s_waitcnt(((n) & 15) | ((n) >> 4) << 14 | 0x70); \
  MEET()

// The BM x 256 tile (BM 256, 192 or 128) of the product at (m0, n0), K slice kslice, by eight wavefronts 2 (M) x 4 (N).
//
// The two rows of wavefronts, one wavefront of each on every SIMD, run half a phase apart: while one multiplies (16 MFMAs, 64
// rows x 32 columns x 64 deep of its part), the other reads the fragments of its next phase from LDS and requests operands,
// and a barrier changes the roles. Reads, address arithmetic and the wait for a place in the memory queue then stand beside
// the other wavefront's MFMAs instead of in front of the own ones. (One loop for all wavefronts with loads and reads dealt
// between the MFMAs and a barrier per K-tile, us: 16384 x 37888 x 3584 3360, 8192 x 8192 x 8192 798, 2048 x 37888 x 3584
// 473, so: 2920, 695, 399, i.e. 1.52, 1.58 and 1.39 PFLOP/s. With 32x32x16 MFMAs: 3183, 764, 423: they move twice as much
// of the accumulators per flop, and the clock of a power-limited part shows it. A phase of 32 MFMAs, 64 x 64: 2962, 703, 400.)
//
// Every phase reads one piece of an operand tile and frees its place in the LDS ring a phase later, so the ring is filled
// piece by piece, as far ahead as it goes: BM = 256: 16 KiB halves in the order A0 W1 A1 W0', one per phase (half 0, 1 of A: rows 0..63, 64..127 of
// each row of wavefronts, half 0, 1 of W: columns 0..31, 32..63 of each wavefront; ' the next K-tile's), ten of them in
// 160 KiB, i.e. nearly two and a half K-tiles. BM = 128: A | W1 W0' in two phases, three K-tiles in 144 KiB.
// Operands are requested through buffer descriptors whose size ends with the matrix: rows beyond it, and K-tiles beyond the
// slice (size 0), are zeros that cost no traffic. Without BUFFER by plain addresses, the last row and K-tile again in their place.
template <int BM, int EPI, bool HD128, bool BUFFER>
__device__ __forceinline__ void wide_product(const GemmArgs& a, int m0, int n0, int kslice, int part, char* smem) {
  static_assert(BM == 256 || (BM == 192 && BUFFER) || BM == 128, "two halves of A, or one");
  constexpr bool SWAP = EPI == ME_QKV_ROPE && HD128;
  constexpr int NH = BM == 128 ? 1 : 2, TMH = BM / NH / 32, TM = TMH * NH, U = 8192;    // U: what one load of every wavefront fills
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm = wave >> 2, wn = wave & 3, r16 = lane & 15, quad = lane >> 4;
  int kt0, KT;
  slice_tiles(a, kslice, kt0, KT);

  floatx4 acc[TM][4];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  // Offsets of the 16 bytes that this lane requests. A half is 128 LDS rows in 16 spans of 8; a wavefront fills spans `wave`
  // and 8 + wave. All of a row is in the vector offset, which the bounds check covers; the scalar offset advances along K.
  const bf16_t *Ab = a.A + (size_t)m0 * a.K + kt0 * 64, *Wb = a.W + (size_t)n0 * a.K + kt0 * 64;
  const unsigned row_bytes = (unsigned)a.K * 2u;
  const unsigned a_size = (unsigned)min(a.M - m0, BM) * row_bytes - kt0 * 128, w_size = (unsigned)min(a.N - n0, 256) * row_bytes - kt0 * 128;
  unsigned aoff[NH][2], woff[2][2];
  const bf16_t *aptr[NH][2], *wptr[2][2];                // without BUFFER, in place of the offsets
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int r = (p * 8 + wave) * 8 + (lane >> 3);
    const unsigned chunk = ((lane & 7) ^ ((r >> 1) & 7)) * 16;
#pragma unroll
    for (int h = 0; h < NH; ++h) {                       // rows beyond the half (BM = 192: 96 of 128) are zeros
      const int wr = r / (16 * TMH), row = wr * 16 * TM + h * 16 * TMH + r - wr * 16 * TMH;
      aoff[h][p] = wr < 2 ? (unsigned)row * row_bytes + chunk : 0x7fffffffu;
      if constexpr (!BUFFER) aptr[h][p] = Ab + (size_t)min(row, a.M - 1 - m0) * a.K + chunk / 2;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = (r >> 5) * 64 + h * 32 + (r & 31);
      woff[h][p] = (unsigned)(SWAP ? swap56(c) : c) * row_bytes + chunk;
      if constexpr (!BUFFER) wptr[h][p] = Wb + (size_t)min(SWAP ? swap56(c) : c, a.N - 1 - n0) * a.K + chunk / 2;
    }
  }
  // Unit p of half h of A (W) of K-tile t, to unit `slot` of the ring
  auto load_a = [&](int h, int p, int slot, int t) {
    if constexpr (BUFFER) {
      const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)Ab, 0, t < KT ? a_size : 0u, 0x00020000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, LDS_PTR(smem + slot * U + wave * 1024), 16, aoff[h][p], t * 128, 0, 0);
    } else {
      __builtin_amdgcn_global_load_lds(GLB_PTR(aptr[h][p] + min(t, KT - 1) * 64), LDS_PTR(smem + slot * U + wave * 1024), 16, 0, 0);
    }
  };
  auto load_w = [&](int h, int p, int slot, int t) {
    if constexpr (BUFFER) {
      const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)Wb, 0, t < KT ? w_size : 0u, 0x00020000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, LDS_PTR(smem + slot * U + wave * 1024), 16, woff[h][p], t * 128, 0, 0);
    } else {
      __builtin_amdgcn_global_load_lds(GLB_PTR(wptr[h][p] + min(t, KT - 1) * 64), LDS_PTR(smem + slot * U + wave * 1024), 16, 0, 0);
    }
  };

  // A fragment is 16 rows x 32 of K: lane l has row l % 16, chunk l / 16 (of 4; chunks 4..7 are the second 32). The rows of a
  // lane's fragments differ by multiples of 16, so they share their swizzle.
  const int sw = (r16 >> 1) & 7, c0 = (quad ^ sw) << 4, c1 = c0 ^ 64;
  const int abase = (wm * 16 * TMH + r16) * 128, bbase = (wn * 32 + r16) * 128;
  bf16x8 af[TMH][2], b0[2][2], b1[2][2];
  auto read_a = [&](int slot) {
    const char* p = smem + slot * U + abase;
#pragma unroll
    for (int i = 0; i < TMH; ++i) {
      af[i][0] = *(const bf16x8*)(p + i * 2048 + c0);
      af[i][1] = *(const bf16x8*)(p + i * 2048 + c1);
    }
  };
  auto read_w = [&](int slot, bf16x8 (&b)[2][2]) {
    const char* p = smem + slot * U + bbase;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      b[j][0] = *(const bf16x8*)(p + j * 2048 + c0);
      b[j][1] = *(const bf16x8*)(p + j * 2048 + c1);
    }
  };
  auto mma = [&](int hm, int hn, const bf16x8 (&b)[2][2]) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < TMH; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[hm * TMH + i][hn * 2 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j][kk], af[i][kk], acc[hm * TMH + i][hn * 2 + j], 0, 0, 0);
  };
  if constexpr (NH == 2) {
    // Position s of the stream of halves: s = 0 is W0 of K-tile 0; of K-tile t A0 is 4t + 1, W1 4t + 2, A1 4t + 3 and the next
    // one's W0 4t + 4. Phase s reads half s. Its first part requests half s + 9, in the place of half s - 1, which
    // the later row of wavefronts has read in the first part of phase s - 1; eight halves are newer than the next one read.
    auto load_half = [&](int s, int t) {                 // s modulo 20, t the K-tile that the half belongs to
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        if (s & 1) load_a((s & 3) >> 1, p, s % 10 * 2 + p, t);
        else load_w((s & 3) >> 1, p, s % 10 * 2 + p, t);
      }
    };
#pragma unroll
    for (int s = 0; s < 9; ++s) load_half(s, s >> 2);
    LANDED_AND_MEET(14);                                         // s = 0 and 1
    load_half(9, 2);
    read_w(0, b0);
    LANDED_AND_MEET(16);
    if (wm == 1) { MEET(); }
    auto step = [&](auto phase, int t) {
      constexpr int S = decltype(phase)::value * 4;      // 4t modulo 20
      read_a((S + 1) % 10 * 2);
      load_half(S + 10, t + 2);
      LANDED_AND_MEET(16);
      mma(0, 0, b0);
      MEET();
      read_w((S + 2) % 10 * 2, b1);
      load_half(S + 11, t + 2);
      LANDED_AND_MEET(16);
      mma(0, 1, b1);
      MEET();
      read_a((S + 3) % 10 * 2);
      load_half(S + 12, t + 3);
      LANDED_AND_MEET(16);
      mma(1, 0, b0);
      MEET();
      read_w((S + 4) % 10 * 2, b0);                      // after the last K-tile: zeros, never used
      load_half(S + 13, t + 3);
      LANDED_AND_MEET(16);
      mma(1, 1, b1);
      MEET();
    };
    for (int t = 0;;) {
      step(std::integral_constant<int, 0>{}, t); if (++t >= KT) break;
      step(std::integral_constant<int, 1>{}, t); if (++t >= KT) break;
      step(std::integral_constant<int, 2>{}, t); if (++t >= KT) break;
      step(std::integral_constant<int, 3>{}, t); if (++t >= KT) break;
      step(std::integral_constant<int, 4>{}, t); if (++t >= KT) break;
    }
  } else {
    // Position s of the stream of units: 0 and 1 are W0 of K-tile 0; of K-tile t A is 6t + 2, 3, W1 6t + 4, 5 and the next
    // one's W0 6t + 6, 7. The first phase of a K-tile reads A and requests 6t + 16 .. 18, the second W1 and W0' and requests
    // 6t + 19 .. 21, each into places read a phase before at the latest.
    auto load_unit = [&](int s, int t) {                 // s modulo 18, t: s belongs to K-tile t (6t + 2 <= s < 6t + 8)
      const int r = (s + 4) % 6;
      if (r < 2) load_a(0, r, s % 18, t);
      else if (r < 4) load_w(1, r - 2, s % 18, t);
      else load_w(0, r - 4, s % 18, t + 1);
    };
#pragma unroll
    for (int s = 0; s < 16; ++s) load_unit(s, (s + 4) / 6 - 1);
    LANDED_AND_MEET(12);                                         // W0 and A of K-tile 0
    read_w(0, b0);
    LANDED_AND_MEET(12);
    if (wm == 1) { MEET(); }
    auto step = [&](auto phase, int t) {
      constexpr int S = decltype(phase)::value * 6;      // 6t modulo 18
      read_a(S + 2);
      load_unit(S + 16, t + 2); load_unit(S + 17, t + 2); load_unit(S + 18, t + 2);
      LANDED_AND_MEET(11);
      mma(0, 0, b0);
      MEET();
      read_w(S + 4, b1);
      read_w((S + 6) % 18, b0);                          // after the last K-tile: zeros, never used
      load_unit(S + 19, t + 2); load_unit(S + 20, t + 3); load_unit(S + 21, t + 3);
      LANDED_AND_MEET(12);
      mma(0, 1, b1);
      MEET();
    };
    for (int t = 0;;) {
      step(std::integral_constant<int, 0>{}, t); if (++t >= KT) break;
      step(std::integral_constant<int, 1>{}, t); if (++t >= KT) break;
      step(std::integral_constant<int, 2>{}, t); if (++t >= KT) break;
    }
  }
  if (wm == 0) { MEET(); }                               // both rows of wavefronts have met the same barriers
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  epilogue<BM, 256, 2, EPI, HD128>(a, acc, m0, n0, wm, wn, kslice, part, smem);
}

// The BM x BN tile of the product at (m0, n0), K slice kslice, for products of few rows or few tiles: the k-step is bound by
// the latency of the operand loads and by what a wavefront issues per k-step, not by the matrix pipe. So the ring holds S whole
// K-tiles, nearly all of them in flight, and a load is one vector instruction (us with the addresses computed per load, and
// the last K-tiles in loops of their own / so: 256 x 2048 x 1024 8.3 / 7.2, 1024 x 1536 x 1536 13.0 / 11.0,
// 256 x 1536 x 8960 in 5 slices 14.9 / 12.7, gate/up of 256 x 5632 x 1024 9.0 / 7.5).
template <int BM, int BN, int NWM, int S, int EPI, bool HD128, bool BUFFER>
__device__ __forceinline__ void ring_product(const GemmArgs& a, int m0, int n0, int kslice, int part, char* smem) {
  static_assert(BUFFER || BN > 64, "whole heads");
  constexpr bool SWAP = EPI == ME_QKV_ROPE && HD128;
  constexpr int NWN = BN / 64, NW = NWM * NWN;        // wavefronts: NWM along M x NWN along N, 64 columns each
  constexpr int WM = BM / NWM, TM = WM / 16, TN = 4;
  constexpr int LA = (BM / 8 + NW - 1) / NW, LB = (BN / 8 + NW - 1) / NW, NLD = LA + LB;   // loads per thread and operand tile
  constexpr int STG = (BM + BN) * 128;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm = wave / NWN, wn = wave % NWN;
  const int r16 = lane & 15, quad = lane >> 4;
  int kt0, KT;
  slice_tiles(a, kslice, kt0, KT);

  floatx4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto mma = [&](const bf16x8 (&af)[TM], const bf16x8 (&bfr)[TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
  };
  auto read_frags = [&](const char* st, int kk, bf16x8 (&af)[TM], bf16x8 (&bfr)[TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i) af[i] = lds_frag(st, wm * WM + i * 16 + r16, kk * 4 + quad);
#pragma unroll
    for (int j = 0; j < TN; ++j) bfr[j] = lds_frag(st + BM * 128, wn * 64 + j * 16 + r16, kk * 4 + quad);
  };
  // Load j of a K-tile fills 1 KiB of LDS (8 rows) per wavefront; where the wavefronts outnumber the last spans of an operand
  // tile, some fetch the last one again. BUFFER: by descriptors that end with the matrix (and are empty behind the slice), so
  // that a load is one vector instruction, with all of a row in the offset that the bounds check covers.
  const unsigned row_bytes = (unsigned)a.K * 2u;
  constexpr bool HALF_HEAD = SWAP && BN == 64;
  const int w0 = HALF_HEAD ? n0 & ~127 : n0, w_rows = HALF_HEAD ? 128 : BN;
  const unsigned a_size = (unsigned)min(a.M - m0, BM) * row_bytes - kt0 * 128, w_size = (unsigned)min(a.N - w0, w_rows) * row_bytes - kt0 * 128;
  const bf16_t *Ab = a.A + (size_t)m0 * a.K + kt0 * 64, *Wb = a.W + (size_t)w0 * a.K + kt0 * 64;
  int dst[NLD];
  unsigned off[NLD];
#pragma unroll
  for (int j = 0; j < NLD; ++j) {
    const int spans = j < LA ? BM / 8 : BN / 8, span = min((j < LA ? j : j - LA) * NW + wave, spans - 1);
    const int row = span * 8 + (lane >> 3), w_row = HALF_HEAD ? swap56(n0 - w0 + row) : SWAP ? swap56(row) : row;
    dst[j] = (j < LA ? 0 : BM * 128) + span * 1024;
    off[j] = (unsigned)(j < LA ? row : w_row) * row_bytes + ((lane & 7) ^ ((row >> 1) & 7)) * 16;
  }
  // loads [lo, hi) of K-tile t
  auto issue = [&](int t, char* st, auto lo, auto hi) {
    if constexpr (BUFFER) {
      const auto ra = __builtin_amdgcn_make_buffer_rsrc((void*)Ab, 0, t < KT ? a_size : 0u, 0x00020000);
      const auto rw = __builtin_amdgcn_make_buffer_rsrc((void*)Wb, 0, t < KT ? w_size : 0u, 0x00020000);
#pragma unroll
      for (int j = decltype(lo)::value; j < decltype(hi)::value; ++j)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(j < LA ? ra : rw, LDS_PTR(st + dst[j]), 16, off[j], t * 128, 0, 0);
    } else {
      const int src = t < KT ? t : KT - 1;             // behind the slice: redundant loads
#pragma unroll
      for (int j = decltype(lo)::value; j < decltype(hi)::value; ++j) {
        if (j < LA) load_span_async<NW, BM / 8>(a.A, m0, a.M, a.K, (kt0 + src) * 64, st, j, wave);
        else load_span_async<NW, BN / 8, SWAP>(a.W, n0, a.N, a.K, (kt0 + src) * 64, st + BM * 128, j - LA, wave);
      }
    }
  };
  constexpr std::integral_constant<int, 0> FIRST{};
  constexpr std::integral_constant<int, NLD / 2> MID{};
  constexpr std::integral_constant<int, NLD> LAST{};
#define SGB __builtin_amdgcn_sched_group_barrier
  // fragment reads, then MFMAs with a load after each of the first
  auto order = [&](auto loads) {
    constexpr int N = decltype(loads)::value;
    SGB(0x100, TM + TN, 0);
#pragma unroll
    for (int i = 0; i < N && i < TM * TN; ++i) {
      SGB(0x008, 1, 0);
      SGB(0x010, 1, 0);
    }
    SGB(0x008, TM * TN, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // own loads of all but the newest S - 2 K-tiles have landed and own fragment reads are done, then everybody's
  static_assert((S - 2) * NLD < 63, "the counter's range");
#pragma unroll
  for (int t = 0; t < S - 1; ++t) issue(t, smem + t * STG, FIRST, LAST);
  LANDED_AND_MEET((S - 2) * NLD);
  bf16x8 a0[TM], b0[TN], a1[TM], b1[TN];
  issue(S - 1, smem + (S - 1) * STG, FIRST, MID);
  char* cur = smem;                                    // slot of K-tile kt, and of kt + S once kt has been read
  char* last = smem + (S - 1) * STG;                   // slot of K-tile kt - 1, and of kt - 1 + S
  read_frags(cur, 0, a0, b0);
  // A K-tile's slot is free once all have read its second half, a barrier and half of its MFMAs before the next K-tile
  // begins: the first loads of K-tile kt + S follow there, the others a half later.
  for (int kt = 0; kt < KT; ++kt) {
    char* nxt = cur + STG == smem + S * STG ? smem : cur + STG;
    read_frags(cur, 1, a1, b1);
    issue(kt + S - 1, last, MID, LAST);
    mma(a0, b0);
    order(std::integral_constant<int, NLD - NLD / 2>{});
    LANDED_AND_MEET((S - 2) * NLD);
    read_frags(nxt, 0, a0, b0);                        // after the last K-tile: not used
    issue(kt + S, cur, FIRST, MID);
    mma(a1, b1);
    order(std::integral_constant<int, NLD / 2>{});
    last = cur;
    cur = nxt;
  }
#undef SGB
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  epilogue<BM, BN, NWM, EPI, HD128>(a, acc, m0, n0, wm, wn, kslice, part, smem);
}

template <int BM, int BN, int NWM, int S, int EPI, bool HD128, bool BUFFER>
__device__ __forceinline__ void tile_product(const GemmArgs& a, int m0, int n0, int kslice, int part, char* smem) {
  if constexpr (BN == 256) wide_product<BM, EPI, HD128, BUFFER>(a, m0, n0, kslice, part, smem);
  else ring_product<BM, BN, NWM, S, EPI, HD128, BUFFER>(a, m0, n0, kslice, part, smem);
}

// REST: the tiles cover the first columns only, in whole rounds of the 256 CUs; what is left, too little for another round,
// is cut into tiles of 128 rows and REST columns, which further workgroups of the same launch take as CUs come free.
template <int BM, int BN, int NWM, int S, int EPI, bool HD128, int REST, bool BUFFER>
__global__ void __launch_bounds__(NWM * BN) gemm_mfma_kernel(GemmArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  TileAt at;
  if constexpr (REST != 0) {
    const int block = (int)blockIdx.x - a.rest_block;
    if (block >= 0) {
      if (!tile_of(block, a.rest_m_tiles, a.rest_n_tiles, 1, at)) return;
      tile_product<128, REST, REST == 256 ? 2 : 4, REST == 256 ? 3 : 5, EPI, HD128, BUFFER>(a, at.m * 128, a.n_tiles * BN + at.n * REST,
                                                                                            0, a.n_tiles + at.n, smem);
      return;
    }
  }
  if (!tile_of(blockIdx.x, a.m_tiles, a.n_tiles, a.ksplit, at)) return;
  tile_product<BM, BN, NWM, S, EPI, HD128, BUFFER>(a, at.m * BM, at.n * BN, at.kslice, at.n, smem);
}

template <int BM, int BN, int NWM, int S, int EPI, bool HD128, int REST = 0, bool BUFFER = true>
static void launch_variant(const GemmArgs& a, hipStream_t s) {
  constexpr int smem = BN == 256 && BM > 128 ? 5 * 256 * 128 : S * (BM + BN) * 128;   // the rest's tiles take no more
  static bool configured = false;
  if (!configured) {
    (void)hipFuncSetAttribute((const void*)gemm_mfma_kernel<BM, BN, NWM, S, EPI, HD128, REST, BUFFER>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    configured = true;
  }
  const int grid = REST ? a.rest_block + tile_grid(a.rest_m_tiles * a.rest_n_tiles) : tile_grid(a.m_tiles * a.n_tiles * a.ksplit);
  gemm_mfma_kernel<BM, BN, NWM, S, EPI, HD128, REST, BUFFER><<<grid, NWM * BN, smem, s>>>(a);
}

// The tile shapes of the plan, and what one 64-deep k-step of a workgroup costs when a few CUs are busy and when all 256 are. The two
// wide ones are for products that fill the chip, where operand traffic counts (2048 x 37888 x 3584 to float: 469, 539, 635, 715 us in
// this order); the narrow ones put four to eight times as many workgroups on a short product and have more of its loads in flight
// (256 x 2048 x 1536: 32.1, 20.6, 12.4, 8.8 us). The last is for up to 32 rows (the positions of a generated block), where
// all that counts is how fast the weights stream: with K in slices and cold weights, 16 x 1536 x 8960 takes 7.9 us and 16 x 3584 x
// 18944 25.3, HBM's rate, where a kernel that loaded weights to registers and walked K wavefront by wavefront took 10.9 and 31.2.
// The costs (us) were those of earlier loops and weigh the tiles against each other: the present ones take 0.90 and 1.25, 0.56
// and 0.73, 0.31 and 0.42, 0.20 and 0.28 (192 x 256: 0.74 and 1.01, 64 x 64: 0.21 and 0.22, 32 x 64: 0.17 and 0.17). The slices of K,
// and with them the order of a product's sums, hang on this table.
struct TileShape { int bm, bn; double lat, full; };
static const TileShape kTiles[MFMA_TILES] = {{256, 256, 1.15, 1.7}, {128, 256, 0.68, 1.04}, {128, 128, 0.46, 0.65}, {64, 128, 0.33, 0.41}, {32, 128, 0.30, 0.36}};

// Tiles that only mfma_gemm_tile gives, behind those of the plan.
enum { TILE_64 = MFMA_TILES, TILE_32, TILE_192, TILE_SHORT /* 64 x 128, three K-tiles */, ALL_TILES };

int mfma_gemm_ring(int tile, int M, int N, int K, int ksplit);
int mfma_gemm_rest(int M, int N, int K, bool wide_only, int* n_tiles);
bool mfma_gate_up_192(int M, int N, int K, int tile);

// The launch of a product in tile `tile`. BUFFER: operands through buffer descriptors; without, tiles that are only
// refinements become the plan's.
template <int EPI, bool HD128, bool BUFFER>
static void launch_tile_of(GemmArgs& a, int tile, hipStream_t s) {
  a.part_tiles = mfma_lmhead_tiles(a.N);
  if constexpr (BUFFER) {
    if constexpr (EPI != ME_LMHEAD)
      if (tile == TILE_64 || tile == TILE_32) {
        a.m_tiles = tile == TILE_64 ? (a.M + 63) / 64 : (a.M + 31) / 32;
        a.n_tiles = (a.N + 63) / 64;
        if (tile == TILE_64) launch_variant<64, 64, 4, 4, EPI, HD128>(a, s);
        else launch_variant<32, 64, 2, 6, EPI, HD128>(a, s);
        return;
      }
    if (tile == TILE_192) {
      a.m_tiles = (a.M + 191) / 192;
      a.n_tiles = (a.N + 255) / 256;
      launch_variant<192, 256, 2, 5, EPI, HD128>(a, s);
      return;
    }
  } else {
    if (tile == TILE_64 || tile == TILE_32) tile = 3;
    if (tile == TILE_192) tile = 0;
  }
  if constexpr (EPI != ME_LMHEAD)
    if (tile == TILE_SHORT) {
      a.m_tiles = (a.M + 63) / 64;
      a.n_tiles = (a.N + 127) / 128;
      launch_variant<64, 128, 4, 3, EPI, HD128, 0, BUFFER>(a, s);
      return;
    }
  if constexpr (EPI == ME_SWIGLU)
    if (mfma_gate_up_192(a.M, a.N, a.K, tile)) {
      a.m_tiles = (a.M + 127) / 128;
      a.n_tiles = (a.N + 191) / 192;
      launch_variant<128, 192, 2, 4, EPI, HD128, 0, BUFFER>(a, s);
      return;
    }
  a.m_tiles = (a.M + kTiles[tile].bm - 1) / kTiles[tile].bm;
  a.n_tiles = (a.N + kTiles[tile].bn - 1) / kTiles[tile].bn;
  if (tile == 0) {
    const int rest = EPI == ME_RESIDUAL || a.ksplit > 1 ? 0 : mfma_gemm_rest(a.M, a.N, a.K, EPI == ME_LMHEAD, &a.n_tiles);
    if (rest) {
      a.rest_block = tile_grid(a.m_tiles * a.n_tiles);
      a.rest_m_tiles = (a.M + 127) / 128;
      a.rest_n_tiles = (a.N - 256 * a.n_tiles + rest - 1) / rest;
    }
    if constexpr (EPI != ME_RESIDUAL) {
      if (rest == 256) launch_variant<256, 256, 2, 5, EPI, HD128, 256, BUFFER>(a, s);
      if constexpr (EPI != ME_LMHEAD)
        if (rest == 128) launch_variant<256, 256, 2, 5, EPI, HD128, 128, BUFFER>(a, s);
    }
    if (!rest) launch_variant<256, 256, 2, 5, EPI, HD128, 0, BUFFER>(a, s);
  }
  else if (tile == 1) launch_variant<128, 256, 2, 3, EPI, HD128, 0, BUFFER>(a, s);
  else if constexpr (EPI != ME_LMHEAD) {
    // four wavefronts along M: two per SIMD cover each other's LDS reads (us, two along M / four: 1024 x 2048 x 1536 in 64 x 128
    // tiles 13.9 / 12.2, 1024 x 1536 x 1536 13.6 / 11.2, 256 x 2048 x 1024 9.8 / 8.3)
    if (tile == 2) launch_variant<128, 128, 4, 5, EPI, HD128, 0, BUFFER>(a, s);
    else if (mfma_gemm_ring(tile, a.M, a.N, a.K, a.ksplit) == 6) launch_variant<64, 128, 4, 6, EPI, HD128, 0, BUFFER>(a, s);
    else if (tile == 3) launch_variant<64, 128, 4, 3, EPI, HD128, 0, BUFFER>(a, s);
    else launch_variant<32, 128, 2, 4, EPI, HD128, 0, BUFFER>(a, s);
  }
}
