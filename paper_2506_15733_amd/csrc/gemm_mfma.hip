// Which tile a product of the bf16 MFMA family gets, how its K and its last columns are cut, and the launches
// (kernels: gemm_mfma.h).
#include "gemm_mfma.h"

int mfma_lmhead_tiles(int V) { return (V + 255) / 256; }

// K-tiles in the LDS ring of the kernel that takes a product. 64 x 128: six, in one workgroup per CU, where few
// workgroups walk a long K; else half of that and two workgroups per CU, which fill it sooner and leave no nearly empty
// last round (16 x 37888 x 3584, 296 workgroups: 62.2 -> 60.3 us).
int mfma_gemm_ring(int tile, int M, int N, int K, int ksplit) {
  const TileShape& ts = kTiles[tile];
  const long wgs = (long)((M + ts.bm - 1) / ts.bm) * ((N + ts.bn - 1) / ts.bn) * ksplit;
  static const int ring[MFMA_TILES] = {5, 3, 5, 3, 4};
  return tile == 3 && wgs <= 256 && K / 64 > 11 * ksplit ? 6 : ring[tile];
}

// Operands are requested in 16-byte pieces through descriptors of at most 256 rows, whose offsets have 32 bits. Any others get
// the plan's tile by plain addresses (us, weights 4 bytes beside the grid / on it: head of 2048 x 152064 x 3584 1729 / 1559, gate/up of
// 2048 x 37888 x 3584 446 / 402, 256 x 1536 x 8960 20.2 / 17.1; all in 128 x 128 tiles 713 for the second and 23.7 for the third).
// Their kernels are compiled in a file of their own: in the code object of the others, which they do not change by an
// instruction, they spread these so far apart that a pass of many short launches took 1.1 % longer (555 rows of d = 1024).
void launch_tile_off_grid(int epi, bool hd128, GemmArgs& a, int tile, hipStream_t s);
static bool buffer_operands(const GemmArgs& a) { return (((uintptr_t)a.A | (uintptr_t)a.W) & 15) == 0 && a.K <= 1 << 22; }

template <int EPI, bool HD128 = false>
static void launch_tile(GemmArgs& a, int tile, hipStream_t s) {
  if (buffer_operands(a)) launch_tile_of<EPI, HD128, true>(a, tile, s);
  else launch_tile_off_grid(EPI, HD128, a, tile, s);
}

// Gate and up in 128 x 192 tiles where the plan says 128 x 256 and a single round does: a few hundred rows then occupy a third
// more CUs, each with 120 KB of operands in flight instead of 96, which is what bounds such a product while its weights come
// from HBM. us with cold weights, in 128 x 256 tiles / so: 256 x 17920 x 1536 30.0 / 26.0, 200 rows 27.7 / 23.8, 100 x 37888 x 3584
// 64.9 / 55.4, 512 x 9728 x 896 17.8 / 15.4; in two rounds it is behind (321 x 17920 x 1536, with the loops of then: 27.7 / 44.3).
// K-tiles for less than two fills of the ring leave nothing in flight to gain. Up to 128 rows, where the weights are read once,
// also in place of 64 x 128 tiles that put two workgroups on some CUs (48 x 37888 x 3584: 66.3 / 50.4).
bool mfma_gate_up_192(int M, int N, int K, int tile) {
  const bool two_narrow = tile == 3 && M > 32 && M <= 128 && (long)((M + 63) / 64) * ((N + 127) / 128) > 256;
  return (tile == 1 || two_narrow) && (long)((M + 127) / 128) * ((N + 191) / 192) <= 256 && K > 512;
}

// Time that wgs workgroups of a tile shape take for a k-step each: in rounds of 256; a round that leaves CUs idle has k-steps
// between the two costs of its tile. The narrow tiles run two workgroups per CU: their last round overlaps the one before, but
// a few more than 256 cost what 512 do, twice one workgroup on a CU (64 x 128: 0.28 us a step at 256 workgroups, 0.52 at 264 and
// 352, 0.56 at 484, 0.82 at 660, 1.45 at 1260; not where 32 rows fill half of the tile and weights are all that streams: 0.96 at
// 296, HBM's rate, for 16 x 37888 x 3584).
static double rounds(int tile, long wgs, int M) {
  const TileShape& ts = kTiles[tile];
  const long whole = tile < 3 || wgs <= 256 ? wgs / 256 : 0, rest = wgs - 256 * whole;
  if (rest > 256) {
    const double per_cu = rest / 256.0, two = rest <= 512 ? 2.2 * ts.lat : 2.0 * ts.lat + 0.34 * (per_cu - 1.0);
    return tile == 3 && M > 32 && two > ts.full * per_cu ? two : ts.full * per_cu;
  }
  return whole * ts.full + (rest ? ts.lat + (ts.full - ts.lat) * rest / 256.0 : 0.0);
}

// Products of more than a round of 256 x 256 tiles: the columns (in tiles, *n_tiles) that fill whole rounds, and the width of
// the 128-row tiles that the rest is cut into, 0 where another round of the large ones takes no longer. *cost: time of a
// k-step over all rounds. A last round of few tiles leaves most CUs idle for as long as a full one (us without a rest / with):
// gate/up of 1024 x 17920 x 1536, 280 tiles, 66 / 50; 2048 rows, 560 tiles, 107 / 96; of 4493 x 37888 x 3584, 2664 tiles, 862 / 847;
// head of 256 x 151936 x 1536, 594 tiles, 138 / 130. About 3 us go to the epilogue and the first loads of the rest.
// The 128-column tiles are for a rest of an eighth of a round at most: they occupy the CUs for half as long again as the 256-column
// ones, which other streams miss (with the loops of then: step of 2184 rows of 7B models, 62 ms, a rest of 52 tiles: 0.9 % longer than without a rest so,
// 0.3 % with the wide ones). For the same reason none from three whole rounds on where half a round or more is left: alone,
// such a rest gains 2 to 5 % of a launch (also then: 16384 x 4608 x 3584 485 / 470 us, 3584 columns 372 / 348), but less than half of the CUs
// would have idled, and a step of 16384 rows on three streams is shorter without (492.3 / 494.5 ms).
static int rest_plan(int M, int N, int K, bool wide_only, int* n_tiles, double* cost) {
  const int m_tiles = (M + 255) / 256, all = (N + 255) / 256;
  const long whole = (long)m_tiles * all / 256;
  *n_tiles = all;
  *cost = rounds(0, (long)m_tiles * all, M);
  const int nb = (int)(256 * whole / m_tiles);
  if (nb == 0 || nb >= all || (whole > 2 && (long)m_tiles * all - 256 * whole >= 128)) return 0;
  int width = 0;
  const bool narrow = !wide_only && (long)m_tiles * (all - nb) <= 32;
  for (int tile = 1; tile <= (narrow ? 2 : 1); ++tile) {
    const int bn = kTiles[tile].bn;
    const double c = whole * kTiles[0].full + rounds(tile, (long)((M + 127) / 128) * ((N - 256 * nb + bn - 1) / bn), M) + 3.0 * 64 / K;
    if (c < *cost) { *cost = c; *n_tiles = nb; width = bn; }
  }
  return width;
}
int mfma_gemm_rest(int M, int N, int K, bool wide_only, int* n_tiles) {
  double cost;
  return rest_plan(M, N, K, wide_only, n_tiles, &cost);
}

// Tile shape and K-split for an M x N x K product whose consumer can sum up to max_split partial products: the pair
// with the least estimated time. The weights cannot arrive faster than HBM delivers them, and about half of that time does
// not overlap with a short walk through K. A launch costs about 3 us beside that, and every extra partial one more M x N float
// write here and one more read in the consumer. Of 64 products without slices (the projections of
// K = 896 to 18944, 34 to 3490 rows, cold weights) 58 get the fastest of the tiles with what mfma_gemm_tile makes of it, the others lose 0.3
// to 10 %.
// A rest competes with the other unsliced tiles only: slices fill their rounds as well as a rest does (product and the
// addition behind it, us with slices / with a rest, with the loops of then: 16384 x 3584 x 18944 1874 / 1870, 4700 rows 653 / 654, 16384 x 1536 x 8960
// 447 / 439), and the order of a product's sums then does not hang on how its last round is cut.
void mfma_gemm_plan(int M, int N, int K, int max_split, bool wide_only, int* tile_out, int* split_out) {
  const int KT = K / 64, shapes = wide_only ? 2 : M <= 32 ? MFMA_TILES : MFMA_TILES - 1;
  const double stream = (double)N * K * 2.0 / 5.2e6;
  double best = 1e30;
  *tile_out = 0; *split_out = 1;
  auto consider = [&](int tile, int sp, double step) {
    const double walk = step * ((KT + sp - 1) / sp) + 0.45 * stream;
    const double t = 3.0 + (walk > stream ? walk : stream) + (2 * sp - 2) * (double)M * N * 4.0 / 4e6;
    if (t < best - 1e-9) { best = t; *tile_out = tile; *split_out = sp; }
  };
  for (int tile = 0; tile < shapes; ++tile) {
    const TileShape& ts = kTiles[tile];
    const long tiles = (long)((M + ts.bm - 1) / ts.bm) * ((N + ts.bn - 1) / ts.bn);
    for (int sp = 1; sp <= max_split && sp <= MFMA_MAX_SPLIT && (sp == 1 || sp * 4 <= KT + 3); ++sp)
      consider(tile, sp, rounds(tile, tiles * sp, M));
  }
  double step;
  int n_tiles;
  if (*split_out == 1 && rest_plan(M, N, K, wide_only, &n_tiles, &step)) consider(0, 1, step);
}

// The plan's tile and slices, or a tile that it does not know with the same slices: all tiles add a slice's products in the same
// order, so these leave the same bits.
// 192 x 256 for 256 x 256 and 128 x 256 where the rounds they take are shorter: fewer rows that only pad, or a single round with more
// CUs in it (us, 256 x 256 / 192 x 256: 1100 x 3584 x 18944 in 3 slices 130 / 119, 1600 rows in 2 186 / 165, gate/up of 1100 x 9728 x
// 896 24.4 / 22.1, head of 555 x 151936 x 1536 270 / 250; but 1600 x 17920 x 1536, 490 / 630 tiles, 78 / 94, 1600 x 37888 x 3584 330 /
// 373, and 1100 x 17920 x 1536, where a rest makes up for the padding, 62.7 / 64.8; against 128 x 256: gate/up of 555 x 37888 x 3584
// 154 / 135, but 1600 x 4608 x 3584 51.8 / 58.5, 1100 rows 52.7 / 62.9). A k-step takes 0.85 of the larger tile's.
// Finer ones where the plan says 64 x 128 and the product leaves CUs without a workgroup of that: what such a launch takes is how
// long its few CUs pull weights from HBM, so more and smaller workgroups are ahead as long as each has a CU to itself. us with cold
// weights, of 64 x 128, 64 x 64 and 32 x 64: 256 x 2048 x 1024 10.3, 7.7, 6.7; 256 x 2048 x 1536 14.8, 10.3, 8.6; 256 x 1024 x 1024 in 4
// slices 6.1, 4.9, 5.4 (512 workgroups of the last, in 2: 5.2). A few CUs with two of the 64 x 64 ones do no harm while the weights are
// few, up to 3.1 M of them (264 to 288 workgroups: 513, 555 and 576 x 2048 x 1536 12.5, 14.4, 14.7 / 12.0, 12.4, 12.5; 650, 704 and 768 x
// 1536 x 1536 13.0, 14.5, 14.5 / 12.4, 12.6, 12.8; 900, 960 and 1024 x 1152 x 896 9.1, 9.8, 9.8 / 8.8, 8.9, 8.9; 1100 and 1152 x 1024 x
// 1024 9.6, 10.2 / 9.1, 9.2; from 3.7 M on they do: 320 x 3584 x 1024 10.9 / 11.3, 256 x 4608 x 896 10.4 / 11.3, 256 x 4608 x 3584 28.1 /
// 32.4, gate/up of 64 x 17920 x 1536 18.3 / 20.1); where many have two, 64 x 128 is ahead (256 x 5632 x 1024: 352, 11.2 / 12.3; 1024 x 2048 x 1536: 512, 14.6 / 16.1).
// beside: the caller said that other launches run beside this one (the models of a step score their blocks at the same time). The
// longer ring of the 64 x 128 tiles takes a CU's LDS to itself, so of two such launches, of 129 to 256 workgroups each, one waits for
// CUs of the other. The short one leaves room for a second workgroup; alone it costs 4 to 7 % of a launch up to 24
// K-tiles, and 7 to 10 % beyond (us, 256 x 5632 x 1024 7.9 / 8.5, 1024 x 2048 x 1536 12.2 / 12.7, 256 x 1536 x 8960 in 5 slices 12.4 /
// 13.3, 256 x 4608 x 3584 18.6 / 20.7). A step of three models of 4 and 16 layers of d = 1024 1260 us with the long ring, 1210 so;
// one of them alone 795 us with the long ring, 805 so.
void mfma_gemm_tile(int M, int N, int K, int max_split, bool wide_only, bool beside, int* tile_out, int* split_out) {
  mfma_gemm_plan(M, N, K, max_split, wide_only, tile_out, split_out);
  if (*tile_out <= 1) {
    const long columns = (long)((N + 255) / 256) * *split_out;
    int n_tiles;
    double large = rounds(*tile_out, (M + kTiles[*tile_out].bm - 1) / kTiles[*tile_out].bm * columns, M), with_rest;
    if (*tile_out == 0 && *split_out == 1 && rest_plan(M, N, K, wide_only, &n_tiles, &with_rest)) large = with_rest;
    if (0.85 * rounds(0, (M + 191) / 192 * columns, M) < 0.97 * large) *tile_out = TILE_192;
  } else if (*tile_out == 3) {
    const long columns = (long)((N + 63) / 64) * *split_out;
    if ((M + 31) / 32 * columns <= 256) *tile_out = TILE_32;
    else if ((M + 63) / 64 * columns <= ((long)N * K <= 13 << 18 ? 288 : 256)) *tile_out = TILE_64;
    else if (beside && mfma_gemm_ring(3, M, N, K, *split_out) == 6 && K / 64 <= 24 * *split_out) *tile_out = TILE_SHORT;
  }
}

// QKV projection with the rotary embedding, the bf16 conversion and the per-candidate transposition of the values
// in the epilogue: no float [M, (Hq+2Hkv)*hd] round trip through memory and no separate kernel. Row m is in-block
// position g.t0 + m % g.L of candidate m / g.L. Returns false when the shape is not taken (head_dim other than 64/128,
// K % 64 != 0, misaligned buffers, parts of blocks other than single positions); the caller then runs the projection and
// the rotary kernel separately.
bool launch_gemm_mfma_qkv_rope(const bf16_t* A, const bf16_t* W, const float* cs, bf16_t* q, bf16_t* kblk, bf16_t* vT,
                               const BatchGeom& g, const ModelDims& md, int Lp, int tile, hipStream_t s) {
  const int M = g.M, N = (md.Hq + 2 * md.Hkv) * md.hd, K = md.d;
  if (K % 64 != 0 || M <= 0 || (md.hd != 64 && md.hd != 128) || (g.L != 1 && (g.t0 != 0 || g.Lk != g.L))) return false;
  if (((uintptr_t)cs & 15) || ((uintptr_t)q & 7) || ((uintptr_t)kblk & 7)) return false;
  GemmArgs a = {};
  a.A = A; a.W = W; a.M = M; a.N = N; a.K = K; a.ksplit = 1;
  a.cs = cs; a.q = q; a.kblk = kblk; a.vT = vT;
  a.Hq = md.Hq; a.Hkv = md.Hkv; a.Lrows = g.L; a.Lk = g.Lk; a.Lp = Lp; a.t0 = g.t0;
  int split = 1;
  if (tile < 0) mfma_gemm_tile(M, N, K, 1, false, false, &tile, &split);
  if (md.hd == 128) launch_tile<ME_QKV_ROPE, true>(a, tile, s);
  else launch_tile<ME_QKV_ROPE, false>(a, tile, s);
  return true;
}

// Whether single positions of more rows than the kernels for few rows take have their rotary embedding in the epilogue. The
// projection can then not be cut into slices of K (up to max_split), so where the plan wants some, only if the whole walk is short or
// every CU's share of it small. Against slices and the rotary kernel's 6 us (us, cold weights): 256 x 2048 x 1536 8.2 + 6.2 / 8.8;
// 48 x 4608 x 3584 11 + 6 / 15, but 128 rows 12.4 + 6 / 20.
bool qkv_rope_position(int M, int N, int K, int max_split) {
  int tile, split;
  mfma_gemm_tile(M, N, K, max_split, false, false, &tile, &split);
  if (split == 1 || K <= 2048) return true;
  mfma_gemm_tile(M, N, K, 1, false, false, &tile, &split);
  return tile == TILE_32;
}

// Returns false when the shape is not one this kernel takes (the caller then uses the SIMT kernel).
// ksplit > 1 (ME_STORE only): C is [ksplit][M][N] and receives the partial products of the K slices.
// tile: index of the tile shape as mfma_gemm_plan gives it, negative = chosen here.
bool launch_gemm_mfma(int epi, const bf16_t* A, const bf16_t* W, int M, int N, int K, float* C, bf16_t* act,
                      const int32_t* tok, float* part_max, float* part_sum, float* zt, int ksplit, int tile,
                      hipStream_t s) {
  if (K % 64 != 0 || M <= 0 || N <= 0) return false;
  if (epi == ME_SWIGLU && (N % 64 != 0 || ((uintptr_t)act & 7))) return false;
  if (ksplit < 1 || (ksplit > 1 && (epi != ME_STORE || ksplit > K / 64))) return false;
  if (tile >= ALL_TILES || (epi == ME_LMHEAD && tile >= 2 && tile != TILE_192)) return false;
  GemmArgs a = {};
  a.A = A; a.W = W; a.M = M; a.N = N; a.K = K; a.C = C; a.act = act; a.tok = tok;
  a.part_max = part_max; a.part_sum = part_sum; a.zt = zt; a.ksplit = ksplit;
  int split = 1;
  if (tile < 0) mfma_gemm_tile(M, N, K, 1, epi == ME_LMHEAD, false, &tile, &split);
  switch (epi) {
    case ME_STORE: launch_tile<ME_STORE>(a, tile, s); break;
    case ME_RESIDUAL: launch_tile<ME_RESIDUAL>(a, tile, s); break;
    case ME_SWIGLU: launch_tile<ME_SWIGLU>(a, tile, s); break;
    case ME_LMHEAD: launch_tile<ME_LMHEAD>(a, tile, s); break;
    default: return false;
  }
  return true;
}
