"""Every tile shape of the bf16 product family, launched by its index on whole-number operands: the sums are exact in float,
so each element has to be equal, whatever the tile, the K-tiles against the length of its LDS ring, the K slices and the
remainders of the last tiles. Only the plan's choice of a tile is left to the other tests."""
import ctypes as C

import pytest
import torch

from host_rules import BatchGeom, ModelDims, library

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
WIDE, TILES = (0, 1, 7), (0, 1, 2, 3, 4, 5, 6, 7, 8)   # those of the plan, 64 x 64, 32 x 64, 192 x 256, 64 x 128 with 3 K-tiles
STORE, RESIDUAL, SWIGLU, HEAD = 0, 1, 2, 3


def launch(epilogue, A, Wt, M, N, K, out=None, act=None, tok=None, pm=None, ps=None, zt=None, split=1, tile=-1):
    f = library()._Z16launch_gemm_mfmaiPKDF16bS0_iiiPfPDF16bPKiS1_S1_S1_iiP12ihipStream_t
    p = C.c_void_p
    f.restype, f.argtypes = C.c_bool, [C.c_int, p, p] + [C.c_int] * 3 + [p] * 6 + [C.c_int] * 2 + [p]
    ptr = lambda t: None if t is None else t.data_ptr()
    return f(epilogue, A.data_ptr(), Wt.data_ptr(), M, N, K, ptr(out), ptr(act), ptr(tok), ptr(pm), ptr(ps), ptr(zt), split, tile,
             torch.cuda.current_stream().cuda_stream)


def whole(shape, seed, top=3):
    g = torch.Generator().manual_seed(seed)
    return torch.randint(-top, top + 1, shape, generator=g).to(torch.bfloat16).to(DEV)


# K-tiles: fewer than any ring holds, one more than a turn of the unrolled loops (5 and 3 K-tiles), several turns; beyond 11 the
# 64 x 128 tile has its longer ring
@pytest.mark.parametrize("k_tiles", [1, 2, 3, 4, 5, 6, 7, 11, 13])
@pytest.mark.parametrize("tile", TILES)
def test_store_and_residual_are_exact(tile, k_tiles):
    K = 64 * k_tiles
    for M, N in ((300, 520), (1, 64), (257, 259)):       # remainders of rows and columns; a row length of no whole 16 bytes
        if tile == 4 and M > 32:
            M = 31                                       # the tile for up to 32 rows
        A, Wt = whole((M, K), 1), whole((N, K), 2)
        want = A.float() @ Wt.float().t()                # exact: sums of at most 832 products of at most 9
        for split in (1, 2, 3):
            if split > k_tiles:
                break
            out = torch.full((split, M, N), float("nan"), device=DEV)
            assert launch(STORE, A, Wt, M, N, K, out, split=split, tile=tile)
            assert torch.equal(out.sum(0), want), (M, N, split)
        assert launch(RESIDUAL, A, Wt, M, N, K, out := want.clone(), tile=tile)
        assert torch.equal(out, 2 * want), (M, N)


@pytest.mark.parametrize("k_tiles", [1, 4, 6])
@pytest.mark.parametrize("tile", WIDE)
def test_vocabulary_head_finds_targets_and_maxima(tile, k_tiles):
    M, N, K = 261, 1000, 64 * k_tiles
    A, Wt = whole((M, K), 3), whole((N, K), 4)
    check_head(A, Wt, A.float() @ Wt.float().t(), tile)


def check_head(A, Wt, z, tile):
    (M, K), N = A.shape, len(Wt)
    tok = torch.randint(0, N, (M,), generator=torch.Generator().manual_seed(5), dtype=torch.int32).to(DEV)
    tiles = -(-N // 256)
    pm, ps = torch.full((2, M, tiles), float("nan"), device=DEV)
    zt = torch.full((M,), float("nan"), device=DEV)
    assert launch(HEAD, A, Wt, M, N, K, tok=tok, pm=pm, ps=ps, zt=zt, tile=tile)
    assert torch.equal(zt, z.gather(1, tok.long()[:, None])[:, 0])
    pad = torch.nn.functional.pad(z, (0, tiles * 256 - N), value=float("-inf")).view(M, tiles, 256)
    assert torch.equal(pm, pad.max(2).values)
    want = (pad.double() - pm.double()[:, :, None]).exp().sum(2)
    # 256 positive terms with 2 ulp each of v_exp_f32, on arguments rounded to float by __expf's product with log2(e)
    assert torch.allclose(ps.double(), want, rtol=256 * 2.0 ** -24, atol=0)


@pytest.mark.parametrize("tile", TILES)
def test_gate_up_columns_meet_their_partners(tile):
    """Gate g and up u of every unit whole numbers: the product is bf16(silu(g) u) up to the rounding of silu."""
    M, F, K = 30 if tile == 4 else 290, 480, 128
    A, Wt = whole((M, K), 6, 1), whole((2 * F, K), 7, 1)
    z = (A.double() @ Wt.double().t()).view(M, F // 32, 2, 32)
    act = torch.full((M, F), float("nan"), dtype=torch.bfloat16, device=DEV)
    assert launch(SWIGLU, A, Wt, M, 2 * F, K, act=act, tile=tile)
    want = (torch.nn.functional.silu(z[:, :, 0]) * z[:, :, 1]).reshape(M, F)
    # half a unit in the last of 8 significant bits is 2^-8 at most; __expf rounds an argument of at most 64 times log2(e) to
    # float, half a unit in the last place of 2^6, and its result, sum, reciprocal and products take a unit each
    assert torch.all((act.double() - want).abs() <= want.abs() * (2.0 ** -8 + 2.0 ** -17 + 8 * 2.0 ** -23) + 1e-30)


def off_the_grid(x):
    """The same values 4 bytes beside the 16-byte grid."""
    return torch.zeros(x.numel() + 2, dtype=x.dtype, device=DEV)[2:].view(x.shape).copy_(x)


@pytest.mark.parametrize("k_tiles", [1, 5, 7])
@pytest.mark.parametrize("epilogue", [STORE, RESIDUAL, SWIGLU, HEAD])
def test_operands_off_the_16_byte_grid(epilogue, k_tiles):
    """The kernels that take plain addresses."""
    M, N, K = 300, 576, 64 * k_tiles
    A, Wt = off_the_grid(whole((M, K), 8, 1)), off_the_grid(whole((N, K), 9, 1))
    z = A.float() @ Wt.float().t()
    for tile in (-1, *(WIDE if epilogue == HEAD else TILES)):
        if epilogue == STORE:
            for split in (1, 2)[:k_tiles]:
                out = torch.full((split, M, N), float("nan"), device=DEV)
                assert launch(STORE, A, Wt, M, N, K, out, split=split, tile=tile)
                assert torch.equal(out.sum(0), z), (tile, split)
        elif epilogue == RESIDUAL:
            assert launch(RESIDUAL, A, Wt, M, N, K, out := z.clone(), tile=tile)
            assert torch.equal(out, 2 * z), tile
        elif epilogue == SWIGLU:
            act = torch.full((M, N // 2), float("nan"), dtype=torch.bfloat16, device=DEV)
            assert launch(SWIGLU, A, Wt, M, N, K, act=act, tile=tile)
            y = z.double().view(M, N // 64, 2, 32)
            ref = (torch.nn.functional.silu(y[:, :, 0]) * y[:, :, 1]).reshape(M, N // 2)
            assert torch.allclose(act.double(), ref, rtol=2.0 ** -8 + 2.0 ** -16, atol=1e-30), tile
        else:
            check_head(A, Wt, z, tile)


@pytest.mark.parametrize("on_grid", [True, False])
@pytest.mark.parametrize("position", [None, 0, 9, 20])   # whole blocks of 21 tokens, or one token of each
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("tile", TILES)
def test_queries_keys_and_values_land_where_they_belong(tile, hd, position, on_grid):
    """Rotations by multiples of a quarter turn: every output is a whole number that bf16 holds."""
    Hq, Hkv, Lk, C_, K, Lp = 5, 2, 21, 1 if tile == 4 else 14 if position is None else 70, 64, 32
    L = Lk if position is None else 1
    M = C_ * L
    A, Wt = whole((M, K), 10, 1), whole(((Hq + 2 * Hkv) * hd, K), 11, 1)
    if not on_grid:
        A, Wt = off_the_grid(A), off_the_grid(Wt)
    turn = torch.randint(0, 4, (M, hd // 2), generator=torch.Generator().manual_seed(12)).to(DEV)
    c, s = torch.tensor([1.0, 0, -1, 0], device=DEV)[turn], torch.tensor([0, 1.0, 0, -1], device=DEV)[turn]
    cs = torch.cat([c, s], 1).contiguous()
    new = lambda *shape: torch.full(shape, float("nan"), dtype=torch.bfloat16, device=DEV)
    q, k, v = new(M, Hq, hd), new(C_, Lk, Hkv, hd), new(C_, Hkv, hd, Lp)
    f = library()._Z25launch_gemm_mfma_qkv_ropePKDF16bS0_PKfPDF16bS3_S3_RK9BatchGeomRK9ModelDimsiiP12ihipStream_t
    p = C.c_void_p
    f.restype, f.argtypes = C.c_bool, [p] * 6 + [C.POINTER(BatchGeom), C.POINTER(ModelDims), C.c_int, C.c_int, p]
    g = BatchGeom(B=1, n=C_, L=L, M=M, t0=position or 0, Lk=Lk, vs=Lp)
    md = ModelDims(d=K, Hq=Hq, Hkv=Hkv, hd=hd)
    assert f(*(t.data_ptr() for t in (A, Wt, cs, q, k, v)), g, md, Lp, tile, torch.cuda.current_stream().cuda_stream)
    y = (A.float() @ Wt.float().t()).view(M, Hq + 2 * Hkv, hd)
    x1, x2 = y[:, :Hq + Hkv, :hd // 2], y[:, :Hq + Hkv, hd // 2:]
    rot = torch.cat([x1 * c[:, None] - x2 * s[:, None], x2 * c[:, None] + x1 * s[:, None]], 2)
    assert torch.equal(q.float(), rot[:, :Hq])
    at = slice(0, Lk) if position is None else slice(position, position + 1)
    want_k, want_v = torch.full_like(k, float("nan")).float(), torch.full_like(v, float("nan")).float()
    want_k[:, at] = rot[:, Hq:].view(C_, L, Hkv, hd)
    want_v[..., at] = y[:, Hq + Hkv:].view(C_, L, Hkv, hd).permute(0, 2, 3, 1)
    if at.stop == Lk:                                    # with the last token, what pads a row of values
        want_v[..., Lk:] = 0
    for got, want in ((k, want_k), (v, want_v)):         # nothing else is written
        assert torch.equal(torch.nan_to_num(got.float(), nan=1e9), torch.nan_to_num(want, nan=1e9))
