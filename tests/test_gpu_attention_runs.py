"""Block attention whose list of key tiles is cut into runs that a second kernel adds, launched with the scratch that a scoring
pass has, against the oracle; and what such a launch must not depend on."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import workload as W
from host_rules import BatchGeom, ModelDims, library

pytestmark = pytest.mark.gpu
DEV, PAGE = "cuda:0", 16


class Operands:
    """Random queries, block keys and values and a paged prefix of one layer, host and device copies."""

    def __init__(self, Hq, Hkv, hd, B, n, L, lens):
        self.Hq, self.Hkv, self.hd, self.B, self.n, self.L, self.lens = Hq, Hkv, hd, B, n, L, lens
        draw = lambda name, *shape: W.rng.normal_tensor(7, name, shape, 1.0, "bf16")
        need = [-(-P // PAGE) for P in lens]
        perm, o = W.rng.permutation(5, "pg", sum(need)), 0
        self.table = np.full((B, max(need)), -1, np.int32)
        for b, k in enumerate(need):
            self.table[b, :k] = perm[o:o + k]
            o += k
        self.q, self.k, self.v = draw("rq", B * n * L, Hq, hd), draw("rk", B * n * L, Hkv, hd), draw("rv", B * n * L, Hkv, hd)
        self.pool = draw("rp", 2, sum(need), Hkv, PAGE, hd)
        self.scale_ends()
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV).to(torch.bfloat16)
        Lp = -(-L // 16) * 16
        vT = np.zeros((B * n, Hkv, hd, Lp), np.float32)
        vT[..., :L] = self.v.reshape(B * n, L, Hkv, hd).transpose(0, 2, 3, 1)
        self.dev = [dev(self.q), dev(self.k), dev(vT), dev(self.pool[0]), dev(self.pool[1].swapaxes(-1, -2))]
        self.lens_dev, self.table_dev = torch.tensor(lens, dtype=torch.int32, device=DEV), torch.from_numpy(self.table).to(DEV)

    def scale_ends(self):
        """Values 16 times as large at the ends of the list and of its first tiles: a key lost, or counted twice, among some thousand
        moves an output by 16 |v| / keys, well beyond the bound below."""
        for b, P in enumerate(self.lens):
            for j in {0, 63, 64, 65, 127, P - 65, P - 64, P - 2, P - 1}:
                if 0 <= j < P:
                    self.pool[1, self.table[b, j // PAGE], :, j % PAGE] *= 16

    def launch(self, scratch_floats=0, n=None):
        """The first n candidates of every beam; the output, and whether the launch used its scratch."""
        n, L = n or self.n, self.L
        part = torch.full((max(scratch_floats, 1),), float("nan"), device=DEV)
        pick = lambda t, rows: t.view(self.B, self.n, rows, *t.shape[1:])[:, :n].reshape(-1, *t.shape[1:]).contiguous()
        q, k, vT = pick(self.dev[0], L), pick(self.dev[1], L), pick(self.dev[2], 1)
        out = torch.full((self.B * n * L, self.Hq * self.hd), float("nan"), dtype=torch.bfloat16, device=DEV)
        Lp = vT.shape[-1]
        g = BatchGeom(B=self.B, n=n, L=L, M=self.B * n * L, len_override=-1, Lk=L, vs=Lp, lens=self.lens_dev.data_ptr(),
                      page_table=self.table_dev.data_ptr(), max_pages=self.table.shape[1], page_tokens=PAGE)
        md = ModelDims(d=self.Hq * self.hd, Hq=self.Hq, Hkv=self.Hkv, hd=self.hd)
        f = library()._Z21launch_attention_mfmaPKDF16bS0_S0_S0_S0_PDF16bRK9BatchGeomRK9ModelDimsiiPfmRK12WeightsAheadP12ihipStream_t
        p = C.c_void_p
        f.restype = C.c_bool
        f.argtypes = [p] * 6 + [C.POINTER(BatchGeom), C.POINTER(ModelDims), C.c_int, C.c_int, p, C.c_size_t, p, p]
        nothing_ahead = (C.c_char * 64)()
        assert f(*(t.data_ptr() for t in (q, k, vT, *self.dev[3:], out)), g, md, Lp, max(self.lens),
                 part.data_ptr() if scratch_floats else None, scratch_floats, nothing_ahead, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        return out.view(self.B, n, L, self.Hq * self.hd), not bool(torch.isnan(part).all())

    def beyond_the_bound(self, out, candidates):
        """Largest error of these candidates as a multiple of what rounding allows: half a unit in the last place of the result
        (2^-8 of it at most), and where the score's own rounding takes a weight over the edge between two bf16 values, 2^-8 of
        that weight's term; four such weights, the largest of the row. 1e-5 for float sums of terms that cancel."""
        worst = 0.0
        for b, i in candidates:
            P, r = self.lens[b], (b * self.n + i) * self.L
            at = np.arange(P)
            pk, pv = (self.pool[o][self.table[b, at // PAGE], :, at % PAGE] for o in (0, 1))
            k, v = np.concatenate([pk, self.k[r:r + self.L]]).astype(float), np.concatenate([pv, self.v[r:r + self.L]]).astype(float)
            q = self.q[r:r + self.L].astype(float)
            mask = np.concatenate([np.ones((self.L, P), bool), np.tril(np.ones((self.L, self.L), bool))], 1)
            want = oracle.attention(q, k, v, mask, "bf16")
            got = out[b, i].float().cpu().numpy().astype(float)
            for h in range(self.Hq):
                cols = slice(h * self.hd, (h + 1) * self.hd)
                kv = h * self.Hkv // self.Hq
                s = np.where(mask, q[:, h] @ k[:, kv].T / np.sqrt(self.hd), -np.inf)
                w = np.exp(s - s.max(1, keepdims=True))
                term = (w / w.sum(1, keepdims=True) * np.abs(v[:, kv]).max(1)).max(1, keepdims=True)
                bound = 2.0 ** -8 * np.abs(want[:, cols]) + 4 * 2.0 ** -8 * term + 1e-5
                worst = max(worst, (np.abs(got[:, cols] - want[:, cols]) / bound).max())
        return worst


# one workgroup of 128 rows per 128 stacked rows of a (beam, kv head, candidate), lists of at least 16 tiles, fewer than 384 workgroups
@pytest.mark.parametrize("Hq,Hkv,hd,B,n,L,lens,cut", [
    (2, 2, 128, 1, 2, 32, [1500], True),          # 32 rows: wavefronts of 16, 25 key tiles in 6 runs
    (3, 1, 64, 2, 2, 7, [2000, 1025], True),      # 21 rows; the runs of the shorter beam hold half as much
    (1, 1, 64, 1, 3, 64, [961], True),            # 64 rows; 17 tiles, 4 runs
    (6, 2, 128, 2, 2, 33, [1, 2900], True),       # 99 rows: wavefronts of 32; runs without a key of the short beam
    (5, 1, 64, 1, 2, 13, [3009], True),           # 65 rows, one beyond a workgroup of 64
    (2, 2, 64, 1, 4, 63, [897], True),            # 63 rows, lists of 15 + 1 tiles: the shortest that is cut
    (2, 2, 64, 1, 4, 63, [895], False),           # one tile fewer
    (1, 1, 128, 2, 30, 70, [2048, 1100], True)])  # blocks of two tiles, 70 rows
def test_runs_against_the_oracle(Hq, Hkv, hd, B, n, L, lens, cut):
    x = Operands(Hq, Hkv, hd, B, n, L, lens)
    some = sorted({(b, i) for b in range(B) for i in (0, n // 2, n - 1)})
    out, used = x.launch(64 << 20)
    assert used == cut
    assert x.beyond_the_bound(out, some) <= 1
    out, used = x.launch()                        # without scratch: one workgroup walks the whole list
    assert not used and x.beyond_the_bound(out, some) <= 1


@pytest.mark.parametrize("hd", [64, 128])
def test_a_candidate_keeps_its_bits_with_more_beside_it(hd):
    """16, 32 and 48 candidates of 80 stacked rows and 2 kv heads, 1500 keys: their lists are cut into 6, 6 and 5 runs, so the
    first two give a candidate the same sums in the same order."""
    x = Operands(4, 2, hd, 1, 48, 40, [1500])
    few, used = x.launch(64 << 20, 16)
    more, also = x.launch(64 << 20, 32)
    assert used and also and torch.equal(few, more[:, :16])
    assert x.beyond_the_bound(x.launch(64 << 20)[0], [(0, 0), (0, 47)]) <= 1
