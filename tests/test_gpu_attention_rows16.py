"""Attention launches whose wavefronts take 16 query rows, and the launches of 32 beside them, against the oracle: numbers of
stacked rows around a wavefront and a workgroup, prefixes around a key tile, and long key lists that one workgroup walks
(those that are cut: test_gpu_attention_runs)."""
import numpy as np
import pytest
import torch

import workload as W
from workload.configs import ModelDesc, Workload
from test_gpu_attention_runs import Operands
from test_gpu_generate import gpu_generate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,hd,Bn,n,L,lens", [
    (1, 1, 64, 1, 1, 1, [64]),                # one row
    (3, 1, 64, 1, 2, 5, [65]),                # 15 rows
    (2, 1, 128, 2, 2, 8, [63, 130]),          # 16
    (1, 1, 128, 1, 3, 17, [16]),              # 17
    (7, 1, 64, 1, 2, 9, [40]),                # 63
    (2, 1, 128, 1, 2, 32, [200]),             # 64
    (5, 1, 64, 1, 2, 13, [200]),              # 65: two workgroups, one row in the second
    (6, 2, 128, 2, 2, 33, [1, 333]),          # 99
    (4, 1, 64, 1, 3, 70, [100]),              # 280, blocks of two key tiles
    (2, 2, 64, 1, 129, 65, [70]),             # 65 rows, 516 workgroups of 64: wavefronts of 32 rows
    (2, 2, 128, 1, 2, 32, [1500]),            # 64 rows, a key list in runs
    (3, 1, 64, 2, 2, 7, [2000, 1025])])
def test_stacked_rows_around_a_wavefront_and_a_workgroup(Hq, Hkv, hd, Bn, n, L, lens):
    """Without scratch, so that no list is cut; the ends of the lists and tiles are many times the rest, so a lost key shows."""
    x = Operands(Hq, Hkv, hd, Bn, n, L, lens)
    out, used = x.launch()
    some = [divmod(c, n) for c in (range(Bn * n) if Bn * n <= 8 else (0, Bn * n // 2, Bn * n - 1))]
    assert not used and x.beyond_the_bound(out, some) <= 1


@pytest.mark.parametrize("n,hq,hkv,hd,lens", [
    (1, 1, 1, 64, (63, 64)), (5, 6, 2, 64, (200, 201)), (4, 4, 1, 64, (64, 65)), (8, 4, 2, 128, (700, 701)),
    (13, 5, 1, 64, (130, 131)), (16, 6, 1, 128, (1024, 1025)), (40, 8, 4, 64, (90, 91))])
def test_generated_positions_equal_scoring(n, hq, hkv, hd, lens):
    """Single positions of 1, 15, 16, 16, 65, 96 and 80 stacked rows: log-likelihoods of the drawn tokens against block scoring,
    within the stated tolerance between the two (2e-2 a token)."""
    from paper_2506_15733_amd import synthetic
    d = hq * hd
    t = ModelDesc("target", 2, d, hq, hkv, hd, 256, 777, "bf16", "lm")
    dr = ModelDesc("draft", 1, d, hq, hkv, hd, 128, 777, "bf16", "lm")
    p = ModelDesc("prm", 1, d, hq, hkv, hd, 128, 777, "bf16", "prm")
    wl = Workload("gen_rows16", t, dr, p, B=1, n=n, L=5, prefix_len=0, lens_range=lens, betas=(1.0,), token_dist="uniform",
                  page_tokens=16, seed=41, u_seed=42)
    step = synthetic.ScoringStep(wl)
    step.prefill()
    u = W.rng.uniform_f64(wl.u_seed, "gen/u16", wl.n * wl.L).reshape(1, wl.n, wl.L)
    cand, logp, tok = gpu_generate(step, "target", u)
    step.cand = torch.from_numpy(cand).to(step.device)
    step.score("target")
    torch.cuda.synchronize()
    assert np.abs(step.tok["target"].cpu().numpy() - tok).max() < 2e-2
    step.close()
