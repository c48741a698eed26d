"""Sampling with one to seven ids per thread, each a kernel of its own: 128 chunks of 256 threads, so up to 32768 permitted ids one
id per thread, up to 65536 two, and so on. (Eight, and the kernel for more: test_gpu_generate.)"""
import numpy as np
import pytest

import oracle
import workload as W
from workload.configs import HostWeights
from test_gpu_generate import compare_generation, gpu_generate, small_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("limit,ids", [(32768, 1), (32769, 2), (65536, 2), (65537, 3), (98304, 3), (98305, 4), (131072, 4), (131073, 5),
                                       (163840, 5), (163841, 6), (196608, 6), (196609, 7), (229376, 7)])
def test_draws_match_the_oracle_at_the_edges_of_the_runs(limit, ids):
    """Logits within 1e-5 move the oracle's running sum by a factor of 1 +- 2e-5; a draw may lie one id beside the oracle's
    within that distance, so the mass of one id, the oracle's largest, is added."""
    from paper_2506_15733_amd import synthetic
    assert ids == -(-(-(-limit // 128)) // 256)
    wl = small_workload("f32", B=1, n=4, L=2, V=limit + 40, seed=18)
    step = synthetic.ScoringStep(wl)
    step.prefill()
    u = W.rng.uniform_f64(5, "gen/runs", wl.n * wl.L).reshape(1, wl.n, wl.L)
    u[0, 0, 0], u[0, 1, 0] = 0.0, 1.0 - 2.0 ** -53           # the first and the last permitted id
    cand, logp, tok = gpu_generate(step, "draft", u, vocab_limit=limit)
    assert cand.max() < limit and cand[0, 0, 0] == 0 and cand[0, 1, 0] == limit - 1
    hw = HostWeights(wl.draft, wl.seed)
    cache = oracle.prefill(wl.draft, hw, wl.prefix_tokens())[0]
    p_max = np.zeros((wl.n, wl.L))
    o_tokens, o_tok, o_blk, _, o_bounds = oracle.generate_blocks(wl.draft, hw, cache, wl.n, wl.L, u[0], vocab_limit=limit,
                                                                 p_max=p_max)
    eta = 2e-5 + p_max.max()
    assert compare_generation(cand[0], tok[0], logp[0], o_tokens, o_tok, o_blk, o_bounds, u[0], 1e-5, eta, p_max) > 0.7
    step.close()
