"""Passes that leave room for others beside them, and the same passes alone."""
import numpy as np
import pytest

import workload as W

pytestmark = pytest.mark.gpu


def test_results_do_not_hang_on_what_runs_beside():
    """The small configuration, whose products take another ring beside others: every score to the bit."""
    from paper_2506_15733_amd import synthetic
    step = synthetic.ScoringStep(W.get_config("c2_small"))
    step.prefill()
    together = step.score_and_select()
    for r in step.ROLES:
        step.out[r].zero_()
        step._fork()
        step.score(r, alone=True)
        step._join()
    alone = step.out
    for r in step.ROLES:
        assert np.array_equal(alone[r].cpu().numpy(), together[r]), r
    assert np.array_equal(step.tok["target"].cpu().numpy(), together["tok_target"])
    step.close()
