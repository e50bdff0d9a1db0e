"""sim_profile: a kernel kind that a step does not launch takes no time (the events
around it are microseconds apart), and one that it launches takes some."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from paper_2111_13072_amd import sim as S
from paper_2111_13072_amd import workload as W

pytestmark = pytest.mark.gpu

ALWAYS = {"sort_scatter", "moments", "carry_chunk_scan", "field_push"}


@pytest.mark.parametrize("n,knobs,more", [
    (1000, {}, set()), (40_000, {}, {"bucket_sums", "bucket_offsets"}),
    (1000, {"sort_bucket": 64}, {"bucket_sums", "bucket_offsets", "sort_rank_move"}),
    (1000, {"carry_chunk": 8}, {"carry_chunk_sums", "carry_apply"}),
    (1000, {"sort_keys": -1}, {"sort_key"})])
def test_profile_times_only_launched_kernels(n, knobs, more):
    print(f"[gpu] profile n={n} {knobs}", file=sys.stderr, flush=True)
    st = W.uniform_shell(n, 5, 5.0, 0.05)
    with S.Sim(S.SimParams(ntilde=W.ntilde_for(n, 5.0), l_max=2, **knobs), st.pos, st.vel,
               np.zeros(8)) as sim:
        first, later = sim.profile(1), sim.profile(2)
    assert {k for k, v in first.items() if v > 0.0} == ALWAYS | more | {"sort_key"}
    assert {k for k, v in later.items() if v > 0.0} == ALWAYS | more
