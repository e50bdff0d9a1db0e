"""The bucket offsets: up to 4096 buckets every scatter block scans the histogram
in LDS and the moments kernel clears it, beyond that kernels of their own do both.
Runs at the limit and across it, with counts of the push pending in the histogram."""
from __future__ import annotations

import sys

import numpy as np
import pytest

import oracle as O
from paper_2111_13072_amd import sim as S
from paper_2111_13072_amd import workload as W

pytestmark = pytest.mark.gpu


def _member(n, seed, n_steps):
    st = W.uniform_shell(n, seed, 5.0, 0.2)
    return S.Member(pos=st.pos, vel=st.vel, u_asy=0.3 * np.cos(np.arange(n_steps)),
                    ntilde=W.ntilde_for(n, 5.0), q_surface0=-2.0)


# One particle per bucket: as many buckets as the LDS holds, one more, and the
# same run through the ranking kernel for large buckets (offsets always apart).
@pytest.mark.parametrize("n", [4095, 4096, 4097])
def test_runs_at_the_limit(n):
    print(f"[gpu] bucket limit n={n}", file=sys.stderr, flush=True)
    m = _member(n, 70 + n, 4)
    out = []
    for bucket in (1, 64):
        with S.Batch(S.SimParams(l_max=3, sort_bucket=bucket), [m]) as b:
            E = b.eval_field(0)
            b.step(3)
            s = b.read_state(0)
            out.append((E, b.read_response(0, 0, 3), s["pos"], s["vel"], s["alive"]))
    assert all(np.isfinite(a).all() for a in out[0])
    for a, c in zip(*out):
        np.testing.assert_array_equal(a, c)
    op = O.Params(ntilde=m.ntilde, l_max=3)
    Eo, _ = O.field(op, m.pos, q_surface=-2.0, u_asy=m.u_asy[0])
    own = np.sqrt(np.sum(Eo * Eo, axis=1))
    scale = np.maximum(own, np.sqrt(np.mean(own * own)))
    assert np.max(np.max(np.abs(out[0][0] - Eo), axis=1) / scale) <= 1e-12


def test_batch_crosses_the_limit_between_steps():
    """3000 buckets, then 5000, then 3000 again, a field evaluation on either side:
    the members' runs equal those of the same members alone."""
    first, second = _member(3000, 81, 14), _member(2000, 82, 9)
    cp = S.SimParams(l_max=3, sort_bucket=1)
    print("[gpu] batch across the bucket limit", file=sys.stderr, flush=True)
    with S.Batch(cp, [], slot_capacity=5400, max_members=2,
                 member_data=2 * S.member_data_bytes(14)) as b:
        i = b.add(first)
        b.step(3)
        j = b.add(second)
        b.step(3)
        E_mid = b.eval_field(j)
        b.step(2)
        s2, q2 = b.read_state(j), b.read_response(j, 0, 5)
        b.remove(j)
        b.step(2)
        E_end = b.eval_field(i)
        b.step(2)
        s1, q1 = b.read_state(i), b.read_response(i, 0, 12)
    for m, steps, at, E, s, q in ((first, 12, 10, E_end, s1, q1), (second, 5, 3, E_mid, s2, q2)):
        with S.Batch(cp, [m]) as a:
            a.step(at)
            Ea = a.eval_field(0)
            a.step(steps - at)
            sa, qa = a.read_state(0), a.read_response(0, 0, steps)
        assert np.isfinite(Ea).all() and np.isfinite(qa).all() and np.isfinite(sa["pos"]).all()
        np.testing.assert_array_equal(E, Ea)
        np.testing.assert_array_equal(q, qa)
        for k in ("pos", "vel", "alive"):
            np.testing.assert_array_equal(s[k], sa[k])
