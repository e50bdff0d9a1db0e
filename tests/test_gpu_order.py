"""The radial order at its edges, against the CPU oracle or between two ways
through the sort.  Bars as in test_gpu_kernels: 1e-12 of the larger of the RMS
field and the particle's own."""
from __future__ import annotations

import sys

import numpy as np
import pytest

import oracle as O
from paper_2111_13072_amd import sim as S
from paper_2111_13072_amd import workload as W

pytestmark = pytest.mark.gpu


def _err(E, Eo):
    own = np.sqrt(np.sum(Eo * Eo, axis=1))
    scale = np.maximum(own, np.sqrt(np.mean(own * own)))
    return float(np.max(np.max(np.abs(E - Eo), axis=1) / scale))


# Radii a few rounding steps of r^2 apart: r^2 has to be formed with the same
# roundings as the definition's key, or such particles change places (each then
# counts on the wrong side of the other: 1e-2 of the field), in the key kernel
# (field evaluation) and in the push (the steps after the first).
@pytest.mark.parametrize("keys", [0, -1], ids=["push", "own-pass"])
def test_order_of_nearly_equal_radii_matches_oracle(keys):
    print(f"[gpu] nearly equal radii keys={keys}", file=sys.stderr, flush=True)
    n = 3000
    nt = W.ntilde_for(n, 5.0)
    st = W.uniform_shell(n, 700 + n, 5.0, 0.08)
    r = np.linalg.norm(st.pos, axis=1)
    pos = st.pos * ((2.0 + 1e-12 * (r - 2.0)) / r)[:, None]
    r2 = (pos[:, 0] ** 2 + pos[:, 1] ** 2) + pos[:, 2] ** 2
    assert np.unique(r2).size < n                  # ties among them, too
    u = np.array([0.2, 0.1, 0.0])
    op = O.Params(ntilde=nt, l_max=4)
    Eo, _ = O.field(op, pos, u_asy=u[0])
    # steps: a common radial speed and no coupling (ntilde 1e30) keep the
    # particles within a few rounding steps of one radius after two moves
    vel = pos * 0.3
    op2 = O.Params(ntilde=1e30, ion_density=0.0, l_max=4)
    ref = O.run(op2, pos, vel, np.zeros(3), 2)
    with S.Sim(S.SimParams(ntilde=nt, l_max=4, sort_keys=keys), pos, st.vel, u) as sim:
        E = sim.eval_field()
    assert _err(E, Eo) <= 1e-12
    with S.Sim(S.SimParams(ntilde=1e30, ion_density=0.0, l_max=4, sort_keys=keys), pos, vel,
               np.zeros(3)) as sim:
        sim.step(2)
        out = sim.read_state()
        E = sim.eval_field()                       # sorted by the push's keys
    assert _err(E, O.field(op2, ref.pos)[0]) <= 1e-12
    np.testing.assert_array_equal(out["pos"], ref.pos)
    np.testing.assert_array_equal(out["vel"], ref.vel)


# A position that is not a number makes every field one, and none is left out:
# its key sorts above every number's, so its bucket has to be the last one where
# a tile selects its records by the key (600 particles in the first bucket's
# shell, past the ranking's LDS window).
def test_field_with_a_nan_position_is_written_everywhere():
    import torch

    n, first = 3000, 600
    print(f"[gpu] NaN positions n={n}", file=sys.stderr, flush=True)
    st = W.uniform_shell(n, 57, 5.0, 0.1)
    pos = st.pos.copy()
    r = np.linalg.norm(pos, axis=1)
    pos[:first] *= ((1.0 + 1e-4 * (r - 1.0)) / r)[:first, None]
    pos[100:300] = np.nan
    dpos = torch.from_numpy(pos).cuda()
    E = torch.full_like(dpos, 7.0)
    S.eval_field_static(S.SimParams(ntilde=W.ntilde_for(n, 5.0), l_max=3), dpos, E)
    assert bool(torch.isnan(E).all())
