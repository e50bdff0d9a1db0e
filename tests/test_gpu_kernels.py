"""Kernel variants at the sizes where their splits can go wrong, against the
CPU oracle.  FP64 bar: 1e-12 of the larger of the RMS field and the particle's
own field.  (The own field counts because a pair at nearly equal place pushes
with ~l_max^2 / sqrt(n) of the RMS field, whose rounding no split of the sum
takes away: 300 particles at l_max 63 reach 7 times the RMS.)"""
from __future__ import annotations

import sys

import numpy as np
import pytest

import oracle as O
from paper_2111_13072_amd import sim as S
from paper_2111_13072_amd import workload as W

pytestmark = pytest.mark.gpu


def _params(n, L, mode=S.SIM_M_FULL, r_out=5.0, **kw):
    nt = W.ntilde_for(n, r_out)
    return (S.SimParams(ntilde=nt, l_max=L, m_mode=mode, r_out=r_out, **kw),
            O.Params(ntilde=nt, l_max=L, m_mode=mode, r_out=r_out))


def _err(E, Eo):
    own = np.sqrt(np.sum(Eo * Eo, axis=1))
    scale = np.maximum(own, np.sqrt(np.mean(own * own)))
    return float(np.max(np.max(np.abs(E - Eo), axis=1) / scale))


# One, two and four blocks of orders per group (l_max 8, 16, 32 on a few
# groups), odd and even l_max (the channel batches end on one or two orders),
# fewer orders than slices, and particle counts around a half, a tile and a
# group.
@pytest.mark.parametrize("n,L,mode", [
    (1, 16, S.SIM_M_FULL), (31, 2, S.SIM_M_FULL), (33, 7, S.SIM_M_FULL), (255, 8, S.SIM_M_FULL),
    (256, 9, S.SIM_M_FULL), (257, 15, S.SIM_M_FULL), (513, 33, S.SIM_M_FULL),
    (300, 63, S.SIM_M_FULL), (257, 1, S.SIM_M_FULL), (255, 1, S.SIM_M_AXISYM),
    (300, 31, S.SIM_M_AXISYM), (66, 64, S.SIM_M_AXISYM)])
def test_order_slices_match_oracle(n, L, mode):
    print(f"[gpu] order slices n={n} L={L} mode={mode}", file=sys.stderr, flush=True)
    sp, op = _params(n, L, mode, q_surface0=-3.0)
    st = W.uniform_shell(n, 600 + n, 5.0, 0.08)
    with S.Sim(sp, st.pos, st.vel, np.array([0.2])) as sim:
        E = sim.eval_field()
    Eo, _ = O.field(op, st.pos, q_surface=-3.0, u_asy=0.2)
    assert _err(E, Eo) <= 1e-12


# The group's ranking inside the moments kernel: windows of one record, of one
# bucket per group, past the LDS window (every particle in two buckets, keys
# that differ in their last digits and by the id alone) and at its edge.
@pytest.mark.parametrize("n,bucket,spread", [(1, 8, 1.0), (257, 1, 1.0), (1024, 256, 1.0),
                                             (1030, 8, 1e-9), (3000, 8, 1e-9),
                                             (700, 256, 0.0)])
def test_group_ranking_matches_oracle(n, bucket, spread):
    print(f"[gpu] group ranking n={n} bucket={bucket} spread={spread}", file=sys.stderr, flush=True)
    sp, op = _params(n, 4, sort_bucket=bucket)
    st = W.uniform_shell(n, 700 + n, 5.0, 0.08)
    r = np.linalg.norm(st.pos, axis=1)
    pos = st.pos * ((2.0 + spread * (r - 2.0)) / r)[:, None]
    if spread == 0.0:   # the same radius to the last bit: signed permutations of one point
        p = np.array([1.1, 0.7, 1.5])
        perms = [p[list(o)] * np.array(s) for o in ((0, 1, 2), (1, 0, 2))
                 for s in ((1, 1, 1), (-1, 1, 1), (1, -1, 1), (1, 1, -1))]
        pos = np.array([perms[i % len(perms)] for i in range(n)])
        pos[: n // 2] *= 1.25
    ids = np.random.default_rng(n).permutation(n).astype(np.uint32) * 3
    with S.Sim(sp, pos, st.vel, np.array([0.0]), ids=ids) as sim:
        E = sim.eval_field()
    Eo, _ = O.field(op, pos, ids=ids)
    assert _err(E, Eo) <= 1e-12


# The axisymmetric field's scan over the lanes of a tile: lanes of one row, of
# every row, partly filled tiles, the largest degree; both precisions (it runs
# in FP64 in either, so the FP32 mode's fields hold 1e-12 too, except for its
# l = 0 term in plain FP64: its rounding of ~1e-16 of the monopole field is far
# below that here).
@pytest.mark.parametrize("precision", [S.SIM_FP64, S.SIM_FP32_COMP], ids=["fp64", "fp32c"])
@pytest.mark.parametrize("n,L", [(1, 1), (2, 1), (17, 2), (49, 5), (64, 1), (65, 64), (300, 21)])
def test_axisymmetric_scan_matches_oracle(n, L, precision):
    print(f"[gpu] axisymmetric scan n={n} L={L} p={precision}", file=sys.stderr, flush=True)
    sp, op = _params(n, L, S.SIM_M_AXISYM, precision=precision)
    st = W.uniform_shell(n, 800 + n, 5.0, 0.08)
    with S.Sim(sp, st.pos, st.vel, np.array([0.1])) as sim:
        E = sim.eval_field()
    Eo, _ = O.field(op, st.pos, u_asy=0.1)
    assert _err(E, Eo) <= 1e-12


# The carries of a member in one kernel: segments of none, one and several
# groups, columns and degrees past a block's, the last member size it takes and
# the first it does not; Q_diff comes from a block of its own (l_max 33: two
# passes over its columns).
@pytest.mark.parametrize("n,L,mode", [(256 * 15, 4, S.SIM_M_FULL), (256 * 17 + 1, 7, S.SIM_M_FULL),
                                      (600, 33, S.SIM_M_FULL), (300, 0, S.SIM_M_FULL),
                                      (131_072, 3, S.SIM_M_FULL), (131_073, 3, S.SIM_M_FULL),
                                      (90_001, 2, S.SIM_M_AXISYM)])
def test_one_kernel_carries_match_chunked(n, L, mode):
    """Against the chunked carries (a tuned chunk length asks for them), which
    the oracle tests pin: the same compensated sums, one rounding apart."""
    print(f"[gpu] one-kernel carries n={n} L={L} mode={mode}", file=sys.stderr, flush=True)
    st = W.uniform_shell(n, 900 + L, 5.0, 0.08)
    out = []
    for chunk in (0, 8):
        sp, _ = _params(n, L, mode, carry_chunk=chunk, q_surface0=-2.0)
        with S.Sim(sp, st.pos, st.vel, np.array([0.3, 0.1, 0.0])) as sim:
            E = sim.eval_field()
            sim.step(3)
            out.append((E, sim.read_response(0, 3), sim.read_state()["pos"]))
    (E0, q0, p0), (E1, q1, p1) = out
    assert _err(E0, E1) <= 1e-13
    assert np.max(np.abs(q0 - q1)) <= 1e-13 * max(np.max(np.abs(q1)), 1e-300)
    assert np.max(np.abs(p0 - p1)) <= 1e-13


# A small member steps in the one-tile-per-block form of the field kernel when
# alone and in the one-tile-per-wave form beside a member of many tiles: the
# same bits (FP64, FP32, FP32 with the near field in FP64; half and whole
# tiles).  The sort, moments and carries differ in form too.
@pytest.mark.parametrize("L,precision,split", [(16, S.SIM_FP64, 0), (5, S.SIM_FP64, -1),
                                               (4, S.SIM_FP32_COMP, 0), (9, S.SIM_FP32_COMP, -1),
                                               (21, S.SIM_FP32_COMP, 0), (0, S.SIM_FP64, 0)])
def test_field_forms_agree_bitwise(L, precision, split):
    print(f"[gpu] field forms L={L} p={precision} split={split}", file=sys.stderr, flush=True)
    common = S.SimParams(l_max=L, precision=precision, near_split=split)

    def member(n, seed):
        st = W.uniform_shell(n, seed, 5.0, 0.2)
        return S.Member(pos=st.pos, vel=st.vel, u_asy=np.array([0.3, 0.1, 0.0]),
                        ntilde=W.ntilde_for(n, 5.0), q_surface0=-2.0)

    small = member(577, 21)
    out = []
    for others in ([], [member(1_100_000, 22)]):
        with S.Batch(common, [small] + others) as b:
            E = b.eval_field(0)
            b.step(3)
            out.append((E, b.read_response(0, 0, 3), b.read_state(0)))
    (E0, q0, s0), (E1, q1, s1) = out
    np.testing.assert_array_equal(E0, E1)
    np.testing.assert_array_equal(q0, q1)
    for k in ("pos", "vel", "alive"):
        np.testing.assert_array_equal(s0[k], s1[k])


@pytest.mark.parametrize("n", [1, 255, 3000])
def test_state_of_index_ids_equals_state_of_any_ids(n):
    """Ids that are the creation indices are put in order on the device, others
    on the host: the same run read both ways (the ids only break ties), with
    absorbed particles, for one member among others."""
    print(f"[gpu] state read n={n}", file=sys.stderr, flush=True)
    st = W.uniform_shell(n, 30 + n, 3.0, 0.6)
    other = W.uniform_shell(300, 31, 3.0, 0.1)
    out = []
    for ids in (None, np.arange(n, dtype=np.uint32) * 5 + 2):
        ms = [S.Member(pos=p.pos, vel=p.vel, u_asy=np.zeros(9), ids=i, r_out=3.0,
                       ntilde=W.ntilde_for(n, 3.0)) for p, i in ((other, None), (st, ids))]
        with S.Batch(S.SimParams(l_max=3), ms) as b:
            first = b.read_state(1)
            b.step(6)
            mid = b.read_state(1)
            b.step(3)
            out.append((first, mid, b.read_state(1)))
    np.testing.assert_array_equal(out[0][0]["pos"], st.pos)
    for a, c in zip(*out):
        for k in ("pos", "vel", "alive"):
            np.testing.assert_array_equal(a[k], c[k])
        assert a["q_surface"] == c["q_surface"] and a["step"] == c["step"]
    if n == 3000:
        assert (out[0][2]["alive"] == 0).any()


# Members whose ranking takes the other ways through a tile's placement, among
# them beside a member of more than a million particles, against the same
# members ranked by the kernel for large buckets (sort_bucket 64): the order is
# exact, so the runs are equal bit for bit.
@pytest.mark.parametrize("n,spread,ties", [(5000, 1.0, False), (3000, 1e-5, False),
                                           (2500, 0.05, True), (70, 1e-9, True)])
def test_placement_equals_large_bucket_ranking(n, spread, ties):
    print(f"[gpu] placement n={n} spread={spread} ties={ties}", file=sys.stderr, flush=True)
    st = W.uniform_shell(n, 41 + n, 5.0, 0.1)
    pos = st.pos.copy()
    r = np.linalg.norm(pos, axis=1)
    half = np.arange(n) % 2 == 0                      # half of them in a thin shell
    pos[half] *= ((2.0 + spread * (r - 3.0) / 2.0) / r)[half, None]
    if ties:                                          # equal radii: mirrored points
        pos[1::4] = pos[0::4][: len(pos[1::4])] * np.array([-1.0, 1.0, 1.0])
    ids = np.random.default_rng(n).permutation(n).astype(np.uint32)
    big = W.uniform_shell(1_050_000, 5, 5.0, 0.1)
    out = []
    for bucket, with_big in ((8, False), (8, True), (64, False), (1, False), (32, False)):
        ms = [S.Member(pos=pos, vel=st.vel, ids=ids, u_asy=np.array([0.2, 0.1, 0.0]),
                       ntilde=W.ntilde_for(n, 5.0))]
        if with_big:
            ms.append(S.Member(pos=big.pos, vel=big.vel, u_asy=np.array([0.2, 0.1, 0.0]),
                               ntilde=W.ntilde_for(1_050_000, 5.0)))
        with S.Batch(S.SimParams(l_max=2, sort_bucket=bucket), ms) as b:
            E = b.eval_field(0)
            b.step(3)
            s = b.read_state(0)
            out.append((E, b.read_response(0, 0, 3), s["pos"], s["vel"], s["alive"]))
    for o in out[1:]:
        for a, c in zip(out[0], o):
            np.testing.assert_array_equal(a, c)
