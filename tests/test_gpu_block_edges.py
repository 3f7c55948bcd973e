"""Edges of the workgroup-per-cell kernel (64 to 126 species, FP64)."""
import dataclasses

import numpy as np
import pytest

from paper_1110_4903_amd import synth

pytestmark = pytest.mark.gpu


def exchange_mech(ns, a, b):
    """Inert species, and one exchange a <=> b of identical thermodynamics with k = 1/s both ways.  The molar
    masses are a power of two, so the Newton matrix of a step h has exactly 1 + h and -h in rows a and b."""
    nasa = []
    for s in range(ns):
        row = [3.5 if s in (a, b) else 2.5 + 0.05 * s, 0, 0, 0, 0, -1000.0, 30.0]
        nasa.append([row, row])
    m = synth.mechanism_from_lists("exchange%d" % ns, ("H",), [[2]] * ns, nasa, [dict(reac=[(a, 1)], prod=[(b, 1)], A=1.0)])
    return dataclasses.replace(m, M=np.full(ns, 32.0))


@pytest.mark.parametrize("ns,a,b", [(64, 0, 1), (66, 65, 3), (95, 94, 93), (126, 70, 125)])
def test_block_kernel_singular_matrix(ns, a, b):
    """From h = 2^53 s on, 1 + h rounds to h and the matrix is singular to the last bit: the attempt fails and
    the step is halved until 2^52 s, as the oracle does, whether the two species balance at the start or not.
    Y within 1e-12 (the sums of a few hundred roundings).  Without halving the cell fails and keeps its state."""
    from oracle import oracle
    from paper_1110_4903_amd import kin
    m = exchange_mech(ns, a, b)
    st = synth.uniform_cells(5, 700, ns, 0.5)   # more cells than are in flight at a time
    st.Y[[a, b], ::2] = st.Y[[a, b], ::2].mean(0)
    dt = 2.0 ** 55
    ref = oracle.OracleMech(m).advance(st.rho, st.T, st.Y, dt, with_sched=True)
    assert np.all(ref[3] == 3)
    with kin.Context(0) as c:
        mid = c.mech_upload(m)
        i = c.state_upload(mid, st.rho, st.T, st.Y)
        c.advance([i], [dt])
        T, Y, status, level = c.download(i)[:4]
        sched = c.download_schedule(i)
        assert np.array_equal(status, ref[2]) and np.array_equal(level, ref[3]) and np.array_equal(sched, ref[5])
        assert np.all(np.abs(T - st.T) <= 1e-12 * st.T)
        assert np.all(np.abs(Y - ref[1]) <= 1e-12)
        c.state_reset(i, st.rho, st.T, st.Y)
        c.advance([i], [dt], opts=kin.solver_opts(L_forced=0))
        T, Y, status = c.download(i)[:3]
        assert np.all(status == 2) and np.array_equal(T, st.T) and np.array_equal(Y, st.Y)
