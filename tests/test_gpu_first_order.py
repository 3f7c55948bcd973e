"""A first advance takes the cells of an instance in the order of their predicted cost from a size on that
depends on the layout; the order never changes a cell.  Instances at and above that size are compared bitwise
with their cells advanced in small instances, which take them as they come, and with a second advance of the
same states, which the first one's iteration counts order."""
import numpy as np
import pytest

from paper_1110_4903_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which,n,part,dt,prec", [("mech36", 2560, 512, 1e-7, "fp64"), ("mech36", 4097, 1024, 1e-7, "fp32lu"),
                                                  ("big", 513, 128, 1e-8, "fp64"), ("big", 1400, 500, 1e-8, "fp64"),
                                                  ("big", 2561, 2000, 1e-9, "fp32lu")])
def test_first_advance_order_is_bitwise_neutral(which, n, part, dt, prec):
    from paper_1110_4903_amd import kin
    m = synth.mechanism("mech36") if which == "mech36" else synth.make_mechanism(synth.MechRecipe(
        "ord66", seed=66, n_elements=4, n_species=66, n_reactions=150, frac_third_body=0.15, frac_irreversible=0.3))
    p = kin.FP64 if prec == "fp64" else kin.FP32_LU
    st = synth.uniform_cells(21, n, m.ns, 0.5)
    Y = np.asarray(st.Y)
    axis = 0 if Y.shape[0] == n else 1
    Tn = np.array(st.T)
    Tn[5] = np.nan   # refused, wherever the order puts it
    with kin.Context(0) as c:
        mid = c.mech_upload(m)
        i = c.state_upload(mid, st.rho, Tn, st.Y)
        runs = []
        for _ in range(2):
            c.state_reset(i, st.rho, Tn, st.Y)
            c.advance([i], [dt], prec=p)
            runs.append(c.download(i)[:5] + (c.download_schedule(i),))
        parts = []
        for a in range(0, n, part):
            s = slice(a, min(a + part, n))
            j = c.state_upload(mid, st.rho[s], Tn[s], np.ascontiguousarray(Y[s] if axis == 0 else Y[:, s]))
            c.advance([j], [dt], prec=p)
            parts.append(c.download(j)[:5] + (c.download_schedule(j),))
            c.instance_release(j)
    for k, x in enumerate(runs[0]):
        whole = np.concatenate([np.asarray(q[k]) for q in parts], axis=axis if np.ndim(x) == 2 else 0)
        assert np.array_equal(np.asarray(x), whole, equal_nan=x.dtype.kind == "f"), k
        assert np.array_equal(np.asarray(x), np.asarray(runs[1][k]), equal_nan=x.dtype.kind == "f"), k
    assert runs[0][2][5] == 3
