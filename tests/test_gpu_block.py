"""GPU parity of the workgroup-per-cell kernel (64 to 126 species, FP64) with the oracle: species counts at
the edges of its matrix (65 and 127 unknowns, 96 and 97 columns with the right-hand side, whole and ragged
strips of 32 columns), mechanisms without third bodies and with many, and the counts just outside, which
other layouts take.  Schedules and iteration counts are the oracle's; T within 1e-9 and Y within 1e-9 of the
largest, as two Newton solutions to 1e-10 of the same sub-steps may differ."""
import numpy as np
import pytest

from paper_1110_4903_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,tb", [(63, 0.15), (64, 0.15), (64, 0.0), (79, 0.5), (94, 0.15), (95, 0.15), (96, 0.0), (110, 0.3),
                                   (126, 0.15), (127, 0.15)])
def test_block_kernel_against_oracle(ns, tb):
    from oracle import oracle
    from paper_1110_4903_amd import kin
    m = synth.make_mechanism(synth.MechRecipe("blk%d" % ns, seed=900 + ns, n_elements=5, n_species=ns, n_reactions=4 * ns + 3,
                                              frac_third_body=tb, frac_irreversible=0.3))
    om = oracle.OracleMech(m)
    n = 6
    st = synth.uniform_cells(11, n, m.ns, 0.5)
    ref = om.advance(st.rho, st.T, st.Y, 2e-8, with_sched=True)
    other = synth.make_mechanism(synth.MechRecipe("blk100", seed=77, n_elements=5, n_species=100, n_reactions=400,
                                                  frac_third_body=0.2, frac_irreversible=0.3))
    so = synth.uniform_cells(12, 600, other.ns, 0.5)
    with kin.Context(0) as c:
        j = c.state_upload(c.mech_upload(other), so.rho, so.T, so.Y)
        c.advance([j], [1e-10])   # leaves its values in the LDS of every compute unit
        i = c.state_upload(c.mech_upload(m), st.rho, st.T, st.Y)
        c.advance([i], [2e-8])
        T, Y, status, _, iters = c.download(i)[:5]
        sched = c.download_schedule(i)
    assert np.array_equal(status, ref[2]) and np.array_equal(iters, ref[4]) and np.array_equal(sched, ref[5])
    assert np.all(np.abs(T - ref[0]) <= 1e-9 * np.abs(ref[0]))
    assert np.all(np.abs(Y - ref[1]) <= 1e-9)


def test_block_kernel_bad_cells_do_not_disturb_others():
    """A cell that is not a number is refused, and the cells beside it advance as without it."""
    from paper_1110_4903_amd import kin
    m = synth.make_mechanism(synth.MechRecipe("blk70", seed=70, n_elements=5, n_species=70, n_reactions=210,
                                              frac_third_body=0.15, frac_irreversible=0.3))
    st = synth.uniform_cells(3, 5, m.ns, 0.5)
    with kin.Context(0) as c:
        mid = c.mech_upload(m)
        i = c.state_upload(mid, st.rho, st.T, st.Y)
        c.advance([i], [1e-7])
        want = c.download(i)
        T = st.T.copy()
        T[2] = np.nan
        j = c.state_upload(mid, st.rho, T, st.Y)
        c.advance([j], [1e-7])
        got = c.download(j)
    keep = [0, 1, 3, 4]
    assert got[2][2] == 3
    for a, b in zip(want[:2], got[:2]):
        a, b = (x if x.shape[0] == 5 else x.T for x in (np.asarray(a), np.asarray(b)))
        assert np.array_equal(a[keep], b[keep])
