"""Cost order of an advance: at sizes where its kernels can go wrong, and by the counts of an advance before."""
import numpy as np
import pytest

from paper_1110_4903_amd import synth

pytestmark = pytest.mark.gpu


def test_first_order_more_threads_than_a_grid_holds():
    """A wavefront for each of 2^26 cells is 2^32 threads: the estimate of the costs takes cells in turns, and
    every cell advances as the closed form has it, the ones at the end too."""
    import torch
    from paper_1110_4903_amd import kin
    from tests.test_gpu_block_edges import exchange_mech
    n = (1 << 26) + 3
    m = exchange_mech(2, 0, 1)
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    dev = dict(device="cuda", dtype=torch.float64)
    rho, T = 0.1 + torch.rand(n, generator=g, **dev), 1000.0 + 2000.0 * torch.rand(n, generator=g, **dev)
    Y = torch.empty(2, n, **dev)
    Y[0] = torch.rand(n, generator=g, **dev)
    Y[1] = 1.0 - Y[0]
    T[5], T[n - 2] = float("nan"), float("nan")   # refused, wherever the order puts them
    dt = 0.25
    torch.cuda.synchronize()
    with kin.Context(0) as c:
        i = c.state_upload(c.mech_upload(m), rho, T, Y)
        c.advance([i], [dt], opts=kin.solver_opts(layout=kin.LAYOUT_GLOBAL))
        T1, Y1 = torch.empty_like(T), torch.empty_like(Y)
        status = torch.full((n,), -1, device="cuda", dtype=torch.int32)
        c.download_device(i, T1, Y1, status=status)
        c.sync()
    bad = torch.nonzero(status).flatten().tolist()
    assert bad == [5, n - 2] and status[5] == 3 and status[n - 2] == 3
    d, want = Y1[0] - Y1[1], (Y[0] - Y[1]) / 1.5
    want[bad] = (Y[0] - Y[1])[bad]
    assert float((d - want).abs().max()) <= 1e-14


@pytest.mark.parametrize("which,n,part,dt,prec", [("mech36", 8192, 2500, 1e-7, "fp64"), ("mech36", 8193, 2500, 1e-7, "fp32lu"),
                                                  ("mech36", 8191, 2500, 1e-7, "fp64"), ("small", 4096, 4000, 1e-7, "fp64"),
                                                  ("small", 9000, 4000, 1e-7, "fp32lu"), ("big", 513, 200, 1e-8, "fp64"),
                                                  ("big", 1025, 500, 1e-8, "fp64"), ("big", 1400, 500, 1e-7, "fp64")])
def test_orders_are_bitwise_neutral(which, n, part, dt, prec):
    """Two advances without a reset, ordered by the estimate and then by the counts of the first, at the sizes
    where each begins, and where one block makes the order and where three kernels do: every cell as in small
    instances, which take their cells as they come.  The counts span several classes."""
    from paper_1110_4903_amd import kin
    m = synth.mechanism("mech36") if which == "mech36" else synth.make_mechanism(synth.MechRecipe(
        "ord_" + which, seed=66, n_elements=4, n_species=66 if which == "big" else 20, n_reactions=150,
        frac_third_body=0.15, frac_irreversible=0.3))
    p = kin.FP64 if prec == "fp64" else kin.FP32_LU
    st = synth.uniform_cells(23, n, m.ns, 0.5)
    st.T[7] = np.nan
    with kin.Context(0) as c:
        mid = c.mech_upload(m)

        def both(s):
            i = c.state_upload(mid, np.ascontiguousarray(st.rho[s]), np.ascontiguousarray(st.T[s]), np.ascontiguousarray(st.Y[:, s]))
            c.advance([i], [dt], prec=p)
            first = c.download(i)[:5] + (c.download_schedule(i),)
            c.advance([i], [dt], prec=p)
            second = c.download(i)[:5] + (c.download_schedule(i),)
            c.instance_release(i)
            return [np.asarray(x) for x in first + second]

        whole = both(slice(0, n))
        parts = [both(slice(a, min(a + part, n))) for a in range(0, n, part)]
    for k, x in enumerate(whole):
        y = np.concatenate([q[k] for q in parts], axis=x.ndim - 1)
        assert np.array_equal(x, y, equal_nan=x.dtype.kind == "f"), k
    assert whole[2][7] == 3
    assert len(np.unique(np.digitize(whole[4], 5 * 2 ** np.arange(7)))) > 2
