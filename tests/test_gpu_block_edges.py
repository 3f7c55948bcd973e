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


def test_block_kernel_more_threads_than_a_grid_holds():
    """2^23 cells are 2^32 threads: every cell advances, in the same way as in a small instance."""
    import torch
    from paper_1110_4903_amd import kin
    ns, n = 64, (1 << 23) + 5
    m = exchange_mech(ns, 0, 1)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    dev = dict(device="cuda", dtype=torch.float64)
    T = 1000.0 + 2000.0 * torch.rand(n, generator=g, **dev)
    rho = 0.1 + torch.rand(n, generator=g, **dev)
    Y = torch.rand(ns, n, generator=g, **dev)
    Y /= Y.sum(0)
    pick = torch.cat([torch.arange(0, n, n // 50, device="cuda"), torch.arange(n - 6, n, device="cuda")])
    dt = 0.25   # k dt = 1/4 each way: the difference shrinks by 1 + 2 k dt
    torch.cuda.synchronize()
    with kin.Context(0) as c:
        mid = c.mech_upload(m)
        i = c.state_upload(mid, rho, T, Y)
        j = c.state_upload(mid, rho[pick].contiguous(), T[pick].contiguous(), Y[:, pick].contiguous())
        c.advance([i], [dt])
        c.advance([j], [dt])
        T1, Y1 = torch.empty_like(T), torch.empty_like(Y)
        status = torch.full((n,), -1, device="cuda", dtype=torch.int32)
        c.download_device(i, T1, Y1, status=status)
        c.sync()
        assert int((status != 0).sum()) == 0
        want = (Y[0] - Y[1]) / 1.5
        assert float((Y1[0] - Y1[1] - want).abs().max()) <= 1e-14 and bool((Y1[2:] == Y[2:]).all())
        part = c.download(j)
        assert np.array_equal(part[0], T1[pick].cpu().numpy()) and np.array_equal(np.asarray(part[1]), Y1[:, pick].cpu().numpy())


def test_block_kernel_batch_holds_no_workspace():
    """The graph of a batched advance holds the matrices of the one-wavefront kernel (1.6 GiB here); a workgroup
    per cell keeps its own on chip, so the batch may take only what the runtime sets up for a graph."""
    import torch
    from paper_1110_4903_amd import kin
    m = exchange_mech(100, 0, 1)
    st = synth.uniform_cells(8, 8192, m.ns, 0.5)
    with kin.Context(0) as c:
        mid = c.mech_upload(m)
        ids = [c.state_upload(mid, st.rho, st.T, st.Y) for _ in range(3)]
        c.advance(ids[2:], [0.25])   # (the kernel's own set-up)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        c.advance(ids[:2], [0.25, 0.25])
        torch.cuda.synchronize()
        assert free - torch.cuda.mem_get_info()[0] < 128 << 20
        want = c.download(ids[2])
        for i in ids[:2]:
            for x, y in zip(c.download(i), want):
                assert np.array_equal(x, y)


@pytest.mark.parametrize("n", [40, 600])
def test_block_kernel_in_a_callers_graph(n):
    """An advance captured by the caller (the launch attribute of the kernel's LDS, the cost order from 513 cells
    on), replayed with eager work between, is the eager advance."""
    import torch
    from paper_1110_4903_amd import kin
    m = synth.make_mechanism(synth.MechRecipe("cap66", seed=66, n_elements=4, n_species=66, n_reactions=150,
                                              frac_third_body=0.15, frac_irreversible=0.3))
    states = [synth.uniform_cells(30 + k, n, m.ns, 0.5) for k in range(3)]
    with kin.Context(0) as c:
        mid = c.mech_upload(m)
        st = states[0]
        want = []
        for q in states:
            j = c.state_upload(mid, q.rho, q.T, q.Y)
            c.advance([j], [1e-8])
            want.append(c.download(j)[:5])
        i = c.state_upload(mid, st.rho, st.T, st.Y)
        torch.cuda.synchronize()
        s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            c.advance([i], [1e-8], stream=s)
        x = torch.zeros(1 << 20, device="cuda")
        for q, w in zip(states + states, want + want):
            c.state_reset(i, q.rho, q.T, q.Y)
            x.add_(1.0)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            for a, b in zip(c.download(i)[:5], w):
                assert np.array_equal(a, b)
