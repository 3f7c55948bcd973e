"""Fluid steps on grids of shapes that leave many lanes without a cell."""
import numpy as np
import pytest

from paper_1110_4903_amd import synth
from tests.test_gpu_fluid import flow_state, scaled_diff
from tests.test_gpu_fluid_ranges import two_range

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,nx,ny", [(9, 75, 50), (16, 65, 130), (36, 401, 250), (64, 129, 65)])
def test_fluid_steps_repeat_bitwise(ns, nx, ny):
    """Steps of the kernels that share a face among wavefronts, on ragged grids: lanes without a cell neither
    read nor change what another lane's cell becomes, so a step repeats to the last bit."""
    from oracle import fluid_oracle as fo
    from paper_1110_4903_amd import kin
    m = two_range(ns, 40 + ns)
    gas = fo.Gas(m)
    Q = np.ascontiguousarray(flow_state(fo, gas, nx, ny, 5, 500.0, 1800.0))
    with kin.Context(0) as ctx:
        mid, want = ctx.mech_upload(m), None
        for k in range(8):
            fid = ctx.fluid_create(mid, nx, ny, 1e-3 / nx, 1e-3 / ny, 1)   # a grid keeps its Newton start temperatures
            ctx.fluid_upload(fid, Q)
            dt = ctx.fluid_max_dt(fid, 0.4)
            ctx.fluid_step(fid, dt)
            ctx.fluid_step(fid, dt, y_first=True)
            got = ctx.fluid_download(fid)
            ctx.fluid_release(fid)
            want = got if want is None else want
            assert np.isfinite(got).all()
            assert np.count_nonzero(got != want) == 0, k


@pytest.mark.parametrize("ns", [4, 9, 16, 19])
@pytest.mark.parametrize("nx,ny", [(31, 1), (130, 1), (2, 1), (16, 2), (33, 2), (17, 3), (70, 3), (200, 4), (20000, 1), (9001, 2)])
def test_fluid_step_flat_grids(nx, ny, ns):
    """Grids of one to four rows, whose tiles along y are up to 32 columns wide, narrow and ragged ones, with one
    wavefront per face and with several.  Gate as for the other fluid parity tests."""
    from oracle import fluid_oracle as fo
    from paper_1110_4903_amd import kin
    m = two_range(ns, 7)
    gas = fo.Gas(m)
    dx = dy = 1e-3 / nx
    Q = np.ascontiguousarray(flow_state(fo, gas, nx, ny, 3, 500.0, 1800.0))
    with kin.Context(0) as ctx:
        fid = ctx.fluid_create(ctx.mech_upload(m), nx, ny, dx, dy, 1)
        ctx.fluid_upload(fid, Q)
        dt = fo.max_dt(gas, Q, dx, dy, 0.4)
        for y_first in (False, True):
            ctx.fluid_step(fid, dt, y_first=y_first)
            Q = fo.fluid_step(gas, Q, dt, dx, dy, "outflow", y_first=y_first)
        d = scaled_diff(ctx.fluid_download(fid), Q)
        assert np.all(d <= 1e-10), d


def test_fluid_step_long_single_row():
    """2^27 cells in a row: a launch of eight lanes a cell along y and four wavefronts a face would be 2^32 threads.
    A uniform flow of all of it stays as it is to 1e-12, but for the roundings of six stages."""
    import torch
    from paper_1110_4903_amd import kin
    from oracle import fluid_oracle as fo
    ns, nx = 17, (1 << 27) + 40
    m = two_range(ns, 7)
    gas = fo.Gas(m)
    q = np.ascontiguousarray(flow_state(fo, gas, 4, 1, 3, 900.0, 901.0))[:, 0, 0]
    Q = torch.empty(ns + 3, 1, nx, device="cuda", dtype=torch.float64)
    Q[:] = torch.as_tensor(q, device="cuda")[:, None, None]
    torch.cuda.synchronize()
    with kin.Context(0) as ctx:
        fid = ctx.fluid_create(ctx.mech_upload(m), nx, 1, 1e-4, 1e-4, 1)
        ctx.fluid_upload(fid, Q)
        ctx.fluid_step(fid, 1e-8)
        out = torch.empty_like(Q)
        assert kin._lib.kin_fluid_download(ctx._h, fid, out.data_ptr(), kin.MEM_DEVICE, None) == kin.OK
        ctx.sync()
    scale = np.abs(q)
    scale[ns:ns + 2] = scale[ns:ns + 2].max()
    for v in range(ns + 3):
        assert float((out[v] - Q[v]).abs().max()) <= 1e-12 * scale[v], v


@pytest.mark.parametrize("ns", [9, 10, 11, 13, 14, 16])
@pytest.mark.parametrize("nx,ny", [(128, 128), (201, 97), (20000, 2)])
def test_fluid_step_two_wavefronts(nx, ny, ns):
    """The species counts that two wavefronts share (of nine only up to 16384 cells), even and odd, on grids at and
    beyond that size.  Gate as for the other fluid parity tests."""
    from oracle import fluid_oracle as fo
    from paper_1110_4903_amd import kin
    m = two_range(ns, 7)
    gas = fo.Gas(m)
    dx, dy = 1e-3 / nx, 1e-3 / ny
    Q = np.ascontiguousarray(flow_state(fo, gas, nx, ny, 3, 500.0, 1800.0))
    with kin.Context(0) as ctx:
        fid = ctx.fluid_create(ctx.mech_upload(m), nx, ny, dx, dy, 1)
        ctx.fluid_upload(fid, Q)
        dt = fo.max_dt(gas, Q, dx, dy, 0.4)
        for y_first in (False, True):
            ctx.fluid_step(fid, dt, y_first=y_first)
            Q = fo.fluid_step(gas, Q, dt, dx, dy, "outflow", y_first=y_first)
        d = scaled_diff(ctx.fluid_download(fid), Q)
        assert np.all(d <= 1e-10), d
