"""Fluid steps on grids of shapes that leave many lanes without a cell."""
import numpy as np
import pytest

from paper_1110_4903_amd import synth
from tests.test_gpu_fluid import flow_state
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
