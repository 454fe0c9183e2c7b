"""Time averages of a lattice whose mean fields exceed 16 and 32 MB a plane, formed and
copied as whole planes on the device path and in blocks of 4M nodes on the host path:
the same bits."""
import numpy as np
import pytest

from paper_2403_15773_amd import inputs

pytestmark = pytest.mark.gpu


def test_means_of_planes_beyond_one_host_block():
    from paper_2403_15773_amd.tslb import Simulation
    nx, ny, nz = 203, 207, 209  # 8.8M nodes: 35 MB a plane, three host blocks
    print("[gpu-test] time averages %dx%dx%d" % (nx, ny, nz), flush=True)
    st = inputs.smooth_state(nx, ny, nz)
    with Simulation(nx=nx, ny=ny, nz=nz, nu=0.02, sigma=0.005, width=3.0, bc=(0, 0, 4, 1, 0, 0), eps=1e-4) as s:
        s.set_state(**{k: st[k] for k in ("rho_dev", "u", "P", "phi")})
        s.stats_start(1)
        s.step(2)
        a = s.stats()
        s.stats_stop()
        b = s.stats()
    assert a["samples"] == b["samples"] == 2
    for k in ("mean_phi", "mean_u", "rms_uz"):
        assert np.array_equal(a[k], b[k]) and np.isfinite(a[k]).all(), k
    assert np.abs(a["mean_u"]).max() > 0.01 and 0.0 < a["mean_phi"].mean() < 1.0
