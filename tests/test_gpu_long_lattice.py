"""A lattice whose work items exceed what one launch takes (2^32 - 1 threads, 4194303
workgroups of 1024): the step goes out in several launches and gives the same bits as
with chunks that fit one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NZ = 4194303 + 1000  # one column; at a plane a workgroup the last 1000 are left for a second launch


def test_work_items_beyond_one_launch():
    from paper_2403_15773_amd.tslb import Simulation
    z = 2 * np.pi / NZ * np.arange(NZ)
    wave = [np.sin(k * z + k).astype(np.float32).reshape(NZ, 1, 1) for k in (7, 3 * NZ // 40, 1001, NZ // 33)]
    st = {"rho_dev": 1e-3 * wave[0], "u": 0.02 * np.stack(wave[:3]), "P": 1e-4 * np.stack(wave + wave[:2]),
          "phi": 0.5 + 0.45 * wave[1]}
    raw = []
    for chunk in (0, 1):
        print("[gpu-test] 1 x 1 x %d, chunk %d" % (NZ, chunk), flush=True)
        with Simulation(nx=1, ny=1, nz=NZ, nu=0.02, sigma=0.005, width=3.0, bc=(0,) * 6, eps=1e-4) as s:
            s.set_kernel("fused", chunk)
            s.set_state(**st)
            s.step(2)
            raw.append(s.get_state_raw())
            assert s.diagnostics()["finite"]
    assert np.array_equal(raw[0], raw[1])
