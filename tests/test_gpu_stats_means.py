"""Time averages formed on the device (while sampling goes on) and on the host (after
it has stopped, when nothing is allocated for them): the same bits."""
import numpy as np
import pytest

from paper_2403_15773_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,components,samples", [((33, 17, 11), 2, 3), ((32, 16, 8), 1, 1), ((61, 45, 23), 2, 7)])
def test_means_are_the_same_bits_on_device_and_host(shape, components, samples):
    from paper_2403_15773_amd.tslb import Simulation
    print("[gpu-test] time averages %s, %d component(s), %d samples" % (shape, components, samples), flush=True)
    st = inputs.smooth_state(*shape)
    if components == 1:
        st["phi"][...] = 0
    with Simulation(nx=shape[0], ny=shape[1], nz=shape[2], nu=0.02, sigma=0.005 if components == 2 else 0.0, width=3.0,
                    bc=(0, 0, 4, 1, 0, 0), components=components, eps=1e-4) as s:
        s.set_state(**{k: st[k] for k in ("rho_dev", "u", "P", "phi")})
        s.stats_start(2)
        s.step(2 * samples)
        a = s.stats()
        again = s.stats()  # the sums are left as they were
        s.step(2)
        c = s.stats()
        s.stats_stop()
        d = s.stats()
        assert a["samples"] == again["samples"] == samples and c["samples"] == d["samples"] == samples + 1
        for k in ("mean_phi", "mean_u", "rms_uz"):
            assert np.array_equal(a[k], again[k]) and np.array_equal(c[k], d[k])
        assert components == 1 or not np.array_equal(a["mean_phi"], c["mean_phi"])
        assert (c["rms_uz"] > 0).any() and np.isfinite(c["rms_uz"]).all()
