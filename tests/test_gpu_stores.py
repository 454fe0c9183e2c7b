"""Stores of the fused step with and without the non-temporal hint.  A lattice
whose state is a few megabytes stores with it, a larger one whose rows do not begin
at cache lines without; a lattice stacked three times along its periodic z axis
crosses that line and has to give three copies of the same bits, and two lattices
that cross it together have to give the bits they give alone."""
import numpy as np
import pytest

from paper_2403_15773_amd import inputs

pytestmark = pytest.mark.gpu

NX, NY, NZ = 61, 76, 48


def _sim(copies, storage, components):
    from paper_2403_15773_amd.tslb import Simulation
    s = Simulation(nx=NX, ny=NY, nz=NZ * copies, nu=0.02, sigma=0.005 if components == 2 else 0.0, width=3.0,
                   bc=(0, 0, 4, 1, 0, 0), components=components, eps=1e-4, storage=storage)
    st = inputs.smooth_state(NX, NY, NZ)
    if components == 1:
        st["phi"][...] = 0
    s.set_state(**{k: np.concatenate([st[k]] * copies, axis=-3) for k in ("rho_dev", "u", "P", "phi")})
    return s


@pytest.mark.parametrize("storage,components", [("fp32", 2), ("fp32", 1), ("fp16", 2), ("bf16", 2), ("fp16q", 2)])
def test_stacked_lattice_gives_the_same_bits(storage, components):
    print("[gpu-test] stores %s, %d component(s): one lattice and three stacked" % (storage, components), flush=True)
    with _sim(1, storage, components) as a, _sim(3, storage, components) as b:
        a.step(6)
        b.step(6)
        pairs = list(zip(a.moments(), b.moments()))
        if components == 2:
            pairs.append((a.phase(), b.phase()))
        for x, y in pairs:
            assert all(np.array_equal(x, y[..., k * NZ:(k + 1) * NZ, :, :]) for k in range(3))


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
def test_group_gives_the_same_bits(storage):
    from paper_2403_15773_amd.tslb import Group
    print("[gpu-test] stores %s: three lattices in one group and alone" % storage, flush=True)
    with _sim(1, storage, 2) as a:
        a.step(6)
        want = a.get_state_raw()
    sims = [_sim(1, storage, 2) for _ in range(3)]
    with Group(hbm_budget_bytes=1 << 30, max_domains=4) as grp:
        for s in sims:
            assert grp.admit(s, 6)
        left = len(sims)
        while left:
            left -= len(grp.poll())
    for s in sims:
        assert np.array_equal(s.get_state_raw(), want)
        s.close()
