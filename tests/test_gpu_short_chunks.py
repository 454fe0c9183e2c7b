"""The shortest z chunks of the fused step (1 to 3 planes a workgroup), which the
library takes by itself on lattices of a few tiles: each chunk starts and ends
its pipeline within the reach of the gradient stencil, next to a wall or across
the period.  The result is bitwise the one of a chunk that covers the lattice."""
import numpy as np
import pytest

from paper_2403_15773_amd import inputs

pytestmark = pytest.mark.gpu

SIZE = (37, 18, 11)  # two tiles in x and y (the second pulled inward), odd in z


def _params(path):
    nx, ny, nz = SIZE
    if path == "vortex":
        return dict(nx=nx, ny=ny, nz=nz, nu=0.01, sigma=0.0, width=3.0, bc=(0,) * 6, components=1)
    p = inputs.jet_params(nx, ny, nz, d=8.0, u=0.05, re=200.0, we=50.0, seed=5)
    if path == "vdjet":
        p.update(density_a=10.0, density_b=1.0, nu_a=0.01, nu_b=0.01)
    if path == "box":
        p.update(bc=(0, 0, 4, 1, 0, 0))
    return p


def _state():
    st = inputs.smooth_state(*SIZE)
    return {k: st[k] for k in ("rho_dev", "u", "P", "phi")}


def _sim(path, storage, chunk):
    from paper_2403_15773_amd.tslb import Simulation
    s = Simulation(**_params(path), eps=1e-4, storage=storage)
    s.set_kernel("fused", chunk)
    st = _state()
    if path == "vortex":
        st["phi"] = np.zeros_like(st["phi"])
    s.set_state(**st)
    return s


@pytest.mark.parametrize("path,storage", [("jet", "fp32"), ("box", "fp32"), ("vortex", "fp32"), ("vdjet", "fp32"),
                                          ("jet", "fp16"), ("box", "bf16"), ("vortex", "fp16q")])
def test_short_chunks_give_the_same_bits(path, storage):
    ref = None
    for chunk in (SIZE[2], 1, 2, 3, 0):
        print("[gpu-test] short chunks %s %s: %d planes" % (path, storage, chunk), flush=True)
        with _sim(path, storage, chunk) as s:
            s.step(9)
            got = s.get_state_raw()
        if ref is None:
            ref = got
        assert np.array_equal(ref, got), chunk


def test_group_of_small_lattices_gives_the_same_bits():
    from paper_2403_15773_amd.tslb import Group
    print("[gpu-test] short chunks: two small lattices in one group", flush=True)
    alone = []
    for path in ("jet", "box"):
        with _sim(path, "fp32", SIZE[2]) as s:
            s.step(9)
            alone.append(s.get_state_raw())
    sims = [_sim(path, "fp32", 0) for path in ("jet", "box")]
    with Group(hbm_budget_bytes=1 << 30, max_domains=4) as grp:
        for s in sims:
            assert grp.admit(s, 9)
        left = len(sims)
        while left:
            left -= len(grp.poll())
    for s, want in zip(sims, alone):
        assert np.array_equal(s.get_state_raw(), want)
        s.close()
