"""20-row tiles with 16-bit moments, which the library takes on some lattices: four
geometry waves that form two pairs of rows a lane, the 13-pair gradient and 16-bit
stores.  Bitwise the result of 16-row tiles, alone and in a group, on lattices of odd
height below and above a tile, walled and periodic, with the shortest chunks and the
library's, and on one large enough to store without the non-temporal hint."""
import numpy as np
import pytest

from paper_2403_15773_amd import inputs

pytestmark = pytest.mark.gpu

HALF = ["fp16", "bf16", "fp16q"]
BOXES = {"low": ((37, 19, 9), (1, 1, 4, 1, 0, 0)), "odd": ((65, 41, 12), (4, 1, 1, 4, 1, 4)),
         "jet": ((48, 44, 30), (1, 1, 1, 1, 2, 3)), "periodic": ((40, 37, 11), (0,) * 6),
         "large": ((90, 81, 96), (0, 0, 4, 1, 0, 0))}  # 16 to 22 MiB, rows inside cache lines


def _sim(box, storage, rows, chunk):
    from paper_2403_15773_amd.tslb import Simulation
    (nx, ny, nz), bc = BOXES[box]
    s = Simulation(nx=nx, ny=ny, nz=nz, nu=0.02, sigma=0.005, width=3.0, bc=bc, eps=1e-4, storage=storage, inlet_u=0.04,
                   inlet_d=10.0, inlet_noise=0.02, seed=3)
    s.set_kernel("fused", chunk)
    s.set_tile(rows)
    assert s.tile_rows == rows
    st = inputs.smooth_state(nx, ny, nz)
    s.set_state(**{k: st[k] for k in ("rho_dev", "u", "P", "phi")})
    return s


@pytest.mark.parametrize("box", sorted(BOXES))
@pytest.mark.parametrize("storage", HALF)
def test_16_bit_moments_at_16_and_20_rows(storage, box):
    raw = []
    for rows, chunk in ((16, 0), (20, 0), (20, 1)):
        print("[gpu-test] %s %s: %d rows, chunk %d" % (box, storage, rows, chunk), flush=True)
        with _sim(box, storage, rows, chunk) as s:
            s.step(9)
            raw.append(s.get_state_raw())
            assert s.diagnostics()["finite"]
    assert np.array_equal(raw[0], raw[1]) and np.array_equal(raw[0], raw[2])


@pytest.mark.parametrize("storage", HALF)
def test_16_bit_members_of_20_rows_in_a_group(storage):
    from paper_2403_15773_amd.tslb import Group
    print("[gpu-test] %s: 20-row members in one group" % storage, flush=True)
    alone = []
    for box in ("odd", "large"):
        with _sim(box, storage, 16, 0) as s:
            s.step(7)
            alone.append(s.get_state_raw())
    sims = [_sim(box, storage, 20, 0) for box in ("odd", "large")]
    with Group(hbm_budget_bytes=1 << 30, max_domains=4) as grp:
        for s in sims:
            assert grp.admit(s, 7)
        left = len(sims)
        while left:
            left -= len(grp.poll())
    for s, want in zip(sims, alone):
        assert np.array_equal(s.get_state_raw(), want)
        s.close()
