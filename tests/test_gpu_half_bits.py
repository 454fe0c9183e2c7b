"""The bits of 16-bit stored moments.  A change of rounding anywhere in the step turns
into other roundings of stored words now and then, which travel; so the 16-bit paths
keep the order of their arithmetic, and their states after some steps from an exactly
representable start are pinned (digests of the step that sums populations, before its
populations crossed columns as records).  1 + rho' takes one rounding from the stored
word in FP16 and BF16."""
import hashlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NX, NY, NZ, STEPS = 100, 90, 96, 4
U = 0.06396  # 13 of the words up to 2 U^2 show a second rounding, more than with most scales
DIGESTS = {("fp16", 1): "b3a1583ca374e36b", ("fp16", 2): "71735eec817756b9",
           ("bf16", 1): "42766e7ec46027f5", ("bf16", 2): "86fcaac9cda1c5e1",
           ("fp16q", 1): "eeaea24cf7a1cc57", ("fp16q", 2): "2332c5ae16aecc5e"}


def _tri(n, period, shift):
    """A triangle wave in [-1, 1] of sixteenths: exact in every type."""
    i = (np.arange(n) * (64 // period) + shift) % 64
    return (np.abs(i - 32) - 16) / 16.0


def _state():
    def field(k, amp):
        x, y, z = _tri(NX, 32, 5 * k), _tri(NY, 16, 11 * k + 3), _tri(NZ, 32, 7 * k + 1)
        return (amp * (z[:, None, None] + 0.5 * y[None, :, None] * x[None, None, :])).astype(np.float32)

    # densities whose stored BF16 word makes 1 + rho' differ by how often it is rounded
    words = (np.arange(0x3C00, 0x4000, dtype=np.uint32) << 16).view(np.float32)  # up to 2 units of U^2
    s2 = np.float32(U * U)
    once = (1.0 + words.astype(np.float64) * float(s2)).astype(np.float32)
    words = words[once != np.float32(1.0) + words * s2]
    rho = (words * s2)[(np.abs(field(1, 8.0)).astype(np.int64) * 5) % words.size]
    phi = np.clip(0.5 + 0.75 * field(20, 1.0), 0.0, 1.0).astype(np.float32)
    return {"rho_dev": rho, "u": np.stack([field(k, 2.0 ** -6) for k in (2, 3, 4)]),
            "P": np.stack([field(k, 2.0 ** -14) for k in range(5, 11)]), "phi": phi}


def digest(storage, components):
    from paper_2403_15773_amd.tslb import Simulation
    st = _state()
    if components == 1:
        st["phi"] = np.zeros_like(st["phi"])
    with Simulation(nx=NX, ny=NY, nz=NZ, nu=2e-3, sigma=5e-4 if components == 2 else 0.0, width=3.0, eps=1e-4,
                    bc=(1, 1, 0, 0, 4, 3), components=components, storage=storage, u_scale=U) as s:
        s.set_state(**st)
        s.step(STEPS)
        assert s.diagnostics()["finite"]
        return hashlib.sha256(s.get_state_raw().tobytes()).hexdigest()[:16]


@pytest.mark.parametrize("components", [1, 2])
@pytest.mark.parametrize("storage", ["fp16", "bf16", "fp16q"])
def test_16_bit_states_keep_their_bits(storage, components):
    got = digest(storage, components)
    print("[gpu-test] %s, %d component(s): %s" % (storage, components, got), flush=True)
    assert got == DIGESTS[storage, components]
