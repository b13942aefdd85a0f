"""The dense kernels of the contact solve at the edges of their tiles, through one FP64 step against the
oracle: a slab landing on the ground while it slides couples all of its bottom vertices, and its friction
makes most rows part of the capacitance system.  Contacts per env: below, at and above one 16-column panel
(14, 16, 33), one panel row per thread and more (256, 272 contacts; up to three rows each in the LU).
Positions within 1e-9 of the body's extent, the bound of the FP64 parity tests (the contact solve stops at
1e-12 m)."""
import numpy as np
import pytest

from oracle import flash_oracle as O
from paper_2604_17513_amd import scenes

pytestmark = pytest.mark.gpu


def _slab(nx, nz):
    rest, tets = scenes.hex_lattice(nx, 1, nz, (0.01 * nx, 0.01, 0.01 * nz), (0.0, 0.0, 0.0))
    env = scenes.EnvDesc(scenes.TET, rest, tets, density=1000.0, young=2e5, poisson=0.35, mu=0.4)
    x0 = rest + np.array([0.0, 5e-4, 0.0])
    v0 = np.zeros_like(rest) + np.array([0.2, -0.3, 0.05])
    return scenes.Scene([env], [x0], [v0], [[scenes.ground()]], scenes.Params(lg_iterations=3), name="slab")


# A base of 14 contacts (14 mod 16) meets the known defect of the base inverse that flash_dense.h states:
# four entries of a 14-column last block are not updated, the inverse is wrong and the solve may diverge.
DEFECT = pytest.mark.xfail(reason="base inverse of 14 mod 16 contacts is inexact (known defect, results kept)",
                           strict=False)


@pytest.mark.parametrize("nx,nz,contacts", [pytest.param(1, 6, 14, marks=DEFECT), (3, 3, 16), (2, 10, 33), (15, 15, 256), (15, 16, 272)])
@pytest.mark.parametrize("fused", [False, True])
def test_landing_slab_matches_oracle(nx, nz, contacts, fused):
    from paper_2604_17513_amd import flash as F
    sc = _slab(nx, nz)
    oe = O.precompute(sc.envs[0], sc.params.h)
    b = F.from_scene(sc, precision=F.FLASH_FP64, fused_lg=fused)
    for s in range(2):
        x0, v0 = b.get_state()
        obs = b.get_obstacles(0)
        b.step(1)
        x1, _ = b.get_state()
        p = b.phase_times()
        c = b.contacts(0)
        ref = O.step(oe, x0, v0, obs, sc.params, tol=1e-12)
        L = np.linalg.norm(sc.envs[0].rest_x.max(0) - sc.envs[0].rest_x.min(0))
        err, tol = np.abs(x1 - ref.x).max(), 1e-9 * max(np.abs(ref.x).max(), L)
        print(f"{nx}x{nz} fused {fused} step {s}: {len(c['vertex'])} contacts, {p['cap_rows_max']:.0f} rows at most, "
              f"max|dq| {err:.2e} (tol {tol:.2e})", flush=True)
        assert len(c["vertex"]) == contacts or s > 0
        assert p["n_factor"] >= 1 or s > 0
        assert err <= tol
