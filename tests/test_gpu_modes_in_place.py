"""The FP64 flow pass with its modes kept in the omega and psi fields (grids whose 18 fields pass
the Infinity Cache), for the kernels the full-size parity workloads do not reach: general transform
lengths and the two-lane column solve of tall channels."""
import numpy as np
import pytest

import oracle as O
from workloads import workload
from workloads.shapes import GridSpec

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import paper_2601_05031_amd as P  # noqa: E402

TOL = 1e-9   # the FP64 bar of the step parity tests


def rel_l2(a, b):
    nb = float(np.linalg.norm(b))
    return float(np.linalg.norm(a - b)) / (nb if nb > 0 else 1.0)


@pytest.mark.parametrize("shape,mc", [((162, 72, 162), 1), ((162, 72, 162), 3), ((48, 260, 162), 1)])
def test_large_ragged_grids_match_the_oracle(shape, mc):
    w = workload("vesicle32", grid=GridSpec(*shape), R0=12.0, rate_V=10.0, k_A=1.0, wall_kind="couette",
                 u0=-0.03, u1=0.05, dt=5e-4, max_cycles=mc, nsteps=2)
    print(f"case modes in place {shape} mc={mc}", flush=True)
    s = P.solver_for(w)
    s.step(w.dt, w.nsteps)
    got = s.fields()
    s.close()
    p = O.Params(model=w.model, kappa=w.kappa, eps=w.eps, rate_V=w.rate_V, k_A=w.k_A)
    ref = O.run(O.Grid(*shape), O.Walls(w.wall_kind, w.u0, w.u1), p, w.phi0(), w.dt, w.nsteps)
    refs = {"phi": ref.phi, "mu": ref.mu}
    for c, ax in enumerate("xyz"):
        refs["omega_" + ax] = ref.omega[c]
        refs["psi_" + ax] = ref.psi[c]
    errs = {k: rel_l2(got[k], refs[k]) for k in refs}
    print("  " + " ".join(f"{k}={v:.1e}" for k, v in errs.items()), flush=True)
    assert max(errs.values()) <= TOL, errs
