"""Column solves at every segment length: row counts M = ny - 2 with all segments long and with some
short, for one scalar problem (vs_poisson_solve) and for the vorticity and stream-vector pair (the
initial state's flow), against the oracle."""
import numpy as np
import pytest

import oracle as O
from workloads import workload
from workloads.shapes import GridSpec

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import paper_2601_05031_amd as P  # noqa: E402
from paper_2601_05031_amd import vs as V  # noqa: E402


def rel_l2(a, b):
    nb = float(np.linalg.norm(b))
    return float(np.linalg.norm(a - b)) / (nb if nb > 0 else 1.0)


# S segments of L rows: all long, all but one long, and one long
ROWS = sorted({m for S, lengths in ((4, range(5, 17)), (8, range(9, 17)), (16, range(9, 17))) for L in lengths
               for m in (S * L, S * L - 1, S * (L - 1) + 1)} | {4, 5, 16, 256, 257})


@pytest.mark.parametrize("nx,nz", [(8, 6), (32, 16)])
def test_every_segment_length(nx, nz):
    worst = 0.0
    for M in ROWS:
        shape = (nx, M + 2, nz)
        w = workload("vesicle32", grid=GridSpec(*shape), shape="sphere", R0=2.0, wall_kind="couette", u0=-0.03,
                     u1=0.05, max_cycles=1, center=(0.45 * nx, 0.5 * (M + 1), 0.4 * nz))
        print(f"case columns {shape}", flush=True)
        s = P.solver_for(w)
        got = s.fields()
        rng = np.random.default_rng(M)
        f, u0 = rng.standard_normal(shape), rng.standard_normal(shape)
        ft, ut = torch.tensor(f, device="cuda"), torch.tensor(u0, device="cuda")
        code, cycles, rel = s.poisson_solve(ft, ut, rtol=1e-12, max_cycles=2)
        s.close()
        g = O.Grid(*shape)
        e = rel_l2(ut.cpu().numpy()[:, 1:-1], O.poisson_solve(f[:, 1:-1], u0[:, 0], u0[:, -1], g))
        assert code == V.VS_OK and e <= 1e-12, (M, e)
        p = O.Params(model=w.model, kappa=w.kappa, eps=w.eps)
        ref = O.init_state(g, O.Walls(w.wall_kind, w.u0, w.u1), p, w.phi0())
        for c, ax in enumerate("xyz"):
            for name, r in (("omega_", ref.omega[c]), ("psi_", ref.psi[c])):
                # the FP64 bar of the step parity tests, on the scale of the whole vector field
                scale = float(np.linalg.norm(ref.omega if name == "omega_" else ref.psi))
                d = float(np.linalg.norm(got[name + ax] - r)) / scale
                worst = max(worst, d)
                assert d <= 1e-9, (M, name + ax, d)
    print(f"  worst {worst:.1e}", flush=True)
