"""The reverse step at the edges of its pair kernels: rows of an odd number of pairs and of few,
walks with a short last slab, one row per tile, and adj_prev 8-byte but not 16-byte aligned, against the oracle."""
import numpy as np
import pytest

import oracle as O
from oracle import adjoint as AD
from workloads import workload
from workloads.shapes import GridSpec

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import paper_2601_05031_amd as P  # noqa: E402


@pytest.mark.parametrize("model", ["bending", "cahn_hilliard"])
@pytest.mark.parametrize("shape", [(16, 9, 4), (12, 8, 18), (54, 40, 6), (36, 70, 108), (96, 40, 64), (6, 7, 512)])
def test_pairs(shape, model):
    print(f"case grad-step {shape} {model}", flush=True)
    nx, ny, nz = shape
    name = "vesicle32" if model == "bending" else "droplet256"
    w = workload(name, grid=GridSpec(*shape), R0=max(1.0, min(shape) / 4.0), wall_kind="couette", u0=-0.03,
                 u1=0.05, rate_V=2.0, k_A=0.7 if model == "bending" else 0.0, max_cycles=1,
                 center=(0.45 * nx, 0.5 * (ny - 1), 0.4 * nz))
    s = P.solver_for(w)
    a = np.random.default_rng(5).standard_normal(shape)
    at = torch.tensor(a, device="cuda")
    flat = torch.full((nx * ny * nz + 2,), 7.0, dtype=torch.float64, device="cuda")
    odd = flat[1:-1].view(shape)
    even = torch.empty(shape, dtype=torch.float64, device="cuda")
    terms = s.grad_step(w.dt, at, odd)
    assert terms == s.grad_step(w.dt, at, even)
    s.close()
    assert torch.equal(odd, even) and flat[0] == 7.0 and flat[-1] == 7.0
    g = O.Grid(*w.grid.shape, h=w.grid.h)
    walls = O.Walls(w.wall_kind, w.u0, w.u1)
    p = O.Params(model=w.model, eta=w.eta, mobility=w.mobility, eps=w.eps, kappa=w.kappa, sigma=w.sigma,
                 gamma0=w.gamma0, rate_V=w.rate_V, k_A=w.k_A, bend_scale=w.bend_scale)
    prev, kappa, scale = AD.grad_step(O.init_state(g, walls, p, w.phi0()), a, w.dt, g, walls, p)
    got = even.cpu().numpy()
    # the bar of the reverse step: 1e-9 relative
    assert np.linalg.norm(got - prev) <= 1e-9 * np.linalg.norm(prev - a)
    assert terms[0] == pytest.approx(kappa if model == "bending" else 0.0, rel=1e-9, abs=1e-15)
    assert terms[1] == pytest.approx(scale, rel=1e-9, abs=1e-15)
