"""Poisson solves of inputs at the edges of what the direct cycle accepts: right-hand sides that
nearly cancel against the wall terms, and arrays that are aligned as doubles only."""
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


# One FP32 cycle of the refined mode. f minus the wall terms is of order one and held in FP64; the
# cycle then loses the FP32 rounding (2^-24) times the condition of the column solves, at most
# 4 (M + 1)^2 / pi^2 <= 425 here: 2.5e-5, and the transforms' few roundings on top: 1e-4. Rounding f to
# FP32 before the subtraction would leave errors of 0.3 (half a unit of a float at 1e7) in rows 1 and M.
@pytest.mark.parametrize("shape", [(32, 9, 48), (48, 6, 96), (32, 33, 64), (64, 7, 32), (32, 8, 128), (32, 6, 192),
                                   (32, 7, 256)])
def test_wall_terms_are_subtracted_before_the_refined_cycle_rounds(shape):
    print(f"case refined poisson {shape}", flush=True)
    w = workload("droplet256", grid=GridSpec(*shape), R0=2.0, max_cycles=4)
    s = P.solver_for(w, precision="fp32_refined")
    rng = np.random.default_rng(11)
    b, u = rng.standard_normal(shape), rng.standard_normal(shape)
    u[:, [0, -1]] = 1e7 * (1.0 + 0.1 * u[:, [0, -1]])
    f = b.copy()
    f[:, 1] += u[:, 0]
    f[:, -2] += u[:, -1]
    ft, ut = torch.tensor(f, device="cuda"), torch.tensor(u, device="cuda")
    code, cycles, rel = s.poisson_solve(ft, ut, rtol=1e-10, max_cycles=1)
    s.close()
    assert code in (V.VS_OK, V.VS_E_NOCONV) and cycles == 1
    got = ut.cpu().numpy()
    assert np.array_equal(got[:, [0, -1]], u[:, [0, -1]])
    zero = np.zeros((shape[0], shape[2]))
    rhs = b[:, 1:-1].copy()
    rhs[:, 0] = f[:, 1] - u[:, 0]
    rhs[:, -1] = f[:, -2] - u[:, -1]
    e = rel_l2(got[:, 1:-1], O.poisson_solve(rhs, zero, zero, O.Grid(*shape)))
    print(f"  relL2={e:.2e} relres={rel:.2e}", flush=True)
    assert e <= 1e-4, e


def odd_view(a):
    """A copy of a at 8 bytes past a 16-byte boundary, inside guard values."""
    flat = torch.full((a.numel() + 3,), 7.0, dtype=torch.float64, device="cuda")
    first = 1 if flat.data_ptr() % 16 == 0 else 2
    v = flat[first:first + a.numel()].view(a.shape)
    v.copy_(a)
    assert v.data_ptr() % 16 == 8
    return flat, first, v


# planes with a kernel of their own, alone and several on a CU, planes of the shared kernel (both sizes),
# and line passes
@pytest.mark.parametrize("shape", [(128, 5, 128), (48, 7, 32), (24, 6, 36), (72, 3, 108), (192, 5, 64), (18, 6, 16)])
@pytest.mark.parametrize("entry", ["state", "noalloc"])
def test_arrays_aligned_as_doubles_only(shape, entry):
    print(f"case poisson alignment {entry} {shape}", flush=True)
    rng = np.random.default_rng(7)
    f, u = (torch.tensor(rng.standard_normal(shape), device="cuda") for _ in range(2))
    if entry == "state":
        s = P.solver_for(workload("droplet256", grid=GridSpec(*shape), R0=1.0, max_cycles=3))
        solve = s.poisson_solve
    else:
        solve = V.poisson_solve_noalloc
    ref = u.clone()
    assert solve(f, ref, rtol=1e-12, max_cycles=2)[:2] == (V.VS_OK, 1)
    ff, f0, fo = odd_view(f)
    uf, u0, uo = odd_view(u)
    assert solve(fo, uo, rtol=1e-12, max_cycles=2)[:2] == (V.VS_OK, 1)
    if entry == "state":
        s.close()
    assert torch.equal(uo, ref) and torch.equal(fo, f)
    for flat, first in ((ff, f0), (uf, u0)):
        assert (flat[:first] == 7.0).all() and (flat[first + f.numel():] == 7.0).all()
