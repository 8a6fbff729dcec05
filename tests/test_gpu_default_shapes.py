"""The launch shapes a grid starts with: register-marching mu with several rows per wave or idle
lanes (bit for bit the LDS tiles), and plane transforms with n_x != n_z (the line passes to
rounding), at row counts and slab lengths that leave remainders."""
import numpy as np
import pytest

from workloads import workload
from workloads.shapes import GridSpec

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import paper_2601_05031_amd as P  # noqa: E402
from paper_2601_05031_amd import vs as V  # noqa: E402

FIELD_NAMES = ["phi", "mu", "omega_x", "omega_y", "omega_z", "psi_x", "psi_y", "psi_z"]
LINES = dict(adv_slab=4, va_maxb=1024, res_maxb=1024, seg_alt=0, mu_kind=0, mu_ni=8, plane=0)


def rel_l2(a, b):
    nb = float(np.linalg.norm(b))
    return float(np.linalg.norm(a - b)) / (nb if nb > 0 else 1.0)


def run(w, shapes, precision="fp64"):
    V.set_launch_shapes(w.grid.shape + (w.grid.h,), shapes)
    s = P.solver_for(w, precision=precision)
    s.step(w.dt, 3)
    f = s.fields()
    s.close()
    V.set_launch_shapes(w.grid.shape + (w.grid.h,), LINES)
    return f


def case(shape, name="vesicle32", mc=1):
    w = workload(name, grid=GridSpec(*shape), R0=min(shape) / 4.0, max_cycles=mc, wall_kind="couette", u0=-0.03,
                 u1=0.05, dt=5e-4)
    return w.with_(rate_V=10.0, k_A=1.0) if name == "vesicle32" else w


# rows of 4 .. 250 values: one to sixteen rows per wave, idle lanes, one, two and four z per lane
@pytest.mark.parametrize("shape", [(8, 5, 4), (12, 9, 16), (12, 11, 24), (16, 13, 32), (12, 21, 36), (16, 17, 48),
                                   (12, 10, 54), (8, 9, 72), (12, 11, 96), (8, 7, 108), (8, 9, 144), (6, 7, 216)])
@pytest.mark.parametrize("mu_kind,mu_ni", [(1, 3), (2, 5)])
def test_register_mu_is_bitwise_the_tile_mu(shape, mu_kind, mu_ni):
    for name in ("vesicle32", "droplet256"):
        w = case(shape, name)
        print(f"case mu {name} {shape} kind={mu_kind} ni={mu_ni}", flush=True)
        ref, got = run(w, LINES), run(w, dict(LINES, mu_kind=mu_kind, mu_ni=mu_ni))
        for k in FIELD_NAMES:
            assert np.array_equal(got[k], ref[k]), (name, k)


def test_register_mu_of_the_refined_mode():
    w = case((32, 12, 48), "droplet256", mc=3)
    ref, got = run(w, LINES, "fp32_refined"), run(w, dict(LINES, mu_kind=2, mu_ni=2), "fp32_refined")
    for k in FIELD_NAMES:
        assert np.array_equal(got[k], ref[k]), k


SIZES = (32, 48, 64, 96, 128)


# every pair of lengths; TOL: the plane and line forms differ by the pairing of the z lines (rounding)
@pytest.mark.parametrize("nx,nz", [(a, b) for a in SIZES for b in SIZES if a != b])
def test_oblong_planes_match_line_transforms(nx, nz):
    w = case((nx, 8, nz), mc=1 if nx < nz else 3)
    print(f"case plane {nx} x {nz}", flush=True)
    ref, got = run(w, LINES), run(w, dict(LINES, plane=1))
    errs = {k: rel_l2(got[k], ref[k]) for k in FIELD_NAMES}
    print("  " + " ".join(f"{k}={v:.1e}" for k, v in errs.items()), flush=True)
    assert max(errs.values()) <= 1e-12, errs


def test_a_batch_with_oblong_planes_is_bitwise_the_single_states():
    ws = [case((32, 9, 64)), case((32, 9, 64)).with_(kappa=0.6, seed=3), case((64, 9, 32))]
    shapes = dict(LINES, plane=1, mu_kind=2, mu_ni=2)
    refs = [run(w, shapes) for w in ws]
    for w in ws:
        V.set_launch_shapes(w.grid.shape + (w.grid.h,), shapes)
    solvers = [P.solver_for(w) for w in ws]
    b = V.Batch(solvers)
    b.step([w.dt for w in ws], 2)
    b.close()
    for s, w, ref in zip(solvers, ws, refs):
        s.step(w.dt, 1)
        got = s.fields()
        s.close()
        for k in FIELD_NAMES:
            assert np.array_equal(got[k], ref[k]), k


# the planes of lengths that share one kernel: idle lanes, several rounds of lines, short last rounds;
# one component (a Poisson solve, walls in the load) and three and six (a step), single and batched
ANY = [(16, 16), (16, 108), (24, 36), (36, 24), (54, 54), (72, 72), (72, 108), (108, 72), (32, 72), (108, 16)]


@pytest.mark.parametrize("nx,nz", ANY)
def test_planes_of_other_lengths_match_line_transforms(nx, nz):
    shape = (nx, 7, nz)
    w = case(shape, "droplet256" if nx > nz else "vesicle32", mc=1 if nx % 3 else 3)
    print(f"case plane any {shape}", flush=True)
    ref, got = run(w, LINES), run(w, dict(LINES, plane=1))
    errs = {k: rel_l2(got[k], ref[k]) for k in FIELD_NAMES}
    print("  " + " ".join(f"{k}={v:.1e}" for k, v in errs.items()), flush=True)
    assert max(errs.values()) <= 1e-12, errs
    rng = np.random.default_rng(nx + nz)
    f, u0 = rng.standard_normal(shape), rng.standard_normal(shape)
    sols = []
    for plane in (0, 1):
        V.set_launch_shapes(shape + (1.0,), dict(LINES, plane=plane))
        s = P.solver_for(w)
        ft, ut = torch.tensor(f, device="cuda"), torch.tensor(u0, device="cuda")
        code, cycles, rel = s.poisson_solve(ft, ut, rtol=1e-12, max_cycles=2)
        s.close()
        assert code == V.VS_OK and cycles == 1
        sols.append(ut.cpu().numpy())
    assert rel_l2(sols[1], sols[0]) <= 1e-12
    solvers = [P.solver_for(w), P.solver_for(w)]
    b = V.Batch(solvers)
    b.step([w.dt, w.dt], 2)
    b.close()
    for s in solvers:
        s.step(w.dt, 1)
        f3 = s.fields()
        s.close()
        for k in FIELD_NAMES:
            assert np.array_equal(f3[k], got[k]), k
    V.set_launch_shapes(shape + (1.0,), LINES)
