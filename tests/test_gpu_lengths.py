"""Steps at the transform lengths of the two-pass register form beyond the power-of-two ones: the
three- and six-component passes against the oracle, and a batch of them against single states. The
refined mode keeps to its own list of lengths."""
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

FIELD_NAMES = ["phi", "mu", "omega_x", "omega_y", "omega_z", "psi_x", "psi_y", "psi_z"]
TOL = 1e-9   # the FP64 bar of the step parity tests
# every new length along x and along z; row counts whose transforms end in a partial block
SHAPES = [(16, 10, 24), (24, 7, 36), (36, 9, 54), (54, 13, 72), (72, 12, 108), (108, 7, 144), (144, 8, 162),
          (162, 6, 216), (216, 6, 16)]


def rel_l2(a, b):
    nb = float(np.linalg.norm(b))
    return float(np.linalg.norm(a - b)) / (nb if nb > 0 else 1.0)


def case(shape):
    return workload("vesicle32", grid=GridSpec(*shape), R0=2.5, rate_V=10.0, k_A=1.0, wall_kind="couette", u0=-0.03,
                    u1=0.05, dt=5e-4, max_cycles=1)


@pytest.mark.parametrize("shape", SHAPES)
def test_steps_match_the_oracle(shape):
    w = case(shape)
    print(f"case lengths {shape}", flush=True)
    s = P.solver_for(w)
    s.step(w.dt, 2)
    got = s.fields()
    s.close()
    p = O.Params(model=w.model, kappa=w.kappa, eps=w.eps, rate_V=w.rate_V, k_A=w.k_A)
    ref = O.run(O.Grid(*shape), O.Walls(w.wall_kind, w.u0, w.u1), p, w.phi0(), w.dt, 2)
    refs = dict(zip(FIELD_NAMES, [ref.phi, ref.mu, *ref.omega, *ref.psi]))
    errs = {k: rel_l2(got[k], refs[k]) for k in refs}
    print("  " + " ".join(f"{k}={v:.1e}" for k, v in errs.items()), flush=True)
    assert max(errs.values()) <= TOL, errs


def test_a_batch_of_them_is_bitwise_the_single_states():
    ws = [case(shape) for shape in SHAPES[2:6]] + [case(SHAPES[2]).with_(seed=5, kappa=0.7)]
    for w in ws:
        V.set_launch_shapes(w.grid.shape + (w.grid.h,), dict(adv_slab=4, va_maxb=1024, res_maxb=1024, seg_alt=0,
                                                             mu_kind=0, mu_ni=8, plane=0))
    refs = []
    for w in ws:
        s = P.solver_for(w)
        s.step(w.dt, 4)
        refs.append(s.fields())
        s.close()
    solvers = [P.solver_for(w) for w in ws]
    b = V.Batch(solvers, nstreams=2)
    b.step([w.dt for w in ws], 4)
    b.close()
    for s, ref in zip(solvers, refs):
        got = s.fields()
        s.close()
        for k in FIELD_NAMES:
            assert np.array_equal(got[k], ref[k]), k


@pytest.mark.parametrize("shape", [(72, 12, 64), (64, 12, 108), (16, 12, 32)])
def test_the_refined_mode_still_refuses_them(shape):
    with pytest.raises(V.VsError) as e:
        P.solver_for(case(shape), precision="fp32_refined", max_cycles=2)
    assert e.value.code == V.VS_E_UNSUPPORTED
