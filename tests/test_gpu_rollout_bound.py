"""rollout_gradient refuses a rollout whose gamma_A takes the forward-Euler bound below dt on the way,
wherever in a checkpoint segment that happens."""
import numpy as np
import pytest

from workloads import workload
from workloads.shapes import GridSpec

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import paper_2601_05031_amd as P  # noqa: E402
from paper_2601_05031_amd import vs as V  # noqa: E402

# the bound is 1.6034e-3 at gamma_A = 0 and 1.570e-3 at the gamma_A = -0.18 that one step of this dt reaches
DT = 1.598e-3


def solver(**kw):
    return P.solver_for(workload("vesicle32", grid=GridSpec(16, 13, 18), R0=4.0, rate_V=3.0, **kw))


@pytest.mark.parametrize("every", [1, 2, 3, 4, 10])
def test_a_bound_that_falls_below_dt_inside_a_segment(every):
    s = solver(k_A=1e3)
    s.step(DT, 1)
    with pytest.raises(V.VsError) as e:
        s.step(DT, 1)
    assert e.value.code == V.VS_E_UNSTABLE
    s.close()
    s = solver(k_A=1e3)
    print(f"case rollout bound every={every}", flush=True)
    with pytest.raises(V.VsError) as e:
        P.rollout_gradient(s, DT, 4, torch.zeros(s.shape, dtype=torch.float64, device="cuda"), every)
    assert e.value.code == V.VS_E_UNSTABLE
    assert s.scalars()["step"] == 1
    s.close()


def test_the_segments_do_not_change_the_gradient():
    """One call a segment (k_A = 0) and one a step give the same bits."""
    outs = []
    for every in (1, 3, 5):
        s = solver(k_A=0.0)
        L, dk, ds, a = P.rollout_gradient(s, 5e-4, 5, torch.zeros(s.shape, dtype=torch.float64, device="cuda"), every)
        outs.append((L, dk, ds, a.cpu().numpy()))
        s.close()
    for o in outs[1:]:
        assert o[:3] == outs[0][:3] and np.array_equal(o[3], outs[0][3])
