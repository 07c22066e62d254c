"""The FP32 and mixed lane-split steps at the states where the step's code branches (fallen
robots, feet on ground and box at once, the box just inside and outside the bounding-sphere
tests, coordinates off the heightfield), against the FP64 oracle and the bounds derived from it
for these arithmetics (parity_utils.fp32_step_bound, mixed_step_bound)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2409_10469_amd import workloads as W
from tests.parity_utils import f32, fp32_step_bound, mixed_step_bound, round_model, round_params, step_error
from tests.test_gpu_step64 import _edge_states

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("arith,bound", [("fp32", fp32_step_bound), ("mixed", mixed_step_bound)])
@pytest.mark.parametrize("workload", [W.FLAT_WALK, W.TERRAIN_WALK, W.BOX_CLIMB, W.BOX_PUSH])
def test_step_at_its_branches(workload, arith, bound):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_10469_amd import binding as B
    print("case: step branches", workload["name"], arith, flush=True)
    md = round_model(W.model_dict(workload, 0))
    p = round_params(W.params_dict(workload, 0, dt=0.01))
    orc = O.Oracle(md)
    ctl = B.Controller(B.Model(md), dict(p, K=1, H=1, nk=2, sigma=0.0, arith=arith, lanes=16))
    xs = _edge_states(workload["scene"])
    us = f32(np.tile(W.STANCE_JOINTS, 4) + np.random.default_rng(3).uniform(-0.3, 0.3, (len(xs), 12)))
    dev = lambda a: torch.as_tensor(np.asarray(a, dtype=np.float32)).cuda().contiguous()
    eps = dev(np.zeros((1, 24)))
    got = []
    for x, u in zip(xs, us):
        ctl.set_nominal(dev(np.repeat(u, 2)))
        got.append(ctl.rollout_batch(dev(x), eps=eps, traj=True)[1][0, 1].cpu().numpy().astype(np.float64))
    want = np.array([orc.step(x, u, p["kp"], p["kd"], p["dt"])[0] for x, u in zip(xs, us)])
    err = step_error(np.array(got), want, box=workload["scene"] == W.SCENE_FREE_BOX)
    lim = np.array([bound(orc, x, u, p["kp"], p["kd"], p["dt"]) for x, u in zip(xs, us)])
    print("step error: max %.2e median %.2e; worst error / bound %.3f at state %d of %d"
          % (err.max(), np.median(err), (err / lim).max(), int((err / lim).argmax()), len(xs)))
    assert (err <= lim).all(), (int((err / lim).argmax()), (err / lim).max())
