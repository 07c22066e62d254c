"""The FP64 step at joint angles far outside the range of a two-part reduction of pi/2 (a
diverging rollout, or a start state that holds them), against the FP64 oracle: the sine and
cosine of any finite FP32 angle are those of the angle itself.  Angles on both sides of 2^40,
where the reduction changes, up to the largest; no position gain, so that the angles act
through the kinematics alone.  The calf's angle is the sum of flexion and knee rounded to
double, as the step defines it; the oracle, which turns by one after the other, is given the
knee angle of that sum (from the host library's sines and cosines, which hold for any angle).  Bar: the FP64 step's 1e-5 per block, from identical FP32
states."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2409_10469_amd import workloads as W
from tests.parity_utils import STEP_TOL, f32, round_model, round_params, step_error

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ANGLES = [3.0, 1e3, 1e6, 1e9, 2.0 ** 39, 2.0 ** 40, np.nextafter(np.float32(2.0 ** 40), np.float32(np.inf)), 2e12, 1e13,
          2.0 ** 53, 2.0 ** 54, 3e16, 1e20, 7e25, 1e30, 2.0 ** 100, 3e38]


def _states(scene):
    rng = np.random.default_rng(70 + scene)
    xs = []
    for a in ANGLES:
        for _ in range(4):
            x = W.initial_state(int(rng.integers(1000)), scene)
            x[19:37] = rng.normal(size=18) * np.r_[0.3, 0.3, 0.3, 1, 1, 1, np.full(12, 2.0)]
            q = np.r_[1.0, 0.1 * rng.normal(size=3)]
            x[3:7] = q / np.linalg.norm(q)
            j = rng.permutation(12)[:rng.integers(1, 7)]
            x[7 + j] = a * rng.choice([-1.0, 1.0], len(j)) * (1.0 if a > 1e38 else rng.uniform(1.0, 1.0 + 1e-6, len(j)))
            xs.append(f32(x))
    return np.array(xs)


@pytest.mark.parametrize("kernel", ["split", "quad"])
@pytest.mark.parametrize("workload", [W.FLAT_WALK, W.BOX_PUSH])
def test_fp64_step_at_far_joint_angles(workload, kernel):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_10469_amd import binding as B
    print("case: fp64 step at far angles", workload["name"], kernel, flush=True)
    md = round_model(W.model_dict(workload, 0))
    p = round_params(W.params_dict(workload, 0, dt=0.01, kp=0.0))
    orc, model = O.Oracle(md), B.Model(md)
    xs = _states(workload["scene"])
    u = f32(np.tile(W.STANCE_JOINTS, 4))
    dev = lambda a: torch.as_tensor(np.asarray(a, dtype=np.float32)).cuda().contiguous()
    if kernel == "quad":
        got = model.sim_step(dev(xs), dev(np.tile(u, (len(xs), 1))), 0.0, p["kd"], p["dt"]).cpu().numpy()
    else:
        ctl = B.Controller(model, dict(p, K=1, H=1, nk=2, sigma=0.0, arith="fp64", lanes=16))
        eps = dev(np.zeros((1, 24)))
        ctl.set_nominal(dev(np.repeat(u, 2)))
        got = np.array([ctl.rollout_batch(dev(x), eps=eps, traj=True)[1][0, 1].cpu().numpy() for x in xs])
    xr = xs.copy()
    turn = lambda a: np.arctan2(np.sin(a), np.cos(a))
    xr[:, 9:19:3] = turn(xs[:, 8:19:3] + xs[:, 9:19:3]) - turn(xs[:, 8:19:3])
    want = np.array([orc.step(x, u, 0.0, p["kd"], p["dt"])[0] for x in xr])
    want[:, 7:19] = xs[:, 7:19] + p["dt"] * want[:, 25:37]
    assert np.isfinite(want).all()
    err = step_error(got.astype(np.float64), want, box=workload["scene"] == W.SCENE_FREE_BOX)
    print("worst block error %.2e at angle %.3g" % (err.max(), ANGLES[int(err.argmax()) // 4]))
    assert err.max() <= STEP_TOL, (err.max(), ANGLES[int(err.argmax()) // 4])
