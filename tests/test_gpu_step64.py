"""The FP64 step on the GPU at the states where its code branches, against the FP64 oracle:
trunk corners on the ground (a fallen robot) and in the static box, feet that touch ground and
box at once, the free box just inside and outside the bounding-sphere tests, coordinates off
the heightfield's edge, angular rates beyond the quaternion series' range, joint angles of many
turns.  Bar: the FP64 step's 1e-5 per block, from identical FP32 states."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2409_10469_amd import workloads as W
from tests.parity_utils import STEP_TOL, f32, round_model, round_params, step_error

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _edge_states(scene):
    rng = np.random.default_rng(50 + scene)
    xs = []

    def add(n, **at):
        for _ in range(n):
            x = W.initial_state(int(rng.integers(1000)), scene)
            x[19:37] = rng.normal(size=18) * np.r_[0.3, 0.3, 0.3, 1, 1, 1, np.full(12, 2.0)]
            q = np.r_[1.0, rng.normal(size=3) * at.get("tilt", 0.1)]
            x[3:7] = q / np.linalg.norm(q)
            for k, v in at.items():
                if k not in ("tilt", "rate", "turns"):
                    x[int(k[1:])] = v() if callable(v) else v
            if "rate" in at:
                w = rng.normal(size=3)
                x[22:25] = at["rate"] * w / np.linalg.norm(w)
            if "turns" in at:
                x[7:19] += at["turns"] * rng.integers(-1, 2, 12)
            xs.append(f32(x))

    far = lambda lo, hi: (lambda: rng.uniform(lo, hi))
    add(4)
    add(6, x2=far(0.03, 0.08), tilt=0.3)          # fallen: trunk corners on the ground
    add(3, rate=99.0)                             # half angle just under 1/2 (dt = 0.01) and over it
    add(3, rate=101.0)
    add(3, rate=700.0)
    add(3, turns=64 * 2 * np.pi)
    if scene == W.SCENE_HEIGHTFIELD:
        add(4, x0=far(1.4, 1.7), x1=far(-1.7, -1.4))
    if scene == W.SCENE_STATIC_BOX:
        add(8, x0=far(0.40, 0.48))                # front feet at the box's face, on the ground
        add(6, x0=far(0.45, 0.6), x2=far(0.2, 0.3), tilt=0.2)
    if scene == W.SCENE_FREE_BOX:
        for d in (0.34, 0.45, 0.53, 0.6, 0.8, 1.2):
            add(3, x37=d, x38=far(-0.1, 0.1))
        add(4, x37=0.36, x2=far(0.04, 0.1), tilt=0.2)
        add(3, x37=0.4, x39=0.16, x47=120.0)
    return np.array(xs)


@pytest.mark.parametrize("kernel", ["split", "quad"])
@pytest.mark.parametrize("workload", [W.FLAT_WALK, W.TERRAIN_WALK, W.BOX_CLIMB, W.BOX_PUSH])
def test_fp64_step_at_its_branches(workload, kernel):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_10469_amd import binding as B
    print("case: fp64 step branches", workload["name"], kernel, flush=True)
    md = round_model(W.model_dict(workload, 0))
    p = round_params(W.params_dict(workload, 0, dt=0.01))
    orc, model = O.Oracle(md), B.Model(md)
    xs = _edge_states(workload["scene"])
    us = f32(np.tile(W.STANCE_JOINTS, 4) + np.random.default_rng(3).uniform(-0.3, 0.3, (len(xs), 12)))
    dev = lambda a: torch.as_tensor(np.asarray(a, dtype=np.float32)).cuda().contiguous()
    if kernel == "quad":
        got = model.sim_step(dev(xs), dev(us), p["kp"], p["kd"], p["dt"]).cpu().numpy().astype(np.float64)
    else:
        ctl = B.Controller(model, dict(p, K=1, H=1, nk=2, sigma=0.0, arith="fp64", lanes=16))
        eps = dev(np.zeros((1, 24)))
        got = []
        for x, u in zip(xs, us):
            ctl.set_nominal(dev(np.repeat(u, 2)))
            _, traj = ctl.rollout_batch(dev(x), eps=eps, traj=True)
            got.append(traj[0, 1].cpu().numpy().astype(np.float64))
        got = np.array(got)
    want = np.array([orc.step(x, u, p["kp"], p["kd"], p["dt"])[0] for x, u in zip(xs, us)])
    err = step_error(got, want, box=workload["scene"] == W.SCENE_FREE_BOX)
    print("worst block error %.2e at state %d of %d" % (err.max(), int(err.argmax()), len(xs)))
    assert err.max() <= STEP_TOL, (err.max(), int(err.argmax()))
