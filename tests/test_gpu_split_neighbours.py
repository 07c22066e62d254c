"""A sample's rollout does not depend on the samples that share its wave (four of them): the
lane-split step takes a short or a long way through its sums by what any of the four touches,
and both have to give the same bits.  The same samples in other orders, beside calm and wild
neighbours (falling robots, feet and trunk against the box): costs bit for bit, and the whole
trajectory of every sample that stays finite."""
import numpy as np
import pytest

from paper_2409_10469_amd import workloads as W
from tests.parity_utils import box_contact_states, f32

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

K, H, NK = 256, 40, 6


def _start(scene, seed):
    if scene == W.SCENE_FREE_BOX:
        return box_contact_states(1, seed=seed)[0]
    x = W.initial_state(seed, scene)
    if scene == W.SCENE_STATIC_BOX:
        x[0] += 0.42
    if seed % 2:
        x[2] -= 0.12  # knees bent by the ground: more of the samples fall
    return f32(x)


@pytest.mark.parametrize("arith", ["fp32", "mixed", "fp64"])
@pytest.mark.parametrize("workload", [W.FLAT_WALK, W.TERRAIN_WALK, W.BOX_CLIMB, W.BOX_PUSH])
def test_rollout_is_the_same_beside_any_neighbours(workload, arith):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_10469_amd import binding as B
    dev = lambda a: torch.as_tensor(np.asarray(a, dtype=np.float32)).cuda().contiguous()
    for seed in range(3):
        print("case: neighbours", workload["name"], arith, seed, flush=True)
        p = W.params_dict(workload, seed, K=K, H=H, nk=NK, dt=0.01, sigma=(0.3, 0.8, 1.2)[seed], arith=arith, lanes=16)
        ctl = B.Controller(B.Model(W.model_dict(workload, seed)), p)
        ctl.set_nominal(dev(W.stance_knots(NK)))
        x0 = dev(_start(workload["scene"], seed))
        rng = np.random.default_rng(20 + seed)
        eps = rng.standard_normal((K, 12 * NK)) * np.where(rng.uniform(size=(K, 1)) < 0.5, 0.1, 1.0)
        costs, traj = [a.cpu().numpy() for a in ctl.rollout_batch(x0, eps=dev(eps), traj=True)]
        assert np.isfinite(costs).mean() > 0.5
        for _ in range(3):
            order = np.r_[0, 1 + rng.permutation(K - 1)]  # sample 0 is the nominal, without noise
            c, t = [a.cpu().numpy() for a in ctl.rollout_batch(x0, eps=dev(eps[order]), traj=True)]
            assert np.array_equal(c, costs[order])
            ok = np.isfinite(c)
            assert np.array_equal(t[ok], traj[order][ok])
