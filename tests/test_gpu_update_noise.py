"""The update over the caller's noise where its rows are read in groups of 4 and where not: knot
counts that are and are not multiples of 4, one chunk of 8 knots and several, odd sample counts,
and noise at an address that is not a multiple of 16.

Tolerances: KNOT_TOL against the oracle, as every update.  The address decides only how the same
values are loaded: the same bits.
"""

import numpy as np
import pytest

from oracle import oracle as O
from paper_2409_10469_amd import workloads as W
from tests.parity_utils import KNOT_TOL, f32, round_model, round_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,nk,H,basis", [(1, 4, 25, 0), (1000, 4, 25, 0), (1025, 6, 25, 0), (2049, 8, 25, 0),
                                          (4097, 8, 25, 0), (70, 12, 12, 3), (1030, 20, 20, 3), (65, 10, 10, 3)])
def test_update_of_given_noise(K, nk, H, basis):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_10469_amd import binding as B

    p = round_params(dict(W.params_dict(W.FLAT_WALK, 0, K=K, nk=nk), H=H, basis=basis))
    ctl = B.Controller(B.Model(round_model(W.model_dict(W.FLAT_WALK, 0))), p)
    rng = np.random.default_rng(K + nk)
    mu = f32(rng.uniform(-0.5, 0.5, 12 * nk))
    eps = f32(rng.standard_normal((K, 12 * nk)))
    costs = f32(rng.uniform(0.5, 1.5, K))
    want, _, rc = O.update(p, costs, mu, eps)
    assert rc == 0

    def dev(a):
        return torch.as_tensor(np.asarray(a, dtype=np.float32)).cuda().contiguous()

    ctl.set_nominal(dev(mu))
    aligned = ctl.update(dev(costs), eps=dev(eps))
    shifted = torch.empty(K * 12 * nk + 1, device="cuda")[1:].reshape(K, 12 * nk)
    shifted.copy_(dev(eps))
    assert np.abs(aligned.cpu().numpy() - want).max() <= KNOT_TOL
    assert torch.equal(aligned, ctl.update(dev(costs), eps=shifted))
