"""GPU tests of what the reductions say about a state that has blown up: a NaN
anywhere has to reach the error norm, the diagnostics and the time step."""
import numpy as np
import pytest

import synthetic
from helpers import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2207_11571_amd import binding
    binding.lib()
    return binding


def _state(N, P, seed):
    return torch.from_numpy(synthetic.random_state(N, P, seed=seed, momentum=0.3)).cuda()


# one block, and as many as there are elements
@pytest.mark.parametrize("N,P", [(1, 1), (3, 2), (9, 6)])
@pytest.mark.parametrize("where", ["first", "last", "middle", "reference", "all"])
def test_error_norm_keeps_nan(B, N, P, where):
    """The error norm of a momentum with a NaN in it is NaN; the others are
    the maxima of the same numbers in torch, exactly."""
    say("error norm with NaN", N, P, where)
    m = B.Mesh(N, P, 100.0)
    q, r = _state(N, P, 1), _state(N, P, 2)
    flat = q.view(5, -1)
    if where == "all":
        q.fill_(float("nan"))
    elif where == "reference":
        r.view(5, -1)[1, flat.shape[1] // 3] = float("nan")
    else:
        flat[2, {"first": 0, "last": flat.shape[1] - 1, "middle": flat.shape[1] // 2}[where]] = float("nan")
    err = torch.zeros(3, dtype=torch.float64, device="cuda")
    B.dg_error_inf(m, q, r, err)
    ref = (q - r).abs().view(5, -1)[1:4].amax(dim=1)
    assert torch.isnan(ref).any()
    assert np.array_equal(err.cpu().numpy(), ref.cpu().numpy(), equal_nan=True)
