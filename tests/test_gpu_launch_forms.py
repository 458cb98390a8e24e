"""GPU tests of launch forms that depend on sizes: the update of a list of
solves past the memory-side cache, and the forcing network apart from the BR1
pass, each against a path that does not take the form."""
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


def _stage_bytes(N, P):
    """State, register, two sets of traces and the viscous fluxes."""
    n = P + 1
    return N ** 3 * (2 * 5 * n ** 3 + 6 * (5 + 5 + 4) * n ** 2) * 8


@pytest.mark.parametrize("P,sizes", [(6, (8, 16)), (8, (6, 13)), (3, (6, 14, 25))])
def test_list_past_the_cache(B, P, sizes):
    """Solves of one order whose stage data exceed 256 MB together and none
    alone, the largest joining the others and leaving them again, so that the
    list passes the limit both ways.  Each ends bitwise in the library's own
    stepping of it."""
    say("list past the cache", P, sizes)
    limit = 256 << 20
    assert sum(_stage_bytes(N, P) for N in sizes) > limit > max(_stage_bytes(N, P) for N in sizes)
    reqs = []
    for j, N in enumerate(sizes):
        m = B.Mesh(N, P, 200.0, Cs=0.1 if j else 0.0)
        q = m.field()
        B.dg_init_tgv(m, q)
        # the others run much longer than it takes to submit the largest
        steps = 20 if N == sizes[-1] else 600
        reqs.append((m, dict(Re=200.0, P=P, N=N, Cs=0.1 if j else 0.0, t_end=(steps - 0.5) * B.dg_stable_dt(m, q))))
    srv = B.Server(3 << 30, max_slots=8)
    ids = [srv.submit(want_state=True, **r) for _, r in reqs]
    srv.drain()
    total = 0
    for rid, (m, r) in zip(ids, reqs):
        _, st = srv.poll(rid)
        assert st.state == B.SOLVE_DONE, st.error
        total += st.n_steps
        q, k = m.field(), m.field(0.0)
        B.dg_init_tgv(m, q)
        B.dg_rk_step(m, q, k, st.dt, st.n_steps)
        torch.cuda.synchronize()
        assert np.array_equal(q.cpu().numpy().ravel(), srv.results(rid)[1]), r
    assert srv.stats()[1] < total   # they shared launches
    srv.close()


# sixteen-element blocks for both passes on half of the CUs (5) and on more
# (13: two launches), as many as there are CUs (16: one launch); hidden widths
# with and without kernels of their own
@pytest.mark.parametrize("N", [5, 13, 16])
@pytest.mark.parametrize("hidden,momenta", [((256, 256, 256), False), ((256, 256), True), ((96, 256), False)])
def test_corrected_step_against_its_parts(B, N, hidden, momenta):
    """A step with the forcing network at every stage against the stages put
    together from the residual and the forcing.  Float64 in another rounding
    order on both sides, as in the plain case: 32 eps of what the divergence
    sums, fluxes of up to 2 E times the derivative's (N / pi) PP^2.  The
    network sees states that differ by less than its bfloat16 rounding."""
    say("corrected step against its parts", N, hidden, momenta)
    io = (1, 2, 3) if momenta else (0, 1, 2, 3, 4)
    dims = [64 * len(io), *hidden, 64 * len(io)]
    norm = [1.0, 0.0, 0.0, 0.0, synthetic.TGV_ENERGY_LEVEL, 0.01, 1.0, 1.0, 1.0, 1.0] + [0.0] * 5 + [1e-2] * 5
    model = B.Model(dims, B.pack_params(synthetic.mlp_init(dims, seed=2)), norm, train=False,
                    activation="relu" if momenta else "tanh", in_vars=io, out_vars=io)
    m = B.Mesh(N, 3, 200.0)
    q, k, r = m.field(), m.field(0.0), m.field()
    B.dg_init_tgv(m, q)
    ref, reg, plain = q.clone(), torch.zeros_like(q), q.clone()
    dt = 0.5 * B.dg_stable_dt(m, q)
    for A, w in ((0.0, 1 / 3), (-5 / 9, 15 / 16), (-153 / 128, 8 / 15)):
        B.dg_residual(m, ref, r)
        B.nn_forcing(model, m, ref, r)
        reg = A * reg + dt * r
        ref += w * reg
    B.dg_rk_step(m, q, k, dt, 1, model=model)
    B.dg_rk_step(m, plain, m.field(0.0), dt, 1)
    eps = np.finfo(float).eps
    tol = 32 * eps * dt * 2 * float(ref[4].abs().max()) * (N / np.pi) * 4 ** 2
    for v in range(5):
        assert float((k[v] - reg[v]).abs().max()) <= tol
        assert float((q[v] - ref[v]).abs().max()) <= tol + 8 * eps * float(ref[v].abs().max())
        if v in io:
            assert float((plain[v] - ref[v]).abs().max()) > 1e3 * tol
