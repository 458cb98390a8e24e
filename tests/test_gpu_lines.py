"""GPU tests of the line kernels' edges: groups of several small elements that
the mesh does not fill, every order with and without viscous fluxes and the
closure, and lists of solves of different sizes in one launch.

Tolerance of the parity checks: float64 on both sides, summation order only --
1e-12 relative L2 per variable, as for the other residual and step checks.
"""
import numpy as np
import pytest

import synthetic
from helpers import field_parity, say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2207_11571_amd import binding
    binding.lib()
    return binding


# P = 1: groups of five elements (8 = 5 + 3, 1); P = 2: of two (27, 1)
@pytest.mark.parametrize("N,P", [(2, 1), (1, 1), (3, 2), (1, 2), (2, 3), (2, 4), (2, 5), (2, 6), (2, 7), (2, 8)])
@pytest.mark.parametrize("Cs,viscous", [(0.0, True), (0.1, True), (0.0, False)])
def test_stage_kernels(B, N, P, Cs, viscous):
    """Residual and two Runge-Kutta steps against the oracle."""
    from oracle import dg, rk
    say("stage kernels", N, P, Cs, viscous)
    prm = dg.Params(N=N, P=P, Re=100.0, Cs=Cs, viscous=viscous)
    q0 = synthetic.random_state(N, P, seed=40 + P, momentum=0.3)
    m = B.Mesh(N, P, 100.0, Cs=Cs, viscous=viscous)
    q = torch.from_numpy(q0).cuda()
    k = m.field(float("nan"))   # contents on entry are ignored
    out = m.field(0.0)
    B.dg_residual(m, q, out)
    dt = 0.2 * dg.stable_dt(dg.to_blocks(q0, N, P), prm)
    B.dg_rk_step(m, q, k, dt, 2)
    torch.cuda.synchronize()
    ref = dg.to_flat(dg.residual(dg.to_blocks(q0, N, P), prm))
    l2, li = field_parity(out.cpu().numpy(), ref, 1e-12)
    assert np.all(l2 < 1e-12) and np.all(li < 1e-11), (l2, li)
    ref = dg.to_flat(rk.integrate(dg.to_blocks(q0, N, P), dt, 2, lambda s, t: dg.residual(s, prm)))
    l2, li = field_parity(q.cpu().numpy(), ref, 1e-12)
    assert np.all(l2 < 1e-12) and np.all(li < 1e-11), (l2, li)


@pytest.mark.parametrize("P", [1, 2, 4, 5, 7])
def test_list_of_solves(B, P):
    """Solves of one order, different meshes and closures, batched by the
    server: each ends bitwise in the library's own stepping of it."""
    say("list of solves", P)
    reqs = [dict(Re=200.0, N=3, Cs=0.0), dict(Re=30.0, N=2, Cs=0.1), dict(Re=1600.0, N=1, Cs=0.0)]
    srv = B.Server(64 << 20, max_slots=8)
    t_end = 0.02 if P < 4 else 0.005
    ids = [srv.submit(Re=r["Re"], P=P, N=r["N"], t_end=t_end, Cs=r["Cs"], want_state=True) for r in reqs]
    srv.drain()
    for rid, r in zip(ids, reqs):
        _, st = srv.poll(rid)
        assert st.state == B.SOLVE_DONE, st.error
        m = B.Mesh(r["N"], P, r["Re"], Cs=r["Cs"])
        q, k = m.field(), m.field(0.0)
        B.dg_init_tgv(m, q)
        B.dg_rk_step(m, q, k, st.dt, st.n_steps)
        torch.cuda.synchronize()
        assert np.array_equal(q.cpu().numpy().ravel(), srv.results(rid)[1])
    srv.close()


# sixteen-element blocks: one, not full (1, 8, 27), several (125), and more
# than half of the CUs (2197: two launches); hidden widths with and without
# kernels of their own
@pytest.mark.parametrize("N", [1, 2, 3, 5, 13])
@pytest.mark.parametrize("hidden,momenta", [((256, 256, 256), False), ((256,), True), ((96, 256), False)])
def test_network_beside_br1_pass(B, N, hidden, momenta):
    """Steps with the forcing network, whose BR1 pass may share the network's
    launch, against the measurement twin, which launches them one after the
    other: bitwise."""
    say("network beside BR1 pass", N, hidden, momenta)
    io = (1, 2, 3) if momenta else (0, 1, 2, 3, 4)
    dims = [64 * len(io), *hidden, 64 * len(io)]
    norm = [1.0, 0.0, 0.0, 0.0, synthetic.TGV_ENERGY_LEVEL, 0.01, 1.0, 1.0, 1.0, 1.0] + [0.0] * 5 + [1e-3] * 5
    model = B.Model(dims, B.pack_params(synthetic.mlp_init(dims, seed=0)), norm, train=False,
                    activation="relu" if momenta else "tanh", in_vars=io, out_vars=io)
    m = B.Mesh(N, 3, 200.0)
    q = torch.from_numpy(synthetic.random_state(N, 3, seed=7, momentum=0.3)).cuda()
    dt = 0.5 * B.dg_stable_dt(m, q)
    q2, k, k2 = q.clone(), m.field(0.0), m.field(0.0)
    B.dg_rk_step(m, q, k, dt, 2, model=model)
    B.dg_profile_steps(m, q2, k2, dt, 2, model=model)
    torch.cuda.synchronize()
    assert torch.isfinite(q).all() and torch.equal(q, q2) and torch.equal(k, k2)


# row blocks of sixteen: one row, one short, one over, two over; one, two and
# three hidden layers of 256; the four input widths with kernels of their own
@pytest.mark.parametrize("batch", [1, 15, 17, 34])
@pytest.mark.parametrize("n_p,momenta,hidden", [(64, False, 3), (64, True, 1), (27, False, 2), (27, True, 3)])
def test_training_rows(B, batch, n_p, momenta, hidden):
    """Loss and gradients of a small batch of indexed rows against the oracle
    with the same bfloat16 weights and activations.  What is left is the
    rounding of the output gradients to bfloat16, 2^-9 relative each, once a
    layer: below 1e-2 relative L2 for the at most four layers here."""
    from oracle import mlp
    say("training rows", batch, n_p, momenta, hidden)
    io = (1, 2, 3) if momenta else (0, 1, 2, 3, 4)
    kind = "relu" if momenta else "tanh"
    dims = [n_p * len(io)] + [256] * hidden + [n_p * len(io)]
    layers = [(W, b + np.float32(0.01)) for W, b in synthetic.mlp_init(dims, seed=4)]
    mu, sig = np.array([1.0, 0, 0, 0, 178.7]), np.array([0.01, 0.5, 0.5, 0.5, 1.0])
    norm = [*mu, *sig, *([0.0] * 5), *([1e-3] * 5)]
    rng = np.random.default_rng(batch)
    rows = batch + 5
    x = (np.repeat(mu, n_p) + np.repeat(sig, n_p) * rng.standard_normal((rows, 5 * n_p))).astype(np.float32)
    y = (1e-3 * rng.standard_normal((rows, 5 * n_p))).astype(np.float32)
    idx = rng.permutation(rows)[:batch].astype(np.int32)
    model = B.Model(dims, B.pack_params(layers), norm, activation=kind, in_vars=io, out_vars=io)
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    B.nn_train_step(model, torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), loss=loss,
                    idx=torch.from_numpy(idx).cuda())
    torch.cuda.synchronize()
    cols = np.concatenate([np.arange(v * n_p, (v + 1) * n_p) for v in io])
    xh = ((x[idx].astype(np.float64) - np.repeat(mu, n_p)) / np.repeat(sig, n_p))[:, cols]
    yt = (y[idx].astype(np.float64) / 1e-3)[:, cols]
    params = [(mlp.bf16_round(W), b.astype(np.float64)) for W, b in layers]
    loss_ref, grads = mlp.mse_loss_and_grads(params, xh, yt, act=kind, quantise=True)
    assert abs(loss.item() / loss_ref - 1) < 1e-3
    for (gW, gb), (rW, rb) in zip(B.unpack_params(model.grad.cpu().numpy().astype(np.float64), dims), grads):
        eW = np.linalg.norm(gW - rW) / np.linalg.norm(rW)
        eb = np.linalg.norm(gb - rb) / np.linalg.norm(rb)
        assert eW < 1e-2 and eb < 1e-2, (eW, eb)


@pytest.mark.parametrize("N,P,viscous", [(13, 8, True), (14, 8, True), (27, 3, False)])
def test_stage_update_past_the_cache(B, N, P, viscous):
    """A step on both sides of 256 MB of stage data (236, 295 and 298 MB)
    against the same stages put together from the residual, on the GPU.
    Float64 on both sides in other rounding orders: 32 eps of what the
    divergence sums, fluxes of up to 2 E times the derivative's (N / pi) PP^2."""
    say("stage update past the cache", N, P, viscous)
    m = B.Mesh(N, P, 200.0, viscous=viscous)
    q, k, r = m.field(), m.field(0.0), m.field()
    B.dg_init_tgv(m, q)
    ref, reg = q.clone(), torch.zeros_like(q)
    dt = 1e-4
    for A, w in ((0.0, 1 / 3), (-5 / 9, 15 / 16), (-153 / 128, 8 / 15)):
        B.dg_residual(m, ref, r)
        reg = A * reg + dt * r
        ref += w * reg
    B.dg_rk_step(m, q, k, dt, 1)
    eps = np.finfo(float).eps
    tol = 32 * eps * dt * 2 * float(ref[4].abs().max()) * (N / np.pi) * (P + 1) ** 2
    for v in range(5):
        assert float((k[v] - reg[v]).abs().max()) <= tol
        assert float((q[v] - ref[v]).abs().max()) <= tol + 8 * eps * float(ref[v].abs().max())


# one block and fewer nodes than it has threads, as many blocks as elements,
# several nodes a thread with an element's node count that does not divide
# the stride
@pytest.mark.parametrize("N,P", [(1, 1), (2, 8), (3, 2), (9, 6), (15, 7)])
def test_diagnostics_over_blocks(B, N, P):
    """Diagnostics and error norm against torch in float64: sums of up to
    1.7 million terms in another order (1e-12 relative; momenta, which
    cancel, relative to the sum of their absolute values), maxima of the
    same numbers, a reciprocal in place of quotients (8 eps)."""
    from oracle import basis
    say("diagnostics over blocks", N, P)
    m = B.Mesh(N, P, 100.0)
    q0 = synthetic.random_state(N, P, seed=70 + P, momentum=0.3)
    q1 = synthetic.random_state(N, P, seed=71 + P, momentum=0.3)
    q, r = (torch.from_numpy(x).cuda() for x in (q0, q1))
    d = B.dg_diagnostics(m, q).cpu().numpy()
    err = torch.full((3,), float("nan"), dtype=torch.float64, device="cuda")
    B.dg_error_inf(m, q, r, err)
    _, w = basis.gauss_legendre(P)
    x = q0.reshape(5, N ** 3, -1)
    wq = np.einsum("k,j,i->kji", w, w, w).ravel() * (np.pi / N) ** 3
    m2 = x[1] ** 2 + x[2] ** 2 + x[3] ** 2
    pr = 0.4 * (x[4] - 0.5 * m2 / x[0])
    eps = np.finfo(float).eps
    assert abs(d[0] - (wq * 0.5 * m2 / x[0]).sum() / (2 * np.pi) ** 3) <= 1e-12 * d[0]
    assert abs(d[1] - (np.sqrt(m2) / x[0] + np.sqrt(1.4 * pr / x[0])).max()) <= 8 * eps * d[1]
    assert d[2] == x[0].min()
    for v in range(5):
        assert abs(d[3 + v] - (wq * x[v]).sum()) <= 1e-12 * (wq * np.abs(x[v])).sum()
    assert np.array_equal(err.cpu().numpy(), np.abs(x - q1.reshape(5, N ** 3, -1))[1:4].reshape(3, -1).max(axis=1))


# 32-row steps over eight wavefronts: one, a few, ten, more than eight each;
# a width that is no multiple of 32
@pytest.mark.parametrize("rows", [16, 80, 160, 1100])
@pytest.mark.parametrize("dims", [(320, 256, 256, 320), (320, 40, 96, 320)])
def test_gradient_of_a_batch(B, rows, dims):
    """The gradient of a batch is the mean of its halves' gradients.  Each
    row's share is the same number in both (its scale differs by a power of
    two), so they differ by the order of float32 sums only: 1e-5 relative L2.
    With a vanishing learning rate the weights and their bf16 copies stay, so
    the whole batch gives the same bits once more."""
    say("gradient of a batch", rows, dims)
    layers = [(W, b + 0.01) for W, b in synthetic.mlp_init(list(dims), seed=9)]
    norm = [1.0, 0.0, 0.0, 0.0, 178.0, 0.01, 1.0, 1.0, 1.0, 1.0] + [0.0] * 5 + [1e-3] * 5
    model = B.Model(list(dims), B.pack_params(layers), norm)
    rng = np.random.default_rng(rows)
    x = rng.standard_normal((2 * rows, 320)).astype(np.float32)
    y = (1e-3 * rng.standard_normal((2 * rows, 320))).astype(np.float32)
    x, y = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    p0 = model.params.clone()

    def grad(a, b):
        loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        B.nn_train_step(model, x[a:b], y[a:b], lr=1e-30, loss=loss)
        return model.grad.clone(), loss.item()

    whole, loss = grad(0, 2 * rows)
    (first, l0), (second, l1) = grad(0, rows), grad(rows, 2 * rows)
    again, _ = grad(0, 2 * rows)
    assert torch.equal(model.params, p0) and torch.equal(again, whole)
    mean = 0.5 * (first.double() + second.double())
    assert float((whole - mean).norm() / mean.norm()) < 1e-5
    assert abs(loss - 0.5 * (l0 + l1)) < 1e-5 * loss


# blocks smaller than a wavefront, equal orders, the widest
@pytest.mark.parametrize("Ps,Pd", [(1, 1), (2, 1), (5, 4), (7, 2), (8, 1), (8, 8)])
def test_filter_orders(B, Ps, Pd):
    """Filter G against the oracle: two roundings per product in up to 27
    sums of order-one terms, 1e-13 of the largest value."""
    from oracle import dg, projection
    say("filter orders", Ps, Pd)
    N = 3
    src = np.random.default_rng(Ps * 10 + Pd).standard_normal((5, N ** 3, (Ps + 1) ** 3))
    ms, md = B.Mesh(N, Ps, 100.0), B.Mesh(N, Pd, 100.0)
    out = md.field(float("nan"))
    B.dg_project(ms, md, torch.from_numpy(src).cuda(), out)
    ref = dg.to_flat(projection.project(dg.to_blocks(src, N, Ps), Ps, Pd))
    assert np.max(np.abs(out.cpu().numpy() - ref)) < 1e-13 * np.max(np.abs(ref))
