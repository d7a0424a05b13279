"""Setting and reading states at the sizes where the way of checking, building or copying them
changes (needs an MI355X): cells checked on the host up to 2048 and on the GPU above; moments
in one copy, in pieces and field by field; the two forms of the equilibrium kernel; amplitudes
with and without the moment kernel."""
import numpy as np
import pytest

from helpers import say
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,q", [(8, 8), (2048, 8), (2049, 16), (6560, 8), (16000, 12), (65537, 48)])
@pytest.mark.parametrize("precision", [0, 2])
def test_state_round_trip_and_refusals(nx, q, precision):
    import paper_2211_16933_amd as elb
    say(f"case state nx={nx} q={q} precision={precision}")
    w = workloads.shock_tube(nx=nx, q=q)
    x = workloads.cell_centres(nx, 1.0)
    w["n"] = w["n"] * (1.0 + 0.1 * np.sin(7.0 * x))
    w["u"] = 0.05 * np.cos(5.0 * x)
    s = elb.Solver(elb.params_from_workload(w, precision=precision))
    s.set_state_moments(w["n"], w["u"], w["T"])
    # FP64 sums over 2Q values of order one, exact on the quadrature: 2Q rounding errors each;
    # q and Pxx - n T pass through FP32 storage in the mixed mode (2Q values of 6e-8)
    tol = 4 * q * 2.3e-16 * 4.0
    tol_q = tol if precision == 0 else 4 * q * 6.0e-8
    n, u, T, qx, pxx = s.moments()
    for got, want in ((n, w["n"]), (u, w["u"]), (T, w["T"])):
        assert np.max(np.abs(got - want)) <= tol
    assert np.max(np.abs(qx)) <= tol_q and np.max(np.abs(pxx - w["n"] * w["T"])) <= tol_q
    k = 2.0 * np.pi
    a, b = s.amplitudes(k)
    assert abs(a - 2.0 / nx * np.sum(w["n"] * np.sin(k * x))) <= 1e-13 * max(1, nx ** 0.5)
    assert abs(b - 2.0 / nx * np.sum(w["n"] * np.cos(k * x))) <= 1e-13 * max(1, nx ** 0.5)
    # refusals name the first bad cell and leave the state as it was
    for cell, field, value, word in ((nx - 1, "n", -1.0, "finite"), (nx // 2, "T", np.nan, "finite"),
                                     (nx - 2, "u", np.inf, "finite"), (nx - 3, "n", 1e9, "eta")):
        f = {key: w[key].copy() for key in ("n", "u", "T")}
        f[field][cell] = value
        f["n"][nx - 1] = -1.0       # a later one that must not be named instead
        with pytest.raises(elb.ElbError) as e:
            s.set_state_moments(f["n"], f["u"], f["T"])
        assert f"cell {cell}:" in str(e.value) and word in str(e.value)
    assert all(np.array_equal(p, r) for p, r in zip(s.moments(), (n, u, T, qx, pxx)))
    s.close()


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("nx,q", [(8, 8), (63, 12), (65, 20), (1000, 12), (4099, 96)])
def test_distribution_round_trip_and_refusals(nx, q, precision):
    """Whole distributions out and in: FP64 bit for bit; FP32 storage holds the deviation from the
    mean state's equilibrium, so a value comes back to half an ulp of its deviation.  The
    equilibrium is evaluated here again; its rounding (Q terms that cancel at the outer nodes)
    is part of what the deviation may be."""
    import paper_2211_16933_amd as elb
    say(f"case distributions nx={nx} q={q} precision={precision}")
    w = workloads.shock_tube(nx=nx, q=q)
    s = elb.Solver(elb.params_from_workload(w, precision=precision))
    s.set_state_moments(w["n"], w["u"], w["T"])
    s.step(3)
    phi, theta = s.dist()
    p, wt = elb.quadrature(q)
    n = phi.sum(1)
    u = phi @ p / n
    T = (phi @ (p * p) + theta.sum(1) - n * u * u) / (3.0 * n)
    nr, ur, Tr = n.mean(), u.mean(), T.mean()
    h, c = [np.ones(q), p], [1.0, ur]
    for l in range(1, q - 1):
        h.append((p * h[l] - np.sqrt(l) * h[l - 1]) / np.sqrt(l + 1))
        c.append((ur * c[l] + (Tr - 1.0) * np.sqrt(l) * c[l - 1]) / np.sqrt(l + 1))
    terms = nr * wt[:, None] * np.array(h).T * np.array(c)   # [node][order]
    refs = [terms.sum(1), 2.0 * Tr * terms.sum(1)]
    noise = 8 * q * 2.3e-16 * np.abs(terms).sum(1)
    fresh = elb.Solver(elb.params_from_workload(w, precision=precision))
    for t in (s, fresh):               # onto a state, and as the first state of a context
        t.set_state_dist(phi, theta)
        a, b = t.dist()
        for got, want, ref in ((a, phi, refs[0]), (b, theta, refs[1])):
            if precision == 0:
                assert np.array_equal(got, want)
            else:
                dev = np.abs(want - ref) + (1.0 + 2.0 * Tr) * noise
                assert np.all(np.abs(got - want) <= 2.0 ** -24 * dev + 2.0 ** -52 * np.abs(want) + 1e-44)
    before = s.dist()
    for bad in (np.nan, np.inf):
        for which in (0, 1):
            arrays = [phi.copy(), theta.copy()]
            arrays[which][nx - 1, q - 1] = bad
            with pytest.raises(elb.ElbError):
                s.set_state_dist(*arrays)
    assert all(np.array_equal(x, y) for x, y in zip(s.dist(), before))
    # FP64: both continue alike (FP32 ghost rows were rounded about different first references)
    if precision == 0:
        s.step(5)
        fresh.step(5)
        assert all(np.array_equal(x, y) for x, y in zip(s.dist(), fresh.dist()))
