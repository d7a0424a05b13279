"""What setting a state promises beyond its values (needs an MI355X): a refused restore leaves a
fresh context without a state, a good one ends a failure, and no state is set while the stream is
captured into a graph; and the copies at the sizes where their way changes."""
import numpy as np
import pytest

from helpers import say
import workloads

pytestmark = pytest.mark.gpu

FP64, FP32, FP32_MIXED = 0, 1, 2


def _tube(nx=65, q=12, precision=FP64, **kw):
    import paper_2211_16933_amd as elb
    w = workloads.shock_tube(nx=nx, q=q)
    return w, elb.Solver(elb.params_from_workload(w, precision=precision), **kw)


@pytest.mark.parametrize("precision", [FP64, FP32, FP32_MIXED])
def test_refused_first_restore_leaves_no_state(precision):
    """A fresh context with end states: refused distributions must not leave the uniform state
    behind that its ghost rows are built from."""
    import paper_2211_16933_amd as elb
    say(f"case refused first restore precision={precision}")
    w, s = _tube(precision=precision)
    s.set_state_moments(w["n"], w["u"], w["T"])
    s.step(3)
    phi, theta = s.dist()
    bad = []
    for which in (0, 1):
        arrays = [phi.copy(), theta.copy()]
        arrays[which][7, 3] = np.nan
        bad.append(arrays)
    if precision != FP64:                       # (FP64 storage has no mean state to refuse)
        bad.append([-phi, theta])
    for arrays in bad:
        _, f = _tube(precision=precision)
        with pytest.raises(elb.ElbError) as e:
            f.set_state_dist(*arrays)
        assert e.value.code == elb.ELB_EINVAL
        for call in (lambda: f.step(1), f.moments, f.dist, f.conserved, lambda: f.amplitudes(1.0)):
            with pytest.raises(elb.ElbError) as e:
                call()
            assert e.value.code == elb.ELB_ESTATE
        f.set_state_dist(phi, theta)            # and a good restore is taken afterwards
        _, g = _tube(precision=precision)
        g.set_state_dist(phi, theta)
        f.step(5)
        g.step(5)
        assert all(np.array_equal(x, y) for x, y in zip(f.dist(), g.dist()))


@pytest.mark.parametrize("precision", [FP64, FP32, FP32_MIXED])
@pytest.mark.parametrize("nx", [65, 2100])
def test_restore_ends_a_failure(precision, nx):
    """A run that failed (a cell of negative density) goes on from a good checkpoint."""
    import paper_2211_16933_amd as elb
    say(f"case restore after a failure nx={nx} precision={precision}")
    w, s = _tube(nx=nx, precision=precision)
    s.set_state_moments(w["n"], w["u"], w["T"])
    s.step(3)
    phi, theta = s.dist()
    broken = phi.copy()
    broken[nx // 2] *= -1.0
    s.set_state_dist(broken, theta)
    s.step(1)
    for call in (s.moments, s.dist, s.conserved, lambda: s.amplitudes(1.0)):
        with pytest.raises(elb.ElbError) as e:
            call()
        assert e.value.code == elb.ELB_ENONFINITE
    s.set_state_dist(phi, theta)
    s.step(2)
    assert all(np.all(np.isfinite(x)) for x in s.moments() + s.dist())
    assert np.all(np.isfinite(s.conserved())) and np.all(np.isfinite(s.amplitudes(1.0)))
    _, f = _tube(nx=nx, precision=precision)
    f.set_state_moments(w["n"], w["u"], w["T"])
    f.set_state_dist(phi, theta)
    f.step(2)
    if precision == FP64:          # (FP32 ghost rows were rounded about other references)
        assert all(np.array_equal(x, y) for x, y in zip(s.dist(), f.dist()))


@pytest.mark.parametrize("nx", [65, 2100])
def test_no_state_is_set_under_capture(nx):
    """The caller captures a step of the context's stream: setting a state is refused, the capture
    goes on, and its replays advance the state that was set before."""
    import torch
    import paper_2211_16933_amd as elb
    say(f"case set under capture nx={nx}")
    stream = torch.cuda.Stream()
    w, s = _tube(nx=nx, stream=stream)
    s.set_state_moments(w["n"], w["u"], w["T"])
    s.step(3)
    phi, theta = s.dist()
    b = elb.BatchSolver([elb.params_from_workload(w, precision=FP64)], stream=stream)
    b.set_state_moments(0, w["n"], w["u"], w["T"])
    before = b.dist(0)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
        s.step(1)
        for call in (lambda: s.set_state_moments(1.1 * w["n"], w["u"], w["T"]), lambda: s.set_state_dist(phi, theta),
                     lambda: b.set_state_moments(0, 1.1 * w["n"], w["u"], w["T"])):
            with pytest.raises(elb.ElbError) as e:
                call()
            assert e.value.code == elb.ELB_EHIP
        s.step(1)
    assert all(np.array_equal(x, y) for x, y in zip(b.dist(0), before))
    _, f = _tube(nx=nx)
    f.set_state_moments(w["n"], w["u"], w["T"])
    f.step(3)
    for _ in range(3):
        with torch.cuda.stream(stream):
            graph.replay()
        s.step(1)
        f.step(3)
        assert all(np.array_equal(x, y) for x, y in zip(s.dist(), f.dist()))


@pytest.mark.parametrize("nx,q", [(408, 40), (409, 8), (410, 8), (512, 40), (6552, 8), (6553, 8), (6554, 8), (6554, 40), (33000, 8)])
@pytest.mark.parametrize("precision", [FP64, FP32])
def test_copies_at_the_edges_of_the_pinned_buffer(nx, q, precision):
    """Readouts and restores whose pieces fill the buffer (16 to 256 KB) to the last value, one cell more
    or less, and whose pieces go part through it, part directly."""
    import paper_2211_16933_amd as elb
    say(f"case copies nx={nx} q={q} precision={precision}")
    w, s = _tube(nx=nx, q=q, precision=precision)
    s.set_state_moments(w["n"], w["u"], w["T"])
    s.step(2)
    phi, theta = s.dist()
    p, _ = elb.quadrature(q)
    n, u, T, qx, pxx = s.moments()
    # sums of q terms in another order: q rounding errors of the largest partial sums, which the
    # outer nodes' cubes scale (below 10 p_max^3 here)
    tol = 16 * q * 2.3e-16 * (1.0 + 10.0 * p[-1] ** 3)
    xi = p - u[:, None]
    e = 0.5 * xi * xi * phi + 0.5 * theta
    for got, want in ((n, phi.sum(1)), (u, phi @ p / n), (T, e.sum(1) / (1.5 * n)), (qx, (xi * e).sum(1)),
                      (pxx, (xi * xi * phi).sum(1))):
        assert np.max(np.abs(got - want)) <= tol
    back = phi[::-1].copy(), theta[::-1].copy()
    s.set_state_dist(*back)
    got = s.dist()
    if precision == FP64:
        assert all(np.array_equal(a, b) for a, b in zip(got, back))
    else:           # deviations below 0.5 in FP32
        assert all(np.max(np.abs(a - b)) <= 0.5 * 2.0 ** -24 + 1e-15 for a, b in zip(got, back))
    assert np.max(np.abs(s.moments()[0] - n[::-1])) <= tol + (0.0 if precision == FP64 else q * 0.5 * 2.0 ** -24)
