"""Distributions read and restored over whole planes, and the moments of every cell (needs an
MI355X): every value, also where there are more than a launch may hold threads for."""
import ctypes

import numpy as np
import pytest

from helpers import say
import workloads

pytestmark = pytest.mark.gpu


def _wave(nx, q):
    return dict(workloads.sound_wave(nx=64, q=q), nx=nx, length=nx / 64.0)


def test_plane_of_2_32_values():
    """FP32 storage, 2^32 + 1304 values per plane: the uniform equilibrium at rest is the
    quadrature weights in every row.  Rows at both ends and around 2^31 and 2^32 values."""
    import psutil
    import torch
    import paper_2211_16933_amd as elb
    q = 200
    nx = (1 << 32) // q + 7
    P = elb.params_from_workload(_wave(nx, q), precision=elb.FP32)
    torch.cuda.empty_cache()
    if psutil.virtual_memory().available < 2 * 8 * nx * q or torch.cuda.mem_get_info()[0] < 1.1 * elb.workspace_bytes(P):
        pytest.skip("not enough host or GPU memory for a plane of 2^32 values")
    say(f"case planes of {nx} x {q} values")
    s = elb.Solver(P)
    one = np.ones(nx)
    s.set_state_moments(one, np.zeros(nx), one)
    phi = np.empty((nx, q))
    rc = elb.lib().elb_get_dist(s._ctx, phi.ctypes.data_as(ctypes.POINTER(ctypes.c_double)), None)
    s.close()
    assert rc == elb.ELB_OK
    _, w = elb.quadrature(q)
    half = (1 << 31) // q
    rows = [0, 1, 6, 100, half - 1, half, half + 1, nx - 8, nx - 7, nx - 1]
    # the state equals its own reference: stored deviations of rounding size in FP32
    worst = max(float(np.max(np.abs(phi[i] - w))) for i in rows)
    say(f"  max |phi - w| = {worst:.2e}")
    assert worst <= 1e-15
    del phi, s
    torch.cuda.empty_cache()


@pytest.mark.parametrize("precision", [0, 1])
def test_planes_beyond_one_sweep_of_a_launch(precision):
    """More values than the threads of a launch (8192 blocks of 256), with a remainder: a periodic
    pattern of 64 cells, repeated, against the 64 cells alone."""
    import paper_2211_16933_amd as elb
    q, copies = 40, 1025
    say(f"case planes of {64 * copies} x {q} values precision={precision}")
    x = workloads.cell_centres(64, 1.0) * 2.0 * np.pi
    fields = 1.0 + 0.1 * np.sin(x), 0.05 * np.cos(x), 1.0 + 0.05 * np.sin(2 * x)
    one = elb.Solver(elb.params_from_workload(_wave(64, q), precision=precision))
    many = elb.Solver(elb.params_from_workload(_wave(64 * copies, q), precision=precision))
    one.set_state_moments(*fields)
    many.set_state_moments(*[np.tile(f, copies) for f in fields])
    # FP64: the same operations, the same bits.  FP32: the mean state, about which the deviations
    # are held, is a sum of another length, so a deviation (below 0.2) may round elsewhere
    tol = 0.0 if precision == 0 else 2.0 ** -24 * 0.2 + 64 * copies * 2.0 ** -53
    state = one.dist()
    assert all(np.max(np.abs(a - np.tile(b, (copies, 1)))) <= 2 * tol for a, b in zip(many.dist(), state))
    if precision == 0:
        assert all(np.array_equal(a, np.tile(b, (copies, 1))) for a, b in zip(many.rhs(), one.rhs()))
    back = [np.tile(b[::-1], (copies, 1)) for b in state]      # another state, restored
    many.set_state_dist(*back)
    assert all(np.max(np.abs(a - b)) <= tol for a, b in zip(many.dist(), back))


def test_moments_of_2_28_cells():
    """2^28 + 77 cells, 16 threads each: the uniform state at rest in every cell."""
    import psutil
    import torch
    import paper_2211_16933_amd as elb
    nx = (1 << 28) + 77
    P = elb.params_from_workload(_wave(nx, 8), precision=elb.FP32)
    torch.cuda.empty_cache()
    if psutil.virtual_memory().available < 16 * 8 * nx or torch.cuda.mem_get_info()[0] < 1.1 * elb.workspace_bytes(P):
        pytest.skip("not enough host or GPU memory for 2^28 cells")
    say(f"case moments of {nx} cells")
    s = elb.Solver(P)
    one = np.ones(nx)
    s.set_state_moments(one, np.zeros(nx), one)
    got = s.moments()
    s.close()
    # the state equals its own reference: sums of 8 values, each rounded to 1e-16
    for f, want in zip(got, (1.0, 0.0, 1.0, 0.0, 1.0)):
        assert f.size == nx and max(abs(f.min() - want), abs(f.max() - want)) <= 1e-14
    del s, got, one
    torch.cuda.empty_cache()
