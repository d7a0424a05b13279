"""The stage kernel's tiles of small problems against its tile of large ones (needs an MI355X).

A problem alone takes the tile that its own number of blocks selects; in a batch with a large
problem of the same Q every instance takes the large-problem tile.  All tiles evaluate the
same expressions in the same order, so the states must agree bit for bit.  The cell counts sit
at the edges of the tiles: one cell more or less than whole tiles of 4 to 32 cells, the
smallest grid, and the first count past the block limit of the smallest tile."""
import numpy as np
import pytest

from helpers import say
import workloads

pytestmark = pytest.mark.gpu

FP64, FP32, FP32_MIXED = 0, 1, 2
FILLER = 33000          # more blocks than any limit of the small tiles


@pytest.mark.parametrize("chi", ["set", "ret"])
@pytest.mark.parametrize("precision", [FP64, FP32, FP32_MIXED])
@pytest.mark.parametrize("q", [8, 12, 16, 20, 24, 32, 40, 48, 64, 96, 200])
def test_small_tiles_match_the_large_one(q, precision, chi):
    import paper_2211_16933_amd as elb
    sizes = [8, 33, 127, 2049, 4100] if q < 200 else [8, 33, 515]
    if chi == "ret":
        sizes = sizes[1:4]
    ws = []
    for nx in sizes:
        w = workloads.shock_tube(nx=nx, q=q, kn=0.05)
        w["chi"] = chi
        ws.append(w)
    filler = dict(workloads.shock_tube(nx=FILLER, q=q), chi=chi)
    if chi == "ret":
        filler["denseness"], filler["kn"] = 0.05, 1e-3   # a ball of a few cells on this grid
    say(f"case tiles q={q} precision={precision} chi={chi} cells={sizes}")
    b = elb.BatchSolver([elb.params_from_workload(w, precision=precision) for w in ws + [filler]])
    for i, w in enumerate(ws + [filler]):
        b.set_state_moments(i, w["n"], w["u"], w["T"])
    b.step(3)
    for i, w in enumerate(ws):
        s = elb.Solver(elb.params_from_workload(w, precision=precision))
        s.set_state_moments(w["n"], w["u"], w["T"])
        s.step(3)
        for x, y in zip(s.dist() + s.moments(), b.dist(i) + b.moments(i)):
            assert np.array_equal(x, y), (w["nx"], "differs from the large-problem tile")
        s.close()
    b.close()


def test_batch_tiles_of_small_problems():
    """A batch of small problems takes small tiles before any tuning, with the same states."""
    import paper_2211_16933_amd as elb
    ws = [workloads.sound_wave(nx=nx, q=16, amplitude=1e-2) for nx in (9, 64, 100)]
    b = elb.BatchSolver([elb.params_from_workload(w, precision=FP64) for w in ws])
    assert b.groups()[0]["strips"] * b.groups()[0]["strip_len"] < 64
    for i, w in enumerate(ws):
        b.set_state_moments(i, w["n"], w["u"], w["T"])
    b.step(60)
    for i, w in enumerate(ws):
        s = elb.Solver(elb.params_from_workload(w, precision=FP64))
        s.set_state_moments(w["n"], w["u"], w["T"])
        s.step(60)
        assert all(np.array_equal(x, y) for x, y in zip(s.dist(), b.dist(i)))


@pytest.mark.parametrize("precision", [FP64, FP32_MIXED])
@pytest.mark.parametrize("q,nx", [(8, 33), (8, 20001), (8, 45001), (12, 8300), (12, 60001), (16, 8300)])
def test_learned_closure_on_every_tile(q, nx, precision):
    """The learned closure inside the stage at cell counts that select each of its tiles, against
    its two separate kernels: the same network arithmetic, with inputs from row moments summed
    in another order, so a bfloat16 rounding may flip here and there (5e-3 of the correction's
    effect, as for a single tile)."""
    import paper_2211_16933_amd as elb
    from paper_2211_16933_amd import learned
    w = workloads.shock_tube(nx=nx, q=q)
    x = workloads.cell_centres(nx, 1.0)
    s = 0.5 * (1.0 + np.tanh((x - 0.5) / 0.05))
    w["n"], w["u"], w["T"] = [a + (b - a) * s for a, b in zip(w["left"], w["right"])]
    norm = learned.make_norm([1.25, 0, 1.1] + [0.0] * 7 + [0.4, -1.3], [0.3, 0.3, 0.3] + [0.5] * 7 + [1.0, 1.0],
                             np.zeros(q), np.full(q, nx / 2000.0), -np.full(12, 1e3), np.full(12, 1e3))
    # (the output scale makes up for the time step, which falls with the cell size, so that the
    # effect of 3 steps stands far above the FP32 rounding at every size)
    say(f"case closure tiles q={q} nx={nx} precision={precision}")
    runs = {}
    for enabled in (0, 1, 2):
        c = elb.Solver(elb.params_from_workload(w, precision=precision, closure=1))
        c.set_state_moments(w["n"], w["u"], w["T"])
        if enabled:
            c.set_closure(learned.init_params(q, 5), norm, enabled)
        c.step(3)
        runs[enabled] = c.dist()[0]
        c.close()
    effect = np.linalg.norm(runs[2] - runs[0])
    assert effect >= 1e-5 * np.linalg.norm(runs[0])
    assert np.linalg.norm(runs[1] - runs[2]) <= 5e-3 * effect
