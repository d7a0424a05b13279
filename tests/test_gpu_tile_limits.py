"""Every tile of the stage kernel at the limits of its range (needs an MI355X).

A problem alone takes the first tile of its Q whose number of blocks is within the tile's limit.
Here it has as many cells as still take the tile, some fewer (a last block that is partly
filled) and one more, which takes the next tile.  The reference is a batch of the same problems
held to the large-problem tile through a tuner cache file; the tile that it runs is asserted.
All tiles evaluate the same expressions in the same order, so the states agree bit for bit."""
import json

import numpy as np
import pytest

from helpers import say
import workloads

pytestmark = pytest.mark.gpu

FP64, FP32, FP32_MIXED = 0, 1, 2

# per Q: the large-problem tile (strips, strip length), then (cells, most blocks) of the others in
# the order in which they are considered; None: taken for any number of blocks
F64 = {8: ((8, 8), (8, 1024), (16, 1024), (32, None)), 12: ((8, 8), (8, 256), (16, 512), (32, 1300)),
       16: ((8, 8), (8, 256), (16, 512), (32, 1024)), 20: ((4, 8), (8, 256), (16, 512)),
       24: ((4, 8), (8, 256), (16, 512)), 32: ((4, 8), (8, 256), (16, 512)), 40: ((8, 8), (8, 256), (16, 512)),
       48: ((4, 8), (8, 256), (16, 512)), 64: ((2, 8), (8, 256)), 96: ((2, 8), (4, 256), (8, 256)),
       200: ((2, 8), (4, 128), (8, 256))}
F32 = {8: ((8, 8), (8, 1024), (16, 1024), (32, None)), 12: ((8, 8), (8, 256), (16, 512), (32, 1300)),
       16: ((8, 8), (16, 512), (32, 1024)), 20: ((8, 8), (8, 256), (16, 256), (32, 1024)),
       24: ((16, 8), (16, 256), (32, 256), (64, 512)), 32: ((8, 8), (8, 256), (16, 256), (32, 512)),
       40: ((8, 8), (8, 256), (16, 256), (32, 512)), 48: ((8, 8), (8, 256), (16, 256), (32, 256)),
       64: ((6, 8), (8, 256), (16, 256), (32, 256)), 96: ((4, 8), (8, 256), (16, 256)),
       200: ((2, 8), (4, 128), (8, 128))}
QS = sorted(F64)
# shapes that only the tuner takes (FP32 modes, chi_SET): they may split a wave's items or the
# coefficient recurrence otherwise, so they agree to rounding (test_gpu_batch.py), not in bits
TUNED = {16: (16, 8), 24: (8, 8), 32: (4, 16), 48: (4, 16), 96: (2, 16)}


def _sizes(tiles):
    sizes = [9]
    for cells, most in tiles[1:]:
        sizes += [cells * most - cells // 2 - 1, cells * most, cells * most + 1] if most else [40001]
    return sizes


def _problem(nx, q, chi):
    w = dict(workloads.shock_tube(nx=nx, q=q, kn=0.05), chi=chi)
    if chi == "ret" and nx > 1000:
        w["denseness"], w["kn"] = 0.05, 1e-3      # a ball of up to a few cells
    return w


@pytest.mark.parametrize("chi", ["set", "ret"])
@pytest.mark.parametrize("precision", [FP64, FP32, FP32_MIXED])
@pytest.mark.parametrize("q", QS)
def test_tiles_at_their_limits_match_the_large_one(q, precision, chi, tmp_path):
    import paper_2211_16933_amd as elb
    tiles = (F64 if precision == FP64 else F32)[q]
    ws = [_problem(nx, q, chi) for nx in _sizes(tiles)]
    say(f"case limits q={q} precision={precision} chi={chi} cells={[w['nx'] for w in ws]}")
    b = elb.BatchSolver([elb.params_from_workload(w, precision=precision) for w in ws])
    for i, w in enumerate(ws):
        b.set_state_moments(i, w["n"], w["u"], w["T"])
    cells = sum(w["nx"] for w in ws)
    key = f"gfx950/{precision}/q{q}{'/ret' if chi == 'ret' else ''}/cells2^{cells.bit_length() - 1}"
    cache = tmp_path / "tiles.json"
    cache.write_text(json.dumps({key: 0}))
    b.tune(str(cache))
    g = b.groups()[0]
    assert (g["strips"], g["strip_len"]) == tiles[0]
    assert json.loads(cache.read_text()) == {key: 0}          # nothing was timed
    b.step(3)
    for i, w in enumerate(ws):
        s = elb.Solver(elb.params_from_workload(w, precision=precision))
        s.set_state_moments(w["n"], w["u"], w["T"])
        s.step(3)
        for x, y in zip(s.dist() + s.moments(), b.dist(i) + b.moments(i)):
            assert np.array_equal(x, y), (w["nx"], "differs from the large-problem tile")
        s.close()
    b.close()


@pytest.mark.parametrize("chi", ["set", "ret"])
@pytest.mark.parametrize("precision", [FP64, FP32, FP32_MIXED])
@pytest.mark.parametrize("q", QS)
def test_every_batch_tile_matches_the_first(q, precision, chi, tmp_path):
    """Each compiled batch tile of a Q, chosen through the cache file, on problems with partly filled
    tiles."""
    import paper_2211_16933_amd as elb
    ws = [_problem(nx, q, chi) for nx in (9, 63, 130, 517)]
    key = f"gfx950/{precision}/q{q}{'/ret' if chi == 'ret' else ''}/cells2^9"
    say(f"case batch tiles q={q} precision={precision} chi={chi}")
    cache = tmp_path / "tiles.json"
    want, seen = None, []
    for v in range(12):
        cache.write_text(json.dumps({key: v}))
        b = elb.BatchSolver([elb.params_from_workload(w, precision=precision) for w in ws])
        for i, w in enumerate(ws):
            b.set_state_moments(i, w["n"], w["u"], w["T"])
        b.tune(str(cache))
        if json.loads(cache.read_text()) != {key: v}:         # past the last: the tuner timed them
            break
        g = b.groups()[0]
        seen.append((g["strips"], g["strip_len"]))
        b.step(3)
        got = [x for i in range(len(ws)) for x in b.dist(i) + b.moments(i)]
        want = want or got
        if precision == FP64 or seen[-1] != TUNED.get(q):
            assert all(np.array_equal(x, y) for x, y in zip(got, want)), seen
        b.close()
    tiles = (F64 if precision == FP64 else F32)[q]
    assert seen[0] == tiles[0] and len(set(seen)) == len(seen) and len(seen) >= len(tiles)


@pytest.mark.parametrize("q", QS)
def test_fixup_tiles_against_repeats(q):
    """The moment fix-up, which batches do not carry: a periodic pattern on each tile against the
    pattern repeated until the large-problem tile takes it.  The stochastic rounding differs from
    cell to cell, so values agree to 9 roundings of FP32 deviations below 1 and what the scheme
    makes of them (a factor of 4 here)."""
    import paper_2211_16933_amd as elb
    tiles = F32[q]

    def run(nx, length):
        w = dict(workloads.sound_wave(nx=nx, q=q, kn=0.05), length=length)
        x = workloads.cell_centres(64, 1.0) * 2.0 * np.pi
        f = [np.tile(v, nx // 64) for v in (1.0 + 0.1 * np.sin(x), 0.05 * np.cos(x), 1.0 + 0.05 * np.sin(2.0 * x))]
        s = elb.Solver(elb.params_from_workload(w, precision=FP32_MIXED, moment_fixup=1))
        s.set_state_moments(*f)
        s.step(3)
        return s.dist() + s.moments()[:3]

    copies = [1] + [max(1, cells * most // 64) for cells, most in tiles[1:] if most]
    copies.append(copies[-1] + 4 * tiles[0][0])
    say(f"case fix-up tiles q={q} copies={copies}")
    runs = [run(64 * c, float(c)) for c in copies]
    for c, r in zip(copies, runs):
        for x, y in zip(r, runs[0]):
            y = np.tile(y, (c, 1) if y.ndim == 2 else c)
            assert np.max(np.abs(x - y)) <= 9 * 4 * 2.0 ** -24
