"""Contexts and batches beside others (needs an MI355X): creating, using and closing one does not
wait for the work of another's stream, and more of them than there are pinned buffers for work as
well."""
import time

import numpy as np
import pytest

from helpers import say
import workloads

pytestmark = pytest.mark.gpu


def _solver(nx, q, stream=None):
    import paper_2211_16933_amd as elb
    w = workloads.shock_tube(nx=nx, q=q)
    s = elb.Solver(elb.params_from_workload(w), stream=stream)
    s.set_state_moments(w["n"], w["u"], w["T"])
    return w, s


def test_close_does_not_wait_for_other_streams():
    import torch
    import paper_2211_16933_amd as elb
    say("case close beside other work")
    busy, mine = torch.cuda.Stream(), torch.cuda.Stream()
    _, big = _solver(65536, 96, busy)
    _, first = _solver(64, 8, mine)          # code objects and the like are loaded here
    first.step(1)
    first.moments()
    first.close()
    big.step(3)
    torch.cuda.synchronize()
    done = torch.cuda.Event()
    t0 = time.perf_counter()
    big.step(1500)                           # 0.4 to 0.5 s
    done.record(busy)
    w, s = _solver(64, 8, mine)
    s.step(2)
    m = s.moments()
    s.close()
    b = elb.BatchSolver([elb.params_from_workload(w)], stream=mine)
    b.set_state_moments(0, w["n"], w["u"], w["T"])
    b.set_graph(False)
    b.step(2)
    mb = b.moments(0)
    b.close()
    early = not done.query()
    t1 = time.perf_counter()
    done.synchronize()
    say(f"  closed after {t1 - t0:.3f} s, the other stream's work ended after {time.perf_counter() - t0:.3f} s")
    assert early
    assert all(np.array_equal(x, y) for x, y in zip(m, mb))


def test_more_contexts_than_pinned_buffers():
    """70 contexts that ask for 256 KB each, where 16 MB are given: those without a buffer copy from
    and to pageable memory, with the same results; closed ones hand theirs on."""
    say("case 70 contexts")
    _, ref = _solver(4000, 12)
    ref.step(2)
    want = ref.moments() + ref.dist() + (ref.conserved(), np.array(ref.amplitudes(2.0)))
    ref.close()
    for _ in range(2):
        many = [_solver(4000, 12)[1] for _ in range(70)]
        for s in many:
            s.step(2)
        for s in many:
            got = s.moments() + s.dist() + (s.conserved(), np.array(s.amplitudes(2.0)))
            assert all(np.array_equal(x, y) for x, y in zip(got, want))
        for s in many[::2] + many[1::2]:
            s.set_state_dist(*want[5:7])
            s.step(1)
            s.close()


def test_contexts_of_several_threads():
    """Eight threads, each with a stream of its own, make, run and close contexts and batches at the
    same time: buffers that pass between them must not be shared."""
    import threading
    import torch
    import paper_2211_16933_amd as elb
    say("case contexts of several threads")
    sizes = [64, 300, 1000, 2500, 4000, 6500, 7000, 12000]
    want = {}
    for nx in sizes:
        _, s = _solver(nx, 12)
        s.step(3)
        want[nx] = s.moments() + s.dist()
        s.close()
    torch.cuda.synchronize()
    wrong = []

    def work(k):
        try:
            stream = torch.cuda.Stream()
            for i in range(12):
                nx = sizes[(k + i) % len(sizes)]
                w, s = _solver(nx, 12, stream)
                b = elb.BatchSolver([elb.params_from_workload(w)], stream=stream)
                b.set_state_moments(0, w["n"], w["u"], w["T"])
                b.set_graph(False)
                s.step(3)
                b.step(3)
                for got in (s.moments() + s.dist(), b.moments(0) + b.dist(0)):
                    if not all(np.array_equal(x, y) for x, y in zip(got, want[nx])):
                        wrong.append((k, i, nx))
                s.close()
                b.close()
        except Exception as e:  # noqa: BLE001
            wrong.append((k, repr(e)))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
