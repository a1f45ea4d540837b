"""Work of other streams and threads beside a batch solve, and requests that arrive
while a server is busy (GPU)."""
import threading
import time

import pytest

import synth
from tests.gpu_util import device, t

pytestmark = pytest.mark.gpu


def _args(net, n, dev, **kw):
    c = synth.sample_cells(net, n, seed=5, **kw)
    return [t(v, dev) for v in (c.T, c.n_H, c.A_V, c.zeta, c.G0, c.x0, c.t_end)]


def test_other_streams_get_in_between():
    # A solve that fills the device for some 0.8 s, in launches of 100 ms: a small
    # kernel waits for the end of one, a small solve (10 ms alone, two
    # synchronisations) of two or three.  The bounds leave twice that.
    import torch
    import paper_2511_10558_amd as ab
    dev = device()
    net = synth.network_for_config("net500")
    g = ab.Network.from_text(net.to_text())
    a = _args(net, 1024, dev, t_end_yr=1e5)
    small = synth.network_for_config("small")
    gs = ab.Network.from_text(small.to_text())
    s = _args(small, 1, dev)
    v = torch.ones(1 << 16, device=dev)
    ab.solve(g, *[x[:2].contiguous() for x in a])
    alone = ab.solve(gs, *s)[0]
    v.mul_(1.0)
    torch.cuda.synchronize()
    out = []

    def batch():
        with torch.cuda.stream(torch.cuda.Stream()):
            out.append(ab.solve(g, *a, lu_reuse=0.3)[1].cpu().numpy())

    th = threading.Thread(target=batch)
    waits = {"kernel": [], "solve": []}
    with torch.cuda.stream(torch.cuda.Stream()):
        th.start()
        time.sleep(0.1)
        while th.is_alive():
            t0 = time.perf_counter()
            v.mul_(1.0)
            torch.cuda.current_stream().synchronize()
            waits["kernel"].append(time.perf_counter() - t0)
            t0 = time.perf_counter()
            x = ab.solve(gs, *s)[0]
            torch.cuda.current_stream().synchronize()
            waits["solve"].append(time.perf_counter() - t0)
            assert torch.equal(x, alone)
    th.join()
    assert (out[0] == 0).all() and len(waits["solve"]) > 0
    print({k: f"max {1e3 * max(w):.1f} ms of {len(w)}" for k, w in waits.items()})
    assert max(waits["kernel"]) < 0.2
    assert max(waits["solve"]) < 0.6


def test_requests_get_in_beside_a_long_one():
    # One request keeps 8 of 64 slots busy; others of a single short cell arrive while
    # it runs.  A launch ends for them within some step attempts (0.3 ms each) and 0.5
    # ms, and their results are handed out within 2 ms of being there.  They take
    # about 6 ms of work; the bounds leave twice that and more.
    import paper_2511_10558_amd as ab
    device()
    net = synth.network_for_config("net200")
    g = ab.Network.from_text(net.to_text())
    long = synth.sample_cells(net, 8, seed=1, t_end_yr=1e6)
    short = synth.sample_cells(net, 1, seed=2, t_end_yr=1e-3)

    def submit(srv, c, **kw):
        return srv.submit(c.T, c.n_H, c.A_V, c.zeta, c.G0, c.x0, c.t_end, **kw)

    with ab.Server(g, max_slots=64) as srv:
        submit(srv, short)
        srv.poll(timeout_ms=10000)
        rid = submit(srv, long, rtol=1e-10)
        time.sleep(0.02)
        admitted, done, finished = [], [], False
        for k in range(20):
            submit(srv, short)
            got = srv.poll(timeout_ms=10000)
            finished |= any(c["id"] == rid for c in got)
            for c in got:
                if c["id"] != rid:
                    admitted.append(c["t_first_admit"] - c["t_submit"])
                    done.append(c["t_done"] - c["t_submit"])
            time.sleep(0.0007 * (k % 5))
        assert not finished, "the long request ended too early to tell"
        t0 = time.perf_counter()
    closed = time.perf_counter() - t0      # with the long request still running
    print(f"admission median {1e3 * sorted(admitted)[10]:.2f} max {1e3 * max(admitted):.2f} ms, "
          f"completion median {1e3 * sorted(done)[10]:.2f} max {1e3 * max(done):.2f} ms")
    assert sorted(admitted)[10] < 4e-3
    assert sorted(done)[10] < 15e-3
    assert closed < 1.0
