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
    # A solve that fills the device for some 0.8 s, in launches of 50 ms: a small
    # kernel waits for the end of one, a small solve (10 ms alone, two
    # synchronisations) of two or three.  The bounds leave four times that.
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
