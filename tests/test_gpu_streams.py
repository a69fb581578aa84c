"""Calls on side streams whose workspace and outputs the call itself allocates: what
is still queued there keeps its memory while other calls and the caller's own
stream allocate, whatever path a decode takes.  Results equal those of calls in
turn, exactly."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_1711_01783_amd as met  # noqa: E402
from met_inputs import PROFILES, make_frames  # noqa: E402
from oracle import code as oc  # noqa: E402

DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _busy(stream):
    with torch.cuda.stream(stream):
        torch.cuda._sleep(4000000)  # about 2 ms: what follows is pending when its call returns


def _overwrite(sizes):
    for n in sizes:  # blocks of the calls' sizes, written by the current stream and dropped
        torch.full((n,), 255, dtype=torch.uint8, device=DEV)


# one launch per decode; launches with a fixed number of iterations; reads of the host in between
@pytest.mark.parametrize("n,b,kw", [(8192, 24, dict()), (4096, 1, dict(posterior=True)),
                                    (8192, 40, dict(fixed_iters=True, check_steps_per_wave=4)),
                                    (8192, 40, dict(check_steps_per_wave=4))])
def test_decode_without_workspace(n, b, kw):
    code = met.Code.build(PROFILES["r0.1"], n, 14)
    ins = []
    for k in range(4):
        bits, llr = make_frames(n, b, 0.22, 100 * k)
        ins.append((torch.from_numpy(llr).to(DEV), met.syndrome(code, torch.from_numpy(bits).to(DEV))))
    ref = [met.decode(code, l, s, 30, **kw) for l, s in ins]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in ins]
    size = met.workspace_bytes(code, b, bool(kw.get("fixed_iters")), bool(kw.get("posterior")))
    print("side streams", n, b, kw, flush=True)
    for rep in range(3):
        outs = []
        for (l, s), st in zip(ins, streams):
            _busy(st)
            outs.append(met.decode(code, l, s, 30, stream=st, **kw))
            _overwrite((size + 256, b * n, b * n * 4))
        again = [met.decode(code, l, s, 30, stream=st, **kw) for (l, s), st in zip(ins, streams)]
        _overwrite((size + 256, b * n, b * n * 4))
        torch.cuda.synchronize()
        for r, o, a in zip(ref, outs, again):
            for k in ("bits", "iterations", "converged", "posterior"):
                x, y, z = getattr(r, k), getattr(o, k), getattr(a, k)
                assert x is None or (torch.equal(x, y) and torch.equal(x, z)), k


@pytest.mark.parametrize("n,b", [(4096, 3), (40001, 70)])
def test_syndromes(n, b):
    co, code = oc.build(PROFILES["r0.1"], n, 3), met.Code.build(PROFILES["r0.1"], n, 3)
    bits = [np.random.default_rng(k).integers(0, 2, (b, n), dtype=np.uint8) for k in range(3)]
    dev = [torch.from_numpy(x).to(DEV) for x in bits]
    met.syndrome(code, dev[0])
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in bits]
    print("side streams, syndromes", n, b, flush=True)
    outs = []
    for x, st in zip(dev, streams):
        _busy(st)
        outs.append(met.syndrome(code, x, stream=st))
        _overwrite((b * code.M, n * 16, n * 8))
    torch.cuda.synchronize()
    for x, o in zip(bits, outs):
        np.testing.assert_array_equal(o.cpu().numpy(), oc.syndrome(co, x))
