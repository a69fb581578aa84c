"""Squeezing (running frames moved to the lowest lanes of their groups once no
group holds more than 32 or 16) against decodes that keep every lane: a frame's
arithmetic does not depend on its lane, so all outputs are equal bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_1711_01783_amd as met  # noqa: E402
from met_inputs import PROFILES, make_frames  # noqa: E402

DEV = "cuda:0"


def _frames(n, b, snrs, seed):
    parts = [make_frames(n, b, s, seed) for s in snrs]
    pick = np.arange(b) % len(snrs)  # frames of several qualities side by side
    bits = np.stack([parts[k][0][i] for i, k in enumerate(pick)])
    llr = np.stack([parts[k][1][i] for i, k in enumerate(pick)])
    return bits, llr


# one to three groups; a third, a fifth and none of the frames never converge
@pytest.mark.parametrize("n,b,snrs", [(8192, 64, (0.3, 0.25, 0.12)), (8191, 33, (0.3, 0.26, 0.24, 0.22, 0.1)),
                                      (6001, 130, (0.3, 0.1)), (9000, 64, (0.4, 0.3)), (8192, 190, (0.3, 0.25, 0.2, 0.1))])
@pytest.mark.parametrize("store", [dict(), dict(c2v_fp16=True), dict(c2v_q8=True), dict(c2v_q8=True, check_lut=True)])
def test_squeeze_equals_whole_groups(n, b, snrs, store):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("squeeze", n, b, snrs, store, flush=True)
    code = met.Code.build(PROFILES["r0.1"], n, 31)
    bits, llr = _frames(n, b, snrs, 60)
    d = torch.from_numpy(llr).to(DEV)
    syn = met.syndrome(code, torch.from_numpy(bits).to(DEV))
    ref = met.decode(code, d, syn, 70, compact=False, check_steps_per_wave=4, **store)
    met.timing_collect()
    met.timing_enable(True)
    got = met.decode(code, d, syn, 70, check_steps_per_wave=4, **store)
    torch.cuda.synchronize()
    met.timing_enable(False)
    used = met.timing_collect()
    for k in ("bits", "iterations", "converged"):
        assert torch.equal(getattr(ref, k), getattr(got, k)), k
    c = got.converged.float().mean().item()
    if b == 64 and c < 1:  # most frames of the one group stop well before the budget
        assert "k_squeeze" in used


def test_run_time_degrees():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(8)
    n, m, b = 1200, 300, 64
    vn, cn = [], []
    for j in range(m):
        for v in rng.choice(n - 200, int(rng.integers(3, 28)), replace=False):
            vn.append(int(v))
            cn.append(j)
    for k in range(200):
        vn.append(n - 200 + k)
        cn.append(k)
    code = met.Code.from_edges(n, m, vn, cn)
    x = rng.integers(0, 2, (b, n)).astype(np.uint8)
    amp = np.where(np.arange(b) % 4 == 0, 0.9, 6.0)[:, None]
    llr = ((1 - 2.0 * x) * amp + rng.standard_normal((b, n))).astype(np.float32)
    d, syn = torch.from_numpy(llr).to(DEV), met.syndrome(code, torch.from_numpy(x).to(DEV))
    print("squeeze, run-time degrees", flush=True)
    ref = met.decode(code, d, syn, 40, compact=False, check_steps_per_wave=4)
    got = met.decode(code, d, syn, 40, check_steps_per_wave=4)
    for k in ("bits", "iterations", "converged"):
        assert torch.equal(getattr(ref, k), getattr(got, k)), k
