"""Every compiled form of the team decoder (frames per group, storage, lanes per
variable node, run-time degrees), whatever the rule would take, against the
launches, bit for bit; and posteriors of check classes in one launch against the
same classes launched apart."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_1711_01783_amd as met  # noqa: E402
from met_inputs import PROFILES, make_frames  # noqa: E402
from tests import team_calls as tc  # noqa: E402

STORES = [(w, dict()) for w in (1, 2, 4, 8, 16)]
STORES += [(w, s) for w in (4, 8, 16) for s in (dict(c2v_fp16=True), dict(c2v_q8=True), dict(c2v_q8=True, check_lut=True))]
MODES = [dict(), dict(fixed_iters=True), dict(posterior=True), dict(fixed_iters=True, posterior=True)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _compare(code, d, syn, max_iter, frames, store, **kw):
    ref = tc.launches(code, d, syn, max_iter, **store, **kw)
    got, used = tc.kernels(lambda: tc.teams(code, d, syn, max_iter, frames, **store, **kw))
    assert used == {"k_team"}
    tc.same(ref, got)


# degrees up to 24, 49 and 99: 1, 4 and 16 lanes per node, by the size of the groups
@pytest.mark.parametrize("frames,store", STORES)
@pytest.mark.parametrize("prof,n,snr", [("r0.1", 4099, 0.24), ("r0.05", 9001, 0.13), ("r0.02", 4100, 0.085),
                                        ("r0.02", 20001, 0.075)])
def test_widths_and_storage(prof, n, snr, frames, store):
    code = met.Code.build(PROFILES[prof], n, 23)
    b = max(3 * frames + 1, 33 if store else 1)
    bits, llr = make_frames(n, b, snr, 60)
    d, syn = torch.from_numpy(llr).to(tc.DEV), met.syndrome(code, torch.from_numpy(bits).to(tc.DEV))
    for kw in MODES:
        print("teams", prof, n, b, "frames in groups of", frames, store, kw, flush=True)
        _compare(code, d, syn, 25, frames, store, **kw)


# the nodes of one frame take 16 lanes each up to the first length, 4 from the second
@pytest.mark.parametrize("n", [68001, 69001])
def test_lanes_per_node(n):
    code = met.Code.build(PROFILES["r0.02"], n, 23)
    bits, llr = make_frames(n, 2, 0.07, 61)
    d, syn = torch.from_numpy(llr).to(tc.DEV), met.syndrome(code, torch.from_numpy(bits).to(tc.DEV))
    print("teams, one frame per group of", n, flush=True)
    _compare(code, d, syn, 12, 1, {})


@pytest.mark.parametrize("frames,store", STORES)
def test_run_time_degrees(frames, store):
    rng = np.random.default_rng(5)
    n, m = 900, 260
    vn, cn = [], []
    for j in range(m):  # degrees 3 to 32, message and degree-1 nodes mixed
        for v in rng.choice(n - 200, int(rng.integers(2, 30)), replace=False):
            vn.append(int(v))
            cn.append(j)
    for k in range(200):  # at most one each
        vn.append(n - 200 + k)
        cn.append(k)
    code = met.Code.from_edges(n, m, vn, cn)
    b = max(2 * frames + 1, 35 if store else 1)
    x = rng.integers(0, 2, (b, n)).astype(np.uint8)
    llr = ((1 - 2.0 * x) * 1.8 + 1.3 * rng.standard_normal((b, n))).astype(np.float32)
    d, syn = torch.from_numpy(llr).to(tc.DEV), met.syndrome(code, torch.from_numpy(x).to(tc.DEV))
    for kw in MODES:
        print("teams, run-time degrees,", b, "frames in groups of", frames, store, kw, flush=True)
        _compare(code, d, syn, 15, frames, store, **kw)


@pytest.mark.parametrize("b", [20, 32, 40])
def test_posteriors_of_classes_in_one_launch(b):
    n = 150001
    code = met.Code.build(PROFILES["r0.05"], n, 21)
    bits, llr = make_frames(n, 192, 0.115, 41)
    d, syn = torch.from_numpy(llr).to(tc.DEV), met.syndrome(code, torch.from_numpy(bits).to(tc.DEV))
    print("posteriors of", b, "frames, and of the same among 192", flush=True)
    for kw in (dict(), dict(fixed_iters=True)):
        one, used = tc.kernels(lambda: met.decode(code, d[:b], syn[:b], 14, posterior=True, check_steps_per_wave=4, **kw))
        apart, sep = tc.kernels(lambda: met.decode(code, d, syn, 14, posterior=True, check_steps_per_wave=4, **kw))
        assert "k_check_set" in used and "k_check<3,1>" not in used
        assert "k_check<3,1>" in sep and "k_check_set" not in sep
        for k in tc.OUTPUTS:
            assert torch.equal(getattr(one, k), getattr(apart, k)[:b]), k
