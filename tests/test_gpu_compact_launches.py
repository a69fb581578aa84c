"""Compaction and squeezing of running frames by the launches (a launch shape asked
for keeps a small decode from the teams): which of them ran is asserted, and all
outputs equal those of groups left alone, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_1711_01783_amd as met  # noqa: E402
from met_inputs import PROFILES, make_frames  # noqa: E402
from tests import team_calls as tc  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _compare(code, x, llr, max_iter, expect, absent=()):
    d = torch.from_numpy(np.ascontiguousarray(llr, dtype=np.float32)).to(tc.DEV)
    syn = met.syndrome(code, torch.from_numpy(np.ascontiguousarray(x)).to(tc.DEV))
    on, used = tc.kernels(lambda: met.decode(code, d, syn, max_iter, check_steps_per_wave=4))
    off, plain = tc.kernels(lambda: met.decode(code, d, syn, max_iter, check_steps_per_wave=4, compact=False))
    assert expect <= used and not set(absent) & used, used
    assert not {"k_team", "k_compact", "k_squeeze"} & plain
    tc.same(off, on)
    return on


def _slow_in(b, slow, n, seed):
    """Frames that stop at once and, where slow, frames that never do."""
    fast_x, fast = make_frames(n, b, 3.0, seed)
    slow_x, never = make_frames(n, b, 0.02, seed + 1)
    return np.where(slow[:, None], slow_x, fast_x), np.where(slow[:, None], never, fast)


# the running frames of two groups fit in one; so few that the remaining group is
# squeezed to 32 or to 16 lanes at the same iteration; and more than half of a
# group's, where nothing is squeezed
@pytest.mark.parametrize("first,second,squeezed", [((50, 64), (64, 74), True), ((0, 16), (127, 128), True),
                                                   ((60, 64), (64, 70), True), ((20, 64), (64, 80), False)])
def test_moves_between_groups(first, second, squeezed):
    n, b = 8192, 128
    code = met.Code.build(PROFILES["r0.1"], n, 5)
    slow = np.zeros(b, dtype=bool)
    slow[slice(*first)] = slow[slice(*second)] = True
    x, llr = _slow_in(b, slow, n, 77)
    print("compaction", first, second, flush=True)
    on = _compare(code, x, llr, 40, {"k_compact"} | ({"k_squeeze"} if squeezed else set()),
                  () if squeezed else ("k_squeeze",))
    conv, it = on.converged.cpu().numpy(), on.iterations.cpu().numpy()
    assert np.all(conv[~slow] == 1) and np.all(it[~slow] <= 2)
    assert np.all(conv[slow] == 0) and np.all(it[slow] == 40)
    np.testing.assert_array_equal(on.bits.cpu().numpy()[~slow], x[~slow])


@pytest.mark.parametrize("prof,n,b,snr,max_iter", [("r0.1", 16384, 768, 0.19, 60), ("r0.05", 6000, 64 * 5 + 17, 0.12, 48),
                                                   ("r0.02", 9000, 130, 0.065, 80), ("r0.05", 12000, 700, 0.10, 64)])
def test_frames_that_stop_one_by_one(prof, n, b, snr, max_iter):
    code = met.Code.build(PROFILES[prof], n, 8)
    x, llr = make_frames(n, b, snr, 99)
    print("compaction", prof, n, b, flush=True)
    on = _compare(code, x, llr, max_iter, {"k_compact"})
    conv = on.converged == 1
    assert 0.2 < conv.float().mean().item() < 1 and on.iterations[conv].unique().numel() > 5
    got = met.syndrome(code, on.bits)
    want = met.syndrome(code, torch.from_numpy(x).to(tc.DEV))
    assert torch.equal((got == want).all(1), conv)


def test_squeezed_twice():
    """One group whose running frames fall to 32 and then to 16 lanes."""
    n, b = 8192, 64
    code = met.Code.build(PROFILES["r0.1"], n, 5)
    parts = [make_frames(n, b, s, 7) for s in (3.0, 0.23, 0.02)]
    kind = np.repeat([0, 1, 2], (30, 22, 12))[np.random.default_rng(2).permutation(b)]
    x = np.stack([parts[k][0][i] for i, k in enumerate(kind)])
    llr = np.stack([parts[k][1][i] for i, k in enumerate(kind)])
    print("squeezing", np.bincount(kind), flush=True)
    on = _compare(code, x, llr, 100, {"k_squeeze"})
    it = on.iterations.cpu().numpy()
    assert it[kind == 0].max() < 8 and it[kind == 1].max() < 90 and np.all(it[kind == 2] == 100)
