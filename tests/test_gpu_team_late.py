"""Teams whose workgroups come late (other work holds compute units when the launch
begins): they are taken in while the team decodes, with results equal to the
launches' bit for bit, and the decode runs at the whole team's speed soon after."""
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


def _inputs(prof, n, b, snr):
    code = met.Code.build(PROFILES[prof], n, 19)
    bits, llr = make_frames(n, b, snr, 70 + b)
    return code, torch.from_numpy(llr).to(tc.DEV), met.syndrome(code, torch.from_numpy(bits).to(tc.DEV))


# delays within the wait for a whole team, beyond it, and beyond most of the decode
@pytest.mark.parametrize("late_us", [2, 15, 60, 400])
@pytest.mark.parametrize("prof,n,b,frames,snr,store", [
    ("r0.1", 4099, 3, 1, 0.24, dict()), ("r0.05", 9001, 16, 2, 0.13, dict()), ("r0.02", 8001, 70, 4, 0.08, dict()),
    ("r0.1", 16384, 40, 8, 0.22, dict(c2v_fp16=True)), ("r0.1", 16384, 40, 16, 0.22, dict(c2v_q8=True, check_lut=True))])
def test_late_workgroups(prof, n, b, frames, snr, store, late_us):
    code, d, syn = _inputs(prof, n, b, snr)
    for kw in (dict(), dict(fixed_iters=True, posterior=True)):
        print("late teams", prof, n, b, "frames in groups of", frames, store, kw, late_us, "us", flush=True)
        tc.same(tc.launches(code, d, syn, 40, **store, **kw),
                tc.teams(code, d, syn, 40, frames, late_us=late_us, **store, **kw))


def test_a_team_grows_to_its_full_size():
    code, d, syn = _inputs("r0.1", 65536, 8, 0.19)

    def ms(late_us):
        met.timing_collect()
        met.timing_enable(True)
        tc.teams(code, d, syn, 600, 1, fixed_iters=True, late_us=late_us)
        met.timing_enable(False)
        return met.timing_collect()["k_team"][1]

    ms(0)
    whole, late = ms(0), ms(60)
    print("600 iterations: whole teams %.2f ms, with workgroups up to 420 us late %.2f ms" % (whole, late), flush=True)
    # an eighth of a team takes several times as long to the end
    assert late < 1.5 * whole + 1.0
