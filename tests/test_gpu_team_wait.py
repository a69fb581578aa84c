"""A team whose wait for its members is cut short (a tiny limit from the host) ends,
and says so: a frame has either its full result or negative iterations, not converged."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_1711_01783_amd as met  # noqa: E402
from met_inputs import PROFILES, make_frames  # noqa: E402
from tests import team_calls as tc  # noqa: E402


@pytest.mark.parametrize("b,frames", [(8, 1), (70, 4)])
@pytest.mark.parametrize("polls", [1, 4, 32])
def test_a_given_up_frame_is_marked(b, frames, polls):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    code = met.Code.build(PROFILES["r0.1"], 4099, 17)
    bits, llr = make_frames(4099, b, 0.25, 40 + b)
    d = torch.from_numpy(llr).to(tc.DEV)
    syn = met.syndrome(code, torch.from_numpy(bits).to(tc.DEV))
    ref = tc.launches(code, d, syn, 20, posterior=True)
    print("teams that wait for", polls, "polls, frames", b, "in groups of", frames, flush=True)
    got = tc.teams(code, d, syn, 20, frames, posterior=True, polls=polls)
    lost = got.iterations < 0
    assert not got.converged[lost].any()
    for k in tc.OUTPUTS:
        assert torch.equal(getattr(got, k)[~lost], getattr(ref, k)[~lost]), k
    if polls == 1:  # no team forms within two looks at its leader's word
        assert lost.any()
    tc.same(ref, tc.teams(code, d, syn, 20, frames, posterior=True))
