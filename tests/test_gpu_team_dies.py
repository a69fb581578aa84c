"""Teams on fewer dies than a batch has groups in its first round (a partitioned
device shows fewer): every frame is decoded, equal to the launches bit for bit."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_1711_01783_amd as met  # noqa: E402
from met_inputs import PROFILES, make_frames  # noqa: E402
from tests import team_calls as tc  # noqa: E402


# one round of 8 groups, an incomplete one with a ragged group, two rounds and a bit
@pytest.mark.parametrize("b,frames", [(16, 2), (5, 1), (70, 4)])
@pytest.mark.parametrize("dies", [1, 2, 3, 7, 8])
def test_every_group_is_decoded(b, frames, dies):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    code = met.Code.build(PROFILES["r0.1"], 4099, 17)
    bits, llr = make_frames(4099, b, 0.25, 40 + b)
    d = torch.from_numpy(llr).to(tc.DEV)
    syn = met.syndrome(code, torch.from_numpy(bits).to(tc.DEV))
    for kw in (dict(), dict(fixed_iters=True, posterior=True)):
        print("teams on", dies, "dies, frames", b, "in groups of", frames, kw, flush=True)
        tc.same(tc.launches(code, d, syn, 20, **kw), tc.teams(code, d, syn, 20, frames, dies=dies, **kw))
