"""Weighted BP on classes of checks with one type of message edges (scales and
gradient sums per class) against the same graph with some of those edges given
another type of the same scale (scales and sums per edge): posteriors are equal
bit for bit, gradients add up."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_1711_01783_amd as met  # noqa: E402
from paper_1711_01783_amd import wbp  # noqa: E402
from met_inputs import PROFILES, make_frames  # noqa: E402

DEV = "cuda:0"


def _relabelled(code, which):
    """The last type-1 edge of the checks of `which` as type 3, the last type-0
    edge as type 4: edges keep their order within the checks."""
    vn, cn, et = code.export()
    et = et.copy()
    for t, other in ((1, 3), (0, 4)):
        pos = np.flatnonzero(et == t)
        last = pos[np.r_[cn[pos][1:] != cn[pos][:-1], True]]
        et[last[which(cn[last])]] = other
    return met.Code.from_edges(code.N, code.M, vn, cn, et)


# every width of a group; all checks (one type per position) or every other one
@pytest.mark.parametrize("prof,n,b", [("r0.1", 2010, 1), ("r0.05", 3000, 3), ("r0.02", 4001, 9), ("r0.1", 4096, 32),
                                      ("r0.02", 2550, 65)])
@pytest.mark.parametrize("every", [1, 2])
def test_class_scales_equal_edge_scales(prof, n, b, every):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("types", prof, n, b, every, flush=True)
    it = 5
    one = met.Code.build(PROFILES[prof], n, 12)
    two = _relabelled(one, lambda j: j % every == 0)
    bits, llr = make_frames(n, b, 0.2, 71)
    d, bt = torch.from_numpy(llr).to(DEV), torch.from_numpy(bits).to(DEV)
    syn = met.syndrome(one, bt)
    w = 1.0 + 0.1 * np.random.default_rng(5).standard_normal((3, it)).astype(np.float32)
    s = 1.0 - 2.0 * bt.float()
    res = []
    for code, rows in ((one, [0, 1, 2]), (two, [0, 1, 2, 1, 0])):
        wt = torch.from_numpy(np.ascontiguousarray(w[rows])).to(DEV).requires_grad_(True)
        post = wbp.weighted_bp(wt, code, d, syn, 2)
        torch.nn.functional.softplus(-s * post).mean().backward()
        res.append((post.detach(), wt.grad.double()))
    (p1, g1), (p2, g2) = res
    assert torch.equal(p1, p2)
    summed = g2[:3].clone()
    summed[1] += g2[3]
    summed[0] += g2[4]
    # the tolerance of the comparison with the 64-bit oracle
    assert torch.allclose(g1, summed, rtol=2e-3, atol=2e-4 * g1.abs().max().item())
    assert torch.all(g1[2, :-1] == 0)
