"""Team decoding (one launch, small frame groups per accelerator die) against the
per-phase launches: the same arithmetic in the same order, so every output is
equal bit for bit (tolerance 0), for every group width, lane split and storage,
with run-time check degrees, ragged groups and posteriors."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_1711_01783_amd as met  # noqa: E402
from met_inputs import PROFILES, make_frames  # noqa: E402

DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _launches(code, llr, syn, max_iter, **kw):
    # asking for a launch shape selects the per-phase launches
    return met.decode(code, llr, syn, max_iter, check_steps_per_wave=4, **kw)


def _kernels(f):
    met.timing_collect()
    met.timing_enable(True)
    try:
        out = f()
        torch.cuda.synchronize()
    finally:
        met.timing_enable(False)
    return out, set(met.timing_collect())


def _compare(code, llr, syn, max_iter, team=True, **kw):
    print("team decode", tuple(llr.shape), max_iter, kw, flush=True)
    ref, plain = _kernels(lambda: _launches(code, llr, syn, max_iter, **kw))
    got, used = _kernels(lambda: met.decode(code, llr, syn, max_iter, **kw))
    assert "k_team" not in plain
    if team is not None:  # None: the rule may send it either way
        assert ("k_team" in used) == team
    for k in ("bits", "iterations", "converged", "posterior"):
        a, b = getattr(ref, k), getattr(got, k)
        assert (a is None and b is None) or torch.equal(a, b), k
    return got


# frames and lengths around the group widths (1, 2, 4, 8, 16 frames per group, 8
# groups at a time), full and partial tiles, degrees 24 to 99
@pytest.mark.parametrize("prof,n,b", [("r0.1", 4096, 1), ("r0.1", 4097, 3), ("r0.05", 5003, 9), ("r0.1", 16384, 16),
                                      ("r0.02", 8001, 17), ("r0.1", 8192, 33), ("r0.1", 4099, 64),
                                      ("r0.02", 16001, 65), ("r0.1", 4500, 131), ("r0.05", 9001, 257)])
@pytest.mark.parametrize("mode", ["early", "fixed", "early+post", "fixed+post"])
def test_team_equals_launches(prof, n, b, mode):
    code = met.Code.build(PROFILES[prof], n, 11)
    bits, llr = make_frames(n, b, {"r0.1": 0.24, "r0.05": 0.13, "r0.02": 0.08}[prof], 900 + b)
    syn = met.syndrome(code, torch.from_numpy(bits).to(DEV))
    out = _compare(code, torch.from_numpy(llr).to(DEV), syn, 25, team=None if "fixed" in mode else True,
                   fixed_iters="fixed" in mode, posterior="post" in mode)
    if mode == "early":
        c = out.converged.cpu().numpy() == 1
        again = met.syndrome(code, out.bits).cpu().numpy()
        np.testing.assert_array_equal((again == syn.cpu().numpy()).all(1), c)


@pytest.mark.parametrize("store", [dict(c2v_fp16=True), dict(c2v_q8=True), dict(c2v_q8=True, check_lut=True)])
@pytest.mark.parametrize("n,b", [(4099, 33), (16384, 64), (6001, 150)])
def test_reduced_storage(store, n, b):
    code = met.Code.build(PROFILES["r0.1"], n, 12)
    bits, llr = make_frames(n, b, 0.23, 77)
    syn = met.syndrome(code, torch.from_numpy(bits).to(DEV))
    for kw in (dict(), dict(fixed_iters=True, posterior=True)):
        _compare(code, torch.from_numpy(llr).to(DEV), syn, 20, team=None if kw else True, **store, **kw)


@pytest.mark.parametrize("b", [1, 2, 6, 20, 64])
def test_run_time_degrees(b):
    rng = np.random.default_rng(5)
    n, m = 900, 260
    vn, cn = [], []
    for j in range(m):  # degrees 2 to 32, message and degree-1 nodes mixed
        for v in rng.choice(n - 200, int(rng.integers(2, 30)), replace=False):
            vn.append(int(v))
            cn.append(j)
    for k in range(200):
        vn.append(n - 200 + k)
        cn.append(int(rng.integers(0, m)) if k else 0)
    deg = np.bincount(cn, minlength=m)
    keep = [k for k in range(len(vn)) if deg[cn[k]] <= 32]
    code = met.Code.from_edges(n, m, [vn[k] for k in keep], [cn[k] for k in keep]) if deg[deg > 32].size == 0 else None
    if code is None:
        pytest.skip("degree beyond the limit")
    x = rng.integers(0, 2, (b, n)).astype(np.uint8)
    llr = ((1 - 2.0 * x) * 1.8 + 1.3 * rng.standard_normal((b, n))).astype(np.float32)
    d = torch.from_numpy(x).to(DEV)
    for kw in (dict(), dict(fixed_iters=True), dict(posterior=True)):
        _compare(code, torch.from_numpy(llr).to(DEV), met.syndrome(code, d), 15, team=None, **kw)


def test_extreme_inputs():
    """Zero, infinite and type-limit LLRs (erased, known and saturated bits)."""
    n, b = 4096, 8
    code = met.Code.build(PROFILES["r0.1"], n, 13)
    bits, llr = make_frames(n, b, 0.26, 5)
    llr[0, ::7] = 0.0
    llr[1, ::5] = np.where(bits[1, ::5] == 1, -np.inf, np.inf)
    llr[2, ::3] = np.where(bits[2, ::3] == 1, np.float32(-3.0e38), np.float32(3.0e38))
    llr[3, ::9] = -0.0
    llr[4] = 0.0
    syn = met.syndrome(code, torch.from_numpy(bits).to(DEV))
    for kw in (dict(), dict(fixed_iters=True, posterior=True)):
        _compare(code, torch.from_numpy(llr).to(DEV), syn, 12, **kw)


def test_streams_and_capture():
    """Concurrent team decodes on four streams, and one in a captured graph
    replayed with new inputs between eager decodes."""
    n, b = 8192, 24
    code = met.Code.build(PROFILES["r0.1"], n, 14)
    ins = []
    for k in range(4):
        bits, llr = make_frames(n, b, 0.22, 100 * k)
        ins.append((torch.from_numpy(llr).to(DEV), met.syndrome(code, torch.from_numpy(bits).to(DEV))))
    ref = [_launches(code, l, s, 40) for l, s in ins]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in ins]
    own = [torch.empty(met.workspace_bytes(code, b) + 256, dtype=torch.uint8, device=DEV) for _ in ins]
    torch.cuda.synchronize()
    print("team decodes on 4 streams", flush=True)
    for rep in range(3):
        outs = [met.decode(code, l, s, 40, stream=st, workspace=w) for (l, s), st, w in zip(ins, streams, own)]
        torch.cuda.synchronize()
        for r, o in zip(ref, outs):
            assert torch.equal(r.bits, o.bits) and torch.equal(r.iterations, o.iterations)
    llr, syn = ins[0][0].clone(), ins[0][1].clone()
    ws = torch.empty(met.workspace_bytes(code, b) + 256, dtype=torch.uint8, device=DEV)
    print("team decode in a graph", flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = met.decode(code, llr, syn, 40, workspace=ws)
    for k in (0, 2, 1, 3):
        llr.copy_(ins[k][0])
        syn.copy_(ins[k][1])
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.bits, ref[k].bits) and torch.equal(out.iterations, ref[k].iterations)
        met.decode(code, *ins[(k + 1) % 4], 40)


def test_large_decodes_keep_the_launches():
    code = met.Code.build(PROFILES["r0.1"], 300000, 15)
    bits, llr = make_frames(300000, 64, 0.3, 9)
    syn = met.syndrome(code, torch.from_numpy(bits).to(DEV))
    _compare(code, torch.from_numpy(llr).to(DEV), syn, 12, team=False)


@pytest.mark.parametrize("n,b,kw", [(200003, 16, dict()), (150001, 32, dict(posterior=True, fixed_iters=True)),
                                    (140003, 65, dict()), (150001, 64, dict(c2v_fp16=True, fixed_iters=True))])
def test_all_classes_in_one_launch(n, b, kw):
    """Four check classes (degrees 11, 12, 2+1 and 3+1) in one launch against the
    same classes in the batched decoder's launches, or, where that has no such
    option, against the class kernels' other step counts: equal bit for bit."""
    code = met.Code.build(PROFILES["r0.05"], n, 21)
    assert len(code.classes()) >= 3
    bits, llr = make_frames(n, b, 0.115, 40)
    d_llr, syn = torch.from_numpy(llr).to(DEV), met.syndrome(code, torch.from_numpy(bits).to(DEV))
    print("check set", n, b, kw, flush=True)
    got, used = _kernels(lambda: met.decode(code, d_llr, syn, 14, compact=False, **kw))
    assert "k_check_set" in used and "k_check<3,1>" not in used
    if kw.get("c2v_fp16"):  # the same frames with 25 others: past the size of one launch per update
        more_bits, more = make_frames(n, 192, 0.115, 41)
        more[:b] = llr
        syn2 = torch.cat([syn, met.syndrome(code, torch.from_numpy(more_bits[b:]).to(DEV))])
        ref, sep = _kernels(lambda: met.decode(code, torch.from_numpy(more).to(DEV), syn2, 14, compact=False, **kw))
        assert "k_check<3,1>" in sep
        assert torch.equal(ref.bits[:b], got.bits) and torch.equal(ref.converged[:b], got.converged)
        return
    ref = met.BatchedDecoder(phase_launches=True, stagger=False)([met.Job(code, d_llr, syn, 14, kw.get("fixed_iters", False))])[0]
    for k in ("bits", "iterations", "converged"):
        assert torch.equal(getattr(ref, k), getattr(got, k)), k
