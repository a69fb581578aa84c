"""Memory that a call with ``stream=`` allocates for itself comes from that stream:
the caching allocator hands freed memory out again in the order of the stream it
was allocated on, so a workspace from the caller's current stream would get its
next owner while `stream` still decodes in it.  The library and the streams are
stand-ins; no GPU."""
import contextlib
import types

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1711_01783_amd as met  # noqa: E402
from met_inputs import PROFILES  # noqa: E402
from paper_1711_01783_amd import api, wbp  # noqa: E402


class _Stream:
    cuda_stream = 7


SIDE, CURRENT = _Stream(), types.SimpleNamespace(cuda_stream=1)


@pytest.fixture
def seen(monkeypatch):
    """Records the stream each tensor is allocated on and marked as used on, and
    checks every pointer that a library call gets against the allocations."""
    active, blocks, marked, calls = [CURRENT], [], [], []

    @contextlib.contextmanager
    def on(s):
        active.append(s)
        try:
            yield
        finally:
            active.pop()

    real_empty, real_like = torch.empty, torch.empty_like

    def track(t):
        blocks.append((t.data_ptr(), t.numel() * t.element_size(), active[-1], t))
        return t

    monkeypatch.setattr(torch.cuda, "Stream", _Stream)
    monkeypatch.setattr(torch.cuda, "stream", on)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: active[-1])
    monkeypatch.setattr(torch, "empty", lambda *a, **k: track(real_empty(*a, **k)))
    monkeypatch.setattr(torch, "empty_like", lambda *a, **k: track(real_like(*a, **k)))
    monkeypatch.setattr(torch.Tensor, "record_stream", lambda t, s: marked.append((t.data_ptr(), s)))
    monkeypatch.setattr(api, "_require", lambda *a: None)
    monkeypatch.setattr(wbp, "_check_weights", lambda *a: None)

    class Lib:
        def __getattr__(self, name):
            if name.endswith("_bytes") or name.startswith("met_code_"):
                return getattr(met.lib, name)

            def call(*args):
                ints = [getattr(a, "value", a) for a in args]
                for a in args:
                    if hasattr(a, "_length_"):  # an array of jobs
                        ints += [getattr(j, f) for j in a for f in ("bits", "iters", "converged")]
                for a in ints:
                    for p, size, s, _ in blocks:
                        if isinstance(a, int) and p <= a < p + max(size, 1):
                            calls.append((name, p, s))
                return 0

            return call

    monkeypatch.setattr(api, "lib", Lib())
    monkeypatch.setattr(wbp, "lib", Lib())
    return types.SimpleNamespace(blocks=blocks, marked=marked, calls=calls, given=torch.zeros)


def _cases():
    n, b, prof = 4096, 64, "r0.1"

    def decode(code, z):
        o = met.decode(code, z(b, n), z(b, code.M, dtype=torch.uint8), 5, stream=SIDE, posterior=True)
        return [o.bits, o.iterations, o.converged, o.posterior], 5

    def few_syndromes(code, z):
        return [met.syndrome(code, z(b, n, dtype=torch.uint8), stream=SIDE)], 1

    def packed_syndromes(code, z):
        k = -(-api._PACKED_SYNDROME_GATHERS // code.E)
        return [met.syndrome(code, z(k, n, dtype=torch.uint8), stream=SIDE)], 2

    def bob(code, z):
        return list(met.mdr_bob(z(b, n), z(b, n, dtype=torch.uint8), stream=SIDE)), 2

    def alice(code, z):
        return [met.mdr_alice(z(b, n), z(b, n), z(b, n // 8), 1.0, stream=SIDE)], 1

    def batched(code, z):
        o = met.decode_batched([met.Job(code, z(b, n), z(b, code.M, dtype=torch.uint8), 5)], stream=SIDE)[0]
        return [o.bits, o.iterations, o.converged], 4

    def weighted(code, z):
        w = z(code.info()["n_edge_types"], 4)
        post, bits, conv, ws = wbp.forward(code, z(b, n), z(b, code.M, dtype=torch.uint8), w, stream=SIDE)
        return [post, bits, conv, wbp.backward(code, z(b, n), w, 0, ws, stream=SIDE)], 6

    return [decode, few_syndromes, packed_syndromes, bob, alice, batched, weighted]


@pytest.mark.parametrize("call", _cases(), ids=lambda f: f.__name__)
def test_memory_of_a_call_comes_from_its_stream(call, seen):
    code = met.Code.build(PROFILES["r0.1"], 4096, 3)
    outs, least = call(code, seen.given)
    assert len({(n, p) for n, p, _ in seen.calls}) >= least
    for name, _, s in seen.calls:
        assert s is SIDE, name
    for o in outs:  # read (and freed) by the caller on its own stream
        assert (o.data_ptr(), CURRENT) in seen.marked


def test_without_a_stream_nothing_changes(seen):
    code = met.Code.build(PROFILES["r0.1"], 4096, 3)
    met.decode(code, seen.given(3, 4096), seen.given(3, code.M, dtype=torch.uint8), 5)
    assert seen.calls and all(s is CURRENT for _, _, s in seen.calls) and not seen.marked
