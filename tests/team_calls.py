"""Calls shared by the tests of the team decoder: a decode by teams of a given shape
into outputs that hold values no decode writes, and the same by launches."""
import ctypes
import types

import torch

import paper_1711_01783_amd as met
from paper_1711_01783_amd._lib import (MET_C2V_FP16, MET_C2V_Q8, MET_CHECK_LUT, MET_FIXED_ITERS, check, lib,
                                       met_team_options)

DEV = "cuda:0"
OUTPUTS = ("bits", "iterations", "converged", "posterior")


def outputs(b, n, posterior):
    return types.SimpleNamespace(
        bits=torch.full((b, n), 7, dtype=torch.uint8, device=DEV),
        iterations=torch.full((b,), -5, dtype=torch.int32, device=DEV),
        converged=torch.full((b,), 9, dtype=torch.uint8, device=DEV),
        posterior=torch.full((b, n), float("nan"), dtype=torch.float32, device=DEV) if posterior else None)


def workspace(code, b):
    # states of groups of 16 frames in all eight slots, whatever the batch
    n = max(met.workspace_bytes(code, b, posterior=True), met.workspace_bytes(code, 128, posterior=True)) + (1 << 20)
    return torch.empty(n, dtype=torch.uint8, device=DEV)


def teams(code, llr, syn, max_iter, frames, posterior=False, fixed_iters=False, c2v_fp16=False, c2v_q8=False,
          check_lut=False, ws=None, stream=None, **options):
    b = int(llr.shape[0])
    o = outputs(b, code.N, posterior)
    ws = workspace(code, b) if ws is None else ws
    off = -ws.data_ptr() % 256
    flags = (MET_FIXED_ITERS * fixed_iters | MET_C2V_FP16 * c2v_fp16 | MET_C2V_Q8 * c2v_q8 | MET_CHECK_LUT * check_lut)
    check(lib.met_decode_teams(
        code.handle, llr.data_ptr(), syn.data_ptr(), b, max_iter, flags, o.bits.data_ptr(), o.iterations.data_ptr(),
        o.converged.data_ptr(), o.posterior.data_ptr() if posterior else None, ctypes.c_void_p(ws.data_ptr() + off),
        ws.numel() - off, ctypes.byref(met_team_options(frames=frames, **options)),
        ctypes.c_void_p((stream or torch.cuda.current_stream()).cuda_stream)))
    torch.cuda.synchronize()
    return o


def kernels(f):
    """f() and the names of the kernels that it launched."""
    met.timing_collect()
    met.timing_enable(True)
    try:
        out = f()
        torch.cuda.synchronize()
    finally:
        met.timing_enable(False)
    return out, set(met.timing_collect())


def launches(code, llr, syn, max_iter, **kw):
    # a launch shape asked for selects the launches
    out, used = kernels(lambda: met.decode(code, llr, syn, max_iter, check_steps_per_wave=4, **kw))
    assert "k_team" not in used
    return out


def same(a, b):
    for k in OUTPUTS:
        x, y = getattr(a, k), getattr(b, k)
        assert (x is None) == (y is None) and (x is None or torch.equal(x, y)), k
