"""Workspaces hold what the path that runs needs: the team decoder's room only where a
decode may run by teams, none in the batched form, and the fixed array of
met_decode_noalloc takes every decode that fits without the frames' flag bytes."""
import ctypes

import pytest

import paper_1711_01783_amd as met
from met_inputs import PROFILES
from paper_1711_01783_amd import _lib

FLAGS = 1024  # bytes per group of 64 frames: one byte per frame and die, two buffers


def _a256(x):
    return -(-x // 256) * 256


def _launches(code, b, c2v=4, w=64):
    """Bytes of the launches' arrays in groups of w frames."""
    st = code.info()
    g = -(-b // w)
    gw, e12, n2, el, m = w * g, st["n_msg_edges"], st["n_msg_vn"], st["n_leaf_edges"], st["M"]
    parts = [max(gw * e12 * c2v, gw * code.N * 4), gw * n2 * 4, gw * n2 * 4, gw * el * 4, g * m * 8, 2 * g * el * 8,
             FLAGS * g, g * 8, gw * 4, 256 + _a256(4 * g) + 64 * 4 * g, 4]
    return sum(_a256(p) for p in parts)


def _batched(code, b):
    jobs = (_lib.met_job * 1)()
    jobs[0].code = code.handle
    jobs[0].llr = jobs[0].syn = jobs[0].bits = jobs[0].iters = jobs[0].converged = 256
    jobs[0].B, jobs[0].max_iter = b, 20
    n = ctypes.c_size_t()
    assert _lib.lib.met_batched_workspace_bytes(jobs, 1, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("prof,n,b", [("r0.1", 262144, 64), ("r0.02", 1000000, 64), ("r0.1", 300001, 128)])
def test_no_room_for_teams_where_none_fits(prof, n, b):
    code = met.Code.build(PROFILES[prof], n, 3)
    assert met.workspace_bytes(code, b) == _launches(code, b)
    assert met.workspace_bytes(code, b, c2v_q8=True) == _launches(code, b, c2v=1)


def test_batched_jobs_hold_no_room_for_teams():
    code = met.Code.build(PROFILES["r0.1"], 65536, 3)
    small = met.Code.build(PROFILES["r0.02"], 4096, 3)

    def control(c, b):  # beside the launches' arrays, in the widest of the groups it may be tuned to take
        return _batched(c, b) - max(_launches(c, b, w=w) for w in (16, 32, 64))

    assert 0 < control(code, 64) == control(code, 640) == control(small, 200) == control(small, 17)


def test_a_workspace_for_more_frames_serves_fewer():
    for prof, n in (("r0.1", 4096), ("r0.05", 65536), ("r0.1", 150001)):
        code = met.Code.build(PROFILES[prof], n, 3)
        for kw in (dict(), dict(posterior=True)):
            need = [met.workspace_bytes(code, b, **kw) for b in range(1, 300)]
            assert need == sorted(need)
        for kw in (dict(c2v_fp16=True), dict(c2v_q8=True, posterior=True)):
            need = [met.workspace_bytes(code, b, **kw) for b in range(33, 300)]
            assert need == sorted(need)


@pytest.mark.parametrize("n,b", [(4209, 3904), (4357, 3776), (4096, 3968), (65536, 192)])
def test_noalloc_takes_what_it_took(n, b):
    """Decodes whose arrays fit in the fixed array with a word of flags per group are
    not refused for their size (they fail later: the code is on no device), and
    those beyond it are."""
    code = met.Code.build(PROFILES["r0.1"], n, 3)
    size = _lib.MET_NOALLOC_SCRATCH_BYTES

    def before(frames):  # with one word per group and buffer for the flags
        g = -(-frames // 64)
        return _launches(code, frames) - FLAGS * g + _a256(16 * g)

    assert before(b) <= size < before(b + 64)
    P = ctypes.c_void_p

    def call(frames):
        return _lib.lib.met_decode_noalloc(code.handle, P(256), P(256), frames, 10, 0, P(256), P(256), P(256), None, None)

    def refused(frames):
        rc = call(frames)
        return rc == -1 and "scratch" in _lib.lib.met_last_error().decode()

    assert not refused(b) and refused(b + 64)
