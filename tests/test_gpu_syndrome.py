"""Packed syndromes against the oracle's H x mod 2, exactly: word widths of 8 to 64
frames, several groups, odd lengths (unaligned rows) and bytes with more than
bit 0 set."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_1711_01783_amd as met  # noqa: E402
from met_inputs import PROFILES  # noqa: E402
from oracle import code as oc  # noqa: E402
from paper_1711_01783_amd._lib import check, lib  # noqa: E402


@pytest.mark.parametrize("n", [1000, 1001, 1003, 4098])
@pytest.mark.parametrize("b", [1, 8, 9, 16, 17, 32, 33, 64, 65, 130])
def test_packed_syndrome(n, b):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("syndrome", n, b, flush=True)
    prof = PROFILES["r0.1" if n % 2 else "r0.05"]
    co, cg = oc.build(prof, n, 3), met.Code.build(prof, n, 3)
    raw = np.random.default_rng(n + b).integers(0, 256, (b, n), dtype=np.uint8)
    ref = oc.syndrome(co, raw & 1)
    d = torch.from_numpy(raw).cuda()
    got = met.syndrome(cg, d)  # few gathers: the plain launch
    plain, packed = torch.empty_like(got), torch.empty_like(got)
    need = ctypes.c_size_t()
    check(lib.met_syndrome_workspace_bytes(cg.handle, b, ctypes.byref(need)))
    ws = torch.full((need.value,), 255, dtype=torch.uint8, device="cuda")
    check(lib.met_syndrome_ex(cg.handle, d.data_ptr(), b, packed.data_ptr(), ws.data_ptr(), need.value,
                              ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    np.testing.assert_array_equal(packed.cpu().numpy(), ref)
    check(lib.met_syndrome(cg.handle, d.data_ptr(), b, plain.data_ptr(),
                           ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    np.testing.assert_array_equal(got.cpu().numpy(), ref)
    np.testing.assert_array_equal(plain.cpu().numpy(), ref)


def test_large_batches_are_packed():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, b = 40001, 70
    co, cg = oc.build(PROFILES["r0.1"], n, 3), met.Code.build(PROFILES["r0.1"], n, 3)
    assert b * cg.E >= met.api._PACKED_SYNDROME_GATHERS
    bits = np.random.default_rng(1).integers(0, 2, (b, n), dtype=np.uint8)
    got = met.syndrome(cg, torch.from_numpy(bits).cuda())
    np.testing.assert_array_equal(got.cpu().numpy(), oc.syndrome(co, bits))
