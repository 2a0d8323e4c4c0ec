"""ctqw_set_state / ctqw_get_state on device buffers that end before the state:
refused before anything is written, whatever the alignment; the state and a
whole buffer's copies are untouched by the refusal.  Buffers of virtual memory
mapped in several pieces hold as much as their pieces together.  Large states
come out and go back bit for bit."""

import ctypes as C

import numpy as np
import pytest

from _helpers import gpu_plan, say

pytestmark = pytest.mark.gpu


def hip_runtime():
    """The HIP runtime that this process has loaded (torch's)."""
    with open("/proc/self/maps") as f:
        path = next(l.split()[-1] for l in f if "libamdhip64" in l)
    return C.CDLL(path)


@pytest.mark.parametrize("N,dtype", [(40, "c64"), (40, "c128"), (300, "c64")])
def test_short_device_buffers_are_refused(N, dtype):
    from paper_1612_00746_amd import _lib as L
    plan = gpu_plan(m=2, statistics="distinguishable", boundary="open", interaction="onsite", dtype=dtype,
                    reals=[(N, np.ones(N - 1), np.zeros(N), 1.0)], dt=0.05, order=4, sites=[1, 2])
    psi = plan.state_numpy()
    hip = hip_runtime()
    size, buf = psi.nbytes, C.c_void_p()
    assert hip.hipMalloc(C.byref(buf), C.c_size_t(size)) == 0
    # the address and what is left of the allocation: whole, an element short, half
    for skip in (0, psi.itemsize, size // 2):
        at = C.c_void_p(buf.value + skip)
        got, put = plan.lib.ctqw_get_state(plan.h, at, 1), plan.lib.ctqw_set_state(plan.h, at, 1)
        say(f"case: state copies N={N} {dtype}, buffer short by {skip} bytes: {got}, {put}")
        assert (got, put) == ((0, 0) if skip == 0 else (L.ERR_DEVICE, L.ERR_DEVICE))
        assert np.array_equal(plan.state_numpy(), psi)
    assert hip.hipFree(buf) == 0


class AllocationProp(C.Structure):
    """hipMemAllocationProp of plain device memory."""
    _fields_ = [("type", C.c_int), ("handle", C.c_int), ("location", C.c_int), ("device", C.c_int),
                ("win32", C.c_void_p), ("flags", C.c_uint32)]


class AccessDesc(C.Structure):
    _fields_ = [("location", C.c_int), ("device", C.c_int), ("flags", C.c_int)]


def test_buffers_mapped_in_pieces():
    """A state across two mappings is read and written like any other."""
    N = 600                                            # 5.8 MB of complex128
    plan = gpu_plan(m=2, statistics="distinguishable", boundary="open", interaction="onsite", dtype="c128",
                    reals=[(N, np.ones(N - 1), np.zeros(N), 1.0)], dt=0.05, order=4, sites=[1, 2])
    plan.propagate(3)
    psi = plan.state_numpy()
    hip, piece = hip_runtime(), 4 << 20
    assert piece < psi.nbytes < 2 * piece
    prop, va, hands = AllocationProp(type=1, location=1), C.c_void_p(), []
    assert hip.hipMemAddressReserve(C.byref(va), C.c_size_t(2 * piece), C.c_size_t(0), None, C.c_uint64(0)) == 0
    for i in range(2):
        h = C.c_void_p()
        assert hip.hipMemCreate(C.byref(h), C.c_size_t(piece), C.byref(prop), C.c_uint64(0)) == 0
        assert hip.hipMemMap(C.c_void_p(va.value + i * piece), C.c_size_t(piece), C.c_size_t(0), h, C.c_uint64(0)) == 0
        hands.append(h)
    acc = AccessDesc(location=1, flags=3)
    assert hip.hipMemSetAccess(va, C.c_size_t(2 * piece), C.byref(acc), C.c_size_t(1)) == 0
    say("case: state copies across two mappings")
    assert plan.lib.ctqw_get_state(plan.h, va, 1) == 0
    host = np.empty_like(psi)
    assert hip.hipMemcpy(host.ctypes.data_as(C.c_void_p), va, C.c_size_t(psi.nbytes), C.c_int(2)) == 0
    assert np.array_equal(host, psi)
    plan.propagate(2)
    assert not np.array_equal(plan.state_numpy(), psi)
    assert plan.lib.ctqw_set_state(plan.h, va, 1) == 0
    assert np.array_equal(plan.state_numpy(), psi)
    for i, h in enumerate(hands):
        assert hip.hipMemUnmap(C.c_void_p(va.value + i * piece), C.c_size_t(piece)) == 0
        assert hip.hipMemRelease(h) == 0
    assert hip.hipMemAddressFree(va, C.c_size_t(2 * piece)) == 0


@pytest.mark.parametrize("N,R,dtype", [(1201, 12, "c64"), (849, 12, "c128"), (1201, 25, "c64")])
def test_large_states_out_and_back(N, R, dtype):
    """States of more than 128 MB (a kernel's copy where the buffer is 16-byte
    aligned, stored to the last-level cache or past it), with an odd number of
    amplitudes and off by one amplitude: the same bits out and back."""
    import torch
    g = np.random.default_rng(N)
    reals = [(N, 1 + 0.1 * g.standard_normal(N - 1), np.zeros(N), 1.0) for _ in range(R)]
    plan = gpu_plan(m=2, statistics="distinguishable", boundary="open", interaction="onsite", dtype=dtype, reals=reals,
                    dt=0.05, order=4, sites=[N // 2, N // 3])
    plan.propagate(3)
    psi = plan.state_numpy()
    assert psi.nbytes > 128 << 20
    for skip in (0, psi.itemsize):
        say(f"case: state copies N={N} R={R} {dtype}, {psi.nbytes} bytes, {skip} into the buffer")
        buf = torch.zeros(psi.nbytes + 64, dtype=torch.uint8, device="cuda")
        at = C.c_void_p(buf.data_ptr() + skip)
        assert plan.lib.ctqw_get_state(plan.h, at, 1) == 0
        got = buf.cpu().numpy()
        assert not got[:skip].any() and not got[skip + psi.nbytes:].any()
        assert np.array_equal(got[skip:skip + psi.nbytes].view(psi.dtype), psi)
        plan.propagate(1)
        assert plan.lib.ctqw_set_state(plan.h, at, 1) == 0
        assert np.array_equal(plan.state_numpy(), psi)
