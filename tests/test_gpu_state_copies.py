"""ctqw_set_state / ctqw_get_state on device buffers that end before the state:
refused before anything is written, whatever the alignment; the state and a
whole buffer's copies are untouched by the refusal."""

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
