"""Autotuning a batch whose runs go on chip: no launch shape has a say there, so
none is timed; the plan keeps its shape, and the time returned is that of a step
of a run, which is what propagate takes."""

import numpy as np
import pytest

from _helpers import gpu_plan, say

pytestmark = pytest.mark.gpu


def test_no_shapes_are_compared(tmp_path, monkeypatch):
    trace, cache = tmp_path / "trace.jsonl", tmp_path / "cache.jsonl"
    monkeypatch.setenv("CTQW_TUNE_TRACE", str(trace))
    reals = [(64, np.ones(63), np.zeros(64), 1.0)] * 300

    def plan(**kw):
        return gpu_plan(m=2, statistics="boson", boundary="open", interaction="onsite", dtype="c64", reals=reals, dt=0.05,
                        order=7, sites=[30, 31], **kw)
    p = plan(launch={"waves_per_block": 2})
    was = p.get_launch()
    best, ms = p.autotune(str(cache), steps=20)
    now = p.get_launch()
    assert all(getattr(best, f) == getattr(was, f) == getattr(now, f) for f, _ in was._fields_)
    assert not trace.exists() and cache.read_text().count("\n") == 1
    p.init_product_state([30, 31])
    p.set_timing(True)
    p.propagate(20)
    total, steps = p.get_timing()
    say(f"case: autotune on chip: {ms * 1e3:.1f} us per step, a run of 20 {total / steps * 1e3:.1f}")
    assert steps == 20 and 0 < ms < 3 * total / steps
    again, ms2 = plan().autotune(str(cache), steps=20)   # from the cache
    assert again.waves_per_block == 2 and ms2 == pytest.approx(ms, rel=1e-3)
    q = plan()
    q.propagate(20)
    assert np.array_equal(p.state_numpy(), q.state_numpy())
