"""The autotuners decide on launches and builds as a program makes them (no GPU).

A stand-in context whose whole builds, without events, take another time than
its class times add up to: classes that are fastest one by one may be slower
together (launches overlap on two streams)."""
import time

import numpy as np
import pytest

from paper_1708_00033_amd import autotune, hfx

A, B = (8192, 1, 0, -1), (32768, 0, 1, -1)


class Fake:
    """Class times by setting (class 0 is faster with A) or precision (class 4
    with FP32); whole builds 5 ms longer where the setting or precision is mixed."""

    def __init__(self, mixed_is_slow):
        self.slow = mixed_is_slow
        self.set = [A] * 21
        self.fp32 = [1] * 21
        self.mode = 0
        self.modes = []
        self.acc = np.zeros(21)
        self.n = 0

    def set_class_tuning(self, cls, *v):
        for k in range(21):
            if cls in (-1, k):
                self.set[k] = tuple(v)

    def set_class_precision(self, cls, on):
        for k in range(21):
            if cls in (-1, k):
                self.fp32[k] = int(on)

    def build_fock_dev(self, d, f, s):
        if self.mode:
            self.n += 1
            for k in range(21):
                self.acc[k] += 10.0 - 5.0 * (k == 0 and self.set[k] == A) + 2.0 * (k != 0 and self.set[k] == A) \
                    - 3.0 * (k == 4 and self.fp32[k]) + 2.0 * (k != 4 and self.fp32[k])
            return
        mixed = len(set(self.set)) > 1 or len(set(self.fp32)) > 1
        time.sleep(0.001 + 0.005 * (mixed == self.slow))

    def kernel_timing(self, on):
        self.mode = int(on)
        if on:
            self.modes.append(int(on))
            self.acc[:] = 0
            self.n = 0

    def kernel_times(self):
        return self.acc.copy(), np.full(21, self.n)


@pytest.mark.parametrize("slow", [True, False])
def test_whole_builds_decide(slow):
    ctx = Fake(slow)
    ctx.fp32 = [0] * 21
    table = autotune.autotune(ctx, 0, 0, 0, candidates=(A, B), reps=1, sync=lambda: None)
    assert ctx.modes and set(ctx.modes) == {hfx.HFX_TIME_LAUNCHES}
    want = [B if slow or k else A for k in range(21)]
    assert list(autotune.summary(table).values()) == want and ctx.set == want
    assert table[hfx.CLASS_NAMES[0]]["ms"] == (10.0 if slow else 5.0)
    assert ctx.mode == 0


@pytest.mark.parametrize("slow", [True, False])
def test_whole_builds_decide_precision(slow):
    ctx = Fake(slow)
    ctx.set = [B] * 21
    table = autotune.autotune_precision(ctx, 0, 0, 0, reps=1, sync=lambda: None)
    assert set(ctx.modes) == {hfx.HFX_TIME_LAUNCHES}
    want = [int(k == 4 and not slow) for k in range(21)]
    assert [table[n]["fp32"] for n in hfx.CLASS_NAMES] == want and ctx.fp32 == want
