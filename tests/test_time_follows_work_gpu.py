"""Calls whose time has to follow the work in them, whatever the shape of the batch: each is set
against a call of about the same work on the other side of a dispatch rule. The margins are wide
(a call may take two to three times its counterpart): they hold for rules that leave the chip to
one workgroup, not for a few per cent."""
import numpy as np
import pytest

from gpu_helpers import torch

pytestmark = pytest.mark.gpu


def _B():
    from paper_2608_13263_amd import binding as B
    return B


def _i32(x):
    return torch().from_numpy(np.ascontiguousarray(x, dtype=np.int32)).cuda()


def _us(fn, calls=8):
    """GPU time of a call in us: the best of five replays of a graph of `calls` calls."""
    t = torch()
    fn()
    t.cuda.synchronize()
    g = t.cuda.CUDAGraph()
    with t.cuda.graph(g):
        for _ in range(calls):
            fn()
    e0, e1 = (t.cuda.Event(enable_timing=True) for _ in range(2))
    best = float("inf")
    for _ in range(6):   # the first one warms up
        e0.record()
        g.replay()
        e1.record()
        t.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) * 1e3 / calls)
    return best


def _append(R, n):
    B = _B()
    start, indptr = _i32(np.arange(R + 1) * (n + 8)), _i32(np.arange(R + 1) * n)
    count, slots, add = _i32(np.zeros(R)), _i32(np.zeros(R * (n + 8))), _i32(np.arange(R * n))
    status = _i32([0])

    def call():
        count.zero_()
        B.append_slots(start, count, slots, indptr, add, status=status)
    us = _us(call)
    assert int(status) == 0 and int(count.sum()) == R * n
    return us


@pytest.mark.parametrize("R", [8, 32, 128])
def test_append_of_many_slots(R):
    """4,096 new slots for each of at most 128 requests, against 129 of them."""
    few, many = _append(R, 4096), _append(129, 4096)
    print(f"[gpu] append {R} x 4096: {few:.1f} us, 129 x 4096: {many:.1f} us", flush=True)
    assert few < 3 * many
