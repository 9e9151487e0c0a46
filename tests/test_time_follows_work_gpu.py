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


def _decode(dtype, H, D, G, S, R, count, bounds, layers=8):
    """us a layer of R requests of `count` slots, under each bound."""
    t, B = torch(), _B()
    blocks = -(-count // S) * R
    g = t.Generator(device="cuda").manual_seed(R + D)
    kv = t.empty((2 * layers, blocks, S, H, D), dtype=t.float16, device="cuda")
    kv = kv.normal_(generator=g).to(dtype)
    cache = B.KVCache(kv, layers, H, D, S)
    per = -(-count // S) * S
    slots = _i32((np.arange(R)[:, None] * per + np.arange(count)).ravel())
    indptr = _i32(np.arange(R + 1) * count)
    q = t.empty((R, H * G, D), device="cuda").normal_(generator=g)
    out, times, first = t.empty_like(q), [], None
    for bound in bounds:
        ws = t.empty(B.decode_workspace_bytes(R, H * G, D, bound) // 4, device="cuda")

        def call():
            for layer in range(layers):
                B.paged_decode(cache, q, indptr, slots, layer, bound, out=out, workspace=ws)
        times.append(_us(call, 2) / layers)
        if first is None:
            first = out.clone()
        assert float((out - first).norm() / first.norm()) < 1.5e-5
    return times


@pytest.mark.parametrize("G", [1, 8])
def test_decode_under_a_loose_bound(G):
    """Bounds 65 times the requests' slots dispatch up to 65 times the workgroups, but the work in
    them is the same: all on one XCD it took seven times as long, in splits as long as the bound
    asks for (one workgroup a head) 2.4 times."""
    tight, loose = _decode(torch().float8_e4m3fn, 8, 128, G, 32, 8, 2000, [2000, 131072])
    print(f"[gpu] decode G={G}: {tight:.1f} us, bound 65 times as large {loose:.1f} us", flush=True)
    assert loose < 1.9 * tight
