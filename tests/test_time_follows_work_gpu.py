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


def _plan_partial(lens, S=16):
    """us of the partial pass's planning: 85% live, one request in two in permuted order."""
    t, B = torch(), _B()
    rng = np.random.default_rng(len(lens))
    blocks = -(-np.asarray(lens) // S)
    M = int(blocks.sum())
    perm = rng.permutation(M + 4000)
    at = np.concatenate([[0], np.cumsum(blocks)])
    slots = []
    for r, n in enumerate(lens):
        s = perm[at[r] + np.arange(n) // S] * S + np.arange(n) % S
        slots.append(rng.permutation(s) if r % 2 else s)
    T = int(np.sum(lens))
    kv = t.zeros((2, perm.size, S, 1, 8), dtype=t.float16, device="cuda")
    live = t.from_numpy((rng.random(T) < 0.85).astype(np.uint8)).cuda()
    batch = B.Batch(_i32(lens), _i32(np.concatenate([[0], np.cumsum(lens)])), _i32(at),
                    _i32(perm[:M]), live, _i32(perm[M:]))
    cache = B.KVCache(kv, 1, 1, 8, S)
    plan, state = B.Plan.allocate(batch, S), B.PlannerState.allocate(perm.size, batch)
    slot_in = _i32(np.concatenate(slots))
    us = _us(lambda: B.plan_partial(cache, batch, slot_in, plan, state), 4)
    assert int(plan.counters[3]) == 0
    return us


def test_partial_planning_of_a_long_request_among_short_ones():
    """One request of 600K tokens, alone and with 511 of 100 beside it: the same planning but for
    the short ones' (left to a single workgroup it took six times as long)."""
    alone, among = _plan_partial([600000]), _plan_partial([600000] + [100] * 511)
    print(f"[gpu] plan_partial 1 x 600K: {alone:.0f} us, among 511 x 100: {among:.0f} us", flush=True)
    assert among < 2.5 * alone


def _build(R, tokens, free_blocks, S=16):
    """us of the table build of R requests of `tokens` tokens, half live."""
    t, B = torch(), _B()
    rng = np.random.default_rng(R)
    M = R * -(-tokens // S)
    perm = rng.permutation(M + free_blocks)
    kv = t.zeros((2, perm.size, S, 1, 8), dtype=t.float16, device="cuda")
    live = t.from_numpy((rng.random(R * tokens) < 0.5).astype(np.uint8)).cuda()
    batch = B.Batch(_i32(np.full(R, tokens)), _i32(np.arange(R + 1) * tokens),
                    _i32(np.arange(R + 1) * (M // R)), _i32(perm[:M]), live, _i32(perm[M:]))
    cache, plan = B.KVCache(kv, 1, 1, 8, S), B.Plan.allocate(batch, S)
    us = _us(lambda: B.build_token_table(cache, batch, plan))
    assert int(plan.counters[3]) == 0
    return us


def test_build_with_a_long_free_list():
    """A pass can use no more of the free list than the batch has table entries: three million free
    blocks cost small requests nothing (looked over to the end, twice the time)."""
    few, many = _build(257, 20, 3000), _build(257, 20, 3000000)
    print(f"[gpu] build, 3K blocks free: {few:.1f} us, 3M: {many:.1f} us", flush=True)
    assert many < 1.5 * few


def _inplace(R, layers, tokens, heads, dim, S=16):
    """us of the in-place copy of R fp8 requests of `tokens` tokens, 0.3 of them live."""
    t, B = torch(), _B()
    rng = np.random.default_rng(R)
    blocks = -(-tokens // S)
    perm = rng.permutation(R * blocks)
    kv = t.zeros((2 * layers, perm.size, S, heads, dim), dtype=t.float8_e4m3fn, device="cuda")
    live = t.from_numpy((rng.random(R * tokens) < 0.3).astype(np.uint8)).cuda()
    batch = B.Batch(_i32(np.full(R, tokens)), _i32(np.arange(R + 1) * tokens),
                    _i32(np.arange(R + 1) * blocks), _i32(perm), live, _i32([]))
    cache, plan = B.KVCache(kv, layers, heads, dim, S), B.Plan.allocate(batch, S, inplace=True)
    B.build_token_table_inplace(cache, batch, plan)
    return _us(lambda: B.repack_inplace(cache, batch, plan), 4)


def test_inplace_copy_of_rows_that_are_no_whole_lines():
    """480-byte rows: 448 (request, plane) pairs against 300, half as much again (1.2 times the time;
    with workgroups of four waves 1.56 times a larger one)."""
    few, more = _inplace(5, 30, 5000, 5, 96), _inplace(7, 32, 5000, 5, 96)
    print(f"[gpu] in place, 300 pairs: {few:.1f} us, 448: {more:.1f} us", flush=True)
    assert more < 1.4 * few
