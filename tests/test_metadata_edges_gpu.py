"""GPU parity of the metadata kernels either side of their dispatch rules: slot mappings and
appends of one launch or two, the free-list check of large batches, and the partial pass's count
by request. Everything is exact."""
import numpy as np
import pytest

from gpu_helpers import torch
from paper_2608_13263_amd import workloads as W
from test_planner_gpu import partial_parity

pytestmark = pytest.mark.gpu


def _B():
    from paper_2608_13263_amd import binding as B
    return B


def _planned(masks, S=8, free=None, inplace=False):
    B = _B()
    shape = W.KVShape(1, 1, 8, S, "fp16")
    inp = W.from_masks(masks, shape, free_blocks=len(masks), seed=1)
    if free is not None:
        inp.free_list = free(inp)
    kv = W.kv_device(shape, inp.num_blocks, 1)
    batch = B.Batch.from_inputs(inp)
    plan = B.Plan.allocate(batch, S, inplace=inplace)
    cache = B.KVCache(kv, 1, 1, 8, S)
    (B.build_token_table_inplace if inplace else B.build_token_table)(cache, batch, plan)
    return inp, batch, plan


@pytest.mark.parametrize("R", [1, 63, 1024, 1025, 2048, 2049, 4096, 4097])
@pytest.mark.parametrize("reserve", [0, 3])
def test_slot_mapping_offsets(R, reserve):
    """2,048 requests is the last batch whose workgroups sum the counts before theirs."""
    t, B = torch(), _B()
    rng = np.random.default_rng(R)
    masks = [list((rng.random(int(n)) < 0.6).astype(int)) for n in rng.integers(1, 12, R)]
    masks[R // 2] = list((rng.random(9000) < 0.5).astype(int))
    inp, batch, plan = _planned(masks)
    if reserve:
        start, count, slots = B.build_slot_table(batch, plan, reserve)
    else:
        start, slots = B.build_slot_mapping(batch, plan)
    t.cuda.synchronize()
    ts, live = plan.token_slot.cpu().numpy(), plan.live_count.cpu().numpy()[:R]
    want = np.concatenate([[0], np.cumsum(live + reserve)])
    assert np.array_equal(start.cpu().numpy(), want)
    got = slots.cpu().numpy()
    if reserve:
        assert np.array_equal(count.cpu().numpy()[:R], live)
    for r in range(R):
        s = ts[inp.tok_indptr[r]:inp.tok_indptr[r + 1]]
        assert np.array_equal(got[want[r]:want[r] + live[r]], s[s >= 0]), r


@pytest.mark.parametrize("R", [1, 64, 65, 128, 129])
@pytest.mark.parametrize("full", [False, True])
def test_append_one_launch(R, full):
    """0 to 40 new slots each, in one launch or two, and one request whose region is too small
    (left alone, the status says so)."""
    t, B = torch(), _B()
    rng = np.random.default_rng(R)
    new = rng.integers(0, 41, R)
    room = new + rng.integers(0, 3, R)
    count = rng.integers(0, 20, R)
    if full:
        new[R // 2], room[R // 2] = 7, 6
    start = np.concatenate([[0], np.cumsum(count + room)])
    indptr = np.concatenate([[0], np.cumsum(new)])
    add = rng.integers(0, 1 << 30, max(int(indptr[-1]), 1))
    slots = np.arange(int(start[-1]) + 1)

    def dev(x):
        return t.from_numpy(np.asarray(x, dtype=np.int32)).cuda()
    d_count, d_slots = dev(count), dev(slots)
    status = B.append_slots(dev(start), d_count, d_slots, dev(indptr), dev(add),
                            status=dev([77]))
    t.cuda.synchronize()
    for r in range(R):
        if new[r] <= room[r]:
            at = start[r] + count[r]
            slots[at:at + new[r]] = add[indptr[r]:indptr[r + 1]]
            count[r] += new[r]
    assert int(status) == (B.STATUS_CODE["VTOKEN_ERR_CAPACITY"] if full else 0)
    assert np.array_equal(d_count.cpu().numpy(), count)
    assert np.array_equal(d_slots.cpu().numpy(), slots)


@pytest.mark.parametrize("spread", ["even", "one", "spare", "unordered"])
@pytest.mark.parametrize("total", [1, 128, 129, 256, 257, 2048, 2049, 16384, 16385])
@pytest.mark.parametrize("R", [1, 2, 3, 8, 64, 65, 128, 129])
def test_append_by_number_of_new_slots(R, total, spread):
    """One launch takes up to 16,384 new slots of one request, 2,048 of 8, 256 of 64 and 128 of
    128 (16 for each of a request's 8 to 1,024 threads): spread evenly, nearly all in one
    request, in a buffer with spare entries at its end, and ranges that are not one after another
    (a negative count, then the same slots once more). The entry without the number gives the
    same."""
    t, B = torch(), _B()
    rng = np.random.default_rng(10 * R + total)
    most = total // 2 if spread in ("spare", "unordered") else total
    new = np.full(R, most // R)
    new[:most % R] += 1
    if spread == "one":
        new[:] = 1 if most > R else 0
        new[R // 2] += most - int(new.sum())
    indptr = np.concatenate([[0], np.cumsum(new)])
    if spread == "unordered" and R > 2:
        indptr[R // 2:] -= indptr[R // 2]
    new = np.diff(indptr)
    room = np.maximum(new, 0) + rng.integers(0, 3, R)
    count = rng.integers(0, 20, R)
    if R > 2:
        room[0] = max(int(new[0]) - 1, 0)         # full (if it appends anything)
        count[1] = -1 if R > 8 else count[1]      # no count of a table: refused
    start = np.concatenate([[0], np.cumsum(np.maximum(count, 0) + room)])
    add = rng.integers(0, 1 << 30, total)
    want, after = np.arange(int(start[-1]) + 1), count.copy()
    full = False
    for r in range(R):
        if new[r] <= 0:
            continue
        if count[r] >= 0 and count[r] + new[r] <= start[r + 1] - start[r]:
            want[start[r] + count[r]:start[r] + count[r] + new[r]] = add[indptr[r]:indptr[r + 1]]
            after[r] += new[r]
        else:
            full = True

    def dev(x):
        return t.from_numpy(np.asarray(x, dtype=np.int32)).cuda()
    ip, d_add, d_start = dev(indptr), dev(add), dev(start)
    for known in (True, False):
        d_count, d_slots, status = dev(count), dev(np.arange(want.size)), dev([77])
        if known:
            B.append_slots(d_start, d_count, d_slots, ip, d_add, status=status)
        else:
            assert B.load_library().vtoken_append_slots(
                R, ip.data_ptr(), d_add.data_ptr(), d_start.data_ptr(), d_count.data_ptr(),
                d_slots.data_ptr(), status.data_ptr(), t.cuda.current_stream().cuda_stream) == 0
        t.cuda.synchronize()
        assert int(status) == (B.STATUS_CODE["VTOKEN_ERR_CAPACITY"] if full else 0)
        assert np.array_equal(d_count.cpu().numpy(), after)
        assert np.array_equal(d_slots.cpu().numpy(), want)


@pytest.mark.parametrize("R", [256, 257, 600])
@pytest.mark.parametrize("bad", [-1, 0, 1])
def test_free_list_entry_outside_the_pool(R, bad):
    """A bad entry before, at and after the last consumed one."""
    t, B = torch(), _B()
    masks = [[1, 0] * 12] * R                       # 24 tokens, 3 blocks, 12 live: 2 blocks
    used = 2 * R

    def free(inp):
        f = np.arange(used + 5, dtype=np.int32) % inp.num_blocks
        f[used - 1 + bad] = inp.num_blocks if R % 2 else -1
        return f
    _, _, plan = _planned(masks, free=free)
    t.cuda.synchronize()
    c = plan.counters.cpu().tolist()
    if bad <= 0:
        assert c[3] == B.STATUS_CODE["VTOKEN_ERR_BLOCK_RANGE"] and c[0] == 0
    else:
        assert c[3] == 0 and c[0] == used


@pytest.mark.parametrize("blocks", [54, 55])
@pytest.mark.parametrize("bad", [0, 53, 54, 55, -1, 0.5, "after", "past"])
def test_free_list_checked_by_the_count(blocks, bad):
    """Large batches look over the usable entries of the free list, from 32,768 on, a share in each
    workgroup of the count (600 requests of 54 blocks: 32,400, left to the admission; of 55: 33,000,
    55 a workgroup): a bad entry at the ends of a share, among the last consumed, after them, and
    past what a pass can use."""
    t, B = torch(), _B()
    R, S = 600, 8
    masks = [([1, 0] * (S // 2)) * blocks] * R
    used = R * -(-blocks // 2)
    at = {"after": used, "past": R * blocks, -1: used - 1, 0.5: used // 2}.get(bad, bad)

    def free(inp):
        f = np.arange(R * blocks + 40, dtype=np.int32) % inp.num_blocks
        f[at] = inp.num_blocks
        return f
    _, _, plan = _planned(masks, free=free)
    t.cuda.synchronize()
    c = plan.counters.cpu().tolist()
    if at < used:
        assert c[3] == B.STATUS_CODE["VTOKEN_ERR_BLOCK_RANGE"] and c[0] == 0
    else:
        assert c[3] == 0 and c[0] == used


@pytest.mark.parametrize("S,reqs,lens,shared", [
    (16, 100, (5200, 5400), 4),       # two tiles a request, shared blocks
    (48, 520, (1000, 1100), 0),       # one workgroup a request, S no power of two
    (64, 20, (26500, 27500), 2),      # slots past 32 in a block, several workgroups a request
    (4, 16, (32500, 33500), 2),       # tables of more entries than the bitmap holds
])
def test_partial_count_by_request(S, reqs, lens, shared):
    """At least 2^19 tokens in long requests: counted by request."""
    inp = W.token_table_inputs(631 + S, W.KVShape(1, 1, 8, S, "fp16"), num_reqs=reqs,
                               len_range=lens, shared_groups=shared, group_size=3,
                               prefix_tokens=256 if shared else 0)
    assert inp.num_tokens >= 1 << 19
    partial_parity(inp, label=f"count by request S={S}")


def _mixed(lens, S, seed):
    """Ragged batch whose every second request holds its tokens in permuted order, half live."""
    rng = np.random.default_rng(seed)
    masks = [(rng.random(n) < 0.5).astype(np.uint8) for n in lens]
    inp = W.from_masks(masks, W.KVShape(1, 1, 8, S, "fp16"), free_blocks=4000, seed=seed)
    slots = []
    for r, n in enumerate(lens):
        ids = inp.block_ids[inp.bt_indptr[r]:inp.bt_indptr[r + 1]].astype(np.int64)
        p = np.arange(n)
        s = ids[p // S] * S + p % S
        slots.append(rng.permutation(s) if r % 2 else s)
    inp.slot_in = np.concatenate(slots).astype(np.int32)
    return inp


@pytest.mark.parametrize("lens", [
    [600000] + [100] * 400,              # one long request first, in the middle, last, alone
    [100] * 200 + [600000] + [90] * 200,
    [80] * 400 + [600001],
    [530000],
    [8192] * 20 + [8193, 30000, 16385] + [5000] * 66,   # just what a request's own workgroups take
    [1] * 300 + [400000, 1, 1, 200000, 3] + [50] * 200,
    [1000] * 520 + [0] * 5 + [90000],                   # more requests than probes of one round
], ids=lambda x: f"{len(x)}x{max(x)}")
def test_partial_count_of_uneven_requests(lens):
    """At least 2^19 tokens and a mean of 1,024, in requests far longer than the mean."""
    inp = _mixed(lens, 16, len(lens))
    assert inp.num_tokens >= 1 << 19 and inp.num_tokens // inp.num_reqs >= 1024
    partial_parity(inp, label=f"uneven R={len(lens)}")


@pytest.mark.parametrize("where", ["own", "rest", "after", "none"])
@pytest.mark.parametrize("cut", [False, True])
def test_partial_count_reports_slots_outside_the_pool(where, cut):
    """A live token's slot past the pool is reported wherever the count finds it - among the tokens
    of a request's own workgroups, in the rest of a long one, past the last request's - and before
    a request's malformed range (cut: the last one ends past the tokens)."""
    t, B = torch(), _B()
    inp = _mixed([600000] + [100] * 300, 16, 5)
    T = inp.num_tokens
    tok = inp.tok_indptr.copy()
    if where == "after":
        tok[-1] -= 1   # (the last token belongs to no request)
        tok[-2] -= 1
    if cut:
        tok[-1] = T + 5
        inp.live[T - 1] = 1
    at = {"own": 3, "rest": 590000, "after": T - 1, "none": 0}[where]
    slots = inp.slot_in.copy()
    if where != "none":
        inp.live[at] = 1
        slots[at] = inp.num_blocks * 16
    cache = B.KVCache(W.kv_device(inp.shape, inp.num_blocks, 1), 1, 1, 8, 16)
    batch = B.Batch.from_inputs(inp)
    batch.tok_indptr = t.from_numpy(tok).cuda()
    plan, state = B.Plan.allocate(batch, 16), B.PlannerState.allocate(inp.num_blocks, batch)
    B.plan_partial(cache, batch, t.from_numpy(slots).cuda(), plan, state)
    t.cuda.synchronize()
    got = int(plan.counters[3])
    if where != "none":
        assert got == B.STATUS_CODE["VTOKEN_ERR_SLOT"]
    else:
        assert got == (B.STATUS_CODE["VTOKEN_ERR_TOK_LEN"] if cut else 0)
