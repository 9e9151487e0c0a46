"""GPU parity of the in-place copy's row walk where its groups, staged move lists and column
slices end: plan and every KV byte against the oracle, exactly."""
import numpy as np
import pytest

from gpu_helpers import full_parity, gpu_pass, plan_to_host, torch
from paper_2608_13263_amd import workloads as W

pytestmark = pytest.mark.gpu


def _all_move(S, n):
    return [0] * S + [1] * n   # a block shorter: admitted, and each of the n rows moves


# (heads, dim, dtype, layers): 16-byte rows; 48; 80; 128; 256; 960 (no whole lines); 1 KiB; 4 KiB
ROWS = [(1, 8, "fp16", 1), (3, 8, "fp16", 2), (5, 8, "bf16", 1), (2, 64, "fp8_e4m3", 1),
        (1, 128, "bf16", 2), (5, 96, "bf16", 1), (4, 128, "bf16", 1), (16, 128, "fp16", 1)]


@pytest.mark.parametrize("heads,dim,dtype,layers", ROWS)
def test_group_and_list_edges(heads, dim, dtype, layers):
    """Chains of k groups of moves and one more or less (groups are 8 instructions of 1 to 64
    rows: 8 to 512), of one staged list (1,024 or 2,048 rows) and one more or less, and lists
    without a move in the middle of a chain."""
    S = 16
    shape = W.KVShape(layers, heads, dim, S, dtype)
    counts = [1, 7, 8, 9, 31, 32, 33, 63, 64, 65, 128, 129, 511, 512, 513, 1023, 1024, 1025,
              2047, 2048, 2049]
    masks = [_all_move(S, n) for n in counts]
    masks.append([1] * 3000 + [0] * S + [1] * 100)                 # lists that move nothing
    masks.append([1] * 2048 + [0] * (S + 1) + [1] * 2047)
    masks.append([1] * 50)                                         # not admitted
    full_parity(W.from_masks(masks, shape, free_blocks=0, seed=heads), seed=dim, inplace=True)


@pytest.mark.parametrize("S", [8, 24, 64, 96])
@pytest.mark.parametrize("reqs", [2, 40])
def test_few_and_many_chains(S, reqs):
    """Either side of the switch from one-wave to four-wave workgroups (1,024 chains: 2 requests
    x 8 planes x 4 slices, 40 x 8 x 4), block sizes above a wave too."""
    rng = np.random.default_rng(S * 100 + reqs)
    shape = W.KVShape(4, 2, 128, S, "bf16")
    masks = [list((rng.random(int(n)) < 0.5).astype(int)) for n in rng.integers(1, 900, reqs)]
    full_parity(W.from_masks(masks, shape, free_blocks=3, seed=S), seed=reqs, inplace=True)


@pytest.mark.parametrize("reqs", [1, 30, 600])
def test_freed_list_in_the_copy_launch(reqs):
    """repack_inplace_free against the copy and free_blocks in two calls: the plan, the freed list
    and every KV byte, with a batch that releases nothing and one that admits nothing too."""
    t = torch()
    from paper_2608_13263_amd import binding as B
    rng = np.random.default_rng(reqs)
    shape = W.KVShape(2, 2, 64, 16, "bf16")
    masks = [list((rng.random(int(n)) < 0.5).astype(int)) for n in rng.integers(1, 300, reqs)]
    for m in (masks, [[1] * len(x) for x in masks], [[0] * len(x) for x in masks]):
        inp = W.from_masks(m, shape, free_blocks=0, seed=reqs)
        kv = W.kv_device(shape, inp.num_blocks, 5)
        kv2 = kv.clone()
        want = gpu_pass(inp, kv, inplace=True)
        batch = B.Batch.from_inputs(inp)
        plan = B.run_pass(B.KVCache(kv2, 2, 2, 64, 16), batch, inplace=True)
        t.cuda.synchronize()
        got = plan_to_host(plan, inp)
        for k in want:
            assert np.array_equal(got[k], want[k]), k
        assert t.equal(kv.view(t.uint8), kv2.view(t.uint8))


# (dtype, layers, heads, dim, S, requests, tokens): what each launch takes stands beside it
LAUNCHES = [
    ("bf16", 32, 2, 64, 48, 7, 3000),       # 896 chains: one wave a workgroup
    ("bf16", 32, 2, 64, 48, 8, 3000),       # 1,024, two slices a row: still
    ("bf16", 32, 2, 64, 48, 31, 900),       # 3,968, short requests
    ("bf16", 32, 2, 64, 48, 32, 1000),      # 4,096: four waves, plain stores (524 MB)
    ("bf16", 32, 2, 64, 48, 10, 7000),      # 1,280 chains of 1.1 GB: one wave, non-temporal
    ("fp8", 16, 8, 128, 16, 8, 2000),       # 2,048 chains, eight slices: four waves, plain
    ("fp8", 32, 4, 128, 16, 8, 300),        # below 96 MiB: non-temporal
    ("bf16", 32, 8, 128, 16, 4, 2100),      # 1.1 GB: non-temporal
    ("bf16", 32, 8, 128, 16, 20, 300),      # 20,480 chains: non-temporal
    ("bf16", 12, 5, 96, 16, 6, 800),        # 144 pairs of 960-byte rows: two slices
    ("bf16", 20, 5, 96, 16, 4, 900),        # 160: one, groups of 16, short requests
    ("bf16", 20, 5, 96, 24, 4, 5000),       # long ones
    ("fp8", 32, 5, 96, 8, 1, 2500),         # 64 pairs of 480-byte rows: four slices
    ("fp8", 32, 5, 96, 16, 7, 3000),        # 448: one
    ("fp8", 80, 5, 96, 16, 30, 400),        # 4,800: four waves, plain
    ("bf16", 1, 3, 8, 16, 9, 2000),         # 48-byte rows
]


@pytest.mark.parametrize("dtype,layers,heads,dim,S,reqs,tokens", LAUNCHES)
def test_every_launch_of_the_row_walk(dtype, layers, heads, dim, S, reqs, tokens):
    """Workgroups of one wave and of four, both kinds of stores, both lengths of the staged list and
    of a group, against the block-staging copy (variant 3) on the same cache: every byte."""
    t = torch()
    from paper_2608_13263_amd import binding as B
    rng = np.random.default_rng(layers * reqs)
    lens = rng.integers(tokens * 3 // 4, tokens * 5 // 4, reqs)
    masks = [(rng.random(int(n)) < 0.4).astype(np.uint8) for n in lens]
    shape = W.KVShape(layers, heads, dim, S, {"fp8": "fp8_e4m3"}.get(dtype, dtype))
    inp = W.from_masks(masks, shape, free_blocks=2, seed=reqs)
    kv = t.randint(0, 256, (2 * layers, inp.num_blocks, S, shape.row_bytes), dtype=t.uint8,
                   device="cuda")
    typed = [x.view(t.uint8 if dtype == "fp8" else t.bfloat16)
             .view(2 * layers, inp.num_blocks, S, heads, dim) for x in (kv, kv.clone())]
    batch = B.Batch.from_inputs(inp)
    for x, variant in zip(typed, (0, 3)):
        cache = B.KVCache(x, layers, heads, dim, S)
        plan = B.Plan.allocate(batch, S, inplace=True)
        B.build_token_table_inplace(cache, batch, plan)
        B.repack_inplace_ex(cache, batch, plan, variant=variant)
        assert int(plan.counters[3]) == 0 and int(plan.counters[1]) > 0
    assert t.equal(typed[0].view(t.uint8), typed[1].view(t.uint8))
