"""Decode splits of several rounds: the running softmax of a wave across its rounds, the query's
three parts, the merge of many records, and the last split that takes what is left."""
import numpy as np
import pytest
import torch

from paper_2608_13263_amd import binding as B

pytestmark = pytest.mark.gpu

DTYPES = {"fp16": torch.float16, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}


def _reference(kv, q, slots, H, D):
    """float64 softmax attention of one request; kv [2][slots][H][D] on the host."""
    G = q.shape[0] // H
    k, v = (kv[i][slots].double().permute(1, 0, 2) for i in (0, 1))
    x = q.double().reshape(H, G, D) * D ** -0.5
    return (torch.softmax(x @ k.transpose(1, 2).contiguous(), -1) @ v).reshape(H * G, D)


@pytest.mark.parametrize("dtype,H,D,G,counts,bound", [
    ("bf16", 2, 128, 4, [63, 64, 65, 511, 512, 513, 1300], 0),   # rounds of 64 tokens
    ("bf16", 1, 128, 8, [1, 255, 256, 257, 129], 0),             # bound not a multiple of 2 units
    ("fp8", 1, 128, 8, [127, 128, 129, 2049, 4100], 0),
    ("fp16", 2, 256, 2, [15, 16, 17, 63, 64, 65, 700], 0),       # 16-token rounds per wave
    ("fp8", 3, 32, 1, [2047, 2048, 2049], 0),                    # heads of a split on one XCD
    ("fp16", 8, 32, 4, [1, 300, 511], 0),
    ("fp8", 2, 64, 2, [511, 512, 513, 5], 0),
    ("bf16", 1, 256, 8, [200, 128, 100], 130),                   # past max_tokens, within its units
    ("bf16", 1, 64, 1, [40000, 9], 0),                           # merge of over 64 records
    ("fp16", 1, 256, 1, [9000, 4200], 0),
    # bounds far above: splits a half, a quarter, an eighth of the host's, where there is room
    ("fp8", 8, 128, 8, [2000, 255, 257, 1], 8000),
    ("fp8", 8, 128, 8, [2000, 257, 0], 131072),
    ("bf16", 8, 128, 1, [1024, 4097, 129], 60000),
    ("fp16", 2, 256, 2, [900, 64, 65], 131072),
    ("bf16", 8, 32, 4, [1500, 513], 131072),
    ("fp8", 4, 64, 2, [1500, 4097], 30000),
    ("bf16", 8, 128, 4, [16000, 40, 700], 60000),
])
def test_decode_rounds(dtype, H, D, G, counts, bound):
    """Against float64; scores rise along every request, so that the running maximum moves in each
    round. Tolerance: the weights' two 16-bit parts, 2^-17 of a value each (random signs)."""
    print(f"[gpu] decode rounds {dtype} H={H} D={D} G={G} counts={counts}", flush=True)
    g = torch.Generator().manual_seed(D + G)
    total = sum(counts)
    kv = torch.randn(2, total, H, D, generator=g)
    kv[0] += 0.002 * torch.arange(total).reshape(-1, 1, 1) / max(1, total // 2000)
    kv = kv.to(DTYPES[dtype])
    q = torch.rand(len(counts), H * G, D, generator=g) + 0.25
    perm = torch.randperm(total, generator=g)
    pool = torch.empty_like(kv.view(torch.uint8)).view(kv.dtype)
    pool.view(torch.uint8)[:, perm] = kv.view(torch.uint8)
    cache = B.KVCache(pool.reshape(2, total, 1, H, D).cuda(), 1, H, D, 1)
    indptr = np.concatenate([[0], np.cumsum(counts)])
    out = B.paged_decode(cache, q.cuda(), torch.tensor(indptr, dtype=torch.int32).cuda(),
                         perm.to(torch.int32).cuda(), 0, bound or max(counts)).cpu().double()
    host = kv.float()
    for r, n in enumerate(counts):
        if n == 0:
            assert (out[r] == 0).all()
            continue
        ref = _reference(host, q[r], slice(int(indptr[r]), int(indptr[r]) + n), H, D)
        scale = float(ref.pow(2).mean().sqrt())
        assert float((out[r] - ref).norm() / ref.norm()) < 1.5e-5, (r, n)
        assert float((out[r] - ref).abs().max()) < 1e-4 * max(scale, 1.0), (r, n)


def test_decode_bound_in_the_middle_of_two_units():
    """16-bit caches at G = 8 promise max_tokens rounded up to two units (256 tokens at head_dim
    128): a request of 200 slots under a bound of 100 is computed, one of 257 is NaN."""
    kv = torch.randn(2, 512, 1, 1, 128, generator=torch.Generator().manual_seed(1)).bfloat16().cuda()
    cache = B.KVCache(kv, 1, 1, 128, 1)
    q = torch.randn(3, 8, 128, generator=torch.Generator().manual_seed(2)).cuda()
    indptr = torch.tensor([0, 200, 457, 457], dtype=torch.int32).cuda()
    slots = torch.arange(457, dtype=torch.int32).cuda()
    out = B.paged_decode(cache, q, indptr, slots, 0, 100)
    full = B.paged_decode(cache, q, indptr, slots, 0, 457)
    assert torch.allclose(out[0], full[0], rtol=1e-4, atol=1e-5)
    assert torch.isnan(out[1]).all() and not torch.isnan(full[1]).any()
    assert (out[2] == 0).all()


@pytest.mark.parametrize("D", [32, 128, 256])
@pytest.mark.parametrize("counts,bound", [([20, 1, 60], 60), ([700, 33, 5000], 5000)])
def test_decode_into_unaligned_buffers(D, counts, bound):
    """q, out and the workspace are aligned to a float: written by the split kernel (one split) and
    by the merge, the same values as in aligned buffers and nothing beside them."""
    g = torch.Generator().manual_seed(D)
    total = sum(counts)
    cache = B.KVCache(torch.randn(2, total, 1, 2, D, generator=g).bfloat16().cuda(), 1, 2, D, 1)
    q = torch.randn(len(counts), 8, D, generator=g).cuda()
    indptr = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32).cuda()
    slots = torch.randperm(total, generator=g).to(torch.int32).cuda()
    want = B.paged_decode(cache, q, indptr, slots, 0, bound)
    need = B.decode_workspace_bytes(len(counts), 8, D, bound) // 4
    for off in (1, 2, 3):
        def shifted(n, fill):
            return torch.full((n + 8,), fill, device="cuda")
        buf, ws, qs = shifted(q.numel(), 7.0), shifted(need, 7.0), shifted(q.numel(), 0.0)
        qs[off:off + q.numel()] = q.flatten()
        B.paged_decode(cache, qs[off:off + q.numel()].view(q.shape), indptr, slots, 0, bound,
                       out=buf[off:off + q.numel()].view(q.shape), workspace=ws[off:off + need])
        assert torch.equal(buf[off:off + q.numel()].view(q.shape), want)
        assert (buf[:off] == 7).all() and (buf[off + q.numel():] == 7).all()
        assert (ws[:off] == 7).all() and (ws[off + need:] == 7).all()
