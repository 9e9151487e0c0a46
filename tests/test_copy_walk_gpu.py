"""The walk of the out-of-place copy: workgroups that take several pieces (parts of destination
blocks, one plane each), for every piece size and for the pieces that share a workgroup."""
import numpy as np
import pytest

from paper_2608_13263_amd import workloads as W
from tests.gpu_helpers import full_parity

pytestmark = pytest.mark.gpu

# (layers, heads, dim, dtype, S): chunks of 16-byte units
GEOMETRIES = [
    (20, 1, 128, "fp8_e4m3", 8),    # 64: one wave per piece, four side by side
    (20, 1, 64, "fp16", 3),         # 24: one wave, partly idle
    (20, 2, 64, "fp16", 8),         # 128: two waves, two side by side
    (20, 5, 96, "fp8_e4m3", 4),     # 120: two waves, the last lanes idle
    (20, 1, 8, "fp16", 70),         # 70, one-unit rows, plan read from memory
    (20, 1, 128, "fp8_e4m3", 32),   # 256: the whole workgroup, one unit each
    (20, 1, 128, "fp16", 24),       # 384: two parts, the second half empty
    (20, 5, 96, "fp8_e4m3", 24),    # 720: two units each, two parts
    (20, 8, 128, "fp8_e4m3", 16),   # 1,024: four units each
    (4, 8, 128, "bf16", 24),        # 3,072: eight units each, two parts
    (4, 8, 128, "bf16", 72),        # 9,216: five parts, plan read from memory
]


def _inputs(layers, heads, dim, dtype, S, reqs, free_blocks, seed):
    rng = np.random.default_rng(seed)
    masks = [(rng.random(int(n)) < 0.4).astype(np.uint8) for n in rng.integers(1, 24 * S, reqs)]
    return W.from_masks(masks, W.KVShape(layers, heads, dim, S, dtype), free_blocks=free_blocks,
                        seed=seed)


@pytest.mark.parametrize("grid,order", [(1, 0), (5, 1), (333, 2), (1 << 15, 1)])
@pytest.mark.parametrize("geometry", GEOMETRIES, ids=str)
def test_walk_of_given_grids(geometry, grid, order):
    """Grids far below, below and above the number of items, both work orders; one workgroup
    walks every piece."""
    reqs = 3 if grid == 1 else 12
    full_parity(_inputs(*geometry, reqs, 200, 7), seed=4, grid=grid, order=order)


@pytest.mark.parametrize("fused", [False, True], ids=["three_calls", "repack_free"])
@pytest.mark.parametrize("room", [20, 210, 4000], ids=["every_item", "walk", "mostly_empty"])
@pytest.mark.parametrize("geometry", GEOMETRIES, ids=str)
def test_walk_of_default_grids(geometry, room, fused):
    """The default grid with a workgroup for every item the buffers hold (no walk), with fewer
    (8,400 items and more of 40 planes), and with most of the room unused; requests past the
    supply are deferred."""
    reqs = 4 if room == 20 else 40
    inp = _inputs(*geometry, reqs, room, 11)
    gpu, orc = full_parity(inp, seed=5, fused=fused)
    assert 0 < orc.used <= room
