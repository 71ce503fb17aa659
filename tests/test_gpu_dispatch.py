"""Parity at the edges of the sizes that choose a kernel: the smallest and the ragged ends of each range, against the oracle."""
import pytest

from tests.test_gpu_parity import _full_parity

pytestmark = pytest.mark.gpu


def _bf16(name, N, L=1, heads=3, d=64, B=16, K=8, kind="gaussian", **kw):
    return dict(name=name, batch=1, heads=heads, d=d, N=N, B=B, K=K, L=L, dtype="bf16", kind=kind, **kw)


@pytest.mark.parametrize("cfg", [
    # lengths that are multiples of the block and of nothing larger: one query tile in all, one tile into the second
    # workgroup, one short of it; a workgroup of the level-0 dK/dV kernel that spans two heads
    _bf16("one_tile", 16, K=4),
    _bf16("tiles_9", 144),
    _bf16("tiles_15_d128", 240, d=128, K=4),
    _bf16("tiles_169", 2704, kind="smooth"),
    _bf16("tiles_33_Le0", 528, Le=0),
    _bf16("blocks32_3", 96, B=32, K=2),
    _bf16("blocks64_5", 320, B=64, K=3),
    # more than 64 level-0 tiles per list at such a length: one wave per query tile
    _bf16("blocks32_K33", 1120, B=32, K=33),
], ids=lambda c: c["name"])
def test_lengths_that_fill_no_workgroup(cfg):
    _full_parity(cfg, 0xD15A + cfg["N"])


def _tile(name, N, B, K, L, d=64, dtype="f32", heads=2, **kw):
    return dict(name=name, batch=1, heads=heads, d=d, N=N, B=B, K=K, L=L, dtype=dtype, kind="gaussian", **kw)


@pytest.mark.parametrize("cfg", [
    # fp32 tiles: blocks of one and a quarter tile, of two, of less than one; every channel count; lists of 64 and of 65 tokens;
    # a dense level with a ragged last tile; coarse lists split over many workgroups; no coarse level in the list
    _tile("B20_d128", 800, 20, 3, 2, d=128),
    _tile("B32_d16", 2048, 32, 2, 2, d=16),
    _tile("B5_d32", 625, 5, 7, 3, d=32),
    _tile("list_64", 256, 16, 3, 1),
    _tile("list_65", 17 * 16, 16, 3, 1, heads=3),
    _tile("split_lists", 8192, 16, 8, 2, heads=1),
    _tile("B64_Le0", 4096, 64, 2, 2, Le=0),
    _tile("bf16_B8_d64", 512, 8, 4, 3, dtype="bf16"),
    _tile("bf16_B16_d32_Le0", 1024, 16, 4, 2, d=32, dtype="bf16", Le=0),
], ids=lambda c: c["name"])
def test_fp32_tiles(cfg):
    _full_parity(cfg, 0xD15B + cfg["N"])
