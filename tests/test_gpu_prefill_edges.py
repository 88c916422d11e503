"""Chunked prefill at the edges of its tiles, units, ring and metadata windows,
against the float64 oracle (tolerance as in the other prefill tests)."""

import pytest

from paper_2609_33536_amd import workloads
from tests import test_gpu_fp8, test_gpu_prefill

pytestmark = pytest.mark.gpu


def _run(case, hq, hkv, **kw):
    if case["dtype"] == "e5m2":
        test_gpu_fp8._run_prefill(case, hq, hkv, **kw)
    else:
        test_gpu_prefill._run_prefill(case, hq, hkv, **kw)


@pytest.mark.parametrize("dtype", ["bf16", "fp16", "e5m2"])
@pytest.mark.parametrize("group,hkv", [(4, 8), (16, 3), (1, 2)])
def test_prefill_tile_unit_and_ring_edges(group, hkv, dtype):
    """Chunks one row below, at and above a query tile (128 / group tokens) and
    a wave's columns; contexts of 1 .. 6 units (32 keys) and one key around a
    unit, with whole, lone and partly filled last blocks; BASE and TARGET units
    mixed.  8 KV heads take the one-XCD-per-head order of the workgroups, 3 and
    2 the other."""
    tile = 128 // group
    prefix = [0, 0, 0, 1, 15, 16, 31, 32, 33, 47, 64, 96, 128, 160]
    chunk = [1, tile, tile + 1, tile - 1 or 1, 1, 16, 1, 2, 31, 1, 32, tile, 33, 1]
    c = workloads.make_prefill_case(prefix, chunk, group * hkv, hkv, dtype=dtype, seed=211, base_fraction=0.6,
                                    spare_blocks=2)
    _run(c, group * hkv, hkv)


@pytest.mark.parametrize("dtype", ["bf16", "e5m2"])
@pytest.mark.parametrize("placement", ["random", "oldest"])
def test_prefill_metadata_window_edges(placement, dtype):
    """Contexts that end one block before, at and after the 64-pair (2048-token)
    windows of the block table."""
    c = workloads.make_prefill_case([2016, 2030, 2048, 2049, 4095], [16, 18, 1, 31, 2], 8, 2, dtype=dtype, seed=212,
                                    base_fraction=0.5, placement=placement, spare_blocks=2)
    _run(c, 8, 2)
    _run(c, 8, 2, use_boundaries=False)
