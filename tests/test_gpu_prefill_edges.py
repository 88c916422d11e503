"""Chunked prefill at the edges of its tiles, units, ring and metadata windows,
against the float64 oracle (tolerance as in the other prefill tests)."""

import numpy as np
import pytest

from paper_2609_33536_amd import workloads
from tests import softmax_rises, test_gpu_fp8, test_gpu_prefill

pytestmark = pytest.mark.gpu


def _run(case, hq, hkv, **kw):
    if case["dtype"] == "e5m2":
        test_gpu_fp8._run_prefill(case, hq, hkv, **kw)
    else:
        test_gpu_prefill._run_prefill(case, hq, hkv, **kw)


def _routed(prefix, chunk, group, hkv, split, monkeypatch):
    """The sequences in batches as each kernel gets them: for the unit-dividing
    one, as many as keep its 32-column workgroups within 256; for the other, all
    of them and one-token prompts until there are more than 512.  The kernel is
    forced, so that a change of the rule does not change what is tested."""
    monkeypatch.setenv("EKV_PREFILL_SPLIT", "1" if split else "0")
    tiles = -(-max(chunk) * group // 32)
    if split:
        per = max(1, 256 // (tiles * hkv))
        return [(prefix[i:i + per], chunk[i:i + per]) for i in range(0, len(chunk), per)]
    pad = max(0, 512 // (tiles * hkv) + 1 - len(chunk))
    return [(prefix + [0] * pad, chunk + [1] * pad)]


@pytest.mark.parametrize("split", [True, False])
@pytest.mark.parametrize("fraction", [0.0, 0.6])
@pytest.mark.parametrize("dtype", ["bf16", "fp16", "e5m2"])
@pytest.mark.parametrize("group,hkv", [(4, 8), (16, 3), (1, 2)])
def test_prefill_tile_unit_and_ring_edges(group, hkv, dtype, fraction, split, monkeypatch):
    """Chunks one row below, at and above a query tile (128 / group tokens) and
    a wave's columns; contexts of 1 .. 6 units (32 keys) and one key around a
    unit, with whole, lone and partly filled last blocks, and waves without a
    unit or with only masked ones; BASE and TARGET units mixed, or TARGET only
    (the native kernels).  8 KV heads take
    the one-XCD-per-head order of the workgroups, 3 and 2 the other."""
    tile = 128 // group
    prefix = [0, 0, 0, 1, 15, 16, 31, 32, 33, 47, 64, 96, 128, 160]
    chunk = [1, tile, tile + 1, tile - 1 or 1, 1, 16, 1, 2, 31, 1, 32, tile, 33, 1]
    for k, (p, c) in enumerate(_routed(prefix, chunk, group, hkv, split, monkeypatch)):
        case = workloads.make_prefill_case(p, c, group * hkv, hkv, dtype=dtype, seed=211 + k,
                                           base_fraction=fraction, spare_blocks=2)
        _run(case, group * hkv, hkv)


@pytest.mark.parametrize("split", [True, False])
@pytest.mark.parametrize("fraction", [0.0, 0.5])
@pytest.mark.parametrize("dtype", ["bf16", "fp16", "e5m2"])
@pytest.mark.parametrize("group,hkv", [(4, 8), (16, 2), (1, 3)])
def test_prefill_contexts_of_few_units(group, hkv, dtype, fraction, split, monkeypatch):
    """Contexts around 4 and 8 units (128 and 256 keys): the 128-column kernel
    takes up to 8 in rounds of 4 and pipelines longer ones; the tiles of one chunk
    fall on both sides, and waves have no unit."""
    monkeypatch.setenv("EKV_PREFILL_SPLIT", "1" if split else "0")
    total = [96, 127, 128, 129, 160, 161, 255, 256, 257, 288, 289, 320]
    chunk = [96, 1, 31, 129, 33, 2, 128 // group + 1, 256, 130, 32, 289, 64]
    case = workloads.make_prefill_case([t - c for t, c in zip(total, chunk)], chunk, group * hkv, hkv, dtype=dtype,
                                       seed=215, base_fraction=fraction, spare_blocks=2)
    _run(case, group * hkv, hkv)


@pytest.mark.parametrize("split", [True, False])
@pytest.mark.parametrize("dtype", ["bf16", "e5m2"])
@pytest.mark.parametrize("placement,fraction", [("random", 0.5), ("oldest", 0.5), ("random", 0.0)])
def test_prefill_metadata_window_edges(placement, fraction, dtype, split, monkeypatch):
    """Contexts that end one block before, at and after the 64-pair (2048-token)
    windows of the block table."""
    for p, c in _routed([2016, 2030, 2048, 2049, 4095], [16, 18, 1, 31, 2], 4, 2, split, monkeypatch):
        case = workloads.make_prefill_case(p, c, 8, 2, dtype=dtype, seed=212, base_fraction=fraction,
                                           placement=placement, spare_blocks=2)
        _run(case, 8, 2)
        _run(case, 8, 2, use_boundaries=False)


@pytest.mark.parametrize("name", ["aligned-bf16", "scale1-bf16-g16", "aligned-e5m2"])
def test_prefill_rescale_in_a_full_launch(name, monkeypatch):
    """The rescaling inputs among enough one-token prompts that the 128-column
    kernel runs them (alone they take the unit-dividing one)."""
    monkeypatch.setenv("EKV_PREFILL_SPLIT", "0")
    case, hq, hkv, scale, dtype = softmax_rises.make(name)
    group, rows = hq // hkv, len(case["q"])
    n = 512 // (-(-int(np.diff(case["cu_q"]).max()) * group // 32) * hkv) + 1
    pad = workloads.make_prefill_case([0] * n, [1] * n, hq, hkv, dtype=dtype, seed=213)
    nb, mb = case["pool"].shape[0], case["block_table"].shape[1]
    bt = np.zeros((n, mb), dtype=np.int32)
    bt[:, :2] = pad["block_table"][:, :2] + nb
    both = dict(case)
    for k in ("pool", "q", "k_new", "v_new", "seq_lens"):
        both[k] = np.concatenate([case[k], pad[k]])
    both["block_table"] = np.concatenate([case["block_table"], bt])
    both["tags"] = np.zeros_like(both["block_table"], dtype=np.uint8)
    both["slots"] = np.concatenate([case["slots"], pad["slots"] + nb * 16]).astype(np.int32)
    both["cu_q"] = np.concatenate([case["cu_q"], rows + pad["cu_q"][1:]]).astype(np.int32)
    _run(both, hq, hkv, out_fp32=True, scale=scale)


@pytest.mark.parametrize("longest", [1010, 1040])
@pytest.mark.parametrize("dtype", ["bf16", "e5m2"])
def test_prefill_one_column_tile_over_many_sequences(dtype, longest):
    """More than 512 workgroups of a few rows each: with a context of 1024 keys
    or more they take the unit-dividing kernel, below it the other."""
    prefix = [longest - 8] + [(7 * s) % 90 for s in range(65)]
    chunk = [8] + [1 + s % 8 for s in range(65)]
    case = workloads.make_prefill_case(prefix, chunk, 32, 8, dtype=dtype, seed=214, base_fraction=0.5, spare_blocks=2)
    _run(case, 32, 8)
