"""Decode with workspaces smaller than the reported size (down to one workgroup
per 8 pairs of blocks), each followed by canary bytes, and the no-allocation
decode where the finest ranges would need more than its 32 MiB of scratch;
against the float64 oracle."""

import numpy as np
import pytest

from oracle import attention as oatt
from oracle import fp8 as ofp8
from oracle import transitions as otr
from paper_2609_33536_amd import ekv, kvpool, workloads
from tests.gpu_util import check_attention, default_scale, require_gpu, words_to_tensor

pytestmark = pytest.mark.gpu
CANARY = 4096


def _prepared(lens, hq, hkv, dtype, seed):
    torch = require_gpu()
    c = workloads.make_decode_case(lens, hq, hkv, seed=seed, base_fraction=0.5, spare_blocks=2, dtype=dtype)
    kv = kvpool.PagedKV(c["pool"], c["block_table"], c["seq_lens"], c["free"], hkv, dtype)
    kv.demote(c["pairs"])
    kv.relower()
    ref = ofp8 if dtype == "e5m2" else otr
    pool, bt, tags, _, _ = ref.demote(c["pool"], c["block_table"], c["tags"], c["pairs"], c["seq_lens"])
    want = (ofp8 if dtype == "e5m2" else oatt).decode(c["q"], pool, bt, tags, c["seq_lens"])
    return kv, words_to_tensor(c["q"], torch, workloads.query_dtype(dtype)), want


def _bytes(grid, group):
    ml = 2 * grid * group * 8
    return 32768 + -(-ml // 256) * 256 + 2 * grid * group * 512


@pytest.mark.parametrize("dtype", ["bf16", "e5m2"])
@pytest.mark.parametrize("group,lens", [(4, [64, 128, 192, 256]), (1, [4096]), (16, [1000, 333, 17]),
                                        (8, [2049, 1, 700, 512, 96])])
def test_decode_with_smaller_workspaces(group, lens, dtype):
    torch = require_gpu()
    hkv = 2
    kv, q, want = _prepared(lens, group * hkv, hkv, dtype, 400 + group)
    batch = kv.batch(group * hkv)
    pairs = len(lens) * hkv * -(-(-(-max(lens) // 16)) // 2)
    least, need = _bytes(max(1, -(-pairs // 8)), group), ekv.decode_workspace_bytes(kv.pool, batch)
    assert need == _bytes(pairs, group)
    out = torch.empty(q.shape, dtype=torch.float32, device="cuda")
    with pytest.raises(ekv.EkvError, match="workspace"):
        ekv.attn_decode(kv.pool, batch, q, out, default_scale(), torch.zeros(least - 1, dtype=torch.uint8, device="cuda"))
    for size in sorted({least, least + 8, (least + need) // 2 + 3, need}):
        memory = torch.zeros(size + CANARY, dtype=torch.uint8, device="cuda")
        memory[size:] = 0xA5
        print(f"decode: group {group} {dtype} workspace {size} of {need}", flush=True)
        for _ in range(2):                                   # the counters are left at zero
            out.fill_(float("nan"))
            ekv.attn_decode(kv.pool, batch, q, out, default_scale(), memory[:size])
            torch.cuda.synchronize()
            check_attention(out.cpu().numpy(), want, True)
        assert bool((memory[size:] == 0xA5).all())


def test_noalloc_decode_of_many_short_sequences_of_wide_groups():
    """128 / 8 heads over an 8-bit pool: one-pair ranges would take 2048
    workgroups (34 MB of partial rows); the scratch holds fewer."""
    torch = require_gpu()
    rng = np.random.default_rng(410)
    kv, q, want = _prepared([1024] + rng.integers(1, 1025, size=39).tolist(), 128, 8, "e5m2", 411)
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
    print("noalloc decode: 40 sequences, 128 / 8 heads, e5m2", flush=True)
    ekv.attn_decode_noalloc(kv.pool, kv.batch(128), q, out, default_scale())
    torch.cuda.synchronize()
    check_attention(out.cpu().numpy(), want, True)
