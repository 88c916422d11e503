"""Chunked prefill over a pool of 12 GiB: consecutive blocks of every sequence
lie more than 4 GiB apart, so the two 32-bit halves of consecutive tile
addresses both change.  Native and mixed batches through both prefill kernels,
against the float64 oracle on a compact copy of the touched blocks."""

import numpy as np
import pytest

from oracle import attention as oatt
from oracle import fp8 as ofp8
from oracle import transitions as otr
from paper_2609_33536_amd import ekv, kvpool, workloads
from tests.gpu_util import check_attention, default_scale, require_gpu, words_to_tensor

pytestmark = pytest.mark.gpu
POOL_BYTES = 12 << 30
HKV = 8


@pytest.fixture(scope="module")
def memory():
    torch = require_gpu()
    mem = torch.zeros(POOL_BYTES, dtype=torch.uint8, device="cuda")
    yield mem
    del mem
    torch.cuda.empty_cache()


@pytest.mark.parametrize("fraction", [0.0, 0.5])
@pytest.mark.parametrize("dtype", ["bf16", "fp16", "e5m2"])
@pytest.mark.parametrize("group,prefix,chunk", [(4, [700, 333, 0], [19, 5, 40]), (1, [400, 90], [33, 64]),
                                                (8, [600, 257], [3, 9]), (16, [500, 75], [6, 2]),
                                                (4, [600] * 24, [130] * 24)])   # the last: the 128-column kernel
def test_prefill_over_a_pool_beyond_4_gib(memory, group, prefix, chunk, dtype, fraction):
    import torch
    case = workloads.make_prefill_case(prefix, chunk, HKV * group, HKV, dtype=dtype, seed=230 + group,
                                       base_fraction=fraction, spare_blocks=2)
    small = case["pool"]                                     # the oracle's pool; block b lies at place[b] on the device
    elem = 1 if dtype == "e5m2" else 2
    flat = memory if elem == 1 else memory.view(torch.int16)
    pool = flat.view(-1, *small.shape[1:])
    nb, used = pool.shape[0], small.shape[0]
    rng = np.random.default_rng(231)
    place = np.empty(used, dtype=np.int64)
    order = [b for s, n in enumerate(case["seq_lens"]) for b in case["block_table"][s, :-(-int(n) // 16)]]
    order += sorted(set(range(used)) - set(order))
    third = nb // 3
    place[order] = np.arange(used) % 3 * third + rng.permutation(third)[:used]   # neighbours 4 GiB apart
    assert len(set(place.tolist())) == used and place.max() < nb
    pool[torch.from_numpy(place).cuda()] = torch.from_numpy(small if elem == 1 else small.view(np.int16)).cuda()
    bt = place[case["block_table"]].astype(np.int32)
    kv = kvpool.PagedKV(pool, bt, case["seq_lens"], place[case["free"]], HKV, dtype)
    new = [torch.from_numpy(x).cuda() if elem == 1 else words_to_tensor(x, torch, dtype)
           for x in (case["k_new"], case["v_new"])]
    slots = case["slots"].astype(np.int64)
    kv.append(torch.from_numpy((place[slots // 16] * 16 + slots % 16).astype(np.int32)).cuda(), *new)
    ref = ofp8 if elem == 1 else otr
    opool, obt, otg = ref.append(small, case["slots"], case["k_new"], case["v_new"]), case["block_table"], case["tags"]
    if len(case["pairs"]):
        kv.demote(case["pairs"])
        opool, obt, otg, _, _ = ref.demote(opool, obt, otg, case["pairs"], case["seq_lens"])
    kv.relower()
    q = words_to_tensor(case["q"], torch, workloads.query_dtype(dtype))
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
    print(f"prefill, 12 GiB pool: group {group} {dtype} BASE {fraction} mode {kv.mode}", flush=True)
    ekv.attn_prefill(kv.pool, kv.batch(HKV * group), q, torch.from_numpy(case["cu_q"]).cuda(), max(chunk), out,
                     default_scale())
    torch.cuda.synchronize()
    args = (case["q"], case["cu_q"], opool, obt, otg, case["seq_lens"])
    want = ofp8.prefill(*args) if elem == 1 else oatt.prefill(*args, dtype)
    check_attention(out.cpu().numpy(), want, True)
