"""GPU check of the attention plan against numpy: the layout of the requests by row blocks, what lies in front of each in pairs and in
cost, and the flat list of tile addresses, for batches of one request to a lane, of several, and of those laid out by a kernel of their own."""
import numpy as np
import pytest
import torch

from paper_2604_09562_amd import binding, synth

pytestmark = pytest.mark.gpu

REQ = np.dtype({"names": ["b", "L", "q0", "q1", "n", "cls", "pre", "cpre"], "formats": ["i4"] * 7 + ["i8"],
                "offsets": [0, 4, 8, 12, 16, 20, 24, 32], "itemsize": 40})


def plan_of(inp, max_q_len):
    """(plan record as int32 words, total cost, request records, flat pair list) that a call leaves in its workspace."""
    d = binding.attention_to_device(inp)
    out, lse, ws = binding.alloc_attention_outputs(d, max_q_len=max_q_len)
    ws.fill_(0xFF)
    binding.ss_spec_verify_attn(d, out, lse, ws, max_q_len=max_q_len)
    torch.cuda.synchronize()
    raw = ws.cpu().numpy()
    plan = raw[:256].view(np.int32)
    at = 256
    req = raw[at:at + 40 * inp["batch"]].view(REQ)
    at += -(-40 * inp["batch"] // 256) * 256
    waves = torch.cuda.get_device_properties(0).multi_processor_count * 4
    at += -(-128 * (waves + 1) // 256) * 256
    pairs = raw[at:at + 8 * int(plan[0])].view(np.int32).reshape(-1, 2)
    return plan, raw[16:24].view(np.int64)[0], req, pairs


@pytest.mark.parametrize("batch", [1, 63, 64, 65, 128, 255, 256, 257, 511, 512, 513, 1024, 1025, 4097])
@pytest.mark.parametrize("hq,hkv,top", [(8, 2, 3), (8, 2, 10), (16, 2, 9)])   # one row block; one to three; one to five
def test_plan(batch, hq, hkv, top):
    rng = np.random.default_rng(batch + top)
    depth = rng.integers(0, top + 1, batch)
    depth[0] = top
    lens = np.maximum(depth + 1, rng.integers(1, 150, batch)).astype(np.int32)
    cfg = synth.CONFIGS[1].scaled(batch=batch, num_q_heads=hq, num_kv_heads=hkv)
    inp = synth.make_attention_inputs(cfg, seed=1, kv_len=lens, depth=depth.astype(np.int32))
    plan, total_cost, req, pairs = plan_of(inp, top + 1)
    G = hq // hkv
    blocks = ((depth + 1) * G + 15) // 16
    kernel = min(5, (21 * G + 15) // 16) if blocks.max() > 2 else 0    # row blocks of the kernel, 0 for those of one class
    cls = kernel - blocks if kernel else np.zeros(batch, np.int64)
    order = np.argsort(cls, kind="stable")
    n = (lens + 31) // 32
    assert np.array_equal(req["b"], order) and np.array_equal(req["cls"], cls[order]) and np.array_equal(req["n"], n[order])
    assert np.array_equal(req["L"], lens[order])
    assert np.array_equal(req["q0"], inp["q_indptr"][order]) and np.array_equal(req["q1"], inp["q_indptr"][order + 1])
    assert np.array_equal(req["pre"], np.cumsum(n[order]) - n[order])
    cost, weight = plan[16:21], plan[21:26]
    u = n[order].astype(np.int64) * cost[cls[order]] + weight[cls[order]]
    assert np.array_equal(req["cpre"], np.cumsum(u) - u) and total_cost == u.sum() * hkv and np.all(weight[cls] > 0)
    assert plan[0] == n.sum() * hkv
    assert np.array_equal(plan[6:11], [(cls <= k).sum() for k in range(5)])
    assert np.array_equal(plan[11:16], [n[cls <= k].sum() * hkv for k in range(5)])
    bt, nblk = inp["block_table"], (lens + 15) // 16
    want = []
    for b in order:
        t = 2 * np.arange(n[b])
        lo, hi = bt[b, t], bt[b, np.minimum(t + 1, nblk[b] - 1)]
        for g in range(hkv):
            want.append(np.stack([lo * hkv + g, hi * hkv + g], 1))
    assert np.array_equal(pairs, np.concatenate(want))
