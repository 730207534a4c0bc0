"""GPU parity of the matrix-core attention kernels whose workgroups are teams: requests of one to five row blocks in one call (laid out by
class), spans that cross classes, units without a pair for some of the team's wavefronts, batches of one and of several requests to a lane of the plan and those laid out by a
kernel of their own."""
import numpy as np
import pytest
import torch

from paper_2604_09562_amd import binding, synth
from tests.test_gpu_attn import check

pytestmark = pytest.mark.gpu

LLAMA8B, FP8_70B = synth.CONFIGS[1], synth.CONFIGS[4]


def _inputs(kv, hq, hkv, lens, depth, seed, tree=False):
    cfg = (LLAMA8B if kv == "bf16" else FP8_70B).scaled(batch=len(lens), num_q_heads=hq, num_kv_heads=hkv)
    k = np.minimum(np.asarray(lens) - 1, depth).astype(np.int32)
    return synth.make_attention_inputs(cfg, seed=seed, kv_len=np.asarray(lens, np.int32), depth=k, tree=tree, nan_tail=True)


@pytest.mark.parametrize("waves", [4, 12, 64, 0])
@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("hq,top", [(4, 20), (8, 19), (16, 9)])   # two KV heads: groups of 2 (to three row blocks), 4 and 8 (to five)
def test_mixed_row_blocks(oracle, hq, top, kv, tree, waves):
    rng = np.random.default_rng(hq)
    depth = np.concatenate([rng.permutation(top + 1), rng.integers(0, top + 1, 12)])
    lens = np.maximum(depth + 1, rng.choice([1, 2, 16, 17, 33, 64, 65, 130, 700, 2049], len(depth)))
    inp = _inputs(kv, hq, 2, lens, depth, seed=waves, tree=tree)
    binding.ss_set_option("attn_path", 2)
    binding.ss_set_option("attn_waves", waves)
    try:
        check(inp, oracle, max_q_len=top + 1, label=f"{kv} {hq} heads tree {tree} waves {waves}")
    finally:
        binding.ss_set_option("attn_path", 0)
        binding.ss_set_option("attn_waves", 0)


@pytest.mark.parametrize("hq,top", [(8, 9), (4, 8), (4, 12)])    # to five, three and four row blocks
@pytest.mark.parametrize("batch", [256, 257, 600, 4096, 4097])   # the largest batch by lanes with classes, the smallest of the layout kernel
def test_large_batches(oracle, batch, hq, top):
    rng = np.random.default_rng(batch)
    depth = rng.integers(0, top + 1, batch)
    lens = np.maximum(depth + 1, rng.integers(1, 70, batch))
    check(_inputs("bf16", hq, 1, lens, depth, seed=1), oracle, max_q_len=top + 1, label=f"{batch} requests, {hq} heads")


# a request to a lane of the plan up to 64, two from 65 on, eight from 257 to 512 without classes
@pytest.mark.parametrize("batch", [1, 2, 63, 64, 65, 257, 512, 513])
@pytest.mark.parametrize("hq,top", [(4, 3), (8, 9)])     # one row block (no classes); one to five
def test_batches_of_a_lane_each(oracle, hq, top, batch):
    rng = np.random.default_rng(batch)
    depth = rng.integers(0, top + 1, batch)
    lens = np.maximum(depth + 1, rng.integers(1, 300, batch))
    check(_inputs("bf16", hq, 1, lens, depth, seed=2), oracle, max_q_len=top + 1, label=f"{batch} requests, {hq} heads")


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_repeated_calls_give_the_same_bits(kv):
    rng = np.random.default_rng(3)
    depth = rng.integers(2, 9, 40)
    inp = _inputs(kv, 64, 8, rng.integers(100, 4000, 40), depth, seed=3)
    d = binding.attention_to_device(inp)
    first = None
    for _ in range(4):
        out, lse, ws = binding.alloc_attention_outputs(d, max_q_len=9)
        binding.ss_spec_verify_attn(d, out, lse, ws, max_q_len=9)
        torch.cuda.synchronize()
        if first is None:
            first = (out, lse)
        assert torch.equal(out, first[0]) and torch.equal(lse, first[1])
