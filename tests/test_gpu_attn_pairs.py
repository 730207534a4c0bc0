"""GPU parity of the matrix-core attention kernel around its pairs of 16-token tiles: cache lengths on both sides of a
tile and a pair, units of one pair, spans from one wavefront to more than the batch fills (with and without the hand-over
inside a workgroup), one to five row blocks, chains and trees."""
import numpy as np
import pytest

from paper_2604_09562_amd import binding, synth
from tests.test_gpu_attn import check

pytestmark = pytest.mark.gpu

LLAMA8B, FP8_70B = synth.CONFIGS[1], synth.CONFIGS[4]
LENS = np.array([1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 95, 97, 500, 2049], dtype=np.int32)


@pytest.mark.parametrize("waves", [4, 8, 32, 0])
@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("hq,depth", [(2, 8), (8, 3), (8, 7), (8, 10), (8, 15), (16, 9)])   # 1, 1, 2, 3, 4 and 5 row blocks
def test_pairs(oracle, hq, depth, kv, tree, waves):
    k = np.minimum(LENS - 1, depth).astype(np.int32)
    cfg = (LLAMA8B if kv == "bf16" else FP8_70B).scaled(batch=len(LENS), num_q_heads=hq, num_kv_heads=2)
    inp = synth.make_attention_inputs(cfg, seed=depth, kv_len=LENS, depth=k, tree=tree, nan_tail=True)
    binding.ss_set_option("attn_path", 2)
    binding.ss_set_option("attn_waves", waves)
    try:
        check(inp, oracle, label=f"{kv} {hq} heads depth {depth} tree {tree} waves {waves}")
    finally:
        binding.ss_set_option("attn_path", 0)
        binding.ss_set_option("attn_waves", 0)
