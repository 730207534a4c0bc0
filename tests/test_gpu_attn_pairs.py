"""GPU parity of the matrix-core attention kernel around its pairs of 16-token tiles: cache lengths on both sides of a
tile and a pair, units of one pair, spans from one wavefront to more than the batch fills (with and without the hand-over
inside a workgroup), one to five row blocks, chains and trees."""
import numpy as np
import pytest
import torch

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


@pytest.mark.parametrize("weight,pairs,pairs_deep", [(0, 0, 0), (1, 1, 1), (4, 2, 2), (17, 9, 9), (64, 32, 32), (3, 2, 8)])
def test_unit_weight_option(weight, pairs, pairs_deep):
    """The plan record (four int32 at the start of the workspace: pairs, spans, unit weight, hand-over) carries the weight the
    spans were cut with: as given, or by the row blocks for the default, also after the option had another value."""
    for hq, depth, want in ((8, 4, pairs), (16, 9, pairs_deep)):
        cfg = LLAMA8B.scaled(batch=4, num_q_heads=hq, num_kv_heads=2, depth=("fixed", depth))
        d = binding.attention_to_device(synth.make_attention_inputs(cfg, seed=1, kv_len=np.full(4, 900, np.int32)))
        out, lse, ws = binding.alloc_attention_outputs(d, max_q_len=depth + 1)
        binding.ss_set_option("attn_unit_weight", 64)
        binding.ss_set_option("attn_unit_weight", weight)
        try:
            binding.ss_spec_verify_attn(d, out, lse, ws, max_q_len=depth + 1)
        finally:
            binding.ss_set_option("attn_unit_weight", 3)
        torch.cuda.synchronize()
        assert ws[:16].view(torch.int32)[2].item() == want, (hq, weight)


@pytest.mark.parametrize("weight", [0, 3, 16, 64])
@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("hq,depth", [(8, 15), (16, 9)])   # 4 and 5 row blocks
def test_many_short_units_over_weights(oracle, hq, depth, kv, tree, weight):
    """Many short units and a few long ones: with the larger weights most spans are empty or hold several whole units."""
    lens = np.array([40] * 30 + [1500, 21, 3000, 33], dtype=np.int32)
    cfg = (LLAMA8B if kv == "bf16" else FP8_70B).scaled(batch=len(lens), num_q_heads=hq, num_kv_heads=2)
    inp = synth.make_attention_inputs(cfg, seed=weight, kv_len=lens, depth=np.minimum(lens - 1, depth).astype(np.int32), tree=tree,
                                      nan_tail=True)
    binding.ss_set_option("attn_path", 2)
    binding.ss_set_option("attn_unit_weight", weight)
    try:
        for waves in (8, 64, 0):
            binding.ss_set_option("attn_waves", waves)
            check(inp, oracle, label=f"{kv} {hq} heads depth {depth} tree {tree} weight {weight} waves {waves}")
    finally:
        binding.ss_set_option("attn_path", 0)
        binding.ss_set_option("attn_unit_weight", 3)
        binding.ss_set_option("attn_waves", 0)


@pytest.mark.parametrize("tokens,hkv,hq,depth,spans,chain", [
    (1000, 8, 32, 4, 128, 0), (1100, 8, 32, 4, 140, 1), (4000, 8, 32, 4, 500, 1),      # two row blocks: the hand-over comes in
    (8200, 8, 32, 4, 1024, 1), (8100, 4, 16, 4, 508, 1),                               # (a full chip)
    (8200, 4, 16, 4, 257, 1), (32000, 1, 4, 4, 250, 1),                                # then spans of four pairs
    (2000, 8, 32, 8, 252, 0), (2200, 8, 32, 8, 138, 0), (20000, 1, 8, 8, 156, 0)])     # three and five row blocks
def test_single_long_requests(oracle, tokens, hkv, hq, depth, spans, chain):
    """One request: the plan record (pairs, spans, unit weight, hand-over) on both sides of its rules, and the result."""
    cfg = LLAMA8B.scaled(batch=1, num_q_heads=hq, num_kv_heads=hkv)
    inp = synth.make_attention_inputs(cfg, seed=tokens, kv_len=np.array([tokens], np.int32), depth=np.array([depth], np.int32))
    check(inp, oracle, max_q_len=depth + 1, label=f"{tokens} tokens over {hkv} KV heads")
    d = binding.attention_to_device(inp)
    out, lse, ws = binding.alloc_attention_outputs(d, max_q_len=depth + 1)
    binding.ss_spec_verify_attn(d, out, lse, ws, max_q_len=depth + 1)
    torch.cuda.synchronize()
    plan = ws[:16].view(torch.int32).tolist()
    assert (plan[1], plan[3]) == (spans, chain), plan


@pytest.mark.parametrize("waves", [4, 0])
@pytest.mark.parametrize("hq,depth", [(8, 1), (4, 7), (8, 5), (4, 15), (8, 9)])   # 1 to 5 row blocks, all of them full
def test_scores_at_the_first_reference(oracle, hq, depth, waves):
    """Scores of exactly -1e30, the reference before any score was seen, have mass until a larger score comes: none of it may stay."""
    cfg = LLAMA8B.scaled(batch=1, num_q_heads=hq, num_kv_heads=1)
    inp = synth.make_attention_inputs(cfg, seed=depth, kv_len=np.array([256], np.int32), depth=np.array([depth], np.int32))
    inp["sm_scale"] = float.fromhex("0x1.17f5bep-1")       # times log2(e) in float32: 1e30 / 2^100
    one = synth.to_bf16_bits(np.array([2.0 ** 50, -2.0 ** 50], np.float32))
    inp["q"][:] = 0
    inp["q"][:, :, 0] = one[0]
    inp["k_cache"][:] = 0
    for pair in (0, 2):                                    # each the first of some wavefront, alone or in a team
        inp["k_cache"][inp["block_table"][0, 2 * pair:2 * pair + 2], :, :, 0] = one[1]
    binding.ss_set_option("attn_path", 2)
    binding.ss_set_option("attn_waves", waves)
    try:
        check(inp, oracle, label=f"{hq} heads depth {depth} waves {waves}")
    finally:
        binding.ss_set_option("attn_path", 0)
        binding.ss_set_option("attn_waves", 0)
