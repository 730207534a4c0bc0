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


# The plan record at the start of the workspace, int32: pairs, whose the spans are, spans, -, -, -, requests and pairs in front of the end of
# each of five classes, what a pair and what opening a unit costs in each.
CHAIN, TEAM, ALONE = 0, 1, 2


def plan_of(inp, max_q_len):
    d = binding.attention_to_device(inp)
    out, lse, ws = binding.alloc_attention_outputs(d, max_q_len=max_q_len)
    binding.ss_spec_verify_attn(d, out, lse, ws, max_q_len=max_q_len)
    torch.cuda.synchronize()
    rec = ws[:104].view(torch.int32).tolist()
    return dict(pairs=rec[0], mode=rec[1], spans=rec[2], cost=rec[16:21], weight=rec[21:26])


@pytest.mark.parametrize("weight", [0, 1, 4, 17, 64, 3])
@pytest.mark.parametrize("batch,hq,depth,mode", [
    (4, 8, 4, TEAM), (64, 8, 4, CHAIN),                                  # two row blocks, in pairs
    (4, 16, 9, TEAM), (260, 16, 9, ALONE)])                              # five, in eighths of a pair
def test_unit_weight_option(batch, hq, depth, mode, weight):
    """What opening a unit is charged when the spans are cut: the option's value for a wavefront (tiles, rounded up to pairs) or the
    default's, also after the option had another value."""
    cfg = LLAMA8B.scaled(batch=batch, num_q_heads=hq, num_kv_heads=2, depth=("fixed", depth))
    inp = synth.make_attention_inputs(cfg, seed=1, kv_len=np.full(batch, 900 if mode != ALONE else 200, np.int32))
    binding.ss_set_option("attn_unit_weight", 64)
    binding.ss_set_option("attn_unit_weight", weight)
    try:
        plan = plan_of(inp, depth + 1)
    finally:
        binding.ss_set_option("attn_unit_weight", 3)
    assert plan["mode"] == mode
    pairs = (weight + 1) // 2
    if hq == 8:
        assert plan["cost"][0] == 1
        assert plan["weight"][0] == (2 if weight == 3 else pairs) * (2 if mode == TEAM else 1)
    elif weight != 3:
        assert plan["weight"] == [pairs * 8 * (4 if mode == TEAM else 1)] * 5
    else:   # five row blocks ... one
        assert plan["cost"] == [9, 9, 8, 8, 8]
        assert plan["weight"] == ([128, 100, 80, 48, 32] if mode == TEAM else [68, 52, 44, 32, 24])


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


@pytest.mark.parametrize("tokens,hkv,hq,depth,spans,mode", [
    (1000, 8, 32, 4, 128, TEAM), (4000, 8, 32, 4, 256, TEAM), (8100, 8, 32, 4, 256, TEAM),   # two row blocks: teams until the chip is full,
    (8200, 8, 32, 4, 1024, CHAIN), (8200, 4, 16, 4, 64, TEAM), (32000, 1, 4, 4, 62, TEAM),  # of sixteen pairs in long units
    (2000, 8, 32, 8, 252, TEAM), (20000, 8, 32, 8, 256, TEAM), (20000, 1, 8, 8, 39, TEAM)])  # three and five row blocks
def test_single_long_requests(oracle, tokens, hkv, hq, depth, spans, mode):
    """One request: whose the spans are and how many, on both sides of the rules, and the result."""
    cfg = LLAMA8B.scaled(batch=1, num_q_heads=hq, num_kv_heads=hkv)
    inp = synth.make_attention_inputs(cfg, seed=tokens, kv_len=np.array([tokens], np.int32), depth=np.array([depth], np.int32))
    check(inp, oracle, max_q_len=depth + 1, label=f"{tokens} tokens over {hkv} KV heads")
    plan = plan_of(inp, depth + 1)
    assert (plan["spans"], plan["mode"]) == (spans, mode), plan


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("batch,hkv,hq,depth,lo,hi,spans,mode", [
    (16, 2, 8, 10, 1, 256, 32, TEAM), (16, 2, 8, 10, 1, 290, None, TEAM),        # whole units of up to eight pairs
    (128, 2, 8, 15, 1, 512, 256, TEAM), (128, 2, 8, 10, 1, 540, None, TEAM),     # of up to sixteen in half as many units as teams
    (255, 2, 16, 9, 1, 200, None, TEAM), (256, 2, 16, 9, 1, 200, None, ALONE),   # five row blocks: two units to a team
    (256, 2, 8, 10, 1, 1300, None, TEAM),                                        # (their pairs too many)
    (16, 2, 8, 4, 1, 128, 32, TEAM), (16, 2, 8, 4, 1, 160, None, TEAM),          # two row blocks: whole units of up to four pairs
    (255, 2, 8, 4, 1, 100, None, TEAM), (256, 2, 8, 4, 1, 100, None, CHAIN)])    # many units
def test_short_units(oracle, batch, hkv, hq, depth, lo, hi, spans, mode, tree, kv):
    """Requests of a few pairs, all row blocks up to the call's: a span per unit, teams and wavefronts by themselves."""
    rng = np.random.default_rng(batch + hi)
    lens = rng.integers(lo, hi + 1, batch).astype(np.int32)
    lens[0] = hi
    k = np.minimum(rng.integers(0, depth + 1, batch), lens - 1).astype(np.int32)
    k[0] = depth
    cfg = (LLAMA8B if kv == "bf16" else FP8_70B).scaled(batch=batch, num_q_heads=hq, num_kv_heads=hkv)
    inp = synth.make_attention_inputs(cfg, seed=batch, kv_len=lens, depth=k, tree=tree, nan_tail=True)
    check(inp, oracle, max_q_len=depth + 1, label=f"{batch} requests of up to {hi}")
    plan = plan_of(inp, depth + 1)
    assert plan["mode"] == (mode if kv == "bf16" or hi != 1300 else ALONE), plan
    assert plan["cost"][0] == 0 if spans else plan["cost"][0] > 0
    assert spans is None or plan["spans"] == spans


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
