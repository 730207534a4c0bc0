"""GPU parity of the streaming attention kernels at shapes that the kernels for short units would serve if the block table were no wider than the
longest request: the same batches with a wide table, whole-unit spans and spans of every kind, and keys turned through LDS."""
import numpy as np
import pytest
import torch

from paper_2604_09562_amd import binding, synth
from tests.helpers import STREAM_COLUMNS, unit_choice, wider
from tests.test_gpu_attn import check, run_gpu
from tests.test_gpu_attn_pairs import ALONE, CHAIN, LENS, TEAM, plan_of

pytestmark = pytest.mark.gpu

LLAMA8B, FP8_70B = synth.CONFIGS[1], synth.CONFIGS[4]


def wide_inputs(kv, hq, hkv, lens, depth, seed, tree=False):
    cfg = (LLAMA8B if kv == "bf16" else FP8_70B).scaled(batch=len(lens), num_q_heads=hq, num_kv_heads=hkv)
    k = np.minimum(np.asarray(lens) - 1, depth).astype(np.int32)
    inp = synth.make_attention_inputs(cfg, seed=seed, kv_len=np.asarray(lens, np.int32), depth=k, tree=tree, nan_tail=True)
    inp = wider(inp, STREAM_COLUMNS)
    if (int(k.max()) + 1) * (hq // hkv) <= 80:
        assert unit_choice(inp, int(k.max()) + 1) == (0, 0)
    return inp


@pytest.mark.parametrize("kv,tree", [("bf16", False), ("fp8", True)])
@pytest.mark.parametrize("batch,hkv,hq,depth,lo,hi,spans,mode", [
    (16, 2, 8, 10, 1, 256, 32, TEAM), (16, 2, 8, 10, 1, 290, None, TEAM),        # whole units of up to eight pairs
    (128, 2, 8, 15, 1, 512, 256, TEAM), (128, 2, 8, 10, 1, 540, None, TEAM),     # of up to sixteen in half as many units as teams
    (255, 2, 16, 9, 1, 200, None, TEAM), (256, 2, 16, 9, 1, 200, None, ALONE),   # five row blocks: two units to a team
    (16, 2, 8, 4, 1, 128, 32, TEAM), (16, 2, 8, 4, 1, 160, None, TEAM),          # two row blocks: whole units of up to four pairs
    (255, 2, 8, 4, 1, 100, None, TEAM), (256, 2, 8, 4, 1, 100, None, CHAIN)])    # many units
def test_short_units(oracle, batch, hkv, hq, depth, lo, hi, spans, mode, kv, tree):
    """A span per unit, teams and wavefronts by themselves, all row blocks up to the call's."""
    rng = np.random.default_rng(batch + hi)
    lens = rng.integers(lo, hi + 1, batch)
    lens[0] = hi
    k = rng.integers(0, depth + 1, batch)
    k[0] = depth
    inp = wide_inputs(kv, hq, hkv, lens, k, seed=batch, tree=tree)
    check(inp, oracle, max_q_len=depth + 1, label=f"{batch} requests of up to {hi}")
    plan = plan_of(inp, depth + 1)
    assert plan["mode"] == mode, plan
    assert plan["cost"][0] == 0 if spans else plan["cost"][0] > 0
    assert spans is None or plan["spans"] == spans


@pytest.mark.parametrize("kv,tree", [("bf16", True), ("fp8", False)])
@pytest.mark.parametrize("hq,depth", [(2, 8), (8, 3), (8, 7), (8, 10), (8, 15), (16, 9)])   # 1, 1, 2, 3, 4 and 5 row blocks
def test_pairs(oracle, hq, depth, kv, tree):
    check(wide_inputs(kv, hq, 2, LENS, depth, seed=depth, tree=tree), oracle, label=f"{kv} {hq} heads depth {depth} tree {tree}")


@pytest.mark.parametrize("tokens,hkv,hq,depth,spans,mode", [
    (1000, 8, 32, 4, 128, TEAM), (4000, 8, 32, 4, 256, TEAM), (8200, 8, 32, 4, 1024, CHAIN), (8200, 4, 16, 4, 64, TEAM),
    (2000, 8, 32, 8, 252, TEAM)])
def test_single_long_requests(oracle, tokens, hkv, hq, depth, spans, mode):
    inp = wide_inputs("bf16", hq, hkv, [tokens], depth, seed=tokens)
    check(inp, oracle, max_q_len=depth + 1, label=f"{tokens} tokens over {hkv} KV heads")
    plan = plan_of(inp, depth + 1)
    assert (plan["spans"], plan["mode"]) == (spans, mode), plan


@pytest.mark.parametrize("batch", [1, 64, 65, 257, 512])
@pytest.mark.parametrize("hq,top", [(4, 3), (8, 9)])     # one row block (no classes); one to five
def test_batches_of_a_lane_each(oracle, hq, top, batch):
    rng = np.random.default_rng(batch)
    depth = rng.integers(0, top + 1, batch)
    lens = np.maximum(depth + 1, rng.integers(1, 300, batch))
    check(wide_inputs("bf16", hq, 1, lens, depth, seed=2), oracle, max_q_len=top + 1, label=f"{batch} requests, {hq} heads")


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_edge_lengths(oracle, kv):
    lens, depth = [1, 9, 16, 17, 32, 5, 48, 255, 256, 257], [0, 8, 3, 8, 0, 4, 8, 2, 8, 7]
    check(wide_inputs(kv, 64 if kv == "fp8" else 32, 8, lens, depth, seed=3), oracle, label=f"edge lengths {kv}")


@pytest.mark.parametrize("hq,depth", [(8, 1), (4, 7), (8, 5), (4, 15), (8, 9)])   # 1 to 5 row blocks, all of them full
def test_scores_at_the_first_reference(oracle, hq, depth):
    """Scores of exactly -1e30, the reference before any score was seen, have mass until a larger score comes: none of it may stay."""
    inp = wide_inputs("bf16", hq, 1, [256], depth, seed=depth)
    inp["sm_scale"] = float.fromhex("0x1.17f5bep-1")       # times log2(e) in float32: 1e30 / 2^100
    one = synth.to_bf16_bits(np.array([2.0 ** 50, -2.0 ** 50], np.float32))
    inp["q"][:] = 0
    inp["q"][:, :, 0] = one[0]
    inp["k_cache"][:] = 0
    for pair in (0, 2):                                    # each the first of some wavefront, alone or in a team
        inp["k_cache"][inp["block_table"][0, 2 * pair:2 * pair + 2], :, :, 0] = one[1]
    check(inp, oracle, label=f"{hq} heads depth {depth}")


@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("lo,hi,mode", [(600, 1400, TEAM), (20, 300, ALONE)])
@pytest.mark.parametrize("hq,top", [(8, 10), (8, 18), (16, 9)])   # to three, five and five row blocks
def test_keys_turned_through_lds(oracle, hq, top, lo, hi, mode, tree):
    """e4m3 with two units and more to a team, a table wide enough for the keys to be turned: units of one to five row blocks in one span, so that
    both block buffers take turns as the keys' place.  The same bits as with keys read as operands, where the narrow table asks for that."""
    rng = np.random.default_rng(top + lo)
    batch = 16
    depth = rng.permutation(np.linspace(0, top, batch).round().astype(int))
    lens = np.maximum(depth + 1, rng.integers(lo, hi + 1, batch))
    cfg = FP8_70B.scaled(batch=batch, num_q_heads=hq, num_kv_heads=2)
    inp = synth.make_attention_inputs(cfg, seed=hi, kv_len=lens.astype(np.int32), depth=depth.astype(np.int32), tree=tree, nan_tail=True)
    wide = wider(inp, 600)                                 # 32 units * 600 tiles: more than 256 to each of 64 wavefronts
    binding.ss_set_option("attn_waves", 64)
    try:
        check(wide, oracle, max_q_len=top + 1, label=f"{hq} heads to depth {top}, {lo}..{hi}")
        assert plan_of(wide, top + 1)["mode"] == mode
        a, b = run_gpu(wide, top + 1), run_gpu(inp, top + 1)
    finally:
        binding.ss_set_option("attn_waves", 0)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


def test_replays_with_a_wide_table():
    """Captured calls of the streaming kernels at a size the short-unit kernels would serve replay to the eager bits."""
    inp = wide_inputs("bf16", 32, 8, [40, 300, 2000, 3900], 8, seed=3)
    d = binding.attention_to_device(inp)
    out, lse, ws = binding.alloc_attention_outputs(d, max_q_len=9)
    binding.ss_spec_verify_attn(d, out, lse, ws, max_q_len=9)
    torch.cuda.synchronize()
    want = out.clone(), lse.clone()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            binding.ss_spec_verify_attn(d, out, lse, ws, max_q_len=9)
    torch.cuda.synchronize()
    for _ in range(3):
        out.fill_(0)
        lse.fill_(0)
        ws.fill_(0xFF)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[0]) and torch.equal(lse, want[1])
