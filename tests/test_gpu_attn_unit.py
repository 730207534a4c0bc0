"""GPU parity of the attention calls whose units are short (a workgroup, or several, to a unit): both sides of every rule that takes a call
there, tile, pair and step edges, shares that a request is too short for, and the same batch with a wider block table, which the streaming
kernels serve."""
import numpy as np
import pytest
import torch

from paper_2604_09562_amd import binding, synth
from tests.helpers import STREAM_COLUMNS, unit_choice, wider
from tests.test_gpu_attn import check

pytestmark = pytest.mark.gpu

LLAMA8B, FP8_70B = synth.CONFIGS[1], synth.CONFIGS[4]
EDGES = [1, 15, 16, 17, 31, 32, 33, 64, 127, 128, 129, 255, 256, 257]


def inputs(kv, hq, hkv, lens, top, seed, tree):
    lens = np.asarray(lens, dtype=np.int32)
    depth = np.minimum(np.random.default_rng(seed).integers(0, top + 1, len(lens)), lens - 1)
    depth[-1] = min(top, lens[-1] - 1)
    cfg = (LLAMA8B if kv == "bf16" else FP8_70B).scaled(batch=len(lens), num_q_heads=hq, num_kv_heads=hkv)
    return synth.make_attention_inputs(cfg, seed=seed, kv_len=lens, depth=depth.astype(np.int32), tree=tree, nan_tail=True)


# longest request, batch, KV heads (256 compute units), on both sides of where the rule (unit_rule.h) takes another number of workgroups to a
# unit, other teams or the streaming kernels; the batches' row bounds move some of the lines
SHAPES = [(700, 14, 2), (769, 14, 2), (900, 14, 2), (1025, 1, 8), (4000, 4, 8), (9000, 14, 1), (16400, 2, 8), (1280, 33, 8), (1281, 33, 8),
          (768, 40, 8), (1024, 40, 8), (1025, 40, 8), (300, 65, 8)]


@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("longest,batch,hkv,group,top", [   # 1, 2, 3, 4 and 5 row blocks at most; 3 to 5 for the large batches
    s + g for s in SHAPES for g in ((1, 15), (2, 12), (4, 10), (8, 7), (8, 9)) if s[1] <= 14 or g[0] >= 4])
def test_shapes(oracle, longest, batch, hkv, group, top, kv, tree):
    lens = (EDGES * 6)[:batch - 1] + [longest]
    inp = inputs(kv, group * hkv, hkv, lens, top, seed=longest + top, tree=tree)
    some = [b for b in range(batch) if b >= batch - 15]       # the oracle's time
    check(inp, oracle, requests=some, max_q_len=top + 1, label=f"{longest} x {batch} over {hkv}")


@pytest.mark.parametrize("kv,tree", [("bf16", False), ("fp8", True)])
@pytest.mark.parametrize("group,top", [(4, 3), (8, 9)])                  # one and five row blocks
@pytest.mark.parametrize("longest,batch,hkv,shares", [                   # (bf16, e4m3), one and five row blocks
    (384, 4, 8, (1, 1, 1, 1)), (400, 4, 8, (4, 4, 1, 1)), (512, 4, 8, (4, 4, 1, 1)), (528, 4, 8, (5, 5, 5, 5)),      # 24, 25, 32, 33 tiles
    (1024, 4, 8, (8, 8, 8, 8)), (1040, 4, 8, (5, 5, 5, 5)), (768, 8, 8, (3, 1, 1, 1)), (784, 8, 8, (4, 4, 4, 4)),    # 64, 65; 48, 49
    (1024, 12, 8, (2, 2, 1, 1)), (1056, 12, 8, (2, 0, 2, 0)), (6160, 4, 8, (8, 0, 8, 0))])
def test_lines_of_the_rule(oracle, longest, batch, hkv, shares, group, top, kv, tree):
    lens = (EDGES * 6)[:batch - 1] + [longest]
    inp = inputs(kv, group * hkv, hkv, lens, top, seed=longest + top, tree=tree)
    assert unit_choice(inp, top + 1)[0] == shares[2 * (kv == "fp8") + (group == 8)]
    check(inp, oracle, max_q_len=top + 1, label=f"{longest} x {batch} over {hkv}")


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("group,top", [(4, 4), (4, 10), (8, 9)])
@pytest.mark.parametrize("longest,batch,hkv", [(700, 14, 2), (3000, 6, 4), (1000, 40, 8), (1000, 66, 8)])
def test_against_the_streaming_kernels(longest, batch, hkv, group, top, kv):
    """Two correct results: bf16 outputs of which each is within a rounding or two of the other's, 32-bit lse."""
    lens = (EDGES * 5)[:batch - 1] + [longest]
    inp = inputs(kv, group * hkv, hkv, lens, top, seed=1, tree=False)
    got = []
    # (320 units of five row blocks are left to the streaming kernels either way)
    assert bool(unit_choice(inp, top + 1)[0]) == ((batch, group) != (40, 8)) and not unit_choice(wider(inp, STREAM_COLUMNS), top + 1)[0]
    for i in (inp, wider(inp, STREAM_COLUMNS)):
        d = binding.attention_to_device(i)
        out, lse, ws = binding.alloc_attention_outputs(d, max_q_len=top + 1)
        binding.ss_spec_verify_attn(d, out, lse, ws, max_q_len=top + 1)
        torch.cuda.synchronize()
        got.append((binding.bf16_bits_to_float(out), lse.cpu().numpy()))
    (a, la), (b, lb) = got
    # each is 2e-3 (e4m3 2.4e-3) from 64 bits in the 2-norm, so they are within 4e-3 (5e-3) of each other
    assert np.linalg.norm(a - b) <= (4e-3 if kv == "bf16" else 5e-3) * np.linalg.norm(a)
    assert np.max(np.abs(la - lb)) < 2e-5


def test_same_bits_every_time():
    inp = inputs("bf16", 32, 8, [40, 300, 2000, 3900], 8, seed=3, tree=False)
    d = binding.attention_to_device(inp)
    first = None
    for _ in range(4):
        out, lse, ws = binding.alloc_attention_outputs(d, max_q_len=9)
        ws.fill_(0xFF)
        binding.ss_spec_verify_attn(d, out, lse, ws, max_q_len=9)
        binding.ss_spec_verify_attn(d, out, lse, ws, max_q_len=9, reuse_plan=True)
        torch.cuda.synchronize()
        first = first or (out, lse)
        assert torch.equal(out, first[0]) and torch.equal(lse, first[1])


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("longest,batch,hkv", [(700, 14, 2), (4000, 4, 8), (1024, 40, 8)])   # one workgroup a unit, several and the merge, many units
def test_captured_calls_replay_exactly(longest, batch, hkv, kv):
    inp = inputs(kv, 4 * hkv, hkv, (EDGES * 6)[:batch - 1] + [longest], 8, seed=longest, tree=False)
    d = binding.attention_to_device(inp)
    out, lse, ws = binding.alloc_attention_outputs(d, max_q_len=9)
    binding.ss_spec_verify_attn(d, out, lse, ws, max_q_len=9)
    torch.cuda.synchronize()
    want = out.clone(), lse.clone()
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
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
