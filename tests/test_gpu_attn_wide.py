"""GPU parity of the streaming attention kernels with wide block tables."""
import numpy as np
import pytest

from paper_2604_09562_amd import binding, synth
from tests.helpers import wider
from tests.test_gpu_attn import check, run_gpu
from tests.test_gpu_attn_pairs import ALONE, TEAM, plan_of

pytestmark = pytest.mark.gpu

FP8_70B = synth.CONFIGS[4]


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
