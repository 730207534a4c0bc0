"""GPU parity of the fp64 acceptance passes where their block arithmetic can go wrong: masked logits (exponentials that
are zero or subnormal), vocabularies around one block per lane of the draw, several blocks per workgroup of the tree walk.
Tokens, lengths and paths equal the oracle's (a draft on a near-tie of the ratio test is excused as in the other tests)."""
import numpy as np
import pytest

from paper_2604_09562_amd import synth
from tests.test_gpu_accept import compare as compare_chain
from tests.test_gpu_tree_sample import compare as compare_tree

pytestmark = pytest.mark.gpu

TINY, LLAMA8B = synth.CONFIGS[:2]


def make(tree, cfg, seed, pad=0):
    return (synth.make_tree_sample_inputs if tree else synth.make_accept_inputs)(cfg, seed=seed, row_pad=pad)


def check(tree, inp, oracle, label):
    (compare_tree if tree else compare_chain)(inp, oracle, label=label)


@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("low", [-np.inf, -715.0, -740.0])
def test_masked_logits(oracle, tree, dtype, low):
    """A third of the vocabulary at -inf, or so low that its exponentials are subnormal, in target and draft rows."""
    cfg = TINY.scaled(batch=8, vocab=9001, logit_dtype=dtype, depth=("uniform", 0, 6), sigma_draft=("fixed", 0.7))
    inp = make(tree, cfg, 3, pad=(-9001) % 8)
    rng = np.random.default_rng(1)
    masked = rng.random(9001) < 1.0 / 3.0
    masked[inp["draft_tokens"]] = False
    masked[:40] = inp["draft_tokens"].min() >= 40   # u_sample = 0 below: the first token with mass comes after a masked run
    for name in ("target_logits", "draft_logits"):
        rows = inp[name][:, :9001]
        rows[:, masked] = synth.store(np.array([low], np.float32), dtype)[0]
    inp["u_sample"][:2] = 0.0
    check(tree, inp, oracle, f"masked at {low}, {dtype}")


@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("vocab", [524288, 524296, 1050000])   # 256, 257 and 513 blocks: one, two and three per lane
def test_more_blocks_than_lanes(oracle, tree, vocab):
    cfg = LLAMA8B.scaled(batch=3, vocab=vocab, depth=("fixed", 2))
    inp = make(tree, cfg, 5)
    inp["u_sample"][:] = np.array([0.02, 0.5, 0.999999], np.float32)
    check(tree, inp, oracle, f"vocab {vocab}")


@pytest.mark.parametrize("batch,vocab", [(300, 9000), (1100, 18000)])   # 2 and 8 (the most) blocks per workgroup, ragged ends
def test_tree_blocks_per_workgroup(oracle, batch, vocab):
    cfg = TINY.scaled(batch=batch, vocab=vocab, logit_dtype="bf16", depth=("uniform", 0, 3), sigma_draft=("fixed", 1.0))
    check(True, make(True, cfg, 2), oracle, f"batch {batch} vocab {vocab}")


@pytest.mark.parametrize("siblings", [1, 7, 20])
def test_tree_star_rejects_every_child(oracle, siblings):
    """All nodes hang under the root and are rejected one after the other: a residual of a residual, as deep as it gets."""
    cfg = TINY.scaled(batch=4, vocab=5000, logit_dtype="bf16", depth=("fixed", siblings), sigma_draft=("fixed", 2.0))
    inp = make(True, cfg, 7)
    inp["tree_parent"] = np.tile(np.concatenate([[-1], np.zeros(siblings)]), 4).astype(np.int32)
    inp["u_accept"][:] = np.float32(0.999999)
    check(True, inp, oracle, f"star of {siblings}")
