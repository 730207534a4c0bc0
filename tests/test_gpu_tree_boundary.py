"""Sampled tree walk: the entries that a pass cannot call before the rejected child's normaliser is exact (r within 1e-4 of the
proposal) and sets aside, none to a run, several, and more than a run holds, after the first rejection at a node, the second and
later ones.  Tokens, lengths and paths equal the oracle's."""
import numpy as np
import pytest

from paper_2604_09562_amd import synth
from tests.test_gpu_tree_sample import compare

pytestmark = pytest.mark.gpu

TINY = synth.CONFIGS[0]


def softmax(x):
    e = np.exp(x - x.max())
    return e / e.sum()


@pytest.mark.parametrize("siblings", [1, 2, 3, 5])
@pytest.mark.parametrize("share", [0.0, 0.001, 0.05, 0.7])   # of a block's 2048 entries at the boundary: about 0, 2, 100, 1400
@pytest.mark.parametrize("vocab", [2000, 9001])
def test_proposals_that_nearly_equal_what_is_left(oracle, siblings, share, vocab):
    """Children of the root, each proposal the residual of the rejections before it but for a token that it overrates (its
    draft, rejected), a relative 1e-5 of noise on `share` of the entries and a factor on the others."""
    B, cfg = 6, TINY.scaled(batch=6, vocab=vocab, logit_dtype="f32", temperature=1.0, depth=("fixed", siblings))
    inp = synth.make_tree_sample_inputs(cfg, seed=11, row_pad=(-vocab) % 4)
    inp["tree_parent"] = np.tile(np.concatenate([[-1], np.zeros(siblings)]), B).astype(np.int32)
    inp["u_accept"][:] = np.float32(0.9)
    rng = np.random.default_rng(siblings * 100 + int(share * 1000))
    for b in range(B):
        t0, d0 = b * (siblings + 1), b * siblings
        r = softmax(inp["target_logits"][t0, :vocab].astype(np.float64))
        for c in range(siblings):
            left = np.flatnonzero(r > 0)
            near = rng.random(vocab) < share
            factor = np.where(near, 1.0 + 1e-5 * rng.standard_normal(vocab), np.exp(0.5 * rng.standard_normal(vocab)))
            low = left[np.argsort(r[left])[len(left) // 4]]      # a token of little mass, so that the normalisers stay level
            factor[low] = 4.0
            q = r * factor
            with np.errstate(divide="ignore"):
                row = np.where(q > 0, np.log(q), -80.0).astype(np.float32)
            inp["draft_logits"][d0 + c, :vocab] = row
            inp["draft_tokens"][d0 + c] = low
            rest = np.maximum(r - softmax(row.astype(np.float64)), 0.0)
            r = rest / rest.sum()
    ref = compare(inp, oracle, f"share {share}, {siblings} siblings, vocab {vocab}")
    assert np.all(ref["accepted_len"] == 0) and np.isfinite(ref["ratio"]).all()   # every child offered and rejected


@pytest.mark.parametrize("vocab", [2048, 20000])
@pytest.mark.parametrize("moved", [200, 600, 1990])   # entries of the first 2000 whose logits trade places
def test_equal_bf16_logits_on_the_boundary(oracle, vocab, moved):
    """A proposal with the target's logits in another order: equal normalisers, and every entry that stayed is exactly on the boundary."""
    B, cfg = 6, TINY.scaled(batch=6, vocab=vocab, logit_dtype="bf16", depth=("fixed", 2))
    inp = synth.make_tree_sample_inputs(cfg, seed=12)
    inp["tree_parent"] = np.tile(np.array([-1, 0, 0], np.int32), B)
    inp["u_accept"][:] = np.float32(0.999)
    rng = np.random.default_rng(moved)
    for b in range(B):
        row = inp["target_logits"][3 * b, :vocab]
        r = softmax(synth.decode_storage(row, "bf16").astype(np.float64) / float(cfg.temperature))
        for c in range(2):
            at = rng.choice(2000, moved, replace=False)
            stored = row.copy()
            stored[at] = row[np.roll(at, 1)]
            inp["draft_logits"][2 * b + c, :vocab] = stored
            q = softmax(synth.decode_storage(stored, "bf16").astype(np.float64) / float(cfg.temperature))
            # overrated most among the tokens with a share in what is left (which is 0 but for rounding where nothing moved)
            inp["draft_tokens"][2 * b + c] = int(np.argmax(np.where(r > 1e-9, q / np.maximum(r, 1e-300), 0.0)))
            r = np.maximum(r - q, 0.0)
            r /= r.sum()
    ref = compare(inp, oracle, f"{moved} moved, vocab {vocab}")
    assert np.all(ref["ratio"][0::2] < 0.999)   # every first child rejected


def few_live(batch, siblings, vocab, live, logit_dtype, seed):
    """Requests whose target row at the root has `live` logits and -inf for the others; every child of the root has that row for a
    proposal.  Returns the batch and the live tokens of each request, in ascending order, each but the last with a free one behind it."""
    cfg = TINY.scaled(batch=batch, vocab=vocab, logit_dtype=logit_dtype, temperature=1.0, depth=("fixed", siblings))
    inp = synth.make_tree_sample_inputs(cfg, seed=seed, row_pad=(-vocab) % 8)
    inp["tree_parent"] = np.tile(np.concatenate([[-1], np.zeros(siblings)]), batch).astype(np.int32)
    inp["u_accept"][:] = np.float32(0.5)
    rng = np.random.default_rng(seed)
    none = synth.store(np.full(1, -np.inf, np.float32), logit_dtype)[0]
    tokens = []
    for b in range(batch):
        at = np.sort(rng.choice(vocab // 8, live, replace=False)) * 8 + rng.integers(0, 6, live)
        row = inp["target_logits"][b * (siblings + 1), :vocab]
        keep = row[at].copy()
        row[:] = none
        row[at] = keep
        inp["draft_logits"][b * siblings:(b + 1) * siblings, :vocab] = row
        tokens.append(at)
    return inp, tokens, none


@pytest.mark.parametrize("logit_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("live", [1, 3, 40, 120])
@pytest.mark.parametrize("vocab", [1000, 9001])
def test_no_residual_of_equal_rows(oracle, vocab, live, logit_dtype):
    """Target row and proposals alike, a first child that neither gives any mass: nothing is left, so r stays what it was, and the second
    child, which r and q weigh alike, is accepted.  (A product that is rounded on one side only leaves 1e-17 of each entry.)"""
    B, siblings = 8, 2
    inp, tokens, _ = few_live(B, siblings, vocab, live, logit_dtype, seed=live)
    for b in range(B):
        inp["draft_tokens"][b * siblings] = tokens[b][0] + 1
        inp["draft_tokens"][b * siblings + 1] = tokens[b][b % live]
    ref = compare(inp, oracle, f"{live} live of {vocab}")
    assert np.all(ref["accepted_nodes"][:, 0] == 2)
    # without the second child: the arg-maximum of the target row
    inp, tokens, _ = few_live(B, 1, vocab, live, logit_dtype, seed=live)
    for b in range(B):
        inp["draft_tokens"][b] = tokens[b][0] + 1
    ref = compare(inp, oracle, f"{live} live of {vocab}, one child")
    assert np.all(ref["accepted_len"] == 0)


@pytest.mark.parametrize("logit_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("live", [3, 40, 120])
def test_no_residual_after_a_second_rejection(oracle, live, logit_dtype):
    """The first proposal has one live logit moved to the token behind it: what is left of the target row is all at that logit's token.  The
    second proposal has only that one, its draft another: nothing is left, r stays, and the third child, that token, is accepted."""
    B, siblings, vocab = 8, 3, 1000
    inp, tokens, none = few_live(B, siblings, vocab, live, logit_dtype, seed=10 + live)
    for b in range(B):
        hot = int(tokens[b][b % live])
        first, second = inp["draft_logits"][b * siblings, :vocab], inp["draft_logits"][b * siblings + 1, :vocab]
        first[hot + 1], first[hot] = first[hot], none     # (in its neighbour's place: the sums of both rows round alike)
        keep = second[hot]
        second[:] = none
        second[hot] = keep
        inp["draft_tokens"][b * siblings:(b + 1) * siblings] = hot + 1, int(tokens[b][(b + 1) % live]), hot
    ref = compare(inp, oracle, f"{live} live, second rejection")
    assert np.all(ref["accepted_nodes"][:, 0] == 3)
