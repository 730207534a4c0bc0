"""GPU parity of sampled acceptance at the edges of its arithmetic: temperatures so small that a row's distribution is its
arg-maxima, logits that are NaN, uniforms that fall on a boundary of the distribution.  Chain and tree walk against the CPU oracle; tokens equal, as in the other acceptance
tests."""
import numpy as np
import pytest

from paper_2604_09562_amd import synth
from tests.test_gpu_accept import compare as compare_chain, run_gpu as run_chain
from tests.test_gpu_tree_sample import compare as compare_tree, run_gpu as run_tree

pytestmark = pytest.mark.gpu

TINY = synth.CONFIGS[0]


def make(tree, cfg, seed, pad=0, **kw):
    return (synth.make_tree_sample_inputs if tree else synth.make_accept_inputs)(cfg, seed=seed, row_pad=pad, **kw)


def check(tree, inp, oracle, label):
    (compare_tree if tree else compare_chain)(inp, oracle, label=label)


@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("temperature", [1e-3, 1e-5, 1e-9, 1e-15, 1e-18, 1e-20, 1e-30])
def test_tiny_temperatures(oracle, tree, dtype, temperature):
    """max / T beyond the range in which it can be rounded: every row's exponentials are 1 at the maximum and 0 elsewhere."""
    cfg = TINY.scaled(batch=24, vocab=3000, logit_dtype=dtype, temperature=temperature, depth=("uniform", 0, 3),
                      sigma_draft=("fixed", 0.2))
    inp = make(tree, cfg, 4)
    # requests without drafts: two equal maxima, so that the uniform decides between them
    rows = inp["target_logits"]
    lone = [b for b in range(24) if inp["depth"][b] == 0]
    assert lone
    for i, b in enumerate(lone):
        rows[inp["q_indptr"][b], [700, 2500]] = synth.store(np.array([20.0 + 3 * i], np.float32), dtype)[0]
        inp["u_sample"][b] = 0.25 if i % 2 else 0.75
    check(tree, inp, oracle, f"T {temperature} {dtype}")


@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("share", [1, 40, 2990])   # NaN entries of each row
def test_nan_logits_carry_no_mass(oracle, tree, dtype, share):
    """A NaN logit counts as masked: requests without drafts draw what they draw with -inf in its place."""
    cfg = TINY.scaled(batch=16, vocab=3000, logit_dtype=dtype, depth=("fixed", 0))
    inp = make(tree, cfg, 6)
    rng = np.random.default_rng(share)
    at = [rng.choice(3000, share, replace=False) for _ in range(16)]
    for value in (-np.inf, np.nan):
        for b in range(16):
            inp["target_logits"][b, at[b]] = synth.store(np.array([value], np.float32), dtype)[0]
        if value != value:
            got = (run_tree if tree else run_chain)(inp)[1]
            assert np.array_equal(got, masked)
        else:
            check(tree, inp, oracle, f"{share} masked, {dtype}")
            masked = (run_tree if tree else run_chain)(inp)[1]


@pytest.mark.parametrize("tree", [False, True])
def test_uniform_on_a_boundary_next_to_masked_runs(tree):
    """Equal masses 1/n with runs of masked entries between them, and u = j/8 where u * n is a whole number: the running sum
    meets the threshold but for its rounding, at a place where lanes without any mass follow.  The token is one of the two
    entries at the boundary, whichever way the sums round."""
    requests = 400
    rows = np.full((requests, 2048), -np.inf, np.float32)
    want = []
    for seed in range(requests):
        rng = np.random.default_rng(seed)
        n = 2 * int(rng.integers(300, 900))
        idx = np.flatnonzero(np.repeat(rng.random(256) < 0.5, 8))
        n = min(n, len(idx) // 2 * 2)
        idx = np.sort(rng.choice(idx, n, replace=False))
        rows[seed, idx] = 0.0
        want.append(idx)
    cfg = TINY.scaled(batch=requests * 7, vocab=2048, logit_dtype="f32", depth=("fixed", 0), temperature=1.0)
    inp = make(tree, cfg, 0)
    inp["target_logits"][:] = synth.store(np.repeat(rows, 7, axis=0), "f32")
    inp["u_sample"][:] = np.tile(np.arange(1, 8, dtype=np.float32) / 8.0, requests)
    got = (run_tree if tree else run_chain)(inp)[1][:, 0]
    for r in range(requests * 7):
        idx, j = want[r // 7], (r % 7 + 1) * len(want[r // 7])
        ok = idx[[j // 8 - 1, j // 8]] if j % 8 == 0 else idx[[j // 8]]
        assert got[r] in ok, (r, int(got[r]), ok)
