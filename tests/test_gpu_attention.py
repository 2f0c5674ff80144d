"""GPU parity of the streaming-softmax attention block (the extension beyond the paper's table:
MatMul -> One-to-One operators -> Softmax -> MatMul in one kernel) against the fp64 oracle, which
evaluates the same operators one by one with a plain row softmax."""
import numpy as np
import pytest

import unit_graphs as U
from parity import TOL, check_against_oracle, check_blocks_against_oracle, rel_err
from workloads import configs

pytestmark = pytest.mark.gpu


def _attention_blocks(s):
    return [d for d in s.plan.describe() if d["family"] == 6]


@pytest.mark.parametrize("args,kw", [
    ((2, 3, 128, 128, 64), dict(dtype="f16", mask="add")),                       # exact tiles
    ((1, 2, 200, 200, 64), dict(dtype="bf16", mask="causal")),                   # ragged queries and keys, causal mask tensor
    ((2, 2, 72, 328, 64), dict(dtype="f16", mask="add", merge_heads=False)),     # cross-attention shape, plain output layout
    ((1, 4, 256, 192, 32), dict(dtype="bf16", mask=None, kt_stored=False)),      # K handed over untransposed, head dimension 32
    ((1, 1, 40, 64, 128), dict(dtype="f16", mask="add")),                        # head dimension 128, fewer queries than a tile
])
def test_attention_block(args, kw):
    spec = U.attention_block(*args, **kw)
    s, _ = check_against_oracle(spec, attention=1)
    blocks = _attention_blocks(s)
    assert len(blocks) == 1 and len([d for d in s.plan.describe() if not d["prepare_only"] and d["family"] != 5]) == 1, s.plan.describe()


@pytest.mark.parametrize("args,kw", [
    ((1, 2, 33, 33, 64), dict(dtype="bf16", mask="causal")),                     # one key past a half tile, mask rows of odd length
    ((2, 2, 77, 77, 64), dict(dtype="f16", mask="add")),                         # 13 keys in the second tile
    ((1, 3, 50, 3, 32), dict(dtype="f16", mask=None, merge_heads=False)),        # fewer keys than a vector of scores
    ((1, 1, 130, 203, 128), dict(dtype="bf16", mask="add")),                     # more queries than a workgroup takes
    ((2, 1, 20, 68, 64), dict(dtype="f16", mask="causal")),                      # a multiple of 4 that is none of 8: mask in vectors
    ((1, 2, 7, 130, 64), dict(dtype="bf16", mask="add")),                        # a multiple of 2
])
def test_attention_block_any_number_of_keys(args, kw):
    """Keys read row by row (the Transpose in front of them joins the block): any number of them."""
    s, _ = check_against_oracle(U.attention_block(*args, kt_stored=False, **kw), attention=1)
    blocks = _attention_blocks(s)
    assert len(blocks) == 1 and len([d for d in s.plan.describe() if not d["prepare_only"] and d["family"] != 5]) == 1, s.plan.describe()


@pytest.mark.parametrize("args,kw", [
    ((1, 2, 70, 253, 64), dict(dtype="bf16", mask="causal")),                    # rows of odd length: groups of four start at any element
    ((2, 1, 9, 131, 32), dict(dtype="f16", mask="where")),                       # truth values; three keys in the last group
    ((1, 3, 64, 66, 64), dict(dtype="bf16", mask="where")),                      # two
    ((1, 1, 33, 5, 32), dict(dtype="f16", mask="causal")),                       # one, behind one whole group
    ((1, 2, 20, 140, 64), dict(dtype="f16", mask="where")),                      # a multiple of 4 that is none of 8
])
def test_attention_masks_of_any_row_length(args, kw):
    s, _ = check_against_oracle(U.attention_block(*args, kt_stored=False, **kw), attention=1)
    assert len(_attention_blocks(s)) == 1, s.plan.describe()


@pytest.mark.parametrize("SK,kt_stored", [(33, False), (130, False), (72, True), (72, False)])
def test_attention_infinite_value_of_the_last_key(SK, kt_stored):
    """An infinite value behind a probability above zero is an infinite result: the keys that fill up the last tile add nothing."""
    from oracle.interp import run_graph
    from paper_2108_13342_amd import api

    spec = U.attention_block(1, 2, 40, SK, 64, dtype="bf16", mask=None, kt_stored=kt_stored)
    v = np.array(spec.tensors["v"].data, dtype=np.float64)
    v[0, 1, SK - 1, 3], v[0, 0, SK - 1, 7] = np.inf, -np.inf
    spec.tensors["v"].data = v
    s = api.Session(spec, attention=1)
    assert len(_attention_blocks(s)) == 1
    s.run()
    got = list(s.result().values())[0]
    want = list(run_graph(spec).values())[0]
    assert np.array_equal(np.isposinf(got), np.isposinf(want)) and np.array_equal(np.isneginf(got), np.isneginf(want)) and not np.isnan(got).any()
    finite = np.isfinite(want)
    assert np.isinf(want).any() and rel_err(got[finite], want[finite]) <= TOL["bf16"]


def test_attention_keys_stored_transposed_need_vectors():
    """K handed over as its transpose is read along the keys: a number that is no multiple of 8 stays three blocks."""
    s, _ = check_against_oracle(U.attention_block(1, 2, 33, 33, 64), attention=1)
    assert not _attention_blocks(s)


def test_attention_off_by_default():
    """Without the option the table decides: Many-to-Many + Many-to-Many stays split."""
    from paper_2108_13342_amd import api
    s = api.Session(U.attention_block(2, 3, 128, 128, 64), fusion=1)
    assert not _attention_blocks(s)
    assert len([d for d in s.plan.describe() if d["family"] in (1, 2)]) == 3


def test_fully_masked_tiles_and_large_scores():
    """Whole key tiles at -1e4 (their probabilities underflow to exactly 0) and scores whose running
    maximum changes late in the row: the rescaling of the partial sums must reproduce the row softmax."""
    spec = U.attention_block(1, 2, 192, 256, 64, dtype="f16", mask="causal")
    q = spec.tensors["q"].data
    q[..., 150:, :] *= 6.0          # rows whose largest score sits in their last key tile
    check_against_oracle(spec, attention=1)


def test_transformer_layers_with_attention_block():
    # reduced variants whose head dimension (32) the template supports
    for name, kw in configs.SMALL_HEAD32.items():
        spec = configs.CONFIGS[name](**kw)
        s, _ = check_against_oracle(spec, attention=1)
        assert len(_attention_blocks(s)) == kw.get("L", 1), name


def test_gpt2_full_size_attention_plan():
    """The benchmark's configuration (tuned plan, attention blocks) at full size against the oracle on one
    sequence; 12 layers of bf16 rounding accumulate as in the plan without the extension."""
    from oracle.interp import run_graph
    from paper_2108_13342_amd import api

    spec = configs.CONFIGS["gpt2_decoder"]()
    s = api.Session(spec, fusion=1, profile=1, tune=1, attention=1)
    assert len(_attention_blocks(s)) == 12
    s.run()
    got = s.result()
    ids = spec.tensors["input_ids"].data
    sub = configs.CONFIGS["gpt2_decoder"](B=1)
    for nm, t in sub.tensors.items():
        if t.kind == "weight" and nm in spec.tensors and spec.tensors[nm].data.shape == t.data.shape:
            t.data = spec.tensors[nm].data
    want = run_graph(sub, feeds={"input_ids": ids[1:2]})
    for name, w in want.items():
        g = got[name][:, 1:2] if name.startswith("present_") else got[name][1:2]
        assert rel_err(g, w) <= TOL["bf16"] * np.sqrt(12), name
