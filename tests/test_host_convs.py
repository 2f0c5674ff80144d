"""Kernels of convolutions compile, whatever stands in front of their operand; no device needed."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(__file__))
import unit_graphs as U
from paper_2108_13342_amd import api


FRONTS = [                                                   # (what stands in front, shape, ...): K on its lanes, in 16 bits
    ("Relu", (2, 16, 1, 1, 8), {}),                          # 2 vectors on 2 lanes
    ("Relu", (2, 24, 8, 8, 16), dict(keep=True)),            # 3 on 4, a channels-last map
    ("Relu", (1, 1160, 1, 1, 9), {}),                     # 145 on a wavefront
    ("Relu", (3, 104, 3, 5, 24), dict(keep=True)),           # 13 on 16
]


def _kernels(spec, **kw):
    g, _ = api.graph_from_spec(spec)
    g.rewrite()
    plan = api.Plan(g, [1] * len(spec.weights()), **kw)
    return [d["kernel_name"].split(":")[1] for d in plan.describe() if not d["prepare_only"]]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("front,args,kw", FRONTS)
def test_operators_in_front_of_a_convolution_of_few_results(front, args, kw, dtype, tmp_path):
    spec = U.front_conv_block(front, *args, dtype=dtype, **kw)
    assert any(k.startswith("dot_") and k.endswith("_front") for k in _kernels(spec, layout=1)), _kernels(spec, layout=1)
    assert api.precompile_spec(spec, cache_dir=str(tmp_path), layout=1) > 0
    assert api.precompile_spec(spec, cache_dir=str(tmp_path), layout=0) > 0


CASTS = [(2, 16, 1, 1, 8), (70, 256, 1, 1, 24), (300, 256, 1, 1, 64), (8, 64, 16, 16, 48)]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("args", CASTS)
def test_pointwise_operand_stored_in_another_type(args, dtype, tmp_path):
    """A Cast that becomes part of the load: the vector paths read the convolution's own type only."""
    spec = U.front_conv_block("Cast", *args, dtype=dtype)
    for layout in (0, 1):
        assert api.precompile_spec(spec, cache_dir=str(tmp_path), layout=layout, rewrite=dtype != "f32") > 0      # (a widening Cast is rewritten away)


@pytest.mark.parametrize("seed", [139, 231, 380])
def test_random_networks_with_operators_in_front(seed, tmp_path):
    assert api.precompile_spec(U.random_cnn(seed, "f16", n_ops=10 + seed % 7), cache_dir=str(tmp_path), layout=1) > 0


def test_environment_does_not_reach_convolution_tiles(monkeypatch):
    """(An override without checks once divided by the wavefront counts it was given.)"""
    spec = U.conv_pair_block(2, 48, 43, 41, 40, 3)
    plain = _kernels(spec, layout=1)
    monkeypatch.setenv("DNNF_CONV_TILE", "32,32,64,0,0,0,2")
    assert _kernels(spec, layout=1) == plain


@pytest.mark.parametrize("args,large", [((1, 64, 107, 107, 474, 3), False), ((1, 64, 107, 107, 480, 3), True),
                                        ((10, 496, 21, 21, 527, 1), False), ((10, 496, 21, 21, 528, 1), True),
                                        ((4, 168, 64, 64, 474, 3), True)])       # 24 K tiles: the store is little of it
def test_tiles_of_results_stored_one_at_a_time(args, large):
    """Channels that are no multiple of 8 and few K tiles: no 128x128 tile, whose store alone would take as long as its loop."""
    names = _kernels(U.conv_pair_block(*args), layout=1)
    name = next(n for n in names if n.startswith("igemm_") and "_dma" in n)
    bm, bn = map(int, name.split("_")[1].split("x")[:2])
    assert (bm * bn >= 128 * 128) == large, names
