"""Rules that choose between forms of a kernel, read from the generated source without a device."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
import unit_graphs as U
from paper_2108_13342_amd import api
from workloads import configs
from workloads.graph import GraphBuilder


def _sources(spec, rewrite=True, **kw):
    """(kernel name, source) of every block that runs per inference."""
    g, _ = api.graph_from_spec(spec)
    if rewrite:
        g.rewrite()
    plan = api.Plan(g, [1] * len(spec.weights()), **kw)
    return [(d["kernel_name"].split(":")[1], plan.block_source(i)) for i, d in enumerate(plan.describe()) if not d["prepare_only"] and d["family"] != 5]


@pytest.mark.parametrize("args,kw,early", [
    ((85, 1040, 1, 1, 44), dict(scale=False), 1),                       # 255 workgroups, three an image
    ((256, 96, 1, 1, 8), dict(scale=False), 1),
    ((257, 96, 1, 1, 8), dict(scale=False), 0),                         # a compute unit gets two workgroups
    ((4, 96, 7, 7, 8), dict(scale=False), 1),                           # a pool in front, 16 bits
    ((4, 96, 7, 7, 8), dict(scale=False, dtype="f32"), 0),              # a pool in front, f32
])
def test_squeeze_excite_weights_up_front(args, kw, early):
    src = [s for n, s in _sources(U.se_tail_block(*args, **kw), squeeze_excite=2) if "fc" in n]
    assert len(src) == 1 and f"#define SE_ALONE {early}\n" in src[0]


@pytest.mark.parametrize("M,K,N,dtype,rewrite,strip", [
    (64, 1024, 1024, "bf16", True, 0),                                  # stored [N][K] after rewriting
    (64, 1004, 1024, "bf16", True, 3),                                  # K no multiple of a vector: stays [K][N]; an XCD's four tiles of 32
    (64, 1024, 1024, "bf16", False, 3),                                 # not rewritten; four tiles of 32
    (64, 1001, 1024, "f32", True, 5),
    (2000, 1001, 300, "f32", True, 11),                                 # an XCD's tiles cover all columns
])
def test_weight_touches_cover_what_the_tiles_read(M, K, N, dtype, rewrite, strip):
    """A run of columns is a run of memory lines only where the weight's rows of K lie one behind the other."""
    src = _sources(U.gemm_block(M, K, N, dtype), rewrite)[0][1]
    assert "#define W_PREFETCH_LINES" in src and "#define W_PF_WHOLE" not in src and "#define W_PREFETCH_LINES" not in _sources(U.gemm_block(M, 900, N, dtype), False)[0][1]
    assert (f"#define W_PF_STRIP {strip}\n" in src) if strip else ("#define W_PF_STRIP" not in src)


@pytest.mark.parametrize("args,dtype,kernel", [
    ((1, 480, 14, 5, 1), "f16", "dw_chan"), ((4, 480, 14, 5, 1), "f16", "dw_chan"),
    ((8, 480, 14, 5, 1), "f16", "dw_lds"), ((5, 672, 14, 5, 1), "f16", "dw_lds"),        # under 128 staged workgroups, and they are done first
    ((8, 240, 14, 5, 1), "f32", "dw_lds"), ((1, 240, 14, 5, 1), "f32", "dw_chan"),
    ((2, 672, 14, 5, 2), "f16", "dw_lds"), ((1, 144, 56, 5, 2), "f16", "dw_chan"),       # small patches; large ones
    ((6, 128, 28, 7, 1), "f16", "dw_chan"), ((16, 128, 28, 7, 1), "f16", "dw_lds"),      # 7x7
])
def test_depthwise_kernel_by_estimate(args, dtype, kernel):
    N, C, H, K, stride = args
    b = GraphBuilder("dw", dtype)
    zeros = lambda shape: np.zeros(shape, dtype=np.float32)
    x = configs._conv(b, b.input("x", (N, 8, H, H), zeros((N, 8, H, H))), b.weight("w0", (C, 8, 1, 1), zeros((C, 8, 1, 1))), None, 1, 0)
    x = configs._un(b, "Relu", x)
    b.mark_output(configs._un(b, "Relu", configs._conv(b, x, b.weight("w", (C, 1, K, K), zeros((C, 1, K, K))), None, stride, K // 2, C)))
    names = [n for n, _ in _sources(b.finish(), layout=1) if n.startswith("dw_")]
    assert len(names) == 1 and names[0].startswith(kernel), names


@pytest.mark.parametrize("rows,inside", [((3, 5), False), ((8, 5), True), ((4, 4), False)])
def test_concat_operands_stay_inside_the_result_only_on_16_byte_boundaries(rows, inside):
    b = GraphBuilder("cat", "f16")
    zeros = lambda shape: np.zeros(shape, dtype=np.float32)
    w = b.weight("w", (16, 7), zeros((16, 7)))
    parts = [configs._un(b, "Relu", configs._matmul(b, b.input(f"x{i}", (r, 16), zeros((r, 16))), w)) for i, r in enumerate(rows)]
    for p in parts:
        b.mark_output(configs._un(b, "Sigmoid", configs._matmul(b, p, b.weight("v" + p, (7, 9), zeros((7, 9))))))
    y = b.op("Concat", parts, (sum(rows), 7), {"axis": 0})
    b.mark_output(y)
    spec = b.finish()
    g, _ = api.graph_from_spec(spec)
    g.rewrite()
    names = [d["kernel_name"] for d in api.Plan(g, [1] * len(spec.weights())).describe() if "Concat" in d["ops"]]
    assert len(names) == 1 and ("alias_concat" in names[0]) == inside, names
