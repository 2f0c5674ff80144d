"""Tile choice of small MatMuls without a device: which form the default rule takes, read from the kernel's name."""
import numpy as np
import pytest

from paper_2108_13342_amd import api
from workloads import configs
from workloads.graph import GraphBuilder


def _kernel(M, K, N, dtype, batch=(), a_transposed=False, weight=True):
    """Name of the MatMul kernel of x @ w; without `weight` both operands are activations, w contiguous along N."""
    b = GraphBuilder("gemm_tiles", dtype)
    zeros = lambda shape: np.zeros(shape, dtype=np.float32)
    if a_transposed:
        x = configs._transpose(b, b.input("x", (K, M), zeros((K, M))), (1, 0))
    else:
        x = b.input("x", batch + (M, K), zeros(batch + (M, K)))
    w = (b.weight if weight else b.input)("w", batch + (K, N), zeros(batch + (K, N)))
    b.mark_output(configs._matmul(b, x, w))
    spec = b.finish()
    g, _ = api.graph_from_spec(spec)
    g.rewrite()
    plan = api.Plan(g, [1] * len([t for t in spec.tensors.values() if t.kind == "weight"]))
    return [d["kernel_name"].split(":")[1] for d in plan.describe() if d["family"] == 2 and not d["prepare_only"]][0]


@pytest.mark.parametrize("M,K,N,kw,tile", [
    # a K that no length divides: the number of tiles counts, not the padding alone
    (40, 3080, 768, {}, "32x32x256_a0b0_w8_dma3"),
    (40, 3136, 768, {}, "32x32x256_a0b0_w8_dma3"),
    (40, 520, 768, {}, "32x32x128_a0b0_w8_dma4"),
    (40, 1000, 768, {}, "32x32x256_a0b0_w8_dma3"),
    (300, 1288, 768, {}, "32x32x128_a0b0_w8_dma4"),
    (33, 3072, 768, {}, "32x32x384_a0b0_w8_dma3"),
    # transposing loaders: fewer, longer tiles
    (640, 640, 64, dict(batch=(6,), weight=False), "32x32x384_a0b1_w8"),
    (320, 640, 640, dict(a_transposed=True, weight=False), "32x32x384_a1b1_w8"),
    (504, 384, 768, dict(a_transposed=True, weight=False), "32x32x384_a1b1_w8"),
    (768, 384, 384, dict(a_transposed=True, weight=False), "32x32x384_a1b1_w8"),
    (896, 896, 64, dict(batch=(8,), weight=False), "32x32x256_a0b1_w8"),
])
def test_length_of_k_tiles_16_bit(M, K, N, kw, tile):
    assert _kernel(M, K, N, "bf16", **kw) == "mfma_" + tile


@pytest.mark.parametrize("K,bk,buffers", [(128, 128, 3), (132, 64, 3), (192, 64, 3), (256, 128, 3), (576, 64, 4), (1000, 128, 3), (3080, 64, 3)])
def test_length_of_k_tiles_f32(K, bk, buffers):
    assert _kernel(256, K, 768, "f32") == f"mfma_32x32x{bk}_a0b0_w8_dma{buffers}"


@pytest.mark.parametrize("M,K,N,tile", [
    (256, 768, 1024, "32x32x64_a0b0_w8_dma4"), (257, 768, 1024, "32x32x128_a0b0_w8"),          # 256 and 288 tiles: straight into LDS, through registers
    (256, 700, 1024, "32x32x64_a0b0_w8_dma3"), (288, 700, 1024, "32x32x64_a0b0_w8"),
])
def test_line_of_direct_to_lds_tiles_f32(M, K, N, tile):
    assert _kernel(M, K, N, "f32") == "mfma_" + tile


@pytest.mark.parametrize("M,K,N,kw,tile", [
    # more than one 32x32 tile per compute unit, both operands read along K: short tiles ...
    (500, 768, 768, {}, "32x32x64_a0b0_dma4"),
    (900, 512, 768, {}, "32x32x64_a0b0_dma4"),
    (900, 768, 768, {}, "32x32x64_a0b0_dma4"),
    (400, 384, 768, {}, "32x32x64_a0b0_dma4"),
    (300, 768, 2304, {}, "32x32x64_a0b0_dma4"),
    # ... whatever the length of K and the size of the weight (more than 4 MB from the second on)
    (900, 1536, 768, {}, "32x32x64_a0b0_dma4"),
    (72, 768, 3072, {}, "32x32x64_a0b0_dma4"),            # 288 tiles
    (96, 1024, 4096, {}, "32x32x64_a0b0_dma4"),           # 384
    (128, 512, 4096, {}, "32x32x64_a0b0_dma4"),
    (128, 512, 4104, {}, "32x32x64_a0b0_dma4"),
    (128, 768, 3072, {}, "32x32x64_a0b0_dma4"),
    # ... unless rows of K start anywhere in a memory line, and K is long or both it and the weight are
    (900, 1528, 768, {}, "32x32x64_a0b0_dma4"),
    (900, 1544, 768, {}, "32x32x128_a0b0_w8_dma3"),
    (200, 1400, 1400, {}, "32x32x64_a0b0_dma4"),
    (64, 1400, 8000, {}, "32x32x128_a0b0_w8_dma3"),
    (72, 776, 3072, {}, "32x32x64_a0b0_dma4"),
    # ... or the chip is not full
    (256, 768, 1024, {}, "32x32x384_a0b0_w8_dma3"),
    (257, 768, 1024, {}, "32x32x64_a0b0_dma4"),
    (512, 512, 64, dict(batch=(12,), weight=False), "32x32x256_a0b1_w8"),
])
def test_short_k_tiles_where_workgroups_hide_each_other(M, K, N, kw, tile):
    assert _kernel(M, K, N, "f16", **kw) == "mfma_" + tile


@pytest.mark.parametrize("M,K,N,dtype,weight,tile", [
    # a transposed left operand: larger tiles from fewer tiles on
    (1000, 768, 512, "bf16", False, "32x32x384_a1b1_w8"),         # 128 tiles of 64x64
    (704, 704, 768, "bf16", False, "64x64x64_a1b1"),              # 132
    (768, 512, 768, "bf16", False, "64x64x64_a1b1"),              # 144
    (904, 1024, 768, "f16", False, "64x64x64_a1b1"),              # 180
    (768, 512, 768, "bf16", True, "64x64x64_a1b0"),
    (904, 768, 768, "bf16", True, "64x64x64_a1b0"),
    (1024, 512, 768, "f32", False, "32x32x128_a1b1_w8"),          # 192
    (960, 256, 832, "f32", False, "64x64x16_a1b1"),               # 195
    (1024, 512, 1024, "f32", False, "64x64x16_a1b1"),             # 256
    (1024, 768, 1024, "f32", False, "64x64x16_a1b1"),
    (1024, 300, 1024, "f32", True, "64x64x16_a1b0"),
    (900, 512, 1000, "f32", True, "64x64x16_a1b0"),               # 240
    (1024, 768, 1024, "f32", True, "32x32x128_a1b0_w8"),
])
def test_line_for_a_transposed_left_operand(M, K, N, dtype, weight, tile):
    assert _kernel(M, K, N, dtype, a_transposed=True, weight=weight) == "mfma_" + tile


@pytest.mark.parametrize("M,K,N,dtype,tile", [
    (384, 256, 1024, "bf16", "32x32x64_a0b0_dma4"), (385, 256, 1024, "bf16", "64x64x64_a0b0_dma4"),              # K below 512: 96 tiles, 112 tiles
    (64, 248, 768, "bf16", "64x64x64_a0b0"), (64, 256, 768, "bf16", "32x32x256_a0b0_w8_dma3"),                  # the smallest K in 16 bits
    (704, 1536, 1024, "f16", "32x32x64_a0b0_dma4"), (768, 1536, 1024, "f16", "64x64x64_a0b0_dma4"),          # 176 tiles, 192 tiles
    (1024, 256, 1024, "f32", "32x32x128_a0b0_w8"), (1088, 256, 1024, "f32", "128x64x16_a0b0"),             # 256 tiles, 272 tiles
    (64, 124, 768, "f32", "64x64x16_a0b0"), (64, 128, 768, "f32", "32x32x128_a0b0_w8_dma3"),                    # the smallest K in f32
])
def test_lines_between_tile_forms(M, K, N, dtype, tile):
    assert _kernel(M, K, N, dtype) == "mfma_" + tile


@pytest.mark.parametrize("M,K,N,batch,tile", [
    # long f32 tiles that would be filled up with zeros on a full chip
    (900, 132, 768, (), "32x32x16_a0b0"),
    (500, 136, 900, (), "32x32x16_a0b0"),
    (1024, 132, 1024, (), "64x64x16_a0b0"),
    (1024, 200, 1024, (), "64x64x16_a0b0"),
    (256, 132, 768, (), "32x32x64_a0b0_w8_dma3"),              # the chip is not full
    (700, 160, 768, (), "32x32x64_a0b0_w8"),              # few zeros
    (1024, 256, 1024, (), "32x32x128_a0b0_w8"),
    (200, 200, 64, (40,), "32x32x128_a0b1_w8"),           # the transposing loader gains all the same
])
def test_f32_tiles_filled_with_zeros(M, K, N, batch, tile):
    assert _kernel(M, K, N, "f32", batch=batch, weight=not batch) == "mfma_" + tile
