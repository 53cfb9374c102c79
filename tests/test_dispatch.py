"""The kernels that the GPU tests' shapes are meant for are the ones the library picks for them on
256 compute units (host functions; no GPU)."""
from tests import test_gpu_attention_range as att
from tests import test_gpu_gemm_tiles as gemm
from tests.gpu_util import ATTENTION, TILES, attention_kernel, block_tiles

CUS = 256


def test_gemm_shapes_take_the_tiles_they_name():
    for name, (m, tiles) in gemm.SHAPES.items():
        assert block_tiles(m, CUS) == tiles, name
    assert {t for _, tiles in gemm.SHAPES.values() for t in tiles} == set(TILES)


def test_attention_shapes_take_the_kernel_they_name():
    for name, s in att.SHAPES.items():
        assert attention_kernel(att.model(name), CUS) == s[4], name
    # head_dim 72 has no k_attn16; every other kernel appears at both, whole and split where it can be
    assert {(s[4], s[1]) for s in att.SHAPES.values()} == {(k, d) for k in ATTENTION for d in (64, 72)} - {("k_attn16", 72)}
    assert {(s[4], s[1], s[5]) for s in att.SHAPES.values() if s[4] != "k_attn_keys"} == {
        (k, d, split) for k, d in (("k_attn_bf16", 64), ("k_attn_bf16", 72), ("k_attn16", 64)) for split in (False, True)}
