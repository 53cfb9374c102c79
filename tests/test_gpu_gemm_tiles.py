"""The bf16 block GEMMs' tile shapes at ragged sizes, against the oracle.

Each shape names the tiles that its QKV, out-projection, MLP-up and MLP-down GEMM take on 256
compute units (asserted against block_gemm_tile in gemm.hip), all six of them among the shapes:
token counts one short of and one past a multiple of the tile heights, and widths whose columns
leave part of a column tile empty."""
import numpy as np
import pytest

from oracle import dit
from paper_2608_16354_amd import inputs as I
from tests.gpu_util import block_tiles, compute_units, mod_input, rel_l2, say, t
from tests.test_gpu_kernels import _OneBlock

pytestmark = pytest.mark.gpu


def _shape(d, heads, hd, f, lat, n_txt):
    return I.ModelShape(n_blocks=1, hidden=d, heads=heads, head_dim=hd, mlp_hidden=f, lat_c=16, lat_t=lat[0],
                        lat_h=lat[1], lat_w=lat[2], patch=2, n_txt=n_txt, dtype="bf16")


SHAPES = {
    "d128-N2-k2": (_shape(128, 2, 64, 128, (1, 2, 2), 1), ("64x64",) * 4),             # two k-steps
    "d128-N129": (_shape(128, 2, 64, 256, (1, 16, 32), 1), ("64x64",) * 4),
    "d640-N257": (_shape(640, 10, 64, 2560, (1, 32, 32), 1), ("64x64",) * 4),
    "d1152-N1537-hd72": (_shape(1152, 16, 72, 4608, (3, 32, 64), 1), ("256x128", "64x64", "256x128", "64x64")),
    "d1920-N1155": (_shape(1920, 30, 64, 7680, (5, 22, 42), 0), ("256x128", "128x128", "256x192", "128x128")),
    "d1920-N2562": (_shape(1920, 30, 64, 7680, (10, 32, 32), 2), ("384x192", "256x128", "256x192", "128x128")),
    "d2176-N2879": (_shape(2176, 34, 64, 6528, (8, 34, 42), 23), ("320x256", "256x128", "320x256", "128x128")),
    "d3072-N2305": (_shape(3072, 48, 64, 12288, (9, 32, 32), 1), ("256x192", "256x128", "384x192", "128x128")),
}


@pytest.fixture(scope="module")
def api():
    from paper_2608_16354_amd import api as A
    A.L.load()
    return A


@pytest.mark.parametrize("name", list(SHAPES))
def test_block_at_tile_edges(api, dev, name):
    import torch
    m, tiles = SHAPES[name]
    assert block_tiles(m, compute_units(dev)) == tiles
    W = I.Weights(m, 130)
    dm = api.DeviceModel(_OneBlock(W, 0), dev)
    ws = api.Workspace(m, 1, dev)
    h = I.hidden_state(m, (60,))
    mod = mod_input(m, (61,))
    dh = t(h[None], dev)
    say("block at tile edges", name, "N =", m.n_tok)
    api.dc_block_forward(dm, 0, t(mod, dev), dh, [0], ws)
    torch.cuda.synchronize()
    got = dh[0].cpu().numpy()
    rng = np.random.default_rng(3)
    rows = np.unique(np.concatenate([[0, m.n_tok - 1, min(63, m.n_tok - 1), min(128, m.n_tok - 1)],
                                     rng.integers(0, m.n_tok, 64)]))
    want = dit.block(dit.Params(W), 0, mod.astype(np.float64), h.astype(np.float64), rows=rows)
    err_h, err_d = rel_l2(got[rows], want), rel_l2(got[rows] - h[rows], want - h[rows])
    say(name, "block rel-L2 h_out", err_h, "update", err_d)
    # bf16 operands: 2^-9 relative rounding of each, independent over the sums
    assert err_h < 1e-2 and err_d < 1e-2
