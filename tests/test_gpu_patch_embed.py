"""The patch embedding at its edges, against the oracle: each patch size, token counts one
off the 16-token strip and the 64-token step, a last column group of one wave, latents whose
base is aligned to 4 and 8 bytes only, and samples outside the index list left alone."""
import numpy as np
import pytest

from oracle import dit
from paper_2608_16354_amd import inputs as I
from tests.gpu_util import rel_l2, say, t
from tests.test_gpu_kernels import _Head

pytestmark = pytest.mark.gpu


def _shape(d, patch, lat, n_txt, dtype):
    return I.ModelShape(n_blocks=1, hidden=d, heads=d // 64, head_dim=64, mlp_hidden=128, lat_c=64 // patch ** 2,
                        lat_t=lat[0], lat_h=lat[1] * patch, lat_w=lat[2] * patch, patch=patch, n_txt=n_txt,
                        dtype=dtype)


CASES = [
    # d, patch, (frames, patch rows, patch columns), text rows, floats the latent's base is off by
    (128, 2, (1, 1, 1), 0, 0),
    (256, 1, (1, 1, 17), 1, 0),
    (320 * 2, 2, (3, 5, 7), 5, 0),        # 105 tokens, groups of 256, 256 and 128 columns
    (1152, 4, (1, 3, 5), 3, 0),
    (1152, 2, (5, 7, 11), 120, 1),
    (640, 4, (1, 9, 7), 2, 2),
    (384, 8, (2, 4, 8), 7, 0),            # 64 tokens
    (3072, 2, (13, 9, 11), 226, 0),
]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d, patch, lat, n_txt, off", CASES)
def test_patch_embed_edges(dev, d, patch, lat, n_txt, off, dtype):
    import torch
    from paper_2608_16354_amd import api
    m = _shape(d, patch, lat, n_txt, dtype)
    W = I.Weights(m, 140)
    dm, ws = api.DeviceModel(_Head(W), dev), api.Workspace(m, 3, dev)
    x = np.stack([I.latent(m, 140, b) for b in range(3)])
    txt = np.stack([I.text(m, 140, b) for b in range(3)])
    room = torch.zeros(x.size + off, device=dev)
    dx = room[off:].view(*x.shape)
    dx.copy_(t(x, dev))
    h = torch.full((3, m.n_tok, d), 7.0, device=dev)
    say("patch embed", dtype, d, patch, lat, "N_v =", m.n_v, "base off by", off)
    api.dc_patch_embed(dm, dx, t(txt, dev), h, [2, 0], ws)
    torch.cuda.synchronize()
    got = h.cpu().numpy()
    assert (got[1] == 7.0).all()
    P = dit.Params(W)
    for b in (0, 2):
        want = dit.embed(P, x[b].astype(np.float64), txt[b])
        err = rel_l2(got[b, : m.n_v], want[: m.n_v])
        say("sample", b, "rel-L2", err)
        # split operands: 2^-17 per product; fp32 sums of 64
        assert err < (1e-5 if dtype == "bf16" else 1e-6)
        assert np.array_equal(got[b, m.n_v:], txt[b])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_txt", [0, 5])
def test_patch_embed_without_video_tokens(dev, n_txt, dtype):
    """A latent of no rows: the text rows are all there is, or nothing."""
    import torch
    from paper_2608_16354_amd import api
    m = _shape(256, 2, (1, 0, 8), n_txt, dtype)
    assert m.n_v == 0 and m.n_tok == n_txt
    one = _shape(256, 2, (1, 1, 8), n_txt, dtype)       # weights whose pos is not empty
    dm, ws = api.DeviceModel(_Head(I.Weights(one, 141)), dev), api.Workspace(one, 2, dev)
    dm.cfg = api.model_cfg(m)
    txt = I.normal((2, n_txt, 256), 1.0, (142,))
    h = torch.full((2, n_txt + 1, 256), 7.0, device=dev)
    say("patch embed without video tokens", dtype, n_txt)
    api.dc_patch_embed(dm, torch.zeros(64, device=dev), t(txt, dev), h, [0, 1], ws)
    torch.cuda.synchronize()
    got = h.cpu().numpy().reshape(-1, 256)
    assert np.array_equal(got[: 2 * n_txt], txt.reshape(-1, 256)) and (got[2 * n_txt:] == 7.0).all()
