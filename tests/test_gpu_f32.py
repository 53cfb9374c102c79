"""The fp32 model's kernels at the edges of their dispatch, against the oracle.

Token counts around the 16-query and 32-key tiles (1 token; one short of, at and one past a
tile), and counts that select each split of the attention on 256 compute units: eight waves
per 16 queries (one round of workgroups), four waves (five rounds of 16 queries against
three of 32), 32 queries per workgroup (two rounds against one)."""
import numpy as np
import pytest

from oracle import calibrate as cal
from oracle import dit
from paper_2608_16354_amd import inputs as I
from tests.gpu_util import mod_input, rel_l2, say, t
from tests.test_gpu_kernels import _OneBlock

pytestmark = pytest.mark.gpu


def _shape(d, lat, n_txt, n_blocks=1):
    return I.ModelShape(n_blocks=n_blocks, hidden=d, heads=d // 64, head_dim=64, mlp_hidden=4 * d, lat_c=16,
                        lat_t=lat[0], lat_h=lat[1], lat_w=lat[2], patch=2, n_txt=n_txt, dtype="f32")


@pytest.fixture(scope="module")
def api():
    from paper_2608_16354_amd import api as A
    A.L.load()
    return A


SHAPES = {
    "N1": _shape(128, (1, 2, 2), 0),
    "N15": _shape(128, (3, 2, 10), 0),
    "N16": _shape(256, (1, 8, 8), 0),
    "N33": _shape(256, (2, 8, 8), 1),
    "N257": _shape(384, (4, 16, 16), 1),
    "N1001-h8": _shape(512, (7, 22, 26), 0),
    "N1429-h12": _shape(768, (4, 38, 36), 61),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_block_forward_f32(api, dev, name):
    import torch
    m = SHAPES[name]
    W = I.Weights(m, 120)
    dm = api.DeviceModel(_OneBlock(W, 0), dev)
    ws = api.Workspace(m, 1, dev)
    h = I.hidden_state(m, (50,))
    mod = mod_input(m, (51,))
    dh = t(h[None], dev)
    say("f32 block_forward", name, "N =", m.n_tok)
    api.dc_block_forward(dm, 0, t(mod, dev), dh, [0], ws)
    torch.cuda.synchronize()
    got = dh[0].cpu().numpy()
    want = dit.block(dit.Params(W), 0, mod.astype(np.float64), h.astype(np.float64))
    err_h, err_d = rel_l2(got, want), rel_l2(got - h, want - h)
    say(name, "block rel-L2 h_out", err_h, "update", err_d)
    # fp32 sums of up to 4 d = 3,072 terms: about sqrt(3072) 2^-24 = 3.3e-6 at worst
    assert err_h < 4e-6 and err_d < 4e-6


@pytest.mark.parametrize("lat,n_txt", [((1, 6, 10), 0), ((3, 10, 12), 5), ((5, 28, 40), 1)])
def test_calibration_at_ragged_token_counts(api, dev, lat, n_txt):
    """15 tokens (less than one tile), 95 (ragged; 21 runs in one group of tangents) and 1,401
    (two tangents per group, several groups)."""
    import torch
    m = _shape(256, lat, n_txt, n_blocks=2)
    W = I.Weights(m, 121)
    K, h_max = (8, 5) if m.n_tok == 95 else (4, 2)
    x1, txt = I.latent(m, 121, 0), I.text(m, 121, 0)
    say("calibration N =", m.n_tok)
    q, d = api.dc_calibrate_tables(api.DeviceModel(W, dev), torch.from_numpy(x1).to(dev),
                                   torch.from_numpy(txt).to(dev), I.sigmas(K), h_max, 1e-6)
    tr = cal.Trace(dit.Params(W), x1.astype(np.float64), txt.astype(np.float64), I.sigmas(K))
    qo, do = cal.run_tables(tr, h_max, 1e-6)
    assert np.array_equal(q == 0.0, qo == 0.0) and np.array_equal(d == 0.0, do == 0.0)
    assert np.allclose(q, qo, rtol=1e-5) and np.allclose(d, do, rtol=1e-6)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_calibration_without_video_tokens(api, dev, dtype):
    """A latent of no rows (text only): nothing to perturb and nothing to measure, every entry 0."""
    import dataclasses
    import torch
    one = dataclasses.replace(_shape(128, (1, 4, 4), 5, n_blocks=1), dtype=dtype)
    m = dataclasses.replace(one, lat_h=0)
    assert m.n_v == 0 and m.n_tok == 5
    dm = api.DeviceModel(I.Weights(one, 124), dev)      # weights whose pos is not empty
    dm.cfg = api.model_cfg(m)
    say("calibration without video tokens", dtype)
    q, d = api.dc_calibrate_tables(dm, torch.zeros(64, device=dev), t(I.normal((5, 128), 1.0, (125,)), dev),
                                   I.sigmas(4), 2, 1e-6)
    assert not q.any() and not d.any()


def test_time_modulation_many_blocks(api, dev):
    """65 blocks: one more than the offsets one launch of the table takes."""
    import torch
    m = _shape(128, (1, 4, 4), 0, n_blocks=65)
    W = I.Weights(m, 123)
    sig = np.array([0.9, 0.1])
    mod = torch.full((2, m.n_blocks + 1, 6, m.hidden), 9.0, device=dev)
    say("time_modulation, 65 blocks")
    api.dc_time_modulation(api.DeviceModel(W, dev), sig, mod, api.Workspace(m, 1, dev))
    torch.cuda.synchronize()
    got = mod.cpu().numpy()
    for k in range(2):
        blocks, head = dit.step_modulation(dit.Params(W), sig[k])
        for l in range(m.n_blocks):
            assert rel_l2(got[k, l], blocks[l]) < 1e-5
        assert rel_l2(got[k, m.n_blocks, :2], head) < 1e-5 and not got[k, m.n_blocks, 2:].any()


@pytest.mark.parametrize("d,K", [(256, 1), (256, 17), (384, 40), (1024, 50), (768, 100), (128, 130)])
def test_time_modulation_tiles(api, dev, d, K):
    """Step counts and widths that select each fp32 GEMM tile of the modulation: 32 x 16 (few
    columns), 64 x 48 for 33 to 128 steps and many columns, 32 x 32; ragged step counts."""
    import torch
    m = _shape(d, (1, 4, 4), 0)
    W = I.Weights(m, 122)
    sig = np.linspace(1.0, 0.02, K)
    mod = torch.zeros((K, m.n_blocks + 1, 6, d), device=dev)
    say("time_modulation d =", d, "K =", K)
    api.dc_time_modulation(api.DeviceModel(W, dev), sig, mod, api.Workspace(m, 1, dev))
    torch.cuda.synchronize()
    got = mod.cpu().numpy()
    P = dit.Params(W)
    for k in {0, 15, 16, 31, 32, K // 2, K - 1} & set(range(K)):
        blocks, head = dit.step_modulation(P, sig[k])
        assert rel_l2(got[k, 0], blocks[0]) < 1e-5
        assert rel_l2(got[k, 1, :2], head) < 1e-5
        assert not got[k, 1, 2:].any()


def _one_off(a, dev):
    """a copied to a base one element past an aligned one."""
    import torch
    room = torch.zeros(a.numel() + 1, device=dev)
    room[1:].copy_(a.reshape(-1))
    return room[1:].view(a.shape)


def test_buffers_at_any_element(api, dev):
    """Position table, bias and output of the fp32 patch embedding, and the offsets and table of the
    modulation, whose bases are aligned to 4 bytes only: the results of aligned buffers, bit for bit."""
    import torch
    m = _shape(256, (2, 6, 10), 0, n_blocks=2)
    dm, ws = api.DeviceModel(I.Weights(m, 126), dev), api.Workspace(m, 1, dev)
    x, sig = t(I.latent(m, 126, 0)[None], dev), np.array([0.7, 0.2, 0.1])

    def run(h, mod):
        say("buffers", "aligned to", int(h.data_ptr()) & -int(h.data_ptr()))
        api.dc_patch_embed(dm, x, None, h, [0], ws)
        api.dc_time_modulation(dm, sig, mod, ws)
        torch.cuda.synchronize()
        return h.clone(), mod.clone()

    h, mod = torch.zeros((1, m.n_tok, 256), device=dev), torch.zeros((3, m.n_blocks + 1, 6, 256), device=dev)
    want = run(h, mod)
    keep = {n: _one_off(dm.g[n], dev) for n in ("pos", "b_pe", "head_mod")}
    for n, a in keep.items():
        setattr(dm.cweights, n, a.data_ptr())
    offsets = [_one_off(b["mod_offset"], dev) for b in dm.blocks]
    for c, a in zip(dm._cblocks, offsets):
        c.mod_offset = a.data_ptr()
    got = run(_one_off(torch.zeros_like(h), dev), _one_off(torch.zeros_like(mod), dev))
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
