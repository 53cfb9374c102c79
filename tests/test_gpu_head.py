"""The bf16 head + Euler kernel at the edges of its dispatch, against the oracle: chunks per wave
0 or 1 (d = 128), 3 and 4, 5 and 6, 8 and 9, 12; token counts of one row, one off a 16-row tile,
and of more rows than one tile per compute unit; every patch size; the residual variant (a reuse
step's g = h_in + r) against the cache-apply path."""
import numpy as np
import pytest

from oracle import dit
from paper_2608_16354_amd import inputs as I
from tests.gpu_util import mod_input, rel_l2, say, t
from tests.test_gpu_kernels import _Head

pytestmark = pytest.mark.gpu


def _shape(d, patch, lat, n_txt=3, n_blocks=1):
    return I.ModelShape(n_blocks=n_blocks, hidden=d, heads=d // 64, head_dim=64, mlp_hidden=128,
                        lat_c=64 // patch ** 2, lat_t=lat[0], lat_h=lat[1] * patch, lat_w=lat[2] * patch,
                        patch=patch, n_txt=n_txt, dtype="bf16")


CASES = [(128, 2, (1, 3, 11)), (768, 1, (1, 1, 1)), (896, 4, (2, 5, 3)), (1280, 8, (1, 5, 7)), (1408, 2, (3, 37, 41)),
         (2048, 1, (2, 4, 4)), (2176, 2, (5, 29, 31)), (3072, 4, (3, 7, 13)), (3072, 2, (1, 1, 17))]


@pytest.mark.parametrize("d, patch, lat", CASES)
def test_head_edges(dev, d, patch, lat):
    import torch
    from paper_2608_16354_amd import api
    m = _shape(d, patch, lat)
    W = I.Weights(m, 150)
    dm, ws = api.DeviceModel(_Head(W), dev), api.Workspace(m, 2, dev)
    g = np.stack([I.hidden_state(m, (70 + b,)) for b in range(2)])
    x = np.stack([I.latent(m, 150, b) for b in range(2)])
    hm = mod_input(m, (72,))[:2]
    dx = t(x, dev)
    say("head edges", d, patch, lat, "N_v =", m.n_v)
    api.dc_head_euler(dm, t(hm, dev), t(g, dev), dx, -0.02, [1], ws)
    torch.cuda.synchronize()
    got = dx.cpu().numpy()
    assert np.array_equal(got[0], x[0])
    v = dit.head(dit.Params(W), hm.astype(np.float64), g[1, : m.n_v].astype(np.float64))
    want = dit.euler(x[1].astype(np.float64), v, 0.52, 0.5)
    err = rel_l2(got[1] - x[1], want - x[1])
    say("head update rel-L2", err)
    # hi + lo operands keep 2^-17 = 7.6e-6; the update is read back from x at fp32: |x| / |update| x
    # 2^-24, about 50 x 6e-8
    assert err < 2e-5


@pytest.mark.parametrize("d", [128, 3072])
def test_head_rows_with_an_outlier_first_value(dev, d):
    """The narrowest and the widest model on rows whose mean is 40 standard deviations from zero, some
    with a first value (the shift of the folded LayerNorm) 900 from the mean."""
    import torch
    from paper_2608_16354_amd import api
    m = _shape(d, 2, (3, 7, 9))
    W = I.Weights(m, 152)
    dm, ws = api.DeviceModel(_Head(W), dev), api.Workspace(m, 1, dev)
    g, x = I.hidden_state(m, (74,)), I.latent(m, 152, 0)
    g[: m.n_v] += np.float32(40 * 0.16)
    g[: m.n_v: 7, 0] += np.float32(900 * 0.16)
    hm = mod_input(m, (75,))[:2]
    dx = t(x[None], dev)
    say("head outlier rows", d)
    api.dc_head_euler(dm, t(hm, dev), t(g[None], dev), dx, -0.02, [0], ws)
    torch.cuda.synchronize()
    v = dit.head(dit.Params(W), hm.astype(np.float64), g[: m.n_v].astype(np.float64))
    want = dit.euler(x.astype(np.float64), v, 0.52, 0.5)
    err = rel_l2(dx[0].cpu().numpy() - x, want - x)
    say("head update rel-L2 (outliers)", err)
    # a row's first value lies at most sqrt(d) = 55 of its own standard deviations from its mean,
    # so y keeps 55 x 2^-17 of the result
    assert err < 55 * 2.0 ** -17


@pytest.mark.parametrize("d, lat", [(128, (1, 3, 11)), (768, (2, 9, 9)), (1280, (1, 5, 7)), (2048, (3, 7, 11)),
                                    (2176, (1, 9, 5))])
def test_reuse_step_matches_cache_apply(dev, d, lat):
    """A two-step sample (refresh, reuse): its second step equals patch embedding, cache apply and
    head called one by one on the sample's own cache (widths up to 2,048 form g in the head)."""
    import torch
    from paper_2608_16354_amd import api
    m = _shape(d, 2, lat)
    W = I.Weights(m, 151)
    w = I.Workload(0, "head-resid", m, 1, 2, 1, None, "inf", 0.5, I.NO_VETO)
    x, txt = I.latent(m, 151, 0), I.text(m, 151, 0)
    dm, ws, sig = api.DeviceModel(W, dev), api.Workspace(m, 1, dev), I.sigmas(2)

    def sample(legal):
        p = I.scene_problem(w, I.Motion(6.0, 0.25)).replace(legal=np.array(legal, np.uint8))
        smp = api.Sampler(dm, [p], sig, t(x[None], dev), t(txt[None], dev))
        say("reuse step", d, lat, legal)
        realized, _ = smp.run()
        torch.cuda.synchronize()
        out, resid = smp.x.clone(), smp.bufs.resid.clone()
        smp.close()
        return realized[:, 0].tolist(), out, resid

    realized, got, resid = sample([0, 1])
    assert realized == [0, 1]
    # the latent after the refresh step: the same step by its own calls
    mod = torch.zeros((2, m.n_blocks + 1, 6, d), device=dev)
    api.dc_time_modulation(dm, sig[:2], mod, ws)
    cfg, xs = api.model_cfg(m), t(x[None], dev)
    h = torch.zeros((1, m.n_tok, d), device=dev)
    g = torch.zeros_like(h)
    api.dc_patch_embed(dm, xs, t(txt[None], dev), h, [0], ws)
    for k in range(2):
        if k == 0:
            g.copy_(h)
            api.dc_block_forward(dm, 0, mod[0, 0].contiguous(), g, [0], ws)
        else:
            api.dc_patch_embed(dm, xs, t(txt[None], dev), h, [0], ws)
            api.dc_cache_apply(cfg, h, resid, g, [0])
        api.dc_head_euler(dm, mod[k, m.n_blocks, :2].contiguous(), g, xs, float(sig[k + 1] - sig[k]), [0], ws)
    torch.cuda.synchronize()
    # the same kernels on the same numbers; the fused g is the same fp32 addition
    assert rel_l2(got.cpu().numpy(), xs.cpu().numpy()) < 1e-6
