"""The bf16 attention kernels over their dispatch, on rows whose scores lie near zero and far from
it, against the oracle.

Shapes for each kernel, ragged, with and without a split tail; each names the kernel it takes on
256 compute units and whether items are split (asserted against attention_kernel and
attention_splits in attention.hip).  The block is reduced to its attention (W_o = I, gate1 = 1,
gate2 = 0), and biases place the scores (log2 units):
  plain      all near zero;
  low        every score of every row near -740;
  first low  the first 64 keys near -350, the others near zero;
  rise       some keys of later tiles about 90 above the others;
  rise, v    the same with values near 2^50.
With low first tiles 2^-m of their maximum m overflows.  A rise past 64 (log2 of the row sum) has
the kernels raise m after the tile, or redo the work where the products with V overflowed."""
import math

import numpy as np
import pytest

from oracle import dit
from paper_2608_16354_amd import inputs as I
from tests.gpu_util import attention_kernel, attention_splits, compute_units, rel_l2, say, t
from tests.test_gpu_edges import _AttentionOnly, _shape

pytestmark = pytest.mark.gpu

# heads, head_dim, frames x rows x columns of patches, text tokens; kernel, split
SHAPES = {
    "hd64-N57": (4, 64, (1, 7, 8), 1, "k_attn_bf16", False),
    "hd72-N63": (16, 72, (1, 7, 8), 7, "k_attn_bf16", False),
    "hd64-N300-h30": (30, 64, (1, 16, 18), 12, "k_attn_keys", False),
    "hd72-N2000-h16": (16, 72, (5, 20, 20), 0, "k_attn_keys", False),
    "hd64-N1155-h30": (30, 64, (5, 11, 21), 0, "k_attn_bf16", True),      # 38 items per XCD, all split
    "hd64-N1700-h30": (30, 64, (5, 16, 21), 20, "k_attn_bf16", False),    # 53 of 96 slots
    "hd72-N3000-h16": (16, 72, (7, 20, 21), 60, "k_attn_bf16", False),    # 48 of 64 slots
    "hd72-N4200-h16": (16, 72, (10, 20, 21), 0, "k_attn_bf16", True),     # 66 items on 64 slots
    "hd64-N2500-h30": (30, 64, (6, 16, 26), 4, "k_attn16", False),        # 75 of 128 slots
    "hd64-N4360-h30": (30, 64, (9, 22, 22), 4, "k_attn16", True),         # 132 items on 128 slots
}


@pytest.fixture(scope="module")
def api():
    from paper_2608_16354_amd import api as A
    A.L.load()
    return A


class _Placed(_AttentionOnly):
    """_AttentionOnly whose first dimension of every head is a constant query times a key value that
    is constant ("low") or carried by channel 0 of the token (the others)."""

    def __init__(self, W, mode):
        super().__init__(W, 1.0)
        self.mode = mode

    def block(self, l, name):
        a = super().block(l, name)
        d, hd = self.m.hidden, self.m.head_dim
        if name == "w_qkv":
            if self.mode != "low":
                a[:, 0] = 0.0
                a[: 2 * d: hd] = 0.0
                a[d: 2 * d: hd, 0] = 2.0
            if self.mode == "rise, v":
                a[2 * d:] *= np.float32(2.0 ** 50)
        elif name == "b_qkv":
            a = a.copy()
            a[:d: hd] = {"plain": 0.0, "low": -64.0, "first low": -32.0}.get(self.mode, 8.0)
            a[d: 2 * d: hd] = 64.0 if self.mode == "low" else 0.0
            if self.mode == "rise, v":
                a[2 * d:] *= np.float32(2.0 ** 50)
        return a


def model(name):
    heads, hd, lat, n_txt = SHAPES[name][:4]
    return _shape(heads * hd, heads, hd, 128, (lat[0], 2 * lat[1], 2 * lat[2]), n_txt, "bf16")


def _case(name, mode, key):
    m = model(name)
    W = _Placed(I.Weights(m, 160), mode)
    h = I.hidden_state(m, (key,))
    h[: m.n_v] /= 0.16                    # rows of unit scale, video and text alike
    if mode != "low":
        h[:, 0] = 0.0
        if mode == "first low":
            h[:64, 0] = 30.0
        elif mode != "plain":
            h[70::97, 0] = 30.0
            h[-1, 0] = 30.0
    mod = np.zeros((6, m.hidden), np.float32)
    mod[2] = 1.0                          # gate1; gate2 = 0: no MLP
    return m, W, h, mod


def _want(m, W, h, rows):
    """The attention of the sampled rows in fp64, with a, q, k and v rounded to bf16 where the
    device rounds them (q after its log2(e)/sqrt(d_h) scale)."""
    d = m.hidden
    z = np.zeros(d)
    a = I.round_bf16(dit.modulate(h.astype(np.float64), z, z, 1e-6).astype(np.float32)).astype(np.float64)
    w, b = W.block(0, "w_qkv").astype(np.float64), W.block(0, "b_qkv").astype(np.float64)
    kv = a @ w[d:].T + b[d:]
    qs = np.float32(1.4426950408889634 / math.sqrt(m.head_dim))
    q = I.round_bf16((a[rows] @ w[:d].T + b[:d]).astype(np.float32) * qs).astype(np.float64)
    k = I.round_bf16(kv[:, :d].astype(np.float32)).astype(np.float64)
    v = I.round_bf16(kv[:, d:].astype(np.float32)).astype(np.float64)
    return dit.attention(q * (math.sqrt(m.head_dim) * math.log(2.0)), k, v, m.heads)


@pytest.mark.parametrize("mode", ["plain", "low", "first low", "rise", "rise, v"])
@pytest.mark.parametrize("name", list(SHAPES))
def test_scores_at_any_place(api, dev, name, mode):
    import torch
    kernel, split = SHAPES[name][4:]
    assert (attention_kernel(model(name), compute_units(dev)), attention_splits(model(name))) == (kernel, split)
    m, W, h, mod = _case(name, mode, 80)
    dm, ws = api.DeviceModel(W, dev), api.Workspace(m, 1, dev)
    dh = t(h[None], dev)
    say("attention range", name, mode, "N =", m.n_tok)
    api.dc_block_forward(dm, 0, t(mod, dev), dh, [0], ws)
    torch.cuda.synchronize()
    got = dh[0].cpu().numpy().astype(np.float64) - h
    assert np.isfinite(got).all()
    rng = np.random.default_rng(4)
    rows = np.unique(np.concatenate([[0, min(127, m.n_tok - 1), m.n_tok - 1], rng.integers(0, m.n_tok, 60)]))
    err = rel_l2(got[rows], _want(m, W, h, rows))
    say(name, mode, "rel-L2", err)
    # P and the output are rounded to bf16: 2^-9 each
    assert err < 5e-3


@pytest.mark.parametrize("name", ["hd64-N300-h30", "hd64-N2500-h30", "hd72-N2000-h16"])
def test_a_rise_costs_little(api, dev, name):
    """Rows whose maximum rises by 90 after the first tile take about as long as ordinary ones
    (redoing the work takes 1.4 to 2.2 times as long; ratios of the medians of 20 launches)."""
    import torch
    us = {}
    for mode in ("ordinary", "rise"):
        m, W, h, mod = _case(name, "rise", 81)
        if mode == "ordinary":
            h[:, 0] = 0.0
        dm, ws = api.DeviceModel(W, dev), api.Workspace(m, 1, dev)
        x, dmod = t(h[None], dev), t(mod, dev)
        dh = [x.clone() for _ in range(21)]
        say("attention time", name, mode)
        times = []
        for y in dh:
            with api.profile(["attention"]) as p:
                api.dc_block_forward(dm, 0, dmod, y, [0], ws)
                torch.cuda.synchronize()
            times.append(p.read()["attention"][1])
        us[mode] = 1e3 * float(np.median(times[1:]))
    say(name, "attention us", us)
    assert us["rise"] < 1.25 * us["ordinary"]
