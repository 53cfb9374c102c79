"""The work a user of this framework has it do, as cases that can be timed and checked.

Each case is one pass through the public entry points of `paper_2608_16354_amd.api`:

  block       dc_block_forward: one transformer block in place on the residual stream of
              the selected scenes (a refresh step runs L of them);
  reuse       the device calls of a reuse step: dc_patch_embed, dc_drift_l1 (the check
              against the refresh input), dc_cache_apply, dc_head_euler;
  refresh     the device calls around the blocks of a refresh step: dc_patch_embed,
              dc_drift_l1 (snapshot), dc_cache_store, dc_head_euler;
  modulation  dc_time_modulation: the conditioning table of a whole sample;
  sample      api.Sampler: a whole cached sample (controller, schedule and device steps);
  calibrate   dc_calibrate_tables: the anchor calibration (trace, head, network tangents).

Shapes come from the framework's own workloads (the small fp32 model, the 12-, 30- and
42-block models) and, off those, from the ranges that the entry points take.
"""
import math

import numpy as np
import torch

from paper_2608_16354_amd import api
from paper_2608_16354_amd import inputs as I

DEV = "cuda:0"
EPS = 1e-6                      # LayerNorm epsilon and the drift denominator's epsilon
WEIGHT_STD = 0.02
N_FREQ = 256


def _case(name, kind, dtype, d, head_dim, latent, n_txt, **more):
    c = {"name": name, "kind": kind, "dtype": dtype, "d": d, "head_dim": head_dim, "mlp": 4 * d,
         "T": latent[0], "H": latent[1], "W": latent[2], "patch": 2, "n_txt": n_txt,
         "blocks": 1, "batch": 1, "K": 1, "h_max": 1, "guidance": 0.0}
    c.update(more)
    return c


def listed():
    full = (13, 60, 90)         # the latent of the 30- and 42-block models: 17,550 video tokens
    return [
        # A block of the small fp32 model (272 tokens): tests, smoke runs, the smallest calls.
        _case("block f32 272x256", "block", "f32", 256, 64, (4, 16, 16), 16),
        # The 30-block model's block on a short low-resolution clip, two scenes of 1,556 tokens:
        # a ragged length between the small model and the full clips.
        _case("block bf16 2x1556x1920", "block", "bf16", 1920, 64, (3, 34, 58), 77, batch=2),
        # The 12-block model's block (head_dim 72, 3,704 tokens): ordinary clips.
        _case("block bf16 3704x1152", "block", "bf16", 1152, 72, (8, 32, 56), 120),
        # The 30-block model's block at full length: the bulk of every refresh step.
        _case("block bf16 17776x1920", "block", "bf16", 1920, 64, full, 226),
        # The 42-block model's block at full length: the widest model and the longest single call.
        _case("block bf16 17776x3072", "block", "bf16", 3072, 64, full, 226),
        # A reuse step of the 12-block model: a handful of short memory-bound launches.
        _case("reuse bf16 3704x1152", "reuse", "bf16", 1152, 72, (8, 32, 56), 120),
        # A reuse step of the 30-block model: what half of its denoising steps consist of.
        _case("reuse bf16 17776x1920", "reuse", "bf16", 1920, 64, full, 226),
        # The calls around the blocks of a refresh step of the 42-block model (d = 3072).
        _case("refresh bf16 17776x3072", "refresh", "bf16", 3072, 64, full, 226),
        # The conditioning table of one 50-step sample of the 30-block model, computed whenever
        # a sampler is created (its size does not depend on the clip).
        _case("modulation 50x30x1920", "modulation", "bf16", 1920, 64, (1, 16, 16), 0, blocks=30, K=50,
              mlp=128),
        # A whole sample of the small fp32 model: latency, launches and the controller.
        _case("sample f32 272x256", "sample", "f32", 256, 64, (4, 16, 16), 16, blocks=2, K=10, h_max=2),
        # A whole 30-step sample of the 12-block model: 8 refresh and 22 reuse steps.
        _case("sample bf16 3704x1152", "sample", "bf16", 1152, 72, (8, 32, 56), 120, blocks=12, K=30,
              h_max=3),
        # Anchor calibration of the small fp32 model: once per model and anchor clip.
        _case("calibrate f32 272x256", "calibrate", "f32", 256, 64, (4, 16, 16), 16, blocks=2, K=10,
              h_max=2),
    ]


# ----------------------------------------------------------------------------
# more cases of the same ranges
# ----------------------------------------------------------------------------
def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _clip(rng, tokens, patch):
    """A latent (T, H, W) of about `tokens` video tokens, odd token counts among them."""
    t = min(13, _log_int(rng, 1, max(1, min(13, tokens // 16))))
    per = max(1, tokens // t)
    hp = max(1, int(round(math.sqrt(per / rng.uniform(1.2, 1.9)))))
    return t, patch * hp, patch * max(1, per // hp)


def _width(rng, lo, hi):
    """A model width and head_dim: multiples of 128 with head_dim 64, now and then head_dim 72."""
    if lo <= 1152 <= hi and rng.random() < 0.25:
        return (2304, 72) if hi >= 2304 and rng.random() < 0.3 else (1152, 72)
    return 128 * _log_int(rng, lo // 128, hi // 128), 64


def draw(rng):
    while True:
        kind = rng.choice(["block"] * 5 + ["reuse"] * 2 + ["refresh"] * 2 + ["modulation", "sample", "calibrate"])
        dtype = "f32" if rng.random() < 0.25 else "bf16"
        more, n_txt = {}, rng.choice([0, 7, 16, 77, 120, 226])
        if kind == "block":
            if dtype == "f32":
                d, hd, tokens = 128 * rng.randint(2, 6), 64, _log_int(rng, 48, 2400)
            else:
                (d, hd), tokens = _width(rng, 256, 3072), _log_int(rng, 64, 17550)
            if tokens < 6000:
                more["batch"] = rng.choice([1, 1, 2, 3])
        elif kind in ("reuse", "refresh"):
            if dtype == "f32":
                d, hd, tokens = 128 * rng.randint(2, 6), 64, _log_int(rng, 48, 2400)
            else:
                (d, hd), tokens = _width(rng, 256, 3072), _log_int(rng, 256, 17550)
            more["batch"] = rng.choice([1, 1, 2, 4] if tokens < 9000 else [1, 2])
        elif kind == "modulation":
            (d, hd), tokens, n_txt = _width(rng, 256, 3072), 64, 0
            more.update(blocks=rng.randint(2, min(42, 30 * 1920 ** 2 // d ** 2)), K=rng.randint(8, 100), mlp=128)
        elif kind == "sample":
            if dtype == "f32":
                d, hd, tokens = 128 * rng.randint(2, 4), 64, _log_int(rng, 48, 600)
                more.update(blocks=rng.randint(2, 4), K=rng.randint(6, 16))
            else:
                (d, hd), tokens = _width(rng, 256, 1152), _log_int(rng, 64, 3600)
                more.update(blocks=rng.randint(2, 12), K=rng.randint(8, 30))
            more.update(h_max=rng.randint(1, 3), batch=rng.choice([1, 1, 2]))
            if rng.random() < 0.25:
                more["guidance"] = 3.0
        else:
            d, hd, tokens = 128 * rng.randint(2, 4), 64, _log_int(rng, 48, 400)
            more.update(blocks=rng.randint(1, 3), K=rng.randint(4, 10), h_max=rng.randint(1, 2))
        patch = more["patch"] = rng.choice([1, 2, 2, 2, 4])
        latent = _clip(rng, tokens, patch) if kind != "modulation" else (1, 16, 16)
        if hd == 72:
            dtype = "bf16"          # fp32 models have head_dim 64
        c = _case("", kind, dtype, d, hd, latent, n_txt, **more)
        del c["name"]
        same_kind = [work(q) for q in listed() if q["kind"] == kind]
        w = work(c)
        if (w["flops"] <= max(q["flops"] for q in same_kind) and
                (kind == "modulation" or w["bytes"] <= max(q["bytes"] for q in same_kind))):
            return c


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------
def _shape(c):
    return I.ModelShape(c["blocks"], c["d"], c["d"] // c["head_dim"], c["head_dim"], c["mlp"],
                        64 // c["patch"] ** 2, c["T"], c["H"], c["W"], c["patch"], c["n_txt"], c["dtype"], EPS)


GLOBALS = {"block": (), "reuse": ("w_pe", "b_pe", "pos", "w_head", "b_head"),
           "modulation": ("w_t1", "b_t1", "w_t2", "b_t2", "w_m", "b_m", "head_mod")}
GLOBALS["refresh"] = GLOBALS["reuse"]
GLOBALS["sample"] = GLOBALS["calibrate"] = I.GLOBAL_TENSORS
BLOCKS = {"block": I.BLOCK_TENSORS[:-1], "reuse": (), "refresh": (), "modulation": ("mod_offset",),
          "sample": I.BLOCK_TENSORS, "calibrate": I.BLOCK_TENSORS}


class _Draws:
    """Seeded normal draws on the GPU, in the order they are asked for."""

    def __init__(self, seed):
        self.g = torch.Generator(DEV)
        self.g.manual_seed(seed)

    def __call__(self, *shape, std=1.0, bf16=False):
        a = torch.randn(shape, generator=self.g, device=DEV) * std
        return a.bfloat16().float() if bf16 else a


class _Weights:
    """Generator weights N(0, 0.02) (rounded to bf16 for bf16 models) of the tensors that the
    case's calls read; the others are zeros.  Serves api.DeviceModel as inputs.Weights does."""

    def __init__(self, c, rnd):
        self.m = _shape(c)
        self._g, self._b = I.tensor_shapes(self.m)
        bf = c["dtype"] == "bf16"
        self.g = {n: rnd(*self._g[n], std=WEIGHT_STD, bf16=bf) for n in GLOBALS[c["kind"]]}
        self.b = [{n: rnd(*self._b[n], std=WEIGHT_STD, bf16=bf) for n in BLOCKS[c["kind"]]}
                  for _ in range(c["blocks"])]
        self._zeros = {}

    def _zero(self, shape):
        return self._zeros.setdefault(shape, np.zeros(shape, np.float32))

    def get(self, name):
        return self.g[name].cpu().numpy() if name in self.g else self._zero(self._g[name])

    def block(self, l, name):
        return self.b[l][name].cpu().numpy() if name in self.b[l] else self._zero(self._b[name])


def _inputs(c, seed):
    """Every input of the case, float32 on the GPU."""
    rnd = _Draws(seed)
    W = _Weights(c, rnd)
    m, B, bf = W.m, c["batch"], c["dtype"] == "bf16"
    v = {"W": W, "m": m}
    if c["kind"] == "block":
        v["mod"] = rnd(6, m.hidden, std=0.1)
        v["h"] = rnd(B, m.n_tok, m.hidden)
        v["h"][:, : m.n_v] *= 0.16      # video rows: the scale of a patch-embedded latent
    elif c["kind"] in ("reuse", "refresh"):
        v["mod0"], v["head_mod"] = rnd(2, m.hidden, std=0.1), rnd(2, m.hidden, std=0.1)
        v["x"], v["txt"] = rnd(B, *m.latent_shape), rnd(B, m.n_txt, m.hidden, bf16=bf)
        if c["kind"] == "reuse":
            v["u_ref"] = rnd(B, m.n_v, m.hidden, bf16=bf)
            v["resid"] = rnd(B, m.n_v, m.hidden, std=0.3, bf16=bf)
        else:
            v["h_out"] = rnd(B, m.n_tok, m.hidden, std=0.5)
    elif c["kind"] in ("sample", "calibrate"):
        v["x"], v["txt"] = rnd(B, *m.latent_shape), rnd(B, m.n_txt, m.hidden, bf16=bf)
        if c["guidance"]:
            v["txt_null"] = rnd(B, m.n_txt, m.hidden, bf16=bf)
    return v


DSIGMA = -0.02


def _legal(c, b):
    """Scene b's legal reuse steps: runs of at most h_max between refreshes, staggered over the
    scenes.  With no response budget the schedule reuses at exactly these steps."""
    a = np.array([(k + b) % (c["h_max"] + 1) != 0 for k in range(c["K"])], np.uint8)
    a[0] = 0
    return a


def _problems(c, m):
    w = I.Workload(0, "case", m, c["batch"], c["K"], c["h_max"], None, "inf", 0.5, I.NO_VETO)
    return [I.scene_problem(w, I.Motion(6.0, 0.25)).replace(legal=_legal(c, b)) for b in range(c["batch"])]


def prepare(case, seed):
    c = case
    v = _inputs(c, seed)
    W, m, B = v["W"], v["m"], c["batch"]
    mdt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    s = {"case": c, "m": m, "dm": api.DeviceModel(W, DEV), "idx": list(range(B))}
    if c["kind"] not in ("sample", "calibrate"):
        s["ws"] = api.Workspace(m, B, DEV)
    if c["kind"] == "block":
        s.update(mod=v["mod"], h=v["h"])
    elif c["kind"] in ("reuse", "refresh"):
        s.update(mod0=v["mod0"], head_mod=v["head_mod"], x=v["x"], txt=v["txt"], cfg=api.model_cfg(m),
                 h_in=torch.zeros((B, m.n_tok, m.hidden), device=DEV))
        if c["kind"] == "reuse":
            s.update(u_ref=v["u_ref"].to(mdt), resid=v["resid"].to(mdt), g=torch.zeros_like(s["h_in"]),
                     sums=torch.zeros((B, 4), dtype=torch.float64, device=DEV))
        else:
            s.update(h_out=v["h_out"], u_ref=torch.zeros((B, m.n_v, m.hidden), dtype=mdt, device=DEV))
            s["resid"] = torch.zeros_like(s["u_ref"])
    elif c["kind"] == "modulation":
        s.update(sigmas=I.sigmas(c["K"])[: c["K"]],
                 mod=torch.zeros((c["K"], m.n_blocks + 1, 6, m.hidden), device=DEV))
    elif c["kind"] == "sample":
        s.update(x=v["x"], txt=v["txt"], sigmas=I.sigmas(c["K"]), problems=_problems(c, m),
                 bufs=api.SamplerBuffers(m, B, c["K"], DEV, branches=2 if c["guidance"] else 1))
        s["guidance"] = (c["guidance"], v["txt_null"]) if c["guidance"] else None
    else:
        s.update(x=v["x"][0], txt=v["txt"][0], sigmas=I.sigmas(c["K"]))
    return s


def run(s):
    c, kind = s["case"], s["case"]["kind"]
    if kind == "block":
        api.dc_block_forward(s["dm"], 0, s["mod"], s["h"], s["idx"], s["ws"])
        return {"h": s["h"]}
    if kind in ("reuse", "refresh"):
        api.dc_patch_embed(s["dm"], s["x"], s["txt"], s["h_in"], s["idx"], s["ws"])
        if kind == "reuse":
            api.dc_drift_l1(s["cfg"], s["h_in"], s["mod0"], s["u_ref"], 0, s["sums"], s["idx"], s["ws"])
            api.dc_cache_apply(s["cfg"], s["h_in"], s["resid"], s["g"], s["idx"])
            api.dc_head_euler(s["dm"], s["head_mod"], s["g"], s["x"], DSIGMA, s["idx"], s["ws"])
            return {"h_in": s["h_in"], "sums": s["sums"], "g": s["g"][:, : s["m"].n_v], "x": s["x"]}
        api.dc_drift_l1(s["cfg"], s["h_in"], s["mod0"], s["u_ref"], 1, None, s["idx"], s["ws"])
        api.dc_cache_store(s["cfg"], s["h_out"], s["h_in"], s["resid"], s["idx"])
        api.dc_head_euler(s["dm"], s["head_mod"], s["h_out"], s["x"], DSIGMA, s["idx"], s["ws"])
        return {"h_in": s["h_in"], "u_ref": s["u_ref"], "resid": s["resid"], "x": s["x"]}
    if kind == "modulation":
        api.dc_time_modulation(s["dm"], s["sigmas"], s["mod"], s["ws"])
        return {"mod": s["mod"]}
    if kind == "sample":
        smp = api.Sampler(s["dm"], s["problems"], s["sigmas"], s["x"], s["txt"], bufs=s["bufs"],
                          guidance=s["guidance"])
        realized, drift = smp.run()
        smp.close()
        return {"x": smp.x, "resid": s["bufs"].resid, "u_ref": s["bufs"].u_ref, "realized": realized,
                "drift": drift}
    q, d = api.dc_calibrate_tables(s["dm"], s["x"], s["txt"], s["sigmas"], c["h_max"], EPS)
    return {"q": q, "d": d}


# ----------------------------------------------------------------------------
# what a pass cannot do without, and what it may be off by
# ----------------------------------------------------------------------------
def _sizes(c):
    m = _shape(c)
    return m.n_tok, m.n_v, m.hidden, m.mlp_hidden, 2 if c["dtype"] == "bf16" else 4


def _block_work(c):
    N, _, d, F, e = _sizes(c)
    return {"bytes": e * (4 * d * d + 2 * d * F) + 8 * N * d * c["batch"],
            "flops": c["batch"] * (2 * N * (4 * d * d + 2 * d * F) + 4 * N * N * d)}


def _edge_work(c, kind):
    """Around the blocks: latent in and out, positions and text in, h_in out; a reuse reads the
    reference input and the cache and writes g, a refresh reads h_out and writes both."""
    N, Nv, d, _, e = _sizes(c)
    B = c["batch"]
    per = 2 * 64 * 4 * Nv + 4 * (N - Nv) * d + 4 * N * d + 2 * e * Nv * d + 4 * Nv * d
    return {"bytes": B * per + e * Nv * d + (4 + e) * 64 * d, "flops": B * 2 * 2 * Nv * 64 * d}


def _modulation_work(c):
    d, K = c["d"], c["K"]
    table = K * (c["blocks"] + 1) * 6 * d
    return {"bytes": 4 * (N_FREQ * d + 7 * d * d + (c["blocks"] + 1) * 6 * d + table),
            "flops": 2 * K * (N_FREQ * d + 7 * d * d) + table}


def _add(*parts):
    return {k: sum(n * p[k] for n, p in parts) for k in ("bytes", "flops")}


def work(case):
    c = case
    if c["kind"] == "block":
        return _block_work(c)
    if c["kind"] in ("reuse", "refresh"):
        return _edge_work(c, c["kind"])
    if c["kind"] == "modulation":
        return _modulation_work(c)
    branches = 2 if c["guidance"] else 1
    one = dict(c, batch=1)
    if c["kind"] == "sample":
        reuse = sum(int(_legal(c, b).sum()) for b in range(c["batch"]))
        refresh = c["batch"] * c["K"] - reuse
        return _add((1, _modulation_work(c)), (branches * refresh * c["blocks"], _block_work(one)),
                    (branches * (reuse + refresh), _edge_work(one, "reuse")))
    # calibrate: the trace, two head evaluations per table entry, and for each entry the network
    # and its tangent at every later step (twice the projections, three times the attention)
    K, N, d = c["K"], *(_sizes(c)[i] for i in (0, 2))
    entries = [(j, h) for j in range(1, K) for h in range(1, c["h_max"] + 1) if j + h <= K]
    tangents = sum(K - j - h for j, h in entries)
    net = _add((c["blocks"], _block_work(one)), (1, _edge_work(one, "refresh")))
    tan = {"bytes": 2 * net["bytes"], "flops": 2 * net["flops"] + c["blocks"] * 4 * N * N * d}
    return _add((1, _modulation_work(c)), (K, net), (2 * len(entries), _edge_work(one, "reuse")),
                (tangents, tan))


# About four times the distance from 64 bits that the path shows (the largest over its outputs).
TOLERANCE = {
    ("block", "f32"): 4e-7,         # 4e-8 to 1e-7: the update is a fraction of h
    ("block", "bf16"): 6e-3,        # up to 1.5e-3 at d = 3072
    ("reuse", "f32"): 6e-7,         # 1.5e-7
    ("reuse", "bf16"): 1.6e-4,      # 2e-6; x 4e-5 where LN rows are rounded to bf16 (d > 2048)
    ("refresh", "f32"): 4e-6,       # resid = h_out - h_in, 1e-6
    ("refresh", "bf16"): 7e-3,      # bf16 outputs: 1.7e-3
    ("modulation", "f32"): 4e-6, ("modulation", "bf16"): 4e-6,      # 1e-6
    ("sample", "f32"): 8e-6,        # resid 2e-6
    ("sample", "bf16"): 1.2e-2,     # resid 3e-3
    ("calibrate", "f32"): 2e-6,     # 3e-7 to 5e-7
    ("calibrate", "bf16"): 2e-3,    # 4e-4: the bf16 trace
}


def tolerance(case):
    return {"rel": TOLERANCE[case["kind"], case["dtype"]]}


# ----------------------------------------------------------------------------
# the same in 64 bits
# ----------------------------------------------------------------------------
def _silu(x):
    return x / (1 + torch.exp(-x))


def _gelu(z):
    return 0.5 * z * (1 + torch.tanh(math.sqrt(2 / math.pi) * (z + 0.044715 * z ** 3)))


def _ln_mod(x, shift, scale):
    xc = x - x.mean(-1, keepdim=True)
    return xc / torch.sqrt((xc * xc).mean(-1, keepdim=True) + EPS) * (1 + scale) + shift


def _sigmas(K):
    return np.array([1.0 - k / K for k in range(K + 1)])


class _Net:
    """The generator in float64 (weights [out, in], y = x W^T + b)."""

    def __init__(self, W):
        self.m = W.m
        self.g = {n: a.double() for n, a in W.g.items()}
        self.b = [{n: a.double() for n, a in b.items()} for b in W.b]

    def attention(self, q, k, v):
        m, out = self.m, []
        for i in range(m.heads):
            sl = slice(i * m.head_dim, (i + 1) * m.head_dim)
            kt, vh = k[:, sl].T.contiguous(), v[:, sl].contiguous()
            out.append(torch.cat([torch.softmax(qq @ kt / math.sqrt(m.head_dim), -1) @ vh
                                  for qq in q[:, sl].split(4096)]))
        return torch.cat(out, 1)

    def block(self, l, mod, h):
        b, d = self.b[l], self.m.hidden
        qkv = _ln_mod(h, mod[0], mod[1]) @ b["w_qkv"].T + b["b_qkv"]
        o = self.attention(qkv[:, :d], qkv[:, d: 2 * d], qkv[:, 2 * d:])
        h = h + mod[2] * (o @ b["w_o"].T + b["b_o"])
        z = _gelu(_ln_mod(h, mod[3], mod[4]) @ b["w_1"].T + b["b_1"])
        return h + mod[5] * (z @ b["w_2"].T + b["b_2"])

    def blocks(self, mods, h):
        for l in range(self.m.n_blocks):
            h = self.block(l, mods[l], h)
        return h

    def patches(self, x):
        m, p = self.m, self.m.patch
        y = x.reshape(m.lat_c, m.lat_t, m.hp, p, m.wp, p).permute(1, 2, 4, 0, 3, 5)
        return y.reshape(m.n_v, m.patch_dim)

    def embed(self, x, txt):
        return torch.cat([self.patches(x) @ self.g["w_pe"].T + self.g["b_pe"] + self.g["pos"], txt])

    def head(self, head_mod, g):
        m, p = self.m, self.m.patch
        tok = _ln_mod(g, head_mod[0], head_mod[1]) @ self.g["w_head"].T + self.g["b_head"]
        y = tok.reshape(m.lat_t, m.hp, m.wp, m.lat_c, p, p).permute(3, 0, 1, 4, 2, 5)
        return y.reshape(m.latent_shape)

    def modulation(self, sigmas):
        """[K, L + 1, 6, d]."""
        m, g = self.m, self.g
        t = 1000 * torch.tensor(np.asarray(sigmas), device=DEV)[:, None]
        i = torch.arange(N_FREQ // 2, dtype=torch.float64, device=DEV)
        arg = t * 10000.0 ** (-i / (N_FREQ // 2))
        e = torch.cat([torch.cos(arg), torch.sin(arg)], 1)
        cond = _silu(e @ g["w_t1"].T + g["b_t1"]) @ g["w_t2"].T + g["b_t2"]
        shared = (_silu(cond) @ g["w_m"].T + g["b_m"]).reshape(-1, 6, m.hidden)
        head = torch.zeros_like(shared)
        head[:, :2] = g["head_mod"] + cond[:, None]
        return torch.stack([shared + b["mod_offset"] for b in self.b] + [head], 1)

    def velocity(self, mods, x, txt):
        """The uncached denoiser output, with what the cache keeps of it."""
        h_in = self.embed(x, txt)
        h = self.blocks(mods, h_in)[: self.m.n_v]
        return self.head(mods[self.m.n_blocks, :2], h), _ln_mod(h_in[: self.m.n_v], *mods[0, :2]), \
            h - h_in[: self.m.n_v]


def _exact_sample(c, v, net):
    m, K, B = net.m, c["K"], c["batch"]
    sig = _sigmas(K)
    mods = net.modulation(sig[:K])
    txts = [v["txt"].double()] + ([v["txt_null"].double()] if c["guidance"] else [])
    xs, resid, u_refs = [], [[None] * B for _ in txts], []
    realized = np.zeros((K, B), np.uint8)
    drift = np.full((K, B), np.nan)
    for b in range(B):
        x, legal, u_ref = v["x"][b].double(), _legal(c, b), None
        for k in range(K):
            mk, vel = mods[k], []
            for i, txt in enumerate(txts):
                h_in = net.embed(x, txt[b])
                hv = h_in[: m.n_v]
                u = _ln_mod(hv, mk[0, 0], mk[0, 1]) if i == 0 else u
                if legal[k]:
                    g = hv + resid[i][b]
                else:
                    g = net.blocks(mk, h_in)[: m.n_v]
                    resid[i][b] = g - hv
                vel.append(net.head(mk[m.n_blocks, :2], g))
            if legal[k]:
                drift[k, b] = float((u - u_ref).abs().sum() / (u.abs().sum() + EPS))
                realized[k, b] = 1
            else:
                u_ref = u
            step = vel[0] if len(vel) == 1 else vel[1] + c["guidance"] * (vel[0] - vel[1])
            x = x + (sig[k + 1] - sig[k]) * step
        xs.append(x)
        u_refs.append(u_ref)
    return {"x": torch.stack(xs), "resid": torch.stack([r for branch in resid for r in branch]),
            "u_ref": torch.stack(u_refs), "realized": realized, "drift": drift}


def _exact_calibrate(c, v, net):
    m, K = net.m, c["K"]
    sig, txt = _sigmas(K), v["txt"][0].double()
    mods = net.modulation(sig[:K])
    xs, us, rs, x = [], [], [], v["x"][0].double()
    for k in range(K):
        vel, u, r = net.velocity(mods[k], x, txt)
        xs.append(x)
        us.append(u)
        rs.append(r)
        x = x + (sig[k + 1] - sig[k]) * vel
    xn = float(x.norm()) + EPS
    q, d = np.zeros((K - 1, c["h_max"])), np.zeros((K - 1, c["h_max"]))
    for j in range(K - 1):
        G = torch.zeros_like(x)
        for h in range(1, c["h_max"] + 1):
            t = j + h
            if t >= K:
                break
            d[j, h - 1] = float((us[t] - us[j]).norm() / (us[t].norm() + EPS))
            hv, hm = net.embed(xs[t], txt)[: m.n_v], mods[t, m.n_blocks, :2]
            dx = (sig[t + 1] - sig[t]) * (net.head(hm, hv + rs[j]) - net.head(hm, hv + rs[t]))
            for k in range(t + 1, K):
                dv = torch.func.jvp(lambda y: net.velocity(mods[k], y, txt)[0], (xs[k],), (dx,))[1]
                dx = dx + (sig[k + 1] - sig[k]) * dv
            G = G + dx
            q[j, h - 1] = float(G.norm()) / xn
    return {"q": q, "d": d}


def exact(case, seed):
    c = case
    v = _inputs(c, seed)
    net, m, B = _Net(v["W"]), v["m"], c["batch"]
    if c["kind"] == "block":
        return {"h": torch.stack([net.block(0, v["mod"].double(), v["h"][b].double()) for b in range(B)])}
    if c["kind"] == "modulation":
        return {"mod": net.modulation(_sigmas(c["K"])[: c["K"]])}
    if c["kind"] == "sample":
        return _exact_sample(c, v, net)
    if c["kind"] == "calibrate":
        return _exact_calibrate(c, v, net)
    out = []
    mod0, hm = v["mod0"].double(), v["head_mod"].double()
    for b in range(B):
        x = v["x"][b].double()
        h_in = net.embed(x, v["txt"][b].double())
        hv = h_in[: m.n_v]
        u = _ln_mod(hv, mod0[0], mod0[1])
        if c["kind"] == "reuse":
            r, w = v["u_ref"][b].double(), hv + v["resid"][b].double()
            sums = torch.stack([(u - r).abs().sum(), u.abs().sum(), (u - r).square().sum(), u.square().sum()])
            out.append({"h_in": h_in, "sums": sums, "g": w, "x": x + DSIGMA * net.head(hm, w)})
        else:
            w = v["h_out"][b, : m.n_v].double()
            out.append({"h_in": h_in, "u_ref": u, "resid": w - hv, "x": x + DSIGMA * net.head(hm, w)})
    return {k: torch.stack([o[k] for o in out]) for k in out[0]}
