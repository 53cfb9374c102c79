"""Helpers for the GPU parity tests (shared seeded inputs, error metrics)."""
import sys

import numpy as np

from paper_2608_16354_amd import inputs as I


def say(*a):
    """Name the case before a GPU step, flushed (a faulting kernel can end the process)."""
    print("[gpu]", *a, flush=True)
    sys.stdout.flush()


def rel_l2(a, b):
    a = np.asarray(a, np.float64)
    b = np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def t(a, dev, dtype=None):
    import torch
    x = torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    return x if dtype is None else x.to(dtype)


def mod_input(m, key, std=0.1):
    """A seeded [6, d] modulation vector set (shift1, scale1, gate1, shift2, scale2, gate2)."""
    return I.normal((6, m.hidden), std, (7000,) + tuple(key))


def compute_units(dev):
    import torch
    return torch.cuda.get_device_properties(dev).multi_processor_count


TILES = ("384x192", "320x256", "256x192", "256x128", "128x128", "64x64")
ATTENTION = ("k_attn_keys", "k_attn_bf16", "k_attn16")


def _native(symbol, *args):
    import ctypes
    from paper_2608_16354_amd import _lib
    f = getattr(_lib.load(), symbol)
    f.restype = ctypes.c_int
    return f(*args)


def block_tiles(m, cus):
    """The library's own choice: the tiles of a block's QKV, out-projection, MLP-up and MLP-down GEMM."""
    d, F = m.hidden, m.mlp_hidden
    return tuple(TILES[_native("_ZN2dc15block_gemm_tileEiiii", m.n_tok, n, k, cus)]
                 for n, k in ((3 * d, d), (d, d), (F, d), (d, F)))


def attention_kernel(m, cus):
    """The library's own choice of the bf16 attention kernel."""
    return ATTENTION[_native("_ZN2dc16attention_kernelEiiii", m.head_dim, m.heads, m.n_tok, cus)]


def attention_splits(m):
    """Whether that kernel splits the items of its last round on the current device."""
    return bool(_native("_ZN2dc16attention_splitsEiii", m.head_dim, m.heads, m.n_tok) & 1)
