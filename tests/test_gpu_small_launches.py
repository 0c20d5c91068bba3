"""GPU parity of the launches that carry more than one of a layer's small kernels, at the sizes where
their workgroups change hands, through one layer against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from mebp_inputs import ALL7, Config, layer_input, make_inputs
from paper_2510_03425_amd.device import DeviceModel

from gpu_util import TOL, rel_l2, say, to_np

pytestmark = pytest.mark.gpu


def _layer_errors(gpu, cfg, layer, seed):
    inp = make_inputs(cfg, seed=seed, norm="random")
    x, dy = layer_input(cfg, seed + 100)
    dm = DeviceModel(inp, device=str(gpu))
    tx, tdy = torch.from_numpy(x).to(gpu), torch.from_numpy(dy).to(gpu)
    ty, dx = torch.full_like(tx, float("nan")), torch.full_like(tx, float("nan"))
    dm.layer_forward(layer, tx, ty)
    dm.layer_backward(layer, tx, tdy, dx)
    torch.cuda.synchronize()
    P = O.decompress_layer(cfg, inp, layer)
    dx_ref, g_ref = O.layer_backward(cfg, layer, P, x, dy)
    errs = {"y": rel_l2(to_np(ty) - x, O.layer_forward(cfg, layer, P, x) - x), "dx": rel_l2(to_np(dx) - dy, dx_ref - dy)}
    for p, (dA, dB) in g_ref.items():
        errs["dA_" + p], errs["dB_" + p] = rel_l2(to_np(dm.dA[layer][p]), dA), rel_l2(to_np(dm.dB[layer][p]), dB)
    say("rel-L2", {k: f"{v:.2e}" for k, v in errs.items()})
    return errs


# attention backward with both halves in one launch (more than one key chunk and one query chunk,
# head dims 64 and 256): one row past a chunk, last chunks of few rows, one and several heads per
# KV head (1, 2, 7 planes per chunk), sliding windows shorter and longer than a chunk
ATTN_CASES = [
    # heads, kv heads, head dim, batch, tokens, window
    (1, 1, 64, 1, 129, 0),
    (7, 1, 64, 1, 257, 0),
    (4, 4, 64, 3, 200, 40),
    (2, 1, 256, 1, 193, 0),
    (2, 2, 256, 2, 330, 150),
]


@pytest.mark.parametrize("case", ATTN_CASES, ids=lambda c: f"h{c[0]}kv{c[1]}-dh{c[2]}-{c[3]}x{c[4]}-w{c[5]}")
def test_attention_backward_in_one_launch(built_lib, gpu, case):
    """Bound: as in every layer test (bf16 operands, 2^-9 a few times in a row); a plane left out or a
    row of the wrong chunk is an error of order one in some gradient."""
    h, kv, dh, b, t, window = case
    cfg = Config(name="attn", n_layers=1, hidden=128, n_heads=h, n_kv_heads=kv, head_dim=dh, ffn=192, vocab=0,
                 act="silu", lora_rank=8, lora_alpha=16.0, lora_modules=ALL7, batch=b, seq=t, window=window,
                 global_every=2 if window else 0)
    say("attention backward", case)
    errs = _layer_errors(gpu, cfg, 0, 21)
    assert max(errs.values()) <= TOL, errs


# a block's input norm with the adapters that read it (and the RoPE table) in one launch: one to
# eight 64-wide super-steps per wave (waves without any; a last one half full; the first width
# past the kernel), one row, one row past a workgroup, and one, two or none of the adapters
NORM_CASES = [
    # hidden, batch, tokens, modules, rank, arch
    (64, 1, 17, "all", 8, {}),
    (96, 1, 2, "all", 16, dict(qkv_bias=True)),
    (512, 3, 11, "qv", 8, dict(sandwich_norm=True)),
    (544, 1, 40, "kg", 16, {}),
    (1088, 1, 33, "all", 16, dict(qk_norm=True, qkv_bias=True)),
    (1568, 2, 16, "qvu", 8, {}),
    (2592, 1, 15, "all", 8, {}),
    (4096, 1, 18, "all", 16, dict(sandwich_norm=True)),
    (4160, 1, 18, "all", 8, {}),
    (320, 1, 70, "od", 8, dict(qkv_bias=True)),
]


@pytest.mark.parametrize("case", NORM_CASES, ids=lambda c: f"d{c[0]}-{c[1]}x{c[2]}-{c[3]}")
def test_norm_and_adapters_in_one_launch(built_lib, gpu, case):
    """Bound: as in every layer test; a wrong chunk of K or row is an error of order one."""
    d, b, t, mods, r, arch = case
    names = dict(q="q", k="k", v="v", o="o", g="gate", u="up", d="down")
    cfg = Config(name="norm", n_layers=1, hidden=d, n_heads=2, n_kv_heads=1, head_dim=64, ffn=192, vocab=0, act="silu",
                 lora_rank=r, lora_alpha=2.0 * r, lora_modules=ALL7 if mods == "all" else tuple(names[m] for m in mods),
                 batch=b, seq=t, **arch)
    say("norm and adapters", case)
    errs = _layer_errors(gpu, cfg, 0, 22)
    assert max(errs.values()) <= TOL, errs
