"""GPU parity of the tile configurations of the forward and the transposed products (gemm_mid.hip)
at the sizes where they can go wrong, through one layer against the fp64 oracle: a single reduction step
(more K ranges than steps), odd step counts, token and column counts that are no multiple of a
tile, every tile shape that the cost model picks, RoPE over head dims 64 / 128 / 256 and
positions that wrap inside a tile.

Bound: the branch (x_out - x_in) is a sum of products of fp16 operands (relative rounding 2^-11
each, a few in a row: norm, q / k / v, O, z) accumulated in fp32, so its rel-L2 error stays below
a few 1e-3; a wrong row, column, step or head is an error of order one in some row.
"""
import numpy as np
import pytest
import torch

import oracle as O
from mebp_inputs import ALL7, Config, layer_input, make_inputs
from paper_2510_03425_amd.device import DeviceModel

from gpu_util import ROW_TOL, TOL, max_row_rel_l2, rel_l2, say, to_np

pytestmark = pytest.mark.gpu

# hidden, heads, kv heads, head dim, ffn, batch, tokens, act, rank
CASES = [
    (64, 1, 1, 64, 192, 1, 33, "silu", 8),        # one K step
    (192, 3, 1, 64, 448, 2, 49, "gelu_tanh", 16),  # three and seven steps, positions wrap in a tile
    (320, 2, 1, 128, 4864, 1, 129, "silu", 16),    # five steps; 129 = one row past a tile
    (576, 3, 1, 256, 3008, 2, 515, "gelu_tanh", 8),  # nine and 47 steps, the widest tile
    (896, 14, 2, 64, 1728, 1, 255, "silu", 8),     # fourteen steps, one row short of a tile
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"d{c[0]}-dh{c[3]}-f{c[4]}-{c[5]}x{c[6]}")
def test_layer_forward_tiles(built_lib, gpu, case):
    d, h, kv, dh, f, b, t, act, r = case
    cfg = Config(name="mid", n_layers=1, hidden=d, n_heads=h, n_kv_heads=kv, head_dim=dh, ffn=f, vocab=0, act=act,
                 lora_rank=r, lora_alpha=2.0 * r, lora_modules=ALL7, batch=b, seq=t)
    inp = make_inputs(cfg, seed=3, norm="random")
    x, _ = layer_input(cfg, 11)
    dm = DeviceModel(inp, device=str(gpu))
    xi = torch.from_numpy(x).to(gpu)
    xo = torch.full_like(xi, float("nan"))
    say("forward tiles", case)
    dm.layer_forward(0, xi, xo)
    torch.cuda.synchronize()
    got = xo.double().cpu().numpy() - x
    ref = O.layer_forward(cfg, 0, O.decompress_layer(cfg, inp, 0), x) - x
    err, row = rel_l2(got, ref), max_row_rel_l2(got, ref)
    say("rel-L2", err, "worst row", row)
    assert err <= 5e-3 and row <= ROW_TOL


# the transposed products reduce over the output features: widths that are no multiple of the
# 64-row step (ffn 688, 208), of the 64-column blocks (hidden 96, 320), one to several segments,
# splits over the grid (long reductions at few tokens) and every tile shape of the plan
BWD_CASES = CASES + [
    (96, 1, 1, 64, 688, 1, 70, "silu", 16),
    (128, 4, 2, 64, 208, 1, 200, "gelu_tanh", 8),
    (256, 2, 1, 128, 6912, 1, 300, "silu", 8),
]


@pytest.mark.parametrize("case", BWD_CASES, ids=lambda c: f"d{c[0]}-dh{c[3]}-f{c[4]}-{c[5]}x{c[6]}")
def test_layer_backward_tiles(built_lib, gpu, case):
    """Bound: gradients are products of bf16 operands (relative rounding 2^-9, three to six in a
    row), 2e-2 as everywhere in these tests; a wrong tile is an error of order one."""
    d, h, kv, dh, f, b, t, act, r = case
    cfg = Config(name="mid", n_layers=1, hidden=d, n_heads=h, n_kv_heads=kv, head_dim=dh, ffn=f, vocab=0, act=act,
                 lora_rank=r, lora_alpha=2.0 * r, lora_modules=ALL7, batch=b, seq=t)
    inp = make_inputs(cfg, seed=4, norm="random")
    x, dy = layer_input(cfg, 12)
    dm = DeviceModel(inp, device=str(gpu))
    tx, tdy = torch.from_numpy(x).to(gpu), torch.from_numpy(dy).to(gpu)
    dx = torch.full_like(tx, float("nan"))
    say("backward tiles", case)
    dm.layer_backward(0, tx, tdy, dx)
    torch.cuda.synchronize()
    dx_ref, g_ref = O.layer_backward(cfg, 0, O.decompress_layer(cfg, inp, 0), x, dy)
    errs = {"dx": rel_l2(to_np(dx) - dy, dx_ref - dy)}
    for p, (dA, dB) in g_ref.items():
        errs["dA_" + p], errs["dB_" + p] = rel_l2(to_np(dm.dA[0][p]), dA), rel_l2(to_np(dm.dB[0][p]), dB)
    row = max_row_rel_l2(to_np(dx) - dy, dx_ref - dy)
    say("rel-L2", {k: f"{v:.2e}" for k, v in errs.items()}, "worst row", row)
    assert max(errs.values()) <= TOL, errs
    assert row <= 2 * ROW_TOL  # (without the residual dy, which the other row checks include)


# LoRA kernels over the token counts where their launch changes shape: rows of 16, 32 and 64 per
# workgroup; outer products by waves over the tokens, over the grid as well (from 2049 tokens on)
# and side by side with a shared u (from 4097 on), with token counts off every step and a rank
# below the tile's 16.
LORA_CASES = [(1, 15, 8), (1, 193, 16), (3, 683, 8), (4, 1023, 16), (3, 1366, 16), (9, 911, 16), (33, 497, 8)]


@pytest.mark.parametrize("case", LORA_CASES, ids=lambda c: f"{c[0]}x{c[1]}-r{c[2]}")
def test_layer_lora_token_counts(built_lib, gpu, case):
    """Same bound as the tiles; a token left out or counted twice changes a gradient of N random
    tokens by 1 / sqrt(N) of its size, so the last tokens are given 40 times the weight."""
    b, t, r = case
    cfg = Config(name="lora", n_layers=1, hidden=64, n_heads=1, n_kv_heads=1, head_dim=64, ffn=192, vocab=0,
                 act="silu", lora_rank=r, lora_alpha=2.0 * r, lora_modules=ALL7, batch=b, seq=t)
    inp = make_inputs(cfg, seed=5, norm="random")
    x, dy = layer_input(cfg, 13)
    dy[-3:] *= 40
    dm = DeviceModel(inp, device=str(gpu))
    tx, tdy = torch.from_numpy(x).to(gpu), torch.from_numpy(dy).to(gpu)
    dx = torch.full_like(tx, float("nan"))
    say("lora token counts", case)
    dm.layer_backward(0, tx, tdy, dx)
    torch.cuda.synchronize()
    dx_ref, g_ref = O.layer_backward(cfg, 0, O.decompress_layer(cfg, inp, 0), x, dy)
    errs = {"dx": rel_l2(to_np(dx) - dy, dx_ref - dy)}
    for p, (dA, dB) in g_ref.items():
        errs["dA_" + p], errs["dB_" + p] = rel_l2(to_np(dm.dA[0][p]), dA), rel_l2(to_np(dm.dB[0][p]), dB)
    say("rel-L2", {k: f"{v:.2e}" for k, v in errs.items()})
    assert max(errs.values()) <= TOL, errs
