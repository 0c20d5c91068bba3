"""The adapters' terms of the products, s u B^T forward and du A backward, carry fp32 bits.

With all base weights zero the fp32 outputs of a layer's products are these terms alone, of the u
and du that the workspace keeps: the O product's h, the down product's output, and the gradients of
the two normalised inputs (where the product is not split over planes; the planes' sum leaves the
gradient in registers).

Bound: sums of up to 48 products of fp32 values in fp32, about 1e-7 of the result (2^-24 a rounding,
random signs); 16 bits in either factor give 2^-17 and more, 4e-6. 1e-6 lies between. From 160
tiles of 256 x 128 and 1024 tokens on the factors have two bf16 parts (2^-17 each): 1e-5.
"""
import numpy as np
import pytest
import torch

import oracle as O
from mebp_inputs import ALL7, PROJ, Config, layer_input, make_inputs
from paper_2510_03425_amd import _lib as L
from paper_2510_03425_amd.device import DeviceModel, slot_index

from gpu_util import TOL, rel_l2, say, to_np

pytestmark = pytest.mark.gpu

# hidden, heads, head dim, ffn, batch, tokens, rank: tiles of 32 .. 128 rows, one and four waves side
# by side, up to eight ranges of the reduction inside a workgroup
CASES = [
    (64, 1, 64, 192, 1, 33, 8),
    (320, 2, 128, 1152, 1, 129, 16),
    (896, 14, 64, 4864, 1, 256, 8),
    (896, 14, 64, 4864, 3, 333, 16),
    (576, 3, 256, 3008, 1, 515, 16),
    (2560, 8, 256, 2048, 1, 640, 16),
    (2560, 8, 256, 2048, 3, 611, 16),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"d{c[0]}-f{c[3]}-{c[4]}x{c[5]}-r{c[6]}")
def test_lora_terms_keep_fp32(built_lib, gpu, case):
    d, h, dh, f, b, t, r = case
    cfg = Config(name="term", n_layers=1, hidden=d, n_heads=h, n_kv_heads=1, head_dim=dh, ffn=f, vocab=0, act="silu",
                 lora_rank=r, lora_alpha=2.0 * r, lora_modules=ALL7, batch=b, seq=t)
    inp = make_inputs(cfg, seed=8, norm="random")
    for p in PROJ:
        q4, sb = inp.base[0][p]
        inp.base[0][p] = (q4, np.zeros_like(sb))
        A, B = inp.lora[0][p]
        B[:] = np.random.default_rng(PROJ.index(p)).standard_normal(B.shape) * 0.1
    x, dy = layer_input(cfg, 14)
    x = (x * 1e-3).astype(np.float32)  # (so that x is small beside the terms that are added to it)
    # (a vocabulary sizes the workspace so that the transposed products read their weights' bf16 copy)
    inp.cfg = cfg.with_(vocab=262144)
    dm = DeviceModel(inp, device=str(gpu))
    dm.ws.fill_(255)  # NaNs
    tx, tdy = torch.from_numpy(x).to(gpu), torch.from_numpy(dy).to(gpu)
    y, dx = torch.empty_like(tx), torch.empty_like(tx)
    N, view = dm.N, lambda name, shape: dm.ws_view(slot_index(name), torch.float32, shape).double()
    A, B = ({p: torch.from_numpy(inp.lora[0][p][i]).to(gpu).double() for p in PROJ} for i in (0, 1))

    two = N >= 1024 and -(-N // 256) * -(-d // 128) >= 160  # (every product below has d columns)

    def close(what, got, ref):
        err = float((got - ref).norm() / ref.norm())
        say(what, f"{err:.2e}")
        assert err <= (1e-5 if two else 1e-6), (what, err)

    say("LoRA terms", case)
    dm.layer_forward(0, tx, y)
    torch.cuda.synchronize()
    u = dict(zip(PROJ, view("lora_u", (len(PROJ), N, r))))
    hh = view("h", (N, d))
    close("o", hh - tx.double(), 2 * u["o"] @ B["o"].t())
    close("down", y.double() - hh, 2 * u["down"] @ B["down"].t())
    dm.ws.fill_(255)
    dm.layer_backward(0, tx, tdy, dx)
    torch.cuda.synchronize()
    du = dict(zip(PROJ, view("lora_du", (len(PROJ), N, r))))
    seen = 0
    for name, ps in (("dc", ("gate", "up")), ("da", ("q", "k", "v"))):
        got = view(name, (N, d))
        if not torch.isnan(got).all():
            close(name, got, sum(du[p] @ A[p] for p in ps))
            seen += 1
    say("gradients seen", seen)


def test_outer_products_in_less_scratch_than_planned(built_lib, gpu):
    """The gate / up launch of dB and dA plans 12 token splits here and the workspace has room for 9.
    Bound: bf16 operands, as in every layer test; the last tokens weigh 40 times the others, so that a
    split left out is an error of order one."""
    b, t, d, f, r = 13, 500, 64, 6912, 8
    cfg = Config(name="outer", n_layers=1, hidden=d, n_heads=1, n_kv_heads=1, head_dim=64, ffn=f, vocab=0, act="silu",
                 lora_rank=r, lora_alpha=2.0 * r, lora_modules=ALL7, batch=b, seq=t)
    inp = make_inputs(cfg, seed=9, norm="random")
    x, dy = layer_input(cfg, 16)
    dy[-3:] *= 40
    dm = DeviceModel(inp, device=str(gpu))
    lo, hi = (L.mebp_workspace_offset(dm.ccfg, b, t, slot_index(n)) for n in ("lora_part", "rope_global"))
    assert (hi - lo) // (2 * (d + f) * r * 4) == 9
    tx, tdy = torch.from_numpy(x).to(gpu), torch.from_numpy(dy).to(gpu)
    dx = torch.full_like(tx, float("nan"))
    say("outer products in less scratch")
    dm.layer_backward(0, tx, tdy, dx)
    torch.cuda.synchronize()
    dx_ref, g_ref = O.layer_backward(cfg, 0, O.decompress_layer(cfg, inp, 0), x, dy)
    errs = {"dx": rel_l2(to_np(dx) - dy, dx_ref - dy)}
    for p, (dA, dB) in g_ref.items():
        errs["dA_" + p], errs["dB_" + p] = rel_l2(to_np(dm.dA[0][p]), dA), rel_l2(to_np(dm.dB[0][p]), dB)
    say("rel-L2", {k: f"{v:.2e}" for k, v in errs.items()})
    assert max(errs.values()) <= TOL, errs
