"""Scales of the compressed weights at addresses that are a multiple of 2 and not of 4, which every
entry point takes: the products that load scales 16 bytes at a time leave them to the kernels that
load them one by one, and the results meet the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from mebp_inputs import ALL7, PROJ, Config, layer_input, make_inputs
from paper_2510_03425_amd import _lib as L
from paper_2510_03425_amd.device import DeviceModel

from gpu_util import TOL, rel_l2, say, to_np

pytestmark = pytest.mark.gpu


def _odd(dm, scale_bits):
    n = scale_bits.size
    t = torch.zeros(n + 3, dtype=torch.int16, device=dm.device)
    first = 1 + t.data_ptr() % 4 // 2
    t[first:first + n] = torch.from_numpy(np.ascontiguousarray(scale_bits).view(np.int16).reshape(-1)).to(dm.device)
    dm.keep.append(t)
    assert t[first:].data_ptr() % 4 == 2
    return t[first:].data_ptr()


def _timed(run):
    L.mebp_kernel_timing(True, 1 << 10)
    try:
        run()
        torch.cuda.synchronize()
        return {k["kernel"] for k in L.mebp_kernel_timing_report()}
    finally:
        L.mebp_kernel_timing(False)


# reductions that are a multiple of 64 (hidden, heads, ffn all are) at few and at many tokens
@pytest.mark.parametrize("batch,seq", [(1, 100), (3, 400)])
def test_odd_scale_addresses(built_lib, gpu, batch, seq):
    cfg = Config(name="odd", n_layers=1, hidden=320, n_heads=4, n_kv_heads=2, head_dim=64, ffn=448, vocab=4160,
                 act="silu", lora_rank=16, lora_alpha=32.0, lora_modules=ALL7, batch=batch, seq=seq)
    inp = make_inputs(cfg, seed=12, norm="random")
    x, dy = layer_input(cfg, 15)
    dm = DeviceModel(inp, device=str(gpu))
    tx, tdy = torch.from_numpy(x).to(gpu), torch.from_numpy(dy).to(gpu)
    y, dx, dxl = (torch.full_like(tx, float("nan")) for _ in range(3))
    aligned = _timed(lambda: dm.layer_forward(0, tx, y))
    for i, p in enumerate(PROJ):
        dm.base[0].w[i].scale = _odd(dm, inp.base[0][p][1])
    dm.emb.scale = _odd(dm, inp.emb[1])
    y.fill_(float("nan"))
    say("odd scale addresses", batch, seq)
    odd = _timed(lambda: dm.layer_forward(0, tx, y))
    # the fused product leaves neither a RoPE launch nor a sum of planes behind; the others do
    say("launches with aligned scales", sorted(aligned), "with odd ones", sorted(odd))
    assert not aligned & {"rope_fwd", "splitk_finalize_rope"} and odd & {"rope_fwd", "splitk_finalize_rope"}
    dm.layer_backward(0, tx, tdy, dx)
    torch.cuda.synchronize()
    P = O.decompress_layer(cfg, inp, 0)
    dx_ref, g_ref = O.layer_backward(cfg, 0, P, x, dy)
    errs = {"y": rel_l2(to_np(y) - x, O.layer_forward(cfg, 0, P, x) - x), "dx": rel_l2(to_np(dx) - dy, dx_ref - dy)}
    for p, (dA, dB) in g_ref.items():
        errs["dA_" + p], errs["dB_" + p] = rel_l2(to_np(dm.dA[0][p]), dA), rel_l2(to_np(dm.dB[0][p]), dB)
    dm.lm_head(tx, dxl)
    torch.cuda.synchronize()
    loss, dxl_ref = O.lm_head_ce(cfg, O.decompress_embedding(cfg, inp), inp.norm_final, x, inp.ids)
    errs["lm_dx"] = rel_l2(to_np(dxl), dxl_ref)
    say("rel-L2", {k: f"{v:.2e}" for k, v in errs.items()}, "loss", dm.loss.item(), loss)
    assert max(errs.values()) <= TOL, errs
    assert abs(dm.loss.item() - loss) <= 1e-3 * abs(loss)
