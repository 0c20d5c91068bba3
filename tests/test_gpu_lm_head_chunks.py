"""GPU parity of the LM head where the last vocabulary chunk is narrower than the others and its dH
product is split into more planes than theirs, under workspace guards."""
import numpy as np
import pytest
import torch

import oracle as O
from mebp_inputs import MINI, make_inputs
from paper_2510_03425_amd import _lib as L
from paper_2510_03425_amd.device import DeviceModel

from gpu_util import TOL, rel_l2, say
from test_lm_head_planes_host import check

pytestmark = pytest.mark.gpu


def test_narrow_last_chunk(built_lib, gpu):
    """Bound: dx as everywhere (bf16 probabilities, fp16 logits); the loss is a mean of fp32 terms
    whose logits have fp16 operands, 1e-3 as in the other LM head tests."""
    hidden, vocab, B, T = 128, 50304, 80, 128
    assert check(hidden, vocab, B, T)
    cfg = MINI.with_(name="chunks", n_layers=1, hidden=hidden, n_heads=1, n_kv_heads=1, head_dim=128, ffn=192,
                     vocab=vocab, batch=B, seq=T)
    inp = make_inputs(cfg, seed=6, norm="random")
    # logits with a standard deviation of about 4: the softmax part of the gradient is then of the
    # size of the target's, and a plane left out or overwritten is an error of order one
    inp.norm_final = (np.asarray(inp.norm_final) * (4 / (0.02 * hidden**0.5))).astype(np.float32)
    gen = torch.Generator().manual_seed(1)
    x = torch.randn((B * T, hidden), generator=gen)
    prev = L.mebp_set_workspace_guards(True)
    try:
        dm = DeviceModel(inp, device=str(gpu))
        tx = x.to(gpu)
        dx = torch.full_like(tx, float("nan"))
        say("LM head, narrow last chunk", hidden, vocab, B, T, "ws bytes", dm.ws_bytes)
        dm.lm_head(tx, dx)
        torch.cuda.synchronize()
    finally:
        L.mebp_set_workspace_guards(prev)
    # the same in 64 bits, some sequences at a time
    E = torch.from_numpy(O.dequant(*inp.emb, hidden, 32).astype(np.float64)).to(gpu)
    w = torch.from_numpy(np.asarray(inp.norm_final, np.float64)).to(gpu)
    ids = torch.from_numpy(np.asarray(inp.ids)).long().to(gpu)
    n, loss, ref = B * (T - 1), 0.0, torch.zeros((B, T, hidden), dtype=torch.float64, device=gpu)
    for b in range(0, B, 8):
        xb = tx.view(B, T, hidden)[b:b + 8].double().requires_grad_()
        hf = xb * torch.rsqrt(xb.square().mean(-1, keepdim=True) + cfg.rms_eps) * w
        lg = hf[:, :-1].reshape(-1, hidden) @ E.t()
        part = torch.nn.functional.cross_entropy(lg, ids[b:b + 8, 1:].reshape(-1), reduction="sum") / n
        ref[b:b + 8] = torch.autograd.grad(part, xb)[0]
        loss += part.item()
    err = rel_l2(dx.cpu().numpy(), ref.view(-1, hidden).cpu().numpy())
    say("loss", dm.loss.item(), loss, "dx rel-L2", err)
    assert abs(dm.loss.item() - loss) <= 1e-3 * abs(loss)
    assert err <= TOL
