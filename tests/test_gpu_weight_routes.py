"""The three ways in which a layer's transposed products get their weights, chosen by the memory that
a call has: a bf16 copy of the whole layer in operand order, one of a product at a time, or the int4
weights themselves. Each is seen by its launches, meets the oracle, and is the same, bit for bit, in
the call that uses the library's own buffer."""
import pytest
import torch

import oracle as O
from mebp_inputs import ALL7, CONFIGS, Config, layer_input, make_inputs
from paper_2510_03425_amd import _lib as L
from paper_2510_03425_amd.device import DeviceModel, ptr, stream_handle

from gpu_util import TOL, rel_l2, say, to_np
from test_gpu_gemm_mid import BWD_CASES

pytestmark = pytest.mark.gpu


def _model(cfg, seed, gpu):
    """A layer of a model whose vocabulary sizes the workspace, without drawing its embedding."""
    inp = make_inputs(cfg.with_(vocab=0), seed=seed, norm="random", n_layers=1)
    inp.cfg = cfg
    return inp, DeviceModel(inp, device=str(gpu))


def _copies(run):
    """Launches that write bf16 weights in `run`."""
    L.mebp_kernel_timing(True, 1 << 10)
    try:
        run()
        torch.cuda.synchronize()
        return sum(k["launches"] for k in L.mebp_kernel_timing_report() if k["kernel"] == "frag_weights")
    finally:
        L.mebp_kernel_timing(False)


def _check(cfg, inp, dm, x, dy, dx):
    dx_ref, g_ref = O.layer_backward(cfg, 0, O.decompress_layer(cfg, inp, 0), x, dy)
    errs = {"dx": rel_l2(to_np(dx) - dy, dx_ref - dy)}
    for p, (dA, dB) in g_ref.items():
        errs["dA_" + p], errs["dB_" + p] = rel_l2(to_np(dm.dA[0][p]), dA), rel_l2(to_np(dm.dB[0][p]), dB)
    say("rel-L2", {k: f"{v:.2e}" for k, v in errs.items()})
    assert max(errs.values()) <= TOL, errs


# the shapes of the tile tests with a vocabulary whose logits (or, from 256 tokens on, whose own
# copy) leave room for a layer's weights
@pytest.mark.parametrize("case", BWD_CASES, ids=lambda c: f"d{c[0]}-dh{c[3]}-f{c[4]}-{c[5]}x{c[6]}")
def test_layer_copy(built_lib, gpu, case):
    d, h, kv, dh, f, b, t, act, r = case
    cfg = Config(name="copy", n_layers=1, hidden=d, n_heads=h, n_kv_heads=kv, head_dim=dh, ffn=f, vocab=262144, act=act,
                 lora_rank=r, lora_alpha=2.0 * r, lora_modules=ALL7, batch=b, seq=t)
    inp, dm = _model(cfg, 4, gpu)
    x, dy = layer_input(cfg, 12)
    tx, tdy = torch.from_numpy(x).to(gpu), torch.from_numpy(dy).to(gpu)
    dx = torch.full_like(tx, float("nan"))
    say("copy of a layer", case)
    assert _copies(lambda: dm.layer_backward(0, tx, tdy, dx)) == 1
    _check(cfg, inp, dm, x, dy, dx)


# model, vocabulary kept, tokens, launches that write copies
STATIC_CASES = [
    ("qwen2.5-0.5b", False, 256, 1),
    ("qwen2.5-0.5b", True, 256, 1),
    ("qwen2.5-0.5b", True, 300, 1),   # (fits the library's buffer with one set of slots)
    ("qwen2.5-0.5b", False, 300, 4),  # one product at a time
    ("gemma3-1b", True, 200, 4),      # (whose whole copy the library's buffer has no room for)
    ("gemma3-1b", True, 100, 1),
    ("qwen2.5-1.5b", True, 128, 0),   # int4 weights
    ("gemma3-1b", False, 64, 0),
]


@pytest.mark.parametrize("case", STATIC_CASES, ids=lambda c: f"{c[0]}-{'v' if c[1] else '0'}-{c[2]}")
def test_library_buffer_takes_the_same_route(built_lib, gpu, case):
    name, vocab, t, copies = case
    cfg = CONFIGS[name].with_(batch=1, seq=t)
    cfg = cfg if vocab else cfg.with_(vocab=0)
    inp, dm = _model(cfg, 5, gpu)
    x, dy = layer_input(cfg, 13)
    tx, tdy = torch.from_numpy(x).to(gpu), torch.from_numpy(dy).to(gpu)
    dx, dx_st = (torch.full_like(tx, float("nan")) for _ in range(2))
    say("library buffer", case, "workspace", dm.ws_bytes)
    assert _copies(lambda: dm.layer_backward(0, tx, tdy, dx)) == copies
    ref = {p: (dm.dA[0][p].clone(), dm.dB[0][p].clone()) for p in dm.dA[0]}
    for p in ref:
        dm.dA[0][p].fill_(float("nan"))
        dm.dB[0][p].fill_(float("nan"))
    static = lambda: L.mebp_layer_recompute_backward_static(dm.ccfg, 0, dm.base[0], dm.lora[0], ptr(tx), ptr(tdy),
                                                            ptr(dx_st), dm.grads[0], dm.B, dm.T, stream_handle())
    assert _copies(static) == copies
    assert torch.equal(dx_st, dx)
    for p, (a, b) in ref.items():
        assert torch.equal(dm.dA[0][p], a) and torch.equal(dm.dB[0][p], b), p
    _check(cfg, inp, dm, x, dy, dx)


# below 256 tokens the LM head keeps no copy of its own and a layer's lie in its logits: whole steps,
# whose LM head and layers take turns there (dx0 is asked for, so every layer needs all its copies)
STEP_CASES = [("qwen2.5-0.5b", 100, 1), ("gemma3-1b", 200, 4), ("qwen2.5-1.5b", 120, 0)]


@pytest.mark.parametrize("case", STEP_CASES, ids=lambda c: f"{c[0]}-{c[1]}")
def test_step_on_each_route(built_lib, gpu, case):
    name, t, copies = case
    cfg = CONFIGS[name].with_(batch=1, seq=t, n_layers=3)
    inp = make_inputs(cfg, seed=7, norm="random")
    dm = DeviceModel(inp, device=str(gpu))
    dx0 = torch.full((dm.N, cfg.hidden), float("nan"), dtype=torch.float32, device=gpu)
    say("step", case, "workspace", dm.ws_bytes)
    assert _copies(lambda: dm.train_step(dx0)) == copies * cfg.n_layers
    ref = O.train_step(cfg, inp, keep_ckpts=False)
    errs = {"dx0": rel_l2(to_np(dx0), ref.dx0)}
    for l in range(cfg.n_layers):
        for p, (dA, dB) in ref.grads[l].items():
            errs[f"dA{l}_{p}"], errs[f"dB{l}_{p}"] = rel_l2(to_np(dm.dA[l][p]), dA), rel_l2(to_np(dm.dB[l][p]), dB)
    say("loss", dm.loss.item(), ref.loss, "worst", max(errs.values()))
    assert abs(dm.loss.item() - ref.loss) <= 1e-3 * abs(ref.loss) and max(errs.values()) <= TOL, errs
    # the same bits as a replayed graph, with eager steps between the replays, and with guards
    eager = dm.loss.clone(), dx0.clone(), dm.grad_probe().clone()
    same = lambda: all(torch.equal(a, b) for a, b in zip(eager, (dm.loss, dx0, dm.grad_probe())))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            dm.train_step(dx0)
    torch.cuda.current_stream().wait_stream(side)
    for i in range(3):
        dx0.fill_(float("nan"))
        say("graph replay", i)
        graph.replay()
        torch.cuda.synchronize()
        assert same()
        dm.train_step(dx0)
        torch.cuda.synchronize()
        assert same()
    prev = L.mebp_set_workspace_guards(True)
    try:
        dm = DeviceModel(inp, device=str(gpu))
        dx0.fill_(float("nan"))
        say("guards")
        dm.train_step(dx0)
        torch.cuda.synchronize()
        assert same()
    finally:
        L.mebp_set_workspace_guards(prev)
