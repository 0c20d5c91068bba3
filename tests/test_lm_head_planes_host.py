"""The LM head's plane buffer holds the planes of every vocabulary chunk, the narrower last one
included (host only: sizes from the layout the library computes).

The library plans a chunk of w columns like a vocabulary of w columns, so the planes of the last
chunk are those of the same call with the vocabulary that is left of it. The split of a shorter
reduction may be the larger one; planes past the buffer would land in the slots behind it.
"""
import functools
import os
import random
import subprocess
import sys

import pytest

from mebp_inputs import CONFIGS, MINI
from paper_2510_03425_amd import _lib as L
from paper_2510_03425_amd.device import make_config, slot_index

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


slot = functools.lru_cache(slot_index)


def _planes(c, B, T):
    lo, hi = (L.mebp_workspace_offset(c, B, T, slot(n)) for n in ("lm_part", "grad"))
    return (hi - lo) // (B * T * c.hidden * 4)  # (the padding behind a slot is below one plane)


def chunk_cols(n_tokens, vocab, mib=512):
    """Columns of a chunk: fp16 logits of `mib` MiB at most, a multiple of 256."""
    return min(vocab, max(256, (mib << 20) // (n_tokens * 2) // 256 * 256))


def _config(hidden, vocab):
    c = make_config(MINI.with_(n_heads=1, n_kv_heads=1, head_dim=128, ffn=192, lora_rank=8))
    c.hidden, c.vocab = hidden, vocab
    return c


def check(hidden, vocab, B, T, mib=512):
    last = vocab % chunk_cols(B * T, vocab, mib)
    whole = _planes(_config(hidden, vocab), B, T)
    if last:
        assert whole >= _planes(_config(hidden, last), B, T), (hidden, vocab, B, T, mib)
    return bool(last)


@pytest.mark.parametrize("hidden,vocab,B,T", [(128, 151936, 136, 64), (128, 50304, 80, 128), (128, 50304, 1, 10240)])
def test_last_chunk_fits(built_lib, hidden, vocab, B, T):
    assert check(hidden, vocab, B, T)


def test_last_chunk_fits_over_shapes(built_lib):
    rng = random.Random(17)
    n = 0
    while n < 4000:
        hidden = 32 * rng.choice([2, 3, 4, 6, 8, 12, 16, 28, 36, 48, 80, 128])
        vocab = 32 * int(2 ** rng.uniform(5, 13.2))
        n += check(hidden, vocab, rng.choice([1, 2, 3, 8]), int(2 ** rng.uniform(7, 13)))


# small chunks (MEBP_LM_CHUNK_MB is read once per process)
@pytest.mark.parametrize("mib,model,tokens", [(32, "qwen2.5-0.5b", range(400, 460)), (16, "qwen2.5-1.5b", range(1400, 1450)),
                                              (16, "gemma3-4b", range(300, 2000, 37))])
def test_last_chunk_fits_with_small_chunks(built_lib, mib, model, tokens):
    c = CONFIGS[model]
    code = ("import tests.test_lm_head_planes_host as t\n"
            f"for n in {list(tokens)}: t.check({c.hidden}, {c.vocab}, 1, n, {mib})\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=dict(os.environ, MEBP_LM_CHUNK_MB=str(mib)),
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
