"""The bf16 copy of the weights that the transposed products read does not enlarge the workspace
(host only): what the products that decompress int4 weights take, with their split planes and the
16-bit copy of one product's weights on large tiles, stays enough for every configured shape."""
import pytest

from mebp_inputs import CONFIGS, MINI
from paper_2510_03425_amd import _lib as L
from paper_2510_03425_amd.device import make_config

SHAPES = ((1, 64), (1, 128), (1, 200), (1, 256), (1, 300), (1, 512), (3, 333), (4, 1024), (8, 2048))
# bytes before there was such a copy: whole model, one layer's calls alone (vocabulary 0)
BYTES = {
    "qwen2.5-0.5b": (
        (57419008, 114838016, 144517888, 482022400, 477371136, 621258752, 861022976, 1308672000, 2776432640),
        (21730048, 43460096, 52342016, 66997248, 66839552, 113022976, 192789248, 542720000, 1988165632)),
    "gemma3-1b": (
        (83452672, 166905344, 201809152, 895323136, 884572928, 1102780416, 1482219520, 1499447296, 3433259008),
        (30547200, 61094400, 62283008, 79721472, 71305472, 141617152, 245760256, 705970176, 2667798528)),
    "qwen2.5-1.5b": (
        (68667136, 137334272, 160110080, 704715776, 693393920, 866138112, 1157867008, 1769652224, 4389634048),
        (30504192, 61008384, 66654208, 85316608, 86464256, 160147456, 291830528, 939606016, 3567157248)),
    "gemma3-4b": (
        (91320064, 182640128, 221888768, 1660271616, 1686068224, 1971025920, 2446200320, 2257043456, 5883691008),
        (37644544, 75289088, 80775424, 103392256, 132222464, 267601920, 460546560, 1309032448, 4893442048)),
}


@pytest.mark.parametrize("model", list(BYTES))
@pytest.mark.parametrize("vocab", [True, False], ids=["model", "layer"])
def test_workspace_is_no_larger(built_lib, model, vocab):
    cfg = CONFIGS[model]
    c = make_config(cfg if vocab else cfg.with_(vocab=0))
    for (B, T), most in zip(SHAPES, BYTES[model][not vocab]):
        assert L.mebp_workspace_bytes(c, B, T) <= most, (B, T)


def test_what_the_static_call_took_still_fits(built_lib):
    for model, (_, layer) in BYTES.items():
        for (B, T), was in zip(SHAPES, layer):
            if was <= L.STATIC_SCRATCH_BYTES:
                c = make_config(CONFIGS[model].with_(vocab=0))
                assert L.mebp_workspace_bytes(c, B, T) <= L.STATIC_SCRATCH_BYTES, (model, B, T)


def test_no_copy_beyond_one_buffer_resource(built_lib):
    """A product reads its copy through one buffer resource, whose offsets have 32 bits: a vocabulary
    chunk of 4 GiB and more in bf16 is decompressed in the product instead."""
    c = make_config(MINI.with_(n_heads=1, n_kv_heads=1, head_dim=128, ffn=192))
    c.hidden = 8192
    for vocab, copied in ((262144 - 64, True), (262144, False), (524288, False)):
        c.vocab = vocab
        assert (L.mebp_workspace_bytes(c, 1, 256) > vocab * c.hidden * 2) == copied, vocab
