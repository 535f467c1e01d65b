"""Parity of the tiles that the projection GEMMs take by estimated time.  Each case
says which (call site, tile) pairs it is there for, with ragged last tiles where the
pair's range has them; test_tile_choice asks the launcher's own choice whether it
takes them, and whether the cases here and in test_gpu_tiles take every kernel that
is compiled.  Method and bounds are those of the tile cases in test_gpu_tiles (which
compares three different sequences: batches of three or more)."""
import pytest

import test_gpu_tiles as tiles
from test_gpu_tiles import torch  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

# name: (arch, d, heads, ffn, seq, batch, seed, what it is for)
CASES = {
    # K dealt to four wave groups; 25 rows of the last tile past the end
    "choice_bert_t39": ("bert", 768, 12, 3072, 13, 3, 2401,
                        "qkv_fwd 32x64, ffn_in_fwd 32x64, ffn_out_fwd 32x32/2, ffn_in_dx 32x32/2, ffn_out_dx 32x64"),
    "choice_bert_t90": ("bert", 1024, 16, 4096, 30, 3, 2408, "o_fwd 32x32/2, o_dx 32x32/2, qkv_dx 32x32/2"),
    "choice_bert_t30": ("bert", 1024, 16, 128, 10, 3, 2409,
                        "qkv_fwd 32x32/2, ffn_in_fwd 32x32/2, ffn_out_dx 32x32/2"),
    "choice_bert_f128": ("bert", 256, 4, 128, 30, 3, 2410, "ffn_out_fwd 32x64, ffn_in_dx 32x64"),
    "choice_llama_f128": ("llama", 256, 2, 128, 30, 3, 2411, "qkv_dx 32x64, ffn_in_dx 32x64, ffn_out_dx 32x64"),
    # F = 960 is no multiple of 128: 64-wide k-tiles in the products over it
    "choice_bert_t300": ("bert", 1024, 16, 960, 100, 3, 2402,
                         "qkv_fwd 64x64, ffn_out_fwd 64x128/k64, ffn_in_dx 64x128/k64"),
    "choice_bert_t2050": ("bert", 256, 4, 512, 50, 41, 2412,
                          "qkv_fwd 64x128, ffn_in_fwd 64x128, ffn_out_fwd 64x64, qkv_dx 64x64, ffn_in_dx 64x64, "
                          "ffn_out_dx 64x128"),
    # 29 of 64 rows past the end
    "choice_llama_t99": ("llama", 1024, 8, 2752, 33, 3, 2403, "qkv_fwd 64x128, ffn_in_fwd 64x128"),
    # 2 F = 1408 = 11 x 128
    "choice_llama_f704": ("llama", 512, 4, 704, 75, 20, 2404,
                          "ffn_out_fwd 64x128/k64, ffn_in_dx 64x64, ffn_out_dx 64x128, ffn_in_fwd 128x128"),
    "choice_llama_t4270": ("llama", 256, 2, 128, 61, 70, 2413, "qkv_dx 64x128, ffn_out_dx 64x64"),
    # 93 rows past the end
    "choice_bert_t1827": ("bert", 768, 12, 3072, 203, 9, 2405,
                          "qkv_fwd 128x192, o_fwd 64x128, ffn_in_fwd 128x192, ffn_out_fwd 64x128, ffn_out_dx 128x192"),
    "choice_bert_t900": ("bert", 768, 12, 64, 30, 30, 2414, "qkv_fwd 128x96"),
    "choice_bert_t8296": ("bert", 256, 4, 960, 61, 136, 2415,
                          "qkv_fwd 256x128, ffn_in_fwd 128x192/2, ffn_out_fwd 128x96, ffn_in_dx 128x96, "
                          "ffn_out_dx 128x192/2"),
    "choice_bert_t4900": ("bert", 256, 2, 1600, 100, 49, 2416,
                          "qkv_fwd 128x128, ffn_in_fwd 128x128/2, ffn_out_dx 128x128/2"),
    "choice_bert_t5400": ("bert", 768, 12, 448, 50, 108, 2417,
                          "qkv_fwd 256x256, ffn_out_fwd 128x192, qkv_dx 128x192, ffn_in_dx 128x192"),
    "choice_llama_t10791": ("llama", 256, 4, 384, 33, 327, 2418,
                            "qkv_fwd 128x128/2, ffn_in_fwd 128x128/2, qkv_dx 128x96, ffn_in_dx 128x96"),
    "choice_llama_d768_t10791": ("llama", 768, 12, 64, 33, 327, 2419,
                                 "o_fwd 128x128/2, o_dx 128x128/2, qkv_dx 128x128/2, ffn_in_dx 128x128/2"),
    "choice_bert_d768_t10791": ("bert", 768, 6, 64, 33, 327, 2420, "qkv_dx 128x128/2"),
    "choice_llama_d1024_t10791": ("llama", 1024, 8, 64, 33, 327, 2421, "qkv_dx 128x192/2"),
    "choice_bert_d1024_t10791": ("bert", 1024, 16, 64, 33, 327, 2422,
                                 "qkv_fwd 128x128/2, o_fwd 128x192/2, o_dx 128x192/2, qkv_dx 128x192/2"),
    "choice_llama_t8296": ("llama", 512, 8, 256, 61, 136, 2423, "ffn_in_dx 128x192"),
    "choice_bert_t4096": ("bert", 1024, 16, 4096, 256, 16, 2406,
                          "qkv_fwd 128x192/2, ffn_in_fwd 256x256, ffn_out_dx 256x256"),
    # a last tile of 192 of 256 rows
    "choice_llama_t4032": ("llama", 1024, 16, 4096, 504, 8, 2407,
                           "qkv_fwd 256x256, ffn_in_fwd 256x256, ffn_out_dx 128x128/2"),
    # a last tile of 132 of 256 rows
    "choice_llama_t32900": ("llama", 256, 4, 768, 100, 329, 2424,
                            "ffn_out_fwd 256x256, qkv_dx 256x256, ffn_in_dx 256x256"),
    "choice_bert_t32900": ("bert", 256, 4, 768, 100, 329, 2425, "ffn_in_dx 256x256"),
    "choice_llama_d2048_t4270": ("llama", 2048, 16, 704, 61, 70, 2426, "ffn_in_dx 256x192, ffn_out_dx 128x128"),
    "choice_llama_d3072_t3201": ("llama", 3072, 24, 1216, 33, 97, 2427, "ffn_out_dx 128x192"),
    # dSwiGLU on 256x256, a last tile of 148 of 256 rows
    "choice_llama_d4096_t4500": ("llama", 4096, 32, 2752, 50, 90, 2428, "ffn_out_dx 256x256"),
}


@pytest.mark.timeout(600)
@pytest.mark.parametrize("name", sorted(CASES))
def test_chosen_tile_parity(torch, monkeypatch, name):  # noqa: F811
    arch, d, h, f, seq, batch, seed, _ = CASES[name]
    monkeypatch.setitem(tiles.TILES, name, tiles._w(name, arch, d, h, f, seq, batch, seed))
    tiles.test_tile_configuration_parity(torch, name)
