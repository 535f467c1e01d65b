"""Parity of the tiles that the projection GEMMs take by estimated time: the
small ones (32x32, 32x64, 64x64, 64x128 with 128- and 64-wide k-tiles), the four-stage
128x192 and the 256x256, each with ragged last tiles where its range has them.
Method and bounds are those of the tile cases in test_gpu_tiles (which compares
three different sequences: batches of three or more)."""
import pytest

import test_gpu_tiles as tiles
from test_gpu_tiles import torch  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

CASES = {
    # 32x32 and 32x64 with K dealt to four wave groups, 25 rows past the end
    "choice_bert_t39": ("bert", 768, 12, 3072, 13, 3, 2401),
    # 32x64 with store, GELU, residual and GELU' epilogues
    "choice_bert_t90": ("bert", 1024, 16, 4096, 30, 3, 2408),
    # 64x64, and 64x128 with 64-wide k-tiles (K = 960 is no multiple of 128)
    "choice_bert_t300": ("bert", 1024, 16, 960, 100, 3, 2402),
    # 64x128 in the rotary and SwiGLU epilogues, 29 of 64 rows past the end
    "choice_llama_t99": ("llama", 1024, 8, 2752, 33, 3, 2403),
    # 64x128 with 64-wide k-tiles in the dX products of a gated block (2 F = 1344 + 64)
    "choice_llama_f704": ("llama", 512, 4, 704, 75, 20, 2404),
    # 128x192 with four stages, 64x128, 93 rows past the end
    "choice_bert_t1827": ("bert", 768, 12, 3072, 203, 9, 2405),
    # 256x256 GELU and GELU'
    "choice_bert_t4096": ("bert", 1024, 16, 4096, 256, 16, 2406),
    # 256x256 SwiGLU, dSwiGLU and rotary, a last tile of 192 of 256 rows
    "choice_llama_t4032": ("llama", 1024, 16, 4096, 504, 8, 2407),
}


@pytest.mark.timeout(600)
@pytest.mark.parametrize("name", sorted(CASES))
def test_chosen_tile_parity(torch, monkeypatch, name):  # noqa: F811
    arch, d, h, f, seq, batch, seed = CASES[name]
    monkeypatch.setitem(tiles.TILES, name, tiles._w(name, arch, d, h, f, seq, batch, seed))
    tiles.test_tile_configuration_parity(torch, name)
