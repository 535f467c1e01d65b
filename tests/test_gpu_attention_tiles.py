"""Attention over more than one tile at the edges of its divisions: 32-row
blocks (per wave), 64-row tiles (two deep in LDS) and 128-row workgroups, causal
and not, at both head widths, down to sequences shorter than one block.  Method
and bounds are those of the tile cases in test_gpu_tiles."""
import pytest

import test_gpu_tiles as tiles
from test_gpu_tiles import torch  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(600)
@pytest.mark.parametrize("seq", [1, 31, 65, 129, 160, 193, 224, 256, 257, 390])
@pytest.mark.parametrize("arch,heads", [("bert", 4), ("bert", 2), ("llama", 4), ("llama", 2)])
def test_attention_tile_edges(torch, monkeypatch, arch, heads, seq):  # noqa: F811
    name = f"attn_{arch}_h{heads}_s{seq}"
    monkeypatch.setitem(tiles.TILES, name, tiles._w(name, arch, 256, heads, 192, seq, 3, 2500 + seq))
    tiles.test_tile_configuration_parity(torch, name)
