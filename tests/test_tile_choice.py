"""The choice of a GEMM tile, on the host: no kernel is compiled that no legal stage
reaches, every kernel is taken by a GPU parity case, and those cases take the tiles
that they are there for."""
import test_gpu_tile_choice
import test_gpu_tiles
import tile_choice as T


def gpu_cases():
    for name, w in test_gpu_tiles.TILES.items():
        yield name, (w.arch, w.d_model, w.n_heads, w.d_ffn, w.seq, w.batch), test_gpu_tiles.TILES_TAKE[name]
    for name, (arch, d, h, f, seq, batch, _, takes) in test_gpu_tile_choice.CASES.items():
        yield name, (arch, d, h, f, seq, batch), takes


def taken(arch, d, h, f, seq, batch):
    return T.taken(arch, seq * batch, d, f, fused=arch == "bert" and d // h == 64 and seq == 128)


def test_no_kernel_without_a_shape():
    for arch in ("bert", "llama"):
        assert T.reached(arch) == T.built(arch)


def test_every_kernel_has_a_gpu_case():
    got = set().union(*(taken(*c) for _, c, _ in gpu_cases()))
    missing = (T.built("bert") | T.built("llama")) - got
    assert not missing, sorted(missing)


def test_gpu_cases_take_their_tiles():
    for name, c, takes in gpu_cases():
        got = {(s, t) for s, _, t in taken(*c)}
        want = {tuple(p.split()) for p in takes.split(", ")}
        assert want <= got, (name, sorted(want - got), sorted(got))
