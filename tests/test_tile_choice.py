"""The choice of a GEMM tile, on the host: no kernel is compiled that no legal stage
reaches."""
import tile_choice as T


def test_no_kernel_without_a_shape():
    for arch in ("bert", "llama"):
        assert T.reached(arch) == T.built(arch)
