"""The fp32 stage at the sizes where its kernels' tiles can go wrong: head
dims that are not multiples of four or fill a tile row, more than one 64-row
attention tile, bottlenecks and token counts off the 16-wide tiles, products
on both tile widths, and frozen weights that are only 4-byte aligned.  fp32
bound of the other parity tests (1e-4)."""
import pytest

from gpu_run import run_gpu
from helpers import TOL, Checker, oracle_run
from paper_2502_19864_amd import binding as B
from paper_2502_19864_amd.stage import Stage
from paper_2502_19864_amd.workloads import Workload, make_inputs

pytestmark = pytest.mark.gpu


class OddWeights(Stage):
    """Frozen matrices one element past a 16-byte boundary."""

    def upload(self, a):
        t = super().upload(a)
        if t.dim() != 2:
            return t
        buf = self.torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
        buf[1:] = t.reshape(-1)
        return buf[1:].view(t.shape)


def _w(name, d, h, f, m, seq, batch, seed, placement="houlsby"):
    return Workload(name, "bert", "f32", 2, d, h, f, m, seq, batch, 0, "dy", seed, placement=placement)


CASES = [
    (_w("f32_dh2", 4, 2, 4, 4, 3, 1, 2501), Stage),
    (_w("f32_dh30_s70", 60, 2, 68, 8, 70, 2, 2502), Stage),
    (_w("f32_dh128_s130", 128, 1, 132, 20, 130, 1, 2503), Stage),
    (_w("f32_dh66_s65", 132, 2, 64, 16, 65, 2, 2504, "ffn"), Stage),
    (_w("f32_wide_tiles", 256, 4, 1024, 32, 64, 8, 2505), Stage),
    (_w("f32_odd_weights", 128, 2, 256, 16, 33, 3, 2506), OddWeights),
]


@pytest.mark.timeout(300)
@pytest.mark.parametrize("w,cls", CASES, ids=[c[0].name for c in CASES])
def test_f32_stage_edges(w, cls):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    inp = make_inputs(w)
    print(f"[{w.name}] d={w.d_model} H={w.n_heads} F={w.d_ffn} m={w.d_adapter} batch={w.batch} seq={w.seq}", flush=True)
    st = cls(w, inp)
    try:
        gpu = run_gpu(torch, st, w, inp, -1, want_dx=True)
    finally:
        st.close()
    ref = oracle_run(w, inp, -1)
    chk = Checker(w.name, tol=TOL["f32"])
    chk("y", gpu["y"], ref["y"])
    chk("dx", gpu["dx"], ref["dx"])
    chk.grads(gpu["grads"], ref["grads"], 0, w.n_blocks)
    chk.done()


class SharedGrads(Stage):
    """Every adapter of the stage adds into the first one's gradients."""

    def __init__(self, w, inp):
        super().__init__(w, inp)
        first = self.adapters[0][1]
        for l, pair in enumerate(self.adapters):
            for t in pair:
                t.update(g_down=first["g_down"], g_up=first["g_up"])
            ca = [B.Adapter(**{k: v.data_ptr() for k, v in t.items()}) for t in pair]
            bw = B.BlockWeights(**{k: v.data_ptr() for k, v in self.frozen[l].items()})
            B.ringada_stage_bind_block(self.handle, l, bw, None if w.placement == "ffn" else ca[0], ca[1],
                                       self.block_mem[l], self.block_bytes, self.sptr)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("dtype,d,f,m,placement", [("f32", 128, 256, 16, "houlsby"), ("f32", 60, 68, 8, "ffn"),
                                                   ("bf16", 256, 192, 64, "houlsby")])
def test_shared_gradients_add_up(dtype, d, f, m, placement):
    """Adapters bound to the same gradient buffers: the backward adds every one's
    gradient, as one adapter after the other.  The sum of up to six fp32 values
    of either run differs by their rounding (2^-20 of the largest)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = Workload("shared", "bert", dtype, 3, d, 2, f, m, 20, 3, 0, "dy", 2507, placement=placement)
    inp = make_inputs(w)
    res = []
    for cls in (Stage, SharedGrads):
        print(f"[shared gradients] {dtype} {placement} {cls.__name__}", flush=True)
        st = cls(w, inp)
        try:
            res.append(run_gpu(torch, st, w, inp, -1, want_dx=True)["grads"])
        finally:
            st.close()
    apart, shared = res
    for k in ("w_down", "w_up"):
        want = sum(pair[a][k].astype("float64") for pair in apart for a in range(2))
        assert abs(shared[0][1][k] - want).max() <= 2.0 ** -20 * abs(want).max(), k
