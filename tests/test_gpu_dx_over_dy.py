"""The input gradient written over the incoming one (dx_in = dy): a pre-RMS stage
reads dy itself as the gradient at its top FFN adapter's output until the weight
gradients at the end of the backward, so that buffer is then copied first.  The
results are the bits of a call with two buffers."""
import pytest

from paper_2502_19864_amd.stage import Stage
from paper_2502_19864_amd.workloads import Workload, make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("placement", ["houlsby", "ffn"])
@pytest.mark.parametrize("arch,d,n_blocks", [("llama", 256, 1), ("llama", 256, 2), ("llama", 2048, 2), ("bert", 256, 2)])
def test_dx_over_dy(arch, d, n_blocks, placement):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = Workload("dx_over_dy", arch, "bf16", n_blocks, d, d // 64, 192, 64, 40, 2, -1, "dy", 2601, placement=placement)
    inp = make_inputs(w)
    st = Stage(w, inp)
    try:
        res = []
        for same in (False, True):
            x, y, dy = st.upload(inp["x"]), st.empty(*inp["x"].shape), st.upload(inp["dy"])
            dx = dy if same else st.empty(*inp["x"].shape)
            st.zero_grads()
            st.forward(x, y, -1)
            st.backward(dy, -1, dx)
            res.append((dx.float().cpu(), st.grads()))
    finally:
        st.close()
    assert torch.equal(res[0][0], res[1][0])
    for a, b in zip(res[0][1], res[1][1]):
        for p, q in zip(a, b):
            assert all((p[k] == q[k]).all() for k in p)
