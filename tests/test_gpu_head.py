"""ringada_head_ce over many workgroups: widths at the edges of the 64-feature
blocks, batches at the edges of the 16 waves and of two samples per wave,
sequences of one position (no rows to zero), and dY in the place of y (the one
workgroup for all features), there also with several chunks of 256 samples and
several blocks of 1024 features.  dY over rows of y that are not read is a call like
any other.  Bounds as in test_gpu_tiles: fp32 sums of exact
inputs 1e-4, the bf16 dY two units in the last place."""
import numpy as np
import pytest

from helpers import TOL, Checker
import oracle as O
from paper_2502_19864_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_classes,batch,seq,d,inplace", [
    (2, 1, 1, 8, False), (2, 16, 3, 64, False), (2, 17, 2, 72, False), (2, 33, 1, 776, False), (3, 15, 2, 56, False),
    (16, 18, 2, 136, False), (1, 5, 2, 128, False), (2, 33, 3, 776, True), (5, 20, 2, 1032, True),
    (2, 257, 1, 1024, True), (2, 300, 2, 2048, True), (5, 300, 1, 1032, True), (16, 513, 2, 2056, True),
    (2, 17, 3, 72, "past"), (5, 3, 2, 136, "past")])
def test_head_blocks(dtype, n_classes, batch, seq, d, inplace):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(1000 * n_classes + batch + d)
    y = torch.randn(batch, seq, d, generator=g).to(tdt)
    wh, bh = 0.05 * torch.randn(d, n_classes, generator=g), 0.1 * torch.randn(n_classes, generator=g)
    lab = torch.randint(0, n_classes, (batch,), generator=g, dtype=torch.int32)
    gwh0, gbh0 = torch.randn(d, n_classes, generator=g), torch.randn(n_classes, generator=g)
    dev = lambda t: t.cuda()  # noqa: E731
    yt, labt, wht, bht = dev(y), dev(lab), dev(wh), dev(bh)
    s = torch.cuda.current_stream().cuda_stream
    runs = []
    for _ in range(2):
        src = yt.clone()
        dyt = src if inplace is True else torch.full_like(yt, float("nan"))
        if inplace == "past":  # over the rows of y past its last position 0, which nobody reads
            buf = torch.full((2 * yt.numel(),), float("nan"), dtype=tdt, device="cuda")
            src, dyt = buf[:yt.numel()].view_as(yt), buf[yt.numel() - (seq - 1) * d:][:yt.numel()].view_as(yt)
            src.copy_(yt)
        gwh, gbh, loss = dev(gwh0), dev(gbh0), torch.full((1,), 2.0, device="cuda")
        B.ringada_head_ce(s, B.BF16 if dtype == "bf16" else B.F32, src, batch, seq, d, wht, bht, n_classes, labt, dyt,
                          gwh, gbh, loss)
        torch.cuda.synchronize()
        runs.append((dyt, gwh, gbh, loss))
    assert all(torch.equal(a, b) for a, b in zip(*runs)), "different bits on the same inputs"
    rloss, rdy, rgwh, rgbh = O.cls_head_ce(y.double().numpy(), wh.double().numpy(), bh.double().numpy(), lab.numpy())
    dyt, gwh, gbh, loss = runs[0]
    chk = Checker(f"head blocks {dtype} C={n_classes} B={batch} S={seq} d={d}", tol=TOL["f32"])
    chk("loss", loss.cpu().numpy(), np.array([rloss]) + 2.0)
    chk("g_wh", gwh.cpu().numpy(), rgwh + gwh0.double().numpy())
    chk("g_bh", gbh.cpu().numpy(), rgbh + gbh0.double().numpy())
    if n_classes > 1:  # one class: the gradient is zero
        dchk = Checker(f"head blocks dy {dtype} C={n_classes} B={batch} S={seq} d={d}",
                       tol=TOL["f32"] if dtype == "f32" else 2.0 ** -7)
        dchk("dy", dyt.float().cpu().numpy(), rdy)
        dchk.done()
    assert torch.all(dyt[:, 1:] == 0), "rows past position 0 must be zeros"
    chk.done()
