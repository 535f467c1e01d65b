"""ringada_loss_mse over its two ways (one workgroup; many, with the partial
sums kept in dY until the last kernel writes those elements), at the line
between them, at odd sizes, on unaligned tensors and in place."""
import numpy as np
import pytest

import oracle as O
from helpers import rel_err
from paper_2502_19864_amd import binding as B

pytestmark = pytest.mark.gpu

ONE = 128 << 10  # bytes per tensor up to which one workgroup does it


@pytest.mark.parametrize("dtype,n,offset,inplace,loss", [
    ("bf16", 1, 0, False, True), ("bf16", 4097, 1, False, True),
    ("bf16", ONE // 2, 0, False, True), ("bf16", ONE // 2 + 1, 0, False, True),
    ("bf16", ONE // 2 + 9, 3, False, True), ("bf16", 1_500_001, 0, False, True),
    ("bf16", 4_194_304, 0, False, True), ("bf16", 300_000, 0, True, True), ("bf16", 300_007, 0, False, False),
    ("f32", ONE // 4, 0, False, True), ("f32", ONE // 4 + 4, 0, False, True), ("f32", 700_003, 1, False, True),
    ("f32", 200_000, 0, True, True)])
def test_mse_sizes(dtype, n, offset, inplace, loss):
    """dY is one rounding of an fp32 value (bf16 2^-8, fp32 2^-22, relative to
    the largest); the loss an fp32 sum of n squares (1e-5).  Twice the same bits."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(2400 + n)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    dev = torch.device("cuda", 0)

    def dev_of(a):
        buf = torch.empty(n + offset + 8, dtype=tdt, device=dev)
        buf[offset:offset + n] = torch.from_numpy(a).to(dev).to(tdt)
        return buf, buf[offset:offset + n]

    (_, y), (_, t) = (dev_of(rng.standard_normal(n).astype(np.float32)) for _ in range(2))
    ref_loss, ref_dy = O.mse_loss(y.double().cpu().numpy(), t.double().cpu().numpy())
    runs = []
    for _ in range(2):
        yy = y.clone() if inplace else y
        buf, dy = dev_of(np.full(n, np.nan, np.float32))
        buf[:offset], buf[offset + n:] = 7.0, 7.0
        dy = yy if inplace else dy
        lt = torch.zeros(1, device=dev) if loss else None
        print(f"[mse] {dtype} n={n} offset={offset} inplace={inplace}", flush=True)
        B.ringada_loss_mse(torch.cuda.current_stream(dev).cuda_stream, B.BF16 if dtype == "bf16" else B.F32, yy, t, n,
                           dy, lt)
        torch.cuda.synchronize()
        assert bool((buf[:offset] == 7).all()) and bool((buf[offset + n:] == 7).all()), "wrote outside dY"
        runs.append((dy.clone(), lt))
    assert torch.equal(runs[0][0], runs[1][0])
    assert rel_err(runs[0][0].double().cpu().numpy(), ref_dy) <= (2.0 ** -8 if dtype == "bf16" else 2.0 ** -22)
    if loss:
        assert torch.equal(runs[0][1], runs[1][1])
        assert abs(float(runs[0][1]) / ref_loss - 1) <= 1e-5
