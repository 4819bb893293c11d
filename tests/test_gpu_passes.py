"""The streaming passes over stored codes, at the edges of their splits (GPU): the
exact residual X^T w - y and the map -X a / (lambda n) against FP64 products of
the dequantised matrix.  Tolerance per entry: a sum of `rows` terms in FP64,
2 rows u sum |terms|."""

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
U = 2.0 ** -53


# one to 16 waves a column group, the rows split over the grid from 512 rows on;
# ragged last chunks and single columns
@pytest.mark.parametrize("rows,cols", [(1, 1), (5, 100), (17, 515), (40, 1000), (64, 33001),
                                       (130, 300001), (300, 70001), (513, 600), (5000, 31),
                                       (4187, 618), (2001, 20001)])
@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("padded", [True, False])
def test_lowp_passes(gpu_lib, dtype, rows, cols, padded):
    print("[passes]", dtype, rows, cols, padded, flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(rows * 7 + cols)
    X = torch.randn(rows, cols, generator=g, device=DEV, dtype=torch.float64)
    Q = gpu_lib.quantize(X, gpu_lib.BF16 if dtype == "bf16" else gpu_lib.FP8_E4M3)
    Xh = Q.dequantize().contiguous()
    if not padded:
        Q = gpu_lib.Quantized(Q.codes.contiguous(), Q.scales, Q.dtype)
    w = torch.randn(rows, generator=g, device=DEV, dtype=torch.float64)
    y = torch.randn(cols, generator=g, device=DEV, dtype=torch.float64)
    _, r = gpu_lib.primal_objective(Q, y, 0.1, w)
    want = Xh.t() @ w - y
    mag = Xh.abs().t() @ w.abs() + y.abs()
    assert bool(((r - want).abs() <= 2 * (rows + 2) * U * mag).all())
    v = gpu_lib.dual_to_primal(Q, w, 0.5)
    want = (Xh.t() @ w) / (-0.5 * rows)
    mag = (Xh.abs().t() @ w.abs()) / (0.5 * rows)
    assert bool(((v - want).abs() <= 2 * (rows + 2) * U * mag).all())
