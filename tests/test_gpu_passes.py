"""The streaming passes, at the edges of their splits and on every boundary that a
row may start on (GPU): the exact residual X^T w - y, the full residual and the map
-X a / (lambda n) against FP64 products (codes: of the dequantised matrix).  Tolerance per entry: a sum of `rows` terms in FP64,
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
                                       (4187, 618), (2001, 20001), (1025, 140001),
                                       (2300, 131072)])
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


# rows that start on odd 8-byte boundaries (odd ld, odd first element) and on
# 16-byte ones; one column, odd and even counts, several parts of a row
@pytest.mark.parametrize("off,pad", [(0, 0), (1, 0), (0, 1), (1, 1), (1, 2)])
@pytest.mark.parametrize("rows,cols", [(3, 1), (40, 33), (257, 1030), (19, 20001), (900, 77)])
def test_f64_rows_on_any_boundary(gpu_lib, rows, cols, off, pad):
    print("[passes] f64", rows, cols, off, pad, flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + cols)
    buf = torch.full((off + rows * (cols + pad) + 1,), float("nan"), device=DEV,
                     dtype=torch.float64)
    X = buf[off:off + rows * (cols + pad)].view(rows, cols + pad)[:, :cols]
    X.copy_(torch.randn(rows, cols, generator=g, device=DEV, dtype=torch.float64))
    vec = torch.randn(rows + 2 * cols + 3, generator=g, device=DEV, dtype=torch.float64)
    w, y, u = vec[1:1 + rows], vec[1 + rows:1 + rows + cols], vec[-cols - 1:-1]
    Xc = X.contiguous()
    _, r = gpu_lib.primal_objective(X, y, 0.1, w)
    want, mag = Xc.t() @ w - y, Xc.abs().t() @ w.abs() + y.abs()
    assert bool(((r - want).abs() <= 2 * (rows + 2) * U * mag).all())
    _, rho = gpu_lib.primal_residual(X, 0.1, w, u)
    want, mag = -0.1 * w - (Xc @ u) / cols, 0.1 * w.abs() + (Xc.abs() @ u.abs()) / cols
    assert bool(((rho - want).abs() <= 2 * (cols + 4) * U * mag).all())
    for m in (1, 16, 31, 64, 100, 129, 256, 300):
        idx = torch.randint(0, rows, (m,), generator=g, device=DEV, dtype=torch.int32)
        G, Yu = gpu_lib.gram(X, idx, 1.0 / cols, 0.5, u)
        Y = Xc[idx.long()]
        want = Y @ Y.t() / cols + 0.5 * torch.eye(m, device=DEV, dtype=torch.float64)
        mag = Y.abs() @ Y.abs().t() / cols + 0.5
        assert bool(((G - want).abs() <= 2 * (cols + 4) * U * mag).all())
        assert bool(((Yu - Y @ u).abs() <= 2 * (cols + 4) * U * (Y.abs() @ u.abs())).all())


# every remainder of a 16-byte chunk, rows shorter than one, one and several tiles,
# each block count of the low-precision Gram; codes from an odd and an aligned byte on.
# Entries are small whole numbers (times 64), so FP32 and FP64 sums are exact.
@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("off,pad", [(0, 0), (1, 0), (0, 1)])
@pytest.mark.parametrize("m", [3, 20, 60, 100, 200])
def test_lowp_gram_ragged_ends(gpu_lib, dtype, m, off, pad):
    print("[passes] lowp gram ends", dtype, m, off, pad, flush=True)
    code = gpu_lib.BF16 if dtype == "bf16" else gpu_lib.FP8_E4M3
    g = torch.Generator(device=DEV)
    g.manual_seed(m)
    idx = torch.randperm(m, generator=g, device=DEV).to(torch.int32)
    for cols in list(range(1, 35)) + [256 + r for r in range(0, 16, 3)] + [4096 + 17]:
        X = 64.0 * torch.randint(-7, 8, (m, cols), generator=g, device=DEV).to(torch.float64)
        X[:, cols // 2] = 448.0     # FP8 row scale 1
        Q = gpu_lib.quantize(X, code)
        if off or pad:
            ld = cols + pad
            buf = torch.zeros(off + m * ld, device=DEV, dtype=Q.codes.dtype)
            view = buf[off:].view(m, ld)[:, :cols]
            view.copy_(Q.codes)
            Q = gpu_lib.Quantized(view, Q.scales, Q.dtype)
        u = torch.randint(-3, 4, (cols,), generator=g, device=DEV).to(torch.float64)
        G, Yu = gpu_lib.gram(Q, idx, 1.0, 0.0, u)
        Y = X[idx.long()].cpu()
        assert torch.equal(G.cpu(), Y @ Y.t()), cols
        assert torch.equal(Yu.cpu(), Y @ u.cpu()), cols
