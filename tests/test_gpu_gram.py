"""The dense FP64 Gram kernels at the edges of their block counts (GPU): every row
count from which another count of 16-row blocks is used, columns at the edges of a
tile and of a slab, against FP64 products.  Tolerance per entry: two sums of `cols`
terms in FP64, 2 cols u sum |terms|."""

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
U = 2.0 ** -53


@pytest.mark.parametrize("m", [1, 16, 17, 33, 65, 128, 129, 144, 145, 160, 161, 176, 192, 193,
                               208, 224, 225, 240, 255, 256, 257, 320, 321, 384, 385, 449, 512])
@pytest.mark.parametrize("cols", [1, 15, 16, 17, 31, 49, 4096 + 5, 33000])
def test_f64_gram_block_counts(gpu_lib, m, cols):
    print("[gram] f64", m, cols, flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(m * 1000 + cols)
    # rows from an odd 8-byte boundary on, NaN around them
    ld = cols + (m + cols) % 3
    buf = torch.full((1 + (m + 3) * ld,), float("nan"), device=DEV, dtype=torch.float64)
    X = buf[1:1 + (m + 3) * ld].view(m + 3, ld)[:, :cols]
    X.copy_(torch.randn(m + 3, cols, generator=g, device=DEV, dtype=torch.float64))
    u = torch.randn(cols, generator=g, device=DEV, dtype=torch.float64)
    idx = torch.randint(0, m + 3, (m,), generator=g, device=DEV).to(torch.int32)
    Y = X[idx.long()].contiguous()
    same = torch.eye(m, device=DEV, dtype=torch.float64)
    for want_u in (True, False):
        G, Yu = gpu_lib.gram(X, idx, 0.5, 0.25, u if want_u else None)
        want, mag = 0.5 * (Y @ Y.t()) + 0.25 * same, 0.5 * (Y.abs() @ Y.abs().t()) + 0.25 * same
        assert bool(((G - want).abs() <= 2 * (cols + 2) * U * mag).all())
        assert torch.equal(G, G.t())
        if want_u:
            want, mag = Y @ u, Y.abs() @ u.abs()
            assert bool(((Yu - want).abs() <= 2 * (cols + 2) * U * mag).all())
