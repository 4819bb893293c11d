"""Outer steps whose Grams are computed ahead run as a chain: the inverse of each
Gram's lower block triangle formed ahead, one launch per dense step.  Checked
against the oracle (GPU) at the edges of its tiles: superblocks that the block
size fills or pads, one to 32 of them, slabs of every width with ragged ends,
rows on odd 8-byte boundaries, repeated indices, exact recomputations between
steps, and the storage formats."""

import numpy as np
import pytest
import scipy.sparse
import torch

import synth
from oracle import bcd, sampler

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _rel(a, b):
    a, b = np.asarray(a), np.asarray(b)
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def _say(*a):
    print("[chain]", *a, flush=True)


# b, s: superblocks of 16 / b blocks: b = 1, 3 (15 rows), 6 (12), 9 (9), 16;
# s b = 256 full, 9 x 28 = 252 in 28 superblocks, a partial last superblock
@pytest.mark.parametrize("b,s", [(1, 1), (1, 37), (3, 17), (4, 64), (6, 25), (8, 32), (9, 28),
                                 (12, 5), (16, 16), (7, 2)])
@pytest.mark.parametrize("n,steps", [(1, 9), (31, 12), (257, 7), (2049, 37)])
def test_primal_chain_matches_oracle(gpu_lib, b, s, n, steps):
    """n = 1, 31: one slab, less than a chunk of it; 2049: a last slab of one
    column; rows of n columns (odd: 8-byte boundaries)."""
    d = max(40, b)
    H = steps * s + s // 2
    _say("primal", b, s, n, H)
    X, y, _ = synth.gaussian_ridge(d, n, 10 * b + s + n)
    w, r = gpu_lib.primal_bcd(X.to(DEV), y.to(DEV), 0.3, b, s, H, 5)
    wo, zo = bcd.primal_bcd(X.numpy(), y.numpy(), 0.3, b, s, H, 5)
    assert _rel(w.cpu(), wo) <= 1e-10
    assert _rel(r.cpu(), zo - y.numpy()) <= 1e-10


@pytest.mark.parametrize("d,b,s", [(30, 4, 8), (33, 5, 20), (1000, 8, 32), (4097, 2, 12),
                                   (70001, 4, 3), (300001, 8, 2)])
def test_dual_chain_matches_oracle(gpu_lib, d, b, s):
    """Slabs of 32 to 1024 columns (and more slabs than 256)."""
    n, H = 60, 21 * s
    _say("dual", d, b, s)
    X, y, _ = synth.gaussian_ridge(d, n, d + b)
    a, w = gpu_lib.dual_bcd(X.t().contiguous().to(DEV), y.to(DEV), 1e-2, b, s, H, 6)
    ao, wo = bcd.dual_bcd(X.numpy(), y.numpy(), 1e-2, b, s, H, 6)
    assert _rel(a.cpu(), ao) <= 1e-10
    assert _rel(w.cpu(), wo) <= 1e-10


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("n,pad,b,s", [(1000, True, 8, 12), (1001, False, 6, 5),
                                       (20003, True, 4, 32), (600001, True, 4, 2)])
def test_chain_codes(gpu_lib, dtype, n, pad, b, s):
    """Stored codes, padded rows and rows on odd boundaries: the residual is that
    of the iterate (FP64 passes over the codes), and the iterate is the FP64
    run's on the dequantised matrix within the Gram's FP32 accumulation."""
    d, steps = 64, 12
    _say("codes", dtype, n, pad, b, s)
    X, y, _ = synth.gaussian_ridge(d, n, n + b)
    Q = gpu_lib.quantize(X.to(DEV), gpu_lib.BF16 if dtype == "bf16" else gpu_lib.FP8_E4M3)
    Xh = Q.dequantize()
    if not pad:
        Q = gpu_lib.Quantized(Q.codes.contiguous(), Q.scales, Q.dtype)
    yd = y.to(DEV)
    w, r = gpu_lib.primal_bcd(Q, yd, 0.1, b, s, steps * s, 8)
    assert _rel(r.cpu(), (Xh.t() @ w - yd).cpu()) <= 1e-11
    wo, _ = bcd.primal_bcd(Xh.cpu().numpy(), y.numpy(), 0.1, b, s, steps * s, 8)
    # each delta solves with a Gram of relative error 2^-24 sqrt(n) (FP8: 1e-5)
    assert _rel(w.cpu(), wo) <= (1e-5 if dtype == "bf16" else 1e-3)


@pytest.mark.parametrize("dtype,n", [("f64", 3001), ("bf16", 3001), ("bf16", 3007),
                                     ("fp8", 3009), ("fp8", 3023)])
@pytest.mark.parametrize("b,s", [(4, 2), (8, 8)])
def test_chain_ragged_columns(gpu_lib, dtype, n, b, s):
    """The columns past the last 16-byte chunk (1 to 15 of them): the residual of every
    one is the iterate's after many steps, in one call and in calls of a step, to the same
    bits."""
    d, steps = 48, 30
    _say("ragged columns", dtype, n, b, s)
    X, y, _ = synth.gaussian_ridge(d, n, n)
    A, yd = X.to(DEV), y.to(DEV)
    Xh = A
    if dtype != "f64":
        A = gpu_lib.quantize(A, gpu_lib.BF16 if dtype == "bf16" else gpu_lib.FP8_E4M3)
        Xh = A.dequantize()
    w, r = gpu_lib.primal_bcd(A, yd, 0.1, b, s, steps * s, 8)
    exact = (Xh.t() @ w - yd).cpu()
    k = n // 16 * 16
    assert _rel(r[k:].cpu(), exact[k:]) <= 1e-11 and _rel(r.cpu(), exact) <= 1e-11
    w1, r1 = torch.zeros_like(w), -yd
    for i in range(steps):
        gpu_lib.primal_bcd(A, yd, 0.1, b, s, s, 8, w=w1, r=r1, h0=i * s,
                           flags=gpu_lib.FLAG_STATE_VALID)
    w2, r2 = torch.zeros_like(w), -yd
    gpu_lib.primal_bcd(A, yd, 0.1, b, s, steps * s, 8, w=w2, r=r2,
                       flags=gpu_lib.FLAG_STATE_VALID)
    assert torch.equal(w1, w2) and torch.equal(r1, r2)


def test_chain_repeated_indices_and_recomputation(gpu_lib):
    """Blocks that repeat indices within a step many times over, with exact
    recomputations between steps, monitor points, and the same run in calls."""
    d, n, b, s, steps = 9, 515, 4, 16, 10
    _say("repeats")
    X, y, _ = synth.gaussian_ridge(d, n, 3)
    rng = np.random.default_rng(1)
    idx = np.concatenate([rng.permutation(d)[:b] for _ in range(steps * s)]).astype(np.int32)
    Xd, yd = X.to(DEV), y.to(DEV)
    ix = torch.tensor(idx, device=DEV)
    wo, zo = bcd.primal_bcd(X.numpy(), y.numpy(), 0.2, b, s, steps * s, 0,
                            explicit_idx=idx.reshape(-1, b))
    w, r = gpu_lib.primal_bcd(Xd, yd, 0.2, b, s, steps * s, 0, explicit_idx=ix)
    assert _rel(w.cpu(), wo) <= 1e-10 and _rel(r.cpu(), zo - y.numpy()) <= 1e-10
    tr = torch.empty(5, dtype=torch.float64, device=DEV)
    w2, r2 = gpu_lib.primal_bcd(Xd, yd, 0.2, b, s, steps * s, 0, explicit_idx=ix, resid_every=3,
                                monitor_every=2, trace=tr)
    assert _rel(w2.cpu(), wo) <= 1e-10 and _rel(r2.cpu(), zo - y.numpy()) <= 1e-10
    w3 = torch.zeros(d, dtype=torch.float64, device=DEV)
    r3 = -yd
    for k0, k1 in ((0, 1), (1, 6), (6, 10)):
        part = ix[k0 * s * b:k1 * s * b].contiguous()
        gpu_lib.primal_bcd(Xd, yd, 0.2, b, s, (k1 - k0) * s, 0, w=w3, r=r3, explicit_idx=part,
                           flags=gpu_lib.FLAG_STATE_VALID)
    w4 = torch.zeros(d, dtype=torch.float64, device=DEV)
    r4 = -yd
    gpu_lib.primal_bcd(Xd, yd, 0.2, b, s, steps * s, 0, w=w4, r=r4, explicit_idx=ix,
                       flags=gpu_lib.FLAG_STATE_VALID)
    assert torch.equal(w3, w4) and torch.equal(r3, r4)


def test_chain_short_workspace_and_pivot(gpu_lib):
    """A caller workspace too small for the chain's buffers (but large enough for
    the solves inside the steps) is accepted; a block that is not positive
    definite is reported."""
    d, n, b, s = 12, 300001, 4, 2
    X, y, _ = synth.gaussian_ridge(d, n, 4)
    Xd, yd = X.to(DEV), y.to(DEV)
    w, r = gpu_lib.primal_bcd(Xd, yd, 0.1, b, s, 20 * s, 1)
    ws = torch.empty(gpu_lib.workspace_bytes(Xd, b, s) // 3, dtype=torch.uint8, device=DEV)
    w1, r1 = gpu_lib.primal_bcd(Xd, yd, 0.1, b, s, 20 * s, 1, workspace=ws)
    assert _rel(w1.cpu(), w.cpu()) <= 1e-12 and _rel(r1.cpu(), r.cpu()) <= 1e-12
    Xb = X.clone()
    Xb[7] = float("nan")
    with pytest.raises(gpu_lib.CabcdError) as e:
        gpu_lib.primal_bcd(Xb.to(DEV), yd, 0.1, b, s, 20 * s, 1)
    assert e.value.status == gpu_lib.ENOTSPD


@pytest.mark.parametrize("b,s", [(16, 32), (9, 32), (8, 64), (5, 40), (16, 8), (4, 3), (1, 300)])
def test_csr_chain_matches_oracle(gpu_lib, b, s):
    """Sparse steps: the split Gram (s b >= 256) and the hash join, one to 32
    superblocks, full and padded."""
    n, d, H = 900, 700, 9 * s + 2
    _say("csr", b, s)
    rng = np.random.default_rng(b + s)
    S = scipy.sparse.random(n, d, 0.03, format="csr", random_state=np.random.RandomState(b * s),
                            data_rvs=rng.standard_normal)
    y = rng.standard_normal(n)
    a, w = gpu_lib.dual_bcd(gpu_lib.CSR.from_scipy(S, DEV), torch.tensor(y, device=DEV), 1e-2, b,
                            s, H, 7)
    ao, wo = bcd.dual_bcd(S.T.tocsc(), y, 1e-2, b, s, H, 7)
    assert _rel(a.cpu(), ao) <= 1e-10
    assert _rel(w.cpu(), wo) <= 1e-10


# one workgroup for runs of steps: one column lane to eight columns a lane, as many rows
# as its registers hold and one less, one to eight superblocks
@pytest.mark.parametrize("d,b,s", [(1, 1, 1), (63, 8, 16), (64, 1, 127), (65, 16, 8), (128, 4, 32),
                                   (129, 7, 9), (257, 16, 2), (512, 8, 4), (513, 4, 4),
                                   (1024, 5, 3), (1025, 8, 1), (2048, 2, 4), (2049, 2, 2),
                                   (4096, 1, 4)])
def test_dual_short_steps_in_one_workgroup(gpu_lib, d, b, s):
    """Against the oracle, and the same bits when the run is split, monitored
    steps and exact recomputations in between; rows on odd 8-byte boundaries."""
    n = max(50, b)            # repeated coordinates from step to step
    H = 23 * s + s // 2
    _say("short dual steps", d, b, s)
    X, y, _ = synth.gaussian_ridge(d, n, d + b + s)
    buf = torch.full((1 + n * (d + 1),), float("nan"), dtype=torch.float64, device=DEV)
    A = buf[1:].view(n, d + 1)[:, :d]
    A.copy_(X.t())
    a, w = gpu_lib.dual_bcd(A, y.to(DEV), 1e-2, b, s, H, 6, resid_every=7)
    ao, wo = bcd.dual_bcd(X.numpy(), y.numpy(), 1e-2, b, s, H, 6)
    assert _rel(a.cpu(), ao) <= 1e-10
    assert _rel(w.cpu(), wo) <= 1e-10
    a1, w1 = gpu_lib.dual_bcd(A, y.to(DEV), 1e-2, b, s, H, 6)
    a2, w2 = gpu_lib.dual_bcd(A, y.to(DEV), 1e-2, b, s, 9 * s, 6)
    a2, w2 = gpu_lib.dual_bcd(A, y.to(DEV), 1e-2, b, s, H - 9 * s, 6, alpha=a2, w=w2,
                              h0=9 * s, flags=gpu_lib.FLAG_STATE_VALID)
    assert torch.equal(a1, a2) and torch.equal(w1, w2)


# sparse steps in two launches up to 64 rows, in three from there on
@pytest.mark.parametrize("b,s", [(1, 1), (1, 64), (1, 65), (3, 21), (5, 7), (7, 9), (8, 8), (16, 4),
                                 (13, 5)])
@pytest.mark.parametrize("kind", ["dual", "primal"])
def test_sparse_steps_of_few_rows(gpu_lib, kind, b, s):
    """Rows without entries, coordinates repeated inside and across steps, exact
    recomputations in between."""
    rows, cols = 70, 900
    _say("sparse few rows", kind, b, s)
    rng = np.random.default_rng(b * s)
    S = scipy.sparse.random(rows, cols, 0.05, random_state=rng, format="csr")
    S.data = rng.standard_normal(S.nnz)
    S = scipy.sparse.csr_matrix(S.multiply((np.arange(rows) % 9 != 4)[:, None]))
    S.eliminate_zeros()
    S.sort_indices()
    H = 13 * s + s // 2
    y = rng.standard_normal(rows if kind == "dual" else cols)
    A = gpu_lib.CSR.from_scipy(S, DEV)
    yd = torch.tensor(y, device=DEV)
    if kind == "dual":
        x, u = gpu_lib.dual_bcd(A, yd, 1e-2, b, s, H, 8, resid_every=5)
        xo, uo = bcd.dual_bcd(S.T.tocsc(), y, 1e-2, b, s, H, 8)
    else:
        x, u = gpu_lib.primal_bcd(A, yd, 1e-2, b, s, H, 8, resid_every=5)
        xo, uo = bcd.primal_bcd(S, y, 1e-2, b, s, H, 8)
        uo = uo - y
    assert _rel(x.cpu(), xo) <= 1e-10
    assert _rel(u.cpu(), uo) <= 1e-10


def _blockwise(dual, A, y, lam, blocks, dt):
    """Block coordinate descent block by block (Alg. 1 / Alg. 3) in precision dt:
    the coordinates and the companion."""
    A, y, lam = A.astype(dt), y.astype(dt), dt(lam)
    rows, cols = A.shape
    n = dt(rows if dual else cols)
    scale, shift, gamma = (1 / (lam * n * n), 1 / n, -1 / (lam * n)) if dual else (1 / n, lam, dt(1))
    x, u = np.zeros(rows, dt), np.zeros(cols, dt) if dual else -y
    for I in blocks:
        Y, b = A[I], len(I)
        c = (Y @ u - x[I] - y[I]) / n if dual else -lam * x[I] - Y @ u / n
        M = np.column_stack([scale * (Y @ Y.T) + shift * np.eye(b, dtype=dt), c])
        for k in range(b):
            M[k + 1:] -= np.outer(M[k + 1:, k] / M[k, k], M[k])
        d = M[:, -1].copy()
        for k in range(b - 1, -1, -1):
            d[k] = (d[k] - M[k, k + 1:-1] @ d[k + 1:]) / M[k, k]
        x[I] += d
        u += gamma * (Y.T @ d)
    return x, u


# one workgroup for runs of steps, a launch a step (few rows, many), sparse steps in two and
# three launches and with the split Gram
@pytest.mark.parametrize("kind,rows,cols,b,s,steps", [
    ("primal", 64, 256, 4, 8, 12), ("primal", 64, 1024, 4, 8, 12), ("primal", 64, 1024, 8, 4, 12),
    ("primal", 256, 4096, 8, 32, 3), ("dual", 64, 128, 4, 8, 12), ("dual", 128, 1000, 8, 16, 8),
    ("dual", 300, 600, 16, 16, 6), ("dual", 200, 514, 5, 20, 4), ("csr primal", 64, 1024, 4, 8, 12),
    ("csr dual", 128, 1000, 8, 16, 8), ("csr primal", 300, 1000, 8, 32, 3),
    ("csr dual", 600, 800, 16, 32, 3)])
@pytest.mark.parametrize("rho,lam", [(0.95, 1e-3), (0.999, 1e-3), (0.9999, 1e-5)])
def test_nearly_collinear_rows(gpu_lib, kind, rows, cols, b, s, steps, rho, lam):
    """Rows with correlation rho (0.95: some superblock rows of the inverse are refined and
    some are not): both results as close to an extended-precision run as substitution comes.  The unit is the error of the descent block by block in FP64
    on the same data; the s-step recurrence by substitution, on the CPU, takes up to 7.3 of
    it over these cases (its right-hand sides are s blocks old), and sums in another order
    are allowed 20."""
    _say("collinear", kind, rows, cols, b, s, rho)
    dual = kind.endswith("dual")
    rng = np.random.default_rng(2)
    v = rng.standard_normal(cols)
    A = np.sqrt(rho) * v + np.sqrt(1 - rho) * rng.standard_normal((rows, cols))
    y = (rng.standard_normal(rows) if dual
         else A.T @ rng.standard_normal(rows) + 0.1 * rng.standard_normal(cols))
    H, seed = s * steps, 3
    blocks = [list(sampler.sample_block(seed, h, b, rows)) for h in range(H)]
    exact = _blockwise(dual, A, y, lam, blocks, np.longdouble)
    plain = _blockwise(dual, A, y, lam, blocks, np.float64)
    Ad = (gpu_lib.CSR.from_scipy(scipy.sparse.csr_matrix(A), DEV) if kind.startswith("csr")
          else torch.tensor(A, device=DEV))
    call = gpu_lib.dual_bcd if dual else gpu_lib.primal_bcd
    out = call(Ad, torch.tensor(y, device=DEV), lam, b, s, H, seed)
    errs = [(float(_rel(g.cpu().numpy(), e)), float(_rel(p, e)))
            for g, p, e in zip(out, plain, exact)]
    _say("  " + ", ".join(f"{e:.1e} = {e / unit:.1f} x {unit:.1e}" for e, unit in errs))
    for e, unit in errs:
        assert e <= 20 * unit


# one workgroup for runs of steps, a launch a step (8 MiB of rows and less, and more), sparse
# steps in two launches and three, the split Gram, and the solves with blocks inverted ahead
# (codes on odd boundaries)
@pytest.mark.parametrize("kind,n,b,s", [("dense", 256, 4, 8), ("dense", 1024, 8, 1),
                                        ("dense", 1024, 16, 8), ("dense", 40000, 4, 8),
                                        ("csr", 1024, 4, 8), ("csr", 1024, 8, 16),
                                        ("csr", 1024, 8, 32), ("bf16", 1001, 4, 8),
                                        ("bf16", 1001, 16, 4)])
def test_block_of_a_step_that_is_not_run(gpu_lib, kind, n, b, s):
    """Rows 62 and 63 make a block that is not positive definite.  A run that its tolerance
    stops before the step that draws it ends well, though that step's Gram was
    computed ahead; a run that reaches it reports the block."""
    _say("block not run", kind, n, b, s)
    d, steps = 64, 4
    rng = np.random.default_rng(4)
    X = rng.standard_normal((d, n))
    y = rng.standard_normal(n)
    # their Gram overflows; nothing else has anything in column 0
    X[:, 0] = y[0] = 0.0
    X[62, 0], X[63, 0] = (1e30, -1e30) if kind == "bf16" else (1e200, -1e200)
    idx = np.concatenate([rng.permutation(62)[:b] for _ in range(steps * s)]).astype(np.int32)
    idx = idx.reshape(-1, b)
    idx[2 * s, :min(b, 2)] = (62, 63)[:min(b, 2)]
    if kind == "csr":
        A = gpu_lib.CSR.from_scipy(scipy.sparse.csr_matrix(X), DEV)
    elif kind == "bf16":
        Q = gpu_lib.quantize(torch.tensor(X, device=DEV), gpu_lib.BF16)
        A = gpu_lib.Quantized(Q.codes.contiguous(), Q.scales, Q.dtype)
    else:
        A = torch.tensor(X, device=DEV)
    ix, yd = torch.tensor(idx.ravel(), device=DEV), torch.tensor(y, device=DEV)
    stats = {}
    w, r = gpu_lib.primal_bcd(A, yd, 0.1, b, s, steps * s, 0, explicit_idx=ix, tol=1e6,
                              check_every=2, stats=stats)
    assert stats["h"] == 2 * s
    Xd = X[:62] if kind != "bf16" else Q.dequantize().cpu().numpy()[:62]
    wo, _ = bcd.primal_bcd(Xd, y, 0.1, b, s, 2 * s, 0, explicit_idx=idx)
    assert _rel(w[:62].cpu(), wo) <= (1e-10 if kind != "bf16" else 1e-4)
    with pytest.raises(gpu_lib.CabcdError) as e:
        gpu_lib.primal_bcd(A, yd, 0.1, b, s, steps * s, 0, explicit_idx=ix)
    assert e.value.status == gpu_lib.ENOTSPD
