"""Batched primal CA-BCD (one persistent launch per round for many problems)
against the CPU oracle, problem by problem.

* With (b, s, seed, H) fixed per problem, each problem's w must equal the
  oracle's Alg. 2 run on that problem alone (same blocks) to 1e-10 relative,
  and r must equal X^T w - y.
* The hipGraph replay and direct launches give bitwise identical results, and
  so does a run split into several calls (the arithmetic is deterministic).
* Autotuned (b, s): every problem reaches a relative objective error of 1e-6
  against its closed-form optimum and is retired by its f_target.
"""

import numpy as np
import pytest
import torch

from oracle import bcd
import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _say(*a):
    print(*a, flush=True)


# (d, n, b, s, H, lambda, seed): ragged last steps, b = d, s*b = 256, odd n
# (rows not 16-byte aligned), many slabs, b = 1, b not a power of two.
CASES = [
    (37, 1001, 4, 3, 50, 1e-2, 11),
    (64, 4096, 8, 8, 200, 1e-3, 12),
    (300, 5000, 16, 16, 96, 1e-3, 13),
    (20, 777, 5, 2, 23, 5e-2, 14),
    (128, 20000, 16, 4, 64, 1e-4, 15),
    (9, 300, 9, 1, 3, 1e-1, 16),
    (50, 4096, 1, 32, 100, 1e-3, 17),
    (200, 3001, 12, 10, 77, 1e-3, 18),
    (33, 65, 16, 16, 40, 1e-2, 19),
    (1, 100, 1, 4, 9, 1e-1, 20),
]


def _problems(cases):
    probs = []
    for i, (d, n, b, s, H, lam, seed) in enumerate(cases):
        X, y, _ = synth.gaussian_ridge(d, n, 500 + i)
        probs.append(dict(X=X.to(DEV), y=y.to(DEV), lam=lam, b=b, s=s, seed=seed, H=H,
                          Xc=X.numpy(), yc=y.numpy()))
    return probs


def _run(gpu_lib, probs, chunks, monitor_every=2, graph=True):
    with gpu_lib.Batch(probs, monitor_every=monitor_every, graph=graph) as B:
        act = None
        for c in chunks:
            act = B.run(c)
        infos = [B.info(p) for p in range(len(probs))]
    torch.cuda.synchronize()
    return act, infos


def test_batch_matches_oracle_per_problem(gpu_lib):
    _say("batch vs oracle,", len(CASES), "problems")
    probs = _problems(CASES)
    act, infos = _run(gpu_lib, probs, [100])
    assert act == 0
    for q, (d, n, b, s, H, lam, seed), inf in zip(probs, CASES, infos):
        assert inf["b"] == b and inf["s"] == s
        assert inf["h"] == H and inf["steps"] == -(-H // s) and not inf["active"]
        assert inf["status"] == gpu_lib.OK and np.isfinite(inf["objective"])
        wo, _ = bcd.primal_bcd(q["Xc"], q["yc"], lam, b, s, H, seed)
        w = q["w"].cpu().numpy()
        err = np.linalg.norm(w - wo) / max(np.linalg.norm(wo), 1e-300)
        _say(f"  d={d} n={n} b={b} s={s} H={H}: rel err {err:.2e}")
        assert err <= 1e-10
        r = q["r"].cpu().numpy()
        assert np.linalg.norm(r - (q["Xc"].T @ w - q["yc"])) <= 1e-10 * np.linalg.norm(q["yc"])


@pytest.mark.parametrize("cheap", [0, 2])
def test_batch_graph_direct_and_split_runs_are_identical(gpu_lib, cheap):
    _say("batch graph / direct / split runs, cheap monitors", cheap)
    cases = CASES[:6]
    runs = []
    for graph, chunks in ((True, [12]), (False, [12]), (True, [2, 1, 3, 4, 2])):
        probs = _problems(cases)
        with gpu_lib.Batch(probs, monitor_every=2, graph=graph, cheap_monitors=cheap) as B:
            for c in chunks:
                B.run(c)
        torch.cuda.synchronize()
        runs.append([(q["w"].cpu().numpy(), q["r"].cpu().numpy()) for q in probs])
    for other in runs[1:]:
        for (w0, r0), (w1, r1) in zip(runs[0], other):
            assert np.array_equal(w0, w1)
            assert np.array_equal(r0, r1)


def test_batch_reslicing_runs_are_identical_and_match_oracle(gpu_lib):
    """Problems retiring at different rounds (their budgets H) make the plan
    re-cut the remaining problems' slabs at the checks every 32 rounds (here at
    round 64, when 2 of 9 remain: a new work list, slabs and partials in the
    pool, graphs captured again): graph, direct and unevenly split runs stay
    bitwise identical and each problem matches the oracle."""
    _say("batch re-slicing")
    cases = [(64, 20000, 8, 4, 4 * H, 1e-3, 40 + H) for H in (8, 12, 20, 28, 36, 44, 60, 200)]
    cases += [(96, 30001, 16, 2, 400, 1e-3, 90)]
    runs = []
    for graph, chunks in ((True, [120]), (False, [120]), (True, [5, 27, 32, 1, 55])):
        probs = _problems(cases)
        with gpu_lib.Batch(probs, monitor_every=4, graph=graph) as B:
            for c in chunks:
                B.run(c)
            infos = [B.info(p) for p in range(len(probs))]
        torch.cuda.synchronize()
        runs.append([(q["w"].cpu().numpy(), q["r"].cpu().numpy()) for q in probs])
    for other in runs[1:]:
        for (w0, r0), (w1, r1) in zip(runs[0], other):
            assert np.array_equal(w0, w1) and np.array_equal(r0, r1)
    for (d, n, b, s, H, lam, seed), inf, q in zip(cases, infos, probs):
        assert inf["h"] == min(H, 120 * s)
        wo, _ = bcd.primal_bcd(q["Xc"], q["yc"], lam, b, s, inf["h"], seed)
        w = q["w"].cpu().numpy()
        assert np.linalg.norm(w - wo) <= 1e-10 * np.linalg.norm(wo)


BIG_CASES = [
    (400, 6000, 16, 32, 3 * 32 * 16 + 5 * 16, 1e-3, 61),   # s b = 512, ragged last step (80 rows)
    (300, 4097, 16, 20, 7 * 20 * 16, 1e-3, 62),            # 320 rows: 2 cross-block Grams
    (200, 3001, 12, 30, 5 * 30 * 12 + 7, 1e-2, 63),        # 360 rows, b not a power of two
    (64, 2000, 8, 4, 120, 1e-3, 64),                       # a small problem beside them
]


@pytest.mark.parametrize("dtype", ["f64", "bf16"])
def test_batch_grams_above_256_rows(gpu_lib, dtype):
    """s b in (256, 512]: every step's Gram assembled from 256-row Grams inside
    the persistent kernel.  FP64: each problem matches the oracle (1e-10).
    BF16: each matches the oracle on the dequantised matrix within 1e-3 (the
    Gram is accumulated in FP32: up to n u_32 ~ 4e-4 relative per entry at
    n = 6000; a misplaced or missing block moves the iterates by O(1))."""
    _say("batch above 256 rows", dtype)
    probs = _problems(BIG_CASES)
    if dtype == "bf16":
        for q in probs:
            Q = gpu_lib.quantize(q["X"], gpu_lib.BF16)
            q["X"], q["Xc"] = Q, Q.dequantize().cpu().numpy()
    act, infos = _run(gpu_lib, probs, [200])
    assert act == 0
    for q, (d, n, b, s, H, lam, seed), inf in zip(probs, BIG_CASES, infos):
        assert inf["b"] == b and inf["s"] == s and inf["h"] == H
        wo, _ = bcd.primal_bcd(q["Xc"], q["yc"], lam, b, s, H, seed)
        w = q["w"].cpu().numpy()
        err = np.linalg.norm(w - wo) / np.linalg.norm(wo)
        _say(f"  d={d} n={n} b={b} s={s}: rel err {err:.2e}")
        assert err <= (1e-10 if dtype == "f64" else 1e-3)


def test_batch_long_monitor_period_runs_without_graph(gpu_lib):
    """A monitor period longer than the 64 rounds a graph may hold launches
    directly: same iterates as a plan with graphs switched off."""
    _say("batch, monitor_every = 100")
    cases = CASES[:4]
    runs = []
    for graph in (True, False):
        probs = _problems(cases)
        with gpu_lib.Batch(probs, monitor_every=100, graph=graph) as B:
            B.run(150)
        torch.cuda.synchronize()
        runs.append([(q["w"].cpu().numpy(), q["r"].cpu().numpy()) for q in probs])
    for (w0, r0), (w1, r1) in zip(*runs):
        assert np.array_equal(w0, w1) and np.array_equal(r0, r1)


def test_batch_without_monitoring(gpu_lib):
    _say("batch, monitor_every = 0")
    cases = CASES[:4]
    probs = _problems(cases)
    act, infos = _run(gpu_lib, probs, [30, 30, 50], monitor_every=0)
    assert act == 0
    for q, (d, n, b, s, H, lam, seed) in zip(probs, cases):
        wo, _ = bcd.primal_bcd(q["Xc"], q["yc"], lam, b, s, H, seed)
        w = q["w"].cpu().numpy()
        assert np.linalg.norm(w - wo) <= 1e-10 * np.linalg.norm(wo)
        r = q["r"].cpu().numpy()   # maintained by the recurrence only
        assert np.linalg.norm(r - (q["Xc"].T @ w - q["yc"])) <= 1e-9 * np.linalg.norm(q["yc"])


def test_batch_autotuned_reaches_1e6(gpu_lib):
    P = 24
    ds, ns, lams = synth.ridge_batch(P, 77, d_range=(32, 512), n_range=(2048, 32768))
    _say("batch autotuned, P =", P)
    probs, fstars = [], []
    for p in range(P):
        X, y, _ = synth.gaussian_ridge(ds[p], ns[p], 900 + p)
        Xc, yc = X.numpy(), y.numpy()
        wst = bcd.ridge_closed_form(Xc, yc, lams[p])
        fst = bcd.primal_objective(Xc, yc, lams[p], wst)
        fstars.append(fst)
        probs.append(dict(X=X.to(DEV), y=y.to(DEV), lam=lams[p], seed=3000 + p,
                          f_target=fst * (1 + 1e-6), Xc=Xc, yc=yc))
    with gpu_lib.Batch(probs, monitor_every=4, cheap_monitors=3) as B:
        rounds, act = 0, P
        while act > 0 and rounds < 4000:
            act = B.run(4)
            rounds += 4
        infos = [B.info(p) for p in range(P)]
    _say(f"  all retired after {rounds} rounds (objective from the maintained residual "
         f"at 3 of 4 monitor points)")
    assert act == 0
    for q, fst, inf, d in zip(probs, fstars, infos, ds):
        # the tuner's range: b in {4, 8, 16}, 4 <= s <= 32, s b <= 256
        assert inf["b"] in (4, 8, 16) and inf["b"] <= d and inf["b"] * inf["s"] <= 256
        assert 4 <= inf["s"] <= 32
        w = q["w"].cpu().numpy()
        rel = (bcd.primal_objective(q["Xc"], q["yc"], q["lam"], w) - fst) / fst
        assert rel <= 1e-6 * (1 + 1e-6)
        assert abs(inf["objective"] - bcd.primal_objective(q["Xc"], q["yc"], q["lam"], w)) \
            <= 1e-12 * fst
    _say("  (b, s) chosen:", sorted({(i["b"], i["s"]) for i in infos}))


def test_batch_bench_size_sampled_problems(gpu_lib):
    """The batched workload at its full size: the benchmark's 256 problems (d
    log-uniform in [32, 1024], n in [4096, 131072], lambda in [1e-6, 1e-1];
    its generator, seeds and storage with rows leading_dim apart), planned with
    the autotuned (b, s) and the benchmark's monitoring, 8 rounds.  Eight
    problems (the smallest and largest d n, the largest s b, five drawn at
    random) against the oracle's Alg. 2 run of the same outer steps with the
    same (b, s) and seed: w to 1e-10, r to X^T w - y."""
    P, rounds = 256, 8
    ds, ns, lams = synth.ridge_batch(P, 1004)
    _say("batch bench size, P =", P, "sum d n =", sum(d * n for d, n in zip(ds, ns)))
    probs = []
    for p in range(P):
        X, y, _ = synth.gaussian_ridge(ds[p], ns[p], 1004 + 1 + p, device=DEV)
        Xp = gpu_lib.empty_dense(ds[p], ns[p], DEV)
        Xp.copy_(X)
        probs.append(dict(X=Xp, y=y, lam=lams[p], seed=2_000_000 + p))
        del X
    torch.cuda.empty_cache()
    with gpu_lib.Batch(probs, monitor_every=4, cheap_monitors=7) as B:
        act = B.run(rounds)
        infos = [B.info(p) for p in range(P)]
    torch.cuda.synchronize()
    assert act == P
    dn = [d * n for d, n in zip(ds, ns)]
    pick = {int(np.argmin(dn)), int(np.argmax(dn)),
            int(np.argmax([i["b"] * i["s"] for i in infos]))}
    pick |= {int(p) for p in np.random.default_rng(5).choice(P, 5, replace=False)}
    for p in sorted(pick):
        inf, q = infos[p], probs[p]
        b, s = inf["b"], inf["s"]
        assert inf["steps"] == rounds and inf["h"] == rounds * s
        Xc = np.ascontiguousarray(q["X"].cpu().numpy())
        yc = q["y"].cpu().numpy()
        wo, _ = bcd.primal_bcd(Xc, yc, q["lam"], b, s, rounds * s, q["seed"])
        w = q["w"].cpu().numpy()
        err = np.linalg.norm(w - wo) / max(np.linalg.norm(wo), 1e-300)
        _say(f"  problem {p}: d={ds[p]} n={ns[p]} b={b} s={s}: rel err {err:.2e}")
        assert err <= 1e-10
        r = q["r"].cpu().numpy()
        assert np.linalg.norm(r - (Xc.T @ w - yc)) <= 1e-10 * np.linalg.norm(yc)
    del probs
    torch.cuda.empty_cache()


def test_batch_one_shot_and_nonfinite(gpu_lib):
    _say("batch one-shot; non-finite data is reported")
    probs = _problems(CASES[:3])
    gpu_lib.primal_bcd_batched(probs, 1000, monitor_every=3)
    for q, (d, n, b, s, H, lam, seed) in zip(probs, CASES[:3]):
        wo, _ = bcd.primal_bcd(q["Xc"], q["yc"], lam, b, s, H, seed)
        assert np.linalg.norm(q["w"].cpu().numpy() - wo) <= 1e-10 * np.linalg.norm(wo)
    probs = _problems(CASES[:3])
    probs[1]["X"][3, 5] = float("nan")
    with pytest.raises(gpu_lib.CabcdError) as e:
        gpu_lib.primal_bcd_batched(probs, 1000, monitor_every=3)
    assert e.value.status in (gpu_lib.ENOTSPD, gpu_lib.ENONFINITE)
    assert "problem 1" in str(e.value)


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
def test_batch_lowp_reaches_1e6_on_dequantised(gpu_lib, dtype):
    """BF16 / FP8 storage: each problem is (X^, y, lambda) with X^ the stored
    matrix; it must reach 1e-6 relative objective error against the closed form
    on X^ and be retired by its target; r at the last monitor point equals
    X^ T w - y.  The distance to the FP64 oracle's iterates on X^ with the same
    blocks is reported, not pinned (the Gram is accumulated in FP32)."""
    P = 12
    ds, ns, lams = synth.ridge_batch(P, 78, d_range=(32, 300), n_range=(2048, 20000),
                                     lam_range=(1e-4, 1e-1))
    code = gpu_lib.BF16 if dtype == "bf16" else gpu_lib.FP8_E4M3
    _say("batch", dtype, "P =", P)
    probs = []
    for p in range(P):
        X, y, _ = synth.gaussian_ridge(ds[p], ns[p], 1200 + p)
        Q = gpu_lib.quantize(X.to(DEV), code)
        if p % 2:   # every other problem with rows starting at any byte
            Q = gpu_lib.Quantized(Q.codes.contiguous(), Q.scales, Q.dtype)
        Xh = Q.dequantize().cpu().numpy()
        yc = y.numpy()
        fst = bcd.primal_objective(Xh, yc, lams[p], bcd.ridge_closed_form(Xh, yc, lams[p]))
        probs.append(dict(X=Q, y=y.to(DEV), lam=lams[p], seed=4000 + p,
                          f_target=fst * (1 + 1e-6), Xh=Xh, yc=yc, fst=fst))
    with gpu_lib.Batch(probs, monitor_every=4) as B:
        rounds, act = 0, P
        while act > 0 and rounds < 4000:
            act = B.run(4)
            rounds += 4
        infos = [B.info(p) for p in range(P)]
    _say(f"  all retired after {rounds} rounds")
    assert act == 0
    for q, inf in zip(probs, infos):
        w = q["w"].cpu().numpy()
        rel = (bcd.primal_objective(q["Xh"], q["yc"], q["lam"], w) - q["fst"]) / q["fst"]
        assert rel <= 1e-6 * (1 + 1e-6)
        r = q["r"].cpu().numpy()
        assert np.linalg.norm(r - (q["Xh"].T @ w - q["yc"])) <= 1e-12 * np.linalg.norm(q["yc"])
    q, inf = probs[0], infos[0]
    wo, _ = bcd.primal_bcd(q["Xh"], q["yc"], q["lam"], inf["b"], inf["s"], inf["h"], q["seed"])
    _say(f"  problem 0: ||w - w_fp64 oracle|| / ||w_fp64|| = "
         f"{np.linalg.norm(q['w'].cpu().numpy() - wo) / np.linalg.norm(wo):.2e} (reported)")


def test_batch_mixed_storage_types_rejected(gpu_lib):
    X, y, _ = synth.gaussian_ridge(16, 256, 1)
    Xd = X.to(DEV)
    probs = [dict(X=Xd, y=y.to(DEV), lam=0.1, b=4, s=2, H=8),
             dict(X=gpu_lib.quantize(Xd, gpu_lib.BF16), y=y.to(DEV), lam=0.1, b=4, s=2, H=8)]
    with pytest.raises(gpu_lib.CabcdError) as e:
        gpu_lib.Batch(probs)
    assert e.value.status == gpu_lib.EINVAL


@pytest.mark.parametrize("b,s", [(1, 1), (5, 3), (4, 4), (8, 4), (9, 7), (16, 4), (16, 8)])
def test_batch_update_row_ranges_and_slab_groups(gpu_lib, b, s):
    """The update and the monitors split a slab's rows into 1, 2, 4 or 8 ranges
    (from 16, 32 and 64 rows on) over units of 128 columns, and slabs are summed
    in groups of eight: row counts at those lines, columns at the edges of a unit
    and from one slab to several groups of them."""
    _say("batch row ranges b=%d s=%d" % (b, s))
    cases = [(max(b, 40), n, b, s, 5 * s + 1, 1e-2, 70 + i)
             for i, n in enumerate((1, 127, 128, 129, 1025, 30011))]
    probs = _problems(cases)
    act, infos = _run(gpu_lib, probs, [3, 4])
    assert act == 0
    for q, (d, n, _, _, H, lam, seed), inf in zip(probs, cases, infos):
        wo, _ = bcd.primal_bcd(q["Xc"], q["yc"], lam, b, s, H, seed)
        w = q["w"].cpu().numpy()
        assert np.linalg.norm(w - wo) <= 1e-10 * max(np.linalg.norm(wo), 1e-300)
        ro = q["Xc"].T @ w - q["yc"]
        assert np.linalg.norm(q["r"].cpu().numpy() - ro) <= 1e-10 * np.linalg.norm(q["yc"])
        f = ro @ ro / (2 * n) + 0.5 * lam * (w @ w)
        assert abs(inf["objective"] - f) <= 1e-10 * f
    assert b * s < 32 or max(inf["nslab"] for inf in infos) > 8


def test_batch_update_pending_at_retirement_is_applied_after_reslicing(gpu_lib):
    """Without monitoring, problems whose budget ends before the slabs are cut
    again still get their last update when the run ends."""
    _say("batch retirement without monitoring")
    cases = [(40, 3000, 4, 4, 16 if i else 800, 1e-2, 80 + i) for i in range(4)]
    probs = _problems(cases)
    _run(gpu_lib, probs, [100], monitor_every=0)
    for q in probs:
        ro = q["Xc"].T @ q["w"].cpu().numpy() - q["yc"]
        assert np.linalg.norm(q["r"].cpu().numpy() - ro) <= 1e-10 * np.linalg.norm(q["yc"])


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("n", [64, 2000, 20011])
def test_batch_lowp_steps_above_256_rows_exact_sums(gpu_lib, dtype, n):
    """One step of 257 to 512 rows over whole-number codes (every sum of the Grams and
    of Y u is exact) ends at the oracle's w to the rounding of its solves; four problems,
    so that workgroups go from Gram to Gram and from problem to problem."""
    _say("batch lowp above 256 rows", dtype, n)
    rng = np.random.default_rng(n)
    probs = []
    for b, s in ((16, 32), (16, 17), (8, 48), (12, 25)):
        d = b * s + 5
        X = rng.integers(-3, 4, (d, n)).astype(np.float64)
        y = rng.integers(-8, 9, n).astype(np.float64)
        code = gpu_lib.BF16 if dtype == "bf16" else gpu_lib.FP8_E4M3
        view = torch.bfloat16 if dtype == "bf16" else torch.float8_e4m3fn
        codes = torch.tensor(X, dtype=torch.float32, device=DEV).to(view).contiguous()
        codes = codes.view(torch.int16 if dtype == "bf16" else torch.uint8)
        Q = gpu_lib.Quantized(codes, torch.ones(d, dtype=torch.float32, device=DEV), code)
        assert np.array_equal(Q.dequantize().cpu().numpy(), X)
        probs.append(dict(X=Q, y=torch.tensor(y, device=DEV), lam=1.0, b=b, s=s, seed=n + b,
                          H=s, Xc=X, yc=y))
    act, infos = _run(gpu_lib, probs, [1], monitor_every=0)
    assert act == 0
    for q in probs:
        wo, zo = bcd.primal_bcd(q["Xc"], q["yc"], q["lam"], q["b"], q["s"], q["H"], q["seed"])
        assert np.linalg.norm(q["w"].cpu().numpy() - wo) <= 1e-11 * np.linalg.norm(wo)
        ro = zo - q["yc"]
        assert np.linalg.norm(q["r"].cpu().numpy() - ro) <= 1e-11 * np.linalg.norm(ro)


@pytest.mark.parametrize("d,n,b,s", [(1024, 66001, 8, 16), (12, 400001, 4, 2), (300, 30001, 16, 16)])
def test_batch_monitors_of_many_slabs(gpu_lib, d, n, b, s):
    """Objectives of exact and maintained monitor points whose slabs are more than a
    workgroup's threads or only a few, and of a run that ends on a pending update."""
    _say("batch monitor slabs", d, n, b, s)
    X, y, _ = synth.gaussian_ridge(d, n, n)
    Xd, yd = X.to(DEV), y.to(DEV)
    q = dict(X=Xd, y=yd, lam=0.05, b=b, s=s, seed=5, H=0)
    with gpu_lib.Batch([q], monitor_every=1, cheap_monitors=2) as B:
        for _ in range(4):
            B.run(1)
            r = Xd.t() @ q["w"] - yd
            f = float(r @ r) / (2 * n) + 0.025 * float(q["w"] @ q["w"])
            assert abs(B.info(0)["objective"] - f) <= 1e-12 * f
            assert float((q["r"] - r).norm()) <= 1e-12 * float(r.norm())
    with gpu_lib.Batch([q], monitor_every=0) as B:
        B.run(3)
    r = Xd.t() @ q["w"] - yd
    assert float((q["r"] - r).norm()) <= 1e-12 * float(r.norm())
