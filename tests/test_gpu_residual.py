"""GPU residual and Jv (through the C ABI) against the FP64 CPU oracle."""
import numpy as np
import pytest

from paper_1709_08803_amd import workloads as W
from oracle import residual as R

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def bim():
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    from paper_1709_08803_amd import bim as B
    B.lib()
    return B


def _gpu_F(B, p, u, prec):
    dp = B.DeviceProblem(p)
    ud = torch.as_tensor(u, device="cuda")
    F = B.residual(dp, ud, prec=prec)
    torch.cuda.synchronize()
    return F.cpu().numpy()


CASES = [
    ("tiny-31x11", lambda: W.tiny(0.7), 1),
    ("61x21-F1.4", lambda: W.working(1.4, N=61, M=21), 2),
    ("ragged-45x9", lambda: W.make_problem(45, 9, -12, 12, 0, 6, 0.9, [W.Bump(0.25, 1.3, 0.9)]), 3),
    ("full-31x13", lambda: W.make_problem(31, 13, -10, 10, -6, 6, 1.2, [W.Bump(0.2, 1.0, 1.0, cy=1.5)],
                                          half_domain=False), 4),
    ("min-3x3", lambda: W.make_problem(3, 3, -1, 1, 0, 1, 0.8, [W.Bump(0.1, 1.0, 1.0)]), 5),
    # a full domain whose y_1 = -30 is not 0 (edge rows through the rectangle's corners)
    ("full-61x61-offset", lambda: W.make_problem(61, 61, -7, 53, -30, 30, 0.6,
                                                 [W.Bump(0.2, 0.71, 0.71, cx=10.0, cy=10.0),
                                                  W.Bump(0.2, 0.71, 0.71, cx=0.0, cy=-10.0)], half_domain=False), 6),
    # surface tension (Section 6): the curvature term of the dynamic rows
    ("tension-31x11", lambda: W.make_problem(31, 11, -16, 16, 0, 10, 1.4, [W.Bump(0.1, 1.0, 1.0)], tau=0.1), 7),
    ("tension-full-31x13", lambda: W.make_problem(31, 13, -10, 10, -6, 6, 1.2, [W.Bump(0.2, 1.0, 1.0, cy=1.5)],
                                                  half_domain=False, tau=0.05), 8),
]


@pytest.mark.parametrize("name,mk,seed", CASES, ids=[c[0] for c in CASES])
def test_residual_fp64_matches_oracle(bim, name, mk, seed):
    p = mk()
    u = W.perturbed_state(p, seed)
    F_ref = R.residual(p, u)
    scale = R.term_magnitude_rows(p, u)
    F = _gpu_F(bim, p, u, "fp64")
    err = np.abs(F - F_ref) / scale
    print(name, "max rel err", err.max())
    assert err.max() <= 1e-12


# The FP64 S2 sums in segments and node by node (from about 10^7 targets times lattice
# nodes on: segments), rows shorter than the segments' reach and too long for the
# fused records, whole and partly filled tiles, two rows per lane; slopes up to ~2.
S2_CASES = [
    (91, 31, True, 1.0), (91, 31, True, 12.0),   # segments, gentle and steep
    (81, 27, True, 12.0),                        # node by node, just below the line
    (65, 45, True, 3.0),                         # rows of 64 targets
    (67, 67, False, 8.0),                        # full domain, two rows per lane, odd row count
    (60, 59, False, 1.0),                        # full domain, one row per lane
    (3, 900, True, 3.0), (3, 700, True, 3.0),    # shortest rows
    (1200, 3, True, 3.0),                        # fewest rows, longer than the fused records take
]


def _s2_integral_extended(A, B, C, s1, s2, t1, t2):
    """The oracle's closed form in extended precision: on strips far longer than wide
    its logarithms cancel (5e-12 of the row's terms at 3 x 900 in FP64)."""
    A, B, C, s1, s2, t1, t2 = (np.asarray(v, dtype=np.longdouble) for v in (A, B, C, s1, s2, t1, t2))

    def G(s, t):
        with np.errstate(divide="ignore", invalid="ignore"):
            Q = A * s * s + B * s * t + C * t * t
            a1 = t / np.sqrt(A) * np.log(2 * A * s + B * t + 2 * np.sqrt(A * Q))
            a2 = s / np.sqrt(C) * np.log(2 * C * t + B * s + 2 * np.sqrt(C * Q))
        return np.where(t == 0, 0, a1) + np.where(s == 0, 0, a2)

    return (G(s2, t2) - G(s1, t2) - G(s2, t1) + G(s1, t1)).astype(np.float64)


@pytest.mark.parametrize("N,M,half,steep", S2_CASES)
def test_residual_fp64_s2_routes_match_oracle(bim, monkeypatch, N, M, half, steep):
    monkeypatch.setattr(R, "s2_integral", _s2_integral_extended)
    L, Ly = 0.25 * (N - 1) / 2, 0.3 * (M - 1)
    p = W.make_problem(N, M, -L, L, 0 if half else -0.4 * Ly, Ly if half else 0.6 * Ly, 0.9,
                       [W.Bump(0.2, 1.0, 1.0, cy=0.0 if half else 0.5)], half_domain=half)
    u = W.perturbed_state(p, 21)
    nb = (N + 1) * M
    u[:nb] *= steep  # elevation and its slopes
    err = np.abs(_gpu_F(bim, p, u, "fp64") - R.residual(p, u)) / R.term_magnitude_rows(p, u)
    print(N, M, "max slope", np.abs(u[:nb]).max(), "max rel err", err.max())
    # as the tolerance of the other FP64 cases: rounding of the row's terms, each a few
    # units in the last place, over sums of up to 10^4
    assert err.max() <= 1e-12


# Slopes far beyond any solution's, where the products of the segments' ratios would leave
# the FP64 range (from about 2800 on with 16 or more rows per chunk), up to and past the
# slope from which targets are summed node by node, and one source chunk (all rows in one
# product, as the allocation-free entry point may run)
@pytest.mark.parametrize("N,M,half,slope,chunks", [(281, 141, True, 3e3, 0), (281, 141, True, 3e4, 0),
                                                   (281, 141, True, 3e6, 0), (151, 300, False, 1e4, 0),
                                                   (151, 100, False, 500.0, 1)])
def test_residual_fp64_steep_surfaces(bim, monkeypatch, N, M, half, slope, chunks):
    import ctypes
    monkeypatch.setattr(R, "s2_integral", _s2_integral_extended)
    L, Ly = 0.05 * (N - 1), 0.1 * (M - 1)
    p = W.make_problem(N, M, -L, L, 0 if half else -0.5 * Ly, Ly if half else 0.5 * Ly, 0.9, [W.Bump(0.2, 1.0, 1.0)],
                       half_domain=half)
    u = W.perturbed_state(p, 21)
    nb = (N + 1) * M
    nf = R.reconstruct(p, u)
    u[:nb] *= slope / max(np.abs(nf.zeta_x).max(), np.abs(nf.zeta_y).max())
    nf = R.reconstruct(p, u)
    zx, zy = R.half_mesh(nf.zeta_x), R.half_mesh(nf.zeta_y)
    steep = np.argsort((zx * zx + zy * zy).reshape(-1))[-40:]  # the steepest targets, and some others
    rng = np.random.default_rng(3)
    some = np.concatenate([steep, rng.choice((N - 1) * M, 60, replace=False)])
    rows = np.unique([R.row_index(p, b, i // (N - 1), i % (N - 1)) for i in some for b in (1, 2)])
    dp = bim.DeviceProblem(p)
    ud = torch.as_tensor(u, device="cuda")
    Fd = torch.empty_like(ud)
    k, t = ctypes.c_double(), ctypes.c_double()
    cfg = ctypes.byref(bim.PairConfig(1, 4, 0, chunks)) if chunks else None
    assert bim.lib().bim_residual_timed(dp.ref(), ud.data_ptr(), Fd.data_ptr(), bim._PREC["fp64"], 1, cfg,
                                        torch.cuda.current_stream().cuda_stream, ctypes.byref(k), ctypes.byref(t)) == 0
    F = Fd.cpu().numpy()
    assert np.isfinite(F).all()
    err = np.abs(F[rows] - R.residual_rows(p, u, rows)) / R.term_magnitude_rows(p, u, rows)
    print(N, M, "max slopes", np.abs(zx).max(), np.abs(zy).max(), "max rel err", err.max())
    # along its valley a form is up to A + C times smaller than its terms, which hold the
    # rounding of A, B, C (one unit each) and of the products (a few)
    assert err.max() <= 1e-12 + 8 * 2.0 ** -52 * (2.0 + zx * zx + zy * zy).max()


@pytest.mark.parametrize("name,mk,seed", CASES[:4], ids=[c[0] for c in CASES[:4]])
def test_residual_fp32c_matches_oracle(bim, name, mk, seed):
    p = mk()
    u = W.perturbed_state(p, seed)
    F_ref = R.residual(p, u)
    scale = R.term_magnitude_rows(p, u)
    F = _gpu_F(bim, p, u, "fp32c")
    err = np.abs(F - F_ref) / scale
    print(name, "fp32c max rel err", err.max())
    assert err.max() <= 5e-7


def test_residual_fp32c_full_size_against_fp64(bim):
    # 181 x 61 (|x| up to 30): the FP32C sums against the FP64 ones, per row
    # relative to the row's sum of term magnitudes (computed by the oracle)
    p = W.working(1.4)
    u = W.perturbed_state(p, 11)
    F64 = _gpu_F(bim, p, u, "fp64")
    F32 = _gpu_F(bim, p, u, "fp32c")
    scale = R.term_magnitude_rows(p, u)
    err = np.abs(F32 - F64) / scale
    print("181x61 fp32c max rel err", err.max(), "median", np.median(err))
    assert err.max() <= 5e-7


@pytest.mark.parametrize("F_num", [0.7, 1.4])
def test_residual_full_size_sampled_rows(bim, F_num):
    # 181 x 61 at the benchmark's launch configuration; the oracle computes a
    # seeded sample of rows one by one (all row kinds, edges included).
    p = W.working(F_num)
    u = W.perturbed_state(p, 11)
    rng = np.random.default_rng(7)
    nb = (p.N + 1) * p.M
    rows = set(rng.choice(3 * nb, 150, replace=False).tolist())
    for blk in range(3):  # corners and edges of every block
        for l in (0, p.M - 1):
            rows.update({blk * nb + l * (p.N + 1) + c for c in (0, 1, 2, p.N)})
    rows = np.array(sorted(rows))
    ref = R.residual_rows(p, u, rows)
    F = _gpu_F(bim, p, u, "fp64")
    F32 = _gpu_F(bim, p, u, "fp32c")
    scale = R.term_magnitude_rows(p, u)[rows]
    e64 = (np.abs(F[rows] - ref) / scale).max()
    e32 = (np.abs(F32[rows] - ref) / scale).max()
    print("181x61 F", F_num, "fp64", e64, "fp32c", e32)
    assert e64 <= 1e-12
    assert e32 <= 5e-7


def test_residual_is_deterministic(bim):
    p = W.working(0.7, N=61, M=21)
    u = W.perturbed_state(p, 1)
    a = _gpu_F(bim, p, u, "fp64")
    b = _gpu_F(bim, p, u, "fp64")
    assert np.array_equal(a, b)
    c = _gpu_F(bim, p, u, "fp32c")
    d = _gpu_F(bim, p, u, "fp32c")
    assert np.array_equal(c, d)


def test_uniform_stream_flat_bottom_is_zero_on_gpu(bim):
    p = W.make_problem(61, 21, -20, 20, 0, 10, 0.7, [])
    F = _gpu_F(bim, p, W.uniform_stream(p), "fp64")
    assert np.abs(F).max() < 1e-12


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-7), ("fp32c", 2e-2)])
def test_jv_matches_oracle_difference_quotient(bim, prec, tol):
    p = W.tiny(0.7)
    u = W.perturbed_state(p, 2)
    v = W.random_direction(p, 3) * 1e-2
    h = 1e-3 if prec == "fp64" else 1e-1
    ref = (R.residual(p, u + h * v) - R.residual(p, u)) / h
    dp = bim.DeviceProblem(p)
    ud, vd = torch.as_tensor(u, device="cuda"), torch.as_tensor(v, device="cuda")
    Fu = bim.residual(dp, ud, prec=prec)
    J = bim.jv(dp, ud, Fu, vd, h=h, prec=prec)
    torch.cuda.synchronize()
    J = J.cpu().numpy()
    err = np.abs(J - ref).max() / np.abs(ref).max()
    print(prec, "jv rel err", err)
    assert err <= tol


def test_jv_full_size_sampled_rows(bim):
    # 181 x 61 (F = 0.7), the quotient (F(u + h v) - F(u)) / h on sampled rows of
    # every kind against the oracle's rows, FP64 within 1e-7 of the largest entry
    p = W.working(0.7)
    u = W.perturbed_state(p, 4)
    v = W.random_direction(p, 5) * 1e-2
    h = 1e-3
    rng = np.random.default_rng(9)
    rows = np.unique(np.concatenate([rng.choice(p.n_unknowns, 300, replace=False),
                                     [R.row_index(p, b, l, k) for b in (0, 1, 2) for l in (0, p.M - 1)
                                      for k in (0, p.N - 2)]]))
    ref = (R.residual_rows(p, u + h * v, rows) - R.residual_rows(p, u, rows)) / h
    dp = bim.DeviceProblem(p)
    ud, vd = torch.as_tensor(u, device="cuda"), torch.as_tensor(v, device="cuda")
    Fu = bim.residual(dp, ud)
    J = bim.jv(dp, ud, Fu, vd, h=h).cpu().numpy()[rows]
    err = np.abs(J - ref).max() / np.abs(ref).max()
    print("181x61 fp64 jv rel err on", rows.size, "rows", err)
    assert err <= 1e-7


def test_jv_default_shift_and_zero_direction(bim):
    p = W.tiny(0.7)
    u = W.perturbed_state(p, 2)
    dp = bim.DeviceProblem(p)
    ud = torch.as_tensor(u, device="cuda")
    Fu = bim.residual(dp, ud)
    z = torch.zeros_like(ud)
    J = bim.jv(dp, ud, Fu, z)  # |v| = 0 -> Jv = 0
    torch.cuda.synchronize()
    assert torch.count_nonzero(J).item() == 0
    v = W.random_direction(p, 3)
    J = bim.jv(dp, ud, Fu, torch.as_tensor(v, device="cuda"))  # default h rule
    eps = 2.0 ** -52
    h = np.sqrt(eps) * (1 + np.linalg.norm(u)) / np.linalg.norm(v)
    ref = (R.residual(p, u + h * v) - R.residual(p, u)) / h
    torch.cuda.synchronize()
    err = np.abs(J.cpu().numpy() - ref).max() / np.abs(ref).max()
    assert err < 1e-4


VARIANTS = [(tpl, unr, rpc) for tpl in (1, 2) for unr in (2, 4, 8) for rpc in (1, 3)]
# explicit chunk counts at 45 x 9 (2 M N = 810 source nodes): ranges that start
# and end inside rows, down to one node per chunk, and one chunk for everything
VARIANTS += [(1, 2, 0, 7), (2, 4, 0, 13), (1, 8, 0, 50), (1, 4, 0, 810), (2, 2, 0, 1), (1, 4, 0, 0), (2, 8, 0, 0)]


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32c", 5e-7)])
def test_every_launch_variant_matches_oracle(bim, prec, tol):
    # the autotuner may pick any of these; all must meet the same bar
    p = W.make_problem(45, 9, -12, 12, 0, 6, 0.9, [W.Bump(0.25, 1.3, 0.9)])  # M odd: a lone last row pair
    u = W.perturbed_state(p, 3)
    F_ref = R.residual(p, u)
    scale = R.term_magnitude_rows(p, u)
    dp = bim.DeviceProblem(p)
    ud = torch.as_tensor(u, device="cuda")
    for cfg in VARIANTS:
        F = torch.empty_like(ud)
        bim.lib()  # loaded
        k, t = bim.residual_timed(dp, ud, prec, iters=1, config=cfg)
        # residual_timed writes into a scratch F; evaluate through the public path with the same shape
        import ctypes
        Fd = torch.empty_like(ud)
        kk, tt = ctypes.c_double(), ctypes.c_double()
        rc = bim.lib().bim_residual_timed(dp.ref(), ud.data_ptr(), Fd.data_ptr(), bim._PREC[prec], 1,
                                          ctypes.byref(bim.PairConfig(*cfg)), torch.cuda.current_stream().cuda_stream,
                                          ctypes.byref(kk), ctypes.byref(tt))
        assert rc == 0
        err = (np.abs(Fd.cpu().numpy() - F_ref) / scale).max()
        assert err <= tol, (cfg, err)


def test_autotuner_choice_is_used_and_correct(bim):
    p = W.working(0.7, N=61, M=21)
    u = W.perturbed_state(p, 4)
    dp = bim.DeviceProblem(p)
    ud = torch.as_tensor(u, device="cuda")
    best, ms = bim.tune_residual(dp, ud, "fp64")
    assert best[0] in (1, 2) and best[1] in (2, 4, 8) and ms > 0
    F = bim.residual(dp, ud, "fp64")
    torch.cuda.synchronize()
    F_ref = R.residual(p, u)
    scale = R.term_magnitude_rows(p, u)
    assert (np.abs(F.cpu().numpy() - F_ref) / scale).max() <= 1e-12


def test_workspace_reuse_across_sizes_streams_and_release(bim):
    """The per-stream workspace of residual() and jv(): a larger problem grows it,
    a smaller one reuses it, another stream gets its own, and after a release the
    next call allocates again; every result equals the first evaluation bit for bit."""
    small = W.tiny(0.7)
    big = W.working(1.4, N=61, M=21)
    cases = {}
    for name, p in (("small", small), ("big", big)):
        dp = bim.DeviceProblem(p)
        u = torch.as_tensor(W.perturbed_state(p, 7), device="cuda")
        cases[name] = (dp, u)
    bim.release_workspaces()
    ref = {k: bim.residual(dp, u).cpu().numpy() for k, (dp, u) in cases.items()}  # small first, then grow
    side = torch.cuda.Stream()
    for order in (("small", "big", "small"), ("big", "small")):
        for k in order:
            dp, u = cases[k]
            assert np.array_equal(bim.residual(dp, u).cpu().numpy(), ref[k]), k
            with torch.cuda.stream(side):
                F = bim.residual(dp, u, stream=side)
            side.synchronize()
            assert np.array_equal(F.cpu().numpy(), ref[k]), (k, "side stream")
        bim.release_workspaces()
    dp, u = cases["small"]
    F0 = bim.residual(dp, u)
    v = torch.ones_like(u)
    J1 = bim.jv(dp, u, F0, v, h=1e-7)
    J2 = bim.jv(dp, u, F0, v, h=1e-7)
    assert torch.equal(J1, J2)
    bim.release_workspaces()


def test_residual_large_mesh_sampled_rows(bim):
    # 541 x 181 (three times finer than the working mesh on the same domain;
    # 9.5e10 pairs per evaluation, 9x the working size) at the default launch
    # shape: a seeded sample of rows, edges and corners included, against the
    # oracle row by row
    p = W.working(1.4, N=541, M=181)
    u = W.perturbed_state(p, 5)
    rng = np.random.default_rng(9)
    nb = (p.N + 1) * p.M
    rows = set(rng.choice(3 * nb, 60, replace=False).tolist())
    for blk in range(3):
        for l in (0, p.M - 1):
            rows.update({blk * nb + l * (p.N + 1) + c for c in (0, 2, p.N)})
    rows = np.array(sorted(rows))
    ref = R.residual_rows(p, u, rows)
    scale = R.term_magnitude_rows(p, u, rows)
    F = _gpu_F(bim, p, u, "fp64")
    F32 = _gpu_F(bim, p, u, "fp32c")
    e64 = (np.abs(F[rows] - ref) / scale).max()
    e32 = (np.abs(F32[rows] - ref) / scale).max()
    print("541x181 fp64", e64, "fp32c", e32)
    assert e64 <= 1e-12
    assert e32 <= 5e-7


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32c", 5e-7)])
@pytest.mark.parametrize("name,mk,seed", CASES, ids=[c[0] for c in CASES])
def test_linear_residual_matches_oracle(bim, name, mk, seed, prec, tol):
    # the linearised residual of Section 4.2 (flat-plane kernel bodies on the
    # GPU) against the oracle's affine form J~ (u - u0) + F_lin(u0), on the
    # half-domain, ragged, full-domain (one image) and minimal meshes; rows are
    # scaled by the nonlinear residual's term magnitudes at the same state
    from oracle import linear as Lin
    p = mk()
    u = W.perturbed_state(p, seed)
    F_ref = Lin.F_lin(p, u)
    scale = R.term_magnitude_rows(p, u)
    dp = bim.DeviceProblem(p)
    F = bim.residual_linear(dp, torch.as_tensor(u, device="cuda"), prec=prec)
    torch.cuda.synchronize()
    err = np.abs(F.cpu().numpy() - F_ref) / scale
    print(name, prec, "linear residual max rel err", err.max())
    assert err.max() <= tol


# The FP64 linear sums are convolutions with kernel tables: R = 1 .. 4 targets per lane (N - 1
# at and past multiples of 64), two blocks of targets, slices of more than one table window
# (N > 256), the smallest mesh, one and several source chunks, both domains
@pytest.mark.parametrize("N,M,half", [(3, 3, True), (65, 3, True), (66, 5, False), (129, 4, True), (130, 3, False),
                                      (193, 3, True), (194, 3, True), (257, 3, False), (300, 3, True)])
def test_linear_convolutions_match_oracle(bim, N, M, half):
    from oracle import linear as Lin
    x, y = (N - 1) / 6.0, (M - 1) / 3.0
    p = W.make_problem(N, M, -x, x, 0.0 if half else -y, y, 0.8, [W.Bump(0.2, 1.1, 0.9, cx=0.3)], half_domain=half)
    u = W.perturbed_state(p, 3)
    F_ref = Lin.F_lin(p, u)
    scale = R.term_magnitude_rows(p, u)
    F = bim.residual_linear(bim.DeviceProblem(p), torch.as_tensor(u, device="cuda"))
    torch.cuda.synchronize()
    err = (np.abs(F.cpu().numpy() - F_ref) / scale).max()
    print(f"{N}x{M}", err)
    assert err <= 1e-12


# Beside the smallest meshes that are summed as convolutions (by nodes and by row length), and
# the pairwise form on their other side
@pytest.mark.parametrize("N,M,half", [(65, 6, True), (66, 6, False), (31, 12, True), (31, 11, True), (24, 32, True),
                                      (24, 31, True), (26, 31, False), (25, 33, False), (18, 43, True), (17, 46, True)])
def test_linear_sums_beside_the_convolution_line(bim, N, M, half):
    from oracle import linear as Lin
    x, y = (N - 1) / 6.0, (M - 1) / 3.0
    p = W.make_problem(N, M, -x, x, 0.0 if half else -y, y, 0.8, [W.Bump(0.2, 1.1, 0.9, cx=0.3)], half_domain=half)
    u = W.perturbed_state(p, 3)
    F = bim.residual_linear(bim.DeviceProblem(p), torch.as_tensor(u, device="cuda"))
    err = (np.abs(F.cpu().numpy() - Lin.F_lin(p, u)) / R.term_magnitude_rows(p, u)).max()
    print(f"{N}x{M}", err)
    assert err <= 1e-12


def _best_us(fn, reps=20):
    import time
    fn()
    best = float("inf")
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(reps):
            fn()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) / reps * 1e6)
    return best


# On narrow meshes the convolution form took up to ten times the pairwise one (3 x 900: 583
# against 60 us; F(u) itself takes 58)
@pytest.mark.parametrize("N,M,half", [(3, 900, True), (5, 900, False), (8, 900, False)])
def test_linear_residual_of_narrow_meshes_is_no_slower_than_the_nonlinear_one(bim, N, M, half):
    L, Ly = (N - 1) / 2.0, float(M - 1)
    p = W.make_problem(N, M, -L, L, 0 if half else -0.5 * Ly, Ly if half else 0.5 * Ly, 0.9, [W.Bump(0.2, 1.0, 1.0)],
                       half_domain=half)
    dp = bim.DeviceProblem(p)
    u = torch.as_tensor(W.perturbed_state(p, 3), device="cuda")
    out = torch.empty_like(u)
    lin, non = _best_us(lambda: bim.residual_linear(dp, u, out=out)), _best_us(lambda: bim.residual(dp, u, out=out))
    print(N, M, "linear", lin, "nonlinear", non)
    assert lin <= 2.0 * non


# The S2 sums of short rows cost less node by node than in segments (3 x 900 58 against 101
# us, with FP32C 54): both sides of the line against the oracle, and no longer the slower one
@pytest.mark.parametrize("N,M,half", [(12, 730, True), (12, 736, True), (24, 183, True), (24, 186, True),
                                      (31, 154, False), (31, 157, False)])
def test_residual_fp64_s2_routes_of_short_rows_match_oracle(bim, monkeypatch, N, M, half):
    test_residual_fp64_s2_routes_match_oracle(bim, monkeypatch, N, M, half, 3.0)


@pytest.mark.parametrize("N,M", [(3, 900), (5, 500)])
def test_residual_fp64_of_short_rows_keeps_near_the_fp32c_one(bim, N, M):
    p = W.make_problem(N, M, -0.5 * (N - 1), 0.5 * (N - 1), 0, float(M - 1), 0.9, [W.Bump(0.2, 1.0, 1.0)])
    dp = bim.DeviceProblem(p)
    u = torch.as_tensor(W.perturbed_state(p, 3), device="cuda")
    out = torch.empty_like(u)
    t64, t32 = _best_us(lambda: bim.residual(dp, u, out=out)), _best_us(lambda: bim.residual(dp, u, "fp32c", out=out))
    print(N, M, "fp64", t64, "fp32c", t32)
    assert t64 <= 1.35 * t32


def test_tuned_batch_and_single_launches_match_oracle(bim):
    # FP64 tunes the kernels of one problem and those of a batch separately; each then runs its own
    # choice (a batch takes that of its largest problem)
    ps = [W.make_problem(45, 15, -12, 12, 0, 6, 0.9, [W.Bump(0.25, 1.3, 0.9)]),
          W.make_problem(31, 13, -10, 10, -6, 6, 1.2, [W.Bump(0.2, 1.0, 1.0, cy=1.5)], half_domain=False)]
    us = [W.perturbed_state(p, 5) for p in ps]
    dps = [bim.DeviceProblem(p) for p in ps]
    uds = [torch.as_tensor(u, device="cuda") for u in us]
    before = [F.cpu().numpy() for F in bim.residual_batched(dps, uds, "fp64")]
    for dp, u in zip(dps, uds):
        best, ms = bim.tune_residual(dp, u, "fp64")
        assert best[0] in (1, 2) and best[1] in (2, 4, 8) and ms > 0
    after = [F.cpu().numpy() for F in bim.residual_batched(dps, uds, "fp64")]
    for i, (p, u) in enumerate(zip(ps, us)):
        ref, scale = R.residual(p, u), R.term_magnitude_rows(p, u)
        for F in (before[i], after[i], bim.residual(dps[i], uds[i]).cpu().numpy()):
            assert (np.abs(F - ref) / scale).max() <= 1e-12


def _bie_rows_extended(p, u, which, idx):
    """Boundary-integral rows `idx` of one boundary ("S" or "B") in extended precision: the oracle's
    steps with every value in numpy's long double."""
    E = np.longdouble
    N, M, dx, dy = p.N, p.M, E(p.dx), E(p.dy)
    x, y = E(p.x1) + dx * np.arange(N), E(p.y1) + dy * np.arange(M)

    def field(f):
        blk = u[f * (N + 1) * M:(f + 1) * (N + 1) * M].reshape(M, N + 1).astype(E)
        inc = 0.5 * dx * (blk[:, 1:-1] + blk[:, 2:])
        return blk[:, :1] + np.concatenate([np.zeros((M, 1), E), np.cumsum(inc, axis=1)], axis=1), blk[:, 1:]

    (zeta, zx), (phi, _), (psi, _) = field(0), field(1), field(2)
    zy = np.empty_like(zeta)
    zy[1:-1] = (zeta[2:] - zeta[:-2]) / (2 * dy)
    zy[-1] = (3 * zeta[-1] - 4 * zeta[-2] + zeta[-3]) / (2 * dy)
    zy[0] = 0 if p.half_domain else (-3 * zeta[0] + 4 * zeta[1] - zeta[2]) / (2 * dy)
    b, bx, by = (a.astype(E) for a in (p.beta, p.beta_x, p.beta_y))
    end = lambda n: np.where((np.arange(n) == 0) | (np.arange(n) == n - 1), E(0.5), E(1))
    w = dx * dy * end(M)[:, None] * end(N)[None]
    layers = (("S", zeta, zx, zy, phi - x, zx, 1), ("B", b, bx, by, psi - x, bx, -1))
    _, a, ax, ay, D, sig, sign = layers["SB".index(which)]
    mid = lambda g, l, k: 0.5 * (g[l, k] + g[l, k + 1])
    out = []
    for i in idx:
        l, k = divmod(int(i), N - 1)
        xs, ys, d, Ds, gx, gy = x[k] + 0.5 * dx, y[l], mid(a, l, k), mid(D, l, k), mid(ax, l, k), mid(ay, l, k)
        ss = sign * mid(sig, l, k)
        A, B, C = 1 + gx * gx, 2 * gx * gy, 1 + gy * gy
        v = E(0)
        for image in (1, -1) if p.half_domain else (1,):
            s, t = (x - xs)[None], (image * y - ys)[:, None]
            for name, h, hx, hy, Dn, sn, sg in layers:
                dz = h - d
                ri = 1 / np.sqrt(s * s + t * t + dz * dz)
                v += (sg * w * ((Dn - (Ds if name == which else 0)) * (dz - s * hx - image * t * hy) * ri ** 3
                                + sn * ri)).sum()
            v -= ss * (w / np.sqrt(A * s * s + B * s * t + C * t * t)).sum()

        def G(s, t):
            Q = A * s * s + B * s * t + C * t * t
            g = t / np.sqrt(A) * np.log(2 * A * s + B * t + 2 * np.sqrt(A * Q)) if t != 0 else E(0)
            return g + (s / np.sqrt(C) * np.log(2 * C * t + B * s + 2 * np.sqrt(C * Q)) if s != 0 else E(0))

        s1, s2, t1, t2 = x[0] - xs, x[-1] - xs, (-y[-1] if p.half_domain else y[0]) - ys, y[-1] - ys
        v += ss * (G(s2, t2) - G(s1, t2) - G(s2, t1) + G(s1, t1)) - E("6.283185307179586476925287") * Ds
        out.append(v)
    return np.array(out)


@pytest.mark.parametrize("N,M,half", [(31, 11, True), (61, 21, True), (70, 40, False)])
def test_fp64_rows_are_no_further_from_extended_precision_than_the_batched_ones(bim, N, M, half):
    # a row's error is mostly the rounding of node values; the one-launch form of one problem forms
    # them in its own order, the batched kernels in that of a plain scan
    p = W.working(0.7, N=N, M=M) if half else W.make_problem(N, M, -10, 20, -10, 10, 0.7, [W.Bump(0.2, 1.0, 1.0)],
                                                             half_domain=False)
    dp = bim.DeviceProblem(p)
    err = {"single": [], "batched": []}
    for seed in range(5):
        u = W.perturbed_state(p, seed)
        ud = torch.as_tensor(u, device="cuda")
        F = {"single": bim.residual(dp, ud).cpu().numpy(), "batched": bim.residual_batched([dp], [ud])[0].cpu().numpy()}
        for block, which in ((1, "S"), (2, "B")):
            idx = np.random.default_rng(seed).choice((N - 1) * M, 60, replace=False)
            ref = _bie_rows_extended(p, u, which, idx)
            rows = [R.row_index(p, block, i // (N - 1), i % (N - 1)) for i in idx]
            for k in F:
                err[k] += [float(e) for e in F[k][rows] - ref]
    rms = {k: float(np.sqrt(np.mean(np.square(v)))) for k, v in err.items()}
    print(N, M, rms)
    assert rms["batched"] < 1e-12  # the reference is the same system
    assert rms["single"] <= rms["batched"]
