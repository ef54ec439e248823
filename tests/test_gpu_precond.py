"""GPU block-banded preconditioner (through the C ABI) against the oracle's P."""
import numpy as np
import pytest

from paper_1709_08803_amd import workloads as W
from oracle import linear as Lin

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def bim():
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    from paper_1709_08803_amd import bim as B
    B.lib()
    return B


CASES = [
    ("tiny-31x11-default", lambda: W.tiny(0.7), -1),
    ("tiny-31x11-h1", lambda: W.tiny(0.7), 1),
    ("31x11-h2", lambda: W.tiny(1.4), 2),
    ("61x21-h1", lambda: W.working(0.7, N=61, M=21), 1),
    ("61x21-default", lambda: W.working(0.7, N=61, M=21), -1),
    ("ragged-45x9-h3", lambda: W.make_problem(45, 9, -12, 12, 0, 6, 0.9, [W.Bump(0.25, 1.3, 0.9)]), 3),
    ("full-31x13", lambda: W.make_problem(31, 13, -10, 10, -6, 6, 1.2, [], half_domain=False), 1),
    # surface tension: P is the preconditioner of the problem without it
    ("tension-31x11-h2", lambda: W.make_problem(31, 11, -16, 16, 0, 10, 1.4, [W.Bump(0.1, 1.0, 1.0)], tau=0.1), 2),
    ("tension-full-31x13", lambda: W.make_problem(31, 13, -10, 10, -6, 6, 1.2, [], half_domain=False, tau=0.05), 1),
    # pivot blocks of s = N + 1 = 192, the largest the register inversion holds
    ("max-block-191x5-h1", lambda: W.make_problem(191, 5, -20, 20, 0, 1, 0.9, [W.Bump(0.25, 1.3, 0.9)]), 1),
    # s = 193, 212, 300: blocks beyond the register kernel, inverted as 2 x 2 block matrices
    # (the leading 192 block and the Schur complement in registers, the rest on the matrix cores)
    ("split-block-192x5-h1", lambda: W.make_problem(192, 5, -20, 20, 0, 1, 0.9, [W.Bump(0.25, 1.3, 0.9)]), 1),
    ("split-block-211x5-h1", lambda: W.make_problem(211, 5, -40, 30, 0, 1, 0.7, [W.Bump(0.2, 1.0, 1.0)]), 1),
    ("split-block-299x5-h2", lambda: W.make_problem(299, 5, -30, 30, 0, 2, 1.2, [W.Bump(0.2, 1.0, 1.0)]), 2),
    # s = 385: the augmented-matrix Gauss-Jordan kernel beyond that
    ("big-block-384x5-h1", lambda: W.make_problem(384, 5, -40, 40, 0, 1, 0.9, [W.Bump(0.25, 1.3, 0.9)]), 1),
]


@pytest.mark.parametrize("name,mk,hb", CASES, ids=[c[0] for c in CASES])
def test_precond_apply_matches_oracle_solve(bim, name, mk, hb):
    p = mk()
    dp = bim.DeviceProblem(p)
    P = bim.Preconditioner(dp, hb)
    if hb < 0:  # the library's default band: max(1, min(10, round(M / 6))) slices
        assert P.band == max(1, min(10, round(p.M / 6)))
    pc_ref = Lin.Preconditioner(p, hb=P.band)
    rng = np.random.default_rng(5)
    for trial in range(2):
        r = rng.standard_normal(p.n_unknowns)
        z_ref = pc_ref.apply(r)
        z = P.apply(torch.as_tensor(r, device="cuda"))
        torch.cuda.synchronize()
        err = np.abs(z.cpu().numpy() - z_ref).max() / np.abs(z_ref).max()
        print(name, "precond rel err", err)
        # the diagonal blocks' conditioning grows with N (their trapezoidal x-integration
        # recurrences): 1e-9 for the 385-wide blocks, 1e-10 up to 300
        assert err <= (1e-10 if p.N + 1 <= 300 else 1e-9)
    P.close()


# Block sizes s = N + 1 at the edges of the setup's tiles: registers of the pivot inversion
# (rows in steps of 32, columns of 64), row panels of the substitutions (64, 128, 192) and
# K steps of 16 and 32 in the products, with K-blocks that end inside a step
@pytest.mark.parametrize("s", [4, 17, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129, 144, 160, 161])
def test_precond_block_sizes_match_oracle_solve(bim, s):
    p = W.make_problem(s - 1, 7, -0.15 * s, 0.15 * s, 0, 2, 0.9, [W.Bump(0.25, 1.3, 0.9)])
    P = bim.Preconditioner(bim.DeviceProblem(p), 2)
    r = np.random.default_rng(s).standard_normal(p.n_unknowns)
    z_ref = Lin.Preconditioner(p, hb=2).apply(r)
    z = P.apply(torch.as_tensor(r, device="cuda")).cpu().numpy()
    err = np.abs(z - z_ref).max() / np.abs(z_ref).max()
    print("s", s, "precond rel err", err)
    assert err <= 1e-10  # as the cases above up to s = 300
    P.close()


def test_precond_full_size_solves_banded_system(bim):
    # 181 x 61: check P z = r with the oracle's banded product (P is never formed on the CPU)
    p = W.working(0.7)
    dp = bim.DeviceProblem(p)
    P = bim.Preconditioner(dp)
    assert P.band == 10
    r = np.random.default_rng(6).standard_normal(p.n_unknowns)
    z = P.apply(torch.as_tensor(r, device="cuda"))
    torch.cuda.synchronize()
    z = z.cpu().numpy()
    res = Lin.banded_matvec(p, z, P.band) - r
    print("181x61 |Pz - r| / |r|", np.abs(res).max() / np.abs(r).max(), "bytes", P.nbytes)
    assert np.abs(res).max() <= 1e-9 * np.abs(r).max()
    P.close()


def test_precond_rejects_bad_band(bim):
    p = W.tiny(0.7)
    dp = bim.DeviceProblem(p)
    with pytest.raises(bim.BimError):
        bim.Preconditioner(dp, p.M)


def test_fp32_storage_operator_solves_the_banded_system(bim):
    """FP32 storage (half the bytes): the block elimination and block LU of P in
    FP64, then, for pivot blocks of 128 < s <= 192, both substitutions that form
    the dense Schur inverse S^-1 in FP32 on FP32 copies of the FP64 factors, and
    the other arrays the apply reads rounded to FP32.  So it is not the FP64
    operator rounded: part of the factorisation runs in FP32.  At 181 x 61 its
    apply still solves the banded system P z = r of the oracle's banded product,
    next to the FP64 one, to FP32 rounding amplified by the conditioning of the
    Schur complement (the FP32 substitutions add ~1e-6, far below that)."""
    p = W.working(0.7)
    dp = bim.DeviceProblem(p)
    r = np.random.default_rng(6).standard_normal(p.n_unknowns)
    rd = torch.as_tensor(r, device="cuda")
    P64 = bim.Preconditioner(dp)
    z64 = P64.apply(rd).cpu().numpy()
    b64 = P64.nbytes
    P64.close()
    P32 = bim.Preconditioner(dp, storage="fp32")
    assert P32.storage == "fp32" and P32.band == 10
    z32 = P32.apply(rd).cpu().numpy()
    z32b = P32.apply(rd).cpu().numpy()
    print("bytes", b64, P32.nbytes)
    assert np.array_equal(z32, z32b)  # a fixed operator
    assert P32.nbytes < 0.51 * b64
    dz = np.abs(z32 - z64).max() / np.abs(z64).max()
    res = np.abs(Lin.banded_matvec(p, z32, 10) - r).max() / np.abs(r).max()
    print("181x61 fp32 storage: |z32 - z64| / |z64|", dz, "|P z32 - r| / |r|", res)
    # FP32 elements carry 6e-8 relative rounding, which the dense Schur-complement
    # inverse amplifies by its conditioning (its products cancel): measured 1.0e-3
    # and 2.6e-3.  A wrong or misplaced array gives O(1); the solves with this P
    # (test_gpu_jfnk) reach the FP64-P solution with about as many iterations.
    assert dz <= 1e-2
    assert res <= 1e-2
    P32.close()


def test_precond_rejects_unknown_storage(bim):
    import ctypes
    p = W.tiny(0.7)
    dp = bim.DeviceProblem(p)
    h = ctypes.c_void_p()
    assert bim.lib().precond_setup_ex(dp.ref(), -1, 2, ctypes.byref(h), None) == -1
    assert not h.value


# bounds: the FP32 rounding of the elements (6e-8) amplified by the
# cancellation in the products with the Schur-complement inverse, which grows as
# the mesh is refined: measured 5.1e-5 and 5.6e-5 on the coarse meshes, 2.65e-3
# at dx = 0.27 (4.1e-3 at 181 x 61, dx = 0.33, where the FP32 substitutions
# leave it unchanged to three digits)
@pytest.mark.parametrize("name,mk,hb,tol", [
    ("odd-s-44x9-h2", lambda: W.make_problem(44, 9, -12, 12, 0, 6, 0.9, [W.Bump(0.25, 1.3, 0.9)]), 2, 2e-4),
    ("even-s-45x9-h3", lambda: W.make_problem(45, 9, -12, 12, 0, 6, 0.9, [W.Bump(0.25, 1.3, 0.9)]), 3, 2e-4),
    # 128 < s <= 384: the substitutions forming S^-1 run in FP32 (odd s; and
    # s = 212, whose pivot blocks are inverted as 2 x 2 block matrices and whose
    # triangular products span two 192-row panels)
    ("fp32-substitutions-150x9-h2", lambda: W.make_problem(150, 9, -20, 20, 0, 4, 1.1, [W.Bump(0.2, 1.0, 1.0)]), 2,
     1e-2),
    ("fp32-substitutions-211x9-h2", lambda: W.make_problem(211, 9, -40, 30, 0, 4, 1.1, [W.Bump(0.2, 1.0, 1.0)]), 2,
     1e-2),
], ids=["odd-s", "even-s", "fp32-substitutions-odd-s", "fp32-substitutions-two-panels"])
def test_fp32_storage_small_meshes_match_oracle(bim, name, mk, hb, tol):
    # FP32 elements read one per lane (odd s: rows not aligned to two elements)
    # or two per lane (even s): both apply the oracle's P to FP32 rounding
    p = mk()
    dp = bim.DeviceProblem(p)
    P = bim.Preconditioner(dp, hb, storage="fp32")
    pc_ref = Lin.Preconditioner(p, hb=hb)
    r = np.random.default_rng(8).standard_normal(p.n_unknowns)
    z = P.apply(torch.as_tensor(r, device="cuda")).cpu().numpy()
    z_ref = pc_ref.apply(r)
    err = np.abs(z - z_ref).max() / np.abs(z_ref).max()
    print(name, "fp32 storage rel err", err)
    assert 0 < err <= tol  # rounded (not bit-equal to FP64), and close
    P.close()


def test_precond_full_domain_with_offset_edges(bim):
    # Full domains whose y_1 is not 0: the offset of the closed-form S2 (K5)
    # integral to the edge y_M through the last row of collocation points must be
    # exactly zero; formed from separately rounded coordinates it can be a few ulp,
    # which made that row's entries non-finite and the last pivot block singular
    # (the 91 x 91 mesh of the paper's two-bump domain did).  P z = r by the
    # oracle's banded product.
    import math
    d = 0.5 * math.sqrt(2.0)
    for N, M, (xlo, xhi, ylo, yhi) in ((91, 91, (-7.0, 53.0, -30.0, 30.0)), (121, 81, (-30.0, 30.0, -20.0, 20.0))):
        p = W.make_problem(N, M, xlo, xhi, ylo, yhi, 0.6,
                           [W.Bump(0.2, d, d, cx=10.0, cy=10.0), W.Bump(0.2, d, d, cx=0.0, cy=-10.0)],
                           half_domain=False)
        print(f"case full {N}x{M}", flush=True)
        dp = bim.DeviceProblem(p)
        P = bim.Preconditioner(dp)
        r = np.random.default_rng(7).standard_normal(p.n_unknowns)
        z = P.apply(torch.as_tensor(r, device="cuda"))
        torch.cuda.synchronize()
        res = Lin.banded_matvec(p, z.cpu().numpy(), P.band) - r
        print(f"full {N}x{M} |Pz - r| / |r|", np.abs(res).max() / np.abs(r).max())
        assert np.abs(res).max() <= 1e-9 * np.abs(r).max()
        P.close()


# The FP64 apply with table-formed banded products (stored bands of 150 MB and more): 1 to 4
# targets per lane, one and two blocks of targets, odd and even s, a slice longer than one
# table window (N > 512), half and full domains, at the working mesh's spacing of 1/3.
# P z = r by the oracle's banded product; the bound is that of the other full-size checks here.
# For s > 192 it holds for the rows of block 2 (the Schur complement's, where the products'
# errors meet): there the slice blocks' 2 x 2 block inverses, which leave 1e-8 to 6e-8 in the
# rows of blocks 1 and 3, have no part.
@pytest.mark.parametrize("N,M,half", [(65, 61, False), (120, 41, True), (129, 41, True), (181, 31, False),
                                      (257, 21, True), (300, 21, True), (600, 5, True)])
def test_table_formed_apply_solves_banded_system(bim, N, M, half):
    x, y = (N - 1) / 6.0, (M - 1) / 3.0
    p = W.make_problem(N, M, -x, x, 0.0 if half else -y, y, 1.2, [W.Bump(0.2, 1.0, 1.0)], half_domain=half)
    dp = bim.DeviceProblem(p)
    P = bim.Preconditioner(dp)
    assert 4 * 8 * M * (2 * P.band + 1) * (N + 1) ** 2 >= 150e6
    r = np.random.default_rng(9).standard_normal(p.n_unknowns)
    z = P.apply(torch.as_tensor(r, device="cuda"))
    torch.cuda.synchronize()
    res = Lin.banded_matvec(p, z.cpu().numpy(), P.band) - r
    nb = (N + 1) * M
    blocks = [np.abs(res[b * nb:(b + 1) * nb]).max() / np.abs(r).max() for b in range(3)]
    print(f"{N}x{M} |Pz - r| / |r| by block", blocks)
    assert blocks[1] <= 1e-9
    assert max(blocks) <= 1e-9 or N + 1 > 192
    P.close()


# The triangular products of the same apply in groups of slices with the factors' blocks between
# them: two groups of even and odd s, several on a half and a full domain, unequal groups (M no
# multiple of their number).  P z = r as above, with that bound.
@pytest.mark.parametrize("N,M,half", [(91, 91, True), (90, 91, True), (131, 131, True), (101, 122, False)])
def test_grouped_triangular_products_solve_banded_system(bim, N, M, half):
    x, y = (N - 1) / 6.0, (M - 1) / 3.0
    p = W.make_problem(N, M, -x, x, 0.0 if half else -y, y, 1.2, [W.Bump(0.2, 1.0, 1.0)], half_domain=half)
    dp = bim.DeviceProblem(p)
    P = bim.Preconditioner(dp)
    r = np.random.default_rng(11).standard_normal(p.n_unknowns)
    for shift in (0, 1):  # z on a 16-byte boundary and 8 bytes off it
        z = torch.empty(p.n_unknowns + 1, dtype=torch.float64, device="cuda")[shift:shift + p.n_unknowns]
        P.apply(torch.as_tensor(r, device="cuda"), out=z)
        torch.cuda.synchronize()
        res = Lin.banded_matvec(p, z.cpu().numpy(), P.band) - r
        print(f"{N}x{M} shift {shift} |Pz - r| / |r|", np.abs(res).max() / np.abs(r).max())
        assert np.abs(res).max() <= 1e-9 * np.abs(r).max()
    P.close()


# Rows of L^-1 and V^-1 in joint launches on one stream (n = (N + 1) M <= 3072) and on two above:
# both sides of the line, few slices, one tile of rows and more.  P z = r with the bound above.
@pytest.mark.parametrize("N,M", [(63, 48), (63, 49), (31, 5), (191, 16), (191, 17)])
def test_triangular_inverses_on_one_and_two_streams(bim, N, M):
    p = W.make_problem(N, M, -(N - 1) / 6.0, (N - 1) / 6.0, 0.0, (M - 1) / 3.0, 1.2, [W.Bump(0.2, 1.0, 1.0)])
    dp = bim.DeviceProblem(p)
    P = bim.Preconditioner(dp)
    r = np.random.default_rng(13).standard_normal(p.n_unknowns)
    z = P.apply(torch.as_tensor(r, device="cuda"))
    torch.cuda.synchronize()
    res = Lin.banded_matvec(p, z.cpu().numpy(), P.band) - r
    print(f"{N}x{M} |Pz - r| / |r|", np.abs(res).max() / np.abs(r).max())
    assert np.abs(res).max() <= 1e-9 * np.abs(r).max()
    P.close()


# Few long slices keep the stored blocks (fewer than s / 160, where the one workgroup per slice
# that forms a3 takes longer than reading them); both sides of the line, P z = r in the rows of
# block 2 as for the other s > 192
@pytest.mark.parametrize("N,M,tables", [(640, 4, False), (639, 4, True)])
def test_tables_need_a_slice_per_160_rows(bim, N, M, tables):
    p = W.make_problem(N, M, -(N - 1) / 6.0, (N - 1) / 6.0, 0.0, (M - 1) / 3.0, 1.2, [W.Bump(0.2, 1.0, 1.0)])
    dp = bim.DeviceProblem(p)
    P = bim.Preconditioner(dp)
    s, w = N + 1, 2 * P.band + 1
    stored = 8 * (4 * M * s * s + 4 * M * w * s * s + (M * s) ** 2 + 4 * M * s)  # the arrays of the blocks
    assert (P.nbytes - stored >= 8 * (2 * N + 1) * s) == tables  # E and the node-value map of a slice
    r = np.random.default_rng(9).standard_normal(p.n_unknowns)
    z = P.apply(torch.as_tensor(r, device="cuda"))
    torch.cuda.synchronize()
    res = Lin.banded_matvec(p, z.cpu().numpy(), P.band) - r
    nb = (N + 1) * M
    blocks = [np.abs(res[b * nb:(b + 1) * nb]).max() / np.abs(r).max() for b in range(3)]
    print(f"{N}x{M} |Pz - r| / |r| by block", blocks)
    assert blocks[1] <= 1e-9
    P.close()


# Blocks longer than 192 rows are inverted as 2 x 2 block matrices, which pivot within their parts
# only; that leaves 1e-8 to 6e-8 of r in the rows of blocks 1 and 3 of P z = r.  The bound is ten
# times that: a wrong entry or a term left out of z1 or z3 is of the order of r.
@pytest.mark.parametrize("N,M", [(257, 21), (300, 21), (600, 5)])
def test_table_formed_apply_bounds_every_block_of_long_slices(bim, N, M):
    p = W.make_problem(N, M, -(N - 1) / 6.0, (N - 1) / 6.0, 0.0, (M - 1) / 3.0, 1.2, [W.Bump(0.2, 1.0, 1.0)])
    dp = bim.DeviceProblem(p)
    P = bim.Preconditioner(dp)
    r = np.random.default_rng(9).standard_normal(p.n_unknowns)
    z = P.apply(torch.as_tensor(r, device="cuda"))
    torch.cuda.synchronize()
    res = Lin.banded_matvec(p, z.cpu().numpy(), P.band) - r
    nb = (N + 1) * M
    blocks = [np.abs(res[b * nb:(b + 1) * nb]).max() / np.abs(r).max() for b in range(3)]
    print(f"{N}x{M} |Pz - r| / |r| by block", blocks)
    assert max(blocks) <= 6e-7
    P.close()
