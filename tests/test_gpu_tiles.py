"""Kernels at the sizes where a tile, a k split or a vector load can go wrong, through the single calls,
against the fp64 oracle.

Tolerance of the split-precision products: an operand is the sum of two bf16 pieces up to 2^-17 of its
size and the product of the two second pieces is dropped, so a product is off by at most 3 x 2^-17 of
|a||b|; two chained products, errors of random sign over the sums: 2 x 3 x 2^-17 = 4.6e-5.  One piece
(bf16 operands): 2^-9 per rounding, four roundings (G or T, V, U, P or D): 7.8e-3."""
import pytest
import torch

import synth_inputs as si
from oracle import tsr_oracle as orc
from gpu_util import check_close, dev, f32, padded

pytestmark = pytest.mark.gpu

TOL = {"split": 4.6e-5, "bf16": 7.8e-3}


@pytest.fixture(scope="module")
def tsr():
    import paper_2602_08007_amd as t
    assert torch.cuda.is_available()
    return t


def _bases(m, n, r, key):
    return si.orthonormal(m, r, si.stream_key(key, 1)).float(), si.orthonormal(n, r, si.stream_key(key, 2)).float()


# the kernels for one small matrix (r <= 128: ranks of one and two 64-wide blocks and their remainders, rows and
# columns around 64, contractions below a vector's width), 64 x 64 tiles (r = 129), 128 x 64 (rank 30 at many units), 128 x 128; k remainders of 1 and 31
# beside whole k-tiles; row remainders of 1, 2 and 127; extents below a vector's (2, 3, 5 and 7)
SIZES = [(2, 3, 2), (5, 7, 3), (7, 65, 5), (64, 64, 64), (65, 97, 33), (127, 129, 65), (1026, 3713, 65), (1151, 4127, 30),
         (641, 4097, 129),
         (1, 1, 1), (33, 31, 4), (63, 129, 63), (130, 1000, 128), (1000, 100, 97), (1001, 1365, 96), (200, 131, 130)]


@pytest.mark.parametrize("m,n,r", SIZES)
@pytest.mark.parametrize("dtype,prec", [(torch.float32, "split"), (torch.bfloat16, "bf16")])
def test_project_sizes(tsr, m, n, r, dtype, prec):
    key = si.stream_key(701, m, n, r)
    G = si.normal((m, n), si.stream_key(key, 3)).to(dtype)
    U, V = _bases(m, n, r, key)
    C = torch.full((r, r), float("nan"), device="cuda")
    tsr.tsr_project_core(dev(G), dev(U), dev(V), C, precision=getattr(tsr, "TSR_PREC_" + prec.upper()))
    # the core of a white gradient is 1 / sqrt(mn / r^2) of its norm: errors relative to what the sums hold
    check_close(C, orc.project_core(G, U, V), TOL[prec] * max(1.0, (min(m, n) / r) ** 0.5), "core")


@pytest.mark.parametrize("m,n,r", [(64, 700, 17), (200, 1000, 64), (1000, 650, 100), (700, 900, 200)])
@pytest.mark.parametrize("dtype,prec", [(torch.bfloat16, "bf16"), (torch.bfloat16, "split"), (torch.float32, "bf16"), (torch.float32, "split")])
def test_project_columns_that_cancel(tsr, m, n, r, dtype, prec):
    """Two halves of the columns whose products cancel to 2^-8 of either (the one is the other with the opposite sign,
    100 columns and more away, so that no range of a k split holds both alike): the precision counts against the sum."""
    key, half = si.stream_key(708, m, n, r), n // 2 - 13
    A = si.normal((m, half), si.stream_key(key, 1)).bfloat16().float()
    G = torch.cat([A, -A, torch.zeros(m, n - 2 * half)], 1)
    V1 = si.normal((half, r), si.stream_key(key, 2)) / half ** 0.5
    V = torch.cat([V1, V1, si.normal((n - 2 * half, r), si.stream_key(key, 3)) / (n - 2 * half) ** 0.5], 0)
    G[:, 2 * half:] = (2.0 ** -8 * si.normal((m, n - 2 * half), si.stream_key(key, 4))).bfloat16().float()
    U = si.orthonormal(m, r, si.stream_key(key, 5)).float()
    C = torch.full((r, r), float("nan"), device="cuda")
    tsr.tsr_project_core(dev(G.to(dtype)), dev(U), dev(V), C, precision=getattr(tsr, "TSR_PREC_" + prec.upper()))
    # and fp32 sums of n products with errors of random sign, 2^8 times the result
    check_close(C, orc.project_core(G, U, V), TOL[prec] + 4 * n ** 0.5 * 2.0 ** -16, "core")


# (the last two: beyond the kernel for one small matrix, with the intermediate on the side of the columns)
@pytest.mark.parametrize("m,n,r", SIZES + [(4 * 259, 259, 150), (33000, 133, 40)])
@pytest.mark.parametrize("prec", ["split", "bf16"])
def test_lift_sizes(tsr, m, n, r, prec):
    key = si.stream_key(702, m, n, r)
    U, V = _bases(m, n, r, key)
    D = si.normal((r, r), si.stream_key(key, 3)).clamp(-1, 1)
    W0 = si.weights(m, n, si.stream_key(key, 4))
    W = dev(W0)
    tsr.tsr_backproject_apply(W, dev(U), dev(V), dev(D), 1.0, 0.1, 0.75, precision=getattr(tsr, "TSR_PREC_" + prec.upper()))
    ref = orc.backproject_apply(orc.f64(W0).copy(), U, V, D, 1.0, f32(0.1), 0.75)
    check_close(orc.f64(W) - orc.f64(W0), ref - orc.f64(W0), TOL[prec], "movement")


# the orthonormalisation and the small SVD around their tile sizes: 16-wide tiles (5, 9, 13 and 17 of them per
# Cholesky kernel; cut in two above 272, with halves of up to 9 and up to 17 tiles, up to 544), 32-wide ones
# (3, 5, 7 and 9) in the tridiagonalization, the variant above 288
@pytest.mark.parametrize("k", [5, 15, 16, 17, 33, 64, 80, 81, 144, 96, 97, 145, 160, 161, 224, 225, 264, 272, 273, 288, 289,
                               303, 417, 528, 543, 544, 545])
def test_refresh_full_sketch_sizes(tsr, k):
    """A sketch as wide as the matrix is high spans everything: the singular values and the leading
    subspaces are those of the matrix, up to the orthonormality the last pass leaves (fp64, stored in
    fp32: below 2^-24 per entry over k columns)."""
    p = min(4, k - 1)
    r, m, n = k - p, k, k + 9
    key = si.stream_key(703, k)
    G = si.normal((m, n), si.stream_key(key, 1))
    G[:, :3] *= 4.0
    U = torch.full((m, r), float("nan"), device="cuda")
    V = torch.full((n, r), float("nan"), device="cuda")
    sigma = torch.full((k,), float("nan"), device="cuda")
    tsr.tsr_refresh_rsvd(dev(G), dev(si.omega(n, k, si.stream_key(key, 2))), r, p, 1, U, V, sigma)
    s = torch.linalg.svdvals(G.double())
    # an fp32 sum of k products is off by at most k x 2^-24 of the sum of their sizes; four such sums in a
    # row bound the way from the matrix to the triangular factor (the passes over Q and over the factor are fp64 and
    # stored in fp32, the product with Q between them is one such sum)
    assert float((sigma.cpu().double() - s).abs().max() / s[0]) < (k + 4) * 2.0 ** -22
    U64, V64, eye = U.cpu().double(), V.cpu().double(), torch.eye(r, dtype=torch.float64)
    for X in (U64, V64):
        assert float(torch.linalg.norm(X.T @ X - eye)) < 2.0 ** -20 * k
    core = U64.T @ G.double() @ V64
    assert float(torch.linalg.norm(core - torch.diag(s[:r])) / torch.linalg.norm(s)) < 2e-5


# the fp64 Gram matrices cut the rows into pieces (multiples of 16) and the columns into 32-wide tiles, one
# per wave: a remainder of one row, row counts around a piece's, one tile, two, one column more, a fourth one
@pytest.mark.parametrize("rows,k", [(1000, 20), (1025, 33), (4097, 64), (130, 65), (33000, 9), (2049, 97)])
def test_refresh_tall_full_sketch(tsr, rows, k):
    """As above with many rows on either side (B^T is as tall as G^T): singular values and orthonormality."""
    p = 4
    r = k - p
    for m, n in ((rows, k), (k, rows)):
        key = si.stream_key(705, m, n)
        G = si.normal((m, n), si.stream_key(key, 1))
        U = torch.full((m, r), float("nan"), device="cuda")
        V = torch.full((n, r), float("nan"), device="cuda")
        sigma = torch.full((k,), float("nan"), device="cuda")
        tsr.tsr_refresh_rsvd(dev(G), dev(si.omega(n, k, si.stream_key(key, 2))), r, p, 0, U, V, sigma)
        s = torch.linalg.svdvals(G.double())
        # fp32 sums of up to `rows` products with errors of random sign
        tol = 4 * (rows ** 0.5 + 4) * 2.0 ** -24
        assert float((sigma.cpu().double() - s).abs().max() / s[0]) < tol
        eye = torch.eye(r, dtype=torch.float64)
        for X in (U.cpu().double(), V.cpu().double()):
            assert float(torch.linalg.norm(X.T @ X - eye)) < 2.0 ** -20 * k


# blocks four times as high as wide beside others: the intermediate of the lift on the side of their rows, and (more than
# three million elements less) on that of their columns, in a launch of its own
@pytest.mark.parametrize("dims", [[(1100, 261, 64), (300, 501, 64), (77, 19, 7)], [(300, 501, 130), (24100, 301, 130), (130, 261, 130)]])
@pytest.mark.parametrize("prec", ["split", "bf16"])
def test_plan_with_tall_blocks(tsr, dims, prec):
    blocks = []
    for i, (m, n, r) in enumerate(dims):
        key = si.stream_key(709, m, n)
        U, V = _bases(m, n, r, key)
        G = U @ torch.diag(torch.linspace(2.0, 1.0, r)) @ V.T + 0.01 * si.normal((m, n), si.stream_key(key, 3))
        z = lambda *x: torch.zeros(*x, device="cuda")  # noqa: E731
        blocks.append(dict(G=dev(G), W=z(m, n), U=dev(U), V=dev(V), M=z(r, r), Vm=z(r, r), C=z(r, r), D=z(r, r)))
    plan = tsr.Plan(blocks, precision=getattr(tsr, "TSR_PREC_" + prec.upper()))
    assert plan.tsr_plan_kernel_path() == 0                    # odd widths: the general kernels in either precision
    for t in (1, 2):
        for b in blocks:
            b["W"].zero_(); b["M"].zero_(); b["Vm"].zero_()
        plan.tsr_step_batched(1, lr=1.0, eps=1.0)
    torch.cuda.synchronize()
    for b in blocks:
        G, U, V, C, D = (orc.f64(b[x]) for x in ("G", "U", "V", "C", "D"))
        check_close(C, orc.project_core(G, U, V), TOL[prec] * max(1.0, (min(G.shape) / U.shape[1]) ** 0.5), "core")
        check_close(orc.f64(b["W"]), -U @ D @ V.T, TOL[prec], "movement")
    plan.close()


def _refresh(tsr, how, G, r, p, q, key):
    """Bases by the single call, or by a plan (a bf16 gradient then takes the other family of kernels)."""
    m, n = G.shape
    om = dev(si.omega(n, r + p, key))
    U, V = torch.full((m, r), float("nan"), device="cuda"), torch.full((n, r), float("nan"), device="cuda")
    if how == "call":
        tsr.tsr_refresh_rsvd(dev(G), om, r, p, q, U, V)
    else:
        z = lambda *s: torch.zeros(*s, device="cuda")  # noqa: E731
        plan = tsr.Plan([dict(G=padded(G, (n + 7) // 8 * 8), W=z(m, n), U=U, V=V, M=z(r, r), Vm=z(r, r), C=z(r, r), D=z(r, r))], with_refresh=True, p=p,
                        precision=tsr.TSR_PREC_BF16 if G.dtype == torch.bfloat16 else tsr.TSR_PREC_SPLIT)
        plan.tsr_refresh_batched([om], q)
        torch.cuda.synchronize()
        plan.close()
    return U.cpu().double(), V.cpu().double()


def _check_full_sketch(G, U, V, k):
    """As test_refresh_full_sketch_sizes, with products in two bf16 pieces (bf16 gradients)."""
    G64, r = G.double(), U.shape[1]
    s = torch.linalg.svdvals(G64)
    core, eye = U.T @ G64 @ V, torch.eye(r, dtype=torch.float64)
    for X in (U, V):
        assert float(torch.linalg.norm(X.T @ X - eye)) < 2.0 ** -20 * k
    assert float((core.diagonal() - s[:r]).abs().max() / s[0]) < (k + 4) * 2.0 ** -22 + 3 * 2.0 ** -17
    assert float(torch.linalg.norm(core - torch.diag(s[:r])) / torch.linalg.norm(s)) < 2e-5 + 3 * 2.0 ** -17


# a plan's bf16 gradients with many rows on either side: the row pieces of the fp64 Gram matrices (see above) behind
# the other family's products
@pytest.mark.parametrize("rows,k", [(1025, 33), (4097, 64), (33000, 16), (2049, 97)])
def test_refresh_tall_full_sketch_of_a_plan(tsr, rows, k):
    for m, n in ((rows, k), (k, rows)):
        key = si.stream_key(710, m, n)
        G = si.normal((m, n), si.stream_key(key, 1)).bfloat16()
        U, V = _refresh(tsr, "plan", G, k - 4, 4, 0, si.stream_key(key, 2))
        _check_full_sketch(G, U, V, k)


def test_refresh_wide_tiles_ragged(tsr, monkeypatch):
    """The 256 x 192 tiles (513 to 576 columns, more than 256 tiles in one launch) at 531 columns, with a row remainder of
    each kind, a tall and a wide block among the others."""
    monkeypatch.setenv("TSR_TUNE_REFRESH_GROUPS", "1")
    k, p = 531, 8
    r = k - p
    shapes = [(700, 536)] * 27 + [(4097, 531), (531, 700), (531, 4097)]
    made, blocks, omegas = {}, [], []
    for m, n in shapes:
        if (m, n) not in made:
            key = si.stream_key(711, m, n)
            G = torch.zeros(m, (n + 7) // 8 * 8, dtype=torch.bfloat16, device="cuda")[:, :n]
            G.copy_(si.normal((m, n), si.stream_key(key, 1)))
            made[m, n] = G, dev(si.omega(n, k, si.stream_key(key, 2)))
        G, om = made[m, n]
        z = lambda *x: torch.zeros(*x, device="cuda")  # noqa: E731
        blocks.append(dict(G=G, W=z(m, n), U=z(m, r), V=z(n, r), M=z(r, r), Vm=z(r, r), C=z(r, r), D=z(r, r)))
        omegas.append(om)
    plan = tsr.Plan(blocks, precision=tsr.TSR_PREC_BF16, with_refresh=True, p=p)
    plan.tsr_refresh_batched(omegas, 0)
    torch.cuda.synchronize()
    for b in blocks[:26]:                                      # the same block: the same bits, wherever its tiles ran
        assert torch.equal(b["U"], blocks[26]["U"]) and torch.equal(b["V"], blocks[26]["V"])
    for b in blocks[27:]:
        _check_full_sketch(b["G"].cpu(), b["U"].cpu().double(), b["V"].cpu().double(), k)
    U, V = (blocks[0][x].cpu().double() for x in ("U", "V"))   # five columns short of everything
    for X in (U, V):
        assert float(torch.linalg.norm(X.T @ X - torch.eye(r, dtype=torch.float64))) < 2.0 ** -20 * k
    plan.close()


# what the fp64 passes of the final orthonormalisation are for: with one power iteration the sketch is singular to fp32
# (the shifted normalisations in it leave small x (100 small)^2 of the small rows' directions)
@pytest.mark.parametrize("how,g", [("plan", torch.bfloat16), ("call", torch.bfloat16), ("plan", torch.float32)])
@pytest.mark.parametrize("small,q", [(1e-4, 0), (1e-4, 1), (3e-4, 1)])
def test_refresh_rows_of_two_scales(tsr, how, g, small, q):
    """Sixty rows that are not zero, two thirds of them `small` times the others (an embedding's gradient with rare
    tokens): the sketch holds their span, and the small ones come back to what one fp32 rounding of the large ones is
    to them, 2^-24 / small; the columns are orthonormal to what the last pass allows, 1e4 x 2^-24.  Medians of five
    matrices: how far a sketch is from dependent columns differs from one to the other."""
    m, n, r, p, lead = 2000, 512, 64, 8, 60
    eye = torch.eye(lead, dtype=torch.float64)
    found = []
    for seed in range(5):
        key = si.stream_key(706, seed)
        at = torch.randperm(m, generator=torch.Generator().manual_seed(seed))[:lead]
        G = torch.zeros(m, n)
        G[at] = si.normal((lead, n), si.stream_key(key, 1))
        G[at[20:]] *= small
        G = G.to(g)
        U, V = _refresh(tsr, how, G, r, p, q, si.stream_key(key, 2))
        U, V, G64, weak = U[:, :lead], V[:, :lead], G.double(), at[20:]
        rel = lambda E, rows: float(torch.linalg.norm(E[rows]) / torch.linalg.norm(G64[rows]))  # noqa: E731
        found.append((rel(G64 - U @ (U.T @ G64), weak), rel(G64 - (G64 @ V) @ V.T, weak),
                      *(float(torch.linalg.norm(X.T @ X - eye, ord=2)) for X in (U, V))))
        assert rel(G64 - U @ (U.T @ G64 @ V) @ V.T, slice(None)) < 2e-5
    median = [sorted(column)[2] for column in zip(*found)]
    assert max(median[:2]) < 2.0 ** -24 / small, median
    assert max(median[2:]) < 1e4 * 2.0 ** -24, median


# the factorization takes four columns at a time, sixteen per tile: dropped columns from every place of a panel on,
# from the first of a tile on, and tiles of nothing else
@pytest.mark.parametrize("rank", [1, 2, 3, 4, 5, 15, 16, 17, 21, 32, 35])
def test_refresh_dropped_columns(tsr, rank):
    """An exactly rank-deficient gradient: the directions beyond its rank are dropped pivots (zero columns of the
    factor), and the leading ones span the gradient.  fp32 sums of up to 150 products: 150 x 2^-24, over the four
    products in a row as above."""
    m, n, r, p = 120, 150, 40, 8
    key = si.stream_key(704, rank)
    G = (si.normal((m, rank), si.stream_key(key, 1)).double() @ si.normal((rank, n), si.stream_key(key, 2)).double()).float()
    U = torch.full((m, r), float("nan"), device="cuda")
    V = torch.full((n, r), float("nan"), device="cuda")
    sigma = torch.full((r + p,), float("nan"), device="cuda")
    tsr.tsr_refresh_rsvd(dev(G), dev(si.omega(n, r + p, si.stream_key(key, 3))), r, p, 1, U, V, sigma)
    U64, V64, s = U.cpu().double(), V.cpu().double(), torch.linalg.svdvals(G.double())
    assert bool(torch.isfinite(U64).all() and torch.isfinite(V64).all())
    tol = 4 * 150 * 2.0 ** -24
    assert float((sigma.cpu().double()[:rank] - s[:rank]).abs().max() / s[0]) < tol
    assert float(sigma[rank:].abs().max() / s[0]) < tol
    # (a direction of rounding may survive the drop, of length one but not orthogonal to the others: the leading ones count)
    U64, V64 = U64[:, :rank], V64[:, :rank]
    back = U64 @ (U64.T @ G.double() @ V64) @ V64.T
    assert float(torch.linalg.norm(back - G.double()) / torch.linalg.norm(G.double())) < tol


@pytest.mark.parametrize("how,g", [("plan", torch.bfloat16), ("call", torch.bfloat16), ("call", torch.float32)])
@pytest.mark.parametrize("rank,r,q", [(1, 40, 1), (5, 40, 1), (16, 40, 0), (35, 40, 1), (100, 560, 1)])
def test_refresh_beyond_the_rank(tsr, how, g, rank, r, q):
    """Rows that are not zero, fewer than r of them: the leading columns are orthonormal, and all r columns, with
    which a step projects, leave the gradient as it is (a column beyond the rank is zero, or orthogonal to the others).
    The last rank of 560 takes the one-kernel small SVD.  Products and storage in fp32 over `rank` rows, four in a row."""
    m, n, p = (120, 152, 8) if r == 40 else (700, 608, 8)
    key = si.stream_key(707, rank)
    G = torch.zeros(m, n)
    G[torch.randperm(m, generator=torch.Generator().manual_seed(rank))[:rank]] = si.normal((rank, n), si.stream_key(key, 1))
    U, V = _refresh(tsr, how, G.to(g), r, p, q, si.stream_key(key, 2))
    G64 = G.to(g).double()
    assert bool(torch.isfinite(U).all() and torch.isfinite(V).all())
    eye = torch.eye(rank, dtype=torch.float64)
    for X in (U[:, :rank], V[:, :rank]):
        assert float(torch.linalg.norm(X.T @ X - eye)) < 4 * rank * 2.0 ** -22
    back = U @ (U.T @ G64 @ V) @ V.T
    assert float(torch.linalg.norm(back - G64) / torch.linalg.norm(G64)) < 4 * (rank + 4) * 2.0 ** -22


# the tridiagonalizations (in registers; from memory down to 288 columns; the one kernel above 544) of what a spectrum
# that ends in zeros leaves: after a few columns rounding of rounding, whose squares underflow
@pytest.mark.parametrize("k", [72, 264, 400, 516, 560])
@pytest.mark.parametrize("spectrum", ["steep 2", "steep 8", "rank 5", "rank 20"])
def test_refresh_spectra_that_end_in_zeros(tsr, k, spectrum):
    kind, by = spectrum.split()
    m, n, r, p = k + 44, k + 24, k - 16, 16
    for seed in range(2):
        key = si.stream_key(712, k, seed, len(kind))
        A, B = si.normal((m, n), si.stream_key(key, 1)), si.normal((n, n), si.stream_key(key, 3))
        if kind == "steep":
            G = torch.linalg.qr(A.double())[0] * 10.0 ** (-torch.arange(n, dtype=torch.float64) / float(by))
        else:
            G = A[:, :int(by)].double() @ B[:int(by)].double()
        G = G.float()
        U, V = torch.full((m, r), float("nan"), device="cuda"), torch.full((n, r), float("nan"), device="cuda")
        sigma = torch.full((k,), float("nan"), device="cuda")
        tsr.tsr_refresh_rsvd(dev(G), dev(si.omega(n, k, si.stream_key(key, 2))), r, p, seed, U, V, sigma)
        assert bool(torch.isfinite(U).all() and torch.isfinite(V).all() and torch.isfinite(sigma).all())
        s = torch.linalg.svdvals(G.double())
        # (sketch and products in fp32 over k columns, four in a row, as above; what the sketch leaves out of a steep
        # spectrum is its tail)
        assert float((sigma.cpu().double() - s[:k]).abs().max() / s[0]) < (k + 4) * 2.0 ** -22


# panels of 128 rows: 343 and 344 (three groups of workers), 1025 (one), 8 (every worker by itself)
@pytest.mark.parametrize("m,n,r,workers,summed", [(43801, 136, 128, 8, True), (44000, 131, 128, 7, True),
                                                  (131077, 257, 256, 4, True), (1000, 136, 128, 8, False)])
def test_projection_sums_workers(tsr, m, n, r, workers, summed):
    """The mean core against the fp64 product of the summed gradients with the bases as the path holds them
    (bf16).  Where the workers are summed before U^T, the sum is kept to two bf16 pieces: the tolerance of the
    split products; else every worker's P is rounded once."""
    gen = torch.Generator(device="cuda").manual_seed(7 * m + workers)
    randn = lambda *s: torch.randn(*s, device="cuda", generator=gen)  # noqa: E731
    ld = (n + 7) // 8 * 8
    G = torch.full((workers, m, ld), float("nan"), dtype=torch.bfloat16, device="cuda")
    G[:, :, :n] = randn(workers, m, n)
    U, V = torch.linalg.qr(randn(m, r))[0].contiguous(), torch.linalg.qr(randn(n, r))[0].contiguous()
    z = lambda *s: torch.zeros(*s, device="cuda")  # noqa: E731
    b = dict(G=G[:, :, :n], W=z(m, n), U=U, V=V, M=z(r, r), Vm=z(r, r), C=z(r, r), D=z(r, r))
    plan = tsr.Plan([b], n_workers=workers, precision=tsr.TSR_PREC_BF16)
    for _ in range(2):
        plan.tsr_step_batched(1, lr=0.0)
    total = sum(G[w, :, :n].double() for w in range(workers)) / workers
    ref = U.bfloat16().double().T @ (total @ V.bfloat16().double())
    check_close(b["C"].cpu(), ref.cpu().numpy(), TOL["split"] if summed else TOL["bf16"], "core")
