"""What the library keeps in the caller's workspace stays inside it."""
import os
import shutil
import subprocess

import pytest
import torch

import synth_inputs as si
from oracle import tsr_oracle as orc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_08007_amd", "csrc")


@pytest.fixture(scope="module")
def tsr():
    import paper_2602_08007_amd as t
    return t


# ------------------------------------------------------------------ scratch of the small SVD (host)
EIG_LAYOUT_CHECK = r"""
#include <cstdio>
#include "eig_layout.h"
int main() {
    for (int k = 1; k <= 544; ++k) {
        size_t end = (size_t)3 * k * k;                       // the LU factors' last entry, and where d begins
        if (tsr::eig_tridiag_at(k) < end) { printf("k = %d: the tridiagonal matrix lies in the LU factors\n", k); return 1; }
        int reflectors = 0;
        for (int b = 0; 16 * b < k; ++b) {
            const int rank = tsr::eig_wy_rank(k, b);
            if (rank < 0 || rank > 16) return 2;
            reflectors += rank;
            for (int row = 0; row < rank; ++row)
                for (int col = 0; col < rank; ++col)
                    if (tsr::eig_wy_at(b, row, col) >= tsr::eig_tridiag_at(k)) {
                        printf("k = %d: entry (%d, %d) of factor %d lies outside\n", k, row, col, b);
                        return 3;
                    }
        }
        if (reflectors != (k > 2 ? k - 2 : 0)) { printf("k = %d: %d reflectors\n", k, reflectors); return 4; }
        // d, e, eigenvalues, radius
        if (tsr::eig_scratch_doubles(k) < tsr::eig_tridiag_at(k) + 3 * (size_t)k + 1) return 5;
    }
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_small_svd_scratch_holds_what_is_indexed(tmp_path):
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(EIG_LAYOUT_CHECK)
    build = subprocess.run(["g++", "-std=c++17", "-Wall", "-I", CSRC, "-o", str(exe), str(src)], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout


# ------------------------------------------------------------------ bytes behind the workspace (GPU)
SENTINEL = 0x5A
TAIL = 8192


class Guarded:
    """A workspace of exactly nbytes with sentinel bytes behind it."""

    def __init__(self, nbytes):
        self.buf = torch.full((nbytes + TAIL,), SENTINEL, dtype=torch.uint8, device="cuda")
        self.ws = self.buf[:nbytes]

    def check(self):
        assert bool((self.buf[self.ws.numel():] == SENTINEL).all()), "bytes behind the workspace were written"


# One product in two bf16 pieces, the coarsest that any path here has (B = Q^T G; the last orthonormalisation
# passes are fp64), is off by at most 3 x 2^-17 of |a||b| (second pieces up to 2^-17 of the first, their product
# dropped).  Long sums average it out; here a sum has one to seventeen terms.
TWO_PIECES = 3 * 2.0 ** -17


def _check_bases(G, U, V, sigma=None):
    """Singular values and bases of a sketch that spans everything: that product, and fp32 sums of k terms (off by
    k x 2^-24 of the sum of their sizes, four in a row)."""
    k, r = min(G.shape), U.shape[1]
    s = torch.linalg.svdvals(G.double())
    U64, V64 = U.cpu().double(), V.cpu().double()
    eye = torch.eye(r, dtype=torch.float64)
    if sigma is not None:
        assert float((sigma.cpu().double()[:k] - s).abs().max() / s[0]) < TWO_PIECES + (k + 4) * 2.0 ** -22
    for X in (U64, V64):
        assert float(torch.linalg.norm(X.T @ X - eye)) < 2.0 ** -20 * max(k, 4)
    core = U64.T @ G.double() @ V64
    assert float(torch.linalg.norm(core - torch.diag(s[:r])) / torch.linalg.norm(s)) < TWO_PIECES + 2e-5


@pytest.mark.gpu
@pytest.mark.parametrize("k", list(range(1, 10)) + [15, 16, 17, 81, 145, 273, 289, 544])
def test_refresh_stays_in_its_workspace(tsr, k):
    p = min(2, k - 1)
    r, m, n = k - p, k, k + 9
    key = si.stream_key(811, k)
    G = si.normal((m, n), si.stream_key(key, 1))
    om = si.omega(n, k, si.stream_key(key, 2)).cuda()
    new = lambda: (torch.full((m, r), float("nan"), device="cuda"), torch.full((n, r), float("nan"), device="cuda"),  # noqa: E731
                   torch.full((k,), float("nan"), device="cuda"))
    g = Guarded(tsr.tsr_refresh_workspace_bytes(m, n, r, p))
    U, V, sigma = new()
    tsr.tsr_refresh_rsvd(G.cuda(), om, r, p, 1, U, V, sigma, ws=g.ws)
    g.check()
    _check_bases(G, U, V, sigma)
    g = Guarded(tsr.tsr_refresh_workers_workspace_bytes(m, n, r, p, 2))
    U, V, sigma = new()
    tsr.tsr_refresh_rsvd_workers(torch.stack([G, G]).cuda(), om, r, p, 1, U, V, sigma, ws=g.ws)
    g.check()
    _check_bases(G, U, V, sigma)
    for A in (G, torch.empty(n, m).copy_(G.T)):
        g = Guarded(tsr.tsr_refresh_exact_workspace_bytes(*A.shape, r))
        U, V, sigma = new()
        if A.shape != G.shape:
            U, V = V, U
        tsr.tsr_refresh_exact_svd(A.cuda(), r, U, V, sigma, ws=g.ws)
        g.check()
        _check_bases(A, U, V, sigma)


@pytest.mark.gpu
@pytest.mark.parametrize("groups", [1, 3])
def test_plan_of_tiny_blocks_refreshes_then_steps(tsr, groups, monkeypatch):
    """Sketches of 3 to 9 columns beside each other in one plan: bases of every block, and the following step
    against the oracle (its tables and the other blocks' buffers lie behind each block's scratch)."""
    monkeypatch.setenv("TSR_TUNE_REFRESH_GROUPS", str(groups))
    p, q, dims = 2, 1, [(k, k + 9) for k in range(3, 10)] * 2
    blocks, omegas, grads = [], [], []
    for i, (m, n) in enumerate(dims):
        key, r = si.stream_key(812, i), m - p
        G = si.normal((m, n), si.stream_key(key, 1))
        grads.append(G)
        z = lambda *s: torch.zeros(*s, device="cuda")  # noqa: E731
        blocks.append(dict(G=G.cuda(), W=z(m, n), U=z(m, r), V=z(n, r), M=z(r, r), Vm=z(r, r), C=z(r, r), D=z(r, r)))
        omegas.append(si.omega(n, m, si.stream_key(key, 2)).cuda())
    plan = tsr.Plan(blocks, with_refresh=True, p=p)
    plan.tsr_refresh_batched(omegas, q)
    plan.tsr_step_batched(1, lr=1.0, eps=1.0)
    torch.cuda.synchronize()
    for G, b in zip(grads, blocks):
        _check_bases(G, b["U"], b["V"])
        C = orc.project_core(G, orc.f64(b["U"]), orc.f64(b["V"]))
        scale = float(abs(C).max())
        assert float(abs(orc.f64(b["C"]) - C).max()) < 1e-4 * scale
        # first Adam step from zero moments, eps = 1: D = C / (|C| + 1); then W = -U D V^T
        W = -orc.f64(b["U"]) @ (C / (abs(C) + 1.0)) @ orc.f64(b["V"]).T
        assert float(abs(orc.f64(b["W"]) - W).max()) < 1e-4 * float(abs(W).max())



# ------------------------------------------------------------------ the built-in scratch (host, GPU)
def _arena(*sizes):
    """Bytes of buffers of these sizes, each on a 256-byte boundary."""
    return sum((s + 255) // 256 * 256 for s in sizes)


def _partials(m, n, k, want_tiles=512):
    """fp32 partial results of an m x n product over k: 128 x 128 tiles, k cut into pieces of at least 256 until
    there are `want_tiles` of them."""
    tiles = -(-m // 128) * -(-n // 128)
    s = min(max(1, want_tiles // tiles), max(1, k // 256))
    s = -(-k // (-(-(-(-k // s)) // 32) * 32))
    return 4 * m * n * s if s > 1 else 0


def _project_bytes(m, n, r):
    return _arena(4 * m * r, _partials(m, r, n), _partials(r, r, m))


# odd products that fill the 16 MiB to the last kilobyte
EDGES = [(9961, 1000, 97), (13118, 1000, 75), (13952, 300, 183), (19876, 300, 141), (40360, 300, 81)]


def test_static_scratch_takes_what_fits_it(tsr):
    limit = tsr.TSR_PROJECT_STATIC_SCRATCH_BYTES
    shapes = list(EDGES)
    for n, r in ((1000, 97), (1000, 75), (300, 183), (777, 33), (5000, 61), (2500, 255)):
        shapes += [(m, n, r) for m in range(r, limit // (4 * r), 3)]
    taken = [s for s in shapes if 0.98 * limit < _project_bytes(*s) <= limit]
    assert set(EDGES) <= set(taken) and len(taken) > 300
    refused = [s for s in taken if tsr.tsr_project_workspace_bytes(*s) > limit]
    assert not refused, refused[:5]


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,r", EDGES[1:3])
def test_static_scratch_at_its_limit(tsr, m, n, r):
    key = si.stream_key(813, m)
    G = si.normal((m, n), si.stream_key(key, 1))
    U, V = si.orthonormal(m, r, si.stream_key(key, 2)).float(), si.orthonormal(n, r, si.stream_key(key, 3)).float()
    C = torch.full((r, r), float("nan"), device="cuda")
    tsr.tsr_project_core_static(G.cuda(), U.cuda(), V.cuda(), C)
    ref = U.double().T @ (G.double() @ V.double())
    # two products in two bf16 pieces or finer; the core of a white gradient is sqrt(r / min(m, n)) of what the sums hold
    assert float(torch.linalg.norm(C.cpu().double() - ref) / torch.linalg.norm(ref)) < 2 * TWO_PIECES * (min(m, n) / r) ** 0.5


# ------------------------------------------------------------------ workspaces smaller than the query's
# Sizes that earlier versions of the library asked for, which a program may hold: the queries return more by now
# (k is cut into more pieces), and what these sizes are enough for is still computed in them.
HELD = [("project", (477, 376, 330), 629760), ("project", (4029, 492, 56), 1078272),
        ("refresh", (463, 491, 4, 16), 188160), ("refresh", (512, 1376, 64, 8), 4243968),
        ("refresh_workers", (324, 509, 20, 4, 2), 371712), ("realign", (296, 1760, 1), 1024), ("realign", (512, 2048, 128), 851968),
        ("one_sided", (4029, 492, 56), 1542912), ("refresh_exact", (200, 700, 50), 6326016)]
# blocks (m, n, r, row pitch), gradient type, workers, precision, refresh, p
HELD_PLANS = [([(390, 2407, 375, 2407), (76, 86, 9, 86)], 0, 1, 0, 1, 0, 52995328), ([(256, 688, 64, 688)] * 6, 1, 1, 1, 1, 8, 17071616),
              ([(768, 2048, 128, 2048)] * 5, 1, 8, 1, 0, 0, 57043968), ([(1000, 300, 64, 300)] * 3, 0, 2, 0, 0, 0, 2604032)]


def _operands(name, dims):
    """Tensors of one call, and the call itself as a function of its workspace (None: one of the query's size)."""
    import paper_2602_08007_amd as t
    gen = torch.Generator(device="cuda").manual_seed(17)
    randn = lambda *s: torch.randn(*s, device="cuda", generator=gen)  # noqa: E731
    new = lambda *s: torch.full(s, float("nan"), device="cuda")  # noqa: E731
    m, n, r = dims[:3]
    G, U, V = randn(m, n), torch.linalg.qr(randn(m, r))[0].contiguous(), torch.linalg.qr(randn(n, r))[0].contiguous()
    G += 30.0 * (U * torch.linspace(2.0, 1.0, r, device="cuda")) @ V.t()
    if name == "project":
        return lambda ws: (t.tsr_project_core(G, U, V, new(r, r), ws=ws),)
    if name == "one_sided":
        return lambda ws: (t.tsr_project_one_sided(G, U, new(n, r), ws=ws), t.tsr_backproject_one_sided(G.clone(), U, V, 1.0, ws=ws))
    if name == "realign":
        U2, V2, M = torch.linalg.qr(U + 0.01 * randn(m, r))[0].contiguous(), torch.linalg.qr(V + 0.01 * randn(n, r))[0].contiguous(), randn(r, r)
        return lambda ws: (t.tsr_realign_moment(U, V, U2, V2, M.clone(), ws=ws),)

    def refresh(ws):
        Un, Vn, sigma = new(m, r), new(n, r), new(min(m, n) if name == "refresh_exact" else r + dims[3])
        if name == "refresh_exact":
            t.tsr_refresh_exact_svd(G, r, Un, Vn, sigma, ws=ws)
        elif name == "refresh":
            t.tsr_refresh_rsvd(G, om, r, dims[3], 1, Un, Vn, sigma, ws=ws)
        else:
            t.tsr_refresh_rsvd_workers(torch.stack([G] * dims[4]), om, r, dims[3], 1, Un, Vn, sigma, ws=ws)
        return sigma[:r], Un @ Un.t(), Vn @ Vn.t()
    om = randn(n, r + dims[3]) if len(dims) > 3 else None
    return refresh


@pytest.mark.gpu
@pytest.mark.parametrize("name,dims,held", HELD)
def test_calls_run_in_a_workspace_held_from_earlier(tsr, name, dims, held):
    assert getattr(tsr, "tsr_%s_workspace_bytes" % name)(*dims) > held
    call = _operands(name, dims)
    g = Guarded(held)
    got = call(g.ws)
    g.check()
    # the same sums in fewer pieces: two results in two bf16 pieces (each off by TWO_PIECES per product, two
    # products), the projectors by that over the relative gap of the spectrum (signal 30 to 60, noise up to the
    # sum of the square roots of the sides: a factor of two at these sizes)
    for a, b in zip(got, call(None)):
        assert bool(torch.isfinite(a).all())
        assert float(torch.linalg.norm(a.double() - b.double()) / torch.linalg.norm(b.double())) < 4 * 2 * TWO_PIECES


@pytest.mark.gpu
@pytest.mark.parametrize("dims,g_dtype,workers,prec,refresh,p,held", HELD_PLANS)
def test_plans_run_in_a_workspace_held_from_earlier(tsr, dims, g_dtype, workers, prec, refresh, p, held):
    import ctypes

    def blocks():
        gen = torch.Generator(device="cuda").manual_seed(18)
        randn = lambda *s: torch.randn(*s, device="cuda", generator=gen)  # noqa: E731
        out, oms = [], []
        for m, n, r, ld in dims:
            U, V = torch.linalg.qr(randn(m, r))[0].contiguous(), torch.linalg.qr(randn(n, r))[0].contiguous()
            G = torch.zeros(workers, m, ld, device="cuda", dtype=torch.bfloat16 if g_dtype else torch.float32)
            G[:, :, :n] = (200.0 * (U * torch.linspace(2.0, 1.0, r, device="cuda")) @ V.t() + randn(workers, m, n)).to(G.dtype)
            z = lambda *s: torch.zeros(*s, device="cuda")  # noqa: E731
            out.append(dict(G=G[:, :, :n] if workers > 1 else G[0, :, :n], W=z(m, n), U=U, V=V, M=z(r, r), Vm=z(r, r), C=z(r, r),
                            D=z(r, r)))
            oms.append(randn(n, r + p))
        return out, oms

    def run(plan, bl, oms):
        if refresh:
            plan.tsr_refresh_batched(oms, 1)
        plan.tsr_step_batched(1, lr=1.0, eps=100.0)
        torch.cuda.synchronize()
        return [b["W"] for b in bl]

    bl, oms = blocks()
    plan = tsr.Plan(bl, n_workers=workers, precision=prec, with_refresh=bool(refresh), p=p)
    assert plan.ws.numel() > held
    want = run(plan, bl, oms)
    bl, oms = blocks()
    probe = tsr.Plan(bl, n_workers=workers, precision=prec, with_refresh=bool(refresh), p=p)      # (its descriptors)
    g = Guarded(held)
    small = object.__new__(tsr.Plan)
    small._handle, small.count, small._keep = ctypes.c_void_p(), len(bl), bl
    assert tsr.lib.tsr_plan_create(probe._descs, len(bl), workers, prec, refresh, p, g.ws.data_ptr(), held,
                                   torch.cuda.current_stream().cuda_stream, ctypes.byref(small._handle)) == 0
    assert small.tsr_plan_kernel_path() == plan.tsr_plan_kernel_path()
    got = run(small, bl, oms)
    g.check()
    small.close()
    # bf16 operands: two roundings (2^-9 each) that fall differently when a sum in fp32 does; else two pieces
    tol = 2 * 2.0 ** -9 if prec else 4 * 2 * TWO_PIECES
    for a, b in zip(got, want):
        assert float(torch.linalg.norm(a.double() - b.double()) / torch.linalg.norm(b.double())) < tol


@pytest.mark.skipif(torch.cuda.is_available(), reason="the calls below pass addresses that hold nothing")
@pytest.mark.parametrize("name,dims,held", HELD)
def test_held_sizes_are_not_refused(tsr, name, dims, held):
    """Without a GPU a call that is accepted ends at its first launch (-5, HIP error); one that is refused for its
    workspace ends before (-4).  A workspace below the smallest is refused."""
    import ctypes
    a, ws, null = ctypes.c_void_p(0x10000), ctypes.c_void_p(0x100000), ctypes.c_void_p(0)
    m, n, r = dims[:3]
    lib = tsr.lib
    call = {
        "project": lambda b: lib.tsr_project_core(a, 0, m, n, n, a, a, r, 1.0, 0, a, 0, ws, b, null),
        "refresh": lambda b: lib.tsr_refresh_rsvd(a, 0, m, n, n, a, r, dims[3], 1, a, a, a, ws, b, null),
        "refresh_workers": lambda b: lib.tsr_refresh_rsvd_workers(a, 0, m, n, n, m * n, dims[4], a, r, dims[3], 1, a, a, a, ws, b, null),
        "realign": lambda b: lib.tsr_realign_moment(a, a, a, a, m, n, r, a, ws, b, null),
        "one_sided": lambda b: lib.tsr_project_one_sided(a, 0, m, n, n, a, r, 1.0, 0, a, 0, ws, b, null),
        "refresh_exact": lambda b: lib.tsr_refresh_exact_svd(a, 0, m, n, n, r, a, a, a, ws, b, null),
    }[name]
    assert call(held) != -4
    assert call(256) == -4


# ------------------------------------------------------------------ host work of a single call (host)
def test_a_single_call_is_built_in_constant_time(tsr):
    """The launch of one matrix decodes its tiles from the block index: nothing the host prepares for it grows
    with the matrix (the query builds the same program as the call)."""
    import time

    def best(*dims):
        t = float("inf")
        for _ in range(50):
            start = time.perf_counter()
            for _ in range(20):
                tsr.tsr_project_workspace_bytes(*dims)
            t = min(t, time.perf_counter() - start)
        return t
    # 25008 tiles of 128 x 128 against four
    assert best(200000, 8192, 512) < 5 * best(256, 256, 128)
