"""The dense eigensolver (spectra, exact NormPre-L) at the sizes where its
kernels change: orders around the one-workgroup block of the reduction (256),
around each change of threads and columns per thread of the per-column
launches up to the largest order, active sides longer and shorter than the other, and spectra with
clusters, zeros and no coupling at all."""
import math

import numpy as np
import pytest
import torch

from oracle import normpre_oracle as O
from paper_2609_36692_amd import normpre as N
from paper_2609_36692_amd import workloads as WL
from parity_util import check_update

pytestmark = pytest.mark.gpu

U16, U24 = 2.0 ** -11, 2.0 ** -24


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = N.normpre_init(0)
    yield c
    N.normpre_destroy(c)


def _inputs(shape, kind="lowrank", seed=0):
    wl = WL.Workload("t", 90 + seed, [shape], kind, 1.0, rank=8)
    return WL.make_matrix(wl, 0, "cpu", shape=shape)


def _momentum(kind, shape):
    if kind == "identity":          # orthonormal rows: Gamma = I, no reflection anywhere
        m = torch.zeros(shape)
        m.diagonal().fill_(3.0)
        return m
    if kind == "repeated":          # 16 groups of equal orthogonal rows: clusters and exact zeros
        m = torch.zeros(shape)
        m[torch.arange(shape[0]), torch.arange(shape[0]) % 16] = 2.0
        return m
    if kind == "zero":
        return torch.zeros(shape)
    if kind == "rank4":             # computed eigenvalues of rounding size, of either sign
        gen = torch.Generator().manual_seed(5)
        return torch.randn(shape[0], 4, generator=gen) @ torch.randn(4, shape[1], generator=gen)
    w, g, mp = _inputs(shape, kind, seed=13)
    return (0.95 * mp + g) * torch.linspace(0.3, 3.0, shape[0])[:, None]


@pytest.mark.parametrize("shape,t,kind", [
    ((1, 300), 0, "lowrank"), ((2, 300), 0, "lowrank"), ((33, 64), 0, "lowrank"), ((255, 300), 0, "lowrank"),
    ((256, 400), 0, "lowrank"), ((257, 400), 0, "lowrank"), ((511, 600), 0, "lowrank"), ((577, 600), 0, "lowrank"),
    ((770, 900), 1, "lowrank"), ((1090, 1200), 0, "student_t"), ((2113, 2200), 0, "student_t"),
    ((900, 257), 0, "lowrank"), ((300, 1100), 1, "lowrank"), ((700, 1), 0, "lowrank"),
    ((300, 600), 0, "identity"), ((300, 600), 0, "repeated"), ((290, 310), 0, "zero"),
    ((700, 300), 0, "rank4"), ((260, 800), 1, "rank4"), ((600, 290), 0, "repeated"), ((310, 290), 0, "zero")])
def test_spectrum_of_the_rounded_psi(ctx, shape, t, kind):
    print(f"spectrum shape={shape} t={t} {kind}", flush=True)
    m = _momentum(kind, shape)
    w = torch.zeros(shape)
    hp = N.normpre_default_hparams(step=t)
    eig = N.normpre_spectrum(ctx, N.NORMPRE_SPECTRUM_GAMMA, w.cuda(), m.cuda(), hp)
    psi = O.diagonal_gram_normalize(O.orient(m.double().numpy(), t % 2)).astype(np.float16).astype(np.float64)
    ref = np.sort(np.linalg.eigvalsh(psi @ psi.T))[::-1]
    assert eig.shape == ref.shape and np.all(np.diff(eig) <= 1e-12 * max(ref[0], 1.0))
    n = min(shape)
    # Each of the n reflections rounds the stored fp32 matrix once (2^-24 of
    # entries of at most lambda_max); the Gram accumulates in fp32; a Psi entry
    # whose fp32 and fp64 values straddle an fp16 rounding boundary is off by
    # one unit, rare enough to stay within the same order.
    tol = (2.0 * n + 256.0) * U24 * max(ref[0], 1e-300)
    err = float(np.max(np.abs(eig - ref)))
    print(f"  max error {err:.2e} (tol {tol:.1e}) lambda_max {ref[0]:.3f}", flush=True)
    assert err <= tol


# The largest orders (above 4096 the per-column launches have 1024 threads, and the
# multisection's matrix takes more than 64 KB of LDS): rows 0.8 e_i + 0.6 e_{i+1} in
# random order, whose Gamma is a permuted tridiagonal Toeplitz matrix of known
# eigenvalues d + 2 o cos(k pi / (n + 1)), d and o from the rounded entries.
@pytest.mark.parametrize("n", [4097, 5000, 8192])
def test_spectrum_of_large_orders(ctx, n):
    print(f"spectrum order {n}", flush=True)
    i = torch.arange(n, device="cuda")
    r = torch.randperm(n, generator=torch.Generator().manual_seed(3)).cuda()
    m = torch.zeros(n, (n + 4) // 4 * 4, device="cuda")
    m[r, i] = 0.8
    m[r, i + 1] = 0.6
    eig = N.normpre_spectrum(ctx, N.NORMPRE_SPECTRUM_GAMMA, torch.zeros_like(m), m, N.normpre_default_hparams(step=0))
    a, b = (float(np.float16(v)) for v in (0.8, 0.6))
    ref = a * a + b * b + 2.0 * a * b * np.cos(np.arange(1, n + 1) * math.pi / (n + 1))
    assert eig.shape == ref.shape and np.all(np.diff(eig) <= 1e-12)
    tol = (2.0 * n + 256.0) * U24 * ref[0]
    err = float(np.max(np.abs(eig - ref)))
    print(f"  max error {err:.2e} (tol {tol:.1e})", flush=True)
    assert err <= tol


def _exact(ctx, mats, t, rank, flags=0):
    Ws, Gs, Ms = ([x[i].cuda().clone() for x in mats] for i in range(3))
    hp = N.normpre_default_hparams(lr=1.0, weight_decay=0.0, step=t, rank=rank,
                                   flags=N.NORMPRE_FLAG_L_EXACT | flags)
    N.normpre_step(ctx, N.NORMPRE_VARIANT_L, Ws, Gs, Ms, hp)
    torch.cuda.synchronize()
    for i, (mat, W) in enumerate(zip(mats, Ws)):
        ref = O.normpre_step(*(x.numpy() for x in mat), t, O.HParams(lr=1.0, weight_decay=0.0, rank=rank), "L",
                             matrix_id=i, l_mode="exact")
        kappa = math.sqrt(float(np.sum(ref["lam_sel"]))) / max(np.linalg.norm(ref["t"]), 1e-300)
        u = mat[0].double().numpy() - W.cpu().double().numpy()
        err = check_update(f"L exact {tuple(mat[0].shape)} r={rank} t={t}", u, ref["update"],
                           max(1e-2, 8.0 * U16 * kappa))
        print(f"  matrix {i}: update err {err:.2e}, |C| = {len(ref['lam_sel'])}", flush=True)


# Active side longer than the other (fewer nonzero eigenvalues than wanted,
# and more), equal, one longer; above the order whose inverse iteration keeps
# its factors in LDS.
@pytest.mark.parametrize("shape,t,rank", [((500, 20), 0, 32), ((900, 31), 0, 32), ((20, 500), 1, 8),
                                          ((400, 390), 0, 32), ((390, 400), 0, 32), ((520, 520), 1, 48),
                                          ((640, 400), 0, 4), ((2810, 2830), 0, 8)])
def test_exact_either_side(ctx, shape, t, rank):
    print(f"L exact shape={shape} t={t} r={rank}", flush=True)
    _exact(ctx, [_inputs(shape, seed=21)], t, rank)


# Matrices of different shapes whose eigenproblems have one order are solved
# together; others of another order in the same step.
@pytest.mark.parametrize("t", [0, 1])
def test_exact_pooled_orders(ctx, t):
    shapes = [(600, 450), (450, 700), (600, 450), (520, 500), (700, 450)]
    print(f"L exact pooled t={t}", flush=True)
    _exact(ctx, [_inputs(sh, seed=30 + i) for i, sh in enumerate(shapes)], t, 16)
