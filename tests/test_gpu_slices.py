"""The FP64 products of the compression.  The expansion (Y = A C with C's columns
in LDS slices) at its edges: one column, every slice width, a cut last block, slices of different
widths, orbital counts that are no multiple of 16, the largest count whose
slices fit and the first one past it, and grids whose last tile is cut.  The
reduction (16 x 16 blocks dealt out to waves): the first size that takes it, one
to several workgroup rows, cut blocks, real orbitals, rows that start at no
multiple of 16 bytes."""
import numpy as np
import pytest

import oracle as O
from paper_1601_07159_amd import synth
from tests._helpers import ggrid, ogrid, to_gpu, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nb,nx", [(12, 1, 1), (8, 17, 33), (12, 80, 81), (12, 97, 48), (16, 136, 64),
                                     (8, 145, 96), (16, 256, 70), (16, 304, 40), (16, 608, 17),
                                     (16, 609, 17)])
def test_apply_products(n, nb, nx):
    from paper_1601_07159_amd import ace
    print(f"expansion products n={n} nb={nb} nx={nx}", flush=True)
    L = 0.43 * n
    g, gg = ogrid(n, L), ggrid(n, L)
    rng = np.random.default_rng(nb)
    xi = rng.standard_normal((nb, n ** 3)) + 1j * rng.standard_normal((nb, n ** 3))
    X = rng.standard_normal((nx, n ** 3)) + 1j * rng.standard_normal((nx, n ** 3))
    Y = to_np(ace.apply(to_gpu(xi.reshape(nb, n, n, n), "fp64"), to_gpu(X.reshape(nx, n, n, n), "fp64"),
                        gg, "fp64")).reshape(nx, -1)
    ref = -g.dV * (xi.conj() @ X.T).T @ xi
    # sums over N_g and then nb: sqrt(4096 + 609) eps = 1.5e-14 of the largest
    # value, ten times that
    assert np.max(np.abs(Y - ref)) <= 1.5e-13 * np.max(np.abs(ref))


@pytest.mark.parametrize("nb,nx", [(97, 48), (136, 64), (145, 96), (256, 70), (304, 40), (608, 33),
                                   (609, 33)])
def test_apply_products_by_slices(nb, nx):
    """The same on a grid of enough points for slices of more than 80 orbitals."""
    from paper_1601_07159_amd import ace
    n = 24
    print(f"expansion by slices nb={nb} nx={nx}", flush=True)
    L = 0.43 * n
    g = ogrid(n, L)
    rng = np.random.default_rng(nb)
    xi = rng.standard_normal((nb, n ** 3)) + 1j * rng.standard_normal((nb, n ** 3))
    X = rng.standard_normal((nx, n ** 3)) + 1j * rng.standard_normal((nx, n ** 3))
    Y = to_np(ace.apply(to_gpu(xi.reshape(nb, n, n, n), "fp64"), to_gpu(X.reshape(nx, n, n, n), "fp64"),
                        ggrid(n, L), "fp64")).reshape(nx, -1)
    ref = -g.dV * (xi.conj() @ X.T).T @ xi
    # sums over N_g and then nb: sqrt(13824 + 609) eps = 2.7e-14 of the largest
    # value, ten times that
    assert np.max(np.abs(Y - ref)) <= 2.7e-13 * np.max(np.abs(ref))


@pytest.mark.parametrize("n,nb", [(8, 1), (12, 15), (16, 80), (16, 81), (16, 136), (16, 257)])
def test_triangular_products(n, nb):
    from paper_1601_07159_amd import ace
    print(f"triangular products n={n} nb={nb}", flush=True)
    L = 0.43 * n
    g = ogrid(n, L)
    rng = np.random.default_rng(nb)
    X = rng.standard_normal((nb, n ** 3)) + 1j * rng.standard_normal((nb, n ** 3))
    Q = to_np(ace.orthonormalize(to_gpu(X.reshape(nb, n, n, n), "fp64"), ggrid(n, L), "fp64"))
    Q = Q.reshape(nb, -1)
    assert np.max(np.abs(g.dV * (Q.conj() @ Q.T) - np.eye(nb))) <= 1e-12
    # Q spans X in order: R = <Q, X> is upper triangular
    R = g.dV * (Q.conj() @ X.T)
    assert np.max(np.abs(np.tril(R, -1))) <= 1e-12 * np.max(np.abs(R))
    assert np.max(np.abs(R.T @ Q - X)) <= 1e-12 * np.max(np.abs(X))


@pytest.mark.parametrize("prec", ["fp32", "fp64", "real32", "real64"])
@pytest.mark.parametrize("n,nb,pad", [(12, 48, 0), (12, 49, 0), (16, 81, 1), (16, 136, 0),
                                      (16, 193, 0), (16, 257, 2)])
def test_gram_products(prec, n, nb, pad):
    import torch
    from paper_1601_07159_amd import ace
    print(f"gram products prec={prec} n={n} nb={nb} pad={pad}", flush=True)
    L = 0.43 * n
    g = ogrid(n, L)
    rng = np.random.default_rng(nb)
    X = rng.standard_normal((nb, n ** 3)) + 1j * rng.standard_normal((nb, n ** 3))
    x = to_gpu(X, prec)
    pad *= 2 if prec.startswith("real") else 1     # real rows hold pairs
    rows = torch.zeros(nb, n ** 3 + pad, dtype=x.dtype, device="cuda")
    rows[:, :n ** 3] = x
    # pad 1: rows of FP32 data start between multiples of 16 bytes
    x = rows[:, :n ** 3]
    Q = to_np(ace.orthonormalize(x, ggrid(n, L), prec)).reshape(nb, -1)
    # FP64 sums; Q is stored in the data type: eps sqrt(N_g) / sqrt(N_g) per
    # entry of the Gram matrix of unit vectors, ten times that
    eps = 6e-8 if prec.endswith("32") else 1.1e-16
    tol = 10 * eps if prec.endswith("32") else 1e-12
    S = g.dV * (Q.conj() @ Q.T)
    if prec.startswith("real"):
        S = S.real
    assert np.max(np.abs(S - np.eye(nb))) <= tol


@pytest.mark.parametrize("nb", [89, 112, 136, 161])
@pytest.mark.parametrize("bad", [None, 0, 15, 16, 65, 88])
def test_panel_factorisation(nb, bad):
    """Cholesky by panels: whole and cut last panels, one to several workgroups;
    the first pivot that is not positive is reported (a zero vector's)."""
    import torch
    from paper_1601_07159_amd import ace
    n = 12
    print(f"panel factorisation nb={nb} bad={bad}", flush=True)
    L = 0.43 * n
    g = ogrid(n, L)
    rng = np.random.default_rng(nb)
    X = rng.standard_normal((nb, n ** 3)) + 1j * rng.standard_normal((nb, n ** 3))
    if bad is not None:
        X[bad] = 0.0
    info = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    Q = ace.orthonormalize(to_gpu(X.reshape(nb, n, n, n), "fp64"), ggrid(n, L), "fp64", info=info)
    torch.cuda.synchronize()
    assert int(info.item()) == (0 if bad is None else bad + 1)
    if bad is None:
        Q = to_np(Q).reshape(nb, -1)
        # 1728 products per entry of unit vectors: sqrt(1728) eps = 5e-15, with
        # a margin of a hundred for the factor's condition
        assert np.max(np.abs(g.dV * (Q.conj() @ Q.T) - np.eye(nb))) <= 5e-13


@pytest.mark.parametrize("prec", ["fp32", "mixed", "real32"])
@pytest.mark.parametrize("n,nb,nx", [(12, 31, 64), (12, 49, 33), (16, 64, 80), (16, 136, 17),
                                     (16, 130, 257), (24, 40, 96)])
def test_apply_products_fp32(prec, n, nb, nx):
    """FP32 reductions by blocks: one below the first size, cut blocks, several
    workgroup rows, chains of less and of more than four chunks."""
    from paper_1601_07159_amd import ace
    print(f"fp32 products prec={prec} n={n} nb={nb} nx={nx}", flush=True)
    L = 0.43 * n
    g = ogrid(n, L)
    rng = np.random.default_rng(nb + nx)
    xi = rng.standard_normal((nb, n ** 3)) + 1j * rng.standard_normal((nb, n ** 3))
    X = rng.standard_normal((nx, n ** 3)) + 1j * rng.standard_normal((nx, n ** 3))
    if prec == "real32":
        xi, X = xi.real, X.real
    Y = to_np(ace.apply(to_gpu(xi.reshape(nb, n, n, n), prec), to_gpu(X.reshape(nx, n, n, n), prec),
                        ggrid(n, L), prec)).reshape(nx, -1)
    ref = -g.dV * (xi.conj() @ X.T).T @ xi
    # FP32 rounding of the inputs and of chains of at most 256 products:
    # sqrt(256) 6e-8 = 1e-6 of the whole, twice that
    assert np.linalg.norm(Y - ref) <= 2e-6 * np.linalg.norm(ref)


@pytest.mark.parametrize("prec,nb,nx", [("fp64", 256, 256), ("fp64", 128, 128), ("fp64", 200, 120),
                                        ("fp32", 256, 256), ("real64", 256, 256)])
def test_noalloc_sizes(prec, nb, nx):
    """The allocation-free apply takes every size up to 256 x 256 and gives what
    apply gives, bit for bit (the grid is large enough for the full K split)."""
    import ctypes
    import torch
    from paper_1601_07159_amd import _lib, ace
    n = 24
    print(f"allocation-free apply prec={prec} nb={nb} nx={nx}", flush=True)
    gg = ggrid(n, 0.43 * n)
    dt = {"fp64": torch.complex128, "fp32": torch.complex64, "real64": torch.float64}[prec]
    gen = torch.Generator(device="cuda").manual_seed(nb)
    xi = torch.randn(nb, n ** 3, dtype=dt, device="cuda", generator=gen)
    X = torch.randn(nx, n ** 3, dtype=dt, device="cuda", generator=gen)
    Y = torch.full_like(X, float("nan"))
    ctx = ace.Context()
    g = gg.as_c()
    ctx._bind_stream()
    st = _lib.load().ace_apply_noalloc(
        ctx._h, ctypes.byref(g), ace._prec(prec), ctypes.c_void_p(xi.data_ptr()), nb, xi.stride(0),
        ctypes.c_void_p(X.data_ptr()), nx, X.stride(0), ctypes.c_void_p(Y.data_ptr()), Y.stride(0))
    assert st == 0
    assert torch.equal(Y, ctx.apply(xi, X, gg, prec))
    ctx.close()


@pytest.mark.parametrize("n,nb,nx", [(24, 96, 96), (24, 100, 100), (24, 256, 130), (16, 256, 250),
                                     (48, 256, 256)])
def test_reduction_forms(n, nb, nx):
    """FP64 reductions by blocks that fill their waves and that do not, with few and
    with many splits (256 x 256: fewer, so that the partials fit the allocation-free
    apply)."""
    import ctypes
    import torch
    from paper_1601_07159_amd import _lib, ace
    print(f"reduction forms n={n} nb={nb} nx={nx}", flush=True)
    gg = ggrid(n, 0.43 * n)
    gen = torch.Generator(device="cuda").manual_seed(nb)
    xi = torch.randn(nb, n ** 3, dtype=torch.complex128, device="cuda", generator=gen)
    X = torch.randn(nx, n ** 3, dtype=torch.complex128, device="cuda", generator=gen)
    Y = torch.full_like(X, float("nan"))
    ctx = ace.Context()
    g = gg.as_c()
    ctx._bind_stream()
    st = _lib.load().ace_apply_noalloc(
        ctx._h, ctypes.byref(g), ace._prec("fp64"), ctypes.c_void_p(xi.data_ptr()), nb, xi.stride(0),
        ctypes.c_void_p(X.data_ptr()), nx, X.stride(0), ctypes.c_void_p(Y.data_ptr()), Y.stride(0))
    assert st == 0
    assert torch.equal(Y, ctx.apply(xi, X, gg, "fp64"))
    ctx.close()
    ref = -gg.dV * ((xi.conj() @ X.T.contiguous()).T.contiguous() @ xi)
    # sums over N_g and then nb: sqrt(N_g + nb) eps of the largest value, ten times that
    tol = 10 * np.sqrt(n ** 3 + nb) * 2.2e-16
    assert float((Y - ref).abs().max()) <= tol * float(ref.abs().max())


@pytest.mark.parametrize("prec,nb,nx", [("fp64", 96, 17), ("fp64", 161, 32), ("fp32", 272, 17)])
def test_small_imaginary_parts(prec, nb, nx):
    """Orbitals that are all but real: the imaginary parts of <xi_a, X_b> are as
    exact as their own terms, not as the real parts.  xi is the identity on its
    first nb grid points, where Y = V_ACE X then holds -<xi_a, X_b> itself."""
    from paper_1601_07159_amd import ace
    n = 24
    print(f"small imaginary parts prec={prec} nb={nb} nx={nx}", flush=True)
    L, K = 0.43 * n, n ** 3
    g = ogrid(n, L)
    small, eps = (1e-8, 1.1e-16) if prec == "fp64" else (1e-4, 6e-8)
    t = 2 * np.pi * np.arange(K) / K
    kx, ky = np.arange(nb)[:, None], np.arange(nx)[:, None]
    xi = 1 + 0.4 * np.cos((kx % 17 + 1) * t) + 1j * small * np.sin((kx % 13 + 1) * t)
    X = 1 + 0.4 * np.cos((ky + 2) * t) + 1j * small * np.cos((ky + 5) * t)
    xi[:, :nb] = np.eye(nb)
    dt = np.complex128 if prec == "fp64" else np.complex64
    xi, X = xi.astype(dt), X.astype(dt)
    Y = to_np(ace.apply(to_gpu(xi.reshape(nb, n, n, n), prec), to_gpu(X.reshape(nx, n, n, n), prec),
                        ggrid(n, L), prec)).reshape(nx, -1)[:, :nb]
    ld = np.longdouble
    xr, xm, Xr, Xm = (v.astype(ld) for v in (xi.real, xi.imag, X.real, X.imag))
    ref = -ld(g.dV) * (Xm @ xr.T - Xr @ xm.T)
    # chains of 128 terms, each at most 3 small, added up over K points: a random
    # walk of sqrt(128) roundings in each chain, times ten (the real parts' own
    # rounding, K g.dV eps, is 1e8 and 1e4 times the terms')
    bound = 10 * np.sqrt(128) * eps * 3 * small * K * g.dV
    assert np.max(np.abs(Y.imag - ref)) <= bound


@pytest.mark.parametrize("prec,nb,nx", [("fp64", 96, 48), ("fp32", 272, 48), ("fp32", 96, 72)])
def test_small_imaginary_parts_expanded(prec, nb, nx):
    """The same for the expansion by slices, more orbitals than three products
    are taken for: Im Y is as exact as its own terms."""
    from paper_1601_07159_amd import ace
    n = 24
    print(f"small imaginary parts, expanded prec={prec} nb={nb} nx={nx}", flush=True)
    L, K = 0.43 * n, n ** 3
    g = ogrid(n, L)
    small, eps = (1e-8, 1.1e-16) if prec == "fp64" else (1e-6, 6e-8)
    t = 2 * np.pi * np.arange(K) / K
    kx, ky = np.arange(nb)[:, None], np.arange(nx)[:, None]
    xi = 1 + 0.4 * np.cos((kx % 17 + 1) * t) + 1j * small * np.sin((kx % 13 + 1) * t)
    X = 1 + 0.4 * np.cos((ky + 2) * t) + 1j * small * np.cos((ky + 5) * t)
    dt = np.complex128 if prec == "fp64" else np.complex64
    xi, X = xi.astype(dt), X.astype(dt)
    Y = to_np(ace.apply(to_gpu(xi.reshape(nb, n, n, n), prec), to_gpu(X.reshape(nx, n, n, n), prec),
                        ggrid(n, L), prec)).reshape(nx, -1)
    ld = np.longdouble
    xr, xm, Xr, Xm = (v.astype(ld) for v in (xi.real, xi.imag, X.real, X.imag))
    cr, cm = -(xr @ Xr.T + xm @ Xm.T), -(xr @ Xm.T - xm @ Xr.T)
    at = np.random.default_rng(nx).integers(0, K, 48)
    ref = ld(g.dV) * (xr[:, at].T @ cm + xm[:, at].T @ cr).T
    # terms xi_r C_m and xi_m C_r of at most 1.4 * 3 small K dV and small * 2 K dV,
    # nb of each; a random walk of the reduction's chains (128 terms) and of the
    # expansion's (2 nb), times ten
    bound = 10 * (np.sqrt(128) + np.sqrt(2 * nb)) * eps * nb * 6.2 * small * K * g.dV
    assert np.max(np.abs(Y[:, at].imag - ref)) <= bound


@pytest.mark.parametrize("prec,nb,nx", [("real64", 96, 48), ("real64", 161, 33), ("real32", 272, 48)])
def test_real_neighbours(prec, nb, nx):
    """Real orbitals go through the products as pairs of grid values: the small
    value of a pair is as exact as its own terms, whatever its neighbour."""
    from paper_1601_07159_amd import ace
    n = 24
    print(f"real neighbours prec={prec} nb={nb} nx={nx}", flush=True)
    L, K = 0.43 * n, n ** 3
    g = ogrid(n, L)
    small, eps, dt = (1e-8, 1.1e-16, np.float64) if prec == "real64" else (1e-6, 6e-8, np.float32)
    t = 2 * np.pi * np.arange(K) / K
    xi = 1 + 0.4 * np.cos((np.arange(nb)[:, None] % 17 + 1) * t)
    X = (1 + 0.4 * np.cos((np.arange(nx)[:, None] + 2) * t)).astype(dt)
    xi[:, 1::2] *= small
    xi = xi.astype(dt)
    Y = to_np(ace.apply(to_gpu(xi.reshape(nb, n, n, n), prec), to_gpu(X.reshape(nx, n, n, n), prec),
                        ggrid(n, L), prec)).real.reshape(nx, -1)
    ld = np.longdouble
    xi, X = xi.astype(ld), X.astype(ld)
    at = 2 * np.random.default_rng(nx).integers(0, K // 2, 48) + 1
    ref = -ld(g.dV) * (xi[:, at].T @ (xi @ X.T)).T
    # nb terms of at most 1.4 small times 2 K dV; a random walk of the reduction's
    # chains (128 terms) and of the expansion's (nb), times ten
    bound = 10 * (np.sqrt(128) + np.sqrt(nb)) * eps * nb * 2.8 * small * K * g.dV
    assert np.max(np.abs(Y[:, at] - ref)) <= bound
