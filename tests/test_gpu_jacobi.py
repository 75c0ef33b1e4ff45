"""Rayleigh-Ritz at the edges of the Jacobi eigensolver's forms: one, two and
three vectors, the last size of the small and of the middle form with the
vectors turned along and the first ones past them, an odd count (padded), the last size with A in LDS and the first
ones in global memory, and the counts where a lane of the vector kernel takes a
second and a third pair."""
import numpy as np
import pytest

import oracle as O
from paper_1601_07159_amd import synth
from tests._helpers import ggrid, ogrid, to_gpu, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [1, 2, 3, 15, 16, 17, 31, 32, 33, 63, 87, 88, 89, 128, 129, 257])
def test_ritz_pairs(nb):
    from paper_1601_07159_amd import ace
    n, L = 16, 12.0
    print(f"ritz pairs nb={nb}", flush=True)
    g = ogrid(n, L)
    X = O.orthonormalize(synth.smooth_orbitals(n, L, nb, seed=nb), g).reshape(nb, -1)
    rng = np.random.default_rng(nb)
    H = rng.standard_normal((nb, nb)) + 1j * rng.standard_normal((nb, nb))
    H = 0.5 * (H + H.conj().T)
    # rows: (H X)_b = sum_a H_ab x_a, so that <x_a, (H X)_b> = H_ab
    HX = H.T @ X
    ctx = ace.Context()
    shape = (nb, n, n, n)
    Xg, Hg, e = ctx.rayleigh_ritz(to_gpu(X.reshape(shape), "fp64"), to_gpu(HX.reshape(shape), "fp64"),
                                  ggrid(n, L), "fp64")
    Xg, Hg, e = to_np(Xg).reshape(nb, -1), to_np(Hg).reshape(nb, -1), e.cpu().numpy()
    # rounding of nb products per entry and some ten sweeps of nb rotations:
    # 257 * 10 * eps = 6e-13 of the norm
    tol = 1e-11 * np.linalg.norm(H)
    assert np.max(np.abs(e - np.linalg.eigvalsh(H))) <= tol
    scale = np.sqrt(g.dV)
    assert np.max(np.linalg.norm(scale * (Hg - e[:, None] * Xg), axis=1)) <= tol
    assert np.max(np.abs(g.dV * (Xg.conj() @ Xg.T) - np.eye(nb))) <= 1e-11
    ctx.close()
