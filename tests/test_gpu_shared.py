"""Builds whose phi and psi are one array, with fewer bands than orbitals (any
n_band >= 1 is allowed): the transposed copies of the split-line passes hold
every orbital that either takes, and pair symmetry is used only where the bands
include all orbitals."""
import pytest

import oracle as O
from paper_1601_07159_amd import synth
from tests._helpers import ggrid, ogrid, rel, to_gpu, to_np, tol

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec,nocc,nband", [
    (40, "fp64", 20, 10), (40, "fp64", 33, 12), (72, "fp32", 20, 10), (48, "fp64", 12, 11)])
def test_fewer_bands_without_symmetry(n, prec, nocc, nband):
    from paper_1601_07159_amd import ace
    print(f"shared array, no symmetry n={n} prec={prec} nocc={nocc} nband={nband}", flush=True)
    L = 0.43 * n
    x = synth.smooth_orbitals(n, L, nocc, seed=n)
    xg = to_gpu(x, prec)
    gg = ggrid(n, L)
    ref = O.build_W(x, x[:nband], ogrid(n, L))
    ctx = ace.Context()
    ctx.set_tuning("symmetry", 0)
    W = ctx.build_W(xg, xg[:nband], gg, prec)
    assert rel(to_np(W), ref) <= tol(prec)
    ctx.close()


@pytest.mark.parametrize("n,prec,nocc,nband", [
    (12, "fp64", 2, 1), (16, "fp32", 17, 16), (16, "fp64", 9, 3), (48, "fp64", 17, 16),
    (16, "real64", 9, 4), (16, "real32", 17, 16)])
def test_fewer_bands(n, prec, nocc, nband):
    from paper_1601_07159_amd import ace
    print(f"shared array n={n} prec={prec} nocc={nocc} nband={nband}", flush=True)
    L = 0.43 * n
    x = synth.smooth_orbitals(n, L, nocc, seed=n + nocc)
    if prec.startswith("real"):
        x = x.real
    xg, gg, og = to_gpu(x, prec), ggrid(n, L), ogrid(n, L)
    ref = O.build_W(x, x[:nband], og)
    ctx = ace.Context()
    assert rel(to_np(ctx.build_W(xg, xg[:nband], gg, prec)), ref) <= tol(prec)
    # blocks of pairs, the last ones short
    for pairs in (2, 5, 60):
        ctx.set_pair_budget(pairs * n ** 3 * (16 if prec.endswith("64") else 8))
        assert rel(to_np(ctx.build_W(xg, xg[:nband], gg, prec)), ref) <= tol(prec)
    ctx.set_pair_budget(0)
    if not prec.startswith("real"):
        a = ctx.apply_h(xg[:nband], gg, prec, phi=xg)
        b = ctx.apply_h(xg[:nband].clone(), gg, prec, phi=xg)
        assert rel(to_np(a), to_np(b)) <= tol(prec)
    ctx.close()


@pytest.mark.parametrize("form", [1, 2])
def test_fewer_bands_batched(form):
    import torch
    from paper_1601_07159_amd import ace
    print(f"shared array, batched form {form}", flush=True)
    sizes = [(16, 9, 3), (12, 5, 8), (16, 17, 16)]
    inst, refs = [], []
    for n, nocc, nband in sizes:
        L = 0.43 * n
        x = synth.smooth_orbitals(n, L, max(nocc, nband), seed=n + nband)
        xg = to_gpu(x, "fp64")
        refs.append(O.build_W(x[:nocc], x[:nband], ogrid(n, L)))
        inst.append(dict(grid=ggrid(n, L), phi=xg[:nocc], psi=xg[:nband],
                         W=torch.zeros_like(xg[:nband])))
    ctx = ace.Context()
    ctx.set_tuning("batch_form", form)
    for _ in range(2):
        ctx.build_batched(inst, "fp64")
        for d, ref in zip(inst, refs):
            assert rel(to_np(d["W"]), ref) <= tol("fp64")
    ctx.close()
