"""The slab and plane passes on split lines (every size and precision that takes
them) against the quad forms, which have the oracle tests: runs of pairs with
every kind of remainder, the symmetric, rectangular and blocked plans, orbitals
with a larger leading dimension, the direct energy, and a captured call whose
workspace has no room for the transposed orbitals."""
import pytest

from paper_1601_07159_amd import synth
from tests._helpers import ggrid, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec,nocc,nband", [
    (40, "fp64", 29, 33),   # runs of 8 (slab) and 4 (plane) and their remainders
    (40, "fp64", 16, 16),   # the fewest pairs that take it
    (40, "fp64", 15, 15),   # quads
    (48, "fp64", 17, 18),   # runs of 3
    (64, "fp64", 12, 13),   # runs of 2
    (72, "fp64", 11, 14),
    (72, "fp32", 22, 25),   # runs of 8; a last wave half filled
    (72, "fp32", 9, 9),
    (64, "fp32", 17, 20),   # plane pass only
])
def test_split_lines_equal_quads(n, prec, nocc, nband):
    import torch
    from paper_1601_07159_amd import ace
    print(f"split lines n={n} prec={prec} nocc={nocc} nband={nband}", flush=True)
    L = 0.43 * n
    gg = ggrid(n, L, "erfc", 0.2)
    base = to_gpu(synth.smooth_orbitals(n, L, 6, seed=n), prec)
    gen = torch.Generator(device="cuda").manual_seed(nband)
    mix = torch.randn(nband, 6, dtype=base.dtype, device="cuda", generator=gen)
    x = torch.zeros(nband, 2, n, n, n, dtype=base.dtype, device="cuda")[:, 0]
    for b in range(nband):
        for k in range(6):
            x[b] += mix[b, k] * base[k]
    pair = n ** 3 * base.element_size()
    out = []
    for shape in (0, 4):
        ctx = ace.Context()
        ctx.set_tuning("fft_shape", shape)
        ctx.set_tuning("accum_shape", 16)
        r = [ctx.build_W(x[:nocc], x, gg, prec), ctx.build_W(x[:nocc].clone(), x, gg, prec),
             ctx.exchange_energy(x[:nocc].contiguous(), gg, prec)]
        ctx.set_tuning("pair_budget", 37 * pair)
        r += [ctx.build_W(x[:nocc], x, gg, prec), ctx.exchange_energy(x[:nocc].contiguous(), gg, prec)]
        ctx.close()
        out.append(r)
    # FP64: some 3 log2(n) roundings per value on each of the two transforms,
    # 40 eps = 9e-15 of the largest value; FP32 likewise 40 eps =
    # 5e-6
    for a, b in zip(*out):
        err = float((a - b).abs().max() / b.abs().max())
        assert err <= (1e-14 if prec == "fp64" else 5e-6), err


def test_captured_without_room_for_copies():
    import torch
    from paper_1601_07159_amd import ace
    n, nocc, nband = 48, 12, 14
    print("split lines: captured without room for the copies", flush=True)
    gg = ggrid(n, 0.43 * n)
    x = to_gpu(synth.smooth_orbitals(n, 0.43 * n, nband, seed=5), "fp64")
    ref = ace.Context()
    ctx = ace.Context()
    W = torch.zeros_like(x)
    ctx.set_tuning("fft_shape", 4)       # takes no copies
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        ctx.build_W(x[:nocc], x, gg, "fp64", out=W)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    ctx.set_tuning("fft_shape", 0)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.build_W(x[:nocc], x, gg, "fp64", out=W)
    for rep in range(3):
        x.mul_(1.0 + rep)
        W.zero_()
        graph.replay()
        torch.cuda.synchronize()
        want = ref.build_W(x[:nocc], x, gg, "fp64")
        # 40 eps of the largest value, as above
        assert float((W - want).abs().max() / want.abs().max()) <= 1e-14
    del graph
    ctx.close()
    ref.close()


@pytest.mark.parametrize("n,prec,nocc,nband", [(48, "fp64", 12, 14), (72, "fp32", 9, 11)])
def test_captured_after_reserve(n, prec, nocc, nband):
    import torch
    from paper_1601_07159_amd import ace
    print(f"split lines: captured after reserve n={n} prec={prec}", flush=True)
    gg = ggrid(n, 0.43 * n)
    x = to_gpu(synth.smooth_orbitals(n, 0.43 * n, nband, seed=6), prec)
    own = x[:nocc].flip(0).contiguous()
    ref, ctx = ace.Context(), ace.Context()
    ctx.reserve(gg, prec, nocc, nband, nband)
    Ws, Wo, e = torch.zeros_like(x), torch.zeros_like(x), torch.zeros((), dtype=torch.float64,
                                                                      device="cuda")

    def path(c, W1, W2, en):
        c.build_W(x[:nocc], x, gg, prec, out=W1)
        c.build_W(own, x, gg, prec, out=W2)
        return c.exchange_energy(own, gg, prec, out=en)

    path(ref, torch.zeros_like(x), torch.zeros_like(x), torch.zeros_like(e))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        path(ctx, Ws, Wo, e)
    for rep in range(3):
        x.mul_(1.0 + 0.5 * rep)
        own.mul_(1.0 - 0.25 * rep)
        Ws.zero_(), Wo.zero_()
        graph.replay()
        torch.cuda.synchronize()
        W1, W2, en = torch.zeros_like(x), torch.zeros_like(x), torch.zeros_like(e)
        path(ref, W1, W2, en)
        torch.cuda.synchronize()
        # the same kernels on the same data
        assert torch.equal(Ws, W1) and torch.equal(Wo, W2) and torch.equal(e, en)
    del graph
    ctx.close()
    ref.close()


@pytest.mark.parametrize("n,nocc,nband", [(24, 10, 40), (32, 12, 40), (40, 10, 30)])
def test_chunks_take_the_form_of_the_build(n, nocc, nband):
    """FP64 builds of many pairs cut into bands blocks of few: the same lines, so
    the same results bit for bit (every band's orbitals stay in one chunk); the
    direct energy in chunks of pairs likewise."""
    import torch
    from paper_1601_07159_amd import ace
    print(f"band blocks n={n} nocc={nocc} nband={nband}", flush=True)
    gg = ggrid(n, 0.43 * n, "erfc", 0.2)
    x = to_gpu(synth.smooth_orbitals(n, 0.43 * n, nband, seed=n), "fp64")
    phi = x[:nocc].clone()
    ctx = ace.Context()
    W, e = ctx.build_W(phi, x, gg, "fp64"), ctx.exchange_energy(x, gg, "fp64")
    ctx.set_tuning("jblock", 8)
    assert torch.equal(ctx.build_W(phi, x, gg, "fp64"), W)
    ctx.set_pair_budget(50 * n ** 3 * 16)
    assert torch.equal(ctx.exchange_energy(x, gg, "fp64"), e)
    ctx.close()


@pytest.mark.parametrize("n,prec,nocc,nband", [
    (64, "real32", 17, 20), (64, "real32", 9, 9), (72, "real32", 12, 13),  # plane pass alone
    (72, "fp32", 22, 25), (72, "fp32", 9, 9)])                             # slab and plane
def test_fp32_split_lines_are_the_quads_bit_for_bit(n, prec, nocc, nband):
    """FP32 lines round every product as the quad forms do."""
    import torch
    from paper_1601_07159_amd import ace
    print(f"fp32 split lines n={n} prec={prec} nocc={nocc} nband={nband}", flush=True)
    for kind, mu in (("coulomb", 0.0), ("erfc", 0.2)):
        gg = ggrid(n, 0.43 * n, kind, mu)
        x = to_gpu(synth.smooth_orbitals(n, 0.43 * n, nband, seed=n + nocc), prec)
        gen = torch.Generator(device="cuda").manual_seed(n)
        x += 1e-3 * torch.randn(x.shape, dtype=x.dtype, device="cuda", generator=gen)
        out = []
        for shape in (0, 4):
            ctx = ace.Context()
            ctx.set_tuning("fft_shape", shape)
            out.append([ctx.build_W(x[:nocc], x, gg, prec), ctx.build_W(x[:nocc].clone(), x, gg, prec)])
            if prec == "fp32":
                out[-1].append(ctx.exchange_energy(x[:nocc].contiguous(), gg, prec))
            ctx.close()
        for a, b in zip(*out):
            assert torch.equal(a, b)
