"""The GEMM kernels for outputs of few tiles against float64, at the edges of their tiles, of their ring of LDS stages and of the reduction
segments; nothing outside the output is written."""
import pytest
import torch

from paper_2506_03077_amd import binding as sb

pytestmark = pytest.mark.gpu

TILES = [(128, 128), (128, 64), (64, 64)]


def run(M, N, Ks, tb, out, tile, seed=0):
    gen = torch.Generator(device="cuda").manual_seed(seed + M + N + sum(Ks))
    r = lambda *s: (torch.randn(s, generator=gen, device="cuda") * 0.5).bfloat16()
    As, Bs = [r(M, k) for k in Ks], [r(N, k) if tb else r(k, N) for k in Ks]
    ldc = N + 16
    buf = torch.full((M + 2, ldc), 77.0, dtype=out, device="cuda")
    assert sb.debug_gemm_few(As, Bs, buf[1:M + 1, :N], tb, tile) == 1
    want = sum(a.double().cpu() @ (b.double().cpu().t() if tb else b.double().cpu()) for a, b in zip(As, Bs))
    got = buf[1:M + 1, :N].double().cpu()
    # fp32 sums of exact products: rounding of the partial sums, at most K 2^-24 of the sum of magnitudes, far less on average; bf16: half an ulp more
    mag = sum(a.double().abs().cpu() @ (b.double().abs().cpu().t() if tb else b.double().abs().cpu()) for a, b in zip(As, Bs))
    bound = mag * sum(Ks) ** 0.5 * 2.0 ** -24 + (want.abs() * 2.0 ** -8 if out == torch.bfloat16 else 0.0)
    assert bool(((got - want).abs() <= bound + 1e-30).all())
    buf[1:M + 1, :N] = 77.0
    assert bool((buf == 77.0).all())


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("tb", [True, False])
@pytest.mark.parametrize("out", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M,N,Ks", [
    (1, 8, (128,)), (64, 64, (128,)), (65, 72, (256,)), (129, 136, (384,)), (128, 128, (512,)),       # 1 .. 4 (or twice as many) steps
    (63, 200, (640,)), (300, 328, (768,)), (127, 1000, (1152,)),                                       # past the ring, ragged tiles
    (200, 264, (256, 384)), (130, 72, (128, 128, 128)), (70, 136, (1024, 128, 640))])                  # segments, odd and even, of one step
def test_few_tiles_match_fp64(tile, tb, out, M, N, Ks):
    run(M, N, Ks, tb, out, tile)


@pytest.mark.parametrize("tile", TILES[:2])
@pytest.mark.parametrize("tb", [True, False])
@pytest.mark.parametrize("Ks", [(64,), (192,), (320, 64), (64, 64, 64)])      # 64-wide steps: odd numbers of them
def test_few_tiles_odd_steps(tile, tb, Ks):
    run(200, 136, Ks, tb, torch.float32, tile)


def test_few_tiles_refuse_what_they_do_not_take():
    r = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")
    C = torch.zeros((64, 64), device="cuda")
    assert sb.debug_gemm_few([r(64, 192)], [r(64, 192)], C, True, (64, 64)) == 0       # 64 x 64 tiles take 128-wide steps
    assert sb.debug_gemm_few([r(64, 100)], [r(64, 100)], C, True, (128, 64)) == 0      # a ragged reduction
    assert sb.debug_gemm_few([r(64, 128)], [r(64, 128)], C, True, (32, 64)) == 0       # no such tile
    assert sb.debug_gemm_few([r(64, 128)], [r(60, 128)], torch.zeros((64, 60), device="cuda"), True, (64, 64)) == 0   # rows of 8 columns


def _check(got, pairs, tb):   # as in run()
    wide = [(a.double().cpu(), b.double().cpu().t() if tb else b.double().cpu()) for a, b in pairs]
    want, mag = sum(a @ b for a, b in wide), sum(a.abs() @ b.abs() for a, b in wide)
    bound = mag * sum(a.shape[1] for a, _ in wide) ** 0.5 * 2.0 ** -24 + (want.abs() * 2.0 ** -8 if got.dtype == torch.bfloat16 else 0.0)
    assert bool(((got.double().cpu() - want).abs() <= bound + 1e-30).all())


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("tb", [True, False])
@pytest.mark.parametrize("out", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n", [1, 2, 8])
def test_problems_of_their_own_sizes_in_one_launch(tile, tb, out, n):
    """Every workgroup finds its problem, of one to twelve tiles and one or two operand pairs, by its number."""
    sizes = [(130, 72, 256), (1, 8, 128), (64, 200, 640), (257, 64, 128), (128, 128, 384), (65, 264, 256), (7, 16, 1152), (200, 136, 512)][:n]
    gen = torch.Generator(device="cuda").manual_seed(3)
    r = lambda *s: (torch.randn(s, generator=gen, device="cuda") * 0.5).bfloat16()
    pair = lambda M, N, K: (r(M, K), r(N, K) if tb else r(K, N))
    first, second = [pair(*s) for s in sizes], [pair(*s) if i % 2 else None for i, s in enumerate(sizes)]
    bufs = [torch.full((M + 2, N + 8), 77.0, dtype=out, device="cuda") for M, N, _ in sizes]
    Cs = [b[1:-1, :-8] for b in bufs]
    assert sb.debug_gemm_few_problems([a for a, _ in first], [b for _, b in first], Cs, tb, tile, [p and p[0] for p in second], [p and p[1] for p in second]) == 1
    for C, one, two, buf in zip(Cs, first, second, bufs):
        _check(C, [one] + ([two] if two else []), tb)
        C.fill_(77.0)
        assert bool((buf == 77.0).all())
