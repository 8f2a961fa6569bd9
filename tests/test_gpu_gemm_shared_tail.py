"""A last round of 129 to 160 tiles whose reductions are shared with the CUs that have no tile: ends of that range, whole rounds before it, ragged
rows, columns and pieces, one operand pair and two, scratch that holds NaN."""
import pytest
import torch

from paper_2506_03077_amd import binding as sb

pytestmark = pytest.mark.gpu


# rows, columns, K: 129 tiles (127 helpers, two last tiles in eight pieces), 140, 160 (64 last tiles in one piece), 256 + 130
@pytest.mark.parametrize("M,N,K", [(700, 11008, 5440), (2500, 3584, 5888), (2560, 4088, 7168), (2560, 9976, 5504)])
@pytest.mark.parametrize("layout", ["nt", "nn"])
@pytest.mark.parametrize("pair", [False, True])
def test_shared_tail(M, N, K, layout, pair):
    tb = layout == "nt"
    K = -(-K // 128) * 64 if pair else K
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    r = lambda *s: torch.randn(s, generator=gen, device="cuda").bfloat16()
    ops = [(r(M, K), r(N, K) if tb else r(K, N)) for _ in range(2 if pair else 1)]
    want = sum(a.double() @ (b.double().t() if tb else b.double()) for a, b in ops)
    scratch = torch.full((64 << 20,), 0xFF, dtype=torch.uint8, device="cuda")
    got = []
    for _ in range(2):
        C = torch.full((M, N), float("nan"), device="cuda")
        more = dict(A2=ops[1][0], B2=ops[1][1]) if pair else {}
        assert sb.debug_gemm(ops[0][0], ops[0][1], C, M, N, K, False, tb, scratch=scratch, **more) == 1
        got.append(C)
    assert bool((scratch.view(torch.int32)[:65536] != -1).any()), "nothing was shared"
    # sums of K products of N(0, 1) values in fp32, in any order: below K ulp of the typical sum sqrt(K)
    terms = K * len(ops)
    assert float((got[0].double() - want).abs().max()) <= terms * 2.0 ** -23 * terms ** 0.5
    assert torch.equal(got[0], got[1])


# 129 tiles, two of them cut up; steps of their rest: 33, 42 and 49 do not make eight pieces of equal length, 35 in two operand pairs, 48 does
@pytest.mark.parametrize("steps,pair,pieces", [(76, False, 7), (95, False, 7), (110, False, 7), (80, True, 7), (107, False, 8)])
def test_no_piece_is_without_a_step(steps, pair, pieces):
    """A piece that starts behind the last step would write a tile of zeros, which the sum then adds."""
    M, N, K = 700, 11008, 64 * steps // (2 if pair else 1)
    gen = torch.Generator(device="cuda").manual_seed(steps)
    r = lambda *s: torch.randn(s, generator=gen, device="cuda").bfloat16()
    ops = [(r(M, K), r(N, K)) for _ in range(2 if pair else 1)]
    want = sum(a.double() @ b.double().t() for a, b in ops)
    scratch, C = torch.full((64 << 20,), 0xFF, dtype=torch.uint8, device="cuda"), torch.full((M, N), float("nan"), device="cuda")
    more = dict(A2=ops[1][0], B2=ops[1][1]) if pair else {}
    assert sb.debug_gemm(ops[0][0], ops[0][1], C, M, N, K, False, True, scratch=scratch, **more) == 1
    slots = scratch.view(torch.int32).view(256, -1)
    written = (slots != -1).any(dim=1)
    assert int(written.sum()) == 127 + 2 * pieces and bool((slots[written] != 0).any(dim=1).all())
    terms = 64 * steps
    assert float((C.double() - want).abs().max()) <= terms * 2.0 ** -23 * terms ** 0.5


def test_other_tails_are_not_shared():
    """128 tiles split evenly, 161 and more are left whole."""
    for tiles_m, tiles_n in ((8, 16), (7, 23)):
        M, N, K = tiles_m * 256, tiles_n * 256, 8192
        A, B = torch.ones(M, K, device="cuda").bfloat16(), torch.ones(N, K, device="cuda").bfloat16()
        C = torch.empty(M, N, device="cuda")
        scratch = torch.full((64 << 20,), 0xFF, dtype=torch.uint8, device="cuda")
        assert sb.debug_gemm(A, B, C, M, N, K, False, True, scratch=scratch) == 1
        assert bool((C == K).all())
        assert bool((scratch.view(torch.int32) != -1).any()) == (tiles_m * tiles_n == 128)
