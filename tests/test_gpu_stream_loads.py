"""The weight-streaming kernel reads its weights as a stream where one row tile holds all rows, and as ordinary loads where several share
them; it leaves its results as a stream from some size on.  The same sums in the same order, so the same bits."""
import pytest
import torch

import paper_2511_16193_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("row_tiles", [2, 3, 4, 5])
@pytest.mark.parametrize("N,K,splits,wide", [(128, 256, 1, False), (768, 1024, 4, False), (768, 512, 2, True)])
def test_one_row_tile_and_several_give_the_same_bits(row_tiles, N, K, splits, wide):
    M = 32 * row_tiles - 5                                 # the last tile is not full
    g = torch.Generator().manual_seed(M + N)
    a = torch.randn((M, K), generator=g).to(torch.bfloat16).cuda()
    w = (torch.randn((N, K), generator=g) * 0.05).to(torch.bfloat16).cuda()
    ap, wp = P.op_pack_rows(a), P.op_pack_weight(w)
    one = P.op_gemm_bf16_ws(ap, wp, M, splits, wide, row_tiles)
    several = P.op_gemm_bf16_ws(ap, wp, M, splits, wide, 1)
    assert torch.equal(one, several)
    want = a.double() @ w.double().T
    # fp32 sums of K products of bf16 values: K roundings of 2^-24 of the sum of magnitudes bound the error
    bound = K * 2.0 ** -24 * (a.double().abs() @ w.double().abs().T) + 1e-30
    assert bool(((one.double().sum(0) - want).abs() <= bound).all())


@pytest.mark.parametrize("N,K,splits,wide,rows", [(768, 1024, 4, False, 128), (1024, 768, 1, True, 128), (1024, 1024, 2, False, 96)])
def test_results_left_ordinarily_and_as_a_stream_have_the_same_bits(N, K, splits, wide, rows):
    g = torch.Generator().manual_seed(N)
    a = torch.randn((rows, K), generator=g).to(torch.bfloat16).cuda()
    wp = P.op_pack_weight((torch.randn((N, K), generator=g) * 0.05).to(torch.bfloat16).cuda())
    # rows x the narrower side below 96 K, and at it
    few, all_rows = (P.op_gemm_bf16_ws(P.op_pack_rows(a[:m].contiguous()), wp, m, splits, wide, 5) for m in (rows - 1, rows))
    assert torch.equal(few, all_rows[:, :rows - 1])
