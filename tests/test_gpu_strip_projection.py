"""The narrow-strip projection kernel: every height and width in both of its forms, rows and strips that end inside a tile, reductions
shorter than its ring and of an odd number of fills, more strips than CUs -- bit for bit the weight-streaming kernel's sums, and
against float64 products."""
import numpy as np
import pytest
import torch

from oracle import model as M

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def bf16(shape, std, seed):
    return (torch.randn(shape, generator=torch.Generator().manual_seed(seed)) * std).to(torch.bfloat16)


def rows_of(tiles):
    return sorted({max(1, 32 * tiles - 37), 32 * tiles - 15, 32 * tiles})


@pytest.mark.parametrize("features", [128, 160, 224])
@pytest.mark.parametrize("tiles", [1, 2, 3, 4, 5, 6, 8, 10])
def test_plain_strips(tiles, features):
    """Tolerance as in the other projection tests: fp32 sums of K <= 576 products of magnitude 0.02."""
    from paper_2511_16193_amd import op_gemm_bf16_strip, op_gemm_bf16_ws, op_pack_rows, op_pack_weight
    for N, K, splits in [(384, 64, 1), (384, 64, 2), (384, 576, 3), (384, 448, 1), (41088, 64, 1)]:
        w = bf16((N, K), 0.02, K).to(DEV)
        wp = op_pack_weight(w)
        for rows in rows_of(tiles) if N < 1000 else [32 * tiles]:
            a = bf16((rows, K), 1.0, rows).to(DEV)
            ap = op_pack_rows(a)
            got = op_gemm_bf16_strip(ap, wp, rows, tiles, features, splits)
            if K % (64 * splits) == 0:
                assert torch.equal(got, op_gemm_bf16_ws(ap, wp, rows, splits=splits, wide=False)), (N, K, splits, rows)
            if N < 1000:
                want = M.matmul_wt(a.cpu().float().numpy().astype(np.float64), w.cpu().float().numpy())
                assert np.max(np.abs(got.cpu().numpy().astype(np.float64).sum(axis=0) - want)) < 1e-4, (N, K, splits, rows)


@pytest.mark.parametrize("features", [128, 160, 224])
@pytest.mark.parametrize("tiles", [1, 2, 3, 4, 5, 6, 8, 10])
def test_gated_strips(tiles, features):
    """std 1: gates of ordinary size; std 200: from about -150 to 150, where the exponential leaves the range of floats."""
    from paper_2511_16193_amd import op_gemm_bf16_strip, op_gemm_bf16_tall, op_pack_rows, op_pack_weight
    for F, K, std in [(384, 64, 1.0), (384, 320, 200.0), (20608, 64, 1.0)]:
        w = bf16((2 * F, K), 0.02, K).to(DEV)
        wp = op_pack_weight(w)
        for rows in rows_of(tiles) if F < 1000 else [32 * tiles]:
            a = bf16((rows, K), std, rows).to(DEV)
            ap = op_pack_rows(a)
            got = op_gemm_bf16_strip(ap, wp, rows, tiles, features, gated=True)
            real = lambda t: t[:rows].float()
            unpack = lambda t: t.view(-1, F // 16, 2, 32, 8).permute(0, 3, 1, 2, 4).reshape(-1, F)
            ref = op_gemm_bf16_tall(ap, wp, rows, None, gated=True)
            assert torch.equal(real(unpack(got)), real(unpack(ref))), (F, K, rows)
            if F < 1000:
                x = a.cpu().double() @ w.cpu().double().T
                gate, up = torch.nn.functional.silu(x[:, :F]), x[:, F:]
                want, slack = (gate * up).float(), (gate.abs() + 1.1 * up.abs()).float()
                err = (real(unpack(got)).cpu() - want).abs()
                # sums within 1e-4 std (silu's slope is 1.1 at most), then a bf16 rounding
                assert bool((err <= 2.0 ** -8 * want.abs() * 1.01 + 1e-4 * std * slack + 1e-8 * std * std).all()), (F, K, rows)


@pytest.mark.parametrize("tiles,features,splits", [(0, 128, 1), (7, 128, 1), (9, 128, 1), (11, 128, 1), (2, 128, 1), (3, 96, 1), (3, 192, 1), (3, 256, 1), (3, 128, 4)])
def test_strips_that_do_not_exist_are_refused(tiles, features, splits):
    """70 rows, 64 inputs: heights and widths that there are not, rows left uncovered, splits finer than a fill."""
    from paper_2511_16193_amd import SvError, op_gemm_bf16_strip
    a, w = torch.zeros((96, 64), dtype=torch.bfloat16, device=DEV), torch.zeros((256, 64), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(SvError):
        op_gemm_bf16_strip(a, w, 70, tiles, features, splits)
