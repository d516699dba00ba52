"""The narrow-strip projection kernel: every height and width in both of its forms, rows and strips that end inside a tile, reductions
shorter than its ring and of odd numbers of fills, more strips than CUs -- bit for bit the weight-streaming kernel's sums, and
against float64 products."""
import numpy as np
import pytest
import torch

from harness import LOGIT_TOL
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


@pytest.mark.parametrize("K,splits", [(576, 2), (448, 2), (192, 2)])
@pytest.mark.parametrize("features", [128, 160, 224])
@pytest.mark.parametrize("tiles", [1, 2, 3, 4, 5, 6, 8, 10])
def test_odd_numbers_of_fills(tiles, features, K, splits):
    """9, 7 and 3 fills a split: the loop over pairs of fills, then the one left over, with the ring wrapped round and not.  The
    weight-streaming kernel has no such splits: against float64 (tolerance as above), and the sums of tall tiles, bit for bit."""
    from paper_2511_16193_amd import op_gemm_bf16_strip, op_gemm_bf16_tall, op_pack_rows, op_pack_weight
    rows, N = 32 * tiles - 5, 384
    a, w = bf16((rows, K), 1.0, tiles).to(DEV), bf16((N, K), 0.02, K).to(DEV)
    ap, wp = op_pack_rows(a), op_pack_weight(w)
    got = op_gemm_bf16_strip(ap, wp, rows, tiles, features, splits)
    need = (rows + 63) // 64
    assert torch.equal(got, op_gemm_bf16_tall(ap, wp, rows, (max(3, need), 1, 0, 0), splits))
    halves = [slice(s * K // splits, (s + 1) * K // splits) for s in range(splits)]
    for s, h in enumerate(halves):
        want = M.matmul_wt(a[:, h].cpu().float().numpy().astype(np.float64), w[:, h].cpu().float().numpy())
        assert np.max(np.abs(got[s].cpu().numpy().astype(np.float64) - want)) < 1e-4, s


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


@pytest.mark.parametrize("rows", [5, 100, 200, 400])
def test_weights_that_start_off_16_bytes_keep_the_weight_streaming_kernel(rows):
    """One decoding step with packed projections 8 bytes past a 16-byte boundary: the bits of the step that is told to take that kernel
    everywhere, and within the step tests' tolerance of the step with the same weights on the boundary (which takes the launches for a few rows at 5, else strips, and tall tiles
    from 200 rows on)."""
    import paper_2511_16193_amd as P
    d, ff, V = 256, 2048, 4096
    lw = {"ln1": bf16((d,), 0.05, 1) + 1, "wqkv": bf16((512, d), 0.02, 2), "wo": bf16((d, 256), 0.02, 3),
          "ln2": bf16((d,), 0.05, 4) + 1, "w_gate_up": bf16((2 * ff, d), 0.02, 5), "w_down": bf16((d, ff), 0.02, 6)}
    lw = {n: P.op_pack_weight(t.to(DEV)) if t.dim() == 2 else t.to(DEV) for n, t in lw.items()}
    head = P.op_pack_weight(bf16((V, d), 0.02, 8).to(DEV))
    embed, norm = bf16((V, d), 0.5, 7).to(DEV), (bf16((d,), 0.05, 9) + 1).to(DEV)

    def off(t):
        return torch.cat([t.new_zeros(4), t.flatten()])[4:].view(t.shape)

    def step(shift, mode):
        place = off if shift else lambda t: t
        w = {"embed": embed, "lm_head": place(head), "final_norm": norm,
             "layers": [{n: place(t) if t.dim() > 1 else t for n, t in lw.items()}]}
        assert (w["lm_head"].data_ptr() % 16 != 0) == shift and (w["layers"][0]["wo"].data_ptr() % 16 != 0) == shift
        model = dict(n_layers=1, d_model=d, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ff=ff, vocab=V, n_experts=0, top_k=0,
                     d_expert=0, dtype="bf16", rope_theta=1.0e4, rms_eps=1.0e-6)
        ver = P.Verifier(model, w, packed=True, max_batch=rows, max_k=1, max_chains=1, max_seqs=rows, page_size=32, num_pages=rows + 4,
                         max_pages_per_seq=2, verify_mode=P.SV_MATCH, sample_mode=P.SV_EXP_RACE, temperature=1.0, device=DEV)
        ver.set_option(P.SV_OPT_GEMM_TILE, mode)
        kv = bf16((2, 7, 1, 128), 1.0, 10).to(DEV)
        for b in range(rows):
            ver.seq_add(b, 7)
            ver.kv_write(b, 0, 0, kv[0], kv[1])
        u = torch.rand((rows, 1, 1), generator=torch.Generator().manual_seed(11)).to(DEV)
        out = {"accepted_len": torch.zeros(rows, dtype=torch.int32, device=DEV), "out_tokens": torch.zeros((rows, 1), dtype=torch.int32, device=DEV),
               "best_chain": torch.zeros(rows, dtype=torch.int32, device=DEV), "logits": torch.full((rows, 1, V), float("nan"), device=DEV)}
        ver.step(list(range(rows)), torch.arange(rows, dtype=torch.int32, device=DEV) * 19 % V, None, None, u, out=out)
        torch.cuda.synchronize()
        ver.close()
        return out["logits"]

    kept = step(True, -1)
    assert torch.equal(kept, step(True, 0))
    assert float((kept - step(False, -1)).abs().max()) < LOGIT_TOL["bf16"]
    assert float(kept.std()) > 0.1
