"""The tall projection kernel: every combination of tall and short row tiles in both of its forms, strips beyond the output's
width, reductions shorter than its ring, short tiles behind and beside the tall ones -- against float64 products and, bit for
bit, the weight-streaming kernel -- and in the launch plan's own tiles inside a step."""
import numpy as np
import pytest
import torch

from oracle import model as M
from harness import LOGIT_TOL

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def bf16(shape, std, seed):
    return (torch.randn(shape, generator=torch.Generator().manual_seed(seed)) * std).to(torch.bfloat16)


@pytest.mark.parametrize("rows", [1, 64, 193, 257, 385, 512, 961])
@pytest.mark.parametrize("K,splits", [(64, 1), (192, 3), (1024, 2)])
def test_whole_and_short_row_tiles_match_float64_product(rows, K, splits):
    """Tolerance as in the other projection tests: fp32 sums of K <= 1024 products of magnitude 0.02."""
    from paper_2511_16193_amd import op_gemm_bf16_ws, op_pack_rows, op_pack_weight
    a, w = bf16((rows, K), 1.0, rows), bf16((512, K), 0.02, K)
    want = M.matmul_wt(a.float().numpy().astype(np.float64), w.float().numpy())
    got = op_gemm_bf16_ws(op_pack_rows(a.to(DEV)), op_pack_weight(w.to(DEV)), rows, splits=splits, wide=True, row_tiles=8)
    torch.cuda.synchronize()
    assert np.max(np.abs(got.cpu().numpy().astype(np.float64).sum(axis=0) - want)) < 1e-4


@pytest.mark.parametrize("rows", [129, 161, 225, 321, 385, 450, 650, 865, 897, 1025, 1601, 1665])
def test_step_equals_the_weight_streaming_kernel(rows):
    """One decoding step of `rows` requests in the launch plan's own tiles (an LM head of 297 strips, the narrow projections,
    from 161 rows on the gated gate/up form), against the same step without the tall kernel.  One layer: two correct
    implementations (the splits of a reduction differ) stay within the tolerance of the step tests."""
    import paper_2511_16193_amd as P
    d, ff, V = 256, 18944, 38016
    lw = {"ln1": bf16((d,), 0.05, 1) + 1, "wqkv": bf16((512, d), 0.02, 2), "wo": bf16((d, 256), 0.02, 3),
          "ln2": bf16((d,), 0.05, 4) + 1, "w_gate_up": bf16((2 * ff, d), 0.02, 5), "w_down": bf16((d, ff), 0.02, 6)}
    lw = {n: P.op_pack_weight(t.to(DEV)) if t.dim() == 2 else t.to(DEV) for n, t in lw.items()}
    w = {"embed": bf16((V, d), 0.5, 7).to(DEV), "lm_head": P.op_pack_weight(bf16((V, d), 0.02, 8).to(DEV)),
         "final_norm": (bf16((d,), 0.05, 9) + 1).to(DEV), "layers": [lw]}
    model = dict(n_layers=1, d_model=d, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ff=ff, vocab=V, n_experts=0, top_k=0,
                 d_expert=0, dtype="bf16", rope_theta=1.0e4, rms_eps=1.0e-6)
    ver = P.Verifier(model, w, packed=True, max_batch=rows, max_k=1, max_chains=1, max_seqs=rows, page_size=32, num_pages=rows + 4,
                     max_pages_per_seq=2, verify_mode=P.SV_MATCH, sample_mode=P.SV_EXP_RACE, temperature=1.0, device=DEV)
    ids = list(range(rows))
    kv = bf16((2, 7, 1, 128), 1.0, 10).to(DEV)
    for b in ids:
        ver.seq_add(b, 7)
        ver.kv_write(b, 0, 0, kv[0], kv[1])
    x0 = torch.arange(rows, dtype=torch.int32, device=DEV) * 19 % V
    u = torch.rand((rows, 1, 1), generator=torch.Generator().manual_seed(11)).to(DEV)
    logits = []
    for mode in (0, -1):
        ver.set_option(P.SV_OPT_GEMM_TILE, mode)
        ver.seq_set_lens(ids, [7] * rows)
        out = {"accepted_len": torch.zeros(rows, dtype=torch.int32, device=DEV), "out_tokens": torch.zeros((rows, 1), dtype=torch.int32, device=DEV),
               "best_chain": torch.zeros(rows, dtype=torch.int32, device=DEV), "logits": torch.full((rows, 1, V), float("nan"), device=DEV)}
        ver.step(ids, x0, None, None, u, out=out)
        torch.cuda.synchronize()
        logits.append(out["logits"])
    assert float((logits[0] - logits[1]).abs().max()) < LOGIT_TOL["bf16"]
    assert float(logits[0].std()) > 0.1
    ver.close()


PAIRS = [(h, ht) for h in (3, 4, 5) for ht in range(h)]


def tiles_of(h, ht, n):
    """n tall tiles and, if there is a height for them, two short ones; the rows they cover but for 37 of the last."""
    nt = 2 if ht else 0
    return (h, n, ht, nt), 64 * (h * n + ht * nt) - 37


@pytest.mark.parametrize("N,K,splits", [
    (384, 64, 1),                     # two fills for a ring of three; the last strip half beyond the output
    (384, 64, 2),                     # one fill a split
    (384, 576, 3),                    # six fills a split
    (65664, 64, 1),                   # 257 strips: two tall tiles a strip fill two rounds, the short ones stand beside them
])
@pytest.mark.parametrize("h,ht", PAIRS)
def test_every_pair_of_heights_equals_the_weight_streaming_kernel(h, ht, N, K, splits):
    """Both kernels add the slices of a split in the same order: equal bits.  float64 tolerance as above."""
    from paper_2511_16193_amd import op_gemm_bf16_tall, op_gemm_bf16_ws, op_pack_rows, op_pack_weight
    tall, rows = tiles_of(h, ht, 2 if N > 1000 else 1)
    a, w = bf16((rows, K), 1.0, rows).to(DEV), bf16((N, K), 0.02, K).to(DEV)
    ap, wp = op_pack_rows(a), op_pack_weight(w)
    got = op_gemm_bf16_tall(ap, wp, rows, tall, splits)
    if K % (64 * splits) == 0:
        assert torch.equal(got, op_gemm_bf16_ws(ap, wp, rows, splits=splits, wide=False))
    if N < 1000:
        want = M.matmul_wt(a.cpu().float().numpy().astype(np.float64), w.cpu().float().numpy())
        assert np.max(np.abs(got.cpu().numpy().astype(np.float64).sum(axis=0) - want)) < 1e-4


@pytest.mark.parametrize("K,splits", [(576, 2), (192, 2)])
@pytest.mark.parametrize("h,ht", PAIRS)
def test_odd_numbers_of_fills(h, ht, K, splits):
    """9 and 3 fills a split, which the weight-streaming kernel has no form for: every split against its float64 product."""
    from paper_2511_16193_amd import op_gemm_bf16_tall, op_pack_rows, op_pack_weight
    tall, rows = tiles_of(h, ht, 1)
    a, w = bf16((rows, K), 1.0, rows).to(DEV), bf16((384, K), 0.02, K).to(DEV)
    got = op_gemm_bf16_tall(op_pack_rows(a), op_pack_weight(w), rows, tall, splits)
    for s in range(splits):
        part = slice(s * K // splits, (s + 1) * K // splits)
        want = M.matmul_wt(a[:, part].cpu().float().numpy().astype(np.float64), w[:, part].cpu().float().numpy())
        assert np.max(np.abs(got[s].cpu().numpy().astype(np.float64) - want)) < 1e-4, s


@pytest.mark.parametrize("F,K", [(384, 64), (384, 640), (33024, 64)])
@pytest.mark.parametrize("h,ht", PAIRS)
def test_every_gated_pair_of_heights_equals_the_weight_streaming_kernel(h, ht, F, K):
    from paper_2511_16193_amd import op_gemm_bf16_tall, op_pack_rows, op_pack_weight
    tall, rows = tiles_of(h, ht, 2 if F > 1000 else 1)
    a, w = bf16((rows, K), 1.0, rows).to(DEV), bf16((2 * F, K), 0.02, K).to(DEV)
    ap, wp = op_pack_rows(a), op_pack_weight(w)
    got = op_gemm_bf16_tall(ap, wp, rows, tall, gated=True)
    assert torch.equal(got, op_gemm_bf16_tall(ap, wp, rows, None, gated=True))
    if F < 1000:
        x = a.cpu().double() @ w.cpu().double().T
        gate, up = torch.nn.functional.silu(x[:, :F]), x[:, F:]
        pack = lambda t: op_pack_rows(t.to(torch.bfloat16).to(DEV)).float()
        want, slack = pack(gate * up), pack(gate.abs() + 1.1 * up.abs())
        # sums within 1e-4 as above (silu's slope is 1.1 at most), then one bf16 spacing where a boundary lies between
        assert bool(((got.float() - want).abs() <= 2.0 ** -7 * want.abs() + 1e-4 * slack).all())
        assert float((got.float() != want).float().mean()) < 0.01


@pytest.mark.parametrize("which", ["weights", "rows"])
def test_operands_off_16_bytes_take_the_weight_streaming_kernel(which):
    """The same sums through every entry point that can ask for tall tiles; a split of an odd number of fills, which the other kernel has
    no form for, is refused."""
    from paper_2511_16193_amd import SvError, op_gemm_bf16_tall, op_gemm_bf16_ws, op_pack_rows, op_pack_weight
    M_, N, K = 260, 512, 192
    ap, wp = op_pack_rows(bf16((M_, K), 1.0, 1).to(DEV)), op_pack_weight(bf16((N, K), 0.02, 2).to(DEV))
    off = lambda t: torch.cat([t.new_zeros(4), t.flatten()])[4:].view(t.shape)
    a, w = (off(ap), wp) if which == "rows" else (ap, off(wp))
    assert a.data_ptr() % 16 or w.data_ptr() % 16
    assert torch.equal(op_gemm_bf16_tall(a, w, M_, (4, 1, 1, 1), 3), op_gemm_bf16_tall(ap, wp, M_, (4, 1, 1, 1), 3))
    assert torch.equal(op_gemm_bf16_ws(a, w, M_, splits=3, wide=True, row_tiles=8), op_gemm_bf16_ws(ap, wp, M_, splits=3, wide=True, row_tiles=8))
    rows = lambda t: t.view(-1, N // 32, 2, 32, 8).permute(0, 3, 1, 2, 4).reshape(-1, N // 2)[:M_]
    assert torch.equal(rows(op_gemm_bf16_tall(a, w, M_, (4, 1, 1, 1), gated=True)), rows(op_gemm_bf16_tall(ap, wp, M_, (4, 1, 1, 1), gated=True)))
    with pytest.raises(SvError):
        op_gemm_bf16_tall(a, w, M_, (4, 1, 1, 1), 2)


@pytest.mark.parametrize("tall", [(2, 2, 0, 0), (6, 1, 0, 0), (4, 1, 4, 1), (4, 1, 2, 0), (4, 1, 0, 1), (4, 0, 2, 2), (4, 1, 0, 0), (4, 3, 0, 0), (3, 1, 1, 3)])
def test_tiles_that_do_not_fit_the_rows_are_refused(tall):
    """260 rows: heights that do not exist, short tiles without a height, rows left uncovered, tiles of padding alone."""
    from paper_2511_16193_amd import SvError, op_gemm_bf16_tall
    a, w = torch.zeros((288, 64), dtype=torch.bfloat16, device=DEV), torch.zeros((256, 64), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(SvError):
        op_gemm_bf16_tall(a, w, 260, tall)
