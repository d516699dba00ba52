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


def _bf16(shape, seed, std=1.0):
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda:0").normal_(0.0, std, generator=torch.Generator("cuda:0").manual_seed(seed))


# Weights of 256 MiB and less are read as they come, larger ones as a stream (a pass of a model counts all that it reads): the same bits.
# 131072 x 1024 bf16 are 256 MiB.
@pytest.mark.parametrize("rows,row_tiles,features", [(5, 0, 0), (96, 3, 0), (5, 1, 128), (40, 2, 160), (96, 3, 224), (128, 4, 128), (160, 5, 160)])
def test_weights_that_the_cache_holds_and_larger_ones_give_the_same_bits(rows, row_tiles, features):
    N, K = 131072, 1024
    w = _bf16((N + 128, K), 11, 0.05)
    ap = P.op_pack_rows(_bf16((rows, K), rows))
    if features:
        small, large = (P.op_gemm_bf16_strip(ap, P.op_pack_weight(w[:n]), rows, row_tiles, features) for n in (N, N + 128))
    else:
        small, large = (P.op_gemm_bf16_ws(ap, P.op_pack_weight(w[:n]), rows, 1, False, row_tiles) for n in (N, N + 128))
    assert torch.equal(small[0], large[0, :, :N])
    a, some = _bf16((rows, K), rows).double(), w[:256].double()
    bound = K * 2.0 ** -24 * (a.abs() @ some.abs().T) + 1e-30          # as above
    assert bool(((small[0, :, :256].double() - a @ some.T).abs() <= bound).all())


@pytest.mark.parametrize("rows,row_tiles,features", [(5, 1, 128), (77, 3, 160), (160, 5, 224)])
def test_gated_strips_of_weights_that_the_cache_holds_and_larger_ones_give_the_same_bits(rows, row_tiles, features):
    F, K = 65536, 1024
    gate, up = _bf16((F + 128, K), 12, 0.05), _bf16((F + 128, K), 13, 0.05)
    ap = P.op_pack_rows(_bf16((rows, K), rows))
    small, large = (P.op_gemm_bf16_strip(ap, P.op_pack_weight(torch.cat([gate[:f], up[:f]])), rows, row_tiles, features, gated=True) for f in (F, F + 128))
    tiles = (rows + 31) // 32                              # packed order [row tile][feature / 16][64][8]
    small, large = small.view(tiles, F // 16, 64, 8), large.view(tiles, F // 16 + 8, 64, 8)
    assert torch.equal(small, large[:, :F // 16])


@pytest.mark.parametrize("hq,k", [(4, 1), (16, 1), (16, 2), (16, 3), (16, 5)])      # per kv head 2, 8 to 48 stacked rows: one to four row tiles
def test_attention_over_keys_from_the_cache_and_as_a_stream_has_the_same_bits(hq, k):
    hd, hkv, n, lens = 128, 1 if hq == 16 else 2, 1 + k, (37, 1500)
    out = []
    for vocab in (1024, 140032):                           # an LM head of 140032 x 1024: more than the cache holds
        d, cap = 1024, 1600
        z = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda:0")
        weights = {"embed": z(vocab, d), "lm_head": z(vocab, d), "final_norm": z(d), "layers": [
            {"ln1": z(d), "wqkv": z((hq + 2 * hkv) * hd, d), "wo": z(d, hq * hd), "ln2": z(d), "w_gate_up": z(256, d), "w_down": z(d, 128)}]}
        model = dict(n_layers=1, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=128, vocab=vocab, n_experts=0, top_k=0, d_expert=0,
                     dtype="bf16", rope_theta=1.0e4, rms_eps=1.0e-6)
        ver = P.Verifier(model, weights, packed=True, max_batch=2, max_k=k, max_chains=1, max_seqs=2, page_size=64, num_pages=60, max_pages_per_seq=26,
                         verify_mode=P.SV_MATCH, sample_mode=P.SV_EXP_RACE, temperature=1.0, device="cuda:0")
        for b, L in enumerate(lens):
            kv = _bf16((2, L + n, hkv, hd), 20 + b)
            ver.seq_add(b, L + n)
            ver.kv_write(b, 0, 0, kv[0], kv[1])
            ver.seq_set_len(b, L)
        out.append(ver.op_attention([0, 1], n, k, 0, _bf16((2 * n, hq, hd), 30)).clone())
        ver.close()
    assert torch.equal(out[0], out[1]) and float(out[0].float().std()) > 0.01


def test_experts_that_the_cache_holds_and_more_give_the_same_bits():
    E, d, F, top_k = 64, 2048, 1024, 4                     # 12 MiB an expert: five rows may choose 20 of them, six 24
    a = _bf16((6, d), 41)
    args = (_bf16((E, d), 42, 0.05), _bf16((E, 2 * F, d), 43, 0.02), _bf16((E, d, F), 44, 0.02), top_k)
    few, more = P.op_moe_ffn(a[:5].contiguous(), *args), P.op_moe_ffn(a, *args)
    assert torch.equal(few[1], more[1][:5]) and torch.equal(few[0], more[0][:5])


def test_an_expert_of_more_rows_than_a_group_gives_the_bits_of_its_tiles_alone():
    """All 96 rows choose expert 3: its weights are read twice and ordinarily, the others', which one group covers, as a stream; 32 rows at a
    time every strip is read once."""
    E, d, F, top_k, rows = 64, 2048, 1024, 2, 96
    a = _bf16((rows, d), 51)
    a[:, 0] = 8.0
    router = _bf16((E, d), 52, 0.02)
    router[:, 0] = 0.0
    router[3, 0] = 4.0
    args = (router, _bf16((E, 2 * F, d), 53, 0.02), _bf16((E, d, F), 54, 0.02), top_k)
    out, ids, _ = P.op_moe_ffn(a, *args)
    assert bool((ids[:, 0] == 3).all()) and len(ids[:, 1].unique()) > 20
    for r0 in range(0, rows, 32):
        part, part_ids, _ = P.op_moe_ffn(a[r0:r0 + 32].contiguous(), *args)
        assert torch.equal(part_ids, ids[r0:r0 + 32]) and torch.equal(part, out[r0:r0 + 32])
