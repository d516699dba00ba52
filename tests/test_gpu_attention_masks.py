"""What a row of the attention must not see: NaN and infinity in masked cache entries."""
import pytest
import torch

import paper_2511_16193_amd as P

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def verifier(dtype, hd, hq, hkv, layers, *, page, pages, k, chains, ff=128, d=None, vocab=1024, weights=None, **kw):
    d = d or hq * hd
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    model = dict(n_layers=layers, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=ff, vocab=vocab, n_experts=0, top_k=0,
                 d_expert=0, dtype=dtype, rope_theta=1.0e4, rms_eps=1.0e-12)
    if weights is None:
        z = lambda *s: torch.zeros(s, dtype=dt, device=DEV)
        weights = {"embed": z(vocab, d), "lm_head": z(vocab, d), "final_norm": z(d), "layers": [
            {"ln1": z(d), "wqkv": z((hq + 2 * hkv) * hd, d), "wo": z(d, hq * hd), "ln2": z(d), "w_gate_up": z(2 * ff, d), "w_down": z(d, ff)}] * layers}
    return P.Verifier(model, weights, packed=dtype == "bf16", max_batch=2, max_k=k, max_chains=chains, max_seqs=2, page_size=page,
                      num_pages=2 * pages, max_pages_per_seq=pages, verify_mode=P.SV_MATCH, sample_mode=P.SV_EXP_RACE, temperature=1.0,
                      device=DEV, **kw)


@pytest.mark.parametrize("dtype,hd,hq,hkv,page,chains,k", [
    ("fp32", 64, 4, 2, 64, 2, 3),
    ("fp32", 128, 4, 4, 32, 3, 4),
    ("bf16", 64, 8, 2, 64, 2, 5),         # head_dim 64: the generic kernel
    ("bf16", 128, 4, 2, 96, 2, 5),        # a page size that is no power of two: the generic kernel
    ("bf16", 128, 8, 1, 64, 4, 10),       # 41 rows of 8 heads, 328 stacked rows: the generic kernel
])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_masked_entries_do_not_reach_a_row(dtype, hd, hq, hkv, page, chains, k, bad):
    """The second chain's entries, the last draft's of the first and whatever an earlier owner left behind the rows are NaN or
    infinite: the rows that do not see them come out bit for bit as with finite entries there."""
    n, lens, cap = 1 + chains * k, (37, 300), 448
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    ver = verifier(dtype, hd, hq, hkv, 1, page=page, pages=-(-cap // page), k=k, chains=chains)
    g = torch.Generator().manual_seed(3)
    kv = [torch.randn((2, cap, hkv, hd), generator=g).to(dt).to(DEV) for _ in lens]
    q = torch.randn((2 * n, hq, hd), generator=g).to(dt).to(DEV)
    got = []
    for value in (0.5, bad):
        for b, L in enumerate(lens):
            ver.seq_add(b, cap - 8)
            x = kv[b].clone()
            x[:, L + k] = value                             # chain 0's last draft
            x[:, L + 1 + k: L + 1 + 2 * k] = value          # chain 1
            x[:, L + n:] = value                            # left by an earlier owner
            ver.kv_write(b, 0, 0, x[0, : cap - 8].contiguous(), x[1, : cap - 8].contiguous())
            ver.seq_set_len(b, L)
        got.append(ver.op_attention([0, 1], n, k, 0, q).view(2, n, -1).float().cpu())
        for b in (0, 1):
            ver.seq_remove(b)
    clean = [j for j in range(n) if j != k and not k < j <= 2 * k]
    assert torch.equal(got[0][:, clean], got[1][:, clean])
    assert bool(torch.isfinite(got[1][:, clean]).all()) and float(got[1][:, clean].std()) > 0.01
    seen = got[1][:, [k] + list(range(k + 1, 2 * k + 1))]
    assert not bool(torch.isfinite(seen).any())             # a row that sees such an entry shows it
    ver.close()


@pytest.mark.parametrize("dtype,hd,hq,hkv,page,lens", [
    ("fp32", 64, 4, 2, 64, (127, 253)),   # the rows' own keys run across the end of a tile and of a chunk of 256 keys
    ("fp32", 128, 4, 4, 32, (253, 510)),
    ("bf16", 64, 8, 2, 64, (253, 510)),
    ("bf16", 128, 4, 2, 96, (28, 766)),   # inside the first tile; around three chunks
])
def test_generic_attention_around_the_ends_of_tiles_and_chunks(dtype, hd, hq, hkv, page, lens):
    k, n, cap = 5, 6, 800
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    ver = verifier(dtype, hd, hq, hkv, 1, page=page, pages=-(-cap // page), k=k, chains=1)
    g = torch.Generator().manual_seed(5)
    kv = [torch.randn((2, cap, hkv, hd), generator=g).to(dt) for _ in lens]
    q = torch.randn((2 * n, hq, hd), generator=g).to(dt)
    for b, L in enumerate(lens):
        ver.seq_add(b, L + n)
        ver.kv_write(b, 0, 0, kv[b][0, : L + n].contiguous().to(DEV), kv[b][1, : L + n].contiguous().to(DEV))
        ver.seq_set_len(b, L)
    got = ver.op_attention([0, 1], n, k, 0, q.to(DEV)).view(2, n, hq, hd).double().cpu()
    for b, L in enumerate(lens):
        for j in range(n):
            x = kv[b][:, : L + j + 1].double().repeat_interleave(hq // hkv, dim=2)
            p = torch.softmax(torch.einsum("hd,khd->hk", q.view(2, n, hq, hd)[b, j].double(), x[0]) / hd ** 0.5, dim=-1)
            want = torch.einsum("hk,khd->hd", p, x[1])
            # the output's own rounding (bf16 keeps 8 significant bits: half a unit of the last is 2^-8 of the value at most) and fp32 sums
            # of some 800 keys, scores of magnitude ten among them
            bound = (2.0 ** -8 * want.abs() if dtype == "bf16" else 0.0) + 2e-5 * torch.einsum("hk,khd->hd", p, x[1].abs())
            assert bool(((got[b, j] - want).abs() <= bound).all()), (b, j)
    ver.close()
