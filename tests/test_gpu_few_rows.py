"""A dense decoder layer over up to sixteen rows: norm, rotary, append and residual inside the projections."""
import numpy as np
import pytest
import torch

import paper_2511_16193_amd as P
from harness import Case, LOGIT_TOL
from oracle import verify as OV
import workloads as W

pytestmark = pytest.mark.gpu
DEV, THETA, EPS = "cuda:0", 1.0e4, 1.0e-6


def _t(shape, seed, std=1.0, dtype=torch.bfloat16):
    return (torch.randn(shape, generator=torch.Generator().manual_seed(seed)) * std).to(dtype)


def _round(x):
    return x.to(torch.bfloat16).double()


def _norm(x, gain):
    return _round(x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * gain.double())


def _rotate(x, pos):                                       # [rows, heads, hd], halves paired
    half = x.shape[-1] // 2
    angle = pos.double()[:, None] * THETA ** (-torch.arange(half, dtype=torch.float64) / half)
    c, s = torch.cos(angle)[:, None], torch.sin(angle)[:, None]
    return torch.cat([x[..., :half] * c - x[..., half:] * s, x[..., half:] * c + x[..., :half] * s], -1)


@pytest.mark.parametrize("rows,d,hq,hkv,hd,ff", [
    (1, 256, 2, 1, 128, 128),            # one step of the reduction a wave; fewer feature operands than a work-group holds
    (7, 384, 4, 2, 64, 1216),            # twelve steps over eight waves; head_dim 64; 76 gate operands, the last work-group whole
    (8, 1024, 8, 2, 128, 17152),         # most rows that are normalised on the way in; 1072 gate operands, 5 a work-group, 2 in the last
    (5, 1024, 8, 8, 128, 20736),         # 1296 gate operands: 7 a work-group, 1 in the last
    (3, 6144, 8, 1, 128, 192),           # the widest rows that are; 32 features of O and down a work-group
    (4, 6272, 8, 1, 128, 192),           # wider: a norm of its own
    (9, 1024, 8, 2, 128, 1024),          # more rows: QKV and O only
    (16, 512, 4, 4, 128, 8320),          # down over 8320 inputs
])
def test_layer_against_float64(rows, d, hq, hkv, hd, ff):
    """One row a request behind zero to five cached keys, rounded to bf16 where the path rounds.  A value that the two sums put on different sides of a
    rounding boundary moves by at most one unit, 2^-8 of it, and so does everything behind it: 2^-8 of what the layer adds to the residual,
    by the 2-norm, and one unit of a cache entry plus 2^-8 of the entries' size."""
    g = lambda *shape, seed, std=None: _t(shape, seed, std or shape[-1] ** -0.5)
    w = {"ln1": 1 + _t((d,), 1, 0.1), "wqkv": g((hq + 2 * hkv) * hd, d, seed=2), "wo": g(d, hq * hd, seed=3), "ln2": 1 + _t((d,), 4, 0.1),
         "w_gate_up": g(2 * ff, d, seed=5, std=2 * d ** -0.5), "w_down": g(d, ff, seed=6)}
    on = {n: x.to(DEV) if x.dim() == 1 else P.op_pack_weight(x.to(DEV)) for n, x in w.items()}
    vocab = 128
    model = dict(n_layers=1, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=ff, vocab=vocab, n_experts=0, top_k=0, d_expert=0, dtype="bf16",
                 rope_theta=THETA, rms_eps=EPS)
    z = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device=DEV)
    ver = P.Verifier(model, {"embed": z(vocab, d), "lm_head": z(vocab, d), "final_norm": z(d), "layers": [on]}, packed=True, max_batch=rows, max_k=1,
                     max_chains=1, max_seqs=rows, page_size=64, num_pages=2 * rows, max_pages_per_seq=2, verify_mode=P.SV_MATCH,
                     sample_mode=P.SV_EXP_RACE, temperature=1.0, device=DEV)
    lens = [b % 6 for b in range(rows)]
    old = [_t((2, max(L, 1), hkv, hd), 20 + b) for b, L in enumerate(lens)]
    for b, L in enumerate(lens):
        ver.seq_add(b, L + 1)
        if L:
            ver.kv_write(b, 0, 0, old[b][0].to(DEV), old[b][1].to(DEV))
        ver.seq_set_len(b, L)
    h = _t((rows, d), 9, 1.5, torch.float32)
    got = ver.op_layer(list(range(rows)), 1, 0, 0, h.to(DEV)).double().cpu()
    entries = [tuple(x.double().cpu()[lens[b]] for x in ver.kv_read(b, 0, 0, lens[b] + 1)) for b in range(rows)]
    ver.close()

    h0, pos = h.double(), torch.tensor(lens)
    qkv = (_norm(h0, w["ln1"]) @ w["wqkv"].double().T).view(rows, hq + 2 * hkv, hd)
    q, k, v = _round(_rotate(qkv[:, :hq], pos)), _round(_rotate(qkv[:, hq:hq + hkv], pos)), _round(qkv[:, hq + hkv:])
    for b in range(rows):
        for have, want in zip(entries[b], (k[b], v[b])):
            assert float(((have - want).abs() - 2.0 ** -7 * want.abs()).max()) <= 2.0 ** -8 * float(want.std()), (b, lens[b])
    attn = torch.empty((rows, hq, hd), dtype=torch.float64)
    for b, L in enumerate(lens):
        keys, vals = (torch.cat([old[b][i].double()[:L], (k, v)[i][b][None]]).repeat_interleave(hq // hkv, 1) for i in (0, 1))
        p = torch.softmax((q[b][None] * keys).sum(-1) / hd ** 0.5, 0)
        attn[b] = (p[..., None] * vals).sum(0)
    h1 = h0 + _round(attn.view(rows, hq * hd)) @ w["wo"].double().T
    gate, up = (_norm(h1, w["ln2"]) @ w["w_gate_up"].double().T).chunk(2, -1)
    want = h1 + _round(torch.nn.functional.silu(gate) * up) @ w["w_down"].double().T
    assert float((got - want).norm() / (want - h0).norm()) < 2.0 ** -8


@pytest.mark.parametrize("cached,lens", [([0], [8]), ([70, 3, 0], [7, 5, 3]), ([40], [1])])       # 8, 15 and 1 rows
def test_prefill_of_a_few_rows_is_the_oracles_causal_pass(cached, lens):
    shape = W.Shape("few-bf16", 2, 256, 8, 2, 128, 512, 2048, dtype="bf16", batch=len(lens), k=4, seed=91)
    case = Case(shape, cached, verify_mode=OV.STOCHASTIC, synthetic_kv=True, extra_tokens=24, packed=True)
    prompts = W.make_tokens((len(lens), max(lens)), shape.vocab, shape.seed, "prompt")
    lo = np.stack([OV.prefill(case.spec, case.wn, case.caches[b], prompts[b, :n])[-1] for b, n in enumerate(lens)])
    ld = case.ver.prefill_batch(list(range(len(lens))), torch.from_numpy(prompts).to(torch.int32), lens).cpu().numpy()
    assert np.max(np.abs(lo - ld)) < LOGIT_TOL["bf16"]
    for b, n in enumerate(lens):
        for layer in range(shape.n_layers):
            kd, vd = case.ver.kv_read(b, layer, cached[b], n)
            ko, vo = case.caches[b].k[layer][cached[b]:cached[b] + n], case.caches[b].v[layer][cached[b]:cached[b] + n]
            assert np.max(np.abs(kd.float().cpu().numpy() - ko)) < 0.03 and np.max(np.abs(vd.float().cpu().numpy() - vo)) < 0.03
    case.close()


@pytest.mark.parametrize("rows", [5, 12])
@pytest.mark.parametrize("off", [("wo", "w_down"), ("w_down", "wqkv"), ("w_gate_up", "wo"), ("wqkv", "w_gate_up"), ("w_down", None)])
def test_layers_of_which_one_matrix_starts_off_16_bytes(rows, off):
    """That one keeps the launch with planes, which the next norm adds up whoever runs it, beside neighbours that take the others along: the logits of the
    step whose matrices all start at 16 bytes, but for values that another order of the sums rounds to another bf16 number (2^-8 of
    them), through two layers: 2^-7 by the 2-norm."""
    d, ff, V = 256, 1152, 2048
    g = lambda *shape, seed, std: _t(shape, seed, std)
    layers = [{"ln1": 1 + _t((d,), 9 * l + 1, 0.1), "wqkv": g(512, d, seed=9 * l + 2, std=d ** -0.5), "wo": g(d, 256, seed=9 * l + 3, std=0.1), "ln2": 1 + _t((d,), 9 * l + 4, 0.1),
               "w_gate_up": g(2 * ff, d, seed=9 * l + 5, std=2 * d ** -0.5), "w_down": g(d, ff, seed=9 * l + 6, std=0.05)} for l in range(2)]
    layers = [{n: P.op_pack_weight(x.to(DEV)) if x.dim() == 2 else x.to(DEV) for n, x in w.items()} for w in layers]
    top = {"embed": _t((V, d), 40).to(DEV), "lm_head": P.op_pack_weight(_t((V, d), 41, d ** -0.5).to(DEV)), "final_norm": (1 + _t((d,), 42, 0.1)).to(DEV)}
    model = dict(n_layers=2, d_model=d, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ff=ff, vocab=V, n_experts=0, top_k=0, d_expert=0, dtype="bf16",
                 rope_theta=THETA, rms_eps=EPS)
    kv = _t((2, 7, 1, 128), 43).to(DEV)

    def moved(x):
        y = torch.cat([x.new_zeros(4), x.flatten()])[4:].view(x.shape)
        assert y.data_ptr() % 16 == 8
        return y

    def step(off):
        ws = [{n: moved(x) if n == o else x for n, x in w.items()} for w, o in zip(layers, off)]
        ver = P.Verifier(model, dict(top, layers=ws), packed=True, max_batch=rows, max_k=1, max_chains=1, max_seqs=rows, page_size=32, num_pages=rows + 4,
                         max_pages_per_seq=2, verify_mode=P.SV_MATCH, sample_mode=P.SV_EXP_RACE, temperature=1.0, device=DEV)
        for b in range(rows):
            ver.seq_add(b, 7)
            for l in range(2):
                ver.kv_write(b, l, 0, kv[0], kv[1])
        u = torch.rand((rows, 1, 1), generator=torch.Generator().manual_seed(44)).to(DEV)
        out = ver.step(list(range(rows)), (torch.arange(rows, dtype=torch.int32) * 19).to(DEV), None, None, u, want_logits=True)
        entries = torch.cat([torch.cat(ver.kv_read(b, 1, 7, 1)) for b in range(rows)]).double()
        torch.cuda.synchronize()
        ver.close()
        return out["logits"].double(), entries

    for got, want in zip(step(off), step((None, None))):
        assert float((got - want).norm() / want.norm()) < 2.0 ** -7
