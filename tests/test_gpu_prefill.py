"""Prefill passes at the edges of how they are cut, and a step with more stacked rows than the MFMA attention takes, against the
oracle."""
import numpy as np
import pytest
import torch

from oracle import verify as OV
import workloads as W
from harness import Case, compare_step, LOGIT_TOL

pytestmark = pytest.mark.gpu

SHAPE = W.Shape("prefill-bf16", 2, 256, 8, 2, 128, 512, 2048, dtype="bf16", batch=2, k=4, seed=61)


@pytest.mark.parametrize("cached,lens", [
    ([0, 0], [2300, 1900]),        # 4200 tokens: two passes, the first prompt split between them
    ([0, 0, 0], [64, 16, 16]),     # groups of 64 stacked rows (16 tokens x 4 heads) that end exactly
    ([2500, 1090], [37, 1]),       # few rows over a long cache: keys cut into pieces, merged
    ([1023, 31, 0], [2, 33, 1]),   # rows that start in the last key of a tile, a single-token prompt
])
def test_prefill_is_the_oracles_causal_pass(cached, lens):
    shape = W.scaled_down(SHAPE, batch=len(lens))
    case = Case(shape, cached, verify_mode=OV.STOCHASTIC, synthetic_kv=True, extra_tokens=max(lens) + 8, packed=True)
    prompts = W.make_tokens((len(lens), max(lens)), shape.vocab, shape.seed, "prompt")
    lo = np.stack([OV.prefill(case.spec, case.wn, case.caches[b], prompts[b, :n])[-1] for b, n in enumerate(lens)])
    ld = case.ver.prefill_batch(list(range(len(lens))), torch.from_numpy(prompts).to(torch.int32), lens).cpu().numpy()
    assert np.max(np.abs(lo - ld)) < LOGIT_TOL["bf16"]
    assert np.array_equal(case.device_lengths(), [a + n for a, n in zip(cached, lens)])
    for b, n in enumerate(lens):
        # layer 0 sees equal inputs: the entries differ where rounding does; behind it every entry may, by little
        for layer, frac, atol in ((0, 0.01, 0.02), (shape.n_layers - 1, None, 0.03)):
            kd, vd = case.ver.kv_read(b, layer, cached[b], n)
            ko, vo = case.caches[b].k[layer][cached[b]:cached[b] + n], case.caches[b].v[layer][cached[b]:cached[b] + n]
            kd, vd = kd.float().cpu().numpy(), vd.float().cpu().numpy()
            assert np.max(np.abs(kd - ko)) < atol and np.max(np.abs(vd - vo)) < atol
            assert frac is None or (np.mean(kd != ko) <= frac and np.mean(vd != vo) <= frac)
    case.close()


@pytest.mark.parametrize("dtype,packed,experts,hd,page,cached,lens", [
    ("bf16", True, 0, 128, 64, [0] * 33, [4] * 31 + [3, 1]),      # 33 last rows of 128: two operand tiles, the most that are taken alone
    ("bf16", True, 0, 128, 64, [0] * 33, [4] * 30 + [3, 2, 2]),   # of 127: one row short of that, all rows go on
    ("bf16", True, 0, 128, 64, [5, 70], [63, 1]),                 # one tile of 64 rows, a prompt of one token
    ("bf16", True, 64, 128, 64, [3, 0], [40, 24]),                # experts: the last rows alone are routed
    ("bf16", False, 0, 128, 64, [0, 9], [90, 17]),                # row-major weights
    ("bf16", True, 0, 64, 64, [0, 9], [90, 17]),                  # the generic attention, packed output
    ("bf16", True, 0, 128, 96, [0, 9], [90, 17]),                 # the same by the page size
    ("fp32", False, 0, 64, 64, [0, 9, 0], [90, 17, 17]),          # fp32, norms and rotary as launches of their own behind it
])
def test_last_layer_of_a_prefill_on_the_prompts_last_rows(dtype, packed, experts, hd, page, cached, lens):
    # (experts: weights with which no row's last kept and first dropped expert are closer than 2.6e-3 of their probability in the first
    # layer, 9e-3 for the rows that the last one routes; the two sides' inputs of a layer differ by some 1e-3)
    shape = W.Shape("last-rows", 2, 256, 8, 2, hd, 0 if experts else 512, 2048, dtype=dtype, batch=len(lens), k=4, seed=105 if experts else 83,
                    n_experts=experts, top_k=4 if experts else 0, d_expert=128 if experts else 0)
    case = Case(shape, cached, verify_mode=OV.STOCHASTIC, synthetic_kv=True, extra_tokens=max(lens) + 8, packed=packed, page_size=page)
    prompts = W.make_tokens((len(lens), max(lens)), shape.vocab, shape.seed, "prompt")
    lo = np.stack([OV.prefill(case.spec, case.wn, case.caches[b], prompts[b, :n])[-1] for b, n in enumerate(lens)])
    ld = case.ver.prefill_batch(list(range(len(lens))), torch.from_numpy(prompts).to(torch.int32), lens).cpu().numpy()
    assert np.max(np.abs(lo - ld)) < LOGIT_TOL[dtype]
    assert np.array_equal(case.device_lengths(), [a + n for a, n in zip(cached, lens)])
    for b, n in enumerate(lens):
        kd, vd = case.ver.kv_read(b, shape.n_layers - 1, cached[b], n)
        ko, vo = case.caches[b].k[-1][cached[b]:cached[b] + n], case.caches[b].v[-1][cached[b]:cached[b] + n]
        assert np.max(np.abs(kd.float().cpu().numpy() - ko)) < 0.03 and np.max(np.abs(vd.float().cpu().numpy() - vo)) < 0.03
    case.close()


def test_prefill_behind_rejected_drafts():
    """A step's rejected drafts leave the host's bounds of the lengths above the live ones; the prompts that follow without the
    lengths being read back start at the live ends, and see nothing of what was rejected."""
    shape = W.Shape("behind-bf16", 2, 256, 8, 2, 128, 512, 2048, dtype="bf16", batch=3, k=8, seed=73)
    case = Case(shape, [30, 250, 1200], verify_mode=OV.STOCHASTIC, sample_mode=OV.SAMPLE_EXP_RACE, packed=True, extra_tokens=160)
    x0 = W.make_tokens((3,), shape.vocab, shape.seed, "x0")
    q = W.make_random_q((3, 1, 8), shape.vocab, 1.0, shape.seed)
    r, g = case.step(x0, W.sample_from(q, shape.seed).numpy(), q, W.make_uniforms((3, 1, 9), shape.seed))
    assert np.array_equal(g["accepted_len"], r.accepted_len) and (r.accepted_len < 8).sum() >= 2
    lens = [120, 40, 1]
    prompts = W.make_tokens((3, 120), shape.vocab, shape.seed, "prompt")
    lo = np.stack([OV.prefill(case.spec, case.wn, case.caches[b], prompts[b, :n])[-1] for b, n in enumerate(lens)])
    ld = case.ver.prefill_batch([0, 1, 2], torch.from_numpy(prompts).to(torch.int32), lens).cpu().numpy()
    assert np.max(np.abs(lo - ld)) < LOGIT_TOL["bf16"]
    assert np.array_equal(case.device_lengths(), [c.length for c in case.caches])
    case.close()


def test_step_with_hundreds_of_stacked_rows():
    """16 q heads on one kv head, three chains of eight drafts: 400 stacked rows, the generic attention's."""
    shape = W.Shape("stacked-bf16", 2, 256, 16, 1, 128, 512, 2048, dtype="bf16", batch=3, k=8, n_chains=3, seed=67)
    case = Case(shape, [5, 333, 2100], verify_mode=OV.STOCHASTIC, sample_mode=OV.SAMPLE_EXP_RACE, packed=True)
    x0 = W.make_tokens((3,), shape.vocab, shape.seed, "x0")
    q = W.make_random_q((3, 3, 8), shape.vocab, 1.0, shape.seed)
    drafts = W.sample_from(q, shape.seed).numpy()
    r, g = case.step(x0, drafts, q, W.make_uniforms((3, 3, 9), shape.seed))
    err, exempt, diverged = compare_step(r, g, "bf16", 8)
    assert err < LOGIT_TOL["bf16"] and len(diverged) <= 1
    case.close()


def bf16_of(x):
    """float64 -> the bf16 nearest to it, straight from 64 bits (ties to even)."""
    f = x.to(torch.float64)
    m, e = torch.frexp(f)
    return torch.ldexp(torch.round(m * 256), e - 8)


@pytest.mark.parametrize("cached", [0, 2100])
def test_prefill_sums_unrounded_softmax_weights(cached):
    """A layer whose output is its attention's: identity output projection, no feed-forward, an embedding a thousandth of the
    attention's size.  The next layer's V (identity weights) then shows the normalised rows as they are, so that every output of
    the attention that was rounded to another bf16 value than the exact one is seen.  q = k / 4, so that the cache holds all that
    the exact attention (float64) needs.

    Bound: with fp32 weights an output's error is that of fp32 sums, a few 1e-7 of the largest V in view (4); outputs of a few
    hundred to two thousand keys are 0.1 to 0.03, where bf16 values lie 2^-11 to 2^-13 apart.  So up to 5e-4 of the outputs lie
    close enough to a boundary to cross it.  Weights of two bf16 terms, 2^-17 off each, move 1.3e-3 of them."""
    import paper_2511_16193_amd as P
    dev, n, hq, hd = "cuda:0", 300, 4, 128
    d, V = hq * hd, 1024
    g = torch.Generator().manual_seed(5)
    rnd = lambda *s, std=1.0: (torch.randn(s, generator=g) * std).to(torch.bfloat16)
    wk = rnd(hd, d, std=d ** -0.5)
    wqkv = torch.cat([wk / 4] * hq + [wk, rnd(hd, d, std=d ** -0.5)])
    eye = torch.eye(d, dtype=torch.bfloat16)
    second = torch.zeros(((hq + 2) * hd, d), dtype=torch.bfloat16)
    second[-hd:, :hd] = torch.eye(hd)
    one, zero = torch.ones(d, dtype=torch.bfloat16), torch.zeros
    layers = [{"ln1": one, "wqkv": w, "wo": eye, "ln2": one, "w_gate_up": zero((128, d), dtype=torch.bfloat16), "w_down": zero((d, 64), dtype=torch.bfloat16)}
              for w in (wqkv, second)]
    embed = rnd(V, d, std=2.0 ** -10)
    w = {"embed": embed, "lm_head": rnd(V, d), "final_norm": one, "layers": layers}
    w = P.pack_weights({k: v.to(dev) if k != "layers" else [{a: b.to(dev) for a, b in lw.items()} for lw in v] for k, v in w.items()})
    model = dict(n_layers=2, d_model=d, n_q_heads=hq, n_kv_heads=1, head_dim=hd, d_ff=64, vocab=V, n_experts=0, top_k=0, d_expert=0,
                 dtype="bf16", rope_theta=1.0e4, rms_eps=1.0e-12)
    ver = P.Verifier(model, w, packed=True, max_batch=1, max_k=4, max_chains=1, max_seqs=1, page_size=64, num_pages=48,
                     max_pages_per_seq=46, verify_mode=P.SV_MATCH, sample_mode=P.SV_EXP_RACE, temperature=1.0, device=dev)
    ver.seq_add(0, cached)
    if cached:
        kv = rnd(2, cached, 1, hd).to(dev)
        ver.kv_write(0, 0, 0, kv[0], kv[1])
        ver.kv_write(0, 1, 0, kv[0], kv[1])
    tokens = torch.randint(0, V, (n,), generator=g)
    ver.prefill(0, tokens)
    k, v = (x[:, 0].double().cpu() for x in ver.kv_read(0, 0, 0, cached + n))
    shown = ver.kv_read(0, 1, cached, n)[1][:, 0].double().cpu()
    ver.close()
    s = k[cached:] @ k.T / 4 / hd ** 0.5
    s = s.masked_fill(torch.arange(cached + n)[None] > cached + torch.arange(n)[:, None], float("-inf"))
    o = bf16_of(torch.softmax(s, -1) @ v)
    h = (embed.double()[tokens] + o.repeat(1, hq)).float()
    want = bf16_of((h * (1 / torch.sqrt((h.double() ** 2).mean(-1, keepdim=True) + 1e-12)).float()).double()[:, :hd])
    moved = float((shown != want).double().mean())
    print("moved", moved)
    assert float((shown - want).abs().max()) < 0.02 * float(want.abs().max())
    assert moved < 1e-3


def other_verifier(case, *, prefill_rows, num_pages, pages_per_seq, page_size=64, max_k=0):
    """A second context over the case's weights, its cache holding what the case's oracle caches hold."""
    from paper_2511_16193_amd import Verifier
    B, dt = len(case.lengths), torch.bfloat16 if case.shape.dtype == "bf16" else torch.float32
    ver = Verifier(case.shape.model_fields(), case.wd, max_batch=B, max_k=max_k, max_chains=1, max_seqs=B, page_size=page_size, num_pages=num_pages,
                   max_pages_per_seq=pages_per_seq, verify_mode=case.verify_mode, packed=case.packed,
                   prefill_rows=prefill_rows, device=case.device)
    for b, L in enumerate(case.lengths):
        ver.seq_add(b, int(L))
        for l in range(case.shape.n_layers) if L else ():
            k, v = (torch.from_numpy(x[l][:L]).to(dt).to(case.device).contiguous() for x in (case.caches[b].k, case.caches[b].v))
            ver.kv_write(b, l, 0, k, v)
    return ver


def case_of(dtype, packed, vocab, cached, **kw):
    shape = W.Shape("passes", 2, 256, 8, 2, kw.pop("hd", 128), 512, vocab, dtype=dtype, batch=len(cached), k=0, seed=91)
    case = Case(shape, cached, verify_mode=OV.STOCHASTIC, packed=packed, extra_tokens=kw.pop("extra", 16), **kw)
    case.packed = packed
    return case


@pytest.mark.parametrize("dtype,packed,vocab,B,n,rows", [
    ("bf16", True, 2048, 72, 4, 160),     # passes that end 40 and 32 prompts, taken alone: kept rows cross an operand tile in mid-pass
    ("bf16", True, 2048, 100, 2, 100),    # 50 and 50 of 100 rows: too many to be taken alone
    ("bf16", False, 2048, 72, 4, 160),
    ("fp32", False, 2048, 72, 4, 160),
    ("bf16", True, 128, 24, 4, 64),       # a small vocabulary: no room to keep normalised rows, an LM head for each pass
])
def test_prompts_that_end_in_several_passes(dtype, packed, vocab, B, n, rows):
    case = case_of(dtype, packed, vocab, [0] * B, hd=64 if dtype == "fp32" else 128)
    ver = other_verifier(case, prefill_rows=rows, num_pages=B + 2, pages_per_seq=2)
    prompts = W.make_tokens((B, n), vocab, 91, "prompt")
    lo = np.stack([OV.prefill(case.spec, case.wn, case.caches[b], prompts[b])[-1] for b in range(B)])
    tokens = torch.from_numpy(prompts).to(torch.int32)
    ld = ver.prefill_batch(list(range(B)), tokens, [n] * B)
    assert np.max(np.abs(lo - ld.cpu().numpy())) < LOGIT_TOL[dtype]
    last = case.shape.n_layers - 1
    entries = [ver.kv_read(b, last, 0, n) for b in range(B)]
    ver.seq_set_lens(list(range(B)), [0] * B)
    assert ver.prefill_batch(list(range(B)), tokens, [n] * B, want_logits=False) is None      # nothing beyond the cache entries
    for b in range(B):
        assert ver.seq_len(b) == n and all(torch.equal(x, y) for x, y in zip(entries[b], ver.kv_read(b, last, 0, n)))
    ver.close()
    case.close()


@pytest.mark.parametrize("cached,lens", [
    ([5000, 3000], [70, 64]),             # the last rows' keys in pieces, of both
    ([5000, 0], [70, 70]),                # of one; the other's output comes from one piece
])
def test_last_rows_alone_over_keys_in_pieces(cached, lens):
    case = case_of("bf16", True, 2048, cached, extra=max(lens) + 8)
    prompts = W.make_tokens((2, max(lens)), 2048, 91, "prompt")
    lo = np.stack([OV.prefill(case.spec, case.wn, case.caches[b], prompts[b, :n])[-1] for b, n in enumerate(lens)])
    ld = case.ver.prefill_batch([0, 1], torch.from_numpy(prompts).to(torch.int32), lens).cpu().numpy()
    assert np.max(np.abs(lo - ld)) < LOGIT_TOL["bf16"]
    case.close()


@pytest.mark.parametrize("vocab", [2048, 128])    # normalised rows kept until the last pass; no room for them
def test_pages_that_run_out_in_a_later_pass(vocab):
    """The second of two passes does not get its pages: the error, the first prompt's logits, and lengths and cache as the first pass left them."""
    import ctypes as C
    lens = [40, 40, 20]                               # 64 rows and 36
    case = case_of("bf16", True, vocab, [0, 0, 0], extra=48)
    ver = other_verifier(case, prefill_rows=64, num_pages=4, pages_per_seq=3, page_size=32, max_k=1)
    prompts = W.make_tokens((3, 40), vocab, 91, "prompt")
    want = OV.prefill(case.spec, case.wn, case.caches[0], prompts[0])[-1]
    tokens = torch.from_numpy(prompts).to(torch.int32).to(case.device)
    out = torch.full((3, vocab), 77.0, dtype=torch.float32, device=case.device)
    rc = ver.lib.verify_prefill_batch(ver.ctx, (C.c_int32 * 3)(0, 1, 2), 3, C.c_void_p(tokens.data_ptr()), 40, (C.c_int32 * 3)(*lens), C.c_void_p(out.data_ptr()))
    assert rc == -2 and ver.lib.verify_last_error(ver.ctx).decode() == "need 2 more pages, 1 free"
    assert np.max(np.abs(out[0].cpu().numpy() - want)) < LOGIT_TOL["bf16"] and bool((out[1:] == 77.0).all())
    assert [ver.seq_len(b) for b in range(3)] == [40, 24, 0]
    ver.seq_remove(0)                                  # its pages let the others go on
    rest = torch.zeros((2, 20), dtype=torch.int32)
    rest[0, :16], rest[1] = tokens[1, 24:].cpu(), tokens[2, :20].cpu()
    ld = ver.prefill_batch([1, 2], rest, [16, 20]).cpu().numpy()
    for b in (1, 2):
        lo = OV.prefill(case.spec, case.wn, case.caches[b], prompts[b, :lens[b]])[-1]
        assert np.max(np.abs(ld[b - 1] - lo)) < LOGIT_TOL["bf16"]
    ver.close()
    case.close()


def test_more_last_rows_than_the_work_list_holds():
    """4096 prompts of two tokens and 33 q heads on one kv head: every prompt's last row lies in two work items, and the list has no room for those
    again.  The last layer then takes all rows; the prompts a thousand at a time do not come to that."""
    import paper_2511_16193_amd as P
    dev, B, d, hq, hd, V = "cuda:0", 4096, 128, 33, 128, 256
    g = torch.Generator(dev).manual_seed(3)
    rnd = lambda *s, std=1.0: torch.empty(s, dtype=torch.bfloat16, device=dev).normal_(0.0, std, generator=g)
    one = torch.ones(d, dtype=torch.bfloat16, device=dev)
    w = P.pack_weights({"embed": rnd(V, d), "lm_head": rnd(V, d, std=0.1), "final_norm": one, "layers": [
        {"ln1": one, "wqkv": rnd((hq + 2) * hd, d, std=0.1), "wo": rnd(d, hq * hd, std=0.02), "ln2": one, "w_gate_up": rnd(256, d, std=0.1),
         "w_down": rnd(d, 128, std=0.1)} for _ in range(2)]})
    model = dict(n_layers=2, d_model=d, n_q_heads=hq, n_kv_heads=1, head_dim=hd, d_ff=128, vocab=V, n_experts=0, top_k=0, d_expert=0, dtype="bf16",
                 rope_theta=1.0e4, rms_eps=1.0e-6)
    ver = P.Verifier(model, w, packed=True, max_batch=B, max_k=1, max_chains=1, max_seqs=B, page_size=32, num_pages=B + 4, max_pages_per_seq=1,
                     verify_mode=P.SV_MATCH, prefill_rows=0, device=dev)
    tokens = torch.randint(0, V, (B, 2), generator=g, device=dev).to(torch.int32)
    for b in range(B):
        ver.seq_add(b, 0)
    all_at_once = ver.prefill_batch(list(range(B)), tokens, [2] * B)
    ver.seq_set_lens(list(range(B)), [0] * B)
    by_parts = torch.cat([ver.prefill_batch(list(range(b, b + 1024)), tokens[b:b + 1024], [2] * 1024) for b in range(0, B, 1024)])
    assert float((all_at_once - by_parts).abs().max()) < LOGIT_TOL["bf16"] and float(by_parts.std()) > 0.1
    ver.close()
