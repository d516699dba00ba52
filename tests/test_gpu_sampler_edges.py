"""The sampler's parts and the race's shortcut at the edges, on given logits against the oracle."""
import numpy as np
import pytest
import torch

from oracle import verify as OV
from test_gpu_ops import DEV, oracle_sample, random_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N,k,V,temp,scale", [
    (5, 1, 2, 1000, 1.0, 1.0),        # a vocabulary of less than one load per thread: one part
    (3, 2, 3, 4100, 1.0, 8.0),        # few rows: many parts, the last one short; peaked distributions
    (700, 1, 2, 2048, 1.0, 1.0),      # many rows, two parts
    (4, 3, 2, 16384, 0.02, 1.0),      # log-probabilities in the thousands: what the hardware exponential flushes to zero
    (6, 1, 4, 33001, 1.0, 3.0),       # a width that is no multiple of four: scalar loads
])
@pytest.mark.parametrize("vmode", [OV.STOCHASTIC, OV.MATCH, OV.GREEDY])
def test_sampler_edges(B, N, k, V, temp, scale, vmode):
    from paper_2511_16193_amd import op_sample
    logits, drafts, q, u = random_case(B, N, k, V, 40 + V % 7)
    logits = (logits * scale).astype(np.float32)
    rng = np.random.default_rng(3)
    best = np.argmax(logits, axis=-1)
    for c in range(N):                                  # half of the drafts are the target's favourite, so windows go on
        rows = np.concatenate([best[:, :1], best[:, 1 + c * k: 1 + (c + 1) * k]], axis=1)[:, :k]
        drafts[:, c] = np.where(rng.random((B, k)) < 0.5, rows, drafts[:, c])
    lens = rng.integers(0, k + 1, B)
    lens[0] = 0
    with_q = vmode == OV.STOCHASTIC
    a, out, chain, margin = oracle_sample(logits, drafts, q if with_q else None, u, vmode, OV.SAMPLE_EXP_RACE, temp, lens)
    ga, gout, gchain = op_sample(torch.from_numpy(logits).to(DEV), torch.from_numpy(drafts).to(torch.int32).to(DEV).contiguous(),
                                 torch.as_tensor(q).to(DEV).contiguous() if with_q else None, torch.from_numpy(u).to(DEV),
                                 verify_mode=vmode, sample_mode=OV.SAMPLE_EXP_RACE, temperature=temp,
                                 draft_lens=torch.from_numpy(lens).to(torch.int32).to(DEV))
    ga, gout, gchain = ga.cpu().numpy(), gout.cpu().numpy(), gchain.cpu().numpy()
    bad = [b for b in range(B) if not (ga[b] == a[b] and gchain[b] == chain[b] and np.array_equal(gout[b], out[b]))]
    # fp32 logits of magnitude |x| / temp carry 2^-24 of it: closer decisions than twice that are not decided
    tol = max(1e-5, 2.0 ** -22 * float(np.abs(logits).max()) / temp)
    assert all(margin[b] < tol for b in bad), [(b, margin[b], ga[b], a[b], gout[b], out[b]) for b in bad]
    assert len(bad) <= max(1, B // 8)


@pytest.mark.parametrize("vmode", [OV.STOCHASTIC, OV.MATCH])
def test_inverse_cdf_over_a_row_of_nan_supplies_a_token_of_its_own(vmode):
    """No id of a NaN row has a weight: id 0 is supplied, not what a draw of an earlier call left in the scratch."""
    from paper_2511_16193_amd.binding import op_sample_static
    V = 1000
    logits = torch.zeros((2, 1, V), device=DEV)
    logits[:, 0, 777] = 50.0
    drafts = torch.zeros((2, 1, 0), dtype=torch.int32, device=DEV)
    u = torch.full((2, 1, 1), 0.5, device=DEV)
    acc, best = (torch.empty(2, dtype=torch.int32, device=DEV) for _ in range(2))
    got = []
    for poison in (False, True):
        if poison:
            logits[1, 0, 5] = float("nan")
        toks = torch.full((2, 1), -7, dtype=torch.int32, device=DEV)
        op_sample_static(logits, drafts, None, u, acc, toks, best, verify_mode=vmode, sample_mode=OV.SAMPLE_INVERSE_CDF)
        got.append(toks.cpu().numpy()[:, 0].tolist())
    assert got == [[777, 777], [777, 0]]


@pytest.mark.parametrize("vmode", [OV.STOCHASTIC, OV.MATCH])
def test_nan_logits_of_an_odd_vocabulary_count_as_none(vmode):
    """Rows that are read one id at a time skip a NaN: the outcome is that of minus infinity in its place."""
    from paper_2511_16193_amd import op_sample
    B, N, k, V = 6, 2, 3, 1001
    logits, drafts, q, u = random_case(B, N, k, V, 9)
    got = []
    for value in (-np.inf, np.nan):
        x = logits.astype(np.float32)
        x[:, :, 17::250] = value
        d = np.where(drafts % 250 == 17, 3, drafts)
        out = op_sample(torch.from_numpy(x).to(DEV), torch.from_numpy(d).to(torch.int32).to(DEV).contiguous(),
                        torch.as_tensor(q).to(DEV).contiguous() if vmode == OV.STOCHASTIC else None, torch.from_numpy(u).to(DEV),
                        verify_mode=vmode, sample_mode=OV.SAMPLE_EXP_RACE)
        got.append([t.cpu().numpy() for t in out])
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    assert all((t >= -1).all() and (t < V).all() for t in (got[1][1],))


@pytest.mark.parametrize("N", [1024, 1025, 50000])
@pytest.mark.parametrize("vmode", [OV.GREEDY, OV.STOCHASTIC, OV.MATCH])
def test_any_number_of_chains(N, vmode):
    """One chain far behind the others agrees with the target, and so does the last: the lower of the two is kept."""
    from paper_2511_16193_amd import op_sample
    V = 64
    logits = torch.zeros((1, 1 + N, V), device=DEV)
    logits[:, :, 5] = 60.0
    drafts = torch.full((1, N, 1), 9, dtype=torch.int32, device=DEV)
    drafts[0, [N - 3, N - 1]] = 5
    u = torch.full((1, N, 2), 0.5, device=DEV)
    acc, toks, best = op_sample(logits, drafts, None, u, verify_mode=vmode, sample_mode=OV.SAMPLE_EXP_RACE)
    assert (acc.item(), best.item(), toks.cpu().tolist()) == (1, N - 3, [[5, 5]])


def test_step_on_buffers_that_start_between_16_byte_boundaries():
    """Logits, draft probabilities and norm gains one element into their allocations (a slice of a larger tensor): the outcome is
    that of aligned ones, bit for bit."""
    import paper_2511_16193_amd as P
    import workloads as W
    from harness import to_device
    shape = W.Shape("offset-bf16", 2, 256, 8, 2, 128, 512, 2048, dtype="bf16", batch=3, k=3, n_chains=2, seed=71)
    B, N, k, V = 3, 2, 3, shape.vocab

    def apart(t):
        big = torch.empty(t.numel() + 1, dtype=t.dtype, device=DEV)
        out = big[1:].view(t.shape)
        out.copy_(t)
        return out

    q = W.make_random_q((B, N, k), V, 1.0, 5)
    drafts = W.sample_from(q, 5).to(torch.int32).to(DEV).contiguous()
    u = torch.from_numpy(W.make_uniforms((B, N, k + 1), 5)).to(DEV)
    x0 = torch.tensor([3, 5, 7], dtype=torch.int32, device=DEV)
    got = []
    for move in (lambda t: t, apart):
        w = P.pack_weights(to_device(W.make_weights(shape, "cpu")))
        w["final_norm"] = move(w["final_norm"])
        for lw in w["layers"]:
            lw["ln1"], lw["ln2"] = move(lw["ln1"]), move(lw["ln2"])
        ver = P.Verifier(shape.model_fields(), w, packed=True, max_batch=B, max_k=k, max_chains=N, num_pages=16, max_pages_per_seq=4)
        for b in range(B):
            ver.seq_add(b, 0)
            ver.prefill(b, torch.arange(20 + b, dtype=torch.int32))
        out = {"accepted_len": torch.zeros(B, dtype=torch.int32, device=DEV), "best_chain": torch.zeros(B, dtype=torch.int32, device=DEV),
               "out_tokens": torch.zeros((B, k + 1), dtype=torch.int32, device=DEV), "logits": move(torch.zeros((B, 1 + N * k, V), device=DEV))}
        ver.step([0, 1, 2], x0, drafts, move(q.to(DEV)), u, out=out)
        torch.cuda.synchronize()
        got.append({n: t.cpu() for n, t in out.items()})
        ver.close()
    assert all(torch.equal(got[0][n], got[1][n]) for n in got[0]) and float(got[0]["logits"].std()) > 0.1
