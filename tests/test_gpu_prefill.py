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
        for layer, frac, atol in ((0, 0.01, 0.02), (shape.n_layers - 1, 1.0, 0.03)):    # as in the step tests: layer 0 sees equal inputs
            kd, vd = case.ver.kv_read(b, layer, cached[b], n)
            ko, vo = case.caches[b].k[layer][cached[b]:cached[b] + n], case.caches[b].v[layer][cached[b]:cached[b] + n]
            kd, vd = kd.float().cpu().numpy(), vd.float().cpu().numpy()
            assert np.max(np.abs(kd - ko)) < atol and np.max(np.abs(vd - vo)) < atol
            assert np.mean(kd != ko) <= frac and np.mean(vd != vo) <= frac
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
