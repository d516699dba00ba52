"""The exponential race where one id holds most of the probability, so that its score rules the others out from the start, and where none does."""
import numpy as np
import pytest
import torch

from oracle import verify as OV
from harness import decide
import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("k,V,temp,peak,sure,one_hot", [
    (0, 4099, 1.0, 12.0, 0.0, True),          # plain decoding: the likeliest id is drawn as a rule
    (3, 4099, 1.0, 12.0, 0.0, True),          # wrong one-hot drafts: the residual is led by the likeliest id
    (3, 8192, 0.7, 6.0, 0.97, False),         # the draft distribution holds more of that id than the target: no residual there
    (3, 8192, 1.0, 8.0, 0.3, False),          # and less of it
    (3, 40961, 1.0, 0.0, 0.0, False),         # nearly flat: its score rules little out
])
def test_race_from_a_peaked_row_matches_oracle(k, V, temp, peak, sure, one_hot):
    """Identical fp32 logits on both sides: accepted lengths and tokens are identical except where the oracle's own margin is below 1e-5 (fp32
    against fp64 evaluation of exp and log)."""
    from paper_2511_16193_amd import op_sample
    B = 24
    rng = np.random.default_rng(V + k)
    logits = rng.standard_normal((B, 1 + k, V)).astype(np.float32)
    top = rng.integers(0, V, (B, 1 + k))
    np.put_along_axis(logits, top[..., None], peak + 1.5, -1)
    drafts = rng.integers(0, V, (B, 1, k))
    q = None
    if not one_hot:
        q = W.make_random_q((B, 1, k), V, 1.0, 3).numpy() * (1 - sure)
        if sure:
            np.put_along_axis(q[:, 0], top[:, :k, None], np.take_along_axis(q[:, 0], top[:, :k, None], -1) + sure, -1)
        q = q.astype(np.float32)
    u = W.make_uniforms((B, 1, k + 1), 11)
    a, out, best, margin = decide(logits, drafts, q, u, OV.STOCHASTIC, OV.SAMPLE_EXP_RACE, temp, None)
    ga, gout, _ = op_sample(torch.from_numpy(logits).to(DEV), torch.from_numpy(drafts).to(torch.int32).to(DEV).contiguous(),
                            None if q is None else torch.from_numpy(q).to(DEV).contiguous(), torch.from_numpy(u).to(DEV),
                            verify_mode=OV.STOCHASTIC, sample_mode=OV.SAMPLE_EXP_RACE, temperature=temp, draft_lens=None)
    ga, gout = ga.cpu().numpy(), gout.cpu().numpy()
    bad = [b for b in range(B) if ga[b] != a[b] or not np.array_equal(gout[b], out[b])]
    assert all(margin[b] < 1e-5 for b in bad) and len(bad) <= 3
