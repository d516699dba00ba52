"""A prefill's attention with four and with two waves a work-group, on both sides of where one gives way to the other."""
import numpy as np
import pytest
import torch

from oracle import verify as OV
import workloads as W
from harness import Case, LOGIT_TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cached,n", [(0, 2048), (0, 2049), (70, 2100)])      # 64, 65 and 66 groups of 64 stacked rows, eight kv heads
def test_prefill_of_about_512_work_groups(cached, n):
    shape = W.Shape("waves-bf16", 2, 256, 16, 8, 128, 512, 2048, dtype="bf16", batch=1, k=4, seed=63)
    case = Case(shape, [cached], verify_mode=OV.STOCHASTIC, synthetic_kv=True, extra_tokens=n + 8, packed=True)
    prompt = W.make_tokens((1, n), shape.vocab, shape.seed, "prompt")
    lo = OV.prefill(case.spec, case.wn, case.caches[0], prompt[0])[-1]
    ld = case.ver.prefill_batch([0], torch.from_numpy(prompt).to(torch.int32), [n]).cpu().numpy()[0]
    assert np.max(np.abs(lo - ld)) < LOGIT_TOL["bf16"]
    kd, vd = case.ver.kv_read(0, 1, cached, n)                                # they stand behind the first layer's attention of every row
    ko, vo = case.caches[0].k[1][cached:cached + n], case.caches[0].v[1][cached:cached + n]
    assert np.max(np.abs(kd.float().cpu().numpy() - ko)) < 0.03 and np.max(np.abs(vd.float().cpu().numpy() - vo)) < 0.03
    case.close()
