"""What a context asks of its caller: the workspace of a step alone, and what wider prefill passes add to it (host arithmetic)."""
import ctypes

import pytest

from paper_2511_16193_amd import binding as B


def size(rows=None, *, dense=True, batch=1, k=4, chains=1, pages=300):
    m = (B.SvModel(28, 3584, 28, 4, 128, 18944, 152064, 0, 0, 0, B.SV_BF16, 1e6, 1e-6) if dense
         else B.SvModel(48, 2048, 32, 4, 128, 0, 151936, 128, 8, 768, B.SV_BF16, 1e6, 1e-6))
    rt = B.SvRuntime(batch, k, chains, batch, 64, pages, pages, 1, 1, 1.0, None, 0, None, 0)
    f = B.lib().verify_workspace_bytes if rows is None else B.lib().sv_workspace_bytes
    return f(ctypes.byref(m), ctypes.byref(rt), *(() if rows is None else (rows,)))


def test_a_step_alone_needs_no_room_for_prefill():
    """Five rows of the 7B shape, and three a request of the expert one: logits, split-K planes and attention partials of the
    step, in MB rounded up; the same sizes as with prefill_rows = 0."""
    assert 0 < size(pages=110) < 8e6 and 0 < size(dense=False, batch=5, k=3, pages=60) < 62e6
    assert size(0) == size() and size(-1) == size()


def test_prefill_rows_are_paid_for_by_the_row():
    """A row of a prefill pass costs its activations and one split-K plane of the widest projection that has one: about
    0.12 MB on the 7B shape.  What it does not cost is the fp32 gate/up output, which no kernel of a packed model writes."""
    sizes = [size(r) for r in (0, 1024, 2048, 4096)]
    assert sizes == sorted(sizes) and sizes[3] < 520e6
    assert size(1 << 20) == size(4096)                       # no pass takes more
    assert size(4096, pages=4) == size(256, pages=4)         # nor more than the cache holds


@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("rows", [0, 96])
@pytest.mark.gpu
def test_prefill_through_narrow_passes(packed, rows):
    """The same prompts through a workspace of a step's rows, of 96 and of the default: other passes, the same cache up to
    roundings.  Row-major weights with a wide feed-forward: the default's passes are those the gate/up product has room for."""
    import numpy as np
    import torch
    import workloads as W
    from harness import Case, LOGIT_TOL
    from oracle import verify as OV
    shape = W.Shape("passes-bf16", 2, 256, 8, 2, 128, 2048, 2048, dtype="bf16", batch=2, k=4, seed=61)
    lens = [1700, 300]
    case = Case(shape, [0, 0], verify_mode=OV.STOCHASTIC, synthetic_kv=False, extra_tokens=1720, packed=packed)
    prompts = W.make_tokens((2, 1700), shape.vocab, shape.seed, "prompt")
    want = np.stack([OV.prefill(case.spec, case.wn, case.caches[b], prompts[b, :n])[-1] for b, n in enumerate(lens)])
    narrow = B.Verifier(shape.model_fields(), case.wd, max_batch=2, max_k=4, max_seqs=2, page_size=64, num_pages=60, max_pages_per_seq=30,
                        packed=packed, prefill_rows=rows)
    assert narrow.workspace.numel() < case.ver.workspace.numel()
    for ver in (case.ver, narrow):
        for b in (0, 1):
            if ver is narrow:
                ver.seq_add(b, 0)
        got = ver.prefill_batch([0, 1], torch.from_numpy(prompts).to(torch.int32), lens).cpu().numpy()
        assert np.max(np.abs(got - want)) < LOGIT_TOL["bf16"]
        assert [ver.seq_len(b) for b in (0, 1)] == lens
    narrow.close()
    case.close()


@pytest.mark.gpu
def test_a_full_device_gets_a_context_of_a_steps_workspace(monkeypatch):
    import torch
    import workloads as W
    from harness import to_device
    shape = W.Shape("full-bf16", 1, 256, 8, 2, 128, 512, 2048, dtype="bf16", batch=1, k=4, seed=61)
    w = to_device(W.make_weights(shape, "cpu"))
    make = lambda **kw: B.Verifier(shape.model_fields(), w, max_batch=1, max_k=4, num_pages=80, max_pages_per_seq=80, **kw)
    step = make(prefill_rows=0).workspace.numel()
    empty = torch.empty

    def full(*shape_, **kw):
        if kw.get("dtype") == torch.uint8 and shape_[0] > step and shape_[0] != pool:
            raise torch.cuda.OutOfMemoryError("no room")
        return empty(*shape_, **kw)

    pool = make().kv_pool.numel()
    monkeypatch.setattr(B.torch, "empty", full)
    assert make().workspace.numel() == step
    with pytest.raises(torch.cuda.OutOfMemoryError):
        make(prefill_rows=4096)
