"""The launch plans of a step's packed projections, host arithmetic: every one is a launch that its kernel takes."""
import pytest

from paper_2511_16193_amd import SvError, op_gemm_step_plan

# QKV, O, down; LM head; gate/up of the 7B-, 32B- and expert-shaped decoders, and small models
SHAPES = {0: [(4608, 3584), (3584, 3584), (3584, 18944), (7168, 5120), (5120, 5120), (5120, 27648), (5120, 2048), (2048, 4096), (256, 1024), (1536, 64)],
          1: [(152064, 3584), (152064, 5120), (151936, 2048), (2048, 256)],
          2: [(37888, 3584), (55296, 5120), (1024, 256)]}


@pytest.mark.parametrize("form", [0, 1, 2])
def test_step_plans_are_launchable(form):
    for M in [1, 5, 33, 40, 96, 128, 129, 147, 160, 161, 192, 200, 320, 321, 500, 640, 777, 800, 1000, 1280, 2048, 2304, 3600, 4096]:
        for N, K in SHAPES[form]:
            p = op_gemm_step_plan(M, N, K, form)
            s, at = p["splits"], (M, N, K, form, p)
            assert 1 <= s <= 16 and (form == 0 or s == 1), at
            if p["tall"]:
                h, n, ht, nt = p["tall"]
                assert h in (3, 4, 5) and 0 <= ht < h and n >= 1 and (nt > 0) == (ht > 0), at
                rows = 64 * (h * n + ht * nt)
                assert rows >= M > rows - 64 * (ht or h), at                # all rows, and no tile of padding alone
                assert K % (32 * s) == 0 and M > 128, at
            elif form == 2:
                assert M <= 160, at
            else:
                mt = p["row_tiles"]
                assert K % (64 * s) == 0 and (not p["wide"] or N % 256 == 0) and 1 <= mt <= 5, at
                assert mt * 32 * ((M + 32 * mt - 1) // (32 * mt)) < M + 32 * mt, at


def test_what_is_no_projection_of_a_step_is_refused():
    for args in [(0, 256, 64, 0), (5, 200, 64, 0), (5, 256, 32, 0), (5, 384, 64, 2), (5, 256, 64, 3), (5, 256, 64, -1)]:
        with pytest.raises(SvError):
            op_gemm_step_plan(*args)
