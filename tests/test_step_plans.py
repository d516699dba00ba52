"""The launch plans of a step's packed projections and of a prefill's attention, host arithmetic: every one is a launch that its kernel takes."""
import pytest

from paper_2511_16193_amd import SvError, op_gemm_step_launch, op_gemm_step_plan, op_prefill_waves

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


ROWS = [1, 5, 33, 40, 96, 97, 128, 129, 147, 160, 161, 192, 200, 256, 289, 320, 321, 500, 777, 1280, 2304, 4096]


@pytest.mark.parametrize("experts", [False, True])
@pytest.mark.parametrize("form", [0, 1, 2, 4])
def test_step_launches_are_launchable(form, experts):
    """What a step really launches: each of the kernels occurs, in a form that it takes, and where it is neither a strip nor the launch for a
    few rows it is the launch that op_gemm_step_plan gives."""
    seen = set()
    for M in ROWS:
        for N, K in SHAPES[form & 3]:
            p, wide = op_gemm_step_launch(M, N, K, form, experts=experts), op_gemm_step_plan(M, N, K, form & 3)
            s, at = p["splits"], (M, N, K, form, p)
            seen.add(p["kernel"])
            assert 1 <= s <= 16 and (form in (0, 4) or s == 1), at
            if p["kernel"] == "few":
                assert M <= (8 if form == 2 else 16) and form != 1 and not experts, at
                assert (s, p["wide"], p["row_tiles"], p["features"], p["tall"]) == (1, False, 0, 0, None), at
                assert op_gemm_step_launch(M, N, K, form, tile_mode=0)["kernel"] == "ws", at
            elif p["kernel"] == "strip":
                assert p["features"] in (128, 160, 224) and p["row_tiles"] in (1, 2, 3, 4, 5, 6, 8, 10), at
                assert p["row_tiles"] * 32 >= M > 32 * (p["row_tiles"] - (1 if p["row_tiles"] <= 6 else 2)) and M <= 320, at
                assert K % (32 * s) == 0 and p["tall"] is None and not p["wide"], at
                if experts:                                                 # the splits, and the bits, of the launch it replaces
                    assert s == wide["splits"], at
            elif p["kernel"] == "tall":
                assert (p["tall"], s) == (wide["tall"], wide["splits"]) and p["row_tiles"] == p["features"] == 0, at
            else:
                assert wide["tall"] is None and p["features"] == 0 and p["tall"] is None, at
                assert (s, p["wide"], p["row_tiles"]) == (wide["splits"], wide["wide"], wide["row_tiles"]), at
    assert seen >= ({"strip", "tall"} if form == 2 else {"ws", "tall", "strip"}) and ("few" in seen) == (form != 1 and not experts)


@pytest.mark.parametrize("N,K,form,most", [
    (4608, 3584, 4, 16), (3584, 3584, 0, 16), (37888, 3584, 2, 8), (3584, 18944, 0, 8),          # QKV, O, gate/up and down of the 7B-shaped decoder
    (7168, 5120, 4, 16), (5120, 5120, 0, 8), (55296, 5120, 2, 8), (5120, 27648, 0, 8),           # of the 32B-shaped one
    (10240, 5120, 4, 0), (10240, 5120, 0, 0),                              # more than 8192 features
    (37888, 6208, 2, 0), (57600, 3584, 2, 0),                              # rows too wide to be normalised inside; more gate features than 7 x 16 x 256
    (4096, 128, 4, 0), (152064, 3584, 1, 0),                               # no step for every wave; an LM head
    (1024, 4096, 0, 16), (1024, 4160, 0, 8), (1024, 6144, 0, 8), (2048, 6656, 0, 0), (1024, 16384, 0, 0), (2432, 8192, 0, 0),     # narrow: long reductions are
    (512, 10240, 0, 8), (512, 10752, 0, 0), (640, 10240, 0, 0), (2560, 8192, 0, 16), (2560, 24576, 0, 8),                         # split instead, where they
    (2048, 11008, 0, 8), (896, 4864, 0, 16), (1024, 17152, 0, 8), (2048, 16384, 4, 16), (32768, 2048, 2, 8),                      # can be in eight
])
def test_a_few_rows(N, K, form, most):
    """Up to `most` rows norm, rotary or residual ride in the projection, unless experts, the option or the weights' alignment forbid it."""
    for M in (1, 5, 8, 9, 12, 16, 17):
        assert (op_gemm_step_launch(M, N, K, form)["kernel"] == "few") == (M <= most), (M, N, K, form)
        for kw in (dict(experts=True), dict(aligned=False), dict(tile_mode=0), dict(tile_mode=1)):
            assert op_gemm_step_launch(M, N, K, form, **kw)["kernel"] != "few", (M, N, K, form, kw)


@pytest.mark.parametrize("tile_mode", [-1, 0, 1])
@pytest.mark.parametrize("form", [0, 1, 2])
def test_weights_off_16_bytes_keep_the_kernel_with_ordinary_loads(form, tile_mode):
    """The tall kernel and the strips request 16 bytes a lane straight into LDS; the weight-streaming kernel loads into registers."""
    for M in ROWS:
        for N, K in SHAPES[form]:
            p = op_gemm_step_launch(M, N, K, form, tile_mode=tile_mode, aligned=False)
            assert p["kernel"] == "ws", (M, N, K, p)
            if form != 2:
                assert K % (64 * p["splits"]) == 0 and (not p["wide"] or N % 256 == 0) and 1 <= p["row_tiles"] <= 5, (M, N, K, p)


@pytest.mark.parametrize("F,K,kernels", [
    (18944, 3584, {9: "strip", 96: "strip", 160: "strip", 161: "strip", 320: "strip", 321: "tall"}),
    (27648, 5120, {9: "strip", 160: "strip", 192: "strip", 321: "tall"}),
    (28672, 8192, {5: "strip", 160: "strip"}),                             # 256 strips of 112 features
    (29568, 8192, {5: "ws", 64: "ws", 96: "ws", 160: "ws", 161: "tall", 320: "tall"}),       # 462 strips, a last round of 206
    (32768, 4096, {5: "ws", 160: "ws"}),                                   # 256 strips of the weight-streaming kernel: one round
    (49152, 6144, {5: "strip", 64: "strip", 160: "strip", 161: "tall", 320: "tall"}),        # 384 of them: a second round in any case
    (14336, 4096, {160: "strip", 256: "strip", 320: "tall"}),
    (5632, 2048, {128: "strip", 129: "ws", 160: "ws", 161: "strip"}),      # 44 strips of five 32-row tiles fit the CUs at once
    (6528, 2048, {160: "ws"}), (6656, 2048, {160: "strip"}),               # 51 and 52 strips
])
def test_gate_up_takes_strips_where_they_are_measured_to_pay(F, K, kernels):
    for M, kernel in kernels.items():
        p = op_gemm_step_launch(M, 2 * F, K, 2)
        assert p["kernel"] == kernel, (M, F, K, p)
        if kernel == "strip" and F < 40000:                                 # one round of work-groups
            assert -(-2 * F // p["features"]) <= 256, (M, F, K, p)


def test_strips_of_short_reductions():
    """Beyond a few rows: up to 4096 inputs strips of one, two or five row tiles, if the weights are 24 MB; longer ones take strips up to
    160 rows."""
    for M in ROWS[2:]:
        for N, K in [(4608, 3584), (3584, 3584), (6144, 4096), (4096, 4096)]:
            assert (op_gemm_step_launch(M, N, K)["kernel"] == "strip") == (M <= 64 or 129 <= M <= 160), (M, N, K)
        for N, K in [(5120, 2048), (2048, 4096), (1152, 896), (2048, 1024)]:
            p, wide = op_gemm_step_launch(M, N, K), op_gemm_step_plan(M, N, K)
            assert p["kernel"] != "strip" and (p["splits"], p["tall"]) == (wide["splits"], wide["tall"]), (M, N, K, p)
    for M in (17, 40, 96, 160):
        for N, K in [(3584, 18944), (5120, 27648), (4096, 14336), (7168, 5120), (10240, 8192)] + [(896, 4864), (2048, 11008)] * (M < 160):
            assert op_gemm_step_launch(M, N, K)["kernel"] == "strip", (M, N, K)
    assert op_gemm_step_launch(320, 3584, 18944)["kernel"] == "strip"


@pytest.mark.parametrize("N,K,kernels", [
    (152064, 3584, {96: "ws", 97: "strip", 160: "strip", 192: "strip", 320: "strip", 321: "tall", 2304: "tall"}),
    (151936, 2048, {96: "ws", 192: "strip", 320: "strip", 400: "tall"}),
    (151936, 1024, {176: "ws", 192: "ws", 320: "strip", 640: "tall"}),     # short reductions: tall tiles by the line of the other projections
    (151936, 896, {176: "ws", 192: "ws"}),
    (50304, 1024, {128: "strip", 192: "tall", 256: "tall", 320: "tall"}),  # tall tiles expected ahead of one round of strips
])
def test_lm_heads(N, K, kernels):
    for M, kernel in kernels.items():
        p = op_gemm_step_launch(M, N, K, 1)
        assert p["kernel"] == kernel and p["splits"] == 1, (M, N, K, p)


def test_what_is_no_projection_of_a_step_is_refused():
    for args in [(0, 256, 64, 0), (5, 200, 64, 0), (5, 256, 32, 0), (5, 384, 64, 2), (5, 256, 64, 3), (5, 256, 64, -1)]:
        with pytest.raises(SvError):
            op_gemm_step_plan(*args)
        with pytest.raises(SvError):
            op_gemm_step_launch(*args)
    with pytest.raises(SvError):
        op_gemm_step_launch(5, 256, 64, 0, tile_mode=2)


def _prompt(group, n, cached=0, cut=1):
    """Keys of a prompt's attention items: 64 stacked rows each, cut into equal parts of whole 32-key tiles."""
    total = cached + n
    part = (-(-total // cut) + 31) // 32 * 32
    ends = [cached + (min(64 * (g + 1), group * n) - 1) // group + 1 for g in range(-(-group * n // 64))]
    return [max(1, min(e, at + part) - at) for e in ends for at in range(0, total, part)]


@pytest.mark.parametrize("heads,keys,waves", [
    (4, _prompt(7, 777), 4), (4, _prompt(7, 1100), 4), (8, _prompt(2, 2048), 4),       # one prompt: 340, 484 and 512 work-groups, the shortest share places
    (8, _prompt(2, 2049), 2), (4, _prompt(7, 1200), 2),                                # more than 512
    (4, _prompt(7, 400) * 2, 2), (4, _prompt(7, 300) * 2, 2), (16, _prompt(1, 260) * 4, 2),       # several short ones: 352, 264, 320
    (8, _prompt(4, 100, 4000, 4) * 2, 2), (8, _prompt(5, 64, 1000) * 8, 2), (8, _prompt(5, 40, 16000, 16), 2),    # pieces of one length, more than 256
    (8, [1000] * 32, 4), (8, [1000] * 33, 2), (8, [4096] * 64, 4), (8, [4096] * 65, 2),
    (4, [256], 4), (4, [255], 2), (4, [255] * 64, 2),
    (1, [600] * 256 + [60], 4), (1, [60] + [600] * 256, 4), (1, [600] * 256 + [61], 2), (1, [511] * 256 + [1], 2), (16, [512] * 16 + [48], 4),
])
def test_waves_of_a_prefills_attention(heads, keys, waves):
    """Four where every work-group has a place, or those that wait for one are short."""
    assert op_prefill_waves(keys, heads) == waves


def test_prefill_waves_refuses_nonsense():
    for keys, heads in (([], 4), ([100], 0), ([100, 0], 4)):
        with pytest.raises(SvError):
            op_prefill_waves(keys, heads)
