"""silu(gate) * up as the projections' epilogues form it: the fp32 result against 64 bits, and beside what float operations with the
library's exponential and division give; gates beyond the range of the exponential, infinities and NaN in every kernel that has the epilogue.

A gate (an up value) is made exactly: one input of a row is not zero, and a weight row has the value there."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def plain(g, u):
    return g / (1.0 + torch.exp(-g)) * u


def test_fp32_layer_is_as_close_to_64_bits_as_plain_float_operations():
    """A layer without attention output, its rows one spike of sqrt(d), which the norm makes 32 exactly, down the identity: h_out is
    silu(g) * u.  Bound: the exponential's argument 2^-25 (two-part product) and its instruction 2^-23, the sum 2^-24, the quotient after one
    Newton step 2^-23, the last product 2^-24: 6 units of 2^-24, and the smallest normal number where the result leaves their range."""
    import paper_2511_16193_amd as P
    d, layers = 1024, 8
    gen = torch.Generator().manual_seed(5)
    gates = [torch.rand(d, generator=gen) * 40 - 20, torch.randn(d, generator=gen), torch.rand(d, generator=gen) * 2 - 1,
             torch.linspace(-87, 88, d), torch.linspace(-110, -80, d), torch.exp2(torch.linspace(-126, 0, d)), -torch.exp2(torch.linspace(-126, 0, d)),
             torch.linspace(80, 3000, d)]
    ups = [torch.randn(d, generator=gen).to(torch.float32) for _ in range(layers)]
    lws = []
    for g, u in zip(gates, ups):
        gu = torch.zeros((2 * d, d))
        gu[:d, 0], gu[d:, 0] = g / 32, u / 32
        lws.append({"ln1": torch.ones(d), "wqkv": torch.zeros((192, d)), "wo": torch.zeros((d, 64)), "ln2": torch.ones(d), "w_gate_up": gu,
                    "w_down": torch.eye(d)})
    w = {"embed": torch.zeros((128, d), device=DEV), "lm_head": torch.zeros((128, d), device=DEV), "final_norm": torch.ones(d, device=DEV),
         "layers": [{n: t.to(DEV).contiguous() for n, t in lw.items()} for lw in lws]}
    model = dict(n_layers=layers, d_model=d, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ff=d, vocab=128, n_experts=0, top_k=0, d_expert=0,
                 dtype="fp32", rope_theta=1.0e4, rms_eps=0.0)
    ver = P.Verifier(model, w, max_batch=1, max_k=1, max_chains=1, max_seqs=1, page_size=32, num_pages=4, max_pages_per_seq=2,
                     verify_mode=P.SV_GREEDY, sample_mode=P.SV_EXP_RACE, temperature=1.0, device=DEV)
    ver.seq_add(0, 1)
    for l in range(layers):
        ver.kv_write(0, l, 0, torch.zeros((1, 1, 64), device=DEV), torch.zeros((1, 1, 64), device=DEV))
    h = torch.zeros((1, d), device=DEV)
    h[0, 0] = 32.0
    units, units_plain = [], []
    for l, (lw, u) in enumerate(zip(lws, ups)):
        got = ver.op_layer([0], 1, 0, l, h)[0, 1:].cpu().double()
        g, u = (32 * lw["w_gate_up"][:d, 0])[1:], (32 * lw["w_gate_up"][d:, 0])[1:]
        want = g.double() / (1 + torch.exp(-g.double())) * u.double()
        err = (got - want).abs()
        near = err <= 6 * 2.0 ** -24 * want.abs() + 2.0 ** -126
        # e^-g beyond the floats (g < -88.73) makes plain operations return 0 where the value is still about 2^-121: 0 or nearer to it
        lost = (g < -88.72) & (err <= want.abs())
        assert bool((near | lost).all()), (l, g[~(near | lost)][:4], got[~(near | lost)][:4])
        if l < 3:
            units.append((err / want.abs() * 2 ** 24).numpy())
            units_plain.append(((plain(g.to(DEV), u.to(DEV)).cpu().double() - want).abs() / want.abs() * 2 ** 24).numpy())
    ver.close()
    units, units_plain = np.concatenate(units), np.concatenate(units_plain)
    print("units of 2^-24, mean and largest:", units.mean(), units.max(), "float operations:", units_plain.mean(), units_plain.max())
    # the two differ in few results, by a unit in the last place: 1 % of the mean covers 3069 values
    assert units.mean() <= 1.01 * units_plain.mean() and units.max() <= units_plain.max() + 1


@pytest.mark.parametrize("rows,kernel", [(5, "ws"), (150, "ws"), (5, "strip"), (320, "strip"), (200, "tall")])
def test_gates_at_and_beyond_the_ends_of_the_range(rows, kernel):
    """g / (1 + e^-g) * u in IEEE terms: +inf * u, NaN for -inf, a zero (or what a denormal rounds to) where e^-g overflows."""
    import paper_2511_16193_amd as P
    inf, nan = float("inf"), float("nan")
    g0 = torch.tensor([inf, -inf, nan, 0.0, -0.0, 2.0 ** -126, -(2.0 ** -126), 20.0, -20.0, 87.0, -87.0, 88.5, -88.0, -88.5, -89.0, -100.0, -104.0, -110.0,
                       -150.0, 150.0, 1e4, -1e4, 1e38, -1e38, 3.3e38, -3.3e38])
    u0 = torch.tensor([1.0, -2.0, 0.0, inf, -inf, nan, 3e-38, 1e30])
    F, K = 384, 64
    g, u = torch.zeros(F), torch.zeros(F)
    pairs = torch.cartesian_prod(g0, u0)
    g[:len(pairs)], u[:len(pairs)] = pairs[:, 0], pairs[:, 1]
    g, u = g.to(torch.bfloat16), u.to(torch.bfloat16)
    w = torch.zeros((2 * F, K), dtype=torch.bfloat16)
    w[:F, 0], w[F:, 0] = g, u
    a = torch.zeros((rows, K), dtype=torch.bfloat16)
    a[:, 0] = 1.0
    ap, wp = P.op_pack_rows(a.to(DEV)), P.op_pack_weight(w.to(DEV))
    tiles = (rows + 31) // 32
    got = (P.op_gemm_bf16_strip(ap, wp, rows, tiles, 160, gated=True) if kernel == "strip"
           else P.op_gemm_bf16_tall(ap, wp, rows, (4, 1, 0, 0) if kernel == "tall" else None, gated=True))
    got = got.view(-1, F // 16, 2, 32, 8).permute(0, 3, 1, 2, 4).reshape(-1, F)[:rows].float().cpu()
    assert torch.equal(got.nan_to_num(1.5), got[:1].nan_to_num(1.5).expand_as(got))
    gd, ud = g.double(), u.double()
    silu = gd / (1 + torch.exp(-gd))                                        # (64 bits do not overflow where 32 do: 0 or nearly 0)
    want = silu * ud
    lost = (gd < -88.72) & torch.isfinite(gd)                               # e^-g beyond the floats: 0, or nearer to the value
    tiny = lost | ((silu.abs() < 2.0 ** -125) & torch.isfinite(silu))       # a zero or a denormal in 32 bits: times inf NaN or inf
    for i in range(F):
        x, y = float(got[0, i]), float(want[i])
        at = (float(g[i]), float(u[i]), x, y)
        if tiny[i] and np.isinf(float(u[i])):
            assert np.isnan(x) or np.isinf(x), at
        elif np.isnan(y):
            assert np.isnan(x), at
        elif abs(y) > 3.3e38:
            assert x == np.sign(y) * inf or abs(x / y - 1) < 0.01, at
        else:
            assert abs(x - y) <= (1.0 if lost[i] else 2.0 ** -8 * 1.01) * abs(y) + 2.0 ** -125 * max(1.0, abs(float(u[i]))), at
