"""The expert layer at the edges of its launches: a whole operand tile of rows and one more, one to four row tiles per expert,
the most experts, and the router's reduction in sixteen parts."""
import pytest

import workloads as W
from oracle import verify as OV
from harness import Case, LOGIT_TOL, compare_step
from test_gpu_moe import test_moe_ffn_matches_oracle as check_ffn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,top_k,F", [
    (1, 256, 64, 8, 128),          # one row
    (32, 256, 256, 8, 128),        # a whole operand tile, the most experts: most of them chosen by no row
    (33, 256, 64, 8, 128),         # one row more: grouped and gathered
    (384, 128, 64, 8, 128),        # 48 rows an expert on average: the last count of the two-tile launch, some in two groups
    (386, 128, 64, 8, 128),        # the first of the four-tile launch: groups of one, two and three tiles
])
def test_ffn_at_launch_edges(T, d, E, top_k, F):
    check_ffn(T, d, E, top_k, F, 0.0)


def test_step_with_the_router_in_sixteen_parts():
    """d_model 2048 and 20 rows: sixteen work-groups share the router's reduction, the products read the activations' own tile."""
    shape = W.Shape("moe-tile", 2, 2048, 8, 2, 128, 0, 2048, dtype="bf16", n_experts=64, top_k=4, d_expert=128, batch=4, k=4, seed=83)
    case = Case(shape, [5, 60, 200, 333], verify_mode=OV.STOCHASTIC, sample_mode=OV.SAMPLE_EXP_RACE, packed=True)
    x0 = W.make_tokens((4,), shape.vocab, shape.seed, "x0")
    q = W.make_random_q((4, 1, 4), shape.vocab, 1.0, shape.seed)
    r, g = case.step(x0, W.sample_from(q, shape.seed).numpy(), q, W.make_uniforms((4, 1, 5), shape.seed))
    err, exempt, diverged = compare_step(r, g, "bf16", 4)
    assert err < LOGIT_TOL["bf16"] and len(diverged) <= 1
    case.close()


@pytest.mark.parametrize("T", [20, 300])
def test_matrices_that_end_where_their_memory_ends(T):
    """Stacks of 64 and 32 MiB, whole allocations: the weights requested ahead of the last strips' products, and the rows
    ahead of the last fills', have nothing behind them that may be read."""
    check_ffn(T, 1024, 64, 8, 256, 0.0)


@pytest.mark.parametrize("T", [20, 40])                # choice and grouping in one launch, and in two
@pytest.mark.parametrize("dead", [0, 70])
def test_an_expert_without_a_probability_is_not_chosen(T, dead):
    """One expert's router row is NaN, so are its logits: the choice is that among the others."""
    import torch
    import paper_2511_16193_amd as P
    d, E, top_k, F = 256, 128, 8, 128
    g = torch.Generator().manual_seed(T)
    rnd = lambda *s, std=1.0: (torch.randn(s, generator=g) * std).to(torch.bfloat16)
    a, w_router, w_gate_up, w_down = rnd(T, d), rnd(E, d, std=0.3), rnd(E, 2 * F, d, std=0.06), rnd(E, d, F, std=0.09)
    w_router[dead] = float("nan")
    out, ids, wts = (x.cpu() for x in P.op_moe_ffn(a.cuda(), w_router.cuda(), w_gate_up.cuda(), w_down.cuda(), top_k))
    logits = a.double() @ w_router.double().T
    logits[:, dead] = float("-inf")
    top, want = torch.sort(torch.softmax(logits, -1), -1, descending=True)
    clear = (top[:, : top_k + 1].diff(dim=-1).abs() > 1e-4 * top[:, :1]).all(-1)      # no two choices that rounding could swap
    assert clear.sum() >= T // 2
    assert torch.equal(ids[clear].long(), want[clear, :top_k])
    assert float((wts[clear] - (top[:, :top_k] / top[:, :top_k].sum(-1, keepdim=True))[clear]).abs().max()) < 5e-5     # as in test_moe_ffn_matches_oracle
    assert not bool((ids == dead).any()) and bool(torch.isfinite(out).all())
