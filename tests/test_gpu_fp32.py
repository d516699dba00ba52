"""fp32 models at sizes where the projection tiles and the attention's chunks end raggedly, against the oracle."""
import numpy as np
import pytest

from oracle import verify as OV
import workloads as W
from harness import Case, compare_step, LOGIT_TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,k,chains,hd,d,ff,vocab,lo,hi", [
    (1, 0, 1, 64, 128, 333, 1001, 0, 0),        # one row, reductions of 333 and vocabularies of 1001: no whole 16-byte pieces
    (4, 3, 1, 64, 252, 64, 515, 254, 258),      # 16 rows; contexts that end around a chunk of 256 keys
    (3, 5, 2, 128, 128, 1024, 640, 30, 700),    # 33 rows; several chunks, two chains, head_dim 128
    (6, 2, 1, 128, 128, 64, 515, 250, 262),     # head_dim 128: contexts that end around a chunk of 256 keys
    (6, 2, 1, 128, 128, 64, 515, 506, 546),     # and around two, in the first tiles of the third
    (220, 4, 1, 64, 64, 128, 2053, 1, 40),      # 1100 rows: 64-row tiles per wave, remainders in rows and features
])
def test_fp32_step(batch, k, chains, hd, d, ff, vocab, lo, hi):
    shape = W.Shape("f32-edge", 2, d, 4, 2, hd, ff, vocab, dtype="fp32", rope_theta=1e4, batch=batch, k=k, n_chains=chains, seed=31)
    rng = np.random.default_rng(7)
    case = Case(shape, rng.integers(lo, hi + 1, size=batch), verify_mode=OV.STOCHASTIC, sample_mode=OV.SAMPLE_EXP_RACE)
    x0 = W.make_tokens((batch,), vocab, shape.seed, "x0")
    q = W.make_random_q((batch, chains, k), vocab, 1.0, shape.seed) if k else None
    drafts = W.sample_from(q, shape.seed).numpy() if k else np.zeros((batch, 1, 0), dtype=np.int64)
    r, g = case.step(x0, drafts, q, W.make_uniforms((batch, chains, k + 1), shape.seed))
    err, exempt, diverged = compare_step(r, g, "fp32", k)
    assert err < LOGIT_TOL["fp32"] and len(diverged) <= 1
    case.close()


@pytest.mark.parametrize("batch,k,hd,d,ff,vocab", [
    (1, 0, 128, 4, 31, 7),            # one reduction group, most of it beyond the end; fewer features than a tile
    (4, 3, 64, 260, 130, 2061),       # 16 rows, one whole tile; the vocabulary ends in a tile of 13 features
    (17, 0, 64, 1024, 516, 1026),     # 17 rows; the longest reduction that the projections normalise themselves
    (17, 0, 128, 1028, 516, 1026),    # just beyond it: norms and rotary as launches of their own
    (51, 4, 64, 64, 320, 128),        # 255 rows, 16 tiles of gate/up features in 16 rows: the last that a CU each holds
    (52, 4, 64, 64, 320, 128),        # 260 rows: one tile more than CUs
])
def test_fp32_step_where_norms_and_rotary_ride_in_the_projections(batch, k, hd, d, ff, vocab):
    shape = W.Shape("f32-fused", 2, d, 4, 2, hd, ff, vocab, dtype="fp32", rope_theta=1e4, batch=batch, k=k, n_chains=1, seed=33)
    case = Case(shape, np.random.default_rng(9).integers(0, 70, size=batch), verify_mode=OV.STOCHASTIC, sample_mode=OV.SAMPLE_EXP_RACE)
    x0 = W.make_tokens((batch,), vocab, shape.seed, "x0")
    q = W.make_random_q((batch, 1, k), vocab, 1.0, shape.seed) if k else None
    drafts = W.sample_from(q, shape.seed).numpy() if k else np.zeros((batch, 1, 0), dtype=np.int64)
    r, g = case.step(x0, drafts, q, W.make_uniforms((batch, 1, k + 1), shape.seed))
    err, exempt, diverged = compare_step(r, g, "fp32", k)
    assert err < LOGIT_TOL["fp32"] and len(diverged) <= 1
    case.close()


@pytest.mark.parametrize("batch,k,hd,d,ff,vocab", [
    (1, 0, 64, 64, 4097, 64),         # one row; one feature more in gate/up than a CU a tile
    (4, 3, 64, 132, 4112, 4097),      # 16 rows; gate/up and the vocabulary just beyond that line
    (4, 3, 64, 68, 4103, 64),         # down over 4103 inputs: no whole 16-byte pieces
    (17, 0, 64, 64, 4097, 4097),      # 17 rows: 32-row tiles beyond the line
])
def test_fp32_step_of_few_rows_over_many_features(batch, k, hd, d, ff, vocab):
    shape = W.Shape("f32-wide", 2, d, 4, 2, hd, ff, vocab, dtype="fp32", rope_theta=1e4, batch=batch, k=k, n_chains=1, seed=37)
    case = Case(shape, np.random.default_rng(11).integers(0, 70, size=batch), verify_mode=OV.STOCHASTIC, sample_mode=OV.SAMPLE_EXP_RACE)
    x0 = W.make_tokens((batch,), vocab, shape.seed, "x0")
    q = W.make_random_q((batch, 1, k), vocab, 1.0, shape.seed) if k else None
    drafts = W.sample_from(q, shape.seed).numpy() if k else np.zeros((batch, 1, 0), dtype=np.int64)
    r, g = case.step(x0, drafts, q, W.make_uniforms((batch, 1, k + 1), shape.seed))
    err, exempt, diverged = compare_step(r, g, "fp32", k)
    assert err < LOGIT_TOL["fp32"] and len(diverged) <= 1
    case.close()
