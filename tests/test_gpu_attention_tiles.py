"""Attention of more than 48 stacked rows: pieces of every small number of 32-key tiles."""
import numpy as np
import pytest
import torch

import paper_2511_16193_amd as P
from oracle import model as M
from oracle import verify as OV
import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _bf16(shape, seed):
    return torch.randn(shape, generator=torch.Generator().manual_seed(seed)).to(torch.bfloat16)


@pytest.mark.parametrize("k,chains,group,max_tiles", [(8, 1, 7, 4), (8, 3, 5, 4), (5, 2, 7, 4), (8, 3, 5, 3), (8, 1, 7, 2)])   # row tiles 4, 4 + 4, 3 + 2, 3 x 3, 2 + 2
def test_every_small_number_of_tiles(k, chains, group, max_tiles):
    """One to eleven tiles, the last one whole, nearly empty or nearly full: each of the two waves takes none to six, so the loop over tiles
    runs every number of times around its first, last and skipped trips.  Tolerance as for the other lengths: the output is rounded to bf16, and the
    softmax weights to 16 significant bits: 2^-8 (|want| + sum_j p_j |v_j|)."""
    hkv, hd, n = 2, 128, 1 + chains * k
    lens = [max(0, 32 * t + part - n) for t in range(1, 12) for part in (0, 1, 31)]
    B, hq = len(lens), hkv * group
    model = dict(n_layers=1, d_model=256, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=512, vocab=2048, dtype="bf16", rope_theta=1e6, rms_eps=1e-6)
    ver = P.Verifier(model, W.make_weights(W.Shape("attn", 1, 256, hq, hkv, hd, 512, 2048), DEV), max_batch=B, max_k=k, max_chains=chains, max_seqs=B,
                     page_size=64, num_pages=B * 8, max_pages_per_seq=8, verify_mode=0)
    q = _bf16((B * n, hq, hd), 3)
    kv = [_bf16((2, L + n, hkv, hd), 10 + b) for b, L in enumerate(lens)]
    for b, L in enumerate(lens):
        ver.seq_add(b, L + n)
        ver.kv_write(b, 0, 0, kv[b][0].to(DEV), kv[b][1].to(DEV))
        ver.seq_set_len(b, L)
    ver.set_option(P.SV_OPT_ATTN_MAX_ROW_TILES, max_tiles)
    got = ver.op_attention(list(range(B)), n, k, 0, q.to(DEV)).float().cpu().numpy().reshape(B, n, hq, hd)
    ver.close()
    _, _, vis = OV.new_token_layout(k, chains)
    for b, L in enumerate(lens):
        mask = np.concatenate([np.ones((n, L), dtype=bool), vis], axis=1)
        qb, (kb, vb) = q[b * n:(b + 1) * n].double().numpy(), kv[b].double().numpy()
        want, spread = M.attend(qb, kb, vb, mask), M.attend(qb, kb, np.abs(vb), mask)
        assert np.all(np.abs(got[b] - want) <= 2.0 ** -8 * (np.abs(want) + spread) + 1e-6), (b, L, float(np.max(np.abs(got[b] - want))))
