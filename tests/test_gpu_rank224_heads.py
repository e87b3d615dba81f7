"""Rank 193 to 224 with five to eight heads per KV head, where the attention
kernel keeps the split's latent values in its gather buffers: one tile, one pair
of tiles, several pairs per workgroup, odd counts."""

import numpy as np
import pytest
import torch

import paper_2608_00528_amd as s4r
import workloads as W
from oracle import decode
from tests.gpu_util import cfg_from_workload, oracle_cfg, rel_err_rows, to_gpu_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,B,rank,m", [
    (16, 2, 1, 224, 9), (16, 2, 1, 204, 17), (14, 2, 2, 224, 40), (64, 8, 8, 204, 333), (56, 8, 8, 224, 610),
    (16, 2, 1, 200, 1030),
])
def test_rank_224_with_many_heads(hq, hkv, B, rank, m):
    L, window = m + 150, 8
    wl = W.CONFIGS["llama8b_32k"].scaled(name="r224", batch=B, n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rank=rank,
                                         r_true=48, N=L + 4, window=window, topk=m - window, n_needles=3)
    st = W.latent_state(wl, seed=m)
    c = cfg_from_workload(wl)
    g = to_gpu_state(c, st)
    idx = torch.empty((B, m), dtype=torch.int32, device="cuda")
    args = (g["q"], g["sink_k"], g["sink_v"], g["bases_k"], g["bases_v"], g["coef_k"], g["coef_v"], s4r.alloc_workspace(c))
    out = s4r.decode_step(c, L, *args, idx_out=idx)
    again = s4r.decode_step(c, L, *args)
    full = s4r.full_recon_decode(c, L, *args)
    torch.cuda.synchronize()
    assert torch.equal(out, again)
    theta = oracle_cfg(c)["rope_theta"]
    state = (st["sink_k"], st["sink_v"], st["bases_k"], st["bases_v"], st["coef_k"], st["coef_v"], L, hkv, theta)
    ref, _, _ = decode.sparse_attention(st["q"], idx.cpu().numpy().astype(np.int64), *state)
    # bf16 storage: the parity tests' output bound
    assert rel_err_rows(out.cpu().numpy(), ref) <= 2e-2
    assert rel_err_rows(full.cpu().numpy(), decode.full_reconstruction_decode(st["q"], *state)) <= 2e-2
