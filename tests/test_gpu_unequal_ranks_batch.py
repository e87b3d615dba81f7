"""Unequal key and value ranks where a batch's selected tokens need more than one
round of the chip's workgroups (they have no second kernel to fall back on)."""

import numpy as np
import pytest
import torch

import paper_2608_00528_amd as s4r
import workloads as W
from oracle import decode
from tests.gpu_util import cfg_from_workload, check_selection, oracle_cfg, rel_err_rows, to_gpu_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,rank,rank_v,m", [
    (16, 96, 160, 1536), (16, 96, 160, 1537), (16, 128, 192, 2075), (32, 64, 192, 1600),
])
def test_more_than_one_round(hq, rank, rank_v, m):
    # 16 sequences x 16 KV heads = 256 pairs: three splits of 32 tiles (1536 tokens) are one round
    B, window = 16, 8
    L = m + 300
    wl = W.CONFIGS["llama8b_32k"].scaled(name="rounds", batch=B, n_q_heads=hq, n_kv_heads=16, head_dim=64, rank=rank,
                                         rank_v=rank_v, r_true=48, N=L + 4, window=window, topk=m - window,
                                         n_needles=3)
    st = W.latent_state(wl, seed=m)
    c = cfg_from_workload(wl)
    g = to_gpu_state(c, st)
    idx = torch.empty((B, m), dtype=torch.int32, device="cuda")
    out = s4r.decode_step(c, L, g["q"], g["sink_k"], g["sink_v"], g["bases_k"], g["bases_v"], g["coef_k"], g["coef_v"],
                          s4r.alloc_workspace(c), idx_out=idx)
    torch.cuda.synchronize()
    oc = oracle_cfg(c, wl.pool_mode, wl.group_agg)
    a = decode.relevance(st["q"], None, st["bases_k"], st["coef_k"], L, c.n_kv_heads, wl.pool_kernel, wl.pool_mode,
                         wl.group_agg)["a_tilde"]
    idx_np = idx.cpu().numpy().astype(np.int64)
    check_selection(idx_np, decode.select(a, L, window, wl.topk), a, L, window, wl.topk)
    ref, _, _ = decode.sparse_attention(st["q"], idx_np, st["sink_k"], st["sink_v"], st["bases_k"], st["bases_v"],
                                        st["coef_k"], st["coef_v"], L, c.n_kv_heads, oc["rope_theta"])
    # bf16 storage: the parity tests' output bound
    assert rel_err_rows(out.cpu().numpy(), ref) <= 2e-2
