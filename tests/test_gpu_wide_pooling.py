"""Pooling windows wider than the shared-window form (9) at each chunk width of
the relevance kernel (256, 512 and 1024 positions) and past 16 query columns."""

import numpy as np
import pytest
import torch

import paper_2608_00528_amd as s4r
import workloads as W
from oracle import decode
from tests.gpu_util import cfg_from_workload, to_gpu_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,wq,kappa,mode,agg", [
    (1, 1, 11, "max", "mean"), (2, 32, 65, "avg", "mean"), (32, 1, 9, "max", "mean"), (32, 1, 11, "avg", "max"),
    (64, 1, 11, "max", "max"), (64, 2, 65, "avg", "mean"),
])
def test_wide_pooling(batch, wq, kappa, mode, agg):
    # two groups: 1024 workgroups of 1024 positions at batch 64, of 512 at batch 32
    L = 16387
    wl = W.CONFIGS["llama8b_32k"].scaled(name="pool", batch=batch, n_q_heads=4, n_kv_heads=2, head_dim=64, rank=32,
                                         r_true=24, N=L + 4, window=8, topk=300, q_window=wq, pool_kernel=kappa,
                                         pool_mode=mode, group_agg=agg)
    st = W.latent_state(wl, seed=kappa)
    c = cfg_from_workload(wl)
    g = to_gpu_state(c, st)
    idx = torch.empty((batch, s4r.num_selected(c, L)), dtype=torch.int32, device="cuda")
    scores = torch.empty((batch, L), dtype=torch.float32, device="cuda")
    s4r.decode_step(c, L, g["q"], g["sink_k"], g["sink_v"], g["bases_k"], g["bases_v"], g["coef_k"], g["coef_v"],
                    s4r.alloc_workspace(c), qwin_prev=g.get("qwin_prev"), idx_out=idx, scores_out=scores)
    torch.cuda.synchronize()
    a = decode.relevance(st["q"], st["qwin_prev"], st["bases_k"], st["coef_k"], L, c.n_kv_heads, kappa, mode,
                         agg)["a_tilde"]
    got = scores.cpu().numpy().astype(np.float64)
    # fp32 probabilities of a few ulp each, sums in fp64: the scores' bound of the parity tests
    assert (np.abs(got - a) / np.maximum(np.abs(a), 1e-30)).max() <= 5e-6
    assert np.array_equal(idx.cpu().numpy(), decode.select(got, L, wl.window, wl.topk))
