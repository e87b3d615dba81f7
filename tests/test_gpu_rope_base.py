"""RoPE bases over the whole accepted range: off (0), below 1 (angles of more than
a revolution per position at the highest pairs), 1, and large."""

import numpy as np
import pytest
import torch

import paper_2608_00528_amd as s4r
import workloads as W
from oracle import decode
from tests.gpu_util import cfg_from_workload, dev, oracle_cfg, rel_err_rows, to_gpu_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("theta", [0.0, 0.01, 0.1, 0.3, 1.0, 5e6])
@pytest.mark.parametrize("dtype,dh", [("bf16", 128), ("bf16", 64), ("fp32", 128), ("fp32", 64)])
def test_rope_base(theta, dtype, dh):
    L = 900
    wl = W.CONFIGS["llama8b_32k"].scaled(name="theta", batch=2, n_q_heads=8, n_kv_heads=2, head_dim=dh, rank=32,
                                         r_true=24, N=L + 4, window=8, topk=200, rope_theta=theta, dtype=dtype,
                                         n_needles=3)
    st = W.latent_state(wl, seed=4)
    c = cfg_from_workload(wl)
    g = to_gpu_state(c, st)
    ws = s4r.alloc_workspace(c)
    m = s4r.num_selected(c, L)
    idx = torch.empty((2, m), dtype=torch.int32, device="cuda")
    out = s4r.decode_step(c, L, g["q"], g["sink_k"], g["sink_v"], g["bases_k"], g["bases_v"], g["coef_k"], g["coef_v"],
                          ws, idx_out=idx)
    torch.cuda.synchronize()
    idx_np = idx.cpu().numpy().astype(np.int64)
    th = oracle_cfg(c)["rope_theta"]
    args = (st["q"], idx_np, st["sink_k"], st["sink_v"], st["bases_k"], st["bases_v"], st["coef_k"], st["coef_v"], L,
            wl.n_kv_heads, th)
    ref, _, _ = decode.sparse_attention(*args)
    # the parity tests' output bounds per storage type
    assert rel_err_rows(out.cpu().numpy(), ref) <= (2e-2 if dtype == "bf16" else 1e-4)
    # attention over given rows: fp32 throughout
    rows = [dev(np.stack([x[b][idx_np[b]] @ B_[b, 0].T for b in range(2)]), torch.float32)
            for x, B_ in ((st["coef_k"], st["bases_k"]), (st["coef_v"], st["bases_v"]))]
    out = s4r.sparse_attn(c, L, g["q"], g["sink_k"], g["sink_v"], idx, *rows, ws)
    torch.cuda.synchronize()
    assert rel_err_rows(out.cpu().numpy(), ref) <= 1e-4
