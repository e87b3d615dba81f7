"""Selection at the edges of its kernels: one workgroup with 4, 8, 16 or 32
keys per thread, chunks of 2048 positions beyond; ties at every level."""

import numpy as np
import pytest
import torch

import paper_2608_00528_amd as s4r
import workloads as W
from oracle import decode
from tests.gpu_util import cfg_from_workload, dev, to_gpu_state

pytestmark = pytest.mark.gpu

SIZES = [1, 63, 65, 2048, 4096, 4097, 8193, 16384, 16385, 32768, 32769, 70001]


def _scores(kind, n, rng):
    if kind == "spread":                       # ten decades: a few members per bin
        return np.exp(rng.uniform(-20, 0, n))
    if kind == "levels":                       # plateaus of exact ties over several sub-bins
        return rng.integers(0, 7, n) / 7.0
    if kind == "equal":
        return np.full(n, 0.25)
    if kind == "low_bits":                     # one sub-bin, told apart by the last key bits, many ties
        return 1.0 + rng.integers(0, 300, n) * 2.0 ** -23
    return np.zeros(n)                         # the lowest key


@pytest.mark.parametrize("kind", ["spread", "levels", "equal", "low_bits", "zero"])
def test_select_sizes(kind):
    rng = np.random.default_rng(5)
    for n in SIZES:
        for k in {1, min(n, 700), max(1, n // 3), n}:
            window, B = (5 if n % 2 else 0), 2
            L = n + window
            c = s4r.make_config(batch=B, n_q_heads=2, n_kv_heads=1, head_dim=64, rank=32,
                                capacity=(L + 15) // 16 * 16, window=window, topk=k)
            sc = np.stack([_scores(kind, L, rng) for _ in range(B)]).astype(np.float32)
            idx = s4r.select_topk(c, L, dev(sc, torch.float32), s4r.alloc_workspace(c))
            ref = decode.select(sc.astype(np.float64), L, window, k)
            assert np.array_equal(idx.cpu().numpy(), ref), f"{kind}: n = {n}, k = {k}"


@pytest.mark.parametrize("n_hist", [4095, 4097, 8192, 16384, 16385, 33000])
def test_fused_selection_sizes(n_hist):
    wl = W.CONFIGS["llama8b_32k"].scaled(name="sel", batch=2, n_q_heads=8, n_kv_heads=2, head_dim=64, rank=32, r_true=24,
                                         N=n_hist + 8 + 4, window=8, topk=n_hist // 10)
    st = W.latent_state(wl, seed=n_hist)
    c = cfg_from_workload(wl)
    g = to_gpu_state(c, st)
    idx = torch.empty((2, s4r.num_selected(c, wl.L)), dtype=torch.int32, device="cuda")
    scores = torch.empty((2, wl.L), dtype=torch.float32, device="cuda")
    s4r.decode_step(c, wl.L, g["q"], g["sink_k"], g["sink_v"], g["bases_k"], g["bases_v"], g["coef_k"], g["coef_v"],
                    s4r.alloc_workspace(c), idx_out=idx, scores_out=scores)
    ref = decode.select(scores.cpu().numpy().astype(np.float64), wl.L, wl.window, wl.topk)
    assert np.array_equal(idx.cpu().numpy(), ref)
