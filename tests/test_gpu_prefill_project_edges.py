"""The prompt's bulk projection at the edges of its row blocks (128 rows, tiles
of 16) and of its 64-dim steps (unrolled by three, the rest after the loop)."""

import numpy as np
import pytest
import torch

import paper_2608_00528_amd as s4r

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hkv,dh,nb,rank,n,B", [
    (1, 64, 1, 32, 1, 1), (2, 64, 1, 64, 16, 2), (3, 64, 1, 96, 127, 1), (4, 64, 1, 128, 129, 1),
    (5, 64, 1, 160, 17, 3), (4, 128, 2, 96, 255, 1), (6, 64, 1, 192, 128, 1), (8, 128, 1, 160, 300, 2),
    (7, 64, 1, 100, 1000, 1),
])
def test_projection_edges(hkv, dh, nb, rank, n, B):
    rng = np.random.default_rng(n + rank)
    Dp = hkv * dh
    cap = 16384                                                  # (a workspace that holds the transposed bases)
    c = s4r.make_config(batch=B, n_q_heads=hkv, n_kv_heads=hkv, head_dim=dh, rank=rank, basis_groups=nb, capacity=cap)
    rs = s4r.rank_stride(rank)
    bf = lambda *s: torch.from_numpy(rng.standard_normal(s)).to(torch.bfloat16)  # noqa: E731
    rows = [bf(B, n, Dp) for _ in range(2)]
    bases = [bf(B, nb, Dp // nb, rank) for _ in range(2)]
    coef = [torch.full((B, cap, nb * rs), 3.0, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    s4r.prefill_project(c, n, *[x.cuda() for x in rows], *[s4r.pad_latent(x, rank).cuda() for x in bases], *coef,
                        s4r.alloc_workspace(c))
    torch.cuda.synchronize()
    for x, basis, got in zip(rows, bases, coef):
        g = s4r.unpack_coef(c, cap, got).cpu().to(torch.float64).numpy().reshape(B, cap, nb, rs)
        a = x.to(torch.float64).numpy().reshape(B, n, nb, Dp // nb)
        w = basis.to(torch.float64).numpy()
        ref = np.einsum("bnkd,bkdr->bnkr", a, w)
        # fp32 sums of Dp / nb exact products, then one rounding to bf16
        bound = 2.0 ** -8 * np.abs(ref) + (Dp // nb) * 2.0 ** -24 * np.einsum("bnkd,bkdr->bnkr", np.abs(a), np.abs(w))
        assert np.all(np.abs(g[:, :n, :, :rank] - ref) <= bound)
        assert np.all(g[:, :n, :, rank:] == 0)                   # padding columns of a rank off 32
        assert np.all(g[:, n:] == 3.0)                           # rows past the prompt untouched


@pytest.mark.parametrize("hkv,dh,rank,n,B", [(8, 128, 192, 5, 2), (16, 64, 160, 16, 4), (4, 64, 96, 30, 1)])
def test_projection_in_the_queried_workspace(hkv, dh, rank, n, B):
    """A capacity so small that the transposed bases are the larger part of the
    workspace: what the size query says is enough, and its last byte is not passed."""
    rng = np.random.default_rng(n + rank)
    Dp, cap = hkv * dh, (n + 15) // 16 * 16
    c = s4r.make_config(batch=B, n_q_heads=hkv, n_kv_heads=hkv, head_dim=dh, rank=rank, capacity=cap)
    size = s4r.workspace_size(c)
    assert size >= 2 * B * Dp * rank * 2
    guarded = torch.full((size + 4096,), 7, dtype=torch.uint8, device="cuda")
    rows = [torch.from_numpy(rng.standard_normal((B, n, Dp))).to(torch.bfloat16) for _ in range(2)]
    bases = [torch.from_numpy(rng.standard_normal((B, 1, Dp, rank))).to(torch.bfloat16) for _ in range(2)]
    coef = [torch.zeros((B, cap, rank), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    s4r.prefill_project(c, n, *[x.cuda() for x in rows], *[x.cuda() for x in bases], *coef, guarded[:size])
    torch.cuda.synchronize()
    assert torch.all(guarded[size:] == 7)
    for x, basis, got in zip(rows, bases, coef):
        a, w = x.to(torch.float64).numpy(), basis[:, 0].to(torch.float64).numpy()
        g = s4r.unpack_coef(c, n, got).cpu().to(torch.float64).numpy()
        bound = 2.0 ** -8 * np.abs(a @ w) + Dp * 2.0 ** -24 * (np.abs(a) @ np.abs(w))
        assert np.all(np.abs(g - a @ w) <= bound)
