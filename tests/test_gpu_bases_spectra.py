"""Basis construction over the widths its kernels are built for and the spectra
where an eigensolver can go wrong: flat, low rank with zeros wanted, repeated
eigenvalues, a matrix that splits, and input that is not finite."""

import numpy as np
import pytest
import torch

import paper_2608_00528_amd as s4r

pytestmark = pytest.mark.gpu


def _rows(kind, n, Dp, rng):
    if kind == "decaying":
        return rng.standard_normal((n, 48)) @ rng.standard_normal((48, Dp)) + 0.05 * rng.standard_normal((n, Dp))
    if kind == "white":
        return rng.standard_normal((n, Dp))
    if kind == "low_rank":                     # exact in bf16: eigenvalue 9 on is zero
        return rng.integers(-2, 3, (n, 8)) @ rng.integers(-1, 2, (8, Dp))
    if kind == "repeated":                     # unit vectors, each the same number of times
        return np.eye(Dp)[np.arange(n) % Dp]
    return np.zeros((n, Dp))                   # "zero"


@pytest.mark.parametrize("kind,hkv,nb,rank,rank_v,n,center", [
    ("decaying", 2, 1, 32, 0, 300, False), ("decaying", 4, 1, 96, 160, 700, True), ("decaying", 6, 1, 192, 0, 800, False),
    ("white", 8, 1, 160, 0, 2000, False), ("white", 8, 2, 100, 0, 600, True), ("decaying", 10, 1, 64, 0, 600, False),
    ("white", 16, 1, 256, 0, 900, False), ("low_rank", 4, 1, 40, 0, 500, False), ("repeated", 2, 1, 64, 0, 768, False),
    ("zero", 2, 1, 32, 0, 300, False),
])
def test_bases_spectra(kind, hkv, nb, rank, rank_v, n, center):
    rng = np.random.default_rng(n + rank)
    dh, eta, B = 128, 1.0, 1
    Dp = hkv * dh
    c = s4r.make_config(batch=B, n_q_heads=hkv, n_kv_heads=hkv, head_dim=dh, rank=rank, rank_v=rank_v, basis_groups=nb,
                        capacity=(n + 15) // 16 * 16)
    S = [torch.from_numpy(_rows(kind, n, Dp, rng)).to(torch.bfloat16)[None] for _ in range(2)]
    got = s4r.prefill_bases(c, n, *[x.cuda() for x in S], eta=eta, center=center)
    again = s4r.prefill_bases(c, n, *[x.cuda() for x in S], eta=eta, center=center)
    torch.cuda.synchronize()
    dg = Dp // nb
    for x, basis, rep, r in zip(S, got, again, (rank, rank_v or rank)):
        assert torch.equal(basis, rep)
        Q_all = basis[0].cpu().to(torch.float64).numpy()
        assert np.all(Q_all[:, :, r:] == 0)                      # padding columns
        for g in range(nb):
            X = x[0, :, g * dg:(g + 1) * dg].to(torch.float64).numpy()
            norm = np.linalg.norm(X, axis=1, keepdims=True)
            X = X / np.where(norm > 0, norm, 1.0)
            if center:
                X = X - X.mean(axis=0)
            w = np.linalg.eigvalsh(X.T @ X)[::-1]
            Q = Q_all[g, :, :r]
            # bf16 rounding of the entries: 2^-9 relative each
            assert np.abs(Q.T @ Q - np.eye(r)).max() <= 1e-2
            V, _ = np.linalg.qr(Q)
            captured = np.linalg.norm(X @ V) ** 2
            assert captured >= (1 - 1e-4) * w[:r].sum() - 1e-9
            # each column's own energy: largest first, within the rounding
            own = ((X @ Q) ** 2).sum(axis=0)
            assert np.all(np.abs(own - w[:r]) <= 1e-2 * w[:r] + 2e-5 * w[0])


def test_bases_of_input_that_is_not_finite():
    rng = np.random.default_rng(3)
    n, Dp, rank = 400, 256, 32
    c = s4r.make_config(batch=2, n_q_heads=2, n_kv_heads=2, head_dim=128, rank=rank, capacity=400)
    S = [torch.from_numpy(rng.standard_normal((2, n, Dp))).to(torch.bfloat16) for _ in range(2)]
    S[0][1, n - 1, 7] = float("nan")                             # a sampled row of the second sequence's keys
    bk, bv = s4r.prefill_bases(c, n, *[x.cuda() for x in S], eta=1.0)
    torch.cuda.synchronize()
    assert torch.isnan(bk[1]).all()
    assert torch.isfinite(bk[0]).all() and torch.isfinite(bv).all()


def _degenerate(kind, n, Dp, k, rng):
    if kind == "orthogonal":                   # k mutually orthogonal +-1 rows, each repeated: k equal eigenvalues
        H = np.ones((1, 1))
        while len(H) < Dp:
            H = np.block([[H, H], [H, -H]])
        pick = H[rng.permutation(Dp)[:k]][:, rng.permutation(Dp)] * rng.choice([-1, 1], (1, Dp))
        return pick[np.arange(n) % k]
    if kind == "few":                          # k distinct rows: zeros from eigenvalue k + 1 on
        return rng.standard_normal((k, Dp))[np.arange(n) % k]
    if kind == "blocks":                       # k copies of one block on the diagonal: multiplicity k
        b, m = Dp // k, n // k
        X, src = np.zeros((n, Dp)), rng.standard_normal((m, b))
        for i in range(k):
            X[i * m:(i + 1) * m, i * b:(i + 1) * b] = src
        return X
    return np.full((n, Dp), 1.5)               # "constant"


@pytest.mark.parametrize("kind,hkv,rank,n,k", [
    ("orthogonal", 2, 16, 288, 16), ("orthogonal", 2, 64, 320, 64), ("orthogonal", 2, 160, 320, 160),
    ("orthogonal", 2, 256, 512, 256), ("orthogonal", 4, 160, 480, 160), ("orthogonal", 4, 256, 768, 256),
    ("orthogonal", 8, 128, 384, 128), ("orthogonal", 8, 256, 512, 256), ("orthogonal", 16, 160, 480, 160),
    ("few", 2, 256, 300, 1), ("few", 4, 64, 300, 2), ("few", 4, 256, 300, 3), ("few", 8, 160, 300, 5),
    ("few", 8, 256, 300, 3), ("few", 16, 192, 300, 1), ("blocks", 2, 96, 512, 4), ("blocks", 8, 160, 1024, 2),
    ("blocks", 8, 256, 1024, 8), ("constant", 4, 64, 300, 1), ("constant", 8, 256, 300, 1),
])
def test_bases_of_coinciding_eigenvalues(kind, hkv, rank, n, k):
    """Wanted eigenvalues that are equal: whichever vectors of their space come
    out, they are orthonormal and hold its energy."""
    dh, draws = 128, 3
    Dp = hkv * dh
    c = s4r.make_config(batch=draws, n_q_heads=hkv, n_kv_heads=hkv, head_dim=dh, rank=rank, capacity=(n + 15) // 16 * 16)
    rng = np.random.default_rng(n + rank + k)
    S = [torch.from_numpy(np.stack([_degenerate(kind, n, Dp, k, rng) for _ in range(draws)])).to(torch.bfloat16)
         for _ in range(2)]
    got = s4r.prefill_bases(c, n, *[x.cuda() for x in S], eta=1.0)
    again = s4r.prefill_bases(c, n, *[x.cuda() for x in S], eta=1.0)
    torch.cuda.synchronize()
    for x, basis, rep in zip(S, got, again):
        assert torch.equal(basis, rep)
        for b in range(draws):
            X = x[b].to(torch.float64).numpy()
            X = X / np.linalg.norm(X, axis=1, keepdims=True)
            w = np.linalg.eigvalsh(X.T @ X)[::-1]
            Q = basis[b, 0, :, :rank].cpu().to(torch.float64).numpy()
            # bf16 rounding of the entries, 2^-9 relative each: the bounds of the spectra above
            off = np.abs(Q.T @ Q - np.eye(rank)).max()
            assert off <= 1e-2, f"{kind} {Dp} rank {rank}: orthonormal to {off:.1e}"
            own = ((X @ Q) ** 2).sum(axis=0)
            assert np.all(np.abs(own - w[:rank]) <= 1e-2 * w[:rank] + 2e-5 * w[0])
