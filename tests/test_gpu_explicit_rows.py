"""The separately callable reconstruction and attention over given rows, at the
edges of their row splits, chunks of 32 rows, tiles of 16 and head groups."""

import numpy as np
import pytest
import torch

import paper_2608_00528_amd as s4r
from oracle import decode
from tests.gpu_util import dev, rel_err_rows

pytestmark = pytest.mark.gpu


def _draw(hq, hkv, dh, rank, nb, n_sink, m, L, B, dtype, seed):
    rng = np.random.default_rng(seed)
    c = s4r.make_config(batch=B, n_q_heads=hq, n_kv_heads=hkv, head_dim=dh, rank=rank, basis_groups=nb,
                        capacity=(L + 15) // 16 * 16, n_sink=n_sink, window=8, topk=max(m, 8) - 8,
                        rope_theta=10000.0, dtype=dtype)
    Dp, dt = hkv * dh, s4r.storage_dtype(c)
    idx = np.stack([np.sort(rng.permutation(L)[:m]) for _ in range(B)]).reshape(B, m)
    rnd = lambda *s: torch.from_numpy(rng.standard_normal(s)).to(dt)  # noqa: E731
    return c, idx, rnd(B, hq, dh), rnd(B, n_sink, Dp), rnd(B, n_sink, Dp), rng


@pytest.mark.parametrize("hq,hkv,dh,n_sink,m,B,dtype", [
    (8, 2, 64, 4, 1, 1, "fp32"), (4, 4, 128, 0, 8, 2, "bf16"), (16, 8, 128, 4, 33, 1, "bf16"),
    (28, 4, 128, 4, 64, 1, "bf16"), (32, 8, 128, 4, 513, 1, "fp32"), (32, 4, 64, 2, 1000, 3, "bf16"),
    (16, 1, 128, 0, 2500, 1, "bf16"), (32, 8, 128, 4, 0, 1, "bf16"),
])
def test_attention_over_rows(hq, hkv, dh, n_sink, m, B, dtype):
    L = max(m, 64) * 2 + 3
    c, idx, q, sk, sv, rng = _draw(hq, hkv, dh, 32, 1, n_sink, m, L, B, dtype, 100 + m)
    Dp = hkv * dh
    kh, vh = (rng.standard_normal((B, m, Dp)).astype(np.float32) for _ in range(2))
    f64 = lambda x: x.to(torch.float64).numpy()  # noqa: E731
    pos = np.concatenate([np.broadcast_to(np.arange(n_sink), (B, n_sink)), n_sink + idx], axis=1)
    ref = decode.attend(f64(q), np.concatenate([f64(sk), kh], axis=1), np.concatenate([f64(sv), vh], axis=1), pos,
                        np.full(B, n_sink + L - 1), 10000.0, hkv)
    ws = s4r.alloc_workspace(c)
    g = lambda x: None if x.numel() == 0 else x.cuda()  # noqa: E731
    args = (g(q), g(sk), g(sv), dev(idx.astype(np.int32), torch.int32), dev(kh, torch.float32), dev(vh, torch.float32))
    out = s4r.sparse_attn(c, L, *args, ws)
    again = s4r.sparse_attn(c, L, *args, ws)
    torch.cuda.synchronize()
    # fp32 logits of a few units over 128 products and a softmax of m terms: some 1e-6
    err = rel_err_rows(out.cpu().numpy(), ref)
    print(f"[rows] {hq}/{hkv} d{dh} m={m} {dtype}: err {err:.2e}", flush=True)
    assert err < 3e-5
    assert torch.equal(out, again)


@pytest.mark.parametrize("hq,hkv,dh,rank,nb,m,B,dtype", [
    (8, 2, 64, 32, 2, 5, 1, "fp32"), (8, 8, 128, 160, 1, 16, 2, "bf16"), (32, 8, 128, 204, 1, 17, 1, "bf16"),
    (4, 4, 128, 192, 1, 100, 1, "fp32"), (16, 4, 64, 96, 2, 301, 2, "bf16"),
])
def test_reconstruction(hq, hkv, dh, rank, nb, m, B, dtype):
    L = 2 * m + 40
    c, idx, _, _, _, rng = _draw(hq, hkv, dh, rank, nb, 0, m, L, B, dtype, 7 * m)
    dt, Dp = s4r.storage_dtype(c), hkv * dh
    rnd = lambda *s: torch.from_numpy(rng.standard_normal(s)).to(dt)  # noqa: E731
    bases = [rnd(B, nb, Dp // nb, rank) for _ in range(2)]
    coefs = [rnd(B, c.capacity, nb * rank) for _ in range(2)]
    pad = lambda x: s4r.pad_latent(x, rank, nb if x.shape[-1] == nb * rank else 1)  # noqa: E731
    got = s4r.reconstruct(c, L, dev(idx.astype(np.int32), torch.int32),
                          *[s4r.pad_latent(x, rank).cuda() for x in bases],
                          *[s4r.pack_coef(c, c.capacity, pad(x).cuda()) for x in coefs])
    torch.cuda.synchronize()
    for out, basis, coef in zip(got, bases, coefs):
        rows = np.stack([coef[b].to(torch.float64).numpy()[idx[b]] for b in range(B)])
        ref = decode.reconstruct(rows, basis.to(torch.float64).numpy())
        # up to 224 products of unit normals in fp32: some 1e-6 of a row's largest value
        assert rel_err_rows(out.cpu().numpy(), ref) < 1e-5


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("sinks,rows", [(True, False), (False, True), (True, True)])
def test_logits_of_minus_infinity(dtype, sinks, rows):
    """Keys whose logits overflow to -inf weigh nothing, whether they are all the
    sinks or all rows of a split; NaN when no key is left."""
    hq, hkv, dh, n_sink, m = 4, 2, 64, 3, 40
    c, idx, q, sk, sv, rng = _draw(hq, hkv, dh, 32, 1, n_sink, m, 100, 1, dtype, 5)
    c.rope_theta = 0.0                         # no rotation: the first dim alone decides
    q[..., 0] = 100.0
    kh, vh = (rng.standard_normal((1, m, hkv * dh)).astype(np.float32) for _ in range(2))
    lost_s = np.full(n_sink, sinks)
    lost_r = np.full(m, rows)
    if not sinks:
        lost_r[:8] = False                     # one split keeps its rows
    sk.view(1, n_sink, hkv, dh)[:, lost_s, :, 0] = -3e38
    kh.reshape(1, m, hkv, dh)[:, lost_r, :, 0] = -3e38
    out = s4r.sparse_attn(c, 100, q.cuda(), sk.cuda(), sv.cuda(), dev(idx.astype(np.int32), torch.int32),
                          dev(kh, torch.float32), dev(vh, torch.float32), s4r.alloc_workspace(c)).cpu().numpy()
    if sinks and rows:
        assert np.isnan(out).all()
        return
    f64 = lambda x: x.to(torch.float64).numpy()  # noqa: E731
    keys = np.concatenate([f64(sk)[:, ~lost_s], kh[:, ~lost_r]], axis=1)
    vals = np.concatenate([f64(sv)[:, ~lost_s], vh[:, ~lost_r]], axis=1)
    ref = decode.attend(f64(q), keys, vals, np.zeros((1, keys.shape[1])), np.zeros(1), 0.0, hkv)
    # logits up to about 40, whose fp32 rounding of 4e-6 goes through the exponential
    assert rel_err_rows(out, ref) < 1e-4


@pytest.mark.parametrize("hkv,dh,rank,m,B,dtype", [
    # four, two and one tile of 16 rows per workgroup, rows left over in each
    (8, 128, 160, 1025, 1, "bf16"), (8, 128, 32, 1023, 1, "bf16"), (4, 64, 224, 1000, 1, "bf16"),
    (16, 64, 96, 530, 2, "bf16"), (8, 128, 96, 2049, 1, "fp32"), (8, 128, 128, 515, 1, "fp32"),
    (8, 64, 192, 257, 3, "fp32"), (4, 128, 256, 700, 2, "fp32"), (2, 64, 64, 65, 1, "fp32"),
])
def test_reconstruction_tiles_per_workgroup(hkv, dh, rank, m, B, dtype):
    L = 2 * m + 40
    c, idx, _, _, _, rng = _draw(hkv, hkv, dh, rank, 1, 0, m, L, B, dtype, m)
    dt, Dp = s4r.storage_dtype(c), hkv * dh
    rnd = lambda *s: torch.from_numpy(rng.standard_normal(s)).to(dt)  # noqa: E731
    bases, coefs = [rnd(B, 1, Dp, rank) for _ in range(2)], [rnd(B, c.capacity, rank) for _ in range(2)]
    idx[:, 7] = [-1, L, L + 5][:B]                               # out of range: a NaN row, nothing else
    guard = [torch.full((B * m * Dp + 512,), 3.0, device="cuda") for _ in range(2)]
    s4r.reconstruct(c, L, dev(idx.astype(np.int32), torch.int32), *[x.cuda() for x in bases],
                    *[s4r.pack_coef(c, c.capacity, x.cuda()) for x in coefs],
                    *[x[:B * m * Dp].view(B, m, Dp) for x in guard])
    torch.cuda.synchronize()
    keep = np.arange(m) != 7
    for out, basis, coef in zip(guard, bases, coefs):
        assert torch.all(out[B * m * Dp:] == 3.0)
        got = out[:B * m * Dp].view(B, m, Dp).cpu().numpy()
        assert np.isnan(got[:, 7]).all()
        rows = np.stack([coef[b].to(torch.float64).numpy()[idx[b][keep]] for b in range(B)])
        # up to 256 products of unit normals in fp32: some 1e-6 of a row's largest value
        assert rel_err_rows(got[:, keep], decode.reconstruct(rows, basis.to(torch.float64).numpy())) < 1e-5
