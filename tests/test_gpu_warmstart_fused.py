"""The fused passes of the warm-start network at the sizes where their tiles, remainders and
dispatch rules can go wrong: the forward pass against the per-layer products (bit for bit), a
training step against the FP64 gradients, the features against the descriptors."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


def bf16(a):
    """Round to the nearest bf16 (ties to even), as float64."""
    u = np.ascontiguousarray(a, dtype=np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000
    return u.astype(np.uint32).view(np.float32).astype(np.float64)


def _rounded_step(p, X, T, mask):
    """Loss and gradients in FP64 with the tensors that the library keeps in bf16 rounded."""
    B = X.shape[0]
    A1 = bf16(np.maximum(X @ p["W1"] + p["b1"], 0))
    A2 = bf16(np.maximum(A1 @ p["W2"] + p["b2"], 0))
    Z = A2 @ p["W3"] + p["b3"]
    loss = mlp.loss(Z, T, mask)
    P = mlp.masked_softmax(Z, mask)
    d3 = bf16(mask * (P * (T * mask).sum(1, keepdims=True) - T) / B)
    d2 = bf16((d3 @ p["W3"].T) * (A2 > 0))
    d1 = bf16((d2 @ p["W2"].T) * (A1 > 0))
    return loss, {"W1": X.T @ d1, "b1": d1.sum(0), "W2": A1.T @ d2, "b2": d2.sum(0),
                  "W3": A2.T @ d3, "b3": d3.sum(0)}


def _flat(p):
    return np.concatenate([np.asarray(p[k], np.float32).ravel() for k in mlp.PARAMS])


def _net(F, H, A, batch, params):
    from paper_2408_14778_amd.warmstart import WarmStartNet
    net = WarmStartNet(F, H, A, max_batch=batch)
    net.set_params(_flat(params))
    return net


def _params(F, H, A, seed):
    rng = np.random.default_rng(seed)
    p = mlp.init(F, H, A, seed=seed)
    for k in ("b1", "b2", "b3"):
        p[k] = rng.standard_normal(p[k].shape) * 0.1
    return {k: bf16(v) for k, v in p.items()}


# rows: one, around a 32- and a 64-row tile, around the switches to 64 rows (16,384) and to
# 128 rows (32,768, at most 4 slots) per workgroup; H = 64 with more inputs than hidden units
@pytest.mark.parametrize("F,H,A,rows", [
    (96, 256, 4, 1), (96, 256, 4, 31), (96, 256, 4, 33), (96, 256, 3, 16383), (96, 256, 4, 16385),
    (96, 256, 4, 32767), (96, 256, 4, 32769), (16, 256, 8, 32800), (128, 128, 1, 65),
    (112, 64, 4, 63), (96, 64, 8, 129)])
def test_forward_rows(F, H, A, rows):
    import torch
    net = _net(F, H, A, rows, _params(F, H, A, F + H))
    x = np.random.default_rng(rows).standard_normal((rows, F)).astype(np.float32)
    x = torch.from_numpy(x).to("cuda").to(torch.bfloat16)
    # a prefix of 4,096 rows per call of the per-layer path: its activations fit its device array
    out = torch.empty((rows, A), dtype=torch.float32, device="cuda")
    for s in range(0, rows, 4096):
        net.forward_noalloc(x[s:s + 4096], out[s:s + 4096])
    got = net.forward(x)
    assert torch.isfinite(got).all()
    assert torch.equal(got, out)


# rows: the smallest fused step, one below it (the per-layer path), a ragged tile, a split of the
# reductions with a remainder, the switch to 64 rows per workgroup
@pytest.mark.parametrize("F,H,A,rows", [
    (96, 256, 4, 63), (96, 256, 4, 64), (48, 128, 4, 129), (96, 256, 4, 545), (64, 64, 8, 700),
    (128, 128, 3, 2049), (96, 256, 4, 16400)])
def test_training_step(F, H, A, rows):
    """Loss and gradients against FP64 with the same tensors rounded: what is left is FP32
    accumulation (1e-4 relative for these lengths) and values that it moves over a bf16 rounding
    boundary (2^-8 of single terms), so 1e-2 of each array's largest entry. The update: Adam's
    first step, and the weights in every layout that the passes read."""
    import torch
    rng = np.random.default_rng(rows)
    p = _params(F, H, A, 3)
    X = bf16(rng.standard_normal((rows, F)))
    mask = (rng.random((rows, A)) < 0.8).astype(np.float64)
    mask[:, 0] = 1.0
    T = rng.random((rows, A)) * mask
    T /= T.sum(axis=1, keepdims=True)
    net = _net(F, H, A, rows, p)
    x = torch.from_numpy(X.astype(np.float32)).to("cuda").to(torch.bfloat16)
    loss = net.train_step(x, torch.from_numpy(T.astype(np.float32)).to("cuda"),
                          torch.from_numpy(mask.astype(np.float32)).to("cuda"), lr=1e-3)
    g = net.grads()
    ref_loss, ref = _rounded_step(p, X, T, mask)
    assert abs(loss - ref_loss) <= 1e-3 * abs(ref_loss)
    at = 0
    for k in mlp.PARAMS:
        n = ref[k].size
        rel = np.abs(g[at:at + n] - ref[k].ravel()).max() / np.abs(ref[k]).max()
        assert rel < 1e-2, (k, rel)
        at += n
    # Adam's first step moves every weight by lr times the gradient's sign (up to eps)
    step = _flat(p) - net.params()
    moved = np.abs(g) > 1e-6
    np.testing.assert_allclose(step[moved], 1e-3 * np.sign(g[moved]), rtol=0.02, atol=1e-6)
    # and the copies that the passes read are those of the new weights
    from paper_2408_14778_amd.warmstart import WarmStartNet
    fresh = WarmStartNet(F, H, A, max_batch=rows)
    fresh.set_params(net.params())
    assert torch.equal(net.forward(x), fresh.forward(x))
    n = min(rows, 4096)
    a, b = (torch.empty((n, A), dtype=torch.float32, device="cuda") for _ in range(2))
    net.forward_noalloc(x[:n], a)
    fresh.forward_noalloc(x[:n], b)
    assert torch.equal(a, b)
    # the backward pass too: a second step (moments differ, gradients do not depend on them)
    t2 = torch.from_numpy(T.astype(np.float32)).to("cuda")
    m2 = torch.from_numpy(mask.astype(np.float32)).to("cuda")
    net.train_step(x, t2, m2, lr=0.0)
    fresh.train_step(x, t2, m2, lr=0.0)
    assert np.array_equal(net.grads(), fresh.grads())


@pytest.mark.parametrize("n,F,skew", [(1, 96, 0), (63, 96, 0), (65, 96, 0), (200, 81, 0),
                                      (130, 88, 0), (70, 100, 0), (64, 40, 0), (77, 96, 1)])
def test_features(n, F, skew):
    """Every feature of include/cfr_warmstart.h's descriptor, widths below, at and above the 81
    meaningful ones, and a descriptor array that is not 16-byte aligned (skew)."""
    import torch

    from paper_2408_14778_amd import warmstart
    rng = np.random.default_rng(n)
    d = np.zeros((n, 16), dtype=np.int16)
    d[:, 0] = rng.integers(1, 3, n)
    d[:, 1] = rng.integers(0, 13, n)
    d[:, 2] = rng.integers(0, 4, n)          # 3 is out of the one-hot's range
    d[:, 3:6] = rng.integers(-1, 13, (n, 3))
    d[:, 6] = rng.integers(0, 6, n)
    d[:, 7] = rng.integers(0, 6, n)
    d[:, 8:10] = rng.integers(0, 60, (n, 2))
    d[:, 10] = rng.integers(2, 400, n)
    d[:, 11] = rng.integers(1, 16, n)
    d[:, 12] = rng.integers(0, 16, n)
    d[:, 13] = rng.integers(1, 4, n)
    d[:, 14] = rng.integers(4, 14, n)
    d[:, 15] = rng.integers(0, 5, n)
    bel = rng.dirichlet(np.ones(13), (5, 2)).astype(np.float32)
    f = np.zeros((n, 81))
    for i, r in enumerate(d.astype(np.int64)):
        def hot(base, width, c):
            if 0 <= c < width:
                f[i, base + c] = 1.0
        hot(0, 13, r[1]); hot(13, 2, r[0] - 1); hot(15, 3, r[2])
        for c in r[3:6]:
            hot(18, 13, c)
        hot(31, 4, r[6]); hot(35, 5, r[7])
        me, op, st = float(r[8]), float(r[9]), float(r[10])
        f[i, 40:44] = me / st, op / st, (me + op) / st, (op - me) / max(me + op, 1.0)
        f[i, 44:48] = [(r[11] >> s) & 1 for s in range(4)]
        f[i, 48:52] = r[12] / 16.0, r[13] / 3.0, np.log(st) / np.log(1000.0), r[14] / 13.0
        bo, bm = bel[r[15], 2 - r[0]], bel[r[15], r[0] - 1]
        f[i, 52:65], f[i, 65:78] = bo, bm
        f[i, 78], f[i, 79], f[i, 80] = bo[:r[1]].sum(), bo[r[1] + 1:].sum(), 1.0
    ref = np.zeros((n, F))
    ref[:, :min(F, 81)] = f[:, :F]
    buf = torch.zeros(n * 16 + skew, dtype=torch.int16, device="cuda")
    buf[skew:] = torch.from_numpy(d.ravel()).to("cuda")
    got = warmstart.features(buf[skew:].view(n, 16), torch.from_numpy(bel).to("cuda"), F)
    # one rounding to bf16 (2^-9) of values computed in fp32
    np.testing.assert_allclose(got.float().cpu().numpy(), ref, rtol=2.0 ** -8, atol=1e-6)
