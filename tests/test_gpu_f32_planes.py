"""The float32 passes on bfloat16 planes: operands are split into three
bfloat16 values and six plane products formed, so their error must stay that of
float32 arithmetic, whatever the magnitudes of the operands."""
import numpy as np
import pytest
import torch

from oracle import mra_oracle as O
from paper_2207_10284_amd import inputs
from tests.parity import dev, host

U = 2.0 ** -24


def _bf16_round(x):
    """float32 -> nearest bfloat16 (ties to even) as float32."""
    u = x.view(np.uint32).astype(np.uint64)
    r = (u + 0x7FFF + ((u >> 16) & 1)) >> 16 << 16
    return r.astype(np.uint32).view(np.float32)


def split3(x):
    """The device's split: hi the upper half of the bits, mid the remainder
    rounded, lo what is left."""
    hi = (x.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
    r = x - hi
    mid = _bf16_round(r)
    return hi, mid, _bf16_round(r - mid)


def test_planes_sum_to_the_value():
    r = np.random.Generator(np.random.PCG64(5))
    x = (r.standard_normal(1 << 16) * np.exp2(r.integers(-90, 120, 1 << 16))).astype(np.float32)
    x[:6] = [0.0, -0.0, np.finfo(np.float32).max, -np.finfo(np.float32).max, 1.0, np.float32(1) - np.float32(U)]
    hi, mid, lo = split3(x)
    assert np.isfinite(hi).all() and np.isfinite(mid).all() and np.isfinite(lo).all()
    total = hi.astype(np.float64) + mid.astype(np.float64) + lo.astype(np.float64)
    assert np.array_equal(total, x.astype(np.float64))
    # the dropped products mid*lo, lo*mid, lo*lo, each relative to x*y
    ax = np.maximum(np.abs(x.astype(np.float64)), 1e-300)
    rm, rl = (np.abs(p.astype(np.float64)) / ax for p in (mid, lo))
    assert rm.max() <= 2.0 ** -7 and rl.max() <= 2.0 ** -16
    assert rm.max() * rl.max() <= 2.0 ** -23


@pytest.mark.gpu
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("n,m,scale", [(32, 1, 1.0), (96, 2, 1e-3), (352, 7, 2.5)])
def test_forward_and_gradients(gpu, d, n, m, scale):
    """One to eleven blocks: forward and gradients of the sparse-only variant
    (tiles only) against the float64 oracle. With logits up to M in magnitude a
    float32 dot product of d terms is off by at most (d + 2) u M (M taken over
    the sums of magnitudes), a weight by that plus a few u, and every result is
    a sum of such terms: 4 (d + 2) u (1 + M) of the result's largest entry
    bounds all of them with room for the sums over the row."""
    q, k, v = inputs.random_qkv(900 + n + d, 1, 2, n, d, "f32", scale=scale)
    g = np.random.Generator(np.random.PCG64(n + d)).standard_normal(q.shape).astype(np.float32)
    tq, tk, tv, tg = (dev(a) for a in (q, k, v, g))
    idx = torch.empty(1, 2, n // 32, m, dtype=torch.int32, device="cuda")
    lse = torch.empty(1, 2, n, device="cuda")
    out = gpu.sparse_attention_forward(tq, tk, tv, m, idx_out=idx, lse_out=lse)
    grads = gpu.attention_backward(tq, tk, tv, out, tg, lse, idx, coarse=False)
    gi = host(idx).astype(np.int64)
    for h in range(2):
        qd, kd, vd, gd = (a[0, h].astype(np.float64) for a in (q, k, v, g))
        M = (np.abs(qd) @ np.abs(kd).T).max() / np.sqrt(d)
        tol = 4 * (d + 2) * U * (1 + M)
        keep = np.zeros((n // 32, n // 32), bool)
        np.put_along_axis(keep, gi[0, h], True, axis=1)
        keep = keep.repeat(32, 0).repeat(32, 1)
        P = np.where(keep, qd @ kd.T / np.sqrt(d), -np.inf)
        A = np.exp(P - P.max(1, keepdims=True))
        A /= A.sum(1, keepdims=True)
        Z = A @ vd
        dP = A * (gd @ vd.T - (gd * Z).sum(1, keepdims=True))
        # dQ, dK: sums whose terms may cancel, so measured against their magnitudes
        mag = A * (np.abs(gd) @ np.abs(vd).T + np.abs(gd * Z).sum(1, keepdims=True))
        refs = (dP @ kd / np.sqrt(d), dP.T @ qd / np.sqrt(d), A.T @ gd)
        mags = (mag @ np.abs(kd) / np.sqrt(d), mag.T @ np.abs(qd) / np.sqrt(d), A.T @ np.abs(gd))
        assert np.abs(host(out)[0, h] - Z).max() <= tol * np.abs(vd).max()
        for got, ref, big in zip(grads, refs, mags):
            assert np.abs(host(got)[0, h] - ref).max() <= tol * big.max()
