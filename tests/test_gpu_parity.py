"""GPU parity: the HIP kernels (through the C ABI) against the float64 oracle
on the same seeded inputs. Bars: selection bit-exact except near-ties (within
1e-6 relative of the m-th score, lower index first); outputs within 1e-5 max
row-normwise relative error for float32 inputs and 2e-2 for bfloat16 inputs.
"""
import math

import numpy as np
import pytest
import torch

from oracle import mra_oracle as O
from paper_2207_10284_amd import inputs
from tests.parity import TOL, check_selection, dev, err_stats, host, record, row_rel_err

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _say(*a):
    print(*a, flush=True)


# ------------------------------------------------------------------ per step
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_pool(gpu, dtype, d):
    _say("pool", dtype, d)
    q, k, v = inputs.random_qkv(101 + d, 2, 3, 160, d, dtype, scale=3.0)
    qp, kp, vp = gpu.pool(dev(q, dtype), dev(k, dtype), dev(v, dtype))
    torch.cuda.synchronize()
    for a, g in ((q, qp), (k, kp), (v, vp)):
        ref = O.pool_batched(a, 32)
        # float32 sum of 32 terms: |error| <= 31 u sum|x| / 32
        bound = 31 * U * O.pool_batched(np.abs(a), 32) + 1e-30
        assert (np.abs(host(g) - ref) <= bound).all()
    # one tensor alone
    qp2, kp2, vp2 = gpu.pool(dev(q, dtype))
    assert kp2 is None and vp2 is None
    assert torch.equal(qp2, qp)


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("n", [32, 96, 2112])
def test_coarse_scores(gpu, d, n):
    _say("coarse", d, n)
    r = np.random.Generator(np.random.PCG64(7 + n + d))
    qp = r.standard_normal((2, 3, n // 32, d)).astype(np.float32) * 2
    kp = r.standard_normal((2, 3, n // 32, d)).astype(np.float32) * 2
    S = host(gpu.coarse_scores(dev(qp), dev(kp)))
    ref = O.coarse_batched(qp, kp)
    # float64 accumulation, one rounding to float32
    mag = np.einsum("bhxd,bhyd->bhxy", np.abs(qp.astype(np.float64)), np.abs(kp.astype(np.float64))) / math.sqrt(d)
    assert (np.abs(S - ref) <= U * np.abs(ref) + 1e-12 * mag).all()


@pytest.mark.parametrize("nb,m", [(1, 1), (5, 2), (16, 4), (64, 63), (100, 8), (128, 16), (1024, 32), (2048, 5)])
def test_select_exact(gpu, nb, m):
    _say("select", nb, m)
    r = np.random.Generator(np.random.PCG64(nb * 31 + m))
    S = r.standard_normal((2, 3, nb, nb)).astype(np.float32)
    S[0, 0] = np.round(S[0, 0] * 2) / 2            # many exact ties
    S[0, 1] = 0.0
    S[0, 1, :, ::3] = -0.0                         # -0 ranks equal to +0
    S[1, 0, :, -1] = np.inf
    S[1, 0, :, 0] = -np.inf
    idx = host(gpu.select(dev(S), m)).astype(np.int64)
    ref = O.select_batched(S.astype(np.float64), m)
    assert np.array_equal(idx, ref)


def test_select_budget_extremes(gpu):
    S = np.random.Generator(np.random.PCG64(3)).standard_normal((1, 2, 40, 40)).astype(np.float32)
    assert np.array_equal(host(gpu.select(dev(S), 40)), np.broadcast_to(np.arange(40), (1, 2, 40, 40)))
    assert gpu.select(dev(S), 0).shape == (1, 2, 40, 0)


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("nb,m", [(1, 0), (1, 1), (7, 3), (128, 16), (1024, 32)])
def test_coarse_term(gpu, d, nb, m):
    _say("coarse_term", d, nb, m)
    r = np.random.Generator(np.random.PCG64(nb + m + d))
    S = (r.standard_normal((1, 3, nb, nb)) * 8).astype(np.float32)
    vp = r.standard_normal((1, 3, nb, d)).astype(np.float32)
    idx = O.select_batched(S.astype(np.float64), m)
    cmax, csum, cvec = gpu.coarse_term(dev(S), torch.from_numpy(idx.astype(np.int32)).cuda(), dev(vp))
    M, c, L = O.coarse_term_batched(S.astype(np.float64), idx, vp, 32)
    gM, gc, gL = host(cmax), host(csum), host(cvec)
    fin = np.isfinite(M)
    assert np.array_equal(np.isfinite(gM), fin) and (gM[fin] == M[fin]).all()    # max is exact
    # float32 exp (a few ulp) and float32 sums of at most nb terms
    tol = (nb + 8) * U
    assert (np.abs(gc - c) <= tol * c).all()
    bound = tol * c[..., None] * np.abs(vp.astype(np.float64)).max(axis=2, keepdims=True)
    assert (np.abs(gL - L) <= bound + 1e-30).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_tile_pass(gpu, dtype, d):
    """Tile pass alone, given the oracle's selection and coarse term."""
    _say("tile", dtype, d)
    B, H, n, m = 2, 3, 320, 3
    q, k, v = inputs.random_qkv(500 + d, B, H, n, d, dtype, scale=1.5)
    Z, idx = O.mra_batched(q, k, v, 32, m)
    qp, kp, vp = (O.pool_batched(a, 32) for a in (q, k, v))
    S = O.coarse_batched(qp, kp)
    M, c, L = O.coarse_term_batched(S, idx, vp, 32)
    out = gpu.block_sddmm_spmm(dev(q, dtype), dev(k, dtype), dev(v, dtype),
                               torch.from_numpy(idx.astype(np.int32)).cuda(),
                               dev(M), dev(c), dev(L))
    err = row_rel_err(host(out), Z)
    _say("  err", err)
    assert err <= TOL[dtype]


# ------------------------------------------------------------------ whole pass
def _forward_and_check(gpu, q, k, v, m, dtype, tol=None):
    tq, tk, tv = dev(q, dtype), dev(k, dtype), dev(v, dtype)
    B, H, n, d = q.shape
    idx = torch.empty(B, H, n // 32, m, dtype=torch.int32, device="cuda")
    out = gpu.attention_forward(tq, tk, tv, m, idx_out=idx)
    gi = host(idx).astype(np.int64)
    differ = 0
    for b in range(B):
        for h in range(H):
            S = O.coarse_logits(O.block_mean(q[b, h], 32), O.block_mean(k[b, h], 32))
            differ += check_selection(gi[b, h], S, m)
    Z, _ = O.mra_batched(q, k, v, 32, m, idx=gi)     # oracle under the GPU's (valid) selection
    err = row_rel_err(host(out), Z)
    assert err <= (tol or TOL[dtype]), err
    return out, idx, err, differ


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("B,H,n,m", [(1, 1, 32, 0), (1, 1, 32, 1), (2, 3, 160, 2), (1, 2, 512, 0),
                                     (1, 2, 512, 5), (1, 1, 512, 16), (1, 3, 1056, 7)])
def test_forward_small(gpu, dtype, d, B, H, n, m):
    _say("forward", dtype, d, B, H, n, m)
    q, k, v = inputs.random_qkv(1000 + n + d + m, B, H, n, d, dtype, scale=1.2)
    _, _, err, differ = _forward_and_check(gpu, q, k, v, m, dtype)
    _say("  err", err, "rows with tie swaps", differ)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("n,m", [(6400, 9), (22400, 12), (48000, 10)])
def test_forward_wide_heads(gpu, dtype, d, n, m):
    """Heads of 200, 700 and 1500 blocks: the fused selection kernel's 8-, 16-
    and 32-register tiers (16-key logit tiles spread over the waves with a
    ragged last tile, coarse-term batches past the head's last block)."""
    _say("forward wide", dtype, d, n, m)
    q, k, v = inputs.random_qkv(3000 + n + d, 1, 2 if n < 10000 else 1, n, d, dtype, scale=1.2)
    _, _, err, differ = _forward_and_check(gpu, q, k, v, m, dtype)
    _say("  err", err, "rows with tie swaps", differ)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,m", [(6400, 9), (22400, 12), (48000, 10)])
def test_forward_matches_stepwise_bitwise_wide(gpu, dtype, n, m):
    """The fused forward equals the step-wise calls bit for bit on wide heads
    too (selection, coarse term and output)."""
    q, k, v = inputs.random_qkv(78 + n, 1, 2, n, 64, dtype)
    nb = n // 32
    tq, tk, tv = dev(q, dtype), dev(k, dtype), dev(v, dtype)
    idx_f = torch.empty(1, 2, nb, m, dtype=torch.int32, device="cuda")
    out_f = gpu.attention_forward(tq, tk, tv, m, idx_out=idx_f)
    qp, kp, vp = gpu.pool(tq, tk, tv)
    S = gpu.coarse_scores(qp, kp)
    idx = gpu.select(S, m)
    cm, cs, cv = gpu.coarse_term(S, idx, vp)
    out = gpu.block_sddmm_spmm(tq, tk, tv, idx, cm, cs, cv)
    assert torch.equal(idx, idx_f)
    assert torch.equal(out, out_f)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_forward_matches_stepwise_bitwise(gpu, dtype, d):
    """The one-call forward (for float32 its tile pass reads K and V copied
    into matrix-core operand order by the pooling pass) equals the step-wise
    calls (row-major K and V) bit for bit."""
    q, k, v = inputs.random_qkv(77 + d, 2, 2, 640, d, dtype)
    m = 4
    tq, tk, tv = dev(q, dtype), dev(k, dtype), dev(v, dtype)
    idx_f = torch.empty(2, 2, 20, m, dtype=torch.int32, device="cuda")
    out_f = gpu.attention_forward(tq, tk, tv, m, idx_out=idx_f)
    qp, kp, vp = gpu.pool(tq, tk, tv)
    S = gpu.coarse_scores(qp, kp)
    idx = gpu.select(S, m)
    cm, cs, cv = gpu.coarse_term(S, idx, vp)
    out = gpu.block_sddmm_spmm(tq, tk, tv, idx, cm, cs, cv)
    assert torch.equal(idx, idx_f)
    assert torch.equal(out, out_f)
    out_s = gpu.sparse_attention_forward(tq, tk, tv, m)
    assert torch.equal(gpu.block_sddmm_spmm(tq, tk, tv, idx), out_s)


# ------------------------------------------------------------------ invariants
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_unit_values_give_unit_output(gpu, dtype):
    q, k, _ = inputs.random_qkv(11, 1, 2, 512, 64, dtype, scale=3.0)
    v = np.ones_like(q)
    for m in (0, 3, 16):
        out = host(gpu.attention_forward(dev(q, dtype), dev(k, dtype), dev(v, dtype), m))
        assert np.abs(out - 1).max() <= (2e-6 if dtype == "f32" else 2 ** -8)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_zero_queries(gpu, dtype):
    _, k, v = inputs.random_qkv(12, 1, 2, 512, 64, dtype)
    q = np.zeros_like(k)
    m = 5
    idx = torch.empty(1, 2, 16, m, dtype=torch.int32, device="cuda")
    out = host(gpu.attention_forward(dev(q, dtype), dev(k, dtype), dev(v, dtype), m, idx_out=idx))
    assert np.array_equal(host(idx), np.broadcast_to(np.arange(m), (1, 2, 16, m)))
    ref = np.broadcast_to(v.astype(np.float64).mean(axis=2, keepdims=True), out.shape)
    assert row_rel_err(out, ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_constant_blocks_exact(gpu, dtype):
    """Q, K constant within each 32-row block: the approximation is exact for
    every budget, so the GPU output must match exact attention."""
    r = np.random.Generator(np.random.PCG64(13))
    qb = r.standard_normal((1, 2, 8, 64)); kb = r.standard_normal((1, 2, 8, 64))
    cast = inputs.round_to_bf16 if dtype == "bf16" else (lambda a: a.astype(np.float32))
    q = cast(np.repeat(qb, 32, axis=2)); k = cast(np.repeat(kb, 32, axis=2))
    v = cast(r.standard_normal((1, 2, 256, 64)))
    ref = np.stack([np.stack([O.exact_attention(q[0, h], k[0, h], v[0, h]) for h in range(2)])])
    for m in (0, 1, 3, 8):
        out = host(gpu.attention_forward(dev(q, dtype), dev(k, dtype), dev(v, dtype), m))
        assert row_rel_err(out, ref) <= TOL[dtype], m


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_full_budget_is_exact_attention(gpu, dtype):
    q, k, v = inputs.random_qkv(14, 1, 2, 384, 64, dtype, scale=2.0)
    out = host(gpu.attention_forward(dev(q, dtype), dev(k, dtype), dev(v, dtype), 12))
    ref = np.stack([np.stack([O.exact_attention(q[0, h], k[0, h], v[0, h]) for h in range(2)])])
    assert row_rel_err(out, ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_large_logits_finite(gpu, dtype):
    """Logits of magnitude ~500: the output stays finite and within the error
    that a float32 dot product of length d allows. A float32 logit carries an
    absolute error up to (d+2) u c sum_t |q_t k_t|; the normalised output moves
    by at most about twice the largest logit error (relative)."""
    q, k, v = inputs.random_qkv(15, 1, 1, 512, 64, dtype, scale=12.0)
    d = q.shape[-1]
    mag = (np.abs(q[0, 0]).astype(np.float64) @ np.abs(k[0, 0]).astype(np.float64).T).max() / math.sqrt(d)
    tol = max(TOL[dtype], 2 * (d + 2) * U * mag)
    for m in (0, 2, 16):
        out, _, err, _ = _forward_and_check(gpu, q, k, v, m, dtype, tol=tol)
        assert torch.isfinite(out.float()).all()
        _say("  large logits m", m, "err", err, "tol", tol)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_reference_restart(gpu, dtype, d):
    """The first selected block of every row has logits near -2 while a later
    selected block has logits of 120: relative to the first block's max the
    later weights would overflow, so the tile pass computes the row again
    relative to its exact max. The result matches the oracle, is finite, and
    the forward agrees bitwise with the step-wise calls."""
    _say("restart", dtype, d)
    n, m = 256, 4
    r = np.random.Generator(np.random.PCG64(4242 + d))
    logit = np.full(n // 32, -2.0)
    logit[1], logit[6] = 2.0, 120.0                 # selected: blocks 0, 1, 2 (ties), 6
    q = np.zeros((1, 1, n, d)); q[..., 0] = 16.0
    k = np.zeros((1, 1, n, d)); k[0, 0, :, 0] = np.repeat(logit, 32) * math.sqrt(d) / 16.0
    v = r.standard_normal((1, 1, n, d))
    if dtype == "bf16":
        k, v = inputs.round_to_bf16(k), inputs.round_to_bf16(v)
    else:
        k, v = k.astype(np.float32).astype(np.float64), v.astype(np.float32).astype(np.float64)
    out, idx, err, _ = _forward_and_check(gpu, q, k, v, m, dtype)
    assert (host(idx)[0, 0] == np.array([0, 1, 2, 6])).all()
    assert torch.isfinite(out.float()).all()
    tq, tk, tv = dev(q, dtype), dev(k, dtype), dev(v, dtype)
    qp, kp, vp = gpu.pool(tq, tk, tv)
    S = gpu.coarse_scores(qp, kp)
    sel = gpu.select(S, m)
    cm, cs, cv = gpu.coarse_term(S, sel, vp)
    o1 = gpu.block_sddmm_spmm(tq, tk, tv, sel, cm, cs, cv)
    assert torch.equal(o1, out)
    _say("  restart err", err)


def test_empty_problems(gpu):
    e = torch.empty(0, 2, 64, 64, device="cuda")
    assert gpu.attention_forward(e, e, e, 1).shape == e.shape
    e = torch.empty(1, 2, 0, 64, device="cuda")
    assert gpu.attention_forward(e, e, e, 0).shape == e.shape


# ------------------------------------------------------------------ workloads at full size
@pytest.mark.parametrize("name", list(inputs.WORKLOADS))
def test_workload_full_size(gpu, name):
    """Each workload at its real shape, in the launch configuration the
    benchmark times (one mra_attention_forward call). Every block-row of
    every head is checked: its selection against the oracle's float64 scores
    (exact except near-ties) and its 32 output rows against the oracle
    evaluated under the GPU's selection (Sec. 4.2 Alg. 1 per block-row,
    eq. actual_approx_mat_form, Sec. 4.3 Alg. 2)."""
    w = inputs.WORKLOADS[name]
    _say("workload", name)
    q, k, v = inputs.make_qkv(w)
    tq, tk, tv = dev(q, w.dtype), dev(k, w.dtype), dev(v, w.dtype)
    idx = torch.empty(w.B, w.H, w.nb, w.budget, dtype=torch.int32, device="cuda")
    out = gpu.attention_forward(tq, tk, tv, w.budget, idx_out=idx)
    torch.cuda.synchronize()
    out_h = out.float().cpu().numpy()
    gi = idx.cpu().numpy().astype(np.int64)
    del tq, tk, tv, out
    Zall = np.empty(out_h.shape)
    differ = 0
    for b in range(w.B):
        for h in range(w.H):
            qh, kh = q[b, h].astype(np.float64), k[b, h].astype(np.float64)
            S = O.coarse_logits(O.block_mean(qh, 32), O.block_mean(kh, 32))
            differ += check_selection(gi[b, h], S, w.budget)
            Zall[b, h], _, _ = O.mra_factored_rows(qh, kh, v[b, h], 32, w.budget, idx=gi[b, h])
    st = err_stats(out_h, Zall)
    record("MRA-2", name, w.dtype, w.B * w.H, w.B * w.H * w.nb, st, TOL[w.dtype], differ)
    _say(f"  {name}: max row rel err {st['row']:.3e} over {w.B * w.H * w.nb} block-rows, tie swaps {differ}")
    assert st["row"] <= TOL[w.dtype]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("B,H,n,m", [(1, 1, 512, 1), (1, 1, 512, 2), (1, 1, 512, 3), (1, 1, 512, 5), (1, 2, 4096, 9),
                                     (1, 3, 2752, 7), (1, 8, 4096, 3), (1, 9, 4096, 3)])
def test_rows_shared_by_waves(gpu, dtype, d, B, H, n, m):
    """16 to 1152 block-rows: one, two or four waves per row (by the number of
    rows, at most one per tile), tiles that do not divide among the waves, and
    both sides of the lines at 256 and 1024 rows."""
    _say("shared rows", dtype, d, B, H, n, m)
    q, k, v = inputs.random_qkv(5000 + n + m + d, B, H, n, d, dtype, scale=1.3)
    _, _, err, _ = _forward_and_check(gpu, q, k, v, m, dtype)
    _say("  err", err)


@pytest.mark.parametrize("d", [32, 64, 128])
def test_shared_rows_without_valid_entries(gpu, d):
    """Rows whose list holds fewer valid entries than the waves that share it
    (none, one, two of four): the waves without a tile add nothing."""
    n = 256
    q, k, v = inputs.random_qkv(5100 + d, 1, 1, n, d, "bf16")
    idx = np.full((1, 1, 8, 4), -1, np.int32)
    for x in range(1, 8):
        idx[0, 0, x, :x % 4] = np.arange(x % 4) * 2
    tq, tk, tv = (dev(a, "bf16") for a in (q, k, v))
    M = torch.full((1, 1, 8), 0.5, device="cuda")
    c = torch.full((1, 1, 8), 32.0, device="cuda")
    L = torch.full((1, 1, 8, d), 16.0, device="cuda")
    out = host(gpu.block_sddmm_spmm(tq, tk, tv, torch.from_numpy(idx).cuda(), M, c, L))[0, 0]
    qd, kd, vd = (a[0, 0].astype(np.float64) for a in (q, k, v))
    for x in range(8):
        cols = np.concatenate([np.arange(32 * y, 32 * y + 32) for y in idx[0, 0, x] if y >= 0] or [np.arange(0)])
        P = qd[32 * x:32 * x + 32] @ kd[cols].T / math.sqrt(d)
        E = np.exp(P)
        ref = (E @ vd[cols] + np.exp(0.5) * 16.0) / (E.sum(1, keepdims=True) + np.exp(0.5) * 32.0)
        assert row_rel_err(out[32 * x:32 * x + 32], ref) <= TOL["bf16"], x


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_shared_rows_weigh_as_one_wave(gpu, dtype, d):
    """A head of 16 block-rows alone (four waves per row), among 40 (two) and
    among 65 (one): the weights, rounded to bfloat16 there, are the same, so the
    row sums differ by the order of their additions only. Each of the two sums
    of 32 m positive terms is off by at most 32 m u, its logarithm by as much,
    and the log normaliser is rounded twice more; an output entry is a sum of
    as many terms, rounded to its type."""
    _say("shared rows, weights", dtype, d)
    H, n, m = 65, 512, 7
    q, k, v = inputs.random_qkv(5200 + d, 1, H, n, d, dtype, scale=1.6)
    r = np.random.Generator(np.random.PCG64(d))
    idx = np.sort(np.argsort(r.random((1, H, n // 32, n // 32)), axis=-1)[..., :m], axis=-1).astype(np.int32)
    args = [dev(q, dtype), dev(k, dtype), dev(v, dtype), torch.from_numpy(idx).cuda()]

    def tiles(heads):
        lse = torch.empty(1, heads, n, device="cuda")
        out = gpu.block_sddmm_spmm(*(t[:, :heads].contiguous() for t in args), lse_out=lse)
        return out.float(), lse

    whole, lse = tiles(H)
    order = 2 * 32 * m * U
    ulp = U if dtype == "f32" else 2.0 ** -8
    for heads in (1, 40):
        o, l = tiles(heads)
        far = (l - lse[:, :heads]).abs().max()
        _say("  heads", heads, "lse", float(far))
        assert far <= order + 4 * U * lse.abs().max()
        assert (o - whole[:, :heads]).abs().sub(2 * ulp * whole[:, :heads].abs()).max() <= 2 * order * np.abs(v).max()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("H,m,hot", [(130, 6, 1), (130, 6, 5), (40, 6, 1), (40, 6, 2), (40, 6, 5), (1, 2, 1), (1, 6, 1),
                                     (1, 6, 4), (1, 6, 5), (1, 3, 2)])
def test_reference_restart_shared_rows(gpu, dtype, d, H, m, hot):
    """The restart with one wave per block-row (1040 rows), two (320 rows, or two
    tiles) and four (8 rows): the tile at place `hot` of each list has logits
    near 120 above the first one's, so its weights overflow the first tile's
    reference in whichever wave has it (its first tile or its second), and the
    whole row, the waves that saw nothing included, is formed again. An error of
    a logit of magnitude 120 moves a weight by (d + 2) u 120."""
    _say("restart, shared rows", dtype, d, H, m, hot)
    n = 256
    r = np.random.Generator(np.random.PCG64(100 * d + 10 * m + hot))
    q, k, v = (0.3 * r.standard_normal((1, H, n, d)) for _ in range(3))
    logit = np.full(n // 32, -2.0)
    logit[hot + 1] = 120.0
    q[..., 0] = 16.0
    k[..., 0] = np.repeat(logit, 32) * math.sqrt(d) / 16.0
    q, k, v = (inputs.round_to_bf16(a) if dtype == "bf16" else a.astype(np.float32) for a in (q, k, v))
    idx = np.broadcast_to(np.arange(1, m + 1, dtype=np.int32), (1, H, n // 32, m)).copy()
    lse = torch.empty(1, H, n, device="cuda")
    out = gpu.block_sddmm_spmm(dev(q, dtype), dev(k, dtype), dev(v, dtype), torch.from_numpy(idx).cuda(), lse_out=lse)
    assert torch.isfinite(out.float()).all() and torch.isfinite(lse).all()
    tol = max(TOL[dtype], 2 * (d + 2) * U * 130)
    cols = slice(32, 32 * (m + 1))
    for h in (0, H - 1):
        qd, kd, vd = (a[0, h].astype(np.float64) for a in (q, k, v))
        P = qd @ kd[cols].T / math.sqrt(d)
        L = np.log(np.exp(P - 120).sum(1)) + 120
        ref = np.exp(P - L[:, None]) @ vd[cols]
        assert np.abs(host(out)[0, h] - ref).max() <= tol * np.abs(vd[cols]).max()
        assert np.abs(host(lse)[0, h] - L).max() <= tol
