"""The native binding of the forward calls and of mra_attention against the
Python autograd function and the refusals of the calls."""
import numpy as np
import pytest
import torch

from paper_2207_10284_amd import inputs
from tests.parity import dev

pytestmark = pytest.mark.gpu


def _inputs(dtype, n=160, d=32, B=2, H=3):
    q, k, v = (dev(a, dtype) for a in inputs.random_qkv(61, B, H, n, d, dtype))
    g = torch.randn(q.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(3)).to(q.dtype)
    return q, k, v, g


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("variant,budget,prior", [("mra2", 2, False), ("mra2", 0, False), ("mra2s", 3, False),
                                                  ("global", 7, True), ("global", 9, False)])
def test_node_matches_the_python_function(gpu, dtype, variant, budget, prior):
    """Same calls in the same order, so the same bits: output and gradients,
    with a gradient that is not contiguous, and with one input only."""
    print("node", dtype, variant, budget, flush=True)
    q, k, v, g = _inputs(dtype)
    g = g.transpose(2, 3).contiguous().transpose(2, 3)
    res = []
    for f in (gpu.mra_attention, gpu.MraAttention.apply):
        a = [t.clone().requires_grad_(True) for t in (q, k, v)]
        z = f(*a, budget, variant, prior)
        res.append((z.detach(), *torch.autograd.grad(z, a, g)))
    for x, y in zip(*res):
        assert torch.equal(x, y)
    k2 = k.clone().requires_grad_(True)
    gpu.mra_attention(q, k2, v, budget, variant, prior).backward(g)
    assert torch.equal(k2.grad, res[0][2])
    assert not gpu.mra_attention(q, k, v, budget, variant, prior).requires_grad


def test_saved_tensor_hooks_see_every_tensor(gpu):
    """A hook that moves what is saved to host memory and back gives the same
    gradients (the node keeps no address from its forward)."""
    q, k, v, g = _inputs("bf16")
    a = [t.clone().requires_grad_(True) for t in (q, k, v)]
    ref = torch.autograd.grad(gpu.mra_attention(*a, 2), a, g)
    seen = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: (seen.append(t.shape), t.cpu())[1], lambda t: t.cuda()):
        z = gpu.mra_attention(*a, 2)
    got = torch.autograd.grad(z, a, g)
    assert len(seen) == 9                      # q, k, v, z, log normalisers, selection, three block means
    for x, y in zip(ref, got):
        assert torch.equal(x, y)


def test_another_stream(gpu):
    """Calls go to the caller's current stream, the backward to its forward's."""
    q, k, v, g = _inputs("f32")
    a = [t.clone().requires_grad_(True) for t in (q, k, v)]
    ref = torch.autograd.grad(gpu.mra_attention(*a, 2), a, g)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        z = gpu.mra_attention(*a, 2)
    got = torch.autograd.grad(z, a, g)
    torch.cuda.synchronize()
    for x, y in zip(ref, got):
        assert torch.equal(x, y)


def test_refusals(gpu):
    q, k, v, _ = _inputs("f32")
    for call in (gpu.attention_forward, gpu.sparse_attention_forward, gpu.attention_forward_global, gpu.mra_attention):
        with pytest.raises(ValueError):
            call(q.cpu(), k.cpu(), v.cpu(), 2)
        with pytest.raises(ValueError):
            call(q, k[:, :2], v, 2)
        with pytest.raises(ValueError):
            call(q.transpose(0, 1), k.transpose(0, 1), v.transpose(0, 1), 2)
        with pytest.raises(TypeError):
            call(q.half(), k.half(), v.half(), 2)
        with pytest.raises(gpu.MraError) as e:
            call(q, k, v, 6 if call is not gpu.attention_forward_global else 26)
        assert e.value.status == 1
    with pytest.raises(ValueError):
        gpu.attention_forward(q, k, v, 2, idx_out=torch.empty(2, 3, 5, 3, dtype=torch.int32, device="cuda"))
    with pytest.raises(gpu.MraError) as e:
        gpu.attention_forward(q, k, v, 2, workspace=torch.empty(256, dtype=torch.uint8, device="cuda"))
    assert e.value.status == 4
    with pytest.raises(ValueError):
        gpu.mra_attention(q, k, v, 2, "none")
    with pytest.raises(RuntimeError):
        torch.func.vmap(lambda a: gpu.mra_attention(a, k, v, 2))(q.expand(2, *q.shape))
    with torch.autograd.forward_ad.dual_level(), pytest.raises(RuntimeError):
        gpu.mra_attention(torch.autograd.forward_ad.make_dual(q, torch.ones_like(q)), k, v, 2)


def test_errors_of_the_backward(gpu):
    """What the backward refuses (here tensors that a saved-tensor hook swapped)
    is the exception of the Python function: ValueError by the checks, MraError
    with its status by the library; a hook's own exception and an exhausted
    allocator come through as they are."""
    q, k, v, g = _inputs("f32")

    def backward(f, unpack):
        a = [t.clone().requires_grad_(True) for t in (q, k, v)]
        with torch.autograd.graph.saved_tensors_hooks(lambda t: t, unpack):
            z = f(*a, 2, "mra2", False)
        z.backward(g)

    def boom(t):
        raise LookupError("unpack")

    def wider(t):                              # a selection of more columns than there are
        return torch.zeros(2, 3, 5, 6, dtype=torch.int32, device="cuda") if t.dtype == torch.int32 else t

    for f in (gpu.MraAttention.apply, gpu.mra_attention):
        with pytest.raises(ValueError, match="ROCm device"):
            backward(f, lambda t: t.cpu())
        with pytest.raises(LookupError, match="unpack"):
            backward(f, boom)
        with pytest.raises(gpu.MraError) as e:
            backward(f, wider)
        assert e.value.status == 1
    with torch.autograd.graph.saved_tensors_hooks(boom, lambda t: t), pytest.raises(LookupError, match="unpack"):
        gpu.mra_attention(q.clone().requires_grad_(True), k, v, 2)
    big = [torch.zeros(8, 16, 4096, 64, device="cuda") for _ in range(3)]
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    try:
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (8 << 20)) / total)
        for call in (gpu.attention_forward, gpu.mra_attention):
            with pytest.raises(torch.OutOfMemoryError):
                call(*big, 8)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)


def test_refusals_name_what_they_expect(gpu):
    q, k, v, _ = _inputs("f32")
    short = torch.empty(2, device="cuda")
    for call, width in ((gpu.attention_forward, 2), (gpu.sparse_attention_forward, 2), (gpu.attention_forward_global, 5)):
        with pytest.raises(ValueError, match=rf"idx must be .* of shape \(2, 3, 5, {width}\)"):
            call(q, k, v, 2, idx_out=short.int())
        with pytest.raises(ValueError, match=r"lse_out must be .* of shape \(2, 3, 160\)"):
            call(q, k, v, 2, lse_out=short)


class _Tagged(torch.Tensor):
    pass


def test_tensor_subclass_gets_its_own_type(gpu):
    """The result of a call on a tensor subclass is of that type (its empty_like
    makes it), with the values of the plain call."""
    q, k, v, g = _inputs("f32")
    t = [x.as_subclass(_Tagged) for x in (q, k, v)]
    for call in (gpu.attention_forward, gpu.sparse_attention_forward, gpu.attention_forward_global, gpu.mra_attention):
        z = call(*t, 2)
        assert type(z) is _Tagged
        assert torch.equal(z.as_subclass(torch.Tensor), call(q, k, v, 2))
    assert type(gpu.attention_forward(*(torch.nn.Parameter(x) for x in (q, k, v)), 2)) is torch.Tensor
    with pytest.raises(ValueError):
        gpu.mra_attention(q, k, v, 2, ["mra2"])
