"""Launches of more than 2^31 threads, whose grid goes on along y, for the
kernels that move lists: the separate unpack, both directions of the tensor
layout, and the one-call step.  16 or 32 bytes to a thread make these the
largest buffers of the tests, 34 to 69 GB.  (The grid's arithmetic at any size runs on
the host, in test_grid_host.py.)
"""

import numpy as np
import pytest
import torch

import paper_1801_03855_amd as tc
from tests.helpers import host_f32

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.fixture(autouse=True)
def _memory():
    torch.cuda.empty_cache()
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


def _numbered(n, salt):
    """Element e's bits are a hash of e, as binary32 storage."""
    out = torch.empty(n, dtype=torch.int32, device=DEV)
    step = 1 << 28
    for at in range(0, n, step):
        e = torch.arange(at, min(at + step, n), device=DEV)
        out[at:at + step] = (e * 2654435761 + salt).bitwise_and_(0x7fffffff).to(torch.int32)
    return out.view(torch.float32)


def test_separate_unpack():
    """64 lanes to 256 elements: 2^31 threads are 2^33 elements."""
    sizes = [(1 << 33) - 1_003, 5, 4_011]
    g = tc.Group(sizes)
    n = g.numel
    flat = _numbered(n, 1)
    store = torch.full((n + 16,), 7.0, device=DEV)
    lists = [list(store[1:1 + n].split(sizes))]
    tc.unpack(tc.TensorList(g, lists), [flat])
    assert torch.equal(store[1:1 + n].view(torch.int32), flat.view(torch.int32))
    assert bool((store[:1] == 7).all()) and bool((store[n + 1:] == 7).all())


def _same(got, want):
    """Slots of one copy against the tensor's, in pieces."""
    for at in range(0, got.shape[0], 1 << 26):
        if not torch.equal(got[at:at + (1 << 26)].view(torch.int32), want[at:at + (1 << 26)].contiguous().view(torch.int32)):
            return False
    return True


def test_tensor_layout_unpack():
    """Slot-aligned lists, K = 8: 512 threads to 256 elements of every copy."""
    K = 8
    sizes = [(1 << 30) - 76, 4, 1_035]
    g = tc.Group(sizes)
    n = g.numel
    T = _numbered(tc.tensor_numel(g, K), 2)
    store = torch.zeros(K, n + 9, device=DEV)
    assert store.stride(0) % 4 == 0
    tc.unpack_tensor(tc.TensorList(g, [list(row[:n].split(sizes)) for row in store]), T)
    want = T.view(-1, K, 4)
    for k in range(K):
        assert _same(store[k, : n // 4 * 4].view(-1, 4), want[: n // 4, k]), f"copy {k}"
        assert torch.equal(store[k, n // 4 * 4:n].view(torch.int32), want[-1, k, : n % 4].view(torch.int32)), f"copy {k}"
        assert not store[k, n:].any()


def test_tensor_layout_pack():
    """K = 8: 256 threads to 256 elements of every copy.  The copies are the same tensors."""
    K = 8
    sizes = [(1 << 31) - 77, 3, 1_032]
    g = tc.Group(sizes)
    n = g.numel
    flat = _numbered(n, 3)
    T = torch.zeros(tc.tensor_numel(g, K), device=DEV)
    tc.pack_tensor(tc.TensorList(g, [list(flat.split(sizes))] * K), T)
    got = T.view(-1, K, 4)
    for k in range(K):
        assert _same(flat[: n // 4 * 4].view(-1, 4), got[: n // 4, k]), f"copy {k}"
        assert torch.equal(flat[n // 4 * 4:].view(torch.int32), got[-1, k, : n % 4].view(torch.int32)), f"copy {k}"


def test_pipeline():
    """K = 8: 256 threads to 128 elements of every copy, so 2^31 are 2^30 elements."""
    K, eta, rho = 8, 0.05, 2.25
    sizes = [(1 << 30) - 77, 3, 1_031]
    g = tc.Group(sizes)
    n, m = g.numel, tc.tensor_numel(g, K)
    gen = torch.Generator(device=DEV).manual_seed(5)
    grad = torch.randn(n, generator=gen, device=DEV).mul_(0.01)
    grads = tc.TensorList(g, [list(grad.split(sizes))] * K)  # one set of gradients for all workers
    store = torch.zeros(K, n, device=DEV)
    params = tc.TensorList(g, [list(row.split(sizes)) for row in store])
    x = torch.randn(m, generator=gen, device=DEV).mul_(0.05)
    xc = torch.randn(n, generator=gen, device=DEV).mul_(0.05)
    mean = torch.zeros(n, device=DEV)
    at = np.unique(np.concatenate([np.random.default_rng(6).integers(0, n, 100_000), np.arange(64), np.arange(n - 2_000, n),
                                   np.arange((1 << 30) - 1_000, (1 << 30) + 600)]))
    ti = torch.from_numpy(at).to(DEV)
    pos = [(ti // 4 * K + k) * 4 + ti % 4 for k in range(K)]
    hx, hc, hg = [host_f32(x[p]) for p in pos], host_f32(xc[ti]), host_f32(grad[ti])
    tc.easgd_pipeline_tensor(grads, params, None, mean, x, xc, eta, rho)
    # binary32, the kernels' own sequence with every fma's product exact in binary64
    e, r = np.float32(eta), np.float32(rho)
    d = [v - hc for v in hx]
    new = [host_f32(x[p]) for p in pos]
    for k in range(K):
        t = (r.astype(np.float64) * d[k] + hg).astype(np.float32)
        ref = (-e.astype(np.float64) * t + hx[k]).astype(np.float32)
        # rounding twice (binary64, then binary32) may differ from an fma by one unit
        assert np.max(np.abs(new[k] - ref) / np.maximum(np.abs(ref), 1e-3)) < 2.0 ** -22, f"x[{k}]"
        assert np.array_equal(new[k], host_f32(store[k][ti])), f"parameters {k}"
    total = sum(v.astype(np.float64) for v in d)
    assert np.max(np.abs(host_f32(xc[ti]) - (hc + eta * rho * total))) < 1e-6
    assert np.max(np.abs(host_f32(mean[ti]) - hg)) < 1e-8
