"""Tensor-layout pack and unpack at the edges of their tiles: 16 to 128 lanes
of 16 bytes per copy (by K, type, direction and alignment), copies in groups of
one 128-byte line (K = 16, 24, 32, 48, 64), tiles that lie in one tensor, in a
few and in more than 32, zero-size tensors and the last, partial slot.  Bit for
bit the oracle's index map.
"""

import numpy as np
import pytest
import torch

import paper_1801_03855_amd as tc
from tests.test_gpu_pipeline_tiles import RENUMBERED, _groups, _lists

pytestmark = pytest.mark.gpu

DEV = "cuda"
KS = [1, 2, 4, 5, 7, 8, 9, 13, 15, 16, 17, 24, 31, 32, 33, 40, 48, 64]


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("K", KS)
def test_pack_and_unpack(orc, K, dtype, shift):
    code = np.uint32 if dtype == torch.float32 else np.uint16
    whole = torch.int32 if dtype == torch.float32 else torch.int16
    rng = np.random.default_rng(100 * K + shift)
    for sizes in _groups() + [[5000, 3, 4099]]:
        g = tc.Group(sizes)
        n, m = g.numel, tc.tensor_numel(g, K)
        what = f"K={K} {dtype} shift={shift} n={n} in {len(sizes)}"
        rows = _lists(sizes, K, dtype, shift)
        flat = [rng.integers(0, 2 ** (8 * code().itemsize), n, dtype=code) for _ in range(K)]
        for row, f in zip(rows, flat):
            at = 0
            for t in row:
                t.view(whole).copy_(torch.from_numpy(f[at:at + t.numel()].view(np.dtype(f"i{code().itemsize}"))))
                at += t.numel()
        # padding positions are never written
        want = orc.tensor_from_copies([f.view(np.float32) if code == np.uint32 else f for f in flat], fill=0)
        T = torch.zeros(m, dtype=dtype, device=DEV)
        tc.pack_tensor(tc.TensorList(g, rows), T)
        got = T.view(whole).cpu().numpy().view(code)
        assert np.array_equal(got, want.view(code)), f"{what}: pack"
        # unpack: every copy's tensors, and nothing around them
        back = _lists(sizes, K, dtype, shift)
        tc.unpack_tensor(tc.TensorList(g, back), T)
        for a, b in zip(back, rows):
            assert torch.equal(a[0]._base.view(whole), b[0]._base.view(whole)), f"{what}: unpack"


def _interleaved(sizes, K, dtype, shift, seed):
    """Lists of random bits, and what they are interleaved (zeros past the last element)."""
    whole = torch.int32 if dtype == torch.float32 else torch.int16
    n = sum(sizes)
    rows = _lists(sizes, K, dtype, shift)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    want = torch.zeros(-(-n // 4), K, 4, dtype=whole, device=DEV)
    for k, row in enumerate(rows):
        lim = torch.iinfo(whole)
        bits = torch.randint(lim.min, lim.max, (n,), generator=gen, device=DEV, dtype=whole)
        for t, v in zip(row, torch.split(bits, sizes)):
            t.view(whole).copy_(v)
        want[: n // 4, k] = bits[: n // 4 * 4].view(-1, 4)
        if n % 4:
            want[-1, k, : n % 4] = bits[n // 4 * 4:]
    return rows, want


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("K", [1, 2, 4, 7, 8, 13, 16, 17, 24, 32, 33, 48, 64])
def test_renumbered_tiles(K, dtype, shift):
    """Both directions where the tiles are renumbered in runs, the last not full."""
    g = tc.Group(RENUMBERED)
    rows, want = _interleaved(RENUMBERED, K, dtype, shift, 300 * K + shift)
    T = torch.zeros(tc.tensor_numel(g, K), dtype=dtype, device=DEV)
    tc.pack_tensor(tc.TensorList(g, rows), T)
    assert torch.equal(T.view(want.dtype).view(want.shape), want), f"K={K} {dtype} shift={shift}: pack"
    back = _lists(RENUMBERED, K, dtype, shift)
    tc.unpack_tensor(tc.TensorList(g, back), T)
    for a, b in zip(back, rows):
        assert torch.equal(a[0]._base.view(want.dtype), b[0]._base.view(want.dtype)), f"K={K} {dtype} shift={shift}: unpack"


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("K,below", [(5, True), (5, False), (6, False), (7, True), (7, False)])
def test_large_bfloat16_pack(K, below, shift):
    """On both sides of 48 M elements of all copies, where K = 5 and 7 change
    their tile; every copy is its own bits, odd sizes and a partial slot."""
    n = (48 << 20) // K + (-5 if below else 262_147)
    cuts = np.sort(np.random.default_rng(K).choice(n, 500, replace=False))
    sizes = [int(v) for v in np.diff(np.concatenate([[0], cuts, [n]]))]
    g = tc.Group(sizes)
    assert (g.numel < -(-(48 << 20) // K)) == below
    rows, want = _interleaved(sizes, K, torch.bfloat16, shift, K)
    T = torch.zeros(tc.tensor_numel(g, K), dtype=torch.bfloat16, device=DEV)
    tc.pack_tensor(tc.TensorList(g, rows), T)
    assert torch.equal(T.view(torch.int16).view(want.shape), want), f"K={K} n={n} shift={shift}"


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("K", [1, 3, 8])
def test_separate_pack_and_unpack(K, dtype, shift, offset):
    """Flat copies: a wave's 256 or 512 elements, unpack and, from 256 to 4,096
    chunks (the last groups at K = 8), pack; flat buffers at any alignment."""
    whole = torch.int32 if dtype == torch.float32 else torch.int16
    rng = np.random.default_rng(7)
    odd = [int(v) for v in rng.integers(1, 3000, 100)]
    many = [int(v) for v in rng.integers(0, 12, 25_000)]
    for sizes in _groups() + [odd, many]:
        g = tc.Group(sizes)
        n = g.numel
        what = f"K={K} {dtype} shift={shift} offset={offset} n={n} in {len(sizes)}"
        rows, back = _lists(sizes, K, dtype, shift), _lists(sizes, K, dtype, shift)
        flats = [torch.zeros(n + 16, dtype=dtype, device=DEV) for _ in range(K)]
        want = []
        for k, row in enumerate(rows):
            bits = torch.randint(-2 ** 15, 2 ** 15, (n,), generator=torch.Generator(device=DEV).manual_seed(k), device=DEV)
            want.append(bits.to(whole))
            for t, v in zip(row, torch.split(want[-1], sizes)):
                t.view(whole).copy_(v)
        tc.pack(tc.TensorList(g, rows), [f[offset:offset + n] for f in flats])
        for f, w in zip(flats, want):
            assert torch.equal(f[offset:offset + n].view(whole), w), f"{what}: pack"
            assert not f[:offset].any() and not f[offset + n:].any(), f"{what}: beside the flat copy"
        tc.unpack(tc.TensorList(g, back), [f[offset:offset + n] for f in flats])
        for a, b in zip(back, rows):
            assert torch.equal(a[0]._base.view(whole), b[0]._base.view(whole)), f"{what}: unpack"
