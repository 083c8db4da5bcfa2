"""The one-call step at the edges of its tiles: 64 or 32 slots per workgroup
(by K and gradient type), lists at any alignment, tiles that lie in one tensor,
in a few and in more than 32, zero-size tensors, and the last, partial slot.
Bit for bit the four calls' results, which other tests hold to the oracle.
"""

import numpy as np
import pytest
import torch

import paper_1801_03855_amd as tc

pytestmark = pytest.mark.gpu

DEV = "cuda"
KS = [1, 2, 3, 4, 7, 8, 9, 13, 14, 15, 16, 17, 24, 31, 32, 33]
# 120 odd sizes, 600,011 elements: from 262,144 / K elements on (of bfloat16
# lists twice that), the tiles are renumbered in runs, the last one not full
RENUMBERED = [int(v) for v in np.random.default_rng(2).integers(1, 8_000, 119)]
RENUMBERED.append(600_011 - sum(RENUMBERED))


def _groups():
    rng = np.random.default_rng(1)
    one = [[n] for n in (1, 3, 4, 127, 128, 129, 255, 256, 257, 260, 511, 1027)]
    tiny = [int(v) for v in rng.integers(0, 6, 700)]          # more than 32 tensors to a tile, zeros among them
    few = [130, 0, 0, 61, 66, 255, 1, 513, 4, 97, 0]
    large = [1024, 64, 260, 2048 + 4, 8]                     # every boundary on a slot
    # long runs of zero-size tensors inside a slot, and where a slot ends
    empties = [5] + [0] * 40 + [2] + [0] * 90 + [1] + [0] * 35 + [1] + [0] * 37 + [3, 250, 0, 129]
    return one + [tiny, few, large, empties]


def _lists(sizes, K, dtype, shift):
    """Per-layer tensors of every copy; tensor t of copy k starts `shift * (k + t)` elements past an aligned place."""
    out = []
    for k in range(K):
        buf = torch.zeros(sum(s + 24 for s in sizes), dtype=dtype, device=DEV)
        at, row = 0, []
        for t, s in enumerate(sizes):
            at = -(-at // 8) * 8
            d = shift * (k + t) % 8
            row.append(buf[at + d:at + d + s])
            at += d + s
        out.append(row)
    return out


def _check(sizes, K, gdt, shift, gen):
    g = tc.Group(sizes)
    n, m = g.numel, tc.tensor_numel(g, K)
    gl, pl, pl2 = _lists(sizes, K, gdt, shift), _lists(sizes, K, torch.float32, shift), _lists(sizes, K, torch.float32, shift)
    for row in gl:
        for t in row:
            t.copy_(torch.randn(t.shape, generator=gen, device=DEV) * 0.01)
    grads, params, params2 = tc.TensorList(g, gl), tc.TensorList(g, pl), tc.TensorList(g, pl2)
    x = torch.randn(m, generator=gen, device=DEV) * 0.05
    xc = torch.randn(n, generator=gen, device=DEV) * 0.05
    x2, xc2 = x.clone(), xc.clone()
    G, G2 = (torch.zeros(m, dtype=gdt, device=DEV) for _ in range(2))
    mean, mean2 = (torch.zeros(n, device=DEV) for _ in range(2))
    tc.pack_tensor(grads, G)
    tc.reduce_tensor(g, K, G, mean, "avg")
    tc.easgd_step_tensor(g, K, x, G, xc, 0.05, 2.25)
    tc.unpack_tensor(params, x)
    x3, xc3 = x2.clone(), xc2.clone()
    tc.easgd_pipeline_tensor(grads, params2, G2, mean2, x2, xc2, 0.05, 2.25)
    what = f"K={K} {gdt} shift={shift} n={n} in {len(sizes)}"
    flat = lambda rows: torch.cat([t for row in rows for t in row])  # noqa: E731
    for name, a, b in (("packed gradients", G2, G), ("average", mean2, mean), ("workers", x2, x), ("center", xc2, xc),
                       ("parameters", flat(pl2), flat(pl))):
        assert torch.equal(a, b), f"{what}: {name}"
    # nothing around the parameters is written
    assert all(torch.equal(a[0]._base, b[0]._base) for a, b in zip(pl, pl2) if a), f"{what}: beside the parameters"
    # the packed gradients left out: the parameters are written again, and
    # nothing around them
    mean2.zero_()
    for a, b in zip(pl, pl2):  # 7 everywhere, in the expected storage outside the tensors
        b[0]._base.fill_(7.0)
        values = [t.clone() for t in a]
        a[0]._base.fill_(7.0)
        for t, v in zip(a, values):
            t.copy_(v)
    tc.easgd_pipeline_tensor(grads, params2, None, mean2, x3, xc3, 0.05, 2.25)
    assert torch.equal(mean2, mean) and torch.equal(x3, x) and torch.equal(xc3, xc), f"{what}: not packed"
    assert all(torch.equal(a[0]._base, b[0]._base) for a, b in zip(pl, pl2)), f"{what}: parameters, not packed"


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("gdt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("K", KS)
def test_tiles_equal_the_four_calls(K, gdt, shift):
    gen = torch.Generator(device=DEV).manual_seed(100 * K + shift)
    for sizes in _groups():
        _check(sizes, K, gdt, shift, gen)


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("gdt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("K", [1, 2, 4, 8, 13, 16, 17, 24, 32])
def test_renumbered_tiles(K, gdt, shift):
    _check(RENUMBERED, K, gdt, shift, torch.Generator(device=DEV).manual_seed(200 * K + shift))
