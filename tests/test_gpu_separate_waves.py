"""The separate-buffer kernels, which split the copies of a 64-slot tile over
the waves of a workgroup: copies per wave change at K = 2/3, 6/7, 12/13/14/15,
16/17, 24/25 and 32/33, tiles end every 256 elements (512 for the bfloat16
reduction), and where a buffer is not aligned to a slot's bytes (16 of binary32,
8 of bfloat16) all of them are read and written with unaligned accesses.  Integer inputs with steps that are powers of two make every result
exact in binary32, so all of them are compared bit for bit with the oracle;
the grid past 2^31 threads is compared at sampled places.
"""

import numpy as np
import pytest
import torch

import oracle
import paper_1801_03855_amd as tc
from paper_1801_03855_amd import workloads as wl
from tests.helpers import assert_close, assert_exact, easgd_mags, host_f32, host_stored

pytestmark = pytest.mark.gpu

DEV = "cuda"
KS = [1, 2, 3, 5, 6, 7, 8, 12, 13, 14, 15, 16, 17, 23, 24, 25, 31, 32, 33, 63, 64]
# one element to a slot's edge, a tile's (256 and 512 elements), and several tiles
NS = [1, 3, 4, 255, 256, 257, 511, 513, 516, 4 * 64 * 5 + 2]


MIXED = "mixed"  # every buffer at another offset


def _buffers(values, offset):
    """Each as its own buffer, starting `offset` elements after an aligned address, in storage filled with 7."""
    out = []
    for i, v in enumerate(values):
        o = (3 * i + 1) % 8 if offset == MIXED else offset
        b = torch.full((v.numel() + 16,), 7.0, dtype=v.dtype, device=DEV)[o:o + v.numel()]
        b.copy_(v)
        out.append(b)
    return out


def _assert_nothing_beside(buffers, what):
    for i, b in enumerate(buffers):
        o, base = b.storage_offset(), b._base
        assert bool((base[:o] == 7).all()) and bool((base[o + b.numel():] == 7).all()), f"{what}: beside buffer {i}"


@pytest.mark.parametrize("offset", [0, 1, 2, MIXED])
@pytest.mark.parametrize("gdt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("K", KS)
def test_every_operation_exact(orc, K, gdt, offset):
    for N in NS:
        g = tc.Group([N])
        what = f"K={K} N={N} {gdt} offset={offset}"
        # |values| <= 128: bfloat16 gradients are exact too
        x0 = wl.integer_values(N, K, 128, seed=10 * K + N, device=DEV)
        g0 = [v.to(gdt) for v in wl.integer_values(N, K, 128, seed=20 * K + N, device=DEV)]
        c0 = wl.integer_values(N, 1, 128, seed=30 * K + N, device=DEV)
        h_x = [host_f32(v).astype(np.float64) for v in x0]
        h_g = [host_stored(v) for v in g0]
        h_c = host_f32(c0[0]).astype(np.float64)
        gs = _buffers(g0, offset)
        sums = orc.reduce(h_g, oracle.SUM)

        out = _buffers([torch.zeros(N)], offset)[0]
        tc.reduce(g, gs, out, "sum")
        assert_exact(host_f32(out), sums, f"{what}: sum")

        xs, xc = _buffers(x0, offset), _buffers(c0, offset)[0]
        xs2, xc2 = _buffers(x0, offset), _buffers(c0, offset)[0]
        tc.easgd_step(g, xs, gs, xc, 0.125, 0.5)
        out.zero_()
        tc.reduce_easgd_step(g, xs2, gs, xc2, out, 0.125, 0.5, "sum")
        rx, rc = [v.copy() for v in h_x], h_c.copy()
        orc.easgd_step(rx, h_g, rc, 0.125, 0.5)
        assert_exact(host_f32(out), sums, f"{what}: fused sum")
        for name, ws, c in (("step", xs, xc), ("fused", xs2, xc2)):
            assert_exact(host_f32(c), rc, f"{what}: {name} center")
            for i in range(K):
                assert_exact(host_f32(ws[i]), rx[i], f"{what}: {name} x[{i}]")
            _assert_nothing_beside([*ws, c, out], f"{what}: {name}")

        xs = _buffers(x0, offset)
        tc.sgd_step(g, xs, gs, 0.25)
        rx = [v.copy() for v in h_x]
        orc.sgd_step(rx, h_g, 0.25)
        for i in range(K):
            assert_exact(host_f32(xs[i]), rx[i], f"{what}: sgd x[{i}]")
        _assert_nothing_beside(xs, f"{what}: sgd")

        for bcast in (False, True) if gdt == torch.float32 else (False,):
            xs, gb = _buffers(x0, offset), _buffers(g0, offset)
            tc.sync_sgd_step(g, xs, gb, 0.5, 0.25, bcast)
            rx = [v.copy() for v in h_x]
            S = orc.sync_sgd(rx, h_g, 0.5, 0.25)
            for i in range(K):
                assert_exact(host_f32(xs[i]), rx[i], f"{what}: sync x[{i}]")
                assert np.array_equal(host_stored(gb[i]), S.astype(np.float32) if bcast else h_g[i]), f"{what}: g[{i}]"
            _assert_nothing_beside([*xs, *gb], f"{what}: sync")


@pytest.mark.parametrize("K", KS)
def test_bfloat16_gradients_on_an_8_byte_boundary(orc, K):
    """bfloat16 gradients 4 and 12 elements into a bucket, beside aligned
    binary32 buffers: slots of 8 bytes, two of which make no aligned 16."""
    for N in NS:
        g = tc.Group([N])
        what = f"K={K} N={N}"
        x0 = wl.integer_values(N, K, 128, seed=60 * K + N, device=DEV)
        g0 = [v.to(torch.bfloat16) for v in wl.integer_values(N, K, 128, seed=70 * K + N, device=DEV)]
        c0 = wl.integer_values(N, 1, 128, seed=80 * K + N, device=DEV)[0]
        h_g = [host_stored(v) for v in g0]
        gs = [_buffers([v], 4 if i % 2 == 0 else 12)[0] for i, v in enumerate(g0)]
        assert all(v.data_ptr() % 16 == 8 for v in gs)
        sums = orc.reduce(h_g, oracle.SUM)
        out = torch.zeros(N, device=DEV)
        tc.reduce(g, gs, out, "sum")
        assert_exact(host_f32(out), sums, f"{what}: sum")
        xs, xc = [v.clone() for v in x0], c0.clone()
        out.zero_()
        tc.reduce_easgd_step(g, xs, gs, xc, out, 0.125, 0.5, "sum")
        rx, rc = [host_f32(v).astype(np.float64) for v in x0], host_f32(c0).astype(np.float64)
        orc.easgd_step(rx, h_g, rc, 0.125, 0.5)
        assert_exact(host_f32(out), sums, f"{what}: fused sum")
        assert_exact(host_f32(xc), rc, f"{what}: center")
        for i in range(K):
            assert_exact(host_f32(xs[i]), rx[i], f"{what}: x[{i}]")


@pytest.mark.parametrize("offset", [0, MIXED])
@pytest.mark.parametrize("gdt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("K", range(2, 17))
def test_one_wave_for_all_copies(orc, K, gdt, offset):
    """The steps between 1.5 and 6 M elements of all copies (2.5 and 4.5 M from K =
    13 on) and the binary32 reduction between 3.3 and 8 M, where one wave takes
    every copy: the last size below, the first inside, an odd one, and the first
    above."""
    lo, hi = (1_500_000, 6_000_000) if K <= 12 else (2_500_000, 4_500_000)
    for N in (-(-lo // K) - 1, -(-lo // K), 3_400_000 // K | 1, -(-hi // K)):
        g = tc.Group([N])
        what = f"K={K} N={N} {gdt} offset={offset}"
        x0 = wl.integer_values(N, K, 128, seed=10 * K, device=DEV)
        g0 = [v.to(gdt) for v in wl.integer_values(N, K, 128, seed=20 * K, device=DEV)]
        c0 = wl.integer_values(N, 1, 128, seed=30 * K, device=DEV)
        h_g = [host_stored(v) for v in g0]
        gs = _buffers(g0, offset)
        sums = orc.reduce(h_g, oracle.SUM)
        rx, rc = [host_f32(v).astype(np.float64) for v in x0], host_f32(c0[0]).astype(np.float64)
        orc.easgd_step(rx, h_g, rc, 0.125, 0.5)
        out = _buffers([torch.zeros(N)], offset)[0]
        tc.reduce(g, gs, out, "sum")
        assert_exact(host_f32(out), sums, f"{what}: sum")
        for fused in (False, True):
            xs, xc = _buffers(x0, offset), _buffers(c0, offset)[0]
            if fused:
                out.zero_()
                tc.reduce_easgd_step(g, xs, gs, xc, out, 0.125, 0.5, "sum")
                assert_exact(host_f32(out), sums, f"{what}: fused sum")
            else:
                tc.easgd_step(g, xs, gs, xc, 0.125, 0.5)
            assert_exact(host_f32(xc), rc, f"{what}: center, fused={fused}")
            for i in range(K):
                assert_exact(host_f32(xs[i]), rx[i], f"{what}: x[{i}], fused={fused}")
            _assert_nothing_beside([*xs, xc, out], f"{what}: fused={fused}")
        bcast = gdt == torch.float32
        xs, gb = _buffers(x0, offset), _buffers(g0, offset)
        rx = [host_f32(v).astype(np.float64) for v in x0]
        S = orc.sync_sgd(rx, h_g, 0.5, 0.25)
        tc.sync_sgd_step(g, xs, gb, 0.5, 0.25, bcast)
        for i in range(K):
            assert_exact(host_f32(xs[i]), rx[i], f"{what}: sync x[{i}]")
            assert np.array_equal(host_stored(gb[i]), S.astype(np.float32) if bcast else h_g[i]), f"{what}: g[{i}]"
        _assert_nothing_beside([*xs, *gb], f"{what}: sync")


@pytest.mark.parametrize("offset", [0, 1, 2, MIXED])
@pytest.mark.parametrize("K,R", [(1, 1), (2, 2), (3, 2), (5, 5), (7, 6), (8, 0), (16, 6), (17, 6), (25, 1), (32, 6),
                                 (33, 6), (64, 6)])
def test_async_exact(orc, K, R, offset):
    """alpha = 1/4 and at most six exchanges: 7 bits and 2 more for each."""
    for N in NS:
        g = tc.Group([N])
        x0 = wl.integer_values(N, K, 128, seed=40 * K + N, device=DEV)
        c0 = wl.integer_values(N, 1, 128, seed=50 * K + N, device=DEV)
        order = [int(w) for w in np.random.default_rng(K + N).permutation(K)[:R]]
        xs, xc = _buffers(x0, offset), _buffers(c0, offset)[0]
        tc.elastic_async(g, xs, xc, order, 0.25)
        rx = [host_f32(v).astype(np.float64) for v in x0]
        rc = host_f32(c0[0]).astype(np.float64)
        orc.elastic_async(rx, rc, order, 0.25)
        assert_exact(host_f32(xc), rc, f"K={K} R={R} N={N} offset={offset}: center")
        for i in range(K):
            assert_exact(host_f32(xs[i]), rx[i], f"K={K} R={R} N={N} offset={offset}: x[{i}]")
        _assert_nothing_beside([*xs, xc], f"K={K} R={R} N={N} offset={offset}")


@pytest.mark.parametrize("offset", [0, MIXED])
@pytest.mark.parametrize("K,R", [(33, 33), (33, 9), (40, 16), (48, 17), (64, 63), (64, 64)])
def test_async_ahead_equals_one_at_a_time(orc, K, R, offset):
    """More than 32 workers: below 1 M elements eight exchanges' loads go ahead.
    The same elements, in a group of that size and in one just below, come out
    the same bits; a sample of them is compared with the oracle."""
    N = 1_000_000
    gen = torch.Generator(device=DEV).manual_seed(K + R)
    x0 = [torch.randn(N, generator=gen, device=DEV).mul_(0.05) for _ in range(K)]
    c0 = torch.randn(N, generator=gen, device=DEV).mul_(0.05)
    order = [int(w) for w in np.random.default_rng(R).permutation(K)[:R]]
    got = []
    for n in (N, N - 3):
        xs, xc = _buffers([v[:n] for v in x0], offset), _buffers([c0[:n]], offset)[0]
        tc.elastic_async(tc.Group([n]), xs, xc, order, 0.05)
        _assert_nothing_beside([*xs, xc], f"K={K} R={R} n={n}")
        got.append((xs, xc))
    for i in range(K):
        assert torch.equal(got[0][0][i][:N - 3], got[1][0][i]), f"K={K} R={R} x[{i}]"
    assert torch.equal(got[0][1][:N - 3], got[1][1]), f"K={K} R={R} center"
    at = torch.cat([torch.arange(500), torch.arange(N - 500, N - 3)]).to(DEV)
    rx, rc = [host_f32(v[at]).astype(np.float64) for v in x0], host_f32(c0[at]).astype(np.float64)
    mag = np.abs(rc) + sum(np.abs(v) for v in rx)
    orc.elastic_async(rx, rc, order, float(np.float32(0.05)))
    assert_close(host_f32(got[1][1][at]), rc, mag, "center")
    for i in range(K):
        assert_close(host_f32(got[1][0][i][at]), rx[i], mag, f"x[{i}]")


def test_grid_past_2_31_threads(orc):
    """K = 12: 256 elements per 768 lanes, so 720 M elements are more than 2^31
    threads and the grid goes on along y (byte offsets still fit 32 bits)."""
    K, N, eta, rho = 12, 720_000_001, 0.05, 2.25
    g = tc.Group([N])
    gen = torch.Generator(device=DEV).manual_seed(3)
    x0 = torch.randn(N + 1, generator=gen, device=DEV).mul_(0.05)[1:]
    g0 = torch.randn(N + 1, generator=gen, device=DEV).mul_(0.01)[1:]
    xs = []
    for i in range(K):
        xs.append(torch.empty(N + 1, device=DEV)[1:])
        torch.add(x0, 0.001 * i, out=xs[-1])
    gs = [g0] * K
    xc = x0.clone().resize_(N + 1)[1:]
    xc.copy_(x0)
    at = torch.from_numpy(np.unique(np.concatenate([np.random.default_rng(4).integers(0, N, 100_000), np.arange(64),
                                                    np.arange(N - 64, N), np.arange(2 ** 31 // 3 - 512, 2 ** 31 // 3 + 512)])))
    h_x, h_c, h_g = [host_f32(t[at]) for t in xs], host_f32(xc[at]), [host_f32(g0[at])] * K
    tc.easgd_step(g, xs, gs, xc, eta, rho)
    torch.cuda.synchronize()
    rx, rc = [v.astype(np.float64) for v in h_x], h_c.astype(np.float64)
    mx, mc = easgd_mags(h_x, h_g, h_c, eta, rho)
    orc.easgd_step(rx, h_g, rc, eta, rho)
    for i in range(K):
        assert_close(host_f32(xs[i][at]), rx[i], mx[i], f"x[{i}]")
    assert_close(host_f32(xc[at]), rc, mc, "center")
