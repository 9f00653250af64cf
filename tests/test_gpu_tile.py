"""The tile contraction of stride-1 rulebooks (forward and input gradient) and
the weight gradient at the sizes where it can go wrong: rows around the tile of 64 and the work-group
of 256, both its kernels (four waves on one tile; four tiles sharing their
weights), pair lists and the mask-sorted view, channel counts around the
16-channel step and the 64-column block, and operands that the bf16 split
cannot hold.

Reference: the sums in float64 over the rulebook's own pair lists.  Bound: a
sum of n products, each rounded once and added in any order, is off by at most
(n + 4) 2^-24 sum |terms|; x - g_in is rounded before it (one more), and the
dropped products of the split stay below 2^-24 of their term."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gen import random_sites, stream_rng  # noqa: E402

from helpers import dev, host  # noqa: E402

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


@pytest.fixture()
def scn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1505_02890_amd as m
    m.lib()
    yield m
    m.set_dense_forward()


def _layer(scn, f, m, n, cin, cout, seed, shuffle=True):
    rng = stream_rng(seed, 7)
    c = random_sites(rng, 1, (m, m, m), n, shuffle=shuffle)
    rb = scn.build_rulebook(dev(c), (1, m, m, m), f, 1)
    x = rng.standard_normal((n, cin)).astype(np.float32)
    g = rng.standard_normal(cin).astype(np.float32)
    W = (rng.standard_normal((rb.K, cin, cout)) * 0.1).astype(np.float32)
    b = rng.standard_normal(cout).astype(np.float32)
    _, ir, orr = (t.long().cpu() for t in rb.export())
    return rb, x, g, W, b, ir, orr


def _forward(rb, ir, orr, x, g, W, b):
    """(y, sum of |terms|) in float64 on the CPU"""
    d = [torch.from_numpy(np.asarray(a, np.float64)) for a in (x - g, x.astype(np.float64) - g, g,
                                                               W, b)]
    y = torch.zeros(rb.a_out, W.shape[2], dtype=torch.float64)
    s = torch.zeros_like(y)
    pre, spre = d[4].clone(), d[4].abs()
    for k in range(rb.K):
        i, o = ir[rb.offsets[k]:rb.offsets[k + 1]], orr[rb.offsets[k]:rb.offsets[k + 1]]
        y.index_add_(0, o, d[1][i] @ d[3][k])
        s.index_add_(0, o, d[1][i].abs() @ d[3][k].abs())
        pre += d[2] @ d[3][k]
        spre += d[2].abs() @ d[3][k].abs()
    return (y + pre).numpy(), (s + spre).numpy()


def _check(got, want, mass, terms):
    err = np.abs(got.astype(np.float64) - want)
    assert np.all(err <= (terms + 8) * U * mass + 1e-30), float(np.max(err / (mass + 1e-30)) / U)


SIZES = [
    # f, m, n, cin, cout, dense view
    (2, 9, 1, 16, 16, False), (2, 9, 2, 1, 1, False), (1, 9, 64, 16, 64, False),
    (1, 9, 63, 32, 65, False), (1, 9, 65, 48, 3, False), (1, 17, 255, 33, 64, False),
    (1, 17, 257, 17, 100, True), (3, 12, 300, 64, 64, False), (3, 12, 300, 64, 64, True),
    (3, 10, 500, 15, 31, True), (2, 14, 1000, 160, 96, False), (2, 14, 1000, 176, 256, True),
    # enough tiles for the shared-weights kernel, forward and input gradient
    (2, 48, 20000, 32, 130, False), (2, 48, 20000, 80, 130, True), (2, 60, 45001, 192, 16, False),
    (2, 60, 45001, 200, 40, True), (1, 60, 131073, 16, 8, False), (1, 60, 131009, 7, 5, True),
]


@pytest.mark.parametrize("case", SIZES)
def test_tile_sizes(scn, case):
    f, m, n, cin, cout, view = case
    scn.set_dense_forward(0 if view else 1 << 40, 1)
    rb, x, g, W, b, ir, orr = _layer(scn, f, m, n, cin, cout, 11, shuffle=n % 2 == 1)
    assert rb.dense_view == (view and rb.a_out > 0)
    y, _ = scn.conv_fwd(rb, dev(x), dev(g), dev(W), dev(b))
    want, mass = _forward(rb, ir, orr, x, g, W, b)
    _check(host(y), want, mass, rb.K * cin)
    rng = stream_rng(12, 1)
    dy = rng.uniform(-1, 1, (rb.a_out, cout)).astype(np.float32)
    dx = scn.conv_bwd(rb, dev(x), dev(g), dev(W), None, None, dev(dy), need=("dx",))["dx"]
    dy64, W64 = torch.from_numpy(dy).double(), torch.from_numpy(W).double()
    want = torch.zeros(n, cin, dtype=torch.float64)
    mass = torch.zeros_like(want)
    for k in range(rb.K):
        i, o = ir[rb.offsets[k]:rb.offsets[k + 1]], orr[rb.offsets[k]:rb.offsets[k + 1]]
        want.index_add_(0, i, dy64[o] @ W64[k].t())
        mass.index_add_(0, i, dy64[o].abs() @ W64[k].t().abs())
    _check(host(dx), want.numpy(), mass.numpy(), rb.K * cout)


@pytest.mark.parametrize("big", [False, True])
@pytest.mark.parametrize("view", [False, True])
def test_values_past_the_split(scn, view, big):
    """Infinities, NaN and floats that round past bf16's largest value: the
    same entries are infinite and NaN as in fp32, and the others as close as
    ever.  Values whose low parts are subnormal in bf16 lose no more than
    those parts (2^-126 at most per factor)."""
    scn.set_dense_forward(0 if view else 1 << 40, 1)
    n, cout = (20000, 130) if big else (900, 40)
    rb, x, g, W, b, ir, orr = _layer(scn, 2, 48 if big else 14, n, 32, cout, 21)
    g[:] = 0
    W = (np.abs(W) + 0.01).astype(np.float32)
    for r, v in ((3, np.inf), (100, -np.inf), (200, np.nan), (300, 3.4e38), (400, -3.402e38),
                 (500, 1e-37), (600, 3e38)):
        x[r, r % 32] = v
    W[:, 300 % 32] *= 1e-3  # 3.4e38 itself stays in range
    with np.errstate(all="ignore"):
        want, mass = _forward(rb, ir, orr, x, g, W, b)
        f32 = want.astype(np.float32)
    y = host(scn.conv_fwd(rb, dev(x), dev(g), dev(W), dev(b))[0])
    assert np.array_equal(np.isnan(y), np.isnan(want))
    assert np.array_equal(np.isinf(y), np.isinf(f32))
    assert np.array_equal(y[np.isinf(y)], f32[np.isinf(y)])
    ok = np.isfinite(f32) & np.isfinite(mass)
    _check(y[ok], want[ok], mass[ok], rb.K * 32)


def _weight_gradient(rb, ir, orr, x, g, dy):
    """(dW, sum of |terms|) in float64; dW = sum (x - g)^T dy + g^T sum dy"""
    xs, d = torch.from_numpy(x.astype(np.float64) - g), torch.from_numpy(dy.astype(np.float64))
    g64 = torch.from_numpy(g.astype(np.float64))
    dW = torch.zeros(rb.K, x.shape[1], dy.shape[1], dtype=torch.float64)
    mass = torch.zeros_like(dW)
    for k in range(rb.K):
        i, o = ir[rb.offsets[k]:rb.offsets[k + 1]], orr[rb.offsets[k]:rb.offsets[k + 1]]
        dW[k] = xs[i].t() @ d[o] + torch.outer(g64, d.sum(0))
        mass[k] = xs[i].abs().t() @ d[o].abs() + torch.outer(g64.abs(), d.abs().sum(0))
    return dW.numpy(), mass.numpy()


@pytest.mark.parametrize("case", [
    # f, s, m, n, cin, cout: one pair, around a stage of 16 and four waves of
    # them, several chunks, quads and single floats, several blocks
    (1, 1, 9, 1, 4, 4), (1, 1, 9, 15, 64, 64), (1, 1, 9, 16, 1, 1), (1, 1, 9, 17, 65, 64),
    (1, 1, 9, 63, 16, 130), (1, 1, 9, 64, 3, 5), (1, 1, 9, 65, 128, 68), (2, 1, 14, 1000, 33, 34),
    (3, 1, 40, 30000, 64, 60), (3, 2, 12, 300, 32, 96), (2, 2, 30, 5000, 7, 64),
    (1, 1, 60, 131073, 8, 12),
])
def test_weight_gradient_sizes(scn, case):
    f, s, m, n, cin, cout = case
    rng = stream_rng(31, 7)
    c = random_sites(rng, 1, (m, m, m), n, shuffle=True)
    rb = scn.build_rulebook(dev(c), (1, m, m, m), f, s)
    x = rng.standard_normal((n, cin)).astype(np.float32)
    g = rng.standard_normal(cin).astype(np.float32)
    W = rng.standard_normal((rb.K, cin, cout)).astype(np.float32)
    dy = rng.uniform(-1, 1, (rb.a_out, cout)).astype(np.float32)
    _, ir, orr = (t.long().cpu() for t in rb.export())
    got = scn.conv_bwd(rb, dev(x), dev(g), dev(W), None, None, dev(dy))
    want, mass = _weight_gradient(rb, ir, orr, x, g, dy)
    _check(host(got["dW"]), want, mass, max(rb.n_pairs // rb.K, 1))
    # special values reach exactly the entries they reach in fp32
    x[0, cin - 1] = np.inf
    dy[rb.a_out - 1, 0] = -3.402e38
    with np.errstate(all="ignore"):
        want, mass = _weight_gradient(rb, ir, orr, x, g, dy)
    got = host(scn.conv_bwd(rb, dev(x), dev(g), dev(W), None, None, dev(dy))["dW"])
    ok = np.isfinite(want) & (np.abs(mass) < 3e38)
    assert not np.any(np.isfinite(got) & np.isinf(want))
    assert np.array_equal(np.isnan(got[ok]), np.isnan(want[ok]))
    _check(got[ok], want[ok], mass[ok], max(rb.n_pairs // rb.K, 1))


@pytest.mark.parametrize("view", [False, True])
@pytest.mark.parametrize("case", [
    # f, m, n, cin, cout: reductions of 1, 8, 16, 27, 32, 54, 64.. entries (one
    # to three tiles of 32), one tile, ragged tiles, more tiles than waves
    (1, 9, 1, 1, 4), (2, 9, 40, 1, 64), (2, 12, 700, 2, 33), (3, 14, 900, 1, 130),
    (2, 16, 1500, 4, 64), (3, 12, 500, 2, 64), (3, 14, 700, 3, 60), (2, 64, 60000, 1, 32),
    (3, 30, 3000, 1, 64),
])
def test_few_channels(scn, case, view):
    """First layers: the forward, and the weight and bias gradients alone
    (which take another path than all gradients together)."""
    f, m, n, cin, cout = case
    scn.set_dense_forward(0 if view else 1 << 40, 1)
    rb, x, g, W, b, ir, orr = _layer(scn, f, m, n, cin, cout, 41)
    y, go = scn.conv_fwd(rb, dev(x), dev(g), dev(W), dev(b), relu=True)
    want, mass = _forward(rb, ir, orr, x, g, W, b)
    _check(host(y), np.maximum(want, 0), mass, rb.K * cin)
    rng = stream_rng(43, 1)
    dy = rng.uniform(-1, 1, (rb.a_out, cout)).astype(np.float32)
    dg = rng.uniform(-1, 1, cout).astype(np.float32)
    for relu in (False, True):
        args = (rb, dev(x), dev(g), dev(W), y, go, dev(dy), dev(dg))
        got = scn.conv_bwd(*args, relu=relu, need=("dW", "dbias"))
        again = scn.conv_bwd(*args, relu=relu, need=("dW", "dbias"))
        assert torch.equal(got["dW"], again["dW"]) and torch.equal(got["dbias"], again["dbias"])
        d = dy * (host(y) > 0) if relu else dy
        dgr = dg * (host(go) > 0) if relu else dg
        want, mass = _weight_gradient(rb, ir, orr, x, g, d)
        gd = np.outer(g, dgr.astype(np.float64))
        _check(host(got["dW"]), want + gd, mass + np.abs(gd), rb.a_out)
        s64 = d.astype(np.float64)
        _check(host(got["dbias"]), s64.sum(0) + dgr, np.abs(s64).sum(0) + np.abs(dgr), rb.a_out)
    # special values
    x[n // 2, cin - 1] = np.inf
    dy[rb.a_out // 2, cout - 1] = np.nan
    with np.errstate(all="ignore"):
        want, mass = _forward(rb, ir, orr, x, g, W, b)
        got = host(scn.conv_fwd(rb, dev(x), dev(g), dev(W), dev(b))[0])
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.array_equal(got[np.isinf(got)], want[np.isinf(want)])
        want, mass = _weight_gradient(rb, ir, orr, x, g, dy)
        got = host(scn.conv_bwd(rb, dev(x), dev(g), dev(W), None, None, dev(dy),
                                need=("dW", "dbias"))["dW"])
    ok = np.isfinite(want)
    assert not np.any(np.isfinite(got) & ~ok)
    _check(got[ok], want[ok], mass[ok], rb.a_out)


@pytest.mark.parametrize("big", [False, True])
@pytest.mark.parametrize("view", [False, True])
@pytest.mark.parametrize("c", [4, 5, 7, 19, 20, 31, 33, 35, 60, 61])
def test_ragged_rows(scn, c, view, big):
    """Rows whose channels divide nothing, from pointers that are 4-byte
    aligned only: forward (with and without allocations: the same bits) and
    input gradient.  The next row's channels are NaN at the ends, so a read
    past a row shows."""
    n, m = (70000, 60) if big else (700, 14)
    scn.set_dense_forward(0 if view else 1 << 40, 1)
    rb, x, g, W, b, ir, orr = _layer(scn, 2, m, n, c, 24, 51)
    buf = torch.full((n * c + 8,), float("nan"), device="cuda")
    for at in (1, 4):
        xd = buf[at:at + n * c].view(n, c)
        xd.copy_(dev(x))
        assert xd.is_contiguous()
        y, _ = scn.conv_fwd(rb, xd, dev(g), dev(W), dev(b))
        again, _ = scn.conv_fwd(rb, xd, dev(g), dev(W), dev(b), noalloc=True)
        assert torch.equal(y, again)
        want, mass = _forward(rb, ir, orr, x, g, W, b)
        _check(host(y), want, mass, rb.K * c)
        buf.fill_(float("nan"))
    Wt = np.ascontiguousarray(W.transpose(0, 2, 1))  # [K][24][c]: dy has c channels
    dy = stream_rng(53, 1).uniform(-1, 1, (rb.a_out, c)).astype(np.float32)
    dbuf = torch.full((rb.a_out * c + 8,), float("nan"), device="cuda")
    dyd = dbuf[3:3 + rb.a_out * c].view(rb.a_out, c)
    dyd.copy_(dev(dy))
    x24 = torch.zeros(n, 24, device="cuda")
    dx = scn.conv_bwd(rb, x24, torch.zeros(24, device="cuda"), dev(Wt), None, None, dyd,
                      need=("dx",))["dx"]
    dy64, W64 = torch.from_numpy(dy).double(), torch.from_numpy(Wt).double()
    want, mass = torch.zeros(n, 24, dtype=torch.float64), torch.zeros(n, 24, dtype=torch.float64)
    for k in range(rb.K):
        i, o = ir[rb.offsets[k]:rb.offsets[k + 1]], orr[rb.offsets[k]:rb.offsets[k + 1]]
        want.index_add_(0, i, dy64[o] @ W64[k].t())
        mass.index_add_(0, i, dy64[o].abs() @ W64[k].t().abs())
    _check(host(dx), want.numpy(), mass.numpy(), rb.K * c)


@pytest.mark.parametrize("cout", [1, 2, 3])
def test_input_gradient_of_few_outputs(scn, cout):
    """Output gradients of one to three channels."""
    n = 3000
    rb, x, g, W, b, ir, orr = _layer(scn, 2, 20, n, 40, cout, 55)
    dy = stream_rng(56, 1).uniform(-1, 1, (rb.a_out, cout)).astype(np.float32)
    dx = scn.conv_bwd(rb, dev(x), dev(g), dev(W), None, None, dev(dy), need=("dx",))["dx"]
    dy64, W64 = torch.from_numpy(dy).double(), torch.from_numpy(W).double()
    want, mass = torch.zeros(n, 40, dtype=torch.float64), torch.zeros(n, 40, dtype=torch.float64)
    for k in range(rb.K):
        i, o = ir[rb.offsets[k]:rb.offsets[k + 1]], orr[rb.offsets[k]:rb.offsets[k + 1]]
        want.index_add_(0, i, dy64[o] @ W64[k].t())
        mass.index_add_(0, i, dy64[o].abs() @ W64[k].t().abs())
    _check(host(dx), want.numpy(), mass.numpy(), rb.K * cout)


def test_ragged_channels_take_no_more_memory(scn):
    """A channel count that is no multiple of 16 asks for no more device
    memory than the next one that is: rows are not copied to be padded."""
    rb, *_ = _layer(scn, 2, 60, 30000, 1, 1, 57)
    from paper_1505_02890_amd import _lib
    for c in (5, 35, 50, 100):
        up = -(-c // 16) * 16
        ws = [_lib.lib().scn_conv_bwd_workspace_bytes(rb.handle, 64, v, 0) for v in (c, up)]
        assert ws[0] <= ws[1], (c, ws)
    asked = []

    def alloc(nbytes, stream):
        asked.append(nbytes)
        return torch.cuda.caching_allocator_alloc(int(nbytes), stream=int(stream))

    def free(ptr, stream):
        torch.cuda.caching_allocator_delete(int(ptr))

    try:
        scn.set_allocator(alloc, free)
        for c in (35, 48):
            z = torch.zeros(c, device="cuda")
            scn.conv_fwd(rb, torch.zeros(rb.a_in, c, device="cuda"), z,
                         torch.zeros(rb.K, c, 48, device="cuda"))
            asked.append(0)
    finally:
        torch.cuda.synchronize()
        scn.set_allocator()
    cut = asked.index(0)
    assert sum(asked[:cut]) <= sum(asked[cut:])


@pytest.mark.parametrize("case", [
    # f, m, n, cin, cout, view: sparse lists from pairs (fill below 0.4, past
    # 5500 full steps) and, just short of that, in tiles; the view's narrow
    # layers (odd steps, rows off 64 bytes, 32 channels and few offsets) and
    # their neighbours; full masks
    (3, 40, 5000, 64, 64, False), (3, 40, 1200, 64, 64, False), (3, 24, 9000, 40, 70, False),
    (2, 40, 20000, 61, 128, False), (2, 12, 1728, 64, 64, False),
    (2, 30, 3000, 16, 64, True), (2, 30, 3000, 20, 33, True), (2, 30, 3000, 32, 64, True),
    (3, 20, 700, 32, 64, True), (2, 30, 3000, 32, 65, True), (2, 30, 3000, 48, 64, True),
    (2, 30, 3000, 60, 20, True), (2, 30, 3000, 64, 64, True), (2, 30, 3000, 68, 8, True),
    (2, 30, 3000, 84, 8, True), (2, 30, 3000, 100, 64, True), (2, 30, 3000, 112, 64, True),
    (2, 30, 3000, 132, 64, True), (2, 30, 3000, 19, 64, True), (3, 20, 700, 3, 32, True),
    (3, 20, 700, 3, 65, True), (3, 20, 700, 4, 64, True), (3, 10, 1000, 3, 40, True),
    (2, 12, 1728, 16, 64, True), (2, 12, 1728, 3, 64, True), (2, 12, 1728, 4, 40, True),
])
def test_routes(scn, case):
    """Forwards on either side of the lines between the kernels, from aligned
    rows and from rows that are not."""
    f, m, n, cin, cout, view = case
    scn.set_dense_forward(0 if view else 1 << 40, 1)
    rb, x, g, W, b, ir, orr = _layer(scn, f, m, n, cin, cout, 61)
    assert rb.dense_view == view
    want, mass = _forward(rb, ir, orr, x, g, W, b)
    buf = torch.empty(n * cin + 4, device="cuda")
    gbuf = torch.empty(cin + 1, device="cuda")
    gd = gbuf[1:]
    gd.copy_(dev(g))
    for at in (0, 1):
        xd = buf[at:at + n * cin].view(n, cin)
        xd.copy_(dev(x))
        for relu in (False, True):
            y, go = scn.conv_fwd(rb, xd, gd, dev(W), dev(b), relu=relu)
            again, _ = scn.conv_fwd(rb, xd, gd, dev(W), dev(b), relu=relu, noalloc=True)
            assert torch.equal(y, again)
            _check(host(y), np.maximum(want, 0) if relu else want, mass, rb.K * cin)
    # an infinite first channel (padding of short rows may read it)
    x[n // 2, 0] = np.inf
    with np.errstate(all="ignore"):
        want, _ = _forward(rb, ir, orr, x, g, W, b)
    got = host(scn.conv_fwd(rb, dev(x), dev(g), dev(W), dev(b))[0])
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(got[np.isinf(got)], want[np.isinf(want)])


def _rms(a):
    return float(np.sqrt(np.mean(np.square(np.asarray(a, np.float64)))))


@pytest.mark.parametrize("view", [False, True])
def test_few_channels_rounding(scn, view):
    """First layers of one and three channels: the rms error of the forward and
    of a weight gradient without cancellation is within one half unit in the
    last place of the rms result, 2^-24.  (A last rounding alone gives 0.43 of
    that; sums that truncate with every product of the matrix core, or add
    hundreds of partial sums in 32 bits, come to 1.2 to 1.5.)"""
    scn.set_dense_forward(0 if view else 1 << 40, 1)
    for f, m, n, cin, cout in ((3, 60, 40000, 1, 64), (3, 12, 1500, 2, 64), (2, 30, 20000, 2, 32)) + \
            (() if view else ((3, 60, 40000, 3, 64),)):
        rb, x, g, W, b, ir, orr = _layer(scn, f, m, n, cin, cout, 71)
        g[:] = 0
        b[:] = 0
        y = host(scn.conv_fwd(rb, dev(x), dev(g), dev(W), dev(b))[0])
        want, _ = _forward(rb, ir, orr, x, g, W, b)
        assert _rms(y - want) <= U * _rms(want), (f, n, cin)
        x = np.abs(x)
        dy = stream_rng(73, 1).uniform(0, 1, (rb.a_out, cout)).astype(np.float32)
        got = scn.conv_bwd(rb, dev(x), dev(g), dev(W), None, None, dev(dy), need=("dW", "dbias"))
        want, _ = _weight_gradient(rb, ir, orr, x, g, dy)
        assert _rms(host(got["dW"]) - want) <= U * _rms(want), (f, n, cin)


@pytest.mark.parametrize("case", [(4, 4), (5, 61), (35, 50), (64, 66), (67, 129), (130, 7)])
def test_weight_gradient_ragged(scn, case):
    """Channel counts that divide nothing, from pointers that are 4-byte aligned
    only, with NaN around the tensors."""
    cin, cout = case
    n = 2100
    rb, x, g, W, b, ir, orr = _layer(scn, 2, 22, n, cin, cout, 81)
    dy = stream_rng(82, 1).uniform(-1, 1, (rb.a_out, cout)).astype(np.float32)
    want, mass = _weight_gradient(rb, ir, orr, x, g, dy)

    def odd(a):
        buf = torch.full((a.size + 8,), float("nan"), device="cuda")
        v = buf[3:3 + a.size].view(*a.shape)
        v.copy_(dev(a))
        return v

    got = scn.conv_bwd(rb, odd(x), odd(g), dev(W), None, None, odd(dy))
    _check(host(got["dW"]), want, mass, max(rb.n_pairs // rb.K, 1))


# Near-full grids: lists full enough for the tile kernels, 2000 rows for the one
# that shares a tile among four waves, 68000 for the one that shares weights.
GRIDS = {"split": (13, 2000), "wg": (41, 68000)}


def _dx_reference(rb, ir, orr, W, dy):
    d, W64 = torch.from_numpy(dy).double(), torch.from_numpy(W).double()
    dx = torch.zeros(rb.a_in, W.shape[1], dtype=torch.float64)
    for k in range(rb.K):
        i, o = ir[rb.offsets[k]:rb.offsets[k + 1]], orr[rb.offsets[k]:rb.offsets[k + 1]]
        dx.index_add_(0, i, d[o] @ W64[k].t())
    return dx.numpy()


@pytest.mark.parametrize("c", [16, 32, 35, 64, 80, 96])
@pytest.mark.parametrize("grid", ["split", "wg"])
@pytest.mark.parametrize("view", [False, True])
def test_tile_precision(scn, c, grid, view):
    """Forward, input gradient and weight gradient against 64-bit sums, as rms:
    within eight units of 2^-24.  A kernel that lost one of the six products
    would be off by 30 or more (test_split_products)."""
    m, n = GRIDS[grid]
    scn.set_dense_forward(0 if view else 1 << 40, 1)
    rb, x, g, W, b, ir, orr = _layer(scn, 2, m, n, c, 64, 91)
    want, _ = _forward(rb, ir, orr, x, g, W, b)
    y = host(scn.conv_fwd(rb, dev(x), dev(g), dev(W), dev(b))[0])
    assert _rms(y - want) <= 8 * U * _rms(want)
    Wt = np.ascontiguousarray(W.transpose(0, 2, 1))  # dy has c channels
    x64 = stream_rng(92, 1).standard_normal((n, 64)).astype(np.float32)
    dy = stream_rng(93, 1).standard_normal((rb.a_out, c)).astype(np.float32)
    z = np.zeros(64, np.float32)
    got = scn.conv_bwd(rb, dev(x64), dev(z), dev(Wt), None, None, dev(dy))
    want = _dx_reference(rb, ir, orr, Wt, dy)
    assert _rms(host(got["dx"]) - want) <= 8 * U * _rms(want)
    want, _ = _weight_gradient(rb, ir, orr, x64, z, dy)
    assert _rms(host(got["dW"]) - want) <= 8 * U * _rms(want)


@pytest.mark.parametrize("grid", ["split", "wg"])
@pytest.mark.parametrize("view", [False, True])
@pytest.mark.parametrize("c", [35, 64])
def test_special_values_stay_local(scn, c, grid, view):
    """An infinity, a NaN and a value past bf16's range in the rows or weights of
    each contraction: the results that they enter are as in fp32, all others
    keep their bits."""
    m, n = GRIDS[grid]
    scn.set_dense_forward(0 if view else 1 << 40, 1)
    rb, x, g, W, b, ir, orr = _layer(scn, 2, m, n, c, 64, 95)
    g[:] = 0
    special = ((n // 7, 3, np.inf), (n // 3, c - 1, np.nan), (n // 2, 0, 3.4e38))
    W = (np.abs(W) + 0.01).astype(np.float32) * np.float32(0.01)

    def same(got, plain, want, reached):
        f32 = want.astype(np.float32)
        assert np.array_equal(got[~reached], plain[~reached])
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.array_equal(got[np.isinf(got)], f32[np.isinf(f32)])
        ok = reached & np.isfinite(f32)
        # what is finite here has 3.4e38 in it, which dwarfs its other terms
        assert np.allclose(got[ok], want[ok], rtol=1e-5, atol=0)

    def hit(rows_in, rows_out, num):
        """outputs that take any of the special rows"""
        r = np.zeros(num, bool)
        src = np.zeros(max(rb.a_in, rb.a_out), bool)
        src[[s[0] for s in special]] = True
        r[rows_out.numpy()[src[rows_in.numpy()]]] = True
        return r

    with np.errstate(all="ignore"):
        plain = host(scn.conv_fwd(rb, dev(x), dev(g), dev(W), dev(b))[0])
        xs = x.copy()
        for r, ch, v in special:
            xs[r, ch] = v
        want, _ = _forward(rb, ir, orr, xs, g, W, b)
        got = host(scn.conv_fwd(rb, dev(xs), dev(g), dev(W), dev(b))[0])
        same(got, plain, want, np.repeat(hit(ir, orr, rb.a_out)[:, None], 64, 1))

        Wt = np.ascontiguousarray(W.transpose(0, 2, 1))
        x64 = stream_rng(96, 1).standard_normal((n, 64)).astype(np.float32)
        z = np.zeros(64, np.float32)
        dy = stream_rng(97, 1).uniform(-1, 1, (rb.a_out, c)).astype(np.float32)
        ds = dy.copy()
        for r, ch, v in special:
            ds[r, ch] = v
        plain = scn.conv_bwd(rb, dev(x64), dev(z), dev(Wt), None, None, dev(dy), need=("dx", "dW"))
        got = scn.conv_bwd(rb, dev(x64), dev(z), dev(Wt), None, None, dev(ds), need=("dx", "dW"))
        same(host(got["dx"]), host(plain["dx"]), _dx_reference(rb, ir, orr, Wt, ds),
             np.repeat(hit(orr, ir, rb.a_in)[:, None], 64, 1))
        want, _ = _weight_gradient(rb, ir, orr, x64, z, ds)
        a, p = host(got["dW"]), host(plain["dW"])
        chans = np.zeros(c, bool)
        chans[[s[1] for s in special]] = True
        assert np.array_equal(a[:, :, ~chans], p[:, :, ~chans])
        ok = np.isfinite(want)
        assert not np.any(np.isfinite(a) & ~ok)
        assert np.array_equal(np.isnan(a[ok]), np.isnan(want[ok]))
        # weights of the input gradient: one NaN reaches the inputs' column alone,
        # and there the inputs with that offset
        Wn = Wt.copy()
        Wn[1, 5, 2] = np.nan
        got = host(scn.conv_bwd(rb, dev(x64), dev(z), dev(Wn), None, None, dev(dy),
                                need=("dx",))["dx"])
        reached = np.zeros((rb.a_in, 64), bool)
        reached[ir[rb.offsets[1]:rb.offsets[2]].numpy(), 5] = True
        assert np.array_equal(np.isnan(got), reached)
        rest, was = np.delete(got, 5, 1), np.delete(host(plain["dx"]), 5, 1)
        assert np.array_equal(rest, was)
        # inputs of the column without that offset may be summed again in fp32
        ref = _dx_reference(rb, ir, orr, Wt, dy)[:, 5]
        keep = ~reached[:, 5]
        assert _rms(got[keep, 5] - ref[keep]) <= 8 * U * _rms(ref)


@pytest.mark.parametrize("view", [False, True])
def test_few_channels_special_values_stay_local(scn, view):
    """As above for the first layers' weight gradient, whose sums run over all
    outputs: one infinite output gradient changes its column alone."""
    scn.set_dense_forward(0 if view else 1 << 40, 1)
    for cin, cout in ((1, 64), (3, 70)):
        rb, x, g, W, b, ir, orr = _layer(scn, 3, 30, 3000, cin, cout, 98)
        dy = stream_rng(99, 1).uniform(-1, 1, (rb.a_out, cout)).astype(np.float32)
        need = ("dW", "dbias")
        plain = host(scn.conv_bwd(rb, dev(x), dev(g), dev(W), None, None, dev(dy), need=need)["dW"])
        dy[rb.a_out // 3, 9] = np.inf
        x[5, cin - 1] = np.nan
        got = host(scn.conv_bwd(rb, dev(x), dev(g), dev(W), None, None, dev(dy), need=need)["dW"])
        with np.errstate(all="ignore"):
            want, _ = _weight_gradient(rb, ir, orr, x, g, dy)
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.array_equal(got[np.isinf(got)], want[np.isinf(want)])
        reached = np.zeros_like(got, bool)
        reached[:, cin - 1] = True
        reached[:, :, 9] = True
        assert np.array_equal(got[~reached], plain[~reached])


def _scaled(a, e):
    """a * 2^e, rounded to float32 once (2^e itself may be subnormal)"""
    return np.ldexp(a.astype(np.float64), e).astype(np.float32)


@pytest.mark.parametrize("e", [-100, -112, -120, -126])
@pytest.mark.parametrize("kind", ["split", "wg", "few"])
@pytest.mark.parametrize("view", [False, True])
def test_tiny_operands(scn, e, kind, view):
    """Rows, weights and output gradients whose low parts lie below bf16's last
    bit (2^-133): as close to 64-bit sums as at any other scale.  Whole tensors,
    then single rows, columns and channels beside ordinary ones."""
    m, n = GRIDS["wg" if kind == "wg" else "split"]
    c = 3 if kind == "few" else 64
    scn.set_dense_forward(0 if view else 1 << 40, 1)
    rb, x, g, W, b, ir, orr = _layer(scn, 2, m, n, c, 64, 101)
    g[:] = 0
    b[:] = 0
    dy = stream_rng(102, 1).standard_normal((rb.a_out, 64)).astype(np.float32)

    def close(got, want, rows=Ellipsis):
        got, want = got[rows], want[rows]
        assert _rms(got - want) <= 8 * U * _rms(want) + 2.0 ** -148

    def fwd(x, W):
        y = host(scn.conv_fwd(rb, dev(x), dev(g), dev(W), dev(b))[0])
        return y, _forward(rb, ir, orr, x, g, W, b)[0]

    def bwd(x, W, dy):
        need = ("dW", "dbias") if kind == "few" else ("dx", "dW")
        r = scn.conv_bwd(rb, dev(x), dev(g), dev(W), None, None, dev(dy), need=need)
        dx = None if kind == "few" else (host(r["dx"]), _dx_reference(rb, ir, orr, W, dy))
        return dx, (host(r["dW"]), _weight_gradient(rb, ir, orr, x, g, dy)[0])

    close(*fwd(_scaled(x, e), W))
    close(*fwd(x, _scaled(W, e)))
    for args in ((_scaled(x, e), W, dy), (x, _scaled(W, e), dy), (x, W, _scaled(dy, e))):
        dx, dW = bwd(*args)
        if dx is not None:
            close(*dx)
        close(*dW)
    # every output of one batch of rows tiny: inputs in a corner of the grid
    co = rb.export()[0].cpu().numpy()
    far = (co[:, 1:] >= m // 2 + 1).all(1)
    reach = np.zeros(n, bool)
    reach[ir.numpy()[far[orr.numpy()]]] = True
    xs = np.where(reach[:, None], _scaled(x, e), x)
    near_only = far & ~np.isin(np.arange(rb.a_out), orr.numpy()[~reach[ir.numpy()]])
    assert near_only.any()
    close(*fwd(xs, W), rows=near_only)
    # one column of weights, one channel of dy and x
    Ws, ds, xc = W.copy(), dy.copy(), x.copy()
    Ws[:, :, 37], ds[:, 37], xc[:, c - 1] = _scaled(W[:, :, 37], e), _scaled(dy[:, 37], e), \
        _scaled(x[:, c - 1], e)
    close(*fwd(x, Ws), rows=(slice(None), 37))
    _, dW = bwd(xc, W, ds)
    close(*dW, rows=(slice(None), slice(0, c - 1), 37))
    close(*dW, rows=(slice(None), c - 1, slice(0, 37)))
