"""Kernels at the edges of their tiles.  Convolutions: every row length, one and
many planes per block, both output widths, outputs that start off a vector
boundary, infinite inputs.  Halo fill: rows of any length and start.  Reductions: rows of one and several strides, fewer
rows than blocks, remainders.  Substep: slabs of one to four planes,
boxes of any width.  Optimizer: arrays of
unequal sizes in one launch."""
import threading

import pytest
import torch

from paper_2103_01597_amd import mhd, nn

pytestmark = pytest.mark.gpu


def _taps(x, n, batch, cin):
    """x shifted by each of the 27 taps, [27][cells][cin] (periodic)."""
    v = x.view(batch, n, n, n, cin)
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                yield v.roll((-dz, -dy, -dx), (1, 2, 3)).reshape(-1, cin)


def _off(count, dtype):
    """An output of count elements that starts one element past an aligned address."""
    return torch.zeros(count + 9, dtype=dtype, device="cuda")[1:count + 1]


@pytest.mark.parametrize("n,batch", [(16, 1), (16, 5), (32, 3), (64, 2)])
@pytest.mark.parametrize("cin,cout", [(8, 8), (8, 32), (32, 8), (32, 32)])
def test_conv_exact_on_whole_numbers(n, batch, cin, cout):
    # products and sums of small whole numbers are exact in FP32 in any order, so
    # the only rounding left is the result's own to BF16
    g = torch.Generator(device="cuda").manual_seed(n + batch + cin + cout)

    def ints(*shape):
        return torch.randint(-4, 5, shape, generator=g, device="cuda").float()

    cells = batch * n ** 3
    x, w, bias = ints(cells, cin), ints(cout, 27, cin), ints(cout)
    w_pad = torch.empty(32 * 27 * cin, dtype=torch.bfloat16, device="cuda")
    wt_pad = torch.empty(32 * 27 * cout, dtype=torch.bfloat16, device="cuda")
    nn.prepare_weights(w, cin, cout, w_pad, wt_pad)
    xb = x.to(torch.bfloat16)
    ref = sum(v @ w[:, t].t() for t, v in enumerate(_taps(x, n, batch, cin))) + bias

    y = _off(cells * cout, torch.float32)
    nn.conv3d_fwd(xb, w_pad, bias, n, batch, cin, cout, 1, y=y)
    assert torch.equal(y.view(cells, cout), ref)
    z, a = _off(cells * cout, torch.bfloat16), _off(cells * cout, torch.bfloat16)
    nn.conv3d_fwd(xb, w_pad, bias, n, batch, cin, cout, 0, z=z, a=a)
    assert torch.equal(z.view(cells, cout), ref.to(torch.bfloat16))
    big = ref.abs() >= 16  # GELU(v) is v or (to FP32) zero there
    assert torch.equal(a.view(cells, cout)[big], ref.clamp(min=0).to(torch.bfloat16)[big])

    # data gradient into cin channels where GELU' is exactly one
    dz, zp = ints(cells, cout), _off(cells * cin, torch.bfloat16)
    zp.fill_(16.0)
    dp = _off(cells * cin, torch.bfloat16)
    nn.conv3d_dgrad(dz.to(torch.bfloat16), wt_pad, zp, n, batch, cout, cin, dp)
    back = sum(v @ w[:, 26 - t] for t, v in enumerate(_taps(dz, n, batch, cout)))
    assert torch.equal(dp.view(cells, cin), back.to(torch.bfloat16))


@pytest.mark.parametrize("cin", [8, 32])
def test_conv_infinite_input_reaches_its_neighbours_only(cin):
    n, cells = 16, 16 ** 3
    x = torch.ones(cells, cin, device="cuda")
    x[(3 * n + 0) * n + 15, 2] = float("inf")
    w = torch.ones(32, 27, cin, device="cuda")
    w_pad = torch.empty(32 * 27 * cin, dtype=torch.bfloat16, device="cuda")
    nn.prepare_weights(w, cin, 32, w_pad)
    y = torch.empty(cells * 32, device="cuda")
    nn.conv3d_fwd(x.to(torch.bfloat16), w_pad, torch.zeros(32, device="cuda"), n, 1, cin, 32, 1, y=y)
    ref = sum(v.sum(1, keepdim=True) for v in _taps(x, n, 1, cin)).expand(cells, 32)
    assert torch.equal(y.view(cells, 32), ref)


@pytest.mark.parametrize("n,batch", [(16, 1), (16, 5), (32, 3), (64, 2)])
@pytest.mark.parametrize("cin,cout", [(8, 8), (8, 32), (32, 8), (32, 32)])
def test_weight_gradient_exact_on_whole_numbers(n, batch, cin, cout):
    # every partial sum is a whole number below 16 * 2^19 < 2^24: exact in FP32
    g = torch.Generator(device="cuda").manual_seed(n + batch + cin + cout)
    cells = batch * n ** 3
    x = torch.randint(-4, 5, (cells, cin), generator=g, device="cuda").float()
    dz = torch.randint(-4, 5, (cells, cout), generator=g, device="cuda").float()
    ws = torch.empty(nn.wgrad_workspace_floats(n, batch), device="cuda")
    dw, db = _off(cout * 27 * cin, torch.float32), _off(cout, torch.float32)
    nn.conv3d_wgrad(x.to(torch.bfloat16), dz.to(torch.bfloat16), n, batch, cin, cout, ws, dw, db)
    ref = torch.stack([dz.t() @ v for v in _taps(x, n, batch, cin)], 1)
    assert torch.equal(dw.view(cout, 27, cin), ref)
    assert torch.equal(db, dz.sum(0))


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,order", [((1, 1, 1), 8), ((2, 3, 5), 8), ((1, 40, 70), 2), ((16, 16, 16), 6), ((17, 15, 33), 6),
                                     ((30, 5, 9), 4), ((31, 64, 3), 2), ((65, 33, 8), 8), ((2500, 3, 2), 6), ((9001, 2, 1), 6)])
def test_halo_fill_of_any_row(n, order, prec, offset):
    # rows of any length, in whole and broken units, from aligned and other addresses:
    # padded coordinate s holds the interior cell (s - r) mod n, nothing else changes
    S = mhd.Solver(*n, prec, order=order)
    g = torch.Generator(device="cuda").manual_seed(sum(n))
    total = S.layout.total_elems
    room = torch.randn(total + 16, generator=g, device="cuda", dtype=torch.float64).to(S.torch_dtype)
    f = room[offset:offset + total]
    before = room.clone()
    want = S.interior_view(f).clone()
    for axis, m in ((3, n[0]), (2, n[1]), (1, n[2])):
        want = want.index_select(axis, (torch.arange(m + 2 * S.r, device="cuda") - S.r) % m)
    S.halo_periodic(f)
    assert torch.equal(S.grid_view(f), want)
    S.grid_view(f).copy_(S.grid_view(before[offset:offset + total]))
    assert torch.equal(room, before)
    S.close()


@pytest.mark.parametrize("prec", ["f64", "f32c"])
@pytest.mark.parametrize("n", [(1, 1, 1), (300, 17, 5), (257, 3, 33), (8, 8, 200), (64, 64, 37), (513, 70, 40)])
def test_reductions_exact_on_whole_numbers(n, prec):
    # whole numbers below 2^53 in any order, twice (the second call finds what the first left)
    S = mhd.Solver(*n, precision=prec)
    f = S.zeros()
    f += 1e6  # the halo is not part of it
    g = torch.Generator(device="cuda").manual_seed(sum(n))
    v = torch.randint(-1000, 1001, n[::-1], generator=g, device="cuda").double()
    S.interior_view(f)[3].copy_(v)
    for _ in range(2):
        assert S.reduce(f, 3, "sum") == v.sum().item()
        assert S.reduce(f, 3, "sumsq") == (v * v).sum().item()
        assert S.reduce(f, 3, "maxabs") == v.abs().max().item()
        assert S.reduce(f, 3, "min") == v.min().item()
        assert S.reduce(f, 3, "max") == v.max().item()
        assert S.reduce(f, 3, "nonfinite") == 0.0
    S.interior_view(f)[3][-1, -1, -1] = float("nan")
    assert S.reduce(f, 3, "nonfinite") == 1.0
    assert S.reduce(f, 3, "min") != S.reduce(f, 3, "min")
    S.close()


@pytest.mark.parametrize("n", [(32, 32, 32), (64, 64, 64), (9, 3, 5)])
def test_reductions_leave_nothing_behind(n):
    # one context used by several threads at once has no defined values, but whatever
    # such calls do must not reach the calls after them
    S = mhd.Solver(*n)
    f = S.zeros()
    v = torch.arange(n[0] * n[1] * n[2], device="cuda").double().view(n[::-1])
    S.interior_view(f)[0].copy_(v)
    torch.cuda.synchronize()

    def many(stream):
        for _ in range(50):
            S.reduce(f, 0, "sum", stream=stream)

    threads = [threading.Thread(target=many, args=(torch.cuda.Stream(),)) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for op, want in (("sum", v.sum().item()), ("max", v.max().item()), ("min", 0.0), ("nonfinite", 0.0)):
        assert S.reduce(f, 0, op) == want
    S.interior_view(f)[0].add_(1.0)
    assert S.reduce(f, 0, "min") == 1.0
    S.close()


@pytest.mark.parametrize("order", [2, 4, 6, 8])
@pytest.mark.parametrize("prec", ["f64", "f32c", "f32"])
def test_thin_slabs_equal_full_substep(prec, order):
    # every cell's arithmetic is the same in any box: bit for bit
    S = mhd.Solver(45, 19, 10, precision=prec, order=order)
    g = torch.Generator(device="cuda").manual_seed(order)
    f = torch.randn(S.layout.total_elems, generator=g, device="cuda", dtype=torch.float64) * 1e-2
    f = f.to(S.torch_dtype)
    S.halo_periodic(f)
    old = torch.randn(f.numel(), generator=g, device="cuda").to(f) * 1e-3
    comp = torch.randn(f.numel(), generator=g, device="cuda").to(f) * 1e-9 if prec == "f32c" else None
    for s in (0, 1, 2):
        got = []
        for cuts in ((0, 10), (0, 1, 3, 6, 10)):
            out, w, c = f.clone(), old.clone(), None if comp is None else comp.clone()
            for a, b in zip(cuts, cuts[1:]):
                S.rk3_substep_box(s, (0, 45, 0, 19, a, b), f, out, w, c)
            got.append((out, w, c))
        for full, thin in zip(*got):
            assert full is None or torch.equal(full, thin)
        assert bool(torch.isfinite(got[0][0]).all())
    S.close()


@pytest.mark.parametrize("order", [2, 4, 6, 8])
@pytest.mark.parametrize("prec", ["f64", "f32c", "f32"])
@pytest.mark.parametrize("nx", [70, 69])
def test_box_reads_its_own_surroundings_only(nx, prec, order):
    # boxes of any width, from even and odd columns, in grids with even and odd rows (planes
    # fetched in pairs or by cells): the full substep's bits inside, with NaN wherever the
    # box's stencil does not reach, and nothing changed outside
    n = (nx, 21, 12)
    S = mhd.Solver(*n, precision=prec, order=order)
    g = torch.Generator(device="cuda").manual_seed(order)
    f = (torch.randn(S.layout.total_elems, generator=g, device="cuda", dtype=torch.float64) * 1e-2).to(S.torch_dtype)
    S.halo_periodic(f)
    old = torch.randn(f.numel(), generator=g, device="cuda").to(f) * 1e-3
    comp = torch.randn(f.numel(), generator=g, device="cuda").to(f) * 1e-9 if prec == "f32c" else None
    out, w, c = f.clone(), old.clone(), None if comp is None else comp.clone()
    S.rk3_substep(1, f, out, w, c)
    r = S.r
    for b in ((0, 3, 0, 21, 0, 12), (nx - 1, nx, 0, 21, 2, 12), (2, 35, 4, 13, 1, 4), (33, 66, 20, 21, 0, 12), (32, 64, 8, 16, 5, 6), (0, nx, 0, 21, 0, 12)):
        inside = lambda t, k=0: S.grid_view(t)[:, r + b[4] - k:r + b[5] + k, r + b[2] - k:r + b[3] + k, r + b[0] - k:r + b[1] + k]  # noqa: E731
        around = torch.full_like(f, float("nan"))
        inside(around, r).copy_(inside(f, r))
        got = [torch.full_like(f, 7.0), old.clone(), None if comp is None else comp.clone()]
        want = [torch.full_like(f, 7.0), old.clone(), None if comp is None else comp.clone()]
        S.rk3_substep_box(1, b, around, *got)
        for a, e, full in zip(got, want, (out, w, c)):
            if e is not None:
                inside(e).copy_(inside(full))
                assert torch.equal(a, e), b
    S.close()


@pytest.mark.parametrize("n,prec,order", [((16, 16, 16), "f64", 6), ((40, 33, 20), "f32c", 2), ((64, 24, 30), "f32", 8)])
def test_captured_steps_equal_eager_ones(n, prec, order):
    # two steps recorded by the caller and replayed, with eager work and waits between
    # the replays: the same bits each time
    S = mhd.Solver(*n, precision=prec, order=order)
    g = torch.Generator(device="cuda").manual_seed(order)
    f0 = (torch.randn(S.layout.total_elems, generator=g, device="cuda", dtype=torch.float64) * 1e-2).to(S.torch_dtype)

    def state():
        return [f0.clone(), S.zeros()], S.zeros(), S.zeros() if prec == "f32c" else None

    (fe, we, ce), (fc, wc, cc) = state(), state()
    S.step(fe, 0, we, ce, 1e-3, 2)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        assert S.step(fc, 0, wc, cc, 1e-3, 2) == 0
    assert torch.equal(fc[0], f0)  # recorded, not run
    for _ in range(4):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(S.interior_view(fc[0]), S.interior_view(fe[0])) and torch.equal(wc, we)
        assert ce is None or torch.equal(cc, ce)
        assert S.reduce(fc[0], 1, "maxabs") > 0
        S.step(fe, 0, we, ce, 1e-3, 2)
    S.close()


@pytest.mark.parametrize("sizes", [(1,), (256, 1), (6912, 32, 27648, 0, 6912, 8), (257, 255, 256, 1, 2, 3, 4, 5)])
def test_updates_in_one_launch_equal_one_by_one(sizes):
    g = torch.Generator(device="cuda").manual_seed(len(sizes))
    parts = [tuple(torch.rand(n + 1, generator=g, device="cuda")[1:] for _ in range(4)) for n in sizes if n]
    alone = [tuple(t.clone() for t in q) for q in parts]
    for t in (1, 2):
        nn.adam_parts(parts, 1e-3, t)
        for p, gr, m, v in alone:
            nn.adam(p, gr, m, v, 1e-3, t)
    for a, b in zip(parts, alone):
        assert all(torch.equal(x, y) for x, y in zip(a, b))
    pads = []
    for cin, cout in ((8, 8), (8, 32), (32, 32), (32, 8)):
        w = torch.randn(cout, 27, cin, generator=g, device="cuda")
        pads.append((w, cin, cout) + tuple(torch.full((32 * 27 * c,), 7.0, dtype=torch.bfloat16, device="cuda") for c in (cin, cout)))
    nn.prepare_weights_parts(pads)
    for w, cin, cout, wp, wt in pads:
        wide = torch.zeros(32, 27, cin, device="cuda")
        wide[:cout] = w
        assert torch.equal(wp.view(32, 27, cin), wide.to(torch.bfloat16))
        flip = torch.zeros(32, 27, cout, device="cuda")
        flip[:cin] = w.flip(1).permute(2, 1, 0)
        assert torch.equal(wt.view(32, 27, cout), flip.to(torch.bfloat16))


@pytest.mark.parametrize("sizes", [(3, 0, 300), (0, 5, 0, 0, 257), (256, 0), (0, 0), (1,) * 8, (40,) * 9, (7, 0, 300) * 6])
def test_updates_of_any_number_of_arrays(sizes):
    # arrays without elements (at an address of their own) between others, and more arrays
    # than one launch takes: as many calls of one array
    g = torch.Generator(device="cuda").manual_seed(len(sizes))
    parts = [tuple(torch.rand(n + 1, generator=g, device="cuda") for _ in range(4)) for n in sizes]
    alone = [tuple(t.clone() for t in q) for q in parts]
    rows = (nn.AdamPart * len(sizes))(*[nn.AdamPart(*[t.data_ptr() for t in q], n) for q, n in zip(parts, sizes)])
    if len(sizes) <= nn.MAX_PARTS:
        nn._chk("adam", nn.lib().mhdnn_adam_parts(rows, len(sizes), 1e-3, 0.9, 0.999, 1e-8, 1, nn._st()))
    else:
        nn.adam_parts([tuple(t[:n] if n else t[:1] for t in q) for q, n in zip(parts, sizes) if n], 1e-3, 1)
    for q, n in zip(alone, sizes):
        if n:
            nn.adam(*[t[:n] for t in q], 1e-3, 1)
    for a, b in zip(parts, alone):
        assert all(torch.equal(x, y) for x, y in zip(a, b))


def test_closure_of_more_layers_than_one_launch_takes(monkeypatch):
    # inference takes any depth: the layers' weights are prepared however many there are
    deep = ((8, 32, True),) + ((32, 32, True),) * 8 + ((32, 8, False),)
    monkeypatch.setattr(nn, "LAYERS", deep)
    net = nn.Closure(seed=1)
    for (cin, cout, _), w, wp in zip(deep, net.w, net.w_pad):
        assert torch.equal(wp.view(32, 27, cin)[:cout], w.to(torch.bfloat16))
    x = torch.randn(16 ** 3 * 8, device="cuda").to(torch.bfloat16)
    y, _ = net.forward(x, 16, 1)
    assert bool(torch.isfinite(y).all())
    net.step([torch.ones_like(p) for p in net.params], 1e-3)
    assert all(bool((p != 0).any()) for p in net.params)
