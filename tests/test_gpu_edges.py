"""The convolutions at the edges of their tiles: every row length, one and many
planes per block, both output widths, outputs that start off a vector boundary,
and infinite inputs."""
import pytest
import torch

from paper_2103_01597_amd import nn

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
