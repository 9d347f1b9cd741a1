"""Tiles dealt to the workgroups round by round: every tile once, for odd tiles that no XCD, some or all of them take."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _weights(n, k, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn((n, k), generator=g, device="cuda") * 0.02


# workgroups are at most as many as compute units (256): one to ten tiles each, 1, 7, 8, 255 and 0 left over
@pytest.mark.parametrize("tiles", [256 + 1, 2 * 256 + 7, 2 * 256 + 255, 5 * 256 + 8, 10 * 256, 264, 200, 101])
@pytest.mark.parametrize("fmt", ["int8", "w8a8", "int4", "bf16"])
def test_every_tile_once(fmt, tiles):
    from paper_2603_01399_amd import binding as qb
    m, n, k = 5, 16 * tiles, 2560
    w = _weights(n, k, tiles)
    x = (torch.randn((m, k), device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))).to(torch.bfloat16)
    y = torch.full((m, n), float("nan"), dtype=torch.bfloat16, device="cuda")
    xd = x.double()
    if fmt == "int8":
        q, s = qb.quantize_weights(w)
        qb.w8_linear(x, q, s, n, y=y)
        wd = qb.unpack_weights(q, n, k).double() * s.double()[:, None]
    elif fmt == "w8a8":
        q, s = qb.quantize_weights(w)
        qb.w8a8_linear(x, q, s, n, y=y)
        wd = qb.unpack_weights(q, n, k).double() * s.double()[:, None]
        amax = x.float().abs().amax(1, keepdim=True)
        xd = torch.clamp(torch.round(x.float() * (127.0 / amax)), -127, 127).double() * (amax / 127.0).double()
    elif fmt == "int4":
        packed = qb.quantize_weights_w4(w)
        qb.w4_linear(x, packed, n, y=y)
        q, s = qb.unpack_weights_w4(packed, n, k)
        wd = (q.view(n, -1, 128).double() * s.double()[..., None]).view(n, k)
    else:
        qb.bf16_linear(x, qb.pack_bf16_weights(w), n, y=y)
        wd = w.to(torch.bfloat16).double()
    want = xd @ wd.t()
    # a bf16 rounding (2^-9) and fp32 sums of k terms of the size of the row's norm product
    bound = want.abs() * 2.0 ** -8 + 1e-5 * xd.norm(dim=1)[:, None] * wd.norm(dim=1)[None]
    torch.cuda.synchronize()
    assert bool(((y.double() - want).abs() <= bound).all())


# K in two to eight slices, whose workgroups lie in four, two or all XCDs by turns
@pytest.mark.parametrize("m,tiles,k", [(8, 67, 14336), (8, 320, 25600), (32, 131, 8192), (32, 323, 16384), (16, 517, 13312)])
def test_every_tile_of_every_slice(m, tiles, k):
    from paper_2603_01399_amd import binding as qb
    n = 16 * tiles
    w = _weights(n, k, tiles)
    x = (torch.randn((m, k), device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))).to(torch.bfloat16)
    q, s = qb.quantize_weights(w)
    y = torch.full((m, n), float("nan"), dtype=torch.bfloat16, device="cuda")
    qb.w8_linear(x, q, s, n, y=y, workspace=qb.make_workspace(m, n, k))
    wd = qb.unpack_weights(q, n, k).double() * s.double()[:, None]
    want = x.double() @ wd.t()
    bound = want.abs() * 2.0 ** -8 + 1e-5 * x.double().norm(dim=1)[:, None] * wd.norm(dim=1)[None]      # as above
    torch.cuda.synchronize()
    assert bool(((y.double() - want).abs() <= bound).all())


@pytest.mark.parametrize("pairs", [256 + 9, 3 * 256 + 128])
def test_gate_and_up_stay_together(pairs):
    from paper_2603_01399_amd import binding as qb
    m, inter, k = 8, 16 * pairs, 2560
    w = _weights(2 * inter, k, pairs)
    x = (torch.randn((m, k), device="cuda", generator=torch.Generator(device="cuda").manual_seed(2))).to(torch.bfloat16)
    q, s = qb.quantize_weights(w)
    y = torch.full((m, inter), float("nan"), dtype=torch.bfloat16, device="cuda")
    qb.w8_gateup_swiglu(x, q, s, inter, y=y)
    both = (x.double() @ (qb.unpack_weights(q, 2 * inter, k).double() * s.double()[:, None]).t()).view(m, pairs, 2, 16)
    gate, up = (both[:, :, i].reshape(m, inter).to(torch.bfloat16).double() for i in (0, 1))
    want = torch.nn.functional.silu(gate).to(torch.bfloat16).double() * up
    torch.cuda.synchronize()
    # each of gate, silu, up and the product rounded to bf16, gate and up within a rounding of the exact ones: six times 2^-9
    assert bool(((y.double() - want).abs() <= 6 * 2.0 ** -9 * want.abs() + 1e-3).all())


@pytest.mark.parametrize("tiles", [256 + 1, 9 * 256 + 255, 2000 + 37])
@pytest.mark.parametrize("fmt", ["int8", "w8a8", "int4", "bf16"])
def test_equal_logits_give_the_lowest_row(fmt, tiles):
    """Rows that tie lie in tiles of one workgroup, of neighbours and of others."""
    from paper_2603_01399_amd import binding as qb
    v, k, m = 16 * tiles, 2560, 3
    w = torch.zeros((v, k), device="cuda")
    tied = [16 * t for t in (tiles - 1, 256, 255, 70, 38) if t < tiles]
    w[tied] = 0.05
    h = torch.ones((m, k), dtype=torch.bfloat16, device="cuda")
    draft = torch.full((m - 1,), min(tied), dtype=torch.int32, device="cuda")
    ws = qb.make_workspace(m, v, k)
    if fmt == "int8":
        out = qb.lmhead_verify(h, *qb.quantize_weights(w), v, draft, ws)
    elif fmt == "w8a8":
        out = qb.w8a8_lmhead_verify(h, *qb.quantize_weights(w), v, draft, ws)
    elif fmt == "int4":
        out = qb.w4_lmhead_verify(h, qb.quantize_weights_w4(w), v, draft, ws)
    else:
        out = qb.bf16_lmhead_verify(h, qb.pack_bf16_weights(w), v, draft, ws)
    torch.cuda.synchronize()
    assert np.array_equal(out[0].cpu().numpy(), [min(tied)] * m) and int(out[1]) == m - 1
