"""Tiles dealt to the workgroups round by round: every tile once, for odd tiles that no XCD, some or all of them take."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _weights(n, k, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn((n, k), generator=g, device="cuda") * 0.02


def _dealt_k(fmt):
    return 3072 if fmt == "bf16" else 2560      # (bf16 weights of up to 16 tokens are in registers where a wave's share is whole slots: K = 1024 i)


# workgroups are at most as many as compute units (256): one to ten tiles each, 1, 7, 8, 255 and 0 left over
@pytest.mark.parametrize("tiles", [256 + 1, 2 * 256 + 7, 2 * 256 + 255, 5 * 256 + 8, 10 * 256, 264, 200, 101])
@pytest.mark.parametrize("fmt", ["int8", "w8a8", "int4", "bf16"])
def test_every_tile_once(fmt, tiles):
    from paper_2603_01399_amd import binding as qb
    m, n, k = 5, 16 * tiles, _dealt_k(fmt)
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


# K in two to eight slices, whose workgroups lie in four, all, two, all, four, all and one of the XCDs; some with a tile more than others
@pytest.mark.parametrize("slices,m,tiles,k", [(2, 8, 517, 13312), (3, 32, 131, 6144), (4, 32, 67, 8192), (5, 16, 101, 9216), (6, 32, 67, 12288),
                                              (7, 16, 67, 13312), (8, 32, 67, 16384), (5, 16, 517, 13312), (5, 8, 320, 25600),
                                              (3, 8, 67, 14336), (4, 32, 131, 8192), (4, 32, 323, 16384)])
def test_every_tile_of_every_slice(slices, m, tiles, k):
    from paper_2603_01399_amd import binding as qb
    n = 16 * tiles
    w = _weights(n, k, tiles)
    x = (torch.randn((m, k), device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))).to(torch.bfloat16)
    q, s = qb.quantize_weights(w)
    y = torch.full((m, n), float("nan"), dtype=torch.bfloat16, device="cuda")
    sums = 4 * slices * m * n
    assert qb.lib().quasar_w8_fused_workspace_bytes(m, n, k, 0, 1) == sums       # (the same division of K)
    ws = torch.full((max(sums, qb.workspace_bytes(m, n, k)) + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    qb.w8_linear(x, q, s, n, y=y, workspace=ws)
    wd = qb.unpack_weights(q, n, k).double() * s.double()[:, None]
    want = x.double() @ wd.t()
    bound = want.abs() * 2.0 ** -8 + 1e-5 * x.double().norm(dim=1)[:, None] * wd.norm(dim=1)[None]      # as above
    torch.cuda.synchronize()
    assert bool(((y.double() - want).abs() <= bound).all())
    # every partial sum was written, and nothing behind them
    assert not bool((ws[:sums].view(torch.int32) == 0xA5A5A5A5 - 2 ** 32).any()) and bool((ws[sums:] == 0xA5).all())


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


def _tiles_of(workgroup, rounds, cus):
    """Tiles of a workgroup of a vocabulary of `rounds` whole rounds and a part of one, in the order it takes them."""
    xcd, at = workgroup & 7, workgroup >> 3
    return [xcd * (cus >> 3) + min(xcd, cus & 7) + at + u * cus for u in range(rounds)] + [rounds * cus + workgroup]


# 17 rounds and the left-over tile: a wave finishes its workgroup's every 16th (8th) tile.  Which of them tie: the first and one of the same
# wave, one of another wave; the second and the left-over one, which the same wave finishes; the left-over one and the whole
# round in front; tiles of three workgroups, the lowest not in the first round
@pytest.mark.parametrize("ties", [[(9, 0), (9, 1), (9, 16)], [(9, 1), (9, 17)], [(9, 16), (9, 17)], [(9, 5), (3, 6), (250, 4)]])
@pytest.mark.parametrize("m", [3, 20])
@pytest.mark.parametrize("fmt", ["int8", "w8a8", "int4", "bf16"])
def test_equal_logits_give_the_lowest_row(fmt, m, ties):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    k, tiles = _dealt_k(fmt), 17 * cus + 40
    v = 16 * tiles
    tied = sorted(_tiles_of(b, 17, cus)[u] for b, u in ties)
    w = torch.zeros((v, k), device="cuda")
    # row 5 of each tile; of the lowest one also its other rows behind it, in the same lane and in others
    w[[16 * t + 5 for t in tied]] = 0.05
    w[16 * tied[0] + 6:16 * tied[0] + 16] = 0.05
    want = 16 * tied[0] + 5
    _lowest_of_equals(fmt, w, m, want)


@pytest.mark.parametrize("tiles", [256 + 1, 9 * 256 + 255, 2000 + 37])
@pytest.mark.parametrize("fmt", ["int8", "w8a8", "int4", "bf16"])
def test_equal_logits_of_several_workgroups(fmt, tiles):
    w = torch.zeros((16 * tiles, _dealt_k(fmt)), device="cuda")
    tied = [16 * t for t in (tiles - 1, 256, 255, 70, 38) if t < tiles]
    w[tied] = 0.05
    _lowest_of_equals(fmt, w, 3, min(tied))


def _lowest_of_equals(fmt, w, m, want):
    from paper_2603_01399_amd import binding as qb
    v, k = w.shape
    h = torch.ones((m, k), dtype=torch.bfloat16, device="cuda")
    draft = torch.full((m - 1,), want, dtype=torch.int32, device="cuda")
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
    assert np.array_equal(out[0].cpu().numpy(), [want] * m) and int(out[1]) == m - 1
