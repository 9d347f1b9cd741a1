"""Fused linears with scratch: the normalisation as a launch of its own and K split over workgroups, against the same entry points
without scratch (every workgroup normalises, K in one piece: the routes that the layer tests hold to the oracle)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _call(qb, x, wq, sc, N, gamma, residual, y, gated, ws, room):
    """Through the C entries, which take the scratch they are given."""
    ptr = lambda t: None if t is None else t.data_ptr()
    M, K = x.shape
    head = (x.data_ptr(), M, K, x.stride(0), ptr(gamma), 1e-6, wq.data_ptr(), sc.data_ptr())
    tail = (y.data_ptr(), y.stride(0), ptr(ws), room, qb._stream())
    if gated:
        qb._check("gated", qb.lib().quasar_w8_gateup_swiglu_split(*head, N // 2, *tail))
    else:
        qb._check("fused", qb.lib().quasar_w8_linear_fused_split(*head, N, ptr(residual), 0 if residual is None else residual.stride(0), *tail))


# K: first beyond each rule, ragged, split in two to seven slices; the last two normalise in more than one round of registers or split K in eight
@pytest.mark.parametrize("M,N,K", [(1, 16 * 22, 8256), (8, 16 * 258, 12288), (9, 16 * 258, 4160), (16, 16 * 40, 8256), (8, 16 * 128, 14336), (12, 16 * 320, 25600),
                                   (17, 16 * 258, 2112), (32, 16 * 700, 4096), (31, 16 * 40, 5184), (32, 16 * 320, 25600), (20, 16 * 16, 33024)])
@pytest.mark.parametrize("kind", ["norm", "residual", "both", "gated"])
def test_fused_with_scratch(M, N, K, kind):
    from paper_2603_01399_amd import binding as qb
    print("fused apart", M, N, K, kind, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(K + M)
    x = torch.full((M, K + 72), float("nan"), dtype=torch.bfloat16, device="cuda")[:, :K]
    x.copy_(torch.randn(M, K, generator=gen, device="cuda"))
    x[:, 17::331] *= 8
    if M > 4:
        x[1] = 0.0
        x[2] *= 1e-3
    wq, sc = qb.quantize_weights(torch.randn(N, K, generator=gen, device="cuda") * 0.02)
    gamma = (1 + 0.2 * torch.randn(K, generator=gen, device="cuda")).bfloat16() if kind != "residual" else None
    out = N // 2 if kind == "gated" else N
    residual = torch.randn(M, out, generator=gen, device="cuda").bfloat16() if kind in ("residual", "both") else None
    need = qb.lib().quasar_w8_gateup_workspace_bytes(M, N // 2, K, 1) if kind == "gated" else \
        qb.lib().quasar_w8_fused_workspace_bytes(M, N, K, gamma is not None, residual is not None)
    want = torch.empty((M, out), dtype=torch.bfloat16, device="cuda")
    _call(qb, x, wq, sc, N, gamma, residual, want, kind == "gated", None, 0)
    for room in (need, need // 2, 15):
        ws = torch.full((need + 256,), 0xA5, dtype=torch.uint8, device="cuda")
        y = torch.full((M, out + 24), 7.0, dtype=torch.bfloat16, device="cuda")
        got = y[:, :out]
        if residual is not None:
            got.copy_(residual)                                    # in place: y is the residual
        _call(qb, x, wq, sc, N, gamma, residual if residual is None else got, got, kind == "gated", ws, room)
        # another order of the row sums may move a normalised value, and of the sums an output, by one bf16 unit: the bound of
        # the fused linears against the oracle
        assert float((got.double() - want.double()).abs().max() / want.double().abs().max()) <= 6e-3
        assert bool((y[:, out:] == 7.0).all()) and bool((ws[room:] == 0xA5).all())
    # the binding brings its own scratch
    again = qb.w8_gateup_swiglu(x, wq, sc, out, gamma=gamma) if kind == "gated" else \
        qb.w8_linear_fused(x, wq, sc, N, gamma=gamma, residual=residual)
    assert float((again.double() - want.double()).abs().max() / want.double().abs().max()) <= 6e-3


@pytest.mark.parametrize("kind", ["w8a8", "int4", "residual", "norm", "gated"])
def test_without_memory_for_scratch(kind):
    """Calls whose scratch does not fit the memory that is left run without it, as the entry points do that take none."""
    from paper_2603_01399_amd import binding as qb
    print("no memory for scratch", kind, flush=True)
    M, N, K = 32, 16 * 320, 8192
    gen = torch.Generator(device="cuda").manual_seed(9)
    w = torch.randn(N, K, generator=gen, device="cuda") * 0.02
    packed = (qb.quantize_weights_w4(w),) if kind == "int4" else qb.quantize_weights(w)
    gamma = (1 + 0.2 * torch.randn(K, generator=gen, device="cuda")).bfloat16()
    x, res = torch.randn(M, K, generator=gen, device="cuda").bfloat16(), torch.randn(M, N, generator=gen, device="cuda").bfloat16()
    y = torch.empty((M, N // 2 if kind == "gated" else N), dtype=torch.bfloat16, device="cuda")
    call = {"w8a8": lambda: qb.w8a8_linear(x, *packed, N, y=y), "int4": lambda: qb.w4_linear(x, *packed, N, y=y),
            "residual": lambda: qb.w8_linear_fused(x, *packed, N, residual=res, y=y),
            "norm": lambda: qb.w8_linear_fused(x, *packed, N, gamma=gamma, y=y),
            "gated": lambda: qb.w8_gateup_swiglu(x, *packed, N // 2, gamma=gamma, y=y)}[kind]
    want = call().clone()
    got = torch.empty_like(want)
    del w
    torch.cuda.empty_cache()
    total, hold = torch.cuda.get_device_properties(0).total_memory, []
    torch.cuda.set_per_process_memory_fraction(min(1.0, (torch.cuda.memory_reserved() + (64 << 20)) / total))
    try:
        for size in (1 << 24, 1 << 21, (1 << 20) + 512, 1 << 20, 1 << 14):      # both of the pools: what is left is less than any scratch
            with pytest.raises(torch.OutOfMemoryError):
                for _ in range(1 << 14):
                    hold.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
        y.fill_(7.0)
        call()
        got.copy_(y)
        torch.cuda.synchronize()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
        hold.clear()
        torch.cuda.empty_cache()
    # (another order of the sums: the bound above; W8A8: integers, the same bits)
    assert float((got.double() - want.double()).abs().max() / want.double().abs().max()) <= (0.0 if kind == "w8a8" else 6e-3)
