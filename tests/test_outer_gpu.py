"""The kernel that walks a workgroup's tiles side by side with K outermost, over its tile counts (1 to 8 and more rounds), ragged
shares of K and the divisions of K over workgroups."""
import pytest
import torch

from paper_2603_01399_amd import synth
from gpu_util import bf16_to_dev, f32_to_dev

pytestmark = pytest.mark.gpu


def _activations(M, K, rows=None):
    """M rows of K values out of a wider buffer whose other columns are NaN."""
    x = torch.full((M, K + 72), float("nan"), dtype=torch.bfloat16, device="cuda")[:, :K]
    x.copy_(bf16_to_dev(synth.activations_bf16(M, K, seed=synth.seed_for(28, M, K))))
    return x


# K: first beyond the kernel that quantises for itself, ragged, several slices; N: one tile, 1 + 1/256 tiles a compute unit, all counts,
# one tile more than eight a compute unit
@pytest.mark.parametrize("M,N,K", [(1, 16, 8256), (1, 16, 10304), (8, 16 * 257, 12288), (5, 16 * 320, 25600), (8, 16 * 700, 8256), (7, 16 * 2049, 8256),
                                   (9, 16 * 40, 5184), (16, 16 * 257, 8192), (12, 16 * 1000, 6208), (16, 16 * 320, 25600),
                                   (17, 16, 1024), (17, 16, 1088), (32, 16 * 64, 1088), (24, 16 * 257, 4160), (32, 16 * 600, 1024), (31, 16 * 1000, 1024),
                                   (32, 16 * 1200, 2048), (18, 16 * 1500, 1088), (32, 16 * 1700, 1024), (32, 16 * 2049, 1088),
                                   (32, 16 * 320, 25600), (32, 16 * 256, 12288), (20, 16 * 16, 33024)])
@pytest.mark.parametrize("smoothed", [False, True])
def test_w8a8_apart(M, N, K, smoothed):
    from paper_2603_01399_amd import binding as qb
    print("w8a8 apart", M, N, K, smoothed, flush=True)
    x = _activations(M, K)
    if M >= 8:
        x[1] = 0.0
        x[2] = x[2] * 2.0 ** -126
        x[3, 5] = float("inf")
        x[4, K // 2] = float("nan")
    w = f32_to_dev(synth.normal_weights(N, K, seed=synth.seed_for(29, 7, K))) if N <= 512 else \
        torch.randn(N, K, device="cuda", generator=torch.Generator("cuda").manual_seed(29 + K)) * 0.02
    smooth = torch.exp2(torch.rand(K, device="cuda") * 4 - 2) if smoothed else None
    wq, sc = qb.quantize_weights(w)
    codes, dx = qb.quantize_activations(x, smooth)
    acc = (codes.double() @ qb.unpack_weights(wq, N, K).double().t()).float()          # exact integers, one rounding
    want = (acc * (dx[:, None] * sc.float()[None])).bfloat16()
    y = torch.full((M, N + 24), 7.0, dtype=torch.bfloat16, device="cuda")
    head = K // 64 * 64 * (8 if M <= 8 else 16 if M <= 16 else 32) + 128
    need = max(qb.lib().quasar_w8a8_workspace_bytes(M, N, K), head)            # (which shapes use scratch: test_rules.py)
    got = qb.w8a8_linear(x, wq, sc, N, smooth=smooth, y=y[:, :N])
    same = got.view(torch.int16) == want.view(torch.int16)
    assert bool((same | (got.isnan() & want.isnan())).all())
    assert bool((y[:, N:] == 7.0).all())
    # scratch that holds no partial sums, and none: the same bits (through the C entry, which takes what it is given)
    for room in (need, head, head - 1):
        ws = torch.full((need + 256,), 0xA5, dtype=torch.uint8, device="cuda")
        y2 = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
        qb._check("w8a8", qb.lib().quasar_w8a8_linear_split(x.data_ptr(), M, K, x.stride(0), None if smooth is None else smooth.data_ptr(),
                                                            wq.data_ptr(), sc.data_ptr(), N, y2.data_ptr(), N, ws.data_ptr(), room, qb._stream()))
        same = y2.view(torch.int16) == want.view(torch.int16)
        assert bool((same | (y2.isnan() & want.isnan())).all())
        assert bool((ws[room:] == 0xA5).all())


@pytest.mark.parametrize("M,N,K", [(1, 16, 12416), (8, 16 * 320, 25600), (5, 16 * 1300, 12416), (8, 16 * 2049, 12416),
                                   (9, 16, 8320), (16, 16 * 256, 12288), (13, 16 * 700, 8320), (16, 16 * 1500, 8320), (16, 16 * 1537, 8320),
                                   (17, 16 * 40, 5120), (32, 16 * 64, 4736), (32, 16 * 256, 4224), (17, 16, 5120), (32, 16 * 257, 5120), (24, 16 * 700, 4224), (32, 16 * 1000, 4224),
                                   (31, 16 * 1200, 4224), (32, 16 * 1600, 5120), (32, 16 * 2049, 4224), (32, 16 * 320, 25600), (20, 16 * 16, 33024)])
def test_w4_outer(M, N, K):
    """Outputs against a 64-bit product with the dequantised codes: 4e-3 of max|y|, as for the kernel that holds x."""
    from paper_2603_01399_amd import binding as qb
    print("w4 outer", M, N, K, flush=True)
    x = _activations(M, K)
    x[M // 2] = x[M // 2].abs()                                    # all positive: the largest offset
    w = torch.randn(N, K, device="cuda", generator=torch.Generator("cuda").manual_seed(30 + K)) * 0.02
    packed = qb.quantize_weights_w4(w)
    codes, steps = qb.unpack_weights_w4(packed, N, K)
    what = (codes.double().view(N, -1, 128) * steps.double()[..., None]).view(N, K)
    want = x.double() @ what.t()
    y = torch.full((M, N + 24), 7.0, dtype=torch.bfloat16, device="cuda")
    qb.w4_linear(x, packed, N, y=y[:, :N])
    assert float((y[:, :N].double() - want).abs().max() / want.abs().max()) <= 4e-3
    assert bool((y[:, N:] == 7.0).all())
    assert torch.equal(y[:, :N].view(torch.int16), qb.w4_linear(x, packed, N).view(torch.int16))
    need = qb.lib().quasar_w4_workspace_bytes(M, N, K)
    for room in (0, need, need - 1):                               # no scratch, and scratch of exactly one plan or less
        ws = torch.full((max(need, 0) + 256,), 0xA5, dtype=torch.uint8, device="cuda")
        y2 = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
        qb._check("w4", qb.lib().quasar_w4_linear_split(x.data_ptr(), M, K, x.stride(0), packed.data_ptr(), N, y2.data_ptr(), N,
                                                        ws.data_ptr(), max(room, 0), qb._stream()))
        assert float((y2.double() - want).abs().max() / want.abs().max()) <= 4e-3
        assert bool((ws[max(room, 0):] == 0xA5).all())


@pytest.mark.parametrize("kind", ["w8a8", "int4", "fused", "gated"])
def test_scratch_routes_under_capture(kind):
    """The routes that take scratch from torch's allocator, captured and replayed with new inputs and eager work in between."""
    from paper_2603_01399_amd import binding as qb
    M, N, K = 20, 16 * 40, 8192
    print("capture", kind, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5)
    w = torch.randn(N, K, generator=gen, device="cuda") * 0.02
    wq, sc = qb.quantize_weights(w)
    w4 = qb.quantize_weights_w4(w)
    gamma = (1 + 0.2 * torch.randn(K, generator=gen, device="cuda")).bfloat16()
    x = torch.randn(M, K, generator=gen, device="cuda").bfloat16()
    y = torch.empty((M, N // 2 if kind == "gated" else N), dtype=torch.bfloat16, device="cuda")
    res = torch.randn(M, N, generator=gen, device="cuda").bfloat16()
    call = {"w8a8": lambda y: qb.w8a8_linear(x, wq, sc, N, y=y), "int4": lambda y: qb.w4_linear(x, w4, N, y=y),
            "fused": lambda y: qb.w8_linear_fused(x, wq, sc, N, gamma=gamma, residual=res, y=y),
            "gated": lambda y: qb.w8_gateup_swiglu(x, wq, sc, N // 2, gamma=gamma, y=y)}[kind]
    call(y)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(y)
    for _ in range(4):
        x.copy_(torch.randn(M, K, generator=gen, device="cuda"))
        want = call(torch.empty_like(y))
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("M,V,K", [(17, 16, 1024), (24, 2048, 2048), (17, 2064, 1024), (32, 16 * 300, 1088), (24, 16 * 1100, 4096), (32, 16 * 257, 5120), (20, 16 * 40, 6144), (20, 16 * 40, 6208)])
@pytest.mark.parametrize("smoothed", [False, True])
def test_w8a8_vocabulary_of_many_tokens(M, V, K, smoothed):
    """Codes from a launch of their own, then the argmax: bit for bit the stated arithmetic, ties to the lowest index."""
    from paper_2603_01399_amd import binding as qb
    print("w8a8 vocabulary", M, V, K, smoothed, flush=True)
    x = _activations(M, K)
    x[1] = 0.0                                                     # every logit equal: index 0
    w = torch.randn(V, K, device="cuda", generator=torch.Generator("cuda").manual_seed(31 + K)) * 0.02
    w[V // 2:] = w[:V - V // 2]                                    # every row twice
    smooth = torch.exp2(torch.rand(K, device="cuda") * 4 - 2) if smoothed else None
    wq, sc = qb.quantize_weights(w)
    codes, dx = qb.quantize_activations(x, smooth)
    acc = (codes.double() @ qb.unpack_weights(wq, V, K).double().t()).float()
    want = (acc * (dx[:, None] * sc.float()[None])).double()
    top = want.max(1, keepdim=True).values
    want = torch.where(want == top, torch.arange(V, device="cuda")[None], V).min(1).values.int()
    draft = want[:-1].clone()
    draft[M // 2:] += 1
    ws = qb.make_workspace(M, V, K)
    room = torch.full((ws.nbytes + 256,), 0xA5, dtype=torch.uint8, device="cuda")
    am, accepted = qb.w8a8_lmhead_verify(x, wq, sc, V, draft.contiguous(), room[:ws.nbytes], smooth=smooth)
    assert torch.equal(am, want) and int(accepted) == M // 2 and bool((room[ws.nbytes:] == 0xA5).all())
    # the codes lie 512 KB behind the start; short calls make none
    apart = (V > 2048 or M * K > 60000) and K <= 6144
    assert bool((room[1 << 19:(1 << 19) + M * K // 2] != 0xA5).any()) == apart
