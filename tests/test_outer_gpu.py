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
@pytest.mark.parametrize("M,N,K", [(1, 16, 8256), (8, 16 * 257, 12288), (5, 16 * 320, 25600), (8, 16 * 700, 8256), (7, 16 * 2049, 8256),
                                   (9, 16 * 40, 5184), (16, 16 * 257, 8192), (12, 16 * 1000, 6208), (16, 16 * 320, 25600),
                                   (17, 16, 1024), (32, 16 * 64, 1088), (24, 16 * 257, 4160), (32, 16 * 600, 1024), (31, 16 * 1000, 1024),
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
    need = qb.lib().quasar_w8a8_workspace_bytes(M, N, K)
    assert need > 0
    got = qb.w8a8_linear(x, wq, sc, N, smooth=smooth, y=y[:, :N])
    same = got.view(torch.int16) == want.view(torch.int16)
    assert bool((same | (got.isnan() & want.isnan())).all())
    assert bool((y[:, N:] == 7.0).all())
    # scratch that holds no partial sums, and none: the same bits (through the C entry, which takes what it is given)
    head = K // 64 * 64 * (8 if M <= 8 else 16 if M <= 16 else 32) + 128
    for room in (need, head, head - 1):
        ws = torch.full((need + 256,), 0xA5, dtype=torch.uint8, device="cuda")
        y2 = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
        qb._check("w8a8", qb.lib().quasar_w8a8_linear(x.data_ptr(), M, K, x.stride(0), None if smooth is None else smooth.data_ptr(),
                                                      wq.data_ptr(), sc.data_ptr(), N, y2.data_ptr(), N, ws.data_ptr(), room, qb._stream()))
        same = y2.view(torch.int16) == want.view(torch.int16)
        assert bool((same | (y2.isnan() & want.isnan())).all())
        assert bool((ws[room:] == 0xA5).all())
