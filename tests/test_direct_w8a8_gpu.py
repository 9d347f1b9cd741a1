"""The W8A8 kernel that keeps its activation codes in registers, over its register forms and ragged shares of K: outputs equal,
bit for bit, the stated arithmetic on the codes and step sizes of the stand-alone activation quantiser - for ordinary tokens, a
zero token, one so small that the reciprocal step overflows, and tokens with infinities and NaN."""
import pytest
import torch

from paper_2603_01399_amd import synth
from gpu_util import bf16_to_dev, f32_to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [64, 960, 1088, 2112, 3136, 4160, 5184, 7680, 8192, 12288])
@pytest.mark.parametrize("M,N", [(1, 16), (8, 16 * 261), (16, 16 * 40), (32, 16 * 261)])
@pytest.mark.parametrize("smoothed", [False, True])
def test_w8a8_forms(M, N, K, smoothed):
    from paper_2603_01399_amd import binding as qb
    print("direct w8a8", M, N, K, smoothed, flush=True)
    x = bf16_to_dev(synth.activations_bf16(M, K, seed=synth.seed_for(24, M, K)))
    if M >= 8:
        x[1] = 0.0
        x[2] = x[2] * 2.0 ** -126
        x[3, 5] = float("inf")
        x[4, K // 2] = float("nan")
    w = f32_to_dev(synth.normal_weights(N, K, seed=synth.seed_for(25, M, K)))
    smooth = torch.exp2(torch.rand(K, device="cuda") * 4 - 2) if smoothed else None
    wq, sc = qb.quantize_weights(w)
    codes, dx = qb.quantize_activations(x, smooth)
    acc = (codes.double() @ qb.unpack_weights(wq, N, K).double().t()).float()          # exact integers, one rounding
    want = (acc * (dx[:, None] * sc.float()[None])).bfloat16()
    got = qb.w8a8_linear(x, wq, sc, N, smooth=smooth)
    same = got.view(torch.int16) == want.view(torch.int16)
    assert bool((same | (got.isnan() & want.isnan())).all())
