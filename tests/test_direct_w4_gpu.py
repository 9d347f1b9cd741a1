"""The 4-bit kernel that keeps its activations in registers, over its register forms, ragged shares of K and tile remainders:
outputs against a 64-bit product with the dequantised codes (one bf16 rounding of an fp32 sum; the codes' bias of 136 taken out
of the accumulator leaves about 1e-5: 4e-3 of max|y| as for the 8-bit linear), argmax and accepted length of planted winners."""
import pytest
import torch

from paper_2603_01399_amd import synth
from gpu_util import bf16_to_dev, f32_to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [128, 1920, 2048, 2176, 4096, 4224, 5120, 6400, 8192, 12288])
@pytest.mark.parametrize("M,N", [(1, 16), (8, 16 * 261), (9, 16 * 40), (16, 16 * 261), (32, 16 * 261)])
def test_w4_forms(M, N, K):
    from paper_2603_01399_amd import binding as qb
    print("direct w4", M, N, K, flush=True)
    x = bf16_to_dev(synth.activations_bf16(M, K, seed=synth.seed_for(26, M, K)))
    x[M // 2] = x[M // 2].abs()                                    # all positive: the largest offset
    w = f32_to_dev(synth.normal_weights(N, K, seed=synth.seed_for(27, M, K)))
    packed = qb.quantize_weights_w4(w)
    codes, steps = qb.unpack_weights_w4(packed, N, K)
    what = (codes.double().view(N, -1, 128) * steps.double()[..., None]).view(N, K)
    want = x.double() @ what.t()
    y = qb.w4_linear(x, packed, N)
    assert float((y.double() - want).abs().max() / want.abs().max()) <= 4e-3
    assert torch.equal(y.view(torch.int16), qb.w4_linear(x, packed, N).view(torch.int16))
    if M > 1:
        draft = want.argmax(1).int()[:-1].contiguous()
        draft[M // 2:] += 1
        top = want.topk(2, dim=1).values
        clear = (top[:, 0] - top[:, 1]) > 1e-3 * want.abs().max()
        am, acc = qb.w4_lmhead_verify(x, packed, N, draft, qb.make_workspace(M, N, K))
        assert torch.equal(am[clear], want.argmax(1).int()[clear])
        hit = am[:-1] == draft
        assert int(acc) == int(hit.int().cumprod(0).sum())
