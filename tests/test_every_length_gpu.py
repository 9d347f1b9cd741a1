"""Every K that a caller may pass, through every entry point and group of token counts: each length lands on a form that is built
and sums every one of its products once.  Activations are 1 and weights whole numbers, so every fp32 sum is exact in any order
and the outputs are known: K (7 K for 4-bit weights, whose step size is then 1), rounded to bf16 once."""
import pytest
import torch

pytestmark = pytest.mark.gpu
N = 32
LENGTHS = list(range(64, 13313, 64)) + [16384, 20480, 25600]


@pytest.fixture(scope="module")
def qb():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2603_01399_amd import binding
    return binding


@pytest.mark.parametrize("M", [2, 9, 17])
@pytest.mark.parametrize("kind", ["int8", "int8+ws", "bf16", "bf16+ws", "w8a8", "w8a8+smooth", "int4", "norm", "norm+residual",
                                  "residual", "swiglu", "norm+swiglu", "head int8", "head bf16", "head w8a8", "head int4",
                                  "sampled head"])
def test_every_length(qb, kind, M):
    print("every length", kind, M, flush=True)
    dev = "cuda"
    ones = torch.ones(M, max(LENGTHS), dtype=torch.bfloat16, device=dev)
    codes = torch.ones(N * max(LENGTHS), dtype=torch.int8, device=dev)
    wide = torch.ones(N * max(LENGTHS), dtype=torch.bfloat16, device=dev)
    sc = torch.ones(N, dtype=torch.bfloat16, device=dev)
    smooth = torch.ones(max(LENGTHS), dtype=torch.float32, device=dev)
    res = torch.full((M, N), 3.0, dtype=torch.bfloat16, device=dev)
    draft = torch.zeros(M - 1, dtype=torch.int32, device=dev)
    ws = torch.empty(1 << 23, dtype=torch.uint8, device=dev)
    ua, us = torch.full((M - 1,), 0.5, device=dev), torch.full((M,), 0.5, device=dev)
    for K in LENGTHS:
        if "int4" in kind and K % 128:
            continue
        x, gamma = ones[:, :K].contiguous(), ones[0, :K].contiguous()
        q, w16, sm = codes[:N * K], wide[:N * K], smooth[:K]
        k16 = torch.tensor(float(K)).bfloat16().float()
        want, tol = float(k16), 0.0
        if kind.startswith("int8"):
            y = qb.w8_linear(x, q, sc, N, workspace=ws if "ws" in kind else None)
        elif kind.startswith("bf16"):
            y = qb.bf16_linear(x, w16, N, workspace=ws if "ws" in kind else None)
        elif kind.startswith("w8a8"):
            y, tol = qb.w8a8_linear(x, q, sc, N, smooth=sm if "smooth" in kind else None), 2.0 ** -7    # 127 K (1 / 127): one ulp
        elif kind == "int4":
            y = qb.w4_linear(x, qb.quantize_weights_w4(torch.full((N, K), 7.0, device=dev)), N)
            want = float(torch.tensor(7.0 * K).bfloat16())
        elif kind.startswith("norm") and "swiglu" not in kind:
            r = res if "residual" in kind else None
            y = qb.w8_linear_fused(x, q, sc, N, gamma=gamma, eps=0.0, residual=r)
            want = float((k16 + 3.0).bfloat16()) if r is not None else want
        elif kind == "residual":
            y, want = qb.w8_linear_fused(x, q, sc, N, residual=res), float((k16 + 3.0).bfloat16())
        elif "swiglu" in kind:
            y = qb.w8_gateup_swiglu(x, q, sc, N // 2, gamma=gamma if "norm" in kind else None, eps=0.0)
            want = float((k16 * k16).bfloat16())                 # silu(K) = K from K = 64 on
        elif kind == "sampled head":
            acc, tok, pd = qb.lmhead_verify_sample(x, q, sc, N, draft, 1.0, ua, us)
            assert int(acc) == 0 and 0 < int(tok) < N and torch.allclose(pd, torch.full_like(pd, 1.0 / N), rtol=1e-5), K
            continue
        else:
            fn = {"head int8": lambda: qb.lmhead_verify(x, q, sc, N, draft, ws), "head bf16": lambda: qb.bf16_lmhead_verify(x, w16, N, draft, ws),
                  "head w8a8": lambda: qb.w8a8_lmhead_verify(x, q, sc, N, draft, ws, smooth=sm),
                  "head int4": lambda: qb.w4_lmhead_verify(x, qb.quantize_weights_w4(torch.full((N, K), 7.0, device=dev)), N, draft, ws)}[kind]
            am, acc = fn()
            assert not am.any() and int(acc) == M - 1, K          # equal logits: the lowest index
            continue
        err = float((y.float() - want).abs().max())
        assert err <= tol * want, (K, err, want)
