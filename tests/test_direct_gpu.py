"""The streaming kernel that holds its activations in registers: every register form (slots of 64 k per wave), ragged shares
of K over the waves, tile remainders, both weight types.  Without a workspace its sums are taken in the order of the kernel
that stages the activations in LDS, so the two must agree bit for bit; with one, and for the fused forms, the outputs are held
to the bar of the linear (one bf16 rounding of an fp32 sum: 4e-3 of max|y|) against a 64-bit product of the same codes."""
import pytest
import torch

from paper_2603_01399_amd import synth
from gpu_util import bf16_to_dev, f32_to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qb():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2603_01399_amd import binding
    return binding


def bits(t):
    return t.contiguous().view(torch.int16)


def rel(y, want):
    return float((y.double() - want).abs().max() / want.abs().max())


def make(qb, M, N, K):
    x = bf16_to_dev(synth.activations_bf16(M, K, seed=synth.seed_for(20, M, K)))
    w = f32_to_dev(synth.normal_weights(N, K, seed=synth.seed_for(21, M, K)))
    wq, sc = qb.quantize_weights(w)
    what = qb.unpack_weights(wq, N, K).double() * sc.double()[:, None]
    return x, w, wq, sc, what


# K: one step; fewer steps than waves; 17, 33, 49, 65, 81 steps (two to six slots, ragged); seven and eight slots; two chunks of
# them; 129 and 160 steps (ten slots, and the twenty of eight waves at 9 to 16 tokens, ragged and full); twelve and 24
KS = [64, 960, 1088, 2112, 3136, 4160, 5184, 6208, 7168, 7680, 8192, 8256, 10240, 12288]


@pytest.mark.parametrize("K", KS)
@pytest.mark.parametrize("M,N", [(1, 16), (8, 16 * 261), (9, 16 * 261), (16, 16 * 40), (17, 16 * 261), (32, 16 * 40)])
def test_linear_forms(qb, M, N, K):
    print("direct linear", M, N, K, flush=True)
    x, w, wq, sc, what = make(qb, M, N, K)
    want = x.double() @ what.t()
    wp = qb.pack_bf16_weights(w)
    want16 = x.double() @ w.to(torch.bfloat16).double().t()
    ws = qb.make_workspace(M, N, K)
    ws.fill_(0xFF)
    plain, plain16 = qb.w8_linear(x, wq, sc, N), qb.bf16_linear(x, wp, N)
    free, free16 = qb.w8_linear(x, wq, sc, N, workspace=ws), qb.bf16_linear(x, wp, N, workspace=ws)
    for y, ref in ((plain, want), (free, want), (plain16, want16), (free16, want16)):
        assert rel(y, ref) <= 4e-3
    qb.set_tuning(16, 2, 4)                    # two workgroups per compute unit: the staged kernel
    try:
        staged, staged16 = qb.w8_linear(x, wq, sc, N), qb.bf16_linear(x, wp, N)
    finally:
        qb.set_tuning(16, 1, 4)
    assert torch.equal(bits(plain), bits(staged)) and torch.equal(bits(plain16), bits(staged16))


@pytest.mark.parametrize("K", [64, 1088, 3136, 4160, 6208, 7168, 8256, 10240, 12288])
@pytest.mark.parametrize("M", [3, 8, 16, 32])
def test_fused_forms(qb, M, K):
    N = 16 * 22
    print("direct fused", M, N, K, flush=True)
    x, _, wq, sc, what = make(qb, M, N, K)
    gamma = bf16_to_dev(synth.activations_bf16(1, K, seed=synth.seed_for(22, M, K)))[0].contiguous()
    res = bf16_to_dev(synth.activations_bf16(M, N, seed=synth.seed_for(23, M, K)))
    xd = x.double()
    norm = ((xd * torch.rsqrt((xd * xd).mean(1, keepdim=True) + 1e-6)).bfloat16().double() * gamma.double()).bfloat16().double()
    lin = norm @ what.t()
    assert rel(qb.w8_linear_fused(x, wq, sc, N, gamma=gamma, eps=1e-6), lin) <= 6e-3
    assert rel(qb.w8_linear_fused(x, wq, sc, N, gamma=gamma, eps=1e-6, residual=res), lin.bfloat16().double() + res.double()) <= 6e-3
    assert rel(qb.w8_linear_fused(x, wq, sc, N, residual=res), (xd @ what.t()).bfloat16().double() + res.double()) <= 6e-3
    gu = lin.bfloat16().double().view(M, N // 32, 2, 16)
    act = (torch.nn.functional.silu(gu[:, :, 0]).bfloat16().double() * gu[:, :, 1]).reshape(M, N // 2)
    assert rel(qb.w8_gateup_swiglu(x, wq, sc, N // 2, gamma=gamma, eps=1e-6), act) <= 1e-2


@pytest.mark.parametrize("M,N,K", [(32, 16 * 22, 4096), (32, 16 * 1026, 5120), (27, 16 * 1026, 4160)])
def test_fused_norm_of_many_tokens(qb, M, N, K):
    """The normalised forms of 17 to 32 tokens: eight slots a wave, and ten where there are many tiles."""
    print("direct fused norm", M, N, K, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(N + K)
    x = torch.randn(M, K, generator=gen, device="cuda").bfloat16()
    gamma = (1 + 0.2 * torch.randn(K, generator=gen, device="cuda")).bfloat16()
    wq, sc = qb.quantize_weights(torch.randn(N, K, generator=gen, device="cuda") * 0.02)
    what = qb.unpack_weights(wq, N, K).float() * sc.float()[:, None]
    xd = x.double()
    norm = ((xd * torch.rsqrt((xd * xd).mean(1, keepdim=True) + 1e-6)).bfloat16().double() * gamma.double()).bfloat16()
    lin = torch.cat([norm.double() @ what[i:i + 4096].double().t() for i in range(0, N, 4096)], 1)
    assert rel(qb.w8_linear_fused(x, wq, sc, N, gamma=gamma, eps=1e-6), lin) <= 6e-3
    gu = lin.bfloat16().double().view(M, N // 32, 2, 16)
    act = (torch.nn.functional.silu(gu[:, :, 0]).bfloat16().double() * gu[:, :, 1]).reshape(M, N // 2)
    assert rel(qb.w8_gateup_swiglu(x, wq, sc, N // 2, gamma=gamma, eps=1e-6), act) <= 1e-2


@pytest.mark.parametrize("M", [2, 9, 17])
def test_sampling_statistics_taken_while_streaming(qb, M):
    """Softmax statistics per workgroup of the streaming kernel against those taken from the finished logits (a workspace with
    room for no more): the same decisions and token, probabilities within a few fp32 roundings of sums of 4800 terms."""
    V, K = 16 * 300, 512
    print("direct sampling", M, V, K, flush=True)
    x, _, wq, sc, what = make(qb, M, V, K)
    p = torch.softmax(x.double() @ what.t() / 0.8, 1)
    draft = p.argmax(1).int()[:-1].contiguous()
    ua = (p.max(1).values * 0.9).float()
    ua[M // 2] = 0.999
    us = torch.rand(M, device="cuda")
    full = qb.lmhead_verify_sample(x, wq, sc, V, draft, 0.8, ua, us)
    least = torch.empty(M * V * 4 + 32 * 32 * 2 * 4, dtype=torch.uint8, device="cuda")
    small = qb.lmhead_verify_sample(x, wq, sc, V, draft, 0.8, ua, us, workspace=least)
    assert int(full[0]) == int(small[0]) and int(full[1]) == int(small[1])
    assert torch.allclose(full[2], small[2], rtol=1e-5, atol=0)
    assert torch.allclose(full[2].double(), p[:-1].gather(1, draft.long()[:, None])[:, 0], rtol=1e-3, atol=0)


# K: one step; one slot a wave; pairs of shares that begin in the middle of a slot (bf16), up to the longest K in one piece
@pytest.mark.parametrize("K", [64, 512, 576, 960, 1024, 1088, 1216, 1344, 1408])
@pytest.mark.parametrize("M,N", [(17, 16), (17, 16 * 261), (32, 16 * 600)])
def test_order_of_many_tokens(qb, M, N, K):
    """More than 16 tokens, K in one piece: a workspace changes nothing, and the sums are those of the staged kernel."""
    print("direct order", M, N, K, flush=True)
    x, w, wq, sc, _ = make(qb, M, N, K)
    wp = qb.pack_bf16_weights(w)
    ws = qb.make_workspace(M, N, K)
    plain, plain16 = qb.w8_linear(x, wq, sc, N), qb.bf16_linear(x, wp, N)
    assert torch.equal(bits(plain), bits(qb.w8_linear(x, wq, sc, N, workspace=ws)))
    assert torch.equal(bits(plain16), bits(qb.bf16_linear(x, wp, N, workspace=ws)))
    am, am16 = (f(None, ws)[0] for f in (lambda d, s: qb.lmhead_verify(x, wq, sc, N, d, s),
                                         lambda d, s: qb.bf16_lmhead_verify(x, wp, N, d, s)))
    qb.set_tuning(16, 2, 4)
    try:
        assert torch.equal(bits(plain), bits(qb.w8_linear(x, wq, sc, N)))
        assert torch.equal(bits(plain16), bits(qb.bf16_linear(x, wp, N)))
        assert torch.equal(am, qb.lmhead_verify(x, wq, sc, N, None, ws)[0])
        assert torch.equal(am16, qb.bf16_lmhead_verify(x, wp, N, None, ws)[0])
    finally:
        qb.set_tuning(16, 1, 4)


@pytest.mark.parametrize("M,K", [(1, 12288), (16, 8192), (32, 4096)])
def test_a_workspace_too_small_changes_nothing(qb, M, K):
    """K in several pieces, but no room for the partial sums: the order of the call without a workspace."""
    N = 16 * 4400
    print("direct small workspace", M, N, K, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(K)
    x = torch.randn(M, K, generator=gen, device="cuda").bfloat16()
    wq = torch.randint(-127, 128, (N * K,), generator=gen, device="cuda", dtype=torch.int8)
    sc = torch.full((N,), 0.01, dtype=torch.bfloat16, device="cuda")
    small = torch.empty(4 * M * N, dtype=torch.uint8, device="cuda")
    assert torch.equal(bits(qb.w8_linear(x, wq, sc, N)), bits(qb.w8_linear(x, wq, sc, N, workspace=small)))


@pytest.mark.parametrize("M,V,K", [(9, 16 * 256 * 17, 1024), (16, 16 * 256 * 17, 4096), (16, 16 * 600, 8256), (16, 16 * 600, 12288),
                                   (32, 16 * 256 * 17, 1024), (32, 16 * 600, 4096), (32, 16 * 600, 5120)])
def test_sampling_statistics_over_many_tiles(qb, M, V, K):
    """The running softmax statistics over several tiles of a wave (17 tiles a workgroup of 16 or 8 waves), two blocks of
    tokens and the longer forms."""
    print("direct sampling, many tiles", M, V, K, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(V + K)
    x = torch.randn(M, K, generator=gen, device="cuda").bfloat16()
    wq, sc = qb.quantize_weights(torch.randn(V, K, generator=gen, device="cuda") * (2.0 / K ** 0.5))
    what = qb.unpack_weights(wq, V, K).float() * sc.float()[:, None]
    logits = torch.cat([x.double() @ what[i:i + 4096].double().t() for i in range(0, V, 4096)], 1)
    p = torch.softmax(logits / 0.8, 1)
    draft = p.argmax(1).int()[:-1].contiguous()
    ua = (p.max(1).values * 0.9).float()
    ua[M // 2] = 0.999
    us = torch.rand(M, generator=gen, device="cuda") * 0.98 + 0.01
    full = qb.lmhead_verify_sample(x, wq, sc, V, draft, 0.8, ua, us)
    least = torch.empty(M * V * 4 + 32 * 32 * 2 * 4, dtype=torch.uint8, device="cuda")
    small = qb.lmhead_verify_sample(x, wq, sc, V, draft, 0.8, ua, us, workspace=least)
    assert int(full[0]) == int(small[0]) == M // 2
    assert torch.allclose(full[2], small[2], rtol=1e-5, atol=0)
    assert torch.allclose(full[2].double(), p[:-1].gather(1, draft.long()[:, None])[:, 0], rtol=1e-3, atol=0)
    # either token covers the drawn point as the 64-bit sums have it, within 1e-4 of the mass (fp32 logits and sums)
    mass = p[M // 2].clone()
    mass[int(draft[M // 2])] = 0.0
    c = torch.cumsum(mass, 0)
    for tok in (int(full[1]), int(small[1])):
        point = float(us[M // 2]) * float(c[-1])
        assert 0 <= tok < V and float(c[tok] - mass[tok]) - 1e-4 * float(c[-1]) <= point < float(c[tok]) + 1e-4 * float(c[-1])


def test_rounding_of_the_normalised_activations(qb):
    """The pair conversion of the fused normalisation rounds to nearest, ties to even, over the exponents of bf16: the products
    of all pairs of 8-bit significands, read back through a weight matrix that picks one channel per row.

    x are whole numbers whose squares have the mean 2^14 exactly, so the normalised x are x / 128 exactly and gamma's product with
    them is the only rounding.  Row n has code 1 at channel n and 127 at a channel whose input is zero (its step size is
    1), so y[m, n] is that channel's operand itself."""
    print("rounding of normalised activations", flush=True)
    K, live = 256, 128                                            # channels 128 .. 255 are zero
    w = torch.zeros(live, K, device="cuda")
    w[:, :live] = torch.eye(live, device="cuda")
    w[:, K - 1] = 127.0
    wq, sc = qb.quantize_weights(w)
    assert bool((sc == 1).all())
    gen = torch.Generator().manual_seed(3)
    for trial in range(8):
        # 124 numbers of 8 bits, then four squares that complete the sum of 256 x 2^14 = 128 x 32768 (Lagrange)
        v = torch.randint(128, 232, (live - 4,), generator=gen)
        left = K * 2 ** 14 - int((v * v).sum())
        while not 20000 <= left <= 150000:
            i = int(torch.randint(live - 4, (1,), generator=gen))
            v[i] = min(255, max(128, int(v[i]) + (8 if left > 85000 else -8)))
            left = K * 2 ** 14 - int((v * v).sum())
        four = four_squares(left)
        x = torch.zeros(1, K)
        x[0, :live] = torch.cat([v, torch.tensor(four)]).float()
        sign = torch.where(torch.rand(K, generator=gen) < 0.5, -1.0, 1.0)
        x = (x * sign).bfloat16()
        assert int((x.double() ** 2).sum()) == K * 2 ** 14
        for e in (-100, -30, -1, 0, 7, 60, 110):
            gamma = (torch.randint(128, 256, (K,), generator=gen).float() * 2.0 ** (e - 7)).bfloat16()
            exact = x.double() / 128 * gamma.double()
            want = exact.float().bfloat16()                       # 16-bit products: exact in fp32, rounded once, ties to even
            y = qb.w8_linear_fused(x.cuda(), wq, sc, live, gamma=gamma.cuda(), eps=0.0)
            assert torch.equal(bits(y.cpu()), bits(want[:, :live])), (trial, e)


def four_squares(n):
    """Four whole numbers up to 255 whose squares add up to n."""
    for a in range(min(255, int(n ** 0.5)), -1, -1):
        for b in range(min(255, int((n - a * a) ** 0.5)), -1, -1):
            r = n - a * a - b * b
            if r > 2 * 255 ** 2:
                break
            for c in range(min(255, int(r ** 0.5)), -1, -1):
                d = int(round((r - c * c) ** 0.5))
                if c * c + d * d == r and d <= 255:
                    return [a, b, c, d]
    raise AssertionError(n)


# K: two to five chunks, of 12 to 16 steps, a short last one; tiles: one, several a workgroup and a remainder
@pytest.mark.parametrize("K", [1472, 1536, 2048, 2560, 3072, 3136, 4096, 4160, 5120])
@pytest.mark.parametrize("M,V", [(17, 16), (32, 16 * 261), (24, 16 * 1100)])
def test_order_of_many_tokens_in_chunks(qb, M, V, K):
    """More than 16 tokens, K in chunks: argmax and accepted length of rows whose exact logits are equal (the winner is the row
    whose sum rounds up most, so it shows the order of the sum) are those of the staged kernel."""
    print("direct chunks", M, V, K, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(K + V)
    half = torch.randn(M, K // 2, generator=gen, device="cuda").bfloat16()
    x = torch.cat([half, half], 1).contiguous()
    codes = torch.randint(-127, 128, (K,), generator=gen, device="cuda").float()
    codes[0] = 127.0
    swap = torch.rand(V, K // 2, generator=gen, device="cuda") < 0.5
    lo, hi = codes[:K // 2].expand(V, -1), codes[K // 2:].expand(V, -1)
    w = torch.cat([torch.where(swap, hi, lo), torch.where(swap, lo, hi)], 1) / 128.0
    wq, sc = qb.quantize_weights(w)
    wp = qb.pack_bf16_weights(w)
    ws = qb.make_workspace(M, V, K)
    draft = torch.zeros(M - 1, dtype=torch.int32, device="cuda")
    now = [t.clone() for f in (lambda: qb.lmhead_verify(x, wq, sc, V, draft, ws), lambda: qb.bf16_lmhead_verify(x, wp, V, draft, ws)) for t in f()]
    qb.set_tuning(16, 2, 4)
    try:
        staged = [t.clone() for f in (lambda: qb.lmhead_verify(x, wq, sc, V, draft, ws), lambda: qb.bf16_lmhead_verify(x, wp, V, draft, ws)) for t in f()]
    finally:
        qb.set_tuning(16, 1, 4)
    assert all(torch.equal(a, b) for a, b in zip(now, staged))
    assert V == 16 or len(set(now[0].tolist())) > M // 2
