"""Rules of the host code that a size query shows (no GPU: they count 256 compute units then)."""
import pytest


@pytest.fixture(scope="module")
def lib():
    from paper_2603_01399_amd import binding
    return binding.lib()


# (M, N, K) int8 and the least and most slices among those near the best time that was measured, of one call and of calls from the host
@pytest.mark.parametrize("M,N,K,least,most", [(8, 3072, 14336, 4, 4), (16, 1024, 25600, 7, 8), (32, 1024, 16384, 8, 8), (20, 512, 5248, 6, 6),
                                              (12, 3072, 9216, 1, 1), (1, 2048, 9216, 1, 1), (6, 512, 9216, 1, 1), (1, 512, 9216, 1, 1)])
def test_slices_of_a_long_k(lib, M, N, K, least, most):
    """Many slices where the second launch is cheap beside them; one where it is not, or the kernel ends before the host has launched twice."""
    slices = lib.quasar_w8_fused_workspace_bytes(M, N, K, 0, 1) // (4 * M * N) or 1
    assert least <= slices <= most


@pytest.mark.parametrize("M,I,K", [(32, 28672, 8192), (32, 16384, 6144), (9, 2048, 4160), (8, 2048, 8256), (32, 2048, 2112), (17, 16, 2112), (32, 2048, 2048)])
def test_scratch_of_the_gateup_form(lib, M, I, K):
    """Normalised activations and nothing else: the form never splits K."""
    apart = K > (8192 if M <= 8 else 4096 if M <= 16 else 2048)
    assert lib.quasar_w8_gateup_workspace_bytes(M, I, K, 1) == (2 * M * K if apart else 0)
    assert lib.quasar_w8_gateup_workspace_bytes(M, I, K, 0) == 0
    for bad in ((M, I + 8, K), (M, 0, K), (M, -16, K), (M, 1 << 26, K), (33, I, K), (M, I, K + 1), (M, 1 << 62, K)):
        assert lib.quasar_w8_gateup_workspace_bytes(*bad, 1) == 0


# where a call is so short that it is the host that launches it which bounds it, and where the activations' registers do
@pytest.mark.parametrize("M,N,K,apart", [(17, 16, 1024, False), (24, 4096, 1024, False), (25, 16, 1024, True), (32, 1024, 1024, True), (17, 16, 1088, True),
                                         (9, 16, 5120, False), (9, 16, 5184, True), (8, 4096, 8192, False), (1, 4096, 8256, False),
                                         (8, 1024, 10240, False), (8, 8192, 8256, True), (8, 8192, 9216, False), (8, 12288, 9216, True),
                                         (8, 25600, 10240, False), (1, 16, 10304, True), (8, 4096, 12288, True)])
def test_w8a8_quantised_apart(lib, M, N, K, apart):
    assert (lib.quasar_w8a8_workspace_bytes(M, N, K) > 0) == apart


@pytest.mark.parametrize("M,N,K,split", [(17, 16, 4224, False), (32, 256, 5120, False), (32, 1024, 4608, False), (32, 512, 5120, False), (32, 1024, 5120, True),
                                         (32, 2048, 5120, False), (32, 4096, 5120, False), (32, 4112, 4224, True), (17, 16, 5248, True), (16, 256, 8320, True)])
def test_w4_split(lib, M, N, K, split):
    assert (lib.quasar_w4_workspace_bytes(M, N, K) > 0) == split


@pytest.mark.parametrize("M,N,K,split", [(9, 16, 5184, False), (16, 1024, 6144, False), (16, 1024, 6400, True), (32, 256, 4096, True)])
def test_w8a8_split(lib, M, N, K, split):
    head = K // 64 * 64 * (8 if M <= 8 else 16 if M <= 16 else 32) + 128
    assert (lib.quasar_w8a8_workspace_bytes(M, N, K) > head) == split
