"""Rules of the host code that a size query shows (no GPU: they count 256 compute units then)."""
import pytest


@pytest.fixture(scope="module")
def lib():
    from paper_2603_01399_amd import binding
    return binding.lib()


# (M, N, K) int8 and the least and most slices among those within 3 % of the best time that was measured
@pytest.mark.parametrize("M,N,K,least,most", [(16, 256, 16384, 8, 8), (16, 256, 25600, 7, 8), (16, 1024, 25600, 7, 8), (6, 512, 9216, 1, 1),
                                              (1, 512, 9216, 1, 1)])
def test_slices_of_a_long_k(lib, M, N, K, least, most):
    """Many slices where the second launch is cheap beside them; one where the kernel ends before the host has launched twice."""
    slices = lib.quasar_w8_fused_workspace_bytes(M, N, K, 0, 1) // (4 * M * N) or 1
    assert least <= slices <= most
