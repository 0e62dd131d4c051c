"""Small products of more than 64 rows on the kernel of 16 x 16 blocks, against the oracle: edges of blocks and slices,
K split over blocks, the accumulating call, and both sides of the dispatch's lines."""
import numpy as np
import pytest

from tests.gpu_util import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_10949_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def ro():
    from oracle import ring_oracle
    return ring_oracle


@pytest.fixture(scope="module")
def wl():
    from paper_2104_10949_amd import workloads
    return workloads


SHAPES = [(65, 1, 2), (66, 17, 34), (128, 128, 784), (127, 129, 62), (1000, 10, 130), (300, 33, 1026), (128, 10, 2048),
          (80, 16, 9000),                        # K split over blocks
          (12288, 16, 64), (12289, 16, 64),      # 768 blocks of z, and one row of them more
          (8208, 16, 32), (12288, 16, 98), (96, 768, 416), (96, 768, 418),   # lines of three and of two rounds
          (320, 29, 3680),                       # K split, and the grid still one round
          (96, 768, 512), (96, 769, 512)]        # 4608 (block, slice) units, and beyond


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_small_products(cg, ro, wl, M, N, K):
    say(f"small product M={M} N={N} K={K}")
    ops = [wl.draw_ring((r, K), 9600 + i) for i, r in enumerate((M, M, N, N))]
    dev = [cg.to_device(a) for a in ops]
    want = ro.party_matmul(*ops)
    assert np.array_equal(cg.to_host(cg.cg_share_matmul(*dev)), want)
    base = wl.draw_ring((M, N), 9610)
    got = cg.to_device(base)
    cg.cg_share_matmul_acc(*dev, got)
    assert np.array_equal(cg.to_host(got), base + want)
