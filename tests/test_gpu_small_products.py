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


# blocks of 8 x 8, 8 x 16 and 16 x 8 up to a full round, and one block more
BLOCKS = [(8, 8, 2), (9, 7, 34), (7, 9, 600), (128, 128, 32), (128, 136, 62), (1032, 24, 70), (2048, 8, 34), (2056, 8, 34), (8, 4096, 66),
          (24, 1368, 34)]


@pytest.mark.parametrize("M,N,K", BLOCKS)
def test_blocks_of_eight(cg, ro, wl, M, N, K):
    test_small_products(cg, ro, wl, M, N, K)


# odd K and operands at odd words: pairs of the left operand that reach into the next row, the last of them into the end of the
# tensor; split over blocks, streamed over tiles of unequal slices, whole tiles streamed
ODD = [(1, 130, 33), (129, 65, 31), (1000, 77, 1531), (700, 1030, 2051), (40000, 64, 33), (128, 64, 1), (257, 700, 95)]


@pytest.mark.parametrize("M,N,K", ODD)
@pytest.mark.parametrize("at", [0, 1])
def test_rows_of_odd_length(cg, ro, wl, M, N, K, at):
    say(f"odd rows M={M} N={N} K={K} first word {at}")
    ops = [wl.draw_ring((r, K), 9650 + i) for i, r in enumerate((M, M, N, N))]
    dev = []
    for a in ops:   # behind the last word lies something else
        whole = torch.full((a.size + at + 8,), -1, dtype=torch.int64, device="cuda")
        whole[at:at + a.size].copy_(cg.to_device(a).view(-1))
        dev.append(whole[at:at + a.size].view(*a.shape))
    got = cg.cg_share_matmul(*dev)
    rows = sorted({i for i in (0, 1, 127, 128, 129, M // 2, M - 2, M - 1) if 0 <= i < M})
    want = ro.party_matmul(ops[0][rows], ops[1][rows], ops[2], ops[3])
    assert np.array_equal(cg.to_host(got[rows].contiguous()), want)
