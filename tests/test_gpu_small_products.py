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
# tensor; unsplit, split over blocks, whole tiles streamed, and (ODD_STREAMED) runs of slices that begin and end inside a tile
ODD = [(1, 130, 33), (129, 65, 31), (1000, 77, 1531), (700, 1030, 2051), (40000, 64, 33), (128, 64, 1), (257, 700, 95)]
ODD_STREAMED = [(1, 5975, 591), (1568, 256, 2305), (16507, 127, 1055)]


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


@pytest.mark.parametrize("M,N,K", ODD_STREAMED)
@pytest.mark.parametrize("at", [0, 1])
def test_rows_of_odd_length_streamed(cg, ro, wl, M, N, K, at):
    test_rows_of_odd_length(cg, ro, wl, M, N, K, at)


@pytest.mark.parametrize("M,N,K", ODD_STREAMED)
def test_rows_of_odd_length_streamed_and_added(cg, wl, M, N, K):
    say(f"odd rows added M={M} N={N} K={K}")
    dev = [cg.to_device(wl.draw_ring((r, K), 9660 + i)) for i, r in enumerate((M, M, N, N))]
    base = cg.to_device(wl.draw_ring((M, N), 9664))
    got = cg.cg_share_matmul_acc(*dev, base.clone())
    assert torch.equal(got, base + cg.cg_share_matmul(*dev))   # (the product itself: see above)


# more than one round of unsplit tiles whose last one is shared out: first layers and a weight gradient, one tile to half a round
# of them left over, in parts of one slice or several, the last one shorter; plainly stored and added
TAIL_LAYERS = [((3, 105, 105, 5), (64, 5, 5, 5), (1, 1), (2, 2)), ((1, 104, 106, 3), (130, 7, 7, 3), (1, 1), (3, 3)),
               ((1, 182, 181, 7), (64, 5, 5, 7), (1, 1), (2, 2)), ((3, 128, 128, 10), (64, 5, 5, 10), (1, 1), (2, 2)),
               ((1, 213, 213, 11), (64, 5, 5, 11), (1, 1), (2, 2)), ((1, 204, 204, 24), (60, 3, 3, 24), (1, 1), (1, 1)),
               ((1, 198, 198, 27), (61, 3, 3, 27), (1, 1), (1, 1))]


@pytest.mark.parametrize("xs,ws,st,pd", TAIL_LAYERS)
def test_last_round_of_a_first_layer(cg, ro, wl, xs, ws, st, pd):
    say(f"split tail conv x={xs} w={ws}")
    ops = [wl.draw_ring(s, 9680 + i) for i, s in enumerate((xs, xs, ws, ws))]
    dev = [cg.to_device(a) for a in ops]
    z = torch.full(cg.conv_out_shape(xs, ws, st, pd), 77, dtype=torch.int64, device="cuda")
    got = cg.cg_share_conv2d(*dev, stride=st, pad=pd, z_i=z)
    want = ro.party_conv2d(*ops, st, pd)
    assert np.array_equal(cg.to_host(got), want)
    base = wl.draw_ring(tuple(got.shape), 9690)
    acc = cg.to_device(base)
    cg.cg_share_conv2d_acc(*dev, acc, stride=st, pad=pd)
    assert np.array_equal(cg.to_host(acc), base + want)


TAIL_GRADIENTS = [(4200, 512, 140), (257 * 128, 64, 129), (128 * 64 + 1, 256, 200), (3071, 1023, 250), (11387, 256, 285),
                  (20864, 128, 224), (307 * 128 - 1, 64, 256)]


@pytest.mark.parametrize("M,N,K", TAIL_GRADIENTS)
def test_last_round_of_a_weight_gradient(cg, ro, wl, M, N, K):
    say(f"split tail matmul_t M={M} N={N} K={K}")
    ops = [wl.draw_ring((K, r), 9695 + i) for i, r in enumerate((M, M, N, N))]
    z = torch.full((M, N), 77, dtype=torch.int64, device="cuda")
    got = cg.cg_share_matmul_t(*[cg.to_device(a) for a in ops], True, True, z_i=z)
    plain = cg.cg_share_matmul(*[cg.to_device(np.ascontiguousarray(a.T)) for a in ops])
    assert torch.equal(got, plain)
    want = ro.party_matmul(*[np.ascontiguousarray(a.T)[-130:] for a in ops[:2]], *[np.ascontiguousarray(a.T) for a in ops[2:]])
    assert np.array_equal(cg.to_host(got[-130:].contiguous()), want)
