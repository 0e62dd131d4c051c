"""Gradients of fully connected layers at small batch (the right operand stored transposed) on their own kernels, against the
oracle: edges of 32-column blocks and 16-row blocks, runs of column blocks of unequal length, K that ends inside a slice."""
import numpy as np
import pytest

from tests.gpu_util import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# one slice of K, both operands transposed; the last ones take more than one block of columns per wave
OUTER = [(2, 2, 1), (10, 34, 8), (32, 32, 32), (34, 66, 31), (130, 2050, 17), (512, 1026, 32), (512, 8194, 32), (2050, 4098, 3)]
# few rows on the left: one and two row blocks, several groups of them; one turn of a wave and several, waves with a turn less and waves
# without a slice (see test_gradients_of_small_batches_run_on_their_own_kernels)
ROWS = [(1, 2, 2), (16, 32, 32), (17, 34, 34), (32, 8194, 66), (3, 1000, 258), (512, 66, 62), (32, 8192, 512), (31, 8194, 514),
        (33, 2050, 258), (70, 2562, 162), (96, 2050, 130), (10, 4098, 1024)]
# ... as long as the rule takes them at these widths
LONG_ROWS = [(8, 8194, 4098), (32, 8194, 1026)]
# what neither takes: odd columns, odd rows, more rows or fewer columns than pay
OTHERS = [(33, 65, 32, True), (35, 66, 16, True), (32, 33, 64, False), (300, 66, 1000, False), (31, 130, 1000, False), (48, 4098, 34, False)]


@pytest.fixture(scope="module")
def cg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_10949_amd import binding
    binding.lib()
    return binding


def check(cg, M, N, K, trans_x, at=0):
    from oracle import ring_oracle as ro
    from paper_2104_10949_amd import workloads as wl
    say(f"fully connected gradient M={M} N={N} K={K} trans_x={trans_x} first word {at}")
    ops = [wl.draw_ring((K, M) if trans_x else (M, K), 9900 + i) for i in range(2)] + [wl.draw_ring((K, N), 9902 + i) for i in range(2)]

    def place(a):
        t = torch.zeros(a.size + at, dtype=torch.int64, device="cuda")[at:].view(*a.shape)
        t.copy_(cg.to_device(a))
        return t
    z = torch.full((M * N + 64,), 0x5A5A5A5A, dtype=torch.int64, device="cuda")
    got = cg.cg_share_matmul_t(*[place(a) for a in ops], trans_x, True, z_i=z[:M * N].view(M, N))
    rows = sorted({i for i in (0, 1, 2, 15, 16, 17, 31, 32, 33, M // 2, M - 2, M - 1) if 0 <= i < M})
    left = [np.ascontiguousarray(a.T if trans_x else a)[rows] for a in ops[:2]]
    want = ro.party_matmul(*left, *[np.ascontiguousarray(a.T) for a in ops[2:]])
    assert np.array_equal(cg.to_host(got[rows].contiguous()), want)
    plain = cg.cg_share_matmul(*[cg.to_device(np.ascontiguousarray(a.T if trans_x else a)) for a in ops[:2]],
                               *[cg.to_device(np.ascontiguousarray(a.T)) for a in ops[2:]])
    assert torch.equal(got, plain)
    assert bool((z[M * N:] == 0x5A5A5A5A).all())


@pytest.mark.parametrize("M,N,K", OUTER)
def test_weight_gradient(cg, M, N, K):
    check(cg, M, N, K, True)


@pytest.mark.parametrize("M,N,K", ROWS)
def test_input_gradient(cg, M, N, K):
    check(cg, M, N, K, False)


@pytest.mark.parametrize("M,N,K", LONG_ROWS)
def test_input_gradient_of_extreme_words(cg, M, N, K):
    """Every digit of the left operand's sum and of the right operand -128, the largest products, against the ring product of
    the words; and random words."""
    check(cg, M, N, K, False)
    say(f"fully connected gradient of extreme words M={M} N={N} K={K}")
    word = 0x7F7F7F7F7F7F7F80
    x = torch.full((M, K), word, dtype=torch.int64, device="cuda")
    w = torch.full((K, N), word, dtype=torch.int64, device="cuda")
    got = cg.cg_share_matmul_t(x, torch.zeros_like(x), w, torch.zeros_like(w), False, True)
    want = K * word * word % (1 << 64)
    assert bool((got == (want - (1 << 64) if want >> 63 else want)).all())


@pytest.mark.parametrize("M,N,K,trans_x", OTHERS)
def test_shapes_of_the_tiled_kernel(cg, M, N, K, trans_x):
    check(cg, M, N, K, trans_x)


@pytest.mark.parametrize("trans_x", [True, False])
def test_operands_at_odd_words(cg, trans_x):
    check(cg, 32, 64, 32, trans_x, at=1)
