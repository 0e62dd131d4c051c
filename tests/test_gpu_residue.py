"""The residue route of the workspace entry points (share_gemm_rns.hip) against the oracle, bit for bit.

The route is taken where it is the faster one and the scratch memory holds it: cg_*_workspace_bytes then asks for more
than the digit planes take.  Every output is compared with the plain kernel's, rows of it with the oracle's.
"""
import threading

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


def poisoned(nbytes):
    return torch.full((nbytes // 8 + 2,), 0x5A5A5A5A5A5A5A5A, dtype=torch.int64, device="cuda")


def sampled(n):   # edges of tiles and a few others
    return sorted({i for i in (0, 1, 15, 16, 127, 128, 255, 256, n // 2, n - 17, n - 2, n - 1) if 0 <= i < n})


# the small tile, the large one, multiples of nothing, the longest K of 18 moduli and the first of 19
SHAPES = [(1150, 1145, 3001), (1023, 2047, 3001), (2048, 2048, 2048), (3001, 2047, 2050), (2048, 2048, 5500),
          (1290, 1283, 5501), (1800, 2040, 9002),
          (1167, 1361, 3048), (1214, 1361, 957), (770, 1691, 5739)]   # the small tile with 18 and 19 moduli


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_matmul(cg, ro, wl, M, N, K):
    say(f"residue route matmul M={M} N={N} K={K}")
    need = cg.cg_share_matmul_workspace_bytes(M, N, K)
    assert cg.cg_share_matmul_prefers_workspace(M, N, K) and need > cg.cg_share_matmul_digit_workspace_bytes(M, N, K)
    ops = [wl.draw_ring((r, K), 9100 + i) for i, r in enumerate((M, M, N, N))]
    dev = [cg.to_device(a) for a in ops]
    plain = cg.cg_share_matmul(*dev)
    got = cg.cg_share_matmul_ws(*dev, poisoned(need))
    assert torch.equal(got, plain)
    rows = sampled(M)
    want = ro.party_matmul(ops[0][rows], ops[1][rows], ops[2], ops[3])
    assert np.array_equal(cg.to_host(got[rows]), want)


# every modulus on the small tile (see test_every_modulus_runs_on_one_tile...)
SMALL_TILE_SHAPES = [(1077, 1133, 1913)]


@pytest.mark.parametrize("M,N,K", SMALL_TILE_SHAPES)
def test_matmul_on_the_small_tile_alone(cg, ro, wl, M, N, K):
    test_matmul(cg, ro, wl, M, N, K)


@pytest.mark.parametrize("x_word,w_word", [(0x7F7F7F7F7F7F7F80, 0x7F7F7F7F7F7F7F80), (0x7F7F7F7F7F7F7F80, 0x7F7F7F7F7F7F7F7F),
                                           (0x8080808080808080, 0x8080808080808080), (0x7F7F7F7F7F7F7F7F, 0x8080808080808080),
                                           (0x7F7F7F7F7F7F7F7F, 0x7F7F7F7F7F7F7F7F), (0x8000000000000000, 0x8000000000000000),
                                           (0, 0), (1, 0xFFFFFFFFFFFFFFFF)])
@pytest.mark.parametrize("K", [5500, 9000])
def test_largest_integers(cg, x_word, w_word, K):
    """w_b = 0, so both terms of every product are x_word * w_word: with the word of the largest signed-digit value
    (0x7F..7F80, eight digits of -128) and the longest K of 18 moduli the integer is as near to half the moduli's product as
    it gets, 0.4943 of it."""
    M, N = 2048, 2048
    say(f"residue route constant words {x_word:016x} {w_word:016x} K={K}")
    signed = lambda w: w - (1 << 64) if w >> 63 else w
    x = torch.full((M, K), signed(x_word), dtype=torch.int64, device="cuda")
    w = torch.full((N, K), signed(w_word), dtype=torch.int64, device="cuda")
    need = cg.cg_share_matmul_workspace_bytes(M, N, K)
    assert need > cg.cg_share_matmul_digit_workspace_bytes(M, N, K)
    got = cg.cg_share_matmul_ws(x, x, w, torch.zeros_like(w), poisoned(need))
    want = signed(2 * K * x_word * w_word % (1 << 64))
    assert bool((got == want).all())


CONVS = [((32, 16, 16, 256), (256, 3, 3, 256), 1, 1), ((32, 32, 32, 256), (128, 3, 3, 256), 1, 1),
         ((9, 27, 25, 200), (500, 3, 3, 200), 1, 1), ((12, 40, 38, 192), (520, 5, 5, 192), 2, 2)]


@pytest.mark.parametrize("xs,ws,stride,pad", CONVS)
def test_conv(cg, ro, wl, xs, ws, stride, pad):
    say(f"residue route conv x={xs} w={ws} stride={stride} pad={pad}")
    st, pd = (stride, stride), (pad, pad)
    need = cg.cg_share_conv2d_workspace_bytes(xs, ws, st, pd)
    assert cg.cg_share_conv2d_prefers_workspace(xs, ws, st, pd)
    assert need > cg.cg_share_conv2d_digit_workspace_bytes(xs, ws, st, pd)
    ops = [wl.draw_ring(s, 9200 + i) for i, s in enumerate((xs, xs, ws, ws))]
    dev = [cg.to_device(a) for a in ops]
    plain = cg.cg_share_conv2d(*dev, stride=st, pad=pd)
    got = cg.cg_share_conv2d_ws(*dev, poisoned(need), stride=st, pad=pd)
    assert torch.equal(got, plain)
    last = ops[0][-1:], ops[1][-1:]
    want = ro.party_conv2d(*last, ops[2][:40], ops[3][:40], st, pd)
    assert np.array_equal(cg.to_host(got[-1:, :, :, :40].contiguous()), want)


def test_longest_contraction(cg):
    """K at the end of the route, words whose residues modulo 256 are -128 on both sides (the inverse multiplied into the
    right one is odd): 2 * 65000 products of 2^14, 0.992 of what an accumulator holds."""
    M, N, K, word = 2048, 2048, 65000, 0x7F7F7F7F7F7F7F80
    say(f"residue route K={K}, largest accumulators")
    need = cg.cg_share_matmul_workspace_bytes(M, N, K)
    assert need > cg.cg_share_matmul_digit_workspace_bytes(M, N, K)
    assert cg.cg_share_matmul_workspace_bytes(M, N, K + 2) == cg.cg_share_matmul_digit_workspace_bytes(M, N, K + 2)
    x = torch.full((M, K), word, dtype=torch.int64, device="cuda")
    w = torch.full((N, K), word, dtype=torch.int64, device="cuda")
    got = cg.cg_share_matmul_ws(x, x, w, torch.zeros_like(w), poisoned(need))
    want = 2 * K * word * word % (1 << 64)
    assert bool((got == (want - (1 << 64) if want >> 63 else want)).all())


def device_ring(shape, seed):   # drawn on the GPU: gigabytes of words
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return torch.randint(-2 ** 63, 2 ** 63 - 1, shape, dtype=torch.int64, device="cuda", generator=gen)


# residues of one modulus just below 2^31 bytes, on the left, on the right, and gathered
@pytest.mark.parametrize("M,N", [(262142, 512), (512, 262143)])
def test_largest_planes(cg, ro, M, N):
    K = 4096
    say(f"residue route near the limit of a plane M={M} N={N} K={K}")
    more = (M + (M > N), N + (N > M), K)
    assert cg.cg_share_matmul_workspace_bytes(*more) == cg.cg_share_matmul_digit_workspace_bytes(*more)
    need = cg.cg_share_matmul_workspace_bytes(M, N, K)
    assert need > cg.cg_share_matmul_digit_workspace_bytes(M, N, K)
    dev = [device_ring((r, K), 9800 + i) for i, r in enumerate((M, M, N, N))]
    got = cg.cg_share_matmul_ws(*dev, poisoned(need))
    assert torch.equal(got, cg.cg_share_matmul(*dev))
    host = [cg.to_host(t[-40:].contiguous()) for t in dev]
    assert np.array_equal(cg.to_host(got[-40:, -40:].contiguous()), ro.party_matmul(*host))
    del dev, got
    torch.cuda.empty_cache()


def test_largest_gathered_plane(cg, ro):
    xs, ws = (8, 362, 362, 1024), (256, 3, 3, 1024)
    say(f"residue route near the limit of a plane, conv x={xs} w={ws}")
    need = cg.cg_share_conv2d_workspace_bytes(xs, ws, (1, 1), (1, 1))
    assert need > cg.cg_share_conv2d_digit_workspace_bytes(xs, ws, (1, 1), (1, 1))
    dev = [device_ring(s, 9850 + i) for i, s in enumerate((xs, xs, ws, ws))]
    got = cg.cg_share_conv2d_ws(*dev, poisoned(need), stride=(1, 1), pad=(1, 1))
    assert torch.equal(got, cg.cg_share_conv2d(*dev, stride=(1, 1), pad=(1, 1)))
    # the last image's last corner
    host = [cg.to_host(t[-1:, -4:, -4:].contiguous()) for t in dev[:2]] + [cg.to_host(t[-8:].contiguous()) for t in dev[2:]]
    want = ro.party_conv2d(*host, (1, 1), (1, 1))[:, 1:, 1:]
    assert np.array_equal(cg.to_host(got[-1:, -3:, -3:, -8:].contiguous()), want)
    del dev, got
    torch.cuda.empty_cache()


# both tiles with 18 and with 19 moduli on gathered patches: even and odd channel counts, windows, strides and paddings
# that differ along the axes, 1 x 1 windows with a stride or padding, and the 1 x 1 layer that is a product of rows
GATHERS = [((2, 25, 51, 180), (384, 3, 5, 180), (1, 2), (0, 1)), ((4, 58, 33, 53), (104, 5, 5, 53), (2, 1), (1, 1)),
           ((1, 23, 41, 511), (1108, 1, 1, 511), (1, 1), (1, 2)), ((3, 58, 10, 234), (336, 2, 3, 234), (2, 1), (1, 2)),
           ((6, 12, 60, 249), (66, 5, 5, 249), (2, 1), (3, 0)), ((4, 19, 29, 223), (71, 5, 5, 223), (1, 1), (1, 2)),
           ((4, 26, 16, 126), (224, 5, 3, 126), (2, 1), (2, 2)), ((5, 40, 29, 63), (223, 5, 3, 63), (2, 1), (0, 1)),
           ((5, 39, 11, 816), (972, 1, 1, 816), (1, 2), (1, 2)), ((1, 51, 30, 831), (507, 1, 1, 831), (1, 1), (1, 1)),
           ((4, 13, 59, 226), (138, 5, 5, 226), (1, 1), (0, 1)), ((5, 51, 9, 447), (264, 5, 3, 447), (2, 1), (1, 2)),
           ((3, 10, 56, 427), (224, 5, 3, 427), (1, 1), (0, 1)), ((4, 43, 45, 697), (976, 1, 1, 697), (1, 1), (0, 0))]


@pytest.mark.parametrize("xs,ws,st,pd", GATHERS)
def test_gathers(cg, ro, wl, xs, ws, st, pd):
    say(f"residue route conv x={xs} w={ws} stride={st} pad={pd}")
    assert cg.cg_share_conv2d_prefers_workspace(xs, ws, st, pd)
    ops = [wl.draw_ring(s, 9250 + i) for i, s in enumerate((xs, xs, ws, ws))]
    dev = [cg.to_device(a) for a in ops]
    plain = cg.cg_share_conv2d(*dev, stride=st, pad=pd)
    got = cg.cg_share_conv2d_ws(*dev, poisoned(cg.cg_share_conv2d_workspace_bytes(xs, ws, st, pd)), stride=st, pad=pd)
    assert torch.equal(got, plain)
    n = ws[0]
    for image, lo in ((0, 0), (xs[0] - 1, n - 40)):
        want = ro.party_conv2d(ops[0][image:image + 1], ops[1][image:image + 1], ops[2][lo:lo + 40], ops[3][lo:lo + 40], st, pd)
        assert np.array_equal(cg.to_host(got[image:image + 1, :, :, lo:lo + 40].contiguous()), want)


# right operands so large that all XCDs take one modulus at a time: the small tile, the large one, both
IN_STEP = [((3, 9, 19, 478), (2562, 3, 3, 478), (1, 1), (1, 1)), ((2, 23, 12, 508), (2286, 3, 3, 508), (1, 1), (1, 1)),
           ((3, 11, 14, 638), (1898, 3, 3, 638), (1, 1), (1, 1))]
IN_STEP_DGRADS = [((3, 22, 8, 578), (876, 5, 5, 578), (2, 2)), ((3, 11, 16, 2199), (538, 3, 3, 2199), (1, 1)),
                  ((4, 18, 9, 2332), (474, 3, 3, 2332), (1, 1))]


@pytest.mark.parametrize("xs,ws,st,pd", IN_STEP)
def test_gathers_of_one_modulus_at_a_time(cg, ro, wl, xs, ws, st, pd):
    test_gathers(cg, ro, wl, xs, ws, st, pd)


# the input gradient of unit-stride layers: 18 and 19 moduli, channel counts of any kind, padding beyond the window, windows that
# differ along the axes, and the 1 x 1 layer, which is a product of rows
DGRADS = [((32, 16, 16, 256), (256, 3, 3, 256), (1, 1)), ((5, 33, 21, 130), (200, 3, 5, 130), (0, 2)),
          ((4, 25, 25, 257), (300, 3, 3, 257), (4, 1)), ((6, 21, 20, 333), (321, 5, 5, 333), (2, 2)),
          ((8, 16, 16, 1025), (2049, 1, 1, 1025), (0, 0))]


@pytest.mark.parametrize("xs,ws,pd", DGRADS)
def test_input_gradient(cg, ro, wl, xs, ws, pd):
    say(f"residue route input gradient x={xs} w={ws} pad={pd}")
    need = cg.cg_share_conv2d_dgrad_workspace_bytes(xs, ws, (1, 1), pd)
    assert need > 0
    gs = (xs[0], xs[1] + 2 * pd[0] - ws[1] + 1, xs[2] + 2 * pd[1] - ws[2] + 1, ws[0])
    ops = [wl.draw_ring(s, 9260 + i) for i, s in enumerate((gs, gs, ws, ws))]
    dev = [cg.to_device(a) for a in ops]
    buf = poisoned(need + 512)
    got = cg.cg_share_conv2d_dgrad_ws(*dev, xs, buf[:need // 8], pad=pd)
    assert bool((buf[need // 8:] == 0x5A5A5A5A5A5A5A5A).all())
    plain = cg.cg_share_conv2d_dgrad_ws(*dev, xs, None, pad=pd)
    assert torch.equal(got, plain)
    for unusable in (buf[:need // 8 - 2], buf[1:need // 8 + 1]):   # too small, 8-byte aligned: the route without
        assert torch.equal(cg.cg_share_conv2d_dgrad_ws(*dev, xs, unusable, pad=pd), plain)
    assert torch.equal(cg.cg_share_conv2d_dgrad(*dev, xs, pad=pd), plain)   # scratch memory of its own
    last = [a[-1:] for a in ops[:2]]
    want = ro.party_conv2d_dgrad(*last, *ops[2:], (1,) + xs[1:], (1, 1), pd)
    assert np.array_equal(cg.to_host(got[-1:].contiguous()), want)


@pytest.mark.parametrize("xs,ws,pd", IN_STEP_DGRADS)
def test_input_gradient_of_one_modulus_at_a_time(cg, ro, wl, xs, ws, pd):
    test_input_gradient(cg, ro, wl, xs, ws, pd)


def test_input_gradient_without_scratch_of_its_own(cg, wl, monkeypatch):
    """Captured, on a named stream, beyond the limit or where the allocator refuses the call keeps no memory; a graph's replays
    follow the operands."""
    xs, ws, pd = (32, 16, 16, 256), (256, 3, 3, 256), (1, 1)
    say("input gradient captured, on a named stream, beyond the limit and refused")
    dev = [cg.to_device(wl.draw_ring(s, 9270 + i)) for i, s in enumerate((xs, xs, ws, ws))]
    want = cg.cg_share_conv2d_dgrad(*dev, xs, pad=pd)
    dx = torch.empty_like(want)
    torch.cuda.synchronize()
    need = cg.cg_share_conv2d_dgrad_workspace_bytes(xs, ws, (1, 1), pd)

    def taken(**kw):
        before = torch.cuda.memory_allocated()
        torch.cuda.reset_peak_memory_stats()
        cg.cg_share_conv2d_dgrad(*dev, xs, pad=pd, dx_i=dx, **kw)
        return torch.cuda.max_memory_allocated() - before

    assert taken() >= need   # what the others do without
    side = torch.cuda.Stream()
    assert taken(stream=side) == 0
    side.synchronize()
    assert torch.equal(dx, want)
    with monkeypatch.context() as m:
        m.setattr(cg, "SCRATCH_LIMIT", need - 1)
        dx.fill_(77)
        assert taken() == 0 and torch.equal(dx, want)
    with monkeypatch.context() as m:   # taken by someone else after it was seen free
        def refuse(*a, **kw):
            raise torch.OutOfMemoryError("no memory")
        m.setattr(torch, "empty", refuse)
        dx.fill_(77)
        assert taken() == 0
    assert torch.equal(dx, want)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        assert taken() == 0
    for i in range(3):
        for t in dev:
            t.add_(i + 1)
        want = cg.cg_share_conv2d_dgrad(*dev, xs, pad=pd)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(dx, want)


def test_input_gradient_where_memory_is_short(cg, wl, monkeypatch):
    """A program that has no room for the scratch memory keeps its cached blocks: nothing is asked for, and nothing released."""
    xs, ws, pd = (32, 16, 16, 256), (256, 3, 3, 256), (1, 1)
    say("input gradient where memory is short")
    dev = [cg.to_device(wl.draw_ring(s, 9280 + i)) for i, s in enumerate((xs, xs, ws, ws))]
    want = cg.cg_share_conv2d_dgrad(*dev, xs, pad=pd)
    dx = torch.empty_like(want)
    need, total = cg.cg_share_conv2d_dgrad_workspace_bytes(xs, ws, (1, 1), pd), torch.cuda.mem_get_info()[1]

    def run():
        dx.fill_(77)
        torch.cuda.empty_cache()   # the block of a call before
        del [torch.empty(64 << 20, dtype=torch.uint8, device="cuda")][0]   # a block of the program's own
        before, stats = torch.cuda.memory_reserved(), torch.cuda.memory_stats()
        cg.cg_share_conv2d_dgrad(*dev, xs, pad=pd, dx_i=dx)
        torch.cuda.synchronize()
        after, taken = torch.cuda.memory_stats(), torch.cuda.memory_reserved() - before
        assert all(after[k] == stats[k] for k in ("num_alloc_retries", "num_ooms"))
        assert torch.equal(dx, want)
        return taken

    assert run() >= need   # there is room
    torch.cuda.empty_cache()
    try:
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (96 << 20)) / total)
        assert run() == 0
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    monkeypatch.setattr(torch.cuda, "mem_get_info", lambda device=None: (total // 8 + need - 1, total))
    assert run() == 0


def test_input_gradient_while_another_thread_captures(cg, wl):
    """A capture in the default mode forbids allocations to every thread; the call is no part of it and leaves it valid."""
    xs, ws, pd = (32, 16, 16, 256), (256, 3, 3, 256), (1, 1)
    say("input gradient while another thread captures a graph")
    dev = [cg.to_device(wl.draw_ring(s, 9290 + i)) for i, s in enumerate((xs, xs, ws, ws))]
    want = cg.cg_share_conv2d_dgrad(*dev, xs, pad=pd)
    dx, counter = torch.empty_like(want), torch.zeros(64, dtype=torch.int64, device="cuda")
    graph, side, errors = torch.cuda.CUDAGraph(), torch.cuda.Stream(), []
    torch.cuda.synchronize()
    capturing, called = threading.Event(), threading.Event()

    def capture():
        try:
            with torch.cuda.graph(graph):   # (empties the allocator's cache: the call below has to allocate)
                counter.add_(1)
                capturing.set()
                called.wait(30)
                counter.add_(1)
        except Exception as e:
            errors.append(e)
        finally:
            capturing.set()
    thread = threading.Thread(target=capture)
    thread.start()
    try:
        assert capturing.wait(30)
        with torch.cuda.stream(side):
            cg.cg_share_conv2d_dgrad(*dev, xs, pad=pd, dx_i=dx)
    finally:
        called.set()
        thread.join()
    assert not errors, errors
    torch.cuda.synchronize()
    assert torch.equal(dx, want)
    for i in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert bool((counter == 2 * (i + 1)).all())


def test_scratch_of_the_digit_planes_is_still_enough(cg, wl):
    """A caller that brings no more than the digit planes take, or memory the route cannot use, gets the same words."""
    M, N, K = 2000, 2040, 2044
    say("residue route with the digit planes' scratch memory")
    planes, need = cg.cg_share_matmul_digit_workspace_bytes(M, N, K), cg.cg_share_matmul_workspace_bytes(M, N, K)
    assert need > planes
    dev = [cg.to_device(wl.draw_ring((r, K), 9300 + i)) for i, r in enumerate((M, M, N, N))]
    want = cg.cg_share_matmul(*dev)
    for nbytes in (planes, need - 16, need):
        buf = torch.full((nbytes // 8 + 64,), 7, dtype=torch.int64, device="cuda")
        got = cg.cg_share_matmul_ws(*dev, buf[:nbytes // 8])
        assert torch.equal(got, want)
        assert bool((buf[nbytes // 8:] == 7).all())


@pytest.mark.parametrize("K", [3001, 3008])
def test_workspace_that_the_residues_cannot_use(cg, wl, K):
    """Missing, misaligned or overlapping scratch memory: the next route where there is one without it (odd K), the
    documented error where the digit route applies and the fault lies within its bytes."""
    M, N = 2048, 2040
    say(f"residue route, unusable workspace K={K}")
    need, digits = cg.cg_share_matmul_workspace_bytes(M, N, K), cg.cg_share_matmul_digit_workspace_bytes(M, N, K)
    assert need > digits and (digits == 0) == bool(K % 2)
    dev = [cg.to_device(wl.draw_ring((r, K), 9700 + i)) for i, r in enumerate((M, M, N, N))]
    want = cg.cg_share_matmul(*dev)
    whole = torch.empty(need // 8 + M * N + 8, dtype=torch.int64, device="cuda")
    z_at = lambda byte: whole[byte // 8:byte // 8 + M * N].view(M, N)
    beyond = (digits + 255) // 256 * 256 + 256   # inside the residues' bytes, behind the digits'
    cases = [(whole[1:], None, cg.CG_ERR_ALIGN), (None, None, cg.CG_ERR_NULL), (whole, z_at(64), cg.CG_ERR_ALIAS),
             (whole, z_at(beyond), cg.CG_OK), (whole[:digits // 8], None, cg.CG_OK)]
    for ws, z, status in cases:
        if K % 2 or status == cg.CG_OK:
            assert torch.equal(cg.cg_share_matmul_ws(*dev, ws, z_i=z), want)
        else:
            with pytest.raises(cg.CgError) as e:
                cg.cg_share_matmul_ws(*dev, ws, z_i=z)
            assert e.value.status == status


def test_operands_at_odd_words(cg, wl):
    """Bases that are 8-byte aligned only, K even: word loads and stores, and the digit planes do not apply."""
    M, N, K = 1408, 1400, 3004
    say("residue route, operands at odd words")
    at_odd = lambda shape: torch.empty(shape[0] * shape[1] + 1, dtype=torch.int64, device="cuda")[1:].view(shape)
    dev = []
    for i, r in enumerate((M, M, N, N)):
        dev.append(at_odd((r, K)))
        dev[-1].copy_(cg.to_device(wl.draw_ring((r, K), 9500 + i)))
    z = at_odd((M, N))
    want = cg.cg_share_matmul(*dev)
    cg.cg_share_matmul_ws(*dev, poisoned(cg.cg_share_matmul_workspace_bytes(M, N, K + 1)), z_i=z)
    assert torch.equal(z, want)


def test_captured(cg, wl):
    """Three launches and no other node: replays with other operands in the same buffers give their products."""
    M, N, K = 1150, 1145, 3001
    say("residue route in a HIP graph")
    dev = [torch.empty((r, K), dtype=torch.int64, device="cuda") for r in (M, M, N, N)]
    ws = poisoned(cg.cg_share_matmul_workspace_bytes(M, N, K))
    z = torch.empty((M, N), dtype=torch.int64, device="cuda")
    fill = lambda seed: [d.copy_(cg.to_device(wl.draw_ring(tuple(d.shape), seed + i))) for i, d in enumerate(dev)]
    fill(9400)
    cg.cg_share_matmul_ws(*dev, ws, z_i=z)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cg.cg_share_matmul_ws(*dev, ws, z_i=z)
    for seed in (9410, 9420, 9430):
        fill(seed)
        want = cg.cg_share_matmul(*dev)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(z, want)


def small_tile_bytes(M, N, words, x_rows, taps):
    """What the route takes with every modulus on the small tile: operands' planes, and the result's in whole tiles of 128."""
    up = lambda v, a: -(-v // a) * a
    nmod, line = 18 if taps * words <= 5500 else 19, -(-words // 64) * 128
    return up((x_rows + 1) * line * nmod, 256) + up(N * taps * line * nmod, 256) + up(up(M, 128) * up(N, 128) * nmod, 256)


def check_small_tile_scratch(plain, call, need, small):
    """With that much memory, where the call asks for a little more, the residues still run: the result's planes that end there
    are written, and nothing behind them.  With less they do not."""
    assert small < need and small % 16 == 0
    for nbytes, taken in ((need - 16, True), (small, True), (small - 16, False)):
        buf = poisoned(need + 512)
        got = call(buf[:nbytes // 8])
        assert torch.equal(got, plain)
        assert bool((buf[small // 8 - 64:small // 8] == 0x5A5A5A5A5A5A5A5A).all()) == (not taken), nbytes
        assert bool((buf[nbytes // 8:] == 0x5A5A5A5A5A5A5A5A).all())


@pytest.mark.parametrize("M,N,K", [(893, 1949, 2505), (1167, 1361, 3048)])
def test_scratch_of_the_small_tile_is_still_enough(cg, wl, M, N, K):
    say(f"residue route with the small tile's scratch memory M={M} N={N} K={K}")
    dev = [cg.to_device(wl.draw_ring((r, K), 9410 + i)) for i, r in enumerate((M, M, N, N))]
    check_small_tile_scratch(cg.cg_share_matmul(*dev), lambda ws: cg.cg_share_matmul_ws(*dev, ws),
                             cg.cg_share_matmul_workspace_bytes(M, N, K), small_tile_bytes(M, N, K, M, 1))


def test_scratch_of_the_small_tile_is_still_enough_for_a_layer(cg, wl):
    xs, ws = (6, 9, 25, 58), (401, 3, 3, 58)
    say(f"residue route with the small tile's scratch memory x={xs} w={ws}")
    dev = [cg.to_device(wl.draw_ring(s, 9420 + i)) for i, s in enumerate((xs, xs, ws, ws))]
    check_small_tile_scratch(cg.cg_share_conv2d(*dev, pad=(1, 1)), lambda w: cg.cg_share_conv2d_ws(*dev, w, pad=(1, 1)),
                             cg.cg_share_conv2d_workspace_bytes(xs, ws, (1, 1), (1, 1)), small_tile_bytes(6 * 225, 401, 58, 6 * 225, 9))
