"""GPU parity of the share-truncation step (local arithmetic of every party, through the C-ABI)
against the CPU oracle, bit for bit, and the protocol's error bound on the opened result."""
import numpy as np
import pytest

from tests.gpu_util import first_mismatch, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

K0, K1, K2 = bytes(range(16)), bytes(range(16, 32)), bytes(range(32, 48))


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


@pytest.mark.parametrize("n,first", [(1, 0), (1, 1), (2, 1), (3, 4), (255, 7), (256, 0), (1001, 3), ((1 << 20) + 5, 2 ** 40 + 1)])
def test_prf_words_match_the_oracle(cg, ro, n, first):
    say(f"cg_prf_words n={n} first={first}")
    got = cg.to_host(cg.cg_prf_words(K1, 77, first, n))
    assert not first_mismatch(got, ro.prf_words(K1, 77, first, n))


# a wave takes 64 blocks = 128 words, 256 blocks = 512 words share the constants of the first two rounds, a workgroup
# takes one chunk up to 32768 words, a chunk for each of its 16 waves up to 524288, then runs of chunks: around each of these, and
# where the block index carries into byte 1, byte 2 and its upper word
@pytest.mark.parametrize("n,first", [(127, 1), (128, 0), (129, 383), (514, 511), (1500, 2 ** 17 - 700), (3000, 2 ** 33 - 1001),
                                     (262144, 6), (262145, 127), (300001, 2 ** 25 - 150001), (524288, 510), (560003, 12)])
def test_prf_streams_at_the_edges_of_their_work_split(cg, ro, wl, n, first):
    say(f"prf streams at work-split edges n={n} first={first}")
    z, m = wl.draw_ring((n + 1,), 911), wl.draw_ring((n + 1,), 912)
    dz, dm = cg.to_device(z), cg.to_device(m)
    assert not first_mismatch(cg.to_host(cg.cg_prf_words(K1, 77, first, n)), ro.prf_words(K1, 77, first, n))
    for s in (0, 1):   # 16-byte aligned and not
        zs, ms = z[s:s + n], m[s:s + n]
        got = cg.to_host(cg.cg_trunc1_local(dz[s:s + n], dm[s:s + n], K1, K0, 31, first, 16, K1, 32))
        assert not first_mismatch(got, ro.trunc1_local(zs, ms, K1, K0, 31, first, 16, K1, 32))
        got = cg.to_host(cg.cg_breshare(dz[s:s + n], K1, K0, 31, first))
        assert not first_mismatch(got, ro.breshare(zs, K1, K0, 31, first))


def test_prf_stream_longer_than_one_run_per_compute_unit(cg, ro):
    # a workgroup holds the constants of 512 groups: more than 256 * 2044 chunks need more workgroups than compute units
    per_wg = 2044 * 128
    n = 256 * per_wg + 3 * 128 + 5
    say(f"cg_prf_words n={n}")
    got = cg.cg_prf_words(K1, 77, 130, n)
    for at in (0, per_wg - 300, 255 * per_wg - 300, 256 * per_wg - 300, n - 600):
        assert not first_mismatch(cg.to_host(got[at:at + 600]), ro.prf_words(K1, 77, 130 + at, 600))


@pytest.mark.parametrize("d", [0, 1, 16, 20, 63])
@pytest.mark.parametrize("n,first", [(1, 0), (2, 1), (257, 5), (100003, 8)])
def test_local_step_matches_the_oracle(cg, ro, wl, n, first, d):
    say(f"cg_trunc1_local n={n} first={first} d={d}")
    z, m = wl.draw_ring((n,), 900 + n), wl.draw_ring((n,), 901 + n)
    dz, dm = cg.to_device(z), cg.to_device(m)
    # P_1's step: message and mask
    got = cg.to_host(cg.cg_trunc1_local(dz, dm, K1, K0, 31, first, d, K1, 32))
    assert not first_mismatch(got, ro.trunc1_local(z, m, K1, K0, 31, first, d, K1, 32))
    # P_0's step: neither
    got = cg.to_host(cg.cg_trunc1_local(dz, None, K0, K2, 31, first, d))
    assert not first_mismatch(got, ro.trunc1_local(z, None, K0, K2, 31, first, d))
    # in place over z
    out = cg.cg_trunc1_local(dz, dm, K1, K0, 31, first, d, K1, 32, out=dz)
    assert out.data_ptr() == dz.data_ptr()
    assert not first_mismatch(cg.to_host(dz), ro.trunc1_local(z, m, K1, K0, 31, first, d, K1, 32))


def test_local_step_on_edge_words(cg, ro):
    edge = np.array([0, 1, 0xFFFF, 0x10000, (1 << 63) - 1, 1 << 63, (1 << 63) + 1, (1 << 64) - 1, (1 << 64) - 0x10001,
                     0x8080808080808080, 0x7F7F7F7F7F7F7F7F], dtype=np.uint64)
    same = bytes(16)
    for d in (0, 1, 16, 63):
        say(f"cg_trunc1_local edge words d={d}")
        got = cg.to_host(cg.cg_trunc1_local(cg.to_device(edge), None, same, same, 0, 0, d))
        assert not first_mismatch(got, ro.trunc1_local(edge, None, same, same, 0, 0, d))


def test_product_then_truncation_opens_to_the_fixed_point_product(cg, ro, wl):
    # three parties: local product, blinded message, local truncation steps; opened result vs the real product
    M, N, K, t = 48, 40, 96, wl.FRAC_BITS
    say(f"matmul + truncation, three parties, {M}x{N}x{K}")
    rng = np.random.default_rng(1234)
    xr, yr = rng.uniform(-1, 1, (M, K)), rng.normal(0, 0.05, (N, K))
    x, y = ro.encode(xr, t), ro.encode(yr, t)
    sx = ro.share(x, wl.draw_ring(x.shape, 1), wl.draw_ring(x.shape, 2))
    sy = ro.share(y, wl.draw_ring(y.shape, 3), wl.draw_ring(y.shape, 4))
    keys = (K0, K1, K2)
    z = []
    for i in range(3):
        ops = [cg.to_device(a) for a in (*ro.party_pair(sx, i), *ro.party_pair(sy, i))]
        z.append(cg.cg_share_matmul(*ops))
    n = M * N
    msg = cg.cg_reshare(z[2], K2, K1, 5, 0)                                   # round 1: P_2 -> P_1
    s0 = cg.cg_trunc1_local(z[0], None, K0, K2, 5, 0, t)                      # P_0
    s1 = cg.cg_trunc1_local(z[1], msg, K1, K0, 5, 0, t, K1, 6)                # P_1
    s2 = cg.cg_prf_words(K1, 6, 0, n).view(M, N)                              # P_1 and P_2
    torch.cuda.synchronize()
    # bit-exact against the oracle's run of the same protocol on the oracle's products
    zo = [ro.party_matmul(*ro.party_pair(sx, i), *ro.party_pair(sy, i)) for i in range(3)]
    so = ro.trunc1_protocol(zo, keys, nonce=5, first=0, d=t, mask_nonce=6)
    for got, want in zip((s0, s1, s2), so):
        assert not first_mismatch(cg.to_host(got), want)
    # and the opened value is the product at scale 2^t, at most one unit below the floor
    opened = cg.to_host(cg.cg_reconstruct(s0, s1, s2)).astype(np.int64)
    exact = (ro.matmul(x, y).astype(np.int64)) >> t
    assert set(np.unique(opened - exact).tolist()) <= {-1, 0}
    real = (np.rint(xr * 2 ** t) / 2 ** t) @ (np.rint(yr * 2 ** t) / 2 ** t).T
    assert np.max(np.abs(opened / 2 ** t - real)) <= 2.0 ** -t * 2


def test_truncation_argument_errors(cg):
    z = torch.zeros(16, dtype=torch.int64, device="cuda")
    for d in (-1, 64):
        with pytest.raises(cg.CgError) as e:
            cg.cg_trunc1_local(z, None, K0, K2, 0, 0, d)
        assert e.value.status == cg.CG_ERR_SHAPE
    with pytest.raises(cg.CgError) as e:
        cg.cg_trunc1_local(z[:8], None, K0, K2, 0, 0, 16, out=z[4:12])
    assert e.value.status == cg.CG_ERR_ALIAS


def test_fc_stack_chained_through_the_truncation_protocol(cg, ro, wl):
    """The FC stack of configuration 2 (784-128-128-10, batch 128) evaluated layer by layer on shares:
    three parties' local products, bias add and the two-round truncation on the GPU, so that every layer's
    output is back at scale 2^t in replicated form.  ReLU is not part of this library: between layers the
    test opens the activations, clips them on the host and shares them again.  The decoded logits must match
    a float64 network on the same grid-rounded parameters."""
    t = wl.FRAC_BITS
    layers = wl.config_layers(2)
    rng = np.random.default_rng(2024)
    keys = (K0, K1, K2)
    x_real = np.rint(rng.uniform(0, 1, size=(layers[0].M, layers[0].K)) * 2 ** t) / 2 ** t
    act_real = x_real
    act = ro.encode(x_real, t)
    nonce = 100
    for li, L in enumerate(layers):
        say(f"chained FC stack: layer {li} {L.gemm}")
        w_real = np.rint(rng.normal(0, 0.05, size=(L.N, L.K)) * 2 ** t) / 2 ** t
        b_real = np.rint(rng.normal(0, 0.1, size=(L.N,)) * 2 ** t) / 2 ** t
        w, b = ro.encode(w_real, t), ro.encode(b_real, 2 * t)          # the bias joins the product at scale 2^2t
        sx = ro.share(act, wl.draw_ring(act.shape, 10 * li + 1), wl.draw_ring(act.shape, 10 * li + 2))
        sw = ro.share(w, wl.draw_ring(w.shape, 10 * li + 3), wl.draw_ring(w.shape, 10 * li + 4))
        sb = ro.share(b, wl.draw_ring(b.shape, 10 * li + 5), wl.draw_ring(b.shape, 10 * li + 6))
        dx, dw, db = ([cg.to_device(s) for s in sh] for sh in (sx, sw, sb))
        z = []
        for i in range(3):
            zi = cg.cg_share_matmul(dx[i], dx[(i + 1) % 3], dw[i], dw[(i + 1) % 3])
            # additive share of the bias: party i adds component i (passed for both slots, second result unused)
            zi, _ = cg.cg_share_bias_add(zi, zi, db[i], db[i])
            z.append(zi)
        n = z[0].numel()
        msg = cg.cg_reshare(z[2], keys[2], keys[1], nonce, 0)
        s0 = cg.cg_trunc1_local(z[0], None, keys[0], keys[2], nonce, 0, t)
        s1 = cg.cg_trunc1_local(z[1], msg, keys[1], keys[0], nonce, 0, t, keys[1], nonce + 1)
        s2 = cg.cg_prf_words(keys[1], nonce + 1, 0, n).view_as(s0)
        nonce += 2
        opened = cg.to_host(cg.cg_reconstruct(s0, s1, s2)).astype(np.int64)
        pre_real = act_real @ w_real.T + b_real
        assert np.max(np.abs(opened / 2 ** t - pre_real)) < 5e-3, f"layer {li}"
        if li + 1 < len(layers):
            opened = np.maximum(opened, 0)                               # host-side ReLU between layers
            act = opened.astype(np.uint64)
            act_real = np.maximum(pre_real, 0)
    assert opened.shape == (layers[-1].M, layers[-1].N)


def test_fc_stack_evaluated_entirely_on_shares(cg, ro, wl):
    """Configuration 2's FC stack with nothing opened between layers: product, bias, truncation protocol and
    ReLU (sign-bit circuit + three share products) all on shares, every party's local step on the GPU.  Only the
    logits are opened; they must match a float64 network on the same grid-rounded parameters."""
    from tests.gpu_util import gpu_relu
    t = wl.FRAC_BITS
    layers = wl.config_layers(2)
    rng = np.random.default_rng(2025)
    keys = (K0, K1, K2)
    x_real = np.rint(rng.uniform(0, 1, size=(layers[0].M, layers[0].K)) * 2 ** t) / 2 ** t
    enc = ro.encode(x_real, t)
    act = tuple(cg.to_device(s) for s in ro.share(enc, wl.draw_ring(enc.shape, 1), wl.draw_ring(enc.shape, 2)))
    act_real = x_real
    nonce = 1000
    for li, L in enumerate(layers):
        say(f"FC stack on shares: layer {li} {L.gemm}")
        w_real = np.rint(rng.normal(0, 0.05, size=(L.N, L.K)) * 2 ** t) / 2 ** t
        b_real = np.rint(rng.normal(0, 0.1, size=(L.N,)) * 2 ** t) / 2 ** t
        w, b = ro.encode(w_real, t), ro.encode(b_real, 2 * t)
        dw = [cg.to_device(s) for s in ro.share(w, wl.draw_ring(w.shape, 10 * li + 3), wl.draw_ring(w.shape, 10 * li + 4))]
        db = [cg.to_device(s) for s in ro.share(b, wl.draw_ring(b.shape, 10 * li + 5), wl.draw_ring(b.shape, 10 * li + 6))]
        z = []
        for i in range(3):
            zi = cg.cg_share_matmul(act[i], act[(i + 1) % 3], dw[i], dw[(i + 1) % 3])
            zi, _ = cg.cg_share_bias_add(zi, zi, db[i], db[i])
            z.append(zi)
        n = z[0].numel()
        msg = cg.cg_reshare(z[2], keys[2], keys[1], nonce, 0)
        s0 = cg.cg_trunc1_local(z[0], None, keys[0], keys[2], nonce, 0, t)
        s1 = cg.cg_trunc1_local(z[1], msg, keys[1], keys[0], nonce, 0, t, keys[1], nonce + 1)
        s2 = cg.cg_prf_words(keys[1], nonce + 1, 0, n).view_as(s0)
        pre = (s0, s1, s2)
        pre_real = act_real @ w_real.T + b_real
        if li + 1 < len(layers):
            # first hidden layer: sign bit from the word-parallel adder; second: from the pruned circuit on planes
            act = gpu_relu(cg, pre, keys, nonce + 2, sliced=(li == 1))
            act_real = np.maximum(pre_real, 0)
        nonce += 4
    torch.cuda.synchronize()
    logits = cg.to_host(cg.cg_reconstruct(*pre)).astype(np.int64) / 2 ** t
    assert logits.shape == (layers[-1].M, layers[-1].N)
    assert np.max(np.abs(logits - pre_real)) < 5e-3
    # same predicted class wherever the reference's top two logits are further apart than the fixed-point error
    top2 = np.sort(pre_real, axis=1)[:, -2:]
    clear = top2[:, 1] - top2[:, 0] > 1e-3
    assert clear.sum() > 100
    assert np.array_equal(np.argmax(logits, axis=1)[clear], np.argmax(pre_real, axis=1)[clear])


ACC_MATMUL = [
    (100, 70, 90),          # one pass, plain read-add-write
    (128, 64, 16384),       # K split over blocks: atomic adds into the value already there
    (130, 70, 16400),       # ... with ragged tiles; more than one accumulator segment per block
    (700, 700, 1100),       # tile counts that take the streamed distribution
    (32, 512, 8192),        # the 32-row tile of the long fully connected layers
]


@pytest.mark.parametrize("M,N,K", ACC_MATMUL)
def test_product_added_to_the_zero_share_is_the_reshared_product(cg, ro, wl, M, N, K):
    """cg_share_matmul_acc on an output that holds alpha_i gives z_i + alpha_i: the oracle's reshare of its product."""
    say(f"matmul_acc M={M} N={N} K={K}")
    x_a, x_b = wl.draw_ring((M, K), 1), wl.draw_ring((M, K), 2)
    y_a, y_b = wl.draw_ring((N, K), 3), wl.draw_ring((N, K), 4)
    z = cg.cg_zero_share(K0, K2, 77, 5, M * N).view(M, N)
    cg.cg_share_matmul_acc(*(cg.to_device(a) for a in (x_a, x_b, y_a, y_b)), z)
    want = ro.reshare(ro.party_matmul(x_a, x_b, y_a, y_b), K0, K2, 77, 5)
    assert not first_mismatch(cg.to_host(z), want)


@pytest.mark.parametrize("case", [
    (2, 12, 12, 64, 128, 3, 3, (1, 1), (1, 1)),        # 32-channel gather
    (2, 9, 7, 3, 20, 5, 5, (2, 1), (2, 2)),            # per-word gather
    (8, 14, 14, 256, 256, 3, 3, (1, 1), (1, 1)),       # streamed distribution
    (2, 14, 14, 64, 96, 1, 1, (1, 1), (0, 0)),         # pointwise: the plain product
])
def test_convolution_added_to_the_zero_share(cg, ro, wl, case):
    B, H, W, Cin, Cout, kh, kw, stride, pad = case
    say(f"conv2d_acc {case}")
    xs, ws = (B, H, W, Cin), (Cout, kh, kw, Cin)
    x_a, x_b, w_a, w_b = wl.draw_ring(xs, 1), wl.draw_ring(xs, 2), wl.draw_ring(ws, 3), wl.draw_ring(ws, 4)
    want = ro.party_conv2d(x_a, x_b, w_a, w_b, stride, pad)
    z = cg.cg_zero_share(K1, K0, 78, 0, want.size).view(want.shape)
    cg.cg_share_conv2d_acc(*(cg.to_device(a) for a in (x_a, x_b, w_a, w_b)), z, stride=stride, pad=pad)
    assert not first_mismatch(cg.to_host(z), ro.reshare(want, K1, K0, 78, 0))


def test_two_products_summed_into_one_output(cg, ro, wl):
    M, N, K = 96, 80, 200
    ops = [[wl.draw_ring((M, K) if j < 2 else (N, K), 10 * t + j) for j in range(4)] for t in range(2)]
    z = cg.cg_share_matmul(*(cg.to_device(a) for a in ops[0]))
    cg.cg_share_matmul_acc(*(cg.to_device(a) for a in ops[1]), z)
    want = ro.party_matmul(*ops[0]) + ro.party_matmul(*ops[1])
    assert not first_mismatch(cg.to_host(z), want)
