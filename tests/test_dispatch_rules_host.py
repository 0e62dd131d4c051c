"""The rules that share a call out over the chip, evaluated on the host: the library's own objects are linked into a small
program that prints what the launchers decide.  No GPU is used."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2104_10949_amd", "csrc")

PROGRAM = r"""
#include <stdio.h>
#include <string.h>
#include "prf.h"
#include "share_gemm.h"
#include "share_gemm_rns.h"
#include "share_gemm_split.h"
static void print_split(const cg::WorkSplit& s) {
    printf("%d %lld %d %d %d %u\n", s.ksplit, (long long)s.stream_per, s.tail.first, s.tail.tiles, s.tail.per, s.grid);
}
int main(int argc, char** argv) {
    if (!strcmp(argv[1], "argument_bytes")) printf("%zu\n", sizeof(cg::GemmParams));
    long long a[9];
    while (scanf("%lld %lld %lld %lld %lld %lld %lld %lld %lld", a, a + 1, a + 2, a + 3, a + 4, a + 5, a + 6, a + 7, a + 8) == 9) {
        if (!strcmp(argv[1], "prf")) {
            const cg::PrfSplit s = cg::prf_split((uint64_t)a[0], (size_t)a[1]);
            printf("%llu %u %u\n", (unsigned long long)s.blocks, s.waves, s.per_wg);
        } else if (!strncmp(argv[1], "residue", 7)) {   // M N words x_rows gathered kh kw stride_h stride_w
            cg::RnsParams p = {};
            p.M = (int)a[0]; p.N = (int)a[1]; p.words = (int)a[2]; p.x_rows = (int)a[3]; p.conv = (int)a[4];
            p.kh = (int)a[5]; p.kw = (int)a[6]; p.sh = (int)a[7]; p.sw = !strcmp(argv[1], "residue_fit") ? p.sh : (int)a[8];
            p.Ho = p.Wo = 1;
            const bool fits = cg::rns_plan(&p);
            if (!strcmp(argv[1], "residue_shares"))   // moduli on the large tile, on the small one, the first of each; XCDs in step
                printf("%d %d %d %d %d %d\n", p.large.count, p.small.count, p.large.first, p.small.first, p.nmod, p.by_rounds);
            else if (!strcmp(argv[1], "residue_fit")) {   // a[8]: bytes at hand; fits or not, moduli on the large tile, bytes taken
                const bool held = fits && cg::rns_fit(&p, (unsigned long long)a[8]);
                printf("%d %d %llu\n", held, held ? p.large.count : -1, held ? (unsigned long long)cg::rns_workspace_bytes(p) : 0ull);
            } else
                printf("%d %d %llu\n", fits ? p.tile : 0, p.nmod, fits ? (unsigned long long)cg::rns_workspace_bytes(p) : 0ull);
        } else if (!strcmp(argv[1], "split_odd_rows")) {   // M N K
            print_split(cg::split_work<cg::A_LINEAR_SCALAR, cg::B_SCALAR>((a[0] + 127) / 128 * ((a[1] + 63) / 64), (int)((a[2] + 31) / 32)));
        } else if (!strcmp(argv[1], "split_gather")) {
            print_split(cg::split_work<cg::A_CONV_GEN, cg::B_SCALAR>((a[0] + 127) / 128 * ((a[1] + 63) / 64), (int)((a[2] + 31) / 32)));
        } else if (!strcmp(argv[1], "split_transposed")) {
            print_split(cg::split_work<cg::A_TRANS, cg::B_TRANS>((a[0] + 127) / 128 * ((a[1] + 63) / 64), (int)((a[2] + 31) / 32)));
        } else {   // small, outer, rows_t: M N K accumulate
            cg::GemmParams p = {};
            p.M = (int)a[0]; p.N = (int)a[1]; p.K = p.lda = (int)a[2]; p.z_add = (int)a[3];
            printf("%d\n", (!strcmp(argv[1], "outer") ? cg::share_gemm_outer_applies(p) :
                            !strcmp(argv[1], "rows_t") ? cg::share_gemm_rows_t_pays(p) : cg::share_gemm_small_applies(p)) ? 1 : 0);
        }
    }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    """rules(what, rows of numbers) -> rows of numbers printed by the program"""
    from paper_2104_10949_amd import build as b
    objects = [os.path.join(CSRC, o) for _, o, _ in b.UNITS]
    if not all(os.path.exists(o) for o in objects):
        b.build()
    d = tmp_path_factory.mktemp("rules")
    src, exe = str(d / "rules.cpp"), str(d / "rules")
    with open(src, "w") as f:
        f.write(PROGRAM)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), src, *objects, "-L", os.path.join(rocm, "lib"), "-lamdhip64",
                    "-Wl,-rpath," + os.path.join(rocm, "lib"), "-o", exe], check=True)

    def ask(what, rows):
        text = "".join(" ".join(str(v) for v in (tuple(r) + (0,) * 9)[:9]) + "\n" for r in rows)
        out = subprocess.run([exe, what], input=text, capture_output=True, text=True, check=True, timeout=60).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]

    return ask


def test_prf_runs_are_even_over_the_compute_units(rules):
    """One workgroup runs per compute unit, so the slowest of 256 takes ceil(blocks / 256) runs of per_wg chunks: within
    5 % of an even share for long calls, and never more than a workgroup's constants have room for."""
    full = 256 * 2044 * 128   # words of one full run per compute unit
    cases = [(f, n) for f in (0, 1, 127, 130, 2 ** 40 + 77)
             for n in (1, 2, 128, 129, 32768, 262144, 300001, 1 << 20, 5000000, 1 << 26, full - 128, full, full + 128, 70000000,
                       int(1.5 * full), 2 * full + 5, 140000000, int(2.5 * full), 1 << 28, 1 << 30, (1 << 33) + 12345)]
    for (first, n), (blocks, waves, per_wg) in zip(cases, rules("prf", cases)):
        chunks = (first + n - 1) // 128 - first // 128 + 1
        assert (blocks - 1) * per_wg < chunks <= blocks * per_wg < 2 ** 62, (first, n)
        assert 1 <= per_wg <= 2044 and blocks < 2 ** 31, (first, n)
        assert waves == 16, (first, n)   # short calls too: they are little more than the fill of the tables
        slowest = -(-blocks // 256) * per_wg
        assert slowest <= max(1.05 * chunks / 256, chunks / 256 + 1), (first, n, blocks, per_wg)


# (M, N, K), taken by the plain call, taken by the accumulating call: both sides of every line for more than 64 rows
SMALL = [((128, 128, 784), 1, 1), ((65, 1, 2), 1, 1), ((80, 16, 28800), 1, 1), ((4096, 16, 576), 1, 1),
         ((4112, 16, 32), 1, 1), ((4112, 16, 352), 1, 1), ((4112, 16, 354), 1, 0), ((4112, 16, 416), 1, 0), ((4112, 16, 418), 0, 0),
         ((8192, 16, 32), 1, 1), ((8208, 16, 32), 0, 0), ((8208, 16, 34), 1, 1), ((12288, 16, 32), 0, 0), ((12288, 16, 64), 1, 1),
         ((12288, 16, 96), 1, 1), ((12288, 16, 98), 1, 0), ((12288, 16, 192), 1, 0), ((12288, 16, 194), 0, 0),
         ((12289, 16, 64), 0, 0), ((512, 512, 64), 0, 0), ((96, 768, 416), 1, 0), ((64, 768, 512), 1, 1), ((64, 16384, 32), 1, 1),
         ((64, 1152, 512), 1, 1), ((64, 1168, 512), 0, 0), ((16, 65536, 4096), 1, 1)]


def test_small_products_of_more_than_64_rows_by_rounds_of_the_chip(rules):
    got = rules("small", [s + (0,) for s, _, _ in SMALL])
    acc = rules("small", [s + (1,) for s, _, _ in SMALL])
    assert [(s, g[0], a[0]) for (s, _, _), g, a in zip(SMALL, got, acc)] == SMALL


def _residue_row(xs, ws, st, pd):
    B, H, W, C = xs
    N, kh, kw, _ = ws
    rows = kh == kw == 1 and st == (1, 1) and pd == (0, 0)
    M = B * ((H + 2 * pd[0] - kh) // st[0] + 1) * ((W + 2 * pd[1] - kw) // st[1] + 1)
    return (M, N, C, B * H * W, int(not rows), kh, kw) + tuple(st)


def test_the_residue_tests_reach_every_instantiation(rules):
    """Tile and number of moduli follow from a model: a change of it must not leave a kernel without a test."""
    from paper_2104_10949_amd import binding as b
    from tests import test_gpu_residue as t
    layers = [(xs, ws, (s, s), (p, p)) for xs, ws, s, p in t.CONVS] + t.GATHERS
    rows = [(M, N, K, M, 0, 1, 1, 1, 1) for M, N, K in t.SHAPES] + [_residue_row(*l) for l in layers]
    needs = [b.cg_share_matmul_workspace_bytes(*s) for s in t.SHAPES] + [b.cg_share_conv2d_workspace_bytes(*l) for l in layers]
    seen = set()
    for row, need, (tile, nmod, nbytes) in zip(rows, needs, rules("residues", rows)):
        assert need == nbytes, row   # the route is taken: its bytes are more than the digit planes'
        seen.add((tile, nmod, row[4]))
    assert seen == {(tile, nmod, gathered) for tile in (128, 256) for nmod in (18, 19) for gathered in (0, 1)}


def test_every_modulus_runs_on_one_tile_and_the_residue_tests_reach_all_shares(rules):
    """All moduli on the large tile, all on the small one, and both sizes in one call, of rows and of patches; 2048^3, whose best share
    is modelled 3 % faster than the large tile alone, stays on that."""
    assert rules("residue_shares", [(2048, 2048, 2048, 2048, 0, 1, 1, 1, 1)])[0][:2] == (18, 0)
    from tests import test_gpu_residue as t
    layers = [(xs, ws, (s, s), (p, p)) for xs, ws, s, p in t.CONVS] + t.GATHERS
    rows = [(M, N, K, M, 0, 1, 1, 1, 1) for M, N, K in t.SHAPES + t.SMALL_TILE_SHAPES] + [_residue_row(*l) for l in layers]
    seen = set()
    for row, (large, small, first_large, first_small, nmod, _) in zip(rows, rules("residue_shares", rows)):
        assert large >= 0 and small >= 0 and large + small == nmod and (first_large, first_small) == (0, large), row
        seen.add((large > 0, small > 0, row[4]))
    assert seen == {(large, small, gathered) for large, small in ((True, False), (False, True), (True, True)) for gathered in (0, 1)}


def test_large_right_operands_are_taken_one_modulus_at_a_time(rules):
    """... and the residue tests reach that with every share of the tiles, of patches and with a flipped filter."""
    from paper_2104_10949_amd import binding as b
    from tests import test_gpu_residue as t
    forward = [_residue_row(*l) for l in t.IN_STEP]
    # an input gradient is a forward layer of the gradient, its filter the right operand
    backward = [_residue_row(xs[:3] + (ws[0],), (xs[3],) + ws[1:3] + (ws[0],), (1, 1), pd) for xs, ws, pd in t.IN_STEP_DGRADS]
    needs = [b.cg_share_conv2d_workspace_bytes(*l) for l in t.IN_STEP] + \
            [b.cg_share_conv2d_dgrad_workspace_bytes(xs, ws, (1, 1), pd) for xs, ws, pd in t.IN_STEP_DGRADS]
    shares = rules("residue_shares", forward + backward)
    assert needs == [r[2] for r in rules("residues", forward + backward)]   # the route is taken
    assert all(s[5] for s in shares)
    every = {(True, False), (False, True), (True, True)}
    assert {(s[0] > 0, s[1] > 0) for s in shares[:3]} == {(s[0] > 0, s[1] > 0) for s in shares[3:]} == every


def test_memory_for_the_small_tile_alone_is_enough_where_it_is_the_better_one(rules):
    """A mix of both tiles pads the result's planes to multiples of 256; a call with a little less runs on the small tile alone."""
    from tests import test_gpu_residue as t
    rows = [(M, N, K, M, 0, 1, 1, 1, 1) for M, N, K in t.SHAPES + t.SMALL_TILE_SHAPES + [(893, 1949, 2505), (1403, 1870, 1271)]]
    mixed = 0
    for row, (tile, _, need), (large, *_) in zip(rows, rules("residues", rows), rules("residue_shares", rows)):
        small = t.small_tile_bytes(*row[:4], 1)
        ask = lambda nbytes: rules("residue_fit", [row[:8] + (nbytes,)])[0]
        assert ask(need) == ask(need + 1) == (1, large, need), row
        if tile == 128 and small < need:
            mixed += 1
            assert ask(need - 1) == ask(small) == (1, 0, small), row
        else:
            assert tile == 256 or small == need, row
        assert ask(min(need, small) - 1) == (0, -1, 0) and (tile == 128 or ask(need - 1) == (0, -1, 0)), row
    assert mixed >= 3


def test_gradients_of_small_batches_run_on_their_own_kernels(rules):
    from tests import test_gpu_fc_gradients as t
    assert all(r == (1,) for r in rules("outer", t.OUTER))
    assert all(r == (1,) for r in rules("rows_t", t.ROWS + t.LONG_ROWS))
    assert all(r == (0,) for r in rules("outer", [s[:3] for s in t.OTHERS if s[3]]))
    assert all(r == (0,) for r in rules("rows_t", [s[:3] for s in t.OTHERS if not s[3]]))
    # one block of rows where the tiled kernel measured as fast or faster
    assert all(r == (0,) for r in rules("rows_t", [(4, 1132, 624), (4, 1874, 694), (4, 1766, 576), (1, 1626, 894)]))
    # one and two row blocks; a single turn of a wave, several and waves with one turn less; groups of rows, the last one ragged
    seen = {(M > 16, min(2, (-(-K // 32) + 3) // 4), -(-K // 32) % 4 != 0) for M, N, K in t.ROWS + t.LONG_ROWS}
    assert seen >= {(two, turns, uneven) for two in (False, True) for turns in (1, 2) for uneven in (False, True)} - {(True, 1, False), (False, 1, False)}
    assert any(M > 64 and M % 32 and -(-K // 32) > 4 for M, N, K in t.ROWS)


def test_odd_rows_reach_every_distribution(rules):
    """Unsplit, split over blocks, whole tiles walked, and runs of slices that begin and end inside a tile."""
    from tests import test_gpu_small_products as t
    kinds = {}
    for (M, N, K), (ksplit, per, *_) in zip(t.ODD + t.ODD_STREAMED, rules("split_odd_rows", t.ODD + t.ODD_STREAMED)):
        nk = -(-K // 32)
        kinds.setdefault("classic" if per == 0 and ksplit == 1 else "split" if per == 0 else "tiles" if ksplit == 1 else "runs", []).append((M, N, K))
        if per and ksplit == 1:
            assert per % nk == 0
    assert set(kinds) == {"classic", "split", "tiles", "runs"} and kinds["runs"] == t.ODD_STREAMED
    for M, N, K in t.ODD_STREAMED:
        per = rules("split_odd_rows", [(M, N, K)])[0][1]
        assert per % -(-K // 32) and -(-K // 32) % per


def test_arguments_of_the_tiled_kernels_take_six_lines(rules):
    """A block's first load waits for them; a seventh line of 64 bytes cost 0.2 us a call."""
    assert rules("argument_bytes", [])[0][0] <= 6 * 64


def test_split_tails_reach_every_form(rules):
    """tail tiles 1 .. 128, parts of one slice and of several, a last part shorter than the others, fewer parts than there is room for"""
    from tests import test_gpu_small_products as t
    layers = []
    for xs, ws, st, pd in t.TAIL_LAYERS:
        M, N, C, _, _, kh, kw, _, _ = _residue_row(xs, ws, st, pd)
        layers.append((M, N, C * kh * kw))
    for what, shapes in (("split_gather", layers), ("split_transposed", t.TAIL_GRADIENTS)):
        seen = set()
        for (M, N, K), (ksplit, stream_per, first, tail, per, grid) in zip(shapes, rules(what, shapes)):
            tiles, nk = -(-M // 128) * -(-N // 64), -(-K // 32)
            parts = -(-nk // per)
            assert ksplit == 1 and stream_per == 0 and first == tiles - tail and first % 256 == 0, (M, N, K)
            assert (parts - 1) * per < nk <= parts * per and grid == first + tail * parts <= first + 256, (M, N, K)
            seen |= {"one slice" if per == 1 else "several slices", "uneven" if nk % per else "even"}
            seen |= {"half a round"} if tail == 128 else set()
            seen |= {"room left"} if parts < min(nk, 256 // tail) else set()
        assert seen == {"one slice", "several slices", "uneven", "even", "half a round", "room left"}, what


# Taken or not, moduli on the large tile, and whole calls in microseconds without residues and with them: as they run, all moduli on the
# large tile, all on the small one.
LAYERS = [(((15, 69, 69, 896), (144, 5, 5, 896), (2, 2), (2, 2)), 0, None, 4301, 3652, 3641, 4527),
          (((4, 101, 101, 1024), (352, 3, 3, 1024), (1, 2), (1, 1)), 1, 17, 3996, 3181, 3196, 3489),
          (((13, 5, 5, 1136), (1008, 7, 7, 1136), (1, 1), (3, 3)), 0, None, 1334, 1683, 1822, 1677),
          (((20, 13, 13, 1296), (224, 5, 5, 1296), (2, 2), (2, 2)), 0, None, 597, 662, 759, 660),
          (((35, 4, 4, 1104), (496, 7, 7, 1104), (1, 1), (3, 3)), 0, None, 1041, 1125, 1278, 1127),
          (((32, 16, 16, 256), (256, 3, 3, 256), (1, 1), (1, 1)), 1, 16, 247, 177, 195, 191),
          (((32, 8, 8, 512), (512, 3, 3, 512), (1, 1), (1, 1)), 1, 16, 252, 181, 224, 197),
          (((32, 32, 32, 128), (128, 3, 3, 128), (1, 1), (1, 1)), 1, 0, 260, 231, 355, 233),
          (((32, 64, 64, 64), (64, 3, 3, 64), (1, 1), (1, 1)), 0, None, 280, 493, 815, 500),
          (((32, 64, 64, 64), (128, 3, 3, 64), (1, 1), (1, 1)), 0, None, 527, 547, 879, 552)]
PRODUCTS = [((7548, 529, 23105), 1, 19, 6225, 6191, 6193, 8962), ((423, 2509, 10029), 0, None, 751, 776, 775, 835),
            ((734, 1713, 3433), 1, 12, 276, 264, 266, 304), ((1000, 777, 1531), 0, None, 96, 84, 105, 84),
            ((4096, 4096, 4096), 1, 18, 3444, 2142, 2143, 2609), ((2048, 2048, 2048), 1, 18, 451, 361, 361, 416),
            ((2048, 2048, 512), 0, None, 121, 132, 129, 124), ((1024, 1024, 1024), 0, None, 72, 72, 81, 73),
            ((512, 4096, 4096), 0, None, 477, 441, 471, 523)]


def test_residues_and_their_tiles_are_chosen_where_they_measured_faster(rules):
    """(Three of those that are not taken would be faster with residues: the rule is fitted to a slower product.)"""
    from paper_2104_10949_amd import binding as b
    rows = [_residue_row(*l) for l, *_ in LAYERS] + [(M, N, K, M, 0, 1, 1, 1, 1) for (M, N, K), *_ in PRODUCTS]
    needs = [b.cg_share_conv2d_workspace_bytes(*l) for l, *_ in LAYERS] + [b.cg_share_matmul_workspace_bytes(*p) for p, *_ in PRODUCTS]
    for (what, taken, share, without, runs, large, small), need, (_, _, nbytes), got in \
            zip(LAYERS + PRODUCTS, needs, rules("residues", rows), rules("residue_shares", rows)):
        assert (need == nbytes) == bool(taken), what
        if taken:
            assert got[0] == share and runs <= 1.02 * min(without, large, small), what


def test_residue_kernels_keep_their_accumulators_in_registers(tmp_path):
    """The product kernels wait for their loads by count: a spilled register's reload waits for all of them, every step."""
    llvm = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
    fat, elf = str(tmp_path / "fat"), str(tmp_path / "elf")
    subprocess.run([os.path.join(llvm, "llvm-objcopy"), "--dump-section", ".hip_fatbin=" + fat,
                    os.path.join(CSRC, "share_gemm_rns.o"), "/dev/null"], check=True)
    subprocess.run([os.path.join(llvm, "clang-offload-bundler"), "--unbundle", "--type=o", "--input=" + fat, "--output=" + elf,
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
    notes = subprocess.run([os.path.join(llvm, "llvm-readelf"), "--notes", elf], capture_output=True, text=True, check=True).stdout
    names = re.findall(r"\.name:\s+(\S*rns_gemm\S*)", notes)
    assert len(names) == 4
    assert set(re.findall(r"\.vgpr_spill_count:\s+(\d+)", notes)) == {"0"}
    assert set(re.findall(r"\.private_segment_fixed_size:\s+(\d+)", notes)) == {"0"}
