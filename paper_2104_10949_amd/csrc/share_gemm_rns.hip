// One party's local product on replicated shares through residues: half the matrix work of the digit form.
//
// z = x_a*(w_a + w_b) + x_b*w_a mod 2^64 needs 36 products of signed bytes per word product when the words are cut
// into digits.  Here the same sum is computed as an INTEGER.  Read as signed numbers the words are below 2^63.01, so
// with the 2*K products of one output the integer is below 2^127.02 * K, and its residues modulo 18 pairwise coprime
// numbers of at most eight bits (product 2^140.45) determine it for K up to 5551 words; a nineteenth (2^147.9)
// reaches beyond what the 32-bit accumulators hold.  One product of bytes per modulus: 18 instead of 36.
//   1. rns_planes_kernel   every operand word -> 18 signed residues, each to the plane of its modulus
//   2. rns_gemm_kernel     one int8 matrix product per modulus; accumulators reduced to a byte at the end of a tile
//   3. rns_combine_kernel  the residues r_m of an output -> sum_m r_m * (P / p_m) - k * P  (mod 2^64)
// The inverses (P / p_m)^-1 mod p_m of the Chinese remainder theorem are multiplied into the right operand's residues,
// and k = round(sum_m r_m / p_m): the integer lies within 0.499 P of zero (that is what RNS_K_18 says), the rounded
// sum is exact to 3e-4, so k is the right one.
//
// Exact matrix products through int8 products modulo such numbers and the Chinese remainder theorem are a published
// method (Ozaki, Uchino and Imamura, "Ozaki Scheme II", 2025, there for floating-point products).
//
// Measured on MI355X in one run, whole calls, the better of the plain kernel and the digit planes against residues: 4096^3 3444 -> 2142 us
// (2115 - 2237 over several cards), 2048^3 451 -> 361, 3072 x 3072 x 1024 525 -> 411; 3x3 layers at batch 32: 16 x 16 x 256 -> 256
// 247 -> 177 (175 - 187), 8 x 8 x 512 -> 512 252 -> 181, the 5x5 one 644 -> 420.  At 4096^3: conversion 330 us (52 bytes per word pair at 5.2 TB/s: memory), product
// 1700-1780 us (the matrix pipes are busy 83 % of the cycles, at the clock that random operands leave), combination 90 us.
// Where operands or outputs are large against M*N*K, or the grid leaves most of a round empty, the three passes cost
// more than they save; the caller's rule compares both.
#include "share_gemm_rns.h"

#include <type_traits>
#include <utility>

#include "share_digits.h"

namespace cg {
namespace {

constexpr int MAX_MOD = 19;
constexpr int MODULI[MAX_MOD] = {256, 255, 253, 251, 247, 241, 239, 233, 229, 227,
                                 223, 217, 211, 199, 197, 193, 191, 181, 179};

constexpr int centred(int v, int p) {   // representative in [-p/2, p/2)
    v %= p;
    if (v < 0) v += p;
    return 2 * v >= p ? v - p : v;
}
// the product of the other moduli of the set, mod p_m and mod 2^64
constexpr int cofactor_mod(int nm, int m) {
    int v = 1;
    for (int j = 0; j < nm; ++j)
        if (j != m) v = v * MODULI[j] % MODULI[m];
    return v;
}
constexpr u64 cofactor(int nm, int m) {   // m == nm: the product of all, negated (the term of k)
    u64 v = m == nm ? ~0ull : 1ull;
    for (int j = 0; j < nm; ++j)
        if (j != m) v *= (u64)MODULI[j];
    return v;
}
constexpr int cofactor_inverse(int nm, int m) {
    const int c = cofactor_mod(nm, m);
    for (int i = 1; i < MODULI[m]; ++i)
        if (c * i % MODULI[m] == 1) return i;
    return 0;
}
// 2^(8l) mod p_m for four digits from l0 on, centred, as one dword; times the inverse for the right operand
constexpr u32 digit_coefs(int nm, int m, int l0, bool right) {
    u32 v = 0;
    for (int j = 0; j < 4; ++j) {
        int c = right ? cofactor_inverse(nm, m) : 1;
        for (int l = 0; l < l0 + j; ++l) c = c * 256 % MODULI[m];
        v |= ((u32)centred(c, MODULI[m]) & 255u) << (8 * j);
    }
    return v;
}
// digit d of the cofactors of moduli 4g .. 4g+3, one dword; the entry behind the last modulus belongs to k
constexpr u32 cofactor_digits(int nm, int g, int d) {
    u32 v = 0;
    for (int j = 0; j < 4; ++j) {
        const int m = 4 * g + j;
        // k sits in the last byte of the last group
        const int e = g == 4 && j == 3 ? nm : (m < nm ? m : -1);
        if (e < 0) continue;
        const u64 t = (cofactor(nm, e) + 0x8080808080808080ull) ^ 0x8080808080808080ull;
        v |= ((u32)(t >> (8 * d)) & 255u) << (8 * j);
    }
    return v;
}
// round(2^22 / p_m) as two signed digits
constexpr u32 quotient_digits(int nm, int g, int d) {
    u32 v = 0;
    for (int j = 0; j < 4; ++j) {
        const int m = 4 * g + j;
        if (m >= nm) continue;
        const int c = ((1 << 23) / MODULI[m] + 1) / 2;
        const int lo = centred(c, 256);
        v |= (u32)((d ? (c - lo) / 256 : lo) & 255) << (8 * j);
    }
    return v;
}

template <class F, int... I>
__device__ __forceinline__ void for_each_index(F f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}

// The low byte of t mod p, centred, for |t| < 2^22.1: q = round(t / p) read off the mantissa of t / p + 1.5 * 2^23
// (q * p has the low byte the biased mantissa times p has, since 2^22 * p ends in zeros).  t / p is at least
// 1 / (2 p) away from a half and computed to 8e-4, so the result lies in [-p/2, p/2] and fits a byte.
__device__ __forceinline__ u32 reduce_byte(int t, float t_float, float inv_p, int neg_p) {
    const float q = __builtin_fmaf(t_float, inv_p, 12582912.0f);
    return (u32)(__mul24((int)__float_as_uint(q), neg_p) + t);
}

// hi * c + lo of the halves of v, hi signed and lo not, for |c| <= 2^15: an and and one multiply-add that picks the half
__device__ __forceinline__ int fold16(int v, int c) {
    int r = v & 0xffff;
    asm("v_mad_i32_i16 %0, %1, %2, %0 op_sel:[1,0,0,0]" : "+v"(r) : "v"(v), "s"(c));
    return r;
}

__device__ __forceinline__ u32 pack4(u32 a, u32 b, u32 c, u32 d) {
    const u32 lo = __builtin_amdgcn_perm(b, a, 0x0c0c0400u);
    const u32 hi = __builtin_amdgcn_perm(d, c, 0x0c0c0400u);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

__device__ __forceinline__ u32 fast_div(u32 n, FastDiv d) { return (__umulhi(n, d.mul) + n) >> d.shift; }

// ---- 1. operands to residues --------------------------------------------------------------------------------------
// Plane layout: [modulus][slice of 64 words][tap][term][row][64 bytes]; the terms are x_a, x_b on the left and
// w_a + w_b, w_a on the right.  The rows a tile of the product reads in a step (one term of one slice) follow each
// other: 16 KB in one run for 256 rows of a matrix.
// A thread takes 8 words of both shares; 8 lanes write one row, a wave 8 rows of one slice.  FLIP: row (tap, n) of the right operand
// has its words at [word][taps - 1 - tap][n] of a filter; the 8 rows of a wave are neighbours in n.
template <int NM, bool RIGHT, bool FLIP = false>
__device__ __forceinline__ void planes_part(const u64* __restrict__ a, const u64* __restrict__ b, char* __restrict__ out,
                                            u64 plane, u32 unit, int words, int slices, u32 rows, u32 out_rows, u32 taps,
                                            FastDiv div_slices, FastDiv div_taps, bool vec) {
    const u32 rows8 = fast_div(unit >> 6, div_slices);
    const u32 slice = (unit >> 6) - rows8 * (u32)slices;
    const u32 row = rows8 * 8u + ((unit >> 3) & 7u);
    if (row >= out_rows * taps) return;
    // words k, k + 1 of every sixteen: the eight lanes of a row read whole lines (any order within a slice will do, as
    // long as both operands have it)
    const int k = (int)(slice * 64u + (unit & 7u) * 2u);
    u64 va[8], vb[8];
    // (row of the plane and tap: a filter's own order is [row][tap])
    const u32 major = fast_div(row, div_taps);
    const u32 out_row = FLIP ? row - major * out_rows : major, tap = FLIP ? major : row - major * taps;
    const size_t at = FLIP ? ((size_t)k * taps + (taps - 1u - tap)) * out_rows + out_row : (size_t)row * (size_t)words + (size_t)k;
    const size_t pitch = FLIP ? (size_t)taps * out_rows : 1;
    // (a whole slice apart from the last one of a row: with a test around every load the loads wait for one another, and converting a filter
    // of 848 x 3 x 3 x 1104 takes 139 us instead of 113)
    if (!FLIP && vec && row < rows && slice * 64u + 64u <= (u32)words) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const ulonglong2 ta = *reinterpret_cast<const ulonglong2*>(a + at + 16 * j);
            const ulonglong2 tb = *reinterpret_cast<const ulonglong2*>(b + at + 16 * j);
            va[2 * j] = ta.x; va[2 * j + 1] = ta.y;
            vb[2 * j] = tb.x; vb[2 * j + 1] = tb.y;
        }
    } else if (!FLIP && vec) {   // an even number of words: both of a pair are there or none
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool in = row < rows && k + 16 * j < words;
            const ulonglong2 zero = {0, 0};
            const ulonglong2 ta = in ? *reinterpret_cast<const ulonglong2*>(a + at + 16 * j) : zero;
            const ulonglong2 tb = in ? *reinterpret_cast<const ulonglong2*>(b + at + 16 * j) : zero;
            va[2 * j] = ta.x; va[2 * j + 1] = ta.y;
            vb[2 * j] = tb.x; vb[2 * j + 1] = tb.y;
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int w = 16 * (j >> 1) + (j & 1);
            const bool in = row < rows && k + w < words;
            va[j] = in ? a[at + w * pitch] : 0;
            vb[j] = in ? b[at + w * pitch] : 0;
        }
    }
    u32 d[2][8][2];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const u64 first = RIGHT ? va[j] + vb[j] : va[j], second = RIGHT ? va[j] : vb[j];
        const u64 t0 = (first + 0x8080808080808080ull) ^ 0x8080808080808080ull;
        const u64 t1 = (second + 0x8080808080808080ull) ^ 0x8080808080808080ull;
        d[0][j][0] = (u32)t0; d[0][j][1] = (u32)(t0 >> 32);
        d[1][j][0] = (u32)t1; d[1][j][1] = (u32)(t1 >> 32);
    }
    char* dst = out + ((size_t)(slice * taps + tap) * 2u * out_rows + out_row) * 64u + (unit & 7u) * 8u;
    const size_t term_bytes = (size_t)out_rows * 64u;
    for_each_index([&](auto mi) {
        constexpr int m = decltype(mi)::value;
        constexpr u32 c_lo = digit_coefs(NM, m, 0, RIGHT), c_hi = digit_coefs(NM, m, 4, RIGHT);
        constexpr float inv_p = 1.0f / (float)MODULI[m];
#pragma unroll
        for (int term = 0; term < 2; ++term) {
            u32 r[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                int t = __builtin_amdgcn_sdot4((int)d[term][j][0], (int)c_lo, 0, false);
                t = __builtin_amdgcn_sdot4((int)d[term][j][1], (int)c_hi, t, false);
                r[j] = reduce_byte(t, (float)t, inv_p, -MODULI[m]);
            }
            u2 v;
            v.x = pack4(r[0], r[1], r[2], r[3]);
            v.y = pack4(r[4], r[5], r[6], r[7]);
            *reinterpret_cast<u2*>(dst + (size_t)m * plane + term * term_bytes) = v;
        }
    }, std::make_integer_sequence<int, NM>{});
}

template <int NM, bool FLIP>
__global__ __launch_bounds__(256) void rns_planes_kernel(RnsParams p, u32 x_blocks, u32 x_units, u32 w_units, int vec) {
    if (blockIdx.x < x_blocks) {
        const u32 unit = blockIdx.x * 256u + threadIdx.x;
        if (unit < x_units)
            planes_part<NM, false>(p.x_a, p.x_b, p.xp, p.x_plane, unit, p.words, p.slices, (u32)p.x_rows, (u32)p.x_rows + 1u, 1u,
                                   p.div_slices, FastDiv{1u, 0u}, vec);
    } else {
        const u32 unit = (blockIdx.x - x_blocks) * 256u + threadIdx.x;
        if (unit < w_units)
            planes_part<NM, true, FLIP>(p.w_a, p.w_b, p.wp, p.w_plane, unit, p.words, p.slices, (u32)(p.N * p.kh * p.kw),
                                        (u32)p.N, (u32)(p.kh * p.kw), p.div_slices, FLIP ? p.div_n : p.div_taps, vec);
    }
}

// ---- 2. one int8 product per modulus ------------------------------------------------------------------------------
struct ModConst {
    int p, shift16;   // shift16: 2^16 mod p, centred
    float inv;
};
constexpr ModConst mod_const(int m) {
    return ModConst{MODULI[m], centred(65536, MODULI[m]), 1.0f / (float)MODULI[m]};
}
__constant__ const ModConst MOD_CONST[MAX_MOD] = {
    mod_const(0), mod_const(1), mod_const(2), mod_const(3), mod_const(4), mod_const(5), mod_const(6),
    mod_const(7), mod_const(8), mod_const(9), mod_const(10), mod_const(11), mod_const(12), mod_const(13),
    mod_const(14), mod_const(15), mod_const(16), mod_const(17), mod_const(18)};

constexpr int GROUP_M = 4;   // tile rows taken together down the columns

// A block computes one BM x BN tile for one modulus.  A step is one term of one slice: 64 bytes per row, which go to
// LDS directly, into the oldest of four buffers.  LDS row r holds its four 16-byte pieces at positions
// (piece ^ (-(r >> 2) & 3)); the loads place them by choosing which piece each lane fetches.  A 16-byte read of a wave runs in
// four turns of 16 lanes: lanes 0-3, 12-15, 20-27, then 4-11, 16-19, 28-31, then the same of the upper half.  A turn of a
// fragment load therefore reads four rows in four of two pieces, and this order puts them in 16 different groups of four banks
// (SQ_LDS_BANK_CONFLICT 0; with (r >> 2) & 3, made for 16 lanes in a row, half of the LDS cycles were conflicts).
template <int BM, int BN, int WM, int WN, bool CONV>
__global__ __launch_bounds__(64 * WM * WN, 2) void rns_gemm_kernel(RnsParams p) {
    constexpr int NW = WM * WN;
    constexpr bool BIG = BM == 256;
    constexpr u32 SLOTS = BIG ? 256u : 512u;   // blocks that run at one time
    constexpr int TM = BM / WM / 16, TN = BN / WN / 16;   // 16 x 16 results of a wave
    constexpr int LA = BM / 16 / NW, LB = BN / 16 / NW;   // 1 KB loads of a wave per step
    __shared__ __attribute__((aligned(1024))) char buf0[(BM + BN) * 64];
    __shared__ __attribute__((aligned(1024))) char buf1[(BM + BN) * 64];
    __shared__ __attribute__((aligned(1024))) char buf2[(BM + BN) * 64];
    __shared__ __attribute__((aligned(1024))) char buf3[(BM + BN) * 64];

    // Each of the 8 XCDs takes a contiguous run of (modulus, tile): its L2 then holds few moduli's planes, and
    // neighbouring tiles share rows.  The run is one of the whole grid, or (by_rounds) of the blocks that run at one time, see
    // rns_plan.
    u32 first = 0, total = gridDim.x, at = blockIdx.x;
    if (p.by_rounds) {
        first = at & ~(SLOTS - 1u);
        at &= SLOTS - 1u;
        total = min(total - first, SLOTS);
    }
    const u32 xcd = at & 7u, left = total & 7u;
    const u32 logical = first + xcd * (total >> 3) + (xcd < left ? xcd : left) + (at >> 3);
    const RnsPart& part = BIG ? p.large : p.small;
    const u32 mod_at = fast_div(logical, part.div_tiles), mod = (u32)part.first + mod_at;
    const u32 tile = logical - mod_at * (u32)(part.tiles_m * part.tiles_n);
    const u32 group = fast_div(tile, part.div_group);
    const u32 in_group = tile - group * (u32)(GROUP_M * part.tiles_n);
    const u32 group_rows = min((u32)GROUP_M, (u32)part.tiles_m - group * GROUP_M);
    const u32 tile_n = in_group / group_rows;
    const u32 tile_m = group * GROUP_M + (in_group - tile_n * group_rows);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    __amdgpu_buffer_rsrc_t rs_x = make_rsrc(p.xp + (size_t)mod * p.x_plane, (u32)p.x_plane);
    __amdgpu_buffer_rsrc_t rs_w = make_rsrc(p.wp + (size_t)mod * p.w_plane, (u32)p.w_plane);
    const u32 x_step = ((u32)p.x_rows + 1u) * 64u, w_step = (u32)p.N * 64u;

    u32 x_off[LA], w_off[LB];
    int iy0[LA], ix0[LA];
    u32 corner[LA];   // offset of the window's first pixel
    const u32 piece = (u32)((lane & 3) ^ (-(lane >> 4) & 3)) * 16u;
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const u32 m = tile_m * BM + (u32)(wave * LA + i) * 16u + (u32)(lane >> 2);
        if (CONV) {
            const u32 b = fast_div(m, p.div_howo), rest = m - b * (u32)(p.Ho * p.Wo);
            const u32 oy = fast_div(rest, p.div_wo), ox = rest - oy * (u32)p.Wo;
            iy0[i] = (int)oy * p.sh - p.ph;
            ix0[i] = (int)ox * p.sw - p.pw;
            corner[i] = ((b * (u32)p.H + (u32)iy0[i]) * (u32)p.W + (u32)ix0[i]) * 64u + piece;   // (mod 2^32)
            if (m >= (u32)p.M) iy0[i] = -(1 << 30);   // rows beyond M: never inside the image
        } else {
            x_off[i] = min(m, (u32)p.x_rows) * 64u + piece;
        }
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const u32 n = tile_n * BN + (u32)(wave * LB + i) * 16u + (u32)(lane >> 2);
        w_off[i] = min(n, (u32)p.N - 1u) * 64u + piece;
    }

    int tap_r = 0, tap_c = 0;
    u32 x_at = 0, w_at = 0;
    // load number i of the LA + LB that bring a wave's share of a step's lines to LDS
    auto fetch = [&](char* buf, int i) {
        if (i < LA)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs_x, (__attribute__((address_space(3))) void*)(buf + (wave * LA + i) * 1024), 16, (int)x_off[i],
                (int)x_at, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs_w, (__attribute__((address_space(3))) void*)(buf + BM * 64 + (wave * LB + i - LA) * 1024), 16,
                (int)w_off[i - LA], (int)w_at, 0, 0);
    };
    auto window = [&]() {   // the rows of the tap that begins
        const u32 tap = (u32)(tap_r * p.W + tap_c) * 64u;
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const bool in = (u32)(iy0[i] + tap_r) < (u32)p.H & (u32)(ix0[i] + tap_c) < (u32)p.W;
            x_off[i] = in ? corner[i] + tap : (u32)p.x_rows * 64u;   // (any piece of the row of zeros)
        }
    };
    v4i acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    const int wave_m = wave / WN, wave_n = wave % WN;
    const int frag = (lane & 15) * 64 + ((lane >> 4) ^ (-(lane >> 2) & 3)) * 16;
    auto left_frag = [&](const char* buf, int i) {
        return *reinterpret_cast<const v4i*>(buf + frag + (wave_m * TM + i) * 1024);
    };
    auto right_frag = [&](const char* buf, int j) {
        return *reinterpret_cast<const v4i*>(buf + frag + BM * 64 + (wave_n * TN + j) * 1024);
    };
    auto multiply_one = [&](int i, int j, const v4i (&xf)[TM], const v4i (&wf)[TN]) {
        // the right operand's rows first: a lane then owns four columns of a row
        acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wf[j], xf[i], acc[i][j], 0, 0, 0);
    };
    auto multiply = [&](int i, const v4i (&xf)[TM], const v4i (&wf)[TN]) {
#pragma unroll
        for (int j = 0; j < TN; ++j) multiply_one(i, j, xf, wf);
    };

    // Fragments of the next step are read while this one is multiplied: a left fragment's registers take the next one
    // as soon as their row of products is issued, the right operand's are double-buffered.  The step's one barrier
    // stands GAP rows in, where a wave has every fragment of the step in registers and the next step's lines have
    // landed; the loads into the buffer just read are spread over the remaining rows (issued in one run they hold a
    // wave back for as long as the address unit takes for all waves' loads) and have three steps to arrive.
    constexpr int GAP = TM / 4, ROWS = TM - GAP;
    constexpr int FETCHES = (LA + LB + ROWS - 1) / ROWS, READS = (TN + ROWS - 1) / ROWS;   // per row
    static_assert(2 * FETCHES <= TN && READS <= 2, "places for the requests of a row");
    const int steps = 2 * p.slices * p.kh * p.kw;
    v4i x[TM], w0[TN], w1[TN];
    int left_steps = steps;   // steps whose lines are still to be fetched
    // Order of the steps of a gathered operand: slice by slice, in a slice tap by tap, the two terms of a tap one after
    // the other: the taps of a slice find the lines they share in the L2.  (Tap by tap over all slices, every tap came from
    // beyond it where the image is wide: 3x3 stride 2 layers up to 2.3 times the time, e.g. 15 x 69 x 69 x 896 -> 144 5x5 10.2
    // -> 4.5 ms.)  `second` is known where a step stands, so the window's arithmetic needs no branch; with one, and a
    // word more per row, 14 registers of the large tile spilled, and their reloads waited for every load in flight: 17 % of the call.
    auto advance = [&](bool second) {
        w_at += w_step;
        if (!CONV || !second) {
            x_at += x_step;
        } else {
            const bool row_end = ++tap_c == p.kw;
            tap_c = row_end ? 0 : tap_c;
            tap_r += row_end;
            const bool slice_end = tap_r == p.kh;
            tap_r = slice_end ? 0 : tap_r;
            x_at += slice_end ? x_step : 0u - x_step;
        }
        if (--left_steps <= 0) {   // views of no bytes: the loads behind the last step move nothing
            rs_x = make_rsrc(p.xp, 0);
            rs_w = make_rsrc(p.wp, 0);
        }
    };
    // The wave's own loads to LDS of all but the last two steps have landed and its fragments have arrived, and then
    // everyone's.  (__syncthreads() would wait for the last two steps as well.)
    auto landed = [&]() {
        asm volatile("" ::: "memory");
        static_assert(2 * (LA + LB) < 16, "vmcnt's low field");
        __builtin_amdgcn_s_waitcnt(0x0070 | (2 * (LA + LB)));   // vmcnt, lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto step = [&](char* cur, const char* next, const v4i (&w)[TN], v4i (&w_next)[TN], bool second) {
#pragma unroll
        for (int i = 0; i < GAP; ++i) multiply(i, x, w);
        __builtin_amdgcn_sched_barrier(0);
        landed();
        if (CONV && !second) window();
        // the requests spread over the products, one at most between two on the large tile (the small one's rows are too short for
        // that: two fragments after the first product): what a wave issues in a run keeps its matrix core waiting
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                multiply_one(GAP + i, j, x, w);
                if (i == 0) {
                    if (j < GAP) x[j] = left_frag(next, j);
                } else if (j == 0) {
                    x[GAP + i - 1] = left_frag(next, GAP + i - 1);
                }
#pragma unroll
                for (int f = 0; f < FETCHES; ++f)
                    if (j == 1 + f * 2 && i * FETCHES + f < LA + LB) fetch(cur, i * FETCHES + f);
#pragma unroll
                for (int f = 0; f < READS; ++f)
                    if (j == (2 + f * 2) % TN && i * READS + f < TN) w_next[i * READS + f] = right_frag(next, i * READS + f);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        x[TM - 1] = left_frag(next, TM - 1);
        advance(second);
    };
    auto fetch_all = [&](char* buf, bool second) {
        if (CONV && !second) window();
#pragma unroll
        for (int f = 0; f < LA + LB; ++f) fetch(buf, f);
        advance(second);
    };
    fetch_all(buf0, false);
    fetch_all(buf1, true);
    fetch_all(buf2, false);
    landed();
    fetch_all(buf3, true);
#pragma unroll
    for (int i = 0; i < TM; ++i) x[i] = left_frag(buf0, i);
#pragma unroll
    for (int j = 0; j < TN; ++j) w0[j] = right_frag(buf0, j);
    // (an even number of steps; the last one reads fragments that nobody uses)
    for (int s = steps >> 2; s > 0; --s) {
        step(buf0, buf1, w0, w1, false);
        step(buf1, buf2, w1, w0, true);
        step(buf2, buf3, w0, w1, false);
        step(buf3, buf0, w1, w0, true);
    }
    if (steps & 2) {
        step(buf0, buf1, w0, w1, false);
        step(buf1, buf2, w1, w0, true);
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);   // no load may reach LDS once the block has given it up

    // Accumulators to residues: v = hi * 2^16 + lo with lo unsigned, and hi * (2^16 mod p) + lo is below 2^22.1.  A row of blocks
    // at a time and stage by stage, so that no instruction waits for the one before it.
    const ModConst mc = MOD_CONST[mod];
    char* out = p.rp + (size_t)mod * p.r_plane;
    const u32 blocks_n = (u32)p.blocks_n;
    const u32 bm = tile_m * (BM / 16) + (u32)(wave_m * TM), bn = tile_n * (BN / 16) + (u32)(wave_n * TN);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        int t[TN][4];
        float f[TN][4];
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) t[j][e] = fold16(acc[i][j][e], mc.shift16);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) f[j][e] = (float)t[j][e];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) t[j][e] = (int)reduce_byte(t[j][e], f[j][e], mc.inv, -mc.p);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < TN; ++j)
            *reinterpret_cast<u32*>(out + ((size_t)(bm + i) * blocks_n + bn + j) * 256u + lane * 4) =
                pack4((u32)t[j][0], (u32)t[j][1], (u32)t[j][2], (u32)t[j][3]);
    }
}

// ---- 3. residues to words -----------------------------------------------------------------------------------------
// Result planes: [modulus][16 x 16 block][lane of the product kernel][4 columns]; a thread takes four outputs.
template <int NM>
__global__ __launch_bounds__(256) void rns_combine_kernel(RnsParams p, u32 quads, int zvec) {
    const u32 q = blockIdx.x * 256u + threadIdx.x;
    if (q >= quads) return;
    const u32 block = q >> 6, lane = q & 63u;
    const u32 bm = fast_div(block, p.div_blocks_n), bn = block - bm * (u32)p.blocks_n;
    const u32 m = bm * 16u + (lane & 15u), n = bn * 16u + (lane >> 4) * 4u;
    if (m >= (u32)p.M || n >= (u32)p.N) return;
    const char* src = p.rp + (size_t)q * 4u;
    u32 r[20];
#pragma unroll
    for (int i = 0; i < 20; ++i) r[i] = i < NM ? *reinterpret_cast<const u32*>(src + (size_t)i * p.r_plane) : 0u;
    u32 g[5][4];   // [group of four moduli][output]
#pragma unroll
    for (int i = 0; i < 5; ++i) transpose4(r[4 * i], r[4 * i + 1], r[4 * i + 2], r[4 * i + 3], g[i]);
    u64 z[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        int k_lo = 1 << 21, k_hi = 0;
        for_each_index([&](auto gi) {
            constexpr int i = decltype(gi)::value;
            constexpr u32 c0 = quotient_digits(NM, i, 0), c1 = quotient_digits(NM, i, 1);
            k_lo = __builtin_amdgcn_sdot4((int)g[i][e], (int)c0, k_lo, false);
            k_hi = __builtin_amdgcn_sdot4((int)g[i][e], (int)c1, k_hi, false);
        }, std::make_integer_sequence<int, 5>{});
        const u32 k = (u32)((k_lo + (k_hi << 8)) >> 22);
        const u32 last = (g[4][e] & 0x00ffffffu) | (k << 24);
        int s[8];
        for_each_index([&](auto di) {
            constexpr int d = decltype(di)::value;
            int v = 0;
            for_each_index([&](auto gi) {
                constexpr int i = decltype(gi)::value;
                constexpr u32 c = cofactor_digits(NM, i, d);
                v = __builtin_amdgcn_sdot4((int)(i == 4 ? last : g[i][e]), (int)c, v, false);
            }, std::make_integer_sequence<int, 5>{});
            s[d] = v;
        }, std::make_integer_sequence<int, 8>{});
        // |s| < 2^19: neighbours combine in 32 bits, the upper half only matters mod 2^32
        const int64_t lo = (int64_t)(s[0] + (s[1] << 8)) + (int64_t)(s[2] + (s[3] << 8)) * 65536;
        const u32 hi = (u32)s[4] + ((u32)s[5] << 8) + ((u32)s[6] << 16) + ((u32)s[7] << 24);
        z[e] = (u64)lo + ((u64)hi << 32);
    }
    u64* dst = p.z + (size_t)m * (size_t)p.N + n;
    if (zvec && n + 4u <= (u32)p.N) {
        reinterpret_cast<ulonglong2*>(dst)[0] = ulonglong2{z[0], z[1]};
        reinterpret_cast<ulonglong2*>(dst)[1] = ulonglong2{z[2], z[3]};
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (n + (u32)e < (u32)p.N) dst[e] = z[e];
    }
}

uint64_t up256(uint64_t v) { return (v + 255) / 256 * 256; }

template <int BM, int BN, int WM, int WN>
hipError_t launch_gemm(const RnsParams& p, const RnsPart& part, hipStream_t stream) {
    const u32 grid = (u32)(part.tiles_m * part.tiles_n * part.count);
    if (grid == 0) return hipSuccess;
    if (p.conv) hipLaunchKernelGGL((rns_gemm_kernel<BM, BN, WM, WN, true>), dim3(grid), dim3(64 * WM * WN), 0, stream, p);
    else        hipLaunchKernelGGL((rns_gemm_kernel<BM, BN, WM, WN, false>), dim3(grid), dim3(64 * WM * WN), 0, stream, p);
    return hipGetLastError();
}

template <int NM>
hipError_t run(const RnsParams& p, hipStream_t stream) {
    const u32 x_units = ((u32)p.x_rows + 8u) / 8u * (u32)p.slices * 64u;   // x_rows and the row of zeros
    const u32 w_units = ((u32)(p.N * p.kh * p.kw) + 7u) / 8u * (u32)p.slices * 64u;
    const u32 x_blocks = (x_units + 255u) / 256u, w_blocks = (w_units + 255u) / 256u;
    const int vec = p.words % 2 == 0 && (((uintptr_t)p.x_a | (uintptr_t)p.x_b | (uintptr_t)p.w_a | (uintptr_t)p.w_b) & 15) == 0;
    auto planes = p.flip ? rns_planes_kernel<NM, true> : rns_planes_kernel<NM, false>;
    hipLaunchKernelGGL(planes, dim3(x_blocks + w_blocks), dim3(256), 0, stream, p, x_blocks, x_units, w_units, vec);
    if (hipError_t e = hipGetLastError()) return e;
    if (hipError_t e = launch_gemm<256, 256, 2, 4>(p, p.large, stream)) return e;
    if (hipError_t e = launch_gemm<128, 128, 2, 2>(p, p.small, stream)) return e;
    const u32 quads = (u32)(p.r_plane / 4);
    const int zvec = p.N % 2 == 0 && ((uintptr_t)p.z & 15) == 0;
    hipLaunchKernelGGL((rns_combine_kernel<NM>), dim3((quads + 255u) / 256u), dim3(256), 0, stream, p, quads, zvec);
    return hipGetLastError();
}

// The first `large` moduli on the large tile and the others on the small one
void set_parts(RnsParams* p, int large) {
    auto set = [&](RnsPart& part, int edge, int first, int count) {
        part.tiles_m = (int)((p->M + (int64_t)edge - 1) / edge);
        part.tiles_n = (int)((p->N + (int64_t)edge - 1) / edge);
        part.first = first; part.count = count;
    };
    set(p->large, 256, 0, large);
    set(p->small, 128, large, p->nmod - large);
}

// ... and all that follows from it
void share_moduli(RnsParams* p, int large) {
    set_parts(p, large);
    for (RnsPart* part : {&p->large, &p->small}) {
        part->div_tiles = make_fast_div((uint32_t)(part->tiles_m * part->tiles_n));
        part->div_group = make_fast_div((uint32_t)(GROUP_M * part->tiles_n));
    }
    const RnsPart& pitch = large > 0 ? p->large : p->small;   // the result's planes hold whole tiles of the larger size
    const int edge = large > 0 ? 256 : 128;
    p->blocks_n = pitch.tiles_n * (edge / 16);
    p->div_blocks_n = make_fast_div((uint32_t)p->blocks_n);
    p->r_plane = (uint64_t)pitch.tiles_m * pitch.tiles_n * edge * edge;
}

}  // namespace

bool rns_plan(RnsParams* p) {
    const int64_t taps = (int64_t)p->kh * p->kw, K = taps * p->words;
    if (K > RNS_K_MAX) return false;
    p->nmod = K <= RNS_K_18 ? 18 : 19;
    p->slices = (p->words + 63) / 64;
    const uint64_t x_plane = (uint64_t)(p->x_rows + (int64_t)1) * p->slices * 128u;
    const uint64_t w_plane = (uint64_t)p->N * taps * p->slices * 128u;
    const int64_t tm = (p->M + (int64_t)255) / 256, tn = (p->N + (int64_t)255) / 256;
    // planes are addressed with 32-bit offsets, results with 32-bit quad numbers
    if (x_plane >= (1ull << 31) || w_plane >= (1ull << 31) || (uint64_t)tm * (uint64_t)tn * 65536u >= (1ull << 31))
        return false;
    p->x_plane = x_plane;
    p->w_plane = w_plane;
    // With one size of tile for all moduli: the less modelled time, in microseconds, by which the caller's rule decides
    // (fitted to the kernels as they were before the shares below and before reads without bank conflicts, 3 - 6 % slower).  A step is a tap of a slice.  The chip takes 256 of the large tile's
    // blocks at a time and 512 of the small one's; a part of the time goes with the rounds and a part with the blocks (a
    // compute unit with one small block runs it faster).  Strided layers leave half of every line they gather unused.
    // The residues that are read once (those of a matrix, of a filter) come on top.  Small against large tile, whole
    // calls: 423 / 366 us at 2048^3, 359 / 330 us at 1023 x 2047 x 3001, but 83 / 102 us at 1000 x 777 x 1531; 3x3 layer
    // 16 x 16 x 256 -> 256 at batch 32 189 / 193 us, the 5x5 one 472 / 446 us.  Coefficients: least squares over whole calls with either
    // tile forced, 1300 products (M, N 65 .. 16384, K 64 .. 65000) and 1900 layers (1 .. 64 images of 4 x 4 .. 128 x 128, 16 .. 2048
    // channels, windows of 1 .. 7, strides of 1 .. 3); eight in ten within 6 % for the large tile, 20 % for the small one.
    struct Shape { int edge, slots; double round_step, block_step, fixed, per_mb; };
    static const Shape shapes[3][2] = {   // rows of a matrix, patches, patches of a strided layer
        {{256, 256, 0.96, 0.37, 6.0, 0.012}, {128, 512, 0.31, 0.54, 2.5, 0.075}},
        {{256, 256, 1.08, 0.27, 5.5, 0.05}, {128, 512, 0.34, 0.48, 1.7, 0.13}},
        {{256, 256, 1.07, 0.34, 7.4, 0.06}, {128, 512, 0.33, 0.68, 3.0, 0.12}}};
    const int kind = !p->conv ? 0 : p->sh == 1 && p->sw == 1 ? 1 : 2;
    const double steps = (double)(taps * p->slices), once_mb = 1.0e-6 * p->nmod * (double)(w_plane + (p->conv ? 0 : x_plane));
    double best = 0.0;
    for (const Shape& t : shapes[kind]) {
        const int64_t tiles_m = (p->M + (int64_t)t.edge - 1) / t.edge, tiles_n = (p->N + (int64_t)t.edge - 1) / t.edge;
        const int64_t blocks = tiles_m * tiles_n * p->nmod, rounds = (blocks + t.slots - 1) / t.slots;
        const double cost = steps * ((double)rounds * t.round_step + (double)blocks / t.slots * t.block_step) +
                            (double)rounds * t.fixed + once_mb * t.per_mb;
        if (best != 0.0 && cost >= best) continue;
        best = cost;
        p->tile = t.edge;
    }
    p->product_us = best;
    // Which moduli run on the large tile and which on the small one.  The large tile asks half as much of the L1 (half
    // of its 64 bytes a clock, where the small tile takes all), but its rounds are the coarser ones, so whole rounds of it go first
    // and the moduli that would leave its last round partly empty run on the small tile: the 3x3 layer 16 x 16 x 256 -> 256 at
    // batch 32, 191 us with five rounds of the small tile alone (4.5 of work), 179 with two rounds of the large one (16
    // moduli) and half a round of the other.  Modelled as above, and a last round of at most one small block per
    // compute unit takes 0.6 of a full one.  Coefficients: least squares over 8000 whole calls, 2013 shapes (products of M, N 100 .. 8192,
    // K 128 .. 8192; layers of 1 .. 64 images of 4 x 4 .. 112 x 112, 32 .. 1024 channels, windows of 1, 3, 5, strides of 1 and 2) with four
    // shares of the moduli each: nine calls in ten within 14 %; the share chosen is within 2 % of the best one measured for
    // nine shapes in ten, 13 % at worst.
    struct Split { double round_step, block_step, fixed, per_mb; };
    static const Split splits[3][2] = {{{0.714, 0.715, 8.2, 0.0}, {0.300, 0.637, 2.9, 0.033}},
                                       {{0.932, 0.208, 8.2, 0.0}, {0.527, 0.204, 3.7, 0.0}},
                                       {{0.872, 0.384, 8.1, 0.053}, {0.443, 0.465, 4.05, 0.020}}};
    auto cost = [&](const RnsPart& part, const Split& t, int slots) {
        if (part.count == 0) return 0.0;
        const int64_t blocks = (int64_t)part.tiles_m * part.tiles_n * part.count, rounds = (blocks + slots - 1) / slots;
        const bool half = slots == 512 && blocks % 512 != 0 && blocks % 512 <= 256;
        return steps * (((double)rounds - (half ? 0.4 : 0.0)) * t.round_step + (double)blocks / slots * t.block_step) +
               (double)rounds * t.fixed + once_mb / p->nmod * part.count * t.per_mb;
    };
    auto modelled = [&](int large) {
        set_parts(p, large);
        return cost(p->large, splits[kind][0], 256) + cost(p->small, splits[kind][1], 512);
    };
    // Both tiles in one call take 3 us and 3 % more than modelled (one launch more, and the last blocks of the first leave compute units
    // idle), and the other tile alone must be modelled 1 % faster than the one of the rule above: of 2250 calls with the modelled share, all
    // moduli on the large tile and all on the small one measured, the choice takes 1.004 of the best of the three on average (1.005 by
    // modelled time alone, 1.012 with one tile).  Of 900 other layers and 300 products against the code before there were shares four are
    // more than 2 % slower, at most 4 % (by modelled time alone 6 of 900, up to 26 %); all together take 0.94 of its time.
    int best_large = p->tile == 256 ? p->nmod : 0;
    best = modelled(best_large);
    if (const double other = modelled(p->nmod - best_large); other < 0.99 * best) {
        best = other;
        best_large = p->nmod - best_large;
    }
    for (int large = 1; large < p->nmod; ++large) {
        const double us = 1.03 * modelled(large) + 3.0;
        if (us >= best) continue;
        best = us;
        best_large = large;
    }
    share_moduli(p, best_large);
    // An XCD reads the whole right operand once per GROUP_M tile rows, eight moduli's at a time where every XCD has a run of
    // its own.  The last-level cache of 256 MB holds eight of up to some 20 MB; beyond, the XCDs take one modulus
    // together: 34 MB (4096^3) 2154 -> 2097 us, 8192 x 8192 x 2048 4466 -> 4294, 22 MB (2048 x 2048 x 5400) 863 -> 856, 17 MB 1178 / 1178 at
    // 4096 x 4096 x 2048 and 2446 / 2557 at 8192 x 8192 x 1024, 6 MB (3072 x 3072 x 1024) 411 / 422.
    p->by_rounds = p->w_plane >= (20u << 20);
    p->div_slices = make_fast_div((uint32_t)p->slices);
    p->div_taps = make_fast_div((uint32_t)taps);
    p->div_n = make_fast_div((uint32_t)p->N);
    p->div_howo = make_fast_div((uint32_t)(p->conv ? p->Ho * p->Wo : 1));
    p->div_wo = make_fast_div((uint32_t)(p->conv ? p->Wo : 1));
    return true;
}

uint64_t rns_workspace_bytes(const RnsParams& p) {
    return up256(p.x_plane * p.nmod) + up256(p.w_plane * p.nmod) + up256(p.r_plane * p.nmod);
}

bool rns_fit(RnsParams* p, uint64_t bytes) {
    if (bytes < rns_workspace_bytes(*p) && p->tile == 128) share_moduli(p, 0);
    return bytes >= rns_workspace_bytes(*p);
}

hipError_t launch_share_gemm_rns(RnsParams p, void* workspace, hipStream_t stream) {
    p.xp = static_cast<char*>(workspace);
    p.wp = p.xp + up256(p.x_plane * p.nmod);
    p.rp = p.wp + up256(p.w_plane * p.nmod);
    return p.nmod == 18 ? run<18>(p, stream) : run<19>(p, stream);
}

}  // namespace cg
