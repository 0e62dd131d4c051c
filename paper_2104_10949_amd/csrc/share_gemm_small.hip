// The party's local product (CryptGPU Sec. III-B, "Multiplication" and "Convolutions and matrix
// multiplication") for a left operand of few rows (fully connected layers at small batch) and for other small ones.
//
// Such a product is a few microseconds of matrix work, so what counts is the length of the chain
// launch -> load -> split -> multiply -> store and how many compute units share it, not the rate of any
// unit.  A block owns one 16 x 16 block of z (or 8 rows or columns of one, where that still fits one round of the chip); its waves
// share out the 32-word slices of K and never wait for
// each other until the end.  For v_mfma_i32_16x16x64_i8 a lane supplies 16 contraction bytes of one row, so
// lane (r, g) ends up with the sixteen words of row r that make up k-group g (g = 2 * share + half of the
// slice), splits them into eight signed digits in its own registers (which is the operand layout of the
// instruction), and the wave issues the 36 digit-pair products of the slice.  The waves' partial results
// meet in LDS; one plain store per element, or an atomic add when K is
// also split over blocks.
// Same arithmetic as share_gemm_kernel: digits, accumulators P_0..P_7, one fold at the end (the launcher takes
// products of at most 511 slices per wave).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "share_digits.h"
#include "share_gemm_split.h"

namespace cg {
namespace {

constexpr int SMALL_WAVES = 8;        // waves of a block: two per SIMD, 256 registers each
constexpr int SMALL_MAX_SLICES = 511 * SMALL_WAVES;  // a wave's i32 accumulators stay exact for 511 slices (see share_gemm.hip)
// Which products the launcher takes.  The lines were measured with blocks of 16 x 16 only and sums through LDS atomics; with the kernels
// as they are (1160 calls on both sides) they hold for the plain call, and lie low: two rounds win up to 15 slices (0.91 of the tiled kernel's
// time, 1.01 at worst), four rounds with three and four (0.93), 17 .. 64 rows up to 6000 units (0.93).  The call that adds to z takes 0.94 at
// 4600 units, single shapes up to 1.28.
// Measured against share_gemm_kernel at M = 8, 32, 64, N = 64 .. 4096, K = 128 .. 25088: with one 16-row block every shape up to the
// slice limit (3.5 us against 11 us at K = 128, 285 against 369 us at 8 x 4096 x 25088); with two to four row blocks the right operand is read once per row
// block, and the tiled kernel wins from about 4600 (16 x 16 block, slice) units on.
// With more than 64 rows the same unit line holds and the rounds of the chip set a second one (a block fills a compute
// unit; 1030 shapes with M = 65 .. 12288, N = 10 .. 2448, K = 32 .. 14720, whole calls against share_gemm_kernel).  Up to
// 256 blocks: 128 x 128 x 784 14.5 -> 8.8 us, 256 x 256 x 128 11.8 -> 4.1, 1024 x 64 x 512 14.0 -> 8.3.  Two rounds: won up to
// 13 slices (0.95 of the tiled kernel's time at worst, 1.04 at 14).  Three: a single slice is not worth three folds
// (12288 x 16 x 32 6.6 -> 8.1 us), two and more are (0.91 of the time at 12288 x 16 x 64).  A fourth round never pays (512 x 512 x 64
// 9.7 -> 10.9).  The tiled kernel needs no clearing launch when it adds to z, so those lines lie lower: 11 slices in two
// rounds (0.96; 1.11 at 12), 2 and 3 in three (0.92; 1.08 at four).
constexpr int SMALL_ONE_BLOCK_ROWS = 16;
constexpr int64_t SMALL_MAX_UNITS = 4608;
constexpr int SMALL_MANY_ROWS = 64;
// K is split over blocks as well as long as the grid stays within one round (one block per compute unit fits):
// 320 x 29 x 3680, 40 blocks of z, split in 7 (280 blocks) 18.5 us, in 6 (240) 10.7
constexpr int64_t SMALL_ROUND_BLOCKS = 256;

// Sixteen words (eight 16-byte registers, word 2i in v[i].xy and word 2i+1 in v[i].zw) -> eight digit
// registers: byte 4j + t of d[l] is digit l of word 4j + t.
__device__ __forceinline__ void split16(u4 (&v)[8], v4i (&d)[8]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        u32 lo[4] = {v[2 * j].x, v[2 * j].z, v[2 * j + 1].x, v[2 * j + 1].z};
        u32 hi[4] = {v[2 * j].y, v[2 * j].w, v[2 * j + 1].y, v[2 * j + 1].w};
#pragma unroll
        for (int t = 0; t < 4; ++t) recode(lo[t], hi[t]);
        u32 dl[4], dh[4];
        transpose4(lo[0], lo[1], lo[2], lo[3], dl);
        transpose4(hi[0], hi[1], hi[2], hi[3], dh);
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            d[l][j] = (int)dl[l];
            d[4 + l][j] = (int)dh[l];
        }
    }
}

__device__ __forceinline__ u4 add64x2(u4 a, u4 b) {
    const u64 s0 = (((u64)a.y << 32) | a.x) + (((u64)b.y << 32) | b.x);
    const u64 s1 = (((u64)a.w << 32) | a.z) + (((u64)b.w << 32) | b.z);
    u4 r;
    r.x = (u32)s0; r.y = (u32)(s0 >> 32); r.z = (u32)s1; r.w = (u32)(s1 >> 32);
    return r;
}

// grid: x = block of COLS columns of z, y = block of ROWS rows, z = range of K slices (gridDim.z > 1: z is cleared or
// holds the value to add to, and every block adds atomically).  Rows of the operands past M or N are
// replaced by the last row: their products land in elements that are never stored.
//
// A slice on its way to the matrix instruction.  Memory wants neighbouring lanes on neighbouring bytes, the
// instruction wants lane (r, g) to hold words of row r only, so the raw words cross a wave-private LDS
// buffer: four regions (x_a, x_b, w_a + w_b, w_a) of 16 rows x 256 bytes.  Loads and LDS writes run with sixteen
// lanes along the sixteen 16-byte pieces of a row's slice (four rows per instruction); the read-back has lane
// (r, g) take the eight pieces of half g & 1 of row r in region g >> 1.  Piece p of row r sits at piece
// p ^ r, rows 4 .. 11 with the halves exchanged: a 16-byte read runs in turns of 16 lanes (0-3, 12-15, 20-27, then 4-11, 16-19,
// 28-31, then the same of the upper half), so a turn of the read-back takes eight rows' piece of one half and the other
// eight rows' piece of the other, and these are sixteen different groups of four banks.  With plain p ^ r every turn met
// a conflict: 32 x 512 x 512 7.38 -> 7.23 us, 128 x 128 x 784 10.29 -> 10.21.  No barrier is involved: a wave reads what it wrote
// itself.
template <int ROWS, int COLS>
__global__ __launch_bounds__(SMALL_WAVES * 64) void share_gemm_small_kernel(const GemmParams p) {
    __shared__ __attribute__((aligned(16))) char stage[SMALL_WAVES][4][16 * 256];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // said to be uniform: the slice loop runs on the scalar unit

    const int n0 = blockIdx.x * COLS, m0 = blockIdx.y * ROWS;
    const u32 K = (u32)p.K;
    const int nk = (int)((K + 31) >> 5);
    const int per = (nk + (int)gridDim.z - 1) / (int)gridDim.z;
    const int ks_begin = (int)blockIdx.z * per;
    const int ks_end = ks_begin + per < nk ? ks_begin + per : nk;

    // loading side: piece lp of rows lr, lr + 4, lr + 8, lr + 12 of the block, through buffer views (the whole left
    // operand; the right operand from the block's first row on) whose range check turns an offset of OOB into zeros
    const int lp = lane & 15, lr = lane >> 4;
    auto swizzle = [](int r) { return r ^ (((r >> 2) ^ (r >> 3)) & 1) << 3; };   // r, or r ^ 8 for rows 4 .. 11
    const u64 b_left = (u64)(p.N - n0) * K * 8u;
    const __amdgpu_buffer_rsrc_t rs_xa = make_rsrc(p.x_a, (u32)((u64)p.M * K * 8u)),
                                 rs_xb = make_rsrc(p.x_b, (u32)((u64)p.M * K * 8u)),
                                 rs_wa = make_rsrc(p.w_a + (u64)n0 * K, b_left > 0x7FFFFFFFull ? 0x7FFFFFFFu : (u32)b_left),
                                 rs_wb = make_rsrc(p.w_b + (u64)n0 * K, b_left > 0x7FFFFFFFull ? 0x7FFFFFFFu : (u32)b_left);
    u32 a_off[4], b_off[4];
    int st_off[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = 4 * j + lr;
        a_off[j] = (u32)(m0 + r < p.M ? m0 + r : p.M - 1) * K * 8u + 16u * lp;
        b_off[j] = (u32)(n0 + r < p.N ? r : p.N - 1 - n0) * K * 8u + 16u * lp;
        st_off[j] = r * 256 + ((lp ^ swizzle(r)) << 4);
    }
    // multiplying side: lane (r16, kg)
    const int r16 = lane & 15, kg = lane >> 4;
    char* const my_stage = &stage[wave][0][0];
    const char* const rd = my_stage + (kg >> 1) * 4096 + r16 * 256;   // x_a / x_b, and + 8192: w_a + w_b / w_a
    int rd_off[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) rd_off[i] = ((8 * (kg & 1) + i) ^ swizzle(r16)) << 4;

    constexpr int AJ = ROWS / 4, BJ = COLS / 4;   // loads of four rows each
    u4 rxa[AJ], rxb[AJ], rwa[BJ], rwb[BJ];
    // words 2 lp, 2 lp + 1 of slice ks of the four rows (K is even: the pair is inside or outside K as a whole)
    auto load = [&](int ks) {
        const u32 at = (32u * (u32)ks + 2u * (u32)lp < K ? 0u : OOB) + 256u * (u32)ks;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j < AJ) rxa[j] = __builtin_amdgcn_raw_buffer_load_b128(rs_xa, a_off[j] + at, 0, 0);
            if (j < AJ) rxb[j] = __builtin_amdgcn_raw_buffer_load_b128(rs_xb, a_off[j] + at, 0, 0);
            if (j < BJ) rwa[j] = __builtin_amdgcn_raw_buffer_load_b128(rs_wa, b_off[j] + at, 0, 0);
            if (j < BJ) rwb[j] = __builtin_amdgcn_raw_buffer_load_b128(rs_wb, b_off[j] + at, 0, 0);
        }
    };

    v4i acc[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) acc[s] = v4i{0, 0, 0, 0};
    int ks = ks_begin + wave;
    if (ks < ks_end) load(ks);
    while (ks < ks_end) {   // uniform over the wave
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j < AJ) *reinterpret_cast<u4*>(my_stage + st_off[j]) = rxa[j];
            if (j < AJ) *reinterpret_cast<u4*>(my_stage + 4096 + st_off[j]) = rxb[j];
            if (j < BJ) *reinterpret_cast<u4*>(my_stage + 8192 + st_off[j]) = add64x2(rwa[j], rwb[j]);
            if (j < BJ) *reinterpret_cast<u4*>(my_stage + 12288 + st_off[j]) = rwa[j];
        }
        const int next = ks + SMALL_WAVES;
        if (next < ks_end) load(next);
        __builtin_amdgcn_wave_barrier();   // (compiler only) the reads below follow the writes above
        u4 ra[8], rb[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            ra[i] = *reinterpret_cast<const u4*>(rd + rd_off[i]);
            rb[i] = *reinterpret_cast<const u4*>(rd + 8192 + rd_off[i]);
        }
        __builtin_amdgcn_wave_barrier();
        v4i ad[8], bd[8];
        split16(ra, ad);
        split16(rb, bd);
#pragma unroll
        for (int l = 0; l < 8; ++l)
#pragma unroll
            for (int m = 0; m + l < 8; ++m)
                acc[l + m] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ad[l], bd[m], acc[l + m], 0, 0, 0);
        ks = next;
    }
    // fold: sum_s sext(P_s) << 8s, P_4..P_7 only reach bits 32..63; lane (c, g) holds rows 4g .. 4g+3 of
    // column c of the block.  A wave leaves its sums where its words were staged.
    u64* const part = reinterpret_cast<u64*>(my_stage);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        u64 v = (u64)(int64_t)acc[0][i];
        v += (u64)(int64_t)acc[1][i] << 8;
        v += (u64)(int64_t)acc[2][i] << 16;
        v += (u64)(int64_t)acc[3][i] << 24;
        const u32 hi = (u32)acc[4][i] + ((u32)acc[5][i] << 8) + ((u32)acc[6][i] << 16) + ((u32)acc[7][i] << 24);
        v += (u64)hi << 32;
        part[(4 * kg + i) * 16 + r16] = v;
    }
    __syncthreads();
    if (tid < 256) {
        const int row = m0 + (tid >> 4), col = n0 + (tid & 15);
        if ((tid >> 4) < ROWS && (tid & 15) < COLS && row < p.M && col < p.N) {
            u64* dst = p.z + (u64)row * (u64)p.N + (u64)col;
            u64 v = 0;
#pragma unroll
            for (int k = 0; k < SMALL_WAVES; ++k) v += reinterpret_cast<const u64*>(&stage[k][0][0])[tid];
            if (gridDim.z > 1) atomicAdd(reinterpret_cast<unsigned long long*>(dst), (unsigned long long)v);
            else *dst = p.z_add ? *dst + v : v;
        }
    }
}

// ---- products whose right operand is stored transposed, [K, N] with N contiguous (gradients of a fully connected layer) --------
// A lane of the matrix instruction wants sixteen consecutive k of one column.  In this storage sixteen lanes on
// neighbouring pairs of columns read 256 contiguous bytes of every k, so the words go straight from memory to the lane that
// splits them: no LDS, no exchange.  The three terms are taken as (x_a + x_b)*w_a + x_a*w_b here: a lane then loads one share of the right
// operand, and the sum is formed on the left, which is split once per wave.

// Sixteen words of a column (the first or the second of a lane's pairs) -> eight digit registers
template <int SECOND>
__device__ __forceinline__ void split_column(const u4 (&v)[16], v4i (&d)[8]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        u32 lo[4], hi[4], dl[4], dh[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            lo[t] = SECOND ? v[4 * j + t].z : v[4 * j + t].x;
            hi[t] = SECOND ? v[4 * j + t].w : v[4 * j + t].y;
            recode(lo[t], hi[t]);
        }
        transpose4(lo[0], lo[1], lo[2], lo[3], dl);
        transpose4(hi[0], hi[1], hi[2], hi[3], dh);
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            d[l][j] = (int)dl[l];
            d[4 + l][j] = (int)dh[l];
        }
    }
}

// The right operand of one lane: a pair of columns of the share that its half-wave takes, words k = 32 ks + 16 (g & 1) + j,
// j = 0 .. 15.  Rows past K are replaced by the last one: the left operand's words there are zeros.
struct PairColumn {
    const u64* base;   // the pair in row 0
    __device__ __forceinline__ void load(u4 (&v)[16], int ks, int g, u32 K, u32 N) const {
        const u32 want = 32u * (u32)ks + 16u * (u32)(g & 1), row = want < K ? want : K - 1u;
        u32 last = K - 1u - row;
        asm volatile("" : "+v"(last));   // (the sixteen offsets are computed here and not kept in registers across a loop)
        const char* const p = reinterpret_cast<const char*>(base + (u64)row * N);
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const u32 r = (u32)j < last ? (u32)j : last;
            v[j] = *reinterpret_cast<const u4*>(p + (u64)(u32)__umul24(r, N * 8u));
        }
    }
};

// element i of the four that a lane holds of a block
__device__ __forceinline__ u64 fold_element(const v4i (&acc)[8], int i) {
    u64 v = (u64)(int64_t)acc[0][i];
    v += (u64)(int64_t)acc[1][i] << 8;
    v += (u64)(int64_t)acc[2][i] << 16;
    v += (u64)(int64_t)acc[3][i] << 24;
    const u32 hi = (u32)acc[4][i] + ((u32)acc[5][i] << 8) + ((u32)acc[6][i] << 16) + ((u32)acc[7][i] << 24);
    return v + ((u64)hi << 32);
}

__device__ __forceinline__ void multiply36(const v4i (&a)[8], const v4i (&b)[8], v4i (&acc)[8]) {
#pragma unroll
    for (int l = 0; l < 8; ++l)
#pragma unroll
        for (int m = 0; m + l < 8; ++m)
            acc[l + m] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[l], b[m], acc[l + m], 0, 0, 0);
}

// Both operands transposed and K <= 32, one slice: the weight gradient at batches of up to 32.  A wave splits 32 rows of the
// left operand once and walks along `per` blocks of 32 columns; nothing is shared between waves, so a block is one wave and
// short calls spread over all compute units (eight waves to a block: 7.9 us instead of 4.7 at 64 x 512 x 32, a compute unit's loads
// one after the other).  Block q of 16 rows holds rows 2 r + q, block c of 16 columns columns 2 r + c: a lane's pairs in memory.
// Bound: the vector ALU (split and fold, 690 instructions beside 144 matrix instructions) and, on long outputs, the loads' latency.
__global__ __launch_bounds__(64, 2) void share_gemm_outer_kernel(const GemmParams p, u32 runs, u32 per) {
    const int lane = threadIdx.x, r16 = lane & 15, g = lane >> 4;
    const bool low = g < 2;
    const u32 rows = blockIdx.x / runs, c0 = (blockIdx.x - rows * runs) * per * 32u;
    const u32 K = (u32)p.K, N = (u32)p.N, M = (u32)p.M, m0 = rows * 32u;
    if (m0 >= M || c0 >= N) return;
    const u32 blocks = (N - c0 + 31u) / 32u < per ? (N - c0 + 31u) / 32u : per;
    auto column = [&](u32 b) { const u32 n = c0 + 32u * b + 2u * (u32)r16; return n < N ? n : N - 2u; };   // (N is even)
    PairColumn right;
    v4i ad[2][8];
    u4 w[16];
    {
        const __amdgpu_buffer_rsrc_t rxa = make_rsrc(p.x_a, K * M * 8u), rxb = make_rsrc(p.x_b, K * M * 8u);
        const u32 m = m0 + 2u * (u32)r16 < M ? m0 + 2u * (u32)r16 : M - 2u, off = ((u32)(16 * (g & 1)) * M + m) * 8u;
        u4 x[16], y[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            x[j] = __builtin_amdgcn_raw_buffer_load_b128(rxa, off + (u32)j * M * 8u, 0, 0);
            y[j] = __builtin_amdgcn_raw_buffer_load_b128(rxb, low ? off + (u32)j * M * 8u : OOB, 0, 0);   // else zero
        }
        right.base = (low ? p.w_a : p.w_b) + column(0);
        right.load(w, 0, g, K, N);
#pragma unroll
        for (int j = 0; j < 16; ++j) x[j] = add64x2(x[j], y[j]);
        split_column<0>(x, ad[0]);
        split_column<1>(x, ad[1]);
    }
    const u64 z_left = (u64)(M - m0) * N * 8u;
    const __amdgpu_buffer_rsrc_t rz = make_rsrc(p.z + (u64)m0 * N, z_left > 0x7FFFFFFFull ? 0x7FFFFFFFu : (u32)z_left);
    for (u32 b = 0; b < blocks; ++b) {
        v4i bd[2][8];
        split_column<0>(w, bd[0]);
        split_column<1>(w, bd[1]);
        const u32 n = c0 + 32u * b + 2u * (u32)r16;
        if (b + 1 < blocks) {
            right.base = (low ? p.w_a : p.w_b) + column(b + 1);
            right.load(w, 0, g, K, N);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            u64 v[2][4];   // (one block's accumulators at a time: two do not fit beside the digits and the words on their way)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                v4i acc[8];
#pragma unroll
                for (int s = 0; s < 8; ++s) acc[s] = v4i{0, 0, 0, 0};
                multiply36(ad[q], bd[c], acc);
#pragma unroll
                for (int i = 0; i < 4; ++i) v[c][i] = fold_element(acc, i);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {   // rows past M lie outside the view, columns past N are sent there
                const u4 out = {(u32)v[0][i], (u32)(v[0][i] >> 32), (u32)v[1][i], (u32)(v[1][i] >> 32)};
                const u32 off = ((u32)(2 * (4 * g + i) + q) * N + n) * 8u;
                __builtin_amdgcn_raw_buffer_store_b128(out, rz, n < N ? off : OOB, 0, 0);
            }
        }
    }
}

// Few rows on the left, row-major: the input gradient at small batch.  A block owns 16 RB rows x 32 columns of z, its four waves
// (one per SIMD, 512 registers: the next slice's words arrive while this one is split and multiplied) share out the slices of K.
// The left operand crosses a wave-private LDS buffer as in share_gemm_small_kernel.  Bound: memory (the right operand, read once
// per 16 RB rows).  32 x 8192 x 512: 32.2 -> 22.3 us (67 MB of right operand, 13 us at 5 TB/s); with 16-column loads of 8 bytes
// and w_a read for both terms 24.5.
template <int RB>
__global__ __launch_bounds__(256, 1) void share_gemm_rows_t_kernel(const GemmParams p) {
    __shared__ __attribute__((aligned(16))) char stage[4][RB * 2][16 * 256];
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
    const bool low = g < 2;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = blockIdx.x * 32, m0 = blockIdx.y * 16 * RB;
    const u32 K = (u32)p.K, N = (u32)p.N;
    const int nk = (int)((K + 31) >> 5);
    const int lp = lane & 15, lr = lane >> 4;
    auto swizzle = [](int r) { return r ^ (((r >> 2) ^ (r >> 3)) & 1) << 3; };
    const __amdgpu_buffer_rsrc_t rs_xa = make_rsrc(p.x_a, (u32)((u64)p.M * K * 8u)), rs_xb = make_rsrc(p.x_b, (u32)((u64)p.M * K * 8u));
    u32 a_off[RB][4];
    int st_off[4], rd_off[8];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = 4 * j + lr;
#pragma unroll
        for (int q = 0; q < RB; ++q) a_off[q][j] = (u32)(m0 + 16 * q + r < p.M ? m0 + 16 * q + r : p.M - 1) * K * 8u + 16u * lp;
        st_off[j] = r * 256 + ((lp ^ swizzle(r)) << 4);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) rd_off[i] = (g >> 1) * 4096 + r16 * 256 + (((8 * (g & 1) + i) ^ swizzle(r16)) << 4);
    char* const my_stage = &stage[wave][0][0];

    u4 rx[RB][2][4];
    auto load_x = [&](int ks) {
        const u32 at = (32u * (u32)ks + 2u * (u32)lp < K ? 0u : OOB) + 256u * (u32)ks;
#pragma unroll
        for (int q = 0; q < RB; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                rx[q][0][j] = __builtin_amdgcn_raw_buffer_load_b128(rs_xa, a_off[q][j] + at, 0, 0);
                rx[q][1][j] = __builtin_amdgcn_raw_buffer_load_b128(rs_xb, a_off[q][j] + at, 0, 0);
            }
    };
    u4 w[16];
    const u32 pair = (u32)(n0 + 2 * r16 < p.N ? n0 + 2 * r16 : p.N - 2);   // (N is even)
    const PairColumn right = {(low ? p.w_a : p.w_b) + pair};
    v4i acc[RB][2][8];
#pragma unroll
    for (int q = 0; q < RB; ++q)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int s = 0; s < 8; ++s) acc[q][c][s] = v4i{0, 0, 0, 0};
    int ks = wave;
    if (ks < nk) {
        right.load(w, ks, g, K, N);
        load_x(ks);
    }
    while (ks < nk) {   // uniform over the wave
        const int next = ks + 4;   // past the end: nothing is read
        v4i ad[RB][8], bd[2][8];
        split_column<0>(w, bd[0]);
        split_column<1>(w, bd[1]);
        if (next < nk) right.load(w, next, g, K, N);
#pragma unroll
        for (int q = 0; q < RB; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                *reinterpret_cast<u4*>(my_stage + 8192 * q + st_off[j]) = add64x2(rx[q][0][j], rx[q][1][j]);
                *reinterpret_cast<u4*>(my_stage + 8192 * q + 4096 + st_off[j]) = rx[q][0][j];
            }
        if (next < nk) load_x(next);
        __builtin_amdgcn_wave_barrier();   // (compiler only) the reads below follow the writes above
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            u4 raw[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) raw[i] = *reinterpret_cast<const u4*>(my_stage + 8192 * q + rd_off[i]);
            split16(raw, ad[q]);
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int q = 0; q < RB; ++q) multiply36(ad[q], bd[c], acc[q][c]);
        ks = next;
    }
    // the waves' partial sums meet in LDS, [wave][row][32 columns]
    __syncthreads();
    u64* const part = reinterpret_cast<u64*>(&stage[0][0][0]);
#pragma unroll
    for (int q = 0; q < RB; ++q)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) part[(wave * 16 * RB + 16 * q + 4 * g + i) * 32 + 2 * r16 + c] = fold_element(acc[q][c], i);
    __syncthreads();
    for (int e = tid; e < 16 * RB * 32; e += 256) {
        const int row = m0 + e / 32, col = n0 + e % 32;
        if (row < p.M && col < p.N) {
            u64 v = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) v += part[k * 16 * RB * 32 + e];
            p.z[(u64)row * N + (u64)col] = v;
        }
    }
}

}  // namespace

// Row-major operands with 16-byte loads (K even, 16-byte aligned bases), few blocks of z, and a K whose
// slices, shared out over a block's waves, fit one fold.
bool share_gemm_small_applies(const GemmParams& p) {
    const int64_t nk = (p.K + 31) / 32;
    if (p.lda != p.K || nk > SMALL_MAX_SLICES) return false;
    if ((p.N + 15) / 16 > (1 << 20)) return false;   // grid size in threads stays below 2^32
    if (p.M <= SMALL_ONE_BLOCK_ROWS) return true;
    const int64_t tiles = ((int64_t)p.M + 15) / 16 * (((int64_t)p.N + 15) / 16);
    if (tiles * nk > SMALL_MAX_UNITS) return false;
    if (p.M <= SMALL_MANY_ROWS) return true;
    const int64_t rounds = (tiles + SMALL_ROUND_BLOCKS - 1) / SMALL_ROUND_BLOCKS;
    if (rounds == 1) return true;
    if (rounds == 2) return nk <= (p.z_add ? 11 : 13);
    return rounds == 3 && nk >= 2 && (nk <= 3 || !p.z_add);
}

hipError_t launch_share_gemm_small(const GemmParams& p, hipStream_t stream) {
    const int64_t tiles_m = (p.M + 15) / 16, tiles_n = (p.N + 15) / 16, tiles = tiles_m * tiles_n;
    const int nk = (p.K + 31) / 32;
    // K is split over blocks as well when the blocks of z alone would leave compute units idle, as long as a
    // wave keeps at least two slices
    int64_t ksplit = 1;
    if (tiles < SMALL_ROUND_BLOCKS) {
        ksplit = SMALL_ROUND_BLOCKS / tiles;
        const int64_t most = nk / (2 * SMALL_WAVES);
        if (ksplit > most) ksplit = most;
        if (ksplit < 1) ksplit = 1;
    }
    if (ksplit > 1 && !p.z_prezeroed && !p.z_add)
        if (hipError_t e = launch_zero_words(p.z, (size_t)p.M * (size_t)p.N, stream)) return e;
    auto launch = [&](auto kernel, int rows, int cols) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((p.N + cols - 1) / cols), (unsigned)((p.M + rows - 1) / rows), (unsigned)ksplit),
                           dim3(SMALL_WAVES * 64), 0, stream, p);
    };
    // Blocks of 8 rows and columns leave half of the matrix instruction's rows and columns to words that nobody stores, but a
    // compute unit's loads, which are what such a call waits for, are those of half as many rows: 32 x 512 x 512 7.3 -> 6.5 us,
    // 128 x 128 x 784 9.6 -> 8.8, 8 x 1000 x 512 7.3 -> 6.0 (of it 0.2 us by sums that meet without LDS atomics).
    const int64_t m8 = ((int64_t)p.M + 7) / 8, n8 = ((int64_t)p.N + 7) / 8;
    if (ksplit == 1 && m8 * n8 <= SMALL_ROUND_BLOCKS) launch(share_gemm_small_kernel<8, 8>, 8, 8);
    else if (ksplit == 1 && m8 * tiles_n <= SMALL_ROUND_BLOCKS) launch(share_gemm_small_kernel<8, 16>, 8, 16);
    else if (ksplit == 1 && tiles_m * n8 <= SMALL_ROUND_BLOCKS) launch(share_gemm_small_kernel<16, 8>, 16, 8);
    else launch(share_gemm_small_kernel<16, 16>, 16, 16);
    return hipGetLastError();
}

namespace {
bool pairs_aligned(const void* a, const void* b) { return (((uintptr_t)a | (uintptr_t)b) & 15) == 0; }
}  // namespace

// 697 shapes of M 10 .. 4096, N 32 .. 16384, K 1 .. 32 against share_gemm_kernel, whole calls: 0.61 - 0.83 of its time with at most
// one wave per SIMD (7.3 -> 4.6 us), 0.64 - 1.04 where the tiled kernel needs more than one round of its 128 x 64 tiles (512 x 8192 x 32 17.3 ->
// 14.1 us, 4096 x 4096 x 32 57 -> 49); in between the waves share a SIMD while the tiles still run in one round (1.02, 1.07 at worst).
bool share_gemm_outer_applies(const GemmParams& p) {
    if (p.K > 32 || p.z_add || p.N % 2 != 0 || p.M % 2 != 0 || p.N >= (1 << 21) || p.M >= (1 << 21)) return false;
    if (!pairs_aligned(p.w_a, p.w_b) || !pairs_aligned(p.x_a, p.x_b) || ((uintptr_t)p.z & 15) != 0) return false;
    const int64_t units = ((int64_t)p.M + 31) / 32 * (((int64_t)p.N + 31) / 32), tiles = ((int64_t)p.M + 127) / 128 * (((int64_t)p.N + 63) / 64);
    return units <= 1024 || tiles > 256;
}

hipError_t launch_share_gemm_outer(const GemmParams& p, hipStream_t stream) {
    const int64_t row_tiles = (p.M + (int64_t)31) / 32, cols = (p.N + (int64_t)31) / 32;
    int64_t per = (row_tiles * cols + 2047) / 2048;
    if (per > cols) per = cols;
    const int64_t runs = (cols + per - 1) / per, waves = row_tiles * runs;
    hipLaunchKernelGGL(share_gemm_outer_kernel, dim3((unsigned)waves), dim3(64), 0, stream, p, (u32)runs, (u32)per);
    return hipGetLastError();
}

// Modelled time in microseconds, or 0 where the kernel does not apply: turns of a wave times rounds of the chip, and the right
// operand once per group of rows (fitted over 692 shapes of M 2 .. 300, N 10 .. 16384, K 8 .. 8192, nine in ten within 8 %).
static double rows_t_us(const GemmParams& p) {
    const int64_t nk = (p.K + (int64_t)31) / 32;
    if (p.lda != p.K || p.z_add || p.M > 512 || nk > 511 * 4 || p.N % 2 != 0 || p.N >= (1 << 21) || !pairs_aligned(p.w_a, p.w_b)) return 0.0;
    const int64_t groups = p.M <= 16 ? 1 : (p.M + 31) / 32, blocks = (p.N + (int64_t)31) / 32 * groups;
    const double turns = (double)((nk + 3) / 4), rounds = (double)((blocks + 255) / 256);
    const double mb = 16.0e-6 * (double)groups * (double)p.N * (double)p.K;
    return p.M <= 16 ? 1.1 + rounds * (1.87 * turns + 1.28) + 0.080 * mb : 1.2 + rounds * (2.69 * turns + 2.27) + 0.083 * mb;
}

// Few rows against a transposed right operand: both kernels' modelled times, the tiled one's in the terms of its launcher (slices in
// rounds, rounds, megabytes of right operand; over the same 692 shapes nine in ten within 13 %).  With one block of rows the kernel must be
// modelled 14 % faster: of 1379 other shapes the 14 between that and 5 % took 1.0 of the tiled kernel's time, up to 1.10 (4 x 1766 x 576
// 12.4 -> 13.7 us), the 789 of up to 16 rows beyond it 18.0 ms -> 10.8, at most 0.94 each, the 576 of more rows
// 6.95 -> 5.24, one of them, by 5 % (30 x 13090 x 284 30.3 -> 31.7).
bool share_gemm_rows_t_pays(const GemmParams& p) {
    const double few = rows_t_us(p);
    if (few == 0.0) return false;
    const int64_t rows = (p.M + (int64_t)127) / 128, tiles = rows * ((p.N + (int64_t)63) / 64);
    const int nk = (p.K + 31) / 32, ks = choose_ksplit(tiles, nk);
    const double tiled = 2.42 * classic_cost(tiles, nk, ks) + (ks > 1 ? 0.4 : 0.0) +
                         1.92 * (double)((tiles * ks + ROUND_BLOCKS - 1) / ROUND_BLOCKS) +
                         0.124 * 16.0e-6 * (double)rows * (double)p.N * (double)p.K;
    return few < (p.M <= 16 ? 0.86 : 0.95) * tiled;
}

hipError_t launch_share_gemm_rows_t(const GemmParams& p, hipStream_t stream) {
    const dim3 grid((unsigned)((p.N + (int64_t)31) / 32), (unsigned)(p.M <= 16 ? 1 : (p.M + 31) / 32));
    if (p.M <= 16) hipLaunchKernelGGL((share_gemm_rows_t_kernel<1>), grid, dim3(256), 0, stream, p);
    else hipLaunchKernelGGL((share_gemm_rows_t_kernel<2>), grid, dim3(256), 0, stream, p);
    return hipGetLastError();
}

}  // namespace cg
