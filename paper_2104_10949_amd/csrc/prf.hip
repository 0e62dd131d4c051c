// Zero shares from an AES-128 PRF and the reshare step z_i + alpha_i
// (CryptGPU Sec. III-B "Protocol initialization", "Multiplication"; Sec. IV
// "Pseudorandom generators on the GPU": AES is the PRF).
//
// alpha_i[j] = F(k_i, j) - F(k_{i-1}, j) mod 2^64.  F(k, j) is AES-128 in counter
// mode: input block = (block index j >> 1 as 64-bit little-endian, nonce as 64-bit
// little-endian), output word = ciphertext bytes 0..7 (j even) or 8..15 (j odd) as
// a little-endian integer.  One thread encrypts one block under both keys and
// produces two consecutive words of alpha.
//
// AES rounds use the classic 32-bit table formulation of FIPS-197: the table
// T0[x] = (2 S[x], S[x], S[x], 3 S[x]); the other three columns of the MixColumns
// matrix are its byte rotations T1 = rotl8(T0), T2 = rotl16(T0), T3 = rotl24(T0).
// With all four in memory a column is four lookups and two three-input xors; the last round takes S-box bytes
// from the table that has them in the right place.  The LDS serves a wave's lookup in two halves of 32 lanes
// (the counters show two cycles each and no conflict), so 32 copies of an entry are enough: a row of 256 bytes
// holds entry x of T0 and of T1, 32 copies each, 64 KiB further on lie T2 and T3 (128 KiB per block of up to 16
// waves).  Lane i reads byte 65536 p + 256 x + 128 t + 4 (i % 32), always from its own bank, and the
// address is ONE byte permute of (state word, lane constant) with 128 t as the instruction's offset.  Round keys are
// expanded on the host and passed by value.
//
// Two rounds shared by 256 counters.  In counter mode 256 consecutive block indices differ
// in one input byte, so of the first round only one lookup differs between them, and of the second
// the four lookups that this one column feeds; the rest of both rounds is one constant
// per column and is computed once per run of 256 counters ("group") and stream (counter-mode
// caching, Bernstein and Schwabe, "New AES software speed records", 2008).  A block is
// 5 + 7*16 + 16 = 133 lookups instead of 160.
//
// Bound: the LDS (133 lookups of two cycles per wave, stream and block of AES, 87 of the 119 us of the measured call; by
// the counters busy 72 % of the cycles), with the vector ALU behind it (59 %; about 215 instructions per AES block, 128 of them lookup addresses; 290 with two tables,
// whose columns needed a rotation, 64 copies each).  Measured: the truncation step with both streams on
// 2^23 words 167 -> 126 us (of that 30 us by the shared rounds and short-call launch shape, 8 us by keys in
// registers and three-input xors), 128.5 -> 119.6 by four tables; a zero share of 2^15 words 8.7 -> 5.9 us (all compute units
// instead of 17, tables read from device memory and filled 16 bytes at a time, keys requested ahead of them).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "prf.h"

namespace cg {

namespace {

typedef uint32_t u32;
typedef uint64_t u64;

// ---- tables (built by the compiler) and key schedule (host) --------------------
// S-box via discrete logarithms to the generator 3 of GF(2^8)*, then the affine map.
struct AesTables {
    uint8_t sbox[256] = {};
    u32 t0[256] = {};
    constexpr AesTables() {
        uint8_t exp3[256] = {}, log3[256] = {};
        uint8_t x = 1;
        for (int i = 0; i < 255; ++i) {
            exp3[i] = x;
            log3[x] = (uint8_t)i;
            const uint8_t x2 = (uint8_t)((x << 1) ^ ((x & 0x80) ? 0x1B : 0));  // x * 2
            x = (uint8_t)(x2 ^ x);                                             // x * 3
        }
        for (int v = 0; v < 256; ++v) {
            const uint8_t inv = v ? exp3[(255 - log3[v]) % 255] : 0;
            uint8_t s = inv;
            s ^= (uint8_t)((inv << 1) | (inv >> 7));
            s ^= (uint8_t)((inv << 2) | (inv >> 6));
            s ^= (uint8_t)((inv << 3) | (inv >> 5));
            s ^= (uint8_t)((inv << 4) | (inv >> 4));
            s ^= 0x63;
            sbox[v] = s;
            const uint8_t s2 = (uint8_t)((s << 1) ^ ((s & 0x80) ? 0x1B : 0));
            const uint8_t s3 = (uint8_t)(s2 ^ s);
            t0[v] = (u32)s2 | ((u32)s << 8) | ((u32)s << 16) | ((u32)s3 << 24);
        }
    }
};

constexpr AesTables host_tables{};
__device__ const AesTables device_tables{};   // (device memory: passed as an argument it would be read over the host link)

// Round keys as 44 little-endian column words.
void expand_key(const uint8_t key[16], u32 rk[44]) {
    const uint8_t* sb = host_tables.sbox;
    for (int i = 0; i < 4; ++i)
        rk[i] = (u32)key[4 * i] | ((u32)key[4 * i + 1] << 8) | ((u32)key[4 * i + 2] << 16) | ((u32)key[4 * i + 3] << 24);
    u32 rcon = 1;
    for (int i = 4; i < 44; ++i) {
        u32 t = rk[i - 1];
        if ((i & 3) == 0) {
            t = (t >> 8) | (t << 24);  // RotWord on little-endian bytes
            t = (u32)sb[t & 0xFF] | ((u32)sb[(t >> 8) & 0xFF] << 8) | ((u32)sb[(t >> 16) & 0xFF] << 16) |
                ((u32)sb[t >> 24] << 24);
            t ^= rcon;
            rcon = (rcon << 1) ^ ((rcon & 0x80) ? 0x11B : 0);
        }
        rk[i] = rk[i - 4] ^ t;
    }
}

// Round keys of the streams of a launch: F(self, .), F(prev, .) if the launch forms alpha, then the mask stream.
struct PrfKeys {
    u32 rk[3][44];
};

// ---- device ------------------------------------------------------------------
constexpr int PRF_MAX_WAVES = 16;      // waves of a block; its tables leave room for one block per compute unit
constexpr int PRF_MAX_GROUPS = 512;    // groups of 256 counters whose constants a block can hold
constexpr int PRF_MAX_CHUNKS = 4 * (PRF_MAX_GROUPS - 1);   // chunks of 64 counters, the first anywhere in its group

// Entry of table T<TABLE> for byte B of a state word.  Byte 0 of the LDS address = 4 * (lane % 32) and byte 2 = which pair
// of tables come from the lane constant `lc` = 4 * (lane % 32) | 0x0100, byte 1 = the state byte; the second table of a
// pair lies 128 bytes on, which is the instruction's own offset.
// v_perm_b32(S0, S1, sel): selector values 0-3 pick bytes of S1, 4-7 bytes of S0, 0x0c gives 0.
template <int B, int TABLE>
__device__ __forceinline__ u32 lut(const char* __restrict__ tbl, u32 state, u32 lc) {
    constexpr u32 sel = 0x0C000000u | (TABLE >= 2 ? 0x00010000u : 0x000C0000u) | ((u32)(4 + B) << 8);
    return *reinterpret_cast<const u32*>(tbl + __builtin_amdgcn_perm(state, lc, sel) + (TABLE & 1) * 128);
}

__device__ __forceinline__ u32 rotl8(u32 v) { return __builtin_amdgcn_alignbit(v, v, 24); }

// a ^ b ^ c in one instruction (truth table 0x96); the compiler leaves two xors
__device__ __forceinline__ u32 xor3(u32 a, u32 b, u32 c) { return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96); }

// one output column of a full round: bytes 0..3 taken from state words a, b, c, d
__device__ __forceinline__ u32 column(const char* tbl, u32 lc, u32 a, u32 b, u32 c, u32 d, u32 rk) {
    return xor3(xor3(lut<0, 0>(tbl, a, lc), lut<1, 1>(tbl, b, lc), rk), lut<2, 2>(tbl, c, lc), lut<3, 3>(tbl, d, lc));
}

// one output word of the last round: S-box bytes of byte 0 of a, 1 of b, 2 of c, 3 of d, each from a table that has it in
// that place (T3 in bytes 0 and 1, T1 in bytes 2 and 3)
__device__ __forceinline__ u32 last_column(const char* tbl, u32 lc, u32 a, u32 b, u32 c, u32 d, u32 rk) {
    const u32 lo = __builtin_amdgcn_perm(lut<1, 3>(tbl, b, lc), lut<0, 3>(tbl, a, lc), 0x0C0C0500u);
    const u32 hi = __builtin_amdgcn_perm(lut<3, 1>(tbl, d, lc), lut<2, 1>(tbl, c, lc), 0x07020C0Cu);
    return xor3(lo, hi, rk);
}

// What a group of 256 counters shares of rounds 1 and 2: column 0 after round 1 without the lookup of the counter's
// byte 0, and the four columns after round 2 without the lookup that each takes from that column.
__device__ __forceinline__ void group_constants(const char* __restrict__ tbl, u32 lc, const u32* __restrict__ rk,
                                                u64 first_block, u64 nonce, u32& c1, uint4& c2) {
    const u32 s0 = (u32)first_block ^ rk[0], s1 = (u32)(first_block >> 32) ^ rk[1], s2 = (u32)nonce ^ rk[2],
              s3 = (u32)(nonce >> 32) ^ rk[3];
    c1 = xor3(lut<1, 1>(tbl, s1, lc), lut<2, 2>(tbl, s2, lc), lut<3, 3>(tbl, s3, lc)) ^ rk[4];
    const u32 n1 = column(tbl, lc, s1, s2, s3, s0, rk[5]);
    const u32 n2 = column(tbl, lc, s2, s3, s0, s1, rk[6]);
    const u32 n3 = column(tbl, lc, s3, s0, s1, s2, rk[7]);
    c2.x = xor3(lut<1, 1>(tbl, n1, lc), lut<2, 2>(tbl, n2, lc), lut<3, 3>(tbl, n3, lc)) ^ rk[8];
    c2.y = xor3(lut<0, 0>(tbl, n1, lc), lut<1, 1>(tbl, n2, lc), lut<2, 2>(tbl, n3, lc)) ^ rk[9];
    c2.z = xor3(lut<0, 0>(tbl, n2, lc), lut<1, 1>(tbl, n3, lc), lut<3, 3>(tbl, n1, lc)) ^ rk[10];
    c2.w = xor3(lut<0, 0>(tbl, n3, lc), lut<2, 2>(tbl, n1, lc), lut<3, 3>(tbl, n2, lc)) ^ rk[11];
}

// Round keys 3..10 of the streams of a launch and the byte that meets the counter's byte 0, fetched once per wave and
// kept in registers over all of its chunks: those of the first stream in scalar registers, those of the others in
// vector registers (96 keys do not fit the scalar file, and keys fetched as the rounds go are scalar loads whose
// out-of-order completion makes every wait for a lookup a wait for all of them).
template <int NS>
struct RoundKeys {
    u32 k0[NS], k[NS][8][4];
    __device__ __forceinline__ void load(const PrfKeys& keys) {
#pragma unroll
        for (int e = 0; e < NS; ++e) {
            k0[e] = keys.rk[e][0];
#pragma unroll
            for (int r = 0; r < 8; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    k[e][r][c] = keys.rk[e][12 + 4 * r + c];
                    if (e > 0) asm volatile("" : "+v"(k[e][r][c]));
                }
        }
    }
};

// NS independent encryptions side by side, round by round, of counter byte 0 = `byte0` in the group with constants
// c1, c2.
template <int NS>
__device__ __forceinline__ void aes_blocks(const char* __restrict__ tbl, u32 lc, const RoundKeys<NS>& key, u32 byte0,
                                           const u32 (&c1)[NS], const uint4 (&c2)[NS], u32 (&out)[NS][4]) {
    u32 s[NS][4];
#pragma unroll
    for (int e = 0; e < NS; ++e) {
        const u32 t = c1[e] ^ lut<0, 0>(tbl, byte0 ^ key.k0[e], lc);
        s[e][0] = c2[e].x ^ lut<0, 0>(tbl, t, lc);
        s[e][1] = c2[e].y ^ lut<3, 3>(tbl, t, lc);
        s[e][2] = c2[e].z ^ lut<2, 2>(tbl, t, lc);
        s[e][3] = c2[e].w ^ lut<1, 1>(tbl, t, lc);
    }
#pragma unroll
    for (int r = 0; r < 7; ++r) {
#pragma unroll
        for (int e = 0; e < NS; ++e) {
            const u32 n0 = column(tbl, lc, s[e][0], s[e][1], s[e][2], s[e][3], key.k[e][r][0]);
            const u32 n1 = column(tbl, lc, s[e][1], s[e][2], s[e][3], s[e][0], key.k[e][r][1]);
            const u32 n2 = column(tbl, lc, s[e][2], s[e][3], s[e][0], s[e][1], key.k[e][r][2]);
            const u32 n3 = column(tbl, lc, s[e][3], s[e][0], s[e][1], s[e][2], key.k[e][r][3]);
            s[e][0] = n0; s[e][1] = n1; s[e][2] = n2; s[e][3] = n3;
        }
    }
#pragma unroll
    for (int e = 0; e < NS; ++e) {
        out[e][0] = last_column(tbl, lc, s[e][0], s[e][1], s[e][2], s[e][3], key.k[e][7][0]);
        out[e][1] = last_column(tbl, lc, s[e][1], s[e][2], s[e][3], s[e][0], key.k[e][7][1]);
        out[e][2] = last_column(tbl, lc, s[e][2], s[e][3], s[e][0], s[e][1], key.k[e][7][2]);
        out[e][3] = last_column(tbl, lc, s[e][3], s[e][0], s[e][1], s[e][2], key.k[e][7][3]);
    }
}

// floor(v / 2^d) of v read as a two's-complement integer
__device__ __forceinline__ u64 asr64(u64 v, int d) { return (u64)((int64_t)v >> d); }

// For the words j = first .. first + n - 1 of the PRF streams:
//   out = asr64((z ? z : 0) + (msg ? msg : 0) + [ALPHA] (F(self, j) - F(prev, j)), d)  -/+  [MASK] F(mask, j)
// (alpha under `nonce`, the mask stream under `mask_nonce`; the mask is subtracted unless add_mask), or, for
// binary shares (xor_mode, ALPHA only):  out = (z ? z : 0) ^ F(self, j) ^ F(prev, j).
// One thread handles one AES block = two consecutive words of each stream; a wave takes chunks of 64 consecutive
// blocks, aligned to 64, of the workgroup's run of `per_wg` chunks.  `pairs`: first is even and z, msg and out are
// 16-byte aligned, so that a thread's two words are one access.
template <bool ALPHA, bool MASK>
__global__ __launch_bounds__(64 * PRF_MAX_WAVES) void prf_combine_kernel(const u64* z, const u64* msg,
                                                          u64* out, size_t n, u64 first, u64 nonce,
                                                          u64 mask_nonce, int d, bool add_mask, bool xor_mode,
                                                          bool pairs, u32 per_wg, const PrfKeys keys) {
    constexpr int NS = (ALPHA ? 2 : 0) + (MASK ? 1 : 0);
    __shared__ __attribute__((aligned(16))) u32 tables[2 * 256 * 64];  // (T0, T1) then (T2, T3), 32 copies of an entry
    __shared__ uint4 group_c2[NS][PRF_MAX_GROUPS];
    __shared__ u32 group_c1[NS][PRF_MAX_GROUPS];
    // The keys first: their way from the argument buffer passes while the tables are filled.
    RoundKeys<NS> key;
    key.load(keys);
    // 16 bytes, i.e. four of the 32 copies, of an entry of one table of either pair per thread and trip
#pragma unroll 4
    for (u32 i = threadIdx.x; i < 256 * 16; i += blockDim.x) {
        const u32 t = device_tables.t0[i >> 4], v0 = i & 8u ? rotl8(t) : t, v2 = (v0 << 16) | (v0 >> 16);
        reinterpret_cast<uint4*>(tables)[i] = uint4{v0, v0, v0, v0};
        reinterpret_cast<uint4*>(tables)[256 * 16 + i] = uint4{v2, v2, v2, v2};
    }
    __syncthreads();
    const char* tbl = reinterpret_cast<const char*>(tables);
    const u32 lane = threadIdx.x & 63;
    const u32 lc = ((lane & 31u) << 2) | 0x0100u;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), waves = blockDim.x >> 6;
    const u64 b_first = first >> 1, b_last = (first + n - 1) >> 1;  // n >= 1
    const u64 ch_last = b_last >> 6;
    const u64 ch0 = (b_first >> 6) + (u64)blockIdx.x * per_wg;      // the workgroup's chunks: ch0 .. ch_end - 1
    const u64 ch_end = ch0 + per_wg <= ch_last + 1 ? ch0 + per_wg : ch_last + 1;
    const u64 g0 = ch0 >> 2;
    if (ch0 < ch_end) {   // uniform over the workgroup
        const u32 groups = (u32)(((ch_end - 1) >> 2) - g0) + 1;     // at most PRF_MAX_GROUPS: see the launcher
        const u32 jobs = NS * ((groups + 63) / 64);
        for (u32 job = wave; job < jobs; job += waves) {
            const u32 e = job % NS, g = job / NS * 64 + lane;
            if (g < groups) {
                u32 c1;
                uint4 c2;
                group_constants(tbl, lc, keys.rk[e], (g0 + g) << 8, MASK && e == NS - 1 ? mask_nonce : nonce, c1, c2);
                group_c1[e][g] = c1;
                group_c2[e][g] = c2;
            }
        }
    }
    __syncthreads();
    for (u64 ch = ch0 + wave; ch < ch_end; ch += waves) {
        const u32 g = (u32)((ch >> 2) - g0);
        u32 c1[NS], ct[NS][4];
        uint4 c2[NS];
#pragma unroll
        for (int e = 0; e < NS; ++e) {
            c1[e] = group_c1[e][g];
            c2[e] = group_c2[e][g];
        }
        const u64 block = ch * 64 + lane;
        const u64 j0 = 2 * block, j1 = j0 + 1;  // word indices
        const bool in0 = j0 >= first && j0 - first < n, in1 = j1 >= first && j1 - first < n;
        // the operands are requested ahead of the encryption
        u64 z0 = 0, z1 = 0;
        if (pairs && in0 && in1) {
            const size_t j = j0 - first;
            if (z) {
                const ulonglong2 v = *reinterpret_cast<const ulonglong2*>(z + j);
                z0 = v.x; z1 = v.y;
            }
            if (msg) {
                const ulonglong2 v = *reinterpret_cast<const ulonglong2*>(msg + j);
                z0 += v.x; z1 += v.y;
            }
        } else {
            if (in0) z0 = (z ? z[j0 - first] : 0) + (msg ? msg[j0 - first] : 0);
            if (in1) z1 = (z ? z[j1 - first] : 0) + (msg ? msg[j1 - first] : 0);
        }
        aes_blocks<NS>(tbl, lc, key, ((u32)(ch & 3) << 6) | lane, c1, c2, ct);
        u64 w0 = 0, w1 = 0, r0 = 0, r1 = 0;
        if constexpr (ALPHA) {
            const u64 a0 = ((u64)ct[0][1] << 32) | ct[0][0], a1 = ((u64)ct[0][3] << 32) | ct[0][2];
            const u64 b0 = ((u64)ct[1][1] << 32) | ct[1][0], b1 = ((u64)ct[1][3] << 32) | ct[1][2];
            w0 = xor_mode ? a0 ^ b0 : a0 - b0;
            w1 = xor_mode ? a1 ^ b1 : a1 - b1;
        }
        if constexpr (MASK) {
            r0 = ((u64)ct[NS - 1][1] << 32) | ct[NS - 1][0];
            r1 = ((u64)ct[NS - 1][3] << 32) | ct[NS - 1][2];
            if (!add_mask) { r0 = 0 - r0; r1 = 0 - r1; }
        }
        const u64 v0 = xor_mode ? z0 ^ w0 : asr64(z0 + w0, d) + r0;
        const u64 v1 = xor_mode ? z1 ^ w1 : asr64(z1 + w1, d) + r1;
        if (pairs && in0 && in1) {
            *reinterpret_cast<ulonglong2*>(out + (j0 - first)) = ulonglong2{v0, v1};
        } else {
            if (in0) out[j0 - first] = v0;
            if (in1) out[j1 - first] = v1;
        }
    }
}

}  // namespace

// The tables take a compute unit's LDS, so one workgroup runs per compute unit.  Short calls spread over all of them,
// longer ones take a run of chunks each, always with 16 waves, which fill the tables together: 100 words (zero share)
// 5.67 us with eight waves, 5.53 with 16, 5.35 with the keys requested ahead of the tables (5.37 with one table fill of
// 16 waves and no shared rounds); from 2^21 words on all three are equal.  A run longer than a workgroup has room for is cut so that every compute unit gets the same number of
// equal runs: with full runs and a shorter rest, a call of 70 million words (257 .. 511 runs) took the time of two whole rounds, 1208 us
// where it now takes 648 (zero share).
PrfSplit prf_split(uint64_t first, size_t n) {
    constexpr u64 CUS = 256;
    const u64 chunks = (((first + n - 1) >> 1) >> 6) - ((first >> 1) >> 6) + 1;
    const u64 per_cu = (chunks + CUS - 1) / CUS;
    const u64 rounds = (per_cu + PRF_MAX_CHUNKS - 1) / PRF_MAX_CHUNKS;
    PrfSplit s;
    s.waves = PRF_MAX_WAVES;
    s.per_wg = (u32)((chunks + CUS * rounds - 1) / (CUS * rounds));
    s.blocks = (chunks + s.per_wg - 1) / s.per_wg;
    return s;
}

hipError_t launch_prf_combine(const uint64_t* z, const uint64_t* msg, uint64_t* out, size_t n,
                              const uint8_t* key_self, const uint8_t* key_prev, uint64_t nonce, uint64_t first, int d,
                              const uint8_t* key_mask, uint64_t mask_nonce, bool add_mask, hipStream_t stream,
                              bool xor_mode) {
    if (n == 0) return hipSuccess;
    const bool alpha = key_self && key_prev, mask = key_mask != nullptr;
    if (!alpha && !mask) return hipErrorInvalidValue;
    if (xor_mode && (mask || msg || d != 0)) return hipErrorInvalidValue;
    PrfKeys keys = {};
    if (alpha) {
        expand_key(key_self, keys.rk[0]);
        expand_key(key_prev, keys.rk[1]);
    }
    if (mask) expand_key(key_mask, keys.rk[alpha ? 2 : 0]);
    const uintptr_t bases = (uintptr_t)z | (uintptr_t)msg | (uintptr_t)out;
    const bool pairs = first % 2 == 0 && bases % 16 == 0;
    const PrfSplit split = prf_split(first, n);
    const dim3 g((unsigned)split.blocks), b(64 * split.waves);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, g, b, 0, stream, z, msg, out, n, (u64)first, (u64)nonce, (u64)mask_nonce, d, add_mask,
                           xor_mode, pairs, split.per_wg, keys);
    };
    if (alpha && mask) launch(prf_combine_kernel<true, true>);
    else if (alpha) launch(prf_combine_kernel<true, false>);
    else launch(prf_combine_kernel<false, true>);
    return hipGetLastError();
}

hipError_t launch_zero_share(const uint64_t* z, uint64_t* out, size_t n, const uint8_t key_self[16],
                             const uint8_t key_prev[16], uint64_t nonce, uint64_t first, hipStream_t stream) {
    return launch_prf_combine(z, nullptr, out, n, key_self, key_prev, nonce, first, 0, nullptr, 0, false, stream, false);
}

}  // namespace cg
