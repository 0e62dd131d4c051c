// Internal interface of the residue route (share_gemm_rns.hip): one party's product through residues modulo
// 18 or 19 pairwise coprime numbers of eight bits.
#ifndef CG_SHARE_GEMM_RNS_H
#define CG_SHARE_GEMM_RNS_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "share_gemm.h"

namespace cg {

// Longest contraction, in words, for which the exact product stays within the range of the first 18 moduli, and of
// all 19 (there the bound is the 32-bit accumulator: 2 * K products of at most 2^14).
constexpr int64_t RNS_K_18 = 5500;
constexpr int64_t RNS_K_MAX = 65000;

// The product of some of the moduli on square tiles of one size.
struct RnsPart {
    int tiles_m, tiles_n;
    int first, count;                        // moduli first .. first + count - 1
    FastDiv div_tiles, div_group;
};

struct RnsParams {
    const uint64_t *x_a, *x_b, *w_a, *w_b;   // shares: left rows of `words` words, right rows of taps * words words
    uint64_t* z;                             // [M, N] row-major
    char *xp, *wp, *rp;                      // residues of the left operand, of the right one, of the result
    uint64_t x_plane, w_plane, r_plane;      // bytes per modulus
    int M, N;
    int words, slices;                       // words of a row per tap, and the 64-word slices they take
    int x_rows;                              // rows of the left operand (pixels); row x_rows of a plane is zero
    int conv;                                // the left operand's rows are gathered tap by tap
    int flip;                                // the right operand is stored [words, taps in reverse, N] (a filter, for its input gradient)
    int H, W, Ho, Wo, kh, kw, sh, sw, ph, pw;
    int nmod;
    RnsPart large, small;                    // which moduli run on tiles of 256 and which on tiles of 128
    int tile;                                // the size that would be taken for all moduli, were it one (256 or 128)
    int by_rounds;                           // the XCDs work on one modulus at a time
    int blocks_n;                            // 16 x 16 blocks of the result's planes along N
    double product_us;                       // modelled time of the product with that size for all moduli
    FastDiv div_slices, div_taps, div_n, div_howo, div_wo, div_blocks_n;
};

// Fills every size of p that follows from M, N, words, x_rows and the window; false where the route does not apply
// (an operand's plane beyond a buffer view, K beyond RNS_K_MAX).
bool rns_plan(RnsParams* p);
// Bytes of scratch memory: xp, wp and rp one after the other, each from a multiple of 256 on.
uint64_t rns_workspace_bytes(const RnsParams& p);
// Can a planned call run in this much memory?  Moduli on the large tile pad the result's planes to multiples of 256; a caller who
// brings what the small tile alone takes, where that is the better one of both, gets all moduli on it.
bool rns_fit(RnsParams* p, uint64_t bytes);
hipError_t launch_share_gemm_rns(RnsParams p, void* workspace, hipStream_t stream);

}  // namespace cg
#endif
