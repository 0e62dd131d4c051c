// How the launcher of the tiled kernel (share_gemm.hip) shares the tiles and K slices of a product out over the chip.  Host code without
// a call of the runtime: the tests ask it which distribution a shape takes.
#ifndef CG_SHARE_GEMM_SPLIT_H
#define CG_SHARE_GEMM_SPLIT_H

#include "share_gemm.h"

namespace cg {

// Blocks that run at one time: a block's LDS leaves room for one block per compute unit.
constexpr int ROUND_BLOCKS = 256;
// A K range of a split holds at least this many slices.
constexpr int SPLIT_MIN_SLICES = 2;
// Cost of the fixed part of a block (prologue, fold of the accumulators into z), in
// units of one K slice of the main loop, with a plain store and with atomic adds.
constexpr double SPLIT_COST_PLAIN = 1.0, SPLIT_COST_ATOMIC = 2.0;
// The streamed distribution must beat the classic one by this factor of modelled time to be used, by a little more where the
// right operand comes in 8-byte loads: the model has the fold of a run's second tile but not its prologue, which waits longer for those
// (1000 x 777 x 1531, 0.858: 95 us streamed, 88 classic; of 700 odd products none is more than 2 % slower than with 8-byte loads on both
// sides and no streaming, and all together take 0.885 of the time).
constexpr double STREAM_MARGIN = 0.88, STREAM_MARGIN_SCALAR = 0.84;
// A last round that is at most half full shares its tiles out over all compute units where that shortens it by this many slices
// (a launch that clears the tiles and the atomic adds cost about two).
constexpr int TAIL_MIN_SAVING = 3;
// Several rounds of unsplit tiles of at most this many slices are run as one round of blocks that
// each walk through whole tiles.
constexpr int PERSIST_MAX_SLICES = 32;

inline int choose_ksplit(int64_t tiles, int nk) {
    // A block's 160 KB of LDS leaves room for one block per compute unit, so a grid runs
    // in rounds of 256 blocks and the last round costs as much as a full one.  Splitting
    // K makes the blocks shorter, which fills the chip when the tiles alone cannot and
    // shrinks the idle part of the last round otherwise.  The split count with the least
    // modelled time wins: rounds * (slices per block + fixed cost per block).
    const int units = ROUND_BLOCKS;
    int64_t max_split = 8 * units / tiles;  // at most eight rounds' worth of blocks
    if (max_split > nk / SPLIT_MIN_SLICES) max_split = nk / SPLIT_MIN_SLICES;
    int best = 1;
    double best_cost = 0;
    for (int64_t ks = 1; ks <= (max_split < 1 ? 1 : max_split); ++ks) {
        const int64_t per = (nk + ks - 1) / ks;
        const int64_t eff = (nk + per - 1) / per;  // no empty splits
        if (eff != ks) continue;
        const int64_t rounds = (tiles * eff + units - 1) / units;
        const double cost = (double)rounds * ((double)per + (eff > 1 ? SPLIT_COST_ATOMIC : SPLIT_COST_PLAIN));
        if (ks == 1 || cost < best_cost * 0.97) {  // a split must pay for itself by a margin
            best = (int)eff;
            best_cost = cost;
        }
    }
    return best;
}

// Modelled time of the classic distribution with `ks` splits, in K slices (see choose_ksplit).
inline double classic_cost(int64_t tiles, int nk, int ks) {
    const int64_t per = (nk + ks - 1) / ks;
    const int64_t rounds = (tiles * ks + ROUND_BLOCKS - 1) / ROUND_BLOCKS;
    return (double)rounds * ((double)per + (ks > 1 ? SPLIT_COST_ATOMIC : SPLIT_COST_PLAIN));
}

// The streamed distribution is compiled for the address generators of the large layers only.
template <int AMODE, int BMODE>
struct CanStream {
    static constexpr bool value = (AMODE == A_LINEAR_VEC && BMODE == B_VEC) || (AMODE == A_LINEAR_SCALAR && BMODE == B_SCALAR) ||
                                  (AMODE == A_CONV_C32 && BMODE == B_VEC) ||
                                  (AMODE == A_CONV_C32 && BMODE == B_FLIP_C32) || (AMODE == A_TRANS && BMODE == B_PATCH_T) ||
                                  (AMODE == A_PATCH_T && BMODE == B_TRANS);
};

// The weight gradient's classic instantiation spills registers inside the loop (its streamed one does not,
// and is 7 % faster on the same ranges over the VGG-shaped layers): only the streamed one is built.  The input
// gradient keeps both: its unsplit tiles gain more from the classic order's neighbouring tiles per XCD.
template <int AMODE, int BMODE>
struct StreamOnly {
    static constexpr bool value = (AMODE == A_TRANS && BMODE == B_PATCH_T) || (AMODE == A_PATCH_T && BMODE == B_TRANS);
};

// The split tail is compiled where a product of a few slices per tile and no streamed instantiation is ordinary work: general gathers
// (first layers) and the gradients of fully connected layers.  An instantiation of its own: the selects that find a block's part
// cost the others 0.3 - 0.5 us a call.  7x7 stem on 224 x 224 x 3, batch 8, 784 tiles of five slices: 87.5 -> 80 us; weight gradient
// 4200 x 512 x 256, 264 tiles of eight: 62 -> 44.
template <int AMODE, int BMODE>
struct CanTail {
    static constexpr bool value = AMODE == A_CONV_GEN && BMODE != B_FLIP_GEN;
    static_assert(!value || !CanStream<AMODE, BMODE>::value, "a streamed instantiation spreads the slices itself");
};
template <>
struct CanTail<A_TRANS, B_TRANS> {
    static constexpr bool value = true;
};

// Split tail: the tiles from `first` on (launch order) are those of a last round that would be partly empty; each is shared by several
// blocks of `per` slices, which add into cleared elements.  An argument of its own kernels: as fields of GemmParams these 24 bytes took
// the arguments of every other kernel into a seventh line of 64 bytes, 0.2 us a call.
struct TailSplit {
    int first, tiles, per;   // (none: tiles 0)
    FastDiv div;             // tiles
};

struct WorkSplit {
    int ksplit;              // K ranges of a tile
    int64_t stream_per;      // (tile, slice) units per block of the streamed distribution, 0: classic
    TailSplit tail;
    unsigned grid;           // blocks
};

template <int AMODE, int BMODE>
WorkSplit split_work(int64_t tiles, int nk) {
    WorkSplit q = {};
    q.ksplit = choose_ksplit(tiles, nk);
    q.grid = (unsigned)(tiles * q.ksplit);
    // Streamed distribution: one block per compute unit, each taking an equal run of (tile, slice)
    // units.  A block pays the fixed cost once per tile its run touches (about per/nk + 1 of them).
    // Worth it when the classic grid leaves a round partly empty.
    const int64_t units = tiles * nk;
    if (CanStream<AMODE, BMODE>::value && units >= 3 * ROUND_BLOCKS && units < ((int64_t)1 << 40)) {
        const int64_t per = (units + ROUND_BLOCKS - 1) / ROUND_BLOCKS;
        const double streamed = (double)per + SPLIT_COST_ATOMIC * ((double)per / nk + 1.0);
        constexpr double margin = BMODE == B_SCALAR ? STREAM_MARGIN_SCALAR : STREAM_MARGIN;
        if (streamed < margin * classic_cost(tiles, nk, q.ksplit)) {
            q.stream_per = per;
            q.ksplit = 2;  // any value above 1: the folds add atomically into a zero-filled z
            q.grid = (unsigned)((units + per - 1) / per);
        }
    }
    // Whole tiles streamed: when the classic grid needs several rounds of unsplit tiles with a short K, one
    // block per compute unit walks through an equal run of whole tiles instead.  The kernel's pipeline then
    // runs on from tile to tile (no prologue, no block launch in between) and every tile is still stored
    // plainly.  Measured: 3-9 % on layers of up to 16 slices; with a long K the fixed part of a tile does not
    // matter and the classic order, which keeps the tiles an XCD runs at one time next to each other, is
    // 1-2 % faster.
    // Row-major left operands only: a patch gather re-reads the rows of neighbouring tiles, which hit in L2
    // when the neighbours run at the same time and miss when one block takes them one after the other
    // (measured on the 3x3 layers of the VGG-shaped step: twice the memory reads for 1-3 % of time).
    if (CanStream<AMODE, BMODE>::value && (AMODE == A_LINEAR_VEC || AMODE == A_LINEAR_SCALAR) && q.stream_per == 0 && q.ksplit == 1 &&
        tiles > ROUND_BLOCKS && nk <= PERSIST_MAX_SLICES) {
        const int64_t tiles_per_block = (tiles + ROUND_BLOCKS - 1) / ROUND_BLOCKS;
        q.stream_per = tiles_per_block * nk;
        q.grid = (unsigned)((tiles + tiles_per_block - 1) / tiles_per_block);
    }
    // The weight gradient runs the streamed kernel also where the classic distribution is the better one: a
    // run of one split's slices is that distribution, tile after tile instead of split after split.
    if (StreamOnly<AMODE, BMODE>::value && q.stream_per == 0) {
        q.stream_per = (nk + q.ksplit - 1) / q.ksplit;
        q.grid = (unsigned)((units + q.stream_per - 1) / q.stream_per);
    }
    // Split tail: several rounds of unsplit tiles whose last one is at most half full
    const int64_t tail = tiles % ROUND_BLOCKS;
    if (CanTail<AMODE, BMODE>::value && q.stream_per == 0 && q.ksplit == 1 && tiles > ROUND_BLOCKS && tail > 0 && tail <= ROUND_BLOCKS / 2) {
        int64_t parts = ROUND_BLOCKS / tail < nk ? ROUND_BLOCKS / tail : nk;
        const int64_t per = (nk + parts - 1) / parts;
        parts = (nk + per - 1) / per;
        if (nk - per >= TAIL_MIN_SAVING) {
            q.tail = TailSplit{(int)(tiles - tail), (int)tail, (int)per, make_fast_div((uint32_t)tail)};
            q.grid = (unsigned)(q.tail.first + tail * parts);
        }
    }
    return q;
}

}  // namespace cg
#endif
