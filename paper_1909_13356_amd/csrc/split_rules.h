// Rules on counts alone, without HIP types: how work lists are cut.
#pragma once
#include <cstdint>

#ifdef __HIPCC__
#define LSS_RULE __host__ __device__ inline
#else
#define LSS_RULE inline
#endif

namespace lss {

// The M2L plan holds pair indices in 32 bits (tiles, blocks, each box's pairs);
// a longer list is run class by class, whose segments are 64-bit.
inline bool m2l_plan_holds(int64_t npairs) { return npairs <= INT32_MAX; }

// Pieces of the node range (chunks of `tile` nodes) for a direct sum of
// `tiles` tiles of `tile` targets.  1024 tiles of 256 targets fill the 256 CUs
// four deep; below 640 the last round of workgroups leaves CUs idle (600 tiles:
// up to 3 on a CU where the average is 2.3), so the nodes are split until up to
// 2048 workgroups run.  Targets times pieces stay below 2^19, so the partial
// sums (64 bytes per target and piece) and the buffers of n targets fit the 48
// MiB of the allocation-free entry point at every n.
//   whole: every tile walks all the chunks (one mesh).  A piece has as many as
// the rounding up of the average gives, and there are no more pieces than that
// leaves with any (144 chunks in up to 128 pieces: 72 of two; mixed, 4096
// targets on 36 864 nodes: 0.267 -> 0.225 ms).  In a batch a tile walks its own
// meshes, cut by its own average, and the last pieces of a short range are
// empty: fewer pieces would make the others longer (FP64, seven meshes with 300
// to 3000 targets each 1 to 3% slower).
inline int direct_pieces(int64_t tiles, int64_t chunks, int tile, bool whole) {
    const int64_t full = (int64_t)2048 * (256 / tile);
    if (tiles >= full * 5 / 16) return 1;
    int64_t most = full / tiles < chunks ? full / tiles : chunks;
    if (most > 1024) most = 1024;
    if (!whole) return (int)most;
    const int64_t per = (chunks + most - 1) / most;
    return (int)((chunks + per - 1) / per);
}

// Targets times pieces that a context allocates for on a call of n targets: what
// the call needs while every chunk is a piece, else the most that any call can
// need.  It does not fall as n grows (what a call needs does: 104 000 targets in
// five pieces need more than 110 000 in four), so that a call of fewer targets
// allocates nothing.
inline int64_t direct_partials_kept(int64_t n, int64_t chunks, int tile) {
    const int64_t full = (int64_t)2048 * (256 / tile), tiles = (n + tile - 1) / tile;
    const int64_t most = chunks < 1024 ? chunks : 1024;
    if (most <= 1 || tiles >= full * 5 / 16) return 0;
    return full / tiles >= most ? n * most : (int64_t)1 << 19;
}

// Piece k of the nodes [lo, hi), in whole chunks
LSS_RULE void piece_range(int tile, int64_t k, int64_t pieces, int64_t &lo, int64_t &hi) {
    const int64_t chunks = (hi - lo + tile - 1) / tile;
    const int64_t per = (chunks + pieces - 1) / pieces * tile;
    const int64_t a = lo + k * per;
    lo = a < hi ? a : hi;
    hi = lo + per < hi ? lo + per : hi;
}

}  // namespace lss
