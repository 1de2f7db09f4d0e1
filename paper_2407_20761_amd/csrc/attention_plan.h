// Which workgroup of an attention launch does which tile, and in which shape dK / dV runs: the host's side of
// attention.hip, free of device code so that the plan query and a host-only build share it.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/omnibal.h"

namespace ob {

constexpr int ST = 64;   // rows of a streamed tile

// Order of the tiles: heaviest first.  The work of a tile is the number of streamed tiles it walks;
// in a causal batch that differs by an order of magnitude between the first and the last tile of a
// long segment, and a launch that hands out the tiles segment by segment ends with a few workgroups
// on the heaviest tiles of the last segment while the rest of the chip idles (simulated on the
// benchmark's batches: 20 % of the forward's and 40 % of the dK/dV kernel's duration).  The host
// sorts the tiles by work (ties: natural order) and passes the order as a kernel argument:
// entry = segment << 16 | unit in segment.  A unit is one tile, or, where the 64-row tiles of dK / dV are more than the
// table holds, 2 or 4 consecutive ones (to 114688 and 229376 tokens): its workgroups have consecutive places in the
// launch, those past the segment's end nothing to do.  (dK / dV of 80000 tokens in 76 segments, 16 / 4 heads of 64: 1235 us
// in natural order, 1109 in units of two; of 70000 in 70, 2 / 1 heads of 128: 459 and 313.)  n == 0 (more units than the
// table holds, or a segment or unit number beyond 16 bits): natural order, found by find_tile.
struct TileOrder {
    static constexpr int CAP = 896;
    int n, unit_log2;
    uint32_t e[CAP];
};
// tile in its segment of place `rank` of the launch, e = ord.e[rank >> ord.unit_log2]
__host__ __device__ __forceinline__ int tile_of_rank(const TileOrder &ord, uint32_t e, int rank) {
    return (int)((e & 0xFFFFu) << ord.unit_log2) | (rank & ((1 << ord.unit_log2) - 1));
}

// shapes of dK / dV: pairs of 32 key rows, query rows of a streamed tile, threads.  Heads of 64: two pairs, two pairs with tiles of 32,
// six pairs; heads of 128: four pairs, two as 32 x 32 blocks on eight waves, two pairs.  Shape 2 is bidirectional:
// causal, two pairs were nowhere the best of the three (one segment of 64, 8 heads: 9.8 us, four pairs 9.5, blocks 10.0; of 128 11.4, 13.9, 11.4).
constexpr int dkv_np(int d, int shape) { return d == 64 && shape == 2 ? 6 : d == 128 && shape == 0 ? 4 : 2; }
constexpr int dkv_sr(int d, int shape) { return d == 64 && shape == 1 ? 32 : 64; }
constexpr int dkv_threads(int d, int shape) { return d == 128 && shape == 1 ? 512 : 128 * dkv_np(d, shape); }

// Consecutive query tiles that one descriptor of a dK / dV wave serves: a lane's offset advances by sr rows of ld2 bytes per tile and
// has 32 bits, in which `run` whole tiles of rows have to fit; a stride that they do not fit at gets a descriptor per tile.
constexpr int DKV_RUN = 64;
__host__ __device__ constexpr int dkv_run(uint32_t ld2, int sr) { return ld2 <= UINT32_MAX / (uint32_t)(DKV_RUN * sr) ? DKV_RUN : 1; }
// Whether the rows of one tile fit at all (64 rows of 67 MB do not).  Where not, a piece of it, 1 KB (8 rows of a head of 64, 4 of 128), is asked
// for by itself at the lanes' offsets from its own first row: those of the tile, of which 32 bits are kept, less that row's.
__host__ __device__ constexpr bool dkv_tile_fits(uint32_t ld2, int sr) { return ld2 <= UINT32_MAX / (uint32_t)sr; }
__host__ __device__ constexpr uint32_t dkv_piece_offset(uint32_t voff, uint32_t row, uint32_t ld2) { return voff - row * ld2; }

// the order of a launch; returns its places (workgroups per head): as many as tiles, or whole units of them
int make_order(const ob_segments *seg, int tile_rows, bool causal, bool kv_side, TileOrder &ord);
int dkv_shape(const ob_segments *seg, int nkv, int group, int d, bool causal);

}  // namespace ob
