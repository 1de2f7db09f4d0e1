// How a GEMM is cut into workgroups: the host's side of gemm.hip, free of device code so that the size queries, the
// plan queries and a host-only build share it.
#pragma once
#include <stddef.h>

namespace ob {

constexpr int KSTEP = 64;        // k per "K step", the unit the host's plan counts and slices in (two ring slots)
// contractions at least this long deal their patches round-robin to the XCDs (measured: shorter ones
// lose up to 1.8 %, longer ones gain 2.4 - 3.5 %)
constexpr int INTERLEAVE_MIN_K = 8192;

// The kind of tile, and which tiles have their contraction split.
// 256 x 256 | 128 x 128, two to a CU | 128 x 128 over a ring of eight slots | 64 x 64, eight slots, two to a CU | 192 x 256
enum TileKind { BIG = 0, SMALL = 1, DEEP = 2, FINE = 3, MID = 4 };
constexpr int tile_rows(TileKind kind) { return kind == BIG ? 256 : kind == MID ? 192 : kind == FINE ? 64 : 128; }
constexpr int tile_cols(TileKind kind) { return kind == MID ? 256 : tile_rows(kind); }
struct Plan {
    TileKind kind;
    int n_full, n_tail, splits, k_chunk;   // splits == 1: every tile whole
    size_t part_bytes() const { return splits > 1 ? (size_t)splits * n_tail * tile_rows(kind) * tile_cols(kind) * 4 : 0; }
};
constexpr int GEMM_GROUP_MAX = 4;
struct RowCut {
    int m;              // rows of the first launch; 0: one launch
    Plan head, rest;    // m == 0: rest is the plan of the whole
};

// compute units of the current device (256 when no device answers)
int compute_units();
// the tiles of one kind that cover M x N
int tiles_of(TileKind kind, int M, int N);
// bytes of slice sums that a GEMM may fill
size_t scratch_bytes(int M, int N, int K);
// the launches of a GEMM; layout 0 "NT", 1 "NN", 2 "TN"; `scratch`: bytes for slice sums
RowCut make_row_cut(int layout, int M, int N, int K, size_t scratch);
// GEMMs with an activation in the epilogue: layouts of gemm_any() beyond the three (internal).  Whether such a launch is taken instead of two, and its
// plan; `scratch`: the GEMM alone would have room for slice sums
enum { GEMM_NT_GELU = 3, GEMM_NN_GELU_BWD = 4, GEMM_NN_SWIGLU_BWD = 5 };
bool gemm_act_fuses(int layout, int M, int N, int K, bool scratch, Plan *plan = nullptr);
// rows of column sums that the last two leave: two per row of tiles
inline int gemm_act_colsums(const Plan &p, int M) { return 2 * ((M + tile_rows(p.kind) - 1) / tile_rows(p.kind)); }
// the same for a group of up to GEMM_GROUP_MAX "TN" GEMMs over one K: true: one launch, p; false: one by one.  has_ws: there is scratch, of ws_bytes
bool make_group_plan(int count, const int *M, const int *N, int K, bool has_ws, size_t ws_bytes, Plan &p);

}  // namespace ob
