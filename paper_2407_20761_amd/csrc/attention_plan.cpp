// Order of work and launch shapes of the attention kernels.
#include "attention_plan.h"

#include <algorithm>
#include <cmath>

#include "gemm_plan.h"
#include "ob_internal.h"

namespace ob {

namespace {

int count_tiles(const ob_segments *seg, int tile_rows) {
    long n = 0;
    for (int j = 0; j < seg->n_seg; ++j)
        n += (seg->cu_host[j + 1] - seg->cu_host[j] + tile_rows - 1) / tile_rows;
    return (int)n;
}

}  // namespace

// Order of work of a launch whose workgroups own `tile_rows` rows of a segment and stream 64-row
// tiles of the other side: descending number of streamed tiles, ties in natural order.  `kv_side`:
// the workgroup owns key rows and streams query tiles (from its diagonal on when causal); otherwise
// it owns query rows and streams key tiles (up to its diagonal when causal).  A unit counts as its first
// tile, on the key side the heaviest of them.  No heap memory.
int make_order(const ob_segments *seg, int tile_rows, bool causal, bool kv_side, TileOrder &ord) {
    ord.n = ord.unit_log2 = 0;
    const int n_tiles = count_tiles(seg, tile_rows), max_log2 = kv_side && tile_rows == 64 ? 2 : 0;
    int log2 = 0, n_units = n_tiles;
    while (n_units > TileOrder::CAP && log2 < max_log2) n_units = count_tiles(seg, tile_rows << ++log2);
    if (n_units > TileOrder::CAP || seg->n_seg > 0xFFFF) return n_tiles;
    const int unit_rows = tile_rows << log2;
    uint64_t key[TileOrder::CAP];
    int n = 0;
    for (int j = 0; j < seg->n_seg; ++j) {
        const int a = seg->cu_host[j], len = seg->cu_host[j + 1] - a;
        const int nt = (len + unit_rows - 1) / unit_rows;
        if (nt > 0xFFFF) return n_tiles;
        for (int t = 0; t < nt; ++t) {
            int rows = len;                                            // streamed rows
            if (causal && kv_side) rows = len - (t * unit_rows) / ST * ST;
            else if (causal) rows = std::min(len, (t + 1) * unit_rows);
            const uint32_t w = (uint32_t)((rows + ST - 1) / ST);
            // ascending sort of (~work, natural index); the entry rides in the low half
            key[n] = ((uint64_t)(0xFFFFFu - w) << 44) | ((uint64_t)n << 32) | ((uint32_t)j << 16) | (uint32_t)t;
            ++n;
        }
    }
    std::sort(key, key + n);
    for (int i = 0; i < n; ++i) ord.e[i] = (uint32_t)key[i];
    ord.n = n;
    ord.unit_log2 = log2;
    return n << log2;
}

// Which of its shapes dK / dV runs in (see the kernels).  An estimate of each shape's duration, to compare the shapes by and up to half as much again as the
// microseconds it takes (one segment of 7168, 32 / 8 heads: 1120 in four pairs, measured 754): the trips (64
// query rows against a workgroup's key rows) that a CU has to make at the rate of a full chip, or the longest chain of
// trips (the first key rows of the longest segment, all query heads of a group) at the rate its workgroup sees, whichever is longer, and what the
// blocks take to finish two trips behind their scores.  Over 480 launches of one segment or of ViT tiles measured in every shape
// (profiles/dkv_shape_choice.csv: 64 - 16400 tokens, 1 - 25 key / value heads, groups of 1 - 6, both masks; the 64 of texts were fitted to as well, but it does
// not hold their lengths) the picks are 0.25 % slower in the mean than the fastest shape; fifteen more than 3 %, the worst 7.6 % (one segment of 7168, 10
// heads of 64: 166 us, with tiles of 64 154).  Eight of the fifteen are one bias: bidirectional launches of heads of 128 that keep four pairs where blocks are
// 3.3 - 5.5 % faster (five ViT tiles, 48 / 8 heads: 328 us, blocks 311).
namespace {
struct DkvShape { int kv_rows; double full, chain, ends; };
constexpr DkvShape DKV_64[] = {{64, 0.81, 1.1, 0}, {64, 0.70, 1.53, 0}};                                // SR = 64, SR = 32 (six pairs: below)
constexpr DkvShape DKV_128[] = {{128, 1.69, 2.5, 0}, {64, 2.4, 0.85, 1.5}, {64, 2.8, 1.25, 0}};      // four pairs, blocks, two pairs
}  // namespace
int dkv_shape(const ob_segments *seg, int nkv, int group, int d, bool causal) {
    int best = 0;
    double t_best = 0;
    for (int i = 0; i < (d == 128 && !causal ? 3 : 2); ++i) {      // (shape 2 is bidirectional)
        const DkvShape &sh = d == 128 ? DKV_128[i] : DKV_64[i];
        double sum = 0, chain = 0;
        for (int j = 0; j < seg->n_seg; ++j) {
            const double len = seg->cu_host[j + 1] - seg->cu_host[j], tiles = ceil(len / sh.kv_rows), first = ceil(len / 64);
            sum += tiles * first - (causal ? 0.5 * tiles * (tiles - 1) * sh.kv_rows / 64 : 0.0);
            chain = std::max(chain, first);
        }
        // (no segment longer than 64 rows: half of four pairs have nothing to do, and a trip is theirs that have; causal, 8 heads: 9.5 us, blocks 10.0,
        // 32 heads over 8: 14.9 and 14.3)
        const double trip = sh.kv_rows == 128 && chain == 1 ? 1.5 : sh.chain;
        const double t = group * std::max(sum * nkv / compute_units() * sh.full, chain * trip) + sh.ends;
        if (i == 0 || t < t_best) { t_best = t; best = i; }
    }
    // six pairs where two would need a second round (of two workgroups to a CU) and they do not: 520 or 176 workgroups, one segment
    // of 4097, 48 / 8 heads: 568 us with SR = 32, 635 with 64, 539; ten ViT tiles x 4 heads in groups of 4, 680 or 240: 116, 123,
    // 115; but three tiles x 10 heads, 510 or 180: 29, 28, 34
    if (d == 64 && !causal && (long)count_tiles(seg, 64) * nkv > 2 * compute_units() &&
        (long)count_tiles(seg, 32 * dkv_np(64, 2)) * nkv <= compute_units())
        return 2;
    return best;
}

}  // namespace ob
