// Which tiles a GEMM is cut into, decided from its sizes by an estimate of the launch's duration.
#include "gemm_plan.h"

#include <cmath>

#include "ob_internal.h"

namespace ob {

// compute units of the current device, asked once (256 on MI355X, also when no device answers: the
// size queries must work on a host without a GPU)
int compute_units() {
    static const int cus = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
            n = 256;
        (void)hipGetLastError();
        return n;
    }();
    return cus;
}
int tiles_of(TileKind kind, int M, int N) {
    return ((M + tile_rows(kind) - 1) / tile_rows(kind)) * ((N + tile_cols(kind) - 1) / tile_cols(kind));
}

namespace {

int slots_of(TileKind kind) { return (kind == SMALL || kind == FINE ? 2 : 1) * compute_units(); }   // workgroups the chip holds at a time
// The tail of `tiles` tiles cut into at most z slices of whole trips of the two-step loop; false: that cuts nothing.
bool cut(TileKind kind, int tiles, int nk, int z, Plan &p) {
    const int n_tail = tiles % slots_of(kind), chunk = ((nk + z - 1) / z + 1) & ~1;
    if (n_tail == 0 || nk < 16 || nk / z < 8 || (nk + chunk - 1) / chunk < 2) return false;
    p = Plan{kind, tiles - n_tail, n_tail, (nk + chunk - 1) / chunk, chunk};   // every slice has at least one K step
    return true;
}

// operands and result, once; the weights (N x K) of a launch that is not `cold` lie in the memory-side cache
double bytes_of(int M, int N, int K, bool cold = true) { return 2.0 * ((double)M * K + (cold ? (double)N * K : 0.0) + (double)M * N); }

// Duration of a launch in microseconds.  Fitted to 2564 GEMMs (64 - 16400 rows on either side, the linears of seven
// models, the three layouts; cold operands, N(0, 1) data), each measured with every kind of tile, whole and with
// its tail in 2, 3, 4, 5, 6, 8 slices (profiles/gemm_tile_choice.csv): over them the choices are 0.26 % slower than the best measured kind and 7.4 % faster
// than the choices of an estimate with big and small tiles alone, 22 more than 2 % slower than those (worst 15 %: 256 x 4096 x 4096
// "NN" 22.5 -> 25.8); run against that library, 2598 shapes, 8.0 % faster, 22 more than 2 % slower.
//  * big tiles come in rounds of one per CU, and the tiles of an incomplete last round take as long as a full one; a K
//    step takes 1.23 on a full chip, 1.1 while half the chip or less is at work (the clock is higher), prologue and
//    epilogue as much as 4.67 more (nothing else runs on the CU meanwhile).  "TN" takes a tenth more and 6.4: its outputs are
//    weights, many for few K steps (6144 x 6144 over 800 tokens: 74, small tiles 68);
//  * a 192 x 256 tile takes 0.82 of a big one's step for 0.75 of its work, with 2.6 for its ends, 4 in several rounds: for rows that fit it better,
//    or a round that it fills and big tiles do not (3072 x 4096 x 4096, 256 tiles instead of 192: 85 -> 76; 3075 x 3200 x 12800,
//    221 instead of 169: 235 -> 208).  In "NT" a launch that fills f of its rounds takes 0.3 (1 - f) more: with few rows every
//    weight comes from HBM and B's loads have a slot and a half to land (557 x 12800 x 3200, 150 tiles: 62, small ones 54; not
//    so, `cold` false, behind a launch that has just read the same weights);
//  * a small tile with a CU to itself is bound by what the CU takes in from beyond the L2 (50 - 75 bytes per ns, also
//    with a ring twice as deep, with eight waves, or with lines fetched ahead by another wave: 0.5 per K step of 32 KB).
//    Two to a CU take 0.94 each, and, out of step as they are, hide each other's epilogues and fill the last round
//    gradually: a round that is f full adds 0.4 + 0.735 f (520 tiles, 1.02 rounds, 26 against 20 for 192 x 256 ones), but a launch
//    that gives any CU two lasts as long as two (300 tiles over K = 7175 106, 93 big ones in two slices 91);
//  * a deep one has the CU to itself as well, with four instead of two K steps on their way.  Only "NT" has it: there
//    B's loads have a slot and a half to land in the shallow ring, too little when the weights come from HBM
//    (557 x 4096 x 4096: 50 -> 36 us; 557 x 6144 x 4096: 51 -> 38), and it keeps its rate when tiles are many enough for
//    rounds;
//  * a fine one takes in half of a small one's bytes per K step, so a launch too small to give every CU a tile is done
//    in little more than half the time on four times the CUs (557 x 1024 x 1024 10.3 -> 7.0, 1025 x 768 x 2112
//    15.6 -> 10.9, 768 x 768 over 1500 tokens 13.8 -> 9.4), while a full chip loses by its 16 instead of 8 KB per 1 MFLOP,
//    most of all in "TN", whose operands it reads 128 bytes at a time;
//  * the slices' sums cost 4 bytes per element and slice at 3.4 TB/s and 2.9 for the second launch;
//  * operands and result pass at 6 TB/s at best, at 4.7 in the short rows of fine tiles (64 x 6144 x 32768 "NN": fine ones 98,
//    small ones 85): the fourth root of the fourth powers, so that of two plans bound by memory the better one stays ahead.
double estimate_us(int layout, TileKind kind, int nk, double bytes, const Plan &p, bool cold = true) {
    const double cus = compute_units();
    const bool sliced = p.splits > 1, tn = layout == 2;
    const double whole = sliced ? p.n_full : 0, tail = sliced ? (double)p.n_tail * p.splits : p.n_full + p.n_tail;
    const int k_tail = sliced ? p.k_chunk : nk;
    const double sums = sliced ? tail * tile_rows(kind) * tile_cols(kind) * 4 / 3.38e6 + 2.94 : 0.0;
    const bool alone = whole == 0 && tail <= cus;
    // tiles that share a CU in twos; the last of their rounds is `part` full
    const double pairs = tail / (2 * cus), part = pairs - ceil(pairs) + 1;
    auto paired = [&](double step, double edge, double last, double least) { return fmax(pairs + last, least) * (nk + edge) * step; };
    auto paired_slices = [&](double step, double edge) { return (whole / (2 * cus) * (nk + edge) + ceil(pairs) * (k_tail + edge)) * step; };
    double t = 0;
    switch (kind) {
    case MID:
    case BIG: {
        const double rounds = ceil(tail / cus), fill = (whole + tail) / (rounds * cus + whole);
        const double edge = kind == MID ? (whole + tail <= cus ? 2.6 : 4.0) : tn ? 6.4 : 4.67;
        const double rate = kind == BIG ? (tn ? 1.115 : 1.0) : 0.82 * (layout == 0 && cold ? 1 + 0.3 * (1 - fill) : 1.0);
        t = (whole / cus * (nk + edge) + rounds * (k_tail + edge)) * (1.1 + 0.13 * fmax(0.0, 2 * fill - 1)) * rate;
        break;
    }
    case SMALL: {
        const double edge = tn ? 2.7 : 1.17;
        t = alone ? (k_tail + 2.86) * (layout == 0 ? 0.566 : 0.521)
                  : sliced ? paired_slices(0.939, edge) : paired(0.939, edge, 0.4 - 0.265 * part, 0.95);
        break;
    }
    case DEEP: t = whole / cus * (nk + 4.0) * 0.536 + ceil(tail / cus) * (k_tail + 4.0) * (alone ? 0.51 : 0.536); break;
    case FINE:
        t = alone ? (k_tail + 5.82) * 0.236 : sliced ? paired_slices(0.49, 3.0) : paired(tn ? 0.532 : 0.403, 3.0, 0.355, tn ? 0.955 : 1.04);
        break;
    }
    t += sums + 1.5;
    const double moved = bytes / (kind == FINE ? 4.7e6 : 6e6), t2 = t * t, m2 = moved * moved;
    return sqrt(sqrt(t2 * t2 + m2 * m2));
}

// The scratch that a GEMM may fill with slice sums, and that the size queries report, is part of the interface:
// programs size buffers by it, once for the largest batch.  So it is a rule of its own, and the plan of a launch
// stays within it (that costs 0.26 % over the measured shapes).
Plan scratch_plan(TileKind whole_kind, double t_whole, int tiles_big, int tiles_small, int nk) {
    auto rule = [&](TileKind kind, const Plan &p) {
        const double cus = compute_units(), w = (double)p.n_tail * p.splits;
        const double sums = w * (kind == BIG ? 65536.0 : 16384.0) * 4.0 / 4e6 + 3.0;
        if (kind == BIG) return p.n_full / cus * (nk + 5) * 1.3 + ceil(w / cus) * (p.k_chunk + 5) * 1.3 + sums;
        if (p.n_full == 0 && w <= cus) return (p.k_chunk + 3) * 0.47 + sums;
        return p.n_full / (2 * cus) * (nk + 1) * 0.9 + ceil(w / (2 * cus)) * (p.k_chunk + 1) * 0.9 + sums;
    };
    Plan best{whole_kind, whole_kind == BIG ? tiles_big : tiles_small, 0, 1, 0}, p;
    double t_best = 0.93 * t_whole;
    for (TileKind kind : {SMALL, BIG})
        for (int z = 2; z <= 8; ++z) {
            const int tiles = kind == BIG ? tiles_big : tiles_small;
            if (tiles == 0 || !cut(kind, tiles, nk, z, p)) continue;
            const double t = rule(kind, p);
            if (t < t_best) { t_best = t; best = p; }
        }
    return best;
}

}  // namespace

size_t scratch_bytes(int M, int N, int K) {
    const int big = tiles_of(BIG, M, N), small = tiles_of(SMALL, M, N), nk = (K + KSTEP - 1) / KSTEP;
    const double cus = compute_units();
    const double t_big = ceil(big / cus) * (nk + 5) * 1.3;
    const double t_small = small <= cus ? (nk + 3) * 0.47 : (small / (2 * cus) + 0.4) * (nk + 1) * 0.9;
    return scratch_plan(t_big <= t_small ? BIG : SMALL, fmin(t_big, t_small), big, small, nk).part_bytes();
}

namespace {

// 192 x 256 tiles where they fill at least seven eighths of their columns (11275 x 640 x 2560, five sixths, inside a step:
// "NT" 63, "NN" 47 us, small tiles 47 and 39; 12300 x 768 x 2112, all: 43 and 54)
bool mid_fits(int layout, int N) { return layout != 2 && 8L * N >= 7L * 256 * ((N + 255) / 256); }

// what a plan of a kind other than big and small tiles, and a split, has to promise over the others: within the scatter of the
// estimate the launch of fewer, larger and whole tiles is the safer one
constexpr double KIND_MARGIN = 1.018, SPLIT_MARGIN = 1 / 0.97;

// `scratch`: bytes for slice sums; t (may be null): the estimated duration
Plan make_plan(int layout, int M, int N, int K, size_t scratch, bool cold, double *t_out = nullptr) {
    const int nk = (K + KSTEP - 1) / KSTEP;
    const double bytes = bytes_of(M, N, K, cold);
    Plan best{BIG, 0, 0, 1, 0}, p;
    double t_best = -1;
    auto consider = [&](double margin) {
        const double t = estimate_us(layout, p.kind, nk, bytes, p, cold);
        if (t_best >= 0 && t * margin >= t_best) return;
        t_best = t * margin;
        best = p;
        if (t_out) *t_out = t;
    };
    for (TileKind kind : {BIG, SMALL, DEEP, FINE, MID}) {
        if ((kind == DEEP && layout != 0) || (kind == MID && !mid_fits(layout, N))) continue;
        const int tiles = tiles_of(kind, M, N);
        const double margin = kind == BIG || kind == SMALL ? 1.0 : KIND_MARGIN;
        p = Plan{kind, tiles, 0, 1, 0};
        consider(margin);
        for (int z = 2; z <= 8 && scratch; ++z)
            if (cut(kind, tiles, nk, z, p) && p.part_bytes() <= scratch) consider(margin * SPLIT_MARGIN);
    }
    return best;
}

}  // namespace

// Rows of a GEMM whose big (or 192-row) tiles fill whole rounds, and the rest as a launch of its own with the tiles
// that suit it.  A row of tiles that spills over a round costs the chip a round: 12300 rows are 48 rows of tiles and
// twelve rows of values, 16 tiles more than three rounds of 4096 columns (over K = 1024 104 us, cut 93; the 557 rows of
// a short text through 28672 columns, 45 of them cut off, 141 -> 127; 5125 x 3200 x 3200 95 -> 86; 8200 x 3200 x 12800,
// the rest in 192-row tiles, 507 -> 466).  The rest's columns are read a second time, out of the memory-side cache, and
// its launch starts on a chip that has run empty (3 us, and 3 % for a rest of smaller tiles).  It has to promise 3 % over a
// launch of whole tiles, and no more than 1 % less than one with slices, which hold less than they promise: of 420 launches
// measured with and without (profiles/gemm_row_cut.csv) it cuts 357, 3.8 % faster in the mean, eight of them more than 2 % slower
// (the worst 4 %: the last 271 of 15375 rows through 3200 x 12800).  K-contiguous A only: a cut of the tokens of "TN" is a split of its
// contraction.
RowCut make_row_cut(int layout, int M, int N, int K, size_t scratch) {
    double t_best;
    RowCut best{0, {}, make_plan(layout, M, N, K, scratch, true, &t_best)};
    if (layout == 2) return best;
    t_best *= best.rest.splits > 1 ? 1.01 : 0.97;
    const int nk = (K + KSTEP - 1) / KSTEP, cus = compute_units();
    for (TileKind kind : {BIG, MID}) {
        const int tn = tiles_of(kind, 1, N), tiles = tiles_of(kind, M, N);
        if (tiles <= cus || (kind == MID && !mid_fits(layout, N))) continue;
        const int m = (int)((long)(tiles / cus) * cus / tn) * tile_rows(kind);
        if (m == 0 || m >= M) continue;
        const Plan head{kind, tiles_of(kind, m, N), 0, 1, 0};
        double t;
        const Plan rest = make_plan(layout, M - m, N, K, scratch, false, &t);
        t = (t + estimate_us(layout, kind, nk, bytes_of(m, N, K), head)) * (rest.kind == BIG || rest.kind == MID ? 1.0 : 1.03) + 3.0;
        if (t < t_best) { t_best = t; best = RowCut{m, head, rest}; }
    }
    return best;
}

// An activation goes into the epilogue of the GEMM in front of it where that is one pass over small tiles: a launch (4 us of the calls that
// such sizes make) and a pass over the result are gone, and where two tiles share a CU one's epilogue runs beside the other's products.  Calls
// with -> without: step of hidden 256, 64 tokens 78.6 -> 83.4 us, 964 tokens 128.9 -> 133.0, of hidden 640 and three ViT tiles 299 -> 308, of 768 with
// SwiGLU, 3200 tokens 376 -> 381, forward of a ViT tile of hidden 1024 86.5 -> 88.1, hand-over of four tiles 75.4 -> 80.2.  SwiGLU's backward, two
// tensors in and two out, only where a CU has another tile to work on meanwhile (136 tiles of 128 x 128, 964 tokens: 17.2 us, apart 9.9 + 5.3).
// Big tiles have the CU to themselves and their epilogues reach HBM together: apart (7B block of 16384 tokens: the GEMM grew by 0.37 ms for a pass
// of 0.41).
bool gemm_act_fuses(int layout, int M, int N, int K, bool scratch, Plan *plan) {
    const int base = layout == GEMM_NT_GELU ? 0 : 1;
    const RowCut c = make_row_cut(base, M, N, K, scratch ? scratch_bytes(M, N, K) : 0);
    if (plan) *plan = c.rest;
    if (layout == GEMM_NN_SWIGLU_BWD && c.rest.kind == SMALL && c.rest.n_full + c.rest.n_tail <= compute_units()) return false;
    return c.m == 0 && c.rest.splits == 1 && c.rest.kind != BIG && c.rest.kind != MID;
}

namespace {

// The scratch of a group of "TN" GEMMs over one K: 256 x 256 tiles, the slices of the combined list's tail.
Plan group_scratch_plan(int total_tiles, int K) {
    const int nk = (K + KSTEP - 1) / KSTEP;
    return scratch_plan(BIG, ceil((double)total_tiles / compute_units()) * (nk + 5) * 1.3, total_tiles, 0, nk);
}

}  // namespace

// fp32 sums of the slices of the tiles whose contraction may be split; 0 for a GEMM without such tiles
size_t gemm_workspace_bytes(int, int M, int N, int K) { return scratch_bytes(M, N, K); }

size_t gemm_tn_group_workspace_bytes(int count, const GemmTN *g, int K) {
    int total = 0;
    size_t single = 0;
    for (int i = 0; i < count; ++i) {
        total += tiles_of(BIG, g[i].M, g[i].N);
        const size_t b = scratch_bytes(g[i].M, g[i].N, K);
        if (b > single) single = b;
    }
    const size_t grouped = group_scratch_plan(total, K).part_bytes();
    return grouped > single ? grouped : single;
}

// The weight gradients of a block in one launch, in tiles of one kind.  One list of tiles leaves one incomplete round
// instead of four, and the last tiles of one GEMM (with their read of R) hide behind the next one's: for up to 8K tokens
// it is the faster way wherever the estimate does not promise the opposite (backward of a block, us, one by one -> grouped: 300M
// ViT 1025 tokens 250 -> 226, 12300 1042 -> 940; 6B ViT 3075 1808 -> 1709; 7B model 557 770 -> 744, 4000 3091 -> 3007).
// Longer contractions keep their own launch order over the XCDs (see INTERLEAVE_MIN_K) unless it promises 7 % (the four
// gradients of the 6B ViT over 11275 tokens, promised 9 %: 2242 -> 2077; its backward over 16400, promised 5 %: 7550 -> 7600; 7B model 16327, 1 %: 11664 -> 11693).
bool make_group_plan(int count, const int *M, const int *N, int K, bool has_ws, size_t ws_bytes, Plan &p) {
    const int nk = (K + KSTEP - 1) / KSTEP;
    double t_single = 0.0, bytes = 0.0;
    int total[4] = {0, 0, 0, 0};           // tiles of each kind
    // (without what "TN" adds to big and small tiles: in a list, and among what else a backward launches, their stores are
    // hidden; a block's gradients over 420 tokens of the 7B model in big tiles 557, in small ones 580)
    auto time = [&](const Plan &q, double moved) { return estimate_us(q.kind == FINE ? 2 : 1, q.kind, nk, moved, q); };
    for (int i = 0; i < count; ++i) {
        const Plan p1 = make_plan(2, M[i], N[i], K, has_ws ? scratch_bytes(M[i], N[i], K) : 0, true);
        t_single += time(p1, bytes_of(M[i], N[i], K));
        bytes += bytes_of(M[i], N[i], K);
        for (TileKind kind : {BIG, SMALL, FINE}) total[kind] += tiles_of(kind, M[i], N[i]);
    }
    p = group_scratch_plan(total[BIG], K);
    double t_group = time(p, bytes);
    for (TileKind kind : {SMALL, FINE}) {
        const Plan q{kind, total[kind], 0, 1, 0};
        const double t = time(q, bytes);
        if (t < t_group) { t_group = t; p = q; }
    }
    return count > 1 && has_ws && ws_bytes >= p.part_bytes() && t_group <= (K < INTERLEAVE_MIN_K ? 1.0 : 0.93) * t_single;
}

}  // namespace ob
