// How many workgroups, and rows of partial sums, the row kernels and column reductions take for a size: shared by the
// kernels' launchers, the buffer layouts, and a host-only build.
#pragma once

namespace ob {

// Norm backward.
// rows of H <= 1024 elements, enough of them: 256 workgroups of eight row-walking waves (12300 x 1024: 22 us, a row per
// workgroup 61)
inline bool norm_bwd_folds(int T, int H) { return H <= 1024 && T >= 2048; }
// Otherwise a row per workgroup at a time, two workgroups of up to four waves to a CU or one of five to eight: 16327 x 4096
// 97 us (1024 workgroups 108, 256 99; a row per wave with a partial each 117), 16400 x 3200 75 (89, 96; 96),
// 1500 x 4096 16 (36), 32741 x 6144 276 (1024 workgroups 300; 256 threads with four vectors each 384).  Rows of one or two waves have
// too few bytes in flight in two workgroups: four from 4096 rows on, where the reduction of twice the partials costs less than that
// gains (with it, 16400 x 1088 55 -> 38, x 1536 58 -> 42, x 2048 62 -> 52, 4100 x 1088 17.7 -> 16.3; 2047 x 1088 13.2 -> 15.0).
inline int norm_bwd_workgroups(int T, int H) {
    const int n = norm_bwd_folds(T, H) || H > 4096 ? 256 : H <= 2048 && T >= 4096 ? 1024 : 512;
    return T < n ? T : n;
}
// Rows of partial sums that the workspace has room for: at least as many as workgroups.  (Up to twice as
// many from 1024 rows on: programs size buffers by what the size queries report, so the region stays as it is while most launches take
// half.)
inline int norm_bwd_partials(int T, int H) { return norm_bwd_folds(T, H) ? 256 : T < 1024 ? T : 1024; }

// column sums of a [T, C] tensor
inline int colsum_partials(int T) { return T < 256 ? T : 256; }

// The same beside a pass over the tensor, workgroups of eight waves on eight rows x 512 columns: as many as the chip holds at once (four to a CU),
// none beyond (10752 x 6144: 1020 of them 72 us, 1032 77; 516 86), at most one per eight rows.
inline int cols_pass_partials(int T, int C, int cus, int max_partials) {
    const int blocks = (C + 511) / 512, n = 4 * cus / blocks > 1 ? 4 * cus / blocks : 1;
    const int most = (T + 7) / 8 < max_partials ? (T + 7) / 8 : max_partials;
    return n < most ? n : most;
}

// Hand-over: the widest row of its norm, and the rows of partial sums that the workspace has a region of its own for.
inline int subsample_max_width() { return 16384; }
inline int subsample_wgrad_partials(int n_tok) { return n_tok < 64 ? n_tok : 64; }

}  // namespace ob
