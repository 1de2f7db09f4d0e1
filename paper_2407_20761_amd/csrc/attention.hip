// Flash-style variable-length attention for gfx950 (steps a4 and b4 of the block).
//
// A packed batch is a concatenation of segments (cu offsets); a token attends only inside its own
// segment, bidirectionally (ViT tile) or causally (LLM sample).  Work is tiled per segment, so
// score tiles that would straddle two segments are never formed, and causal tiles above the
// diagonal are skipped.
//
// All matrix products run on the 32x32x16 bf16 MFMA in "transposed" form: the wavefront's 32 query
// rows (forward, dQ) or 32 key rows (dK/dV) sit on the MFMA's column index, which is the lane
// index.  Each lane therefore owns ONE row of the softmax: row max / row sum are in-register
// reductions plus a single exchange between lane l and lane l+32, and the probabilities a lane
// holds in its accumulator registers are, without any data movement, exactly the 8-value k-slices
// the next MFMA wants as its second operand (accumulator register 8 (u%2) + e of row-tile u/2
// carries streamed row 16 u + 8 (e/4) + 4 (l/32) + e%4, and the other operand is fetched from LDS
// in that same order).
//
// The streamed 64-row tiles (K and V; Q and dO in the dK/dV kernel) are copied global -> LDS
// asynchronously (buffer loads that write LDS directly, two stages, the next tile in flight while
// the current one is multiplied) in their natural [row][D] layout.  Products that contract over D
// read 16-byte fragments; products that contract over the streamed rows read the same tile with
// the transposing LDS read (ds_read_b64_tr_b16), so no tile is ever stored twice.  16-byte chunks
// are XOR-swizzled by the row so that both kinds of read are free of bank conflicts.
#include <cmath>
#include <type_traits>

#include "attention_plan.h"
#include "ob_internal.h"

namespace ob {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

namespace {

#define OB_LDS __attribute__((address_space(3)))

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;
constexpr float NEG_BIG = -1.0e30f;
constexpr float RESCALE_LOG2 = 8.0f;  // the forward's reference maximum may lag the row maximum by this much (base-2 log)
constexpr int QT = 128;  // rows owned by a workgroup (4 waves x 32)
constexpr int WAIT_VM0 = 0x0F70;  // s_waitcnt vmcnt(0) only

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// The value of lane l ^ 32, in one vector instruction (v_permlane32_swap exchanges the upper half of its
// first register with the lower half of its second; given the same value twice, every lane ends up with
// its own value in one of the two results and its partner's in the other): __shfl_xor goes through the
// LDS crossbar, a round trip in the middle of the forward's dependent chain maximum -> exponentials.
__device__ __forceinline__ void both_halves(float x, float &a, float &b) {
#if defined(__HIP_DEVICE_COMPILE__)
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
#else
    a = b = x;
#endif
}
__device__ __forceinline__ float max_halves(float x) {
    float a, b;
    both_halves(x, a, b);
    return fmaxf(a, b);
}
__device__ __forceinline__ float sum_halves(float x) {
    float a, b;
    both_halves(x, a, b);
    return a + b;
}

// XOR applied to the 16-byte chunk index of tile row r.  D = 128 (16 chunks per 256-byte row):
// 16 consecutive rows get 16 different values (conflict-free fragment reads) and the 4 rows of a
// transposing read differ in bits 2-3 (they land in different 64-byte groups).  D = 64 (8 chunks
// per 128-byte row, two rows per bank window): the same two properties with 3 bits.
template <int D>
__device__ __forceinline__ int swz(int r) {
    return D == 128 ? (((r & 3) << 2) | ((r >> 2) & 3)) : ((((r >> 1) & 1) << 2) | ((r >> 2) & 3));
}

// Wave-level loads global -> LDS of N pieces, 16 bytes per lane (4 for the second form), lane i to byte 16 i (4 i) of its piece (lanes past the
// descriptor's range deliver zeros).  A piece is 1 KB behind the one before, piece SKIP 1 + SKIP.  As instructions: the compiler
// counts the builtin among the accesses that a later LDS read may have to wait for, and where stages are parts of one array it waits for the loads
// just issued in front of the first read of every trip.  What has to have landed is said by the s_waitcnt in front of each barrier.
// The compiler does not look inside either, so a block keeps the distances itself, whatever stands in front of it: five wait states from a vector instruction
// that wrote a part of the descriptor (a v_readlane that brings a spilled one back) to the first load, one from m0 to each.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"      // (m0 is a reserved register, never preserved across a clobber: that is what is meant)
#define OB_TO_LDS(WIDTH, P) "s_add_i32 m0, %[at], %[d" P "]\n\ts_nop 0\n\tbuffer_load_" WIDTH " %[v" P "], %[rsrc], 0 offen lds\n\t"
#define OB_PIECE(P) [d##P] "i"((FIRST + P < SKIP ? FIRST + P : FIRST + P + SKIP) * 1024), [v##P] "v"(voff[FIRST + P])
template <int N, int SKIP = N, int FIRST = 0>
__device__ __forceinline__ void load_lds16(u32x4 rsrc, unsigned char OB_LDS *dst, const uint32_t *voff) {
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(N == 1 || N == 2 || N % 4 == 0, "pieces");
    const uint32_t at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)dst);
    if constexpr (N == 1)
        asm volatile("s_nop 2\n\t" OB_TO_LDS("dwordx4", "0") : : [at] "s"(at), OB_PIECE(0), [rsrc] "s"(rsrc) : "m0", "scc", "memory");
    else if constexpr (N == 2)
        asm volatile("s_nop 2\n\t" OB_TO_LDS("dwordx4", "0") OB_TO_LDS("dwordx4", "1")
                     : : [at] "s"(at), OB_PIECE(0), OB_PIECE(1), [rsrc] "s"(rsrc) : "m0", "scc", "memory");
    else
        asm volatile("s_nop 2\n\t" OB_TO_LDS("dwordx4", "0") OB_TO_LDS("dwordx4", "1") OB_TO_LDS("dwordx4", "2") OB_TO_LDS("dwordx4", "3")
                     : : [at] "s"(at), OB_PIECE(0), OB_PIECE(1), OB_PIECE(2), OB_PIECE(3), [rsrc] "s"(rsrc) : "m0", "scc", "memory");
    if constexpr (N > 4) load_lds16<N - 4, SKIP, FIRST + 4>(rsrc, dst, voff);
#endif
}
__device__ __forceinline__ void load_lds4(u32x4 rsrc, unsigned char OB_LDS *dst, uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int FIRST = 0, SKIP = 1;
    const uint32_t at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)dst), voff[1] = {v};
    asm volatile("s_nop 2\n\t" OB_TO_LDS("dword", "0") : : [at] "s"(at), OB_PIECE(0), [rsrc] "s"(rsrc) : "m0", "scc", "memory");
#endif
}
#undef OB_PIECE
#undef OB_TO_LDS
#pragma clang diagnostic pop
// descriptor of the `bytes_left` bytes from `base` on (clamped to [0, 2^32 - 1], in scalar instructions: the compiler's
// own 64-bit compares go through the vector unit)
__device__ __forceinline__ u32x4 make_rsrc(const void *base, long bytes_left) {
    const uint64_t b = (uint64_t)base;
    u32x4 r = {(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b), (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)), 0u, 0x00020000u};
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t num;
    asm("s_cmp_eq_u32 %2, 0\n\ts_cselect_b32 %0, %1, -1\n\ts_cmp_lt_i32 %2, 0\n\ts_cselect_b32 %0, 0, %0"
        : "=&s"(num)
        : "s"(__builtin_amdgcn_readfirstlane((uint32_t)bytes_left)),
          "s"(__builtin_amdgcn_readfirstlane((int32_t)(bytes_left >> 32)))
        : "scc");
    r[2] = num;
#endif
    return r;
}

// 16 bytes of LDS per lane (a restrict argument says that no load to LDS in flight touches them: without it the compiler waits
// for all of those first)
template <class V>
__device__ __forceinline__ V lds16(const unsigned char OB_LDS *__restrict__ p) { return *(const V OB_LDS *)p; }

// s_waitcnt operand: at most `vm` vector-memory operations pending, no LDS operation
constexpr int wait_vm_lds0(int vm) { return (vm & 15) | ((vm >> 4) << 14) | 0x70; }

// The barrier instruction alone: what has to be complete in front of it is said by an s_waitcnt (__syncthreads() waits for every
// load in flight); the empty statements keep the compiler from moving LDS accesses across.
__device__ __forceinline__ void bare_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Per-lane addressing of one streamed [ROWS][D] tile family.
template <int D, int ROWS = ST>
struct Tile {
    static constexpr int RB = D * 2;            // bytes per tile row
    static constexpr int BYTES = ROWS * RB;
    static constexpr int CPR = RB / 16;         // chunks per row
    static constexpr int RPI = 1024 / RB;       // rows filled by one wave-level load
    static constexpr int LD = ROWS / RPI / 4;   // wave-level loads per wave per tile
    uint32_t voff[LD];                          // global byte offset of this lane's chunk (row-in-tile part)
    int rr[D / 16];                             // LDS offset of the 16-byte fragment read, per D-step t
    int tro[2][D / 32];                         // LDS offset of the transposing read, per half s and D-tile dt

    __device__ __forceinline__ void init(int ld, int wave, int lane) {
#pragma unroll
        for (int p = 0; p < LD; ++p) {
            const int row = (wave * LD + p) * RPI + lane / CPR;
            const int ch = (lane % CPR) ^ swz<D>(row);
            voff[p] = ((uint32_t)row * (uint32_t)ld + ch * 8) * 2u;
        }
        const int x = lane & 31, h = lane >> 5;
#pragma unroll
        for (int t = 0; t < D / 16; ++t) rr[t] = x * RB + (((2 * t + h) ^ swz<D>(x)) * 16);
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int dt = 0; dt < D / 32; ++dt) tro[s][dt] = tr_offset(lane, s, dt);
    }
    static __device__ __forceinline__ int tr_offset(int lane, int s, int dt) {
        const int b = lane >> 4, q = lane & 15, kq = q >> 2, c = q & 3, hb = b >> 1;
        const int row = 8 * s + 4 * hb + kq;  // + 16 u
        const int chunk = 4 * dt + 2 * (b & 1) + (c >> 1);
        return row * RB + ((chunk ^ swz<D>(row)) * 16) + (c & 1) * 8;
    }
    // asynchronous copy of rows [row0, row0 + ROWS) of a [*, ld] matrix (column offset folded into
    // `base`); rows past the end of the matrix arrive as zeros
    __device__ __forceinline__ void issue(const unsigned char *base, long bytes_left,
                                          unsigned char OB_LDS *__restrict__ dst, int wave) const {
        const uint64_t b = (uint64_t)base;
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
        // the checked range: bytes_left clamped to [0, 2^32 - 1], in scalar instructions (the compiler's own
        // 64-bit compares go through the vector unit)
        uint32_t num = 0;
#if defined(__HIP_DEVICE_COMPILE__)
        asm("s_cmp_eq_u32 %2, 0\n\ts_cselect_b32 %0, %1, -1\n\ts_cmp_lt_i32 %2, 0\n\ts_cselect_b32 %0, 0, %0"
            : "=&s"(num)
            : "s"(__builtin_amdgcn_readfirstlane((uint32_t)bytes_left)),
              "s"(__builtin_amdgcn_readfirstlane((int32_t)(bytes_left >> 32)))
            : "scc");
#endif
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(((uint64_t)hi << 32) | lo), 0, (int)num, 0x00020000);
#pragma unroll
        for (int p = 0; p < LD; ++p)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, dst + (wave * LD + p) * 1024, 16, voff[p], 0, 0, 0);
    }
    // lane l: tile row 32 mt + l % 32, elements 16 t + 8 (l / 32) .. +7
    __device__ __forceinline__ bf16x8 frag_row(const unsigned char OB_LDS *__restrict__ tile, int mt, int t) const {
        return *(const bf16x8 OB_LDS *)(tile + rr[t] + mt * 32 * RB);
    }
    // lane l: column 32 dt + l % 32, rows 16 u + 8 (e / 4) + 4 (l / 32) + e % 4 for e = 0..7
    __device__ __forceinline__ bf16x8 frag_tr(const unsigned char OB_LDS *__restrict__ tile, int dt, int u) const {
        return frag_at(tile, tro[0][dt], tro[1][dt], u);
    }
    static __device__ __forceinline__ bf16x8 frag_at(const unsigned char OB_LDS *__restrict__ tile, int off0, int off1, int u) {
#if defined(__HIP_DEVICE_COMPILE__)  // gfx950-only builtin, hidden from the host pass
        typedef __attribute__((ext_vector_type(4))) short s16x4;
        typedef __attribute__((ext_vector_type(8))) short s16x8;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 OB_LDS *)(tile + off0 + u * 16 * RB));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 OB_LDS *)(tile + off1 + u * 16 * RB));
        return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#else
        return bf16x8{};
#endif
    }
};

// accumulator registers 8 (u % 2) .. +7 of a 32x32 tile -> the 8-slot second operand of step u
__device__ __forceinline__ bf16x8 pack8(const f32x16 &a, int base) {
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (__bf16)a[base + e];
    return o;
}

// Rotary backward folded into the epilogues of the backward kernels.  A lane holds, of one token's head
// row, accumulator (dt, r) = column 32 dt + 8 (r / 4) + 4 lh + r % 4: the rotary pair (i, i + D/2) is
// (dt, r) and (dt + D/64, r) of the same lane.  The gradient is rotated by minus the token's angle
// pos * base^(-2 i / D), pos = distance to the segment's first token (log2_base <= 0: no rotary).
// Sine and cosine come from the hardware's functions of the angle in revolutions, reduced to [0, 1)
// first: an absolute error of a few 1e-4 rad at positions in the thousands, an order of magnitude
// below the bf16 rounding of the result.
// x1: accumulator tile dt, x2: dt + D/64.
template <int D>
__device__ __forceinline__ void rotary_bwd_pair(f32x16 &x1, f32x16 &x2, int dt, int pos, float log2_base, int lh) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = 32 * dt + 8 * (r >> 2) + 4 * lh + (r & 3);
        const float theta = __builtin_amdgcn_exp2f(-2.0f * (float)i / (float)D * log2_base);
        float rev = (float)pos * theta * 0.15915494309189535f;
        rev -= floorf(rev);
        const float sn = __builtin_amdgcn_sinf(rev), cs = __builtin_amdgcn_cosf(rev);
        const float a = x1[r], b = x2[r];
        x1[r] = a * cs + b * sn;
        x2[r] = b * cs - a * sn;
    }
}
template <int D>
__device__ __forceinline__ void rotary_bwd_row(f32x16 (&acc)[D / 32], int pos, float log2_base, int lh) {
#pragma unroll
    for (int dt = 0; dt < D / 64; ++dt) rotary_bwd_pair<D>(acc[dt], acc[dt + D / 64], dt, pos, log2_base, lh);
}

// Which workgroup does which tile.  The launch is one-dimensional: workgroup b works on tile
// b / heads for head slot b % heads, so all heads of a tile are dispatched together, and (workgroups
// being dealt round-robin to the 8 XCDs) head slot hs runs on XCD hs % 8: with a head count that is a
// multiple of 8 the slots are renumbered so that an XCD only ever sees heads [x heads/8, (x+1) heads/8),
// i.e. the query heads of one key/value group (and that group's K and V) stay in one XCD's L2.
__device__ __forceinline__ int head_of_slot(int hs, int heads) {
    return (heads & 7) == 0 ? (hs & 7) * (heads >> 3) + (hs >> 3) : hs;
}

// Which segment-aligned tile (of `tile_rows` rows) has number `tile` when tiles are numbered segment
// by segment.  Thread j looks at segment j (256 segments per round), an inclusive scan over the
// workgroup gives each segment's first tile number, and the thread whose range holds `tile`
// publishes the answer -- one global-memory round trip instead of a serial walk over cu.
struct TileInfo { int seg_start, seg_end, row0; };
__device__ __forceinline__ TileInfo find_tile(const int32_t *__restrict__ cu, int n_seg, int tile_rows,
                                              int *sh /* >= 8 ints */, int tile) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool scans = tid < 256;  // waves past the fourth only take part in the barriers
    if (tid == 0) sh[2] = -1;
    int base = 0;  // tiles in the segments of earlier rounds
    for (int j0 = 0; j0 < n_seg; j0 += 256) {
        const int j = j0 + tid;
        int a = 0, b = 0, nt = 0;
        if (scans && j < n_seg) {
            a = cu[j];
            b = cu[j + 1];
            nt = (b - a + tile_rows - 1) / tile_rows;
        }
        int incl = nt;  // inclusive scan inside the wave
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o);
            if (lane >= o) incl += up;
        }
        __syncthreads();  // sh[4..7] free (previous round consumed)
        if (scans && lane == 63) sh[4 + wave] = incl;
        __syncthreads();
        int before = base;
        for (int w = 0; w < (wave & 3); ++w) before += sh[4 + w];
        const int first = before + incl - nt;  // number of this segment's first tile
        if (scans && nt > 0 && tile >= first && tile < first + nt) {
            sh[0] = a;
            sh[1] = b;
            sh[2] = a + (tile - first) * tile_rows;
        }
        base += sh[4] + sh[5] + sh[6] + sh[7];
    }
    __syncthreads();
    TileInfo t;
    t.seg_start = __builtin_amdgcn_readfirstlane(sh[0]);
    t.seg_end = __builtin_amdgcn_readfirstlane(sh[1]);
    t.row0 = __builtin_amdgcn_readfirstlane(sh[2]);
    return t;
}

// the tile of place `rank` in the order of work; UNITS (dK / dV): the table may hold units of several tiles, and row0 < 0:
// that place of its unit lies past the segment's end
template <bool UNITS>
__device__ __forceinline__ TileInfo pick_tile(const TileOrder &ord, int rank, const int32_t *__restrict__ cu,
                                              int n_seg, int tile_rows, int *sh) {
    if (ord.n == 0) return find_tile(cu, n_seg, tile_rows, sh, rank);
    const uint32_t e = ord.e[UNITS ? rank >> ord.unit_log2 : rank];
    const int seg = (int)(e >> 16);
    TileInfo t;
    t.seg_start = __builtin_amdgcn_readfirstlane(cu[seg]);
    t.seg_end = __builtin_amdgcn_readfirstlane(cu[seg + 1]);
    t.row0 = t.seg_start + (UNITS ? tile_of_rank(ord, e, rank) : (int)(e & 0xFFFFu)) * tile_rows;
    if (UNITS && t.row0 >= t.seg_end) t.row0 = -1;
    return t;
}

// ------------------------------------------------------------------------------------------------
// forward:  S^T = K Q^T,  online softmax per lane,  O^T += V^T P^T
// ------------------------------------------------------------------------------------------------
// LDS reads are issued one batch ahead of the MFMAs that consume them (explicit double buffers and
// scheduling groups): left alone, the compiler emits read / wait / MFMA triples and every MFMA
// pays a full LDS round trip.
#define OB_SCHED_READS_THEN_MFMA(n_reads, n_mfma)                 \
    do {                                                          \
        __builtin_amdgcn_sched_group_barrier(0x100, (n_reads), 0); \
        __builtin_amdgcn_sched_group_barrier(0x008, (n_mfma), 0);  \
        __builtin_amdgcn_sched_barrier(0);                         \
    } while (0)

template <int D, bool CAUSAL, bool MASK>
__device__ __forceinline__ void fwd_tile(const unsigned char OB_LDS *__restrict__ ks,
                                         const unsigned char OB_LDS *__restrict__ vs, const Tile<D> &tl,
                                         const bf16x8 (&qf)[D / 16], f32x16 (&acc_o)[D / 32], float &m_run,
                                         float &l_run, int kv0, int seg_end, int q_row, float sl2) {
    const int lh = (threadIdx.x & 63) >> 5;
    constexpr int HB = 2;                 // K fragments (D-steps) per batch
    constexpr int R = D == 128 ? 3 : 2;   // batches in flight (ring depth)
    constexpr int PER = (D / 16) / HB;    // batches per 32-row tile
    constexpr int NB = 2 * PER;
    constexpr int DT = D / 32;
    f32x16 acc_s[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_s[mt][r] = 0.f;
    bf16x8 fa[R][HB], fb[2][DT];
#pragma unroll
    for (int b = 0; b < R - 1; ++b)
#pragma unroll
        for (int i = 0; i < HB; ++i) fa[b][i] = tl.frag_row(ks, b / PER, (b % PER) * HB + i);
#pragma unroll
    for (int b = 0; b < NB; ++b) {  // batch b: row tile b / PER, D-steps (b % PER) HB ..
        constexpr int AHEAD = R - 1;
        if (b + AHEAD < NB) {
#pragma unroll
            for (int i = 0; i < HB; ++i)
                fa[(b + AHEAD) % R][i] = tl.frag_row(ks, (b + AHEAD) / PER, ((b + AHEAD) % PER) * HB + i);
        } else if (b + AHEAD == NB) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) fb[0][dt] = tl.frag_tr(vs, dt, 0);
        }
#pragma unroll
        for (int i = 0; i < HB; ++i)
            acc_s[b / PER] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[b % R][i], qf[(b % PER) * HB + i], acc_s[b / PER], 0, 0, 0);
        if (b + AHEAD < NB) OB_SCHED_READS_THEN_MFMA(HB, HB);
        else if (b + AHEAD == NB) OB_SCHED_READS_THEN_MFMA(2 * DT, HB);
        else OB_SCHED_READS_THEN_MFMA(0, HB);
    }
    // the running maximum is kept on the raw scores; the softmax scale rides in the exponent's FMA
    float mx = NEG_BIG;
    if (MASK) {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int kv = kv0 + mt * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
                const bool ok = kv < seg_end && (!CAUSAL || kv <= q_row);
                const float s = ok ? acc_s[mt][r] : NEG_BIG;
                acc_s[mt][r] = s;
                mx = fmaxf(mx, s);
            }
    } else {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, acc_s[mt][r]);
    }
    mx = max_halves(mx);
    // The reference maximum m_run of a row only has to keep the exponentials in range, it need not be
    // the true maximum: it follows the row maximum when that has outgrown it by more than 2^RESCALE_LOG2
    // in some row of the wave (probabilities then reach at most 2^RESCALE_LOG2, harmless in fp32 sums
    // and in bf16 operands), so the accumulators are rescaled a few times per row instead of at almost
    // every tile (with random scores some row of 32 finds a new maximum in nearly every tile).
    if (__any((mx - m_run) * sl2 > RESCALE_LOG2)) {
        const float m_new = fmaxf(m_run, mx);
        const float alpha = fast_exp2((m_run - m_new) * sl2);
        l_run *= alpha;
#pragma unroll
        for (int i = 0; i < D / 32; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc_o[i][r] *= alpha;
        m_run = m_new;
    }
    const float c = m_run * sl2;
    float psum = 0.f;
    // The exponentials of contraction step u + 1 (8 per lane, then their rounding to bf16) are issued
    // between the MFMAs of step u, one MFMA to a few vector instructions: a wave's own element-wise
    // work then runs in the shadow of its own matrix instructions.
    auto probs = [&](int u) {
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float p = fast_exp2(acc_s[u >> 1][8 * (u & 1) + e] * sl2 - c);
            psum += p;
            o[e] = (__bf16)p;
        }
        return o;
    };
    bf16x8 pb = probs(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < ST / 16; ++u) {
        bf16x8 pn = pb;
        if (u + 1 < ST / 16) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) fb[(u + 1) & 1][dt] = tl.frag_tr(vs, dt, u + 1);
            pn = probs(u + 1);
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
            acc_o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[u & 1][dt], pb, acc_o[dt], 0, 0, 0);
        if (u + 1 < ST / 16) {
            __builtin_amdgcn_sched_group_barrier(0x100, 2 * DT, 0);        // next step's V fragments
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);         // one MFMA
                __builtin_amdgcn_sched_group_barrier(0x002, (28 + DT - 1) / DT, 0);   // its share of 28 vector instructions
            }
            __builtin_amdgcn_sched_barrier(0);
        } else {
            OB_SCHED_READS_THEN_MFMA(0, DT);
        }
        pb = pn;
    }
    l_run += psum;
}

// (D = 64: 128 registers, four waves on a SIMD)
template <int D, bool CAUSAL>
__global__ __launch_bounds__(256, D == 64 ? 4 : 2) void attn_fwd_kernel(
    const __bf16 *__restrict__ q, const __bf16 *__restrict__ k, const __bf16 *__restrict__ v,
    __bf16 *__restrict__ o, float *__restrict__ lse, int ldq, int ldkv, int ldo,
    const int32_t *__restrict__ cu, int n_seg, int T, int group, float scale, int heads, TileOrder ord) {
    __shared__ __attribute__((aligned(1024))) unsigned char k_s0[Tile<D>::BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char v_s0[Tile<D>::BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char k_s1[Tile<D>::BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char v_s1[Tile<D>::BYTES];
    __shared__ int sh[8];
    const int rank = blockIdx.x / heads;
    const TileInfo ti = pick_tile<false>(ord, rank, cu, n_seg, QT, sh);
    if (ti.row0 < 0) return;
    const int head = head_of_slot(blockIdx.x - rank * heads, heads), kvh = head / group;
    const int lane = threadIdx.x & 63, lx = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q_row = min(ti.row0 + wave * 32 + lx, ti.seg_end - 1);
    const bool q_live = ti.row0 + wave * 32 + lx < ti.seg_end;
    const int wave_q_last = min(ti.row0 + wave * 32 + 31, ti.seg_end - 1);
    const float sl2 = scale * LOG2E;

    Tile<D> tl;
    tl.init(ldkv, wave, lane);
    const unsigned char *kbase = (const unsigned char *)(k + kvh * D);
    const unsigned char *vbase = (const unsigned char *)(v + kvh * D);
    const long kv_bytes = (long)T * ldkv * 2 - (long)kvh * D * 2;  // from kbase / vbase to the end

    bf16x8 qf[D / 16];
#pragma unroll
    for (int t = 0; t < D / 16; ++t)
        qf[t] = *(const bf16x8 *)(q + (size_t)q_row * ldq + head * D + 16 * t + 8 * lh);
    f32x16 acc_o[D / 32];
#pragma unroll
    for (int i = 0; i < D / 32; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_o[i][r] = 0.f;
    float m_run = NEG_BIG, l_run = 0.f;

    const int kv_end = CAUSAL ? min(ti.seg_end, ti.row0 + QT) : ti.seg_end;
    const int n_tiles = (kv_end - ti.seg_start + ST - 1) / ST;
    unsigned char OB_LDS *const ks0 = (unsigned char OB_LDS *)k_s0, *const ks1 = (unsigned char OB_LDS *)k_s1;
    unsigned char OB_LDS *const vs0 = (unsigned char OB_LDS *)v_s0, *const vs1 = (unsigned char OB_LDS *)v_s1;
    {
        const long off = (long)ti.seg_start * ldkv * 2;
        tl.issue(kbase + off, kv_bytes - off, ks0, wave);
        tl.issue(vbase + off, kv_bytes - off, vs0, wave);
    }
    // Tiles before the workgroup's first row (causal) or before the ragged end need no mask; they
    // run in a loop of their own whose body is a single straight path (with several paths per
    // iteration the register allocator shuffles the accumulators between homes every iteration).
    const int n_main = CAUSAL ? (ti.row0 - ti.seg_start) / ST : (ti.seg_end - ti.seg_start) / ST;
    int j = 0;
#define OB_FWD_ITER(MASKED, KS, VS, KS_NEXT, VS_NEXT)                                                     \
    {                                                                                                    \
        const int kv0 = ti.seg_start + j * ST;                                                           \
        __builtin_amdgcn_s_waitcnt(WAIT_VM0);                                                            \
        __syncthreads();                                                                                 \
        if (j + 1 < n_tiles) {                                                                           \
            const long off = (long)(kv0 + ST) * ldkv * 2;                                                \
            tl.issue(kbase + off, kv_bytes - off, (KS_NEXT), wave);                                      \
            tl.issue(vbase + off, kv_bytes - off, (VS_NEXT), wave);                                      \
        }                                                                                                \
        if (!(MASKED))                                                                                   \
            fwd_tile<D, CAUSAL, false>((KS), (VS), tl, qf, acc_o, m_run, l_run, kv0, ti.seg_end, q_row,  \
                                       sl2);                                                             \
        else if (!(CAUSAL && kv0 > wave_q_last))                                                         \
            fwd_tile<D, CAUSAL, true>((KS), (VS), tl, qf, acc_o, m_run, l_run, kv0, ti.seg_end, q_row,   \
                                      sl2);                                                              \
        ++j;                                                                                             \
    }
    // two tiles per trip: the stage buffers are then compile-time constants and every LDS address is
    // a register plus an immediate offset
    while (j + 1 < n_main) {
        OB_FWD_ITER(false, ks0, vs0, ks1, vs1)
        OB_FWD_ITER(false, ks1, vs1, ks0, vs0)
    }
#define OB_FWD_ANY(MASKED) OB_FWD_ITER(MASKED, (j & 1) ? ks1 : ks0, (j & 1) ? vs1 : vs0, (j & 1) ? ks0 : ks1, (j & 1) ? vs0 : vs1)
    while (j < n_main) OB_FWD_ANY(false)
    while (j < n_tiles) OB_FWD_ANY(true)
#undef OB_FWD_ANY
#undef OB_FWD_ITER
    const float l_tot = sum_halves(l_run);
    if (!q_live) return;
    const float inv = 1.0f / l_tot;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            bf16x4 ov;
#pragma unroll
            for (int e = 0; e < 4; ++e) ov[e] = (__bf16)(acc_o[dt][4 * g + e] * inv);
            *(bf16x4 *)(o + (size_t)q_row * ldo + head * D + dt * 32 + g * 8 + lh * 4) = ov;
        }
    if (lh == 0) lse[(size_t)head * T + q_row] = (m_run * sl2 + __builtin_amdgcn_logf(l_tot)) * LN2;
}

// ------------------------------------------------------------------------------------------------
// backward, part 1: dQ.  A workgroup owns 128 query rows of one head (four wavefronts, 32 rows
// each) and streams the segment's 64-row key/value tiles (up to the diagonal when causal); P is
// rebuilt from the saved log-sum-exp.  A wave takes the two 32-row halves of a streamed tile one
// after the other through the three products
//   S^T = K Q^T,  P = 2^(scale log2(e) S - lse2),  dP^T = V dO^T,  dS^T = P (dP^T - Delta),
//   dQ^T += K^T dS^T
// so its state between the products is that of a 32 x 32 block (two such waves fit on a SIMD; two
// workgroups share a CU and, as nothing synchronises them, their phases drift apart).  Every K / V
// tile a workgroup copies serves 128 query rows: the first layout, two waves per 32 query rows each
// on one half of the tile with their partial dQ added at the end, asked the L2 for twice the bytes
// per MFMA (4.7 GB per launch on the 7B-shaped batch, 10 TB/s) and had a barrier per 24 MFMAs.
// ------------------------------------------------------------------------------------------------
template <int D, bool CAUSAL, bool MASK>
__device__ __forceinline__ void dq_half(const unsigned char OB_LDS *__restrict__ ks,
                                        const unsigned char OB_LDS *__restrict__ vs, const Tile<D> &tl,
                                        const bf16x8 (&qf)[D / 16], const bf16x8 (&dof)[D / 16],
                                        f32x16 (&acc_dq)[D / 32], float lse2, float dlt, int kv_first,
                                        int seg_end, int q_row, float sl2) {
    // ks / vs point at a 32-row half of the K / V tile; kv_first is its first key row
    const int lh = (threadIdx.x & 63) >> 5;
    constexpr int HB = 2;             // D-steps per batch (a batch reads HB fragments of K and HB of V)
    constexpr int NB = (D / 16) / HB;
    constexpr int DT = D / 32;
    f32x16 acc_s, acc_dp;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc_s[r] = acc_dp[r] = 0.f;
    bf16x8 fk[2][HB], fv[2][HB], fb[2][DT];
#pragma unroll
    for (int i = 0; i < HB; ++i) {
        fk[0][i] = tl.frag_row(ks, 0, i);
        fv[0][i] = tl.frag_row(vs, 0, i);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (b + 1 < NB) {
#pragma unroll
            for (int i = 0; i < HB; ++i) {
                fk[(b + 1) & 1][i] = tl.frag_row(ks, 0, (b + 1) * HB + i);
                fv[(b + 1) & 1][i] = tl.frag_row(vs, 0, (b + 1) * HB + i);
            }
        } else {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) fb[0][dt] = tl.frag_tr(ks, dt, 0);
        }
#pragma unroll
        for (int i = 0; i < HB; ++i) {
            acc_s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fk[b & 1][i], qf[b * HB + i], acc_s, 0, 0, 0);
            acc_dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fv[b & 1][i], dof[b * HB + i], acc_dp, 0, 0, 0);
        }
        if (b + 1 < NB) OB_SCHED_READS_THEN_MFMA(2 * HB, 2 * HB); else OB_SCHED_READS_THEN_MFMA(2 * DT, 2 * HB);
    }
    // dS of contraction step h (8 values per lane, rounded to bf16); step 1's are worked out between the
    // MFMAs of step 0, so the wave's own element-wise work runs in the shadow of its matrix instructions
    auto dscores = [&](int h) {
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int r = 8 * h + e;
            bool ok = true;
            if (MASK) {
                const int kv = kv_first + 8 * (r >> 2) + 4 * lh + (r & 3);
                ok = kv < seg_end && (!CAUSAL || kv <= q_row);
            }
            const float p = ok ? fast_exp2(acc_s[r] * sl2 - lse2) : 0.f;
            o[e] = (__bf16)(p * (acc_dp[r] - dlt));
        }
        return o;
    };
    const bf16x8 ds0 = dscores(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) fb[1][dt] = tl.frag_tr(ks, dt, 1);
    const bf16x8 ds1 = dscores(1);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
        acc_dq[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[0][dt], ds0, acc_dq[dt], 0, 0, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 2 * DT, 0);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, (MASK ? 60 : 36) / DT, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
        acc_dq[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[1][dt], ds1, acc_dq[dt], 0, 0, 0);
    OB_SCHED_READS_THEN_MFMA(0, DT);
}

template <int D, bool CAUSAL>
__global__ __launch_bounds__(256, 2) void attn_bwd_dq_kernel(
    const __bf16 *__restrict__ d_o, const __bf16 *__restrict__ q, const __bf16 *__restrict__ k,
    const __bf16 *__restrict__ v, const __bf16 *__restrict__ o, const float *__restrict__ lse,
    float *__restrict__ lse2_all, float *__restrict__ delta, __bf16 *__restrict__ dq, int ldq, int ldkv, int ldo,
    const int32_t *__restrict__ cu, int n_seg, int T, int group, float scale, float rot_log2_base, int heads,
    TileOrder ord) {
    __shared__ __attribute__((aligned(1024))) unsigned char k_s0[Tile<D>::BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char v_s0[Tile<D>::BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char k_s1[Tile<D>::BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char v_s1[Tile<D>::BYTES];
    __shared__ int sh[8];
    const int rank = blockIdx.x / heads;
    const TileInfo ti = pick_tile<false>(ord, rank, cu, n_seg, QT, sh);
    if (ti.row0 < 0) return;
    const int head = head_of_slot(blockIdx.x - rank * heads, heads), kvh = head / group;
    const int lane = threadIdx.x & 63, lx = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q_row = min(ti.row0 + wave * 32 + lx, ti.seg_end - 1);
    const bool q_live = ti.row0 + wave * 32 + lx < ti.seg_end;
    const int wave_q_last = min(ti.row0 + wave * 32 + 31, ti.seg_end - 1);
    const bool wave_live = ti.row0 + wave * 32 < ti.seg_end;   // a wave past the segment's end only copies
    const float sl2 = scale * LOG2E;
    constexpr int DT = D / 32, HALF = 32 * Tile<D>::RB;

    Tile<D> tl;
    tl.init(ldkv, wave, lane);
    const unsigned char *kbase = (const unsigned char *)(k + kvh * D);
    const unsigned char *vbase = (const unsigned char *)(v + kvh * D);
    const long kv_bytes = (long)T * ldkv * 2 - (long)kvh * D * 2;

    bf16x8 qf[D / 16], dof[D / 16];
#pragma unroll
    for (int t = 0; t < D / 16; ++t) {
        qf[t] = *(const bf16x8 *)(q + (size_t)q_row * ldq + head * D + 16 * t + 8 * lh);
        dof[t] = *(const bf16x8 *)(d_o + (size_t)q_row * ldo + head * D + 16 * t + 8 * lh);
    }
    // The row statistics of the backward: Delta = sum_d dO O and the log-sum-exp in base-2 units.  The
    // wave holds its rows of dO already; each lane adds its half of the row, the other half sits 32
    // lanes away.  Both are also written out: the dK / dV kernel, launched behind this one, reads them.
    const float lse2 = lse[(size_t)head * T + q_row] * LOG2E;
    float dlt = 0.f;
#pragma unroll
    for (int t = 0; t < D / 16; ++t) {
        const bf16x8 of = *(const bf16x8 *)(o + (size_t)q_row * ldo + head * D + 16 * t + 8 * lh);
#pragma unroll
        for (int e = 0; e < 8; ++e) dlt += (float)dof[t][e] * (float)of[e];
    }
    dlt = sum_halves(dlt);
    if (q_live && lh == 0) {
        lse2_all[(size_t)head * T + q_row] = lse2;
        delta[(size_t)head * T + q_row] = dlt;
    }
    f32x16 acc_dq[DT];
#pragma unroll
    for (int i = 0; i < DT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_dq[i][r] = 0.f;

    const int kv_end = CAUSAL ? min(ti.seg_end, ti.row0 + QT) : ti.seg_end;
    const int n_tiles = (kv_end - ti.seg_start + ST - 1) / ST;
    unsigned char OB_LDS *const ks0 = (unsigned char OB_LDS *)k_s0, *const ks1 = (unsigned char OB_LDS *)k_s1;
    unsigned char OB_LDS *const vs0 = (unsigned char OB_LDS *)v_s0, *const vs1 = (unsigned char OB_LDS *)v_s1;
    {
        const long off = (long)ti.seg_start * ldkv * 2;
        tl.issue(kbase + off, kv_bytes - off, ks0, wave);
        tl.issue(vbase + off, kv_bytes - off, vs0, wave);
    }
    const int n_main = CAUSAL ? (ti.row0 - ti.seg_start) / ST : (ti.seg_end - ti.seg_start) / ST;
    int j = 0;
#define OB_DQ_ITER(MASKED, KS, VS, KS_NEXT, VS_NEXT)                                                          \
    {                                                                                                        \
        const int kv0 = ti.seg_start + j * ST;                                                               \
        __builtin_amdgcn_s_waitcnt(WAIT_VM0);                                                                \
        __syncthreads();                                                                                     \
        if (j + 1 < n_tiles) {                                                                               \
            const long off = (long)(kv0 + ST) * ldkv * 2;                                                    \
            tl.issue(kbase + off, kv_bytes - off, (KS_NEXT), wave);                                          \
            tl.issue(vbase + off, kv_bytes - off, (VS_NEXT), wave);                                          \
        }                                                                                                    \
        _Pragma("unroll") for (int hf = 0; hf < 2; ++hf) {                                                   \
            const int kv_first = kv0 + 32 * hf;                                                              \
            if (!(MASKED)) {                                                                                 \
                if (wave_live)                                                                               \
                    dq_half<D, CAUSAL, false>((KS) + hf * HALF, (VS) + hf * HALF, tl, qf, dof, acc_dq, lse2,  \
                                              dlt, kv_first, ti.seg_end, q_row, sl2);                        \
            } else if (wave_live && kv_first < ti.seg_end && !(CAUSAL && kv_first > wave_q_last))            \
                dq_half<D, CAUSAL, true>((KS) + hf * HALF, (VS) + hf * HALF, tl, qf, dof, acc_dq, lse2, dlt,  \
                                         kv_first, ti.seg_end, q_row, sl2);                                  \
        }                                                                                                    \
        ++j;                                                                                                 \
    }
    while (j + 1 < n_main) {  // two tiles per trip: the stage buffers are compile-time constants
        OB_DQ_ITER(false, ks0, vs0, ks1, vs1)
        OB_DQ_ITER(false, ks1, vs1, ks0, vs0)
    }
#define OB_DQ_ANY(MASKED) OB_DQ_ITER(MASKED, (j & 1) ? ks1 : ks0, (j & 1) ? vs1 : vs0, (j & 1) ? ks0 : ks1, (j & 1) ? vs0 : vs1)
    while (j < n_main) OB_DQ_ANY(false)
    while (j < n_tiles) OB_DQ_ANY(true)
#undef OB_DQ_ANY
#undef OB_DQ_ITER
    if (!q_live) return;
    if (rot_log2_base > 0.f) rotary_bwd_row<D>(acc_dq, q_row - ti.seg_start, rot_log2_base, lh);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            bf16x4 ov;
#pragma unroll
            for (int e = 0; e < 4; ++e) ov[e] = (__bf16)(acc_dq[dt][4 * g + e] * scale);
            *(bf16x4 *)(dq + (size_t)q_row * ldq + head * D + dt * 32 + g * 8 + lh * 4) = ov;
        }
}

// ------------------------------------------------------------------------------------------------
// backward, part 2: dK, dV.  A workgroup owns 64 or 128 key rows of one head and streams the segment's
// 64- or 32-row query tiles (from the diagonal on when causal).  Its wavefronts form pairs, one
// pair per 32 key rows, and the two waves of a pair split the four products between them:
//   role P (first half of the waves):   S = Q K^T,  P = 2^(scale log2(e) S - lse2),  dV^T += dO^T P
//   role G (second half of the waves):  dP = dO V^T,  dS = P (dP - Delta),           dK^T += Q^T dS
// P travels from the first to the second through LDS in the packed operand layout both use.  Each
// wave keeps half of the state a single wave would need (so two fit on a SIMD and one's MFMAs hide
// the other's element-wise work and LDS waits), and no product is computed twice.  Both roles run
// "row-fragment tile x held rows -> 32x32 scores" and "transposed tile x packed scores -> output";
// role G does the second one tile late (see the kernel), so that it never waits for its partner.
// A wave raises its priority for its matrix products: of two waves on a SIMD the one with MFMAs to issue goes first and
// the other one's element-wise work fills the gaps (7B-shaped batch and 6B ViT tiles 1.7 %, one segment
// of 7168 2.9 %, both builds in turn; a fixed priority for either role loses, the forward and dQ gain nothing).
// ------------------------------------------------------------------------------------------------
// scores of a streamed tile of 32 MT rows against the 32 held rows: acc[mt] = rows 32 mt .. of the tile
template <int D, int MT>
__device__ __forceinline__ void dkv_scores(const unsigned char OB_LDS *__restrict__ tile, const Tile<D, 32 * MT> &tl,
                                           const bf16x8 (&held)[D / 16], f32x16 (&acc)[MT]) {
    constexpr int HB = D / 32, NB = MT * (D / 16) / HB, PER = NB / MT;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mt][r] = 0.f;
    bf16x8 fr[2][HB];
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < HB; ++i) fr[0][i] = tl.frag_row(tile, 0, i);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (b + 1 < NB) {
#pragma unroll
            for (int i = 0; i < HB; ++i)
                fr[(b + 1) & 1][i] = tl.frag_row(tile, (b + 1) / PER, ((b + 1) % PER) * HB + i);
        }
#pragma unroll
        for (int i = 0; i < HB; ++i)
            acc[b / PER] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[b & 1][i], held[(b % PER) * HB + i], acc[b / PER], 0, 0, 0);
        if (b + 1 < NB) OB_SCHED_READS_THEN_MFMA(HB, HB); else OB_SCHED_READS_THEN_MFMA(0, HB);
    }
    __builtin_amdgcn_s_setprio(0);
}

// role P: probabilities of the 32 MT x 32 score tile, packed as the second operands of the 2 MT
// 16-row contraction steps (pk[mt][h] serves step 2 mt + h)
template <bool CAUSAL, bool MASK, int MT>
__device__ __forceinline__ void dkv_probs(const f32x16 (&s)[MT], const unsigned char OB_LDS *__restrict__ lse2_s,
                                          int q0, int seg_end, int kv_row, float sl2, bf16x8 (&pk)[MT][2]) {
    const int lh = (threadIdx.x & 63) >> 5;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        f32x16 p;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 l4 = lds16<f32x4>(lse2_s + (mt * 32 + 8 * g + 4 * lh) * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                bool ok = true;
                if (MASK) {
                    const int qr = q0 + mt * 32 + 8 * g + 4 * lh + e;
                    ok = qr < seg_end && (!CAUSAL || kv_row <= qr);
                }
                const float pe = fast_exp2(s[mt][4 * g + e] * sl2 - l4[e]);
                p[4 * g + e] = ok ? pe : 0.f;
            }
        }
        pk[mt][0] = pack8(p, 0);
        pk[mt][1] = pack8(p, 8);
    }
}

// role G: dS = P (dP - Delta), in place of the packed probabilities
template <int MT>
__device__ __forceinline__ void dkv_dscores(const f32x16 (&dp)[MT], const unsigned char OB_LDS *__restrict__ dlt_s,
                                            bf16x8 (&pk)[MT][2]) {
    const int lh = (threadIdx.x & 63) >> 5;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        f32x16 ds;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 d4 = lds16<f32x4>(dlt_s + (mt * 32 + 8 * g + 4 * lh) * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = 4 * g + e;
                ds[r] = (float)pk[mt][r >> 3][r & 7] * (dp[mt][r] - d4[e]);
            }
        }
        pk[mt][0] = pack8(ds, 0);
        pk[mt][1] = pack8(ds, 8);
    }
}

// out^T += tile^T x packed scores, contracting over the tile's rows
template <int D, int MT>
__device__ __forceinline__ void dkv_outputs(const unsigned char OB_LDS *__restrict__ tile, const Tile<D, 32 * MT> &tl,
                                            const bf16x8 (&pk)[MT][2], f32x16 (&acc_out)[D / 32]) {
    constexpr int DT = D / 32;
    bf16x8 tf[2][DT];
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) tf[0][dt] = tl.frag_tr(tile, dt, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 2 * MT; ++u) {
        if (u + 1 < 2 * MT) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) tf[(u + 1) & 1][dt] = tl.frag_tr(tile, dt, u + 1);
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
            acc_out[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tf[u & 1][dt], pk[u >> 1][u & 1], acc_out[dt], 0, 0, 0);
        if (u + 1 < 2 * MT) OB_SCHED_READS_THEN_MFMA(2 * DT, DT); else OB_SCHED_READS_THEN_MFMA(0, DT);
    }
    __builtin_amdgcn_s_setprio(0);
}

// role P: the products of dkv_outputs (probabilities pk of the tile before), the probabilities of the tile at hand between them:
// two products, their operands read two products ahead, to 16 / D x 16 values per lane
template <int D, int MT>
__device__ __forceinline__ void dkv_outputs_probs(const unsigned char OB_LDS *__restrict__ tile, const Tile<D, 32 * MT> &tl,
                                                  const bf16x8 (&pk)[MT][2], f32x16 (&acc_out)[D / 32], const f32x16 (&s)[MT],
                                                  const unsigned char OB_LDS *__restrict__ lse2_s, float sl2, bf16x8 (&pn)[MT][2]) {
    constexpr int DT = D / 32, PER = DT / 2, NB = 2 * MT * PER, EL = 8 / PER;      // batches of two products; values per lane and batch
    const int lh = (threadIdx.x & 63) >> 5;
    bf16x8 tf[2][2];
    f32x4 l4[2][EL / 4];
    auto read = [&](int b) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) tf[b & 1][i] = tl.frag_tr(tile, 2 * (b % PER) + i, b / PER);
#pragma unroll
        for (int g = 0; g < EL / 4; ++g) l4[b & 1][g] = lds16<f32x4>(lse2_s + (2 * EL * b + 8 * g + 4 * lh) * 4);
    };
    read(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int u = b / PER, e0 = (b % PER) * EL;
        if (b + 1 < NB) read(b + 1);
#pragma unroll
        for (int e = 0; e < EL; ++e)
            pn[u >> 1][u & 1][e0 + e] = (__bf16)fast_exp2(s[u >> 1][8 * (u & 1) + e0 + e] * sl2 - l4[b & 1][e >> 2][e & 3]);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int dt = 2 * (b % PER) + i;
            acc_out[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tf[b & 1][i], pk[u >> 1][u & 1], acc_out[dt], 0, 0, 0);
        }
        if (b + 1 < NB) __builtin_amdgcn_sched_group_barrier(0x100, 4 + EL / 4, 0);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, EL * 5 / 4, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// role G: the products of dkv_scores, dS = P (dP - Delta) of the tile before, in place of its probabilities pk, between them
template <int D, int MT>
__device__ __forceinline__ void dkv_scores_dscores(const unsigned char OB_LDS *__restrict__ tile, const Tile<D, 32 * MT> &tl,
                                                   const bf16x8 (&held)[D / 16], f32x16 (&acc)[MT], const f32x16 (&dp)[MT],
                                                   const unsigned char OB_LDS *__restrict__ dlt_s, bf16x8 (&pk)[MT][2]) {
    constexpr int KT = D / 16, PER = KT / 2, NB = MT * PER, EL = 16 * MT / NB;       // batches of two products; values per lane and batch
    const int lh = (threadIdx.x & 63) >> 5;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mt][r] = 0.f;
    bf16x8 fr[2][2];
    f32x4 d4[2][EL / 4];
    auto read = [&](int b) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) fr[b & 1][i] = tl.frag_row(tile, b / PER, 2 * (b % PER) + i);
#pragma unroll
        for (int g = 0; g < EL / 4; ++g) d4[b & 1][g] = lds16<f32x4>(dlt_s + (2 * EL * b + 8 * g + 4 * lh) * 4);
    };
    read(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (b + 1 < NB) read(b + 1);
#pragma unroll
        for (int e = 0; e < EL; ++e) {
            const int r = EL * b + e, mt = r >> 4;                          // accumulator register r % 16 of row tile mt
            const float p = (float)pk[mt][(r >> 3) & 1][r & 7];
            pk[mt][(r >> 3) & 1][r & 7] = (__bf16)(p * (dp[mt][r & 15] - d4[b & 1][e >> 2][e & 3]));
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
            acc[b / PER] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[b & 1][i], held[2 * (b % PER) + i], acc[b / PER], 0, 0, 0);
        if (b + 1 < NB) __builtin_amdgcn_sched_group_barrier(0x100, 2 + EL / 4, 0);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, EL * 7 / 4, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// dK / dV comes in three shapes per head size (NP pairs of waves, each pair owning 32 key rows, query tiles of SR rows; or blocks, a
// kernel of its own further down), of which dkv_shape() takes the one its estimate of the launch favours:
//  * D = 64: two pairs, so that workgroups which nothing synchronises share a CU and a 1025-row segment wastes
//    6 % of the rows (six pairs in step: 12 %).  SR = 32 needs 34 KB of LDS and under 128 registers: four
//    workgroups to the CU, the better rate when the chip is full (12 ViT tiles x 16 heads: 128 us, against 140
//    with SR = 64 and 161 for six pairs).  SR = 64 has half the barriers and stage switches to a row, and as a wave has its SIMD nearly to
//    itself its element-wise work goes between its own products: the shorter
//    chain when one long segment keeps the launch waiting (texts of 8187 tokens in all, 16 / 4 heads: 92 us, SR = 32 114;
//    with the element-wise work in a stretch of its own 110).  Six pairs remain for bidirectional launches that two pairs would need a second round
//    for (one segment of 4097, 8 heads in groups of 6: 539 us, against 568 with SR = 32).
//  * D = 128: four pairs on one CU, eight waves in step, the better rate when the chip is full (texts of
//    16384 tokens, 32 / 8 heads, and other batches of its size: 612 us, blocks 776); blocks for launches that wait for their longest walk; two pairs,
//    bidirectional, one trip less from scores to results, for walks of a few tiles (one segment of 64, 8 heads: 8.9 us, blocks 9.9; of 320, 25 heads
//    15.0 and 15.5).
// All shapes of a head size add up the query rows of a key row in the same order, set by DKV_ORDER_Q and (causal) the
// place in whole tiles of dkv_whole() key rows: which of them runs does not show in the result, so a packed batch
// still gives bit for bit what its segments give alone.
constexpr int DKV_ORDER_Q = 64;   // the ragged end of the query rows is one masked step of up to this many rows
constexpr int dkv_whole(int d) { return d == 64 ? 64 : 128; }

// The query tiles that a workgroup of dK / dV walks, in the order of work: the masked ones (causal: on the diagonal; either way the
// ragged end) of every query head of the group, then the mask-free ones of every head -- the sums do not care, and one loop per kind keeps
// the accumulators in place.  `dead`: causal query rows before the whole's first key row see none of its keys; a part's dead tiles lie
// before its own first key row and are left out.
template <int D, bool CAUSAL, int KVT, int SR>
struct DkvWalk {
    static constexpr int WHOLE = CAUSAL ? dkv_whole(D) : KVT;    // key rows of the whole that the workgroup's may be a part of
    static_assert(WHOLE % KVT == 0 && KVT % SR == 0, "parts of whole tiles");
    int q_begin, dead, n_head, n_diag, n_end, n_mid, n_masked, n_all;
    __device__ __forceinline__ DkvWalk(const TileInfo &ti, int group) {
        const int whole_row0 = ti.row0 - (ti.row0 - ti.seg_start) % WHOLE;
        q_begin = CAUSAL ? whole_row0 : ti.seg_start;
        dead = CAUSAL ? (ti.row0 - whole_row0) / SR : 0;
        const int n_iter = (ti.seg_end - q_begin + SR - 1) / SR;
        // causal: only the first WHOLE / SR query tiles touch some key's diagonal; either way only the last
        // tile can be ragged.  The tiles in between need no mask.
        n_head = CAUSAL ? min(WHOLE / SR, n_iter) : 0;
        const int n_mid_end = max(n_head, (ti.seg_end - q_begin) / DKV_ORDER_Q * (DKV_ORDER_Q / SR));
        n_diag = n_head - dead;
        n_end = n_iter - n_mid_end;
        n_mid = n_mid_end - n_head;
        n_masked = group * (n_diag + n_end);
        n_all = n_masked + group * n_mid;
    }
    // first query row of masked tile j of a head
    __device__ __forceinline__ int masked_row(int j) const {
        const int diag = dead + j, end = n_head + n_mid + j - n_diag;
        return q_begin + (j < n_diag ? diag : end) * SR;
    }
};

// One wave's requests for them: LD pieces of each tile (1 KB apiece) and, global -> LDS as well, the tile's row statistics.  The order of
// work is runs of consecutive tiles: per head the diagonal and the ragged end, then per head what lies between.  A descriptor serves
// a run (or dkv_run() tiles of it, so that the offsets inside stay below 2^32) and a lane's offsets advance, a handful of instructions per
// tile where making descriptors anew took a hundred, as long as four products, in front of every tile's first one (with the loads as
// instructions of their own, see load_lds16(), 7B-shaped batch 667 -> 612 us, 16 tiles of the 6B ViT 636 -> 596, 12 of the 300M ViT 148 -> 138).  APART: for rows of which not even one tile fits, each piece has a descriptor
// of its own and the lanes' offsets count from the piece's first row.
template <int D, bool CAUSAL, int KVT, int SR, int LD, int SKIP = LD, bool APART = false>
struct DkvRequests {
    const DkvWalk<D, CAUSAL, KVT, SR> &w;
    const unsigned char *base;
    const float *stat_base;
    long ld2;                     // bytes from row to row
    int T, head0, group, piece0;  // the wave's first piece
    uint32_t (&first)[LD], voff[LD], stat_voff;
    int n_issued, run_left, part_left, part_row, part_head, next_part, next_head;
    u32x4 rsrc, stat_rsrc;
    __device__ __forceinline__ DkvRequests(const DkvWalk<D, CAUSAL, KVT, SR> &walk, const void *base_, long ld2_, const float *stat_, int T_,
                                           int head0_, int group_, int piece0_, uint32_t (&first_)[LD])
        : w(walk), base((const unsigned char *)base_), stat_base(stat_), ld2(ld2_), T(T_), head0(head0_), group(group_), piece0(piece0_), first(first_),
          stat_voff(0), n_issued(0), run_left(0), part_left(0), part_row(0), part_head(0),
          next_part(walk.n_masked == 0 ? 2 : walk.n_diag > 0 ? 0 : 1), next_head(0),
          rsrc{0, 0, 0, 0}, stat_rsrc{0, 0, 0, 0} {}
    __device__ __forceinline__ void next_run(int lane) {
        if (part_left == 0) {                          // (only called while there are tiles left)
            const int f0 = w.dead, f1 = w.n_head + w.n_mid, f2 = w.n_head, c0 = w.n_diag, c1 = w.n_end, c2 = w.n_mid;
            const int part = next_part;
            part_row = w.q_begin + (part == 0 ? f0 : part == 1 ? f1 : f2) * SR;
            part_left = part == 0 ? c0 : part == 1 ? c1 : c2;
            part_head = head0 + next_head;
            const bool same = part == 0 && c1 > 0, last = next_head + 1 == group;
            next_part = same ? 1 : part == 2 || last ? 2 : c0 > 0 ? 0 : 1;
            next_head = same ? next_head : last ? 0 : next_head + 1;
        }
        run_left = APART ? 1 : min(part_left, dkv_run((uint32_t)ld2, SR));
        const long off = (long)part_row * ld2 + (long)part_head * D * 2;
        rsrc = make_rsrc(base + off, (long)T * ld2 - off);
        stat_rsrc = make_rsrc(stat_base + (size_t)part_head * T + part_row, (long)(T - part_row) * 4);
#pragma unroll
        for (int p = 0; p < LD; ++p) voff[p] = first[p];
        stat_voff = lane * 4;
        part_left -= run_left;
        part_row += run_left * SR;
    }
    // APART: the wave's pieces of the tile that next_run() has come to
    template <int P = 0>
    __device__ __forceinline__ void issue_apart(unsigned char OB_LDS *pieces) {
        const int in_tile = (piece0 + (P < SKIP ? P : P + SKIP)) * Tile<D, SR>::RPI;      // the piece's first row
        const long off = (long)(part_row - SR + in_tile) * ld2 + (long)part_head * D * 2;
        voff[P] = dkv_piece_offset(first[P], in_tile, (uint32_t)ld2);
        load_lds16<1, SKIP, P>(make_rsrc(base + off, (long)T * ld2 - off), pieces, voff);
        if constexpr (P + 1 < LD) issue_apart<P + 1>(pieces);
    }
    // the next tile: the wave's pieces of it to `pieces`, if `copies`; its statistics to stat, if `stats`
    __device__ __forceinline__ void issue(unsigned char OB_LDS *pieces, bool copies, unsigned char OB_LDS *stat, bool stats, int lane) {
        if (n_issued >= w.n_all) return;
        if (run_left == 0) next_run(lane);
        if constexpr (APART) {
            if (copies) issue_apart(pieces);
        } else if (copies) {
            load_lds16<LD, SKIP>(rsrc, pieces, voff);
#pragma unroll
            for (int p = 0; p < LD; ++p) voff[p] += (uint32_t)(SR * ld2);
        }
        if (stats) load_lds4(stat_rsrc, stat, stat_voff);
        stat_voff += SR * 4;
        --run_left;
        ++n_issued;
    }
};

template <int D, bool CAUSAL, int NP, int SR, bool APART = false>
__global__ __launch_bounds__(128 * NP, D == 128 || NP == 6 ? 1 : SR == 32 ? 4 : 2) void attn_bwd_dkv_kernel(
    const __bf16 *__restrict__ d_o, const __bf16 *__restrict__ q, const __bf16 *__restrict__ k,
    const __bf16 *__restrict__ v, const float *__restrict__ lse2_all, const float *__restrict__ delta,
    __bf16 *__restrict__ dk, __bf16 *__restrict__ dv, int ldq, int ldkv, int ldo,
    const int32_t *__restrict__ cu, int n_seg, int T, int group, float scale, float rot_log2_base, int heads,
    TileOrder ord) {
    // three stages of the streamed Q and dO tiles (the results are formed one tile behind the scores, see
    // below), two buffers for the probabilities on their way from one role to the other, row statistics
    __shared__ __attribute__((aligned(1024))) unsigned char tiles_s[6 * Tile<D, SR>::BYTES];
    constexpr int KVT = 32 * NP, MT = SR / 32, PB = MT * 2048;
    __shared__ __attribute__((aligned(1024))) unsigned char p_s[2 * NP * PB];  // [buffer][pair]: 2 MT x 64 lanes x 16 B
    __shared__ __attribute__((aligned(256))) unsigned char stat_s[6 * 256];    // lse2 x 3 stages, Delta x 3 stages
    __shared__ int sh[8];
    const int rank = blockIdx.x / heads;
    const TileInfo ti = pick_tile<true>(ord, rank, cu, n_seg, KVT, sh);
    if (ti.row0 < 0) return;
    // one workgroup per key/value head: the group's query heads run one after another
    const int kvh = head_of_slot(blockIdx.x - rank * heads, heads);
    const int lane = threadIdx.x & 63, lx = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool role_g = wave >= NP;  // false: S, P, dV;  true: dP, dS, dK
    const int pair = role_g ? wave - NP : wave;
    const int kv_row = min(ti.row0 + pair * 32 + lx, ti.seg_end - 1);
    const bool kv_live = ti.row0 + pair * 32 + lx < ti.seg_end;
    const int pair_kv_first = ti.row0 + pair * 32;
    const float sl2 = scale * LOG2E;
    constexpr int KT = D / 16, DT = D / 32;
    constexpr bool FUSE = NP == 2 && SR == 64;      // one or two waves to a SIMD: element-wise work between the wave's own products

    // the wave copies the tile it reads row fragments from: Q (role P) or dO (role G)
    Tile<D, SR> tl;
    tl.init(role_g ? ldo : ldq, pair, lane);
    f32x16 acc_out[DT];  // dV^T (role P) or dK^T (role G)
#pragma unroll
    for (int i = 0; i < DT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_out[i][r] = 0.f;

    constexpr int BYTES = Tile<D, SR>::BYTES;

    const DkvWalk<D, CAUSAL, KVT, SR> w(ti, group);

    // the whole walk once per role, chosen outside the loops: each role's loop then carries only its own registers
    auto walk = [&](auto role_tag) __attribute__((always_inline)) {
    constexpr bool RG = decltype(role_tag)::value;
    unsigned char OB_LDS *const tiles = (unsigned char OB_LDS *)tiles_s;
    // (where in the array a role's two rings start is part of every lane's offsets: what is added per stage and row tile fits an
    // instruction's 16-bit offset)
    constexpr int OWN_AT = RG ? 3 * BYTES : 0, OTHER_AT = RG ? 0 : 3 * BYTES;
#pragma unroll
    for (int t = 0; t < KT; ++t) tl.rr[t] += OWN_AT;
#pragma unroll
    for (int i = 0; i < 2 * DT; ++i) tl.tro[i / DT][i % DT] += OTHER_AT;
    unsigned char OB_LDS *const stat = (unsigned char OB_LDS *)stat_s + (RG ? 3 * 256 : 0);
    unsigned char OB_LDS *const p_mine = (unsigned char OB_LDS *)p_s + pair * PB + lane * 16;
    // four waves of a role copy a tile, or two half of it each
    constexpr int TLD = Tile<D, SR>::LD, LDW = NP == 2 ? 2 * TLD : TLD;
    const long ld2 = (RG ? (long)ldo : (long)ldq) * 2;
    uint32_t first[LDW];
#pragma unroll
    for (int p = 0; p < LDW; ++p) first[p] = tl.voff[p % TLD] + (p < TLD ? 0u : (uint32_t)(SR / 2 * ld2));
    unsigned char OB_LDS *const pieces = tiles + OWN_AT + pair * TLD * 1024;
    DkvRequests<D, CAUSAL, KVT, SR, LDW, TLD, APART> req(w, RG ? d_o : q, ld2, RG ? delta : lse2_all, T, kvh * group, group, pair * TLD, first);
    auto request = [&](int stage) __attribute__((always_inline)) {
        req.issue(pieces + stage * BYTES, pair < 4, stat + stage * 256, pair == 0, lane);
    };
    request(0);
    bf16x8 kvf[KT];     // held rows: K (role P) or V (role G)
    {
        const __bf16 *src = (RG ? v : k) + (size_t)kv_row * ldkv + kvh * D + 8 * lh;
#pragma unroll
        for (int t = 0; t < KT; ++t) kvf[t] = *(const bf16x8 *)(src + 16 * t);
    }
#pragma unroll
    for (int t = 0; t < KT; ++t) asm volatile("" : "+v"(kvf[t]));      // have landed: no wait for them inside the loops

    // The dK side runs one tile behind: in the trip of tile n the role-P wave does S, P, dV of tile n
    // and leaves P in buffer n % 2, while the role-G wave first finishes tile n - 1 (dS from the P it
    // finds in buffer (n - 1) % 2 and the dP it kept in registers, then dK) and then forms dP of tile
    // n.  One barrier per tile, the role-G wave never waits for its partner inside a
    // trip, and the two waves of a SIMD start a trip in different kinds of work (MFMAs / element-wise).
    // FUSE: over the mask-free tiles dV runs one tile behind as well, P of tile n between its products, and dS of tile n - 1 goes between
    // those of dP of tile n.
    // Stage n % 3 holds tile n: the load of tile n + 1 overwrites tile n - 2, which nobody needs any more.
    int n = 0, q0 = 0, m_j = 0;
    bool live_prev = false, owed = false;      // tile n - 1 took part; (role P) its dV is still to come
    bf16x8 pk[MT][2];            // role P: P of tile n - 1
    f32x16 dp_keep[MT];          // role G: dP of tile n - 1
    auto trip = [&](auto general_tag, auto masked_tag, int S, int PREV, int NEXT, bool owe) __attribute__((always_inline)) {
        constexpr bool GEN = decltype(general_tag)::value, MASK = decltype(masked_tag)::value;
        __builtin_amdgcn_s_waitcnt(wait_vm_lds0(0));
        bare_barrier();
        if (GEN) request(NEXT);      // (the masked tiles' trips are short and each takes a descriptor of its own)
        // (GEN: one after the other, each step behind a test)  a masked tile entirely before this pair's keys contributes nothing
        const bool live = !GEN || (n < w.n_all && !(MASK && CAUSAL && q0 + SR - 1 < pair_kv_first));
        unsigned char OB_LDS *const p_new = p_mine + (n & 1) * (NP * PB), *const p_old = p_mine + ((n & 1) ^ 1) * (NP * PB);
        const bool late = !GEN || (RG ? live_prev : owed);
        if constexpr (!RG) {
            f32x16 acc_x[MT];
            if (live) dkv_scores<D, MT>(tiles + S * BYTES, tl, kvf, acc_x);
            if (!GEN) request(NEXT);
            if constexpr (FUSE && !GEN) {
                bf16x8 pn[MT][2];
                dkv_outputs_probs<D, MT>(tiles + PREV * BYTES, tl, pk, acc_out, acc_x, stat + S * 256, sl2, pn);
#pragma unroll
                for (int i = 0; i < 2 * MT; ++i) pk[i >> 1][i & 1] = pn[i >> 1][i & 1];
            } else {
                if (FUSE && late) dkv_outputs<D, MT>(tiles + PREV * BYTES, tl, pk, acc_out);
                if (live) dkv_probs<CAUSAL, MASK, MT>(acc_x, stat + S * 256, q0, ti.seg_end, kv_row, sl2, pk);
            }
            if (live) {
#pragma unroll
                for (int i = 0; i < 2 * MT; ++i) *(bf16x8 OB_LDS *)(p_new + i * 1024) = pk[i >> 1][i & 1];
                if (GEN || !FUSE) {
                    if (!owe) dkv_outputs<D, MT>(tiles + S * BYTES, tl, pk, acc_out);
                }
            }
            owed = owe && live;
        } else {
            bf16x8 pn[MT][2];
            if (late) {
#pragma unroll
                for (int i = 0; i < 2 * MT; ++i) pn[i >> 1][i & 1] = lds16<bf16x8>(p_old + i * 1024);
            }
            if constexpr (FUSE && !GEN) {
                f32x16 acc_x[MT];
                dkv_scores_dscores<D, MT>(tiles + S * BYTES, tl, kvf, acc_x, dp_keep, stat + PREV * 256, pn);
                request(NEXT);
                dkv_outputs<D, MT>(tiles + PREV * BYTES, tl, pn, acc_out);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) dp_keep[mt] = acc_x[mt];
            } else {
                if (late) {
                    dkv_dscores<MT>(dp_keep, stat + PREV * 256, pn);
                    dkv_outputs<D, MT>(tiles + PREV * BYTES, tl, pn, acc_out);
                }
                if (!GEN) request(NEXT);
                if (live) dkv_scores<D, MT>(tiles + S * BYTES, tl, kvf, dp_keep);
            }
        }
        live_prev = live;
        ++n;
    };
    int st = 0;
    auto slow = [&](auto masked_tag, bool owe) __attribute__((always_inline)) {
        const int s_ = st, p_ = st == 0 ? 2 : st - 1, n_ = st == 2 ? 0 : st + 1;
        trip(std::true_type{}, masked_tag, s_, p_, n_, owe);
        st = n_;
    };
    while (n < w.n_masked) {
        q0 = w.masked_row(m_j);
        if (++m_j == w.n_diag + w.n_end) m_j = 0;
        slow(std::true_type{}, false);
    }
    // The mask-free tiles: three to a trip, constant stage addresses, a single straight path, from a tile on stage 0 on; where the
    // products of dV lag behind, the tile in front of them leaves its own to the first of them.
    const int lead = !FUSE && live_prev && n % 3 == 0 ? n : n + 3 - n % 3;      // the first tile of the first three (never the very first)
    const bool threes = !APART && lead + 3 <= w.n_all;      // (APART: rare, in the small form)
    while (threes && n < lead) slow(std::false_type{}, FUSE && n + 1 == lead);
    while (threes && n + 3 <= w.n_all) {
        trip(std::false_type{}, std::false_type{}, 0, 2, 1, FUSE);
        trip(std::false_type{}, std::false_type{}, 1, 0, 2, FUSE);
        trip(std::false_type{}, std::false_type{}, 2, 1, 0, FUSE);
    }
    while (n <= w.n_all) slow(std::false_type{}, false);
    };
    if (role_g) walk(std::true_type{}); else walk(std::false_type{});
    if (!kv_live) return;
    // dV^T / dK^T of the whole group of query heads sit in the accumulators: one rounding to bf16
    const float out_scale = role_g ? scale : 1.0f;
    __bf16 *const dst = role_g ? dk : dv;
    if (role_g && rot_log2_base > 0.f) rotary_bwd_row<D>(acc_out, kv_row - ti.seg_start, rot_log2_base, lh);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            bf16x4 ov;
#pragma unroll
            for (int e = 0; e < 4; ++e) ov[e] = (__bf16)(acc_out[dt][4 * g + e] * out_scale);
            *(bf16x4 *)(dst + (size_t)kv_row * ldkv + kvh * D + dt * 32 + g * 8 + lh * 4) = ov;
        }
}

// ------------------------------------------------------------------------------------------------
// dK / dV of 64 key rows of a head of 128 by eight waves, for launches whose longest walk keeps everything waiting.  A
// trip (one query tile of 64 rows) is half the work of a trip of four pairs, and all of it is dealt to the eight waves in 32 x 32 blocks:
// query half a and key half b of S (four waves of role P) and of dP (four of role G), columns 32 a and 32 a + 64 of key half b of dV (P)
// and of dK (G).  Nothing in a trip waits for anything of the same trip but a wave's own scores:
//   role P: S of tile n;  P of tile n between the products of dV of tile n - 1
//   role G: dP of tile n;  dS of tile n - 1 between the products of dK of tile n - 2
// P and dS go through LDS in the packed operand layout, two buffers each; Q has four stages and dO three.  What bounds a
// trip is the LDS: reads at 256 bytes per clock, writes at 79, 1500 clocks of a trip's 2500 (its products take 1024 of a SIMD's).
// Against two pairs (four waves that take both blocks of a key half), causal and bidirectional: one segment of 557, 32 / 8 heads 54 -> 44 and 47 -> 40 us, of
// 2000 147 -> 118 and 148 -> 140, of 2000, 12 / 2 heads 214 -> 171 and 203 -> 176 (before the requests had running descriptors two pairs took 61, 187 and
// 271, causal); a full chip is better off with four pairs (16384 tokens, 32 / 8 heads 612 us, here 776).
// The sums are those of the other shapes, in their order.
// ------------------------------------------------------------------------------------------------
struct DkvBlocks {
    static constexpr int D = 128, SR = 64, KVT = 64, Q_STAGES = 4, DO_STAGES = 3, LSE_STAGES = 2, DLT_STAGES = 3;
    static constexpr int BYTES = Tile<D, SR>::BYTES, BLK = 2048, BUF = 4 * BLK;      // a packed 32 x 32 block, the four of a tile
    static constexpr int Q_AT = 0, DO_AT = Q_STAGES * BYTES, P_AT = DO_AT + DO_STAGES * BYTES, DS_AT = P_AT + 2 * BUF,
                         LSE_AT = DS_AT + 2 * BUF, DLT_AT = LSE_AT + LSE_STAGES * 256, TOTAL = DLT_AT + DLT_STAGES * 256;
    static_assert(TOTAL + 64 <= 160 * 1024, "LDS");
};
template <bool CAUSAL>
__global__ __launch_bounds__(512, 2) void attn_bwd_dkv_blocks_kernel(
    const __bf16 *__restrict__ d_o, const __bf16 *__restrict__ q, const __bf16 *__restrict__ k,
    const __bf16 *__restrict__ v, const float *__restrict__ lse2_all, const float *__restrict__ delta,
    __bf16 *__restrict__ dk, __bf16 *__restrict__ dv, int ldq, int ldkv, int ldo,
    const int32_t *__restrict__ cu, int n_seg, int T, int group, float scale, float rot_log2_base, int heads,
    TileOrder ord) {
    using B = DkvBlocks;
    constexpr int D = B::D, SR = B::SR, KT = D / 16, BUF = B::BUF, LD = Tile<D, SR>::LD;
    __shared__ __attribute__((aligned(1024))) unsigned char lds_s[B::TOTAL];
    __shared__ int sh[8];
    unsigned char OB_LDS *const lds = (unsigned char OB_LDS *)lds_s;
    const int rank = blockIdx.x / heads;
    const TileInfo ti = pick_tile<true>(ord, rank, cu, n_seg, B::KVT, sh);
    if (ti.row0 < 0) return;
    const int kvh = head_of_slot(blockIdx.x - rank * heads, heads);
    const int lane = threadIdx.x & 63, lx = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool role_g = wave >= 4;
    const int w4 = wave & 3, a = w4 & 1, b = w4 >> 1;
    const int kv_row = min(ti.row0 + b * 32 + lx, ti.seg_end - 1);
    const bool kv_live = ti.row0 + b * 32 + lx < ti.seg_end;
    const float sl2 = scale * LOG2E;

    Tile<D, SR> tl;
    tl.init(role_g ? ldo : ldq, w4, lane);
    int tro[2][2], rr[KT];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int s = 0; s < 2; ++s) tro[s][i] = Tile<D, SR>::tr_offset(lane, s, a + 2 * i);
#pragma unroll
    for (int t = 0; t < KT; ++t) rr[t] = tl.rr[t] + a * 32 * Tile<D, SR>::RB;
    f32x16 acc_out[2];     // columns 32 (a + 2 i) .. of dV^T (role P) or dK^T (role G)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_out[i][r] = 0.f;
    const DkvWalk<D, CAUSAL, B::KVT, SR> w(ti, group);

    auto walk = [&](auto role_tag) __attribute__((always_inline)) {
    constexpr bool RG = decltype(role_tag)::value;
    constexpr int OWN_STAGES = RG ? B::DO_STAGES : B::Q_STAGES, OTHER_STAGES = RG ? B::Q_STAGES : B::DO_STAGES;
    constexpr int STAT_STAGES = RG ? B::DLT_STAGES : B::LSE_STAGES;
    unsigned char OB_LDS *const own = lds + (RG ? B::DO_AT : B::Q_AT);         // operand of the scores: dO (G), Q (P)
    unsigned char OB_LDS *const other = lds + (RG ? B::Q_AT : B::DO_AT);       // operand of the result
    unsigned char OB_LDS *const stat = lds + (RG ? B::DLT_AT : B::LSE_AT);
    unsigned char OB_LDS *const p_blk = lds + B::P_AT + (b * 2 + a) * B::BLK + lane * 16;       // own block of the scores
    unsigned char OB_LDS *const ds_blk = lds + B::DS_AT + (b * 2 + a) * B::BLK + lane * 16;
    unsigned char OB_LDS *const out_blk = lds + (RG ? B::DS_AT : B::P_AT) + b * 2 * B::BLK + lane * 16;   // the four steps of a result
    DkvRequests<D, CAUSAL, B::KVT, SR, LD> req(w, RG ? d_o : q, (RG ? (long)ldo : (long)ldq) * 2, RG ? delta : lse2_all, T, kvh * group, group,
                                              w4 * LD, tl.voff);
    auto next = [](int stage, int stages) __attribute__((always_inline)) { return stage + 1 == stages ? 0 : stage + 1; };
    int st_issue = 0, st_stat_issue = 0;                                       // stages of the tile to request next
    auto request = [&]() __attribute__((always_inline)) {
        req.issue(own + st_issue * B::BYTES + w4 * LD * 1024, true, stat + st_stat_issue * 256, true, lane);
        st_issue = next(st_issue, OWN_STAGES);
        st_stat_issue = next(st_stat_issue, STAT_STAGES);
    };
    request();
    bf16x8 kvf[KT];     // held rows: K (role P) or V (role G)
    {
        const __bf16 *src = (RG ? v : k) + (size_t)kv_row * ldkv + kvh * D + 8 * lh;
#pragma unroll
        for (int t = 0; t < KT; ++t) kvf[t] = *(const bf16x8 *)(src + 16 * t);
    }
#pragma unroll
    for (int t = 0; t < KT; ++t) asm volatile("" : "+v"(kvf[t]));      // have landed: no wait for them inside the loops
    // stages: of the tile whose scores are formed, of its row statistics (G: of the tile before), of the tile whose share of the
    // result is formed
    int st_own = 0, st_stat = 0, st_other = 0;
    f32x16 dp_keep;     // role G: dP of tile n - 1
#pragma unroll
    for (int r = 0; r < 16; ++r) dp_keep[r] = 0.f;
    int n = 0, q0 = 0, m_j = 0;
    // GEN: each step behind a test (the first trips, in which there is nothing to finish yet, and the last)
    auto trip = [&](auto general_tag, auto masked_tag) __attribute__((always_inline)) {
        constexpr bool GEN = decltype(general_tag)::value, MASK = decltype(masked_tag)::value;
        __builtin_amdgcn_s_waitcnt(wait_vm_lds0(0));
        bare_barrier();
        if (GEN) request();
        const bool has_score = !GEN || n < w.n_all;
        const bool has_late = !GEN || (n >= 1 && n <= w.n_all);                       // dV, dS of tile n - 1
        const bool has_out = RG ? !GEN || (n >= 2 && n <= w.n_all + 1) : has_late, has_elem = RG ? has_late : has_score;
        const unsigned char OB_LDS *const sc = own + st_own * B::BYTES, *const ot = other + st_other * B::BYTES;
        const int buf = n & 1;
        bf16x8 fr[KT], of[4], tf[4][2], pk[2];
        f32x4 row4[4];                                                                // lse2 (P), Delta (G)
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
        if (has_score) {
#pragma unroll
            for (int t = 0; t < KT; ++t) fr[t] = lds16<bf16x8>(sc + rr[t]);
        }
        if (!GEN) __builtin_amdgcn_sched_barrier(0);
        if (has_elem) {
#pragma unroll
            for (int g = 0; g < 4; ++g) row4[g] = lds16<f32x4>(stat + st_stat * 256 + (a * 32 + 8 * g + 4 * lh) * 4);
        }
        if (RG && has_late) {
#pragma unroll
            for (int i = 0; i < 2; ++i) pk[i] = lds16<bf16x8>(p_blk + (buf ^ 1) * BUF + i * 1024);
        }
        if (has_out) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                of[u] = lds16<bf16x8>(out_blk + (RG ? buf : buf ^ 1) * BUF + u * 1024);
#pragma unroll
                for (int i = 0; i < 2; ++i) tf[u][i] = Tile<D, SR>::frag_at(ot, tro[0][i], tro[1][i], u);
            }
        }
        if (has_score) {
#pragma unroll
            for (int t = 0; t < KT; ++t) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[t], kvf[t], s, 0, 0, 0);
        }
        if (!GEN) {
            __builtin_amdgcn_sched_barrier(0);
            request();
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (has_elem) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int r = 8 * h + e, g = r >> 2;
                    if constexpr (RG) {
                        pk[h][e] = (__bf16)((float)pk[h][e] * (dp_keep[r] - row4[g][r & 3]));
                    } else {
                        const int qr = q0 + a * 32 + 8 * g + 4 * lh + (r & 3);
                        const bool ok = !MASK || (qr < ti.seg_end && (!CAUSAL || kv_row <= qr));
                        const float p = fast_exp2(s[r] * sl2 - row4[g][r & 3]);
                        pk[h][e] = (__bf16)(ok ? p : 0.f);
                    }
                }
            }
            if (has_out) {
#pragma unroll
                for (int u = 2 * h; u < 2 * h + 2; ++u)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        acc_out[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tf[u][i], of[u], acc_out[i], 0, 0, 0);
            }
            if (!GEN) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, RG ? 8 : 6, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (has_elem) {
            unsigned char OB_LDS *const dst = RG ? ds_blk + (buf ^ 1) * BUF : p_blk + buf * BUF;
#pragma unroll
            for (int i = 0; i < 2; ++i) *(bf16x8 OB_LDS *)(dst + i * 1024) = pk[i];
        }
        if (RG && has_score) dp_keep = s;
        st_own = next(st_own, OWN_STAGES);
        if (has_out) st_other = next(st_other, OTHER_STAGES);
        if (has_elem) st_stat = next(st_stat, STAT_STAGES);
        ++n;
    };
    while (n < w.n_masked) {
        q0 = w.masked_row(m_j);
        if (++m_j == w.n_diag + w.n_end) m_j = 0;
        trip(std::true_type{}, std::true_type{});
    }
    while (n < 2) trip(std::true_type{}, std::false_type{});
    while (n < w.n_all) trip(std::false_type{}, std::false_type{});
    while (n < w.n_all + 2) trip(std::true_type{}, std::false_type{});
    };
    if (role_g) walk(std::true_type{}); else walk(std::false_type{});
    if (!kv_live) return;
    const float out_scale = role_g ? scale : 1.0f;
    __bf16 *const dst = role_g ? dk : dv;
    if (role_g && rot_log2_base > 0.f) rotary_bwd_pair<D>(acc_out[0], acc_out[1], a, kv_row - ti.seg_start, rot_log2_base, lh);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            bf16x4 ov;
#pragma unroll
            for (int e = 0; e < 4; ++e) ov[e] = (__bf16)(acc_out[i][4 * g + e] * out_scale);
            *(bf16x4 *)(dst + (size_t)kv_row * ldkv + kvh * D + (a + 2 * i) * 32 + g * 8 + lh * 4) = ov;
        }
}

// algorithmic forward FLOPs: 4 nq d sum_seg A(s), A = s^2 or s (s + 1) / 2 (causal)
double attn_flops(const ob_segments *seg, int nq, int d, bool causal) {
    double area = 0;
    for (int j = 0; j < seg->n_seg; ++j) {
        const double len = seg->cu_host[j + 1] - seg->cu_host[j];
        area += causal ? len * (len + 1) / 2 : len * len;
    }
    return 4.0 * nq * d * area;
}

// explicit instantiations (the host pass otherwise drops launch stubs of kernels reached only
// through the dispatch macro below)
#define OB_ATTN_INSTANCES(D, C)                                                                               \
    template __global__ void attn_fwd_kernel<D, C>(const __bf16 *, const __bf16 *, const __bf16 *, __bf16 *,  \
                                                   float *, int, int, int, const int32_t *, int, int, int,    \
                                                   float, int, TileOrder);                                    \
    template __global__ void attn_bwd_dq_kernel<D, C>(const __bf16 *, const __bf16 *, const __bf16 *,         \
                                                      const __bf16 *, const __bf16 *, const float *, float *, \
                                                      float *, __bf16 *, int, int, int, const int32_t *, int, \
                                                      int, int, float, float, int, TileOrder);                \
    OB_DKV_INSTANCE(D, C, dkv_np(D, 0), dkv_sr(D, 0))                                                         \
    OB_DKV_INSTANCE(D, C, dkv_np(D, 0), dkv_sr(D, 0), true)
#define OB_DKV_INSTANCE(D, C, ...)                                                                                \
    template __global__ void attn_bwd_dkv_kernel<D, C, __VA_ARGS__>(const __bf16 *, const __bf16 *, const __bf16 *,    \
                                                           const __bf16 *, const float *, const float *,      \
                                                           __bf16 *, __bf16 *, int, int, int,                 \
                                                           const int32_t *, int, int, int, float, float, int, \
                                                           TileOrder);
OB_ATTN_INSTANCES(64, true)
OB_ATTN_INSTANCES(64, false)
OB_DKV_INSTANCE(64, true, dkv_np(64, 1), dkv_sr(64, 1))
OB_DKV_INSTANCE(64, false, dkv_np(64, 1), dkv_sr(64, 1))
OB_DKV_INSTANCE(64, false, dkv_np(64, 2), dkv_sr(64, 2))
OB_DKV_INSTANCE(128, false, dkv_np(128, 2), dkv_sr(128, 2))
OB_ATTN_INSTANCES(128, true)
OB_ATTN_INSTANCES(128, false)
#define OB_BLOCKS_INSTANCE(C)                                                                                     \
    template __global__ void attn_bwd_dkv_blocks_kernel<C>(const __bf16 *, const __bf16 *, const __bf16 *,         \
                                                           const __bf16 *, const float *, const float *,      \
                                                           __bf16 *, __bf16 *, int, int, int,                 \
                                                           const int32_t *, int, int, int, float, float, int, \
                                                           TileOrder);
OB_BLOCKS_INSTANCE(true)
OB_BLOCKS_INSTANCE(false)
#undef OB_BLOCKS_INSTANCE
#undef OB_DKV_INSTANCE
#undef OB_ATTN_INSTANCES

// the kernel of each shape
template <int D, bool CAUSAL, int SHAPE> constexpr auto attn_bwd_dkv = attn_bwd_dkv_kernel<D, CAUSAL, dkv_np(D, SHAPE), dkv_sr(D, SHAPE)>;
template <bool CAUSAL> constexpr auto attn_bwd_dkv<128, CAUSAL, 1> = attn_bwd_dkv_blocks_kernel<CAUSAL>;
template <int D, bool CAUSAL> constexpr auto attn_bwd_dkv_0 = attn_bwd_dkv<D, CAUSAL, 0>;
template <int D, bool CAUSAL> constexpr auto attn_bwd_dkv_1 = attn_bwd_dkv<D, CAUSAL, 1>;
template <int D, bool CAUSAL> constexpr auto attn_bwd_dkv_apart = attn_bwd_dkv_kernel<D, CAUSAL, dkv_np(D, 0), dkv_sr(D, 0), true>;

}  // namespace

#define OB_ATTN_DISPATCH(KERNEL, GRID, THREADS, ...)                                                      \
    do {                                                                                           \
        if (d == 64 && causal)                                                                     \
            hipLaunchKernelGGL((KERNEL<64, true>), GRID, dim3(THREADS), 0, s, __VA_ARGS__);            \
        else if (d == 64)                                                                          \
            hipLaunchKernelGGL((KERNEL<64, false>), GRID, dim3(THREADS), 0, s, __VA_ARGS__);           \
        else if (causal)                                                                           \
            hipLaunchKernelGGL((KERNEL<128, true>), GRID, dim3(THREADS), 0, s, __VA_ARGS__);           \
        else                                                                                       \
            hipLaunchKernelGGL((KERNEL<128, false>), GRID, dim3(THREADS), 0, s, __VA_ARGS__);          \
    } while (0)

void launch_attn_fwd(const void *q, const void *k, const void *v, void *o, float *lse, int ldq,
                     int ldkv, int ldo, const ob_segments *seg, int nq, int nkv, int d, float scale,
                     int mask, hipStream_t s) {
    const bool causal = mask == OB_MASK_SEG_CAUSAL;
    ProfScope prof(K_ATTN_FWD, s, attn_flops(seg, nq, d, causal));
    TileOrder ord;
    const int tiles = make_order(seg, QT, causal, false, ord);
    const dim3 grid((unsigned)tiles * nq);
    OB_ATTN_DISPATCH(attn_fwd_kernel, grid, 256, (const __bf16 *)q, (const __bf16 *)k, (const __bf16 *)v,
                     (__bf16 *)o, lse, ldq, ldkv, ldo, seg->cu_dev, seg->n_seg, seg->total_tokens,
                     nq / nkv, scale, nq, ord);
}

void launch_attn_bwd(const void *d_o, const void *q, const void *k, const void *v, const void *o, const float *lse,
                     float *lse2, float *delta, void *dq, void *dk, void *dv, int ldq, int ldkv, int ldo,
                     const ob_segments *seg, int nq, int nkv, int d, float scale, int mask, float rotary_base,
                     hipStream_t s) {
    const bool causal = mask == OB_MASK_SEG_CAUSAL;
    const int T = seg->total_tokens, group = nq / nkv;
    const float rot = rotary_base > 1.f ? log2f(rotary_base) : 0.f;
    {
        // dQ = dS K: 1 of the 4 backward products; the kernel also forms Delta and the base-2 log-sum-exp
        ProfScope prof(K_ATTN_BWD_DQ, s, 0.5 * attn_flops(seg, nq, d, causal));
        TileOrder ord;
        const int tiles = make_order(seg, QT, causal, false, ord);
        const dim3 grid_q((unsigned)tiles * nq);
        OB_ATTN_DISPATCH(attn_bwd_dq_kernel, grid_q, 256, (const __bf16 *)d_o, (const __bf16 *)q,
                         (const __bf16 *)k, (const __bf16 *)v, (const __bf16 *)o, lse, lse2, delta, (__bf16 *)dq, ldq,
                         ldkv, ldo, seg->cu_dev, seg->n_seg, seg->total_tokens, nq / nkv, scale, rot, nq, ord);
    }
    ProfScope prof(K_ATTN_BWD_DKV, s, 1.5 * attn_flops(seg, nq, d, causal));  // dV, dP, dK
    TileOrder ord;
    const int best = dkv_shape(seg, nkv, group, d, causal);
    // (in 32 bits: a stride is below 2^31 elements.  All shapes give the same bits)
    const bool apart = !dkv_tile_fits(2u * (uint32_t)(ldq > ldo ? ldq : ldo), dkv_sr(d, best));
    const int shape = apart || (causal && best == 2) ? 0 : best;      // (no causal kernel of shape 2)
    const int kvt = 32 * dkv_np(d, shape), places = make_order(seg, kvt, causal, true, ord);
    const dim3 grid_kv((unsigned)places * nkv);
#define OB_DKV_ARGS (const __bf16 *)d_o, (const __bf16 *)q, (const __bf16 *)k, (const __bf16 *)v, lse2, delta, (__bf16 *)dk,  \
                    (__bf16 *)dv, ldq, ldkv, ldo, seg->cu_dev, seg->n_seg, T, group, scale, rot, nkv, ord
    const int threads = dkv_threads(d, shape);
    if (apart) OB_ATTN_DISPATCH(attn_bwd_dkv_apart, grid_kv, threads, OB_DKV_ARGS);
    else if (shape == 0) OB_ATTN_DISPATCH(attn_bwd_dkv_0, grid_kv, threads, OB_DKV_ARGS);
    else if (shape == 1) OB_ATTN_DISPATCH(attn_bwd_dkv_1, grid_kv, threads, OB_DKV_ARGS);
    else if (d == 64) hipLaunchKernelGGL((attn_bwd_dkv<64, false, 2>), grid_kv, dim3(threads), 0, s, OB_DKV_ARGS);
    else hipLaunchKernelGGL((attn_bwd_dkv<128, false, 2>), grid_kv, dim3(threads), 0, s, OB_DKV_ARGS);
#undef OB_DKV_ARGS
}

}  // namespace ob
