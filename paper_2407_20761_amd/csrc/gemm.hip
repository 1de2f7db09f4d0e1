// bf16 MFMA GEMM for gfx950 (steps a2, a5, a7, a9 and their dgrad / wgrad counterparts).
//
//   C[M,N] = op(A) * op(B) (+ bias[N]) (+ R[M,N])      bf16 in, fp32 accumulate, bf16 out
//   "NT" A[M,K] B[N,K] (forward)   "NN" A[M,K] B[K,N] (dgrad)   "TN" A[K,M] B[K,N] (wgrad, K = tokens)
//
// One workgroup (4 wavefronts, each a 128x128 block of 8x8 MFMA 16x16x32 tiles, 256 accumulator
// registers) owns a 256x256 tile of C and walks K in steps of 32 over a ring of four LDS slots; launches
// that such tiles would leave partly idle take 192x256, 128x128 or 64x64 ones, the last two also over
// a ring of eight slots (which one, and why: estimate_us in gemm_plan.cpp).  The
// 16x16x32 shape reads and writes half the accumulator registers per FLOP of the 32x32x16 one; under
// sustained load the chip is power-limited, and a register-fed loop of it sustains 2010 against
// 1725-1790 TFLOP/s on random data.
//
// A wave has its SIMD to itself, so every instruction that is not an MFMA takes an issue slot that
// only the gaps between MFMAs can hide (three per gap), and what moves data through registers costs
// more than its slot: a 16-byte-per-lane LDS write holds the issue back for as long as its kilobyte
// takes to leave the registers (with both operands staged through registers the loop ran 7 - 12 %
// longer).  Hence
//  * every tile goes global -> LDS directly (buffer loads that write to LDS), one load per run of
//    8 MFMAs, issued one to two slots before its use;
//  * a K-major operand ([k][rows], as it lies in memory: B of "NN", both of "TN") has four slots of 32 k
//    and its fragments come out of transposing LDS reads, so dgrad and wgrad need no re-layout pass;
//  * a K-contiguous operand ([row][k]: A of "NT" and "NN", B of "NT") moves in whole 128-byte rows, two
//    slots at a time (a slot at a time it would fetch every cache line twice); a fragment is one
//    16-byte LDS read.  A has a ring of three such pairs of slots, so its loads have two slots to land;
//    B of "NT" has two (160 KB of LDS hold 96 + 64 KB), its loads go out as soon as the barrier has
//    freed their pair and have a slot and a half;
//  * the descriptor arithmetic of the next slot is a dozen scalar instructions dealt over the gaps of
//    one run (left to the compiler it was some 35 instructions with 64-bit vector compares in one
//    place, 5 % of the loop).
// The hardware range check of the buffer descriptor turns every access past the end of an operand into
// zeros: whole rows beyond M / N of a K-contiguous operand, the ragged token tail of K and slots past
// the last.  (Columns beyond M / N of a K-major operand wrap into its next row instead; they only
// feed outputs beyond M / N, which are never stored.)  16-byte chunks are XOR-swizzled on the way in
// (the global address of each lane's chunk is free to choose) so that LDS reads are bank-conflict free.
// The weight-side rows are the MFMA's first operand, so a lane's accumulators are runs of four
// consecutive output columns; the epilogue transposes them through LDS into full-row stores.
#include <type_traits>

#include "act.h"
#include "gemm_plan.h"
#include "ob_internal.h"

namespace ob {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;

namespace {

#define OB_LDS __attribute__((address_space(3)))

constexpr int BK = 32;           // k per ring slot: 4 chunks of 16 bytes = 64 bytes per row of a K-contiguous operand
constexpr int ROW_BYTES = BK * 2;

// Workgroups are dealt round-robin to the 8 XCDs; give each XCD one contiguous range of the `count`
// work items that the workgroups [first, first + count) of a launch stand for (first % 8 == 0).
__device__ __forceinline__ int xcd_chunk(int pid, int count, bool interleave) {
    const int per = count >> 3, rem = count & 7;
    const int xcd = pid & 7, loc = pid >> 3;
    // interleave: blocks of 32 consecutive items (what one XCD holds at a time) are dealt round-robin
    // to the XCDs instead, so that at any time the 8 XCDs work on neighbouring blocks
    if (interleave && (count & 255) == 0) return (((loc >> 5) << 3) + xcd) * 32 + (loc & 31);
    return (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + loc;
}
// tile id -> (tile_m, tile_n): ids walk groups of GM tile-rows column by column, so the tiles
// resident on one XCD at a time share A and B panels in that XCD's L2.
__device__ __forceinline__ void tile_of_id(int tile, int tiles_m, int tiles_n, int &tm, int &tn) {
    constexpr int GM = 8;
    const int width = GM * tiles_n;
    const int group = tile / width;
    const int first_m = group * GM;
    const int gsz = min(tiles_m - first_m, GM);
    const int in_group = tile - group * width;
    tm = first_m + in_group % gsz;
    tn = in_group / gsz;
}

// The tiles [n_full, n_full + n_tail) of a GEMM, those of an incomplete last round, have their
// contraction cut into `splits` slices of k_chunk K steps; a slice leaves the fp32 sums of its
// BM x BN tile at part[slice][tile - n_full] and tail_sum_kernel adds the slices.
struct TailSplit {
    float *part;          // null: no tile is split
    int n_full, n_tail, splits, k_chunk;
};

template <int BM, int BN, int WM, int WN>
struct Cfg {
    static constexpr int NW = WM * WN;
    static constexpr int TA = BM / WM / 16, TB = BN / WN / 16;   // 16x16 MFMA tiles per wave, each way
    static constexpr int SLOT = (BM + BN) * ROW_BYTES;
    static_assert(BM / 16 / NW * 2 == TA && BN / 16 / NW * 2 == TB, "TA / 2 and TB / 2 pieces of 1 KB per wave and slot");
    static_assert(TA == TB || (TA == 6 && TB == 8), "the schedules below");
};

// One operand's part of the ring; a fragment of the 16x16x32 MFMA is 16 x-values by 32 k, lane l
// holding x = l % 16, k = 8 (l / 16) .. +7.
//
// KMAJOR = true: the source is [K, X] with x contiguous.  A slot holds [32 k][X / 8 chunks of 16 B]
//   (8 x-values per chunk) and is filled by buffer loads that write straight to LDS: the 64 lanes
//   of one load deliver 16 bytes each to 1 KB of consecutive LDS addresses (lane i at 16 i), and which
//   16 bytes of global memory a lane asks for is free to choose: the chunk at physical position p
//   of row k is logical chunk p ^ 4 (k & 3) ^ 2 ((k >> 3 ^ k >> 4) & 1).  A fragment is two
//   transposing 8-byte reads (ds_read_b64_tr_b16): inside a group of 16 lanes, lane 4 k' + c
//   addresses the 4 x-values [4c, 4c + 4) of row k' of a 4 x 16 block, and lane p receives column p,
//   i.e. 4 consecutive k of one x.  The four groups of a read sit at k, k + 8, k + 16, k + 24 over
//   the same x; the second swizzle term puts any two of them that could be served together 32 bytes
//   apart.
// KMAJOR = false: the source is [X, K] with k contiguous.  A load that filled 16 rows of one slot would
//   take 64 bytes of each: half a cache line, whose other half the load for the next slot would
//   fetch again once the line has left the first-level cache (measured: a quarter slower than whole
//   lines).  So this operand's slots come in pairs, [x][8 chunks of 16 B] (64 k), the chunk c of row x
//   at position c ^ row_swizzle(x), filled a pair at a time: one load takes 8 rows of 128 bytes and
//   lands lane-linear in a 1 KB piece of LDS (the swizzle is applied by the choice of each lane's
//   global address).  A fragment is one 16-byte read per lane, from the chunks 0-3 (even slot) or
//   4-7 (odd slot).
template <int X, int NW, int T, bool KMAJOR>
struct Operand {
    static constexpr int LD = KMAJOR ? X / 16 / NW : X / 8 / NW;   // loads per wave: per slot / per two slots
    static constexpr int ROWB = X * 2;
    uint64_t base;                               // (uniform) address of the slot / pair of slots to describe next
    long left;                                   // bytes from there to the end of the source (may be negative)
    uint32_t step;                               // bytes from one to the next
    uint32_t num;                                // checked range of the one at hand
    uint32_t voff[LD];
    int rd[KMAJOR ? T : 2];                      // LDS read offsets (from the ring's start): per tile i (k-major) / per slot of the pair

    // k-contiguous layout.  The LDS serves a 16-byte read 16 lanes at a time (measured with a probe
    // of lane pairs): within each half of the wavefront, first the lanes whose index bits 2, 3, 4 have
    // even parity, then the others.  For these fragments such a group is all 16 rows, the rows with
    // bit 2 ^ bit 3 = 0 at chunk c and the others at c ^ 1 (or the other way round); rows alternate
    // between the two 128-byte halves of the banks, so among the 8 rows of one parity
    // swizzle(x) ^ bit 2 ^ bit 3 has to take 8 different values.
    static __device__ __forceinline__ int row_swizzle(int x) { return (x >> 1) & 7; }
    // K-major layout: the XOR of a chunk of row k.  X = 64: rows of 128 bytes, two to a pass over the banks; the 32-byte
    // pieces of a transposing read's rows k, k + 2 and of its groups k, k + 8 are kept apart (the four groups of 512
    // bytes take two passes anyway).
    static __device__ __forceinline__ int k_swizzle(int k) {
        if (X == 64) return 2 * ((k >> 1) & 1) + 4 * ((k >> 3) & 1);
        return (4 * (k & 3)) ^ (2 * (((k >> 3) ^ (k >> 4)) & 1));
    }

    // ld = source leading dimension (elements); x0 = first tile row; total_bytes = size of the
    // source; wave_x0 = first x-value of this wave's part of the tile; region = where in the ring this
    // operand's slots start (part of every per-lane offset, so that what is added per slot, tile and
    // piece fits an instruction's 16-bit offset field)
    __device__ __forceinline__ void init(const __bf16 *src, int ld, int x0, long total_bytes, int wave,
                                         int lane, int wave_x0, int region) {
        if (!KMAJOR) {
            set((const unsigned char *)(src + (size_t)x0 * ld), total_bytes - (long)x0 * ld * 2, 2 * ROW_BYTES, 0);
#pragma unroll
            for (int p = 0; p < LD; ++p) {
                const int row = (wave * LD + p) * 8 + (lane >> 3);
                const int ch = (lane & 7) ^ row_swizzle(row);
                voff[p] = ((uint32_t)row * (uint32_t)ld + ch * 8) * 2u;
            }
            const int lx = lane & 15, lq = lane >> 4;
#pragma unroll
            for (int h = 0; h < 2; ++h) rd[h] = region + (wave_x0 + lx) * 2 * ROW_BYTES + (((4 * h + lq) ^ row_swizzle(lx)) * 16);
        } else {
            set((const unsigned char *)(src + x0), total_bytes - (long)x0 * 2, (uint32_t)BK * (uint32_t)ld * 2u, 0);
            constexpr int KPB = 1024 / ROWB, CPR = ROWB / 16;
#pragma unroll
            for (int p = 0; p < LD; ++p) {
                const int blk = wave * LD + p, k = blk * KPB + lane / CPR;
                const int ch = (lane % CPR) ^ k_swizzle(k);
                voff[p] = ((uint32_t)k * (uint32_t)ld + ch * 8) * 2u;
            }
            // group b of 16 lanes reads k = 8 b + (0..3) (and + 4 with the second read); inside the
            // group lane 4 kq + c addresses x-values [4c, 4c + 4) of row kq
            const int b = lane >> 4, q = lane & 15, kq = q >> 2, c = q & 3;
#pragma unroll
            for (int i = 0; i < T; ++i) {
                const int chunk = (wave_x0 + 16 * i) / 8 + (c >> 1);
                rd[i] = region + (8 * b + kq) * ROWB + ((chunk ^ k_swizzle(8 * b + kq)) * 16) + (c & 1) * 8;
            }
        }
    }
    // the contraction starts `first` steps into the source (all arguments uniform)
    __device__ __forceinline__ void set(const unsigned char *b, long l, uint32_t step_bytes, int first) {
        base = (uint64_t)b + (uint64_t)first * step_bytes;
        left = l - (long)first * step_bytes;
        step = step_bytes;
    }
    // start the contraction `ksteps` K steps (64 k) into the source
    __device__ __forceinline__ void skip(int ksteps) {
        set((const unsigned char *)base, left, step, KMAJOR ? 2 * ksteps : ksteps);
    }
    // Descriptor of the slot (pair) at hand, then on to the next one, in five steps of two to four scalar
    // instructions (to be placed between different pairs of MFMAs).  The range a descriptor can check is
    // 32 bits wide: a source with more than 4 GB left is clamped (no access of a slot reaches that far
    // from the base), one past its end is empty, and so is any slot when k_left < 1 (every load
    // returns zeros without touching memory).  Written as scalar instructions: the compiler's own
    // 64-bit compares go through the vector unit, a few dozen instructions per slot that a wave alone
    // on its SIMD cannot hide.
    template <int STEP>
    __device__ __forceinline__ void next_step(int k_left, __amdgpu_buffer_rsrc_t &r) {
#if defined(__HIP_DEVICE_COMPILE__)
        if (STEP == 0)
            asm("s_cmp_eq_u32 %2, 0\n\ts_cselect_b32 %0, %1, -1"
                : "=s"(num) : "s"((uint32_t)left), "s"((int32_t)(left >> 32)) : "scc");
        if (STEP == 1)
            asm("s_cmp_lt_i32 %1, 0\n\ts_cselect_b32 %0, 0, %0" : "+s"(num) : "s"((int32_t)(left >> 32)) : "scc");
        if (STEP == 2) asm("s_cmp_gt_i32 %1, 0\n\ts_cselect_b32 %0, %0, 0" : "+s"(num) : "s"(k_left) : "scc");
#endif
        if (STEP == 3) r = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)num, 0x00020000);
        if (STEP == 4) {
            base += step;
            left -= step;
        }
    }
    // k-major: piece p (1 KB per wave) of this wave's share of the slot behind `rsrc`: global -> LDS,
    // lane i to byte 16 i of the piece; lanes past the end of the source (rows beyond K) deliver zeros
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rsrc, unsigned char OB_LDS *__restrict__ dst, int wave, int p) const {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (void OB_LDS *)(dst + (wave * LD + p) * 1024), 16, voff[p], 0, 0, 0);
    }
    // k-contiguous: piece p (8 rows of 64 k) of this wave's share of the pair of slots behind `rsrc`
    // (rows beyond M / N deliver zeros): global -> the pair at `dst` (this operand's region included)
    __device__ __forceinline__ void load_pair(__amdgpu_buffer_rsrc_t rsrc, unsigned char OB_LDS *__restrict__ dst, int wave, int p) const {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (void OB_LDS *)(dst + (wave * LD + p) * 1024), 16, voff[p], 0, 0, 0);
    }
    // fragment for MFMA tile i (16 x-values) out of the slot at `tile` (k-contiguous: slot h of the
    // pair at `tile`)
    __device__ __forceinline__ bf16x8 frag(const unsigned char OB_LDS *__restrict__ tile, int i, int h) const {
        if (!KMAJOR) {
            return *(const bf16x8 OB_LDS *)(tile + rd[h] + i * 16 * 2 * ROW_BYTES);
        } else {
#if defined(__HIP_DEVICE_COMPILE__)
            typedef __attribute__((ext_vector_type(4))) short s16x4;
            typedef __attribute__((ext_vector_type(8))) short s16x8;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 OB_LDS *)(tile + rd[i]));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 OB_LDS *)(tile + rd[i] + 4 * ROWB));
            const s16x8 v8 = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            return __builtin_bit_cast(bf16x8, v8);
#else
            return bf16x8{};
#endif
        }
    }
};

// acc += first x second, in place in the accumulation registers.  Written as an instruction: the
// builtin's destination is not tied to its addend for this shape, and the register allocator then
// moves accumulators around the loop.
__device__ __forceinline__ void mfma(f32x4 &acc, bf16x8 first, bf16x8 second) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(first), "v"(second));
}

// The bare barrier instruction: __syncthreads() carries a fence as well, which waits for every load
// to LDS still in flight, the ones for the slots further ahead included.  What has to be complete at a
// barrier is said by the s_waitcnt in front of it; the empty statement keeps the compiler from moving
// LDS accesses across.
__device__ __forceinline__ void wg_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// s_waitcnt operand: at most `vm` vector-memory operations and `lgkm` LDS operations still pending
constexpr int waitcnt(int vm, int lgkm) { return (vm & 15) | ((vm >> 4) << 14) | 0x70 | (lgkm << 8); }

// State of one wave in the K loop.  The contraction advances one ring slot (32 k) at a time: TA runs,
// run g multiplying A fragment g with all TB B fragments.  (T below: TA = TB; 192 x 256 tiles, TA = 6 and TB = 8, have
// the same order of loads, with two in some runs.)  Between its MFMAs a run carries two or
// three fragment reads for the slot after (the next B fragment g into the other B set, the next A
// fragment g - 1 into the register run g - 1 has just finished with) and one step of the refill:
//  * a k-major operand refills, for NS slots ahead, the slot whose last reader has passed the barrier
//    behind run 0: its T / 2 loads go straight to LDS, from run 1 on (A first; with both operands k-major
//    the last load of B falls into run 0 of the slot after);
//  * a k-contiguous operand refills two slots at a time, T loads, straight to LDS as well: between the
//    barrier of an odd slot, when both slots of a pair are free, and the barrier two slots on there
//    are 2 T runs.  A has three pairs: the pair freed last is filled for three K steps further on, so
//    any of those runs will do.  B has two: the pair freed is the one read next but one, so its loads
//    go out in the odd slot's own runs and the barrier two slots on waits for them.
template <int BM, int BN, int WM, int WN, bool AK, bool BKM, int NS>
struct KLoop {
    using C = Cfg<BM, BN, WM, WN>;
    static constexpr int TA = C::TA, TB = C::TB;
    static_assert(TA == TB || !AK, "a rectangular tile's K-major A would need a swizzle of its own");
    Operand<BM, C::NW, TA, AK> opa;
    Operand<BN, C::NW, TB, BKM> opb;
    __amdgpu_buffer_rsrc_t ra, rb, ra_n, rb_n;
    int ka_left, kb_left;                        // slots (k-major) / pairs of slots (k-contiguous) not yet described
    int wave;
    bf16x8 af[TA], bfr[2][TB];

    // The descriptors of the next slot (pair), ten steps (five per operand, see Operand::next_step); ra_n
    // and rb_n take over behind run 0 of the slot they are for.
    template <int STEP>
    __device__ __forceinline__ void next_step() {
        if (STEP < 5) opa.template next_step<STEP>(ka_left, ra_n);
        else opb.template next_step<STEP - 5>(kb_left, rb_n);
        if (STEP == 4) --ka_left;
        if (STEP == 9) --kb_left;
    }
    __device__ __forceinline__ void prepare_a() {
        next_step<0>();
        next_step<1>();
        next_step<2>();
        next_step<3>();
        next_step<4>();
    }
    __device__ __forceinline__ void prepare_b() {
        next_step<5>();
        next_step<6>();
        next_step<7>();
        next_step<8>();
        next_step<9>();
    }
    __device__ __forceinline__ void next_a() {
        prepare_a();
        ra = ra_n;
    }
    __device__ __forceinline__ void next_b() {
        prepare_b();
        rb = rb_n;
    }
    // The ring holds A's slots, then B's: a k-major operand's NS one after the other, a k-contiguous
    // one's in pairs: B's two, A's three (160 KB of LDS hold 64 + 96 KB).  A's pairs are used in turn,
    // which does not go into the four slots of a trip: where k-contiguous A is read and filled are
    // run-time offsets.
    static constexpr int A_SLOT = BM * ROW_BYTES, B_SLOT = BN * ROW_BYTES, A_PAIRS = NS / 2 + 1;
    static constexpr int A_BYTES = AK ? NS * A_SLOT : A_PAIRS * 2 * A_SLOT, RING_BYTES = A_BYTES + NS * B_SLOT;
    static constexpr int A_BASE = AK ? 0 : NS * B_SLOT, B_BASE = AK ? A_BYTES : 0;   // (transposing reads stay in the lower 128 KB)
    int a_cur, a_nxt, a_fill;                    // k-contiguous A: the pair of the slot at hand, of the one after, the one being filled
    // fragment i of operand A (j of B) out of the slot in ring position S (`own`: the slot at hand, else the one after it)
    __device__ __forceinline__ bf16x8 a_frag(const unsigned char OB_LDS *__restrict__ ring, int S, int i, bool own) const {
        if (AK) return opa.frag(ring + S * A_SLOT, i, 0);
        return opa.frag(ring + (own || (S & 1) ? a_cur : a_nxt), i, S & 1);
    }
    __device__ __forceinline__ bf16x8 b_frag(const unsigned char OB_LDS *__restrict__ ring, int S, int j) const {
        return opb.frag(ring + (BKM ? S : S & ~1) * B_SLOT, j, S & 1);       // (the operand's offsets start at its region)
    }
    // Position of run g of slot S among the 2 TA runs between the barrier of an odd slot and the barrier
    // two slots on: the odd slot's runs 1 .. TA-1, the even slot's runs, run 0 of the next odd slot.
    static constexpr int position(int S, int g) { return (S & 1) ? (g == 0 ? 2 * TA - 1 : g - 1) : TA - 1 + g; }
    // the piece of k-contiguous A that the run at position q loads (-1: none): next to k-contiguous B
    // the even slot's runs; next to k-major B, whose loads sit in runs 1 .. TB/2 of every slot, the
    // other runs (192 x 256: two of these four runs carry a second piece, see piece_a2)
    static constexpr int piece_a(int q) {
        if (AK) return -1;
        if (!BKM) return q >= TA - 1 && q < 2 * TA - 1 ? q - (TA - 1) : -1;      // the even slot's runs
        if (TA != TB) return q == 4 ? 0 : q == 5 ? 2 : q == 10 ? 3 : q == 11 ? 5 : -1;
        return q >= TA / 2 && q < TA ? q - TA / 2 : (q >= TA + TA / 2 ? q - TA : -1);
    }
    static constexpr int piece_a2(int q) { return TA != TB && BKM && (q == 4 || q == 10) ? piece_a(q) + 1 : -1; }
    // (B k-contiguous: A is as well, there is no layout with A alone k-major.)  B's pieces go out in the
    // odd slot's runs 1 .. TA-1, as early as its pair is free, the rest as a second load of the first of them
    static constexpr int piece_b(int q) {
        if (BKM) return -1;
        return q < TA - 1 ? q : -1;
    }
    static constexpr int piece_b2(int q) { return !BKM && q < TB - (TA - 1) ? TA - 1 + q : -1; }
    // the B fragments of the slot after that run g >= 1 reads: as many as there are runs, the rest in the first of them
    static constexpr int read_b(int g) { return TA == TB ? g : g <= 3 ? 2 * g - 2 : g + 2; }
    static constexpr int read_b2(int g) { return TA == TB ? (g == 1 ? 0 : -1) : g <= 3 ? 2 * g - 1 : -1; }
    // the pair of slots (0: slots 0 and 1; 1: slots 2 and 3) that the runs of slot S refill
    static constexpr int pair_of(int S, int g) { return (S & 1) ? (g == 0 ? ((S + 1) / 2) & 1 : (S - 1) / 2) : ((S / 2) + 1) & 1; }

    // Run g of the slot in ring position S: its TB MFMAs and between them, never more than one memory
    // instruction between two MFMAs (a 16x16x32 MFMA keeps the pipe busy for four issue slots of a
    // lone wave, and whatever sits between two of them beyond three slots is lost: scalar
    // instructions count).  Run 0 reads its slot's own last A fragment (the register was busy until
    // now) and moves the descriptors on; the others read ahead in the slot after (run 1 one B fragment
    // more, which makes up for run 0).
    template <int S, int g>
    __device__ __forceinline__ void run(f32x4 (&acc)[TA][TB], unsigned char OB_LDS *__restrict__ ring) {
        constexpr int AT_2 = TB > 2 ? 2 : 1, AT_RB = 0, AT_RA = 1, AT_RX = TB >= 8 ? 2 : 1, AT_DL = TB > 2 ? TB / 2 + 1 : 1, AT_RQ = TB >= 8 ? TB / 2 + 2 : TB - 1;
        constexpr int set = S & 1, q = position(S, g), pa = piece_a(q), pa2 = piece_a2(q), pb = piece_b(q), pb2 = piece_b2(q);
        constexpr int N = (S + 1) % NS, P = (S + NS - 1) % NS, pair = pair_of(S, g);
#pragma unroll
        for (int j = 0; j < TB; ++j) {
            mfma(acc[g][j], bfr[set][j], af[g]);
            __builtin_amdgcn_sched_barrier(0);
            if (g == 0) {
                if (j == AT_RA) af[TA - 1] = a_frag(ring, S, TA - 1, true);
                // the last load of the slot before, when both operands go straight to LDS
                if (AK && BKM && j == AT_2) opb.load(rb, ring + B_BASE + P * B_SLOT, wave, TB / 2 - 1);
                // (small tiles: the descriptors of this slot's loads are worked out here, see below)
                if (TB < 8 && (AK || (S & 1)) && j == 0) prepare_a();
                if (TB < 8 && (BKM || (S & 1)) && j == AT_2) prepare_b();
            } else {
                if (j == AT_RB) bfr[set ^ 1][read_b(g)] = b_frag(ring, N, read_b(g));
                if (j == AT_RA) af[g - 1] = a_frag(ring, N, g - 1, false);
                if (read_b2(g) >= 0 && j == AT_RX) bfr[set ^ 1][read_b2(g) >= 0 ? read_b2(g) : 0] = b_frag(ring, N, read_b2(g) >= 0 ? read_b2(g) : 0);
                if (j == AT_RQ) {
                    if (AK && g - 1 < TA / 2) opa.load(ra, ring + A_BASE + S * A_SLOT, wave, g - 1);
                    if (BKM && !AK && g - 1 < TB / 2) opb.load(rb, ring + B_BASE + S * B_SLOT, wave, g - 1);
                    if (BKM && AK && g - 1 >= TA / 2) opb.load(rb, ring + B_BASE + S * B_SLOT, wave, g - 1 - TA / 2);
                }
            }
            // Descriptors: a k-major operand moves on every slot, a k-contiguous one every other, behind run 0.
            // The ten steps of working the next ones out are dealt over the gaps of runs 2 - 4 of the slot
            // before that no memory instruction uses (a wave alone on its SIMD has three issue slots per gap).
            if (TB >= 8 && g >= 2 && g <= 4 && (j == 3 || j == 4 || j == 5 || j == 7)) {
                constexpr int first = (g - 2) * 4;
                const int step_no = first + (j == 7 ? 3 : j - 3);
                if (AK || !(S & 1)) {
                    if (step_no == 0) next_step<0>();
                    if (step_no == 1) next_step<1>();
                    if (step_no == 2) next_step<2>();
                    if (step_no == 3) next_step<3>();
                    if (step_no == 4) next_step<4>();
                }
                if (BKM || !(S & 1)) {
                    if (step_no == 5) next_step<5>();
                    if (step_no == 6) next_step<6>();
                    if (step_no == 7) next_step<7>();
                    if (step_no == 8) next_step<8>();
                    if (step_no == 9) next_step<9>();
                }
            }
            if (pa >= 0 && j == AT_RQ) opa.load_pair(ra, ring + A_BASE + a_fill, wave, pa);
            if (pb >= 0 && j == AT_RQ) opb.load_pair(rb, ring + B_BASE + pair * 2 * B_SLOT, wave, pb);
            if (pa2 >= 0 && j == AT_DL) opa.load_pair(ra, ring + A_BASE + a_fill, wave, pa2);
            if (pb2 >= 0 && j == AT_DL) opb.load_pair(rb, ring + B_BASE + pair * 2 * B_SLOT, wave, pb2);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (g == 0) {
            if (AK || (S & 1)) ra = ra_n;
            if (BKM || (S & 1)) rb = rb_n;
            // behind the barrier of an odd slot its pair is free: the runs from here on fill it, and
            // read the pair after it
            if (!AK && (S & 1)) {
                a_fill = a_cur;
                a_nxt = a_cur == (A_PAIRS - 1) * 2 * A_SLOT ? 0 : a_cur + 2 * A_SLOT;
            }
        }
        if (!AK && (S & 1) && g == TA - 1) a_cur = a_nxt;
    }
    template <int S, int g>
    __device__ __forceinline__ void runs_from(f32x4 (&acc)[TA][TB], unsigned char OB_LDS *__restrict__ ring) {
        if constexpr (g < TA) {
            run<S, g>(acc, ring);
            runs_from<S, g + 1>(acc, ring);
        }
    }
    // the loads of at most this many slots, the newest, may still be on their way at a barrier
    // (both operands k-contiguous: at the barrier of an odd slot, behind which B's pair filled two slots
    // before is read, the T loads of A since; at that of an even slot nothing new is read)
    static constexpr int vm_pending(int S) { return AK || BKM ? (TA + TB) / 2 * (NS - 2) : (S & 1) ? TA * (NS / 2 - 1) + TB * (NS / 2 - 2) : 63; }
    // The slot in ring position S.  On entry bfr[S & 1] and af[0 .. T-2] hold its fragments; on return
    // those of the slot after.
    template <int S>
    __device__ __forceinline__ void slot(f32x4 (&acc)[TA][TB], unsigned char OB_LDS *__restrict__ ring) {
        run<S, 0>(acc, ring);
        // own reads of this slot and own writes to LDS landed, own loads to the slot after in LDS (every
        // run issues one load, and the last one to the slot after went out NS - 2 slots ago or earlier),
        // then the barrier: the slot after is complete and nobody reads this one any more
        __builtin_amdgcn_s_waitcnt(waitcnt(vm_pending(S), 0));
        wg_barrier();
        runs_from<S, 1>(acc, ring);
    }
    // Before the first slot: the ring filled as the loop expects to find it, what the first slot needs
    // requested first.  k-major: the first NS slots, all but what run 0 of the first slot issues.
    // k-contiguous B: its two pairs.  k-contiguous A: the first two pairs and of the third what the runs
    // in front of the loop's first would have asked for (positions 0 .. T-2).
    // prologue_later(): the number of loads it issues after the last one that the first slot needs.
    static constexpr int prologue_later() {
        if (!AK && !BKM) return (NS / 2 - 1) * (TA + TB);
        int n = 0;
        for (int q = 0; q < TA - 1; ++q) n += (piece_a(q) >= 0 ? 1 : 0) + (piece_a2(q) >= 0 ? 1 : 0);
        n += AK ? (NS - 1) * TA / 2 : (NS / 2 - 1) * TA;
        n += (NS - 1) * TB / 2 - (AK ? 1 : 0);
        return n;
    }
    __device__ __forceinline__ void prologue(unsigned char OB_LDS *__restrict__ ring) {
        next_a();
#pragma unroll
        for (int p = 0; p < (AK ? TA / 2 : TA); ++p) {
            if (AK) opa.load(ra, ring + A_BASE, wave, p);
            else opa.load_pair(ra, ring + A_BASE, wave, p);
        }
        next_b();
#pragma unroll
        for (int p = 0; p < (BKM ? TB / 2 : TB); ++p) {
            if (BKM) opb.load(rb, ring + B_BASE, wave, p);
            else opb.load_pair(rb, ring + B_BASE, wave, p);
        }
        // the rest in the order of its use: a barrier of the loop waits for all but a fixed number of
        // the newest loads
#pragma unroll
        for (int sl = 1; sl < NS; ++sl) {
            if (AK) {
                next_a();
#pragma unroll
                for (int p = 0; p < TA / 2; ++p) opa.load(ra, ring + A_BASE + sl * A_SLOT, wave, p);
            }
            if (BKM) {
                next_b();
#pragma unroll
                for (int p = 0; p < TB / 2; ++p)
                    if (!(AK && sl == NS - 1 && p == TB / 2 - 1)) opb.load(rb, ring + B_BASE + sl * B_SLOT, wave, p);
            }
            if (!BKM && (sl & 1) && sl < NS - 1) {
                next_b();
#pragma unroll
                for (int p = 0; p < TB; ++p) opb.load_pair(rb, ring + B_BASE + (sl + 1) * B_SLOT, wave, p);
            }
            if (!AK && (sl & 1) && sl < NS - 1) {
                next_a();
#pragma unroll
                for (int p = 0; p < TA; ++p) opa.load_pair(ra, ring + A_BASE + (sl + 1) * A_SLOT, wave, p);
            }
            if (!AK && sl == NS - 1) {
                next_a();
#pragma unroll
                for (int q = 0; q < TA - 1; ++q) {
                    if (piece_a(q) >= 0) opa.load_pair(ra, ring + A_BASE + NS * A_SLOT, wave, piece_a(q));
                    if (piece_a2(q) >= 0) opa.load_pair(ra, ring + A_BASE + NS * A_SLOT, wave, piece_a2(q));
                }
                a_cur = a_nxt = 0;
                a_fill = NS * A_SLOT;
            }
        }
        // what runs 2 - 4 of the slot before the first would have left: the descriptors that take over
        // behind run 0 of the first slot
        if (TB >= 8 && AK) prepare_a();
        if (TB >= 8 && BKM) prepare_b();
    }
};

// One workgroup's work: tile (tile_m, tile_n) of C, whole, or (sliced) K steps [kz k_chunk, ...) of it with
// the fp32 sums left at part[kz][tail_tile].
// What becomes of the tile on its way out.  EPI_ROWS: row m of the result is row rows[m] of C (no residual).  The others apply an
// activation to the rounded result x, for launches of one pass over small tiles (gemm_act_fuses(), where the rule stands):
//   EPI_GELU        C = x (+ bias), act[m, n] = GELU(C), act in place of R
//   EPI_GELU_BWD    C = x GELU'(up), up in place of R
//   EPI_SWIGLU_BWD  C[m, n], C[m, N + n]: the gradients of gate and up for x, that of their product; up [M, 2 N] in place of R
// The last two leave the fp32 sums of each half tile's columns of C at colsum[2 tile_m + wave row][C's columns] (may be null: in place of the bias).
enum { EPI_PLAIN = 0, EPI_ROWS, EPI_GELU, EPI_GELU_BWD, EPI_SWIGLU_BWD };
template <int BM, int BN, int WM, int WN, bool AK, bool BKM, int NS, int EPI = EPI_PLAIN>
__device__ __forceinline__ void gemm_tile(
    int M, int N, int K, const __bf16 *__restrict__ A, int lda, const __bf16 *__restrict__ B,
    int ldb, __bf16 *__restrict__ Cm, int ldc, const __bf16 *__restrict__ bias,
    const __bf16 *R, int ldr, int tile_m, int tile_n, bool sliced, int kz, int tail_tile, const TailSplit &ts,
    const void *__restrict__ side = nullptr) {       // rows, act or up
    constexpr bool ROWS = EPI == EPI_ROWS;
    const int32_t *__restrict__ rows = (const int32_t *)side;
    using C = Cfg<BM, BN, WM, WN>;
    constexpr int TA = C::TA, TB = C::TB;
    __shared__ __attribute__((aligned(1024))) unsigned char ring_mem[KLoop<BM, BN, WM, WN, AK, BKM, NS>::RING_BYTES];
    const int m0 = __builtin_amdgcn_readfirstlane(tile_m) * BM;
    const int n0 = __builtin_amdgcn_readfirstlane(tile_n) * BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;

    KLoop<BM, BN, WM, WN, AK, BKM, NS> lp;
    lp.wave = wave;
    lp.opa.init(A, lda, m0, (AK ? (long)K : (long)M) * lda * 2, wave, lane, wm * (BM / WM), lp.A_BASE);
    lp.opb.init(B, ldb, n0, (BKM ? (long)K : (long)N) * ldb * 2, wave, lane, wn * (BN / WN), lp.B_BASE);

    f32x4 acc[TA][TB];
    unsigned char OB_LDS *ring = (unsigned char OB_LDS *)ring_mem;
    // a slice covers K steps [k_first, k_first + nk); two ring slots to the K step
    const int k_first = kz * ts.k_chunk;
    const int nk = sliced ? min(ts.k_chunk, (K + KSTEP - 1) / KSTEP - k_first) : (K + KSTEP - 1) / KSTEP;
    lp.opa.skip(k_first);
    lp.opb.skip(k_first);
    lp.ka_left = AK ? 2 * nk : nk;
    lp.kb_left = BKM ? 2 * nk : nk;
    lp.prologue(ring);
    // the accumulators are cleared while the first loads are on their way (the empty statement pins the 256
    // moves here: left alone they sink behind the wait for those loads)
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) {
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
            asm volatile("" : "+a"(acc[i][j]));
        }
    constexpr int later = KLoop<BM, BN, WM, WN, AK, BKM, NS>::prologue_later();
    __builtin_amdgcn_s_waitcnt(waitcnt(later < 63 ? later : 63, 0));
    wg_barrier();
#pragma unroll
    for (int j = 0; j < TB; ++j) lp.bfr[0][j] = lp.b_frag(ring, 0, j);
#pragma unroll
    for (int i = 0; i < TA - 1; ++i) lp.af[i] = lp.a_frag(ring, 0, i, true);

    // once round the ring per trip: a single straight path with immediate LDS addresses.  There is no
    // separate tail (several ways into the epilogue make the register allocator move the
    // accumulators between homes): the last slots also read ahead and load (fragments that are never
    // used, zeros from past the end of K), and the count of slots is rounded up to whole trips with
    // slots of zeros.
    for (int kt = 0; kt < 2 * nk; kt += NS) {
        lp.template slot<0>(acc, ring);
        lp.template slot<1>(acc, ring);
        lp.template slot<2>(acc, ring);
        lp.template slot<3>(acc, ring);
        if constexpr (NS == 8) {
            if (kt + 4 >= 2 * nk) break;
            lp.template slot<4>(acc, ring);
            lp.template slot<5>(acc, ring);
            lp.template slot<6>(acc, ring);
            lp.template slot<7>(acc, ring);
        }
    }
    static_assert(NS == 4 || NS == 8, "the trip above names the slots");

    // the MFMAs above are opaque to the compiler's hazard handling: let the last ones retire before
    // the accumulators are read
    asm volatile("s_nop 15");
    asm volatile("s_nop 15");
    // every wave is done reading the ring and every load still in flight has landed in it (zeros from
    // past the end of K); then the ring serves as transposition slabs.  A lane holds, per MFMA tile, output row m = lane % 16 and columns
    // n = 4 (lane / 16) + (0..3): stored directly, every lane of a store would touch a different
    // cache line.  Each wave writes two tile rows (32 output rows) to its slab as fp32 and reads
    // them back so that 16 (or 8) consecutive lanes cover one contiguous row segment; bias and
    // residual are added on the way out, then one rounding to bf16.
    __builtin_amdgcn_s_waitcnt(waitcnt(0, 0));
    __syncthreads();
    constexpr int CW = BN / WN;            // columns of the wave's tile
    constexpr int RSTR = CW * 4 + 16;      // fp32 row stride in LDS, padded against bank conflicts
    constexpr int LPR = CW / 8;            // lanes per row on the way out (8 columns each)
    constexpr int RPI = 64 / LPR;          // rows per read instruction
    static_assert(32 * RSTR <= 4 * C::SLOT / C::NW, "slab does not fit the wave's LDS share");
    unsigned char OB_LDS *slab = ring + wave * (4 * C::SLOT / C::NW);
    const int lx = lane & 15, lq = lane >> 4;
    const int n_out = n0 + wn * CW + (lane % LPR) * 8;
    float bv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) bv[e] = 0.f;
    if (EPI < EPI_GELU_BWD && bias && n_out < N) {
        const bf16x8 b8 = *(const bf16x8 *)(bias + n_out);
#pragma unroll
        for (int e = 0; e < 8; ++e) bv[e] = (float)b8[e];
    }
    auto put = [&](int ii) {   // tile rows 2 ii and 2 ii + 1 of the wave into its slab
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < TB; ++j)
                *(f32x4 OB_LDS *)(slab + (16 * h + lx) * RSTR + (j * 16 + lq * 4) * 4) = acc[2 * ii + h][j];
    };
    float cs[2][8];
#pragma unroll
    for (int e = 0; e < 8; ++e) cs[0][e] = cs[1][e] = 0.f;
    // One straight path per kind of output (MODE 0: bf16; 1: bf16 with the residual added; 2: the fp32 sums
    // of a slice, the whole tile: sums beyond M and N are never read by tail_sum_kernel) and per kind of
    // tile (CHECK: some rows or columns lie past M or N): with the choices inside the loop every row read
    // was a round trip to LDS of its own.  All reads of a pair of tile rows are issued together; the next
    // pair is written to the slab behind them (a wave's LDS accesses execute in order) while the rows
    // just read are rounded and stored.
    auto out = [&](auto mode, auto check) {
        constexpr int MODE = decltype(mode)::value;
        constexpr bool CHECK = decltype(check)::value;
        constexpr int NR = 32 / RPI;
        // The residual's rows are all asked for first: vmcnt counts stores too, and loads behind a pair's stores waited for the memory to
        // take those (16400 x 3200 x 3200, NT: 285 us with the loads pair by pair, 265, 252 without a residual; weight gradient
        // 9600 x 3200 over 3075 rows, accumulated: 166, 151, 145).  Registers of the K loop's fragments hold them.
        bf16x8 res[MODE == 1 ? TA / 2 : 1][NR];
        if constexpr (MODE == 1) {
#pragma unroll
            for (int ii = 0; ii < TA / 2; ++ii)
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    const int m = m0 + wm * (BM / WM) + ii * 32 + lane / LPR + r * RPI;
                    if (!CHECK || (m < M && n_out < N)) res[ii][r] = *(const bf16x8 *)(R + (size_t)m * ldr + n_out);
                }
        }
        put(0);
#pragma unroll
        for (int ii = 0; ii < TA / 2; ++ii) {
            f32x4 lo[NR], hi[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int row = r * RPI + lane / LPR;
                lo[r] = *(const f32x4 OB_LDS *)(slab + row * RSTR + (lane % LPR) * 32);
                hi[r] = *(const f32x4 OB_LDS *)(slab + row * RSTR + (lane % LPR) * 32 + 16);
            }
            if (ii + 1 < TA / 2) put(ii + 1);
            const int m_first = m0 + wm * (BM / WM) + ii * 32 + lane / LPR;
            bf16x8 r8[NR], g8[NR];
            if (EPI >= EPI_GELU_BWD) {
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if (!CHECK || (m_first + r * RPI < M && n_out < N)) {
                        const __bf16 *up = (const __bf16 *)side + (size_t)(m_first + r * RPI) * ldc + n_out;
                        r8[r] = *(const bf16x8 *)up;
                        if (EPI == EPI_SWIGLU_BWD) g8[r] = *(const bf16x8 *)(up + N);
                    }
            }
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int m = m_first + r * RPI;
                if (MODE == 2) {
                    float *dst = ts.part + ((size_t)(kz * ts.n_tail + tail_tile) * BM + (m - m0)) * BN + (n_out - n0);
                    *(f32x4 *)dst = lo[r];
                    *(f32x4 *)(dst + 4) = hi[r];
                } else if (!CHECK || (m < M && n_out < N)) {
                    float o8[8];
#pragma unroll
                    for (int e = 0; e < 4; ++e) { o8[e] = lo[r][e] + bv[e]; o8[4 + e] = hi[r][e] + bv[4 + e]; }
                    if (MODE == 1) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) o8[e] += (float)res[ii][r][e];
                    }
                    bf16x8 o;
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[e] = (__bf16)o8[e];
                    if constexpr (EPI == EPI_GELU) {
                        bf16x8 act;
#pragma unroll
                        for (int e = 0; e < 8; ++e) act[e] = (__bf16)gelu_f((float)o[e]);
                        *(bf16x8 *)((__bf16 *)side + (size_t)m * ldc + n_out) = act;
                    }
                    if constexpr (EPI == EPI_GELU_BWD) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            o[e] = (__bf16)((float)o[e] * gelu_grad_f((float)r8[r][e]));
                            cs[0][e] += (float)o[e];
                        }
                    }
                    if constexpr (EPI == EPI_SWIGLU_BWD) {
                        bf16x8 ou;
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const SwigluGrad w = swiglu_grad_f((float)o[e], (float)r8[r][e], (float)g8[r][e]);
                            o[e] = (__bf16)w.gate;
                            ou[e] = (__bf16)w.up;
                            cs[0][e] += (float)o[e];
                            cs[1][e] += (float)ou[e];
                        }
                        *(bf16x8 *)(Cm + (size_t)m * ldc + N + n_out) = ou;
                    }
                    if constexpr (EPI >= EPI_GELU_BWD) *(bf16x8 *)(Cm + (size_t)m * ldc + n_out) = o;
                    else __builtin_nontemporal_store(o, (bf16x8 *)(Cm + (size_t)(ROWS ? rows[m] : m) * ldc + n_out));
                }
            }
        }
    };
    using std::integral_constant;
    const bool inside = m0 + BM <= M && n0 + BN <= N;
    if constexpr (EPI >= EPI_GELU) {
        if (inside) out(integral_constant<int, 0>{}, integral_constant<bool, false>{});
        else out(integral_constant<int, 0>{}, integral_constant<bool, true>{});
        if constexpr (EPI >= EPI_GELU_BWD) {
            if (!bias) return;
            // a lane's columns are the same in every row it has: over the lanes of the same columns, then one row of sums per wave row
            constexpr int HALVES = EPI == EPI_SWIGLU_BWD ? 2 : 1;
#pragma unroll
            for (int half = 0; half < HALVES; ++half)
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int d = LPR; d < 64; d <<= 1) cs[half][e] += __shfl_xor(cs[half][e], d);
            if (lane < LPR && n_out < N) {
                float *dst = (float *)bias + (size_t)(2 * tile_m + wm) * ldc + n_out;
#pragma unroll
                for (int half = 0; half < HALVES; ++half) {
                    *(f32x4 *)(dst + half * N) = f32x4{cs[half][0], cs[half][1], cs[half][2], cs[half][3]};
                    *(f32x4 *)(dst + half * N + 4) = f32x4{cs[half][4], cs[half][5], cs[half][6], cs[half][7]};
                }
            }
        }
        return;
    }
    if (sliced) out(integral_constant<int, 2>{}, integral_constant<bool, false>{});
    else if (inside && R) out(integral_constant<int, 1>{}, integral_constant<bool, false>{});
    else if (inside) out(integral_constant<int, 0>{}, integral_constant<bool, false>{});
    else if (R) out(integral_constant<int, 1>{}, integral_constant<bool, true>{});
    else out(integral_constant<int, 0>{}, integral_constant<bool, true>{});
}

// EPI other than plain: R is the row list, act or up (one more argument would make the argument block 128 bytes long, and a launch of that is 0.2 us
// slower: 2567 x 768 x 256 6.0 -> 6.2)
template <int BM, int BN, int WM, int WN, bool AK, bool BKM, int NS, int EPI = EPI_PLAIN>
__global__ __launch_bounds__(WM * WN * 64) void gemm_kernel(
    int M, int N, int K, const __bf16 *__restrict__ A, int lda, const __bf16 *__restrict__ B,
    int ldb, __bf16 *__restrict__ Cm, int ldc, const __bf16 *__restrict__ bias,
    const __bf16 *R, int ldr, int tiles_m, int tiles_n, TailSplit ts) {
    // workgroups [0, n_full): whole tiles; then slice after slice of the tail tiles
    const int pid = blockIdx.x, n_whole = ts.part ? ts.n_full : (int)gridDim.x;
    const bool sliced = pid >= n_whole;
    const int kz = sliced ? (pid - n_whole) / ts.n_tail : 0;
    const bool interleave = K >= INTERLEAVE_MIN_K;
    const int tail_tile = sliced ? xcd_chunk((pid - n_whole) % ts.n_tail, ts.n_tail, interleave) : 0;
    int tile_m, tile_n;
    tile_of_id(sliced ? n_whole + tail_tile : xcd_chunk(pid, n_whole, interleave), tiles_m, tiles_n, tile_m, tile_n);
    gemm_tile<BM, BN, WM, WN, AK, BKM, NS, EPI>(M, N, K, A, lda, B, ldb, Cm, ldc, bias, EPI == EPI_PLAIN ? R : nullptr, ldr, tile_m, tile_n,
                                                sliced, kz, tail_tile, ts, R);
}

// Several GEMMs of one layout over the same contraction length K in ONE launch (the weight gradients of a
// block: K = tokens).  Their tiles are numbered one GEMM after the other and dealt to the chip as one list,
// so the chip sees one incomplete last round (cut into slices as for a single GEMM) instead of one per GEMM:
// for a narrow model every weight gradient alone is less than a round of tiles.
struct GemmGroup {
    static constexpr int MAX = GEMM_GROUP_MAX;
    int n;
    int first[MAX + 1];   // first[p]: number of the first tile of GEMM p; first[n]: all tiles
    int M[MAX], N[MAX], lda[MAX], ldb[MAX], ldc[MAX], ldr[MAX], tiles_m[MAX], tiles_n[MAX];
    const __bf16 *A[MAX], *B[MAX], *R[MAX];
    __bf16 *C[MAX];
};
__device__ __forceinline__ int group_member(const GemmGroup &g, int tile) {
    int p = 0;
#pragma unroll
    for (int i = 1; i < GEMM_GROUP_MAX; ++i) p += (i < g.n && tile >= g.first[i]) ? 1 : 0;
    return __builtin_amdgcn_readfirstlane(p);
}

template <int BM, int BN, int WM, int WN, bool AK, bool BKM, int NS>
__global__ __launch_bounds__(WM * WN * 64) void gemm_group_kernel(GemmGroup g, int K, TailSplit ts) {
    const int pid = blockIdx.x, n_whole = ts.part ? ts.n_full : (int)gridDim.x;
    const bool sliced = pid >= n_whole;
    const int kz = sliced ? (pid - n_whole) / ts.n_tail : 0;
    const bool interleave = K >= INTERLEAVE_MIN_K;
    const int tail_tile = sliced ? xcd_chunk((pid - n_whole) % ts.n_tail, ts.n_tail, interleave) : 0;
    const int tile = sliced ? n_whole + tail_tile : xcd_chunk(pid, n_whole, interleave);
    const int p = group_member(g, tile);
    int tile_m, tile_n;
    tile_of_id(tile - g.first[p], g.tiles_m[p], g.tiles_n[p], tile_m, tile_n);
    gemm_tile<BM, BN, WM, WN, AK, BKM, NS>(g.M[p], g.N[p], K, g.A[p], g.lda[p], g.B[p], g.ldb[p], g.C[p], g.ldc[p], nullptr,
                                       g.R[p], g.ldr[p], tile_m, tile_n, sliced, kz, tail_tile, ts);
}
template __global__ void gemm_group_kernel<256, 256, 2, 2, true, true, 4>(GemmGroup, int, TailSplit);
template __global__ void gemm_group_kernel<128, 128, 2, 2, true, true, 4>(GemmGroup, int, TailSplit);
template __global__ void gemm_group_kernel<64, 64, 2, 2, true, true, 8>(GemmGroup, int, TailSplit);

#define OB_GEMM_INSTANCE(BM, BN, AK, BKM, NS, ...)                                                        \
    template __global__ void gemm_kernel<BM, BN, 2, 2, AK, BKM, NS __VA_OPT__(,) __VA_ARGS__>(                              \
        int, int, int, const __bf16 *, int, const __bf16 *, int, __bf16 *, int, const __bf16 *,    \
        const __bf16 *, int, int, int, TailSplit);
OB_GEMM_INSTANCE(256, 256, false, false, 4)
OB_GEMM_INSTANCE(128, 128, false, false, 4)
OB_GEMM_INSTANCE(128, 128, false, false, 8)
OB_GEMM_INSTANCE(192, 256, false, false, 4)
OB_GEMM_INSTANCE(192, 256, false, true, 4)
OB_GEMM_INSTANCE(64, 64, false, false, 8)
OB_GEMM_INSTANCE(64, 64, false, true, 8)
OB_GEMM_INSTANCE(64, 64, true, true, 8)
OB_GEMM_INSTANCE(256, 256, false, true, 4)
OB_GEMM_INSTANCE(128, 128, false, true, 4)
OB_GEMM_INSTANCE(256, 256, true, true, 4)
OB_GEMM_INSTANCE(128, 128, true, true, 4)
OB_GEMM_INSTANCE(256, 256, false, false, 4, EPI_ROWS)
OB_GEMM_INSTANCE(128, 128, false, false, 4, EPI_ROWS)
OB_GEMM_INSTANCE(128, 128, false, false, 8, EPI_ROWS)
OB_GEMM_INSTANCE(192, 256, false, false, 4, EPI_ROWS)
OB_GEMM_INSTANCE(64, 64, false, false, 8, EPI_ROWS)
OB_GEMM_INSTANCE(128, 128, false, false, 4, EPI_GELU)
OB_GEMM_INSTANCE(128, 128, false, false, 8, EPI_GELU)
OB_GEMM_INSTANCE(64, 64, false, false, 8, EPI_GELU)
OB_GEMM_INSTANCE(128, 128, false, true, 4, EPI_GELU_BWD)
OB_GEMM_INSTANCE(64, 64, false, true, 8, EPI_GELU_BWD)
OB_GEMM_INSTANCE(128, 128, false, true, 4, EPI_SWIGLU_BWD)
OB_GEMM_INSTANCE(64, 64, false, true, 8, EPI_SWIGLU_BWD)
#undef OB_GEMM_INSTANCE
template <class... A>
constexpr size_t arg_bytes(void (*)(A...)) {
    size_t n = 0;
    ((n = align_up(n, alignof(A)) + sizeof(A)), ...);
    return n;
}
static_assert(arg_bytes((decltype(&gemm_kernel<64, 64, 2, 2, true, true, 8>))nullptr) <= 120, "see gemm_kernel");

// C = sum over the slices of the tail tiles' fp32 sums (+ bias) (+ R); 8 outputs per lane, slices
// added in order
template <int BM, int BN>
__global__ __launch_bounds__(256) void tail_sum_kernel(TailSplit ts, int M, int N, int tiles_m, int tiles_n,
                                                       const __bf16 *__restrict__ bias, const __bf16 *R, int ldr,
                                                       __bf16 *__restrict__ Cm, int ldc, const int32_t *__restrict__ rows) {
    constexpr int PER_TILE = BM * BN / 8 / 256;      // workgroups per tile
    const int t = blockIdx.x / PER_TILE;
    const int e = ((blockIdx.x % PER_TILE) * 256 + threadIdx.x) * 8;
    int tile_m, tile_n;
    tile_of_id(ts.n_full + t, tiles_m, tiles_n, tile_m, tile_n);
    const int m = tile_m * BM + e / BN, n = tile_n * BN + e % BN;
    if (m >= M || n >= N) return;
    const float *src = ts.part + (size_t)t * (BM * BN) + e;
    const size_t slice = (size_t)ts.n_tail * (BM * BN);
    f32x4 lo = *(const f32x4 *)src, hi = *(const f32x4 *)(src + 4);
    for (int z = 1; z < ts.splits; ++z) {
        lo += *(const f32x4 *)(src + z * slice);
        hi += *(const f32x4 *)(src + z * slice + 4);
    }
    float o8[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) { o8[i] = lo[i]; o8[4 + i] = hi[i]; }
    if (bias) {
        const bf16x8 b8 = *(const bf16x8 *)(bias + n);
#pragma unroll
        for (int i = 0; i < 8; ++i) o8[i] += (float)b8[i];
    }
    if (R) {
        const bf16x8 r8 = *(const bf16x8 *)(R + (size_t)m * ldr + n);
#pragma unroll
        for (int i = 0; i < 8; ++i) o8[i] += (float)r8[i];
    }
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (__bf16)o8[i];
    *(bf16x8 *)(Cm + (size_t)(rows ? rows[m] : m) * ldc + n) = o;
}

// the same for the tail tiles of a group of GEMMs
template <int BM, int BN>
__global__ __launch_bounds__(256) void tail_sum_group_kernel(TailSplit ts, GemmGroup g) {
    constexpr int PER_TILE = BM * BN / 8 / 256;
    const int t = blockIdx.x / PER_TILE;
    const int e = ((blockIdx.x % PER_TILE) * 256 + threadIdx.x) * 8;
    const int tile = ts.n_full + t;
    const int p = group_member(g, tile);
    int tile_m, tile_n;
    tile_of_id(tile - g.first[p], g.tiles_m[p], g.tiles_n[p], tile_m, tile_n);
    const int m = tile_m * BM + e / BN, n = tile_n * BN + e % BN;
    if (m >= g.M[p] || n >= g.N[p]) return;
    const float *src = ts.part + (size_t)t * (BM * BN) + e;
    const size_t slice = (size_t)ts.n_tail * (BM * BN);
    f32x4 lo = *(const f32x4 *)src, hi = *(const f32x4 *)(src + 4);
    for (int z = 1; z < ts.splits; ++z) {
        lo += *(const f32x4 *)(src + z * slice);
        hi += *(const f32x4 *)(src + z * slice + 4);
    }
    float o8[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) { o8[i] = lo[i]; o8[4 + i] = hi[i]; }
    const __bf16 *R = g.R[p];
    if (R) {
        const bf16x8 r8 = *(const bf16x8 *)(R + (size_t)m * g.ldr[p] + n);
#pragma unroll
        for (int i = 0; i < 8; ++i) o8[i] += (float)r8[i];
    }
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (__bf16)o8[i];
    *(bf16x8 *)(g.C[p] + (size_t)m * g.ldc[p] + n) = o;
}

template <int BM, int BN, int WM, int WN, bool AK, bool BKM, int NS>
void launch_tile(int M, int N, int K, const void *A, int lda, const void *B, int ldb, void *C, int ldc,
                 const void *bias, const void *R, int ldr, float *part, const Plan &p, const int32_t *rows, hipStream_t s) {
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    const TailSplit ts{p.splits > 1 ? part : nullptr, p.n_full, p.n_tail, p.splits, p.k_chunk};
    const dim3 grid(p.n_full + p.n_tail * p.splits), block(WM * WN * 64);
#define OB_GEMM_ARGS M, N, K, (const __bf16 *)A, lda, (const __bf16 *)B, ldb, (__bf16 *)C, ldc, (const __bf16 *)bias,     \
                     (const __bf16 *)(rows ? (const void *)rows : R), ldr, tiles_m, tiles_n, ts
    if constexpr (!AK && !BKM) {
        if (rows) hipLaunchKernelGGL((gemm_kernel<BM, BN, WM, WN, AK, BKM, NS, EPI_ROWS>), grid, block, 0, s, OB_GEMM_ARGS);
        else hipLaunchKernelGGL((gemm_kernel<BM, BN, WM, WN, AK, BKM, NS>), grid, block, 0, s, OB_GEMM_ARGS);
    } else
        hipLaunchKernelGGL((gemm_kernel<BM, BN, WM, WN, AK, BKM, NS>), grid, block, 0, s, OB_GEMM_ARGS);
#undef OB_GEMM_ARGS
    if (p.splits > 1)
        hipLaunchKernelGGL((tail_sum_kernel<BM, BN>), dim3(p.n_tail * (BM * BN / 8 / 256)), dim3(256), 0, s, ts, M, N,
                           tiles_m, tiles_n, (const __bf16 *)bias, (const __bf16 *)R, ldr, (__bf16 *)C, ldc, rows);
}

template <bool AK, bool BKM>
void launch_plan(const Plan &p, int M, int N, int K, const void *A, int lda, const void *B, int ldb, void *C, int ldc,
                 const void *bias, const void *R, int ldr, float *part, hipStream_t s, const int32_t *rows) {
    if (p.kind == BIG) launch_tile<256, 256, 2, 2, AK, BKM, 4>(M, N, K, A, lda, B, ldb, C, ldc, bias, R, ldr, part, p, rows, s);
    else if (p.kind == SMALL) launch_tile<128, 128, 2, 2, AK, BKM, 4>(M, N, K, A, lda, B, ldb, C, ldc, bias, R, ldr, part, p, rows, s);
    else if (p.kind == FINE) launch_tile<64, 64, 2, 2, AK, BKM, 8>(M, N, K, A, lda, B, ldb, C, ldc, bias, R, ldr, part, p, rows, s);
    else if (p.kind == MID) {
        if constexpr (!AK) launch_tile<192, 256, 2, 2, AK, BKM, 4>(M, N, K, A, lda, B, ldb, C, ldc, bias, R, ldr, part, p, rows, s);
    } else if constexpr (!AK && !BKM) launch_tile<128, 128, 2, 2, AK, BKM, 8>(M, N, K, A, lda, B, ldb, C, ldc, bias, R, ldr, part, p, rows, s);
}

// `part` (may be null: nothing is split) has room for scratch_bytes()
template <bool AK, bool BKM>
void launch_layout(int layout, int M, int N, int K, const void *A, int lda, const void *B, int ldb, void *C, int ldc,
                   const void *bias, const void *R, int ldr, float *part, hipStream_t s, const int32_t *rows = nullptr) {
    const RowCut cut = make_row_cut(layout, M, N, K, part ? scratch_bytes(M, N, K) : 0);
    if (cut.m) {
        launch_plan<AK, BKM>(cut.head, cut.m, N, K, A, lda, B, ldb, C, ldc, bias, R, ldr, part, s, rows);
        M -= cut.m;
        A = (const __bf16 *)A + (size_t)cut.m * lda;
        if (R) R = (const __bf16 *)R + (size_t)cut.m * ldr;
        if (rows) rows += cut.m;
        else C = (__bf16 *)C + (size_t)cut.m * ldc;
    }
    launch_plan<AK, BKM>(cut.rest, M, N, K, A, lda, B, ldb, C, ldc, bias, R, ldr, part, s, rows);
}

}  // namespace

// ws (may be null): gemm_workspace_bytes(0, M, N, K) bytes
void launch_gemm_nt(int M, int N, int K, const void *A, int lda, const void *B, int ldb, void *C,
                    int ldc, const void *bias, const void *R, int ldr, hipStream_t s, int k_algo, void *ws) {
    ProfScope prof(K_GEMM, s, 2.0 * M * N * (k_algo > 0 ? k_algo : K));
    launch_layout<false, false>(0, M, N, K, A, lda, B, ldb, C, ldc, bias, R, ldr, (float *)ws, s);
}
// the same with row m of the result stored as row rows[m] of C
void launch_gemm_nt_rows(int M, int N, int K, const void *A, int lda, const void *B, int ldb, void *C, int ldc,
                         const void *bias, const int32_t *rows, hipStream_t s, void *ws) {
    ProfScope prof(K_GEMM, s, 2.0 * M * N * K);
    launch_layout<false, false>(0, M, N, K, A, lda, B, ldb, C, ldc, bias, nullptr, 0, (float *)ws, s, rows);
}

// The weight gradients of a block in one launch: C_p[M_p, N_p] = A_p[K, M_p]^T B_p[K, N_p] (+ R_p), p < count <= 4, all
// over the same K, in tiles of one kind
int gemm_tn_group(int count, const GemmTN *g, int K, void *ws, size_t ws_bytes, hipStream_t s) {
    if (count < 1 || count > GEMM_GROUP_MAX) return fail(OB_EINVAL, "gemm group: %d members", count);
    int M[GEMM_GROUP_MAX], N[GEMM_GROUP_MAX];
    double flops = 0.0;
    for (int i = 0; i < count; ++i) { M[i] = g[i].M; N[i] = g[i].N; flops += 2.0 * M[i] * N[i] * K; }
    Plan p;
    if (!make_group_plan(count, M, N, K, ws != nullptr, ws_bytes, p)) {
        for (int i = 0; i < count; ++i)
            if (int rc = gemm_any(2, g[i].M, g[i].N, K, g[i].A, g[i].B, g[i].C, nullptr, g[i].R, ws, ws_bytes, s)) return rc;
        return OB_OK;
    }
    GemmGroup grp{};
    grp.n = count;
    int first = 0;
    for (int i = 0; i < count; ++i) {
        const int t = tile_rows(p.kind);
        grp.first[i] = first;
        grp.M[i] = g[i].M; grp.N[i] = g[i].N;
        grp.A[i] = (const __bf16 *)g[i].A; grp.lda[i] = g[i].M;
        grp.B[i] = (const __bf16 *)g[i].B; grp.ldb[i] = g[i].N;
        grp.C[i] = (__bf16 *)g[i].C; grp.ldc[i] = g[i].N;
        grp.R[i] = (const __bf16 *)g[i].R; grp.ldr[i] = g[i].N;
        grp.tiles_m[i] = (g[i].M + t - 1) / t; grp.tiles_n[i] = (g[i].N + t - 1) / t;
        first += grp.tiles_m[i] * grp.tiles_n[i];
    }
    for (int i = count; i <= GEMM_GROUP_MAX; ++i) grp.first[i] = first;
    ProfScope prof(K_GEMM, s, flops);
    const TailSplit ts{p.splits > 1 ? (float *)ws : nullptr, p.n_full, p.n_tail, p.splits, p.k_chunk};
    const dim3 grid(p.n_full + p.n_tail * p.splits);
    if (p.kind == BIG) hipLaunchKernelGGL((gemm_group_kernel<256, 256, 2, 2, true, true, 4>), grid, dim3(256), 0, s, grp, K, ts);
    else if (p.kind == SMALL) hipLaunchKernelGGL((gemm_group_kernel<128, 128, 2, 2, true, true, 4>), grid, dim3(256), 0, s, grp, K, ts);
    else hipLaunchKernelGGL((gemm_group_kernel<64, 64, 2, 2, true, true, 8>), grid, dim3(256), 0, s, grp, K, ts);
    if (p.splits > 1)
        hipLaunchKernelGGL((tail_sum_group_kernel<256, 256>), dim3(p.n_tail * (256 * 256 / 8 / 256)), dim3(256), 0, s, ts, grp);
    return check_launch("gemm group");
}

// one launch of small tiles with an activation in its epilogue (Plan p whole, see gemm_act_fuses())
template <int BM, int NS, bool BKM, int EPI>
static void launch_act(int M, int N, int K, const void *A, const void *B, void *C, int ldc, const void *bias, const void *side,
                       const Plan &p, hipStream_t s) {
    const TailSplit ts{nullptr, 0, 0, 1, 0};
    hipLaunchKernelGGL((gemm_kernel<BM, BM, 2, 2, false, BKM, NS, EPI>), dim3(p.n_full + p.n_tail), dim3(256), 0, s, M, N, K,
                       (const __bf16 *)A, K, (const __bf16 *)B, BKM ? N : K, (__bf16 *)C, ldc, (const __bf16 *)bias,
                       (const __bf16 *)side, ldc, (M + BM - 1) / BM, (N + BM - 1) / BM, ts);
}

// layout 0 ("NT"): A[M,K] B[N,K]; 1 ("NN"): A[M,K] B[K,N]; 2 ("TN"): A[K,M] B[K,N].  All three
// run natively: a K-major operand is staged as it lies in memory and transposed by the LDS read.
// The timed span of a GEMM with split tiles includes the kernel that sums the slices.
int gemm_any(int layout, int M, int N, int K, const void *A, const void *B, void *C,
             const void *bias, const void *R, void *ws, size_t ws_bytes, hipStream_t s) {
    ProfScope prof(K_GEMM, s, 2.0 * M * N * K);
    if (layout > 2) {      // GEMM_NT_GELU ...: R is act or up, bias of the last two the column sums
        Plan p;
        if (!gemm_act_fuses(layout, M, N, K, ws != nullptr, &p)) return fail(OB_EINVAL, "gemm: activation in a launch that has none");
        if (layout == GEMM_NT_GELU) {
            if (p.kind == FINE) launch_act<64, 8, false, EPI_GELU>(M, N, K, A, B, C, N, bias, R, p, s);
            else if (p.kind == DEEP) launch_act<128, 8, false, EPI_GELU>(M, N, K, A, B, C, N, bias, R, p, s);
            else launch_act<128, 4, false, EPI_GELU>(M, N, K, A, B, C, N, bias, R, p, s);
        } else if (layout == GEMM_NN_GELU_BWD) {
            if (p.kind == FINE) launch_act<64, 8, true, EPI_GELU_BWD>(M, N, K, A, B, C, N, bias, R, p, s);
            else launch_act<128, 4, true, EPI_GELU_BWD>(M, N, K, A, B, C, N, bias, R, p, s);
        } else {
            if (p.kind == FINE) launch_act<64, 8, true, EPI_SWIGLU_BWD>(M, N, K, A, B, C, 2 * N, bias, R, p, s);
            else launch_act<128, 4, true, EPI_SWIGLU_BWD>(M, N, K, A, B, C, 2 * N, bias, R, p, s);
        }
        return check_launch("gemm with activation");
    }
    float *part = ws && ws_bytes >= gemm_workspace_bytes(layout, M, N, K) ? (float *)ws : nullptr;
    if (layout == 0)
        launch_layout<false, false>(0, M, N, K, A, K, B, K, C, N, bias, R, N, part, s);
    else if (layout == 1)
        launch_layout<false, true>(1, M, N, K, A, K, B, N, C, N, bias, R, N, part, s);
    else
        launch_layout<true, true>(2, M, N, K, A, M, B, N, C, N, bias, R, N, part, s);
    return check_launch("gemm");
}

}  // namespace ob
