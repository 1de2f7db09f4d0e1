// Row-wise kernels of the hand-over between a ViT stack and an LLM stack on one mixed pipeline
// stage (App. A; the "token sub-sampling" named in Sec. 5.4): the 2 x 2 patch gather fused with
// the LayerNorm that follows it (forward, backward, gain / beta gradients) and the row
// scatter / gather that places the connector's output on the visual rows of the packed LLM
// batch.  All HBM-bound: every byte is read once and written once, 16 bytes per lane.
//
// Tile layout of the ViT output: g*g + 1 rows per tile, class token first, then the patches
// row-major.  Sub-sampled token (r, c) of a tile, r, c < g/2, has 4 Hv channels; channel block
// 2 dr + dc is patch (2 r + dr, 2 c + dc).
#include "ob_internal.h"

namespace ob {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

namespace {

constexpr int THREADS = 256;

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// first ViT row (patch (2r, 2c)) behind sub-sampled token i
__device__ __forceinline__ long first_patch_row(int i, int g) {
    const int half = g >> 1, per_tile = half * half;
    const int t = i / per_tile, rc = i - t * per_tile, r = rc / half, c = rc - r * half;
    return (long)t * (g * g + 1) + 1 + (long)(2 * r) * g + 2 * c;
}

// element offset into v of the 8 channels [8 c8, 8 c8 + 8) of sub-sampled token whose first
// patch row is row0
__device__ __forceinline__ size_t gather_offset(long row0, int c8, int g, int Hv) {
    const int col = c8 * 8, b = col / Hv, off = col - b * Hv;
    return (size_t)(row0 + (b >> 1) * g + (b & 1)) * Hv + off;
}

// The row kernels below: persistent workgroups of WG threads, split into G groups of S threads that each own a token
// at a time, NV vectors of 8 channels per thread.  A token's loads are issued one token ahead, so that the barriers of
// the row sums (one per sum: the LDS words alternate) never leave the memory pipe empty.
// Backward, (WG, S, NV): (1024, 256, 2) for rows of up to 4096 channels; wider ones take four vectors per thread and 512 threads,
// (512, 256, 4) to 8192 and (512, 512, 4) to 16384, so that the column sums fit 256 registers (with 1024
// threads and two vectors it spilled 60: 463 us for 10752 x 12800).
// Forward, no sums to keep: a token per workgroup, (256, 256, 2), (256, 256, 4) and (1024, 1024, 2) at the same widths, as many
// workgroups as have tokens up to what the chip holds well (fwd_workgroups); for more than 3072 tokens of the widest rows
// (512, 512, 4), two to a CU (of 12800 channels 2048 24.7 us, with 1024 threads 24.0, 4096 41.6 and 42.6, 6144 60.8 and 61.8).  In the backward's shapes few tokens meet
// few CUs and barriers of 16 waves: 1280 tokens of 4096 channels 10.4 us, so 7.0; 768 of 4352 8.7 and 5.8; 6144 of
// 4096 25.4 and 21.3; 1280 of 12800 18.1 and 16.2.

// sums of a (and b) over the S threads of the caller's group; `red` alternates between two halves
template <int WG, int S>
__device__ __forceinline__ float2 group_sum(float a, float b, float2 *__restrict__ red, int &half) {
    a = wave_sum(a);
    b = wave_sum(b);
    const int wave = threadIdx.x >> 6, first = (threadIdx.x / S) * (S / 64);
    float2 *r = red + half * (WG / 64);
    half ^= 1;
    if ((threadIdx.x & 63) == 0) r[wave] = make_float2(a, b);
    __syncthreads();
    float2 t = make_float2(0.f, 0.f);
#pragma unroll
    for (int w = 0; w < S / 64; ++w) { t.x += r[first + w].x; t.y += r[first + w].y; }
    return t;
}

// un[i] = LayerNorm(gather(v, i)) * gamma + beta;  stats[i] = (mean, rstd)
template <int WG, int S, int NV>
__global__ __launch_bounds__(WG) void subsample_norm_fwd_kernel(
    const __bf16 *__restrict__ v, const __bf16 *__restrict__ gamma, const __bf16 *__restrict__ beta,
    __bf16 *__restrict__ un, float *__restrict__ stats, int n_tok, int g, int Hv, float eps) {
    constexpr int G = WG / S;
    __shared__ float2 red[2 * (WG / 64)];
    const int W = 4 * Hv, nvec = W / 8, lane = threadIdx.x % S, stride = gridDim.x * G;
    bf16x8 gm[NV], bt[NV], nx[NV];
    int src[NV];                            // offset of this thread's channels from the token's first patch row
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int c8 = lane + k * S;
        src[k] = c8 < nvec ? (int)gather_offset(0, c8, g, Hv) : -1;
        nx[k] = bf16x8{};
    }
    auto fetch = [&](int i) {
        const __bf16 *row = v + (size_t)first_patch_row(i, g) * Hv;
#pragma unroll
        for (int k = 0; k < NV; ++k)
            if (src[k] >= 0) nx[k] = *(const bf16x8 *)(row + src[k]);
    };
    int half = 0, i = blockIdx.x * G + threadIdx.x / S;
    if (i < n_tok) fetch(i);
#pragma unroll
    for (int k = 0; k < NV; ++k) {          // (behind the first token's loads, which the first sum waits for)
        const int c8 = lane + k * S;
        gm[k] = c8 < nvec ? *(const bf16x8 *)(gamma + c8 * 8) : bf16x8{};
        bt[k] = c8 < nvec ? *(const bf16x8 *)(beta + c8 * 8) : bf16x8{};
    }
    for (int first = blockIdx.x * G; first < n_tok; first += stride, i += stride) {   // (same trip count for every thread)
        float x[NV][8], s = 0.f, q = 0.f;
#pragma unroll
        for (int k = 0; k < NV; ++k)
#pragma unroll
            for (int e = 0; e < 8; ++e) { x[k][e] = (float)nx[k][e]; s += x[k][e]; }
        if (i + stride < n_tok) fetch(i + stride);
        const float mean = group_sum<WG, S>(s, 0.f, red, half).x / W;
#pragma unroll
        for (int k = 0; k < NV; ++k)
            if (src[k] >= 0) {
#pragma unroll
                for (int e = 0; e < 8; ++e) { const float d = x[k][e] - mean; q += d * d; }
            }
        const float rstd = rsqrtf(group_sum<WG, S>(q, 0.f, red, half).x / W + eps);
        if (i >= n_tok) continue;
        if (lane == 0) {
            stats[2 * (size_t)i] = mean;
            stats[2 * (size_t)i + 1] = rstd;
        }
#pragma unroll
        for (int k = 0; k < NV; ++k)
            if (src[k] >= 0) {
                bf16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (__bf16)((x[k][e] - mean) * rstd * (float)gm[k][e] + (float)bt[k][e]);
                *(bf16x8 *)(un + (size_t)i * W + (lane + k * S) * 8) = o;
            }
    }
}

// du = LayerNorm backward of dun at a sub-sampled token, written to the four patch rows of dv it was gathered from; the
// class row of every tile is zeroed (it feeds nothing): together every element of dv is written exactly once.  Each
// group keeps its column sums of dun * xhat (gain) and dun (beta) in registers; the workgroup's groups are added through
// LDS, in order, into partial[blockIdx.x][2][W].  (A kernel of its own for the column sums read dun and v again.)
template <int WG, int S, int NV>
__global__ __launch_bounds__(WG) void subsample_norm_bwd_kernel(
    const __bf16 *__restrict__ dun, const __bf16 *__restrict__ v, const float *__restrict__ stats,
    const __bf16 *__restrict__ gamma, __bf16 *__restrict__ dv, float *__restrict__ partial, int n_tok, int n_tiles, int g,
    int Hv) {
    constexpr int G = WG / S;
    __shared__ float2 red[2 * (WG / 64)];
    __shared__ __attribute__((aligned(16))) float fold[G > 1 ? WG * NV * 8 : 4];
    const int W = 4 * Hv, nvec = W / 8, lane = threadIdx.x % S, group = threadIdx.x / S, stride = gridDim.x * G;
    const bf16x8 zero{};
    for (int t = blockIdx.x; t < n_tiles; t += gridDim.x)
        for (int c8 = threadIdx.x; c8 < Hv / 8; c8 += WG) *(bf16x8 *)(dv + (size_t)t * (g * g + 1) * Hv + c8 * 8) = zero;
    bf16x8 gm[NV], nx[NV], nd[NV];
    float dg[NV][8], db[NV][8], nmean = 0.f, nrstd = 0.f;
    int src[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int c8 = lane + k * S;
        gm[k] = c8 < nvec ? *(const bf16x8 *)(gamma + c8 * 8) : zero;
        src[k] = c8 < nvec ? (int)gather_offset(0, c8, g, Hv) : -1;
        nx[k] = nd[k] = zero;
#pragma unroll
        for (int e = 0; e < 8; ++e) dg[k][e] = db[k][e] = 0.f;
    }
    auto fetch = [&](int i) {
        const __bf16 *row = v + (size_t)first_patch_row(i, g) * Hv;
        nmean = stats[2 * (size_t)i];
        nrstd = stats[2 * (size_t)i + 1];
#pragma unroll
        for (int k = 0; k < NV; ++k)
            if (src[k] >= 0) {
                nx[k] = *(const bf16x8 *)(row + src[k]);
                nd[k] = *(const bf16x8 *)(dun + (size_t)i * W + (lane + k * S) * 8);
            }
    };
    int half = 0, i = blockIdx.x * G + group;
    if (i < n_tok) fetch(i);
    for (int first = blockIdx.x * G; first < n_tok; first += stride, i += stride) {
        const bool live = i < n_tok;
        const float mean = nmean, rstd = nrstd;
        bf16x8 tx[NV], td[NV];
        float s1 = 0.f, s2 = 0.f;
#pragma unroll
        for (int k = 0; k < NV; ++k) { tx[k] = nx[k]; td[k] = nd[k]; }
        if (i + stride < n_tok) fetch(i + stride);
        if (live) {
#pragma unroll
            for (int k = 0; k < NV; ++k)
#pragma unroll
                for (int e = 0; e < 8; ++e) {       // (threads past the row hold zeros: dun = 0 adds nothing)
                    const float d = (float)td[k][e], xh = ((float)tx[k][e] - mean) * rstd, dxh = d * (float)gm[k][e];
                    dg[k][e] += d * xh;
                    db[k][e] += d;
                    s1 += dxh;
                    s2 += dxh * xh;
                }
        }
        const float2 sum = group_sum<WG, S>(s1, s2, red, half);
        if (!live) continue;
        const float m1 = sum.x / W, m2 = sum.y / W;
        __bf16 *out = dv + (size_t)first_patch_row(i, g) * Hv;
#pragma unroll
        for (int k = 0; k < NV; ++k)
            if (src[k] >= 0) {
                bf16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float xh = ((float)tx[k][e] - mean) * rstd, dxh = (float)td[k][e] * (float)gm[k][e];
                    o[e] = (__bf16)(rstd * (dxh - m1 - xh * m2));
                }
                *(bf16x8 *)(out + src[k]) = o;
            }
    }
    auto write = [&](const float (&a)[NV][8], float *__restrict__ dst) {
        if constexpr (G == 1) {
#pragma unroll
            for (int k = 0; k < NV; ++k)
                if (src[k] >= 0) {
                    *(f32x4 *)(dst + (lane + k * S) * 8) = f32x4{a[k][0], a[k][1], a[k][2], a[k][3]};
                    *(f32x4 *)(dst + (lane + k * S) * 8 + 4) = f32x4{a[k][4], a[k][5], a[k][6], a[k][7]};
                }
        } else {
            constexpr int ROW = S * NV * 8;
            __syncthreads();
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                *(f32x4 *)(fold + group * ROW + (lane + k * S) * 8) = f32x4{a[k][0], a[k][1], a[k][2], a[k][3]};
                *(f32x4 *)(fold + group * ROW + (lane + k * S) * 8 + 4) = f32x4{a[k][4], a[k][5], a[k][6], a[k][7]};
            }
            __syncthreads();
            for (int c = threadIdx.x; c < W; c += WG) {
                float t = fold[c];
#pragma unroll
                for (int j = 1; j < G; ++j) t += fold[j * ROW + c];
                dst[c] = t;
            }
        }
    };
    write(dg, partial + (size_t)blockIdx.x * 2 * W);
    write(db, partial + (size_t)blockIdx.x * 2 * W + W);
}

// small[i] = big[rows[i]].  One workgroup per row.
__global__ __launch_bounds__(THREADS) void rows_gather_kernel(__bf16 *__restrict__ small, const __bf16 *__restrict__ big,
                                                              const int32_t *__restrict__ rows, int H) {
    const size_t i = blockIdx.x, r = (size_t)rows[i];
    for (int c8 = threadIdx.x; c8 < H / 8; c8 += THREADS) *(bf16x8 *)(small + i * H + c8 * 8) = *(const bf16x8 *)(big + r * H + c8 * 8);
}

}  // namespace

// Workgroups (of a token at a time) of the forward: one per token while the chip holds them, then as few trips of equal length as
// keep `most` of them at work.  Of 4352 channels 768 tokens in 768 workgroups 5.8 us, in 512 7.1, 1024 tokens in 1024 8.3, in 512 7.7;
// of 4096 1280 in 1280 7.0, in 640 7.8, 2048 in 1024 9.2, in 512 10.4.  The widest rows have a CU to themselves, or share it in twos.
static int fwd_workgroups(int n_tok, int Hv) {
    const int whole = Hv <= 1024 ? 1536 : Hv <= 2048 ? 768 : 256, most = Hv <= 1024 ? 1024 : Hv <= 2048 || n_tok > 3072 ? 512 : 256;
    if (n_tok <= whole) return n_tok;
    const int trips = (n_tok + most - 1) / most;
    return (n_tok + trips - 1) / trips;
}

void launch_subsample_norm_fwd(const void *v, const void *gamma, const void *beta, void *un, float *stats,
                               int n_tok, int g, int Hv, float eps, hipStream_t s) {
    ProfScope prof(K_CONN_FWD, s, 16.0 * n_tok * Hv);   // 4 Hv bf16 in, 4 Hv bf16 out
    const dim3 grid(fwd_workgroups(n_tok, Hv));
#define OB_ARGS (const __bf16 *)v, (const __bf16 *)gamma, (const __bf16 *)beta, (__bf16 *)un, stats, n_tok, g, Hv, eps
    if (Hv <= 1024) hipLaunchKernelGGL((subsample_norm_fwd_kernel<256, 256, 2>), grid, dim3(256), 0, s, OB_ARGS);
    else if (Hv <= 2048) hipLaunchKernelGGL((subsample_norm_fwd_kernel<256, 256, 4>), grid, dim3(256), 0, s, OB_ARGS);
    else if (n_tok <= 3072) hipLaunchKernelGGL((subsample_norm_fwd_kernel<1024, 1024, 2>), grid, dim3(1024), 0, s, OB_ARGS);
    else hipLaunchKernelGGL((subsample_norm_fwd_kernel<512, 512, 4>), grid, dim3(512), 0, s, OB_ARGS);
#undef OB_ARGS
}

// workgroups of the backward that there are tokens for
static int token_groups(int n_tok, int Hv) { return Hv <= 1024 ? (n_tok + 3) / 4 : Hv <= 2048 ? (n_tok + 1) / 2 : n_tok; }

int launch_subsample_norm_bwd_wgrad(const void *dun, const void *v, const float *stats, const void *gamma, void *dv,
                                    float *partial, int max_partials, int n_tok, int n_tiles, int g, int Hv, hipStream_t s) {
    ProfScope prof(K_CONN_BWD, s, 24.0 * n_tok * Hv);   // dun and v in, dv out
    int wgs = token_groups(n_tok, Hv);
    if (wgs > 256) wgs = 256;
    if (wgs > max_partials) wgs = max_partials;
#define OB_ARGS (const __bf16 *)dun, (const __bf16 *)v, stats, (const __bf16 *)gamma, (__bf16 *)dv, partial, n_tok, n_tiles, g, Hv
    if (Hv <= 1024) hipLaunchKernelGGL((subsample_norm_bwd_kernel<1024, 256, 2>), dim3(wgs), dim3(1024), 0, s, OB_ARGS);
    else if (Hv <= 2048) hipLaunchKernelGGL((subsample_norm_bwd_kernel<512, 256, 4>), dim3(wgs), dim3(512), 0, s, OB_ARGS);
    else hipLaunchKernelGGL((subsample_norm_bwd_kernel<512, 512, 4>), dim3(wgs), dim3(512), 0, s, OB_ARGS);
#undef OB_ARGS
    return wgs;
}

void launch_rows_gather(void *small, const void *big, const int32_t *rows_dev, int n_rows, int H, hipStream_t s) {
    ProfScope prof(K_ROWS, s, 4.0 * n_rows * H);
    hipLaunchKernelGGL(rows_gather_kernel, dim3(n_rows), dim3(THREADS), 0, s, (__bf16 *)small, (const __bf16 *)big, rows_dev, H);
}

}  // namespace ob
