// HBM-bound row-wise and elementwise kernels of the block (steps a1, a3, a6, a8 and their
// backward counterparts b1, b3, b6, b8, bias-gradient column sums).
// bf16 in / out, fp32 arithmetic, 16-byte loads and stores; one workgroup per token row for the
// row-wise ones so every byte is read once and written once.
#include "act.h"
#include "gemm_plan.h"
#include "ob_internal.h"

namespace ob {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

namespace {

constexpr int NORM_THREADS = 256;
constexpr int MAX_VEC = 4;  // 8-element vectors per thread: H <= 256 * 8 * 4 = 8192

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// sum over the workgroup; every thread gets the result.  `red` holds one float per wave.
__device__ __forceinline__ float block_sum(float v, float *red) {
    v = wave_sum(v);
    const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[wave] = v;
    __syncthreads();
    float t = 0.f;
    for (int w = 0; w < nw; ++w) t += red[w];
    return t;
}

template <bool LAYERNORM>
__global__ __launch_bounds__(NORM_THREADS) void norm_fwd_kernel(
    const __bf16 *__restrict__ x, const __bf16 *__restrict__ gamma, const __bf16 *__restrict__ beta,
    __bf16 *__restrict__ h, float *__restrict__ stats, int T, int H, float eps) {
    __shared__ float red[NORM_THREADS / 64];
    const int row = blockIdx.x;
    const int nvec = H / 8;
    const __bf16 *xr = x + (size_t)row * H;
    float v[MAX_VEC][8];
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < MAX_VEC; ++i) {
        const int c = threadIdx.x + i * NORM_THREADS;
        if (c < nvec) {
            const bf16x8 t = *(const bf16x8 *)(xr + c * 8);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                v[i][e] = (float)t[e];
                s += LAYERNORM ? v[i][e] : v[i][e] * v[i][e];
            }
        }
    }
    s = block_sum(s, red);
    float mean = 0.f, rstd;
    if (LAYERNORM) {
        mean = s / H;
        float q = 0.f;
#pragma unroll
        for (int i = 0; i < MAX_VEC; ++i) {
            const int c = threadIdx.x + i * NORM_THREADS;
            if (c < nvec) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float dlt = v[i][e] - mean;
                    q += dlt * dlt;
                }
            }
        }
        q = block_sum(q, red);
        rstd = rsqrtf(q / H + eps);
    } else {
        rstd = rsqrtf(s / H + eps);
    }
    if (threadIdx.x == 0) {
        stats[2 * (size_t)row] = mean;
        stats[2 * (size_t)row + 1] = rstd;
    }
#pragma unroll
    for (int i = 0; i < MAX_VEC; ++i) {
        const int c = threadIdx.x + i * NORM_THREADS;
        if (c < nvec) {
            const bf16x8 g = *(const bf16x8 *)(gamma + c * 8);
            bf16x8 o;
            if (LAYERNORM && beta) {
                const bf16x8 b = *(const bf16x8 *)(beta + c * 8);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    o[e] = (__bf16)((v[i][e] - mean) * rstd * (float)g[e] + (float)b[e]);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (__bf16)((v[i][e] - mean) * rstd * (float)g[e]);
            }
            *(bf16x8 *)(h + (size_t)row * H + c * 8) = o;
        }
    }
}

// The same forward for narrow rows (H <= 2048): a workgroup per row would leave most lanes idle and
// pay two workgroup barriers per row, so a wavefront owns a row (NV vectors of 8 per lane, row sums
// by wave reduction), walks rows slot, slot + n_slots, ... with the next row's loads in flight, and
// keeps gamma and beta in registers.
template <bool LAYERNORM, int NV>
__global__ __launch_bounds__(256) void norm_fwd_wave_kernel(
    const __bf16 *__restrict__ x, const __bf16 *__restrict__ gamma, const __bf16 *__restrict__ beta,
    __bf16 *__restrict__ h, float *__restrict__ stats, int T, int H, float eps) {
    const int nvec = H / 8, lane = threadIdx.x & 63;
    const int slot = blockIdx.x * 4 + (threadIdx.x >> 6), n_slots = gridDim.x * 4;
    bf16x8 g[NV], b[NV], nx[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = lane + 64 * i;
        g[i] = c < nvec ? *(const bf16x8 *)(gamma + c * 8) : bf16x8{};
        b[i] = LAYERNORM && beta && c < nvec ? *(const bf16x8 *)(beta + c * 8) : bf16x8{};
        nx[i] = bf16x8{};
    }
    auto fetch = [&](int row) {
#pragma unroll
        for (int i = 0; i < NV; ++i)
            if (lane + 64 * i < nvec) nx[i] = *(const bf16x8 *)(x + (size_t)row * H + (lane + 64 * i) * 8);
    };
    if (slot < T) fetch(slot);
    for (int row = slot; row < T; row += n_slots) {
        float v[NV][8];
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i)      // lanes past the end of the row hold zeros
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                v[i][e] = (float)nx[i][e];
                sum += LAYERNORM ? v[i][e] : v[i][e] * v[i][e];
            }
        if (row + n_slots < T) fetch(row + n_slots);
        sum = wave_sum(sum);
        float mean = 0.f, rstd;
        if (LAYERNORM) {
            mean = sum / H;
            float q = 0.f;
#pragma unroll
            for (int i = 0; i < NV; ++i)
                if (lane + 64 * i < nvec)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float dlt = v[i][e] - mean;
                        q += dlt * dlt;
                    }
            rstd = rsqrtf(wave_sum(q) / H + eps);
        } else {
            rstd = rsqrtf(sum / H + eps);
        }
        if (lane == 0) {
            stats[2 * (size_t)row] = mean;
            stats[2 * (size_t)row + 1] = rstd;
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int c = lane + 64 * i;
            if (c < nvec) {
                bf16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (__bf16)((v[i][e] - mean) * rstd * (float)g[i][e] + (float)b[i][e]);
                *(bf16x8 *)(h + (size_t)row * H + c * 8) = o;
            }
        }
    }
}

// dx = dres + rstd * (dxhat - mean(dxhat) [LayerNorm only] - xhat * mean(dxhat * xhat)),
// dxhat = dh * gamma.  Each workgroup walks rows blockIdx.x, +gridDim.x, ... and keeps its
// column sums of dh * xhat (dgamma) and dh (dbeta) in registers; they are written once to
// partial[blockIdx.x][2][H] and summed by reduce_partials_kernel.
// CSUM: the kernel also leaves the column sums of dres and of its output dx (as stored, after rounding) in
// csum[blockIdx.x][2][H]: the bias gradients of the two linears around the norm, which would otherwise
// each take a pass of their own over a [T, H] tensor the kernel has in registers anyway.
// Bound: HBM.  Two vectors of 8 per thread and as many threads as the row needs (H <= 512 * 16), so that several
// workgroups share a CU; a row's loads are issued one row ahead, its two sums take one barrier (the LDS words alternate).
template <bool LAYERNORM, bool CSUM>
__global__ __launch_bounds__(512) void norm_bwd_kernel(
    const __bf16 *__restrict__ dh, const __bf16 *__restrict__ x, const float *__restrict__ stats,
    const __bf16 *__restrict__ gamma, const __bf16 *__restrict__ dres, __bf16 *__restrict__ dx,
    float *__restrict__ partial, float *__restrict__ csum, int T, int H) {
    constexpr int NV = 2;
    __shared__ float2 red[2][8];
    const int nvec = H / 8, nt = blockDim.x, waves = nt >> 6;
    bf16x8 g[NV], nx[NV], nd[NV], nr[NV];
    float dg[NV][8], db[NV][8], sr[CSUM ? NV : 1][8], sx[CSUM ? NV : 1][8];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = threadIdx.x + i * nt;
        g[i] = c < nvec ? *(const bf16x8 *)(gamma + c * 8) : bf16x8{};
        nx[i] = nd[i] = nr[i] = bf16x8{};
#pragma unroll
        for (int e = 0; e < 8; ++e) dg[i][e] = db[i][e] = 0.f;
        if (CSUM) {
#pragma unroll
            for (int e = 0; e < 8; ++e) sr[i][e] = sx[i][e] = 0.f;
        }
    }
    float nmean = 0.f, nrstd = 0.f;
    auto fetch = [&](int row) {
        nmean = stats[2 * (size_t)row];
        nrstd = stats[2 * (size_t)row + 1];
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int c = threadIdx.x + i * nt;
            if (c < nvec) {
                nx[i] = *(const bf16x8 *)(x + (size_t)row * H + c * 8);
                nd[i] = *(const bf16x8 *)(dh + (size_t)row * H + c * 8);
                nr[i] = *(const bf16x8 *)(dres + (size_t)row * H + c * 8);
            }
        }
    };
    int half = 0;
    if ((int)blockIdx.x < T) fetch(blockIdx.x);
    for (int row = blockIdx.x; row < T; row += gridDim.x) {
        const float mean = nmean, rstd = nrstd;
        bf16x8 cx[NV], cd[NV], cr[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) { cx[i] = nx[i]; cd[i] = nd[i]; cr[i] = nr[i]; }
        if (row + (int)gridDim.x < T) fetch(row + gridDim.x);
        float s1 = 0.f, s2 = 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if ((int)threadIdx.x + i * nt < nvec) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float d = (float)cd[i][e], xh = ((float)cx[i][e] - mean) * rstd, dxh = d * (float)g[i][e];
                    dg[i][e] += d * xh;
                    db[i][e] += d;
                    s1 += dxh;
                    s2 += dxh * xh;
                }
            }
        }
        s1 = LAYERNORM ? wave_sum(s1) : 0.f;
        s2 = wave_sum(s2);
        if ((threadIdx.x & 63) == 0) red[half][threadIdx.x >> 6] = make_float2(s1, s2);
        __syncthreads();
        s1 = s2 = 0.f;
        for (int w = 0; w < waves; ++w) { s1 += red[half][w].x; s2 += red[half][w].y; }
        half ^= 1;
        s1 /= H;
        s2 /= H;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int c = threadIdx.x + i * nt;
            if (c < nvec) {
                bf16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float xh = ((float)cx[i][e] - mean) * rstd, dxh = (float)cd[i][e] * (float)g[i][e];
                    o[e] = (__bf16)((float)cr[i][e] + rstd * (dxh - s1 - xh * s2));
                }
                *(bf16x8 *)(dx + (size_t)row * H + c * 8) = o;
                if (CSUM) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        sr[i][e] += (float)cr[i][e];
                        sx[i][e] += (float)o[e];
                    }
                }
            }
        }
    }
    auto write = [&](const float (&a)[8], float *__restrict__ dst) {
        *(f32x4 *)dst = f32x4{a[0], a[1], a[2], a[3]};
        *(f32x4 *)(dst + 4) = f32x4{a[4], a[5], a[6], a[7]};
    };
    const size_t base = (size_t)blockIdx.x * 2 * H;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = threadIdx.x + i * nt;
        if (c < nvec) {
            write(dg[i], partial + base + c * 8);
            write(db[i], partial + base + H + c * 8);
            if (CSUM) {
                write(sr[CSUM ? i : 0], csum + base + c * 8);
                write(sx[CSUM ? i : 0], csum + base + H + c * 8);
            }
        }
    }
}

// The same backward for many narrow rows (H <= 1024), one wavefront per row: no workgroup barrier in the walk, the
// row sums are wave reductions, and the next row's loads are in flight while the current row is
// worked on.  The workgroup's eight waves add their column sums in LDS, in wave order, and leave one partial,
// partial[blockIdx.x][2][H].
constexpr int FOLD_WAVES = 8;
template <bool LAYERNORM, bool CSUM>
__global__ __launch_bounds__(64 * FOLD_WAVES) void norm_bwd_wave_kernel(
    const __bf16 *__restrict__ dh, const __bf16 *__restrict__ x, const float *__restrict__ stats,
    const __bf16 *__restrict__ gamma, const __bf16 *__restrict__ dres, __bf16 *__restrict__ dx,
    float *__restrict__ partial, float *__restrict__ csum, int T, int H) {
    constexpr int NV = 2, W = FOLD_WAVES;
    const int nvec = H / 8, lane = threadIdx.x & 63;
    const int slot = blockIdx.x * W + (threadIdx.x >> 6), n_slots = gridDim.x * W;
    bf16x8 g[NV];
    float dg[NV][8], db[NV][8];
    float sr[CSUM ? NV : 1][8], sx[CSUM ? NV : 1][8];   // column sums of dres and of dx (see norm_bwd_kernel)
#pragma unroll
    for (int i = 0; i < (CSUM ? NV : 1); ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) sr[i][e] = sx[i][e] = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = lane + 64 * i;
#pragma unroll
        for (int e = 0; e < 8; ++e) dg[i][e] = db[i][e] = 0.f;
        g[i] = c < nvec ? *(const bf16x8 *)(gamma + c * 8) : bf16x8{};
    }
    bf16x8 nx[NV], nd[NV], nr[NV];
    float nmean = 0.f, nrstd = 0.f;
    auto fetch = [&](int row) {
        nmean = stats[2 * (size_t)row];
        nrstd = stats[2 * (size_t)row + 1];
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int c = lane + 64 * i;
            if (c < nvec) {
                nx[i] = *(const bf16x8 *)(x + (size_t)row * H + c * 8);
                nd[i] = *(const bf16x8 *)(dh + (size_t)row * H + c * 8);
                nr[i] = *(const bf16x8 *)(dres + (size_t)row * H + c * 8);
            }
        }
    };
    if (slot < T) fetch(slot);
    for (int row = slot; row < T; row += n_slots) {
        const float mean = nmean, rstd = nrstd;
        bf16x8 cx[NV], cd[NV], cr[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) { cx[i] = nx[i]; cd[i] = nd[i]; cr[i] = nr[i]; }
        if (row + n_slots < T) fetch(row + n_slots);
        float s1 = 0.f, s2 = 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if (lane + 64 * i < nvec) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float d = (float)cd[i][e];
                    const float xh = ((float)cx[i][e] - mean) * rstd;
                    const float dxh = d * (float)g[i][e];
                    dg[i][e] += d * xh;
                    db[i][e] += d;
                    s1 += dxh;
                    s2 += dxh * xh;
                }
            }
        }
        s2 = wave_sum(s2) / H;
        s1 = LAYERNORM ? wave_sum(s1) / H : 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int c = lane + 64 * i;
            if (c < nvec) {
                bf16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float xh = ((float)cx[i][e] - mean) * rstd;
                    const float dxh = (float)cd[i][e] * (float)g[i][e];
                    o[e] = (__bf16)((float)cr[i][e] + rstd * (dxh - s1 - xh * s2));
                }
                *(bf16x8 *)(dx + (size_t)row * H + c * 8) = o;
                if (CSUM) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        sr[i][e] += (float)cr[i][e];
                        sx[i][e] += (float)o[e];
                    }
                }
            }
        }
    }
    constexpr int HMAX = 64 * 8 * NV;
    __shared__ float red[W][2][HMAX];
    const int wave = threadIdx.x >> 6;
    auto fold = [&](const float (&a)[NV][8], const float (&b)[NV][8], float *__restrict__ out) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int c = lane + 64 * i;
            if (c < nvec) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    red[wave][0][c * 8 + e] = a[i][e];
                    red[wave][1][c * 8 + e] = b[i][e];
                }
            }
        }
        __syncthreads();
        for (int c = threadIdx.x; c < 2 * H; c += 64 * W) {
            const int which = c >= H ? 1 : 0, col = c - which * H;
            float sum = red[0][which][col];
#pragma unroll
            for (int w = 1; w < W; ++w) sum += red[w][which][col];
            out[c] = sum;   // [2][H]
        }
        __syncthreads();
    };
    fold(dg, db, partial + (size_t)blockIdx.x * 2 * H);
    if constexpr (CSUM) fold(sr, sx, csum + (size_t)blockIdx.x * 2 * H);
}

// out[c] = (accumulate ? out[c] : 0) + sum_p partial[p * stride + c]; fixed summation order.
// A workgroup owns 32 columns; its RG groups of 32 lanes each sum every RG-th partial (eight
// independent chains per lane to keep loads in flight: the kernel is a chain of dependent memory
// latencies, a few hundred partials deep), then the RG sums are combined in LDS.
constexpr int REDUCE_THREADS = 512, RG = REDUCE_THREADS / 32;
__device__ __forceinline__ void reduce_columns(const float *__restrict__ partial, int n_part, int stride,
                                               __bf16 *__restrict__ out, int C, int accumulate) {
    __shared__ float red[RG][32];
    const int col = threadIdx.x & 31, pl = threadIdx.x >> 5;
    const int c = blockIdx.x * 32 + col;
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (c < C) {
        int p = pl;
        for (; p + 7 * RG < n_part; p += 8 * RG) {
#pragma unroll
            for (int u = 0; u < 8; ++u) s[u] += partial[(size_t)(p + u * RG) * stride + c];
        }
        for (; p < n_part; p += RG) s[0] += partial[(size_t)p * stride + c];
    }
    red[pl][col] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    __syncthreads();
    if (pl == 0 && c < C) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < RG; ++i) t += red[i][col];
        if (accumulate) t += (float)out[c];
        out[c] = (__bf16)t;
    }
}

__global__ __launch_bounds__(REDUCE_THREADS) void reduce_partials_kernel(const float *__restrict__ partial,
                                                              int n_part, int stride,
                                                              __bf16 *__restrict__ out, int C,
                                                              int accumulate) {
    reduce_columns(partial, n_part, stride, out, C, accumulate);
}

// the reductions of one block's backward pass in one launch: blockIdx.y picks the job
__global__ __launch_bounds__(REDUCE_THREADS) void reduce_batch_kernel(ReduceBatch b, int accumulate) {
    const ReduceJob j = b.job[blockIdx.y];
    if ((int)blockIdx.x * 32 >= j.C) return;
    reduce_columns(j.partial, j.n_part, j.stride, (__bf16 *)j.out, j.C, accumulate);
}

// partial[blockIdx.z][blockIdx.y][c] = sum over the rows blockIdx.y, +gridDim.y, ... of in[row][c], in = in0 or in1
__global__ __launch_bounds__(256) void colsum_kernel(const __bf16 *__restrict__ in0, const __bf16 *__restrict__ in1, int T, int C,
                                                     int ld, float *__restrict__ partial) {
    const __bf16 *in = blockIdx.z ? in1 : in0;
    const int c8 = blockIdx.x * 256 + threadIdx.x;  // 8-column vector index
    if (c8 * 8 >= C) return;
    float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const __bf16 *src = in + c8 * 8;
    const int g = gridDim.y;
    int row = blockIdx.y;
    // four rows' loads in flight; the rows are added in the order they are walked
    for (; row + 3 * g < T; row += 4 * g) {
        bf16x8 t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) t[u] = *(const bf16x8 *)(src + (size_t)(row + u * g) * ld);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e) s[e] += (float)t[u][e];
    }
    for (; row < T; row += g) {
        const bf16x8 t = *(const bf16x8 *)(src + (size_t)row * ld);
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] += (float)t[e];
    }
    float *dst = partial + ((size_t)blockIdx.z * g + blockIdx.y) * C + c8 * 8;
    *(f32x4 *)dst = f32x4{s[0], s[1], s[2], s[3]};
    *(f32x4 *)(dst + 4) = f32x4{s[4], s[5], s[6], s[7]};
}

// segment index of token t: the j with cu[j] <= t < cu[j+1]
__device__ __forceinline__ int find_segment(const int32_t *__restrict__ cu, int n_seg, int t) {
    int lo = 0, hi = n_seg;  // invariant: cu[lo] <= t < cu[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (cu[mid] <= t) lo = mid; else hi = mid;
    }
    return lo;
}

// In-place rotation of the first n_heads_rot heads of each row of qkv (the q heads then the k
// heads are contiguous there): pair (i, i + d/2) by sign * pos * base^(-2 i / d).
// One workgroup per token.  The angle depends on (token, i) only, so its cosine and sine are
// computed once per token (d/2 values, in LDS) and shared by all heads; the token's position is
// its distance to the largest segment start not behind it, found by one wave in parallel.
__global__ __launch_bounds__(256) void rotary_kernel(__bf16 *__restrict__ qkv, int ld, int T,
                                                     int n_heads_rot, int d,
                                                     const int32_t *__restrict__ cu, int n_seg,
                                                     float log2_base, float sign) {
    const int t = blockIdx.x;
    const int half = d / 2;   // <= 64
    __shared__ float cs_s[64], sn_s[64];
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        int start = 0;
        for (int j0 = 0; j0 < n_seg; j0 += 64) {
            const int j = j0 + lane;
            const int c = j < n_seg ? cu[j] : 0;
            start = max(start, c <= t ? c : 0);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) start = max(start, __shfl_xor(start, o));
        if (lane < half) {
            const float theta = exp2f(-2.0f * (float)lane / (float)d * log2_base);
            float sn, cs;
            sincosf((float)(t - start) * theta, &sn, &cs);
            cs_s[lane] = cs;
            sn_s[lane] = sn * sign;
        }
    }
    __syncthreads();
    const int per_head = half / 8;
    for (int w = threadIdx.x; w < n_heads_rot * per_head; w += blockDim.x) {
        const int head = w / per_head, i0 = (w % per_head) * 8;
        __bf16 *p = qkv + (size_t)t * ld + head * d + i0;
        const bf16x8 a = *(const bf16x8 *)p, b = *(const bf16x8 *)(p + half);
        bf16x8 oa, obb;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float cs = cs_s[i0 + e], sn = sn_s[i0 + e];
            const float x1 = (float)a[e], x2 = (float)b[e];
            oa[e] = (__bf16)(x1 * cs - x2 * sn);
            obb[e] = (__bf16)(x2 * cs + x1 * sn);
        }
        *(bf16x8 *)p = oa;
        *(bf16x8 *)(p + half) = obb;
    }
}

// GELU: act[t, f] = gelu(up[t, f]): one flat array, a vector of 8 per thread.  (Two per thread halve the workgroups, and the last of them
// end alone: forward of 8M elements 10.1 us, with one 8.3; backward of 6M 10.2 and 8.1, of 32M 37.4 and 35.2; of 200M no difference.)
__global__ __launch_bounds__(256) void gelu_fwd_kernel(const __bf16 *__restrict__ up, __bf16 *__restrict__ act, long n_vec) {
    for (long i = blockIdx.x * 256L + threadIdx.x; i < n_vec; i += gridDim.x * 256L) {
        const bf16x8 u = *(const bf16x8 *)(up + i * 8);
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (__bf16)gelu_f((float)u[e]);
        *(bf16x8 *)(act + i * 8) = o;
    }
}
__global__ __launch_bounds__(256) void gelu_bwd_kernel(const __bf16 *__restrict__ dact, const __bf16 *__restrict__ up,
                                                       __bf16 *__restrict__ dup, long n_vec) {
    for (long i = blockIdx.x * 256L + threadIdx.x; i < n_vec; i += gridDim.x * 256L) {
        const bf16x8 u = *(const bf16x8 *)(up + i * 8), d = *(const bf16x8 *)(dact + i * 8);
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (__bf16)((float)d[e] * gelu_grad_f((float)u[e]));
        *(bf16x8 *)(dup + i * 8) = o;
    }
}

// Passes over a [T, C] tensor that leave its column sums beside it: a workgroup of eight waves owns 512 columns (a vector of 8 per lane)
// and walks rows 8 blockIdx.y + wave, + 8 gridDim.y, ...; its waves' sums are added in order.  partial[blockIdx.y][c].  Bound by HBM,
// like the flat passes, without the sums' own reading of the result: 10752 x 6144, GELU's backward, gather and both sums 146 us, here
// 116; 12300 x 4096, GELU's backward and its sums 66 and 54.  (Four rows' loads at a time were slower by 2 to 10 %,
// with the next four asked for ahead by a third.)
constexpr int COLS_WAVES = 8, COLS_BLOCK = 512;
template <class Pass>
__device__ __forceinline__ void cols_pass(const Pass &pass, int T, int C, float *__restrict__ partial) {
    __shared__ float red[COLS_WAVES][COLS_BLOCK];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = blockIdx.x * COLS_BLOCK + lane * 8, step = COLS_WAVES * gridDim.y;
    float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (c < C) {
        for (int row = COLS_WAVES * blockIdx.y + wave; row < T; row += step) {
            const bf16x8 o = pass(row, C, c);
#pragma unroll
            for (int e = 0; e < 8; ++e) s[e] += (float)o[e];
        }
    }
    *(f32x4 *)&red[wave][lane * 8] = f32x4{s[0], s[1], s[2], s[3]};
    *(f32x4 *)&red[wave][lane * 8 + 4] = f32x4{s[4], s[5], s[6], s[7]};
    __syncthreads();
    const int col = blockIdx.x * COLS_BLOCK + threadIdx.x;
    if (col >= C) return;
    float sum = red[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < COLS_WAVES; ++w) sum += red[w][threadIdx.x];
    partial[(size_t)blockIdx.y * C + col] = sum;
}

struct GeluBwdPass {
    const __bf16 *__restrict__ dact, *__restrict__ up;
    __bf16 *__restrict__ dup;
    __device__ __forceinline__ bf16x8 operator()(int row, int C, int c) const {
        const size_t i = (size_t)row * C + c;
        const bf16x8 u = *(const bf16x8 *)(up + i), d = *(const bf16x8 *)(dact + i);
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (__bf16)((float)d[e] * gelu_grad_f((float)u[e]));
        *(bf16x8 *)(dup + i) = o;
        return o;
    }
};
__global__ __launch_bounds__(64 * COLS_WAVES) void gelu_bwd_cols_kernel(const __bf16 *__restrict__ dact, const __bf16 *__restrict__ up,
                                                                        __bf16 *__restrict__ dup, int T, int C, float *__restrict__ partial) {
    cols_pass(GeluBwdPass{dact, up, dup}, T, C, partial);
}

struct GatherPass {
    const __bf16 *__restrict__ big;
    const int32_t *__restrict__ rows;
    __bf16 *__restrict__ small;
    __device__ __forceinline__ bf16x8 operator()(int row, int C, int c) const {
        const bf16x8 x = *(const bf16x8 *)(big + (size_t)rows[row] * C + c);
        *(bf16x8 *)(small + (size_t)row * C + c) = x;
        return x;
    }
};
__global__ __launch_bounds__(64 * COLS_WAVES) void rows_gather_cols_kernel(__bf16 *__restrict__ small, const __bf16 *__restrict__ big,
                                                                           const int32_t *__restrict__ rows, int T, int C, float *__restrict__ partial) {
    cols_pass(GatherPass{big, rows, small}, T, C, partial);
}

// SwiGLU: up row = [gate (F) | up (F)], act = silu(gate) * up.  A thread's first row and column by one 32-bit division
// (the launch has less than 2^32 threads), the next ones by adding the grid's stride.
struct RowCol {
    long row;
    unsigned col, drow, dcol, fv;     // in vectors of 8
    __device__ __forceinline__ RowCol(unsigned fv_) : fv(fv_) {
        const unsigned i = blockIdx.x * 256u + threadIdx.x, stride = gridDim.x * 256u;
        row = i / fv;
        col = i % fv;
        drow = stride / fv;
        dcol = stride % fv;
    }
    __device__ __forceinline__ void next() {
        row += drow;
        col += dcol;
        if (col >= fv) { col -= fv; ++row; }
    }
};
__global__ __launch_bounds__(256) void swiglu_fwd_kernel(const __bf16 *__restrict__ up, __bf16 *__restrict__ act, int T, int F) {
    for (RowCol p(F / 8); p.row < T; p.next()) {
        const long t = p.row;
        const unsigned c = p.col * 8;
        const bf16x8 g = *(const bf16x8 *)(up + t * 2 * F + c);
        const bf16x8 u = *(const bf16x8 *)(up + t * 2 * F + F + c);
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float gz = (float)g[e];
            o[e] = (__bf16)(gz * sigmoid_f(gz) * (float)u[e]);
        }
        *(bf16x8 *)(act + t * F + c) = o;
    }
}
__global__ __launch_bounds__(256) void swiglu_bwd_kernel(const __bf16 *__restrict__ dact, const __bf16 *__restrict__ up,
                                                         __bf16 *__restrict__ dup, int T, int F) {
    for (RowCol p(F / 8); p.row < T; p.next()) {
        const long t = p.row;
        const unsigned c = p.col * 8;
        const bf16x8 da = *(const bf16x8 *)(dact + t * F + c);
        const bf16x8 g = *(const bf16x8 *)(up + t * 2 * F + c);
        const bf16x8 u = *(const bf16x8 *)(up + t * 2 * F + F + c);
        bf16x8 og, ou;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const SwigluGrad r = swiglu_grad_f((float)da[e], (float)g[e], (float)u[e]);
            og[e] = (__bf16)r.gate;
            ou[e] = (__bf16)r.up;
        }
        *(bf16x8 *)(dup + t * 2 * F + c) = og;
        *(bf16x8 *)(dup + t * 2 * F + F + c) = ou;
    }
}

__global__ __launch_bounds__(256) void mask_kernel(const int32_t *__restrict__ cu, int n_seg, int T,
                                                   int causal, uint8_t *__restrict__ out) {
    const int i = blockIdx.x;
    const int seg = find_segment(cu, n_seg, i);
    const int a = cu[seg], b = causal ? i + 1 : cu[seg + 1];
    for (int j = threadIdx.x; j < T; j += 256) out[(size_t)i * T + j] = (j >= a && j < b) ? 1 : 0;
}

}  // namespace

template <int NV>
static void launch_norm_fwd_wave(int norm, const void *x, const void *gamma, const void *beta, void *h, float *stats,
                                 int T, int H, float eps, int groups, hipStream_t s) {
    if (norm == OB_LAYERNORM)
        hipLaunchKernelGGL((norm_fwd_wave_kernel<true, NV>), dim3(groups), dim3(256), 0, s, (const __bf16 *)x,
                           (const __bf16 *)gamma, (const __bf16 *)beta, (__bf16 *)h, stats, T, H, eps);
    else
        hipLaunchKernelGGL((norm_fwd_wave_kernel<false, NV>), dim3(groups), dim3(256), 0, s, (const __bf16 *)x,
                           (const __bf16 *)gamma, (const __bf16 *)nullptr, (__bf16 *)h, stats, T, H, eps);
}

void launch_norm_fwd(int norm, const void *x, const void *gamma, const void *beta, void *h,
                     float *stats, int T, int H, float eps, hipStream_t s) {
    ProfScope prof(K_NORM_FWD, s, 4.0 * T * H);
    if (H <= 2048) {
        const int groups = (T + 3) / 4 < 1024 ? (T + 3) / 4 : 1024;      // 4 rows at a time per workgroup
        if (H <= 512) launch_norm_fwd_wave<1>(norm, x, gamma, beta, h, stats, T, H, eps, groups, s);
        else if (H <= 1024) launch_norm_fwd_wave<2>(norm, x, gamma, beta, h, stats, T, H, eps, groups, s);
        else launch_norm_fwd_wave<4>(norm, x, gamma, beta, h, stats, T, H, eps, groups, s);
        return;
    }
    if (norm == OB_LAYERNORM)
        hipLaunchKernelGGL(norm_fwd_kernel<true>, dim3(T), dim3(NORM_THREADS), 0, s, (const __bf16 *)x,
                           (const __bf16 *)gamma, (const __bf16 *)beta, (__bf16 *)h, stats, T, H, eps);
    else
        hipLaunchKernelGGL(norm_fwd_kernel<false>, dim3(T), dim3(NORM_THREADS), 0, s, (const __bf16 *)x,
                           (const __bf16 *)gamma, (const __bf16 *)nullptr, (__bf16 *)h, stats, T, H, eps);
}

// csum (may be null): [norm_bwd_workgroups(T, H)][2][H] fp32, column sums of dres and of dx per partial
void launch_norm_bwd(int norm, const void *dh, const void *x, const float *stats, const void *gamma,
                     const void *dres, void *dx, float *partial, int T, int H, hipStream_t s, float *csum) {
    ProfScope prof(K_NORM_BWD, s, 8.0 * T * H);
    const int nb = norm_bwd_workgroups(T, H);
    const bool folds = norm_bwd_folds(T, H);
    const int threads = folds ? 64 * FOLD_WAVES : (H / 16 + 63) / 64 * 64;
#define OB_NB(LN, CS)                                                                                          \
    hipLaunchKernelGGL((folds ? norm_bwd_wave_kernel<LN, CS> : norm_bwd_kernel<LN, CS>), dim3(nb), dim3(threads), 0, s, (const __bf16 *)dh, \
                       (const __bf16 *)x, stats, (const __bf16 *)gamma, (const __bf16 *)dres, (__bf16 *)dx,    \
                       partial, csum, T, H)
    if (norm == OB_LAYERNORM) { if (csum) OB_NB(true, true); else OB_NB(true, false); }
    else { if (csum) OB_NB(false, true); else OB_NB(false, false); }
#undef OB_NB
}

void launch_reduce_partials(const float *partial, int n_part, int stride, void *out, int C,
                            int accumulate, hipStream_t s) {
    ProfScope prof(K_REDUCE, s, 4.0 * n_part * C);
    hipLaunchKernelGGL(reduce_partials_kernel, dim3((C + 31) / 32), dim3(REDUCE_THREADS), 0, s, partial, n_part,
                       stride, (__bf16 *)out, C, accumulate);
}

int launch_reduce_batch(const ReduceBatch &b, int accumulate, hipStream_t s) {
    if (b.overflow) return fail(OB_EINVAL, "reduce batch: more than %d column reductions in one launch", ReduceBatch::MAX);
    if (b.n == 0) return OB_OK;
    double work = 0.0;
    int max_c = 0;
    for (int i = 0; i < b.n; ++i) {
        work += 4.0 * b.job[i].n_part * b.job[i].C;
        if (b.job[i].C > max_c) max_c = b.job[i].C;
    }
    ProfScope prof(K_REDUCE, s, work);
    hipLaunchKernelGGL(reduce_batch_kernel, dim3((max_c + 31) / 32, b.n), dim3(REDUCE_THREADS), 0, s, b, accumulate);
    return OB_OK;
}


void launch_colsum(const void *in, int T, int C, int ld, float *partial, hipStream_t s) {
    ProfScope prof(K_COLSUM, s, 2.0 * T * C);
    dim3 grid((C / 8 + 255) / 256, colsum_partials(T));
    hipLaunchKernelGGL(colsum_kernel, grid, dim3(256), 0, s, (const __bf16 *)in, (const __bf16 *)nullptr, T, C, ld, partial);
}

void launch_colsum_pair(const void *in0, const void *in1, int T, int C, int n_part, float *partial, hipStream_t s) {
    ProfScope prof(K_COLSUM, s, 4.0 * T * C);
    dim3 grid((C / 8 + 255) / 256, n_part, 2);
    hipLaunchKernelGGL(colsum_kernel, grid, dim3(256), 0, s, (const __bf16 *)in0, (const __bf16 *)in1, T, C, C, partial);
}

void launch_rotary(void *qkv, int ld, int T, int n_heads_rot, int d, const int32_t *cu_dev, int n_seg,
                   float base, float sign, hipStream_t s) {
    ProfScope prof(K_ROTARY, s, 4.0 * T * n_heads_rot * d);
    hipLaunchKernelGGL(rotary_kernel, dim3(T), dim3(256), 0, s, (__bf16 *)qkv, ld, T, n_heads_rot, d,
                       cu_dev, n_seg, log2f(base), sign);
}

// workgroups of an element-wise pass over n_vec vectors of 8, 256 to a workgroup: at most 65536
static int act_blocks(long n_vec) { return (int)((n_vec + 255) / 256 < 65536 ? (n_vec + 255) / 256 : 65536); }

void launch_act_fwd(int mlp, const void *up, void *act, int T, int F, hipStream_t s) {
    ProfScope prof(K_ACT_FWD, s, (mlp == OB_SWIGLU ? 6.0 : 4.0) * T * F);
    const long n_vec = (long)T * (F / 8);
    if (mlp == OB_SWIGLU)
        hipLaunchKernelGGL(swiglu_fwd_kernel, dim3(act_blocks(n_vec)), dim3(256), 0, s, (const __bf16 *)up, (__bf16 *)act, T, F);
    else
        hipLaunchKernelGGL(gelu_fwd_kernel, dim3(act_blocks(n_vec)), dim3(256), 0, s, (const __bf16 *)up, (__bf16 *)act, n_vec);
}

void launch_act_bwd(int mlp, const void *dact, const void *up, void *dup, int T, int F, hipStream_t s) {
    ProfScope prof(K_ACT_BWD, s, (mlp == OB_SWIGLU ? 10.0 : 6.0) * T * F);
    const long n_vec = (long)T * (F / 8);
    if (mlp == OB_SWIGLU)
        hipLaunchKernelGGL(swiglu_bwd_kernel, dim3(act_blocks(n_vec)), dim3(256), 0, s, (const __bf16 *)dact,
                           (const __bf16 *)up, (__bf16 *)dup, T, F);
    else
        hipLaunchKernelGGL(gelu_bwd_kernel, dim3(act_blocks(n_vec)), dim3(256), 0, s, (const __bf16 *)dact,
                           (const __bf16 *)up, (__bf16 *)dup, n_vec);
}

int launch_gelu_bwd_cols(const void *dact, const void *up, void *dup, int T, int C, float *partial, int max_partials, hipStream_t s) {
    ProfScope prof(K_ACT_BWD, s, 6.0 * T * C);
    const int n = cols_pass_partials(T, C, compute_units(), max_partials);
    hipLaunchKernelGGL(gelu_bwd_cols_kernel, dim3((C + COLS_BLOCK - 1) / COLS_BLOCK, n), dim3(64 * COLS_WAVES), 0, s, (const __bf16 *)dact,
                       (const __bf16 *)up, (__bf16 *)dup, T, C, partial);
    return n;
}

int launch_rows_gather_cols(void *small, const void *big, const int32_t *rows_dev, int n_rows, int H, float *partial, int max_partials,
                            hipStream_t s) {
    ProfScope prof(K_ROWS, s, 4.0 * n_rows * H);
    const int n = cols_pass_partials(n_rows, H, compute_units(), max_partials);
    hipLaunchKernelGGL(rows_gather_cols_kernel, dim3((H + COLS_BLOCK - 1) / COLS_BLOCK, n), dim3(64 * COLS_WAVES), 0, s, (__bf16 *)small,
                       (const __bf16 *)big, rows_dev, n_rows, H, partial);
    return n;
}

void launch_mask(const int32_t *cu_dev, int n_seg, int T, int mask, uint8_t *out, hipStream_t s) {
    hipLaunchKernelGGL(mask_kernel, dim3(T), dim3(256), 0, s, cu_dev, n_seg, T,
                       mask == OB_MASK_SEG_CAUSAL ? 1 : 0, out);
}

}  // namespace ob
