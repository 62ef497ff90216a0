// gfx950 kernels that are no templates (embedding, a prompt's last row, the sampling launch, what runs while a model is loaded and what checks the hardware's
// layouts): one translation unit has them, the runtime's.
#pragma once

#include "ee_prefill.hpp"

namespace ee {

// Probabilistic verification: workgroups (part of the vocabulary, row of the head launch before them, whose logits and candidates they
// read).  The one whose row's decision is the last of the second launch applies the accept rule and publishes, as the
// head launch's last workgroup does under exact-match verification.
__global__ void __launch_bounds__(SAMPLE_WAVES * 64) ee_sample_sum_kernel(PassArgs a_by_value)
{
    extern __shared__ __align__(16) char lds[];
    const PassArgs &a = warmed_arguments();
    sample_sum_stage(a, lds);
}

__global__ void __launch_bounds__(SAMPLE_WAVES * 64) ee_sample_kernel(PassArgs a_by_value)
{
    extern __shared__ __align__(16) char lds[];
    const PassArgs &a = warmed_arguments();
    if (!sample_draw_stage(a, lds)) return;
    int *lastf = reinterpret_cast<int *>(lds + SAMPLE_LDS_BYTES - 16);   // behind the sampling's and the accept step's arrays
    if (threadIdx.x == 0) {
        wait_vmem();                                                     // the decision is visible before it is counted
        const int before = __hip_atomic_fetch_add(a.sm.count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *lastf = before == (int)gridDim.y - 1 ? 1 : 0;
        if (*lastf) __hip_atomic_store(a.sm.count, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (*lastf) accept_stage(a, lds);
}

// embedding
__global__ void __launch_bounds__(WG_THREADS) ee_misc_kernel(PassArgs a_by_value)
{
    extern __shared__ __align__(16) char lds[];
    const PassArgs &a = warmed_arguments();
    embed_stage(a, lds);
}

// ------------------------------------------------------------------ prefill: embedding, last row

__device__ __forceinline__ float pf_block_sum(float s, float *red)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    float t = 0.f;
    for (int w = 0; w < PF_THREADS / 64; ++w) t += red[w];
    return t;
}

// one workgroup per row: h = the token's embedding (or the supplied row), first layer's GEMM input, sum of squares
__global__ void __launch_bounds__(PF_THREADS) pf_embed_kernel(PfArgs a)
{
    __shared__ float red[PF_THREADS / 64];
    const int m = blockIdx.x, tok = a.tokens[m];
    const uint16_t *src = tok >= 0 ? a.emb + (size_t)tok * a.d : a.emb_rows + (size_t)m * a.d;
    float sq = 0.f;
    for (int c = threadIdx.x * 4; c < a.d; c += PF_THREADS * 4) {
        const uint2 r = *reinterpret_cast<const uint2 *>(src + c);
        const float v[4] = {__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xFFFF0000u), __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xFFFF0000u)};
        *reinterpret_cast<float4 *>(a.b.h + (size_t)m * a.d + c) = make_float4(v[0], v[1], v[2], v[3]);
        sq += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
        const float4 g = *reinterpret_cast<const float4 *>(a.gain + c);
        const float x[4] = {v[0] * g.x, v[1] * g.y, v[2] * g.z, v[3] * g.w};
        pf_store_split4(a.b.xn, a.b.rt, m, c, x);
    }
    sq = pf_block_sum(sq, red);
    if (threadIdx.x == 0) a.ss_out[m] = sq;
}

// one workgroup: the chunk's last row as the input of a one-row LM-head launch (xh, sums of squares)
__global__ void __launch_bounds__(PF_THREADS) pf_last_kernel(PfArgs a, uint16_t *xh, float *ss_h)
{
    __shared__ float red[PF_THREADS / 64];
    const float *h = a.b.h + (size_t)(a.rows - 1) * a.d;
    float sq = 0.f;
    for (int c = threadIdx.x * 4; c < a.d; c += PF_THREADS * 4) {
        const float4 v = *reinterpret_cast<const float4 *>(h + c), g = *reinterpret_cast<const float4 *>(a.gain + c);
        sq += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
        const float x[4] = {v.x * g.x, v.y * g.y, v.z * g.z, v.w * g.w};
        store_split4(xh, 1, 0, c, x);
    }
    sq = pf_block_sum(sq, red);
    for (int g = threadIdx.x; g < SS_LD; g += PF_THREADS) ss_h[g] = g == 0 ? sq : 0.f;
}

// ------------------------------------------------------------------ load-time kernels

// source row of output column n for the row orders the stages expect
__device__ __forceinline__ int perm_row(int perm, int n, int d, int hd, int F)
{
    if (perm == PERM_QKV) {
        int sect = n / d, c = n - sect * d;
        if (sect >= 2) return n;
        int head = c / hd, e = c - head * hd;
        int src_e = (e & 1) ? (e >> 1) + (hd >> 1) : (e >> 1);  // RoPE pair (j, j+hd/2) -> columns (2j, 2j+1)
        return sect * d + head * hd + src_e;
    }
    if (perm == PERM_GU) {
        int tile = n >> 4, r = n & 15;
        int p = tile >> 1, which = tile & 1;                     // gate tile p, up tile p, gate tile p+1, ...
        return which * F + p * 16 + r;
    }
    return n;
}

// cos and sin of position blockIdx.x's angle for RoPE pair threadIdx.x, in double
__global__ void rope_table_kernel(float2 *tab, double base, int hd)
{
    const int j = threadIdx.x;
    const double ang = (double)blockIdx.x * pow(base, -2.0 * (double)j / (double)hd);
    tab[(size_t)blockIdx.x * blockDim.x + j] = make_float2((float)cos(ang), (float)sin(ang));
}

// row-major bf16 src[N][K] -> the tiled layout of GemmPlan; block g writes workgroup g's tiles,
// sub-wave `sub` of the block those of streaming wave w = sub, sub + nsub, ...
__global__ void tile_weights_kernel(const uint16_t *__restrict__ src, uint4 *__restrict__ dst, GemmPlan pl,
                                    int perm, int d, int hd, int F)
{
    const int g = blockIdx.x;
    int nt0, n_local;
    wg_units(pl, g, nt0, n_local);
    if (n_local == 0) return;
    const int lane = threadIdx.x & 63, sub = threadIdx.x >> 6, nsub = blockDim.x >> 6;
    const int S0 = wave_ksteps(pl.KTs, 0);
    const int kt_first = (g & ((1 << pl.ksl) - 1)) * pl.KTs;   // K split over workgroups: this workgroup's slice
    for (int w = sub; w < SWAVES; w += nsub) {
        const int S_w = wave_ksteps(pl.KTs, w);
        int seq = 0;
        for (int g0 = 0; g0 < n_local; g0 += GROUP_TILES) {
            const int nl = min(GROUP_TILES, n_local - g0);
            for (int s = 0; s < S_w; ++s)
                for (int nt = 0; nt < nl; ++nt) {
                    int n = (nt0 + g0 + nt) * 16 + (lane & 15);
                    int k0 = (kt_first + w + SWAVES * s) * 32 + (lane >> 4) * 8;
                    uint16_t v[8];
                    int row = n < pl.N ? perm_row(perm, n, d, hd, F) : -1;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        int k = k0 + e;
                        v[e] = (row >= 0 && k < pl.K) ? src[(size_t)row * pl.K + k] : (uint16_t)0;
                    }
                    uint4 o;
                    o.x = v[0] | ((uint32_t)v[1] << 16);
                    o.y = v[2] | ((uint32_t)v[3] << 16);
                    o.z = v[4] | ((uint32_t)v[5] << 16);
                    o.w = v[6] | ((uint32_t)v[7] << 16);
                    const size_t step = (size_t)seq + (size_t)s * nl + nt;
                    dst[((step * pl.nwg + g) * SWAVES + w) * 64 + lane] = o;
                }
            seq += S0 * nl;
        }
    }
}

// how many of a matrix's weights have which exponent (row order does not matter)
__global__ void exponent_count_kernel(const uint16_t *__restrict__ src, size_t n, unsigned *counts)
{
    __shared__ unsigned own[256];
    for (int i = threadIdx.x; i < 256; i += blockDim.x) own[i] = 0;
    __syncthreads();
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) atomicAdd(&own[(src[i] >> 7) & 0xFF], 1u);
    __syncthreads();
    for (int i = threadIdx.x; i < 256; i += blockDim.x)
        if (own[i]) atomicAdd(&counts[i], own[i]);
}

// The packed form of the same tiles (PACK_TILE), for the window of 16 exponents from `base`; weights outside it are appended
// to list[] in any order (count[0] of them; those past `cap` are counted only) unless list is null.
struct EscapeFound {
    int n, k;
    unsigned bits;
};
__global__ void pack_weights_kernel(const uint16_t *__restrict__ src, unsigned char *__restrict__ dst, GemmPlan pl, int perm, int d, int hd, int F,
                                    int base, EscapeFound *list, int cap, int *count)
{
    const int g = blockIdx.x;
    int nt0, n_local;
    wg_units(pl, g, nt0, n_local);
    if (n_local == 0) return;
    const int lane = threadIdx.x & 63, sub = threadIdx.x >> 6, nsub = blockDim.x >> 6;
    const int S0 = wave_ksteps(pl.KTs, 0);
    const int kt_first = (g & ((1 << pl.ksl) - 1)) * pl.KTs;
    for (int w = sub; w < SWAVES; w += nsub) {
        const int S_w = wave_ksteps(pl.KTs, w);
        int seq = 0;
        for (int g0 = 0; g0 < n_local; g0 += GROUP_TILES) {
            const int nl = min(GROUP_TILES, n_local - g0);
            for (int s = 0; s < S_w; ++s)
                for (int nt = 0; nt < nl; ++nt) {
                    const int n = (nt0 + g0 + nt) * 16 + (lane & 15);
                    const int k0 = (kt_first + w + SWAVES * s) * 32 + (lane >> 4) * 8;
                    const int row = n < pl.N ? perm_row(perm, n, d, hd, F) : -1;
                    unsigned low[2] = {0, 0}, var = 0;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int k = k0 + e;
                        if (row < 0 || k >= pl.K) continue;   // padding: code 0, which is not zero: the column is dropped, or every pass clears the input there (the gate/up launch: gemm_group)
                        const unsigned bits = src[(size_t)row * pl.K + k];
                        const int rel = (int)((bits >> 7) & 0xFF) - base;
                        if (rel >= 0 && rel < 16) {
                            low[e >> 2] |= (((unsigned)(rel & 1) << 7) | (bits & 0x7F)) << (8 * (e & 3));
                            const unsigned v = ((bits & 0x8000) | ((unsigned)(rel >> 1) << 8)) << (16 * (e & 1));
                            const int rot = 4 * (e >> 1);
                            var |= rot ? (v << rot) | (v >> (32 - rot)) : v;
                        } else if (list) {
                            const int i = atomicAdd(count, 1);
                            if (i < cap) list[i] = EscapeFound{n, k, bits};
                        }
                    }
                    const size_t step = (size_t)seq + (size_t)s * nl + nt;
                    unsigned *o = reinterpret_cast<unsigned *>(dst + ((step * pl.nwg + g) * SWAVES + w) * PACK_TILE) + lane * 3;
                    o[0] = low[0];
                    o[1] = low[1];
                    o[2] = var;
                }
            seq += S0 * nl;
        }
    }
}

// counts the x in [0, x_max] with div_small(x, d) != x / d, for every divisor of the list
__global__ void div_small_check_kernel(const int *__restrict__ divisors, int n_div, int x_max, unsigned long long *bad)
{
    unsigned long long mine = 0;
    for (int j = blockIdx.y; j < n_div; j += gridDim.y) {
        const int d = divisors[j];
        for (long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x; x <= x_max; x += (long long)gridDim.x * blockDim.x)
            mine += div_small((int)x, d) != (int)x / d ? 1 : 0;
    }
    if (mine) atomicAdd(bad, mine);
}

__global__ void bf16_to_f32_kernel(const uint16_t *__restrict__ src, float *__restrict__ dst, int n)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = bf16_to_f32(src[i]);
}

// Checks the lane layout of v_mfma_f32_16x16x32_bf16 that the kernels assume:
// A[i][k] from lane (i + 16*(k/8)) element k%8, B[k][j] likewise with j, and
// D[i][j] in lane (j + 16*(i/4)) element i%4.  out[lane*4 + r] receives D.
__global__ void mfma_layout_probe_kernel(const uint4 *a, const uint4 *b, float *out)
{
    bf16x8_t A = __builtin_bit_cast(bf16x8_t, a[threadIdx.x]);
    bf16x8_t B = __builtin_bit_cast(bf16x8_t, b[threadIdx.x]);
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, B, acc, 0, 0, 0);
    for (int r = 0; r < 4; ++r) out[threadIdx.x * 4 + r] = acc[r];
}

// plain copy of n 16-byte words: the reference for what the HBM traffic counters read per byte
__global__ void __launch_bounds__(256) ee_copy_kernel(const uint4 *__restrict__ src, uint4 *__restrict__ dst, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) dst[i] = src[i];
}

// the same for v_mfma_f32_16x16x16bf16_1k: A[i][k] from lane (i + 16*(k/4)) element k%4,
// B[k][j] likewise with j, D as above
__global__ void mfma16_layout_probe_kernel(const uint2 *a, const uint2 *b, float *out)
{
    s16x4_t A = __builtin_bit_cast(s16x4_t, a[threadIdx.x]);
    s16x4_t B = __builtin_bit_cast(s16x4_t, b[threadIdx.x]);
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(A, B, acc, 0, 0, 0);
    for (int r = 0; r < 4; ++r) out[threadIdx.x * 4 + r] = acc[r];
}

}  // namespace ee
