// gfx950 kernels of a prefill chunk of many rows (prompt tokens, embedding rows).
//
// A verify pass has up to 48 rows and is bound by streaming the weights once; its kernels give
// every workgroup whole n-tiles and copy the whole input into each of them.  A prompt has
// hundreds of rows: streamed 16 or 48 at a time, every group of rows pays for the whole model's
// weights again.  The kernels here take up to PF_ROWS rows at once and are bound by the
// matrix cores and by what feeds them from the L2:
//   pf_gemm_kernel   output tile of n-tiles x row tiles per workgroup, both operands through LDS
//   pf_att_kernel    causal attention of the chunk over the cache, 64 or 128 query rows per workgroup
//   pf_embed_kernel  embedding gather, first norm input
//   pf_last_kernel   the last row as the LM head's input
// Arithmetic is that of the verify pass: bf16 weights, every other operand as two bf16 terms, fp32
// accumulation, residual stream, norms and softmax; the same weight tiles (GemmPlan's order) and
// the same KV records are used, so nothing is stored twice.
#pragma once

#include "ee_kernels.hpp"

namespace ee {

constexpr int PF_ROWS = 2048;     // rows of one chunk (a multiple of 128)
constexpr int PF_THREADS = 256;   // four waves

// Buffers of a prefill chunk (per session, for `16 * rt` rows).  GEMM inputs are stored as MFMA
// operands: [k-tile][term][row tile][lane][8] bf16, lane = (k % 32 / 8) * 16 + row % 16, so that
// one operand of 16 rows x 32 k is one contiguous kilobyte, read by lane number.
struct PfScratch {
    float *h;          // [rows][d]  residual stream
    float *q;          // [rows][d]  queries after RoPE
    uint16_t *xn;      // gain * h, input of QKV and gate/up
    uint16_t *attn;    // attention output
    uint16_t *u;       // silu(gate) * up
    float *ss;         // [slots][rows]  partial sums of h^2 of the rows (two buffers, see ss_in / ss_out)
    int rt;            // row tiles the buffers are laid out for
};

struct PfArgs {
    PfScratch b;
    int rows;                 // rows of this chunk
    int pos0;                 // position of row 0 (a multiple of KV_PAGE)
    int layer;
    int d, F, H, hd;
    float eps, att_scale;
    // GEMM
    const uint4 *W;           // the layer's weights in GemmPlan's order
    const int2 *tab;          // [NT] per n-tile: first tile and distance between k-tiles 8 apart, in tiles of 1 KB
    int NT, KT, N;
    int nb, mb;               // workgroup tiles along N and along the rows
    int ks;                   // workgroups that share a tile, each with its part of K
    float *part;              // ks > 1: [tile][part][wave][accumulator][lane][4] partial tiles
    int *part_count;          // ks > 1: [tile] parts delivered; zero between launches
    const float *gain;        // O / DN: gain of the next GEMM input, or nullptr
    const float *ss_in;       // partial sums of squares of the input's rows (QKV, GU)
    int ss_slots;
    float *ss_out;            // O / DN
    // attention, KV write
    uint16_t *kpool, *vpool;
    const float2 *rope;
    const int *page_table;
    int contig_base, n_pages;
    // embedding
    const int *tokens;
    const uint16_t *emb_rows, *emb;
};

__device__ __forceinline__ size_t pf_index(int rt, int m, int k, int term)
{
    return ((size_t)((k >> 5) * 2 + term) * rt + (m >> 4)) * 512 + ((k & 31) >> 3) * 128 + (m & 15) * 8 + (k & 7);
}

// four consecutive columns k .. k+3 (k a multiple of 4) of row m, as two bf16 terms
__device__ __forceinline__ void pf_store_split4(uint16_t *x, int rt, int m, int k, const float *v)
{
    uint32_t h[2], l[2];
    split_bf16(v[0], v[1], h[0], l[0]);
    split_bf16(v[2], v[3], h[1], l[1]);
    const size_t i = pf_index(rt, m, k, 0);
    *reinterpret_cast<EE_GLOBAL u32x2_t *>(as_global_mut(x) + i) = (u32x2_t){h[0], h[1]};
    *reinterpret_cast<EE_GLOBAL u32x2_t *>(as_global_mut(x) + i + (size_t)rt * 512) = (u32x2_t){l[0], l[1]};
}

// Stages of the ring a tile shape uses.  One group of waves: 48 to 72 KB, so that two workgroups (2 x 2: three) share
// a compute unit and one's barrier and epilogue run under the other's products.  Several groups: 128 to 144 KB, the
// workgroup has the unit to itself.
constexpr int pf_stages(int wn, int wm, int grp) { return grp > 1 ? 144 / (grp * (wn + 2 * wm) * 2) : (wn + 2 * wm) * 2 >= 32 ? 2 : ((wn + 2 * wm) * 2 >= 24 ? 3 : 4); }
constexpr size_t pf_gemm_lds(int wn, int wm, int grp) { return (size_t)grp * pf_stages(wn, wm, grp) * (wn + 2 * wm) * 2048 + (size_t)wm * 32 * 4 + 16; }
constexpr size_t pf_tile_floats(int wn, int wm) { return (size_t)wn * wm * 1024; }

// One GEMM of the chunk.  Workgroup tile: 2 WN n-tiles x 2 WM row tiles, four waves as 2 x 2, each
// WN x WM accumulators.  Per k-tile of 32 the stage's W tiles and both terms of the X tiles travel to
// LDS (1 KB per load instruction, already in operand order: every LDS read is a contiguous
// kilobyte), NS stages in a ring, one barrier per k-tile.
// Bound by the matrix cores (busy 51 to 63 % of a launch), by a step's barrier and operand reads beside them, and by a last
// round of tiles that leaves part of the chip idle (gate/up of 2041 rows: 1376 tiles on 512 places).  2041 rows, 7B shape, both
// terms' products counted: gate/up 537 to 581 us (1.27 to 1.37 PFLOP/s), QKV 311 to 335 (1.23 to 1.32), down 288 to 301 (1.22 to
// 1.28), output projection 121 to 125 (1.10 to 1.13; 256 workgroups, one per unit); the spread is that of machines.  The same
// rows in chunks of 16 through the streaming kernels: 3 ms per chunk, 486 ms per prompt against 46 ms.
// With few rows the tiles do not cover the chip and a workgroup alone on its unit needs 0.19 us (2 x 2, four groups of waves)
// to 0.91 us (8 x 4) per k-tile, mostly a chain of barrier, LDS reads and products: then ks workgroups
// share a tile, each with a part of K, and GRP groups of four waves share a workgroup's K, group g taking the
// k-tiles g, g + GRP, ... through a ring of its own (pf_choose).  64 rows, 7B shape, us without / with: down 86 / 29,
// output 35 / 18, QKV 40 / 34; four groups instead of one, 1280-wide model, 64 rows: QKV 16 / 11, gate/up 13 / 9.
// (A deeper ring, operands read a stage ahead into registers, the 32x32x16 instruction and starting places along K
// that differ between workgroups: each within 3 % or slower.)
template <int KIND, int WN, int WM, int GRP>
__global__ void __launch_bounds__(PF_THREADS * GRP, GRP > 1 ? GRP : 2) pf_gemm_kernel(PfArgs a)
{
    constexpr int BNT = 2 * WN, BMT = 2 * WM, NS = pf_stages(WN, WM, GRP);
    constexpr int WL = BNT / 4, XL = 2 * BMT / 4;            // loads per wave and stage
    constexpr int PER = WL + XL;
    constexpr unsigned STAGE = (BNT + 2 * BMT) * 1024;
    static_assert(BNT % 4 == 0 && BMT % 2 == 0, "tile shape");
    extern __shared__ __align__(16) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, grp = __builtin_amdgcn_readfirstlane(tid >> 8), wave = __builtin_amdgcn_readfirstlane((tid >> 6) & 3);
    const int wn = wave & 1, wm = wave >> 1;
    // Workgroups are dealt to the XCDs round-robin; each XCD gets a contiguous run of the tile
    // sequence, which walks groups of four n-blocks over all row blocks: the workgroups that run together on
    // an XCD then share a few W and X blocks in its L2.
    const int T = a.nb * a.mb * a.ks;
    int t, part = 0;
    {
        const int x = blockIdx.x % NUM_XCD, j = blockIdx.x / NUM_XCD;
        const int base = T / NUM_XCD, extra = T % NUM_XCD;
        t = x * base + min(x, extra) + j;
        if (a.ks > 1) {                                      // the parts of a tile follow each other
            const int tile = div_small(t, a.ks);
            part = t - tile * a.ks;
            t = tile;
        }
    }
    const int tile = t;
    const int kt_lo = a.ks > 1 ? div_small(a.KT * part, a.ks) : 0, kt_hi = a.ks > 1 ? div_small(a.KT * (part + 1), a.ks) : a.KT;
    const int gsz = 4 * a.mb, tg = div_small(t, gsz), rem = t - tg * gsz;
    const int gw = min(4, a.nb - tg * 4);
    const int mblk = div_small(rem, gw), nblk = tg * 4 + (rem - mblk * gw);
    const int nt0 = nblk * BNT, mt0 = mblk * BMT;

    float *rstd = reinterpret_cast<float *>(lds + GRP * NS * STAGE);
    char *ring = lds + grp * NS * STAGE;                     // this group's ring
    const unsigned lds0 = lds_offset(ring);
    // this wave's share of a stage
    const char *wbase[WL];
    int wstride[WL];
#pragma unroll
    for (int i = 0; i < WL; ++i) {
        const int2 e = a.tab[min(nt0 + wave * WL + i, a.NT - 1)];
        wbase[i] = reinterpret_cast<const char *>(uniform_ptr(reinterpret_cast<const char *>(a.W) + (size_t)__builtin_amdgcn_readfirstlane(e.x) * 1024));
        wstride[i] = __builtin_amdgcn_readfirstlane(e.y);
    }
    const uint16_t *X = KIND == G_O ? a.b.attn : (KIND == G_DN ? a.b.u : a.b.xn);
    const int term = wave >> 1, xt0 = (wave & 1) * XL;       // waves 0, 1: hi term, 2, 3: lo term; XL row tiles each
    const char *xbase = reinterpret_cast<const char *>(X) + ((size_t)term * a.b.rt) * 1024;
    int xrow[XL];
#pragma unroll
    for (int i = 0; i < XL; ++i) xrow[i] = min(mt0 + xt0 + i, a.b.rt - 1);
    const size_t xstep = (size_t)2 * a.b.rt * 1024;
    const int lane16 = lane * 16;
    auto request = [&](int kt, int buf) __attribute__((always_inline)) {
        const unsigned dst = lds0 + buf * STAGE;
#pragma unroll
        for (int i = 0; i < WL; ++i)
            load_lds_kb(wbase[i] + ((size_t)(kt >> 3) * wstride[i] + (kt & 7)) * 1024, lane16, dst + (wave * WL + i) * 1024);
#pragma unroll
        for (int i = 0; i < XL; ++i)
            load_lds_kb(xbase + (size_t)kt * xstep + (size_t)xrow[i] * 1024, lane16, dst + (BNT + term * BMT + xt0 + i) * 1024);
    };
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (kt_lo + grp + s * GRP < kt_hi) request(kt_lo + grp + s * GRP, s);
    // row factors of the norm
    if (KIND == G_QKV || KIND == G_GU) {
        for (int r = tid; r < BMT * 16; r += PF_THREADS * GRP) {
            const int m = min(mt0 * 16 + r, a.rows - 1);
            float s = 0.f;
#pragma unroll 8
            for (int j = 0; j < a.ss_slots; ++j) s += as_global(a.ss_in)[(size_t)j * a.b.rt * 16 + m];
            rstd[r] = 1.0f / sqrtf(s / (float)a.d + a.eps);
        }
    }

    f32x4_t acc[WN][WM];
#pragma unroll
    for (int i = 0; i < WN; ++i)
#pragma unroll
        for (int j = 0; j < WM; ++j) acc[i][j] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

    int buf = 0;
    for (int kt0 = kt_lo; kt0 < kt_hi; kt0 += GRP) {         // (all groups run the same number of rounds)
        const int kt = kt0 + grp;
        // this wave's loads of stage kt have landed; after the barrier everybody's have, and nobody
        // reads the buffer of stage kt - 1 any more
        if (kt + (NS - 2) * GRP < kt_hi)
            wait_pending<PER *(NS - 2)>();
        else
            wait_pending<0>();
        lds_barrier();
        if (kt + (NS - 1) * GRP < kt_hi) request(kt + (NS - 1) * GRP, buf == 0 ? NS - 1 : buf - 1);
        const char *st = ring + buf * STAGE;
        buf = buf + 1 == NS ? 0 : buf + 1;
        if (GRP > 1 && kt >= kt_hi) continue;
        const char *sw = st + (wn * WN) * 1024 + lane16;
        const char *sx = st + (BNT + wm * WM) * 1024 + lane16;
        bf16x8_t w[WN], xh[WM], xl[WM];
#pragma unroll
        for (int i = 0; i < WN; ++i) w[i] = *reinterpret_cast<const bf16x8_t *>(sw + i * 1024);
#pragma unroll
        for (int j = 0; j < WM; ++j) {
            xh[j] = *reinterpret_cast<const bf16x8_t *>(sx + j * 1024);
            xl[j] = *reinterpret_cast<const bf16x8_t *>(sx + (BMT + j) * 1024);
        }
#pragma unroll
        for (int j = 0; j < WM; ++j) {
#pragma unroll
            for (int i = 0; i < WN; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[i], xh[j], acc[i][j], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < WN; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[i], xl[j], acc[i][j], 0, 0, 0);
        }
    }

    if (GRP > 1) {
        // the groups' partial tiles meet in LDS; group 0 adds them up in group order and goes on
        lds_barrier();
        float4 *mine = reinterpret_cast<float4 *>(lds) + ((size_t)grp * 4 + wave) * (WN * WM * 64) + lane;
        if (grp > 0) {
#pragma unroll
            for (int i = 0; i < WN; ++i)
#pragma unroll
                for (int j = 0; j < WM; ++j) mine[(i * WM + j) * 64] = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
        }
        lds_barrier();
        if (grp == 0) {
#pragma unroll
            for (int q = 1; q < GRP; ++q)
#pragma unroll
                for (int i = 0; i < WN; ++i)
#pragma unroll
                    for (int j = 0; j < WM; ++j) {
                        const float4 x = mine[(size_t)q * 4 * (WN * WM * 64) + (i * WM + j) * 64];
                        acc[i][j] += (f32x4_t){x.x, x.y, x.z, x.w};
                    }
        }
    }
    if (a.ks > 1) {
        // K shared by several workgroups: the partial tiles meet in memory and the workgroup that arrives last adds
        // them up in the order of the parts and goes on alone.  Nothing waits.
        int *lastf = reinterpret_cast<int *>(lds + GRP * NS * STAGE + WM * 32 * 4);
        constexpr int TILE_B = WN * WM * 4096;               // bytes of a partial tile
        const WRes mem = buffer_resource(a.part + (size_t)tile * a.ks * (TILE_B / 4));
        const int off = wave * (WN * WM * 1024) + lane16;
#pragma unroll
        for (int i = 0; i < WN; ++i)
#pragma unroll
            for (int j = 0; j < WM; ++j)
                if (grp == 0) store_dev128(mem, part * TILE_B + off + (i * WM + j) * 1024, make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]));
        wait_vmem();      // this workgroup's part is visible device-wide ...
        __syncthreads();  // ... for every wave, before it is counted
        if (tid == 0) {
            const int before = __hip_atomic_fetch_add(a.part_count + tile, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *lastf = before == a.ks - 1 ? 1 : 0;
            if (*lastf) __hip_atomic_store(a.part_count + tile, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (!*lastf || grp > 0) return;
#pragma unroll
        for (int j = 0; j < WM; ++j) {
            f32x4_t total[WN];
#pragma unroll
            for (int i = 0; i < WN; ++i) total[i] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
            for (int p = 0; p < a.ks; ++p) {
                float4 x[WN];
#pragma unroll
                for (int i = 0; i < WN; ++i) x[i] = load_dev128(mem, p * TILE_B + off + (i * WM + j) * 1024);
#pragma unroll
                for (int i = 0; i < WN; ++i) total[i] += (f32x4_t){x[i].x, x[i].y, x[i].z, x[i].w};
            }
#pragma unroll
            for (int i = 0; i < WN; ++i) acc[i][j] = total[i];
        }
    }
    if (GRP > 1 && grp > 0) return;
    // epilogue from the accumulators: lane holds columns n .. n+3 (n = n-tile * 16 + (lane >> 4) * 4) of row m
    const int quad = lane >> 4, lm = lane & 15;
#pragma unroll
    for (int j = 0; j < WM; ++j) {
        const int m = (mt0 + wm * WM + j) * 16 + lm;
        const bool live = m < a.rows;
        if (KIND == G_GU) {
            const float rs = rstd[(wm * WM + j) * 16 + lm];
#pragma unroll
            for (int i = 0; i < WN; i += 2) {
                const int nt = nt0 + wn * WN + i;
                float o[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float g = acc[i][j][e] * rs, u = acc[i + 1][j][e] * rs;
                    o[e] = g / (1.0f + __expf(-g)) * u;
                }
                if (live && nt < a.NT) pf_store_split4(a.b.u, a.b.rt, m, (nt >> 1) * 16 + quad * 4, o);
            }
        } else if (KIND == G_O || KIND == G_DN) {
            float sq = 0.f;
            EE_GLOBAL float *hp = as_global_mut(a.b.h) + (size_t)min(m, a.rows - 1) * a.d;
            f32x4_t hv[WN], gv[WN];
#pragma unroll
            for (int i = 0; i < WN; ++i) {
                const int n = min((nt0 + wn * WN + i) * 16, a.d - 16) + quad * 4;
                hv[i] = *reinterpret_cast<const EE_GLOBAL f32x4_t *>(hp + n);
                gv[i] = a.gain ? *as_global(reinterpret_cast<const f32x4_t *>(a.gain + n)) : (f32x4_t){0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int i = 0; i < WN; ++i) {
                const int nt = nt0 + wn * WN + i, n = nt * 16 + quad * 4;
                if (live && nt < a.NT) {
                    const f32x4_t v = hv[i] + acc[i][j];
                    *reinterpret_cast<EE_GLOBAL f32x4_t *>(hp + n) = v;
                    sq += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
                    if (a.gain) {
                        const float x[4] = {v[0] * gv[i][0], v[1] * gv[i][1], v[2] * gv[i][2], v[3] * gv[i][3]};
                        pf_store_split4(a.b.xn, a.b.rt, m, n, x);
                    }
                }
            }
            sq += __shfl_xor(sq, 16, 64);
            sq += __shfl_xor(sq, 32, 64);
            if (quad == 0 && live) as_global_mut(a.ss_out)[(size_t)(nblk * 2 + wn) * a.b.rt * 16 + m] = sq;
        } else {
            const float rs = rstd[(wm * WM + j) * 16 + lm];
            const int pos = a.pos0 + min(m, a.rows - 1);
            const int page = a.contig_base >= 0 ? a.contig_base + pos / KV_PAGE : as_global(a.page_table)[pos / KV_PAGE];
            const size_t rec0 = (((size_t)a.layer * a.n_pages + page) * a.H) * KV_PAGE * 2 * a.hd;
            const int slot = pos % KV_PAGE;
#pragma unroll
            for (int i = 0; i < WN; ++i) {
                const int nt = nt0 + wn * WN + i;
                if (nt >= a.NT) continue;
                // an n-tile lies inside one head of one of the three sections
                const int sect = div_small(nt * 16, a.d), c0 = nt * 16 - sect * a.d, head = div_small(c0, a.hd), e = c0 - head * a.hd + quad * 4;
                float v[4] = {acc[i][j][0] * rs, acc[i][j][1] * rs, acc[i][j][2] * rs, acc[i][j][3] * rs};
                if (sect < 2) {  // columns are pair-interleaved inside a head: (e, e+1) = RoPE pair e/2
                    const f32x4_t cs = *as_global(reinterpret_cast<const f32x4_t *>(a.rope + (size_t)pos * (a.hd >> 1) + (e >> 1)));
                    const float y0 = v[0] * cs[0] - v[1] * cs[1], y1 = v[1] * cs[0] + v[0] * cs[1];
                    const float y2 = v[2] * cs[2] - v[3] * cs[3], y3 = v[3] * cs[2] + v[2] * cs[3];
                    v[0] = y0; v[1] = y1; v[2] = y2; v[3] = y3;
                }
                if (!live) continue;
                if (sect == 0) {
                    *reinterpret_cast<EE_GLOBAL f32x4_t *>(as_global_mut(a.b.q) + (size_t)m * a.d + c0 + quad * 4) = (f32x4_t){v[0], v[1], v[2], v[3]};
                } else {
                    uint32_t vh[2], vl[2];
                    split_bf16(v[0], v[1], vh[0], vl[0]);
                    split_bf16(v[2], v[3], vh[1], vl[1]);
                    const size_t rec = rec0 + (size_t)head * KV_PAGE * 2 * a.hd;
                    if (sect == 1) {
                        EE_GLOBAL uint16_t *kr = as_global_mut(a.kpool) + rec + (size_t)slot * 2 * a.hd + e;
                        *reinterpret_cast<EE_GLOBAL u32x2_t *>(kr) = (u32x2_t){vh[0], vh[1]};
                        *reinterpret_cast<EE_GLOBAL u32x2_t *>(kr + a.hd) = (u32x2_t){vl[0], vl[1]};
                    } else {
                        EE_GLOBAL uint16_t *vr = as_global_mut(a.vpool) + rec + slot;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            vr[(size_t)(e + r) * KV_PAGE] = (uint16_t)(vh[r >> 1] >> (16 * (r & 1)));
                            vr[(size_t)(a.hd + e + r) * KV_PAGE] = (uint16_t)(vl[r >> 1] >> (16 * (r & 1)));
                        }
                    }
                }
            }
        }
    }
}

// ------------------------------------------------------------------ attention

constexpr int PF_ATT_GROUPS = 2;          // groups of four waves that share a block's positions
constexpr int PF_ATT_THREADS = PF_ATT_GROUPS * 256;
constexpr int pf_att_stage(int hd) { return 4 * KV_PAGE * 2 * hd * 2; }   // bytes: K and V of two pages
constexpr size_t pf_att_lds(int hd, int n_pages) { return (size_t)2 * PF_ATT_GROUPS * pf_att_stage(hd) + (size_t)n_pages * 4; }

// Workgroup = (head, block of 64 RT query rows); wave w of either group has row tiles w RT .. of the block.  The groups
// walk the cached positions 32 (two pages) at a time up to the block's last row's position, group g the steps g, g + 2, ...;
// K and V of a step are shared by the group's four waves through LDS (two buffers per group).  Scores as S^T = K . q^T
// (16x16x32, two operands of 16 positions per 32 values): row 4 q + r of operand p is position 8 q + 4 p + r of the
// step, so that a lane holds eight consecutive positions of one row; those are, without any exchange, the k-slots of the second
// product O^T = V^T . P^T (16x16x32 over the step), and the V operand's eight positions are 16 contiguous bytes of the page.
// A row's maximum, sum and output stay in the lanes of its column: the running rescale needs no exchange either.
// Two bf16 terms of q, K, P and V, three MFMAs each.  At the end group 1's results join group 0's through LDS.
// Bound by a step's chain (copy, scores, softmax, second product: 2 us whatever the model) where workgroups are few, by
// vector instructions and LDS reads beside the products otherwise.  One workgroup per compute unit, the longest blocks first:
// a long block's chain is halved and the short ones fill the end.  us per launch against one group of waves per workgroup, two
// workgroups per unit (V in 8-byte reads, every score masked and scaled): 32 heads of 128, 64 rows 7.3 -> 7.5, 256 18.3 -> 13.5,
// 640 46.8 -> 27.5, 2041 183 -> 117 (0.88 PFLOP/s with all three products counted); 10 heads, 700 rows 42.5 -> 25; 4 heads of 64, 2000
// rows 72 -> 35.
// RT = 2 halves the K and V traffic per row and is used once its blocks are more than the compute units: 32 heads of 128, RT = 1 / 2,
// 900 rows (256 blocks of 128) 40.5 / 46.2, 1300 rows 77 / 64, 2041 rows 154 / 117; 40 heads of 128, 769 rows (280 blocks) 39.7 / 40.0,
// 896 rows 47.8 / 46.7, 1100 rows 68 / 59, 2041 rows 192 / 160.  (32 heads of 64, whose blocks are half the work: 1300 rows 32 / 43,
// 2041 rows 69 / 72, a line that lies too low for them.)  2041 rows: the matrix cores are busy 38 % of the launch, and 30 % of the LDS
// cycles are conflicts (a score operand's lanes of both pages fall into the same half of the banks, V's lanes of a quad take 16
// bytes of every 32; not measured apart).
template <int HD, int RT>
__global__ void __launch_bounds__(PF_ATT_THREADS, 2) pf_att_kernel(PfArgs a)
{
    constexpr int KT = HD / 32, NT = HD / 16;
    constexpr int PAGE_B = KV_PAGE * 2 * HD * 2;             // bytes of one (page, head) record of K or of V
    constexpr int FR = PAGE_B / 1024;                        // kilobytes of it
    constexpr unsigned STAGE = pf_att_stage(HD);
    constexpr int BR = 64 * RT;
    extern __shared__ __align__(16) char lds[];
    int *pages = reinterpret_cast<int *>(lds + 2 * PF_ATT_GROUPS * STAGE);
    const int tid = threadIdx.x, lane = tid & 63, grp = __builtin_amdgcn_readfirstlane(tid >> 8), wave = __builtin_amdgcn_readfirstlane((tid >> 6) & 3);
    const int lm = lane & 15, quad = lane >> 4;
    const int n_blk = (a.rows + BR - 1) / BR;
    // heads fastest; the row blocks with the most positions first, so that the short ones fill the end
    const int head = blockIdx.x % a.H, blk = n_blk - 1 - blockIdx.x / a.H;
    const int r0 = blk * BR, nr = min(BR, a.rows - r0);
    const int n_pos = a.pos0 + r0 + nr;
    const int n_pg = (n_pos + KV_PAGE - 1) / KV_PAGE, steps = (n_pg + 1) / 2;
    for (int i = tid; i < n_pg; i += PF_ATT_THREADS) pages[i] = a.contig_base >= 0 ? a.contig_base + i : as_global(a.page_table)[i];

    // q of this wave's rows as MFMA operands
    const int row0 = r0 + wave * 16 * RT;                    // first row of this wave
    bf16x8_t qh[RT][KT], ql[RT][KT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const float *qp = a.b.q + (size_t)min(row0 + t * 16 + lm, a.rows - 1) * a.d + head * HD + quad * 8;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
            const f32x4_t x = *as_global(reinterpret_cast<const f32x4_t *>(qp + kt * 32)), y = *as_global(reinterpret_cast<const f32x4_t *>(qp + kt * 32 + 4));
            split_bf16x8(x, y, qh[t][kt], ql[t][kt]);
        }
    }
    wait_vmem();
    __syncthreads();                                         // the page list is there; no load is pending

    // wave w copies K (w even) or V (w odd) of page w >> 1 of its group's step; K is gathered into operand order
    const bool is_v = wave & 1;
    const int src_off = is_v ? lane * 16 : lm * (2 * HD * 2) + quad * 16;
    const char *ring = lds + grp * 2 * STAGE;                // this group's two buffers
    const unsigned lds0 = lds_offset(ring);
    auto request = [&](int step, int buf) __attribute__((always_inline)) {
        const int page = __builtin_amdgcn_readfirstlane(pages[min(2 * step + (wave >> 1), n_pg - 1)]);
        const size_t rec = (((size_t)a.layer * a.n_pages + page) * a.H + head) * PAGE_B;
        const char *src = reinterpret_cast<const char *>(is_v ? a.vpool : a.kpool) + rec;
        const unsigned dst = lds0 + buf * STAGE + wave * PAGE_B;   // [page 0: K, V][page 1: K, V]
#pragma unroll
        for (int f = 0; f < FR; ++f)                          // K: operand (32 values kt, term) = f; V: plain copy
            load_lds_kb(uniform_ptr(src + (is_v ? f * 1024 : (f & 1) * HD * 2 + (f >> 1) * 64)), src_off, dst + f * 1024);
    };
    if (grp < steps) request(grp, 0);

    // the score operands' lanes: row lm of operand p is position 8 (lm >> 2) + 4 p + (lm & 3) of the step; V: the lane's eight positions
    int koff[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int pos = 8 * (lm >> 2) + 4 * p + (lm & 3);
        koff[p] = (pos / KV_PAGE) * (2 * PAGE_B) + (quad * 16 + pos % KV_PAGE) * 16;
    }
    const int voff = PAGE_B + (quad >> 1) * (2 * PAGE_B) + lm * 32 + (quad & 1) * 16;

    f32x4_t O[RT][NT];
    float mx[RT], sum[RT];                                   // maxima of the scaled scores, times log2(e)
    const float scale = a.att_scale * 1.44269504f;
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        mx[t] = ATT_NEG;
        sum[t] = 0.f;
#pragma unroll
        for (int n = 0; n < NT; ++n) O[t][n] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    }
    const int wave_last = a.pos0 + min(row0 + 16 * RT, a.rows) - 1;   // last position a row of this wave sees
    for (int round = 0; round * PF_ATT_GROUPS < steps; ++round) {     // (both groups run the same number of rounds)
        const int step = round * PF_ATT_GROUPS + grp;
        wait_pending<0>();
        lds_barrier();
        if (step + PF_ATT_GROUPS < steps) request(step + PF_ATT_GROUPS, (round + 1) & 1);
        if (step >= steps || step * 32 > wave_last || row0 >= a.rows) continue;
        const char *st = ring + (round & 1) * STAGE;
        f32x4_t S[RT][2];
#pragma unroll
        for (int t = 0; t < RT; ++t) S[t][0] = S[t][1] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const bf16x8_t kh = *reinterpret_cast<const bf16x8_t *>(st + koff[p] + (2 * kt) * 1024);
                const bf16x8_t kl = *reinterpret_cast<const bf16x8_t *>(st + koff[p] + (2 * kt + 1) * 1024);
#pragma unroll
                for (int t = 0; t < RT; ++t) {
                    S[t][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh, qh[t][kt], S[t][p], 0, 0, 0);
                    S[t][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kl, qh[t][kt], S[t][p], 0, 0, 0);
                    S[t][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh, ql[t][kt], S[t][p], 0, 0, 0);
                }
            }
        bf16x8_t Ph[RT], Pl[RT];
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            float s[8], local = ATT_NEG;
#pragma unroll
            for (int e = 0; e < 8; ++e) s[e] = S[t][e >> 2][e & 3];
            if (step * 32 + 31 > a.pos0 + row0 + t * 16) {   // (some row of the tile does not see the whole step)
                const int last = a.pos0 + row0 + t * 16 + lm - step * 32 - quad * 8;
#pragma unroll
                for (int e = 0; e < 8; ++e) s[e] = e <= last ? s[e] : -INFINITY;   // (weighs nothing, also in a row that sees no position of the step)
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) local = fmaxf(local, s[e]);
            local = fmaxf(local, __shfl_xor(local, 16, 64));
            local = fmaxf(local, __shfl_xor(local, 32, 64)) * scale;
            if (__any(local > mx[t])) {
                const float m_new = fmaxf(mx[t], local), f = __builtin_amdgcn_exp2f(mx[t] - m_new);
                mx[t] = m_new;
                sum[t] *= f;
#pragma unroll
                for (int n = 0; n < NT; ++n)
#pragma unroll
                    for (int r = 0; r < 4; ++r) O[t][n][r] *= f;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                s[e] = __builtin_amdgcn_exp2f(fmaf(s[e], scale, -mx[t]));
                sum[t] += s[e];
            }
            split_bf16x8((f32x4_t){s[0], s[1], s[2], s[3]}, (f32x4_t){s[4], s[5], s[6], s[7]}, Ph[t], Pl[t]);
        }
#pragma unroll
        for (int n = 0; n < NT; ++n) {                       // V record: [term][dim][16 positions]
            const bf16x8_t Vh = *reinterpret_cast<const bf16x8_t *>(st + voff + n * 512);
            const bf16x8_t Vl = *reinterpret_cast<const bf16x8_t *>(st + voff + HD * 32 + n * 512);
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                O[t][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Vh, Ph[t], O[t][n], 0, 0, 0);
                O[t][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Vh, Pl[t], O[t][n], 0, 0, 0);
                O[t][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Vl, Ph[t], O[t][n], 0, 0, 0);
            }
        }
    }
    // group 1's results: [tile of the wave][outputs, maximum and sum][lane].  A row of which it saw no position has the maximum
    // ATT_NEG there, and weighs nothing (group 0 sees position 0 of every row).
    lds_barrier();                                           // the last step has been read
    constexpr int REC = (NT * 4 + 2) * 64;                   // floats of a row tile
    static_assert(4 * RT * REC * 4 <= 2 * PF_ATT_GROUPS * (int)STAGE, "inside the ring");
    float *rec = reinterpret_cast<float *>(lds) + wave * RT * REC;
    if (grp == 1) {
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            float *w = rec + t * REC;
#pragma unroll
            for (int n = 0; n < NT; ++n) *reinterpret_cast<float4 *>(w + (n * 64 + lane) * 4) = make_float4(O[t][n][0], O[t][n][1], O[t][n][2], O[t][n][3]);
            *reinterpret_cast<float2 *>(w + NT * 256 + lane * 2) = make_float2(mx[t], sum[t]);
        }
    }
    lds_barrier();
    if (grp == 1) return;
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const float *w = rec + t * REC;
        const float2 o = *reinterpret_cast<const float2 *>(w + NT * 256 + lane * 2);
        const float m_all = fmaxf(mx[t], o.x), f0 = __builtin_amdgcn_exp2f(mx[t] - m_all), f1 = __builtin_amdgcn_exp2f(o.x - m_all);
        float s = sum[t] * f0 + o.y * f1;
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        const int m = row0 + t * 16 + lm;
        const float inv = 1.0f / s, c0 = f0 * inv, c1 = f1 * inv;
        if (m < a.rows) {
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const float4 x = load_f4(w + (n * 64 + lane) * 4);
                const float v[4] = {O[t][n][0] * c0 + x.x * c1, O[t][n][1] * c0 + x.y * c1, O[t][n][2] * c0 + x.z * c1, O[t][n][3] * c0 + x.w * c1};
                pf_store_split4(a.b.attn, a.b.rt, m, head * HD + n * 16 + quad * 4, v);
            }
        }
    }
}

// The address of a GEMM kernel of the chunk; the kernels are in translation units of their own (ee_pf_gemm_*.hip).
typedef void (*pf_kernel_t)(PfArgs);
template <int KIND, int WN, int WM, int GRP>
pf_kernel_t pf_gemm_of();
// The tile shapes there are: wn, wm, groups (pf_gemm_kernel)
#define EE_PF_SHAPES(X) X(8, 4, 1) X(4, 4, 1) X(4, 2, 1) X(2, 2, 1) X(4, 4, 2) X(4, 2, 2) X(2, 2, 4)

}  // namespace ee
