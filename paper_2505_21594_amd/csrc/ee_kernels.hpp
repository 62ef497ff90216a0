// gfx950 kernels of the verification pass.
//
// A segment of the pass (embedding, a range of layers, optionally an LM head with its
// accept step) is a list of stages, one launch each.  Per layer (Eq. 3 of the paper,
// f = Llama-2 block) there are five:
//   QKV   x_hat . [Wq;Wk;Wv]^T, * rstd, RoPE, q -> scratch, k/v -> paged bf16 cache
//   ATT   causal attention of the new rows over the cache         -> attn
//   O     h += attn . Wo^T
//   GU    u = silu(rstd * x_hat.Wg^T) * (rstd * x_hat.Wu^T)
//   DN    h += u . Wd^T
// Head (z^(l) = LMHead(h^(l)); accept rule of Eq. 2 / Eq. 5; confidence of Eq. 4):
//   HEAD    x_hat . W_lm^T, * rstd, argmax candidate and softmax denominator per workgroup
//   ACCEPT  global argmax (lowest id wins ties), confidence, accept length, publication
//           to pinned host memory (run by the head launch's last workgroup; the host commits).
// Kernels: ee_gemm_kernel<KIND, XC> for the GEMM kinds (rows <= 8 XC, at most 48),
// ee_att_kernel, ee_misc_kernel (embedding).
//
// Every GEMM stage streams the weights once (HBM-bound).  A workgroup owns whole
// n-tiles for the full K, so its outputs are complete after a cross-wave sum in
// LDS and the element-wise epilogue runs in the same stage.  RMSNorm is split:
// the GEMM input is g * h (written by the stage that produces h), the row factor
// rstd = 1/sqrt(mean(h^2)+eps), from per-workgroup partial sums, multiplies the fp32 result.
#pragma once

#include "ee_device.hpp"

namespace ee {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_t;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2_t;
typedef __attribute__((ext_vector_type(3))) unsigned int u32x3_t;

// Pointers read from descriptors in memory are generic to the compiler, and generic loads go
// through the flat path, whose completion also counts against the LDS counter: a wait for an
// LDS read would then drain every weight load in flight.  These helpers state that the
// address is global memory.
#define EE_GLOBAL __attribute__((address_space(1)))
#define EE_LDS __attribute__((address_space(3)))
template <typename T>
__device__ __forceinline__ const EE_GLOBAL T *as_global(const T *p)
{
    return (const EE_GLOBAL T *)(p);
}
// The same for stores.  One generic (flat) access anywhere in a kernel also makes the compiler
// treat the order of returning loads as unknown and wait for all of them at every use.
template <typename T>
__device__ __forceinline__ EE_GLOBAL T *as_global_mut(T *p)
{
    return (EE_GLOBAL T *)(p);
}

// A buffer as a resource in scalar registers: the device-scope accesses below need it (a cache policy per access).
typedef __amdgpu_buffer_rsrc_t WRes;
__device__ __forceinline__ WRes buffer_resource(const void *ptr)
{
    // raw buffer, no stride, maximal range (offsets stay inside the buffer).  The
    // pointer is the same in every lane; saying so keeps the resource in scalar registers.
    const unsigned long long p = reinterpret_cast<unsigned long long>(ptr);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)p), hi = __builtin_amdgcn_readfirstlane((unsigned)(p >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(((unsigned long long)hi << 32) | lo), 0, 0x7FFFFFFF, 0x00020000);
}

__device__ __forceinline__ uint4 load_global16(const void *p)
{
    u32x4_t v = *as_global(reinterpret_cast<const u32x4_t *>(p));
    return make_uint4(v[0], v[1], v[2], v[3]);
}

// Device-scope accesses for the small buffers that one launch's workgroups exchange among
// themselves (attention partials of a split position range, argmax candidates of a head):
// stores write through to memory and loads bypass the per-XCD L2.  Everything else is read-only
// in a launch or crosses a kernel boundary.
__device__ __forceinline__ void store_dev64(void *p, uint2 v)
{
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), ((unsigned long long)v.y << 32) | v.x,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_dev32(float *p, float v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// the same for 16 or 8 bytes at byte offset `off` of a buffer: device-scope cache policy (sc1)
constexpr int CACHE_POLICY_DEVICE = 16;
__device__ __forceinline__ void store_dev128(WRes r, int off, float4 v)
{
    __builtin_amdgcn_raw_buffer_store_b128((u32x4_t){__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)},
                                           r, off, 0, CACHE_POLICY_DEVICE);
}
__device__ __forceinline__ float4 load_dev128(WRes r, int off)
{
    const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, CACHE_POLICY_DEVICE);
    return make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3]));
}
__device__ __forceinline__ void store_dev64(WRes r, int off, float2 v)
{
    __builtin_amdgcn_raw_buffer_store_b64((u32x2_t){__float_as_uint(v.x), __float_as_uint(v.y)}, r, off, 0, CACHE_POLICY_DEVICE);
}
__device__ __forceinline__ float2 load_dev64(WRes r, int off)
{
    const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, CACHE_POLICY_DEVICE);
    return make_float2(__uint_as_float(v[0]), __uint_as_float(v[1]));
}
__device__ __forceinline__ float load_dev32(const float *p)
{
    return __hip_atomic_load(as_global(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The value itself, but opaque to the optimiser: keeps per-thread index arithmetic of a stage
// from being hoisted to the kernel's start, where it would occupy registers throughout.
__device__ __forceinline__ int opaque(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}
// The launch arguments are several hundred bytes; the compiler fetches their fields where it
// needs them, and every first touch of another 64-byte line is a miss of the scalar cache that
// the wave has to wait out: about 0.22 us each, eight or more in a row at the start of every
// launch.  This reads one word of every line at once, so the misses overlap, and returns the
// argument block through a pointer the compiler cannot trace back, so that none of its own
// fetches can be scheduled before these.  One block of assembly with its wait: the compiler would take the
// register as free as soon as the loads were issued.
__device__ __forceinline__ const PassArgs &warmed_arguments()
{
    unsigned long long ka = reinterpret_cast<unsigned long long>((const void *)__builtin_amdgcn_kernarg_segment_ptr());
    unsigned word;
    constexpr int LINES = (sizeof(PassArgs) + 63 - 4) / 64;   // last word read lies inside the block
    asm volatile(".set ee_line, 0\n\t"
                 ".rept %2\n\t"
                 "s_load_dword %0, %1, ee_line\n\t"
                 ".set ee_line, ee_line + 64\n\t"
                 ".endr\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&s"(word), "+s"(ka)
                 : "n"(LINES)
                 : "memory");
    return *(const PassArgs *)(const __attribute__((address_space(4))) PassArgs *)ka;
}
// all vector memory operations of this wave have completed
// (the builtin, not inline assembly: the compiler's own bookkeeping of loads in flight sees it,
// so code after it is not made to wait again for loads that this wait has already covered)
__device__ __forceinline__ void wait_vmem()
{
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), other counters untouched
    asm volatile("" ::: "memory");
}
// One kilobyte from memory straight into LDS: lane l's 16 bytes at src + off land at LDS byte
// dst + 16 l.  Inline assembly because the compiler makes every LDS read wait for all such loads it
// knows of; here a stage is read while the next ones are on their way, and the kernels wait
// themselves (wait_pending, then a barrier).  No vector register is written; M0 is, and needs one wait
// state before it is used.
__device__ __forceinline__ void load_lds_kb(const void *src, int off, unsigned dst)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(off), "s"(src), "s"(dst)
                 : "m0", "memory");
}
// The same for a packed tile: lane l's 12 bytes at src + off land at dst + 16 l.
__device__ __forceinline__ void load_lds_packed(const void *src, int off, unsigned dst)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx3 %0, %1"
                 :
                 : "v"(off), "s"(src), "s"(dst)
                 : "m0", "memory");
}
template <bool PK>
__device__ __forceinline__ void load_lds_tile(const void *src, int lane, unsigned dst)
{
    if (PK)
        load_lds_packed(src, lane * 12, dst);
    else
        load_lds_kb(src, lane * 16, dst);
}
template <int N>
__device__ __forceinline__ void wait_pending()   // at most N vector memory operations of this wave are pending
{
    static_assert(N < 64, "vmcnt has 6 bits");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ const void *uniform_ptr(const void *p)
{
    const unsigned long long v = reinterpret_cast<unsigned long long>(p);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return reinterpret_cast<const void *>(((unsigned long long)hi << 32) | lo);
}

// LDS byte offset of the dynamic LDS block's start
__device__ __forceinline__ unsigned lds_offset(const char *p)
{
    return __builtin_amdgcn_readfirstlane((unsigned)reinterpret_cast<unsigned long long>((const EE_LDS char *)p));
}
// Workgroup barrier that orders LDS accesses only.  __syncthreads() also waits for every
// vector memory operation of the wave, i.e. for all weight tiles a streaming wave has in
// flight; nothing that crosses these barriers goes through global memory.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// two values as bf16, round to nearest even, packed (a in the low half): one instruction
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    typedef __attribute__((ext_vector_type(2))) float f32x2_t;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){a, b}, bf16x2_t));
}

// ------------------------------------------------------------------ rows

// Fields of session s's descriptor.  Session 0's descriptor travels by value in the launch
// arguments, so the common one-session pass needs no load from memory to find them, and no upload.
// (written so that the two sources are never merged into one pointer of unknown address space)
template <typename T>
__device__ __forceinline__ T sess_pick(bool first, const T &own, const T *other)
{
    T v = own;
    if (!first) v = *as_global(other);
    return v;
}
#define EE_SESS(a, s, field) sess_pick((s) == 0, (a).sess0.field, &(a).sess[s].field)

__device__ __forceinline__ int row_pos(const PassArgs &a, int r)
{
    if (a.mode == 1) return a.pf_pos0 + r;
    int s = div_small(r, a.M);
    return EE_SESS(a, s, kv_len) + (r - s * a.M);
}

// draft i of session s
__device__ __forceinline__ int draft_of(const PassArgs &a, int s, int i)
{
    int v = a.sess0.drafts[i];
    if (s != 0) v = *as_global(&a.sess[s].drafts[i]);
    return v;
}

__device__ __forceinline__ int row_token(const PassArgs &a, int r)
{
    if (a.mode == 1) return a.pf_tokens[r];
    int s = div_small(r, a.M), i = r - s * a.M;
    return i == 0 ? EE_SESS(a, s, pending) : draft_of(a, s, i - 1);
}

// ------------------------------------------------------------------ LDS map

struct Misc {  // views into the misc region of the LDS block
    float *rstd;       // [rows]
    float *rowss;      // [rows]  this workgroup's sum of h^2 per row (O / DN stages)
    int *pos;          // [rows]
    long long *kvoff;  // [rows]  element offset of the row's (layer, page, head 0) record in the KV pools
    float *bestv;      // [rows]
    int *besti;        // [rows]
    float *sume;       // [rows]  sum of exp(logit - bestv) over the columns seen so far
    int *lastf;        // "this workgroup finished the head launch last"
};

constexpr int MISC_BYTES = EE_MAX_ROWS * (8 + 6 * 4) + 64;

__device__ __forceinline__ Misc misc_views(const StageLds &ly, char *lds)
{
    Misc m;
    char *p = lds + ly.misc_off;
    const int R = EE_MAX_ROWS;
    m.kvoff = reinterpret_cast<long long *>(p);
    p += (size_t)R * 8;
    m.rstd = reinterpret_cast<float *>(p);
    p += (size_t)R * 4;
    m.rowss = reinterpret_cast<float *>(p);
    p += (size_t)R * 4;
    m.pos = reinterpret_cast<int *>(p);
    p += (size_t)R * 4;
    m.bestv = reinterpret_cast<float *>(p);
    p += (size_t)R * 4;
    m.besti = reinterpret_cast<int *>(p);
    p += (size_t)R * 4;
    m.sume = reinterpret_cast<float *>(p);
    p += (size_t)R * 4;
    m.lastf = reinterpret_cast<int *>(p);
    return m;
}

// ------------------------------------------------------------------ weight-stream geometry

__device__ __host__ inline void wg_units(const GemmPlan &pl, int g, int &nt0, int &n_local)
{
    const int j = g >> pl.ksl;
    nt0 = (j * pl.base + (j < pl.rem ? j : pl.rem)) * pl.tpu;
    n_local = g < pl.nwg ? (pl.base + (j < pl.rem ? 1 : 0)) * pl.tpu : 0;  // workgroups past the stage's count own nothing
}

// k-steps of streaming wave w: its k-tiles are w, w + SWAVES, ...
__device__ __host__ inline int wave_ksteps(int KT, int w) { return KT > w ? (KT - w + SWAVES - 1) / SWAVES : 0; }

// ------------------------------------------------------------------ GEMM stage

struct GemmIn {
    const char *x;      // the input (already scaled by the norm gain) as two bf16 terms, k-tile-major (x_index); K split: the slice
    const float *ss;    // [rows][SS_LD] partial sums of squares for rstd, or nullptr
};

// GEMM inputs are stored the way the stages consume them: [k-tile][term][row][32] bf16 with
// `rows` = the rows of this pass, term 0 = hi, 1 = lo.  A range of k-tiles (all rows, both
// terms) is then one contiguous range, which 1 KB loads copy straight into LDS, and the 16 rows x
// 4 quads of one MFMA operand read one contiguous kilobyte of LDS.
__device__ __forceinline__ size_t x_index(int rows, int m, int k, int term)
{
    return ((size_t)((k >> 5) * 2 + term) * rows + m) * 32 + (k & 31);
}

// split x into two bf16 terms: hi = bf16(x), lo = bf16(x - hi).  The MFMA takes bf16 operands;
// feeding both terms keeps about 16 mantissa bits of the activations (weights are exact
// bf16).  The matrix cores idle most of the time in the HBM-bound loop, so the second MFMA
// per tile is free.
// Two values at a time, packed: six instructions for both (about twenty with the rounding done in integers).
__device__ __forceinline__ void split_bf16(float a, float b, uint32_t &hi, uint32_t &lo)
{
    hi = pack_bf16(a, b);
    lo = pack_bf16(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xFFFF0000u));
}

// four consecutive columns k .. k+3 (k a multiple of 4) of row m
__device__ __forceinline__ void store_split4(uint16_t *x, int rows, int m, int k, const float *v)
{
    uint32_t h[2], l[2];
    split_bf16(v[0], v[1], h[0], l[0]);
    split_bf16(v[2], v[3], h[1], l[1]);
    *reinterpret_cast<EE_GLOBAL u32x2_t *>(as_global_mut(x) + x_index(rows, m, k, 0)) = (u32x2_t){h[0], h[1]};
    *reinterpret_cast<EE_GLOBAL u32x2_t *>(as_global_mut(x) + x_index(rows, m, k, 1)) = (u32x2_t){l[0], l[1]};
}

// rstd[m] = 1/sqrt(sum_g ss[m][g] / d + eps) into LDS, fixed summation order; helper waves only, for
// rows <= 8 XC.  A row's partial sums are one kilobyte (slots past the workgroups stay zero), all of a
// wave's rows are requested together.  (With the slots of a row apart, as [g][m], these few kilobytes were
// 64 cache lines per load: as many requests as the whole GEMM input, in front of the weight stream.)
template <int XC>
struct RowFactors {
    f32x4_t v[2 * XC];
    __device__ __forceinline__ void request(const float *ss, int rows, int hwave, int lane)
    {
#pragma unroll
        for (int i = 0; i < 2 * XC; ++i) {
            const int m = min(hwave + i * HWAVES, rows - 1);
            v[i] = *as_global(reinterpret_cast<const f32x4_t *>(ss + (size_t)m * SS_LD + lane * 4));
        }
    }
    __device__ __forceinline__ void finish(int rows, int d, float eps, float *rstd_lds, int hwave, int lane)
    {
#pragma unroll
        for (int i = 0; i < 2 * XC; ++i) {
            float s = (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
            const int m = hwave + i * HWAVES;
            if (lane == 0 && m < rows) rstd_lds[m] = 1.0f / sqrtf(s / (float)d + eps);
        }
    }
};

__device__ __forceinline__ bool cand_better(float v, int i, float bv, int bi)
{
    return v > bv || (v == bv && i < bi);
}

__device__ __forceinline__ float4 load_f4(const float *p) { return *reinterpret_cast<const float4 *>(p); }

// Adapters of several exits in one launch: which of them this workgroup works for.
template <int KIND>
__device__ __forceinline__ int exit_of()
{
    return KIND == G_AD || KIND == G_AU ? (int)blockIdx.y : 0;
}

struct GemmEpi {           // what the O / DN / AU epilogue produces besides h
    const float *gain_xn;  // gain of the next GEMM input (xn), or nullptr
    const float *gain_xh;  // gain of the LM-head input (xh, at the exit's head rows), or nullptr
    float *ss_out;         // [rows][SS_LD] partial sums of h^2, or nullptr
    float *ss_head;        // [head rows][SS_LD] partial sums of squares of the LM-head input's rows (at the head rows), or nullptr
    const float *bias;     // AD / AU: bias per output column
    int xa_out;            // DN: also emit h itself as the adapters' input (xa)
};

// Epilogue of one chunk of gn n-tiles starting at n-tile nt_first: sum the nsum partial tiles in
// the slot buffer (the streaming waves', or the K splits' when K is split over workgroups; fixed
// order), apply the stage's element-wise tail.  All threads.
// Packed weights: `corr` are the chunk's sums over the escapes, in the slot buffer's order (CORR false: the partial tiles hold them).
template <int KIND, bool PK, bool CORR>
__device__ __forceinline__ void gemm_epilogue(const PassArgs &a, const StageLds &ly, int nt_first,
                                              int gn, int rows, const GemmEpi &ep, const Misc &mi, char *lds, const int nsum, const float *corr)
{
    const ModelDev &md = a.mdv;
    const float *slots = reinterpret_cast<const float *>(lds);
    const int tid = opaque(threadIdx.x);
    const size_t wstride = (size_t)ly.chunk * rows * 16;  // floats per wave in the slot buffer
    const int exit = exit_of<KIND>();
    const float *hsrc = KIND == G_AU && a.ha ? a.ha + (size_t)exit * rows * md.d : a.sc.h;
    if (KIND == G_GU) {
        const int items = (gn >> 1) * rows * 4;
        for (int idx = tid; idx < items; idx += WG_THREADS) {
            int p = div_small(idx, rows * 4), rem = idx - p * rows * 4;
            int m = rem >> 2, qd = rem & 3;
            const float *sg = slots + ((size_t)(2 * p) * rows + m) * 16 + qd * 4;
            const float *su = sg + (size_t)rows * 16;
            float4 G = make_float4(0.f, 0.f, 0.f, 0.f), U = G;
#pragma unroll 2
            for (int w = 0; w < nsum; ++w) {
                float4 x = *reinterpret_cast<const float4 *>(sg + w * wstride);
                float4 y = *reinterpret_cast<const float4 *>(su + w * wstride);
                G.x += x.x; G.y += x.y; G.z += x.z; G.w += x.w;
                U.x += y.x; U.y += y.y; U.z += y.z; U.w += y.w;
            }
            float rs = mi.rstd[m];
            if (PK) {
                if (CORR) {
                    const float4 x = load_f4(corr + ((2 * p) * rows + m) * 16 + qd * 4), y = load_f4(corr + ((2 * p + 1) * rows + m) * 16 + qd * 4);
                    G.x += x.x; G.y += x.y; G.z += x.z; G.w += x.w;
                    U.x += y.x; U.y += y.y; U.z += y.z; U.w += y.w;
                }
                rs *= a.entry.wscale;
            }
            float g[4] = {G.x * rs, G.y * rs, G.z * rs, G.w * rs}, u[4] = {U.x * rs, U.y * rs, U.z * rs, U.w * rs};
            float o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = g[e] / (1.0f + __expf(-g[e])) * u[e];
            const int f = ((nt_first >> 1) + p) * 16 + qd * 4;
            store_split4(a.sc.u, rows, m, f, o);
        }
        return;
    }
    float *zbuf = reinterpret_cast<float *>(lds + ly.zbuf_off);  // head: [rows][chunk*16] logits of this chunk; O/DN: squares
    const int items = gn * rows * 4;
    for (int idx = tid; idx < items; idx += WG_THREADS) {
        int ntg = div_small(idx, rows * 4), rem = idx - ntg * rows * 4;
        int m = rem >> 2, qd = rem & 3;
        const int n = (nt_first + ntg) * 16 + qd * 4;  // four consecutive output columns
        // What the item reads from global memory is requested first, all of it at once: the sum of
        // the partial tiles below then runs while it is on its way (one after the other, after the
        // sum, these loads were two memory latencies at the end of every launch).
        f32x4_t g_a = (f32x4_t){0.f, 0.f, 0.f, 0.f}, g_b = g_a, g_c = g_a;
        int qkv_sect = 0, qkv_c = 0, qkv_head = 0, qkv_e = 0, qkv_ses = 0;
        if (KIND == G_O || KIND == G_DN || KIND == G_AU) {
            if (n < md.d) {
                g_a = *as_global(reinterpret_cast<const f32x4_t *>(hsrc + (size_t)m * md.d + n));
                if (KIND == G_AU) g_b = *as_global(reinterpret_cast<const f32x4_t *>(ep.bias + n));
                if (ep.gain_xn) g_b = *as_global(reinterpret_cast<const f32x4_t *>(ep.gain_xn + n));
                if (ep.gain_xh) g_c = *as_global(reinterpret_cast<const f32x4_t *>(ep.gain_xh + n));
            }
        } else if (KIND == G_QKV) {
            qkv_sect = div_small(n, md.d);
            qkv_c = n - qkv_sect * md.d;
            qkv_head = div_small(qkv_c, md.hd);
            qkv_e = qkv_c - qkv_head * md.hd;
            qkv_ses = a.mode == 1 ? 0 : div_small(m, a.M);
            if (qkv_sect < 2)  // (cos, sin) of the row's position for the RoPE pairs of these four columns
                g_a = *as_global(reinterpret_cast<const f32x4_t *>(EE_SESS(a, qkv_ses, rope) + (size_t)mi.pos[m] * (md.hd >> 1) + (qkv_e >> 1)));
        } else if (KIND == G_AD) {
            if (n < md.A) g_a = *as_global(reinterpret_cast<const f32x4_t *>(ep.bias + n));
        }
        const float *sp = slots + ((size_t)ntg * rows + m) * 16 + qd * 4;
        float4 S = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
        for (int w = 0; w < nsum; ++w) {
            float4 x = *reinterpret_cast<const float4 *>(sp + w * wstride);
            S.x += x.x; S.y += x.y; S.z += x.z; S.w += x.w;
        }
        if (PK) {
            if (CORR) {
                const float4 x = load_f4(corr + idx * 4);
                S.x += x.x; S.y += x.y; S.z += x.z; S.w += x.w;
            }
            const float f = a.entry.wscale;
            S.x *= f; S.y *= f; S.z *= f; S.w *= f;
        }
        if (KIND == G_AD) {
            // hidden units of the exit head's adapters: silu(W_down . h + b_down)
            if (n < md.A) {
                const f32x4_t b = g_a;
                float pre[4] = {S.x + b[0], S.y + b[1], S.z + b[2], S.w + b[3]}, o[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = pre[e] / (1.0f + __expf(-pre[e]));
                store_split4(a.sc.t + exit * a.t_next, rows, m, n, o);
            }
        } else if (KIND == G_O || KIND == G_DN || KIND == G_AU) {
            float sq = 0.f;
            if (n < md.d) {
                EE_GLOBAL f32x4_t *hp = reinterpret_cast<EE_GLOBAL f32x4_t *>(as_global_mut(a.sc.h) + (size_t)m * md.d + n);
                const f32x4_t hv = g_a;
                float v[4] = {hv[0] + S.x, hv[1] + S.y, hv[2] + S.z, hv[3] + S.w};
                if (KIND == G_AU) {  // a side branch: a = h + W_up . t + b_up feeds the exit's LM head, h stays as it is
                    const f32x4_t b = g_b;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] += b[e];
                } else {
                    *hp = (f32x4_t){v[0], v[1], v[2], v[3]};
                }
                if (ep.xa_out) {
                    store_split4(a.sc.xa, rows, m, n, v);
                    if (KIND == G_DN && a.ha) *reinterpret_cast<EE_GLOBAL f32x4_t *>(as_global_mut(a.ha) + (size_t)(a.head_row0 + m) * md.d + n) = (f32x4_t){v[0], v[1], v[2], v[3]};
                }
                sq = v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
                if (ep.gain_xn) {
                    const f32x4_t g = g_b;
                    float x[4] = {v[0] * g[0], v[1] * g[1], v[2] * g[2], v[3] * g[3]};
                    store_split4(a.sc.xn, rows, m, n, x);
                }
                if (ep.gain_xh) {
                    const f32x4_t g = g_c;
                    float x[4] = {v[0] * g[0], v[1] * g[1], v[2] * g[2], v[3] * g[3]};
                    store_split4(a.sc.xh, a.head_rows, a.head_row0 + exit * rows + m, n, x);
                }
            }
            zbuf[idx] = sq;  // (ntg, m, quad) order
        } else if (KIND == G_QKV) {
            const int d = md.d, hd = md.hd;
            const float rs = mi.rstd[m];
            float v[4] = {S.x * rs, S.y * rs, S.z * rs, S.w * rs};
            const int sect = qkv_sect, c = qkv_c, head = qkv_head, e = qkv_e, ses = qkv_ses;
            if (sect < 2) {
                // columns are pair-interleaved inside a head: (e, e+1) = RoPE pair e/2
                const f32x4_t cs = g_a;
                float y0 = v[0] * cs[0] - v[1] * cs[1], y1 = v[1] * cs[0] + v[0] * cs[1];
                float y2 = v[2] * cs[2] - v[3] * cs[3], y3 = v[3] * cs[2] + v[2] * cs[3];
                v[0] = y0; v[1] = y1; v[2] = y2; v[3] = y3;
            }
            if (sect == 0) {
                *reinterpret_cast<EE_GLOBAL f32x4_t *>(as_global_mut(a.sc.q) + (size_t)m * d + c) = (f32x4_t){v[0], v[1], v[2], v[3]};
            } else {
                // cached value = hi + lo, two bf16 terms.  K: [position][term][hd]; V transposed
                // inside the page: [term][hd][position] (see the attention stage)
                uint32_t vh[2], vl[2];
                split_bf16(v[0], v[1], vh[0], vl[0]);
                split_bf16(v[2], v[3], vh[1], vl[1]);
                const size_t rec = mi.kvoff[m] + (size_t)head * KV_PAGE * 2 * hd;  // this (page, head) record
                const int slot = mi.pos[m] % KV_PAGE;
                if (sect == 1) {
                    EE_GLOBAL uint16_t *kr = as_global_mut(EE_SESS(a, ses, kpool)) + rec + (size_t)slot * 2 * hd + e;
                    *reinterpret_cast<EE_GLOBAL u32x2_t *>(kr) = (u32x2_t){vh[0], vh[1]};
                    *reinterpret_cast<EE_GLOBAL u32x2_t *>(kr + hd) = (u32x2_t){vl[0], vl[1]};
                } else {
                    EE_GLOBAL uint16_t *vr = as_global_mut(EE_SESS(a, ses, vpool)) + rec + slot;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        vr[(size_t)(e + t) * KV_PAGE] = (uint16_t)(vh[t >> 1] >> (16 * (t & 1)));
                        vr[(size_t)(hd + e + t) * KV_PAGE] = (uint16_t)(vl[t >> 1] >> (16 * (t & 1)));
                    }
                }
            }
        } else {  // G_HEAD
            const float rs = mi.rstd[m];
            float z[4] = {S.x * rs, S.y * rs, S.z * rs, S.w * rs};
            float *zr = zbuf + (size_t)m * ly.chunk * 16 + ntg * 16 + qd * 4;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (n + e >= md.V) z[e] = -INFINITY;
                zr[e] = z[e];
            }
            if (a.keep_logits) {
                const int per_head = a.n_sess * a.M, hj = m / per_head;  // the launch's rows: head after head
                EE_GLOBAL float *keep = as_global_mut(a.sc.logits) + ((size_t)(a.head_idx + hj) * md.rows_max + (m - hj * per_head)) * md.V;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < md.V) keep[n + e] = z[e];
            }
        }
    }
    if (KIND == G_O || KIND == G_DN || KIND == G_AU) {
        lds_barrier();
        if (tid < rows) {  // this chunk's sum of squares per row, fixed order
            float t = 0.f;
            for (int ntg = 0; ntg < gn; ++ntg)
                for (int qd = 0; qd < 4; ++qd) t += zbuf[(ntg * rows + tid) * 4 + qd];
            mi.rowss[tid] += t;
        }
    }
    if (KIND == G_HEAD) {
        lds_barrier();
        // Sixteen lanes per row (all rows at once, 48 groups): lane l has column l of every n-tile of the chunk.
        static_assert(WG_THREADS / 16 >= EE_MAX_ROWS && GROUP_TILES <= 8, "a group of lanes per row");
        const int m = tid >> 4, l = tid & 15;
        float z[GROUP_TILES], bv = -INFINITY;
        int bi = 0x7FFFFFFF;
        const float *zr = zbuf + (size_t)min(m, rows - 1) * ly.chunk * 16 + l;
#pragma unroll
        for (int j = 0; j < GROUP_TILES; ++j) {
            z[j] = j < gn ? zr[j * 16] : -INFINITY;
            if (z[j] > bv) {
                bv = z[j];
                bi = (nt_first + j) * 16 + l;
            }
        }
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) {
            const float ov = __shfl_xor(bv, off, 64);
            const int oi = __shfl_xor(bi, off, 64);
            if (cand_better(ov, oi, bv, bi)) {
                bv = ov;
                bi = oi;
            }
        }
        // sum of exp(z - bv) over the chunk's columns (masked columns hold -inf and add 0):
        // the softmax denominator for the confidence score (paper Eq. 4), kept relative to the
        // running maximum like the argmax candidate
        float se = 0.f;
#pragma unroll
        for (int j = 0; j < GROUP_TILES; ++j) se += __expf(z[j] - bv);
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) se += __shfl_xor(se, off, 64);
        if (l == 0 && m < rows && bv > -INFINITY) {  // (a chunk of masked columns only contributes nothing)
            const float ov = mi.bestv[m];
            if (cand_better(bv, bi, ov, mi.besti[m])) {
                mi.sume[m] = mi.sume[m] * __expf(ov - bv) + se;  // exp(-inf) = 0 the first time
                mi.bestv[m] = bv;
                mi.besti[m] = bi;
            } else {
                mi.sume[m] += se * __expf(bv - ov);
            }
        }
    }
}

// K split over workgroups: instead of the epilogue, one chunk of gn n-tiles of this workgroup's
// partial sums (the streaming waves' tiles added up, fixed order, and packed weights' escapes) goes to memory, to
// part[split][n-tile][row][16].  All threads.
template <bool PK>
__device__ __forceinline__ void partial_store(const PassArgs &a, const GemmPlan &pl, const StageLds &ly, int nt_first, int gn,
                                              int rows, const char *lds, const float *corr)
{
    const float *slots = reinterpret_cast<const float *>(lds);
    const int tid = opaque(threadIdx.x);
    const size_t wstride = (size_t)ly.chunk * rows * 16;
    const int sp = blockIdx.x & ((1 << pl.ksl) - 1);
    const WRes out = buffer_resource(a.sc.part + ((size_t)sp * pl.NT + nt_first) * rows * 16);
    const int items = gn * rows * 4;            // (n-tile, row, quad of columns): the slot buffer's own order
    for (int idx = tid; idx < items; idx += WG_THREADS) {
        const float *p = slots + (size_t)idx * 4;
        float4 S = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
        for (int w = 0; w < SWAVES; ++w) {
            float4 x = *reinterpret_cast<const float4 *>(p + w * wstride);
            S.x += x.x; S.y += x.y; S.z += x.z; S.w += x.w;
        }
        if (PK) {
            const float4 x = load_f4(corr + idx * 4);
            S.x += x.x; S.y += x.y; S.z += x.z; S.w += x.w;
        }
        store_dev128(out, idx * 16, S);
    }
}

// K split over workgroups, after the workgroup's last group: count this split in its group's
// counter; the workgroup that arrives last (the counter goes back to zero for the next launch)
// fetches all splits' partial tiles, chunk by chunk, into the slot buffer in split order and
// runs the epilogue on them.  The result does not depend on who arrives last; nothing waits.
template <int KIND, bool PK>
__device__ __forceinline__ void split_finish(const PassArgs &a, const GemmPlan &pl, const StageLds &ly,
                                             const GemmEpi &ep, const Misc &mi, char *lds, int nt0, int n_local)
{
    const int tid = opaque(threadIdx.x);
    const int rows = a.rows, ks = 1 << pl.ksl;
    wait_vmem();      // this workgroup's partial tiles are visible device-wide ...
    __syncthreads();  // ... for every wave, before it is counted
    if (tid == 0) {
        int *cnt = a.sc.part_count + (blockIdx.x >> pl.ksl);
        const int before = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *mi.lastf = before == ks - 1 ? 1 : 0;
        if (*mi.lastf) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!*mi.lastf) return;
    float *slots = reinterpret_cast<float *>(lds);
    const size_t wstride = (size_t)ly.chunk * rows * 16;
    const WRes part = buffer_resource(a.sc.part);
    for (int c0 = 0; c0 < n_local; c0 += ly.chunk) {
        const int gn = min(ly.chunk, n_local - c0);
        const int per = gn * rows * 4;          // 16-byte items of one split's chunk
        for (int idx = tid; idx < ks * per; idx += WG_THREADS) {
            const int s = div_small(idx, per), rem = idx - s * per;
            // (byte offsets stay far below 2^31: the buffer holds splits x n-tiles x rows x 64 bytes)
            *reinterpret_cast<float4 *>(slots + s * wstride + (size_t)rem * 4) =
                load_dev128(part, (int)((((size_t)s * pl.NT + nt0 + c0) * rows * 16 + (size_t)rem * 4) * sizeof(float)));
        }
        lds_barrier();
        gemm_epilogue<KIND, PK, false>(a, ly, nt0 + c0, gn, rows, ep, mi, lds, ks, nullptr);
        lds_barrier();
    }
}

// A streaming wave's ring of stages in LDS.  A stage is one k-step: NL weight tiles and the XC kilobytes
// of the step's input k-tile.  As many stages as fit RING_KB (at least one; WAVE_LDS_KB holds the largest
// stage, NL = 8 with XC = 6): eight waves then have 8 D (NL + XC) KB on their way, 40 (one stage of five tiles: NL = 4,
// XC = 1) to 112.  More does not stream faster where it was measured, a compute unit's requests are served in order and the input's would wait behind
// more weight tiles (ms per pass, headline workload, 8 / 12 / 19 KB: 3.16 / 3.18 / 3.19).
constexpr int RING_KB = 8;
constexpr int WAVE_LDS_KB = GROUP_TILES + (EE_MAX_ROWS + 7) / 8;
// (a division by comparisons: the kernels need it before they know anything else)
__device__ __host__ constexpr int ring_depth(int xc, int nl)
{
    const int per = nl + xc;
    return per <= 2 ? 4 : (per <= 4 ? 2 : 1);
}
constexpr bool ring_depth_ok()
{
    for (int xc = 1; xc <= EE_MAX_ROWS / 8; ++xc)
        for (int nl = 1; nl <= GROUP_TILES; ++nl) {
            const int d = RING_KB / (nl + xc);
            if (ring_depth(xc, nl) != (d < 1 ? 1 : d) || ring_depth(xc, nl) * (nl + xc) > WAVE_LDS_KB) return false;
        }
    return true;
}
static_assert(ring_depth_ok(), "as many stages as fit RING_KB, at least one, inside the wave's part of LDS");

// Lane's offset in the last of the XC kilobytes of an input k-tile: lanes past its end (rows that are no multiple of 8) read its last 16
// bytes again.  What a unit loads is bound by the bytes of its lines.
template <int XC>
__device__ __forceinline__ int x_last_offset(int tile_bytes, int lane)
{
    return min(lane * 16, tile_bytes - (XC - 1) * 1024 - 16);
}

// The start of a GEMM launch: every streaming wave requests the stages its ring holds, before anything else is read or
// worked out.  A launch's instructions come from a cold instruction cache, a line at a time, and its arguments from a
// cold scalar cache: the code up to these requests is 70 instructions (loops, not unrolled) and needs one line of arguments.
// With the requests behind the warming of all arguments and the plan's arithmetic, us per launch, 5 rows of the 7B shape: QKV
// 18.6 -> 18.3, gate/up 30.9 -> 30.0, down 18.1 -> 17.9, head 50.0 -> 49.0; 40 rows, 8 layers, a pass 1390 -> 1372.
template <int KIND, int XC, bool PK>
__device__ __forceinline__ void gemm_entry(char *lds)
{
    typedef unsigned int u32x16_t __attribute__((ext_vector_type(16), aligned(16)));
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = blockIdx.x;
    if (wave >= SWAVES) return;   // (the helper waves do not wait for this line before they ask for the others)
    const u32x16_t v = *(const __attribute__((address_space(4))) u32x16_t *)__builtin_amdgcn_kernarg_segment_ptr();
    const int tile_bytes = v[5], KTs = v[6], nwg = v[7], base = v[8], rem = v[9], tpu = v[10], ksl = v[11];
    if (g >= nwg) return;
    const int nl = min(GROUP_TILES, (base + ((g >> ksl) < rem ? 1 : 0)) * tpu);
    const int stages = min(ring_depth(XC, nl), wave_ksteps(KTs, wave)), lane = threadIdx.x & 63;
    const int x_last = x_last_offset<XC>(tile_bytes, lane);
    const char *wp = reinterpret_cast<const char *>((((unsigned long long)v[1] << 32) | v[0]) + (unsigned)((g * SWAVES + wave) * tile_bytes_of(PK)));
    const char *xp = reinterpret_cast<const char *>((((unsigned long long)v[3] << 32) | v[2]) + (unsigned)(((g & ((1 << ksl) - 1)) * KTs + wave) * tile_bytes));
    if (KIND == G_AD || KIND == G_AU) {   // (w_next, x_next)
        wp += (long long)(((unsigned long long)v[13] << 32) | v[12]) * blockIdx.y;
        xp += (int)v[14] * (int)blockIdx.y;
    }
    unsigned dst = lds_offset(lds) + wave * (WAVE_LDS_KB * 1024);
#pragma unroll 1
    for (int s = 0; s < stages; ++s) {
#pragma unroll 1
        for (int i = 0; i < nl; ++i) {
            load_lds_tile<PK>(wp, lane, dst);
            wp += (int)v[4];
            dst += 1024;
        }
#pragma unroll
        for (int i = 0; i < XC; ++i) load_lds_kb(xp + i * 1024, i == XC - 1 ? x_last : lane * 16, dst + i * 1024);
        dst += XC * 1024;
        xp += SWAVES * tile_bytes;
    }
}

// A lane's eight weights of a packed tile as an MFMA operand (see PACK_TILE): 11 instructions.
__device__ __forceinline__ bf16x8_t unpack_tile(u32x3_t p)
{
    uint32_t o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t low = __builtin_amdgcn_perm(PACK_CONST, p[j >> 1], j & 1 ? 0x04030402u : 0x04010400u);   // [constant, low byte] x 2
        const uint32_t var = j ? __builtin_amdgcn_alignbit(p[2], p[2], 4 * j) : p[2];
        o[j] = (var & PACK_MASK) | (low & ~PACK_MASK);
    }
    return __builtin_bit_cast(bf16x8_t, make_uint4(o[0], o[1], o[2], o[3]));
}

// Packed weights, helper waves: corr[n-tile][row][16] = sum over the group's escapes of delta * x[row][k].  The host has cut
// the group's escapes (sorted by column, then k; K split over workgroups: those of the slice) into one part per helper wave, at column
// boundaries: a sum is one wave's, in list order.  Lane = row; the inputs of eight escapes are requested together, the first
// ones before the wave's other work, whose latencies then overlap.  The escapes themselves come through the scalar cache: a vector load
// would queue behind the 64 requests of the stream.  A wave has 2 to 13 escapes with normally distributed weights, and a request touches a
// line per row: places that hold none are not requested (with them, 48 rows: gate/up of the 7B shape 40.2 us, now 39.0, of a 2048-wide model
// 22.5, now 21.7).
struct EscapeSums {
    typedef unsigned u32x16_t __attribute__((ext_vector_type(16), aligned(64)));
    typedef const __attribute__((address_space(4))) u32x16_t *list_t;
    list_t list;         // the part, eight escapes (the first one is the header) at a time
    u32x16_t now;
    const char *xm;      // this lane's row of k-tile 0
    int n, c1;           // header: places taken, itself included; first column << 8 | end of the columns
    int rows;
    uint16_t hi[8], lo[8];

    __device__ __forceinline__ void load_part(const PassArgs &a, int group, int hwave, int lane)
    {
        const size_t at = ((size_t)((int)blockIdx.x * a.entry.esc_groups + group) * HWAVES + hwave) * a.entry.esc_cap;
        list = (list_t)(a.entry.esc + at);
        now = list[0];
        n = now[0];
        c1 = now[1] & 0xFFFF;
        rows = a.rows;
        xm = reinterpret_cast<const char *>(a.entry.X) + min(lane, rows - 1) * 64;
    }
    __device__ __forceinline__ void request(int j0)
    {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (j0 + j > 0 && j0 + j < n) {
                const int k = now[2 * j + 1] >> 16;
                const char *p = xm + (size_t)(k >> 5) * (rows * 128) + (k & 31) * 2;
                hi[j] = *as_global(reinterpret_cast<const uint16_t *>(p));
                lo[j] = *as_global(reinterpret_cast<const uint16_t *>(p + rows * 64));
            }
    }
    // the escapes' sums into LDS; n_first is the group's first column
    __device__ __forceinline__ void finish(int n_first, int lane, float *corr)
    {
        const bool live = lane < rows;
        for (int c = c1 >> 8; c < (c1 & 0xFF); ++c)
            if (live) corr[((c >> 4) * rows + lane) * 16 + (c & 15)] = 0.f;
        float sum = 0.f;
        int col = -1;
        for (int j0 = 0; j0 < n; j0 += 8) {
            if (j0) {
                now = list[j0 >> 3];
                request(j0);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (j0 + j > 0 && j0 + j < n) {
                    const int c = (int)((now[2 * j + 1] - (unsigned)n_first) & 0xFFFF);
                    if (c != col) sum = 0.f;
                    col = c;
                    sum += __uint_as_float(now[2 * j]) * (bf16_to_f32(hi[j]) + bf16_to_f32(lo[j]));
                    if (live) corr[((c >> 4) * rows + lane) * 16 + (c & 15)] = sum;   // (the last store of a column is its sum)
                }
        }
    }
};

// One group of NL n-tiles (this workgroup's n-tiles nt_first .. nt_first + NL - 1) over all of K,
// for rows <= 8 XC (MT = 16-row tiles).
//
// Streaming wave w walks its k-steps s = 0 .. (k-tile w + SWAVES*s).  Every k-tile of the input is
// used by one wave only, so the wave brings both operands itself: the step's NL weight tiles and
// the k-tile of the input (all rows, both bf16 terms: contiguous) travel from memory straight into a
// ring of D stages in the wave's own part of LDS.  Nothing is shared between waves until the
// cross-wave sum: there is no barrier in the stream, a wave waits for its own oldest stage, reads it,
// requests the stage D further on into the same place and multiplies.
// Weight tiles into NL x MT accumulators, two MFMAs (two input terms) each.
// Bound by HBM: between the first request (gemm_entry) and the last tile the 7B shape streams at 6.2 to 6.7 TB/s
// with 5 rows.  With helper waves that copied input blocks for all streaming waves, a barrier of
// all waves per block and 8 tiles of every wave in registers instead (us per launch, 5 rows / 40
// rows): QKV 20.4 / 36.2 -> 19.6 / 27.8, gate/up 31.5 / 43.4 -> 31.2 / 37.8, down 19.4 / 27.6 -> 19.0 / 27.0,
// LM head 54 / 86 -> 51 / 70.  Packed weights (PK): three quarters of the bytes, unpacked between LDS and the product by the vector unit that
// is idle otherwise.  us per launch plain -> packed: 5 rows QKV 18.2 -> 15.1, output 8.8 -> 8.4, gate/up 30.2 -> 24.2, down 17.6 -> 15.5, head 49.2
// -> 39.8; 16 rows 19.0 -> 18.1, 10.8 -> 10.6, 30.7 -> 25.7, 23.3 -> 21.7, 50.2 -> 42.0; 39 rows (bound by the input's bytes and the LDS passes
// beside the weights; between events, 2 us more each) 27.8 -> 26.0, 17.1 -> 17.0, 38.6 -> 35.1, 27.4 -> 25.4, 59.9 -> 54.5.
//
// Afterwards the accumulators go through LDS, `ly.chunk` n-tiles at a time, for the
// cross-wave sum and the stage's epilogue (all waves).
template <int KIND, int XC, int NL, bool PK>
__device__ __forceinline__ void gemm_group(const PassArgs &a, const GemmPlan &pl, const StageLds &ly,
                                           const uint4 *__restrict__ W, const GemmIn &in, const GemmEpi &ep, const Misc &mi,
                                           char *lds, int nt_first, int seq0, int group)
{
    constexpr int MT = (XC + 1) / 2, D = ring_depth(XC, NL), PER = NL + XC;
    constexpr int NW = MT == 3 && NL > 4 ? (PK ? 2 : 4) : NL;   // weight tiles read at a time (registers: three waves per SIMD)
    const ModelDev &md = a.mdv;
    const int tid = opaque(threadIdx.x), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rows = a.rows;
    f32x4_t acc[NL][MT];                          // streaming waves only

    if (wave < SWAVES) {
        // ---------------- streaming wave
        const int S_w = wave_ksteps(pl.KTs, wave);
        const int lane16 = lane * 16;
        const size_t wstep = (size_t)pl.nwg * SWAVES * tile_bytes_of(PK);   // bytes from one tile of the wave's sequence to the next
        const char *wp = reinterpret_cast<const char *>(W) + (size_t)seq0 * wstep + ((size_t)blockIdx.x * SWAVES + wave) * tile_bytes_of(PK);
        const int tile_bytes = rows * 128;                     // one k-tile of the input: both terms, all rows
        const int x_last = x_last_offset<XC>(tile_bytes, lane);
        const char *xp = in.x + (size_t)wave * tile_bytes;
        const unsigned ring = lds_offset(lds) + wave * (WAVE_LDS_KB * 1024);
        auto request = [&](unsigned dst) __attribute__((always_inline)) {   // the next stage of the sequence
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                load_lds_tile<PK>(wp, lane, dst + i * 1024);
                wp += wstep;
            }
#pragma unroll
            for (int i = 0; i < XC; ++i) load_lds_kb(xp + i * 1024, i == XC - 1 ? x_last : lane16, dst + (NL + i) * 1024);
            xp += SWAVES * tile_bytes;
        };
        if (group == 0) {                                      // (requested at the kernel's start: gemm_entry)
            wp += D * NL * wstep;
            xp += D * SWAVES * tile_bytes;
        } else {
#pragma unroll
            for (int i = 0; i < D; ++i)
                if (i < S_w) request(ring + i * PER * 1024);
        }
#pragma unroll
        for (int nt = 0; nt < NL; ++nt)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
        int brow[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) brow[mt] = min(mt * 16 + (lane & 15), rows - 1) * 64 + (lane >> 4) * 16;  // bytes inside a k-tile's hi rows
        int slot = 0;
        for (int s = 0; s < S_w; ++s) {
            if (s + D <= S_w)
                wait_pending<(D - 1) * PER>();     // the D - 1 stages requested after this one may still be on their way
            else
                wait_pending<0>();
            const char *st = lds + wave * (WAVE_LDS_KB * 1024) + slot * (PER * 1024);
            bf16x8_t w[NW], xh[MT], xl[MT];
            u32x3_t p[NW];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                xh[mt] = *reinterpret_cast<const bf16x8_t *>(st + NL * 1024 + brow[mt]);
                xl[mt] = *reinterpret_cast<const bf16x8_t *>(st + NL * 1024 + brow[mt] + rows * 64);
            }
#pragma unroll
            for (int n0 = 0; n0 < NL; n0 += NW) {
#pragma unroll
                for (int i = 0; i < NW; ++i)
                    if (n0 + i < NL) {
                        if (PK)
                            p[i] = *reinterpret_cast<const u32x3_t *>(st + (n0 + i) * 1024 + lane16);
                        else
                            w[i] = *reinterpret_cast<const bf16x8_t *>(st + (n0 + i) * 1024 + lane16);
                    }
                if (n0 + NW >= NL) {
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the stage has been read: its place is free
                    if (s + D < S_w) request(ring + slot * (PER * 1024));
                    slot = slot + 1 == D ? 0 : slot + 1;
                }
                if (PK) {
#pragma unroll
                    for (int i = 0; i < NW; ++i)
                        if (n0 + i < NL) w[i] = unpack_tile(p[i]);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
                    for (int i = 0; i < NW; ++i)   // the two terms of a tile in separate sweeps: no MFMA waits for the one before it
                        if (n0 + i < NL) acc[n0 + i][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[i], xh[mt], acc[n0 + i][mt], 0, 0, 0);
#pragma unroll
                    for (int i = 0; i < NW; ++i)
                        if (n0 + i < NL) acc[n0 + i][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[i], xl[mt], acc[n0 + i][mt], 0, 0, 0);
                }
            }
        }
    } else if (PK || group == 0) {
        // ---------------- helper wave: what the epilogue needs, row factors and per-row cache addresses
        const int hwave = wave - SWAVES;
        EscapeSums esc;
        RowFactors<XC> rf;
        const bool factors = in.ss && group == 0;
        if (PK) esc.load_part(a, group, hwave, lane);
        if (factors) rf.request(in.ss, rows, hwave, lane);
        if (PK) esc.request(0);
        if (factors) rf.finish(rows, pl.K, md.eps, mi.rstd, hwave, lane);
        const int ht = tid - SWAVES * 64;
        if (KIND == G_QKV && group == 0 && ht < rows) {
            const int m = ht;
            const int pos = row_pos(a, m);
            const int ses = a.mode == 1 ? 0 : div_small(m, a.M);
            const int cbase = EE_SESS(a, ses, contig_base);
            const int page = cbase >= 0 ? cbase + pos / KV_PAGE : as_global(EE_SESS(a, ses, page_table))[pos / KV_PAGE];
            mi.pos[m] = pos;
            mi.kvoff[m] = (((long long)a.layer * EE_SESS(a, ses, n_pages) + page) * md.H) * KV_PAGE * 2 * md.hd;  // record of head 0
        }
        if (PK) esc.finish(nt_first * 16, lane, reinterpret_cast<float *>(lds + ly.corr_off));
        wait_vmem();
        // The down projection's input: the padding columns of its last k-tile (F = 16 mod 32).  Their place depends on the rows, another
        // pass's values may lie there, and a packed padding weight is not zero (PACK_CODE0).  16 bytes a thread: (term, row) and half.  (Nothing waits for it.)
        if (KIND == G_GU && group == 0 && blockIdx.x == 0 && (md.F & 16) && ht < rows * 4) {
            const int row = ht >> 1;   // [term][row] of the last k-tile
            uint16_t *p = a.sc.u + (size_t)(md.F >> 5) * 2 * rows * 32 + row * 32 + 16 + (ht & 1) * 8;
            *reinterpret_cast<EE_GLOBAL u32x4_t *>(as_global_mut(p)) = (u32x4_t){0, 0, 0, 0};
        }
    }
    // ---- cross-wave sum and epilogue, ly.chunk n-tiles at a time (the rings are free now)
    lds_barrier();                                 // every streaming wave has read its last stage
    float *slots = reinterpret_cast<float *>(lds);
    for (int c0 = 0; c0 < NL; c0 += ly.chunk) {
        const int gn = min(ly.chunk, NL - c0);
        if (wave < SWAVES) {
            // D layout: lane holds rows (lane>>4)*4 .. +3 of N, column (lane&15) of M
#pragma unroll
            for (int nt = 0; nt < NL; ++nt)
                if (nt >= c0 && nt < c0 + gn) {
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        const int m = mt * 16 + (lane & 15);
                        if (m < rows)
                            *reinterpret_cast<float4 *>(slots + (((size_t)wave * ly.chunk + (nt - c0)) * rows + m) * 16 + (lane >> 4) * 4) =
                                make_float4(acc[nt][mt][0], acc[nt][mt][1], acc[nt][mt][2], acc[nt][mt][3]);
                    }
                }
        }
        lds_barrier();
        const float *corr = reinterpret_cast<const float *>(lds + ly.corr_off) + c0 * rows * 16;
        if (MT > 1 && pl.ksl)   // (K is split only for launches of more than one row tile)
            partial_store<PK>(a, pl, ly, nt_first + c0, gn, rows, lds, corr);
        else
            gemm_epilogue<KIND, PK, PK>(a, ly, nt_first + c0, gn, rows, ep, mi, lds, SWAVES, corr);
        lds_barrier();
    }
}

// One GEMM stage of this workgroup: its n-tiles in groups of up to GROUP_TILES.
template <int KIND, int XC, bool PK>
__device__ __forceinline__ void gemm_stage_t(const PassArgs &a, const GemmPlan &pl, const StageLds &ly,
                             const uint4 *__restrict__ W, const GemmIn &in_all, const GemmEpi &ep, char *lds)
{
    constexpr int MT = (XC + 1) / 2;
    const ModelDev &md = a.mdv;
    const int tid = opaque(threadIdx.x);
    const int rows = a.rows;
    const Misc mi = misc_views(ly, lds);
    int nt0, n_local;
    wg_units(pl, blockIdx.x, nt0, n_local);

    const int hrow = tid - SWAVES * 64;   // the first helper wave: one lane per row, here and in hand_over
    static_assert(EE_MAX_ROWS <= 64, "one lane per row");
    if (hrow >= 0 && hrow < rows) {
        mi.bestv[hrow] = -INFINITY;
        mi.besti[hrow] = 0x7FFFFFFF;
        mi.sume[hrow] = 0.f;
        mi.rowss[hrow] = 0.f;
    }
    if (n_local > 0) {
        const int S0 = wave_ksteps(pl.KTs, 0);
        // K split over workgroups: this workgroup's slice of the input (k-tile-major: a contiguous range)
        const GemmIn in = {MT > 1 ? in_all.x + (size_t)(blockIdx.x & ((1 << pl.ksl) - 1)) * pl.KTs * (128 * rows) : in_all.x, in_all.ss};
        int seq = 0;  // tiles of a wave's sequence before the group (waves with fewer k-steps leave their slots unused)
        for (int g0 = 0; g0 < n_local; g0 += GROUP_TILES) {
            const int nl = min(GROUP_TILES, n_local - g0);
#define EE_GROUP(NLV) \
    case NLV: gemm_group<KIND, XC, NLV, PK>(a, pl, ly, W, in, ep, mi, lds, nt0 + g0, seq, g0 / GROUP_TILES); break;
            switch (nl) {
                EE_GROUP(1) EE_GROUP(2) EE_GROUP(3) EE_GROUP(4) EE_GROUP(5) EE_GROUP(6) EE_GROUP(7) EE_GROUP(8)
            }
#undef EE_GROUP
            seq += S0 * nl;
        }
        if (MT > 1 && pl.ksl) split_finish<KIND, PK>(a, pl, ly, ep, mi, lds, nt0, n_local);
    }
    // what the workgroup hands to the following launch
    auto hand_over = [&](int slot, bool mine) __attribute__((always_inline)) {
        const float ss = mine ? mi.rowss[hrow] : 0.f;
        if (ep.ss_out) as_global_mut(ep.ss_out)[(size_t)hrow * SS_LD + slot] = ss;
        if (ep.ss_head) as_global_mut(ep.ss_head)[(size_t)(a.head_row0 + exit_of<KIND>() * rows + hrow) * SS_LD + slot] = ss;
        if (KIND == G_HEAD) {  // device-scope stores: the accept step may run in another workgroup of this launch
            store_dev64(a.sc.cand + (size_t)hrow * SS_LD + slot,
                        make_uint2(__float_as_uint(mine ? mi.bestv[hrow] : -INFINITY), (unsigned)(mine ? mi.besti[hrow] : 0x7FFFFFFF)));
            store_dev32(a.sc.cand_sum + (size_t)hrow * SS_LD + slot, mine ? mi.sume[hrow] : 0.f);
        }
    };
    if (hrow >= 0 && hrow < rows) {
        if (MT > 1 && pl.ksl && n_local > 0) {
            // K split: the group's result was worked out by whichever of its workgroups arrived last; it
            // fills the slots of the whole group, the result in the first, so that what the following
            // launch adds up (in slot order) does not depend on who that was
            if (*mi.lastf) {
                const int ks = 1 << pl.ksl, first = (int)blockIdx.x & ~(ks - 1);
                for (int j = 0; j < ks; ++j) hand_over(first + j, j == 0);
            }
        } else {
            hand_over((int)blockIdx.x, true);
        }
    }
}

// ------------------------------------------------------------------ embedding

// h = embedding of each row's token (or the supplied embedding row); workgroup g owns the
// columns [g*cw, (g+1)*cw) and also emits the first layer's GEMM input and its share of h^2
__device__ __forceinline__ void embed_stage(const PassArgs &a, char *lds)
{
    const ModelDev &md = a.mdv;
    const int d = md.d, rows = a.rows, tid = threadIdx.x;
    const int cw = (div_small(d + a.nwg - 1, a.nwg) + 3) & ~3;  // columns per workgroup, multiple of 4
    const int n0 = blockIdx.x * cw;
    const int nq = max(0, min(cw, d - n0)) >> 2;          // quads of columns here
    float *sq = reinterpret_cast<float *>(lds);           // [rows][cw/4]
    const float *gain = md.g_attn;
    for (int it = tid; it < rows * nq; it += WG_THREADS) {
        int m = div_small(it, nq), c = n0 + (it - m * nq) * 4;
        int tok = row_token(a, m);
        const uint16_t *src = tok >= 0 ? md.emb + (size_t)tok * d + c : a.pf_emb + (size_t)m * d + c;
        uint2 r = *reinterpret_cast<const uint2 *>(src);
        float v[4] = {__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xFFFF0000u), __uint_as_float(r.y << 16),
                      __uint_as_float(r.y & 0xFFFF0000u)};
        *reinterpret_cast<float4 *>(a.sc.h + (size_t)m * d + c) = make_float4(v[0], v[1], v[2], v[3]);
        sq[it] = v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
        float4 g = *reinterpret_cast<const float4 *>(gain + c);
        float x[4] = {v[0] * g.x, v[1] * g.y, v[2] * g.z, v[3] * g.w};
        store_split4(a.sc.xn, rows, m, c, x);
    }
    __syncthreads();
    if (tid < rows) {
        float t = 0.f;
        for (int j = 0; j < nq; ++j) t += sq[tid * nq + j];
        as_global_mut(a.sc.ss_a)[(size_t)tid * SS_LD + blockIdx.x] = t;
    }
}

// ------------------------------------------------------------------ attention

constexpr float ATT_NEG = -1.0e30f;  // finite stand-in for "no position seen yet"

__device__ __forceinline__ uint2 load_global8(const void *p)
{
    u32x2_t v = *as_global(reinterpret_cast<const u32x2_t *>(p));
    return make_uint2(v[0], v[1]);
}

typedef __attribute__((ext_vector_type(4))) short s16x4_t;

// eight values as an MFMA operand's two bf16 terms
__device__ __forceinline__ void split_bf16x8(f32x4_t x, f32x4_t y, bf16x8_t &hi, bf16x8_t &lo)
{
    uint32_t h[4], l[4];
    split_bf16(x[0], x[1], h[0], l[0]);
    split_bf16(x[2], x[3], h[1], l[1]);
    split_bf16(y[0], y[1], h[2], l[2]);
    split_bf16(y[2], y[3], h[3], l[3]);
    hi = __builtin_bit_cast(bf16x8_t, make_uint4(h[0], h[1], h[2], h[3]));
    lo = __builtin_bit_cast(bf16x8_t, make_uint4(l[0], l[1], l[2], l[3]));
}

// floats of one row's partial result in LDS (output, maximum, sum, padding to 16 bytes) ...
constexpr int att_rec(int hd) { return hd + 4; }
// ... and of one item's in memory: [ATT_ROWS][hd] outputs, [ATT_ROWS][2] maxima and sums (16-byte accesses without padding)
constexpr int att_item(int hd) { return ATT_ROWS * (hd + 2); }
constexpr size_t att_lds(int hd, int rows) { return (size_t)WAVES * (rows < ATT_ROWS ? rows : ATT_ROWS) * att_rec(hd) * sizeof(float) + 16; }

// Workgroup = (split of the cache's pages, head, session or chunk of up to ATT_ROWS = 16 query
// rows); the host picks the number of splits from the pages, the head size and the items (attention_splits: one where
// there are few pages, otherwise enough for the workgroups to cover the chip).  Where sessions have splits of their own the grid is (head, split of
// session after session): heads vary fastest, so that the XCDs, which workgroups are dealt to in turn, get equal shares of long and short
// sessions.  Elsewhere splits do: a head's splits, which pull on one stretch of the cache, are then on XCDs of their own (one session, 5 rows, heads
// fastest / splits fastest: 32 heads of 128 at 512 positions 10.9 / 10.6 us, at 4096 31.1 / 30.0, of 64 at 4096 19.1 / 17.4).  Wave w takes the pages
// pg_lo + w, pg_lo + w + WAVES, ... of the split (16 positions each), both products on the matrix cores:
//   scores  S[pos][row] = K . q^T     v_mfma_f32_16x16x32_bf16, A = 16 cached positions x 32
//           values straight from the page (lane l: position l & 15, values (l >> 4) * 8 ..),
//           B = the rows' q; three MFMAs per 32 values (k_hi q_hi + k_lo q_hi + k_hi q_lo);
//   output  O[dim][row] = V^T . P     v_mfma_f32_16x16x16bf16_1k, B = p in the layout the score
//           MFMA left it in (lane l: row l & 15, positions (l >> 4) * 4 ..), A = V, which the
//           cache stores transposed inside a page ([term][dim][position]) so that a lane's
//           four positions are 8 contiguous bytes; p and V as two bf16 terms, three MFMAs.
// A row's maximum, sum and output live in the lanes of its column, so the running rescale from page to
// page needs no exchange.  q and the cached k use the same pair-interleaved order inside a head, so
// their dot product is unchanged.  The waves' un-normalised results are merged through LDS in wave
// order.  With one split the normalised output is written directly; otherwise every workgroup
// writes its partial and counts itself in the unit's counter, and the one that arrives
// last merges the unit's partials in split order (the result does not depend on arrival order)
// and clears the counter for the next launch.  Nothing waits.
// With few rows the launch is a chain of latencies (arguments, K and V, merge, count, final merge), and
// its instructions are executed once, from a cold instruction cache: the code is kept short, one loop over
// pages (K of the next page requested as soon as this one's scores are done).  us per launch against a
// version that unrolled eight pages per wave and looped over work items: 5 rows at 512 positions 11.8 ->
// 9.0, the smallest model 7.3 -> 5.4; eight sessions of 640 positions (175 MB of cache) 34.2 -> 33.6.
template <int HD>
__device__ __forceinline__ void att_stage(const PassArgs &a, char *lds)
{
    constexpr int KT = HD / 32;  // 32-value steps of a score
    constexpr int NT = HD / 16;  // 16-dim tiles of the output
    constexpr int REC = att_rec(HD);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15, quad = lane >> 4;
    const int M = a.M;
    int sp = blockIdx.x, hh = blockIdx.y, s = a.mode == 1 ? 0 : blockIdx.z, n_splits = a.att_splits;
    const int ch = a.mode == 1 ? blockIdx.z : 0;
    if (a.att_starts) {
        sp = blockIdx.y;
        hh = blockIdx.x;
        const unsigned long long upto = a.att_starts & ((2ull << sp) - 1);
        const int first = 63 - __builtin_clzll(upto);
        s = __builtin_popcountll(upto) - 1;
        n_splits = sp - first + 1 + __builtin_ctzll(a.att_starts >> (sp + 1));
        sp -= first;
    }
    const int r0 = ch * ATT_ROWS, nr = min(ATT_ROWS, M - r0);
    const int P = a.mode == 1 ? a.pf_pos0 : EE_SESS(a, s, kv_len);  // position of the first row
    const int n_pg = (P + r0 + nr + KV_PAGE - 1) / KV_PAGE;         // pages visible to the chunk's last row
    const int pg_lo = div_small(n_pg * sp, n_splits), pg_hi = div_small(n_pg * (sp + 1), n_splits);
    const int cbase = EE_SESS(a, s, contig_base), n_pages = EE_SESS(a, s, n_pages);
    const int *page_table = EE_SESS(a, s, page_table);
    const uint16_t *kpool = EE_SESS(a, s, kpool), *vpool = EE_SESS(a, s, vpool);
    const int mrow = min(lm, nr - 1);                               // rows past the chunk repeat its last row
    const int last_pos = P + r0 + mrow;                             // last position this lane's row may see
    f32x4_t O[NT];
    float mx = ATT_NEG, sum = 0.f;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) O[nt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    int pg = pg_lo + wave;
    if (pg < pg_hi) {
        uint4 kh[KT], kl[KT];
        uint2 vh[NT], vl[NT];
        auto record = [&](int page_idx) __attribute__((always_inline)) {   // first element of the (page, head) record
            const int page = cbase >= 0 ? cbase + page_idx : __builtin_amdgcn_readfirstlane(as_global(page_table)[page_idx]);
            return (((size_t)a.layer * n_pages + page) * a.H + hh) * (size_t)(KV_PAGE * 2 * HD);
        };
        auto request_k = [&](size_t rec) __attribute__((always_inline)) {
            const uint16_t *kb = reinterpret_cast<const uint16_t *>(uniform_ptr(kpool + rec));
            const unsigned off = lm * (2 * HD) + quad * 8;
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                kh[kt] = load_global16(kb + off + kt * 32);
                kl[kt] = load_global16(kb + off + HD + kt * 32);
            }
        };
        auto request_v = [&](size_t rec) __attribute__((always_inline)) {
            const uint16_t *vb = reinterpret_cast<const uint16_t *>(uniform_ptr(vpool + rec));
            const unsigned off = lm * KV_PAGE + quad * 4;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                vh[nt] = load_global8(vb + off + nt * 16 * KV_PAGE);
                vl[nt] = load_global8(vb + off + (HD + nt * 16) * KV_PAGE);
            }
        };
        // the rows' q, K and V of the first page travel together
        f32x4_t qraw[KT][2];
        {
            const float *qp = a.sc.q + (size_t)(s * M + r0 + mrow) * a.d + hh * HD + quad * 8;
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                qraw[kt][0] = *as_global(reinterpret_cast<const f32x4_t *>(qp + kt * 32));
                qraw[kt][1] = *as_global(reinterpret_cast<const f32x4_t *>(qp + kt * 32 + 4));
            }
        }
        size_t rec = record(pg);
        request_k(rec);
        request_v(rec);
        bf16x8_t qh[KT], ql[KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) split_bf16x8(qraw[kt][0], qraw[kt][1], qh[kt], ql[kt]);
        for (;;) {
            f32x4_t S = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                const bf16x8_t Ah = __builtin_bit_cast(bf16x8_t, kh[kt]), Al = __builtin_bit_cast(bf16x8_t, kl[kt]);
                S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ah, qh[kt], S, 0, 0, 0);
                S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Al, qh[kt], S, 0, 0, 0);
                S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ah, ql[kt], S, 0, 0, 0);
            }
            const int pos0 = pg * KV_PAGE + quad * 4;
            pg += WAVES;
            const bool more = pg < pg_hi;
            if (more) {
                rec = record(pg);
                request_k(rec);
            }
            float m_new = mx;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                S[r] = pos0 + r <= last_pos ? S[r] * a.att_scale : ATT_NEG;
                m_new = fmaxf(m_new, S[r]);
            }
            m_new = fmaxf(m_new, __shfl_xor(m_new, 16, 64));
            m_new = fmaxf(m_new, __shfl_xor(m_new, 32, 64));
            const float f = __expf(mx - m_new);
            mx = m_new;
            sum *= f;
            uint32_t ph[2], pl[2];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                S[r] = S[r] > 0.5f * ATT_NEG ? __expf(S[r] - mx) : 0.f;
                sum += S[r];
            }
            split_bf16(S[0], S[1], ph[0], pl[0]);
            split_bf16(S[2], S[3], ph[1], pl[1]);
            const s16x4_t Ph = __builtin_bit_cast(s16x4_t, make_uint2(ph[0], ph[1])), Pl = __builtin_bit_cast(s16x4_t, make_uint2(pl[0], pl[1]));
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                for (int r = 0; r < 4; ++r) O[nt][r] *= f;
                const s16x4_t Vh = __builtin_bit_cast(s16x4_t, vh[nt]), Vl = __builtin_bit_cast(s16x4_t, vl[nt]);
                O[nt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(Vh, Ph, O[nt], 0, 0, 0);
                O[nt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(Vh, Pl, O[nt], 0, 0, 0);
                O[nt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(Vl, Ph, O[nt], 0, 0, 0);
            }
            if (!more) break;
            request_v(rec);
        }
        sum += __shfl_xor(sum, 16, 64);
        sum += __shfl_xor(sum, 32, 64);
    }
    // this wave's record: lane holds O[dims nt*16 + quad*4 ..][row lm]
    float *wbuf = reinterpret_cast<float *>(lds);                   // [WAVES][nr][REC]
    int *lastf = reinterpret_cast<int *>(wbuf + (size_t)WAVES * nr * REC);
    if (lm < nr) {
        float *w = wbuf + (wave * nr + lm) * REC;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) *reinterpret_cast<float4 *>(w + nt * 16 + quad * 4) = make_float4(O[nt][0], O[nt][1], O[nt][2], O[nt][3]);
        if (quad == 0) {
            w[HD] = mx;
            w[HD + 1] = sum;
        }
    }
    lds_barrier();
    // merge the waves, fixed order; thread = (row, four dims)
    const int i = tid / (HD / 4), e = (tid - i * (HD / 4)) * 4;
    const bool mine = i < nr;                                       // WG_THREADS >= ATT_ROWS * HD / 4
    float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
    float den = 0.f, gm = ATT_NEG;
    static_assert(WG_THREADS >= ATT_ROWS * HD / 4, "one thread per row and four dims");
    if (mine) {
        const int act = min(WAVES, pg_hi - pg_lo);                  // waves that had a page
        const float *w0 = wbuf + i * REC;
        for (int w = 0; w < act; ++w) gm = fmaxf(gm, w0[w * nr * REC + HD]);
        for (int w = 0; w < act; ++w) {
            const float *wr = w0 + w * nr * REC;
            const float f = __expf(wr[HD] - gm);
            const float4 o = load_f4(wr + e);
            num.x += o.x * f; num.y += o.y * f; num.z += o.z * f; num.w += o.w * f;
            den += wr[HD + 1] * f;
        }
    }
    if (n_splits > 1) {
        const int unit = (ch + s) * a.H + hh;                       // (one of them is 0)
        const WRes part = buffer_resource(a.sc.att_part + (size_t)unit * a.att_splits * att_item(HD));
        constexpr int SP_BYTES = att_item(HD) * 4, MS = ATT_ROWS * HD * 4;
        if (mine) {
            store_dev128(part, sp * SP_BYTES + (i * HD + e) * 4, num);
            if (e == 0) store_dev64(part, sp * SP_BYTES + MS + i * 8, make_float2(gm, den));
        }
        wait_vmem();      // this workgroup's partials are visible device-wide ...
        __syncthreads();  // ... for every wave, before it is counted
        if (tid == 0) {
            const int before = __hip_atomic_fetch_add(a.sc.att_count + unit, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *lastf = before == n_splits - 1 ? 1 : 0;
            if (*lastf) __hip_atomic_store(a.sc.att_count + unit, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (!*lastf) return;
        if (mine) {
            // eight splits' loads in flight together; a second round only for more than eight
            num = make_float4(0.f, 0.f, 0.f, 0.f);
            den = 0.f;
            gm = ATT_NEG;
            for (int k0 = 0; k0 < n_splits; k0 += 8) {
                float4 pv[8];
                float2 pm[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int off = min(k0 + k, n_splits - 1) * SP_BYTES;
                    pv[k] = load_dev128(part, off + (i * HD + e) * 4);
                    pm[k] = load_dev64(part, off + MS + i * 8);
                }
                float m_new = gm;
#pragma unroll
                for (int k = 0; k < 8; ++k) m_new = fmaxf(m_new, pm[k].x);
                const float f0 = __expf(gm - m_new);
                gm = m_new;
                num.x *= f0; num.y *= f0; num.z *= f0; num.w *= f0;
                den *= f0;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const float f = k0 + k < n_splits ? __expf(pm[k].x - gm) : 0.f;
                    num.x += pv[k].x * f; num.y += pv[k].y * f; num.z += pv[k].z * f; num.w += pv[k].w * f;
                    den += pm[k].y * f;
                }
            }
        }
    }
    if (mine) {
        const float inv = 1.0f / den;
        const float v[4] = {num.x * inv, num.y * inv, num.z * inv, num.w * inv};
        store_split4(a.sc.attn, a.rows, s * M + r0 + i, hh * HD + e, v);
    }
}

// ------------------------------------------------------------------ accept

__device__ __forceinline__ int2 load_cand(const int2 *p)
{
    const unsigned long long v = __hip_atomic_load(as_global(reinterpret_cast<const unsigned long long *>(p)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_int2((int)(unsigned)v, (int)(unsigned)(v >> 32));
}

// One workgroup: global argmax per row, confidence, accept rule per session, publication.
// Reads the candidates with device scope: they may have been written earlier in this launch.
__device__ __forceinline__ void accept_stage(const PassArgs &a, char *lds)
{
    const int rows = a.rows, M = a.M;  // rows of the head launch: head after head, session after session, M rows each
    int *tok = reinterpret_cast<int *>(lds);
    float *conf = reinterpret_cast<float *>(lds) + EE_MAX_ROWS;
    const int l = threadIdx.x & 15, m = threadIdx.x >> 4;   // sixteen lanes per row, all rows at once
    if (m < rows) {
        // all of the row's candidates and partial sums are requested before the first is used
        constexpr int PER = SS_LD / 16;                     // workgroups per lane
        int2 c[PER];
        float sg[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int g = min(l + 16 * j, a.nwg - 1);       // (slots past the workgroups: the last candidate again, counted once)
            c[j] = load_cand(a.sc.cand + (size_t)m * SS_LD + g);
            sg[j] = load_dev32(a.sc.cand_sum + (size_t)m * SS_LD + g);
        }
        float bv = -INFINITY;
        int bi = 0x7FFFFFFF;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const float v = __int_as_float(c[j].x);
            if (cand_better(v, c[j].y, bv, bi)) {
                bv = v;
                bi = c[j].y;
            }
        }
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) {
            float ov = __shfl_xor(bv, off, 64);
            int oi = __shfl_xor(bi, off, 64);
            if (cand_better(ov, oi, bv, bi)) {
                bv = ov;
                bi = oi;
            }
        }
        // confidence (paper Eq. 4): max softmax = 1 / sum_j exp(z_j - z_max), from the
        // workgroups' sums, each rescaled from its own maximum to the global one
        float se = 0.f;
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (l + 16 * j < a.nwg && sg[j] > 0.f) se += sg[j] * __expf(__int_as_float(c[j].x) - bv);
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) se += __shfl_xor(se, off, 64);
        if (l == 0) {
            tok[m] = bi;
            conf[m] = 1.0f / se;
        }
    }
    __syncthreads();
    // one thread per (head of this launch, session)
    if ((int)threadIdx.x < a.n_heads * a.n_sess) {
        const int hj = div_small(threadIdx.x, a.n_sess), s = threadIdx.x - hj * a.n_sess, head = a.head_idx + hj;
        ee_verify_result *res = EE_SESS(a, s, result);
        const int *t = tok + (hj * a.n_sess + s) * M;
        const float *cf = conf + (hj * a.n_sess + s) * M;
        if (a.head_kind == HEAD_PREFILL) {
            int last = t[M - 1];
            res->next_token = last;
            res->device_status = 0;
        } else {
            const int gamma = M - 1;
            int delta = 0;
            if (a.sm.on) {
                // probabilistic verification: the rows' decisions were taken by the sampling launch;
                // the tokens published are the ones each row emits if the round ends there
                int *ts = tok + (hj * a.n_sess + s) * M;
                unsigned kept = 0;
                for (int i = 0; i < M; ++i) {
                    const int r = (hj * a.n_sess + s) * M + i;   // the row of the head launch
                    ts[i] = __hip_atomic_load(a.sm.tok + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (i < gamma && __hip_atomic_load(a.sm.kept + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) kept |= 1u << i;
                }
                delta = __builtin_ctz(~kept);   // drafts kept before the first one that is not (bit gamma is never set)
            } else {
                int dr[EE_MAX_M];
#pragma unroll
                for (int i = 0; i < EE_MAX_M - 1; ++i) dr[i] = i < gamma ? draft_of(a, s, i) : -1;
#pragma unroll
                for (int i = 0; i < EE_MAX_M - 1; ++i)
                    if (delta == i && i < gamma && dr[i] == t[i]) delta = i + 1;
            }
            if (a.head_kind == HEAD_EXIT) {
                for (int i = 0; i < M; ++i) {
                    res->exit_tokens[head][i] = t[i];
                    res->exit_conf[head][i] = cf[i];
                }
                res->exit_accept_len[head] = delta;
            } else {
                for (int i = 0; i < M; ++i) {
                    res->final_tokens[i] = t[i];
                    res->final_conf[i] = cf[i];
                }
                res->accept_len = delta;
                res->next_token = t[delta];
                res->device_status = 0;
            }
        }
        __threadfence_system();
    }
}

// ------------------------------------------------------------------ probabilistic verification

// Weights of the cumulative sums are 40-bit fixed point (integers): their sums do not depend on
// the order of addition, so every thread's share [exclusive sum, + own sum) of the cumulative
// distribution tiles it exactly and the search below always ends inside the owner's tokens.
// A weight is at most 1 (largest exp term, or a probability), so a row of fewer than 2^24 tokens cannot overflow 64 bits.
static_assert(DIV_SMALL_MAX < 1 << 24, "the loader refuses vocabularies above DIV_SMALL_MAX");
typedef unsigned long long u64;
constexpr int SAMPLE_LDS_BYTES = 4096;             // the waves' sums and flags; the accept step's rows
constexpr float SAMPLE_UNIT = 1099511627776.0f;  // 2^40

__device__ __forceinline__ u64 fixed_weight(float w) { return (u64)(w * SAMPLE_UNIT); }

// e_k = exp((z_k - zmax) / T): un-normalised probability of token k under the target distribution
__device__ __forceinline__ float target_term(float z, float zmax, float inv_T) { return expf((z - zmax) * inv_T); }

// positive part of q_k - p_k (one fused multiply-add, so that every place that forms it gets the same bits)
__device__ __forceinline__ float residual_term(float e, float inv_Z, float p) { return fmaxf(__fmaf_rn(e, inv_Z, -p), 0.f); }

// sum of one 64-bit value per lane over the wave (every lane gets it)
__device__ __forceinline__ u64 wave_sum(u64 x)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
}

constexpr int SAMPLE_WAVES = 16;
constexpr int SAMPLE_BLOCKS = 2;                                     // blocks of 64 tokens a wave holds
constexpr int SAMPLE_PART = SAMPLE_WAVES * SAMPLE_BLOCKS * 64;       // tokens of a workgroup
__host__ __device__ constexpr int sample_parts(int V) { return (V + SAMPLE_PART - 1) / SAMPLE_PART; }

// One row of one head under probabilistic verification (Eq. 2 / Eq. 5 of the paper with the
// draft model's distributions; the keep / replace rule of the speculative sampling scheme the
// paper builds on).  q = softmax(z / T) of the row's logits.  Row i < gamma: its draft x is kept
// iff u_i * p_i(x) < q(x), and if the round ends here the row emits a token drawn from the
// positive part of q - p_i; row gamma emits a token drawn from q.  Drawing = inversion of the
// cumulative sum in token order with the row's number v_i: the first token whose cumulative
// weight exceeds v_i * (sum of the weights).
//
// Workgroup = (part of SAMPLE_PART tokens, row), two launches.  The first sums its part's exponentials (the row's largest logit
// comes from the head launch's candidates); the second, with Z from all parts, sums the residual weights, and the workgroup
// that arrives last at the row's counter has all parts' sums: it finds the part the target lies in, then the wave, the block and the
// token.  The sums are integers: the cumulative sum up to a token is the earlier parts' totals + the earlier waves' + a
// scan inside the wave, whatever the order they were added in.
// Bound by latencies (loads, sums, one arrival each for row and launch).  32000 tokens, 5 rows: 4.8 + 15.4 us in two launches; one workgroup per
// row, which was bound by one unit's vector instructions (about 45 per token), 28 us.
struct SampleRow {
    int ses, i, rr, hj;                                          // session, row of it; row of the head, head of the launch
    const EE_GLOBAL float *z, *p, *uv;                           // logits, the draft's distribution, the session's u, v and 1 / temperature
};
__device__ __forceinline__ SampleRow sample_row(const PassArgs &a, int r)
{
    const int V = a.mdv.V, M = a.M, gamma = M - 1, per_head = a.n_sess * M;   // the launch's rows: head after head, session after session
    SampleRow w;
    w.hj = div_small(r, per_head);
    w.rr = r - w.hj * per_head;
    w.ses = div_small(w.rr, M);
    w.i = w.rr - w.ses * M;
    w.z = as_global(a.sc.logits) + ((size_t)(a.head_idx + w.hj) * a.mdv.rows_max + w.rr) * V;
    w.p = as_global(a.sm.probs) + ((size_t)w.ses * gamma + min(w.i, gamma - 1)) * V;
    w.uv = as_global(a.sm.uv) + (size_t)w.ses * (2 * gamma + 2);
    return w;
}
// largest logit of the row: the best of the head launch's candidates
__device__ __forceinline__ float sample_max(const PassArgs &a, int r, int lane)
{
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < SS_LD / 64; ++j) {
        const int g = lane + 64 * j;
        if (g < a.plan0.nwg) mx = fmaxf(mx, __int_as_float(as_global(a.sc.cand)[(size_t)r * SS_LD + g].x));
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    return mx;
}
// this lane's tokens of the wave's share: first + 64 j + lane; exponentials of the logits, past the row's end 0
__device__ __forceinline__ void sample_terms(const SampleRow &w, int first, int V, int lane, float zmax, float inv_T, float (&e)[SAMPLE_BLOCKS])
{
#pragma unroll
    for (int j = 0; j < SAMPLE_BLOCKS; ++j) {
        const int k = first + 64 * j + lane;
        e[j] = -INFINITY;
        if (k < V) e[j] = w.z[k];
    }
#pragma unroll
    for (int j = 0; j < SAMPLE_BLOCKS; ++j) e[j] = target_term(e[j], zmax, inv_T);
}
__device__ __forceinline__ void sample_drafted(const SampleRow &w, int first, int V, int lane, float (&p)[SAMPLE_BLOCKS])
{
#pragma unroll
    for (int j = 0; j < SAMPLE_BLOCKS; ++j) {
        const int k = first + 64 * j + lane;
        p[j] = 0.f;
        if (k < V) p[j] = w.p[k];
    }
}
// sum of one value per wave over the workgroup; every thread gets it, wtot[] keeps the waves' values
__device__ __forceinline__ u64 sample_block_sum(u64 x, u64 *wtot, int wave, int lane)
{
    x = wave_sum(x);
    if (lane == 0) wtot[wave] = x;
    __syncthreads();
    u64 t = 0;
#pragma unroll
    for (int w = 0; w < SAMPLE_WAVES; ++w) t += wtot[w];
    return t;
}

__device__ __forceinline__ void sample_sum_stage(const PassArgs &a, char *lds)
{
    const int part = blockIdx.x, r = blockIdx.y, V = a.mdv.V, parts = gridDim.x;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const SampleRow w = sample_row(a, r);
    float e[SAMPLE_BLOCKS];
    const float inv_T = w.uv[2 * (a.M - 1) + 1], zmax = sample_max(a, r, lane);
    sample_terms(w, part * SAMPLE_PART + wave * (SAMPLE_BLOCKS * 64), V, lane, zmax, inv_T, e);
    u64 sum = 0;
#pragma unroll
    for (int j = 0; j < SAMPLE_BLOCKS; ++j) sum += fixed_weight(e[j]);
    sum = sample_block_sum(sum, reinterpret_cast<u64 *>(lds), wave, lane);
    if (threadIdx.x == 0) as_global_mut(a.sm.sums)[(size_t)r * parts + part] = sum;
}

// sum of a row's parts in [0, n); every lane gets it
__device__ __forceinline__ u64 sample_load_sum(const u64 *s, int n, int lane)
{
    u64 t = 0;
    for (int i = lane; i < n; i += 64) t += __hip_atomic_load(as_global(s + i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return wave_sum(t);
}

// true in the workgroup that leaves the row's decision behind (thread 0 stores it)
__device__ __forceinline__ bool sample_draw_stage(const PassArgs &a, char *lds)
{
    static_assert(SAMPLE_WAVES * 8 + 32 <= SAMPLE_LDS_BYTES && EE_MAX_ROWS * 8 <= SAMPLE_LDS_BYTES, "LDS of the sampling launch");
    const int r = blockIdx.y, V = a.mdv.V, parts = gridDim.x, gamma = a.M - 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    u64 *wtot = reinterpret_cast<u64 *>(lds);                    // [SAMPLE_WAVES]
    int *flag = reinterpret_cast<int *>(wtot + SAMPLE_WAVES);    // arrived last; the token
    const SampleRow w = sample_row(a, r);
    const bool drafted = w.i < gamma;
    const u64 *sums_e = a.sm.sums + (size_t)r * parts;
    u64 *sums_r = a.sm.sums + ((size_t)a.head_rows + r) * parts;
    const float inv_T = w.uv[2 * gamma + 1], v_row = w.uv[gamma + w.i], zmax = sample_max(a, r, lane);
    float e[SAMPLE_BLOCKS], pc[SAMPLE_BLOCKS];
    int part = blockIdx.x;
    const int mine = wave * (SAMPLE_BLOCKS * 64);
    if (drafted) {
        sample_drafted(w, part * SAMPLE_PART + mine, V, lane, pc);
        sample_terms(w, part * SAMPLE_PART + mine, V, lane, zmax, inv_T, e);
    }
    const u64 Zi = sample_load_sum(sums_e, parts, lane);
    const float inv_Z = 1.0f / (float)((double)Zi * (1.0 / (double)SAMPLE_UNIT));
    if (drafted) {
        u64 sum = 0;
#pragma unroll
        for (int j = 0; j < SAMPLE_BLOCKS; ++j) sum += fixed_weight(residual_term(e[j], inv_Z, pc[j]));
        sum = sample_block_sum(sum, wtot, wave, lane);
        if (tid == 0) {
            __hip_atomic_store(sums_r + part, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            wait_vmem();                                         // visible before it is counted
            int *cnt = a.sm.count + 1 + r;
            const int before = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *flag = before == parts - 1 ? 1 : 0;
            if (*flag) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (!*flag) return false;
    } else if (part != 0) {
        return false;                                            // (a row that draws from q has all it needs from the first launch)
    }
    // all parts' sums are there
    const u64 *tot = sums_e;
    u64 w_total = Zi;
    bool residual = false;
    int kept = 0;
    if (drafted) {
        const int x = draft_of(a, w.ses, w.i);
        const float qx = target_term(w.z[x], zmax, inv_T) * inv_Z;
        kept = w.uv[w.i] * w.p[x] < qx ? 1 : 0;
        const u64 W = sample_load_sum(sums_r, parts, lane);
        if (W > 0) {  // otherwise q = p: the draft is always kept and the row never emits; it then draws from q
            residual = true;
            tot = sums_r;
            w_total = W;
        }
    }
    // the first token whose cumulative weight exceeds the target; v < 1, so target < w_total
    const double vd = (double)v_row;
    u64 target = (u64)(vd * (double)w_total);
    if (target >= w_total) target = w_total - 1;
    // the target's part: 64 parts at a time
    u64 run = 0;
    for (int p0 = 0; p0 < parts; p0 += 64) {
        const u64 own = p0 + lane < parts ? __hip_atomic_load(as_global(tot + p0 + lane), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
        u64 incl = own;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const u64 o = __shfl_up(incl, off, 64);
            if (lane >= off) incl += o;
        }
        const unsigned long long hit = __ballot(run + incl > target);
        if (hit) {
            const int h = __builtin_ctzll(hit);
            part = p0 + h;
            run += __shfl(incl, h, 64) - __shfl(own, h, 64);
            break;
        }
        run += __shfl(incl, 63, 64);
    }
    // its tokens
    const int first = part * SAMPLE_PART + mine;
    sample_terms(w, first, V, lane, zmax, inv_T, e);
    if (residual) sample_drafted(w, first, V, lane, pc);
    u64 wk[SAMPLE_BLOCKS], own = 0;
#pragma unroll
    for (int j = 0; j < SAMPLE_BLOCKS; ++j) {
        wk[j] = fixed_weight(residual ? residual_term(e[j], inv_Z, pc[j]) : e[j]);
        own += wk[j];
    }
    if (tid == 0) flag[1] = 0;                                   // the token where no weight is positive (NaN or infinite logits, 1 / temperature infinite)
    __syncthreads();                                             // (wtot is read above)
    sample_block_sum(own, wtot, wave, lane);
    for (int k = 0; k < wave; ++k) run += wtot[k];
    if (run <= target && target < run + wtot[wave]) {            // at most one wave
        bool done = false;
#pragma unroll
        for (int j = 0; j < SAMPLE_BLOCKS; ++j) {
            u64 incl = wk[j];
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const u64 o = __shfl_up(incl, off, 64);
                if (lane >= off) incl += o;
            }
            const unsigned long long hit = __ballot(run + incl > target);
            if (!done && hit) {
                if (lane == 0) flag[1] = first + 64 * j + __builtin_ctzll(hit);
                done = true;
            }
            run += __shfl(incl, 63, 64);
        }
    }
    __syncthreads();
    if (tid == 0) {
        __hip_atomic_store(a.sm.tok + r, flag[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(a.sm.kept + r, kept, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return true;
}

// ------------------------------------------------------------------ kernels of the pass
//
// Stage list of a segment: [EMBED] { QKV ATT O GU DN } x layers [AD AU] [HEAD]; one launch per stage.
// The accept step runs inside the head's launch, in the workgroup that finishes last.

// Where the input's sums of squares are and what the epilogue produces, by GEMM kind (what varies inside a kind travels in the arguments).
template <int KIND>
__device__ __forceinline__ GemmIn gemm_input(const PassArgs &a)
{
    const char *x = reinterpret_cast<const char *>(a.entry.X);
    if (KIND == G_AD || KIND == G_AU) x += a.entry.x_next * (int)blockIdx.y;
    return GemmIn{x, KIND == G_QKV ? a.sc.ss_a : (KIND == G_GU ? a.sc.ss_f : (KIND == G_HEAD ? a.sc.ss_h : nullptr))};
}

template <int KIND>
__device__ __forceinline__ GemmEpi gemm_epi(const PassArgs &a)
{
    GemmEpi ep = {nullptr, nullptr, nullptr, nullptr, nullptr, 0};
    if (KIND == G_O) {
        ep.gain_xn = a.gain_xn;
        ep.ss_out = a.sc.ss_f;
    } else if (KIND == G_DN) {
        ep.gain_xn = a.gain_xn;                // null after the last layer
        ep.gain_xh = a.gain_xh;                // set where an exit (or the final head) takes this layer's output
        ep.ss_head = a.gain_xh ? a.sc.ss_h : nullptr;
        ep.xa_out = a.xa_out;                  // the exit's adapters come first
        ep.ss_out = a.sc.ss_a;
    } else if (KIND == G_AD) {
        ep.bias = a.bias + (int)blockIdx.y * a.bias_next;
    } else if (KIND == G_AU) {
        ep.bias = a.bias + (int)blockIdx.y * a.bias_next;
        ep.gain_xh = a.gain_xh + (int)blockIdx.y * a.gain_next;
        ep.ss_head = a.sc.ss_h;
    }
    return ep;
}

// One GEMM of the pass, for rows <= 8 XC (gemm_kernel_of gives its address: ee_gemm_*.hip).  The kind is a template parameter: every instruction of a launch is
// executed once, at the speed of instruction-cache misses, and neither its start nor its epilogue holds another kind's
// code.  Against one kernel for all kinds, us per launch, 5 rows of the 7B shape, before the first requests went ahead
// of everything else (gemm_entry): QKV 19.6 -> 18.5, O 10.2 -> 9.1, gate/up 31.2 -> 30.8, down 19.0 -> 18.2, head
// 51.2 -> 49.8; the smallest model's launches 4.9-6.7 -> 3.8-4.8.
template <int KIND, int XC, bool PK>
__global__ void __launch_bounds__(WG_THREADS) ee_gemm_kernel(PassArgs a_by_value)
{
    extern __shared__ __align__(16) char lds[];
    gemm_entry<KIND, XC, PK>(lds);
    const PassArgs &a = warmed_arguments();
    const char *W = reinterpret_cast<const char *>(a.entry.W);
    if (KIND == G_AD || KIND == G_AU) W += a.entry.w_next * blockIdx.y;
    gemm_stage_t<KIND, XC, PK>(a, a.plan0, a.lay, reinterpret_cast<const uint4 *>(W), gemm_input<KIND>(a), gemm_epi<KIND>(a), lds);
    if (KIND == G_HEAD && a.fuse_accept) {
        // The workgroup whose candidates arrive last also runs the accept step
        // (one launch less per head); the counter is left at zero.
        int *lastf = misc_views(a.lay, lds).lastf;
        wait_vmem();      // this workgroup's candidates are visible device-wide ...
        __syncthreads();  // ... for every wave, before it is counted
        if (threadIdx.x == 0) {
            const int before = __hip_atomic_fetch_add(a.sc.head_count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *lastf = before == a.nwg - 1 ? 1 : 0;
            if (*lastf) __hip_atomic_store(a.sc.head_count, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (*lastf) accept_stage(a, lds);
    }
}

template <int HD>
__global__ void __launch_bounds__(WG_THREADS) ee_att_kernel(PassArgs a_by_value)
{
    extern __shared__ __align__(16) char lds[];
    const PassArgs &a = warmed_arguments();
    att_stage<HD>(a, lds);
}

}  // namespace ee
