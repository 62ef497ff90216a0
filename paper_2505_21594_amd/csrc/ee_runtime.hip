// Host runtime and C ABI of libeeverify (declarations and semantics: include/ee.h).
#include <fcntl.h>
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>
#include <sys/stat.h>
#include <unistd.h>

#include <algorithm>
#include <climits>
#include <new>
#include <tuple>
#include <utility>
#include <vector>

#include "ee_once.hpp"

using namespace ee;

// ------------------------------------------------------------------ errors

static thread_local char g_err[512] = "";

static int fail(int code, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return code;
}

#define HIP_TRY(expr)                                                                          \
    do {                                                                                       \
        hipError_t e_ = (expr);                                                                \
        if (e_ != hipSuccess)                                                                  \
            return fail(EE_EDEVICE, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, __LINE__); \
    } while (0)

extern "C" const char *ee_last_error(void) { return g_err; }

// ------------------------------------------------------------------ objects

struct ee_model {
    ee_model_config cfg;
    int device;
    int nwg;
    size_t lds_budget;           // dynamic LDS bytes each launch asks for
    ModelDev host_md;            // the descriptor the launches carry by value
    // Weight-stream plans and tiled weights per GEMM kind (a launch gets its plan and weights by
    // value): [0] every workgroup streams whole rows of K, [1] K split over groups of workgroups
    // (launches of more than 16 rows; only the kinds where it pays have one, nwg = 0 otherwise).
    // One allocation per kind and variant, layer l (adapters: stored exit l) at w + l * wstride (uint4 units).
    GemmPlan plan[2][G_KINDS];
    const uint4 *w[2][G_KINDS];
    long long wstride[2][G_KINDS];
    // The same weights packed (PACK_TILE), what launches of up to 48 rows stream: per slice (pk_bytes each; one allocation
    // per kind and variant, layers apart in it cost 0.3 % of a pass), for the slices that have them; the others, and prefill, take w.
    struct PackedSlice {
        const unsigned char *w;      // nullptr: not packed
        size_t esc;                  // first escape in m->escapes
        int groups, cap;
        float scale;
    };
    unsigned char *pk[2][G_KINDS];
    size_t pk_bytes[2][G_KINDS];
    std::vector<PackedSlice> packed[2][G_KINDS];   // empty: the kind is not packed
    const Escape *escapes;           // all matrices' lists
    const int2 *tile_tab[G_KINDS];   // prefill GEMMs: where the tiles of an n-tile lie (PfArgs::tab; trunk kinds only)
    std::vector<void *> allocs;  // every device allocation of the model
    const float *g_exit[EE_MAX_EXITS];
    // exit-head adapters (per stored exit): biases of the hidden units and the summed output biases
    const float *ad_bdown[EE_MAX_EXITS];
    const float *ad_bup[EE_MAX_EXITS];
};

struct ee_session {
    const ee_model *m;
    unsigned flags;
    int max_ctx, max_gamma;
    hipStream_t stream;
    hipStream_t run_stream;          // stream the pass this session leads is enqueued on (its own, or the first
                                     // group leader's when a batch runs as several groups)
    hipEvent_t ev_start, ev_final, ev_exit[EE_MAX_EXITS];
    // KV cache
    int n_pages;
    uint16_t *kpool, *vpool;
    int *dev_page_table;
    int *host_page_table;            // pinned mirror
    std::vector<int> free_pages;     // LIFO free list of physical pages
    int pages_used;                  // logical pages mapped
    float2 *rope;
    // staging
    float *host_sample;              // pinned staging of a sampled pass: draft distributions, then u, then v (EE_SAMPLING)
    hipStream_t copy_stream;         // uploads of a sampled pass's distributions (EE_SAMPLING)
    hipEvent_t ev_copy;
    float *dev_sample;               // device copy of the same
    int *dev_sample_out;             // [3 * EE_MAX_ROWS + 1] rows' tokens, keep flags, arrival counters (launch, rows)
    unsigned long long *dev_sample_sums;   // SampleDev::sums
    int *dev_pf_tokens;
    int *host_pf_tokens;             // pinned
    uint16_t *dev_pf_emb;
    ee_verify_result *result;        // pinned, mapped
    ee_verify_result *dev_result;
    SessDev *dev_sessdev;            // [EE_MAX_BATCH] per-pass session descriptors
    SessDev *host_sessdev;           // pinned staging for them
    PfScratch pf;                    // buffers of a prefill chunk
    float *pf_ss[2];                 // sums of squares: after the FFN block / embedding, after the attention block
    float *pf_part;                  // partial tiles of prefill GEMMs whose K is shared by several workgroups
    size_t pf_part_cap;              // floats of them
    int *pf_part_count;              // [PF_PART_TILES] parts delivered
    int pf_cap;                      // rows of the largest prefill chunk
    Scratch sc;
    int att_items_cap;               // attention work items the partials buffer has room for
    int att_splits_opt;              // EE_OPT_ATT_SPLITS (0: chosen per pass)
    int head_batch;                  // EE_OPT_HEAD_BATCH: exit heads per launch of the LM head
    bool scatter_pages;              // EE_OPT_SCATTER_PAGES
    int pf_gemm_opt, pf_att_opt;     // EE_OPT_PREFILL_GEMM, EE_OPT_PREFILL_ATT_ROWS (0: chosen per launch)
    int flight_row0;                 // first row of this session in the pass in flight
    unsigned long long popped_mask;  // exits of the pass in flight that ee_exit_pop has handed out
    std::vector<hipEvent_t> lt_events;   // EE_TIME_LAUNCHES: event pairs around every launch of the pass
    std::vector<int> lt_codes;           // what each timed launch ran (EE_LAUNCH_* code)
    std::vector<void *> allocs;
    // the session's state
    int kv_len;
    int pending;
    bool has_pending;
    bool in_flight;                  // a verify pass was enqueued and not yet waited for
    int flight_gamma, flight_exits;
    ee_session *leader;              // session whose stream/events carry the pass in flight
};

// ------------------------------------------------------------------ planning

static pass_kernel_t gemm_kernel(int kind, int rows, bool packed)
{
    switch (kind) {
    case G_QKV: return gemm_kernel_of<G_QKV>(rows, packed);
    case G_O: return gemm_kernel_of<G_O>(rows, packed);
    case G_GU: return gemm_kernel_of<G_GU>(rows, packed);
    case G_DN: return gemm_kernel_of<G_DN>(rows, packed);
    case G_AD: return gemm_kernel_of<G_AD>(rows, packed);
    case G_AU: return gemm_kernel_of<G_AU>(rows, packed);
    default: return gemm_kernel_of<G_HEAD>(rows, packed);
    }
}

static pass_kernel_t att_kernel(int hd) { return hd == 128 ? ee_att_kernel<128> : ee_att_kernel<64>; }

constexpr size_t PF_PART_FLOATS = (size_t)12 << 20;   // partial tiles of one launch: at most 48 MB
constexpr int PF_PART_TILES = 4096;

struct PfShape {
    int wn, wm;                  // a wave's accumulators: n-tiles x row tiles (workgroup: twice that each way)
    int grp;                     // groups of four waves that share the workgroup's K
    double t1, t2;               // us per k-tile: a workgroup alone on its compute unit; per workgroup where a unit has `occ`
    int occ;
    pf_kernel_t gemm[G_DN + 1];
};
#define EE_PF_SHAPE(WN, WM, GRP, T1, T2, OCC)                                                    \
    {WN, WM, GRP, T1, T2, OCC, {pf_gemm_of<G_QKV, WN, WM, GRP>(), pf_gemm_of<G_O, WN, WM, GRP>(), \
                                pf_gemm_of<G_GU, WN, WM, GRP>(), pf_gemm_of<G_DN, WN, WM, GRP>()}}
static const PfShape PF_SHAPES[] = {
    EE_PF_SHAPE(8, 4, 1, 0.908, 0.716, 2), EE_PF_SHAPE(4, 4, 1, 0.529, 0.407, 2), EE_PF_SHAPE(4, 2, 1, 0.356, 0.247, 2),
    EE_PF_SHAPE(2, 2, 1, 0.226, 0.186, 3), EE_PF_SHAPE(4, 4, 2, 0.480, 0.462, 1), EE_PF_SHAPE(4, 2, 2, 0.285, 0.300, 1),
    EE_PF_SHAPE(2, 2, 4, 0.190, 0.222, 1)};

static pf_kernel_t pf_att(int hd, int rt)
{
    return hd == 128 ? (rt == 2 ? pf_att_kernel<128, 2> : pf_att_kernel<128, 1>) : (rt == 2 ? pf_att_kernel<64, 2> : pf_att_kernel<64, 1>);
}

// Shape of the workgroup tile and parts of K of one prefill GEMM: the least estimated time.  The estimate, in us:
// per k-tile (PfShape) t1 where a workgroup is alone on its compute unit (a chain of latencies), t2 per workgroup
// where a unit has several (occ fit), and in a last round that gives only some units more than one at least 1.4 t1 (where two share
// a unit, each is slower than alone); a split adds the exchange of the partial tiles (4, 1 per part read one after the other, and the
// bytes at 3.5 TB/s).  What is the same for all choices, such as the launch itself, is left out.  Least-squares fit to every shape
// with 1 to 8 parts, QKV, O, GU and DN of the 7B shape at 64 to 2041 rows, of the 13B shape at 128 to 1400 and of a 1280-wide model at
// 61 to 700; then the four-group shape's t1 and the exchange set by the splits of few rows that this fit gave away (7B shape, 17 to
// 64 rows: down 29.4 -> 28.7, with t1 0.199 and 4.8 + 0.6 per part; 65 to 128: output 22.1 -> 21.2; 2048-wide, 193 to 256 rows: down
// 23.0 -> 20.6, 1281 to 1344: 84 -> 70).  Over 292 GEMMs (six models 256 to 5120 wide, 4 to 25 row counts from 17 to 2041)
// its choice is on average 2.0 % above the best measured one, at worst 25 % (gate/up of 2041 rows of the smallest model, 2 us); before the
// fit it was 3.1 %, 34 % (7B shape, 640 rows: output 64 -> 58; 256: down 68 -> 59; 900: down 181 -> 149).
struct PfChoice {
    const PfShape *shape;
    int nb, mb, ks;
};
static PfChoice pf_choose(const ee_model *m, const GemmPlan &pl, int rows, int forced)
{
    PfChoice best = {};
    if (forced) {   // EE_OPT_PREFILL_GEMM
        const PfShape &s = PF_SHAPES[forced % 16 - 1];
        best = {&s, (pl.NT + 2 * s.wn - 1) / (2 * s.wn), (rows + 32 * s.wm - 1) / (32 * s.wm), std::min(forced / 16, pl.KT)};
        const size_t tiles = (size_t)best.nb * best.mb;
        while (best.ks > 1 && (tiles > PF_PART_TILES || tiles * best.ks * pf_tile_floats(s.wn, s.wm) > PF_PART_FLOATS)) --best.ks;
        return best;
    }
    double best_t = 0;
    const double cu = m->nwg;
    for (const PfShape &s : PF_SHAPES) {
        const int nb = (pl.NT + 2 * s.wn - 1) / (2 * s.wn), mb = (rows + 32 * s.wm - 1) / (32 * s.wm);
        for (int ks : {1, 2, 3, 4, 6, 8}) {
            const size_t part = (size_t)nb * mb * ks * pf_tile_floats(s.wn, s.wm);
            if (ks > 1 && (pl.KT < 8 * ks || part > PF_PART_FLOATS || nb * mb > PF_PART_TILES)) break;
            double left = (double)nb * mb * ks, f = 0;
            const double slots = cu * s.occ;
            while (left > slots) {   // full rounds
                f += s.occ * s.t2;
                left -= slots;
            }
            f += left <= cu ? s.t1 : std::max(1.4 * s.t1, left / cu * s.t2);
            double t = f * ((pl.KT + ks - 1) / ks);
            if (ks > 1) t += 4.0 + ks + (double)part * 8.0 / 3.5e6;
            if (!best.shape || t < best_t) {
                best = {&s, nb, mb, ks};
                best_t = t;
            }
        }
    }
    return best;
}

// Floats of partial tiles the prefill GEMMs of chunks of up to `rows` rows need: the largest choice of pf_choose, which
// sees the rows in blocks of 64 (the narrowest row tile).
static size_t pf_part_floats(const ee_model *m, int rows, int forced)
{
    size_t need = 0;
    for (int r = 64; r < rows + 64; r += 64)
        for (int k = G_QKV; k <= G_DN; ++k) {
            const PfChoice ch = pf_choose(m, m->plan[0][k], r, forced);
            if (ch.ks > 1) need = std::max(need, (size_t)ch.nb * ch.mb * ch.ks * pf_tile_floats(ch.shape->wn, ch.shape->wm));
        }
    return need;
}

// n-tiles the busiest workgroup owns
static int plan_max_local(const GemmPlan &p)
{
    int mx = 0;
    for (int g = 0; g < p.nwg; ++g) {
        int nt0, n_local;
        wg_units(p, g, nt0, n_local);
        mx = std::max(mx, n_local);
    }
    return mx;
}

// ksl > 0: K split over groups of 1 << ksl workgroups where the k-tiles divide evenly (otherwise the plan comes back unsplit)
static GemmPlan make_plan(int N, int K, int tpu, int nwg_max, int ksl = 0)
{
    GemmPlan p;
    memset(&p, 0, sizeof p);
    p.N = N;
    p.K = K;
    p.NT = (N + 15) / 16;
    p.NT = (p.NT + tpu - 1) / tpu * tpu;
    p.KT = (K + 31) / 32;
    p.tpu = tpu;
    const int U = p.NT / tpu;
    p.KTs = p.KT;
    if (ksl > 0 && p.KT % (1 << ksl) == 0 && (nwg_max >> ksl) >= 1) {
        p.ksl = ksl;
        p.KTs = p.KT >> ksl;
    }
    // the fewest (groups of) workgroups that do not raise the busiest one's share
    const int groups_max = nwg_max >> p.ksl;
    const int most = (U + groups_max - 1) / groups_max, groups = std::min(groups_max, (U + most - 1) / most);
    p.nwg = groups << p.ksl;
    p.base = U / groups;
    p.rem = U % groups;
    // every wave's sequence has room for the busiest wave's k-steps of every n-tile
    p.steps = wave_ksteps(p.KTs, 0) * plan_max_local(p);
    return p;
}

// LDS map of one GEMM launch with `rows` rows (see StageLds)
static bool plan_lds(const GemmPlan &p, int rows, size_t lds_total, bool packed, StageLds &ly)
{
    const size_t misc = (MISC_BYTES + 255) / 256 * 256;
    const size_t corr = packed ? ((size_t)GROUP_TILES * rows * 64 + 255) / 256 * 256 : 0;
    if (lds_total < misc + corr + 4096) return false;
    const size_t avail = (lds_total - misc - corr) / 256 * 256;
    memset(&ly, 0, sizeof ly);
    if (avail < (size_t)SWAVES * WAVE_LDS_KB * 1024) return false;
    // cross-wave sum: SWAVES partial tiles plus one logits / squares tile per n-tile of a chunk
    int chunk = (int)(avail / ((size_t)rows * 64 * (SWAVES + 1)));
    chunk = std::min(chunk, GROUP_TILES);
    if (p.tpu == 2) chunk &= ~1;
    if (chunk < p.tpu) return false;
    ly.chunk = chunk;
    ly.zbuf_off = (int)((size_t)SWAVES * chunk * rows * 64);
    ly.corr_off = (int)avail;
    ly.misc_off = (int)(avail + corr);
    return true;
}

template <typename T>
static int dev_alloc(std::vector<void *> &list, T **out, size_t count, bool zero = true)
{
    void *p = nullptr;
    size_t bytes = std::max<size_t>(count * sizeof(T), 256);
    HIP_TRY(hipMalloc(&p, bytes));
    list.push_back(p);
    if (zero) HIP_TRY(hipMemset(p, 0, bytes));
    *out = reinterpret_cast<T *>(p);
    return EE_OK;
}

// the same for memory that the caller can do without: false, and no error left behind, if there is none
static bool try_alloc(std::vector<void *> &list, unsigned char **out, size_t bytes)
{
    void *p = nullptr;
    if (hipMalloc(&p, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    list.push_back(p);
    *out = static_cast<unsigned char *>(p);
    return true;
}

static size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// ------------------------------------------------------------------ model load

namespace {
struct FileMap {
    void *p = MAP_FAILED;
    size_t n = 0;
    ~FileMap()
    {
        if (p != MAP_FAILED) munmap(p, n);
    }
};
}  // namespace

// concatenates the sources row-wise in a device buffer and writes layer slice `dst` in tile order
static int upload_tiled(const ee_model *m, const GemmPlan &pl, int perm, const uint16_t *const *srcs, int n_src,
                        size_t elems_each, uint16_t *tmp, uint4 *dst)
{
    for (int i = 0; i < n_src; ++i)
        HIP_TRY(hipMemcpy(tmp + (size_t)i * elems_each, srcs[i], elems_each * 2, hipMemcpyHostToDevice));
    hipLaunchKernelGGL(tile_weights_kernel, dim3(pl.nwg), dim3(512), 0, 0, tmp, dst, pl, perm,
                       m->cfg.d_model, m->cfg.head_dim, m->cfg.d_ffn);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipDeviceSynchronize());
    return EE_OK;
}

static int upload_gain(const uint16_t *src, int d, uint16_t *tmp, float *dst)
{
    HIP_TRY(hipMemcpy(tmp, src, (size_t)d * 2, hipMemcpyHostToDevice));
    hipLaunchKernelGGL(bf16_to_f32_kernel, dim3((d + 255) / 256), dim3(256), 0, 0, tmp, dst, d);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipDeviceSynchronize());
    return EE_OK;
}

// Packs one matrix (its rows are in tmp, in file order) into slice `slice` of every variant of its kind, where that pays.
// A launch's stream gets a quarter shorter, but the helper waves' chain (list, then inputs, then sums) takes 5 us whatever the matrix:
// with less than 128 KB of weights per compute unit it is what the launch waits for.  us per launch, plain / packed, 5 rows: 1280-wide
// model QKV (9 MB) 5.3 / 6.4, 2048-wide QKV (25 MB) 7.4 / 8.2, down (22 MB) 9.4 / 9.2, 2560-wide QKV (38 MB, between events) 11.1 / 10.7, gate/up
// (70 MB) 14.7 / 13.6; 7B shape: output (34 MB) 8.8 / 8.4, down 17.6 / 15.5, QKV 18.2 / 15.1, gate/up 30.2 / 24.2, head 49.2 / 39.8.
constexpr int PACK_MIN_TILES = 32768;          // 32 MB
constexpr int PACK_TILES_PER_ESCAPE = 8;       // at most one escape per so many tiles of 512 weights (normally distributed ones: per 20)
static int pack_slice(ee_model *m, int kind, int perm, size_t slice, size_t n_elems, const uint16_t *tmp, void *work, size_t work_bytes, std::vector<Escape> &lists)
try {
    const GemmPlan &p0 = m->plan[0][kind];
    const int cap = p0.NT * p0.KT / PACK_TILES_PER_ESCAPE;
    if ((size_t)cap * sizeof(EscapeFound) + 2048 > work_bytes) return fail(EE_EDEVICE, "ee_model_load: packing buffer too small");
    unsigned *counts = static_cast<unsigned *>(work);                               // [256] exponents, then the escapes found
    EscapeFound *found = reinterpret_cast<EscapeFound *>(static_cast<char *>(work) + 2048);
    HIP_TRY(hipMemset(counts, 0, 2048));
    hipLaunchKernelGGL(exponent_count_kernel, dim3(1024), dim3(256), 0, 0, tmp, n_elems, counts);
    HIP_TRY(hipGetLastError());
    unsigned h[256];
    HIP_TRY(hipMemcpy(h, counts, sizeof h, hipMemcpyDeviceToHost));
    int base = 1, top = 0;
    size_t in_base = 0;
    for (int b = 1; b + 15 < 255; ++b) {
        size_t in = 0;
        for (int e = b; e < b + 16; ++e) in += h[e];
        if (in > in_base) {
            in_base = in;
            base = b;
        }
    }
    for (int e = 0; e < 255; ++e)
        if (h[e]) top = e;
    // (infinities and NaN are left alone, and so is a window so far off that moving it could overflow a sum)
    if (n_elems - in_base > (size_t)cap || h[255] || top + PACK_EXP0 - base > 160 || std::abs(PACK_EXP0 - base) > 32) return EE_OK;
    std::vector<EscapeFound> esc;
    for (int v = 0; v < 2; ++v) {
        if (m->packed[v][kind].empty()) continue;
        const GemmPlan &pl = m->plan[v][kind];
        unsigned char *dst = m->pk[v][kind] + slice * m->pk_bytes[v][kind];
        HIP_TRY(hipMemset(counts, 0, 4));
        hipLaunchKernelGGL(pack_weights_kernel, dim3(pl.nwg), dim3(512), 0, 0, tmp, dst, pl, perm,
                           m->cfg.d_model, m->cfg.head_dim, m->cfg.d_ffn, base, v == 0 ? found : nullptr, cap, reinterpret_cast<int *>(counts));
        HIP_TRY(hipGetLastError());
        if (v == 0) {
            int n = 0;
            HIP_TRY(hipMemcpy(&n, counts, sizeof n, hipMemcpyDeviceToHost));
            if (n > cap) return EE_OK;
            esc.resize((size_t)n);
            if (n) HIP_TRY(hipMemcpy(esc.data(), found, (size_t)n * sizeof(EscapeFound), hipMemcpyDeviceToHost));
        }
        // by slice of K, column and k; then cut into one part per helper wave of every workgroup and group, at column boundaries
        const int slice_k = pl.KTs * 32;
        auto key = [slice_k](const EscapeFound &e) { return std::make_tuple(e.k / slice_k, e.n, e.k); };
        std::sort(esc.begin(), esc.end(), [&](const EscapeFound &a, const EscapeFound &b) { return key(a) < key(b); });
        const int groups = (plan_max_local(pl) + GROUP_TILES - 1) / GROUP_TILES;
        struct Part {
            int first, end, col0, col1;
        };
        std::vector<Part> parts;
        int most = 0;
        for (int g = 0; g < pl.nwg; ++g) {
            int nt0, n_local;
            wg_units(pl, g, nt0, n_local);
            for (int gr = 0; gr < groups; ++gr) {
                const int c0 = (nt0 + std::min(n_local, gr * GROUP_TILES)) * 16, c1 = (nt0 + std::min(n_local, (gr + 1) * GROUP_TILES)) * 16;
                const int sl = g & ((1 << pl.ksl) - 1);
                auto at = [&](int col) {
                    return (int)(std::lower_bound(esc.begin(), esc.end(), std::make_tuple(sl, col, 0), [&](const EscapeFound &e, const std::tuple<int, int, int> &t) { return key(e) < t; }) - esc.begin());
                };
                Part p = {at(c0), 0, c0, 0};
                const int e0 = p.first, e1 = at(c1);
                for (int w = 1; w <= HWAVES; ++w) {
                    const int e = e0 + (int)((long long)(e1 - e0) * w / HWAVES);
                    p.col1 = w < HWAVES && e < e1 ? std::max(p.col0, esc[(size_t)e].n) : (w < HWAVES && e1 == e0 ? c0 + (c1 - c0) * w / HWAVES : c1);
                    p.end = at(p.col1);
                    parts.push_back(Part{p.first, p.end, p.col0 - c0, p.col1 - c0});
                    most = std::max(most, p.end - p.first);
                    p.first = p.end;
                    p.col0 = p.col1;
                }
            }
        }
        if (most > ESCAPES_MAX) return EE_OK;
        const int cap = (most + 8) & ~7;
        const size_t at = lists.size();
        lists.resize(at + parts.size() * (size_t)cap, Escape{0.f, 0});
        for (size_t i = 0; i < parts.size(); ++i) {
            const Part &p = parts[i];
            Escape *t = &lists[at + i * (size_t)cap];
            const int n = p.end - p.first, places = n + 1;
            memcpy(&t->delta, &places, 4);
            t->kn = (unsigned)p.col0 << 8 | (unsigned)p.col1;
            for (int j = 0; j < n; ++j) {
                const EscapeFound &e = esc[(size_t)(p.first + j)];
                const unsigned bits = e.bits << 16;
                float w;
                memcpy(&w, &bits, 4);
                t[1 + j] = Escape{ldexpf(w, PACK_EXP0 - base) - PACK_CODE0, (unsigned)e.k << 16 | ((unsigned)e.n & 0xFFFF)};
            }
        }
        m->packed[v][kind][slice] = {dst, at, groups, cap, ldexpf(1.0f, base - PACK_EXP0)};
    }
    return EE_OK;
} catch (const std::bad_alloc &) {
    return fail(EE_EDEVICE, "ee_model_load: out of host memory");
}

// Gives back the room of a kind's slices that stayed plain: the others move into an allocation of their size, if there is one.
static int trim_packed(ee_model *m, int v, int kind)
{
    std::vector<ee_model::PackedSlice> &slices = m->packed[v][kind];
    const size_t bytes = m->pk_bytes[v][kind], kept = (size_t)std::count_if(slices.begin(), slices.end(), [](const ee_model::PackedSlice &s) { return s.w; });
    unsigned char *to = nullptr;
    if (kept == slices.size() || (kept && !try_alloc(m->allocs, &to, kept * bytes))) return EE_OK;
    m->allocs.erase(std::find(m->allocs.begin(), m->allocs.end(), m->pk[v][kind]));
    const unsigned char *from = std::exchange(m->pk[v][kind], to);
    for (ee_model::PackedSlice &s : slices) {
        if (!s.w) continue;
        HIP_TRY(hipMemcpy(to, s.w, bytes, hipMemcpyDeviceToDevice));
        s.w = to;
        to += bytes;
    }
    HIP_TRY(hipFree(const_cast<unsigned char *>(from)));
    return EE_OK;
}

// which GEMM kinds get a K-split tile order in models loaded for more than 16 rows, and the splits (ee_tune_k_split)
static unsigned g_ksplit_kinds = (1u << G_O) | (1u << G_DN);
static int g_ksplit_log2 = KSPLIT_LOG2;

extern "C" int ee_tune_k_split(unsigned kind_mask, int log2_splits)
{
    if (log2_splits < 1 || (1 << log2_splits) > SWAVES || kind_mask >= (1u << G_KINDS))
        return fail(EE_EINVAL, "ee_tune_k_split: mask %u, log2 splits %d (mask below %u, 1 <= log2 splits <= 3)", kind_mask, log2_splits, 1u << G_KINDS);
    g_ksplit_kinds = kind_mask;
    g_ksplit_log2 = log2_splits;
    return EE_OK;
}

extern "C" int ee_model_free(ee_model *m)
{
    if (!m) return EE_OK;
    hipSetDevice(m->device);
    for (void *p : m->allocs) hipFree(p);
    delete m;
    return EE_OK;
}

extern "C" int ee_model_load_form(const char *path, int device, int max_rows, int form, ee_model **out)
{
    if (!path || !out) return fail(EE_EINVAL, "ee_model_load: null argument");
    if (form < EE_FORM_AUTO || form > EE_FORM_PACKED) return fail(EE_EINVAL, "ee_model_load: form %d not in [%d,%d]", form, EE_FORM_AUTO, EE_FORM_PACKED);
    if (max_rows < 1 || max_rows > EE_MAX_ROWS) return fail(EE_EINVAL, "ee_model_load: max_rows %d not in [1,%d]", max_rows, EE_MAX_ROWS);
    *out = nullptr;
    int fd = open(path, O_RDONLY);
    if (fd < 0) return fail(EE_EIO, "ee_model_load: cannot open %s", path);
    struct stat st;
    if (fstat(fd, &st) != 0) {
        close(fd);
        return fail(EE_EIO, "ee_model_load: cannot stat %s", path);
    }
    FileMap fm;
    fm.n = (size_t)st.st_size;
    if (fm.n < 256) {
        close(fd);
        return fail(EE_EFORMAT, "ee_model_load: %s is shorter than a header", path);
    }
    fm.p = mmap(nullptr, fm.n, PROT_READ, MAP_SHARED, fd, 0);
    close(fd);
    if (fm.p == MAP_FAILED) return fail(EE_EIO, "ee_model_load: cannot map %s", path);
    const uint8_t *b = static_cast<const uint8_t *>(fm.p);
    if (memcmp(b, "EEVMODL1", 8) != 0) return fail(EE_EFORMAT, "ee_model_load: bad magic in %s", path);
    uint32_t u[8];
    memcpy(u, b + 8, sizeof u);
    if (u[0] != 1) return fail(EE_EFORMAT, "ee_model_load: unsupported version %u", u[0]);
    ee_model_config c;
    memset(&c, 0, sizeof c);
    c.n_layers = (int)u[1];
    c.d_model = (int)u[2];
    c.n_heads = (int)u[3];
    c.head_dim = (int)u[4];
    c.d_ffn = (int)u[5];
    c.vocab = (int)u[6];
    c.n_exits = (int)u[7];
    memcpy(&c.rope_base, b + 40, 4);
    memcpy(&c.rms_eps, b + 44, 4);
    if (c.n_layers < 1 || c.n_layers > 4096 || c.d_model < 16 || c.n_heads < 1 || c.d_ffn < 1 || c.vocab < 1 ||
        c.n_exits < 0 || c.n_exits > EE_MAX_EXITS || (long long)c.n_heads * c.head_dim != c.d_model)
        return fail(EE_EFORMAT, "ee_model_load: inconsistent header");
    if (c.head_dim != 64 && c.head_dim != 128)
        return fail(EE_EFORMAT, "ee_model_load: head_dim %d unsupported (64 or 128)", c.head_dim);
    if (c.d_model % 16 != 0 || c.d_ffn % 2 != 0)
        return fail(EE_EFORMAT, "ee_model_load: d_model must be a multiple of 16, d_ffn even");
    uint32_t ex[EE_MAX_EXITS], ad[2];
    static_assert(EE_MAX_EXITS == 40, "the header's exit table has 40 entries");
    memcpy(ex, b + 48, sizeof ex);
    memcpy(ad, b + 208, sizeof ad);
    const int n_ad = (int)ad[0], ad_w = (int)ad[1];
    if ((n_ad == 0) != (ad_w == 0) || n_ad < 0 || n_ad > 64 || ad_w < 0 || ad_w > 4096 || (n_ad * ad_w) % 16 != 0)
        return fail(EE_EFORMAT, "ee_model_load: bad adapter shape %d x %d (the hidden units together must be a multiple of 16)", n_ad, ad_w);
    const size_t A = (size_t)n_ad * (size_t)ad_w;
    c.n_adapters = n_ad;
    c.adapter_width = ad_w;
    for (int i = 0; i < c.n_exits; ++i) {
        c.exit_layers[i] = (int)ex[i];
        if (c.exit_layers[i] < 1 || c.exit_layers[i] >= c.n_layers || (i > 0 && c.exit_layers[i] <= c.exit_layers[i - 1]))
            return fail(EE_EFORMAT, "ee_model_load: bad exit layer list");
    }
    const size_t d = (size_t)c.d_model, F = (size_t)c.d_ffn, V = (size_t)c.vocab;
    // tensor offsets: each tensor starts on a 256-byte boundary, fixed order
    size_t off = 256;
    auto take = [&](size_t elems) -> const uint16_t * {
        off = align_up(off, 256);
        const uint16_t *p = reinterpret_cast<const uint16_t *>(b + off);
        off += elems * 2;
        return p;
    };
    struct LayerSrc {
        const uint16_t *g_attn, *wq, *wk, *wv, *wo, *g_ffn, *wg, *wu, *wd;
    };
    const uint16_t *emb = take(V * d);
    std::vector<LayerSrc> ls((size_t)c.n_layers);
    for (auto &l : ls) {
        l.g_attn = take(d);
        l.wq = take(d * d);
        l.wk = take(d * d);
        l.wv = take(d * d);
        l.wo = take(d * d);
        l.g_ffn = take(d);
        l.wg = take(F * d);
        l.wu = take(F * d);
        l.wd = take(d * F);
    }
    const uint16_t *g_final = take(d);
    const uint16_t *w_lm = take(V * d);
    const uint16_t *g_exit_src[EE_MAX_EXITS];
    for (int i = 0; i < c.n_exits; ++i) g_exit_src[i] = take(d);
    struct AdapterSrc {
        const uint16_t *down, *bdown, *up, *bup;
    };
    std::vector<AdapterSrc> ads((size_t)(A ? c.n_exits : 0));
    for (auto &x : ads) {
        x.down = take(A * d);
        x.bdown = take(A);
        x.up = take(d * A);
        x.bup = take((size_t)n_ad * d);
    }
    if (off > fm.n) return fail(EE_EFORMAT, "ee_model_load: %s is truncated (%zu < %zu bytes)", path, fm.n, off);

    int n_dev = 0;
    HIP_TRY(hipGetDeviceCount(&n_dev));
    if (device < 0 || device >= n_dev) return fail(EE_EINVAL, "ee_model_load: device %d of %d", device, n_dev);
    HIP_TRY(hipSetDevice(device));
    hipDeviceProp_t prop;
    HIP_TRY(hipGetDeviceProperties(&prop, device));
    if (strncmp(prop.gcnArchName, "gfx950", 6) != 0)
        return fail(EE_EDEVICE, "ee_model_load: device %d is %s, this library is built for gfx950 only", device, prop.gcnArchName);

    ee_model *m = new (std::nothrow) ee_model();
    if (!m) return fail(EE_EDEVICE, "out of host memory");
    m->device = device;
    m->nwg = std::min(prop.multiProcessorCount, SS_LD);   // one workgroup per compute unit; the accept step reads at most 256 candidates per row
    c.max_rows = max_rows;
    c.n_workgroups = m->nwg;
    m->cfg = c;
    ModelDev &md = m->host_md;
    memset(&md, 0, sizeof md);
    md.L = c.n_layers;
    md.d = c.d_model;
    md.H = c.n_heads;
    md.hd = c.head_dim;
    md.F = c.d_ffn;
    md.V = c.vocab;
    md.eps = c.rms_eps;
    md.att_scale = (float)(1.0 / sqrt((double)c.head_dim));
    md.Kpad_d = (int)align_up(d, 32);
    md.Kpad_F = (int)align_up(F, 32);
    md.rows_max = max_rows;
    md.A = (int)A;
    md.Kpad_A = (int)align_up(A, 32);
    if (c.d_ffn % 16 != 0) {
        ee_model_free(m);
        return fail(EE_EFORMAT, "ee_model_load: d_ffn must be a multiple of 16");
    }

    // ---- weight-stream plans (independent of the rows) and the LDS block every launch asks for
    size_t lds_cap = prop.sharedMemPerBlock;
    {
        int optin = 0;
        if (hipDeviceGetAttribute(&optin, hipDeviceAttributeSharedMemPerBlockOptin, device) == hipSuccess && optin > 0)
            lds_cap = std::max(lds_cap, (size_t)optin);
    }
    auto plan_of = [&](int kind, int ksl) {
        switch (kind) {
        case G_QKV: return make_plan(3 * c.d_model, c.d_model, 1, m->nwg, ksl);
        case G_O: return make_plan(c.d_model, c.d_model, 1, m->nwg, ksl);
        case G_GU: return make_plan(2 * c.d_ffn, c.d_model, 2, m->nwg, ksl);
        case G_DN: return make_plan(c.d_model, c.d_ffn, 1, m->nwg, ksl);
        case G_HEAD: return make_plan(c.vocab, c.d_model, 1, m->nwg, ksl);
        case G_AD: return make_plan(A ? (int)A : 16, c.d_model, 1, m->nwg, ksl);
        default: return make_plan(c.d_model, A ? (int)A : 32, 1, m->nwg, ksl);
        }
    };
    memset(m->plan, 0, sizeof m->plan);
    memset(m->w, 0, sizeof m->w);
    memset(m->wstride, 0, sizeof m->wstride);
    for (int k = 0; k < G_KINDS; ++k) m->plan[0][k] = plan_of(k, 0);
    if (max_rows > 16) {
        // Launches of more than 16 rows: K split four ways for the projections whose input is as large
        // as, or larger than, a workgroup's share of the weights (see GemmPlan).  Those weights are
        // kept in both tile orders; launches of up to 16 rows keep using the unsplit one.
        const unsigned kinds = g_ksplit_kinds;
        const int ksl = g_ksplit_log2;
        for (int k = 0; k < G_KINDS; ++k)
            if ((kinds >> k) & 1u) {
                const GemmPlan p = plan_of(k, ksl);
                if (p.ksl > 0) m->plan[1][k] = p;
            }
    }
    m->lds_budget = lds_cap / 256 * 256;   // the whole block: more than half of it also keeps a compute unit to one workgroup
    for (int v = 0; v < 2; ++v)
        for (int k = 0; k < G_KINDS; ++k) {
            const GemmPlan &pl = m->plan[v][k];
            if (pl.nwg == 0) continue;
            StageLds ly;
            if (!plan_lds(pl, max_rows, m->lds_budget, false, ly)) {
                ee_model_free(m);
                return fail(EE_EDEVICE, "ee_model_load: max_rows %d needs more LDS than the device's %zu bytes", max_rows, lds_cap);
            }
            // the kernels' exact small-integer division (div_small) covers column numbers
            if (pl.N > DIV_SMALL_MAX) {
                ee_model_free(m);
                return fail(EE_EFORMAT, "ee_model_load: a weight matrix with %d rows is beyond what the kernels' index arithmetic covers", pl.N);
            }
            // The kernels count tiles in ints (PfArgs::tab), 1 KB each; larger matrices than this have never been run.
            if ((long long)pl.steps * pl.nwg * SWAVES * 1024 >= (1LL << 31)) {
                ee_model_free(m);
                return fail(EE_EFORMAT, "ee_model_load: a weight matrix of %d x %d exceeds the 2 GiB a matrix may take", pl.N, pl.K);
            }
            m->wstride[v][k] = (long long)pl.steps * pl.nwg * SWAVES * 64;
        }
    {
        const size_t att = att_lds(c.head_dim, ATT_ROWS);
        const size_t emb = (size_t)max_rows * (((c.d_model + m->nwg - 1) / m->nwg + 3) / 4 + 1) * sizeof(float);
        if (att > m->lds_budget || emb > m->lds_budget) {
            ee_model_free(m);
            return fail(EE_EDEVICE, "ee_model_load: not enough LDS");
        }
        std::vector<pass_kernel_t> ks = {att_kernel(64), att_kernel(128), ee_misc_kernel};
        for (int k = 0; k < G_KINDS; ++k)
            for (int rows = 8; rows <= EE_MAX_ROWS; rows += 8)
                for (bool packed : {false, true}) ks.push_back(gemm_kernel(k, rows, packed));
        for (pass_kernel_t k : ks) {
            hipError_t fe = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)m->lds_budget);
            if (fe != hipSuccess) {
                ee_model_free(m);
                return fail(EE_EDEVICE, "hipFuncSetAttribute(%zu bytes LDS): %s", m->lds_budget, hipGetErrorString(fe));
            }
        }
    }

    {
        std::vector<std::pair<const void *, size_t>> ks;
        for (const PfShape &sh : PF_SHAPES)
            for (pf_kernel_t k : sh.gemm) ks.push_back({reinterpret_cast<const void *>(k), pf_gemm_lds(sh.wn, sh.wm, sh.grp)});
        for (int rt = 1; rt <= 2; ++rt) ks.push_back({reinterpret_cast<const void *>(pf_att(c.head_dim, rt)), pf_att_lds(c.head_dim, ATT_MAX_SPLITS * ATT_TILES * WAVES)});
        for (const auto &k : ks) {
            hipError_t fe = hipFuncSetAttribute(k.first, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.second);
            if (fe != hipSuccess) {
                ee_model_free(m);
                return fail(EE_EDEVICE, "hipFuncSetAttribute(%zu bytes LDS): %s", k.second, hipGetErrorString(fe));
            }
        }
    }

    int rc = EE_OK;
    uint16_t *tmp = nullptr;
    size_t tmp_elems = std::max({V * d, 3 * d * d, 2 * F * d, A * d});
    void *tmp_raw = nullptr;
    if (hipMalloc(&tmp_raw, tmp_elems * 2) != hipSuccess) {
        ee_model_free(m);
        return fail(EE_EDEVICE, "ee_model_load: cannot allocate the upload buffer");
    }
    tmp = static_cast<uint16_t *>(tmp_raw);

    void *pack_work = nullptr;
    size_t pack_work_bytes = 0;
    auto bail = [&](int code) {
        hipFree(tmp_raw);
        hipFree(pack_work);
        ee_model_free(m);
        return code;
    };

    // embedding table stays row-major
    uint16_t *dev_emb = nullptr;
    if ((rc = dev_alloc(m->allocs, &dev_emb, V * d, false)) != EE_OK) return bail(rc);
    if (hipMemcpy(dev_emb, emb, V * d * 2, hipMemcpyHostToDevice) != hipSuccess) return bail(fail(EE_EDEVICE, "upload of the embedding table failed"));
    md.emb = dev_emb;

    // tiled weights: one allocation per GEMM kind and variant, layers at a fixed stride.  Tile slots that no wave's
    // sequence reaches (a wave without k-steps, the shorter sequences' tails) are never read; they stay zero.
    float *g_attn = nullptr, *g_ffn = nullptr, *g_final_d = nullptr;
    const size_t Lz = (size_t)c.n_layers;
    uint4 *wdev[2][G_KINDS];
    memset(wdev, 0, sizeof wdev);
    for (int v = 0; v < 2; ++v)
        for (int k = 0; k < G_KINDS; ++k) {
            if (m->plan[v][k].nwg == 0 || ((k == G_AD || k == G_AU) && !A)) continue;
            const size_t slices = k == G_HEAD ? 1 : ((k == G_AD || k == G_AU) ? (size_t)c.n_exits : Lz);
            if ((rc = dev_alloc(m->allocs, &wdev[v][k], std::max<size_t>(slices, 1) * (size_t)m->wstride[v][k], true)) != EE_OK) return bail(rc);
            m->w[v][k] = wdev[v][k];
        }
    // Packed forms.  They come on top of the plain ones, which prefill reads (10 GB for the 7B shape, 13 with the K-split order): where the
    // caller leaves it open, only if all of them take at most an eighth of the memory that is free now, so that little is taken from the
    // sessions and models still to come, and where an allocation fails the kind stays plain.
    std::vector<Escape> lists;
    {
        size_t free_bytes = 0, total_bytes = 0, need = 0;
        if (hipMemGetInfo(&free_bytes, &total_bytes) != hipSuccess) free_bytes = 0;
        bool want[G_KINDS] = {};
        for (int k = G_QKV; k <= G_HEAD; ++k) {
            const GemmPlan &p0 = m->plan[0][k];
            StageLds ly;
            want[k] = (long long)p0.NT * p0.KT >= PACK_MIN_TILES && p0.K <= 65536;
            for (int v = 0; v < 2; ++v) {
                const GemmPlan &pl = m->plan[v][k];
                if (pl.nwg == 0) continue;
                want[k] = want[k] && plan_lds(pl, max_rows, m->lds_budget, true, ly);
                m->pk_bytes[v][k] = (size_t)pl.steps * pl.nwg * SWAVES * PACK_TILE;
                if (want[k]) need += m->pk_bytes[v][k] * (k == G_HEAD ? 1 : Lz);
            }
            if (want[k]) pack_work_bytes = std::max(pack_work_bytes, (size_t)p0.NT * p0.KT / PACK_TILES_PER_ESCAPE * sizeof(EscapeFound) + 2048);
        }
        if (form == EE_FORM_PLAIN || (form == EE_FORM_AUTO && need > free_bytes / 8)) pack_work_bytes = 0;
        if (pack_work_bytes && hipMalloc(&pack_work, pack_work_bytes) != hipSuccess) {
            (void)hipGetLastError();
            pack_work = nullptr;
            if (form == EE_FORM_PACKED) return bail(fail(EE_EDEVICE, "ee_model_load: no memory for packing the weights"));
        }
        for (int k = G_QKV; pack_work && k <= G_HEAD; ++k)
            for (int v = 0; v < 2; ++v) {
                const size_t slices = k == G_HEAD ? 1 : Lz;
                if (!want[k] || m->plan[v][k].nwg == 0 || (v == 1 && m->packed[0][k].empty())) continue;
                if (!try_alloc(m->allocs, &m->pk[v][k], slices * m->pk_bytes[v][k])) {
                    if (form == EE_FORM_PACKED) return bail(fail(EE_EDEVICE, "ee_model_load: no memory for the packed weights"));
                    continue;
                }
                if (hipMemset(m->pk[v][k], 0, slices * m->pk_bytes[v][k]) != hipSuccess) return bail(fail(EE_EDEVICE, "clearing of a packed matrix failed"));
                m->packed[v][k].assign(slices, ee_model::PackedSlice{nullptr, 0, 0, 0, 0.f});
            }
    }
    // every variant of a kind from the same upload
    auto tile_all = [&](int kind, int perm, const uint16_t *const *srcs, int n_src, size_t elems_each, size_t slice) {
        for (int v = 0; v < 2; ++v) {
            if (!wdev[v][kind]) continue;
            const int r = upload_tiled(m, m->plan[v][kind], perm, srcs, v == 0 ? n_src : 0, elems_each, tmp,
                                       wdev[v][kind] + slice * (size_t)m->wstride[v][kind]);
            if (r != EE_OK) return r;
        }
        return !m->packed[0][kind].empty() ? pack_slice(m, kind, perm, slice, n_src * elems_each, tmp, pack_work, pack_work_bytes, lists) : (int)EE_OK;
    };
    if ((rc = dev_alloc(m->allocs, &g_attn, Lz * d, false)) != EE_OK) return bail(rc);
    if ((rc = dev_alloc(m->allocs, &g_ffn, Lz * d, false)) != EE_OK) return bail(rc);
    if ((rc = dev_alloc(m->allocs, &g_final_d, d, false)) != EE_OK) return bail(rc);
    for (int l = 0; l < c.n_layers; ++l) {
        const LayerSrc &s = ls[(size_t)l];
        const uint16_t *qkv[3] = {s.wq, s.wk, s.wv};
        const uint16_t *gu[2] = {s.wg, s.wu};
        const uint16_t *so[1] = {s.wo}, *sd[1] = {s.wd};
        if ((rc = tile_all(G_QKV, PERM_QKV, qkv, 3, d * d, (size_t)l)) != EE_OK) return bail(rc);
        if ((rc = tile_all(G_O, PERM_NONE, so, 1, d * d, (size_t)l)) != EE_OK) return bail(rc);
        if ((rc = tile_all(G_GU, PERM_GU, gu, 2, F * d, (size_t)l)) != EE_OK) return bail(rc);
        if ((rc = tile_all(G_DN, PERM_NONE, sd, 1, d * F, (size_t)l)) != EE_OK) return bail(rc);
        if ((rc = upload_gain(s.g_attn, c.d_model, tmp, g_attn + (size_t)l * d)) != EE_OK) return bail(rc);
        if ((rc = upload_gain(s.g_ffn, c.d_model, tmp, g_ffn + (size_t)l * d)) != EE_OK) return bail(rc);
    }
    {
        const uint16_t *lm[1] = {w_lm};
        if ((rc = tile_all(G_HEAD, PERM_NONE, lm, 1, V * d, 0)) != EE_OK) return bail(rc);
        if ((rc = upload_gain(g_final, c.d_model, tmp, g_final_d)) != EE_OK) return bail(rc);
        float *ges = nullptr;   // (one allocation, exit after exit: adapters of several exits share a launch)
        if (c.n_exits && (rc = dev_alloc(m->allocs, &ges, (size_t)c.n_exits * d, false)) != EE_OK) return bail(rc);
        for (int i = 0; i < c.n_exits; ++i) {
            float *ge = ges + (size_t)i * d;
            if ((rc = upload_gain(g_exit_src[i], c.d_model, tmp, ge)) != EE_OK) return bail(rc);
            m->g_exit[i] = ge;
        }
    }
    if (A) {
        // adapters: weights in tile order per stored exit; biases as fp32, the bottlenecks' output biases summed in order
        float *bds = nullptr, *bus = nullptr;
        if (c.n_exits && (rc = dev_alloc(m->allocs, &bds, (size_t)c.n_exits * A, false)) != EE_OK) return bail(rc);
        if (c.n_exits && (rc = dev_alloc(m->allocs, &bus, (size_t)c.n_exits * d, false)) != EE_OK) return bail(rc);
        for (int i = 0; i < c.n_exits; ++i) {
            const uint16_t *sd_[1] = {ads[(size_t)i].down}, *su_[1] = {ads[(size_t)i].up};
            if ((rc = tile_all(G_AD, PERM_NONE, sd_, 1, A * d, (size_t)i)) != EE_OK) return bail(rc);
            if ((rc = tile_all(G_AU, PERM_NONE, su_, 1, d * A, (size_t)i)) != EE_OK) return bail(rc);
            float *bd = bds + (size_t)i * A, *bu = bus + (size_t)i * d;
            std::vector<float> hb(std::max(A, d));
            auto bf = [](uint16_t v) {
                uint32_t u32 = (uint32_t)v << 16;
                float f;
                memcpy(&f, &u32, 4);
                return f;
            };
            for (size_t r = 0; r < A; ++r) hb[r] = bf(ads[(size_t)i].bdown[r]);
            if (hipMemcpy(bd, hb.data(), A * 4, hipMemcpyHostToDevice) != hipSuccess) return bail(fail(EE_EDEVICE, "upload of adapter biases failed"));
            for (size_t col = 0; col < d; ++col) {
                float acc = 0.f;
                for (int j = 0; j < n_ad; ++j) acc += bf(ads[(size_t)i].bup[(size_t)j * d + col]);
                hb[col] = acc;
            }
            if (hipMemcpy(bu, hb.data(), d * 4, hipMemcpyHostToDevice) != hipSuccess) return bail(fail(EE_EDEVICE, "upload of adapter biases failed"));
            m->ad_bdown[i] = bd;
            m->ad_bup[i] = bu;
        }
    }
    for (int k = G_QKV; k <= G_DN; ++k) {
        const GemmPlan &pl = m->plan[0][k];
        std::vector<int2> tab((size_t)pl.NT, make_int2(0, 0));
        const int S0 = wave_ksteps(pl.KTs, 0);
        for (int g = 0; g < pl.nwg; ++g) {
            int nt0, n_local, seq = 0;
            wg_units(pl, g, nt0, n_local);
            for (int g0 = 0; g0 < n_local; g0 += GROUP_TILES) {
                const int nl = std::min(GROUP_TILES, n_local - g0);
                for (int i = 0; i < nl; ++i)
                    tab[(size_t)(nt0 + g0 + i)] = make_int2(((seq + i) * pl.nwg + g) * SWAVES, nl * pl.nwg * SWAVES);
                seq += S0 * nl;
            }
        }
        int2 *dev = nullptr;
        if ((rc = dev_alloc(m->allocs, &dev, tab.size(), false)) != EE_OK) return bail(rc);
        if (hipMemcpy(dev, tab.data(), tab.size() * sizeof(int2), hipMemcpyHostToDevice) != hipSuccess) return bail(fail(EE_EDEVICE, "upload of a tile table failed"));
        m->tile_tab[k] = dev;
    }
    if (!lists.empty()) {
        Escape *dev = nullptr;
        if ((rc = dev_alloc(m->allocs, &dev, lists.size(), false)) != EE_OK) return bail(rc);
        if (hipMemcpy(dev, lists.data(), lists.size() * sizeof(Escape), hipMemcpyHostToDevice) != hipSuccess) return bail(fail(EE_EDEVICE, "upload of the escapes failed"));
        m->escapes = dev;
    }
    for (int v = 0; v < 2; ++v)
        for (int k = G_QKV; k <= G_HEAD; ++k)
            if ((rc = trim_packed(m, v, k)) != EE_OK) return bail(rc);
    md.g_attn = g_attn;
    md.g_ffn = g_ffn;
    md.g_final = g_final_d;
    hipFree(tmp_raw);
    hipFree(pack_work);
    tmp_raw = pack_work = nullptr;
    if (hipDeviceSynchronize() != hipSuccess) return bail(fail(EE_EDEVICE, "device error while loading the model"));
    *out = m;
    return EE_OK;
}

extern "C" int ee_model_load_ex(const char *path, int device, int max_rows, ee_model **out)
{
    return ee_model_load_form(path, device, max_rows, EE_FORM_AUTO, out);
}

extern "C" int ee_model_load(const char *path, int device, ee_model **out)
{
    return ee_model_load_ex(path, device, 16, out);
}

extern "C" int ee_model_packed_bytes(const ee_model *m, size_t *bytes)
{
    if (!m || !bytes) return fail(EE_EINVAL, "ee_model_packed_bytes: null argument");
    *bytes = 0;
    for (int v = 0; v < 2; ++v)
        for (int k = G_QKV; k <= G_HEAD; ++k)
            if (m->pk[v][k])
                for (const ee_model::PackedSlice &s : m->packed[v][k]) *bytes += s.w ? m->pk_bytes[v][k] : 0;
    return EE_OK;
}

extern "C" int ee_model_info(const ee_model *m, ee_model_config *out)
{
    if (!m || !out) return fail(EE_EINVAL, "ee_model_info: null argument");
    *out = m->cfg;
    return EE_OK;
}

// ------------------------------------------------------------------ sessions

// Splits of the cache's pages per attention unit.  Few pages (10 of heads of 64, 5 of 128): one, whose waves take a page
// each; the exchange and the merge of several cost 1.3 us.  Up to 8 pages (one round of the merge) of few heads: one per page, as
// long as the items cover at most half the compute units.  Otherwise one per two pages, rounded up, or fewer: as many as occupy
// every compute unit (one unit alone pulls a head's cache too slowly).  No more than ATT_TILES pages per wave, and no more items
// than the leader's partials buffer holds.  us per launch, one split / one per two pages / one per page (32 heads: at most 8):
//   4 heads of 64:    5 rows, 8 pages 4.6 / 5.4 / 5.2, 10 pages 5.3 / 5.5 / 6.0, 11 pages 5.5 / 5.5 / 5.9; 16 rows, 10 pages 5.9 / 5.8 / 6.3
//   10 heads of 128:  5 rows, 5 pages 6.0 / 6.1 / 6.0, 6 pages 6.3 / 6.2 / 6.0, 8 pages 7.1 / 6.3 / 6.0, 9 pages 7.8 / 6.2 / 6.7;
//                     16 rows, 5 pages 6.6 / 6.9 / 6.7, 6 pages 7.1 / 7.1 / 6.7, 8 pages 8.0 / 7.1 / 6.7, 9 pages 9.0 / 7.0 / 7.7
//   32 heads of 128:  5 rows, 5 pages 5.9 / 6.4 / 6.3, 6 pages 6.3 / 6.5 / 6.5, 8 pages 7.2 / 6.5 / 6.9, 9 pages 7.9 / 6.6 / 7.0;
//                     16 rows, 5 pages 6.5 / 7.2 / 7.0, 6 pages 6.9 / 7.1 / 7.2, 8 pages 8.1 / 7.3 / 7.5, 9 pages 8.7 / 7.3 / 7.6
// Returns 0 when the buffer is too small for the context.
static int attention_splits(const ee_session *lead, int items_cap, int n_sess, int M, int n_pos_max)
{
    const ee_model *m = lead->m;
    const int chunks = (M + ATT_ROWS - 1) / ATT_ROWS;
    const int units = n_sess * m->cfg.n_heads * chunks;
    const int pages = (n_pos_max + KV_PAGE - 1) / KV_PAGE;
    const int forced = (pages + ATT_TILES * WAVES - 1) / (ATT_TILES * WAVES);
    const int cap = std::min(ATT_MAX_SPLITS, items_cap / std::max(units, 1));
    int s = std::min(m->nwg / std::max(units, 1), (pages + 1) / 2);
    if (pages * m->cfg.head_dim <= 640)
        s = 1;
    else if (pages <= 8 && units * pages <= m->nwg / 2)
        s = pages;
    if (lead->att_splits_opt > 0) s = lead->att_splits_opt;
    s = std::max(std::max(1, s), forced);
    if (forced > cap) return 0;
    return std::min(s, cap);
}

// Splits of a batch by session: pages per split are the same for all, so that a session has as many splits as its own pages ask for,
// instead of the number that attention_splits gives all of them.  Taken where the launch's estimated time is lower by 5 %: a
// start, an exchange if anything is split (its merge takes eight at a time), the pages of the largest workgroup and a compute unit's share of
// all pages (a little more than the larger of the two), and a second round where the workgroups outnumber the units (one fits a unit).  us, fitted
// to 670 batches of 2 to 16 sessions of 9 to 9000 positions, 4 to 40 heads of 64 and 128 and every number of splits (6 % off, root mean square).
// Against the number all have, us a launch: 32 heads of 128 over 1048, 396 and 9 positions 22.8 -> 16.1, 20 over ten of 888 to 11 27.1 -> 15.1, 16 of 64 over
// twelve of 1064 to 9 17.3 -> 12.4; those batches 5 % on average, one in a hundred slower by up to 9 %.
static void attention_splits_by_session(const ee_session *lead, int items_cap, ee_session *const *sessions, int n_sess, int M, PassArgs &a)
{
    const ee_model *m = lead->m;
    const int H = m->cfg.n_heads, units = n_sess * H;
    if (n_sess < 2 || lead->att_splits_opt > 0) return;
    int pages[EE_MAX_BATCH], most = 0, all = 0;
    for (int i = 0; i < n_sess; ++i) {
        pages[i] = (sessions[i]->kv_len + M + KV_PAGE - 1) / KV_PAGE;
        most = std::max(most, pages[i]);
        all += pages[i];
    }
    struct Cost {
        float start, row, exchange, merge, page, share, round, rounds;
    };
    static constexpr Cost COST[2] = {{5.6f, 0.05f, 1.6f, 0.8f, 0.18f, 0.35f, 1.2f, 2.4f}, {5.4f, 0.145f, 1.55f, 0.55f, 0.385f, 0.73f, 1.65f, 2.8f}};   // heads of 64, of 128
    const Cost &c = COST[m->cfg.head_dim > 64];
    const float nwg = (float)m->nwg, share = c.share * (float)(all * H) / nwg;
    auto estimate = [&](int s, int items) {
        const float largest = c.page * (float)((most + s - 1) / s), more = ((float)items - nwg) / nwg;
        return c.start + c.row * (float)M + (s > 1 ? c.exchange : 0.f) + (s > 8 ? c.merge : 0.f) + sqrtf(hypotf(largest * largest, share * share)) +
               (more > 0.f ? c.round + c.rounds * more : 0.f);
    };
    float best = 0.95f * estimate(a.att_splits, units * a.att_splits);
    const int forced = (most + ATT_TILES * WAVES - 1) / (ATT_TILES * WAVES);
    for (int s = std::max(forced, 1); s <= std::min({ATT_MAX_SPLITS, items_cap / units, most}); ++s) {
        const int per = (most + s - 1) / s;
        unsigned long long starts = 0;
        int total = 0;
        for (int i = 0; i < n_sess; ++i) {
            starts |= total < 64 ? 1ull << total : 0;
            total += (pages[i] + per - 1) / per;
        }
        const float t = estimate(s, H * total);
        if (t >= best || total > 63) continue;
        best = t;
        a.att_splits = s;
        a.att_starts = starts | 1ull << total;
    }
}

extern "C" int ee_session_free(ee_session *s)
{
    if (!s) return EE_OK;
    hipSetDevice(s->m->device);
    if (s->stream) hipStreamSynchronize(s->stream);
    if (s->copy_stream) hipStreamSynchronize(s->copy_stream);
    for (void *p : s->allocs) hipFree(p);
    if (s->host_page_table) hipHostFree(s->host_page_table);
    if (s->host_sample) hipHostFree(s->host_sample);
    if (s->host_pf_tokens) hipHostFree(s->host_pf_tokens);
    if (s->result) hipHostFree(s->result);
    if (s->host_sessdev) hipHostFree(s->host_sessdev);
    if (s->ev_start) hipEventDestroy(s->ev_start);
    if (s->ev_final) hipEventDestroy(s->ev_final);
    for (hipEvent_t e : s->ev_exit)
        if (e) hipEventDestroy(e);
    for (hipEvent_t e : s->lt_events) hipEventDestroy(e);
    if (s->ev_copy) hipEventDestroy(s->ev_copy);
    if (s->copy_stream) hipStreamDestroy(s->copy_stream);
    if (s->stream) hipStreamDestroy(s->stream);
    delete s;
    return EE_OK;
}

extern "C" int ee_session_create(const ee_model *m, int max_ctx, int max_gamma, unsigned flags, ee_session **out)
{
    if (!m || !out) return fail(EE_EINVAL, "ee_session_create: null argument");
    *out = nullptr;
    if (max_gamma < 1 || max_gamma > EE_MAX_M - 1) return fail(EE_EINVAL, "ee_session_create: max_gamma %d not in [1,%d]", max_gamma, EE_MAX_M - 1);
    if (max_gamma + 1 > m->cfg.max_rows) return fail(EE_EINVAL, "ee_session_create: max_gamma+1 exceeds the model's max_rows %d", m->cfg.max_rows);
    // attention keeps at most ATT_TILES pages per wave and ATT_MAX_SPLITS splits per head
    const int ctx_cap = ATT_MAX_SPLITS * ATT_TILES * WAVES * KV_PAGE;
    if (max_ctx < max_gamma + 2 || max_ctx > ctx_cap)
        return fail(EE_EINVAL, "ee_session_create: max_ctx %d out of range (at most %d)", max_ctx, ctx_cap);
    HIP_TRY(hipSetDevice(m->device));
    ee_session *s = new (std::nothrow) ee_session();
    if (!s) return fail(EE_EDEVICE, "out of host memory");
    s->m = m;
    s->flags = flags;
    s->max_ctx = max_ctx;
    s->max_gamma = max_gamma;
    s->leader = s;
    s->head_batch = 1;
    const ee_model_config &c = m->cfg;
    const int rows_max = c.max_rows;
    const size_t d = (size_t)c.d_model;
    int rc = EE_OK;
#define S_TRY(expr)                  \
    do {                             \
        rc = (expr);                 \
        if (rc != EE_OK) {           \
            ee_session_free(s);      \
            return rc;               \
        }                            \
    } while (0)
#define S_HIP(expr)                                                                          \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess) {                                                              \
            ee_session_free(s);                                                              \
            return fail(EE_EDEVICE, "%s failed: %s", #expr, hipGetErrorString(e_));          \
        }                                                                                    \
    } while (0)

    S_HIP(hipStreamCreate(&s->stream));
    s->run_stream = s->stream;
    S_HIP(hipEventCreate(&s->ev_start));
    S_HIP(hipEventCreate(&s->ev_final));
    for (int i = 0; i < EE_MAX_EXITS; ++i) S_HIP(hipEventCreate(&s->ev_exit[i]));

    s->n_pages = (max_ctx + KV_PAGE - 1) / KV_PAGE;
    size_t kv_elems = (size_t)c.n_layers * s->n_pages * c.n_heads * KV_PAGE * 2 * c.head_dim;  // hi and lo terms
    S_TRY(dev_alloc(s->allocs, &s->kpool, kv_elems));
    S_TRY(dev_alloc(s->allocs, &s->vpool, kv_elems));
    S_TRY(dev_alloc(s->allocs, &s->dev_page_table, (size_t)s->n_pages));
    S_HIP(hipHostMalloc(reinterpret_cast<void **>(&s->host_page_table), (size_t)s->n_pages * sizeof(int), hipHostMallocDefault));
    memset(s->host_page_table, 0, (size_t)s->n_pages * sizeof(int));
    // LIFO free list: the first logical page gets the highest physical page, so
    // the mapping is never the identity
    for (int p = s->n_pages - 1; p >= 0; --p) s->free_pages.push_back(p);  // handed out in ascending order
    s->pages_used = 0;

    // RoPE table in double: angle = pos * base^(-2j/hd)
    S_TRY(dev_alloc(s->allocs, &s->rope, (size_t)max_ctx * (c.head_dim / 2), false));
    hipLaunchKernelGGL(rope_table_kernel, dim3(max_ctx), dim3(c.head_dim / 2), 0, 0, s->rope, (double)c.rope_base, c.head_dim);
    S_HIP(hipGetLastError());

    {
        // prefill: a chunk of up to pf_cap rows at once (pf_gemm_kernel and friends).  Per row 18 d + 4 F bytes and the
        // partial tiles: for 2048 positions 290 MB with the 7B shape (a seventh of the cache of its 32 layers), 15 MB
        // with 4 layers of 256 (nine tenths).  Padding columns (K not a multiple of 32) are read and
        // must stay zero; the buffers need no clearing otherwise.
        const ModelDev &pm = m->host_md;
        s->pf_cap = std::min(PF_ROWS, (int)align_up((size_t)max_ctx, 16));
        const size_t cap = (size_t)s->pf_cap, pf_rows = std::max<size_t>(cap, (size_t)rows_max);
        const bool pad = pm.Kpad_d != pm.d || pm.Kpad_F != pm.F;
        // One allocation for all of them (a dozen separate ones made creating a session 5 ms longer).
        const size_t slots = 2 * (((size_t)pm.d + 63) / 64);   // two per workgroup tile of the narrowest shape
        const size_t part = s->pf_part_cap = pf_part_floats(m, s->pf_cap, 0);
        size_t bytes = 0;
        auto place = [&](size_t n) {
            const size_t at = bytes;
            bytes += align_up(n, 256);
            return at;
        };
        const size_t at_xn = place(4 * cap * pm.Kpad_d), at_attn = place(4 * cap * pm.Kpad_d), at_u = place(4 * cap * pm.Kpad_F), padded = bytes;
        const size_t at_h = place(4 * cap * d), at_q = place(4 * cap * d), at_s0 = place(4 * slots * cap), at_s1 = place(4 * slots * cap);
        const size_t at_part = place(4 * part), at_tok = place(4 * pf_rows), at_emb = place(2 * pf_rows * d);
        unsigned char *base = nullptr;
        S_TRY(dev_alloc(s->allocs, &base, bytes, false));
        if (pad) S_HIP(hipMemset(base, 0, padded));
        PfScratch &b = s->pf;
        b.rt = s->pf_cap / 16;
        b.xn = reinterpret_cast<uint16_t *>(base + at_xn);
        b.attn = reinterpret_cast<uint16_t *>(base + at_attn);
        b.u = reinterpret_cast<uint16_t *>(base + at_u);
        b.h = reinterpret_cast<float *>(base + at_h);
        b.q = reinterpret_cast<float *>(base + at_q);
        s->pf_ss[0] = reinterpret_cast<float *>(base + at_s0);
        s->pf_ss[1] = reinterpret_cast<float *>(base + at_s1);
        s->pf_part = reinterpret_cast<float *>(base + at_part);
        s->dev_pf_tokens = reinterpret_cast<int *>(base + at_tok);
        s->dev_pf_emb = reinterpret_cast<uint16_t *>(base + at_emb);
        S_TRY(dev_alloc(s->allocs, &s->pf_part_count, (size_t)PF_PART_TILES));
        S_HIP(hipHostMalloc(reinterpret_cast<void **>(&s->host_pf_tokens), pf_rows * sizeof(int), hipHostMallocDefault));
    }
    S_HIP(hipHostMalloc(reinterpret_cast<void **>(&s->result), sizeof(ee_verify_result), hipHostMallocMapped));
    memset(s->result, 0, sizeof(ee_verify_result));
    S_HIP(hipHostGetDevicePointer(reinterpret_cast<void **>(&s->dev_result), s->result, 0));
    S_TRY(dev_alloc(s->allocs, &s->dev_sessdev, EE_MAX_BATCH));
    S_HIP(hipHostMalloc(reinterpret_cast<void **>(&s->host_sessdev), EE_MAX_BATCH * sizeof(SessDev), hipHostMallocDefault));

    Scratch &sc = s->sc;
    const ModelDev &md = m->host_md;
    S_TRY(dev_alloc(s->allocs, &sc.h, (size_t)rows_max * d));
    S_TRY(dev_alloc(s->allocs, &sc.q, (size_t)rows_max * d));
    S_TRY(dev_alloc(s->allocs, &sc.xn, (size_t)2 * rows_max * md.Kpad_d + X_SLACK));
    S_TRY(dev_alloc(s->allocs, &sc.xh, (size_t)2 * rows_max * md.Kpad_d + X_SLACK));
    S_TRY(dev_alloc(s->allocs, &sc.attn, (size_t)2 * rows_max * md.Kpad_d + X_SLACK));
    S_TRY(dev_alloc(s->allocs, &sc.u, (size_t)2 * rows_max * md.Kpad_F + X_SLACK));
    S_TRY(dev_alloc(s->allocs, &sc.xa, (size_t)2 * rows_max * md.Kpad_d + X_SLACK));
    S_TRY(dev_alloc(s->allocs, &sc.t, (size_t)2 * rows_max * std::max(md.Kpad_A, 32) + X_SLACK));
    if (md.A) S_TRY(dev_alloc(s->allocs, &sc.ha, (size_t)rows_max * d));
    S_TRY(dev_alloc(s->allocs, &sc.ss_h, (size_t)SS_LD * rows_max));
    S_TRY(dev_alloc(s->allocs, &sc.ss_a, (size_t)SS_LD * rows_max));
    S_TRY(dev_alloc(s->allocs, &sc.ss_f, (size_t)SS_LD * rows_max));
    {
        // items = units * splits; splits are chosen per pass and clamped to this room.  Units: a
        // batch of sessions with one chunk of rows each, or one session with the rows of a prefill chunk.
        const size_t max_units = (size_t)c.n_heads * std::max<size_t>(EE_MAX_BATCH, (rows_max + ATT_ROWS - 1) / ATT_ROWS);
        const size_t forced = ((size_t)s->n_pages + ATT_TILES * WAVES - 1) / (ATT_TILES * WAVES);
        const size_t max_items = max_units * std::max<size_t>(forced, 2) + (size_t)m->nwg;
        s->att_items_cap = (int)max_items;
        S_TRY(dev_alloc(s->allocs, &sc.att_part, max_items * att_item(c.head_dim)));
        S_TRY(dev_alloc(s->allocs, &sc.att_count, max_units));
        S_TRY(dev_alloc(s->allocs, &sc.head_count, 1));
    }
    if (flags & (EE_KEEP_LOGITS | EE_SAMPLING))
        S_TRY(dev_alloc(s->allocs, &sc.logits, (size_t)(EE_MAX_EXITS + 1) * rows_max * c.vocab));
    if (flags & EE_SAMPLING) {
        // room for the draft distributions of every row a pass led by this session can carry
        const size_t n = (size_t)rows_max * c.vocab + (size_t)EE_MAX_BATCH * (2 * EE_MAX_M + 2);
        S_HIP(hipHostMalloc(reinterpret_cast<void **>(&s->host_sample), n * sizeof(float), hipHostMallocDefault));
        S_TRY(dev_alloc(s->allocs, &s->dev_sample, n));
        S_HIP(hipStreamCreate(&s->copy_stream));
        S_HIP(hipEventCreateWithFlags(&s->ev_copy, hipEventDisableTiming));
        S_TRY(dev_alloc(s->allocs, &s->dev_sample_out, 3 * EE_MAX_ROWS + 1));
        S_TRY(dev_alloc(s->allocs, &s->dev_sample_sums, (size_t)2 * rows_max * sample_parts(c.vocab)));
    }
    {
        // partial tiles of the K-split launches: [split][n-tile][row][16] floats for the largest split kind
        size_t part = 0;
        for (int k = 0; k < G_KINDS; ++k)
            if (m->plan[1][k].nwg > 0) part = std::max(part, ((size_t)m->plan[1][k].NT << m->plan[1][k].ksl) * rows_max * 16);
        if (part) {
            S_TRY(dev_alloc(s->allocs, &sc.part, part));
            S_TRY(dev_alloc(s->allocs, &sc.part_count, (size_t)m->nwg));
        }
    }
    S_TRY(dev_alloc(s->allocs, &sc.cand, (size_t)SS_LD * rows_max));
    S_TRY(dev_alloc(s->allocs, &sc.cand_sum, (size_t)SS_LD * rows_max));
    S_HIP(hipDeviceSynchronize());
#undef S_TRY
#undef S_HIP
    *out = s;
    return EE_OK;
}

// map logical pages so that positions [0, upto) are backed; upload new entries
static int ensure_pages(ee_session *s, int upto, hipStream_t stream)
{
    int need = (upto + KV_PAGE - 1) / KV_PAGE;
    if (need > s->n_pages) return fail(EE_ECAPACITY, "KV cache: %d positions exceed max_ctx %d", upto, s->max_ctx);
    int first_new = s->pages_used;
    while (s->pages_used < need) {
        if (s->free_pages.empty()) return fail(EE_ECAPACITY, "KV cache: out of pages");
        s->host_page_table[s->pages_used++] = s->free_pages.back();
        s->free_pages.pop_back();
    }
    if (s->pages_used > first_new)
        HIP_TRY(hipMemcpyAsync(s->dev_page_table + first_new, s->host_page_table + first_new,
                               (size_t)(s->pages_used - first_new) * sizeof(int), hipMemcpyHostToDevice, stream));
    return EE_OK;
}

static void release_pages(ee_session *s, int keep_positions)
{
    int keep = (keep_positions + KV_PAGE - 1) / KV_PAGE;
    while (s->pages_used > keep) s->free_pages.push_back(s->host_page_table[--s->pages_used]);
}

static void fill_sessdev(SessDev &sd, const ee_session *s)
{
    sd.page_table = s->dev_page_table;
    sd.kpool = s->kpool;
    sd.vpool = s->vpool;
    sd.rope = s->rope;
    sd.result = s->dev_result;
    sd.n_pages = s->n_pages;
    sd.kv_len = s->kv_len;
    sd.pending = s->pending;
    // the common case: the session's pages are consecutive (a fresh pool hands them out in
    // ascending order and a rollback returns them in the order that restores it)
    sd.contig_base = s->pages_used > 0 ? s->host_page_table[0] : 0;
    for (int i = 1; i < s->pages_used; ++i)
        if (s->host_page_table[i] != s->host_page_table[0] + i) {
            sd.contig_base = -1;
            break;
        }
}

// host mirror of the kernels' stage list: [EMBED] { QKV ATT O GU DN } x layers [AD AU] [HEAD];
// returns the stage's EE_LAUNCH_* code (for a GEMM stage: its GemmKind), or -1 past the end
static int launch_code(const PassArgs &a, int ph)
{
    const int per_layer = 5;
    int idx = ph - (a.do_embed ? 1 : 0);
    if (idx < 0) return EE_LAUNCH_EMBED;
    const int nl = a.layer_end - a.layer_begin;
    if (idx < per_layer * nl) {
        const int r = idx % per_layer;
        if (r == 0) return EE_LAUNCH_QKV;
        if (r == 1) return EE_LAUNCH_ATT;
        return EE_LAUNCH_O + (r - 2);
    }
    idx -= per_layer * nl;
    if (a.head_kind != HEAD_NONE) {
        const int n_ad = a.adapter && (!a.ha || a.head_stage) ? 2 : 0;   // (adapters of several exits: with the last of them)
        if (idx < n_ad) return EE_LAUNCH_ADAPTER_DOWN + idx;
        if (idx == n_ad && a.head_stage) return EE_LAUNCH_HEAD;
    }
    return -1;
}

// Draft distributions and numbers of a sampled pass that are not on their way to the device yet.
struct SampleUpload {
    const ee_sampling *sp;   // [n_sessions], null once uploaded
    int n_sessions, gamma;
};

// [session][gamma][V] distributions, then per session u, v and 1 / temperature (SampleDev).  The copy runs on a
// stream of its own and the pass's stream waits for it: called when the launches before the first sampling
// launch have been enqueued, the staging (512 KB for four drafts of 32000 tokens) and the transfer
// take place while the layers run.
static int upload_sampling(ee_session *lead, SampleUpload &up)
{
    const size_t V = (size_t)lead->m->cfg.vocab, np = (size_t)up.n_sessions * up.gamma * V, blk = 2 * (size_t)up.gamma + 2;
    for (int b = 0; b < up.n_sessions; ++b) {
        const ee_sampling &q = up.sp[b];
        memcpy(lead->host_sample + (size_t)b * up.gamma * V, q.draft_probs, (size_t)up.gamma * V * sizeof(float));
        float *uv = lead->host_sample + np + (size_t)b * blk;
        memcpy(uv, q.u, (size_t)up.gamma * sizeof(float));
        memcpy(uv + up.gamma, q.v, (size_t)(up.gamma + 1) * sizeof(float));
        uv[2 * up.gamma + 1] = 1.0f / q.temperature;
    }
    HIP_TRY(hipMemcpyAsync(lead->dev_sample, lead->host_sample, (np + (size_t)up.n_sessions * blk) * sizeof(float), hipMemcpyHostToDevice, lead->copy_stream));
    HIP_TRY(hipEventRecord(lead->ev_copy, lead->copy_stream));
    HIP_TRY(hipStreamWaitEvent(lead->run_stream, lead->ev_copy, 0));
    up.sp = nullptr;
    return EE_OK;
}

static const uint16_t *gemm_input_of(const Scratch &sc, int kind)
{
    switch (kind) {
    case G_O: return sc.attn;
    case G_DN: return sc.u;
    case G_AD: return sc.xa;
    case G_AU: return sc.t;
    case G_HEAD: return sc.xh;
    default: return sc.xn;
    }
}

// Whether a launch of so many rows streams the packed form of a matrix that has one.  Up to 16 rows, with K split and in the LM head always.  Beyond,
// unpacking and the escapes' sums cost every n-tile a time that grows with the rows, and the bytes saved are K's: both forms meet at K = 64 a
// row, whatever the columns.  us plain / packed at 32, 39 and 48 rows: gate/up of 4 n-tiles a unit, K 2048 16.6 / 17.0, 17.8 / 19.2, 19.1 / 21.7; 2304 19.1 / 18.6,
// 20.4 / 20.6, 21.7 / 23.6; 2560 20.4 / 19.3, 21.8 / 21.3, 23.1 / 24.5; 3072 23.1 / 21.6, 24.7 / 23.3, 26.5 / 26.2; QKV, K 2560 15.8 / 15.8, 17.3 / 17.6,
// 18.4 / 19.2; 3072 20.2 / 18.9, 21.8 / 20.8, 23.1 / 22.7; 4096 25.5 / 23.4, 27.9 / 25.9, 29.6 / 28.1.
static bool packed_pays(int kind, const GemmPlan &p, int rows) { return rows <= 16 || p.ksl > 0 || kind == G_HEAD || p.K >= 64 * rows; }

// Enqueues the stages of one segment, one launch each, on the leader's stream.
// `many`: the adapters of the group's n_heads exits in one launch each, from stored exit adapter_slot on, `adapter_step` apart.
static int launch_segment(ee_session *lead, PassArgs &a, int adapter_slot, SampleUpload *up = nullptr, bool many = false, int adapter_step = 0)
{
    const ee_model *m = lead->m;
    const int per_layer = 5;
    const int rows = a.rows;
    for (int ph = 0;; ++ph) {
        const int code = launch_code(a, ph);
        if (code < 0) break;
        const bool gemm = code != EE_LAUNCH_EMBED && code != EE_LAUNCH_ATT;
        const int idx = ph - (a.do_embed ? 1 : 0);
        a.layer = a.layer_begin + std::max(idx, 0) / per_layer;
        // what the O, DN, AD and AU epilogues produce and read (gemm_epi)
        a.gain_xn = a.gain_xh = a.bias = nullptr;
        a.xa_out = 0;
        const bool adapter_stage = code == EE_LAUNCH_ADAPTER_DOWN || code == EE_LAUNCH_ADAPTER_UP;
        const int head_row0 = a.head_row0;
        if (adapter_stage && many) a.head_row0 = 0;   // (this launch writes the head rows of all exits of the group)
        if (code == EE_LAUNCH_O) a.gain_xn = a.mdv.g_ffn + (size_t)a.layer * a.d;
        if (code == EE_LAUNCH_DN) {
            if (a.layer + 1 < m->cfg.n_layers) a.gain_xn = a.mdv.g_attn + (size_t)(a.layer + 1) * a.d;
            if (a.layer + 1 == a.layer_end && a.head_kind != HEAD_NONE) {
                a.xa_out = a.adapter;
                if (!a.adapter) a.gain_xh = a.head_gain;
            }
        }
        if (code == EE_LAUNCH_ADAPTER_DOWN) a.bias = a.ad_bdown;
        if (code == EE_LAUNCH_ADAPTER_UP) {
            a.bias = a.ad_bup;
            a.gain_xh = a.ad_gain;
        }
        a.fuse_accept = (code == EE_LAUNCH_HEAD && !a.sm.on) ? 1 : 0;
        a.rows = code == EE_LAUNCH_HEAD ? a.head_rows : rows;   // the head launch carries the rows of all exits of its group
        pass_kernel_t k = code == EE_LAUNCH_ATT ? att_kernel(m->cfg.head_dim) : ee_misc_kernel;
        if (gemm) {  // the stage's plan, LDS map and weights travel with the launch
            static_assert(EE_LAUNCH_QKV == G_QKV && EE_LAUNCH_HEAD == G_HEAD && EE_LAUNCH_ADAPTER_DOWN == G_AD && EE_LAUNCH_ADAPTER_UP == G_AU,
                          "launch codes of GEMM stages are their GemmKind");
            const int slice = code == EE_LAUNCH_HEAD ? 0 : (code >= EE_LAUNCH_ADAPTER_DOWN ? adapter_slot : a.layer);
            // more than 16 rows: the K-split variant of the kind, where the model has one and the scratch its buffers
            const int v = (a.rows > 16 && m->plan[1][code].nwg > 0 && a.sc.part) ? 1 : 0;
            a.plan0 = m->plan[v][code];
            GemmEntry &en = a.entry;
            const bool packed = (size_t)slice < m->packed[v][code].size() && m->packed[v][code][slice].w && packed_pays(code, a.plan0, a.rows);
            k = gemm_kernel(code, a.rows, packed);
            if (packed) {
                const ee_model::PackedSlice &ps = m->packed[v][code][slice];
                en.W = reinterpret_cast<const uint4 *>(ps.w);
                en.esc = m->escapes + ps.esc;
                en.esc_groups = (uint16_t)ps.groups;
                en.esc_cap = (uint16_t)ps.cap;
                en.wscale = ps.scale;
            } else {
                en.W = m->w[v][code] + (size_t)slice * m->wstride[v][code];
            }
            en.X = gemm_input_of(a.sc, code);
            if (adapter_stage) {
                const int K = code == EE_LAUNCH_ADAPTER_DOWN ? a.mdv.Kpad_d : a.mdv.Kpad_A;
                if (code == EE_LAUNCH_ADAPTER_DOWN && many) en.X = lead->sc.xa;   // (a.sc.xa is the last exit's)
                en.w_next = (long long)m->wstride[v][code] * 16 * adapter_step;
                en.x_next = 4 * a.rows * K;
                a.t_next = 2 * a.rows * a.mdv.Kpad_A;
                a.bias_next = adapter_step * (code == EE_LAUNCH_ADAPTER_DOWN ? a.mdv.A : a.d);
                a.gain_next = adapter_step * a.d;
            }
            en.wstep = a.plan0.nwg * SWAVES * tile_bytes_of(packed);
            en.tile_bytes = a.rows * 128;
            en.KTs = a.plan0.KTs;
            en.nwg = a.plan0.nwg;
            en.base = a.plan0.base;
            en.rem = a.plan0.rem;
            en.tpu = a.plan0.tpu;
            en.ksl = a.plan0.ksl;
            if (!plan_lds(a.plan0, a.rows, m->lds_budget, packed, a.lay)) return fail(EE_EDEVICE, "no LDS layout for %d rows", a.rows);
        }
        const bool timed = (lead->flags & EE_TIME_LAUNCHES) && a.mode == 0;
        if (timed) {
            const size_t i = lead->lt_codes.size();
            while (lead->lt_events.size() < 2 * (i + 1)) {
                hipEvent_t ev;
                HIP_TRY(hipEventCreate(&ev));
                lead->lt_events.push_back(ev);
            }
            lead->lt_codes.push_back(code);
            HIP_TRY(hipEventRecord(lead->lt_events[2 * i], lead->run_stream));
        }
        if (code == EE_LAUNCH_ATT)
            hipLaunchKernelGGL(k, a.att_starts ? dim3(a.H, 63 - __builtin_clzll(a.att_starts)) : dim3(a.att_splits, a.H, a.mode == 1 ? (a.M + ATT_ROWS - 1) / ATT_ROWS : a.n_sess),
                               dim3(WG_THREADS), att_lds(m->cfg.head_dim, a.M), lead->run_stream, a);
        else
            hipLaunchKernelGGL(k, dim3(m->nwg, adapter_stage && many ? a.n_heads : 1), dim3(WG_THREADS), m->lds_budget, lead->run_stream, a);
        HIP_TRY(hipGetLastError());
        a.head_row0 = head_row0;
        if (timed) HIP_TRY(hipEventRecord(lead->lt_events[2 * lead->lt_codes.size() - 1], lead->run_stream));
        if (code == EE_LAUNCH_HEAD && a.sm.on) {
            // probabilistic verification: the rows' keep tests and draws, workgroups of SAMPLE_PART tokens of a head row,
            // then the accept rule and the publication (in the workgroup that finishes last)
            if (up && up->sp) {
                const int rc = upload_sampling(lead, *up);
                if (rc != EE_OK) return rc;
            }
            if (timed) {
                const size_t i = lead->lt_codes.size();
                while (lead->lt_events.size() < 2 * (i + 1)) {
                    hipEvent_t ev;
                    HIP_TRY(hipEventCreate(&ev));
                    lead->lt_events.push_back(ev);
                }
                lead->lt_codes.push_back(EE_LAUNCH_SAMPLE);
                HIP_TRY(hipEventRecord(lead->lt_events[2 * i], lead->run_stream));
            }
            const dim3 grid(sample_parts(m->cfg.vocab), a.head_rows);
            hipLaunchKernelGGL(ee_sample_sum_kernel, grid, dim3(SAMPLE_WAVES * 64), SAMPLE_LDS_BYTES, lead->run_stream, a);
            HIP_TRY(hipGetLastError());
            hipLaunchKernelGGL(ee_sample_kernel, grid, dim3(SAMPLE_WAVES * 64), SAMPLE_LDS_BYTES, lead->run_stream, a);
            HIP_TRY(hipGetLastError());
            if (timed) HIP_TRY(hipEventRecord(lead->lt_events[2 * lead->lt_codes.size() - 1], lead->run_stream));
        }
    }
    a.rows = rows;
    return EE_OK;
}

static void base_args(const ee_session *lead, PassArgs &a)
{
    memset(&a, 0, sizeof a);
    a.mdv = lead->m->host_md;
    a.sc = lead->sc;
    a.nwg = lead->m->nwg;
    a.H = lead->m->host_md.H;
    a.d = lead->m->host_md.d;
    a.Kpad_d = lead->m->host_md.Kpad_d;
    a.att_scale = lead->m->host_md.att_scale;
    a.keep_logits = (lead->flags & EE_KEEP_LOGITS) ? 1 : 0;
}

static int finish_flight(ee_session *s)
{
    if (!s->in_flight) return EE_OK;
    ee_session *lead = s->leader;
    HIP_TRY(hipEventSynchronize(lead->ev_final));
    s->in_flight = false;
    if (s->result->device_status != 0) return fail(EE_EDEVICE, "a device-side wait gave up during the pass; results are invalid");
    if (!(s->flags & EE_NO_AUTOCOMMIT)) {
        s->kv_len += s->result->accept_len + 1;
        s->pending = s->result->next_token;
    }
    return EE_OK;
}

// ------------------------------------------------------------------ prefill

// All layers of one prefill chunk of many rows; the chunk's tokens and embedding rows are on the device.
static int prefill_chunk(ee_session *s, int start, int rows)
{
    const ee_model *m = s->m;
    const ee_model_config &c = m->cfg;
    const ModelDev &md = m->host_md;
    const SessDev &sd = s->host_sessdev[0];
    PfArgs a;
    memset(&a, 0, sizeof a);
    a.b = s->pf;
    a.rows = rows;
    a.pos0 = start;
    a.d = md.d;
    a.F = md.F;
    a.H = md.H;
    a.hd = md.hd;
    a.eps = md.eps;
    a.att_scale = md.att_scale;
    a.kpool = sd.kpool;
    a.vpool = sd.vpool;
    a.rope = sd.rope;
    a.page_table = sd.page_table;
    a.contig_base = sd.contig_base;
    a.n_pages = sd.n_pages;
    a.tokens = s->dev_pf_tokens;
    a.emb_rows = s->dev_pf_emb;
    a.emb = md.emb;
    a.part = s->pf_part;
    a.part_count = s->pf_part_count;
    a.gain = md.g_attn;
    a.ss_out = s->pf_ss[0];
    hipLaunchKernelGGL(pf_embed_kernel, dim3(rows), dim3(PF_THREADS), 0, s->stream, a);
    HIP_TRY(hipGetLastError());
    int slots = 1;                                          // partial sums per row in pf_ss[0]
    auto gemm = [&](int kind, int layer) {
        const GemmPlan &pl = m->plan[0][kind];
        const PfChoice ch = pf_choose(m, pl, rows, s->pf_gemm_opt);
        const PfShape &sh = *ch.shape;
        a.W = m->w[0][kind] + (size_t)layer * m->wstride[0][kind];
        a.tab = m->tile_tab[kind];
        a.NT = pl.NT;
        a.KT = pl.KT;
        a.N = pl.N;
        a.nb = ch.nb;
        a.mb = ch.mb;
        a.ks = ch.ks;
        hipLaunchKernelGGL(sh.gemm[kind], dim3(a.nb * a.mb * a.ks), dim3(PF_THREADS * sh.grp), pf_gemm_lds(sh.wn, sh.wm, sh.grp), s->stream, a);
    };
    for (int l = 0; l < c.n_layers; ++l) {
        a.layer = l;
        a.ss_in = s->pf_ss[0];
        a.ss_slots = slots;
        gemm(G_QKV, l);
        const int rt = s->pf_att_opt ? s->pf_att_opt / 64 : (md.H * ((rows + 127) / 128) > m->nwg ? 2 : 1);
        hipLaunchKernelGGL(pf_att(md.hd, rt), dim3(md.H * ((rows + 64 * rt - 1) / (64 * rt))), dim3(PF_ATT_THREADS),
                           pf_att_lds(md.hd, s->pages_used), s->stream, a);
        a.gain = md.g_ffn + (size_t)l * md.d;
        a.ss_out = s->pf_ss[1];
        gemm(G_O, l);
        a.ss_in = s->pf_ss[1];
        a.ss_slots = 2 * a.nb;
        gemm(G_GU, l);
        a.gain = l + 1 < c.n_layers ? md.g_attn + (size_t)(l + 1) * md.d : nullptr;
        a.ss_out = s->pf_ss[0];
        gemm(G_DN, l);
        slots = 2 * a.nb;
        HIP_TRY(hipGetLastError());
    }
    return EE_OK;
}

extern "C" int ee_prefill_embeds(ee_session *s, const uint16_t *emb_bf16, int n_emb, const int32_t *tokens, int n,
                                 unsigned flags, int32_t *first_token)
{
    if (!s) return fail(EE_EINVAL, "ee_prefill: null session");
    if (n_emb < 0 || n < 0 || (n_emb > 0 && !emb_bf16) || (n > 0 && !tokens)) return fail(EE_EINVAL, "ee_prefill: bad arguments");
    const ee_model *m = s->m;
    const ee_model_config &c = m->cfg;
    for (int i = 0; i < n; ++i)
        if (tokens[i] < 0 || tokens[i] >= c.vocab) return fail(EE_EINVAL, "ee_prefill: token %d at %d outside [0,%d)", tokens[i], i, c.vocab);
    const bool hold = (flags & EE_HOLD_LAST) != 0;
    if (hold && n < 1) return fail(EE_EINVAL, "ee_prefill: EE_HOLD_LAST needs at least one token");
    const int total = n_emb + n - (hold ? 1 : 0);
    if (!hold && total < 1) return fail(EE_EINVAL, "ee_prefill: empty prompt");
    if (total + 1 > s->max_ctx) return fail(EE_ECAPACITY, "ee_prefill: %d rows do not fit max_ctx %d", total, s->max_ctx);
    HIP_TRY(hipSetDevice(m->device));
    int rc = finish_flight(s);
    if (rc != EE_OK && rc != EE_EDEVICE) return rc;
    HIP_TRY(hipStreamSynchronize(s->stream));
    // reset
    s->run_stream = s->stream;
    release_pages(s, 0);
    // all pages are free here: hand them out in ascending order (a fresh session's pages are then
    // consecutive and the kernels skip the table lookup) or, as a test aid, in descending order
    std::sort(s->free_pages.begin(), s->free_pages.end());
    if (!s->scatter_pages) std::reverse(s->free_pages.begin(), s->free_pages.end());
    s->kv_len = 0;
    s->has_pending = false;
    s->leader = s;
    s->flight_gamma = 0;
    s->flight_exits = 0;
    s->result->device_status = 0;
    if ((rc = ensure_pages(s, total + 1, s->stream)) != EE_OK) return rc;

    fill_sessdev(s->host_sessdev[0], s);
    // More rows than a pass of this model carries: the many-row kernels, in chunks of nearly equal size.  us with
    // them / in streamed chunks of 16 rows: 7B shape, 4 layers, 24 rows 646 / 816, 48 rows 673 / 1238; 1280-wide model, 3
    // layers, 24 rows 204 / 233.  (A streamed pass of 48 rows takes 600: models loaded for that many keep it.)
    const bool many = total > c.max_rows;
    const int n_chunks = (total + s->pf_cap - 1) / s->pf_cap;
    const int chunk = many ? std::min(s->pf_cap, (int)align_up((size_t)((total + n_chunks - 1) / n_chunks), 128)) : total;
    const size_t d = (size_t)c.d_model;
    for (int start = 0; start < total; start += chunk) {
        const int rows = std::min(chunk, total - start);
        if (start > 0) HIP_TRY(hipStreamSynchronize(s->stream));  // the chunk before has read the staging buffers
        for (int i = 0; i < rows; ++i) {
            int r = start + i;
            s->host_pf_tokens[i] = r < n_emb ? -1 : tokens[r - n_emb];
        }
        HIP_TRY(hipMemcpyAsync(s->dev_pf_tokens, s->host_pf_tokens, (size_t)rows * sizeof(int), hipMemcpyHostToDevice, s->stream));
        if (start < n_emb) {
            int ne = std::min(rows, n_emb - start);
            HIP_TRY(hipMemcpyAsync(s->dev_pf_emb, emb_bf16 + (size_t)start * d, (size_t)ne * d * 2, hipMemcpyHostToDevice, s->stream));
        }
        const bool last = (start + rows == total) && !hold;
        PassArgs a;
        base_args(s, a);
        a.n_sess = 1;
        a.M = many ? 1 : rows;   // many rows: the head launch sees the last one only
        a.rows = a.M;
        a.mode = 1;
        a.pf_tokens = s->dev_pf_tokens;
        a.pf_emb = s->dev_pf_emb;
        a.pf_pos0 = 0;
        a.layer_begin = 0;
        a.layer_end = c.n_layers;
        a.do_embed = 1;
        a.head_kind = last ? HEAD_PREFILL : HEAD_NONE;
        a.head_idx = 0;
        a.head_gain = m->host_md.g_final;
        a.n_heads = 1;
        a.head_rows = a.rows;
        a.head_row0 = 0;
        a.head_stage = 1;
        a.sess = s->dev_sessdev;
        a.sess0 = s->host_sessdev[0];
        if (!many) {
            a.att_splits = attention_splits(s, s->att_items_cap, 1, rows, rows);
            if (a.att_splits == 0) return fail(EE_ECAPACITY, "ee_prefill: context too long for the session's attention scratch");
        } else {
            if ((rc = prefill_chunk(s, start, rows)) != EE_OK) return rc;
            if (!last) continue;
            PfArgs p;
            memset(&p, 0, sizeof p);
            p.b = s->pf;
            p.rows = rows;
            p.d = c.d_model;
            p.gain = m->host_md.g_final;
            hipLaunchKernelGGL(pf_last_kernel, dim3(1), dim3(PF_THREADS), 0, s->stream, p, s->sc.xh, s->sc.ss_h);
            HIP_TRY(hipGetLastError());
            a.layer_begin = c.n_layers;
            a.do_embed = 0;
        }
        if ((rc = launch_segment(s, a, 0)) != EE_OK) return rc;
    }
    HIP_TRY(hipStreamSynchronize(s->stream));
    s->kv_len = total;
    if (hold) {
        s->pending = tokens[n - 1];
    } else {
        if (s->result->device_status != 0) return fail(EE_EDEVICE, "a device-side wait gave up during prefill");
        s->pending = s->result->next_token;
        if (first_token) *first_token = s->pending;
    }
    s->has_pending = true;
    return EE_OK;   // (kv_len and pending travel with every launch's arguments: nothing is enqueued behind the wait above)
}

extern "C" int ee_prefill(ee_session *s, const int32_t *tokens, int n, unsigned flags, int32_t *first_token)
{
    return ee_prefill_embeds(s, nullptr, 0, tokens, n, flags, first_token);
}

// ------------------------------------------------------------------ verify

static int check_exits(const ee_model *m, const int32_t *exit_layers, int n_exits, const float **gains, int *slots)
{
    if (n_exits < 0 || n_exits > EE_MAX_EXITS || (n_exits > 0 && !exit_layers))
        return fail(EE_EINVAL, "ee_verify: n_exits %d not in [0,%d]", n_exits, EE_MAX_EXITS);
    for (int e = 0; e < n_exits; ++e) {
        if (exit_layers[e] < 1 || exit_layers[e] > m->cfg.n_layers - 1)
            return fail(EE_EINVAL, "ee_verify: exit layer %d not in [1,%d]", exit_layers[e], m->cfg.n_layers - 1);
        if (e > 0 && exit_layers[e] <= exit_layers[e - 1]) return fail(EE_EINVAL, "ee_verify: exit layers must increase strictly");
        gains[e] = nullptr;
        for (int i = 0; i < m->cfg.n_exits; ++i)
            if (m->cfg.exit_layers[i] == exit_layers[e]) {
                gains[e] = m->g_exit[i];
                slots[e] = i;
            }
        if (!gains[e]) return fail(EE_EINVAL, "ee_verify: the model stores no exit gain for layer %d", exit_layers[e]);
    }
    return EE_OK;
}

// ------------------------------------------------------------------ static scratch (ee_verify_static)

// Scratch of one single-session pass for callers that must not allocate.  One copy per GPU the
// library is loaded on, held until the process ends.  In host code the array's name is only a
// handle: its device address comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) unsigned char scratch[EE_STATIC_SCRATCH_BYTES];

constexpr int EE_MAX_DEVICES = 64;
static void *g_scratch_ptr[EE_MAX_DEVICES];   // per device: address of that GPU's copy of `scratch`

static int static_scratch_ptr(int device, unsigned char **out)
{
    if (device < 0 || device >= EE_MAX_DEVICES) return fail(EE_EINVAL, "device %d: at most %d devices", device, EE_MAX_DEVICES);
    if (!g_scratch_ptr[device]) {   // the model's device is current here
        void *p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        g_scratch_ptr[device] = p;
    }
    *out = static_cast<unsigned char *>(g_scratch_ptr[device]);
    return EE_OK;
}

// fills n 16-byte words with zeros (a kernel, not hipMemsetAsync: callers may be capturing a graph)
__global__ void __launch_bounds__(256) ee_zero_kernel(uint4 *p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// Lays the pass's scratch buffers out in the static array (sizes for M rows of this model),
// points a.sc at them, picks the attention splits for that room and enqueues the clearing of
// the part in use: the array keeps the last call's contents, and the padding columns of the GEMM
// inputs and the attention / head counters must start at zero.  per_group (exits whose heads share a launch
// of the LM head, EE_OPT_HEAD_BATCH) comes in as what the session asks for and goes out as what fits: the
// LM head's input holds the rows of a whole group.  It is lowered rather than the call refused, or
// the attention given fewer splits: results do not depend on it, only when the exits are published.
static int use_static_scratch(ee_session *lead, PassArgs &a, int M, int n_pos_max, int &per_group)
{
    const ee_model *m = lead->m;
    const ModelDev &md = m->host_md;
    unsigned char *base = nullptr;
    int rc = static_scratch_ptr(m->device, &base);
    if (rc != EE_OK) return rc;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        unsigned char *p = base + off;
        off += align_up(std::max<size_t>(bytes, 16), 256);
        return p;
    };
    const size_t rows = (size_t)M, d = (size_t)md.d;
    Scratch sc;
    memset(&sc, 0, sizeof sc);
    auto lay_out = [&](size_t head_rows) {   // everything but the attention partials; behind every GEMM input lie X_SLACK elements of the next buffers
        off = 0;
        sc.h = reinterpret_cast<float *>(take(rows * d * 4));
        sc.q = reinterpret_cast<float *>(take(rows * d * 4));
        sc.xn = reinterpret_cast<uint16_t *>(take(2 * rows * md.Kpad_d * 2));
        sc.xh = reinterpret_cast<uint16_t *>(take(2 * head_rows * md.Kpad_d * 2));
        sc.attn = reinterpret_cast<uint16_t *>(take(2 * rows * md.Kpad_d * 2));
        sc.u = reinterpret_cast<uint16_t *>(take(2 * rows * md.Kpad_F * 2));
        sc.xa = reinterpret_cast<uint16_t *>(take(2 * rows * md.Kpad_d * 2));
        sc.t = reinterpret_cast<uint16_t *>(take(2 * rows * std::max(md.Kpad_A, 32) * 2));
        sc.ss_h = reinterpret_cast<float *>(take((size_t)SS_LD * md.rows_max * 4));
        sc.ss_a = reinterpret_cast<float *>(take((size_t)SS_LD * md.rows_max * 4));
        sc.ss_f = reinterpret_cast<float *>(take((size_t)SS_LD * md.rows_max * 4));
        sc.cand = reinterpret_cast<int2 *>(take((size_t)SS_LD * md.rows_max * 8));
        sc.cand_sum = reinterpret_cast<float *>(take((size_t)SS_LD * md.rows_max * 4));
        sc.att_count = reinterpret_cast<int *>(take((size_t)md.H * 4));
        sc.head_count = reinterpret_cast<int *>(take(4));
    };
    lay_out(rows);
    sc.logits = lead->sc.logits;   // kept logits are an output of the session, not scratch
    // attention partials: what is left, at most one item per compute unit and split
    const size_t item_bytes = (size_t)att_item(md.hd) * 4;
    if (off + (size_t)md.H * item_bytes > EE_STATIC_SCRATCH_BYTES)
        return fail(EE_ECAPACITY, "ee_verify_static: %d rows of this model need more than the %d bytes of static scratch", M, EE_STATIC_SCRATCH_BYTES);
    const int items_cap = (int)std::min<size_t>((EE_STATIC_SCRATCH_BYTES - off) / item_bytes, (size_t)md.H * ATT_MAX_SPLITS);
    a.att_splits = attention_splits(lead, items_cap, 1, M, n_pos_max);
    if (a.att_splits == 0)
        return fail(EE_ECAPACITY, "ee_verify_static: a context of %d positions needs more than the %d bytes of static scratch", n_pos_max, EE_STATIC_SCRATCH_BYTES);
    const size_t part_bytes = (size_t)md.H * a.att_splits * item_bytes;
    const size_t left = EE_STATIC_SCRATCH_BYTES - off - align_up(part_bytes, 256);
    per_group = std::min<int>(per_group, 1 + (int)(left / align_up(4 * rows * md.Kpad_d, 256)));
    lay_out(per_group * rows);
    sc.att_part = reinterpret_cast<float *>(take(part_bytes));
    a.sc = sc;
    hipLaunchKernelGGL(ee_zero_kernel, dim3(256), dim3(256), 0, lead->run_stream, reinterpret_cast<uint4 *>(base), off / 16);
    HIP_TRY(hipGetLastError());
    return EE_OK;
}

// One pass for all sessions of the call: rows = n_sessions * (gamma + 1) share one stream of the
// weights; the first session leads (its stream, events and scratch carry the pass).
// static_scratch: run the pass on the library's static scratch array instead of the leader's own
// buffers (ee_verify_static); nothing on this path allocates.
static int verify_impl(ee_session *const *sessions, int n_sessions, const int32_t *const *drafts, int gamma,
                       const int32_t *exit_layers, int n_exits, const ee_verify_result **outs, bool static_scratch,
                       const ee_sampling *sp = nullptr)
{
    if (!sessions || !drafts || n_sessions < 1 || n_sessions > EE_MAX_BATCH)
        return fail(EE_EINVAL, "ee_verify: n_sessions %d not in [1,%d]", n_sessions, EE_MAX_BATCH);
    for (int i = 0; i < n_sessions; ++i)
        if (!sessions[i] || !drafts[i]) return fail(EE_EINVAL, "ee_verify: null session or drafts");
    ee_session *lead = sessions[0];
    const ee_model *m = lead->m;
    const ee_model_config &c = m->cfg;
    const int M = gamma + 1;
    if (gamma < 1) return fail(EE_EINVAL, "ee_verify: gamma %d < 1", gamma);
    for (int i = 0; i < n_sessions; ++i) {
        ee_session *s = sessions[i];
        if (s->m != m) return fail(EE_EINVAL, "ee_verify_batch: sessions of different models");
        if (gamma > s->max_gamma) return fail(EE_EINVAL, "ee_verify: gamma %d exceeds the session's max_gamma %d", gamma, s->max_gamma);
        for (int j = 0; j < i; ++j)
            if (sessions[j] == s) return fail(EE_EINVAL, "ee_verify_batch: session listed twice");
        for (int j = 0; j < gamma; ++j)
            if (drafts[i][j] < 0 || drafts[i][j] >= c.vocab)
                return fail(EE_EINVAL, "ee_verify: draft token %d outside [0,%d)", drafts[i][j], c.vocab);
        if (((s->flags ^ lead->flags) & EE_NO_AUTOCOMMIT) != 0)
            return fail(EE_EINVAL, "ee_verify_batch: sessions mix EE_NO_AUTOCOMMIT settings");
    }
    if (n_sessions * M > c.max_rows) return fail(EE_EINVAL, "ee_verify: %d rows exceed the model's max_rows %d", n_sessions * M, c.max_rows);
    if (sp) {   // sp[b]: session b's draft distributions and uniform numbers
        if (static_scratch) return fail(EE_EINVAL, "ee_verify_sampled: not with the static scratch");
        for (int b = 0; b < n_sessions; ++b) {
            const ee_sampling &q = sp[b];
            if (!(sessions[b]->flags & EE_SAMPLING)) return fail(EE_ESTATE, "ee_verify_sampled: session %d was created without EE_SAMPLING", b);
            if (!q.draft_probs || !q.u || !q.v) return fail(EE_EINVAL, "ee_verify_sampled: null draft_probs, u or v");
            if (!(q.temperature > 0.f) || !std::isfinite(q.temperature)) return fail(EE_EINVAL, "ee_verify_sampled: temperature must be positive");
            for (int i = 0; i < gamma; ++i)
                if (!(q.u[i] >= 0.f && q.u[i] < 1.f)) return fail(EE_EINVAL, "ee_verify_sampled: u[%d] not in [0,1)", i);
            for (int i = 0; i <= gamma; ++i)
                if (!(q.v[i] >= 0.f && q.v[i] < 1.f)) return fail(EE_EINVAL, "ee_verify_sampled: v[%d] not in [0,1)", i);
            for (int i = 0; i < gamma; ++i) {   // the drafts' own probabilities; the full rows are the caller's responsibility
                const float px = q.draft_probs[(size_t)i * c.vocab + drafts[b][i]];
                if (!(px >= 0.f && px <= 1.f)) return fail(EE_EINVAL, "ee_verify_sampled: draft_probs[%d][draft] = %g is not a probability", i, (double)px);
            }
        }
    }
    const float *gains[EE_MAX_EXITS];
    int slots[EE_MAX_EXITS];
    int rc = check_exits(m, exit_layers, n_exits, gains, slots);
    if (rc != EE_OK) return rc;
    HIP_TRY(hipSetDevice(m->device));
    int n_pos_max = 0;
    for (int i = 0; i < n_sessions; ++i) {
        ee_session *s = sessions[i];
        if ((rc = finish_flight(s)) != EE_OK) return rc;
        if (!s->has_pending) return fail(EE_ESTATE, "ee_verify: session has no pending token (call ee_prefill first)");
        if (s->kv_len + M > s->max_ctx) return fail(EE_ECAPACITY, "ee_verify: kv_len %d + %d rows exceed max_ctx %d", s->kv_len, M, s->max_ctx);
        n_pos_max = std::max(n_pos_max, s->kv_len + M);
    }
    PassArgs a;
    base_args(lead, a);
    lead->run_stream = lead->stream;
    // Exit heads run in groups of up to head_batch consecutive exits: every exit deposits its
    // LM-head input rows when its layer is done, and the last one of the group runs the LM head
    // over the rows of all of them (one stream of W_lm per group), after which the group's results
    // are published together.  head_batch = 1: every exit is published right after its layer.
    int per_group = std::max(1, std::min({lead->head_batch, n_exits, c.max_rows / (n_sessions * M)}));
    if (static_scratch) {
        if ((rc = use_static_scratch(lead, a, M, n_pos_max, per_group)) != EE_OK) return rc;
    } else {
        a.att_splits = attention_splits(lead, lead->att_items_cap, n_sessions, M, n_pos_max);
        if (a.att_splits == 0)
            return fail(EE_ECAPACITY, "ee_verify_batch: a context of %d positions needs more attention scratch than the first session holds "
                                      "(list the session with the largest max_ctx first)", n_pos_max);
        attention_splits_by_session(lead, lead->att_items_cap, sessions, n_sessions, M, a);
    }
    // everything below is enqueued on the leader's stream; other sessions' own
    // streams are idle here (their last pass has been waited for)
    for (int i = 0; i < n_sessions; ++i) {
        ee_session *s = sessions[i];
        if (s != lead) HIP_TRY(hipStreamSynchronize(s->stream));
        if ((rc = ensure_pages(s, s->kv_len + M, lead->run_stream)) != EE_OK) return rc;
        s->result->gamma = gamma;
        s->result->n_exits = n_exits;
        s->result->device_status = 0;
    }
    a.n_sess = n_sessions;
    a.M = M;
    a.rows = n_sessions * M;
    a.mode = 0;
    if (sp) {
        const size_t np = (size_t)n_sessions * gamma * c.vocab;
        a.sm.probs = lead->dev_sample;
        a.sm.uv = lead->dev_sample + np;
        a.sm.on = 1;
        a.sm.tok = lead->dev_sample_out;
        a.sm.kept = lead->dev_sample_out + EE_MAX_ROWS;
        a.sm.count = lead->dev_sample_out + 2 * EE_MAX_ROWS;
        a.sm.sums = lead->dev_sample_sums;
        a.keep_logits = 1;   // the sampling launch reads the head launch's logits
    }
    // The first session's descriptor, drafts included, travels with every launch's arguments; a pass of
    // several sessions uploads all of them in one copy (a copy is a launch of its own: 4 us and a gap).
    for (int i = 0; i < n_sessions; ++i) {
        fill_sessdev(lead->host_sessdev[i], sessions[i]);
        memcpy(lead->host_sessdev[i].drafts, drafts[i], (size_t)gamma * sizeof(int));
    }
    if (n_sessions > 1)
        HIP_TRY(hipMemcpyAsync(lead->dev_sessdev, lead->host_sessdev, (size_t)n_sessions * sizeof(SessDev), hipMemcpyHostToDevice, lead->run_stream));
    a.sess = lead->dev_sessdev;
    a.sess0 = lead->host_sessdev[0];

    HIP_TRY(hipEventRecord(lead->ev_start, lead->run_stream));
    lead->lt_codes.clear();
    SampleUpload upload = {sp, n_sessions, gamma};
    int layer = 0;
    for (int e = 0; e <= n_exits; ++e) {
        const bool fin = (e == n_exits);
        const int g_first = fin ? e : e / per_group * per_group;             // first exit of e's group
        const int g_size = fin ? 1 : std::min(per_group, n_exits - g_first);
        a.layer_begin = layer;
        a.layer_end = fin ? c.n_layers : exit_layers[e];
        a.do_embed = (e == 0) ? 1 : 0;
        a.head_kind = fin ? HEAD_FINAL : HEAD_EXIT;
        a.head_idx = g_first;
        a.head_gain = fin ? m->host_md.g_final : gains[e];
        a.n_heads = g_size;
        a.head_rows = g_size * a.rows;
        a.head_row0 = (e - g_first) * a.rows;
        a.head_stage = (e - g_first == g_size - 1) ? 1 : 0;
        a.adapter = (!fin && m->host_md.A > 0) ? 1 : 0;
        a.ad_bdown = a.adapter ? m->ad_bdown[slots[e]] : nullptr;
        a.ad_bup = a.adapter ? m->ad_bup[slots[e]] : nullptr;
        // The adapters of a group's exits run together, in front of the group's head launch, which is what their results wait for: two
        // launches instead of two per exit (7 exits of the 7B shape, 5 rows: 83 us in 14 launches, now 11 + 23).  Where the exits'
        // weights lie a constant number of slices apart, and nothing of it is split over workgroups.
        int slot = fin ? 0 : slots[e], step = 0;
        bool many = a.adapter && g_size > 1 && lead->sc.ha && !static_scratch;
        if (many) {
            step = slots[g_first + 1] - slots[g_first];
            for (int j = 1; j < g_size; ++j) many = many && slots[g_first + j] - slots[g_first + j - 1] == step;
            for (int k : {(int)G_AD, (int)G_AU}) many = many && (a.rows <= 16 || m->plan[1][k].nwg == 0);
        }
        a.ha = many ? lead->sc.ha : nullptr;
        if (!static_scratch) a.sc.xa = lead->sc.xa + (many ? (size_t)(e - g_first) * 2 * a.rows * m->host_md.Kpad_d : 0);
        if (many) {   // (the first exit's)
            slot = slots[g_first];
            a.ad_bdown = m->ad_bdown[slot];
            a.ad_bup = m->ad_bup[slot];
            a.ad_gain = gains[g_first];
        } else {
            a.ad_gain = a.head_gain;
        }
        if ((rc = launch_segment(lead, a, slot, &upload, many, step)) != EE_OK) return rc;
        if (fin) {
            HIP_TRY(hipEventRecord(lead->ev_final, lead->run_stream));
        } else if (a.head_stage) {
            for (int j = g_first; j <= e; ++j) HIP_TRY(hipEventRecord(lead->ev_exit[j], lead->run_stream));
        }
        layer = a.layer_end;
    }
    for (int i = 0; i < n_sessions; ++i) {
        ee_session *s = sessions[i];
        s->in_flight = true;
        s->leader = lead;
        s->flight_gamma = gamma;
        s->flight_exits = n_exits;
        s->flight_row0 = i * M;
        s->popped_mask = 0;
        if (outs) outs[i] = s->result;
    }
    return EE_OK;
}

extern "C" int ee_verify_batch(ee_session *const *sessions, int n_sessions, const int32_t *const *drafts, int gamma,
                               const int32_t *exit_layers, int n_exits, const ee_verify_result **outs)
{
    return verify_impl(sessions, n_sessions, drafts, gamma, exit_layers, n_exits, outs, false);
}

extern "C" int ee_verify(ee_session *s, const int32_t *draft_tokens, int gamma, const int32_t *exit_layers, int n_exits,
                         const ee_verify_result **out)
{
    if (!s) return fail(EE_EINVAL, "ee_verify: null session");
    ee_session *ss[1] = {s};
    const int32_t *dd[1] = {draft_tokens};
    const ee_verify_result *oo[1] = {nullptr};
    int rc = verify_impl(ss, 1, dd, gamma, exit_layers, n_exits, oo, false);
    if (rc == EE_OK && out) *out = oo[0];
    return rc;
}

extern "C" int ee_verify_sampled(ee_session *s, const int32_t *draft_tokens, int gamma, const int32_t *exit_layers, int n_exits,
                                 const ee_sampling *sampling, const ee_verify_result **out)
{
    if (!s) return fail(EE_EINVAL, "ee_verify_sampled: null session");
    if (!sampling) return fail(EE_EINVAL, "ee_verify_sampled: null sampling arguments");
    ee_session *ss[1] = {s};
    const int32_t *dd[1] = {draft_tokens};
    const ee_verify_result *oo[1] = {nullptr};
    int rc = verify_impl(ss, 1, dd, gamma, exit_layers, n_exits, oo, false, sampling);
    if (rc == EE_OK && out) *out = oo[0];
    return rc;
}

extern "C" int ee_verify_sampled_batch(ee_session *const *sessions, int n_sessions, const int32_t *const *drafts, int gamma,
                                       const int32_t *exit_layers, int n_exits, const ee_sampling *samplings,
                                       const ee_verify_result **outs)
{
    if (!samplings) return fail(EE_EINVAL, "ee_verify_sampled_batch: null sampling arguments");
    return verify_impl(sessions, n_sessions, drafts, gamma, exit_layers, n_exits, outs, false, samplings);
}

extern "C" int ee_verify_static(ee_session *s, const int32_t *draft_tokens, int gamma, const int32_t *exit_layers, int n_exits,
                                const ee_verify_result **out)
{
    if (!s) return fail(EE_EINVAL, "ee_verify_static: null session");
    if (s->flags & EE_TIME_LAUNCHES) return fail(EE_ESTATE, "ee_verify_static: not for EE_TIME_LAUNCHES sessions (their event pairs are created on demand)");
    ee_session *ss[1] = {s};
    const int32_t *dd[1] = {draft_tokens};
    const ee_verify_result *oo[1] = {nullptr};
    int rc = verify_impl(ss, 1, dd, gamma, exit_layers, n_exits, oo, true);
    if (rc == EE_OK && out) *out = oo[0];
    return rc;
}

// ------------------------------------------------------------------ waiting

static int exit_event(ee_session *s, int exit_idx, hipEvent_t *ev)
{
    if (!s) return fail(EE_EINVAL, "null session");
    if (s->flight_exits < 0 || exit_idx < 0 || exit_idx >= s->flight_exits)
        return fail(EE_EINVAL, "exit index %d not in [0,%d)", exit_idx, s->flight_exits);
    *ev = s->leader->ev_exit[exit_idx];
    return EE_OK;
}

extern "C" int ee_wait_exit(ee_session *s, int exit_idx)
{
    hipEvent_t ev;
    int rc = exit_event(s, exit_idx, &ev);
    if (rc != EE_OK) return rc;
    if (s->flight_gamma == 0) return fail(EE_ESTATE, "ee_wait_exit: no verify pass was enqueued");
    HIP_TRY(hipEventSynchronize(ev));
    return EE_OK;
}

extern "C" int ee_query_exit(ee_session *s, int exit_idx)
{
    hipEvent_t ev;
    int rc = exit_event(s, exit_idx, &ev);
    if (rc != EE_OK) return rc;
    if (s->flight_gamma == 0) return fail(EE_ESTATE, "ee_query_exit: no verify pass was enqueued");
    hipError_t e = hipEventQuery(ev);
    if (e == hipSuccess) return EE_OK;
    if (e == hipErrorNotReady) return EE_NOT_READY;
    return fail(EE_EDEVICE, "hipEventQuery: %s", hipGetErrorString(e));
}

extern "C" int ee_wait_final(ee_session *s)
{
    if (!s) return fail(EE_EINVAL, "null session");
    if (s->flight_gamma == 0) return fail(EE_ESTATE, "ee_wait_final: no verify pass was enqueued");
    return finish_flight(s);
}

extern "C" int ee_query_final(ee_session *s)
{
    if (!s) return fail(EE_EINVAL, "null session");
    if (s->flight_gamma == 0) return fail(EE_ESTATE, "ee_query_final: no verify pass was enqueued");
    if (!s->in_flight) return EE_OK;
    hipError_t e = hipEventQuery(s->leader->ev_final);
    if (e == hipSuccess) return EE_OK;
    if (e == hipErrorNotReady) return EE_NOT_READY;
    return fail(EE_EDEVICE, "hipEventQuery: %s", hipGetErrorString(e));
}

// ------------------------------------------------------------------ sender queue, latency model

// s^(e) of Alg. 2: the largest confidence among the rows the exit's result consists of
static float exit_score(const ee_verify_result *r, int e)
{
    float sc = 0.f;
    for (int i = 0; i <= r->exit_accept_len[e] && i < EE_MAX_M; ++i) sc = std::max(sc, r->exit_conf[e][i]);
    return sc;
}

extern "C" int ee_exit_pop(ee_session *s, int wait, int *exit_idx, float *score)
{
    if (!s || !exit_idx) return fail(EE_EINVAL, "null argument");
    if (s->flight_gamma == 0) return fail(EE_ESTATE, "ee_exit_pop: no verify pass was enqueued");
    ee_session *lead = s->leader;
    HIP_TRY(hipSetDevice(s->m->device));
    for (;;) {
        if (!s->in_flight || hipEventQuery(lead->ev_final) == hipSuccess) {  // the final result is there: Q_e is reset
            s->popped_mask = ~0ull;
            return EE_DONE;
        }
        int best = -1, first_unpublished = -1;
        float best_sc = -1.f;
        for (int e = 0; e < s->flight_exits; ++e) {
            if (s->popped_mask & (1ull << e)) continue;
            const hipError_t q = hipEventQuery(lead->ev_exit[e]);
            if (q == hipSuccess) {
                const float sc = exit_score(s->result, e);
                if (sc > best_sc) {
                    best_sc = sc;
                    best = e;
                }
            } else if (q == hipErrorNotReady) {
                if (first_unpublished < 0) first_unpublished = e;
            } else {
                return fail(EE_EDEVICE, "hipEventQuery: %s", hipGetErrorString(q));
            }
        }
        if (best >= 0) {
            s->popped_mask |= 1ull << best;
            *exit_idx = best;
            if (score) *score = best_sc;
            return EE_OK;
        }
        if (first_unpublished < 0) return EE_DONE;
        if (!wait) return EE_NOT_READY;
        HIP_TRY(hipEventSynchronize(lead->ev_exit[first_unpublished]));
    }
}

extern "C" int ee_exit_order(ee_session *s, int *order, float *scores)
{
    if (!s || !order) return fail(EE_EINVAL, "null argument");
    if (s->flight_gamma == 0) return fail(EE_ESTATE, "ee_exit_order: no verify pass was enqueued");
    int rc = finish_flight(s);
    if (rc != EE_OK) return rc;
    const int n = s->flight_exits;
    float sc[EE_MAX_EXITS];
    for (int e = 0; e < n; ++e) {
        sc[e] = exit_score(s->result, e);
        order[e] = e;
    }
    std::stable_sort(order, order + n, [&](int a, int b) { return sc[a] > sc[b]; });  // ties: the earlier exit first
    if (scores)
        for (int i = 0; i < n; ++i) scores[i] = sc[order[i]];
    return EE_OK;
}

extern "C" int ee_latency_model(const ee_latency_params *p, ee_latency *out)
{
    if (!p || !out) return fail(EE_EINVAL, "null argument");
    if (!(p->tau > 0.0) || !(p->T_q > 0.0) || p->n < 1 || p->gamma < 1 || !(p->r >= 0.0 && p->r <= 1.0) || p->T_p < 0.0 ||
        p->T_c < 0.0 || p->T_r < 0.0)
        return fail(EE_EINVAL, "ee_latency_model: tau, T_q, n > 0, gamma >= 1, 0 <= r <= 1 and non-negative times are required");
    const double n = (double)p->n, g = (double)p->gamma, rounds = n / p->tau;
    out->ar_ms = 2.0 * p->T_c + n * p->T_q;
    out->sd_ms = rounds * (2.0 * p->T_c + g * p->T_p + p->T_q);
    out->fsd_ms = rounds * (2.0 * p->T_c + p->r * g * p->T_p + (1.0 - p->r) * p->T_r + p->T_q);
    out->ar_ms_per_token = out->ar_ms / n;
    out->sd_ms_per_token = out->sd_ms / n;
    out->fsd_ms_per_token = out->fsd_ms / n;
    out->speedup_ar_to_sd = out->ar_ms / out->sd_ms;
    out->speedup_sd_to_fsd = out->sd_ms / out->fsd_ms;
    out->c = p->T_p / p->T_q;
    out->projected_sd_to_fsd = (g * out->c + 1.0) / (p->r * g * out->c + 1.0);
    return EE_OK;
}

extern "C" int ee_pass_time_ms(ee_session *s, int exit_idx, float *ms)
{
    if (!s || !ms) return fail(EE_EINVAL, "null argument");
    if (s->flight_gamma == 0) return fail(EE_ESTATE, "ee_pass_time_ms: no verify pass was enqueued");
    if (s->in_flight) return fail(EE_ESTATE, "ee_pass_time_ms: the pass has not been waited for");
    if (exit_idx < 0 || exit_idx > s->flight_exits) return fail(EE_EINVAL, "exit index %d not in [0,%d]", exit_idx, s->flight_exits);
    ee_session *lead = s->leader;
    hipEvent_t ev = exit_idx == s->flight_exits ? lead->ev_final : lead->ev_exit[exit_idx];
    HIP_TRY(hipEventElapsedTime(ms, lead->ev_start, ev));
    return EE_OK;
}

// ------------------------------------------------------------------ state

extern "C" int ee_kv_truncate(ee_session *s, int new_len)
{
    if (!s) return fail(EE_EINVAL, "null session");
    HIP_TRY(hipSetDevice(s->m->device));
    int rc = finish_flight(s);
    if (rc != EE_OK) return rc;
    if (new_len < 0 || new_len > s->kv_len) return fail(EE_EINVAL, "ee_kv_truncate: %d not in [0, kv_len=%d]", new_len, s->kv_len);
    s->kv_len = new_len;
    release_pages(s, new_len);
    return EE_OK;
}

extern "C" int ee_set_pending(ee_session *s, int32_t token)
{
    if (!s) return fail(EE_EINVAL, "null session");
    if (token < 0 || token >= s->m->cfg.vocab) return fail(EE_EINVAL, "ee_set_pending: token %d outside [0,%d)", token, s->m->cfg.vocab);
    HIP_TRY(hipSetDevice(s->m->device));
    int rc = finish_flight(s);
    if (rc != EE_OK) return rc;
    s->pending = token;
    s->has_pending = true;
    return EE_OK;
}

extern "C" int ee_kv_len(ee_session *s, int *out)
{
    if (!s || !out) return fail(EE_EINVAL, "null argument");
    int rc = finish_flight(s);
    if (rc != EE_OK) return rc;
    *out = s->kv_len;
    return EE_OK;
}

extern "C" int ee_pending(ee_session *s, int32_t *out)
{
    if (!s || !out) return fail(EE_EINVAL, "null argument");
    int rc = finish_flight(s);
    if (rc != EE_OK) return rc;
    if (!s->has_pending) return fail(EE_ESTATE, "ee_pending: no pending token");
    *out = s->pending;
    return EE_OK;
}

extern "C" int ee_debug_logits(ee_session *s, int head_idx, float *out)
{
    if (!s || !out) return fail(EE_EINVAL, "null argument");
    if (s->flight_gamma == 0) return fail(EE_ESTATE, "ee_debug_logits: no verify pass was enqueued");
    ee_session *lead = s->leader;
    if (!(lead->flags & EE_KEEP_LOGITS))
        return fail(EE_ESTATE, "ee_debug_logits: the session that led the pass was created without EE_KEEP_LOGITS");
    if (head_idx < 0 || head_idx > s->flight_exits) return fail(EE_EINVAL, "head index %d not in [0,%d]", head_idx, s->flight_exits);
    HIP_TRY(hipSetDevice(s->m->device));
    HIP_TRY(hipEventSynchronize(lead->ev_final));
    const size_t V = (size_t)s->m->cfg.vocab, rows_max = (size_t)s->m->cfg.max_rows;
    const int M = s->flight_gamma + 1;
    HIP_TRY(hipMemcpy(out, lead->sc.logits + ((size_t)head_idx * rows_max + (size_t)s->flight_row0) * V, (size_t)M * V * sizeof(float),
                      hipMemcpyDeviceToHost));
    return EE_OK;
}

extern "C" int ee_session_option(ee_session *s, int option, int value)
{
    if (!s) return fail(EE_EINVAL, "null session");
    int rc = finish_flight(s);
    if (rc != EE_OK) return rc;
    switch (option) {
    case EE_OPT_ATT_SPLITS:
        if (value < 0 || value > ATT_MAX_SPLITS) return fail(EE_EINVAL, "EE_OPT_ATT_SPLITS: %d not in [0,%d]", value, ATT_MAX_SPLITS);
        s->att_splits_opt = value;
        return EE_OK;
    case EE_OPT_HEAD_BATCH:
        if (value < 1 || value > EE_MAX_EXITS) return fail(EE_EINVAL, "EE_OPT_HEAD_BATCH: %d not in [1,%d]", value, EE_MAX_EXITS);
        s->head_batch = value;
        return EE_OK;
    case EE_OPT_SCATTER_PAGES:
        if (value != 0 && value != 1) return fail(EE_EINVAL, "EE_OPT_SCATTER_PAGES: %d not 0 or 1", value);
        s->scatter_pages = value != 0;
        return EE_OK;
    case EE_OPT_PREFILL_GEMM: {
        constexpr int shapes = sizeof PF_SHAPES / sizeof PF_SHAPES[0];
        if (value != 0 && (value < 0 || value % 16 < 1 || value % 16 > shapes || value / 16 < 1 || value / 16 > 8))
            return fail(EE_EINVAL, "EE_OPT_PREFILL_GEMM: %d is neither 0 nor 16 * parts (1..8) + shape (1..%d)", value, shapes);
        const size_t need = value ? pf_part_floats(s->m, s->pf_cap, value) : 0;
        if (need > s->pf_part_cap) {   // (the former room stays part of the session's one allocation)
            HIP_TRY(hipSetDevice(s->m->device));
            if ((rc = dev_alloc(s->allocs, &s->pf_part, need, false)) != EE_OK) return rc;
            s->pf_part_cap = need;
        }
        s->pf_gemm_opt = value;
        return EE_OK;
    }
    case EE_OPT_PREFILL_ATT_ROWS:
        if (value != 0 && value != 64 && value != 128) return fail(EE_EINVAL, "EE_OPT_PREFILL_ATT_ROWS: %d not 0, 64 or 128", value);
        s->pf_att_opt = value;
        return EE_OK;
    default:
        return fail(EE_EINVAL, "ee_session_option: unknown option %d", option);
    }
}

// EE_TIME_LAUNCHES sessions: what every launch of the last verify pass ran and how long the
// stream spent between the events recorded right before and right after it.
extern "C" int ee_launch_times(ee_session *s, int32_t *codes, float *ms, int max_launches, int *n_launches)
{
    if (!s || !codes || !ms || !n_launches) return fail(EE_EINVAL, "null argument");
    if (!(s->flags & EE_TIME_LAUNCHES)) return fail(EE_ESTATE, "ee_launch_times: session was created without EE_TIME_LAUNCHES");
    HIP_TRY(hipSetDevice(s->m->device));
    int rc = finish_flight(s);
    if (rc != EE_OK) return rc;
    const int n = std::min((int)s->lt_codes.size(), max_launches);
    for (int i = 0; i < n; ++i) {
        codes[i] = s->lt_codes[i];
        HIP_TRY(hipEventElapsedTime(&ms[i], s->lt_events[2 * i], s->lt_events[2 * i + 1]));
    }
    *n_launches = n;
    return EE_OK;
}

// Measurement aid: `reps` launches of a plain copy kernel (ee_copy_kernel) moving `bytes` bytes
// each between two freshly allocated device buffers.  Profiled with the HBM traffic counters it
// gives the counter reading of a known number of bytes read and written.
extern "C" int ee_debug_copy(int device, size_t bytes, int reps)
{
    HIP_TRY(hipSetDevice(device));
    if (bytes < 16 || reps < 1) return fail(EE_EINVAL, "ee_debug_copy: bytes %zu, reps %d", bytes, reps);
    void *src = nullptr, *dst = nullptr;
    HIP_TRY(hipMalloc(&src, bytes));
    if (hipMalloc(&dst, bytes) != hipSuccess) {
        hipFree(src);
        return fail(EE_EDEVICE, "ee_debug_copy: out of memory");
    }
    hipMemset(src, 0x3C, bytes);
    hipMemset(dst, 0, bytes);
    for (int r = 0; r < reps; ++r)
        hipLaunchKernelGGL(ee_copy_kernel, dim3(4096), dim3(256), 0, 0, static_cast<const uint4 *>(src), static_cast<uint4 *>(dst), bytes / 16);
    hipError_t e = hipDeviceSynchronize();
    hipFree(src);
    hipFree(dst);
    if (e != hipSuccess) return fail(EE_EDEVICE, "ee_debug_copy: %s", hipGetErrorString(e));
    return EE_OK;
}

extern "C" int ee_device_synchronize(int device)
{
    HIP_TRY(hipSetDevice(device));
    HIP_TRY(hipDeviceSynchronize());
    return EE_OK;
}

// ------------------------------------------------------------------ self-check of the MFMA lane layout

// Fills A[16][32] and B[32][16] with small integers, runs one MFMA through the
// lane layout the kernels assume and compares with the plain product.
// Returns EE_OK when every element agrees.
extern "C" int ee_debug_div_small(int device, const int32_t *divisors, int n, long long *mismatches)
{
    if (!divisors || !mismatches || n < 1 || n > 65536) return fail(EE_EINVAL, "ee_debug_div_small: bad argument");
    for (int i = 0; i < n; ++i)
        if (divisors[i] < 1) return fail(EE_EINVAL, "ee_debug_div_small: divisor %d", divisors[i]);
    HIP_TRY(hipSetDevice(device));
    int *dd = nullptr;
    unsigned long long *dbad = nullptr, bad = 0;
    HIP_TRY(hipMalloc(reinterpret_cast<void **>(&dd), (size_t)n * sizeof(int)));
    HIP_TRY(hipMalloc(reinterpret_cast<void **>(&dbad), sizeof bad));
    HIP_TRY(hipMemcpy(dd, divisors, (size_t)n * sizeof(int), hipMemcpyHostToDevice));
    HIP_TRY(hipMemset(dbad, 0, sizeof bad));
    hipLaunchKernelGGL(div_small_check_kernel, dim3(256, std::min(n, 256)), dim3(256), 0, 0, dd, n, DIV_SMALL_MAX, dbad);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipMemcpy(&bad, dbad, sizeof bad, hipMemcpyDeviceToHost));
    hipFree(dd);
    hipFree(dbad);
    *mismatches = (long long)bad;
    return EE_OK;
}

extern "C" int ee_debug_mfma_layout(int device)
{
    HIP_TRY(hipSetDevice(device));
    uint16_t ha[64 * 8], hb[64 * 8];
    float A[16][32], B[32][16];
    for (int i = 0; i < 16; ++i)
        for (int k = 0; k < 32; ++k) A[i][k] = (float)((i * 7 + k * 3) % 13 - 6);
    for (int k = 0; k < 32; ++k)
        for (int j = 0; j < 16; ++j) B[k][j] = (float)((k * 5 + j * 11) % 9 - 4);
    auto bf = [](float f) {
        uint32_t u;
        memcpy(&u, &f, 4);
        return (uint16_t)(u >> 16);  // small integers are exact in bf16
    };
    for (int l = 0; l < 64; ++l)
        for (int e = 0; e < 8; ++e) {
            ha[l * 8 + e] = bf(A[l & 15][(l >> 4) * 8 + e]);
            hb[l * 8 + e] = bf(B[(l >> 4) * 8 + e][l & 15]);
        }
    uint4 *da = nullptr, *db = nullptr;
    float *dout = nullptr;
    HIP_TRY(hipMalloc(reinterpret_cast<void **>(&da), sizeof ha));
    HIP_TRY(hipMalloc(reinterpret_cast<void **>(&db), sizeof hb));
    HIP_TRY(hipMalloc(reinterpret_cast<void **>(&dout), 256 * sizeof(float)));
    HIP_TRY(hipMemcpy(da, ha, sizeof ha, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(db, hb, sizeof hb, hipMemcpyHostToDevice));
    hipLaunchKernelGGL(mfma_layout_probe_kernel, dim3(1), dim3(64), 0, 0, da, db, dout);
    HIP_TRY(hipGetLastError());
    float out[256];
    HIP_TRY(hipMemcpy(out, dout, sizeof out, hipMemcpyDeviceToHost));
    hipFree(da);
    hipFree(db);
    hipFree(dout);
    int bad = 0;
    for (int l = 0; l < 64; ++l)
        for (int r = 0; r < 4; ++r) {
            int i = (l >> 4) * 4 + r, j = l & 15;
            float ref = 0.f;
            for (int k = 0; k < 32; ++k) ref += A[i][k] * B[k][j];
            if (out[l * 4 + r] != ref) ++bad;
        }
    if (bad) return fail(EE_EDEVICE, "MFMA 16x16x32 lane layout differs from the assumed one in %d of 256 elements", bad);

    // v_mfma_f32_16x16x16bf16_1k: the first 16 k of the same matrices, four k per lane
    uint16_t ga[64 * 4], gb[64 * 4];
    for (int l = 0; l < 64; ++l)
        for (int e = 0; e < 4; ++e) {
            ga[l * 4 + e] = bf(A[l & 15][(l >> 4) * 4 + e]);
            gb[l * 4 + e] = bf(B[(l >> 4) * 4 + e][l & 15]);
        }
    uint2 *ea = nullptr, *eb = nullptr;
    HIP_TRY(hipMalloc(reinterpret_cast<void **>(&ea), sizeof ga));
    HIP_TRY(hipMalloc(reinterpret_cast<void **>(&eb), sizeof gb));
    HIP_TRY(hipMalloc(reinterpret_cast<void **>(&dout), 256 * sizeof(float)));
    HIP_TRY(hipMemcpy(ea, ga, sizeof ga, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(eb, gb, sizeof gb, hipMemcpyHostToDevice));
    hipLaunchKernelGGL(mfma16_layout_probe_kernel, dim3(1), dim3(64), 0, 0, ea, eb, dout);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipMemcpy(out, dout, sizeof out, hipMemcpyDeviceToHost));
    hipFree(ea);
    hipFree(eb);
    hipFree(dout);
    bad = 0;
    for (int l = 0; l < 64; ++l)
        for (int r = 0; r < 4; ++r) {
            int i = (l >> 4) * 4 + r, j = l & 15;
            float ref = 0.f;
            for (int k = 0; k < 16; ++k) ref += A[i][k] * B[k][j];
            if (out[l * 4 + r] != ref) ++bad;
        }
    if (bad) return fail(EE_EDEVICE, "MFMA 16x16x16 lane layout differs from the assumed one in %d of 256 elements", bad);
    return EE_OK;
}
