// Structures shared by the host runtime and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/ee.h"

namespace ee {

constexpr int SWAVES = 8;                // streaming waves: weight tiles -> MFMA
constexpr int HWAVES = 4;                // helper waves: work out what the epilogue needs while the others stream
constexpr int WAVES = SWAVES + HWAVES;   // three per SIMD, 168 VGPRs each
constexpr int WG_THREADS = WAVES * 64;
constexpr int GROUP_TILES = 8;           // n-tiles whose accumulators a streaming wave keeps in registers at once
constexpr int KV_PAGE = 16;              // positions per KV page
constexpr int ATT_ROWS = 16;             // query rows of one attention item (one MFMA tile)
constexpr int ATT_TILES = 8;             // KV pages a wave takes at most per launch of the attention
constexpr int ATT_MAX_SPLITS = 16;
constexpr int KSPLIT_LOG2 = 2;           // many-row launches: workgroups (1 << this) that share n-tiles and split K (at most SWAVES)

// Weight layout of one GEMM y = x . W^T, W[N][K] row-major in the model file.
//
// A tile is the A operand of one v_mfma_f32_16x16x32_bf16: 16 rows of N by 32
// columns of K, stored as 64 lanes x 16 bytes, lane l holding
// W[nt*16 + (l & 15)][kt*32 + (l >> 4)*8 .. +7]  (1 KB per tile).
//
// The N axis is cut into units of `tpu` n-tiles (1, or 2 for a gate/up pair);
// workgroup g owns a contiguous range of units (`base`, and one more if g < `rem`) for the whole of K, so
// every output element is complete inside one workgroup.  Its n-tiles are taken in groups
// of up to GROUP_TILES; streaming wave w owns the k-tiles w, w + SWAVES, w + 2 SWAVES, ...
// ("k-steps" s = 0, 1, ...) and walks
//   for group : for k-step s : for n-tile of the group : tile(n-tile, k-tile w + SWAVES*s)
// keeping one accumulator per n-tile of the group in registers for the whole of K.  The order
// does not depend on the number of rows.
// In memory the tiles are interleaved over the whole chip: the i-th tile of the
// sequence of wave w of workgroup g sits at tile slot (i*nwg + g)*SWAVES + w, so at any
// moment all waves together read one contiguous window (measured: up to 15 % more
// HBM bandwidth than one contiguous range per wave).  `steps` is the longest sequence.
struct GemmPlan {
    int N, K;        // logical shape (N counts rows after concatenation / interleaving)
    int NT, KT;      // tiles along N and K (K zero-padded to 32)
    int tpu;         // n-tiles per unit
    int base, rem;   // units per workgroup: the first `rem` have base + 1.  Workgroups are dealt to the chip's 8 XCDs
                     // round-robin and every XCD has its own path to memory: the larger shares are spread evenly too.
    int steps;       // tile slots per wave (longest wave sequence)
    int nwg;         // workgroups that take part in this stage kind: the fewest that keep the busiest one's
                     // share unchanged, so that all of them get (nearly) the same share; the rest idle.
                     // Half of the compute units already saturate HBM, uneven shares only lengthen the tail.
    // K split over workgroups (many-row launches): 1 << ksl consecutive workgroups share the same
    // n-tiles and take one slice of KTs k-tiles each (workgroup g: n-tiles of g >> ksl, slice
    // g & (splits - 1)); their partial tiles meet in memory and the one that arrives last adds them
    // up and runs the epilogue.  A workgroup then reads only its slice of the input.  ksl = 0, KTs = KT: no split.
    int ksl, KTs;
};

// LDS map of one GEMM launch, chosen on the host from the rows of the launch:
//   [rings of the streaming waves | later: partial tiles] [misc]
// While a group streams, wave w's ring of stages (weight tiles and input k-tiles) is the w-th
// WAVE_LDS_KB kilobytes.  Afterwards the same space holds the waves' partial tiles for the
// cross-wave sum ([wave][n-tile of the chunk][row][16] floats, `chunk` n-tiles at a time) and,
// behind them at zbuf_off, one [row][chunk*16] float tile for the head's logits / the squares of the
// residual stream.
// Packed weights: behind them, at corr_off, the group's sums over the weights that the packed form leaves out,
// [n-tile of the group][row][16] floats, in a place of their own: the helper waves fill it while the rings are in use.
struct StageLds {
    int chunk;       // n-tiles reduced at a time
    int zbuf_off;
    int corr_off;
    int misc_off;
};

// Packed weights: the same tiles in the same slots, a weight in 12 bits instead of 16.  The bf16 weights of a
// matrix lie in few binades: with its 16 most common neighbouring exponents as a window, sign, mantissa and 4 bits of
// exponent say all but about one weight in 10000 of a normal distribution.  Those others stand in the tile as the
// smallest value of the window (code 0), and in a list of the matrix with the difference to what they should be;
// helper waves add the list's products to the sums while the weights stream (EscapeSums).  The difference is fp32: exact for weights between
// 2^-31 and 2^9 on the moved scale below (its window ends at 2), beyond that off by 2^-39 or by 2^-24 of the weight; and as the product is the sum
// of two, an infinite input times a positive weight below the window is no infinity but NaN.
// A tile is 64 lanes x 12 bytes: dwords A and B the low bytes of the lane's eight bf16 values, C their variable high bits (sign and
// upper three exponent bits, PACK_MASK, of pair j rotated left by 4 j).  The window's exponents are moved to 112 .. 127 (a power of two that
// the epilogue takes back exactly, GemmEntry::wscale): the constant exponent bits are 0111, and unpacking is a byte permute, a rotate and a
// bit-field insert per pair of weights.
constexpr int PACK_TILE = 768;
constexpr int PACK_EXP0 = 112;                   // where the window's smallest exponent is moved to
constexpr unsigned PACK_CONST = 0x38383838u;     // the constant exponent bits in a bf16's high byte
constexpr unsigned PACK_MASK = 0x87008700u;      // the variable bits of a pair's high bytes
constexpr float PACK_CODE0 = 1.0f / 32768.0f;    // what code 0 unpacks to
__host__ __device__ constexpr int tile_bytes_of(bool packed) { return packed ? PACK_TILE : 1024; }

// A weight that the packed form leaves out: what its column's sum misses per unit of x[k] (in the window's scale), and where.
struct Escape {
    float delta;
    unsigned kn;     // k << 16 | (column & 0xFFFF)
};
// A helper wave's part of a group's escapes: the first place is the header (delta: places taken, itself included, as an integer; kn: the
// part's first column in the group << 8 | the end of its columns), then the escapes.  Parts are multiples of eight places.
constexpr int ESCAPES_MAX = 63;
static_assert(sizeof(Escape) == 8, "eight are a scalar load");
static_assert(GROUP_TILES * 16 < 256, "a column of a group in eight bits");

// Per-row partial results of the workgroups (sums of squares, argmax candidates) are stored [row][SS_LD],
// one slot per workgroup.
constexpr int SS_LD = 256;

// GEMM inputs are followed by at least this many elements that may be read: a k-tile is copied in whole kilobytes (what
// lies behind its rows ends up in lanes whose products are dropped).
constexpr int X_SLACK = 512;

constexpr int NUM_XCD = 8;
// x / d for 0 <= x <= DIV_SMALL_MAX and d >= 1.  The GPU has no integer division: a 32-bit one is
// about 40 instructions in a dependent chain, a 64-bit one several hundred, and the kernels divide
// by run-time values on the way to their first load, at every block boundary of the stream and in
// every epilogue item.  One reciprocal (1 ulp) and one multiply give the exact quotient in this
// range: (x + 0.5) / d is at least 0.5 / d away from an integer and the error of the product is
// below (x + 0.5) / d * 1.8e-7, which is less than 0.5 / d for x < 2.7e6.
constexpr int DIV_SMALL_MAX = 2500000;
__host__ __device__ inline int div_small(int x, int d)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return (int)(((float)x + 0.5f) * __builtin_amdgcn_rcpf((float)d));
#else
    return x / d;
#endif
}

enum RowPerm { PERM_NONE = 0, PERM_QKV = 1, PERM_GU = 2 };
enum GemmKind { G_QKV = 0, G_O = 1, G_GU = 2, G_DN = 3, G_HEAD = 4, G_AD = 5, G_AU = 6, G_KINDS = 7 };  // AD / AU: an exit head's adapter, down and up

struct ModelDev {
    int L, d, H, hd, F, V;
    float eps, att_scale;
    int Kpad_d, Kpad_F;                  // K rounded up to 32
    int rows_max;
    int A, Kpad_A;                       // hidden units of an exit head's adapters (all bottlenecks together; 0: none), rounded up to 32
    const float *g_attn, *g_ffn;         // [L][d]
    const float *g_final;
    const uint16_t *emb;                 // [V][d] bf16, row-major
};

struct SessDev {
    const int *page_table;               // logical page -> physical page
    uint16_t *kpool, *vpool;             // per (layer, page, head) a record of KV_PAGE*2*hd bf16, value = hi + lo:
                                         // K [position][term][hd], V [term][hd][position]
    const float2 *rope;                  // [max_ctx][hd/2] (cos, sin)
    ee_verify_result *result;            // device address of the pinned result block
    int n_pages;
    int kv_len;                          // positions cached before this pass
    int pending;                         // token of row 0
    int drafts[EE_MAX_M - 1];            // this pass's drafts
    int contig_base;                     // >= 0: logical page i is physical page contig_base + i (no table lookup needed)
};

struct Scratch {
    float *h;            // [rows_max][d]        residual stream
    float *q;            // [rows_max][d]        queries after RoPE (pair-interleaved inside each head)
    // GEMM inputs as two bf16 terms each (x = hi + lo up to ~16 mantissa bits), written by the
    // stage that produces them, k-tile-major: [k-tile][term][row of the pass][32]
    uint16_t *xn;        // [Kpad_d/32][2][rows][32]  gain * h for the next QKV or gate/up GEMM
    uint16_t *xh;        // [Kpad_d/32][2][head rows][32]  head_gain * (h, or h after the adapters) for the LM head; the rows
                         // of all exits that share one launch of the head, exit after exit
    uint16_t *attn;      // [Kpad_d/32][2][rows][32]  attention output
    uint16_t *u;         // [Kpad_F/32][2][rows][32]  silu(gate)*up
    uint16_t *xa;        // [Kpad_d/32][2][rows][32]  h itself: input of an exit head's adapters (exit after exit where they share a launch)
    uint16_t *t;         // [Kpad_A/32][2][rows][32]  the adapters' hidden units after the activation (exit after exit)
    float *ha;           // [rows_max][d]        h after the layers of the exits whose adapters share a launch, or nullptr
    float *ss_h;         // [rows_max][SS_LD]        partial sums of squares of the LM-head input's rows (head rows)
    float *ss_a;         // [rows_max][SS_LD]        partial sums of h^2 after the FFN block / embedding
    float *ss_f;         // [rows_max][SS_LD]        partial sums of h^2 after the attention block
    float *att_part;     // [items][ATT_ROWS * (hd+2)] attention partials (att_item; only when the position range is split)
    int *att_count;      // [units] items of the unit that have delivered their partials; zero between launches
    int *head_count;     // workgroups of a head launch that have delivered their candidates; zero between launches
    float *part;         // [K split][n-tile][rows][16] partial tiles of a launch whose K is split over workgroups
    int *part_count;     // [nwg] splits of a group of workgroups that have delivered their partial tiles; zero between launches
    float *logits;       // [heads][rows_max][V] when logits are kept
    int2 *cand;          // [rows_max][SS_LD]        per-workgroup argmax candidates (value bits, index)
    float *cand_sum;     // [rows_max][SS_LD]        sum over the workgroup's columns of exp(logit - candidate value)
};

enum HeadKind { HEAD_NONE = 0, HEAD_EXIT = 1, HEAD_FINAL = 2, HEAD_PREFILL = 3 };

// Probabilistic verification: inputs and per-row decisions.
struct SampleDev {
    const float *probs;  // [session][gamma][V]  the draft model's distributions
    const float *uv;     // per session 2 gamma + 2 floats: [gamma] the keep tests' uniform numbers, [gamma+1] the rows'
                         // sampling numbers, 1 / temperature
    int on;              // 1: the pass decides by the draft probabilities instead of by exact match
    int *tok;            // [head rows]  token a row emits if the round ends there
    int *kept;           // [head rows]  1: the row's draft passes its test
    int *count;          // rows of a sampling launch that have delivered, then [head rows] parts of a row; zero between launches
    unsigned long long *sums;   // [2][head rows][parts]  the parts' sums of exponentials, of residual weights (40-bit fixed point)
};

// What a GEMM launch needs to request its first weights and input: one line of the launch arguments, read with one
// scalar load (see gemm_entry).
struct GemmEntry {
    const uint4 *W;                      // the stage's weights
    const uint16_t *X;                   // its input
    int wstep;                           // bytes from one tile of a wave's sequence to the next
    int tile_bytes;                      // bytes of one k-tile of the input: all rows, both terms
    int KTs, nwg, base, rem, tpu, ksl;   // of the plan
    union {
        struct {
            const Escape *esc;           // packed weights: [workgroup][esc_groups][HWAVES][esc_cap]
            uint16_t esc_groups, esc_cap; // groups of n-tiles of the busiest workgroup; places of a part
            float wscale;                // packed weights: what the sums are multiplied by (a power of two)
        };
        struct {
            long long w_next;            // adapters of several exits in one launch (blockIdx.y): bytes from one exit's weights
            int x_next, unused;          // and input to the next one's
        };
    };
};
static_assert(sizeof(GemmEntry) == 64, "one line");

struct PassArgs {
    GemmEntry entry;                     // (first: the kernels read it at the start of their arguments)
    ModelDev mdv;                        // the model descriptor by value
    GemmPlan plan0;                      // plan and LDS map of the launch's GEMM stage
    StageLds lay;
    Scratch sc;
    int nwg;
    int n_sess, M, rows;                 // rows = n_sess * M
    int mode;                            // 0 verify, 1 prefill (a prompt of up to rows_max rows, or the last row's head)
    const int *pf_tokens;                // prefill: [rows] token ids, < 0 => embedding row
    const uint16_t *pf_emb;              // prefill: [rows][d] bf16
    int pf_pos0;                         // prefill: position of row 0; always 0, a prompt of more rows than a pass takes the
                                         // many-row kernels.  Written as a constant in the kernels the QKV launch of the 13B
                                         // shape is 0.4 us longer (27.4 against 27.0, 1253 against 1241 us for 8 layers).
    int layer_begin, layer_end;          // (host) layers [begin, end) of this segment, 0-based
    int do_embed;
    int head_kind, head_idx;             // head_idx: result slot of the (first) head of this segment's head launch
    const float *head_gain;
    int n_heads;                         // exit heads evaluated by the head launch (their rows follow each other)
    int head_rows;                       // rows of the head launch: n_heads * rows
    int head_row0;                       // first head row this segment's exit writes (its position in the group)
    int head_stage;                      // 1: this segment ends with the head launch (else its exit only deposits its rows)
    int adapter;                         // 1: the exit has adapters (stages AD, AU between the last layer and the head)
    const float *ad_bdown, *ad_bup;      // adapter biases: [A] and [d] (the bottlenecks' output biases summed)
    const float *ad_gain;                // (host) gain of the head behind the adapters: the exit's, or the group's first exit's
    int keep_logits;
    int fuse_accept;                     // the head launch also runs the accept step (in the workgroup that finishes last)
    int att_splits;                      // splits of the position range (of the session with the most)
    unsigned long long att_starts;       // != 0: sessions have splits of their own, one behind the other in the grid: bit i is set where a
                                         // session's first one is i, and behind the last session's last; 0: all have att_splits
    int H, d, Kpad_d;                    // copies of the model descriptor's fields for the attention kernel
    float att_scale;
    int layer;                           // layer of this launch's stage
    const float *gain_xn, *gain_xh;      // O, DN: gain of the next GEMM input; DN, AU: gain of the LM head's input (each may be null)
    const float *bias;                   // AD, AU: bias per output column
    int t_next, bias_next, gain_next;    // AD, AU of several exits: elements of t, biases and gains from one exit to the next
    float *ha;                           // adapters of several exits: [head rows][d] h after each exit's layer (DN writes, AU reads), or nullptr
    int xa_out;                          // DN: also emit h itself as the adapters' input
    const SessDev *sess;                 // device array [n_sess] (passes of several sessions only)
    SessDev sess0;                       // session 0: a pass of one session needs nothing but its launch arguments
    SampleDev sm;
};

typedef void (*pass_kernel_t)(PassArgs);
// The kernel of a GEMM kind for so many rows.  Defined per kind in a translation unit of its own (ee_gemm_*.hip): they are compiled side by side.
template <int KIND>
pass_kernel_t gemm_kernel_of(int rows, bool packed);

}  // namespace ee
