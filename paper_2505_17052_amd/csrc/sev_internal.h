// Internal declarations shared by the translation units of libsev.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <vector>

#include "../../include/sev.h"

#define SEV_PAGE 16
#define SEV_ATT_MAX_CP 256   // pages per attention work item, upper bound (a block of 8 waves x 16 pairs)
#define SEV_ATT_MAX_CHUNK 128   // pages per chunk when sequences are split over several blocks of 4 waves

// ---------------------------------------------------------------------------
// error plumbing (host)
// ---------------------------------------------------------------------------
int sev_fail(int code, const char *fmt, ...);
#define SEV_HIP(expr)                                                                      \
    do {                                                                                   \
        hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess)                                                              \
            return sev_fail(SEV_EHIP, "%s: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, __LINE__); \
    } while (0)

// ---------------------------------------------------------------------------
// packed activation layout for the matrix-core GEMMs ("xpack")
//
// A [M][K] activation matrix is carried as two bf16 planes (hi = bf16(x),
// lo = bf16(x - hi)), already arranged as MFMA 16x16x32 operand fragments:
//   [K/32 k-steps][row units of 16][plane 2][lane 64][8 bf16]
// lane = (m % 16) + 16 * ((k / 8) % 4), element = k % 8.  One fragment is 1 KiB.
// units = row units of the buffer: ceil(M/16) rounded up to a multiple of 8.
// ---------------------------------------------------------------------------
__host__ __device__ inline int64_t xpack_index(int m, int k, int plane, int units) {
    return ((((int64_t)(k >> 5) * units + (m >> 4)) * 2 + plane) << 9) + (((m & 15) + (((k >> 3) & 3) << 4)) << 3) +
           (k & 7);
}

inline int sev_row_units(int rows) { return (rows + 127) / 128 * 8; }

struct LayerOffsets {
    size_t wqkv, wo, wgu, wd, g_attn, g_ffn;
};

struct sev_model {
    sev_model_desc d;
    char *arena;
    size_t arena_bytes;
    size_t off_embed, off_lm, off_gfinal;
    std::vector<LayerOffsets> layers;
    int n_qkv;   // (Hq + 2 Hkv) * hd
    int q_dim;   // Hq * hd
    int kv_dim;  // Hkv * hd
};

// Per-call description handed to the plan kernel by value (together with PlanDev it stays below the 4 KiB that a
// kernel's arguments may take; slots are below 65536, see sev_kv_create).
struct PlanArgs {
    int B, k_max;
    int first;                // row of the token array that belongs to request 0
    int tail;                 // 1: rows of blocks that are already in the cache (end of a prefill): the slots' state is left alone
    int pad_tokens;           // > 0: attention walks every request's pages up to this many tokens (padded-KV comparison variant)
    uint16_t slot[SEV_MAX_BATCH];
    int32_t prefix[SEV_MAX_BATCH];
    int32_t nd[SEV_MAX_BATCH];
    int32_t tok0[SEV_MAX_BATCH];   // token of node i of request b: tokens[(first + b) * k_max + tok0[b] + i], counted in 64 bits
};

// Device-side call plan (one per sev_kv; rebuilt by every verify).
struct DevPlan {
    // per request
    int32_t *req_slot, *req_P, *req_n, *req_row0;
    // per row (draft node)
    int32_t *row_req, *row_node;
    int32_t *row_kvloc;       // physical page * 16 + token in page of the cache position P + node the row is written to
    unsigned long long *row_anc;
    float2 *row_cs;           // [rows][hd/2] (cos, sin) of pos * theta_i
    double *theta;            // [hd/2] theta_i = base^(-2i/hd), written once when the handle is created
    // attention work items (bf16 path): a = {row group, first page, pages, prefix length},
    // b = {draft nodes, first row, request, 0}; pages = physical page ids of the chunk, SEV_ATT_MAX_CP per item
    int4 *it_a, *it_b;
    int32_t *it_pages;
    int4 *mg_rec;             // [merge groups] {row group (of 32 or 128 rows) | chunks << 16, first work item, draft nodes | item stride << 16, first row}
    int causal;               // 1: blocks are chains (node i sees nodes <= i; any length), 0: trees (ancestor masks, <= 64 nodes)
};

enum ProfClass { PROF_GEMM_QKV = 0, PROF_GEMM_O, PROF_GEMM_GU, PROF_GEMM_DOWN, PROF_GEMM_LM, PROF_ATTN, PROF_OTHER, PROF_N };

struct ProfSpan {
    hipEvent_t a, b;
    int cls;
};

// Tile-shape overrides for tuning experiments, read from the environment ONCE, when the handle is created:
// SEV_TUNE_QKV / _O / _GU / _DOWN = "MT,NT,S,PF" (MT row tiles of 32, or -MT row units of 16; S = 0 keeps the automatic split; NT = 0: blocks of one column tile), SEV_TUNE_TPB = column tiles
// per block of the gate/up GEMM, SEV_TUNE_CP = pages per attention chunk, SEV_TUNE_QUAD = 0: no attention blocks of four
// row groups, n > 0: always, with chunks of n pages.  Unset (the normal case): all zero, quad -1.
struct Tune {
    int gemm[4][4];
    bool has_gemm[4];
    int tpb, cp, quad;
};

// Tile configuration of a matrix-core GEMM (choose_cfg in kernels_bf16.hip).
struct GemmCfg {
    int MR, NT, S;          // row units of 16 per block, column tiles per wave (0: one tile per block, whose waves share K), K slices
    bool half;              // the last of the NT column tiles is shared by two waves: 4 (NT - 1) + 2 tiles per block
    int T;                  // column tiles per block (cols() unless a narrower block fills the chip better)
    int cols() const { return half ? 4 * (NT - 1) + 2 : 4 * NT; }
};
#define SEV_KEPT_UNITS 128   // row counts (in units of 16) whose configurations a handle keeps

// What the stochastic rule found at one node of a tree (sample_nodes_kernel).
enum { NODE_OPEN = 0, NODE_ACCEPTED, NODE_REJECTED };      // nothing yet; accepted `child`; rejected nrej of the children below `child`
#define SEV_NODE_REJ 4       // rejections worked off there
struct SampleNode {
    int state, child, nrej;
    int rej[SEV_NODE_REJ];   // the rejected children whose residual counts, and its normalisers
    float R[SEV_NODE_REJ];
};

struct sev_kv {
    const sev_model *model;
    Tune tune;
    std::vector<GemmCfg> gemm_kept;          // [5 GEMMs][SEV_KEPT_UNITS]; MR = 0: not chosen yet
    int max_req, max_rows, page_size;
    int64_t n_pages;
    char *pool;
    size_t pool_bytes;
    size_t layer_stride;      // bytes between layers in the pool
    size_t v_offset;          // bytes from a layer's K pages to its V pages
    int max_pages_per_req;

    // device state (one allocation: `ws`)
    char *ws;
    size_t ws_bytes;
    int32_t *page_table;      // [max_req][max_pages_per_req]
    int32_t *seq_len, *next_tok;             // [max_req]
    int32_t *pend_n, *pend_a, *pend_bonus, *pend_P;   // [max_req] pending block: size, accepted, bonus, prefix length at verify
    int32_t *pend_path;       // [max_req][SEV_MAX_DRAFT]
    uint32_t *err_flags;      // [1]
    DevPlan plan;
    int max_items, max_groups;

    // activations
    float *h;                 // [rows][d] residual stream
    float *part;              // split-K exchange buffer / f32 scratch
    size_t part_elems;
    unsigned long long *ssq[2];   // bf16: fixed-point sums of squares of the residual rows (two buffers, used alternately)
    void *xa;                 // normed activations (xpack for bf16, [rows][d] f32 otherwise)
    void *q_buf;              // bf16: q hi/lo planes [2][rows][Hq*hd]; f32: qkv [rows][n_qkv]
    void *o_buf;              // attention output (xpack K=q_dim, or f32 [rows][q_dim])
    void *act;                // SwiGLU output (xpack K=d_ffn, or f32 [rows][d_ffn])
    float *att_o;             // attention partials [items*Hkv][32][hd]
    float2 *att_ml;           // [items*Hkv][32] (running max, sum)
    float *lm_val;            // [tiles][rows] partial arg-max values
    int32_t *lm_idx;
    int32_t *row_argmax;      // [rows]
    uint16_t *tail_q;         // bf16, end of a prefill: q planes [2][requests][Hq*hd] and residual rows [requests][d] of the last
    float *tail_h;            //   token of every prompt that ends in the chunk
    SampleNode *sample_nodes; // [rows]
    float2 *row_stats;        // [rows] (largest logit, sum of exp((logit - max) / T)) of the stochastic rule
    float *logits_f32;        // f32 path only: [rows][vocab]

    // host mirrors
    std::vector<int> host_pages;   // pages assigned per slot
    std::vector<char> host_tree;   // per slot: the last verified block was a tree (its commit may have to move K/V); 2: captured
    // profiling
    int prof_on;
    std::vector<ProfSpan> spans;
    double prof_ms[PROF_N];
    int64_t prof_n[PROF_N];
};

struct Prof {
    sev_kv *kv;
    hipStream_t st;
    int cls;
    hipEvent_t a, b;
    bool on;
    Prof(sev_kv *kv_, hipStream_t st_, int cls_);
    ~Prof();
};

// ---------------------------------------------------------------------------
// launchers (defined in the kernel translation units)
// ---------------------------------------------------------------------------
// Work list of the attention over one batch of blocks (see pick_chunk_pages).
struct AttList {
    int n_items, n_groups, sib, chunk_pages;
    bool direct;
    int quad;                // row groups of 32 query rows per work item: 1, or 4 (a block of four waves that share K/V in LDS)
};

// What the output head leaves for the acceptance: the arg-max of every row, or what it is taken from.
enum HeadKind { HEAD_ROWS, HEAD_PARTS, HEAD_LOGITS };
struct HeadOut {
    HeadKind kind;
    const int32_t *rows;      // HEAD_ROWS: [rows]
    const float *val;         // HEAD_PARTS: [n_part][stride] largest values and their columns; HEAD_LOGITS: [rows][n_part] logits
    const int32_t *idx;
    int n_part, stride;
};

bool sev_capturing(hipStream_t st);

// common
void launch_fill_f32(float *p, float v, int64_t n, hipStream_t st);
void launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t st);
void launch_plan(const sev_kv *kv, const PlanArgs &pa, const int32_t *draft_tokens, const int32_t *parents,
                 const AttList &att, hipStream_t st);
void launch_theta(const sev_kv *kv, hipStream_t st);
void launch_accept(const sev_kv *kv, const HeadOut &ho, int B, int k_max, int mode, const int32_t *draft_tokens, const int32_t *parents,
                   int32_t *accept_len, int32_t *bonus, int32_t *accept_path, int32_t *argmax_out, hipStream_t st);
void launch_sample(const sev_kv *kv, int B, int k_max, int rows, const int32_t *tokens, const int32_t *parents, const float *logits,
                   const float *draft_probs, float2 *stats, float temperature, const float *u_acc, const float *u_emit,
                   int32_t *accept_len, int32_t *emitted, int32_t *accept_path, hipStream_t st);
void launch_prefill_state(const sev_kv *kv, const PlanArgs &pa, const int32_t *row, hipStream_t st);
void launch_commit(const sev_kv *kv, const int32_t *slots_dev_by_value, int B, bool rollback, hipStream_t st);
void launch_kv_copy(const sev_kv *kv, int slot, int layer, int start, int n, void *k, void *v, int to_cache, hipStream_t st);
void launch_argmax_rows_f32(const float *logits, int rows, int vocab, int32_t *out, hipStream_t st);

// f32 path
void launch_pack_f32(float *dst, const float *src, int64_t n, hipStream_t st);
// both: head = nullptr takes the arg-max of every row into kv->row_argmax (prefill); else it says where to find it
void f32_forward(const sev_model *m, sev_kv *kv, int rows, int B, float *logits_out, HeadOut *head, hipStream_t st);

// bf16 path
void launch_pack_bf16(uint16_t *dst, const uint16_t *src, int n_rows, int K, int mode, int tile_add, hipStream_t st);

// End of a prefill chunk: only the last token of each of F prompts is wanted from the last layer on (F = 0: none).
struct TailRows {
    int F;
    PlanArgs pa;                     // the F tokens as blocks of one node behind their own prefix
    AttList att;
    int32_t src[SEV_MAX_BATCH];      // their rows in the chunk
    const int32_t *tokens;
};
void bf16_forward(const sev_model *m, sev_kv *kv, int rows, int B, const AttList &att, float *logits_out, const TailRows *tail, HeadOut *head,
                  hipStream_t st);
