// Kernels shared by both precisions: call plan, acceptance, KV commit, cache import/export.
#include <algorithm>

#include "sev_internal.h"
#include "kv_layout.h"
#include "row_ops.h"

// ---------------------------------------------------------------------------
// fills
// ---------------------------------------------------------------------------
__global__ void fill_f32_kernel(float *p, float v, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}
__global__ void fill_i32_kernel(int32_t *p, int32_t v, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}
void launch_fill_f32(float *p, float v, int64_t n, hipStream_t st) {
    if (n > 0) hipLaunchKernelGGL(fill_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, v, n);
}
void launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t st) {
    if (n > 0) hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, v, n);
}

// ---------------------------------------------------------------------------
// call plan: everything the forward pass needs to know about the batch,
// derived on the device from the lengths passed by value.
//
// Per request: row range, prefix length, slot.  Per draft node (row): request,
// node index, rotary position P + depth, ancestor-or-self bit mask, token.
// Per row and rotary frequency: (cos, sin) of pos * base^(-2i/hd), evaluated in
// double so that positions in the thousands keep full float accuracy.
// For the matrix-core attention: the list of (request, row group, KV chunk)
// work items and the per (request, row group) merge groups.
//
// One kernel, bound by latency alone: every block scans the (at most 256) requests' sizes itself and then fills its
// own share, so no block waits for another and no second launch is needed.  The first n_row_blocks blocks take 16 rows
// of one request each, the next n_item_blocks four work items (one per wave), and the last, one per row, gather the rows' embeddings
// (a kernel of its own behind the plan took 1.6-14 us and a launch).  The ancestor sets of a tree come from pointer
// doubling in LDS (six rounds for 64 nodes); a depth is the number of ancestors.  (One thread per request walking
// its tree, and a second kernel for the tables, took 55 + 6 us for 8 trees of 64 nodes and 5 + 5 us for 16 chains of 8.)
// ---------------------------------------------------------------------------
struct PlanDev {
    DevPlan p;
    int32_t *seq_len, *pend_n, *pend_P;
    uint32_t *err;
    int vocab, hd, G;          // G = query heads per KV head
    int chunk_pages;
    int group_rows;            // query rows per work item (32, or 128 where four waves share the K/V)
    const int32_t *tokens, *parents;
    const int32_t *page_table;
    int max_pages;
    EmbedArgs emb;
};
static_assert(sizeof(PlanArgs) + sizeof(PlanDev) + 64 <= 4096, "kernel arguments of the plan");

#define PLAN_ROWS 16           // rows per row block
#define PLAN_ITEMS 4           // work items per item block

__global__ void theta_kernel(double *theta, int hd, double rope_base) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < hd / 2) theta[i] = pow(rope_base, -2.0 * (double)i / (double)hd);
}

void launch_theta(const sev_kv *kv, hipStream_t st) {
    const int hd = kv->model->d.head_dim;
    hipLaunchKernelGGL(theta_kernel, dim3((hd / 2 + 63) / 64), dim3(64), 0, st, kv->plan.theta, hd, (double)kv->model->d.rope_base);
}

// largest b in [0, B) with first[b] <= m (first ascends, first[0] = 0; entries of empty requests never win)
__device__ __forceinline__ int plan_find(const int *first, int B, int m) {
    int lo = 0, hi = B - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first[mid] <= m) lo = mid; else hi = mid - 1;
    }
    return lo;
}

template <bool BF16>
__global__ __launch_bounds__(256) void plan_kernel(PlanArgs a, PlanDev d, int n_row_blocks, int n_item_blocks, int n_items) {
    __shared__ int s_first[4][SEV_MAX_BATCH];                  // per request: first row, merge group, work item, row block
    __shared__ int s_tot[4][4];
    __shared__ unsigned long long s_anc[2][SEV_MAX_DRAFT];
    __shared__ int s_up[2][SEV_MAX_DRAFT];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int B = a.B;
    int mine[4] = {0, 0, 0, 0};
    if (t < B) {
        const int n = a.nd[t];
        const int pages = (max(a.prefix[t] + n, a.pad_tokens) + SEV_PAGE - 1) / SEV_PAGE;
        mine[0] = n;
        mine[1] = (d.G * n + d.group_rows - 1) / d.group_rows;
        mine[2] = mine[1] * ((pages + d.chunk_pages - 1) / d.chunk_pages);
        mine[3] = (n + PLAN_ROWS - 1) / PLAN_ROWS;
    }
    int inc[4] = {mine[0], mine[1], mine[2], mine[3]};
#pragma unroll
    for (int o = 1; o < 64; o <<= 1)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int y = __shfl_up(inc[q], o);
            if (lane >= o) inc[q] += y;
        }
    if (lane == 63)
#pragma unroll
        for (int q = 0; q < 4; ++q) s_tot[q][wave] = inc[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        int before = 0;
        for (int w = 0; w < wave; ++w) before += s_tot[q][w];
        s_first[q][t] = before + inc[q] - mine[q];
    }
    __syncthreads();

    const int blk = blockIdx.x;
    if (blk < n_row_blocks) {                                   // 16 rows of one request
        const int b = plan_find(s_first[3], B, blk);
        const int i0 = (blk - s_first[3][b]) * PLAN_ROWS;
        const int slot = a.slot[b], P = a.prefix[b], n = a.nd[b], row0 = s_first[0][b];
        if (i0 == 0 && t == 0) {
            if (!a.tail) {
                if (d.seq_len[slot] != P) atomicOr(d.err, 1u);
                d.pend_n[slot] = 0;                             // a new verify drops whatever was pending
                d.pend_P[slot] = P;
            }
            d.p.req_slot[b] = slot;
            d.p.req_P[b] = P;
            d.p.req_n[b] = n;
            d.p.req_row0[b] = row0;
        }
        int cur = 0;
        if (d.parents) {                                        // trees: n <= 64 nodes, parents precede children
            if (t < SEV_MAX_DRAFT) {
                int par = -1;
                if (t < n) {
                    par = d.parents[b * a.k_max + t];
                    if (par < -1 || par >= t) { atomicOr(d.err, 2u); par = -1; }
                }
                s_anc[0][t] = 1ull << t;
                s_up[0][t] = par;
            }
            __syncthreads();
            for (int r = 0; r < 6; ++r, cur ^= 1) {             // after r rounds: the ancestors up to 2^r - 1 levels up
                if (t < SEV_MAX_DRAFT) {
                    const int up = s_up[cur][t];
                    s_anc[cur ^ 1][t] = s_anc[cur][t] | (up >= 0 ? s_anc[cur][up] : 0ull);
                    s_up[cur ^ 1][t] = up >= 0 ? s_up[cur][up] : -1;
                }
                __syncthreads();
            }
        }
        if (t < PLAN_ROWS && i0 + t < n) {
            const int i = i0 + t, row = row0 + i;
            const int tok = d.tokens[(size_t)(a.first + b) * a.k_max + a.tok0[b] + i];
            if (tok < 0 || tok >= d.vocab) atomicOr(d.err, 4u);
            const unsigned long long anc = d.parents ? s_anc[cur][i] : (i < 63 ? (2ull << i) - 1ull : ~0ull);
            d.p.row_req[row] = b;
            d.p.row_node[row] = i;
            d.p.row_anc[row] = anc;
            d.p.row_kvloc[row] = d.page_table[(size_t)slot * d.max_pages + (P + i) / SEV_PAGE] * SEV_PAGE + (P + i) % SEV_PAGE;
        }
        const int half = d.hd / 2, rows = min(PLAN_ROWS, n - i0);
        for (int e = t; e < rows * half; e += 256) {
            const int r = e / half, i = e - r * half, node = i0 + r;
            const int pos = P + (d.parents ? __popcll(s_anc[cur][node]) - 1 : node);
            double s, c;
            sincos((double)pos * d.p.theta[i], &s, &c);
            d.p.row_cs[(size_t)(row0 + node) * half + i] = make_float2((float)c, (float)s);
        }
        return;
    }
    if (blk >= n_row_blocks + n_item_blocks) {                  // the embedding of one row
        __shared__ float s_red[4];
        const int m = blk - n_row_blocks - n_item_blocks, b = plan_find(s_first[0], B, m);
        const int tok = d.tokens[(size_t)(a.first + b) * a.k_max + a.tok0[b] + (m - s_first[0][b])];
        embed_row<BF16>(d.emb, m, tok < 0 || tok >= d.vocab ? 0 : tok, s_red);      // (the row's own block flags such a token)
        return;
    }
    // attention work items.  A request's pages are split evenly over its chunks; item order: chunk by chunk, the row
    // groups of one chunk side by side (the attention kernel puts them on one XCD, where the chunk is then fetched from
    // memory once for all of them).  The page list is padded with the chunk's last page, so that the attention kernel
    // can load its page ids without knowing the chunk length.
    const int it = (blk - n_row_blocks) * PLAN_ITEMS + wave;
    if (it >= n_items) return;
    const int b = plan_find(s_first[2], B, it);
    const int slot = a.slot[b], P = a.prefix[b], n = a.nd[b];
    const int pages = (max(P + n, a.pad_tokens) + SEV_PAGE - 1) / SEV_PAGE;
    const int groups = (d.G * n + d.group_rows - 1) / d.group_rows, chunks = (pages + d.chunk_pages - 1) / d.chunk_pages;
    const int cpp = (pages + chunks - 1) / chunks;
    const int local = it - s_first[2][b], c = local / groups, rg = local - c * groups;
    const int p0 = c * cpp, np = min(cpp, pages - p0);
    if (lane == 0) {
        d.p.it_a[it] = make_int4(rg, p0, np, P);
        d.p.it_b[it] = make_int4(n, s_first[0][b], b, slot);
        if (c == 0) d.p.mg_rec[s_first[1][b] + rg] = make_int4(rg | (chunks << 16), it, n | (groups << 16), s_first[0][b]);
    }
#pragma unroll
    for (int i = lane; i < SEV_ATT_MAX_CP; i += 64)
        d.p.it_pages[(size_t)it * SEV_ATT_MAX_CP + i] = d.page_table[(size_t)slot * d.max_pages + p0 + min(i, np - 1)];
}

void launch_plan(const sev_kv *kv, const PlanArgs &pa, const int32_t *draft_tokens, const int32_t *parents,
                 const AttList &att, hipStream_t st) {
    const int n_items = att.n_items;
    PlanDev d;
    d.p = kv->plan;
    d.seq_len = kv->seq_len;
    d.pend_n = kv->pend_n;
    d.pend_P = kv->pend_P;
    d.err = kv->err_flags;
    d.vocab = kv->model->d.vocab;
    d.hd = kv->model->d.head_dim;
    d.G = kv->model->d.n_q_heads / kv->model->d.n_kv_heads;
    d.chunk_pages = att.chunk_pages;
    d.group_rows = 32 * att.quad;
    d.tokens = draft_tokens;
    d.parents = parents;
    d.page_table = kv->page_table;
    d.max_pages = kv->max_pages_per_req;
    int row_blocks = 0, rows = 0;
    for (int b = 0; b < pa.B; ++b) {
        row_blocks += (pa.nd[b] + PLAN_ROWS - 1) / PLAN_ROWS;
        rows += pa.nd[b];
    }
    const sev_model *m = kv->model;
    const bool bf = m->d.dtype == SEV_BF16;
    d.emb.E = m->arena + m->off_embed;
    d.emb.h = kv->h;
    d.emb.d = m->d.d_model;
    d.emb.g = (const float *)(m->arena + m->layers[0].g_attn);
    d.emb.xa = (uint16_t *)kv->xa;
    d.emb.ssq_out = kv->ssq[1];
    d.emb.ssq_clear = kv->ssq[0];
    d.emb.units = sev_row_units(rows);
    const int item_blocks = (n_items + PLAN_ITEMS - 1) / PLAN_ITEMS;
    if (pa.tail) rows = 0;                              // (their rows are in the stream already)
    const dim3 grid((unsigned)(row_blocks + item_blocks + rows));
    if (bf) hipLaunchKernelGGL((plan_kernel<true>), grid, dim3(256), 0, st, pa, d, row_blocks, item_blocks, n_items);
    else hipLaunchKernelGGL((plan_kernel<false>), grid, dim3(256), 0, st, pa, d, row_blocks, item_blocks, n_items);
}

// ---------------------------------------------------------------------------
// greedy acceptance (paper section 4.1: accepted candidates plus one additional
// token from the server's own forward pass).  One block per request.  First the arg-max of its rows, from what the head left
// (HEAD_PARTS: the matrix-core GEMM's partial results; HEAD_LOGITS: float32 logits; HEAD_ROWS: it is there already): the lanes
// of a wave take the request's rows side by side (16 bytes to 256 of a line), the waves different parts.  Then one wave, one lane
// per candidate: a step of the walk is a ballot over (parent, token), so it is two loads deep whatever the tree (a thread
// per request, searching the children in memory, took 50 us for 8 trees of 64 nodes and 11 us for chains of 8).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void arg_max(float &v, int &i, float ov, int oi) {
    if (ov > v || (ov == v && oi < i)) { v = ov; i = oi; }       // lowest index wins ties
}

#define ACCEPT_WAVES 16
template <int HEAD>
__global__ __launch_bounds__(HEAD == HEAD_ROWS ? 64 : ACCEPT_WAVES * 64) void accept_kernel(DevPlan p, HeadOut ho, int k_max, int mode, const int32_t *tokens,
                                                                                            const int32_t *parents, const int32_t *next_tok, int32_t *pend_n,
                                                                                            int32_t *pend_a, int32_t *pend_bonus, int32_t *pend_path,
                                                                                            int32_t *accept_len, int32_t *bonus_out, int32_t *path_out,
                                                                                            int32_t *argmax_out) {
    const int b = blockIdx.x, c = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int slot = p.req_slot[b], n = p.req_n[b], row0 = p.req_row0[b];
    int am = 0;
    if constexpr (HEAD == HEAD_ROWS) {
        am = c < n ? ho.rows[row0 + c] : 0;
    } else {
        __shared__ float s_v[ACCEPT_WAVES][64];
        __shared__ int s_i[ACCEPT_WAVES][64];
        if constexpr (HEAD == HEAD_PARTS) {
            const int R = n > 1 ? 2 << (31 - __clz(n - 1)) : 1, sub = c / R, per = 64 / R;      // a power of two of lanes for the rows
            const size_t at = row0 + min(c & (R - 1), n - 1);
            float v = -INFINITY;
            int i = 0x7fffffff;
#pragma unroll 8
            for (int q = wave * per + sub; q < ho.n_part; q += ACCEPT_WAVES * per)
                arg_max(v, i, ho.val[(size_t)q * ho.stride + at], ho.idx[(size_t)q * ho.stride + at]);
            for (int o = R; o < 64; o *= 2) {
                const float ov = __shfl_xor(v, o);
                const int oi = __shfl_xor(i, o);
                arg_max(v, i, ov, oi);
            }
            s_v[wave][c] = v;
            s_i[wave][c] = i;
            __syncthreads();
            if (wave) return;
            for (int w = 1; w < ACCEPT_WAVES; ++w) arg_max(v, i, s_v[w][c], s_i[w][c]);
            am = c < n ? i : 0;
        } else {
            for (int r = wave; r < n; r += ACCEPT_WAVES) {
                const float *row = ho.val + (size_t)(row0 + r) * ho.n_part;
                float v = -INFINITY;
                int i = 0x7fffffff;
#pragma unroll 8
                for (int q = c; q < ho.n_part; q += 64) arg_max(v, i, row[q], q);
                for (int o = 1; o < 64; o *= 2) {
                    const float ov = __shfl_xor(v, o);
                    const int oi = __shfl_xor(i, o);
                    arg_max(v, i, ov, oi);
                }
                if (c == 0) s_i[0][r] = i;
            }
            __syncthreads();
            if (wave) return;
            am = c < n ? s_i[0][c] : 0;
        }
    }
    const bool live = c < n;
    const int tok = live ? tokens[(size_t)b * k_max + c] : -1;
    int par = live ? (parents ? parents[(size_t)b * k_max + c] : c - 1) : -2;
    if (live && (par < -1 || par >= c)) par = -1;
    int a = 0, want = next_tok[slot], mine = -1;
    if (mode == 1) {                       // append: keep the whole chain
        a = n;
        mine = live ? c : -1;
        want = __shfl(am, n - 1);
    } else {
        int cur = -1;
        while (true) {
            const unsigned long long hit = __ballot(par == cur && tok == want);     // children come after their parent; the lowest matching index wins
            if (!hit) break;
            cur = __ffsll((long long)hit) - 1;
            if (c == a) mine = cur;
            ++a;
            want = __shfl(am, cur);
        }
    }
    pend_path[(size_t)slot * SEV_MAX_DRAFT + c] = mine;
    if (path_out && c < k_max) path_out[(size_t)b * k_max + c] = mine;
    if (argmax_out && live) argmax_out[row0 + c] = am;
    if (c == 0) {
        pend_n[slot] = n;
        pend_a[slot] = a;
        pend_bonus[slot] = want;
        accept_len[b] = a;
        bonus_out[b] = want;
    }
}

void launch_accept(const sev_kv *kv, const HeadOut &ho, int B, int k_max, int mode, const int32_t *draft_tokens, const int32_t *parents,
                   int32_t *accept_len, int32_t *bonus, int32_t *accept_path, int32_t *argmax_out, hipStream_t st) {
#define SEV_ACCEPT(HEAD_, THREADS_)                                                                                                      \
    hipLaunchKernelGGL((accept_kernel<HEAD_>), dim3(B), dim3(THREADS_), 0, st, kv->plan, ho, k_max, mode, draft_tokens, parents, kv->next_tok, \
                       kv->pend_n, kv->pend_a, kv->pend_bonus, kv->pend_path, accept_len, bonus, accept_path, argmax_out)
    if (ho.kind == HEAD_PARTS) SEV_ACCEPT(HEAD_PARTS, ACCEPT_WAVES * 64);
    else if (ho.kind == HEAD_LOGITS) SEV_ACCEPT(HEAD_LOGITS, ACCEPT_WAVES * 64);
    else SEV_ACCEPT(HEAD_ROWS, 64);
#undef SEV_ACCEPT
}

// ---------------------------------------------------------------------------
// commit / rollback (paper section 4.2: the cache follows the accepted tokens)
// ---------------------------------------------------------------------------
struct SlotList {
    int32_t s[SEV_MAX_BATCH];
};

// grid (ceil(L*Hkv*hd/256), B).  Each thread owns one (layer, kv head, element) and moves it for the
// accepted nodes in ascending order; destinations never lie ahead of a source still to be read
// because an accepted node's index is at least its depth.
template <typename T, bool BF16>
__global__ void commit_copy_kernel(SlotList sl, KvGeom g, const int32_t *page_table, int max_pages,
                                   const int32_t *pend_n, const int32_t *pend_a, const int32_t *pend_P,
                                   const int32_t *pend_path) {
    const int slot = sl.s[blockIdx.y];
    if (pend_n[slot] == 0) return;
    const int a = pend_a[slot], P = pend_P[slot];
    const int32_t *path = pend_path + (size_t)slot * SEV_MAX_DRAFT;
    bool moved = false;
    for (int j = 0; j < a; ++j) moved |= (path[j] != j);
    if (!moved) return;
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    const int per_layer = g.Hkv * g.hd;
    if (idx >= g.L * per_layer) return;
    const int layer = idx / per_layer, rem = idx - layer * per_layer, h = rem / g.hd, e = rem - h * g.hd;
    const int32_t *pt = page_table + (size_t)slot * max_pages;
    T *base = (T *)(g.pool + (size_t)layer * g.layer_stride);
    T *vbase = (T *)(g.pool + (size_t)layer * g.layer_stride + g.v_offset);
    for (int j = 0; j < a; ++j) {
        const int src = P + path[j], dst = P + j;
        if (src == dst) continue;
        const size_t so = (size_t)pt[src / SEV_PAGE] * g.Hkv + h, dofs = (size_t)pt[dst / SEV_PAGE] * g.Hkv + h;
        const int blk = SEV_PAGE * g.hd;
        base[dofs * blk + k_in_page<BF16>(dst % SEV_PAGE, e, g.hd)] = base[so * blk + k_in_page<BF16>(src % SEV_PAGE, e, g.hd)];
        vbase[dofs * blk + v_in_page<BF16>(dst % SEV_PAGE, e, g.hd)] = vbase[so * blk + v_in_page<BF16>(src % SEV_PAGE, e, g.hd)];
    }
}

__global__ void commit_state_kernel(SlotList sl, int B, int rollback, int32_t *seq_len, int32_t *next_tok,
                                    int32_t *pend_n, const int32_t *pend_a, const int32_t *pend_bonus) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const int slot = sl.s[b];
    if (pend_n[slot] == 0) return;
    if (!rollback) {
        seq_len[slot] += pend_a[slot];
        next_tok[slot] = pend_bonus[slot];
    }
    pend_n[slot] = 0;
}

// After a chunk of a prefill: every listed slot grows by its tokens; a prompt that ended takes the arg-max after its last
// token as its next token (row[b] = its entry of row_argmax), the others have none yet (row[b] = -1).
struct PrefillState {
    uint16_t slot[SEV_MAX_BATCH];
    int32_t n[SEV_MAX_BATCH], row[SEV_MAX_BATCH];
};

__global__ void prefill_state_kernel(PrefillState s, int B, const int32_t *row_argmax, int32_t *seq_len, int32_t *next_tok) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const int slot = s.slot[b];
    seq_len[slot] += s.n[b];
    next_tok[slot] = s.row[b] >= 0 ? row_argmax[s.row[b]] : -1;
}

void launch_prefill_state(const sev_kv *kv, const PlanArgs &pa, const int32_t *row, hipStream_t st) {
    PrefillState s;
    for (int b = 0; b < pa.B; ++b) {
        s.slot[b] = pa.slot[b];
        s.n[b] = pa.nd[b];
        s.row[b] = row[b];
    }
    hipLaunchKernelGGL(prefill_state_kernel, dim3((pa.B + 63) / 64), dim3(64), 0, st, s, pa.B, kv->row_argmax, kv->seq_len, kv->next_tok);
}

// ---------------------------------------------------------------------------
// stochastic verification (paper section 4.1: the draft/verify cycle preserves the server
// model's output distribution, by the accept / resample rule of speculative sampling, in its
// multi-step form for trees; section 5: temperature 0.7).  All random numbers are inputs.
//
// softmax_stats_kernel: one block per row: the row's largest logit and the sum of
//   exp((logit - max) / T).
// sample_walk_kernel: one block per request.  The block's root must be the server's own previous
//   token.  At the current node, with p = the server distribution computed there, the children
//   are tried in index order: child c (token x, edge distribution q_c) is accepted iff
//   u_acc[c] * q_c(x) < p(x); a rejection replaces p by the normalised residual max(0, p - q_c)
//   (the normaliser is a block-wide sum over the vocabulary, in a fixed order); an acceptance
//   moves to c.  When no child is left the emitted token is drawn from the current p by inverse
//   CDF in token-id order: sums of groups of 64 consecutive ids, a scan over the groups, then a
//   scan inside the group that holds u_emit * total.  Chains are trees whose node i has parent
//   i - 1.
// ---------------------------------------------------------------------------
#define SEV_MAX_REJ 16   // rejected siblings remembered at one node

__global__ __launch_bounds__(1024) void softmax_stats_kernel(const float *logits, int vocab, float inv_t, float2 *stats) {
    // one pass with a running maximum (the sum is rescaled whenever the maximum grows); 16-byte loads where the
    // row allows it; the partial (max, sum) pairs are combined in a fixed order
    __shared__ float red_m[16], red_s[16];
    const float *row = logits + (size_t)blockIdx.x * vocab;
    float m = -INFINITY, sum = 0.f;
    auto take = [&](float x) {
        if (x > m) { sum *= expf((m - x) * inv_t); m = x; }       // exp(-inf) = 0 covers the first element
        sum += expf((x - m) * inv_t);
    };
    const bool vec = ((vocab & 3) == 0) && ((((size_t)blockIdx.x * vocab) & 3) == 0) && ((((uintptr_t)logits) & 15) == 0);
    if (vec) {
        const float4 *r4 = (const float4 *)row;
        for (int i = threadIdx.x; i < (vocab >> 2); i += 1024) {
            const float4 x = r4[i];
            const float mx4 = fmaxf(fmaxf(x.x, x.y), fmaxf(x.z, x.w));
            if (mx4 > m) { sum *= expf((m - mx4) * inv_t); m = mx4; }
            sum += expf((x.x - m) * inv_t) + expf((x.y - m) * inv_t) + expf((x.z - m) * inv_t) + expf((x.w - m) * inv_t);
        }
    } else {
        for (int v = threadIdx.x; v < vocab; v += 1024) take(row[v]);
    }
    // wave, then block: (m, s) pairs merge as s = s_a * exp((m_a - m) / T) + s_b * exp((m_b - m) / T)
    auto merge = [&](float mo, float so) {
        const float mn = fmaxf(m, mo);
        const float a = (m == -INFINITY) ? 0.f : expf((m - mn) * inv_t), b = (mo == -INFINITY) ? 0.f : expf((mo - mn) * inv_t);
        sum = sum * a + so * b;
        m = mn;
    };
    for (int o = 32; o > 0; o >>= 1) merge(__shfl_xor(m, o), __shfl_xor(sum, o));
    if ((threadIdx.x & 63) == 0) { red_m[threadIdx.x >> 6] = m; red_s[threadIdx.x >> 6] = sum; }
    __syncthreads();
    if (threadIdx.x == 0) {
        m = red_m[0]; sum = red_s[0];
#pragma unroll
        for (int w = 1; w < 16; ++w) merge(red_m[w], red_s[w]);
        stats[blockIdx.x] = make_float2(m, sum);
    }
}

// Division by a number that a whole pass divides by: its reciprocal once, then a quotient and one correction with the exact remainder, which rounds as
// x / y does (as long as nothing underflows) in three instructions instead of about eleven.  The passes over the vocabulary below are bound by
// their vector instructions and load latencies: 128256 ids, one rejection and the draw on one compute
// unit: 86 us with divisions, 69 without, 57 with several places of a row requested together (current4).
struct Divisor {
    float y, inv;             // inv = 0: y is too small or not finite, divide
    __device__ __forceinline__ void set(float y_) {
        y = y_;
        inv = y_ > 1e-30f && y_ < 1e30f ? 1.0f / y_ : 0.f;
    }
    __device__ __forceinline__ Divisor uniform() const {      // the same for all lanes: the branch below is then a scalar one
        Divisor d;
        d.y = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(y)));
        d.inv = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(inv)));
        return d;
    }
    __device__ __forceinline__ float of(float x) const {
        if (inv == 0.f) return x / y;
        const float q = x * inv;
        return fmaf(fmaf(-q, y, x), inv, q);
    }
};

struct WalkState {
    int cur, a, nrej, child, action;       // action: 0 accepted a child, 1 rejected one (in rej[nrej]), 2 no child left
    int rej[SEV_MAX_REJ + 1];
    Divisor R[SEV_MAX_REJ + 1];
    Divisor den;                           // sum behind the softmax of `cur`
    float top;                             // its largest logit
    int path[SEV_MAX_DRAFT];
};

// A request's block during the walk: its tokens and (sanitised) parents in LDS, and for every node the outcome of its acceptance test
// against the plain softmax at its parent: the test the walk needs as long as no sibling was rejected at that
// parent, taken for all nodes at once instead of one after the other along the path.
struct WalkBlock {
    int tk[SEV_MAX_DRAFT], par[SEV_MAX_DRAFT], acc0[SEV_MAX_DRAFT];
};

#define WALK_BATCH 4
struct WalkIn {
    const float *logits, *draft_probs;     // the request's rows
    const float2 *stats;
    const float *u_acc;
    int vocab, n;
    float inv_t;
    bool vec;                              // rows can be read 16 bytes at a time
    __device__ __forceinline__ WalkIn(const float *logits_, const float *draft_probs_, const float2 *stats_, const float *u_acc_, int b, int row0, int n_,
                                      int k_max, int vocab_, float inv_t_)
        : logits(logits_ + (size_t)row0 * vocab_), draft_probs(draft_probs_ + (size_t)row0 * vocab_), stats(stats_ + row0),
          u_acc(u_acc_ + (size_t)b * k_max), vocab(vocab_), n(n_), inv_t(inv_t_),
          vec(((vocab_ & 3) == 0) && ((((uintptr_t)logits_ | (uintptr_t)draft_probs_) & 15) == 0)) {}
    __device__ __forceinline__ void block(WalkBlock &w, const int32_t *tokens, const int32_t *parents) const {      // tokens, parents: the request's
        const int c = threadIdx.x;
        if (c >= n) return;
        const int q0 = parents ? parents[c] : c - 1;
        const int q = (q0 < -1 || q0 >= c) ? -1 : q0;
        int x = tokens[c];
        if (x < 0 || x >= vocab) x = 0;                 // the embedding step has flagged it and used id 0 as well
        w.tk[c] = x;
        w.par[c] = q;
        int ok = 0;
        if (q >= 0) {
            const float2 st = stats[q];
            const float px = expf((logits[(size_t)q * vocab + x] - st.x) * inv_t) / st.y;
            ok = u_acc[c] * draft_probs[(size_t)c * vocab + x] < px;
        }
        w.acc0[c] = ok;
    }
    __device__ __forceinline__ void enter(WalkState &s) const {      // (one thread) the node's softmax
        const float2 st = stats[s.cur];
        s.top = st.x;
        s.den.set(st.y);
    }
    // value at token v of the current distribution: the node's softmax, then one residual step per rejected sibling
    __device__ __forceinline__ float current(const WalkState &s, int v) const {
        float r = s.den.of(expf((logits[(size_t)s.cur * vocab + v] - s.top) * inv_t));
        for (int j = 0; j < s.nrej; ++j) r = s.R[j].of(fmaxf(r - draft_probs[(size_t)s.rej[j] * vocab + v], 0.f));
        return r;
    }
    // the same for four consecutive ids at each of WALK_BATCH places i, i + stride, .. (in units of four ids; past the end: the last ones again).
    // All places of a row are requested together: one after the other, a pass would wait a memory latency per place and row.
    __device__ __forceinline__ void current4(const WalkState &s, int i, int stride, float4 (&r)[WALK_BATCH]) const {
        const int last = (vocab >> 2) - 1;
        const Divisor den = s.den.uniform();
        const float top = s.top;
        const float4 *row = (const float4 *)(logits + (size_t)s.cur * vocab);
#pragma unroll
        for (int u = 0; u < WALK_BATCH; ++u) r[u] = row[min(i + u * stride, last)];
#pragma unroll
        for (int u = 0; u < WALK_BATCH; ++u)
            r[u] = make_float4(den.of(expf((r[u].x - top) * inv_t)), den.of(expf((r[u].y - top) * inv_t)), den.of(expf((r[u].z - top) * inv_t)),
                               den.of(expf((r[u].w - top) * inv_t)));
        for (int j = 0; j < s.nrej; ++j) {
            const float4 *qrow = (const float4 *)(draft_probs + (size_t)s.rej[j] * vocab);
            const Divisor R = s.R[j].uniform();
            float4 q[WALK_BATCH];
#pragma unroll
            for (int u = 0; u < WALK_BATCH; ++u) q[u] = qrow[min(i + u * stride, last)];
#pragma unroll
            for (int u = 0; u < WALK_BATCH; ++u)
                r[u] = make_float4(R.of(fmaxf(r[u].x - q[u].x, 0.f)), R.of(fmaxf(r[u].y - q[u].y, 0.f)), R.of(fmaxf(r[u].z - q[u].z, 0.f)),
                                   R.of(fmaxf(r[u].w - q[u].w, 0.f)));
        }
    }
    // the next child of the current node and its test (one thread)
    __device__ __forceinline__ void try_child(WalkState &s, const WalkBlock &w) const {
        s.action = 2;
        for (int c = s.child; c < n; ++c) {
            if (w.par[c] != s.cur) continue;
            const int x = w.tk[c];
            s.child = c + 1;
            const bool ok = s.nrej == 0 ? w.acc0[c] != 0 : u_acc[c] * draft_probs[(size_t)c * vocab + x] < current(s, x);
            if (ok) {
                s.cur = c;
                s.path[s.a++] = c;
                s.nrej = 0;
                s.action = 0;
                enter(s);
            } else {
                s.rej[s.nrej] = c;
                s.action = 1;
            }
            break;
        }
    }
    // normaliser of the residual against the rejected child: a block-wide pass over the vocabulary, thread t at ids t, t + 1024, ...
    // (coalesced); wave sums, then the 16 wave totals in order
    __device__ __forceinline__ void reject(WalkState &s, float *s_part, uint32_t *err) const {
        const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
        const float *qrow = draft_probs + (size_t)s.rej[s.nrej] * vocab;
        float sum = 0.f;
        if (vec) {
            const int end = vocab >> 2;
            for (int i = t; i < end; i += 1024 * WALK_BATCH) {
                float4 r[WALK_BATCH], q[WALK_BATCH];
#pragma unroll
                for (int u = 0; u < WALK_BATCH; ++u) q[u] = ((const float4 *)qrow)[min(i + 1024 * u, end - 1)];
                current4(s, i, 1024, r);
#pragma unroll
                for (int u = 0; u < WALK_BATCH; ++u)
                    if (i + 1024 * u < end)
                        sum += (fmaxf(r[u].x - q[u].x, 0.f) + fmaxf(r[u].y - q[u].y, 0.f)) + (fmaxf(r[u].z - q[u].z, 0.f) + fmaxf(r[u].w - q[u].w, 0.f));
            }
        } else {
            for (int v = t; v < vocab; v += 1024) sum += fmaxf(current(s, v) - qrow[v], 0.f);
        }
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
        if (lane == 0) s_part[wave] = sum;
        __syncthreads();
        if (t == 0) {
            float tot = 0.f;
            for (int i = 0; i < 16; ++i) tot += s_part[i];
            if (s.nrej >= SEV_MAX_REJ) atomicOr(err, 8u);           // more rejected siblings than the walk remembers
            else if (tot > 0.f) { s.R[s.nrej].set(tot); ++s.nrej; }    // an empty residual leaves the distribution as it is
        }
        __syncthreads();
    }
};

// Trees: the tests at all nodes that the walk may reach, one block per node, so that the passes over the vocabulary that follow rejected
// siblings run side by side and not one after the other along the path.  What happens at a node does not depend on how the walk came there.  A node is
// left out if an ancestor's first child passes its test and the way to the node leads through another child.  At most SEV_NODE_REJ rejections are worked off,
// so that a node with many children which the walk never sees cannot hold it up; the walk goes on from there.
// 6 trees of up to 40 nodes, 128256 ids: the walk alone 455 us, 254 with the nodes' blocks in front of it and the passes below.
__global__ __launch_bounds__(1024) void sample_nodes_kernel(DevPlan p, int k_max, const int32_t *tokens, const int32_t *parents, const float *logits,
                                                            const float *draft_probs, const float2 *stats, int vocab, float inv_t, const float *u_acc,
                                                            SampleNode *out) {
    __shared__ WalkState s;
    __shared__ WalkBlock w;
    __shared__ float s_part[16];
    __shared__ int s_go;
    const int row = blockIdx.x, b = p.row_req[row], node = p.row_node[row], t = threadIdx.x;
    const int n = p.req_n[b];
    const WalkIn in(logits, draft_probs, stats, u_acc, b, p.req_row0[b], n, k_max, vocab, inv_t);
    in.block(w, tokens + (size_t)b * k_max, parents + (size_t)b * k_max);
    if (t == 0) { s.cur = node; s.a = 0; s.nrej = 0; s.child = node + 1; s.action = 1; s_go = 1; in.enter(s); }
    __syncthreads();
    if (t < n && t < node) {                             // thread q: is q an ancestor whose first child bars the way?
        int at = node;
        while (at > t && w.par[at] != t) at = w.par[at];
        if (at > t) {
            int first = t + 1;
            while (w.par[first] != t) ++first;           // (at the latest `at`)
            if (first != at && w.acc0[first]) s_go = 0;
        }
    }
    __syncthreads();
    if (s_go) {
        for (int pass = 0;; ++pass) {
            if (t == 0) {
                if (pass < SEV_NODE_REJ) in.try_child(s, w);
                else s.action = 3;
            }
            __syncthreads();
            if (s.action != 1) break;
            in.reject(s, s_part, nullptr);
        }
    }
    if (t == 0) {
        SampleNode &o = out[row];
        o.state = !s_go ? NODE_OPEN : s.action == 0 ? NODE_ACCEPTED : NODE_REJECTED;
        o.child = s.action == 0 && s_go ? s.cur : s.child;
        o.nrej = s_go && s.action != 0 ? s.nrej : 0;
        for (int j = 0; j < SEV_NODE_REJ; ++j)
            if (j < o.nrej) { o.rej[j] = s.rej[j]; o.R[j] = s.R[j].y; }
    }
}

__global__ __launch_bounds__(1024) void sample_walk_kernel(DevPlan p, int k_max, const int32_t *tokens, const int32_t *parents,
                                                           const float *logits, const float *draft_probs, const float2 *stats, int vocab,
                                                           float inv_t, const float *u_acc, const float *u_emit, const int32_t *next_tok,
                                                           uint32_t *err, int32_t *pend_n, int32_t *pend_a, int32_t *pend_bonus,
                                                           int32_t *pend_path, int32_t *accept_len, int32_t *emitted, int32_t *path_out,
                                                           const SampleNode *nodes) {
    __shared__ WalkState s;
    __shared__ WalkBlock w;
    __shared__ float s_part[16];
    __shared__ int s_pick, s_state[SEV_MAX_DRAFT], s_child[SEV_MAX_DRAFT];
    extern __shared__ float s_grp[];                    // [ceil(vocab / 64)] sums of 64 consecutive ids (draw pass)
    const int b = blockIdx.x, t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const int n_groups = (vocab + 63) >> 6;
    const int slot = p.req_slot[b], n = p.req_n[b], row0 = p.req_row0[b];
    const WalkIn in(logits, draft_probs, stats, u_acc, b, row0, n, k_max, vocab, inv_t);
    in.block(w, tokens + (size_t)b * k_max, parents ? parents + (size_t)b * k_max : nullptr);
    if (nodes && t < n) { s_state[t] = nodes[row0 + t].state; s_child[t] = nodes[row0 + t].child; }
    const bool vec = in.vec;
    auto current = [&](int v) { return in.current(s, v); };
    __syncthreads();
    if (t == 0) {
        s.cur = -1;
        s.a = 0;
        s.nrej = 0;
        for (int c = 0; c < n; ++c)
            if (w.par[c] == -1 && w.tk[c] == next_tok[slot]) { s.cur = c; break; }
        if (s.cur >= 0) { s.path[0] = s.cur; s.a = 1; s.child = s.cur + 1; }
        if (nodes && s.cur >= 0) {                       // as far as the nodes' own blocks have come
            while (s_state[s.cur] == NODE_ACCEPTED) {    // (a child's index is larger than its parent's)
                s.cur = s_child[s.cur];
                s.path[s.a++] = s.cur;
                s.child = s.cur + 1;
            }
            if (s_state[s.cur] == NODE_REJECTED) {      // (its first rejections)
                const SampleNode &o = nodes[row0 + s.cur];
                s.child = o.child;
                s.nrej = o.nrej;
                for (int j = 0; j < o.nrej; ++j) { s.rej[j] = o.rej[j]; s.R[j].set(o.R[j]); }
            }
        }
        if (s.cur >= 0) in.enter(s);
    }
    __syncthreads();
    int tok = next_tok[slot];
    if (s.cur >= 0) {
        for (int guard = 0; guard <= 2 * SEV_MAX_DRAFT; ++guard) {          // every round consumes a child or ends the walk
            if (t == 0) in.try_child(s, w);
            __syncthreads();
            const int action = s.action;
            if (action == 0) {
                __syncthreads();                                              // everyone has read the action before thread 0 writes the next one
                continue;
            }
            if (action == 1) {
                in.reject(s, s_part, err);
                continue;
            }
            // the draw: inverse CDF of the current distribution in token-id order.  Sums of groups of 64 consecutive ids
            // go to LDS (a wave per group, lanes = ids); wave 0 then finds the group that holds u_emit * total (every
            // lane sums a run of groups, a scan over the lanes, then that lane's groups in order) and the id inside it.
            if (vec) {
                // a wave takes 256 ids = four groups at a time, a lane four consecutive ids, 16 lanes a group
                for (int sg0 = wave; sg0 * 256 < vocab; sg0 += 16 * WALK_BATCH) {
                    float4 r[WALK_BATCH];
                    in.current4(s, sg0 * 64 + lane, 1024, r);
#pragma unroll
                    for (int u = 0; u < WALK_BATCH; ++u) {
                        const int sg = sg0 + 16 * u;
                        float x = 4 * (sg * 64 + lane) < vocab ? (r[u].x + r[u].y) + (r[u].z + r[u].w) : 0.f;
                        for (int o = 8; o > 0; o >>= 1) x += __shfl_xor(x, o);
                        const int g = sg * 4 + (lane >> 4);
                        if ((lane & 15) == 0 && g < n_groups) s_grp[g] = x;
                    }
                }
            } else {
                for (int g = wave; g < n_groups; g += 16) {
                    const int v = g * 64 + lane;
                    float r = v < vocab ? current(v) : 0.f;
                    for (int o = 32; o > 0; o >>= 1) r += __shfl_xor(r, o);
                    if (lane == 0) s_grp[g] = r;
                }
            }
            __syncthreads();
            if (wave == 0) {
                const int gpl = (n_groups + 63) >> 6;                        // groups per lane
                float ls = 0.f;
                for (int i = 0; i < gpl; ++i) {
                    const int g = lane * gpl + i;
                    ls += g < n_groups ? s_grp[g] : 0.f;
                }
                float inc = ls;                                              // inclusive scan over the lanes
                for (int o = 1; o < 64; o <<= 1) {
                    const float y = __shfl_up(inc, o);
                    if (lane >= o) inc += y;
                }
                const float target = u_emit[b] * __shfl(inc, 63);
                const unsigned long long hit = __ballot(target < inc);
                const int L = hit ? __ffsll((long long)hit) - 1 : 63;
                float cum = __shfl(inc - ls, L);                             // weight before lane L's groups
                int gsel = min((L + 1) * gpl, n_groups) - 1;
                for (int i = 0; i < gpl; ++i) {                              // uniform: every lane walks lane L's groups
                    const int g = L * gpl + i;
                    if (g >= n_groups) break;
                    const float gs = s_grp[g];
                    if (target < cum + gs) { gsel = g; break; }
                    cum += gs;
                }
                const int v = gsel * 64 + lane;
                const float w = v < vocab ? current(v) : 0.f;
                float winc = w;
                for (int o = 1; o < 64; o <<= 1) {
                    const float y = __shfl_up(winc, o);
                    if (lane >= o) winc += y;
                }
                const unsigned long long first = __ballot(target < cum + winc && w > 0.f), any = __ballot(w > 0.f);
                int pick;
                if (first) pick = gsel * 64 + __ffsll((long long)first) - 1;
                else if (any) pick = gsel * 64 + 63 - __clzll((long long)any);       // rounding at the very end: the last id with weight
                else pick = min(gsel * 64, vocab - 1);
                if (lane == 0) s_pick = pick;
            }
            __syncthreads();
            tok = s_pick;
            break;
        }
    }
    __syncthreads();
    if (t < SEV_MAX_DRAFT) pend_path[(size_t)slot * SEV_MAX_DRAFT + t] = t < s.a ? s.path[t] : -1;
    if (path_out && t < k_max) path_out[(size_t)b * k_max + t] = t < s.a ? s.path[t] : -1;
    if (t == 0) {
        const int a = s.a;
        pend_n[slot] = n;
        pend_a[slot] = a;
        pend_bonus[slot] = tok;
        accept_len[b] = a;
        emitted[b] = tok;
    }
}

void launch_sample(const sev_kv *kv, int B, int k_max, int rows, const int32_t *tokens, const int32_t *parents, const float *logits,
                   const float *draft_probs, float2 *stats, float temperature, const float *u_acc, const float *u_emit,
                   int32_t *accept_len, int32_t *emitted, int32_t *accept_path, hipStream_t st) {
    const int vocab = kv->model->d.vocab;
    const float inv_t = 1.0f / temperature;
    hipLaunchKernelGGL(softmax_stats_kernel, dim3(rows), dim3(1024), 0, st, logits, vocab, inv_t, stats);
    if (parents)
        hipLaunchKernelGGL(sample_nodes_kernel, dim3(rows), dim3(1024), 0, st, kv->plan, k_max, tokens, parents, logits, draft_probs, stats, vocab, inv_t, u_acc,
                           kv->sample_nodes);
    hipLaunchKernelGGL(sample_walk_kernel, dim3(B), dim3(1024), (size_t)((vocab + 63) / 64) * 4, st, kv->plan, k_max, tokens, parents, logits, draft_probs, stats, vocab,
                       inv_t, u_acc, u_emit, kv->next_tok, kv->err_flags, kv->pend_n, kv->pend_a, kv->pend_bonus, kv->pend_path, accept_len,
                       emitted, accept_path, parents ? kv->sample_nodes : nullptr);
}

KvGeom sev_kv_geom(const sev_kv *kv);

void launch_commit(const sev_kv *kv, const int32_t *slots, int B, bool rollback, hipStream_t st) {
    SlotList sl;
    for (int b = 0; b < B; ++b) sl.s[b] = slots ? slots[b] : b;
    KvGeom g = sev_kv_geom(kv);
    // accepted candidates of a chain are in place already (candidate j sits at position P + j): only trees may have to move
    // (a captured commit may be replayed after any block)
    bool trees = !rollback && sev_capturing(st);
    for (int b = 0; b < B; ++b) trees |= kv->host_tree[sl.s[b]] != 0;
    if (!rollback && trees) {
        const int n = g.L * g.Hkv * g.hd;
        dim3 grid((n + 255) / 256, B);
        if (kv->model->d.dtype == SEV_BF16)
            hipLaunchKernelGGL((commit_copy_kernel<uint16_t, true>), grid, dim3(256), 0, st, sl, g, kv->page_table,
                               kv->max_pages_per_req, kv->pend_n, kv->pend_a, kv->pend_P, kv->pend_path);
        else
            hipLaunchKernelGGL((commit_copy_kernel<float, false>), grid, dim3(256), 0, st, sl, g, kv->page_table,
                               kv->max_pages_per_req, kv->pend_n, kv->pend_a, kv->pend_P, kv->pend_path);
    }
    hipLaunchKernelGGL(commit_state_kernel, dim3((B + 63) / 64), dim3(64), 0, st, sl, B, rollback ? 1 : 0, kv->seq_len,
                       kv->next_tok, kv->pend_n, kv->pend_a, kv->pend_bonus);
}

// ---------------------------------------------------------------------------
// cache import / export: plain [n][Hkv][hd] <-> paged layout
// ---------------------------------------------------------------------------
template <typename T, bool BF16>
__global__ void kv_copy_kernel(KvGeom g, const int32_t *pt, int layer, int start, int n, T *k, T *v, int to_cache) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = (int64_t)n * g.Hkv * g.hd;
    if (idx >= total) return;
    const int e = (int)(idx % g.hd), h = (int)((idx / g.hd) % g.Hkv), t = (int)(idx / ((int64_t)g.hd * g.Hkv));
    const int tok = start + t;
    const size_t blk = (size_t)SEV_PAGE * g.hd;
    const size_t pb = ((size_t)pt[tok / SEV_PAGE] * g.Hkv + h) * blk;
    T *kp = (T *)(g.pool + (size_t)layer * g.layer_stride) + pb + k_in_page<BF16>(tok % SEV_PAGE, e, g.hd);
    T *vp = (T *)(g.pool + (size_t)layer * g.layer_stride + g.v_offset) + pb + v_in_page<BF16>(tok % SEV_PAGE, e, g.hd);
    if (to_cache) { *kp = k[idx]; *vp = v[idx]; }
    else { k[idx] = *kp; v[idx] = *vp; }
}

void launch_kv_copy(const sev_kv *kv, int slot, int layer, int start, int n, void *k, void *v, int to_cache,
                    hipStream_t st) {
    KvGeom g = sev_kv_geom(kv);
    const int64_t total = (int64_t)n * g.Hkv * g.hd;
    if (total == 0) return;
    const int32_t *pt = kv->page_table + (size_t)slot * kv->max_pages_per_req;
    dim3 grid((unsigned)((total + 255) / 256));
    if (kv->model->d.dtype == SEV_BF16)
        hipLaunchKernelGGL((kv_copy_kernel<uint16_t, true>), grid, dim3(256), 0, st, g, pt, layer, start, n,
                           (uint16_t *)k, (uint16_t *)v, to_cache);
    else
        hipLaunchKernelGGL((kv_copy_kernel<float, false>), grid, dim3(256), 0, st, g, pt, layer, start, n, (float *)k,
                           (float *)v, to_cache);
}

// ---------------------------------------------------------------------------
// row-wise arg-max over materialised logits (lowest index wins ties)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void argmax_rows_kernel(const float *logits, int vocab, int32_t *out) {
    __shared__ float sv[256];
    __shared__ int si[256];
    const float *row = logits + (size_t)blockIdx.x * vocab;
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    for (int i = threadIdx.x; i < vocab; i += 256) {
        const float v = row[i];
        if (v > bv || (v == bv && i < bi)) { bv = v; bi = i; }
    }
    sv[threadIdx.x] = bv;
    si[threadIdx.x] = bi;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            const float v = sv[threadIdx.x + s];
            const int i = si[threadIdx.x + s];
            if (v > sv[threadIdx.x] || (v == sv[threadIdx.x] && i < si[threadIdx.x])) { sv[threadIdx.x] = v; si[threadIdx.x] = i; }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = si[0];
}

void launch_argmax_rows_f32(const float *logits, int rows, int vocab, int32_t *out, hipStream_t st) {
    hipLaunchKernelGGL(argmax_rows_kernel, dim3(rows), dim3(256), 0, st, logits, vocab, out);
}
