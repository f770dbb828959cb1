// float32 path: straightforward kernels for float32 models.  Every step of the forward pass
// (embedding, RMSNorm, projections, rotary embedding + cache append, masked attention over the
// paged cache, SwiGLU, output head) is computed here in float32 with plain FMA arithmetic.
#include "sev_internal.h"
#include "kv_layout.h"

KvGeom sev_kv_geom(const sev_kv *kv);

__global__ void copy_f32_kernel(float *dst, const float *src, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}
void launch_pack_f32(float *dst, const float *src, int64_t n, hipStream_t st) {
    if (n > 0) hipLaunchKernelGGL(copy_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, dst, src, n);
}

// ---------------------------------------------------------------------------
// Y[m][c] = sum_k X[m][k] * W[c][k], with the norm in front and the stage behind it fused in.
//
// Up to 16 rows a wave owns P column PAIRS x all R rows and splits K over its lanes (16 bytes per lane and matrix row), so nothing goes
// through LDS and no barrier is needed; the 64 partial sums are then folded by exchanging halves (an accumulator array of
// V values takes V - 1 exchanges instead of 6 V) and every group of 64 / V lanes ends up with one finished pair.  A pair
// is what the following stage has to see together: the two halves of a rotary pair, gate and up of one feed-forward
// column, or just two neighbouring columns.
//
// What binds it at the sizes this path is for (a few rows, K of a few hundred) is latency and the number of launches: K
// is one to three loads deep per lane, all in flight at once, and the norm (its sum of squares is a by-product of reading
// X), rotary embedding, cache append, SwiGLU and residual addition cost no launch of their own.  The kernel before it
// took K in steps of 32 through LDS, two barriers each, with N / 64 blocks: O and down (N = 256) ran on 4 blocks and took
// 38 us on average with K = 256 and 688 and four rows; 3.5 us now.  One request, 4 candidates: 548 -> 76 us a step.
// ---------------------------------------------------------------------------
enum { F32_PLAIN = 0, F32_RESID, F32_SWIGLU, F32_QKV };

struct GemmF32 {
    const float *X, *W, *gain;       // gain: RMS norm of X in front (its gains), or null
    float *Y;
    int M, K, N, n_pairs;            // N: row stride of Y
    float inv_k, eps;
    // F32_QKV
    const float2 *row_cs;
    const int32_t *row_kvloc;
    float *k_layer, *v_layer;
    int hd, Hq, Hkv;
};

// columns of pair j
template <int EPI>
__device__ __forceinline__ void f32_cols(const GemmF32 &g, int j, int &c0, int &c1) {
    if constexpr (EPI == F32_SWIGLU) { c0 = j; c1 = g.n_pairs + j; }
    else if constexpr (EPI == F32_QKV) { const int half = g.hd >> 1, head = j / half; c0 = head * g.hd + j - head * half; c1 = c0 + half; }
    else { c0 = 2 * j; c1 = min(2 * j + 1, g.N - 1); }
}

// what happens to the finished pair j of row m
template <int EPI>
__device__ __forceinline__ void f32_finish(const GemmF32 &g, int m, int j, float va, float vb) {
    int c0, c1;
    f32_cols<EPI>(g, j, c0, c1);
    float *y = g.Y + (size_t)m * g.N;
    if constexpr (EPI == F32_SWIGLU) {
        y[j] = va / (1.0f + expf(-va)) * vb;
    } else if constexpr (EPI == F32_QKV) {
        // rotary embedding of q and k; k and v go to the paged cache at position P + node
        const int half = g.hd >> 1, head = j / half, i = j - head * half;
        if (head < g.Hq + g.Hkv) {
            const float2 cs = g.row_cs[(size_t)m * half + i];
            const float t = va * cs.x - vb * cs.y;
            vb = vb * cs.x + va * cs.y;
            va = t;
        }
        if (head < g.Hq) {
            y[c0] = va;
            y[c1] = vb;
        } else {
            const bool is_k = head < g.Hq + g.Hkv;
            const int loc = g.row_kvloc[m], h = head - g.Hq - (is_k ? 0 : g.Hkv);
            float *c = (is_k ? g.k_layer : g.v_layer) + (((size_t)(loc >> 4) * g.Hkv + h) * SEV_PAGE + (loc & 15)) * g.hd + i;
            c[0] = va;
            c[half] = vb;
        }
    } else if constexpr (EPI == F32_RESID) {
        y[c0] += va;
        if (c1 != c0) y[c1] += vb;
    } else {
        y[c0] = va;
        if (c1 != c0) y[c1] = vb;
    }
}

// Sum over the wave of V values per lane: lane ends up with value lane / (64 / V).
template <int V>
__device__ __forceinline__ float wave_sum_split(float (&a)[V], int lane) {
    int off = 32;
#pragma unroll
    for (int cnt = V; cnt > 1; cnt >>= 1, off >>= 1) {
        const bool up = lane & off;
#pragma unroll
        for (int i = 0; i < V / 2; ++i)
            if (i < cnt / 2) {
                const float keep = up ? a[i + cnt / 2] : a[i], send = up ? a[i] : a[i + cnt / 2];
                a[i] = keep + __shfl_xor(send, off);
            }
    }
    for (; off > 0; off >>= 1) a[0] += __shfl_xor(a[0], off);
    return a[0];
}

template <int R, int P, int EPI, bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmF32 g) {
    constexpr int V = R * P, E = VEC ? 4 : 1;
    const int lane = threadIdx.x & 63;
    const int pair0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * P;
    if (pair0 >= g.n_pairs) return;                           // (no barrier in this kernel)
    const float *w0[P], *w1[P], *x[R];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        int c0, c1;
        f32_cols<EPI>(g, min(pair0 + p, g.n_pairs - 1), c0, c1);
        w0[p] = g.W + (size_t)c0 * g.K;
        w1[p] = g.W + (size_t)c1 * g.K;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = g.X + (size_t)min(r, g.M - 1) * g.K;
    float a0[V], a1[V], ss[R];
#pragma unroll
    for (int i = 0; i < V; ++i) a0[i] = a1[i] = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) ss[r] = 0.f;
    auto load = [&](const float *p, float (&v)[E]) {
        if constexpr (VEC) {
            const float4 q = *(const float4 *)p;
            v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
        } else v[0] = *p;
    };
    const bool norm = g.gain != nullptr;
#pragma unroll (R * P <= 8 ? 2 : 1)
    for (int k = lane * E; k < g.K; k += 64 * E) {            // (VEC: K is a multiple of 4)
        float wa[P][E], wb[P][E], gn[E];
#pragma unroll
        for (int p = 0; p < P; ++p) { load(w0[p] + k, wa[p]); load(w1[p] + k, wb[p]); }
        if (norm) load(g.gain + k, gn);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float xv[E];
            load(x[r] + k, xv);
            if (norm) {
#pragma unroll
                for (int e = 0; e < E; ++e) { ss[r] += xv[e] * xv[e]; xv[e] *= gn[e]; }
            }
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    a0[p * R + r] += xv[e] * wa[p][e];
                    a1[p * R + r] += xv[e] * wb[p][e];
                }
        }
    }
    float va = wave_sum_split<V>(a0, lane), vb = wave_sum_split<V>(a1, lane);
    constexpr int LPV = 64 / V;
    const int idx = lane / LPV, p = idx / R, m = idx - p * R, j = pair0 + p;
    if (norm) {
        float sq[V];                                          // the same fold, so that every lane ends with its own row's sum
#pragma unroll
        for (int i = 0; i < V; ++i) sq[i] = ss[i % R];
        const float rs = 1.0f / sqrtf(wave_sum_split<V>(sq, lane) * g.inv_k + g.eps);
        va *= rs;
        vb *= rs;
    }
    if (lane % LPV || m >= g.M || j >= g.n_pairs) return;
    f32_finish<EPI>(g, m, j, va, vb);
}

// The same for more than 16 rows, where the kernel above would read each matrix row from the caches once per 16 rows of X,
// which bound it: a block of 256 threads owns 16 pairs x 16 R rows, stages K in steps of 32 through LDS (the next step's
// loads in flight behind the products of this one) and a thread keeps one pair of R rows.  Sums run over 8 products each
// (four of them per value and step), are folded once a step and added to a total that carries its rounding errors along, so
// that the logits are no further from a 64-bit forward than with the kernel above (2.0e-7 of their norm with K = 256 and 688
// in both; 2.0e-7 against 2.9e-7 with K = 2048 and 5504).  A step of the two-layer 256-wide shape with the kernel above and
// with this one: 64 rows 217 -> 133 us, 256 rows 581 -> 141, 1024 rows 1809 -> 196.
template <int R, int EPI, bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_tile_kernel(GemmF32 g) {
    constexpr int TM = 16 * R, KS = 32, LD = KS + 4, NX = R / 2;      // LD: rows stay 16-byte aligned and spread over the banks
    static_assert(R % 2 == 0, "a step of X must be a whole number of 16 bytes per thread");
    __shared__ float4 Ws[32 * LD / 4], Xs[TM * LD / 4];
    __shared__ float s_ss[TM];
    const int t = threadIdx.x, lr = t >> 3, lk = (t & 7) * 4;          // loads: matrix row, place in the K step
    const int pl = t & 15, rl = t >> 4;                                // products: pair, row
    const int pair0 = blockIdx.x * 16, m0 = blockIdx.y * TM;
    int c0, c1;
    f32_cols<EPI>(g, min(pair0 + (lr & 15), g.n_pairs - 1), c0, c1);
    const float *w = g.W + (size_t)(lr < 16 ? c0 : c1) * g.K, *x[NX];
#pragma unroll
    for (int i = 0; i < NX; ++i) x[i] = g.X + (size_t)min(m0 + lr + 32 * i, g.M - 1) * g.K;
    const bool norm = g.gain != nullptr;
    auto load = [&](const float *p, int k) {                           // past the end: zeros
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (VEC) {
            if (k < g.K) v = *(const float4 *)(p + k);
        } else {
            if (k < g.K) v.x = p[k];
            if (k + 1 < g.K) v.y = p[k + 1];
            if (k + 2 < g.K) v.z = p[k + 2];
            if (k + 3 < g.K) v.w = p[k + 3];
        }
        return v;
    };
    auto add = [](float &sum, float &err, float v) {                   // sum + v, its rounding error kept for the next one
        const float y = v - err, s = sum + y, e = (s - sum) - y;
        err = fabsf(e) < INFINITY ? e : 0.f;                           // an infinite sum has none (and would turn to NaN with one)
        sum = s;
    };
    float ss[NX], ss_err[NX], a0[R], a1[R], e0[R], e1[R];
#pragma unroll
    for (int i = 0; i < NX; ++i) ss[i] = ss_err[i] = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) a0[r] = a1[r] = e0[r] = e1[r] = 0.f;
    float4 wn = load(w, lk), xn[NX], gn = make_float4(1.f, 1.f, 1.f, 1.f);
#pragma unroll
    for (int i = 0; i < NX; ++i) xn[i] = load(x[i], lk);
    if (norm) gn = load(g.gain, lk);
    for (int k0 = 0; k0 < g.K; k0 += KS) {
        Ws[(lr * LD + lk) / 4] = wn;
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            float4 v = xn[i];
            if (norm) {
                add(ss[i], ss_err[i], (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w));
                v = make_float4(v.x * gn.x, v.y * gn.y, v.z * gn.z, v.w * gn.w);
            }
            Xs[((lr + 32 * i) * LD + lk) / 4] = v;
        }
        __syncthreads();
        if (k0 + KS < g.K) {
            wn = load(w, k0 + KS + lk);
#pragma unroll
            for (int i = 0; i < NX; ++i) xn[i] = load(x[i], k0 + KS + lk);
            if (norm) gn = load(g.gain, k0 + KS + lk);
        }
        float4 p0[R], p1[R];
#pragma unroll
        for (int r = 0; r < R; ++r) p0[r] = p1[r] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int k = 0; k < KS; k += 4) {
            const float4 wa = Ws[(pl * LD + k) / 4], wb = Ws[((16 + pl) * LD + k) / 4];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float4 v = Xs[((rl + 16 * r) * LD + k) / 4];
                p0[r].x += v.x * wa.x; p0[r].y += v.y * wa.y; p0[r].z += v.z * wa.z; p0[r].w += v.w * wa.w;
                p1[r].x += v.x * wb.x; p1[r].y += v.y * wb.y; p1[r].z += v.z * wb.z; p1[r].w += v.w * wb.w;
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            add(a0[r], e0[r], (p0[r].x + p0[r].y) + (p0[r].z + p0[r].w));
            add(a1[r], e1[r], (p1[r].x + p1[r].y) + (p1[r].z + p1[r].w));
        }
        __syncthreads();                                               // the next step overwrites the tiles
    }
    if (norm) {
#pragma unroll
        for (int i = 0; i < NX; ++i) {
#pragma unroll
            for (int o = 1; o < 8; o <<= 1) ss[i] += __shfl_xor(ss[i], o);
            if ((t & 7) == 0) s_ss[lr + 32 * i] = ss[i];
        }
        __syncthreads();
    }
    const int j = pair0 + pl;
    if (j >= g.n_pairs) return;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int m = m0 + rl + 16 * r;
        if (m >= g.M) continue;
        const float rs = norm ? 1.0f / sqrtf(s_ss[rl + 16 * r] * g.inv_k + g.eps) : 1.0f;
        f32_finish<EPI>(g, m, j, a0[r] * rs, a1[r] * rs);
    }
}

template <int EPI>
static void gemm_f32(GemmF32 g, hipStream_t st) {
    const bool vec = g.K % 4 == 0;       // matrices start on 256 bytes (or a multiple of K values behind that), so every row is 16-byte aligned then
    // From 17 rows on the blocks of the tile kernel: a step of 16 rows takes 131 us with either (two-layer 256-wide shape), of
    // 32 rows 137 and 132, of 128 rows 335 and 136; with matrices eight times as wide 16 rows take 664 and 783, 32 rows 1026
    // and 805.  64 rows per block (half the reads of W) where those still give every compute unit one.
    if (g.M > 16) {
        const unsigned pb = (unsigned)((g.n_pairs + 15) / 16);
        const bool tall = (int64_t)pb * ((g.M + 63) / 64) >= 256;
        const dim3 grid(pb, (unsigned)((g.M + (tall ? 63 : 31)) / (tall ? 64 : 32)));
        if (tall && vec) hipLaunchKernelGGL((gemm_f32_tile_kernel<4, EPI, true>), grid, dim3(256), 0, st, g);
        else if (tall) hipLaunchKernelGGL((gemm_f32_tile_kernel<4, EPI, false>), grid, dim3(256), 0, st, g);
        else if (vec) hipLaunchKernelGGL((gemm_f32_tile_kernel<2, EPI, true>), grid, dim3(256), 0, st, g);
        else hipLaunchKernelGGL((gemm_f32_tile_kernel<2, EPI, false>), grid, dim3(256), 0, st, g);
        return;
    }
    // rows of a wave: all of them; two pairs per wave (half the reads of X) only where there are waves enough without them
    // (4 per compute unit)
    const int R = g.M <= 4 ? 4 : (g.M <= 8 ? 8 : 16);
    const int P = R == 16 && g.n_pairs >= 2048 ? 2 : 1;
    const dim3 grid((unsigned)((g.n_pairs + 4 * P - 1) / (4 * P)));
#define SEV_F32_LAUNCH(R_, P_)                                                                                                \
    do {                                                                                                                      \
        if (vec) hipLaunchKernelGGL((gemm_f32_kernel<R_, P_, EPI, true>), grid, dim3(256), 0, st, g);                         \
        else hipLaunchKernelGGL((gemm_f32_kernel<R_, P_, EPI, false>), grid, dim3(256), 0, st, g);                            \
    } while (0)
    if (R == 4) SEV_F32_LAUNCH(4, 1);
    else if (R == 8) SEV_F32_LAUNCH(8, 1);
    else if (P == 1) SEV_F32_LAUNCH(16, 1);
    else SEV_F32_LAUNCH(16, 2);
#undef SEV_F32_LAUNCH
}

// ---------------------------------------------------------------------------
// Masked attention of one (row, query head) per block over the request's paged cache: all prefix positions, plus the
// block's nodes that are ancestors-or-self of the row's node (chains: the nodes up to the row's own, whatever the length).
//
// LPK lanes share a key (four of its dims each), so a block walks 256 / LPK keys at a time with an online softmax per lane
// group; the groups meet once, at the end, in LDS.  Four keys of a group are in flight together.  Latency binds it (a
// prefix of 64 is one round of loads).  One wave per (row, head) that took the keys one after the other needed 0.7 us per
// key: 46.6 us at 68 positions, 6.4 us now (8 chains of 16 on prefixes of 100 to 1000: a step of 2135 us, now 386).
// ---------------------------------------------------------------------------
template <int LPK, bool VEC>
__global__ __launch_bounds__(256) void attn_f32_kernel(const float *qkv, float *out, DevPlan p, const float *Kl, const float *Vl, int Hkv, int hd,
                                                       const int32_t *page_table, int max_pages, int Hq, int n_qkv, float scale) {
    constexpr int NG = 256 / LPK, U = 4;
    __shared__ float s_m[NG], s_l[NG], s_o[NG * LPK * 4];
    const int m = blockIdx.x, j = blockIdx.y, e = threadIdx.x % LPK, gid = threadIdx.x / LPK;
    const int b = p.row_req[m], P = p.req_P[b], n = p.req_n[b], slot = p.req_slot[b];
    const unsigned long long anc = p.row_anc[m];
    const int node = p.row_node[m];
    const int h = (j * Hkv) / Hq;
    const int32_t *pt = page_table + (size_t)slot * max_pages;
    const int d0 = 4 * e;
    auto load = [&](const float *v, float (&o)[4]) {
        if constexpr (VEC) {
            const float4 q = d0 < hd ? *(const float4 *)(v + d0) : make_float4(0.f, 0.f, 0.f, 0.f);
            o[0] = q.x; o[1] = q.y; o[2] = q.z; o[3] = q.w;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = d0 + i < hd ? v[d0 + i] : 0.f;
        }
    };
    float q[4], acc[4] = {0.f, 0.f, 0.f, 0.f};
    load(qkv + (size_t)m * n_qkv + j * hd, q);
    float mx = -INFINITY, den = 0.f;
    const int T = p.causal ? P + node + 1 : P + n;
    for (int t0 = gid; t0 < T; t0 += NG * U) {
        float kf[U][4], vf[U][4], s[U];
        bool vis[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = t0 + u * NG, tc = min(t, T - 1);
            vis[u] = t < T && (p.causal || t < P || ((anc >> (t - P)) & 1ull));
            const size_t at = (((size_t)pt[tc / SEV_PAGE] * Hkv + h) * SEV_PAGE + tc % SEV_PAGE) * hd;
            load(Kl + at, kf[u]);
            load(Vl + at, vf[u]);
        }
        float mn = mx;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float d = (q[0] * kf[u][0] + q[1] * kf[u][1]) + (q[2] * kf[u][2] + q[3] * kf[u][3]);
#pragma unroll
            for (int o = LPK / 2; o > 0; o >>= 1) d += __shfl_xor(d, o);
            s[u] = d * scale;
            if (vis[u]) mn = fmaxf(mn, s[u]);
        }
        const float base = mn == -INFINITY ? 0.f : mn, corr = expf(mx - base);
        den *= corr;
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] *= corr;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float pe = vis[u] ? expf(s[u] - base) : 0.f;
            den += pe;
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] += vis[u] ? pe * vf[u][i] : 0.f;
        }
        mx = mn;
    }
    if (e == 0) { s_m[gid] = mx; s_l[gid] = den; }
#pragma unroll
    for (int i = 0; i < 4; ++i) s_o[(gid * LPK + e) * 4 + i] = acc[i];
    __syncthreads();
    float top = -INFINITY;                                    // every row sees itself: some group has a finite maximum
#pragma unroll
    for (int g = 0; g < NG; ++g) top = fmaxf(top, s_m[g]);
    if ((int)threadIdx.x < hd) {
        float l = 0.f, o = 0.f;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const float w = expf(s_m[g] - top);
            l += w * s_l[g];
            o += w * s_o[g * LPK * 4 + threadIdx.x];
        }
        out[(size_t)m * (Hq * hd) + j * hd + threadIdx.x] = o / l;
    }
}

static void attn_f32(const sev_model *m, sev_kv *kv, int rows, int layer, hipStream_t st) {
    const sev_model_desc &d = m->d;
    const KvGeom g = sev_kv_geom(kv);
    const float *K = (const float *)(g.pool + (size_t)layer * g.layer_stride), *V = (const float *)((const char *)K + g.v_offset);
    const float scale = 1.0f / sqrtf((float)d.head_dim);
    const bool vec = d.head_dim % 4 == 0;
#define SEV_ATTN_F32(LPK_)                                                                                                    \
    do {                                                                                                                      \
        if (vec) hipLaunchKernelGGL((attn_f32_kernel<LPK_, true>), dim3(rows, d.n_q_heads), dim3(256), 0, st, (const float *)kv->q_buf, (float *)kv->o_buf,  \
                                    kv->plan, K, V, d.n_kv_heads, d.head_dim, kv->page_table, kv->max_pages_per_req, d.n_q_heads, m->n_qkv, scale);       \
        else hipLaunchKernelGGL((attn_f32_kernel<LPK_, false>), dim3(rows, d.n_q_heads), dim3(256), 0, st, (const float *)kv->q_buf, (float *)kv->o_buf,      \
                                kv->plan, K, V, d.n_kv_heads, d.head_dim, kv->page_table, kv->max_pages_per_req, d.n_q_heads, m->n_qkv, scale);           \
    } while (0)
    if (d.head_dim <= 32) SEV_ATTN_F32(8);
    else if (d.head_dim <= 64) SEV_ATTN_F32(16);
    else if (d.head_dim <= 128) SEV_ATTN_F32(32);
    else SEV_ATTN_F32(64);
#undef SEV_ATTN_F32
}

void f32_forward(const sev_model *m, sev_kv *kv, int rows, int B, float *logits_out, HeadOut *head, hipStream_t st) {
    (void)B;
    const sev_model_desc &d = m->d;
    const KvGeom geo = sev_kv_geom(kv);
    auto W = [&](size_t off) { return (const float *)(m->arena + off); };
    float *h = kv->h, *qkv = (float *)kv->q_buf, *ob = (float *)kv->o_buf, *act = (float *)kv->act;
    // X [rows][K] (normed in front where there are gains) times W, n_pairs column pairs, into rows of N
    auto gemm = [&](const float *X, const float *gain, const float *Wm, float *Y, int N, int n_pairs, int K) {
        GemmF32 g = {};
        g.X = X; g.W = Wm; g.gain = gain; g.Y = Y;
        g.M = rows; g.K = K; g.N = N; g.n_pairs = n_pairs;
        g.inv_k = 1.0f / (float)K; g.eps = d.rms_eps;
        return g;
    };
    for (int l = 0; l < d.n_layers; ++l) {
        const LayerOffsets &lo = m->layers[l];
        GemmF32 q = gemm(h, W(lo.g_attn), W(lo.wqkv), qkv, m->n_qkv, m->n_qkv / 2, d.d_model);
        q.row_cs = kv->plan.row_cs; q.row_kvloc = kv->plan.row_kvloc;
        q.k_layer = (float *)(geo.pool + (size_t)l * geo.layer_stride);
        q.v_layer = (float *)(geo.pool + (size_t)l * geo.layer_stride + geo.v_offset);
        q.hd = d.head_dim; q.Hq = d.n_q_heads; q.Hkv = d.n_kv_heads;
        gemm_f32<F32_QKV>(q, st);
        attn_f32(m, kv, rows, l, st);
        gemm_f32<F32_RESID>(gemm(ob, nullptr, W(lo.wo), h, d.d_model, (d.d_model + 1) / 2, m->q_dim), st);
        gemm_f32<F32_SWIGLU>(gemm(h, W(lo.g_ffn), W(lo.wgu), act, d.d_ffn, d.d_ffn, d.d_model), st);
        gemm_f32<F32_RESID>(gemm(act, nullptr, W(lo.wd), h, d.d_model, (d.d_model + 1) / 2, d.d_ffn), st);
    }
    float *lg = logits_out ? logits_out : kv->logits_f32;
    gemm_f32<F32_PLAIN>(gemm(h, W(m->off_gfinal), W(m->off_lm), lg, d.vocab, (d.vocab + 1) / 2, d.d_model), st);
    // a request's block of the acceptance reads its rows by itself where they are short (a kernel less); longer ones want more blocks
    if (head && d.vocab <= 4096) {
        *head = {HEAD_LOGITS, nullptr, lg, nullptr, d.vocab, 0};
        return;
    }
    launch_argmax_rows_f32(lg, rows, d.vocab, kv->row_argmax, st);
    if (head) *head = {HEAD_ROWS, kv->row_argmax, nullptr, nullptr, 0, 0};
}
