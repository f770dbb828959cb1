// bfloat16 path for gfx950: matrix-core GEMMs that stream re-tiled bf16 weights once per step,
// paged-KV verification attention, and the fused element-wise stages between them.
//
// Precision recipe.  Weights and the KV cache are bf16.  Every activation that feeds a matrix
// core is carried as TWO bf16 planes, hi = bf16(x) and lo = bf16(x - hi), and multiplied in two
// MFMAs that accumulate into the same float32 registers; the residual stream, norms, rotary
// embedding, softmax and all accumulations are float32.  (A single bf16 plane per activation
// accumulates ~3 % relative error over 32 layers; the split keeps it near 1e-5.)
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <math.h>

#include <algorithm>
#include <iterator>
#include <type_traits>

#include "sev_internal.h"
#include "kv_layout.h"
#include "row_ops.h"

KvGeom sev_kv_geom(const sev_kv *kv);

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // native 16-byte vector (keeps staging arrays in registers)

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;          // round to nearest even (finite inputs)
}

// hi/lo split of one float: hi = bf16(x), lo = bf16(x - hi)
__device__ __forceinline__ void split_bf16(float x, uint32_t &hi, uint32_t &lo) {
    hi = f32_to_bf16_bits(x);
    lo = f32_to_bf16_bits(x - bf16_bits_to_f32(hi));
}

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// ---------------------------------------------------------------------------
// weight re-tiling: canonical [rows][K] bf16 -> [tile of 32 rows][K/32][fragment 2][lane 64][8], where lane l of fragment f
// holds W[16 f + l % 16][8 (l / 16) .. + 7 of the k-step]: exactly the A operand of a 16x16x32 MFMA.
//
// mode 0: source tile t lands at destination tile t + tile_add (plain, or a row range of a fused matrix).
// mode 1 / 2 (gate / up of the SwiGLU pair): destination tile t holds feed-forward columns
// [16t, 16t+16) of BOTH matrices, the gate in fragment 0 and up in fragment 1, so that an MFMA output lane owns the
// gate and the up value of the same 4 columns.
// mode 3 (q, k, v projections, head_dim 128): the same inside every head, with the two
// halves of the head in the roles of gate and up: tile 4*head + t holds the head's dims 16t .. 16t+15 and those dims + 64,
// so that a lane owns both members of a rotary pair (i, i + 64).
// ---------------------------------------------------------------------------
__global__ void pack_bf16_kernel(uint4 *dst, const uint16_t *src, int K, int64_t n_chunks, int mode, int tile_add) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n_chunks) return;
    const int ksteps = K >> 5;
    const int lane = (int)(c & 63), f = (int)(c >> 6) & 1;
    const int64_t tk = c >> 7;
    const int kt = (int)(tk % ksteps);
    const int64_t t = tk / ksteps;                   // destination tile
    const int n = lane & 15;
    const int k = kt * 32 + 8 * (lane >> 4);
    int64_t row;
    if (mode == 0) {
        row = (t - tile_add) * 32 + 16 * f + n;
    } else if (mode == 3) {
        const int64_t tt = t - tile_add;
        row = (tt >> 2) * 128 + f * 64 + (tt & 3) * 16 + n;
    } else {
        if (f != mode - 1) return;                   // this launch fills only its own fragments
        row = t * 16 + n;
    }
    dst[c] = *(const uint4 *)(src + row * K + k);
}

// n_rows source rows.  modes 0, 3: destination tiles tile_add .. tile_add + n_rows/32 - 1;
// modes 1, 2: destination tiles 0 .. n_rows/16 - 1.
void launch_pack_bf16(uint16_t *dst, const uint16_t *src, int n_rows, int K, int mode, int tile_add, hipStream_t st) {
    const bool whole = mode == 0 || mode == 3;
    const int64_t tiles = whole ? n_rows / 32 : n_rows / 16;
    const int64_t n_chunks = tiles * (K / 32) * 128;
    uint4 *d = (uint4 *)dst + (whole ? (int64_t)tile_add * (K / 32) * 128 : 0);
    hipLaunchKernelGGL(pack_bf16_kernel, dim3((unsigned)((n_chunks + 255) / 256)), dim3(256), 0, st, d, src, K, n_chunks,
                       mode, 0);
}

// ---------------------------------------------------------------------------
// skinny-M GEMM on the matrix cores:  Y[M][N] = X[M][K] * W[N][K]^T, with the stage that follows
// the GEMM fused into its epilogue.
//
// A block of 4 waves covers MR row units of 16 (up to 160 rows) and 4*NT column tiles of 32; wave w owns NT column tiles.
// Weights go global -> registers, one fully coalesced 1 KiB fragment per load, PF stages ahead; each weight byte is read
// once per row block.  Activations (hi and lo planes, already in fragment order) go global -> LDS once per block and are
// shared by the 4 waves.
// MFMA 16x16x32: A = 16 columns of a weight tile (fragment 0 or 1 of it, 32 k), B = activation unit (32 k x 16 rows), so a
// lane ends up with 4 consecutive output columns of one row per register quad.
//
// Matrix work of this chip is bound by its power: 32x32x16 on random hi/lo operands sustains 1.75-1.83 PFLOP/s (at 1.76 GHz),
// 16x16x32 with the two planes of a product back to back on the same accumulators 2.11-2.15 (at 2.1 GHz; the second product
// moves only the low bits of sums that the first has just read).  The same with the planes apart: 1.95-2.0.
// grid: 1-D over (column group, split-K slice, row block of MR units); see the block index decode.
//
// Split-K.  With S = 1 the block runs the epilogue itself.  With S > 1 it stores its accumulators
// in register order (coalesced 1 KiB stores, layout [slice][column tile][row unit][fragment]) and gemm_fixup_kernel,
// one wave per 32 columns x 16 rows, adds the S slices in slice order and runs the same epilogue code.
//
// Normalisation.  RMSNorm scales row m by r[m] = 1/rms(h[m]) and column k by the gain g[k].  The
// producer of an activation matrix writes split(h * g) and the rows' sums of squares; the
// consuming GEMM multiplies its accumulators by r[m] (the scale commutes with the contraction).
//
// Epilogues (per 32 columns x 16 rows):
//   EPI_QKV    rotary embedding of q and k (weight rows of every head are interleaved so that a
//              lane holds both members of 4 rotary pairs), q -> hi/lo planes for the attention
//              kernel, k and v -> bf16 into the paged cache at position P + node
//   EPI_RESID  h += Y; xout = split(h * gain); adds the tile's sums of squares to ssq_out and
//              clears the buffer the next producer will add to
//   EPI_SWIGLU act = split(silu(gate) * up), gate and up rows interleaved in the weight tiles
//   EPI_ARGMAX arg-max of every row over the block's columns (+ optional float32 logits); never split
// ---------------------------------------------------------------------------
// A pipeline stage is KS steps of 32 k.  An odd number of units does not fill whole loads of 256 threads: narrow blocks take two k-steps
// per stage; in wide ones, whose registers that would not fit, half of the threads have no part in the stage's last load.
__host__ __device__ constexpr int gemm_ks(int MR, int NT) { return MR % 2 && NT <= 2 ? 2 : 1; }

enum { EPI_QKV = 0, EPI_SWIGLU = 1, EPI_ARGMAX = 2, EPI_RESID = 3 };

struct GemmArgs {
    const uint4 *W;          // re-tiled weights
    const uint4 *X;          // xpack activations
    int n_tiles, k_steps, units_total, M, N;      // k_steps of 32; units_total: row units of the operand buffers
    int col_groups, m_blocks, splits;   // grid decomposition (see the kernel's block index decode)
    float *part;             // split-K exchange: [S][column tile][row unit][2][64 lanes] float4
    const unsigned long long *ssq_in;   // [rows] sums of squares of the input rows, or null (input is not a normed stream)
    float inv_d, eps;
    // EPI_RESID
    float *h;                // residual stream [M][N]
    const float *gain;       // gains of the norm that follows
    uint16_t *xout;          // xpack (K = N) of h * gain
    unsigned long long *ssq_out, *ssq_clear;   // [rows]
    // EPI_SWIGLU
    uint16_t *act;           // xpack with K = N/2 (N counts gate and up rows)
    // EPI_QKV
    const float2 *row_cs;    // [rows][64] (cos, sin)
    const int32_t *row_kvloc; // [rows] physical page * 16 + token in page of the row's cache position
    int Hq, Hkv;
    char *k_layer;           // K pages of this layer; V pages follow at v_offset
    size_t v_offset;
    uint16_t *q_planes;      // [2][M][Hq*128]
    // EPI_ARGMAX
    float *lm_val;           // [col groups][lm_stride]
    int32_t *lm_idx;
    int lm_stride;
    float *logits;           // optional: [M][N]
};

// Epilogue of 32 columns x 16 rows held in MFMA register order: lane (row = lane % 16, q = lane / 16) owns columns
// 4q + r (r = 0..3) in acc0 and 16 + 4q + r in acc1.  T = column tile, m = the lane's row, nsub = 4q.
// tile_pre issues every load the epilogue needs that does not depend on the accumulators (so that a
// caller can overlap them with its own loads); tile_epilogue consumes them and returns the lane's
// share of the tile's sum of squares (EPI_RESID).
struct TilePre {
    float rs;                // RMS scale of the row
    float4 hv[2], gn[2];     // EPI_RESID: residual values and gains of the lane's 8 columns
    float4 cs[2];            // EPI_QKV: (cos, sin) of the lane's 4 rotary pairs
    int kvloc;               // EPI_QKV: physical page * 16 + token in page of the row's cache position
};

template <int EPI, bool RS_KNOWN = false>
__device__ __forceinline__ TilePre tile_pre(const GemmArgs &g, int T, int m, int nsub, float rs_known = 1.0f) {
    TilePre p;
    p.rs = rs_known;
    p.kvloc = 0;
    if (m >= g.M) return p;
    if (!RS_KNOWN && g.ssq_in) p.rs = rms_scale(g.ssq_in[m], g.inv_d, g.eps);
    if constexpr (EPI == EPI_RESID) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int nn = T * 32 + 16 * j + nsub;
            p.hv[j] = *(const float4 *)(g.h + (size_t)m * g.N + nn);
            p.gn[j] = *(const float4 *)(g.gain + nn);
        }
    } else if constexpr (EPI == EPI_QKV) {
        const int hy = T >> 2, i0 = 16 * (T & 3) + nsub;
        if (hy >= g.Hq) p.kvloc = g.row_kvloc[m];
        if (hy < g.Hq + g.Hkv) {
            p.cs[0] = *(const float4 *)(g.row_cs + (size_t)m * 64 + i0);
            p.cs[1] = *(const float4 *)(g.row_cs + (size_t)m * 64 + i0 + 2);
        }
    }
    return p;
}

template <int EPI>
__device__ __forceinline__ float tile_epilogue(const GemmArgs &g, const f32x4 &acc0, const f32x4 &acc1, int T, int m, int nsub, const TilePre &p) {
    float ss = 0.f;
    if (m >= g.M) return ss;
    const float rs = p.rs;
    if constexpr (EPI == EPI_RESID) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int nn = T * 32 + 16 * j + nsub;
            const f32x4 &a = j ? acc1 : acc0;
            float4 v = p.hv[j];
            v.x += a[0]; v.y += a[1]; v.z += a[2]; v.w += a[3];
            *(float4 *)(g.h + (size_t)m * g.N + nn) = v;
            ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
            const float4 gn = p.gn[j];
            uint32_t hi[2], lo[2];
            split_pack2(v.x * gn.x, v.y * gn.y, hi[0], lo[0]);
            split_pack2(v.z * gn.z, v.w * gn.w, hi[1], lo[1]);
            *(uint2 *)(g.xout + xpack_index(m, nn, 0, g.units_total)) = make_uint2(hi[0], hi[1]);
            *(uint2 *)(g.xout + xpack_index(m, nn, 1, g.units_total)) = make_uint2(lo[0], lo[1]);
        }
    } else if constexpr (EPI == EPI_SWIGLU) {
        // acc0 holds the gate and acc1 the up values of feed-forward columns 16 T + nsub .. + 3
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float gt = acc0[r] * rs, up = acc1[r] * rs;
            v[r] = gt * __builtin_amdgcn_rcpf(1.0f + __expf(-gt)) * up;      // (v_rcp_f32: 1 ulp; a division is ten instructions more)
        }
        uint32_t hi[2], lo[2];
        split_pack2(v[0], v[1], hi[0], lo[0]);
        split_pack2(v[2], v[3], hi[1], lo[1]);
        const int f0 = T * 16 + nsub;
        *(uint2 *)(g.act + xpack_index(m, f0, 0, g.units_total)) = make_uint2(hi[0], hi[1]);
        *(uint2 *)(g.act + xpack_index(m, f0, 1, g.units_total)) = make_uint2(lo[0], lo[1]);
    } else if constexpr (EPI == EPI_QKV) {
        // tile T = 4 * head + t: acc0 holds dims 16 t + nsub .. + 3 of the head, acc1 the same dims + 64 (the rotary partners)
        const size_t qd = (size_t)g.Hq * 128;
        const int hy = T >> 2, i0 = 16 * (T & 3) + nsub;
        float va[4], vb[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            va[r] = acc0[r] * rs;
            vb[r] = acc1[r] * rs;
        }
        if (hy < g.Hq + g.Hkv) {
            const float cs[4] = {p.cs[0].x, p.cs[0].z, p.cs[1].x, p.cs[1].z}, sn[4] = {p.cs[0].y, p.cs[0].w, p.cs[1].y, p.cs[1].w};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float x = va[r], y = vb[r];
                va[r] = x * cs[r] - y * sn[r];
                vb[r] = y * cs[r] + x * sn[r];
            }
        }
        if (hy < g.Hq) {
            uint32_t hi[2], lo[2];
            const size_t o = (size_t)m * qd + (size_t)hy * 128 + i0;
            split_pack2(va[0], va[1], hi[0], lo[0]);
            split_pack2(va[2], va[3], hi[1], lo[1]);
            *(uint2 *)(g.q_planes + o) = make_uint2(hi[0], hi[1]);
            *(uint2 *)(g.q_planes + (size_t)g.M * qd + o) = make_uint2(lo[0], lo[1]);
            split_pack2(vb[0], vb[1], hi[0], lo[0]);
            split_pack2(vb[2], vb[3], hi[1], lo[1]);
            *(uint2 *)(g.q_planes + o + 64) = make_uint2(hi[0], hi[1]);
            *(uint2 *)(g.q_planes + (size_t)g.M * qd + o + 64) = make_uint2(lo[0], lo[1]);
        } else {
            const int kvh = hy < g.Hq + g.Hkv ? hy - g.Hq : hy - g.Hq - g.Hkv, tk = p.kvloc & 15;
            const size_t pb = ((size_t)(p.kvloc >> 4) * g.Hkv + kvh) * (SEV_PAGE * 128);
            if (hy < g.Hq + g.Hkv) {
                uint16_t *kc = (uint16_t *)g.k_layer + pb;
                *(uint2 *)(kc + k_in_page<true>(tk, i0, 128)) =
                    make_uint2(f32_to_bf16_bits(va[0]) | (f32_to_bf16_bits(va[1]) << 16),
                               f32_to_bf16_bits(va[2]) | (f32_to_bf16_bits(va[3]) << 16));
                *(uint2 *)(kc + k_in_page<true>(tk, i0 + 64, 128)) =
                    make_uint2(f32_to_bf16_bits(vb[0]) | (f32_to_bf16_bits(vb[1]) << 16),
                               f32_to_bf16_bits(vb[2]) | (f32_to_bf16_bits(vb[3]) << 16));
            } else {
                uint16_t *vc = (uint16_t *)(g.k_layer + g.v_offset) + pb;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    vc[v_in_page<true>(tk, i0 + r, 128)] = (uint16_t)f32_to_bf16_bits(va[r]);
                    vc[v_in_page<true>(tk, i0 + 64 + r, 128)] = (uint16_t)f32_to_bf16_bits(vb[r]);
                }
            }
        }
    }
    return ss;
}

// Adds a block's per-row sums of squares (one value per lane < 16 and wave, in red[wave][row]) to
// ssq_out and clears ssq_clear; rows = number of rows covered, m0 = first row.
template <int STRIDE>
__device__ __forceinline__ void ssq_commit(const GemmArgs &g, float (*red)[STRIDE], int rows, int m0, bool clear) {
    __syncthreads();
    if ((int)threadIdx.x < rows) {
        const int t = threadIdx.x, m = m0 + t;
        if (m < g.M) {
            atomicAdd(g.ssq_out + m, ssq_fix((red[0][t] + red[1][t]) + (red[2][t] + red[3][t])));
            if (clear) g.ssq_clear[m] = 0ull;
        }
    }
}

// Kernel arguments live in memory and are fetched with scalar loads where the compiler first needs
// them; an argument block of several cache lines can then cost one memory latency per line, one after
// the other, in the middle of the kernel.  Naming one field of every line at the kernel's entry makes
// all of those fetches start together.
#define SEV_ARGS_NOW(...) asm volatile("" : : __VA_ARGS__)

// The arguments the prologue needs first (pointers and grid decomposition) are passed as leading
// scalars as well: the library is built with kernel-argument preloading, which hands the first 16
// dwords of the argument block to the wave in registers at launch, so the first loads can be issued
// without waiting for a scalar load of the argument block.
//
// HALF: the wave's last column tile is shared with the wave beside it, each of the two doing half of the row units, so that
// a block covers 4 (NT - 1) + 2 column tiles (6, 10 or 14) and every wave has the same MR (NT - 1/2) units of work.  The
// odd wave of a pair carries its row units in the order "upper half first": its shared tile then uses the same registers
// as the even wave's, and no fragment is indexed by a run-time value.
//
// Accumulators.  Left to itself the compiler gives every product of this instruction a destination of its own and moves
// accumulators about in the loop (60-300 moves in 256 products), so mfma_pair names the accumulator file and ties source and
// destination in an assembly statement.  Such statements keep their order, which makes the loop's instruction order the one written here.

// acc += w * (hi plane) + w * (lo plane).  The products of a pair follow each other on the same accumulators, which needs no wait
// states, and their operands come from loads, which the compiler awaits.
__device__ __forceinline__ void mfma_pair(f32x4 &acc, u32x4 w, u32x4 hi, u32x4 lo) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %3, %0" : "+a"(acc) : "v"(w), "v"(hi), "v"(lo));
}

template <int MR, int NT, int EPI, int PF, bool HALF = false>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(const uint4 *W_, const uint4 *X_, int n_tiles_, int k_steps_, int units_total_,
                                                        int col_groups_, int m_blocks_, int splits_, GemmArgs g) {
    g.W = W_; g.X = X_; g.n_tiles = n_tiles_; g.k_steps = k_steps_; g.units_total = units_total_;
    g.col_groups = col_groups_; g.m_blocks = m_blocks_; g.splits = splits_ & 0xffff;
    const int tpb = splits_ >> 16;                      // column tiles per block: 4 * NT, or fewer (the last wave then has fewer tiles)
    constexpr int KS = gemm_ks(MR, NT);
    constexpr int NF = 2 * NT;                          // weight fragments per wave and k-step: two per column tile
    constexpr int XI = (KS * MR + 1) / 2;               // 16-byte activation loads per thread and stage
    constexpr bool XHALF = KS * MR % 2 != 0;            // the last of them by the first 128 threads alone
    constexpr int G = KS * MR;                          // groups of products per stage: one activation unit x all weight fragments
    constexpr int AHEAD = G < PF ? G : PF - 1;          // an activation unit is read from LDS that many groups before its products
    static_assert(PF >= 3, "X(st+2) is written while X(st) and X(st+1) are read");
    extern __shared__ u32x4 xs[];                       // [PF buffers][KS k-steps][MR][2 planes][64 lanes], a stage filled up to whole loads
    __shared__ float red[4][MR * 16 < 128 ? 128 : MR * 16];
    constexpr int STAGE_U4 = XI * 256;                  // uint4 per stage
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // Block index decode, XCD-aware: consecutive block ids go round-robin to the 8 XCDs, each with its
    // own L2.  Blocks that share weight tiles (the row blocks of one column group) get ids 8 apart,
    // i.e. land on the same XCD back to back, so the second read can hit that L2.
    int q = blockIdx.x >> 3;
    const int mb = q % g.m_blocks;
    q /= g.m_blocks;
    const int split = q % g.splits;
    const int cg = (q / g.splits) * 8 + (blockIdx.x & 7);
    if (cg >= g.col_groups) return;                      // whole block leaves before any barrier
    const int block_tiles = min(tpb, g.n_tiles - cg * tpb);
    // column tile a of the wave, within the block: those past block_tiles do not exist (the wave then only helps with the activations)
    auto lct = [&](int a) { return !HALF ? wave * NT + a : (a < NT - 1 ? wave * (NT - 1) + a : 4 * (NT - 1) + (wave >> 1)); };
    auto have = [&](int a) { return lct(a) < block_tiles; };
    auto coltile = [&](int a) { return cg * tpb + lct(a); };
    const int u0 = mb * MR;                              // first row unit
    constexpr int MH = MR / 2;
    static_assert(!HALF || MR % 2 == 0, "a shared tile is split into two halves of the row units");
    const int par = HALF ? wave & 1 : 0;
    auto ru = [&](int b) { return !HALF ? b : (b < MH ? b + par * MH : b - par * MH); };      // row unit behind register slot b
    auto rows_of = [&](int a) { return HALF && a == NT - 1 ? MH : MR; };                       // slots of column tile a
    const int n_stages = g.k_steps / KS;
    const int s_begin = (int)((unsigned)n_stages * (unsigned)split / (unsigned)g.splits);          // small numbers: 32-bit division
    const int s_end = (int)((unsigned)n_stages * (unsigned)(split + 1) / (unsigned)g.splits);
    const int n = s_end - s_begin;
    const int mrow = lane & 15, nsub = 4 * (lane >> 4);

    f32x4 acc[NF][MR];
#pragma unroll
    for (int a = 0; a < NF; ++a)
#pragma unroll
        for (int b = 0; b < MR; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[a][b][r] = 0.f;

    // Both streams are read at a uniform address plus a 32-bit offset of the thread, so that a stage costs a few scalar
    // instructions and no vector ones: with one wave per SIMD everything that is issued between two products beyond three
    // instructions or so is idle time of the matrix pipe (64-bit addresses per load and stage: about 290 cycles of a stage).
    // Weights: tiles the wave does not have are clamped to a valid one, so idle waves load harmlessly.
    const char *const W = (const char *)g.W + (size_t)cg * tpb * g.k_steps * 2048;
    unsigned woff[NT];
#pragma unroll
    for (int a = 0; a < NT; ++a) woff[a] = (unsigned)((min(coltile(a), g.n_tiles - 1) - cg * tpb) * g.k_steps) * 2048u + lane * 16u;
    // The gate/up GEMM reads its weights through a buffer descriptor that covers exactly the block's column tiles: a
    // tile the wave does not have (blocks of fewer than 4 * NT tiles, the matrix edge) lies past the descriptor's
    // end, where a load returns zeros and reads nothing, so the loop stays free of branches and the missing tile
    // costs no memory traffic.
    constexpr bool WBUF = EPI == EPI_SWIGLU && MR <= 4;      // the 128-row blocks never run narrower than 4 * NT tiles
    const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc((void *)W, 0, block_tiles * g.k_steps * 2048, 0x00020000);
    if constexpr (WBUF) {
#pragma unroll
        for (int a = 0; a < NT; ++a) woff[a] = (unsigned)(lct(a) * g.k_steps) * 2048u + lane * 16u;
    }
    auto load_w = [&](int f, unsigned at) -> u32x4 {      // 16 bytes per lane of the k-step at byte `at` of a tile: fragment f & 1 of the wave's column tile f / 2
        // The streaming hint keeps the weights from displacing the activations in the L2s (gate/up: 7 % faster with it).
        // The QKV projection streams the fewest weights per activation byte and is 4 % faster with plain loads.  Blocks of 96
        // and 128 rows keep the hint although their row blocks share the weights through an L2; plain loads there, timed in
        // turn: 192 rows of the 8B shape gate/up 88.6 -> 89.8 us and QKV behind it 33.5 -> 34.4, 416 rows down 105.2 -> 106.7,
        // 480 rows of the 70B shape O 131.3 -> 132.9.  The one that gains from plain loads is down of the 70B shape at 176 rows
        // (178.5 -> 176.4, where gate/up loses twice that).
        if constexpr (WBUF) return __builtin_amdgcn_raw_buffer_load_b128(wrs, woff[f >> 1] + (f & 1) * 1024, at, 2);      // 2: streaming hint
        else if constexpr (EPI == EPI_QKV) return *(const u32x4 *)(W + at + woff[f >> 1] + (f & 1) * 1024);
        else return __builtin_nontemporal_load((const u32x4 *)(W + at + woff[f >> 1] + (f & 1) * 1024));
    };
    // Software pipeline.  Loads return in issue order, so a wait on one load drains every older one:
    // to keep PF stages in flight, weights AND activations are fetched PF stages ahead into registers
    // and consumed in the order they were issued.  At the start of stage st (slot u = st % PF):
    //   LDS buffers u and (u+1) % PF hold X(st) and X(st+1);  wreg[u] holds W(st);  xreg[u] holds X(st+2).
    // The activation units pass through a ring of PF register pairs: during a group's products the unit AHEAD groups later
    // is read from LDS, so that no product waits for LDS and the reads are spread evenly.  X(st+2) goes from registers into
    // the LDS buffer after next, whose contents (stage st-1 or older) were last read before the barrier that ended stage st-1;
    // one barrier per stage.  (Buffers and ring close with the loop body, so that no place is computed at run time.)
    // The loop body is PF stages of straight-line code (no branches), which lets the compiler's
    // wait-count bookkeeping follow the loads across the back-edge.  What a body prefetches past the slice's end wraps around to
    // its start (cached) and is never multiplied.
    u32x4 wreg[PF][KS][NF];
    u32x4 xreg[PF][XI];
    u32x4 xf[PF][2];
    unsigned xoff[XI];
#pragma unroll
    for (int i = 0; i < XI; ++i) {
        const int u = threadIdx.x + 256 * i;
        const int ksl = u / (MR * 128), within = u - ksl * (MR * 128);
        xoff[i] = XHALF && ksl == KS ? 0x80000000u : (unsigned)((ksl * g.units_total + u0) * 128 + within) * 16u;
    }
    // (XHALF: the activations through a buffer descriptor too; a thread without a part reads past its end, i.e. zeros and no memory)
    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc((void *)g.X, 0, g.k_steps * g.units_total * 2048, 0x00020000);
    const size_t x_stage = (size_t)KS * g.units_total * 2048;       // bytes per stage of all row units
    const int n_pad = (n + PF - 1) / PF * PF;
    // Where the activations are small enough to stay in an L2 (4 MiB) beside the weight stream, every column group walks its K range
    // from a different starting stage and wraps around: blocks that run at the same time then do not all read the same few KiB
    // of activations, i.e. hammer a few L2 channels while the others idle (8B shape, QKV: 64 rows 17.4 -> 15.4 us, 32 rows
    // 13.9 -> 12.9).  Larger ones are fetched chunk by chunk once for all column groups of an XCD, which then have to
    // walk together (rotated: down of the 8B shape at 64 rows 28 -> 39 us, of the 70B shape 83 -> 112, gate/up of that shape at 256 rows
    // 335 -> 363).  In between, from 1.5 to 2.5 MiB, the two are within 3 % of each other.
    const bool resident = g.m_blocks * MR * g.k_steps <= 768;              // 2 KiB per unit and step
    const int rot = resident ? (int)((unsigned)cg * (unsigned)n / (unsigned)g.col_groups) : 0;
    // where the two streams stand: the next stage to be requested, counted within the slice, and its address
    const char *const x_first = (const char *)g.X + (size_t)s_begin * x_stage, *x_at = x_first + (size_t)rot * x_stage;
    const unsigned xb_first = (unsigned)s_begin * (unsigned)x_stage;
    unsigned xb_at = xb_first + (unsigned)rot * (unsigned)x_stage;
    const unsigned w_first = (unsigned)s_begin * (KS * 2048u);
    unsigned w_at = w_first + (unsigned)rot * (KS * 2048u);
    int x_i = rot, w_i = rot;
    auto x_next = [&]() {
        if constexpr (XHALF) xb_at += (unsigned)x_stage;
        else x_at += x_stage;
        if (++x_i == n) { x_i = 0; x_at = x_first; xb_at = xb_first; }
    };
    auto w_next = [&]() {
        w_at += KS * 2048u;
        if (++w_i == n) { w_i = 0; w_at = w_first; }
    };
    auto load_x = [&](int i) -> u32x4 {
        if constexpr (XHALF) return __builtin_amdgcn_raw_buffer_load_b128(xrs, xoff[i], xb_at, 0);
        else return *(const u32x4 *)(x_at + xoff[i]);
    };

    {
        u32x4 x0[XI], x1[XI];
#pragma unroll
        for (int i = 0; i < XI; ++i) x0[i] = load_x(i);
        x_next();
#pragma unroll
        for (int i = 0; i < XI; ++i) x1[i] = load_x(i);
        x_next();
#pragma unroll
        for (int u = 0; u < PF; ++u) {
#pragma unroll
            for (int i = 0; i < XI; ++i) xreg[u][i] = load_x(i);
            x_next();
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int f = 0; f < NF; ++f) wreg[u][ks][f] = load_w(f, w_at + ks * 2048u);
            w_next();
        }
#pragma unroll
        for (int i = 0; i < XI; ++i) {
            xs[threadIdx.x + 256 * i] = x0[i];
            xs[STAGE_U4 + threadIdx.x + 256 * i] = x1[i];
        }
    }
    // a block that runs the epilogue itself fetches its rows' sums of squares now, so that the row scales are
    // there when the loop ends
    unsigned long long sq_rows[MR];
#pragma unroll
    for (int b = 0; b < MR; ++b) {
        const int m = (u0 + ru(b)) * 16 + mrow;
        sq_rows[b] = (g.splits == 1 && g.ssq_in && m < g.M) ? g.ssq_in[m] : 0ull;
    }
    // the rest of the argument block (epilogue pointers): fetched now, behind the first loads
    if constexpr (EPI == EPI_QKV) SEV_ARGS_NOW("s"(g.part), "s"(g.ssq_in), "s"(g.row_cs), "s"(g.q_planes));
    else if constexpr (EPI == EPI_ARGMAX) SEV_ARGS_NOW("s"(g.part), "s"(g.ssq_in), "s"(g.lm_val), "s"(g.logits));
    else SEV_ARGS_NOW("s"(g.part), "s"(g.ssq_in), "s"(g.act));
    __syncthreads();
    const u32x4 *const xr = xs + lane, *const xr_lo = xr + par * MH * 128, *const xr_hi = xr - par * MH * 128;
    u32x4 *const xw = xs + threadIdx.x;
    auto read_unit = [&](int buf, int grp, u32x4 (&to)[2]) {      // group grp of the stage in LDS buffer buf
        const int ks = grp / MR, b = grp % MR;
        const u32x4 *p = (!HALF ? xr : b < MH ? xr_lo : xr_hi) + buf * STAGE_U4 + (ks * MR + b) * 128;
        to[0] = p[0];
        to[1] = p[64];
    };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) read_unit(0, i, xf[i]);

    // One group of PF stages.  The last group of a slice issues no global loads: what it would
    // prefetch lies beyond the slice, and the epilogue would have to wait for those loads to return
    // before it may reuse their registers.
    // Everything a stage has to do besides its products is spread between them, a few instructions at a time: two LDS reads ahead
    // of a group, one activation register at a time into LDS and requested anew from the second pair on, a weight fragment
    // requested anew right after its last product.
    auto group = [&](int base, auto load_tag) {
        constexpr bool LOAD = decltype(load_tag)::value;
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            if constexpr (!LOAD) {
                if (base + u >= n) break;               // padding of the slice (uniform): nothing left to multiply
            }
            int pair = 0;
#pragma unroll
            for (int grp = 0; grp < G; ++grp) {
                const int ks = grp / MR, b = grp % MR, slot = (u * G + grp) % PF, far = (u * G + grp + AHEAD) % PF;
                if (grp + AHEAD < G) read_unit(u, grp + AHEAD, xf[far]);
                else read_unit((u + 1) % PF, grp + AHEAD - G, xf[far]);
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    if (b >= rows_of(f >> 1)) continue;
                    mfma_pair(acc[f][b], wreg[u][ks][f], xf[slot][0], xf[slot][1]);
                    if (pair % 2 == 1 && pair / 2 < XI) {
                        const int i = pair / 2;
                        xw[(u + 2) % PF * STAGE_U4 + 256 * i] = xreg[u][i];
                        if constexpr (LOAD) xreg[u][i] = load_x(i);
                    }
                    ++pair;
                    if constexpr (LOAD) {
                        if (b == rows_of(f >> 1) - 1) wreg[u][ks][f] = load_w(f, w_at + ks * 2048u);
                    }
                }
            }
            if constexpr (LOAD) {
                x_next();
                w_next();
            }
            __syncthreads();
        }
    };
    for (int base = 0; base + PF < n_pad; base += PF) group(base, std::true_type{});
    group(n_pad - PF, std::false_type{});
    asm volatile("s_nop 15\n\ts_nop 15");              // the last products must have left the pipe before their sums are read
#pragma unroll
    for (int a = 0; a < NF; ++a)
#pragma unroll
        for (int b = 0; b < MR; ++b) asm volatile("" : "+a"(acc[a][b]));

    // ------------------------------------------------------------------ split-K: hand the slice to the fix-up kernel
    if (g.splits > 1) {
        // exchange layout [slice][column tile][row unit][2][64 lanes] float4: register order, 1 KiB per store instruction
#pragma unroll
        for (int a = 0; a < NT; ++a)
            if (have(a)) {
#pragma unroll
                for (int b = 0; b < rows_of(a); ++b) {
                    float4 *mine = (float4 *)g.part + (((size_t)split * g.n_tiles + coltile(a)) * g.units_total + u0 + ru(b)) * 128 + lane;
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const f32x4 &v = acc[2 * a + j][b];
                        mine[j * 64] = make_float4(v[0], v[1], v[2], v[3]);
                    }
                }
            }
        return;
    }

    // ------------------------------------------------------------------ epilogues
    if constexpr (EPI != EPI_ARGMAX) {
        float ss[MR];
#pragma unroll
        for (int b = 0; b < MR; ++b) {
            ss[b] = 0.f;
            const int m = (u0 + ru(b)) * 16 + mrow;
            const float rs_b = g.ssq_in ? rms_scale(sq_rows[b], g.inv_d, g.eps) : 1.0f;
#pragma unroll
            for (int a = 0; a < NT; ++a)
                if (b < rows_of(a) && have(a)) {
                    const TilePre pre = tile_pre<EPI, true>(g, coltile(a), m, nsub, rs_b);
                    ss[b] += tile_epilogue<EPI>(g, acc[2 * a][b], acc[2 * a + 1][b], coltile(a), m, nsub, pre);
                }
        }
        if constexpr (EPI == EPI_RESID) {
#pragma unroll
            for (int b = 0; b < MR; ++b) {
                ss[b] += __shfl_xor(ss[b], 16);
                ss[b] += __shfl_xor(ss[b], 32);
                if (lane < 16) red[wave][ru(b) * 16 + mrow] = ss[b];
            }
            ssq_commit(g, red, MR * 16, u0 * 16, cg == 0);
        }
    } else {
        // arg-max over the block's columns for every row (lowest index wins ties); the row scale is
        // positive, so it only matters for the logits that are written out.  The waves meet in the activations' LDS, which
        // nobody reads any more (the last stage ended with a barrier): what the acceptance reads per row is a quarter of the waves' results.
        float *const wave_val = (float *)xs;
        int *const wave_idx = (int *)(wave_val + 4 * MR * 16);
#pragma unroll
        for (int b = 0; b < MR; ++b) {
            const int m = (u0 + ru(b)) * 16 + mrow;
            const float rsb = (g.logits && g.ssq_in && m < g.M) ? rms_scale(sq_rows[b], g.inv_d, g.eps) : 1.0f;
            float bv = -INFINITY;
            int bi = 0x7fffffff;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                if (b >= rows_of(f >> 1) || !have(f >> 1)) continue;
                const int nn = coltile(f >> 1) * 32 + 16 * (f & 1) + nsub;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float v = acc[f][b][r];
                    if (v > bv) { bv = v; bi = nn + r; }       // indices ascend, so ">" keeps the lowest
                }
                if (g.logits && m < g.M)
                    *(float4 *)(g.logits + (size_t)m * g.N + nn) = make_float4(acc[f][b][0] * rsb, acc[f][b][1] * rsb, acc[f][b][2] * rsb, acc[f][b][3] * rsb);
            }
#pragma unroll
            for (int o = 16; o < 64; o *= 2) {
                const float ov = __shfl_xor(bv, o);
                const int oi = __shfl_xor(bi, o);
                if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
            }
            if (lane < 16) {
                wave_val[wave * MR * 16 + ru(b) * 16 + mrow] = bv;
                wave_idx[wave * MR * 16 + ru(b) * 16 + mrow] = bi;
            }
        }
        __syncthreads();
        const int t = threadIdx.x, m = u0 * 16 + t;
        if (t < MR * 16 && m < g.M) {
            float bv = wave_val[t];
            int bi = wave_idx[t];
#pragma unroll
            for (int v = 1; v < 4; ++v) {
                const float ov = wave_val[v * MR * 16 + t];
                const int oi = wave_idx[v * MR * 16 + t];
                if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
            }
            g.lm_val[(size_t)cg * g.lm_stride + m] = bv;
            g.lm_idx[(size_t)cg * g.lm_stride + m] = bi;
        }
    }
}

// The same GEMM for small matrices: a block takes one column tile x MR row units, its four waves a quarter of K each, and their sums meet in LDS, so that
// a short contraction is spread over the chip without a fix-up kernel.  Operands go straight from memory to the products (both are stored in
// fragment order), four k-steps at a time with the next four under way; no barrier before the sums.  It reads the activations again for
// every column tile, which is what bounds its range (see choose_cfg).  (Eight waves per block are slower everywhere: 512-wide model, down 7.2 -> 7.6 us.)
// Event-timed (about 5 us of each), 25 rows of a model 512 wide, us: QKV 7.1 -> 6.6, O with its fix-up 9.6 -> 6.4, gate/up 7.6 -> 6.5, down with its fix-up
// 9.5 -> 7.2, head over 4224 ids 12.0 -> 6.8; of one 1024 wide: QKV 10.7 -> 6.6, O 9.9 -> 6.4, gate/up 11.6 -> 7.5, down 11.3 -> 9.9.
template <int MR, int EPI>
__global__ __launch_bounds__(256) void gemm_narrow_kernel(const uint4 *W_, const uint4 *X_, int n_tiles_, int k_steps_, int units_total_,
                                                                int m_blocks_, GemmArgs g) {
    g.W = W_; g.X = X_; g.n_tiles = n_tiles_; g.k_steps = k_steps_; g.units_total = units_total_;
    constexpr int STEPS = 4;
    __shared__ f32x4 sums[4][2 * MR][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = blockIdx.x >> 3, mb = q % m_blocks_, T = q / m_blocks_ * 8 + (blockIdx.x & 7);      // the row blocks of a tile on one XCD
    if (T >= g.n_tiles) return;                          // whole block leaves before any barrier
    const int u0 = mb * MR, mrow = lane & 15, nsub = 4 * (lane >> 4);
    const int k0 = g.k_steps * wave / 4, k1 = g.k_steps * (wave + 1) / 4;      // (a wave without a step loads the first and adds nothing)
    const u32x4 *const wp = (const u32x4 *)g.W + (size_t)T * g.k_steps * 128 + lane;
    const u32x4 *const xp = (const u32x4 *)g.X + (size_t)u0 * 128 + lane;
    const size_t x_step = (size_t)g.units_total * 128;
    u32x4 w[2][STEPS][2], x[2][STEPS][MR][2];
    auto load = [&](int buf, int k) {
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            const int at = max(min(k + i, k1 - 1), 0);   // past the wave's share: the last step again
            w[buf][i][0] = wp[(size_t)at * 128];
            w[buf][i][1] = wp[(size_t)at * 128 + 64];
#pragma unroll
            for (int b = 0; b < MR; ++b) {
                x[buf][i][b][0] = xp[at * x_step + b * 128];
                x[buf][i][b][1] = xp[at * x_step + b * 128 + 64];
            }
        }
    };
    load(0, k0);
    // the epilogue's own loads: wave b finishes row unit b
    const int m = (u0 + wave) * 16 + mrow;
    TilePre pre;
    if (wave < MR) pre = tile_pre<EPI>(g, T, m, nsub);
    f32x4 acc[2][MR];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int b = 0; b < MR; ++b) acc[f][b] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto products = [&](int buf, int k) {
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            if (k + i >= k1) break;                      // (uniform)
#pragma unroll
            for (int b = 0; b < MR; ++b)
#pragma unroll
                for (int f = 0; f < 2; ++f) {
                    acc[f][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(w[buf][i][f]), as_bf16x8(x[buf][i][b][0]), acc[f][b], 0, 0, 0);
                    acc[f][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(w[buf][i][f]), as_bf16x8(x[buf][i][b][1]), acc[f][b], 0, 0, 0);
                }
        }
    };
    for (int k = k0; k < k1; k += 2 * STEPS) {
        load(1, k + STEPS);
        products(0, k);
        load(0, k + 2 * STEPS);
        products(1, k + STEPS);
    }
#pragma unroll
    for (int b = 0; b < MR; ++b)
#pragma unroll
        for (int f = 0; f < 2; ++f) sums[wave][2 * b + f][lane] = acc[f][b];
    __syncthreads();
    if (wave >= MR) return;
    f32x4 a0 = sums[0][2 * wave][lane], a1 = sums[0][2 * wave + 1][lane];
#pragma unroll
    for (int v = 1; v < 4; ++v) {
        a0 += sums[v][2 * wave][lane];
        a1 += sums[v][2 * wave + 1][lane];
    }
    if constexpr (EPI == EPI_ARGMAX) {
        const int nn = T * 32 + nsub;
        float bv = -INFINITY;
        int bi = 0x7fffffff;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const float v = r < 4 ? a0[r] : a1[r - 4];
            if (v > bv) { bv = v; bi = nn + (r < 4 ? r : 12 + r); }      // indices ascend, so ">" keeps the lowest
        }
        if (g.logits && m < g.M) {
            float *to = g.logits + (size_t)m * g.N + nn;
            *(float4 *)to = make_float4(a0[0] * pre.rs, a0[1] * pre.rs, a0[2] * pre.rs, a0[3] * pre.rs);
            *(float4 *)(to + 16) = make_float4(a1[0] * pre.rs, a1[1] * pre.rs, a1[2] * pre.rs, a1[3] * pre.rs);
        }
#pragma unroll
        for (int o = 16; o < 64; o *= 2) {
            const float ov = __shfl_xor(bv, o);
            const int oi = __shfl_xor(bi, o);
            if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
        }
        if (lane < 16 && m < g.M) {
            g.lm_val[(size_t)T * g.lm_stride + m] = bv;
            g.lm_idx[(size_t)T * g.lm_stride + m] = bi;
        }
    } else {
        float ss = tile_epilogue<EPI>(g, a0, a1, T, m, nsub, pre);
        if constexpr (EPI == EPI_RESID) {
            ss += __shfl_xor(ss, 16);
            ss += __shfl_xor(ss, 32);
            if (lane < 16 && m < g.M) {
                atomicAdd(g.ssq_out + m, ssq_fix(ss));
                if (T == 0) g.ssq_clear[m] = 0ull;
            }
        }
    }
}

// Split-K fix-up: block (group of 4 column tiles, row unit) of 4 waves; wave w sums the S slices of 32 columns x 16 rows
// (column tile 4 * group + w, row unit ru) in slice order and runs the epilogue.
template <int EPI>
__global__ __launch_bounds__(256) void gemm_fixup_kernel(const float *part_, const void *pa_, const void *pb_, const unsigned long long *ssq_in_,
                                                         int units_real_, int units_total_, int splits_, int n_tiles_, int M_, int N_, int heads_,
                                                         GemmArgs g) {
    __shared__ float red[4][128];
    // leading scalars (preloaded at wave launch): everything the first loads need; pa_ / pb_ are the residual stream and
    // the gains (EPI_RESID) or the rotary table and the rows' cache locations (EPI_QKV); heads_ = query heads | KV heads << 16
    g.part = const_cast<float *>(part_); g.ssq_in = ssq_in_; g.units_total = units_total_;
    g.splits = splits_; g.n_tiles = n_tiles_; g.M = M_; g.N = N_;
    g.Hq = heads_ & 0xffff; g.Hkv = heads_ >> 16;
    if constexpr (EPI == EPI_RESID) { g.h = (float *)const_cast<void *>(pa_); g.gain = (const float *)pb_; }
    if constexpr (EPI == EPI_QKV) { g.row_cs = (const float2 *)pa_; g.row_kvloc = (const int32_t *)pb_; }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int unit = blockIdx.x % units_real_, grp = blockIdx.x / units_real_;
    const int T = grp * 4 + wave;
    const int mrow = lane & 15, nsub = 4 * (lane >> 4);
    const int m = unit * 16 + mrow;
    const size_t slice_stride = (size_t)g.n_tiles * g.units_total * 128;
    const float4 *src = (const float4 *)g.part + ((size_t)min(T, g.n_tiles - 1) * g.units_total + unit) * 128 + lane;
    f32x4 acc[2];
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[0][r] = acc[1][r] = 0.f;
    const bool live = T < g.n_tiles;
    float ss = 0.f;
    if (live) {
        const TilePre pre = tile_pre<EPI>(g, T, m, nsub);       // issued ahead of the slice loads
        for (int s0 = 0; s0 < g.splits; s0 += 8) {
            float4 v[8][2];
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    v[u][j] = src[(size_t)min(s0 + u, g.splits - 1) * slice_stride + j * 64];
            if (s0 == 0) {                                      // the rest of the argument block, behind the first loads
                if constexpr (EPI == EPI_QKV) SEV_ARGS_NOW("s"(g.q_planes), "s"(g.k_layer), "s"(g.inv_d));
                else SEV_ARGS_NOW("s"(g.xout), "s"(g.ssq_out), "s"(g.act), "s"(g.inv_d));
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (s0 + u < g.splits) {
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        acc[j][0] += v[u][j].x; acc[j][1] += v[u][j].y;
                        acc[j][2] += v[u][j].z; acc[j][3] += v[u][j].w;
                    }
                }
        }
        ss = tile_epilogue<EPI>(g, acc[0], acc[1], T, m, nsub, pre);
    }
    if constexpr (EPI == EPI_RESID) {
        ss += __shfl_xor(ss, 16);
        ss += __shfl_xor(ss, 32);
        if (lane < 16) red[wave][mrow] = ss;
        ssq_commit(g, red, 16, unit * 16, grp == 0);
    }
}

// ---------------------------------------------------------------------------
// final arg-max over the per-block partial results of the LM-head GEMM; one block per row
__global__ __launch_bounds__(256) void lm_reduce_kernel(const float *val, const int32_t *idx, int n_part, int stride,
                                                        int32_t *out) {
    __shared__ float sv[256];
    __shared__ int si[256];
    const int m = blockIdx.x;
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    for (int p = threadIdx.x; p < n_part; p += 256) {
        const float v = val[(size_t)p * stride + m];
        const int i = idx[(size_t)p * stride + m];
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
    if (threadIdx.x == 0) out[m] = si[0];
}

// ---------------------------------------------------------------------------
// verification attention over the paged bf16 cache (head_dim 128, 16-token pages).
//
// Work item = (request, group of 32 query rows, KV chunk) x KV head.  The 32 rows are
// (query head in the GQA group) x (draft node), so every K/V byte is read once for the whole
// group.  The waves of a block (4, or 8 when a block takes a whole sequence) take alternate page pairs
// (32 keys) of the chunk; per pair a wave runs
//   S^T = K Q^T   : 8 k-steps of MFMA 32x32x16, A = keys (32 keys x 16 dims; the in-page K layout
//                   makes every 16-lane group read 256 contiguous bytes), B = q (hi and lo planes,
//                   kept in registers for the whole chunk)
//   O^T += V^T P^T: MFMA 32x32x16 per 32-dim tile and page; a lane of the S^T result holds 16 keys of
//                   ONE query, and the in-page V layout is chosen so that exactly those keys are the
//                   contraction slots of the lane's B operand: probabilities never leave registers
// with an online softmax per query row (one cross-lane exchange per pair: the other 16 keys of the
// row sit in lane ^ 32); then the waves' partial (max, sum, O) are merged through LDS.  A block that
// saw only a chunk writes its partial result for the cross-chunk merge; a block that saw the whole
// sequence (DIRECT) normalises and writes the O projection's operand itself.  Masking: keys < P are visible to every row; key P + j is visible
// to a row iff bit j of the row's ancestor mask is set.
// ---------------------------------------------------------------------------
// Online softmax over one pair of pages, first half.  sh: scores of the lane's query (row `node` of the block; row_live: it
// exists) against keys 8j + 4 half + r of the pair (register 4j + r); jbase = draft-node index of the lane's first key
// (negative: prefix); pages = how many pages of the pair belong to the chunk.  Masks the scores, moves the running maximum, rescales the running sum and the accumulators, and returns the
// exponents' offset.
// MASKED = false: a pair whose 32 keys all lie in the committed prefix (every row sees every key); most pairs are.
template <bool MASKED>
__device__ __forceinline__ float attn_max(const f32x16 &sh, float (&sc)[16], int jbase, int pages, unsigned long long anc, int node, bool row_live, int causal,
                                         float scale_log2e, float &mrun, float &lrun, f32x16 (&oacc)[4]) {
    // (no memory access sits under control flow inside a pair step: the compiler's wait counts then stay exact)
    float mx = -INFINITY;
    // sc holds the raw scores (masked ones: -inf); the softmax scale goes into the one multiply-add in front of
    // each exponential
    if constexpr (!MASKED) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            sc[r] = sh[r];
            mx = fmaxf(mx, sc[r]);
        }
    }
#pragma unroll
    for (int j4 = 0; MASKED && j4 < 4; ++j4) {
        // 4-bit visibility of keys j..j+3: prefix keys (index < 0) always, draft key i iff ancestor bit i
        // (the mask has no bits at or above n); plain shifts and selects
        const int j = jbase + 8 * j4;
        const unsigned up = j < 64 ? (unsigned)(anc >> max(j, 0)) : 0u;             // j >= 0 (the tail of the last page can reach past 63)
        const unsigned dn = (unsigned)((anc << (-max(j, -3))) | ((1ull << (-max(j, -3))) - 1ull));   // -3 <= j < 0
        unsigned vis4 = j >= 0 ? up : (j <= -4 ? 0xFu : dn);
        // chains (any length): key j is visible iff j <= the row's own node index
        const int dcs = node - j;
        const unsigned visc = dcs >= 3 ? 0xFu : (dcs < 0 ? 0u : (2u << dcs) - 1u);
        vis4 = causal ? (row_live ? visc : 0xFu) : vis4;
        vis4 = (j4 >> 1) < pages ? vis4 : 0u;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float v = ((vis4 >> r) & 1u) ? sh[4 * j4 + r] : -INFINITY;
            sc[4 * j4 + r] = v;
            mx = fmaxf(mx, v);
        }
    }
    const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);      // (lanes & 31, that + 32)
    mx = fmaxf(__uint_as_float(both[0]), __uint_as_float(both[1])) * scale_log2e;      // (the scale is positive)
    const float mnew = fmaxf(mrun, mx);
    const float muse = (mnew == -INFINITY) ? 0.f : mnew;
    const float alpha = __builtin_amdgcn_exp2f(mrun - muse);
    mrun = mnew;
    lrun *= alpha;
    // the running maximum rarely moves after the first pairs: the 64 accumulator registers are rescaled only when
    // some row's maximum did (alpha is exactly 1 otherwise, so skipping changes nothing)
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0ull) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[t][r] *= alpha;
    }
    return muse;
}

// Second half: the probabilities, two scores at a time, as hi/lo planes, and their sum.
__device__ __forceinline__ void attn_exp2(float (&sc)[16], int r, float scale_log2e, float muse) {
    sc[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[r], scale_log2e, -muse));
    sc[r + 1] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[r + 1], scale_log2e, -muse));
}
__device__ __forceinline__ void attn_split(const float (&sc)[16], int r, float &ps, uint32_t (&ph)[8], uint32_t (&pl_)[8]) {
    ps += sc[r] + sc[r + 1];
    split_pack2(sc[r], sc[r + 1], ph[r / 2], pl_[r / 2]);
}

// ONCE: every K/V byte is read by exactly one block (each request has a single row group); its loads then carry the
// streaming hint.
template <int WAVES, bool DIRECT, bool ONCE>
__global__ __launch_bounds__(WAVES * 64, WAVES == 4 ? 2 : 1) void attn_bf16_kernel(const int4 *it_a_, const int4 *it_b_, const int32_t *it_pages_,
                                                                                    const uint16_t *q_planes, char *pool_, size_t layer_off_, size_t v_off_,
                                                                                    int M, int heads_,
                                                                                    DevPlan p, KvGeom g, int n_items_sib,
                                                                                    float *att_o, float2 *att_ml, float scale_log2e,
                                                                                    uint16_t *o_pack, int units) {
    // (leading scalars: preloaded at wave launch; layer_off_ = layer * layer stride of the pool, v_off_ = offset of the
    // V pages, heads_ = query heads | KV heads << 16)
    p.it_a = const_cast<int4 *>(it_a_); p.it_b = const_cast<int4 *>(it_b_); p.it_pages = const_cast<int32_t *>(it_pages_);
    const int Hq = heads_ & 0xffff;
    g.Hkv = heads_ >> 16;
    g.v_offset = v_off_;
    extern __shared__ float lds[];                    // WAVES merge slots: 64 accumulator registers + max + sum per lane
    // Block index -> (work item, KV head).  Consecutive block ids go round-robin to the 8 XCDs, each with its own L2.  A set
    // is the `sib` row groups of one (request, chunk): items that read the same K/V, side by side in the work list.  The
    // blocks of a (set, KV head) pair run on one XCD at about the same time, and its K/V comes from memory once (trees of 64
    // nodes, 8 row groups: 45 ns per page against 78 ns when the groups are spread over the XCDs).  sib = 1 when the requests
    // differ in their number of row groups.  The pairs go round the XCDs, so that few or unequal sets fill all of them (one
    // tree of 64 nodes on 16 tokens 17.7 -> 11.0 us against whole sets per XCD, 9 ragged trees on up to 2900 39 -> 30);
    // equal requests in a multiple of 8 sets fill them as well with whole sets, which an XCD then walks head by head, a page
    // of all heads at a time (16 trees of 24 nodes on 1000 tokens: 36.2 us by pairs, 33.8 by sets).  The grid is padded to
    // whole rounds of 8; the padding leaves before the barrier.
    const int n_items = n_items_sib & 0xffffff, sib = n_items_sib >> 24;
    const int jb = (int)(blockIdx.x >> 3), xcd = (int)(blockIdx.x & 7);
    int item, kvh;
    if (sib > 1 && n_items % (8 * sib) == 0) {
        const int tb = jb / g.Hkv;
        kvh = jb - tb * g.Hkv;
        item = (tb / sib * 8 + xcd) * sib + tb % sib;
    } else {
        const int pair = jb / sib * 8 + xcd, set = pair / g.Hkv;
        kvh = pair - set * g.Hkv;
        item = set * sib + jb % sib;
    }
    if (item >= n_items) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave index as a scalar: loop bounds stay uniform
    // everything the block needs to know comes from two 16-byte loads and one page-id load, all independent
    const int4 ia = p.it_a[item], ib = p.it_b[item];
    const int rg = ia.x, page0 = ia.y, npages = ia.z, P = ia.w, n = ib.x, row0 = ib.y;
    const int npairs = (npages + 1) >> 1;
    const int my_pairs = npairs > wave ? (npairs - wave + WAVES - 1) / WAVES : 0;   // this wave takes pairs wave, wave+WAVES, ...
    int pt_val;                                         // lane j < 32: page (j&1) of this wave's pair j/2
    {
        const int pidx = 2 * (wave + WAVES * ((lane & 31) >> 1)) + (lane & 1);
        pt_val = p.it_pages[(size_t)item * SEV_ATT_MAX_CP + pidx];    // the list is padded with the last page
    }
    const int G = Hq / g.Hkv;
    const int qrow = lane & 31, half = lane >> 5;
    const size_t page_stride = (size_t)g.Hkv * 4096;
    const size_t qd = (size_t)Hq * 128;
    // K fragment of k-step ks: lane (key = lane % 32 -> page (key / 16), token key % 16; dims 16 ks + 8 half .. +7)
    //   byte offset in the page block: ((2 ks + half) * 16 + token) * 16
    // V fragment of (dim tile dt, page): lane (dim = lane % 32, half) -> 16 bytes at ((dt * 64 + lane) * 16)
    const char *Kl = pool_ + layer_off_ + (size_t)kvh * 4096 + (half * 16 + (lane & 15)) * 16;
    const char *Vl = pool_ + layer_off_ + g.v_offset + (size_t)kvh * 4096 + lane * 16;
    const int kpage_sel = (lane >> 4) & 1;             // which page of the pair this lane's key belongs to

    // K and V fragments of one page pair live in registers; the keys of the next pair are requested as
    // soon as the score MFMAs have consumed the current ones, the values right after the PV MFMAs.  Two
    // blocks share a compute unit, so the other block's waves fill the time a wave waits for its loads.
    // Where the cache is read once, its loads carry the streaming hint, which keeps q, the page lists and the partial
    // results in the L2s (8-12 % faster on workloads of 0.3-0.5 GB of K/V per layer).  Requests with several row groups
    // (trees, wide GQA groups) re-read their K/V through the L2s, which the hint would defeat (measured: 60 % slower
    // with 8 groups, 20 % with 2).
    auto ld = [](const char *p_) -> u32x4 {
        if constexpr (ONCE) return __builtin_nontemporal_load((const u32x4 *)p_);
        else return *(const u32x4 *)p_;
    };
    u32x4 kf[8], vf[2][4];
    auto load_k = [&](int i) {
        const int pg = __shfl(pt_val, 2 * i + kpage_sel);
        const char *a = Kl + (size_t)pg * page_stride;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) kf[ks] = ld(a + ks * 512);
    };
    auto load_v = [&](int i) {
        const char *a0 = Vl + (size_t)__shfl(pt_val, 2 * i) * page_stride, *a1 = Vl + (size_t)__shfl(pt_val, 2 * i + 1) * page_stride;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) {
            vf[0][dt] = ld(a0 + dt * 1024);
            vf[1][dt] = ld(a1 + dt * 1024);
        }
    };
    load_k(0);                                             // padded page list: always a valid page, even for an idle wave
    load_v(0);
    SEV_ARGS_NOW("s"(p.row_anc), "s"(p.causal), "s"(att_o), "s"(att_ml), "s"(o_pack));   // the rest of the argument block, behind the first loads

    // query fragments of this lane's row (hi and lo planes, 8 k-steps): 64 registers for the whole chunk
    const int R = rg * 32 + qrow;
    const bool row_live = R < G * n;
    u32x4 qf[2][8];
    unsigned long long anc = 0ull;
    const int hg = row_live ? R / n : 0, node = row_live ? R - hg * n : 0;
    {
        const uint16_t *qp = q_planes + (size_t)(row0 + node) * qd + (size_t)(kvh * G + hg) * 128 + 8 * half;
#pragma unroll
        for (int pl = 0; pl < 2; ++pl)
#pragma unroll
            for (int ks = 0; ks < 8; ++ks)
                qf[pl][ks] = *(const u32x4 *)(qp + (size_t)pl * M * qd + 16 * ks);     // dead rows read row (row0, head 0): harmless, never stored
        anc = p.row_anc[row0 + node];
        if (!row_live) anc = 0ull;
    }
    // Everything loaded so far (the first K and V fragments, q, the ancestor mask) is awaited HERE, once: the loop's
    // first MFMA needs most of it anyway.  Left to the loop, the compiler's wait-count bookkeeping has to assume at
    // every iteration that the q loads of the prologue may still be pending behind the K and V loads, and makes each
    // iteration's score MFMAs wait for the V fragments requested just before, i.e. for a whole memory latency.
#pragma unroll
    for (int pl = 0; pl < 2; ++pl)
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) asm volatile("" : : "v"(qf[pl][ks]));
    asm volatile("" : : "v"(anc));

    f32x16 oacc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[t][r] = 0.f;
    float mrun = -INFINITY, lrun = 0.f;

    auto pair_step = [&](int i, auto prefetch_tag, auto masked_tag) {
        constexpr bool PREFETCH = decltype(prefetch_tag)::value;
        constexpr bool MASKED = decltype(masked_tag)::value;
        const int lp0 = 2 * (wave + WAVES * i);             // chunk-local pages of the pair
        // scores of this lane's query against keys 8j + 4*half + r of the pair (j = 0..3 -> register 4j + r)
        f32x16 sh;
#pragma unroll
        for (int r = 0; r < 16; ++r) sh[r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            sh = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kf[ks]), as_bf16x8(qf[0][ks]), sh, 0, 0, 0);
            sh = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kf[ks]), as_bf16x8(qf[1][ks]), sh, 0, 0, 0);
        }
        if (PREFETCH) load_k(i + 1);
        uint32_t ph[8], pl_[8];
        float sc[16];
        const float muse = attn_max<MASKED>(sh, sc, (page0 + lp0) * 16 + 4 * half - P, npages - lp0, anc, node, row_live, p.causal, scale_log2e, mrun, lrun, oacc);
        float ps = 0.f;
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            attn_exp2(sc, r, scale_log2e, muse);
            attn_split(sc, r, ps, ph, pl_);
        }
        lrun += ps;
        // page kk of the pair is contraction step kk: its 8 slots of this lane are score registers 8kk .. 8kk+7
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const bf16x8 pH = as_bf16x8((u32x4){ph[4 * kk], ph[4 * kk + 1], ph[4 * kk + 2], ph[4 * kk + 3]});
            const bf16x8 pL = as_bf16x8((u32x4){pl_[4 * kk], pl_[4 * kk + 1], pl_[4 * kk + 2], pl_[4 * kk + 3]});
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) {
                oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vf[kk][dt]), pH, oacc[dt], 0, 0, 0);
                oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vf[kk][dt]), pL, oacc[dt], 0, 0, 0);
            }
        }
        if (PREFETCH) load_v(i + 1);
    };
    // pairs in key order: first those that lie wholly inside the prefix, then the few that hold draft nodes, the end of
    // the last page or padding
    // pair i covers keys [(page0 + lp0) * 16, (page0 + lp0 + 2) * 16), lp0 = 2 (wave + WAVES i): inside the prefix iff
    // 2 (wave + WAVES i) <= P / 16 - page0 - 2
    const int room = P / 16 - page0 - 2;
    const int n_plain = (room >= 0 && (room >> 1) >= wave) ? min(my_pairs - 1, ((room >> 1) - wave + WAVES) / WAVES) : 0;     // (the last pair always takes the general path)
    int i = 0;
    for (; i < n_plain; ++i) pair_step(i, std::true_type{}, std::false_type{});
    for (; i + 1 < my_pairs; ++i) pair_step(i, std::true_type{}, std::true_type{});
    if (my_pairs > 0) pair_step(my_pairs - 1, std::false_type{}, std::true_type{});

    // ---- merge the waves through LDS in one step: every wave publishes its (max, sum, O) in the
    // accumulators' own register layout; then wave w reduces register quads [w * QW, (w + 1) * QW) of all
    // waves (a quad = 4 consecutive dims of the lane's query) and stores them, so that the reduction and
    // the stores are spread over the whole block.
    f32x4 *slotO = (f32x4 *)lds;                        // [WAVES][16 register quads][64 lanes]
    float *slotM = lds + WAVES * 16 * 64 * 4;           // [WAVES][64 lanes] (max), then the same for sums
    float *slotL = slotM + WAVES * 64;
    slotM[wave * 64 + lane] = mrun;
    slotL[wave * 64 + lane] = lrun;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            slotO[(wave * 16 + t * 4 + j) * 64 + lane] = (f32x4){oacc[t][4 * j], oacc[t][4 * j + 1], oacc[t][4 * j + 2], oacc[t][4 * j + 3]};
    __syncthreads();
    float mall = -INFINITY;
#pragma unroll
    for (int v = 0; v < WAVES; ++v) mall = fmaxf(mall, slotM[v * 64 + lane]);
    const float mfin = (mall == -INFINITY) ? 0.f : mall;
    float wsc[WAVES];
    float l = 0.f;
#pragma unroll
    for (int v = 0; v < WAVES; ++v) {
        wsc[v] = __builtin_amdgcn_exp2f(slotM[v * 64 + lane] - mfin);
        l += slotL[v * 64 + lane] * wsc[v];
    }
    l += __shfl_xor(l, 32);                             // the other half of the row's keys
    constexpr int QW = 16 / WAVES;
    const float inv = DIRECT ? 1.0f / l : 1.0f;
    const size_t base = ((size_t)item * g.Hkv + kvh) * 32;
    if (!DIRECT && wave == 0 && half == 0) att_ml[base + qrow] = make_float2(mall, l);
#pragma unroll
    for (int qi = 0; qi < QW; ++qi) {
        const int q = wave * QW + qi;                   // register quad: dims 32 (q / 4) + 8 (q % 4) + 4 half .. +3 of this lane's query
        f32x4 o = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < WAVES; ++v) {
            const f32x4 x = slotO[(v * 16 + q) * 64 + lane];
#pragma unroll
            for (int r = 0; r < 4; ++r) o[r] += x[r] * wsc[v];
        }
        const int dim = 32 * (q >> 2) + 8 * (q & 3) + 4 * half;
        if constexpr (DIRECT) {
            // the block saw the whole sequence: normalise and write hi/lo fragments for the O projection
            if (row_live) {
                uint32_t hi[2], lo[2];
                split_pack2(o[0] * inv, o[1] * inv, hi[0], lo[0]);
                split_pack2(o[2] * inv, o[3] * inv, hi[1], lo[1]);
                const int m = row0 + node, kk = (kvh * G + hg) * 128 + dim;
                *(uint2 *)(o_pack + xpack_index(m, kk, 0, units)) = make_uint2(hi[0], hi[1]);
                *(uint2 *)(o_pack + xpack_index(m, kk, 1, units)) = make_uint2(lo[0], lo[1]);
            }
        } else {
            *(float4 *)(att_o + (base + qrow) * 128 + dim) = make_float4(o[0], o[1], o[2], o[3]);
        }
    }
}

// The same attention for requests with many query rows (prefill chunks, large trees): a block of 4 waves takes four row
// groups (128 query rows) of a request, a wave each, and walks the pages with all of them, so that a page pair comes
// through the L2 once per 128 rows: it is staged in LDS (two buffers of 16 KiB, one barrier per pair; a wave fetches one
// of the pair's four 4 KiB page blocks, one pair ahead in registers).  The waves need no merge, and on chains the walk
// ends at the last key that the block's rows see.
//
// With K/V read per row group (attn_bf16_kernel) this work was bound by the bytes that the compute units can pull (16 KiB
// per pair and wave, 35 bytes per ns and unit): 1.85 us per pair step and SIMD.  Now 0.85 us; its 32 MFMAs are 0.5 us of
// that, staging 0.2 us (0.65 us without it).  The rest is the vector work, which is therefore spread between the MFMAs.
// grid: Hkv x n_items; KV head = block id % Hkv, which with 8 KV heads puts all blocks of a head on one XCD.
template <bool DIRECT>
__global__ __launch_bounds__(256, 2) void attn_bf16_shared_kernel(const int4 *it_a, const int4 *it_b, const int32_t *it_pages, const uint16_t *q_planes,
                                                                  const char *pool, size_t layer_off, size_t v_off, int M, int heads,
                                                                  const unsigned long long *row_anc, int causal, int n_items, float scale_log2e,
                                                                  float *att_o, float2 *att_ml, uint16_t *o_pack, int units) {
    __shared__ u32x4 kv[2][1024];                       // per buffer: K page 0, K page 1, V page 0, V page 1 of one head
    const int Hq = heads & 0xffff, Hkv = heads >> 16, G = Hq / Hkv;
    const int kvh = (int)blockIdx.x % Hkv, idx = (int)blockIdx.x / Hkv;
    // Items of a request ascend in work on chains (later rows see more keys).  They are taken from the top and from the
    // bottom in turn, the other way round in the second half of the grid: neighbours then add up to the same work, and so do
    // blocks half the grid apart, whichever of them share a compute unit.
    const int pr = idx >> 1;
    const int item = ((idx & 1) != 0) == (4 * pr >= n_items) ? n_items - 1 - pr : pr;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int4 ia = it_a[item], ib = it_b[item];
    const int page0 = ia.y, npages = ia.z, P = ia.w, n = ib.x, row0 = ib.y;
    const int rows = G * n, R0 = ia.x * 128;
    // keys that query rows first .. last of the request (row R = query head R / n of the group, node R % n) see
    auto keys = [&](int first, int last) {
        if (first >= rows) return 0;
        last = min(last, rows - 1);
        const int hf = first / n, hl = last / n;
        return P + (!causal || hf != hl ? n : last - hl * n + 1);
    };
    auto pairs = [&](int k) { return (max(0, min(npages, (k + SEV_PAGE - 1) / SEV_PAGE - page0)) + 1) >> 1; };
    const int n_pairs = pairs(keys(R0, R0 + 127)), my_pairs = pairs(keys(R0 + 32 * wave, R0 + 32 * wave + 31));
    // this wave fetches page (wave & 1) of every pair, K or V; its page ids of up to 128 pairs sit in two registers
    const int32_t *pl = it_pages + (size_t)item * SEV_ATT_MAX_CP + (wave & 1);
    const int pt0 = pl[2 * lane], pt1 = pl[128 + 2 * lane];
    const size_t page_stride = (size_t)Hkv * 4096;
    const char *src = pool + layer_off + (wave >> 1 ? v_off : 0) + (size_t)kvh * 4096 + lane * 16;
    u32x4 sa[4], sb[4];
    auto load = [&](int i, u32x4 (&to)[4]) {
        const int pg = i < 64 ? __builtin_amdgcn_readlane(pt0, i) : __builtin_amdgcn_readlane(pt1, i - 64);
        const char *a = src + (size_t)pg * page_stride;
#pragma unroll
        for (int j = 0; j < 4; ++j) to[j] = *(const u32x4 *)(a + j * 1024);
    };
    auto put = [&](int buf, const u32x4 (&from)[4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j) kv[buf][wave * 256 + j * 64 + lane] = from[j];
    };
    const int last = max(n_pairs - 1, 0), ahead = wave >> 1 ? 1 : 2;      // the keys run one pair ahead of the values
    load(0, sa);                                         // (the page list is padded: always a valid page)
    load(min(1, last), sb);

    const int qrow = lane & 31, half = lane >> 5;
    const int R = R0 + 32 * wave + qrow;
    const bool row_live = R < rows;
    const int hg = row_live ? R / n : 0, node = row_live ? R - hg * n : 0;
    u32x4 qf[2][8];
    {
        const uint16_t *qp = q_planes + (size_t)(row0 + node) * Hq * 128 + (size_t)(kvh * G + hg) * 128 + 8 * half;
#pragma unroll
        for (int pn = 0; pn < 2; ++pn)
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) qf[pn][ks] = *(const u32x4 *)(qp + (size_t)pn * M * Hq * 128 + 16 * ks);     // dead rows read row (row0, head 0)
    }
    const unsigned long long anc = row_live ? row_anc[row0 + node] : 0ull;
    f32x16 oacc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[t][r] = 0.f;
    float mrun = -INFINITY, lrun = 0.f;

    const u32x4 *kb = kv[0] + ((lane >> 4) & 1) * 256 + half * 16 + (lane & 15), *vb = kv[0] + 512 + lane;
    f32x16 sh;
    // Pair i: softmax of its scores, and its values.  The scores of pair i + 1 are computed in between, MFMA by MFMA among
    // the vector instructions of this pair's probabilities: a wave by itself then keeps the matrix pipe and the vector unit
    // busy at the same time.
    auto step = [&](int i, auto masked_tag) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        float sc[16];
        const float muse = attn_max<MASKED>(sh, sc, (page0 + 2 * i) * 16 + 4 * half - P, npages - 2 * i, anc, node, row_live, causal, scale_log2e, mrun, lrun, oacc);
        const u32x4 *ki = kb + ((i + 1) & 1) * 1024, *vi = vb + (i & 1) * 1024;
        u32x4 f[4];                                      // the next four fragments: keys, then values, four products ahead
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) f[ks] = ki[ks * 32];
        auto next = [&](int j) { return j < 8 ? ki[j * 32] : vi[((j - 8) >> 2) * 256 + ((j - 8) & 3) * 64]; };
        uint32_t ph[8], pl_[8];
        float ps = 0.f;
        __builtin_amdgcn_sched_barrier(0);               // (the scheduler left alone puts the vector instructions in front of the MFMAs)
#pragma unroll
        for (int r = 0; r < 16; ++r) sh[r] = 0.f;        // (past the last pair the scores are those of a buffer's old contents: never used)
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            sh = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(f[ks & 3]), as_bf16x8(qf[0][ks]), sh, 0, 0, 0);
            attn_exp2(sc, 2 * ks, scale_log2e, muse);
            __builtin_amdgcn_sched_barrier(0);
            sh = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(f[ks & 3]), as_bf16x8(qf[1][ks]), sh, 0, 0, 0);
            attn_split(sc, 2 * ks, ps, ph, pl_);
            f[ks & 3] = next(ks + 4);
            __builtin_amdgcn_sched_barrier(0);
        }
        lrun += ps;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const bf16x8 pH = as_bf16x8((u32x4){ph[4 * kk], ph[4 * kk + 1], ph[4 * kk + 2], ph[4 * kk + 3]});
            const bf16x8 pL = as_bf16x8((u32x4){pl_[4 * kk], pl_[4 * kk + 1], pl_[4 * kk + 2], pl_[4 * kk + 3]});
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) {
                const bf16x8 v = as_bf16x8(f[dt]);
                oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, pH, oacc[dt], 0, 0, 0);
                oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, pL, oacc[dt], 0, 0, 0);
                if (kk == 0) {
                    f[dt] = next(12 + dt);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    };
    // Buffer i & 1 holds pair i.  In step i the keys of pair i + 1 and the values of pair i are read; the keys of pair i + 2
    // and the values of pair i + 1 go where those of i and i - 1 were last read before the previous barrier, and what comes
    // two steps later is requested (past the end: the last pair once more).
    put(0, sa);
    if (ahead == 2) put(1, sb);
    load(min(ahead, last), sa);
    load(min(ahead + 1, last), sb);
    __syncthreads();
    {
        u32x4 f[8];
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) f[ks] = kb[ks * 32];
#pragma unroll
        for (int r = 0; r < 16; ++r) sh[r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            sh = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(f[ks]), as_bf16x8(qf[0][ks]), sh, 0, 0, 0);
            sh = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(f[ks]), as_bf16x8(qf[1][ks]), sh, 0, 0, 0);
        }
    }
    __syncthreads();                                    // step 0 overwrites the keys of pair 0
    // pairs of two pages that all rows of the wave see: in the prefix, on chains up to the first row's own node
    const int Rw = R0 + 32 * wave;
    const int seen = causal && Rw < rows && Rw / n == min(Rw + 31, rows - 1) / n ? P + Rw % n + 1 : P;
    const int n_plain = max(0, min(my_pairs, min(seen / SEV_PAGE - page0, npages) >> 1));
    auto stage = [&](int i, u32x4 (&st)[4]) {
        put((i + ahead) & 1, st);
        load(min(i + ahead + 2, last), st);
    };
    // Two steps a turn, one per staging register set (a plain pair left over takes the masked path; so does, wholly masked,
    // the step that fills up an odd count).  Three loops: one with branches around the steps copies the accumulators.
    int i = 0;
    for (; i + 1 < n_plain; i += 2) {
        stage(i, sa);
        step(i, std::false_type{});
        __syncthreads();
        stage(i + 1, sb);
        step(i + 1, std::false_type{});
        __syncthreads();
    }
    for (; i < my_pairs; i += 2) {
        stage(i, sa);
        step(i, std::true_type{});
        __syncthreads();
        stage(i + 1, sb);
        step(i + 1, std::true_type{});
        __syncthreads();
    }
    for (; i < n_pairs; i += 2) {                       // rows of this wave see no more, those of another wave do
        stage(i, sa);
        __syncthreads();
        stage(i + 1, sb);
        __syncthreads();
    }

    const float l = lrun + __shfl_xor(lrun, 32);        // the other half of the row's keys
    const size_t base = ((size_t)item * Hkv + kvh) * 128 + 32 * wave + qrow;
    if (!DIRECT && half == 0) att_ml[base] = make_float2(mrun, l);
    const float inv = 1.0f / l;
#pragma unroll
    for (int q = 0; q < 16; ++q) {                      // register quad: dims 32 (q / 4) + 8 (q % 4) + 4 half .. +3
        const int dim = 32 * (q >> 2) + 8 * (q & 3) + 4 * half;
        const float o[4] = {oacc[q >> 2][4 * (q & 3)], oacc[q >> 2][4 * (q & 3) + 1], oacc[q >> 2][4 * (q & 3) + 2], oacc[q >> 2][4 * (q & 3) + 3]};
        if constexpr (DIRECT) {
            if (row_live) {
                uint32_t hi[2], lo[2];
                split_pack2(o[0] * inv, o[1] * inv, hi[0], lo[0]);
                split_pack2(o[2] * inv, o[3] * inv, hi[1], lo[1]);
                const int m = row0 + node, kk = (kvh * G + hg) * 128 + dim;
                *(uint2 *)(o_pack + xpack_index(m, kk, 0, units)) = make_uint2(hi[0], hi[1]);
                *(uint2 *)(o_pack + xpack_index(m, kk, 1, units)) = make_uint2(lo[0], lo[1]);
            }
        } else {
            *(float4 *)(att_o + base * 128 + dim) = make_float4(o[0], o[1], o[2], o[3]);
        }
    }
}

// cross-chunk merge + normalisation; writes the attention output as hi/lo fragments for the O projection.
// grid (merge groups, Hkv, row groups of 8 per work item), 256 threads: thread owns (row q = t/32, 4 dims).
// The kernel is a load latency or two deep, and a compute unit keeps about 20 KB of loads in flight: blocks of 8 rows spread the partial results over
// the whole chip (16 requests of one row group: 512 blocks; with 32 rows per block 128).  Attention and merge of a layer against blocks of 32 rows and batches
// of four, us: one request on 8000 tokens (33 chunks) 25.6 -> 18.8, two on up to 2500 18.3 -> 14.4, a tree of 32 nodes on 1000 15.0 -> 13.1, 32 chains of the 70B shape 101.5 -> 99.6.
template <int PER>
__global__ __launch_bounds__(256) void attn_merge_kernel(const int4 *mg_rec, const float *att_o, const float2 *att_ml, uint16_t *o_pack,
                                                         int Hq, int Hkv, int units) {
    // (all arguments are scalars: preloaded at wave launch; one 16-byte record describes the group of PER query rows)
    const int grpi = blockIdx.x, kvh = blockIdx.y;
    const int4 rec = mg_rec[grpi];
    const int rg = rec.x & 0xffff, cnt = rec.x >> 16, item0 = rec.y, n = rec.z & 0xffff, stride = rec.z >> 16, row0 = rec.w, G = Hq / Hkv;
    const int sub = 8 * blockIdx.z + (threadIdx.x >> 5), d0 = (threadIdx.x & 31) * 4;      // row of the work item
    const int R = rg * PER + sub;
    if (R >= G * n) return;
    const int hg = R / n, node = R - hg * n;
    // chunks are combined four (of many: eight) at a time with a running maximum: all loads of a batch are issued together
    float mg = -INFINITY, l = 0.f, acc[4] = {0.f, 0.f, 0.f, 0.f};
    auto batch = [&](int c0, auto count_tag) {
        constexpr int N = decltype(count_tag)::value;
        float2 ml[N];
        float4 o[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const size_t base = ((size_t)(item0 + min(c0 + u, cnt - 1) * stride) * Hkv + kvh) * PER + sub;
            ml[u] = att_ml[base];
            o[u] = *(const float4 *)(att_o + base * 128 + d0);
        }
        float mb = mg;
#pragma unroll
        for (int u = 0; u < N; ++u) mb = (c0 + u < cnt) ? fmaxf(mb, ml[u].x) : mb;
        const float muse = (mb == -INFINITY) ? 0.f : mb;
        const float keep = exp2f(mg - muse);
        l *= keep;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] *= keep;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const float sc = (c0 + u < cnt) ? exp2f(ml[u].x - muse) : 0.f;
            l += sc * ml[u].y;
            acc[0] += sc * o[u].x; acc[1] += sc * o[u].y;
            acc[2] += sc * o[u].z; acc[3] += sc * o[u].w;
        }
        mg = mb;
    };
    if (cnt <= 4) batch(0, std::integral_constant<int, 4>{});
    else
        for (int c0 = 0; c0 < cnt; c0 += 8) batch(c0, std::integral_constant<int, 8>{});
    const float inv = 1.0f / l;
    const int m = row0 + node, k0 = (kvh * G + hg) * 128 + d0;
    uint32_t hi[2], lo[2];
    split_pack2(acc[0] * inv, acc[1] * inv, hi[0], lo[0]);
    split_pack2(acc[2] * inv, acc[3] * inv, hi[1], lo[1]);
    *(uint2 *)(o_pack + xpack_index(m, k0, 0, units)) = make_uint2(hi[0], hi[1]);
    *(uint2 *)(o_pack + xpack_index(m, k0, 1, units)) = make_uint2(lo[0], lo[1]);
}

// ---------------------------------------------------------------------------
// host orchestration of one forward pass
// ---------------------------------------------------------------------------
enum { G_QKV = 0, G_O, G_GU, G_DOWN, G_LM };

// Tile configuration of one GEMM: row units per block MR, column tiles per wave NT, split-K slices S.
//
// The row units go into the fewest row blocks that an MR allows (every row block reads the weights again through the L2s), and of
// what remains the block shape with the smallest estimated time is taken.  The estimate, in us, adds up
//   the main loop: products of the fullest unit's rounds (0.028 per row unit, column tile and k-step, 12 % less in the wide blocks) and bytes into the units
//     (weights from memory at 12.4 MB/us and re-reads with the activations at 20.4, slower where blocks do not fill the chip),
//     which overlap in part: root of the sum of squares; and a barrier and its skew per stage,
//   what follows it: the epilogue (per unit and tile of the block), or a split's partial sums out (per block) and through the
//     fix-up kernel.
// Its constants are fitted to which shape is best, not to times: 9000 timings of 256 (GEMM, row count) pairs, 8 to 2048 rows of five
// shapes, where its choice is 1.3 % off the best shape on average, more than 5 % in 9 % of them and 19 % at most.  (The rules by
// cases before it, for row tiles of 32, were 15 % off in the same pairs: 80 rows of the 8B shape, gate/up 64.5 -> 48.2 us, down 38.1 -> 31.5;
// 64 rows of the 70B shape, down 112 -> 83; 128 rows, gate/up 251 -> 200.)
// Blocks of 12 and 16 column tiles over 80 to 160 rows give it the row counts whose blocks of 8 tiles need a second, half-empty round
// (4800 timings more, of 38 row counts of two shapes: 1.4 % off the best for gate/up, 3 % for the others): 323 rows of the 8B shape, gate/up in 112 x 384
// blocks 133.7 -> 116.9 us (225 blocks, one round; 96 x 256 were 448), 304 rows 129 -> 122, 192 rows of the 70B shape 304 -> 263.
// The handle's tuning overrides (struct Tune: read from the environment when the handle was created) replace the choice in experiments.
static GemmCfg choose_cfg(int which, int rows, int n_tiles, int k_steps, size_t part_elems, const Tune &tune) {
    static const int row_units[] = {1, 2, 3, 4, 5, 6, 7, 8, 10};
    const int units = (rows + 15) / 16, units_total = sev_row_units(rows);
    const size_t slice = (size_t)n_tiles * units_total * 512;            // floats of one slice in the exchange buffer
    GemmCfg best = {0, 0, 1, false, 0};
    double best_us = 0;
    auto slices_fit = [&](int MR, int NT, int S) { return S == 1 || (k_steps / gemm_ks(MR, NT) / S >= 4 && (size_t)S * slice <= part_elems); };
    auto consider = [&](GemmCfg c, int s_min, int s_max, double epilogue) {
        const int mb = (units + c.MR - 1) / c.MR, cg = (n_tiles + c.cols() - 1) / c.cols();
        const double nt = c.half ? c.NT - 0.5 : c.NT, weights = n_tiles * (double)k_steps * 2048e-6, acts = (double)cg * mb * c.MR * k_steps * 2048e-6;      // MB
        c.T = c.cols();
        for (c.S = s_min; c.S <= s_max && slices_fit(c.MR, c.NT, c.S); ++c.S) {
            const int blocks = cg * mb * c.S, rounds = ((cg + 7) / 8 * mb * c.S + 31) / 32;      // column group c runs on XCD c % 8 (32 units)
            const double steps = (double)rounds * k_steps / c.S;
            const double idle = cbrt(256.0 * ((blocks + 255) / 256) / blocks);
            const double products = (c.NT > 2 ? 0.0246 : 0.028) * steps * c.MR * nt, bytes = (weights / 12.4 + (acts + (mb - 1) * weights) / 20.4) * idle * idle;
            double us = sqrt(products * products + bytes * bytes) + 0.0085 * steps / gemm_ks(c.MR, c.NT);
            if (c.S == 1) us += epilogue * rounds * c.MR * nt;
            else us += 1.8 + 0.63 * c.S * units * n_tiles * 2048e-6 + 4.7 * rounds * c.MR * std::min(c.T, n_tiles) * 2.048e-3;
            if (!best.MR || us < best_us) { best = c; best_us = us; }
        }
    };
    // Blocks of one column tile whose waves share K (gemm_narrow_kernel): their estimate is the bytes into the fullest unit, weights and activations alike, at 52 KB/us,
    // less what the caches make of it and 1.4 us at least, 0.6 us per further round of blocks, and 0.05 us per MB of weights, which come from memory (QKV of the 8B shape at
    // 16 rows: 12.8 us, in split blocks 10.3).  A split's fix-up kernel costs 1.5 us more than the other estimate says where everything is that small.
    // Against 160 timings (4 to 256 rows of models 512 to 4096 wide) the choice between the two is 1.4 % off the better one on average (without these blocks 11 %).
    auto consider_narrow = [&](double factor) {
        for (int MR : {1, 2}) {
            const int mb = (units + MR - 1) / MR, rounds = ((n_tiles + 7) / 8 * mb + 31) / 32;
            const double us = factor * std::max(1.4, rounds * (double)k_steps * 2.048 * (1 + MR) / 52.0 - 0.8) + 0.6 * (rounds - 1) + 0.05 * n_tiles * k_steps * 2048e-6;
            if (MR <= units && us < best_us + (best.S > 1 ? 1.5 : 0.0)) {
                best = GemmCfg{MR, 0, 1, false, 1};
                best_us = us;
            }
        }
    };
    const bool xbuf = (int64_t)k_steps * units_total < 1 << 20;            // an odd number of units in wide blocks: operand within 2 GiB (a buffer descriptor)
    if (which == G_LM) {
        // Never split.  Above 64 rows the wide blocks: the shape with the fewest products (rounds of the fullest XCD times a block's units and
        // tiles), on a tie the one with fewer row blocks.  8B shape with its logits, us: 80 rows in 80 x 512 blocks 174, in 80 x 256 192; 192 rows in 96 x 512
        // 293, in 96 x 256 358; 304 rows in 80 x 512 464, in 128 x 512 521; 400 rows in 80 x 512 572, in 128 x 512 708; 480 rows in 160 x 384
        // 651, in 128 x 512 729.  64 x 256 blocks take up to four times as long per product, but fill the chip where a vocabulary is small.
        double least = 0;
        auto lm = [&](int MR, int NT, double factor) {
            const int mb = (units + MR - 1) / MR, cg = (n_tiles + 4 * NT - 1) / (4 * NT), rounds = ((cg + 7) / 8 * mb + 31) / 32;
            const double products = factor * rounds * MR * NT;
            if (mb * MR > units_total || (MR % 2 && !xbuf) || (best.MR && products >= least)) return;
            best = GemmCfg{MR, NT, 1, false, 0};
            least = products;
        };
        if (units <= 4) lm((units + 1) / 2 * 2, 2, 1.0);
        else {
            for (int MR : {8, 7, 6, 5}) lm(MR, 4, 1.0);
            lm(10, 3, 1.0);
            lm(4, 2, 1.5);
        }
        const GemmCfg wide = best;
        best.MR = 0;
        consider(wide, 1, 1, 0.6);
        consider_narrow(1.15);
        return best;
    }
    int seen = 0;
    for (int MR : row_units) {
        const int mb = (units + MR - 1) / MR;
        if (mb == seen || MR > units || mb * MR > units_total) continue;      // (blocks must stay inside the operand buffers)
        seen = mb;                                           // the smallest MR of every number of row blocks
        for (int NT : {1, 2, 3, 4})
            for (bool half : {false, true}) {
                // which instances there are (launch_gemm)
                if (NT == 1 && half) continue;
                if (NT == 2 && half && (which != G_QKV || MR != 4)) continue;
                if (NT >= 3 && (MR < 5 || (NT == 4 && MR == 10))) continue;
                if (NT >= 3 && MR % 2 && !xbuf) continue;
                if (NT >= 3 && half && (NT == 3 || MR != 8 || which != G_GU)) continue;
                const GemmCfg c = {MR, NT, 1, half, 0};
                const int cg = (n_tiles + c.cols() - 1) / c.cols();
                consider(c, 1, std::min(16, std::max(1, 256 / (cg * mb))), which == G_QKV ? 1.45 : 1.0);
            }
    }
    consider_narrow(1.0);
    if (tune.has_gemm[which] && tune.gemm[which][1] == 0) {      // "-MR,0,1,4": blocks of one column tile
        if (tune.gemm[which][0] == -1 || tune.gemm[which][0] == -2) best = GemmCfg{-tune.gemm[which][0], 0, 1, false, 1};
    } else if (tune.has_gemm[which]) {                          // "MT,NT,S,PF": MT row tiles of 32 (-MT: row units), NT > 10: half tiles; S = 0 keeps the automatic split
        const int mt = tune.gemm[which][0], nt = tune.gemm[which][1], sp = tune.gemm[which][2], pf = tune.gemm[which][3];
        const bool half = nt > 10;                           // 15 (QKV), 35 (gate/up): a shared half tile
        const int MR = mt < 0 ? -mt : 2 * mt;
        const bool known = std::find(std::begin(row_units), std::end(row_units), MR) != std::end(row_units);
        if (known && (half ? ((which == G_QKV && MR == 4 && nt == 15) || (which == G_GU && MR == 8 && nt == 35)) :
                             (nt == 1 || nt == 2 || ((nt == 3 || nt == 4) && MR >= 5 && !(nt == 4 && MR == 10) && (MR % 2 == 0 || xbuf)))) &&
            sp >= 0 && sp <= 32 && pf == 4 && (units + MR - 1) / MR * MR <= units_total && sp <= std::max(1, k_steps / gemm_ks(MR, nt)) &&
            (sp <= 1 || (size_t)sp * slice <= part_elems)) {
            best.MR = 0;
            const GemmCfg c = {MR, half ? nt / 10 + 1 : nt, 1, half, 0};
            const int blocks = (n_tiles + c.cols() - 1) / c.cols() * ((units + MR - 1) / MR);
            consider(c, 1, std::min(16, std::max(1, 256 / blocks)), 1.0);
            if (sp > 0) best.S = sp;
        }
    }
    // The unsplit gate/up GEMM, when it leaves compute units idle: blocks one or two column tiles narrower (the last
    // wave of a block then has fewer tiles than the others) if that brings the block count closer to the number of
    // compute units.  With few rows the kernel is bound by the requests a compute unit can keep in flight, so every
    // unit counts: the 8B shape has 896 column tiles, 112 x 2 = 224 blocks of 8 or 128 x 2 = 256 blocks of 7.
    if (best.S == 1 && which == G_GU && best.NT && best.MR <= 4 && !best.half) {
        const int m_blocks = (units + best.MR - 1) / best.MR;
        auto blocks_t = [&](int t) { return ((n_tiles + t - 1) / t) * m_blocks; };
        for (int t = 4 * best.NT - 1; t >= 3 * best.NT + 1; --t)
            if (blocks_t(4 * best.NT) < 256 && blocks_t(t) <= 256 && blocks_t(t) > blocks_t(best.T)) best.T = t;
    }
    if (tune.tpb) {                                      // tuning experiments: tiles per block of the gate/up GEMM
        const int t = tune.tpb;
        if (which == G_GU && best.S == 1 && best.NT && best.MR <= 4 && !best.half && t >= 3 * best.NT + 1 && t <= 4 * best.NT) best.T = t;
    }
    return best;
}

// The choice depends on the handle's model and the number of row units alone; it is kept with the handle for up to 2048 rows.
static GemmCfg gemm_cfg(sev_kv *kv, int which, int rows, int n_tiles, int k_steps) {
    const int units = (rows + 15) / 16;
    GemmCfg *kept = units <= SEV_KEPT_UNITS ? &kv->gemm_kept[which * SEV_KEPT_UNITS + units - 1] : nullptr;
    if (kept && kept->MR) return *kept;
    const GemmCfg c = choose_cfg(which, rows, n_tiles, k_steps, kv->part_elems, kv->tune);
    if (kept) *kept = c;
    return c;
}

// one wave per 32 columns x 16 rows; ga.splits slices in the exchange buffer
template <int EPI>
static void launch_fixup(const GemmArgs &ga, hipStream_t st) {
    const int units = (ga.M + 15) / 16;
    hipLaunchKernelGGL((gemm_fixup_kernel<EPI>), dim3((unsigned)((ga.n_tiles + 3) / 4 * units)), dim3(256), 0, st, (const float *)ga.part,
                       EPI == EPI_QKV ? (const void *)ga.row_cs : (const void *)ga.h, EPI == EPI_QKV ? (const void *)ga.row_kvloc : (const void *)ga.gain,
                       ga.ssq_in, units, ga.units_total, ga.splits, ga.n_tiles, ga.M, ga.N, ga.Hq | (ga.Hkv << 16), ga);
}

template <int EPI>
static void launch_gemm(GemmArgs ga, const GemmCfg &c, hipStream_t st) {
    if (!c.NT) {
        const int m_blocks = ((ga.M + 15) / 16 + c.MR - 1) / c.MR;
        const dim3 narrow((unsigned)((ga.n_tiles + 7) / 8 * 8 * m_blocks));
        if (c.MR == 2) hipLaunchKernelGGL((gemm_narrow_kernel<2, EPI>), narrow, dim3(256), 0, st, ga.W, ga.X, ga.n_tiles, ga.k_steps, ga.units_total, m_blocks, ga);
        else hipLaunchKernelGGL((gemm_narrow_kernel<1, EPI>), narrow, dim3(256), 0, st, ga.W, ga.X, ga.n_tiles, ga.k_steps, ga.units_total, m_blocks, ga);
        return;
    }
    ga.col_groups = (ga.n_tiles + c.T - 1) / c.T;
    ga.m_blocks = ((ga.M + 15) / 16 + c.MR - 1) / c.MR;
    ga.splits = c.S;
    const int g8 = (ga.col_groups + 7) / 8 * 8;
    dim3 grid((unsigned)(g8 * ga.m_blocks * ga.splits));
#define SEV_LAUNCH(MR_, NT_, PF_, ...)                                                                                \
    hipLaunchKernelGGL((gemm_bf16_kernel<MR_, NT_, EPI, PF_ __VA_OPT__(, ) __VA_ARGS__>), grid, dim3(256), (PF_) * ((gemm_ks(MR_, NT_) * (MR_) + 1) / 2) * 4096, st, ga.W, ga.X, ga.n_tiles, ga.k_steps,         \
                       ga.units_total, ga.col_groups, ga.m_blocks, ga.splits | (c.T << 16), ga)
#define SEV_BY_NT(MR_, PF_)                                                                                           \
    do {                                                                                                              \
        if (c.NT == 2) SEV_LAUNCH(MR_, 2, PF_); else SEV_LAUNCH(MR_, 1, (MR_ % 2 ? 3 : 4));                               \
    } while (0)
    if constexpr (EPI == EPI_ARGMAX) {
        if (c.MR == 10) SEV_LAUNCH(10, 3, 3);
        else if (c.MR == 8) SEV_LAUNCH(8, 4, 3);
        else if (c.MR == 7) SEV_LAUNCH(7, 4, 3);
        else if (c.MR == 6) SEV_LAUNCH(6, 4, 3);
        else if (c.MR == 5) SEV_LAUNCH(5, 4, 3);
        else if (c.MR == 4) SEV_LAUNCH(4, 2, 4);
        else SEV_LAUNCH(2, 2, 4);
    } else if (c.half) {
        if constexpr (EPI == EPI_SWIGLU) SEV_LAUNCH(8, 4, 3, true);
        if constexpr (EPI == EPI_QKV) SEV_LAUNCH(4, 2, 4, true);
    } else if (c.NT == 4) {
        if (c.MR == 8) SEV_LAUNCH(8, 4, 3);
        else if (c.MR == 7) SEV_LAUNCH(7, 4, 3);
        else if (c.MR == 6) SEV_LAUNCH(6, 4, 3);
        else SEV_LAUNCH(5, 4, 3);
    } else if (c.NT == 3) {
        if (c.MR == 10) SEV_LAUNCH(10, 3, 3);
        else if (c.MR == 8) SEV_LAUNCH(8, 3, 3);
        else if (c.MR == 7) SEV_LAUNCH(7, 3, 3);
        else if (c.MR == 6) SEV_LAUNCH(6, 3, 3);
        else SEV_LAUNCH(5, 3, 3);
    }
    else if (c.MR == 10) SEV_BY_NT(10, 3);
    else if (c.MR == 8) SEV_BY_NT(8, 3);
    else if (c.MR == 7) SEV_BY_NT(7, 3);
    else if (c.MR == 6) SEV_BY_NT(6, 3);
    else if (c.MR == 5) SEV_BY_NT(5, 3);
    else if (c.MR == 4) SEV_BY_NT(4, 4);
    else if (c.MR == 3) SEV_BY_NT(3, 3);
    else if (c.MR == 2) SEV_BY_NT(2, 4);
    else SEV_BY_NT(1, 3);
#undef SEV_BY_NT
#undef SEV_LAUNCH
    if constexpr (EPI != EPI_ARGMAX) {
        if (c.S > 1) launch_fixup<EPI>(ga, st);
    }
}

// Rows of a chunk picked into compact buffers: q planes and residual stream of the tokens that a prefill still needs in its
// last layer.  One block per row.
struct TailSrc {
    int32_t row[SEV_MAX_BATCH];
};
__global__ __launch_bounds__(256) void tail_gather_kernel(TailSrc src, const uint4 *q, const uint4 *h, uint4 *q2, uint4 *h2, int M, int F, int q8, int h4) {
    const int i = blockIdx.x, r = src.row[i];
    for (int c = threadIdx.x; c < 2 * q8; c += 256) {
        const int pl = c >= q8, e = c - pl * q8;
        q2[((size_t)pl * F + i) * q8 + e] = q[((size_t)pl * M + r) * q8 + e];
    }
    for (int c = threadIdx.x; c < h4; c += 256) h2[(size_t)i * h4 + c] = h[(size_t)r * h4 + c];
}

void bf16_forward(const sev_model *m, sev_kv *kv, int rows, int B, const AttList &att_all, float *logits_out, const TailRows *tail, HeadOut *head, hipStream_t st) {
    AttList att = att_all;
    const sev_model_desc &d = m->d;
    KvGeom g = sev_kv_geom(kv);
    int units = sev_row_units(rows);                     // row units of the operand buffers
    auto Wp = [&](size_t off) { return (const uint4 *)(m->arena + off); };
    auto Gp = [&](size_t off) { return (const float *)(m->arena + off); };
    uint16_t *xa = (uint16_t *)kv->xa, *qp = (uint16_t *)kv->q_buf, *op = (uint16_t *)kv->o_buf, *act = (uint16_t *)kv->act;
    const float scale_log2e = 1.4426950408889634f / sqrtf((float)d.head_dim);

    const GemmCfg pq = gemm_cfg(kv, G_QKV, rows, m->n_qkv / 32, d.d_model / 32);
    GemmCfg po, pg, pd;
    auto choose = [&]() {
        po = gemm_cfg(kv, G_O, rows, d.d_model / 32, m->q_dim / 32);
        pg = gemm_cfg(kv, G_GU, rows, d.d_ffn / 16, d.d_model / 32);
        pd = gemm_cfg(kv, G_DOWN, rows, d.d_model / 32, d.d_ffn / 32);
    };
    choose();
    GemmArgs base;
    memset(&base, 0, sizeof(base));
    base.units_total = units;
    base.M = rows;
    base.part = kv->part;
    base.inv_d = 1.0f / (float)d.d_model;
    base.eps = d.rms_eps;
    base.h = kv->h;
    for (int l = 0; l < d.n_layers; ++l) {
        const LayerOffsets &lo = m->layers[l];
        {   // QKV projection; rotary embedding, q planes and the cache append in its epilogue
            Prof p(kv, st, PROF_GEMM_QKV);
            GemmArgs ga = base;
            ga.W = Wp(lo.wqkv); ga.X = (const uint4 *)xa; ga.n_tiles = m->n_qkv / 32; ga.k_steps = d.d_model / 32;
            ga.N = m->n_qkv; ga.ssq_in = kv->ssq[1];
            ga.row_cs = kv->plan.row_cs; ga.row_kvloc = kv->plan.row_kvloc; ga.Hq = d.n_q_heads; ga.Hkv = d.n_kv_heads;
            ga.k_layer = g.pool + (size_t)l * g.layer_stride; ga.v_offset = g.v_offset; ga.q_planes = qp;
            launch_gemm<EPI_QKV>(ga, pq, st);
        }
        if (tail && l == d.n_layers - 1) {
            // The rest of the last layer and the head only feed the next token of the prompts that end here: their last
            // rows go on alone, as blocks of one node (of 8 chunks of 512 rows at the 8B shape: LM head 8 x 0.81 ms, and
            // attention, O, gate/up and down of the last layer 8 x 0.45 ms for rows nobody reads).
            if (!tail->F) return;
            TailSrc src;
            memcpy(src.row, tail->src, sizeof(src.row));
            hipLaunchKernelGGL(tail_gather_kernel, dim3(tail->F), dim3(256), 0, st, src, (const uint4 *)qp, (const uint4 *)kv->h, (uint4 *)kv->tail_q,
                               (uint4 *)kv->tail_h, rows, tail->F, m->q_dim / 8, d.d_model / 4);
            launch_plan(kv, tail->pa, tail->tokens, nullptr, tail->att, st);
            rows = tail->F;
            B = tail->F;
            att = tail->att;
            units = sev_row_units(rows);
            qp = kv->tail_q;
            base.h = kv->tail_h;
            base.M = rows;
            base.units_total = units;
            choose();
        }
        {
            Prof p(kv, st, PROF_ATTN);
            const bool once = att.n_groups == B;         // one row group per request: every K/V byte is read by one block
#define SEV_ATTN(WAVES_, DIRECT_, ONCE_, THREADS_, LDS_)                                                                                   \
    hipLaunchKernelGGL((attn_bf16_kernel<WAVES_, DIRECT_, ONCE_>), dim3((unsigned)((att.n_items / att.sib * d.n_kv_heads + 7) / 8 * 8 * att.sib)), dim3(THREADS_), LDS_, st, \
                       kv->plan.it_a, kv->plan.it_b, kv->plan.it_pages, qp, g.pool, (size_t)l * g.layer_stride, g.v_offset, rows,           \
                       d.n_q_heads | (d.n_kv_heads << 16), kv->plan, g, att.n_items | (att.sib << 24), kv->att_o, kv->att_ml, scale_log2e, op, units)
            if (att.quad > 1) {                          // blocks of 128 query rows, K/V through LDS
                const dim3 grid((unsigned)(att.n_items * d.n_kv_heads));
#define SEV_ATTN_SHARED(DIRECT_)                                                                                                            \
    hipLaunchKernelGGL((attn_bf16_shared_kernel<DIRECT_>), grid, dim3(256), 0, st, (const int4 *)kv->plan.it_a, (const int4 *)kv->plan.it_b,      \
                       (const int32_t *)kv->plan.it_pages, (const uint16_t *)qp, (const char *)g.pool, (size_t)l * g.layer_stride, g.v_offset, rows,  \
                       d.n_q_heads | (d.n_kv_heads << 16), (const unsigned long long *)kv->plan.row_anc, kv->plan.causal, att.n_items, scale_log2e,  \
                       kv->att_o, kv->att_ml, op, units)
                if (att.direct) SEV_ATTN_SHARED(true); else SEV_ATTN_SHARED(false);
#undef SEV_ATTN_SHARED
            } else if (att.direct) {                     // one block of 8 waves per (request, row group, KV head): no chunks, no merge
                const size_t lds = (size_t)(8 * 64 * 64 + 2 * 8 * 64) * 4;      // 8 merge slots
                if (once) SEV_ATTN(8, true, true, 512, lds); else SEV_ATTN(8, true, false, 512, lds);
            } else {
                const size_t lds = (size_t)(4 * 64 * 64 + 2 * 4 * 64) * 4;   // 4 merge slots
                if (once) SEV_ATTN(4, false, true, 256, lds); else SEV_ATTN(4, false, false, 256, lds);
            }
#define SEV_MERGE(PER_)                                                                                                                     \
    hipLaunchKernelGGL((attn_merge_kernel<PER_>), dim3(att.n_groups, d.n_kv_heads, PER_ / 8), dim3(256), 0, st, (const int4 *)kv->plan.mg_rec,  \
                       (const float *)kv->att_o, (const float2 *)kv->att_ml, op, d.n_q_heads, d.n_kv_heads, units)
            if (!att.direct) {
                if (att.quad > 1) SEV_MERGE(128); else SEV_MERGE(32);
            }
#undef SEV_MERGE
#undef SEV_ATTN
        }
        {   // output projection; residual add, FFN-norm operand and scale in its epilogue
            Prof p(kv, st, PROF_GEMM_O);
            GemmArgs ga = base;
            ga.W = Wp(lo.wo); ga.X = (const uint4 *)op; ga.n_tiles = d.d_model / 32; ga.k_steps = m->q_dim / 32;
            ga.N = d.d_model; ga.gain = Gp(lo.g_ffn); ga.xout = xa; ga.ssq_out = kv->ssq[0]; ga.ssq_clear = kv->ssq[1];
            launch_gemm<EPI_RESID>(ga, po, st);
        }
        {   // gate/up projection with fused SwiGLU
            Prof p(kv, st, PROF_GEMM_GU);
            GemmArgs ga = base;
            ga.W = Wp(lo.wgu); ga.X = (const uint4 *)xa; ga.n_tiles = d.d_ffn / 16; ga.k_steps = d.d_model / 32;
            ga.N = 2 * d.d_ffn; ga.act = act; ga.ssq_in = kv->ssq[0];
            launch_gemm<EPI_SWIGLU>(ga, pg, st);
        }
        {   // down projection; residual add, next norm's operand and scale in its epilogue
            Prof p(kv, st, PROF_GEMM_DOWN);
            GemmArgs ga = base;
            ga.W = Wp(lo.wd); ga.X = (const uint4 *)act; ga.n_tiles = d.d_model / 32; ga.k_steps = d.d_ffn / 32;
            ga.N = d.d_model; ga.gain = (l + 1 < d.n_layers) ? Gp(m->layers[l + 1].g_attn) : Gp(m->off_gfinal); ga.xout = xa;
            ga.ssq_out = kv->ssq[1]; ga.ssq_clear = kv->ssq[0];
            launch_gemm<EPI_RESID>(ga, pd, st);
        }
    }
    {   // LM head with fused arg-max
        Prof p(kv, st, PROF_GEMM_LM);
        const GemmCfg pl = gemm_cfg(kv, G_LM, rows, d.vocab / 32, d.d_model / 32);
        GemmArgs ga = base;
        ga.W = Wp(m->off_lm); ga.X = (const uint4 *)xa; ga.n_tiles = d.vocab / 32; ga.k_steps = d.d_model / 32; ga.N = d.vocab;
        ga.ssq_in = kv->ssq[1];
        ga.lm_val = kv->lm_val; ga.lm_idx = kv->lm_idx; ga.lm_stride = units * 16; ga.logits = logits_out;
        launch_gemm<EPI_ARGMAX>(ga, pl, st);
        const int n_part = pl.NT ? (ga.n_tiles + 4 * pl.NT - 1) / (4 * pl.NT) : ga.n_tiles;
        if (head) *head = {HEAD_PARTS, nullptr, kv->lm_val, kv->lm_idx, n_part, ga.lm_stride};
        else hipLaunchKernelGGL(lm_reduce_kernel, dim3(rows), dim3(256), 0, st, kv->lm_val, kv->lm_idx, n_part, ga.lm_stride,
                                kv->row_argmax);
    }
}
