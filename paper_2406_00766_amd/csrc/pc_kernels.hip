// HIP kernels (gfx950) and their launchers for the layered forward / backward passes.
//
// Node buffers are row-major [node offset][sample], samples contiguous (l_prod in R^{N x B},
// l_sum in R^{M x B} of Sec. 4.3), row stride Bs = B rounded up to 32.
//
// Log-probabilities are kept as  log p(node, b) = R[block, b] + l[node, b]:  R is an integer-valued
// float per (block, sample) and l a small fp32 residual.  Deep circuits reach log-probabilities of
// -10^4 and below, where one fp32 holds only ~1e-3 absolute -- too coarse for the ratios p_c / p_n of
// Def. 2.  Product blocks renormalise (R = sum of the children's R + round(column max), l = rest);
// a sum block takes R = max of its children's R; differences of R are exact, so every exp() below
// sees a small, accurately known argument.  The paper stores plain fp32 log-probabilities.
//
// Sum layers use v_mfma_f32_32x32x2_f32.  Operand layout of that instruction (wave64):
//   A (32 x 2): lane holds A[i = lane % 32][k = lane / 32]
//   B (2 x 32): lane holds B[k = lane / 32][j = lane % 32]
//   D (32 x 32): register r of a lane holds D[i = 8 * (r / 4) + 4 * (lane / 32) + r % 4][j = lane % 32]
// With sum nodes on i and samples on j, every lane owns one sample column, so the per-sample
// running maximum of the log-sum-exp is a per-lane scalar.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>

#include "pc_device.h"
#include "pc_internal.h"
#include "pc_kernels.h"

namespace pc {

// The running maximum is only a reference: it is raised (and the accumulator rescaled) when a chunk exceeds it by
// more than PC_LAZY nats, not at every new maximum -- with 64 columns per wave some column has a new maximum in
// almost every chunk, and the rescale costs a multiplication per accumulator register.  Terms reach e^(PC_UP + PC_LAZY).
#define PC_LAZY 8.0f

// ------------------------------------------------------------------------------------------
// small utility kernels
// ------------------------------------------------------------------------------------------
__global__ void k_fill(float *p, int64_t n, float v)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

__global__ void k_readout(const float *__restrict__ l, const float *__restrict__ R, int64_t root_row, int64_t root_blk,
                          int64_t Bs, int32_t B, float *__restrict__ ll)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B) ll[b] = R[root_blk * Bs + b] + l[root_row * Bs + b];
}

// ------------------------------------------------------------------------------------------
// input layer (categorical): l[n,b] = log table[t][x_b,v][k]
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_input_fwd(const float *__restrict__ tables, const int32_t *__restrict__ xT,
                                                   const int32_t *__restrict__ ids, const int32_t *__restrict__ var,
                                                   const int32_t *__restrict__ tab, int32_t K, int32_t n_cats,
                                                   int64_t Bs, float *__restrict__ l, float *__restrict__ R)
{
    const int u = blockIdx.x;
    const int64_t b = (int64_t)blockIdx.y * 256 + threadIdx.x;
    if (b >= Bs) return;
    R[(int64_t)(ids[u] / K) * Bs + b] = 0.0f;                           // an input block's reference
    const int32_t xv = xT[(int64_t)var[u] * Bs + b];
    float *out = l + (int64_t)ids[u] * Bs + b;
    if (xv < 0) {
        const float v = xv == -1 ? 0.0f : PC_NEG_INF;
        for (int k = 0; k < K; ++k) out[(int64_t)k * Bs] = v;
        return;
    }
    const float *row = tables + ((int64_t)tab[u] * n_cats + xv) * K;
    if ((K & 3) == 0) {
        for (int k = 0; k < K; k += 4) {
            const float4 t = *reinterpret_cast<const float4 *>(row + k);
            out[(int64_t)(k + 0) * Bs] = __logf(t.x);
            out[(int64_t)(k + 1) * Bs] = __logf(t.y);
            out[(int64_t)(k + 2) * Bs] = __logf(t.z);
            out[(int64_t)(k + 3) * Bs] = __logf(t.w);
        }
    } else {
        for (int k = 0; k < K; ++k) out[(int64_t)k * Bs] = __logf(row[k]);
    }
}

// The same through an LDS tile (input_tile)
template <int KC, int COLS>
__global__ __launch_bounds__(256) void k_input_fwd_tile(const float *__restrict__ tables, const int32_t *__restrict__ xT,
                                                        const int32_t *__restrict__ ids, const int32_t *__restrict__ var,
                                                        const int32_t *__restrict__ tab, int32_t n_rows, int32_t n_by_xcd, int32_t n_ct, int32_t K,
                                                        int32_t n_cats, int64_t Bs, float *__restrict__ l, float *__restrict__ R)
{
    extern __shared__ float smem[];
    const InputTile t = n_by_xcd ? input_tile_at((int)blockIdx.x, n_rows, n_by_xcd, n_ct) : InputTile{(int)blockIdx.x, (int)blockIdx.y};
    input_tile<KC, COLS, false>(smem, t.block, (int64_t)t.col * COLS, tables, xT, nullptr, 0, 0, ids, var, tab, K, n_cats, Bs, l, R);
}

// table_flow[t][x_b,v][k] += F[n,b] for observed variables.
// The first two variants bring a [K rows x 64 samples] tile of the flow buffer into LDS with coalesced 16-byte
// loads along the batch, then turn it: a group of lanes owns consecutive nodes k of ONE sample, so every add
// touches consecutive floats of one table row.
//   hist : one workgroup per input block; the adds go into an LDS copy of the block's [n_cats x K] table slice
//          (LDS float atomics), flushed once with coalesced read-modify-writes (atomics only if the table is
//          shared by several blocks).  Used when the slice fits in LDS.
//   direct: one workgroup per (block, 64 samples); global float atomics, 64 consecutive floats per wave op.
//   sorted: below; used for tables of up to 1024 categories when hist does not apply.
__device__ inline void input_bwd_load_tile(const float *__restrict__ F, const int32_t *__restrict__ xT, int32_t id,
                                           int32_t var, int32_t K, int64_t Bs, int64_t b0, float *tile, int *cats)
{
    for (int idx = threadIdx.x; idx < K * 16; idx += 256) {
        const int row = idx >> 4, c4 = (idx & 15) * 4;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (b0 + c4 < Bs) v = *reinterpret_cast<const float4 *>(F + (int64_t)(id + row) * Bs + b0 + c4);
        float *dst = tile + row * 65 + c4;
        dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
    }
    if (threadIdx.x < 64) cats[threadIdx.x] = (b0 + threadIdx.x < Bs) ? xT[(int64_t)var * Bs + b0 + threadIdx.x] : -1;
}

__global__ __launch_bounds__(256) void k_input_bwd_hist(const float *__restrict__ F, const int32_t *__restrict__ xT,
                                                        const int32_t *__restrict__ ids, const int32_t *__restrict__ var,
                                                        const int32_t *__restrict__ tab, int32_t K, int32_t n_cats,
                                                        int64_t Bs, float *__restrict__ table_flow, int lps, int atomic_flush)
{
    extern __shared__ float smem[];
    float *hist = smem, *tile = smem + (size_t)n_cats * K;
    int *cats = reinterpret_cast<int *>(tile + K * 65);
    const int u = blockIdx.x;
    const int32_t id = ids[u];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int spi = 64 / lps;                                          // samples per wave instruction
    const int kl = lane % lps, sl = lane / lps;
    for (int i = threadIdx.x; i < n_cats * K; i += 256) hist[i] = 0.0f;
    for (int64_t b0 = 0; b0 < Bs; b0 += 64) {
        __syncthreads();
        input_bwd_load_tile(F, xT, id, var[u], K, Bs, b0, tile, cats);
        __syncthreads();
        for (int s = wave * spi + sl; s < 64; s += 4 * spi) {
            const int cat = cats[s];
            if (cat < 0) continue;
            for (int k = kl; k < K; k += lps) {
                const float f = tile[k * 65 + s];
                if (f != 0.0f) atomicAdd(hist + cat * K + k, f);
            }
        }
    }
    __syncthreads();
    float *dst = table_flow + (int64_t)tab[u] * n_cats * K;
    for (int i = threadIdx.x; i < n_cats * K; i += 256) {
        const float v = hist[i];
        if (v != 0.0f) { if (atomic_flush) atomicAdd(dst + i, v); else dst[i] += v; }
    }
}

__global__ __launch_bounds__(256) void k_input_bwd_direct(const float *__restrict__ F, const int32_t *__restrict__ xT,
                                                          const int32_t *__restrict__ ids, const int32_t *__restrict__ var,
                                                          const int32_t *__restrict__ tab, int32_t K, int32_t n_cats,
                                                          int64_t Bs, float *__restrict__ table_flow, int lps)
{
    extern __shared__ float smem[];
    float *tile = smem;
    int *cats = reinterpret_cast<int *>(tile + K * 65);
    const int u = blockIdx.x;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int spi = 64 / lps;
    const int kl = lane % lps, sl = lane / lps;
    input_bwd_load_tile(F, xT, ids[u], var[u], K, Bs, (int64_t)blockIdx.y * 64, tile, cats);
    __syncthreads();
    float *base = table_flow + (int64_t)tab[u] * n_cats * K;
    for (int s = wave * spi + sl; s < 64; s += 4 * spi) {
        const int cat = cats[s];
        if (cat < 0) continue;
        for (int k = kl; k < K; k += lps) {
            const float f = tile[k * 65 + s];
            if (f != 0.0f) atomicAdd(base + (int64_t)cat * K + k, f);
        }
    }
}

// Third variant, for tables with at most 1024 categories: one workgroup per (input block, slab of SB samples).
// The slab's samples are ordered by category with a counting sort in LDS; the block's [K x SB] flows are brought
// into an LDS tile with the columns in that order, so the samples of a category sit side by side, and every category
// that occurs gets ONE add per node -- the sum over its samples -- instead of one per sample.  The adds that remain
// are atomic even where the workgroup is the only writer of its rows: an atomic is sent and forgotten, a plain
// read-modify-write waits for its read (measured: 0.87 against 0.55 ms on 12 K blocks).  The order of the samples of
// a category is whatever the sort's atomics gave, so sums may differ in the last bit between runs, as with the
// other variants.
template <int NT>
__global__ __launch_bounds__(NT) void k_input_bwd_sorted(const float *__restrict__ F, const int32_t *__restrict__ xT,
                                                          const int32_t *__restrict__ ids, const int32_t *__restrict__ var,
                                                          const int32_t *__restrict__ tab, int32_t K, int32_t n_cats,
                                                          int64_t Bs, float *__restrict__ table_flow, int SB, int lpc)
{
    extern __shared__ float smem[];
    const int LDT = SB + 1;                                             // odd row stride: column reads conflict-free
    float *tile = smem;                                                 // [K][SB + 1], columns ordered by category
    int *cats = reinterpret_cast<int *>(tile + (size_t)K * LDT);        // [SB] category of a sample, < 0: no flow
    int *pos = cats + SB;                                               // [SB] column of a sample in the tile, -1: none
    int *start = pos + SB;                                              // [n_cats + 1] counts, then segment starts
    int *wsum = start + n_cats + 1;                                     // [NT / 64] scan scratch
    constexpr int NV = 4;                                               // 16-byte loads in flight per thread
    constexpr int PT = 1024 / NT;                                       // samples and categories of a thread, at most
    const int u = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int64_t b0 = (int64_t)blockIdx.y * SB;
    const int nb = (int)((Bs - b0) < SB ? (Bs - b0) : SB);              // samples of this slab (a multiple of 32)
    const int32_t id = ids[u];

    // flows of the block: 16-byte loads along the batch, on their way while the samples are sorted
    const int n4 = nb / 4, total = K * n4;
    const uint32_t inv_n4 = 0xffffffffu / (uint32_t)n4 + 1;             // idx / n4 = umulhi(idx, inv_n4): idx < 2^16, 8 <= n4 <= 256
    float4 v[NV];
    auto load = [&](int base0) {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int idx = base0 + tid + NT * j;
            const int row = (int)__umulhi((uint32_t)idx, inv_n4), c4 = (idx - row * n4) * 4;
            v[j] = idx < total ? *reinterpret_cast<const float4 *>(F + (int64_t)(id + row) * Bs + b0 + c4) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    load(0);
    for (int c = tid; c <= n_cats; c += NT) start[c] = 0;
    for (int i = tid; i < nb; i += NT) cats[i] = xT[(int64_t)var[u] * Bs + b0 + i];
    __syncthreads();
    // counting sort: rank inside the category, counts -> exclusive scan -> columns
    int rank[PT];                                                       // SB <= 1024: at most PT samples per thread
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        const int i = tid + NT * j;
        rank[j] = (i < nb && cats[i] >= 0) ? atomicAdd(start + cats[i], 1) : 0;
    }
    __syncthreads();
    const int per = (n_cats + NT - 1) / NT;                             // categories per thread (<= PT)
    int loc[PT], tot = 0;
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        const int c = tid * per + j;
        loc[j] = (j < per && c < n_cats) ? start[c] : 0;
        tot += loc[j];
    }
    int incl = tot;                                                     // inclusive scan over the wave, then over the waves
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int run = incl - tot;
    for (int w2 = 0; w2 < wave; ++w2) run += wsum[w2];
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        const int c = tid * per + j;
        if (j < per && c < n_cats) { start[c] = run; run += loc[j]; }
    }
    if (tid == NT - 1) start[n_cats] = run;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        const int i = tid + NT * j;
        if (i < nb) pos[i] = cats[i] >= 0 ? start[cats[i]] + rank[j] : -1;
    }
    __syncthreads();
    // columns scattered into category order; rows of a tile of more than NT * NV quads come in further rounds
    for (int base0 = 0; base0 < total; base0 += NT * NV) {
        if (base0 > 0) load(base0);
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int idx = base0 + tid + NT * j;
            if (idx >= total) break;
            const int row = (int)__umulhi((uint32_t)idx, inv_n4), c4 = (idx - row * n4) * 4;
            float *dst = tile + row * LDT;
            const int p0 = pos[c4], p1 = pos[c4 + 1], p2 = pos[c4 + 2], p3 = pos[c4 + 3];
            if (p0 >= 0) dst[p0] = v[j].x;
            if (p1 >= 0) dst[p1] = v[j].y;
            if (p2 >= 0) dst[p2] = v[j].z;
            if (p3 >= 0) dst[p3] = v[j].w;
        }
    }
    __syncthreads();
    // one group of lpc lanes per category at a time; a lane owns nodes k, k + lpc, ...
    const int grp = tid / lpc, kl = tid % lpc, n_grp = NT / lpc;
    float *base = table_flow + (int64_t)tab[u] * n_cats * K;
    for (int c = grp; c < n_cats; c += n_grp) {
        const int s0 = start[c], s1 = start[c + 1];
        if (s0 == s1) continue;
        for (int k = kl; k < K; k += lpc) {
            const float *src = tile + k * LDT;
            float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f, a3 = 0.0f;
            int sidx = s0;
            for (; sidx + 4 <= s1; sidx += 4) { a0 += src[sidx]; a1 += src[sidx + 1]; a2 += src[sidx + 2]; a3 += src[sidx + 3]; }
            for (; sidx < s1; ++sidx) a0 += src[sidx];
            const float acc = (a0 + a1) + (a2 + a3);
            if (acc != 0.0f) atomicAdd(base + (int64_t)c * K + k, acc);
        }
    }
}

// Group of launch row `row` in a set (wave-uniform).  Kernels are instantiated for one group (MULTI = false: the deep
// narrow circuits, where anything extra shows in a launch of a few microseconds) and for several: there the group
// index is found with a few scalar compares and the group's fields are read from the argument at that index (one
// more dependent scalar load, which launches with several groups -- thousands of workgroups -- hide).
struct GroupRow { int32_t r, width; const int32_t *ids, *nbr, *par, *aux; };
template <int ROWS>
__device__ inline GroupRow locate_row(const GroupSet &gs, int row)
{
    if (ROWS == PC_ROWS_CSR) return GroupRow{row, 0, gs.ids[0], gs.nbr[0] + gs.par[0][row], nullptr, gs.aux[0]};
    if (ROWS == PC_ROWS_ONE) return GroupRow{row, gs.width[0], gs.ids[0], gs.nbr[0], gs.par[0], gs.aux[0]};   // a set of one group
    int g = 0;                                                          // groups are in row order: count the starts passed
#pragma unroll
    for (int i = 1; i < PC_MAX_SET; ++i) g += (i < gs.n && row >= gs.first[i]) ? 1 : 0;
    return GroupRow{row - gs.first[g], gs.width[g], gs.ids[g], gs.nbr[g], gs.par[g], gs.aux[g]};
}

template <int>
__device__ inline GroupRow locate_row(const GroupDev &g, int row) { return GroupRow{row, g.width, g.ids, g.nbr, g.par, g.aux}; }

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

__device__ inline void bf16_split2(float a, float b, uint32_t &hi, uint32_t &lo)
{
    const floatx2 v = {a, b};
    const bf16x2 h = __builtin_convertvector(v, bf16x2);               // round to nearest even
    const floatx2 hf = __builtin_convertvector(h, floatx2);
    const bf16x2 l = __builtin_convertvector(v - hf, bf16x2);
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, l);
}

// One 1 KiB tile of the value planes read by the bf16 sum kernels (see there): exp(X + sh) of 16 node rows x 32 columns,
// split into hi and lo bf16 values; lane (j = lane % 32, h = lane / 32) owns rows 8 h .. 8 h + 7 of column j.  `sh` is
// the lane's shift (per column), -inf for a column without flow.  row0 = first node row of the slice.
// `src` points at the lane's column in the slice's first row (global rows, or a tile in LDS), `ld` is its row stride.
__device__ inline void split_value_rows(const float *src, int64_t ld, float sh, int64_t row0, int ct, int n_ct,
                                        uint4 *__restrict__ Ph, uint4 *__restrict__ Pl, int lane)
{
    const int h = lane >> 5;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = __expf(src[(8 * h + e) * ld] + sh);
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) bf16_split2(v[2 * e], v[2 * e + 1], hi[e], lo[e]);
    const int64_t tile = (row0 / 16) * n_ct + ct;
    Ph[tile * 64 + lane] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    Pl[tile * 64 + lane] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
}
__device__ inline void split_value_tile(const float *__restrict__ X, float sh, int64_t row0, int ct, int n_ct, int64_t Bs,
                                        uint4 *__restrict__ Ph, uint4 *__restrict__ Pl, int lane)
{
    split_value_rows(X + row0 * Bs + (int64_t)ct * 32 + (lane & 31), Bs, sh, row0, ct, n_ct, Ph, Pl, lane);
}

// ------------------------------------------------------------------------------------------
// product layers: forward adds child log-probs (Sec. 3); backward adds parent flows (Def. 2)
// ------------------------------------------------------------------------------------------
// Block-wise product kernels.  Workgroup = one node block x 64 sample columns; thread (rg, cl) owns rows
// rg, rg+16, ... of 4 adjacent columns (16-byte accesses along the batch), so a K-row block is K/16 rows
// deep per thread and all its loads are independent.  Column maxima over the K rows go through one
// shuffle stage (4 row groups per wave) and one LDS stage (4 waves).
template <int CL>
__device__ inline void block_col_max(float (&mx)[4], float (*red)[64], int wave, int cl)
{
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (CL == 8) mx[v] = fmaxf(mx[v], __shfl_xor(mx[v], 8));
        mx[v] = fmaxf(mx[v], __shfl_xor(mx[v], 16));
        mx[v] = fmaxf(mx[v], __shfl_xor(mx[v], 32));
    }
    if ((threadIdx.x & 63) < CL) {
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave][cl * 4 + v] = mx[v];
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int c = cl * 4 + v;
        mx[v] = fmaxf(fmaxf(red[0][c], red[1][c]), fmaxf(red[2][c], red[3][c]));
    }
}

// Both kernels walk the row's real neighbours (count in the row's flag word) U at a time: the U neighbour ids are
// fetched first, then all their loads are issued together, so a row costs one memory round trip per U neighbours
// instead of one per neighbour (small layers are latency-bound).  RPT = rows per thread = ceil(K / 16).

// forward (Sec. 3): s = sum of the children's residuals; the column maximum over the K rows is rounded to an
// integer and moved into R.  ACC = double for rows with many children (a leaf product over 98 pixels adds up to
// -540, where one fp32 step is 6e-5: summed in fp32 the residuals -- and with them every flow ratio p_c / p_n below --
// would be off by up to 1e-3); the rounded maximum is subtracted in that precision, the small residual is stored as fp32.
template <typename ACC> struct Acc4 { ACC x, y, z, w; };
// `l` is the base the children are read from, `lout` the base the block's own rows are written to: the same buffer,
// except in the product-scratch mode (Sec. 5), where product rows live in a window that every product layer reuses.
template <int RPT, int U, int ROWS, int CL, typename ACC, bool PLANES>
__global__ __launch_bounds__(256) void k_prod_fwd(const float *__restrict__ l, float *__restrict__ lout, float *__restrict__ R,
                                                  const GroupSet gs, int32_t K, int64_t Bs, uint4 *__restrict__ Ph,
                                                  uint4 *__restrict__ Pl)
{
    __shared__ float red[4][64];
    const GroupRow gr = locate_row<ROWS>(gs, blockIdx.x);
    const int r = gr.r;
    constexpr int RG = 256 / CL;                                        // row groups: a thread owns rows rg, rg + RG, ...
    const int rg = threadIdx.x / CL, cl = threadIdx.x % CL, wave = threadIdx.x >> 6;
    const int64_t b = (int64_t)blockIdx.y * (4 * CL) + cl * 4;
    const bool in = b < Bs;                                            // Bs is a multiple of 32: b..b+3 all inside
    const int32_t *row_nbr = gr.nbr + (int64_t)r * gr.width;
    const int32_t cnt = gr.aux[r] >> 8;
    const int32_t id = gr.ids[r];
    Acc4<ACC> s[RPT];
    float mx[4] = {PC_NEG_INF, PC_NEG_INF, PC_NEG_INF, PC_NEG_INF};
    float4 rsum = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int i = 0; i < RPT; ++i) s[i] = Acc4<ACC>{0, 0, 0, 0};
    if (in) {
        for (int j0 = 0; j0 < cnt; j0 += U) {
            int32_t ch[U];
#pragma unroll
            for (int u = 0; u < U; ++u) ch[u] = j0 + u < cnt ? row_nbr[j0 + u] : 0;
            float4 t[U][RPT], tr[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool on = j0 + u < cnt;                          // uniform over the workgroup
#pragma unroll
                for (int i = 0; i < RPT; ++i) {
                    const int k = rg + RG * i;
                    t[u][i] = (on && k < K) ? *reinterpret_cast<const float4 *>(l + (int64_t)(ch[u] + k) * Bs + b)
                                            : make_float4(0.f, 0.f, 0.f, 0.f);
                }
                tr[u] = (on && rg == 0) ? *reinterpret_cast<const float4 *>(R + (int64_t)(ch[u] / K) * Bs + b)
                                        : make_float4(0.f, 0.f, 0.f, 0.f);
            }
            // the U values of a round are added in fp32, the rounds in ACC (double for rows of many children: a running
            // fp32 sum of a hundred residuals loses more than the flows' tolerance allows, a sum of U does not)
#pragma unroll
            for (int i = 0; i < RPT; ++i) {
                float4 part = t[0][i];
#pragma unroll
                for (int u = 1; u < U; ++u) { part.x += t[u][i].x; part.y += t[u][i].y; part.z += t[u][i].z; part.w += t[u][i].w; }
                s[i].x += (ACC)part.x; s[i].y += (ACC)part.y; s[i].z += (ACC)part.z; s[i].w += (ACC)part.w;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) { rsum.x += tr[u].x; rsum.y += tr[u].y; rsum.z += tr[u].z; rsum.w += tr[u].w; }
        }
#pragma unroll
        for (int i = 0; i < RPT; ++i)
            if (rg + RG * i < K) {
                mx[0] = fmaxf(mx[0], (float)s[i].x); mx[1] = fmaxf(mx[1], (float)s[i].y);
                mx[2] = fmaxf(mx[2], (float)s[i].z); mx[3] = fmaxf(mx[3], (float)s[i].w);
            }
    }
    block_col_max<CL>(mx, red, wave, cl);
    if (!PLANES && !in) return;
    float sh4[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) sh4[v] = mx[v] > PC_NEG_INF ? rintf(mx[v]) : 0.0f;
    if (in) {
        const float (&sh)[4] = sh4;
        if (rg == 0)
            *reinterpret_cast<float4 *>(R + (int64_t)(id / K) * Bs + b) = make_float4(rsum.x + sh[0], rsum.y + sh[1], rsum.z + sh[2], rsum.w + sh[3]);
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int k = rg + RG * i;
            if (k < K)
                *reinterpret_cast<float4 *>(lout + (int64_t)(id + k) * Bs + b) =
                    make_float4((float)(s[i].x - (ACC)sh[0]), (float)(s[i].y - (ACC)sh[1]), (float)(s[i].z - (ACC)sh[2]),
                                (float)(s[i].w - (ACC)sh[3]));
        }
    }
    if (PLANES) {
        // the block's tile again as bf16 operand planes for a sum layer that runs on the bf16 matrix cores (this saves
        // the launch of k_split_p), taken from a copy of the tile in LDS: a lane of the plane layout owns eight rows of one
        // column, a thread here four columns of RPT rows
        constexpr int LDT = 4 * CL + 1;
        __shared__ float ptile[PLANES ? 128 * LDT : 1];
        if (in) {
#pragma unroll
            for (int i = 0; i < RPT; ++i) {
                const int k = rg + RG * i;
                if (k < K) {
                    float *dst = ptile + k * LDT + cl * 4;
                    dst[0] = (float)(s[i].x - (ACC)sh4[0]); dst[1] = (float)(s[i].y - (ACC)sh4[1]);
                    dst[2] = (float)(s[i].z - (ACC)sh4[2]); dst[3] = (float)(s[i].w - (ACC)sh4[3]);
                }
            }
        }
        __syncthreads();
        const int n_ct = (int)(Bs / 32), lane = threadIdx.x & 63;
        constexpr int CTW = CL / 8;                                     // 32-column tiles of the workgroup
        for (int it = wave; it < (K / 16) * CTW; it += 4) {
            const int ks = it / CTW, cw = it % CTW, ct = (int)blockIdx.y * CTW + cw;
            if (ct < n_ct)
                split_value_rows(ptile + 16 * ks * LDT + cw * 32 + (lane & 31), LDT, PC_UP, (int64_t)id + 16 * ks, ct, n_ct, Ph, Pl, lane);
        }
    }
}

// backward (Def. 2): rows = child blocks (sum / input blocks), neighbours = their product parents in this layer;
// F_child += sum of the parents' flows ('=' where this is the first layer that feeds the block, flag bit 1, so
// the flow buffer is never cleared).  Where this layer is the last one that feeds a SUM block (flag bit 0) its
// flow is final, so log_nf = log F - l (Alg. 3 / 4) and its column maximum per block are produced here.
// `Fpar` is the base the parents' (product blocks') flows are read from, `F` the base of the rows' own flows: the same
// buffer, except in the product-scratch mode, where product rows live in a window.
template <int RPT, int U, int ROWS, int CL, bool PLANES>
__global__ __launch_bounds__(256) void k_prod_bwd(const float *__restrict__ l, float *__restrict__ F, const float *__restrict__ Fpar,
                                                  float *__restrict__ N, float *__restrict__ nfmax, const GroupSet gs, int32_t K,
                                                  int64_t Bs, uint4 *__restrict__ Ph, uint4 *__restrict__ Pl)
{
    __shared__ float red[4][64];
    const GroupRow gr = locate_row<ROWS>(gs, blockIdx.x);
    const int r = gr.r;
    constexpr int RG = 256 / CL;                                        // row groups: a thread owns rows rg, rg + RG, ...
    const int rg = threadIdx.x / CL, cl = threadIdx.x % CL, wave = threadIdx.x >> 6;
    const int64_t b = (int64_t)blockIdx.y * (4 * CL) + cl * 4;
    const bool in = b < Bs;
    const int32_t *row_nbr = gr.nbr + (int64_t)r * gr.width;
    const int32_t id = gr.ids[r];
    const int32_t fl = gr.aux[r];                                       // uniform over the workgroup
    bool final_flow = (fl & 1) != 0;
    const bool first = ROWS == PC_ROWS_CSR || (fl & 2) != 0;
    int32_t cnt = fl >> 8;
    if (ROWS == PC_ROWS_CSR) {                                          // parents from the highest layer down: those from layer
        const int32_t *lay = gs.nbr[1] + gs.par[0][r];                  // width[1] on belong to this launch
        int32_t in_launch = cnt;
        while (lay[in_launch - 1] < gs.width[1]) --in_launch;           // the first one always does
        final_flow = final_flow && in_launch == cnt;
        cnt = in_launch;
    }
    float4 f[RPT], lv[RPT];
    if (in) {
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int k = rg + RG * i;
            f[i] = (k < K && !first) ? *reinterpret_cast<const float4 *>(F + (int64_t)(id + k) * Bs + b)
                                     : make_float4(0.f, 0.f, 0.f, 0.f);
            // the block's own log-probabilities, needed only for log_nf: fetched with everything else
            lv[i] = (k < K && final_flow) ? *reinterpret_cast<const float4 *>(l + (int64_t)(id + k) * Bs + b)
                                          : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        for (int j0 = 0; j0 < cnt; j0 += U) {
            int32_t pa[U];
#pragma unroll
            for (int u = 0; u < U; ++u) pa[u] = j0 + u < cnt ? row_nbr[j0 + u] : 0;
            float4 t[U][RPT];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool on = j0 + u < cnt;                          // uniform over the workgroup
#pragma unroll
                for (int i = 0; i < RPT; ++i) {
                    const int k = rg + RG * i;
                    t[u][i] = (on && k < K) ? *reinterpret_cast<const float4 *>(Fpar + (int64_t)(pa[u] + k) * Bs + b)
                                            : make_float4(0.f, 0.f, 0.f, 0.f);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int i = 0; i < RPT; ++i) {
                    f[i].x += t[u][i].x; f[i].y += t[u][i].y; f[i].z += t[u][i].z; f[i].w += t[u][i].w;
                }
        }
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int k = rg + RG * i;
            if (k < K) *reinterpret_cast<float4 *>(F + (int64_t)(id + k) * Bs + b) = f[i];
        }
    }
    if (!final_flow) return;
    float mx[4] = {PC_NEG_INF, PC_NEG_INF, PC_NEG_INF, PC_NEG_INF};
    float4 nfv[PLANES ? RPT : 1];
    if (in) {
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int k = rg + RG * i;
            if (k < K) {
                float4 nf;
                nf.x = (f[i].x > 0.0f && lv[i].x > PC_NEG_INF) ? __logf(f[i].x) - lv[i].x : PC_NEG_INF;
                nf.y = (f[i].y > 0.0f && lv[i].y > PC_NEG_INF) ? __logf(f[i].y) - lv[i].y : PC_NEG_INF;
                nf.z = (f[i].z > 0.0f && lv[i].z > PC_NEG_INF) ? __logf(f[i].z) - lv[i].z : PC_NEG_INF;
                nf.w = (f[i].w > 0.0f && lv[i].w > PC_NEG_INF) ? __logf(f[i].w) - lv[i].w : PC_NEG_INF;
                *reinterpret_cast<float4 *>(N + (int64_t)(id + k) * Bs + b) = nf;
                if (PLANES) nfv[i] = nf;
                mx[0] = fmaxf(mx[0], nf.x); mx[1] = fmaxf(mx[1], nf.y); mx[2] = fmaxf(mx[2], nf.z); mx[3] = fmaxf(mx[3], nf.w);
            }
        }
    }
    block_col_max<CL>(mx, red, wave, cl);
    if (in && rg == 0) *reinterpret_cast<float4 *>(nfmax + (int64_t)(id / K) * Bs + b) = make_float4(mx[0], mx[1], mx[2], mx[3]);
    if (PLANES) {
        // exp(log_nf - column maximum + PC_UP) of the block as bf16 operand planes for a sum layer whose backward pass
        // runs on the bf16 matrix cores (saves the launch of k_split_p), taken from a copy of the tile in LDS (row K: the
        // column maxima)
        constexpr int LDT = 4 * CL + 1;
        __shared__ float ptile[PLANES ? 129 * LDT : 1];
        if (in) {
#pragma unroll
            for (int i = 0; i < RPT; ++i) {
                const int k = rg + RG * i;
                if (k < K) {
                    float *dst = ptile + k * LDT + cl * 4;
                    dst[0] = nfv[i].x; dst[1] = nfv[i].y; dst[2] = nfv[i].z; dst[3] = nfv[i].w;
                }
            }
            if (rg == 0) {
                float *dst = ptile + 128 * LDT + cl * 4;
                dst[0] = mx[0]; dst[1] = mx[1]; dst[2] = mx[2]; dst[3] = mx[3];
            }
        }
        __syncthreads();
        const int n_ct = (int)(Bs / 32), lane = threadIdx.x & 63;
        constexpr int CTW = CL / 8;                                     // 32-column tiles of the workgroup
        for (int it = wave; it < (K / 16) * CTW; it += 4) {
            const int ks = it / CTW, cw = it % CTW, ct = (int)blockIdx.y * CTW + cw;
            if (ct >= n_ct) continue;
            const float top = ptile[128 * LDT + cw * 32 + (lane & 31)];
            split_value_rows(ptile + 16 * ks * LDT + cw * 32 + (lane & 31), LDT, top > PC_NEG_INF ? PC_UP - top : PC_NEG_INF,
                             (int64_t)id + 16 * ks, ct, n_ct, Ph, Pl, lane);
        }
    }
}

// ------------------------------------------------------------------------------------------
// product layers over input blocks in classes of equal parents (LayerTab::cls_*, ::tile)
// ------------------------------------------------------------------------------------------
// The leaf regions of a RAT-SPN: every product adds up the blocks of two classes (49 + 49), every class is added up by eight
// products.  k_prod_fwd asks L2 for a block once per product (13 GB for 1.6 GB of rows at D = 784, B = 512, and L2 is what it
// waits for).  Here a workgroup takes 4 x 4 products at once: at each place of the products' rows stand four blocks of the one or of
// the other side's classes, each loaded once and added to the four products that have it.  The sums are those of k_prod_fwd to the
// last bit -- four children in fp32, the fours in double, children ascending --; sums of a class taken once and added up by the
// products would need two reads per product instead, but round differently, and three EM steps on the same batch turn
// differences of 6e-5 in single weights into 3e-3.
// D = 784, B = 512: 1.01 ms -> 0.43.  Thread (k, c): row k, two adjacent columns; C2 column pairs per workgroup, T x T products, in 128
// registers for four waves per SIMD (0.57 ms with three).  The four tiles that share their classes run one
// after another on one XCD (workgroup h runs on XCD h mod 8), for the blocks to be in its L2.  So do the two column tiles of a
// 128-byte line where a tile has 16 columns (K = 64): on two XCDs each line was fetched twice (300 variables, K = 64, B = 1000: k_prod_fwd 322 us,
// tiles 350, now 295; B = 512 158, 142, 126).
template <int C2, int T>
__global__ __launch_bounds__(512, 4) void k_prod_tile(float *__restrict__ l, float *__restrict__ R, const int32_t *tile_words, int32_t n_tiles,
                                                   const int32_t *order_words, const int32_t *blk_words, int32_t K, int64_t Bs)
{
    typedef const int32_t __attribute__((address_space(4))) *TabPtr;       // (read as constants: scalar loads)
    __shared__ float red[T * T][8][2 * C2];                                // [product][wave][column]
    constexpr int U = 4;                                                // children of a round
    constexpr int PARTS = 16 / (T * T);                                 // workgroups of a 4 x 4 tile
    const int32_t n4 = (n_tiles * PARTS + 3) & ~3;
    const int32_t h = (int32_t)blockIdx.x, q = h >> 3, m = ((q >> 2) * 8 + (h & 7)) * 4 + (q & 3);
    constexpr int LINE = C2 < 16 ? 16 / C2 : 1;                         // column tiles of a line (Bs is a multiple of 32 columns)
    const int32_t part = m / LINE % n4, ti = part / PARTS, i0 = T * (part % PARTS / (4 / T)), j0 = T * (part % PARTS % (4 / T));
    const int64_t col0 = (int64_t)(m / LINE / n4 * LINE + m % LINE) * (2 * C2), b = col0 + 2 * (threadIdx.x % C2);
    if (ti >= n_tiles || col0 >= Bs) return;                            // the whole workgroup
    const TabPtr tw = (TabPtr)(uintptr_t)tile_words + PROD_TILE_WORDS * (int64_t)ti, blk = (TabPtr)(uintptr_t)blk_words;
    const TabPtr order = (TabPtr)(uintptr_t)order_words + tw[24];
    const int k = threadIdx.x / C2, wave = threadIdx.x >> 6;
    const int32_t n = tw[25];
    double2 s[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) { s[i][j] = make_double2(0, 0); }
    int32_t at_a = 0, at_b = 0, ids[U][T];
    uint32_t sides = 0;
    auto places = [&](int32_t p0) {                                     // the blocks at the places p0 .. p0 + U - 1 of the products' rows
        sides = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool on = p0 + u < n;
            const int sd = on ? (order[(p0 + u) >> 5] >> ((p0 + u) & 31)) & 1 : 0;
#pragma unroll
            for (int i = 0; i < T; ++i) ids[u][i] = on ? blk[sd ? tw[4 + j0 + i] + at_b : tw[i0 + i] + at_a] : 0;
            at_b += on && sd; at_a += on && !sd;
            sides |= (uint32_t)sd << u;
        }
    };
    places(0);
    for (int32_t p0 = 0; p0 < n; p0 += U) {
        float2 y[U][T];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < T; ++i) y[u][i] = *reinterpret_cast<const float2 *>(l + (int64_t)(ids[u][i] + k) * Bs + b);
        const uint32_t sides_now = sides;                               // (past the end: the null block's rows, 0)
        places(p0 + U);
        float2 part[T][T];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool sd = (sides_now >> u) & 1;                       // uniform
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int j = 0; j < T; ++j) {
                    const float2 x = sd ? y[u][j] : y[u][i];
                    part[i][j].x = u == 0 ? x.x : part[i][j].x + x.x; part[i][j].y = u == 0 ? x.y : part[i][j].y + x.y;
                }
        }
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int j = 0; j < T; ++j) { s[i][j].x += (double)part[i][j].x; s[i][j].y += (double)part[i][j].y; }
    }
    // renormalise: the column maxima of a product's K rows
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) {
            float mx = (float)s[i][j].x, my = (float)s[i][j].y;
#pragma unroll
            for (int o = C2; o < 64; o <<= 1) { mx = fmaxf(mx, __shfl_xor(mx, o)); my = fmaxf(my, __shfl_xor(my, o)); }
            if ((threadIdx.x & 63) < C2) { red[T * i + j][wave][2 * (threadIdx.x % C2)] = mx; red[T * i + j][wave][2 * (threadIdx.x % C2) + 1] = my; }
        }
    __syncthreads();
    const int n_waves = (int)blockDim.x >> 6, c0 = 2 * (threadIdx.x % C2);
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) {
            const int32_t id = tw[8 + 4 * (i0 + i) + j0 + j];
            if (id == 0) continue;
            float mx = PC_NEG_INF, my = PC_NEG_INF;
            for (int w = 0; w < n_waves; ++w) { mx = fmaxf(mx, red[T * i + j][w][c0]); my = fmaxf(my, red[T * i + j][w][c0 + 1]); }
            mx = mx > PC_NEG_INF ? rintf(mx) : 0.0f;
            my = my > PC_NEG_INF ? rintf(my) : 0.0f;
            if (k == 0) *reinterpret_cast<float2 *>(R + (int64_t)(id / K) * Bs + b) = make_float2(mx, my);   // (R of input blocks is 0)
            *reinterpret_cast<float2 *>(l + (int64_t)(id + k) * Bs + b) = make_float2((float)(s[i][j].x - (double)mx), (float)(s[i][j].y - (double)my));
        }
}

// Backward, the flow that a class's blocks share is summed once and stored to each (0.49 -> 0.25 ms at D = 784, B = 512).  Workgroup = one
// class x 4 CL columns as in k_prod_bwd; gridDim.z shares of the class's blocks, each of which sums the parents again (they are few).
template <int RPT, int U, int CL>
__global__ __launch_bounds__(256) void k_class_bwd(float *F, const ClassesDev c, int32_t K, int64_t Bs)
{
    constexpr int RG = 256 / CL;
    const int rg = threadIdx.x / CL, cl = threadIdx.x % CL;
    const int64_t b = (int64_t)blockIdx.y * (4 * CL) + cl * 4;
    if (b >= Bs) return;
    const int32_t p1 = c.par_ptr[blockIdx.x + 1];
    float4 f[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) f[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int32_t p0 = c.par_ptr[blockIdx.x]; p0 < p1; p0 += U) {
        float4 t[U][RPT];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool on = p0 + u < p1;                               // uniform over the workgroup
            const int32_t pa = on ? c.par[p0 + u] : 0;
#pragma unroll
            for (int i = 0; i < RPT; ++i) {
                const int k = rg + RG * i;
                t[u][i] = (on && k < K) ? *reinterpret_cast<const float4 *>(F + (int64_t)(pa + k) * Bs + b) : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < RPT; ++i) { f[i].x += t[u][i].x; f[i].y += t[u][i].y; f[i].z += t[u][i].z; f[i].w += t[u][i].w; }
    }
    const bool first = c.first[blockIdx.x] != 0;
    const int32_t j1 = c.ptr[blockIdx.x + 1];
    for (int32_t j = c.ptr[blockIdx.x] + (int32_t)blockIdx.z; j < j1; j += (int32_t)gridDim.z) {
        const int32_t id = c.blk[j];
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int k = rg + RG * i;
            if (k >= K) continue;
            float4 *dst = reinterpret_cast<float4 *>(F + (int64_t)(id + k) * Bs + b);
            float4 v = f[i];
            if (!first) { const float4 old = *dst; v = make_float4(old.x + v.x, old.y + v.y, old.z + v.z, old.w + v.w); }
            *dst = v;
        }
    }
}

// ------------------------------------------------------------------------------------------
// generic sum-layer kernels (any K, one thread per output, no matrix cores) -- the node x sample
// parallelisation of Sec. 3, kept for block sizes the MFMA kernels do not cover
// ------------------------------------------------------------------------------------------
__device__ inline void lse_push(float &m, float &s, float t)
{
    if (t > m) { s = s * __expf(m - t) + 1.0f; m = t; }
    else s += __expf(t - m);
}

__global__ __launch_bounds__(256) void k_sum_fwd_generic(const float *__restrict__ theta, const float *__restrict__ lch,
                                                         float *__restrict__ l, float *__restrict__ R, const int32_t *__restrict__ ids,
                                                         const int32_t *__restrict__ nbr, const int32_t *__restrict__ par,
                                                         int32_t n_rows, int32_t width, int32_t K, int64_t Bs)
{
    const int64_t total = (int64_t)n_rows * K * Bs;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t row = t / Bs, b = t - row * Bs;
        const int32_t r = (int32_t)(row / K), i = (int32_t)(row - (int64_t)r * K);
        float Rn = PC_NEG_INF;
        for (int j = 0; j < width; ++j)
            if (par[(int64_t)r * width + j] != 0) Rn = fmaxf(Rn, R[(int64_t)(nbr[(int64_t)r * width + j] / K) * Bs + b]);
        float m = PC_NEG_INF, s = 0.0f;
        for (int j = 0; j < width; ++j) {
            const int32_t ns = nbr[(int64_t)r * width + j], ps = par[(int64_t)r * width + j];
            if (ps == 0) continue;
            const float d = R[(int64_t)(ns / K) * Bs + b] - Rn;
            for (int jj = 0; jj < K; ++jj) {
                const float th = theta[(int64_t)ps + (int64_t)i * K + jj];
                const float v = lch[(int64_t)(ns + jj) * Bs + b] + d;
                if (th > 0.0f && v > PC_NEG_INF) lse_push(m, s, __logf(th) + v);
            }
        }
        l[(int64_t)(ids[r] + i) * Bs + b] = m > PC_NEG_INF ? m + __logf(s) : PC_NEG_INF;
        if (i == 0) R[(int64_t)(ids[r] / K) * Bs + b] = Rn;
    }
}

__global__ __launch_bounds__(256) void k_sum_bwd_child_generic(const float *__restrict__ theta, const float *__restrict__ l,
                                                               const float *__restrict__ R, const float *__restrict__ N,
                                                               float *__restrict__ F, const int32_t *__restrict__ ids,
                                                               const int32_t *__restrict__ nbr, const int32_t *__restrict__ par,
                                                               const int32_t *__restrict__ flags, int32_t n_rows,
                                                               int32_t width, int32_t K, int64_t Bs)
{
    const int64_t total = (int64_t)n_rows * K * Bs;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t row = t / Bs, b = t - row * Bs;
        const int32_t r = (int32_t)(row / K), jj = (int32_t)(row - (int64_t)r * K);
        const float Rc = R[(int64_t)(ids[r] / K) * Bs + b];
        float m = PC_NEG_INF, s = 0.0f;
        for (int j = 0; j < width; ++j) {
            const int32_t ms = nbr[(int64_t)r * width + j], ps = par[(int64_t)r * width + j];
            if (ps == 0) continue;
            const float d = Rc - R[(int64_t)(ms / K) * Bs + b];
            for (int i = 0; i < K; ++i) {
                const float th = theta[(int64_t)ps + (int64_t)i * K + jj];
                const float nf = N[(int64_t)(ms + i) * Bs + b] + d;
                if (th > 0.0f && nf > PC_NEG_INF) lse_push(m, s, __logf(th) + nf);
            }
        }
        const int64_t at = (int64_t)(ids[r] + jj) * Bs + b;
        const float lc = l[at];
        const float add = (m > PC_NEG_INF && lc > PC_NEG_INF) ? __expf(m + __logf(s) + lc) : 0.0f;
        F[at] = (flags[r] & 2) ? add : F[at] + add;                     // first layer that feeds the block stores
    }
}

__global__ __launch_bounds__(256) void k_sum_bwd_param_generic(const float *__restrict__ theta, const float *__restrict__ l,
                                                               const float *__restrict__ R, const float *__restrict__ N,
                                                               float *__restrict__ G, const int32_t *__restrict__ ids,
                                                               const int32_t *__restrict__ nbr, const int32_t *__restrict__ par,
                                                               int32_t n_rows, int32_t width, int32_t K, int64_t Bs, int32_t B,
                                                               int atomic)
{
    const int64_t per_row = (int64_t)width * K * K;
    const int64_t total = (int64_t)n_rows * per_row;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
        const int32_t r = (int32_t)(t / per_row);
        int64_t rem = t - (int64_t)r * per_row;
        const int32_t j = (int32_t)(rem / ((int64_t)K * K));
        rem -= (int64_t)j * K * K;
        const int32_t i = (int32_t)(rem / K), jj = (int32_t)(rem - (int64_t)i * K);
        const int32_t ns = nbr[(int64_t)r * width + j], ps = par[(int64_t)r * width + j];
        if (ps == 0) continue;
        const float th = theta[(int64_t)ps + (int64_t)i * K + jj];
        if (!(th > 0.0f)) continue;
        const float *nrow = N + (int64_t)(ids[r] + i) * Bs;
        const float *lrow = l + (int64_t)(ns + jj) * Bs;
        const float *Rs = R + (int64_t)(ids[r] / K) * Bs, *Rc = R + (int64_t)(ns / K) * Bs;
        const float lth = __logf(th);                                   // inside the exponent: every term is an edge flow <= 1
        float acc = 0.0f;
        for (int b = 0; b < B; ++b) {
            const float nf = nrow[b], lc = lrow[b];
            if (nf > PC_NEG_INF && lc > PC_NEG_INF) acc += __expf(nf + lc + (Rc[b] - Rs[b]) + lth);
        }
        float *dst = G + (int64_t)ps + (int64_t)i * K + jj;
        if (atomic) atomicAdd(dst, acc); else *dst += acc;
    }
}

// ------------------------------------------------------------------------------------------
// small-block sum-layer kernels (K in {1, 2, 4, 8}): block-based parallelisation (Sec. 4.1) on the vector
// ALU.  A thread owns one sample column of one node block: it reads each of the K neighbour values once,
// exponentiates it once and uses it for all K outputs of the block -- the K-fold cut in reloads and in
// exponentials that Sec. 4.1 describes.  The K x K weights have workgroup-uniform addresses and ride in scalar
// registers.  Linear-space accumulators with a running maximum, as in the MFMA kernels.
// ------------------------------------------------------------------------------------------
// Two-factor split of a parameter-flow term exp(log_nf_s + l_c + dR) of one sample (dR = R_child - R_sum, an exact
// integer).  With a = max_s log_nf_s over the sum block and g = a + dR -- the children are product blocks, whose
// largest residual lies within +-0.5 of 0, so e^g is the size of the sample's largest term in this block pair, and
// theta p_c / p_s <= 1 with theta >= FLT_MIN bounds g by 87.3 --
//   first factor  exp(log_nf_s - a + s_b)            <= e^s_b
//   second factor exp(l_c + g - s_b - PC_SPLIT_SCALE) <= e^(s_b + 0.5)     with s_b = (g - PC_SPLIT_SCALE) / 2 <= 31.65
// Any per-sample shift is valid (it only moves scale between the factors); this one gives both factors the same
// head-room, so each keeps 87 + s_b nats below its largest value.  The products carry the fixed scale e^-PC_SPLIT_SCALE,
// taken out again when the flow is written: a sum over up to 2^21 samples times a thousand tied instances of terms
// as large as 1 / FLT_MIN then still fits fp32.  What is lost: a product below FLT_MIN, i.e. a term below
// FLT_MIN * e^PC_SPLIT_SCALE = 3.2e-28, and -- only in a sample with g > 23.4, which takes a weight below e^-23 on an
// edge that nevertheless carries the block's largest flow ratio -- a term below e^(g / 2 - 75) whose factor underflows
// (at most e^-31.4).  (A fixed first shift of 31 lost every term of a sample with g < -32, the common case of a block
// pair that carries little flow.)
#define PC_SPLIT_SCALE 24.0f
#define PC_SPLIT_CAP 32.5f
#define PC_SPLIT_OUT 2.6489122e10f   /* e^24 */
__device__ inline float pc_split_shift(float g) { return fminf(fmaxf(0.5f * (g - PC_SPLIT_SCALE), -40.0f), 31.5f); }
// flow += theta * sum * e^24 without leaving the fp32 range on the way: theta may be FLT_MIN (theta * sum would be
// subnormal) and the sum as large as e^85 (sum * e^24 would overflow); theta * 2^40 is a normal number below 2^41 and
// (theta * 2^40) * sum = flow * 2^5.4
__device__ inline float pc_flow_out(float th, float sum) { return ((th * 0x1p+40f) * sum) * (PC_SPLIT_OUT * 0x1p-40f); }
template <int K>
__global__ __launch_bounds__(256) void k_sum_fwd_small(const float *__restrict__ theta, const float *__restrict__ lch,
                                                       float *__restrict__ l, float *__restrict__ R, const int32_t *__restrict__ ids,
                                                       const int32_t *__restrict__ nbr, const int32_t *__restrict__ par,
                                                       const int32_t *__restrict__ flags, int32_t width, int64_t Bs)
{
    const int r = blockIdx.x;
    const int64_t b = (int64_t)blockIdx.y * 256 + threadIdx.x;
    if (b >= Bs) return;
    const int32_t *row_nbr = nbr + (int64_t)r * width, *row_par = par + (int64_t)r * width;
    const int32_t cnt = flags[r] >> 8, id = ids[r];
    float acc[K];
#pragma unroll
    for (int i = 0; i < K; ++i) acc[i] = 0.0f;
    float m = PC_NEG_INF, Rrow = PC_NEG_INF;                            // Rrow: largest child reference seen so far
    // U neighbours at a time: their ids first, then all their loads together -- one memory round trip per U
    // neighbours (with one thread per sample column nothing else hides that latency at the smallest block sizes)
    constexpr int U = K == 1 ? 8 : K == 2 ? 4 : K == 4 ? 2 : 1;
    for (int j0 = 0; j0 < cnt; j0 += U) {
        int32_t nsv[U], pov[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int jc = j0 + u < cnt ? j0 + u : cnt - 1;             // past the end: the last neighbour again, unused
            nsv[u] = row_nbr[jc];
            pov[u] = row_par[jc];
        }
        float vv[U][K], RBv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int jj = 0; jj < K; ++jj) vv[u][jj] = lch[(int64_t)(nsv[u] + jj) * Bs + b];
            RBv[u] = R[(int64_t)(nsv[u] / K) * Bs + b];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (j0 + u >= cnt) break;                                   // uniform over the workgroup
            const float *th = theta + pov[u];
            const float(&v)[K] = vv[u];
            const float RB = RBv[u];
            const float Rn = fmaxf(Rrow, RB);
            m += Rrow - Rn;                                             // exact integer shift; -inf stays -inf
            Rrow = Rn;
            const float d = RB - Rrow;
            float bm = v[0];
#pragma unroll
            for (int jj = 1; jj < K; ++jj) bm = fmaxf(bm, v[jj]);
            bm += d;
            if (bm > m + PC_LAZY) {
                const float sc = pc_half_scale(m - bm);                 // m = -inf: the accumulators are 0
#pragma unroll
                for (int i = 0; i < K; ++i) acc[i] = acc[i] * sc * sc;
                m = bm;
            }
            const float sh = m > PC_NEG_INF ? d - m + PC_UP : 0.0f;     // dead column: v = -inf -> p = 0
            float pv[K];
#pragma unroll
            for (int jj = 0; jj < K; ++jj) pv[jj] = __expf(v[jj] + sh);
#pragma unroll
            for (int i = 0; i < K; ++i) {
#pragma unroll
                for (int jj = 0; jj < K; ++jj) acc[i] = fmaf(th[i * K + jj], pv[jj], acc[i]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < K; ++i) l[(int64_t)(id + i) * Bs + b] = acc[i] > 0.0f ? m - PC_UP + __logf(acc[i]) : PC_NEG_INF;
    R[(int64_t)(id / K) * Bs + b] = Rrow;
}

template <int K>
__global__ __launch_bounds__(256) void k_sum_bwd_small(const float *__restrict__ theta, const float *__restrict__ l,
                                                       const float *__restrict__ R, const float *__restrict__ N,
                                                       const float *__restrict__ nfmax, float *__restrict__ F,
                                                       const int32_t *__restrict__ ids, const int32_t *__restrict__ nbr,
                                                       const int32_t *__restrict__ par, const int32_t *__restrict__ flags,
                                                       int32_t width, int64_t Bs)
{
    const int r = blockIdx.x;
    const int64_t b = (int64_t)blockIdx.y * 256 + threadIdx.x;
    if (b >= Bs) return;
    const int32_t *row_nbr = nbr + (int64_t)r * width, *row_par = par + (int64_t)r * width;
    const int32_t fl = flags[r], id = ids[r];
    const int32_t cnt = fl >> 8;
    const bool first = (fl & 2) != 0;
    const float Rc = R[(int64_t)(id / K) * Bs + b];
    float lown[K];
#pragma unroll
    for (int jj = 0; jj < K; ++jj) lown[jj] = l[(int64_t)(id + jj) * Bs + b];
    float acc[K];
#pragma unroll
    for (int jj = 0; jj < K; ++jj) acc[jj] = 0.0f;
    float m = PC_NEG_INF;
    constexpr int U = K == 1 ? 8 : K == 2 ? 4 : K == 4 ? 2 : 1;         // neighbours in flight, as in the forward kernel
    for (int j0 = 0; j0 < cnt; j0 += U) {
        int32_t msv[U], pov[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int jc = j0 + u < cnt ? j0 + u : cnt - 1;
            msv[u] = row_nbr[jc];
            pov[u] = row_par[jc];
        }
        float nvv[U][K], Rp[U], bmv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int i = 0; i < K; ++i) nvv[u][i] = N[(int64_t)(msv[u] + i) * Bs + b];
            Rp[u] = R[(int64_t)(msv[u] / K) * Bs + b];
            bmv[u] = nfmax[(int64_t)(msv[u] / K) * Bs + b];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (j0 + u >= cnt) break;                                   // uniform over the workgroup
            const float *th = theta + pov[u];
            const float(&nv)[K] = nvv[u];
            const float d = Rc - Rp[u];
            const float bm = bmv[u] + d;
            if (bm > m + PC_LAZY) {
                const float sc = pc_half_scale(m - bm);
#pragma unroll
                for (int jj = 0; jj < K; ++jj) acc[jj] = acc[jj] * sc * sc;
                m = bm;
            }
            const float sh = m > PC_NEG_INF ? d - m + PC_UP : 0.0f;
            float pv[K];
#pragma unroll
            for (int i = 0; i < K; ++i) pv[i] = __expf(nv[i] + sh);
#pragma unroll
            for (int i = 0; i < K; ++i)
#pragma unroll
                for (int jj = 0; jj < K; ++jj) acc[jj] = fmaf(th[i * K + jj], pv[i], acc[jj]);
        }
    }
#pragma unroll
    for (int jj = 0; jj < K; ++jj) {
        const int64_t at = (int64_t)(id + jj) * Bs + b;
        const float add = (acc[jj] > 0.0f && lown[jj] > PC_NEG_INF) ? __expf(__logf(acc[jj]) + (m - PC_UP) + lown[jj]) : 0.0f;
        if (first) F[at] = add;                                         // first layer that feeds the block stores
        else if (add > 0.0f) F[at] += add;
    }
}

// Backward to the parameters for small blocks, by parameter block like k_param_flow_mfma: one wave per parameter
// block, lanes = samples.  Per pass a lane holds IG x K partial sums of the two-factor products (the same
// balanced split as the MFMA kernel); at the end the 64 lanes are reduced with an exchange-and-halve butterfly
// (each step a lane hands half of its values to its partner and adds the partner's other half), which costs
// about 4 operations per value instead of 12.
template <int K, int IG>
__global__ __launch_bounds__(256) void k_param_flow_small(const float *__restrict__ theta, const float *__restrict__ l,
                                                          const float *__restrict__ R, const float *__restrict__ N,
                                                          const float *__restrict__ nfmax, float *__restrict__ G,
                                                          const int32_t *__restrict__ pf_pb, const int32_t *__restrict__ pf_ptr,
                                                          const int32_t *__restrict__ pf_sum, const int32_t *__restrict__ pf_child,
                                                          int32_t n_pb, int64_t Bs)
{
    constexpr int A = IG * K;                                           // values per lane and pass
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int64_t pidx = (int64_t)blockIdx.x * 4 + wave;
    if (pidx >= n_pb) return;                                           // wave-uniform; no workgroup barrier below
    const int32_t pb = pf_pb[pidx];
    const int i0 = pf_ptr[pidx], i1 = pf_ptr[pidx + 1];
    for (int ig = 0; ig < K; ig += IG) {
        float acc[A];
#pragma unroll
        for (int a = 0; a < A; ++a) acc[a] = 0.0f;
        for (int inst = i0; inst < i1; ++inst) {
            const int32_t ms = pf_sum[inst], ns = pf_child[inst];
            for (int64_t b = lane; b < Bs; b += 64) {
                const float mx = nfmax[(int64_t)(ms / K) * Bs + b];
                const float dR = R[(int64_t)(ns / K) * Bs + b] - R[(int64_t)(ms / K) * Bs + b];
                const bool live = mx > PC_NEG_INF;                      // dead sample: both factors 0
                const float sb = pc_split_shift(mx + dR);
                const float qa = live ? sb - mx : PC_NEG_INF;
                const float qb = live ? mx + dR - sb - PC_SPLIT_SCALE : PC_NEG_INF;
                float fa[IG], fb[K];
#pragma unroll
                for (int i = 0; i < IG; ++i) fa[i] = __expf(N[(int64_t)(ms + ig + i) * Bs + b] + qa);
#pragma unroll
                for (int jj = 0; jj < K; ++jj) fb[jj] = __expf(fminf(l[(int64_t)(ns + jj) * Bs + b] + qb, PC_SPLIT_CAP));
#pragma unroll
                for (int i = 0; i < IG; ++i)
#pragma unroll
                    for (int jj = 0; jj < K; ++jj) acc[i * K + jj] = fmaf(fa[i], fb[jj], acc[i * K + jj]);
            }
        }
        // reduce over the 64 lanes
        int cur = A, idx = 0;                                           // idx: first of the values this lane still holds
#pragma unroll
        for (int dist = 32; dist >= 1; dist >>= 1) {
            if (cur > 1) {
                const int h = cur / 2;
                const bool up = (lane & dist) != 0;
#pragma unroll
                for (int e = 0; e < A / 2; ++e) {
                    if (e < h) {
                        const float lo = acc[e], hi = acc[e + h];
                        const float give = up ? lo : hi, keep = up ? hi : lo;
                        acc[e] = keep + __shfl_xor(give, dist);
                    }
                }
                idx += up ? h : 0;
                cur = h;
            } else {
                acc[0] += __shfl_xor(acc[0], dist);
            }
        }
        // cur values per lane; lanes that differ only in the bits of the plain-sum steps hold copies
        constexpr int HALVINGS = A >= 64 ? 6 : (A == 32 ? 5 : A == 16 ? 4 : A == 8 ? 3 : A == 4 ? 2 : A == 2 ? 1 : 0);
        constexpr int COPIES = 64 >> HALVINGS;
        if ((lane & (COPIES - 1)) == 0) {
#pragma unroll
            for (int e = 0; e < (A >= 64 ? A / 64 : 1); ++e) {
                const int a = idx + e;                                  // = i * K + jj inside this pass
                const int64_t at = (int64_t)pb + (int64_t)ig * K + a;
                const float th = theta[at];
                if (th > 0.0f) G[at] += pc_flow_out(th, acc[e]);
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// K = 16 on the matrix cores: one block is one v_mfma_f32_16x16x4_f32 tile
// ------------------------------------------------------------------------------------------
// A (16 x 4): lane holds A[lane % 16][lane / 16], B (4 x 16): B[lane / 16][lane % 16], D: register r holds
// D[4 * (lane / 16) + r][lane % 16].  Forward and backward to the children: a wave owns one node block x 32 columns; per
// neighbour block step e pairs lane group g with node 4 g + e, so the forward weights are one 16-byte load per lane (the
// block's 1 KiB, coalesced) and nothing goes through LDS.  U neighbours are requested together.  SPLIT = 4: the waves of a
// workgroup share one tile and deal the neighbours among them (launches too small to fill the chip).  References as in the
// other kernels: forward the largest integer reference of a live neighbour, backward the running maximum of the parents'.
// What bounds it: exponentials (a quarter of the vector rate) and MFMAs in turn, eight of each per neighbour.  Measured on
// 28 sets of 1024 x 1024, 30 % of the 16 x 16 blocks kept, B = 333 (6.2 GFLOP): forward 526 -> 179 us, backward 432 -> 165 us
// against the vector kernel (64 columns per wave: 205 and 216 us, the operands of four neighbours then take 170 - 210 registers).
// Rows: GroupSet, or GroupDev for a layer of one group.  The set is 332 bytes of kernel arguments in six cache lines, each read before
// anything else can be: 5 sets of 256 x 256, B = 64, forward 5.5, backward 5.6 and 4.8 us a launch with the set, 5.3, 5.5 and 4.1 with
// the group alone.
template <bool BWD, int SPLIT, class Rows>
__global__ __launch_bounds__(256) void k_sum_16(const float *__restrict__ theta, const float *__restrict__ X, float *__restrict__ l,
                                                float *__restrict__ R, const float *__restrict__ nfmax, float *__restrict__ F,
                                                const Rows rows, int64_t Bs)
{
    constexpr int K = 16, U = 4, NC = 2;
    __shared__ floatx4 part[SPLIT > 1 ? 4 : 1][NC][SPLIT > 1 ? 64 : 1];
    __shared__ float pref[SPLIT > 1 ? 4 : 1][NC][16];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 4, j16 = lane & 15;
    const GroupRow gr = locate_row<PC_ROWS_MULTI>(rows, blockIdx.x);
    const int r = gr.r;
    const int64_t cg = SPLIT > 1 ? blockIdx.y : (int64_t)blockIdx.y * 4 + wave;   // group of NC column tiles
    if (SPLIT == 1 && cg * NC * 16 >= Bs) return;
    int64_t col[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) col[c] = (cg * NC + c) * 16 + j16;     // Bs is a multiple of 32
    const int32_t *row_nbr = gr.nbr + (int64_t)r * gr.width, *row_par = gr.par + (int64_t)r * gr.width;
    const int32_t id = gr.ids[r], fl = gr.aux[r], cnt = fl >> 8;
    float Rown[NC];
    floatx4 lown[BWD ? NC : 1];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        Rown[c] = BWD ? R[(int64_t)(id / K) * Bs + col[c]] : 0.0f;
        if (BWD)
#pragma unroll
            for (int e = 0; e < 4; ++e) lown[c][e] = l[(int64_t)(id + 4 * g + e) * Bs + col[c]];
    }
    floatx4 acc[NC];
    float m[NC];                                                        // reference of acc, -inf: nothing live yet
#pragma unroll
    for (int c = 0; c < NC; ++c) { acc[c] = floatx4{0.f, 0.f, 0.f, 0.f}; m[c] = PC_NEG_INF; }

    const int first_j = SPLIT > 1 ? wave : 0;
    for (int j0 = first_j; j0 < cnt; j0 += U * SPLIT) {
        floatx4 th[U], v[U][NC];
        float rb[U][NC], bm[BWD ? U : 1][NC];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = j0 + u * SPLIT < cnt ? j0 + u * SPLIT : j0;   // past the end: the first again, unused
            const int32_t ns = row_nbr[j], ps = row_par[j];
            if (BWD) {
#pragma unroll
                for (int e = 0; e < 4; ++e) th[u][e] = theta[(int64_t)ps + (4 * g + e) * K + j16];
            } else {
                th[u] = *reinterpret_cast<const floatx4 *>(theta + (int64_t)ps + j16 * K + 4 * g);
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[u][c][e] = X[(int64_t)(ns + 4 * g + e) * Bs + col[c]];
                rb[u][c] = R[(int64_t)(ns / K) * Bs + col[c]];
                if (BWD) bm[u][c] = nfmax[(int64_t)(ns / K) * Bs + col[c]];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (j0 + u * SPLIT >= cnt) break;                           // wave-uniform
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const float d = BWD ? Rown[c] - rb[u][c] : rb[u][c];
                const float top = BWD ? bm[u][c] + d : d;
                if (__any(top > (BWD ? m[c] + PC_LAZY : m[c]))) {       // a larger reference (forward: unless the block is dead)
                    float live = v[u][c][0];
                    if (!BWD) {
                        live = fmaxf(fmaxf(live, v[u][c][1]), fmaxf(v[u][c][2], v[u][c][3]));
                        live = fmaxf(live, __shfl_xor(live, 16)); live = fmaxf(live, __shfl_xor(live, 32));
                    }
                    const bool raise = (BWD ? top > m[c] + PC_LAZY : top > m[c] && live > PC_NEG_INF);
                    const float mn = raise ? top : m[c];
                    const float sc = mn > PC_NEG_INF ? pc_half_scale(m[c] - mn) : 1.0f;
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[c][e] = acc[c][e] * sc * sc;
                    m[c] = mn;
                }
                const float sh2 = m[c] > PC_NEG_INF ? (d - m[c] + PC_UP) * PC_LOG2E : 0.0f;   // dead so far: v = -inf
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float p = __builtin_amdgcn_exp2f(fmaf(v[u][c][e], PC_LOG2E, sh2));
                    acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(th[u][e], p, acc[c], 0, 0, 0);
                }
            }
        }
    }
    if (SPLIT > 1) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            part[wave][c][lane] = acc[c];
            if (g == 0) pref[wave][c][j16] = m[c];
        }
        __syncthreads();
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (SPLIT > 1) {
            if (wave != c % 4) continue;                                // wave-uniform
            float mt = PC_NEG_INF;
#pragma unroll
            for (int w = 0; w < 4; ++w) mt = fmaxf(mt, pref[w][c][j16]);
            floatx4 tot = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float mw = pref[w][c][j16], sc = mw > PC_NEG_INF ? pc_half_scale(mw - mt) : 0.0f;
                const floatx4 pw = part[w][c][lane];
#pragma unroll
                for (int e = 0; e < 4; ++e) tot[e] += pw[e] * sc * sc;
            }
            acc[c] = tot;
            m[c] = mt;
        }
        if (!BWD && g == 0) R[(int64_t)(id / K) * Bs + col[c]] = m[c] > PC_NEG_INF ? m[c] : 0.0f;   // all dead: any finite reference
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t at = (int64_t)(id + 4 * g + e) * Bs + col[c];
            if (BWD) {
                const float add = m[c] > PC_NEG_INF ? __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(acc[c][e]) + (lown[c][e] + (m[c] - PC_UP)) * PC_LOG2E)
                                                    : 0.0f;
                if (fl & 2) F[at] = add;                                // first layer that feeds the block stores
                else if (add > 0.0f) F[at] += add;
            } else {
                // ln(sum) - PC_UP, the logarithm taken of sum / 2^24 (as in k_sum_mfma)
                l[at] = fmaf(__builtin_amdgcn_logf(acc[c][e] * 0x1p-24f), 0.6931471805599453f, 16.635532333f - PC_UP);
            }
        }
    }
}

// Parameter flows, K = 16: by parameter block as in k_param_flow_mfma, the batch on the reduction index: a wave takes one
// 16 x 16 block (n_split > 1: a share of its pairs, added atomically) and 16 samples per four MFMAs, lane (row, g) holding
// samples 4 g .. 4 g + 3 of its row -- 16-byte loads, no staging.  Per 64 samples the shifts of the two factors are computed once,
// lane = sample, and handed round through LDS (2 KiB per workgroup; LDS operations of one wave complete in order): 262 -> 216 us
// against every lane computing the shifts of its own samples, 382 us on the vector ALU (34 312 blocks, B = 333).
__global__ __launch_bounds__(256) void k_param_flow_16(const float *__restrict__ theta, const float *__restrict__ l,
                                                       const float *__restrict__ R, const float *__restrict__ N,
                                                       const float *__restrict__ nfmax, float *__restrict__ G,
                                                       const int32_t *__restrict__ pf_pb, const int32_t *__restrict__ pf_ptr,
                                                       const int32_t *__restrict__ pf_sum, const int32_t *__restrict__ pf_child,
                                                       int32_t n_pb, int32_t n_split, int64_t Bs)
{
    constexpr int K = 16, CH = 4;
    __shared__ float q[4][2][64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 4, j16 = lane & 15;
    const int64_t w = (int64_t)blockIdx.x * 4 + wave;
    const int pidx = (int)(w / n_split), spl = (int)(w % n_split);
    if (pidx >= n_pb) return;                                           // wave-uniform; no workgroup barrier below
    const int32_t pb = pf_pb[pidx];
    const int i0 = pf_ptr[pidx], i1 = pf_ptr[pidx + 1];
    floatx4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    for (int inst = i0 + spl; inst < i1; inst += n_split) {
        const int32_t ms = pf_sum[inst], ns = pf_child[inst];
        const float *np = N + (int64_t)(ms + j16) * Bs + 4 * g, *lp = l + (int64_t)(ns + j16) * Bs + 4 * g;
        for (int64_t b = 0; b < Bs; b += 64) {                          // Bs is a multiple of 32: the last round may be a half one
            const bool whole = b + 64 <= Bs;
            floatx4 nf[CH], lc[CH];
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int64_t at = b + (c < 2 || whole ? 16 * c : 0);
                nf[c] = *reinterpret_cast<const floatx4 *>(np + at);
                lc[c] = *reinterpret_cast<const floatx4 *>(lp + at);
            }
            const int64_t bl = b + (whole ? lane : lane & 31);
            const float mx = nfmax[(int64_t)(ms / K) * Bs + bl];
            const float gg = mx + (R[(int64_t)(ns / K) * Bs + bl] - R[(int64_t)(ms / K) * Bs + bl]), sb = pc_split_shift(gg);
            const bool live = mx > PC_NEG_INF && (whole || lane < 32);  // dead sample: both factors 0
            q[wave][0][lane] = live ? (sb - mx) * PC_LOG2E : PC_NEG_INF;
            q[wave][1][lane] = live ? (gg - sb - PC_SPLIT_SCALE) * PC_LOG2E : PC_NEG_INF;
            __builtin_amdgcn_wave_barrier();                            // the lanes below read what others wrote
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const floatx4 qa = *reinterpret_cast<const floatx4 *>(&q[wave][0][16 * c + 4 * g]);
                const floatx4 qb = *reinterpret_cast<const floatx4 *>(&q[wave][1][16 * c + 4 * g]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float a = __builtin_amdgcn_exp2f(fmaf(nf[c][e], PC_LOG2E, qa[e]));
                    const float p = __builtin_amdgcn_exp2f(fminf(fmaf(lc[c][e], PC_LOG2E, qb[e]), PC_SPLIT_CAP * PC_LOG2E));
                    acc[c & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, p, acc[c & 1], 0, 0, 0);
                }
            }
            __builtin_amdgcn_wave_barrier();                            // and write anew in the next round
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int64_t at = (int64_t)pb + (4 * g + e) * K + j16;
        const float th = theta[at], inc = pc_flow_out(th, acc[0][e] + acc[1][e]);
        if (th > 0.0f) {                                                // theta = 0: no flow (and never 0 * inf)
            if (n_split > 1) atomicAdd(G + at, inc); else G[at] += inc;
        }
    }
}

// ------------------------------------------------------------------------------------------
// MFMA sum-layer kernels (K % 32 == 0).  Workgroup = 4 waves; a wave owns 32 sample columns.
// ------------------------------------------------------------------------------------------

// Forward (role of Alg. 1) and backward-to-children (role of Alg. 4) share one kernel.
//
// A wave owns a tile of TM = 32*RT rows of one node block x 32 sample columns and a share of the row's
// neighbour chunks (KC = 32 nodes per chunk).  The rows are sum nodes (forward) or child product nodes
// (backward).  A workgroup holds 4 waves: SPLIT of them share one output tile and take the chunks
// round-robin (split of the reduction dimension, so that small batches still fill every SIMD with two
// waves -- a wave cannot overlap its own VALU work with its own MFMAs, a second wave can), the other
// factor 4/SPLIT spans adjacent column tiles.  Per chunk and wave:
//   * forward: the theta sub-block [TM x KC] (row = sum node, contiguous along the children) is fetched with
//     coalesced 16-byte loads and staged in a wave-private LDS tile only to reach the MFMA A-operand layout (LDS
//     operations of one wave complete in order, so no barrier and no double buffer are needed), then read back
//     whole into registers with 16-byte reads;
//   * backward: the operand is the transpose -- lane i needs theta[parent][child i] -- and that IS coalesced in
//     memory (32 consecutive children of one parent row), so it goes straight from L2 into the A-operand layout;
//   * the KC x 32 neighbour values go straight from L2 into the MFMA B-operand layout;
//   * the chunks follow one another without software pipelining: the loop needs 75-150 registers, so 3-6 waves
//     share a SIMD and hide each other's waits.  (A pipelined version -- two operand sets, theta of chunk c+1
//     staged during the arithmetic of chunk c, 190-230 registers, two waves per SIMD -- was slower in every
//     configuration measured, and so was prefetching only the next theta sub-block.)  The exception is a launch
//     too small to put more than one wave on a SIMD (the top layers of a deep narrow circuit, a root): there the
//     PF instantiation requests the next chunk before it works on the current one.
//   forward : value = l (log-prob residual) + (R_child - R_sum); the chunk maximum is taken in registers
//   backward: value = N (log F - l of the parent) + (R_child - R_parent); the block maximum is nfmax
// Values are shifted by the running per-sample maximum, exponentiated in registers and multiplied on
// the matrix cores (MFMA step q of a chunk pairs lanes 0-31 with node 8*(q/4) + q%4 and lanes 32-63 with
// node 8*(q/4) + 4 + q%4, so that one 16-byte LDS read yields the A operands of four steps); the
// accumulator stays in linear space and is rescaled when the maximum grows (the same sum as the
// per-block log-space update of the accumulator in Alg. 1 / Alg. 4, with one log per output instead of one
// per block).  Partial sums of the SPLIT waves are merged through LDS at the end.  No lane-dependent
// branch surrounds an MFMA.
template <int K, int RT, int SPLIT, bool BWD, bool MULTI, int MODE>
__global__ __launch_bounds__(SPLIT > 4 ? 64 * SPLIT : 256, SPLIT > 4 ? 1 : 2) void k_sum_mfma(const float *__restrict__ theta, float *__restrict__ l,
                                                     float *__restrict__ R, const float *__restrict__ N,
                                                     const float *__restrict__ nfmax, float *__restrict__ F,
                                                     const GroupSet gs, int64_t Bs)
{
    constexpr int KC = 32;
    constexpr int TM = 32 * RT;
    constexpr int SUB = K / TM;
    constexpr int NQ = KC / 2;                                          // MFMA steps per chunk
    constexpr int CPB = K / KC;                                         // chunks per neighbour block
    constexpr int WAVES = SPLIT > 4 ? SPLIT : 4;
    constexpr int NCT = WAVES / SPLIT;                                  // column tiles per workgroup
    constexpr int ES = RT * 16 / SPLIT;                                 // results per lane that a wave writes
    constexpr int NF4 = TM * KC / 4 / 64;                               // forward: 16-byte loads per lane per chunk
    constexpr int LDA = KC + 4;                                         // LDS row stride (floats): b128 reads conflict-free
    constexpr int TILE = BWD ? 0 : TM * LDA;                            // the backward kernel stages nothing
    constexpr int XCH = RT * 16 * 64 + 128;                             // one partial accumulator, its maxima and references
    constexpr int WSZ = TILE > XCH ? TILE : XCH;
    static_assert(K % TM == 0 && ES * SPLIT == RT * 16, "tile shape");
    __shared__ float lds[WAVES * WSZ];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int ct = wave / SPLIT, sp = wave % SPLIT;
    constexpr bool PART = MODE == 3;                                    // one row, its chunks in gs.first[2] parts, results to F (sum_parts)
    const GroupRow gr = locate_row<MULTI ? PC_ROWS_MULTI : PC_ROWS_ONE>(gs, PART ? 0 : blockIdx.x / SUB);
    const int r = gr.r, sub = blockIdx.x % SUB;
    const int64_t col0 = ((int64_t)blockIdx.y * NCT + ct) * 32;
    const bool active = col0 < Bs;                                      // wave-uniform
    const int64_t col = (active ? col0 : 0) + l32;
    const int32_t *row_nbr = gr.nbr + (int64_t)r * gr.width, *row_par = gr.par + (int64_t)r * gr.width;
    const int32_t id = gr.ids[r];
    const int32_t fl = gr.aux[r];                                       // wave-uniform
    // backward: the first layer of the sweep that feeds this block stores its flow, later ones accumulate
    const bool first = (fl & 2) != 0;
    float *buf = lds + wave * WSZ;
    const int n_row = (fl >> 8) * CPB;                                  // real neighbours; padding sits at the end of a row
    const int share = PART ? (n_row + gs.first[2] - 1) / gs.first[2] : n_row, chunk0 = PART ? (int)(blockIdx.x / SUB) * share : 0;
    const int n_chunks = PART ? min(chunk0 + share, n_row) : n_row;
    const int part = PART ? (int)blockIdx.x / SUB : 0;
    const int32_t part_row = PART ? row_nbr[part] : 0, part_top = PART ? row_nbr[gs.first[2] + part / (K / 2)] + part % (K / 2) * 2 : 0;

    // block reference of this row.  Backward: the row's own.  Forward: the maximum of the children's, found
    // on the fly -- Rrow is the maximum over the chunks seen so far and the running maximum m is relative to it
    float Rrow = PC_NEG_INF;
    if (BWD) Rrow = R[(int64_t)(id / K) * Bs + col];

    floatx16 acc[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[rt][e] = 0.0f;
    float m = PC_NEG_INF;
    // backward: the rows' own log-probabilities are needed only at the end; fetched now, their latency is hidden
    // behind the whole reduction (short reductions are latency-bound)
    // (the tile's rows through one buffer descriptor at its first row: per-lane offset = rows 4 * half + (0..3) of a
    // group of 8 rows and the column, scalar offset per row -- no per-element address arithmetic)
    // (a wave's results are the elements sp * ES, sp * ES + 1, ... of its tile's accumulators)
    auto row_off = [&](int q) { return __builtin_amdgcn_readfirstlane((int)((int64_t)(q / 16 * 32 + 8 * (q % 16 / 4) + q % 4) * Bs * 4)); };
    float lown[BWD ? ES : 1];
    const int ooff = (int)(((int64_t)(4 * half) * Bs + col) * 4);
    if (BWD) {
        const __amdgpu_buffer_rsrc_t rl =
            __builtin_amdgcn_make_buffer_rsrc((void *)(l + (int64_t)(id + sub * TM) * Bs), 0, PC_BUF_RANGE, PC_BUF_FLAGS);
#pragma unroll
        for (int k = 0; k < ES; ++k)
            lown[k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rl, ooff, row_off(sp * ES + k), 0));
    }

    // Operands of one chunk: `ar` the MFMA A operands (theta), `v` the neighbour values with their block scalars;
    // forward only: `th` carries the theta sub-block from global memory to the LDS tile.
    // All loads of the loop are buffer loads: a wave-uniform descriptor per chunk (base = first row of the chunk), a
    // loop-invariant per-lane byte offset and a compile-time scalar offset, so they need no vector address
    // arithmetic (the vector ALU issues instead of the matrix cores, not beside them).
    struct Operands {
        floatx4 th[BWD ? 1 : NF4];
        float ar[NQ][RT], v[NQ];
        float rb, bm;
    };
    const float *vsrc = N;                                              // forward: the children's log-probabilities (passed as N)
    int voff[4];                                                        // neighbour values: rows 0-3 of a group of 8 rows
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) voff[rr] = (int)(((int64_t)(4 * half + rr) * Bs + col) * 4);
    int soff[NQ / 4];                                                   // groups of 8 rows
#pragma unroll
    for (int g = 0; g < NQ / 4; ++g) soff[g] = __builtin_amdgcn_readfirstlane((int)((int64_t)(8 * g) * Bs * 4));
    // theta: forward, 16-byte pieces of rows of the sub-block; backward, one child column of parent rows 0 / 4
    const int toff = BWD ? ((4 * half) * K + l32) * 4 : ((lane / (KC / 4)) * K + (lane % (KC / 4)) * 4) * 4;

    float sh2 = 0.0f;
    constexpr bool PF = MODE == 1, WAIT_ALL = MODE == 2;                // schedules chosen by the launcher, see below
    // loads of chunk c into an operand set (nothing is computed on the loaded values here: any arithmetic would wait)
    auto load_chunk = [&](int c, Operands &o) {
        const int j = c / CPB, kc = c % CPB;
        const int32_t ps = row_par[j];
        const float *tb = BWD ? theta + (int64_t)ps + (int64_t)(kc * KC) * K + sub * TM
                              : theta + (int64_t)ps + (int64_t)(sub * TM) * K + kc * KC;
        const __amdgpu_buffer_rsrc_t rth = __builtin_amdgcn_make_buffer_rsrc((void *)tb, 0, PC_BUF_RANGE, PC_BUF_FLAGS);
        if (BWD) {
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    o.ar[q][rt] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                                rth, toff, ((8 * (q / 4) + (q % 4)) * K + rt * 32) * 4, 0));
        } else {
#pragma unroll
            for (int i = 0; i < NF4; ++i)                               // 64 lanes cover 64 / (KC / 4) rows
                o.th[i] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(
                                                          rth, toff, i * (64 / (KC / 4)) * K * 4, 0));
        }
        const int32_t ns = row_nbr[j];
        const float *src = vsrc + (int64_t)(ns + kc * KC) * Bs;
        const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc((void *)src, 0, PC_BUF_RANGE, PC_BUF_FLAGS);
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            o.v[q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rv, voff[q % 4], soff[q / 4], 0));
        o.rb = (R + (int64_t)(ns / K) * Bs)[(uint32_t)col];
        if (BWD) o.bm = (nfmax + (int64_t)(ns / K) * Bs)[(uint32_t)col];
    };
    // arithmetic of a loaded chunk
    auto run_chunk = [&](Operands &o) {
        // ---- forward: theta registers -> LDS tile -> A operands of the whole chunk ----
        if (!BWD) {
#pragma unroll
            for (int i = 0; i < NF4; ++i) {
                const int t = lane + i * 64;
                *reinterpret_cast<floatx4 *>(buf + (t / (KC / 4)) * LDA + (t % (KC / 4)) * 4) = o.th[i];
            }
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int g = 0; g < NQ / 4; ++g) {
                    const floatx4 a4 = *reinterpret_cast<const floatx4 *>(buf + (rt * 32 + l32) * LDA + 8 * g + 4 * half);
                    o.ar[4 * g + 0][rt] = a4[0]; o.ar[4 * g + 1][rt] = a4[1];
                    o.ar[4 * g + 2][rt] = a4[2]; o.ar[4 * g + 3][rt] = a4[3];
                }
        }
        // ---- per-chunk scalars: reference, maximum, rescale of the accumulator; leaves sh2 for the exponentials ----
        {
            if (!BWD) {                                                 // a larger reference: m moves by an exact integer
                const float Rn = fmaxf(Rrow, o.rb);
                m += Rrow - Rn;                                         // -inf stays -inf (rb is finite)
                Rrow = Rn;
            }
            const float d = BWD ? Rrow - o.rb : o.rb - Rrow;            // exact integer <= 0
            float cmax;
            if (BWD) {
                cmax = o.bm + d;
            } else {
                cmax = PC_NEG_INF;
#pragma unroll
                for (int q = 0; q < NQ; ++q) cmax = fmaxf(cmax, o.v[q]);
                cmax = fmaxf(cmax, __shfl_xor(cmax, 32)) + d;
            }
            const float m_new = cmax > m + PC_LAZY ? cmax : m;          // -inf + 8 = -inf: the first finite chunk sets it
            const bool dead = !(m_new > PC_NEG_INF);                    // every term of this column so far is 0
            if (__any(m_new != m)) {
                const float scale = dead ? 1.0f : pc_half_scale(m - m_new);   // m = -inf: acc is 0 anyway
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[rt][e] = acc[rt][e] * scale * scale;
            }
            m = m_new;
            // exp(v + d - m) = exp2(v * log2e + sh2); dead column: v = -inf -> 0
            sh2 = dead ? 0.0f : (d - m_new + PC_UP) * PC_LOG2E;
        }
        // ---- the chunk's MFMA steps ----
        // WAIT_ALL (backward, long reductions, at most two waves per SIMD): all loads of the chunk are waited for
        // before the first MFMA.  Left alone, the compiler lets each MFMA wait for just its own operand, and the matrix
        // pipe then runs in stop-and-go behind the loads for the whole chunk (config 4: 82 -> 78 us per layer).  With
        // more waves per SIMD, or rows of a few chunks, it is faster the other way (dense 1024 x 1024 layers at K = 32:
        // 2.2 against 3.4 ms), and a run-time test here costs as much as the wait itself -- hence an instantiation of
        // its own.  (The forward kernel waits in any case: its
        // chunk maximum needs every value.)  0x0F70 = vmcnt(0), the other counters at their maxima.
        if (WAIT_ALL) __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const float p = __builtin_amdgcn_exp2f(fmaf(o.v[q], PC_LOG2E, sh2));
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) acc[rt] = __builtin_amdgcn_mfma_f32_32x32x2f32(o.ar[q][rt], p, acc[rt], 0, 0, 0);
        }
    };
    if (!PF) {
        Operands o;
        for (int c = chunk0 + sp; c < n_chunks; c += SPLIT) {
            load_chunk(c, o);
            run_chunk(o);
        }
    } else {
        // small launches (one wave per SIMD or fewer): nobody else hides this wave's loads, so the next chunk is
        // requested before the current one is worked on -- two operand sets, chunks in pairs
        Operands oa, ob;
        if (sp < n_chunks) load_chunk(sp, oa);
        int c = sp;
        for (; c + SPLIT < n_chunks; c += 2 * SPLIT) {
            load_chunk(c + SPLIT, ob);
            run_chunk(oa);
            if (c + 2 * SPLIT < n_chunks) load_chunk(c + 2 * SPLIT, oa);
            run_chunk(ob);
        }
        if (c < n_chunks) run_chunk(oa);
    }

    // Merge of the SPLIT waves' partial sums: each takes its share of the elements from all of them, and writes them.
    float res[ES];
    if (SPLIT == 1) {
#pragma unroll
        for (int q = 0; q < ES; ++q) res[q] = acc[q / 16][q % 16];
    } else {
#pragma unroll
        for (int q = 0; q < RT * 16; ++q) buf[q * 64 + lane] = acc[q / 16][q % 16];   // (the wave's own staging tile until now)
        buf[RT * 16 * 64 + lane] = m;
        if (!BWD) buf[RT * 16 * 64 + 64 + lane] = Rrow;
        __syncthreads();
        const float *part = lds + ct * SPLIT * WSZ;
        float sc[SPLIT], Ro[BWD ? 1 : SPLIT];
#pragma unroll
        for (int s = 0; s < SPLIT; ++s) {
            sc[s] = part[s * WSZ + RT * 16 * 64 + lane];
            if (!BWD) Ro[BWD ? 0 : s] = part[s * WSZ + RT * 16 * 64 + 64 + lane];   // -inf: that wave had no chunk (its sum is 0)
        }
        if (!BWD) {                                                     // all partial sums to the largest reference
#pragma unroll
            for (int s = 0; s < SPLIT; ++s) Rrow = fmaxf(Rrow, Ro[BWD ? 0 : s]);
#pragma unroll
            for (int s = 0; s < SPLIT; ++s) sc[s] = Ro[BWD ? 0 : s] > PC_NEG_INF ? sc[s] + (Ro[BWD ? 0 : s] - Rrow) : PC_NEG_INF;
        }
#pragma unroll
        for (int s = 0; s < SPLIT; ++s) m = fmaxf(s == 0 ? sc[0] : m, sc[s]);
        const bool dead = !(m > PC_NEG_INF);
#pragma unroll
        for (int k = 0; k < ES; ++k) res[k] = 0.0f;
#pragma unroll
        for (int s = 0; s < SPLIT; ++s) {
            const float h = dead ? 0.0f : pc_half_scale(sc[s] - m);
#pragma unroll
            for (int k = 0; k < ES; ++k) res[k] += part[s * WSZ + (sp * ES + k) * 64 + lane] * h * h;
        }
    }
    if (!active) return;
    if (PART) {                                                         // K rows of sums, their maximum's shift and reference (k_sum_merge)
        float *po = F + (int64_t)part_row * Bs + col;
#pragma unroll
        for (int k = 0; k < ES; ++k) {
            const int q = sp * ES + k;
            po[(int64_t)(sub * TM + q / 16 * 32 + 8 * (q % 16 / 4) + 4 * half + q % 4) * Bs] = res[k];
        }
        if (sub == 0 && sp == 0) F[(int64_t)(part_top + half) * Bs + col] = half ? Rrow : m;
        return;
    }
    if (!BWD && sub == 0 && sp == 0 && half == 0) R[(int64_t)(id / K) * Bs + col] = Rrow;
    // Results out.  The rows are addressed through one buffer descriptor at the tile's first row with a scalar offset
    // per row.  Backward: log and exp are the hardware's base-2 instructions (the accumulator of a column with any
    // term is a normal number -- the largest term is at least FLT_MIN * e^PC_UP -- so no denormal care is needed).
    float *out = BWD ? F : l;
    const __amdgpu_buffer_rsrc_t ro =
        __builtin_amdgcn_make_buffer_rsrc((void *)(out + (int64_t)(id + sub * TM) * Bs), 0, PC_BUF_RANGE, PC_BUF_FLAGS);
    const float mb = (m - PC_UP) * PC_LOG2E;
#pragma unroll
    for (int k = 0; k < ES; ++k) {
        const int so = row_off(sp * ES + k);
        const float a = res[k];
        if (BWD) {
            const float lg = __builtin_amdgcn_logf(a);                  // log2; a = 0 -> -inf
            const float lc = lown[k];
            // exp(ln a + (m - PC_UP) + lc); a = 0 or lc = -inf gives exp2(-inf) = 0
            const float add = __builtin_amdgcn_exp2f(lg + fmaf(lc, PC_LOG2E, mb));
            if (first) {
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, add), ro, ooff, so, 0);
            } else if (add > 0.0f) {
                const float old = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ro, ooff, so, 0));
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, old + add), ro, ooff, so, 0);
            }
        } else {
            // ln a + (m - PC_UP), with the logarithm taken of a / 2^24: the accumulator of a live column is around
            // e^PC_UP, and a base-2 logarithm near 0 is far more accurate in absolute terms than one near 29 --
            // these errors add up from layer to layer (a log-likelihood near 0 has an absolute tolerance of 1e-5).
            // a = 0: -inf.  (a >= FLT_MIN * e^PC_UP > 2^-98, so a / 2^24 is a normal number.)
            const float v = fmaf(__builtin_amdgcn_logf(a * 0x1p-24f), 0.6931471805599453f, m + (16.635532333f - PC_UP));
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), ro, ooff, so, 0);
        }
    }
}

// The parts of a row (k_sum_mfma, MODE 3; 32 at most) merged as the waves of a workgroup merge theirs.  Workgroup = 8 rows x 32 columns,
// thread = one of them; all its loads are requested at once.  at: the children, in whose rows of `part` the parts lie (sum_parts).  ll not null:
// the row is the root's, node 0 of it is read out.
__global__ __launch_bounds__(256) void k_sum_merge(const float *__restrict__ part, const int32_t *__restrict__ at, int32_t n_parts, float *__restrict__ l, float *__restrict__ R,
                                                   const int32_t *__restrict__ ids, int32_t K, int64_t Bs, float *__restrict__ ll, int32_t B)
{
    __shared__ float scale[32][32], top[2][8][32];                      // a part's factor; the threads' largest references and shifts
    const int c32 = threadIdx.x & 31, g = threadIdx.x >> 5;
    const int64_t col = (int64_t)blockIdx.y * 32 + c32;
    const int row = (int)blockIdx.x * 8 + g;
    const float *p = part + col;
    const int32_t id = ids[0];
    float v[32];
#pragma unroll
    for (int s = 0; s < 32; ++s) v[s] = s < n_parts ? p[(int64_t)(at[min(s, n_parts - 1)] + row) * Bs] : 0.0f;
    const int32_t top0 = at[n_parts], top1 = at[n_parts + 1];           // 16 parts to a block of 32
    float ms[4], Ro[4], Rm = PC_NEG_INF, m = PC_NEG_INF;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int s = g + 8 * i;
        const float *top_rows = p + (int64_t)(K == 32 && i >= 2 ? top1 + 2 * (s - 16) : top0 + 2 * s) * Bs;
        ms[i] = s < n_parts ? top_rows[0] : PC_NEG_INF;
        Ro[i] = s < n_parts ? top_rows[Bs] : PC_NEG_INF;                // -inf: a part without chunks
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) Rm = fmaxf(Rm, Ro[i]);
    top[0][g][c32] = Rm;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) Rm = fmaxf(Rm, top[0][i][c32]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        ms[i] = Ro[i] > PC_NEG_INF ? ms[i] + (Ro[i] - Rm) : PC_NEG_INF;
        m = fmaxf(m, ms[i]);
    }
    top[1][g][c32] = m;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) m = fmaxf(m, top[1][i][c32]);
#pragma unroll
    for (int i = 0; i < 4; ++i) scale[g + 8 * i][c32] = m > PC_NEG_INF ? pc_half_scale(ms[i] - m) : 0.0f;
    __syncthreads();
    float sum = 0.0f;
#pragma unroll
    for (int s = 0; s < 32; ++s) {
        const float h = scale[s][c32];
        sum += v[s] * h * h;
    }
    const float out = fmaf(__builtin_amdgcn_logf(sum * 0x1p-24f), 0.6931471805599453f, m + (16.635532333f - PC_UP));
    l[(int64_t)(id + row) * Bs + col] = out;
    if (row == 0) R[(int64_t)(id / K) * Bs + col] = Rm;
    if (row == 0 && ll && col < B) ll[col] = Rm + out;
}

// ------------------------------------------------------------------------------------------
// Long dense reductions on the bf16 matrix cores (fp32 values split in two)
// ------------------------------------------------------------------------------------------
// The fp32 MFMA rate (157 TFLOP/s) is a sixteenth of the bf16 rate.  Every term of a sum node is non-negative, so a
// product theta * p can be taken as  th*ph + th*pl + tl*ph  with theta = th + tl and p = ph + pl split into two bf16
// values each (8 + 8 significant bits, round to nearest): three bf16 MFMAs with fp32 accumulation per fp32 MFMA's
// worth of work, relative error of a term about 2^-17, no cancellation.  Used for rows with long reductions (the
// dense layers of a large HMM), where the fp32 kernel is bound by the matrix cores.
//
// Operands are prepared once, in the order the MFMA wants them, so that the main loop is loads and MFMAs only:
//   * theta planes (k_split_theta, once per forward pass): per parameter block and (32-row tile rt, 16-column slice
//     ks) one 1 KiB tile -- lane (i = lane % 32, h = lane / 32) owns theta[32 rt + i][16 ks + 8 h .. + 7] as 8 bf16;
//   * value planes (k_split_p, per product layer): p = exp(l + PC_UP) of the residual log-probabilities -- at most
//     e^(PC_UP + 0.5), a product block's largest residual is within 0.5 of 0 -- per (16-node slice, 32-column tile)
//     one 1 KiB tile: lane (j = lane % 32, h) owns p[16 slice + 8 h .. + 7][32 tile + j].
// What the fp32 kernel does per value (running maximum, exponential) happens per child BLOCK here: a block's values
// are relative to its integer reference R_c, the block's partial sums are accumulated on their own and added to the
// row's accumulator with the factor exp(R_c - R_row) (R_row = largest reference so far; the accumulator is rescaled
// when it grows).  v_mfma_f32_32x32x16_bf16: A 32 x 16, B 16 x 32, D as for the fp32 instruction.

// theta [n_blocks][K][K] fp32 -> planes Th, Tl of 1 KiB tiles [block][rt][ks][lane][8]; TRANSPOSED: the tiles of
// theta^T (rows = children), for the backward kernel.  One wave per tile.
template <bool TRANSPOSED>
__global__ __launch_bounds__(256) void k_split_theta(const float *__restrict__ theta, int64_t n_tiles, int32_t K,
                                                     uint4 *__restrict__ Th, uint4 *__restrict__ Tl)
{
    const int64_t tile = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (tile >= n_tiles) return;
    const int lane = threadIdx.x & 63, i = lane & 31, h = lane >> 5;
    const int nks = K / 16, nrt = K / 32;
    const int ks = (int)(tile % nks), rt = (int)((tile / nks) % nrt);
    const int64_t pb = tile / ((int64_t)nks * nrt);
    const float *src = theta + pb * K * K;
    float v[8];
    if (!TRANSPOSED) {
        const float4 *q = reinterpret_cast<const float4 *>(src + (int64_t)(32 * rt + i) * K + 16 * ks + 8 * h);
        const float4 a = q[0], b = q[1];
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = src[(int64_t)(16 * ks + 8 * h + e) * K + 32 * rt + i];
    }
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) bf16_split2(v[2 * e], v[2 * e + 1], hi[e], lo[e]);
    Th[tile * 64 + lane] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    Tl[tile * 64 + lane] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
}

// value planes of the given node blocks: X = l (forward: residual log-probabilities of product blocks) gives
// exp(l + PC_UP); with a block reference `ref` (backward: X = log_nf of sum blocks, ref = their column maxima) gives
// exp(X - ref + PC_UP).  One wave per (block, 16-node slice, 32-column tile).
__global__ __launch_bounds__(256) void k_split_p(const float *__restrict__ X, const float *__restrict__ ref,
                                                 const int32_t *__restrict__ blk_ids, int32_t n_blk, int32_t K, int64_t Bs,
                                                 uint4 *__restrict__ Ph, uint4 *__restrict__ Pl)
{
    const int n_ct = (int)(Bs / 32), nks = K / 16;
    const int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (item >= (int64_t)n_blk * nks * n_ct) return;
    const int lane = threadIdx.x & 63;
    const int ct = (int)(item % n_ct), ks = (int)((item / n_ct) % nks);
    const int32_t id = blk_ids[item / ((int64_t)n_ct * nks)];
    float sh = PC_UP;
    if (ref) {
        const float r = ref[(int64_t)(id / K) * Bs + (int64_t)ct * 32 + (lane & 31)];
        sh = r > PC_NEG_INF ? PC_UP - r : PC_NEG_INF;                   // a block without flow: every factor 0
    }
    split_value_tile(X, sh, (int64_t)id + 16 * ks, ct, n_ct, Bs, Ph, Pl, lane);
}

// Sum layer on the planes, forward (rows = sum blocks, neighbours = their product children) and backward to the
// children (rows = product blocks, neighbours = their sum parents, theta planes transposed).  Workgroup = 4 waves that
// share one output tile of 64 rows x 32 CT columns and take the row's neighbour blocks in turn (a split of the
// reduction); at the end the tile's 32 x 32 parts are dealt to the waves, which merge the four partial sums through
// LDS and write the results.  Per 16-node slice a wave fetches 2 + 2 theta tiles and CT + CT value tiles
// (hi and lo planes, 16 bytes per lane each, 1 KiB per wave load) and issues 6 CT MFMAs; the operands of D slices are
// in flight at any time (a ring of D register sets that runs across the neighbour blocks).
//   forward : block scale = R_c (integer reference of the child block); result l = ln(sum) - PC_UP relative to the
//             largest reference, which becomes the row's own
//   backward: block scale = nfmax_s + (R_row - R_s) (column maximum of the parent's log_nf, brought to the row's
//             reference); result F += exp(ln(sum) + scale - PC_UP + l_row)
// Measured on 4096 x 4096 layers at B = 256: 40 us per layer with CT = 1 and 32-34 us with CT = 2 (one workgroup per
// CU, one wave per SIMD) against 80 us on the fp32 matrix cores; the matrix work itself is 10 us.  The rest is the
// rate at which a CU's vector memory pipeline delivers the 1 KiB operand loads (a 128-byte line per 4.8 cycles,
// whatever the ring depth; CT = 2 needs two thirds of the bytes per MFMA) on top of some 20 us that do not depend on
// the traffic (launch, row headers, the per-block folds, the merge, the epilogue).
template <int K, int D, bool BWD, int CT>
__global__ __launch_bounds__(256, CT == 1 ? 2 : 1) void k_sum_bf16(const uint4 *__restrict__ Th, const uint4 *__restrict__ Tl,
                                                                   const uint4 *__restrict__ Ph, const uint4 *__restrict__ Pl,
                                                                   float *__restrict__ l, float *__restrict__ R,
                                                                   const float *__restrict__ nfmax, float *__restrict__ F,
                                                                   const GroupSet gs, int64_t Bs)
{
    constexpr int NKS = K / 16, NRT = K / 32, SUB = K / 64;
    static_assert(NKS % D == 0, "the ring must divide a block's slices");
    __shared__ float lds[2 * CT * 3 * 1024 + 4 * CT * 64];              // partial tiles of the merge and the waves' references
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const GroupRow gr = locate_row<PC_ROWS_ONE>(gs, blockIdx.x / SUB);
    const int r = gr.r, sub = blockIdx.x % SUB;
    const int n_ct = (int)(Bs / 32);
    const int ct0 = blockIdx.y * CT;
    const int64_t col0 = (int64_t)ct0 * 32 + l32;                       // column of tile c: col0 + 32 c
    const int32_t *row_nbr = gr.nbr + (int64_t)r * gr.width, *row_par = gr.par + (int64_t)r * gr.width;
    const int32_t id = gr.ids[r];
    const int32_t fl = gr.aux[r];
    const int cnt = fl >> 8;
    float Rown[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) Rown[c] = BWD ? R[(int64_t)(id / K) * Bs + col0 + 32 * c] : 0.0f;

    floatx16 acc[2][CT], blk[2][CT];
    float m[CT], cm[CT];                                                // reference of the accumulator, of the current block
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        m[c] = PC_NEG_INF;
        cm[c] = PC_NEG_INF;
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[rt][c][e] = 0.0f;
    }

    struct Ops { uint4 ah[2], al[2], bh[CT], bl[CT]; };
    const int n_my = cnt > wave ? (cnt - wave + 3) / 4 : 0;             // neighbour blocks wave, wave + 4, ...
    auto load_slice = [&](int32_t ns, int32_t ps, int ks, Ops &o) {
        const int64_t ta = (((int64_t)(ps / (K * K)) * NRT + 2 * sub) * NKS + ks) * 64 + lane;   // rt advances by NKS tiles
        const int64_t tb = ((int64_t)(ns / 16 + ks) * n_ct + ct0) * 64 + lane;
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) { o.ah[rt] = Th[ta + (int64_t)rt * NKS * 64]; o.al[rt] = Tl[ta + (int64_t)rt * NKS * 64]; }
#pragma unroll
        for (int c = 0; c < CT; ++c) { o.bh[c] = Ph[tb + 64 * c]; o.bl[c] = Pl[tb + 64 * c]; }
    };
    // The loop over the wave's neighbour blocks is straight-line inside (every slot of the ring is refilled
    // unconditionally: past the last block the refill repeats that block and is never used), so that the compiler can
    // count the loads in flight and wait for just the oldest set; a branch around a load makes it wait for all of them.
    Ops o[D];
    int32_t ns_cur = 0, ps_cur = 0;
    if (n_my > 0) {
        ns_cur = row_nbr[wave];
        ps_cur = row_par[wave];
#pragma unroll
        for (int d = 0; d < D; ++d) load_slice(ns_cur, ps_cur, d, o[d]);
    }
    for (int bi = 0; bi < n_my; ++bi) {
        const int jn = wave + 4 * (bi + 1 < n_my ? bi + 1 : bi);
        const int32_t ns_nxt = row_nbr[jn], ps_nxt = row_par[jn];
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const float Rn = R[(int64_t)(ns_cur / K) * Bs + col0 + 32 * c];   // finite
            cm[c] = BWD ? nfmax[(int64_t)(ns_cur / K) * Bs + col0 + 32 * c] + (Rown[c] - Rn) : Rn;
        }
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            Ops &cur = o[ks % D];
            if (ks == 0) {
#pragma unroll
                for (int c = 0; c < CT; ++c)
#pragma unroll
                    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                        for (int e = 0; e < 16; ++e) blk[rt][c][e] = 0.0f;
            }
            // three products per tile, small ones first; the tiles take turns so that no MFMA waits for the one before
#pragma unroll
            for (int step = 0; step < 3; ++step)
#pragma unroll
                for (int c = 0; c < CT; ++c)
#pragma unroll
                    for (int rt = 0; rt < 2; ++rt) {
                        const bf16x8 a = __builtin_bit_cast(bf16x8, step == 0 ? cur.al[rt] : cur.ah[rt]);
                        const bf16x8 b = __builtin_bit_cast(bf16x8, step == 1 ? cur.bl[c] : cur.bh[c]);
                        blk[rt][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, blk[rt][c], 0, 0, 0);
                    }
            if (ks + D < NKS) load_slice(ns_cur, ps_cur, ks + D, cur);
            else load_slice(ns_nxt, ps_nxt, ks + D - NKS, cur);
            __builtin_amdgcn_sched_barrier(0);                          // keeps the refill here, D - 1 slices ahead of its use
        }
        // the block's partial sums join the row's accumulator, both brought to the larger reference
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const float mn = fmaxf(m[c], cm[c]);
            const float sa = m[c] > PC_NEG_INF ? __expf(m[c] - mn) : 0.0f, sb = cm[c] > PC_NEG_INF ? __expf(cm[c] - mn) : 0.0f;
            m[c] = mn;
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[rt][c][e] = acc[rt][c][e] * sa + blk[rt][c][e] * sb;
        }
        ns_cur = ns_nxt;
        ps_cur = ps_nxt;
    }

    // Merge and results: the 2 CT tiles of 32 x 32 outputs are dealt to the waves, tile u = 2 c + rt to wave u; every
    // wave leaves its partial sums of the tiles it does not own in LDS (three sets per tile) and its references.
    constexpr int NU = 2 * CT;
    float *mref = lds + NU * 3 * 1024;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
            const int u = c * 2 + rt;
            if (wave != u) {
                float *dst = lds + (u * 3 + (wave < u ? wave : wave - 1)) * 1024;
#pragma unroll
                for (int e = 0; e < 16; ++e) dst[e * 64 + lane] = acc[rt][c][e];
            }
        }
        mref[(wave * CT + c) * 64 + lane] = m[c];
    }
    __syncthreads();
    const bool first = (fl & 2) != 0;                                   // backward: the first layer that feeds the block stores
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        if (wave != u) continue;                                        // uniform: a wave takes one of the branches
        const int c = u / 2, rt = u % 2;
        const int64_t col = col0 + 32 * c;
        // backward: the rows' own log-probabilities (and, where this layer accumulates, the flows so far) are all
        // requested before the first of them is used -- a load inside the per-element branch would be waited for on its
        // own, 16 times
        floatx16 lown, fold;
        if (BWD) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int64_t at = (int64_t)(id + sub * 64 + rt * 32 + 8 * (e / 4) + 4 * half + (e % 4)) * Bs + col;
                lown[e] = l[at];
                fold[e] = first ? 0.0f : F[at];
            }
        }
        float mw[4], mt = PC_NEG_INF;                                   // the four waves' references of this column; -inf: no block
#pragma unroll
        for (int w = 0; w < 4; ++w) { mw[w] = mref[(w * CT + c) * 64 + lane]; mt = fmaxf(mt, mw[w]); }
        floatx16 tot;
#pragma unroll
        for (int e = 0; e < 16; ++e) tot[e] = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float sc = mw[w] > PC_NEG_INF ? __expf(mw[w] - mt) : 0.0f;
            if (w == u) {
#pragma unroll
                for (int e = 0; e < 16; ++e) tot[e] += acc[rt][c][e] * sc;
            } else {
                const float *src = lds + (u * 3 + (w < u ? w : w - 1)) * 1024;
#pragma unroll
                for (int e = 0; e < 16; ++e) tot[e] += src[e * 64 + lane] * sc;
            }
        }
        if (!BWD && sub == 0 && rt == 0 && half == 0) R[(int64_t)(id / K) * Bs + col] = mt;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int row = sub * 64 + rt * 32 + 8 * (e / 4) + 4 * half + (e % 4);
            const int64_t at = (int64_t)(id + row) * Bs + col;
            if (!BWD) {
                // ln(sum) - PC_UP, the logarithm taken of sum / 2^24 (see the fp32 kernel)
                l[at] = fmaf(__builtin_amdgcn_logf(tot[e] * 0x1p-24f), 0.6931471805599453f, 16.635532333f - PC_UP);
            } else {
                // exp(ln(sum) + (m - PC_UP) + l_row); sum = 0 or l_row = -inf gives exp2(-inf) = 0
                const float lg = __builtin_amdgcn_logf(tot[e]);
                const float add = __builtin_amdgcn_exp2f(lg + (lown[e] + (mt - PC_UP)) * PC_LOG2E);
                F[at] = fold[e] + (mt > PC_NEG_INF ? add : 0.0f);
            }
        }
    }
}

// Backward to the parameters (role of Alg. 3), organised by PARAMETER BLOCK instead of by layer: one launch
// covers every parameter block of the circuit after the backward sweep.  A wave owns a TMW x TNW tile
// (up to 64 x 64) of one K x K parameter block and reduces over the batch of every (sum block, child
// block) pair that uses the block -- all tied instances, e.g. the T-1 transition layers of an HMM
// (App. A.3) -- in registers, so each flow element is read-modified-written once per call, without
// atomics and without the per-layer accumulation that closes Alg. 3.
//
// Each term exp(log_nf_s + l_c) is split into two fp32 factors around a per-sample shift (any shift is
// valid: it only moves scale between the factors) -- the balanced split defined with PC_SPLIT_SCALE above.  Alg. 3
// shifts by the block maximum a alone, which can drop products of order one when a weight is as small as FLT_MIN.
//
// Per chunk of 32 samples a wave fetches its TMW rows of N and TNW rows of l with 16-byte loads along
// the batch, applies the exponentials, and stages both tiles in wave-private LDS (row stride 36 floats)
// to reach the MFMA operand layouts (batch index on k: step q pairs lanes 0-31 with sample 8*(q/4) + q%4
// and lanes 32-63 with sample 8*(q/4) + 4 + q%4); loads of the next chunk are issued before the
// arithmetic of the current one.
//
// ORDERED: the four waves of a workgroup take the chunks of one block and add up their parts in LDS, in a fixed order: no atomics, so the
// flow repeats to the bit (launch_param_flow).
template <int K, int RT, int CT, bool ONE, bool ORDERED>
__global__ __launch_bounds__(256, 2) void k_param_flow_mfma(const float *__restrict__ theta, const float *__restrict__ l,
                                                            const float *__restrict__ R, const float *__restrict__ N,
                                                            const float *__restrict__ nfmax, float *__restrict__ G,
                                                            const int32_t *__restrict__ pf_pb, const int32_t *__restrict__ pf_ptr,
                                                            const int32_t *__restrict__ pf_sum, const int32_t *__restrict__ pf_child,
                                                            int32_t n_pb, int32_t n_split, int64_t Bs)
{
    constexpr int TMW = 32 * RT, TNW = 32 * CT;
    constexpr int TPB = (K / TMW) * (K / TNW);                          // wave tiles per parameter block
    constexpr int LD = 36;                                              // LDS row stride: 16-byte rows, b128 reads conflict-free
    constexpr int NA4 = TMW * 8 / 64, NB4 = TNW * 8 / 64;               // 16-byte loads per lane per chunk
    // ONE (short reductions): a single tile per wave, used for N's factors and then for l's (LDS operations of one wave
    // complete in order) -- half the LDS, twice the workgroups per CU; the second staging then waits for the first
    // operand read, which costs more than it gains once a block has 16 chunks or more.
    constexpr int TLD = ONE ? (TMW > TNW ? TMW : TNW) : TMW + TNW;
    __shared__ float lds[4 * TLD * LD];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    // n_split > 1 (a handful of parameter blocks with many tied pairs each, e.g. a small HMM): the chunks of a block's pairs
    // are dealt to n_split waves, which add their partial flows atomically
    const int64_t wtile = (int64_t)blockIdx.x * 4 + wave;
    const int64_t tile = ORDERED ? blockIdx.x : wtile / n_split;
    const int spl = ORDERED ? wave : (int)(wtile % n_split);
    const int pidx = (int)(tile / TPB), tin = (int)(tile % TPB);
    static_assert(!ORDERED || TPB == 1, "a workgroup is one block's");
    if (pidx >= n_pb) return;                                           // wave-uniform; ORDERED: there are n_pb workgroups
    const int r0 = (tin / (K / TNW)) * TMW, c0 = (tin % (K / TNW)) * TNW;
    const int32_t pb = pf_pb[pidx];
    const int i0 = pf_ptr[pidx], i1 = pf_ptr[pidx + 1];
    float *Qs = lds + wave * TLD * LD, *Ps = ONE ? Qs : Qs + TMW * LD;
    const int srow = lane >> 3, sc4 = (lane & 7) * 4;                   // staging: 8 lanes x 16 bytes per row of 32 samples

    floatx16 acc[RT][CT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[rt][ct][e] = 0.0f;

    const int chunks_per_inst = (int)(Bs / 32);
    const int all = (i1 - i0) * chunks_per_inst, share = n_split == 1 ? all : (all + n_split - 1) / n_split;
    const int chunk0 = min(spl * share, all), n_chunks = min(share, all - chunk0);
    floatx4 nf_next[NA4], lc_next[NB4], mx_next, rs_next, rc_next;

#define PC_ISSUE(C)                                                                                                   \
    do {                                                                                                              \
        const int inst_ = i0 + (chunk0 + (C)) / chunks_per_inst;                                                      \
        const int64_t b0_ = (int64_t)((chunk0 + (C)) % chunks_per_inst) * 32 + sc4;                                   \
        const int32_t ms_ = pf_sum[inst_], ns_ = pf_child[inst_];                                                     \
        const float *np_ = N + (int64_t)(ms_ + r0 + srow) * Bs + b0_;                                                 \
        const float *lp_ = l + (int64_t)(ns_ + c0 + srow) * Bs + b0_;                                                 \
        _Pragma("unroll") for (int i = 0; i < NA4; ++i) nf_next[i] = *reinterpret_cast<const floatx4 *>(np_ + (int64_t)(8 * i) * Bs); \
        _Pragma("unroll") for (int i = 0; i < NB4; ++i) lc_next[i] = *reinterpret_cast<const floatx4 *>(lp_ + (int64_t)(8 * i) * Bs); \
        mx_next = *reinterpret_cast<const floatx4 *>(nfmax + (int64_t)(ms_ / K) * Bs + b0_);                          \
        rs_next = *reinterpret_cast<const floatx4 *>(R + (int64_t)(ms_ / K) * Bs + b0_);                              \
        rc_next = *reinterpret_cast<const floatx4 *>(R + (int64_t)(ns_ / K) * Bs + b0_);                              \
    } while (0)

    if (n_chunks > 0) PC_ISSUE(0);
    for (int c = 0; c < n_chunks; ++c) {
        // exponentials of the fetched chunk, staged in the wave's LDS tiles
        floatx4 qa, qb;                                                 // per-sample shifts in log2 units
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool live = mx_next[e] > PC_NEG_INF;
            const float g = mx_next[e] + (rc_next[e] - rs_next[e]);
            const float sb = pc_split_shift(g);
            qa[e] = live ? (sb - mx_next[e]) * PC_LOG2E : PC_NEG_INF;                      // dead sample: both factors 0
            qb[e] = live ? (g - sb - PC_SPLIT_SCALE) * PC_LOG2E : PC_NEG_INF;
        }
#pragma unroll
        for (int i = 0; i < NA4; ++i) {
            floatx4 q;
#pragma unroll
            for (int e = 0; e < 4; ++e) q[e] = __builtin_amdgcn_exp2f(fmaf(nf_next[i][e], PC_LOG2E, qa[e]));
            *reinterpret_cast<floatx4 *>(Qs + (8 * i + srow) * LD + sc4) = q;
        }
        // operands of the whole chunk into registers (LDS operations of one wave complete in order); with a single tile
        // the first operand has to be read before the second is staged
        float areg[16][RT], breg[16][CT];
#define PC_READ_AREG()                                                                                                \
    _Pragma("unroll") for (int rt = 0; rt < RT; ++rt)                                                                 \
        _Pragma("unroll") for (int g = 0; g < 4; ++g) {                                                               \
            const floatx4 a4 = *reinterpret_cast<const floatx4 *>(Qs + (rt * 32 + l32) * LD + 8 * g + 4 * half);      \
            areg[4 * g + 0][rt] = a4[0]; areg[4 * g + 1][rt] = a4[1]; areg[4 * g + 2][rt] = a4[2]; areg[4 * g + 3][rt] = a4[3]; \
        }
        if (ONE) PC_READ_AREG();
#pragma unroll
        for (int i = 0; i < NB4; ++i) {
            floatx4 p;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                p[e] = __builtin_amdgcn_exp2f(fminf(fmaf(lc_next[i][e], PC_LOG2E, qb[e]), PC_SPLIT_CAP * PC_LOG2E));
            *reinterpret_cast<floatx4 *>(Ps + (8 * i + srow) * LD + sc4) = p;
        }
        if (c + 1 < n_chunks) PC_ISSUE(c + 1);
        if (!ONE) PC_READ_AREG();
#undef PC_READ_AREG
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const floatx4 b4 = *reinterpret_cast<const floatx4 *>(Ps + (ct * 32 + l32) * LD + 8 * g + 4 * half);
                breg[4 * g + 0][ct] = b4[0]; breg[4 * g + 1][ct] = b4[1]; breg[4 * g + 2][ct] = b4[2]; breg[4 * g + 3][ct] = b4[3];
            }
#pragma unroll
        for (int q = 0; q < 16; ++q)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
                    acc[rt][ct] = __builtin_amdgcn_mfma_f32_32x32x2f32(areg[q][rt], breg[q][ct], acc[rt][ct], 0, 0, 0);
    }
#undef PC_ISSUE

    if constexpr (ORDERED) {
        const int64_t at = (int64_t)pb + (int64_t)(threadIdx.x >> 3) * K + sc4;      // 16 bytes of the block per thread
        const floatx4 th = *reinterpret_cast<const floatx4 *>(theta + at), old = *reinterpret_cast<const floatx4 *>(G + at);
#pragma unroll
        for (int e = 0; e < 16; ++e) Qs[(8 * (e / 4) + 4 * half + (e % 4)) * LD + l32] = acc[0][0][e];
        __syncthreads();
        floatx4 sum = {0.0f, 0.0f, 0.0f, 0.0f}, out;
#pragma unroll
        for (int w = 0; w < 4; ++w) sum += *reinterpret_cast<const floatx4 *>(lds + w * TLD * LD + (threadIdx.x >> 3) * LD + sc4);
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = th[e] > 0.0f ? pc_flow_out(th[e], sum[e]) : 0.0f;
        *reinterpret_cast<floatx4 *>(G + at) = old + out;
        return;
    }
    // Results out, 32 x 32 at a time through the wave's LDS tile, so that theta and the flows come as 16-byte loads that are all
    // requested together.  (Element by element in the accumulator's layout, a load of theta, a test, a load of the flow and a store after
    // the other, a block of one chunk was 32 memory latencies: PD of 97 K parameter blocks, B = 20 443 -> 249 us, B = 256 831 -> 791; RAT-SPN of 28.6 K,
    // B = 16 146 -> 66.)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const int64_t at0 = (int64_t)pb + (int64_t)(r0 + rt * 32 + srow) * K + c0 + ct * 32 + sc4;
            floatx4 th[4], old[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) th[i] = *reinterpret_cast<const floatx4 *>(theta + at0 + 8 * i * K);
            if (n_split == 1) {
#pragma unroll
                for (int i = 0; i < 4; ++i) old[i] = *reinterpret_cast<const floatx4 *>(G + at0 + 8 * i * K);
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) Qs[(8 * (e / 4) + 4 * half + (e % 4)) * LD + l32] = acc[rt][ct][e];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const floatx4 sum = *reinterpret_cast<const floatx4 *>(Qs + (8 * i + srow) * LD + sc4);
                floatx4 out;
#pragma unroll
                for (int e = 0; e < 4; ++e) out[e] = th[i][e] > 0.0f ? pc_flow_out(th[i][e], sum[e]) : 0.0f;   // theta = 0: no flow (never 0 * inf)
                if (n_split == 1) {
                    *reinterpret_cast<floatx4 *>(G + at0 + 8 * i * K) = old[i] + out;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) if (th[i][e] > 0.0f) atomicAdd(G + at0 + 8 * i * K + e, out[e]);
                }
            }
        }
}

// The same computation for K = 64 and 128 with the staging shared by the workgroup: the four waves own the four
// quarters of one K x K parameter block, and every fetched row is used by two of them.  Per chunk of 32 samples the
// 256 threads fetch and exponentiate the K rows of N and the K rows of l ONCE (K / 32 + K / 32 sixteen-byte loads per
// thread; the per-wave kernel needs four times as many at K = 128) into a workgroup tile in LDS; each wave then reads
// the K / 2 + K / 2 rows of its quarter.  Two forms (template parameter ONE, see inside): for long reductions the tile
// is double-buffered, so one barrier per chunk suffices, and the loads run two chunks ahead of the arithmetic -- a
// chunk's matrix work (1.7 us) is shorter than a trip to HBM, which some of a chunk's loads always take; for short
// reductions one tile and one register set, and many more waves per SIMD.
template <int K, bool ONE, bool BF>
__global__ __launch_bounds__(256, 2) void k_param_flow_mfma_wg(const float *__restrict__ theta, const float *__restrict__ l,
                                                               const float *__restrict__ R, const float *__restrict__ N,
                                                               const float *__restrict__ nfmax, float *__restrict__ G,
                                                               const int32_t *__restrict__ pf_pb, const int32_t *__restrict__ pf_ptr,
                                                               const int32_t *__restrict__ pf_sum, const int32_t *__restrict__ pf_child,
                                                               int32_t n_split, int64_t Bs)
{
    constexpr int LD = 36;                                              // LDS row stride: 16-byte rows, b128 reads conflict-free
    // BF (long reductions): the factors are split into hi / lo bf16 values when they are staged -- four planes (Q hi, Q
    // lo, P hi, P lo) of K rows x 32 samples, row stride 80 bytes (16-byte reads of 16 consecutive rows hit distinct
    // banks) -- and a product is qh*ph + qh*pl + ql*ph on v_mfma_f32_32x32x16_bf16: 24 MFMAs of 32 cycles per chunk and
    // wave instead of 64 of 64 cycles; all terms are non-negative, relative error about 2^-17.
    constexpr int LDB = 20;                                             // bf16 planes: row stride in dwords
    constexpr int TILE = BF ? 4 * K * LDB : 2 * K * LD;                 // K rows of factors from N, K rows from l
    constexpr int Q = K / 2, QT = Q / 32;                               // a wave's quarter: Q x Q, QT x QT MFMA tiles
    static_assert(!(BF && ONE), "the bf16 form exists for long reductions only");
    constexpr int NL = K / 32;                                          // 16-byte loads per thread, chunk and array
    static_assert(K == 64 || K == 128, "workgroup-shared parameter-flow kernel");
    // ONE (short reductions -- a parameter block used by one pair, B / 32 chunks -- and many small workgroups): one LDS
    // tile, one register set, operands in two halves: at K = 64 68 registers and 18 KB of LDS, seven waves per SIMD hide
    // the waits and the second barrier per chunk.  Otherwise (long reductions: tied blocks, e.g. the 31 layers of an
    // HMM): two tiles, loads two chunks ahead -- two workgroups of K = 128 fit a CU either way, and the loop has to hide
    // its own waits.
    __shared__ float lds[(ONE ? 1 : 2) * TILE];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int r0 = (wave >> 1) * Q, c0 = (wave & 1) * Q;                // this wave's quarter of the block
    // n_split > 1: the chunks of a block's pairs are dealt to n_split workgroups, which add their partial flows atomically
    // (a handful of blocks with many tied pairs each would otherwise keep a handful of workgroups busy)
    const int pidx = blockIdx.x / n_split, spl = blockIdx.x % n_split;
    const int32_t pb = pf_pb[pidx];
    const int i0 = pf_ptr[pidx], i1 = pf_ptr[pidx + 1];
    const int srow = threadIdx.x >> 3, sc4 = (threadIdx.x & 7) * 4;     // staging: 8 threads x 16 bytes per row, 32 rows per pass

    floatx16 acc[QT][QT];
#pragma unroll
    for (int rt = 0; rt < QT; ++rt)
#pragma unroll
        for (int ct = 0; ct < QT; ++ct)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[rt][ct][e] = 0.0f;

    const int chunks_per_inst = (int)(Bs / 32);
    const int all = (i1 - i0) * chunks_per_inst, share = n_split == 1 ? all : (all + n_split - 1) / n_split;
    const int chunk0 = min(spl * share, all), n_chunks = min(share, all - chunk0);
    // two register sets of fetched tiles (loads two chunks ahead)
    floatx4 nfA[NL], lcA[NL], mxA, rsA, rcA;
    floatx4 nfB[NL], lcB[NL], mxB, rsB, rcB;
    const int voff = (int)(((int64_t)srow * Bs + sc4) * 4), voff1 = sc4 * 4;
    int soff[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) soff[i] = __builtin_amdgcn_readfirstlane((int)((int64_t)(32 * i) * Bs * 4));

#define PC_ISSUE(C, NF, LC, MX, RS, RC)                                                                               \
    do {                                                                                                              \
        const int inst_ = i0 + (chunk0 + (C)) / chunks_per_inst;                                                      \
        const int64_t b0_ = (int64_t)((chunk0 + (C)) % chunks_per_inst) * 32;                                         \
        const int32_t ms_ = pf_sum[inst_], ns_ = pf_child[inst_];                                                     \
        const __amdgpu_buffer_rsrc_t rn_ = __builtin_amdgcn_make_buffer_rsrc((void *)(N + (int64_t)ms_ * Bs + b0_), 0, PC_BUF_RANGE, PC_BUF_FLAGS); \
        const __amdgpu_buffer_rsrc_t rl_ = __builtin_amdgcn_make_buffer_rsrc((void *)(l + (int64_t)ns_ * Bs + b0_), 0, PC_BUF_RANGE, PC_BUF_FLAGS); \
        _Pragma("unroll") for (int i = 0; i < NL; ++i)                                                                \
            NF[i] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rn_, voff, soff[i], 0));        \
        _Pragma("unroll") for (int i = 0; i < NL; ++i)                                                                \
            LC[i] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rl_, voff, soff[i], 0));        \
        const __amdgpu_buffer_rsrc_t rm_ = __builtin_amdgcn_make_buffer_rsrc((void *)(nfmax + (int64_t)(ms_ / K) * Bs + b0_), 0, PC_BUF_RANGE, PC_BUF_FLAGS); \
        const __amdgpu_buffer_rsrc_t rs_ = __builtin_amdgcn_make_buffer_rsrc((void *)(R + (int64_t)(ms_ / K) * Bs + b0_), 0, PC_BUF_RANGE, PC_BUF_FLAGS); \
        const __amdgpu_buffer_rsrc_t rc_ = __builtin_amdgcn_make_buffer_rsrc((void *)(R + (int64_t)(ns_ / K) * Bs + b0_), 0, PC_BUF_RANGE, PC_BUF_FLAGS); \
        MX = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rm_, voff1, 0, 0));                    \
        RS = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rs_, voff1, 0, 0));                    \
        RC = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rc_, voff1, 0, 0));                    \
    } while (0)

    // exponentials of a fetched chunk into tile T of the workgroup (this thread's rows srow, srow + 32, ...)
#define PC_STAGE(T, NF, LC, MX, RS, RC)                                                                               \
    do {                                                                                                              \
        float *Qt_ = lds + (T) * TILE, *Pt_ = Qt_ + K * LD;                                                           \
        floatx4 qa, qb;                                                 /* per-sample shifts in log2 units */         \
        _Pragma("unroll") for (int e = 0; e < 4; ++e) {                                                               \
            const bool live = MX[e] > PC_NEG_INF;                                                                     \
            const float g_ = MX[e] + (RC[e] - RS[e]);                                                                 \
            const float sb_ = pc_split_shift(g_);                                                                     \
            qa[e] = live ? (sb_ - MX[e]) * PC_LOG2E : PC_NEG_INF;       /* dead sample: both factors 0 */             \
            qb[e] = live ? (g_ - sb_ - PC_SPLIT_SCALE) * PC_LOG2E : PC_NEG_INF;                                       \
        }                                                                                                             \
        _Pragma("unroll") for (int i = 0; i < NL; ++i) {                                                              \
            floatx4 q, p;                                                                                             \
            _Pragma("unroll") for (int e = 0; e < 4; ++e) {                                                           \
                q[e] = __builtin_amdgcn_exp2f(fmaf(NF[i][e], PC_LOG2E, qa[e]));                                       \
                p[e] = __builtin_amdgcn_exp2f(fminf(fmaf(LC[i][e], PC_LOG2E, qb[e]), PC_SPLIT_CAP * PC_LOG2E));      \
            }                                                                                                         \
            *reinterpret_cast<floatx4 *>(Qt_ + (32 * i + srow) * LD + sc4) = q;                                       \
            *reinterpret_cast<floatx4 *>(Pt_ + (32 * i + srow) * LD + sc4) = p;                                       \
        }                                                                                                             \
    } while (0)

    // this wave's operands from tile T, then the products -- in two halves of eight steps (half the operand registers)
#define PC_MATH(T)                                                                                             \
    do {                                                                                                              \
        const float *Qt_ = lds + (T) * TILE + r0 * LD, *Pt_ = lds + (T) * TILE + (K + c0) * LD;                       \
        _Pragma("unroll") for (int h2 = 0; h2 < 2; ++h2) {                                                            \
            float areg[8][QT], breg[8][QT];                                                                           \
            _Pragma("unroll") for (int rt = 0; rt < QT; ++rt)                                                         \
                _Pragma("unroll") for (int g = 0; g < 2; ++g) {                                                       \
                    const floatx4 a4 = *reinterpret_cast<const floatx4 *>(Qt_ + (rt * 32 + l32) * LD + 8 * (2 * h2 + g) + 4 * half); \
                    areg[4 * g + 0][rt] = a4[0]; areg[4 * g + 1][rt] = a4[1]; areg[4 * g + 2][rt] = a4[2]; areg[4 * g + 3][rt] = a4[3]; \
                    const floatx4 b4 = *reinterpret_cast<const floatx4 *>(Pt_ + (rt * 32 + l32) * LD + 8 * (2 * h2 + g) + 4 * half); \
                    breg[4 * g + 0][rt] = b4[0]; breg[4 * g + 1][rt] = b4[1]; breg[4 * g + 2][rt] = b4[2]; breg[4 * g + 3][rt] = b4[3]; \
                }                                                                                                     \
            _Pragma("unroll") for (int q = 0; q < 8; ++q)                                                             \
                _Pragma("unroll") for (int rt = 0; rt < QT; ++rt)                                                     \
                    _Pragma("unroll") for (int ct = 0; ct < QT; ++ct)                                                 \
                        acc[rt][ct] = __builtin_amdgcn_mfma_f32_32x32x2f32(areg[q][rt], breg[q][ct], acc[rt][ct], 0, 0, 0); \
        }                                                                                                             \
    } while (0)

    // the same with the factors split into bf16 planes (BF)
#define PC_STAGE_BF(T, NF, LC, MX, RS, RC)                                                                            \
    do {                                                                                                              \
        uint32_t *Qh_ = reinterpret_cast<uint32_t *>(lds) + (T) * TILE, *Ql_ = Qh_ + K * LDB, *Ph_ = Ql_ + K * LDB,   \
                 *Pl_ = Ph_ + K * LDB;                                                                                \
        floatx4 qa, qb;                                                                                               \
        _Pragma("unroll") for (int e = 0; e < 4; ++e) {                                                               \
            const bool live = MX[e] > PC_NEG_INF;                                                                     \
            const float g_ = MX[e] + (RC[e] - RS[e]);                                                                 \
            const float sb_ = pc_split_shift(g_);                                                                     \
            qa[e] = live ? (sb_ - MX[e]) * PC_LOG2E : PC_NEG_INF;                                                     \
            qb[e] = live ? (g_ - sb_ - PC_SPLIT_SCALE) * PC_LOG2E : PC_NEG_INF;                                       \
        }                                                                                                             \
        _Pragma("unroll") for (int i = 0; i < NL; ++i) {                                                              \
            floatx4 q, p;                                                                                             \
            _Pragma("unroll") for (int e = 0; e < 4; ++e) {                                                           \
                q[e] = __builtin_amdgcn_exp2f(fmaf(NF[i][e], PC_LOG2E, qa[e]));                                       \
                p[e] = __builtin_amdgcn_exp2f(fminf(fmaf(LC[i][e], PC_LOG2E, qb[e]), PC_SPLIT_CAP * PC_LOG2E));      \
            }                                                                                                         \
            uint32_t h0, l0, h1, l1;                                                                                  \
            const int at_ = (32 * i + srow) * LDB + (sc4 >> 1);                                                       \
            bf16_split2(q[0], q[1], h0, l0); bf16_split2(q[2], q[3], h1, l1);                                         \
            *reinterpret_cast<uint2 *>(Qh_ + at_) = make_uint2(h0, h1);                                               \
            *reinterpret_cast<uint2 *>(Ql_ + at_) = make_uint2(l0, l1);                                               \
            bf16_split2(p[0], p[1], h0, l0); bf16_split2(p[2], p[3], h1, l1);                                         \
            *reinterpret_cast<uint2 *>(Ph_ + at_) = make_uint2(h0, h1);                                               \
            *reinterpret_cast<uint2 *>(Pl_ + at_) = make_uint2(l0, l1);                                               \
        }                                                                                                             \
    } while (0)
#define PC_MATH_BF(T)                                                                                                 \
    do {                                                                                                              \
        const uint32_t *Qh_ = reinterpret_cast<const uint32_t *>(lds) + (T) * TILE, *Ql_ = Qh_ + K * LDB,             \
                       *Ph_ = Ql_ + K * LDB, *Pl_ = Ph_ + K * LDB;                                                    \
        _Pragma("unroll") for (int ks = 0; ks < 2; ++ks) {                                                            \
            bf16x8 ah[QT], al[QT], bh[QT], bl[QT];                                                                    \
            _Pragma("unroll") for (int rt = 0; rt < QT; ++rt) {                                                       \
                const int ra_ = (r0 + rt * 32 + l32) * LDB + 8 * ks + 4 * half, rb_ = (c0 + rt * 32 + l32) * LDB + 8 * ks + 4 * half; \
                ah[rt] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(Qh_ + ra_));                     \
                al[rt] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(Ql_ + ra_));                     \
                bh[rt] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(Ph_ + rb_));                     \
                bl[rt] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(Pl_ + rb_));                     \
            }                                                                                                         \
            _Pragma("unroll") for (int rt = 0; rt < QT; ++rt)                                                         \
                _Pragma("unroll") for (int ct = 0; ct < QT; ++ct) {                                                   \
                    acc[rt][ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[rt], bh[ct], acc[rt][ct], 0, 0, 0);      \
                    acc[rt][ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[rt], bl[ct], acc[rt][ct], 0, 0, 0);      \
                    acc[rt][ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[rt], bh[ct], acc[rt][ct], 0, 0, 0);      \
                }                                                                                                     \
        }                                                                                                             \
    } while (0)

    // n_chunks is the same for all four waves, so every wave reaches every barrier
    if (ONE) {
        if (n_chunks > 0) PC_ISSUE(0, nfA, lcA, mxA, rsA, rcA);
        for (int c = 0; c < n_chunks; ++c) {
            if (c > 0) __syncthreads();                                 // the tile has been read by everybody
            PC_STAGE(0, nfA, lcA, mxA, rsA, rcA);
            if (c + 1 < n_chunks) PC_ISSUE(c + 1, nfA, lcA, mxA, rsA, rcA);
            __syncthreads();
            PC_MATH(0);
        }
    } else {
    if (n_chunks > 0) PC_ISSUE(0, nfA, lcA, mxA, rsA, rcA);
    if (n_chunks > 1) PC_ISSUE(1, nfB, lcB, mxB, rsB, rcB);
    int c = 0;
    for (; c + 1 < n_chunks; c += 2) {                                  // pairs of chunks; a last single chunk follows
        if (BF) PC_STAGE_BF(0, nfA, lcA, mxA, rsA, rcA); else PC_STAGE(0, nfA, lcA, mxA, rsA, rcA);
        if (c + 2 < n_chunks) PC_ISSUE(c + 2, nfA, lcA, mxA, rsA, rcA);
        __syncthreads();
        if (BF) PC_MATH_BF(0); else PC_MATH(0);
        if (BF) PC_STAGE_BF(1, nfB, lcB, mxB, rsB, rcB); else PC_STAGE(1, nfB, lcB, mxB, rsB, rcB);
        if (c + 3 < n_chunks) PC_ISSUE(c + 3, nfB, lcB, mxB, rsB, rcB);
        __syncthreads();
        if (BF) PC_MATH_BF(1); else PC_MATH(1);
    }
    if (c < n_chunks) {
        if (BF) PC_STAGE_BF(0, nfA, lcA, mxA, rsA, rcA); else PC_STAGE(0, nfA, lcA, mxA, rsA, rcA);
        __syncthreads();
        if (BF) PC_MATH_BF(0); else PC_MATH(0);
    }
    }
#undef PC_ISSUE
#undef PC_STAGE
#undef PC_MATH
#undef PC_STAGE_BF
#undef PC_MATH_BF

    // flows out: all loads of a 32 x 32 tile first, then the arithmetic, then the stores (a load between two stores
    // would be waited for on its own); theta = 0: no flow (and never 0 * inf)
#pragma unroll
    for (int rt = 0; rt < QT; ++rt)
#pragma unroll
        for (int ct = 0; ct < QT; ++ct) {
            floatx16 thv, gv;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int i = r0 + rt * 32 + 8 * (e / 4) + 4 * half + (e % 4);
                const int64_t at = (int64_t)pb + (int64_t)i * K + c0 + ct * 32 + l32;
                thv[e] = theta[at];
                gv[e] = G[at];
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int i = r0 + rt * 32 + 8 * (e / 4) + 4 * half + (e % 4);
                const int64_t at = (int64_t)pb + (int64_t)i * K + c0 + ct * 32 + l32;
                const float inc = thv[e] > 0.0f ? pc_flow_out(thv[e], acc[rt][ct][e]) : 0.0f;
                if (n_split > 1) { if (inc != 0.0f) atomicAdd(G + at, inc); }
                else G[at] = gv[e] + inc;
            }
        }
}

// ------------------------------------------------------------------------------------------
// EM update
// ------------------------------------------------------------------------------------------
// Parameters: a wave takes one row of a row group (the weights of one sum node over all its parameter blocks), sums its flows
// and updates its weights; the flows stay in registers between the two, so they are read once and a pass needs no row sums
// in memory.  V consecutive columns per access; a row of more than 64 V NR columns is read a second time.  Bound by HBM: theta
// and flows read and written once.  Measured on the 49 140 blocks of 64 x 64 of a 3072-variable tree (3.2 GB moved): 0.55 ms,
// 5.8 TB/s, where the sums took 0.16 and the update 0.56 ms.
// SEG: much longer rows are cut into segments, and a wave takes one row of a segment: their sums come from k_em_row_sums (part),
// every segment adds up those of its group.  Measured on one row of 10 000 blocks of 32 columns: 1519 us by one wave, so 40 us.
template <int V, int NR, bool SEG>
__device__ inline void em_theta_rows(int g, int first_row, int row_step, float *__restrict__ theta, float *__restrict__ G, const int32_t *__restrict__ ptr,
                                     const int32_t *__restrict__ list, const int32_t *__restrict__ pb_rows, const int32_t *__restrict__ pb_cols,
                                     const int32_t *__restrict__ group_nch, int32_t n_groups, const int32_t *__restrict__ seg,
                                     const float *__restrict__ part, int32_t K, float step, float pc)
{
    typedef float vec __attribute__((ext_vector_type(V)));
    const int lane = threadIdx.x & 63;
    const int32_t *blk = list + ptr[g];
    const int n = ptr[g + 1] - ptr[g], kv = K / V, tot = n * kv;
    const int rows = g < n_groups ? pb_rows[blk[0]] : 0;
    const float share = g < n_groups ? pc / (float)(SEG ? seg[3 * g + 2] : group_nch[g]) : 0.0f;
    const vec zero = {};
    for (int i = first_row; i < K; i += row_step) {
        if (i >= rows) {                                                // wave-uniform: placeholders, unused blocks
            for (int q = lane; q < tot; q += 64)
                *reinterpret_cast<vec *>(G + (int64_t)blk[q / kv] * K * K + (int64_t)i * K + (q % kv) * V) = zero;
            continue;
        }
        vec f[NR];
        int64_t at[NR];
        int cols[NR];                                                   // real columns from the access on
        const bool held = tot <= 64 * NR;                               // uniform over the workgroup
        float s = 0.0f;
        auto place = [&](int q, int64_t &where, int &c) {
            const int b = blk[q / kv], j = (q % kv) * V;
            where = (int64_t)b * K * K + (int64_t)i * K + j;
            c = pb_cols[b] - j;
        };
        auto add = [&](vec x, int c) {
#pragma unroll
            for (int e = 0; e < V; ++e) s += e < c ? x[e] : 0.0f;
        };
        if (held) {
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int q = lane + 64 * r;
                cols[r] = 0;
                if (q < tot) { place(q, at[r], cols[r]); f[r] = *reinterpret_cast<const vec *>(G + at[r]); }
            }
#pragma unroll
            for (int r = 0; r < NR; ++r) if (!SEG && lane + 64 * r < tot) add(f[r], cols[r]);
        } else if (!SEG) {
            for (int q = lane; q < tot; q += 64) { place(q, at[0], cols[0]); add(*reinterpret_cast<const vec *>(G + at[0]), cols[0]); }
        }
        if (SEG) {
            const int first = seg[3 * g], n_seg = seg[3 * g + 1];
            for (int t = lane; t < n_seg; t += 64) s += part[(int64_t)(first + t) * K + i];
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        const float z = s + pc;
        auto update = [&](vec x, int64_t where, int c) {
            if (z > 0.0f && c > 0) {
                vec w = *reinterpret_cast<const vec *>(theta + where);
#pragma unroll
                for (int e = 0; e < V; ++e) if (e < c) w[e] = (1.0f - step) * w[e] + step * ((x[e] + share) / z);
                *reinterpret_cast<vec *>(theta + where) = w;
            }
            *reinterpret_cast<vec *>(G + where) = zero;
        };
        if (held) {
#pragma unroll
            for (int r = 0; r < NR; ++r) if (lane + 64 * r < tot) update(f[r], at[r], cols[r]);
        } else {
            for (int q = lane; q < tot; q += 64) { place(q, at[0], cols[0]); update(*reinterpret_cast<const vec *>(G + at[0]), at[0], cols[0]); }
        }
    }
}

template <int V, int NR, bool SEG>
__global__ __launch_bounds__(256) void k_em_theta(float *__restrict__ theta, float *__restrict__ G, const int32_t *__restrict__ ptr,
                                                  const int32_t *__restrict__ list, const int32_t *__restrict__ pb_rows,
                                                  const int32_t *__restrict__ pb_cols, const int32_t *__restrict__ group_nch,
                                                  int32_t n_groups, const int32_t *__restrict__ seg, const float *__restrict__ part,
                                                  int32_t K, float step, float pc)
{
    const int wave = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
    em_theta_rows<V, NR, SEG>(blockIdx.x, blockIdx.y * n_waves + wave, gridDim.y * n_waves, theta, G, ptr, list, pb_rows, pb_cols, group_nch, n_groups, seg,
                              part, K, step, pc);
}

// Row sums of the segments of long rows: a wave per row of a segment.
template <int V>
__global__ __launch_bounds__(256) void k_em_row_sums(const float *__restrict__ G, const int32_t *__restrict__ ptr,
                                                     const int32_t *__restrict__ list, const int32_t *__restrict__ pb_rows,
                                                     const int32_t *__restrict__ pb_cols, int32_t K, float *__restrict__ part)
{
    typedef float vec __attribute__((ext_vector_type(V)));
    const int g = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n_waves = blockDim.x >> 6;
    const int32_t *blk = list + ptr[g];
    const int kv = K / V, tot = (ptr[g + 1] - ptr[g]) * kv, rows = pb_rows[blk[0]];
    for (int i = blockIdx.y * n_waves + wave; i < rows; i += gridDim.y * n_waves) {
        float s = 0.0f;
        for (int q = lane; q < tot; q += 64) {
            const int b = blk[q / kv], j = (q % kv) * V, c = pb_cols[b] - j;
            const vec x = *reinterpret_cast<const vec *>(G + (int64_t)b * K * K + (int64_t)i * K + j);
#pragma unroll
            for (int e = 0; e < V; ++e) s += e < c ? x[e] : 0.0f;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        if (lane == 0) part[(int64_t)g * K + i] = s;
    }
}

// Tables whose flows one workgroup can hold in registers (16 float4 per thread): column sums and update in one pass, the flows
// read once.  K a power of two >= 4; a thread owns nodes 4 kq .. 4 kq + 3 of every R-th category, the partial column sums of the
// R rows of threads meet in LDS.  Measured on 12 288 tables of 256 x 64 (3.2 GB moved): 0.64 ms against 0.20 + 0.59 ms.
// THETA: small models, where a launch costs as much as the work, have the parameters in the same launch: n_tables workgroups for the
// tables, then those of k_em_theta, `shares` of a row group (16 x 32 HMM: 3.9 + 3.0 us, together 3.9).
template <int NT, bool THETA>
__global__ __launch_bounds__(NT) void k_em_tables_whole(float *__restrict__ tables, float *__restrict__ Gt, int32_t K, int32_t n_cats,
                                                        float step, float pc, int32_t n_tables, float *__restrict__ theta, float *__restrict__ G,
                                                        const EmDev em, int32_t shares)
{
    __shared__ float4 red[NT];
    if constexpr (THETA)
        if ((int)blockIdx.x >= n_tables) {
            const int q = (int)blockIdx.x - n_tables;
            em_theta_rows<4, 1, false>(q / shares, q % shares * 4 + (int)(threadIdx.x >> 6), shares * 4, theta, G, em.ptr, em.list, em.pb_rows, em.pb_cols,
                                       em.group_nch, em.n_groups, nullptr, nullptr, K, step, pc);
            return;
        }
    const float share = pc / (float)n_cats;
    const int k4n = K / 4, kq = threadIdx.x % k4n, rs = threadIdx.x / k4n, R = NT / k4n;
    float4 *tb = reinterpret_cast<float4 *>(tables + (int64_t)blockIdx.x * n_cats * K) + kq;
    float4 *gb = reinterpret_cast<float4 *>(Gt + (int64_t)blockIdx.x * n_cats * K) + kq;
    float4 g[16], z = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int c = rs + i * R;
        g[i] = c < n_cats ? gb[(int64_t)c * k4n] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) { z.x += g[i].x; z.y += g[i].y; z.z += g[i].z; z.w += g[i].w; }
    red[threadIdx.x] = z;
    __syncthreads();
    for (int o = NT / 2; o >= k4n; o >>= 1) {                           // the distances are multiples of k4n
        if ((int)threadIdx.x < o) {
            const float4 v = red[threadIdx.x + o];
            z.x += v.x; z.y += v.y; z.z += v.z; z.w += v.w;
            red[threadIdx.x] = z;
        }
        __syncthreads();
    }
    const float4 zr = red[kq];
    z = make_float4(zr.x + pc, zr.y + pc, zr.z + pc, zr.w + pc);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int c = rs + i * R;
        if (c >= n_cats) break;
        float4 w = tb[(int64_t)c * k4n];
        if (z.x > 0.0f) w.x = (1.0f - step) * w.x + step * ((g[i].x + share) / z.x);
        if (z.y > 0.0f) w.y = (1.0f - step) * w.y + step * ((g[i].y + share) / z.y);
        if (z.z > 0.0f) w.z = (1.0f - step) * w.z + step * ((g[i].z + share) / z.z);
        if (z.w > 0.0f) w.w = (1.0f - step) * w.w + step * ((g[i].w + share) / z.w);
        tb[(int64_t)c * k4n] = w;
        gb[(int64_t)c * k4n] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

// ztab[t*K + k] += sum over a slab of categories of table_flow[t][c][k]
__global__ __launch_bounds__(256) void k_em_tabsum(const float *__restrict__ Gt, int32_t K, int32_t n_cats,
                                                   int32_t cats_per_block, float *__restrict__ ztab)
{
    const int t = blockIdx.x;
    const int c0 = blockIdx.y * cats_per_block;
    const int c1 = min(n_cats, c0 + cats_per_block);
    for (int k = threadIdx.x; k < K; k += 256) {
        float s = 0.0f;
        for (int c = c0; c < c1; ++c) s += Gt[((int64_t)t * n_cats + c) * K + k];
        atomicAdd(ztab + (int64_t)t * K + k, s);
    }
}

// The same for K a multiple of 4 (K <= 128): a thread owns four consecutive nodes, the 256 threads cover
// 1024 / K categories per pass with 16-byte loads (four in flight per thread), partial sums meet in LDS.
__global__ __launch_bounds__(256) void k_em_tabsum_v4(const float *__restrict__ Gt, int32_t K, int32_t n_cats,
                                                      int32_t cats_per_block, float *__restrict__ ztab)
{
    __shared__ float4 red[256];
    const int t = blockIdx.x;
    const int c0 = blockIdx.y * cats_per_block;
    const int c1 = min(n_cats, c0 + cats_per_block);
    const int k4n = K / 4, kq = threadIdx.x % k4n, rs = threadIdx.x / k4n, R = 256 / k4n;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (rs < R) {
        const float4 *src = reinterpret_cast<const float4 *>(Gt + (int64_t)t * n_cats * K) + kq;
        for (int c = c0 + rs; c < c1; c += 4 * R) {
            float4 v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                v[j] = c + j * R < c1 ? src[(int64_t)(c + j * R) * k4n] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int j = 0; j < 4; ++j) { acc.x += v[j].x; acc.y += v[j].y; acc.z += v[j].z; acc.w += v[j].w; }
        }
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x < k4n) {
        float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int r2 = 0; r2 < R; ++r2) {
            const float4 v = red[r2 * k4n + threadIdx.x];
            sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
        }
        float *dst = ztab + (int64_t)t * K + threadIdx.x * 4;
        atomicAdd(dst + 0, sum.x); atomicAdd(dst + 1, sum.y); atomicAdd(dst + 2, sum.z); atomicAdd(dst + 3, sum.w);
    }
}

__global__ __launch_bounds__(256) void k_em_tables(float *__restrict__ tables, float *__restrict__ Gt,
                                                   const float *__restrict__ ztab, int32_t K, int32_t n_cats,
                                                   int64_t total, float step, float pc)
{
    const float share = pc / (float)n_cats;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t tc = i / K;
        const int k = (int)(i - tc * K);
        const int64_t t = tc / n_cats;
        const float z = ztab[t * K + k] + pc;
        if (z > 0.0f) {
            const float nw = (Gt[i] + share) / z;
            tables[i] = (1.0f - step) * tables[i] + step * nw;
        }
        Gt[i] = 0.0f;
    }
}

// The same for K a multiple of 4: one table per blockIdx.x, a thread owns four consecutive nodes of one category
// (16-byte accesses, 32-bit index arithmetic, the column sums of the table read once per thread).
__global__ __launch_bounds__(256) void k_em_tables_v4(float *__restrict__ tables, float *__restrict__ Gt,
                                                      const float *__restrict__ ztab, int32_t K, int32_t n_cats,
                                                      float step, float pc)
{
    const float share = pc / (float)n_cats;
    const int t = blockIdx.x;
    const int k4n = K / 4, kq = threadIdx.x % k4n, rs = threadIdx.x / k4n, R = 256 / k4n;
    if (rs >= R) return;
    const float4 zr = *reinterpret_cast<const float4 *>(ztab + (int64_t)t * K + kq * 4);
    const float4 z = make_float4(zr.x + pc, zr.y + pc, zr.z + pc, zr.w + pc);
    float4 *tb = reinterpret_cast<float4 *>(tables + (int64_t)t * n_cats * K) + kq;
    float4 *gb = reinterpret_cast<float4 *>(Gt + (int64_t)t * n_cats * K) + kq;
    for (int c = blockIdx.y * R + rs; c < n_cats; c += gridDim.y * R) {
        const int64_t at = (int64_t)c * k4n;
        const float4 g = gb[at];
        float4 w = tb[at];
        if (z.x > 0.0f) w.x = (1.0f - step) * w.x + step * ((g.x + share) / z.x);
        if (z.y > 0.0f) w.y = (1.0f - step) * w.y + step * ((g.y + share) / z.y);
        if (z.z > 0.0f) w.z = (1.0f - step) * w.z + step * ((g.z + share) / z.z);
        if (z.w > 0.0f) w.w = (1.0f - step) * w.w + step * ((g.w + share) / z.w);
        tb[at] = w;
        gb[at] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

// ------------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------------
static thread_local Profiler *g_prof = nullptr;
void set_profiler(Profiler *p) { g_prof = p; }

hipEvent_t Profiler::get()
{
    if (!pool.empty()) { hipEvent_t e = pool.back(); pool.pop_back(); return e; }
    hipEvent_t e = nullptr;
    (void)hipEventCreate(&e);
    return e;
}

void Profiler::collect(int64_t *launches, double *ms)
{
    for (Rec &r : recs) {
        float t = 0.0f;
        if (hipEventSynchronize(r.b) == hipSuccess && hipEventElapsedTime(&t, r.a, r.b) == hipSuccess) {
            launches[r.cls] += 1;
            ms[r.cls] += t;
        }
        pool.push_back(r.a);
        pool.push_back(r.b);
    }
    recs.clear();
}

Profiler::~Profiler()
{
    for (Rec &r : recs) { (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
    for (hipEvent_t e : pool) (void)hipEventDestroy(e);
}

Timed::Timed(int cls, hipStream_t stream) : s(stream)
{
    if (!g_prof) return;
    hipEvent_t a = g_prof->get();
    b = g_prof->get();
    (void)hipEventRecord(a, s);
    g_prof->recs.push_back({cls, a, b});
}
Timed::~Timed() { if (b) (void)hipEventRecord(b, s); }

static inline int grid_for(int64_t items, int per_block = 256, int cap = 1 << 16)
{
    int64_t g = (items + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

static bool g_force_generic = false;
void set_force_generic(bool on) { g_force_generic = on; }
static inline bool use_mfma(int32_t K) { return !g_force_generic && (K == 32 || K == 64 || K == 128); }
static inline bool use_small(int32_t K) { return !g_force_generic && (K == 1 || K == 2 || K == 4 || K == 8); }
static inline bool use_16(int32_t K) { return !g_force_generic && K == 16; }
#define PC_DISPATCH_SMALL(KERNEL, ...)                                                                     \
    do {                                                                                                   \
        if (K == 1) hipLaunchKernelGGL((KERNEL<1>), __VA_ARGS__);                                          \
        else if (K == 2) hipLaunchKernelGGL((KERNEL<2>), __VA_ARGS__);                                     \
        else if (K == 4) hipLaunchKernelGGL((KERNEL<4>), __VA_ARGS__);                                     \
        else hipLaunchKernelGGL((KERNEL<8>), __VA_ARGS__);                                                 \
    } while (0)

void launch_fill(float *p, int64_t n, float v, hipStream_t s)
{
    Timed timed(KC_MISC, s);
    if (n <= 0) return;
    hipLaunchKernelGGL(k_fill, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, p, n, v);
}

void launch_readout(const float *l, const float *R, int64_t root_row, int64_t root_blk, int64_t Bs, int32_t B, float *ll,
                    hipStream_t s)
{
    Timed timed(KC_MISC, s);
    hipLaunchKernelGGL(k_readout, dim3((B + 255) / 256), dim3(256), 0, s, l, R, root_row, root_blk, Bs, B, ll);
}

// Columns of an input tile, 0: no tile (larger blocks: it costs occupancy, rows are long enough).
int input_tile_cols(const GroupDev &g, int32_t K, int64_t Bs)
{
    if ((K & 3) != 0 || K > 64) return 0;
    return K == 32 && g.n_rows * (Bs / 128) >= 2048 ? 128 : 64;
}

// Blocks of which the tiles run on one XCD (input_tile_at): a table row that several of them need is then in its L2.  That pays where the tables of
// all blocks are more than an L2 holds, in whole eights (with a share of nine blocks one XCD has twice the others': B = 65536 45 us, all in turn 30).
// In turn / by XCD, 256 categories: K = 64, 12 288 blocks, B = 256 280 / 254 us, 2000 blocks, B = 1000 194 / 161, 65 blocks, B = 30000
// 125 / 121, 33 blocks 52 / 54; K = 32, 2000 blocks, B = 1000 86 / 80, 257 blocks, B = 1500 15.2 / 14.4, but B = 8000 68 / 73 and 600 blocks,
// B = 3000 65 / 68; K = 20 600 blocks, B = 1000 17.7 / 19.5, B = 3000 53 / 61.
int input_by_xcd(const GroupDev &g, int32_t K, int64_t Bs)
{
    const bool pays = K == 64 ? g.n_rows >= 64 : K == 32 && g.n_rows >= 256 && Bs <= 1536;
    return pays ? g.n_rows & ~7 : 0;
}

void launch_input_fwd(const float *tables, const int32_t *xT, const GroupDev &g, int32_t K, int32_t n_cats, int64_t Bs,
                      float *l, float *R, hipStream_t s)
{
    Timed timed(KC_INPUT_FWD, s);
    if (g.n_rows == 0) return;
    const int cols = input_tile_cols(g, K, Bs);
    if (cols > 0) {
        // a dimension of a grid takes fewer than 2^32 threads (512 blocks of 4 nodes at 2^21 samples are as many)
        const int64_t n_ct = (Bs + cols - 1) / cols;
        const int by_xcd = g.n_rows * n_ct < (1 << 24) ? input_by_xcd(g, K, Bs) : 0;
        const dim3 grid = by_xcd ? dim3((unsigned)(g.n_rows * n_ct)) : dim3((unsigned)g.n_rows, (unsigned)n_ct);
#define PC_INPUT_TILE(KK, CC) hipLaunchKernelGGL((k_input_fwd_tile<KK, CC>), grid, dim3(256), ((size_t)K * (CC + 1) + CC) * 4, s, tables, xT, g.ids, g.nbr, g.par, \
                                                 g.n_rows, by_xcd, (int32_t)n_ct, K, n_cats, Bs, l, R)
        if (cols == 128) PC_INPUT_TILE(32, 128);
        else if (K == 32) PC_INPUT_TILE(32, 64);
        else if (K == 64) PC_INPUT_TILE(64, 64);
        else PC_INPUT_TILE(0, 64);
#undef PC_INPUT_TILE
    } else {
        dim3 grid((unsigned)g.n_rows, (unsigned)((Bs + 255) / 256));
        hipLaunchKernelGGL(k_input_fwd, grid, dim3(256), 0, s, tables, xT, g.ids, g.nbr, g.par, K, n_cats, Bs, l, R);
    }
}

void launch_input_bwd(const float *F, const int32_t *xT, const GroupDev &g, int32_t K, int32_t n_cats, int64_t Bs,
                      float *table_flow, hipStream_t s)
{
    if (g.n_rows == 0) return;
    Timed timed(KC_INPUT_BWD, s);
    int lps = 1;                                                       // lanes per sample: next power of two >= K, at most 64
    while (lps < K && lps < 64) lps <<= 1;
    const size_t tile_bytes = ((size_t)K * 65 + 64) * 4;
    const size_t hist_bytes = (size_t)n_cats * K * 4 + tile_bytes;
    // more than 64 KB of dynamic LDS has to be allowed per kernel, once on every device the library runs on
    static std::atomic<uint64_t> attr_set{0};
    int dev = 0;
    (void)hipGetDevice(&dev);
    const uint64_t bit = 1ull << (dev & 63);
    if (!(attr_set.load(std::memory_order_relaxed) & bit)) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(k_input_bwd_hist), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  96 * 1024);
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(k_input_bwd_sorted<256>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  96 * 1024);
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(k_input_bwd_sorted<512>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  96 * 1024);
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(k_input_bwd_sorted<1024>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  96 * 1024);
        attr_set.fetch_or(bit, std::memory_order_relaxed);
    }
    // slab of samples for the sorted variant: a [K x SB] tile of at most 66 KB, two workgroups per CU.  Threads by the tile: 256 up to 16 KB (K = 32,
    // B = 128, 25 088 blocks 157 us, with 512 194), 512 up to 48 KB (B = 352 345, with 256 468, with 1024 415), then 1024 (B = 512 486, with 512
    // 542).  Four 16-byte loads of a thread are on their way during the sort, the whole tile up to 16 KB, 32 KB and 64 KB; what is left of a tile
    // of 32 to 48 KB or of the largest follows behind it.  256 threads at every size had wanted tiles of 34 KB, four workgroups per CU, and more
    // adds per category (B = 512 618; K = 64, 12 288 blocks, B = 256 507, now 322; 1568 blocks, B = 512 138, now 100).  Half as many workgroups
    // pay for few blocks, too: 4 blocks of 64, B = 512 16 -> 10, 64 blocks 17 -> 11, 16 blocks of 128 17 -> 11, 64 of 32 15 -> 9.
    int SB = 1024;
    while (SB > 32 && (size_t)K * (SB + 1) * 4 > 66 * 1024) SB >>= 1;
    if (SB > Bs) SB = (int)Bs;
    const size_t sorted_bytes = ((size_t)K * (SB + 1) + 2 * (size_t)SB + n_cats + 1 + 16) * 4;
    if (hist_bytes <= 96 * 1024 && (int64_t)n_cats * 4 <= Bs) {           // many samples per category: privatise in LDS
        hipLaunchKernelGGL(k_input_bwd_hist, dim3((unsigned)g.n_rows), dim3(256), hist_bytes, s, F, xT, g.ids, g.nbr, g.par, K,
                           n_cats, Bs, table_flow, lps, g.tied ? 1 : 0);
    } else if (n_cats <= 1024 && SB >= 64) {                             // few samples per category: combine them first
        const int n_slabs = (int)((Bs + SB - 1) / SB);
        dim3 grid((unsigned)g.n_rows, (unsigned)n_slabs);
#define PC_SORTED(NT) hipLaunchKernelGGL(k_input_bwd_sorted<NT>, grid, dim3(NT), sorted_bytes, s, F, xT, g.ids, g.nbr, g.par, K, n_cats, Bs, table_flow, SB, lps)
        const int64_t tile = (int64_t)K * SB * 4;
        if (tile <= 16 * 1024) PC_SORTED(256);
        else if (tile <= 48 * 1024) PC_SORTED(512);
        else PC_SORTED(1024);
#undef PC_SORTED
    } else {
        dim3 grid((unsigned)g.n_rows, (unsigned)((Bs + 63) / 64));
        hipLaunchKernelGGL(k_input_bwd_direct, grid, dim3(256), tile_bytes, s, F, xT, g.ids, g.nbr, g.par, K, n_cats, Bs,
                           table_flow, lps);
    }
}

// rows per thread and neighbours in flight by block size: 8-16 outstanding 16-byte loads per thread (at K = 32 eight
// neighbours in flight cost a fifth of the occupancy and 15 % of the PD's product-layer time)
#define PC_DISPATCH_PROD_M(KERNEL, MULTI, ...)                                                             \
    do {                                                                                                   \
        if (narrow) {                                /* 32 columns per workgroup: twice the workgroups, half the rows per thread */ \
            if (K <= 32) hipLaunchKernelGGL((KERNEL(1, 8, MULTI, 8)), __VA_ARGS__);                        \
            else if (K <= 64) hipLaunchKernelGGL((KERNEL(2, 4, MULTI, 8)), __VA_ARGS__);                   \
            else hipLaunchKernelGGL((KERNEL(4, 4, MULTI, 8)), __VA_ARGS__);                                \
        } else if (K <= 16) hipLaunchKernelGGL((KERNEL(1, 8, MULTI, 16)), __VA_ARGS__);                    \
        else if (K <= 32) hipLaunchKernelGGL((KERNEL(2, 4, MULTI, 16)), __VA_ARGS__);                      \
        else if (K <= 64) hipLaunchKernelGGL((KERNEL(4, 4, MULTI, 16)), __VA_ARGS__);                      \
        else hipLaunchKernelGGL((KERNEL(8, 2, MULTI, 16)), __VA_ARGS__);                                   \
    } while (0)
#define PC_DISPATCH_PROD(KERNEL, ...)                                                                      \
    do {                                                                                                   \
        if (gs.n > 1) PC_DISPATCH_PROD_M(KERNEL, PC_ROWS_MULTI, __VA_ARGS__);                              \
        else PC_DISPATCH_PROD_M(KERNEL, PC_ROWS_ONE, __VA_ARGS__);                                         \
    } while (0)
#define PC_PROD_FWD_F32(RPT, U, MULTI, CL) k_prod_fwd<RPT, U, MULTI, CL, float, false>
#define PC_PROD_FWD_F64(RPT, U, MULTI, CL) k_prod_fwd<RPT, U, MULTI, CL, double, false>
#define PC_PROD_FWD_F32_P(RPT, U, MULTI, CL) k_prod_fwd<RPT, U, MULTI, CL, float, true>
#define PC_PROD_FWD_F64_P(RPT, U, MULTI, CL) k_prod_fwd<RPT, U, MULTI, CL, double, true>
#define PC_PROD_BWD(RPT, U, MULTI, CL) k_prod_bwd<RPT, U, MULTI, CL, false>
#define PC_PROD_BWD_P(RPT, U, MULTI, CL) k_prod_bwd<RPT, U, MULTI, CL, true>
// small launches (the deep narrow circuits) use 32-column workgroups
static inline bool prod_narrow(const GroupSet &gs, int64_t Bs) { return (int64_t)gs.first[gs.n] * ((Bs + 63) / 64) < 1024; }

// Sets of at most PC_MAX_SET groups, widest rows first (the longest rows start first, so they do not trail the launch).
std::vector<GroupSet> make_group_sets(const std::vector<GroupDev> &groups)
{
    std::vector<const GroupDev *> order;
    for (const GroupDev &g : groups)
        if (g.n_rows > 0) order.push_back(&g);
    std::stable_sort(order.begin(), order.end(), [](const GroupDev *a, const GroupDev *b) { return a->width > b->width; });
    std::vector<GroupSet> sets;
    for (size_t i = 0; i < order.size(); ++i) {
        if (i % PC_MAX_SET == 0) { sets.emplace_back(); std::memset(&sets.back(), 0, sizeof(GroupSet)); }
        GroupSet &gs = sets.back();
        const GroupDev &g = *order[i];
        const int k = gs.n++;
        gs.first[k + 1] = gs.first[k] + g.n_rows;
        gs.width[k] = g.width;
        gs.ids[k] = g.ids; gs.nbr[k] = g.nbr; gs.par[k] = g.par; gs.aux[k] = g.aux;
    }
    return sets;
}
static inline int32_t set_rows(const GroupSet &gs) { return gs.first[gs.n]; }
static inline int32_t set_width(const GroupSet &gs)
{
    int32_t w = 0;
    for (int k = 0; k < gs.n; ++k) w = std::max(w, gs.width[k]);
    return w;
}

void launch_prod_fwd(const float *l, float *lout, float *R, const std::vector<GroupSet> &sets, int32_t K, int64_t Bs, void *Ph, void *Pl,
                     hipStream_t s)
{
    uint4 *ph = (uint4 *)Ph, *pl = (uint4 *)Pl;                          // non-null: also write the bf16 value planes
    for (const GroupSet &gs : sets) {
        Timed timed(KC_PROD_FWD, s);
        const bool narrow = prod_narrow(gs, Bs);
        dim3 grid((unsigned)set_rows(gs), (unsigned)(narrow ? (Bs + 31) / 32 : (Bs + 63) / 64));
        // rows with more than eight children (leaf products over many variables) are summed in double
        if (ph && (K % 16) == 0) {
            if (set_width(gs) > 8) PC_DISPATCH_PROD(PC_PROD_FWD_F64_P, grid, dim3(256), 0, s, l, lout, R, gs, K, Bs, ph, pl);
            else PC_DISPATCH_PROD(PC_PROD_FWD_F32_P, grid, dim3(256), 0, s, l, lout, R, gs, K, Bs, ph, pl);
        } else if (set_width(gs) > 8) PC_DISPATCH_PROD(PC_PROD_FWD_F64, grid, dim3(256), 0, s, l, lout, R, gs, K, Bs, ph, pl);
        else PC_DISPATCH_PROD(PC_PROD_FWD_F32, grid, dim3(256), 0, s, l, lout, R, gs, K, Bs, ph, pl);
    }
}

// rows of several layers as one launch of neighbour lists (CSR); K is 32, 64 or 128
static GroupSet csr_set(const RowsDev &rows)
{
    GroupSet gs;
    std::memset(&gs, 0, sizeof(gs));
    gs.n = 1;
    gs.first[1] = rows.n_rows;
    gs.width[0] = rows.max_nbr; gs.width[1] = rows.li0;
    gs.ids[0] = rows.ids; gs.nbr[0] = rows.list; gs.nbr[1] = rows.lay; gs.par[0] = rows.start; gs.aux[0] = rows.aux;
    return gs;
}

#define PC_DISPATCH_CLASS(KERNEL, U, ...)                                                                  \
    do {                                                                                                   \
        if (narrow) {                                                                                      \
            if (K <= 32) hipLaunchKernelGGL((KERNEL<1, U, 8>), __VA_ARGS__);                               \
            else if (K <= 64) hipLaunchKernelGGL((KERNEL<2, U, 8>), __VA_ARGS__);                          \
            else hipLaunchKernelGGL((KERNEL<4, U / 2, 8>), __VA_ARGS__);                                   \
        } else if (K <= 16) hipLaunchKernelGGL((KERNEL<1, U, 16>), __VA_ARGS__);                           \
        else if (K <= 32) hipLaunchKernelGGL((KERNEL<2, U, 16>), __VA_ARGS__);                             \
        else if (K <= 64) hipLaunchKernelGGL((KERNEL<4, U / 2, 16>), __VA_ARGS__);                         \
        else hipLaunchKernelGGL((KERNEL<8, U / 4, 16>), __VA_ARGS__);                                      \
    } while (0)
// Where k_prod_fwd sums rows of more than eight children in fours of fp32 and double beyond, in launches that fill the chip (a narrow one
// takes eights at K = 32, and tiles would leave most CUs idle: RAT-SPN of 100 variables, B = 3, 38.5 -> 44 us), and where the tiles hold 6 of
// 16 products and more: sets of two classes (4 of 16) have nothing to share, RAT-SPNs of 784 and 300 variables, four replicas, depth 4, S / K =
// 2, B = 480, k_prod_fwd -> 4 x 4: K = 32 146 -> 156, 70 -> 66 us, K = 64 283 -> 277, 115 -> 129; 2 x 2 at K = 32 225, 93.  Sets of
// five (25 of 64): 784 variables, depth 3, B = 256 392 -> 236 (K = 32), 751 -> 490 (K = 64); of three (9 of 16): 163 -> 103, 288 -> 242.
bool prod_takes_tiles(int32_t K, int32_t n_rows, int32_t n_tiles, int32_t width, int64_t Bs)
{
    return (K == 32 || K == 64) && width > 8 && n_rows >= 6 * (int64_t)n_tiles && (int64_t)n_rows * ((Bs + 63) / 64) >= 1024;
}

// 2 x 2 products a workgroup where 4 x 4 make less than 192 workgroups, which full tiles can at K = 32 only.  RAT-SPNs at K = 32, k_prod_fwd / 2 x 2 /
// 4 x 4: 128 workgroups 297 / 241 / 257, 72 / 53 / 64, 71 / 59 / 70 us (784, 400, 300 variables), 248 .. 256 564 / 381 / 265, 116 / 75 / 70, 123 / 90 /
// 75, 384 178 / 127 / 119.  At K = 64 4 x 4 are the faster ones from the smallest launches on (240 .. 256 workgroups 150 / 138 / 108, 202 / 164 / 142,
// 752 / 633 / 496).
ProdTile prod_tile_shape(int32_t n_tiles, int32_t K, int64_t Bs)
{
    if (K == 64) return ProdTile{8, 4};
    return ProdTile{16, (int64_t)n_tiles * (Bs / 32) < 192 ? 2 : 4};
}
void launch_prod_fwd_tiles(float *l, float *R, const int32_t *tile, int32_t n_tiles, const int32_t *order, const int32_t *cls_blk, int32_t K,
                           int64_t Bs, hipStream_t s)
{
    Timed timed(KC_PROD_FWD, s);
    const ProdTile t = prod_tile_shape(n_tiles, K, Bs);
    const bool small = t.side == 2;
    const int64_t wgs = (int64_t)((n_tiles * (small ? 4 : 1) + 3) & ~3) * (Bs / (2 * t.pairs));
    const dim3 grid((unsigned)((wgs + 31) / 32 * 32));
#define PC_PROD_TILE(CC, TT) hipLaunchKernelGGL((k_prod_tile<CC, TT>), grid, dim3(512), 0, s, l, R, tile, n_tiles, order, cls_blk, K, Bs)
    if (K == 64) PC_PROD_TILE(8, 4);
    else if (small) PC_PROD_TILE(16, 2);
    else PC_PROD_TILE(16, 4);
#undef PC_PROD_TILE
}

void launch_prod_bwd_classes(float *F, const ClassesDev &c, int32_t K, int64_t Bs, hipStream_t s)
{
    Timed timed(KC_PROD_BWD, s);
    const bool narrow = (int64_t)c.n * ((Bs + 63) / 64) < 1024;
    const int64_t tiles = (int64_t)c.n * (narrow ? (Bs + 31) / 32 : (Bs + 63) / 64);
    const int shares = (int)std::max<int64_t>(1, std::min<int64_t>(4096 / tiles, c.avg / 4));
    dim3 grid((unsigned)c.n, (unsigned)(narrow ? (Bs + 31) / 32 : (Bs + 63) / 64), (unsigned)shares);
    PC_DISPATCH_CLASS(k_class_bwd, 8, grid, dim3(256), 0, s, F, c, K, Bs);
}

void launch_prod_fwd_rows(float *l, float *R, const RowsDev &rows, int32_t K, int64_t Bs, hipStream_t s)
{
    if (rows.n_rows == 0) return;
    Timed timed(KC_PROD_FWD, s);
    const GroupSet gs = csr_set(rows);
    const bool narrow = prod_narrow(gs, Bs);
    dim3 grid((unsigned)rows.n_rows, (unsigned)(narrow ? (Bs + 31) / 32 : (Bs + 63) / 64));
    if (rows.max_nbr > 8) PC_DISPATCH_PROD_M(PC_PROD_FWD_F64, PC_ROWS_CSR, grid, dim3(256), 0, s, l, l, R, gs, K, Bs, nullptr, nullptr);
    else PC_DISPATCH_PROD_M(PC_PROD_FWD_F32, PC_ROWS_CSR, grid, dim3(256), 0, s, l, l, R, gs, K, Bs, nullptr, nullptr);
}

void launch_prod_bwd_rows(const float *l, float *F, float *N, float *nfmax, const RowsDev &rows, int32_t K, int64_t Bs, void *Ph,
                          void *Pl, hipStream_t s)
{
    if (rows.n_rows == 0) return;
    Timed timed(KC_PROD_BWD, s);
    const GroupSet gs = csr_set(rows);
    const bool narrow = prod_narrow(gs, Bs);
    dim3 grid((unsigned)rows.n_rows, (unsigned)(narrow ? (Bs + 31) / 32 : (Bs + 63) / 64));
    uint4 *ph = (uint4 *)Ph, *pl = (uint4 *)Pl;
    if (ph) PC_DISPATCH_PROD_M(PC_PROD_BWD_P, PC_ROWS_CSR, grid, dim3(256), 0, s, l, F, F, N, nfmax, gs, K, Bs, ph, pl);
    else PC_DISPATCH_PROD_M(PC_PROD_BWD, PC_ROWS_CSR, grid, dim3(256), 0, s, l, F, F, N, nfmax, gs, K, Bs, nullptr, nullptr);
}

void launch_prod_bwd(const float *l, float *F, const float *Fpar, float *N, float *nfmax, const std::vector<GroupSet> &sets, int32_t K,
                     int64_t Bs, void *Ph, void *Pl, hipStream_t s)
{
    uint4 *ph = (uint4 *)Ph, *pl = (uint4 *)Pl;                          // non-null: also write the bf16 planes of finished sum blocks
    for (const GroupSet &gs : sets) {
        Timed timed(KC_PROD_BWD, s);
        const bool narrow = prod_narrow(gs, Bs);
        dim3 grid((unsigned)set_rows(gs), (unsigned)(narrow ? (Bs + 31) / 32 : (Bs + 63) / 64));
        if (ph && (K % 16) == 0) PC_DISPATCH_PROD(PC_PROD_BWD_P, grid, dim3(256), 0, s, l, F, Fpar, N, nfmax, gs, K, Bs, ph, pl);
        else PC_DISPATCH_PROD(PC_PROD_BWD, grid, dim3(256), 0, s, l, F, Fpar, N, nfmax, gs, K, Bs, ph, pl);
    }
}

// forward / backward-to-children: (K, rows per wave tile / 32, waves sharing one tile)
#define PC_SUM_CASE(KK, RR, SS, BWD, ...)                                                                  \
    if (K == KK && rt == RR && split == SS) {                                                              \
        if (gs.n > 1) hipLaunchKernelGGL((k_sum_mfma<KK, RR, SS, BWD, true, 0>), __VA_ARGS__);             \
        else if (RR == 1 && prefetch) hipLaunchKernelGGL((k_sum_mfma<KK, 1, SS, BWD, false, 1>), __VA_ARGS__); \
        else if (BWD && wait_all) hipLaunchKernelGGL((k_sum_mfma<KK, RR, SS, BWD, false, BWD ? 2 : 0>), __VA_ARGS__); \
        else hipLaunchKernelGGL((k_sum_mfma<KK, RR, SS, BWD, false, 0>), __VA_ARGS__);                     \
        break;                                                                                             \
    }
// eight or sixteen waves to a tile: rows of 32 (pick_sum_shape), a register budget without a second operand set at sixteen
#define PC_SUM_WIDE(KK, SS, BWD, ...)                                                                      \
    if (K == KK && rt == 1 && split == SS) {                                                               \
        if (gs.n > 1) hipLaunchKernelGGL((k_sum_mfma<KK, 1, SS, BWD, true, 0>), __VA_ARGS__);              \
        else if (SS == 8 && prefetch) hipLaunchKernelGGL((k_sum_mfma<KK, 1, SS, BWD, false, SS == 8 ? 1 : 0>), __VA_ARGS__); \
        else hipLaunchKernelGGL((k_sum_mfma<KK, 1, SS, BWD, false, 0>), __VA_ARGS__);                      \
        break;                                                                                             \
    }
#define PC_DISPATCH_SUM(BWD, ...)                                                                         \
    do {                                                                                                  \
        PC_SUM_WIDE(32, 8, BWD, __VA_ARGS__) PC_SUM_WIDE(64, 8, BWD, __VA_ARGS__) PC_SUM_WIDE(128, 8, BWD, __VA_ARGS__)            \
        PC_SUM_WIDE(32, 16, BWD, __VA_ARGS__) PC_SUM_WIDE(64, 16, BWD, __VA_ARGS__) PC_SUM_WIDE(128, 16, BWD, __VA_ARGS__)         \
        PC_SUM_CASE(32, 1, 1, BWD, __VA_ARGS__) PC_SUM_CASE(32, 1, 2, BWD, __VA_ARGS__) PC_SUM_CASE(32, 1, 4, BWD, __VA_ARGS__)    \
        PC_SUM_CASE(64, 1, 1, BWD, __VA_ARGS__) PC_SUM_CASE(64, 1, 2, BWD, __VA_ARGS__) PC_SUM_CASE(64, 1, 4, BWD, __VA_ARGS__)    \
        PC_SUM_CASE(64, 2, 1, BWD, __VA_ARGS__) PC_SUM_CASE(64, 2, 2, BWD, __VA_ARGS__) PC_SUM_CASE(64, 2, 4, BWD, __VA_ARGS__)    \
        PC_SUM_CASE(128, 1, 1, BWD, __VA_ARGS__) PC_SUM_CASE(128, 1, 2, BWD, __VA_ARGS__) PC_SUM_CASE(128, 1, 4, BWD, __VA_ARGS__) \
        PC_SUM_CASE(128, 2, 1, BWD, __VA_ARGS__) PC_SUM_CASE(128, 2, 2, BWD, __VA_ARGS__) PC_SUM_CASE(128, 2, 4, BWD, __VA_ARGS__) \
    } while (0)

// Tile shape for the forward / backward-to-children kernel: the largest row tile (least exp work and
// neighbour traffic per flop) that still leaves two waves per SIMD (2048 waves on 256 CUs), splitting
// the reduction over up to four waves when rows x columns alone are too few, and over eight or sixteen where each still has
// two chunks: a wave has one or two chunks in flight, 1.2 us of latency each (a RAT-SPN's root over 256 blocks of 32 nodes, one tile:
// 79 us with four waves).  Four -> up to sixteen: HMM H = 4096, B = 10, per layer forward 39 -> 28 us, backward 41 -> 27;
// H = 3072 in blocks of 64, B = 40 31 -> 23, 32 -> 21; RAT-SPN of 784 variables, B = 16, forward pass 300 -> 251.  (Eight from one chunk a wave
// on: PD of 5 x 5 cells, B = 100 106 -> 108 us.)
static void pick_sum_shape(int32_t K, int32_t n_rows, int32_t width, int64_t Bs, int &rt, int &split)
{
    const int64_t col_tiles = (Bs + 31) / 32;
    const int64_t want = 2048;
    rt = K / 32 > 2 ? 2 : K / 32;                                      // 64-row wave tiles at most (register budget)
    while (rt > 1 && (int64_t)n_rows * (K / (32 * rt)) * col_tiles * 4 < want) rt >>= 1;
    const int64_t tiles = (int64_t)n_rows * (K / (32 * rt)) * col_tiles;
    split = 1;
    while (split < (rt == 1 ? 16 : 4) && tiles * split < want && (int64_t)width * (K / 32) >= (split < 4 ? 2 : 4) * split) split <<= 1;
}

// Forward, a layer of one row block with a long row (a root): parts of the row to as many workgroups of four waves, two chunks to a wave and more,
// and a launch that merges them.  One workgroup per tile reads through one CU's 64 bytes a clock, 8 KiB a chunk.  The parts lie in
// rows that belong to the row's children in an array that nobody reads them from (N; with recomputed products the window of F): the rows of the
// first child are the first part's sums, and so on; two rows a part, its shift and reference, follow in those of the next child or, at K = 32, two
// (they are there: parts <= width * K / 256, and 64 chunks).
// Root over 256 blocks of 32 nodes, sixteen waves and the readout / parts, merge and readout in one: B = 16 51 + 4 / 6 + 4 us, B = 512 49 + 5 / 9 + 5;
// at 32 tiles, RAT-SPN of 64 variables, all sum launches of a forward pass: K = 32, B = 1000 166 / 133, K = 128, S = 512, B = 256 81 / 45.  Both lines
// lie inside what pays: 64 tiles of 128 (B = 500) 108 / 78, rows of 48 chunks of 32 (R = 3, S = 128, B = 500) 29 / 21.
static int sum_parts(int32_t K, int32_t n_groups, int32_t n_rows, int32_t width, int64_t Bs)
{
    const int64_t chunks = (int64_t)width * (K / 32), tiles = (K / 32) * ((Bs + 31) / 32);
    if (n_groups != 1 || n_rows != 1 || chunks < 64 || tiles > 32) return 1;
    return (int)std::min<int64_t>(std::min<int64_t>(32, chunks / 8), 512 / tiles);
}

void sum_kernel_name(char (&name)[64], const GroupSet &gs, bool bwd, int32_t K, int64_t Bs)
{
    const char *dir = bwd ? "bwd" : "fwd";
    if (use_mfma(K)) {
        int rt, split;
        pick_sum_shape(K, set_rows(gs), set_width(gs), Bs, rt, split);
        if (!bwd && sum_parts(K, gs.n, set_rows(gs), set_width(gs), Bs) > 1) std::snprintf(name, sizeof(name), "k_sum_mfma<%d, 1, 4, false, false, 3>", (int)K);
        else std::snprintf(name, sizeof(name), "k_sum_mfma<%d, %d, %d, %s>", (int)K, rt, split, bwd ? "true" : "false");
    } else if (use_16(K)) {
        std::snprintf(name, sizeof(name), "k_sum_16<%s>", bwd ? "true" : "false");
    } else if (use_small(K)) {
        std::snprintf(name, sizeof(name), "k_sum_%s_small<%d>", dir, (int)K);
    } else {
        std::snprintf(name, sizeof(name), bwd ? "k_sum_bwd_child_generic" : "k_sum_fwd_generic");
    }
}

// K = 16: forward (F null; X = l of the children) or backward to the children (X = log_nf).  The neighbours of a row
// are dealt to four waves where the tiles alone leave less than a wave per SIMD.  All groups of the layer in one launch: three launches
// of 28 sets of 1024 x 1024, 30 % kept, B = 333 took 161 us forward and 158 backward, one 143 and 145.
static void launch_sum_16(const float *theta, const float *X, float *l, float *R, const float *nfmax, float *F, const GroupSet &gs, int64_t Bs,
                          hipStream_t s)
{
    const int64_t cgs = Bs / 32;
    const bool split = (int64_t)set_rows(gs) * cgs < 1024 && set_width(gs) >= 8;
    const dim3 grid((unsigned)set_rows(gs), (unsigned)(split ? cgs : (cgs + 3) / 4));
    const GroupDev one{gs.first[1], gs.width[0], gs.ids[0], gs.nbr[0], gs.par[0], false, gs.aux[0]};
#define PC_SUM_16(BB, SS)                                                                                                     \
    do {                                                                                                                      \
        if (gs.n > 1) hipLaunchKernelGGL((k_sum_16<BB, SS, GroupSet>), grid, dim3(256), 0, s, theta, X, l, R, nfmax, F, gs, Bs);     \
        else hipLaunchKernelGGL((k_sum_16<BB, SS, GroupDev>), grid, dim3(256), 0, s, theta, X, l, R, nfmax, F, one, Bs);      \
    } while (0)
    if (F) { if (split) PC_SUM_16(true, 4); else PC_SUM_16(true, 1); }
    else { if (split) PC_SUM_16(false, 4); else PC_SUM_16(false, 1); }
#undef PC_SUM_16
}

bool launch_sum_fwd(const float *theta, const float *lch, float *l, float *R, float *part, const std::vector<GroupSet> &sets, int32_t K,
                    int64_t Bs, float *ll, int32_t B, hipStream_t s)
{
    bool read_out = false;
    if (use_mfma(K)) {
        for (const GroupSet &gs : sets) {
            Timed timed(KC_SUM_FWD, s);
            const int parts = sets.size() == 1 ? sum_parts(K, gs.n, set_rows(gs), set_width(gs), Bs) : 1;
            if (parts > 1) {
                GroupSet ps = gs;
                ps.first[2] = parts;
                const dim3 grid((unsigned)(parts * (K / 32)), (unsigned)(Bs / 32));
#define PC_SUM_PART(KK) hipLaunchKernelGGL((k_sum_mfma<KK, 1, 4, false, false, 3>), grid, dim3(256), 0, s, theta, l, R, lch, (const float *)nullptr, part, ps, Bs)
                if (K == 32) PC_SUM_PART(32); else if (K == 64) PC_SUM_PART(64); else PC_SUM_PART(128);
#undef PC_SUM_PART
                hipLaunchKernelGGL(k_sum_merge, dim3((unsigned)(K / 8), (unsigned)(Bs / 32)), dim3(256), 0, s, part, gs.nbr[0], parts, l, R, gs.ids[0], K, Bs, ll, B);
                read_out = ll != nullptr;
                continue;
            }
            int rt, split;
            pick_sum_shape(K, set_rows(gs), set_width(gs), Bs, rt, split);
            const int waves = std::max(split, 4);
            const int64_t cols_per_wg = 32 * (waves / split);
            dim3 grid((unsigned)(set_rows(gs) * (K / (32 * rt))), (unsigned)((Bs + cols_per_wg - 1) / cols_per_wg));
            const bool prefetch = (int64_t)grid.x * grid.y * waves <= 1024;   // at most one wave per SIMD
            // long reductions at two waves per SIMD or fewer: see WAIT_ALL in the kernel
            const bool wait_all = (int64_t)set_width(gs) * (K / 32) >= 16 * split && (int64_t)grid.x * grid.y * waves <= 2048;
            (void)wait_all;
            PC_DISPATCH_SUM(false, grid, dim3(64 * waves), 0, s, theta, l, R, lch, (const float *)nullptr,
                            (float *)nullptr, gs, Bs);
        }
        return read_out;
    }
    if (use_16(K)) {
        for (const GroupSet &gs : sets) {
            Timed timed(KC_SUM_FWD, s);
            launch_sum_16(theta, lch, l, R, nullptr, nullptr, gs, Bs, s);
        }
        return read_out;
    }
    // other block sizes: one launch per group
    for (const GroupSet &gs : sets) for (int k = 0; k < gs.n; ++k) {
        const GroupDev g{gs.first[k + 1] - gs.first[k], gs.width[k], gs.ids[k], gs.nbr[k], gs.par[k], false, gs.aux[k]};
        Timed timed(KC_SUM_FWD, s);
        if (use_small(K)) {
            dim3 grid((unsigned)g.n_rows, (unsigned)((Bs + 255) / 256));
            PC_DISPATCH_SMALL(k_sum_fwd_small, grid, dim3(256), 0, s, theta, lch, l, R, g.ids, g.nbr, g.par, g.aux, g.width, Bs);
        } else {
            const int64_t items = (int64_t)g.n_rows * K * Bs;
            hipLaunchKernelGGL(k_sum_fwd_generic, dim3(grid_for(items)), dim3(256), 0, s, theta, lch, l, R, g.ids, g.nbr, g.par,
                               g.n_rows, g.width, K, Bs);
        }
    }
    return read_out;
}

void launch_sum_bwd_child(const float *theta, const float *l, const float *R, const float *N, const float *nfmax, float *F,
                          const std::vector<GroupSet> &sets, int32_t K, int64_t Bs, hipStream_t s)
{
    if (use_mfma(K)) {
        for (const GroupSet &gs : sets) {
            Timed timed(KC_SUM_BWD_CHILD, s);
            int rt, split;
            pick_sum_shape(K, set_rows(gs), set_width(gs), Bs, rt, split);
            const int waves = std::max(split, 4);
            const int64_t cols_per_wg = 32 * (waves / split);
            dim3 grid((unsigned)(set_rows(gs) * (K / (32 * rt))), (unsigned)((Bs + cols_per_wg - 1) / cols_per_wg));
            const bool prefetch = (int64_t)grid.x * grid.y * waves <= 1024;   // at most one wave per SIMD
            // long reductions at two waves per SIMD or fewer: see WAIT_ALL in the kernel
            const bool wait_all = (int64_t)set_width(gs) * (K / 32) >= 16 * split && (int64_t)grid.x * grid.y * waves <= 2048;
            (void)wait_all;
            PC_DISPATCH_SUM(true, grid, dim3(64 * waves), 0, s, theta, const_cast<float *>(l), const_cast<float *>(R), N, nfmax,
                            F, gs, Bs);
        }
        return;
    }
    if (use_16(K)) {
        for (const GroupSet &gs : sets) {
            Timed timed(KC_SUM_BWD_CHILD, s);
            launch_sum_16(theta, N, const_cast<float *>(l), const_cast<float *>(R), nfmax, F, gs, Bs, s);
        }
        return;
    }
    // other block sizes: one launch per group
    for (const GroupSet &gs : sets) for (int k = 0; k < gs.n; ++k) {
        const GroupDev g{gs.first[k + 1] - gs.first[k], gs.width[k], gs.ids[k], gs.nbr[k], gs.par[k], false, gs.aux[k]};
        Timed timed(KC_SUM_BWD_CHILD, s);
        if (use_small(K)) {
            dim3 grid((unsigned)g.n_rows, (unsigned)((Bs + 255) / 256));
            PC_DISPATCH_SMALL(k_sum_bwd_small, grid, dim3(256), 0, s, theta, l, R, N, nfmax, F, g.ids, g.nbr, g.par, g.aux,
                              g.width, Bs);
        } else {
            const int64_t items = (int64_t)g.n_rows * K * Bs;
            hipLaunchKernelGGL(k_sum_bwd_child_generic, dim3(grid_for(items)), dim3(256), 0, s, theta, l, R, N, F, g.ids, g.nbr,
                               g.par, g.aux, g.n_rows, g.width, K, Bs);
        }
    }
}

void launch_sum_bwd_param_generic(const float *theta, const float *l, const float *R, const float *N, float *G,
                                  const GroupDev &g, int32_t K, int64_t Bs, int32_t B, hipStream_t s)
{
    if (g.n_rows == 0) return;
    Timed timed(KC_SUM_BWD_PARAM, s);
    const int64_t items = (int64_t)g.n_rows * g.width * K * K;
    hipLaunchKernelGGL(k_sum_bwd_param_generic, dim3(grid_for(items)), dim3(256), 0, s, theta, l, R, N, G, g.ids, g.nbr,
                       g.par, g.n_rows, g.width, K, Bs, B, g.tied ? 1 : 0);
}

static int bf16_enabled()                                              // PC_BF16=0 keeps every layer on the fp32 matrix cores
{
    static const int on = [] { const char *e = std::getenv("PC_BF16"); return (e && e[0] == '0') ? 0 : 1; }();
    return on;
}

bool use_flow() { return !g_force_generic; }
bool param_flow_by_block(int32_t K) { return use_mfma(K) || use_16(K) || use_small(K); }

void launch_param_flow(const float *theta, const float *l, const float *R, const float *N, const float *nfmax, float *G,
                       const ParamFlowDev &pf, int32_t K, int64_t Bs, hipStream_t s)
{
    if (pf.n_pb == 0) return;
    Timed timed(KC_SUM_BWD_PARAM, s);
    if (use_small(K)) {
        const dim3 grid((unsigned)((pf.n_pb + 3) / 4));
#define PC_PF_SMALL(KK, IG)                                                                                         \
    hipLaunchKernelGGL((k_param_flow_small<KK, IG>), grid, dim3(256), 0, s, theta, l, R, N, nfmax, G, pf.pb, pf.ptr, \
                       pf.sum, pf.child, pf.n_pb, Bs)
        if (K == 1) PC_PF_SMALL(1, 1);
        else if (K == 2) PC_PF_SMALL(2, 2);
        else if (K == 4) PC_PF_SMALL(4, 4);
        else PC_PF_SMALL(8, 8);
#undef PC_PF_SMALL
    } else if (use_16(K)) {
        // few blocks with many tied pairs each: split the pairs over waves until the launch has some 1024 of them
        const int n_split = (int)std::max<int64_t>(1, std::min<int64_t>(pf.n_pairs / pf.n_pb, 1024 / pf.n_pb));
        hipLaunchKernelGGL(k_param_flow_16, dim3((unsigned)(((int64_t)pf.n_pb * n_split + 3) / 4)), dim3(256), 0, s, theta, l, R, N, nfmax, G,
                           pf.pb, pf.ptr, pf.sum, pf.child, pf.n_pb, n_split, Bs);
    } else if (K == 32) {
        // few blocks with many tied pairs each: their chunks are dealt to waves, which add their parts atomically.  Two chunks to a wave until the
        // launch has 256 of them, one up to 24 waves a block, four until it has 512 (with two, 94 chunks of each of 12 blocks, HMM of 64 x 96, B = 64,
        // took 18.2 us, now 15.1).  At most 64 waves a block: their adds meet on the same addresses.  Whole pairs dealt out / now: 16 x 32,
        // B = 32 6.1 / 6.1 us (two chunks a wave 7.5), B = 128 12.5 / 9.4, B = 512 37.5 / 15.7; 64 x 64, B = 64 10.9 / 12.7, B = 512 40.6 / 30.7;
        // 32 x 128, B = 32 8.8 / 9.4, B = 512 56 / 33; two blocks with 256 waves each 27, now 21.
        // From 128 blocks on the result has a fixed order: up to 255 blocks four waves of one workgroup to a block of four chunks and more
        // (132 blocks, HMM of 64 x 352, B = 128, one wave 267 us, three that add atomically 95, now 71; B = 32 71, 30, 21; 240 blocks, 4 x 480,
        // B = 128 18, 15, 7), then one.
        const int64_t avg_pairs = pf.n_pairs / pf.n_pb, chunks = avg_pairs * (Bs / 32);
        const bool ordered = avg_pairs >= 2 && chunks >= 4 && pf.n_pb >= 128 && pf.n_pb < 256;
        int n_split = ordered ? 4 : 1;
        if (avg_pairs >= 2 && pf.n_pb < 128) {
            const int64_t few = std::min(std::max(std::min<int64_t>(avg_pairs, 24), chunks / 2), (int64_t)256 / pf.n_pb);
            n_split = (int)std::max<int64_t>(1, std::min<int64_t>(std::max(few, std::min(chunks / 4, (int64_t)512 / pf.n_pb)), 64));
        }
        const unsigned wgs = (unsigned)(((int64_t)pf.n_pb * n_split + 3) / 4);
        const bool one = (int64_t)pf.n_pairs * (Bs / 32) < 12 * (int64_t)pf.n_pb * n_split;   // fewer than 12 chunks per wave on average
#define PC_PF_32(ONE, ORDERED) hipLaunchKernelGGL((k_param_flow_mfma<32, 1, 1, ONE, ORDERED>), dim3(wgs), dim3(256), 0, s, theta, l, R, N, nfmax, G, \
                                                  pf.pb, pf.ptr, pf.sum, pf.child, pf.n_pb, n_split, Bs)
        if (ordered && one) PC_PF_32(true, true);
        else if (ordered) PC_PF_32(false, true);
        else if (one) PC_PF_32(true, false);
        else PC_PF_32(false, false);
#undef PC_PF_32
    } else {
        // few blocks with many tied pairs each: the pairs are dealt to workgroups until the launch has some 256 of them; where that leaves
        // short reductions (below), their chunks, two or more to each.  Up to 512 workgroups with eight chunks each, or up to 32 a block with five
        // (K = 64: two): a workgroup's adds meet those of the block's others.  256 workgroups and pairs / now: HMM of 4 x 64, B = 512 36 / 7 us, 32 x 64
        // 39 / 14, 32 x 512, B = 77 42 / 31 (1024 workgroups 34), 64 x 128, B = 128 14.3 / 12.6 (84 of two chunks a block 17.4); K = 128 4 x 128, B = 128
        // 29 / 18, 16 x 512, B = 300 65 / 57, B = 128 33.5 / 29 (24 of two chunks 38), 64 x 256, B = 128 37 / 41 (84 of two chunks 57), 64 x 512, B = 1
        // 30 / 30 (25 of two 38).  128 blocks and more keep one each: a fixed order.
        int n_split = pf.n_pb >= 128 ? 1 : (int)std::max<int64_t>(1, std::min<int64_t>(pf.n_pairs / pf.n_pb, 256 / pf.n_pb));
        const int64_t chunks = pf.n_pairs * (Bs / 32) / pf.n_pb;
        if (n_split > 1 && chunks < 64 * n_split) {
            const int64_t half = std::min(chunks / 2, (int64_t)256 / pf.n_pb), few = std::min(chunks / (K == 64 ? 2 : 5), (int64_t)32);
            const int64_t most = std::min(128, 512 / pf.n_pb);
            n_split = (int)std::max<int64_t>(n_split, std::min(std::max({half, few, chunks / 8}), most));
        }
        // short reductions (fewer than 64 chunks per workgroup on average): the single-tile form
        const bool one = (int64_t)pf.n_pairs * (Bs / 32) < 64 * (int64_t)pf.n_pb * n_split;
#define PC_PF_WG(KK, ONE, BF)                                                                                       \
    hipLaunchKernelGGL((k_param_flow_mfma_wg<KK, ONE, BF>), dim3((unsigned)pf.n_pb * n_split), dim3(256), 0, s, theta, l, R, N, \
                       nfmax, G, pf.pb, pf.ptr, pf.sum, pf.child, n_split, Bs)
        // long reductions (128 chunks per workgroup or more: tied blocks of a large model): bf16-split products
        const bool bf = bf16_enabled() && (int64_t)pf.n_pairs * (Bs / 32) >= 128 * (int64_t)pf.n_pb * n_split;
        if (bf && !one && g_prof) g_prof->bf16_launches[KC_SUM_BWD_PARAM] += 1;
        if (K == 64 && one) PC_PF_WG(64, true, false);
        else if (K == 64 && bf) PC_PF_WG(64, false, true);
        else if (K == 64) PC_PF_WG(64, false, false);
        else if (one) PC_PF_WG(128, true, false);
        else if (bf) PC_PF_WG(128, false, true);
        else PC_PF_WG(128, false, false);
#undef PC_PF_WG
    }
}

// ---- bf16-split path for long dense reductions ----
// A layer takes the bf16 kernel when its rows are long (at least 2048 children: the fp32 kernel is bound by the matrix
// cores there) and the launch has a workgroup for every fourth CU at least.
bool sum_layer_takes_bf16(int32_t K, int32_t n_groups, int32_t n_rows, int32_t width, int64_t Bs)
{
    if (!bf16_enabled() || g_force_generic || (K != 64 && K != 128) || n_groups != 1) return false;
    return (int64_t)width * K >= 2048 && (int64_t)n_rows * (K / 64) * (Bs / 32) >= 128;
}

void launch_split_theta(const float *theta, int64_t n_blocks, int32_t K, bool transposed, void *Th, void *Tl, hipStream_t s)
{
    Timed timed(KC_SPLIT, s);
    const int64_t n_tiles = n_blocks * (K / 32) * (K / 16);
    const dim3 grid((unsigned)((n_tiles + 3) / 4));
    if (transposed) hipLaunchKernelGGL(k_split_theta<true>, grid, dim3(256), 0, s, theta, n_tiles, K, (uint4 *)Th, (uint4 *)Tl);
    else hipLaunchKernelGGL(k_split_theta<false>, grid, dim3(256), 0, s, theta, n_tiles, K, (uint4 *)Th, (uint4 *)Tl);
}

void launch_split_p(const float *X, const float *ref, const int32_t *blk_ids, int32_t n_blk, int32_t K, int64_t Bs, void *Ph,
                    void *Pl, hipStream_t s)
{
    if (n_blk == 0) return;
    Timed timed(KC_SPLIT, s);
    const int64_t items = (int64_t)n_blk * (K / 16) * (Bs / 32);
    hipLaunchKernelGGL(k_split_p, dim3((unsigned)((items + 3) / 4)), dim3(256), 0, s, X, ref, blk_ids, n_blk, K, Bs, (uint4 *)Ph,
                       (uint4 *)Pl);
}

void launch_sum_bf16(const void *Th, const void *Tl, const void *Ph, const void *Pl, float *l, float *R, const float *nfmax,
                     float *F, bool bwd, const GroupSet &gs, int32_t K, int64_t Bs, hipStream_t s)
{
    Timed timed(bwd ? KC_SUM_BWD_CHILD : KC_SUM_FWD, s);
    if (g_prof) g_prof->bf16_launches[bwd ? KC_SUM_BWD_CHILD : KC_SUM_FWD] += 1;
    // 64 x 64 tiles per wave (two thirds of the operand bytes per MFMA) where they still give every CU a workgroup;
    // PC_BF16_CT=1 / 2 forces one form (measurements)
    static const int force_ct = getenv("PC_BF16_CT") ? atoi(getenv("PC_BF16_CT")) : 0;
    const int64_t tiles64 = (int64_t)set_rows(gs) * (K / 64) * (Bs / 64);
    const bool wide = Bs % 64 == 0 && (force_ct ? force_ct == 2 : tiles64 >= 200);
    const dim3 grid((unsigned)(set_rows(gs) * (K / 64)), (unsigned)(Bs / (wide ? 64 : 32)));
#define PC_BF16_SUM(KK, BB)                                                                                            \
    do {                                                                                                               \
        if (wide) hipLaunchKernelGGL((k_sum_bf16<KK, 2, BB, 2>), grid, dim3(256), 0, s, (const uint4 *)Th, (const uint4 *)Tl, \
                                     (const uint4 *)Ph, (const uint4 *)Pl, l, R, nfmax, F, gs, Bs);                     \
        else hipLaunchKernelGGL((k_sum_bf16<KK, 2, BB, 1>), grid, dim3(256), 0, s, (const uint4 *)Th, (const uint4 *)Tl, \
                                (const uint4 *)Ph, (const uint4 *)Pl, l, R, nfmax, F, gs, Bs);                          \
    } while (0)
    if (K == 64) { if (bwd) PC_BF16_SUM(64, true); else PC_BF16_SUM(64, false); }
    else { if (bwd) PC_BF16_SUM(128, true); else PC_BF16_SUM(128, false); }
#undef PC_BF16_SUM
}

void launch_em(float *theta, float *tables, float *theta_flow, float *table_flow, const EmDev &em, int32_t K,
               int32_t n_tables, int32_t n_cats, float step, float pc, hipStream_t s)
{
    // one workgroup per table where it can hold the flows and there are enough tables, or too little data to share out
    const int64_t per_table = (int64_t)n_cats * K;
    const bool whole = K >= 4 && (K & (K - 1)) == 0 && per_table <= 65536 && (n_tables >= 64 || per_table <= 8192);
    // up to the workgroups the chip holds at once with the tables' registers: beyond, the launch is little beside the work
    const int32_t shares = (K + 3) / 4;
    if (whole && per_table <= 16384 && em.n_seg == 0 && (K & 3) == 0 && em.avg_list * (K / 4) <= 64 && n_tables + (int64_t)em.n_all * shares <= 1024) {
        Timed timed(KC_EM, s);
        hipLaunchKernelGGL((k_em_tables_whole<256, true>), dim3((unsigned)(n_tables + em.n_all * shares)), dim3(256), 0, s, tables, table_flow, K, n_cats, step,
                           pc, n_tables, theta, theta_flow, em, shares);
        return;
    }
    {
        Timed timed(KC_EM, s);
        // up to four rows per wave, fewer where that leaves less than eight waves per SIMD; registers for the average row
        const bool v4 = (K & 3) == 0;
        const int waves = std::min(4, K), tot = em.avg_list * (v4 ? K / 4 : K);
        const int rpw = (int)std::max<int64_t>(1, std::min<int64_t>(4, (int64_t)em.n_all * K / 8192));
        const dim3 grid((unsigned)em.n_all, (unsigned)((K + rpw * waves - 1) / (rpw * waves))), blk((unsigned)(64 * waves));
#define PC_EM_THETA(V, NR)                                                                                                \
    hipLaunchKernelGGL((k_em_theta<V, NR, false>), grid, blk, 0, s, theta, theta_flow, em.ptr, em.list, em.pb_rows, em.pb_cols, \
                       em.group_nch, em.n_groups, nullptr, nullptr, K, step, pc)
        if (v4) {
            if (tot <= 64) PC_EM_THETA(4, 1);
            else if (tot <= 256) PC_EM_THETA(4, 4);
            else PC_EM_THETA(4, 16);
        } else {
            if (tot <= 64) PC_EM_THETA(1, 1);
            else PC_EM_THETA(1, 16);
        }
#undef PC_EM_THETA
        if (em.n_seg > 0) {
            const dim3 sgrid((unsigned)em.n_seg, (unsigned)((K + waves - 1) / waves));
#define PC_EM_SEG(V)                                                                                                      \
    do {                                                                                                                  \
        hipLaunchKernelGGL((k_em_row_sums<V>), sgrid, blk, 0, s, theta_flow, em.seg_ptr, em.list, em.pb_rows, em.pb_cols, K, em.part); \
        hipLaunchKernelGGL((k_em_theta<V, 4, true>), sgrid, blk, 0, s, theta, theta_flow, em.seg_ptr, em.list, em.pb_rows, em.pb_cols, \
                           nullptr, em.n_seg, em.seg, em.part, K, step, pc);                                              \
    } while (0)
            if (v4) PC_EM_SEG(4);
            else PC_EM_SEG(1);
#undef PC_EM_SEG
        }
    }
    if (whole) {
        Timed timed(KC_EM, s);
        const dim3 grid((unsigned)n_tables);
#define PC_EM_WHOLE(NN) \
    hipLaunchKernelGGL((k_em_tables_whole<NN, false>), grid, dim3(NN), 0, s, tables, table_flow, K, n_cats, step, pc, n_tables, nullptr, nullptr, em, 0)
        if (per_table <= 16384) PC_EM_WHOLE(256);
        else if (per_table <= 32768) PC_EM_WHOLE(512);
        else PC_EM_WHOLE(1024);
#undef PC_EM_WHOLE
        return;
    }
    launch_fill(em.ztab, (int64_t)n_tables * K, 0.0f, s);
    Timed timed(KC_EM, s);
    if ((K & 3) == 0) {                                                // 16-byte accesses
        const int rows_per_pass = 256 / (K / 4);
        // about 2048 workgroups when the tables are few, at least four loads per thread
        const int64_t max_slabs = std::max<int64_t>(1, n_cats / (4 * rows_per_pass));
        const int64_t slabs = std::min<int64_t>(max_slabs, std::max<int64_t>(1, 2048 / n_tables));
        const int cats_per_block = (int)((n_cats + slabs - 1) / slabs);
        dim3 grid((unsigned)n_tables, (unsigned)((n_cats + cats_per_block - 1) / cats_per_block));
        hipLaunchKernelGGL(k_em_tabsum_v4, grid, dim3(256), 0, s, table_flow, K, n_cats, cats_per_block, em.ztab);
        // enough workgroups per table to fill the chip when there are few tables, one pass otherwise
        const int per_table = (int)std::min<int64_t>((n_cats + rows_per_pass - 1) / rows_per_pass,
                                                     std::max<int64_t>(1, 4096 / n_tables));
        hipLaunchKernelGGL(k_em_tables_v4, dim3((unsigned)n_tables, (unsigned)per_table), dim3(256), 0, s, tables, table_flow,
                           em.ztab, K, n_cats, step, pc);
    } else {
        const int cats_per_block = 64;
        dim3 grid((unsigned)n_tables, (unsigned)((n_cats + cats_per_block - 1) / cats_per_block));
        hipLaunchKernelGGL(k_em_tabsum, grid, dim3(256), 0, s, table_flow, K, n_cats, cats_per_block, em.ztab);
        const int64_t total = (int64_t)n_tables * n_cats * K;
        hipLaunchKernelGGL(k_em_tables, dim3(grid_for(total)), dim3(256), 0, s, tables, table_flow, em.ztab, K, n_cats, total,
                           step, pc);
    }
}

}  // namespace pc
