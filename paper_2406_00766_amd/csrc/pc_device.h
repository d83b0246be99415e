// Constants and device helpers shared by the kernel files (internal).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace pc {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

#define PC_NEG_INF (-__builtin_inff())
#define PC_LOG2E 1.4426950408889634f
// Sum-layer terms are theta * exp(value - running maximum + PC_UP).  The maximum is taken over the values alone (as in
// Alg. 1 / Alg. 4), so without the upward shift a term with a large weight whose value lies 87 nats below that of a
// child with a weight near FLT_MIN would be flushed to zero although it dominates the sum.  With it every term or
// factor that underflows is at least e^-20 smaller than the largest term kept, and nothing can overflow.  The shift
// is kept small because the result is  maximum - PC_UP + log(sum): the larger the two cancelling parts, the larger
// the absolute rounding error of a log-probability near zero.
#define PC_UP 20.0f
// Rescaling an accumulator when the running maximum grows by -delta: the factor exp(delta) itself may leave the
// fp32 range where accumulator * factor does not (the accumulator can be as large as e^28 times the term count),
// so the factor is applied as two multiplications by exp(delta / 2); below delta = -174 the result is nil anyway.
__device__ inline float pc_half_scale(float delta) { return __expf(0.5f * fmaxf(delta, -174.0f)); }

// buffer descriptors: raw (stride 0), 2 GiB window from the base, 32-bit data format
#define PC_BUF_RANGE 0x7fffffff
#define PC_BUF_FLAGS 0x00020000

// Category of variable v in sample b: -1 if marginalised (mask, or a padding column b >= B), -2 if out of range.
__device__ inline int32_t pc_category(const int32_t *x, const uint8_t *mask, int64_t b, int32_t v, int32_t B, int32_t D, int32_t n_cats)
{
    if (b >= B) return -1;
    const int64_t at = b * D + v;
    const int32_t c = x[at];
    if (mask && mask[at]) return -1;
    return c < 0 || c >= n_cats ? -2 : c;
}

// Which tile of the input layer a workgroup takes: of the first n_by_xcd blocks (a multiple of eight, input_by_xcd) those of a block one after
// another on one XCD (workgroup h runs on XCD h mod 8), of the others the tiles of all XCDs in turn.
struct InputTile { int block, col; };
__device__ inline InputTile input_tile_at(int h, int n_rows, int n_by_xcd, int n_ct)
{
    const int q = h >> 3, rest = h - n_by_xcd * n_ct, others = n_rows - n_by_xcd;
    return rest < 0 ? InputTile{q / n_ct * 8 + (h & 7), q % n_ct} : InputTile{n_by_xcd + rest % others, rest / others};
}

// Input layer through an LDS tile, for K a multiple of 4: one workgroup per (block u, COLS samples).  K / 4 lanes fetch one
// sample's table row with 16-byte loads (every global read is a whole contiguous row), the logs go into a
// [K x COLS] tile, and the tile leaves as 16-byte stores along the batch -- no access is narrower than a row.
// KC: the block size at compile time, 0 any multiple of 4; COLS columns per workgroup.  Bound: the chain of a workgroup -- block, categories,
// table rows, stores --, of which a CU holds eight; a thread's table rows are requested together, and wide tiles carry more per chain.
// One row after the other / together / 128 columns, K = 32: RAT-SPN of 784 variables, B = 512 577 / 553 / 496 us, PD of 1024
// variables, B = 256 93 / 89 / 85; launches of a few thousand workgroups lose with wide tiles (RAT-SPN of 784, B = 16 52 -> 56), 256 columns do
// (641), and so does K = 64 with 128 (784-variable tree, B = 512 68 -> 82): the tiles leave room for fewer workgroups.
// Direct: the categories are read from x (and mask) itself, not from its transpose xT.
template <int KC, int COLS, bool DIRECT>
__device__ inline void input_tile(float *smem, int u, int64_t b0, const float *__restrict__ tables, const int32_t *__restrict__ x,
                                  const uint8_t *__restrict__ mask, int32_t B, int32_t D, const int32_t *__restrict__ ids,
                                  const int32_t *__restrict__ var, const int32_t *__restrict__ tab, int32_t K_, int32_t n_cats, int64_t Bs,
                                  float *__restrict__ l, float *__restrict__ R)
{
    constexpr int LD = COLS + 1, N = KC ? COLS * KC / 1024 : 1, C4 = COLS / 4;
    const int K = KC ? KC : K_;
    float *tile = smem;                                                 // [K][LD]
    int *cats = reinterpret_cast<int *>(tile + K * LD);
    if (threadIdx.x < COLS) {
        const int64_t b = b0 + threadIdx.x;
        cats[threadIdx.x] = DIRECT ? pc_category(x, mask, b, var[u], B, D, n_cats) : b < Bs ? x[(int64_t)var[u] * Bs + b] : -1;
    }
    __syncthreads();
    const int lps = K / 4;                                              // lanes per sample
    const float *tbase = tables + (int64_t)tab[u] * n_cats * K;
    for (int idx0 = threadIdx.x; idx0 < COLS * lps; idx0 += 256 * N) {
        float4 r[N];
        int xv[N];
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int idx = idx0 + 256 * n, sidx = idx / lps, kl = idx - sidx * lps;
            xv[n] = cats[sidx];
            r[n] = xv[n] >= 0 ? *reinterpret_cast<const float4 *>(tbase + (int64_t)xv[n] * K + kl * 4) : make_float4(1.f, 1.f, 1.f, 1.f);
        }
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int idx = idx0 + 256 * n, sidx = idx / lps, kl = idx - sidx * lps;
            float4 t = make_float4(__logf(r[n].x), __logf(r[n].y), __logf(r[n].z), __logf(r[n].w));
            if (xv[n] < 0) {
                const float v = xv[n] == -1 ? 0.0f : PC_NEG_INF;        // marginalised / tail : out-of-range category
                t = make_float4(v, v, v, v);
            }
            float *dst = tile + (kl * 4) * LD + sidx;
            dst[0] = t.x; dst[LD] = t.y; dst[2 * LD] = t.z; dst[3 * LD] = t.w;
        }
    }
    __syncthreads();
    const int32_t id = ids[u];
    if (threadIdx.x < COLS && b0 + threadIdx.x < Bs) R[(int64_t)(id / K) * Bs + b0 + threadIdx.x] = 0.0f;   // an input block's reference
    for (int idx = threadIdx.x; idx < K * C4; idx += 256) {
        const int row = idx / C4, c4 = (idx % C4) * 4;
        if (b0 + c4 < Bs) {
            const float *src = tile + row * LD + c4;
            *reinterpret_cast<float4 *>(l + (int64_t)(id + row) * Bs + b0 + c4) = make_float4(src[0], src[1], src[2], src[3]);
        }
    }
}

}  // namespace pc
