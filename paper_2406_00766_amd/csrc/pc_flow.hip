// Dataflow sum layers: every sum layer from a given layer to the root in ONE launch per direction.
//
// A layer of a deep narrow circuit is a few microseconds of latency: a launch, a table row, the operands, the result.
// Launched one by one the layers of a 784-variable tree cost 83 x (product + sum) launches of 5 us each per direction
// while the chip idles.  Here a layer's tiles are TASKS of one launch.  A task is (sum or product block, tile of 16 RT of
// its rows, tile of 16 NC columns); workgroups take tasks by a ticket counter, in layer order, and a task that needs
// values of an earlier task reads them straight from the result buffer until they are there:
//   * the rows a task publishes are filled with a sentinel (a NaN bit pattern no result has) before the launch; a consumer
//     loads the values it needs with device-scope loads and repeats the load while any of them is the sentinel.  Data and
//     signal are one word, so a hand-over costs one store and one load -- 0.5 - 0.7 us between workgroups (measured) where a kernel
//     boundary costs that of the launch and the consumer's cold start, which here is over before the values arrive: a
//     waiting workgroup holds its weights in registers already.
//   * no wait can last for ever: a task waits only for tasks with lower tickets, tickets are taken by running workgroups
//     in increasing order and worked off in that order, so the lowest unfinished task never waits.  (No assumption about
//     how many workgroups are resident.)  A bound on the polls ends the launch all the same should that ever be untrue: the
//     task that gave up publishes NaN, its readers pass NaN on, and the host is told through a word in its memory.
//
// Forward (role of Alg. 1): a task computes 16 RT sum nodes.  Its neighbours' values are the PRODUCTS of their children's
// log-probabilities, formed here from the children's rows (Sec. 3: a sum of log-probabilities), so a product layer is
// not on the path from layer to layer at all; the product blocks' own rows are written by one ordinary launch after this
// one (k_prod_fwd over all layers).  Backward (role of Alg. 4): a task computes 16 RT product nodes' flows; log_nf of its
// parents (sum blocks) is formed here from their own parents' flows, and F, log_nf of the sum and input blocks are written
// by one launch of k_prod_bwd afterwards.
//
// Arithmetic: v_mfma_f32_16x16x4_f32.  A (16 x 4): lane holds A[lane % 16][lane / 16]; B (4 x 16): lane holds
// B[lane / 16][lane % 16]; D: register r holds D[4 * (lane / 16) + r][lane % 16].  Reduction in chunks of 32 neighbour
// nodes, step (c2, e) pairs lane group g with node 16 c2 + 4 g + e, so that the forward weights are 16-byte loads.  The W
// waves of a workgroup split the chunks and meet in LDS once.  A chunk's values are brought to an integer reference (the
// rounded column maximum joins R), so every exponential sees an argument <= 0.5 and results need no running maximum.
//
// What bounds it: the chain through the layers.  Measured (time stamps of the tasks of one layer): values seen 0.5 - 0.7 us
// after they were published, 0.4 - 0.5 us to exponentials and MFMAs (up to 128 neighbour nodes; at 512, 1 us: the waves of a CU
// share its matrix cores), 0.2 - 0.5 us to merge and publish: 1.3 us at 32 nodes, 1.5 at 128, 2.2 at 512.  Launch time over layers:
// 1.4 us at 32 nodes (HMM 16 x 32), 3.5 us on a 784-variable tree with M = 128, B = 512, 4.6 us at 512 (HMM 32 x 512), against
// 7 - 13 us for a layer's two launches; what the stamps do not account for is not attributed (products that wait for several
// children in turn; polls that read every operand of the wave again).  Before -> now, whole passes: forward, HMM T = 16, H = 32, one sample 137 -> 29 us; forward,
// 784-variable tree, M = 128, B = 100 908 -> 350 us; forward + backward, the same tree at B = 512 2.70 -> 1.69 ms; HMM T = 32, H = 512,
// B = 77 865 -> 390 us.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pc_device.h"
#include "pc_kernels.h"

namespace pc {

#define PC_SENTINEL 0xFFFFFFFFu

// Device-scope 4- and 16-byte accesses (sc1); every dword of a 16-byte access is a word of its own.  (A polling loop needs a
// compiler barrier so that it loads again; a volatile access would be system-scope.)
#define PC_AUX_DEVICE 16
__device__ inline floatx4 mail_load(const float *tile, int voff)
{
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)tile, 0, PC_BUF_RANGE, PC_BUF_FLAGS);
    return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, PC_AUX_DEVICE));
}
__device__ inline float flow_load(const float *p)
{
    return __builtin_bit_cast(float, __hip_atomic_load(reinterpret_cast<const uint32_t *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
// maximum over the four lane groups of a column (lanes j, j + 16, j + 32, j + 48)
__device__ inline float max_over_groups(float v)
{
    // (as instructions: of the builtins' two results the compiler keeps one when the operands are equal)
    float a = v, b = v;
    asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    a = b = fmaxf(a, b);
    asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    return fmaxf(a, b);
}
__device__ inline bool is_sentinel(float v) { return __builtin_bit_cast(uint32_t, v) == PC_SENTINEL; }
__device__ inline float no_sentinel(float v) { return v == v ? v : __builtin_bit_cast(float, 0x7FC00000u); }   // one NaN for all

__device__ inline bool flow_give_up(int spin, int wait_limit, int32_t *ticket, int32_t *fault)
{
    if (spin < wait_limit && ((spin & 1023) != 1023 || __hip_atomic_load(ticket + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)) return false;
    __hip_atomic_store(ticket + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(fault, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return true;
}

// Fills before a dataflow launch: a block's K rows (contiguous, K Bs values) are dealt to workgroups in shares of PC_FILL_SHARE
// values, and with them its row of R or nothing.  fill_shares: of one block.
#define PC_FILL_SHARE 4096
static __host__ __device__ inline int fill_shares(int32_t K, int64_t Bs) { return (int)((K * Bs + PC_FILL_SHARE - 1) / PC_FILL_SHARE); }
__device__ inline void fill_share(float *X, float *Y, float *R, int32_t id, int share, int32_t K, int64_t Bs, float value)
{
    const floatx4 v = {value, value, value, value};
#pragma unroll
    for (int k = 0; k < PC_FILL_SHARE; k += 1024) {
        const int64_t i = (int64_t)share * PC_FILL_SHARE + k + 4 * threadIdx.x;   // K Bs, Bs and the share are multiples of 32
        if (i < K * Bs) {
            *reinterpret_cast<floatx4 *>(X + (int64_t)id * Bs + i) = v;
            if (Y) *reinterpret_cast<floatx4 *>(Y + (int64_t)id * Bs + i) = v;
        }
        if (R && i < Bs) *reinterpret_cast<floatx4 *>(R + (int64_t)(id / K) * Bs + i) = v;
    }
}

// Start of a forward pass in one launch: x -> xT (see below), the sentinels of the sum blocks the dataflow launch will publish,
// the null block's rows (l = 0, R = 0; mail = 0 where a direction has a dataflow launch) and the ticket words.  One workgroup per block
// takes longer than the rest of the launch at a large batch: the null block alone, forward pass of a 3 x 32 HMM at B = 131072, 561 us
// instead of 88; the published ones, this launch for a 16 x 128 HMM in blocks of 128 at B = 4096, 23 us instead of 16.
// xT[v][b] = category, -1 if marginalised (mask, or padding column b >= B), -2 if out of range.
__global__ __launch_bounds__(256) void k_begin_forward(const int32_t *__restrict__ x, const uint8_t *__restrict__ mask, int32_t B,
                                                       int32_t D, int64_t Bs, int32_t n_cats, int32_t *__restrict__ xT, int32_t n_xb,
                                                       int32_t n_xtiles, float *__restrict__ l, float *__restrict__ R,
                                                       float *__restrict__ mail, bool null_mail, const int32_t *__restrict__ ent,
                                                       int32_t n_ent, int32_t K, int32_t *ticket)
{
    __shared__ int32_t tile[32][33];
    if ((int)blockIdx.x >= n_xtiles) {
        const int q = (int)blockIdx.x - n_xtiles;
        const int n_sh = fill_shares(K, Bs), b = q / n_sh, share = q % n_sh;
        if (b < n_ent) fill_share(mail, nullptr, R, ent[4 * b], share, K, Bs, __builtin_bit_cast(float, PC_SENTINEL));
        else fill_share(l, null_mail ? mail : nullptr, R, 0, share, K, Bs, 0.0f);
        if (q == 0 && threadIdx.x < 2) ticket[threadIdx.x] = 0;
        return;
    }
    const int b0 = ((int)blockIdx.x % n_xb) * 32, v0 = ((int)blockIdx.x / n_xb) * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;           // 256 threads: ty in 0..7
    for (int r = ty; r < 32; r += 8) {
        const int b = b0 + r, v = v0 + tx;
        int32_t val = -1;
        if (b < B && v < D) {
            const int64_t idx = (int64_t)b * D + v;
            val = x[idx];
            if (val < 0 || val >= n_cats) val = -2;
            if (mask && mask[idx]) val = -1;
        }
        tile[r][tx] = val;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        const int v = v0 + r, b = b0 + tx;
        if (v < D && b < Bs) xT[(int64_t)v * Bs + b] = tile[tx][r];
    }
}

// Start of a backward pass in one launch.  Workgroups < n_init * n_cb: blocks without parents, which no layer of the sweep
// writes.  An entry >= 0 is a sum block: the root (flow 1 on node 0 of real samples with non-zero probability, Def. 2) or a
// sum block nobody uses (flow 0); its log_nf rows and block maximum are set as well.  An entry < 0 is ~offset of another
// block (the null block, a product or input block nobody uses): its flow rows are zeroed.  One workgroup per entry and 256
// columns.  Workgroups behind them: the sentinels of the product blocks the dataflow launch will publish, its tickets.
__global__ __launch_bounds__(256) void k_begin_backward(const float *__restrict__ l, float *__restrict__ F, float *__restrict__ N,
                                                        float *__restrict__ nfmax, const int32_t *__restrict__ blk_ids, int32_t n_init,
                                                        int32_t n_cb, int32_t root_id, int32_t K, int64_t Bs, int32_t B,
                                                        const int32_t *__restrict__ ent, int32_t n_ent, int32_t *ticket)
{
    if ((int)blockIdx.x >= n_init * n_cb) {
        const int q = (int)blockIdx.x - n_init * n_cb;
        const int n_sh = fill_shares(K, Bs);
        if (q < n_ent * n_sh) fill_share(N, nullptr, nullptr, ent[4 * (q / n_sh)], q % n_sh, K, Bs, __builtin_bit_cast(float, PC_SENTINEL));
        else if (threadIdx.x < 2) ticket[threadIdx.x] = 0;
        return;
    }
    const int32_t entry = blk_ids[blockIdx.x / n_cb];
    const int64_t b = (int64_t)(blockIdx.x % n_cb) * 256 + threadIdx.x;
    if (b >= Bs) return;
    if (entry < 0) {
        const int32_t id = ~entry;
        for (int k = 0; k < K; ++k) F[(int64_t)(id + k) * Bs + b] = 0.0f;
        return;
    }
    const int32_t id = entry;
    float top = PC_NEG_INF, f0 = 0.0f;
    if (id == root_id) {
        const float lv = l[(int64_t)id * Bs + b];
        const bool live = b < B && lv > PC_NEG_INF;
        f0 = live ? 1.0f : 0.0f;
        top = live ? -lv : PC_NEG_INF;
    }
    for (int k = 0; k < K; ++k) {
        F[(int64_t)(id + k) * Bs + b] = k == 0 ? f0 : 0.0f;
        N[(int64_t)(id + k) * Bs + b] = k == 0 ? top : PC_NEG_INF;
    }
    nfmax[(int64_t)(id / K) * Bs + b] = top;
}

// Tables (built by compile_flow):
//   ent  4 words per task block, in task order: node offset, first neighbour record, neighbour records, 1 for the root
//   rec  16 words per neighbour: parameter offset; start of its list; list items; neighbour's node offset; its layer; the first
//        five items and then their layers.  A list holds items (node offset, layer); an item of layer li0 or above is waited for.
//        Forward: the neighbour is a product block, the list its children; a neighbour below layer li0 has been evaluated
//        already and stands for itself.  Backward: the neighbour is a sum block, the list its product parents, or itself
//        (layer -1) where it has none.
// `mail` (the rows of log_nf that are not in use at the time: sum rows forward, product rows backward) carries the published
// values in MFMA operand order: per block, 16 rows and 16 columns one 1 KiB tile, lane (j, g) holding rows 4 g .. 4 g + 3 of
// column j -- one 16-byte load per lane where the row-major buffer would take four loads of 4 x 64 bytes, and no line shared
// by two column tiles.
template <int W, int RT, int NCH, bool BWD, bool EXACT>
__global__ __launch_bounds__(64 * W, W >= 8 ? 1 : 2) void k_flow(const float *__restrict__ theta, float *__restrict__ l, float *R,
                                                                 float *__restrict__ F, float *mail,
                                                                 const int32_t *__restrict__ ent, const int32_t *__restrict__ rec,
                                                                 const int32_t *__restrict__ list, int32_t n_tasks, int32_t n_ct,
                                                                 int32_t K, int64_t Bs, int32_t li0, int32_t *ticket,
                                                                 float *__restrict__ ll, int32_t B, int32_t wait_limit,
                                                                 int32_t *fault)
{
    constexpr int TPW = (RT + W - 1) / W;                               // 16 x 16 result tiles that a wave writes
    __shared__ floatx4 part[2][W][RT][W > 1 ? 64 : 1];                              // partial sums of the waves, double-buffered over tasks
    __shared__ float pref[2][W][16];                                    // and their references
    __shared__ int32_t s_ticket[2];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, g = lane >> 4, j16 = lane & 15;
    const int ks = 31 - __builtin_clz(K);                               // K is 32, 64 or 128
    const int TM = 16 * RT, subs = K / TM, cpb = K >> 5;

    struct Task { int32_t ct, sub, row0, rec0, root, C; };              // C: chunks of 32 neighbour nodes
    auto decode = [&](int t) -> Task {
        if (t >= n_tasks) return Task{0, 0, 0, 0, 0, 0};
        const int q = t / n_ct, e = 4 * (q / subs);
        return Task{t % n_ct, q % subs, ent[e], ent[e + 1], ent[e + 3], ent[e + 2] * cpb};
    };

    // operands of this wave's chunks cb, cb + W, ... (NCH of them; past the end the first one again, given the value -inf)
    floatx4 th[NCH][2][RT], v[NCH][2], own_l[BWD ? NCH : 1][2];
    float base[NCH];
    int32_t koff[NCH], own[NCH], cnt[NCH];
    const int32_t *rp[NCH];
    // item n of chunk i if it is (wait) / is not (!wait) one to wait for, else the null block (value 0); any: there is one
    auto item = [&](int i, int n, bool wait, int &any) -> int32_t {
        if (cnt[i] < 0) { if (n == 0 && !wait) { any = 1; return own[i]; } return 0; }
        if (n >= cnt[i]) return 0;
        int32_t it, lay;
        if (n < 5) { it = rp[i][5 + n]; lay = rp[i][10 + n]; }
        else { it = list[2 * (rp[i][1] + n)]; lay = list[2 * (rp[i][1] + n) + 1]; }
        if ((lay >= li0) != wait) return 0;
        any = 1;
        return it;
    };
    auto row_values = [&](const float *X, int32_t id, int i, int64_t col, floatx4 (&x)[2]) {
        const float *src = X + (int64_t)(id + koff[i] + 4 * g) * Bs + col;
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k >> 2][k & 3] = src[(int64_t)(16 * (k >> 2) + (k & 3)) * Bs];
    };
    auto request = [&](const Task &T, int cb) {
        const int64_t col = (int64_t)T.ct * 16 + j16;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int cc = cb + W * i < T.C ? cb + W * i : cb;
            const int32_t *r = rec + 16 * (int64_t)(T.rec0 + cc / cpb);
            rp[i] = r;
            koff[i] = (cc % cpb) * 32;
            cnt[i] = r[2]; own[i] = r[3];
            if (!BWD && r[4] < li0) cnt[i] = -1;                        // evaluated before this launch
            const float *tb = theta + r[0] + (BWD ? koff[i] * K + T.sub * TM : T.sub * TM * K + koff[i]);
#pragma unroll
            for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    if (BWD) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) th[i][c2][rt][e] = tb[(16 * c2 + 4 * g + e) * K + rt * 16 + j16];
                    } else {
                        th[i][c2][rt] = *reinterpret_cast<const floatx4 *>(tb + (rt * 16 + j16) * K + 16 * c2 + 4 * g);
                    }
                }
            // the first item if it is there already (else zeros from the null block); backward: the sum block's own rows
            int any = 0;
            const int32_t it = item(i, 0, false, any);
            row_values(BWD ? F : l, it, i, col, v[i]);
            if (BWD) row_values(l, own[i], i, col, own_l[i]);
            base[i] = R[(int64_t)((BWD ? own[i] : it) >> ks) * Bs + col];
        }
    };

    int nxt = 0;
    if (threadIdx.x == 0) nxt = atomicAdd(ticket, 1);
    if (W > 1) {
        if (threadIdx.x == 0) s_ticket[1] = nxt;
        __syncthreads();
    }
    int t = __builtin_amdgcn_readfirstlane(W > 1 ? s_ticket[1] : nxt);
    for (int buf = 0; t < n_tasks; buf ^= 1) {
        if (threadIdx.x == 0) nxt = atomicAdd(ticket, 1);               // arrives while this task is worked on
        const Task T = decode(t);
        if (wave < T.C) request(T, wave);
        const int64_t col = (int64_t)T.ct * 16 + j16;

        float lown[TPW][4], Rrow = 0.0f;                                // backward: the rows' own log-probabilities, R of their block
        if (BWD) {
#pragma unroll
            for (int k = 0; k < TPW; ++k) {
                const int rt = wave + W * k < RT ? wave + W * k : 0;
#pragma unroll
                for (int r = 0; r < 4; ++r) lown[k][r] = l[(int64_t)(T.row0 + T.sub * TM + rt * 16 + 4 * g + r) * Bs + col];
            }
            Rrow = R[(int64_t)(T.row0 >> ks) * Bs + col];
        }

        floatx4 acc[RT];
        float ref = PC_NEG_INF;                                         // reference of acc; -inf: nothing live yet
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt] = floatx4{0.f, 0.f, 0.f, 0.f};

        for (int cb = wave; cb < T.C;) {
            // Values: the sum of the list items' rows (forward: log-probabilities; backward: flows).  One item of every chunk's
            // list at a time, the null block past its end: a branch around a load makes the compiler wait for all before it.
            int max_cnt = 0, since = 0;
#pragma unroll
            for (int i = 0; i < NCH; ++i) {
                max_cnt = max(max_cnt, cnt[i]);
                if (BWD) base[i] = Rrow - base[i];
            }
            // A running fp32 sum of several log-probabilities loses more than the flows' tolerance allows, so every four items its
            // integer part moves into the reference (exactly: no value lies above the column's maximum).  EXACT (launches with
            // products of more than eight children, which the product kernels sum in double): the rounding error of every
            // addition is kept beside the sum (Knuth's two-sum) and added once the integer part is out.  Products of 12 children
            // of -80 nats: largest error of the sum layer above 6.7e-5 -> 1.0e-6.  An instantiation of its own, as carrying it in
            // every launch cost 1 - 5 % of a pass (HMM 16 x 32, one sample 29.1 -> 30.5 us), and in it the tasks that have such a
            // product (3072-variable tree, forward 2.71 -> 2.66 ms against all tasks).
            floatx4 low[EXACT ? NCH : 1][2];
            if (EXACT) {
#pragma unroll
                for (int i = 0; i < NCH; ++i) low[i][0] = low[i][1] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
            auto settle = [&]() {
#pragma unroll
                for (int i = 0; i < NCH; ++i) {
                    float cm = v[i][0][0];
#pragma unroll
                    for (int k = 1; k < 8; ++k) cm = fmaxf(cm, v[i][k >> 2][k & 3]);
                    cm = max_over_groups(cm);
                    cm = cm > PC_NEG_INF ? rintf(cm) : 0.0f;
                    base[i] += cm;
#pragma unroll
                    for (int k = 0; k < 8; ++k) v[i][k >> 2][k & 3] -= cm;
                }
            };
            const bool exact = EXACT && max_cnt > 8;                    // wave-uniform: this task has such a product
            auto add_item = [&](const floatx4 (&x)[NCH][2], const float (&xr)[NCH]) {
                if (exact) {
#pragma unroll
                    for (int i = 0; i < NCH; ++i)
#pragma unroll
                        for (int k = 0; k < 8; ++k) {
                            const float a = v[i][k >> 2][k & 3], y = x[i][k >> 2][k & 3], s = a + y, t = s - a;
                            low[EXACT ? i : 0][k >> 2][k & 3] += (a - (s - t)) + (y - t);   // NaN where s = -inf: not used then
                        }
                }
#pragma unroll
                for (int i = 0; i < NCH; ++i) {
#pragma unroll
                    for (int k = 0; k < 8; ++k) v[i][k >> 2][k & 3] += x[i][k >> 2][k & 3];
                    if (!BWD) base[i] += xr[i];
                }
                if (!BWD && !exact && (++since & 3) == 3) settle();
            };
            for (int n = 1; n < max_cnt; ++n) {                         // items of earlier launches (the first: requested before)
                int32_t its[NCH];
                int any = 0;
#pragma unroll
                for (int i = 0; i < NCH; ++i) its[i] = item(i, n, false, any);
                if (!any) continue;
                floatx4 x[NCH][2];
                float xr[NCH];
#pragma unroll
                for (int i = 0; i < NCH; ++i) {
                    row_values(BWD ? F : l, its[i], i, col, x[i]);
                    if (!BWD) xr[i] = R[(int64_t)(its[i] >> ks) * Bs + col];
                }
                add_item(x, xr);
            }
            for (int n = 0; n < max_cnt; ++n) {                         // items of this launch: poll until they are there
                int32_t its[NCH];
                int any = 0;
#pragma unroll
                for (int i = 0; i < NCH; ++i) its[i] = item(i, n, true, any);
                if (!any) continue;
                floatx4 x[NCH][2];
                float xr[NCH];
                for (int spin = 0;; ++spin) {
                    asm volatile("" ::: "memory");
                    int missing = 0;
#pragma unroll
                    for (int i = 0; i < NCH; ++i) {
                        const float *src = mail + (int64_t)(its[i] + koff[i]) * Bs + (int64_t)T.ct * 256;
                        x[i][0] = mail_load(src, 16 * lane);
                        x[i][1] = mail_load(src + 16 * Bs, 16 * lane);
                        if (!BWD) xr[i] = flow_load(R + (int64_t)(its[i] >> ks) * Bs + col);
                    }
#pragma unroll
                    for (int i = 0; i < NCH; ++i) {
#pragma unroll
                        for (int k = 0; k < 8; ++k) missing |= is_sentinel(x[i][k >> 2][k & 3]);
                        if (!BWD) missing |= is_sentinel(xr[i]);
                    }
                    if (!__any(missing)) break;
                    if (flow_give_up(spin, wait_limit, ticket, fault)) {    // NaN in all its results (a factor 0 below keeps it)
#pragma unroll
                        for (int i = 0; i < NCH; ++i)
#pragma unroll
                            for (int k = 0; k < 8; ++k) x[i][k >> 2][k & 3] = __builtin_nanf("");
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
                add_item(x, xr);
            }
            if (exact) {
                settle();
#pragma unroll
                for (int i = 0; i < NCH; ++i)
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const float a = v[i][k >> 2][k & 3];
                        v[i][k >> 2][k & 3] = a > PC_NEG_INF ? a + low[EXACT ? i : 0][k >> 2][k & 3] : a;
                    }
            }
            // log_nf of the parents; integer reference of each chunk; the largest live one
            float nref = ref;
#pragma unroll
            for (int i = 0; i < NCH; ++i) {
                float cm = PC_NEG_INF;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    float x = v[i][k >> 2][k & 3];
                    if (BWD) {
                        const float lo = own_l[i][k >> 2][k & 3];
                        x = lo > PC_NEG_INF ? __logf(x) - lo : PC_NEG_INF;   // flow 0: -inf; NaN (a wait given up) stays NaN
                    }
                    if (cb + W * i >= T.C) x = PC_NEG_INF;
                    v[i][k >> 2][k & 3] = x;
                    cm = fmaxf(cm, x);
                }
                cm = max_over_groups(cm);
                const bool live = cm > PC_NEG_INF;
                cm = live ? rintf(cm) : 0.0f;
#pragma unroll
                for (int k = 0; k < 8; ++k) v[i][k >> 2][k & 3] -= cm;
                base[i] = live ? base[i] + cm : PC_NEG_INF;
                nref = fmaxf(nref, base[i]);
            }
            if (cb != wave) {                                           // not the first batch: rescale
                const float sc = nref > PC_NEG_INF ? pc_half_scale(ref - nref) : 1.0f;
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[rt][r] = acc[rt][r] * sc * sc;
            }
            ref = nref;
#pragma unroll
            for (int i = 0; i < NCH; ++i) {
                // exp(v + base - ref + PC_UP) = exp2(v * log2e + sh2); dead: v = -inf
                const float sh2 = base[i] > PC_NEG_INF ? (base[i] - ref + PC_UP) * PC_LOG2E : 0.0f;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const float p = __builtin_amdgcn_exp2f(fmaf(v[i][k >> 2][k & 3], PC_LOG2E, sh2));
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        acc[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(th[i][k >> 2][rt][k & 3], p, acc[rt], 0, 0, 0);
                }
            }
            cb += W * NCH;
            if (cb < T.C) request(T, cb);
        }
        // the waves' partial sums meet in LDS; tile rt goes to wave rt % W
        if (W > 1) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) part[buf][wave][rt][lane] = acc[rt];
            if (g == 0) pref[buf][wave][j16] = ref;
            if (threadIdx.x == 0) s_ticket[buf] = nxt;
            __syncthreads();
        }
        t = __builtin_amdgcn_readfirstlane(W > 1 ? s_ticket[buf] : nxt);
#pragma unroll
        for (int k = 0; k < TPW; ++k) {
            const int rt = wave + W * k;
            if (rt >= RT) break;                                        // wave-uniform
            float top = PC_NEG_INF;
            floatx4 tot = {0.f, 0.f, 0.f, 0.f}, val;
            if (W == 1) {
                top = ref;
                tot = acc[k];
            } else {
                float rw[W];
#pragma unroll
                for (int w = 0; w < W; ++w) { rw[w] = pref[buf][w][j16]; top = fmaxf(top, rw[w]); }
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    const float sc = rw[w] > PC_NEG_INF ? pc_half_scale(rw[w] - top) : 0.0f;
                    const floatx4 pw = part[buf][w][rt][lane];
#pragma unroll
                    for (int r = 0; r < 4; ++r) tot[r] += pw[r] * sc * sc;
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (BWD) {
                    // exp(ln(sum) + (ref - PC_UP) + l_row); sum = 0 or l_row = -inf gives exp2(-inf) = 0
                    const float add = __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(tot[r]) + (lown[k][r] + (top - PC_UP)) * PC_LOG2E);
                    val[r] = top > PC_NEG_INF || tot[r] != tot[r] ? no_sentinel(add) : 0.0f;
                } else {
                    // ln(sum) - PC_UP relative to the largest reference, the logarithm taken of sum / 2^24: a base-2 logarithm
                    // near 0 is far more accurate in absolute terms than one near 29, and these errors add up over the layers
                    val[r] = no_sentinel(fmaf(__builtin_amdgcn_logf(tot[r] * 0x1p-24f), 0.6931471805599453f, 16.635532333f - PC_UP));
                }
            }
            const int rrow = T.sub * TM + rt * 16;
            const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(mail + (int64_t)(T.row0 + rrow) * Bs + (int64_t)T.ct * 256), 0, PC_BUF_RANGE, PC_BUF_FLAGS);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(__attribute__((ext_vector_type(4))) unsigned, val), rm, 16 * lane, 0, PC_AUX_DEVICE);
            if (!BWD && rrow == 0 && g == 0) {
                const float rs = top > PC_NEG_INF ? top : 0.0f;         // all children dead: any finite reference
                __hip_atomic_store(R + (int64_t)(T.row0 >> ks) * Bs + col, rs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (T.root && col < B) ll[col] = rs + val[0];
            }
            float *out = (BWD ? F : l) + (int64_t)(T.row0 + rrow + 4 * g) * Bs + col;
#pragma unroll
            for (int r = 0; r < 4; ++r) out[(int64_t)r * Bs] = val[r];
        }
    }
}

// ---- launchers ----
void launch_begin_forward(const int32_t *x, const uint8_t *mask, int32_t B, int32_t D, int64_t Bs, int32_t n_cats, int32_t *xT,
                          float *l, float *R, float *mail, bool null_mail, const int32_t *ent, int32_t n_ent, int32_t K,
                          int32_t *ticket, hipStream_t s)
{
    Timed timed(KC_MISC, s);
    const int n_xb = (int)((Bs + 31) / 32), n_xt = n_xb * ((D + 31) / 32);
    hipLaunchKernelGGL(k_begin_forward, dim3((unsigned)(n_xt + (n_ent + 1) * fill_shares(K, Bs))), dim3(256), 0, s, x, mask, B, D, Bs, n_cats, xT, n_xb,
                       n_xt, l, R, mail, null_mail, ent, n_ent, K, ticket);
}

void launch_begin_backward(const float *l, float *F, float *N, float *nfmax, const int32_t *blk_ids, int32_t n_blk, int32_t root_id,
                           int32_t K, int64_t Bs, int32_t B, const int32_t *ent, int32_t n_ent, int32_t *ticket, hipStream_t s)
{
    Timed timed(KC_MISC, s);
    const int n_cb = (int)((Bs + 255) / 256);
    hipLaunchKernelGGL(k_begin_backward, dim3((unsigned)(n_blk * n_cb + n_ent * fill_shares(K, Bs) + 1)), dim3(256), 0, s, l, F, N, nfmax, blk_ids, n_blk,
                       n_cb, root_id, K, Bs, B, ent, n_ent, ticket);
}

void launch_flow(const float *theta, float *l, float *R, float *F, float *mail, bool bwd, const FlowDev &f, int32_t K, int64_t Bs, int32_t B,
                 int32_t *ticket, float *ll, int32_t wait_limit, int32_t *fault, hipStream_t s)
{
    if (f.n_ent == 0) return;
    Timed timed(bwd ? KC_SUM_BWD_CHILD : KC_SUM_FWD, s);
    // As many waves as a row has chunks of 32 neighbour nodes, up to eight (a single one needs no merge: 29 against 34 us for an HMM of
    // 16 x 32 states); row tiles of 32 halve the number of tasks that read a neighbour and win from 64 tasks per layer on, tiles
    // of 16 leave a shorter chain before.  Measured with 1 - 16 waves, 16 - 64 rows, 16 and 32 columns, 1 - 4 chunks at once: 32
    // columns lost everywhere, 64 rows won 1 - 2 % on 128- and 256-state trees and lost elsewhere.
    // Workgroups: enough to hold a layer's tasks and the next ones' operands; those beyond that only poll.  256 / 320 / 512 measured:
    // eight waves (one workgroup per CU is 256) HMM T = 60, H = 1024, B = 20 1110 / 1133 / 1189 us, T = 32, H = 512, B = 77 385 / 404 /
    // 394; one and two waves, trees of 800 variables, M = 32 259 / 256 / 260 (with 2048: 297) and 500 variables 266 / 267 / 273, HMM
    // T = 50, H = 64, B = 400 277 / 281 / 290, 784 variables, M = 64 722 / 721 / 729; four waves, M = 128, B = 512 1714 / 1719 / 1704.
    // Below 256 all of them lose (784 variables, M = 64 at 192: 749).
    const int chunks = f.max_nbr * (K / 32);
#define PC_FLOW(WW, RR, HH)                                                                                                  \
    do {                                                                                                                     \
        const int n_ct = (int)(Bs / 16);                                                                                     \
        const int64_t tasks = (int64_t)f.n_ent * (K / (16 * RR)) * n_ct;                                                     \
        const int grid = (int)std::min<int64_t>(tasks, WW == 8 ? 256 : WW == 4 ? 512 : 320);                                 \
        if (bwd) hipLaunchKernelGGL((k_flow<WW, RR, HH, true, false>), dim3(grid), dim3(64 * WW), 0, s, theta, l, R, F, mail, f.ent, f.rec, \
                                    f.list, (int)tasks, n_ct, K, Bs, f.li0, ticket, ll, B, wait_limit, fault);               \
        else if (f.max_items > 8) hipLaunchKernelGGL((k_flow<WW, RR, HH, false, true>), dim3(grid), dim3(64 * WW), 0, s, theta, l, R, F, \
                                mail, f.ent, f.rec, f.list, (int)tasks, n_ct, K, Bs, f.li0, ticket, ll, B, wait_limit, fault);     \
        else hipLaunchKernelGGL((k_flow<WW, RR, HH, false, false>), dim3(grid), dim3(64 * WW), 0, s, theta, l, R, F, mail, f.ent, f.rec, \
                                f.list, (int)tasks, n_ct, K, Bs, f.li0, ticket, ll, B, wait_limit, fault);                   \
    } while (0)
    if (chunks == 1) {
        if ((int64_t)f.n_ent * (K / 16) * (Bs / 16) >= 64 * (int64_t)f.n_levels) PC_FLOW(1, 2, 1);
        else PC_FLOW(1, 1, 1);
    } else if (chunks == 2) PC_FLOW(2, 2, 1);
    else if (chunks <= 4) PC_FLOW(4, 2, 1);
    else if (chunks <= 8) PC_FLOW(8, 2, 1);
    else PC_FLOW(8, 2, 2);
#undef PC_FLOW
}

}  // namespace pc
