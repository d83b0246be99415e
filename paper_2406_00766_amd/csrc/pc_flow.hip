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
// What bounds it: the chain through the layers.  Measured (time stamps of the tasks of one layer, forward, from the layer before
// being published): values seen after 0.6 - 0.9 us (1.4 at 512 neighbour nodes; 0.57 us is the bare hand-over between two
// workgroups, 0.45 on one XCD), 0.4 us at 32 nodes, 0.55 at 128, 1.3 at 512 to exponentials and MFMAs (there the eight waves of a CU
// share its matrix cores for 0.85 us), 0.2 - 0.4 us to merge and publish: 1.2, 1.9 and 3.5 us a layer.  Three things had made that 1.4, 2.3
// and 4.8 us: tickets drawn a task ahead, so that a workgroup could be left with a task of the very next layer and find its
// weights unrequested; table words read through the vector memory pipe between two polls; lists in the order of the ids, so
// that the value that arrives last was not the last to be asked for.  Before -> now: forward + backward of an HMM T = 32, H = 512, B = 77
// 163 + 228 -> 126 + 201 us; T = 60, H = 1024, B = 20 523 + 606 -> 281 + 431; 784-variable tree, M = 128, B = 100 349 + 462 -> 316 +
// 438; 500 variables, M = 64, B = 30 137 + 148 -> 114 + 128; HMM T = 50, H = 64, B = 400 114 + 210 -> 98 + 192.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pc_device.h"
#include "pc_internal.h"
#include "pc_kernels.h"

namespace pc {

#define PC_SENTINEL 0xFFFFFFFFu

// Device-scope accesses (sc1); every dword of a wider access is a word of its own.  (A polling loop needs a
// compiler barrier so that it loads again; a volatile access would be system-scope.)
#define PC_AUX_DEVICE 16
__device__ inline floatx4 mail_load(const float *tile, int voff)
{
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)tile, 0, PC_BUF_RANGE, PC_BUF_FLAGS);
    return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, PC_AUX_DEVICE));
}
template <int N>
__device__ inline void mail_store(float *tile, int voff, const float (&v)[N])
{
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)tile, 0, PC_BUF_RANGE, PC_BUF_FLAGS);
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    uint32_t w[N];
#pragma unroll
    for (int k = 0; k < N; ++k) w[k] = __builtin_bit_cast(uint32_t, v[k]);
    if constexpr (N == 4) __builtin_amdgcn_raw_buffer_store_b128(u4{w[0], w[1], w[2], w[3]}, r, voff, 0, PC_AUX_DEVICE);
    else if constexpr (N == 2) __builtin_amdgcn_raw_buffer_store_b64(u2{w[0], w[1]}, r, voff, 0, PC_AUX_DEVICE);
    else __builtin_amdgcn_raw_buffer_store_b32(w[0], r, voff, 0, PC_AUX_DEVICE);
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
// xT[v][b] = pc_category.
// KI = 32, 64: a small input layer of blocks of that size in the same launch, which saves its own (3.3 us of the 17.6 of a 16 x 32 HMM's
// query); its workgroups read x itself, a line per sample where xT would be one for 16 (input_in_begin).
template <int KI>
__global__ __launch_bounds__(256) void k_begin_forward(const int32_t *__restrict__ x, const uint8_t *__restrict__ mask, int32_t B,
                                                       int32_t D, int64_t Bs, int32_t n_cats, int32_t *__restrict__ xT, int32_t n_xb,
                                                       int32_t n_xtiles, float *__restrict__ l, float *__restrict__ R,
                                                       float *__restrict__ mail, bool null_mail, const int32_t *__restrict__ ent,
                                                       int32_t n_ent, int32_t K, int32_t *ticket, const float *__restrict__ tables,
                                                       const int32_t *__restrict__ in_ids, const int32_t *__restrict__ in_var,
                                                       const int32_t *__restrict__ in_tab, int32_t n_in, int32_t n_by_xcd)
{
    if constexpr (KI != 0) {
        const int n_ct = (int)((Bs + 63) / 64);
        if ((int)blockIdx.x < n_in * n_ct) {
            __shared__ float smem[KI * 65 + 64];
            const InputTile t = input_tile_at((int)blockIdx.x, n_in, n_by_xcd, n_ct);
            input_tile<KI, 64, true>(smem, t.block, (int64_t)t.col * 64, tables, x, mask, B, D, in_ids, in_var, in_tab, KI, n_cats, Bs, l, R);
            return;
        }
    }
    const int block = KI ? (int)blockIdx.x - n_in * (int)((Bs + 63) / 64) : (int)blockIdx.x;
    __shared__ int32_t tile[32][33];
    if (block >= n_xtiles) {
        const int q = block - n_xtiles;
        const int n_sh = fill_shares(K, Bs), b = q / n_sh, share = q % n_sh;
        if (b < n_ent) fill_share(mail, nullptr, R, ent[4 * b], share, K, Bs, __builtin_bit_cast(float, PC_SENTINEL));
        else fill_share(l, null_mail ? mail : nullptr, R, 0, share, K, Bs, 0.0f);
        if (q == 0 && threadIdx.x < 2) ticket[threadIdx.x] = 0;
        return;
    }
    const int b0 = (block % n_xb) * 32, v0 = (block / n_xb) * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;           // 256 threads: ty in 0..7
    for (int r = ty; r < 32; r += 8) {
        const int b = b0 + r, v = v0 + tx;
        const int32_t val = v < D ? pc_category(x, mask, b, v, B, D, n_cats) : -1;
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
//        Items stand in the order in which they will be there, so those to wait for are the end of the list and the last is
//        the one that arrives last.  Forward: the neighbour is a product block, the list its children; a neighbour below layer
//        li0 has been evaluated already and stands for itself.  Backward: the neighbour is a sum block, the list its product
//        parents, or itself (layer -1) where it has none.
// They are read as constants, through the scalar cache: a vector load of a table word between two polls was a memory latency
// of the chain.
// `mail` (the rows of log_nf that are not in use at the time: sum rows forward, product rows backward) carries the published
// values in MFMA operand order: per block, 16 rows and 16 columns one 1 KiB tile, lane (j, g) holding rows 4 g .. 4 g + 3 of
// column j -- one 16-byte load per lane where the row-major buffer would take four loads of 4 x 64 bytes, and no line shared
// by two column tiles.
typedef const int32_t __attribute__((address_space(4))) *TabPtr;
template <int N> struct FloatVec { typedef float type __attribute__((ext_vector_type(N))); };
template <> struct FloatVec<1> { typedef float type; };

template <int W, int RT, int NCH, bool BWD, bool EXACT>
__global__ __launch_bounds__(64 * W, W >= 8 ? 1 : 2) void k_flow(const float *__restrict__ theta, float *__restrict__ l, float *R,
                                                                 float *__restrict__ F, float *mail, const int32_t *ent_words,
                                                                 const int32_t *rec_words, const int32_t *list_words,
                                                                 int32_t n_tasks, int32_t n_ct, int32_t K, int64_t Bs, int32_t li0,
                                                                 int32_t *ticket, float *__restrict__ ll, int32_t B,
                                                                 int32_t wait_limit, int32_t *fault)
{
    // Results: the RT tiles of 256 words are dealt to the waves in equal shares, VL consecutive words a lane, so that merge and logarithms
    // of a task take all its waves (dealt tile by tile two of four or eight worked: 0.1 us a layer).
    constexpr int VL = W == 1 ? 4 : RT * 4 / W > 0 ? RT * 4 / W : 1;
    constexpr int TPW = W == 1 ? RT : 1;                                // tiles of a wave's share
    constexpr int RW = W == 1 ? 1 : RT * 4 / VL;                        // waves that have a share
    __shared__ floatx4 part[2][W][RT][W > 1 ? 64 : 1];                  // partial sums of the waves, double-buffered over tasks
    __shared__ float pref[2][W][16];                                    // and their references
    __shared__ int32_t s_ticket[2];
    const TabPtr ent = (TabPtr)(uintptr_t)ent_words, rec = (TabPtr)(uintptr_t)rec_words, list = (TabPtr)(uintptr_t)list_words;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, g = lane >> 4, j16 = lane & 15;
    const int ks = 31 - __builtin_clz(K);                               // K is 32, 64 or 128
    const int TM = 16 * RT, subs = K / TM, cpb = K >> 5;
    // first word of this lane's share and the tile it lies in; word 4 u + r of a tile is row 4 (u / 16) + r of column u % 16
    const int word0 = W == 1 ? 4 * lane : wave * VL * 64 % 256 + VL * lane;
    const int rt0 = W == 1 ? 0 : wave * VL * 64 / 256 % RT;
    const int rj = (word0 >> 2) & 15, rr = 4 * (word0 >> 6) + (word0 & 3);

    struct Task { int32_t ct, sub, row0, rec0, root, C; };              // C: chunks of 32 neighbour nodes
    auto decode = [&](int t) -> Task {
        const int q = t / n_ct, e = 4 * (q / subs);
        return Task{t % n_ct, q % subs, ent[e], ent[e + 1], ent[e + 3], ent[e + 2] * cpb};
    };
    // Tickets: the next task of this workgroup.  (Lane 0 of wave 0 draws; the other lanes' accesses lie outside the buffer's range and do
    // nothing.  A branch around the atomic makes the compiler wait for its result at the branch's end.)
    const __amdgpu_buffer_rsrc_t ticket_word = __builtin_amdgcn_make_buffer_rsrc((void *)ticket, 0, 4, PC_BUF_FLAGS);
    auto draw = [&]() -> int { return __builtin_amdgcn_raw_ptr_buffer_atomic_add_i32(1, ticket_word, threadIdx.x == 0 ? 0 : 4, 0, 0); };

    // operands of this wave's chunks cb, cb + W, ... (NCH of them; past the end the first one again, given the value -inf)
    floatx4 th[NCH][2][RT], v[NCH][2], own_l[BWD ? NCH : 1][2];
    float base[NCH];
    int32_t koff[NCH], own[NCH], cnt[NCH], pre[NCH];                    // list items; those at the beginning that are there already
    TabPtr rp[NCH];
    auto item = [&](int i, int n) -> int32_t {                          // item n of chunk i's list
        if (!BWD && rp[i][4] < li0) return own[i];                      // evaluated before this launch
        return n < 5 ? rp[i][5 + n] : list[2 * (rp[i][1] + n)];
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
            const TabPtr r = rec + 16 * (int64_t)(T.rec0 + cc / cpb);
            rp[i] = r;
            koff[i] = (cc % cpb) * 32;
            cnt[i] = r[2]; own[i] = r[3];
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
            if (BWD) {
                pre[i] = r[10] < li0 ? cnt[i] : 0;                      // the block itself, or parents that are all waited for
            } else if (r[4] < li0) {
                cnt[i] = pre[i] = 1;
            } else {
                int p = 0;
#pragma unroll
                for (int k = 0; k < 5; ++k) p += k < cnt[i] && r[10 + k] < li0;
                if (p == 5)
                    while (p < cnt[i] && list[2 * (r[1] + p) + 1] < li0) ++p;
                pre[i] = p;
            }
            // the first item if it is there already (else zeros from the null block); backward: the sum block's own rows
            const int32_t it = pre[i] > 0 ? item(i, 0) : 0;
            row_values(BWD ? F : l, it, i, col, v[i]);
            if (BWD) row_values(l, own[i], i, col, own_l[i]);
            base[i] = R[(int64_t)((BWD ? own[i] : it) >> ks) * Bs + col];
        }
    };

    int nxt = draw();
    if (W > 1) {
        if (threadIdx.x == 0) s_ticket[1] = nxt;
        __syncthreads();
    }
    int t = __builtin_amdgcn_readfirstlane(W > 1 ? s_ticket[1] : nxt);
    for (int buf = 0; t < n_tasks; buf ^= 1) {
        const Task T = decode(t);
        if (wave < T.C) request(T, wave);
        const int64_t col = (int64_t)T.ct * 16 + j16, rcol = (int64_t)T.ct * 16 + rj;

        float lown[TPW][VL], Rrow = 0.0f;                               // backward: the rows' own log-probabilities, R of their block
        if (BWD) {
#pragma unroll
            for (int k = 0; k < TPW; ++k)
#pragma unroll
                for (int r = 0; r < VL; ++r) lown[k][r] = l[(int64_t)(T.row0 + T.sub * TM + (rt0 + k) * 16 + rr + r) * Bs + rcol];
            Rrow = R[(int64_t)(T.row0 >> ks) * Bs + col];
        }

        floatx4 acc[RT];
        float ref = PC_NEG_INF;                                         // reference of acc; -inf: nothing live yet
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt] = floatx4{0.f, 0.f, 0.f, 0.f};

        for (int cb = wave; cb < T.C;) {
            // Values: the sum of the list items' rows (forward: log-probabilities; backward: flows).  One item of every chunk's
            // list at a time, the null block where a list has none: a branch around a load makes the compiler wait for all before it.
            int max_pre = 0, max_wait = 0, max_cnt = 0, since = 0;
#pragma unroll
            for (int i = 0; i < NCH; ++i) {
                max_pre = max(max_pre, pre[i]);
                max_wait = max(max_wait, cnt[i] - pre[i]);
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
            for (int n = 1; n < max_pre; ++n) {                         // items of earlier launches (the first: requested before)
                floatx4 x[NCH][2];
                float xr[NCH];
#pragma unroll
                for (int i = 0; i < NCH; ++i) {
                    const int32_t it = n < pre[i] ? item(i, n) : 0;
                    row_values(BWD ? F : l, it, i, col, x[i]);
                    if (!BWD) xr[i] = R[(int64_t)(it >> ks) * Bs + col];
                }
                add_item(x, xr);
            }
            // Items of this launch: poll until they are there.  The chunks' lists end together; the words of the next items are requested
            // before the poll.
            int32_t its[NCH];
            auto items_from_end = [&](int w) {
#pragma unroll
                for (int i = 0; i < NCH; ++i) its[i] = w >= 0 && cnt[i] - 1 - w >= pre[i] ? item(i, cnt[i] - 1 - w) : 0;
            };
            items_from_end(max_wait - 1);
            for (int w = max_wait - 1; w >= 0; --w) {
                floatx4 x[NCH][2];
                float xr[NCH];
                const float *src[NCH], *rsrc[NCH];
#pragma unroll
                for (int i = 0; i < NCH; ++i) {
                    src[i] = mail + (int64_t)(its[i] + koff[i]) * Bs + (int64_t)T.ct * 256;
                    rsrc[i] = R + (int64_t)(its[i] >> ks) * Bs + col;
                }
                items_from_end(w - 1);
                bool lost = false;
                for (int spin = 0;; ++spin) {
                    asm volatile("" ::: "memory");
#pragma unroll
                    for (int i = 0; i < NCH; ++i) {
                        x[i][0] = mail_load(src[i], 16 * lane);
                        x[i][1] = mail_load(src[i] + 16 * Bs, 16 * lane);
                        if (!BWD) xr[i] = flow_load(rsrc[i]);
                    }
                    uint32_t most = 0;                                  // the sentinel is the largest word
#pragma unroll
                    for (int i = 0; i < NCH; ++i) {
#pragma unroll
                        for (int k = 0; k < 8; ++k) most = max(most, __builtin_bit_cast(uint32_t, x[i][k >> 2][k & 3]));
                        if (!BWD) most = max(most, __builtin_bit_cast(uint32_t, xr[i]));
                    }
                    if (!__any(most == PC_SENTINEL)) break;
                    if (flow_give_up(spin, wait_limit, ticket, fault)) { lost = true; break; }
                    __builtin_amdgcn_s_sleep(1);
                }
                add_item(x, xr);
                if (lost) {                                             // NaN in all its results (a factor 0 below keeps it)
#pragma unroll
                    for (int i = 0; i < NCH; ++i)
#pragma unroll
                        for (int k = 0; k < 8; ++k) v[i][k >> 2][k & 3] = __builtin_nanf("");
                }
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
        // The next ticket, drawn where nothing of this task waits for memory any more.  Drawn at the task's beginning, every
        // workgroup held two tickets that could lie anything from one task to two grids apart, and some had the very next layer's
        // behind a task they still worked on (HMM T = 32, H = 512, B = 77: the last weights of a layer arrived 1.7 us after its
        // values, 4.8 us a layer; now 3.5); drawn between values and MFMAs it kept the MFMAs waiting (HMM 16 x 32, one sample 29 -> 34 us).
        nxt = draw();
        if (W > 1) {                                                    // the waves' partial sums meet in LDS
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) part[buf][wave][rt][lane] = acc[rt];
            if (g == 0) pref[buf][wave][j16] = ref;
            __syncthreads();
        }
#pragma unroll
        for (int k = 0; k < TPW; ++k) {
            if (W > RW && wave >= RW) break;                            // wave-uniform
            const int rt = rt0 + k;
            float top = PC_NEG_INF, tot[VL], val[VL];
            if (W == 1) {
                top = ref;
#pragma unroll
                for (int r = 0; r < VL; ++r) tot[r] = acc[k][r];
            } else {
                typedef typename FloatVec<VL>::type Share;
                float rw[W];
                Share pw[W];
#pragma unroll
                for (int w = 0; w < W; ++w) rw[w] = pref[buf][w][rj];
#pragma unroll
                for (int w = 0; w < W; ++w) pw[w] = *reinterpret_cast<const Share *>(reinterpret_cast<const float *>(part[buf][w][rt]) + word0);
#pragma unroll
                for (int w = 0; w < W; ++w) top = fmaxf(top, rw[w]);
#pragma unroll
                for (int r = 0; r < VL; ++r) tot[r] = 0.0f;
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    const float sc = rw[w] > PC_NEG_INF ? pc_half_scale(rw[w] - top) : 0.0f;
#pragma unroll
                    for (int r = 0; r < VL; ++r) tot[r] += reinterpret_cast<const float *>(&pw[w])[r] * sc * sc;
                }
            }
#pragma unroll
            for (int r = 0; r < VL; ++r) {
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
            mail_store<VL>(mail + (int64_t)(T.row0 + rrow) * Bs + (int64_t)T.ct * 256, 4 * word0, val);
            if (!BWD && rrow == 0 && rr == 0) {
                const float rs = top > PC_NEG_INF ? top : 0.0f;         // all children dead: any finite reference
                __hip_atomic_store(R + (int64_t)(T.row0 >> ks) * Bs + rcol, rs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (T.root && rcol < B) ll[rcol] = rs + val[0];
            }
            float *out = (BWD ? F : l) + (int64_t)(T.row0 + rrow + rr) * Bs + rcol;
#pragma unroll
            for (int r = 0; r < VL; ++r) out[(int64_t)r * Bs] = val[r];
        }
        if (W > 1) {
            if (threadIdx.x == 0) s_ticket[buf] = nxt;
            __syncthreads();
        }
        t = __builtin_amdgcn_readfirstlane(W > 1 ? s_ticket[buf] : nxt);
    }
}


struct ChainLink { int32_t id, nbr, src, in, par, root, next_par; };    // a link's words (ChainTab)

// ------------------------------------------------------------------------------------------
// Chains: the same layers where each is one block of 32 or 64 nodes that takes values of the layer before it only (ChainTab; an HMM of
// as many states).  A wave walks the whole chain for the columns its lanes hold a node each of (two of 32 nodes, one of 64), so the
// values of a layer stay in registers; nothing is polled and nothing published.
// Bound: the dependent instructions of a layer, one wave's.  A product of a K x K block and a column is K instructions on the vector ALU --
// a lane has its node's row of the weights in registers, the operand comes from the lane's row of sixteen by DPP -- and every
// column has a wave of its own for them, where the matrix cores take sixteen columns at the price of 512 cycles for 32 nodes (k_chain_wide)
// and most of a small batch's are padding.  For it to be that and not the memory, nothing in a layer may wait: operands that do not
// depend on the chain are requested four layers ahead (the stores between are counted with the loads, so one layer ahead is a wait
// for the last layer's stores), weights are loaded where they change, those of the next change when this one's are taken over.
// Layers of HMMs of 16 and 32 layers, k_chain_wide or k_flow -> here: 32 nodes 0.6 us -> 0.3 forward, 0.9 -> 0.4 backward (B = 128; launches of 16
// layers 13.7 -> 8.2 and 19.9 -> 10.4 us); 64 nodes 1.6 -> 0.45, 1.8 -> 0.5.  pc_forward_static, 16 x 32, one sample, the whole pass 15.4 -> 7.2 us.
// (DPP in assembly: the compiler turns these into a move and an operation each)
template <int K> __device__ inline float chain_max(float v)             // over a column's lanes
{
#define PC_ROR(N) "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_ror:" #N " row_mask:0xf bank_mask:0xf\n\t"
    asm(PC_ROR(8) PC_ROR(4) PC_ROR(2) PC_ROR(1) : "+v"(v));
#undef PC_ROR
    float a = v, b = v;
    asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
    a = b = __builtin_amdgcn_fmed3f(a, b, __builtin_inff());            // (fmaxf would quiet both first)
    if (K == 64) {
        asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
        a = __builtin_amdgcn_fmed3f(a, b, __builtin_inff());
    }
    return a;
}
// sum over n of w[n] p(node n of this lane's column)
template <int K> __device__ inline float chain_dot(const float (&w)[K], float p)
{
    float q[K / 16];                                                    // nodes 16 i + j of the column in lane j of every row of sixteen
    q[0] = q[1] = p;
    asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(q[0]), "+v"(q[1]));
    if constexpr (K == 64) {
        q[2] = q[0]; q[3] = q[1];
        asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(q[0]), "+v"(q[2]));
        asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(q[1]), "+v"(q[3]));
    }
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
#define PC_FMA(A, W, J) "v_fmac_f32_dpp %" #A ", %4, %" #W " row_newbcast:" #J " row_mask:0xf bank_mask:0xf\n\t"
#pragma unroll
    for (int i = 0; i < K / 16; ++i)
        asm("s_nop 1\n\t" PC_FMA(0, 5, 0) PC_FMA(1, 6, 1) PC_FMA(2, 7, 2) PC_FMA(3, 8, 3) PC_FMA(0, 9, 4) PC_FMA(1, 10, 5) PC_FMA(2, 11, 6) PC_FMA(3, 12, 7)
            PC_FMA(0, 13, 8) PC_FMA(1, 14, 9) PC_FMA(2, 15, 10) PC_FMA(3, 16, 11) PC_FMA(0, 17, 12) PC_FMA(1, 18, 13) PC_FMA(2, 19, 14) PC_FMA(3, 20, 15)
            : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3])
            : "v"(q[i]), "v"(w[16 * i]), "v"(w[16 * i + 1]), "v"(w[16 * i + 2]), "v"(w[16 * i + 3]), "v"(w[16 * i + 4]), "v"(w[16 * i + 5]), "v"(w[16 * i + 6]),
              "v"(w[16 * i + 7]), "v"(w[16 * i + 8]), "v"(w[16 * i + 9]), "v"(w[16 * i + 10]), "v"(w[16 * i + 11]), "v"(w[16 * i + 12]), "v"(w[16 * i + 13]),
              "v"(w[16 * i + 14]), "v"(w[16 * i + 15]));
#undef PC_FMA
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

struct ChainIn { const float *tables; const int32_t *x; const uint8_t *mask; int32_t D, n_cats; };   // what DIRECT reads

// DIRECT: the input blocks' values come from the tables, and nothing is kept but ll (pc_forward_static): the whole pass.
// Backward, N not null: the root and the null block are the only blocks that no layer of the sweep writes, and this launch writes them
// (as k_begin_backward).
template <int K, bool BWD, bool DIRECT>
__device__ inline void walk_chain(const float *__restrict__ theta, float *l, float *R, float *F, const int32_t *link_words, int32_t n_links, int64_t Bs,
                                  float *__restrict__ ll, int32_t B, const ChainIn &in, float *N = nullptr, float *nfmax = nullptr)
{
    constexpr int D = 4;                                                // links whose operands are under way
    const int lane = threadIdx.x & 63, node = lane % K;
    const int64_t col = ((int64_t)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * (64 / K) + lane / K;
    const TabPtr table = (TabPtr)(uintptr_t)link_words;
    const int at = (int)((node * Bs + col) * 4), col_off = (int)(col * 4), first_off = node == 0 ? col_off : -1;   // -1: beyond every descriptor
    auto buf = [](const void *p, int bytes) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, PC_BUF_FLAGS); };
    auto load = [](__amdgpu_buffer_rsrc_t r, int voff) { return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, 0, 0)); };
    auto store = [](float v, __amdgpu_buffer_rsrc_t r, int voff) { __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), r, voff, 0, 0); };
    auto words = [&](int k) -> ChainLink {
        const TabPtr w = table + CHAIN_WORDS * (k < n_links ? k : n_links - 1);
        return ChainLink{w[0], w[1], w[2], w[3], w[4], w[5], w[6]};
    };

    // DIRECT: rows of the tables (below 0: pc_category's), lane i those of link i of this run of 64, and of the columns of this wave
    int32_t trow[64 / K] = {};
    auto rows_of = [&](int k0) {
        const int k = k0 + lane < n_links ? k0 + lane : n_links - 1;
        const int32_t *w = link_words + CHAIN_WORDS * (int64_t)n_links + 2 * (int64_t)k;
        const int32_t var = w[0], tab = w[1];
#pragma unroll
        for (int c = 0; c < 64 / K; ++c) {
            const int32_t cat = pc_category(in.x, in.mask, col - lane / K + c, var, B, in.D, in.n_cats);
            trow[c] = cat >= 0 ? tab * in.n_cats + cat : cat;
        }
    };

    struct Operands { float a, b, Ra, Rb; int32_t row; };               // forward: the input's value (its reference is 0); backward: l of both blocks, their references
    auto request = [&](int k, const ChainLink &w, Operands &o) {
        if (DIRECT) {
            int32_t r = __builtin_amdgcn_readlane(trow[0], k & 63);
            if (K == 32) {
                const int32_t r1 = __builtin_amdgcn_readlane(trow[K == 32 ? 1 : 0], k & 63);
                r = lane < 32 ? r : r1;
            }
            o.row = r;
            o.a = in.tables[(int64_t)max(r, 0) * K + node];
        } else if (BWD) {
            o.a = load(buf(l + (int64_t)w.nbr * Bs, PC_BUF_RANGE), at);
            o.b = load(buf(l + (int64_t)w.id * Bs, PC_BUF_RANGE), at);
            o.Ra = load(buf(R + (int64_t)(w.nbr / K) * Bs, PC_BUF_RANGE), col_off);
            o.Rb = load(buf(R + (int64_t)(w.id / K) * Bs, PC_BUF_RANGE), col_off);
        } else {
            o.a = load(buf(l + (int64_t)w.in * Bs, PC_BUF_RANGE), at);   // (no input block: the null block's rows, 0)
        }
    };
    float w[K], wn[K];                                                  // this lane's weights; those after the next change
    auto weights = [&](int32_t par) {
        if (BWD) {
#pragma unroll
            for (int n = 0; n < K; ++n) wn[n] = theta[(int64_t)par + n * K + node];
        } else {
            const floatx4 *src = reinterpret_cast<const floatx4 *>(theta + par + node * K);
#pragma unroll
            for (int n = 0; n < K / 4; ++n) {
                const floatx4 t = src[n];
                wn[4 * n] = t[0]; wn[4 * n + 1] = t[1]; wn[4 * n + 2] = t[2]; wn[4 * n + 3] = t[3];
            }
        }
    };

    ChainLink cur = words(0), next, far;
    weights(cur.par);
    // the values that the first link takes have been there before this launch (backward: the root's own flow, or 0 of an unused block)
    float x = 0.0f, Rx = 0.0f;
    if (BWD && N) {
        const float lv = load(buf(l + (int64_t)cur.nbr * Bs, PC_BUF_RANGE), at);
        const bool live = node == 0 && col < B && lv > PC_NEG_INF;
        x = live ? 1.0f : 0.0f;
        store(x, buf(F + (int64_t)cur.nbr * Bs, PC_BUF_RANGE), at);
        store(live ? -lv : PC_NEG_INF, buf(N + (int64_t)cur.nbr * Bs, PC_BUF_RANGE), at);
        store(live ? -lv : PC_NEG_INF, buf(nfmax + (int64_t)(cur.nbr / K) * Bs, PC_BUF_RANGE), first_off);
        store(0.0f, buf(F, PC_BUF_RANGE), at);
    } else if (BWD) x = load(buf(F + (int64_t)cur.nbr * Bs, PC_BUF_RANGE), at);
    else if (!DIRECT) { x = load(buf(l + (int64_t)cur.src * Bs, PC_BUF_RANGE), at); Rx = R[(int64_t)(cur.src / K) * Bs + col]; }
    // (the stores of a link go to a descriptor of no bytes here: the compiler waits for a count of accesses that holds on all paths into the loop)
    Operands ops[D];
    const __amdgpu_buffer_rsrc_t none = buf(theta, 0);
    auto ahead = [&](int k0, int i) {
        request(k0 + i, words(k0 + i), ops[i]);
        asm volatile("" ::: "memory");
        if (!DIRECT) store(0.0f, none, at);
        if (!DIRECT && !BWD) store(0.0f, none, at);
        if (!BWD) store(0.0f, none, at);
        asm volatile("" ::: "memory");
    };
    int32_t par = 0;
    auto link = [&](int k, Operands &o) {
        if (cur.par != par) {                                           // uniform
            par = cur.par;
#pragma unroll
            for (int n = 0; n < K; ++n) { w[n] = wn[n]; asm volatile("" : "+v"(w[n])); }   // (waits in here, not where the paths meet)
            weights(cur.next_par);
        }
        const bool taken = cur.src != 0 || (BWD && k == 0);             // uniform
        const float xt = taken ? x : 0.0f;
        float y, base, val;
        if (BWD) {
            y = o.a > PC_NEG_INF ? __logf(xt) - o.a : PC_NEG_INF;       // flow 0: -inf
            base = o.Rb - o.Ra;
        } else if (DIRECT) {
            const float e = o.row >= 0 ? __logf(o.a) : o.row == -1 ? 0.0f : PC_NEG_INF;
            y = xt + (cur.in != 0 ? e : 0.0f);
            base = taken ? Rx : 0.0f;
        } else {
            y = xt + o.a;
            base = taken ? Rx : 0.0f;
        }
        const float lown = o.b;
        request(k + D, far, o);
        const ChainLink now = cur;
        const int bytes = k < n_links ? PC_BUF_RANGE : 0;               // (the links are rounded up to whole turns of the loop)
        cur = next; next = words(k + 2); far = words(k + D + 1);
        float cm = chain_max<K>(y);
        const bool live = cm > PC_NEG_INF;
        cm = live ? rintf(cm) : 0.0f;
        base = live ? base + cm : PC_NEG_INF;                           // the reference: there is but one chunk
        // exp(y - cm + PC_UP); dead: y = -inf
        const float p = __builtin_amdgcn_exp2f(fmaf(y - cm, PC_LOG2E, live ? PC_UP * PC_LOG2E : 0.0f));
        const float sum = chain_dot<K>(w, p);
        if (BWD) {                                                      // as in k_flow
            const float add = __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(sum) + (lown + (base - PC_UP)) * PC_LOG2E);
            val = live ? add : 0.0f;
            store(val, buf(F + (int64_t)now.id * Bs, bytes), at);
        } else {
            val = fmaf(__builtin_amdgcn_logf(sum * 0x1p-24f), 0.6931471805599453f, 16.635532333f - PC_UP);
            Rx = live ? base : 0.0f;                                    // all children dead: any finite reference
            if (!DIRECT) {
                store(val, buf(l + (int64_t)now.id * Bs, bytes), at);
                store(Rx, buf(R + (int64_t)(now.id / K) * Bs, bytes), first_off);
            }
            store(Rx + val, buf(ll, now.root && k < n_links ? 4 * B : 0), first_off);
        }
        x = val;
        asm volatile("" :: "s"(cur.id), "s"(cur.nbr), "s"(cur.src), "s"(cur.in), "s"(cur.par), "s"(cur.root));   // the words are here by now
    };
    for (int k0 = 0; k0 < n_links; k0 += DIRECT ? 64 : n_links) {       // (DIRECT: a lane has the rows of one link in 64)
        if (DIRECT) rows_of(k0);
        const int k1 = DIRECT ? min(k0 + 64, n_links) : n_links;
        next = words(k0 + 1); far = words(k0 + D);
#pragma unroll
        for (int i = 0; i < D; ++i) ahead(k0, i);
        asm volatile("" : "+v"(x), "+v"(Rx));                           // (waited for here)
        for (int k = k0; k < k1; k += D) { link(k, ops[0]); link(k + 1, ops[1]); link(k + 2, ops[2]); link(k + 3, ops[3]); }
    }
}

template <bool BWD>
__global__ __launch_bounds__(256) void k_chain(const float *__restrict__ theta, float *l, float *R, float *F, float *N, float *nfmax, const int32_t *link_words, int32_t n_links,
                                               int64_t Bs, float *__restrict__ ll, int32_t B)
{
    walk_chain<32, BWD, false>(theta, l, R, F, link_words, n_links, Bs, ll, B, ChainIn{}, N, nfmax);
}
template <bool BWD>
__global__ __launch_bounds__(256) void k_walk64(const float *__restrict__ theta, float *l, float *R, float *F, float *N, float *nfmax, const int32_t *link_words, int32_t n_links,
                                                int64_t Bs, float *__restrict__ ll, int32_t B)
{
    walk_chain<64, BWD, false>(theta, l, R, F, link_words, n_links, Bs, ll, B, ChainIn{}, N, nfmax);
}
template <int K>
__global__ __launch_bounds__(256) void k_walk_pass(const float *__restrict__ theta, const int32_t *link_words, int32_t n_links, float *__restrict__ ll,
                                                   int32_t B, const ChainIn in)
{
    walk_chain<K, false, true>(theta, nullptr, nullptr, nullptr, link_words, n_links, 0, ll, B, in);
}

// The same for large batches of 32 nodes: one wave per 16 columns, on the matrix cores; in MFMA layout the results of one layer are the
// operands of the next lane by lane.  Bound: the instructions of a layer, some 250 of one wave, 0.6 us against 1.1 us for a task of
// k_flow with its hand-over.
template <bool BWD>
__global__ __launch_bounds__(64) void k_chain_wide(const float *__restrict__ theta, float *l, float *R, float *F, const int32_t *link_words,
                                                   int32_t n_links, int64_t Bs, float *__restrict__ ll, int32_t B)
{
    constexpr int K = 32;
    const int lane = threadIdx.x, g = lane >> 4, j16 = lane & 15;
    const int64_t col = (int64_t)blockIdx.x * 16 + j16;
    const TabPtr table = (TabPtr)(uintptr_t)link_words;
    const int row4 = (int)(Bs * 4), tile_off = (int)((4 * g * Bs + col) * 4), col_off = (int)(col * 4);   // bytes: a row; row 4 g of a tile
    const int first_off = g == 0 ? col_off : -1;                        // beyond every descriptor: lanes without row 0 of a tile
    auto buf = [](const void *p, int bytes) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, PC_BUF_FLAGS); };
    auto load = [](__amdgpu_buffer_rsrc_t r, int voff, int soff) { return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0)); };
    auto store = [](float v, __amdgpu_buffer_rsrc_t r, int voff, int soff) { __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), r, voff, soff, 0); };

    auto words = [&](int k) -> ChainLink {
        const TabPtr w = table + CHAIN_WORDS * (k < n_links ? k : n_links - 1);
        return ChainLink{w[0], w[1], w[2], w[3], w[4], w[5], 0};
    };
    auto rows = [&](const float *X, int32_t row, floatx4 (&x)[2]) {     // 32 rows in operand order: lane (j, g), rows 16 c2 + 4 g + e of column j
        const __amdgpu_buffer_rsrc_t r = buf(X + (int64_t)row * Bs, PC_BUF_RANGE);
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k >> 2][k & 3] = load(r, tile_off, (16 * (k >> 2) + (k & 3)) * row4);
    };
    struct Operands {
        floatx4 th[2][2], in[2], lown[2];
        float base, Rrow;
        int32_t id, src, root;
    };
    // what a link reads that the chain does not compute
    auto request = [&](const ChainLink &w, Operands &o) {
        o.id = w.id; o.src = w.src; o.root = w.root;
        const __amdgpu_buffer_rsrc_t r = buf(theta + w.par, PC_BUF_RANGE);
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int c2 = 0; c2 < 2; ++c2) {
                if (BWD) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) o.th[c2][rt][e] = load(r, (4 * g * K + j16) * 4, ((16 * c2 + e) * K + 16 * rt) * 4);
                } else {
                    o.th[c2][rt] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, (j16 * K + 4 * g) * 4, 64 * K * rt + 64 * c2, 0));
                }
            }
        const int32_t from = BWD ? w.nbr : w.in;                        // (no input block: the null block's rows, 0)
        rows(l, from, o.in);
        o.base = load(buf(R + (int64_t)(from / K) * Bs, PC_BUF_RANGE), col_off, 0);
        if (BWD) {
            rows(l, w.id, o.lown);
            o.Rrow = load(buf(R + (int64_t)(w.id / K) * Bs, PC_BUF_RANGE), col_off, 0);
        }
    };

    // the values that the first link takes have been there before this launch (backward: the root's own flow, or 0 of an unused block)
    ChainLink w = words(0);
    floatx4 x[2];
    rows(BWD ? F : l, BWD ? w.nbr : w.src, x);
    float Rx = BWD ? 0.0f : R[(int64_t)(w.src / K) * Bs + col];
    auto link = [&](int k, const Operands &o, Operands &ahead) {
        request(w, ahead);                                              // link k + 1
        w = words(k + 2);
        const bool taken = o.src != 0 || (BWD && k == 0);               // uniform
        float base = BWD ? o.Rrow - o.base : o.base + (taken ? Rx : 0.0f), cm = PC_NEG_INF;
        floatx4 v[2], acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}}, val[2];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float y = taken ? x[e >> 2][e & 3] : 0.0f;
            if (BWD) {
                const float lo = o.in[e >> 2][e & 3];
                y = lo > PC_NEG_INF ? __logf(y) - lo : PC_NEG_INF;       // flow 0: -inf
            } else {
                y += o.in[e >> 2][e & 3];
            }
            v[e >> 2][e & 3] = y;
            cm = fmaxf(cm, y);
        }
        cm = max_over_groups(cm);
        const bool live = cm > PC_NEG_INF;
        cm = live ? rintf(cm) : 0.0f;
        base = live ? base + cm : PC_NEG_INF;                           // the reference: there is but one chunk
        // exp(v - cm + PC_UP); dead: v = -inf
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float p = __builtin_amdgcn_exp2f(fmaf(v[e >> 2][e & 3] - cm, PC_LOG2E, live ? PC_UP * PC_LOG2E : 0.0f));
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) acc[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(o.th[e >> 2][rt][e & 3], p, acc[rt], 0, 0, 0);
        }
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {                               // as in k_flow
                if (BWD) {
                    const float add = __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(acc[rt][r]) + (o.lown[rt][r] + (base - PC_UP)) * PC_LOG2E);
                    val[rt][r] = live ? add : 0.0f;
                } else {
                    val[rt][r] = fmaf(__builtin_amdgcn_logf(acc[rt][r] * 0x1p-24f), 0.6931471805599453f, 16.635532333f - PC_UP);
                }
            }
        const __amdgpu_buffer_rsrc_t out = buf((BWD ? F : l) + (int64_t)o.id * Bs, PC_BUF_RANGE);
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r) store(val[rt][r], out, tile_off, (16 * rt + r) * row4);
        if (!BWD) {
            Rx = live ? base : 0.0f;                                    // all children dead: any finite reference
            store(Rx, buf(R + (int64_t)(o.id / K) * Bs, PC_BUF_RANGE), first_off, 0);
            store(Rx + val[0][0], buf(ll, o.root ? 4 * B : 0), first_off, 0);
        }
        x[0] = val[0]; x[1] = val[1];
        asm volatile("" :: "s"(w.id), "s"(w.nbr), "s"(w.src), "s"(w.in), "s"(w.par), "s"(w.root));   // the words are here by now
    };
    Operands a, b;                                                      // in turn: a copy would be some forty moves a layer
    request(w, a);
    w = words(1);
    for (int k = 0; k < n_links; k += 2) {
        link(k, a, b);
        if (k + 1 < n_links) link(k + 1, b, a);
    }
}

// ---- launchers ----
// A small input layer joins the begin of the pass.  Up to 4096 workgroups: beyond, a launch is nothing beside them, and they would read x a line
// per sample.
bool input_in_begin(const GroupDev &in, int32_t K, int64_t Bs) { return (K == 32 || K == 64) && in.n_rows * ((Bs + 63) / 64) <= 4096; }

void launch_begin_forward(const int32_t *x, const uint8_t *mask, int32_t B, int32_t D, int64_t Bs, int32_t n_cats, int32_t *xT,
                          float *l, float *R, float *mail, bool null_mail, const int32_t *ent, int32_t n_ent, int32_t K,
                          int32_t *ticket, const float *tables, const GroupDev &in, hipStream_t s)
{
    const bool with_input = input_in_begin(in, K, Bs);
    Timed timed(with_input ? KC_INPUT_FWD : KC_MISC, s);
    const int n_xb = (int)((Bs + 31) / 32), n_xt = n_xb * ((D + 31) / 32);
    const unsigned wgs = (unsigned)(n_xt + (n_ent + 1) * fill_shares(K, Bs) + (with_input ? in.n_rows * ((Bs + 63) / 64) : 0));
#define PC_BEGIN(KI) hipLaunchKernelGGL(k_begin_forward<KI>, dim3(wgs), dim3(256), 0, s, x, mask, B, D, Bs, n_cats, xT, n_xb, n_xt, l, R, mail, null_mail, \
                                        ent, n_ent, K, ticket, tables, in.ids, in.nbr, in.par, in.n_rows, input_by_xcd(in, K, Bs))
    if (with_input && K == 32) PC_BEGIN(32);
    else if (with_input) PC_BEGIN(64);
    else PC_BEGIN(0);
#undef PC_BEGIN
}

void launch_begin_backward(const float *l, float *F, float *N, float *nfmax, const int32_t *blk_ids, int32_t n_blk, int32_t root_id,
                           int32_t K, int64_t Bs, int32_t B, const int32_t *ent, int32_t n_ent, int32_t *ticket, hipStream_t s)
{
    Timed timed(KC_MISC, s);
    const int n_cb = (int)((Bs + 255) / 256);
    hipLaunchKernelGGL(k_begin_backward, dim3((unsigned)(n_blk * n_cb + n_ent * fill_shares(K, Bs) + 1)), dim3(256), 0, s, l, F, N, nfmax, blk_ids, n_blk,
                       n_cb, root_id, K, Bs, B, ent, n_ent, ticket);
}

// As many waves as a row has chunks of 32 neighbour nodes, up to eight (a single one needs no merge: an HMM of 16 x 32
// states, a chain of its own kernel since, 29 against 34 us); in longer rows a wave takes two or four chunks at once (HMM T = 60, H = 1024, B = 20, rows of 32 chunks: forward 421
// us two at a time, 324 four; fewer waves with two chunks each lost everywhere but on a 3072-variable tree's forward pass, 2587 ->
// 2502), but no more than two where the products' rounding errors are kept: four take 256 registers and spill (PD of 4 x 4 cells, rows of
// 24 chunks, K = 64, B = 32 62 us four at a time, 44 two; K = 32, B = 64 86, 58).  Row tiles of 32 halve the number of tasks that read a neighbour, tiles of 16 leave a shorter chain and win where
// the widest layer has at most 128 tasks of them, 16 -> 32: HMM T = 60, H = 1024, B = 20 (128 tasks) 281 -> 324 us, T = 40, H = 256, B =
// 10 (32) 90 -> 100, T = 50, H = 64, B = 400 (104) 98 -> 101; T = 32, H = 512, B = 77 (192) 131 -> 126, trees (thousands in their lower
// layers) of 784 variables, M = 128, B = 512 788 -> 650, of 500, M = 64, B = 30 120 -> 114.  64 rows and 32 columns lost.
FlowShape flow_shape(const FlowDev &f, bool bwd, int32_t K, int64_t Bs)
{
    const int chunks = f.max_nbr * (K / 32);
    const bool exact = !bwd && f.max_items > 8;
    return FlowShape{chunks <= 2 ? chunks : chunks <= 4 ? 4 : 8, f.max_level * (int64_t)(K / 16) * (Bs / 16) <= 128 ? 1 : 2,
                     chunks <= 8 ? 1 : chunks <= 16 || exact ? 2 : 4, exact};
}

void launch_flow(const float *theta, float *l, float *R, float *F, float *mail, bool bwd, const FlowDev &f, int32_t K, int64_t Bs, int32_t B,
                 int32_t *ticket, float *ll, int32_t wait_limit, int32_t *fault, hipStream_t s)
{
    if (f.n_ent == 0) return;
    Timed timed(bwd ? KC_SUM_BWD_CHILD : KC_SUM_FWD, s);
    // Workgroups: enough to hold a layer's tasks and the next ones' operands; those beyond that only poll.  256 / 512 measured: eight waves
    // (one workgroup per CU is 256) HMM T = 32, H = 512, B = 77 126 / 154 us, T = 40, H = 256, B = 10 90 / 98; one and two waves, trees of
    // 800 variables, M = 32, B = 300 166 / 167, HMM T = 50, H = 64, B = 400 98 / 101; four waves, trees, no difference.
    const FlowShape sh = flow_shape(f, bwd, K, Bs);
#define PC_FLOW(WW, RR, HH)                                                                                                  \
    do {                                                                                                                     \
        const int n_ct = (int)(Bs / 16);                                                                                     \
        const int64_t tasks = (int64_t)f.n_ent * (K / (16 * RR)) * n_ct;                                                     \
        const int grid = (int)std::min<int64_t>(tasks, WW == 8 ? 256 : WW == 4 ? 512 : 320);                                 \
        if (bwd) hipLaunchKernelGGL((k_flow<WW, RR, HH, true, false>), dim3(grid), dim3(64 * WW), 0, s, theta, l, R, F, mail, f.ent, f.rec, \
                                    f.list, (int)tasks, n_ct, K, Bs, f.li0, ticket, ll, B, wait_limit, fault);               \
        else if (sh.exact) hipLaunchKernelGGL((k_flow<WW, RR, HH == 4 ? 2 : HH, false, true>), dim3(grid), dim3(64 * WW), 0, s, theta, l, R, F, \
                                mail, f.ent, f.rec, f.list, (int)tasks, n_ct, K, Bs, f.li0, ticket, ll, B, wait_limit, fault);     \
        else hipLaunchKernelGGL((k_flow<WW, RR, HH, false, false>), dim3(grid), dim3(64 * WW), 0, s, theta, l, R, F, mail, f.ent, f.rec, \
                                f.list, (int)tasks, n_ct, K, Bs, f.li0, ticket, ll, B, wait_limit, fault);                   \
    } while (0)
#define PC_FLOW_ROWS(WW, HH) do { if (sh.tiles == 1) PC_FLOW(WW, 1, HH); else PC_FLOW(WW, 2, HH); } while (0)
    if (sh.waves == 1) PC_FLOW_ROWS(1, 1);
    else if (sh.waves == 2) PC_FLOW_ROWS(2, 1);
    else if (sh.waves == 4) PC_FLOW_ROWS(4, 1);
    else if (sh.chunks == 1) PC_FLOW_ROWS(8, 1);
    else if (sh.chunks == 2) PC_FLOW_ROWS(8, 2);
    else PC_FLOW_ROWS(8, 4);
#undef PC_FLOW_ROWS
#undef PC_FLOW
}

// Columns up to which a chain has a wave per column (two columns at K = 32).  HMMs, forward + backward, another kernel (k_chain_wide at K = 32,
// k_flow at 64; k_begin_backward's 4 us come on top) / here: K = 32, 32 layers, B = 128 61 / 31 us, 2048 62 / 43, 4096 63 / 84, four layers
// 2048 11 / 14; K = 64, 32 layers, B = 128 103 / 40, 2048 201 / 157, 4096 393 / 315, eight layers 4096 forward 53 / 46, six 41 / 43, 2048 47 / 49.
// Where most links have weights of their own, loading them counts: K = 32, 16 layers, B = 256 34 / 23, 1024 34 / 29, 2048 35 / 39; K = 64 58 / 35,
// 512 62 / 44, 1024 65 / 71.  Chains of fewer than six layers of 64: two, B = 256 11.5 / 10.8, 512 15 / 14, 2048 11 / 18 forward, four
// 19 / 12, 24 / 15, 35 / 40.  These two are walked to 256 columns, one workgroup on a CU; more would pay up to some 512.
bool chain_walks(bool few_weights, int32_t n_links, int32_t K, int64_t Bs)
{
    return Bs <= (!few_weights || (K == 64 && n_links < 6) ? 256 : K == 32 || n_links < 8 ? 2048 : 4096);
}
// Waves of a workgroup of a walk: one while every workgroup has a CU for itself, where waves of one CU wait for each other's weights (K = 64,
// 16 layers, B = 256 26 us, with two 28, four 36; weights of their own 35, 41, 65), then two (B = 512 32, 29, 38), then four, which share them
// (B = 2048 100, 116, 87).
static int walk_waves(int64_t waves) { return waves <= 256 ? 1 : waves <= 512 ? 2 : 4; }

void launch_chain(const float *theta, float *l, float *R, float *F, float *N, float *nfmax, bool bwd, const ChainDev &c, int32_t K, int64_t Bs, int32_t B,
                  float *ll, hipStream_t s)
{
    Timed timed(bwd ? KC_SUM_BWD_CHILD : KC_SUM_FWD, s);
    if (c.walks) {
        const int wgw = walk_waves(Bs * K / 64);
        const dim3 grid((unsigned)(Bs * K / 64 / wgw)), block(64 * wgw);
        if (K == 32 && bwd) hipLaunchKernelGGL(k_chain<true>, grid, block, 0, s, theta, l, R, F, N, nfmax, c.words, c.n_links, Bs, ll, B);
        else if (K == 32) hipLaunchKernelGGL(k_chain<false>, grid, block, 0, s, theta, l, R, F, N, nfmax, c.words, c.n_links, Bs, ll, B);
        else if (bwd) hipLaunchKernelGGL(k_walk64<true>, grid, block, 0, s, theta, l, R, F, N, nfmax, c.words, c.n_links, Bs, ll, B);
        else hipLaunchKernelGGL(k_walk64<false>, grid, block, 0, s, theta, l, R, F, N, nfmax, c.words, c.n_links, Bs, ll, B);
        return;
    }
    const dim3 grid((unsigned)(Bs / 16));
    if (bwd) hipLaunchKernelGGL(k_chain_wide<true>, grid, dim3(64), 0, s, theta, l, R, F, c.words, c.n_links, Bs, ll, B);
    else hipLaunchKernelGGL(k_chain_wide<false>, grid, dim3(64), 0, s, theta, l, R, F, c.words, c.n_links, Bs, ll, B);
}

void launch_walk_pass(const float *theta, const float *tables, const int32_t *x, const uint8_t *mask, const ChainDev &c, int32_t K, int32_t B,
                      int32_t n_vars, int32_t n_cats, float *ll, hipStream_t s)
{
    const ChainIn in{tables, x, mask, n_vars, n_cats};
    const int wgw = walk_waves(((int64_t)B * K + 63) / 64), cols = 64 / K * wgw;
    const dim3 grid((unsigned)((B + cols - 1) / cols)), block(64 * wgw);
    if (K == 32) hipLaunchKernelGGL(k_walk_pass<32>, grid, block, 0, s, theta, c.words, c.n_links, ll, B, in);
    else hipLaunchKernelGGL(k_walk_pass<64>, grid, block, 0, s, theta, c.words, c.n_links, ll, B, in);
}

}  // namespace pc
