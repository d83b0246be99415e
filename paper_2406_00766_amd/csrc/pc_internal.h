// Internal structures of libpc (not part of the C ABI).
#pragma once
#include <cstdint>
#include <string>
#include <vector>

#include "pc.h"

namespace pc {

enum : int { KIND_INPUT = 0, KIND_PRODUCT = 1, KIND_SUM = 2 };

// Flags of one row (= one child block) of a layer's backward tables.
//   BWD_FINAL  product layer, sum child: this is the last layer that adds to the child's flow, which is complete
//              afterwards (log_nf of Alg. 3 / 4 is produced here)
//   BWD_FIRST  this is the first layer of the backward sweep that adds to the child's flow: the kernel stores
//              instead of accumulating, so the flow buffer needs no clearing (the '=' of Alg. 4's last line)
// The per-row word of a group (GroupTab::aux) holds these flags in its low byte and the row's number of real
// neighbours (the rest of the row is padding) from bit AUX_COUNT_SHIFT up.
enum : int32_t { BWD_FINAL = 1, BWD_FIRST = 2, AUX_COUNT_SHIFT = 8 };
inline int32_t bwd_row_flags(int layer_kind, int child_kind, int32_t layer_depth, int32_t last_parent_depth,
                             int32_t first_parent_depth)
{
    int32_t f = 0;
    if (layer_kind == KIND_PRODUCT && child_kind == KIND_SUM && last_parent_depth == layer_depth) f |= BWD_FINAL;
    if (first_parent_depth == layer_depth) f |= BWD_FIRST;
    return f;
}

// Words of a tile of products (LayerTab::tile): starts of the member lists of four classes of the first and four of the second
// set; the node offsets of the 4 x 4 products, 0: none; start of the order's bits; children of a product.
constexpr int PROD_TILE_WORDS = 32;

// One group of a layer: rows padded to a common width (Sec. 4.3).
struct GroupTab {
    int32_t n_rows = 0, width = 0;
    std::vector<int32_t> ids, nbr, par;              // host copies
    std::vector<int32_t> aux;                        // per row: neighbour count << AUX_COUNT_SHIFT | BWD_* flags
    int32_t *d_ids = nullptr, *d_nbr = nullptr, *d_par = nullptr, *d_aux = nullptr;
    bool tied_in_group = false;                       // a parameter block occurs twice: flows need atomics
};

struct LayerTab {
    int32_t kind = 0, depth = 0;
    std::vector<GroupTab> fwd, bwd;
    std::vector<int32_t> blk_ids;                     // node offsets of all blocks of the layer, ascending
    int32_t *d_blk_ids = nullptr;
    // product-scratch mode (Sec. 5): a product layer's blocks are one contiguous id range that lives in the scratch
    // window; a sum layer has its own parameter-flow table (its products are gone when the sweep moves on)
    int32_t scr_first_block = -1;                     // product layers: id of the first block of the layer
    std::vector<int32_t> pf_pb, pf_ptr, pf_sum, pf_child;
    int32_t *d_pf_pb = nullptr, *d_pf_ptr = nullptr, *d_pf_sum = nullptr, *d_pf_child = nullptr;
    // Product layer over input blocks many of which have the same product parents here: its children by equal parents (and equal
    // BWD_FIRST), so that the flow of a class is summed once and not once per block.  Empty where few do.
    std::vector<int32_t> cls_ptr, cls_blk;            // class -> its input blocks (node offsets, ascending)
    std::vector<int32_t> cls_par_ptr, cls_par, cls_first;   // class -> its product parents (node offsets, ascending); 1: the flow is stored
    int32_t *d_cls_ptr = nullptr, *d_cls_blk = nullptr, *d_cls_par_ptr = nullptr, *d_cls_par = nullptr, *d_cls_first = nullptr;
    // Such a layer whose product blocks are the pairs of two sets of classes each: tiles of up to 4 x 4 of them, PROD_TILE_WORDS words
    // (k_prod_tile), and the order of the two classes' blocks in the products' rows, a bit per block.  Empty elsewhere.
    std::vector<int32_t> tile, tile_order;
    int32_t *d_tile = nullptr, *d_tile_order = nullptr;
};

// Tables of the dataflow launches (pc_flow.hip), for K = 32, 64, 128 and circuits that keep their product values.  Entries
// are in task order -- forward: sum blocks by ascending layer, backward: product blocks by descending layer -- so the layers
// from any given one to the root are a suffix (forward) or a prefix (backward).
struct FlowTab {
    std::vector<int32_t> ent, rec, list;              // words as described in pc_flow.hip
    std::vector<int32_t> count_from, max_nbr_from;    // per layer index: entries in that layer and above; most neighbours of one
    int32_t *d_ent = nullptr, *d_rec = nullptr, *d_list = nullptr;
};
// The same launches where the circuit is a chain of single blocks of 32 or 64 nodes (k_chain): CHAIN_WORDS words per sum layer (forward,
// ascending) or product layer (backward, descending), and per layer index how many of them from there up, -1: a layer there is no link
// of a chain.
//   0 node offset of the layer's block  1 its neighbour's (a product block; backward: a sum block)  2 the block whose published values
//   the neighbour takes, 0: none  3 forward: the input block multiplied to them, 0: none  4 parameter offset  5 1 for the root
//   6 the next parameter offset that is another, or this
// few_weights: most links have the parameters of the one before.  whole: forward, the links and their input blocks are all there is, and
// each link takes the one before; every link's variable and table then follow the words of the last
constexpr int CHAIN_WORDS = 8;    // two links to a line of the scalar cache: with 12 words the backward pass of k_chain_wide took 8 % longer
struct ChainTab {
    std::vector<int32_t> words, from;
    int32_t n_links = 0;
    bool few_weights = false, whole = false;
    int32_t *d_words = nullptr;
};
// The product layers that belong to them, as rows with neighbour lists (CSR): forward, product blocks by ascending layer with
// their children; backward, sum and input blocks by descending layer of their highest product parent, with their product
// parents from the highest layer down (lay: the parents' layers).
struct RowTab {
    std::vector<int32_t> ids, start, list, lay, aux;  // aux: neighbours << AUX_COUNT_SHIFT | 1 for a sum block
    std::vector<int32_t> count_from, max_nbr_from;    // per layer index: rows in that layer and above; most neighbours of one
    int32_t *d_ids = nullptr, *d_start = nullptr, *d_list = nullptr, *d_lay = nullptr, *d_aux = nullptr;
};

}  // namespace pc

struct pc_circuit {
    int32_t K = 0, n_blocks = 0, root_block = 0, n_param_blocks = 0;
    int32_t n_vars = 0, n_cats = 0, n_tables = 0;
    std::vector<pc::LayerTab> layers;
    int32_t root_layer = 0;                           // not always the last one: blocks the root does not reach may lie deeper

    // EM normalisation: parameter block -> (row group, real rows, real cols); row group (of short rows) -> child count
    int32_t n_em_groups = 0;
    std::vector<int32_t> pb_group, pb_rows, pb_cols, group_nch;
    std::vector<int32_t> em_ptr, em_list;             // row group -> its parameter blocks (CSR); groups without rows at the end
    int32_t *d_em_ptr = nullptr, *d_em_list = nullptr;
    int32_t *d_pb_rows = nullptr, *d_pb_cols = nullptr, *d_group_nch = nullptr;
    // groups of long rows, not among those above, in segments: their blocks (CSR into em_list) and three words each -- first
    // segment and number of segments of the group, child count of the group
    std::vector<int32_t> em_seg_ptr, em_seg;
    int32_t *d_em_seg_ptr = nullptr, *d_em_seg = nullptr;
    float *d_em_part = nullptr;                       // [segments * K] row sums of flows
    float *d_ztab = nullptr;                          // [n_tables * K] column sums of table flows

    // parameter-centric flow tables: parameter block offset -> CSR list of (sum block, child block) node offsets
    std::vector<int32_t> pf_pb, pf_ptr, pf_sum, pf_child;
    int32_t *d_pf_pb = nullptr, *d_pf_ptr = nullptr, *d_pf_sum = nullptr, *d_pf_child = nullptr;

    // blocks without parents, which no layer of the backward sweep writes.  Sum blocks (the root among them) as
    // node offsets; other blocks and the null block as ~offset
    std::vector<int32_t> init_ids;
    int32_t *d_init_ids = nullptr;

    // per input block (in the order of the input layer): the block whose flow rows hold its flows as well -- the first of its class
    // (LayerTab::cls_blk) where the class has all its parents, else itself
    std::vector<int32_t> flow_rep;
    int32_t *d_flow_rep = nullptr;

    // dataflow launches (empty where they do not apply)
    pc::FlowTab flow_fwd, flow_bwd;
    pc::ChainTab chain_fwd, chain_bwd;
    std::vector<int64_t> sum_edges;                   // per layer (sum layers): block pairs,
    std::vector<int32_t> max_items;                   // most children of a product block that it reads,
    // per layer, what its tasks read (sum layer: forward, product layer: backward): most values waited for at one neighbour, chunks of
    // 32 neighbour nodes in the longest row
    std::vector<int32_t> flow_waits, flow_chunks;
    std::vector<uint8_t> flow_cut;                    // per layer: a dataflow part may begin here (a product layer, and no product
                                                      // block below it is read by a sum block above it)
    pc::RowTab prod_fwd_rows, prod_bwd_rows;
    static constexpr int32_t kWaitLimit = 1 << 22;    // polls of a wait before it is given up: some seconds
    int32_t wait_limit = kWaitLimit;
    int32_t *fault = nullptr, *d_fault = nullptr;     // a word of pinned host memory, set by a launch that gave up; its device address

    // product-scratch mode: product log-probabilities live in a window of max_window_blocks blocks behind the
    // n_persistent_blocks input and sum blocks
    bool product_scratch = false;
    int32_t n_persistent_blocks = 0, max_window_blocks = 0;

    void *d_arena = nullptr;                          // one device allocation behind every d_* above
    size_t arena_bytes = 0;
    bool on_device = false;

    // analysis results handed from compile_host to build_tables_device (cleared afterwards)
    std::vector<int32_t> an_depth, an_last_parent_depth, an_first_parent_depth;

    // optional per-kernel-class timing (pc_profile_*)
    void *profiler = nullptr;                         // pc::Profiler*, owned
    void *plan = nullptr;                             // launch plan (group sets per layer), owned
    int64_t prof_launches[16] = {0};
    double prof_ms[16] = {0.0};

    // state linking pc_backward to the preceding pc_forward
    const void *fw_workspace = nullptr;
    const void *fw_theta = nullptr, *fw_tables = nullptr, *fw_x = nullptr, *fw_mask = nullptr;
    int32_t fw_B = -1;
};

namespace pc {

void set_error(const std::string &msg);
pc_status fail(pc_status st, const std::string &msg);

// Host part of compilation: validation, layering, grouping, table construction, EM maps.
// tables_on_host = false leaves the sum / product layer tables to build_tables_device.
pc_status compile_host(const pc_dag *dag, pc_circuit *c, bool tables_on_host);
// Whether a layer is narrow enough for the dataflow launches at row stride Bs (narrower at a smaller one).
bool flow_narrow(const pc_circuit *c, size_t layer, int64_t Bs);
// Microseconds that such a layer gains from them (negative: loses).
double flow_gain(const pc_circuit *c, size_t layer, int64_t Bs);
// Microseconds more that it takes as the first layer of the launch.
double flow_start_up(const pc_circuit *c, size_t layer, int64_t Bs);
// Device part of compilation: transposes the block graph, sorts neighbour lists and fills every forward and
// backward table with HIP kernels; allocates the handle's device arena and uploads the remaining metadata.
pc_status build_tables_device(const pc_dag *dag, pc_circuit *c, void *stream);
// Alg. 2 (App. A.1): ascending group capacities for the given neighbour counts.
std::vector<int32_t> partition_groups(const std::vector<int32_t> &counts, int32_t max_groups, int32_t tol_permille);

}  // namespace pc
