// Launchers of the HIP kernels (internal).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

namespace pc {

struct GroupDev {            // device view of one table group
    int32_t n_rows, width;
    const int32_t *ids, *nbr, *par;
    bool tied;
    const int32_t *aux;      // per row: real neighbours << 8 | bit 0 flow final after this layer | bit 1 first layer to write it
};

// Table groups of one layer that one launch covers (a kernel argument, passed by value).  Rows of the launch are
// numbered through the groups; group g holds rows first[g] .. first[g + 1].
constexpr int PC_MAX_SET = 8;
struct GroupSet {
    int32_t n;
    int32_t first[PC_MAX_SET + 1];
    int32_t width[PC_MAX_SET];
    const int32_t *ids[PC_MAX_SET], *nbr[PC_MAX_SET], *par[PC_MAX_SET], *aux[PC_MAX_SET];
};

// The same for rows given as neighbour lists (CSR) instead of padded groups: ids[0], nbr[0] = list, par[0] = start, aux[0];
// backward: nbr[1] = the neighbours' layers, width[1] = first layer whose neighbours count.
constexpr int PC_ROWS_ONE = 0, PC_ROWS_MULTI = 1, PC_ROWS_CSR = 2;

struct ParamFlowDev {        // parameter blocks with the (sum block, child block) pairs that use them
    int32_t n_pb;
    const int32_t *pb, *ptr, *sum, *child;
    int64_t n_pairs;         // entries of sum / child
};

struct FlowDev {             // a dataflow launch (pc_flow.hip): entries from layer li0 to the root
    const int32_t *ent, *rec, *list;
    int32_t n_ent, max_nbr, li0, max_level; // max_level: entries of the widest layer
    int32_t max_items;       // forward: most children of a product block that is read
};

struct ChainDev {            // a dataflow launch over a chain (k_chain): its links in the order they are worked off
    const int32_t *words;
    int32_t n_links;         // 0: not a chain
    bool walks;              // a wave per column (k_chain, k_walk64), else one per sixteen (k_chain_wide)
};

struct RowsDev {             // product-layer rows of a dataflow launch as neighbour lists
    const int32_t *ids, *start, *list, *lay, *aux;
    int32_t n_rows, max_nbr, li0;
};

struct ClassesDev {          // input blocks in classes of equal product parents (LayerTab::cls_*)
    int32_t n, avg;          // classes; blocks of one, on average
    const int32_t *ptr, *blk, *par_ptr, *par, *first;
};

struct EmDev {               // row groups with their parameter blocks; those from n_groups on have no rows; segments of long rows
    int32_t n_groups, n_all, avg_list, n_seg;
    const int32_t *ptr, *list, *pb_rows, *pb_cols, *group_nch, *seg_ptr, *seg;
    float *part, *ztab;
};

void set_force_generic(bool on);

// Optional per-launch timing: when a profiler is installed, every launcher brackets its kernel with two
// HIP events on the launch stream; totals per kernel class are summed when the profile is read.
enum KernelClass : int {
    KC_MISC = 0, KC_INPUT_FWD, KC_PROD_FWD, KC_SUM_FWD, KC_LOGNF, KC_SUM_BWD_CHILD, KC_SUM_BWD_PARAM, KC_PROD_BWD,
    KC_INPUT_BWD, KC_EM, KC_SPLIT, KC_COUNT
};
struct Profiler {
    struct Rec { int cls; hipEvent_t a, b; };
    std::vector<Rec> recs;
    int64_t bf16_launches[16] = {0};                    // per class: launches that ran on the bf16 matrix cores
    std::vector<hipEvent_t> pool;
    hipEvent_t get();
    void collect(int64_t *launches, double *ms);      // waits for the recorded events, adds to the totals
    ~Profiler();
};
void set_profiler(Profiler *p);                        // nullptr switches timing off
struct Timed {                                          // brackets one kernel launch
    hipStream_t s;
    hipEvent_t b = nullptr;
    Timed(int cls, hipStream_t stream);
    ~Timed();
};

void launch_fill(float *p, int64_t n, float v, hipStream_t s);
void launch_readout(const float *l, const float *R, int64_t root_row, int64_t root_blk, int64_t Bs, int32_t B, float *ll,
                    hipStream_t s);
int input_tile_cols(const GroupDev &g, int32_t K, int64_t Bs);
int input_by_xcd(const GroupDev &g, int32_t K, int64_t Bs);
void launch_input_fwd(const float *tables, const int32_t *xT, const GroupDev &g, int32_t K, int32_t n_cats, int64_t Bs,
                      float *l, float *R, hipStream_t s);
void launch_input_bwd(const float *F, const int32_t *xT, const GroupDev &g, int32_t K, int32_t n_cats, int64_t Bs,
                      float *table_flow, hipStream_t s);
// The four layer launchers take all table groups of the layer, packed into sets by make_group_sets: the groups of a
// layer are independent of one another, and one launch covers a whole set.
std::vector<GroupSet> make_group_sets(const std::vector<GroupDev> &groups);
// Ph / Pl non-null: the kernel also writes the bf16 value planes of its rows (see launch_split_p)
// l: base the children are read from, lout: base the products are written to (the same, except in the product-scratch mode)
void launch_prod_fwd(const float *l, float *lout, float *R, const std::vector<GroupSet> &sets, int32_t K, int64_t Bs, void *Ph, void *Pl,
                     hipStream_t s);
// Fpar: base the parents' flows are read from (= F, except in the product-scratch mode)
void launch_prod_bwd(const float *l, float *F, const float *Fpar, float *N, float *nfmax, const std::vector<GroupSet> &sets, int32_t K,
                     int64_t Bs, void *Ph, void *Pl, hipStream_t s);
// Product layer over classes of input blocks: forward, tiles of products (LayerTab::tile); backward, a class's flow stored to its blocks
bool prod_takes_tiles(int32_t K, int32_t n_rows, int32_t n_tiles, int32_t width, int64_t Bs);   // width: most children of a product
struct ProdTile { int pairs, side; };                                   // k_prod_tile's template arguments: column pairs, side x side products
ProdTile prod_tile_shape(int32_t n_tiles, int32_t K, int64_t Bs);
void launch_prod_fwd_tiles(float *l, float *R, const int32_t *tile, int32_t n_tiles, const int32_t *order, const int32_t *cls_blk, int32_t K,
                           int64_t Bs, hipStream_t s);
void launch_prod_bwd_classes(float *F, const ClassesDev &c, int32_t K, int64_t Bs, hipStream_t s);
// the product layers of a dataflow launch: all their rows in one launch
void launch_prod_fwd_rows(float *l, float *R, const RowsDev &rows, int32_t K, int64_t Bs, hipStream_t s);
void launch_prod_bwd_rows(const float *l, float *F, float *N, float *nfmax, const RowsDev &rows, int32_t K, int64_t Bs, void *Ph,
                          void *Pl, hipStream_t s);
// lch: base the product children are read from; l: base of the sum rows written; part: base of scratch
// rows for the product children.  ll not null:
// the layer is the root alone; true if it has been read out into ll[0 .. B)
void sum_kernel_name(char (&name)[64], const GroupSet &gs, bool bwd, int32_t K, int64_t Bs);
bool launch_sum_fwd(const float *theta, const float *lch, float *l, float *R, float *part, const std::vector<GroupSet> &sets, int32_t K,
                    int64_t Bs, float *ll, int32_t B, hipStream_t s);
void launch_sum_bwd_child(const float *theta, const float *l, const float *R, const float *N, const float *nfmax, float *F,
                          const std::vector<GroupSet> &sets, int32_t K, int64_t Bs, hipStream_t s);
void launch_sum_bwd_param_generic(const float *theta, const float *l, const float *R, const float *N, float *G,
                                  const GroupDev &g, int32_t K, int64_t Bs, int32_t B, hipStream_t s);
// bf16-split path (long dense reductions): operand planes and the kernels that read them
bool sum_layer_takes_bf16(int32_t K, int32_t n_groups, int32_t n_rows, int32_t width, int64_t Bs);
void launch_split_theta(const float *theta, int64_t n_blocks, int32_t K, bool transposed, void *Th, void *Tl, hipStream_t s);
void launch_split_p(const float *X, const float *ref, const int32_t *blk_ids, int32_t n_blk, int32_t K, int64_t Bs, void *Ph,
                    void *Pl, hipStream_t s);
void launch_sum_bf16(const void *Th, const void *Tl, const void *Ph, const void *Pl, float *l, float *R, const float *nfmax,
                     float *F, bool bwd, const GroupSet &gs, int32_t K, int64_t Bs, hipStream_t s);
bool param_flow_by_block(int32_t K);
bool use_flow();
void launch_param_flow(const float *theta, const float *l, const float *R, const float *N, const float *nfmax, float *G,
                       const ParamFlowDev &pf, int32_t K, int64_t Bs, hipStream_t s);
void launch_em(float *theta, float *tables, float *theta_flow, float *table_flow, const EmDev &em, int32_t K,
               int32_t n_tables, int32_t n_cats, float step, float pc, hipStream_t s);

// pc_flow.hip: the first launch of a forward / backward pass (ent, n_ent: blocks the dataflow launch will publish) and the
// dataflow launch itself (fault: set to 1 if a wait was given up after wait_limit polls)
// (in: the input layer, evaluated here if input_in_begin)
struct FlowShape { int waves, tiles, chunks; bool exact; };             // k_flow's template arguments: waves, row tiles of 16, chunks per wave
FlowShape flow_shape(const FlowDev &f, bool bwd, int32_t K, int64_t Bs);
bool input_in_begin(const GroupDev &in, int32_t K, int64_t Bs);
void launch_begin_forward(const int32_t *x, const uint8_t *mask, int32_t B, int32_t D, int64_t Bs, int32_t n_cats, int32_t *xT,
                          float *l, float *R, float *mail, bool null_mail, const int32_t *ent, int32_t n_ent, int32_t K,
                          int32_t *ticket, const float *tables, const GroupDev &in, hipStream_t s);
void launch_begin_backward(const float *l, float *F, float *N, float *nfmax, const int32_t *blk_ids, int32_t n_blk, int32_t root_id,
                           int32_t K, int64_t Bs, int32_t B, const int32_t *ent, int32_t n_ent, int32_t *ticket, hipStream_t s);
bool chain_walks(bool few_weights, int32_t n_links, int32_t K, int64_t Bs);
// N, nfmax not null (backward, where it walks): the launch does k_begin_backward's work for the root and the null block
void launch_chain(const float *theta, float *l, float *R, float *F, float *N, float *nfmax, bool bwd, const ChainDev &c, int32_t K, int64_t Bs, int32_t B,
                  float *ll, hipStream_t s);
// the whole of a forward pass that keeps nothing but ll, over a circuit that is a chain from its inputs to the root (ChainTab::whole)
void launch_walk_pass(const float *theta, const float *tables, const int32_t *x, const uint8_t *mask, const ChainDev &c, int32_t K, int32_t B,
                      int32_t n_vars, int32_t n_cats, float *ll, hipStream_t s);
void launch_flow(const float *theta, float *l, float *R, float *F, float *mail, bool bwd, const FlowDev &f, int32_t K, int64_t Bs, int32_t B,
                 int32_t *ticket, float *ll, int32_t wait_limit, int32_t *fault, hipStream_t s);

}  // namespace pc
