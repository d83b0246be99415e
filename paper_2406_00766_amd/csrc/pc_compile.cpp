// Host side of pc_compile: validation, layering by depth (Sec. 3), grouping of node blocks by
// neighbour count (Sec. 4.3, App. A.1 / Alg. 2) and construction of the forward and backward
// index tensors (Sec. 4.3, App. A.2).  Integer work only.
//
// Canonical form (the paper leaves ordering open; these rules make the tables unique):
//   * node offset of block u is (u+1)*K, offset 0 is the null block; parameter offset of block p
//     is (p+1)*K*K, offset 0 is the all-zero block; padding entries are 0 / 0;
//   * depth(input) = 0, depth(n) = 1 + max depth(children); layers: inputs, then for each depth the
//     product blocks, then the sum blocks;
//   * blocks ascend by id inside a layer and inside a group; a block joins the smallest capacity
//     that holds its count; a row lists its neighbours by ascending node offset;
//   * product layers get the same forward / backward table pair as sum layers.
#include <algorithm>
#include <array>
#include <cstring>
#include <limits>
#include <map>
#include <numeric>
#include <unordered_map>

#include "pc_internal.h"

namespace pc {

static thread_local std::string g_last_error;
void set_error(const std::string &msg) { g_last_error = msg; }
pc_status fail(pc_status st, const std::string &msg) { g_last_error = msg; return st; }
const char *last_error_cstr() { return g_last_error.c_str(); }

// Alg. 2 with the following reading of the printed listing: group counts are tried from 1 upwards
// and the first one whose optimal padded size is within sum*(1+tol) wins (the text asks for the
// fewest groups), else max_groups; the back-pointers are followed through decreasing group count;
// the result is the set of distinct capacities; integer arithmetic throughout; on equal cost the
// smallest split index wins.
std::vector<int32_t> partition_groups(const std::vector<int32_t> &counts, int32_t max_groups, int32_t tol_permille)
{
    std::vector<int32_t> caps;
    if (counts.empty()) return caps;
    std::map<int32_t, int64_t> hist;
    for (int32_t v : counts) ++hist[v];
    std::vector<int64_t> val, cum;
    int64_t running = 0, total = 0;
    for (auto &kv : hist) {
        val.push_back(kv.first);
        running += kv.second;
        cum.push_back(running);
        total += (int64_t)kv.first * kv.second;
    }
    const int L = (int)val.size();
    const int G = std::max<int32_t>(1, max_groups);
    const int64_t target = total + (total * (int64_t)tol_permille + 999) / 1000;

    // cost[n][i]: least padded size of the i+1 smallest distinct counts using at most n capacities,
    // the largest of which is val[i]
    std::vector<std::vector<int64_t>> cost(G + 1, std::vector<int64_t>(L, 0));
    std::vector<std::vector<int32_t>> prev(G + 1, std::vector<int32_t>(L, 0));
    for (int i = 0; i < L; ++i) cost[1][i] = val[i] * cum[i];
    int n_sel = 1;
    if (cost[1][L - 1] > target) {
        n_sel = G;
        for (int n = 2; n <= G; ++n) {
            cost[n][0] = val[0] * cum[0];
            prev[n][0] = 0;
            for (int i = 1; i < L; ++i) {
                int64_t best = std::numeric_limits<int64_t>::max();
                int32_t arg = -1;
                for (int j = 0; j < i; ++j) {
                    const int64_t cand = cost[n - 1][j] + val[i] * (cum[i] - cum[j]);
                    if (cand < best) { best = cand; arg = j; }
                }
                cost[n][i] = best;
                prev[n][i] = arg;
            }
            if (cost[n][L - 1] <= target) { n_sel = n; break; }
        }
    }
    int i = L - 1;
    for (int n = n_sel; n >= 1; --n) {
        caps.push_back((int32_t)val[i]);
        if (n > 1) i = prev[n][i];
    }
    std::sort(caps.begin(), caps.end());
    caps.erase(std::unique(caps.begin(), caps.end()), caps.end());
    return caps;
}

namespace {

struct Row {
    int64_t id;                                        // node offset of the row's own block
    std::vector<std::pair<int64_t, int64_t>> nbrs;     // (neighbour node offset, parameter offset)
};

bool fits_i32(int64_t v) { return v >= 0 && v <= std::numeric_limits<int32_t>::max(); }

// rows arrive in ascending id; neighbours get sorted here
pc_status build_groups(std::vector<Row> &rows, int32_t max_groups, int32_t tol_permille,
                       std::vector<GroupTab> &out)
{
    std::vector<int32_t> counts(rows.size());
    for (size_t r = 0; r < rows.size(); ++r) counts[r] = (int32_t)rows[r].nbrs.size();
    const std::vector<int32_t> caps = partition_groups(counts, max_groups, tol_permille);
    out.assign(caps.size(), GroupTab());
    for (size_t g = 0; g < caps.size(); ++g) out[g].width = caps[g];
    for (Row &row : rows) {
        const int32_t cnt = (int32_t)row.nbrs.size();
        const size_t g = std::lower_bound(caps.begin(), caps.end(), cnt) - caps.begin();
        GroupTab &gt = out[g];
        std::sort(row.nbrs.begin(), row.nbrs.end());
        if (!fits_i32(row.id)) return fail(PC_ERR_TOO_LARGE, "node offset exceeds int32");
        gt.ids.push_back((int32_t)row.id);
        gt.aux.push_back(cnt << AUX_COUNT_SHIFT);
        for (int32_t j = 0; j < gt.width; ++j) {
            int64_t a = 0, p = 0;
            if (j < cnt) { a = row.nbrs[j].first; p = row.nbrs[j].second; }
            if (!fits_i32(a) || !fits_i32(p)) return fail(PC_ERR_TOO_LARGE, "table entry exceeds int32");
            gt.nbr.push_back((int32_t)a);
            gt.par.push_back((int32_t)p);
        }
        ++gt.n_rows;
    }
    for (GroupTab &gt : out) {
        std::vector<int32_t> ps;
        for (int32_t p : gt.par) if (p != 0) ps.push_back(p);
        std::sort(ps.begin(), ps.end());
        gt.tied_in_group = std::adjacent_find(ps.begin(), ps.end()) != ps.end();
    }
    return PC_OK;
}

// Chains (ChainTab): one block a layer with one neighbour, which takes the values of the sum layer before (forward) or of the product
// layer above (backward), or none of this launch.
void compile_chain(const pc_dag *d, pc_circuit *c, const std::vector<int32_t> &par_ptr, const std::vector<int32_t> &par_of,
                   const std::vector<int64_t> &par_edge, const std::vector<int32_t> &layer_of, int32_t from)
{
    const int32_t K = d->K, L = (int32_t)c->layers.size();
    auto off = [&](int32_t u) { return (u + 1) * K; };
    auto only = [&](int32_t li) { return li >= 0 && li < L && c->layers[li].blk_ids.size() == 1 ? c->layers[li].blk_ids[0] / K - 1 : -1; };
    auto fwd_link = [&](int32_t li, std::vector<int32_t> &w) -> bool {
        const int32_t u = only(li);
        if (u < 0 || d->child_ptr[u + 1] - d->child_ptr[u] != 1) return false;
        const int32_t p = d->child[d->child_ptr[u]];
        if (layer_of[p] != li - 1) return false;
        w = {off(u), off(p), 0, 0, (d->param_blk[d->child_ptr[u]] + 1) * K * K, u == d->root_block ? 1 : 0, 0, 0};
        for (int64_t e = d->child_ptr[p]; e < d->child_ptr[p + 1]; ++e) {
            const int32_t k = d->child[e];
            int32_t &at = d->type[k] == KIND_INPUT ? w[3] : w[2];
            if (at != 0 || (d->type[k] == KIND_SUM && k != only(li - 2))) return false;
            at = off(k);
        }
        return true;
    };
    auto bwd_link = [&](int32_t li, std::vector<int32_t> &w) -> bool {
        const int32_t u = only(li);
        if (u < 0 || par_ptr[u + 1] - par_ptr[u] != 1) return false;
        const int32_t s = par_of[par_ptr[u]], ns = par_ptr[s + 1] - par_ptr[s];
        if (layer_of[s] != li + 1 || ns > 1) return false;
        w = {off(u), off(s), 0, 0, (d->param_blk[par_edge[par_ptr[u]]] + 1) * K * K, 0, 0, 0};
        // a flow that is there already (the root's, or 0 of an unused block) is read by the first link only
        if (ns == 0) return s != d->root_block || c->chain_bwd.words.empty();
        const int32_t p = par_of[par_ptr[s]];
        w[2] = off(p);
        return p == only(li + 2) && par_ptr[p] != par_ptr[p + 1];
    };
    for (ChainTab *t : {&c->chain_fwd, &c->chain_bwd}) t->from.assign(L + 1, 0);
    std::vector<std::vector<int32_t>> fwd;
    for (int32_t li = L; li-- > from;) {
        const bool sums = c->layers[li].kind == KIND_SUM;
        c->chain_fwd.from[li] = c->chain_fwd.from[li + 1]; c->chain_bwd.from[li] = c->chain_bwd.from[li + 1];
        int32_t &n = (sums ? c->chain_fwd : c->chain_bwd).from[li];
        std::vector<int32_t> w;
        if (n < 0 || (K != 32 && K != 64) || !(sums ? fwd_link(li, w) : bwd_link(li, w))) { n = -1; continue; }
        ++n;
        if (sums) fwd.push_back(w);
        else c->chain_bwd.words.insert(c->chain_bwd.words.end(), w.begin(), w.end());
    }
    for (size_t k = fwd.size(); k-- > 0;) c->chain_fwd.words.insert(c->chain_fwd.words.end(), fwd[k].begin(), fwd[k].end());
    for (ChainTab *t : {&c->chain_fwd, &c->chain_bwd}) {
        const size_t n = t->words.size() / CHAIN_WORDS;
        t->n_links = (int32_t)n;
        size_t changes = 0;
        for (size_t k = n; k-- > 0;) {
            int32_t *w = t->words.data() + k * CHAIN_WORDS;
            w[6] = k + 1 == n ? w[4] : w[CHAIN_WORDS + 4] != w[4] ? w[CHAIN_WORDS + 4] : w[CHAIN_WORDS + 6];
            changes += k + 1 < n && w[CHAIN_WORDS + 4] != w[4];
        }
        t->few_weights = changes <= 1 + n / 8;
    }
    std::vector<int32_t> &fw = c->chain_fwd.words;
    bool whole = from == 1 && c->chain_fwd.from[1] > 0 && d->n_blocks == 3 * c->chain_fwd.from[1];
    for (int32_t k = 0; whole && k < c->chain_fwd.from[1]; ++k) {
        const int32_t *w = fw.data() + k * CHAIN_WORDS;
        whole = w[3] != 0 && par_ptr[w[3] / K] - par_ptr[w[3] / K - 1] == 1 && w[2] == (k ? w[-CHAIN_WORDS] : 0);
    }
    c->chain_fwd.whole = whole;
    for (int32_t k = 0; whole && k < c->chain_fwd.from[1]; ++k) {
        const int32_t in = fw[k * CHAIN_WORDS + 3] / K - 1;
        fw.insert(fw.end(), {d->in_var[in], d->in_table[in]});
    }
}

// Tables of the dataflow launches (pc_internal.h, pc_flow.hip), for the layers such a launch may cover at some batch size.
void compile_flow(const pc_dag *d, pc_circuit *c, const std::vector<int32_t> &par_ptr, const std::vector<int32_t> &par_of,
                  const std::vector<int64_t> &par_edge)
{
    const int32_t n = d->n_blocks, K = d->K, L = (int32_t)c->layers.size();
    std::vector<int32_t> layer_of(n, 0);
    for (int32_t li = 0; li < L; ++li)
        for (int32_t id : c->layers[li].blk_ids) layer_of[id / K - 1] = li;
    auto off = [&](int32_t u) { return (u + 1) * K; };

    c->sum_edges.assign(L, 0);
    c->max_items.assign(L, 0);
    c->flow_waits.assign(L, 0);
    c->flow_chunks.assign(L, 0);
    std::vector<int32_t> readers(n, 0);                   // product parents that are read themselves, of a sum block
    for (int32_t u = 0; u < n; ++u)
        if (d->type[u] == KIND_SUM) readers[u] = (int32_t)std::count_if(par_of.begin() + par_ptr[u], par_of.begin() + par_ptr[u + 1],
                                                                       [&](int32_t p) { return par_ptr[p] != par_ptr[p + 1]; });
    c->flow_cut.assign(L + 1, 0);
    int32_t reach = 0;                                    // highest layer that reads a product block of the layers so far
    for (int32_t li = 0; li < L; ++li) {
        const LayerTab &T = c->layers[li];
        c->flow_cut[li] = li > 0 && T.kind == KIND_PRODUCT && reach < li;
        int64_t row = 0;                                  // block pairs of the longest row
        int32_t waits = 0;                                // most values that a task waits for at one neighbour
        for (int32_t id : T.blk_ids) {
            const int32_t u = id / K - 1;
            if (T.kind == KIND_SUM) {
                c->sum_edges[li] += d->child_ptr[u + 1] - d->child_ptr[u];
                row = std::max<int64_t>(row, d->child_ptr[u + 1] - d->child_ptr[u]);
                for (int64_t e = d->child_ptr[u]; e < d->child_ptr[u + 1]; ++e) {
                    const int64_t k0 = d->child_ptr[d->child[e]], k1 = d->child_ptr[d->child[e] + 1];
                    c->max_items[li] = std::max(c->max_items[li], (int32_t)(k1 - k0));
                    if (k1 - k0 <= 12)                    // (a layer that reads longer ones is out: flow_narrow)
                        waits = std::max(waits, (int32_t)std::count_if(d->child + k0, d->child + k1, [&](int32_t k) { return d->type[k] == KIND_SUM; }));
                }
            } else if (T.kind == KIND_PRODUCT) {
                for (int32_t k = par_ptr[u]; k < par_ptr[u + 1]; ++k) {
                    reach = std::max(reach, layer_of[par_of[k]]);
                    waits = std::max(waits, readers[par_of[k]]);
                }
                row = std::max<int64_t>(row, par_ptr[u + 1] - par_ptr[u]);
            }
        }
        c->flow_waits[li] = waits;
        c->flow_chunks[li] = (int32_t)std::min<int64_t>(row * (K / 32), 1 << 20);
    }
    int32_t from = L;                                     // the part at the smallest batch holds those at all others
    for (int32_t li = L; li-- > 1 && flow_narrow(c, li, 32);) if (c->flow_cut[li]) from = li;
    if (from == L) return;

    for (FlowTab *f : {&c->flow_fwd, &c->flow_bwd}) { f->count_from.assign(L + 1, 0); f->max_nbr_from.assign(L + 1, 0); }
    for (RowTab *r : {&c->prod_fwd_rows, &c->prod_bwd_rows}) { r->count_from.assign(L + 1, 0); r->max_nbr_from.assign(L + 1, 0); r->start.assign(1, 0); }
    // list of every product block's children and of every sum block's product parents (or itself): (node offset, layer), in the order
    // in which the sweep produces them
    std::vector<int32_t> list_at(n, 0), list_n(n, 0);
    for (int32_t u = 0; u < n; ++u) {
        if (d->type[u] == KIND_INPUT || layer_of[u] < from) continue;
        std::vector<int32_t> &to = d->type[u] == KIND_PRODUCT ? c->flow_fwd.list : c->flow_bwd.list;
        list_at[u] = (int32_t)(to.size() / 2);
        if (d->type[u] == KIND_PRODUCT) {
            std::vector<int32_t> ch(d->child + d->child_ptr[u], d->child + d->child_ptr[u + 1]);
            std::sort(ch.begin(), ch.end(), [&](int32_t a, int32_t b) { return layer_of[a] != layer_of[b] ? layer_of[a] < layer_of[b] : a < b; });
            for (int32_t k : ch) to.insert(to.end(), {off(k), layer_of[k]});
        } else {
            std::vector<int32_t> pa;
            for (int32_t k = par_ptr[u]; k < par_ptr[u + 1]; ++k)       // an unused product parent has flow 0
                if (par_ptr[par_of[k]] != par_ptr[par_of[k] + 1]) pa.push_back(par_of[k]);
            std::stable_sort(pa.begin(), pa.end(), [&](int32_t a, int32_t b) { return layer_of[a] > layer_of[b]; });
            for (int32_t k : pa) to.insert(to.end(), {off(k), layer_of[k]});
            // the root or an unused sum block (its own flow rows are initialised); one whose parents are all unused: flow 0
            if ((int32_t)(to.size() / 2) == list_at[u]) to.insert(to.end(), {par_ptr[u] == par_ptr[u + 1] ? off(u) : 0, -1});
        }
        list_n[u] = (int32_t)(to.size() / 2) - list_at[u];
    }
    auto add_rec = [&](FlowTab &f, int32_t par, int32_t nbr) {
        const int32_t at = list_at[nbr], cnt = list_n[nbr];
        f.rec.insert(f.rec.end(), {par, at, cnt, off(nbr), layer_of[nbr]});
        for (int w = 0; w < 2; ++w)
            for (int32_t k = 0; k < 5; ++k) f.rec.push_back(k < cnt ? f.list[2 * (at + k) + w] : -1);
        f.rec.push_back(0);
    };
    for (int32_t li = from; li < L; ++li) {
        const LayerTab &T = c->layers[li];
        for (int32_t id : T.blk_ids) {
            const int32_t u = id / K - 1;
            std::vector<std::pair<int32_t, int64_t>> ch;
            for (int64_t e = d->child_ptr[u]; e < d->child_ptr[u + 1]; ++e) ch.emplace_back(d->child[e], e);
            std::sort(ch.begin(), ch.end());
            if (T.kind == KIND_SUM) {
                FlowTab &f = c->flow_fwd;
                f.ent.insert(f.ent.end(), {id, (int32_t)(f.rec.size() / 16), (int32_t)ch.size(), u == d->root_block ? 1 : 0});
                for (auto &k : ch) add_rec(f, (d->param_blk[k.second] + 1) * K * K, k.first);
                ++f.count_from[li];
                f.max_nbr_from[li] = std::max(f.max_nbr_from[li], (int32_t)ch.size());
            } else {
                RowTab &r = c->prod_fwd_rows;
                r.ids.push_back(id);
                for (auto &k : ch) r.list.push_back(off(k.first));
                r.start.push_back((int32_t)r.list.size());
                r.aux.push_back((int32_t)ch.size() << AUX_COUNT_SHIFT);
                ++r.count_from[li];
                r.max_nbr_from[li] = std::max(r.max_nbr_from[li], (int32_t)ch.size());
            }
        }
    }
    for (int32_t li = L; li-- > from;) {
        const LayerTab &T = c->layers[li];
        if (T.kind != KIND_PRODUCT) continue;
        for (int32_t id : T.blk_ids) {
            const int32_t u = id / K - 1, n_par = par_ptr[u + 1] - par_ptr[u];
            if (n_par == 0) continue;
            FlowTab &f = c->flow_bwd;
            f.ent.insert(f.ent.end(), {id, (int32_t)(f.rec.size() / 16), n_par, 0});
            for (int32_t k = par_ptr[u]; k < par_ptr[u + 1]; ++k) add_rec(f, (d->param_blk[par_edge[k]] + 1) * K * K, par_of[k]);
            ++f.count_from[li];
            f.max_nbr_from[li] = std::max(f.max_nbr_from[li], n_par);
        }
    }
    // backward rows: blocks with product parents of these layers, by descending layer of the highest one
    std::vector<std::vector<int32_t>> by_top(L);
    for (int32_t u = 0; u < n; ++u) {
        if (d->type[u] == KIND_PRODUCT) continue;
        int32_t top = 0;
        for (int32_t k = par_ptr[u]; k < par_ptr[u + 1]; ++k) top = std::max(top, layer_of[par_of[k]]);
        if (top >= from) by_top[top].push_back(u);
    }
    for (int32_t li = L; li-- > from;)
        for (int32_t u : by_top[li]) {
            RowTab &r = c->prod_bwd_rows;
            std::vector<int32_t> pa(par_of.begin() + par_ptr[u], par_of.begin() + par_ptr[u + 1]);
            std::stable_sort(pa.begin(), pa.end(), [&](int32_t a, int32_t b) { return layer_of[a] > layer_of[b]; });
            r.ids.push_back(off(u));
            for (int32_t p : pa) { r.list.push_back(off(p)); r.lay.push_back(layer_of[p]); }
            r.start.push_back((int32_t)r.list.size());
            r.aux.push_back((int32_t)pa.size() << AUX_COUNT_SHIFT | (d->type[u] == KIND_SUM ? 1 : 0));
            ++r.count_from[li];
            r.max_nbr_from[li] = std::max(r.max_nbr_from[li], (int32_t)pa.size());
        }
    compile_chain(d, c, par_ptr, par_of, par_edge, layer_of, from);
    auto accumulate = [&](std::vector<int32_t> &cnt, std::vector<int32_t> &most) {
        for (int32_t li = L; li-- > 0;) { cnt[li] += cnt[li + 1]; most[li] = std::max(most[li], most[li + 1]); }
    };
    for (FlowTab *f : {&c->flow_fwd, &c->flow_bwd}) accumulate(f->count_from, f->max_nbr_from);
    for (RowTab *r : {&c->prod_fwd_rows, &c->prod_bwd_rows}) accumulate(r->count_from, r->max_nbr_from);
}

// Tiles of a product layer whose classes are there already (LayerTab::tile): the product blocks must be the pairs of classes of two
// sets each, and the blocks of a pair's classes must alternate in the same order in every product of the sets.
void compile_product_tiles(LayerTab &T, int32_t K, int32_t n)
{
    const int32_t n_cls = (int32_t)T.cls_first.size();
    std::vector<std::array<int32_t, 2>> of_row(n, {-1, -1});                // product block -> its two classes
    std::vector<std::vector<int32_t>> next(n_cls);
    for (int32_t q = 0; q < n_cls; ++q)
        for (int32_t k = T.cls_par_ptr[q]; k < T.cls_par_ptr[q + 1]; ++k) {
            auto &two = of_row[T.cls_par[k] / K - 1];
            if (two[1] >= 0) return;
            two[two[0] < 0 ? 0 : 1] = q;
        }
    for (int32_t id : T.blk_ids) {
        const auto &two = of_row[id / K - 1];
        if (two[1] < 0) return;
        next[two[0]].push_back(two[1]); next[two[1]].push_back(two[0]);
    }
    auto blocks = [&](int32_t q) { return T.cls_ptr[q + 1] - T.cls_ptr[q]; };
    std::vector<int32_t> side(n_cls, -1), tile, order, row_at(n_cls, -1);
    for (int32_t q0 = 0; q0 < n_cls; ++q0) {
        if (side[q0] >= 0) continue;
        std::vector<int32_t> set[2], todo(1, q0);                            // the component of q0, two-coloured
        side[q0] = 0;
        while (!todo.empty()) {
            const int32_t q = todo.back();
            todo.pop_back();
            set[side[q]].push_back(q);
            for (int32_t o : next[q]) {
                if (side[o] == side[q]) return;
                if (side[o] < 0) { side[o] = 1 - side[q]; todo.push_back(o); }
            }
        }
        for (auto &v : set) std::sort(v.begin(), v.end());
        if (set[1].empty()) return;
        // a product for every pair, checked before the tiles are laid out: without it there are up to (classes / 8)^2 of them for a number of
        // products that grows with the classes only (16 000 classes in a ring: 409 MB and 1.2 s)
        for (int32_t q : set[0]) if (next[q].size() != set[1].size()) return;
        // the order in which the blocks of a pair's classes stand in a product's row: that of the first pair, a bit per block, 1 for the
        // second set's.  It is every pair's where at each change of sides all blocks of the one place come before all of the next.
        const int32_t na = blocks(set[0][0]), nb = blocks(set[1][0]), n_pos = na + nb, at = (int32_t)order.size();
        std::vector<int32_t> lo[2], hi[2];
        for (int h = 0; h < 2; ++h) {
            lo[h].assign(h ? nb : na, std::numeric_limits<int32_t>::max()); hi[h].assign(h ? nb : na, 0);
            for (int32_t q : set[h]) {
                if (blocks(q) != (h ? nb : na)) return;
                for (int32_t k = 0; k < blocks(q); ++k) {
                    const int32_t id = T.cls_blk[T.cls_ptr[q] + k];
                    lo[h][k] = std::min(lo[h][k], id); hi[h][k] = std::max(hi[h][k], id);
                }
            }
        }
        order.resize(order.size() + (n_pos + 31) / 32, 0);
        for (int32_t i = 0, j = 0, last = -1; i + j < n_pos;) {
            const int32_t h = i < na && (j == nb || T.cls_blk[T.cls_ptr[set[0][0]] + i] < T.cls_blk[T.cls_ptr[set[1][0]] + j]) ? 0 : 1;
            if (last >= 0 && last != h && hi[last][last ? j - 1 : i - 1] >= lo[h][h ? j : i]) return;
            int32_t &word = order[at + ((i + j) >> 5)];
            word = (int32_t)((uint32_t)word | (uint32_t)h << ((i + j) & 31));
            ++(h ? j : i);
            last = h;
        }
        const size_t first_tile = tile.size();
        const int32_t ta = ((int32_t)set[0].size() + 3) / 4, tb = ((int32_t)set[1].size() + 3) / 4;
        for (int32_t i = 0; i < ta; ++i)
            for (int32_t j = 0; j < tb; ++j) {
                std::vector<int32_t> w(PROD_TILE_WORDS, 0);
                for (int32_t k = 0; k < 4; ++k) {                            // (past the end: the last class again, without a product)
                    w[k] = T.cls_ptr[set[0][std::min<size_t>(4 * i + k, set[0].size() - 1)]];
                    w[4 + k] = T.cls_ptr[set[1][std::min<size_t>(4 * j + k, set[1].size() - 1)]];
                }
                w[24] = at; w[25] = n_pos;
                tile.insert(tile.end(), w.begin(), w.end());
            }
        for (auto &v : set) for (size_t k = 0; k < v.size(); ++k) row_at[v[k]] = (int32_t)k;
        for (int32_t qa : set[0])
            for (int32_t k = T.cls_par_ptr[qa]; k < T.cls_par_ptr[qa + 1]; ++k) {
                const auto &two = of_row[T.cls_par[k] / K - 1];
                const int32_t qb = two[0] == qa ? two[1] : two[0], i = row_at[qa], j = row_at[qb];
                int32_t &at16 = tile[first_tile + PROD_TILE_WORDS * (size_t)(i / 4 * tb + j / 4) + 8 + 4 * (i % 4) + j % 4];
                if (at16 != 0) return;                                       // two products of one pair
                at16 = T.cls_par[k];
            }
    }
    T.tile = std::move(tile);
    T.tile_order = std::move(order);
}

// Classes of input blocks with equal product parents (LayerTab::cls_*), and the tiles of the products over them.
void compile_classes(const pc_dag *d, pc_circuit *c, const std::vector<int32_t> &par_ptr, const std::vector<int32_t> &par_of)
{
    const int32_t n = d->n_blocks, K = d->K;
    std::vector<int32_t> layer_of(n, 0), rep(n);
    for (int32_t li = 0; li < (int32_t)c->layers.size(); ++li)
        for (int32_t id : c->layers[li].blk_ids) layer_of[id / K - 1] = li;
    for (int32_t u = 0; u < n; ++u) rep[u] = u;
    std::vector<uint8_t> seen(n, 0);
    for (int32_t li = 0; li < (int32_t)c->layers.size(); ++li) {
        LayerTab &T = c->layers[li];
        if (T.kind != KIND_PRODUCT) continue;
        int64_t reads = 0;                                // block rows that the product kernels read
        bool inputs_only = true;
        std::vector<int32_t> members;
        for (int32_t id : T.blk_ids) {
            const int32_t u = id / K - 1;
            reads += d->child_ptr[u + 1] - d->child_ptr[u];
            for (int64_t e = d->child_ptr[u]; e < d->child_ptr[u + 1]; ++e) {
                const int32_t ch = d->child[e];
                inputs_only = inputs_only && d->type[ch] == KIND_INPUT;
                if (!seen[ch]) { seen[ch] = 1; members.push_back(ch); }
            }
            if (!inputs_only) break;
        }
        const bool shared = inputs_only && 2 * (int64_t)members.size() <= reads;
        for (int32_t u : members) seen[u] = shared;
        if (!shared) continue;
        members.clear();                                  // again, ascending
        for (int32_t u = 0; u < n; ++u) if (seen[u]) { seen[u] = 0; members.push_back(u); }
        // Classes: blocks with equal parents in this layer and equal BWD_FIRST (lists are ascending), told apart by a hash that is unique to
        // a class.  Only a class's first list is kept; sorting the blocks by hash and list took five times as long (25 K blocks of a
        // RAT-SPN of 784 variables: 8.2 ms, now 1.7; pc_compile 9.1 -> 7.2 ms).
        std::unordered_map<uint64_t, int32_t> found;
        std::vector<std::pair<uint64_t, int32_t>> cls;    // hash, number in the order of first blocks
        std::vector<int32_t> at, at_ptr(1, 0), size, first, of(members.size());
        for (size_t i = 0; i < members.size(); ++i) {
            const int32_t u = members[i], b = at_ptr.back();
            uint64_t hash = 0;
            int32_t q = -1;
            for (int32_t k = par_ptr[u]; k < par_ptr[u + 1]; ++k)
                if (layer_of[par_of[k]] == li) at.push_back((par_of[k] + 1) * K);
            at.push_back(c->an_first_parent_depth[u] == T.depth ? -1 : -2);
            for (size_t k = b; k < at.size(); ++k) hash = (hash ^ (uint32_t)at[k]) * 0x9E3779B97F4A7C15ull;
            for (;; ++hash) {
                const auto it = found.try_emplace(hash, (int32_t)cls.size());
                q = it.first->second;
                if (it.second) {
                    cls.push_back({hash, q}); size.push_back(0); first.push_back(u);
                    at_ptr.push_back((int32_t)at.size());
                    break;
                }
                if (std::equal(at.begin() + at_ptr[q], at.begin() + at_ptr[q + 1], at.begin() + b, at.end())) { at.resize(b); break; }
            }
            of[i] = q;
            ++size[q];
            if (par_ptr[u + 1] - par_ptr[u] == at_ptr[q + 1] - 1 - at_ptr[q]) rep[u] = first[q];
        }
        if (2 * cls.size() > members.size()) continue;    // too few blocks share their parents
        std::sort(cls.begin(), cls.end());
        T.cls_ptr.assign(1, 0); T.cls_par_ptr.assign(1, 0);
        std::vector<int32_t> next(cls.size());
        for (const auto &hq : cls) {
            const int32_t q = hq.second, last = at_ptr[q + 1] - 1;
            next[q] = T.cls_ptr.back();
            T.cls_ptr.push_back(T.cls_ptr.back() + size[q]);
            T.cls_par.insert(T.cls_par.end(), at.begin() + at_ptr[q], at.begin() + last);
            T.cls_par_ptr.push_back((int32_t)T.cls_par.size());
            T.cls_first.push_back(at[last] == -1 ? 1 : 0);
        }
        T.cls_blk.resize(members.size());
        for (size_t i = 0; i < members.size(); ++i) T.cls_blk[next[of[i]]++] = (members[i] + 1) * K;
        compile_product_tiles(T, K, n);
    }
    for (int32_t id : c->layers[0].blk_ids) c->flow_rep.push_back((rep[id / K - 1] + 1) * K);
}

}  // namespace

// A dataflow task repeats its neighbours' products and exponentials for every 16 or 32 rows, so a layer that fills the chip is
// better off in the layer kernels; a narrow one costs them two launches and cold starts (5 + 5 us) where its tasks take
// 1.2 - 4 us.  Measured, with the kernels as they were when the lines were drawn, on hidden Chow-Liu trees (M = 32, 128, 256; B = 100 .. 512), HMMs and RAT-SPNs: the line lies at 2048
// tiles of 16 x 16 results (sum layer: forward, product layer: backward) and 16384 tile-chunks (16 x 16 results x 32 neighbour
// nodes) per layer, and half or twice that makes 5 % of a pass.  Product blocks of many children (RAT-SPN leaves: 57 - 98)
// are summed one child at a time by every task that reads them and belong in their own launch.
bool flow_narrow(const pc_circuit *c, size_t li, int64_t Bs)
{
    const LayerTab &t = c->layers[li];
    const int64_t ct = Bs / 16;
    if ((int64_t)t.blk_ids.size() * (c->K / 16) * ct > 2048) return false;
    return t.kind != KIND_SUM || (c->sum_edges[li] * (c->K / 16) * (c->K / 32) * ct <= 16384 && c->max_items[li] <= 12);
}

// What a layer gains from the dataflow launch, in us: a sum layer in the forward, a product layer in the backward pass.  The constants were
// set with earlier kernels; both sides below are measured with these, and the lines they draw stand, some us on the launches' side.
// Forward, a task takes the sum blocks among its products' children one after the other, each in 1.2 us and 0.12 us more per
// chunk of 32 neighbour nodes in the row; a layer's own two launches take 10.8 us.  Measured on a sum layer and a root that reads
// products of 5 / 6 / 7 / 8 / 10 / 12 sum blocks, B = 60, launches -> dataflow: rows of 4 chunks 22.2 -> 16.0, 21.8 -> 16.4, 22.2 -> 16.9, 23.4 ->
// 17.6, 23.9 -> 21.2, 23.2 -> 24.6 us (taken up to 8); of 16 chunks 25.4 -> 23.7, 26.9 -> 25.3, 27.0 -> 27.5, 27.5 -> 31.0, 32.1 -> 38.8, 33.3 ->
// 44.6 us; of 32 chunks 39.8 -> 44.1 us and more (none taken).  Many tiles take 7 ns each, whatever their rows: HMMs of 16 layers of one
// block, launches -> dataflow: 64 nodes, B = 1024 / 2048 / 4096 / 8192 (256 .. 2048 tiles a layer) 128 -> 46, 140 -> 72, 143 -> 124, 158 -> 232
// us (the last not taken), 128 nodes, B = 1024 / 2048 / 4096 (512 .. 2048 tiles) 154 -> 87, 162 -> 140, 193 -> 244 us (the last not taken).
// A chain of blocks of 32 (k_chain) has no such tasks, yet is priced by the same formula: 16 layers, B = 2048 / 8192 / 16384 / 32768 123 -> 26,
// 141 -> 38, 151 -> 56, 185 -> 96 us, of which the formula takes the first two.
// Backward, it takes the product parents of its sum blocks one after the other, each in 0.5 us and 0.06 us more per chunk, and
// what the workgroups do in all grows with tiles and waits; the launches take 11.5 us.  Measured on seven layers whose sum
// blocks feed 4 / 8 / 12 / 16 / 24 products, launches -> dataflow: one block of 32 nodes per layer, B = 30, 77 -> 37, 77 -> 46, 82 ->
// 59, 82 -> 69, 87 -> 91 us (taken up to 16), B = 300 108 -> 69, 109 -> 84, 117 -> 97, 125 -> 108, 131 -> 149 us (up to 8); four blocks of 32, B = 30, 77 ->
// 43, 83 -> 58, 95 -> 74, 93 -> 87, 100 -> 114 us (up to 8); one block of 128, B = 300, 204 -> 163, 216 -> 194, 225 -> 223, 237 -> 274 us (4).
static double flow_tiles(const pc_circuit *c, size_t li, int64_t Bs)
{
    return (double)((int64_t)c->layers[li].blk_ids.size() * (c->K / 16) * (Bs / 16));
}
static double flow_load(const pc_circuit *c, size_t li, int64_t Bs) { return flow_tiles(c, li, Bs) * (1 + c->flow_waits[li] / 8.0); }
double flow_gain(const pc_circuit *c, size_t li, int64_t Bs)
{
    const double waits = c->flow_waits[li], chunks = c->flow_chunks[li], load = flow_load(c, li, Bs);
    if (c->layers[li].kind == KIND_SUM) return 10.8 - std::max(std::max(waits, 1.0) * (1.2 + 0.12 * chunks), 0.007 * flow_tiles(c, li, Bs));
    return 11.5 - std::max(2 + waits * (0.5 + 0.06 * chunks) + 0.003 * load, 0.007 * load);
}
// The first layer of the launch finds neither weights nor values requested ahead.  Forward passes of 3 x 64 and 3 x 128 HMMs, 1024 tiles a
// layer, launches -> dataflow 30.7 -> 35.8 and 42.0 -> 48.6 us, half the tiles 29.0 -> 23.7 and 39.8 -> 36.3 (taken); backward passes 771 -> 774 and
// 886 -> 888, where the layers' gain alone would be 20 us.  With earlier kernels the backward pass of a RAT-SPN's root over 256 product blocks of
// 32 nodes, B = 16 (1024 tiles): 90 us in launches, 100 as dataflow.
double flow_start_up(const pc_circuit *c, size_t li, int64_t Bs)
{
    return c->layers[li].kind == KIND_PRODUCT ? 0.04 * flow_load(c, li, Bs) : 0.012 * flow_tiles(c, li, Bs);
}

pc_status compile_host(const pc_dag *d, pc_circuit *c, bool tables_on_host)
{
    if (!d) return fail(PC_ERR_ARG, "dag is NULL");
    if (d->K < 1 || d->n_blocks < 1) return fail(PC_ERR_ARG, "K and n_blocks must be positive");
    if (!d->type || !d->n_real || !d->child_ptr || !d->in_var || !d->in_table)
        return fail(PC_ERR_ARG, "a dag array is NULL");
    const int32_t n = d->n_blocks, K = d->K;
    const int64_t n_edges = d->child_ptr[n];
    if (d->child_ptr[0] != 0 || n_edges < 0) return fail(PC_ERR_ARG, "child_ptr must start at 0");
    if (n_edges > 0 && (!d->child || !d->param_blk)) return fail(PC_ERR_ARG, "child / param_blk is NULL");
    if (d->root_block < 0 || d->root_block >= n || d->type[d->root_block] != KIND_SUM)
        return fail(PC_ERR_ARG, "root_block must name a sum block");
    if (d->n_param_blocks < 0 || d->n_vars < 1 || d->n_cats < 1 || d->n_tables < 1)
        return fail(PC_ERR_ARG, "n_param_blocks / n_vars / n_cats / n_tables out of range");
    if ((int64_t)(n + 1) * K > std::numeric_limits<int32_t>::max())
        return fail(PC_ERR_TOO_LARGE, "node offsets exceed int32");
    if (((int64_t)d->n_param_blocks + 1) * K * K > std::numeric_limits<int32_t>::max())
        return fail(PC_ERR_TOO_LARGE, "parameter offsets exceed int32");
    if ((int64_t)d->n_tables * d->n_cats > std::numeric_limits<int32_t>::max())
        return fail(PC_ERR_TOO_LARGE, "categorical table rows exceed int32");
    if (K > 128) return fail(PC_ERR_ARG, "block sizes above 128 are not supported");

    for (int32_t u = 0; u < n; ++u) {
        if (d->type[u] > KIND_SUM) return fail(PC_ERR_ARG, "unknown block type");
        if (d->n_real[u] < 1 || d->n_real[u] > K) return fail(PC_ERR_ARG, "n_real out of range");
        const int64_t e0 = d->child_ptr[u], e1 = d->child_ptr[u + 1];
        if (e1 < e0) return fail(PC_ERR_ARG, "child_ptr not monotone");
        if (d->type[u] == KIND_INPUT) {
            if (e1 != e0) return fail(PC_ERR_NOT_ALTERNATING, "input block with children");
            if (d->in_var[u] < 0 || d->in_var[u] >= d->n_vars) return fail(PC_ERR_ARG, "in_var out of range");
            if (d->in_table[u] < 0 || d->in_table[u] >= d->n_tables) return fail(PC_ERR_ARG, "in_table out of range");
            continue;
        }
        if (e1 == e0) return fail(PC_ERR_NOT_BLOCK_SPARSE, "inner block without children");
        std::vector<int32_t> seen;
        for (int64_t e = e0; e < e1; ++e) {
            const int32_t ch = d->child[e];
            if (ch < 0 || ch >= n) return fail(PC_ERR_ARG, "child id out of range");
            if (d->type[u] == KIND_SUM) {
                if (d->type[ch] != KIND_PRODUCT) return fail(PC_ERR_NOT_ALTERNATING, "sum block with a non-product child");
                if (d->param_blk[e] < 0 || d->param_blk[e] >= d->n_param_blocks)
                    return fail(PC_ERR_ARG, "param_blk out of range");
            } else if (d->type[ch] == KIND_PRODUCT) {
                return fail(PC_ERR_NOT_ALTERNATING, "product block with a product child");
            }
            seen.push_back(ch);
        }
        std::sort(seen.begin(), seen.end());
        if (std::adjacent_find(seen.begin(), seen.end()) != seen.end())
            return fail(PC_ERR_NOT_BLOCK_SPARSE, "duplicate (parent, child) block pair");
    }

    // Longest-path depth by peeling blocks whose children are all done (also detects cycles).
    std::vector<int32_t> depth(n, 0), pending(n, 0), par_ptr(n + 1, 0);
    for (int64_t e = 0; e < n_edges; ++e) ++par_ptr[d->child[e] + 1];
    for (int32_t u = 0; u < n; ++u) par_ptr[u + 1] += par_ptr[u];
    std::vector<int32_t> par_of(n_edges), fill(par_ptr.begin(), par_ptr.end() - 1);
    std::vector<int64_t> par_edge(n_edges);
    for (int32_t u = 0; u < n; ++u)
        for (int64_t e = d->child_ptr[u]; e < d->child_ptr[u + 1]; ++e) {
            const int32_t at = fill[d->child[e]]++;
            par_of[at] = u;
            par_edge[at] = e;
        }
    std::vector<int32_t> ready;
    for (int32_t u = 0; u < n; ++u) {
        pending[u] = (int32_t)(d->child_ptr[u + 1] - d->child_ptr[u]);
        if (pending[u] == 0) ready.push_back(u);
    }
    int32_t done = 0, max_depth = 0;
    while (!ready.empty()) {
        const int32_t u = ready.back();
        ready.pop_back();
        ++done;
        max_depth = std::max(max_depth, depth[u]);
        for (int32_t k = par_ptr[u]; k < par_ptr[u + 1]; ++k) {
            const int32_t p = par_of[k];
            depth[p] = std::max(depth[p], depth[u] + 1);
            if (--pending[p] == 0) ready.push_back(p);
        }
    }
    if (done != n) return fail(PC_ERR_CYCLE, "the block graph has a cycle");

    if (par_ptr[d->root_block + 1] != par_ptr[d->root_block]) return fail(PC_ERR_ARG, "the root block must not have parents");
    // Product-scratch mode (Sec. 5): a product block is evaluated as late as possible -- in the layer right before the
    // sum blocks that read it (all of one depth) -- so that a product layer is read by the next sum layer only and its
    // values can share one scratch.  Product blocks nobody reads form a last layer of their own.
    c->product_scratch = d->product_scratch != 0;
    if (c->product_scratch) {
        bool orphan = false;
        for (int32_t u = 0; u < n; ++u) {
            if (d->type[u] != KIND_PRODUCT) continue;
            if (par_ptr[u] == par_ptr[u + 1]) { orphan = true; continue; }
            const int32_t ds = depth[par_of[par_ptr[u]]];
            for (int32_t k = par_ptr[u]; k < par_ptr[u + 1]; ++k)
                if (depth[par_of[k]] != ds) return fail(PC_ERR_ARG, "product_scratch: a product block is read by sum blocks of different depths");
            depth[u] = ds;
        }
        if (orphan) {
            for (int32_t u = 0; u < n; ++u)
                if (d->type[u] == KIND_PRODUCT && par_ptr[u] == par_ptr[u + 1]) depth[u] = max_depth + 1;
            max_depth += 1;
        }
    }
    // per block: the smallest and the largest depth among its parents (the last and the first layer of the
    // backward sweep that feed it; all parents of a block are of one kind, so a depth names one layer)
    std::vector<int32_t> last_parent_depth(n, -1), first_parent_depth(n, -1);
    for (int32_t u = 0; u < n; ++u)
        for (int32_t k = par_ptr[u]; k < par_ptr[u + 1]; ++k) {
            const int32_t dp = depth[par_of[k]];
            if (last_parent_depth[u] < 0 || dp < last_parent_depth[u]) last_parent_depth[u] = dp;
            if (dp > first_parent_depth[u]) first_parent_depth[u] = dp;
        }
    // blocks no layer of the backward sweep writes: sum blocks as node offsets (flow and log_nf initialised),
    // other blocks and the null block as ~offset (flow zeroed only)
    c->init_ids.clear();
    c->init_ids.push_back(~0);
    // (product-scratch mode: product blocks nobody reads are the last layer; their window is cleared when the backward
    // sweep reaches it, and their rows do not exist in the flow buffer)
    for (int32_t u = 0; u < n; ++u)
        if (last_parent_depth[u] < 0 && !(c->product_scratch && d->type[u] == KIND_PRODUCT))
            c->init_ids.push_back(d->type[u] == KIND_SUM ? (u + 1) * K : ~((u + 1) * K));

    c->K = K; c->n_blocks = n; c->root_block = d->root_block; c->n_param_blocks = d->n_param_blocks;
    c->n_vars = d->n_vars; c->n_cats = d->n_cats; c->n_tables = d->n_tables;
    c->layers.clear();
    c->an_depth = depth;                                  // kept for the device table builder
    c->an_last_parent_depth = last_parent_depth;
    c->an_first_parent_depth = first_parent_depth;

    // bucket blocks: layer key = 2*depth + (sum ? 1 : 0); inputs are layer 0
    std::vector<std::vector<int32_t>> bucket(2 * (size_t)max_depth + 2);      // max_depth includes the layer of unread products
    for (int32_t u = 0; u < n; ++u) {
        const size_t key = d->type[u] == KIND_INPUT ? 0 : 2 * (size_t)depth[u] + (d->type[u] == KIND_SUM ? 1 : 0);
        bucket[key].push_back(u);
    }
    for (size_t key = 0; key < bucket.size(); ++key) {
        const std::vector<int32_t> &blocks = bucket[key];
        if (blocks.empty()) continue;
        LayerTab layer;
        layer.kind = key == 0 ? KIND_INPUT : d->type[blocks[0]];
        layer.depth = key == 0 ? 0 : depth[blocks[0]];
        for (int32_t u : blocks) {
            layer.blk_ids.push_back((u + 1) * K);
            if (u == d->root_block) c->root_layer = (int32_t)c->layers.size();
        }
        if (layer.kind == KIND_INPUT) {
            GroupTab g;
            g.n_rows = (int32_t)blocks.size();
            g.width = 1;
            for (int32_t u : blocks) {
                g.ids.push_back((u + 1) * K);
                g.nbr.push_back(d->in_var[u]);
                g.par.push_back(d->in_table[u]);
            }
            std::vector<int32_t> tabs = g.par;                          // a table shared by several blocks: flows collide
            std::sort(tabs.begin(), tabs.end());
            g.tied_in_group = std::adjacent_find(tabs.begin(), tabs.end()) != tabs.end();
            layer.fwd.push_back(std::move(g));
        } else if (tables_on_host) {
            std::vector<Row> fwd_rows;
            std::map<int32_t, Row> by_child;                       // ordered: ascending child block id
            for (int32_t u : blocks) {
                Row r;
                r.id = (int64_t)(u + 1) * K;
                for (int64_t e = d->child_ptr[u]; e < d->child_ptr[u + 1]; ++e) {
                    const int32_t ch = d->child[e];
                    const int64_t p = layer.kind == KIND_SUM ? ((int64_t)d->param_blk[e] + 1) * K * K : 0;
                    r.nbrs.emplace_back((int64_t)(ch + 1) * K, p);
                    Row &br = by_child[ch];
                    br.id = (int64_t)(ch + 1) * K;
                    br.nbrs.emplace_back(r.id, p);
                }
                fwd_rows.push_back(std::move(r));
            }
            std::vector<Row> bwd_rows;
            for (auto &kv : by_child) bwd_rows.push_back(std::move(kv.second));
            pc_status st = build_groups(fwd_rows, d->max_groups, d->tol_permille, layer.fwd);
            if (st != PC_OK) return st;
            st = build_groups(bwd_rows, d->max_groups, d->tol_permille, layer.bwd);
            if (st != PC_OK) return st;
            for (GroupTab &gt : layer.bwd)
                for (size_t i = 0; i < gt.ids.size(); ++i) {
                    const int32_t ch = gt.ids[i] / K - 1;
                    gt.aux[i] |= bwd_row_flags(layer.kind, d->type[ch], layer.depth, last_parent_depth[ch],
                                               first_parent_depth[ch]);
                }
        }
        if (c->product_scratch && layer.kind == KIND_PRODUCT) {
            layer.scr_first_block = blocks.front();
            if (blocks.back() - blocks.front() + 1 != (int32_t)blocks.size())
                return fail(PC_ERR_ARG, "product_scratch: the product blocks of a layer must have consecutive ids (pc_order_for_scratch)");
            c->max_window_blocks = std::max(c->max_window_blocks, (int32_t)blocks.size());
        }
        c->layers.push_back(std::move(layer));
    }
    if (c->product_scratch) {
        // input and sum blocks first, product blocks behind them; every sum layer reads the product layer before it
        c->n_persistent_blocks = 0;
        for (int32_t u = 0; u < n; ++u) if (d->type[u] != KIND_PRODUCT) ++c->n_persistent_blocks;
        for (int32_t u = 0; u < n; ++u)
            if ((d->type[u] == KIND_PRODUCT) != (u >= c->n_persistent_blocks))
                return fail(PC_ERR_ARG, "product_scratch: input and sum blocks must come before the product blocks (pc_order_for_scratch)");
        std::vector<int32_t> layer_of(n, 0);
        for (size_t li = 0; li < c->layers.size(); ++li)
            for (int32_t id : c->layers[li].blk_ids) layer_of[id / K - 1] = (int32_t)li;
        for (size_t li = 0; li < c->layers.size(); ++li) {
            LayerTab &L = c->layers[li];
            if (L.kind != KIND_SUM) continue;
            std::map<int32_t, std::vector<std::pair<int32_t, int32_t>>> users;        // parameter block -> pairs of this layer
            for (int32_t id : L.blk_ids) {
                const int32_t u = id / K - 1;
                for (int64_t e = d->child_ptr[u]; e < d->child_ptr[u + 1]; ++e) {
                    if (layer_of[d->child[e]] != (int32_t)li - 1) return fail(PC_ERR_ARG, "product_scratch: a sum layer must read the product layer before it");
                    users[d->param_blk[e]].emplace_back(id, (d->child[e] + 1) * K);
                }
            }
            L.pf_ptr.assign(1, 0);
            for (auto &kv : users) {
                L.pf_pb.push_back((kv.first + 1) * K * K);
                for (auto &sc : kv.second) { L.pf_sum.push_back(sc.first); L.pf_child.push_back(sc.second); }
                L.pf_ptr.push_back((int32_t)L.pf_sum.size());
            }
        }
    }

    // EM normalisation map.  A sum node's weights span all parameter blocks of its block's edges;
    // tied sum blocks must share that whole list (else the normalisation is ill defined).
    const int32_t P = d->n_param_blocks;
    c->pb_group.assign(P + 1, -1);
    c->pb_rows.assign(P + 1, 0);
    c->pb_cols.assign(P + 1, 0);
    c->group_nch.clear();
    std::vector<std::vector<int32_t>> group_list;
    for (int32_t u = 0; u < n; ++u) {
        if (d->type[u] != KIND_SUM) continue;
        std::vector<int32_t> list;
        int32_t nch = 0;
        for (int64_t e = d->child_ptr[u]; e < d->child_ptr[u + 1]; ++e) {
            list.push_back(d->param_blk[e]);
            nch += d->n_real[d->child[e]];
        }
        std::vector<int32_t> sorted = list;
        std::sort(sorted.begin(), sorted.end());
        if (std::adjacent_find(sorted.begin(), sorted.end()) != sorted.end())
            return fail(PC_ERR_TIE, "a sum block uses one parameter block for two children");
        const int32_t g0 = c->pb_group[list[0] + 1];
        if (g0 < 0) {
            for (int32_t p : list)
                if (c->pb_group[p + 1] >= 0) return fail(PC_ERR_TIE, "sum blocks share only part of their parameter blocks");
            const int32_t g = (int32_t)group_list.size();
            size_t k = 0;
            for (int64_t e = d->child_ptr[u]; e < d->child_ptr[u + 1]; ++e, ++k) {
                c->pb_group[list[k] + 1] = g;
                c->pb_rows[list[k] + 1] = d->n_real[u];
                c->pb_cols[list[k] + 1] = d->n_real[d->child[e]];
            }
            group_list.push_back(list);
            c->group_nch.push_back(nch);
        } else {
            if (group_list[g0] != list) return fail(PC_ERR_TIE, "sum blocks share only part of their parameter blocks");
            size_t k = 0;
            for (int64_t e = d->child_ptr[u]; e < d->child_ptr[u + 1]; ++e, ++k)
                if (c->pb_rows[list[k] + 1] != d->n_real[u] || c->pb_cols[list[k] + 1] != d->n_real[d->child[e]])
                    return fail(PC_ERR_TIE, "tied parameter blocks with different numbers of real nodes");
        }
    }
    // Parameter blocks of every group of short rows, then one group without rows per block that no sum block uses and for the
    // padding block: the EM kernel only clears their flows.  Rows of more than 2048 accesses (k_em_theta) go in segments of 256
    // accesses, at most 1024 of them, so that they are as many waves' work: one wave takes 26 us for a row of 2048, 104 us for 8000
    // and 1.5 ms for 80 000; in segments 16 and 40 us.  Shorter rows would only pay the two launches (a RAT-SPN's EM step, whose
    // root has 2048 accesses beside 0.7 ms of other rows' work: 769 -> 778 us).
    const int32_t row_acc = (K & 3) == 0 ? K / 4 : K;
    auto is_long = [&](const std::vector<int32_t> &list) { return (int64_t)list.size() * row_acc > 2048; };
    c->em_ptr.assign(1, 0);
    c->em_list.clear();
    std::vector<int32_t> nch_of = std::move(c->group_nch);
    c->group_nch.clear();
    for (size_t g = 0; g < group_list.size(); ++g) {
        if (is_long(group_list[g])) continue;
        for (int32_t p : group_list[g]) c->em_list.push_back(p + 1);
        c->em_ptr.push_back((int32_t)c->em_list.size());
        c->group_nch.push_back(nch_of[g]);
    }
    c->n_em_groups = (int32_t)c->group_nch.size();
    for (int32_t p = 0; p <= P; ++p)
        if (c->pb_group[p] < 0) { c->em_list.push_back(p); c->em_ptr.push_back((int32_t)c->em_list.size()); }
    c->em_seg_ptr.assign(1, (int32_t)c->em_list.size());
    c->em_seg.clear();
    for (size_t g = 0; g < group_list.size(); ++g) {
        const std::vector<int32_t> &list = group_list[g];
        if (!is_long(list)) continue;
        const size_t len = std::max<size_t>(256 / row_acc, (list.size() + 1023) / 1024);
        const int32_t first = (int32_t)c->em_seg_ptr.size() - 1, n_seg = (int32_t)((list.size() + len - 1) / len);
        for (size_t k = 0; k < list.size(); ++k) {
            c->em_list.push_back(list[k] + 1);
            if (k % len == len - 1 || k + 1 == list.size()) {
                c->em_seg_ptr.push_back((int32_t)c->em_list.size());
                c->em_seg.insert(c->em_seg.end(), {first, n_seg, nch_of[g]});
            }
        }
    }

    // Parameter-centric flow tables (App. A.3): every (sum block, child block) pair that uses a parameter
    // block, so that the flows of tied edges are reduced together; pairs in ascending sum-block order.
    std::vector<std::vector<std::pair<int32_t, int32_t>>> users(P);
    for (int32_t u = 0; u < n; ++u) {
        if (d->type[u] != KIND_SUM) continue;
        for (int64_t e = d->child_ptr[u]; e < d->child_ptr[u + 1]; ++e)
            users[d->param_blk[e]].emplace_back((u + 1) * K, (d->child[e] + 1) * K);
    }
    c->pf_pb.clear(); c->pf_ptr.assign(1, 0); c->pf_sum.clear(); c->pf_child.clear();
    for (int32_t p = 0; p < P; ++p) {
        if (users[p].empty()) continue;
        c->pf_pb.push_back((p + 1) * K * K);
        for (auto &sc : users[p]) { c->pf_sum.push_back(sc.first); c->pf_child.push_back(sc.second); }
        c->pf_ptr.push_back((int32_t)c->pf_sum.size());
    }
    if (!c->product_scratch && (K == 32 || K == 64 || K == 128)) compile_flow(d, c, par_ptr, par_of, par_edge);
    if (!c->product_scratch) compile_classes(d, c, par_ptr, par_of);
    return PC_OK;
}

}  // namespace pc
