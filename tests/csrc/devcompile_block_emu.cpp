// CPU run of the device tree compiler's other two passes (the steps of
// paper_2205_03251_amd/csrc/devcompile_core.h that k_dc_up_block, k_dc_up_walk
// and the emission by a thread per node run), checked tree by tree against
// compile_tree: code words, parents, inputs, node counts, STORE flags, stack
// bound and the index of large subtrees.
//
// Blocks of `span` positions (small ones, so that most trees leave theirs) are
// finished in a random order, each by its terminals' walks in a random
// interleaving; then the listed walks go on, interleaved at random, also
// between a walk's look at its parent's slot and the atomic that follows.
// Emission runs chunks and nodes in random orders.
//
// Input (stdin, text): vtype n_inputs chunk_nodes index_min_size n_trees seed
// span n_records, n_trees + 1 offsets, the ops bytes, and n_records points as
// (tree, node) pairs in tree order.  Output: "ok chunks <n> listed <l> between
// <b>", or a line naming the first difference (exit status 1).
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <random>
#include <string>
#include <vector>

#include "../../paper_2205_03251_amd/csrc/devcompile_core.h"

using namespace gpe;

namespace {

std::function<void()> g_between;               // runs other walks inside a look at a slot

struct CpuMem {
    static int32_t ld(const int32_t* p)
    {
        const int32_t v = *p;
        if (g_between) g_between();
        return v;
    }
    static void st(int32_t* p, int32_t v) { *p = v; }
    static uint64_t fetch_or64(uint64_t* p, uint64_t v)
    {
        const uint64_t o = *p;
        *p = o | v;
        return o;
    }
    static void err(int32_t* p, int32_t v) { *p |= v; }
    static uint32_t exchange(uint32_t* p, uint32_t v)
    {
        std::swap(*p, v);
        return v;
    }
    static void fetch_or(uint32_t* p, uint32_t v) { *p |= v; }
    static void add(uint32_t* p, uint32_t v) { *p += v; }
};

[[noreturn]] void fail(const std::string& what)
{
    std::printf("mismatch: %s\n", what.c_str());
    std::exit(1);
}

template <class T> T rd()
{
    long long v;
    if (std::scanf("%lld", &v) != 1) fail("short input");
    return (T)v;
}

}  // namespace

int main()
{
    const int vtype = rd<int>(), n_inputs = rd<int>();
    const int64_t C = rd<int64_t>(), index_min = rd<int64_t>(), n_trees = rd<int64_t>();
    std::mt19937_64 rng(rd<uint64_t>());
    const int64_t span = rd<int64_t>(), n_pts = rd<int64_t>();
    if (C > kDcPackMaxC || span < 1 || span > 4096) fail("chunk target or span out of range");
    std::vector<int64_t> off(n_trees + 1);
    for (auto& v : off) v = rd<int64_t>();
    const int64_t n = off[n_trees];
    std::vector<uint8_t> ops(n);
    for (auto& v : ops) v = rd<uint8_t>();
    std::vector<std::vector<int64_t>> pts(n_trees);
    for (int64_t i = 0; i < n_pts; ++i) {
        const int64_t t = rd<int64_t>();
        pts[t].push_back(rd<int64_t>());
    }

    std::vector<int32_t> endl(n), parl(n);
    for (int64_t t = 0; t < n_trees; ++t) {
        const int64_t s = off[t];
        std::vector<int32_t> st;
        for (int64_t i = off[t + 1] - s - 1; i >= 0; --i) {
            endl[s + i] = (int32_t)(i + 1);
            if (ops[s + i] & kFuncBit) {
                const int32_t l = st.back(), r = st[st.size() - 2];
                st.resize(st.size() - 2);
                endl[s + i] = endl[s + r];
                parl[s + l] = parl[s + r] = (int32_t)i;
            }
            st.push_back((int32_t)i);
        }
        parl[s] = -1;
    }
    std::vector<int32_t> info(n, -7), len(n, -7), rec;
    std::vector<uint8_t> ncut(n, 0), big(n, 7);
    std::vector<uint64_t> slot64(n, 0);
    int32_t err = 0;
    DcNodes q{};
    q.ops = ops.data();
    q.offsets = off.data();
    q.n_trees = n_trees;
    q.n = n;
    q.endl = endl.data();
    q.parl = parl.data();
    q.info = info.data();
    q.len = len.data();
    q.slot64 = slot64.data();
    q.ncut = ncut.data();
    q.big = index_min > 0 ? big.data() : nullptr;
    q.big_min = index_min;
    q.err = &err;
    q.boolean = vtype == 1;
    q.S = 10;
    q.C = std::max<int64_t>(2, C);

    // blocks
    struct Walk {
        int64_t v, s;
        int32_t p;
        uint32_t w;
    };
    std::vector<Walk> listed;
    std::vector<int64_t> blocks;
    for (int64_t b = 0; b < n; b += span) blocks.push_back(b);
    std::shuffle(blocks.begin(), blocks.end(), rng);
    for (int64_t base : blocks) {
        const int64_t end = std::min(n, base + span);
        std::vector<uint32_t> word(end - base, 0);
        std::vector<uint16_t> par(end - base), rgt(end - base);
        for (int64_t v = base; v < end; ++v) {
            const int64_t s = off[dc_tree_of(q, v)];
            dc_block_node(q, s, v, base, end, &par[v - base], &rgt[v - base]);
        }
        const DcBlock blk{word.data(), par.data(), rgt.data()};
        std::vector<std::pair<int, uint32_t>> th;
        for (int64_t v = base; v < end; ++v)
            if (!(ops[v] & kFuncBit)) {
                word[v - base] = kDcBlockLeaf;
                th.push_back({(int)(v - base), dc_leaf_word(dc_foldable_op(q, ops[v]))});
            }
        while (!th.empty()) {
            const size_t i = (size_t)(rng() % th.size());
            const int at = dc_block_step<CpuMem>(q, blk, base, th[i].first, &th[i].second);
            if (at >= 0) {
                th[i].first = at;
                continue;
            }
            if (at == -2) {
                const int64_t v = base + th[i].first;
                listed.push_back(Walk{v, off[dc_tree_of(q, v)], parl[v], th[i].second});
            }
            th[i] = th.back();
            th.pop_back();
        }
        for (int64_t v = base; v < end; ++v)
            if (!(ops[v] & kFuncBit) || rgt[v - base] != kDcOutside)
                dc_block_result(q, v, word[v - base],
                                (ops[v] & kFuncBit) && off[dc_tree_of(q, v)] + endl[v] - v >= index_min);
    }
    const size_t n_listed = listed.size();

    // walks; a walk that is taken up runs alone in `listed`'s place until its step is done
    long between = 0;
    std::function<void()> one = [&]() {
        const size_t i = (size_t)(rng() % listed.size());
        Walk x = listed[i];
        listed[i] = listed.back();
        listed.pop_back();
        x.v = dc_walk_step<CpuMem>(q, x.s, x.v, &x.p, &x.w);
        if (x.v >= 0 && x.p >= 0) listed.push_back(x);
    };
    for (size_t i = 0; i < listed.size();) {
        if (listed[i].p < 0) {
            listed[i] = listed.back();
            listed.pop_back();
        } else {
            ++i;
        }
    }
    int depth = 0;
    g_between = [&]() {
        if (listed.empty() || depth >= 3 || rng() % 2) return;
        ++depth;
        for (int k = (int)(rng() % 4); k > 0 && !listed.empty(); --k, ++between) one();
        --depth;
    };
    while (!listed.empty()) one();
    g_between = nullptr;
    if (err) fail("inconsistent index " + std::to_string(err));
    for (int64_t g = 0; g < n; ++g)
        if (info[g] < 0) fail("node " + std::to_string(g) + " never finished");

    // records, as the host compiler numbers them, and the STORE words' lengths
    CompileOptions opt;
    opt.vtype = vtype;
    opt.n_inputs = n_inputs;
    opt.chunk_nodes = C;
    opt.stack_slots = 10;
    opt.index_min_size = index_min;
    std::vector<TreeProg> want(n_trees);
    std::vector<DcStored> stored;
    for (int64_t t = 0; t < n_trees; ++t) {
        const int64_t s = off[t], np = (int64_t)pts[t].size();
        std::string why;
        if (!compile_tree(ops.data() + s, off[t + 1] - s, opt, pts[t].data(), np, &want[t], &why)) fail(why);
        std::vector<int64_t> lv_off(np + 1, 0);
        std::vector<DcPathLevel> lv;
        std::vector<uint8_t> pop(np);
        std::vector<int32_t> pend(np);
        for (int64_t p = 0; p < np; ++p) {
            int32_t below = (int32_t)pts[t][p];
            pop[p] = ops[s + below];
            pend[p] = endl[s + below];
            for (int32_t a = parl[s + below]; a >= 0; below = a, a = parl[s + a]) {
                const int32_t l = a + 1, r = endl[s + l], sib = below != l ? l : r;
                lv.push_back(DcPathLevel{a, sib, (ops[s + a] & 3) | (below != l ? 4 : 0), ops[s + sib]});
            }
            lv_off[p + 1] = (int64_t)lv.size();
        }
        std::vector<Spine> spines;
        dc_tree_records(s, np, pts[t].data(), pop.data(), pend.data(), lv_off.data(), lv.data(), &spines, &stored);
    }
    if (!stored.empty()) {
        std::vector<uint8_t> cut(stored.size());
        for (size_t i = 0; i < stored.size(); ++i) cut[i] = dc_cut(q, stored[i].node) ? 1 : 0;
        std::vector<int32_t> inc(stored.size());
        dc_store_words(stored.data(), cut.data(), stored.size(), inc.data());
        rec.assign(n, -1);
        for (size_t i = 0; i < stored.size(); ++i) {
            len[stored[i].node] += inc[i];
            rec[stored[i].node] = stored[i].rec;
        }
        q.rec = rec.data();
    }

    // chunk roots, the chunk graph
    std::vector<int64_t> roots, root, tstart, cbase;
    for (int64_t g = 0; g < n; ++g)
        if (dc_finish(q, g)) roots.push_back(g);
    std::vector<int32_t> ctree, ids;
    if (!dc_number_chunks(roots, off.data(), n_trees, &root, &tstart, &ctree, &ids, &cbase))
        fail("a tree without its root chunk");
    const int64_t nch = (int64_t)root.size();
    std::vector<int64_t> key(nch), end(nch), code_off(nch + 1, 0), nodes(nch), in_off;
    std::vector<int32_t> rend(nch), parent(nch, -1), load_idx(nch, -1), inputs;
    for (int64_t j = 0; j < nch; ++j) key[j] = dc_load_key(q, roots[j], off[dc_tree_of(q, roots[j])]);
    for (int64_t k = 0; k < nch; ++k) {
        rend[k] = endl[root[k]];
        end[k] = tstart[k] + rend[k];
        code_off[k + 1] = code_off[k] + len[root[k]] + 1;
    }
    if (!dc_chunk_graph(roots, ids, rend, root, tstart, key, &parent, &load_idx, &nodes, &in_off, &inputs))
        fail("inconsistent chunk graph");

    // emission by a thread per node
    std::vector<uint32_t> place(n, 0), id(n, 0), frame(nch), code(code_off[nch] + 1, 0xdeadbeefu);
    std::vector<int32_t> max_slot(nch, -9);
    std::vector<uint8_t> stores(nch, 9);
    for (int64_t g = 0; g < n; ++g) dc_add_place_steps<CpuMem>(q, g, place.data());
    for (int64_t k = 0; k < nch; ++k) dc_add_id_steps<CpuMem>(n, k, root[k], end[k], parent[k], id.data());
    for (int64_t g = 1; g < n; ++g) {
        place[g] += place[g - 1];
        id[g] += id[g - 1];
    }
    DcChunks ck{};
    ck.n = nch;
    ck.root = root.data();
    ck.code_off = code_off.data();
    ck.code = code.data();
    ck.parent = parent.data();
    ck.load_idx = load_idx.data();
    ck.max_slot = max_slot.data();
    ck.stores = stores.data();
    std::vector<int64_t> order(std::max(n, nch));
    for (size_t i = 0; i < order.size(); ++i) order[i] = (int64_t)i;
    std::shuffle(order.begin(), order.end(), rng);
    for (int64_t k : order)
        if (k < nch) dc_emit_chunk(q, ck, place.data(), k, frame.data());
    std::shuffle(order.begin(), order.end(), rng);
    for (int64_t g : order)
        if (g < n) dc_emit_node(q, ck, place.data(), id.data(), frame.data(), g);

    for (int64_t t = 0; t < n_trees; ++t) {
        const int64_t s = off[t], b = cbase[t], nc = cbase[t + 1] - b;
        const TreeProg& h = want[t];
        const std::string T = "tree " + std::to_string(t) + ": ";
        if ((int64_t)h.chunks.size() != nc) fail(T + "chunks");
        int32_t ms = 0;
        for (int64_t i = 0; i < nc; ++i) {
            const int64_t k = b + i;
            const Chunk& c = h.chunks[i];
            const std::string K = T + "chunk " + std::to_string(i) + ": ";
            if ((parent[k] >= 0 ? parent[k] - (int32_t)b : -1) != c.parent) fail(K + "parent");
            if (root[k] - s != c.root_node || nodes[k] != c.nodes) fail(K + "root or nodes");
            if ((stores[k] != 0) != c.stores || stores[k] > 1) fail(K + "stores");
            if (code_off[k + 1] - code_off[k] != c.code_len) fail(K + "code length");
            for (int64_t w = 0; w < c.code_len; ++w)
                if (code[code_off[k] + w] != h.code[c.code_off + w]) fail(K + "word " + std::to_string(w));
            if (in_off[k + 1] - in_off[k] != (int64_t)c.inputs.size()) fail(K + "input count");
            for (size_t j = 0; j < c.inputs.size(); ++j)
                if (inputs[in_off[k] + (int64_t)j] - (int32_t)b != c.inputs[j]) fail(K + "input " + std::to_string(j));
            ms = std::max(ms, max_slot[k] + 1);
        }
        if (ms != h.max_stack) fail(T + "max stack");
        if (index_min > 0) {
            std::vector<SubtreeEnd> bl;
            for (int64_t i = s; i < off[t + 1]; ++i) {
                if (big[i] > 1) fail(T + "large-subtree flag never written");
                if (big[i]) bl.push_back({(int32_t)(i - s), endl[i]});
            }
            if (bl != h.big_ends) fail(T + "large subtrees");
        }
    }
    std::printf("ok chunks %lld listed %zu between %ld\n", (long long)nch, n_listed, between);
    return 0;
}
