// Host-side retrieval drafter over the short-term context (Section 4.2; Algorithm 2 with the
// trie as the only structure): an n-gram trie with continuation counts, the greedy search path,
// and the depth-first extraction of a draft tree.  Plain C++ on host memory; no GPU involved.
// It produces the token / parent arrays that the verification step takes.
//
// What bounds it is finding a node's child: a prompt of 4096 tokens in a trie of depth 8 takes 32768 lookups.  Nodes are
// therefore plain records in one array, linked to their siblings by number, and the n-grams of a text are followed by where
// they end, not by where they begin, so that the lookups of one token (one per n-gram length) do not wait for each other.
// Of the 17 to 18 thousand nodes of such a trie 3.4 have no child and 13.3 a single one, which its parent leads to: only
// the children of nodes with two or more are in a table (one for all, open addressing, 8 bytes per slot).  Measured on one
// core: one request (prompt of 4096 tokens, 64 draft trees and search paths) 222 to 227 us, 351 when every edge had a slot, 2560
// with a hash map of edges and a vector of children per node, walked n-gram by n-gram; 65536 tokens of text that repeats
// little inserted in 7.8 ms, 40 when every edge had a slot.
#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <new>
#include <vector>

#include "reader.h"

struct reader_trie {
    struct Node {
        int32_t token;
        int32_t count;                    // how often the n-gram that ends here was seen
        int32_t parent;
        int32_t newest;                   // child created last (0: none; the root is nobody's child)
        int32_t older;                    // sibling created before this one (0: none)
    };
    struct Slot {
        int32_t token;
        int32_t child;                    // 0: free
    };
    int32_t max_depth;
    std::vector<Node> nodes;              // nodes[0] is the root (empty n-gram)
    std::vector<Slot> slots;              // edges (parent, token) -> child of nodes with several; a power of two of them, at most three quarters in use
    size_t used = 0;                      // slots in use
    int shift;                            // 64 - log2(slots)

    size_t slot_of(int32_t node, int32_t token) const {
        const uint64_t key = ((uint64_t)(uint32_t)node << 32) | (uint32_t)token;
        return (size_t)((key * 0x9e3779b97f4a7c15ull) >> shift);     // multiplicative hashing, the golden ratio's bits
    }
    int32_t child(int32_t node, int32_t token) const {
        const int32_t newest = nodes[node].newest;
        if (newest == 0 || nodes[newest].token == token) return newest;
        if (nodes[newest].older == 0) return 0;
        const size_t mask = slots.size() - 1;
        size_t i = slot_of(node, token);
        while (slots[i].child != 0 && !(slots[i].token == token && nodes[slots[i].child].parent == node)) i = (i + 1) & mask;
        return slots[i].child;
    }
    void enter(int32_t c) {
        const size_t mask = slots.size() - 1;
        size_t i = slot_of(nodes[c].parent, nodes[c].token);
        while (slots[i].child != 0) i = (i + 1) & mask;
        slots[i] = {nodes[c].token, c};
        ++used;
    }
    // Room for `more` further nodes: the records, and a slot for each and for the only child that it may make one of two.
    void make_room(size_t more) {
        const size_t need = nodes.size() + more;
        if (need > nodes.capacity()) nodes.reserve(std::max(need, 2 * nodes.capacity()));
        const size_t edges = std::min(used + 2 * more, need);
        grow_table(edges + edges / 3 + 1);
    }
    void grow_table(size_t want) {
        if (want <= slots.size()) return;
        int log2 = 64 - shift;
        while (((size_t)1 << log2) < want) ++log2;
        std::vector<Slot> fresh((size_t)1 << log2, Slot{0, 0});
        slots.swap(fresh);
        shift = 64 - log2;
        used = 0;
        for (size_t c = 1; c < nodes.size(); ++c)
            if (nodes[nodes[nodes[c].parent].newest].older != 0) enter((int32_t)c);
    }
    int32_t add(int32_t node, int32_t token) {
        const int32_t c = (int32_t)nodes.size(), newest = nodes[node].newest;
        nodes.push_back({token, 0, node, 0, newest});
        nodes[node].newest = c;
        if (newest != 0) {
            if (nodes[newest].older == 0) enter(newest);
            enter(c);
        }
        return c;
    }
    // the most frequent continuation, the earliest of equals (which is met last)
    int32_t best_child(int32_t node) const {
        int32_t best = nodes[node].newest;
        for (int32_t c = nodes[best].older; c != 0; c = nodes[c].older)
            if (nodes[c].count >= nodes[best].count) best = c;
        return best;
    }
    // The `most` best continuations by descending count, equal counts in order of creation (children of one node
    // have increasing numbers).
    void best_children(int32_t node, size_t most, std::vector<int32_t> &c) const {
        c.clear();
        for (int32_t i = nodes[node].newest; i != 0; i = nodes[i].older) c.push_back(i);
        const auto better = [&](int32_t a, int32_t b) {
            return nodes[a].count != nodes[b].count ? nodes[a].count > nodes[b].count : a < b;
        };
        if (c.size() > most) {
            std::partial_sort(c.begin(), c.begin() + most, c.end(), better);
            c.resize(most);
        } else {
            std::sort(c.begin(), c.end(), better);
        }
    }
};

namespace {

// The tails of a context that are in the trie, as the context grows: node[len] is where the tail of `len` tokens
// ends.  With an n-gram every n-gram inside it is in the trie too, so the known tails are those of 1..known tokens.
struct Tails {
    const reader_trie &t;
    std::vector<int32_t> node;
    int32_t known = 0;
    explicit Tails(const reader_trie &trie, int32_t longest) : t(trie), node((size_t)std::min(longest, trie.max_depth - 1) + 1, 0) {}
    void append(int32_t token) {
        const int32_t most = std::min(known + 1, (int32_t)node.size() - 1);
        known = 0;
        for (int32_t len = most; len >= 1; --len) {
            node[len] = t.child(node[len - 1], token);      // (node[0], the empty tail, is the root)
            if (node[len] != 0 && known == 0) known = len;
        }
    }
    // The node reached by the longest tail that is in the trie, has a continuation and leaves room below it
    // (Section 4.2: a tail that is not present loses its first token and is tried again).  At least one token
    // of context is kept.  0: no continuation known.
    int32_t descend() const {
        for (int32_t len = known; len >= 1; --len)
            if (t.nodes[node[len]].newest != 0) return node[len];
        return 0;
    }
    void start(const int32_t *ctx, int32_t n) {
        for (int32_t i = std::max(0, n - (t.max_depth - 1)); i < n; ++i) append(ctx[i]);
    }
};

}  // namespace

extern "C" reader_trie *reader_trie_create(int32_t max_depth) {
    if (max_depth < 2 || max_depth > 4096) return nullptr;
    reader_trie *t = new (std::nothrow) reader_trie;
    if (!t) return nullptr;
    t->max_depth = max_depth;
    try {
        t->slots.assign(64, reader_trie::Slot{0, 0});
        t->shift = 64 - 6;
        t->nodes.push_back({-1, 0, -1, 0, 0});
    } catch (const std::bad_alloc &) {
        delete t;
        return nullptr;
    }
    return t;
}

extern "C" void reader_trie_destroy(reader_trie *t) { delete t; }

extern "C" int64_t reader_trie_nodes(const reader_trie *t) { return t ? (int64_t)t->nodes.size() : -1; }

extern "C" int reader_trie_insert(reader_trie *t, const int32_t *tokens, int64_t n) {
    if (!t || n < 0 || (n > 0 && !tokens)) return READER_EINVAL;
    try {
        // at[d]: the node of the n-gram of d tokens that ends in front of the current token (at[0]: the root)
        const int32_t D = t->max_depth;
        std::vector<int32_t> at((size_t)std::min<int64_t>(D, n) + 1, 0);
        // (more than half of the n-grams of a text are new: growing by doubling would move and fault in all of it again; a
        // quarter of them need a slot)
        const size_t fresh = (size_t)std::min<int64_t>(std::min<int64_t>(n, D) * (n / 8) * 5, 1 << 20);
        if (t->nodes.size() + fresh > t->nodes.capacity()) t->nodes.reserve(std::max(t->nodes.size() + fresh, 2 * t->nodes.capacity()));
        t->grow_table(t->used + fresh / 2);
        for (int64_t j = 0; j < n; ++j) {
            const int32_t token = tokens[j], longest = (int32_t)std::min<int64_t>(j, D - 1);
            if (t->nodes.size() + (size_t)longest + 1 > 0x7fffffffu) return READER_EUNSUPPORTED;
            t->make_room((size_t)longest + 1);
            for (int32_t d = longest; d >= 0; --d) {
                int32_t c = t->child(at[d], token);
                if (c == 0) c = t->add(at[d], token);
                ++t->nodes[c].count;
                at[d + 1] = c;
            }
        }
    } catch (const std::bad_alloc &) {
        return READER_EUNSUPPORTED;
    }
    return READER_OK;
}

extern "C" int32_t reader_trie_search_path(const reader_trie *t, const int32_t *suffix, int32_t n_suffix, int32_t depth,
                                           int32_t *path_tokens) {
    if (!t || n_suffix < 0 || depth < 0 || (n_suffix > 0 && !suffix) || (depth > 0 && !path_tokens)) return -1;
    try {   // (no exception may cross the C boundary: running out of memory is reported as a bad call)
        Tails tails(*t, n_suffix > 0x7fffffff - depth ? 0x7fffffff : n_suffix + depth);
        tails.start(suffix, n_suffix);
        int32_t k = 0;
        while (k < depth) {
            const int32_t at = tails.descend();
            if (at == 0) break;
            const int32_t token = t->nodes[t->best_child(at)].token;
            path_tokens[k++] = token;
            tails.append(token);
        }
        return k;
    } catch (const std::bad_alloc &) {
        return -1;
    }
}

extern "C" int32_t reader_trie_extract_tree(const reader_trie *t, const int32_t *suffix, int32_t n_suffix,
                                            int32_t max_depth, int32_t budget, int32_t *tokens, int32_t *parents) {
    if (!t || n_suffix < 1 || !suffix || max_depth < 0 || budget < 1 || !tokens || !parents) return -1;
    tokens[0] = suffix[n_suffix - 1];      // the root is the last committed token
    parents[0] = -1;
    int32_t used = 1;
    // depth-first, most frequent continuation first, within the depth and the node budget
    struct Frame { int32_t trie_node, tree_node, depth; };
    try {
        Tails tails(*t, n_suffix);
        tails.start(suffix, n_suffix);
        const int32_t start = tails.descend();
        if (start == 0) return used;
        std::vector<Frame> stack;
        std::vector<int32_t> c;
        stack.push_back({start, 0, 0});
        while (!stack.empty() && used < budget) {
            const Frame f = stack.back();
            stack.pop_back();
            int32_t me = f.tree_node;
            if (f.depth > 0) {                  // (the start node itself is the root, already numbered)
                me = used++;
                tokens[me] = t->nodes[f.trie_node].token;
                parents[me] = f.tree_node;
            }
            if (f.depth < max_depth) {
                t->best_children(f.trie_node, (size_t)(budget - used), c);   // (no more than that can still be visited)
                for (auto it = c.rbegin(); it != c.rend(); ++it) stack.push_back({*it, me, f.depth + 1});   // best on top
            }
        }
    } catch (const std::bad_alloc &) {
        return -1;
    }
    return used;
}

extern "C" int32_t reader_tree_attach_path(int32_t *tokens, int32_t *parents, int32_t n_nodes, int32_t capacity,
                                           int32_t at_node, const int32_t *path_tokens, int32_t k) {
    if (!tokens || !parents || n_nodes < 1 || capacity < n_nodes || at_node < 0 || at_node >= n_nodes || k < 0 ||
        (k > 0 && !path_tokens))
        return -1;
    int32_t prev = at_node;
    for (int32_t i = 0; i < k && n_nodes < capacity; ++i) {
        tokens[n_nodes] = path_tokens[i];
        parents[n_nodes] = prev;
        prev = n_nodes++;
    }
    return n_nodes;
}

extern "C" double reader_self_repetition(const int32_t *prompt, int64_t n_prompt, const int32_t *response,
                                         int64_t n_response) {
    if (n_prompt < 0 || n_response < 0 || (n_prompt > 0 && !prompt) || (n_response > 0 && !response)) return -1.0;
    if (n_response == 0) return 0.0;
    // history = prompt, then the processed part of the response; a match must lie inside it
    try {
        std::vector<int32_t> hist(prompt, prompt + n_prompt);
        hist.reserve((size_t)(n_prompt + n_response));
        int64_t ptr = 0, advances = 0;
        while (ptr < n_response) {
            int64_t best = 0;
            const int64_t h = (int64_t)hist.size();
            for (int64_t s = 0; s < h; ++s) {
                if (hist[s] != response[ptr]) continue;
                int64_t len = 0;
                while (s + len < h && ptr + len < n_response && hist[s + len] == response[ptr + len]) ++len;
                best = std::max(best, len);
            }
            const int64_t step = best > 0 ? best : 1;
            hist.insert(hist.end(), response + ptr, response + ptr + step);
            ptr += step;
            ++advances;
        }
        return (double)n_response / (double)advances;
    } catch (const std::bad_alloc &) {
        return -1.0;
    }
}
