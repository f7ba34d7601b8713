// Device code of the acceptance and compaction steps, shared by their own kernels and by the launches of
// reader_verify_step: the tails do both, and so do workgroups of the attention launch of short problems; or the attention launch
// accepts, of short problems and in the 128-row ring kernel, and the tail appends.
//
// Acceptance (Algorithm 5; Appendix C invariants 2-3): one 64-lane wavefront per
// sequence.  Each lane owns up to two tree nodes.  A node "matches" when its drafted
// token equals the base model's token at its parent; the matches of all nodes are
// gathered with two wavefront ballots.  Every lane then walks its nodes' parent
// chains to get their ancestor-or-self sets as 128-bit masks; a node is accepted
// iff its whole set lies inside the match ballot, and its depth is the set's
// population count minus one.  A wavefront max-reduction over (depth, lowest id)
// picks the terminal node; the nodes of its ancestor set scatter themselves into
// `path` at their own depth.
//
// Compaction (Section 4.3 / Algorithm 4, applied every step): one workgroup per
// sequence copies the accepted rows with 128-bit accesses and then bumps seq_lens.
#pragma once

#include "internal.h"

namespace reader {

// LDS the acceptance of one sequence needs.
struct AcceptShared {
    int par[READER_MAX_T];
    int target[READER_MAX_T];        // the base model's tokens, so that target[parent] is an LDS read
    int path[READER_MAX_T];          // the accepted path, to report and for a compaction that follows in the same workgroup
    unsigned long long term[2];
    int accept_len;
};

// Orders a wavefront's LDS accesses for the compiler; the hardware executes those of one wavefront in order.
__device__ __forceinline__ void wave_lds_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// The tokens and parents of a lane's two nodes, asked for ahead of the acceptance.
struct AcceptTokens {
    int par[2], draft[2], target[2];
};
__device__ __forceinline__ AcceptTokens accept_load(const AcceptParams &p, int b, int lane) {
    AcceptTokens a;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int i = lane + 64 * s;
        const bool in = i < p.T;
        a.par[s] = in ? p.parents[(size_t)b * p.T + i] : -1;
        a.draft[s] = in ? p.draft[(size_t)b * p.T + i] : 0;
        a.target[s] = in ? p.target[(size_t)b * p.T + i] : 0;
    }
    return a;
}

// Acceptance of sequence b by one wavefront, without barriers, in three parts, so that a caller can put other work between
// them: the tokens go into LDS, the path is chosen from there (LDS only), the results are written out.
struct AcceptNodes {
    int draft[2], par[2];      // drafted token and parent of the lane's two nodes (-1: none, or a bad link)
    bool valid[2];
};
__device__ __forceinline__ AcceptNodes accept_stage(const AcceptParams &p, int lane, const AcceptTokens &tok, AcceptShared &sh) {
    AcceptNodes nd;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int i = lane + 64 * s, pi = tok.par[s];
        nd.draft[s] = tok.draft[s];
        nd.valid[s] = i < p.T && ((i == 0) ? (pi == -1) : (pi >= 0 && pi < i));
        nd.par[s] = nd.valid[s] ? pi : -1;
        if (i < p.T) {
            sh.par[i] = nd.par[s];
            sh.target[i] = tok.target[s];
        }
    }
    wave_lds_order();
    return nd;
}

// Returns the number of accepted nodes, leaves the path in sh.path and the status bits to report in `bits`.
__device__ inline int accept_choose(const AcceptParams &p, int lane, const AcceptNodes &nd, AcceptShared &sh, int &bits) {
    const int T = p.T;
    bool match[2] = {false, false}, bad_tree = false;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int i = lane + 64 * s;
        if (i < T) {
            match[s] = (i == 0) || (nd.valid[s] && nd.draft[s] == sh.target[nd.par[s]]);   // (target[parent] comes from LDS)
            bad_tree |= !nd.valid[s];
        }
    }
    const unsigned long long m_lo = __ballot(match[0]), m_hi = __ballot(match[1]);

    // ancestor-or-self sets by walking the parent chain (at most T steps, always ends)
    unsigned long long a_lo[2] = {0ull, 0ull}, a_hi[2] = {0ull, 0ull};
    int key[2] = {-1, -1};
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int i = lane + 64 * s;
        if (i < T) {
            int t = i;
            for (int step = 0; step < T && t >= 0; ++step) {
                if (t < 64) a_lo[s] |= 1ull << t; else a_hi[s] |= 1ull << (t - 64);
                t = sh.par[t];
            }
            const bool ok = ((a_lo[s] & ~m_lo) == 0) && ((a_hi[s] & ~m_hi) == 0);
            const int depth = __popcll(a_lo[s]) + __popcll(a_hi[s]) - 1;
            if (ok) key[s] = depth * 256 + (255 - i);   // deeper first, then lower node id
        }
    }
    int best = max(key[0], key[1]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) best = max(best, __shfl_xor(best, off));
    // the root always qualifies, so best >= 255
    const int term = 255 - (best & 255), depth_term = best >> 8;
    const int n_out = min(depth_term, p.max_path - 1);
    if (lane == (term & 63)) {
        // (a choice, not an index: an indexed array would live in scratch memory)
        sh.term[0] = term < 64 ? a_lo[0] : a_lo[1];
        sh.term[1] = term < 64 ? a_hi[0] : a_hi[1];
    }
    wave_lds_order();
    const unsigned long long t_lo = sh.term[0], t_hi = sh.term[1];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int i = lane + 64 * s;
        const bool on_path = ((s == 0 ? t_lo : t_hi) >> lane) & 1ull;
        if (i < T && on_path) {
            const int depth = __popcll(a_lo[s]) + __popcll(a_hi[s]) - 1;
            if (depth < p.max_path) sh.path[depth] = i;
        }
    }
    if (lane == 0) sh.accept_len = n_out;
    wave_lds_order();
    bits = (__ballot(bad_tree) != 0ull ? READER_STATUS_BAD_TREE : 0) | (depth_term > n_out ? READER_STATUS_BAD_PATH : 0);
    return n_out;
}

__device__ __forceinline__ void accept_report(const AcceptParams &p, int b, int lane, int n, int bits, const AcceptShared &sh) {
    for (int j = lane; j < p.max_path; j += 64) p.path[(size_t)b * p.max_path + j] = j <= n ? sh.path[j] : -1;
    if (lane == 0) {
        p.accept_len[b] = n;
        p.bonus[b] = sh.target[sh.path[n]];
        if (p.status && bits) atomicOr(p.status, bits);
    }
}

// all of it; the number of accepted nodes and the path are left in `sh` too
__device__ inline void accept_path_wave(const AcceptParams &p, int b, int lane, AcceptShared &sh) {
    const AcceptNodes nd = accept_stage(p, lane, accept_load(p, b, lane), sh);
    int bits;
    const int n = accept_choose(p, lane, nd, sh, bits);
    accept_report(p, b, lane, n, bits, sh);
}

// What compaction needs that does not depend on the accepted path: the old length and the page
// ids of the positions a path could be appended to.  Loaded up front so that, in the fused tail
// kernel, they travel while the acceptance runs.
struct CompactShared {
    int L;
    int page[READER_MAX_T];   // page id of position L + j (or -1 past the page table)
};

// Called by all 256 threads of the workgroup, before a barrier.
__device__ inline void kv_compact_prefetch(const CompactParams &p, int b, int tid, CompactShared &cs) {
    const int L = p.seq_lens[b];
    if (tid == 0) cs.L = L;
    if (tid < p.max_path) {
        const long long pos = (long long)L + tid;
        const bool in_table = L >= 0 && pos < (long long)p.max_pages * READER_PAGE_SIZE;
        cs.page[tid] = in_table ? p.page_table[(size_t)b * p.max_pages + pos / READER_PAGE_SIZE] : -1;
    }
}

// Called by all 256 threads of the workgroup, after kv_compact_prefetch and a barrier.
// n = accept_len of the sequence, path = its accepted path (global or LDS).
__device__ inline void kv_compact_body(const CompactParams &p, int b, int tid, int n, const int *path,
                                       const CompactShared &cs) {
    const int L = cs.L;

    // Every item this sequence would touch is checked before anything is written.
    int bad = 0;
    if (n < 0 || n > p.max_path - 1 || L < 0 || (long long)L + n + 1 > (long long)p.max_pages * READER_PAGE_SIZE) {
        bad = READER_STATUS_BAD_PATH;
    } else {
        for (int j = tid; j <= n; j += 256) {
            const int node = path[j];
            if (node < 0 || node >= p.T) bad |= READER_STATUS_BAD_PATH;
            const int page = cs.page[j];
            if (page < 0 || page >= p.num_pages) bad |= READER_STATUS_BAD_PAGE;
        }
    }
    // the barriers also order every thread's read of seq_lens before its update below
    const int bad_path = __syncthreads_or(bad & READER_STATUS_BAD_PATH);
    const int bad_page = __syncthreads_or(bad & READER_STATUS_BAD_PAGE);
    if (bad_path || bad_page) {
        if (tid == 0 && p.status)
            atomicOr(p.status, (bad_path ? READER_STATUS_BAD_PATH : 0) | (bad_page ? READER_STATUS_BAD_PAGE : 0));
        return;
    }

    const int chunks_per_head = p.D / 8;                 // 16-byte chunks
    const int chunks_per_row = p.Hkv * chunks_per_head;  // one position, all kv heads, K or V
    // A thread keeps its place inside a position (K or V, head, chunk) and walks the path entries, eight at a
    // time: their rows are asked for together and stored afterwards (taken one by one, every accepted token
    // costs a trip to memory).  The loads carry no condition (an entry past the path reads the last one
    // again), so that they stay together in front of the stores.
    // (held in a native vector type: an array of uint4 goes through scratch memory, one more trip)
    typedef unsigned int held_t __attribute__((ext_vector_type(4)));
    constexpr int kBatch = 8;
    for (int rem = tid; rem < 2 * chunks_per_row; rem += 256) {
        const int which = rem / chunks_per_row;
        const int c = rem - which * chunks_per_row;
        const int h = c / chunks_per_head;
        const int dc = c - h * chunks_per_head;
        const uint16_t *tree = (which ? p.v_tree : p.k_tree) + ((size_t)b * p.T * p.Hkv + h) * p.D + dc * 8;
        uint16_t *cache = (which ? p.v_cache : p.k_cache) + (size_t)h * READER_PAGE_SIZE * p.D + dc * 8;
        for (int j0 = 0; j0 <= n; j0 += kBatch) {
            held_t held[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                held[u] = *reinterpret_cast<const held_t *>(tree + (size_t)path[min(j0 + u, n)] * p.Hkv * p.D);
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int j = j0 + u;
                if (j <= n) {
                    const long long page = cs.page[j];
                    const int slot = (L + j) % READER_PAGE_SIZE;
                    *reinterpret_cast<held_t *>(cache + ((size_t)page * p.Hkv * READER_PAGE_SIZE + slot) * p.D) = held[u];
                }
            }
        }
    }
    if (tid == 0) p.seq_lens[b] = L + n + 1;
}

// The rows of a sequence's path, appended by 256 threads in the launch behind the attention; the path is chosen here too unless that
// launch has (then it is fetched next to what kv_compact_prefetch fetches, so that the next trip to memory is the rows').
template <bool kAccept>
__device__ __forceinline__ void step_tail(const AcceptParams &ap, const CompactParams &cp, int b, int tid) {
    __shared__ CompactShared cs;
    if constexpr (kAccept) {
        __shared__ AcceptShared sh;
        // (in-cache layout, no tree tensors: the in-place move of the accepted rows follows as a launch of its own)
        const bool append = cp.k_tree != nullptr;
        if (append) kv_compact_prefetch(cp, b, tid, cs);   // on its way while the path is being chosen
        if (tid < 64) accept_path_wave(ap, b, tid, sh);
        if (!append) return;
        __syncthreads();
        kv_compact_body(cp, b, tid, sh.accept_len, sh.path, cs);
    } else {
        __shared__ int path[READER_MAX_T];
        const int n = cp.accept_len[b];
        if (tid < cp.max_path) path[tid] = cp.path[(size_t)b * cp.max_path + tid];
        kv_compact_prefetch(cp, b, tid, cs);
        __syncthreads();
        kv_compact_body(cp, b, tid, n, path, cs);
    }
}

// The accepted rows of a sequence, moved by wavefronts that share no barrier (inside the attention launch of a fused step).
// Every wavefront checks for itself what the sequence would touch, one path entry per lane and half, and notes where each
// entry's row is and goes.  A thread keeps its column of a position (K or V, head, chunk) and walks the entries in order,
// eight loads ahead of eight stores.  Tree tensors: row path[j] goes to position L + j.  Rows in the cache already (k_tree
// null): position L + path[j] moves to L + j; path[j] >= j, so a destination is never the source of a later entry, and an
// earlier one of the column has been read.
struct TailShared {
    AcceptShared accept;
    long long src[READER_MAX_T], dst[READER_MAX_T];   // in values, of head 0 and chunk 0; dst < 0: in place already
};
struct TailLane {
    int L, bad;             // old length, status bits (0: go); the same in all lanes
};
__device__ __forceinline__ TailLane tail_check(const CompactParams &p, int b, int lane, TailShared &sh) {
    TailLane t;
    t.L = __builtin_amdgcn_readfirstlane(p.seq_lens[b]);
    t.bad = READER_STATUS_BAD_PATH;
    const int n = sh.accept.accept_len;
    const bool move = p.k_tree == nullptr;
    const long long mapped = (long long)p.max_pages * READER_PAGE_SIZE, page_values = (long long)p.Hkv * READER_PAGE_SIZE * p.D;
    const int32_t *table = p.page_table + (size_t)b * p.max_pages;
    if (t.L < 0 || (long long)t.L + n + 1 > mapped) return t;
    int bad = 0;
    for (int j = lane; j <= n; j += 64) {
        const int node = sh.accept.path[j], to = t.L + j;
        const long long from = (long long)t.L + node;
        if (move && from >= mapped) { bad |= READER_STATUS_BAD_PATH; continue; }
        const int dst_page = table[to / READER_PAGE_SIZE], src_page = move ? table[from / READER_PAGE_SIZE] : 0;
        if (dst_page < 0 || dst_page >= p.num_pages || src_page < 0 || src_page >= p.num_pages) { bad |= READER_STATUS_BAD_PAGE; continue; }
        sh.src[j] = move ? src_page * page_values + from % READER_PAGE_SIZE * p.D : ((long long)b * p.T + node) * p.Hkv * p.D;
        sh.dst[j] = move && node == j ? -1 : dst_page * page_values + to % READER_PAGE_SIZE * p.D;
    }
    wave_lds_order();
    t.bad = (__ballot(bad & READER_STATUS_BAD_PATH) != 0ull ? READER_STATUS_BAD_PATH : 0) |
            (__ballot(bad & READER_STATUS_BAD_PAGE) != 0ull ? READER_STATUS_BAD_PAGE : 0);
    return t;
}
constexpr int kTailBatch = 8;
typedef unsigned int tail_held_t __attribute__((ext_vector_type(4)));
// A thread's column `col` (below 2 Hkv D / 8): where its 16 bytes of a row of the source and of the cache are.
struct TailColumn {
    const uint16_t *src;
    uint16_t *dst;
};
__device__ __forceinline__ TailColumn tail_column(const CompactParams &p, int col) {
    const int chunks = p.D / 8, per_row = p.Hkv * chunks, which = col >= per_row ? 1 : 0, c = col - which * per_row;
    const int h = c / chunks, dc = c - h * chunks;
    TailColumn t;
    t.dst = (which ? p.v_cache : p.k_cache) + (size_t)h * READER_PAGE_SIZE * p.D + dc * 8;
    t.src = p.k_tree ? (which ? p.v_tree : p.k_tree) + (size_t)h * p.D + dc * 8 : t.dst;
    return t;
}
__device__ __forceinline__ void tail_load(const TailColumn &col, const TailShared &sh, int j0, tail_held_t (&held)[kTailBatch]) {
    const int n = sh.accept.accept_len;
#pragma unroll
    for (int u = 0; u < kTailBatch; ++u) held[u] = *reinterpret_cast<const tail_held_t *>(col.src + sh.src[min(j0 + u, n)]);
}
__device__ __forceinline__ void tail_store(const TailColumn &col, const TailShared &sh, int j0, const tail_held_t (&held)[kTailBatch]) {
    const int n = sh.accept.accept_len;
#pragma unroll
    for (int u = 0; u < kTailBatch; ++u) {
        const long long to = j0 + u <= n ? sh.dst[j0 + u] : -1;
        if (to >= 0) *reinterpret_cast<tail_held_t *>(col.dst + to) = held[u];
    }
}

}  // namespace reader
