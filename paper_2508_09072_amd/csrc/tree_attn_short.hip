// Tree-masked attention (Section 3.2 of the READER paper) for short problems: the flavour of the main kernel whose
// time is latency and not bandwidth.
//
// With few users or short contexts a compute unit has a handful of key tiles to look at, and a launch of the ring
// kernels (tree_attn_mfma.hip, tree_attn_wide.hip) spends a good part of its time before the first of them is asked
// for: scan of all lengths, cut of the tile axis, tile list in LDS, barriers in between.  Here everything that can
// be is fixed by the host, and the rest is asked for at once:
//   - a static grid: workgroup (split s, kv head, sequence and row chunk) takes the s-th of n_splits equal shares of
//     its pair's tiles, so nothing is searched for (of the other sequences' lengths only the sum is wanted, where pairs
//     are cut: a pair that the ring kernels could leave whole stays whole);
//   - one trip to memory brings the length, the page ids of the sequence (into registers of the wavefronts that
//     copy, asked for before the length is known), the parent pointers and the query rows; a second one the keys;
//   - no list and no barrier in front of the main loop;
//   - the fused step is this one launch (see kJoin below).
// The main loop is that of the 128-row ring kernel: wavefronts 0..3 compute 32 query rows each, 4..7 copy 64-key
// tiles HBM -> LDS into a ring of four buffers, one barrier per tile.
//
// What bounds a launch: its chain of trips to memory and then the computation, one wavefront per SIMD working through
// operand reads, products, softmax, products (about 2000 cycles per tile at head dimension 128, 1024 of them matrix
// instructions), not the copies (with the computation left out the same launch ends 4 us sooner, with the copies
// left out 1 us).  Measured against the ring kernels, main launch and merge: one prompt of 4 K tokens, 64 nodes x 4
// grouped heads 21.5 -> 20.4 us; 16-node tree on 512 tokens 14.7 -> 11.4; three sequences of 0.7 - 2.5 K tokens
// 21.3 -> 18.7; 32 sequences of 0.4 - 0.9 K with 752 query rows per kv head 95 -> 76; 39 sequences of 68 tokens
// 16.7 -> 7.6.
#include <hip/hip_ext.h>

#include <mutex>

#include "accept_compact.h"
#include "arrivals.h"
#include "internal.h"
#include "tree_attn_common.h"

namespace reader {

namespace {

constexpr int kShortRows = 128;
constexpr int kShortStages = 4;
constexpr int kPageRegs = 4;              // page ids a copying wavefront holds: one per lane and register, i.e. 256 tiles

// Profiling build (-DREADER_WG_STAMPS): thread `who` of the workgroup notes the time at point k
#ifdef READER_WG_STAMPS
#define READER_STAMP(k, who)                                                                              \
    do {                                                                                                  \
        const unsigned at_ = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;              \
        if (p.stamps && threadIdx.x == (who) && at_ < kStampedWgs)                                        \
            p.stamps[(size_t)at_ * kWgStamps + (k)] = (long long)__builtin_amdgcn_s_memrealtime();         \
    } while (0)
#else
#define READER_STAMP(k, who) do { } while (0)
#endif

// Head dimension 128: one workgroup per compute unit (its ring takes 128 KB of LDS), one computing wavefront per SIMD
// with registers to spare, which it uses to have its operands read long before they are needed.  Head dimension 64:
// half the ring, so two workgroups per compute unit if a wavefront makes do with 128 registers; the two computing
// wavefronts of a SIMD then fill each other's waits (measured, 32 sequences with 752 query rows per kv head: 76 us
// against 89 us with the deeper prefetch and one workgroup).
#ifdef READER_WG_STAMPS
constexpr int kWavesPerSimd64 = 2;        // (the time stamps take registers)
#else
constexpr int kWavesPerSimd64 = 4;
#endif

// Merge of the n_splits records of every query row.  A record is laid out [chunk of 8 values][row]; a wavefront takes four rows
// of four chunks (64 contiguous bytes per chunk of a record, 64 of an output row), and its four groups of 16 lanes every fourth
// record each, four or eight of them asked for together: up to 32 records are one trip to memory.  Weights against the largest of the
// lane's references, then against that of all four groups: two swaps and a maximum, two swaps and additions.
//
// What bounds it: alone, a launch; inside the attention launch, one wavefront's instructions, each waiting for the one before.
// Before, a thread per row and chunk folded one record after the other into its state (two exponentials and 36 instructions
// per record, four wavefronts' states through LDS): inside the launch, 24 pairs of 100 rows in ten shares, 3.5 us where this takes
// 2.2; as a launch of its own, 16-layer decoding step of three users 265 -> 255 us.
//
// kAgent: the records are read past the caches of this XCD.  kUnits: sets of four rows and four chunks that the wavefront takes
// together, `unit` and every `step`-th behind it below `end` (few records leave a lane room for several).
template <int D, bool kAgent, int kUnits, int kBatch>
__device__ __forceinline__ void merge_rows(const AttnParams &p, int b, int hkv, int unit, int step, int end) {
    constexpr int kQuads = D / 32;                           // sets of four chunks in a row
    constexpr size_t kRec = attn_slot_floats(D, kShortRows);   // (64 records stay below 2^32 bytes)
    const int lane = threadIdx.x & 63, g = lane >> 4, n = p.n_splits;
    // (four wavefronts side by side: eight rows of eight chunks, so that the halves of a line of 128 bytes are fetched together)
    int m_row[kUnits], c[kUnits];
    const char *rec[kUnits];
    unsigned row_at[kUnits], m_at[kUnits];
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
        const int at = min(unit + u * step, end - 1);        // (a unit too many is the last one again, and not written)
        const int in8 = at % (2 * kQuads), quad = (in8 >> 2) * 2 + (in8 & 1), block = at / (2 * kQuads) * 2 + ((in8 >> 1) & 1);
        const int chunk = block / (kShortRows / 4), r = block % (kShortRows / 4) * 4 + (lane & 3);
        c[u] = quad * 4 + ((lane >> 2) & 3);
        m_row[u] = unit + u * step < end ? chunk * kShortRows + r : p.M;
        // (rows past the last one of a block are in the records too, with whatever bytes)
        rec[u] = reinterpret_cast<const char *>(p.workspace + ((size_t)(b * p.Hkv + hkv) * p.n_row_chunks + chunk) * n * kRec);
        row_at[u] = (c[u] * kShortRows + r) * 16;
        m_at[u] = (kShortRows * (D / 2) + r) * 4;
    }
    float m[kUnits], l[kUnits], acc[kUnits][8];
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
        m[u] = -INFINITY;
        l[u] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[u][e] = 0.f;
    }
#pragma unroll 1
    for (int j0 = g; j0 - g < n; j0 += 4 * kBatch) {
        float ms[kUnits][kBatch], ls[kUnits][kBatch];
        uint4 v[kUnits][kBatch];
#pragma unroll
        for (int u = 0; u < kUnits; ++u)
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                const unsigned at = (unsigned)min(j0 + 4 * i, n - 1) * (unsigned)(kRec * sizeof(float));   // (a record read twice is only a load)
                const uint4 *row = reinterpret_cast<const uint4 *>(rec[u] + (at + row_at[u]));
                const float *m_rec = reinterpret_cast<const float *>(rec[u] + (at + m_at[u]));
                const float *l_rec = reinterpret_cast<const float *>(rec[u] + (at + m_at[u] + kShortRows * 4));
                v[u][i] = kAgent ? agent_load16(row) : *row;
                ms[u][i] = kAgent ? agent_load(m_rec) : *m_rec;
                ls[u][i] = kAgent ? agent_load(l_rec) : *l_rec;
            }
#pragma unroll
        for (int u = 0; u < kUnits; ++u) {
            float m_new = m[u];
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                if (j0 + 4 * i >= n) ms[u][i] = -INFINITY;
                m_new = fmaxf(m_new, ms[u][i]);
            }
            const float ref = m_new == -INFINITY ? 0.f : m_new, old = __builtin_amdgcn_exp2f(m[u] - ref);
            l[u] *= old;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[u][e] *= old;
            m[u] = m_new;
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                // (a share that saw no key of this row wrote no values: whatever is there is dropped, not weighted)
                const bool none = ms[u][i] == -INFINITY;
                const float w = none ? 0.f : ls[u][i] * __builtin_amdgcn_exp2f(ms[u][i] - ref);
                const uint32_t x[4] = {none ? 0u : v[u][i].x, none ? 0u : v[u][i].y, none ? 0u : v[u][i].z, none ? 0u : v[u][i].w};
                l[u] += w;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc[u][2 * e] = __builtin_fmaf(w, __uint_as_float(x[e] << 16), acc[u][2 * e]);
                    acc[u][2 * e + 1] = __builtin_fmaf(w, __uint_as_float(x[e] & 0xffff0000u), acc[u][2 * e + 1]);
                }
            }
        }
    }
    // over the four groups of lanes
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
        float m_all = m[u];
        {
            const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(m_all), __float_as_uint(m_all), false, false);
            m_all = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
            const auto b2 = __builtin_amdgcn_permlane16_swap(__float_as_uint(m_all), __float_as_uint(m_all), false, false);
            m_all = fmaxf(__uint_as_float(b2[0]), __uint_as_float(b2[1]));
        }
        const float mine = m[u] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[u] - m_all);
        auto total = [&](float x) {
            x *= mine;
            const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
            x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
            const auto b2 = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
            return __uint_as_float(b2[0]) + __uint_as_float(b2[1]);
        };
        l[u] = total(l[u]);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[u][e] = total(acc[u][e]);
        if (m_row[u] < p.M && g == 0) {
            const float inv = 1.f / l[u];                    // (> 0: every row sees its own tree node)
            // m / G without an integer division: m + 0.5 is 0.5 / G away from the next multiple of G, far more than rounding
            const int node = (int)(((float)m_row[u] + 0.5f) * p.g_rcp), group = m_row[u] - node * p.G;
            *reinterpret_cast<uint4 *>(p.out + (((size_t)b * p.T + node) * p.Hq + hkv * p.G + group) * D + c[u] * 8) =
                make_uint4(pack_bf16x2(acc[u][0] * inv, acc[u][1] * inv), pack_bf16x2(acc[u][2] * inv, acc[u][3] * inv),
                           pack_bf16x2(acc[u][4] * inv, acc[u][5] * inv), pack_bf16x2(acc[u][6] * inv, acc[u][7] * inv));
            if (p.lse && c[u] == 0)
                p.lse[((size_t)b * p.Hq + hkv * p.G + group) * p.T + node] = (m_all + __builtin_amdgcn_logf(l[u])) * kLn2;
        }
    }
}

// As a launch of its own: a wavefront per unit, blocks of four.
template <int D>
__device__ __forceinline__ void merge_block(const AttnParams &p, int b, int hkv, int block) {
    const int unit = block * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (p.n_splits > 16) merge_rows<D, false, 1, 8>(p, b, hkv, unit, 1, unit + 1);
    else merge_rows<D, false, 1, 4>(p, b, hkv, unit, 1, unit + 1);
}

// Inside the attention launch: the rows that fall to share s of the pair's chunk, by the eight wavefronts of a workgroup.
// Records that were all written on this XCD are in its L2 (and in no first-level cache: nobody has read them in this launch before
// all of them were there, and no line of 128 bytes holds two pairs' records); others are read past it (kAgent).
// With few shares a wavefront has several units to do, and takes up to four of them together: one trip to memory,
// not one each (64 pairs' chunks of 128 rows, two shares each 21.2 -> 18.2 us, three 17.7 -> 16.8).
template <int D, bool kAgent>
__device__ __forceinline__ void merge_share(const AttnParams &p, int b, int hkv, int chunk, int s) {
    constexpr int kQuads = D / 32;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = p.n_splits, step = n * 8;
    const int first = chunk * (kShortRows / 4) * kQuads, end = first + (min(kShortRows, p.M - chunk * kShortRows) + 7) / 8 * 2 * kQuads;
    auto all = [&](auto units_c, auto batch_c) __attribute__((always_inline)) {
        constexpr int kUnits = decltype(units_c)::value, kBatch = decltype(batch_c)::value;
#pragma unroll 1
        for (int u = first + s * 8 + wave; u < end; u += step * kUnits) merge_rows<D, kAgent, kUnits, kBatch>(p, b, hkv, u, step, end);
    };
    if (!kAgent && n <= 4) all(std::integral_constant<int, 4>{}, std::integral_constant<int, 1>{});
    else if (!kAgent && n <= 8) all(std::integral_constant<int, 2>{}, std::integral_constant<int, 2>{});
    else if (n <= 16) all(std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{});
    else all(std::integral_constant<int, 1>{}, std::integral_constant<int, 8>{});
}

// The argument of the fused step's kernels (parts of it are read where they are used: late_argument).
struct StepParams {
    JoinParams join;           // (of the launch that waits inside)
    AttnParams attn;
    AcceptParams accept;
    CompactParams compact;
};
// This launch's marks in the workspace header: of every workgroup that works on a share whether its part of the records is
// written, and whether it reads nothing of the cache and the lengths any more; of those that keep a sequence's cache whether
// they have left, and whether any of them has.
struct Marks {
    mark_t *written, *landed, *keepers, *any_left, token;
    int n_wg;
    __device__ __forceinline__ explicit Marks(const AttnParams &p, const JoinParams &j) {
        written = reinterpret_cast<mark_t *>(p.redo);
        landed = written + (p.n_splits > 1 ? kMaxMarks / 2 : 0);      // (whole pairs leave no record)
        keepers = reinterpret_cast<mark_t *>(p.pair_info);
        any_left = reinterpret_cast<mark_t *>(p.range_tiles);
        token = j.token;
        n_wg = p.B * p.Hkv * p.n_row_chunks * p.n_splits;
    }
};

// Compaction of sequence b by NT threads (`t` of them this one) that share no barrier, behind a path that is in sh.accept:
// the rows that were asked for ahead are in `held`.
template <int NT>
__device__ __forceinline__ void keep_rows(const CompactParams &cp, int b, int t, const TailLane &tail, const TailShared &sh,
                                          bool held_first, tail_held_t (&held)[kTailBatch]) {
    if (tail.bad == 0) {
#pragma unroll 1
        for (int c = t; c < 2 * cp.Hkv * (cp.D / 8); c += NT) {
            const TailColumn column = tail_column(cp, c);
#pragma unroll 1
            for (int j0 = 0; j0 <= sh.accept.accept_len; j0 += kTailBatch) {
                if (!held_first || c != t || j0 != 0) tail_load(column, sh, j0, held);
                tail_store(column, sh, j0, held);
            }
        }
    }
    if (t == 0) {
        if (tail.bad == 0) cp.seq_lens[b] = tail.L + sh.accept.accept_len + 1;
        else if (cp.status) atomicOr(cp.status, tail.bad);
    }
}

// The sequences whose own workgroup has left, by one wavefront of a workgroup whose keys have landed, if it is the last.
__device__ __forceinline__ void keep_for_others(const AttnParams &p, const Marks &marks, int lane, TailShared &sh) {
    auto everybody = [&] { return all_here(marks.landed, marks.n_wg, marks.token, lane); };
    act_for_those_who_left(AgentMarks{lane}, marks.keepers, p.B, marks.token, everybody, [&](int b) __attribute__((always_inline)) {
        const AcceptParams ap = late_argument<AcceptParams, offsetof(StepParams, accept)>();
        const CompactParams cp = late_argument<CompactParams, offsetof(StepParams, compact)>();
        int bits;
        const AcceptNodes nodes = accept_stage(ap, lane, accept_load(ap, b, lane), sh.accept);
        (void)accept_choose(ap, lane, nodes, sh.accept, bits);          // (reported by the workgroup that left)
        const TailLane tail = tail_check(cp, b, lane, sh);
        tail_held_t held[kTailBatch];
        keep_rows<64>(cp, b, lane, tail, sh, false, held);
        wave_lds_order();                                               // (before the next one's nodes go where these were)
    });
}

// A workgroup that keeps one sequence's cache in a fused step: it accepts while the others attend, has the accepted rows ready,
// and when every one of the others has read its keys and the lengths it appends them (a slot behind one sequence's end may
// lie inside the prefix of another: forks of unequal length that share a partly filled page).
constexpr int kKeeperThreads = 256;
__device__ __forceinline__ void keep_sequence(const AttnParams &p, const JoinParams &j, int b, TailShared &sh, int &s_append) {
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid >= kKeeperThreads) return;
    const Marks marks(p, j);
    const CompactParams cp = late_argument<CompactParams, offsetof(StepParams, compact)>();
    if (tid < 64) accept_path_wave(late_argument<AcceptParams, offsetof(StepParams, accept)>(), b, lane, sh.accept);
    __syncthreads();
    const TailLane tail = tail_check(cp, b, lane, sh);
    tail_held_t held[kTailBatch];
    const bool ahead = tail.bad == 0 && tid < 2 * cp.Hkv * (cp.D / 8);
    if (ahead) tail_load(tail_column(cp, tid), sh, 0, held);
    READER_STAMP(kStampAccepted, 0);
    if (tid < 64) {
        const bool go = keep(AgentMarks{lane}, marks.keepers + b, marks.any_left, marks.token,
                             [&] { return all_here(marks.landed, marks.n_wg, marks.token, lane); }, (unsigned)j.wait_ticks * kKeeperPatience);
        if (lane == 0) s_append = go ? 1 : 0;
    }
    __syncthreads();
    if (s_append) keep_rows<kKeeperThreads>(cp, b, tid, tail, sh, ahead, held);
    READER_STAMP(kStampAppended, 0);
}

// What a workgroup whose launch waits inside keeps in LDS for its wavefronts.
struct JoinShared {
    mark_t left;        // shares of the pair whose workgroups have left, one bit each
    int complete;       // all shares have written their records
    int local;          // ... on this workgroup's XCD
    int append;         // (a keeper's) the rows may be appended
};

// kStep, kJoin: the fused step in one launch.  Workgroups that keep a sequence's cache each (keep_sequence) accept meanwhile, and
// append when everybody's keys have landed; the shares of a cut pair wait for one another and merge its rows together, on one
// XCD.  A second launch costs 4 to 5 us, of which 2.2 are the launch.  What takes its place, from time stamps: 0.25 us until a
// share's records are written through, 0.6 to 0.8 until the last one's mark is seen, 2.0 for the merge of ten shares of 24 pairs with
// 100 rows (0.9 on 512 tokens at head dimension 64); and an append that ends before the last share's rows.
// Whole steps: 512 tokens 10.0 -> 8.0 us, five sequences of 100 tokens, whole pairs, 12.8 -> 8.9; with the tree in the cache
// (three launches before) 19.7 -> 12.5.  Acceptance by the first copying wavefront of an attention workgroup instead made that
// workgroup's first keys 0.9 us late and its append 1.7; merging inside the launches of reader_tree_attn as well gained nothing
// with an earlier merge (one prompt of 4 K tokens 16.1 -> 15.8 us, 512 tokens 7.4 -> 8.4; other shapes, and today's merge, not tried).
//
// Whole pairs of more sequences than run at once: the keepers, last in the grid, come to run when nobody waits for a place
// any more (44 sequences of 237 tokens, 24 nodes, 29.8 -> 24.2 us, at head dimension 64 17.5 -> 14.0).
//
// kStep alone: a step of more launches than one (on a stream that is being captured, of more workgroups than there are marks for,
// or where a pair's shares leave a keeper no place).  Acceptance reads tokens only and writes nothing that an attention launch
// reads, so the first copying wavefront of a sequence's first workgroup does it: the tokens arrive with the page ids, and when
// the last tile has landed it chooses the path, while the others compute that tile and write their records.  The accepted rows
// wait for the next launch, as everybody reads the lengths.  Where pairs are cut and the second launch has little to merge (the
// rule is at the launch) acceptance stood in front of the append there and made it the longest job: one prompt of 4 K tokens 17.9 ->
// 17.3 us (half of that with the path chosen in front of the wait for the first tile, which that workgroup's others then wait for), 8 K
// 22.3 -> 21.5, 128 nodes 22.3 -> 21.4.  Whole pairs (44 sequences of 237 tokens, captured), chosen in front of the first tile before,
// 30.6 -> 27.2.
template <int D, bool kStep, bool kJoin>
__device__ __forceinline__ void tree_attn_short_body(const AttnParams &p, const JoinParams &j) {
    constexpr bool kDeep = D == 128;
    constexpr int CW = 4, kS = kShortStages;
    using G = Geometry<D, CW>;
    constexpr int kCopiesPerTile = 2 * G::kCopies;   // per copying wavefront
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    char *ring = smem;                                                               // [kS][kStageBytes]
    int *s_par = reinterpret_cast<int *>(smem + kS * G::kStageBytes);                // [4][READER_MAX_T]: one copy per computing wavefront
    int *s_hole = s_par + 4 * READER_MAX_T;                                          // [kS][4]: quarter of the tile behind a bad page id
    JoinShared *s_join = reinterpret_cast<JoinShared *>(s_hole + 4 * kS);            // (where the launch waits inside)
    TailShared *s_tail = reinterpret_cast<TailShared *>(s_join + (kJoin ? 1 : 0));   // (the fused step; not all of it where the launch does not wait)
    AcceptShared *s_accept = &s_tail->accept;
    const unsigned ring_lds = (unsigned)(size_t)(lds_char *)ring;

    READER_STAMP(kStampEntry, 0);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int split, hkv, chunk, b, wg = 0;
    if constexpr (kJoin) {
        // All shares of a pair's chunk get ids that are equal modulo 8: one XCD, whose L2 then holds the records to be merged.
        const int k = blockIdx.x >> 3, pairs = p.B * p.Hkv, units = pairs * p.n_row_chunks;
        if (k >= j.units_per_xcd * p.n_splits) {
            keep_sequence(p, j, blockIdx.x - kNumXCD * j.units_per_xcd * p.n_splits, *s_tail, s_join->append);
            return;
        }
        // (quotients of small numbers by way of floats: exact)
        split = __builtin_amdgcn_readfirstlane((int)(((float)k + 0.5f) * j.units_per_xcd_rcp));
        const int unit = ((blockIdx.x + j.spread * split) & 7) + 8 * (k - split * j.units_per_xcd);
        if (unit >= units) return;
        chunk = p.n_row_chunks == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)(((float)unit + 0.5f) * j.pairs_rcp));
        const int pair = unit - chunk * pairs;
        b = p.B == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)(((float)pair + 0.5f) * j.hkv_rcp));
        hkv = pair - b * p.Hkv;
        wg = unit * p.n_splits + split;
    } else {
        split = blockIdx.x, hkv = blockIdx.y;
        chunk = p.n_row_chunks == 1 ? 0 : blockIdx.z / p.B, b = blockIdx.z - chunk * p.B;
    }
    const int32_t *table = p.page_table + (size_t)b * p.max_pages;
    bool whole = p.n_splits == 1;      // the pair's tiles are all this workgroup's (or all another one's): no record
    // this workgroup's tiles [lo, hi) of the pair (prefix tiles, then tree tiles), once the length is there
    int L, n_pre, lo, hi;
    auto share = [&]() {
        L = __builtin_amdgcn_readfirstlane(clamp_len(p, p.seq_lens, b));
        n_pre = (L + kTile - 1) / kTile;
        const int n_all = n_pre + p.n_tree_tiles;
        if (p.keep_whole) {
            // The ring kernels give each of n_ranges workgroups an even share of all tiles (and pair_cost positions a
            // pair).  A pair that fits one such share may have been finished in place there, in fp32 and rounded once: it
            // is not cut here either.  Its workgroup has no more to do than one of the ring kernels'.
            int v = 0;
            for (int i = lane; i < p.B; i += 64) v += (clamp_len(p, p.seq_lens, i) + kTile - 1) / kTile + p.n_tree_tiles + p.pair_cost;
            const int all = p.Hkv * __builtin_amdgcn_readlane(wave_inclusive_scan(v), 63);   // (below 2^30: at most 256 pairs are cut)
            if ((n_all - 1) * p.n_ranges < all) {
                lo = split == 0 ? 0 : n_all;
                hi = n_all;
                whole = kJoin;
                return;
            }
        }
        lo = (int)(((float)(split * n_all) + 0.5f) * p.split_rcp);         // (exact: the host keeps the products below 2^22)
        hi = (int)(((float)((split + 1) * n_all) + 0.5f) * p.split_rcp);
        lo = __builtin_amdgcn_readfirstlane(lo);
        hi = __builtin_amdgcn_readfirstlane(hi);
    };
    int bad = 0;
    bool some_left = false;            // a keeper has left before this workgroup's keys had landed

    if (wave >= 4) {
        // ---------------- wavefronts that only move data ----------------
        const int cw = wave - 4;              // takes the 16 keys of page 4 t + cw of prefix tile t
        const int n_table = min(p.max_pages, (p.max_seq_len + READER_PAGE_SIZE - 1) / READER_PAGE_SIZE);
        int page[kPageRegs];
        int page_base = 0;                    // tile whose page is in lane 0 of page[0]
        auto fetch_pages = [&]() {
#pragma unroll
            for (int i = 0; i < kPageRegs; ++i) {
                const int at = (page_base + i * 64 + lane) * 4 + cw;
                page[i] = at < n_table ? table[at] : -1;
            }
        };
        const bool early = n_table <= kPageRegs * 64 * 4;   // all the sequence can have: asked for before its length is known
        if (early) fetch_pages();
        const bool side = kStep && !kJoin && cw == 0 && chunk == 0 && hkv == 0 && split == 0;
        AcceptTokens tok;
        if (side) tok = accept_load(late_argument<AcceptParams, offsetof(StepParams, accept)>(), b, lane);
        share();
        if (!early) {
            page_base = lo;
            fetch_pages();
        }
        const CopyLane<D, CW> cl = make_copy_lane<D, CW>(p, cw, lane);
        // page ids of the tree rows where those live in the cache (rows of a tile are not aligned to pages)
        int tree_page[2] = {-1, -1};
        if (p.tree_in_cache && hi > n_pre) {
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) {
                const int row = tt * kTile + cw * 16 + (lane & 15);
                if (row < p.T) tree_page[tt] = table[(L + row) >> 4];      // (inside the table: checked on the host)
            }
        }
#pragma unroll
        for (int i = 0; i < kPageRegs; ++i) asm volatile("" : "+v"(page[i]));   // (waited for in front of the copies)
        AcceptNodes nodes;
        if (side) nodes = accept_stage(late_argument<AcceptParams, offsetof(StepParams, accept)>(), lane, tok, *s_accept);    // (here with the page ids: a wait behind the copies would be for those too)
        READER_STAMP(kStampRange, 256);
        auto issue = [&](int t) {
            const unsigned at = (unsigned)(t - lo) % kS;
            const unsigned dst = ring_lds + at * G::kStageBytes + cw * G::kRowsPerWave * G::kRowBytes;
            const char *zeros = reinterpret_cast<const char *>(kZeroRow) + (lane & 15) * 16;
            if (t < n_pre) {
                const int i = t - page_base;
                const int id = __builtin_amdgcn_readlane(i < 64 ? page[0] : i < 128 ? page[1] : i < 192 ? page[2] : page[3], i & 63);
                const int n_valid = L - t * kTile - cw * 16;               // rows of this wavefront that exist
                const bool fits = id >= 0 && id < p.num_pages;
                const bool hole = !fits && n_valid > 0;
                if (hole) bad |= READER_STATUS_BAD_PAGE;
                if (lane == 0) s_hole[at * 4 + cw] = hole ? 1 : 0;
                const int blk = __builtin_amdgcn_readfirstlane((fits ? id : 0) * p.Hkv + hkv);   // (below 2^31: checked on the host)
                const size_t off = (size_t)blk * (READER_PAGE_SIZE * G::kRowBytes);
                const char *kb = reinterpret_cast<const char *>(p.k_cache) + off, *vb = reinterpret_cast<const char *>(p.v_cache) + off;
                if (fits && n_valid >= 16) {
#pragma unroll
                    for (int c = 0; c < G::kCopies; ++c) copy16_uniform(kb, cl.k_cache_off[c], dst + c * 1024);
#pragma unroll
                    for (int c = 0; c < G::kCopies; ++c) copy16_uniform(vb, cl.v_cache_off[c], dst + G::kTileBytes + c * 1024);
                } else {
#pragma unroll
                    for (int c = 0; c < G::kCopies; ++c) {
                        const bool ok = fits && cl.row[c] - cw * 16 < n_valid;
                        copy16_lane(ok ? kb + cl.k_cache_off[c] : zeros, dst + c * 1024);
                        copy16_lane(ok ? vb + cl.v_cache_off[c] : zeros, dst + G::kTileBytes + c * 1024);
                    }
                }
            } else {
                const int tt = t - n_pre;
                if (lane == 0) s_hole[at * 4 + cw] = 0;
                const size_t origin = (((size_t)b * p.T + tt * kTile) * p.Hkv + hkv) * G::kRowBytes;
#pragma unroll
                for (int c = 0; c < G::kCopies; ++c) {
                    bool ok = tt * kTile + cl.row[c] < p.T;
                    const char *ks, *vs;
                    if (p.tree_in_cache) {
                        const int pos = L + tt * kTile + cl.row[c], in_quarter = cl.row[c] - cw * 16;
                        const int id = __shfl(tt == 0 ? tree_page[0] : tree_page[1], in_quarter);
                        if (ok && !(id >= 0 && id < p.num_pages)) { bad |= READER_STATUS_BAD_PAGE; ok = false; }
                        const size_t off = (((size_t)id * p.Hkv + hkv) * READER_PAGE_SIZE + (pos & 15)) * G::kRowBytes;
                        const unsigned in_row = (unsigned)in_quarter * G::kRowBytes;   // (the lane's offsets count from row 0 of a page)
                        ks = reinterpret_cast<const char *>(p.k_cache) + off + (cl.k_cache_off[c] - in_row);
                        vs = reinterpret_cast<const char *>(p.v_cache) + off + (cl.v_cache_off[c] - in_row);
                    } else {
                        ks = reinterpret_cast<const char *>(p.k_tree) + origin + cl.k_tree_off[c];
                        vs = reinterpret_cast<const char *>(p.v_tree) + origin + cl.v_tree_off[c];
                    }
                    copy16_lane(ok ? ks : zeros, dst + c * 1024);
                    copy16_lane(ok ? vs : zeros, dst + G::kTileBytes + c * 1024);
                }
            }
        };
#pragma unroll 1
        for (int i = 0; i < kS - 1 && lo + i < hi; ++i) {
            issue(lo + i);
            if (i == 0) READER_STAMP(kStampItem0Issued, 256);
        }
#pragma unroll 1
        for (int t = lo; t < hi; ++t) {
            // this wavefront's part of tile t has landed once at most its copies of the tiles behind it are outstanding
            const int ahead = hi - 1 - t;
            if (ahead >= kS - 2) wait_vmcnt<(kS - 2) * kCopiesPerTile>();
            else if (ahead == 1) wait_vmcnt<kCopiesPerTile>();
            else wait_vmcnt<0>();
            __syncthreads();   // tile t is complete in LDS; every wavefront is done with tile t - 1
            if (t + kS - 1 < hi) issue(t + kS - 1);
        }
        if (p.status && bad) atomicOr(p.status, bad);
        if (side) {
            const AcceptParams ap = late_argument<AcceptParams, offsetof(StepParams, accept)>();
            int bits;
            const int n = accept_choose(ap, lane, nodes, *s_accept, bits);
            accept_report(ap, b, lane, n, bits, *s_accept);
        }
        if constexpr (!kJoin) {
            return;
        } else {
            if (lo >= hi) __syncthreads();     // (no tile, so no barrier yet: now every wavefront has read the lengths)
            if (cw == 0) {
                const Marks marks(p, j);          // (the keys of the last tile are in LDS)
                some_left = arrive(AgentMarks{lane}, marks.landed + wg, marks.any_left, marks.token);
            }
        }
    }

    // ---------------- wavefronts that only compute ----------------
    if (wave < 4) {
    const int n = lane & 31, h = lane >> 5;
    const int row_local = wave * 32 + n;
    const int m_row = chunk * kShortRows + row_local;                        // query row inside the pair
    const bool row_real = m_row < p.M;
    const bool wave_active = chunk * kShortRows + wave * 32 < p.M;
    // m / G without an integer division: m + 0.5 is 0.5 / G away from the next multiple of G, far more than rounding
    const int node = row_real ? (int)(((float)m_row + 0.5f) * p.g_rcp) : 0;
    const int group = row_real ? m_row - node * p.G : 0;
    // (the length first: the page ids, which the first keys wait for, are then in front of the query rows)
    share();
    bf16x8 qf[G::kKSteps];
    if (wave_active) {
        const uint16_t *qrow = p.q + (((size_t)b * p.T + node) * p.Hq + hkv * p.G + group) * D + h * 8;
#pragma unroll
        for (int kk = 0; kk < G::kKSteps; ++kk) qf[kk] = __builtin_bit_cast(bf16x8, ld16(qrow + kk * 16));
    }
    int *my_par = s_par + wave * READER_MAX_T;
    int par_raw[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) par_raw[i] = lane + 64 * i < p.T ? p.parents[(size_t)b * p.T + lane + 64 * i] : -1;

    // ancestor-or-self sets of this lane's query row, where this share reaches the tree tiles
    uint32_t anc[4] = {0u, 0u, 0u, 0u};
    if (hi > n_pre && wave_active) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int t = lane + 64 * i;
            if (t < p.T) {
                const bool valid = t == 0 ? par_raw[i] == -1 : (par_raw[i] >= 0 && par_raw[i] < t);
                if (!valid) bad = READER_STATUS_BAD_TREE;                   // (a bad link counts as a root link)
                my_par[t] = valid ? par_raw[i] : -1;
            }
        }
        int t = row_real ? node : -1;
        while (__any(t >= 0)) {                                              // (parents decrease: at most T steps)
            if (t >= 0) {
                const uint32_t bit = 1u << (t & 31);
#pragma unroll
                for (int w = 0; w < 4; ++w) anc[w] |= (t >> 5) == w ? bit : 0u;
                t = my_par[t];
            }
        }
    }

    // per-lane LDS offsets of the operand reads inside a stage
    int k_rd[G::kKSteps];
#pragma unroll
    for (int kk = 0; kk < G::kKSteps; ++kk) k_rd[kk] = n * G::kRowBytes + (((2 * kk + h) ^ swizzle_k<D>(n)) << 4);
    int v_rd[G::kOBlocks];
    {
        const int i16 = lane & 15, g16 = (lane >> 4) & 1;
        const int key_lo = 4 * h + (i16 >> 2), c_lo = 2 * g16 + ((i16 & 3) >> 1);
#pragma unroll
        for (int db = 0; db < G::kOBlocks; ++db)
            v_rd[db] = G::kTileBytes + key_lo * G::kRowBytes + ((((db * 4) | c_lo) ^ swizzle_v<D>(key_lo)) << 4) + (i16 & 1) * 8;
    }

    f32x16 o[G::kOBlocks];
#pragma unroll
    for (int db = 0; db < G::kOBlocks; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    const float c2 = p.scale_log2;
    // the reference of a row is only raised when its maximum outgrows it by 2^8: weights stay <= 256, rescales are rare
    const float grow_margin = 8.f / c2;

#pragma unroll 1
    for (int t = lo; t < hi; ++t) {
        const unsigned at = (unsigned)(t - lo) % kS;
        const char *stage = ring + at * G::kStageBytes;
        __syncthreads();       // tile t is complete in LDS
        if (t == lo) READER_STAMP(kStampTileLanded, 0);
        if (t == lo + 1) READER_STAMP(kStampFirstTile, 0);
        if (!wave_active) continue;
        const int4 hole = *reinterpret_cast<const int4 *>(s_hole + at * 4);
        // S^T = K.Q^T: two 32-key blocks, two independent chains.  All operand fragments are asked for before they are
        // needed: a read takes some 130 cycles, four matrix instructions.
        bf16x8 ka[G::kKSteps][2];
#pragma unroll
        for (int kk = 0; kk < G::kKSteps; ++kk) {
            ka[kk][0] = *reinterpret_cast<const bf16x8 *>(stage + k_rd[kk]);
            ka[kk][1] = *reinterpret_cast<const bf16x8 *>(stage + k_rd[kk] + 32 * G::kRowBytes);
        }
        s16x4 vh[4][G::kOBlocks][2];   // V^T fragments of the four 16-key steps
        auto read_v_step = [&](int ks) {
#pragma unroll
            for (int db = 0; db < G::kOBlocks; ++db) {
                const char *src = stage + v_rd[db] + ks * 16 * G::kRowBytes;
                vh[ks][db][0] = lds_read_tr16(src);                         // keys +0..3 (+4h)
                vh[ks][db][1] = lds_read_tr16(src + 8 * G::kRowBytes);      // keys +8..11 (+4h)
            }
        };
        f32x16 s[2];
#pragma unroll
        for (int i = 0; i < 16; ++i) { s[0][i] = 0.f; s[1][i] = 0.f; }
#pragma unroll
        for (int kk = 0; kk < G::kKSteps; ++kk) {
            s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[kk][0], qf[kk], s[0], 0, 0, 0);
            s[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[kk][1], qf[kk], s[1], 0, 0, 0);
        }
        if constexpr (kDeep) {
            read_v_step(0);
            read_v_step(1);
            __builtin_amdgcn_sched_group_barrier(0x100, 2 * G::kKSteps + 1, 0);
#pragma unroll
            for (int j = 0; j < 2 * G::kKSteps; ++j) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        } else {
            __builtin_amdgcn_sched_group_barrier(0x100, 5, 0);
#pragma unroll
            for (int j = 0; j < 2 * G::kKSteps - 4; ++j) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
        }

        uint32_t pk[2][8];     // weights, bf16 pairs, in B-operand order
        auto weights = [&]() {
            const float mc = (m_run == -INFINITY) ? 0.f : m_run * c2;
            float l0 = 0.f, l1 = 0.f;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 16; i += 2) {
                    const float p0 = __builtin_amdgcn_exp2f(s[kb][i] * c2 - mc), p1 = __builtin_amdgcn_exp2f(s[kb][i + 1] * c2 - mc);
                    l0 += p0;
                    l1 += p1;
                    pk[kb][i >> 1] = pack_bf16x2(p0, p1);
                }
            return l0 + l1;
        };
        // A whole prefix tile behind the first takes its weights against the running references at once; the row maxima
        // are looked for only if one of them comes out huge (bf16 and fp32 share the exponent range: nothing is lost).
        const int n_valid = t < n_pre ? L - t * kTile : 0;
        const int holes = __builtin_amdgcn_readfirstlane(hole.x | hole.y << 1 | hole.z << 2 | hole.w << 3);
        // (head dimension 64 looks for them in every tile: the second way to the weights takes too many registers there)
        bool careful = !kDeep || t == lo || n_valid < kTile || holes != 0;
        float lsum = 0.f;
        if (kDeep && !careful) {
            lsum = weights();
            careful = __any(!(lsum < 0x1p40f));
        }
        if (careful) {
            // which keys this lane's row attends to; score i of block kb is key (i / 4) * 8 + 4 h + i % 4 of the block
            uint32_t bits[2] = {0xffffffffu, 0xffffffffu};
            if (t >= n_pre) {
                const bool second = t > n_pre;
                bits[0] = second ? anc[2] : anc[0];
                bits[1] = second ? anc[3] : anc[1];
            } else {
                if (n_valid < kTile) {
                    bits[0] = n_valid >= 32 ? 0xffffffffu : (1u << n_valid) - 1u;
                    bits[1] = n_valid <= 32 ? 0u : (1u << (n_valid - 32)) - 1u;
                }
                bits[0] &= (holes & 1 ? 0xffff0000u : 0xffffffffu) & (holes & 2 ? 0x0000ffffu : 0xffffffffu);
                bits[1] &= (holes & 4 ? 0xffff0000u : 0xffffffffu) & (holes & 8 ? 0x0000ffffu : 0xffffffffu);
            }
            if (__any((bits[0] & bits[1]) != 0xffffffffu)) {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    const uint32_t mine = bits[kb] >> (4 * h);
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if (!((mine >> ((i >> 2) * 8 + (i & 3))) & 1u)) s[kb][i] = -INFINITY;
                }
            }
            float mx0 = fmaxf(s[0][0], s[0][1]), mx1 = fmaxf(s[1][0], s[1][1]);
#pragma unroll
            for (int i = 2; i < 16; i += 2) {
                mx0 = fmaxf(fmaxf(mx0, s[0][i]), s[0][i + 1]);
                mx1 = fmaxf(fmaxf(mx1, s[1][i]), s[1][i + 1]);
            }
            float mx = fmaxf(mx0, mx1);
            {   // the other half of the row's keys sits in lane ^ 32
                const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
                mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
            }
            const bool grow = mx > m_run + grow_margin;     // also the first finite maximum (m_run = -inf)
            if (__any(grow)) {
                const float alpha = grow ? __builtin_amdgcn_exp2f((m_run - mx) * c2) : 1.f;   // m_run = -inf gives 0
                m_run = grow ? mx : m_run;
                l_run *= alpha;
                if (t != lo) {
#pragma unroll
                    for (int db = 0; db < G::kOBlocks; ++db)
#pragma unroll
                        for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
                }
            }
            // (a row whose every key so far was skipped gets a finite reference, so low that the first real score
            // overflows the check above and is handled here)
            if (holes) m_run = fmaxf(m_run, -1e30f);
            lsum = weights();
        }
        l_run += lsum;
        if constexpr (kDeep) {
            read_v_step(2);
            read_v_step(3);
        } else {
            read_v_step(0);
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            if (!kDeep && ks + 1 < 4) read_v_step(ks + 1);
            const int kb = ks >> 1, m2 = ks & 1;
            u32x4 pv;
            pv.x = pk[kb][4 * m2]; pv.y = pk[kb][4 * m2 + 1]; pv.z = pk[kb][4 * m2 + 2]; pv.w = pk[kb][4 * m2 + 3];
#pragma unroll
            for (int db = 0; db < G::kOBlocks; ++db) {
                const s16x8 a8 = __builtin_shufflevector(vh[ks][db][0], vh[ks][db][1], 0, 1, 2, 3, 4, 5, 6, 7);
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a8), __builtin_bit_cast(bf16x8, pv), o[db], 0, 0, 0);
            }
        }
        if constexpr (kDeep) {         // (the reads of the last two steps go out ahead of all products)
            __builtin_amdgcn_sched_group_barrier(0x100, 4 * G::kOBlocks, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 4 * G::kOBlocks, 0);
        }
    }
    READER_STAMP(kStampLastTile, 0);

    // ---- a pair that was not split is normalised and written out, a share leaves a record for the merge
    if (wave_active) {
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
        l_run = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
        const float inv = l_run > 0.f ? 1.f / l_run : 0.f;                   // (a row may see no key of a share)
        const size_t slot = ((((size_t)b * p.Hkv + hkv) * p.n_row_chunks + chunk) * p.n_splits + split);
        float *rec = p.workspace + slot * attn_slot_floats(D, kShortRows);
        uint16_t *orow = p.out + (((size_t)b * p.T + node) * p.Hq + hkv * p.G + group) * D;
        // A lane holds, per 8-wide chunk of the row, 4 values and its partner lane (lane ^ 32) the other 4: one half-wave
        // swap per pair of chunks gives every lane whole 16-byte chunks.  Records are [D / 8 chunks][rows][8 values].
#pragma unroll
        for (int db = 0; db < G::kOBlocks; ++db)
#pragma unroll
            for (int i4 = 0; i4 < 4; i4 += 2) {
                const uint32_t a0 = pack_bf16x2(o[db][4 * i4] * inv, o[db][4 * i4 + 1] * inv);
                const uint32_t a1 = pack_bf16x2(o[db][4 * i4 + 2] * inv, o[db][4 * i4 + 3] * inv);
                const uint32_t b0 = pack_bf16x2(o[db][4 * i4 + 4] * inv, o[db][4 * i4 + 5] * inv);
                const uint32_t b1 = pack_bf16x2(o[db][4 * i4 + 6] * inv, o[db][4 * i4 + 7] * inv);
                const auto s0 = __builtin_amdgcn_permlane32_swap(a0, b0, false, false);
                const auto s1 = __builtin_amdgcn_permlane32_swap(a1, b1, false, false);
                u32x4 w;
                w.x = s0[0]; w.y = s1[0]; w.z = s0[1]; w.w = s1[1];
                const int c = db * 4 + i4 + h;
                if (row_real && lo < hi) {                 // (of an empty share the merge looks at the maxima only)
                    u32x4 *rec16 = reinterpret_cast<u32x4 *>(rec) + (size_t)c * kShortRows + row_local;
                    if (whole) *reinterpret_cast<u32x4 *>(orow + c * 8) = w;
                    else if (kJoin) agent_store16(rec16, w);
                    else __builtin_nontemporal_store(w, rec16);
                }
            }
        if (row_real && h == 0) {
            float m_exp2 = m_run * c2;
            asm volatile("" : "+v"(m_exp2));      // (rounded here in every kernel: the lse of a whole pair has the bits of one from a record)
            if (!whole) {
                float *m_rec = rec + kShortRows * (D / 2) + row_local, *l_rec = m_rec + kShortRows;
                if constexpr (kJoin) {
                    agent_store(m_rec, m_exp2);
                    agent_store(l_rec, l_run);
                } else {
                    *m_rec = m_exp2;
                    *l_rec = l_run;
                }
            } else if (p.lse && lo < hi) {
                p.lse[((size_t)b * p.Hq + hkv * p.G + group) * p.T + node] = (m_exp2 + __builtin_amdgcn_logf(l_run)) * kLn2;
            }
        }
        READER_STAMP(kStampExit, 0);
    }
    if (p.status && bad) atomicOr(p.status, bad);
    if constexpr (kJoin) {
        if (lo >= hi) __syncthreads();
        wait_vmcnt<0>();                       // this wavefront's part of the record is where the others will look for it
    }
    }
    if constexpr (kJoin) {
        auto merge = [&]() __attribute__((always_inline)) {
            __syncthreads();                   // the records are written
            READER_STAMP(kStampWritten, 0);
            if (wave == 0) {
                const Marks marks(p, j);
                const mark_t xcc = my_xcc();
                const mark_t *of_pair = marks.written + (wg - split);
                mark_t seen = 0;
                auto look = [&] {
                    seen = agent_load(of_pair + min(lane, p.n_splits - 1));
                    return (bool)__all((seen & ~kMarkBits) == marks.token);
                };
                const bool complete = meet(AgentMarks{lane}, marks.written + wg, marks.token | xcc, look, (unsigned)j.wait_ticks);
                const mark_t have_left = __ballot((seen & kStateBits) == kLeft);
                const bool here = __all((seen & (kMarkBits & ~kStateBits)) == xcc);
                if (lane == 0) {
                    s_join->complete = complete ? 1 : 0;
                    s_join->local = here ? 1 : 0;
                    s_join->left = have_left;
                }
            }
            __syncthreads();
            READER_STAMP(kStampSeen, 0);
            if (!__builtin_amdgcn_readfirstlane(s_join->complete)) return;
            const mark_t left = s_join->left;
            const int local = __builtin_amdgcn_readfirstlane(s_join->local);
            // The rows of the pair's chunk are shared out among its shares' workgroups; those of the ones that have left are
            // done by everybody who is there (twice the same bytes, if by several).
#pragma unroll 1
            for (int s = 0; s < p.n_splits; ++s) {
                if (s != split && !__builtin_amdgcn_readfirstlane((int)((left >> s) & 1))) continue;
                if (local) merge_share<D, false>(p, b, hkv, chunk, s);
                else merge_share<D, true>(p, b, hkv, chunk, s);
            }
            READER_STAMP(kStampMerged, 0);
        };
        if (!whole) merge();
        if (some_left) {              // (one wavefront)
            const Marks marks(p, j);
            keep_for_others(p, marks, lane, *s_tail);
        }
    }
}

template <int D>
__global__ __launch_bounds__(kThreads, D == 64 ? kWavesPerSimd64 : 2) void tree_attn_short_kernel(AttnParams p) {
    tree_attn_short_body<D, false, false>(p, JoinParams());
}
template <int D>
__global__ __launch_bounds__(kThreads, D == 64 ? kWavesPerSimd64 : 2) void tree_attn_short_kernel(StepParams p) {   // (cut pairs of a step whose paths it chooses; a trace tells the two apart by their argument)
    tree_attn_short_body<D, true, false>(p.attn, JoinParams());
}
template <int D>
__global__ __launch_bounds__(kThreads, D == 64 ? kWavesPerSimd64 : 2) void verify_short_kernel(StepParams p) {
    tree_attn_short_body<D, true, false>(p.attn, JoinParams());
}
template <int D>
__global__ __launch_bounds__(kThreads, D == 64 ? kWavesPerSimd64 : 2) void verify_short_join_kernel(StepParams p) {
    tree_attn_short_body<D, true, true>(p.attn, p.join);
}

// What its first loads need stands in front of the other arguments, one by one: those words arrive in scalar registers with the
// launch (members of a structure do not), and the records are not asked for a trip to memory later.  16-layer decoding step of three
// users 259.6 -> 254.0 us.  (The same in front of the attention kernels' arguments: a step of 512 tokens 7.98 -> 8.12, one prompt of 4 K
// tokens alike; in front of verify_tail_short_kernel's, where the path and the append are what takes time: 17.7 -> 18.5 us.)
template <int D>
__global__ __launch_bounds__(256) void merge_short_kernel(float *workspace, uint16_t *out, int32_t n_splits, int32_t M, int32_t Hkv,
                                                          int32_t n_row_chunks, int32_t T, int32_t Hq, int32_t G, float g_rcp, AttnParams p) {
    p.workspace = workspace, p.out = out, p.n_splits = n_splits, p.M = M, p.Hkv = Hkv, p.n_row_chunks = n_row_chunks;
    p.T = T, p.Hq = Hq, p.G = G, p.g_rcp = g_rcp;
    merge_block<D>(p, blockIdx.z, blockIdx.y, blockIdx.x);
}

// Second launch of the fused step where pairs were cut: one workgroup per sequence that appends the rows of its path, and chooses
// that first where the attention launch has not, then the merge blocks.  The jobs touch disjoint data.
template <int D, bool kAccept>
__global__ __launch_bounds__(256) void verify_tail_short_kernel(AttnParams p, AcceptParams ap, CompactParams cp, int merge_blocks) {
    if ((int)blockIdx.x >= p.B) {
        const int m = blockIdx.x - p.B, pair = m / merge_blocks, seq = pair / p.Hkv;
        merge_block<D>(p, seq, pair - seq * p.Hkv, m - pair * merge_blocks);
        return;
    }
    step_tail<kAccept>(ap, cp, blockIdx.x, threadIdx.x);
}

template <int D, bool kStep, bool kJoin, bool kCut = false>
hipError_t launch_main(const AttnParams &p, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop, const AcceptParams *ap,
                       const CompactParams *cp, const JoinParams *jp) {
    using G = Geometry<D, 4>;
    constexpr size_t lds = (size_t)kShortStages * G::kStageBytes + (4 * READER_MAX_T + 4 * kShortStages) * sizeof(int) +
                           (kJoin ? sizeof(JoinShared) : 0) + (kStep ? (kJoin ? sizeof(TailShared) : sizeof(AcceptShared)) : 0);
    static_assert(kStep || !kJoin, "only the fused step waits inside a launch");
    const void *kernel = kJoin ? reinterpret_cast<const void *>(&verify_short_join_kernel<D>)
                       : kCut  ? reinterpret_cast<const void *>(static_cast<void (*)(StepParams)>(&tree_attn_short_kernel<D>))
                       : kStep ? reinterpret_cast<const void *>(&verify_short_kernel<D>)
                               : reinterpret_cast<const void *>(static_cast<void (*)(AttnParams)>(&tree_attn_short_kernel<D>));
    {
        static std::mutex guard;             // host threads may call in at the same time
        static bool allowed = false;
        std::lock_guard<std::mutex> lock(guard);
        if (!allowed) {
            const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) { (void)hipGetLastError(); return note_hip_error("hipFuncSetAttribute(short attention LDS size)", e); }
            allowed = true;
        }
    }
    const dim3 grid = kJoin ? dim3(kNumXCD * jp->units_per_xcd * p.n_splits + p.B) : dim3(p.n_splits, p.Hkv, p.B * p.n_row_chunks);
    const bool timed = ev_start && ev_stop;
    auto go = [&](auto *fn, const char *name, auto... args) {
        if (timed) hipExtLaunchKernelGGL(fn, grid, dim3(kThreads), lds, stream, ev_start, ev_stop, 0, args...);
        else hipLaunchKernelGGL(fn, grid, dim3(kThreads), lds, stream, args...);
        return note_hip_error(name, hipGetLastError());
    };
    if constexpr (kJoin) return go(verify_short_join_kernel<D>, "launch verify_short_join_kernel", StepParams{*jp, p, *ap, *cp});
    else if constexpr (kCut) return go(static_cast<void (*)(StepParams)>(&tree_attn_short_kernel<D>), "launch tree_attn_short_kernel", StepParams{JoinParams(), p, *ap, *cp});
    else if constexpr (kStep) return go(verify_short_kernel<D>, "launch verify_short_kernel", StepParams{JoinParams(), p, *ap, *cp});
    else return go(static_cast<void (*)(AttnParams)>(&tree_attn_short_kernel<D>), "launch tree_attn_short_kernel", p);
}

template <int D>
hipError_t launch_all(const AttnParams &p, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop, const AcceptParams *ap,
                      const CompactParams *cp, const JoinParams *jp) {
    const bool step = ap && cp;
    if (step && jp) return launch_main<D, true, true>(p, stream, ev_start, ev_stop, ap, cp, jp);
    if (step && p.n_splits == 1) {
        const hipError_t e = launch_main<D, true, false>(p, stream, ev_start, ev_stop, ap, cp, nullptr);
        if (e != hipSuccess || !cp->k_tree) return e;      // (in-cache layout: the rows move in a launch of their own)
        return launch_kv_compact(*cp, stream);
    }
    // Who accepts where pairs are cut.  In the attention launch acceptance lengthens a copying wavefront's work; in the second one
    // it stands in front of an append, beside the merge of B Hkv M rows.  Up to as many rows as here the append is the longer of the
    // two, and the step 0.3 to 1.6 us shorter without acceptance in front of it (16 sequences of 8 heads, 0.2 to 0.8 K positions, 16
    // rows, head dimension 64: 15.4 -> 14.9 us).  With more the merge is, and acceptance beside it costs nothing, in the attention launch 0.2 to
    // 1.8 us (the same with 128 rows 20.1 -> 21.8; 32 of 4 heads at head dimension 128 24.9 -> 25.7).
    const bool rides = step && p.B * p.Hkv * ((p.M + 7) / 8) <= 640;
    const hipError_t e = rides ? launch_main<D, true, false, true>(p, stream, ev_start, ev_stop, ap, cp, nullptr)
                               : launch_main<D, false, false>(p, stream, ev_start, ev_stop, nullptr, nullptr, nullptr);
    if (e != hipSuccess || p.n_splits == 1) return e;
    const int blocks = (p.M + 7) / 8 * (D / 64);           // of 8 rows x 8 chunks, four wavefronts
    if (step && (!rides || cp->k_tree)) {                  // (in-cache layout: the rows move in a launch of their own)
        const dim3 grid(p.B + p.B * p.Hkv * blocks);
        if (rides) hipLaunchKernelGGL((verify_tail_short_kernel<D, false>), grid, dim3(256), 0, stream, p, *ap, *cp, blocks);
        else hipLaunchKernelGGL((verify_tail_short_kernel<D, true>), grid, dim3(256), 0, stream, p, *ap, *cp, blocks);
        return note_hip_error("launch verify_tail_short_kernel", hipGetLastError());
    }
    hipLaunchKernelGGL(merge_short_kernel<D>, dim3(blocks, p.Hkv, p.B), dim3(256), 0, stream, p.workspace, p.out, p.n_splits, p.M, p.Hkv,
                       p.n_row_chunks, p.T, p.Hq, p.G, p.g_rcp, p);
    return note_hip_error("launch merge_short_kernel", hipGetLastError());
}

}  // namespace

hipError_t launch_tree_attn_short(const AttnParams &p, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop,
                                  const AcceptParams *ap, const CompactParams *cp, const JoinParams *jp) {
    return p.D == 64 ? launch_all<64>(p, stream, ev_start, ev_stop, ap, cp, jp) : launch_all<128>(p, stream, ev_start, ev_stop, ap, cp, jp);
}

}  // namespace reader
