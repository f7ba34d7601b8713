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
//   - no list and no barrier in front of the main loop.
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
        const unsigned wg = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;               \
        if (p.stamps && threadIdx.x == (who) && wg < kStampedWgs)                                         \
            p.stamps[(size_t)wg * kWgStamps + (k)] = (long long)__builtin_amdgcn_s_memrealtime();         \
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

// kStep: the fused step where no pair is cut.  Acceptance reads tokens only and writes nothing that an attention launch
// reads, so the first copying wavefront of a sequence's first workgroup chooses the path while the first tiles are on their
// way and reports it when it has no more tiles to ask for.  The accepted rows wait for the next launch: a slot behind one
// sequence's end may lie inside the prefix of another one that this launch still reads (forks of unequal length that share a
// partly filled page), and so do the lengths, which every workgroup reads.  Whole steps, against acceptance in the second
// launch too: five sequences of 100 tokens, 32 nodes, 15.8 -> 14.6 us; 44 of 237, 24 nodes, 28.3 -> 27.3, at head dimension
// 64 14.9 -> 14.3; 64 of 300 to 500, 20 nodes, 40.7 -> 40.3.  (Cut pairs need a second launch for their merge anyway, which
// accepts as well.)
template <int D, bool kStep>
__device__ __forceinline__ void tree_attn_short_body(const AttnParams &p, const AcceptParams &ap) {
    constexpr bool kDeep = D == 128;
    constexpr int CW = 4, kS = kShortStages;
    using G = Geometry<D, CW>;
    constexpr int kCopiesPerTile = 2 * G::kCopies;   // per copying wavefront
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    char *ring = smem;                                                               // [kS][kStageBytes]
    int *s_par = reinterpret_cast<int *>(smem + kS * G::kStageBytes);                // [4][READER_MAX_T]: one copy per computing wavefront
    int *s_hole = s_par + 4 * READER_MAX_T;                                          // [kS][4]: quarter of the tile behind a bad page id
    AcceptShared *s_accept = reinterpret_cast<AcceptShared *>(s_hole + 4 * kS);      // (the fused step only)
    const unsigned ring_lds = (unsigned)(size_t)(lds_char *)ring;

    READER_STAMP(kStampEntry, 0);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int split = blockIdx.x, hkv = blockIdx.y;
    const int chunk = p.n_row_chunks == 1 ? 0 : blockIdx.z / p.B, b = blockIdx.z - chunk * p.B;
    const int32_t *table = p.page_table + (size_t)b * p.max_pages;
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
                return;
            }
        }
        lo = (int)(((float)(split * n_all) + 0.5f) * p.split_rcp);         // (exact: the host keeps the products below 2^22)
        hi = (int)(((float)((split + 1) * n_all) + 0.5f) * p.split_rcp);
        lo = __builtin_amdgcn_readfirstlane(lo);
        hi = __builtin_amdgcn_readfirstlane(hi);
    };
    int bad = 0;

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
        const bool side = kStep && cw == 0 && chunk == 0 && hkv == 0;
        AcceptTokens tok;
        if (side) tok = accept_load(ap, b, lane);
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
        if (side) nodes = accept_stage(ap, lane, tok, *s_accept);    // (here with the page ids: a wait behind the copies would be for those too)
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
        int accepted = 0, step_bits = 0;
        if (side) accepted = accept_choose(ap, lane, nodes, *s_accept, step_bits);
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
        if (side) accept_report(ap, b, lane, accepted, step_bits, *s_accept);
        return;
    }

    // ---------------- wavefronts that only compute ----------------
    const int n = lane & 31, h = lane >> 5;
    const int row_local = wave * 32 + n;
    const int m_row = chunk * kShortRows + row_local;                        // query row inside the pair
    const bool row_real = m_row < p.M;
    const bool wave_active = chunk * kShortRows + wave * 32 < p.M;
    const float g_rcp = 1.0f / (float)p.G;
    // m / G without an integer division: m + 0.5 is 0.5 / G away from the next multiple of G, far more than rounding
    const int node = row_real ? (int)(((float)m_row + 0.5f) * g_rcp) : 0;
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
    if (!wave_active) return;
    {
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
        l_run = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    }
    const bool whole = gridDim.x == 1;
    const float inv = l_run > 0.f ? 1.f / l_run : 0.f;                       // (a row may see no key of a share)
    const size_t slot = ((((size_t)b * p.Hkv + hkv) * p.n_row_chunks + chunk) * gridDim.x + split);
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
            if (row_real && (whole || lo < hi)) {          // (of an empty share the merge looks at the maxima only)
                if (whole) *reinterpret_cast<u32x4 *>(orow + c * 8) = w;
                else __builtin_nontemporal_store(w, reinterpret_cast<u32x4 *>(rec) + (size_t)c * kShortRows + row_local);
            }
        }
    if (row_real && h == 0) {
        if (!whole) {
            rec[kShortRows * (D / 2) + row_local] = m_run * c2;
            rec[kShortRows * (D / 2 + 1) + row_local] = l_run;
        } else if (p.lse) {
            p.lse[((size_t)b * p.Hq + hkv * p.G + group) * p.T + node] = (m_run * c2 + __builtin_amdgcn_logf(l_run)) * kLn2;
        }
    }
    READER_STAMP(kStampExit, 0);
    if (p.status && bad) atomicOr(p.status, bad);
}

template <int D>
__global__ __launch_bounds__(kThreads, D == 64 ? kWavesPerSimd64 : 2) void tree_attn_short_kernel(AttnParams p) {
    tree_attn_short_body<D, false>(p, AcceptParams());
}
template <int D>
__global__ __launch_bounds__(kThreads, D == 64 ? kWavesPerSimd64 : 2) void verify_short_kernel(AttnParams p, AcceptParams ap) {
    tree_attn_short_body<D, true>(p, ap);
}

// Merge of the n_splits records of every query row.  A record is laid out [chunk of 8 values][row], so a wavefront takes 16
// consecutive rows of four chunks: its loads fetch 256 contiguous bytes per chunk.  With more than eight shares the four
// wavefronts of a workgroup take a quarter of the shares each and fold their states through LDS in the order of the shares.
//
// What bounds it: a launch, one trip to memory for the records (other compute units have just written them past the
// caches) and the way back; loads are few and asked for together, four or eight records at a time.  As one thread per row and chunk
// in row order, eight records at a time whether there were that many or not, it took 6.6 us where this takes 4.2 (three
// sequences of 0.7 - 2.5 K tokens, ten shares of 24 pairs with 100 rows; four wavefronts per row from nine shares on there).
template <int D>
__device__ __forceinline__ void merge_short_body(const AttnParams &p, int b, int hkv, int block) {
    constexpr int kQuads = D / 32;                           // sets of four chunks in a row
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_splits = p.n_splits;
    const bool four = p.merge_groups == 4;
    const int unit = four ? block : block * 4 + wave;        // 16 rows x 4 chunks
    const int m = (unit / kQuads) * 16 + (lane & 15), c = (unit % kQuads) * 4 + (lane >> 4);
    const bool live = m < p.M;
    const int chunk = m / kShortRows, r = m % kShortRows;
    constexpr size_t kRec = attn_slot_floats(D, kShortRows);
    const float *rec = p.workspace + ((size_t)(b * p.Hkv + hkv) * p.n_row_chunks + (live ? chunk : 0)) * n_splits * kRec;
    const int share = four ? (n_splits + 3) >> 2 : n_splits, first = four ? wave * share : 0, last = min(n_splits, first + share);
    MergeState st;
    auto take = [&](auto batch_c) __attribute__((always_inline)) {
        constexpr int kBatch = decltype(batch_c)::value;
        for (int s0 = first; s0 < last; s0 += kBatch) {
            float ms[kBatch], ls[kBatch];
            uint4 v[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const float *part = rec + (size_t)min(s0 + j, last - 1) * kRec;
                v[j] = reinterpret_cast<const uint4 *>(part)[c * kShortRows + r];
                ms[j] = part[kShortRows * (D / 2) + r];
                ls[j] = part[kShortRows * (D / 2 + 1) + r];
            }
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                if (s0 + j >= last || ms[j] == -INFINITY) continue;      // (no key of that share for this row)
                st.fold_record(ms[j], ls[j], v[j]);
            }
        }
    };
    // (a second round is a second trip to memory, a record read twice only a load)
    if (share > 4) take(std::integral_constant<int, 8>{});
    else take(std::integral_constant<int, 4>{});
    if (four) {
        __shared__ float s_state[3][10][64];
        if (!st.gather(s_state, wave, lane)) return;
    }
    if (!live) return;
    // m / G without an integer division: m + 0.5 is 0.5 / G away from the next multiple of G, far more than rounding
    const int node = (int)(((float)m + 0.5f) * (1.0f / (float)p.G)), group = m - node * p.G;
    *reinterpret_cast<uint4 *>(p.out + (((size_t)b * p.T + node) * p.Hq + hkv * p.G + group) * D + c * 8) = st.result();
    if (p.lse && c == 0)
        p.lse[((size_t)b * p.Hq + hkv * p.G + group) * p.T + node] = (st.m + __builtin_amdgcn_logf(st.l)) * kLn2;
}

template <int D>
__global__ __launch_bounds__(256) void merge_short_kernel(AttnParams p) {
    merge_short_body<D>(p, blockIdx.z, blockIdx.y, blockIdx.x);
}

// Tail of the fused step where pairs were cut: one workgroup per sequence that accepts a path and appends its rows, then the
// merge blocks.  The jobs touch disjoint data.
template <int D>
__global__ __launch_bounds__(256) void verify_tail_short_kernel(AttnParams p, AcceptParams ap, CompactParams cp, int merge_blocks) {
    if ((int)blockIdx.x >= p.B) {
        const int m = blockIdx.x - p.B, pair = m / merge_blocks, seq = pair / p.Hkv;
        merge_short_body<D>(p, seq, pair - seq * p.Hkv, m - pair * merge_blocks);
        return;
    }
    __shared__ AcceptShared sh;
    __shared__ CompactShared cs;
    const int b = blockIdx.x, tid = threadIdx.x;
    const bool append = cp.k_tree != nullptr;       // (in-cache layout: the rows move in a launch of their own)
    if (append) kv_compact_prefetch(cp, b, tid, cs);
    if (tid < 64) accept_path_wave(ap, b, tid, sh);
    if (!append) return;
    __syncthreads();
    kv_compact_body(cp, b, tid, sh.accept_len, sh.path, cs);
}

template <int D, bool kStep>
hipError_t launch_main(const AttnParams &p, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop, const AcceptParams *ap) {
    using G = Geometry<D, 4>;
    constexpr size_t lds = (size_t)kShortStages * G::kStageBytes + (4 * READER_MAX_T + 4 * kShortStages) * sizeof(int) +
                           (kStep ? sizeof(AcceptShared) : 0);
    {
        static std::mutex guard;             // host threads may call in at the same time
        static bool allowed = false;
        std::lock_guard<std::mutex> lock(guard);
        if (!allowed) {
            const void *kernel = kStep ? reinterpret_cast<const void *>(&verify_short_kernel<D>) : reinterpret_cast<const void *>(&tree_attn_short_kernel<D>);
            const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) { (void)hipGetLastError(); return note_hip_error("hipFuncSetAttribute(short attention LDS size)", e); }
            allowed = true;
        }
    }
    const dim3 grid(p.n_splits, p.Hkv, p.B * p.n_row_chunks);
    const bool timed = ev_start && ev_stop;
    if constexpr (kStep) {
        if (timed) hipExtLaunchKernelGGL(verify_short_kernel<D>, grid, dim3(kThreads), lds, stream, ev_start, ev_stop, 0, p, *ap);
        else hipLaunchKernelGGL(verify_short_kernel<D>, grid, dim3(kThreads), lds, stream, p, *ap);
    } else {
        if (timed) hipExtLaunchKernelGGL(tree_attn_short_kernel<D>, grid, dim3(kThreads), lds, stream, ev_start, ev_stop, 0, p);
        else hipLaunchKernelGGL(tree_attn_short_kernel<D>, grid, dim3(kThreads), lds, stream, p);
    }
    return note_hip_error(kStep ? "launch verify_short_kernel" : "launch tree_attn_short_kernel", hipGetLastError());
}

template <int D>
hipError_t launch_all(const AttnParams &p, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop, const AcceptParams *ap,
                      const CompactParams *cp) {
    if (ap && cp && p.n_splits == 1) {
        const hipError_t e = launch_main<D, true>(p, stream, ev_start, ev_stop, ap);
        if (e != hipSuccess || !cp->k_tree) return e;      // (in-cache layout: the rows move in a launch of their own)
        return launch_kv_compact(*cp, stream);
    }
    const hipError_t e = launch_main<D, false>(p, stream, ev_start, ev_stop, nullptr);
    if (e != hipSuccess || p.n_splits == 1) return e;
    const int units = (p.M + 15) / 16 * (D / 32);          // of 16 rows x 4 chunks
    const int blocks = p.merge_groups == 4 ? units : (units + 3) / 4;
    if (ap && cp) {
        hipLaunchKernelGGL(verify_tail_short_kernel<D>, dim3(p.B + p.B * p.Hkv * blocks), dim3(256), 0, stream, p, *ap, *cp, blocks);
        return note_hip_error("launch verify_tail_short_kernel", hipGetLastError());
    }
    hipLaunchKernelGGL(merge_short_kernel<D>, dim3(blocks, p.Hkv, p.B), dim3(256), 0, stream, p);
    return note_hip_error("launch merge_short_kernel", hipGetLastError());
}

}  // namespace

hipError_t launch_tree_attn_short(const AttnParams &p, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop,
                                  const AcceptParams *ap, const CompactParams *cp) {
    return p.D == 64 ? launch_all<64>(p, stream, ev_start, ev_stop, ap, cp) : launch_all<128>(p, stream, ev_start, ev_stop, ap, cp);
}

}  // namespace reader
