// Periodic rearrangement of a padded KV cache (Section 4.3 / Algorithm 4 of the READER paper):
// per sample, internal padding is removed and the real entries are concatenated tightly, in
// place, so that padding may only remain at the end.
//
// Two kernels.
//   plan:   one workgroup per sample scans its validity flags: every valid position gets its
//           destination (the number of valid positions before it), noted the other way round:
//           source[d] = the position whose row goes to d; the sample's new length n, its old
//           extent (last valid position + 1) and its first hole are noted; for the positions
//           from n on (their slots of `source` are free) it is noted whether they held a row;
//           the flags become ones-then-zeros.
//   apply:  two kinds of workgroup in one launch, which never touch the same bytes.
//           Movers, one per (sample, kv head, layer), walk the destinations from the first hole
//           to n in passes: all rows of a pass are loaded (128-bit accesses) before any is
//           stored, and sources never lie to the left of their destinations, so the move is
//           safe in place (a pass writes [a, a + P); the sources of later passes lie at or
//           behind a + P); a source at or behind n is cleared once it has been read.  Rows in
//           front of the first hole are not touched, so a pass moves only what acceptance spans
//           of unequal length have left out of place: few rows, scattered (memory serves such
//           pieces at a fraction of its streaming rate).
//           Clearers take the positions between n and the old extent that held no row: per
//           (sample, layer) one stretch of K and one of V, contiguous but for the few sources
//           in it, cut into pieces for as many workgroups as fill the GPU.  This is most of the
//           traffic of a pass (a short prompt leaves a long hole in front of the first decoding
//           step); as plain stores it runs at the rate of a fill, with the movers underneath.
#include "internal.h"

namespace reader {

namespace {

constexpr int kPlanThreads = 1024;
constexpr int kPlanPerThread = 8;                    // consecutive positions of a thread per round
constexpr int kPlanRound = kPlanThreads * kPlanPerThread;

// The 8 flags of positions j0.. of a sample as bits; positions from S on count as empty.
__device__ inline unsigned plan_flags(const uint8_t *valid, int j0, int S, bool aligned) {
    unsigned mask = 0u;
    if (aligned && j0 + kPlanPerThread <= S) {
        const uint64_t w = *reinterpret_cast<const uint64_t *>(valid + j0);
#pragma unroll
        for (int i = 0; i < kPlanPerThread; ++i) mask |= ((w >> (8 * i)) & 0xff) != 0 ? 1u << i : 0u;
    } else {
        bool f[kPlanPerThread];
#pragma unroll
        for (int i = 0; i < kPlanPerThread; ++i) f[i] = j0 + i < S && valid[j0 + i] != 0;
#pragma unroll
        for (int i = 0; i < kPlanPerThread; ++i) mask |= f[i] ? 1u << i : 0u;
    }
    return mask;
}

// One workgroup per sample: few of them, so what counts is how many steps follow one another.  A thread takes 8
// consecutive positions of a round; the flags of a round (8192 positions) are asked for together and stay in
// registers for the second half, where a sample of one round, the usual case, reads nothing again; the count of the
// flags in front of a lane comes from ballots, not from a chain of shuffles.  16 samples of 4405 slots: 5.6 us (11.9 when
// the second half read the flags again, a trip to memory for every 1024 of them, and all threads met in two atomics).
__global__ __launch_bounds__(kPlanThreads) void rearrange_plan_kernel(RearrangeParams p) {
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint8_t *valid = p.valid + (size_t)b * p.S;
    int32_t *source = p.dest + (size_t)b * p.S;
    const bool aligned = (reinterpret_cast<uintptr_t>(valid) & 7) == 0;   // (the same for all threads)
    __shared__ int s_wsum[kPlanThreads / 64];
    __shared__ int s_first_hole, s_extent;
    if (tid == 0) { s_first_hole = p.S; s_extent = 0; }

    int carry = 0;
    unsigned mask = 0u;
    for (int base = 0; base < p.S; base += kPlanRound) {
        const int j0 = base + tid * kPlanPerThread;
        mask = plan_flags(valid, j0, p.S, aligned);
        unsigned before = 0u;                          // valid positions of the lanes in front, in this wavefront
        int mine_all = 0;                              // ... and of all its lanes
#pragma unroll
        for (int i = 0; i < kPlanPerThread; ++i) {
            const uint64_t set = __ballot((mask >> i) & 1u);
            before = __builtin_amdgcn_mbcnt_hi((unsigned)(set >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)set, before));
            mine_all += __popcll(set);
        }
        if (lane == 0) s_wsum[wave] = mine_all;
        __syncthreads();
        int woff = 0, total = 0;
#pragma unroll
        for (int w = 0; w < kPlanThreads / 64; ++w) {
            const int x = s_wsum[w];
            if (w < wave) woff += x;
            total += x;
        }
        int d = carry + woff + (int)before;            // valid positions in front of j0
#pragma unroll
        for (int i = 0; i < kPlanPerThread; ++i)
            if ((mask >> i) & 1u) source[d++] = j0 + i;
        // the wavefront's first hole and last valid position: the lane that holds it reports it
        const uint64_t holes = __ballot(mask != (1u << kPlanPerThread) - 1u), held = __ballot(mask != 0u);
        if (holes != 0 && lane == (int)__builtin_ctzll(holes)) {
            const int j = j0 + __builtin_ctz(~mask);
            if (j < p.S) atomicMin(&s_first_hole, j);
        }
        if (held != 0 && lane == 63 - (int)__builtin_clzll(held)) atomicMax(&s_extent, j0 + 32 - __builtin_clz(mask));
        carry += total;
        __syncthreads();
    }
    // every flag has been read; all threads know the new length (carry)
    for (int base = 0; base < p.S; base += kPlanRound) {
        const int j0 = base + tid * kPlanPerThread;
        if (p.S > kPlanRound) mask = plan_flags(valid, j0, p.S, aligned);
        uint64_t w = 0;
#pragma unroll
        for (int i = 0; i < kPlanPerThread; ++i) {
            const int j = j0 + i;
            if (j >= carry && j < p.S) source[j] = (mask >> i) & 1u;   // (destinations end at carry - 1: these slots are free)
            w |= j < carry ? 1ull << (8 * i) : 0ull;
        }
        if (aligned && j0 + kPlanPerThread <= p.S) {
            *reinterpret_cast<uint64_t *>(valid + j0) = w;
        } else {
#pragma unroll
            for (int i = 0; i < kPlanPerThread; ++i)
                if (j0 + i < p.S) valid[j0 + i] = (uint8_t)(w >> (8 * i));
        }
    }
    if (tid == 0) {
        p.new_len[b] = carry;
        int32_t *meta = p.dest + (size_t)p.B * p.S + (size_t)b * 4;
        meta[0] = carry;
        meta[1] = s_extent;
        meta[2] = s_first_hole;
    }
}

constexpr int kApplyThreads = 256;
constexpr int kMoveSub = 4;                          // groups of rows a mover's thread carries through one pass
constexpr int kZeroPerThread = 8;                    // 16-byte stores per clearer thread and tensor
constexpr int kZeroChunks = kApplyThreads * kZeroPerThread;   // 16-byte chunks of K (and of V) a clearer takes at a time

template <int D>
__device__ inline void rearrange_move(const RearrangeParams &p, int b, int hkv, int layer) {
    constexpr int kThreadsPerRow = D / 8;            // 16-byte chunks of one (position, kv head) row
    constexpr int kRowsPerGroup = kApplyThreads / kThreadsPerRow;
    const int tid = threadIdx.x, r = tid / kThreadsPerRow, c = tid % kThreadsPerRow;
    const int32_t *source = p.dest + (size_t)b * p.S;
    const int32_t *meta = p.dest + (size_t)p.B * p.S + (size_t)b * 4;
    const int n = meta[0], extent = meta[1], first_hole = meta[2];
    if (first_hole >= extent) return;               // no hole inside the sample: nothing to do

    const size_t pos_stride = (size_t)p.Hkv * D;    // elements between consecutive positions
    uint16_t *k = p.k_pad + (((size_t)layer * p.B + b) * p.S) * pos_stride + (size_t)hkv * D + c * 8;
    uint16_t *v = p.v_pad + (((size_t)layer * p.B + b) * p.S) * pos_stride + (size_t)hkv * D + c * 8;
    const uint4 zero = make_uint4(0u, 0u, 0u, 0u);

    // destinations first_hole .. n - 1, in passes of kMoveSub groups: the sources of a pass are asked for
    // together, then their rows, so that a pass costs two memory round trips
    for (int base = first_hole; base < n; base += kRowsPerGroup * kMoveSub) {
        int src[kMoveSub];
        uint4 kv[kMoveSub], vv[kMoveSub];
#pragma unroll
        for (int u = 0; u < kMoveSub; ++u) {
            const int d = base + u * kRowsPerGroup + r;
            src[u] = d < n ? source[d] : -1;
        }
#pragma unroll
        for (int u = 0; u < kMoveSub; ++u) {
            kv[u] = zero; vv[u] = zero;
            if (src[u] >= 0) {
                kv[u] = *reinterpret_cast<const uint4 *>(k + (size_t)src[u] * pos_stride);
                vv[u] = *reinterpret_cast<const uint4 *>(v + (size_t)src[u] * pos_stride);
            }
        }
        __syncthreads();   // every row of the pass is in registers (the barrier waits for the loads)
#pragma unroll
        for (int u = 0; u < kMoveSub; ++u) {
            const int d = base + u * kRowsPerGroup + r;
            if (src[u] >= 0) {
                *reinterpret_cast<uint4 *>(k + (size_t)d * pos_stride) = kv[u];
                *reinterpret_cast<uint4 *>(v + (size_t)d * pos_stride) = vv[u];
                if (src[u] >= n) {                   // (no destination lies there: they end at n - 1)
                    *reinterpret_cast<uint4 *>(k + (size_t)src[u] * pos_stride) = zero;
                    *reinterpret_cast<uint4 *>(v + (size_t)src[u] * pos_stride) = zero;
                }
            }
        }
    }
}

// The `lanes` clearers of a (sample, layer) take the pieces of its stretch in turn.
__device__ inline void rearrange_clear(const RearrangeParams &p, int b, int first_piece, int lanes, int layer) {
    const int32_t *held_row = p.dest + (size_t)b * p.S;             // meaningful from position n on
    const int32_t *meta = p.dest + (size_t)p.B * p.S + (size_t)b * 4;
    const int n = meta[0], extent = meta[1], first_hole = meta[2];
    if (first_hole >= extent) return;
    const unsigned per_pos = (unsigned)p.Hkv * p.D / 8;              // 16-byte chunks of a position
    const unsigned positions = (unsigned)(extent - n);
    const size_t chunks = (size_t)positions * per_pos;
    const size_t stride = (size_t)lanes * kZeroChunks;               // from one piece of this workgroup to its next
    size_t begin = (size_t)first_piece * kZeroChunks;
    if (begin >= chunks) return;
    const size_t at = (((size_t)layer * p.B + b) * p.S + n) * per_pos;
    uint4 *k = reinterpret_cast<uint4 *>(p.k_pad) + at, *v = reinterpret_cast<uint4 *>(p.v_pad) + at;
    const uint4 zero = make_uint4(0u, 0u, 0u, 0u);

    // Bound by the stores (0.9 GB at 5.3 TB/s; the movers' scattered 0.14 GB add their own 25 us).  A chunk's position is
    // kept with its place in the position and moved on by additions, not found by a division per chunk.
    const unsigned row_pos = kApplyThreads / per_pos, row_rem = kApplyThreads % per_pos;   // from a thread's chunk to its next
    const unsigned jump_pos = (unsigned)(stride / per_pos), jump_rem = (unsigned)(stride % per_pos);
    unsigned pos = (unsigned)((begin + threadIdx.x) / per_pos), rem = (unsigned)((begin + threadIdx.x) % per_pos);
    auto held_of_piece = [&](int *held) {
        unsigned at_pos = pos, at_rem = rem;
#pragma unroll
        for (int i = 0; i < kZeroPerThread; ++i) {
            held[i] = at_pos < positions ? held_row[n + (int)at_pos] : 1;
            at_pos += row_pos;
            at_rem += row_rem;
            if (at_rem >= per_pos) { at_rem -= per_pos; ++at_pos; }
        }
    };
    // The notes of the next piece are asked for in front of this one's stores: the memory counter is in order, and a
    // wait for notes asked for behind them is a wait for the stores.
    int held[kZeroPerThread];
    held_of_piece(held);
    for (;;) {
        const size_t next = begin + stride;
        pos += jump_pos;
        rem += jump_rem;
        if (rem >= per_pos) { rem -= per_pos; ++pos; }
        int held_next[kZeroPerThread];
        if (next < chunks) held_of_piece(held_next);
#pragma unroll
        for (int i = 0; i < kZeroPerThread; ++i) {
            if (held[i] == 0) {                                       // (a position that held a row is its mover's)
                k[begin + (size_t)i * kApplyThreads + threadIdx.x] = zero;
                v[begin + (size_t)i * kApplyThreads + threadIdx.x] = zero;
            }
        }
        if (next >= chunks) break;
        begin = next;
#pragma unroll
        for (int i = 0; i < kZeroPerThread; ++i) held[i] = held_next[i];
    }
}

// 1-D grid: the movers of all layers first (their scattered accesses take longest), then the clearers
template <int D>
__global__ __launch_bounds__(kApplyThreads) void rearrange_apply_kernel(RearrangeParams p, int lanes) {
    const int per_layer = p.B * p.Hkv, movers = per_layer * p.NL;
    if ((int)blockIdx.x < movers) {
        const int layer = blockIdx.x / per_layer, i = blockIdx.x - layer * per_layer, b = i / p.Hkv;
        rearrange_move<D>(p, b, i - b * p.Hkv, layer);
    } else {
        const int c = blockIdx.x - movers, per = p.B * lanes;
        const int layer = c / per, i = c - layer * per, b = i / lanes;
        rearrange_clear(p, b, i - b * lanes, lanes, layer);
    }
}

}  // namespace

hipError_t launch_kv_rearrange(const RearrangeParams &p, hipStream_t stream) {
    hipLaunchKernelGGL(rearrange_plan_kernel, dim3(p.B), dim3(kPlanThreads), 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return note_hip_error("launch rearrange_plan_kernel", e);
    if (p.NL == 0) return hipSuccess;
    // clearers per (sample, layer): enough for 32 workgroups per compute unit over the whole grid, four times what is
    // resident, so that samples with short and long stretches even out (8, 16, 32 and 64 of them: 213, 205, 202 and 202 us
    // for 8 layers of 16 samples, 0.9 GB to clear; 22.3, 23.1, 21.9 and 22.3 for 27 layers of 8); no more than the
    // longest stretch has pieces
    const size_t longest = (size_t)p.S * p.Hkv * p.D / 8;            // chunks of one tensor a sample can have to clear
    const long long most = (long long)((longest + kZeroChunks - 1) / kZeroChunks);
    long long lanes = (32LL * kNumCU + (long long)p.B * p.NL - 1) / ((long long)p.B * p.NL);
    lanes = lanes < 1 ? 1 : (lanes > most ? most : lanes);
    if ((long long)p.NL * p.B * (p.Hkv + lanes) > 0x7fffffffLL) lanes = 1;   // (NL * B * (Hkv + 1) fits: checked by the caller)
    const dim3 grid((unsigned)((long long)p.NL * p.B * (p.Hkv + lanes)));
    if (p.D == 64)
        hipLaunchKernelGGL(rearrange_apply_kernel<64>, grid, dim3(kApplyThreads), 0, stream, p, (int)lanes);
    else
        hipLaunchKernelGGL(rearrange_apply_kernel<128>, grid, dim3(kApplyThreads), 0, stream, p, (int)lanes);
    return note_hip_error("launch rearrange_apply_kernel", hipGetLastError());
}

}  // namespace reader
