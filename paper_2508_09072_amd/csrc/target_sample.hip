// The base model's tokens under a sampling policy with coupled uniforms (Appendix C,
// randomized decoding): the policy is a map F(distribution, u) with one uniform per decoding
// position, shared by the plain run and the speculative run.  Here F is inverse-CDF sampling of
// softmax(logits / temperature): the lowest index whose cumulative probability exceeds u.
// Node n of sequence b stands for the position depth(n) behind the root, so all nodes of one
// depth draw with the same uniform, uniforms[b][depth(n)].
//
// One workgroup per (sequence, node) row, one pass over the row (256 KB at vocabulary 128256,
// as large as the step's KV stream): the row is cut into slots of 2048 consecutive tokens (four
// 16-byte loads per lane), a wavefront reduces a slot to (maximum, sum of exp relative to that
// maximum) and leaves the pair in LDS, with the loads of its next slot on their way meanwhile.
// The rest is one wavefront's work without a barrier (a barrier per reduction made the end of a
// row as long as a third of its stream): the slots' sums, brought to the row maximum, are scanned
// in index order to find the slot that crosses u * total, and only that slot (4 KB, still in
// cache) is read again to find the token.  All sums are fp32: where u * total falls within rounding of a
// token boundary the neighbouring token may come out.
#include <stdlib.h>

#include "internal.h"

namespace reader {

namespace {

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
constexpr int kGroup = 4;            // 512-token blocks (64 lanes x 8 tokens) per slot

// Wavefront reductions on the vector ALU's lane-crossing paths (no LDS traffic): four shifts
// inside each row of 16 lanes leave the row's result in its last lane, two row broadcasts
// carry it on to lane 63, which is read back as a wavefront-uniform value.
template <int kCtrl, int kRowMask>
__device__ inline float dpp_from(float identity, float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(identity), __float_as_int(v), kCtrl, kRowMask, 0xf, false));
}
__device__ inline float wave_max(float v) {
    v = fmaxf(v, dpp_from<0x111, 0xf>(-INFINITY, v));   // row_shr:1
    v = fmaxf(v, dpp_from<0x112, 0xf>(-INFINITY, v));   // row_shr:2
    v = fmaxf(v, dpp_from<0x114, 0xf>(-INFINITY, v));   // row_shr:4
    v = fmaxf(v, dpp_from<0x118, 0xf>(-INFINITY, v));   // row_shr:8
    v = fmaxf(v, dpp_from<0x142, 0xa>(-INFINITY, v));   // row_bcast:15 into rows 1 and 3
    v = fmaxf(v, dpp_from<0x143, 0xc>(-INFINITY, v));   // row_bcast:31 into rows 2 and 3
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ inline float wave_sum(float v) {
    v += dpp_from<0x111, 0xf>(0.f, v);
    v += dpp_from<0x112, 0xf>(0.f, v);
    v += dpp_from<0x114, 0xf>(0.f, v);
    v += dpp_from<0x118, 0xf>(0.f, v);
    v += dpp_from<0x142, 0xa>(0.f, v);
    v += dpp_from<0x143, 0xc>(0.f, v);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
// Scaled logits never exceed this: a +inf logit (or a product that overflows) sits exactly
// there, so that it takes all the probability, shared among equals, instead of producing NaNs.
constexpr float kCeil = 0x1p127f;
// bf16 bits -> logit * c as fp32; a NaN carries no probability
__device__ inline float scaled(uint32_t bits16_hi, float c) {
    const float x = __uint_as_float(bits16_hi);
    return x != x ? -INFINITY : fminf(x * c, kCeil);
}
// A weight relative to its slot's maximum lies in [0, 1] (rounding may leave the largest a hair above); the
// weight of a NaN logit is a NaN and becomes 0 here.  Written so that the compiler folds it into the
// instruction that makes the weight (its result clamp), at no cost.
__device__ inline float unit_clamp(float w) { return fminf(fmaxf(w, 0.f), 1.f); }
// Inclusive prefix sum across the wavefront, by the same lane-crossing paths.
__device__ inline float wave_scan(float v) {
    v += dpp_from<0x111, 0xf>(0.f, v);
    v += dpp_from<0x112, 0xf>(0.f, v);
    v += dpp_from<0x114, 0xf>(0.f, v);
    v += dpp_from<0x118, 0xf>(0.f, v);
    v += dpp_from<0x142, 0xa>(0.f, v);
    v += dpp_from<0x143, 0xc>(0.f, v);
    return v;
}
__device__ inline float lane_value(float v, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); }

// Row layout: `head` tokens in front of the first 16-byte boundary, n_vec groups of 8 tokens,
// a tail of fewer than 8.  Statistics slot 0 is the head, slot 1 + k block k of the aligned
// part, the last slot the tail.
// kSampleThreads: 256, 512 or 1024, see the launch code.  What bounds it: memory for many long rows (2048 rows of
// 128 K tokens 6.2 TB/s, 87.4 -> 84.5 us), else the chain of one row, i.e. launch, one trip for its tokens, the sums, one
// trip for the chosen slot (one row of 32 K tokens 9.2 -> 6.9 us, 512 rows of 128 K tokens 29.2 -> 25.7).
template <int kSampleThreads>
__global__ __launch_bounds__(kSampleThreads) void target_sample_kernel(const uint16_t *__restrict__ logits,
                                                                       const int32_t *__restrict__ parents,
                                                                       const float *__restrict__ uniforms,
                                                                       int32_t *__restrict__ out, int T, int V, float c) {
    constexpr int kSampleWaves = kSampleThreads / 64;
    extern __shared__ float2 s_stat[];        // (maximum, sum) per slot
    __shared__ float s_u;
    const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = row / T, node = row - b * T;
    const uint16_t *src = logits + (size_t)row * V;

    const int head = min(V, (int)(((16 - ((uintptr_t)src & 15)) & 15) >> 1));
    const int n_vec = (V - head) / 8;
    const int n_blocks = (n_vec + 63) / 64, n_groups = (n_blocks + kGroup - 1) / kGroup;
    const int tail_at = head + n_vec * 8, n_slots = n_groups + 2;
    const uint4 *vec = reinterpret_cast<const uint4 *>(src + head);

    // slots: a wavefront takes the four blocks of a slot at once.  Per token: widen, half a three-way
    // maximum, one fused multiply-add, exp2 (a NaN becomes weight 0 in its result clamp), add;
    // per slot: one maximum and one sum across the wavefront.  Lanes past the end of the row hold
    // -inf bit patterns, so nothing is selected per token.
    const u32x4_t nothing = {0xff80ff80u, 0xff80ff80u, 0xff80ff80u, 0xff80ff80u};
    auto fetch = [&](int grp, u32x4_t (&w)[kGroup]) {
#pragma unroll
        for (int j = 0; j < kGroup; ++j) {
            const int g = (grp * kGroup + j) * 64 + lane;
            w[j] = grp < n_groups && g < n_vec ? __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(vec + g)) : nothing;
        }
    };
    u32x4_t w[kGroup], next[kGroup];
    fetch(wave, w);

    // The last wavefront, its first loads on their way, finds the depth of the node and with it the row's uniform (a
    // parent pointer that does not lead towards the root ends the walk: the tree checks belong to
    // reader_validate_tree / the attention kernel).  The pointers sit in its lanes.
    if (wave == kSampleWaves - 1) {
        const int32_t *par = parents + (size_t)b * T;
        const int p0 = lane < T ? par[lane] : -1, p1 = lane + 64 < T ? par[lane + 64] : -1;
        int n = node, d = 0;
        while (n > 0 && d < T) {
            const int pn = n < 64 ? __builtin_amdgcn_readlane(p0, n) : __builtin_amdgcn_readlane(p1, n - 64);
            if (pn < 0 || pn >= n) break;
            n = pn;
            ++d;
        }
        const float u = uniforms[(size_t)b * T + d];
        if (lane == 0) s_u = u < 0.f ? 0.f : u;
    }
    // head and tail: at most 7 tokens each, wavefront 0 and 1
    if (wave < 2) {
        const int at = wave == 0 ? 0 : tail_at, cnt = wave == 0 ? head : V - tail_at;
        float2 st = make_float2(-INFINITY, 0.f);
        if (cnt > 0) {
            const float y = lane < cnt ? scaled((uint32_t)src[at + lane] << 16, c) : -INFINITY;
            st.x = wave_max(y);
            st.y = wave_sum(st.x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(y - st.x));
        }
        if (lane == 0) s_stat[wave == 0 ? 0 : n_slots - 1] = st;
    }
    for (int grp = wave; grp < n_groups; grp += kSampleWaves) {
        fetch(grp + kSampleWaves, next);
        float x[8 * kGroup];
#pragma unroll
        for (int j = 0; j < kGroup; ++j) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[8 * j + 2 * e] = __uint_as_float(w[j][e] << 16);
                x[8 * j + 2 * e + 1] = __uint_as_float(w[j][e] & 0xffff0000u);
            }
        }
        // (the maximum of a NaN and a number is the number: a NaN never becomes the maximum unless all are)
        float m = fmaxf(x[0], -INFINITY);
#pragma unroll
        for (int e = 1; e < 8 * kGroup; e += 2) m = fmaxf(fmaxf(m, x[e]), e + 1 < 8 * kGroup ? x[e + 1] : -INFINITY);
        m = wave_max(m);
        float s0 = 0.f, s1 = 0.f, m_store;
        if (m * c < kCeil) {                              // (wavefront-uniform)
            const float mc = fmaxf(m, -0x1p126f) * c;     // a slot of nothing but -inf: every weight becomes exp2(-inf) = 0
#pragma unroll
            for (int e = 0; e < 8 * kGroup; e += 2) {
                s0 += unit_clamp(__builtin_amdgcn_exp2f(__builtin_fmaf(x[e], c, -mc)));
                s1 += unit_clamp(__builtin_amdgcn_exp2f(__builtin_fmaf(x[e + 1], c, -mc)));
            }
            m_store = m * c;
        } else {
            // a +inf logit, or one so large that scaling overflows: go through the clamped values
#pragma unroll
            for (int e = 0; e < 8 * kGroup; e += 2) {
                s0 += __builtin_amdgcn_exp2f(fminf(fmaxf(x[e], -INFINITY) * c, kCeil) - kCeil);
                s1 += __builtin_amdgcn_exp2f(fminf(fmaxf(x[e + 1], -INFINITY) * c, kCeil) - kCeil);
            }
            m_store = kCeil;                              // some token of the slot sits at the ceiling
        }
        const float s = wave_sum(s0 + s1);
        if (lane == 0) s_stat[1 + grp] = make_float2(m_store, s);
#pragma unroll
        for (int j = 0; j < kGroup; ++j) w[j] = next[j];
    }
    __syncthreads();
    if (wave != 0) return;

    // ---- the end of the row, wavefront 0: lane t owns the slots [t * per, (t + 1) * per)
    const int per = (n_slots + 63) / 64, first_slot = lane * per, end_slot = min(n_slots, first_slot + per);
    float m_row = -INFINITY;
    for (int i = first_slot; i < end_slot; ++i) m_row = fmaxf(m_row, s_stat[i].x);
    m_row = wave_max(m_row);
    // (m_row = -inf: no token has any probability, every weight below is 0 and no slot is chosen)
    float mine = 0.f;
    for (int i = first_slot; i < end_slot; ++i) {
        const float2 st = s_stat[i];
        const float wgt = st.x == -INFINITY ? 0.f : st.y * __builtin_amdgcn_exp2f(st.x - m_row);
        s_stat[i].y = wgt;              // the slot's weight relative to the row maximum (read again by this lane only)
        mine += wgt;
    }
    const float incl = wave_scan(mine), total = lane_value(incl, 63);
    // u * total, kept below the total so that some slot crosses it
    const float thr = fminf(s_u * total, total * (1.f - 0x1p-23f));
    // The slot that crosses the threshold: the first whose cumulative weight exceeds it.  Each
    // lane looks at its own slots; rounding of the per-lane sums may let no lane (or two)
    // see the crossing, so the lowest claimed slot wins, and the last slot with weight that
    // starts at or below the threshold stands in when nobody claims.
    int claim = -1, stand_in = -1;
    float claim_front = 0.f, stand_in_front = 0.f;      // weight in front of them
    {
        float cum = incl - mine;
        for (int i = first_slot; i < end_slot; ++i) {
            const float wgt = s_stat[i].y;
            if (wgt > 0.f && cum <= thr) {
                stand_in = i;
                stand_in_front = cum;
                if (claim < 0 && thr < cum + wgt) { claim = i; claim_front = cum; }
            }
            cum += wgt;
        }
    }
    const unsigned long long claims = __ballot(claim >= 0), others = __ballot(stand_in >= 0);
    int slot = -1;
    float front = 0.f;
    if (claims != 0ull) {
        const int l = __ffsll((long long)claims) - 1;
        slot = __builtin_amdgcn_readlane(claim, l);
        front = lane_value(claim_front, l);
    } else if (others != 0ull) {
        const int l = 63 - __clzll((long long)others);
        slot = __builtin_amdgcn_readlane(stand_in, l);
        front = lane_value(stand_in_front, l);
    }
    if (slot < 0) {                     // no weight anywhere, or weights that are not numbers
        if (lane == 0) out[row] = 0;
        return;
    }

    // Inside the slot: its tokens are read again (all of them asked for together) and their weights scanned in index
    // order, block by block (a lane's 8 tokens are consecutive, the lanes of a block follow each other; the four
    // blocks' scans do not wait for each other, only the sums in front of them add up).
    int pick = 0x7fffffff, last_pos = -1;
    if (slot == 0 || slot == n_slots - 1) {             // head or tail: up to 7 tokens, one per lane
        const int at = slot == 0 ? 0 : tail_at, cnt = slot == 0 ? head : V - tail_at;
        const float y = lane < cnt ? scaled((uint32_t)src[at + lane] << 16, c) : -INFINITY;
        const float wgt = y == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(y - m_row);
        const float cum = front + (wave_scan(wgt) - wgt);
        if (wgt > 0.f) {
            if (thr < cum + wgt) pick = at + lane;
            last_pos = at + lane;
        }
    } else {
        u32x4_t again[kGroup];
#pragma unroll
        for (int j = 0; j < kGroup; ++j) {
            const int g = ((slot - 1) * kGroup + j) * 64 + lane;
            again[j] = g < n_vec ? *reinterpret_cast<const u32x4_t *>(vec + g) : nothing;
        }
        float wgt[kGroup][8], lane_sum[kGroup], incl_l[kGroup];
#pragma unroll
        for (int j = 0; j < kGroup; ++j) {
            lane_sum[j] = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float y = scaled(e & 1 ? again[j][e >> 1] & 0xffff0000u : again[j][e >> 1] << 16, c);
                wgt[j][e] = y == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(y - m_row);
                lane_sum[j] += wgt[j][e];
            }
            incl_l[j] = wave_scan(lane_sum[j]);
        }
        float carry = front;
#pragma unroll
        for (int j = 0; j < kGroup; ++j) {
            const int first = head + (((slot - 1) * kGroup + j) * 64 + lane) * 8;
            float cum = carry + (incl_l[j] - lane_sum[j]);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (wgt[j][e] > 0.f) {
                    if (pick == 0x7fffffff && thr < cum + wgt[j][e]) pick = first + e;
                    last_pos = first + e;
                }
                cum += wgt[j][e];
            }
            carry += lane_value(incl_l[j], 63);
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        pick = min(pick, __shfl_xor(pick, off));
        last_pos = max(last_pos, __shfl_xor(last_pos, off));
    }
    // the slot's own sum, added up in another order, may stop just short of the threshold
    if (lane == 0) out[row] = pick != 0x7fffffff ? pick : (last_pos >= 0 ? last_pos : 0);
}

}  // namespace

hipError_t launch_target_sample(const uint16_t *logits, const int32_t *parents, const float *uniforms, int32_t *out,
                                int B, int T, int V, float temperature, hipStream_t stream) {
    // one (maximum, sum) slot per kGroup blocks of 512 tokens, plus the unaligned head and tail of the row
    // (the kernel computes the same number from the row's alignment; this is its upper bound)
    const int n_slots = ((V / 8 + 63) / 64 + kGroup - 1) / kGroup + 2;
    const float c = 1.44269504088896340736f / temperature;
    // Wavefronts per row: 16 while every row can have a compute unit of its own (60 rows of 128 K tokens: 13.6 us, 14.8
    // with eight, 18.3 with four), eight beyond (1600 rows of 16 K: 15.6 us; 22.4 with sixteen, 17.3 with four), four
    // where many rows have no more than four slots each (4096 rows of 8 K: 19.9 us, 22.8 with eight).
    const long long rows = (long long)B * T;
    const int nt = rows <= kNumCU ? 1024 : rows > 4 * kNumCU && n_slots <= 6 ? 256 : 512;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(B * T), dim3(nt), (size_t)n_slots * sizeof(float2), stream, logits, parents, uniforms, out, T, V, c);
    };
    if (nt == 1024) launch(target_sample_kernel<1024>);
    else if (nt == 512) launch(target_sample_kernel<512>);
    else launch(target_sample_kernel<256>);
    return note_hip_error("launch target_sample_kernel", hipGetLastError());
}

}  // namespace reader
