// The base model's greedy tokens from its logits (Algorithm 5: "compare base logits with
// drafted tokens"): target_tokens[r] = argmax_v logits[r][v] for the B*T rows of one
// verification step.  The logits of a step are as large as its KV stream (vocabulary 128256:
// 256 KB per row), so this is a plain streaming reduction: one workgroup per row, 128-bit
// loads (eight in flight per thread until the row ends; in rounds, each asked for when the one
// before was scanned, 512 rows took 23.1 us and now 22.1, 6.0 TB/s), a running (value, index)
// per thread, then a wavefront and a workgroup reduction.  The workgroup is 512 threads wide, 1024 when there are few rows
// (measured: from 1024 rows on 512 threads are the fastest).
// Ties go to the lowest index; a NaN is never larger than anything (a row of NaNs gives 0).
#include <type_traits>

#include "internal.h"

namespace reader {

namespace {

struct Best {
    float v;
    int i;
};

__device__ inline void take(Best &b, float v, int i) {
    // strictly larger, or equal with a lower index (indices arrive out of order across threads)
    if (v > b.v || (v == b.v && i < b.i)) { b.v = v; b.i = i; }
}

// The same for values that arrive in increasing index order (a thread's own scan): an equal value never wins.
// (Half the vector instructions per logit of `take`; with `take` the kernel was bound by them, not by memory.)
__device__ inline void first_larger(Best &b, float v, int i) {
    if (v > b.v) { b.v = v; b.i = i; }
}

template <int NT>
__global__ __launch_bounds__(NT) void target_argmax_kernel(const uint16_t *__restrict__ logits, int32_t *__restrict__ out,
                                                           int V) {
    const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint16_t *src = logits + (size_t)row * V;
    Best best = {-INFINITY, 0x7fffffff};
    // rows start at any multiple of 2 bytes: up to seven logits in front of the first 16-byte boundary and up to seven
    // behind the last one go to a thread each.  (All threads load, under the index they load from, and the value is
    // looked at last: a load under a condition would be waited for where it ends.)
    const int head = min(V, (int)(((16 - ((uintptr_t)src & 15)) & 15) >> 1));
    const int n_vec = (V - head) / 8;
    const int edge_i = tid < head ? tid : min(tid + n_vec * 8, V - 1);
    const uint4 *vec = reinterpret_cast<const uint4 *>(src + head);
    auto scan = [&](const uint4 &w, int c) {
        const uint32_t u[4] = {w.x, w.y, w.z, w.w};
        const int base = head + c * 8;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            first_larger(best, __uint_as_float(u[e] << 16), base + 2 * e);
            first_larger(best, __uint_as_float(u[e] & 0xffff0000u), base + 2 * e + 1);
        }
    };
    // Read once: streamed past the caches (about a sixth more bandwidth out of HBM than plain loads).  A register's next
    // load is asked for as soon as its group is scanned, so that a thread's loads stay in flight until the row ends; no
    // load stands under a condition (behind one the compiler waits for all of them).  Threads without a group of their
    // own read the row's last one again, under that one's indices, which changes nothing.
    const int rounds = (n_vec + NT - 1) / NT;
    auto stream = [&](auto n_loads) {
        constexpr int N = decltype(n_loads)::value;
        uint4 w[N];
#pragma unroll
        for (int j = 0; j < N; ++j) w[j] = load_stream16(vec + min(tid + j * NT, n_vec - 1));
        const uint32_t edge = src[edge_i];
        int r = 0;
        for (; r + N < rounds; r += N) {
#pragma unroll
            for (int j = 0; j < N; ++j) {
                scan(w[j], min(tid + (r + j) * NT, n_vec - 1));
                w[j] = load_stream16(vec + min(tid + (r + j + N) * NT, n_vec - 1));
                __builtin_amdgcn_sched_barrier(0);   // (the scheduler would gather the loads behind the last scan)
            }
        }
#pragma unroll
        for (int j = 0; j < N; ++j)
            if (r + j < rounds) scan(w[j], min(tid + (r + j) * NT, n_vec - 1));
        take(best, __uint_as_float(edge << 16), edge_i);
    };
    // (rows of up to four rounds would ask eight times for loads that four of them repeat)
    if (rounds > 4) stream(std::integral_constant<int, 8>());
    else if (rounds > 0) stream(std::integral_constant<int, 4>());
    else take(best, __uint_as_float((uint32_t)src[edge_i] << 16), edge_i);

#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const float ov = __shfl_xor(best.v, off);
        const int oi = __shfl_xor(best.i, off);
        take(best, ov, oi);
    }
    __shared__ float s_v[NT / 64];
    __shared__ int s_i[NT / 64];
    if (lane == 0) { s_v[wave] = best.v; s_i[wave] = best.i; }
    __syncthreads();
    if (wave == 0) {
        constexpr int NW = NT / 64;
        Best b = {lane < NW ? s_v[lane] : -INFINITY, lane < NW ? s_i[lane] : 0x7fffffff};
#pragma unroll
        for (int off = NW / 2; off >= 1; off >>= 1) {
            const float ov = __shfl_xor(b.v, off);
            const int oi = __shfl_xor(b.i, off);
            take(b, ov, oi);
        }
        int token = __shfl(b.i, 0);
        if (__shfl(b.v, 0) == -INFINITY) {
            // nothing but -inf and NaN, which no scan has told apart: the first that is not a NaN
            token = 0;
            for (int base = 0; base < V; base += 64) {
                const int i = min(base + lane, V - 1);
                const unsigned long long held = __ballot((src[i] & 0x7fff) <= 0x7f80);
                if (held != 0ull) { token = min(base + (int)__builtin_ctzll(held), V - 1); break; }
            }
        }
        if (lane == 0) out[row] = token;
    }
}

}  // namespace

hipError_t launch_target_argmax(const uint16_t *logits, int32_t *out, int rows, int V, hipStream_t stream) {
    // threads per row so that the rows of the launch fill the chip's 256 x 2048 thread slots
    // (measured: 1024 threads per row are ahead up to 768 rows, 512 beyond)
    if (rows <= 768) hipLaunchKernelGGL((target_argmax_kernel<1024>), dim3(rows), dim3(1024), 0, stream, logits, out, V);
    else hipLaunchKernelGGL((target_argmax_kernel<512>), dim3(rows), dim3(512), 0, stream, logits, out, V);
    return note_hip_error("launch target_argmax_kernel", hipGetLastError());
}

}  // namespace reader
