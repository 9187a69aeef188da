// k_accept.hip -- speculative-decoding acceptance: target probabilities of the draft tokens, leading run.
//
// After a miss or a rejected lookahead the k draft tokens of the draft model
// g are verified by the target model f in one forward pass (Section 4.3,
// speculative decoding): token t_j is accepted when P_f(t_j) >= P_g(t_j),
// starting from the first token, and f takes over at the first failure.
// P_f(t_j) is the softmax probability of t_j under f's logits at position j,
// so each (query, position) row of V logits is read once: a workgroup keeps a
// running (maximum, sum of exponentials relative to it) per thread over
// 16-byte chunks of the row, merges the pairs across the workgroup, and
// divides the token's exponential by the sum.  The kernel is bound by reading
// the logits, which it reads once, with non-temporal loads.  A second kernel finds, per query, the first rejected position
// with a wave ballot.
#include "common.hpp"
#include "launch.hpp"

namespace lacache {

namespace {

constexpr int kUnroll = 4;  // 16-byte chunks in flight per thread

// merge two (max, sum of exp(x - max)) pairs; -inf maxima carry an empty sum
__device__ inline void lse_merge(float& m, float& s, float m2, float s2) {
    const float M = fmaxf(m, m2);
    if (M == -__builtin_inff()) return;
    s = (m == -__builtin_inff() ? 0.0f : s * __expf(m - M)) + (m2 == -__builtin_inff() ? 0.0f : s2 * __expf(m2 - M));
    m = M;
}

// fold up to 8 logits into the running pair
__device__ inline void lse_add8(float& m, float& s, const float x[8]) {
    float cm = x[0];
#pragma unroll
    for (int e = 1; e < 8; ++e) cm = fmaxf(cm, x[e]);
    if (cm > m) {
        s = (m == -__builtin_inff()) ? 0.0f : s * __expf(m - cm);
        m = cm;
    }
    if (m == -__builtin_inff()) return;
#pragma unroll
    for (int e = 0; e < 8; ++e) s += __expf(x[e] - m);
}

// 8 logits from 16-byte aligned memory, by non-temporal loads (each logit is read once)
__device__ inline void load_chunk(const char* p, int dtype, float x[8]) {
    if (dtype == 0) {
        const u32x4 a = __builtin_nontemporal_load((const u32x4*)p), b = __builtin_nontemporal_load((const u32x4*)p + 1);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            x[t] = __uint_as_float(a[t]);
            x[4 + t] = __uint_as_float(b[t]);
        }
    } else {
        const u32x4 a = __builtin_nontemporal_load((const u32x4*)p);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            x[2 * t] = __uint_as_float(a[t] << 16);
            x[2 * t + 1] = __uint_as_float(a[t] & 0xFFFF0000u);
        }
    }
}

__device__ inline float load_one(const char* row, int dtype, int v) {
    return dtype == 0 ? ((const float*)row)[v] : bf16_to_f32(((const uint16_t*)row)[v]);
}

}  // namespace

// One workgroup per (query, position) row, grid-stride over the rows.  A row that does not start on a 16-byte
// boundary (a vocabulary that is no multiple of 8) has its first elements taken one by one up to the next: 5120
// rows of 128,257 bfloat16 logits take 211 us, as those of 128,256 do (205 us), and took 875 us one by one.
// Workgroups of 256 threads where the rows fill the chip (5120 rows: 205 us, 222 us with 1024) or are short, of 1024
// where a row's own chain of loads is the bound (accept_many_waves): 1 to 20 rows of 128,256 logits 14 us against
// 22 to 26 us a call, 256 rows 21 against 38 us, 1024 rows 50 against 59 us.
template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_token_prob(const void* __restrict__ logits, int dtype, int V,
                                                         const int32_t* __restrict__ tokens, int64_t rows,
                                                         float* __restrict__ p_target) {
    __shared__ float sm[kThreads / 64], ss[kThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const size_t esz = dtype == 0 ? 4 : 2;
    for (int64_t row = blockIdx.x; row < rows; row += gridDim.x) {
        const char* r = (const char*)logits + row * (int64_t)V * esz;
        float m = -__builtin_inff(), s = 0.0f;
        // elements before the first whole chunk (all of them if no element starts on the boundary)
        int head = (uintptr_t)r % esz == 0 ? (int)(((0 - (uintptr_t)r) & 15) / esz) : V;
        if (head > V) head = V;
        const char* rc = r + head * esz;
        const int nchunks = (V - head) / 8;
        int c = tid;
        for (; c + (kUnroll - 1) * kThreads < nchunks; c += kUnroll * kThreads) {
            float x[kUnroll][8];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) load_chunk(rc + (size_t)(c + u * kThreads) * 8 * esz, dtype, x[u]);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) lse_add8(m, s, x[u]);
        }
        for (; c < nchunks; c += kThreads) {
            float x[8];
            load_chunk(rc + (size_t)c * 8 * esz, dtype, x);
            lse_add8(m, s, x);
        }
        // the elements before and after the chunks, one by one
        const int rest = V - nchunks * 8;
        for (int v = tid; v < rest; v += kThreads) {
            float x[8];
            x[0] = load_one(r, dtype, v < head ? v : nchunks * 8 + v);
#pragma unroll
            for (int e = 1; e < 8; ++e) x[e] = -__builtin_inff();
            lse_add8(m, s, x);
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            const float m2 = __shfl_xor(m, o, kWave), s2 = __shfl_xor(s, o, kWave);
            lse_merge(m, s, m2, s2);
        }
        if (lane == 0) {
            sm[wid] = m;
            ss[wid] = s;
        }
        __syncthreads();
        if constexpr (kThreads > 256) {
            // Sixteen pairs one after another would scale the first ones fifteen times, and each scaling rounds: the
            // sums of 12,000 to 50,000 logits were 2 to 29 % further from 64 bits than with four waves (root mean square
            // of the relative error 7.9e-8 and 6.3e-8 at 12,000).  Here each is scaled once: 5.2e-8, and 1 us less.
            if (wid == 0) {
                const float mw = lane < kThreads / 64 ? sm[lane] : -__builtin_inff();
                const float sw = lane < kThreads / 64 ? ss[lane] : 0.0f;
                m = wave_reduce(mw, [](float a, float b) { return fmaxf(a, b); });
                s = wave_sum_f32(mw == -__builtin_inff() ? 0.0f : sw * __expf(mw - m));
            }
        } else if (tid == 0) {
            for (int w = 1; w < kThreads / 64; ++w) lse_merge(m, s, sm[w], ss[w]);
        }
        if (tid == 0) {
            const int t = tokens[row];
            float p = 0.0f;
            if (t >= 0 && t < V) p = __expf(load_one(r, dtype, t) - m) / s;
            p_target[row] = p;
        }
        __syncthreads();  // sm / ss are rewritten by the next row
    }
}

// One wave per query: the accepted length is the first position whose target probability is below the
// draft's (k if none).
__global__ __launch_bounds__(256) void k_accept_len(const float* __restrict__ p_target,
                                                    const float* __restrict__ p_draft, int B, int k,
                                                    int32_t* __restrict__ accept_len) {
    const int lane = threadIdx.x & 63;
    for (int64_t b = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); b < B; b += (int64_t)gridDim.x * 4) {
        int len = k;
        for (int j0 = 0; j0 < k; j0 += 64) {
            const int j = j0 + lane;
            const bool reject = j < k && !(p_target[b * k + j] >= p_draft[b * k + j]);
            const uint64_t rej = __ballot(reject);
            if (rej != 0ull) {
                len = j0 + __ffsll((unsigned long long)rej) - 1;
                break;
            }
        }
        if (lane == 0) accept_len[b] = len;
    }
}

hipError_t launch_accept_length(const void* logits, int dtype, int V, const int32_t* tokens, const float* p_draft,
                                int B, int k, int32_t* accept_len, float* p_target, hipStream_t s) {
    const int64_t rows = (int64_t)B * k;
    if (rows <= 0) return hipSuccess;
    if (accept_many_waves(rows, V, dtype))
        k_token_prob<1024><<<dim3((unsigned)rows), dim3(1024), 0, s>>>(logits, dtype, V, tokens, rows, p_target);
    else
        k_token_prob<256><<<dim3((unsigned)grid_blocks(rows)), dim3(256), 0, s>>>(logits, dtype, V, tokens, rows,
                                                                                 p_target);
    k_accept_len<<<dim3((unsigned)grid_blocks(((int64_t)B + 3) / 4)), dim3(256), 0, s>>>(p_target, p_draft, B, k,
                                                                                         accept_len);
    return hipGetLastError();
}

}  // namespace lacache
