// k_calibrate.hip -- threshold calibration from benign pairs: pair cosines, then an exact percentile.
//
// Appendix A.2 sets each threshold to a percentile of the cosine similarities
// of benign pairs, capped from above (tau_c = min(0.80, P5) over paraphrase
// query pairs, tau_a = min(0.70, P10) over their response prefixes).  The pair
// cosine is the one the lookup computes: both vectors normalised in double and
// rounded once to bfloat16 (the same routine as every stored vector), their
// products accumulated in float32, clamped to [-1, 1].  The percentile is
// linear between the closest ranks, h = (n - 1) p / 100 (the paper does not
// say; this is numpy's default), from the two order statistics floor(h) and
// floor(h) + 1, which an exact radix select finds without sorting: three
// histogram passes over the orderable 32-bit keys of the similarities (11,
// 11 and 10 bits), each ended by a scan, in the workgroup that finishes last,
// that fixes those bits of both ranks' keys (1M similarities: 12 + 9 + 9 us).
#include <mutex>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"

namespace lacache {

namespace {

constexpr int kBins = 2048;  // histogram bins of the widest pass (11 bits)
constexpr int kPasses = 3;
__constant__ const int kShift[kPasses] = {21, 10, 0};
__constant__ const int kBits[kPasses] = {11, 11, 10};

}  // namespace

// One wave per pair: normalise a[j] and b[j] as stored vectors are, and dot the rounded values in column order per
// lane, then across the wave (products of two bfloat16 values are exact in float32).  NC > 0: d <= 512 NC and each
// lane keeps its 8 NC columns of both rows in registers, read once; the norms are summed in the order row_norm
// uses, so the rounded values are those of the stored vectors.  Square root and reciprocal, 60 double-precision
// operations that every lane needs of both norms, run once for the two (one norm in each half of the wave).
// CHUNKED: both arrays have rows of whole aligned 16-byte chunks (row_is_chunked), loaded and rounded without branches;
// else the rows are loaded chunk by chunk in turn and every element takes its own test for the division, in fewer
// registers than rounding whole rows needs (100k pairs of 900 bfloat16 columns 218 us, 244 us in one kernel with the
// chunked rows; of 1500 427 and 530 us).
// NC = 0: any d, the rows read once for the norms and once for the dot.
template <int NC, bool CHUNKED>
__device__ __forceinline__ void pair_cosine(const void* __restrict__ a, const void* __restrict__ b, int dtype, int d,
                                            int64_t j, float* __restrict__ sims) {
    const int lane = threadIdx.x & 63;
    const size_t esz = dtype == 0 ? 4 : 2;
    const char* ra = (const char*)a + j * d * esz;
    const char* rb = (const char*)b + j * d * esz;
    float acc = 0.0f;
    if constexpr (NC > 0) {
        float xa[NC][8], xb[NC][8];
        if constexpr (CHUNKED) {
            RawRow<NC> wa, wb;
            // Non-temporally, as each row is read once; but not float32 rows of more than one chunk per lane: a lane's two
            // pieces of a chunk are loaded one after the other, so every line is asked for twice (100k pairs of 2048
            // float32 columns 370 us, 300 us with plain loads, of 1024 174 and 168 us; of 2048 bfloat16 ones 167 and
            // 173 us).
            if (NC == 1 || dtype != 0) {
                int ln = lane;
                if constexpr (NC > 1) __asm__ volatile("" : "+v"(ln));  // else both branches' loads become plain ones
                row_load<NC, true>(ra, dtype, d, true, ln, wa);
                row_load<NC, true>(rb, dtype, d, true, ln, wb);
            } else {
                row_load<NC>(ra, dtype, d, true, lane, wa);
                row_load<NC>(rb, dtype, d, true, lane, wb);
            }
            row_unpack_chunks<NC>(dtype, d, lane, wa, xa);
            row_unpack_chunks<NC>(dtype, d, lane, wb, xb);
        } else {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                load8f(ra, dtype, d, lane * 8 + 512 * c, xa[c]);
                load8f(rb, dtype, d, lane * 8 + 512 * c, xb[c]);
            }
        }
        double sa = 0.0, sb = 0.0;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                sa += (double)xa[c][e] * (double)xa[c][e];
                sb += (double)xb[c][e] * (double)xb[c][e];
            }
        sa = wave_sum_f64(sa), sb = wave_sum_f64(sb);
        if constexpr (CHUNKED) {
            const double n = __builtin_sqrt(lane < 32 ? sa : sb);
            const float rnf = quotient_rcp_f32(n);
            const double na = __shfl(n, 0, kWave), nb = __shfl(n, 32, kWave);
            const float rna = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(rnf), 0));
            const float rnb = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(rnf), 32));
            if (__ballot(n == 0.0) == 0ull) {  // a zero vector normalises to zero and scores 0
                uint32_t pa[NC * 4], pb[NC * 4];
                quantise_row<NC>(xa, na, rna, d, lane, pa);
                quantise_row<NC>(xb, nb, rnb, d, lane, pb);
#pragma unroll
                for (int k = 0; k < NC * 4; ++k) {
                    acc += __uint_as_float(pa[k] << 16) * __uint_as_float(pb[k] << 16);
                    acc += __uint_as_float(pa[k] & 0xFFFF0000u) * __uint_as_float(pb[k] & 0xFFFF0000u);
                }
            }
        } else if (sa != 0.0 && sb != 0.0) {
            const double na = __builtin_sqrt(sa), nb = __builtin_sqrt(sb);
            const float rna = quotient_rcp_f32(na), rnb = quotient_rcp_f32(nb);
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if (lane * 8 + 512 * c + e >= d) continue;
                    acc += bf16_rne_quotient_f32(xa[c][e], na, rna) * bf16_rne_quotient_f32(xb[c][e], nb, rnb);
                }
        }
    } else {
        const double na = row_norm(ra, dtype, d, true, lane);
        const double nb = row_norm(rb, dtype, d, true, lane);
        if (na != 0.0 && nb != 0.0) {
            const float rna = quotient_rcp_f32(na), rnb = quotient_rcp_f32(nb);
            for (int j0 = lane * 8; j0 < d; j0 += 512) {
                float va[8], vb[8];
                load8f(ra, dtype, d, j0, va);
                load8f(rb, dtype, d, j0, vb);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if (j0 + e >= d) continue;
                    acc += bf16_rne_quotient_f32(va[e], na, rna) * bf16_rne_quotient_f32(vb[e], nb, rnb);
                }
            }
        }
    }
    acc = wave_sum_f32(acc);
    if (lane == 0) sims[j] = fminf(fmaxf(acc, -1.0f), 1.0f);
}

// state[0..1]: the key bits found so far for rank 0 / rank 1; state[2..3]: the ranks still to skip inside the
// current prefix; state[4]: workgroups that have added their histogram.  hist: [2][kBins] counts.
__device__ inline void select_init(uint32_t* state, uint32_t* hist, uint32_t r0, uint32_t r1) {
    for (int i = threadIdx.x; i < 2 * kBins; i += blockDim.x) hist[i] = 0u;
    if (threadIdx.x < 5) state[threadIdx.x] = threadIdx.x == 2 ? r0 : threadIdx.x == 3 ? r1 : 0u;
}

// The pair cosines; the first workgroup also sets up the selection that follows on the stream.
// LOOP: grid-stride over the pairs, for more pairs than one grid holds; else one pair per wave (the loop's
// carried state costs registers, and with them occupancy).
// Bound by the vector ALU beside HBM.  1M pairs of 1024 bfloat16 columns: 710 us (5.8 TB/s), 945 us with the rounding
// test and its division branch at every element, both norms in every lane and loads that waited for each other.
template <int NC, bool LOOP, bool CHUNKED>
__global__ __launch_bounds__(256) void k_pair_cosine(const void* __restrict__ a, const void* __restrict__ b,
                                                     int dtype, int d, int64_t n, float* __restrict__ sims,
                                                     uint32_t* __restrict__ state, uint32_t* __restrict__ hist,
                                                     uint32_t r0, uint32_t r1) {
    if (blockIdx.x == 0) select_init(state, hist, r0, r1);
    const int64_t j0 = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (LOOP) {
        for (int64_t j = j0; j < n; j += (int64_t)gridDim.x * 4) pair_cosine<NC, CHUNKED>(a, b, dtype, d, j, sims);
    } else {
        if (j0 >= n) return;
        pair_cosine<NC, CHUNKED>(a, b, dtype, d, j0, sims);
    }
}

// Adds 1 to h[bin] for the lanes with `on`.  Similarities crowd into few bins (cosines of 0.5 .. 1 share all but the
// last two bits of the first pass), so the lanes that agree with the first one are counted by one addition.
__device__ inline void hist_add(uint32_t* h, uint32_t bin, bool on) {
    const uint64_t m = __ballot(on);
    if (m == 0ull) return;
    const uint32_t lead = (uint32_t)__builtin_amdgcn_readlane((int)bin, __ffsll((unsigned long long)m) - 1);
    const uint64_t same = __ballot(on && bin == lead);
    if ((threadIdx.x & 63) == 0) atomicAdd(&h[lead], (uint32_t)__popcll(same));
    if (on && bin != lead) atomicAdd(&h[bin], 1u);
}

// Histogram (in LDS) of bits [shift, shift + bits) of the keys whose higher bits equal each rank's prefix p0, p1;
// only the first one while the prefixes are equal.  Elements first, first + step, ... of sims.
__device__ inline void select_count(const float* __restrict__ sims, int64_t n, int64_t first, int64_t step, int pass,
                                    uint32_t p0, uint32_t p1, uint32_t* h) {
    const int shift = kShift[pass], hi = shift + kBits[pass];  // bits above hi are fixed by the earlier passes
    const uint32_t mask = (uint32_t)((1u << kBits[pass]) - 1u);
    const bool two = p0 != p1;
    constexpr int kAhead = 8;  // similarities on their way at once
    for (int64_t i0 = first; i0 - (int)(threadIdx.x & 63) < n; i0 += kAhead * step) {  // whole waves
        float v[kAhead];
#pragma unroll
        for (int t = 0; t < kAhead; ++t) v[t] = i0 + t * step < n ? sims[i0 + t * step] : 0.0f;
#pragma unroll
        for (int t = 0; t < kAhead; ++t) {
            const bool in = i0 + t * step < n;
            const uint32_t key = order_f32(v[t]);
            const uint32_t bin = (key >> shift) & mask;
            hist_add(h, bin, in && (hi >= 32 || (key >> hi) == (p0 >> hi)));
            if (two) hist_add(h + kBins, bin, in && (key >> hi) == (p1 >> hi));
        }
    }
}

constexpr int kSelectThreads = 1024;

// One workgroup of T threads: for each rank, the bin holding it (counts read through count(i), scanned in bin
// order) fixes this pass's bits of its key; the counts of the bins before it are skipped.  Each thread takes
// kBins / T consecutive bins, a block-wide exclusive scan gives the count before them, and the one thread whose
// bins hold the rank walks them.  `state` may be LDS or global memory.
template <int T, class Count>
__device__ inline void select_scan(int pass, uint32_t* state, bool two, Count count, uint32_t (&wsum)[2][T / 64]) {
    constexpr int kPer = kBins / T;  // bins per thread in the widest pass
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int shift = kShift[pass], per = (1 << kBits[pass]) / T;
    const uint32_t rank[2] = {state[2], state[3]};
    uint32_t cnt[2][kPer], tot[2] = {0u, 0u};
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            cnt[k][i] = i < per ? count((two ? k * kBins : 0) + tid * per + i) : 0u;
            tot[k] += cnt[k][i];
        }
    uint32_t incl[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        incl[k] = tot[k];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t t = __shfl_up(incl[k], o, kWave);
            if (lane >= o) incl[k] += t;
        }
        if (lane == 63) wsum[k][wid] = incl[k];
    }
    __syncthreads();  // every thread has read the ranks before any is rewritten
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        uint32_t run = incl[k] - tot[k];
        for (int w = 0; w < wid; ++w) run += wsum[k][w];
        if (run <= rank[k] && rank[k] < run + tot[k]) {
            bool found = false;
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                if (found || i >= per) continue;
                if (rank[k] < run + cnt[k][i]) {
                    state[k] |= (uint32_t)(tid * per + i) << shift;
                    state[2 + k] = rank[k] - run;
                    found = true;
                } else {
                    run += cnt[k][i];
                }
            }
        }
    }
    __syncthreads();
}

// P = x_lo + (h - lo) (x_hi - x_lo) in double from the two order statistics; out[0] = P, out[1] = min(cap, P).
__device__ inline void select_result(const uint32_t* state, double frac, float cap, float* __restrict__ out) {
    const double lo = (double)unorder_f32(state[0]);
    const double hi = (double)unorder_f32(state[1]);
    const double P = lo + frac * (hi - lo);
    out[0] = (float)P;
    out[1] = (float)fmin((double)cap, P);
}

// One pass of the selection over many similarities: every workgroup adds its histogram to the global one, and the
// last one to do so (no workgroup waits for another) scans it, clears it for the next pass and, in the last pass,
// writes the result.
__global__ __launch_bounds__(kSelectThreads) void k_select_pass(const float* __restrict__ sims, int64_t n, int pass,
                                                     uint32_t* __restrict__ state, uint32_t* __restrict__ hist,
                                                     double frac, float cap, float* __restrict__ out) {
    __shared__ uint32_t h[2 * kBins];
    __shared__ uint32_t wsum[2][kSelectThreads / 64];
    __shared__ bool last;
    const int tid = threadIdx.x;
    const uint32_t p0 = state[0], p1 = state[1];
    const bool two = p0 != p1;
    const int bins = two ? 2 * kBins : kBins;
    for (int i = tid; i < bins; i += kSelectThreads) h[i] = 0u;
    __syncthreads();
    select_count(sims, n, (int64_t)blockIdx.x * kSelectThreads + tid,
                 (int64_t)gridDim.x * kSelectThreads, pass, p0, p1, h);
    __syncthreads();
    for (int i = tid; i < bins; i += kSelectThreads)
        if (h[i] != 0u) atomicAdd(&hist[i], h[i]);
    last_workgroup_wait();
    __syncthreads();
    if (tid == 0) last = atomicAdd(&state[4], 1u) == gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    select_scan<kSelectThreads>(pass, state, two, [&](int i) {
        return __hip_atomic_load(&hist[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }, wsum);
    for (int i = tid; i < bins; i += kSelectThreads) hist[i] = 0u;
    if (tid == 0) {
        state[4] = 0u;
        if (pass == kPasses - 1) select_result(state, frac, cap, out);
    }
}

// The whole selection over few similarities in one workgroup.
__global__ __launch_bounds__(kSelectThreads) void k_select_few(const float* __restrict__ sims, int64_t n, uint32_t r0,
                                                     uint32_t r1, double frac, float cap, float* __restrict__ out) {
    __shared__ uint32_t h[2 * kBins];
    __shared__ uint32_t state[5];
    __shared__ uint32_t wsum[2][kSelectThreads / 64];
    select_init(state, h, r0, r1);
    __syncthreads();
    for (int pass = 0; pass < kPasses; ++pass) {
        const uint32_t p0 = state[0], p1 = state[1];
        select_count(sims, n, threadIdx.x, kSelectThreads, pass, p0, p1, h);
        __syncthreads();
        select_scan<kSelectThreads>(pass, state, p0 != p1, [&](int i) { return h[i]; }, wsum);
        for (int i = threadIdx.x; i < 2 * kBins; i += kSelectThreads) h[i] = 0u;
        __syncthreads();
    }
    if (threadIdx.x == 0) select_result(state, frac, cap, out);
}

// Scratch of the allocation-free calibration entry point (lacache_calibrate_noalloc): the selection's state
// and histograms, kCalibScratchWords words.  Every GPU the library runs on holds its own copy for the life of
// the process; all such calls on one GPU share it (the pair kernel clears it at the start of each call, so calls
// ordered on one stream are independent; calls that overlap on one GPU race).
static __device__ __align__(256) uint32_t scratch[kCalibScratchWords];

hipError_t calibrate_static_scratch(uint32_t** out) {
    // the array's device address, taken once per device with that device current (the host-side name of the
    // array is no device address); devices past the cache's range look it up on every call
    static std::mutex mu;
    static uint32_t* addr[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    if (dev >= 0 && dev < 64 && addr[dev]) {
        *out = addr[dev];
        return hipSuccess;
    }
    uint32_t* p = nullptr;
    e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64) addr[dev] = p;
    *out = p;
    return hipSuccess;
}

// Similarities up to which one workgroup selects, in one launch instead of three.  Whole call, one workgroup / many,
// us: 14 / 22 for 500 pairs, 18 / 26 for 4096, 34 / 41 for 16384, 56 / 48 for 32768 (nine launches: 31, 45, 52, 64).
constexpr int64_t kSelectFew = 16384;

hipError_t launch_calibrate(const void* a, const void* b, int dtype, int d, int64_t n, float percentile, float cap,
                            float* sims, float* tau, uint32_t* scratch, int num_cu, hipStream_t s) {
    if (n <= 0) return hipErrorInvalidValue;
    const double h = (double)(n - 1) * ((double)percentile / 100.0);
    int64_t lo = (int64_t)h;  // h >= 0: truncation is floor
    if (lo > n - 1) lo = n - 1;
    const int64_t hi = lo + 1 < n ? lo + 1 : lo;
    const double frac = lo == hi ? 0.0 : h - (double)lo;
    uint32_t* state = scratch;
    uint32_t* hist = scratch + 64;
    const dim3 grid((unsigned)grid_blocks((n + 3) / 4)), block(256);
    const bool loop = (n + 3) / 4 > kMaxGridBlocks;
    const bool chunked = row_is_chunked((const char*)a, d) && row_is_chunked((const char*)b, d);
    auto pairs = [&](auto kernel) {
        kernel<<<grid, block, 0, s>>>(a, b, dtype, d, n, sims, state, hist, (uint32_t)lo, (uint32_t)hi);
    };
    auto columns = [&](auto nc) {
        constexpr int NC = decltype(nc)::value;
        if (chunked)
            pairs(loop ? k_pair_cosine<NC, true, true> : k_pair_cosine<NC, false, true>);
        else
            pairs(loop ? k_pair_cosine<NC, true, false> : k_pair_cosine<NC, false, false>);
    };
    if (d <= 512)
        columns(std::integral_constant<int, 1>{});
    else if (d <= 1024)
        columns(std::integral_constant<int, 2>{});
    else if (d <= 2048)
        columns(std::integral_constant<int, 4>{});
    else
        pairs(loop ? k_pair_cosine<0, true, false> : k_pair_cosine<0, false, false>);
    if (n <= kSelectFew) {
        k_select_few<<<dim3(1), dim3(kSelectThreads), 0, s>>>(sims, n, (uint32_t)lo, (uint32_t)hi, frac, cap, tau);
        return hipGetLastError();
    }
    // at least 16 similarities per thread, and few workgroups: each adds its non-zero bins to the global histogram
    // and counts itself, at the same few addresses as the others
    int64_t blocks = (n + kSelectThreads * 16 - 1) / (kSelectThreads * 16);
    if (blocks > num_cu / 2) blocks = num_cu / 2;
    if (blocks < 1) blocks = 1;
    for (int pass = 0; pass < kPasses; ++pass)
        k_select_pass<<<dim3((unsigned)blocks), dim3(kSelectThreads), 0, s>>>(sims, n, pass, state, hist, frac, cap,
                                                                             tau);
    return hipGetLastError();
}

}  // namespace lacache
