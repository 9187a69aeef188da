// common.hpp -- types, store layout and device helpers shared by the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lacache {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kWave = 64;

// ---------------------------------------------------------------------------
// Store layout of the normalised bfloat16 keys ("tiled"):
//   a 16-row x 32-column block of the key matrix is one contiguous 1 KiB
//   "chunk", ordered [c = col/8 % 4][r = row % 16][e = col % 8];
//   chunks are ordered [row/16][col/32].
// Lane l of a wave reading the chunk as 64 x 16 bytes gets row l%16 and
// columns 8*(l/16) .. 8*(l/16)+7 -- exactly the A/B operand fragment of
// v_mfma_f32_16x16x32_bf16 -- so every operand load is one fully coalesced
// 1 KiB wave access, and a run of 16 keys is d_pad*32 contiguous bytes.
// The same layout holds the normalised queries in scratch.
// ---------------------------------------------------------------------------
__host__ __device__ inline int64_t tiled_offset(int64_t row, int32_t col, int32_t kc /* d_pad / 32 */) {
    return ((row >> 4) * kc + (col >> 5)) * 512 + (((col >> 3) & 3) * 16 + (row & 15)) * 8 + (col & 7);
}

// ---------------------------------------------------------------------------
// Rounding of a double to bfloat16, once, to nearest with ties to even.
// Normal range (|v| >= 2^-126): round the 52-bit double significand to 7
// stored bits by adding just under half an ulp plus the kept lsb and
// truncating; a carry moves into the exponent by itself.  Below 2^-126 the
// bfloat16 grid is uniform with spacing 2^-133 (subnormals): round v*2^133 to
// an integer.  Overflow gives infinity.
// ---------------------------------------------------------------------------
__host__ __device__ inline uint64_t f64_bits(double v) {
    uint64_t b;
    __builtin_memcpy(&b, &v, sizeof b);
    return b;
}

__host__ __device__ inline uint16_t bf16_rne_from_f64(double v) {
    const uint64_t b = f64_bits(v);
    const uint16_t sign = (uint16_t)((b >> 48) & 0x8000u);
    const uint64_t mag = b & 0x7FFFFFFFFFFFFFFFull;
    const int e = (int)(mag >> 52) - 1023;
    if (e >= -126) {
        uint64_t m = mag + ((1ull << 44) - 1) + ((mag >> 45) & 1);
        const int e2 = (int)(m >> 52) - 1023;
        if (e2 > 127) return (uint16_t)(sign | 0x7F80u);
        return (uint16_t)(sign | ((uint32_t)(e2 + 127) << 7) | (uint32_t)((m >> 45) & 0x7F));
    }
    const double s = __builtin_rint(__builtin_ldexp(__builtin_fabs(v), 133));
    return (uint16_t)(sign | (uint16_t)s);
}

// bfloat16 rounding of the quotient v / n of a float32 v, identical to bf16_rne_from_f64(v / n) with the
// division correctly rounded (call that double q), computed as f = v * rnf in float32, where rnf is 1 / n
// rounded to double and then to float32 (quotient_rcp_f32).  The roundings of rn, rnf, f and q (at most
// 2^-53, 2^-24, 2^-24 and 2^-53 relative) put f within 2^-23 (1 + 2^-28) |v / n| of q: at most 2 float32 units
// in the last place of f's binade, plus a sliver.  Every bfloat16 rounding midpoint is a float32 with low 16
// bits 0x8000, and the only one closer to f than 2^14 such units is the one inside f's own bfloat16 interval;
// so unless f's low 16 bits are within 2 of 0x8000, no midpoint lies between f and q and both round to the
// same bfloat16.  The fallback window is twice that (within 4).  Those rare cases, zero,
// values below 2^-125 (where the float32 product loses relative precision) and rows whose reciprocal is not
// a normal float32 (rnf = 0, so every product is zero) divide instead.
// The reciprocal for bf16_rne_quotient_fast: 1 / n rounded to double, then to float32, or 0 where that double
// is not a normal float32.
__host__ __device__ inline float quotient_rcp_f32(double n) {
    const double rn = 1.0 / n;
    return (rn >= 0x1p-126 && rn < 0x1p127) ? (float)rn : 0.0f;
}

// The rounding without the division: the result as the float32 of the same value (its low 16 bits zero), and
// whether it may be wrong, when the caller must take bf16_rne_quotient_f32 instead.
__host__ __device__ inline float bf16_rne_quotient_fast(float v, float rnf, bool& exact_needed) {
    const float f = v * rnf;
    uint32_t u;
    __builtin_memcpy(&u, &f, 4);
    exact_needed = (u & 0x7FFFFFFFu) < 0x01000000u || (u & 0xFFFFu) - 0x7FFCu <= 8u;
    u = (u + 0x7FFFu + ((u >> 16) & 1u)) & 0xFFFF0000u;
    float r;
    __builtin_memcpy(&r, &u, 4);
    return r;
}

// The result as the float32 of the same value (its low 16 bits zero); rnf = quotient_rcp_f32(n).
__host__ __device__ inline float bf16_rne_quotient_f32(float v, double n, float rnf) {
    bool exact_needed;
    const float r = bf16_rne_quotient_fast(v, rnf, exact_needed);
    if (!exact_needed) return r;
    float vv = v;
#if defined(__HIP_DEVICE_COMPILE__)
    // convert here, on the rare path, rather than keep a double of every element live across the caller's loop
    __asm__ volatile("" : "+v"(vv));
#endif
    const uint32_t u = (uint32_t)bf16_rne_from_f64((double)vv / n) << 16;
    float e;
    __builtin_memcpy(&e, &u, 4);
    return e;
}
__host__ __device__ inline uint16_t bf16_rne_quotient(float v, double n, float rnf) {
    const float r = bf16_rne_quotient_f32(v, n, rnf);
    uint32_t u;
    __builtin_memcpy(&u, &r, 4);
    return (uint16_t)(u >> 16);
}

// The lane index computed afresh (not kept live across a main loop whose registers are all in use).
__device__ inline int fresh_lane() {
    int r;
    __asm__ volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(r));
    return r;
}

// Workgroup barrier that orders LDS accesses only: loads from memory stay in flight across it.
__device__ inline void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ inline float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Elements j0 .. j0+7 of a row as floats (0 beyond d; bfloat16 widens exactly): one or two 16-byte loads when
// the chunk is whole and 16-byte aligned, element loads otherwise.  The values are the same either way.
__device__ inline void load8f(const void* row, int dtype, int d, int j0, float v[8]) {
    const size_t esz = dtype == 0 ? 4 : 2;
    const char* p = (const char*)row + (size_t)j0 * esz;
    if (j0 + 8 <= d && ((uintptr_t)p & 15) == 0) {
        if (dtype == 0) {
            const float4 x = ((const float4*)p)[0], y = ((const float4*)p)[1];
            v[0] = x.x, v[1] = x.y, v[2] = x.z, v[3] = x.w, v[4] = y.x, v[5] = y.y, v[6] = y.z, v[7] = y.w;
        } else {
            const uint4 x = *(const uint4*)p;
            const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                v[2 * t] = __uint_as_float(w[t] << 16);
                v[2 * t + 1] = __uint_as_float(w[t] & 0xFFFF0000u);
            }
        }
        return;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
        v[e] = (j0 + e < d) ? (dtype == 0 ? ((const float*)row)[j0 + e] : bf16_to_f32(((const uint16_t*)row)[j0 + e]))
                            : 0.0f;
}

// The same elements as doubles.
__device__ inline void load8(const void* row, int dtype, int d, int j0, double v[8]) {
    float f[8];
    load8f(row, dtype, d, j0, f);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (double)f[e];
}

// ---------------------------------------------------------------------------
// Wave-wide butterfly reductions: every lane ends with the same value, and
// the combination order is fixed (lanes 32 apart first, then 16, 8, 4, 2, 1),
// so results are run-to-run identical.  The exchanges run on the vector ALU
// (DPP and the row swaps), not through LDS: a step costs a few cycles
// instead of an LDS round trip, and these chains are most of what the
// kernels of a small call wait for.
// ---------------------------------------------------------------------------
// {a, b} = {x of this lane, x of lane ^ M}, in an order that every half of a wider value shares.
template <int M>
__device__ __forceinline__ void xor_exchange(uint32_t x, uint32_t& a, uint32_t& b) {
    if constexpr (M == 32 || M == 16) {
        const auto r = M == 32 ? __builtin_amdgcn_permlane32_swap(x, x, false, false)
                               : __builtin_amdgcn_permlane16_swap(x, x, false, false);
        a = r[0], b = r[1];
    } else {
        a = x;
        if constexpr (M == 8) b = __builtin_amdgcn_update_dpp(x, x, 0x128, 0xF, 0xF, false);  // row_ror:8
        if constexpr (M == 4) {  // even groups of 4 lanes take from 4 above, odd ones from 4 below
            b = __builtin_amdgcn_update_dpp(x, x, 0x104, 0xF, 0x5, false);
            b = __builtin_amdgcn_update_dpp(b, x, 0x114, 0xF, 0xA, false);
        }
        if constexpr (M == 2) b = __builtin_amdgcn_update_dpp(x, x, 0x4E, 0xF, 0xF, false);  // quad_perm 2,3,0,1
        if constexpr (M == 1) b = __builtin_amdgcn_update_dpp(x, x, 0xB1, 0xF, 0xF, false);  // quad_perm 1,0,3,2
    }
}
template <int M, class T, class Op>
__device__ __forceinline__ T xor_combine(T x, Op op) {
    if constexpr (sizeof(T) == 4) {
        uint32_t a, b;
        xor_exchange<M>(__builtin_bit_cast(uint32_t, x), a, b);
        return op(__builtin_bit_cast(T, a), __builtin_bit_cast(T, b));
    } else {
        const uint64_t u = __builtin_bit_cast(uint64_t, x);
        uint32_t al, bl, ah, bh;
        xor_exchange<M>((uint32_t)u, al, bl);
        xor_exchange<M>((uint32_t)(u >> 32), ah, bh);
        return op(__builtin_bit_cast(T, (uint64_t)ah << 32 | al), __builtin_bit_cast(T, (uint64_t)bh << 32 | bl));
    }
}
template <class T, class Op>
__device__ __forceinline__ T wave_reduce(T x, Op op) {
    x = xor_combine<32>(x, op);
    x = xor_combine<16>(x, op);
    x = xor_combine<8>(x, op);
    x = xor_combine<4>(x, op);
    x = xor_combine<2>(x, op);
    return xor_combine<1>(x, op);
}
__device__ inline double wave_sum_f64(double x) {
    return wave_reduce(x, [](double a, double b) { return a + b; });
}
__device__ inline float wave_sum_f32(float x) {
    return wave_reduce(x, [](float a, float b) { return a + b; });
}
__device__ inline uint64_t umax64(uint64_t a, uint64_t b) { return a > b ? a : b; }
__device__ inline uint64_t wave_max_u64(uint64_t x) { return wave_reduce(x, umax64); }

// ---------------------------------------------------------------------------
// "The last workgroup to finish goes on": every workgroup publishes its part with device-wide atomic
// operations only, calls this, and after a workgroup barrier one thread adds 1 to a counter; the workgroup
// that counts last reads the parts with device-wide atomic loads.  The order rests on gfx950, not on the language's
// memory model, in which relaxed operations order nothing between workgroups: there, device-wide atomic operations take
// effect where all XCDs see them, and s_waitcnt returns when this wave's have, so they come before the counter.  It
// holds only for words that are written and read by device-wide atomics alone.  A device-wide release fence in
// its place writes the XCD's L2 back (25 us per pass of 256 workgroups).  Not for another target without a look at it.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void last_workgroup_wait() {
#if defined(__HIP_DEVICE_COMPILE__) && !defined(__gfx950__)
#error "last_workgroup_wait orders atomics as gfx950 does; use __threadfence() elsewhere"
#endif
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
}

// ---------------------------------------------------------------------------
// One wave L2-normalises one input row and rounds it to bfloat16: the sum of
// squares is taken in double (lane-local in column order, then the butterfly
// above), n = sqrt in double, and each component v / n is rounded once to
// bfloat16.  A zero row (or live == false) gives zeros, as do the columns
// d .. d_pad-1.  Lane l produces columns 8l + 512t .. 8l + 512t + 7 and hands
// them, packed, to emit(j0, u32x4).  Every kernel that quantises a vector
// (insert, query staging, lookahead check, calibration pairs) goes through
// row_norm and quantise8, so equal inputs quantise to identical bits wherever
// they are stored or compared.
// ---------------------------------------------------------------------------
__device__ inline double row_norm(const void* row, int dtype, int d, bool live, int lane) {
    double ss = 0.0;
    if (live) {
        for (int j0 = lane * 8; j0 < d; j0 += 512) {
            double v[8];
            load8(row, dtype, d, j0, v);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (j0 + e < d) ss += v[e] * v[e];
        }
    }
    ss = wave_sum_f64(ss);
    return __builtin_sqrt(ss);
}

// Columns j0 .. j0+7 of the normalised row as packed bfloat16 (zeros beyond d, for a zero norm or dead rows).
__device__ inline u32x4 quantise8(const void* row, int dtype, int d, int j0, double n, bool live) {
    uint16_t h[8];
    float v[8];
    if (live && j0 < d && n != 0.0) load8f(row, dtype, d, j0, v);
    const float rnf = quotient_rcp_f32(n);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int j = j0 + e;
        h[e] = 0;
        if (live && j < d && n != 0.0) h[e] = bf16_rne_quotient(v[e], n, rnf);
    }
    u32x4 w;
    w.x = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
    w.y = (uint32_t)h[2] | ((uint32_t)h[3] << 16);
    w.z = (uint32_t)h[4] | ((uint32_t)h[5] << 16);
    w.w = (uint32_t)h[6] | ((uint32_t)h[7] << 16);
    return w;
}

template <class Emit>
__device__ inline void normalise_row(const void* row, int dtype, int d, int d_pad, bool live, int lane, Emit emit) {
    const double n = row_norm(row, dtype, d, live, lane);
    for (int j0 = lane * 8; j0 < d_pad; j0 += 512) emit(j0, quantise8(row, dtype, d, j0, n, live));
}

// A row held in registers: lane l keeps columns l*8 + 512 c .. +7 for c < NC (zeros beyond d, and for rows that
// are not live), the columns row_norm and quantise8 give lane l.  Loading is split in two so that a caller can
// have several rows on their way before it waits for the first: rows of whole 16-byte chunks are loaded without
// branches (lanes past the row read its first chunk and drop it); others element by element in the second half.
template <int NC>
struct RawRow {
    u32x4 lo[NC], hi[NC];  // 16-byte pieces: lo alone for a chunk of bfloat16, both for one of float32
};
__host__ __device__ __forceinline__ bool row_is_chunked(const char* src, int d) {
    return ((uintptr_t)src & 15) == 0 && d % 8 == 0;
}
template <int NC, bool NT = false>
__device__ __forceinline__ void row_load(const char* src, int dtype, int d, bool live, int lane, RawRow<NC>& r) {
    const bool any = live && row_is_chunked(src, d);
    auto at = [&](int c, int half) {
        const int j0 = lane * 8 + 512 * c;
        const u32x4* p = (const u32x4*)(src + (j0 < d ? (size_t)j0 * (dtype == 0 ? 4 : 2) + 16 * half : 0));
        return NT ? __builtin_nontemporal_load(p) : *p;
    };
#pragma unroll
    for (int c = 0; c < NC; ++c) r.lo[c] = any ? at(c, 0) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int c = 0; c < NC; ++c) r.hi[c] = any && dtype == 0 ? at(c, 1) : u32x4{0u, 0u, 0u, 0u};
}
template <int NC>
__device__ __forceinline__ void row_unpack_chunks(int dtype, int d, int lane, const RawRow<NC>& r, float (&x)[NC][8]) {
    if (dtype == 0) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const bool in = lane * 8 + 512 * c < d;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                x[c][t] = __uint_as_float(in ? r.lo[c][t] : 0u);
                x[c][4 + t] = __uint_as_float(in ? r.hi[c][t] : 0u);
            }
        }
    } else {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const bool in = lane * 8 + 512 * c < d;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const uint32_t u = in ? r.lo[c][t] : 0u;
                x[c][2 * t] = __uint_as_float(u << 16);
                x[c][2 * t + 1] = __uint_as_float(u & 0xFFFF0000u);
            }
        }
    }
}
template <int NC>
__device__ __forceinline__ void row_unpack(const char* src, int dtype, int d, bool live, int lane, const RawRow<NC>& r,
                                           float (&x)[NC][8]) {
    if (live && !row_is_chunked(src, d)) {
        // The lane made opaque here: else the addresses and bounds of these elements are formed before the caller's
        // loop over rows and hold 40 registers through it (the forms for 2048 columns spilled 84 to 176 bytes a lane:
        // inserts of 4096 x 1536 float32 rows 26.6 us, 20.1 us so).
        __asm__ volatile("" : "+v"(lane));
#pragma unroll
        for (int c = 0; c < NC; ++c) load8f(src, dtype, d, lane * 8 + 512 * c, x[c]);
        return;
    }
    row_unpack_chunks<NC>(dtype, d, lane, r, x);
}
template <int NC>
__device__ __forceinline__ void row_to_regs(const char* src, int dtype, int d, bool live, int lane, float (&x)[NC][8]) {
    RawRow<NC> r;
    row_load<NC>(src, dtype, d, live, lane, r);
    row_unpack<NC>(src, dtype, d, live, lane, r, x);
}

// Its norm, the squares summed in the order row_norm uses (the zeros it skips add nothing), so the two agree
// bit for bit.
template <int NC>
__device__ __forceinline__ double regs_norm(const float (&x)[NC][8]) {
    double ss = 0.0;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 8; ++e) ss += (double)x[c][e] * (double)x[c][e];
    return __builtin_sqrt(wave_sum_f64(ss));
}

// The row divided by its norm and rounded to bfloat16, two values to a word, as bf16_rne_quotient rounds each:
// the float32 products are rounded in pairs, and a lane with a product that the proof of bf16_rne_quotient_fast
// does not cover (within 2 units of a rounding midpoint, or below 2^-125) goes through the division for it.
// One element in 13,000 is such a one, 7 % of 1024-column rows hold any, so the test is made once per row and
// the loop over a lane's elements is left out of the common path (with a branch per element, bulk inserts of
// 1024-column prefix rows stored 131,000 of them in 79 us; 65 us so).  Rows with zeros (exact as they are, but below
// 2^-125), and last chunks that d does not fill, always go through that loop's first half: inserts of 20,000 x 1024
// bfloat16 entries 45 us, 52 us where half of the elements are zero (48 and 58 us with a branch per element).  A zero norm
// gives zeros.  The whole wave
// calls it, with one n for all lanes; rnf = quotient_rcp_f32(n).
template <int NC>
__device__ __forceinline__ void quantise_row(const float (&x)[NC][8], double n, float rnf, int d, int lane,
                                             uint32_t (&p)[NC * 4]) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    constexpr uint32_t kTiny = 0x01000000u;  // bits of 2^-125
    if (n == 0.0) {
#pragma unroll
        for (int k = 0; k < NC * 4; ++k) p[k] = 0u;
        return;
    }
    uint16_t window = 0xFFFFu;
    float least = __builtin_inff();
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        float low = __builtin_inff();
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float f0 = x[c][2 * t] * rnf, f1 = x[c][2 * t + 1] * rnf;
            const uint16_t w0 = (uint16_t)(__float_as_uint(f0) - 0x7FFEu);
            const uint16_t w1 = (uint16_t)(__float_as_uint(f1) - 0x7FFEu);
            window = w0 < window ? w0 : window;
            window = w1 < window ? w1 : window;
            low = fminf(fminf(__builtin_fabsf(f0), __builtin_fabsf(f1)), low);
            p[c * 4 + t] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{f0, f1}), bf16x2));
        }
        if (lane * 8 + 512 * c < d) least = fminf(least, low);
    }
    if (__ballot(window <= 4u || least < __uint_as_float(kTiny)) == 0ull) return;
    __asm__ volatile("" : "+v"(rnf));  // form the products again rather than keep them all for this rare path
    uint32_t todo = 0u;  // the lane's elements that need the division (zeros are exact as they are)
#pragma unroll
    for (int i = 0; i < NC * 8; ++i) {
        const float v = x[i >> 3][i & 7];
        const uint32_t u = __float_as_uint(v * rnf);
        if ((u & 0xFFFFu) - 0x7FFEu <= 4u || ((u & 0x7FFFFFFFu) < kTiny && v != 0.0f)) todo |= 1u << i;
    }
    while (__ballot(todo != 0u) != 0ull) {
        const int i = todo != 0u ? __ffs(todo) - 1 : NC * 8;
        float v = 0.0f;
#pragma unroll
        for (int k = 0; k < NC * 8; ++k) v = k == i ? x[k >> 3][k & 7] : v;
        const uint32_t h = bf16_rne_from_f64((double)v / n);
#pragma unroll
        for (int k = 0; k < NC * 4; ++k)
            if (k == i >> 1) p[k] = (i & 1) ? (p[k] & 0xFFFFu) | (h << 16) : (p[k] & 0xFFFF0000u) | h;
        todo &= todo - 1u;
    }
}

// The 8 values of chunk c.
template <int N>
__device__ __forceinline__ u32x4 piece(const uint32_t (&p)[N], int c) {
    return u32x4{p[4 * c], p[4 * c + 1], p[4 * c + 2], p[4 * c + 3]};
}

// Dot product of two packed bfloat16 chunks, accumulated into acc in float32 in column order.  bf16 x bf16
// products are exact in float.
__device__ inline float dot8_bf16(u32x4 a, u32x4 b, float acc) {
    const uint32_t av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        acc += __uint_as_float(av[t] << 16) * __uint_as_float(bv[t] << 16);
        acc += __uint_as_float(av[t] & 0xFFFF0000u) * __uint_as_float(bv[t] & 0xFFFF0000u);
    }
    return acc;
}

// ---------------------------------------------------------------------------
// Top-1 candidates as one 64-bit key: high word = the score's bits mapped so
// that unsigned order equals float order, low word = ~index.  The unsigned
// maximum is then "highest score, lowest index among equal scores": a total
// order, so any merge order gives the same winner.  -0 is folded onto +0
// first so that equal scores compare equal.
// ---------------------------------------------------------------------------
__device__ inline uint32_t order_f32(float f) {
    const uint32_t u = __float_as_uint(f + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float unorder_f32(uint32_t o) {
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o);
}
__device__ inline uint64_t pack_top1(float s, int32_t idx) {
    return ((uint64_t)order_f32(s) << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)idx);
}
__device__ inline int32_t unpack_idx(uint64_t p) { return (int32_t)(0xFFFFFFFFu - (uint32_t)(p & 0xFFFFFFFFu)); }
__device__ inline float unpack_score(uint64_t p) { return unorder_f32((uint32_t)(p >> 32)); }

__device__ inline f32x4 mfma16x16x32(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                   0, 0, 0);
}

}  // namespace lacache
