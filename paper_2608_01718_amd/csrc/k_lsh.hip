// k_lsh.hip -- stage 1 through a locality-sensitive index: random-hyperplane signatures, a Hamming-radius
// candidate scan, and exact re-ranking of the candidates.
//
// Section 3 models the cache key as an LSH h(z) of the embedding with the
// gapped collision property of Eq. (1), and Algorithm 1 searches the cache
// with it.  For cosine distance the hash family is random hyperplanes: bit i
// of h(z) is 1 when r_i . z >= 0, so vectors at angle theta agree on a bit
// with probability 1 - theta / pi.  Signatures of the stored (normalised,
// bfloat16-rounded) keys are kept beside the store; a query's candidates are
// the entries within a Hamming radius of its signature (radius 0 is equality
// of hash keys), found by one pass over the signatures (bits / 8 bytes per
// entry instead of the key's d * 2), and re-ranked by their exact similarity.
#include <type_traits>
#include <utility>

#include "verify.hpp"

namespace lacache {

// ---------------------------------------------------------------------------
// Signature bits on the matrix cores.  The hyperplanes are the row operand of
// v_mfma_f32_16x16x32_bf16 and the vectors the column operand, so lane l ends
// with the projections of vector l % 16 on rows 4 q .. 4 q + 3 (q = l / 16) of
// each 16-hyperplane block.  The hyperplanes are stored in the order that
// makes those bits land where the signature keeps them: with W words (2 W
// blocks), row 4 q + i of block hb is hyperplane 8 W q + 4 hb + i, so over all
// blocks lane q of a vector collects bytes W q .. W q + W - 1 of its 4 W
// signature bytes in order and stores them without any exchange.
// ---------------------------------------------------------------------------

// f(0), f(1), ... with compile-time indices.
template <int... Q, class F>
__device__ __forceinline__ void for_each_index(std::integer_sequence<int, Q...>, F f) {
    (f(std::integral_constant<int, Q>{}), ...);
}

// Hyperplane held by row p of the tiled hyperplane matrix.
__host__ __device__ inline int hyperplane_at(int p, int words) {
    return 8 * words * ((p >> 2) & 3) + 4 * (p >> 4) + (p & 3);
}

// x shifted left by one with the sign bit of f + 0 shifted in (f + 0: a negative zero counts as >= 0).
__device__ inline uint32_t push_sign(uint32_t x, float f) {
    return __builtin_amdgcn_alignbit(x, __float_as_uint(f + 0.0f), 31);
}

// The 4 bits (projection >= 0) of block accumulator `lo` in bits 0..3 and of `hi` in bits 4..7.
__device__ inline uint32_t sign_byte(f32x4 lo, f32x4 hi) {
    uint32_t x = 0u;
#pragma unroll
    for (int i = 3; i >= 0; --i) x = push_sign(x, hi[i]);
#pragma unroll
    for (int i = 3; i >= 0; --i) x = push_sign(x, lo[i]);
    return ~x & 0xFFu;
}

// The [32 words][d] row-major bfloat16 hyperplanes as a tiled matrix of d_pad columns (zero padded), its rows in
// the order above.
__global__ __launch_bounds__(256) void k_tile_hyperplanes(const uint16_t* __restrict__ src, int words, int d,
                                                          int d_pad, uint16_t* __restrict__ dst) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= (int64_t)words * 32 * d_pad) return;
    const int p = (int)(t / d_pad), c = (int)(t - (int64_t)p * d_pad);
    dst[tiled_offset(p, c, d_pad >> 5)] = c < d ? src[(int64_t)hyperplane_at(p, words) * d + c] : (uint16_t)0;
}

// Signatures of many rows (building the index, bulk inserts).  The projection of N rows on 32 W hyperplanes is a
// [N][d] x [d][32 W] product of which only the signs are kept: at 256 bits 512 FLOP per 2 key bytes, about the
// balance of the matrix cores and HBM, so both have to stream.  A workgroup is four waves, one per SIMD (two
// workgroups per CU up to 96 bits); a wave multiplies 64 rows by all HB = 2 W hyperplane blocks, so every row is
// read once, straight from memory into operand registers, SETS - 1 steps of 32 columns ahead (what the launch
// holds in flight is what bounds its bandwidth).  The hyperplanes, which every wave needs, pass through LDS in
// two slots of two steps each; a part's fragments (PARTS = 2: half of the blocks) are read while the part before
// it multiplies, which needs one LDS barrier per two steps: after it the slot just drained is refilled.
// 1M x 768 rows: 345 us at 256 bits (1.14 PFLOP/s, rows at 4.5 TB/s), 263 us at 128, 239 us at 64 (6.4 TB/s).
// One wave per 16 rows with both operands from L2 took 1790 us at 256 bits; 128-row x 128-hyperplane waves that
// read every row twice 386 us.
template <int HB, int PARTS, int SETS>
__global__ __launch_bounds__(256, HB <= 6 ? 2 : 1) void k_simhash_bulk(const u32x4* __restrict__ rows_tiled, int kc,
                                                                       int64_t row0, int64_t n,
                                                                       const u32x4* __restrict__ hp_tiled,
                                                                       int n_tiles, uint8_t* __restrict__ sig) {
    constexpr int kRB = 4;                  // 16-row blocks per wave
    constexpr int kHP = HB / PARTS;         // hyperplane blocks per part of a step
    constexpr int kWaves = 4, kBytes = 2 * HB;  // signature bytes of a row
    constexpr int kTile = kWaves * kRB;     // 16-row groups per workgroup tile
    constexpr int kSteps = 2;               // 32-column steps per LDS slot
    constexpr int kSlot = kSteps * HB;      // 1 KiB chunks per slot
    constexpr int kMine = kSlot / kWaves;   // chunks a wave stages per slot
    static_assert(kSlot % kWaves == 0 && SETS % 4 == 0, "");
    __shared__ u32x4 ring[2 * kSlot * 64];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t0 = (int)((int64_t)blockIdx.x * n_tiles / gridDim.x);
    const int t1 = (int)((int64_t)(blockIdx.x + 1) * n_tiles / gridDim.x);
    const int64_t g0 = row0 >> 4;
    const uint32_t lane16 = (uint32_t)lane * 16;

    // rows: chunk (block kb, step j) of the wave's part of a tile at byte (kb * kc + j) * 1024 from the tile's
    // base.  A tile reads at most 255 rows past the call's last one, fewer than the store's 512 spare rows.  The
    // loads run SETS - 1 steps ahead into the next tile; in the last tile they start over, and are not used.
    const char* kbase = (const char*)(rows_tiled + (g0 + (int64_t)t0 * kTile + wv * kRB) * kc * 64);
    const int tile_bytes = kTile * kc * 1024;
    __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc((void*)kbase, 0, 0x7FFFFFFF, 0x00020000);
    int kstep = 0, koff = 0, wrap = (t0 + 1 < t1 ? tile_bytes : 0) - kc * 1024;
    u32x4 kf[SETS][kRB];
    auto rows_load = [&](u32x4 (&dst)[kRB]) {
#pragma unroll
        for (int kb = 0; kb < kRB; ++kb)  // read once: non-temporal
            dst[kb] = __builtin_amdgcn_raw_buffer_load_b128(krs, lane16, koff + kb * kc * 1024, 2);
        koff += 1024;
        if (++kstep == kc) {
            kstep = 0;
            koff += wrap;
        }
    };

    // hyperplanes: chunk c = s * HB + hb of a slot is block hb at its step s; wave wv stages chunks wv, wv + 4, ...
    const __amdgpu_buffer_rsrc_t hrs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)hp_tiled, 0, 0x7FFFFFFF, 0x00020000);
    u32x4 sr[kMine];
    int ld_step = 0;
    auto slot_load = [&]() {
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            const int c = wv + kWaves * i;
            sr[i] = __builtin_amdgcn_raw_buffer_load_b128(hrs, lane16, ((c % HB) * kc + c / HB + ld_step) * 1024, 0);
        }
        ld_step += kSteps;
        if (ld_step == kc) ld_step = 0;
    };
    auto slot_store = [&](int slot) {
#pragma unroll
        for (int i = 0; i < kMine; ++i) ring[(slot * kSlot + wv + kWaves * i) * 64 + lane] = sr[i];
    };
    u32x4 hf[2][kHP];
    auto frags = [&](int slot, int s, int p, u32x4 (&dst)[kHP]) {
#pragma unroll
        for (int hb = 0; hb < kHP; ++hb) dst[hb] = ring[(slot * kSlot + s * HB + p * kHP + hb) * 64 + lane];
    };
    f32x4 acc[kRB][HB];
#pragma unroll
    for (int p = 0; p < SETS - 1; ++p) rows_load(kf[p]);
    slot_load();
    slot_store(0);
    slot_load();
    slot_store(1);
    slot_load();
    lds_barrier();
    frags(0, 0, 0, hf[0]);

    // one part of a step: load the rows SETS - 1 steps ahead, read the next part's fragments, multiply set u (the
    // row loads spread between the multiplications: bursts of loads stall the wave's issue)
    auto part = [&](auto q_tag, bool zero) {
        constexpr int q = decltype(q_tag)::value, u = q / PARTS, p = q % PARTS;
        constexpr int v = (q + 1) % (SETS * PARTS), vu = v / PARTS % 4;  // the next part, its step
        if constexpr (u % 2 == 1 && p == PARTS - 1) {
            lds_barrier();
            slot_store(u / 2 % 2);
            slot_load();
        }
        if constexpr (p == 0) rows_load(kf[(u + SETS - 1) % SETS]);
        frags(vu >> 1, vu & 1, v % PARTS, hf[v & 1]);
#pragma unroll
        for (int kb = 0; kb < kRB; ++kb)
#pragma unroll
            for (int hb = 0; hb < kHP; ++hb) {
                f32x4& c = acc[kb][p * kHP + hb];
                c = mfma16x16x32(hf[q & 1][hb], kf[u][kb], zero ? f32x4{} : c);
            }
#pragma unroll
        for (int i = 0; i < kRB; ++i) {
            if (p == 0) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // VMEM read
            __builtin_amdgcn_sched_group_barrier(0x008, kHP, 0);            // MFMA
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto body = [&](auto first_tag) {
        constexpr bool first = decltype(first_tag)::value;
        for_each_index(std::make_integer_sequence<int, SETS * PARTS>{},
                       [&](auto q) { part(q, first && decltype(q)::value < PARTS); });
    };

    for (int t = t0; t < t1; ++t) {
        wrap = (t + 1 < t1 ? tile_bytes : 0) - kc * 1024;
        body(std::true_type{});
        for (int j = SETS; j < kc; j += SETS) body(std::false_type{});
        // the lane's 4 HB bits of each row, collected from the top down; rel is the row within the call
        const int ln = fresh_lane();
        const int rel0 = (t * kTile + wv * kRB) * 16 - (int)(row0 & 15) + (ln & 15);
        uint8_t* const dst0 = sig + row0 * kBytes + (ln >> 4) * (HB / 2);
#pragma unroll
        for (int kb = 0; kb < kRB; ++kb) {
            uint32_t x[2] = {0u, 0u};
#pragma unroll
            for (int hb = HB - 1; hb >= 0; --hb)
#pragma unroll
                for (int i = 3; i >= 0; --i) x[hb >> 3] = push_sign(x[hb >> 3], acc[kb][hb][i]);
            const int rel = rel0 + kb * 16;
            if (rel >= 0 && rel < n) {
                uint8_t* dst = dst0 + (int64_t)rel * kBytes;
                if constexpr (HB == 16) {
                    *(uint2*)dst = uint2{~x[0], ~x[1]};
                } else if constexpr (HB == 8) {
                    *(uint32_t*)dst = ~x[0];
                } else if constexpr (HB == 4) {
                    *(uint16_t*)dst = (uint16_t)~x[0];
                } else {
#pragma unroll
                    for (int y = 0; y < HB / 2; ++y) dst[y] = (uint8_t)(~x[y >> 2] >> (8 * (y & 3)));
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        kbase += tile_bytes;
        koff -= tile_bytes;
        krs = __builtin_amdgcn_make_buffer_rsrc((void*)kbase, 0, 0x7FFFFFFF, 0x00020000);
    }
}

// One signature byte per lane: blocks b0 (bits 0..3) and b1 (bits 4..7) of the hyperplanes against 16 vectors, S
// column chunks c0 .. c0+S-1, every operand load of the batch issued before its first MFMA.  xat(c) gives the
// lane's piece of vector chunk c.
template <int S, class X>
__device__ __forceinline__ void simhash_batch(X xat, const u32x4* __restrict__ b0, const u32x4* __restrict__ b1,
                                              int c0, f32x4& lo, f32x4& hi) {
    u32x4 x[S], y0[S], y1[S];
#pragma unroll
    for (int u = 0; u < S; ++u) {
        x[u] = xat(c0 + u);
        y0[u] = b0[(c0 + u) * 64];
        y1[u] = b1[(c0 + u) * 64];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < S; ++u) {
        lo = mfma16x16x32(y0[u], x[u], lo);
        hi = mfma16x16x32(y1[u], x[u], hi);
    }
}

// Byte `wv` (0 .. words-1) of every lane's signature bytes for 16 vectors of kc chunks.
template <class X>
__device__ __forceinline__ uint32_t simhash_byte(X xat, const u32x4* __restrict__ hp_tiled, int kc, int wv, int lane) {
    const u32x4* b0 = hp_tiled + (int64_t)(2 * wv) * kc * 64 + lane;
    const u32x4* b1 = b0 + (int64_t)kc * 64;
    f32x4 lo = f32x4{0.f, 0.f, 0.f, 0.f}, hi = f32x4{0.f, 0.f, 0.f, 0.f};
    int c = 0;
    for (; c + 8 <= kc; c += 8) simhash_batch<8>(xat, b0, b1, c, lo, hi);
    if (c < kc) simhash_batch<4>(xat, b0, b1, c, lo, hi);  // kc is a multiple of 4
    return sign_byte(lo, hi);
}

// Signatures of few rows (simhash_by_wave): one wave per (16-row group, signature byte of
// every lane), so that the blocks of a group are computed in parallel.  Rows outside [row0, row0 + n) are not
// written.  Grid-stride over the waves.
__global__ __launch_bounds__(256) void k_simhash_few(const u32x4* __restrict__ rows_tiled, int kc, int64_t row0,
                                                     int64_t n, const u32x4* __restrict__ hp_tiled, int words,
                                                     uint8_t* __restrict__ sig) {
    const int lane = threadIdx.x & 63;
    // groups grow with the wave index, so the first one past the rows ends the loop
    for (int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);; wave += (int64_t)gridDim.x * 4) {
        const int64_t g = (row0 >> 4) + wave / words;
        const int wv = (int)(wave % words);
        if (g * 16 >= row0 + n) break;
        const u32x4* a = rows_tiled + g * kc * 64 + lane;
        const uint32_t byte = simhash_byte([&](int c) { return a[c * 64]; }, hp_tiled, kc, wv, lane);
        const int64_t row = g * 16 + (lane & 15);
        if (row >= row0 && row < row0 + n) sig[row * (4 * words) + (lane >> 4) * words + wv] = (uint8_t)byte;
    }
}

// Query preparation for the LSH lookup, one workgroup of 16 waves per 16 queries: wave w normalises and
// rounds query 16 g + w into the tiled scratch exactly as stored vectors are (zeros past the batch) and
// clears its candidate count; after the barrier wave w < bits / 32 computes byte w of every lane's part of the
// signatures with the MFMA sequence of the stored rows (so a query equal to a stored key gets its signature).
// NC > 0 (d_pad <= 512 NC): the query row is read once into registers, and the rounded queries are also
// kept in LDS (the tiled chunk layout), where the signature MFMAs read them; the hyperplane chunks are
// loaded eight at a time.  NC = 0: any d, the rows read twice and the queries read back from the scratch.
template <int NC>
__global__ __launch_bounds__(1024) void k_lsh_prep(const void* __restrict__ queries, int dtype, int nb, int d,
                                                   int d_pad, uint16_t* __restrict__ qt,
                                                   const u32x4* __restrict__ hp_tiled, int bits,
                                                   uint32_t* __restrict__ sigq, uint32_t* __restrict__ cnt) {
    __shared__ u32x4 qs[NC > 0 ? 16 * 64 * NC : 1];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int g = blockIdx.x;
    const int r = g * 16 + wv;
    const bool live = r < nb;
    const int kc = d_pad >> 5;
    const char* src = (const char*)queries + (live ? (int64_t)r * d * (dtype == 0 ? 4 : 2) : 0);
    if constexpr (NC > 0) {
        float x[NC][8];
        row_to_regs<NC>(src, dtype, d, live, lane, x);
        const double n = regs_norm<NC>(x);
        uint32_t z[NC * 4];
        quantise_row<NC>(x, n, quotient_rcp_f32(n), d, lane, z);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int j0 = lane * 8 + 512 * c, J = j0 >> 3;
            if (j0 < d_pad) {
                const u32x4 w = piece(z, c);
                *(u32x4*)(qt + tiled_offset(r, j0, kc)) = w;
                qs[(J >> 2) * 64 + (J & 3) * 16 + wv] = w;
            }
        }
    } else {
        normalise_row(src, dtype, d, d_pad, live, lane,
                      [&](int j0, u32x4 w) { *(u32x4*)(qt + tiled_offset(r, j0, kc)) = w; });
    }
    if (live && lane == 0) cnt[r] = 0u;
    __syncthreads();
    const int words = bits >> 5;
    if (wv >= words) return;
    const u32x4* a = (const u32x4*)qt + (int64_t)g * kc * 64 + lane;
    auto xat = [&](int c) { return NC > 0 ? qs[c * 64 + lane] : a[c * 64]; };
    const uint32_t byte = simhash_byte(xat, hp_tiled, kc, wv, lane);
    const int row = g * 16 + (lane & 15);
    if (row < nb) ((uint8_t*)sigq)[(int64_t)row * (4 * words) + (lane >> 4) * words + wv] = (uint8_t)byte;
}

// ---------------------------------------------------------------------------
// Candidate scan: every (entry, query) pair whose signatures differ in at most `radius` bits.  Counted with XOR
// and popcount the scan is bound by the vector ALU (two operations per word and pair, 72 us for 100 queries on
// 1M 256-bit signatures); as a contraction it runs on the matrix cores, in 4-bit floats: with key bits as 0 / 1
// and query bits as -1 / +1, their dot product is popc(key & q) - popc(key & ~q), so the Hamming distance is
// popc(q) - dot, and with the accumulator started at radius - popc(q) a pair is a candidate exactly when it
// ends >= 0 (integers up to 256: exact).  v_mfma_f32_16x16x128_f8f6f4 takes 32 elements per lane and operand:
// one signature word, expanded to 4 registers of 8 nibbles by masks and shifts.  Both operands number the
// elements alike, and that is all a dot product needs.  100 queries on 1M 256-bit signatures: 16 us (256: 30 us
// against 176 us, 1024: 92 us against 680 us).
// ---------------------------------------------------------------------------
typedef int i32x8 __attribute__((ext_vector_type(8)));

// The 32 bits of a key word as 32 nibbles, bit 4 i + j in nibble i of word j.  Three bits of each four stay where
// they are (as 0.5, 1 and 2 in E2M1), the fourth, the sign's place, moves down to 1; the query's values make up for it.
__device__ __forceinline__ u32x4 key_nibbles(uint32_t w) {
    return u32x4{w & 0x11111111u, w & 0x22222222u, w & 0x44444444u, (w >> 2) & 0x22222222u};
}
// The query's: +2, +1, +0.5 and +1 where the bit is set, the negative where not.
__device__ __forceinline__ u32x4 query_nibbles(uint32_t w) {
    constexpr uint32_t k = 0x88888888u;
    const u32x4 sign = u32x4{~w << 3, ~w << 2, ~w << 1, ~w} & u32x4{k, k, k, k};
    return sign | u32x4{0x44444444u, 0x22222222u, 0x11111111u, 0x22222222u};
}

// D = A B + c over 128 elements: 16 keys (A rows) x 16 queries (B columns), 4-bit floats, no scaling.
__device__ __forceinline__ f32x4 mfma_fp4(u32x4 a, u32x4 b, f32x4 c) {
    const i32x8 a8{(int)a.x, (int)a.y, (int)a.z, (int)a.w, 0, 0, 0, 0};
    const i32x8 b8{(int)b.x, (int)b.y, (int)b.z, (int)b.w, 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a8, b8, c, 4, 4, 0, 0, 0, 0);
}

constexpr int kScanThreads = 512;
constexpr int kScanQueries = 480;  // queries of one workgroup (grid y): their operands take up to 62 KiB of LDS
constexpr int kScanBlocks = 4;     // 16-key blocks a wave holds expanded while it walks the queries
constexpr int kScanGroups = 4;     // groups of that many whose signatures it loads at once

// Lane l of a block's operands holds words word_of(0, l / 16) (and word_of(1, l / 16): W > 4 words, NM = 2
// products) of vector l % 16, zeros past the signature.
template <int W>
struct ScanWords {
    static constexpr int NM = W > 4 ? 2 : 1;
    __device__ static int word_of(int m, int q) { return W == 8 ? 2 * q + m : 4 * m + q; }
    // the lane's words of row i (0 for a row past the store)
    __device__ static void load(const uint32_t* __restrict__ sig, int64_t i, int64_t n_rows, int q, uint32_t (&w)[NM]) {
        const bool live = i < n_rows;
        if constexpr (W == 8) {
            const uint2 x = live ? *(const uint2*)(sig + i * 8 + 2 * q) : uint2{0u, 0u};
            w[0] = x.x, w[1] = x.y;
        } else {
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const int j = word_of(m, q);
                w[m] = live && j < W ? sig[i * W + j] : 0u;
            }
        }
    }
};

// Candidates are appended to the query's list (at most max_cand kept; cnt counts them all).
template <int W>
__global__ __launch_bounds__(kScanThreads, 4) void k_lsh_scan(const uint32_t* __restrict__ sig_keys, int64_t n_rows,
                                                           const uint32_t* __restrict__ sig_q, int nb, int radius,
                                                           int max_cand, int groups, uint32_t* __restrict__ cnt,
                                                           int32_t* __restrict__ cand) {
    constexpr int NM = ScanWords<W>::NM;
    extern __shared__ u32x4 qop[];                       // [query block][NM][64] query operands, then
    const int q0 = (int)blockIdx.y * kScanQueries;
    const int nq = nb - q0 < kScanQueries ? nb - q0 : kScanQueries;
    const int nblk = (nq + 15) / 16;
    float* start = (float*)(qop + nblk * NM * 64);       // [nblk][16] radius - popc(q)
    const int tid = threadIdx.x, lane = tid & 63;
    auto stage_queries = [&]() {
        for (int e = tid; e < nblk * NM * 64; e += kScanThreads) {
            const int l = e & 63, m = (e >> 6) % NM, q = (e >> 6) / NM * 16 + (l & 15);
            const int j = ScanWords<W>::word_of(m, l >> 4);
            u32x4 v = u32x4{0u, 0u, 0u, 0u};
            if (q < nq && j < W) v = query_nibbles(sig_q[(int64_t)(q0 + q) * W + j]);
            qop[e] = v;
        }
        for (int q = tid; q < nblk * 16; q += kScanThreads) {
            int c = -1;  // no query: never a candidate
            if (q < nq) {
                c = radius;
    #pragma unroll
                for (int j = 0; j < W; ++j) c -= __popc(sig_q[(int64_t)(q0 + q) * W + j]);
            }
            start[q] = (float)c;
        }
    };
    // the wave's entries of a turn: `groups` groups of 64, their words all loaded at once; as each group is
    // expanded its registers take the next turn's words
    const int64_t turn = (int64_t)groups * kScanBlocks * 16;
    const int64_t stride = (int64_t)gridDim.x * (kScanThreads / 64) * turn;
    int64_t i0 = ((int64_t)blockIdx.x * (kScanThreads / 64) + (tid >> 6)) * turn;
    uint32_t w[kScanGroups][kScanBlocks][NM];
    auto load_group = [&](int64_t i, uint32_t (&x)[kScanBlocks][NM]) {
#pragma unroll
        for (int t = 0; t < kScanBlocks; ++t)
            ScanWords<W>::load(sig_keys, i + t * 16 + (lane & 15), n_rows, lane >> 4, x[t]);
    };
    if (i0 < n_rows) {
#pragma unroll
        for (int g = 0; g < kScanGroups; ++g)
            if (g < groups) load_group(i0 + g * kScanBlocks * 16, w[g]);
    }
    __builtin_amdgcn_sched_barrier(0);
    stage_queries();
    __syncthreads();
    for (; i0 < n_rows; i0 += stride) {
#pragma unroll
        for (int g = 0; g < kScanGroups; ++g) {
            if (g >= groups) continue;
            const int64_t ig = i0 + g * kScanBlocks * 16;
            u32x4 a[kScanBlocks][NM];
#pragma unroll
            for (int t = 0; t < kScanBlocks; ++t)
#pragma unroll
                for (int m = 0; m < NM; ++m) a[t][m] = key_nibbles(w[g][t][m]);
            if (i0 + stride < n_rows) load_group(ig + stride, w[g]);
            for (int b = 0; b < nblk; ++b) {
                const float s = start[b * 16 + (lane & 15)];
                f32x4 acc[kScanBlocks];
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    const u32x4 bq = qop[(b * NM + m) * 64 + lane];
#pragma unroll
                    for (int t = 0; t < kScanBlocks; ++t)
                        acc[t] = mfma_fp4(a[t][m], bq, m == 0 ? f32x4{s, s, s, s} : acc[t]);
                }
                float top = acc[0][0];
#pragma unroll
                for (int t = 0; t < kScanBlocks; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) top = fmaxf(top, acc[t][e]);
                if (__ballot(top >= 0.0f) == 0ull) continue;
                // lane l holds rows 4 (l / 16) + e of each block for query l % 16: bit 4 t + e of its candidates
                const int ln = fresh_lane();
                const int q = q0 + b * 16 + (ln & 15);
                const int64_t first = ig + 4 * (ln >> 4), left = n_rows - first;
                uint32_t mine = 0u;
#pragma unroll
                for (int t = 0; t < kScanBlocks; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        mine |= (acc[t][e] >= 0.0f && t * 16 + e < left ? 1u : 0u) << (4 * t + e);
                // A query's candidates among the 64 entries take their places with one addition.  The lists are counted
                // at few addresses, and with an addition per candidate a wide radius waits for nothing else: 16 queries
                // with all of 1M entries candidates 37 ms, 0.2 ms so; 100 queries on 20k entries 24 us, 19.5 us so.
                const uint32_t n = __popc(mine);
                const uint32_t n16 = __shfl_xor(n, 16, kWave), n32 = __shfl_xor(n + n16, 32, kWave);
                const uint32_t all = n + n16 + n32;
                uint32_t pos = 0u;
                if (ln < 16 && all != 0u) pos = atomicAdd(&cnt[q], all);
                pos = __shfl(pos, ln & 15, kWave) + ((ln & 16) ? n16 : 0u) + ((ln & 32) ? n32 : 0u);
                for (; mine != 0u && pos < (uint32_t)max_cand; mine &= mine - 1u, ++pos) {
                    const int k = __ffs(mine) - 1;
                    cand[(int64_t)q * max_cand + pos] = (int32_t)(first + (k >> 2) * 16 + (k & 3));
                }
            }
        }
    }
}

// The same scan by XOR and popcount, for at most kFewQueries queries: the matrix cores work for 16 whatever the
// count, and expanding the signatures costs as much as counting for four (1M 256-bit signatures: 4.6 us against
// 6.6 us for one query; 15 us against 6.9 us for 16).  Each thread takes kScanKeys entries at a time.
constexpr int kFewQueries = 3;
constexpr int kScanKeys = 4;
__global__ __launch_bounds__(256) void k_lsh_scan_few(const uint32_t* __restrict__ sig_keys, int64_t n_rows,
                                                      const uint32_t* __restrict__ sig_q, int nq, int words,
                                                      int radius, int max_cand, uint32_t* __restrict__ cnt,
                                                      int32_t* __restrict__ cand) {
    __shared__ uint32_t sq[kFewQueries * 8];  // [nq][words]
    for (int i = threadIdx.x; i < nq * words; i += 256) sq[i] = sig_q[i];
    __syncthreads();
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x; i0 < n_rows; i0 += kScanKeys * stride) {
        uint32_t k[kScanKeys][8];
#pragma unroll
        for (int e = 0; e < kScanKeys; ++e) {
            const int64_t i = i0 + e * stride;
            if ((words & 3) == 0) {  // 16-byte loads (signature rows are 16-byte aligned then)
                const uint4* p = (const uint4*)(sig_keys + i * words);
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    const uint4 x = (v * 4 < words && i < n_rows) ? p[v] : uint4{0u, 0u, 0u, 0u};
                    k[e][4 * v] = x.x, k[e][4 * v + 1] = x.y, k[e][4 * v + 2] = x.z, k[e][4 * v + 3] = x.w;
                }
            } else {
#pragma unroll
                for (int w = 0; w < 8; ++w) k[e][w] = (w < words && i < n_rows) ? sig_keys[i * words + w] : 0u;
            }
        }
        for (int b = 0; b < nq; ++b) {
            int h[kScanKeys] = {};
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                if (w < words) {
                    const uint32_t qw = sq[b * words + w];
#pragma unroll
                    for (int e = 0; e < kScanKeys; ++e) h[e] += __popc(k[e][w] ^ qw);
                }
            }
#pragma unroll
            for (int e = 0; e < kScanKeys; ++e) {
                const int64_t i = i0 + e * stride;
                if (i < n_rows && h[e] <= radius) {
                    const uint32_t pos = atomicAdd(&cnt[b], 1u);
                    if (pos < (uint32_t)max_cand) cand[(int64_t)b * max_cand + pos] = (int32_t)i;
                }
            }
        }
    }
}

// One wave per query: the exact similarity of each candidate (the query and the entry read from their tiled
// stores, bf16 products summed in float32), the best as a packed top-1 (order-free: highest score, lowest
// index), then the threshold and stage 2 (verify_query); n_cand receives the candidate count.
__global__ __launch_bounds__(256) void k_lsh_verify(const u32x4* __restrict__ keys_tiled,
                                                    const u32x4* __restrict__ qt, int kc, int B,
                                                    const uint32_t* __restrict__ cnt,
                                                    const int32_t* __restrict__ cand, int max_cand,
                                                    int32_t* __restrict__ n_cand, int n_rows, int dtype,
                                                    const VerifyArgs v) {
    const int lane = threadIdx.x & 63;
    const int b = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (b >= B) return;
    const uint32_t c_all = cnt[b];
    const int nc = c_all < (uint32_t)max_cand ? (int)c_all : max_cand;
    const int d_pad = kc * 32;
    uint64_t best = 0ull;
    for (int t = 0; t < nc; ++t) {
        const int32_t i = cand[(int64_t)b * max_cand + t];
        float acc = 0.0f;
        for (int j0 = lane * 8; j0 < d_pad; j0 += 512) {
            const u32x4 kv = *(const u32x4*)((const uint16_t*)keys_tiled + tiled_offset(i, j0, kc));
            const u32x4 qv = *(const u32x4*)((const uint16_t*)qt + tiled_offset(b, j0, kc));
            acc = dot8_bf16(qv, kv, acc);
        }
        acc = wave_sum_f32(acc);
        best = umax64(best, pack_top1(acc, i));
    }
    if (lane == 0) n_cand[b] = (int32_t)c_all;
    verify_query<IN_PLACE>(b, best, unpack_idx(best), unpack_score(best), n_rows, dtype, v, lane);
}

hipError_t launch_tile_hyperplanes(const uint16_t* src, int bits, int d, int d_pad, uint16_t* dst, hipStream_t s) {
    const int64_t total = (int64_t)bits * d_pad;
    if (total <= 0) return hipSuccess;
    k_tile_hyperplanes<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s>>>(src, bits >> 5, d, d_pad, dst);
    return hipGetLastError();
}

template <int HB, int PARTS, int SETS>
static void launch_bulk(const uint16_t* rows_tiled, int kc, int64_t row0, int64_t n, const uint16_t* hp_tiled,
                        uint32_t* sig, int num_cu, hipStream_t s) {
    const int64_t groups = ((row0 + n + 15) >> 4) - (row0 >> 4);
    const int n_tiles = (int)((groups + 15) / 16);
    const int cap = HB <= 6 ? 2 * num_cu : num_cu;  // the workgroups that the registers allow at once
    k_simhash_bulk<HB, PARTS, SETS><<<dim3(n_tiles < cap ? n_tiles : cap), dim3(256), 0, s>>>(
        (const u32x4*)rows_tiled, kc, row0, n, (const u32x4*)hp_tiled, n_tiles, (uint8_t*)sig);
}

hipError_t launch_simhash(const uint16_t* rows_tiled, int d_pad, int64_t row0, int64_t n, const uint16_t* hp_tiled,
                          int bits, uint32_t* sig, int num_cu, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int words = bits >> 5, kc = d_pad >> 5;
    if (simhash_by_wave(n, bits)) {
        const int64_t groups = ((row0 + n + 15) >> 4) - (row0 >> 4);
        k_simhash_few<<<dim3((unsigned)grid_blocks((groups * words + 3) / 4)), dim3(256), 0, s>>>(
            (const u32x4*)rows_tiled, kc, row0, n, (const u32x4*)hp_tiled, words, (uint8_t*)sig);
        return hipGetLastError();
    }
    // d_pad % 256 == 0: whole groups of 8 steps, so the rows are loaded 7 steps ahead where the registers allow
    // (1M x 768 rows, 256 bits: 345 us against 367 us three steps ahead)
    const bool deep = kc % 8 == 0;
    auto run = [&](auto shallow, auto deeper) {
        (deep ? deeper : shallow)(rows_tiled, kc, row0, n, hp_tiled, sig, num_cu, s);
    };
    switch (words) {
        case 1: run(launch_bulk<2, 1, 4>, launch_bulk<2, 1, 4>); break;
        case 2: run(launch_bulk<4, 1, 4>, launch_bulk<4, 1, 4>); break;
        case 3: run(launch_bulk<6, 1, 4>, launch_bulk<6, 1, 4>); break;
        case 4: run(launch_bulk<8, 1, 4>, launch_bulk<8, 1, 8>); break;
        case 5: run(launch_bulk<10, 2, 4>, launch_bulk<10, 2, 8>); break;
        case 6: run(launch_bulk<12, 2, 4>, launch_bulk<12, 2, 8>); break;
        case 7: run(launch_bulk<14, 2, 4>, launch_bulk<14, 2, 8>); break;
        case 8: run(launch_bulk<16, 2, 4>, launch_bulk<16, 2, 8>); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int W>
static void launch_scan(const uint32_t* sig_keys, int64_t n_rows, const uint32_t* sigq, int nb, int radius,
                        int max_cand, uint32_t* cnt, int32_t* cand, int num_cu, hipStream_t s) {
    const int chunks = (nb + kScanQueries - 1) / kScanQueries;
    const int nblk = ((nb < kScanQueries ? nb : kScanQueries) + 15) / 16;
    const size_t lds = (size_t)nblk * (ScanWords<W>::NM * 1024 + 64);
    // Two workgroups per CU are resident (registers, and LDS for the largest batches).  As many groups per wave as
    // let those hold the whole store, so that every signature is on its way at once (16 queries on 1M
    // entries: 6.9 us against 9.0 us with one group at a time); few entries spread over more waves instead.
    const int64_t waves = (int64_t)2 * num_cu * (kScanThreads / 64);
    const int64_t tiles = (n_rows + kScanBlocks * 16 - 1) / (kScanBlocks * 16);
    int64_t groups = (tiles + waves - 1) / waves;
    if (groups > kScanGroups) groups = kScanGroups;
    const int64_t per = groups * (kScanThreads / 64);
    int64_t blocks = (tiles + per - 1) / per;
    if (blocks > 2 * num_cu) blocks = 2 * num_cu;
    k_lsh_scan<W><<<dim3((unsigned)blocks, chunks), dim3(kScanThreads), lds, s>>>(
        sig_keys, n_rows, sigq, nb, radius, max_cand, (int)groups, cnt, cand);
}

hipError_t launch_lsh_lookup(const void* queries, int dtype, int nb, int d, int d_pad, uint16_t* qt,
                             const uint16_t* hp_tiled, int bits, uint32_t* sigq, const uint16_t* keys_tiled,
                             const uint32_t* sig_keys, int64_t n_rows, int radius, int max_cand, uint32_t* cnt,
                             int32_t* cand, int32_t* n_cand, const VerifyArgs& v, int num_cu, hipStream_t s) {
    if (nb <= 0) return hipSuccess;
    const int words = bits >> 5;
    if (words < 1 || words > 8) return hipErrorInvalidValue;
    const dim3 pg((unsigned)((nb + 15) / 16)), pb(1024);
    const u32x4* hp = (const u32x4*)hp_tiled;
    if (d_pad <= 512)
        k_lsh_prep<1><<<pg, pb, 0, s>>>(queries, dtype, nb, d, d_pad, qt, hp, bits, sigq, cnt);
    else if (d_pad <= 1024)
        k_lsh_prep<2><<<pg, pb, 0, s>>>(queries, dtype, nb, d, d_pad, qt, hp, bits, sigq, cnt);
    else if (d_pad <= 2048)
        k_lsh_prep<4><<<pg, pb, 0, s>>>(queries, dtype, nb, d, d_pad, qt, hp, bits, sigq, cnt);
    else
        k_lsh_prep<0><<<pg, pb, 0, s>>>(queries, dtype, nb, d, d_pad, qt, hp, bits, sigq, cnt);
    if (n_rows > 0 && nb <= kFewQueries) {
        // every thread a whole run of kScanKeys entries (no idle slots), at most 8 workgroups per CU
        int64_t blocks = (n_rows + 256 * kScanKeys - 1) / (256 * kScanKeys);
        if (blocks > 8 * num_cu) blocks = 8 * num_cu;
        k_lsh_scan_few<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(sig_keys, n_rows, sigq, nb, words, radius, max_cand,
                                                                   cnt, cand);
    } else if (n_rows > 0) {
        switch (words) {
            case 1: launch_scan<1>(sig_keys, n_rows, sigq, nb, radius, max_cand, cnt, cand, num_cu, s); break;
            case 2: launch_scan<2>(sig_keys, n_rows, sigq, nb, radius, max_cand, cnt, cand, num_cu, s); break;
            case 3: launch_scan<3>(sig_keys, n_rows, sigq, nb, radius, max_cand, cnt, cand, num_cu, s); break;
            case 4: launch_scan<4>(sig_keys, n_rows, sigq, nb, radius, max_cand, cnt, cand, num_cu, s); break;
            case 5: launch_scan<5>(sig_keys, n_rows, sigq, nb, radius, max_cand, cnt, cand, num_cu, s); break;
            case 6: launch_scan<6>(sig_keys, n_rows, sigq, nb, radius, max_cand, cnt, cand, num_cu, s); break;
            case 7: launch_scan<7>(sig_keys, n_rows, sigq, nb, radius, max_cand, cnt, cand, num_cu, s); break;
            default: launch_scan<8>(sig_keys, n_rows, sigq, nb, radius, max_cand, cnt, cand, num_cu, s); break;
        }
    }
    k_lsh_verify<<<dim3((unsigned)((nb + 3) / 4)), dim3(256), 0, s>>>(
        (const u32x4*)keys_tiled, (const u32x4*)qt, d_pad >> 5, nb, cnt, cand, max_cand, n_cand, (int)n_rows,
        dtype, v);
    return hipGetLastError();
}

}  // namespace lacache
