// launch.hpp -- host-side launchers of the gfx950 kernels (called by the C ABI in lacache.cpp).
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <tuple>
#include <utility>

namespace lacache {

// Workgroups of a grid-stride launch: at most 2^20, so that a grid's work-items (blocks x threads, up to
// 1024 threads) stay far below the 2^32 one dispatch can describe, whatever the row or pair count.
constexpr int64_t kMaxGridBlocks = int64_t(1) << 20;
inline int64_t grid_blocks(int64_t want) { return want < 1 ? 1 : (want > kMaxGridBlocks ? kMaxGridBlocks : want); }

// Allow kernel `fn` `bytes` of dynamic LDS on the current device, once per device (bit d of `done`; devices
// past 63 set it on every call).  Safe to call from several threads.
inline hipError_t allow_dynamic_lds(const void* fn, int bytes, std::atomic<uint64_t>& done) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev < 64 ? (uint64_t(1) << dev) : 0;
    if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess && bit) done.fetch_or(bit, std::memory_order_acq_rel);
    return e;
}

// Launch `kernel` on stream s.  With events e0 and e1 (both or neither) the launch goes through
// hipExtLaunchKernel, which takes the kernel's own start and end times into them from its dispatch: no
// event packets of their own on the stream, so timing a kernel does not change the gaps around it.
template <typename... P, typename... A>
hipError_t launch_timed(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t s, hipEvent_t e0,
                        hipEvent_t e1, A... args) {
    static_assert(sizeof...(P) == sizeof...(A), "one argument per kernel parameter");
    if (!e0) {
        kernel<<<grid, block, lds, s>>>(static_cast<P>(args)...);
        return hipGetLastError();
    }
    std::tuple<P...> t{static_cast<P>(args)...};
    return std::apply(
        [&](auto&... v) {
            void* a[] = {(void*)&v...};
            return hipExtLaunchKernel((const void*)kernel, grid, block, a, lds, s, e0, e1, 0);
        },
        t);
}

// Normalise `rows` input rows (dtype 0 f32 / 1 bf16, row-major [rows][d]) and
// store them as bfloat16 at destination rows row0 .. row0+rows-1, zero-filling
// up to rows_pad rows and d_pad columns; `tiled` selects the key layout,
// otherwise row-major [.][d_pad].
hipError_t launch_normalise(const void* in, int dtype, int64_t rows, int64_t rows_pad, int d, int d_pad,
                            uint16_t* out, int64_t row0, bool tiled, hipStream_t s);

// The arrays of an insert or an export: rows of keys (tiled store), of up to kMaxModels prefix-embedding
// models (row-major stores) and of prefix tokens.  Callers' arrays are dense ([n][d], [n][k_cap]).
constexpr int kMaxModels = 8;
struct EntryArrays {
    const void* keys;                 // caller's rows (insert) or the store (export)
    uint16_t* keys_out;               // the store (insert) or the caller's rows (export); null: not wanted
    int d, d_pad;
    int m;
    const void* emb[kMaxModels];
    uint16_t* emb_out[kMaxModels];    // null: not wanted
    int d_resp[kMaxModels], d_pad_resp[kMaxModels];
    const int32_t* tokens;
    int32_t* tokens_out;              // null: not wanted
    int k_cap;
};

// Store n entries at rows row0 .. row0+n-1: vectors normalised and rounded to bfloat16, tokens copied (the store's
// arrays are their bases, not row row0).
hipError_t launch_insert(const EntryArrays& a, int dtype, int64_t n, int64_t row0, hipStream_t s);

// Dense copies of stored rows first .. first+n-1.
hipError_t launch_export(const EntryArrays& a, int64_t first, int n, hipStream_t s);

// The response-prefix embedding models of stage 2 (one per lookahead check of an ensemble).
struct PrefixModels {
    int m;                             // number of models, 1 .. kMaxModels
    const void* la[kMaxModels];        // [B][d_i] lookahead embeddings of the batch (cache dtype)
    const uint16_t* emb[kMaxModels];   // [capacity][d_pad_i] stored normalised prefix embeddings
    int d[kMaxModels], d_pad[kMaxModels];
    float tau[kMaxModels];             // stage-2 threshold of each model
};

// What the end of a lookup needs besides the stage-1 candidates: stage 2's inputs and the outputs of the batch.
struct VerifyArgs {
    PrefixModels models;
    const int32_t* la_tok;   // [B][k]
    int k;
    const int32_t* tokens;   // [capacity][k_cap]
    int k_cap;
    float tau_q;
    int32_t* idx;
    float* score;
    float* resp_score;       // [B][models.m]
    int32_t* decision;
};

// Stage 1, bandwidth-bound path: queries qt (tiled; up to 16 * stream_max_qg rows as one group, zero-padded to
// a multiple of 16, or up to four such groups, zero-padded to whole groups) against n_rows tiled keys.  Writes, for every query b
// and every workgroup p of the launch, the packed top-1 candidate
// part[b * P + p] (P <= kMaxPartials).  Returns the number of partials P through *P_out.
// With events e0 / e1 the kernel's run time is recorded into them (launch_timed).  With qraw (the caller's
// [B][d] query rows, dtype 0 f32 / 1 bf16) the kernel normalises the queries itself and qt is not read; this
// takes d_pad <= 2048 (stream_fused_ncq(d_pad) > 0) and B <= 32.  With `verify` too (lookup_in_one_launch) the
// workgroup that ends last also merges the partials and runs stage 2, so no launch follows; it counts in the slot of
// `ticket` in done (done_slots.hpp: the caller gives every launch the ticket after the last one's).
hipError_t launch_stage1_stream(const uint16_t* keys, const uint16_t* qt, int B, int n_rows, int d_pad,
                                uint64_t* part, int num_cu, int* P_out, hipStream_t s, hipEvent_t e0 = nullptr,
                                hipEvent_t e1 = nullptr, const void* qraw = nullptr, int dtype = 0, int d = 0,
                                const VerifyArgs* verify = nullptr, uint32_t* done = nullptr, uint32_t ticket = 0);
int stream_fused_ncq(int d_pad);
// Whether a lookup of B queries (d_pad columns) on n_rows entries, its prefix models of resp_columns padded columns in
// all, ends in its streaming launch.  That saves a launch, but one workgroup then does what the launch spreads over
// the chip, each wave a query, one model after another.  One launch / two, us a call, back to back: 1, 8, 16 and 32
// queries on 10k x 384 float32 keys 9.6 / 10.8, 10.5 / 11.5, 11.8 / 12.3, 16.6 / 14.5; on 200k x 768 bfloat16 keys
// 53.6 / 53.9, 52.6 / 53.1, 54.3 / 54.1, 60.2 / 56.3; 20k x 768 float32 entries with four models (3200 columns), 1, 8
// and 16 queries 17.1 / 17.7, 19.6 / 19.9, 24.4 / 21.1; bfloat16 ones with two of 1536 and 2048 columns 20.9 / 21.2,
// 23.2 / 22.4, 27.8 / 23.1.  In a replayed graph, where a launch costs less, the two are even up to 4 queries, 8 take
// up to 0.4 us longer in one launch and 16 0.6 to 1.8 us; so 9 to 16 queries take one launch only on the smallest
// stores, where calls wait for the host (16 queries on 10k x 64 bfloat16 keys 9.2 / 10.1 us, on 10k x 384 11.3 / 11.7,
// on 200k x 64 14.7 / 14.6).  Wider keys leave no registers for stage 2 beside the normaliser (176 bytes of scratch a
// lane: 16 queries on 200k x 1536 float32 keys 125 us, 110 us in two launches).
inline bool lookup_in_one_launch(int B, int64_t n_rows, int d_pad, int64_t resp_columns) {
    const int most = n_rows * d_pad <= (int64_t(1) << 23) ? 16 : 8;
    return B <= most && d_pad <= 1024 && B * resp_columns <= 12288;
}
// The kernels (16 qg queries, normalised in up to 512 ncq columns) that have stage 2 in them for it.
constexpr bool stream_ends_lookup(int qg, int ncq) { return qg == 1 && (ncq == 1 || ncq == 2); }

// The streaming pass for more queries than LDS holds, of 769 to 1024 columns (is_wide): B <= kWideQueries (rows of qt
// zero-padded to that); otherwise as launch_stage1_stream with staged queries.
constexpr int kWideQueries = 128;
inline bool is_wide(int B, int d_pad) { return B > 64 && B <= kWideQueries && (d_pad == 896 || d_pad == 1024); }
hipError_t launch_stage1_wide(const uint16_t* keys, const uint16_t* qt, int B, int n_rows, int d_pad, uint64_t* part,
                              int num_cu, int* P_out, hipStream_t s, hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);

// Stage 1, compute-bound path (matrix-core GEMM with a fused row maximum): queries qt (tiled, rows zero-padded
// to a multiple of kGemmQueryTile) against n_rows keys.  The key store must hold whole tiles of kGemmKeyTile
// rows plus one spare tile past the last one (the kernel prefetches into it; its rows are never scored).  Its
// partials name the 16-row group of the candidate (global row / 16) instead of the row; the finalize step
// recovers the row by replaying that group (part_groups = true).
constexpr int kGemmKeyTile = 512;
constexpr int kGemmQueryTile = 128;
hipError_t launch_stage1_gemm(const uint16_t* keys, const uint16_t* qt, int B, int n_rows, int d_pad,
                              uint64_t* part, int num_cu, int* P_out, hipStream_t s, hipEvent_t e0 = nullptr,
                              hipEvent_t e1 = nullptr);

// Merge the P partial candidates of each query (rows, or 16-row groups to replay against keys_tiled and
// the tiled queries qt), threshold, and run stage 2 on hits.  resp_score is [B][models.m].  Every query whose
// group replay does not reproduce its stage-1 score adds 1 to *fallbacks (device memory).
hipError_t launch_finalize_verify(const uint64_t* part, int P, bool part_groups, const uint16_t* keys_tiled,
                                  const uint16_t* qt, int B, int n_rows, int dtype, int d_keys, const VerifyArgs& v,
                                  uint32_t* fallbacks, hipStream_t s);

// Threshold calibration over n pairs (a[j], b[j]) of d-dimensional input vectors: sims[j] = the lookup's
// cosine of the pair; tau[0] = the percentile (linear between the closest ranks), tau[1] = min(cap, tau[0]).
// scratch: kCalibScratchWords words of device memory.
constexpr int kCalibScratchWords = 64 + 2 * 2048;
hipError_t launch_calibrate(const void* a, const void* b, int dtype, int d, int64_t n, float percentile, float cap,
                            float* sims, float* tau, uint32_t* scratch, int num_cu, hipStream_t s);

// Device address, on the current device, of the library's static calibration scratch (kCalibScratchWords words,
// one copy per device, shared by every allocation-free calibration on that device).  Allocates nothing.
hipError_t calibrate_static_scratch(uint32_t** out);

// Speculative-decoding acceptance: p_target[b][j] = softmax(logits[b][j])[tokens[b][j]] (0 for an
// out-of-range token); accept_len[b] = the number of leading positions with p_target >= p_draft.
// Sixteen waves on each row of logits instead of four: few rows of many logits, where a row's own chain of loads is the
// bound; more rows fill the chip with four waves each, and in short ones most of the sixteen hold nothing.  Four /
// sixteen, us a call in a replayed graph: 256 rows of 1000, 4000 and 8192 float32 logits 5.1 / 5.1, 5.6 / 5.9,
// 6.3 / 6.1, of 12,000, 16,000 and 100,003 7.1 / 6.3, 9.2 / 6.9, 25.7 / 23.5; 100 rows of 12,000, 32,000 and 128,256
// bfloat16 ones 6.1 / 5.5, 12.1 / 9.3, 38 / 17.  Beyond 256 rows float32 ones hardly gain (260 rows of 50,257
// 18.9 / 19.2, 512 of 151,936 58.5 / 58.4); 512 rows of 100,003 bfloat16 ones take 38.9 / 22.1, of 8192 6.4 / 7.0, 2048
// of 128,256 88 / 95.
inline bool accept_many_waves(int64_t rows, int V, int dtype) {
    return rows <= 256 ? V >= 12000 : rows <= 1024 && dtype == 1 && V >= 96 * 1024;
}
hipError_t launch_accept_length(const void* logits, int dtype, int V, const int32_t* tokens, const float* p_draft,
                                int B, int k, int32_t* accept_len, float* p_target, hipStream_t s);

// LSH index (random hyperplanes): tiled copy of the raw hyperplanes (their rows in the order the signature
// kernels want), signatures of rows row0 .. row0+n-1 of a
// tiled matrix ([rows][bits / 32] words, bit i of a row is 1 when its projection on hyperplane i is >= 0),
// and the whole LSH lookup of a query batch (query preparation, Hamming-radius candidate scan, exact re-rank,
// threshold and stage 2).
// Whether the signatures of n rows are computed a wave per (16-row group, signature byte) or by the bulk kernel.  The
// first spreads a call over the whole chip but reads the hyperplanes once per group, so its time grows with rows x bits;
// the second lasts at least one tile's chain, whatever the rows.  Both grow with the columns alike.  Few / bulk, us to
// build an index of n rows in place: 64 bits x 2048 columns 28 / 39 at 12288 rows, 41 / 47 at 32768, 53 / 50 at 49152;
// 128 bits x 1024 28 / 30 at 16384, 35 / 31 at 24576; 256 bits x 768 31 / 35 at 12288, 36 / 36 at 16384, 46 / 36 at
// 24576; 256 x 2048 54 / 63, 66 / 63, 91 / 64; 32 bits x 384 20 / 21 at 49152, 22 / 22 at 65536.
inline bool simhash_by_wave(int64_t n, int bits) {
    const int64_t most = 2500000 / bits;
    return n <= (most < 14000 ? 14000 : most);
}
hipError_t launch_tile_hyperplanes(const uint16_t* src, int bits, int d, int d_pad, uint16_t* dst, hipStream_t s);
hipError_t launch_simhash(const uint16_t* rows_tiled, int d_pad, int64_t row0, int64_t n, const uint16_t* hp_tiled,
                          int bits, uint32_t* sig, int num_cu, hipStream_t s);
hipError_t launch_lsh_lookup(const void* queries, int dtype, int nb, int d, int d_pad, uint16_t* qt,
                             const uint16_t* hp_tiled, int bits, uint32_t* sigq, const uint16_t* keys_tiled,
                             const uint32_t* sig_keys, int64_t n_rows, int radius, int max_cand, uint32_t* cnt,
                             int32_t* cand, int32_t* n_cand, const VerifyArgs& v, int num_cu, hipStream_t s);

// Most partials a stage-1 launch may write per query.
constexpr int kMaxPartials = 1024;

}  // namespace lacache
