// Internal declarations shared by the host side of libatf.so and its kernels.
// Not part of the public ABI (include/atf.h is).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace atf {

constexpr int kMaxPairs = 64;     // d/2 for d = 128
constexpr int kChunkPairs = 8;    // pairs per QK K-step and per decode K-cache chunk
constexpr int kMaxChunks = kMaxPairs / kChunkPairs;

// Window table in the form every kernel consumes: per pair the integer threshold
// W_r (keep the pair's term at distance z iff z <= W_r), and per chunk of
// kChunkPairs consecutive pairs the smallest and largest threshold.
struct WindowTable {
    int32_t W[kMaxPairs];
    int32_t chunk_min[kMaxChunks];
    int32_t chunk_max[kMaxChunks];
};

struct PrefillParams {
    const uint16_t* q;   // [B][n_q][h_q][d]
    const uint16_t* k;   // [B][h_kv][d/16][cache_tokens][16] (pair-chunk-major)
    const uint16_t* v;   // [B][h_kv][ceil(cache_tokens/16)][d][16] (see atf_pack_vcache)
    uint16_t* o;         // [B][n_q][h_q][d]
    float* lse;          // [B][h_q][n_q]
    int32_t batch, n_q, n_k, q_pos0, h_q, h_kv, group;
    int32_t cache_tokens;  // tokens each cache entry is allocated for (>= n_k)
    int32_t pos_per_tile;  // query positions per workgroup (rows = positions x group)
    int32_t n_qtiles;
    int32_t mono;        // thresholds non-decreasing in r
    float scale_log2;    // softmax scale * log2(e)
    WindowTable win;
};

// Prefill with RoPE at read time: q and the K cache hold unrotated vectors, rotated
// in the kernel as DecodeParams describes. A type of its own, so that the kernels
// of pre-rotated caches keep their argument block.
struct PrefillRotParams : PrefillParams {
    uint32_t rope_rho_hi[kMaxPairs];
    uint32_t rope_rho_lo[kMaxPairs];
};

struct DecodeParams {
    const uint16_t* q;       // [B][h_q][d]
    const uint16_t* kpcm;    // [B][h_kv][d/16][cache_tokens][16]
    const uint16_t* vpk;     // [B][h_kv][ceil(cache_tokens/16)][d][16] (see atf_pack_vcache)
    uint16_t* o;             // [B][h_q][d]
    float* lse;              // [B][h_q]
    float* ws_m;             // [B][h_q][splits]   running max (log2 domain)
    float* ws_l;             // [B][h_q][splits]   normaliser
    float* ws_o;             // [B][h_q][splits][d] unnormalised output
    int32_t batch, n_k, q_pos, h_q, h_kv, group;
    int32_t cache_tokens;     // tokens each cache entry is allocated for (>= n_k)
    int32_t heads_per_block;  // query heads handled by one workgroup (divides group, <= 32)
    int32_t n_valid;          // keys 0 .. n_valid - 1 are causal
    const int32_t* n_k_rows;  // ragged batch: device [B] keys of each row (clamped to
                              // [0, n_k]), or nullptr: every row has n_k keys
    const int32_t* q_pos_rows;  // ragged batch: device [B] query position of each row
                                // (clamped to [0, 2^31 - 2]), or nullptr: q_pos
    const int32_t* block_table;  // paged caches: device [B][max_pages] page of each row's
                                 // page_tokens-token span (clamped to [0, num_pages)),
                                 // or nullptr: contiguous caches
    int32_t max_pages, num_pages, page_tokens;
    int32_t* ws_plan;         // ragged batch: [B + 1] index of each row's first work item
                              // (written by the split kernel for the merge), else unused
    int32_t splits;           // uniform batch: splits per row; ragged batch: work items the
                              // batch's keys are spread over (a row adds at most one more)
    int32_t split_tokens;     // uniform batch: tokens per split (multiple of the workgroup's
                              // token step); ragged batch: unused (derived on the device)
    float scale_log2;
    WindowTable win;
    // RoPE at read time: q and the K cache hold unrotated vectors; pair r of a vector
    // at position pos is rotated by pos * theta_r, with rho_r = theta_r / (2 pi) mod 1
    // as a 0.64 fixed-point fraction (hi and lo words)
    int32_t rotate;
    int32_t cols16;           // decode_split16_kernel, not decode_split_kernel
    int32_t direct;           // one split per row, which writes the output itself (no merge)
    uint32_t rope_rho_hi[kMaxPairs];
    uint32_t rope_rho_lo[kMaxPairs];
};

// Append of n_new tokens at cache positions pos0 .. (rotate.hip): a NULL k_src or v_src
// leaves that cache alone (the packs).
struct AppendParams {
    const uint16_t* k_src;       // [B][n_new][h_kv][d]
    const uint16_t* v_src;
    uint16_t* k_dst;             // [B][h_kv][d/16][cache_tokens][16], or pages
                                 // [num_pages][h_kv][d/16][page_tokens][16]
    uint16_t* v_dst;             // [B][h_kv][ceil(cache_tokens/16)][d][16], or pages
                                 // [num_pages][h_kv][page_tokens/16][d][16]
    const int32_t* block_table;  // [B][max_pages], or nullptr: contiguous caches
    int32_t batch, n_new, h_kv, pos0;
    int32_t cache_tokens;        // capacity of the contiguous caches
    int32_t zero_tail;           // V: write zeros to the slots of the last block past the source
    int32_t max_pages, num_pages, page_tokens;
};

// With the keys turned on the way in.  A type of its own: 512 bytes more of arguments take 0.3
// us of a launch.
struct AppendRotParams : AppendParams {
    uint32_t rope_rho_hi[kMaxPairs];
    uint32_t rope_rho_lo[kMaxPairs];
};

// One pass of RoPE over a pair-chunk-major K cache (rotate.hip): key t of every (batch,
// kv head) turned to position t, tokens 0 .. n_k - 1.
struct RotateParams {
    const uint16_t* src;   // [B][h_kv][d/16][cache_tokens][16]
    uint16_t* dst;         // same layout; only the tokens named are written
    int32_t batch, n_k, h_kv, cache_tokens;
    uint32_t rope_rho_hi[kMaxPairs];
    uint32_t rope_rho_lo[kMaxPairs];
};

// Kernel launchers (prefill.hip, decode.hip, rotate.hip).  Return the HIP error of the launch.
hipError_t launch_prefill(const PrefillParams& p, int head_dim, hipStream_t stream);
hipError_t launch_prefill_rotating(const PrefillRotParams& p, int head_dim, hipStream_t stream);
// The kernel a prefill takes: 4 or 8 waves per row block of prefill_short_kernel, 0 for
// prefill_kernel, -1 if it is refused (the tests ask).
int32_t prefill_waves(int32_t batch, int32_t n_q, int32_t n_k, int32_t q_pos0, int32_t h_kv, int32_t group,
                      int32_t cache_tokens, const int32_t* thresholds, int32_t head_dim, bool rotate);
hipError_t launch_decode(const DecodeParams& p, int head_dim, hipStream_t stream);
hipError_t launch_append(const AppendRotParams& p, bool turn, int head_dim, hipStream_t stream);
hipError_t launch_rotate_kcache(const RotateParams& p, int head_dim, hipStream_t stream);

// Most splits per (batch, kv head) of a uniform batch, and most work items per column of
// `cols` = kv heads x head subgroups of a ragged one: what the workspace has room for.
int32_t decode_splits(int32_t batch, int32_t h_kv, int64_t n_k);
int32_t decode_ragged_items(int32_t cols);
// The kernel and the numbers a call uses; n_valid bounds a ragged batch's rows.
bool decode_cols16(int32_t batch, int32_t h_q, int32_t h_kv, int32_t head_dim, int64_t n_valid,
                   int64_t cache_tokens, int32_t heads_per_block, bool ragged);
int32_t decode_plan_splits(int32_t batch, int32_t h_q, int32_t h_kv, int64_t n_k, int64_t n_valid,
                           int32_t heads_per_block, bool cols16, bool rotate);
int32_t decode_plan_items(int32_t cols, bool cols16);
// Whether a batch runs without splits (with cols16 only).
bool decode_direct(int32_t batch, int32_t h_q, int32_t h_kv, int32_t head_dim, int64_t n_valid,
                   int32_t heads_per_block, bool rotate, bool ragged);
// Caches from this many tokens are out of the 32-bit lane offsets of decode_split16_kernel
// (they reach over one chunk's stream) and take decode_split_kernel.
constexpr int64_t kDecode16MaxTokens = (int64_t(1) << 27) - 64;
// Tokens handled per decode workgroup iteration (the split granularity).
constexpr int32_t kDecodeTokenStep = 128;
// Largest split count the merge kernel accepts.
constexpr int32_t kDecodeMaxSplits = 4096;
// Query heads one decode workgroup handles at most (columns of its MFMA tiles).
constexpr int32_t kDecodeMaxHeads = 32;
// Size of the library's own decode scratch array (decode.hip), the workspace of
// atf_decode_noalloc; equal to ATF_DECODE_NOALLOC_SCRATCH_BYTES of atf.h.
constexpr size_t kNoAllocScratchBytes = size_t(16) << 20;
// Device address of that array on the current device, resolved once per device
// (hipGetSymbolAddress) and kept for the life of the process.
hipError_t noalloc_scratch(void** out);

}  // namespace atf
