// Host side of libatf.so: argument validation, the window table, the exact
// retained-term count, and dispatch to the gfx950 kernels.  See include/atf.h.
#include "atf.h"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <new>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <string>

#include "atf_internal.hpp"

namespace {

thread_local std::string g_last_error;

int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
int fail(int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return code;
}

constexpr int64_t kPosLimit = 2147483647;  // positions and thresholds are int32 on the device

bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// W_r = floor(w_r), clamped to [0, 2^31 - 1], in fp64.  The default window is
// w_r = k * lambda_r with lambda_r = 2*pi/theta_r (eq:lambda, eq:window); with
// `family` set, w_r = min(max(k_r * lambda_r^gamma + a (r+1)/(d/2), beta), cap)
// (App. A eq:family).  A position-free pair (theta_r == 0) is never pruned.
// Works for any even d <= 2 * max_pairs.
int window_thresholds(const atf_window* w, int32_t* out, int max_pairs) {
    if (w == nullptr || out == nullptr) return fail(ATF_EINVAL, "window: NULL pointer");
    const int d = w->head_dim;
    if (d < 2 || d % 2 != 0 || d / 2 > max_pairs)
        return fail(ATF_EINVAL, "window: head_dim %d must be even, >= 2 and <= %d", d,
                    2 * max_pairs);
    const bool fam = w->family != 0;
    if (fam ? !(w->k >= 0.0) : !(w->k > 0.0))
        return fail(ATF_EINVAL, "window: k must be %s (got %g)", fam ? ">= 0" : "> 0", w->k);
    if (w->inv_freq == nullptr && !(w->rope_base > 1.0 && std::isfinite(w->rope_base)))
        return fail(ATF_EINVAL, "window: rope_base must be finite and > 1 (got %g)",
                    w->rope_base);
    if (fam) {
        if (!std::isfinite(w->gamma))
            return fail(ATF_EINVAL, "window: gamma must be finite (got %g)", w->gamma);
        if (!(w->a >= 0.0) || !std::isfinite(w->a))
            return fail(ATF_EINVAL, "window: a must be finite and >= 0 (got %g)", w->a);
        if (!(w->beta >= 0.0) || !std::isfinite(w->beta))
            return fail(ATF_EINVAL, "window: beta must be finite and >= 0 (got %g)", w->beta);
        if (!(w->cap >= 0.0))
            return fail(ATF_EINVAL, "window: cap must be >= 0 (got %g)", w->cap);
    }
    const double two_pi = 6.283185307179586476925286766559;
    for (int r = 0; r < d / 2; ++r) {
        double theta;
        if (w->inv_freq) {
            theta = w->inv_freq[r];
            if (!(theta >= 0.0) || std::isinf(theta))
                return fail(ATF_EINVAL, "window: inv_freq[%d] = %g must be finite and >= 0", r,
                            theta);
        } else {
            theta = std::pow(w->rope_base, -2.0 * r / d);
        }
        double width;
        if (theta == 0.0) {
            width = HUGE_VAL;  // no wavelength: every distance keeps the pair
        } else if (!fam) {
            width = w->k * (two_pi / theta);
        } else {
            const double kr = w->k_profile ? w->k_profile[r] : w->k;
            if (!(kr >= 0.0))
                return fail(ATF_EINVAL, "window: k_profile[%d] = %g must be >= 0", r, kr);
            width = kr * std::pow(two_pi / theta, w->gamma) + w->a * (r + 1) / (d / 2);
            if (std::isnan(width))
                return fail(ATF_EINVAL, "window: the width of pair %d is undefined (0 * inf)", r);
            width = std::fmin(std::fmax(width, w->beta), w->cap);
        }
        double t = std::floor(width);
        if (!(t < static_cast<double>(kPosLimit))) t = static_cast<double>(kPosLimit);
        if (t < 0.0) t = 0.0;
        out[r] = static_cast<int32_t>(t);
    }
    // Rounded slice (Sec. 3.3): at distance z the window keeps the suffix r >= rf(z)
    // of a non-decreasing table; rounding its length up to whole s-pair steps counted
    // from r = h - 1 keeps pair r iff the top pair of r's step is kept.
    const int h = d / 2, sp = w->slice_pairs;
    if (sp < 0 || sp > h)
        return fail(ATF_EINVAL, "window: slice_pairs %d must be in [0, d/2 = %d]", sp, h);
    if (sp > 1) {
        for (int r = 1; r < h; ++r)
            if (out[r] < out[r - 1])
                return fail(ATF_EINVAL,
                            "window: the rounded slice needs a table non-decreasing in r "
                            "(W[%d] = %d < W[%d] = %d)", r, out[r], r - 1, out[r - 1]);
        for (int r = 0; r < h; ++r) out[r] = out[h - 1 - sp * ((h - 1 - r) / sp)];
    }
    return ATF_OK;
}

int build_table(const atf_window* w, atf::WindowTable* t) {
    std::memset(t, 0, sizeof *t);
    int rc = window_thresholds(w, t->W, atf::kMaxPairs);
    if (rc != ATF_OK) return rc;
    const int pairs = w->head_dim / 2;
    for (int c = 0; c * atf::kChunkPairs < pairs; ++c) {
        int32_t lo = INT32_MAX, hi = 0;
        for (int e = 0; e < atf::kChunkPairs; ++e) {
            const int32_t x = t->W[c * atf::kChunkPairs + e];
            lo = x < lo ? x : lo;
            hi = x > hi ? x : hi;
        }
        t->chunk_min[c] = lo;
        t->chunk_max[c] = hi;
    }
    return ATF_OK;
}

using u128 = unsigned __int128;

// sum_{p=a}^{c} (p + 1), 0 <= a <= c
u128 sum_p_plus_1(int64_t a, int64_t c) {
    if (c < a) return 0;
    const u128 n = static_cast<u128>(c - a + 1);
    return n * static_cast<u128>(a + c + 2) / 2;
}

// Kept keys of one pair with threshold W, summed over rows p in [p0, p1]:
// per row, keys j in [max(0, p - W), min(p, n_k - 1)].
u128 pair_count(int64_t W, int64_t p0, int64_t p1, int64_t n_k) {
    u128 total = 0;
    // rows with p <= n_k - 1: min(p, W) + 1 keys
    {
        const int64_t a = p0, b = p1 < n_k - 1 ? p1 : n_k - 1;
        if (a <= b) {
            const int64_t c = b < W ? b : W;        // rows where p <= W: p + 1 keys
            total += sum_p_plus_1(a, c);
            const int64_t s = a > W + 1 ? a : W + 1;  // rows where p > W: W + 1 keys
            if (s <= b) total += static_cast<u128>(b - s + 1) * static_cast<u128>(W + 1);
        }
    }
    // rows with p >= n_k: n_k keys while p <= W, then n_k + W - p until it hits 0
    {
        const int64_t a = p0 > n_k ? p0 : n_k, b = p1;
        if (a <= b) {
            const int64_t c = b < W ? b : W;
            if (a <= c) total += static_cast<u128>(c - a + 1) * static_cast<u128>(n_k);
            const int64_t x = a > W + 1 ? a : W + 1;
            const int64_t y = b < n_k + W - 1 ? b : n_k + W - 1;
            if (x <= y) {
                const u128 n = static_cast<u128>(y - x + 1);
                total += n * static_cast<u128>(n_k + W) - n * static_cast<u128>(x + y) / 2;
            }
        }
    }
    return total;
}

}  // namespace

namespace atf {

int32_t decode_splits(int32_t batch, int32_t h_kv, int64_t n_k) {
    const int64_t target_groups = 1024;
    int64_t s = (target_groups + int64_t(batch) * h_kv - 1) / (int64_t(batch) * h_kv);
    const int64_t max_s = (n_k + kDecodeTokenStep - 1) / kDecodeTokenStep;
    if (s > max_s) s = max_s;
    if (s > kDecodeMaxSplits) s = kDecodeMaxSplits;
    if (s < 1) s = 1;
    return static_cast<int32_t>(s);
}

int32_t decode_ragged_items(int32_t cols) {
    const int64_t target_groups = 2048;
    int64_t s = (target_groups + cols - 1) / cols;
    if (s > kDecodeMaxSplits - 1) s = kDecodeMaxSplits - 1;
    if (s < 1) s = 1;
    return static_cast<int32_t>(s);
}

namespace {
// rounds of the chip's CUs that a number of equal workgroups takes
constexpr int64_t kDecodeCUs = 256;
int64_t decode_rounds(int64_t groups) { return (groups + kDecodeCUs - 1) / kDecodeCUs; }

// Whether workgroups that share a KV head (35, 39 or 49 heads to one: 5 of 7, 3 of 13, 7 of 7)
// find its keys in the caches wherever on the chip they run: caches of up to 1 GB over their
// number, or 128 MB, beside a last-level cache of 256 MB.  Below it the unsplit 16-column kernel takes 0.2 to
// 1.2 of the time of the split 32-column one (median 0.8 next to it), above it 0.7 to 2.2 (1.0
// next to it; 3,600 calls).
bool decode_shared_fits(int32_t batch, int32_t h_kv, int32_t head_dim, int64_t n_valid, int32_t workgroups) {
    return int64_t(batch) * h_kv * n_valid <= (int64_t(1) << 30) / (4 * head_dim * std::min(workgroups, 8));
}
}  // namespace

// Whether a call's workgroups take decode_split16_kernel: up to 16 heads each, and caches within
// its lane offsets (they reach over one chunk's stream).
//
// Not where several workgroups share a KV head and the batch's caches are large
// (decode_shared_fits): more workgroups are then in flight at places further apart, and keys
// that one has read have left the caches when the next one of the same KV head comes
// (decode_split_kernel -> split16: 146 rows of 86,558 keys, 70/2 heads 3385 -> 4813 us, 270 rows of
// 40,029, 39/1 1607 -> 1879; but 54 rows of 1,255, 70/2 152 -> 75).  A ragged batch's caches are
// not known here, only a bound that is far from them where one row is long (496 rows of 1,905
// keys in all, 99/3 heads, 216 -> 33); large ones lose up to 8 %.
bool decode_cols16(int32_t batch, int32_t h_q, int32_t h_kv, int32_t head_dim, int64_t n_valid,
                   int64_t cache_tokens, int32_t heads_per_block, bool ragged) {
    if (heads_per_block > 16 || cache_tokens >= kDecode16MaxTokens) return false;
    const int32_t workgroups = h_q / h_kv / heads_per_block;
    return ragged || workgroups == 1 || decode_shared_fits(batch, h_kv, head_dim, n_valid, workgroups);
}

// Splits a uniform batch uses, at most the decode_splits() its workspace has room for.
//
// Where several workgroups share a KV head (64 heads to one: two of 32), a multiple of 8 where
// one is near: the workgroups that read the same keys are that many apart, and so on the same
// XCD (16 rows of 123,544 keys, 64/1 heads: 61 splits 235 us, 64, 3 of them empty, 201; but 10
// rows of 14,730, rotating, 58 splits 66 us, 103 with 45 empty 80).
//
// Up to 16 heads per workgroup: as many workgroups as the CUs hold at once, 3 of
// decode_split16_kernel (768) or 2 where it rotates keys (512, at d = 128; its tables are
// made anew by every workgroup), so that the batch runs in one round of equal splits:
// 2^20 keys, 28/4 heads 283 us with 1024, 273 with 768; batch 8 at 32,768 keys, 24/8 heads
// 156 -> 153; rotating, batch 2 at 100,003 keys 65.9 -> 63.5, batch 8 at 8,200 36.1 -> 30.7
// (512; 31.6 with 768).  From 256 (row, KV head) pairs on: the splits that leave the fewest
// rounds of 256, counted in whole rows (decode_direct).  More heads: 1024, two rounds of the
// 2 workgroups per CU of decode_split_kernel (2048 is 6 % slower at 2^20 keys).  The steps
// are then spread evenly: 65 steps over 12 splits are 11 splits, ten of 6 and one of 5, not
// 10 of 6, one of 5 and an empty one.
int32_t decode_plan_splits(int32_t batch, int32_t h_q, int32_t h_kv, int64_t n_k, int64_t n_valid,
                           int32_t heads_per_block, bool cols16, bool rotate) {
    const int64_t room = decode_splits(batch, h_kv, n_k);
    const int64_t cols = int64_t(batch) * (h_q / heads_per_block);
    const int64_t target = rotate ? 512 : 768;
    const int64_t steps = (n_valid + kDecodeTokenStep - 1) / kDecodeTokenStep;
    const bool shared = h_q / h_kv != heads_per_block;
    int64_t s = 1;
    if (!cols16) {
        s = room;
    } else if (cols < kDecodeCUs) {
        s = std::min(room, std::max<int64_t>(1, target / cols));
    } else {
        for (int64_t t = 2; t <= std::min<int64_t>(room, 4); ++t)
            if (decode_rounds(t * cols) * s < decode_rounds(s * cols) * t) s = t;
    }
    s = std::max<int64_t>(1, std::min(s, steps));
    const int64_t per = (steps + s - 1) / s;
    s = std::max<int64_t>(1, (steps + per - 1) / per);
    const int64_t up = (s + 7) / 8 * 8;
    return static_cast<int32_t>(shared && up <= room && 16 * (up - s) <= s ? up : s);
}

// Whether a batch takes one workgroup of 8 waves per (row, KV head), which writes the
// output itself, and no merge.
//
// With 256 such workgroups every CU has one, and splitting only adds the partial states' way
// through memory and the merge (us, split -> direct): 32 rows of 500 keys, 24/8 heads
// 19.8 -> 14.0, of 16,000 306 -> 295; rotating 23.9 -> 18.3, and 173 -> 155 at 8,000.
// Just past a whole round of the CUs some of them take a row more while the others wait, and a
// split plan has smaller pieces to deal out: 24/8 heads, 16,000 keys, 33 rows 310 -> 382, 40
// rows 351 -> 398, 48 rows 409 -> 405, 52 rows 448 -> 423, 66 rows 615 -> 654, 76 rows
// 643 -> 646; 98 rows of 60,000 keys 3018 -> 3145; rotating, 16,000 keys, 33 rows 342 -> 440, 42 rows 385 -> 452, 66
// rows 686 -> 713; d = 64, 16/16 heads, 17 rows 174 -> 213, rotating 184 -> 257, 24 rows
// 241 -> 265, 40 rows 380 -> 401.  So they are split in a second to fourth round of up to 128
// workgroups (from 1,025 pairs on the workspace has room for one split only), if a row is long
// enough to pay for the merge, which grows with its heads, out of what the round leaves idle,
// which falls with the round's workgroups and with the rounds before it: the limit is a fit
// to 1,400 measured calls of 257 to 1,023 pairs, 1 to 16 heads and 300 to 60,000 keys.  264
// pairs of 3 heads, 1,000 keys 33.2 -> 34.7, 2,000 53.4 -> 60.8; of 7, 2,000 59.4 -> 60.1, 8,000
// 179 -> 204; of 16, 4,000 112 -> 110, 8,000 193 -> 206; 528 pairs of 7 heads without a window,
// 8,000 keys 404 -> 415, 60,000 2800 -> 3017.
// Workgroups that share a KV head run unsplit too: their caches are small (decode_cols16; 270
// rows of 40,029 keys, 39/1 heads, would take 2926 for 1615, but 295 rows of 893, rotating,
// 172 -> 75).
// Rotating at d = 64, a CU holds 8 waves of the unsplit kernel and 12 of the split one: with 1
// or 2 heads, whose merge costs least, the latter wins from 1,025 pairs on (2,112 pairs of 1
// head, 300 keys 50 -> 62, 4,000 353 -> 378, 16,000 1242 -> 1261; of 2, 1,000 keys 110 -> 118,
// but 1,056 pairs 66.1 -> 65.6; of 7, 137 -> 120).
//
// With 128 to 255 they win while a row is short: d = 128 39.3 -> 33.8 at 3,840 keys,
// 62.3 -> 68.9 at 5,000 without a window; d = 64 39.5 -> 34.1 at 7,680, 60.4 -> 66.8 at 10,000;
// rotating d = 128 18.8 -> 18.7 at 768, 21.2 -> 21.4 at 1,024, d = 64 14.2 -> 14.0 at 1,024,
// 17.2 -> 18.2 at 1,500.  With fewer they win while a row costs less than the second launch:
// d = 128 12.3 -> 11.5 at 1,280, 12.4 -> 12.3 at 1,600; d = 64 13.4 -> 10.8 at 2,048,
// 13.2 -> 11.2 at 2,560, 13.6 -> 13.7 at 3,000; rotating d = 128 12.1 -> 10.5 at 256,
// 12.0 -> 13.6 at 512, d = 64 13.5 -> 11.8 at 768, 13.3 -> 13.4 at 1,000.
//
// Of a ragged batch only the longest row's bound is known here, and one long row among short
// ones is then one workgroup's work: below 1,024 workgroups the limit is the last of these (8
// to 128 rows up to 300 keys, 24/8 heads 15.2..42.5 -> 11.2..23.1; up to 1,280 14.9 -> 12.4; 64
// rows of d = 64 up to 3,840 18.3 -> 22.0).  From 1,024 the plan and merge of all rows cost
// more than a long row does: 128 rows up to 1,920 73.9 -> 60.3 (but one row of 3,840 keys
// among 127 of one key 39.7 -> 46.2); 512 rows of d = 64 up to 300 keys 54.2 -> 12.1, up to
// 7,680 148.9 -> 131.0, one row of 7,680 among rows of one key 55.5 -> 28.6.
bool decode_direct(int32_t batch, int32_t h_q, int32_t h_kv, int32_t head_dim, int64_t n_valid,
                   int32_t heads_per_block, bool rotate, bool ragged) {
    const int64_t cols = int64_t(batch) * (h_q / heads_per_block);
    if (!ragged && cols >= kDecodeCUs) {
        if (h_q / h_kv != heads_per_block) return true;
        const int64_t rounds = decode_rounds(cols), last = cols - (rounds - 1) * kDecodeCUs;
        if (rounds > 4) return !(rotate && head_dim == 64 && heads_per_block <= 2);
        if (rounds == 1 || last > 128) return true;
        const double keys = (rotate ? 128 : head_dim == 64 ? 512 : 256) * (rounds == 2 ? 1 : 4);
        return n_valid < std::max(!rotate && head_dim == 64 ? 2048.0 : 1024.0,
                                  keys * heads_per_block * std::exp2(double(last) / 48));
    }
    if (cols >= (ragged ? 1024 : 128))
        return n_valid <= (rotate ? (head_dim == 64 ? 1024 : 768)
                                  : head_dim == 64 ? 7680 : ragged ? 2560 : 3840);
    return n_valid <= (rotate ? (head_dim == 64 ? 768 : 256) : (head_dim == 64 ? 2560 : 1280));
}

// Work items the keys of a ragged batch are spread over, at most the decode_ragged_items()
// its workspace has room for.  1536 workgroups, two rounds of decode_split16_kernel's 768
// (rows differ, so one round leaves the CUs of the short ones idle: 768 takes 1.08 times as
// long on 8 rows of 6K to 120K keys of 24/8 heads), against 2048: 8 rows up to 120K keys
// 219 -> 214 us (24/8 heads), 124 -> 120 (28/4); 4 rows up to 60K 65 -> 63, 38 -> 36; 24
// rows up to 30K 159 -> 161, 94 -> 92.  decode_split_kernel keeps 2048 (5-12 % faster than
// 1024, up to 20 % than 4096).
int32_t decode_plan_items(int32_t cols, bool cols16) {
    const int32_t room = decode_ragged_items(cols);
    return cols16 ? std::min(room, std::max(1, 1536 / cols)) : room;
}

}  // namespace atf

extern "C" {

const char* atf_last_error(void) { return g_last_error.c_str(); }

int atf_window_table(const atf_window* w, int32_t* W_out) {
    return window_thresholds(w, W_out, 1 << 20);
}

int atf_retention_profile(int32_t head_dim, int32_t kind, double k_hi, double k_lo,
                          double* k_out) {
    if (k_out == nullptr) return fail(ATF_EINVAL, "retention_profile: NULL output");
    if (head_dim < 2 || head_dim % 2 != 0)
        return fail(ATF_EINVAL, "retention_profile: head_dim %d must be even and >= 2", head_dim);
    if (!(k_hi >= 0.0) || !std::isfinite(k_hi) || !(k_lo >= 0.0) || !std::isfinite(k_lo))
        return fail(ATF_EINVAL, "retention_profile: k_hi, k_lo must be finite and >= 0");
    const int n = head_dim / 2;
    const double span = n > 1 ? double(n - 1) : 1.0;
    switch (kind) {
        case ATF_PROFILE_CONSTANT:
            for (int r = 0; r < n; ++r) k_out[r] = k_hi;
            return ATF_OK;
        case ATF_PROFILE_ARITHMETIC: {
            const double step = (k_hi - k_lo) / span;
            for (int r = 0; r < n; ++r) k_out[r] = k_hi - step * r;
            if (n > 1) k_out[n - 1] = k_lo;
            return ATF_OK;
        }
        case ATF_PROFILE_GEOMETRIC: {
            if (!(k_hi > 0.0) || !(k_lo > 0.0))
                return fail(ATF_EINVAL, "retention_profile: geometric needs k_hi, k_lo > 0");
            const double lr = std::log(k_lo / k_hi) / span;
            for (int r = 0; r < n; ++r) k_out[r] = k_hi * std::exp(lr * r);
            if (n > 1) k_out[n - 1] = k_lo;
            return ATF_OK;
        }
        default:
            return fail(ATF_EINVAL, "retention_profile: unknown kind %d", kind);
    }
}

int atf_count_terms(const atf_window* w, int64_t n_q, int64_t q_pos0, int64_t n_k,
                    uint64_t* retained, uint64_t* causal_cells) {
    if (retained == nullptr || causal_cells == nullptr)
        return fail(ATF_EINVAL, "count_terms: NULL output");
    if (n_q < 0 || q_pos0 < 0 || n_k < 0)
        return fail(ATF_EINVAL, "count_terms: n_q, q_pos0 and n_k must be >= 0");
    if (q_pos0 > INT64_MAX / 4 - n_q || n_k > INT64_MAX / 4)
        return fail(ATF_EINVAL, "count_terms: sizes too large");
    if (w == nullptr) return fail(ATF_EINVAL, "count_terms: NULL window");
    const int pairs = w->head_dim / 2;
    if (w->head_dim < 2 || w->head_dim % 2 || pairs > (1 << 20))
        return fail(ATF_EINVAL, "count_terms: bad head_dim %d", w->head_dim);
    int32_t* W = new (std::nothrow) int32_t[pairs];
    if (!W) return fail(ATF_EINVAL, "count_terms: out of host memory");
    int rc = window_thresholds(w, W, pairs);
    if (rc != ATF_OK) {
        delete[] W;
        return rc;
    }
    u128 ret = 0, cau = 0;
    if (n_q > 0 && n_k > 0) {
        const int64_t p0 = q_pos0, p1 = q_pos0 + n_q - 1;
        for (int r = 0; r < pairs; ++r) ret += pair_count(W[r], p0, p1, n_k);
        cau = pair_count(INT64_MAX / 8, p0, p1, n_k);  // every key kept
    }
    delete[] W;
    if (ret > static_cast<u128>(UINT64_MAX) || cau > static_cast<u128>(UINT64_MAX))
        return fail(ATF_EINVAL, "count_terms: count exceeds 64 bits");
    *retained = static_cast<uint64_t>(ret);
    *causal_cells = static_cast<uint64_t>(cau);
    return ATF_OK;
}

int32_t atf_kcache_chunk_pairs(int32_t head_dim) {
    return (head_dim == 64 || head_dim == 128) ? atf::kChunkPairs : 0;
}

namespace {

// RoPE at read time (q and the K cache unrotated): theta_r = rope_inv_freq[r] if given,
// else the window's frequencies (its inv_freq, or rope_base^(-2r/d)).
struct RopeArgs {
    bool rotate = false;
    const double* inv_freq = nullptr;
};

// rho_r = theta_r / (2 pi) mod 1 as a 0.64 fixed-point fraction, in extended precision
int rope_fractions(const char* fn, const atf_window* w, const double* inv_freq,
                   uint32_t* rho_hi, uint32_t* rho_lo) {
    const int d = w->head_dim;
    const long double two_pi = 6.283185307179586476925286766559L;
    for (int r = 0; r < d / 2; ++r) {
        double th;
        if (inv_freq != nullptr)
            th = inv_freq[r];
        else if (w->inv_freq != nullptr)
            th = w->inv_freq[r];
        else
            th = std::pow(w->rope_base, -2.0 * r / d);
        if (!(th >= 0.0) || std::isinf(th))
            return fail(ATF_EINVAL, "%s: rotation frequency %d = %g must be finite and >= 0", fn, r,
                        th);
        long double f = static_cast<long double>(th) / two_pi;
        if (f >= 1.0L) f -= std::floor(f);
        const long double scaled = f * 18446744073709551616.0L;  // 2^64: exact
        uint64_t fx = scaled >= 18446744073709551615.0L ? UINT64_MAX : static_cast<uint64_t>(scaled);
        rho_hi[r] = static_cast<uint32_t>(fx >> 32);
        rho_lo[r] = static_cast<uint32_t>(fx);
    }
    return ATF_OK;
}

// Shared by atf_prefill (pre-rotated caches) and atf_prefill_unrotated (RoPE applied
// to q and each kept key pair as the kernel reads them).
int prefill_impl(const char* fn, const void* q, const void* k, const void* v, void* o, float* lse,
                 int32_t batch, int64_t n_q, int64_t n_k, int64_t q_pos0, int32_t h_q,
                 int32_t h_kv, int64_t cache_tokens, const atf_window* w, float softmax_scale,
                 void* hip_stream, const RopeArgs& rope) {
    if (w == nullptr) return fail(ATF_EINVAL, "%s: NULL window", fn);
    const int d = w->head_dim;
    if (d != 64 && d != 128)
        return fail(ATF_EUNSUPPORTED, "%s: head_dim %d not built (64 or 128)", fn, d);
    if (batch < 1 || n_q < 0 || n_k < 1 || q_pos0 < 0 || h_q < 1 || h_kv < 1)
        return fail(ATF_EINVAL,
                    "%s: need batch >= 1, n_q >= 0, n_k >= 1, q_pos0 >= 0, heads >= 1", fn);
    if (h_q % h_kv != 0)
        return fail(ATF_EINVAL, "%s: h_q %d not a multiple of h_kv %d", fn, h_q, h_kv);
    const int max_group = d == 64 ? 128 : 256;  // query rows of one prefill workgroup
    if (h_q / h_kv > max_group)
        return fail(ATF_EUNSUPPORTED, "%s: GQA ratio %d above %d not built for d = %d", fn,
                    h_q / h_kv, max_group, d);
    if (q_pos0 + n_q > kPosLimit || n_k > kPosLimit)
        return fail(ATF_EINVAL, "%s: positions must stay below 2^31 - 1", fn);
    if (cache_tokens == 0) cache_tokens = n_k;
    if (cache_tokens < n_k || cache_tokens > kPosLimit)
        return fail(ATF_EINVAL, "%s: cache_tokens %lld must be >= n_k %lld and < 2^31 - 1", fn,
                    (long long)cache_tokens, (long long)n_k);
    if (!std::isfinite(softmax_scale))
        return fail(ATF_EINVAL, "%s: softmax_scale must be finite", fn);
    atf::PrefillRotParams p{};
    int rc = build_table(w, &p.win);
    if (rc != ATF_OK) return rc;
    if (rope.rotate) {
        rc = rope_fractions(fn, w, rope.inv_freq, p.rope_rho_hi, p.rope_rho_lo);
        if (rc != ATF_OK) return rc;
    }
    if (n_q == 0) return ATF_OK;
    if (!q || !k || !v || !o || !lse) return fail(ATF_EINVAL, "%s: NULL tensor pointer", fn);
    if (!aligned(q, 16) || !aligned(k, 16) || !aligned(v, 16) || !aligned(o, 16) ||
        !aligned(lse, 4))
        return fail(ATF_EINVAL, "%s: q/k/v/o must be 16-byte and lse 4-byte aligned", fn);
    const float scale = softmax_scale > 0.f ? softmax_scale : 1.0f / std::sqrt(float(d));
    p.q = static_cast<const uint16_t*>(q);
    p.k = static_cast<const uint16_t*>(k);
    p.v = static_cast<const uint16_t*>(v);
    p.o = static_cast<uint16_t*>(o);
    p.lse = lse;
    p.batch = batch;
    p.n_q = static_cast<int32_t>(n_q);
    p.n_k = static_cast<int32_t>(n_k);
    p.cache_tokens = static_cast<int32_t>(cache_tokens);
    p.q_pos0 = static_cast<int32_t>(q_pos0);
    p.h_q = h_q;
    p.h_kv = h_kv;
    p.group = h_q / h_kv;
    p.scale_log2 = scale * 1.4426950408889634f;
    const hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const hipError_t e = rope.rotate ? atf::launch_prefill_rotating(p, d, st)
                                     : atf::launch_prefill(p, d, st);
    if (e != hipSuccess) return fail(ATF_EHIP, "%s: launch failed: %s", fn, hipGetErrorString(e));
    return ATF_OK;
}

}  // namespace

int atf_prefill(const void* q, const void* k, const void* v, void* o, float* lse,
                int32_t batch, int64_t n_q, int64_t n_k, int64_t q_pos0, int32_t h_q,
                int32_t h_kv, int64_t cache_tokens, const atf_window* w, float softmax_scale,
                void* hip_stream) {
    return prefill_impl("prefill", q, k, v, o, lse, batch, n_q, n_k, q_pos0, h_q, h_kv,
                        cache_tokens, w, softmax_scale, hip_stream, RopeArgs());
}

int atf_prefill_unrotated(const void* q, const void* k, const void* v, void* o, float* lse,
                          int32_t batch, int64_t n_q, int64_t n_k, int64_t q_pos0, int32_t h_q,
                          int32_t h_kv, int64_t cache_tokens, const atf_window* w,
                          const double* rope_inv_freq, float softmax_scale, void* hip_stream) {
    RopeArgs rope;
    rope.rotate = true;
    rope.inv_freq = rope_inv_freq;
    return prefill_impl("prefill_unrotated", q, k, v, o, lse, batch, n_q, n_k, q_pos0, h_q, h_kv,
                        cache_tokens, w, softmax_scale, hip_stream, rope);
}


namespace {
int check_pack(const char* what, const void* src, void* dst, int32_t batch, int64_t n_k,
               int32_t h_kv, int32_t head_dim, size_t dst_bytes) {
    if (head_dim != 64 && head_dim != 128)
        return fail(ATF_EUNSUPPORTED, "%s: head_dim %d not built", what, head_dim);
    if (batch < 1 || n_k < 1 || h_kv < 1 || n_k > kPosLimit)
        return fail(ATF_EINVAL, "%s: need batch >= 1, 1 <= n_k < 2^31, h_kv >= 1", what);
    if (!src || !dst) return fail(ATF_EINVAL, "%s: NULL pointer", what);
    if (!aligned(src, 16) || !aligned(dst, 16))
        return fail(ATF_EINVAL, "%s: pointers must be 16-byte aligned", what);
    const size_t src_bytes = size_t(batch) * size_t(n_k) * size_t(h_kv) * size_t(head_dim) * 2;
    const char* a = static_cast<const char*>(src);
    const char* b = static_cast<const char*>(dst);
    if (a < b + dst_bytes && b < a + src_bytes)
        return fail(ATF_EINVAL, "%s: buffers overlap", what);
    return ATF_OK;
}

size_t vcache_bytes(int32_t batch, int64_t n_k, int32_t h_kv, int32_t head_dim) {
    return size_t(batch) * size_t(h_kv) * size_t((n_k + 15) / 16) * 16 * size_t(head_dim) * 2;
}
}  // namespace

int atf_pack_kcache(const void* k_bshd, void* k_pcm, int32_t batch, int64_t n_k, int32_t h_kv,
                    int32_t head_dim, void* hip_stream) {
    const size_t bytes = size_t(batch) * size_t(n_k) * size_t(h_kv) * size_t(head_dim) * 2;
    int rc = check_pack("pack_kcache", k_bshd, k_pcm, batch, n_k, h_kv, head_dim, bytes);
    if (rc != ATF_OK) return rc;
    atf::AppendRotParams p{};
    p.k_src = static_cast<const uint16_t*>(k_bshd);
    p.k_dst = static_cast<uint16_t*>(k_pcm);
    p.batch = batch;
    p.n_new = p.cache_tokens = static_cast<int32_t>(n_k);
    p.h_kv = h_kv;
    hipError_t e = atf::launch_append(p, false, head_dim, static_cast<hipStream_t>(hip_stream));
    if (e != hipSuccess) return fail(ATF_EHIP, "pack_kcache: launch failed: %s", hipGetErrorString(e));
    return ATF_OK;
}

int atf_rotate_kcache(const void* k_pcm, void* k_rot, int32_t batch, int64_t n_k, int32_t h_kv,
                      int64_t cache_tokens, const atf_window* w, const double* rope_inv_freq,
                      void* hip_stream) {
    const char* fn = "rotate_kcache";
    if (w == nullptr) return fail(ATF_EINVAL, "%s: NULL window", fn);
    const int d = w->head_dim;
    if (d != 64 && d != 128)
        return fail(ATF_EUNSUPPORTED, "%s: head_dim %d not built (64 or 128)", fn, d);
    if (batch < 1 || n_k < 1 || h_kv < 1 || n_k > kPosLimit)
        return fail(ATF_EINVAL, "%s: need batch >= 1, 1 <= n_k < 2^31, h_kv >= 1", fn);
    if (cache_tokens == 0) cache_tokens = n_k;
    if (cache_tokens < n_k || cache_tokens > kPosLimit)
        return fail(ATF_EINVAL, "%s: cache_tokens %lld must be >= n_k %lld and < 2^31 - 1", fn,
                    (long long)cache_tokens, (long long)n_k);
    if (int64_t(batch) * h_kv * (d / 16) > 65535)
        return fail(ATF_EUNSUPPORTED, "%s: batch * h_kv * d/16 above 65535", fn);
    atf::RotateParams p{};
    int rc = rope_fractions(fn, w, rope_inv_freq, p.rope_rho_hi, p.rope_rho_lo);
    if (rc != ATF_OK) return rc;
    if (!k_pcm || !k_rot) return fail(ATF_EINVAL, "%s: NULL pointer", fn);
    if (!aligned(k_pcm, 16) || !aligned(k_rot, 16))
        return fail(ATF_EINVAL, "%s: pointers must be 16-byte aligned", fn);
    const size_t bytes = size_t(batch) * size_t(h_kv) * size_t(d) * size_t(cache_tokens) * 2;
    const char* a = static_cast<const char*>(k_pcm);
    const char* b = static_cast<const char*>(k_rot);
    // in place (the same buffer) is allowed: each thread reads a record, then writes it
    if (a != b && a < b + bytes && b < a + bytes)
        return fail(ATF_EINVAL, "%s: buffers overlap", fn);
    p.src = static_cast<const uint16_t*>(k_pcm);
    p.dst = static_cast<uint16_t*>(k_rot);
    p.batch = batch;
    p.n_k = static_cast<int32_t>(n_k);
    p.h_kv = h_kv;
    p.cache_tokens = static_cast<int32_t>(cache_tokens);
    const hipError_t e = atf::launch_rotate_kcache(p, d, static_cast<hipStream_t>(hip_stream));
    if (e != hipSuccess) return fail(ATF_EHIP, "%s: launch failed: %s", fn, hipGetErrorString(e));
    return ATF_OK;
}

size_t atf_vcache_bytes(int32_t batch, int64_t n_k, int32_t h_kv, int32_t head_dim) {
    if (batch < 1 || n_k < 1 || h_kv < 1 || n_k > kPosLimit || (head_dim != 64 && head_dim != 128))
        return 0;
    return vcache_bytes(batch, n_k, h_kv, head_dim);
}

int atf_pack_vcache(const void* v_bshd, void* v_pack, int32_t batch, int64_t n_k, int32_t h_kv,
                    int32_t head_dim, void* hip_stream) {
    int rc = check_pack("pack_vcache", v_bshd, v_pack, batch, n_k, h_kv, head_dim,
                        (batch >= 1 && n_k >= 1 && h_kv >= 1 && n_k <= kPosLimit)
                            ? vcache_bytes(batch, n_k, h_kv, head_dim) : 0);
    if (rc != ATF_OK) return rc;
    atf::AppendRotParams p{};
    p.v_src = static_cast<const uint16_t*>(v_bshd);
    p.v_dst = static_cast<uint16_t*>(v_pack);
    p.batch = batch;
    p.n_new = p.cache_tokens = static_cast<int32_t>(n_k);
    p.h_kv = h_kv;
    p.zero_tail = 1;
    hipError_t e = atf::launch_append(p, false, head_dim, static_cast<hipStream_t>(hip_stream));
    if (e != hipSuccess) return fail(ATF_EHIP, "pack_vcache: launch failed: %s", hipGetErrorString(e));
    return ATF_OK;
}

namespace {
// Shared by atf_cache_append (keys stored as given) and atf_cache_append_rotated (keys
// turned to their cache positions on the way in: rope != nullptr).
int cache_append_impl(const char* fn, const void* k_new, const void* v_new, void* k_cache,
                      void* v_cache, int32_t batch, int64_t n_new, int64_t pos0, int32_t h_kv,
                      int32_t head_dim, int64_t cache_tokens, void* hip_stream,
                      const atf::AppendRotParams* rope) {
    if (head_dim != 64 && head_dim != 128)
        return fail(ATF_EUNSUPPORTED, "%s: head_dim %d not built", fn, head_dim);
    if (batch < 1 || h_kv < 1 || n_new < 0 || pos0 < 0 || cache_tokens < 1 ||
        cache_tokens > kPosLimit || pos0 > cache_tokens - n_new)
        return fail(ATF_EINVAL,
                    "%s: need batch >= 1, h_kv >= 1, n_new >= 0, pos0 >= 0, "
                    "1 <= cache_tokens < 2^31 and pos0 + n_new <= cache_tokens", fn);
    if (!k_new || !v_new || !k_cache || !v_cache)
        return fail(ATF_EINVAL, "%s: NULL pointer", fn);
    if (!aligned(k_new, 16) || !aligned(v_new, 16) || !aligned(k_cache, 16) || !aligned(v_cache, 16))
        return fail(ATF_EINVAL, "%s: pointers must be 16-byte aligned", fn);
    const size_t row = size_t(h_kv) * size_t(head_dim) * 2;
    const char* bufs[4] = {static_cast<const char*>(k_new), static_cast<const char*>(v_new),
                           static_cast<const char*>(k_cache), static_cast<const char*>(v_cache)};
    const size_t sizes[4] = {size_t(batch) * size_t(n_new) * row, size_t(batch) * size_t(n_new) * row,
                             size_t(batch) * size_t(cache_tokens) * row,
                             vcache_bytes(batch, cache_tokens, h_kv, head_dim)};
    for (int i = 0; i < 4; ++i)
        for (int j = (i < 2 ? 2 : i + 1); j < 4; ++j)  // written buffers against all others
            if (bufs[i] < bufs[j] + sizes[j] && bufs[j] < bufs[i] + sizes[i])
                return fail(ATF_EINVAL, "%s: buffers overlap", fn);
    if (n_new == 0) return ATF_OK;
    atf::AppendRotParams p = rope != nullptr ? *rope : atf::AppendRotParams{};
    p.k_src = static_cast<const uint16_t*>(k_new);
    p.v_src = static_cast<const uint16_t*>(v_new);
    p.k_dst = static_cast<uint16_t*>(k_cache);
    p.v_dst = static_cast<uint16_t*>(v_cache);
    p.batch = batch;
    p.n_new = static_cast<int32_t>(n_new);
    p.h_kv = h_kv;
    p.pos0 = static_cast<int32_t>(pos0);
    p.cache_tokens = static_cast<int32_t>(cache_tokens);
    const hipError_t e = atf::launch_append(p, rope != nullptr, head_dim, static_cast<hipStream_t>(hip_stream));
    if (e != hipSuccess) return fail(ATF_EHIP, "%s: launch failed: %s", fn, hipGetErrorString(e));
    return ATF_OK;
}
}  // namespace

int atf_cache_append(const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                     int32_t batch, int64_t n_new, int64_t pos0, int32_t h_kv, int32_t head_dim,
                     int64_t cache_tokens, void* hip_stream) {
    return cache_append_impl("cache_append", k_new, v_new, k_cache, v_cache, batch, n_new, pos0,
                             h_kv, head_dim, cache_tokens, hip_stream, nullptr);
}

int atf_cache_append_rotated(const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                             int32_t batch, int64_t n_new, int64_t pos0, int32_t h_kv,
                             int64_t cache_tokens, const atf_window* w, const double* rope_inv_freq,
                             void* hip_stream) {
    const char* fn = "cache_append_rotated";
    if (w == nullptr) return fail(ATF_EINVAL, "%s: NULL window", fn);
    const int d = w->head_dim;
    if (d != 64 && d != 128)
        return fail(ATF_EUNSUPPORTED, "%s: head_dim %d not built (64 or 128)", fn, d);
    atf::AppendRotParams rp{};
    const int rc = rope_fractions(fn, w, rope_inv_freq, rp.rope_rho_hi, rp.rope_rho_lo);
    if (rc != ATF_OK) return rc;
    return cache_append_impl(fn, k_new, v_new, k_cache, v_cache, batch, n_new, pos0, h_kv, d,
                             cache_tokens, hip_stream, &rp);
}

namespace {
size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

struct WsLayout {
    size_t off_plan, off_m, off_l, off_o, total;
};

// Partial states of `slots` (split or work item) x h_q heads, after `plan_ints` int32.
WsLayout ws_layout(size_t slots, int32_t h_q, int32_t head_dim, size_t plan_ints) {
    const size_t n = slots * size_t(h_q);
    WsLayout L;
    L.off_plan = 0;
    L.off_m = align_up(plan_ints * 4, 256);
    L.off_l = L.off_m + align_up(n * 4, 256);
    L.off_o = L.off_l + align_up(n * 4, 256);
    L.total = L.off_o + align_up(n * size_t(head_dim) * 4, 256);
    return L;
}

// query heads per decode workgroup: the largest divisor of the group up to 32
int32_t decode_heads_per_block(int32_t group) {
    for (int32_t c = atf::kDecodeMaxHeads; c >= 1; --c)
        if (group % c == 0) return c;
    return 1;
}

WsLayout uniform_layout(int32_t batch, int32_t h_q, int32_t h_kv, int64_t n_k, int32_t head_dim) {
    return ws_layout(size_t(batch) * size_t(atf::decode_splits(batch, h_kv, n_k)), h_q, head_dim, 0);
}

// ragged batch: at most items + batch work items (each row rounds its count up once)
WsLayout ragged_layout(int32_t batch, int32_t h_q, int32_t h_kv, int32_t head_dim) {
    const int32_t cols = h_kv * (h_q / h_kv / decode_heads_per_block(h_q / h_kv));
    const size_t items = size_t(atf::decode_ragged_items(cols)) + size_t(batch);
    return ws_layout(items, h_q, head_dim, size_t(batch) + 1);
}
}  // namespace

size_t atf_decode_workspace_bytes(int32_t batch, int32_t h_q, int32_t h_kv, int64_t n_k,
                                  int32_t head_dim) {
    if (batch < 1 || h_q < 1 || h_kv < 1 || h_q % h_kv || n_k < 1 || n_k > kPosLimit ||
        (head_dim != 64 && head_dim != 128))
        return 0;
    // covers both plans: uniform (atf_decode) and ragged (atf_decode_ragged / _paged)
    const size_t u = uniform_layout(batch, h_q, h_kv, n_k, head_dim).total;
    const size_t r = ragged_layout(batch, h_q, h_kv, head_dim).total;
    return u > r ? u : r;
}

}  // extern "C"

namespace {

// Shared by atf_decode (every row has n_k keys and its query at q_pos) and
// atf_decode_ragged (row b has n_k_rows[b] keys and its query at q_pos_rows[b],
// device arrays; n_k is then their upper bound and q_pos is unused).
struct PagedArgs {
    const int32_t* block_table = nullptr;
    int32_t max_pages = 0, num_pages = 0, page_tokens = 0;
};

int decode_impl(const char* fn, const void* q, const void* k_cache, const void* v_cache, void* o,
                float* lse, int32_t batch, int64_t n_k, int64_t q_pos, const int32_t* n_k_rows,
                const int32_t* q_pos_rows, int32_t h_q, int32_t h_kv, int64_t cache_tokens,
                const atf_window* w, float softmax_scale, void* workspace, size_t workspace_bytes,
                void* hip_stream, const PagedArgs& pg = PagedArgs(), const RopeArgs& rope = RopeArgs()) {
    const bool ragged = n_k_rows != nullptr || q_pos_rows != nullptr;
    if (w == nullptr) return fail(ATF_EINVAL, "%s: NULL window", fn);
    const int d = w->head_dim;
    if (d != 64 && d != 128)
        return fail(ATF_EUNSUPPORTED, "%s: head_dim %d not built (64 or 128)", fn, d);
    if (batch < 1 || n_k < 1 || q_pos < 0 || h_q < 1 || h_kv < 1)
        return fail(ATF_EINVAL, "%s: need batch >= 1, n_k >= 1, q_pos >= 0, heads >= 1", fn);
    if (h_q % h_kv != 0)
        return fail(ATF_EINVAL, "%s: h_q %d not a multiple of h_kv %d", fn, h_q, h_kv);
    if (q_pos >= kPosLimit || n_k > kPosLimit)
        return fail(ATF_EINVAL, "%s: positions must stay below 2^31 - 1", fn);
    if (cache_tokens == 0) cache_tokens = n_k;
    if (cache_tokens < n_k || cache_tokens > kPosLimit)
        return fail(ATF_EINVAL, "%s: cache_tokens %lld must be >= n_k %lld and < 2^31 - 1", fn,
                    (long long)cache_tokens, (long long)n_k);
    if (!std::isfinite(softmax_scale))
        return fail(ATF_EINVAL, "%s: softmax_scale must be finite", fn);
    atf::DecodeParams p{};
    int rc = build_table(w, &p.win);
    if (rc != ATF_OK) return rc;
    if (rope.rotate) {
        rc = rope_fractions(fn, w, rope.inv_freq, p.rope_rho_hi, p.rope_rho_lo);
        if (rc != ATF_OK) return rc;
        p.rotate = 1;
    }
    if (!q || !k_cache || !v_cache || !o || !lse)
        return fail(ATF_EINVAL, "%s: NULL tensor pointer", fn);
    if (ragged && (!n_k_rows || !q_pos_rows))
        return fail(ATF_EINVAL, "%s: NULL row-length or row-position array", fn);
    if (!aligned(q, 16) || !aligned(k_cache, 16) || !aligned(v_cache, 16) || !aligned(o, 16) ||
        !aligned(lse, 4))
        return fail(ATF_EINVAL, "%s: q/k/v/o must be 16-byte and lse 4-byte aligned", fn);
    if (ragged && (!aligned(n_k_rows, 4) || !aligned(q_pos_rows, 4)))
        return fail(ATF_EINVAL, "%s: row arrays must be 4-byte aligned", fn);
    if (pg.block_table != nullptr && !aligned(pg.block_table, 4))
        return fail(ATF_EINVAL, "%s: block table must be 4-byte aligned", fn);
    const WsLayout L = ragged ? ragged_layout(batch, h_q, h_kv, d)
                              : uniform_layout(batch, h_q, h_kv, n_k, d);
    if (workspace == nullptr || workspace_bytes < L.total)
        return fail(ATF_EWORKSPACE, "%s: workspace of %zu bytes needed, %zu given", fn, L.total,
                    workspace == nullptr ? size_t(0) : workspace_bytes);
    if (!aligned(workspace, 16)) return fail(ATF_EINVAL, "%s: workspace must be 16-byte aligned", fn);
    const float scale = softmax_scale > 0.f ? softmax_scale : 1.0f / std::sqrt(float(d));
    const int32_t group = h_q / h_kv;
    const int32_t hpb = decode_heads_per_block(group);
    char* ws = static_cast<char*>(workspace);
    p.q = static_cast<const uint16_t*>(q);
    p.kpcm = static_cast<const uint16_t*>(k_cache);
    p.vpk = static_cast<const uint16_t*>(v_cache);
    p.o = static_cast<uint16_t*>(o);
    p.lse = lse;
    p.ws_plan = ragged ? reinterpret_cast<int32_t*>(ws + L.off_plan) : nullptr;
    p.ws_m = reinterpret_cast<float*>(ws + L.off_m);
    p.ws_l = reinterpret_cast<float*>(ws + L.off_l);
    p.ws_o = reinterpret_cast<float*>(ws + L.off_o);
    p.batch = batch;
    p.n_k = static_cast<int32_t>(n_k);
    p.cache_tokens = static_cast<int32_t>(cache_tokens);
    p.q_pos = static_cast<int32_t>(q_pos);
    p.h_q = h_q;
    p.h_kv = h_kv;
    p.group = group;
    p.heads_per_block = hpb;
    p.n_k_rows = n_k_rows;
    p.q_pos_rows = q_pos_rows;
    p.block_table = pg.block_table;
    p.max_pages = pg.max_pages;
    p.num_pages = pg.num_pages;
    p.page_tokens = pg.page_tokens;
    p.n_valid = static_cast<int32_t>(ragged ? n_k : std::min(q_pos, n_k - 1) + 1);
    p.cols16 = atf::decode_cols16(batch, h_q, h_kv, d, p.n_valid, cache_tokens, hpb, ragged);
    if (ragged) {
        // the work items are laid out on the device from the row arrays: the batch's
        // keys in about `splits` equal spans (multiples of the workgroup's token step)
        // per column, each row cut into whole spans of its own keys
        p.splits = atf::decode_plan_items(h_kv * (group / hpb), p.cols16);
        p.split_tokens = 0;
        p.direct = p.cols16 && atf::decode_direct(batch, h_q, h_kv, d, n_k, hpb, rope.rotate, true);
    } else {
        const bool direct = p.cols16 && atf::decode_direct(batch, h_q, h_kv, d, p.n_valid, hpb, rope.rotate, false);
        const int32_t splits =
            direct ? 1 : atf::decode_plan_splits(batch, h_q, h_kv, n_k, p.n_valid, hpb, p.cols16, rope.rotate);
        p.splits = splits;
        p.direct = direct;
        const auto step_of = [&](int64_t s) {
            const int64_t per = (p.n_valid + s - 1) / s;
            return (per + atf::kDecodeTokenStep - 1) / atf::kDecodeTokenStep * atf::kDecodeTokenStep;
        };
        const int64_t step_tokens = step_of(splits);
        // (the longest plan is what a call is refused by, whichever it uses)
        const int64_t room = atf::decode_splits(batch, h_kv, n_k);
        if (step_of(room) * room >= kPosLimit || step_tokens * splits >= kPosLimit)
            return fail(ATF_EINVAL, "%s: cache too long for the split plan", fn);
        p.split_tokens = static_cast<int32_t>(step_tokens);
    }
    p.scale_log2 = scale * 1.4426950408889634f;
    hipError_t e = atf::launch_decode(p, d, static_cast<hipStream_t>(hip_stream));
    if (e != hipSuccess) return fail(ATF_EHIP, "%s: launch failed: %s", fn, hipGetErrorString(e));
    return ATF_OK;
}

}  // namespace

extern "C" {

int atf_decode(const void* q, const void* k_cache, const void* v_cache, void* o, float* lse,
               int32_t batch, int64_t n_k, int64_t q_pos, int32_t h_q, int32_t h_kv,
               int64_t cache_tokens, const atf_window* w, float softmax_scale, void* workspace,
               size_t workspace_bytes, void* hip_stream) {
    return decode_impl("decode", q, k_cache, v_cache, o, lse, batch, n_k, q_pos, nullptr, nullptr,
                       h_q, h_kv, cache_tokens, w, softmax_scale, workspace, workspace_bytes,
                       hip_stream);
}

int atf_decode_noalloc(const void* q, const void* k_cache, const void* v_cache, void* o,
                       float* lse, int32_t batch, int64_t n_k, int64_t q_pos, int32_t h_q,
                       int32_t h_kv, int64_t cache_tokens, const atf_window* w,
                       float softmax_scale, void* hip_stream) {
    static_assert(atf::kNoAllocScratchBytes == ATF_DECODE_NOALLOC_SCRATCH_BYTES,
                  "scratch size of the header and of the library differ");
    if (w == nullptr) return fail(ATF_EINVAL, "decode_noalloc: NULL window");
    const int d = w->head_dim;
    if (batch >= 1 && h_q >= 1 && h_kv >= 1 && h_q % h_kv == 0 && n_k >= 1 && n_k < kPosLimit &&
        (d == 64 || d == 128)) {
        const size_t need = uniform_layout(batch, h_q, h_kv, n_k, d).total;
        if (need > atf::kNoAllocScratchBytes)
            return fail(ATF_EWORKSPACE,
                        "decode_noalloc: these sizes need %zu bytes of partial states, above the "
                        "%zu-byte scratch array (use atf_decode with a workspace)",
                        need, atf::kNoAllocScratchBytes);
    }
    void* ws = nullptr;
    const hipError_t e = atf::noalloc_scratch(&ws);
    if (e != hipSuccess)
        return fail(ATF_EHIP, "decode_noalloc: scratch address: %s", hipGetErrorString(e));
    // every other argument is checked as atf_decode checks it
    return decode_impl("decode_noalloc", q, k_cache, v_cache, o, lse, batch, n_k, q_pos, nullptr,
                       nullptr, h_q, h_kv, cache_tokens, w, softmax_scale, ws,
                       atf::kNoAllocScratchBytes, hip_stream);
}

int atf_decode_unrotated(const void* q, const void* k_cache, const void* v_cache, void* o,
                         float* lse, int32_t batch, int64_t n_k, int64_t q_pos, int32_t h_q,
                         int32_t h_kv, int64_t cache_tokens, const atf_window* w,
                         const double* rope_inv_freq, float softmax_scale, void* workspace,
                         size_t workspace_bytes, void* hip_stream) {
    RopeArgs rope;
    rope.rotate = true;
    rope.inv_freq = rope_inv_freq;
    return decode_impl("decode_unrotated", q, k_cache, v_cache, o, lse, batch, n_k, q_pos, nullptr,
                       nullptr, h_q, h_kv, cache_tokens, w, softmax_scale, workspace,
                       workspace_bytes, hip_stream, PagedArgs(), rope);
}

int atf_decode_ragged_unrotated(const void* q, const void* k_cache, const void* v_cache, void* o,
                                float* lse, int32_t batch, const int32_t* n_k_rows,
                                const int32_t* q_pos_rows, int64_t max_n_k, int32_t h_q,
                                int32_t h_kv, int64_t cache_tokens, const atf_window* w,
                                const double* rope_inv_freq, float softmax_scale,
                                void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!n_k_rows || !q_pos_rows)
        return fail(ATF_EINVAL, "decode_ragged_unrotated: NULL row-length or row-position array");
    RopeArgs rope;
    rope.rotate = true;
    rope.inv_freq = rope_inv_freq;
    return decode_impl("decode_ragged_unrotated", q, k_cache, v_cache, o, lse, batch, max_n_k, 0,
                       n_k_rows, q_pos_rows, h_q, h_kv, cache_tokens, w, softmax_scale, workspace,
                       workspace_bytes, hip_stream, PagedArgs(), rope);
}

int atf_decode_ragged(const void* q, const void* k_cache, const void* v_cache, void* o, float* lse,
                      int32_t batch, const int32_t* n_k_rows, const int32_t* q_pos_rows,
                      int64_t max_n_k, int32_t h_q, int32_t h_kv, int64_t cache_tokens,
                      const atf_window* w, float softmax_scale, void* workspace,
                      size_t workspace_bytes, void* hip_stream) {
    if (!n_k_rows || !q_pos_rows)
        return fail(ATF_EINVAL, "decode_ragged: NULL row-length or row-position array");
    return decode_impl("decode_ragged", q, k_cache, v_cache, o, lse, batch, max_n_k, 0, n_k_rows,
                       q_pos_rows, h_q, h_kv, cache_tokens, w, softmax_scale, workspace,
                       workspace_bytes, hip_stream);
}

}  // extern "C"

namespace {
int decode_paged_impl(const char* fn, const void* q, const void* k_pages, const void* v_pages,
                      void* o, float* lse, int32_t batch, const int32_t* block_table,
                      int32_t max_pages_per_row, int32_t num_pages, int32_t page_tokens,
                      const int32_t* n_k_rows, const int32_t* q_pos_rows, int64_t max_n_k,
                      int32_t h_q, int32_t h_kv, const atf_window* w, float softmax_scale,
                      void* workspace, size_t workspace_bytes, void* hip_stream,
                      const RopeArgs& rope) {
    if (!block_table) return fail(ATF_EINVAL, "%s: NULL block table", fn);
    if (!n_k_rows || !q_pos_rows)
        return fail(ATF_EINVAL, "%s: NULL row-length or row-position array", fn);
    if (page_tokens < 32 || page_tokens % 32 != 0)
        return fail(ATF_EINVAL, "%s: page_tokens %d must be a positive multiple of 32",
                    fn, page_tokens);
    if (num_pages < 1 || max_pages_per_row < 1)
        return fail(ATF_EINVAL, "%s: need num_pages >= 1 and max_pages_per_row >= 1", fn);
    const int64_t row_cap = int64_t(max_pages_per_row) * page_tokens;
    if (max_n_k > row_cap || row_cap > kPosLimit)
        return fail(ATF_EINVAL, "%s: max_n_k %lld exceeds the %lld tokens a row's pages "
                    "hold (or that exceeds 2^31 - 1)", fn, (long long)max_n_k, (long long)row_cap);
    PagedArgs pg;
    pg.block_table = block_table;
    pg.max_pages = max_pages_per_row;
    pg.num_pages = num_pages;
    pg.page_tokens = page_tokens;
    // the contiguous-cache capacity is the rows' span; the kernel addresses pages instead
    return decode_impl(fn, q, k_pages, v_pages, o, lse, batch, max_n_k, 0, n_k_rows, q_pos_rows,
                       h_q, h_kv, row_cap, w, softmax_scale, workspace, workspace_bytes, hip_stream,
                       pg, rope);
}
}  // namespace

extern "C" {

int atf_decode_paged(const void* q, const void* k_pages, const void* v_pages, void* o, float* lse,
                     int32_t batch, const int32_t* block_table, int32_t max_pages_per_row,
                     int32_t num_pages, int32_t page_tokens, const int32_t* n_k_rows,
                     const int32_t* q_pos_rows, int64_t max_n_k, int32_t h_q, int32_t h_kv,
                     const atf_window* w, float softmax_scale, void* workspace,
                     size_t workspace_bytes, void* hip_stream) {
    return decode_paged_impl("decode_paged", q, k_pages, v_pages, o, lse, batch, block_table,
                             max_pages_per_row, num_pages, page_tokens, n_k_rows, q_pos_rows,
                             max_n_k, h_q, h_kv, w, softmax_scale, workspace, workspace_bytes,
                             hip_stream, RopeArgs());
}

int atf_decode_paged_unrotated(const void* q, const void* k_pages, const void* v_pages, void* o,
                               float* lse, int32_t batch, const int32_t* block_table,
                               int32_t max_pages_per_row, int32_t num_pages, int32_t page_tokens,
                               const int32_t* n_k_rows, const int32_t* q_pos_rows,
                               int64_t max_n_k, int32_t h_q, int32_t h_kv, const atf_window* w,
                               const double* rope_inv_freq, float softmax_scale, void* workspace,
                               size_t workspace_bytes, void* hip_stream) {
    RopeArgs rope;
    rope.rotate = true;
    rope.inv_freq = rope_inv_freq;
    return decode_paged_impl("decode_paged_unrotated", q, k_pages, v_pages, o, lse, batch,
                             block_table, max_pages_per_row, num_pages, page_tokens, n_k_rows,
                             q_pos_rows, max_n_k, h_q, h_kv, w, softmax_scale, workspace,
                             workspace_bytes, hip_stream, rope);
}

namespace {
// Shared by atf_cache_append_paged and atf_cache_append_paged_rotated (rope != nullptr:
// the keys turned to their positions on the way in).
int cache_append_paged_impl(const char* fn, const void* k_new, const void* v_new, void* k_pages,
                            void* v_pages, const int32_t* block_table, int32_t max_pages_per_row,
                            int32_t num_pages, int32_t page_tokens, int32_t batch, int64_t n_new,
                            int64_t pos0, int32_t h_kv, int32_t head_dim, void* hip_stream,
                            const atf::AppendRotParams* rope) {
    if (head_dim != 64 && head_dim != 128)
        return fail(ATF_EUNSUPPORTED, "%s: head_dim %d not built", fn, head_dim);
    if (batch < 1 || h_kv < 1 || n_new < 0 || pos0 < 0)
        return fail(ATF_EINVAL, "%s: need batch >= 1, h_kv >= 1, n_new >= 0, pos0 >= 0", fn);
    if (page_tokens < 32 || page_tokens % 32 != 0)
        return fail(ATF_EINVAL, "%s: page_tokens %d must be a positive multiple of 32", fn,
                    page_tokens);
    if (num_pages < 1 || max_pages_per_row < 1)
        return fail(ATF_EINVAL, "%s: need num_pages >= 1 and max_pages_per_row >= 1", fn);
    const int64_t row_cap = int64_t(max_pages_per_row) * page_tokens;
    if (row_cap > kPosLimit || pos0 + n_new > row_cap)
        return fail(ATF_EINVAL, "%s: tokens %lld .. %lld do not fit the %lld tokens "
                    "of a row's pages", fn, (long long)pos0, (long long)(pos0 + n_new), (long long)row_cap);
    if (!k_new || !v_new || !k_pages || !v_pages || !block_table)
        return fail(ATF_EINVAL, "%s: NULL pointer", fn);
    if (!aligned(k_new, 16) || !aligned(v_new, 16) || !aligned(k_pages, 16) ||
        !aligned(v_pages, 16) || !aligned(block_table, 4))
        return fail(ATF_EINVAL, "%s: tensors must be 16-byte, the table 4-byte aligned", fn);
    if (n_new == 0) return ATF_OK;
    if (int64_t(batch) * n_new * h_kv > kPosLimit)
        return fail(ATF_EINVAL, "%s: too many tokens for one call", fn);
    atf::AppendRotParams p = rope != nullptr ? *rope : atf::AppendRotParams{};
    p.k_src = static_cast<const uint16_t*>(k_new);
    p.v_src = static_cast<const uint16_t*>(v_new);
    p.k_dst = static_cast<uint16_t*>(k_pages);
    p.v_dst = static_cast<uint16_t*>(v_pages);
    p.block_table = block_table;
    p.batch = batch;
    p.n_new = static_cast<int32_t>(n_new);
    p.pos0 = static_cast<int32_t>(pos0);
    p.h_kv = h_kv;
    p.max_pages = max_pages_per_row;
    p.num_pages = num_pages;
    p.page_tokens = page_tokens;
    const hipError_t e = atf::launch_append(p, rope != nullptr, head_dim, static_cast<hipStream_t>(hip_stream));
    if (e != hipSuccess) return fail(ATF_EHIP, "%s: launch failed: %s", fn, hipGetErrorString(e));
    return ATF_OK;
}
}  // namespace

int atf_cache_append_paged(const void* k_new, const void* v_new, void* k_pages, void* v_pages,
                           const int32_t* block_table, int32_t max_pages_per_row,
                           int32_t num_pages, int32_t page_tokens, int32_t batch, int64_t n_new,
                           int64_t pos0, int32_t h_kv, int32_t head_dim, void* hip_stream) {
    return cache_append_paged_impl("cache_append_paged", k_new, v_new, k_pages, v_pages,
                                   block_table, max_pages_per_row, num_pages, page_tokens, batch,
                                   n_new, pos0, h_kv, head_dim, hip_stream, nullptr);
}

int atf_cache_append_paged_rotated(const void* k_new, const void* v_new, void* k_pages,
                                   void* v_pages, const int32_t* block_table,
                                   int32_t max_pages_per_row, int32_t num_pages,
                                   int32_t page_tokens, int32_t batch, int64_t n_new, int64_t pos0,
                                   int32_t h_kv, const atf_window* w, const double* rope_inv_freq,
                                   void* hip_stream) {
    const char* fn = "cache_append_paged_rotated";
    if (w == nullptr) return fail(ATF_EINVAL, "%s: NULL window", fn);
    const int d = w->head_dim;
    if (d != 64 && d != 128)
        return fail(ATF_EUNSUPPORTED, "%s: head_dim %d not built (64 or 128)", fn, d);
    atf::AppendRotParams rp{};
    const int rc = rope_fractions(fn, w, rope_inv_freq, rp.rope_rho_hi, rp.rope_rho_lo);
    if (rc != ATF_OK) return rc;
    return cache_append_paged_impl(fn, k_new, v_new, k_pages, v_pages, block_table,
                                   max_pages_per_row, num_pages, page_tokens, batch, n_new, pos0,
                                   h_kv, d, hip_stream, &rp);
}

}  // extern "C"
