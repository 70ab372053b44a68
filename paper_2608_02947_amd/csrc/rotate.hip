// Writes into the caches: the appends and packs (keys as given or turned to their
// positions on the way in, contiguous or paged caches), and RoPE over a whole unrotated K
// cache in one pass.  Rotation at write time (App. B sets it against rotating at read
// time) costs one read and one write of the keys and every (key, pair) rotation, whatever
// the window keeps; a long prefill over an unrotated cache can take it instead of the
// read-time path when the rotated copy's memory is at hand.
//
// All memory-bound.  Angles are evaluated directly (0.64 fixed-point fraction, v_cos_f32 /
// v_sin_f32 in revolutions), rotated in fp32 and rounded to bf16.
#include "atf_internal.hpp"
#include "rope.hpp"

#include <algorithm>
#include <type_traits>

namespace atf {
namespace {

// Whole cache: one thread per (key, pair-chunk) record; grid y = the (batch, kv head,
// chunk) stream, x over its tokens, so a block's chunk and its 8 frequencies are uniform
// and consecutive threads touch consecutive 32-byte records.
template <int D>
__global__ __launch_bounds__(256) void rotate_kcache_kernel(const RotateParams p) {
    constexpr int kChunks = D / 16;
    const int stream = blockIdx.y;  // (b * h_kv + g) * kChunks + c
    const int c = stream % kChunks;
    const int64_t off = int64_t(stream) * p.cache_tokens * 16;
    const uint16_t* src = p.src + off;
    uint16_t* dst = p.dst + off;
    for (int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x; t < p.n_k;
         t += int64_t(gridDim.x) * 256) {
        const rope::u32x4_t x = *reinterpret_cast<const rope::u32x4_t*>(src + 16 * t);
        const rope::u32x4_t y = *reinterpret_cast<const rope::u32x4_t*>(src + 16 * t + 8);
        float cs8[8], sn8[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float u = rope::revolutions(uint32_t(t), make_uint2(p.rope_rho_hi[8 * c + e],
                                                                      p.rope_rho_lo[8 * c + e]));
            cs8[e] = __builtin_amdgcn_cosf(u);
            sn8[e] = __builtin_amdgcn_sinf(u);
        }
        *reinterpret_cast<rope::u32x4_t*>(dst + 16 * t) = rope::rotate_cs(x, y, 0, cs8, sn8);
        *reinterpret_cast<rope::u32x4_t*>(dst + 16 * t + 8) = rope::rotate_cs(y, x, 1, cs8, sn8);
    }
}

// Append: K and V of the new tokens in one launch.  One wave per unit = (batch, 16-token
// block of cache positions, kv head), heads fastest, so that the waves of a workgroup read
// neighbouring rows of the source ([B][n_new][h_kv][d]).
//   K, turned: one (token, chunk) record per lane and step: 16 bytes of each half of the
//      chunk's pairs in, 32 contiguous bytes of the chunk's stream out; 16 tokens of a chunk
//      are 512 contiguous bytes.
//   K, as given: 16 bytes per lane and step, lanes along a token's row, so that a step reads
//      whole rows and stores whole 32-byte records (as above every store instruction leaves
//      out half of each: packs of 52 x 344 tokens of 4 heads at d = 128 8.1 us -> 7.1, of
//      51 x 3,021 of one at d = 64 8.0 -> 6.4; appends of K and V 1-7 % less).
//   V: a lane takes 2 dims x the 8 tokens of one half of the block's slots (slot 8h + e
//      holds token 8(e/4) + 4h + e%4): eight 4-byte loads, 256 (d = 64: 128) contiguous
//      bytes per token, transposed in registers into two 16-byte stores.  Of a block that
//      the call does not cover whole only the call's slots are written, so the others keep
//      their contents (or become zero past the source when zero_tail is set): a lane takes
//      2 dims, 8 tokens loaded before the first is stored, four stored at a time where the
//      call has them (token by token, load and store, 15 tokens in a block of each of 141 x
//      8 heads took 23.3 us, and 11.0 so; 16 tokens loaded at once need 102 registers for 70, and
//      16,384 whole tokens then take 34.2 us for 33.2).
// Bound by HBM; every load of a unit is in flight before the first store.  One thread per
// (token, chunk) and per (block, dim) with a 64-bit division chain each and 2-byte stores
// of V, in two launches, took 96 us for 16,384 tokens of 8 heads at d = 128 (134 MB moved,
// rotated); this takes 33.2 us (4.0 TB/s).
constexpr int kKeysNone = 0, kKeysAsGiven = 1, kKeysTurned = 2;

template <int D, int kKeys, bool kValues, bool kPaged>
__global__ __launch_bounds__(256) void append_kernel(
    const std::conditional_t<kKeys == kKeysTurned, AppendRotParams, AppendParams> p) {
    constexpr int kChunks = D / 16;
    constexpr int kSteps = D / 64;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63;
    const int blk0 = p.pos0 / 16;
    const int nblk = (p.pos0 + p.n_new - 1) / 16 + 1 - blk0;  // blocks touched
    const uint32_t units = uint32_t(p.batch) * uint32_t(nblk) * uint32_t(p.h_kv);
    for (uint32_t unit = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6)); unit < units;
         unit += gridDim.x * 4) {
        const int g = int(unit % uint32_t(p.h_kv));
        const uint32_t rest = unit / uint32_t(p.h_kv);
        const int blk = blk0 + int(rest % uint32_t(nblk));
        const int b = int(rest / uint32_t(nblk));
        // first token of the block in the source, and the tokens of the block in it
        const int t0 = 16 * blk - p.pos0;
        const int lo = max(0, -t0), hi = min(16, p.n_new - t0);
        // the unit's place in the caches: chunk c of block token t at
        // kd + (c * kstride + t) * 16, dim x at vd + x * 16
        int64_t kd, kstride, vd;
        if constexpr (kPaged) {
            const int page = p.block_table[int64_t(b) * p.max_pages + 16 * blk / p.page_tokens];
            if (page < 0 || page >= p.num_pages) continue;
            const int at = 16 * blk % p.page_tokens;  // a page holds whole blocks
            const int64_t ph = int64_t(page) * p.h_kv + g;
            kd = (ph * kChunks * p.page_tokens + at) * 16;
            kstride = p.page_tokens;
            vd = (ph * (p.page_tokens / 16) + at / 16) * int64_t(D) * 16;
        } else {
            const int64_t bh = int64_t(b) * p.h_kv + g;
            kd = (bh * kChunks * p.cache_tokens + 16 * int64_t(blk)) * 16;
            kstride = p.cache_tokens;
            vd = (bh * ((int64_t(p.cache_tokens) + 15) / 16) + blk) * int64_t(D) * 16;
        }
        // element offset of (block token t, dim 0) in the sources: src0 + t * row
        const int64_t row = int64_t(p.h_kv) * D;
        const int64_t src0 = ((int64_t(b) * p.n_new + t0) * p.h_kv + g) * D;

        // W: the call covers the whole block (no test per token)
        auto move = [&](auto whole_tag) __attribute__((always_inline)) {
            constexpr bool W = decltype(whole_tag)::value;
            u32x4 kx[kSteps], ky[kSteps];
            [[maybe_unused]] uint32_t vx[kSteps][8];
            // a key that is not turned: piece i, 8 dims of half h of token t
            const auto piece = [&](int j, auto f) __attribute__((always_inline)) {
                const int i = lane + 64 * j, t = i / (D / 8), o = i % (D / 8);
                if (W || (t >= lo && t < hi)) f(j & 1 ? ky[j / 2] : kx[j / 2], t, o % kChunks, o / kChunks);
            };
            if constexpr (kKeys == kKeysAsGiven) {
#pragma unroll
                for (int j = 0; j < 2 * kSteps; ++j)
                    piece(j, [&](u32x4& x, int t, int c, int h) __attribute__((always_inline)) {
                        x = *reinterpret_cast<const u32x4*>(p.k_src + src0 + t * row + h * (D / 2) + 8 * c);
                    });
            }
            if constexpr (kKeys == kKeysTurned) {
#pragma unroll
                for (int j = 0; j < kSteps; ++j) {
                    const int t = lane & 15, c = (lane >> 4) + 4 * j;
                    kx[j] = ky[j] = u32x4{0u, 0u, 0u, 0u};
                    if (W || (t >= lo && t < hi)) {
                        const uint16_t* src = p.k_src + src0 + t * row + 8 * c;
                        kx[j] = *reinterpret_cast<const u32x4*>(src);
                        ky[j] = *reinterpret_cast<const u32x4*>(src + D / 2);
                    }
                }
            }
            // one or two tokens, a decode step's: their values loaded with the keys
            [[maybe_unused]] const int end = p.zero_tail ? 16 : hi;
            [[maybe_unused]] uint32_t few[2] = {0u, 0u};
            if constexpr (kValues && !W) {
                if (lane < D / 2 && end - lo <= 2) {
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        if (lo + i < hi) few[i] = *reinterpret_cast<const uint32_t*>(p.v_src + src0 + (lo + i) * row + 2 * lane);
                }
            }
            if constexpr (kValues && W) {
#pragma unroll
                for (int j = 0; j < kSteps; ++j) {
                    const int it = lane + 64 * j, dp = it % (D / 2), h = it / (D / 2);
                    const uint16_t* src = p.v_src + src0 + 4 * h * row + 2 * dp;
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        vx[j][e] = *reinterpret_cast<const uint32_t*>(src + (8 * (e / 4) + e % 4) * row);
                }
            }
            if constexpr (kKeys == kKeysAsGiven) {
#pragma unroll
                for (int j = 0; j < 2 * kSteps; ++j)
                    piece(j, [&](u32x4& x, int t, int c, int h) __attribute__((always_inline)) {
                        *reinterpret_cast<u32x4*>(p.k_dst + kd + (c * kstride + t) * 16 + 8 * h) = x;
                    });
            }
            if constexpr (kKeys == kKeysTurned) {
#pragma unroll
                for (int j = 0; j < kSteps; ++j) {
                    const int t = lane & 15, c = (lane >> 4) + 4 * j;
                    float cs8[8], sn8[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float u = rope::revolutions(uint32_t(16 * blk + t),
                                                          make_uint2(p.rope_rho_hi[8 * c + e], p.rope_rho_lo[8 * c + e]));
                        cs8[e] = __builtin_amdgcn_cosf(u);
                        sn8[e] = __builtin_amdgcn_sinf(u);
                    }
                    const u32x4 x = kx[j], y = ky[j];
                    kx[j] = rope::rotate_cs(x, y, 0, cs8, sn8);
                    ky[j] = rope::rotate_cs(y, x, 1, cs8, sn8);
                    if (W || (t >= lo && t < hi)) {
                        uint16_t* dst = p.k_dst + kd + (c * kstride + t) * 16;
                        *reinterpret_cast<u32x4*>(dst) = kx[j];
                        *reinterpret_cast<u32x4*>(dst + 8) = ky[j];
                    }
                }
            }
            if constexpr (kValues && W) {
#pragma unroll
                for (int j = 0; j < kSteps; ++j) {
                    const int it = lane + 64 * j, dp = it % (D / 2), h = it / (D / 2);
                    uint16_t* dst = p.v_dst + vd + 32 * dp + 8 * h;  // slots of dims 2 dp, 2 dp + 1
                    u32x4 even, odd;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        even[q] = __builtin_amdgcn_perm(vx[j][2 * q + 1], vx[j][2 * q], 0x05040100u);
                        odd[q] = __builtin_amdgcn_perm(vx[j][2 * q + 1], vx[j][2 * q], 0x07060302u);
                    }
                    *reinterpret_cast<u32x4*>(dst) = even;
                    *reinterpret_cast<u32x4*>(dst + 16) = odd;
                }
            }
            if constexpr (kValues && !W) {
                // 2 dims per lane; slots of token 4 q + i: 8 (q % 2) + 4 (q / 2) + i
                if (lane < D / 2 && end - lo <= 2) {
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const int t = lo + i;
                        uint16_t* dst = p.v_dst + vd + 32 * lane + 8 * (t % 8 / 4) + 4 * (t / 8) + t % 4;
                        if (t < end) {
                            dst[0] = uint16_t(few[i]);
                            dst[16] = uint16_t(few[i] >> 16);
                        }
                    }
                } else if (lane < D / 2) {
#pragma unroll 1
                    for (int h8 = lo & 8; h8 < end; h8 += 8) {
                        uint32_t x[8];
#pragma unroll
                        for (int t = 0; t < 8; ++t) {
                            x[t] = 0u;
                            if (h8 + t >= lo && h8 + t < hi)
                                x[t] = *reinterpret_cast<const uint32_t*>(p.v_src + src0 + (h8 + t) * row + 2 * lane);
                        }
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            const int t0 = h8 + 4 * q;  // its slots: 8 q + h8 / 2 on
                            uint16_t* dst = p.v_dst + vd + 32 * lane + 8 * q + h8 / 2;
                            const uint32_t* y = &x[4 * q];
                            if (t0 >= lo && t0 + 4 <= end) {
                                *reinterpret_cast<uint2*>(dst) = make_uint2(__builtin_amdgcn_perm(y[1], y[0], 0x05040100u),
                                                                            __builtin_amdgcn_perm(y[3], y[2], 0x05040100u));
                                *reinterpret_cast<uint2*>(dst + 16) = make_uint2(__builtin_amdgcn_perm(y[1], y[0], 0x07060302u),
                                                                                 __builtin_amdgcn_perm(y[3], y[2], 0x07060302u));
                            } else {
#pragma unroll
                                for (int i = 0; i < 4; ++i)
                                    if (t0 + i >= lo && t0 + i < end) {
                                        dst[i] = uint16_t(y[i]);
                                        dst[16 + i] = uint16_t(y[i] >> 16);
                                    }
                            }
                        }
                    }
                }
            }
        };
        if (hi - lo == 16)
            move(std::true_type{});
        else
            move(std::false_type{});
    }
}

template <int D, int kKeys, bool kValues, bool kPaged>
hipError_t launch_append_k(const AppendRotParams& p, hipStream_t stream) {
    const int64_t nblk = (p.pos0 + p.n_new - 1) / 16 + 1 - p.pos0 / 16;
    const int64_t units = int64_t(p.batch) * nblk * p.h_kv;
    // (16 rows of 128 bytes or more each: 2^31 units do not fit the memory)
    if (units < 1 || units > 0x7fffffff) return hipErrorInvalidConfiguration;
    const int64_t blocks = std::min<int64_t>((units + 3) / 4, 1 << 20);
    (void)hipGetLastError();
    hipLaunchKernelGGL((append_kernel<D, kKeys, kValues, kPaged>), dim3(unsigned(blocks)), dim3(256), 0, stream, p);
    return hipGetLastError();
}

template <int D>
hipError_t launch_append_d(const AppendRotParams& p, bool turn, hipStream_t stream) {
    if (p.block_table != nullptr)
        return turn ? launch_append_k<D, kKeysTurned, true, true>(p, stream)
                    : launch_append_k<D, kKeysAsGiven, true, true>(p, stream);
    if (p.v_src == nullptr) return launch_append_k<D, kKeysAsGiven, false, false>(p, stream);
    if (p.k_src == nullptr) return launch_append_k<D, kKeysNone, true, false>(p, stream);
    return turn ? launch_append_k<D, kKeysTurned, true, false>(p, stream)
                : launch_append_k<D, kKeysAsGiven, true, false>(p, stream);
}

}  // namespace

hipError_t launch_append(const AppendRotParams& p, bool turn, int head_dim, hipStream_t stream) {
    return head_dim == 64 ? launch_append_d<64>(p, turn, stream) : launch_append_d<128>(p, turn, stream);
}

hipError_t launch_rotate_kcache(const RotateParams& p, int head_dim, hipStream_t stream) {
    const int64_t streams = int64_t(p.batch) * p.h_kv * (head_dim / 16);
    if (streams < 1 || streams > 65535 || p.n_k < 1) return hipErrorInvalidConfiguration;
    const int64_t xb = (int64_t(p.n_k) + 255) / 256;
    const dim3 grid(unsigned(xb < 1024 ? xb : 1024), unsigned(streams));
    (void)hipGetLastError();
    if (head_dim == 64)
        hipLaunchKernelGGL(rotate_kcache_kernel<64>, grid, dim3(256), 0, stream, p);
    else
        hipLaunchKernelGGL(rotate_kcache_kernel<128>, grid, dim3(256), 0, stream, p);
    return hipGetLastError();
}

}  // namespace atf
