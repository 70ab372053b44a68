// Windowed causal prefill for gfx950 (CDNA4): tiled attention with an online
// softmax in which the per-RoPE-wavelength window (Sec. 3.2 eq:window) is applied
// as a per-tile slice of the QK contraction axis (Sec. 3.3).
//
// Work decomposition
//   A workgroup of W waves owns 32 W query rows that share one KV head: P = 32W/G
//   consecutive positions x the G query heads of the group (row f -> position
//   f / G, head f % G), so every K/V tile staged in LDS serves all of them.  Each
//   wave owns 32 rows (one MFMA row-block).  W = 8 at d = 128 (two waves per
//   SIMD), W = 4 at d = 64 (three workgroups per CU).  Key tiles of 64 rotate
//   through LDS buffers filled by global_load_lds_dwordx4 (global memory straight
//   into LDS, no register staging) one tile ahead of the compute.
//
// K comes from the pair-chunk-major cache (the decode layout): chunk c of a KV
// head is a stream of 32 bytes per key (dims [8c, 8c+8) then [d/2+8c, d/2+8c+8)),
// so one wave-wide direct load fetches one chunk of 32 keys as 1 KB of contiguous
// memory, and a chunk that no cell of the tile keeps is skipped by one
// wave-uniform branch -- its bytes are never read from HBM.  In LDS the K tile is
// [chunk][32-key block][half][key][8 bf16]: a fragment read of 64 lanes covers
// 1 KB without bank conflicts.  V also comes from the decode cache: 16-token
// blocks stored [d][16 slots], slot 8h + e holding token 8(e/4) + 4h + e%4 of the
// block.  A 64-key tile is four consecutive blocks, one contiguous copy into LDS,
// and the 8 slots a lane needs for the PV operand are 16 contiguous bytes.
//
// Matrix layout (v_mfma_f32_32x32x16_bf16, lane l, c = l % 32, h = l / 32)
//   S^T[key][row] = K[key][dims] * Q^T[dims][row]: A = K fragment (key c, dims
//   8h..8h+7 of the K-step), B = Q fragment (row c, same dims), so lane l holds
//   query row c and keys 8*(v/4) + 4h + v%4 of a 32-key block (v < 16).  One query
//   row per lane pair makes the row max and sum lane-local plus one exchange.
//   O^T[d][row] += V^T[d][key] * P^T[key][row]: the S^T registers, rounded to
//   bf16, are the B operand as they are (element e of lane half h = key
//   8(e/4) + 4h + e%4 of a 16-key group); the V^T operand of lane (dim c, half h)
//   is slots 8h .. 8h+7 of dim row c of the packed block: the same keys.
//
// Window as a K-slice (one K-step = one chunk of 8 rotary pairs = dims
// [8c, 8c+8) and [d/2 + 8c, d/2 + 8c + 8)).  Whether pair r contributes to a cell
// depends only on the cell's distance z (keep iff z <= W_r).
//   Uniform tiles.  When no threshold falls inside the distance range of a wave's
//   tile, every pair is either kept in all of its cells or in none.  With
//   thresholds non-decreasing in r, the kept pairs are a suffix r >= rf, so the
//   tile's QK is the chunks above rf / 8 in full plus chunk rf / 8 with the query
//   dims of the pairs below rf zeroed.  That set stays the same for a run of
//   consecutive tiles (until the next threshold enters the distance range), and
//   each wave runs such a run in a loop compiled for its chunk count: straight
//   matrix code with no per-tile branch.
//   Other tiles (a threshold inside the range, or a table that is not monotone)
//   take the general path: per 32-key block, two ballots classify all pairs at
//   once (kept in every cell / in some cell); whole chunks go into one MFMA each
//   with the query dims of pairs kept nowhere zeroed, and each pair whose
//   threshold lies inside the block's range gets one MFMA of its own whose
//   product is added only to the cells with z <= W_r.
//   Every cell sums exactly its kept pairs.  K chunks that no cell of the
//   workgroup's tile keeps are not loaded into LDS.  With the window off the
//   kernel is compiled without any of this.
//
// Softmax: fp32 in the log2 domain.  The running max is raised only when a row's
// tile max exceeds it by more than kRescale (log2 units); otherwise the stale
// max is kept, probabilities are at most 2^kRescale, and the output and
// normaliser need no rescaling -- the result is the same softmax.  Row sums add
// the fp32 probabilities; the PV MFMA consumes them rounded to bf16.
#include "atf_internal.hpp"
#include "rope.hpp"

#include <algorithm>
#include <type_traits>

namespace atf {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) u32x4_t lds_u32x4;

constexpr int kBN = 64;           // keys per tile
constexpr float kRescale = 8.0f;  // lazy-rescale threshold, log2 units

// 8 waves (256 rows) per workgroup, two waves per SIMD, three LDS stages; the
// windowed kernel at d = 64 instead runs 4 waves (128 rows) per workgroup with two
// LDS stages, so that three workgroups share a CU at its ~160 VGPRs.
template <int D, bool kWin>
struct Cfg {
    static constexpr bool kSmall = D == 64 && kWin;
    static constexpr int kWaves = kSmall ? 4 : 8;
    static constexpr int kThreads = kWaves * 64;
    static constexpr int kRows = kWaves * 32;  // query rows per workgroup
    static constexpr int kStages = kSmall ? 2 : 3;  // LDS buffers per K and V tile
    static constexpr int kMinWavesPerSimd = kSmall ? 3 : 2;
    static constexpr int kHalf = D / 2;
    static constexpr int kChunks = D / 16;
    static constexpr int kKTile = kChunks * kBN * 16;  // bf16; [chunk][block][half][key][8]
    static constexpr int kVBlkBytes = D * 32;          // one packed 16-key V block [d][16]
    static constexpr int kVTile = kBN * D;             // bf16; four packed blocks
    static constexpr int kKPerWave = 2 * kChunks / kWaves;  // K (chunk, block) units per wave
    static constexpr int kVLoads = kVTile / 512;      // wave-wide 1 KB loads per V tile
    static constexpr int kVPer = (kVLoads + kWaves - 1) / kWaves;
    static_assert((2 * kChunks) % kWaves == 0, "K units must spread evenly over the waves");
    static_assert(kVTile % 512 == 0, "V tile must be whole kilobytes");
};

__device__ __forceinline__ f32x16_t mfma(u32x4_t a, u32x4_t b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                   __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

__device__ __forceinline__ f32x16_t zero16() {
    f32x16_t z;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = 0.f;
    return z;
}

// Keep only the pairs whose bit is set in `mask` (bit e = pair 8c+e of the
// chunk); a fragment holds the 8 dims of one half of the chunk, element e in
// dword e/2, low half for even e.
__device__ __forceinline__ u32x4_t keep_pairs(u32x4_t x, uint32_t mask) {
    u32x4_t r;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const uint32_t m = ((mask >> (2 * t)) & 1u ? 0x0000FFFFu : 0u) |
                           ((mask >> (2 * t + 1)) & 1u ? 0xFFFF0000u : 0u);
        r[t] = x[t] & m;
    }
    return r;
}

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// LDS reads at a byte address.  Callers form addresses as (per-lane base below
// 2^18) + (constant), so the compiler folds the constants into the
// instructions' offset fields.
__device__ __forceinline__ u32x4_t lds_read_b128(uint32_t byte_addr) {
    return *(const lds_u32x4*)(uintptr_t)byte_addr;
}
// byte offset of the LDS buffer of a tile.  Passed through readfirstlane so the
// compiler treats it as one opaque scalar per tile instead of re-deriving it in
// every address (which defeats the offset-field folding above).
template <int kStages>
__device__ __forceinline__ uint32_t stage_off(int tile, int buf_bytes) {
    return uint32_t(__builtin_amdgcn_readfirstlane((tile % kStages) * buf_bytes));
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return uint32_t(reinterpret_cast<uintptr_t>((const lds_char*)p)) & 0x3FFFFu;
}

// 16 bytes per lane from global memory straight into LDS: lane i reads base + off
// (base wave-uniform) and its 16 bytes land at byte lds_wave + 16 * i (lds_wave
// wave-uniform).  Issued as inline assembly so that the compiler does not make
// LDS reads of other buffers wait for it; completion is awaited explicitly
// (vm_wait) before the workgroup barrier that publishes the buffer.
__device__ __forceinline__ void load_to_lds(const char* base, uint32_t off, uint32_t lds_wave) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(off), "s"(base), "s"(lds_wave)
                 : "memory", "m0");
}
// wait until this wave's vector memory loads have completed (vmcnt 0 only)
__device__ __forceinline__ void vm_wait() { __builtin_amdgcn_s_waitcnt(0x0F70); }
// workgroup barrier without a memory fence: every LDS read is consumed (waited
// for) before it, and the direct-to-LDS loads are awaited with vm_wait
__device__ __forceinline__ void barrier() { __builtin_amdgcn_s_barrier(); }

// LDS of the rotation tables of the kernels that rotate at read time (dynamic, bytes)
template <int D, bool kWin>
struct RotLds {
    static constexpr int kColStride = D + 4;
    static constexpr unsigned kBytes =
        unsigned(32 * kColStride + Cfg<D, kWin>::kWaves * Cfg<D, kWin>::kKPerWave * 16 + D) * 4u;
};

// Two waves per SIMD (one workgroup per CU): the windowed kernel's registers
// exceed the 128 that four waves per SIMD would leave each wave, even at d = 64.
template <int D, bool kWin, bool kRot>
__global__ __launch_bounds__((Cfg<D, kWin>::kThreads), (Cfg<D, kWin>::kMinWavesPerSimd)) void
prefill_kernel(const std::conditional_t<kRot, PrefillRotParams, PrefillParams> p) {
    using C = Cfg<D, kWin>;
    __shared__ __attribute__((aligned(16))) uint16_t Ks[C::kStages][C::kKTile];
    __shared__ __attribute__((aligned(16))) uint16_t Vs[C::kStages][C::kVTile];
    // rotation at read time (dynamic LDS, after the static buffers): cos and sin of
    // kk * theta_r for the 32 key offsets of a 32-key block (row kk: pairs interleaved
    // as (cos, sin), padded by 16 bytes), then per wave and K unit the cos and sin of
    // the block's first position * theta_r, then rho_r (hi, lo) of every pair
    constexpr int kColStride = RotLds<D, kWin>::kColStride;
    extern __shared__ __attribute__((aligned(16))) float s_rot[];
    float* const s_colcs = s_rot;
    float* const s_base = s_rot + 32 * kColStride;
    uint2* const s_rho = reinterpret_cast<uint2*>(s_base + C::kWaves * C::kKPerWave * 16);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31;
    const int hh = lane >> 5;

    // block -> (position tile, kv head, batch); heavy (late) tiles first.  Blocks
    // are dealt to the 8 XCDs round-robin, so with h_kv * batch a multiple or a
    // divisor of 8 every XCD keeps to fixed KV heads and its L2 serves them.
    const int per_tile = p.h_kv * p.batch;
    const int bid = blockIdx.x;
    const int qt = p.n_qtiles - 1 - bid / per_tile;
    const int rem = bid % per_tile;
    const int g = rem % p.h_kv;
    const int b = rem / p.h_kv;
    const int G = p.group;

    const int i0 = qt * p.pos_per_tile;  // first query row (position index)
    const int npos = min(p.pos_per_tile, p.n_q - i0);
    const int rows_valid = npos * G;
    const int pos_first = p.q_pos0 + i0;
    const int pos_last = pos_first + npos - 1;
    const int key_end = min(p.n_k, pos_last + 1);

    // this lane's row: workgroup row 32 * wave + col
    const int f = 32 * wave + col;
    const bool row_ok = f < rows_valid;
    const int ff = row_ok ? f : 0;
    const int my_qrow = i0 + ff / G;
    const int my_head = g * G + ff % G;
    const int my_pos = p.q_pos0 + my_qrow;
    const int wf0 = 32 * wave;
    const bool wave_active = wf0 < rows_valid;
    const int wf1 = min(wf0 + 31, rows_valid - 1);
    const int wp_min = pos_first + wf0 / G;
    const int wp_max = pos_first + (wave_active ? wf1 : wf0) / G;
    // lane r holds the threshold of pair r (pairs past d/2 never count)
    const int my_w = lane < C::kHalf ? p.win.W[lane] : -1;

    // K: pair-chunk-major streams of cache_tokens keys, chunk c of this head =
    // 32 bytes per key; V: rows of h_kv * d bf16
    const int64_t chunk_bytes = int64_t(p.cache_tokens) * 32;
    const char* kpcm = reinterpret_cast<const char*>(p.k) + (int64_t(b) * p.h_kv + g) * C::kChunks * chunk_bytes;
    const uint32_t k_piece = uint32_t((lane & 31) * 32 + (lane >> 5) * 16);
    // V: packed 16-key blocks [d][16] of this head, ceil(cache_tokens / 16) of them
    const int n_vblk = (p.cache_tokens + 15) / 16;
    const char* vhead = reinterpret_cast<const char*>(p.v) + (int64_t(b) * p.h_kv + g) * n_vblk * int64_t(C::kVBlkBytes);

    // query fragments (B operand): row `col`, dims of half hh of every chunk
    u32x4_t qf[C::kChunks];
    {
        const uint16_t* qrow =
            p.q + ((int64_t(b) * p.n_q + my_qrow) * p.h_q + my_head) * D + hh * C::kHalf;
#pragma unroll
        for (int c = 0; c < C::kChunks; ++c) {
            u32x4_t z = {0u, 0u, 0u, 0u};
            if (row_ok) z = *reinterpret_cast<const u32x4_t*>(qrow + 8 * c);
            // an unrotated query is turned to its position here, once
            if constexpr (kRot)
                z = rope::rotate(z, rope::other_half(z, hh), hh, uint32_t(my_pos), &p.rope_rho_hi[8 * c],
                                 &p.rope_rho_lo[8 * c]);
            qf[c] = z;
        }
    }

    // ---- global -> LDS staging of the tile at key j0 into buffer `buf`.
    // K: the tile is 2 * kChunks units (chunk u / 2, 32-key block u % 2); wave w
    // loads units w, w + 8, ...: lane i reads 16 bytes of key i % 32, half i / 32,
    // so the wave's 1 KB of global memory is contiguous.  A unit whose chunk no
    // cell of the workgroup tile keeps is skipped; the last chunk is always loaded
    // because the QK of a block always multiplies it.  V: the tile's four packed
    // blocks are one contiguous run; wave w copies its kilobytes w, w + W, ...
    // Blocks past the cache's last one re-read that block (their keys are past
    // n_k and masked).
    const uint32_t ks_lds = lds_addr(&Ks[0][0]);
    const uint32_t vs_lds = lds_addr(&Vs[0][0]);
    auto tile_need = [&](int j0) __attribute__((always_inline)) -> uint32_t {
        if (!kWin) return (1u << C::kChunks) - 1u;
        const int zlo = max(0, pos_first - (j0 + kBN - 1));
        uint32_t need = 1u << (C::kChunks - 1);
#pragma unroll
        for (int c = 0; c < C::kChunks; ++c)
            if (p.win.chunk_max[c] >= zlo) need |= 1u << c;
        return need;
    };
    // Fast form for tiles wholly below n_k (all but the last): per wave unit, the
    // stream base and the first tile from which its chunk is kept (chunk c is kept in
    // the tile at j0 iff chunk_max[c] >= pos_first - j0 - 63; the thresholds are >= 0)
    // are fixed, so a tile costs one compare and one 64-bit add per load.
    const char* kbase[C::kKPerWave];
    int kfirst[C::kKPerWave];
#pragma unroll
    for (int t = 0; t < C::kKPerWave; ++t) {
        const int u = wave + C::kWaves * t;
        const int c = u >> 1;
        kbase[t] = kpcm + c * chunk_bytes + (u & 1) * 1024;
        kfirst[t] = 0;
        if (kWin && c != C::kChunks - 1) {
            const int64_t num = int64_t(pos_first) - (kBN - 1) - p.win.chunk_max[c];
            kfirst[t] = num <= 0 ? 0 : int(min(int64_t(INT32_MAX), (num + kBN - 1) / kBN));
        }
    }
    auto issue_fast = [&](int j0, int buf) __attribute__((always_inline)) -> uint32_t {
        uint32_t loaded = 0;
        const int tn = j0 / kBN;
        const int64_t koff = int64_t(j0) * 32;
        const int64_t voff = int64_t(j0) * (2 * D);
        const uint32_t kdst = ks_lds + uint32_t(buf * C::kKTile * 2);
#pragma unroll
        for (int t = 0; t < C::kKPerWave; ++t) {
            const int u = wave + C::kWaves * t;
            if (tn >= kfirst[t]) {
                load_to_lds(kbase[t] + koff, k_piece, kdst + 1024u * u);
                loaded |= 1u << t;
            }
        }
        const uint32_t vdst = vs_lds + uint32_t(buf * C::kVTile * 2);
#pragma unroll
        for (int t = 0; t < C::kVPer; ++t) {
            const int u = wave + C::kWaves * t;
            if constexpr (C::kVLoads % C::kWaves != 0)
                if (u >= C::kVLoads) break;
            load_to_lds(vhead + voff + 1024 * u, uint32_t(lane) * 16u, vdst + 1024u * u);
        }
        return loaded;
    };
    // returns the K units (bit t: unit wave + kWaves t) this wave loaded
    auto issue = [&](int j0, int buf) __attribute__((always_inline)) -> uint32_t {
        if (j0 + kBN <= p.n_k) return issue_fast(j0, buf);
        uint32_t loaded = 0;
        const uint32_t need = tile_need(j0);
        const uint32_t kdst = ks_lds + uint32_t(buf * C::kKTile * 2);
#pragma unroll
        for (int t = 0; t < C::kKPerWave; ++t) {
            const int u = wave + C::kWaves * t;  // unit = (chunk u / 2, 32-key block u % 2)
            const int c = u >> 1;
            if ((need >> c) & 1u) {
                const int jb = min(j0 + 32 * (u & 1), p.n_k - 1);
                uint32_t off = k_piece;
                if (jb + 32 > p.n_k)
                    off = min(uint32_t(lane & 31), uint32_t(p.n_k - 1 - jb)) * 32u + uint32_t(lane >> 5) * 16u;
                load_to_lds(kpcm + c * chunk_bytes + int64_t(jb) * 32, off, kdst + 1024u * u);
                loaded |= 1u << t;
            }
        }
        const uint32_t vdst = vs_lds + uint32_t(buf * C::kVTile * 2);
#pragma unroll
        for (int t = 0; t < C::kVPer; ++t) {
            const int u = wave + C::kWaves * t;
            if (u >= C::kVLoads) break;
            const int blk = min(j0 / 16 + (1024 * u) / C::kVBlkBytes, n_vblk - 1);
            load_to_lds(vhead + int64_t(blk) * C::kVBlkBytes + (1024 * u) % C::kVBlkBytes,
                        uint32_t(lane) * 16u, vdst + 1024u * u);
        }
        return loaded;
    };

    // ---- rotation at read time: each wave turns the K units it loaded, once they have
    // landed and before the barrier that publishes the tile, so each kept (key, pair) of
    // the workgroup's tile is rotated once and pruned chunks (never loaded) never are.
    // Lane l turns 4 pairs (half l / 32 of the unit's 8) of key l % 32: both components
    // from the unit's two halves, angle (block start + l % 32) * theta_r by angle
    // addition of the block start's angle (lanes 0 .. 8 kKPerWave - 1, one pair of one
    // unit each) and the offset's (the table).
    auto rotate_units = [&](int j0, int buf, uint32_t loaded) __attribute__((always_inline)) {
        loaded = __builtin_amdgcn_readfirstlane(loaded);
        if (loaded == 0u) return;
        // block-start angles of all the wave's units at once: lane 8 t + e holds pair
        // 8 c + e of unit t (c its chunk); a unit not loaded gets an unused angle
        if (lane < 8 * C::kKPerWave) {
            const int u = wave + C::kWaves * (lane >> 3);
            const float ub = rope::revolutions(uint32_t(j0 + 32 * (u & 1)), s_rho[8 * (u >> 1) + (lane & 7)]);
            s_base[wave * C::kKPerWave * 16 + 2 * lane] = __builtin_amdgcn_cosf(ub);
            s_base[wave * C::kKPerWave * 16 + 2 * lane + 1] = __builtin_amdgcn_sinf(ub);
        }
        // the wave's own LDS writes complete before its later LDS reads; the fences
        // keep the compiler from moving the reads above the writes
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // every unit's elements are read before any is rotated, so the reads' latencies
        // overlap (reading a unit that was not loaded is harmless: it is not written)
        typedef __attribute__((address_space(3))) uint64_t lds_u64;
        const int kk = lane & 31, gq = lane >> 5;
        uint64_t xv[C::kKPerWave], yv[C::kKPerWave];
#pragma unroll
        for (int t = 0; t < C::kKPerWave; ++t) {
            const int u = wave + C::kWaves * t;
            const uint32_t a0 = ks_lds + uint32_t(buf * C::kKTile * 2) + 1024u * u + uint32_t(kk * 16 + gq * 8);
            xv[t] = *(const lds_u64*)(uintptr_t)a0;
            yv[t] = *(const lds_u64*)(uintptr_t)(a0 + 512u);
        }
#pragma unroll
        for (int t = 0; t < C::kKPerWave; ++t) {
            if (!((loaded >> t) & 1u)) continue;
            const int u = wave + C::kWaves * t;
            const float* cr = &s_colcs[kk * kColStride + 2 * (8 * (u >> 1) + 4 * gq)];
            const float4 cc0 = *reinterpret_cast<const float4*>(cr);
            const float4 cc1 = *reinterpret_cast<const float4*>(cr + 4);
            const float* br = &s_base[(wave * C::kKPerWave + t) * 16 + 8 * gq];
            const float4 bb0 = *reinterpret_cast<const float4*>(br);
            const float4 bb1 = *reinterpret_cast<const float4*>(br + 4);
            const float cC[4] = {cc0.x, cc0.z, cc1.x, cc1.z}, sC[4] = {cc0.y, cc0.w, cc1.y, cc1.w};
            const float cB[4] = {bb0.x, bb0.z, bb1.x, bb1.z}, sB[4] = {bb0.y, bb0.w, bb1.y, bb1.w};
            uint32_t xo[2], yo[2];
#pragma unroll
            for (int w2 = 0; w2 < 2; ++w2) {
                const uint32_t xw = uint32_t(xv[t] >> (32 * w2)), yw = uint32_t(yv[t] >> (32 * w2));
                rope::bf16x2_t xt, yt;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int e = 2 * w2 + h;
                    const float cs = __builtin_fmaf(cB[e], cC[e], -sB[e] * sC[e]);
                    const float sn = __builtin_fmaf(sB[e], cC[e], cB[e] * sC[e]);
                    const float x = __uint_as_float(h ? (xw & 0xFFFF0000u) : (xw << 16));
                    const float y = __uint_as_float(h ? (yw & 0xFFFF0000u) : (yw << 16));
                    xt[h] = (__bf16)rope::turn(x, y, -1.f, cs, sn);
                    yt[h] = (__bf16)rope::turn(y, x, 1.f, cs, sn);
                }
                xo[w2] = __builtin_bit_cast(uint32_t, xt);
                yo[w2] = __builtin_bit_cast(uint32_t, yt);
            }
            const uint32_t a0 = ks_lds + uint32_t(buf * C::kKTile * 2) + 1024u * u + uint32_t(kk * 16 + gq * 8);
            *(lds_u64*)(uintptr_t)a0 = uint64_t(xo[0]) | (uint64_t(xo[1]) << 32);
            *(lds_u64*)(uintptr_t)(a0 + 512u) = uint64_t(yo[0]) | (uint64_t(yo[1]) << 32);
        }
        // the rotated units are complete in LDS before the workgroup barrier, and the
        // fence keeps the compiler from sinking the writes below it
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    };
    // after the barrier: no LDS read of a rotated unit moves above it
    auto rotated_acquire = [&]() __attribute__((always_inline)) {
        if constexpr (kRot) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    };

    // per-lane LDS byte bases of the fragment reads (buffer 0, block 0)
    //   K: unit (chunk c, block kb) at 1 KB * (2 c + kb), half hh, key col
    //   V: packed block q of the tile at q * kVBlkBytes, dim 32 i + col at 1 KB * i,
    //      slots 8 hh .. 8 hh + 7
    const uint32_t k_lane = ks_lds + uint32_t(hh * 512 + col * 16);
    const uint32_t v_lane = vs_lds + uint32_t(col * 32 + hh * 16);

    f32x16_t oacc[D / 32];
#pragma unroll
    for (int i = 0; i < D / 32; ++i) oacc[i] = zero16();
    float m_run = -INFINITY;  // running (possibly stale) max, log2 domain
    float m_thr = -INFINITY;  // m_run + kRescale: a tile max above it raises m_run
    float m_neg = 0.f;        // minus the max the exponentials subtract (0 while m_run = -inf)
    float l_run = 0.f;        // normaliser over this lane's keys
    const float sc = p.scale_log2;
    f32x16_t sacc[2];  // scores of the current tile (two 32-key blocks)
    u32x4_t qb;        // query dims of chunk qb_rf / 8 with the pairs below qb_rf zeroed
    int qb_rf = -1;

    auto k_block = [&](int tile, int kb) __attribute__((always_inline)) -> uint32_t {
        return k_lane + stage_off<C::kStages>(tile, C::kKTile * 2) + uint32_t(kb * 1024);
    };

    // ---- QK of a uniform tile: chunk CF with the boundary operand qb, then the
    // whole chunks above it (for the window off: CF = 0, qb = qf[0])
    auto qk_uniform = [&](int tile, auto cf_tag) __attribute__((always_inline)) {
        constexpr int CF = decltype(cf_tag)::value;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const uint32_t kr = k_block(tile, kb);
            u32x4_t kf[C::kChunks];
#pragma unroll
            for (int c = CF; c < C::kChunks; ++c) kf[c] = lds_read_b128(kr + 2048u * c);
            f32x16_t acc = mfma(kf[CF], qb, zero16());
#pragma unroll
            for (int c = CF + 1; c < C::kChunks; ++c) acc = mfma(kf[c], qf[c], acc);
            sacc[kb] = acc;
        }
    };

    // ---- QK of any tile (general path), per 32-key block
    auto qk_general = [&](int tile) __attribute__((always_inline)) {
        const int j0 = tile * kBN;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const int jb = j0 + 32 * kb;
            const uint32_t kr = k_block(tile, kb);
            u32x4_t kf[C::kChunks];
#pragma unroll
            for (int c = 0; c < C::kChunks; ++c) kf[c] = lds_read_b128(kr + 2048u * c);
            const int zhi = wp_max - jb;
            const int zlo = max(0, wp_min - (jb + 31));
            // all pairs classified at once: lane r holds W_r; bit r of `full` = pair r
            // kept in every cell of the block, of `keep` = kept in some cell
            const uint64_t full = __ballot(my_w >= zhi);
            const uint64_t keep = __ballot(my_w >= zlo);
            // lowest frequencies (largest windows) first: the first MFMA always runs
            // (pairs no cell keeps zeroed) and starts from a zero accumulator
            f32x16_t acc;
#pragma unroll
            for (int c = C::kChunks - 1; c >= 0; --c) {
                const uint32_t fc = uint32_t(full >> (8 * c)) & 0xFFu;
                if (c == C::kChunks - 1) {
                    acc = mfma(kf[c], keep_pairs(qf[c], fc), zero16());
                } else if (fc) {
                    u32x4_t q = qf[c];
                    if (fc != 0xFFu) q = keep_pairs(q, fc);
                    acc = mfma(kf[c], q, acc);
                }
            }
            // pairs whose window ends inside the block, grouped by chunk and threshold:
            // one MFMA per group, added where z <= W_r (register v holds distance
            // zbase - off(v): keep iff off(v) >= thr).  A table whose chunks share one
            // threshold (the rounded slice) needs one MFMA per partial chunk.
            const auto add_kept = [&](u32x4_t k, u32x4_t q, uint32_t pairs, int wr) __attribute__((always_inline)) {
                const f32x16_t pr = mfma(k, keep_pairs(q, pairs), zero16());
                const int thr = my_pos - jb - 4 * hh - wr;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int off = 8 * (v / 4) + (v % 4);
                    acc[v] += off >= thr ? pr[v] : 0.f;
                }
            };
            uint64_t part = keep & ~full;
            if constexpr (D == 64) {
                // chunk by chunk, the operands named at compile time: selecting them by a
                // run-time chunk and re-reading K made a general tile 2.3 times a uniform
                // one (16/16 heads, 8,191 tokens, base 1e4: 222 us, now 207; rounded slice
                // 150).  At d = 128 the eight copies cost 1-2 % from 32K tokens.
                if (part) {
#pragma unroll
                    for (int c = 0; c < C::kChunks; ++c) {
                        uint32_t pc = uint32_t(part >> (8 * c)) & 0xFFu;
                        while (pc) {
                            const int wr = __builtin_amdgcn_readlane(my_w, 8 * c + __builtin_ctz(pc));
                            const uint32_t grp = uint32_t(__ballot(my_w == wr) >> (8 * c)) & pc;
                            pc &= ~grp;
                            add_kept(kf[c], qf[c], grp, wr);
                        }
                    }
                }
            } else {
                while (part) {
                    const int r = __builtin_ctzll(part);
                    const int c = r >> 3;
                    const int wr = p.win.W[r];
                    const uint64_t grp = __ballot(my_w == wr) & part & (0xFFull << (8 * c));
                    part &= ~grp;
                    u32x4_t qc = qf[0];
#pragma unroll
                    for (int cc = 1; cc < C::kChunks; ++cc)
                        if (cc == c) qc = qf[cc];
                    add_kept(lds_read_b128(kr + 2048u * c), qc, uint32_t(grp >> (8 * c)), wr);
                }
            }
            sacc[kb] = acc;
        }
    };

    // ---- causal mask and key bound (only tiles that reach the diagonal or n_k),
    // then the online softmax over the tile (lane = query row; the two lane halves
    // hold disjoint keys), then PV.  One rescale check per tile; the exponentials
    // are branch-free.
    auto softmax_pv = [&](int tile) __attribute__((always_inline)) {
        const int j0 = tile * kBN;
        if (wp_min - (j0 + kBN - 1) < 0 || j0 + kBN > p.n_k) {
            // cell kept iff off <= lim = min(distance base, last key - block start): the
            // score goes through min(s, +inf) if kept, min(s, -inf) if not, the sign bit of
            // lim - off choosing the infinity.  (Written with per-cell compares, the 32
            // lane masks of a tile were all live at once and pushed the kernel's scalar
            // registers into spills.)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                const int jb = j0 + 32 * kb;
                const int lim = min(my_pos - jb, p.n_k - 1 - jb) - 4 * hh;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int off = 8 * (v / 4) + (v % 4);
                    const uint32_t inf = (uint32_t(lim - off) & 0x80000000u) | 0x7F800000u;
                    sacc[kb][v] = fminf(sacc[kb][v], __uint_as_float(inf));
                }
            }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sacc[kb][v]);
        // The two lane halves of a row hold the same m_run and sc > 0, so some lane's half
        // max passes the threshold exactly when some lane's row max does: the halves
        // exchange their maxima only when the running max is raised.
        if (__any(mx * sc > m_thr)) {
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m_run, mx * sc);
            const float m_use = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = exp2_fast(m_run - m_use);
            m_run = m_new;
            m_thr = m_new + kRescale;
            m_neg = -m_use;
            l_run *= alpha;
#pragma unroll
            for (int i = 0; i < D / 32; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) oacc[i][v] *= alpha;
        }
        const uint32_t vb = v_lane + stage_off<C::kStages>(tile, C::kVTile * 2);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            u32x4_t pb[2];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float a = exp2_fast(__builtin_fmaf(sacc[kb][8 * ks + 2 * t], sc, m_neg));
                    const float c2 = exp2_fast(__builtin_fmaf(sacc[kb][8 * ks + 2 * t + 1], sc, m_neg));
                    l_run += a;
                    l_run += c2;
                    bf16x2_t two;
                    two[0] = (__bf16)a;
                    two[1] = (__bf16)c2;
                    pb[ks][t] = __builtin_bit_cast(uint32_t, two);
                }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int i = 0; i < D / 32; ++i)
                    oacc[i] = mfma(lds_read_b128(vb + uint32_t((2 * kb + ks) * C::kVBlkBytes + 1024 * i)),
                                   pb[ks], oacc[i]);
        }
    };

    // The V slots of keys at or past n_k in the LDS copy of a tile that crosses n_k
    // (only the last tile can) are set to zero by the whole workgroup before any
    // wave reads them: the cache past n_k need not hold finite values, and a zero
    // probability does not cancel a NaN in the matrix product.
    auto zero_v_tail = [&](int u) __attribute__((always_inline)) {
        const int j0 = u * kBN;
        if (j0 + kBN <= p.n_k) return;
        uint16_t* vt = &Vs[u % C::kStages][0];
        for (int row = tid; row < 4 * D; row += C::kThreads) {  // row = block * D + dim
            const int kblk = j0 + 16 * (row / D);
#pragma unroll
            for (int sl = 0; sl < 16; ++sl) {
                const int key = kblk + 8 * ((sl & 7) >> 2) + 4 * (sl >> 3) + (sl & 3);
                if (key >= p.n_k) vt[row * 16 + sl] = 0;
            }
        }
        __syncthreads();
    };

    const int n_tiles = (key_end + kBN - 1) / kBN;
    auto active = [&](int tile) __attribute__((always_inline)) { return wave_active && wp_max >= tile * kBN; };
    // one tile: stage the next, compute this one (if the wave has rows there),
    // await this wave's loads of the next tile (and rotate them, for unrotated
    // caches), barrier
    auto run_tile = [&](int u, auto&& qk) __attribute__((always_inline)) {
        uint32_t loaded = 0;
        if (u + 1 < n_tiles) loaded = issue((u + 1) * kBN, (u + 1) % C::kStages);
        zero_v_tail(u);
        if (active(u)) {
            qk(u);
            softmax_pv(u);
        }
        vm_wait();
        if constexpr (kRot) rotate_units((u + 1) * kBN, (u + 1) % C::kStages, loaded);
        barrier();
        rotated_acquire();
    };

    if constexpr (kRot) {
        for (int idx = tid; idx < 32 * C::kHalf; idx += C::kThreads) {
            const int kk = idx / C::kHalf, r = idx % C::kHalf;
            const float u = rope::revolutions(uint32_t(kk), make_uint2(p.rope_rho_hi[r], p.rope_rho_lo[r]));
            s_colcs[kk * kColStride + 2 * r] = __builtin_amdgcn_cosf(u);
            s_colcs[kk * kColStride + 2 * r + 1] = __builtin_amdgcn_sinf(u);
        }
        if (tid < C::kHalf) s_rho[tid] = make_uint2(p.rope_rho_hi[tid], p.rope_rho_lo[tid]);
        __syncthreads();
    }
    {
        const uint32_t loaded = issue(0, 0);
        vm_wait();
        if constexpr (kRot) rotate_units(0, 0, loaded);
        barrier();
        rotated_acquire();
    }

    if constexpr (!kWin) {
        // window off: every tile is the full contraction
        qb = qf[0];
        for (int u = 0; u < n_tiles; ++u)
            run_tile(u, [&](int t) __attribute__((always_inline)) {
                qk_uniform(t, std::integral_constant<int, 0>{});
            });
    } else {
    // Each wave walks the tiles in runs; every tile ends with one barrier on every
    // wave, whichever loop runs it.
    constexpr int kGeneral = 64;  // mode of a general-path tile (chunk counts are 0..7)
    int u = 0;
    while (u < n_tiles) {
        int mode, seg_end;
        if (!active(u)) {
            mode = -1;  // the wave's rows all precede this tile and every later one
            seg_end = n_tiles;
        } else {
            mode = kGeneral;
            seg_end = u + 1;
            if (p.mono) {
                const int zhi = wp_max - u * kBN;                      // largest distance of the tile
                const int zlo = max(0, wp_min - (u * kBN + kBN - 1));  // smallest
                const uint64_t full = __ballot(my_w >= zhi);
                const uint64_t keep = __ballot(my_w >= zlo);
                if (full == keep) {
                    // uniform: kept pairs r >= rf (rf = d/2: none, every score is 0; a
                    // window that ends before the farthest key, base 1e4 at 20,000 tokens,
                    // then has no general tile but those a threshold lies in: 4,000 rows
                    // against 20,000 keys, 16/16 heads, 515 -> 345 us).  The
                    // run lasts while the next threshold below, W[rf - 1], stays under the
                    // tile's smallest distance: wp_min - 64 u' - 63 > W[rf - 1].
                    const int rf = __popcll(~full & (~0ull >> (64 - C::kHalf)));
                    seg_end = n_tiles;
                    if (rf > 0) {
                        const int wlow = p.win.W[rf - 1];
                        const int64_t lim = (int64_t(wp_min) - kBN - wlow) / kBN + 1;
                        seg_end = int(max(int64_t(u) + 1, min(lim, int64_t(n_tiles))));
                    }
                    mode = min(rf >> 3, C::kChunks - 1);
                    if (rf != qb_rf) {
                        qb_rf = rf;
                        u32x4_t qs = qf[0];
#pragma unroll
                        for (int cc = 1; cc < C::kChunks; ++cc)
                            if (cc == mode) qs = qf[cc];
                        // (from rf, not from `full`: 4,096 rows against 2^20 keys 44.04 -> 43.78 ms)
                        qb = keep_pairs(qs, rf < C::kHalf ? (0xFFu << (rf & 7)) & 0xFFu : 0u);
                    }
                }
            }
        }
        switch (mode) {
#define ATF_UNIFORM_RUN(CFV)                                                                    \
    case CFV:                                                                                   \
        if constexpr (CFV < C::kChunks) {                                                       \
            for (; u < seg_end; ++u)                                                            \
                run_tile(u, [&](int t) __attribute__((always_inline)) { qk_uniform(t, std::integral_constant<int, CFV>{}); }); \
        } else { /* not reached: mode < d/16 */                                                 \
            run_tile(u, [&](int t) __attribute__((always_inline)) { qk_general(t); });                                         \
            ++u;                                                                                \
        }                                                                                       \
        break;
            ATF_UNIFORM_RUN(0)
            ATF_UNIFORM_RUN(1)
            ATF_UNIFORM_RUN(2)
            ATF_UNIFORM_RUN(3)
            ATF_UNIFORM_RUN(4)
            ATF_UNIFORM_RUN(5)
            ATF_UNIFORM_RUN(6)
            ATF_UNIFORM_RUN(7)
#undef ATF_UNIFORM_RUN
            case kGeneral:
                run_tile(u, [&](int t) __attribute__((always_inline)) { qk_general(t); });
                ++u;
                break;
            default:  // idle: keep the barrier count
                for (; u < seg_end; ++u) {
                    uint32_t loaded = 0;
                    if (u + 1 < n_tiles) loaded = issue((u + 1) * kBN, (u + 1) % C::kStages);
                    zero_v_tail(u);
                    vm_wait();
                    if constexpr (kRot) rotate_units((u + 1) * kBN, (u + 1) % C::kStages, loaded);
                    barrier();
                    rotated_acquire();
                }
                break;
        }
    }
    }

    if (!wave_active) return;
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (!row_ok) return;
    const float inv = 1.0f / l_tot;
    uint16_t* orow = p.o + ((int64_t(b) * p.n_q + my_qrow) * p.h_q + my_head) * D;
#pragma unroll
    for (int i = 0; i < D / 32; ++i) {
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
            typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
            bf16x4_t out;
#pragma unroll
            for (int t = 0; t < 4; ++t) out[t] = (__bf16)(oacc[i][4 * grp + t] * inv);
            *reinterpret_cast<bf16x4_t*>(orow + 32 * i + 8 * grp + 4 * hh) = out;
        }
    }
    if (hh == 0)
        p.lse[(int64_t(b) * p.h_q + my_head) * p.n_q + my_qrow] =
            m_run * 0.69314718055994531f + logf(l_tot);
}

// ---- Calls with few rows: the keys of a row block split over the waves of its workgroup.
//
// prefill_kernel gives a CU 256 rows (128 at d = 64), so a call with few rows (an
// appended turn, a short prompt) leaves most of the chip idle while a few workgroups
// walk all the keys.  Here a workgroup owns ONE block of 32 rows and its S waves
// take the 32-key blocks u = wave, wave + S, ..., each with its own softmax state; the
// states are merged in LDS at the end, in wave order.  The waves share nothing while
// they stream, so there is no LDS staging and no barrier: operand fragments are 16-byte
// loads from the caches into registers (the decode kernel's form), a block's V issued
// before its QK and the next block's K after it.
//
// What bounds it: every row block reads its keys through L1 by itself (8 to 16 KB per 32
// keys against 64 B per clock), which costs more than the matrix work once every CU is
// full; a row costs about 1.5 times what it does in prefill_kernel, and `short_split`
// takes this kernel only where the idle CUs cost more.  Chunks that no cell keeps are not
// loaded (a fixed number of loads, the pruned ones out of a buffer's range, took 1.3 times
// as long with every CU full).  Measured, windowed, prefill_kernel -> this one: 300 rows
// against 65,836 keys (28 heads on 4, d = 128) 1310 -> 508 us; 16 rows against 20,000 keys
// 321 -> 89 us, at d = 64 239 -> 54 us; a 1,024-token prompt (14 heads on 2, d = 64)
// 28.8 -> 11.4 us.
// Slower: K staged through a per-wave LDS ring (501 us at the 300 rows), two row blocks
// sharing staged tiles of 128 keys with a barrier each (489 us; 184 us at the 16 rows),
// 64 rows per wave with 512 registers (1450 us, spilled).
//
// Rows are grouped as in prefill_kernel (the same position tiles, the same 32 rows to a
// wave) and a block of keys belongs to the same wave whatever n_q is, so chunks of a
// prefill that take this kernel with the same S agree bit for bit.
//
// kRot: queries rotated as they are loaded, the kept chunks of a block's keys in
// registers before their products; angles as in the decode kernel (the block's first
// position, evaluated by lane r for pair r, plus the offset's table entry).
template <int D, bool kWin, bool kRot, int S>
__global__ __launch_bounds__(S * 64, 2) void prefill_short_kernel(
    const std::conditional_t<kRot, PrefillRotParams, PrefillParams> p) {
    constexpr int kChunks = D / 16;
    constexpr int kHalf = D / 2;
    constexpr int kDB = D / 32;
    constexpr int kBlk = 32;  // keys per step of a wave
    constexpr int kVBlkBytes = D * 32;
    constexpr int kParts = Cfg<D, kWin>::kRows / 32;  // row blocks per position tile
    constexpr int kCStride = D + 4;
    __shared__ float red_m[S][32];
    __shared__ float red_l[S][32];
    // While the waves stream: the queries, then (rotation) the (cos, sin) of col * theta_r
    // for the 32 key offsets of a block, rows padded by 16 bytes, and per wave those of the
    // block's first position * theta_r.  Afterwards: the waves' weighted outputs.
    constexpr int kTables = 16 * D + (kRot ? 32 * kCStride + S * D : 0);  // floats
    constexpr int kMerge = S * 32 * (D + 1);
    __shared__ __attribute__((aligned(16))) float shared[kTables > kMerge ? kTables : kMerge];
    uint16_t* const Qs = reinterpret_cast<uint16_t*>(shared);
    float* const s_colcs = shared + 16 * D;
    float* const s_blkcs = s_colcs + 32 * kCStride;
    float* const red_o = shared;  // [S][32][D + 1]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31;
    const int hh = lane >> 5;

    // block -> (position tile, row block, kv head, batch), late rows first; heads vary
    // fastest, as in prefill_kernel, so that each XCD keeps to fixed KV heads
    const int per_tile = p.h_kv * p.batch;
    const int rem = blockIdx.x % per_tile;
    const int tb = blockIdx.x / per_tile;
    const int qt = p.n_qtiles - 1 - tb / kParts;
    const int row0 = 32 * (kParts - 1 - tb % kParts);
    const int g = rem % p.h_kv;
    const int b = rem / p.h_kv;
    const int G = p.group;

    const int i0 = qt * p.pos_per_tile;
    const int rows_valid = min(p.pos_per_tile, p.n_q - i0) * G;
    if (row0 >= rows_valid) return;  // the whole workgroup
    const int pos0 = p.q_pos0 + i0;
    const int my_pos = pos0 + min(row0 + col, rows_valid - 1) / G;
    const int wp_min = pos0 + row0 / G;
    const int wp_max = pos0 + min(row0 + 31, rows_valid - 1) / G;
    const int n_blk = __builtin_amdgcn_readfirstlane((min(p.n_k, wp_max + 1) + kBlk - 1) / kBlk);
    const int my_w = lane < kHalf ? p.win.W[lane] : -1;

    const int64_t chunk_bytes = int64_t(p.cache_tokens) * 32;
    const char* kpcm = reinterpret_cast<const char*>(p.k) + (int64_t(b) * p.h_kv + g) * kChunks * chunk_bytes;
    const int n_vblk = (p.cache_tokens + 15) / 16;
    const char* vhead = reinterpret_cast<const char*>(p.v) + (int64_t(b) * p.h_kv + g) * n_vblk * int64_t(kVBlkBytes);
    const uint32_t piece = uint32_t(col * 32 + hh * 16);

    // The row block's queries: chunk c, half h, row r at 1024 c + 512 h + 16 r (each wave
    // writes whole chunks, lane = (half, row))
    for (int e = tid; e < kChunks * 64; e += S * 64) {
        const int c = __builtin_amdgcn_readfirstlane(e >> 6), fr = row0 + col;
        u32x4_t z = {0u, 0u, 0u, 0u};
        if (fr < rows_valid)
            z = *reinterpret_cast<const u32x4_t*>(p.q + ((int64_t(b) * p.n_q + i0 + fr / G) * p.h_q + g * G + fr % G) * D +
                                                  hh * kHalf + 8 * c);
        if constexpr (kRot)
            z = rope::rotate(z, rope::other_half(z, hh), hh, uint32_t(my_pos), &p.rope_rho_hi[8 * c],
                             &p.rope_rho_lo[8 * c]);
        *reinterpret_cast<u32x4_t*>(&Qs[8 * e]) = z;
    }
    uint2 my_rho = make_uint2(0u, 0u);  // lane r: the rotation fraction of pair r
    if constexpr (kRot) {
        for (int e = tid; e < 32 * kHalf; e += S * 64) {
            const int kk = e / kHalf, r = e % kHalf;
            const float u = rope::revolutions(uint32_t(kk), make_uint2(p.rope_rho_hi[r], p.rope_rho_lo[r]));
            s_colcs[kk * kCStride + 2 * r] = __builtin_amdgcn_cosf(u);
            s_colcs[kk * kCStride + 2 * r + 1] = __builtin_amdgcn_sinf(u);
        }
        if (lane < kHalf) my_rho = make_uint2(p.rope_rho_hi[lane], p.rope_rho_lo[lane]);
    }
    __syncthreads();
    const uint32_t q_lane = lds_addr(Qs) + uint32_t(hh * 512 + col * 16);
    auto q_frag = [&](int c) __attribute__((always_inline)) { return lds_read_b128(q_lane + 1024u * c); };

    f32x16_t oacc[kDB];
#pragma unroll
    for (int i = 0; i < kDB; ++i) oacc[i] = zero16();
    float m_run = -INFINITY, m_thr = -INFINITY, m_neg = 0.f, l_run = 0.f;
    const float sc = p.scale_log2;

    // the window's classification of block u: `full` = pairs kept in every cell, `keep` =
    // pairs kept in some cell (lane r holds W_r)
    auto classify = [&](int u, uint64_t& full, uint64_t& keep) __attribute__((always_inline)) {
        if constexpr (kWin) {
            full = __ballot(my_w >= wp_max - u * kBlk);
            keep = __ballot(my_w >= max(0, wp_min - (u * kBlk + kBlk - 1)));
        } else {
            full = keep = ~0ull;
        }
    };
    // K fragments of block u (A operand: key 32 u + col, half hh of every kept chunk; the
    // last chunk is always multiplied).  One scalar base per block and fixed 32-bit lane
    // offsets (the host checks that the chunks' span fits); keys past n_k - 1 read that key
    // and are masked.
    u32x4_t kf[kChunks];
    uint32_t k_off[kChunks];
#pragma unroll
    for (int c = 0; c < kChunks; ++c) k_off[c] = uint32_t(c) * uint32_t(chunk_bytes) + piece;
    auto load_k = [&](int u, uint64_t keep) __attribute__((always_inline)) {
        const int jb = u * kBlk;
        const char* base = kpcm + int64_t(jb) * 32;
        const uint32_t back = jb + kBlk <= p.n_k ? 0u : uint32_t(max(0, col - (p.n_k - 1 - jb))) * 32u;
#pragma unroll
        for (int c = 0; c < kChunks; ++c)
            if (!kWin || c == kChunks - 1 || ((keep >> (8 * c)) & 0xFFull))
                kf[c] = *reinterpret_cast<const u32x4_t*>(base + (k_off[c] - back));
    };

    // query operands with the dims of the pairs outside qf_full zeroed: remade where a
    // threshold enters or leaves the block's distances
    uint64_t full = 0, keep = 0, qf_full = kWin ? 0 : ~0ull;
    u32x4_t qf[kChunks];
#pragma unroll
    for (int c = 0; c < kChunks; ++c) qf[c] = kWin ? u32x4_t{0u, 0u, 0u, 0u} : q_frag(c);
    if (wave < n_blk) {
        classify(wave, full, keep);
        load_k(wave, keep);
    }
    for (int u = wave; u < n_blk; u += S) {
        const int jb = u * kBlk;
        // V^T fragments (A operand: dim 32 i + col, half hh of each 16-token block; blocks
        // past the last key re-read the last block and are zeroed below)
        u32x4_t vf[2][kDB];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const char* vb = vhead + int64_t(min(2 * u + ks, (p.n_k - 1) / 16)) * kVBlkBytes;
#pragma unroll
            for (int i = 0; i < kDB; ++i) vf[ks][i] = *reinterpret_cast<const u32x4_t*>(vb + 1024 * i + piece);
        }
        if constexpr (kRot) {
            const float ub = rope::revolutions(uint32_t(jb), my_rho);
            float* const blk = &s_blkcs[wave * D];
            if (lane < kHalf) {
                blk[2 * lane] = __builtin_amdgcn_cosf(ub);
                blk[2 * lane + 1] = __builtin_amdgcn_sinf(ub);
            }
            // the wave's own LDS writes complete before its later LDS reads; the fences keep
            // the compiler from moving the reads above the writes
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int c = 0; c < kChunks; ++c) {
                if (!kWin || c == kChunks - 1 || ((keep >> (8 * c)) & 0xFFull))
                    kf[c] = rope::rotate_block(kf[c], hh, &s_colcs[col * kCStride + 16 * c], blk + 16 * c);
                __builtin_amdgcn_sched_barrier(0);  // one chunk's angles at a time in registers
            }
        }
        f32x16_t sacc;  // QK, lowest frequencies first
        if constexpr (kWin) {
            if (full != qf_full) {
                qf_full = full;
#pragma unroll
                for (int c = 0; c < kChunks; ++c)
                    qf[c] = keep_pairs(q_frag(c), uint32_t(full >> (8 * c)) & 0xFFu);
            }
        }
#pragma unroll
        for (int c = kChunks - 1; c >= 0; --c) {
            if (c == kChunks - 1)
                sacc = mfma(kf[c], qf[c], zero16());
            else if (!kWin || ((full >> (8 * c)) & 0xFFull))
                sacc = mfma(kf[c], qf[c], sacc);
        }
        if constexpr (kWin) {
            // pairs whose window ends inside the block, grouped by chunk and threshold: one
            // MFMA per group, added where z <= W_r
            uint64_t part = keep & ~full;
            while (part) {
                const int r = __builtin_ctzll(part);
                const int c = r >> 3;
                const int wr = __builtin_amdgcn_readlane(my_w, r);
                const uint64_t grp = __ballot(my_w == wr) & part & (0xFFull << (8 * c));
                part &= ~grp;
                u32x4_t kc = kf[0];
#pragma unroll
                for (int cc = 1; cc < kChunks; ++cc)
                    if (cc == c) kc = kf[cc];
                const f32x16_t pr = mfma(kc, keep_pairs(q_frag(c), uint32_t(grp >> (8 * c))), zero16());
                const int thr = my_pos - jb - 4 * hh - wr;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int off = 8 * (v / 4) + (v % 4);
                    sacc[v] += off >= thr ? pr[v] : 0.f;
                }
            }
        }
        {
            // the wave's next block (past its last one: this block again, unused)
            const int un = u + S < n_blk ? u + S : u;
            classify(un, full, keep);
            load_k(un, keep);
        }
        if (jb + kBlk > p.n_k) {
            // V slots of keys at or past n_k: zero (the cache there may hold anything, and a
            // zero probability does not cancel a NaN in the matrix product)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const int lim = p.n_k - jb - 16 * ks - 4 * hh;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int e0 = 2 * t, e1 = 2 * t + 1;
                    const uint32_t m = (8 * (e0 / 4) + e0 % 4 < lim ? 0x0000FFFFu : 0u) |
                                       (8 * (e1 / 4) + e1 % 4 < lim ? 0xFFFF0000u : 0u);
#pragma unroll
                    for (int i = 0; i < kDB; ++i) vf[ks][i][t] &= m;
                }
            }
        }
        if (wp_min < jb + kBlk - 1 || jb + kBlk > p.n_k) {
            // cell kept iff off <= lim; see softmax_pv of prefill_kernel
            const int lim = min(my_pos - jb, p.n_k - 1 - jb) - 4 * hh;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int off = 8 * (v / 4) + (v % 4);
                const uint32_t inf = (uint32_t(lim - off) & 0x80000000u) | 0x7F800000u;
                sacc[v] = fminf(sacc[v], __uint_as_float(inf));
            }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sacc[v]);
        if (__any(mx * sc > m_thr)) {
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m_run, mx * sc);
            const float m_use = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = exp2_fast(m_run - m_use);
            m_run = m_new;
            m_thr = m_new + kRescale;
            m_neg = -m_use;
            l_run *= alpha;
#pragma unroll
            for (int i = 0; i < kDB; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) oacc[i][v] *= alpha;
        }
        u32x4_t pb[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float a = exp2_fast(__builtin_fmaf(sacc[8 * ks + 2 * t], sc, m_neg));
                const float c2 = exp2_fast(__builtin_fmaf(sacc[8 * ks + 2 * t + 1], sc, m_neg));
                l_run += a;
                l_run += c2;
                bf16x2_t two;
                two[0] = (__bf16)a;
                two[1] = (__bf16)c2;
                pb[ks][t] = __builtin_bit_cast(uint32_t, two);
            }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < kDB; ++i) oacc[i] = mfma(vf[ks][i], pb[ks], oacc[i]);
    }

    // ---- merge the waves' states in wave order: weights 2^(m_w - M) from all maxima, each
    // wave's weighted output in an LDS slab of its own, then S values summed per output
    const float l_lane = l_run + __shfl_xor(l_run, 32);
    if (hh == 0) {
        red_m[wave][col] = m_run;
        red_l[wave][col] = l_lane;
    }
    __syncthreads();
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < S; ++w) M = fmaxf(M, red_m[w][col]);
    const float wt = m_run == -INFINITY ? 0.f : exp2_fast(m_run - M);
#pragma unroll
    for (int i = 0; i < kDB; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            red_o[(32 * wave + col) * (D + 1) + 32 * i + 8 * (v / 4) + 4 * hh + (v % 4)] = oacc[i][v] * wt;
    __syncthreads();
    for (int e = tid; e < 32 * (D / 8); e += S * 64) {
        const int r = e / (D / 8), x0 = 8 * (e % (D / 8));
        const int fr = row0 + r;
        if (fr >= rows_valid) break;
        float Mr = -INFINITY;
#pragma unroll
        for (int w = 0; w < S; ++w) Mr = fmaxf(Mr, red_m[w][r]);
        float L = 0.f;
#pragma unroll
        for (int w = 0; w < S; ++w)
            // (a wave without a maximum: 0, or NaN if its scores are NaN)
            L += red_m[w][r] == -INFINITY ? red_l[w][r] : red_l[w][r] * exp2_fast(red_m[w][r] - Mr);
        const float inv = 1.0f / L;
        u32x4_t out;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            bf16x2_t two;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float a = 0.f;
#pragma unroll
                for (int w = 0; w < S; ++w) a += red_o[(32 * w + r) * (D + 1) + x0 + 2 * t + h];
                two[h] = (__bf16)(a * inv);
            }
            out[t] = __builtin_bit_cast(uint32_t, two);
        }
        const int qrow = i0 + fr / G, head = g * G + fr % G;
        *reinterpret_cast<u32x4_t*>(p.o + ((int64_t(b) * p.n_q + qrow) * p.h_q + head) * D + x0) = out;
        if (x0 == 0) p.lse[(int64_t(b) * p.h_q + head) * p.n_q + qrow] = Mr * 0.69314718055994531f + logf(L);
    }
}

// Tile geometry and the uniform-run test, shared by both launchers.
template <class P>
hipError_t prepare(P& p, int head_dim, unsigned* blocks, bool* window_on) {
    // the window is off when no threshold is below the largest possible distance;
    // the uniform-run path needs thresholds non-decreasing in r
    const int64_t max_dist = int64_t(p.q_pos0) + p.n_q - 1;
    bool on = false;
    for (int r = 0; r < head_dim / 2; ++r)
        if (int64_t(p.win.W[r]) < max_dist) on = true;
    bool mono = true;
    for (int r = 1; r < head_dim / 2; ++r)
        if (p.win.W[r] < p.win.W[r - 1]) mono = false;
    p.mono = mono ? 1 : 0;
    const int rows = head_dim == 64 ? (on ? Cfg<64, true>::kRows : Cfg<64, false>::kRows)
                                    : (on ? Cfg<128, true>::kRows : Cfg<128, false>::kRows);
    if (p.group < 1 || p.group > rows) return hipErrorInvalidValue;
    p.pos_per_tile = rows / p.group;
    p.n_qtiles = (p.n_q + p.pos_per_tile - 1) / p.pos_per_tile;
    const int64_t n = int64_t(p.n_qtiles) * p.h_kv * p.batch;
    if (n <= 0 || n > 0x7fffffff) return hipErrorInvalidConfiguration;
    *blocks = unsigned(n);
    *window_on = on;
    (void)hipGetLastError();
    return hipSuccess;
}

// Waves per row block of prefill_short_kernel for this call, or 0 for prefill_kernel.
//
// prefill_kernel takes as long as its longest row as long as its workgroups (`blocks` of
// them) do not fill the chip; the short kernel takes as long as the keys of all its row
// blocks together.  So the line lies on x = blocks * (mean keys of a row / keys of the
// longest row): the short kernel's gain, prefill_kernel's time over its own, falls with x
// and passes 1 at (measured over 28/4, 24/8 (d = 128), 14/2 and 16/16 heads (d = 64), 64
// to 5,000 rows, 512 to 40,000 keys)
//   d = 128, windowed: 1.30 at x = 97..116, 1.04-1.18 at 132..145, 0.93-1.06 at 146..173
//   d = 128, off:      1.17-1.18 at 98..116, 0.96-1.09 at 120..132, 0.82-0.95 at 146..173
//   d = 64, windowed (128-row workgroups): 1.26 at 241, 1.23-1.29 at 278..320, 0.92-1.07 at
//   362..402
//   d = 64, off: 1.43 at 139, 1.28 at 160, 1.06-1.16 at 181, 0.93-0.98 at 201..228
// and where keys are rotated as they are read (every row block turns its own keys)
//   d = 128: windowed 1.29-1.55 at 52..63, 0.80-1.02 at 84..98; off 1.03-1.11 at 52..58,
//   0.79-0.90 at 67..72;  d = 64: windowed 1.14-1.63 at 167..200, 0.90-1.03 at 223..241;
//   off 1.05-1.19 at 78..84, 0.84-1.04 at 96..112
// Eight waves instead of four halve the row block's time while every row block has a CU
// to itself (8 waves of its registers fill one): 256 row blocks or fewer (300 rows of
// 24/8 heads against 8,000 keys 64 -> 49 us; 64 rows against 8,000 keys 58 -> 43 us).
// Below about 4,096 keys the merge of the longer list of states takes the gain back (512
// keys: equal).
//
// That holds while the short kernel is bound by its row blocks' own work.  Short prompts are
// bound by what a row block costs before and after its few keys, and then it stops gaining at
// 0.2 to 0.5 of the limit (counted in row blocks, which a call with part tiles has fewer of):
// 8 prompts of 290 tokens of 24/8 heads 20.9 -> 29.0 us, 32 of 48 of 28/4 14.3 -> 22.8, 4 of
// 468 of 32/4 without a window 20.9 -> 28.3, 32 of 160 of 16/1 heads of d = 64 14.1 -> 18.9;
// rotating 16 of 58 of 32/4 17.3 -> 21.9.  From 384 keys on (1,024 without a window, 640 at d
// = 64, rotating 128 and 384) the limit stands; between, a line.
// And where the caches of the batch's entries pass the 256 MB last-level cache, row blocks of
// one entry that do not run at once read its keys from memory again each: 16 x 117 rows against
// 11,166 keys of 16/16 heads of d = 64 (1,024 row blocks) 189 -> 285, but 6 x 132 against 26,240
// of 24/8 (624) 584 -> 489; past 1 GB also where the limit is near: 32 x 9 against 27,936 of 32/4
// (384 row blocks) 441 -> 609, but 16 x 22 against 38,656 half the time.
int short_split(const PrefillParams& p, int head_dim, bool window_on, bool rotate, int64_t blocks) {
    // the short kernel's lane offsets cover all chunks of a token's stream in 32 bits
    if (int64_t(p.cache_tokens) * head_dim * 2 > int64_t(UINT32_MAX)) return 0;
    const int64_t longest = std::min<int64_t>(p.n_k, int64_t(p.q_pos0) + p.n_q);
    const int64_t shortest = std::min<int64_t>(p.n_k, int64_t(p.q_pos0) + 1);
    const int64_t mean = (shortest + longest) / 2;
    const int64_t limit = head_dim == 64 ? (window_on ? (rotate ? 192 : 320) : (rotate ? 80 : 184))
                                         : (rotate ? (window_on ? 64 : 56) : (window_on ? 132 : 120));
    if (blocks * mean > limit * longest) return 0;
    const int64_t per = head_dim == 64 && window_on ? 4 : 8;  // row blocks of a full workgroup of prefill_kernel
    const auto parts = [&](int64_t positions) { return (positions * p.group + 31) / 32; };
    const int64_t entries = int64_t(p.batch) * p.h_kv;
    const int64_t row_blocks = entries * (p.n_q / p.pos_per_tile * parts(p.pos_per_tile) + parts(p.n_q % p.pos_per_tile));
    const int64_t long_from = rotate ? (head_dim == 64 ? 384 : 128) : head_dim == 64 ? 640 : window_on ? 384 : 1024;
    const int64_t tenths = rotate ? 5 : head_dim == 128 && window_on ? 2 : 3;
    if (longest < long_from && 10 * row_blocks * mean * long_from >
                                   per * limit * longest * (tenths * long_from + (10 - tenths) * longest))
        return 0;
    if (rotate || row_blocks <= 256) return blocks * per <= 256 && longest >= 4096 ? 8 : 4;
    const bool many = row_blocks > (window_on ? 768 : head_dim == 64 ? 640 : 512);
    if (many || 10 * blocks * mean > 9 * limit * longest) {
        int64_t kept = 0;  // (key, pair) terms of the last row
        for (int r = 0; r < head_dim / 2; ++r) kept += std::min<int64_t>(p.win.W[r], longest);
        if (entries * (4 * kept + 2 * head_dim * longest) > int64_t(many ? 256 : 1024) << 20) return 0;
    }
    return 4;
}

template <int D, bool kWin, bool kRot, class P>
hipError_t launch_short(const P& p, int64_t blocks, int S, hipStream_t stream) {
    const int64_t n = blocks * (Cfg<D, kWin>::kRows / 32);
    if (n > 0x7fffffff) return hipErrorInvalidConfiguration;
    if (S == 8)
        hipLaunchKernelGGL((prefill_short_kernel<D, kWin, kRot, 8>), dim3(unsigned(n)), dim3(512), 0, stream, p);
    else
        hipLaunchKernelGGL((prefill_short_kernel<D, kWin, kRot, 4>), dim3(unsigned(n)), dim3(256), 0, stream, p);
    return hipGetLastError();
}

template <int D, bool kRot, class P>
hipError_t launch_d(const P& p, unsigned blocks, bool window_on, hipStream_t stream) {
    const int split = short_split(p, D, window_on, kRot, blocks);
    if (split)
        return window_on ? launch_short<D, true, kRot>(p, blocks, split, stream)
                         : launch_short<D, false, kRot>(p, blocks, split, stream);
    constexpr unsigned kLdsOn = kRot ? RotLds<D, true>::kBytes : 0u;
    constexpr unsigned kLdsOff = kRot ? RotLds<D, false>::kBytes : 0u;
    if (window_on)
        hipLaunchKernelGGL((prefill_kernel<D, true, kRot>), dim3(blocks), dim3(Cfg<D, true>::kThreads),
                           kLdsOn, stream, p);
    else
        hipLaunchKernelGGL((prefill_kernel<D, false, kRot>), dim3(blocks),
                           dim3(Cfg<D, false>::kThreads), kLdsOff, stream, p);
    return hipGetLastError();
}

}  // namespace

int32_t prefill_waves(int32_t batch, int32_t n_q, int32_t n_k, int32_t q_pos0, int32_t h_kv, int32_t group,
                      int32_t cache_tokens, const int32_t* thresholds, int32_t head_dim, bool rotate) {
    PrefillParams p{};
    p.batch = batch;
    p.n_q = n_q;
    p.n_k = n_k;
    p.q_pos0 = q_pos0;
    p.h_kv = h_kv;
    p.group = group;
    p.cache_tokens = cache_tokens;
    std::copy_n(thresholds, head_dim / 2, p.win.W);
    unsigned blocks = 0;
    bool window_on = false;
    if (prepare(p, head_dim, &blocks, &window_on) != hipSuccess) return -1;
    return short_split(p, head_dim, window_on, rotate, blocks);
}

hipError_t launch_prefill(const PrefillParams& p_in, int head_dim, hipStream_t stream) {
    PrefillParams p = p_in;
    unsigned blocks = 0;
    bool window_on = false;
    const hipError_t e = prepare(p, head_dim, &blocks, &window_on);
    if (e != hipSuccess) return e;
    return head_dim == 64 ? launch_d<64, false>(p, blocks, window_on, stream)
                          : launch_d<128, false>(p, blocks, window_on, stream);
}

hipError_t launch_prefill_rotating(const PrefillRotParams& p_in, int head_dim, hipStream_t stream) {
    PrefillRotParams p = p_in;
    unsigned blocks = 0;
    bool window_on = false;
    const hipError_t e = prepare(p, head_dim, &blocks, &window_on);
    if (e != hipSuccess) return e;
    return head_dim == 64 ? launch_d<64, true>(p, blocks, window_on, stream)
                          : launch_d<128, true>(p, blocks, window_on, stream);
}

}  // namespace atf
