// Streaming MFMA kernels of the Gated MLP for one token tile (6 to 128 tokens)
// and small weights.
//
// With few tokens and small weights a step takes some 10 us of weight stream
// and as much again of latency: the ramp and barriers of the LDS ring
// (gemm_mfma.hpp) and the split-K exchange.  No weight is shared between
// waves, so here each wave streams its own rows of the weights straight into
// registers and transposes them there, as the GEMV kernels read theirs, and
// feeds the matrix cores: no LDS and no barrier in the k loop.
//
//   * A block owns 64 (or 128) columns of one weight (the down step) or of
//     both (gate/up), over the rows of its split.  Its 4 waves (one per SIMD)
//     take batches of 32 rows in turn.
//   * Of 128 columns, lane l of a wave loads 16 bytes, columns 8 (l % 16) .. +7,
//     of the 8 rows 8 (l / 16) .. +7 of a batch: each load instruction reads
//     four 256-byte row segments.  32 v_perm_b32 transpose the lane's 8 x 8
//     block into eight A fragments of v_mfma_f32_16x16x32_bf16: fragment i
//     holds column 8 (l % 16) + i, and lane group l / 16 the k's 8 (l / 16)
//     .. +7.  64 columns: 8-byte loads, four fragments.
//   * The B fragments are 16-byte loads of 16 token rows (from L2: X or H is
//     small), used for all the columns of a batch.
//   * A batch's registers are loaded again as soon as it is transposed, before
//     its MFMAs; 32 KB are in flight per block, which streams fastest (more
//     queues up in front of the memory: 64 KB 8% slower, 128 KB 11%).
//   * The accumulators of the waves are added through LDS in wave order, the
//     splits by the last block of a tile in split order (the exchange of
//     gemm_mfma.hpp), so the result is bitwise reproducible.  That last block
//     reads (splits x columns x tokens) fp32: with 64 columns a quarter of
//     what 128 read, which is what the narrow tiles are for.
//
// Measured over rotated weights, LDS ring against this (us, gate/up and down):
// D = 1024, F = 4096, T = 48: 21.1 + 26.5 -> 12.2 + 10.3; D = 2048, F = 8192,
// T = 51: 24.5 + 22.3 -> 22.2 + 16.0, of which the weight stream takes 15.4 +
// 10.3 (4.4 and 3.3 TB/s, launch included), the sum over the waves 3.0 + 2.0 and
// the exchange the rest.
#pragma once

#include <type_traits>

#include "common.hpp"
#include "gemm_params.hpp"
#include "tiling.hpp"

namespace gmlp {

// One block's work with NT token tiles of 16 (N <= 16 NT).
template <class S, int EPI, int NT>
__device__ __forceinline__ void stream_tile(const GemmParams &p, int block, f32x4 *red)
{
    __shared__ int s_last;
    constexpr int NW = S::NW, NWAVES = S::NWAVES, DEPTH = S::STAGES;
    constexpr int CPL = S::BMW / 16; // columns per lane
    constexpr int HP = CPL / 4;      // pieces of 4 columns per lane and 16-token tile of a wave's share
    typedef __attribute__((__vector_size__(CPL * 2))) uint32_t Row; // a lane's columns of one row
    static_assert(EPI == EPI_GATE_MUL ? NW == 2 : EPI == EPI_STORE && NW == 1, "gate/up of both weights, or the down step");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, l16 = lane & 15;

    const int ntiles = p.tile_count;
    const int id = xcd_contiguous_id(block, ntiles * p.splits);
    const int split = id / ntiles, tile = id - split * ntiles;
    const int M = p.M, N = p.N, K = p.K;
    const int m0 = tile * S::BMW;
    const int kb = split * p.k_split;
    const int ke = min(K, kb + p.k_split);
    const int nb_all = (ke - kb + 31) >> 5;
    const int nb = (nb_all - wave + NWAVES - 1) / NWAVES; // batches of this wave: wave, wave + NWAVES, ...

    // Lane offsets within a batch, in bytes; out of range (zeros, no fetch)
    // past the last column and the last token.
    const uint32_t w_voff = m0 + CPL * l16 < M ? (uint32_t)(8 * g * M + CPL * l16) * 2u : kOutOfRange;
    const uint32_t x_voff = (uint32_t)(l16 * K + 8 * g) * 2u;

    // Unit u of a wave is weight u % NW of its batch u / NW; DEPTH units are
    // in flight.  A unit's registers are loaded again as soon as it has been
    // transposed, ahead of its MFMAs.  The token fragments of the next batch
    // are issued before those loads: loads complete in order, so they never
    // wait for the weights issued behind them.
    constexpr bool WIDE = CPL == 8;
    auto load_w = [&](Row (&v)[8], int b, int w) __attribute__((always_inline)) {
        const int k0 = kb + 32 * (wave + b * NWAVES);
        const uint32_t voff = k0 + 8 * g < ke ? w_voff : kOutOfRange; // K and the splits are multiples of 8
        const __amdgpu_buffer_rsrc_t r = make_rsrc((w == 0 ? p.w0 : p.w1) + (size_t)min(k0, K - 8) * M + m0);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t soff = (uint32_t)i * (uint32_t)M * 2u;
            if constexpr (WIDE)
                v[i] = __builtin_bit_cast(Row, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, kNonTemporal));
            else
                v[i] = __builtin_bit_cast(Row, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, kNonTemporal));
        }
    };
    auto load_x = [&](u32x4 (&v)[NT], int b) __attribute__((always_inline)) {
        const int k0 = kb + 32 * (wave + b * NWAVES);
        const bool in = k0 + 8 * g < ke;
        const __amdgpu_buffer_rsrc_t r = make_rsrc(p.act + min(k0, K - 8));
#pragma unroll
        for (int t = 0; t < NT; ++t)
            v[t] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                 r, in && 16 * t + l16 < N ? x_voff : kOutOfRange,
                                                 (uint32_t)(16 * t) * (uint32_t)K * 2u, 0));
    };

    f32x4 acc[NW][CPL][NT];
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
        for (int i = 0; i < CPL; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t)
                acc[w][i][t] = f32x4{};
    Row raw[DEPTH][8];
    u32x4 x[2][NT];
    load_x(x[0], 0);
#pragma unroll
    for (int u = 0; u < DEPTH; ++u)
        load_w(raw[u], u / NW, u % NW);
    static_assert(2 * NW % DEPTH == 0, "two batches are whole turns of the ring");
    auto batch = [&](auto odd, int b) __attribute__((always_inline)) {
        constexpr int P = decltype(odd)::value;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            Row(&rw)[8] = raw[(P * NW + w) % DEPTH];
            bf16x8 a[CPL]; // column i of the lane's 8 rows
#pragma unroll
            for (int e = 0; e < CPL / 2; ++e) {
                u32x4 lo, hi;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    lo[j] = __builtin_amdgcn_perm(rw[2 * j + 1][e], rw[2 * j][e], 0x05040100u);
                    hi[j] = __builtin_amdgcn_perm(rw[2 * j + 1][e], rw[2 * j][e], 0x07060302u);
                }
                a[2 * e] = __builtin_bit_cast(bf16x8, lo);
                a[2 * e + 1] = __builtin_bit_cast(bf16x8, hi);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (w + 1 == NW)
                load_x(x[1 - P], b + 1);
            load_w(rw, b + (w + DEPTH) / NW, (w + DEPTH) % NW);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < CPL; ++i)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[w][i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], __builtin_bit_cast(bf16x8, x[P][t]),
                                                                           acc[w][i][t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int b = 0;
    for (; b + 2 <= nb; b += 2) {
        batch(std::integral_constant<int, 0>{}, b);
        batch(std::integral_constant<int, 1>{}, b + 1);
    }
    if (b < nb)
        batch(std::integral_constant<int, 0>{}, b);

    // ---- sum over the waves, through LDS ---------------------------------------
    // Lane l's accumulators [i][t] element r are column 4 CPL g + CPL r + i of
    // token 16 t + l16.  Wave r adds up the CPL columns of group r (HP pieces
    // of 4 columns per token tile) over the waves, in wave order.  A round
    // moves all token tiles of RW weights.
    constexpr int RW = S::RED_WEIGHTS;
    float sum[NW][NT][CPL];
    auto slot = [&](int src, int w, int t, int r, int h) __attribute__((always_inline)) {
        return red + ((((src * RW + w) * NT + t) * 4 + r) * HP + h) * 64 + lane;
    };
    auto own = [&](int w, int t, int r, int h) __attribute__((always_inline)) {
        return f32x4{acc[w][4 * h][t][r], acc[w][4 * h + 1][t][r], acc[w][4 * h + 2][t][r], acc[w][4 * h + 3][t][r]};
    };
#pragma unroll
    for (int w0 = 0; w0 < NW; w0 += RW) {
        if (w0 > 0)
            __syncthreads();
#pragma unroll
        for (int w = 0; w < RW; ++w)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int h = 0; h < HP; ++h)
                        *slot(wave, w, t, r, h) = own(w0 + w, t, r, h);
        __syncthreads();
#pragma unroll
        for (int w = 0; w < RW; ++w)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int h = 0; h < HP; ++h) {
                    f32x4 s = *slot(0, w, t, wave, h);
#pragma unroll
                    for (int q = 1; q < NWAVES; ++q)
                        s += *slot(q, w, t, wave, h);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        sum[w0 + w][t][4 * h + e] = s[e];
                }
    }

    // ---- sum over the splits, by the last block of the tile ---------------------
    constexpr int PIECES = NW * NT * HP; // of this wave
    static_assert(PIECES <= 16, "two splits in flight at least");
    if (p.splits > 1) {
        const __amdgpu_buffer_rsrc_t prs = make_rsrc(p.partial);
        const uint32_t lane_off = lane * 16;
        auto wave_base = [&](int sp) __attribute__((always_inline)) {
            return (uint32_t)(((sp * ntiles + tile) * NWAVES + wave) * PIECES) * 1024u;
        };
        auto piece = [&](int q) __attribute__((always_inline)) {
            const int w = q / (NT * HP), t = q / HP % NT, h = q % HP;
            return f32x4{sum[w][t][4 * h], sum[w][t][4 * h + 1], sum[w][t][4 * h + 2], sum[w][t][4 * h + 3]};
        };
        const uint32_t base = wave_base(split);
#pragma unroll
        for (int q = 0; q < PIECES; ++q)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, piece(q)), prs, lane_off,
                                                   base + q * 1024u, kCoherent);
        wait_vmcnt<0>();
        __syncthreads();
        if (threadIdx.x == 0) {
            const uint32_t before =
                __hip_atomic_fetch_add(p.counters + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_last = before == (uint32_t)(p.splits - 1);
        }
        __syncthreads();
        if (!s_last)
            return;
        if (threadIdx.x == 0)
            __hip_atomic_store(p.counters + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // The other splits' pieces, up to C splits in flight at once, and this
        // block's own at its place in the order.  What does not fill a group
        // takes smaller ones, where a slot past the last reloads the last and
        // is not added: a whole group of spare slots costs as much as one of
        // real ones (down step with whole groups only: D = 1032, F = 1032, T = 8,
        // two splits and 31 spare loads a piece, 10.1 us against 7.0; D = 1024,
        // F = 4096, T = 16, eight splits, 11.0 against 7.6).
        constexpr int C = 32 / PIECES;
        const int others = p.splits - 1;
        f32x4 tot[PIECES];
#pragma unroll
        for (int q = 0; q < PIECES; ++q)
            tot[q] = f32x4{};
        int s0 = 0;
        auto add_group = [&](auto size) __attribute__((always_inline)) {
            constexpr int G = decltype(size)::value;
            f32x4 x[G][PIECES];
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const int o = min(s0 + u, others - 1);
                const uint32_t sb = wave_base(o + (o >= split));
#pragma unroll
                for (int q = 0; q < PIECES; ++q)
                    x[u][q] = __builtin_bit_cast(
                        f32x4, __builtin_amdgcn_raw_buffer_load_b128(prs, lane_off, sb + q * 1024u, kCoherent));
            }
#pragma unroll
            for (int u = 0; u < G; ++u) {
                if (s0 + u == split && split < others)
#pragma unroll
                    for (int q = 0; q < PIECES; ++q)
                        tot[q] += piece(q);
                if (s0 + u < others)
#pragma unroll
                    for (int q = 0; q < PIECES; ++q)
                        tot[q] += x[u][q];
            }
            s0 += G;
        };
        while (s0 + C <= others)
            add_group(std::integral_constant<int, C>{});
        while (s0 + 2 < others)
            add_group(std::integral_constant<int, (C < 8 ? C : 8)>{});
        if (s0 < others)
            add_group(std::integral_constant<int, 2>{});
        if (split == others)
#pragma unroll
            for (int q = 0; q < PIECES; ++q)
                tot[q] += piece(q);
#pragma unroll
        for (int q = 0; q < PIECES; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                sum[q / (NT * HP)][q / HP % NT][4 * (q % HP) + e] = tot[q][e];
    }

    // ---- epilogue: CPL consecutive columns of one token per lane and token tile ----
    const int col = 4 * CPL * g + CPL * wave;
    const __amdgpu_buffer_rsrc_t ro = make_rsrc(p.out + m0);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int tok = 16 * t + l16;
        const bool in = tok < N;
        const float r = EPI != EPI_STORE && p.rrms && in ? p.rrms[tok] : 1.0f;
        const float d = EPI == EPI_STORE && p.rowdiv && in ? p.rowdiv[tok] : 1.0f;
        float y[CPL];
#pragma unroll
        for (int e = 0; e < CPL; ++e) {
            if constexpr (EPI == EPI_STORE) {
                y[e] = sum[0][t][e];
                if (p.rowdiv)
                    y[e] = y[e] / d;
            } else {
                float gv = sum[0][t][e], uv = sum[NW - 1][t][e];
                if (p.rrms) {
                    gv *= r;
                    uv *= r;
                }
                y[e] = gate_act(gv, p.activation, p.beta) * uv;
            }
        }
        const uint32_t off = in && m0 + col < M ? (uint32_t)(tok * M + col) * 2u : kOutOfRange;
        if constexpr (WIDE)
            __builtin_amdgcn_raw_buffer_store_b128(u32x4{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]),
                                                         pack_bf16x2(y[CPL - 4], y[CPL - 3]),
                                                         pack_bf16x2(y[CPL - 2], y[CPL - 1])},
                                                   ro, off, 0, 0);
        else
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])}, ro, off, 0, 0);
    }
}

// A launch of streaming tiles: one token tile, of TN x 32 tokens of which the
// last 16 are left out where N does not reach them.
template <class S, int EPI>
__device__ __forceinline__ void stream_block(const GemmParams &p)
{
    __shared__ __attribute__((aligned(1024))) f32x4 red[S::RED_BYTES / 16];
    if (p.N <= S::BN - 16)
        stream_tile<S, EPI, 2 * S::TN - 1>(p, blockIdx.x, red);
    else
        stream_tile<S, EPI, 2 * S::TN>(p, blockIdx.x, red);
}

} // namespace gmlp
