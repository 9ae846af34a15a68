// Arguments of the MFMA GEMM kernels (gemm_mfma.hpp, gemm_stream.hpp).
#pragma once

#include <stdint.h>

namespace gmlp {

struct GemmParams {
    const uint16_t *w0;  // [K, M] bf16, M contiguous (Wg, or Wd)
    const uint16_t *w1;  // [K, M] bf16 second weight (Wu) of the dual kernel
    const uint16_t *act; // [N, K] bf16, K contiguous (X, or H)
    uint16_t *out;       // [N, M] bf16 (H, or Y)
    float *partial;      // split-K partial sums, fp32, [split][tile of the launch][wave][piece][lane]
    uint32_t *counters;  // split-K arrival counter per output tile (zero on entry and exit)
    int M, N, K;
    int k_split; // K rows per split (a multiple of BK when splits > 1)
    int splits;
    int tiles_m, tiles_n;
    int group_m; // consecutive blocks sweep group_m column tiles before the next token tile
    // This launch computes tiles [tile_base, tile_base + tile_count) of the
    // block order of all tiles_m x tiles_n tiles (a plan can give the tiles
    // of a last, partial round of blocks to a split-K part of their own).
    int tile_base, tile_count;
    // A split-K launch may start with head_blocks blocks (a multiple of 8)
    // that each compute one whole tile over all of K: tiles [0, head_blocks)
    // of the block order, before its split tiles, so those start as soon as
    // CUs free up instead of after the last whole tile.
    int head_blocks;
    // Gate/up epilogue: activation (enum Activation), swish slope, and the
    // per-token RMSNorm scales [N] (nullptr: none).
    int activation;
    float beta;
    const float *rrms;
    // Store epilogue: per-token divisors [N] (nullptr: none).  Softmax+MatMul
    // divides its result rows by the softmax sums here.
    const float *rowdiv;
};

} // namespace gmlp
