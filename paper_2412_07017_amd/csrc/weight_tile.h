// Which weights a wave of the products of up to four row tiles (k_chunk_gemm and its relatives) requests: plain arithmetic, for the device and for tests on the host.
#pragma once
#include "common.h"

namespace asynclm {

// Row q of the lane = tile row 4 q + lane / 16: rows 0..15 start at w0, rows 16..31 at w1 (both the same for the whole wave), off[q] is the
// lane's byte offset from there.  Nothing is fetched for rows from w0 + bytes (w1 + bytes) on.
struct WeightTile { const bf16_t *w0, *w1; uint32_t bytes, off[8]; };

// The part of the tile's run that a request for block `blk` (128 columns) takes: the bytes of the run and the request's start in it.  Not `live`: nothing.
// The range check compares a lane's offset with bytes - base, a difference of unsigned 32-bit numbers: a request that takes nothing (a wave without gate
// rows among them) starts at 0, because with a start past the end the difference wraps and nothing is dropped.
struct RunPart { uint32_t bytes, base; };
__host__ __device__ __forceinline__ RunPart weight_part(const WeightTile& t, int blk, bool live) {
    const uint32_t bytes = live ? t.bytes : 0u;
    return RunPart{bytes, bytes ? (uint32_t)blk * 256 : 0u};
}

// 32 consecutive rows of K columns from w on
__host__ __device__ __forceinline__ WeightTile weight_tile(const bf16_t* w, int K, int lane) {
    WeightTile t;
    t.w0 = t.w1 = w; t.bytes = 64u * (uint32_t)K;
#pragma unroll
    for (int q = 0; q < 8; ++q) t.off[q] = (uint32_t)(4 * q + (lane >> 4)) * (uint32_t)K * 2 + (lane & 15) * 16;
    return t;
}

// Gate rows of a wave-tile: the fewest whole rounds of tiles over the device's waves that 16 rows per tile allow.
inline int gate_rows_per_wave(int F, int waves) {
    int rp = 16;
    for (int m = 1; m <= 64; ++m) {
        rp = (F + waves * m - 1) / (waves * m);
        if (rp <= 16) break;
    }
    return rp < 1 ? 1 : rp > 16 ? 16 : rp;
}

// Of them, those of the wave that starts at gate row n0; none past the last
__host__ __device__ __forceinline__ int gate_rows(int F, int n0, int rp) { const int left = F - n0; return left < 0 ? 0 : left < rp ? left : rp; }

// Gate rows n0 .. n0 + nr - 1 of F into tile rows 0 .., the up rows of the same columns into tile rows 16 ..
__host__ __device__ __forceinline__ WeightTile gate_up_tile(const bf16_t* W, int F, int K, int n0, int nr, int lane) {
    WeightTile t = weight_tile(W, K, lane);
    const int g0 = n0 < F ? n0 : F - 1;
    t.w0 = W + (size_t)g0 * K; t.w1 = W + (size_t)(F + g0) * K; t.bytes = 2u * (uint32_t)nr * (uint32_t)K;
#pragma unroll
    for (int q = 4; q < 8; ++q) t.off[q] = t.off[q - 4];
    return t;
}

}  // namespace asynclm
