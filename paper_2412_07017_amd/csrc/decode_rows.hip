// Several consecutive rows of one sequence per pass over the weights, for the models outside the matrix-core paths: fp32 models and
// bf16 models of sizes that are no multiple of 128.  (bf16 models of such multiples with head_dim 64 or the single-plane cache take passes of
// up to 512 rows on the matrix cores, forward_wide_rows, where memory allows, and only short passes of the smaller ones here: rows_are_faster.)  The arithmetic of a row is
// that of the single-row kernels: fp32 activations, fp32 accumulation on the vector units, the same epilogues.
//
// A single-row pass is bound by the weight stream (8B shape) or by the launches (small models); either cost is nearly the
// same for up to ROWS_MAX rows, so an interrupt or a prompt takes ROWS_MAX tokens per pass (ROWS_PASS_SMALL where all products
// are small) instead of one.  Measured, one
// layer of the 8B shape with the single-plane cache: 152 us for eight rows (QKV 24, attention 9, O 19, gate/up 52, down 45)
// against 8 x 94 us token by token (128 us for up to 32 rows on the matrix cores); the
// tiny fp32 preset's session (64 + 8 tokens, 32 steps) 7.3 -> 3.1 ms with k_rows_gemv alone; 1.91 ms with the kernels for small
// products, here and in decode_kernels.hip.
#include "common.h"
#include "launch.h"
#include "decode_device.h"

#include <algorithm>

namespace asynclm {

struct RowsArgs {
    const void* W;          // [rows, K] row-major
    int32_t rows, K;
    int32_t units, uq, ur;  // row pairs; units / waves and units % waves of the grid
    int32_t done_cap;       // finished row pairs a wave can park in LDS
    int32_t n;              // token rows of this pass (1 .. ROWS_MAX; k_rows_small: .. ROWS_PASS_SMALL, eight per workgroup)
    int32_t pos0, seq;
    const float* x;         // [n][K] input vectors
    const float* gain;      // [K] RMSNorm gain, or nullptr
    float* y;               // [n][y_stride]: RESID y = res + product; SWIGLU the activation
    const float* res;
    int32_t y_stride;
    float* q_out;           // QKV: rotated queries [n][Hq * dh]
    void* kv_layer;
    const float* rope_cos;
    const float* rope_sin;
};

// Eight waves per workgroup, two per SIMD, because the LDS reads of one wave wait behind only 16 products of their own:
// gate/up product of the 8B shape, eight rows, 52 us against 64 us with four waves (four tiles each in flight); with four
// tiles for each of eight waves 56 us (the requests queue up in front of the vectors).
constexpr int ROWS_NW = 8;           // waves per workgroup
constexpr int ROWS_RING = 2;         // weight tiles in flight per wave
constexpr int ROWS_SEG = 4096;      // columns of the input vectors held in LDS at a time: 8 rows x 16 KiB

// Sums NV per-lane values over the wave: lane l < NV returns the total of value rows_index<NV>(l).  Each exchange halves
// the number of values a lane still carries, so NV values cost NV - 1 + 6 - log2(NV) exchanges instead of 6 NV.
template <int NV, int HALF = NV / 2, int MASK = 1>
__device__ __forceinline__ float rows_reduce(float (&v)[NV], int lane) {
    if constexpr (HALF >= 1) {
        const bool up = (lane & MASK) != 0;
#pragma unroll
        for (int i = 0; i < HALF; ++i) {
            const float keep = up ? v[i + HALF] : v[i], send = up ? v[i] : v[i + HALF];
            v[i] = keep + __shfl_xor(send, MASK, 64);
        }
        return rows_reduce<NV, HALF / 2, MASK * 2>(v, lane);
    } else {
        float t = v[0];
#pragma unroll
        for (int m = NV; m < 64; m *= 2) t += __shfl_xor(t, m, 64);
        return t;
    }
}
template <int NV>
__device__ __forceinline__ int rows_index(int lane) {
    int idx = 0, bit = 1;
#pragma unroll
    for (int half = NV / 2; half >= 1; half >>= 1, bit <<= 1) idx |= (lane & bit) ? half : 0;
    return idx;
}

// Columns [4096 seg, ...) of the input vectors -> LDS, planar as in stage_vector ([row][plane][group]), zero past the last
// column.  `ss` (if wanted) takes the squares.
template <typename WT>
__device__ __forceinline__ void rows_stage(float4* xs, int GS, const RowsArgs& a, int seg, float (&ss)[ROWS_MAX], bool count) {
    constexpr int NP = Elem<WT>::EPL / 4;
    constexpr int NT = ROWS_NW * 64;
    const int tid = threadIdx.x, n4 = a.K >> 2, base = seg * (ROWS_SEG / 4);
    for (int l0 = 0; l0 < GS * NP; l0 += 2 * NT) {
        float4 gn[2];
        int k4[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            k4[j] = base + l0 + j * NT + tid;
            gn[j] = a.gain ? as_float4(load16(a.gain + 4 * (size_t)min(k4[j], n4 - 1))) : make_float4(1.f, 1.f, 1.f, 1.f);
        }
        float4 v[ROWS_MAX][2];
#pragma unroll
        for (int r = 0; r < ROWS_MAX; ++r)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                v[r][j] = as_float4(load16(a.x + (size_t)min(r, a.n - 1) * a.K + 4 * (size_t)min(k4[j], n4 - 1)));
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int l = l0 + j * NT + tid;
            if (l >= GS * NP) continue;
            const bool live = k4[j] < n4;
            const int grp = l / NP, pl = l - grp * NP;
#pragma unroll
            for (int r = 0; r < ROWS_MAX; ++r) {
                const float4 x = live ? v[r][j] : make_float4(0.f, 0.f, 0.f, 0.f);
                if (count) ss[r] += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
                xs[(r * NP + pl) * GS + grp] = make_float4(x.x * gn[j].x, x.y * gn[j].y, x.z * gn[j].z, x.w * gn[j].w);
            }
        }
    }
}

// Every wave owns a contiguous share of the row pairs and takes UB of them at a time over all columns, so a vector
// element read from LDS is used for 2 UB weight rows; the weights stream through a ring of register tiles (2 rows x
// 4 wave-wide loads each; ROWS_RING of them) that is requested before the vectors are staged.  SEG: the vectors do not fit LDS as a whole
// (more than 4096 columns): they are staged in segments, again for every UB row pairs.
// The QKV product adds its terms in two levels (8 or 4 per load, then the loads): the single-plane cache rounds keys and
// values to 8 bits of mantissa, and how many of them round the other way is proportional to the error of these sums.
// Bound: the vector units (16 products and two conversions per weight, fp32) and the LDS reads beside the weight stream.
template <typename WT, int EPI, int UB, bool SEG>
__global__ __launch_bounds__(ROWS_NW * 64) void k_rows_gemv(RowsArgs a, Geom g) {
    constexpr int EPL = Elem<WT>::EPL, NP = EPL / 4, R = ROWS_MAX;
    constexpr int TS = ROWS_SEG / (256 * EPL);      // tiles per segment
    constexpr int AHEAD = ROWS_RING / UB > 0 ? ROWS_RING / UB : 1;                // column tiles in flight
    constexpr int NV = 2 * UB * R;
    extern __shared__ float4 lds4[];
    __shared__ float red[ROWS_NW][R];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Kg = a.K / EPL, KT = (Kg + 255) / 256;
    const int GS = min(KT, TS) * 256;
    float4* xs = lds4;
    float* done = reinterpret_cast<float*>(lds4 + (size_t)R * NP * GS) + (size_t)wave * a.done_cap * 2 * R;
    const int gw = (int)blockIdx.x * ROWS_NW + wave;
    const int u0 = gw * a.uq + min(gw, a.ur), cnt = a.uq + (gw < a.ur ? 1 : 0);
    const int nbatch = (a.uq + (a.ur ? 1 : 0) + UB - 1) / UB;      // the same for every wave: staging synchronises them
    const int T = nbatch * KT;
    const WT* W = (const WT*)a.W;

    auto load = [&](uint4 (&v)[8], int batch, int kt, int u) {
        const int unit = min(u0 + min(batch * UB + u, max(cnt - 1, 0)), a.units - 1);   // past the share: its last pair again
        int rA, rB;
        unit_rows<EPI>(unit, a.rows, g, rA, rB);
        const WT* pa = W + (size_t)rA * a.K;
        const WT* pb = W + (size_t)rB * a.K;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int gi = min((kt * 4 + s) * 64 + lane, Kg - 1);
            v[2 * s] = load16_stream(pa + (size_t)gi * EPL);
            v[2 * s + 1] = load16_stream(pb + (size_t)gi * EPL);
        }
    };
    uint4 ring[AHEAD][UB][8];
    int lb = 0, lk = 0;                             // next tile to request
    auto advance = [&](int& b, int& k) { if (++k == KT) { k = 0; ++b; } };
#pragma unroll
    for (int d = 0; d < AHEAD; ++d) {
#pragma unroll
        for (int u = 0; u < UB; ++u) load(ring[d][u], min(lb, nbatch - 1), lk, u);
        advance(lb, lk);
    }
    __builtin_amdgcn_sched_barrier(0);

    float ss[R];
#pragma unroll
    for (int r = 0; r < R; ++r) ss[r] = 0.f;
    rows_stage<WT>(xs, GS, a, 0, ss, true);
    __syncthreads();

    float acc[NV];                                  // [matrix row of the pair][u][token row]
#pragma unroll
    for (int i = 0; i < NV; ++i) acc[i] = 0.f;
    int cb = 0, ck = 0;
    for (int t = 0; t < T; t += AHEAD) {
#pragma unroll
        for (int d = 0; d < AHEAD; ++d) {
            if (t + d >= T) break;                  // uniform
            if (SEG && ck % TS == 0 && t + d > 0) {
                __syncthreads();                    // the previous segment has been read by every wave
                rows_stage<WT>(xs, GS, a, ck / TS, ss, cb == 0);
                __syncthreads();
            }
            const int gl = (SEG ? ck % TS : ck) * 256 + lane;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                float w[2 * UB][EPL];
#pragma unroll
                for (int u = 0; u < UB; ++u) {
                    Elem<WT>::expand(ring[d][u][2 * s], w[u]);
                    Elem<WT>::expand(ring[d][u][2 * s + 1], w[UB + u]);
                }
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    float x[EPL];
#pragma unroll
                    for (int pl = 0; pl < NP; ++pl) {
                        const float4 v = xs[(r * NP + pl) * GS + gl + s * 64];
                        x[4 * pl] = v.x; x[4 * pl + 1] = v.y; x[4 * pl + 2] = v.z; x[4 * pl + 3] = v.w;
                    }
                    if (EPI == EPI_QKV) {           // see below: keys and values may be rounded to 16 bits next
#pragma unroll
                        for (int u = 0; u < 2 * UB; ++u) {
                            float p = w[u][0] * x[0];
#pragma unroll
                            for (int e = 1; e < EPL; ++e) p = fmaf(w[u][e], x[e], p);
                            acc[u * R + r] += p;
                        }
                    } else {
#pragma unroll
                        for (int e = 0; e < EPL; ++e)
#pragma unroll
                            for (int u = 0; u < 2 * UB; ++u) acc[u * R + r] = fmaf(w[u][e], x[e], acc[u * R + r]);
                    }
                }
            }
            if (ck == KT - 1) {
                const float v = rows_reduce<NV>(acc, lane);
                const int i = rows_index<NV>(lane), u = cb * UB + (i / R) % UB;
                if (lane < NV && u < cnt) done[(u * 2 + i / (R * UB)) * R + i % R] = v;
#pragma unroll
                for (int j = 0; j < NV; ++j) acc[j] = 0.f;
            }
            advance(cb, ck);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < UB; ++u) load(ring[d][u], min(lb, nbatch - 1), lk, u);
            advance(lb, lk);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    {
        const float v = rows_reduce<R>(ss, lane);
        if (lane < R) red[wave][rows_index<R>(lane)] = v;
        __syncthreads();
    }
    EpiOut eo{};
    eo.q_out = a.q_out; eo.kv_layer = a.kv_layer; eo.rope_cos = a.rope_cos; eo.rope_sin = a.rope_sin; eo.rows = a.rows; eo.seq = a.seq;
    for (int j = lane; j < cnt * R; j += 64) {
        const int ul = j / R, r = j % R, u = u0 + ul;
        if (r >= a.n) continue;
        float sq = 0.f;
#pragma unroll
        for (int w = 0; w < ROWS_NW; ++w) sq += red[w][r];
        const float sc = a.gain ? 1.f / sqrtf(sq / (float)a.K + g.eps) : 1.f;
        const float sa = done[(ul * 2) * R + r] * sc, sb = done[(ul * 2 + 1) * R + r] * sc;
        float e0 = 0.f, e1 = 0.f;
        eo.y = a.y + (size_t)r * a.y_stride; eo.pos = a.pos0 + r;
        if (EPI == EPI_RESID) {
            const float* res = a.res + (size_t)r * a.y_stride;
            e0 = res[2 * u]; e1 = res[min(2 * u + 1, a.rows - 1)];
        } else if (EPI == EPI_QKV) {
            const int hs = g.dh == 128 ? 6 : 5, i = u & ((1 << hs) - 1);
            const size_t ri = ((size_t)eo.pos << hs) + i;
            e0 = a.rope_cos[ri]; e1 = a.rope_sin[ri];
            eo.q_out = a.q_out + (size_t)r * g.Hq * g.dh;
        }
        finish_unit<WT, EPI>(u, sa, sb, e0, e1, eo, g);
    }
}

// Small products (at most one row pair per wave of the device, one tile of columns per row): the same without ring and staging,
// as k_gemv_small: a wave per row pair, its two rows and the input vectors in registers.  Tiny preset, eight rows: QKV 7.7 -> 4.3 us,
// O 8.4 -> 3.8, gate/up 6.9 -> 4.4, down 8.4 -> 5.8; its session 2.15 -> 1.91 ms.
// Eight rows per workgroup, any number of workgroups beside each other (grid y): where all products are small a pass is as long as
// 128 rows, because eight rows use few of the compute units and a launch costs nearly the same: 64 rows of the tiny preset take 5.5 us for QKV
// (eight: 4.5), 3.9 for O (3.5), 6.9 for gate/up (4.4), 6.0 for down (5.8); its session 1906 -> 1624 us.
template <typename WT, int EPI, int NS>
__global__ __launch_bounds__(256) void k_rows_small(RowsArgs a, Geom g) {
    constexpr int EPL = Elem<WT>::EPL, NP = EPL / 4, R = ROWS_MAX;
    __shared__ float sums[4][3 * R];                // per wave: dot products of the two rows, squares
    {                                               // this workgroup's eight rows of the pass
        const int r0 = blockIdx.y * R;
        a.n = min(a.n - r0, R); a.pos0 += r0;
        a.x += (size_t)r0 * a.K;
        if (EPI == EPI_QKV) a.q_out += (size_t)r0 * g.Hq * g.dh;
        else a.y += (size_t)r0 * a.y_stride;
        if (EPI == EPI_RESID) a.res += (size_t)r0 * a.y_stride;
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int unit = blockIdx.x * 4 + wave, u = min(unit, a.units - 1), Kg = a.K / EPL;
    int rA, rB;
    unit_rows<EPI>(u, a.rows, g, rA, rB);
    const WT* pa = (const WT*)a.W + (size_t)rA * a.K;
    const WT* pb = (const WT*)a.W + (size_t)rB * a.K;
    uint4 wa[NS], wb[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int gi = min(s * 64 + lane, Kg - 1);
        wa[s] = load16_stream(pa + (size_t)gi * EPL); wb[s] = load16_stream(pb + (size_t)gi * EPL);
    }
    // epilogue operands of the row this lane finishes
    const int r = min(lane, a.n - 1);
    EpiOut eo{};
    eo.q_out = a.q_out + (EPI == EPI_QKV ? (size_t)r * g.Hq * g.dh : 0); eo.kv_layer = a.kv_layer;
    eo.rope_cos = a.rope_cos; eo.rope_sin = a.rope_sin; eo.rows = a.rows; eo.seq = a.seq; eo.pos = a.pos0 + r;
    eo.y = a.y + (size_t)r * a.y_stride;
    float e0 = 0.f, e1 = 0.f;
    if (EPI == EPI_RESID) { const float* res = a.res + (size_t)r * a.y_stride; e0 = res[rA]; e1 = res[rB]; }
    if (EPI == EPI_QKV) {
        const int hs = g.dh == 128 ? 6 : 5;
        const size_t ri = ((size_t)eo.pos << hs) + (u & ((1 << hs) - 1));
        e0 = a.rope_cos[ri]; e1 = a.rope_sin[ri];
    }
    float acc[2 * R], ss[R];
#pragma unroll
    for (int i = 0; i < R; ++i) { acc[i] = 0.f; acc[R + i] = 0.f; ss[i] = 0.f; }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int gi = min(s * 64 + lane, Kg - 1);
        const bool live = s * 64 + lane < Kg;
        float fa[EPL], fb[EPL];
        Elem<WT>::expand(wa[s], fa); Elem<WT>::expand(wb[s], fb);
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const size_t k = (size_t)gi * EPL + 4 * q;
            const float4 gn = a.gain ? as_float4(load16(a.gain + k)) : make_float4(1.f, 1.f, 1.f, 1.f);
            float4 x[R];
#pragma unroll
            for (int i = 0; i < R; ++i) x[i] = as_float4(load16(a.x + (size_t)min(i, a.n - 1) * a.K + k));
#pragma unroll
            for (int i = 0; i < R; ++i) {
                float4 v = live ? x[i] : make_float4(0.f, 0.f, 0.f, 0.f);
                ss[i] += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
                v = make_float4(v.x * gn.x, v.y * gn.y, v.z * gn.z, v.w * gn.w);
                acc[i] += fmaf(fa[4 * q + 3], v.w, fmaf(fa[4 * q + 2], v.z, fmaf(fa[4 * q + 1], v.y, fa[4 * q] * v.x)));
                acc[R + i] += fmaf(fb[4 * q + 3], v.w, fmaf(fb[4 * q + 2], v.z, fmaf(fb[4 * q + 1], v.y, fb[4 * q] * v.x)));
            }
        }
    }
    const float t = rows_reduce<2 * R>(acc, lane), q = rows_reduce<R>(ss, lane);
    if (lane < 2 * R) sums[wave][rows_index<2 * R>(lane)] = t;
    if (lane < R) sums[wave][2 * R + rows_index<R>(lane)] = q;
    // (written and read by the same wave)
    if (lane < a.n && unit < a.units) {
        const float sc = a.gain ? 1.f / sqrtf(sums[wave][2 * R + lane] / (float)a.K + g.eps) : 1.f;
        finish_unit<WT, EPI>(u, sums[wave][lane] * sc, sums[wave][R + lane] * sc, e0, e1, eo, g);
    }
}

// Rows of the residual stream of a pass; the sequence grows and the step descriptor gets its number for the output head.
template <typename WT>
__global__ __launch_bounds__(256) void k_rows_embed(const WT* __restrict__ E, RowsTokens tk, int row0, int pos0, int seq, int n, float* __restrict__ x,
                                                    int d, StepDesc* step, SeqState* st) {
    const int r = blockIdx.y;
    if (blockIdx.x == 0 && r == 0 && row0 == 0 && threadIdx.x == 0) {
        step->token = -1; step->pos = pos0; step->seq = seq; step->rows = n;
        st[seq].len = pos0 + n;
    }
    const WT* row = E + (size_t)tk.t[r] * d;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < d; i += gridDim.x * 256) x[(size_t)(row0 + r) * d + i] = Elem<WT>::load1(row + i);
}

// Passes of forward_wide_rows, between the QKV product and the attention: the partial planes of the product are added in split order,
// queries and keys rotated, keys and values stored row by row (rounded to bf16, with the remainder where the cache has a lo plane),
// queries left in fp32.  dh / 8 threads per (row, head), four pairs (i, i + dh / 2) each.  P holds the heads from h0 on.
template <int DH>
__global__ __launch_bounds__(256) void k_rows_rope_kv(const float* __restrict__ P, int S, size_t s_stride, int n_stride, Geom g, RowsPass p,
                                                      const float* __restrict__ rope_cos, const float* __restrict__ rope_sin, bf16_t* __restrict__ kv_layer,
                                                      float* __restrict__ q, int h0) {
    constexpr int half = DH / 2, LPI = DH / 8;
    const int nh = g.Hq + 2 * g.Hkv - h0, item = blockIdx.x * (256 / LPI) + threadIdx.x / LPI, i = 4 * (threadIdx.x % LPI);
    if (item >= p.n * nh) return;
    const int m = item / nh, hl = item - m * nh, h = hl + h0, pos = p.pos0 + m;
    float4 pa[CHUNK_GEMM_MAX_SPLIT], pb[CHUNK_GEMM_MAX_SPLIT];
#pragma unroll
    for (int s = 0; s < CHUNK_GEMM_MAX_SPLIT; ++s) {
        const float* src = P + (size_t)min(s, S - 1) * s_stride + (size_t)m * n_stride + hl * DH + i;
        pa[s] = *reinterpret_cast<const float4*>(src); pb[s] = *reinterpret_cast<const float4*>(src + half);
    }
    float a[4] = {0.f, 0.f, 0.f, 0.f}, b[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < CHUNK_GEMM_MAX_SPLIT; ++s)
        if (s < S) {
            a[0] += pa[s].x; a[1] += pa[s].y; a[2] += pa[s].z; a[3] += pa[s].w;
            b[0] += pb[s].x; b[1] += pb[s].y; b[2] += pb[s].z; b[3] += pb[s].w;
        }
    if (h < g.Hq + g.Hkv) {                                         // values are not rotated
        const float4 c4 = *reinterpret_cast<const float4*>(rope_cos + (size_t)pos * half + i), s4 = *reinterpret_cast<const float4*>(rope_sin + (size_t)pos * half + i);
        const float c[4] = {c4.x, c4.y, c4.z, c4.w}, sn[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float ra = a[e] * c[e] - b[e] * sn[e], rb = b[e] * c[e] + a[e] * sn[e];
            a[e] = ra; b[e] = rb;
        }
    }
    if (h < g.Hq) {
        float* o = q + ((size_t)m * g.Hq + h) * DH + i;
        *reinterpret_cast<float4*>(o) = make_float4(a[0], a[1], a[2], a[3]);
        *reinterpret_cast<float4*>(o + half) = make_float4(b[0], b[1], b[2], b[3]);
        return;
    }
    const int hk = h - g.Hq;
    bf16_t* dst = kv_layer + (size_t)p.seq * g.kv_seq_stride + (hk < g.Hkv ? (size_t)hk * g.kv_head_stride : g.kv_v_offset + (size_t)(hk - g.Hkv) * g.kv_head_stride) +
                  (size_t)pos * DH + i;
    bf16_t ea[4][2], eb[4][2];
#pragma unroll
    for (int e = 0; e < 4; ++e) { split_planes<2>(a[e], ea[e]); split_planes<2>(b[e], eb[e]); }
#pragma unroll
    for (int pl = 0; pl < 2; ++pl) {
        if (pl && !g.kv_lo_offset) break;
        bf16_t* o = dst + (pl ? g.kv_lo_offset : 0);
        *reinterpret_cast<uint2*>(o) = make_uint2(ea[0][pl] | ((uint32_t)ea[1][pl] << 16), ea[2][pl] | ((uint32_t)ea[3][pl] << 16));
        *reinterpret_cast<uint2*>(o + half) = make_uint2(eb[0][pl] | ((uint32_t)eb[1][pl] << 16), eb[2][pl] | ((uint32_t)eb[3][pl] << 16));
    }
}

// ---- launchers ------------------------------------------------------------------------------------------------------

namespace {

template <typename WT>
size_t rows_lds(int K, int units, int grid, int* done_cap) {
    constexpr int EPL = Elem<WT>::EPL, TS = ROWS_SEG / (256 * EPL);
    *done_cap = (units + grid * ROWS_NW - 1) / (grid * ROWS_NW);
    const int kt = (K / EPL + 255) / 256;
    return (size_t)ROWS_MAX * std::min(kt, TS) * 256 * EPL * sizeof(float) + (size_t)ROWS_NW * *done_cap * 2 * ROWS_MAX * sizeof(float);
}

// Workgroups and row pairs per batch: a wave per row pair while they all fit one round (small models), else one
// workgroup per compute unit and two pairs at a time (half the LDS reads per weight).
int rows_grid(int units) { return std::max(1, std::min(decode_gemv_grid(), (units + ROWS_NW - 1) / ROWS_NW)); }
int rows_ub(int units) { return units > ROWS_NW * rows_grid(units) ? 2 : 1; }

constexpr size_t ROWS_LDS_LIMIT = 160 * 1024;

template <typename WT, int EPI>
const void* rows_func(int ub, bool seg) {
    if (ub == 1) return seg ? (const void*)(k_rows_gemv<WT, EPI, 1, true>) : (const void*)(k_rows_gemv<WT, EPI, 1, false>);
    return seg ? (const void*)(k_rows_gemv<WT, EPI, 2, true>) : (const void*)(k_rows_gemv<WT, EPI, 2, false>);
}

template <typename WT>
bool rows_fit(int K, int units) {
    int cap = 0;
    return rows_lds<WT>(K, units, rows_grid(units), &cap) + 1024 <= ROWS_LDS_LIMIT;
}

// k_rows_small takes the product
template <typename WT>
bool rows_small(int K, int units) { return K / Elem<WT>::EPL <= 256 && units <= 4 * decode_gemv_grid(); }

template <typename WT, int EPI>
const void* rows_small_func(int ns) {
    return ns <= 1 ? (const void*)(k_rows_small<WT, EPI, 1>) : ns == 2 ? (const void*)(k_rows_small<WT, EPI, 2>) : (const void*)(k_rows_small<WT, EPI, 4>);
}

template <typename WT, int EPI>
hipError_t launch_rows_t(RowsArgs a, const Geom& g, hipStream_t s) {
    if (rows_small<WT>(a.K, a.units) && a.n >= 1 && a.n <= ROWS_PASS_SMALL && a.K % 8 == 0) {
        Geom gg = g;
        void* params[] = {&a, &gg};
        return hipLaunchKernel(rows_small_func<WT, EPI>((a.K / Elem<WT>::EPL + 63) / 64), dim3((a.units + 3) / 4, (a.n + ROWS_MAX - 1) / ROWS_MAX), dim3(256), params, 0, s);
    }
    const int grid = rows_grid(a.units), ub = rows_ub(a.units);
    const size_t lds = rows_lds<WT>(a.K, a.units, grid, &a.done_cap);
    if (lds + 1024 > ROWS_LDS_LIMIT || a.n < 1 || a.n > ROWS_MAX || a.K % 8) return hipErrorInvalidValue;
    a.uq = a.units / (grid * ROWS_NW); a.ur = a.units % (grid * ROWS_NW);
    Geom gg = g;
    void* params[] = {&a, &gg};
    return hipLaunchKernel(rows_func<WT, EPI>(ub, a.K > ROWS_SEG), dim3(grid), dim3(ROWS_NW * 64), params, lds, s);
}

template <int EPI>
hipError_t launch_rows(int dtype, const RowsArgs& a, const Geom& g, hipStream_t s) {
    return dtype == 0 ? launch_rows_t<float, EPI>(a, g, s) : launch_rows_t<bf16_t, EPI>(a, g, s);
}

template <typename WT, int EPI>
hipError_t rows_attr() {
    for (int ub = 1; ub <= 2; ++ub)
        for (int seg = 0; seg < 2; ++seg)
            if (hipError_t e = hipFuncSetAttribute(rows_func<WT, EPI>(ub, seg != 0), hipFuncAttributeMaxDynamicSharedMemorySize, (int)ROWS_LDS_LIMIT - 1024)) return e;
    return hipSuccess;
}

template <typename WT>
hipError_t rows_attrs() {
    hipError_t e = rows_attr<WT, EPI_QKV>();
    if (!e) e = rows_attr<WT, EPI_RESID>();
    return e ? e : rows_attr<WT, EPI_SWIGLU>();
}

}  // namespace

bool rows_supported(int dtype, const Geom& g) {
    const int nqkv = (g.Hq + 2 * g.Hkv) * g.dh, qd = g.Hq * g.dh, dp = (g.d + 1) / 2;
    return dtype == 0 ? rows_fit<float>(g.d, nqkv / 2) && rows_fit<float>(qd, dp) && rows_fit<float>(g.d, g.F) && rows_fit<float>(g.F, dp)
                      : rows_fit<bf16_t>(g.d, nqkv / 2) && rows_fit<bf16_t>(qd, dp) && rows_fit<bf16_t>(g.d, g.F) && rows_fit<bf16_t>(g.F, dp);
}

template <typename WT>
static bool rows_all_small(const Geom& g) {
    const int nqkv = (g.Hq + 2 * g.Hkv) * g.dh, qd = g.Hq * g.dh, dp = (g.d + 1) / 2;
    return rows_small<WT>(g.d, nqkv / 2) && rows_small<WT>(qd, dp) && rows_small<WT>(g.d, g.F) && rows_small<WT>(g.F, dp);
}

int rows_per_pass(int dtype, const Geom& g) { return (dtype == 0 ? rows_all_small<float>(g) : rows_all_small<bf16_t>(g)) ? ROWS_PASS_SMALL : ROWS_MAX; }

hipError_t rows_init(int dtype) { return dtype == 0 ? rows_attrs<float>() : rows_attrs<bf16_t>(); }

hipError_t launch_rows_embed(int dtype, const void* E, const RowsTokens& tk, int row0, int n, const RowsBuffers& rb, const DecodeBuffers& b, const RowsPass& p,
                             const Geom& g, hipStream_t s) {
    if (n < 1 || n > ROWS_MAX || row0 < 0 || row0 + n > p.n) return hipErrorInvalidValue;
    const dim3 grid((g.d + 255) / 256, n);
    if (dtype == 0) hipLaunchKernelGGL(k_rows_embed<float>, grid, dim3(256), 0, s, (const float*)E, tk, row0, p.pos0, p.seq, p.n, rb.x, g.d, b.step, b.seq_state);
    else hipLaunchKernelGGL(k_rows_embed<bf16_t>, grid, dim3(256), 0, s, (const bf16_t*)E, tk, row0, p.pos0, p.seq, p.n, rb.x, g.d, b.step, b.seq_state);
    return hipGetLastError();
}

hipError_t launch_rows_rope_kv(const ChunkBuffers& c, int S, int MT, void* kv_layer, const RowsBuffers& rb, const DecodeBuffers& b, const RowsPass& p,
                               const Geom& g, hipStream_t s, bool kv_only) {
    const int h0 = kv_only ? g.Hq : 0, nh = g.Hq + 2 * g.Hkv - h0, per = 256 / (g.dh / 8);
    if ((g.dh != 64 && g.dh != 128) || S < 1 || S > CHUNK_GEMM_MAX_SPLIT || p.n < 1 || p.n > MT * 32 || !g.kv_v_offset) return hipErrorInvalidValue;
    auto go = [&](auto k) { hipLaunchKernelGGL(k, dim3((p.n * nh + per - 1) / per), dim3(256), 0, s, c.part, S, (size_t)MT * 32 * nh * g.dh, nh * g.dh, g, p,
                                               b.rope_cos, b.rope_sin, (bf16_t*)kv_layer, rb.q, h0); };
    if (g.dh == 128) go(k_rows_rope_kv<128>);
    else go(k_rows_rope_kv<64>);
    return hipGetLastError();
}

static RowsArgs rows_args(const RowsPass& p) {
    RowsArgs a{};
    a.n = p.n; a.pos0 = p.pos0; a.seq = p.seq;
    return a;
}

hipError_t launch_rows_qkv(int dtype, const void* wqkv, const float* gain, void* kv_layer, const RowsBuffers& rb, const DecodeBuffers& b,
                           const RowsPass& p, const Geom& g, hipStream_t s) {
    RowsArgs a = rows_args(p);
    a.W = wqkv; a.rows = (g.Hq + 2 * g.Hkv) * g.dh; a.K = g.d; a.units = a.rows / 2; a.x = rb.x; a.gain = gain;
    a.q_out = rb.q; a.kv_layer = kv_layer; a.rope_cos = b.rope_cos; a.rope_sin = b.rope_sin;
    return launch_rows<EPI_QKV>(dtype, a, g, s);
}

hipError_t launch_rows_oproj(int dtype, const void* wo, const RowsBuffers& rb, const RowsPass& p, const Geom& g, hipStream_t s) {
    RowsArgs a = rows_args(p);
    a.W = wo; a.rows = g.d; a.K = g.Hq * g.dh; a.units = (g.d + 1) / 2; a.x = rb.o; a.y = rb.x; a.res = rb.x; a.y_stride = g.d;
    return launch_rows<EPI_RESID>(dtype, a, g, s);
}

hipError_t launch_rows_gateup(int dtype, const void* wgu, const float* gain, const RowsBuffers& rb, const RowsPass& p, const Geom& g, hipStream_t s) {
    RowsArgs a = rows_args(p);
    a.W = wgu; a.rows = 2 * g.F; a.K = g.d; a.units = g.F; a.x = rb.x; a.gain = gain; a.y = rb.a; a.y_stride = g.F;
    return launch_rows<EPI_SWIGLU>(dtype, a, g, s);
}

hipError_t launch_rows_down(int dtype, const void* wd, const RowsBuffers& rb, const RowsPass& p, const Geom& g, hipStream_t s) {
    RowsArgs a = rows_args(p);
    a.W = wd; a.rows = g.d; a.K = g.F; a.units = (g.d + 1) / 2; a.x = rb.a; a.y = rb.x; a.res = rb.x; a.y_stride = g.d;
    return launch_rows<EPI_RESID>(dtype, a, g, s);
}

}  // namespace asynclm
