// Append-chunk path on gfx950 (bf16 models): M = 2..CHUNK_MAX rows per forward pass, used by
// interrupt injection and prefill.  Weights are streamed from HBM once per pass; every linear
// map and the causal chunk attention run on the matrix cores (v_mfma_f32_32x32x16_bf16), with
// fp32 accumulation.  Activations are carried as a pair of bf16 planes, hi = bf16(x) and
// lo = bf16(x - hi), and each product is formed as W*hi + W*lo, so the chunk path keeps about
// 16 mantissa bits like the fp32 activations of the single-row path.
//
// Matrix-core operand layout used throughout (wave of 64 lanes, lane = 32 g + i):
//   A[32 x 16]: lane (i, g) holds A[i][8g .. 8g+7]        (8 bf16 = one 16-byte register quad)
//   B[16 x 32]: lane (j, g) holds B[8g .. 8g+7][j]
//   D[32 x 32]: lane (j, g) holds D[8b + 4g + r][j] in register 4b + r  (b, r = 0..3)
// Within a k-block of 128 elements, MFMA step t, lane half g, element e is k = 16 t + 8 g + e.
//
// Memory access.  A wave-wide 16-byte load is cheap when its 64 lanes cover few cache lines, so:
//  * activations (the B operand) are kept in global memory in operand order ("tiled planes"):
//    element (row m, column k) lives at ((((m/32 * K/128 + k/128) * 8 + t) * 2 + g) * 32 + m%32) * 8 + e,
//    and the 64 lanes of a B load read one contiguous KiB;
//  * weights (the A operand, row-major in HBM) are loaded 4 rows x 256 contiguous bytes per
//    instruction and transposed into operand order through a wave-private, XOR-swizzled LDS tile.
// In the chunk attention, which is small next to the weight streaming, every lane instead reads 128
// contiguous bytes of its own K / V^T row (k = 64 g + 8 t + e there).
#include "common.h"
#include "launch.h"
#include "weight_tile.h"

#include <type_traits>

namespace asynclm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ f32x16 mfma_bf16(const uint4& a, const uint4& b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ void split_bf16(float v, bf16_t& hi, bf16_t& lo) {
    hi = f32_to_bf16(v);
    lo = f32_to_bf16(v - __uint_as_float((uint32_t)hi << 16));
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// two fp32 -> two bf16 (round to nearest even) in one 32-bit word, first value in the low half (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16x2(float x, float y) {
    const f32x2 v = {x, y};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// hi = bf16(p), lo = bf16(p - hi) for a pair of values
__device__ __forceinline__ void split_pair(float x, float y, uint32_t& hi, uint32_t& lo) {
    hi = pack_bf16x2(x, y);
    lo = pack_bf16x2(x - __uint_as_float(hi << 16), y - __uint_as_float(hi & 0xffff0000u));
}

// ---------------------------------------------------------------------------------------------
// bookkeeping and small row-wise kernels
// ---------------------------------------------------------------------------------------------

// Row of a workgroup of the row kernels.  A line of a tiled plane holds 16 bytes each of eight consecutive rows; workgroups go
// round robin over the XCDs, so with row = workgroup every line is written in pieces by eight L2 caches.  Eight consecutive
// rows go to one XCD instead, one after the other (rows past the last full 64 keep their place): 1019 rows of the 8B shape with
// two planes 23.6 -> 17.2 us, 2048 rows 48.6 -> 33.9, the first kernel of a 2048-row pass 50 -> 32.
__device__ __forceinline__ int row_of_workgroup(int rows) {
    const int b = blockIdx.x;
    if (b >= (rows & ~63)) return b;
    const int xcd = b & 7, k = b >> 3;
    return ((k >> 3) * 8 + xcd) * 8 + (k & 7);
}

constexpr int ROW_VEC_MAX = 8;      // float4 groups per thread of a row kernel: d <= 8192

// One row by one workgroup: v = x[m] + sum_s P[s][row pm] (S <= SM planes, and the gain of the following norm), returns the sum
// of squares over the workgroup.  Thread tid owns the float4 groups tid + 256 u.  SM: S rounded up to a power of two, because
// the planes past S are requested too (the last one again): with eight always, 1019 rows with two planes took 27.4 instead of 23.6 us.
// Many planes (short passes, one workgroup per compute unit at most): the loads of half a row are all issued before the first use,
// 5.3 us for 16 rows with eight planes against 7.1 one group after the other.  One or two planes (long passes, several workgroups
// per compute unit): one group after the other, 17.4 us for 1019 rows with two planes against 20.3 all at once, 2048 rows 36.5 / 39.5,
// with one plane 30 / 34.7.
template <int SM>
__device__ __forceinline__ float row_gather(const float* __restrict__ xr, const float* __restrict__ Pr, int S,
                                            size_t s_stride, int d4, int tid, const float* __restrict__ gain,
                                            float4 (&v)[ROW_VEC_MAX], float4 (&gn)[ROW_VEC_MAX], float* red) {
    const float4* x4 = reinterpret_cast<const float4*>(xr);
    float ss = 0.f;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
        constexpr int HU = ROW_VEC_MAX / 2, AT_ONCE = SM <= 2 ? 1 : HU;
        if (hf * HU * 256 < d4) {                               // uniform: the upper half only for d > 4096
#pragma unroll
            for (int u0 = hf * HU; u0 < (hf + 1) * HU; u0 += AT_ONCE) {
                float4 p[AT_ONCE][SM];
#pragma unroll
                for (int u = 0; u < AT_ONCE; ++u) {
                    const int i4 = min(tid + 256 * (u0 + u), d4 - 1);       // past the end: a repeated load, dropped below
                    v[u0 + u] = x4[i4];
                    gn[u0 + u] = reinterpret_cast<const float4*>(gain)[i4];
#pragma unroll
                    for (int s = 0; s < SM; ++s)
                        p[u][s] = reinterpret_cast<const float4*>(Pr + (size_t)min(s, S - 1) * s_stride)[i4];
                }
#pragma unroll
                for (int u = 0; u < AT_ONCE; ++u) {
                    float4& w = v[u0 + u];
#pragma unroll
                    for (int s = 0; s < SM; ++s) {
                        const float k = s < S ? 1.f : 0.f;
                        w.x += k * p[u][s].x; w.y += k * p[u][s].y; w.z += k * p[u][s].z; w.w += k * p[u][s].w;
                    }
                    if (tid + 256 * (u0 + u) < d4) ss += w.x * w.x + w.y * w.y + w.z * w.z + w.w * w.w;
                }
                if (AT_ONCE < HU) __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int u = 0; u < HU; ++u) { v[hf * HU + u] = make_float4(0.f, 0.f, 0.f, 0.f); gn[hf * HU + u] = v[hf * HU + u]; }
        }
    }
    ss = wave_sum(ss);
    __syncthreads();
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    return red[0] + red[1] + red[2] + red[3];
}

// four consecutive columns (inside one 8-element group) of one plane
template <int PL>
__device__ __forceinline__ uint2 plane_quad(const bf16_t (&p)[4][PL], int i) {
    return make_uint2(p[0][i] | ((uint32_t)p[1][i] << 16), p[2][i] | ((uint32_t)p[3][i] << 16));
}

// v * sc * gain -> tiled bf16 planes (PL = 2 or 3) at row `mo`
template <int PL>
__device__ __forceinline__ void row_emit(const float4 (&v)[ROW_VEC_MAX], float sc, const float4 (&gain)[ROW_VEC_MAX], int d,
                                         int tid, int mo, bf16_t* __restrict__ out_hi, bf16_t* __restrict__ out_lo, bf16_t* __restrict__ out_lo2) {
    const int d4 = d >> 2;
#pragma unroll
    for (int u = 0; u < ROW_VEC_MAX; ++u) {
        const int i4 = tid + 256 * u;
        if (i4 < d4) {
            const float4 gn = gain[u];
            bf16_t e[4][PL];
            split_planes<PL>(v[u].x * sc * gn.x, e[0]); split_planes<PL>(v[u].y * sc * gn.y, e[1]);
            split_planes<PL>(v[u].z * sc * gn.z, e[2]); split_planes<PL>(v[u].w * sc * gn.w, e[3]);
            const size_t o = tiled_off(mo, 4 * i4, d);       // 4 consecutive columns stay inside one 8-element group
            *reinterpret_cast<uint2*>(out_hi + o) = plane_quad<PL>(e, 0);
            *reinterpret_cast<uint2*>(out_lo + o) = plane_quad<PL>(e, 1);
            if (PL > 2) *reinterpret_cast<uint2*>(out_lo2 + o) = plane_quad<PL>(e, PL - 1);
        }
    }
}

// (three planes carry all of a float: the scale is then formed without the approximate reciprocal root)
template <int PL>
__device__ __forceinline__ float row_scale(float ss, int d, float eps) { return PL > 2 ? 1.f / sqrtf(ss / (float)d + eps) : rsqrtf(ss / (float)d + eps); }

// x[m] += sum_s P[s][m], then RMSNorm with `gain` -> tiled bf16 hi/lo planes.
// One workgroup per row; P has row stride n_stride and split stride s_stride (elements).
template <int SM, int PL>
__global__ __launch_bounds__(256) void k_chunk_resid_norm(float* __restrict__ x, const float* __restrict__ P, int S,
                                                          size_t s_stride, int n_stride, const float* __restrict__ gain,
                                                          float eps, int d, bf16_t* __restrict__ out_hi,
                                                          bf16_t* __restrict__ out_lo, bf16_t* __restrict__ out_lo2) {
    __shared__ float red[4];
    const int m = row_of_workgroup(gridDim.x), tid = threadIdx.x, d4 = d >> 2;
    float* xr = x + (size_t)m * d;
    float4 v[ROW_VEC_MAX], gn[ROW_VEC_MAX];
    const float ss = row_gather<SM>(xr, P + (size_t)m * n_stride, S, s_stride, d4, tid, gain, v, gn, red);
#pragma unroll
    for (int u = 0; u < ROW_VEC_MAX; ++u)
        if (tid + 256 * u < d4) reinterpret_cast<float4*>(xr)[tid + 256 * u] = v[u];
    row_emit<PL>(v, row_scale<PL>(ss, d, eps), gn, d, tid, m, out_hi, out_lo, out_lo2);
}

// First kernel of a pass, one workgroup per row: resolves the token where it is chosen on the device (first row of a
// group), x[m] = E[token], RMSNorm with the first layer's gain -> tiled planes.  The workgroup of a group's first row also
// records the token (in pinned host memory, where the host reads it after the pass) and grows the sequence; the one of the pass's last row fills the step descriptor that the single-row
// kernels read (a pass over one sequence ends with them).
// One launch instead of three (descriptor 4 us, embedding 9 us, norm 6 us for 24 rows of the 8B shape).
template <int PL>
__global__ __launch_bounds__(256) void k_chunk_embed_norm(const bf16_t* __restrict__ E, ChunkTab tab, int rows, StepDesc* step, SeqState* st,
                                                          int32_t* chosen_host, float* __restrict__ x, const float* __restrict__ gain, float eps,
                                                          int d, bf16_t* __restrict__ out_hi, bf16_t* __restrict__ out_lo, bf16_t* __restrict__ out_lo2) {
    __shared__ float red[4];
    const int m = row_of_workgroup(rows), tid = threadIdx.x, d4 = d >> 2;
    const ChunkRow R = tab.row[m];
    const int tok = R.token >= 0 ? R.token : st[R.seq].next_token;
    if (tid == 0) {
        if (m == R.row0) {
            if (R.group >= 0) chosen_host[R.group] = tok;
            st[R.seq].len = R.pos + R.n;
        }
        if (m == rows - 1) { step->token = -1; step->pos = R.pos; step->seq = R.seq; step->rows = rows; }
    }
    const uint2* row = reinterpret_cast<const uint2*>(E + (size_t)tok * d);
    float4 v[ROW_VEC_MAX], gn[ROW_VEC_MAX];
    float ss = 0.f;
#pragma unroll
    for (int u = 0; u < ROW_VEC_MAX; ++u) {
        const int i4 = min(tid + 256 * u, d4 - 1);
        v[u] = gn[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (u * 256 < d4) {                                     // uniform
            const uint2 e = row[i4];
            v[u] = make_float4(bf16_lo(e.x), bf16_hi(e.x), bf16_lo(e.y), bf16_hi(e.y));
            gn[u] = reinterpret_cast<const float4*>(gain)[i4];
        }
    }
#pragma unroll
    for (int u = 0; u < ROW_VEC_MAX; ++u)
        if (tid + 256 * u < d4) {
            reinterpret_cast<float4*>(x + (size_t)m * d)[tid + 256 * u] = v[u];
            ss += v[u].x * v[u].x + v[u].y * v[u].y + v[u].z * v[u].z + v[u].w * v[u].w;
        }
    ss = wave_sum(ss);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    ss = red[0] + red[1] + red[2] + red[3];
    row_emit<PL>(v, row_scale<PL>(ss, d, eps), gn, d, tid, m, out_hi, out_lo, out_lo2);
}

// Last row of group `group` only: out[:] = x[row] + sum_s P[s][row]  (residual stream handed to the
// single-row output head); the step descriptor gets the group's sequence.
__global__ __launch_bounds__(256) void k_chunk_last_row(const float* __restrict__ x, const float* __restrict__ P, int S,
                                                        size_t s_stride, int n_stride, int d, ChunkTab tab,
                                                        int group, StepDesc* step, float* __restrict__ out) {
    const ChunkGroup G = tab.group[group];
    const int row = G.row0 + G.n - 1;
    if (blockIdx.x == 0 && threadIdx.x == 0) step->seq = G.seq;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < d; i += gridDim.x * 256) {
        float v = x[(size_t)row * d + i];
        for (int s = 0; s < S; ++s) v += P[s * s_stride + (size_t)row * n_stride + i];
        out[i] = v;
    }
}

// Workgroup = group: if the group wants logits, its last row (residual + down-projection partials), normalised
// with the final gain, becomes row `head` of the tiled planes that feed the output-head product.
__global__ __launch_bounds__(256) void k_chunk_head_rows(const float* __restrict__ x, const float* __restrict__ P, int S,
                                                         size_t s_stride, int n_stride, const float* __restrict__ gain,
                                                         float eps, int d, ChunkTab tab,
                                                         bf16_t* __restrict__ out_hi, bf16_t* __restrict__ out_lo) {
    __shared__ float red[4];
    const ChunkGroup G = tab.group[blockIdx.x];
    if (G.head < 0) return;
    const int row = G.row0 + G.n - 1, tid = threadIdx.x, d4 = d >> 2;
    float4 v[ROW_VEC_MAX], gn[ROW_VEC_MAX];
    const float ss = row_gather<CHUNK_GEMM_MAX_SPLIT>(x + (size_t)row * d, P + (size_t)row * n_stride, S, s_stride, d4, tid, gain, v, gn, red);
    row_emit<2>(v, rsqrtf(ss / (float)d + eps), gn, d, tid, G.head, out_hi, out_lo, nullptr);
}

// Row `head` of the output-head product of every group that wants logits -> logits of its sequence, greedy argmax (lowest
// index on ties) -> next_token.  grid (groups, CHUNK_LOGIT_SLICES): a workgroup copies a slice of the row (16 bytes per lane)
// and leaves its maximum; the last one of a group merges them.  Bound by the copy: one workgroup per row took 47 us for 16 rows
// of 128256 logits, 24 slices take 13 us.  No fence: partial results are written through and read past the caches, as
// in PipeSync.
__global__ __launch_bounds__(256) void k_chunk_logits(const float* __restrict__ P, int V, ChunkTab tab, float* __restrict__ logits_base,
                                                      SeqState* st, const int32_t* __restrict__ banned, float* part_v, int32_t* part_i,
                                                      int32_t* counters) {
    __shared__ float sv[4];
    __shared__ int si[4];
    __shared__ int s_last;
    const ChunkGroup G = tab.group[blockIdx.x];
    if (G.head < 0) return;
    const float* src = P + (size_t)G.head * V;
    float* dst = logits_base + (size_t)G.seq * V;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ns = gridDim.y;
    const int per = ((V + ns - 1) / ns + 3) & ~3, i0 = min((int)blockIdx.y * per, V), i1 = min(i0 + per, V);      // V is a multiple of 128
    const int32_t* ban = banned + (size_t)G.seq * (1 + BAN_MAX);
    const int nban = ban[0];
    float bv = -INFINITY; int bi = 0x7fffffff;
    auto take = [&](float v, int i) {
        bool allowed = true;
        for (int k = 0; k < nban; ++k) allowed = allowed && i != ban[1 + k];
        if (allowed && (v > bv || (v == bv && i < bi))) { bv = v; bi = i; }
    };
    for (int i = i0 + 4 * tid; i < i1; i += 1024) {
        const float4 v = *reinterpret_cast<const float4*>(src + i);
        *reinterpret_cast<float4*>(dst + i) = v;
        take(v.x, i); take(v.y, i + 1); take(v.z, i + 2); take(v.w, i + 3);
    }
    auto reduce = [&]() {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const float ov = __shfl_xor(bv, o, 64); const int oi = __shfl_xor(bi, o, 64);
            if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
        }
    };
    reduce();
    if (lane == 0) { sv[wave] = bv; si[wave] = bi; }
    __syncthreads();
    const size_t slot = (size_t)blockIdx.x * ns;
    if (tid == 0) {
        for (int w = 1; w < 4; ++w)
            if (sv[w] > bv || (sv[w] == bv && si[w] < bi)) { bv = sv[w]; bi = si[w]; }
        __hip_atomic_store(part_v + slot + blockIdx.y, bv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(part_i + slot + blockIdx.y, bi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // both have reached memory before the arrival is counted
        s_last = __hip_atomic_fetch_add(counters + blockIdx.x, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == ns - 1;
    }
    __syncthreads();
    if (!s_last || wave != 0) return;
    bv = -INFINITY; bi = 0x7fffffff;
    if (lane < ns) {
        bv = __hip_atomic_load(part_v + slot + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bi = __hip_atomic_load(part_i + slot + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    reduce();
    if (lane == 0) { st[G.seq].next_token = bi; counters[blockIdx.x] = 0; }
}

// a[m][f] = silu(sum_s gate) * (sum_s up) -> tiled hi/lo planes
__global__ __launch_bounds__(256) void k_chunk_swiglu(const float* __restrict__ P, int S, size_t s_stride, int n_stride,
                                                      int F, bf16_t* __restrict__ out_hi, bf16_t* __restrict__ out_lo) {
    const int m = blockIdx.y;
    const int f = blockIdx.x * 256 + threadIdx.x;
    if (f >= F) return;
    float gt = 0.f, up = 0.f;
    for (int s = 0; s < S; ++s) {
        const float* p = P + s * s_stride + (size_t)m * n_stride;
        gt += p[f]; up += p[F + f];
    }
    bf16_t hi, lo;
    split_bf16(gt / (1.f + expf(-gt)) * up, hi, lo);
    const size_t o = tiled_off(m, f, F);
    out_hi[o] = hi; out_lo[o] = lo;
}

// Rotary embedding of q and k, K/V cache write (row-major planes and the transposed V planes), scaled q
// as hi/lo planes [Hkv][q_cols][dh] with the columns of a group ordered [q head in the kv group][row] (head_dim 128).
// P holds the heads from h0 on (h0 = Hq: keys and values only).
// The first `nrot` workgroups rotate: 16 threads per (row, q or k head), four pairs (i, i + 64) each, 16-byte loads and 8-byte
// stores.  The others write values: a workgroup takes `vrows` consecutive rows of the pass and two heads, a thread one channel;
// the row that starts a run of eight positions (or a group) takes the whole run, because eight positions of a channel lie
// side by side in the transposed planes: one 16-byte store per plane instead of eight of 2 bytes 16 bytes apart from their
// neighbours'.  2048 rows of the 70B shape 45 -> 28 us, 1019 of the 8B shape 20 -> 15, 24 rows 5.1 as before (latency).
constexpr int ROPE_ITEMS = 16;      // (row, head) pairs per rotating workgroup
__global__ __launch_bounds__(256) void k_chunk_rope_kv(const float* __restrict__ P, int S, size_t s_stride, int n_stride, Geom g, ChunkTab tab,
                                                       int rows, const float* __restrict__ rope_cos, const float* __restrict__ rope_sin,
                                                       bf16_t* __restrict__ kv_layer, bf16_t* __restrict__ q_hi, bf16_t* __restrict__ q_lo, int q_cols,
                                                       int h0, int nrot, int vrows) {
    constexpr int DH = 128, half = 64;
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < nrot) {
        const int nh = g.Hq + g.Hkv - h0, item = blockIdx.x * ROPE_ITEMS + (tid >> 4);
        if (item >= rows * nh) return;
        const int m = item / nh, hl = item - m * nh, h = hl + h0, i = 4 * (tid & 15);
        const ChunkRow R = tab.row[m];
        // all partial products of this thread in one round of loads, added in split order
        float4 pa[CHUNK_GEMM_MAX_SPLIT], pb[CHUNK_GEMM_MAX_SPLIT];
#pragma unroll
        for (int s = 0; s < CHUNK_GEMM_MAX_SPLIT; ++s) {
            const float* p = P + (size_t)min(s, S - 1) * s_stride + (size_t)m * n_stride + hl * DH + i;
            pa[s] = *reinterpret_cast<const float4*>(p); pb[s] = *reinterpret_cast<const float4*>(p + half);
        }
        const float4 c = *reinterpret_cast<const float4*>(rope_cos + (size_t)R.pos * half + i);
        const float4 sn = *reinterpret_cast<const float4*>(rope_sin + (size_t)R.pos * half + i);
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
#pragma unroll
        for (int s = 0; s < CHUNK_GEMM_MAX_SPLIT; ++s)
            if (s < S) {
                a.x += pa[s].x; a.y += pa[s].y; a.z += pa[s].z; a.w += pa[s].w;
                b.x += pb[s].x; b.y += pb[s].y; b.z += pb[s].z; b.w += pb[s].w;
            }
        float ra[4] = {a.x * c.x - b.x * sn.x, a.y * c.y - b.y * sn.y, a.z * c.z - b.z * sn.z, a.w * c.w - b.w * sn.w};
        float rb[4] = {b.x * c.x + a.x * sn.x, b.y * c.y + a.y * sn.y, b.z * c.z + a.z * sn.z, b.w * c.w + a.w * sn.w};
        bf16_t *hi, *lo;
        if (h < g.Hq) {
#pragma unroll
            for (int e = 0; e < 4; ++e) { ra[e] *= g.scale; rb[e] *= g.scale; }
            const int G = g.Hq / g.Hkv, kvh = h / G, gq = h - kvh * G;
            const size_t o = ((size_t)kvh * q_cols + (size_t)G * R.row0 + (size_t)gq * R.n + (m - R.row0)) * DH + i;
            hi = q_hi + o; lo = q_lo + o;
        } else {
            hi = kv_layer + (size_t)R.seq * g.kv_seq_stride + (size_t)(h - g.Hq) * g.kv_head_stride + (size_t)R.pos * DH + i;
            lo = hi + g.kv_lo_offset;
        }
        uint32_t h2[4], l2[4];
        split_pair(ra[0], ra[1], h2[0], l2[0]); split_pair(ra[2], ra[3], h2[1], l2[1]);
        split_pair(rb[0], rb[1], h2[2], l2[2]); split_pair(rb[2], rb[3], h2[3], l2[3]);
        *reinterpret_cast<uint2*>(hi) = make_uint2(h2[0], h2[1]); *reinterpret_cast<uint2*>(hi + half) = make_uint2(h2[2], h2[3]);
        *reinterpret_cast<uint2*>(lo) = make_uint2(l2[0], l2[1]); *reinterpret_cast<uint2*>(lo + half) = make_uint2(l2[2], l2[3]);
        return;
    }
    const int hp = (g.Hkv + 1) / 2, item = blockIdx.x - nrot, vh = (item % hp) * 2 + (tid >> 7), ch = tid & 127;
    const int m0 = item / hp * vrows;
    if (vh >= g.Hkv) return;
    for (int mm = m0; mm < min(m0 + vrows, rows); ++mm) {
        const ChunkRow R = tab.row[mm];
        if ((R.pos & 7) != 0 && mm != R.row0) continue;             // in the run of an earlier row
        const int cnt = min(8 - (R.pos & 7), R.row0 + R.n - mm);
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = 0.f;
        const float* p = P + (size_t)mm * n_stride + (size_t)(g.Hq + g.Hkv - h0 + vh) * DH + ch;
        for (int s = 0; s < S; ++s) {
            float t[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) t[k] = p[s * s_stride + (size_t)min(k, cnt - 1) * n_stride];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] += t[k];
        }
        uint32_t hi[4], lo[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) split_pair(v[2 * k], v[2 * k + 1], hi[k], lo[k]);
        bf16_t* head = kv_layer + (size_t)R.seq * g.kv_seq_stride + (size_t)vh * g.kv_head_stride;
        bf16_t* vt = head + g.kv_vt_offset + vt_tile_off(R.pos, ch);
        if (cnt == 8) {
            *reinterpret_cast<uint4*>(vt) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
            *reinterpret_cast<uint4*>(vt + g.kv_lo_offset) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k < cnt) {
                    vt[k] = (bf16_t)(hi[k >> 1] >> (16 * (k & 1)));
                    vt[g.kv_lo_offset + k] = (bf16_t)(lo[k >> 1] >> (16 * (k & 1)));
                }
        }
        if (g.kv_v_offset) {               // row-major values are only kept for the single-row attention kernel
            bf16_t* vr = head + g.kv_v_offset + (size_t)R.pos * DH + ch;
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k < cnt) {
                    vr[(size_t)k * DH] = (bf16_t)(hi[k >> 1] >> (16 * (k & 1)));
                    vr[g.kv_lo_offset + (size_t)k * DH] = (bf16_t)(lo[k >> 1] >> (16 * (k & 1)));
                }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// skinny GEMM on the matrix cores:  P[s][m][n] = sum_{k in slice s} X[m][k] W[n][k]
// ---------------------------------------------------------------------------------------------
// Which kernel takes a pass (launch_chunk_gemm): up to 32 rows this one (bound by the weight stream, a wave per 32
// weight rows); 33-64 rows k_chunk_gemm_ks (the waves split the k-steps); 65-128 rows k_chunk_gemm_wide, a wave
// per row tile; more rows k_chunk_gemm_big.
// Workgroup = 4 waves on 128 weight rows (32 per wave) and one contiguous run of 128-element k-blocks
// (the S workgroups of a row tile split K and write separate partial planes that the consumer adds in
// a fixed order: no atomics, results are bit-reproducible).
//  * weights stream from HBM through a register ring of GEMM_RING tiles per wave (one tile = the wave's
//    32 rows x 128 columns, loaded 4 rows x 256 contiguous bytes per instruction), are transposed into
//    operand order through a wave-private XOR-swizzled LDS tile and multiplied;
//  * the activations of a k-block (32 rows, hi and lo planes: 16 KiB) are shared by the four waves
//    through a double-buffered LDS tile that the workgroup fills one block ahead.
// The loop body has no conditional code around loads or their uses: the requests past the end of a run fetch nothing (weight_run).
// The compiler sinks loads into conditional users
// and then waits for each load right before its product; the scheduling barriers keep the instruction
// scheduler from doing the same within the straight-line body.

constexpr int GEMM_RING = 4;        // weight tiles per wave in the register ring

template <int PL> struct BStage { uint4 v[2 * PL]; };

// Block `blk` of a wave's weight tile.  Not `live` (past the end of the run): zeros, nothing is fetched.
__device__ __forceinline__ void gemm_a_load(uint4 (&a)[8], const WeightTile& t, int blk, bool live) {
    const RunPart part = weight_part(t, blk, live);
    const __amdgpu_buffer_rsrc_t r0 = weight_run(t.w0, part.bytes), r1 = weight_run(t.w1, part.bytes);
#pragma unroll
    for (int q = 0; q < 8; ++q) a[q] = load16_run(q < 4 ? r0 : r1, t.off[q], part.base);
}

// thread tid stages chunks tid and tid + 256 of the 512 16-byte chunks of each 8 KiB plane tile
// off: the thread's byte offset in a tile, past every tile (DEAD_ROW) if its row is past the pass's last one: such rows cost no traffic.  Gate/up of the
// 8B shape with 40 rows 47.4 -> 44.6 us, 48 rows 47.2 -> 45.9, the head with 16 rows 181 -> 178.8 (with blocks past the end of a run
// neither requested nor multiplied: 24 rows 39.6 -> 39.2, the other products 16.0 -> 15.2 on average).
constexpr uint32_t DEAD_ROW = 0x40000000u;
template <int PL>
__device__ __forceinline__ void gemm_b_load(BStage<PL>& st, const bf16_t* const (&x)[PL], int blk, bool live, uint32_t off) {
#pragma unroll
    for (int p = 0; p < PL; ++p) {
        const __amdgpu_buffer_rsrc_t run = weight_run(x[p] + (size_t)blk * 4096, live ? 8192 : 0);
        st.v[2 * p] = load16_run<false>(run, off); st.v[2 * p + 1] = load16_run<false>(run, off + 4096);
    }
}

template <int PL>
__device__ __forceinline__ void gemm_b_store(const BStage<PL>& st, uint4* buf, int tid) {
#pragma unroll
    for (int h = 0; h < 2 * PL; ++h) buf[(h >> 1) * 512 + (h & 1) * 256 + tid] = st.v[h];
}

// Transposes the weight tile into operand order through the wave's LDS tile (32 rows x 16 chunks of
// 16 bytes, chunk c of row r stored at chunk position c ^ (r & 15)), then multiplies it with the
// activation tile in `bt` ([plane][k-step][lane]).  Three planes: the sums of a block of 128 columns start at zero, smallest plane
// first, and are added to the total as a whole, so that a long row costs about as little accuracy as the vector units' tree of sums.
template <int PL>
__device__ __forceinline__ void gemm_tile_mma(const uint4 (&ta)[8], f32x16& acc, uint4* at, const uint4* bt, int lane) {
    {
        const int r0 = lane >> 4, c = lane & 15;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int r = 4 * q + r0;
            at[r * 16 + (c ^ (r & 15))] = ta[q];
        }
    }
    uint4 a[8];
    {
        const int i = lane & 31, gh = lane >> 5;
#pragma unroll
        for (int k = 0; k < 8; ++k) a[k] = at[i * 16 + ((2 * k + gh) ^ (i & 15))];
    }
    if (PL == 3) {
        f32x16 t;
#pragma unroll
        for (int r = 0; r < 16; ++r) t[r] = 0.f;
        auto b_read = [&](int i) { return bt[(2 - i / 8) * 512 + (i % 8) * 64 + lane]; };      // product i: plane 2 - i / 8, step i % 8
        uint4 b[3] = {b_read(0), b_read(1), b_read(2)};
#pragma unroll
        for (int i = 0; i < 24; ++i) {
            __builtin_amdgcn_sched_barrier(0);
            t = mfma_bf16(a[i % 8], b[i % 3], t);
            __builtin_amdgcn_sched_barrier(0);
            if (i + 3 < 24) b[i % 3] = b_read(i + 3);
        }
        acc += t;
        return;
    }
    // The activation operands of k-step k + 1 are read from LDS while the products of step k run (a wave is alone on
    // its SIMD: nothing else hides the LDS latency).
    uint4 b0[2] = {bt[lane], bt[512 + lane]}, b1[2];
#pragma unroll
    for (int k = 0; k < 8; k += 2) {
        b1[0] = bt[(k + 1) * 64 + lane]; b1[1] = bt[512 + (k + 1) * 64 + lane];
        __builtin_amdgcn_sched_barrier(0);
        acc = mfma_bf16(a[k], b0[0], acc);
        acc = mfma_bf16(a[k], b0[1], acc);
        __builtin_amdgcn_sched_barrier(0);
        if (k + 2 < 8) { b0[0] = bt[(k + 2) * 64 + lane]; b0[1] = bt[512 + (k + 2) * 64 + lane]; }
        __builtin_amdgcn_sched_barrier(0);
        acc = mfma_bf16(a[k + 1], b1[0], acc);
        acc = mfma_bf16(a[k + 1], b1[1], acc);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// SWIGLU (S = 1 only): W holds the gate rows [0, N/2) and the up rows [N/2, N).  Wave-tile t = 4 blockIdx.x + wave
// takes `rp` <= 16 gate rows (columns t rp .. t rp + rp - 1 of the result) into tile rows 0..rp-1 and the matching up
// rows into tile rows 16..16+rp-1: in the accumulator layout a gate product and its up product then sit in the same
// lane (registers 4b + r and 4(b + 2) + r), and the wave writes silu(gate) * up as hi/lo planes in operand order
// (act_hi, act_lo; N/2 columns) without any exchange.  The tile rows beyond rp are not fetched (results
// dropped): the launcher picks rp so that the tiles divide evenly among the waves of the device (14 rows for
// F = 14336 on 256 compute units: 1024 tiles), which a fixed 16 or 32 rows per wave would not.
template <bool SWIGLU, int PL>
__global__ __launch_bounds__(256) void k_chunk_gemm(const bf16_t* __restrict__ W, int N, int K,
                                                    const bf16_t* __restrict__ Xhi, const bf16_t* __restrict__ Xlo, const bf16_t* __restrict__ Xlo2,
                                                    float* __restrict__ P, size_t s_stride, int n_stride, int S, int rows,
                                                    bf16_t* __restrict__ act_hi, bf16_t* __restrict__ act_lo, bf16_t* __restrict__ act_lo2, int rp) {
    extern __shared__ uint4 gemm_lds[];             // [4 waves][512] weight tiles, then [2][PL][512] activation tiles
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint4* at = gemm_lds + wave * 512;
    uint4* bt = gemm_lds + 2048;
    constexpr int BT = PL * 512;                    // chunks in one activation buffer
    const int n0 = SWIGLU ? (blockIdx.x * 4 + wave) * rp : blockIdx.x * 128 + wave * 32;     // SWIGLU: first gate row
    const int nr = SWIGLU ? gate_rows(N >> 1, n0, rp) : 32;                                   // SWIGLU: gate rows of this wave
    const int sp = blockIdx.y;
    const int nblk = K >> 7;
    const int b0 = (int)((unsigned)(nblk * sp) / (unsigned)S), b1 = (int)((unsigned)(nblk * (sp + 1)) / (unsigned)S);   // (K / 128) * S < 2^31
    const int nb = b1 - b0;

    const WeightTile wt = SWIGLU ? gate_up_tile(W, N >> 1, K, n0, nr, lane) : weight_tile(W + (size_t)n0 * K, K, lane);
    const bf16_t* x[PL];
    x[0] = Xhi; x[1] = Xlo;
    if (PL > 2) x[PL - 1] = Xlo2;
    const uint32_t xoff = (tid & 31) < rows ? tid * 16 : DEAD_ROW;

    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;

    if (nb > 0) {
        // The workgroups walk their k-blocks in rotated order, each starting somewhere else: workgroups that all
        // read column block 0 of their own rows at the same time (rows are a multiple of 8 KiB apart) load few memory
        // channels at a time, and how badly depends on where the matrix lies (measured on the gate/up product, whose
        // workgroups all start together: 42 to 52 us for the same shape at different addresses).  Block i of the
        // walk is b0 + (i + rot) mod nb.
        const int rot = (int)((blockIdx.x / 8 + (blockIdx.x & 7) * 4 + blockIdx.y * 3) % (unsigned)nb);
        auto blk = [&](int i) { const int x = min(i, nb - 1) + rot; return b0 + (x >= nb ? x - nb : x); };
        // Waits are in issue order, so the activation loads of block t+2 are issued before the weight loads of
        // the newest block: waiting for the activations of block t+1 (to store them) then leaves the two newest
        // weight tiles in flight.
        constexpr int RING = GEMM_RING;
        uint4 ring[RING][8];
        BStage<PL> st[2];
        gemm_b_load<PL>(st[0], x, blk(0), true, xoff);
        gemm_b_load<PL>(st[1], x, blk(1), 1 < nb, xoff);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < RING - 1; ++u) gemm_a_load(ring[u], wt, blk(u), u < nb);
        gemm_b_store<PL>(st[0], bt, tid);
        __syncthreads();
        static_assert(RING % 2 == 0, "ring slot (u % RING) and activation buffer (u & 1) are static");
        for (int t = 0; t < nb; t += RING) {
#pragma unroll
            for (int u = 0; u < RING; ++u) {
                const int tt = t + u;                       // this block of the walk
                gemm_b_load<PL>(st[u & 1], x, blk(tt + 2), tt + 2 < nb, xoff);
                __builtin_amdgcn_sched_barrier(0);
                gemm_a_load(ring[(u + RING - 1) % RING], wt, blk(tt + RING - 1), tt + RING - 1 < nb);
                __builtin_amdgcn_sched_barrier(0);
                if (tt < nb) gemm_tile_mma<PL>(ring[u % RING], acc, at, bt + (u & 1) * BT, lane);        // uniform
                __builtin_amdgcn_sched_barrier(0);
                gemm_b_store<PL>(st[(u + 1) & 1], bt + ((u + 1) & 1) * BT, tid);
                __syncthreads();
            }
        }
    }

    // lane (j, g) holds D[8b + 4g + r][j] in register 4b + r: four consecutive weight rows of token row j.  Nobody reads rows past the last.
    if ((lane & 31) >= rows) return;
    if (SWIGLU) {
        const int F = N >> 1;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int slot = 8 * b + 4 * (lane >> 5) + r;
                if (slot < nr) {
                    const float gt = acc[4 * b + r], up = acc[4 * (b + 2) + r];
                    bf16_t e[PL];
                    split_planes<PL>(gt / (1.f + expf(-gt)) * up, e);
                    const size_t o = tiled_off(lane & 31, n0 + slot, F);
                    act_hi[o] = e[0]; act_lo[o] = e[1];
                    if (PL > 2) act_lo2[o] = e[PL - 1];
                }
            }
        return;
    }
    float* prow = P + sp * s_stride + (size_t)(lane & 31) * n_stride + n0 + 4 * (lane >> 5);
#pragma unroll
    for (int b = 0; b < 4; ++b) *(float4*)(prow + 8 * b) = make_float4(acc[4 * b], acc[4 * b + 1], acc[4 * b + 2], acc[4 * b + 3]);
}

// ---------------------------------------------------------------------------------------------
// wide GEMM on the matrix cores for passes of 65-128 rows
// ---------------------------------------------------------------------------------------------
// Workgroup = 4 waves on a tile of 128 weight rows x 128 token rows and one run of k-blocks:
//  * every wave multiplies ALL 128 weight rows of the tile with its own row tile (32 token rows):
//    per 16-column k-step 4 weight operands and 2 activation operands (hi, lo) feed 8 products;
//  * the weight block (128 rows x 128 columns) is loaded once per workgroup (4 rows x 256 contiguous bytes
//    per instruction), transposed into operand order through a double-buffered, XOR-swizzled LDS tile that
//    the waves share: one barrier per k-block;
//  * the activations are already in operand order in global memory (tiled planes: one contiguous KiB per
//    wave-wide load) and go straight to registers through a ring of four 2-step units, three units ahead of
//    the products; no wave reads another wave's rows, so they never pass through LDS.

// activations of MW row tiles (one here, two in k_chunk_gemm_ks)
template <int MW, int PL = 2> struct BUnit { uint4 v[MW][2][PL]; };      // [row tile][k-step of the unit][plane]

// x: the row tiles' planes; off: the lane's byte offset in an operand of each, or DEAD_ROW
template <int MW, int PL>
__device__ __forceinline__ void wide_b_load(BUnit<MW, PL>& b, const bf16_t* const (&x)[MW][PL], const uint32_t (&off)[MW], int blk, int unit, bool live) {
#pragma unroll
    for (int j = 0; j < MW; ++j)
#pragma unroll
        for (int p = 0; p < PL; ++p) {
            const __amdgpu_buffer_rsrc_t run = weight_run(x[j][p] + ((size_t)blk * 8 + unit * 2) * 512, live ? 2048 : 0);
#pragma unroll
            for (int st = 0; st < 2; ++st) b.v[j][st][p] = load16_run<false>(run, off[j] + st * 1024);
        }
}

// weight operands of k-step k: all four 32-row tiles of the block in `at`
__device__ __forceinline__ void wide_a_read(uint4 (&a)[4], const uint4* at, int k, int lane) {
    const int i = lane & 31, gh = lane >> 5;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) a[nt] = at[nt * 512 + i * 16 + ((2 * k + gh) ^ (i & 15))];
}

template <int MW>
__device__ __forceinline__ void wide_step(const uint4 (&a)[4], const BUnit<MW>& b, int st, f32x16 (&acc)[4][MW]) {
#pragma unroll
    for (int pl = 0; pl < 2; ++pl)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int j = 0; j < MW; ++j) acc[nt][j] = mfma_bf16(a[nt], b.v[j][st][pl], acc[nt][j]);
}

// The products of three planes: `t` takes the largest, `tl` the other two.
__device__ __forceinline__ void wide_step3(const uint4 (&a)[4], const BUnit<1, 3>& b, int st, f32x16 (&t)[4], f32x16 (&tl)[4]) {
#pragma unroll
    for (int pl = 2; pl >= 0; --pl)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            f32x16& d = pl ? tl[nt] : t[nt];
            d = mfma_bf16(a[nt], b.v[0][st][pl], d);
        }
}

// Three planes (PL = 3): any number of row tiles, four per workgroup; the workgroups of one weight tile sit next to each other on one
// XCD and share the weights in its L2.  The sums of a block of 128 columns start at zero and are added to the total as a whole (see
// gemm_tile_mma); the two small planes have a total of their own.
//
// SWIGLU: W holds the gate rows [0, N/2) and the up rows [N/2, N) of a feed-forward block.  The workgroup
// takes 64 gate rows and the 64 up rows of the same columns (weight-row tiles 0, 1 and 2, 3), and its
// epilogue writes silu(gate) * up as hi/lo planes in operand order (act_hi, act_lo; N/2 columns) instead of
// the fp32 products: S must be 1.
template <bool SWIGLU, int PL>
__global__ __launch_bounds__(256) void k_chunk_gemm_wide(const bf16_t* __restrict__ W, int N, int K,
                                                             const bf16_t* __restrict__ Xhi, const bf16_t* __restrict__ Xlo, const bf16_t* __restrict__ Xlo2,
                                                             float* __restrict__ P, size_t s_stride, int n_stride, int S, int rows,
                                                             bf16_t* __restrict__ act_hi, bf16_t* __restrict__ act_lo, bf16_t* __restrict__ act_lo2) {
    extern __shared__ uint4 gemm_lds[];             // [2 buffers][4 weight-row tiles][512]
    constexpr int QN = 8;                           // weight loads per thread and block: wave w stages rows 32 w ...
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles = N >> 7, MT = (rows + 31) >> 5;
    int q0 = blockIdx.x, my = 0;
    if (PL == 3) {
        const int MY = (MT + 3) >> 2, total = gridDim.x / MY;       // weight tiles x splits
        if ((total & 7) == 0) { const int r = q0 >> 3; my = r % MY; q0 = (r / MY) * 8 + (q0 & 7); }
        else { my = q0 % MY; q0 /= MY; }
    }
    const int ntile = q0 % tiles, sp = q0 / tiles, mtile = my * 4 + wave;
    const int nblk = K >> 7;
    const int b0 = (int)((unsigned)(nblk * sp) / (unsigned)S), b1 = (int)((unsigned)(nblk * (sp + 1)) / (unsigned)S);   // (K / 128) * S < 2^31
    const int nb = b1 - b0, last = b1 - 1;
    const int n0 = ntile * 128;

    // weights: load q of a thread covers row 32 wave + 4 q + lane / 16 of the tile, 16-byte chunk lane % 16
    const int wrow = SWIGLU ? (wave < 2 ? 0 : N >> 1) + ntile * 64 + (wave & 1) * 32 : n0 + wave * 32;
    const WeightTile wt = weight_tile(W + (size_t)wrow * K, K, lane);
    int wslot[QN];
#pragma unroll
    for (int q = 0; q < QN; ++q) {
        const int r = 4 * q + (lane >> 4), c = lane & 15;
        wslot[q] = wave * 512 + r * 16 + (c ^ (r & 15));
    }
    // activations: a row tile per wave; waves past the last tile repeat it and store nothing
    const size_t xo = (size_t)min(mtile, MT - 1) * nblk * 4096;
    const bf16_t* x[1][PL];
    x[0][0] = Xhi + xo; x[0][1] = Xlo + xo;
    const uint32_t xoff[1] = {min(mtile, MT - 1) * 32 + (lane & 31) < rows ? lane * 16u : DEAD_ROW};
    if (PL > 2) x[0][PL - 1] = Xlo2 + xo;

    f32x16 acc[4][1];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[nt][0][r] = 0.f;
    f32x16 bs[PL > 2 ? 4 : 1], tl[PL > 2 ? 4 : 1];                 // three planes: sums of a block, total of the small planes
    if constexpr (PL > 2) {
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) tl[nt] = acc[nt][0];
    }

    if (nb > 0) {
        uint4 wreg[QN];
        BUnit<1, PL> ring[4];
        auto w_load = [&](int blk) { gemm_a_load(wreg, wt, blk, blk <= last); };
        auto w_store = [&](uint4* at) {
#pragma unroll
            for (int q = 0; q < QN; ++q) at[wslot[q]] = wreg[q];
        };
        // issue order = completion order: weights of the first block, three activation units, weights of the second block
        w_load(b0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 3; ++u) wide_b_load<1, PL>(ring[u], x, xoff, b0, u, true);
        __builtin_amdgcn_sched_barrier(0);
        w_store(gemm_lds);
        w_load(b0 + 1);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        for (int t = 0; t < nb; t += 2) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int tt = b0 + t + h;                  // this block, in LDS buffer h
                if (tt > last) break;                       // uniform
                const uint4* at = gemm_lds + h * 2048;
                uint4 a0[4], a1[4];
                wide_a_read(a0, at, 0, lane);
                if constexpr (PL > 2) {
#pragma unroll
                    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                        for (int r = 0; r < 16; ++r) bs[nt][r] = 0.f;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    // unit u + 3 of the stream: the last unit of this block, then the first three of the next
                    wide_b_load<1, PL>(ring[(u + 3) & 3], x, xoff, u == 0 ? tt : tt + 1, (u + 3) & 3, u == 0 || tt < last);
                    __builtin_amdgcn_sched_barrier(0);
                    if (u == 1) {
                        // the next block's weights (requested one block ago) move to the other LDS buffer, whose
                        // readers passed the barrier that ended the previous block; then the block after is requested
                        w_store(gemm_lds + (h ^ 1) * 2048);
                        w_load(tt + 2);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    wide_a_read(a1, at, 2 * u + 1, lane);
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (PL > 2) wide_step3(a0, ring[u], 0, bs, tl);
                    else wide_step<1>(a0, ring[u], 0, acc);
                    __builtin_amdgcn_sched_barrier(0);
                    if (u < 3) wide_a_read(a0, at, 2 * u + 2, lane);
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (PL > 2) wide_step3(a1, ring[u], 1, bs, tl);
                    else wide_step<1>(a1, ring[u], 1, acc);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (PL > 2) {
#pragma unroll
                    for (int nt = 0; nt < 4; ++nt) acc[nt][0] += bs[nt];
                }
                __syncthreads();
            }
        }
        if constexpr (PL > 2) {
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) acc[nt][0] += tl[nt];
        }
    }

    // lane (j, g) holds D[8b + 4g + r][j] in register 4b + r: four consecutive weight rows of token row j
    const int m = mtile * 32 + (lane & 31);
    if (m >= rows) return;
    if (SWIGLU) {
        const int F = N >> 1, f0 = ntile * 64 + 4 * (lane >> 5);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                bf16_t e[4][PL];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float gt = acc[nt][0][4 * b + r], up = acc[nt + 2][0][4 * b + r];
                    split_planes<PL>(gt / (1.f + expf(-gt)) * up, e[r]);
                }
                const size_t o = tiled_off(m, f0 + nt * 32 + 8 * b, F);         // four columns inside one 8-element group
                *reinterpret_cast<uint2*>(act_hi + o) = plane_quad<PL>(e, 0);
                *reinterpret_cast<uint2*>(act_lo + o) = plane_quad<PL>(e, 1);
                if (PL > 2) *reinterpret_cast<uint2*>(act_lo2 + o) = plane_quad<PL>(e, PL - 1);
            }
        return;
    }
    float* prow = P + sp * s_stride + (size_t)m * n_stride + n0 + 4 * (lane >> 5);
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int b = 0; b < 4; ++b)
            *(float4*)(prow + nt * 32 + 8 * b) = make_float4(acc[nt][0][4 * b], acc[nt][0][4 * b + 1], acc[nt][0][4 * b + 2], acc[nt][0][4 * b + 3]);
}

// ---------------------------------------------------------------------------------------------
// large GEMM on the matrix cores for passes of more than 128 rows (prefill, long interrupts, large batched steps)
// ---------------------------------------------------------------------------------------------
// Workgroup = 4 waves, one per SIMD, on a tile of 32 NT weight rows (NT = 4..8) x 256 token rows and one run of k-blocks.
// Every wave multiplies all NT weight-row tiles with its own two row tiles: per 16-column step NT weight and 4 activation
// operands (hi, lo) feed 4 NT products.  Such a pass is bound by the matrix cores and, with operands that are not zero, by
// the power they may take, so the loop is made for few bytes per product and no idle issue slots:
//  * weights and activations of a block of 32 columns go from global memory straight to LDS (16 bytes per lane and load,
//    no registers): three buffers, the block after next is requested while a block is multiplied.  The weights are
//    row-major in memory; the transposition into operand order is the choice of the 16-byte piece a lane loads (LDS row r,
//    piece p holds piece p ^ ((r / 4) & 3) of the row: the 16 rows that a read takes at a time then cover all 64 banks once.  With (r / 2) & 3,
//    eight rows over half of them, 29.4 of the 75.5 M LDS cycles of gate/up of 2048 rows were conflicts, now none of 46.1.  Time does not follow, the
//    power limit binds: 781 and 787 us before, 781 and 784 after (two runs of the kernel trace), in a 16k prompt 727 / 725-726).
//  * every load and every LDS read is issued between two products.  Issued together at the start of a block, the same
//    loads kept the matrix cores idle for 40 % of the time (0.94-1.17 PFLOP/s); spread, the cores are busy 87-91 % of the
//    cycles and the clock drops to the power limit instead (1.3-1.7 GHz with random operands, 2.4 with zeros).
//  * one barrier per block, after the operands of its last step are in registers.
// NT and the split of K come from pick_gemm_plan: the tiles should fill whole rounds of one workgroup per compute unit.
// Measured stand-alone, random operands, counted with both planes: gate/up of the 8B shape (28672 x 4096) 512 rows 204 us =
// 1.18 PFLOP/s, 2048 rows 736 us = 1.31; down of the 70B shape (8192 x 28672), 2048 rows 1.38.  The kernel before this one
// (128 weight rows per workgroup, activations straight to registers): 225 us = 1.07 at 512 rows.  The same matrix
// instruction in a loop without any loads sustains 1.82 PFLOP/s with random operands.

typedef __attribute__((address_space(3))) void* lds_ptr;
typedef const __attribute__((address_space(1))) void* global_ptr;

constexpr int BIG_M = 8;                                    // row tiles per workgroup
template <int NT> struct BigShape {
    static constexpr int W_BYTES = NT * 2048, BUF = W_BYTES + BIG_M * 4096;     // 32 columns: weights, then [row tile][plane][step] KiB
    static constexpr int LW = (2 * NT + 3) / 4, L = LW + 8;                     // loads per wave and block: weights, all
};
template <int NT> struct BigPtrs {
    const bf16_t* w[BigShape<NT>::LW];
    int w_off[BigShape<NT>::LW];
    const bf16_t* x[2][2];                                  // [row tile][plane]
};
struct BigLane { int a0, a1, b, wave; };                    // LDS offsets of the lane's operands: weights of step 0 / 1, activations

// Load j of the wave's share of block `blk` (32 columns) into the buffer at `base`.
template <int NT>
__device__ __forceinline__ void big_load(unsigned char* base, const BigPtrs<NT>& p, int blk, int wave, int j) {
    constexpr int LW = BigShape<NT>::LW;
    if (j < LW) {
        __builtin_amdgcn_global_load_lds((global_ptr)(p.w[j] + (size_t)blk * 32), (lds_ptr)(base + p.w_off[j]), 16, 0, 0);
    } else {
        const int q = j - LW, mt = q >> 2, pl = (q >> 1) & 1, st = q & 1;
        __builtin_amdgcn_global_load_lds((global_ptr)(p.x[mt][pl] + ((size_t)blk * 2 + st) * 512),
                                         (lds_ptr)(base + BigShape<NT>::W_BYTES + (((wave * 2 + mt) * 2 + pl) * 2 + st) * 1024), 16, 0, 0);
    }
}

// The 4 NT products of one step; `between(m)` runs after product m.
template <int NT, class F>
__device__ __forceinline__ void big_mma(const u32x4 (&a)[NT], const u32x4 (&x)[2][2], f32x16 (&acc)[NT][2], F&& between) {
#pragma unroll
    for (int pl = 0; pl < 2; ++pl)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                acc[nt][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[nt]), __builtin_bit_cast(bf16x8, x[j][pl]),
                                                                     acc[nt][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                between((pl * NT + nt) * 2 + j);
                __builtin_amdgcn_sched_barrier(0);
            }
}

// One block.  On entry its data are in `rd` for every wave and nobody reads `wr` any more; a1 / x1 hold the operands of
// the previous block's second step.  Requests block `blk` into `wr`, multiplies the previous second step and this block's
// first one, leaves the operands of its second step in a1 / x1 and the next block complete in LDS for every wave.
// The two pointers never meet (the buffers rotate), which the compiler has to know: it would otherwise wait for all
// loads to LDS before every LDS read.  The empty asm statements keep the reads on their side of the barrier.
template <int NT, bool FIRST>
__device__ __forceinline__ void big_block(const unsigned char* __restrict__ rd, unsigned char* __restrict__ wr, const BigPtrs<NT>& p, int blk,
                                          const BigLane& ln, f32x16 (&acc)[NT][2], u32x4 (&a1)[NT], u32x4 (&x1)[2][2]) {
    constexpr int L = BigShape<NT>::L, LA = (L + 1) / 2, STEP = 4 * NT / LA;
    static_assert(STEP >= 1 && NT + 4 <= 4 * NT, "every load and read of a block has a product to stand behind");
    int oa0 = ln.a0, oa1 = ln.a1, ob = ln.b;
    asm volatile("" : "+v"(oa0), "+v"(oa1), "+v"(ob));
    __builtin_amdgcn_sched_barrier(0);
    u32x4 a0[NT], x0[2][2];
    auto read0 = [&](int m) {
        if (m < NT) a0[m] = *(const u32x4*)(rd + m * 2048 + oa0);
        else if (m < NT + 4) x0[(m - NT) >> 1][(m - NT) & 1] = *(const u32x4*)(rd + ob + (m - NT) * 2048);
    };
    if (FIRST) {
#pragma unroll
        for (int j = 0; j < LA; ++j) big_load<NT>(wr, p, blk, ln.wave, j);
#pragma unroll
        for (int m = 0; m < NT + 4; ++m) read0(m);
    } else {
        big_mma<NT>(a1, x1, acc, [&](int m) { read0(m); if (m % STEP == STEP - 1 && m / STEP < LA) big_load<NT>(wr, p, blk, ln.wave, m / STEP); });
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) asm volatile("" : "+v"(a0[nt]));
#pragma unroll
    for (int j = 0; j < 2; ++j) { asm volatile("" : "+v"(x0[j][0])); asm volatile("" : "+v"(x0[j][1])); }
    __builtin_amdgcn_sched_barrier(0);
    big_mma<NT>(a0, x0, acc, [&](int m) {
        if (m < NT) a1[m] = *(const u32x4*)(rd + m * 2048 + oa1);
        else if (m < NT + 4) x1[(m - NT) >> 1][(m - NT) & 1] = *(const u32x4*)(rd + ob + (m - NT) * 2048 + 1024);
        if (m % STEP == STEP - 1 && m / STEP < L - LA) big_load<NT>(wr, p, blk, ln.wave, LA + m / STEP);
    });
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) asm volatile("" : "+v"(a1[nt]));
#pragma unroll
    for (int j = 0; j < 2; ++j) { asm volatile("" : "+v"(x1[j][0])); asm volatile("" : "+v"(x1[j][1])); }
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(L) : "memory");       // this wave's share of the next block has landed ...
    __builtin_amdgcn_s_barrier();                                   // ... and everybody's
    __builtin_amdgcn_sched_barrier(0);
}

// SWIGLU (S = 1): W holds the gate rows [0, N/2) and the up rows [N/2, N); a weight-row tile is 16 gate rows and the 16 up
// rows of the same columns, which end up in the same lane (registers 4b + r and 4(b + 2) + r), and the epilogue writes
// silu(gate) * up as hi/lo planes in operand order.
template <int NT, bool SWIGLU>
__global__ __launch_bounds__(256) void k_chunk_gemm_big(const bf16_t* __restrict__ W, int N, int K, const bf16_t* __restrict__ Xhi,
                                                        const bf16_t* __restrict__ Xlo, float* __restrict__ P, size_t s_stride, int n_stride,
                                                        int S, int MT, int ntiles, bf16_t* __restrict__ act_hi, bf16_t* __restrict__ act_lo) {
    extern __shared__ __align__(1024) unsigned char big_lds[];      // [3 buffers]
    constexpr int BUF = BigShape<NT>::BUF, L = BigShape<NT>::L, LW = BigShape<NT>::LW;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int MY = (MT + BIG_M - 1) / BIG_M;
    int ntile, my, sp;
    {
        // Workgroups go round robin over the XCDs by linear id.  An XCD takes weight tiles of its own, each with two row
        // blocks next to each other, and all of its tiles before the next pair of row blocks: what its 32 compute units
        // read at a time (16 weight tiles, two row blocks) stays in its L2.
        int q = blockIdx.x;
        const int MG = MY & 1 ? 1 : 2;
        if ((ntiles & 7) == 0) {
            const int xcd = q & 7;
            q >>= 3;
            const int mi = q % MG; q /= MG;
            ntile = (q % (ntiles >> 3)) * 8 + xcd; q /= ntiles >> 3;
            my = (q % (MY / MG)) * MG + mi; sp = q / (MY / MG);
        } else {
            my = q % MY; q /= MY;
            ntile = q % ntiles; sp = q / ntiles;
        }
    }
    const int nblk = K >> 7;                                        // (K / 128) * S < 2^31
    const int b0 = (int)((unsigned)(nblk * sp) / (unsigned)S) * 4, nb = (int)((unsigned)(nblk * (sp + 1)) / (unsigned)S) * 4 - b0;
    const int NR = SWIGLU ? N >> 1 : N;                             // rows of the result
    BigPtrs<NT> p;
#pragma unroll
    for (int j = 0; j < LW; ++j) {
        // load q covers LDS rows 16 q .. 16 q + 15 of the tile, four lanes each; past the end the last one again
        const int q = min(wave * LW + j, 2 * NT - 1);
        const int r = 16 * q + (lane >> 2), c = (lane & 3) ^ ((r >> 2) & 3);
        int row;
        if (SWIGLU) {
            const int f = min((ntile * NT + (r >> 5)) * 16 + (r & 15), NR - 1);
            row = (r & 16) ? NR + f : f;
        } else row = min(ntile * NT * 32 + r, NR - 1);
        p.w[j] = W + (size_t)row * K + c * 8;
        p.w_off[j] = q * 1024;
    }
    int mtile[2];                                                   // past the pass's end: the last tile again, not stored
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        mtile[j] = my * BIG_M + wave * 2 + j;
        const size_t o = (size_t)min(mtile[j], MT - 1) * nblk * 4096 + lane * 8;
        p.x[j][0] = Xhi + o; p.x[j][1] = Xlo + o;
    }
    BigLane ln;
    {
        const int i = lane & 31, gh = lane >> 5, z = (i >> 2) & 3;
        ln.a0 = i * 64 + ((gh ^ z) << 4); ln.a1 = i * 64 + (((2 + gh) ^ z) << 4);
        ln.b = BigShape<NT>::W_BYTES + wave * 8192 + lane * 16; ln.wave = wave;
    }
    f32x16 acc[NT][2];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[nt][j][r] = 0.f;

    if (nb > 0) {
        const int last = b0 + nb - 1;                               // nb >= 4
        u32x4 a1[NT], x1[2][2];
#pragma unroll
        for (int j = 0; j < L; ++j) big_load<NT>(big_lds, p, b0, wave, j);
#pragma unroll
        for (int j = 0; j < L; ++j) big_load<NT>(big_lds + BUF, p, b0 + 1, wave, j);
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"(L) : "memory");
        __builtin_amdgcn_s_barrier();
        big_block<NT, true>(big_lds, big_lds + 2 * BUF, p, b0 + 2, ln, acc, a1, x1);
        int cur = 1;
        for (int i = 1; i < nb; ++i) {
            const int prev = cur == 0 ? 2 : cur - 1;                // the buffer of block i - 1 takes block i + 2
            big_block<NT, false>(big_lds + cur * BUF, big_lds + prev * BUF, p, min(b0 + i + 2, last), ln, acc, a1, x1);
            cur = cur == 2 ? 0 : cur + 1;
        }
        big_mma<NT>(a1, x1, acc, [](int) {});
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // no load may still be on its way to LDS when the workgroup ends
    }

    // lane (j, g) holds D[8b + 4g + r][j] in register 4b + r: four consecutive weight rows of token row j
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (mtile[j] >= MT) continue;
        const int m = mtile[j] * 32 + (lane & 31);
        if (SWIGLU) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    const int f = (ntile * NT + nt) * 16 + 8 * b + 4 * (lane >> 5);
                    uint32_t hi[2], lo[2];
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        float v[2];
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            const float gt = acc[nt][j][4 * b + 2 * r + e], up = acc[nt][j][4 * (b + 2) + 2 * r + e];
                            v[e] = gt / (1.f + expf(-gt)) * up;
                        }
                        split_pair(v[0], v[1], hi[r], lo[r]);
                    }
                    if (f < NR) {
                        const size_t o = tiled_off(m, f, NR);       // four columns inside one 8-element group
                        *reinterpret_cast<uint2*>(act_hi + o) = make_uint2(hi[0], hi[1]);
                        *reinterpret_cast<uint2*>(act_lo + o) = make_uint2(lo[0], lo[1]);
                    }
                }
        } else {
            float* prow = P + sp * s_stride + (size_t)m * n_stride;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const int n = (ntile * NT + nt) * 32 + 8 * b + 4 * (lane >> 5);
                    if (n < NR) *(float4*)(prow + n) = make_float4(acc[nt][j][4 * b], acc[nt][j][4 * b + 1], acc[nt][j][4 * b + 2], acc[nt][j][4 * b + 3]);
                }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// GEMM for passes of 33-64 rows: the four waves of a workgroup split the k-steps
// ---------------------------------------------------------------------------------------------
// With two row tiles k_chunk_gemm is bound by LDS: a wave that owns 32 weight rows uses every activation
// operand it reads for one product only.  Here every wave multiplies the whole tile of the workgroup, 128 weight
// rows x all MT row tiles, but only for two of the eight 16-column steps of each k-block (wave w: steps 2w, 2w+1):
// per step 4 weight operands (from the shared LDS tile, staged as in k_chunk_gemm_wide) and 2 MT activation
// operands (straight from the operand-order planes, two blocks ahead) feed 8 MT products, and no operand
// is read by two waves.  The four partial tiles are added through LDS at the end, in wave order.

template <int MT, bool SWIGLU>
__global__ __launch_bounds__(256) void k_chunk_gemm_ks(const bf16_t* __restrict__ W, int N, int K,
                                                       const bf16_t* __restrict__ Xhi, const bf16_t* __restrict__ Xlo,
                                                       float* __restrict__ P, size_t s_stride, int n_stride, int S, int rows,
                                                       bf16_t* __restrict__ act_hi, bf16_t* __restrict__ act_lo) {
    extern __shared__ uint4 gemm_lds[];             // [2 buffers][4 weight-row tiles][512]; reused by the final sum
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntile = blockIdx.x, sp = blockIdx.y;
    const int nblk = K >> 7;
    const int b0 = (int)((unsigned)(nblk * sp) / (unsigned)S), b1 = (int)((unsigned)(nblk * (sp + 1)) / (unsigned)S);   // (K / 128) * S < 2^31
    const int nb = b1 - b0;
    const int n0 = ntile * 128;

    // weights: load q of a thread covers row 32 wave + 4 q + lane / 16 of the tile, 16-byte chunk lane % 16
    const int wrow = SWIGLU ? (wave < 2 ? ntile * 64 + wave * 32 : (N >> 1) + ntile * 64 + (wave - 2) * 32) : n0 + wave * 32;
    const WeightTile wt = weight_tile(W + (size_t)wrow * K, K, lane);
    const int wr0 = lane >> 4, wc = lane & 15;
    const bf16_t* x[MT][2];
    uint32_t xoff[MT];
#pragma unroll
    for (int j = 0; j < MT; ++j) {
        const size_t o = (size_t)j * nblk * 4096;
        x[j][0] = Xhi + o; x[j][1] = Xlo + o;
        xoff[j] = j * 32 + (lane & 31) < rows ? lane * 16 : DEAD_ROW;
    }

    f32x16 acc[4][MT];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[nt][j][r] = 0.f;

    if (nb > 0) {
        // A block is short (32 products per wave with two row tiles), so the weights of block b0 + i travel in register
        // set i % 2, requested two blocks ahead of their use, and the activations (from L2) one block ahead.  What bounds it is the
        // memory with the activations beside the weights (gate/up of 40 rows 48.9 us when they were loaded whole: 42.4 without them, 45.8 without products);
        // activations two or three blocks ahead 48.5 and 47.0 us, three or four weight sets 48.9 and 47.8, eight waves 48.5, this 46.1 (then less the dead rows).
        // (Three row tiles do not fit the register file this way; they take k_chunk_gemm_wide with an idle wave.)
        static_assert(MT == 2, "register budget");
        // rotated walk over the k-blocks, as in k_chunk_gemm: block i of the walk is b0 + (i + rot) mod nb
        const int rot = (int)((blockIdx.x / 8 + (blockIdx.x & 7) * 4 + blockIdx.y * 3) % (unsigned)nb);
        auto blk = [&](int i) { const int x = min(i, nb - 1) + rot; return b0 + (x >= nb ? x - nb : x); };
        constexpr int NSET = 2, RING = 2, UNROLL = 2;   // LDS buffer u % 2 and ring slot u % RING are static
        uint4 wreg[NSET][8];
        BUnit<MT> ring[RING];
        auto w_load = [&](uint4 (&set)[8], int i) { gemm_a_load(set, wt, blk(i), i < nb); };      // block i of the walk
        auto w_store = [&](const uint4 (&set)[8], uint4* at) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int r = 4 * q + wr0;
                at[wave * 512 + r * 16 + (wc ^ (r & 15))] = set[q];
            }
        };
        // issue order = completion order: weights of the first block, activations of the first, weights of the second
        w_load(wreg[0], 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < RING - 1; ++i) wide_b_load<MT, 2>(ring[i], x, xoff, blk(i), wave, i < nb);
        __builtin_amdgcn_sched_barrier(0);
        w_store(wreg[0], gemm_lds);
        w_load(wreg[NSET - 1], 1);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        for (int t = 0; t < nb; t += UNROLL) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const int tt = t + u;                       // this block of the walk: LDS buffer u % 2, ring slot u % RING
                const uint4* at = gemm_lds + (u & 1) * 2048;
                uint4* other = gemm_lds + ((u & 1) ^ 1) * 2048;   // its readers passed the barrier that ended the previous block
                wide_b_load<MT, 2>(ring[(u + RING - 1) % RING], x, xoff, blk(tt + RING - 1), wave, tt + RING - 1 < nb);
                __builtin_amdgcn_sched_barrier(0);
                w_load(wreg[u & 1], tt + 2);           // this set's previous block was stored one block ago
                __builtin_amdgcn_sched_barrier(0);
                if (tt < nb) {                              // uniform
                    uint4 a0[4], a1[4];
                    wide_a_read(a0, at, 2 * wave, lane);
                    wide_a_read(a1, at, 2 * wave + 1, lane);
                    __builtin_amdgcn_sched_barrier(0);
                    wide_step<MT>(a0, ring[u % RING], 0, acc);
                    __builtin_amdgcn_sched_barrier(0);
                    wide_step<MT>(a1, ring[u % RING], 1, acc);
                    __builtin_amdgcn_sched_barrier(0);
                }
                __builtin_amdgcn_sched_barrier(0);
                w_store(wreg[(u + 1) & 1], other);          // the next block's weights, requested two blocks ago
                __syncthreads();
            }
        }
    }

    // sum of the four waves' partial tiles, one row tile at a time: [wave][weight-row tile][register quad][lane] float4
    float4* ex = reinterpret_cast<float4*>(gemm_lds);
#pragma unroll
    for (int j = 0; j < MT; ++j) {
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                ex[((wave * 4 + nt) * 4 + b) * 64 + lane] = make_float4(acc[nt][j][4 * b], acc[nt][j][4 * b + 1], acc[nt][j][4 * b + 2], acc[nt][j][4 * b + 3]);
        __syncthreads();
        // lane (j, g) holds D[8b + 4g + r][j] in register 4b + r: four consecutive weight rows of token row j
        const int m = j * 32 + (lane & 31);
        if (SWIGLU) {
            if (wave < 2) {                                 // wave w: gate tile w and up tile w + 2 (rows past the last too: a microsecond faster)
                const int F = N >> 1, f0 = ntile * 64 + wave * 32 + 4 * (lane >> 5);
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    float4 gt = ex[((0 * 4 + wave) * 4 + b) * 64 + lane], up = ex[((0 * 4 + wave + 2) * 4 + b) * 64 + lane];
#pragma unroll
                    for (int w = 1; w < 4; ++w) {
                        const float4 g2 = ex[((w * 4 + wave) * 4 + b) * 64 + lane], u2 = ex[((w * 4 + wave + 2) * 4 + b) * 64 + lane];
                        gt.x += g2.x; gt.y += g2.y; gt.z += g2.z; gt.w += g2.w;
                        up.x += u2.x; up.y += u2.y; up.z += u2.z; up.w += u2.w;
                    }
                    const float gv[4] = {gt.x, gt.y, gt.z, gt.w}, uv[4] = {up.x, up.y, up.z, up.w};
                    bf16_t hi[4], lo[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) split_bf16(gv[r] / (1.f + expf(-gv[r])) * uv[r], hi[r], lo[r]);
                    const size_t o = tiled_off(m, f0 + 8 * b, F);       // four columns inside one 8-element group
                    *reinterpret_cast<uint2*>(act_hi + o) = make_uint2(hi[0] | ((uint32_t)hi[1] << 16), hi[2] | ((uint32_t)hi[3] << 16));
                    *reinterpret_cast<uint2*>(act_lo + o) = make_uint2(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16));
                }
            }
        } else if (m < rows) {                              // wave w: weight-row tile w
            float* prow = P + sp * s_stride + (size_t)m * n_stride + n0 + wave * 32 + 4 * (lane >> 5);
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                float4 v = ex[((0 * 4 + wave) * 4 + b) * 64 + lane];
#pragma unroll
                for (int w = 1; w < 4; ++w) {
                    const float4 v2 = ex[((w * 4 + wave) * 4 + b) * 64 + lane];
                    v.x += v2.x; v.y += v2.y; v.z += v2.z; v.w += v2.w;
                }
                *(float4*)(prow + 8 * b) = v;
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------------
// causal chunk attention on the matrix cores (head_dim 128, paired bf16 cache)
// ---------------------------------------------------------------------------------------------
// One wave = one (task, kv head, key split); a task is a tile of 32 query columns of one group, the columns
// of a group being (q head within the kv group, row) pairs, so a single-row group of a 4:1 model fills
// 4 columns and a 24-row group three tiles.  Per 32-key tile the wave loads K and V^T (both planes) at once,
// forms S^T = K Q^T (keys along D rows), does the online softmax per query column, and accumulates
// O^T += V^T P^T.  Key rows are permuted so that the D registers of a lane hold 16 consecutive keys, which
// makes P directly usable as the next B operand.

struct ChunkAttnArgs {
    const bf16_t* q_hi; const bf16_t* q_lo;     // [Hkv][q_cols][128], scaled by 1/sqrt(dh)
    const bf16_t* kv_layer;
    ChunkTab tab;
    float* part_o;      // [unit][128][32]
    float* part_ml;     // [unit][2][32]
    bf16_t* out_hi; bf16_t* out_lo;             // tiled planes (one split: no merge)
    int32_t nsplit /* k_chunk_attn */, q_cols;
};

// K tile (32 keys x 128 channels, one plane) as loaded: instruction q covers rows 4q .. 4q+3, lane l holds
// row 4q + l/16, 16-byte chunk l%16 (1 KiB contiguous per instruction).  Not `live`, here and for the values: past the wave's last tile,
// nothing is fetched (weight_run).  STREAM: nobody else reads these keys and values: they leave no lines in the caches, which is the
// faster way through them (decoding step at 16k keys 26.9 -> 24.7 us, and its merge 5.8 -> 4.7; 16 sequences in the shared-key kernel 73.0 -> 66.3; but where
// two blocks of tasks read the same keys, 48 rows into 16k, 50.5 -> 52.6).
template <bool STREAM>
__device__ __forceinline__ void attn_k_load(uint4 (&kh)[8], uint4 (&kl)[8], const bf16_t* Kp, size_t lo, int tile, bool live, int lane) {
    const bf16_t* p = Kp + (size_t)tile * 32 * 128;
    const __amdgpu_buffer_rsrc_t hi_run = weight_run(p, live ? 8192 : 0), lo_run = weight_run(p + lo, live ? 8192 : 0);
#pragma unroll
    for (int q = 0; q < 8; ++q) { kh[q] = load16_run<STREAM>(hi_run, lane * 16 + q * 1024); kl[q] = load16_run<STREAM>(lo_run, lane * 16 + q * 1024); }
}

// V^T tile (both planes) in operand order: instruction (dt, t) is one contiguous KiB in lane order.
template <bool STREAM>
__device__ __forceinline__ void attn_v_load(uint4 (&vh)[8], uint4 (&vl)[8], const bf16_t* Vt, size_t lo, int tile, bool live, int lane) {
    const bf16_t* p = Vt + (size_t)tile * 8 * 64 * 8;
    const __amdgpu_buffer_rsrc_t hi_run = weight_run(p, live ? 8192 : 0), lo_run = weight_run(p + lo, live ? 8192 : 0);
#pragma unroll
    for (int k = 0; k < 8; ++k) { vh[k] = load16_run<STREAM>(hi_run, lane * 16 + k * 1024); vl[k] = load16_run<STREAM>(lo_run, lane * 16 + k * 1024); }
}

// chunk position of 16-byte chunk c of row r in the wave's LDS tile (conflict-free for the row-wise writes and
// for the reads of the permuted key rows)
__device__ __forceinline__ int attn_k_slot(int r, int c) { return r * 16 + (c ^ ((r & 7) | ((r >> 1) & 8))); }

struct AttnState {
    f32x16 o[4];
    float mrun, lrun;
};

// One 32-key tile: K goes through the wave's LDS tile (attn_stage_k) into A-operand order (key rows permuted so
// that the D registers of a lane hold 16 consecutive keys), then S^T = K Q^T, online softmax, O^T += V^T P^T.
__device__ __forceinline__ void attn_stage_k(const uint4 (&kh)[8], const uint4 (&kl)[8], uint4* kt, int lane) {
    const int r0 = lane >> 4, c = lane & 15;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        kt[attn_k_slot(4 * q + r0, c)] = kh[q];
        kt[512 + attn_k_slot(4 * q + r0, c)] = kl[q];
    }
}

// The per-tile arithmetic outside the matrix cores is what bounds this kernel (a wave is alone on its SIMD and every
// vector instruction takes four cycles), so it is kept short: packed conversions, exp through the hardware exp2,
// and the two steps that most tiles do not need (causal mask away from the diagonal, rescaling of the output when
// no column's maximum moved) are skipped on a wave-uniform test.
__device__ __forceinline__ void attn_tile(AttnState& st, const uint4 (&vh)[8], const uint4 (&vl)[8], const uint4 (&qh)[8],
                                          const uint4 (&ql)[8], const uint4* kt, int key0, int qpos, int lane) {
    const int i = lane & 31, gh = lane >> 5;
    const int krow = (i >> 3) * 4 + (i & 3) + 16 * ((i >> 2) & 1);   // key (within the tile) held in A row i
    // hi.hi + lo.hi + hi.lo accumulate into one register set (back-to-back accumulation), K operands read from LDS
    // two steps ahead
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
    uint4 kq[3][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) { kq[j][0] = kt[attn_k_slot(krow, 2 * j + gh)]; kq[j][1] = kt[512 + attn_k_slot(krow, 2 * j + gh)]; }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        if (t + 2 < 8) {
            kq[(t + 2) % 3][0] = kt[attn_k_slot(krow, 2 * (t + 2) + gh)];
            kq[(t + 2) % 3][1] = kt[512 + attn_k_slot(krow, 2 * (t + 2) + gh)];
        }
        __builtin_amdgcn_sched_barrier(0);
        s = mfma_bf16(kq[t % 3][0], qh[t], s);
        s = mfma_bf16(kq[t % 3][1], qh[t], s);
        s = mfma_bf16(kq[t % 3][0], ql[t], s);
        __builtin_amdgcn_sched_barrier(0);
    }
    // register r of lane (j, g) is key key0 + 16 g + r for query column j
    if (__builtin_amdgcn_ballot_w64(key0 + 31 > qpos) != 0) {        // the tile reaches past some column's position
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (key0 + 16 * gh + r > qpos) s[r] = -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mnew = fmaxf(st.mrun, mx);
    const float msafe = mnew == -INFINITY ? 0.f : mnew;
    const float corr = __expf(st.mrun - msafe);
    float psum = 0.f;
    uint32_t ph[8], pl[8];
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
        const float p0 = __expf(s[r] - msafe), p1 = __expf(s[r + 1] - msafe);
        psum += p0 + p1;
        split_pair(p0, p1, ph[r >> 1], pl[r >> 1]);
    }
    st.lrun = st.lrun * corr + psum;
    if (__builtin_amdgcn_ballot_w64(mnew != st.mrun) != 0) {          // some column's running maximum moved
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) st.o[dt][r] *= corr;
    }
    st.mrun = mnew;
    // consecutive products go to different accumulators
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const uint4 pht = make_uint4(ph[4 * t], ph[4 * t + 1], ph[4 * t + 2], ph[4 * t + 3]);
        const uint4 plt = make_uint4(pl[4 * t], pl[4 * t + 1], pl[4 * t + 2], pl[4 * t + 3]);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) st.o[dt] = mfma_bf16(vh[dt * 2 + t], pht, st.o[dt]);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) st.o[dt] = mfma_bf16(vl[dt * 2 + t], pht, st.o[dt]);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) st.o[dt] = mfma_bf16(vh[dt * 2 + t], plt, st.o[dt]);
    }
}

__global__ __launch_bounds__(256) void k_chunk_attn(ChunkAttnArgs a, Geom g) {
    constexpr int DH = 128;
    extern __shared__ uint4 attn_lds[];                    // [4 waves][hi | lo][512 chunks] K tiles
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = lane & 31, gh = lane >> 5;
    uint4* kt = attn_lds + wave * 1024;
    const int G = g.Hq / g.Hkv;
    const int kvh = blockIdx.x % g.Hkv, split = blockIdx.y * (int)(blockDim.x >> 6) + wave;
    const ChunkTask T = a.tab.task[blockIdx.x / g.Hkv];
    // Columns 32 tile .. 32 tile + 31 of the group are rows first .. first + 31 of one query head, or wrap into the
    // next head (then the group's last row is among them): no column of the tile sees keys past its latest row.
    const int first = (32 * T.tile) % T.n;
    const int Lk = T.pos0 + min(first + 32, T.n);          // keys 0 .. Lk-1 matter to this tile
    const int ntile = (Lk + 31) >> 5;
    const int tps = (ntile + a.nsplit - 1) / a.nsplit;
    const int t0 = split * tps, t1 = min(ntile, t0 + tps);

    const size_t seq_off = (size_t)T.seq * g.kv_seq_stride + (size_t)kvh * g.kv_head_stride;
    const bf16_t* Kp = a.kv_layer + seq_off;
    const bf16_t* Vt = a.kv_layer + g.kv_vt_offset + seq_off;
    const size_t lo = g.kv_lo_offset;

    // this lane's query column: (q head, row r) of the group; columns past the group are computed and dropped
    const int col = 32 * T.tile + i;
    const int qpos = T.pos0 + col % T.n;

    AttnState st;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) st.o[dt][r] = 0.f;
    st.mrun = -INFINITY; st.lrun = 0.f;

    if (t0 < t1) {
        // B operand of S^T = K Q^T: lane (j, g) holds q[j][16 t + 8 g + e]
        uint4 qh[8], ql[8];
        {
            const size_t qo = ((size_t)kvh * a.q_cols + (size_t)G * T.row0 + col) * DH + gh * 8;
#pragma unroll
            for (int t = 0; t < 8; ++t) { qh[t] = load16(a.q_hi + qo + t * 16); ql[t] = load16(a.q_lo + qo + t * 16); }
        }
        // Once K of a tile is staged in LDS its registers take K of the next tile, and the V
        // registers take the next tile's V as soon as the P V product has used them, so the next tile's loads are in
        // flight while a tile is multiplied.  No conditional code around loads or their uses (the compiler would
        // sink the loads next to the uses); past the wave's last tile they fetch nothing (one tile of a wave's five or six at 16k keys, all of its
        // one tile at 1k: the decoding step's attention 28.5 -> 26.9 and 6.8 -> 6.7 us with its last tile not read again, 24 rows at 1.1k 8.8 -> 8.6).
        uint4 kh[8], kl[8], vh[8], vl[8];
        __builtin_amdgcn_sched_barrier(0);          // issue order q, K, V: the waits in the loop count on it
        attn_k_load<false>(kh, kl, Kp, lo, t0, true, lane);
        __builtin_amdgcn_sched_barrier(0);
        attn_v_load<false>(vh, vl, Vt, lo, t0, true, lane);
        __builtin_amdgcn_sched_barrier(0);
        for (int tile = t0; tile < t1; ++tile) {
            const bool more = tile + 1 < t1;
            attn_stage_k(kh, kl, kt, lane);
            __builtin_amdgcn_sched_barrier(0);
            attn_k_load<false>(kh, kl, Kp, lo, tile + 1, more, lane);
            __builtin_amdgcn_sched_barrier(0);
            attn_tile(st, vh, vl, qh, ql, kt, tile * 32, qpos, lane);
            __builtin_amdgcn_sched_barrier(0);
            attn_v_load<false>(vh, vl, Vt, lo, tile + 1, more, lane);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    st.lrun += __shfl_xor(st.lrun, 32, 64);

    const size_t unit = (size_t)blockIdx.x * a.nsplit + split;
    float* po = a.part_o + unit * DH * 32;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r2 = 0; r2 < 16; ++r2) po[(size_t)(dt * 32 + 8 * (r2 >> 2) + 4 * gh + (r2 & 3)) * 32 + i] = st.o[dt][r2];
    if (gh == 0) {
        float* pm = a.part_ml + unit * 64;
        pm[i] = st.mrun; pm[32 + i] = st.lrun;
    }
}

// ---------------------------------------------------------------------------------------------
// single-row decoding attention on the matrix cores, one kernel
// ---------------------------------------------------------------------------------------------
// grid (Hkv, nsplit / waves per workgroup); wave = (kv head, key split), the q heads of the kv group are the first G query columns
// of the tile (the other columns are zero and dropped).  Keys and values of the wave's first tile are requested
// first, then the step's fp32 query, which is split into bf16 pairs while they arrive.  Each wave leaves the G
// useful columns of its partial result ([G][128] + running maximum and sum); k_decode_attn_merge, a kernel of its
// own, merges the splits that had keys.  (Merging in the same kernel by the workgroup that finishes last needs two
// device-wide fences and a ticket before the partial results can be read, a longer chain than a kernel boundary.)
struct DecodeAttnArgs {
    const float* q;             // [Hq][128] rotated, unscaled
    const StepDesc* step;
    const bf16_t* kv_layer;
    float* part_o;              // [Hkv][nsplit][G][128]
    float* part_ml;             // [Hkv][nsplit][2][G]
    float* out;                 // [Hq][128]
    int32_t nsplit;
    unsigned long long* stamps; // stamp mode of the one-stream step: six words for this kernel, six for the merge
    unsigned long long* done_wg; // ... and STAMP_DONE_SLOTS finishing-time words each
};

__global__ __launch_bounds__(256) void k_decode_attn_mfma(DecodeAttnArgs a, Geom g) {
    constexpr int DH = 128;
    extern __shared__ uint4 attn_lds[];                    // [4 waves][hi | lo][512 chunks] K tiles
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    PipeSync stamp{};
    stamp.stamps = a.stamps; stamp.done_wg = a.done_wg;
    const unsigned long long t_start = clock_if(stamp.done_wg != nullptr);
    const int i = lane & 31, gh = lane >> 5;
    uint4* kt = attn_lds + wave * 1024;
    const int G = g.Hq / g.Hkv;
    const int kvh = blockIdx.x, split = blockIdx.y * (int)(blockDim.x >> 6) + wave, nsplit = a.nsplit;
    const int seq = a.step->seq, pos = a.step->pos;
    const int ntile = (pos + 32) >> 5;                     // keys 0 .. pos
    const int tps = (ntile + nsplit - 1) / nsplit;
    const int t0 = split * tps, t1 = min(ntile, t0 + tps);

    const size_t seq_off = (size_t)seq * g.kv_seq_stride + (size_t)kvh * g.kv_head_stride;
    const bf16_t* Kp = a.kv_layer + seq_off;
    const bf16_t* Vt = a.kv_layer + g.kv_vt_offset + seq_off;
    const size_t lo = g.kv_lo_offset;

    if (t0 < t1) {
        AttnState st;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) st.o[dt][r] = 0.f;
        st.mrun = -INFINITY; st.lrun = 0.f;
        uint4 kh[8], kl[8], vh[8], vl[8];
        __builtin_amdgcn_sched_barrier(0);          // issue order K, V, q: the waits in the loop count on it
        attn_k_load<true>(kh, kl, Kp, lo, t0, true, lane);
        __builtin_amdgcn_sched_barrier(0);
        attn_v_load<true>(vh, vl, Vt, lo, t0, true, lane);
        __builtin_amdgcn_sched_barrier(0);
        // B operand of S^T = K Q^T: lane (j, g) holds q[j][16 t + 8 g + e]; column j is q head j of the kv group
        uint4 qh[8], ql[8];
        {
            const float* qp = a.q + (size_t)(kvh * G + min(i, G - 1)) * DH + gh * 8;
            const float sc = i < G ? g.scale : 0.f;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const float4 v0 = *reinterpret_cast<const float4*>(qp + t * 16), v1 = *reinterpret_cast<const float4*>(qp + t * 16 + 4);
                split_pair(v0.x * sc, v0.y * sc, qh[t].x, ql[t].x); split_pair(v0.z * sc, v0.w * sc, qh[t].y, ql[t].y);
                split_pair(v1.x * sc, v1.y * sc, qh[t].z, ql[t].z); split_pair(v1.z * sc, v1.w * sc, qh[t].w, ql[t].w);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        for (int tile = t0; tile < t1; ++tile) {
            const bool more = tile + 1 < t1;
            attn_stage_k(kh, kl, kt, lane);
            __builtin_amdgcn_sched_barrier(0);
            attn_k_load<true>(kh, kl, Kp, lo, tile + 1, more, lane);
            __builtin_amdgcn_sched_barrier(0);
            attn_tile(st, vh, vl, qh, ql, kt, tile * 32, pos, lane);
            __builtin_amdgcn_sched_barrier(0);
            attn_v_load<true>(vh, vl, Vt, lo, tile + 1, more, lane);
            __builtin_amdgcn_sched_barrier(0);
        }
        st.lrun += __shfl_xor(st.lrun, 32, 64);
        if (i < G) {
            // register r2 of accumulator dt is channel 32 dt + 8 (r2 / 4) + 4 gh + r2 % 4 of column i
            const size_t unit = (size_t)kvh * nsplit + split;
            float* po = a.part_o + (unit * G + i) * DH + 4 * gh;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    *reinterpret_cast<float4*>(po + dt * 32 + 8 * q4) =
                        make_float4(st.o[dt][4 * q4], st.o[dt][4 * q4 + 1], st.o[dt][4 * q4 + 2], st.o[dt][4 * q4 + 3]);
            if (gh == 0) {
                float* pm = a.part_ml + unit * 2 * G;
                pm[i] = st.mrun; pm[G + i] = st.lrun;
            }
        }
    }
    step_stamp_done(stamp, t_start, 0);
}

// Merge of the key splits: grid (Hkv, G * 128 / 64), a workgroup writes 64 of the kv group's G x 128 outputs.  Thread =
// (output, quarter of the splits): the splits are few long chains of loads otherwise (96 splits at a long context), the
// four partial sums of an output meet in LDS and are added in a fixed order.
__global__ __launch_bounds__(256) void k_decode_attn_merge(DecodeAttnArgs a, Geom g) {
    constexpr int DH = 128;
    __shared__ float f[8 * CHUNK_ATTN_MAX_SPLIT];          // [G][nused] weights exp(m_s - M) / L
    __shared__ float red[256];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    PipeSync stamp{};
    stamp.stamps = a.stamps ? a.stamps + 6 : nullptr; stamp.done_wg = a.done_wg ? a.done_wg + STAMP_DONE_SLOTS : nullptr;
    const unsigned long long t_start = clock_if(stamp.done_wg != nullptr);
    const int G = g.Hq / g.Hkv;
    const int kvh = blockIdx.x, nsplit = a.nsplit;
    const int ntile = (a.step->pos + 32) >> 5;
    const int tps = (ntile + nsplit - 1) / nsplit;
    const int nused = (ntile + tps - 1) / tps;             // splits that had keys
    const float* ml = a.part_ml + (size_t)kvh * nsplit * 2 * G;
    const int per = (G * DH + (int)gridDim.y - 1) / (int)gridDim.y;
    const int o0 = blockIdx.y * per, o1 = min(o0 + per, G * DH);
    for (int gq = (o0 >> 7) + wave; gq <= ((o1 - 1) >> 7); gq += 4) {      // the q heads this workgroup writes; lanes over splits
        float M = -INFINITY;
        for (int sp = lane; sp < nused; sp += 64) M = fmaxf(M, ml[sp * 2 * G + gq]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) M = fmaxf(M, __shfl_xor(M, o, 64));
        float L = 0.f;
        for (int sp = lane; sp < nused; sp += 64) {
            const float m = ml[sp * 2 * G + gq];
            const float w = m > -INFINITY ? expf(m - M) : 0.f;
            L += ml[sp * 2 * G + G + gq] * w;
            f[gq * nused + sp] = w;
        }
        L = wave_sum(L);
        const float inv = L > 0.f ? 1.f / L : 0.f;
        for (int sp = lane; sp < nused; sp += 64) f[gq * nused + sp] *= inv;
    }
    __syncthreads();
    for (int base = o0; base < o1; base += 64) {
        const int idx = base + lane;
        float acc = 0.f;
        if (idx < o1) {
            const int gq = idx >> 7, ch = idx & (DH - 1);
            const float* po = a.part_o + ((size_t)kvh * nsplit * G + gq) * DH + ch;
            const float* fw = f + gq * nused;
#pragma unroll 8
            for (int sp = wave; sp < nused; sp += 4) acc = fmaf(po[(size_t)sp * G * DH], fw[sp], acc);
        }
        red[tid] = acc;
        __syncthreads();
        if (wave == 0 && idx < o1)
            a.out[(size_t)kvh * G * DH + idx] = (red[lane] + red[64 + lane]) + (red[128 + lane] + red[192 + lane]);
        __syncthreads();
    }
    step_stamp_done(stamp, t_start, 0);
}

// ---------------------------------------------------------------------------------------------
// the same attention for large groups (prefill, long interrupts): keys and values shared by four tasks
// ---------------------------------------------------------------------------------------------
// Workgroup = (block of up to four consecutive tasks of one group, kv head, key split); wave w works on task w of
// the block (128 query columns per workgroup).  The K and V^T tiles of 32 keys (both planes, 32 KiB) go from global memory
// straight to a double-buffered LDS tile (16 bytes per lane and load, eight loads per wave, issued between the products of
// the tile before): K in the swizzled row layout of attn_k_slot, V^T verbatim (it is stored in operand order).  All four
// waves read their operands from there, a quarter of the traffic from L2 of one wave per task.
// What bounds it: products and softmax alternate in a wave, so one wave per SIMD leaves the matrix cores idle during the
// softmax and behind every LDS read.  The kernel is kept to 256 registers (values are read from LDS when they are used,
// the next tile needs no registers), so that two workgroups share a compute unit and one multiplies while the other
// does its softmax.  2048 rows over 8k keys on average (16k prompt of the 8B shape): 1190 -> 735 us a layer and pass
// (698 now = 1.18 PFLOP/s counted with the three hi/lo products); 48 rows into 16.4k keys 66 -> 51 us (48.7 now) against a wave per task.

// Where a wave's eight loads of a tile come from: four of the 16 KiB of K (4 rows each) and four of the 16 of V^T.  LDS in
// 16-byte chunks: K hi [0, 512), K lo [512, 1024), V^T hi [1024, 1536), V^T lo [1536, 2048).
struct WideSrc {
    const bf16_t* k; const bf16_t* v;       // this wave's plane of K and V^T (waves 0, 1: hi, waves 2, 3: lo)
    uint32_t koff[4], voff;                 // the lane's elements within a tile
    int slot;                               // first LDS chunk of the wave's K loads
};
template <bool STREAM>                      // as for attn_k_load
__device__ __forceinline__ void attn_wide_load(uint4* buf, const WideSrc& w, int tile, int j) {
    const bf16_t* src = j < 4 ? w.k + (size_t)tile * 4096 + w.koff[j & 3] : w.v + (size_t)tile * 4096 + w.voff + (j & 3) * 512;
    __builtin_amdgcn_global_load_lds((global_ptr)src, (lds_ptr)(buf + w.slot + (j < 4 ? 0 : 1024) + (j & 3) * 64), 16, 0, STREAM ? 2 : 0);
}

// One tile: multiplies the tile in `rd` (if `work`) and requests tile `next` into `wr` (MORE).  The buffers never meet, see big_block.
template <bool STREAM, bool MORE>
__device__ __forceinline__ void attn_wide_tile(AttnState& st, const uint4* __restrict__ rd, uint4* __restrict__ wr, const WideSrc& w, int next,
                                               const u32x4 (&qh)[8], const u32x4 (&ql)[8], int key0, int qpos, bool work, int lane) {
    if (!work) {                                                    // uniform over the wave
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (MORE) attn_wide_load<STREAM>(wr, w, next, j);
        return;
    }
    const int i = lane & 31, gh = lane >> 5;
    const int krow = (i >> 3) * 4 + (i & 3) + 16 * ((i >> 2) & 1);  // key (within the tile) held in A row i
    int kbase = krow * 16, kx = attn_k_slot(krow, 0) & 15, vbase = 1024 + lane;
    asm volatile("" : "+v"(kbase), "+v"(vbase));                    // the reads stay behind the barrier before this call
    __builtin_amdgcn_sched_barrier(0);
    const u32x4* kt = reinterpret_cast<const u32x4*>(rd);
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
    auto kread = [&](int t, int pl) { return kt[pl * 512 + kbase + ((2 * t + gh) ^ kx)]; };
    auto mma = [](const u32x4& a, const u32x4& b, const f32x16& c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    };
    u32x4 kq[3][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) { kq[j][0] = kread(j, 0); kq[j][1] = kread(j, 1); }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        if (t + 2 < 8) { kq[(t + 2) % 3][0] = kread(t + 2, 0); kq[(t + 2) % 3][1] = kread(t + 2, 1); }
        __builtin_amdgcn_sched_barrier(0);
        s = mma(kq[t % 3][0], qh[t], s);
        if (MORE) attn_wide_load<STREAM>(wr, w, next, t);
        __builtin_amdgcn_sched_barrier(0);
        s = mma(kq[t % 3][1], qh[t], s);
        s = mma(kq[t % 3][0], ql[t], s);
        __builtin_amdgcn_sched_barrier(0);
    }
    // A wave in its products goes before one in its softmax, so that the two waves of a SIMD do not keep step.  The more keys the more it gives; without / with it,
    // us a layer: 2048 rows after 6k keys 603 / 588, after 14k 1270 / 1203; 70B shape, 2048 rows after none 201 / 184, after 2k 550 / 510; 24 rows into 8k 23.9 / 22.0; 48 into
    // 16k 49.8 / 48.7; 16 sequences 66 / 66; 2048 rows after up to 4k and prompts of 300 to 1464 no difference but 1019 tokens 70.8 / 72.2.  (A 16k
    // prompt with the softmax first is as without, with one workgroup of a unit before the other 2 % slower.)
    __builtin_amdgcn_s_setprio(0);
    u32x4 v0[4];                                                    // the first values are on their way during the softmax
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) v0[dt] = kt[vbase + dt * 128];
    __builtin_amdgcn_sched_barrier(0);
    // register r of lane (j, g) is key key0 + 16 g + r for query column j
    if (__builtin_amdgcn_ballot_w64(key0 + 31 > qpos) != 0) {       // the tile reaches past some column's position
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (key0 + 16 * gh + r > qpos) s[r] = -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mnew = fmaxf(st.mrun, mx);
    const float msafe = mnew == -INFINITY ? 0.f : mnew;
    // exp(s - m) as 2^(s log2(e) - m log2(e)) with one fma per score instead of a difference and a product.  m log2(e) is
    // rounded once: a relative error of |m| 2^-24 in all weights of a tile alike, which matters only between tiles whose m
    // differs; the pairs of bf16 that carry q and k put |s| 2^-17 or more into a score.
    constexpr float LOG2E = 1.44269504088896340736f;
    const float corr = __builtin_amdgcn_exp2f((st.mrun - msafe) * LOG2E), mlog = -msafe * LOG2E;
    float psum = 0.f;
    uint32_t ph[8], pl[8];
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(s[r], LOG2E, mlog)), p1 = __builtin_amdgcn_exp2f(fmaf(s[r + 1], LOG2E, mlog));
        psum += p0 + p1;
        split_pair(p0, p1, ph[r >> 1], pl[r >> 1]);
    }
    st.lrun = st.lrun * corr + psum;
    if (__builtin_amdgcn_ballot_w64(mnew != st.mrun) != 0) {        // some column's running maximum moved
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) st.o[dt][r] *= corr;
    }
    st.mrun = mnew;
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    // V^T chunk (plane, dt, t) is KiB plane * 8 + dt * 2 + t of the values; the next group of four is read while one is multiplied
    u32x4 v1[4];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const u32x4 pht = {ph[4 * t], ph[4 * t + 1], ph[4 * t + 2], ph[4 * t + 3]};
        const u32x4 plt = {pl[4 * t], pl[4 * t + 1], pl[4 * t + 2], pl[4 * t + 3]};
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) v1[dt] = kt[vbase + 512 + dt * 128 + t * 64];        // lo plane
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) st.o[dt] = mma(v0[dt], pht, st.o[dt]);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) st.o[dt] = mma(v0[dt], plt, st.o[dt]);
        __builtin_amdgcn_sched_barrier(0);
        if (t == 0) {
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) v0[dt] = kt[vbase + dt * 128 + 64];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) st.o[dt] = mma(v1[dt], pht, st.o[dt]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

__global__ __launch_bounds__(256, 2) void k_chunk_attn_wide(ChunkAttnArgs a, Geom g) {
    constexpr int DH = 128;
    extern __shared__ uint4 attn_lds[];                    // [2 buffers][2048 chunks]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 31, gh = lane >> 5;
    const int G = g.Hq / g.Hkv;
    const int kvh = blockIdx.x % g.Hkv;
    const ChunkPiece piece = a.tab.piece[blockIdx.x / g.Hkv];
    const int split = piece.split;
    const ChunkTaskBlock B = a.tab.block[piece.block];
    const bool live = wave < B.n;
    const int task = B.task0 + min(wave, B.n - 1);
    const ChunkTask T0 = a.tab.task[B.task0];
    const ChunkTask T = a.tab.task[task];
    // keys that matter to the block's columns (its tasks are consecutive tiles of one group), split evenly
    const int Lk = T0.pos0 + min((32 * T0.tile) % T0.n + 32 * B.n, T0.n);
    const int ntile = (Lk + 31) >> 5, nsplit = T0.nsplit;
    const int tps = (ntile + nsplit - 1) / nsplit;
    const int t0 = split * tps, t1 = min(ntile, t0 + tps);
    // and to this wave's own columns: later tiles are loaded for the other waves but not multiplied here
    const int Lw = T.pos0 + min((32 * T.tile) % T.n + 32, T.n);

    const size_t seq_off = (size_t)T.seq * g.kv_seq_stride + (size_t)kvh * g.kv_head_stride;
    WideSrc w;
    {
        const size_t lo = wave >= 2 ? g.kv_lo_offset : 0;
        w.k = a.kv_layer + seq_off + lo; w.v = a.kv_layer + g.kv_vt_offset + seq_off + lo;
        w.slot = wave * 256; w.voff = (wave & 1) * 2048 + lane * 8;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = ((wave & 1) * 4 + j) * 4 + (lane >> 4), c = (lane & 15) ^ (attn_k_slot(r, 0) & 15);
            w.koff[j] = r * 128 + c * 8;
        }
    }
    const int col = 32 * T.tile + i;
    const int qpos = T.pos0 + col % T.n;

    AttnState st;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) st.o[dt][r] = 0.f;
    st.mrun = -INFINITY; st.lrun = 0.f;

    if (t0 < t1) {
        const bool alone = G * T0.n <= 128;                         // one block of tasks: nobody else reads these keys
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (alone) attn_wide_load<true>(attn_lds, w, t0, j);
            else attn_wide_load<false>(attn_lds, w, t0, j);
        }
        u32x4 qh[8], ql[8];
        {
            const size_t qo = ((size_t)kvh * a.q_cols + (size_t)G * T.row0 + col) * DH + gh * 8;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                qh[t] = *(global_u32x4_ptr)(uintptr_t)(a.q_hi + qo + t * 16);
                ql[t] = *(global_u32x4_ptr)(uintptr_t)(a.q_lo + qo + t * 16);
            }
        }
        auto step = [&](auto stream, auto more, int tile) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this wave's share of the tile has landed ...
            __builtin_amdgcn_s_barrier();                           // ... and everybody's, and the other buffer has been read
            __builtin_amdgcn_sched_barrier(0);
            const int cur = (tile - t0) & 1;
            attn_wide_tile<stream.value, more.value>(st, attn_lds + cur * 2048, attn_lds + (cur ^ 1) * 2048, w, min(tile + 1, t1 - 1), qh, ql, tile * 32, qpos,
                                                     live && tile * 32 < Lw, lane);
        };
        // Streamed tiles leave no lines behind, so the last one is not requested again in place of a next one that does not exist, which would come from memory:
        // 24 rows into 4.2k (two tiles a workgroup) 679 -> 673 us, into 16k (eight) 741 -> 735, four layers; batches no difference beyond noise.  Where
        // others read the tiles too the repeat is a cache hit and stays (without it 0.996x on a 16k prompt).
        if (alone) {                                                // uniform
            for (int tile = t0; tile < t1 - 1; ++tile) step(std::true_type{}, std::true_type{}, tile);
            step(std::true_type{}, std::false_type{}, t1 - 1);
        } else
            for (int tile = t0; tile < t1; ++tile) step(std::false_type{}, std::true_type{}, tile);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // no load may still be on its way to LDS when the workgroup ends
    }
    st.lrun += __shfl_xor(st.lrun, 32, 64);
    if (!live) return;

    if (nsplit == 1) {                                              // nothing to merge: the output goes straight to the tiled planes
        if (col >= G * T.n) return;
        const float inv = st.lrun > 0.f ? 1.f / st.lrun : 0.f;
        const int gq = col / T.n, m = T.row0 + col - gq * T.n, hq = kvh * G + gq;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                uint32_t h0, l0, h1, l1;
                split_pair(st.o[dt][4 * q4] * inv, st.o[dt][4 * q4 + 1] * inv, h0, l0);
                split_pair(st.o[dt][4 * q4 + 2] * inv, st.o[dt][4 * q4 + 3] * inv, h1, l1);
                const size_t o = tiled_off(m, hq * DH + dt * 32 + 8 * q4 + 4 * gh, g.Hq * DH);
                *reinterpret_cast<uint2*>(a.out_hi + o) = make_uint2(h0, h1);
                *reinterpret_cast<uint2*>(a.out_lo + o) = make_uint2(l0, l1);
            }
        return;
    }
    const size_t unit = (size_t)T.unit0 * g.Hkv + (size_t)kvh * nsplit + split;
    float* po = a.part_o + unit * DH * 32;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r2 = 0; r2 < 16; ++r2) po[(size_t)(dt * 32 + 8 * (r2 >> 2) + 4 * gh + (r2 & 3)) * 32 + i] = st.o[dt][r2];
    if (gh == 0) {
        float* pm = a.part_ml + unit * 64;
        pm[i] = st.mrun; pm[32 + i] = st.lrun;
    }
}

// Merge the key splits of one (task, kv head) and emit the attention output as tiled hi/lo planes
// (K = Hq*128).  grid (tasks * Hkv, 4): workgroup y handles channels 32 y .. 32 y + 31.
__global__ __launch_bounds__(256) void k_chunk_attn_combine(const float* __restrict__ part_o, const float* __restrict__ part_ml,
                                                            Geom g, ChunkTab tab,
                                                            bf16_t* __restrict__ out_hi, bf16_t* __restrict__ out_lo) {
    constexpr int DH = 128;
    __shared__ float f[CHUNK_ATTN_MAX_SPLIT][32];          // running maximum of every split, then its weight
    __shared__ float fl[CHUNK_ATTN_MAX_SPLIT][32];         // running sum of every split
    __shared__ float red[8][32];
    const int tid = threadIdx.x;
    const int G = g.Hq / g.Hkv;
    const int kvh = blockIdx.x % g.Hkv;
    const ChunkTask T = tab.task[blockIdx.x / g.Hkv];
    const int nsplit = T.nsplit;
    if (nsplit == 1) return;                               // the attention has written the output itself
    const size_t unit = (size_t)T.unit0 * g.Hkv + (size_t)kvh * nsplit;
    const float* ml = part_ml + unit * 64;
    const int j = tid & 31, dl = tid >> 5;                 // column, channel within a run of 8
    const float* po = part_o + unit * DH * 32 + (size_t)(blockIdx.y * 32 + dl) * 32 + j;
    constexpr int PB = 8;                                  // splits whose partial results are requested together
    float p[PB][4];
    auto p_load = [&](int s0) {
#pragma unroll
        for (int k = 0; k < PB; ++k) {
            const int sc = min(s0 + k, nsplit - 1);
#pragma unroll
            for (int u = 0; u < 4; ++u) p[k][u] = po[(size_t)sc * DH * 32 + u * 8 * 32];
        }
    };
    float inv;
    {
        // statistics per query column: thread (column c, slice q) covers splits q, q + 8, ...; partial results meet in
        // LDS.  Maxima and sums of four splits per thread are requested at once, and with the first of them the partial
        // results of the first PB splits, which do not depend on the statistics.
        const int c = tid & 31, q = tid >> 5;
        float m = -INFINITY;
        for (int s0 = q; s0 < nsplit || s0 == q; s0 += 32) {       // every thread runs the first round: it requests p
            float mv[4], lv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int sc = min(s0 + 8 * k, nsplit - 1);
                mv[k] = ml[sc * 64 + c]; lv[k] = ml[sc * 64 + 32 + c];
            }
            if (s0 == q) p_load(0);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (s0 + 8 * k < nsplit) { f[s0 + 8 * k][c] = mv[k]; fl[s0 + 8 * k][c] = lv[k]; m = fmaxf(m, mv[k]); }
        }
        red[q][c] = m;
        __syncthreads();
        float M = red[0][c];
#pragma unroll
        for (int k = 1; k < 8; ++k) M = fmaxf(M, red[k][c]);
        __syncthreads();
        float lp = 0.f;
        for (int sp = q; sp < nsplit; sp += 8) {
            const float w = f[sp][c] > -INFINITY ? expf(f[sp][c] - M) : 0.f;
            lp += fl[sp][c] * w;
            f[sp][c] = w;
        }
        red[q][c] = lp;
        __syncthreads();
        float L = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) L += red[k][c];
        inv = L > 0.f ? 1.f / L : 0.f;
    }
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < nsplit; s += PB) {
        if (s > 0) p_load(s);
#pragma unroll
        for (int k = 0; k < PB; ++k) {
            const float w = s + k < nsplit ? f[min(s + k, CHUNK_ATTN_MAX_SPLIT - 1)][j] : 0.f;
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = fmaf(p[k][u], w, v[u]);
        }
    }
    const int col = 32 * T.tile + j;
    if (col < G * T.n) {
        const int gq = col / T.n, r = col - gq * T.n;
        const int m = T.row0 + r, hq = kvh * G + gq;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int ch = blockIdx.y * 32 + dl + 8 * u;
            v[u] *= inv;
            bf16_t hi, lw;
            split_bf16(v[u], hi, lw);
            const size_t o = tiled_off(m, hq * DH + ch, g.Hq * DH);
            out_hi[o] = hi; out_lo[o] = lw;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------

static bool row_kernel_ok(const Geom& g, int S) { return g.d % 4 == 0 && g.d <= ROW_VEC_MAX * 1024 && S >= 1 && S <= CHUNK_GEMM_MAX_SPLIT; }

template <int PL>
static hipError_t resid_norm_t(const ChunkBuffers& c, int S, int MT, const float* gain, int rows, const Geom& g, hipStream_t s) {
    auto go = [&](auto k) { hipLaunchKernelGGL(k, dim3(rows), dim3(256), 0, s, c.x, c.part, S, (size_t)MT * 32 * g.d, g.d, gain, g.eps, g.d, c.nrm_hi, c.nrm_lo, c.nrm_lo2); };
    if (S == 1) go(k_chunk_resid_norm<1, PL>);
    else if (S == 2) go(k_chunk_resid_norm<2, PL>);
    else if (S <= 4) go(k_chunk_resid_norm<4, PL>);
    else go(k_chunk_resid_norm<CHUNK_GEMM_MAX_SPLIT, PL>);
    return hipGetLastError();
}

hipError_t launch_chunk_resid_norm(const ChunkBuffers& c, int S, int MT, const float* gain,
                                   int rows, const Geom& g, hipStream_t s, int planes) {
    if (!row_kernel_ok(g, S)) return hipErrorInvalidValue;
    return planes == 3 ? resid_norm_t<3>(c, S, MT, gain, rows, g, s) : resid_norm_t<2>(c, S, MT, gain, rows, g, s);
}

hipError_t launch_chunk_embed_norm(const void* E, const ChunkBuffers& c, const float* gain, int rows, const DecodeBuffers& b, const Geom& g,
                                   hipStream_t s, int planes) {
    if (!row_kernel_ok(g, 1)) return hipErrorInvalidValue;
    auto go = [&](auto k) { hipLaunchKernelGGL(k, dim3(rows), dim3(256), 0, s, (const bf16_t*)E, c.tab, rows, b.step, b.seq_state, c.chosen_host, c.x, gain,
                                               g.eps, g.d, c.nrm_hi, c.nrm_lo, c.nrm_lo2); };
    if (planes == 3) go(k_chunk_embed_norm<3>);
    else go(k_chunk_embed_norm<2>);
    return hipGetLastError();
}

hipError_t launch_chunk_last_row(const ChunkBuffers& c, int S, int MT, int group, const DecodeBuffers& b, const Geom& g,
                                 hipStream_t s) {
    hipLaunchKernelGGL(k_chunk_last_row, dim3((g.d + 255) / 256), dim3(256), 0, s, c.x, c.part, S, (size_t)MT * 32 * g.d,
                       g.d, g.d, c.tab, group, b.step, b.x);
    return hipGetLastError();
}

hipError_t launch_chunk_head_rows(const ChunkBuffers& c, int S, int MT, const float* gain, int ngroups, const Geom& g,
                                  hipStream_t s) {
    if (!row_kernel_ok(g, S)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_chunk_head_rows, dim3(ngroups), dim3(256), 0, s, c.x, c.part, S, (size_t)MT * 32 * g.d, g.d, gain,
                       g.eps, g.d, c.tab, c.nrm_hi, c.nrm_lo);
    return hipGetLastError();
}

hipError_t launch_chunk_logits(const ChunkBuffers& c, float* logits_base, const DecodeBuffers& b, int ngroups,
                               const Geom& g, hipStream_t s) {
    hipLaunchKernelGGL(k_chunk_logits, dim3(ngroups, CHUNK_LOGIT_SLICES), dim3(256), 0, s, c.part, g.V, c.tab, logits_base, b.seq_state, b.banned,
                       c.amax_v, c.amax_i, c.amax_counters);
    return hipGetLastError();
}

hipError_t launch_chunk_swiglu(const ChunkBuffers& c, int S, int MT, int rows, const Geom& g, hipStream_t s) {
    hipLaunchKernelGGL(k_chunk_swiglu, dim3((g.F + 255) / 256, rows), dim3(256), 0, s, c.part, S,
                       (size_t)MT * 32 * 2 * g.F, 2 * g.F, g.F, c.act_hi, c.act_lo);
    return hipGetLastError();
}

hipError_t launch_chunk_rope_kv(const ChunkBuffers& c, int S, void* kv_layer, const DecodeBuffers& b, int rows, int MT,
                                const Geom& g, hipStream_t s, bool kv_only) {
    const int h0 = kv_only ? g.Hq : 0, n_qkv = (g.Hq + 2 * g.Hkv - h0) * g.dh;
    const int nrot = (rows * (g.Hq + g.Hkv - h0) + ROPE_ITEMS - 1) / ROPE_ITEMS, vrows = rows > 256 ? 8 : 1, nval = (rows + vrows - 1) / vrows * ((g.Hkv + 1) / 2);
    // few rows: a workgroup per row, most of them with nothing to do, because the runs of several rows one after the other are a
    // chain (16 sequences, 40 rows: 18 us with eight rows per workgroup)
    if (g.dh != 128 || S < 1 || S > CHUNK_GEMM_MAX_SPLIT) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_chunk_rope_kv, dim3(nrot + nval), dim3(256), 0, s, c.part, S, (size_t)MT * 32 * n_qkv, n_qkv, g, c.tab, rows,
                       b.rope_cos, b.rope_sin, (bf16_t*)kv_layer, c.q_hi, c.q_lo, c.q_cols, h0, nrot, vrows);
    return hipGetLastError();
}

constexpr int ATTN_LDS_BYTES = 4 * 1024 * 16;       // k_chunk_attn: per wave one K tile, two planes

constexpr int gemm_lds_bytes(int planes) { return (2048 + 2 * planes * 512) * 16; }    // k_chunk_gemm: weight tiles, two buffers of activations
constexpr int GEMM_WIDE_LDS_BYTES = 2 * 2048 * 16;  // k_chunk_gemm_wide: two buffers of one 128 x 128 weight block
template <bool SWIGLU>
static const void* big_func(int nt) {
    switch (nt) {
        case 4: return (const void*)(k_chunk_gemm_big<4, SWIGLU>);
        case 5: return (const void*)(k_chunk_gemm_big<5, SWIGLU>);
        case 6: return (const void*)(k_chunk_gemm_big<6, SWIGLU>);
        case 7: return (const void*)(k_chunk_gemm_big<7, SWIGLU>);
        case 8: return (const void*)(k_chunk_gemm_big<8, SWIGLU>);
        default: return nullptr;
    }
}
static int big_lds_bytes(int nt) { return 3 * (nt * 2048 + BIG_M * 4096); }

hipError_t chunk_init() {
    hipError_t e;
    if ((e = hipFuncSetAttribute((const void*)(k_chunk_gemm<false, 2>), hipFuncAttributeMaxDynamicSharedMemorySize, gemm_lds_bytes(2)))) return e;
    if ((e = hipFuncSetAttribute((const void*)(k_chunk_gemm<true, 2>), hipFuncAttributeMaxDynamicSharedMemorySize, gemm_lds_bytes(2)))) return e;
    if ((e = hipFuncSetAttribute((const void*)k_chunk_attn, hipFuncAttributeMaxDynamicSharedMemorySize, ATTN_LDS_BYTES))) return e;
    if ((e = hipFuncSetAttribute((const void*)k_chunk_attn_wide, hipFuncAttributeMaxDynamicSharedMemorySize, ATTN_LDS_BYTES))) return e;
    if ((e = hipFuncSetAttribute((const void*)k_decode_attn_mfma, hipFuncAttributeMaxDynamicSharedMemorySize, ATTN_LDS_BYTES))) return e;
    if ((e = hipFuncSetAttribute((const void*)k_chunk_gemm_ks<2, false>, hipFuncAttributeMaxDynamicSharedMemorySize, GEMM_WIDE_LDS_BYTES))) return e;
    if ((e = hipFuncSetAttribute((const void*)k_chunk_gemm_ks<2, true>, hipFuncAttributeMaxDynamicSharedMemorySize, GEMM_WIDE_LDS_BYTES))) return e;
    if ((e = hipFuncSetAttribute((const void*)(k_chunk_gemm_wide<false, 2>), hipFuncAttributeMaxDynamicSharedMemorySize, GEMM_WIDE_LDS_BYTES))) return e;
    for (int nt = 4; nt <= 8; ++nt) {
        if ((e = hipFuncSetAttribute(big_func<false>(nt), hipFuncAttributeMaxDynamicSharedMemorySize, big_lds_bytes(nt)))) return e;
        if ((e = hipFuncSetAttribute(big_func<true>(nt), hipFuncAttributeMaxDynamicSharedMemorySize, big_lds_bytes(nt)))) return e;
    }
    if ((e = hipFuncSetAttribute((const void*)(k_chunk_gemm_wide<true, 2>), hipFuncAttributeMaxDynamicSharedMemorySize, GEMM_WIDE_LDS_BYTES))) return e;
    return hipSuccess;
}

hipError_t chunk_init_wide() {
    hipError_t e;
    if ((e = hipFuncSetAttribute((const void*)(k_chunk_gemm<false, 3>), hipFuncAttributeMaxDynamicSharedMemorySize, gemm_lds_bytes(3)))) return e;
    if ((e = hipFuncSetAttribute((const void*)(k_chunk_gemm<true, 3>), hipFuncAttributeMaxDynamicSharedMemorySize, gemm_lds_bytes(3)))) return e;
    if ((e = hipFuncSetAttribute((const void*)(k_chunk_gemm_wide<false, 3>), hipFuncAttributeMaxDynamicSharedMemorySize, GEMM_WIDE_LDS_BYTES))) return e;
    if ((e = hipFuncSetAttribute((const void*)(k_chunk_gemm_wide<true, 3>), hipFuncAttributeMaxDynamicSharedMemorySize, GEMM_WIDE_LDS_BYTES))) return e;
    return hipSuccess;
}

template <bool SWIGLU>
static hipError_t launch_big(const bf16_t* W, int N, int K, const bf16_t* xhi, const bf16_t* xlo, float* part, int S, int nt, int MT,
                             bf16_t* act_hi, bf16_t* act_lo, hipStream_t s) {
    const void* f = big_func<SWIGLU>(nt);
    if (!f || K % 128 || K / 128 < S) return hipErrorInvalidValue;
    const int per = nt * (SWIGLU ? 16 : 32), rows = SWIGLU ? N / 2 : N, MY = (MT + BIG_M - 1) / BIG_M;
    int ntiles = (rows + per - 1) / per, n_stride = N;
    size_t ps = (size_t)MT * 32 * N;
    void* params[] = {&W, &N, &K, &xhi, &xlo, &part, &ps, &n_stride, &S, &MT, &ntiles, &act_hi, &act_lo};
    return hipLaunchKernel(f, dim3((unsigned)ntiles * MY * S), dim3(256), params, big_lds_bytes(nt), s);
}

hipError_t launch_chunk_gemm(const void* W, int N, int K, const bf16_t* xhi, const bf16_t* xlo, const ChunkBuffers& c,
                             GemmPlan pl, int rows, hipStream_t s) {
    const int S = pl.s, MT = (rows + 31) / 32;
    const dim3 grid(N / 128, S), block(256);
    const size_t ps = (size_t)MT * 32 * N;
    if (S < 1 || S > CHUNK_GEMM_MAX_SPLIT || S > K / 128 || N % 128 || K % 128 || ps * S > c.part_capacity) return hipErrorInvalidValue;
    if (MT < 1 || MT > CHUNK_MAX / 32) return hipErrorInvalidValue;
    // one row tile: weight-streaming kernel, a wave per 32 weight rows; two: the waves split the k-steps; three or four:
    // a wave per row tile (128-row workgroups); more: 256-row workgroups with pl.nt weight-row tiles
    if (MT == 1) {
        hipLaunchKernelGGL((k_chunk_gemm<false, 2>), grid, block, gemm_lds_bytes(2), s, (const bf16_t*)W, N, K, xhi, xlo, nullptr, c.part, ps, N, S, rows, nullptr, nullptr, nullptr, 0);
    } else if (MT == 2) {
        hipLaunchKernelGGL((k_chunk_gemm_ks<2, false>), grid, block, GEMM_WIDE_LDS_BYTES, s, (const bf16_t*)W, N, K, xhi, xlo, c.part, ps, N, S, rows, nullptr, nullptr);
    } else if (MT <= 4) {
        hipLaunchKernelGGL((k_chunk_gemm_wide<false, 2>), dim3((unsigned)(N / 128) * S), block, GEMM_WIDE_LDS_BYTES, s, (const bf16_t*)W, N, K, xhi, xlo, nullptr, c.part, ps, N, S, rows, nullptr, nullptr, nullptr);
    } else return launch_big<false>((const bf16_t*)W, N, K, xhi, xlo, c.part, S, pl.nt, MT, nullptr, nullptr, s);
    return hipGetLastError();
}

// Gate/up product with the SwiGLU in its epilogue (no split-K): W = [gate rows | up rows] (2F x K), result in
// c.act_hi / c.act_lo.
hipError_t launch_chunk_gemm_swiglu(const void* W, int F, int K, const bf16_t* xhi, const bf16_t* xlo, const ChunkBuffers& c,
                                    GemmPlan pl, int rows, hipStream_t s) {
    const int MT = (rows + 31) / 32;
    if (MT < 1 || MT > CHUNK_MAX / 32 || F < 1 || K % 128 || (MT > 1 && F % 64)) return hipErrorInvalidValue;
    const bf16_t* Wb = (const bf16_t*)W;
    if (MT == 1) {
        const int rp = gate_rows_per_wave(F, 4 * std::max(1, decode_gemv_grid())), tiles = (F + rp - 1) / rp;
        hipLaunchKernelGGL((k_chunk_gemm<true, 2>), dim3((tiles + 3) / 4, 1), dim3(256), gemm_lds_bytes(2), s, Wb, 2 * F, K, xhi, xlo, nullptr, nullptr, (size_t)0, 0, 1, rows, c.act_hi, c.act_lo, nullptr, rp);
    } else if (MT == 2) {
        hipLaunchKernelGGL((k_chunk_gemm_ks<2, true>), dim3(F / 64, 1), dim3(256), GEMM_WIDE_LDS_BYTES, s, Wb, 2 * F, K, xhi, xlo, nullptr, (size_t)0, 0, 1, rows, c.act_hi, c.act_lo);
    } else if (MT <= 4) {
        hipLaunchKernelGGL((k_chunk_gemm_wide<true, 2>), dim3((unsigned)(F / 64)), dim3(256), GEMM_WIDE_LDS_BYTES, s, Wb, 2 * F, K, xhi, xlo, nullptr, nullptr, (size_t)0, 0, 1, rows, c.act_hi, c.act_lo, nullptr);
    } else return launch_big<true>(Wb, 2 * F, K, xhi, xlo, nullptr, 1, pl.nt, MT, c.act_hi, c.act_lo, s);
    return hipGetLastError();
}

// Inputs of three planes: one row tile k_chunk_gemm, more k_chunk_gemm_wide.
hipError_t launch_wide_gemm(const void* W, int N, int K, const bf16_t* xhi, const bf16_t* xlo, const bf16_t* xlo2, const ChunkBuffers& c, int S,
                            int rows, hipStream_t s) {
    const int MT = (rows + 31) / 32;
    const size_t ps = (size_t)MT * 32 * N;
    if (S < 1 || S > CHUNK_GEMM_MAX_SPLIT || S > K / 128 || N % 128 || K % 128 || ps * S > c.part_capacity || MT < 1 || MT > WIDE_ROWS_MAX / 32) return hipErrorInvalidValue;
    if (MT == 1)
        hipLaunchKernelGGL((k_chunk_gemm<false, 3>), dim3(N / 128, S), dim3(256), gemm_lds_bytes(3), s, (const bf16_t*)W, N, K, xhi, xlo, xlo2, c.part, ps, N, S, rows, nullptr, nullptr, nullptr, 0);
    else
        hipLaunchKernelGGL((k_chunk_gemm_wide<false, 3>), dim3((unsigned)(N / 128) * S * ((MT + 3) / 4)), dim3(256), GEMM_WIDE_LDS_BYTES, s, (const bf16_t*)W, N, K, xhi, xlo, xlo2,
                           c.part, ps, N, S, rows, nullptr, nullptr, nullptr);
    return hipGetLastError();
}

hipError_t launch_wide_gemm_swiglu(const void* W, int F, int K, const bf16_t* xhi, const bf16_t* xlo, const bf16_t* xlo2, const ChunkBuffers& c,
                                   int rows, hipStream_t s) {
    const int MT = (rows + 31) / 32;
    if (F < 1 || F % 64 || K % 128 || MT < 1 || MT > WIDE_ROWS_MAX / 32) return hipErrorInvalidValue;
    if (MT == 1) {
        const int rp = gate_rows_per_wave(F, 4 * std::max(1, decode_gemv_grid())), tiles = (F + rp - 1) / rp;
        hipLaunchKernelGGL((k_chunk_gemm<true, 3>), dim3((tiles + 3) / 4, 1), dim3(256), gemm_lds_bytes(3), s, (const bf16_t*)W, 2 * F, K, xhi, xlo, xlo2, nullptr, (size_t)0, 0, 1, rows,
                           c.act_hi, c.act_lo, c.act_lo2, rp);
    } else
        hipLaunchKernelGGL((k_chunk_gemm_wide<true, 3>), dim3((unsigned)(F / 64) * ((MT + 3) / 4)), dim3(256), GEMM_WIDE_LDS_BYTES, s, (const bf16_t*)W, 2 * F, K, xhi, xlo, xlo2,
                           nullptr, (size_t)0, 0, 1, rows, c.act_hi, c.act_lo, c.act_lo2);
    return hipGetLastError();
}

hipError_t launch_chunk_attn(const ChunkBuffers& c, const void* kv_layer, int nsplit, int ntasks, const Geom& g, hipStream_t s) {
    if (nsplit < 4 || nsplit % 4 || nsplit > CHUNK_ATTN_MAX_SPLIT || ntasks < 1 || ntasks > CHUNK_MAX_TASKS ||
        (long long)ntasks * g.Hkv * nsplit > CHUNK_ATTN_MAX_UNITS)
        return hipErrorInvalidValue;
    ChunkAttnArgs a{};
    a.q_hi = c.q_hi; a.q_lo = c.q_lo; a.kv_layer = (const bf16_t*)kv_layer; a.tab = c.tab;
    a.part_o = c.attn_o; a.part_ml = c.attn_ml; a.nsplit = nsplit; a.q_cols = c.q_cols;
    // one wave per workgroup (the kernel takes any number up to four): the waves of a small pass then spread over more
    // compute units instead of sharing one unit's memory pipeline (24-row inject 4.19 -> 4.11 ms; no change for the
    // 16-sequence batched step)
    hipLaunchKernelGGL(k_chunk_attn, dim3(ntasks * g.Hkv, nsplit), dim3(64), ATTN_LDS_BYTES / 4, s, a, g);
    hipError_t e = hipGetLastError();
    if (e) return e;
    hipLaunchKernelGGL(k_chunk_attn_combine, dim3(ntasks * g.Hkv, 4), dim3(256), 0, s, c.attn_o, c.attn_ml, g, c.tab,
                       c.att_hi, c.att_lo);
    return hipGetLastError();
}

// The variant for passes made of large groups: one workgroup per kv head, block of up to four tasks and key split of it.
hipError_t launch_chunk_attn_wide(const ChunkBuffers& c, const void* kv_layer, bool merge, int ntasks, int npieces, const Geom& g, hipStream_t s) {
    if (ntasks < 1 || ntasks > CHUNK_MAX_TASKS || npieces < 1 || npieces > CHUNK_ATTN_MAX_UNITS) return hipErrorInvalidValue;
    ChunkAttnArgs a{};
    a.q_hi = c.q_hi; a.q_lo = c.q_lo; a.kv_layer = (const bf16_t*)kv_layer; a.tab = c.tab;
    a.part_o = c.attn_o; a.part_ml = c.attn_ml; a.q_cols = c.q_cols;
    a.out_hi = c.att_hi; a.out_lo = c.att_lo;
    hipLaunchKernelGGL(k_chunk_attn_wide, dim3(npieces * g.Hkv), dim3(256), ATTN_LDS_BYTES, s, a, g);
    hipError_t e = hipGetLastError();
    if (e || !merge) return e;
    hipLaunchKernelGGL(k_chunk_attn_combine, dim3(ntasks * g.Hkv, 4), dim3(256), 0, s, c.attn_o, c.attn_ml, g, c.tab,
                       c.att_hi, c.att_lo);
    return hipGetLastError();
}

hipError_t launch_decode_attn_mfma(const ChunkBuffers& c, const void* kv_layer, int nsplit, const DecodeBuffers& b, const Geom& g,
                                   hipStream_t s, unsigned long long* stamps, unsigned long long* done_wg) {
    const int G = g.Hq / g.Hkv;
    if (g.dh != 128 || G > 8 || nsplit < 4 || nsplit % 4 || nsplit > CHUNK_ATTN_MAX_SPLIT ||
        (long long)g.Hkv * nsplit > CHUNK_ATTN_MAX_UNITS)
        return hipErrorInvalidValue;
    DecodeAttnArgs a{};
    a.q = b.q; a.step = b.step; a.kv_layer = (const bf16_t*)kv_layer;
    a.part_o = c.attn_o; a.part_ml = c.attn_ml; a.out = b.o; a.nsplit = nsplit; a.stamps = stamps; a.done_wg = done_wg;
    // one wave per workgroup (the kernel takes any number up to four): the waves that have keys (35 of the 96 splits of a
    // kv head at a context of 1.1k) then spread over as many compute units instead of sharing one unit's memory pipeline
    // four at a time (8B decode 3.31 -> 3.26 ms per token; two per workgroup the same at 1.1k, 2 % slower at 16k)
    hipLaunchKernelGGL(k_decode_attn_mfma, dim3(g.Hkv, nsplit), dim3(64), ATTN_LDS_BYTES / 4, s, a, g);
    hipError_t e = hipGetLastError();
    if (e) return e;
    hipLaunchKernelGGL(k_decode_attn_merge, dim3(g.Hkv, 2 * G), dim3(256), 0, s, a, g);
    return hipGetLastError();
}

}  // namespace asynclm
