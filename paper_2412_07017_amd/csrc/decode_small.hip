// Decoding step of models so small that a step is a chain of launches and memory round trips (the tiny preset: 7.4 MB of weights):
// three launches per layer instead of five, and none for the start of the step.  What allows it is that a product may leave partial
// vectors behind which the next kernel adds while it reads its input, in a fixed order:
//   k_gemv_small<.., QKV> (decode_kernels.hip)  x + the partial vectors of the layer before (first layer: the token's embedding, and the
//                                      step's bookkeeping) -> norm, q, k, v; one workgroup leaves the sum as the new x
//   k_small_attn_o                     one workgroup per kv head: its attention, then the columns of the O projection that belong to its
//                                      query heads, from registers that were filled while the attention ran -> a partial vector per kv head
//   k_small_mlp                        one workgroup per 16 features: gate and up rows, then the same columns of the down projection
//                                      -> a partial vector per workgroup
//   k_gemv_small<.., STORE>            output head, the same sum first
// Tiny preset, context 100: 5.0 us for attention and O projection (two kernels and a boundary: 4.0 + 3.6), 4.0 for the MLP (2.6 + 2.8), 4.2 for a
// QKV product that adds 47 partial vectors (2.7), 6.8 for the head (5.2), 3.1 for the first kernel (2.9 + 2.7); a step 47.5 -> 41 us as a
// graph, 38 with its seven launches issued one by one, 32 without an event behind the first of them.  16 or 32 features per workgroup make no difference.
#include "common.h"
#include "launch.h"
#include "decode_device.h"

namespace asynclm {

constexpr int MLP_F = 16;               // features per workgroup of k_small_mlp
constexpr int O_BATCH = 16;             // 16-byte loads of the O projection per thread in flight

struct SmallArgs {
    const float* q; const void* kv_layer; const StepDesc* step;
    const void* w;                      // O projection [d][Hq * dh]; gate and up rows [2 F][d]
    const void* wdown;                  // [d][F]
    const float* x; const float* gain;
    const float* parts_in;              // partial vectors of the O projection [Hkv][d]
    float* parts_out;                   // [Hkv][d], [F / MLP_F][d]
    SeqState* grow;                     // the attention of the first layer: sequences, of which the step's one is a token longer now; else null
};

template <int N>
__device__ __forceinline__ float lanes_sum(float v) {
    if constexpr (N == 64) return wave_sum_all(v);
    else return group_sum<N>(v);
}

// Bound by latency: query, keys and values, and the 16 loads per thread of the O projection are all requested in the first microsecond;
// then scores, softmax, P V and the projection follow from registers and LDS.
template <typename WT, int DH, int G, bool PAIR>
__global__ __launch_bounds__(256) void k_small_attn_o(SmallArgs a, Geom g) {
    constexpr int EPL = Elem<WT>::EPL, COLS = G * DH;
    constexpr int LPS = COLS / EPL;                         // lanes that cover this kv head's columns of a row
    constexpr int RPP = 256 / LPS;                          // rows per round of the workgroup
    static_assert(LPS >= 8 && LPS <= 64, "a row's columns lie within a wave");
    extern __shared__ float lds[];
    const int tid = threadIdx.x, kvh = blockIdx.x, sub = tid / LPS, c = tid % LPS, len = a.step->pos + 1;
    const WT* wo = (const WT*)a.w + (size_t)kvh * COLS + c * EPL;
    const size_t stride = (size_t)g.Hq * DH;
    uint4 w[O_BATCH];
    auto load = [&](int r0) {
#pragma unroll
        for (int j = 0; j < O_BATCH; ++j) w[j] = load16(wo + (size_t)min(r0 + j * RPP + sub, g.d - 1) * stride);
    };
    load(0);
    __builtin_amdgcn_sched_barrier(0);
    if (a.grow && kvh == 0 && tid == 0) a.grow[a.step->seq].len = len;
    const WT* Kp = (const WT*)a.kv_layer + (size_t)a.step->seq * g.kv_seq_stride + (size_t)kvh * g.kv_head_stride;
    float mh[G], lh[G];
    attn_split<WT, DH, G, PAIR, 8>(a.q, Kp, Kp + g.kv_v_offset, g.kv_lo_offset, kvh, 0, len, g.scale, lds, mh, lh);
    for (int t = tid; t < COLS; t += 256) {                 // the scores have been read: their place takes the output
        const int h = t / DH, dim = t - h * DH;
        float L = lh[0];
#pragma unroll
        for (int hh = 1; hh < G; ++hh) if (hh == h) L = lh[hh];
        lds[t] = attn_gather<WT, DH, G>(lds, h, dim) / L;
    }
    __syncthreads();
    float o[EPL];
#pragma unroll
    for (int e = 0; e < EPL; e += 4) {
        const float4 v = *reinterpret_cast<const float4*>(lds + c * EPL + e);
        o[e] = v.x; o[e + 1] = v.y; o[e + 2] = v.z; o[e + 3] = v.w;
    }
    float* out = a.parts_out + (size_t)kvh * g.d;
    for (int r0 = 0; r0 < g.d; r0 += O_BATCH * RPP) {
        if (r0) load(r0);
#pragma unroll
        for (int j = 0; j < O_BATCH; ++j) {
            float f[EPL], s = 0.f;
            Elem<WT>::expand(w[j], f);
#pragma unroll
            for (int e = 0; e < EPL; ++e) s = fmaf(f[e], o[e], s);
            s = lanes_sum<LPS>(s);
            const int r = r0 + j * RPP + sub;
            if (c == 0 && r < g.d) out[r] = s;
        }
    }
}

// NS: wave-wide loads per row of d columns (1 or 2).  Every wave forms the whole input vector for itself, as in k_gemv_small.
// Everything that does not depend on the vector (gate, up and down rows) is requested first.
template <typename WT, int NS>
__global__ __launch_bounds__(256) void k_small_mlp(SmallArgs a, Geom g) {
    constexpr int EPL = Elem<WT>::EPL, NP = EPL / 4, FW = MLP_F / 4;       // features per wave
    constexpr int LPS = MLP_F / EPL, RPP = 256 / LPS, ND = 4 * NS;         // down rows: lanes per row, rows per round, rounds in flight
    __shared__ float act[MLP_F];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Kg = g.d / EPL, f0 = blockIdx.x * MLP_F;
    uint4 w[2 * FW][NS], wd[ND];
    float4 xv[NS][NP], gn[NS][NP];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const size_t k = (size_t)min(s * 64 + lane, Kg - 1) * EPL + 4 * q;
            xv[s][q] = as_float4(load16(a.x + k)); gn[s][q] = as_float4(load16(a.gain + k));
        }
#pragma unroll
    for (int j = 0; j < 2 * FW; ++j) {
        const int f = min(f0 + wave * FW + (j >> 1), g.F - 1);
        const WT* row = (const WT*)a.w + (size_t)((j & 1) ? g.F + f : f) * g.d;
#pragma unroll
        for (int s = 0; s < NS; ++s) w[j][s] = load16(row + (size_t)min(s * 64 + lane, Kg - 1) * EPL);
    }
    const int sub = tid / LPS, c = tid % LPS;
    const int fc = min(f0 + c * EPL, g.F - EPL);            // past the last feature (F is a multiple of 8): any columns, times zero
    const WT* wdn = (const WT*)a.wdown + fc;
    auto load_down = [&](int r0) {
#pragma unroll
        for (int j = 0; j < ND; ++j) wd[j] = load16(wdn + (size_t)min(r0 + j * RPP + sub, g.d - 1) * g.F);
    };
    load_down(0);
    float4 sum[NS][NP];                                     // the kv heads' shares of the O projection, then the residual
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int q = 0; q < NP; ++q) sum[s][q] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int p0 = 0; p0 < g.Hkv; p0 += 4) {
        float4 t[4][NS][NP];
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int q = 0; q < NP; ++q)
                    t[p][s][q] = as_float4(load16(a.parts_in + (size_t)min(p0 + p, g.Hkv - 1) * g.d + (size_t)min(s * 64 + lane, Kg - 1) * EPL + 4 * q));
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                float4 u[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) u[p] = p0 + p < g.Hkv ? t[p][s][q] : make_float4(0.f, 0.f, 0.f, 0.f);
                float4& v = sum[s][q];
                v.x += (u[0].x + u[1].x) + (u[2].x + u[3].x); v.y += (u[0].y + u[1].y) + (u[2].y + u[3].y);
                v.z += (u[0].z + u[1].z) + (u[2].z + u[3].z); v.w += (u[0].w + u[1].w) + (u[2].w + u[3].w);
            }
    }
    float ss = 0.f, acc[2 * FW];
#pragma unroll
    for (int j = 0; j < 2 * FW; ++j) acc[j] = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const bool live = s * 64 + lane < Kg;
        float x[EPL];
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const float4 b = xv[s][q], u = sum[s][q], v = live ? make_float4(b.x + u.x, b.y + u.y, b.z + u.z, b.w + u.w) : make_float4(0.f, 0.f, 0.f, 0.f);
            ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
            x[4 * q] = v.x * gn[s][q].x; x[4 * q + 1] = v.y * gn[s][q].y; x[4 * q + 2] = v.z * gn[s][q].z; x[4 * q + 3] = v.w * gn[s][q].w;
        }
#pragma unroll
        for (int j = 0; j < 2 * FW; ++j) {
            float f[EPL];
            Elem<WT>::expand(w[j][s], f);
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[j] = fmaf(f[e], x[e], acc[j]);
        }
    }
    const float sc = rsqrtf(wave_sum_all(ss) / (float)g.d + g.eps);
#pragma unroll
    for (int j = 0; j < FW; ++j) {
        const float gt = wave_sum_all(acc[2 * j]) * sc, up = wave_sum_all(acc[2 * j + 1]) * sc;
        if (lane == 0) act[wave * FW + j] = f0 + wave * FW + j < g.F ? gt / (1.f + expf(-gt)) * up : 0.f;
    }
    __syncthreads();
    float av[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) av[e] = f0 + c * EPL < g.F ? act[c * EPL + e] : 0.f;
    float* out = a.parts_out + (size_t)blockIdx.x * g.d;
    for (int r0 = 0; r0 < g.d; r0 += ND * RPP) {
        if (r0) load_down(r0);
#pragma unroll
        for (int j = 0; j < ND; ++j) {
            float f[EPL], s = 0.f;
            Elem<WT>::expand(wd[j], f);
#pragma unroll
            for (int e = 0; e < EPL; ++e) s = fmaf(f[e], av[e], s);
            s += dpp_move<0xB1>(s);                         // the two or four lanes of a row
            if (LPS == 4) s += dpp_move<0x4E>(s);
            const int r = r0 + j * RPP + sub;
            if (c == 0 && r < g.d) out[r] = s;
        }
    }
}

// ---- launchers ------------------------------------------------------------------------------------------------------

template <typename WT>
static bool small_step_t(const Geom& g) {
    const int cols = g.Hq / g.Hkv * g.dh, lps = cols / Elem<WT>::EPL;
    return lps >= 8 && lps <= 64 && g.d <= SMALL_MAX_D && (size_t)g.d * cols * sizeof(WT) <= SMALL_O_BYTES && g.Hkv <= SMALL_MAX_KV_HEADS && g.d % 8 == 0 && g.F % 8 == 0 && g.F >= 8;
}

bool small_step_supported(int dtype, const Geom& g) {
    return gemv_all_small(dtype, g) && g.kv_v_offset && (dtype == 0 ? small_step_t<float>(g) : small_step_t<bf16_t>(g));
}

// The short step saves the launch that starts a step, two per layer and, launch by launch, the start of a graph; but one workgroup per
// kv head walks all keys and reads all its columns of the O projection, and every workgroup of the next product reads all partial vectors,
// where the other kernels split these.  Difference of the two in us, fitted to 372 random shapes of 1 to 16 layers at six contexts from 10 to 350
// (rms 4 % of a step) and shifted by 1 + 0.6 per layer to the other kernels' side.  On 363 other shapes (2178 points) the choice is more than 3 %
// slower than the other kernels at 3 points (4 % at most), and 0.5 % slower than the better of the two on average (10 % at most).  Short step / the other kernels, us per step: tiny preset's
// shape 32 / 44 (350 keys 38 / 44), with 5 layers 75 / 88 at 110 keys and 81 / 87 at 200; bf16 d 256, 5 layers 89 / 102; but bf16 d 512 with 1024 features,
// 5 layers 105 / 103, two heads per kv head 125 / 108 (144 / 107 at 350 keys), d 1024 163 / 109, eight heads per kv head 153 / 143 (201 / 143 at 275).
bool small_step_pays(int dtype, const Geom& g, int n_layers, int keys) {
    const int es = dtype == 0 ? 4 : 2, G = g.Hq / g.Hkv, w = 4 / es * G;                          // w: bf16 has twice the channels per lane
    const int o_batches = (int)(((size_t)g.d * G * g.dh * es + 65535) / 65536);                    // of the O projection's loads (O_BATCH)
    const int key_batches = (keys - 1) / (2048 * (16 / es) / g.dh), chunks = (keys - 1) / 256;      // beyond the first (attn_split)
    const double part_bytes = (double)(g.Hkv + small_mlp_parts(g)) * g.d * sizeof(float), cache = dtype == 0 ? 0. : g.kv_lo_offset ? 0.9 : -0.4;
    const double layer = 2.4 * (o_batches - 1) + 0.6 * part_bytes / 65536 + 1.4 * key_batches + 0.48 * chunks * w + 0.5 * w + cache - 0.34 * (g.Hq - g.Hkv) - 2.2;
    return keys <= SMALL_MAX_KEYS && layer * n_layers < (n_layers <= SMALL_DIRECT_LAYERS ? 8.2 : 4.0);
}

int small_mlp_parts(const Geom& g) { return (g.F + MLP_F - 1) / MLP_F; }

template <typename WT, int DH, bool PAIR>
static hipError_t launch_attn_o_t(const SmallArgs& a, const Geom& g, hipStream_t s) {
    auto go = [&](auto k, int lds_floats) -> hipError_t {
        const int lds = lds_floats * (int)sizeof(float);
        if (lds > 48 * 1024)
            if (hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, lds)) return e;
        hipLaunchKernelGGL(k, dim3(g.Hkv), dim3(256), lds, s, a, g);
        return hipGetLastError();
    };
    constexpr int EPL = Elem<WT>::EPL;
    switch (g.Hq / g.Hkv) {
        case 1: return go(k_small_attn_o<WT, DH, 1, PAIR>, attn_lds_floats<WT, DH, 1>());
        case 2: return go(k_small_attn_o<WT, DH, 2, PAIR>, attn_lds_floats<WT, DH, 2>());
        case 4: if constexpr (4 * DH / EPL <= 64) return go(k_small_attn_o<WT, DH, 4, PAIR>, attn_lds_floats<WT, DH, 4>()); else return hipErrorInvalidValue;
        case 8: if constexpr (8 * DH / EPL <= 64) return go(k_small_attn_o<WT, DH, 8, PAIR>, attn_lds_floats<WT, DH, 8>()); else return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_small_attn_o(int dtype, const void* kv_layer, const void* wo, const SmallBuffers& sb, const DecodeBuffers& b, const Geom& g, bool first_layer, hipStream_t s) {
    SmallArgs a{};
    if (first_layer) a.grow = b.seq_state;
    a.q = b.q; a.kv_layer = kv_layer; a.step = b.step; a.w = wo; a.parts_out = sb.parts;
    if (dtype == 0) return g.dh == 64 ? launch_attn_o_t<float, 64, false>(a, g, s) : launch_attn_o_t<float, 128, false>(a, g, s);
    if (g.kv_lo_offset) return g.dh == 64 ? launch_attn_o_t<bf16_t, 64, true>(a, g, s) : launch_attn_o_t<bf16_t, 128, true>(a, g, s);
    return g.dh == 64 ? launch_attn_o_t<bf16_t, 64, false>(a, g, s) : launch_attn_o_t<bf16_t, 128, false>(a, g, s);
}

template <typename WT>
static hipError_t launch_mlp_t(const SmallArgs& a, const Geom& g, hipStream_t s) {
    const int ns = (g.d / Elem<WT>::EPL + 63) / 64;
    auto go = [&](auto k) { hipLaunchKernelGGL(k, dim3(small_mlp_parts(g)), dim3(256), 0, s, a, g); return hipGetLastError(); };
    if constexpr (SMALL_MAX_D > 64 * Elem<WT>::EPL)
        if (ns == 2) return go(k_small_mlp<WT, 2>);
    return ns <= 1 ? go(k_small_mlp<WT, 1>) : hipErrorInvalidValue;
}

hipError_t launch_small_mlp(int dtype, const void* wgu, const void* wdown, const float* gain, const float* x, const SmallBuffers& sb, const Geom& g, hipStream_t s) {
    SmallArgs a{};
    a.w = wgu; a.wdown = wdown; a.x = x; a.gain = gain; a.parts_in = sb.parts; a.parts_out = sb.parts + (size_t)g.Hkv * g.d;
    return dtype == 0 ? launch_mlp_t<float>(a, g, s) : launch_mlp_t<bf16_t>(a, g, s);
}

}  // namespace asynclm
