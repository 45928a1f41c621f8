// Epilogues shared by the GEMV (k_gemv.hip) and MFMA (k_mfma.hip) paths of
// the routed projections: weight-row pairing of the two-row kinds and what is
// done with a finished sum (residual add, bias + activation, SwiGLU, rotary
// embedding with KV append).
#pragma once

#include "buddy_internal.h"

namespace buddy {

template <int EPI>
__device__ __forceinline__ void unit_rows(const GemvArgs& g, int u, int& r0, int& r1) {
    if (EPI == EPI_SWIGLU) { r0 = u; r1 = g.f + u; }
    else if (EPI == EPI_QKV) {
        const int half = g.hd >> 1;
        const int hg = u / half, i = u - hg * half;
        r0 = hg * g.hd + i; r1 = r0 + half;
    } else { r0 = 2 * u; r1 = 2 * u + 1; }
}

__device__ __forceinline__ float act_fn(float x, int act) {
    if (act == BUDDY_ACT_GELU_ERF) return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f));
    return x / (1.0f + expf(-x));
}

// SwiGLU of a gate sum v0 and an up sum v1: SiLU(v0) v1.
__device__ __forceinline__ float swiglu(float v0, float v1) { return v0 / (1.0f + expf(-v0)) * v1; }

// Epilogue of one finished row for the single-row kinds.
template <typename TW, int EPI>
__device__ __forceinline__ void epilogue1(const GemvArgs& g, int b, int row, float v) {
    float* y = g.Y + (size_t)b * g.ldy;
    if (EPI == EPI_ADD) y[row] += v;
    else y[row] = act_fn(v + St<TW>::get((const TW*)g.bias, row), g.act);
}

template <typename TW, int EPI>
__device__ __forceinline__ void epilogue(const GemvArgs& g, int b, int u, int r0, int r1,
                                         float v0, float v1) {
    if (EPI == EPI_ADD) {
        float* y = g.Y + (size_t)b * g.ldy;
        y[r0] += v0;
        y[r1] += v1;
    } else if (EPI == EPI_BIAS_ACT) {
        float* y = g.Y + (size_t)b * g.ldy;
        const TW* bias = (const TW*)g.bias;
        y[r0] = act_fn(v0 + St<TW>::get(bias, r0), g.act);
        y[r1] = act_fn(v1 + St<TW>::get(bias, r1), g.act);
    } else if (EPI == EPI_SWIGLU) {
        g.Y[(size_t)b * g.ldy + u] = swiglu(v0, v1);
    } else {  // EPI_QKV
        const int half = g.hd >> 1;
        const int hg = u / half, i = u - hg * half;
        int slot, pos;
        slot_pos(b, g.tok_T, g.pos, g.pos_u, slot, pos);
        if (hg < g.nq + g.nkv) {
            const float2 cs = g.rope[(size_t)pos * half + i];
            const float a0 = v0 * cs.x - v1 * cs.y;
            const float a1 = v1 * cs.x + v0 * cs.y;
            v0 = a0; v1 = a1;
        }
        if (hg < g.nq) {
            float* y = g.Y + (size_t)b * g.ldy + (size_t)hg * g.hd;
            y[i] = v0;
            y[i + half] = v1;
        } else {
            const bool is_k = hg < g.nq + g.nkv;
            const int kvh = is_k ? hg - g.nq : hg - g.nq - g.nkv;
            TW* dst = (TW*)(is_k ? g.kc : g.vc) +
                      (((size_t)slot * g.nkv + kvh) * g.T + pos) * g.hd;
            St<TW>::put(dst, i, v0);
            St<TW>::put(dst, i + half, v1);
        }
    }
}

// Four units or rows u .. u + 3 (u % 4 == 0) of row b at once, for the tiled
// GEMM: 16-byte loads and stores of fp32, 8-byte stores of bf16.  The values
// their arithmetic are those of the epilogues above.  (One element at a
// time, the QKV projection of a 2048-token prompt took 170 us, Llama-8B
// shape; four at a time 146, and 125 on the 256 x 256 tiles, which the
// scattered 4-byte stores had made slower: 189.)
template <int EPI>
__device__ __forceinline__ void epilogue4(const GemvArgs& g, int b, int u, const float* v0, const float* v1) {
    static_assert(EPI == EPI_ADD || EPI == EPI_SWIGLU || EPI == EPI_QKV, "kinds of the tiled GEMM");
    if (EPI == EPI_ADD) {
        float4* y = reinterpret_cast<float4*>(g.Y + (size_t)b * g.ldy + u);
        float4 t = *y;
        t.x += v0[0]; t.y += v0[1]; t.z += v0[2]; t.w += v0[3];
        *y = t;
    } else if (EPI == EPI_SWIGLU) {
        *reinterpret_cast<float4*>(g.Y + (size_t)b * g.ldy + u) =
            make_float4(swiglu(v0[0], v1[0]), swiglu(v0[1], v1[1]), swiglu(v0[2], v1[2]), swiglu(v0[3], v1[3]));
    } else {
        const int half = g.hd >> 1;   // a multiple of 4: the four units are of one head
        const int hg = u / half, i = u - hg * half;
        int slot, pos;
        slot_pos(b, g.tok_T, g.pos, g.pos_u, slot, pos);
        float a0[4], a1[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) { a0[e] = v0[e]; a1[e] = v1[e]; }
        if (hg < g.nq + g.nkv) {
            const float4* rp = reinterpret_cast<const float4*>(g.rope + (size_t)pos * half + i);
            const float4 r0 = rp[0], r1 = rp[1];
            const float c[4] = {r0.x, r0.z, r1.x, r1.z}, s[4] = {r0.y, r0.w, r1.y, r1.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a0[e] = v0[e] * c[e] - v1[e] * s[e];
                a1[e] = v1[e] * c[e] + v0[e] * s[e];
            }
        }
        if (hg < g.nq) {
            float* y = g.Y + (size_t)b * g.ldy + (size_t)hg * g.hd + i;
            *reinterpret_cast<float4*>(y) = make_float4(a0[0], a0[1], a0[2], a0[3]);
            *reinterpret_cast<float4*>(y + half) = make_float4(a1[0], a1[1], a1[2], a1[3]);
        } else {
            const bool is_k = hg < g.nq + g.nkv;
            const int kvh = is_k ? hg - g.nq : hg - g.nq - g.nkv;
            bf16_t* dst = (bf16_t*)(is_k ? g.kc : g.vc) +
                          (((size_t)slot * g.nkv + kvh) * g.T + pos) * g.hd + i;
            *reinterpret_cast<uint2*>(dst) = make_uint2(f2bf(a0[0]) | (uint32_t)f2bf(a0[1]) << 16,
                                                        f2bf(a0[2]) | (uint32_t)f2bf(a0[3]) << 16);
            *reinterpret_cast<uint2*>(dst + half) = make_uint2(f2bf(a1[0]) | (uint32_t)f2bf(a1[1]) << 16,
                                                               f2bf(a1[2]) | (uint32_t)f2bf(a1[3]) << 16);
        }
    }
}

}  // namespace buddy
