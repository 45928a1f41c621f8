// First layer of the Decision Module (and of the Budget Predictor) over a
// batch (gfx950, bf16 weights): the sums W z_b of act(W z_b + bias), with the
// router context z_b = [pooled K / V means | newest hidden state] in fp32.
//
// The routes are decided on these scores, so the context keeps its 24 bits:
// each value enters v_mfma_f32_16x16x32_bf16 as three bf16 parts (the
// rounding of the value, then of the remainders), whose products with the
// bf16 weights accumulate in fp32.  No staging: a lane's eight context values
// of a k-step are its B operand, split in registers.
//
// A workgroup of four wavefronts owns 128 hidden units, 16 sequences and a
// slice of K; wavefront w takes every fourth k-step of the slice, its sums
// meet the others' in LDS, and the workgroup writes them to part[slice][b][unit],
// which the router kernel adds in slice order before bias and activation.
// What bounds this layer is not its few MB but the bytes one CU can fetch
// (about 50 GB/s), so the launch is cut into about 256 workgroups: K slices
// until the grid has them (a workgroup per 16 units over all of K read the
// whole context, pool splits included, 32 times over from 64 CUs: 35.6 us at
// B = 24 on the Llama-8B shape; the GEMV, which passes the weights by each
// sequence in turn, 44.6), and 128 units per workgroup so that four of them,
// not 32, fold a slice's pool splits: 8.3 us at B = 24, 24 at B = 96 (13B MHA
// shape; GEMV 189).
#include <type_traits>

#include "buddy_internal.h"
#include "epilogue.h"

namespace buddy {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kDmWaves = 4;
constexpr int kDmTiles = kDmUnits / 16;   // 16-unit weight tiles of a workgroup

// Eight fp32 context values as three packed bf16 parts against every weight
// tile: acc += a p0, low += a (p1 + p2).  The remainders are exact; where a
// value (or its rounding) is not finite it decides alone, which one test of
// all eight remainders finds.
__device__ __forceinline__ void dm_step(const bf16x8_t* a, const float4& v0, const float4& v1, f32x4_t* acc,
                                        f32x4_t* low) {
    const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
    uint32_t p0[4], p1[4], p2[4];
    float r[8], t = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        p0[e] = pack_bf16x2(v[2 * e], v[2 * e + 1]);
        r[2 * e] = v[2 * e] - __uint_as_float(p0[e] << 16);
        r[2 * e + 1] = v[2 * e + 1] - __uint_as_float(p0[e] & 0xffff0000u);
        t += r[2 * e] + r[2 * e + 1];
    }
    if (!((t - t) == 0.f)) {
#pragma unroll
        for (int e = 0; e < 8; ++e) r[e] = (r[e] - r[e]) == 0.f ? r[e] : 0.f;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        p1[e] = pack_bf16x2(r[2 * e], r[2 * e + 1]);
        p2[e] = pack_bf16x2(r[2 * e] - __uint_as_float(p1[e] << 16),
                            r[2 * e + 1] - __uint_as_float(p1[e] & 0xffff0000u));
    }
    const bf16x8_t b0 = __builtin_bit_cast(bf16x8_t, make_uint4(p0[0], p0[1], p0[2], p0[3]));
    const bf16x8_t b1 = __builtin_bit_cast(bf16x8_t, make_uint4(p1[0], p1[1], p1[2], p1[3]));
    const bf16x8_t b2 = __builtin_bit_cast(bf16x8_t, make_uint4(p2[0], p2[1], p2[2], p2[3]));
#pragma unroll
    for (int x = 0; x < kDmTiles; ++x) {
        acc[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[x], b0, acc[x], 0, 0, 0);
        low[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[x], b1, low[x], 0, 0, 0);
        low[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[x], b2, low[x], 0, 0, 0);
    }
}

__device__ __forceinline__ void add4(float4& v, const float4& t) { v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w; }

template <bool BOTH>   // the K + V context: both feature rows of a split
__global__ __launch_bounds__(64 * kDmWaves) void dm_kernel(GemvArgs g, int B, int slice_steps, float* part) {
    constexpr int kNW = BOTH ? 2 : 1;
    __shared__ float s_red[kDmWaves][16][kDmUnits + 1];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, q = lane >> 4;
    const int h0 = blockIdx.y * kDmUnits, b0 = blockIdx.z * 16;
    // units and sequences past the end repeat the last one; not written
    const int b = min(b0 + i, B - 1);
    const int K = g.K, zsteps = pooled_dim(g.ctx, g.nkv, g.hd) / 32;
    const int first = blockIdx.x * slice_steps, end = min(first + slice_steps, K / 32);
    const bf16_t* w[kDmTiles];
#pragma unroll
    for (int x = 0; x < kDmTiles; ++x)
        w[x] = (const bf16_t*)g.W + (size_t)min(h0 + 16 * x + i, g.N - 1) * K + 8 * q;
    const float* h = g.h + (size_t)b * g.d + 8 * q;
    const float inv_n = 1.0f / (float)(seq_pos(g.pos, g.pos_u, b) + 1);
    const int hsteps = g.hd / 32, hshift = g.hd == 128 ? 2 : 1;   // hd is 64 or 128
    const size_t row = 2 * (size_t)g.hd;   // floats of a split: K sums, V sums
    f32x4_t acc[kDmTiles], low[kDmTiles];
#pragma unroll
    for (int x = 0; x < kDmTiles; ++x) acc[x] = low[x] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

    for (int s = first + wave; s < end; s += kDmWaves) {
        bf16x8_t a[kDmTiles];
#pragma unroll
        for (int x = 0; x < kDmTiles; ++x) a[x] = *reinterpret_cast<const bf16x8_t*>(w[x] + 32 * s);
        float4 v0, v1;
        if (s < zsteps) {
            // pooled features: a step lies in one feature row of one KV head;
            // its split sums are added in split order
            v0 = v1 = make_float4(0.f, 0.f, 0.f, 0.f);
            int hs = s >> hshift, feature = g.ctx == BUDDY_CTX_V;
            if (g.ctx == BUDDY_CTX_KV && hs >= g.nkv) { hs -= g.nkv; feature = 1; }
            const float* pp = g.pool_part + ((size_t)b * g.nkv + hs) * g.pool_max_splits * row +
                              feature * g.hd + 32 * (s & (hsteps - 1)) + 8 * q;
            // NC splits (and, for K + V, both rows of each) with all loads in flight
            auto fold = [&](int c, auto nc) {
                constexpr int NC = decltype(nc)::value, NW = kNW;
                float4 t[NC][NW][2];
#pragma unroll
                for (int x = 0; x < NC; ++x)
#pragma unroll
                    for (int f = 0; f < NW; ++f) {
                        const float* at = pp + (c + x) * row + f * g.hd;
                        t[x][f][0] = *reinterpret_cast<const float4*>(at);
                        t[x][f][1] = *reinterpret_cast<const float4*>(at + 4);
                    }
#pragma unroll
                for (int x = 0; x < NC; ++x)
#pragma unroll
                    for (int f = 0; f < NW; ++f) {
                        add4(v0, t[x][f][0]);
                        add4(v1, t[x][f][1]);
                    }
            };
            int c = 0;
            for (; c + 8 / kNW <= g.pool_splits; c += 8 / kNW) fold(c, std::integral_constant<int, 8 / kNW>());
            for (; c + 2 <= g.pool_splits; c += 2) fold(c, std::integral_constant<int, 2>());
            for (; c < g.pool_splits; ++c) fold(c, std::integral_constant<int, 1>());
            v0.x *= inv_n; v0.y *= inv_n; v0.z *= inv_n; v0.w *= inv_n;
            v1.x *= inv_n; v1.y *= inv_n; v1.z *= inv_n; v1.w *= inv_n;
        } else {
            v0 = *reinterpret_cast<const float4*>(h + 32 * (s - zsteps));
            v1 = *reinterpret_cast<const float4*>(h + 32 * (s - zsteps) + 4);
        }
        dm_step(a, v0, v1, acc, low);
    }
    // D: lane j + 16 (i / 4), element i % 4: unit i, sequence j
#pragma unroll
    for (int x = 0; x < kDmTiles; ++x)
#pragma unroll
        for (int e = 0; e < 4; ++e) s_red[wave][i][16 * x + 4 * q + e] = acc[x][e] + low[x][e];
    __syncthreads();
    for (int t = tid; t < 16 * kDmUnits; t += 64 * kDmWaves) {
        const int u = t % kDmUnits, j = t / kDmUnits;
        if (h0 + u < g.N && b0 + j < B)
            part[((size_t)blockIdx.x * B + b0 + j) * g.N + h0 + u] =
                (s_red[0][j][u] + s_red[1][j][u]) + (s_red[2][j][u] + s_red[3][j][u]);
    }
}

hipError_t launch_dm(const GemvArgs& g, float* part, hipStream_t s) {
    const int B = g.rows.n_max, steps = g.K / 32, slices = dm_slices(B, g.N, g.K);
    const dim3 grid(slices, (g.N + kDmUnits - 1) / kDmUnits, (B + 15) / 16);
    const int per = (steps + slices - 1) / slices;
    if (g.ctx == BUDDY_CTX_K_PLUS_V) dm_kernel<true><<<grid, 64 * kDmWaves, 0, s>>>(g, B, per, part);
    else dm_kernel<false><<<grid, 64 * kDmWaves, 0, s>>>(g, B, per, part);
    return hipGetLastError();
}

}  // namespace buddy
