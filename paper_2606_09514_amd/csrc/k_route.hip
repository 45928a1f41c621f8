// Router-side kernels of the budget-routed decode step (gfx950).
//
//  setup_kernel   publishes the step's positions and budgets to device memory
//                 and the identity row list used by the always-run blocks.
//  pool_kernel    KV-aware planner (Sec. 4.3): sums of the first layer's K
//                 and V rows 0..pos per KV head over a few split position
//                 ranges; the Decision Module's first layer (dm_kernel, or
//                 the GEMV's PRO_POOL in k_gemv.hip) folds the splits into the
//                 means and joins the newest hidden state,
//                 z = [mean K | mean V | h].
//  pool_running_kernel  the same sums kept across steps in caller memory:
//                 only rows not yet summed are read (normally one per
//                 sequence and step).
//  dm_kernel      first layer of the Decision Module (and Budget Predictor)
//                 over a batch, as K-slice sums that route_kernel adds.
//  route_kernel   Decision Module output layer plus prior fusion (Eq. 2),
//                 deterministic top-k by rank counting, zero-fill of the K/V
//                 row of every skipped block (Conclusion: non-executed states
//                 are zero vectors) and, with skipped-KV masking, the step's
//                 entries of the execution map; with a single sequence it
//                 also does the compaction below.
//  compact_kernel grouping by mask (App. C.1): for every routable block the
//                 ascending list of sequences that run it, their count and
//                 each sequence's row in the list (-1 if absent).
//  topk_kernel    the standalone top-k entry point.
// Partial results always travel through a kernel boundary; no kernel here
// synchronises workgroups (device-wide fences are costly across the XCDs).
#include <type_traits>

#include "buddy_internal.h"
#include "epilogue.h"

namespace buddy {

// ------------------------------------------------------------------ setup

__global__ __launch_bounds__(256) void setup_kernel(StepArgs a, Workspace ws) {
    const int t = threadIdx.x;
    if (t < a.B) {
        ws.pos[t] = a.pos[t];
        ws.kb[t] = a.k[t];
        ws.idx_all[t] = t;
    }
    if (t == 0) ws.n_all[0] = a.B;
}

hipError_t launch_setup(const StepArgs& a, const Workspace& ws, hipStream_t s) {
    setup_kernel<<<1, 256, 0, s>>>(a, ws);
    return hipGetLastError();
}

// ------------------------------------------------------------------- pool

struct PoolParams {
    const void* k0; const void* v0;  // first layer's cache base
    const int32_t* pos; int pos_u;
    float* part;
    int T, hd, nkv, splits, max_splits;
};

typedef uint32_t pool_u4 __attribute__((ext_vector_type(4)));
// 16 bytes of a cache row as fp32 (8 bf16 or 4 fp32 values), nontemporal
__device__ __forceinline__ void nt_vec(const bf16_t* q, float* out) {
    const pool_u4 w = __builtin_nontemporal_load(reinterpret_cast<const pool_u4*>(q));
    out[0] = __uint_as_float(w.x << 16); out[1] = __uint_as_float(w.x & 0xffff0000u);
    out[2] = __uint_as_float(w.y << 16); out[3] = __uint_as_float(w.y & 0xffff0000u);
    out[4] = __uint_as_float(w.z << 16); out[5] = __uint_as_float(w.z & 0xffff0000u);
    out[6] = __uint_as_float(w.w << 16); out[7] = __uint_as_float(w.w & 0xffff0000u);
}
__device__ __forceinline__ void nt_vec(const float* q, float* out) {
    const pool_u4 w = __builtin_nontemporal_load(reinterpret_cast<const pool_u4*>(q));
    out[0] = __uint_as_float(w.x); out[1] = __uint_as_float(w.y);
    out[2] = __uint_as_float(w.z); out[3] = __uint_as_float(w.w);
}

template <typename T>
__global__ __launch_bounds__(256) void pool_kernel(PoolParams p) {
    constexpr int V = St<T>::V;
    __shared__ float red[2][256 * V];   // [K|V][row slot][hd] partial sums
    const int s = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x;
    const int n = seq_pos(p.pos, p.pos_u, b) + 1;
    const int cpr = p.hd / V;           // threads per cache row
    const int rpp = 256 / cpr;          // rows per pass
    const int col = tid % cpr, slot = tid / cpr;
    const int len = (n + p.splits - 1) / p.splits;
    const int j0 = s * len, j1 = min(j0 + len, n);
    const size_t base = ((size_t)b * p.nkv + g) * p.T * p.hd;
    const T* K = (const T*)p.k0 + base;
    const T* Vc = (const T*)p.v0 + base;

    float ak[V], av[V];
#pragma unroll
    for (int e = 0; e < V; ++e) ak[e] = av[e] = 0.f;
    // the rows are read once here (this step's first-block attention has
    // already run): nontemporal 16-byte loads, two rows of each cache in
    // flight per thread.  Bound by the stream; four rows in flight were slower
    // (24 sequences of 750 to 3000 rows, Llama-8B shape, 189 MB: 43.7 us
    // against 33.7; 32 x 2000 rows of the 13B MHA shape, 1.3 GB, the same)
#pragma unroll 2
    for (int j = j0 + slot; j < j1; j += rpp) {
        float kr[V], vr[V];
        nt_vec(K + (size_t)j * p.hd + col * V, kr);
        nt_vec(Vc + (size_t)j * p.hd + col * V, vr);
#pragma unroll
        for (int e = 0; e < V; ++e) { ak[e] += kr[e]; av[e] += vr[e]; }
    }
#pragma unroll
    for (int e = 0; e < V; ++e) {
        red[0][slot * p.hd + col * V + e] = ak[e];
        red[1][slot * p.hd + col * V + e] = av[e];
    }
    __syncthreads();
    float* part = p.part + (((size_t)b * p.nkv + g) * p.max_splits) * 2 * p.hd;
    for (int t = tid; t < 2 * p.hd; t += 256) {
        const int which = t / p.hd, e = t % p.hd;
        float acc = 0.f;
        for (int r = 0; r < rpp; ++r) acc += red[which][r * p.hd + e];
        part[(size_t)s * 2 * p.hd + t] = acc;
    }
}

hipError_t launch_pool(const Model& M, const void* k0, const void* v0, int B, int max_pos,
                       int pos_u, int* splits_out, hipStream_t s) {
    const buddy_config& c = M.cfg;
    PoolParams p;
    p.k0 = k0; p.v0 = v0; p.pos = M.ws.pos; p.pos_u = pos_u;
    p.part = M.ws.pool_part;
    p.T = c.max_ctx; p.hd = c.head_dim; p.nkv = c.n_kv_heads; p.max_splits = M.ws.max_pool_splits;
    const int splits = pool_splits(B, c.n_kv_heads, max_pos, p.max_splits);
    p.splits = splits;
    *splits_out = splits;
    dim3 grid(splits, c.n_kv_heads, B);
    if (c.dtype == BUDDY_BF16) pool_kernel<bf16_t><<<grid, 256, 0, s>>>(p);
    else pool_kernel<float><<<grid, 256, 0, s>>>(p);
    return hipGetLastError();
}

// Running sums: one workgroup per (KV head, sequence) owns its record, so
// the sums and the row count need no synchronisation between workgroups.
// Rows n0..pos-1 join the kept sums (n0 = pool_rows; a count of 0 or above
// pos starts over from empty sums); row pos joins only this call's split.
template <typename T>
__global__ __launch_bounds__(1024) void pool_running_kernel(PoolParams p, float* sum,
                                                            int32_t* rows) {
    constexpr int V = St<T>::V;
    __shared__ float red[2][16][128];   // [K|V][wavefront][hd] partial sums
    const int g = blockIdx.x, b = blockIdx.y;
    const int tid = threadIdx.x;
    const int pos = seq_pos(p.pos, p.pos_u, b);
    int32_t* cnt = rows + (size_t)b * p.nkv + g;
    float* rec = sum + ((size_t)b * p.nkv + g) * 2 * p.hd;
    int n0 = *cnt;
    const bool restart = n0 <= 0 || n0 > pos;   // count 0: the kept sums are not read
    if (restart) n0 = 0;
    const int cpr = p.hd / V, rpp = 1024 / cpr;
    const int col = tid % cpr, slot = tid / cpr;
    const size_t base = ((size_t)b * p.nkv + g) * p.T * p.hd;
    const T* K = (const T*)p.k0 + base;
    const T* Vc = (const T*)p.v0 + base;
    float ak[V], av[V];
#pragma unroll
    for (int e = 0; e < V; ++e) ak[e] = av[e] = 0.f;
    for (int j = n0 + slot; j < pos; j += rpp) {
        float kr[V], vr[V];
        St<T>::vec(K + (size_t)j * p.hd + col * V, kr);
        St<T>::vec(Vc + (size_t)j * p.hd + col * V, vr);
#pragma unroll
        for (int e = 0; e < V; ++e) { ak[e] += kr[e]; av[e] += vr[e]; }
    }
    // rows of one wavefront first (lanes cpr apart share a column), then
    // the 16 wavefronts through LDS
    const int lane = tid & 63, wave = tid >> 6;
    for (int o = cpr; o < kWave; o <<= 1) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            ak[e] += __shfl_xor(ak[e], o, kWave);
            av[e] += __shfl_xor(av[e], o, kWave);
        }
    }
    if (lane < cpr) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            red[0][wave][col * V + e] = ak[e];
            red[1][wave][col * V + e] = av[e];
        }
    }
    __syncthreads();   // every thread has also read *cnt before it is replaced
    float* part = p.part + ((size_t)b * p.nkv + g) * p.max_splits * 2 * p.hd;
    for (int t = tid; t < 2 * p.hd; t += 1024) {
        const int which = t / p.hd, e = t % p.hd;
        float acc = restart ? 0.f : rec[t];
        for (int w = 0; w < 16; ++w) acc += red[which][w][e];
        rec[t] = acc;
        part[t] = acc + St<T>::get(which ? Vc : K, (size_t)pos * p.hd + e);
    }
    if (tid == 0) *cnt = pos;
}

hipError_t launch_pool_running(const Model& M, const void* k0, const void* v0, float* pool_sum,
                               int32_t* pool_rows, int B, int pos_u, hipStream_t s) {
    const buddy_config& c = M.cfg;
    PoolParams p;
    p.k0 = k0; p.v0 = v0; p.pos = M.ws.pos; p.pos_u = pos_u;
    p.part = M.ws.pool_part;
    p.T = c.max_ctx; p.hd = c.head_dim; p.nkv = c.n_kv_heads; p.max_splits = M.ws.max_pool_splits;
    p.splits = 1;
    dim3 grid(c.n_kv_heads, B);
    if (c.dtype == BUDDY_BF16) pool_running_kernel<bf16_t><<<grid, 1024, 0, s>>>(p, pool_sum, pool_rows);
    else pool_running_kernel<float><<<grid, 1024, 0, s>>>(p, pool_sum, pool_rows);
    return hipGetLastError();
}

// ------------------------------------------------------- router first layer

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
    // D: lane j + 16 (i / 4), element i % 4: unit i, sequence j.  A sum of the
    // first parts that is not finite stands alone: an infinite weight times a
    // remainder of 0 is NaN, times the value it is not.
#pragma unroll
    for (int x = 0; x < kDmTiles; ++x)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float v = acc[x][e];
            s_red[wave][i][16 * x + 4 * q + e] = (v - v) == 0.f ? v + low[x][e] : v;
        }
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

// ------------------------------------------------------------------ route

// Strict total order of the top-k: a number beats NaN, larger beats smaller,
// equal values go to the lower layer index.
__device__ __forceinline__ bool beats(float sj, int j, float si, int i) {
    const bool nj = isnan(sj), ni = isnan(si);
    if (nj != ni) return ni;
    if (!nj && sj != si) return sj > si;
    return j < i;
}

struct RouteParams {
    // first layer's activations [B][H], or (part != null) its K-slice sums
    // [slices][B][H], to which bias b1 and activation are still to come
    const float* a; int H;
    const float* part; int slices; const void* b1; int act;
    const void* w2; const void* b2; const float* prior; float omega;
    int Lm, B;
    int S, L;                         // start layer (routable blocks S..L-2), blocks
    const uint8_t* route_override;
    uint8_t* mask; uint8_t* mask_out;
    float* scores; float* scores_out;
    void* kc; void* vc;               // cache bases (layer 0)
    int T, hd, nkv, bcap;
    int scores_only;
    int32_t* idx; int32_t* cnt;       // compaction outputs (single-sequence launch)
    volatile int32_t* host_cnt; int32_t seq;
    uint8_t* exec;                    // execution map [L][bcap][T] (masking), or null
    // Budget Predictor: hidden activations [B][Hp] (null: budgets from the
    // step arguments), output layer, and the optional outputs
    const float* pa; int Hp; const void* pw2; const void* pb2;
    const float* ppart; int pslices; const void* pb1;   // as part, slices, b1
    int32_t* k_out; float* logits_out;
};

// Groups by mask the routed blocks of a one-sequence batch and publishes the
// counts (shared by route_kernel at B = 1 and compact_kernel).
__device__ __forceinline__ void publish_counts(volatile int32_t* host_cnt, int Lm, int32_t seq) {
    __threadfence_system();
    host_cnt[Lm] = seq;
}

// One output layer row per wavefront: v[i] = W[i] . a + bias[i] (fp32).
template <typename T>
__device__ __forceinline__ void output_layer(const void* w, const void* bias, const float* a,
                                             int H, int Lm, int wave, int lane, float* v) {
    constexpr int V = St<T>::V;
    const int nv = H / V;              // 16-byte vectors per row
    for (int i = wave; i < Lm; i += 16) {
        float acc = 0.f;
        for (int q = lane; q < nv; q += kWave) {
            float wv[V];
            St<T>::vec((const T*)w + (size_t)i * H + q * V, wv);
#pragma unroll
            for (int e = 0; e < V; ++e) acc += wv[e] * a[q * V + e];
        }
        acc = wave_sum(acc);
        if (lane == 0) v[i] = acc + St<T>::get((const T*)bias, i);
    }
}

// First-layer activations of sequence b from the K-slice sums (in slice
// order), into LDS.  Up to 48 slices one after the other in fp32 left the
// scores further from float64 than the GEMV's tree of lanes (rms over ten
// seeds, Llama-8B shape: 1.48e-7 of the scores at 24 sequences of 3000 rows,
// 1.64e-7 at 16 of 20; GEMV 1.37e-7 and 1.38e-7), so they add up in fp64:
// 1.15e-7 at both, in the same time.
template <typename T>
__device__ __forceinline__ void first_layer(const float* part, int slices, int B, int b, const void* b1,
                                            int act, int H, float* s_a) {
    for (int h = threadIdx.x; h < H; h += 1024) {
        const float* pp = part + (size_t)b * H + h;
        double v = St<T>::get((const T*)b1, h);
#pragma unroll 8
        for (int c = 0; c < slices; ++c) v += pp[(size_t)c * B * H];
        s_a[h] = act_fn((float)v, act);
    }
    __syncthreads();
}

// SLICES: some first layer comes as K-slice sums.
template <typename T, bool SLICES>
__global__ __launch_bounds__(1024) void route_kernel(RouteParams p, StepArgs sa) {
    __shared__ float s_sc[256];
    __shared__ uint8_t s_mask[256];
    __shared__ int s_k;
    __shared__ float s_a[SLICES ? kDmMaxHidden : 1];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Lm = p.Lm;

    // Budget Predictor (Sec. 4.4): k = 1 + argmax of the policy logits (the
    // softmax is monotone), smaller k on equal logits, NaN never chosen
    if (p.pa) {
        if (SLICES && p.ppart) {
            first_layer<T>(p.ppart, p.pslices, p.B, b, p.pb1, p.act, p.Hp, s_a);
            output_layer<T>(p.pw2, p.pb2, s_a, p.Hp, Lm, wave, lane, s_sc);
        } else {
            output_layer<T>(p.pw2, p.pb2, p.pa + (size_t)b * p.Hp, p.Hp, Lm, wave, lane, s_sc);
        }
        __syncthreads();
        if (tid < Lm && p.logits_out) p.logits_out[(size_t)b * Lm + tid] = s_sc[tid];
        if (wave == 0) {
            float bv = 0.f;
            int bi = Lm;                                  // none yet
            for (int i = lane; i < Lm; i += kWave) {
                const float v = s_sc[i];
                if (v == v && (bi == Lm || v > bv)) { bv = v; bi = i; }
            }
            for (int o = kWave / 2; o > 0; o >>= 1) {
                const float ov = __shfl_xor(bv, o, kWave);
                const int oi = __shfl_xor(bi, o, kWave);
                if (oi != Lm && (bi == Lm || ov > bv || (ov == bv && oi < bi))) { bv = ov; bi = oi; }
            }
            if (lane == 0) {
                s_k = (bi == Lm ? 0 : bi) + 1;
                if (p.k_out) p.k_out[b] = s_k;
            }
        }
        __syncthreads();   // s_sc is reused for the scores below
    }
    const int kb = p.pa ? s_k : (int)sa.k[b];

    if (p.route_override) {
        if (tid < Lm) s_mask[tid] = p.route_override[(size_t)b * Lm + tid] != 0;
    } else {
        if (SLICES && p.part) {
            first_layer<T>(p.part, p.slices, p.B, b, p.b1, p.act, p.H, s_a);
            output_layer<T>(p.w2, p.b2, s_a, p.H, Lm, wave, lane, s_sc);
        } else {
            output_layer<T>(p.w2, p.b2, p.a + (size_t)b * p.H, p.H, Lm, wave, lane, s_sc);
        }
        __syncthreads();
        if (p.prior && tid < Lm) s_sc[tid] += p.omega * p.prior[tid];
        __syncthreads();
        if (tid < Lm) {
            p.scores[(size_t)b * Lm + tid] = s_sc[tid];
            if (p.scores_out) p.scores_out[(size_t)b * Lm + tid] = s_sc[tid];
        }
        if (p.scores_only) return;
        if (tid < Lm) {
            const float si = s_sc[tid];
            int rank = 0;
            for (int j = 0; j < Lm; ++j) rank += (j != tid) && beats(s_sc[j], j, si, tid);
            s_mask[tid] = rank < kb;
        }
    }
    __syncthreads();
    if (tid < Lm) {
        p.mask[(size_t)b * Lm + tid] = s_mask[tid];
        if (p.mask_out) p.mask_out[(size_t)b * Lm + tid] = s_mask[tid];
        if (gridDim.x == 1) {   // one sequence: this workgroup is the compaction
            p.idx[(size_t)tid * p.bcap] = 0;
            p.cnt[tid] = s_mask[tid];
            if (p.host_cnt) p.host_cnt[tid] = s_mask[tid];
        }
    }
    if (gridDim.x == 1 && p.host_cnt) {
        __syncthreads();
        if (tid == 0) publish_counts(p.host_cnt, Lm, p.seq);
    }

    // with masking, every block's entry of the execution map at this step's
    // position: 1 for blocks 0..S-1, the last block and the selected ones
    const int pos = sa.pos[b];
    if (p.exec && tid < p.L)
        p.exec[((size_t)tid * p.bcap + b) * p.T + pos] =
            (tid < p.S || tid == p.L - 1) ? 1 : s_mask[tid - p.S];

    // zero-filled K/V row at this step's position for every skipped block,
    // written as 16-byte vectors
    constexpr int VZ = St<T>::V;
    const size_t layer_stride = (size_t)p.bcap * p.nkv * p.T * p.hd;
    const int per_layer = p.nkv * (p.hd / VZ);
    for (int t = tid; t < Lm * per_layer; t += 1024) {
        const int i = t / per_layer, r = t % per_layer;
        if (s_mask[i]) continue;
        const int g = r / (p.hd / VZ), e = (r % (p.hd / VZ)) * VZ;
        const size_t at = (size_t)(i + p.S) * layer_stride +
                          (((size_t)b * p.nkv + g) * p.T + pos) * p.hd + e;
        *reinterpret_cast<uint4*>((T*)p.kc + at) = make_uint4(0u, 0u, 0u, 0u);
        *reinterpret_cast<uint4*>((T*)p.vc + at) = make_uint4(0u, 0u, 0u, 0u);
    }
}

// One workgroup: each wavefront scans the mask columns of every fourth
// routable block over the batch (inv: [Lm][bcap] rows).  When host_cnt (mapped pinned host memory)
// is given, the counts are also published there, followed by the step's
// sequence number once they are visible to the host.
__global__ __launch_bounds__(256) void compact_kernel(const uint8_t* mask, int Lm, int B, int bcap,
                                                      int32_t* idx, int32_t* cnt, int32_t* inv,
                                                      volatile int32_t* host_cnt, int32_t seq) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = wave; i < Lm; i += 4) {
        int base = 0;
        for (int b0 = 0; b0 < B; b0 += kWave) {
            const int bb = b0 + lane;
            const bool sel = bb < B && mask[(size_t)bb * Lm + i];
            const uint64_t bal = __ballot(sel);
            const int before = __popcll(bal & ((1ull << lane) - 1ull));
            if (sel) idx[(size_t)i * bcap + base + before] = bb;
            if (bb < B) inv[(size_t)i * bcap + bb] = sel ? base + before : -1;
            base += __popcll(bal);
        }
        if (lane == 0) {
            cnt[i] = base;
            if (host_cnt) host_cnt[i] = base;
        }
    }
    if (host_cnt) {
        __syncthreads();
        if (tid == 0) publish_counts(host_cnt, Lm, seq);
    }
}

hipError_t launch_route(const Model& M, const void* kc, const void* vc, uint8_t* exec, bool predict,
                        int32_t* k_out, float* logits_out, const StepArgs& a,
                        const uint8_t* route_override, uint8_t* mask_out,
                        float* scores_out, bool scores_only, int32_t publish_seq,
                        hipStream_t s) {
    const buddy_config& c = M.cfg;
    const int B = a.B;
    RouteParams p;
    p.a = M.ws.a; p.H = c.dm_hidden;
    p.w2 = M.dm.w2; p.b2 = M.dm.b2; p.prior = M.dm.prior; p.omega = M.dm.omega;
    p.Lm = n_mid(c); p.B = B;
    p.S = start_layer(c); p.L = c.n_layers;
    p.route_override = route_override;
    p.mask = M.ws.mask; p.mask_out = mask_out;
    p.scores = M.ws.scores; p.scores_out = scores_out;
    p.kc = (void*)kc; p.vc = (void*)vc;
    p.T = c.max_ctx; p.hd = c.head_dim; p.nkv = c.n_kv_heads; p.bcap = c.max_batch;
    p.scores_only = scores_only ? 1 : 0;
    p.idx = M.ws.idx; p.cnt = M.ws.cnt;
    p.host_cnt = publish_seq >= 0 ? M.d_host_cnt : nullptr;
    p.seq = publish_seq;
    p.exec = exec;
    p.pa = predict ? M.pred_a : nullptr; p.Hp = M.pred.hidden;
    p.pw2 = M.pred.w2; p.pb2 = M.pred.b2;
    p.k_out = k_out; p.logits_out = logits_out;
    const int din = pooled_dim(c.router_ctx, c.n_kv_heads, c.head_dim) + c.d_model;
    const bool dm = !route_override && dm_uses_mfma(c, B, c.dm_hidden, din);
    const bool pdm = predict && dm_uses_mfma(c, B, M.pred.hidden, din);
    p.part = dm ? M.ws.dm_part : nullptr;
    p.slices = dm_slices(B, c.dm_hidden, din); p.b1 = M.dm.b1; p.act = c.dm_act;
    p.ppart = pdm ? pred_part(M) : nullptr;
    p.pslices = pdm ? dm_slices(B, M.pred.hidden, din) : 0; p.pb1 = M.pred.b1;
    if (c.dtype == BUDDY_F32) route_kernel<float, false><<<B, 1024, 0, s>>>(p, a);
    else if (dm || pdm) route_kernel<bf16_t, true><<<B, 1024, 0, s>>>(p, a);
    else route_kernel<bf16_t, false><<<B, 1024, 0, s>>>(p, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || scores_only || p.Lm == 0 || B == 1) return e;
    compact_kernel<<<1, 256, 0, s>>>(M.ws.mask, p.Lm, B, c.max_batch, M.ws.idx, M.ws.cnt,
                                     M.ws.inv, p.host_cnt, publish_seq);
    return hipGetLastError();
}

// ---------------------------------------------------------------- prefill

// Zero rows 0..len-1 of a skipped block (16-byte stores) and, with an
// execution map, the block's entries: the gridDim.z workgroups of a
// (block, sequence) share its rows.  Bound by the stores (33.5 MB for one
// skipped block of a 2048-token prompt, Llama-8B shape; eight stores of each
// cache per thread keep the CUs busy: one workgroup per (block, sequence)
// took 144 us for three such blocks, now 10 us).
constexpr int kFillPerThread = 8;
template <typename T>
__global__ __launch_bounds__(256) void prefill_fill_kernel(void* kc, void* vc, uint8_t* exec,
                                                           const uint8_t* mask, const int32_t* len,
                                                           int S, int L, int T_cap, int bcap,
                                                           int nkv, int hd) {
    const int b = blockIdx.y, l = blockIdx.x;      // block l of 0..L-1
    const int n = len[b];
    const int Lm = L - 1 - S;
    const bool run = l < S || l == L - 1 || mask[(size_t)b * Lm + (l - S)];
    const int t0 = blockIdx.z * 256 + threadIdx.x, step = gridDim.z * 256;
    if (exec)
        for (int t = t0; t < n; t += step) exec[((size_t)l * bcap + b) * T_cap + t] = run;
    if (run) return;
    constexpr int V = St<T>::V;
    const int per_row = hd / V;
    const size_t layer = (size_t)l * bcap * nkv * T_cap * hd;
    for (int t = t0; t < nkv * n * per_row; t += step) {
        const int g = t / (n * per_row), r = t - g * n * per_row;
        const int row = r / per_row, e = (r - row * per_row) * V;
        const size_t at = layer + (((size_t)b * nkv + g) * T_cap + row) * hd + e;
        *reinterpret_cast<uint4*>((T*)kc + at) = make_uint4(0u, 0u, 0u, 0u);
        *reinterpret_cast<uint4*>((T*)vc + at) = make_uint4(0u, 0u, 0u, 0u);
    }
}

hipError_t launch_prefill_fill(const Model& M, void* kc, void* vc, uint8_t* exec,
                               const uint8_t* mask, const int32_t* len, int B, int max_len,
                               hipStream_t s) {
    const buddy_config& c = M.cfg;
    const int per_row = c.head_dim / (c.dtype == BUDDY_BF16 ? 8 : 4);
    const size_t vecs = (size_t)c.n_kv_heads * max_len * per_row;
    const size_t want = (vecs + 256 * kFillPerThread - 1) / (256 * kFillPerThread);
    const dim3 grid(c.n_layers, B, want < 1024 ? (unsigned)want : 1024);
    if (c.dtype == BUDDY_BF16)
        prefill_fill_kernel<bf16_t><<<grid, 256, 0, s>>>(kc, vc, exec, mask, len, start_layer(c),
                                                         c.n_layers, c.max_ctx, c.max_batch,
                                                         c.n_kv_heads, c.head_dim);
    else
        prefill_fill_kernel<float><<<grid, 256, 0, s>>>(kc, vc, exec, mask, len, start_layer(c),
                                                        c.n_layers, c.max_ctx, c.max_batch,
                                                        c.n_kv_heads, c.head_dim);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void gather_last_kernel(const float* hidden, int t_stride, int d,
                                                          const int32_t* len, float* out) {
    const int b = blockIdx.x;
    const float* src = hidden + ((size_t)b * t_stride + len[b] - 1) * d;
    for (int i = threadIdx.x; i < d; i += 256) out[(size_t)b * d + i] = src[i];
}

hipError_t launch_gather_last(const float* hidden, int t_stride, int d, const int32_t* len, int B,
                              float* out, hipStream_t s) {
    gather_last_kernel<<<B, 256, 0, s>>>(hidden, t_stride, d, len, out);
    return hipGetLastError();
}

// ----------------------------------------------------------- select_topk

struct TopkArgs {
    int n, rows;
    uint8_t k[kMaxBatch];
};

__global__ __launch_bounds__(256) void topk_kernel(const float* scores, uint8_t* mask, TopkArgs a) {
    __shared__ float s_sc[256];
    const int r = blockIdx.x, tid = threadIdx.x;
    if (tid < a.n) s_sc[tid] = scores[(size_t)r * a.n + tid];
    __syncthreads();
    if (tid < a.n) {
        const float si = s_sc[tid];
        int rank = 0;
        for (int j = 0; j < a.n; ++j) rank += (j != tid) && beats(s_sc[j], j, si, tid);
        mask[(size_t)r * a.n + tid] = rank < (int)a.k[r];
    }
}

// ------------------------------------------------------- path grouping

// Orders the batch by route.  Each sequence's route (mask row, nonzero =
// run) is packed into NWD = ceil(n / 64) 64-bit words, block 0 in the top bit
// of word 0, so that comparing the words as unsigned numbers in order
// compares routes lexicographically with skip before run; a sequence's
// position is the count of (route, index) keys below its own, which is
// unique, and it starts a group when no lower-indexed sequence has its route.
// The work is latency and LDS reads (a batch of 200 with 30 blocks has 6 KB
// of input): rows are packed by wavefront ballots of coalesced bytes, and the
// B^2 comparisons are shared by all 1024 threads, each counting for one
// sequence over a slice of the others.  Up to kGroupOneWg sequences one
// workgroup does everything (B = 200, n = 30: 39.9 us with one thread per
// sequence, now 8.8); beyond, group_rank_kernel's workgroups take 64
// sequences each and leave the group-start flag of a position in the top bit
// of its perm entry, which group_scan_kernel takes out again.
constexpr int kGroupOneWg = 256;
constexpr int32_t kGroupStart = INT32_MIN;

// Packs every route into s_key.
template <int NWD>
__device__ __forceinline__ void group_pack(const uint8_t* mask, int B, int n, uint64_t (*s_key)[NWD]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int kRows = 4;   // rows whose loads are in flight together
    for (int t0 = wave; t0 < B; t0 += 16 * kRows) {
        uint8_t m[kRows][NWD];
#pragma unroll
        for (int r = 0; r < kRows; ++r)
#pragma unroll
            for (int q = 0; q < NWD; ++q)
                m[r][q] = mask[(size_t)min(t0 + 16 * r, B - 1) * n + min(64 * q + lane, n - 1)];
#pragma unroll
        for (int r = 0; r < kRows; ++r)
#pragma unroll
            for (int q = 0; q < NWD; ++q) {
                const uint64_t w = __brevll(__ballot(64 * q + lane < n && m[r][q] != 0));
                if (lane == 0 && t0 + 16 * r < B) s_key[t0 + 16 * r][q] = w;
            }
    }
    __syncthreads();
}

// Sequences t0 .. t0 + m - 1: their positions (s_rank) and whether a lower
// index has the same route (s_dup), over all B keys.  m is a multiple of 64
// and at most 1024; entries past B are computed on key 0 and not used.
template <int NWD>
__device__ __forceinline__ void group_rank(int B, int t0, int m, const uint64_t (*s_key)[NWD],
                                           int32_t* s_rank, int32_t* s_dup) {
    const int tid = threadIdx.x;
    if (tid < m) s_rank[tid] = s_dup[tid] = 0;
    __syncthreads();
    const int slices = 1024 / m, sl = tid / m, tl = tid - sl * m;
    const int t = t0 + tl, len = (B + slices - 1) / slices;
    if (sl < slices && t < B) {
        uint64_t k[NWD];
#pragma unroll
        for (int q = 0; q < NWD; ++q) k[q] = s_key[t][q];
        int rank = 0, dup = 0;
        const int b1 = min(B, (sl + 1) * len);
#pragma unroll 4
        for (int b = sl * len; b < b1; ++b) {
            bool below = false, eq = true;
#pragma unroll
            for (int q = 0; q < NWD; ++q) {
                const uint64_t o = s_key[b][q];
                below = below || (eq && o < k[q]);
                eq = eq && o == k[q];
            }
            const bool before = eq && b < t;
            rank += below || before;
            dup |= before;
        }
        atomicAdd(&s_rank[tl], rank);
        if (dup) atomicOr(&s_dup[tl], 1);
    }
    __syncthreads();
}

// Compacts the group-start flags of the positions (flag of position
// threadIdx.x) into starts and the group count; s_tot: 16 words of LDS.
__device__ __forceinline__ void group_scan(int B, bool flag, int32_t* starts, int32_t* n_groups,
                                           int32_t* s_tot) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const uint64_t bal = __ballot(flag);
    if (lane == 0) s_tot[wave] = __popcll(bal);
    __syncthreads();
    int base = 0, total = 0;
    for (int w = 0; w < 16; ++w) {
        if (w < wave) base += s_tot[w];
        total += s_tot[w];
    }
    if (flag) starts[base + __popcll(bal & ((1ull << lane) - 1ull))] = t;
    if (t == 0) {
        starts[total] = B;
        *n_groups = total;
    }
}

template <int NWD>
__global__ __launch_bounds__(1024) void group_kernel(const uint8_t* mask, int B, int n, int32_t* perm,
                                                     int32_t* starts, int32_t* n_groups) {
    __shared__ uint64_t s_key[kGroupOneWg][NWD];
    __shared__ int32_t s_rank[kGroupOneWg], s_dup[kGroupOneWg], s_flag[kGroupOneWg], s_tot[16];
    const int t = threadIdx.x;
    group_pack<NWD>(mask, B, n, s_key);
    group_rank<NWD>(B, 0, (B + 63) / 64 * 64, s_key, s_rank, s_dup);
    if (t < B) {
        perm[s_rank[t]] = t;
        s_flag[s_rank[t]] = !s_dup[t];
    }
    __syncthreads();
    group_scan(B, t < B && s_flag[t], starts, n_groups, s_tot);
}

template <int NWD>
__global__ __launch_bounds__(1024) void group_rank_kernel(const uint8_t* mask, int B, int n,
                                                          int32_t* perm) {
    __shared__ uint64_t s_key[kMaxGroupBatch][NWD];
    __shared__ int32_t s_rank[64], s_dup[64];
    const int t = threadIdx.x, t0 = blockIdx.x * 64;
    group_pack<NWD>(mask, B, n, s_key);
    group_rank<NWD>(B, t0, 64, s_key, s_rank, s_dup);
    if (t < 64 && t0 + t < B) perm[s_rank[t]] = (t0 + t) | (s_dup[t] ? 0 : kGroupStart);
}

__global__ __launch_bounds__(1024) void group_scan_kernel(int B, int32_t* perm, int32_t* starts,
                                                          int32_t* n_groups) {
    __shared__ int32_t s_tot[16];
    const int t = threadIdx.x;
    const int32_t p = t < B ? perm[t] : 0;
    if (t < B) perm[t] = p & ~kGroupStart;
    group_scan(B, (p & kGroupStart) != 0, starts, n_groups, s_tot);
}

template <int NWD>
static hipError_t launch_group(const uint8_t* mask, int B, int n, int32_t* perm, int32_t* starts,
                               int32_t* n_groups, hipStream_t s) {
    if (B <= kGroupOneWg) {
        group_kernel<NWD><<<1, 1024, 0, s>>>(mask, B, n, perm, starts, n_groups);
        return hipGetLastError();
    }
    group_rank_kernel<NWD><<<(B + 63) / 64, 1024, 0, s>>>(mask, B, n, perm);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    group_scan_kernel<<<1, 1024, 0, s>>>(B, perm, starts, n_groups);
    return hipGetLastError();
}

hipError_t launch_group_by_route(const uint8_t* mask, int B, int n, int32_t* perm, int32_t* starts,
                                 int32_t* n_groups, hipStream_t s) {
    if (n <= 64) return launch_group<1>(mask, B, n, perm, starts, n_groups, s);
    if (n <= 128) return launch_group<2>(mask, B, n, perm, starts, n_groups, s);
    return launch_group<4>(mask, B, n, perm, starts, n_groups, s);
}

hipError_t launch_select_topk(const float* scores, const int32_t* k_host, int B, int n,
                              uint8_t* mask_out, hipStream_t s) {
    for (int r0 = 0; r0 < B; r0 += kMaxBatch) {
        TopkArgs a;
        a.n = n;
        a.rows = B - r0 < kMaxBatch ? B - r0 : kMaxBatch;
        for (int r = 0; r < a.rows; ++r) a.k[r] = (uint8_t)k_host[r0 + r];
        topk_kernel<<<a.rows, 256, 0, s>>>(scores + (size_t)r0 * n, mask_out + (size_t)r0 * n, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace buddy
