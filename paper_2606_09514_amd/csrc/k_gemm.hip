// Tiled MFMA GEMM for projections over many rows (the prompt tokens of a
// routed prefill): Y = W X^T with v_mfma_f32_16x16x32_bf16, fp32 accumulate,
// and the fused epilogues of the decode paths.
//
// A workgroup of WM x WN wavefronts computes a (16 WM TI weight rows) x
// (16 WN TJ rows) tile, each wavefront TI x TJ accumulator tiles of 16 x 16,
// stepping K by 32.  For the two-row kinds (SwiGLU, QKV) the weight rows of
// a tile are 8 WM TI units: their first rows in the upper half of the row
// tiles and their second rows in the lower half, and each wavefront holds
// the first and second rows of the same units.  Three shapes:
//   128 x 128 (2 x 2 wavefronts of 64 x 64), two workgroups per CU;
//   256 x 256 (2 x 4 wavefronts of 128 x 64), one workgroup per CU, which
//     halves the bytes each CU fetches per flop;
//   128 x 256 (2 x 4 wavefronts of 64 x 64), one workgroup per CU: the
//     weights of up to 256 tokens pass once, and twice the grid of the large
//     tile for the 4096-row projections.
// With eight wavefronts the two of each SIMD run in antiphase (below).  What
// bounds the 256 x 256 tile is the MFMA and what does not overlap it: gate/up
// of a 2048-token prompt (Llama-8B shape, three rounds of tiles) 357 us with
// the wavefronts in phase, 328 to 338 in antiphase, 321 with the weights in
// whole lines as well: 1.28 PFLOP/s, where a large library product of random
// bf16 values reaches 1.46 on this card.
// Both operands pass through LDS in MFMA fragment order, so each wavefront
// reads a fragment as one conflict-free 16-byte read per lane (the weights of
// the eight-wavefront tiles lie in whole lines instead, see the loads):
//   A fragment (row tile rt): 1 KB at rt KB of the step's buffer, lane
//     i + 16 q holding tile row 16 rt + i, k = 8 q .. + 7 of the step;
//   B fragment (column tile ct): 1 KB after the A fragments, copied as is
//     from the activations, which the staging kernel already wrote in
//     B-operand order (16 rows x 32 k per contiguous KB).
// Tiles travel straight from memory to LDS (global_load_lds) three K steps
// ahead of the multiply (four buffers); in the 128 x 128 tile each row tile's
// MFMAs start as soon as its own fragment read has landed.
//   D[i][j] (16 x 16): lane j + 16 (i / 4), element i % 4.
#include "buddy_internal.h"
#include "epilogue.h"

namespace buddy {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

typedef __attribute__((address_space(1))) const void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

constexpr int kTileK = 32;
constexpr int kFragBytes = 1024;                 // one 16 x 32 bf16 fragment
constexpr int kBufs = 4;                         // K steps in LDS, three ahead
constexpr int kPairBufs = 3;                     // pairs of K steps of weights in LDS

// s_waitcnt operand: at most n vector-memory operations outstanding, other
// counters unconstrained (gfx9 encoding: vmcnt low bits 3:0 and high bits
// 15:14, expcnt 6:4, lgkmcnt 11:8).
constexpr int vmcnt_at_most(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

// Fragment reads from LDS: 16 bytes at address a (or b) plus immediate
// offsets, issued without a wait.  Written as asm so that the compiler, which
// cannot tell the direct-to-LDS loads into the other buffers from these
// reads, does not make them wait for every load in flight.  LDS reads return
// in issue order, so after a step's reads (the B fragments, then the A
// fragments in row-tile order) lgkmcnt(n) means that all but the last n have
// landed, and the MFMAs of row tile i can start once TI - 1 - i reads remain
// (lds_wait): the first MFMAs wait for 4 + 1 reads, not for all of them.
// Other counted operations the compiler issues only make such a wait longer.
// Until its wait, the compiler believes a read's registers written: the wait
// takes them as operands it modifies, so that nothing reads them earlier.
template <int O0, int O1, int O2, int O3>
__device__ __forceinline__ void lds_issue4(uint32_t a, u32x4_t* x) {
    asm volatile(
        "ds_read_b128 %0, %4 offset:%5\n\t"
        "ds_read_b128 %1, %4 offset:%6\n\t"
        "ds_read_b128 %2, %4 offset:%7\n\t"
        "ds_read_b128 %3, %4 offset:%8"
        : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3])
        : "v"(a), "i"(O0), "i"(O1), "i"(O2), "i"(O3)
        : "memory");
}
// B fragments at b + 0, 1, 2, 3 KB, then A fragments at a + O0 .. O3
template <int O0, int O1, int O2, int O3>
__device__ __forceinline__ void lds_issue8(uint32_t a, uint32_t b, u32x4_t* x, u32x4_t* y) {
    asm volatile(
        "ds_read_b128 %4, %9 offset:0\n\t"
        "ds_read_b128 %5, %9 offset:1024\n\t"
        "ds_read_b128 %6, %9 offset:2048\n\t"
        "ds_read_b128 %7, %9 offset:3072\n\t"
        "ds_read_b128 %0, %8 offset:%10\n\t"
        "ds_read_b128 %1, %8 offset:%11\n\t"
        "ds_read_b128 %2, %8 offset:%12\n\t"
        "ds_read_b128 %3, %8 offset:%13"
        : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(y[0]), "=&v"(y[1]),
          "=&v"(y[2]), "=&v"(y[3])
        : "v"(a), "v"(b), "i"(O0), "i"(O1), "i"(O2), "i"(O3)
        : "memory");
}
template <int N>
__device__ __forceinline__ void lds_wait(u32x4_t& r) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(r) : "i"(N));
}
template <int N>
__device__ __forceinline__ void lds_wait(u32x4_t& r, u32x4_t* y) {
    asm volatile("s_waitcnt lgkmcnt(%5)"
                 : "+v"(r), "+v"(y[0]), "+v"(y[1]), "+v"(y[2]), "+v"(y[3])
                 : "i"(N));
}

// Every fragment of a step: nothing may read them before this wait.
template <int TI>
__device__ __forceinline__ void lds_wait_all(u32x4_t* a, u32x4_t* y) {
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(y[0]), "+v"(y[1]), "+v"(y[2]),
                   "+v"(y[3]));
    if constexpr (TI == 8)
        asm volatile("" : "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]));
}

// One K step's MFMAs, row tile I onwards: each row tile after its own read
// (and, for the first, the B fragments') has landed.
template <int I, int TI, int TJ>
__device__ __forceinline__ void mfma_rows(f32x4_t (&acc)[TI][TJ], u32x4_t* a, u32x4_t* bv) {
    if constexpr (I == 0)
        lds_wait<TI - 1>(a[0], bv);
    else
        lds_wait<TI - 1 - I>(a[I]);
#pragma unroll
    for (int j = 0; j < TJ; ++j)
        acc[I][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8_t, a[I]), __builtin_bit_cast(bf16x8_t, bv[j]), acc[I][j], 0,
            0, 0);
    // keep the next row tile's wait behind these MFMAs (the scheduler would
    // otherwise gather the waits ahead of them)
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (I + 1 < TI) mfma_rows<I + 1>(acc, a, bv);
}

template <int WM, int WN, int TI, int TJ>
struct GemmShape {
    static constexpr int kWaves = WM * WN, kThreads = 64 * kWaves;
    static constexpr int kRowTiles = WM * TI, kColTiles = WN * TJ;
    static constexpr int kRows = 16 * kRowTiles, kCols = 16 * kColTiles;
    // eight wavefronts: antiphase, weights in whole cache lines (pairs of K
    // steps in three buffers), one workgroup per CU
    static constexpr bool kPingPong = kWaves == 8;
    static constexpr int kPairBytes = kRowTiles * 2 * kFragBytes;
    static constexpr int kBufBytes = (kRowTiles + kColTiles) * kFragBytes;
    static constexpr int kLds = kPingPong ? kPairBufs * kPairBytes + kBufs * kColTiles * kFragBytes
                                          : kBufs * kBufBytes;
    // fragments each wavefront loads per K step
    static constexpr int kALoads = kRowTiles / kWaves, kBLoads = kColTiles / kWaves;
    static_assert(kRowTiles % kWaves == 0 && kColTiles % kWaves == 0, "even load split");
    static_assert(kLds <= 160 * 1024, "LDS");
    static_assert(TJ == 4 && (TI == 4 || TI == 8), "wavefront tile");
};

// Four finished units or rows of a token (launch row col, row id b): SwiGLU
// outputs as bf16 into the next projection's staging if asked for, one
// 8-byte store (f % 8 == 0), otherwise the shared epilogues.
template <int EPI>
__device__ __forceinline__ void tile_epilogue(const GemvArgs& g, int units, int col, int b, int u,
                                              const float* v0, const float* v1) {
    if (EPI == EPI_SWIGLU && g.xb_out) {
        *reinterpret_cast<uint2*>(g.xb_out + xb_index(col, u, units)) =
            make_uint2(pack_bf16x2(swiglu(v0[0], v1[0]), swiglu(v0[1], v1[1])),
                       pack_bf16x2(swiglu(v0[2], v1[2]), swiglu(v0[3], v1[3])));
        return;
    }
    epilogue4<EPI>(g, b, u, v0, v1);
}

template <int EPI, int WM, int WN, int TI, int TJ>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_kernel(GemvArgs g, int units, int n, float* part, int ubase) {
    using Sh = GemmShape<WM, WN, TI, TJ>;
    constexpr bool kPaired = EPI == EPI_SWIGLU || EPI == EPI_QKV;
    __shared__ __attribute__((aligned(128))) char s_buf[Sh::kLds];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    // split K (part != null): workgroup z takes K steps [z nk, (z + 1) nk)
    // and writes its fp32 sums to part[z][row][unit] for a separate add
    const int K = g.K, S = K >> 5, nk = K / kTileK / gridDim.z, k0 = blockIdx.z * nk;
    const int u0 = ubase + blockIdx.x * (kPaired ? Sh::kRows / 2 : Sh::kRows);   // first unit or row
    const int t0 = blockIdx.y * Sh::kCols;                               // first row (token)
    const int last_tile = (n - 1) >> 4;                                   // last 16-row column tile

    // Direct global -> LDS loads (each lane's 16 bytes land at the wave's LDS
    // base + 16 lane): wavefront w loads row tiles kALoads w .. and column
    // tiles kBLoads w .. of every step.
    constexpr bool PP = Sh::kPingPong;
    constexpr int kARows = PP ? 2 : 1;        // loads (row addresses) per row tile
    auto weight_row = [&](int r) {            // row r of the tile
        if constexpr (kPaired) {
            const int half = Sh::kRows / 2;
            const int u = min(u0 + (r % half), units - 1);
            int r0, r1;
            unit_rows<EPI>(g, u, r0, r1);
            return r < half ? r0 : r1;
        } else {
            return min(u0 + r, units - 1);
        }
    };
    // A, one step per load: fragment lane i + 16 q holds tile row 16 rt + i,
    // k = 8 q of the step.  PP, two steps per pair of loads: load h of a row
    // tile brings rows 8 h .. 8 h + 7, one whole 128-byte line each (two steps of
    // 32; half lines cost the memory system as many requests as whole ones),
    // lane L's chunk L % 8 of row L / 8 holding source chunk (L % 8) ^ (row % 8),
    // which spreads the fragment reads over the banks.
    const bf16_t* arow[Sh::kALoads][kARows];
#pragma unroll
    for (int t = 0; t < Sh::kALoads; ++t)
#pragma unroll
        for (int h = 0; h < kARows; ++h) {
            const int rl = PP ? 8 * h + (lane >> 3) : lane & 15;
            const int chunk = PP ? (lane & 7) ^ (lane >> 3) : lane >> 4;
            arow[t][h] = (const bf16_t*)g.W + (size_t)weight_row(16 * (Sh::kALoads * wave + t) + rl) * K + 8 * chunk;
        }
    const bf16_t* bfrag[Sh::kBLoads];
#pragma unroll
    for (int t = 0; t < Sh::kBLoads; ++t) {
        const int c = min((t0 >> 4) + Sh::kBLoads * wave + t, last_tile);   // repeats of the last tile are discarded
        bfrag[t] = g.XB + ((size_t)c * S * 64 + lane) * 8;
    }
    constexpr int kBBase = PP ? kPairBufs * Sh::kPairBytes : Sh::kRowTiles * kFragBytes;
    constexpr int kBStep = PP ? Sh::kColTiles * kFragBytes : Sh::kBufBytes;
    // steps (pairs) past the end reload the last one into a buffer that is not
    // read again
    auto issue_b = [&](int kb) {
        const int kc = k0 + min(kb, nk - 1);
#pragma unroll
        for (int t = 0; t < Sh::kBLoads; ++t)
            __builtin_amdgcn_global_load_lds(
                (gptr_t)(bfrag[t] + (size_t)kc * 512),
                (lptr_t)(s_buf + kBBase + (kb % kBufs) * kBStep + (Sh::kBLoads * wave + t) * kFragBytes), 16, 0, 0);
    };
    auto issue_a = [&](int kb) {   // one step's fragments (128 x 128 tile)
        const int kc = k0 + min(kb, nk - 1);
#pragma unroll
        for (int t = 0; t < Sh::kALoads; ++t)
            __builtin_amdgcn_global_load_lds((gptr_t)(arow[t][0] + kc * kTileK),
                                             (lptr_t)(s_buf + (kb % kBufs) * Sh::kBufBytes +
                                                      (Sh::kALoads * wave + t) * kFragBytes),
                                             16, 0, 0);
    };
    auto issue_half = [&](int pair, int pbuf, int h) {   // rows 8 h .. of a pair of steps
        const int kc = k0 + 2 * min(pair, nk / 2 - 1);
#pragma unroll
        for (int t = 0; t < Sh::kALoads; ++t)
            __builtin_amdgcn_global_load_lds((gptr_t)((h ? arow[t][kARows - 1] : arow[t][0]) + kc * kTileK),
                                             (lptr_t)(s_buf + pbuf * Sh::kPairBytes +
                                                      (Sh::kALoads * wave + t) * 2 * kFragBytes + h * kFragBytes),
                                             16, 0, 0);
    };
    constexpr int kLoads = Sh::kALoads + Sh::kBLoads;   // per wavefront and step

    f32x4_t acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[i][j] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    // this wavefront's fragments within a buffer.  Row tiles: paired, its
    // units' first rows (TI/2 tiles from wm TI/2) and second rows (the same
    // TI/2 tiles of the lower half); otherwise TI tiles from wm TI.  Column
    // tiles: TJ from wn TJ.
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)s_buf;
    const uint32_t b_off = lds0 + lane * 16 + kBBase + wn * TJ * kFragBytes;
    constexpr int F = PP ? 2 * kFragBytes : kFragBytes;                 // a row tile's bytes
    // PP: row i = lane % 16 of a tile, chunk 4 u + lane / 16 of step u of the
    // pair, at that chunk ^ (i % 8): bit 6 of the address flips with u
    const uint32_t a_off = lds0 + (PP ? (lane & 15) * 128 + (((lane >> 4) ^ (lane & 7)) * 16) : lane * 16) +
                           (kPaired ? wm * TI / 2 : wm * TI) * F;
    constexpr int kSecond = kPaired ? Sh::kRowTiles / 2 - TI / 2 : 0;   // gap to the second rows

    auto read_frags = [&](uint32_t aa, uint32_t bb, u32x4_t* a, u32x4_t* bv) {
        if constexpr (TI == 4) {
            lds_issue8<0, F, (2 + kSecond) * F, (3 + kSecond) * F>(aa, bb, a, bv);
        } else {
            lds_issue8<0, F, 2 * F, 3 * F>(aa, bb, a, bv);
            lds_issue4<(4 + kSecond) * F, (5 + kSecond) * F, (6 + kSecond) * F, (7 + kSecond) * F>(aa, a + 4);
        }
    };
    if constexpr (Sh::kPingPong) {
        // Two wavefronts per SIMD in antiphase: while wavefronts 0 .. 3 (one
        // per SIMD) multiply a step from registers, wavefronts 4 .. 7 read
        // their next fragments and issue loads, and the other way round, a
        // barrier between the phases.  (In phase, both read LDS and then both
        // multiply: MFMA 44 % busy.)  Early wavefronts read step k in phase 2 k
        // and multiply it in phase 2 k + 1, late ones a phase later.  The loads
        // of step k have landed for everyone after the barrier that ends
        // phase 2 k - 1: each wavefront waits for its own share before it
        // (early: after multiplying step k - 1; late: after reading it), with
        // the loads of steps k + 1 and k + 2, issued by then, in flight.
        // Step k's buffer is refilled with step k + 4's loads by the reads of
        // step k + 1 (phase 2 k + 2 at the earliest): everyone has read step k
        // by the end of phase 2 k + 1, its reads waited for before the barrier.
        // The weights of a pair of steps P arrive in halves, issued while
        // reading steps 2 P - 4 and 2 P - 3, each with the B tiles of the step
        // three ahead: the counts above hold for both, and a pair's buffer (P % 3)
        // held pair P - 3, whose steps everyone has read by then.
        const bool late = wave >= 4;
        issue_half(0, 0, 0);
        issue_half(0, 0, 1);
        issue_b(0);
        issue_half(1, 1, 0);
        issue_b(1);
        issue_half(1, 1, 1);
        issue_b(2);
        __builtin_amdgcn_s_waitcnt(vmcnt_at_most(2 * kLoads));
        asm volatile("s_barrier" ::: "memory");
        if (late) asm volatile("s_barrier" ::: "memory");   // phase 0 is the early wavefronts'
        int pread = 0, pload = 2;                            // pair buffers of this step's reads and loads
        for (int kb = 0; kb < nk; ++kb) {
            u32x4_t a[TI], bv[TJ];
            read_frags((a_off + pread * Sh::kPairBytes) ^ ((kb & 1) * 64), b_off + (kb % kBufs) * kBStep, a, bv);
            issue_half((kb >> 1) + 2, pload, kb & 1);
            issue_b(kb + 3);
            if (kb & 1) {
                pread = pread == kPairBufs - 1 ? 0 : pread + 1;
                pload = pload == kPairBufs - 1 ? 0 : pload + 1;
            }
            lds_wait_all<TI>(a, bv);
            if (late) __builtin_amdgcn_s_waitcnt(vmcnt_at_most(2 * kLoads));
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_barrier" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8_t, a[i]), __builtin_bit_cast(bf16x8_t, bv[j]),
                        acc[i][j], 0, 0, 0);
            __builtin_amdgcn_s_setprio(0);
            if (!late) __builtin_amdgcn_s_waitcnt(vmcnt_at_most(2 * kLoads));
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_barrier" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!late) asm volatile("s_barrier" ::: "memory");  // the late wavefronts' last phase
    } else {
        // At step kb: wait until only the loads of steps kb + 1 and kb + 2 are
        // outstanding, barrier (every wavefront's loads of step kb have landed
        // and every wavefront has read step kb - 1's buffer), refill that
        // buffer with step kb + 3, multiply step kb.
        for (int kb = 0; kb < 3; ++kb) {
            issue_a(kb);
            issue_b(kb);
        }
        for (int kb = 0; kb < nk; ++kb) {
            __builtin_amdgcn_s_waitcnt(vmcnt_at_most(2 * kLoads));
            // a plain barrier: __syncthreads() would also wait for every load
            // in flight (its fence covers the direct-to-LDS writes)
            asm volatile("s_barrier" ::: "memory");
            issue_a(kb + 3);
            issue_b(kb + 3);
            u32x4_t a[TI], bv[TJ];
            const uint32_t sb = (kb % kBufs) * Sh::kBufBytes;
            read_frags(a_off + sb, b_off + sb, a, bv);
            mfma_rows<0>(acc, a, bv);
        }
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_at_most(0));   // the reloads past the end

    // rows (or units) 4 (lane / 16) .. + 3 of each tile, one column (token) per
    // lane: four at a time
    constexpr int NU = kPaired ? TI / 2 : TI;                       // tiles of rows or units
    const int N = kPaired ? 2 * units : units;
    float* pz = part + (size_t)blockIdx.z * n * N;
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
        const int col = t0 + 16 * (wn * TJ + j) + (lane & 15);
        if (col >= n) continue;
        const int b = row_seq(g.rows, col);
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            const int u = u0 + 16 * (wm * NU + i) + 4 * (lane >> 4);
            if (u >= units) continue;                               // units % 4 == 0
            float v0[4], v1[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v0[e] = acc[i][j][e];
                v1[e] = kPaired ? acc[TI - NU + i][j][e] : 0.f;
            }
            if (part) {   // split K: part[split][token][weight row]
                int r0 = u, r1 = u;
                if (kPaired) unit_rows<EPI>(g, u, r0, r1);
                *reinterpret_cast<float4*>(pz + (size_t)col * N + r0) = make_float4(v0[0], v0[1], v0[2], v0[3]);
                if (kPaired)
                    *reinterpret_cast<float4*>(pz + (size_t)col * N + r1) = make_float4(v1[0], v1[1], v1[2], v1[3]);
            } else {
                tile_epilogue<EPI>(g, units, col, b, u, v0, v1);
            }
        }
    }
}

// ----------------------------------------------------------- staging

// Activation staging for the tiled GEMM, RMSNorm folded in: a workgroup of
// 1024 threads takes four rows, 256 threads each, which hold their row in
// registers (KG groups of eight elements per thread, K <= 2048 KG), so that
// it is read once; the bf16 values pass through LDS and leave as 64-byte
// pieces (four rows of an 8-column chunk) of the 16-row fragments.  Rows past
// the last write zeros.  With addpart (split sums of the O projection, [split][row][K]
// by launch row) the residual add happens here, in split order, and the row
// is written back.  Latency bounds a short prompt, so many small workgroups:
// 197 rows of 4096 took 14.8 us with a wavefront per row and 16 rows per
// workgroup (13 workgroups, each row read twice), now 4.4; 2048 rows 18.5 and
// 11.4.
constexpr int kPrepRows = 4;
template <int KG>
__global__ __launch_bounds__(1024) void prep_rows_kernel(GemvArgs g, int n) {
    constexpr int kPitch = KG * 2048 * 2 + 16;   // bytes per LDS row, conflict-free pieces
    __shared__ __attribute__((aligned(16))) char s_rows[kPrepRows * kPitch];
    __shared__ float s_ss[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = tid >> 8, t = tid & 255;
    const int i = kPrepRows * blockIdx.x + r, K = g.K;   // launch row
    const bool live = i < n;
    float* x = const_cast<float*>(g.X) + (size_t)(live ? row_seq(g.rows, i) : 0) * g.ldx;
    float4 v[2 * KG];
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < KG; ++q) {
        const int k = 8 * (t + 256 * q);
        v[2 * q] = v[2 * q + 1] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (!live || k >= K) continue;
        v[2 * q] = *reinterpret_cast<const float4*>(x + k);
        v[2 * q + 1] = *reinterpret_cast<const float4*>(x + k + 4);
    }
    if (g.addpart && live) {
#pragma unroll
        for (int q = 0; q < KG; ++q) {
            const int k = 8 * (t + 256 * q);
            if (k >= K) continue;
            float4 a0 = make_float4(0.f, 0.f, 0.f, 0.f), a1 = a0;
#pragma unroll 4
            for (int z = 0; z < g.addpart_splits; ++z) {
                const float* pz = g.addpart + ((size_t)z * g.addpart_cap + i) * K + k;
                const float4 p0 = *reinterpret_cast<const float4*>(pz), p1 = *reinterpret_cast<const float4*>(pz + 4);
                a0.x += p0.x; a0.y += p0.y; a0.z += p0.z; a0.w += p0.w;
                a1.x += p1.x; a1.y += p1.y; a1.z += p1.z; a1.w += p1.w;
            }
            v[2 * q].x += a0.x; v[2 * q].y += a0.y; v[2 * q].z += a0.z; v[2 * q].w += a0.w;
            v[2 * q + 1].x += a1.x; v[2 * q + 1].y += a1.y; v[2 * q + 1].z += a1.z; v[2 * q + 1].w += a1.w;
            *reinterpret_cast<float4*>(x + k) = v[2 * q];
            *reinterpret_cast<float4*>(x + k + 4) = v[2 * q + 1];
        }
    }
#pragma unroll
    for (int q = 0; q < 2 * KG; ++q) ss += v[q].x * v[q].x + v[q].y * v[q].y + v[q].z * v[q].z + v[q].w * v[q].w;
    ss = wave_sum(ss);
    if (lane == 0) s_ss[wave] = ss;
    __syncthreads();
    ss = (s_ss[4 * r] + s_ss[4 * r + 1]) + (s_ss[4 * r + 2] + s_ss[4 * r + 3]);
    const float inv = 1.0f / sqrtf(ss / (float)K + g.eps);
#pragma unroll
    for (int q = 0; q < KG; ++q) {
        const int k = 8 * (t + 256 * q);
        if (k >= K) continue;
        float gv[8];
        St<bf16_t>::vec((const bf16_t*)g.gain + k, gv);
        const float4 a = v[2 * q], b = v[2 * q + 1];
        *reinterpret_cast<uint4*>(s_rows + r * kPitch + 2 * k) =
            make_uint4(pack_bf16x2(a.x * (inv * gv[0]), a.y * (inv * gv[1])),
                       pack_bf16x2(a.z * (inv * gv[2]), a.w * (inv * gv[3])),
                       pack_bf16x2(b.x * (inv * gv[4]), b.y * (inv * gv[5])),
                       pack_bf16x2(b.z * (inv * gv[6]), b.w * (inv * gv[7])));
    }
    __syncthreads();
    for (int f = tid; f < kPrepRows * (K >> 3); f += 1024) {
        const int rr = f & (kPrepRows - 1), k = 8 * (f / kPrepRows);
        *reinterpret_cast<uint4*>(g.XB + xb_index(kPrepRows * blockIdx.x + rr, k, K)) =
            *reinterpret_cast<const uint4*>(s_rows + rr * kPitch + 2 * k);
    }
}

// Plain conversion (inputs no kernel staged): one workgroup of 16 wavefronts
// per 16-row tile and chunk of kPrepChunk columns; wavefront w converts row w
// into LDS (rows padded by 16 bytes), then every thread writes whole 16-byte
// pieces of the tile's fragments, consecutive threads to consecutive addresses.
constexpr int kPrepChunk = 2048;                 // columns per workgroup
constexpr int kPrepPitch = kPrepChunk * 2 + 16;  // bytes per LDS row

__global__ __launch_bounds__(1024) void prep_tile_kernel(GemvArgs g, int n) {
    __shared__ __attribute__((aligned(16))) char s_rows[16 * kPrepPitch];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile = blockIdx.x, K = g.K, S = K >> 5;
    const int i = 16 * tile + w;                      // this wavefront's row (list index)
    const bool live = i < n;
    const int c0 = blockIdx.y * kPrepChunk, kc = min(kPrepChunk, K - c0);
    const float* x = g.X + (size_t)(live ? row_seq(g.rows, i) : 0) * g.ldx + c0;
    char* row = s_rows + w * kPrepPitch;
    for (int k = 4 * lane; k < kc; k += 256) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (live) v = *reinterpret_cast<const float4*>(x + k);
        *reinterpret_cast<uint2*>(row + 2 * k) = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
    }
    __syncthreads();
    // fragment (k-step s, lane L): row L % 16, columns 32 s + 8 (L / 16) .. + 7
    const int nfrag = (kc >> 5) * 64;
    for (int f = tid; f < nfrag; f += 1024) {
        const int sl = f >> 6, L = f & 63;
        const uint4 v = *reinterpret_cast<const uint4*>(s_rows + (L & 15) * kPrepPitch +
                                                       2 * (32 * sl + 8 * (L >> 4)));
        const size_t frag = ((size_t)tile * S + (c0 >> 5) + sl) * 64 + L;
        *reinterpret_cast<uint4*>(g.XB + frag * 8) = v;
    }
}

static hipError_t launch_prep_tiles(int pro, const GemvArgs& g, hipStream_t s) {
    const int n = g.rows.n_max, tiles = (n + 15) / 16;
    if (pro == PRO_RMSNORM) {
        const int wgs = 16 / kPrepRows * tiles;
        if (g.K <= 2048) prep_rows_kernel<1><<<wgs, 1024, 0, s>>>(g, n);
        else if (g.K <= 4096) prep_rows_kernel<2><<<wgs, 1024, 0, s>>>(g, n);
        else if (g.K <= 8192) prep_rows_kernel<4><<<wgs, 1024, 0, s>>>(g, n);
        else return hipErrorInvalidValue;   // K = d_model (at most 8192, checked at create)
    } else if (pro == PRO_NONE) {
        const int chunks = (g.K + kPrepChunk - 1) / kPrepChunk;
        prep_tile_kernel<<<dim3(tiles, chunks), 1024, 0, s>>>(g, n);
    } else {
        return hipErrorInvalidValue;        // the router context feeds no prompt projection
    }
    return hipGetLastError();
}

constexpr int kCUs = 256;   // compute units of the MI355X: one round of 256 x 256 tiles

// units (weight rows, or row pairs for the two-row kinds) per row tile
template <int EPI, int WM, int WN, int TI, int TJ>
constexpr int tile_units() {
    return EPI == EPI_SWIGLU || EPI == EPI_QKV ? GemmShape<WM, WN, TI, TJ>::kRows / 2
                                               : GemmShape<WM, WN, TI, TJ>::kRows;
}

template <int EPI, int WM, int WN, int TI, int TJ>
static dim3 gemm_grid(int units, int n) {
    constexpr int per = tile_units<EPI, WM, WN, TI, TJ>();
    return dim3((units + per - 1) / per, (n + GemmShape<WM, WN, TI, TJ>::kCols - 1) /
                                             GemmShape<WM, WN, TI, TJ>::kCols);
}

// Units [ubase, uend) of the projection (uend = -1: to the last one).
template <int EPI, int WM, int WN, int TI, int TJ>
static void gemm_launch(const GemvArgs& g, int units, int n, hipStream_t s, float* part = nullptr,
                        int splits = 1, int ubase = 0, int uend = -1) {
    dim3 grid = gemm_grid<EPI, WM, WN, TI, TJ>((uend < 0 ? units : uend) - ubase, n);
    grid.z = splits;
    launch_main(gemm_kernel<EPI, WM, WN, TI, TJ>, grid, dim3(GemmShape<WM, WN, TI, TJ>::kThreads),
                0, s, g, units, n, part, ubase);
}

// Split-K partial sums (part[split][token][weight row]) added in split order,
// then the epilogue, four units (or rows) of a token per thread.
template <int EPI>
__global__ __launch_bounds__(256) void splitk_epi_kernel(GemvArgs g, int units, int n, int splits,
                                                         const float* part) {
    constexpr bool kPaired = EPI == EPI_SWIGLU || EPI == EPI_QKV;
    const int q = units >> 2, N = kPaired ? 2 * units : units;
    for (size_t t = (size_t)blockIdx.x * 256 + threadIdx.x; t < (size_t)n * q;
         t += (size_t)gridDim.x * 256) {
        const int col = (int)(t / q), u = 4 * (int)(t - (size_t)col * q);
        int r0 = u, r1 = u;
        if (kPaired) unit_rows<EPI>(g, u, r0, r1);
        float4 s0 = make_float4(0.f, 0.f, 0.f, 0.f), s1 = s0;
#pragma unroll 4
        for (int z = 0; z < splits; ++z) {
            const float* pz = part + ((size_t)z * n + col) * N;
            const float4 a = *reinterpret_cast<const float4*>(pz + r0);
            s0.x += a.x; s0.y += a.y; s0.z += a.z; s0.w += a.w;
            if (kPaired) {
                const float4 b = *reinterpret_cast<const float4*>(pz + r1);
                s1.x += b.x; s1.y += b.y; s1.z += b.z; s1.w += b.w;
            }
        }
        const float v0[4] = {s0.x, s0.y, s0.z, s0.w}, v1[4] = {s1.x, s1.y, s1.z, s1.w};
        tile_epilogue<EPI>(g, units, col, row_seq(g.rows, col), u, v0, v1);
    }
}

// Tile shapes: weight rows x tokens.
enum Shape { SH_128 = 0, SH_256 = 1, SH_128x256 = 2 };

template <int EPI>
static dim3 shape_grid(int shape, int units, int n) {
    if (shape == SH_256) return gemm_grid<EPI, 2, 4, 8, 4>(units, n);
    if (shape == SH_128x256) return gemm_grid<EPI, 2, 4, 4, 4>(units, n);
    return gemm_grid<EPI, 2, 2, 4, 4>(units, n);
}

// Time of `wgs` workgroups over `steps` K steps, us: rounds over the CUs
// (128 x 128 tiles run two to a CU) times what a step was measured to take
// (Llama-8B and Qwen-7B projections, 64 to 3150 tokens).
static float grid_us(int shape, int wgs, int steps) {
    if (shape == SH_128) {
        const int rest = wgs % (2 * kCUs);
        return steps * (0.74f * (wgs / (2 * kCUs)) + (rest > kCUs ? 0.74f : rest > 0 ? 0.36f : 0.f));
    }
    return steps * (shape == SH_256 ? 0.84f : 0.57f) * ((wgs + kCUs - 1) / kCUs);
}

// The last round of a 256 x 256 grid that does not fill the CUs: the units
// of the row tiles that fill whole rounds stay on 256 x 256 tiles, and the
// rest go to a second launch of 128 x 256 tiles when those take one round
// (0.57 of a large round's 0.84 us a step) instead of a partly idle round of
// the large one (gate/up of a 2048-token prompt, Llama-8B shape, half a round
// left: 95 us on 128 x 128 tiles, two to a CU, now 66).  Returns the first
// unit of the second launch, or units for none.  The outputs are the same bit
// for bit: every output sums its K steps in the same order in either tile.
template <int EPI>
static int gemm_tail_units(int units, int n) {
    const dim3 big = shape_grid<EPI>(SH_256, units, n);
    const int tiles = big.x * big.y, whole = tiles / kCUs * kCUs;
    if (whole == tiles || whole == 0) return units;
    const int ubig = whole / big.y * tile_units<EPI, 2, 4, 8, 4>();
    const dim3 rest = shape_grid<EPI>(SH_128x256, units - ubig, n);
    return (int)(rest.x * rest.y) <= kCUs ? ubig : units;
}

// The projection on one tile shape with K in `splits` parts (1: no partial
// sums), the split sums' epilogue behind it unless the next staging adds them
// (fold: *fold receives the splits); tail: unsplit 256 x 256 tiles with a last
// round on 128 x 256 ones (gemm_tail_units).
template <int EPI>
static hipError_t launch_shape(int shape, int splits, const GemvArgs& g, int units, int n, float* part,
                               hipStream_t s, bool tail = false, int* fold = nullptr) {
    if (splits == 1) part = nullptr;
    if (shape == SH_256) {
        // never with a K split: the split sums added behind are those of every unit
        const int ubig = tail && splits == 1 ? gemm_tail_units<EPI>(units, n) : units;
        gemm_launch<EPI, 2, 4, 8, 4>(g, units, n, s, part, splits, 0, ubig);
        if (ubig < units) gemm_launch<EPI, 2, 4, 4, 4>(g, units, n, s, nullptr, 1, ubig);
    } else if (shape == SH_128x256) {
        gemm_launch<EPI, 2, 4, 4, 4>(g, units, n, s, part, splits);
    } else {
        gemm_launch<EPI, 2, 2, 4, 4>(g, units, n, s, part, splits);
    }
    const hipError_t e = hipGetLastError();
    if (fold) *fold = splits;
    if (e != hipSuccess || splits == 1 || fold) return e;
    const size_t work = (size_t)n * (units / 4);
    const int grid = (int)((work + 255) / 256 < 4096 ? (work + 255) / 256 : 4096);
    splitk_epi_kernel<EPI><<<grid, 256, 0, s>>>(g, units, n, splits, part);
    return hipGetLastError();
}

// Automatic choice: the tile and K split of least estimated time.  Short
// prompts (up to kGemmShortRows tokens) leave most CUs without a tile, so
// their K may split up to eight ways for every kind, as far as the partial
// buffer holds the sums (197 tokens, Llama-8B shape, with the sums' launch:
// O 62 -> 24 us, down 184 -> 47, QKV 67 -> 32, gate/up on 128 x 256 tiles
// 102 -> 81 against 128 x 128 tiles unsplit; 900 tokens, 6 blocks 3040 ->
// 2257, 13B MHA shape, 1500 tokens, 4 blocks 4960 -> 3480); longer ones split
// only the residual adds in two, where that fills the CUs.  Adding split sums
// costs their write and read (about 5 TB/s) and a launch.
template <int EPI>
static hipError_t launch_auto(const GemvArgs& g, int units, float* part, size_t part_elems, hipStream_t s,
                              int* fold) {
    const int n = g.rows.n_max, steps = g.K / kTileK;
    const size_t N = EPI == EPI_ADD ? units : 2 * units;
    const bool few = n <= kGemmShortRows;
    int shape = SH_128, splits = 1;
    float best = 0.f;
    for (int sh : {SH_128, SH_256, SH_128x256})
        for (int z = 1; z <= 8; z *= 2) {
            const dim3 grid = shape_grid<EPI>(sh, units, n);
            const int wgs = grid.x * grid.y;
            if (z > 1 && (!part || !gemm_split_ok(steps, z) || z * n * N > part_elems)) break;
            if (z > 1 && !few && (EPI != EPI_ADD || sh != SH_256 || z > 2 || 2 * wgs < kCUs)) break;
            float us = grid_us(sh, wgs * z, steps / z);
            if (z > 1) us += (fold ? 0.f : 4.f) + (float)z * n * N * 8.f / 5e6f;
            if (sh == SH_256 && z == 1) {
                const int ubig = gemm_tail_units<EPI>(units, n);
                if (ubig < units) us = grid_us(sh, wgs / kCUs * kCUs, steps) + grid_us(SH_128x256, 1, steps);
            }
            if (best == 0.f || us < best) { best = us; shape = sh; splits = z; }
        }
    return launch_shape<EPI>(shape, splits, g, units, n, part, s, true, fold);
}

template <int EPI>
static hipError_t launch_gemm_epi(const GemvArgs& g, int units, int tile, float* part,
                                  size_t part_elems, hipStream_t s, int* fold = nullptr) {
    const int n = g.rows.n_max;
    if (tile == BUDDY_GEMM_TILE_AUTO) return launch_auto<EPI>(g, units, part, part_elems, s, fold);
    if (tile == BUDDY_GEMM_TILE_128) return launch_shape<EPI>(SH_128, 1, g, units, n, nullptr, s, false, fold);
    if (tile != BUDDY_GEMM_TILE_256_SPLIT || EPI != EPI_ADD || !part)
        return launch_shape<EPI>(SH_256, 1, g, units, n, nullptr, s, false, fold);
    // halves of an odd number of steps: the 128 x 128 tile, which takes its
    // weights step by step, gives the same sums
    return launch_shape<EPI>((g.K / kTileK) % 4 == 0 ? SH_256 : SH_128, 2, g, units, n, part, s, false, fold);
}

hipError_t launch_gemm(int pro, int epi, const GemvArgs& g, int tile, float* part, size_t part_elems,
                       hipStream_t s, int* fold) {
    if (pro != PRO_STAGED) {
        hipError_t e = launch_prep_tiles(pro, g, s);
        if (e != hipSuccess) return e;
    }
    if (epi == EPI_QKV)
        return launch_gemm_epi<EPI_QKV>(g, (g.nq + 2 * g.nkv) * (g.hd / 2), tile, part, part_elems, s);
    if (epi == EPI_SWIGLU) return launch_gemm_epi<EPI_SWIGLU>(g, g.f, tile, part, part_elems, s);
    if (epi != EPI_ADD) return hipErrorInvalidValue;
    return launch_gemm_epi<EPI_ADD>(g, g.N, tile, part, part_elems, s, fold);
}

}  // namespace buddy
