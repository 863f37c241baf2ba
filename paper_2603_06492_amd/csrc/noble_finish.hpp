// The last launch of a forward whose x W was computed as float32 partial sums
// over K pieces:
//   y[t][n] = sum over s < S of P[s][t][n]  +  C2[t] W_up[:, n]  +  b[n].
//
// Such a forward runs x W and x W_down in one split-K launch (neither needs
// the branch), then the chain, then this kernel: a layer of few tokens has
// too few output tiles to keep 256 CUs reading W, and its K loop is split
// over the idle ones.  Bound by bytes (S T d_out 4 of partials, which the
// preceding launches left in the memory-side cache) and, for a few tokens, by
// the latency of one round trip: every load is issued before any is waited
// for.  32 tokens x 128 columns per workgroup, one 32 x 32 block per wave;
// W_up's [r][128] tile goes through LDS (transposing reads), C2's fragments
// straight to registers.
#pragma once

#include "noble_gemm_tile.hpp"
#include "noble_skinny.hpp"

namespace noble {

constexpr int kFinRows = 32, kFinCols = 128;

struct FinishArgs {
    const float* P;       // partials [S][T][dout]
    int64_t pstride;      // T * dout
    const uint16_t* C2s;  // [T][R]
    const uint16_t* Wu;   // [G r][dog]
    const float* b;       // [dout] or NULL
    uint16_t* y;          // [T][dout]
    int T, S, G, r, R, dog, dout, pad_;
};

// NC: 64-row chunks of W_up (r <= 64 NC).
template <int NC>
__global__ __launch_bounds__(256) void y_finish_kernel(FinishArgs a) {
    constexpr int kTile = 64 * kFinCols * 2;
    __shared__ __attribute__((aligned(1024))) char lds[NC * kTile];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    const int tiles_n = (a.dog + kFinCols - 1) / kFinCols;
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const int per = a.G * tiles_n;
    const int rb = uni((int)blockIdx.x / per), rem = (int)blockIdx.x - rb * per;
    const int g = uni(rem / tiles_n), n0 = (rem - g * tiles_n) * kFinCols;
    const int row0 = rb * kFinRows, c0 = g * a.r;

    Seg su;
    su.ptr = reinterpret_cast<const char*>(a.Wu + (int64_t)c0 * a.dog);
    su.ld = a.dog;
    su.klen = a.r;
    TileDma<false, kFinCols, 4> dma;
    dma.segment(su, a.dog, n0, wave, lane);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const i32x4 d = dma.desc(64 * c, 64 * c < a.r);
#pragma unroll
        for (int i = 0; i < dma.PER; ++i) dma.load(d, 64 * c, i, lds + c * kTile, wave);
    }

    // C2 fragments: token row0 + r32, ranks 16 s + 8 h .. +7
    const __amdgpu_buffer_rsrc_t rc = rows_rsrc(a.C2s, a.T, row0, a.R, c0, 2);
    u32x4 av[4 * NC];
#pragma unroll
    for (int s = 0; s < 4 * NC; ++s) {
        const int k = 16 * s + 8 * h;
        av[s] = __builtin_bit_cast(
            u32x4, __builtin_amdgcn_raw_buffer_load_b128(rc, k < a.r ? (uint32_t)((r32 * a.R + k) * 2) : kOOB, 0, 0));
    }

    // acc[v]: token row0 + 8(v/4) + 4h + v%4, column n of the group
    const int n = n0 + 32 * wave + r32, col = g * a.dog + n;
    const uint32_t vo = n < a.dog ? (uint32_t)(((4 * h) * a.dout + col) * 4) : kOOB;
    const float bias = (a.b != nullptr && n < a.dog) ? a.b[col] : 0.f;
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    constexpr int kBatch = 4;
    for (int s0 = 0; s0 < a.S; s0 += kBatch) {
        float x[kBatch][16];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const bool live = s0 + i < a.S;
            const __amdgpu_buffer_rsrc_t rp =
                make_rsrc(reinterpret_cast<const char*>(a.P + (live ? (s0 + i) * a.pstride : 0) +
                                                        (int64_t)row0 * a.dout),
                          live ? (int64_t)(a.T - row0) * a.dout * 4 : 0);
#pragma unroll
            for (int v = 0; v < 16; ++v)
                x[i][v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                    rp, vo, (uint32_t)((8 * (v >> 2) + (v & 3)) * a.dout * 4), 0));
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] += x[i][v];
    }

    wait_vmcnt<0>();
    __syncthreads();
    const TileFrag<false, kFinCols, 1> fb(32 * wave, lane);
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int s = 0; s < 4; ++s) mma32<uint16_t>(acc, av[4 * c + s], fb.read(lds + c * kTile, 0, s));

    const __amdgpu_buffer_rsrc_t ry = make_rsrc(reinterpret_cast<const char*>(a.y + (int64_t)row0 * a.dout),
                                                (int64_t)(a.T - row0) * a.dout * 2);
    const uint32_t vy = n < a.dog ? (uint32_t)(((4 * h) * a.dout + col) * 2) : kOOB;
#pragma unroll
    for (int v = 0; v < 16; ++v)
        __builtin_amdgcn_raw_buffer_store_b16((uint16_t)f2bf(acc[v] + bias), ry, vy,
                                              (uint32_t)((8 * (v >> 2) + (v & 3)) * a.dout * 2), kStoreNT);
}

}  // namespace noble
