// The last launch of a forward whose x W was computed as float32 partial sums
// over K pieces:
//   y[t][n] = sum over s < S of P[s][t][n]  +  C2[t] W_up[:, n]  +  b[n].
//
// Such a forward runs x W and x W_down in one split-K launch (neither needs
// the branch), then the chain, then this kernel: a layer of few tokens has
// too few output tiles to keep 256 CUs reading W, and its K loop is split
// over the idle ones.  Bound by bytes (S T d_out 4 of partials, which the
// products store non-temporal, as they do y and dx) and, for a few tokens, by
// the latency of one round trip: the loads of four partials are issued before
// any is waited for.  32 tokens x 128 columns per workgroup, one 32 x 32 block
// per wave; W_up's [r][128] tile goes through LDS (transposing reads), C2's
// fragments straight to registers.
#pragma once

#include "noble_gemm_tile.hpp"
#include "noble_skinny.hpp"

namespace noble {

constexpr int kFinRows = 32, kFinCols = 128;
constexpr int kFinTile = 64 * kFinCols * 2;   // LDS bytes of 64 rows of W_up

struct FinishArgs {
    const float* P;       // partials [S][T][dout]
    int64_t pstride;      // T * dout
    const uint16_t* C2s;  // [T][R]
    const uint16_t* Wu;   // [G r][dog]
    const float* b;       // [dout] or NULL
    uint16_t* y;          // [T][dout]
    int T, S, G, r, R, dog, dout, pad_;
};

// W_up[:, n0 ..] of group g into LDS, [64 NC][128 columns].
template <int NC>
__device__ __forceinline__ void finish_dma(const FinishArgs& a, int c0, int n0, char* lds, int wave, int lane) {
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
        for (int i = 0; i < dma.PER; ++i) dma.load(d, 64 * c, i, lds + c * kFinTile, wave);
    }
}

// acc[v] = the sum of the partials of token row0 + 8(v/4) + 4h + v%4, column
// col (valid: ok), as sum_partials.
__device__ __forceinline__ void finish_sum(const FinishArgs& a, int row0, int col, bool ok, int h, f32x16& acc) {
    const uint32_t vo = ok ? (uint32_t)(((4 * h) * a.dout + col) * 4) : kOOB;
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
}

__device__ __forceinline__ void finish_store(const FinishArgs& a, int row0, int col, bool ok, int h, float bias,
                                             const f32x16& acc) {
    const __amdgpu_buffer_rsrc_t ry = make_rsrc(reinterpret_cast<const char*>(a.y + (int64_t)row0 * a.dout),
                                                (int64_t)(a.T - row0) * a.dout * 2);
    const uint32_t vy = ok ? (uint32_t)(((4 * h) * a.dout + col) * 2) : kOOB;
#pragma unroll
    for (int v = 0; v < 16; ++v)
        __builtin_amdgcn_raw_buffer_store_b16((uint16_t)f2bf(acc[v] + bias), ry, vy,
                                              (uint32_t)((8 * (v >> 2) + (v & 3)) * a.dout * 2), kStoreNT);
}

// Workgroup position: 32 tokens x 128 columns of one group.
struct FinishPos {
    int row0, g, n0;
};
__device__ __forceinline__ FinishPos finish_pos(const FinishArgs& a) {
    const int tiles_n = (a.dog + kFinCols - 1) / kFinCols, per = a.G * tiles_n;
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const int rb = uni((int)blockIdx.x / per), rem = (int)blockIdx.x - rb * per;
    const int g = uni(rem / tiles_n);
    return FinishPos{rb * kFinRows, g, (rem - g * tiles_n) * kFinCols};
}

// NC: 64-row chunks of W_up (r <= 64 NC).
template <int NC>
__global__ __launch_bounds__(256) void y_finish_kernel(FinishArgs a) {
    __shared__ __attribute__((aligned(1024))) char lds[NC * kFinTile];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    const FinishPos q = finish_pos(a);
    const int c0 = q.g * a.r;
    finish_dma<NC>(a, c0, q.n0, lds, wave, lane);

    // C2 fragments: token row0 + r32, ranks 16 s + 8 h .. +7
    const __amdgpu_buffer_rsrc_t rc = rows_rsrc(a.C2s, a.T, q.row0, a.R, c0, 2);
    u32x4 av[4 * NC];
#pragma unroll
    for (int s = 0; s < 4 * NC; ++s) {
        const int k = 16 * s + 8 * h;
        av[s] = __builtin_bit_cast(
            u32x4, __builtin_amdgcn_raw_buffer_load_b128(rc, k < a.r ? (uint32_t)((r32 * a.R + k) * 2) : kOOB, 0, 0));
    }

    const int n = q.n0 + 32 * wave + r32, col = q.g * a.dog + n;
    const bool ok = n < a.dog;
    const float bias = (a.b != nullptr && ok) ? a.b[col] : 0.f;
    f32x16 acc;
    finish_sum(a, q.row0, col, ok, h, acc);

    wait_vmcnt<0>();
    __syncthreads();
    const TileFrag<false, kFinCols, 1> fb(32 * wave, lane);
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int s = 0; s < 4; ++s) mma32<uint16_t>(acc, av[4 * c + s], fb.read(lds + c * kFinTile, 0, s));
    finish_store(a, q.row0, col, ok, h, bias, acc);
}

// The chain and the finish in one launch, for r <= 128 and few enough
// workgroups that all of them run at once: each computes the chain of its 32
// tokens and group (a copy per 128 columns), keeps C2 in LDS and adds C2 W_up.
// Both kernels are latency-bound there (5.4 and 4.5 us at one token), and the
// chain's loads, the partials of y and W_up arrive in the same round trip.
struct ChainFinishArgs {
    BranchArgs c;
    FinishArgs f;
};
template <Act F, int L>
__global__ __launch_bounds__(256) void chain_finish_kernel(ChainFinishArgs args) {
    constexpr int NW = 4, NC = 2;
    using S = SkShape<NW>;
    __shared__ __attribute__((aligned(1024))) char lds[S::lds(L) + NC * kFinTile];
    const BranchArgs& a = args.c;
    const FinishArgs& f = args.f;
    char* mt = lds + NC * kFinTile;
    char* mt2 = mt + S::MT;   // 3-layer form
    char* chi = mt + (L == 3 ? 2 : 1) * S::MT;
    char* clo = chi + S::CT;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5, r = a.r, R = a.R;
    const FinishPos fp = finish_pos(f);
    const ChainPos q{fp.row0, fp.g, fp.g * r};

    if constexpr (L >= 2) m_dma<NW>(a.M + (int64_t)q.g * r * r, r, mt, wave, lane);
    if constexpr (L == 3) m_dma<NW>(a.M2 + (int64_t)q.g * r * r, r, mt2, wave, lane);
    finish_dma<NC>(f, q.c0, fp.n0, lds, wave, lane);
    const int rcol = 32 * wave + r32;   // rank column of the chain
    const bool cv = rcol < r;
    const ChainVec w = chain_vec<L>(a, q, rcol);
    const int n = fp.n0 + 32 * wave + r32, col = q.g * f.dog + n;   // column of y
    const bool ok = n < f.dog;
    const float bias = (f.b != nullptr && ok) ? f.b[col] : 0.f;
    f32x16 hv, acc;
    sum_partials(a, q.row0, q.c0, rcol, h, hv);
    finish_sum(f, q.row0, col, ok, h, acc);

    // H is the same in every workgroup of the group: the first one stores it
    const __amdgpu_buffer_rsrc_t rh = group_rsrc(a.H, a, q, 4);
    const uint32_t vo4 = cv ? (uint32_t)(((4 * h) * R + rcol) * 4) : kOOB;
    auto store_h = [&]() {
        if (a.H != nullptr && fp.n0 == 0)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(hv[v]), rh, vo4,
                                                      (uint32_t)((8 * (v >> 2) + (v & 3)) * R * 4), kStoreNT);
    };
    float c[16];
    chain_fwd<F, L, NW>(hv, w, cv, chi, clo, mt, mt2, wave, lane, rcol, store_h, c);

    // C2 as the next product's operand (the mixing left the tile free)
#pragma unroll
    for (int v = 0; v < 16; ++v)
        *reinterpret_cast<uint16_t*>(chi + ctile_off(8 * (v >> 2) + 4 * h + (v & 3), rcol)) = (uint16_t)f2bf(c[v]);
    wait_vmcnt<0>();   // W_up (the mixing forms have waited already)
    __syncthreads();
    const TileFrag<false, kFinCols, 1> fb(32 * wave, lane);
#pragma unroll
    for (int k = 0; k < NC; ++k)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const u32x4 av = *reinterpret_cast<const u32x4*>(
                chi + k * 4096 + r32 * 128 + (((2 * s + h) ^ (r32 & 7) ^ (r32 >> 3)) << 4));
            mma32<uint16_t>(acc, av, fb.read(lds + k * kFinTile, 0, s));
        }
    finish_store(f, q.row0, col, ok, h, bias, acc);
}

}  // namespace noble
