// float32 grouped MFMA GEMM on 64 x 64 tiles with direct-to-LDS loads.
//
// For launches that gemm_kernel's 128 x 128 tiles would leave CUs idle in (the
// rule is f32_tile's).  Bound by the float32 MFMAs (a chunk is 0.43 us of them
// at full clock) where its tiles fill the CUs, and by the last CU's tiles
// otherwise: hence small tiles, and three LDS stages (48 KB) so that three
// workgroups share a CU.  Against register staging on the same tile, forward /
// backward (us): 2048 x 768 -> 768 62.3 / 101.5 -> 58.7 / 98.8, 64 x 1024 ->
// 1024 63.0 / 68.9 -> 56.2 / 67.8, 2048 x 1024 -> 1024 86.2 / 147.2 -> 82.0 /
// 146.7.
//
// Operands keep their HBM orientation in LDS:
//  - K-major: [64 rows][128 B], 16-byte chunk c of row q at c ^ ((q ^ q/8) & 7);
//    fragments (four k of a row) with ds_read_b128.
//  - MN-major: [32 k][256 B], column n of k-row k at n ^ 32 ((k / 4) & 1);
//    fragments with four ds_read_b32: the two half waves read k-rows four
//    apart, in the two halves of the banks.
#pragma once

#include "noble_gemm_tile.hpp"

namespace noble {

constexpr int kF32Tile = 64, kF32Stages = 3;
constexpr int kF32Op = kF32Tile * 128;   // LDS bytes of one operand tile, either layout

// Loads of one operand tile, one 32-element K chunk at a time: 8 instructions
// of 1 KB shared by four waves.
template <bool KMAJ>
struct F32Dma {
    static constexpr int PER = 2;
    uint32_t vo[PER];
    int kq[PER];
    uint32_t sstep;
    const char* base;
    int64_t bytes, ld;
    int klen;

    __device__ __forceinline__ void segment(const Seg& s, int rows, int row0, int wave, int lane) {
        ld = s.ld;
        klen = s.klen;
        if constexpr (KMAJ) {
            // block b = 4 i + wave holds rows 8b .. 8b+7; lane p -> row 8b + p/8,
            // physical chunk p%8 = logical (p%8) ^ (p/8) ^ (b & 7)
            const int rr = lane >> 3;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                kq[i] = ((lane & 7) ^ rr ^ ((4 * i + wave) & 7)) * 4;
                vo[i] = (uint32_t)(((int64_t)rr * ld + kq[i]) * 4);
            }
            base = s.ptr + (int64_t)row0 * ld * 4;
            bytes = (int64_t)(rows - row0) * ld * 4;
            sstep = (uint32_t)(8 * ld * 4);
        } else {
            // block b holds k-rows 4b .. 4b+3; lane p -> k-row 4b + p/16,
            // physical 16-byte segment p%16 = logical (p%16) ^ 8 (b & 1)
            const int col = row0 + 4 * ((lane & 15) ^ (8 * (wave & 1)));
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                vo[i] = col < rows ? (uint32_t)(((int64_t)(lane >> 4) * ld + col) * 4) : kOOB;
                kq[i] = 0;
            }
            base = s.ptr;
            bytes = (int64_t)klen * ld * 4;
            sstep = (uint32_t)(4 * ld * 4);
        }
    }
    __device__ __forceinline__ void load(int k0, bool live, char* dst, int wave) const {
        const int64_t off = KMAJ ? (int64_t)k0 * 4 : (int64_t)k0 * ld * 4;
        const i32x4 d = make_desc(base + (live ? off : 0), live ? bytes - off : 0);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int b = 4 * i + wave;
            const uint32_t v = KMAJ && k0 + kq[i] >= klen ? kOOB : vo[i];
            dma16(d, dst + b * 1024, v, (uint32_t)__builtin_amdgcn_readfirstlane((int)(sstep * (uint32_t)b)));
        }
    }
};

// Fragment of K step s (8 elements) of the 32 rows / columns from w0.
template <bool KMAJ>
__device__ __forceinline__ u32x4 f32_frag(const char* tile, int w0, int lane, int s) {
    const int r32 = lane & 31, h = lane >> 5;
    if constexpr (KMAJ) {
        return *reinterpret_cast<const u32x4*>(tile + lds_off(w0 + r32, 2 * s + h));
    } else {
        const char* p = tile + (8 * s + 4 * h) * 256 + ((w0 + r32) ^ (32 * h)) * 4;
        u32x4 v;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = *reinterpret_cast<const uint32_t*>(p + 256 * q);
        return v;
    }
}

template <bool AK, bool BKM, bool HAS_BSUM, typename Batch>
__global__ __launch_bounds__(256, 3) void gemm_f32_kernel(Batch batch) {
    constexpr int NST = kF32Stages, STAGE = 2 * kF32Op, kLoads = F32Dma<AK>::PER + F32Dma<BKM>::PER;
    __shared__ __attribute__((aligned(1024))) char lds[NST * STAGE];

    const int bid = blockIdx.x;
    int q = 0;
#pragma unroll
    for (int t = 1; t < Batch::kMax; ++t)
        if (t < batch.count && bid >= batch.p[t].tile_begin) q = t;
    const GemmProblem& P = batch.p[q];
    // XCD-aware order and column groups, as gemm_kernel
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    int L = bid - P.tile_begin;
    if ((P.nblocks & 7) == 0) L = (L & 7) * (P.nblocks >> 3) + (L >> 3);
    const int ntiles = P.tiles_m * P.tiles_n;
    const int piece = uni(L / ntiles), tile = L - piece * ntiles;
    constexpr int GM = 8;
    const int span = GM * P.tiles_n;
    const int grp = tile / span, in = tile - grp * span;
    const int gsz = min(P.tiles_m - grp * GM, GM);
    const int tm = uni(grp * GM + in % gsz), tn = uni(in / gsz);
    const int m0 = tm * kF32Tile, n0 = tn * kF32Tile;
    const int kc0 = uni((int)((int64_t)P.nk * piece / P.split));
    const int kc1 = uni((int)((int64_t)P.nk * (piece + 1) / P.split));
    const int n = kc1 - kc0;

    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const int wm0 = (wave >> 1) * 32, wn0 = (wave & 1) * 32;
    const int r32 = lane & 31, h = lane >> 5;
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    const bool do_bsum = HAS_BSUM && (P.bsum != nullptr) && tm == 0 && wm0 == 0;
    float bs = 0.f;

    if (n > 0) {
        const Operand opA = P.A, opB = P.B;
        F32Dma<AK> da;
        F32Dma<BKM> db;
        // Chunk i of the piece into its stage (past the end: nothing is read).
        // A and B change segments at the same chunk.
        auto load = [&](int i, int st) __attribute__((always_inline)) {
            const int kc = kc0 + i;
            const bool second = kc >= opA.nk1;
            if (i == 0 || kc == opA.nk1) {
                da.segment(second ? opA.s[1] : opA.s[0], opA.rows, m0, wave, lane);
                db.segment(second ? opB.s[1] : opB.s[0], opB.rows, n0, wave, lane);
            }
            const int k0 = (second ? kc - opA.nk1 : kc) * 32;
            da.load(k0, i < n, lds + st * STAGE, wave);
            db.load(k0, i < n, lds + st * STAGE + kF32Op, wave);
        };
#pragma unroll
        for (int i = 0; i < NST - 1; ++i) load(i, i);
        int st = 0;
        for (int i = 0; i < n; ++i) {
            wait_vmcnt<(NST - 2) * kLoads>();   // chunk i has landed
            __syncthreads();                    // for every wave, and all are done with chunk i - 1
            load(i + NST - 1, st == 0 ? NST - 1 : st - 1);
            const char* ta = lds + st * STAGE;
            u32x4 a[4], b[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                a[s] = f32_frag<AK>(ta, wm0, lane, s);
                b[s] = f32_frag<BKM>(ta + kF32Op, wn0, lane, s);
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                mma32<float>(acc, a[s], b[s]);
                if constexpr (HAS_BSUM)
                    if (do_bsum)
#pragma unroll
                        for (int w = 0; w < 4; ++w) bs += __uint_as_float(b[s][w]);
            }
            st = st + 1 == NST ? 0 : st + 1;
        }
        wait_vmcnt<0>();   // no load may reach LDS after the workgroup's end
    }

    if (do_bsum) {
        const float s = bs + __shfl_xor(bs, 32);
        const int col = n0 + wn0 + r32;
        if (h == 0 && col < P.N) unsafeAtomicAdd(P.bsum + col, s);
    }
    // acc[v]: row 8(v/4) + 4h + v%4, column r32 of the wave's block
    const int col = n0 + wn0 + r32;
    const float bias = (P.bias != nullptr && piece == 0 && col < P.N) ? P.bias[col] : 0.f;
    const __amdgpu_buffer_rsrc_t rc =
        make_rsrc(static_cast<const char*>(P.C) + (piece * P.pstride + (int64_t)m0 * P.ldc) * 4,
                  (int64_t)(P.M - m0) * P.ldc * 4);
    const uint32_t vo = col < P.N ? (uint32_t)(((int64_t)(wm0 + 4 * h) * P.ldc + col) * 4) : kOOB;
#pragma unroll
    for (int v = 0; v < 16; ++v)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[v] + bias), rc, vo,
                                              (uint32_t)((int64_t)(8 * (v >> 2) + (v & 3)) * P.ldc * 4), 0);
}

}  // namespace noble
