// bf16 grouped MFMA GEMM for gfx950 with a pinned instruction schedule.
//
// Waves of 32 TM x 32 TN outputs (32 x 32 x 16 MFMAs) in a WM x WN grid;
// operands go straight to LDS with buffer_load ... lds and keep their HBM
// orientation:
//  - K-major tiles: [rows][128 B], 16-byte chunk c of row q at physical chunk
//    c ^ ((q ^ q/8) & 7); fragments with ds_read_b128.
//  - MN-major tiles: [64 k][2 W bytes], W columns; the 64-byte block (32
//    columns) w of k-row k sits at w ^ (k & 3) (w ^ ((k >> 1) & 1) for
//    W = 64), so that the four k-rows a transposing read touches fall in
//    different banks; fragments with two ds_read_b64_tr_b16.
#pragma once

#include "noble_gemm_dma.hpp"

namespace noble {

// Direct-to-LDS loads of one W-row (K-major) or W-column (MN-major) operand
// tile, one 64-element K chunk at a time, shared by NW waves.  The per-lane
// offsets are set up once per K segment; a chunk only needs its descriptor.
template <bool KMAJ, int W, int NW>
struct TileDma {
    static constexpr int ES = 2;
    static constexpr int PER = W / 8 / NW;                       // 1 KB instructions per wave per chunk
    static constexpr int NV = KMAJ ? (NW == 4 && PER > 1 ? 2 : 1) : 1;   // distinct lane offsets
    static_assert(W % (8 * NW) == 0, "whole instructions per wave");
    uint32_t vo[NV];
    int kq[NV];          // K-major: first k of the lane's 16 bytes within the chunk
    uint32_t sstep;      // byte step of one instruction
    const char* base;    // segment base at the tile's first row / column
    int64_t bytes;       // bytes from base to the end of the operand
    int64_t ld;
    int klen;

    __device__ __forceinline__ void segment(const Seg& s, int rows, int row0, int wave, int lane) {
        ld = s.ld;
        klen = s.klen;
        if constexpr (KMAJ) {
            // block b = NW i + wave holds rows 8b .. 8b+7; lane p -> row
            // 8b + p/8, physical chunk p%8 = logical (p%8) ^ (p/8) ^ (b & 7)
            const int rr = lane >> 3;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                kq[v] = ((lane & 7) ^ rr ^ ((NW * v + wave) & 7)) * 8;
                vo[v] = (uint32_t)(((int64_t)rr * ld + kq[v]) * ES);
            }
            base = s.ptr + (int64_t)row0 * ld * ES;
            bytes = (int64_t)(rows - row0) * ld * ES;
            sstep = (uint32_t)(8 * ld * ES);
        } else {
            // block b holds KR k-rows; lane p -> k-row KR b + p/SEG, physical
            // 16-byte segment p%SEG
            constexpr int SEG = W / 8 < 64 ? W / 8 : 64, KR = 64 / SEG;
            const int kr = lane / SEG;
            // k & 3 (or (k >> 1) & 1) of the lane's row: KR b + kr
            const int k = KR * wave + kr;   // NW KR is a multiple of 4: the same for every i
            static_assert((NW * KR) % 4 == 0, "the swizzle repeats over a wave's instructions");
            const int swz = W == 64 ? ((k >> 1) & 1) : (k & 3);
            const int col = row0 + 8 * ((lane % SEG) ^ (4 * swz));
            vo[0] = col < rows ? (uint32_t)(((int64_t)kr * ld + col) * ES) : kOOB;
            kq[0] = 0;
            base = s.ptr;
            bytes = (int64_t)klen * ld * ES;
            sstep = (uint32_t)(KR * ld * ES);
        }
    }
    // Descriptor of the chunk starting at k0 (relative to the segment);
    // live = false: an empty one (its loads store zeros, no memory access).
    __device__ __forceinline__ i32x4 desc(int k0, bool live) const {
        const int64_t off = KMAJ ? (int64_t)k0 * ES : (int64_t)k0 * ld * ES;
        return make_desc(base + (live ? off : 0), live ? bytes - off : 0);
    }
    // Instruction i of this wave.
    __device__ __forceinline__ void load(const i32x4& d, int k0, int i, char* dst, int wave) const {
        const int b = NW * i + wave;
        uint32_t v = vo[NV == 1 ? 0 : i & 1];
        if constexpr (KMAJ) v = k0 + kq[NV == 1 ? 0 : i & 1] < klen ? v : kOOB;
        dma16(d, dst + b * 1024, v, (uint32_t)__builtin_amdgcn_readfirstlane((int)(sstep * (uint32_t)b)));
    }
};

// Fragment reads (32 x 32 x 16) of a wave whose block starts at row / column
// w0 of a W-wide tile (w0 a multiple of 32).
template <bool KMAJ, int W, int T>
struct TileFrag {
    uint32_t base;
    uint32_t off[T];
    __device__ __forceinline__ TileFrag(int w0, int lane) {
        if constexpr (KMAJ) {
            const int r32 = lane & 31, h = lane >> 5;
            base = (uint32_t)(r32 * 128 + ((h ^ (r32 & 7) ^ (r32 >> 3)) << 4));
#pragma unroll
            for (int i = 0; i < T; ++i) off[i] = (uint32_t)((w0 >> 5) + i);
        } else {
            const int g = lane >> 4, j = lane & 15, c = j >> 2;
            const int x = 2 * (g & 1) + ((j & 3) >> 1);
            const int f = W == 64 ? (c >> 1) : c;
            base = (uint32_t)((8 * (g >> 1) + c) * 2 * W + 16 * x + 8 * (j & 1));
#pragma unroll
            for (int i = 0; i < T; ++i) off[i] = (uint32_t)(64 * (((w0 >> 5) + i) ^ f));
        }
    }
    __device__ __forceinline__ u32x4 read(const char* tile, int i, int s) const {
        if constexpr (KMAJ) {
            return *reinterpret_cast<const u32x4*>(
                tile + ((base ^ ((uint32_t)s << 5) ^ ((off[i] & 1) << 6)) + 4096u * off[i]));
        } else {
            const char* p = tile + (base + off[i] + 2u * W * 16 * s);
            const uint64_t lo = ds_read_tr(p);
            const uint64_t hi = ds_read_tr(p + 4 * 2 * W);
            u32x4 v;
            v[0] = (uint32_t)lo;
            v[1] = (uint32_t)(lo >> 32);
            v[2] = (uint32_t)hi;
            v[3] = (uint32_t)(hi >> 32);
            return v;
        }
    }
};

// A K-major, B K-major (BKM) or MN-major; WM x WN waves of 32 TM x 32 TN
// outputs; NST LDS stages of 64-element chunks.
template <bool BKM, int WM, int WN, int TM, int TN, int NST, typename Batch>
__global__ __launch_bounds__(64 * WM * WN, (160 * 1024 / (NST * 32 * (WM * TM + WN * TN) * 128)) * WM * WN / 4)
void gemm_tile_kernel(Batch batch) {
    constexpr int NW = WM * WN, WTM = 32 * TM, WTN = 32 * TN, BM = WM * WTM, BN = WN * WTN;
    constexpr int TA = BM * 128, STAGE = (BM + BN) * 128;
    static_assert(NST >= 3, "the loads of a chunk span two others");
    using DA = TileDma<true, BM, NW>;
    using DB = TileDma<BKM, BN, NW>;
    constexpr int kLoads = DA::PER + DB::PER;
    __shared__ __attribute__((aligned(1024))) char lds[NST * STAGE];

    const int bid = blockIdx.x;
    int q = 0;
#pragma unroll
    for (int t = 1; t < Batch::kMax; ++t)
        if (t < batch.count && bid >= batch.p[t].tile_begin) q = t;
    const GemmProblem& P = batch.p[q];
    int L = bid - P.tile_begin;
    if ((P.nblocks & 7) == 0) L = (L & 7) * (P.nblocks >> 3) + (L >> 3);
    const int ntiles = P.tiles_m * P.tiles_n;
    const int piece = __builtin_amdgcn_readfirstlane(L / ntiles);
    const int tile = L - piece * ntiles;
    constexpr int GM = kGroupM * 256 / BM;
    const int span = GM * P.tiles_n;
    const int grp = tile / span, in = tile - grp * span;
    const int first_m = grp * GM;
    const int gsz = min(P.tiles_m - first_m, GM);
    // Integer divisions run on the vector unit: bring their (uniform) results
    // back to scalars, so that the loads' descriptors and offsets stay scalar.
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const int tm = uni(first_m + in % gsz), tn = uni(in / gsz);
    const int m0 = tm * BM, n0 = tn * BN;
    const int kc0 = uni((int)((int64_t)P.nk * piece / P.split));
    const int kc1 = uni((int)((int64_t)P.nk * (piece + 1) / P.split));
    const int n = kc1 - kc0;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave / WN) * WTM, wn0 = (wave % WN) * WTN;
    const int r32 = lane & 31, h = lane >> 5;

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    if (n > 0) {
        const TileFrag<true, BM, TM> fa(wm0, lane);
        const TileFrag<BKM, BN, TN> fb(wn0, lane);
        const Operand opA = P.A, opB = P.B;
        DA da;
        DB db;
        // Chunk being loaded: its descriptors and K offset.  A and B change
        // segments at the same chunk.
        int k0 = 0;
        i32x4 dsa, dsb;
        auto aim = [&](int i) __attribute__((always_inline)) {   // chunk i of the piece
            const int kc = kc0 + i;
            const bool second = kc >= opA.nk1;
            if (i == 0 || kc == opA.nk1) {
                da.segment(second ? opA.s[1] : opA.s[0], opA.rows, m0, wave, lane);
                db.segment(second ? opB.s[1] : opB.s[0], opB.rows, n0, wave, lane);
            }
            k0 = (second ? kc - opA.nk1 : kc) * 64;
            dsa = da.desc(k0, i < n);
            dsb = db.desc(k0, i < n);
        };
        auto dma = [&](int d, int st) __attribute__((always_inline)) {   // instruction d of kLoads
            char* dst = lds + st * STAGE;
            if (d < DA::PER)
                da.load(dsa, k0, d, dst, wave);
            else
                db.load(dsb, k0, d - DA::PER, dst + TA, wave);
        };
        // Instructions [part_lo(p), part_lo(p + 1)) are part p of a chunk.
        // Part 0 goes out in the last K step of a chunk, parts 1 .. 3 in the
        // first three of the next.
        auto part_lo = [](int p) constexpr { return kLoads * p / 4; };

#pragma unroll
        for (int i = 0; i < NST - 1; ++i) {
            aim(i);
#pragma unroll
            for (int d = 0; d < kLoads; ++d) dma(d, i);
        }
        aim(NST - 1);
#pragma unroll
        for (int d = 0; d < part_lo(1); ++d) dma(d, NST - 1);
        wait_vmcnt<(NST - 2) * kLoads + part_lo(1)>();
        __builtin_amdgcn_s_barrier();

        u32x4 a[2][TM], b[2][TN];
#pragma unroll
        for (int t = 0; t < TM; ++t) a[0][t] = fa.read(lds, t, 0);
#pragma unroll
        for (int t = 0; t < TN; ++t) b[0][t] = fb.read(lds + TA, t, 0);

        int st = 0;   // stage of the chunk being multiplied
        // One K step: MFMAs on fragments cb while the next step's fragments
        // (from stage rs, step s2) and part p of the loads (into stage ds) go out.
        auto step = [&](int cb, int rs, int s2, int p, int ds) __attribute__((always_inline)) {
            constexpr int NM = TM * TN, NR = TM + TN;
            const int nb = cb ^ 1;
            const char* ra = lds + rs * STAGE;
            const char* rb = ra + TA;
            const int d0 = part_lo(p), nd = part_lo(p + 1) - d0;
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                mma32<uint16_t>(acc[m / TN][m % TN], a[cb][m / TN], b[cb][m % TN]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = NR * m / NM; t < NR * (m + 1) / NM; ++t) {
                    if (t < TN)
                        b[nb][t] = fb.read(rb, t, s2);
                    else
                        a[nb][t - TN] = fa.read(ra, t - TN, s2);
                }
#pragma unroll
                for (int d = nd * m / NM; d < nd * (m + 1) / NM; ++d) dma(d0 + d, ds);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto chunk = [&](int i) __attribute__((always_inline)) {
            const int prv = st == 0 ? NST - 1 : st - 1, nxt = st + 1 == NST ? 0 : st + 1;
            step(0, st, 1, 1, prv);
            step(1, st, 2, 2, prv);
            step(0, st, 3, 3, prv);
            // Chunk i + 1 has landed once only the later chunks' loads are
            // outstanding; this wave's reads of chunk i are done (lgkmcnt).
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt((((NST - 2) * kLoads) & 15) | ((((NST - 2) * kLoads) >> 4) << 14) | (7 << 4));
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            aim(i + NST);
            step(1, nxt, 0, 0, st);
            st = nxt;
        };
        // A function of its bounds: with the loop written out here, the compiler
        // computes the offsets of the loads of a K-major B in vector registers.
        auto run = [&](int lo, int hi) __attribute__((always_inline)) {
            for (int i = lo; i < hi; ++i) chunk(i);
        };
        run(0, n);
        wait_vmcnt<0>();   // no load may reach LDS after the workgroup's end
    }

    const bool add_bias = (P.bias != nullptr) && piece == 0;
    const int es = P.out_f32 ? 4 : 2;
    const __amdgpu_buffer_rsrc_t rc =
        make_rsrc(static_cast<const char*>(P.C) + (piece * P.pstride + (int64_t)m0 * P.ldc) * es,
                  (int64_t)(P.M - m0) * P.ldc * es);
    uint32_t voff[TM][TN];
    float bcol[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int col = n0 + wn0 + 32 * j + r32;
        bcol[j] = (add_bias && col < P.N) ? P.bias[col] : 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i)
            voff[i][j] = col < P.N ? (uint32_t)(((int64_t)(wm0 + 32 * i + 4 * h) * P.ldc + col) * es) : kOOB;
    }
    auto epilogue = [&](auto store) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    store(acc[i][j][v] + bcol[j], voff[i][j],
                          (uint32_t)((int64_t)(8 * (v >> 2) + (v & 3)) * P.ldc * es));
    };
    if (P.out_f32)
        epilogue([&](float val, uint32_t vo, uint32_t so) {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(val), rc, vo, so, kStoreNT);
        });
    else
        epilogue([&](float val, uint32_t vo, uint32_t so) {
            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)f2bf(val), rc, vo, so, kStoreNT);
        });
}

}  // namespace noble
