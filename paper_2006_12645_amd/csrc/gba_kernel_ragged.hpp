// gba_kernel_ragged.hpp -- the fused fp16 GEMM + bias + activation for large
// requests that the fast path cannot take (odd sizes, odd leading
// dimensions, 2-byte alignment) on gfx950: M >= BM, N >= BN and, for every
// product that is not empty, K >= 64 (with fp16 accumulation a multiple of
// 32).
//
// The step structure is the 16x16x32 fast path's (gba_kernel16.hpp): a
// BM x BN block tile, 64-deep steps over two LDS stages, one barrier per
// step, four slices of MFMAs with the next slice's fragment reads under
// them, the same LDS layouts.  What differs is the copy: its direct
// global -> LDS loads need 16-byte alignment, so here every 16-byte chunk
// goes through a register, loaded at 2-byte alignment (one instruction on
// gfx950) a whole step before it is written to LDS, which also is where the
// prologue's ReLU is applied.
//
// Edges.  Edge tiles are shifted inside the matrix, as on the fast path.  A
// product whose K is no multiple of 64 has its last step start at K - 64:
// every load stays whole and inside the matrix, and the k that the step
// before has already multiplied are cleared in the registers of both
// operands.
#pragma once

#include "gba_kernel_generic.hpp"
#include "gba_kernel16.hpp"
#include "gba_kernel_thin.hpp"

namespace gba {

// A register-staged copy of an operand tile of R rows contiguous along k
// (LDS as in DmaCopy): instruction i of wave w moves rows 8 (NW i + w) .. + 7.
// Instructions whose rows differ by a multiple of the chunk permutation's
// period share a lane offset; the rest of the address is uniform.
template <int R, int NT, int SW>
struct StageK {
    static constexpr int NW = NT / 64, NI = R / (8 * NW);
    static constexpr int PER = SW == 2 ? 64 : 16;
    static constexpr int NV = (8 * NW) % PER == 0 ? 1 : PER / (8 * NW);
    static_assert(R % (8 * NW) == 0, "rows must divide evenly among the waves");
    unsigned off[NV];
    int chunk[NV];   // k / 8 of the lane's chunk
    int lds0;        // byte offset of instruction 0's chunk in the tile
    int64_t ldb;

    __device__ __forceinline__ void init(int64_t ld, int tid)
    {
        ldb = 2 * ld;
        const int w = tid >> 6, l = tid & 63;
        lds0 = 1024 * w + 16 * l;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            chunk[v] = (l & 7) ^ swz_sel<SW>(8 * (NW * v + w) + (l >> 3));
            off[v] = (unsigned)(8 * w + (l >> 3)) * (unsigned)ldb + 16u * chunk[v];
        }
    }
    __device__ __forceinline__ void load(const _Float16 *tile, int k0, i4 (&r)[NI]) const
    {
        const char *b = reinterpret_cast<const char *>(tile + k0);
#pragma unroll
        for (int i = 0; i < NI; ++i)
            r[i] = __builtin_bit_cast(i4, *reinterpret_cast<const h8u *>(b + (8 * NW * i) * ldb + off[i % NV]));
    }
    // clear the k below z
    __device__ __forceinline__ void clear(i4 (&r)[NI], int z) const
    {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int k = 8 * chunk[i % NV] + 2 * d;
                r[i][d] &= (k >= z ? 0xffff : 0) | (k + 1 >= z ? 0xffff0000 : 0);
            }
    }
};

// 16-element group permutation of reduction row k of a tile contiguous along
// M or N with R elements per row: a fragment read's half-wave touches one
// group of rows k0 + {0..3, 8..11}.
template <int R>
__device__ __forceinline__ int fragT(int k)
{
    if constexpr (R >= 128) return fT16(k);
    else return fthin<4>(k);
}

// The same for an operand contiguous along M or N (LDS as in DmaCopyT).
template <int R, int NT>
struct StageN {
    static constexpr int NW = NT / 64, CPR = R / 8, RPI = 1024 / (2 * R), NI = 64 / (RPI * NW);
    static_assert(R == 64 || R == 128 || R == 256, "rows of 64, 128 or 256 elements");
    static_assert(64 % (RPI * NW) == 0, "rows must divide evenly among the waves");
    static_assert((RPI * NW) % 16 == 0, "instructions share the group permutation");
    unsigned off;
    int row0;        // reduction row of instruction 0's chunk
    int lds0;
    int64_t ldb;

    __device__ __forceinline__ void init(int64_t ld, int tid)
    {
        ldb = 2 * ld;
        const int w = tid >> 6, l = tid & 63, p = l % CPR;
        lds0 = 1024 * w + 16 * l;
        row0 = RPI * w + l / CPR;
        off = (unsigned)row0 * (unsigned)ldb + 2u * (16 * ((p >> 1) ^ fragT<R>(row0)) + 8 * (p & 1));
    }
    __device__ __forceinline__ void load(const _Float16 *tile, int k0, i4 (&r)[NI]) const
    {
        const char *b = reinterpret_cast<const char *>(tile) + k0 * ldb;
#pragma unroll
        for (int i = 0; i < NI; ++i)
            r[i] = __builtin_bit_cast(i4, *reinterpret_cast<const h8u *>(b + (RPI * NW * i) * ldb + off));
    }
    __device__ __forceinline__ void clear(i4 (&r)[NI], int z) const
    {
#pragma unroll
        for (int i = 0; i < NI; ++i)
            if (row0 + RPI * NW * i < z) r[i] = i4{0, 0, 0, 0};
    }
};

template <int BM, int BN, int WM, int WN, int LA, int LB, bool ACC16>
__global__ void __launch_bounds__(64 * WM * WN, BM * BN == 128 * 128 ? 4 : 2) gemm_bias_act_ragged(GemmArgs p)
{
    constexpr int NT = 64 * WM * WN, BK = 64;
    constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 16, TN = WTN / 16, TMH = TM / 2;
    constexpr bool TA = LA == COL, TB = LB == ROW;
    constexpr int G = TB ? 1 : (TN < 4 ? TN : 4);   // B blocks per group of consecutive outputs
    constexpr int ROWB = BK * 2, STAGE = (BM + BN) * ROWB;
    using CopyA = std::conditional_t<TA, StageN<BM, NT>, StageK<BM, NT, 1>>;
    using CopyB = std::conditional_t<TB, StageN<BN, NT>, StageK<BN, NT, 2>>;
    static_assert(TN % G == 0 && TM % 2 == 0, "whole groups and halves");
    __shared__ __attribute__((aligned(16))) char lds[2 * STAGE];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WM, wn = wave / WM;
    const int l16 = lane & 15, g4 = lane >> 4;
    int tm, tn;
    tile_coords(blockIdx.x, gridDim.x, p.tiles_m, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int mc = m0 + BM <= p.M ? m0 : p.M - BM;
    const int nc = n0 + BN <= p.N ? n0 : p.N - BN;

    // Fragment byte offsets inside a stage (as in gba_kernel16.hpp); the
    // second 32-deep half of a 128-byte row is the first's with bit 6 flipped.
    int offa[TA ? TM : 1], offb[TN];
    {
        const int kr = 8 * g4 + (l16 >> 2), c4 = 4 * (l16 & 3);
        if constexpr (TA) {
#pragma unroll
            for (int s = 0; s < TM; ++s)
                offa[s] = kr * (2 * BM) + 32 * (((wm * WTM) / 16 + s) ^ fragT<BM>(kr)) + 2 * c4;
        } else {
            offa[0] = (wm * WTM + l16) * ROWB + ((g4 ^ swzA16(l16)) * 16);
        }
#pragma unroll
        for (int t = 0; t < TN; ++t) {
            if constexpr (TB) {
                offb[t] = BM * ROWB + kr * (2 * BN) + 32 * (((wn * WTN) / 16 + t) ^ fragT<BN>(kr)) + 2 * c4;
            } else {
                const int rb = wn * WTN + perm16<G>(t, l16);
                offb[t] = (BM + rb) * ROWB + ((g4 ^ swzB16(rb)) * 16);
            }
        }
    }

    f4 acc[TN][TM];
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int s = 0; s < TM; ++s) acc[t][s] = f4{0.f, 0.f, 0.f, 0.f};
    auto negate_acc = [&]() {
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int s = 0; s < TM; ++s) acc[t][s] = -acc[t][s];
    };
    auto round16 = [&]() {
        if constexpr (ACC16) {
#pragma unroll
            for (int t = 0; t < TN; ++t)
#pragma unroll
                for (int s = 0; s < TM; ++s)
#pragma unroll
                    for (int e = 0; e < 4; e += 2) {
                        const f2v r = round_f16x2(f2v{acc[t][s][e], acc[t][s][e + 1]});
                        acc[t][s][e] = r[0];
                        acc[t][s][e + 1] = r[1];
                    }
        }
    };

    h8 fa[2][TMH], fb[2][TN];
    auto read_a = [&](int buf, const char *stage, int h, int q) {
#pragma unroll
        for (int s = 0; s < TMH; ++s) {
            if constexpr (TA) fa[buf][s] = read_frag_tr<BM>(stage + offa[q * TMH + s] + h * 32 * (2 * BM));
            else fa[buf][s] = *reinterpret_cast<const h8 *>(stage + (offa[0] ^ (64 * h)) + (q * TMH + s) * 16 * ROWB);
        }
    };
    auto read_b = [&](int buf, const char *stage, int h) {
#pragma unroll
        for (int t = 0; t < TN; ++t) {
            if constexpr (TB) fb[buf][t] = read_frag_tr<BN>(stage + offb[t] + h * 32 * (2 * BN));
            else fb[buf][t] = *reinterpret_cast<const h8 *>(stage + (offb[t] ^ (64 * h)));
        }
    };
    auto mfmas = [&](int abuf, int bbuf, int q) {
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int s = 0; s < TMH; ++s)
                acc[t][q * TMH + s] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[bbuf][t], fa[abuf][s],
                                                                             acc[t][q * TMH + s], 0, 0, 0);
    };

    constexpr int NM = TN * TMH;
    constexpr int NRA = TMH * (TA ? 2 : 1), NRB = NRA + TN * (TB ? 2 : 1);
    constexpr int NC = CopyA::NI + CopyB::NI;   // chunks per thread and step
    // Register sets.  A step of the 64x64 tile is shorter than a memory
    // latency, so it has two (1023^3 RC 10.5 -> 9.7 us; four: 10.8, and a
    // slower start-up: 71 x 71 x 125 4.4 -> 5.0).  The larger tiles have
    // registers for one only: refilled right after it was written to LDS, or
    // (256x256) spread over the two slices after that, since at 2-byte
    // alignment a load takes the address unit up to three times as long as
    // an aligned one (4095^3 RC 177 us in one slice, 139 in two, eight
    // launches at a time; under a sustained load 163).  That tile's sums and
    // copies need a few registers more than there are: in RC they spill
    // outside the loop, in CC two of them in every step.
    constexpr int D = BM * BN <= 64 * 64 ? 2 : 1;
    constexpr bool LATE_B = BM * BN > 128 * 128;
    // The prologue's ReLU as a signed 16-bit max (with the smallest value
    // when there is none).
    const short floor16 = p.pro ? 0 : (short)-32768;
    const s8 floor8 = {floor16, floor16, floor16, floor16, floor16, floor16, floor16, floor16};

#pragma unroll 1
    for (int seg = 0; seg < 2; ++seg) {
        const int K = seg == 0 ? p.K : p.K2;
        if (seg == 1 && p.sub) negate_acc();
        if (K > 0) {
            const _Float16 *X = seg == 0 ? p.A : p.P, *Y = seg == 0 ? p.B : p.Q;
            const int64_t ldx = seg == 0 ? p.lda : p.ldp, ldy = seg == 0 ? p.ldb : p.ldq;
            X += TA ? (int64_t)mc : (int64_t)mc * ldx;
            Y += TB ? (int64_t)nc : (int64_t)nc * ldy;
            CopyA ca;
            CopyB cb;
            ca.init(ldx, tid);
            cb.init(ldy, tid);
            const int nk = (K + BK - 1) / BK;
            const int z = nk * BK - K;   // k of the last step that the one before has

            // D register sets: step s is loaded into set s % D, D steps
            // before it is written to LDS, which is in the third slice of
            // step s - 1.
            i4 ra[D][CopyA::NI], rb[D][CopyB::NI];
            auto load_a = [&](int d, int s) { ca.load(X, s < nk - 1 ? s * BK : K - BK, ra[d]); };
            auto load_b = [&](int d, int s) { cb.load(Y, s < nk - 1 ? s * BK : K - BK, rb[d]); };
            auto clear = [&](int d, int s) {
                if (z > 0 && s == nk - 1) {
                    ca.clear(ra[d], z);
                    cb.clear(rb[d], z);
                }
            };
            auto store = [&](int d, char *stage) {
#pragma unroll
                for (int i = 0; i < CopyA::NI; ++i)
                    *reinterpret_cast<i4 *>(stage + ca.lds0 + 1024 * CopyA::NW * i) = __builtin_bit_cast(
                        i4, (s8)__builtin_elementwise_max(__builtin_bit_cast(s8, ra[d][i]), floor8));
#pragma unroll
                for (int i = 0; i < CopyB::NI; ++i)
                    *reinterpret_cast<i4 *>(stage + BM * ROWB + cb.lds0 + 1024 * CopyB::NW * i) = rb[d][i];
            };

            if (seg == 1) __syncthreads();   // the first product's stages are read
#pragma unroll
            for (int d = 0; d < D; ++d) {
                load_a(d, d);
                load_b(d, d);
            }
            clear(0, 0);
            store(0, lds);
            if (D < nk) {
                load_a(0, D);
                if constexpr (!LATE_B) load_b(0, D);
            }
            wait_vm_lgkm0<63>();
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            read_a(0, lds, 0, 0);
            read_b(0, lds, 0);

            // One step; d: the set that holds step kt+1 and is refilled with
            // step kt+1+D.  Without FILL no step is left to load.
            auto step = [&](auto fill, int kt, int d) {
                constexpr bool FILL = decltype(fill)::value;
                char *cur = lds + (kt & 1) * STAGE, *nxt = lds + ((kt + 1) & 1) * STAGE;
                // slice 0: half 0, first A blocks
                read_a(1, cur, 0, 1);
                if constexpr (LATE_B) {
                    if (FILL || kt + D < nk) load_b(d, kt + D);
                }
                mfmas(0, 0, 0);
                sched_slice<NM, NRA, 0x020, LATE_B ? CopyB::NI : 0, false>();
                // slice 1: half 0, second A blocks (B fragments of half 1 in flight)
                read_a(0, cur, 1, 0);
                read_b(1, cur, 1);
                mfmas(1, 0, 1);
                round16();
                sched_slice<NM, NRB, 0, 0, false>();
                __builtin_amdgcn_sched_barrier(0);
                clear(d, kt + 1);
                // slice 2: half 1, first A blocks, step kt+1 into its stage
                // (and the loads of step kt+1+D)
                read_a(1, cur, 1, 1);
                store(d, nxt);
                if constexpr (FILL && !LATE_B) {
                    load_a(d, kt + 1 + D);
                    load_b(d, kt + 1 + D);
                }
                mfmas(0, 1, 0);
                if constexpr (LATE_B || !FILL) sched_slice<NM, NRA, 0x200, NC, false>();
                else sched_slice2<NM, NRA, 0x200, NC, 0x020, NC>();
                __builtin_amdgcn_sched_barrier(0);
                wait_vm_lgkm0<63>();
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_sched_barrier(0);
                // slice 3: half 1, second A blocks, the first fragments of step kt+1
                read_a(0, nxt, 0, 0);
                read_b(0, nxt, 0);
                if constexpr (FILL && LATE_B) load_a(d, kt + 1 + D);
                mfmas(1, 1, 1);
                round16();
                sched_slice<NM, NRB, 0x020, FILL && LATE_B ? CopyA::NI : 0, false>();
            };
            int kt = 0;
#pragma unroll 1
            for (; kt + 2 * D < nk; kt += D) {
#pragma unroll
                for (int d = 0; d < D; ++d) step(std::true_type{}, kt + d, (d + 1) % D);
            }
            // The last 2 D steps or fewer.
#pragma unroll
            for (int i = 0; i < 2 * D; ++i) {
                if (kt + i >= nk) break;
                if (i < D - 1 && kt + i + 1 + D < nk) step(std::true_type{}, kt + i, (i + 1) % D);
                else step(std::false_type{}, kt + i, (i + 1) % D);
            }
        }
        if (seg == 1 && p.sub) negate_acc();
    }

    // Epilogue on registers: a lane holds, per A block and group of G B
    // blocks, 4 G consecutive outputs of one row, stored W at a time at any
    // alignment; outputs shared with a neighbouring tile are stored by their
    // owner only.
    constexpr int NGRP = TN / G, W = G >= 2 ? 8 : 4, NV = 4 * G / W;
    typedef std::conditional_t<W == 8, h8u, h4u> run;
    const int j0 = nc + wn * WTN + 4 * G * g4;   // column of group 0's first output
    run brow[NGRP][NV];
    if (p.bias_kind == BIAS_ROW) {
#pragma unroll
        for (int tg = 0; tg < NGRP; ++tg)
#pragma unroll
            for (int v = 0; v < NV; ++v)
                brow[tg][v] = *reinterpret_cast<const run *>(p.bias + j0 + 16 * G * tg + W * v);
    }
#pragma unroll
    for (int s = 0; s < TM; ++s) {
        const int i = mc + wm * WTM + 16 * s + l16;
        const _Float16 *const bfull = p.bias + (int64_t)i * p.ldbias + j0;
        _Float16 *const row = p.C + (int64_t)i * p.ldc + j0;
#pragma unroll
        for (int tg = 0; tg < NGRP; ++tg) {
            float x[4 * G];
#pragma unroll
            for (int e = 0; e < 4 * G; ++e) x[e] = acc[tg * G + e / 4][s][e % 4];
            if (p.bias_kind == BIAS_ROW) {
#pragma unroll
                for (int e = 0; e < 4 * G; ++e) x[e] += p.bias_sign * (float)brow[tg][e / W][e % W];
            } else if (p.bias_kind == BIAS_FULL) {
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const run b = *reinterpret_cast<const run *>(bfull + 16 * G * tg + W * v);
#pragma unroll
                    for (int e = 0; e < W; ++e) x[W * v + e] += p.bias_sign * (float)b[e];
                }
            }
            activate(p.act, x);
            if (i < m0) continue;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                run o;
#pragma unroll
                for (int e = 0; e < W; ++e) o[e] = (_Float16)x[W * v + e];
                _Float16 *dst = row + 16 * G * tg + W * v;
                const int j = j0 + 16 * G * tg + W * v;
                if (nc == n0 || j >= n0) {
                    *reinterpret_cast<run *>(dst) = o;
                } else if (j + W > n0) {
#pragma unroll
                    for (int e = 0; e < W; ++e)
                        if (j + e >= n0) dst[e] = o[e];
                }
            }
        }
    }
}

}  // namespace gba
