// gba_kernel_thin.hpp -- the fused fp16 GEMM + bias + activation for a few
// rows (decoding and small inference batches) on gfx950: any leading
// dimension, any K and any (2-byte) alignment, fp32 accumulation.
//
// With a few rows the product is bound by reading B once, and below that by
// latency: the tiled kernels walk K in steps that wait for each other on
// one compute unit per 64 columns.  Here a workgroup owns 16 * TM rows by
// 16 * TN columns, and its up to 16 waves split K between them (the Split-K
// subsection's partition of the reduction inside a thread block).  A wave
// loads its operands' 64-deep slabs into registers D slabs ahead, 16 bytes
// per lane with consecutive lanes along each row, and passes every slab
// through its own corner of LDS to get MFMA fragments; no barrier stands
// between the loads, so most of the panel is in flight after one memory
// latency.  The waves' partial sums meet once in LDS, are added in wave
// order, and the epilogue runs on the sum.
//
// Why through LDS: a fragment's lanes 16 g + c hold chunk g of row c, so a
// fragment loaded straight from memory has consecutive lanes in different
// rows, which the address unit takes at about 16 bytes a clock.
//
// LDS.  An operand contiguous along k (row-major A, column-major B) is kept
// as 16 T rows of 128 bytes, chunk c of row r at c ^ (r % 8); one contiguous
// along N (row-major B) as 64 k rows of 16 T columns, 16-column group t of
// row k at t ^ fthin(k), and read with transposing reads.  Column-major A
// (a few rows: not enough for a 16-byte load) is read element-wise into its
// fragments.
//
// Edges.  Rows of A and columns of a column-major B beyond the matrix are
// read at the last one inside it; a row-major B's last tile is shifted
// inside; neither is stored twice.  The k beyond K of a product's last slab
// are not read and count as zeros.
#pragma once

#include "gba_kernel_generic.hpp"
#include "gba_kernel16.hpp"

namespace gba {

// 16-column group permutation of row k: a transposing read's half-wave
// touches rows k0 + {0..3, 8..11} of one group.
template <int T>
__device__ __forceinline__ int fthin(int k)
{
    if constexpr (T == 2) return (k >> 3) & 1;
    else if constexpr (T == 4) return ((k >> 1) & 1) | (((k >> 3) & 1) << 1);
    else return 0;
}

// A 64-deep slab of an operand contiguous along k: T blocks of 16 rows.
// Instruction i loads rows 8 i .. 8 i + 7, eight lanes (128 bytes) a row.
template <int T>
struct ThinSlabK {
    static constexpr int NI = 2 * T;
    const char *base;   // uniform
    unsigned off[NI];   // lane byte offset of instruction i
    int chunk;          // the lane's 16-byte chunk of its row
    int wr, rd;         // lane byte offsets of the LDS writes and reads

    // first: the tile's first row; ext: rows from it on that exist
    __device__ __forceinline__ void init(const _Float16 *X, int64_t ld, int first, int ext, int lane)
    {
        base = reinterpret_cast<const char *>(X + first * ld);
        chunk = lane & 7;
        const int r0 = lane >> 3;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int r = 8 * i + r0;
            off[i] = (unsigned)(r < ext ? r : ext - 1) * (unsigned)(2 * ld) + 16u * chunk;
        }
        wr = 128 * r0 + 16 * (chunk ^ r0);
        rd = 128 * (lane & 15);
    }
    __device__ __forceinline__ void load(int k0, i4 (&v)[NI]) const
    {
        const char *b = base + 2 * (int64_t)k0;
#pragma unroll
        for (int i = 0; i < NI; ++i) v[i] = __builtin_bit_cast(i4, *reinterpret_cast<const h8u *>(b + off[i]));
    }
    // only n of the 64 k exist
    __device__ __forceinline__ void load_tail(int k0, int n, i4 (&v)[NI]) const
    {
        const char *b = base + 2 * (int64_t)k0;
        const int left = n - 8 * chunk;
#pragma unroll
        for (int i = 0; i < NI; ++i)
            v[i] = __builtin_bit_cast(
                i4, left > 0 ? load8(reinterpret_cast<const _Float16 *>(b + off[i]), left) : zero_h8());
    }
    __device__ __forceinline__ void store(char *lds, const i4 (&v)[NI]) const
    {
#pragma unroll
        for (int i = 0; i < NI; ++i) *reinterpret_cast<i4 *>(lds + wr + 1024 * i) = v[i];
    }
    // fragment of block t for 32-deep half h
    __device__ __forceinline__ h8 frag(const char *lds, int t, int h, int lane) const
    {
        return *reinterpret_cast<const h8 *>(lds + rd + 2048 * t + 16 * ((4 * h + (lane >> 4)) ^ (lane & 7)));
    }
};

// A 64-deep slab of an operand contiguous along N: 64 k rows of 16 T columns.
template <int T>
struct ThinSlabN {
    static constexpr int NI = 2 * T;
    static constexpr int CPR = 2 * T;        // 16-byte chunks per row
    static constexpr int RPI = 64 / CPR;     // rows per instruction
    const char *base;
    int64_t ldb;
    unsigned off;
    int row0, wr[NI], rd[T];

    __device__ __forceinline__ void init(const _Float16 *X, int64_t ld, int first, int, int lane)
    {
        base = reinterpret_cast<const char *>(X + first);
        ldb = 2 * ld;
        row0 = lane / CPR;
        const int chunk = lane % CPR;
        off = (unsigned)row0 * (unsigned)ldb + 16u * chunk;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int k = RPI * i + row0;
            wr[i] = 32 * T * k + 32 * ((chunk >> 1) ^ fthin<T>(k)) + 16 * (chunk & 1);
        }
        // transposing reads: lane 4 j + c of 16-lane group g addresses row
        // 8 g + j at elements 4 c .. 4 c + 3 of the block (the second read
        // of a fragment four rows further: fthin is the same there for T = 2
        // and, with bit 1 of k unchanged, for T = 4)
        const int k = 8 * (lane >> 4) + ((lane & 15) >> 2);
#pragma unroll
        for (int t = 0; t < T; ++t) rd[t] = 32 * T * k + 32 * (t ^ fthin<T>(k)) + 8 * (lane & 3);
    }
    __device__ __forceinline__ void load(int k0, i4 (&v)[NI]) const
    {
        const char *b = base + k0 * ldb;
#pragma unroll
        for (int i = 0; i < NI; ++i)
            v[i] = __builtin_bit_cast(i4, *reinterpret_cast<const h8u *>(b + (RPI * i) * ldb + off));
    }
    __device__ __forceinline__ void load_tail(int k0, int n, i4 (&v)[NI]) const
    {
        const char *b = base + k0 * ldb;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            v[i] = i4{0, 0, 0, 0};
            if (RPI * i + row0 < n) v[i] = __builtin_bit_cast(i4, *reinterpret_cast<const h8u *>(b + (RPI * i) * ldb + off));
        }
    }
    __device__ __forceinline__ void store(char *lds, const i4 (&v)[NI]) const
    {
#pragma unroll
        for (int i = 0; i < NI; ++i) *reinterpret_cast<i4 *>(lds + wr[i]) = v[i];
    }
    __device__ __forceinline__ h8 frag(const char *lds, int t, int h, int) const
    {
        return read_frag_tr<16 * T>(lds + rd[t] + h * 32 * (32 * T));
    }
};

// A 64-deep slab of a column-major A of up to 16 T rows, loaded element-wise
// into its fragments: lane 16 g + c holds row 16 t + c.
template <int T>
struct ThinSlabM {
    static constexpr int NI = 2 * T;
    const char *base;
    int64_t ldb;
    unsigned off[T];
    int g;

    __device__ __forceinline__ void init(const _Float16 *X, int64_t ld, int first, int ext, int lane)
    {
        base = reinterpret_cast<const char *>(X + first);
        ldb = 2 * ld;
        g = lane >> 4;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int r = 16 * t + (lane & 15);
            off[t] = 8u * g * (unsigned)ldb + 2u * (unsigned)(r < ext ? r : ext - 1);
        }
    }
    __device__ __forceinline__ void load(int k0, i4 (&v)[NI]) const
    {
        const char *b = base + k0 * ldb;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int t = 0; t < T; ++t) {
                h8 x;
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = *reinterpret_cast<const _Float16 *>(b + (32 * h + e) * ldb + off[t]);
                v[h * T + t] = __builtin_bit_cast(i4, x);
            }
    }
    __device__ __forceinline__ void load_tail(int k0, int n, i4 (&v)[NI]) const
    {
        const char *b = base + k0 * ldb;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int t = 0; t < T; ++t) {
                h8 x = zero_h8();
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (32 * h + 8 * g + e < n)
                        x[e] = *reinterpret_cast<const _Float16 *>(b + (32 * h + e) * ldb + off[t]);
                v[h * T + t] = __builtin_bit_cast(i4, x);
            }
    }
};

// The most waves of a workgroup: each has 2 (TM + TN) KB of LDS.
template <int TM, int TN>
constexpr int thin_max_waves() { return TM + TN <= 3 ? 16 : 8; }

// TM row blocks and TN column blocks of 16; p.waves waves (the launch's
// block size over 64) split the 64-deep slabs of A.B followed by those of
// P.Q.
template <int LA, int LB, int TM, int TN>
__global__ void __launch_bounds__((64 * thin_max_waves<TM, TN>())) gemm_bias_act_thin(GemmArgs p)
{
    constexpr bool KA = LA == ROW, KB = LB == COL;
    constexpr int D = TM + TN <= 2 ? 4 : TM + TN <= 5 ? 3 : 2;   // slabs in flight per wave
    constexpr int LDSW = 2048 * (TM + TN);                       // LDS bytes per wave
    static_assert(TM * TN * 1024 <= LDSW, "the partial sums reuse the slabs' LDS");
    __shared__ __attribute__((aligned(16))) char lds[thin_max_waves<TM, TN>() * LDSW];
    using SlabA = std::conditional_t<KA, ThinSlabK<TM>, ThinSlabM<TM>>;
    using SlabB = std::conditional_t<KB, ThinSlabK<TN>, ThinSlabN<TN>>;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nw = p.waves;
    // consecutive tiles of an XCD are the row blocks of one column tile and
    // then its neighbours, which share B's lines in the XCD's L2
    int tm, tn;
    tile_coords(blockIdx.x, gridDim.x, p.tiles_m, tm, tn);
    const int m0 = tm * (16 * TM), n0 = tn * (16 * TN);
    const int nc = KB || n0 + 16 * TN <= p.N ? n0 : p.N - 16 * TN;
    char *const la = lds + wave * LDSW, *const lb = la + 2048 * TM;

    f4 acc[TM][TN];
#pragma unroll
    for (int s = 0; s < TM; ++s)
#pragma unroll
        for (int t = 0; t < TN; ++t) acc[s][t] = f4{0.f, 0.f, 0.f, 0.f};

    // The prologue's ReLU as a signed 16-bit max (with the smallest value
    // when there is none), and the sign of P's fragments under a difference.
    const short floor16 = p.pro ? 0 : (short)-32768;
    const s8 floor8 = {floor16, floor16, floor16, floor16, floor16, floor16, floor16, floor16};

    const int slabs_ab = (p.K + 63) / 64, slabs_pq = (p.K2 + 63) / 64;
    const int64_t slabs = (int64_t)slabs_ab + slabs_pq;
    const int64_t mine_lo = slabs * wave / nw, mine_hi = slabs * (wave + 1) / nw;

#pragma unroll 1
    for (int seg = 0; seg < 2; ++seg) {
        const int K = seg == 0 ? p.K : p.K2;
        const int64_t before = seg == 0 ? 0 : slabs_ab;
        const int nseg = seg == 0 ? slabs_ab : slabs_pq;
        const int lo = mine_lo > before ? (int)(mine_lo - before) : 0;
        const int hi = mine_hi - before < nseg ? (int)(mine_hi - before) : nseg;
        if (lo >= hi) continue;
        const short flip16 = seg == 1 && p.sub ? (short)-32768 : 0;
        const s8 flip8 = {flip16, flip16, flip16, flip16, flip16, flip16, flip16, flip16};

        SlabA xa;
        SlabB xb;
        xa.init(seg == 0 ? p.A : p.P, seg == 0 ? p.lda : p.ldp, m0, p.M - m0, lane);
        xb.init(seg == 0 ? p.B : p.Q, seg == 0 ? p.ldb : p.ldq, nc, p.N - nc, lane);

        i4 ra[D][SlabA::NI], rb[D][SlabB::NI];
        auto load = [&](int d, int slab) {
            xa.load(64 * slab, ra[d]);
            xb.load(64 * slab, rb[d]);
        };
        // LDS accesses of one wave complete in order, so its reads see the
        // writes before them; the fences keep the compiler's order.
        auto multiply = [&](int d) {
            __builtin_amdgcn_wave_barrier();
            if constexpr (KA) xa.store(la, ra[d]);
            xb.store(lb, rb[d]);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                h8 fb[TN];
#pragma unroll
                for (int t = 0; t < TN; ++t) fb[t] = xb.frag(lb, t, h, lane);
#pragma unroll
                for (int s = 0; s < TM; ++s) {
                    h8 f;
                    if constexpr (KA) f = xa.frag(la, s, h, lane);
                    else f = __builtin_bit_cast(h8, ra[d][h * TM + s]);
                    f = __builtin_bit_cast(
                        h8, (s8)(__builtin_elementwise_max(__builtin_bit_cast(s8, f), floor8) ^ flip8));
#pragma unroll
                    for (int t = 0; t < TN; ++t)
                        acc[s][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(f, fb[t], acc[s][t], 0, 0, 0);
                }
            }
        };

        // Whole slabs [lo, full), D in flight (the first loads of a range
        // shorter than D repeat its last slab).
        const int full = hi < K / 64 ? hi : K / 64;
        if (lo < full) {
#pragma unroll
            for (int d = 0; d < D; ++d) load(d, lo + d < full ? lo + d : full - 1);
            int slab = lo;
#pragma unroll 1
            for (; slab + 2 * D <= full; slab += D) {
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    multiply(d);
                    load(d, slab + D + d);
                }
            }
            // the last D to 2 D - 1 of them
#pragma unroll
            for (int d = 0; d < D; ++d) {
                if (slab + d < full) multiply(d);
                if (slab + D + d < full) load(d, slab + D + d);
            }
#pragma unroll
            for (int d = 0; d < D; ++d)
                if (slab + D + d < full) multiply(d);
        }
        if (hi > K / 64) {   // this wave has the product's partial last slab
            const int k0 = K / 64 * 64;
            xa.load_tail(k0, K - k0, ra[0]);
            xb.load_tail(k0, K - k0, rb[0]);
            multiply(0);
        }
    }

    // Partial sums to the wave's LDS: register r of lane l of a block is row
    // 4 (l / 16) + r, column l % 16.
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int s = 0; s < TM; ++s)
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                reinterpret_cast<float *>(la)[(s * TN + t) * 256 + 64 * r + lane] = acc[s][t][r];
    __syncthreads();

    // Consecutive threads take consecutive columns of a row.
    for (int e = tid; e < TM * TN * 256; e += 64 * nw) {
        const int col = e & 15, t = (e >> 4) % TN, row = (e / (16 * TN)) & 15, s = e / (256 * TN);
        const float *src =
            reinterpret_cast<const float *>(lds) + (s * TN + t) * 256 + 64 * (row & 3) + 16 * (row >> 2) + col;
        float x[1] = {0.f};
        for (int w = 0; w < nw; ++w) x[0] += src[w * (LDSW / 4)];
        const int i = m0 + 16 * s + row, j = nc + 16 * t + col;
        if (i < p.M && j < p.N && j >= n0) {
            if (p.bias_kind == BIAS_ROW) x[0] += p.bias_sign * (float)p.bias[j];
            else if (p.bias_kind == BIAS_FULL) x[0] += p.bias_sign * (float)p.bias[(int64_t)i * p.ldbias + j];
            activate(p.act, x);
            p.C[(int64_t)i * p.ldc + j] = (_Float16)x[0];
        }
    }
}

}  // namespace gba
