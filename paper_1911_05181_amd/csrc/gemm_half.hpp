// fp32 GEMM through the f16 matrix instructions: C = epilogue(op(A) * op(B)) with fp32 operands, accumulation and
// result, at half the matrix work of the three-term bf16 split (gemm_split.hpp), which it falls back on step by step.
//
// Every operand element, times a power of two that is common to the panel, is split on its way to LDS into two f16 terms,
//     a = a0 + a1 + e   with  a0 = f16(a),  a1 = f16(a - a0)      (round to nearest),
// and a product is the sum of three term products, a0 b1 + a1 b0 + a0 b0, accumulated in fp32.  a0 and a1 hold 23 bits of
// the 24: e is at most 2^-23 |a| (zero for three elements out of four), and the omitted a1 b1 at most 2^-22 |a b|, both
// without a preferred sign.  As three instructions instead of six round the accumulator, the error against 64 bits
// (2-norm) is smaller than the bf16 split's from k of about 100 on: k = 128: 1.4e-7 against 1.6e-7, 480: 2.5e-7 and
// 3.3e-7, 3200: 6.3e-7 and 8.8e-7, 65536: 3.5e-6 and 4.5e-6 (normal operands; softmax deltas: the same from k = 256 on).
// Shorter sums keep the bf16 split (k = 48: 1.04e-7 and 0.90e-7).
//
// Range.  The panel's scale brings the largest element of its first k step and of a sample of the others into [2^14, 2^15), or
// is known (tanh outputs and softmax deltas are at most 1).  Below 2^-2 the terms leave an error of 2^-25 at most whatever
// the element's size, above 65504 f16 ends.  Every element is checked on the way, and its k step noted where needed:
//   - a non-zero element below 2^-8 (which would lose 2^-17 of itself or more): after the other steps, what both terms left
//     of the step's elements is multiplied with the other operand's first term, in f16 with a scale of its own.  Of normal
//     operands 4e-7 of the elements are that small, one step of 256 x 256 x 32 in 150; a mended step costs about one more.
//   - one below 2^-29 or above 65504: the step multiplies zeros and is taken through the three bf16 terms afterwards, into the
//     same accumulators.
// After a few noted steps (4, and one in eight) the rest of the tile's k goes the bf16 way too.  So operands of any range are
// as exact as in gemm_split.hpp, at about its speed: 4096^3 with elements over 60 binades, or with A D and D^-1 B for powers
// of two up to 2^20, 670-700 us, there 590-650.  Non-finite accumulators are recomputed with the fp32 instruction as there.
//
// Signs alternate over C like a chessboard as in gemm_split.hpp, for the same reason.
//
// What bounds it: power, and the vector work beside the products.  The instructions alone (16x16x32, 1.94 PFLOP/s) would allow
// 647 TFLOP/s of fp32 products; 4096^3 takes 350-380 us (360-390 TFLOP/s, matrix pipes busy 58 % of the cycles at 2 GHz),
// against 580-650 with six bf16 products.  A step of 256 x 256 x 32 takes 2.1 us on one compute unit alone and 2.75 us with all
// busy; its products 1.3 us at 2.4 GHz.  The 16x16x32 form is used because it takes less power than 32x32x16 (loops of nothing
// else: 1.94 and 1.73 PFLOP/s at 2.05 and 1.74 GHz); the same kernel with it took 375-385 us.
//
// Layout.  LDS holds two planes per operand and stage: plane, k chunk of 8, row, 8 f16.  The row index is XORed with twice the
// chunk's number, which keeps the 16-byte fragment reads (16 rows of four chunks) and the 8-byte panel stores off each
// other's banks (no conflicts counted).  A and B change roles in the instruction, so that a lane's four results are four
// consecutive columns of a row of C: 16-byte accesses in the epilogue (output layer over 65536 patterns of 400-480-3203: 960 us
// with the 32 x 32 blocks' epilogue, 755 so).  The k loop has one body and one exit, at its end: with others the compiler
// copies accumulators on every turn.  An element's next load is issued right behind its split, a step ahead; the order of
// products, splits and loads is fixed with scheduling barriers.  The barrier of a step lies before its last block of
// products, which cover the latency of the next step's first fragments (540 us instead of 570 for 256 steps alone).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "gemm_split.hpp"

namespace ulsnn {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));

// (members as SplitTile's; no k groups)
template <int BM_, int BN_, int WM_, int WN_, int WAVES_PER_SIMD_>
struct HalfTile {
    static constexpr int BM = BM_, BN = BN_, BK = 32, WM = WM_, WN = WN_, WAVES_PER_SIMD = WAVES_PER_SIMD_;
    static constexpr int THREADS = WM * WN * 64, WAVES = WM * WN;
    static constexpr int WTM = BM / WM, WTN = BN / WN;
    static constexpr int TM = WTM / 32, TN = WTN / 32;      // of the recomputation
    static constexpr int RM = WTM / 16, RN = WTN / 16;      // accumulator blocks
    static_assert(WTM % 32 == 0 && WTN % 32 == 0 && WAVES <= 16, "tile shape");
};

// (sizes in u16 elements) PLANES terms of R rows of one k step
template <int R>
struct HalfPanel {
    static constexpr int CHUNK = R * 8, PLANE = 4 * CHUNK;
};
__device__ __forceinline__ int half_row(int row, int chunk) { return (row ^ (chunk << 1)) * 8; }

constexpr int HALF_NOTED = 32;       // noted steps a tile keeps a list of

// LDS, in u16 elements: two stages of two planes (the bf16 terms use the same memory as one stage of three planes); zeros
// for the fragments of a noted step to read instead, where both planes of the largest sub-tile side have some; flags of the
// two stages and maxima of the two panels by wavefront, two lists of noted steps (128 ints).
template <class Cfg>
struct HalfLds {
    static constexpr int A = HalfPanel<Cfg::BM>::PLANE, B = HalfPanel<Cfg::BN>::PLANE, STAGE = 2 * (A + B);
    static constexpr int SIDE = (Cfg::WTM > Cfg::WTN ? Cfg::WTM : Cfg::WTN) * 8;
    static constexpr int INTS = 2 * STAGE, ZEROS_A = INTS + 2 * (64 + 2 * HALF_NOTED), ZEROS_B = A == B ? ZEROS_A : ZEROS_A + SIDE;
    static constexpr int SIZE = ZEROS_B + (A > B ? A : B) + SIDE;
};

// Two floats times f to two packed pairs of f16 terms.  (v_fma_mixlo_f16 would form a term in one instruction, but takes 6 cycles
// from the matrix instructions beside it; these take at most 2: 16x16x32 with two of them in between 8.3 ns, with two of
// v_fma_mixlo_f16 11.5, alone 7.1.)
__device__ __forceinline__ void half_pair(float x, float y, const float f, unsigned &p0, unsigned &p1)
{
    float rx, ry;
    unsigned a, b;
    asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(a) : "v"(x * f), "v"(y * f));
    asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel_hi:[0,0,1]" : "=v"(rx) : "v"(x), "v"(f), "v"(a));
    asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "=v"(ry) : "v"(y), "v"(f), "v"(a));
    asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(b) : "v"(rx), "v"(ry));
    p0 = a;
    p1 = b;
}
// The first terms, and 2^22 times what both terms leave of x f and y f (2^-25 at most where they are small, 2^-7 where they
// are below 2^16).
__device__ __forceinline__ void half_remainder(float x, float y, const float f, unsigned &p0, unsigned &rest)
{
    float rx, ry;
    unsigned a, b;
    asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(a) : "v"(x * f), "v"(y * f));
    asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel_hi:[0,0,1]" : "=v"(rx) : "v"(x), "v"(f), "v"(a));
    asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "=v"(ry) : "v"(y), "v"(f), "v"(a));
    asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(b) : "v"(rx), "v"(ry));
    asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[0,0,1]" : "=v"(rx) : "v"(rx), "v"(b));
    asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "=v"(ry) : "v"(ry), "v"(b));
    asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(rest) : "v"(rx * 0x1p22f), "v"(ry * 0x1p22f));
    p0 = a;
}

// The largest of 64 lanes' non-negative values.
__device__ __forceinline__ float wave_max(float v)
{
    auto step = [](float v, auto ctrl, auto rows) {
        return fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, decltype(rows)::value, 0xf, false)));
    };
    std::integral_constant<int, 0xf> all;
    v = step(v, std::integral_constant<int, 0x111>{}, all);      // row_shr 1, 2, 4, 8
    v = step(v, std::integral_constant<int, 0x112>{}, all);
    v = step(v, std::integral_constant<int, 0x114>{}, all);
    v = step(v, std::integral_constant<int, 0x118>{}, all);
    v = step(v, std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});      // row_bcast 15, 31
    v = step(v, std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// The same value, as far as the compiler knows another one: what is derived from it is neither formed early nor kept alive.
__device__ __forceinline__ int fresh(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// One thread's share of a panel of R rows: loads, terms, range check.  It comes in units of W k of one row: 4 (KC) or, with
// consecutive lanes on consecutive rows, 8 or 4 (MC; as many as leave every thread one).  All of a thread's units lie at one k
// (KC) or in one row (MC), so one offset serves them.
template <bool KC, int R, int THREADS>
struct HalfPart {
    using P = HalfPanel<R>;
    typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
    static constexpr int W = KC || R * 4 < THREADS ? 4 : 8, NV = R * 32 / W / THREADS;
    static_assert(R * 32 / W % THREADS == 0 && THREADS % (KC ? 16 : R) == 0, "units");
    float reg[NV][W];
    unsigned off;
    float factor;               // scale and sign
    unsigned lo, lowest;        // (bits << 1) - 1 of the smallest magnitudes that two terms hold well, that the remainder does
    unsigned hi;                // bits of the largest

    static __device__ __forceinline__ int row(int tid, int v) { return KC ? tid / 8 + v * (THREADS / 8) : tid % R; }
    static __device__ __forceinline__ int first_k(int tid, int v) { return KC ? tid % 8 * 4 : (tid / R + v * (THREADS / R)) * W; }
    // A k-contiguous operand's rows beyond the matrix lie behind the buffer's end and read as zero (records()), an m-contiguous
    // one's are redirected to its last row.
    __device__ __forceinline__ void init(int ld, int valid, int tid)
    {
        off = KC ? ((unsigned)row(tid, 0) * (unsigned)ld + (unsigned)first_k(tid, 0)) * 4u
                 : ((unsigned)first_k(tid, 0) * (unsigned)ld + (unsigned)min(row(tid, 0), valid - 1)) * 4u;
    }
    static __device__ __forceinline__ int records(int ld, int valid)
    {
        return KC ? (min(valid, R) - 1) * ld * 4 + 128 : SPLIT_NUM_RECORDS;
    }
    template <int V>
    __device__ __forceinline__ void fetch(const __amdgpu_buffer_rsrc_t rs, int ld)
    {
        if constexpr (KC) {
            const floatx4 x = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, V * (THREADS / 8) * ld * 4, 0));
#pragma unroll
            for (int e = 0; e < 4; ++e) reg[V][e] = x[e];
        } else {
#pragma unroll
            for (int e = 0; e < W; ++e)
                reg[V][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off, (V * (THREADS / R) * W + e) * ld * 4, 0));
        }
    }
    // only the first `left` k exist
    __device__ __forceinline__ void fetch_partial(const float *base, int ld, int valid, int left, int tid)
    {
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int e = 0; e < W; ++e) {
                const int k = first_k(tid, v) + e, r = min(row(tid, v), valid - 1);
                reg[v][e] = k < left ? base[KC ? (size_t)r * ld + k : (size_t)k * ld + r] : 0.f;
            }
    }
    // the scale's sign: odd rows negative (`flip`: even ones)
    static __device__ __forceinline__ float sign(int tid, bool flip) { return ((row(tid, 0) & 1) != 0) != flip ? -1.f : 1.f; }
    // One of THREADS samples of the panel over the whole k range: 128 bytes each at a few dozen places.
    static __device__ __forceinline__ float sample(const float *base, int ld, int valid, int k, int tid)
    {
        if (k < 32) return 0.f;
        if constexpr (KC) {
            constexpr int PLACES = THREADS / 8;
            const int at = tid / 8;
            const floatx4 x = load4_any_align(base + (size_t)(at * 37 % min(valid, R)) * ld + (k - 32) / (PLACES - 1) * at + tid % 8 * 4);
            return fmaxf(fmaxf(fabsf(x[0]), fabsf(x[1])), fmaxf(fabsf(x[2]), fabsf(x[3])));
        } else {
            constexpr int PLACES = THREADS / 32;
            const int at = tid / 32;
            return fabsf(base[(size_t)((k - 1) / (PLACES - 1) * at) * ld + min(at * 32 % R + tid % 32, valid - 1)]);
        }
    }
    __device__ __forceinline__ float largest(float m) const
    {
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int e = 0; e < W; ++e) m = fmaxf(m, fabsf(reg[v][e]));
        return m;
    }
    __device__ __forceinline__ void set_scale(int e, float sign)
    {
        factor = sign * __uint_as_float((unsigned)(127 + e) << 23);
        lo = ((unsigned)(127 - 8 - e) << 24) - 1u;
        lowest = ((unsigned)(127 - 29 - e) << 24) - 1u;
        hi = __float_as_uint(65504.f) - ((unsigned)e << 23);
    }

    // first element (of a plane) of unit V's place in a stage
    template <int V>
    static __device__ __forceinline__ int place(int tid)
    {
        const int k = first_k(tid, V), c = k / 8;
        return c * P::CHUNK + half_row(row(tid, V), c) + k % 8;
    }
    template <int PLANES>
    static __device__ __forceinline__ void put(u16 *dst, const unsigned (&p)[PLANES][W / 2])
    {
#pragma unroll
        for (int t = 0; t < PLANES; ++t) {
            if constexpr (W == 4) *reinterpret_cast<uintx2 *>(dst + t * P::PLANE) = uintx2{p[t][0], p[t][1]};
            else *reinterpret_cast<uintx4_t *>(dst + t * P::PLANE) = uintx4_t{p[t][0], p[t][1], p[t][W / 2 - 2], p[t][W / 2 - 1]};
        }
    }
    // `small`: (bits << 1) - 1 of the smallest non-zero magnitude so far (zero becomes the largest number), `large`: the largest
    template <int V>
    __device__ __forceinline__ void store(u16 *lds, int tid, unsigned &small, float &large) const
    {
        unsigned p[2][W / 2];
#pragma unroll
        for (int e = 0; e < W / 2; ++e) {
            const float x = reg[V][2 * e], y = reg[V][2 * e + 1];
            half_pair(x, y, factor, p[0][e], p[1][e]);
            const unsigned a = (__float_as_uint(x) << 1) - 1u, b = (__float_as_uint(y) << 1) - 1u;
            small = min(min(a, b), small);
            large = fmaxf(fmaxf(fabsf(x), fabsf(y)), large);
        }
        put(lds + place<V>(tid), p);
    }
    // what any lane saw: 1 an element that needs its remainder, 2 one that f16 does not hold
    __device__ __forceinline__ int outside(unsigned small, float large) const
    {
        return (__ballot(small < lo) != 0 ? 1 : 0) | (__ballot((unsigned)(small < lowest) | (unsigned)(__float_as_uint(large) > hi)) != 0 ? 2 : 0);
    }
    template <int V>
    __device__ __forceinline__ void store_remainder(u16 *lds, int tid) const
    {
        unsigned p[2][W / 2];
#pragma unroll
        for (int e = 0; e < W / 2; ++e) half_remainder(reg[V][2 * e], reg[V][2 * e + 1], factor, p[0][e], p[1][e]);
        put(lds + place<V>(tid), p);
    }
    template <int V>
    __device__ __forceinline__ void store_bf16(u16 *lds, int tid) const
    {
        unsigned p[3][W / 2];
#pragma unroll
        for (int e = 0; e < W / 2; ++e) split_pair(reg[V][2 * e], reg[V][2 * e + 1], factor, p[0][e], p[1][e], p[2][e]);
        put(lds + place<V>(tid), p);
    }
};

// Epilogue of a wavefront's sub-tile from 16 x 16 blocks, a lane holding four consecutive columns of row lane % 16.  `even` and
// `odd`: what the sums of even and odd columns are multiplied with.  All loads of 16 rows are issued before their first store.
template <int RM, int RN, int EPI>
__device__ __forceinline__ void half_epilogue(const GemmArgs &g, const floatx4 (&acc)[RM][RN], const int row0, const int col0,
                                              const int lane, float *Cout, const int ldc, const float even, const float odd)
{
    typedef floatx4 floatx4_a4 __attribute__((aligned(4)));
    const int col = col0 + 4 * (lane >> 4);
    auto load = [&](const float *src, int c) {
        if (c + 3 < g.N) return (floatx4)*reinterpret_cast<const floatx4_a4 *>(src);
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (c + r < g.N) v[r] = src[r];
        return v;
    };
    floatx4 bias[RN];
#pragma unroll
    for (int b = 0; b < RN; ++b) {
        bias[b] = floatx4{0.f, 0.f, 0.f, 0.f};
        if ((EPI == EPI_BIAS_TANH || EPI == EPI_BIAS) && g.bias) bias[b] = load(g.bias + col + b * 16, col + b * 16);
    }
#pragma unroll
    for (int a = 0; a < RM; ++a) {
        const int row = row0 + a * 16 + (lane & 15);
        if (row < g.M) {
            float *dst = Cout + (size_t)row * ldc + col;
            floatx4 in[RN];
#pragma unroll
            for (int b = 0; b < RN; ++b) {
                if (EPI == EPI_AXPBY && g.beta != 0.f) in[b] = load(dst + b * 16, col + b * 16);
                else if (EPI == EPI_TANHGRAD) in[b] = load(g.aux + (size_t)row * g.ldaux + col + b * 16, col + b * 16);
                else in[b] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int b = 0; b < RN; ++b) {
                floatx4 out;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float v = __builtin_fmaf(acc[a][b][r], (r & 1) ? odd : even, 0.f);
                    if (EPI == EPI_AXPBY) {
                        out[r] = g.alpha * v;
                        if (g.beta != 0.f) out[r] += g.beta * in[b][r];
                    } else if (EPI == EPI_PARTIAL) {
                        out[r] = v;
                    } else if (EPI == EPI_BIAS_TANH) {
                        out[r] = tanh_f32(v + bias[b][r]);
                    } else if (EPI == EPI_BIAS) {
                        out[r] = v + bias[b][r];
                    } else {
                        out[r] = v * (1.0f - in[b][r] * in[b][r]);
                    }
                }
                const int c = col + b * 16;
                if (c + 3 < g.N) {
                    *reinterpret_cast<floatx4_a4 *>(dst + b * 16) = out;
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (c + r < g.N) dst[b * 16 + r] = out[r];
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The product of one tile over the k range [kbeg, kend), written through `Cout` with epilogue EPI; every thread of the
// workgroup must call this.
template <class Cfg, bool A_KC, bool B_KC, int EPI>
__device__ __forceinline__ void half_segment(const GemmArgs &g, const int tile_m, const int tile_n, const int kbeg, const int kend,
                                             const bool flip, float *Cout, const int ldc, u16 *lds)
{
    constexpr int BM = Cfg::BM, BN = Cfg::BN, BK = Cfg::BK, THREADS = Cfg::THREADS, WAVES = Cfg::WAVES;
    constexpr int RM = Cfg::RM, RN = Cfg::RN;
    using PA = HalfPanel<BM>;
    using PB = HalfPanel<BN>;
    using L = HalfLds<Cfg>;
    constexpr int STAGE = L::STAGE, B0 = 2 * PA::PLANE;
    int *flags = reinterpret_cast<int *>(lds + L::INTS);          // [stage][wavefront]
    unsigned *maxima = reinterpret_cast<unsigned *>(flags + 32);  // [operand][wavefront]
    int *to_mend = flags + 64, *to_repeat = to_mend + HALF_NOTED;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / Cfg::WN, wn = wave % Cfg::WN;
    const int wrow = wm * Cfg::WTM, wcol = wn * Cfg::WTN;
    const int i0 = tile_m * BM, j0 = tile_n * BN;
    const int nfull = (kend - kbeg) / BK, left = (kend - kbeg) % BK;
    const int first_full = left ? 1 : 0, steps = nfull + first_full;      // a partial step comes first

    floatx4 acc[RM][RN];
#pragma unroll
    for (int a = 0; a < RM; ++a)
#pragma unroll
        for (int b = 0; b < RN; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
    // Small sub-tiles have the registers to sum k in blocks of 256: the sums err by less than those of the bf16 split's tiles of
    // the same sizes, whose wavefront groups share k.
    constexpr bool BLOCKS = RM * RN <= 4;
    floatx4 total[BLOCKS ? RM : 1][BLOCKS ? RN : 1];
    auto flush = [&](auto first) {
#pragma unroll
        for (int a = 0; a < RM; ++a)
#pragma unroll
            for (int b = 0; b < RN; ++b) {
                total[a][b] = decltype(first)::value ? acc[a][b] : total[a][b] + acc[a][b];
                acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
    };
    if constexpr (BLOCKS) flush(std::true_type{});

    HalfPart<A_KC, BM, THREADS> pa;
    HalfPart<B_KC, BN, THREADS> pb;
    constexpr int NA = decltype(pa)::NV, NU = NA + decltype(pb)::NV;
    pa.init(g.lda, g.M - i0, tid);
    pb.init(g.ldb, g.N - j0, tid);
    const size_t step_a = A_KC ? (size_t)BK : (size_t)BK * g.lda;
    const size_t step_b = B_KC ? (size_t)BK : (size_t)BK * g.ldb;
    const float *const base_a = A_KC ? g.A + (size_t)i0 * g.lda + kbeg : g.A + (size_t)kbeg * g.lda + i0;
    const float *const base_b = B_KC ? g.B + (size_t)j0 * g.ldb + kbeg : g.B + (size_t)kbeg * g.ldb + j0;
    // the operands of a full step; beyond the last one every load reads as zero, without traffic
    const int records_a = pa.records(g.lda, g.M - i0), records_b = pb.records(g.ldb, g.N - j0);
    int next = 0;
    __amdgpu_buffer_rsrc_t rsa, rsb;
    auto point_at = [&](int full) {
        rsa = __builtin_amdgcn_make_buffer_rsrc((void *)(base_a + step_a * full), 0, full < nfull ? records_a : 0, 0x00020000);
        rsb = __builtin_amdgcn_make_buffer_rsrc((void *)(base_b + step_b * full), 0, full < nfull ? records_b : 0, 0x00020000);
    };
    auto fetch_unit = [&](auto j) {
        constexpr int J = decltype(j)::value;
        if constexpr (J < NA) pa.template fetch<J>(rsa, g.lda);
        else pb.template fetch<J - NA>(rsb, g.ldb);
    };
    auto fetch_partial = [&](const int tid) {
        pa.fetch_partial(base_a + step_a * nfull, g.lda, g.M - i0, left, tid);
        pb.fetch_partial(base_b + step_b * nfull, g.ldb, g.N - j0, left, tid);
    };
    auto fetch_next = [&] {
        point_at(next++);
        for_each_index<NU>(fetch_unit);
    };
    // the split of unit J into a stage; behind each operand's last unit its range check
    unsigned small = 0;
    float large = 0.f;
    int outside = 0;
    auto unit = [&](auto j, u16 *stage) {
        constexpr int J = decltype(j)::value;
        if (J == 0 || J == NA) {
            small = 0xffffffffu;
            large = 0.f;
        }
        if constexpr (J < NA) pa.template store<J>(stage, tid, small, large);
        else pb.template store<J - NA>(stage + B0, tid, small, large);
        if (J == NA - 1) outside = pa.outside(small, large);
        if (J == NU - 1) outside |= pb.outside(small, large);
    };
    auto finish = [&](const int st) { flags[st * 16 + wave] = outside; };

    if (left) fetch_partial(tid);
    else fetch_next();

    // Scales: the largest element of the first step and of a sample of the others goes to [2^14, 2^15).
    const float sign_a = pa.sign(tid, flip), sign_b = pb.sign(tid, false);
    int ea = g.exp_a, eb = g.exp_b;
    bool usable = true;
    if (ea == GEMM_EXP_UNKNOWN || eb == GEMM_EXP_UNKNOWN) {
        float ma = pa.sample(base_a, g.lda, g.M - i0, kend - kbeg, tid), mb = pb.sample(base_b, g.ldb, g.N - j0, kend - kbeg, tid);
        ma = pa.largest(ma);
        mb = pb.largest(mb);
        ma = wave_max(ma);
        mb = wave_max(mb);
        maxima[wave] = __float_as_uint(ma);
        maxima[16 + wave] = __float_as_uint(mb);
        __syncthreads();
        unsigned a = 0, b = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            a = max(a, maxima[w]);
            b = max(b, maxima[16 + w]);
        }
        const int fa = __builtin_amdgcn_readfirstlane((int)(a >> 23)), fb = __builtin_amdgcn_readfirstlane((int)(b >> 23));
        // (all zero: as if the largest were 1)
        if (ea == GEMM_EXP_UNKNOWN) ea = a ? 141 - fa : 14;
        if (eb == GEMM_EXP_UNKNOWN) eb = b ? 141 - fb : 14;
        ea = __builtin_amdgcn_readfirstlane(ea);
        eb = __builtin_amdgcn_readfirstlane(eb);
        usable = ea >= 14 - 40 && ea <= 14 + 40 && eb >= 14 - 40 && eb <= 14 + 40;
    }

    constexpr bool A_LONG = RM > RN;
    constexpr int NS = A_LONG ? RN : RM, NL = A_LONG ? RM : RN;
    static_assert(NL % 2 == 0, "fragments of the longer side alternate between two slots");
    constexpr int PS = A_LONG ? PB::PLANE : PA::PLANE, PL = A_LONG ? PA::PLANE : PB::PLANE;

    // Stage 0 takes the first step, the registers the second.
    for (int i = tid; i < L::SIDE / 2; i += THREADS) {
        reinterpret_cast<unsigned *>(lds + L::ZEROS_A)[i] = reinterpret_cast<unsigned *>(lds + L::ZEROS_A + PA::PLANE)[i] = 0;
        reinterpret_cast<unsigned *>(lds + L::ZEROS_B)[i] = reinterpret_cast<unsigned *>(lds + L::ZEROS_B + PB::PLANE)[i] = 0;
    }
    pa.set_scale(ea, sign_a);
    pb.set_scale(eb, sign_b);
    for_each_index<NU>([&](auto j) { unit(j, lds); });
    finish(0);
    fetch_next();
    __syncthreads();
    const int c4 = lane >> 4;
    const int frag_a = c4 * PA::CHUNK + wrow * 8 + half_row(lane & 15, c4), frag_b = B0 + c4 * PB::CHUNK + wcol * 8 + half_row(lane & 15, c4);
    const int frag_s = A_LONG ? frag_b : frag_a, frag_l = A_LONG ? frag_a : frag_b;
    constexpr int ZERO_L = A_LONG ? L::ZEROS_A : L::ZEROS_B;
    int s = 0, n_mend = 0, n_repeat = 0;
    const int in_f16 = usable ? steps : 0;
    // One step: the products of stage s & 1 (of zeros, if it does not fit f16), and the split of the registers, the next step's
    // elements, into the other stage; behind each split the same unit of the step after is loaded.
    // fragments: the shorter side's, the longer side's of two blocks
    half8 f[2][NS], q[2][2];
    auto read_f = [&](const int cur, const int t) {
#pragma unroll
        for (int x = 0; x < NS; ++x) f[t][x] = *reinterpret_cast<const half8 *>(lds + cur + frag_s + x * 128 + t * PS);
    };
    auto read_q = [&](const u16 *from, const int l) {
#pragma unroll
        for (int t = 0; t < 2; ++t) q[l & 1][t] = *reinterpret_cast<const half8 *>(from + l * 128 + t * PL);
    };
    int seen = flags[lane % WAVES];
    read_q(lds + frag_l, 0);
    read_f(0, 1);
    read_f(0, 0);
    bool more = in_f16 > 0;
    if (more)
#pragma unroll 1
    do {
        constexpr int TA[3] = {0, 1, 0}, TB[3] = {1, 0, 0}, TS[3] = {A_LONG ? 1 : 0, A_LONG ? 0 : 1, 0};
        const int cur = (s & 1) * STAGE, st = (s & 1) ^ 1;
        const u16 *ll = lds + cur + frag_l;
        u16 *const other = lds + st * STAGE;
        if (__builtin_expect(__any(seen != 0), 0)) {
            const bool zeros = __any(seen >= 2);
            (zeros ? to_repeat[n_repeat] : to_mend[n_mend]) = s;
            n_repeat += zeros;
            n_mend += !zeros;
            if (zeros) {
                ll = lds + ZERO_L;
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    q[0][t] = half8{};
#pragma unroll
                    for (int x = 0; x < NS; ++x) f[t][x] = half8{};
                }
            }
        }
        point_at(next++);
        auto multiply = [&](auto block, auto term) {
            constexpr int B = decltype(block)::value, T = decltype(term)::value;
#pragma unroll
            for (int x = 0; x < NS; ++x) {
                floatx4 &c = acc[A_LONG ? B : x][A_LONG ? x : B];
                if constexpr (A_LONG) c = __builtin_amdgcn_mfma_f32_16x16x32_f16(f[TB[T]][x], q[B & 1][TA[T]], c, 0, 0, 0);
                else c = __builtin_amdgcn_mfma_f32_16x16x32_f16(q[B & 1][TB[T]], f[TA[T]][x], c, 0, 0, 0);
            }
        };
        for_each_index<NL>([&](auto block) {
            constexpr int B = decltype(block)::value;
            if constexpr (B + 1 < NL) {
                read_q(ll, B + 1);
                for_each_index<3>([&](auto term) { multiply(block, term); });
                // the units are spread over all blocks but the last
                constexpr int U0 = B * NU / (NL - 1), U1 = (B + 1) * NU / (NL - 1);
                for_each_index<U1 - U0>([&](auto j) {
                    unit(std::integral_constant<int, U0 + decltype(j)::value>{}, other);
                    fetch_unit(std::integral_constant<int, U0 + decltype(j)::value>{});
                });
                if constexpr (B == NL - 2) finish(st);
            } else {
                // Behind the barrier the other stage is whole and nothing reads this one: the last block's products cover
                // the latency of the next step's first fragments, each of which takes the place of one no longer needed.
                __syncthreads();
                seen = flags[st * 16 + lane % WAVES];
                read_q(other + frag_l, 0);
                multiply(block, std::integral_constant<int, 0>{});
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (TS[0] == 1) read_f(st * STAGE, 1);
                multiply(block, std::integral_constant<int, 1>{});
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (TS[0] != 1) read_f(st * STAGE, 1);
                multiply(block, std::integral_constant<int, 2>{});
                __builtin_amdgcn_sched_barrier(0);
                read_f(st * STAGE, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        ++s;
        if constexpr (BLOCKS)
            if (s % 8 == 0) flush(std::false_type{});
        more = (s < in_f16) & (n_mend + n_repeat <= min(4 + (s >> 3), HALF_NOTED - 1));
    } while (more);
    __syncthreads();
    const int done = s - n_repeat;
    if constexpr (BLOCKS) {
#pragma unroll
        for (int a = 0; a < RM; ++a)
#pragma unroll
            for (int b = 0; b < RN; ++b) acc[a][b] += total[a][b];
    }
    const int rest = n_repeat + (steps - s);
    if (__builtin_expect(n_mend + rest > 0, 0)) {
        const int tid = fresh(threadIdx.x), lane = tid & 63, c4 = lane >> 4;
        const int frag_a = c4 * PA::CHUNK + wrow * 8 + half_row(lane & 15, c4), frag_b = c4 * PB::CHUNK + wcol * 8 + half_row(lane & 15, c4);
        pa.init(g.lda, g.M - i0, tid);
        pb.init(g.ldb, g.N - j0, tid);
        if (done == 0) ea = eb = 16;      // (nothing in the accumulators yet: the bf16 split's own scale)
        pa.set_scale(ea, sign_a);
        pb.set_scale(eb, sign_b);
        auto fetch_step = [&](const int t) {
            if (t < first_full) {
                fetch_partial(tid);
            } else {
                point_at(t - first_full);
                for_each_index<NU>(fetch_unit);
            }
        };
        int i = 0;
        if (n_mend > 0)
#pragma unroll 1
        do {
            __syncthreads();
            fetch_step(__builtin_amdgcn_readfirstlane(to_mend[i]));
                            // the remainders of both operands, 2^22 times as large as the sums
                            for_each_index<NU>([&](auto j) {
                                constexpr int J = decltype(j)::value;
                                if constexpr (J < NA) pa.template store_remainder<J>(lds, tid);
                                else pb.template store_remainder<J - NA>(lds + B0, tid);
                            });
                            __syncthreads();
                            const u16 *ls = lds + (A_LONG ? B0 + frag_b : frag_a), *ll = lds + (A_LONG ? frag_a : B0 + frag_b);
                            half8 f[2][NS];
            #pragma unroll
                            for (int p = 0; p < 2; ++p)
            #pragma unroll
                                for (int x = 0; x < NS; ++x) f[p][x] = *reinterpret_cast<const half8 *>(ls + x * 128 + p * PS);
            #pragma unroll
                            for (int l = 0; l < NL; ++l) {
                                half8 q[2];
            #pragma unroll
                                for (int p = 0; p < 2; ++p) q[p] = *reinterpret_cast<const half8 *>(ll + l * 128 + p * PL);
            #pragma unroll
                                for (int x = 0; x < NS; ++x) {
                                    floatx4 &c = acc[A_LONG ? l : x][A_LONG ? x : l];
                                    c *= 0x1p22f;
            #pragma unroll
                                    for (int p = 0; p < 2; ++p)
                                        c = A_LONG ? __builtin_amdgcn_mfma_f32_16x16x32_f16(f[p][x], q[p ^ 1], c, 0, 0, 0)
                                                   : __builtin_amdgcn_mfma_f32_16x16x32_f16(q[p], f[p ^ 1][x], c, 0, 0, 0);
                                    c *= 0x1p-22f;
                                }
                                __builtin_amdgcn_sched_barrier(0);
                            }
        } while (++i < n_mend);
        constexpr int B3 = 3 * PA::PLANE;
        auto fetch_repeat = [&] { fetch_step(i < n_repeat ? __builtin_amdgcn_readfirstlane(to_repeat[i]) : s + (i - n_repeat)); };
        i = 0;
        if (rest > 0) {
        __syncthreads();
        fetch_repeat();
#pragma unroll 1
        do {
            // three bf16 terms, two of them per instruction as in split_kernel's MIXED form
            for_each_index<NU>([&](auto j) {
                constexpr int J = decltype(j)::value;
                if constexpr (J < NA) pa.template store_bf16<J>(lds, tid);
                else pb.template store_bf16<J - NA>(lds + B3, tid);
            });
            ++i;
            fetch_repeat();      // (behind the last step: zeros)
            __syncthreads();
            // fragments (t, k half | t, k half): (a1 high, a0 low), (a1 low, a0 high), (a0 high, a2 low), (a0 low, a2 high)
            typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
            constexpr int T0[4] = {1, 1, 0, 0}, T1[4] = {0, 0, 2, 2}, H0[4] = {4, 0, 4, 0}, H1[4] = {0, 4, 0, 4};
            constexpr int TA[6] = {0, 2, 1, 3, 1, 0}, TB[6] = {2, 0, 1, 1, 3, 0};
            auto fragment = [&](const u16 *row, const int plane, const int p) {
                const uintx2 x = *reinterpret_cast<const uintx2 *>(row + T0[p] * plane + H0[p]);
                const uintx2 y = *reinterpret_cast<const uintx2 *>(row + T1[p] * plane + H1[p]);
                return __builtin_bit_cast(bf16x8, uintx4_t{x[0], x[1], y[0], y[1]});
            };
            const u16 *ls = lds + (A_LONG ? B3 + frag_b : frag_a), *ll = lds + (A_LONG ? frag_a : B3 + frag_b);
#pragma unroll
            for (int x0 = 0; x0 < NS; x0 += 2) {
                bf16x8 f[4][2];
#pragma unroll
                for (int p = 0; p < 4; ++p)
#pragma unroll
                    for (int x = 0; x < 2; ++x) f[p][x] = fragment(ls + (x0 + x) * 128, PS, p);
#pragma unroll
                for (int l = 0; l < NL; ++l) {
                    bf16x8 q[4];
#pragma unroll
                    for (int p = 0; p < 4; ++p) q[p] = fragment(ll + l * 128, PL, p);
#pragma unroll
                    for (int p = 0; p < 6; ++p)
#pragma unroll
                        for (int x = 0; x < 2; ++x) {
                            floatx4 &c = acc[A_LONG ? l : x0 + x][A_LONG ? x0 + x : l];
                            c = A_LONG ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[TB[p]][x], q[TA[p]], c, 0, 0, 0)
                                       : __builtin_amdgcn_mfma_f32_16x16x32_bf16(q[TB[p]], f[TA[p]][x], c, 0, 0, 0);
                        }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __syncthreads();
        } while (i < rest);
        }
    }
    const int late = fresh(threadIdx.x) & 63;
    // 0 * x is NaN exactly where x is not finite
    float probe = 0.f;
#pragma unroll
    for (int a = 0; a < RM; ++a)
#pragma unroll
        for (int b = 0; b < RN; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) probe = fmaf(acc[a][b][r], 0.f, probe);
    if (__builtin_expect(__any(probe != 0.0f), 0)) {
        split_fallback<Cfg, A_KC, B_KC, EPI>(g, i0 + wrow, j0 + wcol, kbeg, kend, late, Cout, ldc);
        return;
    }
    const float unscale = __uint_as_float((unsigned)(127 - ea - eb) << 23);
    const float even = ((late & 1) != 0) != flip ? -unscale : unscale;
    half_epilogue<RM, RN, EPI>(g, acc, i0 + wrow, j0 + wcol, late, Cout, ldc, even, -even);
}

template <class Cfg, bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__(Cfg::THREADS, Cfg::WAVES_PER_SIMD) void half_kernel(const GemmArgs g)
{
    __shared__ __attribute__((aligned(16))) u16 lds[HalfLds<Cfg>::SIZE];
    int tile_m, tile_n, z;
    const int splits = gridDim.y;
    work_of_workgroup(blockIdx.y * gridDim.x + blockIdx.x, g.tiles_m, g.tiles_n, splits, tile_m, tile_n, z);
    const int kbeg = z * g.kchunk;
    const int kend = (kbeg + g.kchunk < g.K) ? kbeg + g.kchunk : g.K;
    float *Cout = g.C;
    int ldc = g.ldc;
    if (EPI == EPI_PARTIAL) {
        Cout = g.C + (size_t)z * g.partial_stride;
        ldc = g.N;
    }
    half_segment<Cfg, A_KC, B_KC, EPI>(g, tile_m, tile_n, kbeg, kend, (z & 1) != 0, Cout, ldc, lds);
}

}  // namespace ulsnn
