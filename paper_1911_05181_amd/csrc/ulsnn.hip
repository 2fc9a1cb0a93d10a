// Host side of the C ABI declared in include/ulsnn.h: argument checks, choice of tile shape and k split,
// workspace layout, and the stream-ordered launches.  No device memory is allocated here.
#include "../../include/ulsnn.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <mutex>
#include <type_traits>

#include "gemm_bf16.hpp"
#include "gemm_launch.hpp"
#include "line_search.hpp"
#include "mlp_kernels.hpp"
#include "small_net.hpp"
#include "vec_kernels.hpp"

using namespace ulsnn;

// Built-in scratch of ulsnn_mlp_grad_static (callers that cannot allocate a workspace).  In host code this name is
// only a handle for hipGetSymbolAddress: the device address, one per GPU, is resolved by static_scratch() below.
static __device__ __align__(256) unsigned char scratch[ULSNN_STATIC_SCRATCH_BYTES];

namespace {

// Compute units of the current device (MI355X: 8 XCDs x 32 = 256), read from the runtime once; the planner's
// cost model and the grid sizes of the streaming kernels use it.  Without a device (host-only plan queries) the
// MI355X figure is assumed.
int query_num_cu()
{
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
        return n;
    (void)hipGetLastError();   // no device: not an error of a later launch
    return 256;
}
inline int num_cu()
{
    static const int n = query_num_cu();
    return n;
}
constexpr int SLAB_ROWS = 65536;     // patterns processed per internal pass of the MLP gradient

inline bool is_n(char t) { return t == 'N' || t == 'n'; }
inline bool is_t(char t) { return t == 'T' || t == 't' || t == 'C' || t == 'c'; }
inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// ---------------------------------------------------------------------------------------------------------
// GEMM dispatch: tile shapes, the cost model that picks one (and a k split), and the launchers
// ---------------------------------------------------------------------------------------------------------

struct CfgInfo {
    int bm, bn, bk, threads, occ;   // occ = resident workgroups per compute unit
    double eff;                     // matrix-core efficiency of the steady state relative to the best shape
    const char *name;
};

constexpr CfgInfo CFG_INFO[CFG_COUNT] = {
    {256, 128, 16, 512, 2, 1.00, "256x128"}, {128, 128, 16, 512, 3, 0.98, "128x128w8"},
    {128, 128, 16, 256, 4, 0.97, "128x128"}, {128, 64, 16, 256, 5, 0.93, "128x64"},
    {64, 128, 16, 256, 5, 0.93, "64x128"},   {64, 64, 16, 256, 8, 0.86, "64x64"},
    {64, 64, 64, 512, 2, 0.86, "64x64k64"},
    {160, 128, 16, 256, 3, 1.06, "160x128"},   // (1.06 x the 3-wavefront utilisation = what it sustains: 116 TFLOP/s)
    {64, 64, 32, 512, 4, 0.86, "64x64k32"},
};

struct GemmPlan {
    bool split;      // cfg is a SplitId (gemm_split.hpp), else a CfgId (gemm.hpp)
    int cfg;
    int tiles_m, tiles_n;
    int splits, kchunk;
    double est_us;
};

// Fraction of the matrix-core rate a SIMD reaches with w resident wavefronts (measured: one wavefront cannot
// hide its own LDS, barrier and global-load latency; four can).
inline double simd_utilisation(double w)
{
    static const double u[5] = {0.0, 0.60, 0.78, 0.86, 0.90};
    if (w >= 4.0) return u[4];
    if (w <= 1.0) return u[1];
    const int lo = (int)w;
    return u[lo] + (u[lo + 1] - u[lo]) * (w - lo);
}

// Estimated run time of one launch (+ the split-k reduction), in microseconds.  Not a simulator: a consistent
// way to trade tile efficiency against how evenly the workgroups fill 256 compute units.
double model_us(const CfgInfo &c, bool a_kc, bool b_kc, int m, int n, int k, int splits, int *kchunk_out,
                int *splits_out)
{
    const int chunk = (int)round_up((size_t)(k + splits - 1) / splits, c.bk);
    const int sp = (k + chunk - 1) / chunk;
    *kchunk_out = chunk;
    *splits_out = sp;
    const long tiles = (long)((m + c.bm - 1) / c.bm) * ((n + c.bn - 1) / c.bn);
    const long wgs = tiles * sp;
    const double layout = (!a_kc && !b_kc) ? 0.92 : (a_kc && b_kc) ? 1.0 : 0.97;   // 4-byte LDS reads cost more
    const double cu_rate = 155.0e12 / 256.0 * c.eff * layout;   // flop/s of one compute unit (peak is for 256 of them)
    const double flops_wg = 2.0 * c.bm * c.bn * (double)chunk;
    const double wps = c.threads / 256.0;                                          // wavefronts per SIMD per WG
    const long slots = (long)num_cu() * c.occ;
    const long full = wgs / slots, rem = wgs % slots;
    double t = full * c.occ * flops_wg / (cu_rate * simd_utilisation(c.occ * wps));
    if (rem) {
        const double per_cu = std::ceil((double)rem / num_cu());
        t += per_cu * flops_wg / (cu_rate * simd_utilisation(per_cu * wps));
    }
    t += 3.0e-6 + (double)m * n * sp * 4.0 / 4.0e12;                               // ramp-up and the store burst
    if (sp > 1) t += 3.0e-6 + (double)m * n * (sp + 1.0) * 4.0 / 5.0e12;            // reduction pass
    return t * 1e6;
}

// Choose tile shape and k split (at most `split_limit` slices; 1 = no split).  `cfg_mask` restricts the shapes
// (bit i = CfgId i).
GemmPlan plan_gemm(int m, int n, int k, bool a_kc, bool b_kc, int split_limit, unsigned cfg_mask)
{
    GemmPlan best{};
    best.est_us = 1e30;
    for (int ci = 0; ci < CFG_COUNT; ++ci) {
        if (!(cfg_mask >> ci & 1) || ci == CFG_64K64 || ci == CFG_64K32) continue;
        const CfgInfo &c = CFG_INFO[ci];
        // the 160-row shape exists to avoid padding: only where it computes fewer rows than 128-row tiles would
        if (ci == CFG_160x128 && round_up((size_t)m, 160) >= round_up((size_t)m, 128)) continue;
        const int max_splits = std::max(1, std::min(std::min(64, split_limit), k / (8 * c.bk)));
        for (int s = 1; s <= max_splits; ++s) {
            int chunk, sp;
            const double us = model_us(c, a_kc, b_kc, m, n, std::max(k, 1), s, &chunk, &sp);
            if (sp != s) continue;   // this s collapses onto a smaller split count already seen
            if (us < best.est_us) {
                best.cfg = ci;
                best.tiles_m = (m + c.bm - 1) / c.bm;
                best.tiles_n = (n + c.bn - 1) / c.bn;
                best.splits = sp;
                best.kchunk = chunk;
                best.est_us = us;
            }
        }
    }
    // Unsplit 64x64 launches that cannot fill the chip take the eight-wavefront variants of the tile.  Up to four
    // workgroups per compute unit: k step 32 (2048^3 161 -> 155 us; with more workgroups than that the plain tile's
    // eight small workgroups per CU do better: output layer at 4096 patterns 120 against 124.5 us).  At most one
    // workgroup per compute unit: k step 64; the launch is bound by the latency of its chain of k steps
    // (1024^3 34.5 -> 26.9 us, 512^3 17.8 -> 14.4 us).
    if (best.cfg == CFG_64 && best.splits == 1) {
        const long tiles = (long)best.tiles_m * best.tiles_n;
        CfgId alt = CFG_64;
        if ((cfg_mask >> CFG_64K32 & 1) && tiles <= 4 * num_cu() && k >= 4 * CFG_INFO[CFG_64K32].bk &&
            k % CFG_INFO[CFG_64K32].bk == 0)   // (a partial last step would eat the gain: hidden layer, k = 400)
            alt = CFG_64K32;
        if ((cfg_mask >> CFG_64K64 & 1) && tiles <= num_cu() && k >= 4 * CFG_INFO[CFG_64K64].bk) alt = CFG_64K64;
        if (alt != CFG_64) {
            best.cfg = alt;
            best.kchunk = (int)round_up((size_t)k, CFG_INFO[alt].bk);
        }
    }
    return best;
}

// (launchers: gemm_launch.hpp)
constexpr unsigned ALL_CFGS = (1u << CFG_COUNT) - 1;
// ---------------------------------------------------------------------------------------------------------
// The same products through the bf16 matrix instructions (gemm_split.hpp): tile shapes, cost model, launchers
// ---------------------------------------------------------------------------------------------------------

// Run time of a launch that gives every compute unit r workgroups: base + (r - 1) * base_more + chunk * slope(r), with
// slope(r) = slope_1 (idle + (1 - idle) r) for r <= 1 and slope_r times the rounds beyond, the last of which counts 0.6 + 0.4
// of its share (microseconds, and microseconds per k).  Fitted to launches with r = 1 .. 5, k = 512 and 2048 in three layouts
// and, the tiles of 128 rows and more, to 29 products from 2048^3 to 16384 x 16384 x 2048: mostly within 12 % of the measured
// time where k >= 1000, and the tile it chooses within 3 % of the fastest but for two (6 and 7 %).  Not modelled: the stores
// of a large C under a short k (12000 x 5000 x 64 takes 1.5 times what it says, with every tile).
struct SplitInfo {
    int bm, bn, bk, threads, occ;
    double base, base_more, slope_1, slope_r, idle;
    const char *name;
};
constexpr SplitInfo SPLIT_INFO[SP_COUNT] = {
    {256, 256, 16, 512, 1, 13.5, 8.0, 0.1380, 0.1380, 0.60, "256x256"}, {256, 128, 32, 512, 1, 7.5, 5.0, 0.0760, 0.0750, 0.70, "256x128"},
    {128, 128, 32, 512, 1, 5.7, 3.0, 0.0406, 0.0450, 0.75, "128x128w8"}, {128, 128, 16, 256, 3, 7.7, 1.0, 0.0445, 0.0405, 0.75, "128x128"},
    {128, 64, 32, 512, 2, 5.9, 0.9, 0.0240, 0.0240, 0.75, "128x64"},     {64, 128, 32, 512, 2, 5.9, 0.9, 0.0240, 0.0240, 0.75, "64x128"},
    {64, 64, 32, 256, 3, 4.0, 0.3, 0.0170, 0.0136, 0.75, "64x64"},       {64, 64, 64, 512, 1, 4.2, 2.2, 0.0146, 0.0155, 0.75, "64x64k64"},
    {32, 32, 128, 512, 1, 4.2, 3.0, 0.0061, 0.0061, 0.75, "32x32k128"},
};

double split_model_us(const SplitInfo &c, int m, int n, int k, int splits, int *kchunk_out, int *splits_out)
{
    const int chunk = (int)round_up((size_t)(k + splits - 1) / splits, c.bk);
    const int sp = (k + chunk - 1) / chunk;
    *kchunk_out = chunk;
    *splits_out = sp;
    const double wgs = (double)((m + c.bm - 1) / c.bm) * ((n + c.bn - 1) / c.bn) * sp;
    const double r = wgs / num_cu(), whole = std::ceil(r);
    // A round that leaves compute units idle takes less time than a full one: the chip runs at a higher clock (power bounds
    // these kernels), and a shared compute unit takes the next workgroup as soon as one of its own ends.  4608^3 with
    // 256 x 256 tiles, 27 % of a second round: 1100 us where two full rounds would take 1300.
    const double rounds = 0.6 * whole + 0.4 * r;
    double t = c.base + (whole - 1.0) * c.base_more;
    t += chunk * (r <= 1.0 ? c.slope_1 * (c.idle + (1.0 - c.idle) * r) : c.slope_r * rounds);
    if (sp > 1) t += 3.0 + (double)m * n * (sp + 1.0) * 4.0 / 5.0e6;
    return t;
}

GemmPlan plan_split(int m, int n, int k, int split_limit, unsigned mask)
{
    GemmPlan best{};
    best.est_us = 1e30;
    best.split = true;
    for (int ci = 0; ci < SP_COUNT; ++ci) {
        const SplitInfo &c = SPLIT_INFO[ci];
        if (!(mask >> ci & 1) || (ci == SP_32K128 && k < c.bk)) continue;   // (a step that would be mostly padding)
        const int max_splits = std::max(1, std::min(std::min(64, split_limit), k / 128));
        for (int s = 1; s <= max_splits; ++s) {
            int chunk, sp;
            const double us = split_model_us(c, m, n, k, s, &chunk, &sp);
            if (sp != s || us >= best.est_us) continue;
            best.cfg = ci;
            best.tiles_m = (m + c.bm - 1) / c.bm;
            best.tiles_n = (n + c.bn - 1) / c.bn;
            best.splits = sp;
            best.kchunk = chunk;
            best.est_us = us;
        }
    }
    return best;
}

constexpr unsigned ALL_SPLIT = (1u << SP_COUNT) - 1;

inline const char *plan_name(const GemmPlan &p) { return p.split ? SPLIT_INFO[p.cfg].name : CFG_INFO[p.cfg].name; }

// Launch a product by its plan (either unit).
hipError_t launch_plan(const GemmPlan &p, bool a_kc, bool b_kc, int epi, GemmArgs a, hipStream_t s, bool mixed = false)
{
    a.tiles_m = p.tiles_m;
    a.tiles_n = p.tiles_n;
    a.kchunk = p.kchunk;
    return p.split ? launch_split(p.cfg, p.splits, a_kc, b_kc, epi, mixed, a, s) : launch_fp32(p.cfg, p.splits, a_kc, b_kc, epi, a, s);
}

// Longest k that one workgroup sums through the split.  Its downward rounding grows with k (1.1e-11 k of the result) where
// the other errors grow with the root: at 300,000 the split's error is 5.4e-6 and the fp32 instruction's 7.0e-6, at 2^21
// 2.5e-5 and 1.8e-5; they cross near 800,000.
constexpr int SPLIT_MAX_CHUNK = 1 << 19;

// The plan of a product with the given leading dimensions.  The fp32 instruction serves rows so far apart that a tile
// does not fit the buffer instructions' 32-bit offsets and sums longer than SPLIT_MAX_CHUNK (and ulsnn_sgemm_planned, which
// names its tile shapes).
GemmPlan plan_product(int m, int n, int k, bool a_kc, bool b_kc, int lda, int ldb, int split_limit, unsigned mask = ALL_SPLIT)
{
    if (std::max(lda, ldb) > SPLIT_MAX_LD) return plan_gemm(m, n, k, a_kc, b_kc, split_limit, ALL_CFGS);
    const GemmPlan p = plan_split(m, n, k, split_limit, mask);
    return p.kchunk <= SPLIT_MAX_CHUNK ? p : plan_gemm(m, n, k, a_kc, b_kc, split_limit, ALL_CFGS);
}

inline unsigned grid_for(size_t elems)
{
    return (unsigned)std::min<size_t>((elems + 255) / 256, (size_t)num_cu() * 8);
}

// The reduction that follows a split-k launch: out = epilogue(sum of partials).
hipError_t launch_reduce(int splits, int epi, const GemmArgs &a, const float *partial, hipStream_t s)
{
    const size_t total = (size_t)a.M * a.N;
    if (epi == EPI_TANHGRAD) {
        hipLaunchKernelGGL(splitk_reduce_kernel<true>, dim3(grid_for(total)), dim3(256), 0, s, partial, total, splits,
                           a.C, a.M, a.N, a.ldc, 1.0f, 0.0f, a.aux, a.ldaux);
    } else {
        hipLaunchKernelGGL(splitk_reduce_kernel<false>, dim3(grid_for(total)), dim3(256), 0, s, partial, total,
                           splits, a.C, a.M, a.N, a.ldc, a.alpha, a.beta, (const float *)nullptr, 0);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------
// bf16-operand GEMM dispatch (fp32 accumulation): tile shapes and their costs
// ---------------------------------------------------------------------------------------------------------

using T16_128 = Tile16<128, 128, 2, 2, 4>;   // 256 threads, 4 workgroups / CU (LDS 39 KB each)
using T16_64 = Tile16<64, 64, 2, 2, 8>;      // 256 threads, 8 workgroups / CU
// Steps of 64 k (wide16_kernel): 256 x 256, one workgroup per CU, and 128 x 128, two, both with eight wavefronts.  The sub-tile
// of the large one lies across or along by what each read costs: with both operands k-contiguous 64 x 128 and 128 x 64 measured
// the same on plain products, the hidden delta 237 and 243 us at 65536 patterns; with both m-contiguous (dW2 there) 261 and 249.
using T16_256x256 = Wide16<256, 256, 4, 2, 2>;
using T16_256x256t = Wide16<256, 256, 2, 4, 2>;
using T16_128k64 = Wide16<128, 128, 4, 2, 4>;
// For patterns whose rows are not 16-byte aligned and find no room for an aligned copy: such a product fetches element by element
// and is bound by that, so the tile that fetches least per product wins.  dW1 against the best of 128 x 128 and 64 x 64: 785 x 256
// over 65536 patterns 243 us (396), 2049 x 1024 over 20000 488 (789), 4001 x 1000 over 9000 396 (693); hidden layer 65536 x 256 x 785
// 177 (246), 30000 x 500 x 3001 665 (910).
using T16_256x256u = Tile16<256, 256, 4, 2, 2>;

enum Cfg16Id { CFG16_128 = 0, CFG16_64, CFG16_256x256, CFG16_128K64, CFG16_256x256U, CFG16_COUNT };

// One launch on an otherwise idle chip, in microseconds, by the layout of its operands (0 a k-contiguous A and an m-contiguous B,
// 1 both k-contiguous, 2 both m-contiguous): `base`, `more` per further round of workgroups, and per k of the longest slice
// `slope_1` while every compute unit has at most one workgroup (`idle` of it when hardly any has one), else `slope_r` per round,
// of which the last counts as whole to the part `full`.  `delta`: what forming the output delta multiplies the slopes by (1.0
// where the layout never does).  Fitted to 4300 launches of the gradients' five products over 70 networks and batches (48 to
// 1024 inputs, 32 to 1024 hidden, 10 to 4096 classes, 256 to 40000 patterns), each tile off by 4 (first layout) to 10 percent.
// The tile and slices it picks take longer than the best of those measured by 0.7 percent (output and hidden layer), 1.9 (hidden
// delta), 2.3 (dW2) and 1.2 (dW1); one matrix rate for all layouts, which stood here, by 2, 15, 11 and 5.
// `delta_base`: what forming the delta adds to `base`: over 180 dW2 products of 32 to 800 hidden units, 64 to 3203 classes and 256 to
// 8192 patterns, the 128 x 128 tile with steps of 64 k was taken 29 times where 64 x 64 is 0.7 to 3.5 us faster, now 5 times.
// `waits`: a latency of so many rounds that every `held` rounds, which a compute unit works on together, have once.
struct Tile16Cost {
    double base, more, slope_1, slope_r, idle, full, delta;
    double delta_base = 0.0, waits = 0.0, held = 1.0;
};
// `loose`: the same where the rows of A are not 16-byte aligned (a k-contiguous A, and an m-contiguous one): each element is a load of
// its own, five to ten times the cost per k.  Fitted to 1800 launches of 74 products (49 to 4001 inputs, 700 to 65536 patterns); the
// choice takes 0.6 and 1.6 percent longer than the best measured, the costs of aligned rows 5 and 41.  The round costs of 64 x 64 (eight
// workgroups a compute unit) and of dW1 on 128 x 128 (four) are fitted apart, to 120 products of 20 to 300 hidden units: without `waits`
// several rounds at once seemed to gain nothing, so dW1 of 2049 x 100 over 65536 patterns was cut into 30 slices (383 us, 59 take 320), of
// 1017 x 34 into 32 (64 take 20 us less), and the hidden layer 45001 x 72 x 1017 went to 128 x 128 (204 us, 64 x 64 170).
struct Cfg16Info {
    int bm, bn, bk;
    Tile16Cost cost[3], loose[2];      // (a slope of zero: not offered)
    const char *name;
};
constexpr Cfg16Info CFG16_INFO[CFG16_COUNT] = {
    {128, 128, 32, {{8.6, 1.7, 0.0129, 0.0087, 0.91, 1.00, 1.00}, {7.4, 1.2, 0.0183, 0.0098, 0.76, 1.00, 1.22}, {4.9, 0.1, 0.0156, 0.0090, 0.80, 1.00, 1.75}},
     {{2.9, 0.0, 0.1633, 0.0984, 0.64, 1.00, 1.00}, {3.1, 0.0, 0.1104, 0.0500, 0.76, 0.50, 1.00, 0.0, 0.90, 4.0}}, "bf16 128x128"},
    {64, 64, 32, {{5.3, 0.5, 0.0057, 0.0036, 0.91, 0.97, 1.00}, {5.1, 0.4, 0.0089, 0.0043, 0.83, 1.00, 1.24}, {4.0, 0.0, 0.0074, 0.0040, 0.89, 1.00, 2.05}},
     {{2.0, 0.0, 0.0656, 0.0235, 0.86, 0.50, 1.00, 0.0, 2.60, 8.0}, {5.7, 0.0, 0.0454, 0.0227, 0.84, 0.50, 1.00, 0.0, 0.86, 8.0}}, "bf16 64x64"},
    {256, 256, 64, {{16.0, 14.0, 0.0278, 0.0235, 0.53, 0.47, 1.00}, {9.5, 7.1, 0.0248, 0.0242, 0.72, 0.73, 1.19}, {8.2, 10.0, 0.0240, 0.0228, 0.74, 0.66, 1.45}}, {}, "bf16 256x256"},
    {128, 128, 64, {{6.4, 2.6, 0.0095, 0.0075, 0.73, 1.00, 1.00}, {5.5, 1.5, 0.0096, 0.0080, 0.75, 0.86, 1.33}, {4.6, 2.4, 0.0104, 0.0086, 0.76, 1.00, 1.47, 0.8}}, {}, "bf16 128x128k64"},
    {256, 256, 32, {}, {{2.0, 0.0, 0.2185, 0.2176, 0.84, 1.00, 1.00}, {2.0, 0.0, 0.1582, 0.1571, 0.95, 0.90, 1.00}}, "bf16 256x256u"},
};

struct Gemm16Plan {
    Cfg16Id cfg;
    int tiles_m, tiles_n;
    int splits, kchunk;
    double est_us;
};

// `rows`: ROWS16_WIDE where the operands suit wide16_kernel, which loads whole vectors with 32-bit offsets within a panel of 256
// rows: 16-byte aligned rows shorter than WIDE16_MAX_LD.  ROWS16_LOOSE where those of A are not aligned (never with both operands
// k-contiguous).  `delta`: the product forms the output delta while loading.
constexpr int WIDE16_MAX_LD = 1 << 22;
// Hidden and output layers of up to three steps of 64 k: the loop has too few to hide its loads, and the tile's epilogue is the longer
// (output layer 4096 x 1000 x 64: 10.3 us, 64 x 64 7.5; hidden layer 4096 x 700 x 48: 7.9 and 6.7).  Over 260 such calls of k = 32 to 160
// (1024 to 65536 patterns, 64 to 3200 columns) the best tile with steps of 32 k is 0.06 us behind the best of all.
constexpr int WIDE16_FORWARD_MIN_K = 161;
enum Rows16 { ROWS16_WIDE, ROWS16_ALIGNED, ROWS16_LOOSE };
Gemm16Plan plan_gemm16(int m, int n, int k, bool a_kc, bool b_kc, bool allow_split, size_t max_partial_floats, Rows16 rows, bool delta = false)
{
    Gemm16Plan best{};
    best.est_us = 1e30;
    int max_splits = allow_split ? std::max(1, std::min(64, k / 256)) : 1;
    if ((size_t)m * n > 0) max_splits = (int)std::min<size_t>(max_splits, std::max<size_t>(1, max_partial_floats / ((size_t)m * n)));
    for (int ci = 0; ci < CFG16_COUNT; ++ci) {
        const Cfg16Info &c = CFG16_INFO[ci];
        if (c.bk == 64 && (rows != ROWS16_WIDE || (!b_kc && a_kc && k < WIDE16_FORWARD_MIN_K))) continue;
        const Tile16Cost &t = rows == ROWS16_LOOSE ? c.loose[a_kc ? 0 : 1] : c.cost[a_kc && b_kc ? 1 : a_kc ? 0 : 2];
        if (t.slope_1 == 0.0) continue;
        const int tiles_m = (m + c.bm - 1) / c.bm, tiles_n = (n + c.bn - 1) / c.bn;
        for (int s = 1; s <= max_splits; ++s) {
            const int chunk = (int)round_up((size_t)(std::max(k, 1) + s - 1) / s, c.bk);
            if ((std::max(k, 1) + chunk - 1) / chunk != s) continue;      // (fewer slices, seen already)
            const double r = (double)tiles_m * tiles_n * s / num_cu(), whole = std::ceil(r), slope = delta ? t.delta : 1.0;
            double us = t.base + (delta ? t.delta_base : 0.0) + (whole - 1.0) * t.more;
            us += chunk * slope * (r <= 1.0 ? t.slope_1 * (t.idle + (1.0 - t.idle) * r) : t.slope_r * (t.waits * std::ceil(r / t.held) + t.full * whole + (1.0 - t.full) * r));
            us += (double)m * n * s * (s > 1 || !a_kc ? 4.0 : 2.0) / 8.0e6;      // its stores, beyond what `base` has
            if (s > 1) us += 3.0 + (double)m * n * (s + 1.0) * 4.0 / 5.0e6;       // the reduction
            if (us < best.est_us) {
                best.cfg = (Cfg16Id)ci;
                best.tiles_m = tiles_m;
                best.tiles_n = tiles_n;
                best.splits = s;
                best.kchunk = chunk;
                best.est_us = us;
            }
        }
    }
    return best;
}

template <class Cfg, bool A_KC, bool B_KC, int EPI, int DELTA = 0>
hipError_t launch16_one(const Gemm16Args &a, int splits, hipStream_t s)
{
    const dim3 grid((unsigned)(a.tiles_m * a.tiles_n), (unsigned)splits);
    if constexpr (std::is_same_v<Cfg, T16_256x256> && !A_KC && !B_KC)
        hipLaunchKernelGGL((wide16_kernel<T16_256x256t, A_KC, B_KC, EPI, DELTA>), grid, dim3(Cfg::THREADS), 0, s, a);
    else if constexpr (Cfg::BK == 64)
        hipLaunchKernelGGL((wide16_kernel<Cfg, A_KC, B_KC, EPI, DELTA>), grid, dim3(Cfg::THREADS), 0, s, a);
    else
        hipLaunchKernelGGL((gemm16_kernel<Cfg, A_KC, B_KC, EPI, DELTA>), grid, dim3(Cfg::THREADS), 0, s, a);
    return hipGetLastError();
}

inline bool rows_16b_aligned(const void *p, int ld) { return ((uintptr_t)p & 15) == 0 && (ld & 7) == 0; }

// Columns of C one statistics group of the output-layer epilogue covers: the wavefront sub-tile width of the shape.
inline int stat_group_width(Cfg16Id id)
{
    switch (id) {
        case CFG16_128: return T16_128::WTN;
        case CFG16_256x256: return T16_256x256::WTN;
        case CFG16_128K64: return T16_128k64::WTN;
        default: return T16_64::WTN;
    }
}

// The combinations the MLP gradient needs: NN with bias+tanh / bias / bias + softmax statistics, NT with the tanh'
// mask, NT and TN partials, TN with alpha/beta.
hipError_t launch_gemm16(const Gemm16Plan &p, bool a_kc, bool b_kc, int epi, Gemm16Args a, hipStream_t s)
{
    a.tiles_m = p.tiles_m;
    a.tiles_n = p.tiles_n;
    a.kchunk = p.kchunk;
    a.aligned = rows_16b_aligned(a.A, a.lda) && rows_16b_aligned(a.B, a.ldb);
    const bool c_bf16 = epi == EPI_BIAS_TANH || epi == EPI_TANHGRAD || epi == EPI_BIAS_STATS || epi == EPI_TANH_MSE;
    a.c_vec = ((uintptr_t)a.C & 15) == 0 && (a.ldc % (c_bf16 ? 8 : 4)) == 0;
    a.aux_vec = a.aux != nullptr && rows_16b_aligned(a.aux, a.ldaux);
    auto go = [&](auto cfg) -> hipError_t {
        using Cfg = decltype(cfg);
        if (epi == EPI_BIAS_TANH && a_kc && !b_kc) return launch16_one<Cfg, true, false, EPI_BIAS_TANH>(a, p.splits, s);
        if (epi == EPI_PARTIAL && !a_kc && !b_kc && !a.row_lse) return launch16_one<Cfg, false, false, EPI_PARTIAL>(a, p.splits, s);
        if (epi == EPI_AXPBY && !a_kc && !b_kc && !a.row_lse) return launch16_one<Cfg, false, false, EPI_AXPBY>(a, p.splits, s);
        if constexpr (!std::is_same_v<Cfg, T16_256x256u>) {
            if (epi == EPI_BIAS && a_kc && !b_kc) return launch16_one<Cfg, true, false, EPI_BIAS>(a, p.splits, s);
            if ((epi == EPI_BIAS_STATS || epi == EPI_STATS_ONLY) && a_kc && !b_kc) {
                // one statistics group per wavefront column; the logits' rows must be 16-byte aligned
                if (a.stat_groups != (a.N + Cfg::WTN - 1) / Cfg::WTN || a.stat_stride < (size_t)a.M || !a.stats || !a.label_logit || !a.labels ||
                    (epi == EPI_BIAS_STATS && !a.c_vec))
                    return hipErrorInvalidValue;
                return epi == EPI_BIAS_STATS ? launch16_one<Cfg, true, false, EPI_BIAS_STATS>(a, p.splits, s)
                                             : launch16_one<Cfg, true, false, EPI_STATS_ONLY>(a, p.splits, s);
            }
            if ((epi == EPI_TANH_MSE || epi == EPI_MSE_ONLY) && a_kc && !b_kc) {
                if (a.stat_groups != (a.N + Cfg::WTN - 1) / Cfg::WTN || a.stat_stride < (size_t)a.M || !a.stats || !a.targets || a.ldt < a.N ||
                    (epi == EPI_TANH_MSE && !a.c_vec))
                    return hipErrorInvalidValue;
                return epi == EPI_TANH_MSE ? launch16_one<Cfg, true, false, EPI_TANH_MSE>(a, p.splits, s)
                                           : launch16_one<Cfg, true, false, EPI_MSE_ONLY>(a, p.splits, s);
            }
            if (a.row_lse) {   // a product that forms the output delta from the logits while loading them
                if (!a.aligned || !a.labels) return hipErrorInvalidValue;
                if (a_kc && b_kc && epi == EPI_TANHGRAD) return launch16_one<Cfg, true, true, EPI_TANHGRAD, 1>(a, p.splits, s);
                if (a_kc && b_kc && epi == EPI_PARTIAL) return launch16_one<Cfg, true, true, EPI_PARTIAL, 1>(a, p.splits, s);
                if (!a_kc && !b_kc && epi == EPI_PARTIAL) return launch16_one<Cfg, false, false, EPI_PARTIAL, 2>(a, p.splits, s);
                if (!a_kc && !b_kc && epi == EPI_AXPBY) return launch16_one<Cfg, false, false, EPI_AXPBY, 2>(a, p.splits, s);
                return hipErrorInvalidValue;
            }
            if (epi == EPI_TANHGRAD && a_kc && b_kc) return launch16_one<Cfg, true, true, EPI_TANHGRAD>(a, p.splits, s);
            if (epi == EPI_PARTIAL && a_kc && b_kc) return launch16_one<Cfg, true, true, EPI_PARTIAL>(a, p.splits, s);
        }
        return hipErrorInvalidValue;
    };
    if (CFG16_INFO[p.cfg].bk == 64 && (!a.aligned || (c_bf16 && !a.c_vec))) return hipErrorInvalidValue;   // (plan_gemm16's ROWS16_WIDE)
    return p.cfg == CFG16_128 ? go(T16_128{}) : p.cfg == CFG16_256x256 ? go(T16_256x256{})
         : p.cfg == CFG16_128K64 ? go(T16_128k64{}) : p.cfg == CFG16_256x256U ? go(T16_256x256u{}) : go(T16_64{});
}

// Plan of an unsplit ulsnn_sgemm.
GemmPlan plan_sgemm(int m, int n, int k, bool a_kc, bool b_kc, int lda, int ldb)
{
    return plan_product(m, n, k, a_kc, b_kc, lda, ldb, 1);
}

// Plan of a product that may cut k into at most `slices` slices.  A split costs a second launch (the reduction), so it
// is taken where it beats the unsplit tiles of 64 rows and more.  The 32 x 32 tile, which splits k over the wavefronts
// of a workgroup instead, is preferred to it up to 0.92 of its modelled time: over 48 products of 64 x 64 to 640 x 640 and
// k = 512 to 4096 that is where the measured times cross (512^3 7.3 us, 9.3 split; 256 x 256 x 768 8.6 and 9.0, x 1024
// 10.1 and 8.8; 512 x 512 x 1536 13.4 and 13.0).
GemmPlan plan_sgemm_ws(int m, int n, int k, bool a_kc, bool b_kc, int lda, int ldb, size_t slices)
{
    const GemmPlan one = plan_sgemm(m, n, k, a_kc, b_kc, lda, ldb);
    if (slices < 2) return one;
    const int limit = (int)std::min<size_t>(64, slices);
    if (!one.split) {
        const GemmPlan cut = plan_product(m, n, k, a_kc, b_kc, lda, ldb, limit);
        return (cut.splits > 1 && cut.est_us < 0.8 * one.est_us) ? cut : one;
    }
    const GemmPlan cut = plan_product(m, n, k, a_kc, b_kc, lda, ldb, limit, ALL_SPLIT & ~(1u << SP_32K128));
    return (cut.splits > 1 && one.est_us > 0.92 * cut.est_us) ? cut : one;
}

// ---------------------------------------------------------------------------------------------------------
// MLP gradient: plans and workspace layout for one slab of patterns
// ---------------------------------------------------------------------------------------------------------

constexpr size_t PARTIAL_CAP_FLOATS = (size_t)32 << 20;   // at most 128 MiB of split-k partials per product

struct MlpLayout {
    int slab;                       // rows per pass
    int ldh, ldz;                   // row strides (elements) of H / dA1 and of Z / dO
    int ldw1p, ldw2p;               // bf16 path: row strides of the 16-byte aligned copies of W1 and W2
    size_t floats_pa, floats_pb;    // split-k partial regions: A (dW2) and B (hidden delta, then dW1)
    size_t off_h, off_z, off_da1, off_rowloss, off_pa, off_pb, bytes;
    size_t off_do16, off_w1p, off_w2p, off_zlab, off_lse;   // bf16 path only
};

struct SlabPlans {
    GemmPlan g1, g2, g3, g4, g5;
};

bool desc_ok(const ulsnn_mlp_desc *d)
{
    return d && d->n_in >= 1 && d->n_hid >= 1 && d->n_out >= 1;
}

// Sizes depend on the network and on min(batch, SLAB_ROWS) only, and do not decrease with the batch, so a
// workspace sized for a batch also serves every smaller one.
// Small networks at small batches take a two-launch path (small_net.hpp).  Its scratch: one share of every sum
// per workgroup of SMALL_ROWS patterns.
inline int small_net_stride(const ulsnn_mlp_desc *d)
{
    return (int)round_up((size_t)d->n_in * d->n_hid + (size_t)d->n_hid * d->n_out + d->n_hid + d->n_out + 1, 4);
}
inline bool small_net_shape(const ulsnn_mlp_desc *d, long long batch)
{
    return d->operand_dtype == 0 && d->n_in <= SMALL_MAX_IN && d->n_hid <= SMALL_MAX_HID &&
           d->n_out <= SMALL_MAX_OUT && batch >= 1 && batch <= SMALL_MAX_BATCH &&
           small_net_dense_floats(d->n_in, d->n_hid, d->n_out) <= SMALL_LDS_FLOATS;
}
inline size_t small_net_bytes(const ulsnn_mlp_desc *d, long long batch)
{
    if (!small_net_shape(d, batch)) return 0;
    const size_t groups = (size_t)(batch + SMALL_ROWS - 1) / SMALL_ROWS;
    return round_up(groups * small_net_stride(d) * sizeof(float), 256);
}

MlpLayout mlp_layout(const ulsnn_mlp_desc *d, int batch)
{
    MlpLayout L{};
    const bool bf16 = d->operand_dtype == 1;
    const size_t act = bf16 ? 2 : 4;               // bytes per stored activation (H, dA1)
    L.slab = std::max(1, std::min(batch, SLAB_ROWS));
    L.ldh = (int)round_up((size_t)d->n_hid, 32);
    L.ldz = (int)round_up((size_t)d->n_out, 32);
    L.ldw1p = (int)round_up((size_t)d->n_hid, 8);
    L.ldw2p = (int)round_up((size_t)d->n_out, 8);
    const size_t mn3 = (size_t)d->n_hid * d->n_out, mn5 = (size_t)d->n_in * d->n_hid;
    const size_t mn4 = (size_t)L.slab * d->n_hid;
    L.floats_pa = std::max(std::max(mn3, mn5), std::min(PARTIAL_CAP_FLOATS, 64 * std::max(mn3, mn5)));
    L.floats_pb = std::max(mn4, std::min(PARTIAL_CAP_FLOATS, 16 * mn4));
    size_t off = 0;
    L.off_h = off;        off += round_up((size_t)L.slab * L.ldh * act, 256);
    // fp32: the logits / output delta.  bf16: the softmax statistics of the output layer's epilogue, one
    // (max, sum) pair per row and group of at least 32 columns (the logits themselves live at off_do16)
    L.off_z = off;        off += round_up(bf16 ? (size_t)L.slab * (L.ldz / 32) * sizeof(float2) : (size_t)L.slab * L.ldz * 4, 256);
    L.off_da1 = off;      off += round_up((size_t)L.slab * L.ldh * act, 256);
    L.off_rowloss = off;  off += round_up((size_t)L.slab * 4, 256);
    L.off_pa = off;       off += round_up(L.floats_pa * 4, 256);
    L.off_pb = off;       off += round_up(L.floats_pb * 4, 256);
    if (bf16) {
        L.off_do16 = off; off += round_up((size_t)L.slab * L.ldz * 2, 256);
        L.off_w1p = off;  off += round_up((size_t)d->n_in * L.ldw1p * 2, 256);
        L.off_w2p = off;  off += round_up((size_t)d->n_hid * L.ldw2p * 2, 256);
        L.off_zlab = off; off += round_up((size_t)L.slab * 4, 256);
        L.off_lse = off;  off += round_up((size_t)L.slab * 4, 256);
    }
    L.bytes = std::max(off, small_net_bytes(d, batch));
    return L;
}

// Plans of the five products for `rows` patterns.  A split count is limited by the partial region it writes.
SlabPlans plan_slab(const MlpLayout &L, int n_in, int n_hid, int n_out, int rows)
{
    SlabPlans s;
    auto slices = [](size_t region, int m, int n) { return (int)std::min<size_t>(64, region / ((size_t)m * n)); };
    s.g1 = plan_product(rows, n_hid, n_in, true, false, n_in, n_hid, 1);
    s.g2 = plan_product(rows, n_out, n_hid, true, false, L.ldh, n_out, 1);
    s.g3 = plan_product(n_hid, n_out, rows, false, false, L.ldh, L.ldz, slices(L.floats_pa, n_hid, n_out));
    s.g4 = plan_product(rows, n_hid, n_out, true, true, L.ldz, n_out, slices(L.floats_pb, rows, n_hid));
    s.g5 = plan_product(n_in, n_hid, rows, false, false, n_in, L.ldh, slices(L.floats_pb, n_in, n_hid));
    return s;
}

int check_mlp_args(const ulsnn_mlp_desc *d, const void *W1, const void *W2, const void *X, const void *targets,
                   long long batch, const float *dW1, const float *dW2, const float *loss, bool backward)
{
    if (!d) return ULSNN_ERR_NULL;
    if (d->n_in < 1 || d->n_hid < 1 || d->n_out < 1 || batch < 0) return ULSNN_ERR_DIM;
    if (d->n_in > ULSNN_MAX_LD || d->n_hid > ULSNN_MAX_LD || d->n_out > ULSNN_MAX_LD) return ULSNN_ERR_UNSUPPORTED;
    if (!W1 || !W2 || !loss) return ULSNN_ERR_NULL;
    if (backward && (!dW1 || !dW2)) return ULSNN_ERR_NULL;
    if (batch > 0 && (!X || !targets)) return ULSNN_ERR_NULL;
    const int nb = (d->b1 != nullptr) + (d->b2 != nullptr) + (d->db1 != nullptr) + (d->db2 != nullptr);
    if (backward ? (nb != 0 && nb != 4) : ((d->b1 != nullptr) != (d->b2 != nullptr))) return ULSNN_ERR_NULL;
    if (d->accumulate != 0 && d->accumulate != 1) return ULSNN_ERR_UNSUPPORTED;
    if (d->operand_dtype != 0 && d->operand_dtype != 1) return ULSNN_ERR_UNSUPPORTED;
    return ULSNN_OK;
}

#define HIP_TRY(expr)                                   \
    do {                                                \
        if ((expr) != hipSuccess) return ULSNN_ERR_HIP; \
    } while (0)
#define MARK(stage)                                       \
    do {                                                  \
        if (ev) HIP_TRY(hipEventRecord(ev[stage], s));    \
    } while (0)

// `ev`, if not null, is an array of ULSNN_MLP_STAGES + 1 events recorded at the stage boundaries.
// What one call computes beyond the forward pass.
struct MlpTask {
    const int32_t *labels;   // softmax / cross-entropy output stage (targets == nullptr)
    const float *targets;    // tanh / squared-error output stage of the paper: dense T[batch x n_out]
    bool backward;           // false: loss only (error evaluation), dW1 / dW2 untouched
};

// The share of final_reduce_kernel that adds a product's k slices (none if it was not cut).
ReducePart reduce_part(int splits, int M, int N, int ldc, float *out, const float *partial)
{
    ReducePart r{};
    if (splits < 2) return r;
    const size_t total = (size_t)M * N;
    r.partial = partial; r.stride = total; r.splits = splits;
    r.out = out; r.M = M; r.N = N; r.ldc = ldc;
    r.vec = ldc == N && total % 4 == 0 && ((uintptr_t)out & 15) == 0 && ((uintptr_t)partial & 15) == 0;
    r.blocks = (int)grid_for(r.vec ? total / 4 : total);
    return r;
}

// db2 and db1 of `rows` patterns (c.D, c.ld and the softmax rows are given): slices of at least 16 rows, as many as give
// every compute unit about four workgroups and `region` floats of scratch hold shares for.
template <int KIND0>
hipError_t launch_column_sums(ColumnSumArgs c, const ulsnn_mlp_desc *d, int rows, float *scratch_floats, size_t region,
                              float beta, hipStream_t s)
{
    constexpr int V0 = 64 * ColumnVec<KIND0>::VEC;      // columns per workgroup (the same for D[1])
    c.N[0] = d->n_out; c.N[1] = d->n_hid;
    c.out[0] = d->db2; c.out[1] = d->db1;
    c.rows = rows; c.beta = beta; c.partial = scratch_floats;
    c.blocks0 = (d->n_out + V0 - 1) / V0;
    const int blocks = c.blocks0 + (d->n_hid + V0 - 1) / V0, total = d->n_out + d->n_hid;
    int slices = std::max(1, std::min(4 * num_cu() / blocks, (rows + 15) / 16));
    slices = (int)std::min<size_t>((size_t)slices, std::max<size_t>(1, region / (size_t)total));
    c.slice_rows = (rows + slices - 1) / slices;
    c.slices = (rows + c.slice_rows - 1) / c.slice_rows;
    hipLaunchKernelGGL(column_sum_kernel<KIND0>, dim3((unsigned)blocks, (unsigned)c.slices), dim3(256), 0, s, c);
    hipLaunchKernelGGL(column_sum_join_kernel, dim3((unsigned)((total + 63) / 64)), dim3(256), 0, s, c);
    return hipGetLastError();
}

int mlp_grad_impl16(const ulsnn_mlp_desc *d, const u16 *W1, const u16 *W2, const u16 *X, const MlpTask &task,
                    int batch, float *dW1, float *dW2, float *loss, bool accumulate, hipEvent_t *ev);

// W1v, W2v, Xv point at fp32 (operand_dtype 0) or bf16 (operand_dtype 1) data.
int mlp_grad_impl(const ulsnn_mlp_desc *d, const void *W1v, const void *W2v, const void *Xv,
                  const MlpTask &task, int batch, float *dW1, float *dW2, float *loss, bool accumulate,
                  hipEvent_t *ev = nullptr)
{
    hipStream_t s = (hipStream_t)d->hip_stream;
    const int n_in = d->n_in, n_hid = d->n_hid, n_out = d->n_out;
    const bool biases = d->b1 != nullptr;

    if (batch == 0) {
        if (!accumulate) {
            hipLaunchKernelGGL(zero_kernel, dim3(1), dim3(256), 0, s, loss, (size_t)1);
            if (task.backward) {
                hipLaunchKernelGGL(zero_kernel, dim3(grid_for((size_t)n_in * n_hid)), dim3(256), 0, s, dW1,
                                   (size_t)n_in * n_hid);
                hipLaunchKernelGGL(zero_kernel, dim3(grid_for((size_t)n_hid * n_out)), dim3(256), 0, s, dW2,
                                   (size_t)n_hid * n_out);
            }
            if (biases && task.backward) {
                hipLaunchKernelGGL(zero_kernel, dim3(grid_for(n_hid)), dim3(256), 0, s, d->db1, (size_t)n_hid);
                hipLaunchKernelGGL(zero_kernel, dim3(grid_for(n_out)), dim3(256), 0, s, d->db2, (size_t)n_out);
            }
            HIP_TRY(hipGetLastError());
        }
        return ULSNN_OK;
    }

    if (d->operand_dtype == 1)
        return mlp_grad_impl16(d, (const u16 *)W1v, (const u16 *)W2v, (const u16 *)Xv, task, batch, dW1, dW2, loss,
                               accumulate, ev);
    const float *W1 = (const float *)W1v, *W2 = (const float *)W2v, *X = (const float *)Xv;

    // small network, small batch, no stage timing asked for: two launches instead of nine
    if (!ev && small_net_shape(d, batch)) {
        const size_t need = mlp_layout(d, batch).bytes;
        if (!d->workspace || ((uintptr_t)d->workspace & 255) || d->workspace_bytes < need) return ULSNN_ERR_WORKSPACE;
        SmallNetArgs a{};
        a.n_in = n_in; a.n_hid = n_hid; a.n_out = n_out; a.batch = batch;
        a.W1 = W1; a.W2 = W2; a.b1 = d->b1; a.b2 = d->b2; a.X = X; a.labels = task.labels; a.targets = task.targets;
        a.partial = (float *)d->workspace; a.stride = small_net_stride(d); a.backward = task.backward ? 1 : 0;
        a.strides = small_net_strides(n_in, n_hid, n_out);
        const int groups = (batch + SMALL_ROWS - 1) / SMALL_ROWS;
        const size_t lds = (size_t)small_net_lds_floats(n_in, n_hid, n_out, a.strides) * sizeof(float);
        SmallReduceArgs r{};
        r.partial = a.partial; r.stride = a.stride; r.groups = groups;
        r.n1 = n_in * n_hid; r.n2 = n_hid * n_out; r.n_hid = n_hid; r.n_out = n_out;
        r.dW1 = task.backward ? dW1 : nullptr; r.dW2 = task.backward ? dW2 : nullptr;
        r.db1 = task.backward ? d->db1 : nullptr; r.db2 = task.backward ? d->db2 : nullptr;
        r.loss = loss; r.beta = accumulate ? 1.0f : 0.0f;
        const int total = task.backward ? r.n1 + r.n2 + n_hid + n_out + 1 : 1;
        hipLaunchKernelGGL(small_net_kernel, dim3(groups), dim3(256), lds, s, a);
        hipLaunchKernelGGL(small_reduce_kernel, dim3((total + 63) / 64), dim3(256), 0, s, r);
        HIP_TRY(hipGetLastError());
        return ULSNN_OK;
    }

    const MlpLayout L = mlp_layout(d, batch);
    if (!d->workspace || ((uintptr_t)d->workspace & 255) || d->workspace_bytes < L.bytes)
        return ULSNN_ERR_WORKSPACE;
    char *ws = (char *)d->workspace;
    float *H = (float *)(ws + L.off_h);
    float *Z = (float *)(ws + L.off_z);
    float *dA1 = (float *)(ws + L.off_da1);
    float *row_loss = (float *)(ws + L.off_rowloss);
    float *part_a = (float *)(ws + L.off_pa);
    float *part_b = (float *)(ws + L.off_pb);

    for (int r0 = 0; r0 < batch; r0 += L.slab) {
        const int rows = std::min(L.slab, batch - r0);
        const SlabPlans P = plan_slab(L, n_in, n_hid, n_out, rows);
        const float beta = (r0 > 0 || accumulate) ? 1.0f : 0.0f;
        const float *Xs = X + (size_t)r0 * n_in;
        const int32_t *ys = task.labels ? task.labels + r0 : nullptr;
        const float *ts = task.targets ? task.targets + (size_t)r0 * n_out : nullptr;
        GemmArgs a{};
        MARK(0);

        // H = tanh(Xs W1 + b1)
        a = GemmArgs{};
        a.A = Xs; a.lda = n_in; a.B = W1; a.ldb = n_hid; a.C = H; a.ldc = L.ldh;
        a.M = rows; a.N = n_hid; a.K = n_in; a.alpha = 1.f; a.beta = 0.f; a.bias = d->b1;
        HIP_TRY(launch_plan(P.g1, true, false, EPI_BIAS_TANH, a, s));
        MARK(1);

        // Z = H W2 + b2   (softmax form)   or   Y = tanh(H W2 + b2)   (the paper's form)
        a = GemmArgs{};
        a.A = H; a.lda = L.ldh; a.B = W2; a.ldb = n_out; a.C = Z; a.ldc = L.ldz;
        a.M = rows; a.N = n_out; a.K = n_hid; a.alpha = 1.f; a.beta = 0.f; a.bias = d->b2;
        HIP_TRY(launch_plan(P.g2, true, false, ts ? EPI_BIAS_TANH : EPI_BIAS, a, s));
        MARK(2);

        // output stage: row losses and, for a gradient, the output delta in place of Z; loss (+)= their sum
        const dim3 per_row((unsigned)((rows + 3) / 4));      // four wavefronts, one row each
        if (ts) {
            if (task.backward)
                hipLaunchKernelGGL(mse_delta_kernel<true>, per_row, dim3(256), 0, s, Z, L.ldz, rows, n_out, ts, n_out, row_loss);
            else
                hipLaunchKernelGGL(mse_delta_kernel<false>, per_row, dim3(256), 0, s, Z, L.ldz, rows, n_out, ts, n_out, row_loss);
        } else if (n_out <= 1024) {
            // Narrow rows: 16 lanes or one wavefront each (a workgroup per row: 52955 x 13, 73 us; so 5.8).  At 3203
            // columns both ways take the same time and the workgroup needs fewer registers, so wide rows keep it.
            auto launch = [&](auto lanes, auto v) {
                constexpr int LANES = decltype(lanes)::value, V = decltype(v)::value, PER_WG = 256 / LANES;
                const dim3 grid((unsigned)((rows + PER_WG - 1) / PER_WG));
                if (task.backward)
                    hipLaunchKernelGGL((softmax_ce_narrow_kernel<LANES, V, true>), grid, dim3(256), 0, s, Z, L.ldz, rows, n_out,
                                       ys, row_loss);
                else
                    hipLaunchKernelGGL((softmax_ce_narrow_kernel<LANES, V, false>), grid, dim3(256), 0, s, Z, L.ldz, rows, n_out,
                                       ys, row_loss);
            };
            if (n_out <= 64) launch(std::integral_constant<int, 16>{}, std::integral_constant<int, 1>{});
            else if (n_out <= 256) launch(std::integral_constant<int, 64>{}, std::integral_constant<int, 1>{});
            else launch(std::integral_constant<int, 64>{}, std::integral_constant<int, 4>{});
        } else if (n_out <= 256 * 16) {
            if (task.backward)
                hipLaunchKernelGGL((softmax_ce_kernel<256, 16>), dim3(rows), dim3(256), 0, s, Z, L.ldz, n_out, ys,
                                   row_loss);
            else
                hipLaunchKernelGGL((softmax_ce_kernel<256, 16, false>), dim3(rows), dim3(256), 0, s, Z, L.ldz,
                                   n_out, ys, row_loss);
        } else {
            if (task.backward)
                hipLaunchKernelGGL((softmax_ce_long_kernel<256>), dim3(rows), dim3(256), 0, s, Z, L.ldz, n_out, ys,
                                   row_loss);
            else
                hipLaunchKernelGGL((softmax_ce_long_kernel<256, false>), dim3(rows), dim3(256), 0, s, Z, L.ldz,
                                   n_out, ys, row_loss);
        }
        // the loss sum and the reductions of dW2 and dW1 end the pass in one launch, unless there is none of the latter
        const bool final_reduce = task.backward && (P.g3.splits > 1 || P.g5.splits > 1);
        if (!final_reduce)
            hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(1024), 0, s, row_loss, (long long)rows, loss, beta);
        HIP_TRY(hipGetLastError());
        MARK(3);
        if (!task.backward) {
            MARK(4); MARK(5); MARK(6); MARK(7); MARK(8);
            continue;
        }

        // dW2 (+)= H^T dO   and   dA1 = (dO W2^T) * (1 - H*H): independent of each other
        GemmArgs a3{}, a4{};
        a3.A = H; a3.lda = L.ldh; a3.B = Z; a3.ldb = L.ldz; a3.C = dW2; a3.ldc = n_out;
        a3.M = n_hid; a3.N = n_out; a3.K = rows; a3.alpha = 1.f; a3.beta = beta;
        a4.A = Z; a4.lda = L.ldz; a4.B = W2; a4.ldb = n_out; a4.C = dA1; a4.ldc = L.ldh;
        a4.M = rows; a4.N = n_hid; a4.K = n_out; a4.alpha = 1.f; a4.beta = 0.f; a4.aux = H; a4.ldaux = L.ldh;
        {
            GemmArgs p3 = a3, p4 = a4;
            if (P.g4.splits > 1) { p4.C = part_b; p4.partial_stride = (size_t)a4.M * a4.N; }
            if (P.g3.splits > 1) { p3.C = part_a; p3.partial_stride = (size_t)a3.M * a3.N; }
            HIP_TRY(launch_plan(P.g4, true, true, P.g4.splits > 1 ? EPI_PARTIAL : EPI_TANHGRAD, p4, s, true));   // (summed over patterns)
            HIP_TRY(launch_plan(P.g3, false, false, P.g3.splits > 1 ? EPI_PARTIAL : EPI_AXPBY, p3, s));
        }
        MARK(4);
        if (P.g4.splits > 1) HIP_TRY(launch_reduce(P.g4.splits, EPI_TANHGRAD, a4, part_b, s));
        MARK(5);

        // dW1 (+)= Xs^T dA1
        a = GemmArgs{};
        a.A = Xs; a.lda = n_in; a.B = dA1; a.ldb = L.ldh; a.C = dW1; a.ldc = n_hid;
        a.M = n_in; a.N = n_hid; a.K = rows; a.alpha = 1.f; a.beta = beta;
        {
            GemmArgs p5 = a;     // (the hidden delta's slices are summed: its region is free for dW1's)
            if (P.g5.splits > 1) { p5.C = part_b; p5.partial_stride = (size_t)a.M * a.N; }
            HIP_TRY(launch_plan(P.g5, false, false, P.g5.splits > 1 ? EPI_PARTIAL : EPI_AXPBY, p5, s));
        }
        MARK(6);
        if (final_reduce) {
            FinalReduceArgs f{};
            f.part[0] = reduce_part(P.g3.splits, a3.M, a3.N, a3.ldc, dW2, part_a);
            f.part[1] = reduce_part(P.g5.splits, a.M, a.N, a.ldc, dW1, part_b);
            f.row_loss = row_loss; f.rows = rows; f.loss = loss; f.beta = beta;
            hipLaunchKernelGGL(final_reduce_kernel, dim3((unsigned)(1 + f.part[0].blocks + f.part[1].blocks)), dim3(256), 0, s, f);
            HIP_TRY(hipGetLastError());
        }
        MARK(7);

        // db2 (+)= 1^T dO,  db1 (+)= 1^T dA1
        if (biases) {
            ColumnSumArgs c{};
            c.D[0] = Z; c.ld[0] = L.ldz; c.D[1] = dA1; c.ld[1] = L.ldh;
            HIP_TRY(launch_column_sums<COLUMNS_F32>(c, d, rows, part_a, L.floats_pa, beta, s));
        }
        MARK(8);
    }
    return ULSNN_OK;
}

// The same gradient with X, W1, W2 stored as bf16 (operand_dtype 1): H, the logits and dA1 are kept in bf16 and fed
// to the bf16 matrix instructions, every product accumulates in fp32; the softmax statistics and the loss come from
// the fp32 accumulators of the output layer, the output delta exists only in registers (formed from the bf16 logits
// inside the two products that consume it), and the weight gradients are fp32.
int mlp_grad_impl16(const ulsnn_mlp_desc *d, const u16 *W1, const u16 *W2, const u16 *X, const MlpTask &task,
                    int batch, float *dW1, float *dW2, float *loss, bool accumulate, hipEvent_t *ev)
{
    hipStream_t s = (hipStream_t)d->hip_stream;
    const int n_in = d->n_in, n_hid = d->n_hid, n_out = d->n_out;
    const bool biases = d->b1 != nullptr;
    const MlpLayout L = mlp_layout(d, batch);
    if (!d->workspace || ((uintptr_t)d->workspace & 255) || d->workspace_bytes < L.bytes)
        return ULSNN_ERR_WORKSPACE;
    char *ws = (char *)d->workspace;
    u16 *H = (u16 *)(ws + L.off_h);
    float2 *stats = (float2 *)(ws + L.off_z);
    // one rows x ldz bf16 array: the logits (softmax form; the delta is formed from them inside the backward
    // products and never stored) or the output delta (squared-error form, written by the output layer's epilogue)
    u16 *dO = (u16 *)(ws + L.off_do16);
    u16 *Z16 = dO;
    float *zlab = (float *)(ws + L.off_zlab);
    float *row_lse = (float *)(ws + L.off_lse);
    u16 *dA1 = (u16 *)(ws + L.off_da1);
    float *row_loss = (float *)(ws + L.off_rowloss);
    float *part_a = (float *)(ws + L.off_pa);
    float *part_b = (float *)(ws + L.off_pb);

    // weights whose rows are not 16-byte aligned (n_out = 3203) are copied once into aligned rows, both in one launch
    int ldw1 = n_hid, ldw2 = n_out;
    RepackArgs rp{};
    if (!rows_16b_aligned(W1, ldw1)) {
        u16 *W1p = (u16 *)(ws + L.off_w1p);
        rp.part[0] = {W1, W1p, ldw1, L.ldw1p, n_in, n_hid, (int)grid_for((size_t)n_in * n_hid)};
        W1 = W1p;
        ldw1 = L.ldw1p;
    }
    if (!rows_16b_aligned(W2, ldw2)) {
        u16 *W2p = (u16 *)(ws + L.off_w2p);
        rp.part[1] = {W2, W2p, ldw2, L.ldw2p, n_hid, n_out, (int)grid_for((size_t)n_hid * n_out)};
        W2 = W2p;
        ldw2 = L.ldw2p;
    }
    if (rp.part[0].blocks + rp.part[1].blocks > 0)
        hipLaunchKernelGGL(repack16_kernel, dim3((unsigned)(rp.part[0].blocks + rp.part[1].blocks)), dim3(256), 0, s, rp);
    HIP_TRY(hipGetLastError());

    for (int r0 = 0; r0 < batch; r0 += L.slab) {
        const int rows = std::min(L.slab, batch - r0);
        const float beta = (r0 > 0 || accumulate) ? 1.0f : 0.0f;
        const u16 *Xs = X + (size_t)r0 * n_in;
        const int32_t *ys = task.labels ? task.labels + r0 : nullptr;
        const float *ts = task.targets ? task.targets + (size_t)r0 * n_out : nullptr;
        // Patterns whose rows are not 16-byte aligned (n_in no multiple of 8) are copied into aligned rows too, in the upper
        // half of the partial region where they fit there: both products that read them would go element by element
        // otherwise.  A gradient gains from 128 rows on, whatever the width, because its dW1 walks the rows (9-16-10, 300
        // patterns: 45 -> 37 us; 33-64-40, 1000: 50 -> 38; 401-480-3203, 65536: 1319 -> 1082; with 50 rows nothing).  An error
        // alone reads them once, n_in deep: up to two k steps (n_in <= 64) the launch costs what it saves or more (33-64-40,
        // 1000 patterns: 13.8 -> 15.9, 57-128-100, 30000: 26.2 -> 28.0), beyond it gains (65-480-480, 5000: 29.2 -> 25.6;
        // 401-128-64, 160: 32.6 -> 18.5).
        const int ldx_copy = (int)round_up((size_t)n_in, 8);
        const size_t half_pb = L.floats_pb / 2 / 64 * 64;      // floats, 256-byte aligned
        const bool copy_x = !rows_16b_aligned(Xs, n_in) && (task.backward ? rows >= 128 : n_in > 64) &&
                            (size_t)rows * ldx_copy * sizeof(u16) <= half_pb * sizeof(float);
        const size_t floats_pb = copy_x ? half_pb : L.floats_pb;
        // (The copies of the weights and everything in the workspace are aligned.  The hidden layer of patterns that did not come
        // aligned stays on the steps of 32 k, whose sums do not depend on the tile, so that an error with and without gradient has
        // the same whether or not they are copied.)
        const bool x_aligned = rows_16b_aligned(Xs, n_in), softmax = !ts;
        const Rows16 wide = std::max(std::max(n_in, n_hid), n_out) <= WIDE16_MAX_LD - 32 ? ROWS16_WIDE : ROWS16_ALIGNED;
        const Gemm16Plan p1 = plan_gemm16(rows, n_hid, n_in, true, false, false, 0, x_aligned ? wide : copy_x ? ROWS16_ALIGNED : ROWS16_LOOSE);
        const Gemm16Plan p2 = plan_gemm16(rows, n_out, n_hid, true, false, false, 0, wide);
        const Gemm16Plan p3 = plan_gemm16(n_hid, n_out, rows, false, false, true, L.floats_pa, wide, softmax);
        const Gemm16Plan p4 = plan_gemm16(rows, n_hid, n_out, true, true, true, floats_pb, wide, softmax);
        const Gemm16Plan p5 = plan_gemm16(n_in, n_hid, rows, false, false, true, floats_pb, copy_x || x_aligned ? wide : ROWS16_LOOSE);
        Gemm16Args a{};
        MARK(0);

        int ldx = n_in;
        if (copy_x) {
            u16 *Xp = (u16 *)(part_b + half_pb);
            RepackArgs rx{};
            rx.part[0] = {Xs, Xp, n_in, ldx_copy, rows, n_in, (int)grid_for((size_t)rows * n_in)};
            hipLaunchKernelGGL(repack16_kernel, dim3((unsigned)rx.part[0].blocks), dim3(256), 0, s, rx);
            HIP_TRY(hipGetLastError());
            Xs = Xp;
            ldx = ldx_copy;
        }
        // H = tanh(Xs W1 + b1), stored bf16
        a = Gemm16Args{};
        a.A = Xs; a.lda = ldx; a.B = W1; a.ldb = ldw1; a.C = H; a.ldc = L.ldh;
        a.M = rows; a.N = n_hid; a.K = n_in; a.alpha = 1.f; a.bias = d->b1;
        HIP_TRY(launch_gemm16(p1, true, false, EPI_BIAS_TANH, a, s));
        MARK(1);

        // Z = H W2 + b2 rounded to bf16, with the softmax statistics of every row taken from the fp32 accumulators
        // in the product's epilogue (an error-only call writes the statistics alone)
        a = Gemm16Args{};
        a.A = H; a.lda = L.ldh; a.B = W2; a.ldb = ldw2; a.C = ts ? dO : Z16; a.ldc = L.ldz;
        a.M = rows; a.N = n_out; a.K = n_hid; a.alpha = 1.f; a.bias = d->b2;
        a.stats = stats; a.label_logit = zlab; a.labels = ys; a.targets = ts; a.ldt = n_out;
        const int sgw = stat_group_width(p2.cfg);
        a.stat_groups = (n_out + sgw - 1) / sgw;
        a.stat_stride = (size_t)rows;
        if (ts)   // the paper's output stage (tanh, squared error, delta) entirely in the epilogue
            HIP_TRY(launch_gemm16(p2, true, false, task.backward ? EPI_TANH_MSE : EPI_MSE_ONLY, a, s));
        else
            HIP_TRY(launch_gemm16(p2, true, false, task.backward ? EPI_BIAS_STATS : EPI_STATS_ONLY, a, s));
        MARK(2);

        // row losses (and, softmax form, each row's log-sum-exp for the delta); loss (+)= their sum
        if (ts)
            hipLaunchKernelGGL(mse16_finish_kernel, dim3((rows + 63) / 64), dim3(256), 0, s, rows,
                               (const float2 *)stats, a.stat_stride, a.stat_groups, row_loss);
        else
            hipLaunchKernelGGL(softmax16_finish_kernel, dim3((rows + 63) / 64), dim3(256), 0, s, n_out, rows,
                               (const float2 *)stats, a.stat_stride, a.stat_groups, (const float *)zlab, ys, row_loss,
                               row_lse);
        // the loss sum and the reductions of dW2 and dW1 end the pass in one launch, unless there is none of the latter
        const bool final_reduce = task.backward && (p3.splits > 1 || p5.splits > 1);
        if (!final_reduce)
            hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(1024), 0, s, row_loss, (long long)rows, loss, beta);
        HIP_TRY(hipGetLastError());
        MARK(3);
        if (!task.backward) {
            MARK(4); MARK(5); MARK(6); MARK(7); MARK(8);
            continue;
        }

        // dA1 = (dO W2^T) * (1 - H*H), stored bf16, and dW2 (+)= H^T dO.  Softmax form: both products read the
        // LOGITS and form dO = softmax - onehot on the way into LDS; the delta is never stored (no pass over the
        // 2 x batch x n_out bytes of logits and delta, and no write of the delta, which cost the hidden-delta
        // product a third of its time).  Squared-error form: the delta came out of the output layer's epilogue.
        Gemm16Args a4{};
        a4.A = ts ? dO : Z16; a4.lda = L.ldz; a4.B = W2; a4.ldb = ldw2; a4.C = dA1; a4.ldc = L.ldh;
        a4.M = rows; a4.N = n_hid; a4.K = n_out; a4.alpha = 1.f; a4.aux = H; a4.ldaux = L.ldh;
        Gemm16Args a3{};
        a3.A = H; a3.lda = L.ldh; a3.B = ts ? dO : Z16; a3.ldb = L.ldz; a3.C = dW2; a3.ldc = n_out;
        a3.M = n_hid; a3.N = n_out; a3.K = rows; a3.alpha = 1.f; a3.beta = beta;
        if (!ts) {
            a4.row_lse = row_lse; a4.labels = ys;
            a3.row_lse = row_lse; a3.labels = ys;
        }
        {
            Gemm16Args q4 = a4, q3 = a3;
            if (p4.splits > 1) { q4.C = part_b; q4.partial_stride = (size_t)a4.M * a4.N; }
            if (p3.splits > 1) { q3.C = part_a; q3.partial_stride = (size_t)a3.M * a3.N; }
            HIP_TRY(launch_gemm16(p4, true, true, p4.splits > 1 ? EPI_PARTIAL : EPI_TANHGRAD, q4, s));
            HIP_TRY(launch_gemm16(p3, false, false, p3.splits > 1 ? EPI_PARTIAL : EPI_AXPBY, q3, s));
        }
        MARK(4);
        if (p4.splits > 1) {
            const size_t total = (size_t)a4.M * a4.N;
            hipLaunchKernelGGL((splitk_reduce_kernel<true, true>), dim3(grid_for(total)), dim3(256), 0, s, part_b, total,
                               p4.splits, (void *)dA1, a4.M, a4.N, a4.ldc, 1.0f, 0.0f, (const void *)H, L.ldh);
        }
        HIP_TRY(hipGetLastError());
        MARK(5);

        // dW1 (+)= Xs^T dA1
        a = Gemm16Args{};
        a.A = Xs; a.lda = ldx; a.B = dA1; a.ldb = L.ldh; a.C = dW1; a.ldc = n_hid;
        a.M = n_in; a.N = n_hid; a.K = rows; a.alpha = 1.f; a.beta = beta;
        {
            Gemm16Args q5 = a;   // (the hidden delta's slices are summed: its region is free for dW1's)
            if (p5.splits > 1) { q5.C = part_b; q5.partial_stride = (size_t)a.M * a.N; }
            HIP_TRY(launch_gemm16(p5, false, false, p5.splits > 1 ? EPI_PARTIAL : EPI_AXPBY, q5, s));
        }
        MARK(6);
        if (final_reduce) {
            FinalReduceArgs f{};
            f.part[0] = reduce_part(p3.splits, a3.M, a3.N, a3.ldc, dW2, part_a);
            f.part[1] = reduce_part(p5.splits, a.M, a.N, a.ldc, dW1, part_b);
            f.row_loss = row_loss; f.rows = rows; f.loss = loss; f.beta = beta;
            hipLaunchKernelGGL(final_reduce_kernel, dim3((unsigned)(1 + f.part[0].blocks + f.part[1].blocks)), dim3(256), 0, s, f);
            HIP_TRY(hipGetLastError());
        }
        MARK(7);

        if (biases) {
            ColumnSumArgs c{};
            c.D[0] = ts ? dO : Z16; c.ld[0] = L.ldz; c.D[1] = dA1; c.ld[1] = L.ldh;
            c.row_lse = row_lse; c.labels = ys;
            if (ts) HIP_TRY(launch_column_sums<COLUMNS_BF16>(c, d, rows, part_a, L.floats_pa, beta, s));
            else HIP_TRY(launch_column_sums<COLUMNS_BF16_DELTA>(c, d, rows, part_a, L.floats_pa, beta, s));
        }
        MARK(8);
    }
    return ULSNN_OK;
}

}  // namespace

// ---------------------------------------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------------------------------------

extern "C" {

int ulsnn_sgemm(char transa, char transb, int m, int n, int k, float alpha, const float *A, int lda,
                const float *B, int ldb, float beta, float *C, int ldc, void *hip_stream)
{
    if (!(is_n(transa) || is_t(transa)) || !(is_n(transb) || is_t(transb))) return ULSNN_ERR_TRANS;
    if (m < 0 || n < 0 || k < 0) return ULSNN_ERR_DIM;
    const int cols_a = is_n(transa) ? k : m;
    const int cols_b = is_n(transb) ? n : k;
    if (lda < std::max(1, cols_a) || ldb < std::max(1, cols_b) || ldc < std::max(1, n)) return ULSNN_ERR_LD;
    if (lda > ULSNN_MAX_LD || ldb > ULSNN_MAX_LD) return ULSNN_ERR_UNSUPPORTED;   // 32-bit offsets inside a tile
    if (m == 0 || n == 0) return ULSNN_OK;
    if (!C) return ULSNN_ERR_NULL;
    hipStream_t s = (hipStream_t)hip_stream;
    if (k == 0 || alpha == 0.0f) {
        if (beta == 1.0f) return ULSNN_OK;
        hipLaunchKernelGGL(scale_kernel, dim3(grid_for((size_t)m * n)), dim3(256), 0, s, C, m, n, ldc, beta);
        return hipGetLastError() == hipSuccess ? ULSNN_OK : ULSNN_ERR_HIP;
    }
    if (!A || !B) return ULSNN_ERR_NULL;
    const GemmPlan p = plan_sgemm(m, n, k, is_n(transa), is_t(transb), lda, ldb);
    GemmArgs a{};
    a.A = A; a.B = B; a.C = C; a.M = m; a.N = n; a.K = k; a.lda = lda; a.ldb = ldb; a.ldc = ldc;
    a.alpha = alpha; a.beta = beta;
    return launch_plan(p, is_n(transa), is_t(transb), EPI_AXPBY, a, s) == hipSuccess ? ULSNN_OK : ULSNN_ERR_HIP;
}

int ulsnn_sgemm_ws(char transa, char transb, int m, int n, int k, float alpha, const float *A, int lda,
                   const float *B, int ldb, float beta, float *C, int ldc, void *workspace, size_t workspace_bytes,
                   void *hip_stream)
{
    if (!(is_n(transa) || is_t(transa)) || !(is_n(transb) || is_t(transb))) return ULSNN_ERR_TRANS;
    if (m < 0 || n < 0 || k < 0) return ULSNN_ERR_DIM;
    const int cols_a = is_n(transa) ? k : m;
    const int cols_b = is_n(transb) ? n : k;
    if (lda < std::max(1, cols_a) || ldb < std::max(1, cols_b) || ldc < std::max(1, n)) return ULSNN_ERR_LD;
    if (lda > ULSNN_MAX_LD || ldb > ULSNN_MAX_LD) return ULSNN_ERR_UNSUPPORTED;
    if (workspace_bytes > 0 && (!workspace || ((uintptr_t)workspace & 255) != 0)) return ULSNN_ERR_WORKSPACE;
    if (m == 0 || n == 0 || k == 0 || alpha == 0.0f)
        return ulsnn_sgemm(transa, transb, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, hip_stream);
    if (!C || !A || !B) return ULSNN_ERR_NULL;
    // as many k slices as the planner likes and the workspace can hold partial products for
    const size_t slices = workspace_bytes / ((size_t)m * n * sizeof(float));
    const GemmPlan p = plan_sgemm_ws(m, n, k, is_n(transa), is_t(transb), lda, ldb, slices);
    hipStream_t s = (hipStream_t)hip_stream;
    GemmArgs a{};
    a.A = A; a.B = B; a.C = C; a.M = m; a.N = n; a.K = k; a.lda = lda; a.ldb = ldb; a.ldc = ldc;
    a.alpha = alpha; a.beta = beta;
    if (p.splits == 1)
        return launch_plan(p, is_n(transa), is_t(transb), EPI_AXPBY, a, s) == hipSuccess ? ULSNN_OK : ULSNN_ERR_HIP;
    GemmArgs q = a;
    q.C = (float *)workspace;
    q.partial_stride = (size_t)m * n;
    if (launch_plan(p, is_n(transa), is_t(transb), EPI_PARTIAL, q, s) != hipSuccess) return ULSNN_ERR_HIP;
    return launch_reduce(p.splits, EPI_AXPBY, a, (const float *)workspace, s) == hipSuccess ? ULSNN_OK : ULSNN_ERR_HIP;
}

size_t ulsnn_mlp_grad_workspace_bytes(const ulsnn_mlp_desc *desc, int batch)
{
    if (!desc_ok(desc) || batch < 0) return 0;
    if (batch == 0) return 0;
    return mlp_layout(desc, batch).bytes;
}

int ulsnn_mlp_grad(const ulsnn_mlp_desc *desc, const void *W1, const void *W2, const void *X,
                   const int32_t *labels, int batch, float *dW1, float *dW2, float *loss)
{
    const int rc = check_mlp_args(desc, W1, W2, X, labels, batch, dW1, dW2, loss, true);
    if (rc != ULSNN_OK) return rc;
    return mlp_grad_impl(desc, W1, W2, X, MlpTask{labels, nullptr, true}, batch, dW1, dW2, loss,
                         desc->accumulate != 0);
}

// Device address of `scratch` on the current device, resolved once per device.
static int static_scratch(void **out)
{
    constexpr int MAX_DEVICES = 64;
    static std::mutex mu;
    static void *address[MAX_DEVICES] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return ULSNN_ERR_HIP;
    std::lock_guard<std::mutex> lock(mu);
    if (!address[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return ULSNN_ERR_HIP;
        address[dev] = p;
    }
    *out = address[dev];
    return ULSNN_OK;
}

size_t ulsnn_static_scratch_bytes(void) { return (size_t)ULSNN_STATIC_SCRATCH_BYTES; }

int ulsnn_static_scratch_init(void)
{
    void *p = nullptr;
    return static_scratch(&p);
}

int ulsnn_mlp_grad_static(const ulsnn_mlp_desc *desc, const void *W1, const void *W2, const void *X,
                          const int32_t *labels, int batch, float *dW1, float *dW2, float *loss)
{
    const int rc = check_mlp_args(desc, W1, W2, X, labels, batch, dW1, dW2, loss, true);
    if (rc != ULSNN_OK) return rc;
    if (batch > 0 && mlp_layout(desc, batch).bytes > (size_t)ULSNN_STATIC_SCRATCH_BYTES) return ULSNN_ERR_WORKSPACE;
    ulsnn_mlp_desc d = *desc;
    const int rs = static_scratch(&d.workspace);
    if (rs != ULSNN_OK) return rs;
    d.workspace_bytes = (size_t)ULSNN_STATIC_SCRATCH_BYTES;
    return mlp_grad_impl(&d, W1, W2, X, MlpTask{labels, nullptr, true}, batch, dW1, dW2, loss, d.accumulate != 0);
}

int ulsnn_check_labels(const int32_t *labels, int64_t batch, int n_out, int64_t *count, void *hip_stream)
{
    if (batch < 0 || n_out < 1) return ULSNN_ERR_DIM;
    if (!count || (batch > 0 && !labels)) return ULSNN_ERR_NULL;
    hipLaunchKernelGGL(count_ignored_labels_kernel, dim3(1), dim3(1024), 0, (hipStream_t)hip_stream, labels,
                       (long long)batch, n_out, (long long *)count);
    return hipGetLastError() == hipSuccess ? ULSNN_OK : ULSNN_ERR_HIP;
}

int ulsnn_mlp_loss(const ulsnn_mlp_desc *desc, const void *W1, const void *W2, const void *X,
                   const int32_t *labels, int batch, float *loss)
{
    const int rc = check_mlp_args(desc, W1, W2, X, labels, batch, nullptr, nullptr, loss, false);
    if (rc != ULSNN_OK) return rc;
    return mlp_grad_impl(desc, W1, W2, X, MlpTask{labels, nullptr, false}, batch, nullptr, nullptr, loss,
                         desc->accumulate != 0);
}

int ulsnn_mlp_grad_mse(const ulsnn_mlp_desc *desc, const void *W1, const void *W2, const void *X, const float *T,
                       int batch, float *dW1, float *dW2, float *loss)
{
    const int rc = check_mlp_args(desc, W1, W2, X, T, batch, dW1, dW2, loss, true);
    if (rc != ULSNN_OK) return rc;
    return mlp_grad_impl(desc, W1, W2, X, MlpTask{nullptr, T, true}, batch, dW1, dW2, loss, desc->accumulate != 0);
}

int ulsnn_mlp_mse(const ulsnn_mlp_desc *desc, const void *W1, const void *W2, const void *X, const float *T,
                  int batch, float *loss)
{
    const int rc = check_mlp_args(desc, W1, W2, X, T, batch, nullptr, nullptr, loss, false);
    if (rc != ULSNN_OK) return rc;
    return mlp_grad_impl(desc, W1, W2, X, MlpTask{nullptr, T, false}, batch, nullptr, nullptr, loss,
                         desc->accumulate != 0);
}

int ulsnn_mlp_grad_epoch(const ulsnn_mlp_desc *desc, const void *W1, const void *W2, const void *X,
                         const int32_t *labels, int64_t n_patterns, int chunk, float *dW1, float *dW2,
                         float *loss)
{
    const int rc = check_mlp_args(desc, W1, W2, X, labels, (long long)n_patterns, dW1, dW2, loss, true);
    if (rc != ULSNN_OK) return rc;
    if (chunk < 1) return ULSNN_ERR_DIM;
    if (n_patterns == 0)
        return mlp_grad_impl(desc, W1, W2, nullptr, MlpTask{nullptr, nullptr, true}, 0, dW1, dW2, loss,
                             desc->accumulate != 0);
    const int first = (int)std::min<int64_t>(chunk, n_patterns);
    if (!desc->workspace || ((uintptr_t)desc->workspace & 255) ||
        desc->workspace_bytes < ulsnn_mlp_grad_workspace_bytes(desc, first))
        return ULSNN_ERR_WORKSPACE;
    const size_t elem = desc->operand_dtype == 1 ? 2 : 4;
    for (int64_t p0 = 0; p0 < n_patterns; p0 += chunk) {
        const int rows = (int)std::min<int64_t>(chunk, n_patterns - p0);
        const int r = mlp_grad_impl(desc, W1, W2, (const char *)X + (size_t)p0 * desc->n_in * elem,
                                    MlpTask{labels + p0, nullptr, true}, rows, dW1, dW2, loss,
                                    p0 > 0 || desc->accumulate != 0);
        if (r != ULSNN_OK) return r;
    }
    return ULSNN_OK;
}

int ulsnn_mlp_grad_timed(const ulsnn_mlp_desc *desc, const void *W1, const void *W2, const void *X,
                         const int32_t *labels, int batch, float *dW1, float *dW2, float *loss, float *stage_ms)
{
    const int rc = check_mlp_args(desc, W1, W2, X, labels, batch, dW1, dW2, loss, true);
    if (rc != ULSNN_OK) return rc;
    if (!stage_ms) return ULSNN_ERR_NULL;
    if (batch < 1 || batch > SLAB_ROWS) return ULSNN_ERR_UNSUPPORTED;   // one internal pass only
    hipEvent_t ev[ULSNN_MLP_STAGES + 1];
    int made = 0, out = ULSNN_OK;
    for (; made <= ULSNN_MLP_STAGES; ++made)
        if (hipEventCreate(&ev[made]) != hipSuccess) { out = ULSNN_ERR_HIP; break; }
    if (out == ULSNN_OK)
        out = mlp_grad_impl(desc, W1, W2, X, MlpTask{labels, nullptr, true}, batch, dW1, dW2, loss,
                            desc->accumulate != 0, ev);
    if (out == ULSNN_OK && hipEventSynchronize(ev[ULSNN_MLP_STAGES]) != hipSuccess) out = ULSNN_ERR_HIP;
    if (out == ULSNN_OK)
        for (int i = 0; i < ULSNN_MLP_STAGES; ++i)
            if (hipEventElapsedTime(&stage_ms[i], ev[i], ev[i + 1]) != hipSuccess) out = ULSNN_ERR_HIP;
    for (int i = 0; i < made; ++i) (void)hipEventDestroy(ev[i]);
    return out;
}

// ---------------------------------------------------------------------------------------------------------
// Optimiser step (section 4.2, last paragraph): vector primitives, Polak-Ribiere direction, line search
// ---------------------------------------------------------------------------------------------------------

namespace {

inline unsigned vec_grid(size_t n) { return (unsigned)std::min<size_t>((n + 255) / 256, (size_t)VEC_MAX_BLOCKS); }

inline bool vec_ws_ok(const void *ws, size_t bytes)
{
    return ws && ((uintptr_t)ws & 255) == 0 && bytes >= (size_t)ULSNN_VEC_WORKSPACE_BYTES;
}

// *out (device) = x . y
hipError_t launch_dot(size_t n, const float *x, const float *y, float *out, double *partial, hipStream_t s)
{
    const unsigned nb = vec_grid(n);
    if (vec_aligned(x, y)) hipLaunchKernelGGL((dot_partial_kernel<false, true>), dim3(nb), dim3(256), 0, s, n, x, y, partial);
    else hipLaunchKernelGGL((dot_partial_kernel<false, false>), dim3(nb), dim3(256), 0, s, n, x, y, partial);
    hipLaunchKernelGGL(dot_final_kernel, dim3(1), dim3(256), 0, s, (const double *)partial, (int)nb, out);
    return hipGetLastError();
}

struct LsLayout {
    size_t mlp_bytes, n1, n2;
    size_t off_w1, off_w2, off_g1, off_g2, off_vec, off_scalars, bytes;
};

LsLayout ls_layout(const ulsnn_mlp_desc *d, int batch)
{
    LsLayout L{};
    L.mlp_bytes = round_up(mlp_layout(d, batch).bytes, 256);
    L.n1 = (size_t)d->n_in * d->n_hid;
    L.n2 = (size_t)d->n_hid * d->n_out;
    size_t off = L.mlp_bytes;
    L.off_w1 = off; off += round_up(L.n1 * 4, 256);
    L.off_w2 = off; off += round_up(L.n2 * 4, 256);
    L.off_g1 = off; off += round_up(L.n1 * 4, 256);
    L.off_g2 = off; off += round_up(L.n2 * 4, 256);
    L.off_vec = off; off += round_up((size_t)ULSNN_VEC_WORKSPACE_BYTES, 256);
    L.off_scalars = off; off += 256;
    L.bytes = off;
    return L;
}

// Layout of the batched slopes inside the (otherwise idle) gradient workspace, and how many steps fit at once: 0 if not even
// one does (a subset close to the whole batch of a wide network), then the slopes come from gradients.  So they do where the
// stacked product's extra work, 8 n_hid n_out flop per pattern against a gradient's 6 n_hid n_out + 4 n_in n_hid, outweighs
// its fewer launches: above 15 GFLOP.  Whole searches over 20000 patterns, stacked and with gradients: 400-480-3203 (2.3
// MFLOP per pattern) on a subset of 5500 10.7 and 11.5 ms, 6500 12.3 and 12.7, 8192 14.8 and 14.3; 64-256-4096 on 6500 9.0
// and 9.1, 8192 10.9 and 9.8, 12000 15.3 and 13.2.  Networks of few classes do less work stacked, at any size.
struct SlopeLayout {
    int rows, ldp, lda, ldu;
    int steps;
    size_t off_p, off_q, off_b, off_value, off_a, off_u;
};

SlopeLayout slope_layout(const ulsnn_mlp_desc *d, int rows, size_t bytes)
{
    SlopeLayout S{};
    S.rows = rows;
    S.ldp = (int)round_up((size_t)d->n_hid, 32);
    S.lda = (int)round_up(2 * (size_t)d->n_hid, 32);
    S.ldu = (int)round_up((size_t)d->n_out, 32);
    if (rows > SLAB_ROWS || d->n_hid > ULSNN_MAX_LD / 2) return S;
    if ((double)rows * d->n_hid * (2.0 * d->n_out - 4.0 * d->n_in) > 15.0e9) return S;
    size_t off = 0;
    S.off_p = off; off += round_up((size_t)rows * S.ldp * 4, 256);
    S.off_q = off; off += round_up((size_t)rows * S.ldp * 4, 256);
    S.off_b = off; off += round_up(2 * (size_t)d->n_hid * d->n_out * 4, 256);
    S.off_value = off; off += round_up((size_t)LS_GROUP * rows * 8, 256);
    const size_t per_step = 2 * (size_t)rows * (S.lda + S.ldu) * 4;     // a step's rows of the two stacked matrices
    if (off + per_step + 512 > bytes) return S;
    S.steps = (int)std::min<size_t>(LS_GROUP, (bytes - off - 512) / per_step);
    S.off_a = off;
    S.off_u = off + round_up((size_t)S.steps * 2 * rows * S.lda * 4, 256);
    return S;
}

}  // namespace

int ulsnn_dot(int64_t n, const float *x, const float *y, float *result, void *workspace, size_t workspace_bytes,
              void *hip_stream)
{
    if (n < 0) return ULSNN_ERR_DIM;
    if (!result || (n > 0 && (!x || !y))) return ULSNN_ERR_NULL;
    if (!vec_ws_ok(workspace, workspace_bytes)) return ULSNN_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)hip_stream;
    if (n == 0) {
        hipLaunchKernelGGL(zero_kernel, dim3(1), dim3(256), 0, s, result, (size_t)1);
        return hipGetLastError() == hipSuccess ? ULSNN_OK : ULSNN_ERR_HIP;
    }
    return launch_dot((size_t)n, x, y, result, (double *)workspace, s) == hipSuccess ? ULSNN_OK : ULSNN_ERR_HIP;
}

int ulsnn_axpy(int64_t n, float alpha, const float *x, float *y, void *hip_stream)
{
    if (n < 0) return ULSNN_ERR_DIM;
    if (n == 0) return ULSNN_OK;
    if (!x || !y) return ULSNN_ERR_NULL;
    const dim3 grid(grid_for((size_t)n / 4 + 1));
    if (vec_aligned(x, y)) hipLaunchKernelGGL(add_scaled_kernel<true>, grid, dim3(256), 0, (hipStream_t)hip_stream, (size_t)n, (const float *)y, alpha, x, y);
    else hipLaunchKernelGGL(add_scaled_kernel<false>, grid, dim3(256), 0, (hipStream_t)hip_stream, (size_t)n, (const float *)y, alpha, x, y);
    return hipGetLastError() == hipSuccess ? ULSNN_OK : ULSNN_ERR_HIP;
}

int ulsnn_cg_direction(int64_t n, const float *g_new, const float *g_old, float *d, float *beta, void *workspace,
                       size_t workspace_bytes, void *hip_stream)
{
    if (n < 0) return ULSNN_ERR_DIM;
    if (n > 0 && (!g_new || !d)) return ULSNN_ERR_NULL;
    if (!vec_ws_ok(workspace, workspace_bytes)) return ULSNN_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)hip_stream;
    double *partial = (double *)workspace;
    static_assert(2 * CG_MAX_BLOCKS * sizeof(double) <= ULSNN_VEC_WORKSPACE_BYTES, "partial sums fit the workspace");
    if (n == 0) {
        if (beta) hipLaunchKernelGGL(zero_kernel, dim3(1), dim3(256), 0, s, beta, (size_t)1);
        return hipGetLastError() == hipSuccess ? ULSNN_OK : ULSNN_ERR_HIP;
    }
    const size_t len = (size_t)n;
    const unsigned nb = g_old ? std::min<unsigned>(vec_grid(len / 4 + 1), CG_MAX_BLOCKS) : 0;
    const bool vec = vec_aligned(g_new, g_old, d);
    if (g_old) {
        if (vec) hipLaunchKernelGGL((dot_partial_kernel<true, true>), dim3(nb), dim3(256), 0, s, len, g_new, g_old, partial);
        else hipLaunchKernelGGL((dot_partial_kernel<true, false>), dim3(nb), dim3(256), 0, s, len, g_new, g_old, partial);
    }
    const dim3 grid(std::min<unsigned>(grid_for(len / 4 + 1), 2 * CG_MAX_BLOCKS));
    if (vec) hipLaunchKernelGGL(cg_update_kernel<true>, grid, dim3(256), 0, s, len, g_new, d, (const double *)partial, (int)nb, beta);
    else hipLaunchKernelGGL(cg_update_kernel<false>, grid, dim3(256), 0, s, len, g_new, d, (const double *)partial, (int)nb, beta);
    return hipGetLastError() == hipSuccess ? ULSNN_OK : ULSNN_ERR_HIP;
}

size_t ulsnn_mlp_line_search_workspace_bytes(const ulsnn_mlp_desc *desc, int batch)
{
    if (!desc_ok(desc) || batch < 1) return 0;
    return ls_layout(desc, batch).bytes;
}

int ulsnn_mlp_line_search(const ulsnn_mlp_desc *desc, float *W1, float *W2, const float *d1, const float *d2,
                          const float *X, const int32_t *labels, int batch, int bracket_batch, float alpha0,
                          int max_doublings, ulsnn_line_search_result *result)
{
    if (!desc || !result) return ULSNN_ERR_NULL;
    if (!desc_ok(desc) || batch < 1 || bracket_batch < 1 || max_doublings < 0 || max_doublings > 60 ||
        !(alpha0 > 0.0f) || !std::isfinite(alpha0))
        return ULSNN_ERR_DIM;
    if (!W1 || !W2 || !d1 || !d2 || !X || !labels) return ULSNN_ERR_NULL;
    if (desc->b1 || desc->b2 || desc->db1 || desc->db2 || desc->operand_dtype != 0) return ULSNN_ERR_UNSUPPORTED;
    const LsLayout L = ls_layout(desc, batch);
    if (!desc->workspace || ((uintptr_t)desc->workspace & 255) != 0 || desc->workspace_bytes < L.bytes)
        return ULSNN_ERR_WORKSPACE;
    char *base = (char *)desc->workspace;
    float *T1 = (float *)(base + L.off_w1), *T2 = (float *)(base + L.off_w2);
    float *G1 = (float *)(base + L.off_g1), *G2 = (float *)(base + L.off_g2);
    double *partial = (double *)(base + L.off_vec);
    static_assert(sizeof(LineSearchScalars) <= 256, "scalars fit their workspace slot");
    LineSearchScalars *scal = (LineSearchScalars *)(base + L.off_scalars);
    hipStream_t s = (hipStream_t)desc->hip_stream;
    ulsnn_mlp_desc sub = *desc;
    sub.workspace = base;
    sub.workspace_bytes = L.mlp_bytes;
    sub.accumulate = 0;
    const int nsub = std::min(bracket_batch, batch);
    const unsigned wgrid = grid_for(L.n1 + L.n2);

    // weights at step alpha: the caller's own for alpha == 0, else T = W + alpha d (alpha from the host, or, with
    // alpha_dev, a step the device chose)
    auto weights_at = [&](double alpha, const float *alpha_dev, const float *&w1, const float *&w2) -> hipError_t {
        if (!alpha_dev && alpha == 0.0) {
            w1 = W1; w2 = W2;
            return hipSuccess;
        }
        hipLaunchKernelGGL(add_scaled2_kernel, dim3(wgrid), dim3(256), 0, s, L.n1, (const float *)W1, d1, T1, L.n2,
                           (const float *)W2, d2, T2, (float)alpha, alpha_dev);
        w1 = T1; w2 = T2;
        return hipGetLastError();
    };
    // E(W + alpha d) over all `batch` patterns (one error evaluation, section 6.2), left in *out on the device
    auto error_at = [&](double alpha, const float *alpha_dev, float *out) -> int {
        const float *w1, *w2;
        HIP_TRY(weights_at(alpha, alpha_dev, w1, w2));
        return mlp_grad_impl(&sub, w1, w2, X, MlpTask{labels, nullptr, false}, batch, nullptr, nullptr, out, false);
    };
    // grad E_sub(W + alpha d) . d on the first nsub patterns, left in *out on the device: only its sign is used
    auto slope_at = [&](double alpha, float *out) -> int {
        const float *w1, *w2;
        HIP_TRY(weights_at(alpha, nullptr, w1, w2));
        const int rc = mlp_grad_impl(&sub, w1, w2, X, MlpTask{labels, nullptr, true}, nsub, G1, G2, &scal->E[4], false);
        if (rc != ULSNN_OK) return rc;
        const unsigned nb = vec_grid(L.n1 + L.n2);
        hipLaunchKernelGGL(dot2_partial_kernel, dim3(nb), dim3(256), 0, s, L.n1, (const float *)G1, d1, L.n2,
                           (const float *)G2, d2, partial);
        hipLaunchKernelGGL(dot_final_kernel, dim3(1), dim3(256), 0, s, (const double *)partial, (int)nb, out);
        HIP_TRY(hipGetLastError());
        return ULSNN_OK;
    };

    // The slopes of `cnt` steps, left in scal->slope[0..cnt): from one stacked product (line_search.hpp) where the
    // workspace holds it, else one gradient per step.
    const SlopeLayout B = slope_layout(desc, nsub, L.mlp_bytes);
    float *P = (float *)(base + B.off_p), *Q = (float *)(base + B.off_q), *W2d2 = (float *)(base + B.off_b);
    double *row_value = (double *)(base + B.off_value);
    const int n_in = desc->n_in, n_hid = desc->n_hid, n_out = desc->n_out;
    auto prepare_slopes = [&]() -> int {
        GemmArgs a{};
        a.A = X; a.lda = n_in; a.ldb = n_hid; a.ldc = B.ldp; a.M = nsub; a.N = n_hid; a.K = n_in; a.alpha = 1.f;
        const GemmPlan p = plan_product(nsub, n_hid, n_in, true, false, n_in, n_hid, 1);
        a.B = W1; a.C = P;
        HIP_TRY(launch_plan(p, true, false, EPI_BIAS, a, s));
        a.B = d1; a.C = Q;
        HIP_TRY(launch_plan(p, true, false, EPI_BIAS, a, s));
        HIP_TRY(hipMemcpyAsync(W2d2, W2, L.n2 * 4, hipMemcpyDeviceToDevice, s));
        HIP_TRY(hipMemcpyAsync(W2d2 + L.n2, d2, L.n2 * 4, hipMemcpyDeviceToDevice, s));
        return ULSNN_OK;
    };
    auto slopes_at = [&](const double *alpha, int cnt) -> int {
        if (B.steps == 0) {
            int rc = ULSNN_OK;
            for (int j = 0; j < cnt && rc == ULSNN_OK; ++j) rc = slope_at(alpha[j], &scal->slope[j]);
            return rc;
        }
        for (int j0 = 0; j0 < cnt; j0 += B.steps) {
            LineSearchSteps steps{};
            steps.count = std::min(B.steps, cnt - j0);
            for (int j = 0; j < steps.count; ++j) steps.alpha[j] = (float)alpha[j0 + j];
            float *A = (float *)(base + B.off_a), *U = (float *)(base + B.off_u);
            const size_t half = (size_t)steps.count * nsub;
            hipLaunchKernelGGL(ls_stack_kernel, dim3(grid_for((size_t)nsub * n_hid)), dim3(256), 0, s, (const float *)P,
                               (const float *)Q, B.ldp, nsub, n_hid, steps, A, B.lda);
            GemmArgs a{};
            a.A = A; a.lda = B.lda; a.B = W2d2; a.ldb = n_out; a.C = U; a.ldc = B.ldu;
            a.M = (int)(2 * half); a.N = n_out; a.K = 2 * n_hid; a.alpha = 1.f;
            HIP_TRY(launch_plan(plan_product(a.M, n_out, a.K, true, false, B.lda, n_out, 1), true, false, EPI_BIAS, a, s));
            hipLaunchKernelGGL(ls_slope_row_kernel, dim3((unsigned)((half + 3) / 4)), dim3(256), 0, s, (const float *)U, B.ldu, half, nsub,
                               n_out, labels, row_value);
            hipLaunchKernelGGL(ls_slope_sum_kernel, dim3((unsigned)steps.count), dim3(256), 0, s, (const double *)row_value,
                               nsub, &scal->slope[j0]);
            HIP_TRY(hipGetLastError());
        }
        return ULSNN_OK;
    };

    // The host reads device scalars only where it must decide what to launch next: once per group of GROUP
    // bracketing steps (the steps of a group are evaluated whether or not an earlier one of the group already
    // closed the bracket: a few spare evaluations on the small subset instead of a round trip each), and once at
    // the end.  Vertex, comparison of the errors and the weight update use steps the device computes.
    constexpr int GROUP = LS_GROUP;                   // largest group; the first two hold 2 and 4 steps
    int rc;
    if ((rc = error_at(0.0, nullptr, &scal->E[0])) != ULSNN_OK) return rc;
    if (B.steps > 0 && (rc = prepare_slopes()) != ULSNN_OK) return rc;
    double lo = 0.0, hi = alpha0, prev = 0.0;
    int n_grad = 0;
    bool closed = false;
    int size = 2;
    for (int k0 = 0; k0 <= max_doublings && !closed; k0 += size, size = std::min(2 * size, GROUP)) {
        const int cnt = std::min(size, max_doublings + 1 - k0);
        double alpha[GROUP];
        for (int j = 0; j < cnt; ++j) alpha[j] = (double)alpha0 * std::ldexp(1.0, k0 + j);
        if ((rc = slopes_at(alpha, cnt)) != ULSNN_OK) return rc;
        float h[GROUP] = {};
        HIP_TRY(hipMemcpyAsync(h, scal->slope, cnt * sizeof(float), hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
        for (int j = 0; j < cnt; ++j) {
            hi = (double)alpha0 * std::ldexp(1.0, k0 + j);
            lo = prev;
            ++n_grad;
            if (h[j] >= 0.0f) { closed = true; break; }
            prev = hi;
        }
    }
    const bool lo_zero = lo == 0.0;
    const double mid = 0.5 * (lo + hi);
    if (!lo_zero && (rc = error_at(lo, nullptr, &scal->E[1])) != ULSNN_OK) return rc;
    if ((rc = error_at(mid, nullptr, &scal->E[2])) != ULSNN_OK) return rc;
    if ((rc = error_at(hi, nullptr, &scal->E[3])) != ULSNN_OK) return rc;
    hipLaunchKernelGGL(ls_vertex_kernel, dim3(1), dim3(1), 0, s, scal, (int)lo_zero, (float)lo, (float)hi);
    HIP_TRY(hipGetLastError());
    if ((rc = error_at(0.0, &scal->q, &scal->E[4])) != ULSNN_OK) return rc;   // at the vertex (at mid again if not convex)
    hipLaunchKernelGGL(ls_pick_kernel, dim3(1), dim3(1), 0, s, scal, (int)lo_zero, (float)lo, (float)hi);
    hipLaunchKernelGGL(add_scaled2_kernel, dim3(wgrid), dim3(256), 0, s, L.n1, (const float *)W1, d1, W1, L.n2,
                       (const float *)W2, d2, W2, 0.0f, (const float *)&scal->alpha);
    HIP_TRY(hipGetLastError());
    LineSearchScalars host{};
    HIP_TRY(hipMemcpyAsync(&host, scal, sizeof(host), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    result->alpha = host.alpha;
    result->loss = host.loss;
    result->loss0 = host.E[0];
    result->bracket_lo = (float)lo;
    result->bracket_hi = (float)hi;
    result->error_evaluations = 1 + (lo_zero ? 0 : 1) + 2 + (host.convex ? 1 : 0);   // the algorithm's own count
    result->gradient_evaluations = n_grad;
    return ULSNN_OK;
}

int ulsnn_mlp_grad_describe_plan(const ulsnn_mlp_desc *desc, int batch, char *buf, size_t buf_bytes)
{
    if (!desc || !buf) return ULSNN_ERR_NULL;
    if (!desc_ok(desc) || batch < 1 || buf_bytes < 1) return ULSNN_ERR_DIM;
    const MlpLayout L = mlp_layout(desc, batch);
    const char *what[5] = {"hidden_layer", "output_layer", "dW2", "hidden_delta", "dW1"};
    size_t used = 0;
    auto add = [&](int n) {
        if (n > 0) used = std::min(used + (size_t)n, buf_bytes - 1);
    };
    auto five_lines = [&](const SlabPlans &P) {
        const GemmPlan *g[5] = {&P.g1, &P.g2, &P.g3, &P.g4, &P.g5};
        for (int i = 0; i < 5 && used + 1 < buf_bytes; ++i)
            add(snprintf(buf + used, buf_bytes - used, "%s: tile=%s tiles=%dx%d splits=%d kchunk=%d model_us=%.1f\n",
                         what[i], plan_name(*g[i]), g[i]->tiles_m, g[i]->tiles_n, g[i]->splits, g[i]->kchunk,
                         g[i]->est_us));
    };
    const SlabPlans P = plan_slab(L, desc->n_in, desc->n_hid, desc->n_out, L.slab);
    // (paired_backward: hidden delta and dW2 in one launch, which no plan does any more; the field stays for its readers)
    add(snprintf(buf, buf_bytes, "rows_per_pass=%d paired_backward=0 workspace_bytes=%zu small_network_path=%d\n",
                 L.slab, L.bytes, (int)small_net_shape(desc, batch)));
    five_lines(P);
    const int tail = batch % L.slab;
    if (tail != 0 && used + 1 < buf_bytes) {
        const SlabPlans T = plan_slab(L, desc->n_in, desc->n_hid, desc->n_out, tail);
        add(snprintf(buf + used, buf_bytes - used, "tail_rows=%d paired_backward=0\n", tail));
        five_lines(T);
    }
    return ULSNN_OK;
}

int ulsnn_sgemm_describe_plan(char transa, char transb, int m, int n, int k, char *buf, size_t buf_bytes)
{
    if (!buf) return ULSNN_ERR_NULL;
    if (!(is_n(transa) || is_t(transa)) || !(is_n(transb) || is_t(transb))) return ULSNN_ERR_TRANS;
    if (m < 1 || n < 1 || k < 1 || buf_bytes < 1) return ULSNN_ERR_DIM;
    const GemmPlan p = plan_sgemm(m, n, k, is_n(transa), is_t(transb), is_n(transa) ? k : m, is_n(transb) ? n : k);
    snprintf(buf, buf_bytes, "tile=%s tiles=%dx%d splits=%d kchunk=%d model_us=%.1f\n", plan_name(p),
             p.tiles_m, p.tiles_n, p.splits, p.kchunk, p.est_us);
    return ULSNN_OK;
}

int ulsnn_sgemm_ws_describe_plan(char transa, char transb, int m, int n, int k, size_t workspace_bytes, char *buf,
                                 size_t buf_bytes)
{
    if (!buf) return ULSNN_ERR_NULL;
    if (!(is_n(transa) || is_t(transa)) || !(is_n(transb) || is_t(transb))) return ULSNN_ERR_TRANS;
    if (m < 1 || n < 1 || k < 1 || buf_bytes < 1) return ULSNN_ERR_DIM;
    const int lda = is_n(transa) ? k : m, ldb = is_n(transb) ? n : k;
    const size_t slices = workspace_bytes / ((size_t)m * n * sizeof(float));
    const GemmPlan p = plan_sgemm_ws(m, n, k, is_n(transa), is_t(transb), lda, ldb, slices);
    const GemmPlan cut = plan_product(m, n, k, is_n(transa), is_t(transb), lda, ldb,
                                      (int)std::min<size_t>(64, std::max<size_t>(1, slices)));
    snprintf(buf, buf_bytes, "tile=%s tiles=%dx%d splits=%d kchunk=%d model_us=%.1f (best split plan: %d slices, %.1f us)\n",
             plan_name(p), p.tiles_m, p.tiles_n, p.splits, p.kchunk, p.est_us, cut.splits, cut.est_us);
    return ULSNN_OK;
}

int ulsnn_sgemm_planned(int tile_shape, int k_splits, char transa, char transb, int m, int n, int k, float alpha,
                        const float *A, int lda, const float *B, int ldb, float beta, float *C, int ldc,
                        void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!(is_n(transa) || is_t(transa)) || !(is_n(transb) || is_t(transb))) return ULSNN_ERR_TRANS;
    if (tile_shape < 0 || tile_shape >= CFG_COUNT || k_splits < 1 || m < 0 || n < 0 || k < 0) return ULSNN_ERR_DIM;
    const int cols_a = is_n(transa) ? k : m;
    const int cols_b = is_n(transb) ? n : k;
    if (lda < std::max(1, cols_a) || ldb < std::max(1, cols_b) || ldc < std::max(1, n)) return ULSNN_ERR_LD;
    if (lda > ULSNN_MAX_LD || ldb > ULSNN_MAX_LD) return ULSNN_ERR_UNSUPPORTED;
    if (m == 0 || n == 0) return ULSNN_OK;
    if (!C) return ULSNN_ERR_NULL;
    hipStream_t s = (hipStream_t)hip_stream;
    if (k == 0 || alpha == 0.0f)
        return ulsnn_sgemm(transa, transb, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, hip_stream);
    if (!A || !B) return ULSNN_ERR_NULL;
    const CfgInfo &c = CFG_INFO[tile_shape];
    GemmPlan p{};
    p.cfg = tile_shape;
    p.tiles_m = (m + c.bm - 1) / c.bm;
    p.tiles_n = (n + c.bn - 1) / c.bn;
    p.kchunk = (int)round_up((size_t)(k + k_splits - 1) / k_splits, c.bk);
    p.splits = (k + p.kchunk - 1) / p.kchunk;
    GemmArgs a{};
    a.A = A; a.B = B; a.C = C; a.M = m; a.N = n; a.K = k; a.lda = lda; a.ldb = ldb; a.ldc = ldc;
    a.alpha = alpha; a.beta = beta;
    if (p.splits == 1)
        return launch_plan(p, is_n(transa), is_t(transb), EPI_AXPBY, a, s) == hipSuccess ? ULSNN_OK : ULSNN_ERR_HIP;
    const size_t need = (size_t)p.splits * m * n * sizeof(float);
    if (!workspace || ((uintptr_t)workspace & 255) != 0 || workspace_bytes < need) return ULSNN_ERR_WORKSPACE;
    GemmArgs q = a;
    q.C = (float *)workspace;
    q.partial_stride = (size_t)m * n;
    if (launch_plan(p, is_n(transa), is_t(transb), EPI_PARTIAL, q, s) != hipSuccess) return ULSNN_ERR_HIP;
    return launch_reduce(p.splits, EPI_AXPBY, a, (const float *)workspace, s) == hipSuccess ? ULSNN_OK : ULSNN_ERR_HIP;
}

int ulsnn_device_info(int *compute_units, int *max_shader_clock_khz, int *wall_clock_khz)
{
    int dev = 0, cu = 0, sclk = 0, wall = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipDeviceGetAttribute(&sclk, hipDeviceAttributeClockRate, dev) != hipSuccess ||
        hipDeviceGetAttribute(&wall, hipDeviceAttributeWallClockRate, dev) != hipSuccess) {
        (void)hipGetLastError();
        return ULSNN_ERR_HIP;
    }
    if (compute_units) *compute_units = cu;
    if (max_shader_clock_khz) *max_shader_clock_khz = sclk;
    if (wall_clock_khz) *wall_clock_khz = wall;
    return ULSNN_OK;
}

int ulsnn_clock_probe(double window_ms, unsigned long long *cycles_and_ticks, void *hip_stream)
{
    if (!cycles_and_ticks) return ULSNN_ERR_NULL;
    if (!(window_ms > 0.0) || window_ms > 1000.0) return ULSNN_ERR_DIM;
    int wall_khz = 0;
    const int rc = ulsnn_device_info(nullptr, nullptr, &wall_khz);
    if (rc != ULSNN_OK) return rc;
    if (wall_khz <= 0) return ULSNN_ERR_UNSUPPORTED;
    const unsigned long long ticks = (unsigned long long)(window_ms * (double)wall_khz);
    // one reading takes well over 100 ns (the sleep alone is 32 x 64 cycles): the cap only guards the exit
    const unsigned int max_iterations = (unsigned int)std::min(1.0e8, window_ms * 2.0e4 + 1000.0);
    hipLaunchKernelGGL(clock_probe_kernel, dim3(1), dim3(64), 0, (hipStream_t)hip_stream, ticks, max_iterations,
                       cycles_and_ticks);
    return hipGetLastError() == hipSuccess ? ULSNN_OK : ULSNN_ERR_HIP;
}

double ulsnn_sgemm_flops(int m, int n, int k) { return 2.0 * (double)m * (double)n * (double)k; }

double ulsnn_mlp_loss_flops(int n_in, int n_hid, int n_out, int64_t batch)
{
    return 2.0 * (double)batch * ((double)n_in + n_out) * n_hid;
}

double ulsnn_mlp_grad_flops(int n_in, int n_hid, int n_out, int64_t batch)
{
    return (double)batch * (4.0 * (double)n_in * n_hid + 6.0 * (double)n_hid * n_out);
}

const char *ulsnn_status_string(int status)
{
    switch (status) {
        case ULSNN_OK: return "ok";
        case ULSNN_ERR_NULL: return "null pointer";
        case ULSNN_ERR_TRANS: return "bad transpose flag";
        case ULSNN_ERR_DIM: return "bad dimension";
        case ULSNN_ERR_LD: return "leading dimension too small";
        case ULSNN_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
        case ULSNN_ERR_UNSUPPORTED: return "option not supported by this build";
        case ULSNN_ERR_HIP: return "HIP launch failed";
        default: return "unknown status";
    }
}

int ulsnn_version(void) { return 100; }

}  // extern "C"
