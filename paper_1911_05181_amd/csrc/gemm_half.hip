// Kernels of the two-term f16 split (gemm_half.hpp) for every tile shape, layout and epilogue.
#include "gemm_half.hpp"
#include "gemm_launch.hpp"

namespace ulsnn {
namespace {

using Hp256x256 = HalfTile<256, 256, 4, 2, 2>;    // 512 threads, 1 workgroup / CU: sub-tiles of 64 x 128
using Hp256x128 = HalfTile<256, 128, 8, 2, 4>;    // 1024 threads, 1 workgroup / CU: 32 x 64
using Hp128w8 = HalfTile<128, 128, 4, 2, 4>;      // 512 threads, 2 workgroups / CU: 32 x 64
using Hp128 = HalfTile<128, 128, 2, 2, 2>;        // 256 threads, 2 workgroups / CU: 64 x 64
using Hp128x64 = HalfTile<128, 64, 4, 2, 4>;      // 512 threads, 2 workgroups / CU: 32 x 32
using Hp64x128 = HalfTile<64, 128, 2, 4, 4>;
using Hp64 = HalfTile<64, 64, 2, 2, 4>;           // 256 threads, 4 workgroups / CU: 32 x 32

template <class F>
hipError_t with_half_cfg(int id, F &&f)
{
    switch (id) {
        case HP_256x256: return f(Hp256x256{});
        case HP_256x128: return f(Hp256x128{});
        case HP_128W8: return f(Hp128w8{});
        case HP_128: return f(Hp128{});
        case HP_128x64: return f(Hp128x64{});
        case HP_64x128: return f(Hp64x128{});
        default: return f(Hp64{});
    }
}

template <class Cfg, bool A_KC, bool B_KC, int EPI>
hipError_t launch_half_one(const GemmArgs &a, int splits, hipStream_t s)
{
    const dim3 grid((unsigned)(a.tiles_m * a.tiles_n), (unsigned)splits);
    hipLaunchKernelGGL((half_kernel<Cfg, A_KC, B_KC, EPI>), grid, dim3(Cfg::THREADS), 0, s, a);
    return hipGetLastError();
}

template <class Cfg, int EPI>
hipError_t launch_half_layout(bool a_kc, bool b_kc, const GemmArgs &a, int splits, hipStream_t s)
{
    if (a_kc && !b_kc) return launch_half_one<Cfg, true, false, EPI>(a, splits, s);    // NN
    if (a_kc && b_kc) return launch_half_one<Cfg, true, true, EPI>(a, splits, s);       // NT
    if (!a_kc && !b_kc) return launch_half_one<Cfg, false, false, EPI>(a, splits, s);   // TN
    return launch_half_one<Cfg, false, true, EPI>(a, splits, s);                        // TT
}

}  // namespace

hipError_t launch_half(int cfg, int splits, bool a_kc, bool b_kc, int epi, const GemmArgs &a, hipStream_t s)
{
    return with_half_cfg(cfg, [&](auto c) -> hipError_t {
        using Cfg = decltype(c);
        switch (epi) {
            case EPI_AXPBY: return launch_half_layout<Cfg, EPI_AXPBY>(a_kc, b_kc, a, splits, s);
            case EPI_PARTIAL: return launch_half_layout<Cfg, EPI_PARTIAL>(a_kc, b_kc, a, splits, s);
            case EPI_BIAS_TANH: return launch_half_one<Cfg, true, false, EPI_BIAS_TANH>(a, splits, s);   // NN only
            case EPI_BIAS: return launch_half_one<Cfg, true, false, EPI_BIAS>(a, splits, s);             // NN only
            default: return launch_half_one<Cfg, true, true, EPI_TANHGRAD>(a, splits, s);                // NT only
        }
    });
}

}  // namespace ulsnn
