// One ping-pong or copied tile shape of the LDS-tiled matrix-core kernels (gemm_tile.h, gemm_dma.h), selected by ECLIP_PP_ID at compile time:
// both 16-bit types and the three addressing forms, or (ECLIP_PP_POOL) the form of a copied tile that takes a max-pool along.  One translation unit per shape keeps the build parallel; the
// build script compiles this file once for every id listed in ECLIP_PP_TILES.
#include "gemm_dma.h"

#ifndef ECLIP_PP_ID
#error "compile with -DECLIP_PP_ID=<variant id>"
#endif

namespace eclip {

namespace {

constexpr PPTile kTile = pp_tile(ECLIP_PP_ID);
static_assert(kTile.id == ECLIP_PP_ID, "ECLIP_PP_ID is not in ECLIP_PP_TILES");

[[maybe_unused]] constexpr bool kFloatForm = kTile.loop == LOOP_DMA && dma_acc_in_agprs(kTile.bm, kTile.bn, 4);

template <typename T, int AMODE, int FORM>
void launch_dma(const GemmDev &d, const SeDeal &deal, dim3 grid, hipStream_t s)
{
    hipLaunchKernelGGL((conv_gemm_dma_kernel<T, kTile.bm, kTile.bn, kTile.bk, 2, 2, kTile.rs, AMODE, FORM>), grid, dim3(256),
                       dma_lds_bytes(kTile.bm, kTile.bn, kTile.bk, kTile.rs), s, d.x, d.w, d.x_bytes, d.M, d.N, d.K, d.ldx, d.kt_per,
                       dma_walk(d, deal), (unsigned)(d.tiles_m * d.tiles_n), d.fast.d, d.fast.mul, d, deal);
}

#ifndef ECLIP_PP_POOL
template <typename T, int AMODE>
hipError_t launch_one(const GemmDev &d, const SeDeal &deal, dim3 grid, hipStream_t s)
{
    if constexpr (kTile.loop == LOOP_DMA) {
        if constexpr (kFloatForm)
            if (dma_writes_floats(d)) {
                launch_dma<T, AMODE, DMA_F32>(d, deal, grid, s);
                return hipGetLastError();
            }
        launch_dma<T, AMODE, DMA_PLAIN>(d, deal, grid, s);
    } else
        hipLaunchKernelGGL((conv_gemm_kernel<T, kTile.bm, kTile.bn, kTile.bk, 2, 4, kTile.rs, kTile.loop, AMODE>), grid, dim3(512),
                       lds_bytes(kTile.bm, kTile.bn, kTile.bk, 16, kTile.loop != LOOP_PP_BDIRECT), s, d, deal);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_mode(const GemmDev &d, const SeDeal &deal, dim3 grid, hipStream_t s)
{
    switch (gemm_amode(d, kTile.bk, kTile.loop)) {
    case A_MATRIX: return launch_one<T, A_MATRIX>(d, deal, grid, s);
    case A_UNIFORM: return launch_one<T, A_UNIFORM>(d, deal, grid, s);
    default:
        if constexpr (pp_fast_forms_only(ECLIP_PP_ID)) return hipErrorInvalidValue;          // the planner keeps such layers away (GemmTraits::copied)
        else return launch_one<T, A_GENERAL>(d, deal, grid, s);
    }
}

template <typename T, int AMODE>
hipError_t init_one()
{
    if constexpr (kTile.loop == LOOP_DMA) {
        const int lds = (int)dma_lds_bytes(kTile.bm, kTile.bn, kTile.bk, kTile.rs);
        if constexpr (kFloatForm) {
            const hipError_t e = hipFuncSetAttribute((const void *)conv_gemm_dma_kernel<T, kTile.bm, kTile.bn, kTile.bk, 2, 2, kTile.rs, AMODE, DMA_F32>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess) return e;
        }
        return hipFuncSetAttribute((const void *)conv_gemm_dma_kernel<T, kTile.bm, kTile.bn, kTile.bk, 2, 2, kTile.rs, AMODE, DMA_PLAIN>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    } else
        return hipFuncSetAttribute((const void *)conv_gemm_kernel<T, kTile.bm, kTile.bn, kTile.bk, 2, 4, kTile.rs, kTile.loop, AMODE>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes(kTile.bm, kTile.bn, kTile.bk, 16, kTile.loop != LOOP_PP_BDIRECT));
}

}  // namespace

template <> hipError_t launch_pp<ECLIP_PP_ID>(const GemmDev &d, const SeDeal &deal, int dtype, dim3 grid, hipStream_t s)
{
    return dtype == DT_BF16 ? launch_mode<bf16_t>(d, deal, grid, s) : launch_mode<f16_t>(d, deal, grid, s);
}

template <> hipError_t init_pp<ECLIP_PP_ID>()
{
    hipError_t e;
    if constexpr (!pp_fast_forms_only(ECLIP_PP_ID))
        if ((e = init_one<bf16_t, A_GENERAL>()) != hipSuccess || (e = init_one<f16_t, A_GENERAL>()) != hipSuccess) return e;
    if ((e = init_one<bf16_t, A_UNIFORM>()) != hipSuccess || (e = init_one<bf16_t, A_MATRIX>()) != hipSuccess ||
        (e = init_one<f16_t, A_UNIFORM>()) != hipSuccess || (e = init_one<f16_t, A_MATRIX>()) != hipSuccess)
        return e;
    return hipSuccess;
}

#else

// The pooling form is compiled apart: in one code object with the others it moved these, and BERT-base at 5 x 201 tokens, which has no pool, took 1.1 % longer.
template <typename T>
hipError_t init_pool()
{
    return hipFuncSetAttribute((const void *)conv_gemm_dma_kernel<T, kTile.bm, kTile.bn, kTile.bk, 2, 2, kTile.rs, A_UNIFORM, DMA_POOL>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)dma_lds_bytes(kTile.bm, kTile.bn, kTile.bk, kTile.rs));
}

}  // namespace

template <> hipError_t launch_pp_pool<ECLIP_PP_ID>(const GemmDev &d, const SeDeal &deal, int dtype, dim3 grid, hipStream_t s)
{
    if (gemm_amode(d, kTile.bk, kTile.loop) != A_UNIFORM) return hipErrorInvalidValue;       // conv_gemm_pools
    if (dtype == DT_BF16) launch_dma<bf16_t, A_UNIFORM, DMA_POOL>(d, deal, grid, s);
    else launch_dma<f16_t, A_UNIFORM, DMA_POOL>(d, deal, grid, s);
    return hipGetLastError();
}

template <> hipError_t init_pp_pool<ECLIP_PP_ID>()
{
    const hipError_t e = init_pool<bf16_t>();
    return e == hipSuccess ? init_pool<f16_t>() : e;
}

#endif

}  // namespace eclip
