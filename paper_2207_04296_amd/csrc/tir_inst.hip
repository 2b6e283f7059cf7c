// One translation unit of kernel instantiations; compiled once per TIR_UNIT value so the units
// build in parallel.  Each line of tir_variants.def owned by this unit becomes an explicit
// instantiation of launch_cfg<Cfg<...>>, which the dispatcher references by address.
#include "tir_kernel.h"
#include "tir_conv_rows.h"
#include "tir_conv_blocks.h"
#include "tir_launch.h"

#ifndef TIR_UNIT
#error "compile with -DTIR_UNIT=<n>"
#endif

namespace tir {

template <class C> hipError_t launch_cfg(const Params& p, hipStream_t stream) {
    dim3 grid((unsigned)(p.tiles_m * p.tiles_n), (unsigned)p.batch, 1);
    if constexpr (C::AMODE == A_CONV_PATCH) {
        grid.x = (unsigned)(p.batch_imgs * p.tiles_m * p.tiles_n);
        return launch_kernel(&conv_patch_kernel<C::DT, C::OUT>, grid, dim3(512), stream, p);
    } else if constexpr (C::AMODE == A_CONV_ROWS) {
        grid.x = (unsigned)((p.batch_imgs * p.tiles_m + p.rows_waves - 1) / p.rows_waves * p.tiles_n);
        const unsigned lds = (unsigned)conv_rows_lds(p.R, p.rows_cpr, p.stride_h, p.dil_h, p.PW, C::BN, p.rows_waves);
        return launch_kernel((p.stride_w * p.Cin * C::ES) % 4 == 0 ? &conv_rows_kernel<C::DT, C::OUT, C::BN, false> : &conv_rows_kernel<C::DT, C::OUT, C::BN, true>, grid,
                             dim3((unsigned)p.rows_waves * 64), stream, p, lds);
    } else if constexpr (C::AMODE == A_CONV_BLOCKS) {
        const auto kernel = p.blk_taps == 2 ? &conv_blocks_kernel<C, 2, 2> : p.blk_taps == 3 ? &conv_blocks_kernel<C, 3, 3> : &conv_blocks_kernel<C, 5, 5>;
        return launch_kernel(kernel, grid, dim3(C::THREADS), stream, p, (unsigned)p.blk_lds);
    } else if constexpr (C::AMODE == A_GENERIC || C::AMODE == A_CONV_GENERIC)
        return launch_kernel(&contract_staged_kernel<C>, grid, dim3(C::THREADS), stream, p);
    else if constexpr (C::AMODE == A_UK || C::AMODE == A_UM)
        return launch_kernel(&contract_unaligned_kernel<C>, grid, dim3(C::THREADS), stream, p);
    else {
        grid.z = (unsigned)p.ksplit;
        return launch_kernel(&contract_direct_kernel<C>, grid, dim3(C::THREADS), stream, p);
    }
}

#define TIR_DEFINE(name, DT, OUT, BM, BN, WM, WN, AM, BMO, RB, NS, KW, CW) \
    template hipError_t launch_cfg<Cfg<DT, OUT, BM, BN, WM, WN, AM, BMO, RB, NS, KW, CW>>(const Params&, hipStream_t);
#define TIR_SKIP(...)

#if TIR_UNIT == 0
#define V0 TIR_DEFINE
#else
#define V0 TIR_SKIP
#endif
#if TIR_UNIT == 1
#define V1 TIR_DEFINE
#else
#define V1 TIR_SKIP
#endif
#if TIR_UNIT == 2
#define V2 TIR_DEFINE
#else
#define V2 TIR_SKIP
#endif
#if TIR_UNIT == 3
#define V3 TIR_DEFINE
#else
#define V3 TIR_SKIP
#endif
#if TIR_UNIT == 4
#define V4 TIR_DEFINE
#else
#define V4 TIR_SKIP
#endif
#if TIR_UNIT == 5
#define V5 TIR_DEFINE
#else
#define V5 TIR_SKIP
#endif
#include "tir_variants.def"

}  // namespace tir
