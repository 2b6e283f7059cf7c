// Launcher declarations shared by the instantiation units and the dispatcher.
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>
#include "tir_params.h"

namespace tir {

// Defined (explicitly instantiated) in tir_inst.hip for every line of tir_variants.def.
template <class C> hipError_t launch_cfg(const Params& p, hipStream_t stream);

// Launch with the arguments where they are: the <<<>>> form copies them once more and keeps the launch configuration in
// between (0.25 us of 2.6 us per launch with a 600-byte parameter block).
template <class P> inline hipError_t launch_kernel(void (*kernel)(P), dim3 grid, dim3 block, hipStream_t stream, const P& p, unsigned lds = 0) {
    void* args[] = {const_cast<typename std::remove_const<P>::type*>(&p)};
    const hipError_t e = hipLaunchKernel((const void*)kernel, grid, block, args, lds, stream);
    if (e != hipSuccess) (void)hipGetLastError();          // reported through the return value
    return e;
}

typedef hipError_t (*launch_fn)(const Params&, hipStream_t);

struct Variant {
    const char* name;
    int dt, out, bm, bn, wm, wn, amode, bmode, rowb, nstage, kw, cw;
    launch_fn fn;
};

}  // namespace tir
