// Which kernel runs a whole narrow network (see chain_kernel.h), and its launch.
#include "chain.h"

namespace iodf {

namespace {

const ChainKernel* const kChains[] = {kChain443, kChain423, kChain223, kChain441, kChain421, kChain221, kChain40, kChain20};

const ChainKernel* kernel_for(const ChainArgs& a) {
    const int need = (a.images * a.h * a.w + 31) / 32;
    for (const ChainKernel* t : kChains) {
        if (t->nc_x != a.nc_x || t->nc_t != a.nc_t || t->taps_two != a.taps_two) continue;
        for (int i = 0; i < kChainSizes; ++i)
            if (t[i].tiles >= need) return t + i;
    }
    return nullptr;
}

}  // namespace

size_t chain_lds_bytes(const ChainArgs& a) {
    size_t per = 0;
    for (int nc : {(int)a.nc_x, (int)a.nc_t, (int)a.nc_q}) per += chain_image_bytes(a.h, a.w, chain_pixel_bytes(nc));
    return 2 * kChainConstBytes + per * a.images;
}

bool chain_args_ok(const ChainArgs& a) {
    return a.params && a.state && a.idx && a.batch >= 1 && a.h >= 1 && a.w >= 1 && a.images >= 1 && a.h * a.w <= 32 * kChainMaxTiles &&
           (a.nc_q == 1 || a.nc_q == 2) && a.n_a >= 1 && a.n_a <= 32 * a.nc_q && a.n_out >= 1 && a.n_out <= 32 * a.n_blk_last &&
           (a.n_blk_last == 1 || a.n_blk_last == 2) && (a.taps_last == 1 || a.taps_last == 9) && (a.nc_t != 0) == (a.blocks != 0) &&
           kernel_for(a) && chain_lds_bytes(a) <= kChainMaxLds;
}

hipError_t chain_setup() {
    for (const ChainKernel* t : kChains)
        for (int i = 0; i < kChainSizes; ++i) {
            const hipError_t e = hipFuncSetAttribute((const void*)t[i].kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kChainMaxLds);
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

hipError_t launch_chain(const ChainArgs& a, hipStream_t st) {
    if (a.batch <= 0) return hipSuccess;
    if (!chain_args_ok(a)) return hipErrorInvalidValue;
    const ChainKernel* const k = kernel_for(a);
    const int groups = (a.batch + a.images - 1) / a.images;
    // blocks go round the XCDs, so those beyond the groups sit pf_blocks to an XCD
    const int grid = a.pf_blocks ? (groups + 7) / 8 * 8 + 8 * a.pf_blocks : groups;
    hipLaunchKernelGGL(k->kern, dim3(grid), dim3(k->threads), chain_lds_bytes(a), st, a);
    return hipGetLastError();
}

}  // namespace iodf
