// Which kernel runs a whole narrow network (see chain_kernel.h), and its launch.
#include "chain.h"

namespace iodf {

namespace {

const struct { const ChainKernel* of; int n; } kChains[] = {{kChain443, kChainSizes}, {kChain433, 2}, {kChain423, kChainSizes},
                                                            {kChain223, kChainSizes}, {kChain441, kChainSizes}, {kChain421, kChainSizes},
                                                            {kChain221, kChainSizes}, {kChain40, kChainSizes}, {kChain20, kChainSizes}};

const StripKernel* const kStrips[] = {kStrip443, kStrip433, kStrip423, kStrip223, kStrip441, kStrip421, kStrip221};

size_t strip_lds_bytes(StripPart part, int nc_x, int nc_t, int taps_two, int nc_q, int w, int rows) {
    const int ext = taps_two == 9 ? 1 : 0;
    const size_t px = chain_row_bytes(w, chain_pixel_bytes(nc_x));
    if (part == STRIP_IN) return kChainConstBytes + chain_row_bytes(w, chain_pixel_bytes(nc_q)) * (size_t)(rows + 2);
    if (part == STRIP_LAST) return kChainConstBytes + px * (rows + 2);
    return 2 * kChainConstBytes + px * (rows + 2 + 2 * ext) + chain_row_bytes(w, chain_pixel_bytes(nc_t)) * (size_t)(rows + 2 * ext);
}

const ChainKernel* kernel_for(const ChainArgs& a) {
    const int need = (a.images * a.h * a.w + 31) / 32;
    for (const auto& t : kChains) {
        if (t.of->nc_x != a.nc_x || t.of->nc_t != a.nc_t || t.of->taps_two != a.taps_two) continue;
        for (int i = 0; i < t.n; ++i)
            if (t.of[i].tiles >= need) return t.of + i;
    }
    return nullptr;
}

}  // namespace

size_t chain_lds_bytes(const ChainArgs& a) {
    size_t per = 0;
    for (int nc : {(int)a.nc_x, (int)a.nc_t, (int)a.nc_q}) per += chain_image_bytes(a.h, a.w, chain_pixel_bytes(nc));
    return 2 * kChainConstBytes + per * a.images;
}

int chain_tiles(const ChainArgs& a) {
    const bool ok = a.params && a.state && a.idx && a.batch >= 1 && a.h >= 1 && a.w >= 1 && a.images >= 1 && a.h * a.w <= 32 * kChainMaxTiles &&
           (a.nc_q == 1 || a.nc_q == 2) && a.n_a >= 1 && a.n_a <= 32 * a.nc_q && a.n_out >= 1 && a.n_out <= 32 * a.n_blk_last &&
           (a.n_blk_last == 1 || a.n_blk_last == 2) && (a.taps_last == 1 || a.taps_last == 9) && (a.nc_t != 0) == (a.blocks != 0) &&
           chain_lds_bytes(a) <= kChainMaxLds;
    const ChainKernel* const k = ok ? kernel_for(a) : nullptr;
    return k ? k->tiles : 0;
}

hipError_t chain_setup() {
    for (const auto& t : kChains)
        for (int i = 0; i < t.n; ++i) {
            const hipError_t e = hipFuncSetAttribute((const void*)t.of[i].kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kChainMaxLds);
            if (e != hipSuccess) return e;
        }
    for (const StripKernel* t : kStrips)
        for (int i = 0; i < kStripSizes; ++i)
            for (auto kern : {t[i].kern, t[i].kern_run}) {
                const hipError_t e = kern ? hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kStripMaxLds) : hipSuccess;
                if (e != hipSuccess) return e;
            }
    for (int i = 0; i < kStripIns + kStripLasts; ++i) {
        const StripKernel& k = i < kStripIns ? kStripIn[i] : kStripLast[i - kStripIns];
        const hipError_t e = hipFuncSetAttribute((const void*)k.kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kStripMaxLds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

const StripKernel* strip_kernel_for(StripPart part, int nc_x, int nc_t, int taps_two, int nc_q, int h, int w, int rows) {
    if ((long long)(rows + 4) * 16 * (w + 2) * (w + 2) >= 1 << 20) return nullptr;  // the kernel's divisions by multiplication
    if (rows < 1 || rows > h || strip_lds_bytes(part, nc_x, nc_t, taps_two, nc_q, w, rows) > kStripMaxLds) return nullptr;
    if (part != STRIP_BLOCK) {
        const StripKernel* const t = part == STRIP_IN ? kStripIn : kStripLast;
        for (int i = 0; i < (part == STRIP_IN ? kStripIns : kStripLasts); ++i)
            if (t[i].nc_x == nc_x && (part == STRIP_LAST || t[i].nc_t == nc_q) && rows * w <= 32 * t[i].tiles_two) return t + i;
        return nullptr;
    }
    const int one = rows + (taps_two == 9 ? 2 : 0);
    for (const StripKernel* t : kStrips) {
        if (t->nc_x != nc_x || t->nc_t != nc_t || t->taps_two != taps_two) continue;
        for (int i = 0; i < kStripSizes; ++i)
            if (rows * w <= 32 * t[i].tiles_two && (one < h ? one : h) * w <= 32 * t[i].tiles_one) return t + i;
    }
    return nullptr;
}

// One layer of a workgroup: n_blk blocks of 32 filters over `tiles` tiles, nc chunks of 32 input channels.
static long long layer_macs(int waves, int n_blk, int tiles, int taps, int nc) {
    return 32LL * share_tiles(waves, n_blk, tiles) * 32 * n_blk * taps * 32 * nc;
}

int strip_max_run(const StripKernel& k, int h, int w, int rows) {
    // the loop takes strips that are all alike, and rows that are kept move within LDS without overlapping
    if (!k.kern_run || rows < 2 || h % rows) return 1;
    const long long fresh = 2LL * k.nc_x * (w + 2) * rows;
    const long long kept = 2LL * chain_row_bytes(w, chain_pixel_bytes(k.nc_x)) / 16;  // (nc_t is no larger)
    if (fresh > kStripRunLoads * kStripThreads || kept > kStripRunCopies * kStripThreads) return 1;
    return h / rows < 255 ? h / rows : 255;
}

long long strip_issued_macs(StripPart part, const StripKernel& k, const StripArgs& a) {
    const int waves = kStripThreads / 64;
    long long per = 0;
    if (part == STRIP_IN) per = layer_macs(waves, k.nc_x, k.tiles_two, 9, a.nc_q);
    else if (part == STRIP_LAST) per = layer_macs(waves, a.n_blk_last, k.tiles_two, a.taps_last, k.nc_x);
    else per = layer_macs(waves, k.nc_t, k.tiles_one, 9, k.nc_x) + layer_macs(waves, k.nc_x, k.tiles_two, k.taps_two, k.nc_t);
    const int strips = (a.h + a.rows - 1) / a.rows, runs = (strips + (int)a.run - 1) / (int)a.run;
    if (a.run == 1) return per * strips * a.batch;
    const long long more = layer_macs(waves, k.nc_t, k.tiles_two, 9, k.nc_x) + layer_macs(waves, k.nc_x, k.tiles_two, 9, k.nc_t);
    return (per * runs + more * (strips - runs)) * a.batch;
}

long long chain_issued_macs(const ChainArgs& a) {
    if (!chain_tiles(a)) return 0;
    const ChainKernel& k = *kernel_for(a);
    const int waves = k.threads / 64;
    long long per = layer_macs(waves, k.nc_x, k.tiles, 9, a.nc_q) + layer_macs(waves, a.n_blk_last, k.tiles, a.taps_last, k.nc_x);
    if (a.blocks) per += a.blocks * (layer_macs(waves, k.nc_t, k.tiles, 9, k.nc_x) + layer_macs(waves, k.nc_x, k.tiles, k.taps_two, k.nc_t));
    return per * ((a.batch + a.images - 1) / a.images);
}

hipError_t launch_strip(StripPart part, const StripKernel* k, const StripArgs& a, hipStream_t st) {
    if (a.batch <= 0) return hipSuccess;
    if (!k || !a.params || (part == STRIP_IN ? !a.out || !a.state || !a.idx : !a.in) || (part == STRIP_BLOCK && !a.out) ||
        (part == STRIP_LAST && (!a.state || !a.idx)) ||
        k != strip_kernel_for(part, k->nc_x, k->nc_t, k->taps_two, a.nc_q, a.h, a.w, a.rows) || a.run < 1 ||
        (a.run > 1 && (part != STRIP_BLOCK || (int)a.run > strip_max_run(*k, a.h, a.w, a.rows))))
        return hipErrorInvalidValue;
    const int units = (a.h + a.rows * a.run - 1) / (a.rows * a.run) * a.batch;
    StripArgs b = a;
    b.chunk = (unsigned short)((units + 7) / 8);
    if (units > kStripMaxUnits) return hipErrorInvalidValue;
    hipLaunchKernelGGL(a.run > 1 ? k->kern_run : k->kern, dim3(8 * (b.chunk + b.pf_blocks)), dim3(kStripThreads),
                       strip_lds_bytes(part, k->nc_x, k->nc_t, k->taps_two, a.nc_q, a.w, a.rows), st, b);
    return hipGetLastError();
}

hipError_t launch_chain(const ChainArgs& a, hipStream_t st) {
    if (a.batch <= 0) return hipSuccess;
    if (!chain_tiles(a)) return hipErrorInvalidValue;
    const ChainKernel* const k = kernel_for(a);
    const int groups = (a.batch + a.images - 1) / a.images;
    // blocks go round the XCDs, so those beyond the groups sit pf_blocks to an XCD
    const int grid = a.pf_blocks ? (groups + 7) / 8 * 8 + 8 * a.pf_blocks : groups;
    hipLaunchKernelGGL(k->kern, dim3(grid), dim3(k->threads), chain_lds_bytes(a), st, a);
    return hipGetLastError();
}

}  // namespace iodf
