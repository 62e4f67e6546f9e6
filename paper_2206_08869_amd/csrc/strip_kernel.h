// Strips of images through the layers of a narrow network (see chain.h): the same products and epilogues as
// chain_kernel.h, with the stream x in global memory between launches.
//
// A launch per layer fetches its activations nine times from the L2 (once per tap) and a block's inner tensor goes out
// and comes back. Here a workgroup loads its strip and the rows around it once, runs both convolutions of a block on
// it, the first one on one row more on either side, and writes the result.
//
// Bound. Blocks of two 3x3 layers, 128 wide, strips of four rows of 32 pixels, in clocks of a CU: request to LDS 5000,
// products 9000 + 6000 (matrix cores 6900 + 4600, a quarter of it for the rows that two strips both compute), epilogues
// 3500 + 3100. Two workgroups share a CU, so that the loads and epilogues of one run under the other's products: a pair
// takes 39000 (87 us for the 2048 strips of 256 images; 94 us as two launches layer by layer). With a
// strip or less per CU the length of that chain is what counts, hence strips down to a single row.
//
// Runs. Where strips come in several rounds a workgroup takes any number of them up to all of an image, one below the other (the
// last workgroup of an image may take fewer): a later strip keeps the two rows of t and of x that it shares with the one above, so
// that its first convolution runs over four rows instead of six, and its new rows of x are on their way while the strip above is
// still multiplied. One block of 256 images of 32x32, profiler attached, medians: 82.7 -> 72.8 us (96 channels inside 66.0 -> 56.7),
// of which the priorities below are 1 to 2. The matrix cores' part of a pair of strips falls from 23000 clocks to 18400, in runs of
// four, whose first strip still has six rows, to 19550, and is half of the time (0.49; 96 inside 0.43). A pair's weights, each fragment
// loaded by two waves, are 1.18 MB, 20700 clocks at the 57 bytes a clock that a CU gets: no shorter than the products. The rest is
// epilogues and LDS reads. Dropped: four blocks of 32 filters over four waves in one or both convolutions, half the weights and twice
// the pixel reads (16 blocks of 256 images 1308 us; 1350 in the first, 1385 in the second, 1352 in both).
#pragma once
#include "chain_kernel.h"

namespace iodf {

namespace {

struct StripGeom {
    int img, r0, r1;
    int n;  // strips of this workgroup: rows r0 .. r1 and the n - 1 below, alike
};

__device__ __forceinline__ bool strip_of(const StripArgs& a, StripGeom& g) {
    const int each = a.rows * a.run, strips = (a.h + each - 1) / each;
    const int unit = (int)(blockIdx.x & 7) * a.chunk + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= a.chunk || unit >= strips * a.batch) return false;
    g.img = unit / strips;
    g.r0 = (unit - g.img * strips) * each;
    g.r1 = g.r0 + a.rows < a.h ? g.r0 + a.rows : a.h;
    g.n = (a.h - g.r0 + a.rows - 1) / a.rows;
    g.n = g.n < (int)a.run ? g.n : (int)a.run;
    return true;
}

// Workgroups behind the strips, pf_blocks to an XCD that holds strips (blocks go round the XCDs): what the next launch
// reads first comes into the L2 while compute units would idle.
__device__ __forceinline__ void strip_ahead(const StripArgs& a) {
    const int slot = (int)(blockIdx.x >> 3) - a.chunk, each = a.rows * a.run, units = (a.h + each - 1) / each * a.batch;
    if (slot < 0 || (int)(blockIdx.x & 7) * a.chunk >= units) return;
    touch_lines(a.pf, a.pf_bytes >> 7, slot * kStripThreads + threadIdx.x, a.pf_blocks * kStripThreads);
}

// Rows [y0, y1) of the stream (padding rows and columns included) into LDS, 16 bytes per thread and step, consecutive
// threads on consecutive parts of a 64-channel plane. The first kStripLoads steps' loads are all requested by
// strip_request, before anything else the kernel asks for, so that strip_put waits for one memory latency only.
constexpr int kStripLoads = 9;

template <int NCX>
__device__ __forceinline__ const int8_t* strip_source(const StripArgs& a, const int img, const int y0, const int y1, const int t,
                                                      unsigned& pl, unsigned& k) {
    const unsigned W2 = a.w + 2, per = W2 * 4 * (y1 - y0);
    pl = NCX == 4 && (unsigned)t >= per ? 1u : 0u;
    k = t - pl * per;
    return a.in + ((size_t)img * (a.h + 2) * W2 + (size_t)(y0 + 1) * W2) * 64 + (size_t)pl * a.plane + (size_t)k * 16;
}

template <int NCX, int N>
__device__ __forceinline__ void strip_request(const StripArgs& a, v4i (&v)[N], const int img, const int y0, const int y1,
                                              const int tid) {
    const int total = (a.w + 2) * 4 * (y1 - y0) * (NCX / 2);
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const int t = tid + u * kStripThreads;
        unsigned pl, k;
        v[u] = *(const v4i*)strip_source<NCX>(a, img, y0, y1, t < total ? t : 0, pl, k);
    }
}

template <int NCX, int N>
__device__ __forceinline__ void strip_put(const StripArgs& a, const v4i (&v)[N], unsigned char* x, const int img,
                                          const int y0, const int y1, const unsigned rp, const int tid) {
    constexpr unsigned ps = chain_pixel_bytes(NCX);
    const unsigned per_row = (a.w + 2) * 4, inv = ((1u << kInvBits) + per_row - 1) / per_row;
    const int total = per_row * (y1 - y0) * (NCX / 2);
    auto put = [&](const v4i& d, unsigned pl, unsigned k) {
        const unsigned row = __umul24(k, inv) >> kInvBits, c = k - row * per_row;
        *(v4i*)(x + row * rp + (c >> 2) * ps + pl * 64 + (c & 3) * 16) = d;
    };
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const int t = tid + u * kStripThreads;
        unsigned pl, k;
        (void)strip_source<NCX>(a, img, y0, y1, t, pl, k);
        if (t < total) put(v[u], pl, k);
    }
    if constexpr (N < kStripLoads) return;  // (a run's rows: no more than that)
    for (int t = tid + N * kStripThreads; t < total; t += kStripThreads) {
        unsigned pl, k;
        const v4i d = *(const v4i*)strip_source<NCX>(a, img, y0, y1, t, pl, k);
        put(d, pl, k);
    }
}

// 16 bytes per thread of a layer's constants; the first half of the threads hold them.
__device__ __forceinline__ v4i strip_consts(const gbytes at, const int tid) {
    return *(gv4i)(at + (tid & (kChainConstBytes / 16 - 1)) * 16);
}
__device__ __forceinline__ void strip_put_consts(unsigned char* lds, const v4i& v, const int buf, const int tid) {
    if (tid < kChainConstBytes / 16) *(v4i*)(lds + buf * kChainConstBytes + tid * 16) = v;
}

// Pixel m of rows [y0, y1): row, column; false past the last one (which is repeated).
__device__ __forceinline__ bool strip_pixel(int m, int w, unsigned inv_w, int y0, int y1, int& row, int& col) {
    const int M = (y1 - y0) * w;
    const bool live = m < M;
    m = live ? m : M - 1;
    const int q = (int)(__umul24((unsigned)m, inv_w) >> kInvBits);
    row = y0 + q;
    col = m - q * w;
    return live;
}

// Two workgroups share a compute unit and its waves' turns: the first convolution's products go before all that the other one
// does, which fills the gaps they leave and keeps the two out of step. 16 blocks of 64, 100 and 256 images of 32x32, without
// priorities / both convolutions' products first / the first one's only, in us: 128 inside 427, 744, 1358 / 425, 719, 1338 /
// 406, 692, 1338; 64 inside 281, 485, 875 / 284, 488, 878 / 269, 461, 841. 64 wide, where a third workgroup fits, the second
// one's products go first as well (205 images of 40x32 617, without 637). One workgroup before the other throughout 1364 at 256
// images, epilogues before products 1362. In every kernel of chain_kernel.h, whole networks among them, the latter lose: cfg2
// forward at batch 64 175.4 -> 176.2.
template <bool ON, int P>
__device__ __forceinline__ void wave_priority() {
    if constexpr (ON) __builtin_amdgcn_s_setprio(P);
}

__device__ __forceinline__ void in_register(unsigned& v) { asm volatile("" : "+v"(v)); }

// One residual block. T1, T2: tiles of the first and second convolution. RUN: a.run strips one below the other, else one. The loop
// costs registers (64 inside 162 -> 218, 64 wide 139 -> 157), and 64 inside with them the third workgroup that LDS has room for on
// 16 and 24 columns, so launches of one strip to a workgroup have kernels without it: 16 blocks of 300 images of 32x16 643 -> 600 us;
// 64 wide, when the loop took 181, 160 and 201 images of 32x32 434 -> 402 and 576 -> 536.
template <int NCX, int NCT, int NT2, int T1, int T2, bool RUN>
__global__ __launch_bounds__(kStripThreads, 2) void k_strip_block(const StripArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const unsigned lane16 = lane * 16;
    hold_args(a);
    StripGeom g;
    if (!strip_of(a, g)) return strip_ahead(a);
    constexpr int EXT = NT2 == 3 ? 1 : 0;  // rows of the inner tensor beyond the strip
    const int h = a.h, w = a.w, W2 = w + 2;
    const int xo = g.r0 - 1 - EXT > -1 ? g.r0 - 1 - EXT : -1, xe = g.r1 + 1 + EXT < h + 1 ? g.r1 + 1 + EXT : h + 1;
    const int to = g.r0 - EXT, te = g.r1 + EXT;                          // kept rows of t, and of these the image's
    const int ty0 = to > 0 ? to : 0, ty1 = te < h ? te : h;
    constexpr unsigned psx = chain_pixel_bytes(NCX), pst = chain_pixel_bytes(NCT);
    const unsigned rpx = chain_row_bytes(w, psx), rpt = chain_row_bytes(w, pst);
    constexpr unsigned xb = 2 * kChainConstBytes;
    const unsigned tb = xb + rpx * (xe - xo), end = tb + rpt * (te - to);

    constexpr bool PRIO = strip_largest(NT2 * NT2, T1), BOTH = PRIO && NCX == 2;  // (see wave_priority)
    using ST = Share<4, NCT, T1>;
    using SX = Share<4, NCX, T2>;
    const int tblk = wave % ST::WC * ST::TC, xblk = wave % SX::WC * SX::TC;
    constexpr unsigned w_one = NCT * 9 * NCX * 1024, w_two = NCX * NT2 * NT2 * NCT * 1024;
    const gbytes par = (gbytes)a.params;
    const gbytes p_one = uniform(par + tblk * 9 * NCX * 1024);
    const gbytes p_two = uniform(par + w_one + kChainConstBytes + xblk * NT2 * NT2 * NCT * 1024);
    v4i xv[kStripLoads];
    strip_request<NCX>(a, xv, g.img, xo, xe, tid);
    const v4i c1 = strip_consts(par + w_one, tid), c0 = strip_consts(par + w_one + kChainConstBytes + w_two, tid);
    // 96 filters: in the 16-row form over four tiles and more, else three of the waves take a block of 32 each
    constexpr bool F48 = NCT == 3 && T1 >= 4;
    static_assert(NCT != 3 || (NCX == 4 && NT2 == 3), "what the fragment registers are laid out for");
    constexpr int NWF = NCT == 3 ? 18 : 12;
    const Wave48 f48 = wave48<NCX>(wave & 1, lane);
    const bool one = NCT != 3 || F48 || wave < 3;  // a wave with a share of the first convolution
    v4i wf[NWF];
    static_for<NWF>([&](auto i_) { wf[decltype(i_)::value] = v4i{0, 0, 0, 0}; });
    if constexpr (F48) fetch48<NCX>(wf, uniform(par), f48);
    else if (one) chain_fetch<ST::TC, NCX, 3, 0>(wf, p_one, lane16);
    __builtin_amdgcn_sched_barrier(0);
    const int pad = a.act_unsigned ? (int)0x80808080 : 0;
    for (unsigned o = tb + tid * 16; o < end; o += kStripThreads * 16) *(v4i*)(lds + o) = v4i{pad, pad, pad, pad};
    const unsigned inv_w = ((1u << kInvBits) + w - 1) / w;
    unsigned x_in[ST::TP], t_out[ST::TP], t_in[SX::TP], x_sc[SX::TP], go[SX::TP];
    int live_t = 0, live_x = 0;
    static_for<ST::TP>([&](auto tp_) {
        constexpr int tp = decltype(tp_)::value;
        int row, col;
        if (strip_pixel((wave / ST::WC * ST::TP + tp) * 32 + l32, w, inv_w, ty0, ty1, row, col)) live_t |= 1 << tp;
        x_in[tp] = xb + (row - 1 - xo) * rpx + col * psx + half * 16;
        t_out[tp] = tb + (row - to) * rpt + (col + 1) * pst;
    });
    // (F48) pixel of tile tp, out of l16 as if anew: what is only stored to need not stay in registers meanwhile
    constexpr int TP48 = F48 ? T1 : 1;
    auto pixel48 = [&](int tp, int l16, int& row, int& col) {
        return strip_pixel(((wave >> 1) * TP48 + tp) * 16 + l16, w, inv_w, ty0, ty1, row, col);
    };
    unsigned x_48[TP48];
    if constexpr (F48) {
        static_for<TP48>([&](auto tp_) {
            constexpr int tp = decltype(tp_)::value;
            int row, col;
            (void)pixel48(tp, lane & 15, row, col);
            x_48[tp] = xb + (row - 1 - xo) * rpx + col * psx + (lane >> 4) * 16;
        });
    }
    static_for<SX::TP>([&](auto tp_) {
        constexpr int tp = decltype(tp_)::value;
        int row, col;
        if (strip_pixel((wave / SX::WC * SX::TP + tp) * 32 + l32, w, inv_w, g.r0, g.r1, row, col)) live_x |= 1 << tp;
        t_in[tp] = tb + (row - EXT - to) * rpt + (col + 1 - EXT) * pst + half * 16;
        x_sc[tp] = xb + (row - xo) * rpx + (col + 1) * psx;
        go[tp] = (unsigned)(((g.img * (h + 2) + row + 1) * W2 + col + 1) * 64);
    });
    if constexpr (F48 && !RUN) {
        // worked out here, while the rows are on their way, and not between the products, where the compiler would put them
        // (16 blocks of 64 and 201 images of 32x32 343 -> 334 and 1043 -> 1019 us)
        static_for<TP48>([&](auto tp_) { in_register(x_48[decltype(tp_)::value]); });
        static_for<SX::TP>([&](auto tp_) {
            constexpr int tp = decltype(tp_)::value;
            in_register(t_in[tp]);
            in_register(x_sc[tp]);
            in_register(go[tp]);
        });
    }
    strip_put<NCX>(a, xv, lds + xb, g.img, xo, xe, rpx, tid);
    strip_put_consts(lds, c1, 1, tid);
    strip_put_consts(lds, c0, 0, tid);
    lds_barrier();
    const int* const cst0 = (const int*)lds;
    const int* const cst1 = (const int*)(lds + kChainConstBytes);
    constexpr bool carry = ST::TC == SX::TC;
    constexpr unsigned tcs_two = SX::TC == 2 ? NT2 * NT2 * NCT * 1024 : 0;
    if constexpr (F48) {
        v4i acc[3][TP48];
        const int ch = (wave & 1) * 48 + (lane >> 4) * 4;
        bias48(acc, cst1, ch);
        wave_priority<PRIO, 1>();
        products48<TP48, NCX>(acc, wf, lds, x_48, rpx, uniform(par), f48, [&](auto i_) {
            constexpr int i = decltype(i_)::value;
            if constexpr (i < chain_depth<SX::TC, NCT, NT2>() * SX::TC)
                wf[i] = *(gv4i)(p_two + i % SX::TC * tcs_two + (i / SX::TC) * 1024 + lane16);
        });
        unsigned t_48[TP48];
        int live_48 = 0, l16 = lane & 15;
        asm volatile("" : "+v"(l16));
        static_for<TP48>([&](auto tp_) {
            constexpr int tp = decltype(tp_)::value;
            int row, col;
            if (pixel48(tp, l16, row, col)) live_48 |= 1 << tp;
            t_48[tp] = tb + (row - to) * rpt + (col + 1) * pst;
        });
        wave_priority<PRIO, 0>();
        store48(acc, lds, t_48, live_48, cst1, ch, a.act_unsigned);
    } else if (one) {
        v16i acc[ST::TC][ST::TP];
        chain_bias(acc, cst1, tblk, half);
        wave_priority<PRIO, 1>();
        chain_products<ST::TC, ST::TP, NCX, 3, carry>(acc, wf, lds, x_in, rpx, p_one, p_two, tcs_two, lane16);
        chain_fetch<SX::TC, NCT, NT2, carry ? chain_depth<ST::TC, NCX, 3>() * ST::TC : 0>(wf, p_two, lane16);
        wave_priority<PRIO, 0>();
        chain_store<ST::TC, ST::TP, false>(acc, lds, t_out, live_t, cst1, tblk * 32, half, a.act_unsigned);
    } else {
        chain_fetch<SX::TC, NCT, NT2, 0>(wf, p_two, lane16);
    }
    lds_barrier();
    // The strip's second convolution; with MORE another strip follows, whose new rows are requested in front of it and whose
    // first fragments behind it.
    using SR = Share<4, NCT, T2>;  // a later strip's first convolution
    static_assert(!RUN || (SR::TC == ST::TC && SR::WC == ST::WC), "the same weights to a wave");
    v4i xn[kStripRunLoads];
    auto second = [&](auto more_, const int r0) {
        constexpr bool MORE = decltype(more_)::value;
        // (in a run: fragments' addresses out of the lane as if anew, see below)
        unsigned l16 = lane16;
        Wave48 f = f48;
        if constexpr (RUN) asm volatile("" : "+v"(l16), "+v"(f.lane));
        if constexpr (MORE) {
            int t = tid;
            asm volatile("" : "+v"(t));
            strip_request<NCX>(a, xn, g.img, r0 + a.rows + 2, r0 + 2 * a.rows + 2 < h + 1 ? r0 + 2 * a.rows + 2 : h + 1, t);
        }
        v16i acc[SX::TC][SX::TP];
        chain_bias(acc, cst0, xblk, half);
        if constexpr (MORE && F48) {
            wave_priority<BOTH, 1>();
            chain_products_then<SX::TC, SX::TP, NCT, NT2>(acc, wf, lds, t_in, rpt, p_two, l16, [&](auto i_) {
                constexpr int i = decltype(i_)::value;
                wf[i] = *(gv4i)(uniform(par) + f.at[i % 3] + (i / 3) * 2048 + f.lane);
            });
        } else {
            wave_priority<BOTH, 1>();
            chain_products<SX::TC, SX::TP, NCT, NT2, MORE && carry>(acc, wf, lds, t_in, rpt, p_two, MORE && carry ? p_one : p_two,
                                                                    SR::TC == 2 ? 9 * NCX * 1024 : 0, l16);
            if constexpr (MORE) chain_fetch<SR::TC, NCX, 3, carry ? chain_depth<SX::TC, NCT, NT2>() * SX::TC : 0>(wf, p_one, l16);
        }
        wave_priority<BOTH, 0>();
        chain_store<SX::TC, SX::TP, true, true>(acc, lds, x_sc, live_x, cst0, xblk * 32, half, a.act_unsigned, a.out, a.plane, go);
    };
    if constexpr (RUN) {
        const int rows = a.rows, up = g.r0 - xo;  // row r of the strip at r0 lies in x at row r - r0 + up, in t at r - r0 + 1
        int r0 = g.r0;
#pragma unroll 1
        for (int left = g.n; left > 1; --left) {
            second(std::true_type{}, r0);
            // addresses out of the lane as if anew: what is needed once a strip must not stay in registers meanwhile
            int t = tid;
            asm volatile("" : "+v"(t));
            r0 += rows;
            static_for<SX::TP>([&](auto tp_) { go[decltype(tp_)::value] += rows * W2 * 64; });
            // The last two rows of t, and the last two of x that the next strip reads, become its first. Those of x lie where
            // its new rows go, so they are read before any wave puts those. (Read without a branch: with one, 96 channels inside
            // spilled 14 registers; 16 blocks of 128 and 256 images of 32x32 622 -> 601 and 1103 -> 1069 us.)
            auto keep = [&](v4i& v, unsigned at, unsigned rp, int u, auto put_) {
                const unsigned o = (t + u * kStripThreads) * 16;
                const bool in = o < 2 * rp;
                if constexpr (!decltype(put_)::value) v = *(const v4i*)(lds + at + rows * rp + (in ? o : 0));
                else if (in) *(v4i*)(lds + at + o) = v;
            };
            v4i cx[kStripRunCopies], ct[kStripRunCopies];
            static_for<kStripRunCopies>([&](auto u_) { keep(cx[decltype(u_)::value], xb + up * rpx, rpx, decltype(u_)::value, std::false_type{}); });
            lds_barrier();
            static_for<kStripRunCopies>([&](auto u_) { keep(ct[decltype(u_)::value], tb, rpt, decltype(u_)::value, std::false_type{}); });
            static_for<kStripRunCopies>([&](auto u_) {
                constexpr int u = decltype(u_)::value;
                keep(cx[u], xb + up * rpx, rpx, u, std::true_type{});
                keep(ct[u], tb, rpt, u, std::true_type{});
            });
            const bool bottom = r0 + rows == h;
            strip_put<NCX>(a, xn, lds + xb + (up + 2) * rpx, g.img, r0 + 2, bottom ? h + 1 : r0 + rows + 2, rpx, t);
            lds_barrier();
            if (bottom)  // the row below the image
                for (unsigned o = tb + (rows + 1) * rpt + t * 16; o < tb + (rows + 2) * rpt; o += kStripThreads * 16)
                    *(v4i*)(lds + o) = v4i{pad, pad, pad, pad};
            unsigned l16 = lane16;
            Wave48 f = f48;
            asm volatile("" : "+v"(l16), "+v"(f.lane));
            const int y1 = bottom ? rows : rows + 1;  // rows 1 .. y1 of t, counted from r0
            if constexpr (F48) {
                unsigned at[T2], out[T2];
                int live = 0;
                static_for<T2>([&](auto tp_) {
                    constexpr int tp = decltype(tp_)::value;
                    int row, col;
                    if (strip_pixel(((wave >> 1) * T2 + tp) * 16 + (t & 15), w, inv_w, 1, y1, row, col)) live |= 1 << tp;
                    at[tp] = xb + (row - 1 + up) * rpx + col * psx + ((t & 63) >> 4) * 16;
                    out[tp] = tb + (row + 1) * rpt + (col + 1) * pst;
                });
                v4i acc[3][T2];
                const int ch = (wave & 1) * 48 + (lane >> 4) * 4;
                bias48(acc, cst1, ch);
                wave_priority<PRIO, 1>();
                products48<T2, NCX>(acc, wf, lds, at, rpx, uniform(par), f, [&](auto i_) {
                    constexpr int i = decltype(i_)::value;
                    if constexpr (i < chain_depth<SX::TC, NCT, NT2>() * SX::TC)
                        wf[i] = *(gv4i)(p_two + i % SX::TC * tcs_two + (i / SX::TC) * 1024 + l16);
                });
                wave_priority<PRIO, 0>();
                store48(acc, lds, out, live, cst1, ch, a.act_unsigned);
            } else {
                unsigned at[SR::TP], out[SR::TP];
                int live = 0;
                static_for<SR::TP>([&](auto tp_) {
                    constexpr int tp = decltype(tp_)::value;
                    int row, col;
                    if (strip_pixel((wave / SR::WC * SR::TP + tp) * 32 + (t & 31), w, inv_w, 1, y1, row, col)) live |= 1 << tp;
                    at[tp] = xb + (row - 1 + up) * rpx + col * psx + ((t & 63) >> 5) * 16;
                    out[tp] = tb + (row + 1) * rpt + (col + 1) * pst;
                });
                v16i acc[SR::TC][SR::TP];
                chain_bias(acc, cst1, tblk, half);
                wave_priority<PRIO, 1>();
                chain_products<SR::TC, SR::TP, NCX, 3, carry>(acc, wf, lds, at, rpx, p_one, p_two, tcs_two, l16);
                chain_fetch<SX::TC, NCT, NT2, carry ? chain_depth<SR::TC, NCX, 3>() * SR::TC : 0>(wf, p_two, l16);
                wave_priority<PRIO, 0>();
                chain_store<SR::TC, SR::TP, false>(acc, lds, out, live, cst1, tblk * 32, half, a.act_unsigned);
            }
            lds_barrier();
        }
        second(std::false_type{}, r0);
    } else {
        second(std::false_type{}, g.r0);
    }
}

// Input quantiser and first layer. Little arithmetic behind a chain of latencies, so three workgroups to a CU
// (32x32 maps at batch 256: 33 -> 29 us).
template <int NCX, int NCQ, int T>
__global__ __launch_bounds__(kStripThreads, 3) void k_strip_in(const StripArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const unsigned lane16 = lane * 16;
    hold_args(a);
    StripGeom g;
    if (!strip_of(a, g)) return strip_ahead(a);
    const int h = a.h, w = a.w, W2 = w + 2;
    const int qo = g.r0 - 1, qe = g.r1 + 1, ya = qo > 0 ? qo : 0, yb = qe < h ? qe : h;
    constexpr unsigned psq = chain_pixel_bytes(NCQ);
    const unsigned rpq = chain_row_bytes(w, psq);
    constexpr unsigned qb = kChainConstBytes;
    const unsigned end = qb + rpq * (qe - qo);
    using S = Share<4, NCX, T>;
    const int blk = wave % S::WC * S::TC;
    const gbytes par = (gbytes)a.params;
    const gbytes p = uniform(par + blk * 9 * NCQ * 1024);
    v4i wf[12];
    static_for<12>([&](auto i_) { wf[decltype(i_)::value] = v4i{0, 0, 0, 0}; });
    chain_fetch<S::TC, NCQ, 3, 0>(wf, p, lane16);
    const v4i c0 = strip_consts(par + NCX * 9 * NCQ * 1024, tid);
    for (unsigned o = qb + tid * 16; o < end; o += kStripThreads * 16) *(v4i*)(lds + o) = v4i{0, 0, 0, 0};
    lds_barrier();
    strip_put_consts(lds, c0, 0, tid);
    chain_quant<kStripThreads>(a, lds + qb, g.img, 1, ya, yb, qo, 0, rpq, psq, tid);
    const unsigned inv_w = ((1u << kInvBits) + w - 1) / w;
    unsigned q_in[S::TP], go[S::TP];
    int live = 0;
    static_for<S::TP>([&](auto tp_) {
        constexpr int tp = decltype(tp_)::value;
        int row, col;
        if (strip_pixel((wave / S::WC * S::TP + tp) * 32 + l32, w, inv_w, g.r0, g.r1, row, col)) live |= 1 << tp;
        q_in[tp] = qb + (row - 1 - qo) * rpq + col * psq + half * 16;
        go[tp] = (unsigned)(((g.img * (h + 2) + row + 1) * W2 + col + 1) * 64);
    });
    lds_barrier();
    const int* const cst = (const int*)lds;
    v16i acc[S::TC][S::TP];
    chain_bias(acc, cst, blk, half);
    chain_products<S::TC, S::TP, NCQ, 3, false>(acc, wf, lds, q_in, rpq, p, p, 0, lane16);
    chain_store<S::TC, S::TP, false, true>(acc, lds, q_in, live, cst, blk * 32, half, a.act_unsigned, a.out, a.plane, go);
}

// Last layer. (Three workgroups to a CU would spill: 33 -> 35 us at batch 256.)
template <int NCX, int T>
__global__ __launch_bounds__(kStripThreads, 2) void k_strip_last(const StripArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const unsigned lane16 = lane * 16;
    hold_args(a);
    StripGeom g;
    if (!strip_of(a, g)) return strip_ahead(a);
    const int h = a.h, w = a.w;
    const int xo = g.r0 - 1, xe = g.r1 + 1;
    constexpr unsigned psx = chain_pixel_bytes(NCX), xb = kChainConstBytes;
    const unsigned rpx = chain_row_bytes(w, psx), inv_w = ((1u << kInvBits) + w - 1) / w;
    const gbytes par = (gbytes)a.params;
    v4i xv[kStripLoads];
    strip_request<NCX>(a, xv, g.img, xo, xe, tid);
    const v4i c0 = strip_consts(par + a.n_blk_last * a.taps_last * NCX * 1024, tid);
    const int* const cst = (const int*)lds;
    auto run = [&](auto n_blk_, auto nt_) {
        constexpr int NT = decltype(nt_)::value;
        using S = Share<4, decltype(n_blk_)::value, T>;
        const int blk = wave % S::WC;
        const gbytes p = uniform(par + blk * NT * NT * NCX * 1024);
        v4i wf[12];
        static_for<12>([&](auto i_) { wf[decltype(i_)::value] = v4i{0, 0, 0, 0}; });
        chain_fetch<1, NCX, NT, 0>(wf, p, lane16);
        int ix[16];
        chain_last_channels(a, ix, blk, half);
        unsigned at[S::TP];
        int gp[S::TP];
        static_for<S::TP>([&](auto tp_) {
            constexpr int tp = decltype(tp_)::value;
            int row, col;
            const bool live = strip_pixel((wave / S::WC * S::TP + tp) * 32 + l32, w, inv_w, g.r0, g.r1, row, col);
            at[tp] = xb + (row - (NT == 3) - xo) * rpx + (col + (NT == 1)) * psx + half * 16;
            gp[tp] = live ? (g.img * h + row) * w + col : -1;
        });
        strip_put<NCX>(a, xv, lds + xb, g.img, xo, xe, rpx, tid);
        strip_put_consts(lds, c0, 0, tid);
        lds_barrier();
        v16i acc[1][S::TP];
        chain_bias(acc, cst, blk, half);
        chain_products<1, S::TP, NCX, NT, false>(acc, wf, lds, at, rpx, p, p, 0, lane16);
        chain_last_store<S::TP>(a, acc, gp, ix, cst, blk, half);
    };
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    if (a.taps_last == 9) {
        if (a.n_blk_last == 1) run(I1{}, I3{});
        else run(I2{}, I3{});
    } else {
        if (a.n_blk_last == 1) run(I1{}, I1{});
        else run(I2{}, I1{});
    }
}

}  // namespace

template <int NCX, int NCT, int NT2, int T1, int T2>
constexpr StripKernel strip_kernel() {
    StripKernel k{NCX, NCT, NT2 * NT2, T1, T2, k_strip_block<NCX, NCT, NT2, T1, T2, false>, nullptr};
    if constexpr (strip_largest(NT2 * NT2, T1)) k.kern_run = k_strip_block<NCX, NCT, NT2, T1, T2, true>;
    return k;
}
// Every wave's work is fixed by the tiles a kernel is compiled for, so the small ones are worth their own.
#define IODF_STRIP_TABLE(NAME, NCX, NCT, NT2)                                                                       \
    const StripKernel NAME[kStripSizes] = {strip_kernel<NCX, NCT, NT2, 2, 1>(), strip_kernel<NCX, NCT, NT2, 3, 1>(), \
                                           strip_kernel<NCX, NCT, NT2, 3, 2>(), strip_kernel<NCX, NCT, NT2, 4, 2>(), \
                                           strip_kernel<NCX, NCT, NT2, 6, 4>()};

}  // namespace iodf
