// Convolution layers over few pixels.
#include "conv_direct.h"
#include "conv_dev.h"

namespace iodf {

namespace {

// 16 TC channels x 16 TP pixels per workgroup, the k-tiles split over its KW waves: each wave multiplies whole tiles of
// its share, and the partial sums (integers: any order of addition gives the same result) meet in LDS.
//
// Over few pixels a layer is launch, first operands, the stream of operands into a compute unit (57 bytes a clock, whether
// they hit in its L1 or in the L2) and drain; the matrix cores idle. conv_igemm_lean's 64x64 tile takes 295 KB of them for
// 256 channels, 3x3 (5200 clocks) on 4 to 64 compute units. Small tiles spread the same layer over more units, 74 KB each
// for 16x16. They need no staging: 16 rows x 64 bytes of either operand are 1 KB of consecutive memory and one operand of
// v_mfma_i32_16x16x64_i8, so every wave loads its fragments straight into registers, D k-tiles ahead, and meets no barrier
// before its reduction is done. Four waves: with eight or sixteen a launch takes longer to begin and to add up than its
// shorter shares save (16x16 tiles: cfg5 at batch 1 2.84 ms with four, 2.90 and 3.01 with eight and sixteen).
// Workgroups that fetch the next layer's weights ahead, as the strips have them, cost more than they save here (2.77 ->
// 3.13 ms; each XCD only its own part: 2.81 -> 2.86). One launch, 256 channels, 3x3, at batch 1, against conv_igemm_lean:
// 4x4 to 16x16 maps 5.2 -> 3.3 us, 32x32 5.6 -> 5.0; whole calls at batch 1: cfg5 3500 -> 2775 us, cfg3 (inverse) 3490 -> 2450,
// mid_dense 463 -> 358.
template <int TC, int TP, int KW, int D, int EPI>
__global__ __launch_bounds__(KW * 64) void conv_igemm_direct(const ConvArgs a) {
    constexpr int BC = 16 * TC, BP = 16 * TP, NB = TC * TP, PER = (NB + KW - 1) / KW;
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, quad = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    hold_args(a);
    // whole pixel blocks to an XCD (8 x ncb x npb / 8), as in conv_igemm, or the channel blocks round the XCDs (ncb x npb)
    const bool by_pixels = direct_by_pixels(a, BP);
    const int cb = by_pixels ? blockIdx.y : blockIdx.x, pb = by_pixels ? blockIdx.z * 8 + blockIdx.x : blockIdx.y;
    const int p0 = pb * BP, c0 = cb * BC;
    if (p0 >= a.npix) return;

    const int nkt = a.taps * (a.cin_pad / 64), hw = a.h * a.w, W2 = a.w + 2, PP = (a.h + 2) * W2;
    const int k0 = wave * nkt / KW, n = (wave + 1) * nkt / KW - k0;

    // the stream of k-tiles: weights at wp, pixels at ap + shift. Past this wave's last k-tile all lanes read the same
    // 16 bytes, which nobody uses.
    const unsigned wstep = (unsigned)a.n_pad * 64;
    const bool k3 = a.taps == 9;
    const int plane0 = k3 ? (int)((unsigned)k0 / 9u) : k0, tap0 = k3 ? k0 - plane0 * 9 : 0;
    gbytes wp = (gbytes)a.wgt + (size_t)k0 * wstep + (size_t)c0 * 64;
    gbytes ap = (gbytes)a.in + (size_t)(a.in_chunk0 + plane0) * a.in_plane;
    int row = (int)((unsigned)tap0 / 3u), col = tap0 - row * 3;
    const unsigned wl = l16 * 64 + quad * 16;
    unsigned pl[TP];
    v4i fw[D][TC], fp[D][TP];
    int w_left = n, p_left = n;  // k-tiles not yet requested
    auto issue_w = [&](auto d_) {
        constexpr int d = decltype(d_)::value;
        const unsigned live = (unsigned)(-w_left >> 31);  // all ones while there are any
        const gbytes ws = uniform(w_left > 0 ? wp : (gbytes)a.wgt);
        static_for<TC>([&](auto i_) { constexpr int i = decltype(i_)::value; fw[d][i] = *(gv4i)(ws + ((i * 1024 + wl) & live)); });
        --w_left;
        wp += wstep;
    };
    auto issue_p = [&](auto d_) {
        constexpr int d = decltype(d_)::value;
        const unsigned live = (unsigned)(-p_left >> 31);
        const gbytes as = uniform(p_left > 0 ? ap + (k3 ? (unsigned)((row * W2 + col) * 64) : 0u) : (gbytes)a.in);
        static_for<TP>([&](auto i_) { constexpr int i = decltype(i_)::value; fp[d][i] = *(gv4i)(as + (pl[i] & live)); });
        --p_left;
        if (k3) {
            if (++col == 3) {
                col = 0;
                if (++row == 3) { row = 0; ap += a.in_plane; }
            }
        } else ap += a.in_plane;
    };
    // weights first: where the pixels lie takes a while to work out
    static_for<D>([&](auto d_) { issue_w(d_); });
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int tp = 0; tp < TP; ++tp) {
        int m = p0 + tp * 16 + l16;
        m = m < a.npix ? m : a.npix - 1;
        pl[tp] = (unsigned)(bordered_pos(a, m, hw, W2, PP) - (k3 ? W2 + 1 : 0)) * 64 + quad * 16;
    }
    static_for<D>([&](auto d_) { issue_p(d_); });

    // what the epilogue needs, on its way behind the first k-tiles
    v4i B4[PER], M4[PER], S4[PER], H4[PER];
    long long at[PER];
    int sc[PER];
    static_for<PER>([&](auto i_) {
        constexpr int i = decltype(i_)::value;
        const int b = wave + i * KW, nb = c0 + (b / TP) * 16 + quad * 4;
        B4[i] = M4[i] = S4[i] = H4[i] = v4i{0, 0, 0, 0};
        at[i] = 0;
        sc[i] = 0;
        if (b >= NB || nb >= a.n_store) return;
        B4[i] = *(const v4i*)(a.bias + nb);
        if (EPI == EPI_ANY && a.mode == MODE_RAW) return;
        M4[i] = *(const v4i*)(a.mul + nb);
        S4[i] = *(const v4i*)(a.shift + nb);
        if constexpr (EPI == EPI_FAST_RELU) H4[i] = *(const v4i*)(a.clamp_hi + nb);
        if (a.mode == MODE_ACT) {
            int m = p0 + b % TP * 16 + l16;
            m = m < a.npix ? m : a.npix - 1;
            at[i] = (long long)(a.out_chunk0 + (nb >> 6)) * a.out_plane + (long long)bordered_pos(a, m, hw, W2, PP) * 64 + (nb & 63);
            if (EPI != EPI_FAST_RELU && a.shortcut) sc[i] = *(const int*)(a.out + at[i]);
        }
    });

    v4i acc[NB];
    static_for<NB>([&](auto b_) { acc[decltype(b_)::value] = v4i{0, 0, 0, 0}; });
    auto mma = [&](auto d_) {
        constexpr int d = decltype(d_)::value;
        static_for<NB>([&](auto b_) {
            constexpr int b = decltype(b_)::value;
            acc[b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fw[d][b / TP], fp[d][b % TP], acc[b], 0, 0, 0);
        });
    };
    int kt = 0;
    for (; kt + D < n; kt += D)
        static_for<D>([&](auto d_) {
            mma(d_);
            issue_w(d_);
            issue_p(d_);
        });
    static_for<D>([&](auto d_) {
        if (kt + decltype(d_)::value < n) mma(d_);
    });

    v4i* const part = (v4i*)lds;
    static_for<NB>([&](auto b_) {
        constexpr int b = decltype(b_)::value;
        part[(wave * NB + b) * 64 + lane] = acc[b];
    });
    __syncthreads();
    static_for<PER>([&](auto i_) {
        constexpr int i = decltype(i_)::value;
        const int b = wave + i * KW;
        if (b >= NB) return;
        v4i s = B4[i];
#pragma unroll
        for (int w = 0; w < KW; ++w) s += part[(w * NB + b) * 64 + lane];
        const int nb = c0 + (b / TP) * 16 + quad * 4, m = p0 + b % TP * 16 + l16;
        if (m >= a.npix || nb >= a.n_store) return;
        if constexpr (EPI != EPI_ANY) {
            unsigned R[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) R[e] = 1u << (S4[i][e] - 1);
            using I0 = std::integral_constant<int, 0>;
            const int lo2 = (a.relu && !a.out_unsigned) ? 0 : -128;
            unsigned p4;
            if constexpr (EPI == EPI_FAST_RELU) p4 = pack_relu_quad(s, I0{}, H4[i], M4[i], S4[i], R, a.out_unsigned);
            else if (a.no_ties) p4 = pack_signed_quad<true>(s, I0{}, M4[i], S4[i], R, sc[i], lo2);
            else p4 = pack_signed_quad<false>(s, I0{}, M4[i], S4[i], R, sc[i], lo2);
            *(unsigned*)(a.out + at[i]) = p4;
        } else {
            if (a.mode == MODE_RAW) {  // n_pad is a multiple of 64, so the quad is in bounds
                *(v4i*)(a.partial + (long long)m * a.n_pad + nb) = s;
                return;
            }
            int v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = rq_dev(s[e], M4[i][e], S4[i][e] + (a.rq_fast ? 32 : 0));
            const int bi = m / hw, qi = m - bi * hw;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (nb + e >= a.n_store) continue;
                int y = v[e];
                if (a.mode == MODE_ACT) {
                    if (a.shortcut) y += (int)(int8_t)(sc[i] >> (8 * e)) + (a.sc_unsigned ? 128 : 0);
                    if (a.relu) y = y < 0 ? 0 : y;
                    a.out[at[i] + e] = (int8_t)(a.out_unsigned ? (y > 255 ? 255 : y) - 128 : sat8_dev(y));
                } else {
                    if (a.relu) y = y < 0 ? 0 : y;
                    y = sat8_dev(y);
                    if (a.mode == MODE_COUPLE) a.state[(long long)m * a.state_c + a.idx_b[nb + e]] += a.sign * y;
                    else a.codes[(long long)bi * a.codes_img_stride + a.codes_off + (long long)(nb + e) * hw + qi] = (int8_t)y;
                }
            }
        }
    });
}

}  // namespace

#define IODF_DIRECT(TC, TP, KW, D)                                                                                        \
    DirectTile {                                                                                                          \
        16 * TC, 16 * TP, KW, (size_t)KW * TC * TP * 1024,                                                                \
            {conv_igemm_direct<TC, TP, KW, D, EPI_ANY>, conv_igemm_direct<TC, TP, KW, D, EPI_FAST>, conv_igemm_direct<TC, TP, KW, D, EPI_FAST_RELU>}, \
            "conv_igemm_direct<" #TC "," #TP "," #KW "," #D ">"                                                                 \
    }
const DirectTile kDirect[kDirectTiles] = {
    IODF_DIRECT(1, 1, 4, 5),
    IODF_DIRECT(2, 1, 4, 5),
    IODF_DIRECT(2, 2, 4, 6),
};

}  // namespace iodf
