// Whole networks of at most 128 channels out of LDS (Sec. 4.1, App. B.1): input quantiser, first layer, residual
// blocks, last layer and coupling add (or head codes) in one launch.
//
// A layer of 128 channels over the few pixels of a deep level is too little work for a launch of its own: it is
// mostly launch, first operands and drain. Here a workgroup keeps the features of one or several whole images in
// LDS and runs layer after layer on them; only the weights move, from the L2 straight into registers, in the order
// the matrix cores take them (no LDS, no barrier, a stream that never stops between layers).
//
// Bound, per layer 128 -> 128 channels, 3x3, in clocks of a CU (measured in the kernel; 147 KB of weights at the
// 57 bytes a clock that a CU gets from its L2 are 2600):
//   4x4 maps, 1 tile of pixels:   products 2700, the weights; epilogue and barrier 950
//   8x8 maps, 2 tiles:            products 3950 (matrix cores 2300, LDS reads 2300, weights 2600); 1350 to 1600
//   16x16 maps, 8 tiles:          products 11300 (matrix cores 9200); epilogue 4200, with a shortcut 5000, taken with four
//                                 waves; the eight of the table run one's epilogue under the other's products
#pragma once
#include "chain.h"
#include "conv_dev.h"

namespace iodf {

namespace {

constexpr int kInvBits = 20;  // m / d = m * ceil(2^20 / d) >> 20 for m * d < 2^20

// See hold_args(const ConvArgs&).
__device__ __forceinline__ void hold_args(const ChainArgs& a) {
    asm volatile("" ::"s"(a.params), "s"(a.state), "s"(a.idx), "s"(a.codes), "s"(a.pf_bytes), "s"(a.batch), "s"(a.mul_in));
    const unsigned* const raw = (const unsigned*)&a;  // the bit fields
    static_assert(offsetof(ChainArgs, mul_in) == 56 && sizeof(ChainArgs) == 80, "raw[15 .. 19]");
    asm volatile("" ::"s"(raw[15]), "s"(raw[16]), "s"(raw[17]), "s"(raw[18]), "s"(raw[19]));
}
__device__ __forceinline__ void hold_args(const StripArgs& a) {
    asm volatile("" ::"s"(a.params), "s"(a.in), "s"(a.out), "s"(a.state), "s"(a.idx), "s"(a.codes), "s"(a.plane), "s"(a.batch), "s"(a.mul_in));
    const unsigned* const raw = (const unsigned*)&a;
    static_assert(offsetof(StripArgs, mul_in) == 84 && sizeof(StripArgs) == 112, "raw[22 .. 26], then padding");
    asm volatile("" ::"s"(raw[22]), "s"(raw[23]), "s"(raw[24]), "s"(raw[25]), "s"(raw[26]));
}

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// share_blocks / share_tiles of chain.h as constants: TC blocks and TP tiles to a wave.
template <int NW, int N_BLK, int TILES>
struct Share {
    static constexpr int TC = share_blocks(N_BLK, TILES);
    static constexpr int WC = N_BLK / TC, WP = NW / WC;
    static constexpr int TP = share_tiles(NW, N_BLK, TILES) / WP;
};

// The products of one layer. Weights come in fragments of 1 KB per channel block and step (a step: one tap, 32
// channels). w holds those of the next 12 / TC steps, at most a kernel row: as soon as a step has used its
// fragments their registers take those of a later step of the layer or, in the last kernel row, of the next layer,
// so the stream runs on across layers. Pixels are read from LDS one step ahead, two where a step is only one or two
// products long; the scheduling barriers keep the compiler from moving the reads next to their use.
template <int TC, int NC, int NT>
constexpr int chain_depth() { return NC * NT == 9 || NC * NT < 12 / TC ? NC * NT : 12 / TC; }

// With NEXT = false nothing follows: the last kernel row, unrolled by itself, requests no more than its own fragments (the
// repeats that stood for a next layer's were a sixth to a third of a layer's stream).
template <int TC, int TP, int NC, int NT, bool NEXT = true, int NW>
__device__ __forceinline__ void chain_products(v16i (&acc)[TC][TP], v4i (&w)[NW], const unsigned char* lds,
                                               const unsigned (&at)[TP], const unsigned rowstep, const gbytes wcur,
                                               const gbytes wnext, const unsigned tcs_next, const unsigned lane16) {
    constexpr int S = NC * NT, PS = chain_pixel_bytes(NC), D = chain_depth<TC, NC, NT>();
    constexpr unsigned tcs = TC == 2 ? S * NT * 1024 : 0;
    static_assert(S % D == 0 && D * TC <= NW, "a kernel row is a whole number of rounds of the fragment registers");
    constexpr int PD = S % 2 != 0 || (TP <= 2 && S % 3 == 0) ? 2 : 1;
    static_assert(NT == 1 || S % (PD + 1) == 0, "and of the pixel registers");
    v4i b[PD + 1][TP];
    unsigned ba[TP];
#pragma unroll
    for (int tp = 0; tp < TP; ++tp) ba[tp] = at[tp];
    auto read = [&](auto i_) {
        constexpr int i = decltype(i_)::value;
        static_for<TP>([&](auto tp_) {
            constexpr int tp = decltype(tp_)::value;
            b[i % (PD + 1)][tp] = *(const v4i*)(lds + ba[tp] + (i / NC) * PS + (i % NC) * 32);
        });
    };
    static_for<PD>([&](auto i_) { read(i_); });
    // fragments of this row at wr, of what comes behind it at wn
    auto row = [&](auto end_, const gbytes wr, const gbytes wn, const unsigned ts, const unsigned adv) {
        constexpr bool end = decltype(end_)::value;
        static_for<S>([&](auto i_) {
            constexpr int i = decltype(i_)::value;
            if constexpr (i == S - PD && !end) {
#pragma unroll
                for (int tp = 0; tp < TP; ++tp) ba[tp] += adv;
            }
            if constexpr (i + PD < S) read(std::integral_constant<int, i + PD>{});
            else if constexpr (NT > 1 && !end) read(std::integral_constant<int, i + PD - S>{});
            __builtin_amdgcn_sched_barrier(0);
            static_for<TC>([&](auto tc_) {
                constexpr int tc = decltype(tc_)::value;
                static_for<TP>([&](auto tp_) {
                    constexpr int tp = decltype(tp_)::value;
                    acc[tc][tp] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w[(i % D) * TC + tc], b[i % (PD + 1)][tp], acc[tc][tp], 0, 0, 0);
                });
            });
            static_for<TC>([&](auto tc_) {
                constexpr int tc = decltype(tc_)::value;
                if constexpr (i + D < S) w[(i % D) * TC + tc] = *(gv4i)(wr + tc * tcs + (i + D) * 1024 + lane16);
                else if constexpr (!end) w[(i % D) * TC + tc] = *(gv4i)(wn + tc * ts + (i + D - S) * 1024 + lane16);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
#pragma unroll 1
    for (int r = 0; r < (NEXT ? NT : NT - 1); ++r) {
        const bool last = NEXT && r == NT - 1;
        row(std::false_type{}, uniform(wcur + r * (S * 1024)), uniform(last ? wnext : wcur + (r + 1) * (S * 1024)),
            last ? tcs_next : tcs, last ? 0u : rowstep);
    }
    if constexpr (!NEXT) row(std::true_type{}, uniform(wcur + (NT - 1) * (S * 1024)), wcur, 0, 0);
    // what reads the accumulators next may be an opaque statement, which the compiler gives no wait states
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// The same for layers whose fragment registers hold one kernel row, in front of a layer of the 16-row form: next(i) loads
// what register i holds for it.
template <int TC, int TP, int NC, int NT, int NW, class Next>
__device__ __forceinline__ void chain_products_then(v16i (&acc)[TC][TP], v4i (&w)[NW], const unsigned char* lds,
                                                    const unsigned (&at)[TP], const unsigned rowstep, const gbytes wcur,
                                                    const unsigned lane16, Next next) {
    constexpr int S = NC * NT, PS = chain_pixel_bytes(NC);
    constexpr unsigned tcs = TC == 2 ? S * NT * 1024 : 0;
    static_assert(chain_depth<TC, NC, NT>() == S && S * TC <= NW && S % 3 == 0 && NT == 3, "one row of fragments, pixels two steps ahead");
    v4i b[3][TP];
    unsigned ba[TP];
#pragma unroll
    for (int tp = 0; tp < TP; ++tp) ba[tp] = at[tp];
    auto read = [&](auto i_) {
        constexpr int i = decltype(i_)::value;
        static_for<TP>([&](auto tp_) {
            constexpr int tp = decltype(tp_)::value;
            b[i % 3][tp] = *(const v4i*)(lds + ba[tp] + (i / NC) * PS + (i % NC) * 32);
        });
    };
    read(std::integral_constant<int, 0>{});
    read(std::integral_constant<int, 1>{});
    auto row = [&](auto last_, const gbytes wn) {
        constexpr bool last = decltype(last_)::value;
        static_for<S>([&](auto i_) {
            constexpr int i = decltype(i_)::value;
            if constexpr (i == S - 2 && !last) {
#pragma unroll
                for (int tp = 0; tp < TP; ++tp) ba[tp] += rowstep;
            }
            if constexpr (i + 2 < S) read(std::integral_constant<int, i + 2>{});
            else if constexpr (!last) read(std::integral_constant<int, i + 2 - S>{});
            __builtin_amdgcn_sched_barrier(0);
            static_for<TC>([&](auto tc_) {
                constexpr int tc = decltype(tc_)::value;
                static_for<TP>([&](auto tp_) {
                    constexpr int tp = decltype(tp_)::value;
                    acc[tc][tp] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w[i * TC + tc], b[i % 3][tp], acc[tc][tp], 0, 0, 0);
                });
            });
            static_for<TC>([&](auto tc_) {
                constexpr int tc = decltype(tc_)::value;
                if constexpr (last) next(std::integral_constant<int, i * TC + tc>{});
                else w[i * TC + tc] = *(gv4i)(wn + tc * tcs + i * 1024 + lane16);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
#pragma unroll 1
    for (int r = 1; r < NT; ++r) row(std::false_type{}, uniform(wcur + r * (S * 1024)));
    row(std::true_type{}, wcur);
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// The products of one layer, one block of filters to a wave, over one or two tiles, unrolled whole: the fragment registers are
// a ring that holds R of the network's stream ahead, half a layer of 128 channels or one of 64. load(i) requests what follows R
// behind fragment i. With few tiles the products take as long as the weights need to come, and with 12 ahead the stream
// stood still during every epilogue. 18 layers 128 wide: on one 8x8 map 46.1 -> 40.1 us, on one 4x4 map 32.4 -> 31.4; 64 channels
// inside 35.5 -> 32.1 and 30.1 -> 26.5. (36 ahead: the compiler no longer keeps the ring in place from block to block.)
template <int TP, int NC, int NT, int R, class Load>
__device__ __forceinline__ void chain_products_ring(v16i (&acc)[1][TP], v4i (&w)[R], const unsigned char* lds, const unsigned (&at)[TP],
                                                    const unsigned rowstep, Load load) {
    constexpr int S = NC * NT, F = S * NT, PS = chain_pixel_bytes(NC);
    v4i b[3][TP];
    unsigned ba[TP];
#pragma unroll
    for (int tp = 0; tp < TP; ++tp) ba[tp] = at[tp];
    auto read = [&](auto i_) {
        constexpr int i = decltype(i_)::value, j = i % S;
        static_for<TP>([&](auto tp_) {
            constexpr int tp = decltype(tp_)::value;
            if constexpr (i > 0 && j == 0) ba[tp] += rowstep;
            b[i % 3][tp] = *(const v4i*)(lds + ba[tp] + (j / NC) * PS + (j % NC) * 32);
        });
    };
    read(std::integral_constant<int, 0>{});
    read(std::integral_constant<int, 1>{});
    static_for<F>([&](auto i_) {
        constexpr int i = decltype(i_)::value;
        if constexpr (i + 2 < F) read(std::integral_constant<int, i + 2>{});
        __builtin_amdgcn_sched_barrier(0);
        static_for<TP>([&](auto tp_) {
            constexpr int tp = decltype(tp_)::value;
            acc[0][tp] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w[i % R], b[i % 3][tp], acc[0][tp], 0, 0, 0);
        });
        load(i_);
        __builtin_amdgcn_sched_barrier(0);
    });
    // what reads the accumulators next may be an opaque statement, which the compiler gives no wait states
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Fragment i of a layer at p: four to a base, so that the offsets fit a load's own field and take no registers.
__device__ __forceinline__ v4i fragment(const gbytes p, const int i, const unsigned lane16) {
    return *(gv4i)(uniform(p + (i & ~3) * 1024) + (i & 3) * 1024 + lane16);
}

// Fragments of the first steps of a layer, registers from FROM on.
template <int TC, int NC, int NT, int FROM, int NW>
__device__ __forceinline__ void chain_fetch(v4i (&w)[NW], const gbytes p, const unsigned lane16) {
    constexpr int n = chain_depth<TC, NC, NT>() * TC;
    static_for<n>([&](auto i_) {
        constexpr int i = decltype(i_)::value;
        if constexpr (i >= FROM) w[i] = *(gv4i)(p + (i % TC) * (NC * NT * NT * 1024) + (i / TC) * 1024 + lane16);
    });
}

// Three blocks of 32 filters do not divide over the waves. A layer of 96 filters over four tiles and more therefore runs
// on v_mfma_i32_16x16x64_i8: a wave takes 48 filters, three blocks of 16, and half (a quarter) of the pixels in tiles of
// 16; half a wave's lanes of a 32-filter fragment and of the one behind it are one operand of it. 96 of 128 filters kept,
// against the kernels of 128: one residual block on 256 images of 32x32 85 -> 71 us, 18 layers on 256 of 16x16 146 -> 113.
struct Wave48 {
    unsigned at[3];  // a wave's three blocks of 16 filters: offsets in a layer's fragments
    unsigned lane;   // and a lane's
};

template <int NC>
__device__ __forceinline__ Wave48 wave48(const int col, const int lane) {
    Wave48 f;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        const int g = 3 * col + t;
        f.at[t] = (unsigned)((g >> 1) * (9 * NC * 1024) + (g & 1) * 256);
    }
    const int quad = lane >> 4;
    f.lane = (unsigned)((quad >> 1) * 1024 + (quad & 1) * 512 + (lane & 15) * 16);
    return f;
}

// A step: one tap, 64 channels. w: the fragments of a kernel row's steps, three to a step.
template <int NC>
__device__ __forceinline__ void fetch48(v4i (&w)[18], const gbytes p, const Wave48& f) {
    static_for<18>([&](auto i_) {
        constexpr int i = decltype(i_)::value;
        if constexpr (i < 3 * (NC / 2) * 3) w[i] = *(gv4i)(p + f.at[i % 3] + (i / 3) * 2048 + f.lane);
    });
}

// The products of such a layer. next(i) loads what register i holds for the layer behind it.
template <int TP, int NC, class Next>
__device__ __forceinline__ void products48(v4i (&acc)[3][TP], v4i (&w)[18], const unsigned char* lds, const unsigned (&at)[TP],
                                           const unsigned rowstep, const gbytes p, const Wave48& f, Next next) {
    static_assert(NC == 4, "a step's three fragments and a row's six steps fill the registers");
    constexpr int S = 6, PS = chain_pixel_bytes(NC);
    v4i b[2][TP];
    unsigned ba[TP];
#pragma unroll
    for (int tp = 0; tp < TP; ++tp) ba[tp] = at[tp];
    auto read = [&](auto i_) {
        constexpr int i = decltype(i_)::value;
        static_for<TP>([&](auto tp_) {
            constexpr int tp = decltype(tp_)::value;
            b[i % 2][tp] = *(const v4i*)(lds + ba[tp] + (i / 2) * PS + (i % 2) * 64);
        });
    };
    using I0 = std::integral_constant<int, 0>;
    read(I0{});
    auto row = [&](auto last_, const gbytes wn) {
        constexpr bool last = decltype(last_)::value;
        static_for<S>([&](auto i_) {
            constexpr int i = decltype(i_)::value;
            if constexpr (i + 1 < S) read(std::integral_constant<int, i + 1>{});
            else if constexpr (!last) {
#pragma unroll
                for (int tp = 0; tp < TP; ++tp) ba[tp] += rowstep;
                read(I0{});
            }
            __builtin_amdgcn_sched_barrier(0);
            static_for<3>([&](auto t_) {
                constexpr int t = decltype(t_)::value;
                static_for<TP>([&](auto tp_) {
                    constexpr int tp = decltype(tp_)::value;
                    acc[t][tp] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[i * 3 + t], b[i % 2][tp], acc[t][tp], 0, 0, 0);
                });
            });
            static_for<3>([&](auto t_) {
                constexpr int t = decltype(t_)::value;
                if constexpr (last) next(std::integral_constant<int, i * 3 + t>{});
                else w[i * 3 + t] = *(gv4i)(wn + f.at[t] + i * 2048 + f.lane);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
#pragma unroll 1
    for (int r = 1; r < 3; ++r) row(std::false_type{}, uniform(p + r * (S * 2048)));
    row(std::true_type{}, p);
    // what reads the accumulators next may be an opaque statement, which the compiler gives no wait states
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Its accumulators' start, and its epilogue: a lane holds four consecutive filters of a pixel for every block and tile.
template <int TP>
__device__ __forceinline__ void bias48(v4i (&acc)[3][TP], const int* cst, const int ch) {
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        const v4i b4 = *(const v4i*)(cst + 3 * 128 + ch + 16 * t);
#pragma unroll
        for (int tp = 0; tp < TP; ++tp) acc[t][tp] = b4;
    }
}

template <int TP>
__device__ __forceinline__ void store48(const v4i (&acc)[3][TP], unsigned char* lds, const unsigned (&at)[TP], const int live,
                                        const int* cst, const int ch, const bool act_unsigned) {
    static_for<3>([&](auto t_) {
        constexpr int t = decltype(t_)::value;
        const int n = ch + 16 * t;
        const v4i B = *(const v4i*)(cst + n), M = *(const v4i*)(cst + 128 + n), S = *(const v4i*)(cst + 256 + n);
        unsigned R[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) R[e] = 1u << (S[e] - 1);
        static_for<TP>([&](auto tp_) {
            constexpr int tp = decltype(tp_)::value;
            const unsigned p4 = pack_relu_quad(acc[t][tp], std::integral_constant<int, 0>{}, B, M, S, R, act_unsigned);
            if (live >> tp & 1) *(unsigned*)(lds + at[tp] + n) = p4;
        });
    });
}

// Hidden layer's epilogue: requantise, ReLU or shortcut, 16 channels of a pixel per lane and 32x32 block, into LDS.
// at: where each tile's pixel lies in the output tensor. With OUT the result goes there instead, to out[pixel * 64 ..]
// of 64-channel planes, go = pixel * 64 (the shortcut still comes from LDS).
template <int TC, int TP, bool SHORTCUT, bool OUT = false>
__device__ __forceinline__ void chain_store(const v16i (&acc)[TC][TP], unsigned char* lds, const unsigned (&at)[TP],
                                            const int live, const int* cst, const int ch_base, const int half,
                                            const bool act_unsigned, int8_t* out = nullptr, const unsigned plane = 0,
                                            const unsigned* go = nullptr) {
    static_for<TC>([&](auto tc_) {
        constexpr int tc = decltype(tc_)::value;
        const int ch0 = ch_base + tc * 32;
        v4i Bq[4], Mq[4], Sq[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int nl = ch0 + g * 8 + half * 4;
            if (!SHORTCUT) Bq[g] = *(const v4i*)(cst + nl);
            Mq[g] = *(const v4i*)(cst + 128 + nl);
            Sq[g] = *(const v4i*)(cst + 256 + nl);
        }
        unsigned pk[TP][4];
        if constexpr (SHORTCUT) {
            // the shortcut's 16 bytes sit where the result's go; the regrouping below run backwards
            v4i s4[TP];
            static_for<TP>([&](auto tp_) { s4[decltype(tp_)::value] = *(const v4i*)(lds + at[decltype(tp_)::value] + ch0 + half * 16); });
            __builtin_amdgcn_sched_barrier(0);
            static_for<TP>([&](auto tp_) {
                constexpr int tp = decltype(tp_)::value;
                auto x = __builtin_amdgcn_permlane32_swap((unsigned)s4[tp][0], (unsigned)s4[tp][2], false, false);
                auto u = __builtin_amdgcn_permlane32_swap((unsigned)s4[tp][1], (unsigned)s4[tp][3], false, false);
                auto q01 = __builtin_amdgcn_permlane32_swap(x[0], u[0], false, false);
                auto q23 = __builtin_amdgcn_permlane32_swap(x[1], u[1], false, false);
                pk[tp][0] = q01[0]; pk[tp][1] = q01[1]; pk[tp][2] = q23[0]; pk[tp][3] = q23[1];
            });
        }
        static_for<4>([&](auto g_) {
            constexpr int g = decltype(g_)::value;
            unsigned Rq[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) Rq[e] = 1u << (Sq[g][e] - 1);
            static_for<TP>([&](auto tp_) {
                constexpr int tp = decltype(tp_)::value;
                if constexpr (SHORTCUT)
                    pk[tp][g] = pack_signed_quad<true>(acc[tc][tp], std::integral_constant<int, g * 4>{}, Mq[g], Sq[g], Rq,
                                                       (int)pk[tp][g], act_unsigned ? -128 : 0);
                else
                    pk[tp][g] = pack_relu_quad(acc[tc][tp], std::integral_constant<int, g * 4>{}, Bq[g], Mq[g], Sq[g], Rq, act_unsigned);
            });
        });
        static_for<TP>([&](auto tp_) {
            constexpr int tp = decltype(tp_)::value;
            auto s01 = __builtin_amdgcn_permlane32_swap(pk[tp][0], pk[tp][1], false, false);
            auto s23 = __builtin_amdgcn_permlane32_swap(pk[tp][2], pk[tp][3], false, false);
            auto x = __builtin_amdgcn_permlane32_swap(s01[0], s23[0], false, false);
            auto u = __builtin_amdgcn_permlane32_swap(s01[1], s23[1], false, false);
            const v4i o4 = {(int)x[0], (int)u[0], (int)x[1], (int)u[1]};
            if (live >> tp & 1) {
                if constexpr (OUT) *(v4i*)(out + (size_t)(ch0 >> 6) * plane + go[tp] + (ch0 & 63) + half * 16) = o4;
                else *(v4i*)(lds + at[tp] + ch0 + half * 16) = o4;
            }
        });
    });
}

// Accumulators start at the bias.
template <int TC, int TP>
__device__ __forceinline__ void chain_bias(v16i (&acc)[TC][TP], const int* cst, const int blk, const int half) {
    static_for<TC>([&](auto tc_) {
        constexpr int tc = decltype(tc_)::value;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const v4i b4 = *(const v4i*)(cst + 3 * 128 + (blk + tc) * 32 + g * 8 + half * 4);
            static_for<TP>([&](auto tp_) {
                constexpr int tp = decltype(tp_)::value;
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[tc][tp][g * 4 + e] = b4[e];
            });
        }
    });
}

// Quantised input of rows [ya, yb) of some images: channel c of pixel p is sat8(rq(S[p][idx[c]])). q: the tensor, whose
// first kept row is image row `org`. Four channels to a task, four tasks of a thread at a time: their loads, an index
// and a word behind it each, overlap.
template <int THREADS, class Args>
__device__ __forceinline__ void chain_quant(const Args& a, unsigned char* q, const int img0, const int n_img, const int ya,
                                            const int yb, const int org, const unsigned image, const unsigned row_bytes,
                                            const unsigned pixel, const int tid) {
    const unsigned w = a.w, hw = a.h * a.w, per = (yb - ya) * w;
    const unsigned quads = (a.n_a + 3) >> 2, total = per * n_img * quads;
    const int32_t* const s0 = a.state + ((long long)img0 * hw + ya * w) * a.state_c;
    for (unsigned t0 = tid; t0 < total; t0 += 4 * THREADS) {
        int v[4][4];
        unsigned at[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const unsigned t = t0 + u * THREADS < total ? t0 + u * THREADS : t0, p = t / quads, g = t - p * quads;
            const unsigned im = p / per, k = p - im * per, row = k / w, col = k - row * w;
            const int32_t* const s = s0 + (im * hw + k) * a.state_c;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[u][e] = s[a.idx[g * 4 + e < a.n_a ? g * 4 + e : 0]];
            at[u] = im * image + (ya + row - org) * row_bytes + (col + 1) * pixel + g * 4;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (t0 + u * THREADS >= total) break;
            const unsigned g = (t0 + u * THREADS) % quads;
            unsigned packed = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (g * 4 + e < a.n_a) packed |= ((unsigned)sat8_dev(rq_dev(v[u][e], a.mul_in, a.shift_in)) & 0xffu) << (8 * e);
            *(unsigned*)(q + at[u]) = packed;
        }
    }
}

// Epilogue of the last layer: requantise, then add into the state or write head codes. ix: physical channels of this
// lane's sixteen filters (see chain_last_channels); gp: each tile's pixel, image * hw + q, or -1.
template <class Args>
__device__ __forceinline__ void chain_last_channels(const Args& a, int (&ix)[16], const int blk, const int half) {
    static_for<16>([&](auto r_) {
        constexpr int r = decltype(r_)::value;
        const int n = blk * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
        ix[r] = a.codes ? 0 : a.idx[a.n_a + (n < a.n_out ? n : a.n_out - 1)];
    });
}

template <int TP, class Args>
__device__ __forceinline__ void chain_last_store(const Args& a, const v16i (&acc)[1][TP], const int (&gp)[TP], const int (&ix)[16],
                                                 const int* cst, const int blk, const int half) {
    const int hw = a.h * a.w;
    auto result = [&](int acc, int n) {
        int y;
        if (a.last_fast) y = (__mulhi(acc, cst[128 + n]) + (1 << (cst[256 + n] - 33))) >> (cst[256 + n] - 32);
        else y = rq_dev(acc, cst[128 + n], cst[256 + n]);
        if (a.relu_last) y = y < 0 ? 0 : y;
        return sat8_dev(y);
    };
    if (a.codes) {
        static_for<TP>([&](auto tp_) {
            constexpr int tp = decltype(tp_)::value;
            if (gp[tp] < 0) return;
            const int bi = gp[tp] / hw, qi = gp[tp] - bi * hw;
            int8_t* const cp = a.codes + (long long)bi * a.codes_img_stride + a.codes_off + qi;
            static_for<16>([&](auto r_) {
                constexpr int r = decltype(r_)::value;
                const int n = blk * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
                if (n < a.n_out) cp[n * hw] = (int8_t)result(acc[0][tp][r], n);
            });
        });
        return;
    }
    // The state words this lane updates: all on their way before the first is needed. Lanes past the last pixel
    // and filters past the last one read a word that exists and write nothing.
    static_for<TP>([&](auto tp_) {
        constexpr int tp = decltype(tp_)::value;
        int32_t* const sp = a.state + (long long)(gp[tp] < 0 ? 0 : gp[tp]) * a.state_c;
        int v[16];
        static_for<16>([&](auto r_) { v[decltype(r_)::value] = sp[ix[decltype(r_)::value]]; });
        if (gp[tp] < 0) return;
        static_for<16>([&](auto r_) {
            constexpr int r = decltype(r_)::value;
            const int n = blk * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
            if (n < a.n_out) sp[ix[r]] = v[r] + a.sign * result(acc[0][tp][r], n);
        });
    });
}

// Networks of 3x3 blocks that hold their fragments in a ring (see chain_products_ring).
template <int NCX, int NCT, int NT2, int TILES>
constexpr bool chain_ring() { return NCX == 4 && (NCT == 2 || NCT == 4) && NT2 == 3 && TILES <= 2; }

// NCX, NCT: 32-channel chunks of the stream x and of the tensor t inside a block (0: no blocks); NT2: kernel side of a
// block's second convolution; TILES: 32-pixel tiles of the workgroup's images, rounded up to a power of two.
// (The ring is given 256 registers: with more, the compiler keeps part of it in accumulation registers and moves it back
// every block, behind a wait for all loads.)
template <int NW, int NCX, int NCT, int NT2, int TILES>
__global__ __launch_bounds__(NW * 64, (chain_ring<NCX, NCT, NT2, TILES>() ? 2 : 1)) void k_chain(const ChainArgs a) {
    constexpr int kThreads = NW * 64;
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const unsigned lane16 = lane * 16;
    hold_args(a);

    const int groups = (a.batch + a.images - 1) / a.images;
    if ((int)blockIdx.x >= groups) {
        // workgroups beyond the groups bring the parameters into the L2 of an XCD that has groups (blocks go round the XCDs)
        if ((int)(blockIdx.x & 7) >= groups) return;
        const int base = (groups + 7) >> 3;  // first slot of an XCD that may hold such a block
        touch_lines(a.params, a.pf_bytes >> 7, (((int)blockIdx.x >> 3) - base) * kThreads + tid, a.pf_blocks * kThreads);
        return;
    }
    const int img0 = blockIdx.x * a.images;
    const int n_img = a.batch - img0 < a.images ? a.batch - img0 : a.images;
    const int h = a.h, w = a.w, hw = h * w, M = n_img * hw;

    // LDS: constants of the current and the next layer, then the three tensors, zero-bordered images each
    constexpr unsigned psx = chain_pixel_bytes(NCX), pst = chain_pixel_bytes(NCT);
    const unsigned psq = chain_pixel_bytes(a.nc_q);
    const unsigned rpx = chain_row_bytes(w, psx), rpt = chain_row_bytes(w, pst), rpq = chain_row_bytes(w, psq);
    const unsigned isx = chain_image_bytes(h, w, psx), ist = chain_image_bytes(h, w, pst), isq = chain_image_bytes(h, w, psq);
    constexpr unsigned qb = 2 * kChainConstBytes;
    const unsigned xb = qb + isq * n_img, tb = xb + isx * n_img, end = tb + ist * n_img;

    // Parameter block: sizes of a layer's weights and constants
    const unsigned bytes_in = NCX * 9 * a.nc_q * 1024 + kChainConstBytes;
    constexpr unsigned w_one = NCT * 9 * NCX * 1024, w_two = NCX * NT2 * NT2 * NCT * 1024;
    constexpr unsigned bytes_one = w_one + kChainConstBytes, bytes_block = bytes_one + w_two + kChainConstBytes;
    const gbytes par = (gbytes)a.params;

    using SX = Share<NW, NCX, TILES>;                 // layers that write the stream
    using ST = Share<NW, NCT ? NCT : 1, TILES>;       // first convolution of a block
    using S1 = Share<NW, 1, TILES>;                   // last layer, up to 32 filters
    using S2 = Share<NW, 2, TILES>;                   // ... up to 64
    const int xblk = wave % SX::WC * SX::TC, tblk = wave % ST::WC * ST::TC;

    constexpr bool F48 = NCT == 3;  // a block's first convolution in the 16-row form: two columns of waves
    static_assert(!F48 || (NCX == 4 && NT2 == 3 && TILES >= 4 && SX::TC == 2), "what the fragment registers are laid out for");
    constexpr int TP48 = F48 ? 4 * TILES / NW : 1;
    constexpr bool RING = chain_ring<NCX, NCT, NT2, TILES>();
    constexpr int NWF = RING || F48 ? 18 : 12;
    // one tile, 64 filters: two waves have the first convolution's, the other two go without
    const bool one = !RING || NCT == 4 || TILES > 1 || wave < 2;
    const Wave48 f48 = wave48<NCX>(wave & 1, lane);
    v4i wf[NWF];
    static_for<NWF>([&](auto i_) { wf[decltype(i_)::value] = v4i{0, 0, 0, 0}; });
    const gbytes w_in = par + (size_t)(xblk * 9 * a.nc_q * 1024);
    if (a.nc_q == 1) chain_fetch<SX::TC, 1, 3, 0>(wf, uniform(w_in), lane16);
    else chain_fetch<SX::TC, 2, 3, 0>(wf, uniform(w_in), lane16);
    auto fetch_const = [&](gbytes at) { return tid < kChainConstBytes / 16 ? *(gv4i)(at + tid * 16) : v4i{0, 0, 0, 0}; };
    auto put_const = [&](int buf, const v4i& v) {
        if (tid < kChainConstBytes / 16) *(v4i*)(lds + buf * kChainConstBytes + tid * 16) = v;
    };
    {
        const v4i c0 = fetch_const(par + (bytes_in - kChainConstBytes));
        // padding first: the quantised input's is byte 0, the features' the stored form of code 0
        const int pad = a.act_unsigned ? (int)0x80808080 : 0;
        for (unsigned o = qb + tid * 16; o < end; o += kThreads * 16) {
            const int v = o < xb ? 0 : pad;
            *(v4i*)(lds + o) = v4i{v, v, v, v};
        }
        put_const(0, c0);
    }
    lds_barrier();
    chain_quant<kThreads>(a, lds + qb, img0, n_img, 0, h, -1, isq, rpq, psq, tid);

    // Where the pixels of this wave's tiles lie: image, row, column, as byte offsets of tap (0, 0) in each tensor.
    // Lanes past the last pixel repeat it and store nothing.
    const unsigned inv_w = ((1u << kInvBits) + w - 1) / w, inv_hw = ((1u << kInvBits) + hw - 1) / hw;
    auto pixel_of = [&](int m, int& im, int& row, int& col) {
        const bool live = m < M;
        m = live ? m : M - 1;
        im = (int)(__umul24((unsigned)m, inv_hw) >> kInvBits);
        const int q = m - im * hw;
        row = (int)(__umul24((unsigned)q, inv_w) >> kInvBits);
        col = q - row * w;
        return live;
    };
    unsigned x_of_x[SX::TP], t_of_x[SX::TP], q_of_x[SX::TP], x_of_t[ST::TP], t_of_t[ST::TP];
    int live_x = 0, live_t = 0;
    static_for<SX::TP>([&](auto tp_) {
        constexpr int tp = decltype(tp_)::value;
        int im, row, col;
        if (pixel_of((wave / SX::WC * SX::TP + tp) * 32 + l32, im, row, col)) live_x |= 1 << tp;
        x_of_x[tp] = xb + im * isx + row * rpx + col * psx;
        t_of_x[tp] = tb + im * ist + row * rpt + col * pst + half * 16;
        q_of_x[tp] = qb + im * isq + row * rpq + col * psq + half * 16;
    });
    static_for<ST::TP>([&](auto tp_) {
        constexpr int tp = decltype(tp_)::value;
        int im, row, col;
        if (pixel_of((wave / ST::WC * ST::TP + tp) * 32 + l32, im, row, col)) live_t |= 1 << tp;
        x_of_t[tp] = xb + im * isx + row * rpx + col * psx + half * 16;
        t_of_t[tp] = tb + im * ist + row * rpt + col * pst;
    });
    unsigned x_of_48[TP48], to_48[TP48];
    int live_48 = 0;
    if constexpr (F48) {
        static_for<TP48>([&](auto tp_) {
            constexpr int tp = decltype(tp_)::value;
            int im, row, col;
            if (pixel_of(((wave >> 1) * TP48 + tp) * 16 + (lane & 15), im, row, col)) live_48 |= 1 << tp;
            x_of_48[tp] = xb + im * isx + row * rpx + col * psx + (lane >> 4) * 16;
            to_48[tp] = tb + im * ist + (row + 1) * rpt + (col + 1) * pst;
        });
    }
    unsigned xo[SX::TP], to[ST::TP];  // the pixels themselves
#pragma unroll
    for (int i = 0; i < SX::TP; ++i) xo[i] = x_of_x[i] + rpx + psx;
#pragma unroll
    for (int i = 0; i < ST::TP; ++i) to[i] = t_of_t[i] + rpt + pst;
    lds_barrier();

    const int* const cst0 = (const int*)lds;
    const int* const cst1 = (const int*)(lds + kChainConstBytes);

    // First layer. Behind it every layer's constants alternate between the two buffers: 1, 0, 1, ...
    gbytes blockp = par + bytes_in;
    constexpr bool carry_one = NCT != 0 && SX::TC == ST::TC;  // the stream of fragments runs on between x's layers and t's
    constexpr unsigned tcs_one = ST::TC == 2 ? 9 * NCX * 1024 : 0, tcs_two = SX::TC == 2 ? NT2 * NT2 * NCT * 1024 : 0;
    {
        const v4i cn = fetch_const(NCT ? blockp + w_one : blockp + a.n_blk_last * a.taps_last * NCX * 1024);
        v16i acc[SX::TC][SX::TP];
        chain_bias(acc, cst0, xblk, half);
        if (a.nc_q == 1) chain_products<SX::TC, SX::TP, 1, 3, false>(acc, wf, lds, q_of_x, rpq, uniform(w_in), uniform(w_in), 0, lane16);
        else chain_products<SX::TC, SX::TP, 2, 3, false>(acc, wf, lds, q_of_x, rpq, uniform(w_in), uniform(w_in), 0, lane16);
        if constexpr (F48) fetch48<NCX>(wf, uniform(blockp), f48);
        else if constexpr (RING) {
            const gbytes p = uniform(one ? blockp + tblk * 9 * NCX * 1024 : blockp + bytes_one + xblk * 9 * NCT * 1024);
            static_for<NWF>([&](auto i_) { wf[decltype(i_)::value] = fragment(p, decltype(i_)::value, lane16); });
        } else if constexpr (NCT != 0) chain_fetch<ST::TC, NCX, 3, 0>(wf, uniform(blockp + tblk * 9 * NCX * 1024), lane16);
        chain_store<SX::TC, SX::TP, false>(acc, lds, xo, live_x, cst0, xblk * 32, half, a.act_unsigned);
        put_const(1, cn);
    }
    lds_barrier();
    if constexpr (NCT != 0) {
#pragma unroll 1
        for (int b = 0; b < a.blocks; ++b) {
            const bool last = b + 1 == a.blocks;
            const gbytes p_one = blockp + tblk * 9 * NCX * 1024, p_two = blockp + bytes_one + xblk * NT2 * NT2 * NCT * 1024;
            const gbytes next = last ? blockp : blockp + bytes_block;
            {
                const v4i cn = fetch_const(blockp + bytes_one + w_two);
                if constexpr (F48) {
                    v4i acc[3][TP48];
                    const int ch = (wave & 1) * 48 + (lane >> 4) * 4;
                    bias48(acc, cst1, ch);
                    const gbytes pn = uniform(p_two);
                    products48<TP48, NCX>(acc, wf, lds, x_of_48, rpx, uniform(blockp), f48, [&](auto i_) {
                        constexpr int i = decltype(i_)::value;
                        wf[i] = *(gv4i)(pn + i % 2 * tcs_two + (i / 2) * 1024 + lane16);
                    });
                    store48(acc, lds, to_48, live_48, cst1, ch, a.act_unsigned);
                } else if constexpr (RING) {
                    if (one) {
                        v16i acc[1][ST::TP];
                        chain_bias(acc, cst1, tblk, half);
                        const gbytes p1 = uniform(p_one), p2 = uniform(p_two);
                        chain_products_ring<ST::TP, NCX, 3>(acc, wf, lds, x_of_t, rpx, [&](auto i_) {
                            constexpr int i = decltype(i_)::value, ahead = i + NWF;
                            wf[i % NWF] = ahead < 36 ? fragment(p1, ahead, lane16) : fragment(p2, ahead - 36, lane16);
                        });
                        chain_store<1, ST::TP, false>(acc, lds, to, live_t, cst1, tblk * 32, half, a.act_unsigned);
                    }
                } else {
                    v16i acc[ST::TC][ST::TP];
                    chain_bias(acc, cst1, tblk, half);
                    chain_products<ST::TC, ST::TP, NCX, 3>(acc, wf, lds, x_of_t, rpx, uniform(p_one), uniform(p_two), tcs_two, lane16);
                    constexpr int got = carry_one ? chain_depth<ST::TC, NCX, 3>() * ST::TC : 0;
                    chain_fetch<SX::TC, NCT, NT2, got>(wf, uniform(p_two), lane16);
                    chain_store<ST::TC, ST::TP, false>(acc, lds, to, live_t, cst1, tblk * 32, half, a.act_unsigned);
                }
                put_const(0, cn);
            }
            lds_barrier();
            {
                const v4i cn = fetch_const(last ? blockp + bytes_block + a.n_blk_last * a.taps_last * NCX * 1024 : next + w_one);
                v16i acc[SX::TC][SX::TP];
                chain_bias(acc, cst0, xblk, half);
                unsigned at[SX::TP];  // a 1x1 kernel begins at the pixel itself
#pragma unroll
                for (int i = 0; i < SX::TP; ++i) at[i] = NT2 == 1 ? t_of_x[i] + rpt + pst : t_of_x[i];
                const gbytes p_next = next + tblk * 9 * NCX * 1024;
                if constexpr (F48) {
                    const gbytes pn = uniform(next);
                    chain_products_then<SX::TC, SX::TP, NCT, NT2>(acc, wf, lds, at, rpt, uniform(p_two), lane16, [&](auto i_) {
                        constexpr int i = decltype(i_)::value;
                        wf[i] = *(gv4i)(pn + f48.at[i % 3] + (i / 3) * 2048 + f48.lane);
                    });
                } else if constexpr (RING) {
                    // behind the last block: the last layer's first fragments, where it has as many
                    const gbytes pn = uniform(last ? (a.taps_last == 9 ? blockp + bytes_block + wave % a.n_blk_last * (36 * 1024) : blockp)
                                              : one ? p_next : next + bytes_one + xblk * 9 * NCT * 1024);
                    const gbytes p2 = uniform(p_two);
                    chain_products_ring<SX::TP, NCT, 3>(acc, wf, lds, at, rpt, [&](auto i_) {
                        constexpr int i = decltype(i_)::value, ahead = i + NWF;
                        wf[i % NWF] = ahead < 9 * NCT ? fragment(p2, ahead, lane16) : fragment(pn, ahead - 9 * NCT, lane16);
                    });
                } else {
                    chain_products<SX::TC, SX::TP, NCT, NT2>(acc, wf, lds, at, rpt, uniform(p_two), uniform(p_next), tcs_one, lane16);
                    constexpr int got = carry_one ? chain_depth<SX::TC, NCT, NT2>() * SX::TC : 0;
                    chain_fetch<ST::TC, NCX, 3, got>(wf, uniform(p_next), lane16);
                }
                chain_store<SX::TC, SX::TP, true>(acc, lds, xo, live_x, cst0, xblk * 32, half, a.act_unsigned);
                put_const(1, cn);
            }
            lds_barrier();
            blockp += bytes_block;
        }
    }

    // Last layer: few filters, every wave takes some of the pixels.
    auto last_layer = [&](auto share_, auto nt_) {
        using S = decltype(share_);
        constexpr int NT = decltype(nt_)::value, TP = S::TP;
        const int blk = wave % S::WC;
        const gbytes p = uniform(blockp + blk * NT * NT * NCX * 1024);
        constexpr bool carried = RING && NT == 3;
        if constexpr (!carried) chain_fetch<1, NCX, NT, 0>(wf, p, lane16);
        unsigned at[TP];
        int gp[TP];  // image * hw + pixel, or -1
        static_for<TP>([&](auto tp_) {
            constexpr int tp = decltype(tp_)::value;
            int im, row, col;
            const bool live = pixel_of((wave / S::WC * TP + tp) * 32 + l32, im, row, col);
            at[tp] = xb + im * isx + (row + (NT == 1)) * rpx + (col + (NT == 1)) * psx + half * 16;
            gp[tp] = live ? (img0 + im) * hw + row * w + col : -1;
        });
        int ix[16];
        chain_last_channels(a, ix, blk, half);
        v16i acc[1][TP];
        chain_bias(acc, cst1, blk, half);
        if constexpr (carried)
            chain_products_ring<TP, NCX, NT>(acc, wf, lds, at, rpx, [&](auto i_) {
                constexpr int i = decltype(i_)::value;
                if constexpr (i + NWF < 36) wf[i % NWF] = fragment(p, i + NWF, lane16);
            });
        else chain_products<1, TP, NCX, NT, false>(acc, wf, lds, at, rpx, p, p, 0, lane16);
        chain_last_store<TP>(a, acc, gp, ix, cst1, blk, half);
    };
    using I1 = std::integral_constant<int, 1>;
    using I3 = std::integral_constant<int, 3>;
    if (a.taps_last == 9) {
        if (a.n_blk_last == 1) last_layer(S1{}, I3{});
        else last_layer(S2{}, I3{});
    } else {
        if (a.n_blk_last == 1) last_layer(S1{}, I1{});
        else last_layer(S2{}, I1{});
    }
}

}  // namespace

template <int NW, int NCX, int NCT, int NT2, int TILES>
constexpr ChainKernel chain_kernel() {
    return ChainKernel{NCX, NCT, NCT ? NT2 * NT2 : 0, TILES, NW * 64, k_chain<NW, NCX, NCT, NT2, TILES>};
}
// The kernels of one kind of network, by tiles. Four waves read the fewest bytes for a product; over eight tiles
// eight waves are ahead all the same (16x16 maps at batch 256: 147 us against 150), because two waves of a SIMD fill
// each other's epilogue.
#define IODF_CHAIN_TABLE(NAME, NCX, NCT, NT2)                                                         \
    const ChainKernel NAME[kChainSizes] = {chain_kernel<4, NCX, NCT, NT2, 1>(), chain_kernel<4, NCX, NCT, NT2, 2>(), \
                                           chain_kernel<4, NCX, NCT, NT2, 4>(), chain_kernel<8, NCX, NCT, NT2, 8>()};

}  // namespace iodf
