// Device code the convolution kernels share: vector types, compile-time loops, the fixed-point requantise and the
// arithmetic of the fast epilogues.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <stddef.h>

#include <type_traits>

#include "conv.h"

namespace iodf {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// Global memory by type: a pointer rebuilt from scalar halves would otherwise be a generic one, whose loads also
// count as LDS operations.
typedef const uint8_t __attribute__((address_space(1)))* gbytes;
typedef const v4i __attribute__((address_space(1)))* gv4i;

__device__ __forceinline__ gbytes uniform(gbytes p) {
    const unsigned long long v = (unsigned long long)p;
    return (gbytes)(((unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(v >> 32)) << 32) |
                    (unsigned)__builtin_amdgcn_readfirstlane((unsigned)v));
}

// Compile-time loop: f(std::integral_constant<int, I>) for I = 0..N-1. Keeps every
// accumulator index a constant so the accumulators stay in registers.
template <int I, int N, class F>
__device__ __forceinline__ void static_for_impl(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for_impl<I + 1, N>(f);
    }
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl<0, N>(f);
}

// Reads one word of every 128-byte line of p, lines first, first + stride, ..., so that they sit in this XCD's L2. Four
// independent loads at a time: a thread pays one memory latency a round and not one a line.
__device__ __forceinline__ void touch_lines(const uint8_t* p, const unsigned lines, const unsigned first, const unsigned stride) {
    int sum = 0;
    for (unsigned l = first; l < lines; l += 4 * stride) {
#pragma unroll
        for (unsigned u = 0; u < 4; ++u)
            if (l + u * stride < lines) sum += *(const int*)(p + ((size_t)(l + u * stride) << 7));
    }
    asm volatile("" ::"v"(sum));  // the loads are the point: keep them
}

// Round-half-away-from-zero of acc * M / 2^s, clamped far outside the 8-bit range
// (the caller saturates to 8 bit after adding at most one 8-bit shortcut).
__device__ __forceinline__ int rq_dev(int acc, int M, int s) {
    long long v = (long long)acc * (long long)M;
    long long half = s > 0 ? (1LL << (s - 1)) : 0LL;
    long long r = v >= 0 ? ((v + half) >> s) : -((-v + half) >> s);
    r = r > (1 << 20) ? (1 << 20) : r;
    r = r < -(1 << 20) ? -(1 << 20) : r;
    return (int)r;
}

__device__ __forceinline__ int sat8_dev(int v) { return v > 127 ? 127 : (v < -128 ? -128 : v); }

// Four outputs of one lane, registers I .. I + 3 of its accumulators, requantised and packed into a dword of codes.
// B: clamp bound, M: multiplier, S: shift - 32, R: rounding constant 2^(shift - 33) of the four channels.
template <int I, class Acc>
__device__ __forceinline__ unsigned pack_relu_quad(const Acc& acc, std::integral_constant<int, I>, const v4i& Bq, const v4i& Mq,
                                                   const v4i& Sq, const unsigned (&Rq)[4], const bool out_unsigned) {
    // ReLU without shortcut. The accumulators already hold the bias. Clamping them to
    // [0, hi] first (hi = the smallest value that requantises to 127; the rescale is
    // monotone and steps by at most 1) replaces both the ReLU and the saturation, so
    // every result fits a byte and the last shift can drop it straight into its place
    // in the packed dword.
    unsigned q[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        int av;
        asm("v_med3_i32 %0, %1, 0, %2" : "=v"(av) : "v"(acc[I + e]), "v"(Bq[e]));
        q[e] = __umulhi((unsigned)av, (unsigned)Mq[e]) + Rq[e];
    }
    unsigned p4 = q[0] >> Sq[0];
    asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD "
        "src1_sel:DWORD" : "+v"(p4) : "v"(Sq[1]), "v"(q[1]));
    asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD "
        "src1_sel:DWORD" : "+v"(p4) : "v"(Sq[2]), "v"(q[2]));
    asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD "
        "src1_sel:DWORD" : "+v"(p4) : "v"(Sq[3]), "v"(q[3]));
    return out_unsigned ? p4 ^ 0x80808080u : p4;  // code u is stored as u - 128
}

// NO_TIES: no accumulator of the layer lands exactly between two codes. Rounding half away from zero is then rounding
// half up, one arithmetic shift of the (floored) high word, and the sign needs no handling of its own.
template <bool NO_TIES, int I, class Acc>
__device__ __forceinline__ unsigned pack_signed_quad(const Acc& acc, std::integral_constant<int, I>, const v4i& Mq, const v4i& Sq,
                                                     const unsigned (&Rq)[4], const int sc, const int lo2) {
    // Signed results: a shortcut and / or no ReLU. The accumulators hold the bias. In
    // stored bytes the result is clamp(rq(acc) + shortcut byte, lo, 127): for signed codes
    // lo is 0 with a ReLU and -128 without; for unsigned codes (stored as code - 128, which
    // only occur here together with a shortcut of the same format) the two offsets of 128
    // cancel and ReLU plus saturation to [0, 255] is the clamp to [-128, 127]. The shortcut
    // byte is added sign-extended straight out of its dword and the clamp's second half
    // drops the byte into the packed dword.
    unsigned p4 = 0;
    static_for<4>([&](auto e_) {
        constexpr int e = decltype(e_)::value;
        const int av = acc[I + e];
        int r;
        if constexpr (NO_TIES) {
            r = (__mulhi(av, Mq[e]) + (int)Rq[e]) >> Sq[e];
        } else {
            const int sgn = av >> 31;
            const unsigned q = (__umulhi((unsigned)((av ^ sgn) - sgn), (unsigned)Mq[e]) + Rq[e]) >> Sq[e];
            r = ((int)q ^ sgn) - sgn;
        }
        int t;
        if constexpr (e == 0)
            asm("v_add_u32_sdwa %0, %1, sext(%2) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD "
                "src1_sel:BYTE_0" : "=v"(t) : "v"(r), "v"(sc));
        else if constexpr (e == 1)
            asm("v_add_u32_sdwa %0, %1, sext(%2) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD "
                "src1_sel:BYTE_1" : "=v"(t) : "v"(r), "v"(sc));
        else if constexpr (e == 2)
            asm("v_add_u32_sdwa %0, %1, sext(%2) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD "
                "src1_sel:BYTE_2" : "=v"(t) : "v"(r), "v"(sc));
        else
            asm("v_add_u32_sdwa %0, %1, sext(%2) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD "
                "src1_sel:BYTE_3" : "=v"(t) : "v"(r), "v"(sc));
        t = t < lo2 ? lo2 : t;
        const int hi2 = 127;
        if constexpr (e == 0)
            asm("v_min_i32_sdwa %0, %1, %2 dst_sel:BYTE_0 dst_unused:UNUSED_PRESERVE src0_sel:DWORD "
                "src1_sel:DWORD" : "+v"(p4) : "v"(t), "v"(hi2));
        else if constexpr (e == 1)
            asm("v_min_i32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD "
                "src1_sel:DWORD" : "+v"(p4) : "v"(t), "v"(hi2));
        else if constexpr (e == 2)
            asm("v_min_i32_sdwa %0, %1, %2 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD "
                "src1_sel:DWORD" : "+v"(p4) : "v"(t), "v"(hi2));
        else
            asm("v_min_i32_sdwa %0, %1, %2 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD "
                "src1_sel:DWORD" : "+v"(p4) : "v"(t), "v"(hi2));
    });
    return p4;
}

// Epilogue variants a kernel is compiled for.
enum { EPI_ANY = 0, EPI_FAST = 1, EPI_FAST_RELU = 2 };

// Brings the arguments into registers in one go. Left alone they are loaded where first used, several memory latencies one
// behind the other, the last of them in the epilogue (with conv_igemm_direct's divisions out of its prologue as well: cfg5 at
// batch 1 2660 -> 2440 us, mid_dense 337 -> 307; conv_igemm_lean: cfg3 inverse at batch 50 7140 -> 7005).
__device__ __forceinline__ void hold_args(const ConvArgs& a) {
    asm volatile("" ::"s"(a.in), "s"(a.wgt), "s"(a.bias), "s"(a.mul), "s"(a.shift), "s"(a.clamp_hi), "s"(a.partial), "s"(a.out), "s"(a.idx_b),
                 "s"(a.in_plane), "s"(a.npix), "s"(a.cin_pad), "s"(a.n_pad), "s"(a.n_store), "s"(a.state_c));
    const unsigned* const raw = (const unsigned*)&a;  // in_chunk0, h, w, n_cu and the bit fields
    static_assert(offsetof(ConvArgs, in_chunk0) == 104 && sizeof(ConvArgs) == 120, "raw[26 .. 28]");
    asm volatile("" ::"s"(raw[26]), "s"(raw[27]), "s"(raw[28]));
}

// Pixel index m -> position of the pixel in the zero-bordered image stack, (b * PP + (i+1) * W2 + (j+1)).
// Image sides that are powers of two take shifts; others divide.
__device__ __forceinline__ int bordered_pos(const ConvArgs& a, int m, int hw, int W2, int PP) {
    int b, i, j;
    if (a.log2_w >= 0 && a.log2_hw >= 0) {
        b = m >> a.log2_hw;
        const int q = m & (hw - 1);
        i = q >> a.log2_w;
        j = q & (a.w - 1);
    } else {
        b = m / hw;
        const int q = m - b * hw;
        i = q / a.w;
        j = q - i * a.w;
    }
    return b * PP + (i + 1) * W2 + (j + 1);
}

// Timeline of one output tile (see ConvArgs::trace): stamp `which` of slot `slot`.
__device__ __forceinline__ void trace_stamp(const ConvArgs& a, int slot, int which, int tid) {
    if (a.has_trace && tid == 0) {
        a.trace[8LL * slot + which] = (long long)wall_clock64();
        if (which == 0) a.trace[8LL * slot + 4] = (long long)clock64();
        if (which == 3) a.trace[8LL * slot + 5] = (long long)clock64();
    }
}

}  // namespace iodf
