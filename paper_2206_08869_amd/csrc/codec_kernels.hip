// Prior masses (Sec. 3) and the streaming rANS coder (App. A) on the GPU.
//
// Prior of one latent z with 8-bit mean code m and log-scale code l: mu = 2 m, s = 2^(l/16),
// residual r = z - mu in [-8192, 8191]. Cumulative mass of the symbols below r:
//   G(r) = (r + 8192) + floor((M - 16384) * S((2r - 1) / (2s)) / 2^30),   M = 2^24,
// i.e. one unit of floor mass per symbol plus the logistic CDF at the symbol's lower edge,
// sigma((r - 1/2) / s). S is a 3073-entry table of 2^30 * sigma at steps of 1/64 on [-24, 24],
// interpolated linearly with floor. The symbol's masses are C = G(r), F = G(r + 1) - G(r) >= 1.
//
// Coder: 64-bit state X in [2^31, 2^63), initial 2^31. Encoding a symbol first sheds the low
// 32 bits as a word if X >= F * 2^39, then X <- floor(X / F) * M + C + X mod F. Decoding reads
// the slot X mod M, finds the symbol whose [C, C + F) holds it, restores
// X <- F * floor(X / M) + (X mod M) - C and pulls a word back in when X < 2^31.
// A chunk's latents are dealt round-robin to 16 lanes, each an independent stream encoded
// last-to-first. The chains are serial (encoding: one thread to a lane, what it is fed worked out
// by other waves; decoding: a wave to a lane, or half of one), so these kernels are bound by dependent
// integer latency, not by memory or the vector units.
#include "codec_kernels.h"

#include <cmath>

namespace iodf {

void codec_make_tables(int32_t* sig, int64_t* inv) {
    for (int j = 0; j < kSigEntries; ++j) {
        const long double t = ((long double)j - 1536.0L) / 64.0L;
        // sigma(t) written so that the exponential never overflows: e^t / (1 + e^t) for t < 0
        long double s;
        if (t < 0) {
            const long double e = std::exp(t);
            s = e / (1.0L + e);
        } else {
            s = 1.0L / (1.0L + std::exp(-t));
        }
        sig[j] = (int32_t)std::llround(std::ldexp(s, kSigBits));
    }
    for (int l = -128; l <= 127; ++l) inv[l + 128] = (int64_t)std::llround(std::exp2((368.0L - (long double)l) / 16.0L));
}

namespace {

constexpr long long kMass = 1LL << kMassBits;
constexpr unsigned long long kStateLow = 1ULL << 31;
constexpr int TPB = 256;

// The table in LDS has one entry more than its kSigEntries points, so that the last point has a neighbour too.
constexpr int kSigLds = kSigEntries + 1;

__device__ __forceinline__ void load_sig(int* s_sig, const int32_t* sig) {
    for (int i = threadIdx.x; i < kSigLds; i += blockDim.x) s_sig[i] = sig[i < kSigEntries ? i : kSigEntries - 1];
    __syncthreads();
}

// G(r) = (r + 8192) + floor((M - 16384) * S((2r - 1) * inv) / 2^30), S interpolated between the table's points with
// floor. Everything fits 32-bit products: the argument saturates at +-24 (24 << 24 in its units), where S is 0 and
// 2^30 exactly as the table's ends are; the interpolation's and the mass's shifts are folded into a factor so that the
// result is a product's high word.
__device__ __forceinline__ int cdf(const int* s_sig, int r, unsigned inv) {
    constexpr unsigned tmax = 24u << 24;
    const int t = 2 * r - 1;
    const unsigned a = (unsigned)(t < 0 ? -t : t), lo = a * inv;
    unsigned T = __umulhi(a, inv) ? tmax : lo;
    T = T < tmax ? T : tmax;
    const unsigned u = t < 0 ? tmax - T : tmax + T;
    const unsigned j = u >> 18, frac = u & ((1u << 18) - 1);
    const unsigned s0 = (unsigned)s_sig[j], s1 = (unsigned)s_sig[j + 1];
    const unsigned S = s0 + __umulhi(s1 - s0, frac << 14);
    return (r + kAlphaR) + (int)__umulhi((unsigned)(kMass - 2 * kAlphaR) << 2, S);
}

// codes of latent e of chunk c of one image
__device__ __forceinline__ void codes_of(const ChunkTable& ct, int c, const int8_t* codes_img, int e, int& m, int& l) {
    if (codes_img && ct.code_off[c] >= 0) {
        m = codes_img[ct.code_off[c] + e];
        l = codes_img[ct.code_off[c] + ct.n[c] + e];
    } else {
        m = kDefaultM;
        l = kDefaultL;
    }
}

__device__ __forceinline__ int residual(int z, int m, unsigned& clamped) {
    long long r = (long long)z - 2 * m;
    if (r < -kAlphaR) { r = -kAlphaR; ++clamped; }
    if (r > kAlphaR - 1) { r = kAlphaR - 1; ++clamped; }
    return (int)r;
}

__global__ __launch_bounds__(TPB) void k_prior_cf(const CodecTables t, const ChunkTable ct, const int32_t* __restrict__ z,
                                                  long long d, const int8_t* __restrict__ codes, long long d_codes,
                                                  int batch, int32_t* __restrict__ c_out, int32_t* __restrict__ f_out,
                                                  unsigned long long* errs) {
    __shared__ int s_sig[kSigLds];
    load_sig(s_sig, t.sig);
    unsigned clamped = 0;
    const long long total = (long long)batch * d;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total; i += (long long)gridDim.x * blockDim.x) {
        const int b = (int)(i / d);
        const long long q = i - (long long)b * d;
        int c = 0;
        while (c + 1 < ct.n_chunks && q >= ct.z_off[c + 1]) ++c;
        const int e = (int)(q - ct.z_off[c]);
        int m, l;
        codes_of(ct, c, codes ? codes + (long long)b * d_codes : nullptr, e, m, l);
        const int r = residual(z[i], m, clamped);
        const unsigned inv = (unsigned)t.inv[l + 128];
        const int C = cdf(s_sig, r, inv);
        c_out[i] = C;
        f_out[i] = cdf(s_sig, r + 1, inv) - C;
    }
    if (clamped) atomicAdd(errs, (unsigned long long)clamped);
}

// One workgroup per (image, chunk). A lane's coder is a serial chain (shed a word, divide, multiply, add), but what it
// is fed, the masses of its symbols, depends on nothing in it: the first wave runs the sixteen chains, one to a
// thread, and the other four work out the masses and reciprocals of the next kEncBlock symbols of every lane
// meanwhile. The chain's division X / F (63 by 24 bits, the quotient below 2^39) is a product with 1 / F in double
// precision, off by less than 1.01 in either direction, and one correction.
// Bound: the chain. paper_res64, up to 384 symbols a lane: 65 to 72 us at batch 1, 170 to 190 ns a symbol, the same
// with eight producing waves instead of four; at batch 256, four workgroups to a compute unit, 94 us, 245 ns (eight
// producing waves: 205 us, since two workgroups fit; a thread per lane that also fetched, looked up and divided: 443 us).
constexpr int kEncBlock = 32;
constexpr int kEncThreads = 320;

struct EncSymbol {
    unsigned c, f;  // f = 0: no symbol here
    double rcp;     // 1 / f
};

__global__ __launch_bounds__(kEncThreads) void k_rans_encode(const CodecTables t, const ChunkTable ct,
                                                             const int32_t* __restrict__ z, long long d,
                                                             const int8_t* __restrict__ codes, long long d_codes,
                                                             uint32_t* __restrict__ lane_words, long long lwpi,
                                                             uint32_t* __restrict__ lane_meta, unsigned long long* errs) {
    __shared__ int s_sig[kSigLds];
    __shared__ EncSymbol s_sym[2][kEncBlock * kLanes];
    load_sig(s_sig, t.sig);
    const int nslots = ct.n_chunks * kLanes;
    const int b = blockIdx.x / ct.n_chunks, c = blockIdx.x - b * ct.n_chunks;
    const int n = ct.n[c];
    const int kmax = (n + kLanes - 1) / kLanes, rounds = (kmax + kEncBlock - 1) / kEncBlock;
    const int32_t* zc = z + (long long)b * d + ct.z_off[c];
    const int8_t* ci = codes ? codes + (long long)b * d_codes : nullptr;
    const int j = threadIdx.x;  // the coder's lane (first wave, below kLanes)
    uint32_t* w = lane_words + (long long)b * lwpi + ct.lane_off[c] + (long long)(j & (kLanes - 1)) * ct.lane_cap[c];
    unsigned long long X = kStateLow;
    int nw = 0;
    unsigned clamped = 0;
    // round r holds the symbols at positions kmax - 1 - r * kEncBlock and below, in coding order
    auto produce = [&](int r) {
        for (int s = (int)threadIdx.x - 64; s < kEncBlock * kLanes; s += kEncThreads - 64) {
            const int p = kmax - 1 - r * kEncBlock - s / kLanes, e = p * kLanes + s % kLanes;
            EncSymbol y = {0u, 0u, 0.0};
            if (p >= 0 && e < n) {
                int m, l;
                codes_of(ct, c, ci, e, m, l);
                const int res = residual(zc[e], m, clamped);
                const unsigned inv = (unsigned)t.inv[l + 128];
                y.c = (unsigned)cdf(s_sig, res, inv);
                y.f = (unsigned)cdf(s_sig, res + 1, inv) - y.c;
                y.rcp = 1.0 / (double)y.f;
            }
            s_sym[r & 1][s] = y;
        }
    };
    if (threadIdx.x >= 64 && rounds > 0) produce(0);
    __syncthreads();
    for (int r = 0; r < rounds; ++r) {
        if (threadIdx.x >= 64) {
            if (r + 1 < rounds) produce(r + 1);
        } else if (threadIdx.x < kLanes) {
            EncSymbol y = s_sym[r & 1][j];
            for (int i = 0; i < kEncBlock; ++i) {
                const EncSymbol next = s_sym[r & 1][(i + 1 < kEncBlock ? i + 1 : i) * kLanes + j];
                if (y.f) {
                    if (X >= ((unsigned long long)y.f << 39)) {  // at most once per symbol, so nw <= k < lane_cap
                        w[nw++] = (uint32_t)X;
                        X >>= 32;
                    }
                    unsigned long long q = (unsigned long long)((double)X * y.rcp);
                    long long rem = (long long)(X - q * y.f);
                    if (rem < 0) { --q; rem += y.f; }
                    if (rem >= (long long)y.f) { ++q; rem -= y.f; }
                    X = q * (unsigned long long)kMass + y.c + (unsigned long long)rem;
                }
                y = next;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x < kLanes) {
        uint32_t* mt = lane_meta + ((long long)b * nslots + c * kLanes + j) * 4;
        mt[0] = (uint32_t)nw;
        mt[1] = (uint32_t)X;
        mt[2] = (uint32_t)(X >> 32);
        mt[3] = 0;
    }
    if (clamped) atomicAdd(errs, (unsigned long long)clamped);
}

// `parts` workgroups per image, each for some of the lanes. Container: [0] total words; [1 .. 1 + S) words per lane slot;
// then S pairs (state low, state high); then every slot's words in the order the decoder
// reads them (the reverse of the order they were shed). S = n_chunks * 16.
__global__ __launch_bounds__(TPB) void k_rans_pack(const ChunkTable ct, const uint32_t* __restrict__ lane_words,
                                                   long long lwpi, const uint32_t* __restrict__ lane_meta,
                                                   uint32_t* __restrict__ out, long long cap,
                                                   uint32_t* __restrict__ sizes, unsigned long long* errs, const int parts) {
    __shared__ long long s_off[kMaxChunks * kLanes + 1];
    static_assert(kMaxChunks * kLanes <= TPB, "a thread per slot");
    const int b = blockIdx.x / parts, part = blockIdx.x - b * parts;
    const int nslots = ct.n_chunks * kLanes;
    const long long header = 1 + 3LL * nslots;
    const uint32_t* mt = lane_meta + (long long)b * nslots * 4;
    // s_off[s] = words of the slots before s: an inclusive sum over at most 128 slots, one to a thread
    long long sum = (int)threadIdx.x < nslots ? (long long)mt[4 * threadIdx.x] : 0;
    for (int step = 1; step < nslots; step *= 2) {
        if ((int)threadIdx.x < nslots) s_off[threadIdx.x + 1] = sum;
        __syncthreads();
        if ((int)threadIdx.x < nslots && (int)threadIdx.x >= step) sum += s_off[threadIdx.x + 1 - step];
        __syncthreads();
    }
    if ((int)threadIdx.x < nslots) s_off[threadIdx.x + 1] = sum;
    if (threadIdx.x == 0) s_off[0] = 0;
    __syncthreads();
    const long long total = header + s_off[nslots];
    uint32_t* ob = out + (long long)b * cap;
    if (part == 0 && threadIdx.x == 0) {
        sizes[b] = (uint32_t)total;
        if (cap > 0) ob[0] = (uint32_t)total;
        if (total > cap) atomicAdd(errs + 1, 1ULL);
    }
    for (int s = threadIdx.x; part == 0 && s < nslots; s += blockDim.x) {
        if (1 + s < cap) ob[1 + s] = mt[4 * s];
        if (1 + nslots + 2 * s < cap) ob[1 + nslots + 2 * s] = mt[4 * s + 1];
        if (1 + nslots + 2 * s + 1 < cap) ob[1 + nslots + 2 * s + 1] = mt[4 * s + 2];
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
    for (int s = part * nwaves + wave; s < nslots; s += parts * nwaves) {
        const int c = s / kLanes, j = s % kLanes;
        const long long nw = s_off[s + 1] - s_off[s];
        const uint32_t* w = lane_words + (long long)b * lwpi + ct.lane_off[c] + (long long)j * ct.lane_cap[c];
        for (long long i = lane; i < nw; i += 64) {
            const long long dst = header + s_off[s] + i;
            if (dst < cap) ob[dst] = w[nw - 1 - i];
        }
    }
}

// A whole wave serves one lane, a workgroup four. What hangs on the state is then the same for all 64 threads: the state lives in
// scalar registers, counts come from whole ballots and picked values by v_readlane.
//
// A symbol is found by a guess that is then proved. Where G is all floor mass (13.86 s and more from the mean, the
// logistic's part below 16 of 2^24) the residual is the slot less a constant; elsewhere the logistic alone, inverted
// in single precision, is close. The threads work out G at 64 residuals around the guess, and a ballot shows whether the
// slot lies among them; if not (far from the mean, between the two regimes) the search over all residuals follows, 128
// cut points and then 128 residuals, two to a thread. What a position's codes mean for all this is worked out 64 positions at
// a time, one to a thread. Bound: the chain of some 60 instructions and one LDS read from one state to the next, 320 ns a
// symbol at batch 1. (Half a wave to a lane, three rounds of 32, 32 and 16 cut points, the first a symbol ahead: 500 ns and more.
// A whole wave with two rounds of 128: 440.) Whole calls, paper_iodf64 decode at batch 1 2150 -> 2025 us, cfg2 at batch 300
// 520 -> 495.
constexpr int kDecLanes = 4;

// cdf() with its argument clamped before and after one signed product. inv: min(inv, kTMax), which gives the same G since
// every argument is odd; cap: kTMax / inv + 1, from where on the argument saturates.
constexpr int kTMax = 24 << 24;
__device__ __forceinline__ int cdf_capped(const int* s_sig, int r, int inv, int cap) {
    int t = 2 * r - 1;
    t = t < -cap ? -cap : t > cap ? cap : t;
    t *= inv;  // |t| <= kTMax + inv < 2^30
    t = t < -kTMax ? -kTMax : t > kTMax ? kTMax : t;
    const unsigned u = (unsigned)(t + kTMax), j = u >> 18;
    const unsigned s0 = (unsigned)s_sig[j], s1 = (unsigned)s_sig[j + 1];
    const unsigned S = s0 + __umulhi(s1 - s0, u << 14);
    return (r + kAlphaR) + (int)__umulhi((unsigned)(kMass - 2 * kAlphaR) << 2, S);
}

__global__ __launch_bounds__(64 * kDecLanes) void k_rans_decode_chunk(const CodecTables t, const ChunkTable ct, const int c,
                                                                      const uint32_t* __restrict__ cont, long long cap, int batch,
                                                                      const int8_t* __restrict__ codes, long long d_codes,
                                                                      int32_t* __restrict__ z, long long d,
                                                                      unsigned long long* errs) {
    __shared__ int s_sig[kSigLds];
    load_sig(s_sig, t.sig);
    constexpr int kParts = kLanes / kDecLanes;
    const int b = blockIdx.x / kParts;  // grid = batch * kParts
    const int lane = threadIdx.x & 63;
    const int j = blockIdx.x % kParts * kDecLanes + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nslots = ct.n_chunks * kLanes;
    const long long header = 1 + 3LL * nslots;  // the host has checked cap >= header
    const uint32_t* cb = cont + (long long)b * cap;
    const int n = ct.n[c];
    const int k = __builtin_amdgcn_readfirstlane(j < n ? (n - j + kLanes - 1) / kLanes : 0);
    int32_t* zc = z + (long long)b * d + ct.z_off[c];
    const int8_t* const cm = codes && ct.code_off[c] >= 0 ? codes + (long long)b * d_codes + ct.code_off[c] : nullptr;
    const long long total = cb[0];
    bool bad = total > cap || total < header;
    const int slot = c * kLanes + j;
    // words of the lanes before this one: the wave adds them up together
    unsigned long long sum = 0;
    for (int s = lane; s < slot; s += 64) sum += cb[1 + s];
    for (int x = 32; x; x >>= 1) sum += __shfl_xor(sum, x, 64);
    const long long before = (long long)(((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(sum >> 32)) << 32) |
                                         (unsigned)__builtin_amdgcn_readfirstlane((int)sum));
    long long pos = header + before;
    unsigned nw = cb[1 + slot];
    if (bad || pos + (long long)nw > total) { bad = true; nw = 0; pos = header; }
    // 64 words or codes to a register, one to a thread, requested 64 words or positions before they are needed. Reads
    // stay below pos + nw <= total <= cap and below k: threads past the end repeat the last one.
    const uint32_t* const w = nw ? cb + pos : cb;
    unsigned used = 0;
    auto words_at = [&](unsigned i) { return w[nw ? (i + lane < nw ? i + lane : nw - 1) : 0u]; };
    unsigned w_cur = words_at(0), w_next = words_at(64);
    unsigned long long X = (unsigned long long)cb[1 + nslots + 2 * slot] |
                           ((unsigned long long)cb[1 + nslots + 2 * slot + 1] << 32);
    auto code_at = [&](int p, int what) -> int {
        if (!cm) return what ? kDefaultL : kDefaultM;
        return cm[what * n + (p + lane < k ? p + lane : k - 1) * kLanes + j];
    };
    // what a position's codes mean, one position to a thread
    struct Scale { int m2, inv, cap, tail; float s; };
    auto scale_of = [&](int m, int l) {
        Scale q;
        const int inv = t.inv[l + 128] < kTMax ? (int)t.inv[l + 128] : kTMax;  // 2^23 / scale, rounded
        const float scale = 8388608.0f / (float)inv;
        q.m2 = 2 * m;
        q.inv = inv;
        q.cap = kTMax / inv + 1;
        q.tail = (int)(13.86f * scale) + 1;
        q.s = 0.69314718f * scale;
        return q;
    };
    auto pick = [&](const Scale& q, int i) {
        return Scale{__builtin_amdgcn_readlane(q.m2, i), __builtin_amdgcn_readlane(q.inv, i), __builtin_amdgcn_readlane(q.cap, i),
                     __builtin_amdgcn_readlane(q.tail, i), __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q.s), i))};
    };
    if (k > 0) {
        Scale now = scale_of(code_at(0, 0), code_at(0, 1));
        int m_next = code_at(64, 0), l_next = code_at(64, 1);
        for (int p0 = 0; p0 < k; p0 += 64) {
            const int n_here = k - p0 < 64 ? k - p0 : 64;
            int out = 0;  // this thread's latent of the 64
            Scale q = pick(now, 0);
            for (int i = 0; i < n_here; ++i) {
                const int v = (int)(X & (unsigned long long)(kMass - 1));
                constexpr int A = (int)kMass - 2 * kAlphaR;  // mass of the logistic
                const int u = v - kAlphaR, uh = A - u;       // u = r + A * sigma, about
                // around the guess: 64 residuals from lo on, wholly inside the alphabet
                const float g = q.s * (__log2f((float)(u > 1 ? u : 1)) - __log2f((float)(uh > 1 ? uh : 1)));
                int lo = (int)fminf(fmaxf(g, -8192.0f), 8191.0f);
                lo = u < -q.tail ? u : u - A > q.tail ? u - A : lo;
                lo = (lo < -kAlphaR + 32 ? -kAlphaR + 32 : lo > kAlphaR - 32 ? kAlphaR - 32 : lo) - 32;
                int g0 = cdf_capped(s_sig, lo + lane, q.inv, q.cap);
                const Scale after = pick(now, (i + 1) & 63);
                int idx = __popcll(__ballot(g0 <= v)) - 1;
                int C, F;
                if (__builtin_expect(idx >= 0 && idx < 63, 1)) {
                    C = __builtin_amdgcn_readlane(g0, idx);
                    F = __builtin_amdgcn_readlane(g0, idx + 1) - C;
                } else {
                    // cut points -8192 + 128 (i + 1), i = lane and lane + 64; G(-8192) = 0 <= v < M = G(8192)
                    const int cut = -kAlphaR + (lane + 1) * 128;
                    const int seg = __popcll(__ballot(cdf_capped(s_sig, cut, q.inv, q.cap) <= v)) +
                                    __popcll(__ballot(cdf_capped(s_sig, cut + 64 * 128, q.inv, q.cap) <= v));
                    lo = -kAlphaR + seg * 128;
                    g0 = cdf_capped(s_sig, lo + lane, q.inv, q.cap);
                    const int g1 = cdf_capped(s_sig, lo + 64 + lane, q.inv, q.cap);
                    idx = __popcll(__ballot(g0 <= v)) + __popcll(__ballot(g1 <= v)) - 1;  // G(lo) <= v
                    // both edges of the symbol, worked out by every thread alike
                    C = __builtin_amdgcn_readfirstlane(cdf_capped(s_sig, lo + idx, q.inv, q.cap));
                    F = __builtin_amdgcn_readfirstlane(cdf_capped(s_sig, lo + idx + 1, q.inv, q.cap)) - C;
                }
                if (lane == i) out = lo + idx + q.m2;
                X = (unsigned long long)(unsigned)F * (X >> kMassBits) + (unsigned long long)(unsigned)(v - C);
                if (X >> 31 == 0) {  // below kStateLow
                    if (used < nw) {
                        X = (X << 32) | (unsigned)__builtin_amdgcn_readlane((int)w_cur, (int)(used & 63));
                        if ((++used & 63) == 0) {
                            w_cur = w_next;
                            w_next = words_at(used + 64);
                        }
                    } else { X <<= 32; bad = true; }
                }
                q = after;
            }
            if (p0 + lane < k) zc[(p0 + lane) * kLanes + j] = out;
            now = scale_of(m_next, l_next);
            m_next = code_at(p0 + 128, 0);
            l_next = code_at(p0 + 128, 1);
        }
    }
    if (X != kStateLow || used != nw) bad = true;
    if (bad && lane == 0) atomicAdd(errs + 2, 1ULL);
}

// The same for chunks of at most 32 symbols a lane, with half a wave to a lane and a workgroup to eight lanes. The 2^14 residuals
// are isolated in three rounds (32 * 32 * 16): in each the 32 threads work out G at 32 cut points of the current interval and a ballot
// counts how many lie at or below the slot; the last round works out G at every residual left, so the symbol's mass is two of its
// values. The first round's G (its cut points are the same for every symbol, only the scale differs) is worked out a symbol ahead.
//
// Its chain is longer (500 ns a symbol and more), but a wave brings two lanes on and has less to do before its first symbol. With
// more images than fill the chip's wave slots with a wave to a lane it is the issue of instructions that counts, and for short
// chunks this one is ahead (us, a wave to a lane against half of one): 4096 images of 12 latents 56 against 38, of 192 108 against 98, of two
// chunks of 384 350 to 356 against 326 to 345; 2048 58 against 53 (192), 188 to 192 against 176 to 188 (384). With 48 symbols a lane and more the guess
// pays again where it hits (4096 images of 768 latents 317 against 330, 2048 of two chunks of 1536 623 against 661) and costs little
// where it misses (631 against 625).
constexpr int kHalfLanes = 8, kHalfThreads = 32 * kHalfLanes;

__global__ __launch_bounds__(kHalfThreads) void k_rans_decode_half(const CodecTables t, const ChunkTable ct, const int c,
                                                                   const uint32_t* __restrict__ cont, long long cap, int batch,
                                                                   const int8_t* __restrict__ codes, long long d_codes,
                                                                   int32_t* __restrict__ z, long long d,
                                                                   unsigned long long* errs) {
    __shared__ int s_sig[kSigLds];
    __shared__ unsigned s_inv[256];
    for (int i = threadIdx.x; i < 256; i += kHalfThreads) s_inv[i] = (unsigned)t.inv[i];
    load_sig(s_sig, t.sig);
    constexpr int kParts = kLanes / kHalfLanes;
    const int b = blockIdx.x / kParts;  // grid = batch * kParts
    const int j = blockIdx.x % kParts * kHalfLanes + (threadIdx.x >> 5), helper = threadIdx.x & 31;
    const int half_shift = threadIdx.x & 32;  // this half's first bit in the wave's ballot, its first lane
    auto of_half = [&](int v, int i) { return __builtin_amdgcn_ds_bpermute((half_shift + i) << 2, v); };
    const int nslots = ct.n_chunks * kLanes;
    const long long header = 1 + 3LL * nslots;  // the host has checked cap >= header
    const uint32_t* cb = cont + (long long)b * cap;
    const int n = ct.n[c];
    const int k = j < n ? (n - j + kLanes - 1) / kLanes : 0;
    const int kmax = (n + kLanes - 1) / kLanes;  // the same for every thread, at most 32: ballots stay convergent
    const long long total = cb[0];
    bool bad = total > cap || total < header;
    const int slot = c * kLanes + j;
    // words of the lanes before this one: the half adds them up together
    long long before = 0;
    for (int s = helper; s < slot; s += 32) before += cb[1 + s];
    for (int x = 16; x; x >>= 1) before += __shfl_xor(before, x, 32);
    long long pos = header + before;
    unsigned nw = cb[1 + slot];
    if (bad || pos + (long long)nw > total) { bad = true; nw = 0; pos = header; }
    // a thread's word and codes, of the one position of the chunk that is its own (a symbol pulls in one word at most); reads stay
    // below pos + nw <= total <= cap
    const unsigned w_own = helper < nw ? cb[pos + helper] : 0u;
    int m = kDefaultM, l = kDefaultL;
    if (helper < k) codes_of(ct, c, codes ? codes + (long long)b * d_codes : nullptr, helper * kLanes + j, m, l);
    const int ml_own = (l << 16) | (m & 0xffff);  // mean code in the low half, log-scale code above it
    unsigned used = 0;
    unsigned long long X = (unsigned long long)cb[1 + nslots + 2 * slot] |
                           ((unsigned long long)cb[1 + nslots + 2 * slot + 1] << 32);
    // first round: cut points -8192 + (helper + 1) * 512; the last one is the interval's end, above every slot
    const int cut1 = -kAlphaR + (helper < 31 ? helper + 1 : 31) * 512;
    int ml = of_half(ml_own, 0);
    unsigned inv = s_inv[(ml >> 16) + 128];
    int g1 = cdf(s_sig, cut1, inv);
    int out = 0;  // this thread's latent
    for (int i = 0; i < kmax; ++i) {
        const int ml_after = of_half(ml_own, (i + 1) & 31);
        const unsigned word = (unsigned)of_half((int)w_own, (int)(used & 31));
        const unsigned inv_after = s_inv[(ml_after >> 16) + 128];
        const int v = (int)(X & (unsigned long long)(kMass - 1));
        // G(-8192) = 0 <= v < M = G(8192)
        unsigned below = (unsigned)(__ballot(helper < 31 && g1 <= v) >> half_shift);
        int lo = -kAlphaR + __popc(below) * 512;
        below = (unsigned)(__ballot(helper < 31 && cdf(s_sig, lo + (helper + 1) * 16, inv) <= v) >> half_shift);
        lo += __popc(below) * 16;
        const int g3 = cdf(s_sig, lo + (helper < 16 ? helper : 16), inv);
        below = (unsigned)(__ballot(helper >= 1 && helper < 16 && g3 <= v) >> half_shift);
        const int idx = __popc(below);
        const int C = of_half(g3, idx);
        const int F = of_half(g3, idx + 1) - C;
        g1 = cdf(s_sig, cut1, inv_after);
        if (helper == i) out = lo + idx + 2 * (int)(int16_t)(ml & 0xffff);
        if (i < k) {
            X = (unsigned long long)F * (X >> kMassBits) + (unsigned long long)(v - C);
            if (X < kStateLow) {
                if (used < nw) { X = (X << 32) | word; ++used; }
                else { X <<= 32; bad = true; }
            }
        }
        inv = inv_after;
        ml = ml_after;
    }
    if (helper < k) z[(long long)b * d + ct.z_off[c] + helper * kLanes + j] = out;
    if (X != kStateLow || used != nw) bad = true;
    if (bad && helper == 0) atomicAdd(errs + 2, 1ULL);
}

int grid_for(long long n, int tpb) {
    long long g = (n + tpb - 1) / tpb;
    if (g > 256 * 16) g = 256 * 16;
    return g < 1 ? 1 : (int)g;
}

bool table_ok(const ChunkTable& ct) { return ct.n_chunks >= 1 && ct.n_chunks <= kMaxChunks; }

}  // namespace

hipError_t launch_prior_cf(const CodecTables& t, const ChunkTable& ct, const int32_t* z, long long d,
                           const int8_t* codes, long long d_codes, int batch, int32_t* c_out, int32_t* f_out,
                           unsigned long long* errs, hipStream_t st) {
    if (batch <= 0) return hipSuccess;
    if (!table_ok(ct) || !z || !c_out || !f_out || !errs || !t.sig || !t.inv) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_prior_cf, dim3(grid_for((long long)batch * d, TPB)), dim3(TPB), 0, st, t, ct, z, d, codes, d_codes,
                       batch, c_out, f_out, errs);
    return hipGetLastError();
}

hipError_t launch_rans_encode(const CodecTables& t, const ChunkTable& ct, const int32_t* z, long long d,
                              const int8_t* codes, long long d_codes, int batch, uint32_t* lane_words,
                              long long lane_words_per_image, uint32_t* lane_meta, unsigned long long* errs,
                              hipStream_t st) {
    if (batch <= 0) return hipSuccess;
    if (!table_ok(ct) || !z || !lane_words || !lane_meta || !errs || !t.sig || !t.inv) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_rans_encode, dim3((unsigned)batch * ct.n_chunks), dim3(kEncThreads), 0, st, t, ct, z, d, codes,
                       d_codes, lane_words, lane_words_per_image, lane_meta, errs);
    return hipGetLastError();
}

hipError_t launch_rans_pack(const ChunkTable& ct, const uint32_t* lane_words, long long lane_words_per_image,
                            const uint32_t* lane_meta, int batch, uint32_t* out, long long cap, uint32_t* sizes,
                            unsigned long long* errs, hipStream_t st) {
    if (batch <= 0) return hipSuccess;
    if (!table_ok(ct) || !lane_words || !lane_meta || !out || !sizes || !errs || cap < 0) return hipErrorInvalidValue;
    // One workgroup for all lanes copies their words one lane behind the other, while few images leave the chip idle; each further one
    // works out all lanes' offsets again. As many as give 2048 of them at most (us, one / two / four to an image: 128 images of 64x64
    // 18.3 / 11.6 / 9.1, 1024 31.5 / 24.2 / 26.1, 2048 43.6 / 43.6 / 45.8; of 8x8, 512 7.1 / 7.3 / 6.8, 1024 7.6 / 8.2 / 9.7, 4096 13.5 / 18.2 / 24.2).
    const int parts = batch <= 512 ? 4 : batch <= 1024 ? 2 : 1;
    hipLaunchKernelGGL(k_rans_pack, dim3((unsigned)batch * parts), dim3(TPB), 0, st, ct, lane_words, lane_words_per_image, lane_meta, out,
                       cap, sizes, errs, parts);
    return hipGetLastError();
}

hipError_t launch_rans_decode_chunk(const CodecTables& t, const ChunkTable& ct, int c, const uint32_t* cont,
                                    long long cap, int batch, const int8_t* codes, long long d_codes, int32_t* z,
                                    long long d, unsigned long long* errs, int n_cu, hipStream_t st) {
    if (batch <= 0) return hipSuccess;
    if (!table_ok(ct) || c < 0 || c >= ct.n_chunks || !cont || !z || !errs || !t.sig || !t.inv ||
        cap < 1 + 3LL * ct.n_chunks * kLanes)
        return hipErrorInvalidValue;
    if (rans_decode_by_halves(ct, c, batch, n_cu))
        hipLaunchKernelGGL(k_rans_decode_half, dim3((unsigned)batch * (kLanes / kHalfLanes)), dim3(kHalfThreads), 0, st, t, ct, c, cont, cap,
                           batch, codes, d_codes, z, d, errs);
    else
        hipLaunchKernelGGL(k_rans_decode_chunk, dim3((unsigned)batch * (kLanes / kDecLanes)), dim3(64 * kDecLanes), 0, st, t, ct, c, cont, cap,
                           batch, codes, d_codes, z, d, errs);
    return hipGetLastError();
}

}  // namespace iodf
