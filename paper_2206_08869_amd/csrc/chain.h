// Launch description of a whole narrow network that one workgroup per group of images runs out of LDS (see chain.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace iodf {

constexpr size_t kChainMaxLds = 160 * 1024;
constexpr int kChainMaxTiles = 8;  // 32-pixel tiles of a workgroup
constexpr int kChainConstBytes = 4 * 128 * (int)sizeof(int32_t);

// Bytes a pixel of a tensor with 32 * nc channels takes in LDS: 16 more than its channels, so that the 16-byte
// reads of neighbouring pixels touch different banks.
constexpr unsigned chain_pixel_bytes(int nc) { return nc ? nc * 32 + 16 : 0; }
// A row of w pixels and two of padding, and an image of hw pixels in `rows` such rows: stretched so that the first
// pixel of a row (image) lies, modulo the 64 LDS banks, where the pixel behind the last one of the row (image)
// before would. A read of 32 consecutive pixels then has the banks of one unbroken run, however often it wraps.
__host__ __device__ constexpr unsigned chain_row_bytes(int w, unsigned ps) { return (w + 2) * ps + ((0u - 2 * ps) & 255u); }
__host__ __device__ constexpr unsigned chain_image_bytes(int h, int w, unsigned ps) {
    return ps ? (h + 2) * chain_row_bytes(w, ps) + ((h * w * ps - (h + 2) * chain_row_bytes(w, ps)) & 255u) : 0u;
}

// How the waves of a workgroup divide n_blk blocks of 32 channels x `tiles` tiles of 32 pixels: share_blocks blocks to a
// wave, and as many tiles as it takes; share_tiles is what all waves together then run, `tiles` or more. One block to a
// wave reads the fewest weights but every pixel four times, which over four tiles and more is all that LDS delivers; two
// blocks halve that (strips of 32x32 maps at batch 256, whole call: 8920 -> 8707 us for four tiles).
__host__ __device__ constexpr int share_blocks(int n_blk, int tiles) { return n_blk == 4 && tiles >= 4 ? 2 : 1; }
__host__ __device__ constexpr int share_tiles(int waves, int n_blk, int tiles) {
    const int wp = waves / (n_blk / share_blocks(n_blk, tiles));
    return (tiles + wp - 1) / wp * wp;
}

// Parameters of a network, one block: for every layer its weights and then its constants, in the order first layer,
// (first, second convolution) of every residual block, last layer. Weights are fragments of 1 KB,
// [n_blk][taps * nc][64 lanes][16 bytes]: lane l of fragment (blk, tap * nc + c) holds, for filter 32 * blk + l % 32,
// the channels 32 * c + 16 * (l / 32) .. + 15 of that tap. Constants are int32 [4][128]: clamp bound, multiplier,
// shift, bias; the shift is stored minus 32 except in the last layer.
struct ChainArgs {
    const uint8_t* params;
    int32_t* state;      // int32 pixel-major [npix][state_c]
    const int32_t* idx;  // physical channel of logical channel c; the translation channels begin at n_a
    int8_t* codes;       // nullptr: the last layer adds into the state; else head codes as in conv.h
    long long codes_img_stride, codes_off;
    unsigned pf_bytes;   // size of the block, for the workgroups that fetch it ahead
    int batch, mul_in;
    // bit fields, so that they come out of whole words by scalar loads (bytes and halves took a vector load's latency)
    unsigned h : 16, w : 16;
    unsigned images : 16;  // images of a workgroup
    unsigned blocks : 16;
    unsigned n_a : 16, n_out : 16;
    unsigned state_c : 16, shift_in : 8;
    unsigned taps_two : 4, taps_last : 4;          // 1 or 9
    unsigned nc_x : 4, nc_t : 4, nc_q : 4;         // 32-channel chunks of the stream, the block-internal tensor (0: no blocks), the quantised input
    unsigned n_blk_last : 4;                       // 32-filter blocks of the last layer
    unsigned pf_blocks : 8;
    unsigned act_unsigned : 1, relu_last : 1;
    unsigned last_fast : 1;  // the last layer's shifts are all 33 or more and nothing in it requantises to half a code
    int sign : 2;
};
static_assert(sizeof(ChainArgs) == 80, "five words of fields");

// One kernel: the kind of network it runs, and the 32-pixel tiles its workgroup takes. The tables, one to a kind, are
// spread over several source files because compiling them takes a while.
struct ChainKernel {
    int nc_x, nc_t, taps_two, tiles, threads;
    void (*kern)(const ChainArgs);
};
constexpr int kChainSizes = 4;  // 1, 2, 4 and 8 tiles
extern const ChainKernel kChain433[2], kChain443[], kChain423[], kChain223[], kChain441[], kChain421[], kChain221[], kChain40[], kChain20[];

// A network of the same kinds whose images are too large for one workgroup, or too few to fill the chip with whole
// ones: strips of `rows` rows of an image. The stream x lives in planes as in conv.h and every launch below takes it from
// one buffer to another: first layer (input quantiser included), one residual block, last layer.
struct StripArgs {
    const uint8_t* params;  // the layer's (block's) weights and constants, laid out as for ChainArgs
    const int8_t* in;
    int8_t* out;
    int32_t* state;
    const int32_t* idx;
    int8_t* codes;
    long long codes_img_stride, codes_off;
    const uint8_t* pf;        // what the next launch reads first
    unsigned pf_bytes;
    unsigned plane;
    int batch, mul_in;
    unsigned h : 16, w : 16;
    unsigned rows : 16, chunk : 16;  // chunk: strips per XCD
    unsigned n_a : 16, n_out : 16;
    unsigned state_c : 16, shift_in : 8, pf_blocks : 8;  // pf_blocks: workgroups per XCD behind the strips that bring pf .. pf + pf_bytes into its L2
    unsigned taps_last : 4, nc_q : 4, n_blk_last : 4, act_unsigned : 1, relu_last : 1, last_fast : 1;
    unsigned run : 8;  // strips that a workgroup takes one below the other (blocks; see strip_max_run), else 1
    int sign : 2;
};
static_assert(sizeof(StripArgs) == 112, "five words of fields");
struct StripKernel {
    int nc_x, nc_t, taps_two;
    int tiles_one, tiles_two;  // 32-pixel tiles of the block's first and second convolution (first and last layer: the same)
    void (*kern)(const StripArgs);
    void (*kern_run)(const StripArgs);  // blocks: the form that takes several strips, or nullptr
};
constexpr int kStripThreads = 256;
constexpr int kStripMaxUnits = 8 * 65535;  // strips of a launch: StripArgs::chunk has 16 bits
constexpr size_t kStripMaxLds = 80 * 1024;  // two workgroups to a CU
constexpr int kStripMaxTiles = 6;  // tiles_one of the largest block kernel
// The largest kernel of 3x3 blocks, the one that launches of several rounds of strips take.
__host__ __device__ constexpr bool strip_largest(int taps_two, int tiles_one) { return taps_two == 9 && tiles_one == kStripMaxTiles; }
constexpr int kStripRunLoads = 5, kStripRunCopies = 3;  // 16-byte pieces a thread moves between two strips of a run: new rows; two rows of x, of t
constexpr int kStripSizes = 5, kStripIns = 8, kStripLasts = 4;
extern const StripKernel kStrip433[], kStrip443[], kStrip423[], kStrip223[], kStrip441[], kStrip421[], kStrip221[];
extern const StripKernel kStripIn[], kStripLast[];  // (nc_t of a first layer's kernel: chunks of the quantised input)

size_t chain_lds_bytes(const ChainArgs& a);
// Tiles of the kernel for this network and this many images per workgroup; 0: there is none.
int chain_tiles(const ChainArgs& a);
hipError_t launch_chain(const ChainArgs& a, hipStream_t stream);
// Multiply-accumulates the matrix cores run for a launch: whole tiles, padded widths.
long long chain_issued_macs(const ChainArgs& a);
// The kernel for strips of `rows` rows of h x w images, or nullptr: `block` of the residual networks with these widths,
// or one of the ends (nc_t and taps_two unused).
enum StripPart { STRIP_IN, STRIP_BLOCK, STRIP_LAST };
const StripKernel* strip_kernel_for(StripPart part, int nc_x, int nc_t, int taps_two, int nc_q, int h, int w, int rows);
// Strips of `rows` rows that one workgroup of this block kernel can take one below the other: those of an image, or 1.
int strip_max_run(const StripKernel& k, int h, int w, int rows);
hipError_t launch_strip(StripPart part, const StripKernel* k, const StripArgs& a, hipStream_t stream);
long long strip_issued_macs(StripPart part, const StripKernel& k, const StripArgs& a);
hipError_t chain_setup();

}  // namespace iodf
