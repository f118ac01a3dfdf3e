// Parameters and modes shared by the implicit-GEMM convolution kernels of the bf16 path: kernels_bf16_stream.hip, which streams
// the weights to registers, for layers of whole 128-row panels and 64-channel chunks (variant 0), kernels_bf16.hip, which stages
// them through LDS, for the others.
#pragma once

#include "device_common.h"

namespace demon {

constexpr int MAXSPAN = 64;    // largest (max tap offset - min tap offset) the LDS tiles are sized for

enum { MODE_ACT = 0,   // bias + Snake, bf16 out only                     (dilated conv of a residual unit)
       MODE_RES = 1,   // bias + residual add in fp32, half out in place  (1x1 conv of a residual unit)
       MODE_UP  = 2,   // bias, polyphase scatter, half out               (ConvTranspose1d)
       MODE_DOWN = 3, // bias, half out; columns step two input rows     (strided Conv1d on merged rows)
       MODE_PART = 4 };// MODE_DOWN with K in kConvParts parts: fp32 sums of each out, the bias in those of the first
// MODE_RES, MODE_UP and MODE_DOWN may in addition emit the activated operand of the next layer: EMIT = 0 none, else the
// operand format + 1 (1 bf16, 2 bf16 hi + lo, 3 half).  IN is the operand format of the input.

// No larger than it needs to be: the host bounds a call of empty launches (a gated call whose clips are skipped), and where it is slow to
// issue them (some processes are, from their start to their end) such a call of a 3 s window takes 82 to 84 us with the 144
// bytes that this and the grid come to, 86 to 88 with 152 and with 160, in turn in one process.
struct MfmaParams {
    const uint16_t* xa;      // activated input, 16-bit [rows][cin] in the kernel's IN format; lo plane at xa + in_lo_off
    const uint16_t* w;       // packed weight blocks
    const float* bias;
    hres_t* y;               // residual-stream output; MODE_RES: also the residual source (in place); unused in MODE_ACT
    union {
        uint16_t* ya;        // activated output in the kernel's EMIT format; lo plane at ya + out_lo_off
        float* part;         // MODE_PART: [row][part][cout]
    };
    const float* out_alpha; const float* out_inv_beta;   // Snake applied before writing ya
    const Slot* slots;
    int r_in, cin, cout, ntaps, tap0, tap_step, stride, nchunks, margin;
    int mtiles_x;            // > 0: blockIdx.x enumerates (column tile, row tile), see the kernel; 0: blockIdx.z = row tile
    bool y_dead;             // MODE_RES: y is read only, nothing after this layer reads the sum
    bool xcd_group;          // with mtiles_x: 1 = all row tiles of a column tile on one XCD, 0 = row tiles dealt over the XCDs
    unsigned w_bytes;
    long long in_lo_off, out_lo_off;     // element offsets of the lo planes
};

// MODE_PART: byte offset of a piece's sums in rows of kConvParts x cout floats, from its offset in rows of cout halves and its first
// channel.  A surplus piece of a tile stays out of range: the row of kOutOfRange, times sixteen, would wrap to an offset near
// 2 GiB, inside the sums of a large window.
constexpr unsigned kOutOfRange = 0xf8000000u;
__host__ __device__ constexpr unsigned part_voff(unsigned off, unsigned ch)
{
    return off >= kOutOfRange ? off : (off - ch * 2u) * (kConvParts * 2u) + ch * 4u;
}

// kernels_bf16_stream.hip: weights streamed to registers, on weights packed for the 128 x 128 tile (variant 0).  `rows` is the
// GEMM's M, `ncols` the most columns a window needs, `mode`, `in_fmt` and `emit` as the template arguments of the
// other kernels; `call_slots` the windows of the whole call, `n_slots` those of this launch; launches of more than `max_small`
// 128 x 128 tiles look for no smaller tile, except strided convs of up to 512 merged channels, which may take 128 x 64 unless
// `max_small` is 0.  Dilated convs of seven taps may take 256 x 128 whatever `max_small` is.
hipError_t launch_conv_stream(MfmaParams p, int mode, int in_fmt, int emit, int rows, long long ncols, int n_slots, int call_slots, long long max_small,
                              hipStream_t stream);

}  // namespace demon
