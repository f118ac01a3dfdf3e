// Internal declarations shared by the host code and the kernel launchers of libdemon_vae.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "../../include/demon_vae.h"

namespace demon {

// ---- error reporting -------------------------------------------------------------------------
demon_status fail(demon_status st, const char* fmt, ...);   // records the thread-local message
void clear_error();

// ---- layer stack (host) ----------------------------------------------------------------------
struct Stack {
    int c0 = 0;
    std::vector<int> strides, widths, dilations;
    int res_kernel = 7, head_kernel = 7, out_channels = 2;
    int total_stride() const { int s = 1; for (int v : strides) s *= v; return s; }
};

// Validates the description and copies it. Returns DEMON_OK or INVALID_ARG (message recorded).
demon_status stack_from_config(const demon_vae_config* cfg, Stack* out);
size_t stack_weight_count(const Stack& st);
void stack_receptive_field(const Stack& st, int* left, int* right);
void stack_forward_support(const Stack& st, long long a, long long b, long long* lo, long long* hi);
size_t stack_encoder_weight_count(const Stack& st);
// halo of the windowed encode in latent frames and (optional) the cone in samples before / after a frame
void stack_encoder_receptive_field(const Stack& st, int* left, int* right, long long* samples_left, long long* samples_right);

// ---- windows ---------------------------------------------------------------------------------
// One extended window ("slot") as the kernels see it.  Frames are latent frames; at a level with
// R samples per frame the slot owns workspace rows [row0*R, (row0+len)*R).
struct Slot {
    int row0;     // first workspace frame of the slot (prefix sum of len)
    int len;      // extended length hi - lo
    int clip;
    int lo;       // first latent frame of the extended region
    int crop;     // begin - lo: frames trimmed on the left
    int n_int;    // end - begin: interior frames
    int begin;    // interior start (absolute frame)
    int pad;
};

// ---- kernels (launchers; all asynchronous on `stream`) -----------------------------------------
// Activations live in "row-major time x channels" layout: element (row, c) at row*C + c.

// MFMA operand formats of the bf16 path.  Weights are bf16 values in every format (exact in half as well).
enum OperandFmt { OP_BF16 = 0,     // one bf16 plane
                  OP_BF16X2 = 1,   // hi + lo bf16 planes, two MFMAs per k-step
                  OP_F16 = 2 };    // one IEEE half plane, f16 MFMA

// bytes past a layer's packed weights that its kernel may request (and not use), see weight_rsrc; the parameter allocation ends
// with as many
constexpr unsigned kWeightSlack = 256 * 1024;

struct ConvArgs {
    const void* x;        // activated input [rows_in, cin] (fp32 path: fp32; bf16 path: 16-bit operand)
    void* y;              // output activation [rows_out, cout] (fp32 path: fp32; bf16 path: half); bf16 dilated conv: unused
    void* ya = nullptr;   // activated copy of the output for the next layer (Snake out_alpha/out_inv_beta); fp32 path: fp32
    const void* res;      // residual (same layout as y) or nullptr; bf16 path: must equal y (in place)
    bool y_dead = false;  // bf16 path, with res: y is only read, the sum goes to ya alone
    float* part = nullptr;// bf16 path, strided conv: fp32 sums of the parts of K, [row][kConvParts][cout], instead of y and ya
    const void* w;        // packed weights (layout private to each kernel family)
    const float* bias;    // [cout]
    const float* out_alpha;  const float* out_inv_beta;   // Snake applied before writing ya, or nullptr
    const Slot* slots;    // device
    int n_slots;
    int call_slots;       // windows of the whole call: its launches run beside those of the other group, see two_groups in api.hip
    int max_len;          // longest slot (frames)
    int max_int;          // longest interior (frames)
    int margin;           // rows of the OUTPUT level beyond each window's interior that later layers still
                          // read (the shrinking cone of the receptive field); rows further out are not computed
    int r_in;             // samples per frame of the input level
    int cin, cout;
    int ntaps;            // conv: kernel size; convT: 2
    int dil;              // conv: dilation; convT: unused
    int stride;           // 0 = Conv1d; s > 0 = ConvTranspose1d(kernel 2s, stride s, padding s/2)
    int down = 0;         // s > 0 = strided Conv1d(kernel 2s, stride s, padding s/2) (the encoder); ntaps = 2s, stride = 0
    // bf16 path only: format of the MFMA operand read (x) and of the one emitted (ya), see kernels_bf16.hip
    int in_fmt = OP_BF16, out_fmt = OP_BF16;
    long long in_lo_off = 0, out_lo_off = 0;     // OP_BF16X2: element offset of the lo plane
    long long small_tile_wgs = 1024;             // bf16 path: launches of more 128 x 128 tiles than this look for no smaller tile (conv_bf16.h)
};

// fp32 implicit GEMM on an activated input; y: the residual stream (or nullptr), ya: fp32 operand of the next layer (or nullptr)
hipError_t launch_conv_f32(const ConvArgs& a, hipStream_t stream);
// a residual unit (dilated conv, 1x1 conv) in one kernel, where res_unit_f32_fuses()
bool res_unit_f32_fuses(const ConvArgs& d, const ConvArgs& p);
hipError_t launch_res_unit_f32(const ConvArgs& d, const ConvArgs& p, hipStream_t stream);
// bf16 MFMA implicit GEMM.  `variant` is the tile configuration chosen when the weights were packed.
hipError_t launch_conv_bf16(const ConvArgs& a, int variant, hipStream_t stream);

// Packed weight sizes / packing (host).  w_src is the PyTorch layout: conv [cout, cin, k]; convT [cin, cout, 2s].
size_t packed_f32_count(int cin, int cout, int ntaps, int stride);
void pack_f32(const float* w_src, int cin, int cout, int ntaps, int stride, float* dst);
int  choose_variant_bf16(int cin, int m);   // -1 if unsupported
size_t packed_bf16_count(int cin, int cout, int ntaps, int stride, int variant);
// `as_half`: the 16-bit weights are IEEE half (for a layer whose activation operand is OP_F16), else bf16.
// `permute_rows`: row order of launch_conv_bf16's accumulator tiles (not for the layouts the fused units read).
// `down` = s > 0: a strided Conv1d [cout, cin, 2s] in its merged-row form (see kernels_bf16.hip); ntaps, stride unused.
void pack_bf16(const float* w_src, int cin, int cout, int ntaps, int stride, int variant, bool as_half, bool permute_rows,
               uint16_t* dst, int down = 0);
// The layouts of pack_bf16 / pack_w1_* are row-major within a block; the kernels read every block in fragment order.
// variant_block: rows and K values of a block of a variant's layout.
void to_fragment_order(uint16_t* w, size_t count, int rows, int kc);
void variant_block(int variant, int* rows, int* kc);
uint16_t f32_to_bf16_rne(float v);
uint16_t f32_to_f16_rne(float v);

// Where the head writes the interior rows of the windows: n_frames > 0: the caller's waveform, y[clip][channel][n_frames * r] (the
// windows side by side: crop and stitch are in the address); 0: the window waveforms y[channel][plane], rows as in the workspace.
struct HeadOut { float* y = nullptr; long long plane = 0; int n_frames = 0; };

// Fused residual unit (bf16 path, C = 64 or 128): y = x + W1 snake2(W7 (*) snake1(x) + b7) + b1, x != y.
struct FusedArgs {
    const void* x; void* y;  // residual stream in its HBM storage type (half); y may be nullptr where ya takes all of the output
    uint16_t* ya = nullptr;  // optional: bf16(snake(y; a3, ib3)) for an unfused consumer
    const float* a3 = nullptr; const float* ib3 = nullptr;
    const uint16_t* w7;      // packed as pack_bf16 does for an MT = C, KC = 64 tile
    const uint16_t* w1;      // packed by pack_w1_fused
    const float* b7; const float* b1;
    const float* a1; const float* ib1; const float* a2; const float* ib2;
    const Slot* slots; int n_slots, call_slots, max_len, max_int, margin;
    int r, c, ntaps, dil;
    // optional: the decoder's head in the same kernel (64 channels, the unit feeds nothing else; y is then not written).
    // hw: half-precision MFMA fragments (pack_head_mfma), hb bias, ha / hib the head's Snake, hk its kernel size (odd, <= 7)
    const uint16_t* hw = nullptr; const float* hb = nullptr; const float* ha = nullptr; const float* hib = nullptr;
    HeadOut out; int oc = 0, hk = 0;
};
hipError_t launch_res_unit_fused(const FusedArgs& a, hipStream_t stream);
void pack_w1_fused(const float* w, int C, uint16_t* dst);

// fused residual unit for 256 channels (kernels_bf16_wide.hip): reads the pre-activated bf16 operand, updates the
// half residual stream in place
struct WideArgs {
    const uint16_t* xa; void* y;
    bool y_dead = false;     // y is only read: its sum goes to the consumer's operand alone (ya)
    uint16_t* ya = nullptr;  // optional: bf16(snake(y; a3, ib3)) for the consumer; must not be the buffer of xa
    const float* a3 = nullptr; const float* ib3 = nullptr;
    const uint16_t* w7;      // packed as pack_bf16 does for variant 3 (MT = 256, KC = 32)
    const uint16_t* w1;      // packed by pack_w1_wide
    const float* b7; const float* b1; const float* a2; const float* ib2;
    const Slot* slots; int n_slots, call_slots, max_len, max_int, margin;
    int r, c, ntaps, dil;
    bool staged_only = false;          // the LDS-staged kernel also in launches of few tiles (small_tile_wgs < 0 in the config)
};
hipError_t launch_res_unit_wide(const WideArgs& a, hipStream_t stream);
void pack_w1_wide(const float* w /*[256][256]*/, uint16_t* dst);

struct IoArgs {
    const Slot* slots; int n_slots; int max_len;
};
// latent [n_clips, c0, n_frames] (fp32 or bf16) -> activated operand snake(x; alpha, inv_beta) of the first layer, [frames, c0]:
// fp32 in x0 or, with `xa` (bf16 path), in operand format xa_fmt (lo plane at xa + xa_lo_off).  With `skip` (decode gate, one flag a
// clip): nothing for the windows of flagged clips, and `gated` becomes the table with these windows empty, for the launches after it
hipError_t launch_gather(const void* latent, float* x0, int c0, int n_frames, bool bf16,
                         const Slot* slots, int n_slots, int max_len, hipStream_t stream,
                         uint16_t* xa = nullptr, int xa_fmt = OP_BF16, long long xa_lo_off = 0,
                         const float* alpha = nullptr, const float* inv_beta = nullptr,
                         const int* skip = nullptr, Slot* gated = nullptr);
// encoder stem: Conv1d(k, ch -> C) + bias from the planar fp32 waveform [n_clips, ch, n_frames * S] into the residual
// stream y (half or fp32) of the rows each window needs (interior widened by `margin`); with ya also the activated
// operand snake(y; alpha, inv_beta), fp32 or (half path) in format ya_fmt.  w: fp32 [k][ch][C].
hipError_t launch_stem(const float* wave, void* y, bool y_half, void* ya, int ya_fmt, const float* w, const float* bias,
                       const float* alpha, const float* inv_beta, int ch, int C, int k, int S, int n_frames, int margin,
                       const Slot* slots, int n_slots, int max_len, int max_int, hipStream_t stream);
// the parts that K of the encoder's last convolution is cut into, each summed by workgroups of its own
constexpr int kConvParts = 8;
// encoder: moments of the windows' interior frames -> moments_out fp32 [n_clips, 2 C0, n_frames] and the sampled latent
// [n_clips, C0, n_frames] (bf16 for the half path, fp32 otherwise); eps fp32 [n_clips, C0, n_frames] or nullptr (z = mean)
// with `parts` (half path) the moments are the sums of the parts there, rounded to half; `m`, if given, takes them as the conv would have left them
hipError_t launch_sample(void* m, const float* parts, bool m_half, const float* eps, float* moments_out, void* latent_out, bool latent_bf16,
                         int C0, int n_frames, const Slot* slots, int n_slots, int max_int, hipStream_t stream);
// head: Snake -> Conv1d(k, cin -> oc) -> tanh; output planar fp32 [oc, total_rows]
// `fast` selects the hardware-sine Snake (alpha given in revolutions) used by the bf16 path.
// `x_half`: the input is the bf16 path's half-precision residual stream, else fp32.
hipError_t launch_head(const void* x, bool x_half, const HeadOut& out, const float* w /*[k][cin][oc]*/, const float* bias,
                       const float* alpha, const float* inv_beta, int cin, int oc, int k, int r,
                       bool fast, const Slot* slots, int n_slots, int max_int,
                       hipStream_t stream);
// MFMA head of the bf16 path (cin 32 or 64, oc <= 32); weights packed by pack_head_mfma
size_t head_mfma_frag_count(int cin, int k);          // 16-byte x 64-lane fragments
void pack_head_mfma(const float* w /*[oc][cin][k]*/, int cin, int oc, int k, uint16_t* dst);
hipError_t launch_head_mfma(const void* x, const HeadOut& out, const uint16_t* wfrag, const float* bias, const float* alpha,
                            const float* inv_beta, int cin, int oc, int k, int r,
                            const Slot* slots, int n_slots, int max_len, int max_int, hipStream_t stream);
// crop + stitch + 16-bit render: planar slot waveform -> d_pcm [n_clips, n_frames*S, oc] interleaved int16
hipError_t launch_stitch_pcm16(const float* y, int16_t* pcm, int oc, int S, int n_frames, long long total_rows,
                               const Slot* slots, int n_slots, int max_int, hipStream_t stream);
// window table written on the device (no host copy); per_clip windows and clip_frames extended frames per clip.
hipError_t launch_plan_slots(Slot* dst, int n_clips, int per_clip, int clip_frames, int n_frames, int frame_begin,
                             int frame_end, int window, int halo, hipStream_t stream);
// latent similarity filter: per clip mse = mean((a-b)^2) over n elements and the gate mse < threshold
hipError_t launch_latent_mse(const void* a, const void* b, int n_clips, long long n, bool bf16, float threshold,
                             float* mse, int* unchanged, hipStream_t stream);
// equal-power crossfade of n_planes planar segments of n samples
hipError_t launch_crossfade(const float* tail, long long tail_stride, const float* head, long long head_stride,
                            float* out, long long out_stride, int n_planes, int n, hipStream_t stream);
// debug tap: activation -> fp32 copy; src_type 0 fp32, 1 bf16, 2 half
hipError_t launch_to_f32(const void* x, float* dst, size_t n, int src_type, hipStream_t stream);

}  // namespace demon
