// C ABI of libdemon_vae: decoder construction (weight repacking, workspace), window plans and the
// launch sequence of the windowed decode (paper section 3.6: extend, decode, trim).
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <memory>
#include <mutex>
#include <new>

#include "internal.h"

using namespace demon;

namespace {

constexpr int kMaxSlots = 4096;
constexpr int kPlanCache = 16;
constexpr int kTimingRing = 32;        // decode calls whose events are kept for demon_vae_get_timing
// bf16 path: blocks at least this wide carry their MFMA operands with more mantissa bits than bf16.  There the
// branch gain (weight std x sqrt(fan-in)) is about one, so operand rounding passes into the output at full
// strength.  Default: IEEE half operands on the f16 MFMA for every convolution of such a block (same rate as bf16;
// the operands have the range of the half residual stream they are computed from).  The alternative (config field
// wide_operands) carries hi + lo bf16 pairs instead, for the inputs of the block's transposed conv and of its 1x1
// convs (two MFMAs per k-step there; the dilated convs then take plain bf16).
constexpr int kSplitWidth = 512;
// The head runs inside the last unit: at every size where that is of seven taps (60 s clip 5260 -> 5208 us back to back: 0.74 GB less of
// traffic), else, on the LDS-staged kernel, in calls of at most this many extended frames.
constexpr long long kHeadFusionFrames = 256;
// Defaults of the config fields wide_operands / flags / small_tile_wgs where they are left at 0, from the environment
// (read once when the library is loaded; for A/B timing of a whole program without touching its configs).
const int g_env_wide_fmt = [] {
    const char* e = getenv("DEMON_VAE_WIDE_OPERANDS");
    return (e && strcmp(e, "bf16x2") == 0) ? (int)OP_BF16X2 : (int)OP_F16;
}();
const bool g_env_no_fused = getenv("DEMON_VAE_NO_FUSED") != nullptr;
const bool g_env_one_stream = getenv("DEMON_VAE_ONE_STREAM") != nullptr;
const long long g_env_small_tile_wgs = [] {
    const char* e = getenv("DEMON_VAE_SMALL_TILE_WGS");
    return e ? atoll(e) : 1024ll;
}();

struct ConvLayer {
    int cin = 0, cout = 0, ntaps = 0, dil = 1, stride = 0, variant = -1;
    bool parts = false;                // K in parts, see kConvParts
    int down = 0;                      // s > 0: strided Conv1d(kernel 2s, stride s, padding s/2) of the encoder (ntaps = 2s)
    int in_fmt = OP_BF16;              // bf16 path: format of the activation operand (the weights are packed to match)
    bool generic = true;               // bf16 path: runs on launch_conv_bf16 (row order of its accumulator tiles)
    int margin = 0;                    // output rows beyond the interior that later layers read
    const void* w = nullptr;
    const float* bias = nullptr;
    const float* in_alpha = nullptr;   const float* in_inv_beta = nullptr;
    const float* out_alpha = nullptr;  const float* out_inv_beta = nullptr;
};

// fused: one kernel per unit that reads the half residual stream itself (64, 128 channels);
// wide: one kernel per unit that reads the pre-activated operand (256 channels); else two kernels
struct ResUnit { ConvLayer dilated, pointwise; bool fused = false, wide = false; const uint16_t* w1_fused = nullptr; };
// up: the block's resampling layer -- the decoder's transposed conv (before the units) or the encoder's strided conv (after them)
struct Block { ConvLayer up; std::vector<ResUnit> res; };
// The layer sequence in processing order: a resampling convolution (conv) or a residual unit (unit), and the layer that
// takes this step's output as an activated MFMA operand (bf16 path; nullptr: the next layer reads the residual stream).
struct Step { const ConvLayer* conv = nullptr; const ResUnit* unit = nullptr; const ConvLayer* consumer = nullptr; };

struct Plan {
    bool valid = false;
    int n_clips = 0, n_frames = 0, frame_begin = 0, frame_end = 0, window = 0, halo = 0;      // as the caller gave them
    bool verbatim = false;             // the caller's own windows, see computed_grid
    bool cut = false;                  // each clip in two windows, see cut_clips
    int grid_window = 0, grid_halo = 0;        // the grid that is computed
    int n_slots = 0, max_len = 0, max_int = 0;
    long long total_frames = 0;
    // where a call that runs as two groups of windows is cut: the window whose first extended frame is nearest to half of all
    int split = 0;
    long long split_frame0 = 0;
    Slot* d_slots = nullptr;
    unsigned long long last_use = 0;
    // A call on this grid was recorded into a HIP graph: the graph holds the address of this entry's table (and the
    // grid's launch shapes), so the entry is never evicted while the handle lives.
    bool pinned = false;
    // The kernel that writes this entry's table has only been recorded into a graph so far, not executed: the next call
    // on this grid launches it again (eagerly, or into the graph being recorded, which must not depend on another graph
    // having been replayed first).
    bool table_pending = false;
};

// The device memory a decode call works in besides its inputs and outputs: the handle's own (allocated at create) or,
// for demon_vae_decode_windowed_static, pieces of the static scratch array below.
struct Workspace {
    void* buf[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};
    float* head_out = nullptr;
    Slot* slot_gated = nullptr;
    size_t act_elems = 0;              // elements one activation buffer holds (= offset of the lo plane of a split operand)
};

// Scratch of demon_vae_decode_windowed_static, the entry point for callers that cannot allocate: window table and activation
// buffers of one call.  Every GPU the library runs on holds its own copy until the process ends.
// In host code the array's name is only a handle for hipGetSymbolAddress: kernels get the address looked up there.
constexpr size_t kStaticScratchBytes = DEMON_VAE_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
unsigned char* g_scratch_ptr[kMaxDevices] = {};      // per device: address of its copy of `scratch`
std::mutex g_scratch_mutex;

// Address of the current device's copy of the static scratch array (looked up once per device).
hipError_t static_scratch(int device, unsigned char** out)
{
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[device]) {
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[device] = static_cast<unsigned char*>(ptr);
    }
    *out = g_scratch_ptr[device];
    return hipSuccess;
}

}  // namespace

struct demon_vae {
    Stack st;
    demon_dtype dtype = DEMON_F32;
    int max_frames = 0, max_clips = 0;
    long long cap_frames = 0;
    double frame_flop = 0;             // operations of the convolutions for one latent frame
    long long per_frame = 0;           // largest rate x width of a layer: elements of one latent frame at its widest
    int rf_left = 0, rf_right = 0;
    int device = 0;
    bool has_staged_convs = false;     // bf16 path: some convolution outside the fused units takes an LDS-staged tile
    bool has_split_operands = false;   // bf16 path: some layer carries its operand as hi + lo planes
    bool fuse_f32 = false;             // fp32 path: residual units may run as one kernel
    long long small_tile_wgs = 1024;   // bf16 path: launches of more 128 x 128 tiles than this look for no smaller tile (conv_bf16.h)
    bool head_fusable = false;         // bf16 path: the last layer is a fused 64-channel unit that can run the head in its kernel

    void* d_params = nullptr;          // one allocation: all packed weights, biases, Snake parameters
    std::vector<Block> blocks;         // in processing order (encoder: from the audio rate down)
    std::vector<Step> steps;
    const ConvLayer* first_consumer = nullptr;     // bf16 path: the layer whose operand the gather (stem) writes
    bool encoder = false;              // the mirror path: waveform -> moments / latent
    const float* stem_w = nullptr;  const float* stem_bias = nullptr;      // encoder stem, fp32 [k][channels][C]
    int stem_cout = 0, stem_margin = 0;
    const float* head_w = nullptr;  const float* head_bias = nullptr;
    const uint16_t* head_wfrag = nullptr;   // bf16 path: half-precision MFMA fragments of the head weights (or nullptr)
    const float* head_alpha = nullptr;  const float* head_inv_beta = nullptr;
    int head_cin = 0;

    // fp32 path: residual stream, activated operand of the next layer, branch tensor / next residual stream, all fp32.
    // bf16 path: buf[0], buf[1] residual stream ping/pong (half), buf[2] bf16 activated branch tensor,
    // buf[3], buf[4] bf16 activated operand of the next layer (each bf16 buffer: hi plane + lo plane).
    // head_out: planar window waveforms [out_channels, cap_frames*S], for the 16-bit render only; slot_gated: per-call copy of a window table with
    // the skipped clips emptied (gated decode)
    Workspace ws;
    unsigned char* scratch = nullptr;              // this device's copy of the static scratch array
    Slot* d_slot_arena = nullptr;
    hipStream_t stream2 = nullptr;                 // second lane of the bf16 layer sequence (default priority, non-blocking)
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    Plan plans[kPlanCache];
    unsigned long long use_counter = 0;

    int timing = 0;                    // 0 off, 1 group boundaries, 2 every launch
    std::vector<hipEvent_t> events;    // kTimingRing sets of marks_per_call events
    int marks_per_call = 0;
    int n_marks = 0;                   // marks recorded by the current/last call
    int timed_calls = 0;               // calls recorded since the last set_timing / get_timing

    int tap_layer = -1;
    float* tap_dst = nullptr;
    size_t tap_cap = 0;

    bool callers_grid = false;         // demon_vae_debug_callers_grid
    int last_windows = 0, last_groups = 0;         // what the last call computed (demon_vae_debug_last_grid)
    long long last_frames = 0;
};

namespace {

// Host-side staging of the parameter arena: offsets are assigned while packing, pointers afterwards.
struct Arena {
    std::vector<unsigned char> bytes;
    size_t reserve(size_t n) {
        const size_t off = (bytes.size() + 255) & ~(size_t)255;
        bytes.resize(off + n);
        return off;
    }
};

struct SnakeOff { size_t alpha, inv_beta; };

SnakeOff pack_snake(Arena& ar, const float* alpha, const float* beta, int c, bool fast)
{
    SnakeOff o;
    o.alpha = ar.reserve(sizeof(float) * c);
    o.inv_beta = ar.reserve(sizeof(float) * c);
    float* a = reinterpret_cast<float*>(ar.bytes.data() + o.alpha);
    float* b = reinterpret_cast<float*>(ar.bytes.data() + o.inv_beta);
    for (int i = 0; i < c; ++i) {
        // the fast Snake feeds the hardware sine, which takes revolutions
        a[i] = fast ? (float)((double)alpha[i] / (2.0 * M_PI)) : alpha[i];
        b[i] = (float)(1.0 / ((double)beta[i] + 1e-9));
    }
    return o;
}

size_t pack_floats(Arena& ar, const float* src, size_t n)
{
    const size_t off = ar.reserve(sizeof(float) * n);
    memcpy(ar.bytes.data() + off, src, sizeof(float) * n);
    return off;
}

size_t pack_conv(Arena& ar, const float* w, ConvLayer& L, bool bf16)
{
    if (bf16) {
        const size_t n = packed_bf16_count(L.cin, L.cout, L.ntaps, L.stride, L.variant);
        const size_t off = ar.reserve(n * 2);
        pack_bf16(w, L.cin, L.cout, L.ntaps, L.stride, L.variant, L.in_fmt == OP_F16, L.generic, reinterpret_cast<uint16_t*>(ar.bytes.data() + off), L.down);
        int rows = 0, kc = 0;
        variant_block(L.variant, &rows, &kc);
        to_fragment_order(reinterpret_cast<uint16_t*>(ar.bytes.data() + off), n, rows, kc);
        return off;
    }
    const size_t n = packed_f32_count(L.cin, L.cout, L.ntaps, L.stride);
    const size_t off = ar.reserve(n * 4);
    pack_f32(w, L.cin, L.cout, L.ntaps, L.stride, reinterpret_cast<float*>(ar.bytes.data() + off));
    return off;
}

demon_status hip_fail(hipError_t e, const char* what)
{
    return fail(DEMON_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

// The window grid of one clip, walked on the host: windows, extended frames, longest window and interior.
struct GridCount { long long per_clip = 0, clip_frames = 0; int max_len = 0, max_int = 0; };

GridCount count_grid(int n_frames, int fb, int fe, int window, int halo)
{
    GridCount g;
    for (long long b = fb; b < fe; b += window) {
        const long long e = std::min<long long>(b + window, fe);
        const int len = (int)(std::min<long long>(n_frames, e + halo) - std::max<long long>(0, b - halo));
        g.clip_frames += len;
        g.max_len = std::max(g.max_len, len);
        g.max_int = std::max(g.max_int, (int)(e - b));
        ++g.per_clip;
    }
    return g;
}

#define HIP_TRY(expr, what) do { hipError_t e_ = (expr); if (e_ != hipSuccess) return hip_fail(e_, what); } while (0)

// bf16 path: a window's activation plane is addressed with 32-bit byte offsets through a buffer descriptor
demon_status check_plane(const demon_vae* v, int max_len)
{
    if (v->dtype != DEMON_BF16) return DEMON_OK;
    const long long bytes = (long long)max_len * v->per_frame * 2;
    if (bytes > 0xf0000000ll)
        return fail(DEMON_ERR_UNSUPPORTED, "a window of %d frames has an activation plane of %lld bytes; the kernels address one window "
                    "with 32-bit offsets (limit %lld bytes): decode it in several windows", max_len, bytes, 0xf0000000ll);
    return DEMON_OK;
}

// The window grid that a call computes.  Where every window carries the whole receptive field (or is the clip), a row does not depend
// on the grid: the results are the full decode's bits.  Windows side by side would compute the rows that both read twice -- one row in
// 21 of the decode and one in 6 of the encode with 64 frames, more than half with 16 -- and fill a last tile each, so a call computes each
// clip's span as one window, or as two where cut_clips says so.  In us, the caller's windows of 64 frames / one
// per clip / two (x1920 stack): decode of 250 frames 1085 / 1039 / 1060, 750 frames 2804 / 2713 / 2600, 1500 frames 5474 / 5298 / 5213, four
// clips of 1500 21614 / 20732 / 20778; encode of 250 frames 1298 / 1071 / 1107, 1500 frames 6185 / 5308 / 5213; fp32 decode of the x32 stack,
// 1500 frames 293 / 247.  A window's plane stays below 1 GB, far from the kernels' 32-bit offsets.
// The caller's own grid stays where a window carries less (its rows then depend on it), for the debug tap, whose rows are the caller's windows, and
// where a test asks for it.
struct Grid { int window, halo; };
constexpr long long kRegionBytes = 1ll << 30;

bool callers_own(const demon_vae* v) { return v->callers_grid || (v->tap_layer >= 0 && v->tap_dst); }

// Whether every clip is cut in two, for calls that may run as the two groups below and would otherwise have unequal ones: an odd number of
// clips, with a second stream and no gate (gated, one window a clip / two: one clip of 1500 frames 5191 / 5268, 3 x 150 1730 / 1809).  Per-launch
// timing, which runs one group, times the launches of the grid that calls compute.  A join computes twice the receptive field again (12 frames
// on the x1920 stack) in every clip, and two groups are twice the launches.  In us, one window a clip / two:
//  * one clip: 330 frames 1348 / 1330, 360 frames 1428 / 1429, 400 frames 1510 / 1509, 440 frames 1778 / 1624, 520 frames 1975 / 1880, encode of 400
//    frames 1520 / 1605, 440 frames 1790 / 1703; with LDS-staged convolutions 100 frames 994 / 1000, 200 frames 1395 / 1432, 250 frames 1683 / 1582.
//  * one clip of a smaller stack: what two groups cover is a share of each launch, so it takes as much work to be worth it, and a call that is waited
//    for pays for fork and join as well.  Back to back / waited for, one window, two: 512 to 64 channels at 768 samples a frame (0.63 GFLOP a frame)
//    480 frames 434 / 453, 455 / 513; 600 frames 503 / 520, 520 / 601; 700 frames 631 / 647, 584 / 680; its encode 642 / 659, 610 / 653; with LDS-staged
//    convolutions (0.43) 700 frames 694 / 714, 665 / 761; 900 frames 801 / 824, 771 / 877; 1000 frames 866 / 887, 836 / 899; 1200 frames 1061 / 1073, 967 / 1036, its
//    encode 1075 / 1086, 1005 / 1016.  512 to 96 channels at 32 samples (0.12) 700 frames 215, 258, 1500 frames 319, 331; 128 to 64 at 8 samples, bound by the
//    launches, 700 frames 53, 106.
//  * more clips: decode of 3 x 150 frames 1688 / 1693, 3 x 250 2610 / 2674, 3 x 300 3131 / 3093, 3 x 420 4459 / 4349, 3 x 1500 15595 / 15364, 5 x 150 2590 / 2699,
//    5 x 250 4422 / 4346, 5 x 300 5225 / 5202, 7 x 64 1675 / 1740, 7 x 200 4852 / 4835; encode of 3 x 150 1741 / 1753, 3 x 250 2803 / 2792, 3 x 350 3717 / 3741, 3 x 420
//    4611 / 4499, 3 x 1500 15602 / 15514, 5 x 90 1724 / 1821, 5 x 300 5389 / 5425, 5 x 420 7428 / 7362, 7 x 64 1670 / 1916, 7 x 200 4912 / 5073.  With LDS-staged
//    convolutions (960 to 64 channels) decode of 3 x 230 4369 / 4360, 3 x 300 5732 / 5704, 3 x 400 7555 / 7570, encode of 3 x 230 4755 / 4817, 3 x 400 8013 / 8480.
constexpr double kCutFlop = 430e9;

bool cut_clips(const demon_vae* v, int n_clips, long long span, bool gated)
{
    if (n_clips % 2 == 0 || !v->stream2 || gated || v->frame_flop * span * n_clips < kCutFlop) return false;
    if (n_clips == 1) return span >= (v->has_staged_convs ? 230 : 420);
    return v->encoder ? !v->has_staged_convs && span >= 420 : span >= 300;
}

Grid computed_grid(const demon_vae* v, int n_clips, int n_frames, int fb, int fe, int window, int halo, long long frames_held, bool cut)
{
    const int rf = std::max(v->rf_left, v->rf_right);
    const bool whole_clip = fb == 0 && fe == n_frames && window >= n_frames;
    if (halo < rf && !whole_clip) return {window, halo};
    const long long span = fe - fb;
    const long long most = kRegionBytes / (v->per_frame * (v->dtype == DEMON_BF16 ? 2 : 4)) - 2ll * rf;
    long long k = cut ? 2 : 1;
    if (most > 0 && (span + most - 1) / most > k) k = (span + most - 1) / most + (span + most - 1) / most % 2;
    const int w = (int)((span + k - 1) / k);
    // the halo of the caller's single window is not needed where it is the clip
    const Grid g = {w, w == span && whole_clip ? 0 : rf};
    // more extended frames than the caller's grid (a window cut in two): only where they are held
    if (most < 1 || k * n_clips > kMaxSlots || count_grid(n_frames, fb, fe, g.window, g.halo).clip_frames * n_clips > frames_held) return {window, halo};
    return g;
}

// Whether the layer sequence of a call runs as two groups of windows on two streams: the ramp and tail of one group's launches
// (a last round of workgroups that fills a fraction of the CUs, prologues, epilogues) overlap with the other's.  Both take the
// tiles that the whole call would take.  One / two groups in us on the x1920 stack, windows of 64 frames: 250 frames (286
// extended) 1180 / 1191, 310 frames 1483 / 1462, 600 frames 2603 / 2438, 1500 frames 6102 / 5994, four clips of 1500 frames
// 23.83 / 23.72 ms.  Calls that fit one or two rounds of the chip lose by the split, hence the bound: five windows of 50 frames
// (298 extended) 1182 / 1305, three of 75 frames 1117 / 1228, two of 32 frames 429 / 489.  LDS-staged convolutions have longer
// tails (a stack of 960 to 64 channels): two windows of 40 frames (104 extended) 1046 / 1080, two of 60 (144) 1245 / 1222, 220 frames
// 1935 / 1782.
// One group for a gated call, which may turn out to be launches only, and where a mode wants one ordered launch sequence
// (per-launch timing, debug tap).
long long two_group_frames(const demon_vae* v) { return v->has_staged_convs ? 150 : 320; }

bool two_groups(const demon_vae* v, const Plan* p, bool gated)
{
    return p->split > 0 && p->total_frames >= two_group_frames(v) && !gated && v->stream2 && v->timing < 2 &&
           !(v->tap_layer >= 0 && v->tap_dst);
}

// Looks the window grid up in the plan cache; on a miss the table of the least recently used entry that no graph holds is
// rewritten by a small kernel on the decode stream, so the call stays asynchronous (kernels of earlier calls that still
// read the replaced table precede that kernel on the stream) and can itself be recorded into a graph.
demon_status get_plan(demon_vae* v, int n_clips, int n_frames, int fb, int fe, int window, int halo, bool gated,
                      hipStream_t stream, Plan** out)
{
    ++v->use_counter;
    const bool verbatim = callers_own(v);
    const bool cut = !verbatim && cut_clips(v, n_clips, fe - fb, gated);
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    HIP_TRY(hipStreamIsCapturing(stream, &cap), "hipStreamIsCapturing");
    const bool capturing = cap != hipStreamCaptureStatusNone;
    Plan* victim = nullptr;
    Plan* hit = nullptr;
    // the other grid of the same rows: taken where graphs hold every entry, and by a recorded call where a graph holds it already, so that
    // the graphs of one grid hold one entry
    Plan* alike = nullptr;
    for (Plan& p : v->plans) {
        if (p.valid && p.n_clips == n_clips && p.n_frames == n_frames && p.frame_begin == fb && p.frame_end == fe &&
            p.window == window && p.halo == halo && p.verbatim == verbatim) {
            if (p.cut == cut) { hit = &p; break; }
            alike = &p;
        }
        if (p.pinned) continue;
        if (!victim || (victim->valid && (!p.valid || p.last_use < victim->last_use))) victim = &p;
    }
    if (!hit && alike && (!victim || (capturing && alike->pinned))) hit = alike;
    if (hit) {
        hit->last_use = v->use_counter;
        if (capturing) hit->pinned = true;
        if (hit->table_pending) {
            HIP_TRY(launch_plan_slots(hit->d_slots, hit->n_clips, hit->n_slots / hit->n_clips, (int)(hit->total_frames / hit->n_clips), hit->n_frames,
                                      hit->frame_begin, hit->frame_end, hit->grid_window, hit->grid_halo, stream), "window table");
            if (!capturing) hit->table_pending = false;
        }
        *out = hit;
        return DEMON_OK;
    }
    if (!victim)
        return fail(DEMON_ERR_WORKSPACE, "all %d cached window grids are held by recorded graphs; a further grid needs another handle", kPlanCache);
    // the limits are those of the caller's grid
    GridCount gc = count_grid(n_frames, fb, fe, window, halo);
    long long n_slots = gc.per_clip * n_clips;
    if (n_slots > kMaxSlots)
        return fail(DEMON_ERR_WORKSPACE, "%lld windows exceed the limit of %d", n_slots, kMaxSlots);
    long long total = gc.clip_frames * n_clips;
    if (total > v->cap_frames)
        return fail(DEMON_ERR_WORKSPACE, "extended windows need %lld frames, the workspace holds %lld", total, v->cap_frames);
    const demon_status prc = check_plane(v, gc.max_len);
    if (prc != DEMON_OK) return prc;
    const Grid grid = verbatim ? Grid{window, halo} : computed_grid(v, n_clips, n_frames, fb, fe, window, halo, v->cap_frames, cut);
    gc = count_grid(n_frames, fb, fe, grid.window, grid.halo);
    n_slots = gc.per_clip * n_clips;
    total = gc.clip_frames * n_clips;
    const int idx = (int)(victim - v->plans);
    Slot* d = v->d_slot_arena + (size_t)idx * kMaxSlots;
    victim->valid = false;
    HIP_TRY(launch_plan_slots(d, n_clips, (int)gc.per_clip, (int)gc.clip_frames, n_frames, fb, fe, grid.window, grid.halo, stream), "window table");
    victim->valid = true;
    victim->pinned = capturing;
    victim->table_pending = capturing;
    victim->n_clips = n_clips; victim->n_frames = n_frames; victim->frame_begin = fb; victim->frame_end = fe;
    victim->window = window; victim->halo = halo; victim->verbatim = verbatim; victim->cut = cut;
    victim->grid_window = grid.window; victim->grid_halo = grid.halo;
    victim->n_slots = (int)n_slots; victim->max_len = gc.max_len; victim->max_int = gc.max_int;
    victim->total_frames = total; victim->d_slots = d; victim->last_use = v->use_counter;
    victim->split = 0; victim->split_frame0 = 0;
    long long best = -1, row = 0, i = 0;
    for (int c = 0; c < n_clips; ++c)
        for (long long b = fb; b < fe; b += grid.window, ++i) {
            const long long e = std::min<long long>(b + grid.window, fe);
            const long long d = std::abs(total - 2 * row);
            if (i >= 1 && (best < 0 || d < best)) { best = d; victim->split = (int)i; victim->split_frame0 = row; }
            row += std::min<long long>(n_frames, e + grid.halo) - std::max<long long>(0, b - grid.halo);
        }
    *out = victim;
    return DEMON_OK;
}

// What one call reads and writes besides the handle's own memory.
struct Io {
    // decode: latent in, waveform (fp32 planar or interleaved int16) out, optional per-clip skip flags
    const void* d_latent = nullptr; const int* d_skip = nullptr; float* d_out = nullptr; int16_t* d_pcm = nullptr;
    // encode: waveform in, moments and / or sampled latent out, optional noise of the sampling step
    const float* d_wave = nullptr; const float* d_eps = nullptr; float* d_moments = nullptr; void* d_zout = nullptr;
    int n_frames = 0;
};

// The launch sequence of one call over the windows of `plan`, in the memory of `ws`: the decoder's
// gather | layers | head (| 16-bit render), or the encoder's stem | layers | sampling step.
demon_status run_pass(demon_vae* v, const Workspace& ws, const Plan* plan, const Io& io, hipStream_t stream)
{
    const bool bf = v->dtype == DEMON_BF16;
    const bool enc = v->encoder;
    // the head inside the last unit's kernel, unless the debug tap wants that unit's output in memory
    // (bit-identical either way)
    const bool head_in_unit = v->head_fusable && !(v->tap_layer >= 0 && v->tap_dst) && (v->st.res_kernel == 7 || plan->total_frames <= kHeadFusionFrames);
    const int n_frames = io.n_frames;
    const Slot* slots = plan->d_slots;
    const int ns = plan->n_slots, ml = plan->max_len;
    if (io.d_skip) {
        // gated decode: the gather writes a copy of the table in which the skipped clips' windows are empty, for all kernels after it
        slots = ws.slot_gated;
    }

    // the launches address a group of windows (gs, gn) on a stream gst: all windows on the caller's stream, or two
    // groups of consecutive windows on two streams (see the bf16 path below)
    const int n_groups = two_groups(v, plan, io.d_skip != nullptr) ? 2 : 1;
    v->last_windows = ns; v->last_frames = plan->total_frames; v->last_groups = bf ? n_groups : 1;
    const Slot* gs = slots;
    int gn = ns;
    long long frame0 = 0;
    hipStream_t gst = stream;
    bool marks_on = true;
    auto select_group = [&](int which, hipStream_t on) {
        gs = slots + (which ? plan->split : 0);
        gn = n_groups == 1 ? ns : which ? ns - plan->split : plan->split;
        frame0 = which ? plan->split_frame0 : 0;
        gst = on;
    };
    // The groups can be at different layers at the same time, and the bytes a window occupies depend on the layer's rate x
    // width: in every activation buffer of the bf16 path the second group owns what lies from frame0 x (largest rate x width)
    // on.  `at` is the base from which the rows of the window table, which count from the first window, fall into it.
    auto at = [&](const void* buf, int rate, int width) -> uint16_t* {
        return buf ? (uint16_t*)const_cast<void*>(buf) + (size_t)frame0 * (size_t)(v->per_frame - (long long)rate * width) : nullptr;
    };

    v->n_marks = 0;
    const int ring_base = (v->timed_calls % kTimingRing) * v->marks_per_call;
    auto mark = [&](int level) -> hipError_t {
        if (!marks_on || v->timing < level || v->n_marks >= v->marks_per_call) return hipSuccess;
        return hipEventRecord(v->events[ring_base + v->n_marks++], stream);
    };
    // level 1 marks: start, after gather (stem), after the last convolution, after head (sampling step), after the 16-bit render.
    // level 2 adds a mark after every convolution launch.
    HIP_TRY(mark(1), "event");

    const int S = v->st.total_stride();
    // the head writes the caller's waveform; the 16-bit render takes the windows' waveforms, planar [channel][all rows]
    HeadOut head_out;
    if (io.d_pcm) { head_out.y = ws.head_out; head_out.plane = plan->total_frames * S; }
    else { head_out.y = io.d_out; head_out.plane = (long long)n_frames * S; head_out.n_frames = n_frames; }
    void* cur = ws.buf[0];
    void* other = ws.buf[1];
    int r = enc ? S : 1, layer_id = 0;
    const size_t n_steps = v->steps.size();
    const long long lo_off = (long long)ws.act_elems;        // lo plane of a split bf16 tensor
    auto tap = [&](const void* x, int c) -> hipError_t {
        const int id = layer_id++;
        if (id != v->tap_layer || !v->tap_dst) return hipSuccess;
        const size_t want = (size_t)plan->total_frames * r * c;
        return launch_to_f32(x, v->tap_dst, std::min(want, v->tap_cap), bf ? 2 : 0, stream);
    };
    // A unit before a resampling convolution: that reads the activated operand only and starts the residual stream anew, so the unit's
    // own sum is not written (unless the debug tap reads it).  60 s clip, us, written / not: the 1x1 conv
    // of 512 channels 89 / 77, units of 256 channels 325 / 308, of 128 channels 442 / 400; the clip 5703 / 5633.
    auto residual_dead = [&](size_t si) {
        return v->steps[si].unit && si + 1 < n_steps && v->steps[si + 1].conv && !(v->tap_layer >= 0 && v->tap_dst);
    };
    // samples per frame after a layer
    auto resampled = [](int rate, const ConvLayer& L) { return L.down > 0 ? rate / L.down : L.stride > 0 ? rate * L.stride : rate; };
    auto conv_args = [&](const ConvLayer& L, const void* x, void* y, const void* res) {
        ConvArgs a;
        const int ro = resampled(r, L);
        a.x = at(x, r, L.cin); a.y = at(y, ro, L.cout); a.res = at(res, ro, L.cout); a.w = L.w; a.bias = L.bias;
        a.out_alpha = L.out_alpha; a.out_inv_beta = L.out_inv_beta;
        a.slots = gs; a.n_slots = gn; a.call_slots = ns; a.max_len = ml; a.max_int = plan->max_int; a.margin = L.margin; a.r_in = r;
        a.cin = L.cin; a.cout = L.cout; a.ntaps = L.ntaps; a.dil = L.dil; a.stride = L.stride; a.down = L.down;
        a.in_fmt = L.in_fmt;
        a.in_lo_off = a.out_lo_off = lo_off;
        a.small_tile_wgs = v->small_tile_wgs;
        return a;
    };

    if (!bf) {
        // ---- fp32 path.  Three buffers in rotation: `cur` holds the residual stream h, `act` the activated operand of the
        // next layer (written by the producer of h with that layer's Snake), `other` is free.
        void* act = ws.buf[2];
        if (enc) {
            const ConvLayer& C = *v->first_consumer;
            HIP_TRY(launch_stem(io.d_wave, cur, false, act, 0, v->stem_w, v->stem_bias, C.in_alpha, C.in_inv_beta, v->st.out_channels,
                                v->stem_cout, v->st.head_kernel, S, n_frames, v->stem_margin, slots, ns, ml, plan->max_int, stream), "stem");
        } else {
            const ConvLayer& C = *v->first_consumer;
            HIP_TRY(launch_gather(io.d_latent, (float*)act, v->st.c0, n_frames, false, plan->d_slots, ns, ml, stream, nullptr, 0, 0,
                                  C.in_alpha, C.in_inv_beta, io.d_skip, ws.slot_gated), "gather");
        }
        HIP_TRY(mark(1), "event");
        for (size_t si = 0; si < n_steps; ++si) {
            const Step& T = v->steps[si];
            const ConvLayer* C = T.consumer;
            const bool last = si + 1 == n_steps;
            const bool y_dead = residual_dead(si);
            auto emit_to = [&](ConvArgs& a, void* ya) { if (C) { a.ya = ya; a.out_alpha = C->in_alpha; a.out_inv_beta = C->in_inv_beta; } };
            if (T.conv) {
                ConvArgs a = conv_args(*T.conv, act, other, nullptr);
                emit_to(a, cur);                                       // the old h is not needed any more
                HIP_TRY(launch_conv_f32(a, stream), "resampling convolution");
                HIP_TRY(mark(last ? 1 : 2), "event");
                void* const old = cur;
                cur = other; other = act; act = old;
                r = resampled(r, *T.conv);
                HIP_TRY(tap(cur, T.conv->cout), "debug tap");
            } else {
                const ResUnit& U = *T.unit;
                ConvArgs d = conv_args(U.dilated, act, nullptr, nullptr);
                ConvArgs fused = conv_args(U.pointwise, other, y_dead ? nullptr : cur, cur);
                emit_to(fused, other);                                 // (neighbouring tiles read `act`)
                if (v->fuse_f32 && res_unit_f32_fuses(d, fused)) {
                    HIP_TRY(launch_res_unit_f32(d, fused, stream), "residual unit");
                    std::swap(act, other);
                    HIP_TRY(mark(2), "event");
                    HIP_TRY(mark(last ? 1 : 2), "event");
                    HIP_TRY(tap(cur, U.pointwise.cout), "debug tap");
                    continue;
                }
                d.ya = other;                                          // Snake between the convolutions: the layer's own out_alpha
                HIP_TRY(launch_conv_f32(d, stream), "dilated convolution");
                HIP_TRY(mark(2), "event");
                ConvArgs q = conv_args(U.pointwise, other, y_dead ? nullptr : cur, cur);       // in place on the residual stream
                emit_to(q, act);
                HIP_TRY(launch_conv_f32(q, stream), "pointwise convolution");
                HIP_TRY(mark(last ? 1 : 2), "event");
                HIP_TRY(tap(cur, U.pointwise.cout), "debug tap");
            }
        }
    } else {
        // ---- bf16 path.  h (half) ping-pongs between buf[0] and buf[1]; the activated bf16 operand `a` of the
        // next layer that wants one ping-pongs between buf[3] and buf[4]; buf[2] holds the activated branch tensor
        // between the dilated and the 1x1 conv of a two-kernel unit.  Each producer writes `a` with its consumer's Snake.
        uint16_t* acur = (uint16_t*)ws.buf[3];
        uint16_t* aoth = (uint16_t*)ws.buf[4];
        uint16_t* mid = (uint16_t*)ws.buf[2];
        for (int gi = 0; gi < n_groups; ++gi) {
            select_group(gi, stream);
            if (enc) {
                const ConvLayer* C = v->first_consumer;
                HIP_TRY(launch_stem(io.d_wave, at(ws.buf[0], S, v->stem_cout), true, C ? at(ws.buf[3], S, v->stem_cout) : nullptr,
                                    C ? C->in_fmt : 0, v->stem_w, v->stem_bias, C ? C->in_alpha : nullptr, C ? C->in_inv_beta : nullptr,
                                    v->st.out_channels, v->stem_cout, v->st.head_kernel, S, n_frames, v->stem_margin, gs, gn, ml,
                                    plan->max_int, stream), "stem");
            } else {
                const ConvLayer& U0 = *v->first_consumer;
                HIP_TRY(launch_gather(io.d_latent, nullptr, v->st.c0, n_frames, true, io.d_skip ? plan->d_slots : gs, gn, ml, stream,
                                      at(ws.buf[3], 1, v->st.c0), U0.in_fmt, lo_off, U0.in_alpha, U0.in_inv_beta, io.d_skip, ws.slot_gated), "gather");
            }
        }
        HIP_TRY(mark(1), "event");
        auto layers = [&]() -> demon_status {
            cur = ws.buf[0]; other = ws.buf[1];
            acur = (uint16_t*)ws.buf[3]; aoth = (uint16_t*)ws.buf[4];
            r = enc ? S : 1; layer_id = 0;
            for (size_t si = 0; si < n_steps; ++si) {
                const Step& T = v->steps[si];
                const bool last = si + 1 == n_steps;
                // the layer that consumes this step's output through an activated operand; nullptr when that layer reads the
                // residual stream itself (narrow fused unit, head, sampling step)
                const ConvLayer* C = T.consumer;
                if (T.conv) {
                    ConvArgs a = conv_args(*T.conv, acur, other, nullptr);
                    if (T.conv->parts) { a.y = nullptr; a.part = reinterpret_cast<float*>(at(other, 1, 2 * kConvParts * T.conv->cout)); }
                    if (C) { a.ya = at(aoth, resampled(r, *T.conv), T.conv->cout); a.out_alpha = C->in_alpha; a.out_inv_beta = C->in_inv_beta; a.out_fmt = C->in_fmt; }
                    HIP_TRY(launch_conv_bf16(a, T.conv->variant, gst), "resampling convolution");
                    if (C) std::swap(acur, aoth);
                    HIP_TRY(mark(last ? 1 : 2), "event");
                    std::swap(cur, other);
                    r = resampled(r, *T.conv);
                    if (!T.conv->parts) HIP_TRY(tap(cur, T.conv->cout), "debug tap");     // else after the sampling step
                    continue;
                }
                const ResUnit& U = *T.unit;
                if (U.fused) {
                    FusedArgs f;
                    f.x = at(cur, r, U.dilated.cin); f.y = residual_dead(si) ? nullptr : at(other, r, U.dilated.cin);
                    if (C) { f.ya = at(acur, r, U.dilated.cin); f.a3 = C->in_alpha; f.ib3 = C->in_inv_beta; }
                    f.w7 = (const uint16_t*)U.dilated.w; f.w1 = U.w1_fused;
                    f.b7 = U.dilated.bias; f.b1 = U.pointwise.bias;
                    f.a1 = U.dilated.in_alpha; f.ib1 = U.dilated.in_inv_beta;
                    f.a2 = U.dilated.out_alpha; f.ib2 = U.dilated.out_inv_beta;
                    f.slots = gs; f.n_slots = gn; f.call_slots = ns; f.max_len = ml; f.max_int = plan->max_int; f.margin = U.pointwise.margin;
                    f.r = r; f.c = U.dilated.cin; f.ntaps = U.dilated.ntaps; f.dil = U.dilated.dil;
                    if (C && C->in_fmt != OP_BF16) return fail(DEMON_ERR_UNSUPPORTED, "a fused unit cannot feed a layer with wide operands");
                    if (last && head_in_unit) {
                        f.hw = v->head_wfrag; f.hb = v->head_bias; f.ha = v->head_alpha; f.hib = v->head_inv_beta;
                        f.out = head_out;
                        f.oc = v->st.out_channels; f.hk = v->st.head_kernel;
                    }
                    HIP_TRY(launch_res_unit_fused(f, gst), "fused residual unit");
                    std::swap(cur, other);
                    HIP_TRY(mark(2), "event");
                } else if (U.wide) {
                    WideArgs f;
                    f.xa = at(acur, r, U.dilated.cin); f.y = at(cur, r, U.dilated.cin); f.y_dead = residual_dead(si);
                    if (C) { f.ya = at(aoth, r, U.dilated.cin); f.a3 = C->in_alpha; f.ib3 = C->in_inv_beta; }
                    f.w7 = (const uint16_t*)U.dilated.w; f.w1 = U.w1_fused;
                    f.b7 = U.dilated.bias; f.b1 = U.pointwise.bias;
                    f.a2 = U.dilated.out_alpha; f.ib2 = U.dilated.out_inv_beta;
                    f.slots = gs; f.n_slots = gn; f.call_slots = ns; f.max_len = ml; f.max_int = plan->max_int; f.margin = U.pointwise.margin;
                    f.r = r; f.c = U.dilated.cin; f.ntaps = U.dilated.ntaps; f.dil = U.dilated.dil;
                    if (C && C->in_fmt != OP_BF16) return fail(DEMON_ERR_UNSUPPORTED, "a fused unit cannot feed a layer with wide operands");
                    f.staged_only = v->small_tile_wgs == 0;
                    HIP_TRY(launch_res_unit_wide(f, gst), "fused residual unit (256 channels)");
                    if (C) std::swap(acur, aoth);
                    HIP_TRY(mark(2), "event");
                } else {
                    ConvArgs d = conv_args(U.dilated, acur, nullptr, nullptr);
                    d.ya = at(mid, r, U.dilated.cout); d.out_fmt = U.pointwise.in_fmt;   // Snake between the convolutions: the layer's own out_alpha
                    HIP_TRY(launch_conv_bf16(d, U.dilated.variant, gst), "dilated convolution");
                    HIP_TRY(mark(2), "event");
                    ConvArgs q = conv_args(U.pointwise, mid, cur, cur);   // in place on the residual stream
                    q.y_dead = residual_dead(si);
                    if (C) { q.ya = at(acur, r, U.pointwise.cout); q.out_alpha = C->in_alpha; q.out_inv_beta = C->in_inv_beta; q.out_fmt = C->in_fmt; }
                    HIP_TRY(launch_conv_bf16(q, U.pointwise.variant, gst), "pointwise convolution");
                }
                HIP_TRY(mark(last ? 1 : 2), "event");
                HIP_TRY(tap(cur, U.pointwise.cout), "debug tap");
            }
            return DEMON_OK;
        };
        if (n_groups == 2) {
            marks_on = false;
            HIP_TRY(hipEventRecord(v->ev_fork, stream), "event");
            HIP_TRY(hipStreamWaitEvent(v->stream2, v->ev_fork, 0), "hipStreamWaitEvent");
        }
        demon_status lrc = DEMON_OK;
        for (int gi = 0; gi < n_groups && lrc == DEMON_OK; ++gi) {
            select_group(gi, gi == 1 ? v->stream2 : stream);
            lrc = layers();
        }
        if (n_groups == 2) {
            // also after a failed launch: the second stream joins the caller's again (an open capture stays well-formed)
            const hipError_t e1 = hipEventRecord(v->ev_join, v->stream2);
            const hipError_t e2 = e1 == hipSuccess ? hipStreamWaitEvent(stream, v->ev_join, 0) : e1;
            if (lrc != DEMON_OK) return lrc;
            HIP_TRY(e2, "joining the second stream");
            marks_on = true;
            HIP_TRY(mark(1), "event");                       // after the last convolution
        }
        if (lrc != DEMON_OK) return lrc;
    }
    if (enc) {
        // sampling step on the moments, trim and scatter into the caller's [clip, channel, frame] arrays
        const bool parts = v->steps.back().conv->parts, tapped = parts && v->tap_layer == layer_id && v->tap_dst;
        void* m = !parts ? cur : tapped ? ws.buf[3] : nullptr;
        for (int gi = 0; gi < n_groups; ++gi) {
            select_group(gi, stream);
            const float* sums = parts ? reinterpret_cast<const float*>(at(cur, 1, 4 * kConvParts * v->st.c0)) : nullptr;
            HIP_TRY(launch_sample(at(m, r, 2 * v->st.c0), sums, bf, io.d_eps, io.d_moments, io.d_zout, bf, v->st.c0, n_frames, gs, gn,
                                  plan->max_int, stream), "sampling step");
        }
        if (parts) HIP_TRY(tap(m, 2 * v->st.c0), "debug tap");
        HIP_TRY(mark(1), "event");
        if (v->timing > 0) ++v->timed_calls;
        return DEMON_OK;
    }
    // head, group by group on the caller's stream
    for (int gi = 0; gi < n_groups && !head_in_unit; ++gi) {
        select_group(gi, stream);
        const void* x = at(cur, r, v->head_cin);
        if (v->head_wfrag)
            HIP_TRY(launch_head_mfma(x, head_out, v->head_wfrag, v->head_bias, v->head_alpha, v->head_inv_beta, v->head_cin,
                                     v->st.out_channels, v->st.head_kernel, r, gs, gn, ml, plan->max_int, stream), "head");
        else
            HIP_TRY(launch_head(x, bf, head_out, v->head_w, v->head_bias, v->head_alpha, v->head_inv_beta, v->head_cin,
                                v->st.out_channels, v->st.head_kernel, r, bf, gs, gn, plan->max_int, stream), "head");
    }
    HIP_TRY(mark(1), "event");
    if (io.d_pcm)
        HIP_TRY(launch_stitch_pcm16(ws.head_out, io.d_pcm, v->st.out_channels, r, n_frames, head_out.plane, slots, ns, plan->max_int, stream), "stitch");
    HIP_TRY(mark(1), "event");
    if (v->timing > 0) ++v->timed_calls;
    return DEMON_OK;
}

// Builds a decoder (encoder = false) or its mirror, the encoder (true), on the current device.
demon_status create_impl(const demon_vae_config* cfg, const float* host_weights, size_t n_floats, bool encoder, demon_vae** out)
{
    clear_error();
    if (!out) return fail(DEMON_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (!host_weights) return fail(DEMON_ERR_INVALID_ARG, "host_weights is NULL");
    Stack st;
    demon_status rc = stack_from_config(cfg, &st);
    if (rc != DEMON_OK) return rc;
    if (cfg->dtype != DEMON_F32 && cfg->dtype != DEMON_BF16) return fail(DEMON_ERR_INVALID_ARG, "unknown dtype %d", (int)cfg->dtype);
    if (cfg->max_frames < 1 || cfg->max_clips < 1) return fail(DEMON_ERR_INVALID_ARG, "max_frames and max_clips must be >= 1");
    const size_t need = encoder ? stack_encoder_weight_count(st) : stack_weight_count(st);
    if (n_floats != need) return fail(DEMON_ERR_INVALID_ARG, "got %zu weights, the layer stack needs %zu", n_floats, need);
    const bool bf = cfg->dtype == DEMON_BF16;
    if (cfg->wide_operands < 0 || cfg->wide_operands > 2) return fail(DEMON_ERR_INVALID_ARG, "wide_operands must be 0, 1 or 2");
    if (cfg->flags & ~(DEMON_VAE_FLAG_NO_FUSED | DEMON_VAE_FLAG_ONE_STREAM | DEMON_VAE_FLAG_NO_WIDE_TILE | DEMON_VAE_FLAG_NO_HEAD_FUSION)) return fail(DEMON_ERR_INVALID_ARG, "unknown flag bits 0x%x", (unsigned)cfg->flags);
    // 0 in a field = the default, which the environment may have changed (see the header)
    const int g_wide_fmt = cfg->wide_operands == 1 ? (int)OP_F16 : cfg->wide_operands == 2 ? (int)OP_BF16X2 : g_env_wide_fmt;
    const bool g_allow_fused = !((cfg->flags & DEMON_VAE_FLAG_NO_FUSED) || g_env_no_fused);
    const bool g_dual_stream = !((cfg->flags & DEMON_VAE_FLAG_ONE_STREAM) || g_env_one_stream);
    if (bf) {
        if (st.c0 % 16) return fail(DEMON_ERR_UNSUPPORTED, "bf16 path: latent_channels %d is not a multiple of 16", st.c0);
        for (int c : st.widths)
            if (c % 32) return fail(DEMON_ERR_UNSUPPORTED, "bf16 path: width %d is not a multiple of 32", c);
        for (int d : st.dilations)
            if ((st.res_kernel - 1) * d > 64)
                return fail(DEMON_ERR_UNSUPPORTED, "bf16 path: kernel %d with dilation %d spans more than 64 samples", st.res_kernel, d);
        if (encoder && g_wide_fmt == OP_BF16X2)
            return fail(DEMON_ERR_UNSUPPORTED, "the encoder's strided convolutions take one operand plane: wide_operands = 2 is for decoders");
    }
    if (st.head_kernel > 15) return fail(DEMON_ERR_UNSUPPORTED, "head_kernel %d exceeds 15", st.head_kernel);
    if (encoder && st.widths.back() % 8) return fail(DEMON_ERR_UNSUPPORTED, "encoder: the stem's width %d is not a multiple of 8", st.widths.back());

    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) return fail(DEMON_ERR_HIP, "no HIP device available");

    std::unique_ptr<demon_vae> v(new (std::nothrow) demon_vae);
    if (!v) return fail(DEMON_ERR_HIP, "out of host memory");

    v->st = st; v->dtype = cfg->dtype; v->max_frames = cfg->max_frames; v->max_clips = cfg->max_clips;
    v->encoder = encoder;
    v->fuse_f32 = !bf && g_allow_fused;
    if (cfg->max_extended_frames < 0) return fail(DEMON_ERR_INVALID_ARG, "max_extended_frames must be >= 0");
    v->cap_frames = cfg->max_extended_frames > 0 ? cfg->max_extended_frames : 3ll * cfg->max_frames * cfg->max_clips;
    if (encoder) stack_encoder_receptive_field(st, &v->rf_left, &v->rf_right, nullptr, nullptr);
    else stack_receptive_field(st, &v->rf_left, &v->rf_right);
    v->small_tile_wgs = cfg->small_tile_wgs > 0 ? cfg->small_tile_wgs : cfg->small_tile_wgs < 0 ? 0 : g_env_small_tile_wgs;
    if (hipGetDevice(&v->device) != hipSuccess) return fail(DEMON_ERR_HIP, "hipGetDevice failed");
    {
        // the static scratch array of demon_vae_decode_windowed_static: its address on this device
        const hipError_t se = static_scratch(v->device, &v->scratch);
        if (se != hipSuccess) return hip_fail(se, "hipGetSymbolAddress(static scratch)");
    }

    // ---- pack parameters (offsets first, device pointers after the upload)
    Arena ar;
    struct Pending { ConvLayer* L; size_t w, bias; SnakeOff in, outp; bool has_in, has_out; };
    std::vector<Pending> pend;
    struct FusedFix { ResUnit* U; size_t off; };
    std::vector<FusedFix> fused_fix;
    const int nb = (int)st.strides.size(), nres = (int)st.dilations.size();
    v->blocks.resize(nb);
    for (int b = 0; b < nb; ++b) v->blocks[b].res.resize(nres);

    const float* w = host_weights;
    // one residual unit of width c whose output goes, as an operand, to a layer of format `next_fmt`
    auto pack_unit = [&](ResUnit& U, int c, int j, int next_fmt) -> demon_status {
        ConvLayer& D = U.dilated;
        D.cin = c; D.cout = c; D.ntaps = st.res_kernel; D.dil = st.dilations[j];
        ConvLayer& P = U.pointwise;
        P.cin = c; P.cout = c; P.ntaps = 1; P.dil = 1;
        const bool wide_ops = bf && c >= kSplitWidth;
        P.in_fmt = wide_ops ? g_wide_fmt : (int)OP_BF16;
        if (P.in_fmt == OP_BF16X2) v->has_split_operands = true;
        D.in_fmt = (wide_ops && g_wide_fmt == OP_F16) ? (int)OP_F16 : (int)OP_BF16;
        if (bf) {
            D.variant = choose_variant_bf16(c, c);
            P.variant = choose_variant_bf16(c, c);
            if (D.variant < 0 || P.variant < 0) return fail(DEMON_ERR_UNSUPPORTED, "bf16 path: no kernel for %d channels", c);
        }
        // a fused unit writes plain bf16 operands: a unit stays on the two-kernel path when the layer after it wants
        // its input in a wider format
        const bool feeds_split = next_fmt != OP_BF16;
        U.fused = bf && (c == 64 || c == 128) && (st.res_kernel - 1) * st.dilations[j] <= 64 && !wide_ops && g_allow_fused && !feeds_split;
        if (U.fused) { D.variant = (c == 64) ? 1 : 0; D.generic = false; }     // weight blocks of C x 64
        U.wide = bf && c == 256 && (st.res_kernel - 1) * st.dilations[j] <= 64 && !wide_ops && g_allow_fused && !feeds_split;
        if (U.wide) { D.variant = 3; D.generic = false; }                      // weight blocks of 256 x 32
        Pending pd{&D, 0, 0, {}, {}, true, true};
        pd.in = pack_snake(ar, w, w + c, c, bf);     w += 2 * c;
        pd.w = pack_conv(ar, w, D, bf);              w += (size_t)c * c * st.res_kernel;
        pd.bias = pack_floats(ar, w, c);             w += c;
        pd.outp = pack_snake(ar, w, w + c, c, bf);   w += 2 * c;      // Snake between the two convolutions
        Pending pp{&P, 0, 0, {}, {}, false, false};
        if (U.fused || U.wide) {
            const size_t off = ar.reserve((size_t)c * c * 2);
            uint16_t* w1 = reinterpret_cast<uint16_t*>(ar.bytes.data() + off);
            if (U.wide) pack_w1_wide(w, w1);
            else pack_w1_fused(w, c, w1);
            to_fragment_order(w1, (size_t)c * c, c, U.wide ? 32 : c);
            fused_fix.push_back({&U, off});
        }
        pp.w = pack_conv(ar, w, P, bf);              w += (size_t)c * c;
        pp.bias = pack_floats(ar, w, c);             w += c;
        pend.push_back(pd);
        pend.push_back(pp);
        return DEMON_OK;
    };
    auto wide_fmt_of = [&](int width) { return (bf && width >= kSplitWidth) ? g_wide_fmt : (int)OP_BF16; };

    long long per_frame = st.c0, rate = 1;
    size_t stem_w_off = 0, stem_b_off = 0;
    SnakeOff hs{};  size_t hw = 0, hwf = 0, hb = 0;  bool head_mfma = false;
    const int oc = st.out_channels, hk = st.head_kernel;
    if (!encoder) {
        int cin = st.c0;
        for (int l = 0; l < nb; ++l) {
            const int s = st.strides[l], c = st.widths[l];
            Block& B = v->blocks[l];
            {
                ConvLayer& L = B.up;
                L.cin = cin; L.cout = c; L.ntaps = 2; L.stride = s;
                L.in_fmt = wide_fmt_of(c);
                if (L.in_fmt == OP_BF16X2) v->has_split_operands = true;
                if (bf) {
                    L.variant = choose_variant_bf16(cin, s * c);
                    if (L.variant < 0) return fail(DEMON_ERR_UNSUPPORTED, "bf16 path: no kernel for a %d -> %d stride-%d upsampling", cin, c, s);
                }
                Pending p{&L, 0, 0, {}, {}, true, false};
                p.in = pack_snake(ar, w, w + cin, cin, bf);  w += 2 * cin;
                p.w = pack_conv(ar, w, L, bf);               w += (size_t)cin * c * 2 * s;
                p.bias = pack_floats(ar, w, c);              w += c;
                pend.push_back(p);
            }
            for (int j = 0; j < nres; ++j) {
                // the last unit of a block feeds the next block's transposed conv
                const int next_fmt = (j + 1 == nres && l + 1 < nb) ? wide_fmt_of(st.widths[l + 1]) : (int)OP_BF16;
                rc = pack_unit(B.res[j], c, j, next_fmt);
                if (rc != DEMON_OK) return rc;
            }
            cin = c;
            rate *= s;
            per_frame = std::max(per_frame, rate * c);
        }
        // Rows each layer must produce beyond a window's interior (the receptive-field cone, walked from the
        // head back to the first block): a k-tap conv of dilation d reads d(k-1)/2 rows further out than it
        // writes; a transposed conv writing margin m reads inputs up to (m + p)/s + 1 rows out.
        {
            int m = (st.head_kernel - 1) / 2;
            for (int l = nb - 1; l >= 0; --l) {
                Block& B = v->blocks[l];
                for (int j = nres - 1; j >= 0; --j) {
                    B.res[j].pointwise.margin = m;
                    B.res[j].dilated.margin = m;
                    m += st.dilations[j] * ((st.res_kernel - 1) / 2);
                }
                B.up.margin = m;
                m = (m + st.strides[l] / 2) / st.strides[l] + 1;
            }
        }
        // head: weights as [tap][cin][out_channel] fp32
        hs = pack_snake(ar, w, w + cin, cin, bf);  w += 2 * cin;
        hw = ar.reserve(sizeof(float) * (size_t)hk * cin * oc);
        {
            float* dst = reinterpret_cast<float*>(ar.bytes.data() + hw);
            for (int o = 0; o < oc; ++o)
                for (int i = 0; i < cin; ++i)
                    for (int t = 0; t < hk; ++t) {
                        float val = w[((size_t)o * cin + i) * hk + t];
                        if (bf) { const uint32_t u = (uint32_t)f32_to_bf16_rne(val) << 16; memcpy(&val, &u, 4); }
                        dst[((size_t)t * cin + i) * oc + o] = val;
                    }
        }
        w += (size_t)oc * cin * hk;
        head_mfma = bf && (cin == 64 || cin == 32) && head_mfma_frag_count(cin, hk) <= 40;
        if (head_mfma) {
            // from the bf16-rounded weights, like every other weight of this path
            std::vector<float> wr((size_t)oc * cin * hk);
            for (size_t i = 0; i < wr.size(); ++i) { const uint32_t u = (uint32_t)f32_to_bf16_rne((w - (size_t)oc * cin * hk)[i]) << 16; memcpy(&wr[i], &u, 4); }
            hwf = ar.reserve(head_mfma_frag_count(cin, hk) * 64 * 16);
            pack_head_mfma(wr.data(), cin, oc, hk, reinterpret_cast<uint16_t*>(ar.bytes.data() + hwf));
        }
        hb = pack_floats(ar, w, oc);
        w += oc;
        v->head_cin = cin;
    } else {
        // ---- encoder: stem from the waveform, then per block (from the audio rate down) the units and the strided conv
        for (int s : st.strides) rate *= s;
        const int cs = st.widths[nb - 1];
        v->stem_cout = cs;
        stem_w_off = ar.reserve(sizeof(float) * (size_t)hk * oc * cs);
        {
            // [C][channels][k] -> [k][channels][C]
            float* dst = reinterpret_cast<float*>(ar.bytes.data() + stem_w_off);
            for (int o = 0; o < cs; ++o)
                for (int i = 0; i < oc; ++i)
                    for (int t = 0; t < hk; ++t) {
                        float val = w[((size_t)o * oc + i) * hk + t];
                        if (bf) { const uint32_t u = (uint32_t)f32_to_bf16_rne(val) << 16; memcpy(&val, &u, 4); }
                        dst[((size_t)t * oc + i) * cs + o] = val;
                    }
        }
        w += (size_t)cs * oc * hk;
        stem_b_off = pack_floats(ar, w, cs);  w += cs;
        per_frame = rate * cs;
        for (int b = 0; b < nb; ++b) {
            const int l = nb - 1 - b;
            const int s = st.strides[l], c = st.widths[l];
            const int cn = l > 0 ? st.widths[l - 1] : 2 * st.c0;
            Block& B = v->blocks[b];
            per_frame = std::max(per_frame, rate * c);
            ConvLayer& L = B.up;               // the strided conv after the units
            L.cin = c; L.cout = cn; L.ntaps = 2 * s; L.stride = 0; L.down = s;
            L.in_fmt = (bf && c >= kSplitWidth) ? (int)OP_F16 : (int)OP_BF16;
            for (int j = 0; j < nres; ++j) {
                // the last unit of a block feeds the block's strided conv
                rc = pack_unit(B.res[j], c, j, j + 1 == nres ? L.in_fmt : (int)OP_BF16);
                if (rc != DEMON_OK) return rc;
            }
            if (bf) {
                L.variant = choose_variant_bf16(c * (s / 2), cn);
                if (L.variant == 1) L.variant = cn % 32 == 0 ? 2 : -1;      // the 256-column tile has no strided form
                if (L.variant < 0) return fail(DEMON_ERR_UNSUPPORTED, "bf16 path: no kernel for a %d -> %d stride-%d downsampling", c, cn, s);
            }
            Pending p{&L, 0, 0, {}, {}, true, false};
            p.in = pack_snake(ar, w, w + c, c, bf);  w += 2 * c;
            p.w = pack_conv(ar, w, L, bf);           w += (size_t)cn * c * 2 * s;
            p.bias = pack_floats(ar, w, cn);         w += cn;
            pend.push_back(p);
            rate /= s;
            per_frame = std::max(per_frame, rate * cn);
            // The last one has the longest K (1024 channels, stride 10: 20480) and the fewest columns, one a frame: 12 workgroups for 75 frames and 26 us a
            // launch in one piece, 9 in parts; 72 and 18 for 60 s.  In parts whatever the call's size, so that a value does not depend on that, although very long
            // calls lose by the sums' traffic, in us with an event after the launch, conv and sampling step, one piece / parts: K of 20480 27 + 6 / 8 + 6 up to 400
            // frames, 68 + 13 / 46 + 15 at 6000, 169 + 36 / 170 + 50 at 24000; K of 4096 to 128 rows 9 + 6 / 7 + 6, 15 + 12 / 19 + 14, 40 + 35 / 59 + 40 (that whole
            // encode 354 us before, 314 with the stem's gain).  For K whose 64-channel chunks divide into eight parts of whole stages of two chunks (others, 75 chunks of
            // 960 channels at stride 10, go in one piece), up to 256 rows, and where the sums fit where the residual stream would go.
            L.parts = bf && l == 0 && L.variant == 0 && cn <= 256 && c * (s / 2) % (128 * kConvParts) == 0 && 2ll * kConvParts * cn <= per_frame;
        }
        // Rows each layer must produce beyond a window's interior, walked from the moments back to the stem: a strided
        // conv writing margin m reads inputs up to m s + s/2 rows out, a k-tap conv of dilation d d(k-1)/2 rows further.
        {
            int m = 0;
            for (int b = nb - 1; b >= 0; --b) {
                Block& B = v->blocks[b];
                const int s = st.strides[nb - 1 - b];
                B.up.margin = m;
                m = m * s + s / 2;
                for (int j = nres - 1; j >= 0; --j) {
                    B.res[j].pointwise.margin = m;
                    B.res[j].dilated.margin = m;
                    m += st.dilations[j] * ((st.res_kernel - 1) / 2);
                }
            }
            v->stem_margin = m;
        }
        rate = 1;                              // no window waveforms to hold
    }

    for (const Block& B : v->blocks) {
        auto staged = [&](const ConvLayer& L) { return bf && L.generic && L.variant != 0; };
        if (staged(B.up)) v->has_staged_convs = true;
        for (const ResUnit& U : B.res)
            if (staged(U.dilated)) v->has_staged_convs = true;
    }

    // ---- device memory
    const size_t act_elems = (size_t)v->cap_frames * (size_t)per_frame;
    v->ws.act_elems = act_elems;
    v->per_frame = per_frame;
    const size_t head_bytes = encoder ? 256 : (size_t)v->cap_frames * (size_t)rate * oc * sizeof(float);
    auto cleanup = [&]() {
        if (v->d_params) (void)hipFree(v->d_params);
        for (void* b : v->ws.buf) if (b) (void)hipFree(b);
        if (v->ws.head_out) (void)hipFree(v->ws.head_out);
        if (v->d_slot_arena) (void)hipFree(v->d_slot_arena);
        if (v->ws.slot_gated) (void)hipFree(v->ws.slot_gated);
        if (v->ev_fork) (void)hipEventDestroy(v->ev_fork);
        if (v->ev_join) (void)hipEventDestroy(v->ev_join);
        if (v->stream2) (void)hipStreamDestroy(v->stream2);
    };
    ar.reserve(kWeightSlack);
    hipError_t e = hipMalloc(&v->d_params, ar.bytes.size());
    // fp32 path: 4 bytes per element; bf16 path: half residual stream (2 bytes), bf16 operand buffers with hi and lo planes (4)
    for (int i = 0; e == hipSuccess && i < (bf ? 5 : 3); ++i) e = hipMalloc(&v->ws.buf[i], act_elems * ((bf && i < 2) ? 2 : 4));
    if (e == hipSuccess) e = hipMalloc((void**)&v->ws.head_out, head_bytes);
    if (e == hipSuccess) e = hipMalloc((void**)&v->d_slot_arena, sizeof(Slot) * kMaxSlots * kPlanCache);
    if (e == hipSuccess) e = hipMalloc((void**)&v->ws.slot_gated, sizeof(Slot) * kMaxSlots);
    if (e == hipSuccess && bf && g_dual_stream && v->cap_frames >= two_group_frames(v.get())) {      // else no call can use it
        e = hipStreamCreateWithFlags(&v->stream2, hipStreamNonBlocking);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&v->ev_fork, hipEventDisableTiming);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&v->ev_join, hipEventDisableTiming);
    }
    if (e == hipSuccess) e = hipMemcpy(v->d_params, ar.bytes.data(), ar.bytes.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) { cleanup(); return hip_fail(e, "allocating device memory"); }

    const unsigned char* base = static_cast<const unsigned char*>(v->d_params);
    auto fptr = [&](size_t off) { return reinterpret_cast<const float*>(base + off); };
    for (const Pending& p : pend) {
        p.L->w = base + p.w;
        p.L->bias = fptr(p.bias);
        if (p.has_in) { p.L->in_alpha = fptr(p.in.alpha); p.L->in_inv_beta = fptr(p.in.inv_beta); }
        if (p.has_out) { p.L->out_alpha = fptr(p.outp.alpha); p.L->out_inv_beta = fptr(p.outp.inv_beta); }
    }
    for (const FusedFix& f : fused_fix) f.U->w1_fused = reinterpret_cast<const uint16_t*>(base + f.off);
    if (encoder) {
        v->stem_w = fptr(stem_w_off); v->stem_bias = fptr(stem_b_off);
    } else {
        v->head_alpha = fptr(hs.alpha); v->head_inv_beta = fptr(hs.inv_beta);
        v->head_w = fptr(hw); v->head_bias = fptr(hb);
        if (head_mfma) v->head_wfrag = reinterpret_cast<const uint16_t*>(base + hwf);
    }

    // ---- the layer sequence in processing order, each step with the layer that takes its output as an MFMA operand
    // (bf16 path): the next step's resampling conv or the dilated conv of its unit, unless that unit reads the residual
    // stream itself (narrow fused unit) or nothing follows (head, sampling step)
    for (int b = 0; b < nb; ++b) {
        Block& B = v->blocks[b];
        if (!encoder) { Step t; t.conv = &B.up; v->steps.push_back(t); }
        for (int j = 0; j < nres; ++j) { Step t; t.unit = &B.res[j]; v->steps.push_back(t); }
        if (encoder) { Step t; t.conv = &B.up; v->steps.push_back(t); }
    }
    {
        double r = 1;
        if (encoder) for (int s : st.strides) r *= s;
        for (const Step& t : v->steps) {
            const ConvLayer& L = t.conv ? *t.conv : t.unit->dilated;
            if (t.conv) r = L.down > 0 ? r / L.down : r * L.stride;
            v->frame_flop += 2.0 * r * L.cin * L.cout * (t.conv ? L.ntaps : L.ntaps + 1);
        }
    }
    auto operand_layer = [](const Step& t) -> const ConvLayer* {
        if (t.conv) return t.conv;
        return t.unit->fused ? nullptr : &t.unit->dilated;
    };
    for (size_t i = 0; i + 1 < v->steps.size(); ++i) v->steps[i].consumer = operand_layer(v->steps[i + 1]);
    v->first_consumer = operand_layer(v->steps[0]);
    // the head can run inside the last residual unit's kernel when that unit is the fused 64-channel form
    if (!encoder && head_mfma && !(cfg->flags & DEMON_VAE_FLAG_NO_HEAD_FUSION) && !v->steps.empty()) {
        const Step& last = v->steps.back();
        v->head_fusable = last.unit && last.unit->fused && last.unit->dilated.cin == 64 && oc <= 8 && hk <= 7 &&
                          last.unit->pointwise.margin == (hk - 1) / 2;
    }

    *out = v.release();
    return DEMON_OK;
}

}  // namespace

extern "C" {

demon_status demon_vae_create(const demon_vae_config* cfg, const float* host_weights, size_t n_floats, demon_vae** out)
{
    return create_impl(cfg, host_weights, n_floats, false, out);
}

demon_status demon_vae_create_encoder(const demon_vae_config* cfg, const float* host_weights, size_t n_floats, demon_vae** out)
{
    return create_impl(cfg, host_weights, n_floats, true, out);
}

void demon_vae_destroy(demon_vae* v)
{
    if (!v) return;
    (void)hipFree(v->d_params);
    for (void* b : v->ws.buf) if (b) (void)hipFree(b);
    (void)hipFree(v->ws.head_out);
    (void)hipFree(v->d_slot_arena);
    (void)hipFree(v->ws.slot_gated);
    for (hipEvent_t e : v->events) (void)hipEventDestroy(e);
    if (v->ev_fork) (void)hipEventDestroy(v->ev_fork);
    if (v->ev_join) (void)hipEventDestroy(v->ev_join);
    if (v->stream2) (void)hipStreamDestroy(v->stream2);
    delete v;
}

demon_status demon_vae_receptive_field(const demon_vae* v, int* halo_left, int* halo_right)
{
    if (!v || !halo_left || !halo_right) return fail(DEMON_ERR_INVALID_ARG, "NULL argument");
    *halo_left = v->rf_left; *halo_right = v->rf_right;
    return DEMON_OK;
}

static demon_status decode_checked(demon_vae* v, const void* d_latent, int n_clips, int n_frames,
                                   int frame_begin, int frame_end, int window, int halo, const int* d_skip,
                                   float* d_out, int16_t* d_pcm, void* stream)
{
    clear_error();
    if (!v || !d_latent || (!d_out && !d_pcm)) return fail(DEMON_ERR_INVALID_ARG, "NULL argument");
    if (v->encoder) return fail(DEMON_ERR_INVALID_ARG, "this handle is an encoder (demon_vae_create_encoder): use demon_vae_encode_windowed");
    if (n_clips < 1) return fail(DEMON_ERR_INVALID_ARG, "n_clips must be >= 1");
    if (n_frames < 1) return fail(DEMON_ERR_INVALID_ARG, "n_frames must be >= 1");
    if (frame_begin < 0) return fail(DEMON_ERR_INVALID_ARG, "frame_begin must be >= 0");
    if (frame_end > n_frames) return fail(DEMON_ERR_INVALID_ARG, "frame_end %d exceeds n_frames %d", frame_end, n_frames);
    if (frame_begin >= frame_end) return fail(DEMON_ERR_INVALID_ARG, "empty frame range [%d, %d)", frame_begin, frame_end);
    if (window < 1) return fail(DEMON_ERR_INVALID_ARG, "window must be >= 1");
    if (halo < -1) return fail(DEMON_ERR_INVALID_ARG, "halo must be >= -1");
    if (n_frames > v->max_frames) return fail(DEMON_ERR_WORKSPACE, "n_frames %d exceeds max_frames %d", n_frames, v->max_frames);
    if (n_clips > v->max_clips) return fail(DEMON_ERR_WORKSPACE, "n_clips %d exceeds max_clips %d", n_clips, v->max_clips);
    if (halo == -1) halo = std::max(v->rf_left, v->rf_right);
    Plan* plan = nullptr;
    const demon_status rc = get_plan(v, n_clips, n_frames, frame_begin, frame_end, window, halo, d_skip != nullptr, (hipStream_t)stream, &plan);
    if (rc != DEMON_OK) return rc;
    Io io;
    io.d_latent = d_latent; io.d_skip = d_skip; io.d_out = d_out; io.d_pcm = d_pcm; io.n_frames = n_frames;
    return run_pass(v, v->ws, plan, io, (hipStream_t)stream);
}

demon_status demon_vae_decode_windowed(demon_vae* v, const void* d_latent, int n_clips, int n_frames,
                                       int frame_begin, int frame_end, int window, int halo,
                                       float* d_out, void* stream)
{
    if (!d_out) { clear_error(); return fail(DEMON_ERR_INVALID_ARG, "NULL argument"); }
    return decode_checked(v, d_latent, n_clips, n_frames, frame_begin, frame_end, window, halo, nullptr, d_out, nullptr, stream);
}

demon_status demon_vae_decode_windowed_gated(demon_vae* v, const void* d_latent, int n_clips, int n_frames,
                                             int frame_begin, int frame_end, int window, int halo,
                                             const int* d_skip, float* d_out, void* stream)
{
    if (!d_out || !d_skip) { clear_error(); return fail(DEMON_ERR_INVALID_ARG, "NULL argument"); }
    return decode_checked(v, d_latent, n_clips, n_frames, frame_begin, frame_end, window, halo, d_skip, d_out, nullptr, stream);
}

demon_status demon_vae_decode_windowed_pcm16(demon_vae* v, const void* d_latent, int n_clips, int n_frames,
                                             int frame_begin, int frame_end, int window, int halo,
                                             int16_t* d_pcm, void* stream)
{
    if (!d_pcm) { clear_error(); return fail(DEMON_ERR_INVALID_ARG, "NULL argument"); }
    return decode_checked(v, d_latent, n_clips, n_frames, frame_begin, frame_end, window, halo, nullptr, nullptr, d_pcm, stream);
}

demon_status demon_vae_decode_windowed_static(demon_vae* v, const void* d_latent, int n_clips, int n_frames,
                                              int frame_begin, int frame_end, int window, int halo,
                                              float* d_out, void* stream_)
{
    clear_error();
    hipStream_t stream = (hipStream_t)stream_;
    if (!v || !d_latent || !d_out) return fail(DEMON_ERR_INVALID_ARG, "NULL argument");
    if (v->encoder) return fail(DEMON_ERR_INVALID_ARG, "this handle is an encoder (demon_vae_create_encoder): use demon_vae_encode_windowed");
    if (n_clips < 1) return fail(DEMON_ERR_INVALID_ARG, "n_clips must be >= 1");
    if (n_frames < 1) return fail(DEMON_ERR_INVALID_ARG, "n_frames must be >= 1");
    if (frame_begin < 0) return fail(DEMON_ERR_INVALID_ARG, "frame_begin must be >= 0");
    if (frame_end > n_frames) return fail(DEMON_ERR_INVALID_ARG, "frame_end %d exceeds n_frames %d", frame_end, n_frames);
    if (frame_begin >= frame_end) return fail(DEMON_ERR_INVALID_ARG, "empty frame range [%d, %d)", frame_begin, frame_end);
    if (window < 1) return fail(DEMON_ERR_INVALID_ARG, "window must be >= 1");
    if (halo < -1) return fail(DEMON_ERR_INVALID_ARG, "halo must be >= -1");
    if (halo == -1) halo = std::max(v->rf_left, v->rf_right);
    if (!v->scratch) return fail(DEMON_ERR_HIP, "the static scratch array was not found on this device");

    // the window grid, counted on the host without building it (the table itself is written by a kernel)
    const GridCount gc = count_grid(n_frames, frame_begin, frame_end, window, halo);
    const long long per_clip = gc.per_clip, clip_frames = gc.clip_frames;
    if (per_clip * n_clips > kMaxSlots)
        return fail(DEMON_ERR_WORKSPACE, "%lld windows exceed the limit of %d", per_clip * n_clips, kMaxSlots);
    const long long total = clip_frames * n_clips;
    const demon_status prc = check_plane(v, gc.max_len);
    if (prc != DEMON_OK) return prc;

    // carve the call's memory out of the static array: window table, activation buffers (the head writes the caller's waveform)
    const bool bf = v->dtype == DEMON_BF16;
    const size_t act_elems = (size_t)total * (size_t)v->per_frame;
    const size_t planes = (bf && v->has_split_operands) ? 2 : 1;
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t at = off; off = (at + bytes + 255) & ~(size_t)255; return at; };
    const size_t at_slots = take(sizeof(Slot) * (size_t)(per_clip * n_clips));
    size_t at_buf[5] = {0, 0, 0, 0, 0};
    for (int i = 0; i < (bf ? 5 : 3); ++i) at_buf[i] = take(act_elems * (bf ? (i < 2 ? 2 : 2 * planes) : 4));
    if (off > kStaticScratchBytes)
        return fail(DEMON_ERR_WORKSPACE, "the call needs %zu bytes of scratch for %lld extended frames, the static array holds %zu",
                    off, total, kStaticScratchBytes);
    Workspace ws;
    for (int i = 0; i < (bf ? 5 : 3); ++i) ws.buf[i] = v->scratch + at_buf[i];
    ws.act_elems = act_elems;

    Plan plan;
    plan.valid = true;
    plan.n_clips = n_clips; plan.n_frames = n_frames; plan.frame_begin = frame_begin; plan.frame_end = frame_end;
    plan.window = window; plan.halo = halo;
    const Grid grid = callers_own(v) ? Grid{window, halo} : computed_grid(v, n_clips, n_frames, frame_begin, frame_end, window, halo, total, false);
    const GridCount cc = count_grid(n_frames, frame_begin, frame_end, grid.window, grid.halo);
    plan.n_slots = (int)(cc.per_clip * n_clips); plan.max_len = cc.max_len; plan.max_int = cc.max_int;
    plan.total_frames = cc.clip_frames * n_clips;
    plan.d_slots = reinterpret_cast<Slot*>(v->scratch + at_slots);
    HIP_TRY(launch_plan_slots(plan.d_slots, n_clips, (int)cc.per_clip, (int)cc.clip_frames, n_frames, frame_begin, frame_end, grid.window, grid.halo, stream),
            "window table");
    Io io;
    io.d_latent = d_latent; io.d_out = d_out; io.n_frames = n_frames;
    return run_pass(v, ws, &plan, io, stream);
}

demon_status demon_vae_encode_windowed(demon_vae* v, const float* d_wave, int n_clips, int n_frames,
                                       int frame_begin, int frame_end, int window, int halo,
                                       const float* d_eps, float* d_moments, void* d_latent, void* stream)
{
    clear_error();
    if (!v || !d_wave || (!d_moments && !d_latent)) return fail(DEMON_ERR_INVALID_ARG, "NULL argument");
    if (!v->encoder) return fail(DEMON_ERR_INVALID_ARG, "this handle is a decoder (demon_vae_create): use demon_vae_decode_windowed");
    if (n_clips < 1) return fail(DEMON_ERR_INVALID_ARG, "n_clips must be >= 1");
    if (n_frames < 1) return fail(DEMON_ERR_INVALID_ARG, "n_frames must be >= 1");
    if (frame_begin < 0) return fail(DEMON_ERR_INVALID_ARG, "frame_begin must be >= 0");
    if (frame_end > n_frames) return fail(DEMON_ERR_INVALID_ARG, "frame_end %d exceeds n_frames %d", frame_end, n_frames);
    if (frame_begin >= frame_end) return fail(DEMON_ERR_INVALID_ARG, "empty frame range [%d, %d)", frame_begin, frame_end);
    if (window < 1) return fail(DEMON_ERR_INVALID_ARG, "window must be >= 1");
    if (halo < -1) return fail(DEMON_ERR_INVALID_ARG, "halo must be >= -1");
    if (n_frames > v->max_frames) return fail(DEMON_ERR_WORKSPACE, "n_frames %d exceeds max_frames %d", n_frames, v->max_frames);
    if (n_clips > v->max_clips) return fail(DEMON_ERR_WORKSPACE, "n_clips %d exceeds max_clips %d", n_clips, v->max_clips);
    if ((long long)n_frames * v->st.total_stride() > 0x7fffffffll) return fail(DEMON_ERR_UNSUPPORTED, "clips longer than 2^31 samples");
    if (halo == -1) halo = std::max(v->rf_left, v->rf_right);
    Plan* plan = nullptr;
    const demon_status rc = get_plan(v, n_clips, n_frames, frame_begin, frame_end, window, halo, false, (hipStream_t)stream, &plan);
    if (rc != DEMON_OK) return rc;
    Io io;
    io.d_wave = d_wave; io.d_eps = d_eps; io.d_moments = d_moments; io.d_zout = d_latent; io.n_frames = n_frames;
    return run_pass(v, v->ws, plan, io, (hipStream_t)stream);
}

demon_status demon_vae_encode(demon_vae* v, const float* d_wave, int n_clips, int n_frames, const float* d_eps,
                              float* d_moments, void* d_latent, void* stream)
{
    // one window per clip covering [0, n_frames), no halo: the same kernels as the windowed encode
    return demon_vae_encode_windowed(v, d_wave, n_clips, n_frames, 0, n_frames, n_frames > 0 ? n_frames : 1, 0, d_eps, d_moments, d_latent, stream);
}

demon_status demon_vae_decode(demon_vae* v, const void* d_latent, int n_clips, int n_frames, float* d_out, void* stream)
{
    // one window per clip covering [0, n_frames), no halo: the same kernels as the windowed decode
    return demon_vae_decode_windowed(v, d_latent, n_clips, n_frames, 0, n_frames, n_frames > 0 ? n_frames : 1, 0, d_out, stream);
}

demon_status demon_vae_latent_similarity(const void* d_curr, const void* d_prev, int n_clips, long long elems_per_clip,
                                         demon_dtype dtype, float threshold, float* d_mse, int* d_unchanged, void* stream)
{
    clear_error();
    if (!d_curr || !d_prev || (!d_mse && !d_unchanged)) return fail(DEMON_ERR_INVALID_ARG, "NULL argument");
    if (n_clips < 1 || n_clips > 65535) return fail(DEMON_ERR_INVALID_ARG, "n_clips must be in [1, 65535]");
    if (elems_per_clip < 1) return fail(DEMON_ERR_INVALID_ARG, "elems_per_clip must be >= 1");
    if (dtype != DEMON_F32 && dtype != DEMON_BF16) return fail(DEMON_ERR_INVALID_ARG, "unknown dtype");
    if (!(threshold >= 0.0f)) return fail(DEMON_ERR_INVALID_ARG, "threshold must be >= 0");
    HIP_TRY(launch_latent_mse(d_curr, d_prev, n_clips, elems_per_clip, dtype == DEMON_BF16, threshold, d_mse, d_unchanged,
                              (hipStream_t)stream), "latent similarity");
    return DEMON_OK;
}

demon_status demon_vae_crossfade(const float* d_prev_tail, long long prev_stride, const float* d_next_head, long long next_stride,
                                 float* d_out, long long out_stride, int n_planes, int n_samples, void* stream)
{
    clear_error();
    if (!d_prev_tail || !d_next_head || !d_out) return fail(DEMON_ERR_INVALID_ARG, "NULL argument");
    if (n_planes < 1 || n_planes > 65535) return fail(DEMON_ERR_INVALID_ARG, "n_planes must be in [1, 65535]");
    if (n_samples < 1) return fail(DEMON_ERR_INVALID_ARG, "n_samples must be >= 1");
    if (prev_stride < 0 || next_stride < 0 || out_stride < 0) return fail(DEMON_ERR_INVALID_ARG, "negative plane stride");
    if (n_planes > 1 && out_stride < n_samples) return fail(DEMON_ERR_INVALID_ARG, "output planes overlap");
    HIP_TRY(launch_crossfade(d_prev_tail, prev_stride, d_next_head, next_stride, d_out, out_stride, n_planes, n_samples,
                             (hipStream_t)stream), "crossfade");
    return DEMON_OK;
}

demon_status demon_vae_set_timing(demon_vae* v, int level)
{
    if (!v) return fail(DEMON_ERR_INVALID_ARG, "NULL handle");
    if (level < 0 || level > 2) return fail(DEMON_ERR_INVALID_ARG, "timing level must be 0, 1 or 2");
    size_t launches = 3;                                    // gather, head, 16-bit render
    for (const Block& B : v->blocks) launches += 1 + 2 * B.res.size();
    v->marks_per_call = (int)launches + 1;
    while (level > 0 && v->events.size() < (size_t)v->marks_per_call * kTimingRing) {
        hipEvent_t e;
        hipError_t rc = hipEventCreate(&e);
        if (rc != hipSuccess) return hip_fail(rc, "hipEventCreate");
        v->events.push_back(e);
    }
    v->timing = level;
    v->n_marks = 0;
    v->timed_calls = 0;
    return DEMON_OK;
}

demon_status demon_vae_get_timing(demon_vae* v, float* ms, int capacity, int* n)
{
    if (!v || !n) return fail(DEMON_ERR_INVALID_ARG, "NULL argument");
    const int avail = v->n_marks > 0 ? v->n_marks - 1 : 0;
    *n = avail;
    const int calls = v->timed_calls < kTimingRing ? v->timed_calls : kTimingRing;
    if (!ms || calls == 0) return DEMON_OK;
    for (int i = 0; i < avail && i < capacity; ++i) {
        double sum = 0;
        for (int c = 0; c < calls; ++c) {
            float t = 0;
            const int base = c * v->marks_per_call;
            hipError_t rc = hipEventElapsedTime(&t, v->events[base + i], v->events[base + i + 1]);
            if (rc != hipSuccess) return hip_fail(rc, "hipEventElapsedTime");
            sum += t;
        }
        ms[i] = (float)(sum / calls);
    }
    v->timed_calls = 0;
    return DEMON_OK;
}

void demon_vae_test_pack_bf16(const float* w, int cin, int cout, int ntaps, int stride, int variant, int as_half,
                              int permute_rows, uint16_t* dst)
{
    pack_bf16(w, cin, cout, ntaps, stride, variant, as_half != 0, permute_rows != 0, dst);
}

void demon_vae_test_pack_w1_fused(const float* w, int c, uint16_t* dst) { pack_w1_fused(w, c, dst); }

uint16_t demon_vae_test_f32_to_f16(float v) { return f32_to_f16_rne(v); }

demon_status demon_vae_debug_tap(demon_vae* v, int layer, float* d_dst, size_t capacity)
{
    if (!v) return fail(DEMON_ERR_INVALID_ARG, "NULL handle");
    if (layer >= 0 && !d_dst) return fail(DEMON_ERR_INVALID_ARG, "d_dst is NULL");
    v->tap_layer = layer; v->tap_dst = d_dst; v->tap_cap = capacity;
    return DEMON_OK;
}

demon_status demon_vae_debug_callers_grid(demon_vae* v, int on)
{
    if (!v) return fail(DEMON_ERR_INVALID_ARG, "NULL handle");
    v->callers_grid = on != 0;
    return DEMON_OK;
}

demon_status demon_vae_debug_last_grid(const demon_vae* v, int* n_windows, long long* extended_frames, int* n_groups)
{
    if (!v || !n_windows || !extended_frames || !n_groups) return fail(DEMON_ERR_INVALID_ARG, "NULL argument");
    *n_windows = v->last_windows; *extended_frames = v->last_frames; *n_groups = v->last_groups;
    return DEMON_OK;
}

}  // extern "C"
