// Fused residual unit for 256 channels:
//     h += W1 * snake2(W7 (*) a + b7) + b1,      a = bf16(snake1(h)) written by the producer of h
// in one kernel: the activated branch tensor between the two convolutions never goes to HBM, and the 1x1
// convolution (a short reduction with a long epilogue, bound by HBM when it runs on its own) costs one more
// K loop instead of a launch.  Three kernels with the same results: weights streamed to registers for seven taps (narrow tiles for
// launches of few of them, tall ones else), and the LDS-staged one, first below, for any number of taps.
//
// LDS-staged: workgroup = 4 waves, tile = all 256 channels x 128 time columns, every wave all 256 rows of its 32 columns
// (8 accumulator tiles of 32 x 32).  The dilated convolution runs as in kernels_bf16.hip on the pre-activated
// bf16 operand, with K stages of 32 channels so that two workgroups fit the LDS of a CU.  As in the narrow fused
// unit, a lane of an accumulator tile holds column j and rows 8g + 4h + {0..3}, which after bias + Snake are the
// B fragments of the 1x1 convolution once its K axis is permuted to that order (fused_k_to_channel); its weights,
// 128 KB, do not fit the LDS and are streamed through the weight buffers in 8 blocks of 32 k-slots.
// In the 1x1 convolution the roles are swapped: the fragments are the row operand (rows = time), the weights the
// column operand, so its accumulator tile is [time][output channel slot]; the weight rows are packed so that slot j
// of tile mo is channel 8 j + mo.  A lane then owns 8 consecutive channels (16 bytes of half) of a time row and 32
// lanes the whole row: residual loads and stores are contiguous straight from the accumulators.
// The residual stream is updated in place (only this tile reads or writes its elements); the emitted operand of
// the next layer goes to a second buffer because neighbouring tiles still read this tile's input rows.
#include <algorithm>
#include <type_traits>

#include "device_common.h"

namespace demon {

namespace {

constexpr int W_CH = 256, W_KC = 32, W_LDK = W_KC + 8, W_NT = 128, W_TM = W_CH / 32, W_MAXSPAN = 64;
constexpr int W_XR_MAX = W_NT + W_MAXSPAN;
constexpr int W_SEGS = W_KC / 8, W_RPP = 256 / W_SEGS;
constexpr int W_A_CH = W_CH * W_SEGS, W_A_ITERS = W_A_CH / 256;
constexpr int W_X_ITERS = (W_XR_MAX + W_RPP - 1) / W_RPP;
constexpr int W_NCHUNKS = W_CH / W_KC;

struct WideParams {
    const uint16_t* xa;          // activated input, bf16 [rows][256]
    hres_t* y;                   // residual stream, in place
    uint16_t* ya;                // optional bf16(snake_next(y)) (EMIT); not the buffer of xa
    const uint16_t* w7;          // [chunk][tap] blocks of 256 x 32 bf16
    const uint16_t* w1;          // [chunk] blocks of 256 x 32 bf16, K axis permuted
    const float* b7; const float* b1;
    const float* a2; const float* ib2;    // Snake between the two convolutions (alpha in revolutions, 1/(beta+eps))
    const float* a3; const float* ib3;    // Snake of the consumer (EMIT)
    const Slot* slots;
    int r, ntaps, tap0, tap_step, margin;
    bool y_dead;                 // EMIT: y is read only, nothing after the unit reads the sum
};

template <bool EMIT>
__global__ __launch_bounds__(256) void res_unit_wide_kernel(WideParams p)
{
    fp16_saturate_on();
    constexpr int CH = W_CH, KC = W_KC, LDK = W_LDK, NT = W_NT, TM = W_TM;
    constexpr int A_ITERS = W_A_ITERS, X_ITERS = W_X_ITERS, SEGS = W_SEGS, RPP = W_RPP;
    constexpr int AS_BYTES = 2 * CH * LDK * 2, XS_BYTES = W_XR_MAX * LDK * 2;
    constexpr int SMEM_BYTES = AS_BYTES + XS_BYTES;
    __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM_BYTES];
    __shared__ __attribute__((aligned(16))) float prm[4 * CH];     // b7 | a2 | ib2 | b1
    uint16_t* As = reinterpret_cast<uint16_t*>(smem);
    uint16_t* Xs = reinterpret_cast<uint16_t*>(smem + AS_BYTES);

    const Slot s = p.slots[blockIdx.y];
    const int nrows = s.len * p.r;
    const int out_lo = max(0, s.crop * p.r - p.margin);
    const int out_hi = min(nrows, (s.crop + s.n_int) * p.r + p.margin);
    // Workgroups are dealt to the 8 XCDs round-robin by linear id, and each XCD has its own L2: XCD x takes a contiguous
    // eighth of a window's tiles, in order, so that neighbouring tiles (which share their halo rows) run on the same
    // XCD at about the same time.  The eighths rotate with the window index (the last one may be short).
    const int tiles8 = (int)(gridDim.x >> 3);
    const int tile = (int)((blockIdx.x + blockIdx.y) & 7u) * tiles8 + (int)(blockIdx.x >> 3);
    const int n0 = out_lo + tile * NT;
    if (n0 >= out_hi) return;
    const long long rowbase = (long long)s.row0 * p.r;

    const int last_off = p.tap0 + (p.ntaps - 1) * p.tap_step;
    const int minoff = min(p.tap0, last_off);
    const int XR = NT + max(p.tap0, last_off) - minoff;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wn = tid >> 6;
    const int j = lane & 31, h = lane >> 5;
    const int seg = tid % SEGS;

    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(p.xa + rowbase * CH, (unsigned)nrows * CH * 2u);
    const __amdgpu_buffer_rsrc_t rs_y = make_rsrc(p.y + rowbase * CH, (unsigned)out_hi * CH * (unsigned)sizeof(hres_t));
    const __amdgpu_buffer_rsrc_t rs_ys = make_rsrc(p.y + rowbase * CH, EMIT && p.y_dead ? 0u : (unsigned)out_hi * CH * (unsigned)sizeof(hres_t));
    const __amdgpu_buffer_rsrc_t rs_a = make_rsrc(p.ya + rowbase * CH, EMIT ? (unsigned)out_hi * CH * 2u : 0u);
    const int nstages = W_NCHUNKS * p.ntaps;
    const __amdgpu_buffer_rsrc_t rs_w7 = weight_rsrc(p.w7, (unsigned)nstages * (W_A_CH * 16u));
    const __amdgpu_buffer_rsrc_t rs_w1 = weight_rsrc(p.w1, (unsigned)W_NCHUNKS * (W_A_CH * 16u));

    // Staging pattern of the activations.  An LDS row is 80 bytes (20 banks), so the 8 lanes that one cycle of a 16-byte LDS write serves
    // must not hold two neighbouring rows (rows r and r + 1 overlap in 4 banks): lanes 0..3 of each group of 8 take the
    // four pieces of row r, lanes 4..7 those of row r + 4, which starts 16 banks further.  A pass of 256 threads covers
    // 64 rows; srow is the thread's row within a pass.
    const int srow = 8 * (tid >> 5) + ((tid >> 3) & 3) + 4 * ((tid >> 2) & 1);
    const unsigned a_voff = tid * 16u;
    const unsigned x_voff = ((unsigned)((n0 + minoff + srow) * CH) + seg * 8u) * 2u;     // may wrap "negative": out of range
    constexpr unsigned x_row_step = RPP * CH * 2u;

    u32x4 ra[A_ITERS], rb[A_ITERS];     // rb: second set, only for the blocks of the 1x1 weights (requested two ahead)
    u32x4 rx[X_ITERS];
    auto load_set = [&](u32x4 (&r)[A_ITERS], __amdgpu_buffer_rsrc_t rs, int block) __attribute__((always_inline)) {
        const unsigned base = (unsigned)block * (W_A_CH * 16u);
#pragma unroll
        for (int it = 0; it < A_ITERS; ++it) r[it] = __builtin_amdgcn_raw_buffer_load_b128(rs, a_voff, base + it * 4096u, 0);
    };
    auto store_set = [&](const u32x4 (&r)[A_ITERS], int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < A_ITERS; ++it)
            *reinterpret_cast<u32x4*>(&As[buf * CH * LDK + frag_row<KC>(tid + it * 256) * LDK + frag_piece<KC>(tid + it * 256) * 8]) = r[it];
    };
    auto store_a = [&](int buf) __attribute__((always_inline)) { store_set(ra, buf); };
    auto load_x = [&](int chunk) __attribute__((always_inline)) {
        const unsigned coff = x_voff + (unsigned)(chunk * KC) * 2u;
#pragma unroll
        for (int it = 0; it < X_ITERS; ++it) {
            if (it * RPP >= XR) break;                        // uniform
            rx[it] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, coff + it * x_row_step, 0, 0);
        }
    };
    auto store_x = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < X_ITERS; ++it) {
            if (it * RPP >= XR) break;                        // uniform
            const int xr = srow + it * RPP;
            if (xr >= W_XR_MAX) continue;
            *reinterpret_cast<u32x4*>(&Xs[xr * LDK + seg * 8]) = rx[it];
        }
    };

    // every request of the prologue is issued before the first result is waited for, in the order of use
    load_set(ra, rs_w7, 0);
    load_x(0);
    constexpr int PRM_ITERS = 4 * CH / 256;
    float pv[PRM_ITERS];
#pragma unroll
    for (int it = 0; it < PRM_ITERS; ++it) {
        const float* src = it == 0 ? p.b7 : it == 1 ? p.a2 : it == 2 ? p.ib2 : p.b1;      // 256 threads, 256 channels
        pv[it] = src[tid];
    }
    store_a(0);
    store_x();
#pragma unroll
    for (int it = 0; it < PRM_ITERS; ++it) prm[it * CH + tid] = pv[it];
    __syncthreads();

    // accumulators start at the bias: lane (j, h) holds rows (channels) mi*32 + 8g + 4h + {0..3} of column j
    f32x16 acc[TM];
    auto init_acc = [&](int which) __attribute__((always_inline)) {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 b4 = *reinterpret_cast<const float4*>(&prm[which * CH + mi * 32 + 8 * g + 4 * h]);
                acc[mi][4 * g + 0] = b4.x; acc[mi][4 * g + 1] = b4.y; acc[mi][4 * g + 2] = b4.z; acc[mi][4 * g + 3] = b4.w;
            }
    };
    init_acc(0);

    // ---- dilated conv: K loop over (chunk, tap) stages, fixed order; the last stage is peeled, its shadow hides the
    // fetch of the first block of the 1x1 weights
    int chunk = 0, tap = 0;
    auto mma_stage = [&](int stage) __attribute__((always_inline)) {
        __builtin_amdgcn_s_setprio(1);
        const int off = p.tap0 + tap * p.tap_step - minoff;
        const uint16_t* abase = &As[(stage & 1) * CH * LDK + j * LDK + h * 8];
        const uint16_t* xbase = &Xs[(wn * 32 + j + off) * LDK + h * 8];
        // The stage's 16 MFMAs in the order (k-step, row tile), each weight fragment requested three MFMAs before it is used
        // (four fragment registers in rotation).  Left to itself the compiler reads the first k-step's fragments one at a time
        // into one register set, and each of those MFMAs waits out the full LDS latency of its read.
        static_assert(KC == 32 && TM == 8, "two k-steps of eight row tiles");
        auto afrag = [&](int i) __attribute__((always_inline)) {
            return *reinterpret_cast<const bf16x8*>(abase + (i & 7) * 32 * LDK + (i >> 3) * 16);
        };
        const bf16x8 b0 = *reinterpret_cast<const bf16x8*>(xbase);
        const bf16x8 b1 = *reinterpret_cast<const bf16x8*>(xbase + 16);
        bf16x8 a[4];
        a[0] = afrag(0); a[1] = afrag(1); a[2] = afrag(2);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (i + 3 < 16) a[(i + 3) & 3] = afrag(i + 3);
            acc[i & 7] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i & 3], (i >> 3) ? b1 : b0, acc[i & 7], 0, 0, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);            // b0, b1, three fragments, the fourth
#pragma unroll
        for (int i = 0; i < 12; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
        __builtin_amdgcn_s_setprio(0);
    };
    // Weight blocks are requested two stages ahead, alternating between the two register sets (the second set is otherwise
    // only used by the 1x1 convolution): with one workgroup per CU (a single playback window) nothing else hides the
    // latency of a block's load, and one stage of MFMAs is shorter than it.  The request is unconditional: behind a
    // branch the compiler could not count it, and the wait for the older block would wait for it as well.  In place of the block
    // past the last one the first block of the 1x1 weights is requested.
    auto iter = [&](int stage, u32x4 (&rload)[A_ITERS], const u32x4 (&rstore)[A_ITERS], __amdgpu_buffer_rsrc_t rs, int block) __attribute__((always_inline)) {
        int ntap = tap + 1, nchunk = chunk;
        if (ntap == p.ntaps) { ntap = 0; ++nchunk; }
        const bool new_chunk = nchunk != chunk;
        load_set(rload, rs, block);
        if (new_chunk) load_x(nchunk);
        mma_stage(stage);
        if (new_chunk) {
            __syncthreads();
            store_x();
        }
        store_set(rstore, (stage + 1) & 1);
        __syncthreads();
        tap = ntap; chunk = nchunk;
    };
    load_set(rb, rs_w7, 1);
    static_assert(W_NCHUNKS % 2 == 0, "an even number of stages");
    for (int stage = 0; stage + 2 < nstages; stage += 2) {
        iter(stage, ra, rb, rs_w7, stage + 2);
        iter(stage + 1, rb, ra, rs_w7, stage + 3);
    }
    iter(nstages - 2, ra, rb, rs_w1, 0);
    mma_stage(nstages - 1);

    // ---- Snake on the accumulators; repack them as the B fragments of the 1x1 conv (k step kk = 2 mi + g/2)
    u32x4 mid[CH / 16];
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int c = mi * 32 + 8 * g + 4 * h;
            const float4 a4 = *reinterpret_cast<const float4*>(&prm[CH + c]);
            const float4 i4 = *reinterpret_cast<const float4*>(&prm[2 * CH + c]);
            u32x4& f = mid[2 * mi + g / 2];
            f[2 * (g & 1) + 0] = pack_bf16x2(snake_fast(acc[mi][4 * g + 0], a4.x, i4.x), snake_fast(acc[mi][4 * g + 1], a4.y, i4.y));
            f[2 * (g & 1) + 1] = pack_bf16x2(snake_fast(acc[mi][4 * g + 2], a4.z, i4.z), snake_fast(acc[mi][4 * g + 3], a4.w, i4.w));
        }

    // ---- 1x1 conv: K = 256 channels straight from registers, weights streamed through the two weight buffers; block
    // c + 2 is requested before block c is used (odd blocks travel in ra, even ones in rb).  The residual values of
    // the epilogue are requested in the second half of the loop, where the fragments already used have freed registers.
    __syncthreads();                                   // all waves are done with the last stage's operands
    store_a(0);
    load_set(ra, rs_w1, 1);
    load_set(rb, rs_w1, 2);
    // accumulator tile mo of the 1x1 conv: [time row 8g + 4h + q][channel slot j] = channel 8 j + mo; starts at its bias
#pragma unroll
    for (int mo = 0; mo < TM; ++mo) {
        const float b1v = prm[3 * CH + j * TM + mo];
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[mo][q] = b1v;
    }
    __syncthreads();
    u32x4 resv[16];                                    // 8 halves: the lane's channels of time row gq
    auto row_offset = [&](int gq) -> unsigned {
        return (unsigned)((n0 + wn * 32 + 8 * (gq >> 2) + 4 * h + (gq & 3)) * CH + j * TM) * 2u;
    };
#pragma unroll
    for (int c = 0; c < W_NCHUNKS; ++c) {
        const uint16_t* abase = &As[(c & 1) * CH * LDK + j * LDK + h * 8];
#pragma unroll
        for (int mo = 0; mo < TM; ++mo) {
            const bf16x8 a0 = *reinterpret_cast<const bf16x8*>(abase + mo * 32 * LDK);
            const bf16x8 a1 = *reinterpret_cast<const bf16x8*>(abase + mo * 32 * LDK + 16);
            acc[mo] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, mid[2 * c]), a0, acc[mo], 0, 0, 0);
            acc[mo] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, mid[2 * c + 1]), a1, acc[mo], 0, 0, 0);
        }
        if (c + 1 < W_NCHUNKS) {
            if ((c + 1) & 1) store_set(ra, (c + 1) & 1); else store_set(rb, (c + 1) & 1);
            __syncthreads();
            if (c + 3 < W_NCHUNKS) { if ((c + 3) & 1) load_set(ra, rs_w1, c + 3); else load_set(rb, rs_w1, c + 3); }
        }
        if (c >= W_NCHUNKS / 2) {                      // chunks 4..7 request four time rows each
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int gq = (c - W_NCHUNKS / 2) * 4 + q;
                resv[gq] = __builtin_amdgcn_raw_buffer_load_b128(rs_y, row_offset(gq), 0, 0);
            }
        }
    }
    static_assert(W_NCHUNKS / 2 * 4 == 16, "four time rows per chunk of the second half");

    // ---- residual add, half store in place, optional Snake + bf16 operand for the next layer, straight from the
    // accumulators.  Rows past out_hi are outside the descriptors and dropped.
    float a3v[TM], i3v[TM];
#pragma unroll
    for (int mo = 0; mo < TM; ++mo) {
        a3v[mo] = EMIT ? p.a3[j * TM + mo] : 0.f;
        i3v[mo] = EMIT ? p.ib3[j * TM + mo] : 0.f;
    }
#pragma unroll
    for (int gq = 0; gq < 16; ++gq) {
        const unsigned off = row_offset(gq);
        const f16x8 r = __builtin_bit_cast(f16x8, resv[gq]);
        f16x8 o;
#pragma unroll
        for (int mo = 0; mo < TM; ++mo) o[mo] = (_Float16)keep_f32(acc[mo][gq] + (float)r[mo]);     // fp32 sum, then one rounding
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), rs_ys, off, 0, 0);
        if (EMIT) {
            // the next layer's operand is Snake of the STORED value
            u32x4 sh;
#pragma unroll
            for (int mo = 0; mo < TM; mo += 2)
                sh[mo / 2] = pack_bf16x2(snake_fast((float)o[mo], a3v[mo], i3v[mo]), snake_fast((float)o[mo + 1], a3v[mo + 1], i3v[mo + 1]));
            __builtin_amdgcn_raw_buffer_store_b128(sh, rs_a, off, 0, 0);
        }
    }
}

// The same unit with the weights streamed to registers, for launches of few tiles: 8 waves share the 16 TN columns of a tile, a wave
// owning 32 channels of all of them.  The staged kernel above lasts as long as one workgroup's
// walk over its 64 weight blocks, whatever the launch's size (45 us: two barriers a block, every wave reading all 16 KB of it
// from LDS).  Here a CU reads each weight once, RS k-steps ahead and without a barrier, and the branch tensor goes through LDS
// (its fragments are spread over the waves); what bounds it is the 16 KB of weights a k-step brings into the CU for narrow tiles
// (some 45 bytes per clock) and the MFMAs for wide ones.  Per unit of a window of 8 frames 45 -> 22 us, of 75 frames 51 -> 27.
// K order (chunk of 32 channels, tap, channel; the 1x1 conv's k-slots) and roundings are those of the kernel above: the
// results are bit-identical, whichever kernel a launch takes.
template <int TN, bool EMIT>
__global__ __launch_bounds__(512, 2) void res_unit_wide_stream_kernel(WideParams p)
{
    fp16_saturate_on();
    constexpr int CH = W_CH, NT = 16 * TN, NTAPS = 7, NTH = 512;
    constexpr int KX = 64, LDR = KX + 16;                   // stage of two chunks; rows 10 pieces apart: no bank conflicts
    constexpr int SEGS = KX / 8, RPP = NTH / SEGS, X_ITERS = (NT + W_MAXSPAN + RPP - 1) / RPP, XR = X_ITERS * RPP;
    constexpr int F = 2 * NTAPS, NSTAGES = CH / KX;         // k-steps of 32 in a stage
    constexpr int RS = 7;                     // k-steps of weights in flight
    static_assert(F % RS == 0 && RS * (W_A_CH * 16u) <= kWeightSlack, "static ring indices");
    constexpr int LDM = CH + 16;                            // row of the branch tensor's tile: 34 pieces
    constexpr int LDO = CH + 4;                             // row of the fp32 output tile
    constexpr int X_BYTES = XR * LDR * 2, M_BYTES = NT * LDM * 2, O_BYTES = NT * LDO * 4;
    constexpr int SMEM_XM = 2 * X_BYTES > M_BYTES ? 2 * X_BYTES : M_BYTES, SMEM = SMEM_XM > O_BYTES ? SMEM_XM : O_BYTES;
    __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM];

    const Slot s = p.slots[blockIdx.y];
    const int nrows = s.len * p.r;
    const int out_lo = max(0, s.crop * p.r - p.margin);
    const int out_hi = min(nrows, (s.crop + s.n_int) * p.r + p.margin);
    const int tiles8 = (int)(gridDim.x >> 3);               // XCD x takes a contiguous eighth of the tiles, as above
    const int n0 = out_lo + ((int)((blockIdx.x + blockIdx.y) & 7u) * tiles8 + (int)(blockIdx.x >> 3)) * NT;
    if (n0 >= out_hi) return;
    const long long rowbase = (long long)s.row0 * p.r;
    const int minoff = p.tap0, need = NT + (NTAPS - 1) * p.tap_step;         // tap_step > 0

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = lane & 15, q = lane >> 4;
    const int seg = tid % SEGS, xr0 = tid / SEGS;

    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(p.xa + rowbase * CH, (unsigned)nrows * CH * 2u);
    const __amdgpu_buffer_rsrc_t rs_y = make_rsrc(p.y + rowbase * CH, (unsigned)out_hi * CH * (unsigned)sizeof(hres_t));
    const __amdgpu_buffer_rsrc_t rs_ys = make_rsrc(p.y + rowbase * CH, EMIT && p.y_dead ? 0u : (unsigned)out_hi * CH * (unsigned)sizeof(hres_t));
    const __amdgpu_buffer_rsrc_t rs_a = make_rsrc(p.ya + rowbase * CH, EMIT ? (unsigned)out_hi * CH * 2u : 0u);
    const __amdgpu_buffer_rsrc_t rs_w7 = weight_rsrc(p.w7, (unsigned)(W_NCHUNKS * NTAPS) * (W_A_CH * 16u));
    const __amdgpu_buffer_rsrc_t rs_w1 = weight_rsrc(p.w1, (unsigned)W_NCHUNKS * (W_A_CH * 16u));

    // weights: one block of 256 x 32 per k-step, [16-row unit][lane][8]; this wave's units are 2 wave, 2 wave + 1
    const unsigned w_voff = (unsigned)wave * 2048u + lane * 16u;
    u32x4 a[RS][2];
    auto load_a = [&](int f, int slot, unsigned voff) __attribute__((always_inline)) {
        const unsigned blk = (unsigned)f * (W_A_CH * 16u);
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) a[slot][mi] = __builtin_amdgcn_raw_buffer_load_b128(rs_w7, voff + mi * 1024u, blk, 0);
    };
    // 1x1 weights: channel 8 j + mo lies in slot 32 mo + j (see pack_w1_wide); this lane's channel 16 u + i in unit u
    auto load_a1 = [&](int c, int slot) __attribute__((always_inline)) {
        const unsigned blk = (unsigned)c * (W_A_CH * 16u);
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) {
            const int ch = 32 * wave + 16 * mi + i, sl = (ch & 7) * 32 + (ch >> 3);
            a[slot][mi] = __builtin_amdgcn_raw_buffer_load_b128(rs_w1, (unsigned)((sl >> 4) * 1024 + (q * 16 + (sl & 15)) * 16), blk, 0);
        }
    };

    const unsigned x_voff = ((unsigned)((n0 + minoff + xr0) * CH) + seg * 8u) * 2u;      // may wrap "negative": out of range
    u32x4 rx[X_ITERS];
    auto load_x = [&](int stage) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < X_ITERS; ++it) {
            // rows no tap reads and stages past the last: out of range
            const bool used = stage < NSTAGES && it * RPP < need;
            rx[it] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, used ? x_voff + (unsigned)(it * RPP * CH + stage * KX) * 2u : 0xf8000000u, 0, 0);
        }
    };
    auto store_x = [&](int buf) __attribute__((always_inline)) {
        uint16_t* xs = reinterpret_cast<uint16_t*>(smem + buf * X_BYTES);
#pragma unroll
        for (int it = 0; it < X_ITERS; ++it) *reinterpret_cast<u32x4*>(&xs[(xr0 + it * RPP) * LDR + seg * 8]) = rx[it];
    };

    load_x(0);
#pragma unroll
    for (int f = 0; f < RS; ++f) load_a(f, f, w_voff);
    const int ch0 = 32 * wave + i;                          // this lane's channels: ch0, ch0 + 16
    f32x4 acc[2][TN];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi) {
        const float b = p.b7[ch0 + 16 * mi];
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = f32x4{b, b, b, b};
    }
    store_x(0);
    __syncthreads();

    // activations are the row operand: register e of accumulator (mi, ni) is column 16 ni + 4 q + e, channel ch0 + 16 mi
    auto mma = [&](const u32x4& x, const u32x4 (&w)[2], int ni) __attribute__((always_inline)) {
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, w[mi]), acc[mi][ni], 0, 0, 0);
    };
    for (int stage = 0; stage < NSTAGES; ++stage) {
        load_x(stage + 1);
        const unsigned voff_next = ahead_voff(w_voff, stage + 1 < NSTAGES);
        const uint16_t* xs = reinterpret_cast<const uint16_t*>(smem + (stage & 1) * X_BYTES) + i * LDR + q * 8;
        u32x4 x[2][TN];
        auto read_x = [&](int f, int ni) __attribute__((always_inline)) {
            x[f & 1][ni] = *reinterpret_cast<const u32x4*>(xs + (16 * ni + f % NTAPS * p.tap_step) * LDR + f / NTAPS * 32);
        };
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) read_x(0, ni);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < F; ++f) {
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) {
                if (f + 1 < F) read_x(f + 1, ni);
                mma(x[f & 1][ni], a[f % RS], ni);
                __builtin_amdgcn_sched_barrier(0);
            }
            load_a(stage * F + f + RS, f % RS, f + RS < F ? w_voff : voff_next);
            __builtin_amdgcn_sched_barrier(0);
        }
        store_x((stage + 1) & 1);
        __syncthreads();
    }

    // ---- Snake on the accumulators; the branch tensor goes to LDS as [column][k-slot], where the 8 k-slots of a piece are the
    // channels 32 c + 16 (q / 2) + 4 (q % 2) + {0..3, 8..11} of the 1x1 weights' K axis
#pragma unroll
    for (int f = 0; f < RS; ++f) load_a1(f, f);
    uint16_t* ms = reinterpret_cast<uint16_t*>(smem);
#pragma unroll
    for (int mi = 0; mi < 2; ++mi) {
        const float al = p.a2[ch0 + 16 * mi], ib = p.ib2[ch0 + 16 * mi], b = p.b1[ch0 + 16 * mi];
        const int slot = 32 * wave + 16 * mi + 8 * ((i >> 2) & 1) + 4 * (i >> 3) + (i & 3);
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) {
#pragma unroll
            for (int e = 0; e < 4; ++e) ms[(16 * ni + 4 * q + e) * LDM + slot] = f32_to_bf16_bits(snake_fast(acc[mi][ni][e], al, ib));
            acc[mi][ni] = f32x4{b, b, b, b};
        }
    }
    __syncthreads();

    // ---- 1x1 conv
    const uint16_t* mr = ms + i * LDM + q * 8;
#pragma unroll
    for (int c = 0; c < W_NCHUNKS; ++c) {
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) mma(*reinterpret_cast<const u32x4*>(mr + 16 * ni * LDM + 32 * c), a[c % RS], ni);
        if (c + RS < W_NCHUNKS) load_a1(c + RS, c % RS);
    }

    // ---- residual add, half store in place, optional Snake + bf16 operand, 8 channels of a column at a time through LDS
    constexpr int PPR = CH / 8, ERPP = NTH / PPR, E_ITERS = NT / ERPP;
    const int ec = tid % PPR * 8, er = tid / PPR;
    float a3v[8], i3v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) { a3v[e] = EMIT ? p.a3[ec + e] : 0.f; i3v[e] = EMIT ? p.ib3[ec + e] : 0.f; }
    float* os = reinterpret_cast<float*>(smem);
    u32x4 resv[E_ITERS];
#pragma unroll
    for (int it = 0; it < E_ITERS; ++it) resv[it] = __builtin_amdgcn_raw_buffer_load_b128(rs_y, (unsigned)((n0 + er + it * ERPP) * CH + ec) * 2u, 0, 0);
    __syncthreads();                                        // the branch tensor has been read
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
#pragma unroll
            for (int e = 0; e < 4; ++e) os[(16 * ni + 4 * q + e) * LDO + ch0 + 16 * mi] = acc[mi][ni][e];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < E_ITERS; ++it) {
        // rows past out_hi are outside the descriptors and dropped
        const unsigned off = (unsigned)((n0 + er + it * ERPP) * CH + ec) * 2u;
        const float* src = &os[(er + it * ERPP) * LDO + ec];
        const f16x8 r = __builtin_bit_cast(f16x8, resv[it]);
        f16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (_Float16)keep_f32(src[e] + (float)r[e]);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), rs_ys, off, 0, 0);
        if (EMIT) {
            u32x4 sh;
#pragma unroll
            for (int e = 0; e < 8; e += 2)
                sh[e / 2] = pack_bf16x2(snake_fast((float)o[e], a3v[e], i3v[e]), snake_fast((float)o[e + 1], a3v[e + 1], i3v[e + 1]));
            __builtin_amdgcn_raw_buffer_store_b128(sh, rs_a, off, 0, 0);
        }
    }
}

// The same unit for launches that fill the chip: 4 waves share a tile of 128 columns, a wave owning 64 channels of all of them, two
// workgroups on a CU (256 registers, 70 KB of LDS).  What bound the staged kernel is LDS reads: a wave of 256 channels x 32 columns
// reads 9 KB per 256 cycles of MFMAs, four of them more than the LDS delivers, with two barriers per weight block on top.  64 channels x 128
// columns need 4 KB of streamed weights and 8 KB of LDS reads per 512 cycles of MFMAs, a third of what either path delivers, and
// one barrier per 14 k-steps; the next stage's activations travel two rows of a thread at a time, so that
// accumulators (128 registers), four k-steps of weights (64) and the fragments read ahead fit without spills.
// The dilated conv has the weights as the row operand (a lane ends with four consecutive channels of a column: 8-byte LDS writes of
// the branch tensor), the 1x1 conv the activations (a lane ends with four channels of a row, 16 lanes with 128 bytes: the
// epilogue goes straight to memory).  In calls that are waited for, 60 s clip 389 -> 317 us per unit (1.19 PFLOP/s; HBM traffic and Snake included),
// 375 frames 111 -> 80, encode of 60 s 438 -> 363.  The 1x1 conv goes before the K loop of the other workgroup (s_setprio 2 and 1: 310 -> 307 us; 1 in the
// K loop alone: none).  Bit-identical to the kernels above.
template <bool EMIT>
__global__ __launch_bounds__(256, 2) void res_unit_wide_tall_kernel(WideParams p)
{
    fp16_saturate_on();
    constexpr int CH = W_CH, TM = 4, TN = 8, NT = 16 * TN, NTAPS = 7, NTH = 256;
    constexpr int KX = 64, LDR = KX + 16;                   // stage of two chunks; rows 10 pieces apart: no bank conflicts
    constexpr int SEGS = KX / 8, RPP = NTH / SEGS, X_ITERS = (NT + W_MAXSPAN) / RPP, XR = X_ITERS * RPP;
    constexpr int F = 2 * NTAPS, NSTAGES = CH / KX;         // k-steps of 32 in a stage
    constexpr int RS = 4;                                   // k-steps of weights in flight
    constexpr int XA = 5, XQ = XA + 1;                      // activation fragments read ahead of their MFMAs
    constexpr int LDM = CH + 16;                            // row of the branch tensor's tile: 34 pieces
    constexpr int X_BYTES = XR * LDR * 2, M_BYTES = NT * LDM * 2;
    constexpr int SMEM = 2 * X_BYTES > M_BYTES ? 2 * X_BYTES : M_BYTES;
    static_assert(XR == NT + W_MAXSPAN && X_ITERS == 6 && NSTAGES % 2 == 0 && 2 * F % RS == 0 && W_NCHUNKS % RS == 0, "static indices");
    __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM];

    const Slot s = p.slots[blockIdx.y];
    const int nrows = s.len * p.r;
    const int out_lo = max(0, s.crop * p.r - p.margin);
    const int out_hi = min(nrows, (s.crop + s.n_int) * p.r + p.margin);
    const int tiles8 = (int)(gridDim.x >> 3);               // XCD x takes a contiguous eighth of the tiles, as above
    const int n0 = out_lo + ((int)((blockIdx.x + blockIdx.y) & 7u) * tiles8 + (int)(blockIdx.x >> 3)) * NT;
    if (n0 >= out_hi) return;
    const long long rowbase = (long long)s.row0 * p.r;
    const int minoff = p.tap0;                              // tap_step > 0

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = lane & 15, q = lane >> 4;
    const int seg = tid % SEGS, xr0 = tid / SEGS;

    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(p.xa + rowbase * CH, (unsigned)nrows * CH * 2u);
    const __amdgpu_buffer_rsrc_t rs_y = make_rsrc(p.y + rowbase * CH, (unsigned)out_hi * CH * (unsigned)sizeof(hres_t));
    const __amdgpu_buffer_rsrc_t rs_ys = make_rsrc(p.y + rowbase * CH, EMIT && p.y_dead ? 0u : (unsigned)out_hi * CH * (unsigned)sizeof(hres_t));
    const __amdgpu_buffer_rsrc_t rs_a = make_rsrc(p.ya + rowbase * CH, EMIT ? (unsigned)out_hi * CH * 2u : 0u);
    const __amdgpu_buffer_rsrc_t rs_w7 = weight_rsrc(p.w7, (unsigned)(W_NCHUNKS * NTAPS) * (W_A_CH * 16u));
    const __amdgpu_buffer_rsrc_t rs_w1 = weight_rsrc(p.w1, (unsigned)W_NCHUNKS * (W_A_CH * 16u));

    // weights: one block of 256 x 32 per k-step, [16-row unit][lane][8]; this wave's units are 4 wave .. 4 wave + 3
    const unsigned w_voff = (unsigned)wave * (TM * 1024u) + lane * 16u;
    u32x4 a[RS][TM];
    auto load_a = [&](int f) __attribute__((always_inline)) {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi) a[f % RS][mi] = __builtin_amdgcn_raw_buffer_load_b128(rs_w7, w_voff + mi * 1024u, (unsigned)f * (W_A_CH * 16u), 0);
    };
    // 1x1 weights: lane i of unit mi is channel 64 wave + 4 i + mi, which lies in slot 32 (channel % 8) + channel / 8 (pack_w1_wide)
    const unsigned w1_voff = (unsigned)((8 * (i & 1) + (wave >> 1)) * 1024 + (8 * (wave & 1) + (i >> 1)) * 16 + q * 256);
    auto load_a1 = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi) a[c % RS][mi] = __builtin_amdgcn_raw_buffer_load_b128(rs_w1, w1_voff, (unsigned)c * (W_A_CH * 16u) + mi * 2048u, 0);
    };

    const unsigned x_voff = ((unsigned)((n0 + minoff + xr0) * CH) + seg * 8u) * 2u;      // may wrap "negative": out of range
    u32x4 rx[X_ITERS];
    auto load_x = [&](int stage, int it) __attribute__((always_inline)) {
        rx[it] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, x_voff + (unsigned)(it * RPP * CH + stage * KX) * 2u, 0, 0);
    };
    auto store_x = [&](int buf, int it) __attribute__((always_inline)) {
        *reinterpret_cast<u32x4*>(smem + buf * X_BYTES + ((xr0 + it * RPP) * LDR + seg * 8) * 2) = rx[it];
    };

#pragma unroll
    for (int it = 0; it < X_ITERS; ++it) load_x(0, it);
#pragma unroll
    for (int f = 0; f < RS; ++f) load_a(f);
    f32x4 acc[TM][TN];
    const int ch0 = 64 * wave + 4 * q;                      // dilated conv: register e of (mi, ni) is channel ch0 + 16 mi + e, column 16 ni + i
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) {
        const f32x4 b = *reinterpret_cast<const f32x4*>(p.b7 + ch0 + 16 * mi);
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = b;
    }
#pragma unroll
    for (int it = 0; it < X_ITERS; ++it) store_x(0, it);
    __syncthreads();

    __builtin_amdgcn_s_setprio(1);                          // waves in this loop go first, those in the 1x1 conv before them
    const int tap_bytes = p.tap_step * (LDR * 2);
    auto run_stage = [&](int stage, int half, auto last) __attribute__((always_inline)) {
        constexpr bool LAST = decltype(last)::value;
        // LDS offset of the tap that is read, kept as one running register (left to itself the compiler holds one for every tap)
        unsigned at = half * X_BYTES + (i * LDR + q * 8) * 2;
        u32x4 x[XQ];
        auto read_x = [&](int t) __attribute__((always_inline)) {
            const int f = t / TN, ni = t % TN;
            if (t > 0 && ni == 0) {
                at = f % NTAPS == 0 ? at - (NTAPS - 1) * tap_bytes + 64 : at + tap_bytes;
                asm volatile("" : "+v"(at));
            }
            x[t % XQ] = *reinterpret_cast<const u32x4*>(smem + at + 16 * ni * LDR * 2);
        };
#pragma unroll
        for (int t = 0; t < XA; ++t) read_x(t);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < F; ++f) {
            // the next stage's activations, two rows of a thread at a time
            if (!LAST || half == 0) {
                if (f >= 4 && f % 4 == 0) { store_x(half ^ 1, f / 2 - 2); store_x(half ^ 1, f / 2 - 1); }
                if (f % 4 == 0 && f < 12) { load_x(stage + 1, f / 2); load_x(stage + 1, f / 2 + 1); }
            }
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) {
                const int t = f * TN + ni;
                if (t + XA < F * TN) read_x(t + XA);
#pragma unroll
                for (int mi = 0; mi < TM; ++mi)
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[(half * F + f) % RS][mi]), __builtin_bit_cast(bf16x8, x[t % XQ]), acc[mi][ni], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            // k-steps past the last are the first ones of the 1x1 conv
            if (LAST && half == 1 && f + RS >= F) load_a1(f + RS - F);
            else {
                const unsigned blk = (unsigned)(stage * F + f + RS) * (W_A_CH * 16u);
#pragma unroll
                for (int mi = 0; mi < TM; ++mi) a[(half * F + f) % RS][mi] = __builtin_amdgcn_raw_buffer_load_b128(rs_w7, w_voff + mi * 1024u, blk, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
    };
    for (int stage = 0; stage + 2 < NSTAGES; stage += 2) {
        run_stage(stage, 0, std::false_type{});
        run_stage(stage + 1, 1, std::false_type{});
    }
    run_stage(NSTAGES - 2, 0, std::true_type{});
    run_stage(NSTAGES - 1, 1, std::true_type{});
    __builtin_amdgcn_s_setprio(0);

    // ---- Snake on the accumulators; the branch tensor goes to LDS as [column][k-slot]: channel 16 m + 4 q + e of a group of 32 is
    // k-slot 16 m + 8 (q % 2) + 4 (q / 2) + e of the 1x1 weights' K axis
    uint16_t* ms = reinterpret_cast<uint16_t*>(smem);
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) {
        const f32x4 al = *reinterpret_cast<const f32x4*>(p.a2 + ch0 + 16 * mi), ib = *reinterpret_cast<const f32x4*>(p.ib2 + ch0 + 16 * mi);
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) {
            const f32x4 v = acc[mi][ni];
            u32x2 o;
            o[0] = pack_bf16x2(snake_fast(v[0], al[0], ib[0]), snake_fast(v[1], al[1], ib[1]));
            o[1] = pack_bf16x2(snake_fast(v[2], al[2], ib[2]), snake_fast(v[3], al[3], ib[3]));
            *reinterpret_cast<u32x2*>(&ms[(16 * ni + i) * LDM + 64 * wave + 16 * mi + 8 * (q & 1) + 4 * (q >> 1)]) = o;
        }
    }
    // ---- 1x1 conv, activations as the row operand: register e of (mi, ni) is column 16 ni + 4 q + e, channel 64 wave + 4 i + mi, so
    // that a lane holds four consecutive channels of a column and 16 lanes 128 bytes of it
    const int ec = 64 * wave + 4 * i;
    const f32x4 b1v = *reinterpret_cast<const f32x4*>(p.b1 + ec);
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = f32x4{b1v[mi], b1v[mi], b1v[mi], b1v[mi]};
    __syncthreads();

    u32x2 resv[TN][4];
    unsigned e_voff = (unsigned)((n0 + 4 * q) * CH + ec) * 2u;
    // residual values, requested into the registers that the weights of the 1x1 conv's last k-steps free
    auto load_res = [&](int ni) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) resv[ni][e] = __builtin_amdgcn_raw_buffer_load_b64(rs_y, e_voff + (unsigned)((16 * ni + e) * CH * 2), 0, 0);
    };
    {
        __builtin_amdgcn_s_setprio(2);
        const uint16_t* mr = ms + i * LDM + q * 8;
        constexpr int XA = 3, XQ = XA + 1;
        u32x4 x[XQ];
        auto read_x = [&](int t) __attribute__((always_inline)) { x[t % XQ] = *reinterpret_cast<const u32x4*>(mr + (t % TN) * 16 * LDM + (t / TN) * 32); };
#pragma unroll
        for (int t = 0; t < XA; ++t) read_x(t);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < W_NCHUNKS; ++c) {
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) {
                const int t = c * TN + ni;
                if (t + XA < W_NCHUNKS * TN) read_x(t + XA);
#pragma unroll
                for (int mi = 0; mi < TM; ++mi)
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x[t % XQ]), __builtin_bit_cast(bf16x8, a[c % RS][mi]), acc[mi][ni], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (c + RS < W_NCHUNKS) load_a1(c + RS);
            else if (c + RS > W_NCHUNKS) { load_res(2 * (c + RS - W_NCHUNKS) - 2); load_res(2 * (c + RS - W_NCHUNKS) - 1); }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __builtin_amdgcn_s_setprio(0);
    load_res(TN - 2);
    load_res(TN - 1);
    asm volatile("" : "+v"(e_voff));                        // the 32 offsets are formed again, not kept

    // ---- residual add, half store in place, optional Snake + bf16 operand for the next layer.  Rows past out_hi are outside the
    // descriptors and dropped.
    f32x4 a3v = {0.f, 0.f, 0.f, 0.f}, i3v = {0.f, 0.f, 0.f, 0.f};
    if (EMIT) { a3v = *reinterpret_cast<const f32x4*>(p.a3 + ec); i3v = *reinterpret_cast<const f32x4*>(p.ib3 + ec); }
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned off = e_voff + (unsigned)((16 * ni + e) * CH * 2);
            const f16x4 r = __builtin_bit_cast(f16x4, resv[ni][e]);
            f16x4 o;
#pragma unroll
            for (int mi = 0; mi < TM; ++mi) o[mi] = (_Float16)keep_f32(acc[mi][ni][e] + (float)r[mi]);     // fp32 sum, then one rounding
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, o), rs_ys, off, 0, 0);
            if (EMIT) {
                // the next layer's operand is Snake of the STORED value
                u32x2 sh;
                sh[0] = pack_bf16x2(snake_fast((float)o[0], a3v[0], i3v[0]), snake_fast((float)o[1], a3v[1], i3v[1]));
                sh[1] = pack_bf16x2(snake_fast((float)o[2], a3v[2], i3v[2]), snake_fast((float)o[3], a3v[3], i3v[3]));
                __builtin_amdgcn_raw_buffer_store_b64(sh, rs_a, off, 0, 0);
            }
        }
    }
}

}  // namespace

// W1 [256][256] -> 8 blocks of 256 row slots x 32 k-slots, the K axis in the accumulator row order of the narrow fused
// unit, the rows in the order of the swapped-role accumulator tiles
void pack_w1_wide(const float* w, uint16_t* dst)
{
    for (int c = 0; c < W_NCHUNKS; ++c)
        for (int slot = 0; slot < W_CH; ++slot) {
            const int o = (slot % 32) * W_TM + slot / 32;          // row slot (mo, j) holds output channel 8 j + mo
            for (int e = 0; e < W_KC; ++e) {
                const int kp = c * W_KC + e, kk = kp / 16, h = (kp / 8) % 2, q = kp % 8;
                const int ch = 32 * (kk / 2) + 8 * (2 * (kk % 2) + q / 4) + 4 * h + q % 4;
                dst[((size_t)c * W_CH + slot) * W_KC + e] = f32_to_bf16_rne(w[(size_t)o * W_CH + ch]);
            }
        }
}

hipError_t launch_res_unit_wide(const WideArgs& a, hipStream_t stream)
{
    WideParams p;
    p.xa = a.xa; p.y = (hres_t*)a.y; p.y_dead = a.y_dead; p.ya = a.ya; p.w7 = a.w7; p.w1 = a.w1; p.b7 = a.b7; p.b1 = a.b1;
    p.a2 = a.a2; p.ib2 = a.ib2; p.a3 = a.a3; p.ib3 = a.ib3;
    p.slots = a.slots; p.r = a.r; p.ntaps = a.ntaps;
    p.tap0 = -((a.ntaps - 1) / 2) * a.dil; p.tap_step = a.dil; p.margin = a.margin;
    if (a.c != W_CH || a.ntaps < 1 || (a.ntaps - 1) * a.dil > W_MAXSPAN || a.margin < 0 || !a.xa || !a.y || a.xa == a.ya) return hipErrorInvalidValue;
    if (a.ya ? !a.a3 || !a.ib3 : a.y_dead) return hipErrorInvalidValue;
    // one window's activation plane must fit a 32-bit byte offset (buffer descriptors)
    if ((long long)a.max_len * a.r * a.c * 2 > 0xf0000000ll) return hipErrorInvalidValue;
    const long long out_rows = std::min((long long)a.max_int * a.r + 2ll * a.margin, (long long)a.max_len * a.r);
    auto tiles = [&](int nt) { return (out_rows + nt - 1) / nt; };
    auto grid = [&](int nt) { return dim3((unsigned)(tiles(nt) + 7) / 8 * 8, (unsigned)a.n_slots); };     // whole groups of 8 tiles; the surplus exits at once
    // Seven taps: the narrow streamed tiles run one workgroup of 8 waves per CU, and a launch takes the narrowest one that fits the 256
    // CUs; larger launches take the tall kernel, two workgroups of 4 waves per CU.  Per unit in us, columns 32, 64, 80, 96 in one round (two
    // rounds in brackets) / tall: 13 frames 18, 21, 23, 26 / 28; 40 frames (30), 22, 24, 27 / 29; 75 frames (44), (39), 28, 29 / 31; 110 frames
    // (55), (40), (46), (52) / 33; 150 frames (70), (59), (50), (55) / 49; four windows of 64 frames 3 rounds and more: 109, 81, 94, 82 / 58.
    // Against the LDS-staged kernel: 375 frames 111 -> 80, 60 s clip 389 -> 317.
    const bool streamed = a.ntaps == 7 && !a.staged_only;
#define DEMON_STREAM(TN) \
    if (streamed && tiles(16 * TN) * a.call_slots <= 256) { \
        if (a.ya) hipLaunchKernelGGL((res_unit_wide_stream_kernel<TN, true>), grid(16 * TN), dim3(512), 0, stream, p); \
        else hipLaunchKernelGGL((res_unit_wide_stream_kernel<TN, false>), grid(16 * TN), dim3(512), 0, stream, p); \
        return hipGetLastError(); \
    }
    DEMON_STREAM(2) DEMON_STREAM(4) DEMON_STREAM(5) DEMON_STREAM(6)
#undef DEMON_STREAM
    if (streamed) {
        if (a.ya) hipLaunchKernelGGL((res_unit_wide_tall_kernel<true>), grid(W_NT), dim3(256), 0, stream, p);
        else hipLaunchKernelGGL((res_unit_wide_tall_kernel<false>), grid(W_NT), dim3(256), 0, stream, p);
        return hipGetLastError();
    }
    if (a.ya) hipLaunchKernelGGL((res_unit_wide_kernel<true>), grid(W_NT), dim3(256), 0, stream, p);
    else hipLaunchKernelGGL((res_unit_wide_kernel<false>), grid(W_NT), dim3(256), 0, stream, p);
    return hipGetLastError();
}

}  // namespace demon
