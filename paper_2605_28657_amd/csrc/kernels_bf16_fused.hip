// Fused residual unit for the narrow, high-rate levels (C = 64 or 128 channels):
//     h_out = h + W1 * snake2(W7 (*) snake1(h) + b7) + b1
// in one kernel, so that the activated branch tensor never goes to HBM.  Two kernels: the LDS-staged one, first below, for kernel
// sizes other than 7, and the streamed one.
//
// LDS-staged: the dilated conv runs as in kernels_bf16.hip (implicit GEMM, rows = output channels, columns = time,
// one weight block in LDS, the next waiting in registers), except that the kernel reads the half-precision residual stream itself and
// applies Snake while staging (cheaper in HBM traffic than a separate bf16 operand at these rates),
// and that every wave owns ALL C rows of its 32*TN columns.  A lane of a 32x32 MFMA accumulator tile
// holds column j and rows 8g + 4h + {0..3}; the B operand of the next MFMA wants, for the same column
// j, eight K values per lane.  So after bias + Snake the accumulators ARE the B fragments of the 1x1
// conv, provided its K axis is permuted to the accumulator's row order: k-slot (kk, h, e) <-> channel
// 32 (kk/2) + 8 (2 (kk%2) + e/4) + 4 h + e%4.  The 1x1 weights are packed in that order at create.
// In the 1x1 conv the roles are swapped: these fragments are the row operand (rows = time) and the weights the
// column operand, so its accumulator tile is [time][output channel] and a lane holds one output-channel slot j of
// each of the C/32 channel tiles.  The weight rows are packed so that slot j of tile mo is channel j C/32 + mo:
// a lane then owns C/32 consecutive channels of a time row, 32 lanes a whole row, and residual loads and
// stores are contiguous without a transposition through LDS.
// The result is written to a second buffer (neighbouring tiles still read this tile's input rows).
// With EMIT the kernel also writes bf16(snake_next(h_out)), the operand of the next (unfused) layer.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "device_common.h"

namespace demon {

constexpr int FUSED_MAXSPAN = 64;
constexpr int FUSED_MAXSPAN7 = FUSED_MAXSPAN / 6 * 6;      // of seven taps

struct FusedParams {
    const hres_t* x; hres_t* y;  // EMIT: y may be nullptr, nothing after the unit reads the residual stream
    uint16_t* ya;                // optional activated bf16 copy of y (EMIT)
    const uint16_t* w7;          // [chunk][tap] blocks of C x 64 bf16
    const uint16_t* w1;          // [C][C] bf16, K axis permuted (see above)
    const float* b7; const float* b1;
    const float* a1; const float* ib1;    // Snake on the input (alpha in revolutions, 1/(beta+eps))
    const float* a2; const float* ib2;    // Snake between the two convolutions
    const float* a3; const float* ib3;    // Snake of the consumer (EMIT)
    const Slot* slots;
    int r, ntaps, tap0, tap_step, nchunks, margin;
    // HEAD: the decoder's head (Snake -> Conv1d(hk) -> tanh) on this unit's output, in the same kernel
    const uint16_t* hw;          // half-precision MFMA fragments of the head weights (pack_head_mfma)
    const float* hb; const float* ha; const float* hib;
    HeadOut out;
    int oc, hk;
};

// channel that k-slot kp (0..C-1) of the permuted 1x1 weight matrix multiplies
static inline int fused_k_to_channel(int kp)
{
    const int kk = kp / 16, h = (kp / 8) % 2, e = kp % 8;
    return 32 * (kk / 2) + 8 * (2 * (kk % 2) + e / 4) + 4 * h + e % 4;
}

void pack_w1_fused(const float* w /*[C][C]*/, int C, uint16_t* dst)
{
    const int tm = C / 32;
    for (int slot = 0; slot < C; ++slot) {
        const int o = (slot % 32) * tm + slot / 32;        // row slot (mo, j) holds output channel j * tm + mo
        for (int kp = 0; kp < C; ++kp) dst[(size_t)slot * C + kp] = f32_to_bf16_rne(w[(size_t)o * C + fused_k_to_channel(kp)]);
    }
}

// HEAD (64 channels, no EMIT): the unit is the decoder's last layer before the head.  Its output rows do not go to memory:
// Snake with the head's parameters, rounded to half, they fill an LDS tile (the activation tile's space, free after the K
// loop), the head's weight fragments take the weight buffer, and every wave runs the head's k x 4 k-steps on its 64
// columns exactly as head_mfma_kernel does (same operands, same order: the same bits).  A tile's head outputs need the
// unit's outputs (k-1)/2 columns to both sides, so tiles advance by NT - (k-1) columns and the first and last (k-1)/2
// columns of a tile only serve as context.  Saves the unit's 128-byte-per-row store, the head's read of it and a launch.
constexpr int FUSED_HEAD_MAXK = 7;      // k x 64 weight pieces of 16 bytes travel in two registers per thread

template <int CH, int TN, bool EMIT, bool HEAD = false>
__global__ __launch_bounds__(256, (CH == 128 && TN == 2) ? 2 : 3) void res_unit_fused_kernel(FusedParams p)
{
    static_assert(!HEAD || (CH == 64 && !EMIT), "the head follows a 64-channel unit that feeds nothing else");
    fp16_saturate_on();
    constexpr int KC = 64;
    constexpr int LDK = KC + 8;
    constexpr int NT = 4 * 32 * TN;               // four waves side by side in time
    constexpr int WTN = 32 * TN;
    constexpr int XR_MAX = NT + FUSED_MAXSPAN;
    constexpr int TM = CH / 32;
    constexpr int SEGS = KC / 8;
    constexpr int RPP = 256 / SEGS;
    constexpr int A_CH = CH * SEGS;
    constexpr int A_ITERS = A_CH / 256;
    constexpr int X_ITERS = (XR_MAX + RPP - 1) / RPP;
    constexpr int LD1 = CH + 8;                   // padded row of the 1x1 weight tile
    constexpr int W1_CH = CH * CH / 8;            // 16-byte chunks of the 1x1 weights
    static_assert(A_CH % 256 == 0 && W1_CH % 256 == 0, "staging loops assume whole passes");
    // 64 channels: LDS and registers are budgeted for three workgroups per CU (they hide each other's barriers and latencies
    // markedly better than two).  128 channels: two workgroups per CU with twice the columns per wave (TN = 2, 128
    // accumulator registers): 0.75 instead of 1.25 fragment reads per MFMA, half the weight staging and a quarter less
    // halo per column; per launch the same time as three workgroups of 128 columns, per step 1 % less (less LDS traffic
    // under the power limit).  Its residual values are requested after the 1x1 conv (no registers before).
    // Common to both: one weight buffer (the next block waits in registers and is stored between two
    // barriers), an activation tile without row padding (16-byte pieces XOR-swizzled by the row instead), the 1x1
    // weights and the residual values requested after the K loop.
    constexpr int LDX = KC;                       // unpadded row of the activation tile; piece sg of row r sits at sg ^ (r & 7)
    constexpr int AS_BYTES = CH * LDK * 2, XS_BYTES = XR_MAX * LDX * 2;
    constexpr int SMEM_BYTES = AS_BYTES + XS_BYTES;
    static_assert(CH * LD1 * 2 <= SMEM_BYTES, "the 1x1 weights reuse the buffers of the dilated conv");
    __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM_BYTES];
    // per-channel vectors used after the K loop (bias of both convolutions, Snake between them): read from global
    // memory where they are used, each load would be waited for in turn
    __shared__ __attribute__((aligned(16))) float prm[4 * CH];     // b7 | a2 | ib2 | b1
    uint16_t* As = reinterpret_cast<uint16_t*>(smem);
    uint16_t* Xs = reinterpret_cast<uint16_t*>(smem + AS_BYTES);

    const Slot s = p.slots[blockIdx.y];
    const int nrows = __builtin_amdgcn_readfirstlane(s.len * p.r);        // (the descriptors must be scalar)
    const int out_lo = max(0, s.crop * p.r - p.margin);
    const int out_hi = min(nrows, (s.crop + s.n_int) * p.r + p.margin);
    // Workgroups are dealt to the 8 XCDs round-robin by linear id, and each XCD has its own L2: XCD x takes a contiguous
    // eighth of a window's tiles, in order, so that neighbouring tiles (which share their halo rows) run on the same
    // XCD at about the same time.  The eighths rotate with the window index (the last one may be short).
    const int tiles8 = (int)(gridDim.x >> 3);
    const int tile = (int)((blockIdx.x + blockIdx.y) & 7u) * tiles8 + (int)(blockIdx.x >> 3);
    const int hhalf = HEAD ? (p.hk - 1) / 2 : 0;
    // HEAD: the unit's columns start (k-1)/2 before the interior also at a clip edge (rows before the window are zero)
    const int n0 = HEAD ? s.crop * p.r - hhalf + tile * (NT - 2 * hhalf) : out_lo + tile * NT;
    const int h_lo = s.crop * p.r, h_hi = (s.crop + s.n_int) * p.r;     // HEAD: the interior rows the head produces
    if (HEAD ? (n0 + hhalf >= h_hi) : (n0 >= out_hi)) return;
    const long long rowbase = (long long)__builtin_amdgcn_readfirstlane(s.row0) * p.r;

    const int last_off = p.tap0 + (p.ntaps - 1) * p.tap_step;
    const int minoff = min(p.tap0, last_off);
    const int XR = NT + max(p.tap0, last_off) - minoff;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wn = tid >> 6;
    const int j = lane & 31, h = lane >> 5;
    const int seg = tid % SEGS, xr0 = tid / SEGS;

    // descriptors: one window of the input, the computed part of the window for the outputs
    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(p.x + rowbase * CH, (unsigned)nrows * CH * (unsigned)sizeof(hres_t));
    const __amdgpu_buffer_rsrc_t rs_y = make_rsrc(p.y + rowbase * CH, EMIT && !p.y ? 0u : (unsigned)out_hi * CH * (unsigned)sizeof(hres_t));
    const __amdgpu_buffer_rsrc_t rs_a = make_rsrc(p.ya + rowbase * CH, EMIT ? (unsigned)out_hi * CH * 2u : 0u);
    const __amdgpu_buffer_rsrc_t rs_w = weight_rsrc(p.w7, (unsigned)(p.nchunks * p.ntaps) * (A_CH * 16u));

    const int nstages = p.nchunks * p.ntaps;
    const unsigned a_voff = tid * 16u;
    const unsigned x_voff = ((unsigned)((n0 + minoff + xr0) * CH) + seg * 8u) * (unsigned)sizeof(hres_t);   // may wrap "negative": out of range
    constexpr unsigned x_row_step = RPP * CH * (unsigned)sizeof(hres_t);

    u32x4 ra[A_ITERS];
    u32x4 rx[X_ITERS];           // 8 channels of one row (half)
    float al[8], ib[8];

    auto load_a = [&](int stage) __attribute__((always_inline)) {
        const unsigned base = (unsigned)stage * (A_CH * 16u);
#pragma unroll
        for (int it = 0; it < A_ITERS; ++it) ra[it] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, a_voff, base + it * 4096u, 0);
    };
    auto store_a = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < A_ITERS; ++it) {
            const int q = tid + it * 256;
            *reinterpret_cast<u32x4*>(&As[frag_row<KC>(q) * LDK + frag_piece<KC>(q) * 8]) = ra[it];
        }
    };
    auto load_x = [&](int chunk) __attribute__((always_inline)) {
        const unsigned coff = x_voff + (unsigned)(chunk * KC) * (unsigned)sizeof(hres_t);
#pragma unroll
        for (int it = 0; it < X_ITERS; ++it) {
            if (it * RPP >= XR) break;                        // uniform
            rx[it] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, coff + it * x_row_step, 0, 0);
        }
        const int cbase = chunk * KC + seg * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) { al[e] = p.a1[cbase + e]; ib[e] = p.ib1[cbase + e]; }
    };
    auto store_x = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < X_ITERS; ++it) {
            if (it * RPP >= XR) break;                        // uniform
            const int xr = xr0 + it * RPP;
            if (xr >= XR_MAX) continue;
            u32x4 v;
            const f16x8 hv = __builtin_bit_cast(f16x8, rx[it]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[q] = pack_bf16x2(snake_fast_half(hv[2 * q], al[2 * q], ib[2 * q]), snake_fast_half(hv[2 * q + 1], al[2 * q + 1], ib[2 * q + 1]));
            }
            *reinterpret_cast<u32x4*>(&Xs[xr * LDX + ((seg ^ (xr & 7)) * 8)]) = v;
        }
    };

    u32x4 rw1[W1_CH / 256];      // the 1x1 weights on their way to LDS
    auto load_w1 = [&]() __attribute__((always_inline)) {
        const u32x4* src = reinterpret_cast<const u32x4*>(p.w1);
#pragma unroll
        for (int it = 0; it < W1_CH / 256; ++it) rw1[it] = src[tid + it * 256];
    };

    // every request of the prologue is issued before the first result is waited for, in the order of use
    load_a(0);
    load_x(0);
    constexpr int PRM_ITERS = 4 * CH / 256;
    float pv[PRM_ITERS];
#pragma unroll
    for (int it = 0; it < PRM_ITERS; ++it) {
        const int i = tid + it * 256, which = i / CH, c = i % CH;
        const float* src = which == 0 ? p.b7 : which == 1 ? p.a2 : which == 2 ? p.ib2 : p.b1;
        pv[it] = src[c];
    }
    // The residual values this lane adds in the epilogue are requested in one go after the K loop, in the shadow of the
    // Snake and the 1x1 convolution: loaded where they are used, each would be waited for in turn, a chain of memory
    // latencies per tile (and held through the K loop they cost the registers of the third workgroup).
    // epilogue geometry: lane (j, h) owns channels j TM .. j TM + TM - 1 of time rows 8g + 4h + q of every 32-column tile
    using res_t = std::conditional_t<TM == 2, uint32_t, u32x2>;         // TM halves
    res_t resv[TN][16];
    auto res_offset = [&](int ni, int gq) -> unsigned {
        const int col = n0 + wn * WTN + ni * 32 + 8 * (gq >> 2) + 4 * h + (gq & 3);
        return (unsigned)(col * CH + j * TM) * 2u;
    };
    auto load_res = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
#pragma unroll
            for (int gq = 0; gq < 16; ++gq) {
                if constexpr (TM == 2) resv[ni][gq] = __builtin_amdgcn_raw_buffer_load_b32(rs_x, res_offset(ni, gq), 0, 0);
                else resv[ni][gq] = __builtin_amdgcn_raw_buffer_load_b64(rs_x, res_offset(ni, gq), 0, 0);
            }
    };
    store_a();
    store_x();
#pragma unroll
    for (int it = 0; it < PRM_ITERS; ++it) prm[tid + it * 256] = pv[it];
    __syncthreads();

    // accumulators start at the bias: lane (j, h) holds rows (channels) mi*32 + 8g + 4h + {0..3}
    f32x16 acc[TM][TN];
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 b4 = *reinterpret_cast<const float4*>(&prm[mi * 32 + 8 * g + 4 * h]);
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) {
                acc[mi][ni][4 * g + 0] = b4.x; acc[mi][ni][4 * g + 1] = b4.y;
                acc[mi][ni][4 * g + 2] = b4.z; acc[mi][ni][4 * g + 3] = b4.w;
            }
        }

    // ---- dilated conv: K loop over (chunk, tap) stages, fixed order
    int chunk = 0, tap = 0;
    for (int stage = 0; stage < nstages; ++stage) {
        int ntap = tap + 1, nchunk = chunk;
        if (ntap == p.ntaps) { ntap = 0; ++nchunk; }
        const bool more = stage + 1 < nstages;
        const bool new_chunk = more && nchunk != chunk;
        if (more) load_a(stage + 1);
        if (new_chunk) load_x(nchunk);

        const int off = p.tap0 + tap * p.tap_step - minoff;
        const uint16_t* abase = &As[j * LDK + h * 8];
        const int xrow = wn * WTN + j + off;                  // + ni * 32: the same row & 7
        const uint16_t* xbase = &Xs[xrow * LDX];
        const int r7 = xrow & 7;
#pragma unroll
        for (int ks = 0; ks < KC / 16; ++ks) {
            bf16x8 af[TM], bfr[TN];
#pragma unroll
            for (int mi = 0; mi < TM; ++mi) af[mi] = *reinterpret_cast<const bf16x8*>(abase + mi * 32 * LDK + ks * 16);
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) bfr[ni] = *reinterpret_cast<const bf16x8*>(xbase + ni * 32 * LDX + (((2 * ks + h) ^ r7) * 8));
#pragma unroll
            for (int mi = 0; mi < TM; ++mi)
#pragma unroll
                for (int ni = 0; ni < TN; ++ni)
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[mi], bfr[ni], acc[mi][ni], 0, 0, 0);
        }
        if constexpr (CH == 128) {
            // order of the stage's fragment reads and MFMAs: one k-step's reads plus two ahead, then one read per MFMA, so
            // that a fragment is requested a few MFMAs before it is used instead of right before the MFMAs of its own k-step
            // (the 64-channel form has no registers left for the fragments in flight)
            constexpr int R = (KC / 16) * (TM + TN), M = (KC / 16) * TM * TN;
            constexpr int LEAD = (TM + TN + 2) < R ? (TM + TN + 2) : R;
            constexpr int PAIRS = (R - LEAD) < M ? (R - LEAD) : M;
            __builtin_amdgcn_sched_group_barrier(0x100, LEAD, 0);
#pragma unroll
            for (int i = 0; i < PAIRS; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, M - PAIRS, 0);
        }
        if (more) {
            __syncthreads();                                  // every wave is done with the weight buffer (and the X tile)
            if (new_chunk) store_x();
            store_a();
            __syncthreads();
        }
        tap = ntap; chunk = nchunk;
    }
    constexpr bool RES_LAST = CH == 128 && TN == 2;     // no registers for the residual values until the 1x1 conv is done
    load_w1();
    if (!RES_LAST) load_res();

    // ---- bias + Snake on the accumulators; repack them as the B fragments of the 1x1 conv
    u32x4 mid[CH / 16][TN];      // bf16x8 fragments, built from packed pairs
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int c = mi * 32 + 8 * g + 4 * h;
            const float4 a4 = *reinterpret_cast<const float4*>(&prm[CH + c]);
            const float4 i4 = *reinterpret_cast<const float4*>(&prm[2 * CH + c]);
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) {
                const float v0 = snake_fast(acc[mi][ni][4 * g + 0], a4.x, i4.x);
                const float v1 = snake_fast(acc[mi][ni][4 * g + 1], a4.y, i4.y);
                const float v2 = snake_fast(acc[mi][ni][4 * g + 2], a4.z, i4.z);
                const float v3 = snake_fast(acc[mi][ni][4 * g + 3], a4.w, i4.w);
                u32x4& f = mid[2 * mi + g / 2][ni];
                f[2 * (g & 1) + 0] = pack_bf16x2(v0, v1);
                f[2 * (g & 1) + 1] = pack_bf16x2(v2, v3);
            }
        }
    }

    // ---- stage the 1x1 weights over the (now free) buffers of the dilated conv
    __syncthreads();                                   // all waves are done with the last stage's operands
#pragma unroll
    for (int it = 0; it < W1_CH / 256; ++it) {
        const int q = tid + it * 256;
        *reinterpret_cast<u32x4*>(&As[frag_row<CH>(q) * LD1 + frag_piece<CH>(q) * 8]) = rw1[it];
    }
    __syncthreads();

    // ---- 1x1 conv: K = C channels straight from registers, as the row operand (rows = time); the accumulator tile
    // [time][channel slot] starts at the bias of the lane's channel j TM + mo
#pragma unroll
    for (int mo = 0; mo < TM; ++mo) {
        const float b1v = prm[3 * CH + j * TM + mo];
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[mo][ni][q] = b1v;
    }
#pragma unroll
    for (int kk = 0; kk < CH / 16; ++kk) {
        bf16x8 af[TM];
#pragma unroll
        for (int mo = 0; mo < TM; ++mo) af[mo] = *reinterpret_cast<const bf16x8*>(&As[(mo * 32 + j) * LD1 + kk * 16 + h * 8]);
#pragma unroll
        for (int mo = 0; mo < TM; ++mo)
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
                acc[mo][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, mid[kk][ni]), af[mo], acc[mo][ni], 0, 0, 0);
    }

    if (RES_LAST) load_res();

    // ---- residual add and half store to the other buffer, straight from the accumulators: register 4g + q of tile
    // (mo, ni) is time row 8g + 4h + q, channel j TM + mo.  Rows past out_hi are outside the descriptors and dropped.
    float a3v[TM], i3v[TM];
#pragma unroll
    for (int mo = 0; mo < TM; ++mo) {
        a3v[mo] = EMIT ? p.a3[j * TM + mo] : 0.f;
        i3v[mo] = EMIT ? p.ib3[j * TM + mo] : 0.f;
    }
    const float one = opaque_one();
    // HEAD: the tile of head operands takes the activation tile's space (nothing reads that after the K loop; every wave
    // has passed the barriers that staged the 1x1 weights), rows shifted by (k-1)/2 so that a tap is a row offset >= 0
    constexpr int LDH = CH + 8;
    _Float16* Hs = reinterpret_cast<_Float16*>(smem + AS_BYTES);
    static_assert(!HEAD || (NT + FUSED_HEAD_MAXK - 1) * LDH * 2 <= XS_BYTES, "the head's operand tile fits the activation tile's space");
    float hav[TM], hiv[TM];
    u32x4 rhw[2];                 // the head's weight fragments on their way to LDS (at most 2 x 256 pieces of 16 bytes)
    const int n_hw = HEAD ? p.hk * (CH / 16) * 2 * 8 : 0;
    if constexpr (HEAD) {
#pragma unroll
        for (int mo = 0; mo < TM; ++mo) { hav[mo] = p.ha[j * TM + mo]; hiv[mo] = p.hib[j * TM + mo]; }
        const u32x4* src = reinterpret_cast<const u32x4*>(p.hw);          // [fragment][lane = h * 32 + channel][8 halves]
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int q = tid + it * 256;
            rhw[it] = q < n_hw ? src[(q / 8) * 32 + q % 8] : u32x4{0, 0, 0, 0};
        }
        // rows of the operand tile past the unit's columns (context of columns that are not produced): defined, unused
        for (int q = tid; q < 2 * hhalf * (CH / 2); q += 256) {
            const int rr = q / (CH / 2), cc = q % (CH / 2);
            const int row = rr < hhalf ? rr : NT + rr;
            *reinterpret_cast<uint32_t*>(&Hs[row * LDH + 2 * cc]) = 0u;
        }
    }
#pragma unroll
    for (int ni = 0; ni < TN; ++ni)
#pragma unroll
        for (int gq = 0; gq < 16; ++gq) {
            const unsigned off = res_offset(ni, gq);
            typedef _Float16 halfs_t __attribute__((ext_vector_type(TM)));
            const halfs_t r = __builtin_bit_cast(halfs_t, resv[ni][gq]);
            static_assert(sizeof(halfs_t) == sizeof(res_t), "TM halves");
            halfs_t o;
#pragma unroll
            for (int mo = 0; mo < TM; ++mo) {
                o[mo] = (_Float16)keep_f32(add_half(acc[mo][ni][gq], r[mo], one));       // fp32 sum, then one rounding
            }
            if constexpr (HEAD) {
                // the head's operand: Snake of the (half) value the unit would have stored, in fp32, rounded once to half;
                // rows outside the window are the head conv's zero padding
                const int col = wn * WTN + ni * 32 + 8 * (gq >> 2) + 4 * h + (gq & 3);
                const int n = n0 + col;
                f16x2 av = {(_Float16)0.f, (_Float16)0.f};
                if (n >= 0 && n < nrows) {
                    av[0] = (_Float16)keep_f32(snake_fast_half(o[0], hav[0], hiv[0]));
                    av[1] = (_Float16)keep_f32(snake_fast_half(o[1], hav[1], hiv[1]));
                }
                *reinterpret_cast<f16x2*>(&Hs[(col + hhalf) * LDH + j * TM]) = av;
                continue;
            }
            if constexpr (TM == 2) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, o), rs_y, off, 0, 2);
            else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, o), rs_y, off, 0, 2);
            if (EMIT) {
                // the next layer's operand is Snake of the STORED value
                uint32_t sh[TM / 2];
#pragma unroll
                for (int mo = 0; mo < TM; mo += 2) {
                    const float e0 = snake_fast_half(o[mo], a3v[mo], i3v[mo]);
                    const float e1 = snake_fast_half(o[mo + 1], a3v[mo + 1], i3v[mo + 1]);
                    sh[mo / 2] = pack_bf16x2(e0, e1);
                }
                if constexpr (TM == 2) __builtin_amdgcn_raw_buffer_store_b32(sh[0], rs_a, off, 0, 2);
                else { const u32x2 s2 = {sh[0], sh[1]}; __builtin_amdgcn_raw_buffer_store_b64(s2, rs_a, off, 0, 2); }
            }
        }
    if constexpr (HEAD) {
        // ---- the head on this tile: weights -> LDS (over the 1x1 weights), then per wave 2 column tiles x k taps x 4 k-steps
        uint16_t* Ws = reinterpret_cast<uint16_t*>(smem);          // [fragment][h][channel < 8][8 halves]
        __syncthreads();                                   // the operand tile is complete; nobody reads the 1x1 weights any more
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int q = tid + it * 256;
            if (q < n_hw) reinterpret_cast<u32x4*>(Ws)[q] = rhw[it];
        }
        __syncthreads();
        typedef _Float16 f16x8v __attribute__((ext_vector_type(8)));
        constexpr int KS = CH / 16;
        float hbv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) hbv[q] = (4 * h + q < p.oc) ? p.hb[4 * h + q] : 0.f;
        f32x16 hacc[2];
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int q = 0; q < 16; ++q) hacc[mi][q] = q < 4 ? hbv[q] : 0.f;
        for (int t = 0; t < p.hk; ++t) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                f16x8v bw = {0, 0, 0, 0, 0, 0, 0, 0};
                if (j < 8) bw = *reinterpret_cast<const f16x8v*>(&Ws[(((t * KS + ks) * 2 + h) * 8 + j) * 8]);
#pragma unroll
                for (int mi = 0; mi < 2; ++mi) {
                    const f16x8v av = *reinterpret_cast<const f16x8v*>(&Hs[(wn * WTN + mi * 32 + j + t) * LDH + ks * 16 + h * 8]);
                    // weights as the row operand: the accumulator tile is [output channel][time]
                    hacc[mi] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bw, av, hacc[mi], 0, 0, 0);
                }
            }
        }
        // lane (j, h) holds time column j and output channels 4 h + {0..3} in its first four registers
        const long long origin = head_origin(p.out, s, p.oc, p.r);
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) {
            const int col = wn * WTN + mi * 32 + j;
            const int n = n0 + col;
            if (col < hhalf || col >= NT - hhalf || n < h_lo || n >= h_hi) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int c = 4 * h + q;
                if (c < p.oc) p.out.y[c * p.out.plane + origin + n] = tanhf(hacc[mi][q]);
            }
        }
    }
}

// f(0), f(1), ... with the numbers as types: a loop of this many groups is past the compiler's limit for unrolling
template <int... I, typename Fn>
__device__ __forceinline__ void unrolled(std::integer_sequence<int, I...>, Fn&& f) { (f(std::integral_constant<int, I>{}), ...); }

// The same unit with the weights streamed to registers (seven taps): WM x WN waves, a wave owning 16 TM channels x 16 TN columns, the
// branch tensor through LDS.  What bound the kernel above: two barriers per 8 or 16 KB weight block (a launch of few tiles lasts as long as
// one workgroup's 14 of them), and at 128 channels LDS reads (6 KB per wave and 256 cycles of MFMAs).  Here a stage of 64 channels has all its taps
// between two barriers and the next stage's Snake runs in the shadow of its MFMAs, a quarter row every other group of TM MFMAs.
// Times: a launch with an event after it in a call that is waited for (4 to 5 us of each are the events; in back-to-back steps at the power
// limit the 128-channel units of a 60 s clip take 376 to 399 us on one stream).
//  * 128 channels, large calls: 64 x 128 per wave, 2 x 2 waves, two workgroups per CU (256 registers, 80 KB): a third of the LDS reads.
//    What bounds it now is the two waves of a SIMD: matrix cores busy 50 %, other VALU work (Snake of 1.25 + 1 values per output) 30 %,
//    which overlap in part.  Waves in the K loop go first (s_setprio: -5 %), those in the 1x1 conv before them: at the default priority its 2 k
//    cycles of MFMAs took 9 of a workgroup's 60 k beside the other's K loop (366 -> 346 us; at the loop's own priority 343, and calls the same within
//    0.1 %: 60 s clip 4808 to 4818 us in eight runs of either).
//    60 s clip 428 -> 346 us per unit (with the operand 458 -> 366), 375 frames 104 to 121 -> 89 to 98.
//  * 128 channels, few tiles: 32 x 64 per wave, 4 x 1 waves: window of 13 frames 25 -> 11 us, 75 frames 36 -> 27.
//  * 64 channels: one stage, two by two waves of 32 channels: 13 frames 13 -> 9 us (with the head 19 -> 11), 75 frames 20 -> 17 (28 -> 23),
//    375 frames 62 -> 55.
// K order: (64 channels, tap, channel), as above: the results are the bits of the kernel above.  At 128 channels and 256 columns two stages
// of 64 channels take all of the LDS that two workgroups per CU leave one (rows without padding, the late vectors in a tile that has been
// read).  Stages of 32 channels with padded rows are 0.4 % faster (60 s clip 5401 us, 5424 with these), but another order of the sums:
// another 4.5e-4 of every decode, 2.8e-3 of every encode.
template <int TM, int TN, int WM, int WN, int OCC, bool EMIT, bool HEAD>
__global__ __launch_bounds__(64 * WM * WN, OCC) void res_unit_narrow_stream_kernel(FusedParams p)
{
    fp16_saturate_on();
    constexpr int CH = 16 * TM * WM, NT = 16 * TN * WN, NTAPS = 7, NTH = 64 * WM * WN, KX = 64;
    constexpr bool TIGHT = TM * TN > 24;                    // accumulators take half of the registers, activation tiles half of the LDS
    // stage of KX channels.  Rows 10 pieces apart: no bank conflicts; TIGHT: rows of 8 pieces, piece sg of row r at sg ^ (r & 7)
    constexpr int LDR = TIGHT ? KX : KX + 16;
    constexpr int SEGS = KX / 8, RPP = NTH / SEGS, ROWS = NT + FUSED_MAXSPAN7, X_ITERS = (ROWS + RPP - 1) / RPP, XR = TIGHT ? ROWS : X_ITERS * RPP;
    constexpr int NSTAGES = CH / KX, SX = KX / 32, F = NTAPS * SX, NSTEPS = NSTAGES * F, KS1 = CH / 32;
    constexpr int RS = TIGHT ? 4 : 7;                       // k-steps of weights in flight
    constexpr int XA = TIGHT ? 3 : 5, XQ = XA + 1;          // activation fragments read ahead of their MFMAs
    constexpr int RX = TIGHT ? 2 : X_ITERS;                 // rows of a thread requested ahead
    constexpr int G = F * TN;                               // groups of TM MFMAs in a stage
    constexpr int LDM = CH + 16;
    // per-channel vectors in LDS: (a1, ib1) pairs | b7 | a2 | ib2 | b1 | a3 | ib3 (of the consumer or the head).  TIGHT: the pairs; the vectors
    // from a2 on come in front of the branch tensor during the last stage, where nothing reads the first stage's tile any more
    constexpr int PRM = TIGHT ? 2 * CH : (EMIT || HEAD ? 8 : 6) * CH, M_OFF = TIGHT ? (EMIT ? 5 : 3) * CH * 4 : 0;
    constexpr int X_BYTES = XR * LDR * 2, M_BYTES = M_OFF + NT * LDM * 2;
    constexpr int XS_BYTES = NSTAGES * X_BYTES, SMEM = XS_BYTES > M_BYTES ? XS_BYTES : M_BYTES;
    constexpr unsigned BLOCK = CH * 128u;                   // bytes of a weight block: CH rows x 64 channels
    constexpr int PW = G / X_ITERS, PD = PW >= 8 ? 2 : 1;   // groups a staged row lasts, groups between its quarters
    constexpr int AUX = TIGHT ? 2 : 0;                      // stores of large calls pass the caches by
    // HEAD: weight fragments, then the tile of operands, in the activation tile's space
    constexpr int LDH = CH + 8, HW_BYTES = FUSED_HEAD_MAXK * CH * 16, HW_ITERS = HEAD ? (HW_BYTES / 16 + NTH - 1) / NTH : 1;
    static_assert(!HEAD || (CH == 64 && !EMIT && NT % (32 * WM * WN) == 0 && HW_BYTES + (NT + FUSED_HEAD_MAXK - 1) * LDH * 2 <= SMEM), "the head follows a 64-channel unit that feeds nothing else");
    static_assert(KS1 <= RS && KS1 % TM == 0 && PW >= 4 && (NSTAGES == 1 || NSTAGES == 2), "static indices; a quarter row per group");
    static_assert(!TIGHT || (NSTAGES == 2 && NTH == 2 * CH && M_OFF <= X_BYTES), "vectors loaded by two threads a channel, over the first stage's tile");
    // TIGHT: what the last pass stages past a tile's rows falls on rows of the second tile that are staged later, or on the first stage's pairs,
    // which nothing reads (its Snake takes them from memory)
    static_assert(!TIGHT || (SMEM == XS_BYTES && (X_ITERS * RPP - XR) * LDR * 2 <= 2 * KX * 4), "rows past the second tile");
    static_assert(OCC * (SMEM + PRM * 4) <= 163840, "workgroups on a CU");
    __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM + PRM * 4];
    float* const prm = reinterpret_cast<float*>(smem + SMEM);
    float* const late = TIGHT ? reinterpret_cast<float*>(smem) : prm + 3 * CH;          // a2 | ib2 | b1 | a3 | ib3

    const Slot s = p.slots[blockIdx.y];
    const int nrows = __builtin_amdgcn_readfirstlane(s.len * p.r);        // (the descriptors must be scalar)
    const int out_lo = max(0, s.crop * p.r - p.margin);
    const int out_hi = min(nrows, (s.crop + s.n_int) * p.r + p.margin);
    const int tiles8 = (int)(gridDim.x >> 3);               // XCD x takes a contiguous eighth of the tiles, as above
    const int tile = (int)((blockIdx.x + blockIdx.y) & 7u) * tiles8 + (int)(blockIdx.x >> 3);
    const int hhalf = HEAD ? (p.hk - 1) / 2 : 0;
    const int h_lo = s.crop * p.r, h_hi = (s.crop + s.n_int) * p.r;     // HEAD: the interior rows the head produces
    const int n0 = HEAD ? h_lo - hhalf + tile * (NT - 2 * hhalf) : out_lo + tile * NT;
    if (HEAD ? n0 + hhalf >= h_hi : n0 >= out_hi) return;
    const long long rowbase = (long long)__builtin_amdgcn_readfirstlane(s.row0) * p.r;

    int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    int i = lane & 15, q = lane >> 4;
    const int seg = tid % SEGS, xr0 = tid / SEGS;

    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(p.x + rowbase * CH, (unsigned)nrows * CH * (unsigned)sizeof(hres_t));
    const __amdgpu_buffer_rsrc_t rs_y = make_rsrc(p.y + rowbase * CH, EMIT && !p.y ? 0u : (unsigned)out_hi * CH * (unsigned)sizeof(hres_t));
    const __amdgpu_buffer_rsrc_t rs_a = make_rsrc(p.ya + rowbase * CH, EMIT ? (unsigned)out_hi * CH * 2u : 0u);
    const __amdgpu_buffer_rsrc_t rs_w = weight_rsrc(p.w7, (unsigned)(CH / 64 * NTAPS) * BLOCK);
    const __amdgpu_buffer_rsrc_t rs_w1 = weight_rsrc(p.w1, CH * CH * 2u);

    // weights: blocks of CH x 64 in fragment order, [16-row unit][2 k-steps][lane][8]; this wave's units are TM wm .. TM wm + TM - 1
    const unsigned w_voff = (unsigned)wm * (TM * 2048u) + lane * 16u;
    u32x4 a[RS][TM];
    auto load_a = [&](int g) __attribute__((always_inline)) {              // k-step g: stage, tap, 32 channels of the stage
        const int c32 = g / F * SX + g % SX, tap = g % F / SX;
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
            a[g % RS][mi] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, w_voff, (unsigned)((c32 >> 1) * NTAPS + tap) * BLOCK + (c32 & 1) * 1024u + mi * 2048u, 0);
    };
    // 1x1 weights: lane i of unit mi is channel 16 TM wm + TM i + mi, which lies in slot 32 (channel % (CH / 32)) + channel / (CH / 32)
    auto load_a1 = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi) {
            // the slot of unit mi lies 32 mi after that of unit 0 (TM i and the wave's first channel are multiples of TM <= CH / 32)
            const int ch = 16 * TM * wm + TM * i, sl = ch % KS1 * 32 + ch / KS1;
            a[(NSTEPS + c) % RS][mi] = __builtin_amdgcn_raw_buffer_load_b128(rs_w1, (unsigned)((sl >> 4) * (KS1 * 1024) + q * 256 + (sl & 15) * 16), c * 1024u + mi * (2 * KS1 * 1024u), 0);
        }
    };

    // activations: row j of the staging (j = stage x X_ITERS + pass), 8 channels a thread
    const unsigned x_voff = ((unsigned)((n0 + p.tap0 + xr0) * CH) + seg * 8u) * 2u;      // may wrap "negative": out of range
    auto load_x = [&](int j) __attribute__((always_inline)) -> u32x4 {
        return __builtin_amdgcn_raw_buffer_load_b128(rs_x, x_voff + (unsigned)(j % X_ITERS * RPP * CH + j / X_ITERS * KX) * 2u, 0, 0);
    };
    auto put_x = [&](int j, u32x4 v) __attribute__((always_inline)) {
        const int row = (j / X_ITERS) * XR + xr0 + j % X_ITERS * RPP;                    // counted through both tiles
        *reinterpret_cast<u32x4*>(smem + (row * LDR + (TIGHT ? seg ^ (row & 7) : seg) * 8) * 2) = v;
    };
    auto read_prm = [&](int j, int k) __attribute__((always_inline)) -> f32x4 {          // Snake parameters of channels 2 k, 2 k + 1 of the thread's 8
        return *reinterpret_cast<const f32x4*>(&prm[(j / X_ITERS * KX + seg * 8 + 2 * k) * 2]);
    };
    auto snake2 = [&](uint32_t v, f32x4 pr) __attribute__((always_inline)) -> uint32_t {
        const f16x2 hv = __builtin_bit_cast(f16x2, v);
        return pack_bf16x2(snake_fast_half(hv[0], pr[0], pr[1]), snake_fast_half(hv[1], pr[2], pr[3]));
    };

    // every request of the prologue in the order of use
    // the last rows are those of the largest dilation (0.5 s window 215.2 -> 212.3 us, 3 s 463 -> 459; the units 3 to 8 % with dilations 1 and 3)
    const int rows_read = NT + (NTAPS - 1) * p.tap_step;
    auto staged = [&](int j) __attribute__((always_inline)) { return TIGHT || j < X_ITERS - 1 || j * RPP < rows_read; };
    u32x4 px[X_ITERS], rx[NSTAGES > 1 ? RX : 1];
#pragma unroll
    for (int j = 0; j < X_ITERS; ++j)
        if (staged(j)) px[j] = load_x(j);
    f32x4 pal[2], pib[2];                                    // Snake of the first stage's rows
#pragma unroll
    for (int k = 0; k < 2; ++k) { pal[k] = *reinterpret_cast<const f32x4*>(p.a1 + seg * 8 + 4 * k); pib[k] = *reinterpret_cast<const f32x4*>(p.ib1 + seg * 8 + 4 * k); }
    // per-channel vectors: the first CH threads take half of them, the next CH the others
    constexpr int NPV = EMIT || HEAD ? 4 : 3;
    const int ph = __builtin_amdgcn_readfirstlane(tid / CH), pc = tid % CH;
    const float* const psrc[4] = {ph ? p.a2 : p.a1, ph ? p.ib2 : p.ib1, ph ? p.b1 : p.b7, HEAD ? (ph ? p.hib : p.ha) : (ph ? p.ib3 : p.a3)};
    float pv[NPV];
    f32x4 b7v[TIGHT ? TM : 1];
    int ch0 = 16 * TM * wm + 4 * q;                         // dilated conv: register e of (mi, ni) is channel ch0 + 16 mi + e, column 16 ni + i
    if constexpr (TIGHT) {
        pv[0] = (ph ? p.ib1 : p.a1)[pc];
#pragma unroll
        for (int mi = 0; mi < TM; ++mi) b7v[mi] = *reinterpret_cast<const f32x4*>(p.b7 + ch0 + 16 * mi);
    } else {
#pragma unroll
        for (int k = 0; k < NPV; ++k) pv[k] = psrc[k][pc];
    }
#pragma unroll
    for (int g = 0; g < RS; ++g) load_a(g);
    if constexpr (NSTAGES > 1) {
#pragma unroll
        for (int j = 0; j < RX; ++j) rx[(X_ITERS + j) % RX] = load_x(X_ITERS + j);
    }
#pragma unroll
    for (int j = 0; j < X_ITERS; ++j) {
        if (!staged(j)) break;
        u32x4 v;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = snake2(px[j][k], f32x4{pal[k / 2][k % 2 * 2], pib[k / 2][k % 2 * 2], pal[k / 2][k % 2 * 2 + 1], pib[k / 2][k % 2 * 2 + 1]});
        put_x(j, v);
    }
    if constexpr (TIGHT) { if (pc >= KX) prm[2 * pc + ph] = pv[0]; }
    else {
        if (ph == 0) { prm[2 * pc] = pv[0]; prm[2 * pc + 1] = pv[1]; prm[2 * CH + pc] = pv[2]; }
        else if (ph == 1) { late[pc] = pv[0]; late[CH + pc] = pv[1]; late[2 * CH + pc] = pv[2]; }
        if (NPV == 4 && ph < 2) late[(3 + ph) * CH + pc] = pv[NPV - 1];
    }
    __syncthreads();
    f32x4 acc[TM][TN];
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) {
        const f32x4 b = TIGHT ? b7v[TIGHT ? mi : 0] : *reinterpret_cast<const f32x4*>(&prm[2 * CH + ch0 + 16 * mi]);
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = b;
    }

    // waves in this loop go first: the matrix cores are what the workgroups of a CU share (-5 % per unit)
    __builtin_amdgcn_s_setprio(1);
    const int tap_bytes = p.tap_step * (LDR * 2);
    auto run_stage = [&](auto stage) __attribute__((always_inline)) {
        constexpr int st = decltype(stage)::value;
        // LDS offset of the tap that is read, kept as one running register (left to itself the compiler holds one for every tap)
        unsigned at = st * X_BYTES + ((wn * (16 * TN) + i) * LDR + (TIGHT ? 0 : q * 8)) * 2;
        asm volatile("" : "+v"(at));
        u32x4 x[XQ];
        unsigned pos = 0;                                   // TIGHT: of the k-step's piece
        auto read_x = [&](int t) __attribute__((always_inline)) {
            if (t > 0 && t % (SX * TN) == 0) { at += tap_bytes; asm volatile("" : "+v"(at)); }
            if constexpr (TIGHT) {
                // piece q of the row (at / 128), its swizzle from the row's low bits; the k-step of the other 32 channels is 4 pieces on
                if (t % TN == 0) { pos = t / TN % SX ? pos ^ 64u : at + ((q * 16u) ^ (at >> 3 & 0x70u)); asm volatile("" : "+v"(pos)); }
                x[t % XQ] = *reinterpret_cast<const u32x4*>(smem + pos + 16 * (t % TN) * LDR * 2);
            } else
                x[t % XQ] = *reinterpret_cast<const u32x4*>(smem + at + (16 * (t % TN) * LDR + t / TN % SX * 32) * 2);
        };
        f32x4 pr = st + 1 < NSTAGES ? read_prm((st + 1) * X_ITERS, 0) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < XA; ++t) read_x(t);
        __builtin_amdgcn_sched_barrier(0);
        unrolled(std::make_integer_sequence<int, G>{}, [&](auto group) __attribute__((always_inline)) {
            constexpr int t = decltype(group)::value, ni = t % TN, g = st * F + t / TN;
            // the next stage's activations, in the shadow of the MFMAs: Snake on two values of a row, PD groups of MFMAs apart
            if constexpr (st + 1 < NSTAGES && t < X_ITERS * PW && t % PW >= PW - 1 - 3 * PD && (PW - 1 - t % PW) % PD == 0) {
                constexpr int it = t / PW, k = 3 - (PW - 1 - t % PW) / PD, j = (st + 1) * X_ITERS + it;
                rx[j % RX][k] = snake2(rx[j % RX][k], pr);
                if constexpr (k < 3) pr = read_prm(j, k + 1);
                else {
                    put_x(j, rx[j % RX]);
                    if constexpr (it + 1 < X_ITERS) pr = read_prm(j + 1, 0);
                    if constexpr (j + RX < NSTAGES * X_ITERS) rx[j % RX] = load_x(j + RX);
                }
            }
            if constexpr (TIGHT && st + 1 == NSTAGES) {
                // the vectors of the epilogue: requested here, stored two k-steps later (some twice: a branch would cut the schedule)
                if constexpr (t == 0) {
                    pv[0] = (ph ? p.ib2 : p.a2)[pc]; pv[1] = (ph ? EMIT ? p.ib3 : p.ib2 : p.b1)[pc];
                    if (EMIT) pv[2] = (ph ? p.ib3 : p.a3)[pc];
                }
                if constexpr (t == 2 * TN) {
                    late[ph * CH + pc] = pv[0]; late[(ph ? EMIT ? 4 : 1 : 2) * CH + pc] = pv[1];
                    if (EMIT) late[(ph ? 4 : 3) * CH + pc] = pv[2];
                }
            }
            if (t + XA < G) read_x(t + XA);
#pragma unroll
            for (int mi = 0; mi < TM; ++mi)
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[g % RS][mi]), __builtin_bit_cast(bf16x8, x[t % XQ]), acc[mi][ni], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (ni == TN - 1) {                             // k-steps past the last are those of the 1x1 conv
                if (g + RS < NSTEPS) load_a(g + RS);
                else if (g + RS < NSTEPS + KS1) load_a1(g + RS - NSTEPS);
                __builtin_amdgcn_sched_barrier(0);
            }
        });
        __syncthreads();
    };
    run_stage(std::integral_constant<int, 0>{});
    if constexpr (NSTAGES == 2) run_stage(std::integral_constant<int, 1>{});

    __builtin_amdgcn_s_setprio(0);
    // what the lane's number decides is formed again: nothing of it is held through the loop
    asm volatile("" : "+v"(tid));
    i = tid & 15; q = (tid >> 4) & 3; ch0 = 16 * TM * wm + 4 * q;

    // 1x1 conv, activations as the row operand: register e of (mi, ni) is column 16 ni + 4 q + e, channel 16 TM wm + TM i + mi, so that a
    // lane holds TM consecutive channels of a column and 16 lanes 16 TM of it
    const int ec = 16 * TM * wm + TM * i;
    unsigned e_voff = (unsigned)((n0 + wn * (16 * TN) + 4 * q) * CH + ec) * 2u;
    typedef _Float16 halfs_t __attribute__((ext_vector_type(TM)));
    using res_t = std::conditional_t<TM == 2, uint32_t, u32x2>;
    static_assert(sizeof(halfs_t) == sizeof(res_t), "TM halves");
    res_t resv[TN][4];
    auto load_res = [&](int ni) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned off = e_voff + (unsigned)((16 * ni + e) * CH * 2);
            if constexpr (TM == 2) resv[ni][e] = __builtin_amdgcn_raw_buffer_load_b32(rs_x, off, 0, 0);
            else resv[ni][e] = __builtin_amdgcn_raw_buffer_load_b64(rs_x, off, 0, 0);
        }
    };
    if (!TIGHT) {
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) load_res(ni);
    }

    // ---- Snake on the accumulators; the branch tensor goes to LDS as [column][k-slot]: channel 16 m + 4 q + e of a group of 32 is
    // k-slot 16 m + 8 (q % 2) + 4 (q / 2) + e of the 1x1 weights' K axis
    uint16_t* ms = reinterpret_cast<uint16_t*>(smem + M_OFF);
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) {
        const f32x4 al = *reinterpret_cast<const f32x4*>(&late[ch0 + 16 * mi]), ib = *reinterpret_cast<const f32x4*>(&late[CH + ch0 + 16 * mi]);
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) {
            const f32x4 v = acc[mi][ni];
            u32x2 o;
            o[0] = pack_bf16x2(snake_fast(v[0], al[0], ib[0]), snake_fast(v[1], al[1], ib[1]));
            o[1] = pack_bf16x2(snake_fast(v[2], al[2], ib[2]), snake_fast(v[3], al[3], ib[3]));
            *reinterpret_cast<u32x2*>(&ms[(wn * (16 * TN) + 16 * ni + i) * LDM + 16 * TM * wm + 16 * mi + 8 * (q & 1) + 4 * (q >> 1)]) = o;
        }
    }
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) {
        const float b = late[2 * CH + ec + mi];
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = f32x4{b, b, b, b};
    }
    __syncthreads();
    u32x4 rhw[HW_ITERS];                                    // HEAD: its weight fragments on their way to LDS, [fragment][h][channel < 8][8 halves]
    const int n_hw = HEAD ? p.hk * (CH / 16) * 2 * 8 : 0;
    if constexpr (HEAD) {
        const u32x4* src = reinterpret_cast<const u32x4*>(p.hw);          // [fragment][lane = h * 32 + channel][8 halves]
#pragma unroll
        for (int it = 0; it < HW_ITERS; ++it) {
            const int k = tid + it * NTH;
            rhw[it] = k < n_hw ? src[(k / 8) * 32 + k % 8] : u32x4{0, 0, 0, 0};
        }
    }
    {
        __builtin_amdgcn_s_setprio(2);                      // before the waves in the loop: a seventh of its MFMAs, and the workgroup is nearly done
        const uint16_t* mr = ms + (wn * (16 * TN) + i) * LDM + q * 8;
        constexpr int XA = 3, XQ = XA + 1;
        u32x4 x[XQ];
        auto read_x = [&](int t) __attribute__((always_inline)) { x[t % XQ] = *reinterpret_cast<const u32x4*>(mr + t % TN * 16 * LDM + t / TN * 32); };
#pragma unroll
        for (int t = 0; t < XA; ++t) read_x(t);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < KS1; ++c) {
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) {
                const int t = c * TN + ni;
                if (t + XA < KS1 * TN) read_x(t + XA);
#pragma unroll
                for (int mi = 0; mi < TM; ++mi)
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x[t % XQ]), __builtin_bit_cast(bf16x8, a[(NSTEPS + c) % RS][mi]), acc[mi][ni], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            // the registers of the weights hold the residual values now
            if (TIGHT && c > 0) { load_res(2 * c - 2); load_res(2 * c - 1); }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __builtin_amdgcn_s_setprio(0);
    if (TIGHT) {
#pragma unroll
        for (int ni = 2 * (KS1 - 1); ni < TN; ++ni) load_res(ni);
    }
    asm volatile("" : "+v"(e_voff));                        // the offsets are formed again, not kept

    const float one = opaque_one();
    float a3v[TM], i3v[TM];                                 // Snake of the consumer: the layer that takes the operand, or the head
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) {
        a3v[mi] = NPV == 4 ? late[(NPV == 4 ? 3 : 0) * CH + ec + mi] : 0.f;
        i3v[mi] = NPV == 4 ? late[(NPV == 4 ? 4 : 0) * CH + ec + mi] : 0.f;
    }
    // ---- residual add and half store to the other buffer.  Rows past out_hi are outside the descriptors and dropped.
    // HEAD: Snake of the (half) value the unit would have stored, in fp32, rounded once to half, goes to an LDS tile, rows shifted by
    // (k - 1) / 2 so that a tap is a row offset >= 0; rows outside the window are the head's zero padding
    uint16_t* Ws = reinterpret_cast<uint16_t*>(smem);
    _Float16* Hs = reinterpret_cast<_Float16*>(smem + HW_BYTES);
    if constexpr (HEAD) {
        __syncthreads();                                    // the branch tensor has been read
#pragma unroll
        for (int it = 0; it < HW_ITERS; ++it) {
            const int k = tid + it * NTH;
            if (k < n_hw) reinterpret_cast<u32x4*>(Ws)[k] = rhw[it];
        }
        // rows past the unit's columns (context of columns that are not produced): defined, unused
        for (int k = tid; k < 2 * hhalf * (CH / 2); k += NTH) {
            const int rr = k / (CH / 2), cc = k % (CH / 2);
            *reinterpret_cast<uint32_t*>(&Hs[(rr < hhalf ? rr : NT + rr) * LDH + 2 * cc]) = 0u;
        }
    }
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned off = e_voff + (unsigned)((16 * ni + e) * CH * 2);
            const halfs_t r = __builtin_bit_cast(halfs_t, resv[ni][e]);
            halfs_t o;
#pragma unroll
            for (int mi = 0; mi < TM; ++mi) o[mi] = (_Float16)keep_f32(add_half(acc[mi][ni][e], r[mi], one));     // fp32 sum, then one rounding
            if constexpr (HEAD) {
                const int col = wn * (16 * TN) + 16 * ni + 4 * q + e, n = n0 + col;
                const bool inside = n >= 0 && n < nrows;
#pragma unroll
                for (int mi = 0; mi < TM; ++mi) {
                    const _Float16 v = (_Float16)keep_f32(snake_fast_half(o[mi], a3v[mi], i3v[mi]));
                    o[mi] = inside ? v : (_Float16)0.f;
                }
                *reinterpret_cast<halfs_t*>(&Hs[(col + hhalf) * LDH + ec]) = o;
                continue;
            }
            if constexpr (TM == 2) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, o), rs_y, off, 0, AUX);
            else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, o), rs_y, off, 0, AUX);
            if (EMIT) {
                // the next layer's operand is Snake of the STORED value
                uint32_t sh[TM / 2];
#pragma unroll
                for (int mi = 0; mi < TM; mi += 2)
                    sh[mi / 2] = pack_bf16x2(snake_fast_half(o[mi], a3v[mi], i3v[mi]), snake_fast_half(o[mi + 1], a3v[mi + 1], i3v[mi + 1]));
                if constexpr (TM == 2) __builtin_amdgcn_raw_buffer_store_b32(sh[0], rs_a, off, 0, AUX);
                else { const u32x2 s2 = {sh[0], sh[1]}; __builtin_amdgcn_raw_buffer_store_b64(s2, rs_a, off, 0, AUX); }
            }
        }
    }
    if constexpr (HEAD) {
        // ---- the head on this tile, as in the kernel above: per wave NT / 128 tiles of 32 columns x k taps x 4 k-steps
        __syncthreads();
        constexpr int HT = NT / 32 / (WM * WN), KS = CH / 16;
        const int j = lane & 31, hh = lane >> 5;
        f32x16 hacc[HT];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const float hb = k < 4 && 4 * hh + k < p.oc ? p.hb[4 * hh + k] : 0.f;
#pragma unroll
            for (int mi = 0; mi < HT; ++mi) hacc[mi][k] = hb;
        }
        for (int t = 0; t < p.hk; ++t) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                f16x8 bw = {0, 0, 0, 0, 0, 0, 0, 0};
                if (j < 8) bw = *reinterpret_cast<const f16x8*>(&Ws[(((t * KS + ks) * 2 + hh) * 8 + j) * 8]);
#pragma unroll
                for (int mi = 0; mi < HT; ++mi) {
                    const f16x8 av = *reinterpret_cast<const f16x8*>(&Hs[((wave * HT + mi) * 32 + j + t) * LDH + ks * 16 + hh * 8]);
                    hacc[mi] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bw, av, hacc[mi], 0, 0, 0);
                }
            }
        }
        // lane (j, hh) holds time column j and output channels 4 hh + {0..3} in its first four registers
        const long long origin = head_origin(p.out, s, p.oc, p.r);
#pragma unroll
        for (int mi = 0; mi < HT; ++mi) {
            const int col = (wave * HT + mi) * 32 + j, n = n0 + col;
            if (col < hhalf || col >= NT - hhalf || n < h_lo || n >= h_hi) continue;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int c = 4 * hh + k;
                if (c < p.oc) p.out.y[c * p.out.plane + origin + n] = tanhf(hacc[mi][k]);
            }
        }
    }
}

hipError_t launch_res_unit_fused(const FusedArgs& a, hipStream_t stream)
{
    FusedParams p;
    p.x = (const hres_t*)a.x; p.y = (hres_t*)a.y; p.ya = a.ya; p.w7 = a.w7; p.w1 = a.w1; p.b7 = a.b7; p.b1 = a.b1;
    p.a1 = a.a1; p.ib1 = a.ib1; p.a2 = a.a2; p.ib2 = a.ib2; p.a3 = a.a3; p.ib3 = a.ib3;
    p.slots = a.slots; p.r = a.r; p.ntaps = a.ntaps;
    p.tap0 = -((a.ntaps - 1) / 2) * a.dil; p.tap_step = a.dil;
    p.nchunks = a.c / 64; p.margin = a.margin;
    if ((a.c != 64 && a.c != 128) || (a.ntaps - 1) * a.dil > FUSED_MAXSPAN || a.margin < 0 || a.x == a.y) return hipErrorInvalidValue;
    if (a.ya ? !a.a3 || !a.ib3 : !a.y) return hipErrorInvalidValue;
    // one window's activation plane must fit a 32-bit byte offset (buffer descriptors)
    if ((long long)a.max_len * a.r * a.c * (long long)sizeof(hres_t) > 0xf0000000ll) return hipErrorInvalidValue;
    const long long out_rows = std::min((long long)a.max_int * a.r + 2ll * a.margin, (long long)a.max_len * a.r);
    const bool emit = a.ya != nullptr;
    p.hw = nullptr; p.hb = p.ha = p.hib = nullptr; p.out = {}; p.oc = p.hk = 0;
    if (a.hw) {
        // the unit before the head, with the head in the same kernel: tiles advance by NT - (k - 1) interior columns
        if (a.c != 64 || a.ya || !a.out.y || !a.hb || !a.ha || !a.hib || a.hk < 1 || (a.hk & 1) == 0 || a.hk > FUSED_HEAD_MAXK ||
            a.oc < 1 || a.oc > 8 || a.margin < (a.hk - 1) / 2) return hipErrorInvalidValue;
        p.hw = a.hw; p.hb = a.hb; p.ha = a.ha; p.hib = a.hib; p.out = a.out; p.oc = a.oc; p.hk = a.hk;
    }
    auto tiles = [&](int nt) { return a.hw ? ((long long)a.max_int * a.r + nt - a.hk) / (nt - (a.hk - 1)) : (out_rows + nt - 1) / nt; };
    auto grid = [&](int nt) { return dim3((unsigned)(tiles(nt) + 7) / 8 * 8, (unsigned)a.n_slots); };       // whole groups of 8 tiles; the surplus exits at once
#define DEMON_NARROW(TM, TN, WM, WN, OCC) { \
        if (emit) hipLaunchKernelGGL((res_unit_narrow_stream_kernel<TM, TN, WM, WN, OCC, true, false>), grid(16 * TN * WN), dim3(64 * WM * WN), 0, stream, p); \
        else hipLaunchKernelGGL((res_unit_narrow_stream_kernel<TM, TN, WM, WN, OCC, false, false>), grid(16 * TN * WN), dim3(64 * WM * WN), 0, stream, p); \
        return hipGetLastError(); \
    }
    if (a.ntaps == 7 && a.c == 128) {
        // 64 columns a workgroup up to five of them per CU, else 256.  Per unit (dilation 1, 3, 9 with emitted operand) in us, 64 / 256 columns:
        // 13 frames 11, 10, 12 / 20, 20, 21; 40 frames 17, 16, 18 / 20, 20, 21; 64 frames 23, 22, 24 / 21, 21, 23; 75 frames (1133 tiles) 26, 25, 28 /
        // 28, 28, 31; 95 frames 30, 29, 32 / 28, 29, 32; 110 frames (1656) 35, 34, 38 / 29, 30, 33; 150 frames 43, 43, 47 / 47, 50, 56; 200 frames
        // 57, 56, 61 / 49, 50, 59; 375 frames 104, 102, 111 / 89, 91, 104; 60 s clip 460, 453, 526 / 378, 377, 422.
        if (tiles(64) * a.call_slots <= 1280) DEMON_NARROW(2, 4, 4, 1, 3)
        DEMON_NARROW(4, 8, 2, 2, 2)
    }
    if (a.ntaps == 7 && a.hw) {
        // the columns by the rule below: of 128 columns 122 are the head's, of 256 250 (60 s clip 5210 -> 5180 us, 375 frames 1464 -> 1457)
        if (tiles(128) * a.call_slots <= 2304) hipLaunchKernelGGL((res_unit_narrow_stream_kernel<2, 4, 2, 2, 3, false, true>), grid(128), dim3(256), 0, stream, p);
        else hipLaunchKernelGGL((res_unit_narrow_stream_kernel<2, 8, 2, 2, 3, false, true>), grid(256), dim3(256), 0, stream, p);
        return hipGetLastError();
    }
    // 64 channels.  Per unit in us, LDS-staged / 128 columns / 256 columns: 13 frames 13, 12 / 9, 8 / 10, 10; 75 frames 19 / 17 / 17; 150 frames
    // 30 / 27 / 27; 200 frames 35 / 34 / 32.  Beyond the last-level cache the stores of whole rows of the staged kernel gain nothing: on one
    // stream with an event after the launch (gated calls run so), staged / 256 columns: 375 frames 60 / 55, 500 frames 77 / 72, 600 frames 92 / 93, 1000 frames 160 /
    // 159, 1500 frames 242 / 240, the whole calls 1332 / 1309, 1835 / 1815, 2070 / 2067, 3334 / 3332, 4931 / 4926 (encodes 1356 / 1319, 1852 / 1831, 2163 / 2155, 3449 / 3440,
    // 5037 / 5036); in two groups 60 s 5059 / 5033, its encode 5078 / 5056.
    if (a.ntaps == 7 && a.c == 64) {
        if (tiles(128) * a.call_slots <= 2304) DEMON_NARROW(2, 4, 2, 2, 3)
        DEMON_NARROW(2, 8, 2, 2, 3)
    }
#undef DEMON_NARROW
    if (a.hw) {
        hipLaunchKernelGGL((res_unit_fused_kernel<64, 2, false, true>), grid(256), dim3(256), 0, stream, p);
        return hipGetLastError();
    }
    if (a.c == 64) {
        constexpr int NT = 4 * 32 * 2;
        dim3 grid((unsigned)((out_rows + NT - 1) / NT + 7) / 8 * 8, (unsigned)a.n_slots);       // whole groups of 8 tiles; the surplus exits at once
        if (emit) hipLaunchKernelGGL((res_unit_fused_kernel<64, 2, true>), grid, dim3(256), 0, stream, p);
        else hipLaunchKernelGGL((res_unit_fused_kernel<64, 2, false>), grid, dim3(256), 0, stream, p);
    } else {
        constexpr int NT = 4 * 32 * 2;
        dim3 grid((unsigned)((out_rows + NT - 1) / NT + 7) / 8 * 8, (unsigned)a.n_slots);       // whole groups of 8 tiles; the surplus exits at once
        if (emit) hipLaunchKernelGGL((res_unit_fused_kernel<128, 2, true>), grid, dim3(256), 0, stream, p);
        else hipLaunchKernelGGL((res_unit_fused_kernel<128, 2, false>), grid, dim3(256), 0, stream, p);
    }
    return hipGetLastError();
}

}  // namespace demon
