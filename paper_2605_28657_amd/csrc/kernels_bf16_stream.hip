// Convolutions of the bf16 path with the weights streamed to registers.
//
// What bound the LDS-staged tiles: a launch of few workgroups (a playback window, a short clip) lasted as long as one
// workgroup's walk over K, whatever their number -- two barriers per 8 KB weight block, four blocks in flight, 0.41 us per block
// where its MFMAs take 0.1 -- and a launch that fills the chip read as many LDS bytes per MFMA as the LDS delivers.  Here
//  * a wave streams the fragments of its own GEMM rows from global memory straight to registers, in the order the packed
//    blocks hold them (no LDS, no barrier), RS k-steps ahead in a ring of registers with static indices;
//  * the activation tile, shared by the workgroup's waves, is double-buffered in LDS in stages of SC 64-channel chunks and all
//    their taps: one barrier per stage;
//  * the MFMA is the 16 x 16 x 32 form: half the dependent accumulations of the 32 x 32 x 16 form and tiles small enough to
//    give every SIMD a chain (a dependent 32 x 32 x 16 takes 19 ns, an independent one 13.5; 16 x 16 x 32: 22 and 7.5);
//  * the output tile goes through LDS to 16-byte loads and stores of consecutive channels.
// A CU takes some 45 bytes of weights per clock in, whether they hit its L1 or not, and reads 190 bytes per clock from LDS: the
// large tile gives every wave 32 rows x 128 columns (8 KB of weights and 32 KB of LDS reads per 288 cycles of MFMAs).
// Measured, LDS-staged tile -> here: 1024-channel dilated conv 46 -> 9.6 us (200 columns), 47 -> 17 (830), 258 -> 214 (17000);
// 512 channels 34 -> 21 (4700), 60 s clip 297 (a 128 x 256 tile) -> 266 (1.24 PFLOP/s); 1x1 conv of 1024 channels 13 -> 5 (200), 14 -> 7.6 (830);
// strided conv 1024 -> 128, stride 10: 146 -> 25 (75 columns).  That one, 640 k-steps in a workgroup and a column a frame, lasts as long as one
// walk at any size: with K in eight parts (MODE_PART), which the sampling step sums, 26 -> 9 us at 75 columns and 72 -> 18 at 1500, with an event after the
// launch; encode of 75 frames 509 -> 495, of 60 s 5089 -> 5080.  Eight because an XCD then holds a part: its L2 reads an eighth of weights and activations.
// Every tile adds in the same order (chunk, tap, k-step, for two operand planes hi before lo), so a value does not depend on the tile.
#include <algorithm>
#include <type_traits>

#include "conv_bf16.h"

namespace demon {

namespace {

struct StreamGrid {
    int xm, xn;              // the 8 XCDs as xm groups of 128-row panels x xn groups of column tiles
    int mper;                // row tiles of an XCD
};

// Tile: WM x WN waves of TM x TN accumulator tiles of 16 rows x 16 columns.
// NB: activation buffers, 2, or 1 for layers of a single stage.
// NTAPS: the taps, unrolled, or 0: any number, counted at run time (dilated convs of kernel sizes other than 7).
// The transposed conv's largest tile keeps to the 168 registers of three workgroups per CU (170: +5 %).
template <int TM, int TN, int WM, int WN, int NTAPS, int SC, int SPAN, int MODE, int IN, int NB>
__global__ __launch_bounds__(64 * WM * WN, MODE == MODE_UP && TM * TN == 16 && IN != OP_BF16X2 ? 3 : 1) void conv_stream_kernel(MfmaParams p, StreamGrid sg, int emit)
{
    fp16_saturate_on();
    constexpr int NTH = 64 * WM * WN, MT = 16 * TM * WM, NT = 16 * TN * WN;
    constexpr bool DOWN = MODE == MODE_DOWN || MODE == MODE_PART;
    constexpr int XS = DOWN ? 2 : 1;                       // input rows per GEMM column
    constexpr int XROWS = XS * (NT - 1) + 1 + SPAN;
    // channels of a stage; padded LDS row: 16-byte reads of 16 rows x 4 neighbouring pieces are free of bank conflicts (5.3 cycles
    // a wave, else 8 or more) when the rows lie 2 (mod 4) pieces apart
    constexpr int KX = 64 * SC, LDR = KX + 16 / XS;
    constexpr int NP = IN == OP_BF16X2 ? 2 : 1;
    constexpr int SEGS = KX / 8, RPP = NTH / SEGS, X_ITERS = (XROWS + RPP - 1) / RPP;
    constexpr int XR = X_ITERS * RPP;                      // rows held (whole passes)
    constexpr bool ANY = NTAPS == 0;
    constexpr int F = SC * NTAPS * 2;                      // k-steps of a stage
    // k-steps in flight: a step lasts TM x TN MFMAs of 8 ns, an L2 hit some 400 ns
    constexpr int RS = ANY ? (TM == 1 ? 12 : 8) : TM * F <= 32 ? F : F / 2;
    static_assert(F % RS == 0 && RS % 2 == 0 && RS / 2 * 16384 <= kWeightSlack, "static ring indices");
    const int ntaps = ANY ? p.ntaps : NTAPS;
    constexpr int LDO = MT + 4;                            // padded row of the fp32 output tile
    constexpr int X_BYTES = NP * XR * LDR * 2;
    constexpr int EP = NT * LDO * 4 > NB * X_BYTES && TN % 2 == 0 ? 2 : 1;      // passes of the epilogue
    constexpr int O_BYTES = NT / EP * LDO * 4;
    constexpr int SMEM = NB * X_BYTES > O_BYTES ? NB * X_BYTES : O_BYTES;
    static_assert(NTH % SEGS == 0 && TN % EP == 0, "whole rows per pass");
    __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM];

    const Slot s = p.slots[blockIdx.y];
    const int nrows = s.len * p.r_in;
    const int r_out = (MODE == MODE_UP) ? p.r_in * p.stride : DOWN ? p.r_in / 2 : p.r_in;
    const int nrows_o = s.len * r_out;
    const int out_lo = max(0, s.crop * r_out - p.margin);
    const int out_hi = min(nrows_o, (s.crop + s.n_int) * r_out + p.margin);
    if (out_hi <= out_lo) return;                           // an empty window (a gated clip)
    const int col_lo = (MODE == MODE_UP) ? (out_lo + p.stride / 2) / p.stride : out_lo;
    const int ncols = (MODE == MODE_UP) ? (out_hi - 1 + p.stride / 2) / p.stride + 1 : out_hi;
    // Workgroups are dealt to the 8 XCDs round-robin by linear id (gridDim.x is a multiple of 8), each with its own L2.  XCD
    // (x % xm, x / xm) takes every xm-th panel of 128 rows and every xn-th column tile (rotated by the window): it reads
    // 1/xm of the weights and 1/xn of the activations.  K in parts: an XCD takes one of the eight parts, and reads an eighth of both.
    constexpr int SUB = 128 / MT;                           // row tiles of a panel
    const int part = MODE == MODE_PART ? (int)(blockIdx.x & 7u) : 0;
    const int xcd = MODE == MODE_PART ? 0 : (int)((blockIdx.x + blockIdx.y) & 7u), q8 = (int)(blockIdx.x >> 3), mi8 = q8 % sg.mper;
    const int panel = xcd % sg.xm + sg.xm * (mi8 / SUB), ntile = xcd / sg.xm + sg.xn * (q8 / sg.mper);
    const int n0 = col_lo + ntile * NT;
    if (n0 >= ncols) return;
    const int sub = mi8 % SUB, m0 = panel * 128 + sub * MT;
    const long long rowbase = (long long)s.row0 * p.r_in, rowbase_o = (long long)s.row0 * r_out;
    const int minoff = min(p.tap0, p.tap0 + (ntaps - 1) * p.tap_step);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int i = lane & 15, q = lane >> 4;
    const int seg = tid % SEGS, xr0 = tid / SEGS;

    const __amdgpu_buffer_rsrc_t rs_w = weight_rsrc(p.w, p.w_bytes);
    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(p.xa + rowbase * p.cin, (unsigned)nrows * p.cin * 2u);
    const __amdgpu_buffer_rsrc_t rs_xl = make_rsrc(p.xa + p.in_lo_off + rowbase * p.cin, NP == 2 ? (unsigned)nrows * p.cin * 2u : 0u);

    // ---- weights: blocks of 128 x 64 (16 KB) in fragment order, [16-slot tile][2 k-steps][lane][8].  Slot 32 k + l of a group of
    // 64 is row 2 l + k (see slot_to_row): slot tiles 0, 2 hold rows 0..31 of the group (even, odd), 1, 3
    // rows 32..63.  Unit u of a panel takes them in the order 0, 2, 1, 3; its lane i is row 32 (u / 2) + 2 i + u % 2.
    const int nblocks = p.nchunks * ntaps;
    const int unit0 = sub * (MT / 16) + wm * TM;                             // first unit of this wave in the panel
    const unsigned w_voff = (unsigned)((unit0 & ~3) + (unit0 & 1) * 2 + (unit0 >> 1 & 1)) * 2048u + lane * 16u;
    const unsigned w_tile = (unsigned)panel * (unsigned)nblocks * 16384u;
    // any number of taps: requests past the panel's last block read the next panel's (nobody's after the last panel) and are not used
    const bool more_panels = w_tile + (unsigned)nblocks * 16384u < p.w_bytes;
    u32x4 a[RS][TM];
    auto load_a = [&](int block0, int f, unsigned voff) __attribute__((always_inline)) {     // k-step f from block0 on
        const unsigned blk = w_tile + (unsigned)(block0 + f / 2) * 16384u;
#pragma unroll
        for (int mi = 0; mi < TM; ++mi) a[f % RS][mi] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, voff + ((mi & 1) * 2 + (mi >> 1)) * 2048u + (f & 1) * 1024u, blk, 0);
    };
    auto lane_row = [&](int mi) __attribute__((always_inline)) -> int {      // GEMM row of this lane in the tile
        const int u = unit0 + mi;
        return (u >> 1) * 32 + 2 * i + (u & 1) - sub * MT;
    };

    // ---- activations
    const unsigned x_voff = ((unsigned)((XS * n0 + minoff + xr0) * p.cin) + seg * 8u) * 2u;    // may wrap "negative": out of range
    const unsigned x_row_step = (unsigned)(RPP * p.cin) * 2u;
    const int nstages = MODE == MODE_PART ? p.nchunks / kConvParts / SC : p.nchunks / SC, stage0 = part * nstages;
    u32x4 rx[X_ITERS][NP];
    auto load_x = [&](int stage) __attribute__((always_inline)) {
        const unsigned base = stage < nstages ? x_voff + (unsigned)((stage0 + stage) * KX) * 2u : 0xf8000000u;      // past the last stage: out of range
#pragma unroll
        for (int it = 0; it < X_ITERS; ++it) {
            // any number of taps: rows that no tap reads are out of range too
            const unsigned off = ANY && it * RPP >= XS * (NT - 1) + 1 + (ntaps - 1) * p.tap_step ? 0xf8000000u : base + it * x_row_step;
            rx[it][0] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, off, 0, 0);
            if (NP == 2) rx[it][NP - 1] = __builtin_amdgcn_raw_buffer_load_b128(rs_xl, off, 0, 0);
        }
    };
    auto store_x = [&](int buf) __attribute__((always_inline)) {
        uint16_t* xs = reinterpret_cast<uint16_t*>(smem + buf * X_BYTES);
#pragma unroll
        for (int it = 0; it < X_ITERS; ++it)
#pragma unroll
            for (int pl = 0; pl < NP; ++pl)
                *reinterpret_cast<u32x4*>(&xs[pl * XR * LDR + (xr0 + it * RPP) * LDR + seg * 8]) = rx[it][pl];
    };

    // every request of the prologue in the order of use
    load_x(0);
#pragma unroll
    for (int f = 0; f < RS; ++f) load_a(stage0 * (F / 2), f, ANY ? ahead_voff(w_voff, more_panels || f / 2 < nblocks) : w_voff);
    float bv[TM];
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) bv[mi] = part > 0 ? 0.f : p.bias[(MODE == MODE_UP) ? (m0 + lane_row(mi)) % p.cout : m0 + lane_row(mi)];

    // ---- geometry of the epilogue: piece (row, 8 channels) of the output tile; residual values requested ahead where the
    // registers allow it
    constexpr int PPR = MT / 8, ERPP = NTH / PPR, E_ITERS = (NT / EP + ERPP - 1) / ERPP;
    static_assert(NTH % PPR == 0, "whole rows per pass");
    constexpr int WROWS = NT / EP / WN;                                 // rows of a pass that belong to one wave column
    const int ec = m0 + (tid % PPR) * 8, er0 = tid / PPR;
    auto eoff = [&](int ep, int it) __attribute__((always_inline)) -> unsigned {
        const int r = er0 + it * ERPP;
        if (NT / EP % ERPP != 0 && r >= NT / EP) return kOutOfRange;
        const int n = n0 + r / WROWS * (16 * TN) + ep * WROWS + r % WROWS;
        // transposed conv: column n, row mu lands on the run starting at (n s - p) cout + mu; a negative row wraps: out of range
        return (MODE == MODE_UP ? (unsigned)((n * p.stride - p.stride / 2) * p.cout + ec) : (unsigned)(n * p.cout + ec)) * 2u;
    };
    const unsigned out_bytes = (unsigned)out_hi * p.cout * 2u;
    const __amdgpu_buffer_rsrc_t rs_y = make_rsrc(MODE == MODE_ACT || MODE == MODE_PART ? nullptr : p.y + rowbase_o * p.cout, MODE == MODE_ACT || MODE == MODE_PART ? 0u : out_bytes);
    u32x4 resv[MODE == MODE_RES ? EP : 1][MODE == MODE_RES ? E_ITERS : 1];
    auto load_res = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int ep = 0; ep < EP; ++ep)
#pragma unroll
            for (int it = 0; it < E_ITERS; ++it) resv[ep][it] = __builtin_amdgcn_raw_buffer_load_b128(rs_y, eoff(ep, it), 0, 0);
    };
    constexpr bool EARLY_RES = MODE == MODE_RES && E_ITERS * EP <= 4;
    if (EARLY_RES) load_res();

    f32x4 acc[TM][TN];
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = f32x4{bv[mi], bv[mi], bv[mi], bv[mi]};

    store_x(0);
    __syncthreads();

    // The k-steps are a software pipeline held in source order by scheduling fences: activation fragments AHEAD steps before their
    // MFMAs, the step's weight registers refilled right after them.  (Left to itself the compiler runs one accumulator's whole
    // chain, then the next, waiting out the LDS latency of every fragment.)
    constexpr int AHEAD = TM * TN <= 2 ? 6 : TM * TN <= 4 ? 3 : 1, XD = AHEAD + 1;
    if constexpr (ANY) {
        // One walk over all blocks of K, unrolled by the ring: a block is a tap of a 64-channel chunk, two k-steps.  Fragments are
        // read AH k-steps ahead, past the end of a stage from the same buffer again (in bounds, not used); at the switch to the
        // next stage they are read once more.  1024-channel dilated conv of 9 taps, LDS-staged 128 x 128 tile -> here:
        // 83 -> 26 us (13 frames), 84 -> 32 (75 frames), 199 -> 169 (1000), 306 -> 266 (1500).
        constexpr int RB = RS / 2, AH = TM * TN <= 2 ? 4 : TM * TN <= 6 ? 2 : 1, D = (AH + 1) / 2, XR3 = AH + (AH > 1 ? 2 : 1) - (AH == 2 ? 1 : 0);
        static_assert(RS % XR3 == 0 && NP == 1, "static indices; one operand plane");
        const int nb = SC * ntaps;                                           // blocks of a stage
        const uint16_t* xs = nullptr;
        int off[D + 1], rt = 0, rc = 0, next = 0;                            // LDS offsets of this block and the D after it
        auto push = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int d = 0; d < D; ++d) off[d] = off[d + 1];
            off[D] = next;
            next += p.tap_step * LDR;
            if (++rt == ntaps) { rt = 0; if (++rc == SC) rc = 0; next = rc * 64; }
        };
        u32x4 x[XR3][TN];
        auto read_x = [&](int slot, int at, int ni) __attribute__((always_inline)) {
            x[slot][ni] = *reinterpret_cast<const u32x4*>(xs + at + ni * 16 * LDR);
        };
        int stage = -1, b = nb;
        for (int g0 = 0; g0 < nblocks; g0 += RB) {
#pragma unroll
            for (int u = 0; u < RB; ++u) {
                if (g0 + u >= nblocks) break;
                if (b == nb) {
                    if (stage >= 0) { store_x((stage + 1) & 1); __syncthreads(); }
                    ++stage;
                    load_x(stage + 1);
                    xs = reinterpret_cast<const uint16_t*>(smem + (stage & 1) * X_BYTES) + (wn * (16 * TN) + i) * LDR + q * 8;
                    b = rt = rc = next = 0;
#pragma unroll
                    for (int d = 0; d <= D; ++d) push();
#pragma unroll
                    for (int s = 0; s < AH; ++s)
#pragma unroll
                        for (int ni = 0; ni < TN; ++ni) read_x((2 * u + s) % XR3, off[s / 2] + s % 2 * 32, ni);
                }
                const unsigned voff = ahead_voff(w_voff, more_panels || g0 + u + RB < nblocks);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    const int f = 2 * u + ks;
#pragma unroll
                    for (int ni = 0; ni < TN; ++ni) {
                        read_x((f + AH) % XR3, off[(ks + AH) / 2] + (ks + AH) % 2 * 32, ni);
#pragma unroll
                        for (int mi = 0; mi < TM; ++mi) {
                            if (IN == OP_F16)
                                acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, x[f % XR3][ni]), __builtin_bit_cast(f16x8, a[f][mi]), acc[mi][ni], 0, 0, 0);
                            else
                                acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x[f % XR3][ni]), __builtin_bit_cast(bf16x8, a[f][mi]), acc[mi][ni], 0, 0, 0);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    load_a(g0, f + RS, voff);
                    __builtin_amdgcn_sched_barrier(0);
                }
                push();
                ++b;
            }
        }
        __syncthreads();
    } else {
        // the last stage on its own: nothing is requested past the layer's end
        auto run_stage = [&](int stage, auto last) __attribute__((always_inline)) {
            constexpr bool LAST = decltype(last)::value;
            if (!LAST) load_x(stage + 1);
            const uint16_t* xs = reinterpret_cast<const uint16_t*>(smem + (NB == 2 ? (stage & 1) * X_BYTES : 0)) + (wn * (16 * TN) + i) * XS * LDR + q * 8;
            u32x4 x[XD][TN][NP];
            auto read_x = [&](int f, int ni) __attribute__((always_inline)) {
                const int ks = f & 1, tap = (f / 2) % NTAPS, c = f / (2 * NTAPS);
                const uint16_t* xt = xs + (p.tap0 + tap * p.tap_step - minoff) * LDR + c * 64 + ks * 32 + ni * 16 * XS * LDR;
#pragma unroll
                for (int pl = 0; pl < NP; ++pl) x[f % XD][ni][pl] = *reinterpret_cast<const u32x4*>(xt + pl * XR * LDR);
            };
#pragma unroll
            for (int f = 0; f < AHEAD && f < F; ++f)
#pragma unroll
                for (int ni = 0; ni < TN; ++ni) read_x(f, ni);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int f = 0; f < F; ++f) {
#pragma unroll
                for (int t = 0; t < NP * TN; ++t) {
                    const int pl = t / TN, ni = t % TN;
                    if (pl == 0 && f + AHEAD < F) read_x(f + AHEAD, ni);
                    // activations are the row operand: the accumulator tile is [time][GEMM row].  Two operand planes: the step's hi
                    // values of every column tile, then its lo values, against the same weights.
#pragma unroll
                    for (int mi = 0; mi < TM; ++mi) {
                        const u32x4 w = a[f % RS][mi];
                        if (IN == OP_F16)
                            acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, x[f % XD][ni][pl]), __builtin_bit_cast(f16x8, w), acc[mi][ni], 0, 0, 0);
                        else
                            acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x[f % XD][ni][pl]), __builtin_bit_cast(bf16x8, w), acc[mi][ni], 0, 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (!LAST || f + RS < F) load_a((stage0 + stage) * (F / 2), f + RS, w_voff);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (!LAST) store_x((stage + 1) & 1);
            __syncthreads();
        };
        int stage = 0;
        if constexpr (NB == 2)
            for (; stage + 1 < nstages; ++stage) run_stage(stage, std::false_type{});
        run_stage(stage, std::true_type{});
    }

    // ---- epilogue: register e of lane (i, q) is time row 4 q + e, GEMM row lane_row(mi)
    if (MODE == MODE_RES && !EARLY_RES) load_res();
    float oa[8], ob[8];
    if (emit > 0) {
        const int c0 = (MODE == MODE_UP) ? ec % p.cout : ec;
#pragma unroll
        for (int e = 0; e < 8; e += 4) {
            const f32x4 va = *reinterpret_cast<const f32x4*>(p.out_alpha + c0 + e), vb = *reinterpret_cast<const f32x4*>(p.out_inv_beta + c0 + e);
#pragma unroll
            for (int k = 0; k < 4; ++k) { oa[e + k] = va[k]; ob[e + k] = vb[k]; }
        }
    }
    const __amdgpu_buffer_rsrc_t rs_a = make_rsrc(p.ya + rowbase_o * p.cout, emit > 0 ? out_bytes : 0u);
    const __amdgpu_buffer_rsrc_t rs_ys = MODE == MODE_RES ? make_rsrc(p.y + rowbase_o * p.cout, p.y_dead ? 0u : out_bytes) : rs_y;
    const __amdgpu_buffer_rsrc_t rs_al = make_rsrc(p.ya + p.out_lo_off + rowbase_o * p.cout, emit == 2 ? out_bytes : 0u);
    // K in parts: this part's sums, rows kConvParts x cout apart; nothing past the last row's
    const __amdgpu_buffer_rsrc_t rs_p = make_rsrc(p.part + (rowbase_o * kConvParts + part) * p.cout, MODE == MODE_PART ? ((unsigned)(out_hi - 1) * kConvParts + 1u) * p.cout * 4u : 0u);
    float* os = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int ep = 0; ep < EP; ++ep) {
        if (ep > 0) __syncthreads();
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int ni = 0; ni < TN / EP; ++ni)
#pragma unroll
                for (int e = 0; e < 4; ++e) os[(wn * WROWS + ni * 16 + 4 * q + e) * LDO + lane_row(mi)] = acc[mi][ep * (TN / EP) + ni][e];
        __syncthreads();
#pragma unroll
        for (int it = 0; it < E_ITERS; ++it) {
            if (NT / EP % ERPP != 0 && er0 + it * ERPP >= NT / EP) break;
            const float* src = &os[(er0 + it * ERPP) * LDO + (tid % PPR) * 8];
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = src[e];
            const unsigned off = eoff(ep, it);
            if constexpr (MODE == MODE_PART) {
                const unsigned at = part_voff(off, (unsigned)ec);
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, f32x4{v[0], v[1], v[2], v[3]}), rs_p, at, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, f32x4{v[4], v[5], v[6], v[7]}), rs_p, at + 16u, 0, 0);
                continue;
            }
            if (MODE == MODE_RES) {
                const f16x8 r = __builtin_bit_cast(f16x8, resv[ep][it]);
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = keep_f32(v[e] + (float)r[e]);
            }
            if (MODE != MODE_ACT) {
                // half store of h; the next layer's operand is Snake of the STORED value
                f16x8 hv;
#pragma unroll
                for (int e = 0; e < 8; ++e) { hv[e] = (_Float16)v[e]; v[e] = (float)hv[e]; }
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, hv), rs_ys, off, 0, 0);
            }
            if (emit == 0) continue;                                                  // uniform
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = keep_f32(snake_fast(v[e], oa[e], ob[e]));            // fp32 Snake, then one rounding
            u32x4 o;
            if (emit == 3) {
#pragma unroll
                for (int k = 0; k < 4; ++k) o[k] = pack_f16x2(v[2 * k], v[2 * k + 1]);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) o[k] = pack_bf16x2(v[2 * k], v[2 * k + 1]);
            }
            __builtin_amdgcn_raw_buffer_store_b128(o, rs_a, off, 0, 0);
            if (emit == 2) {                                                          // what the hi plane's rounding left over
                u32x4 lo;
#pragma unroll
                for (int k = 0; k < 4; ++k) lo[k] = pack_bf16x2(v[2 * k] - __uint_as_float(o[k] << 16), v[2 * k + 1] - __uint_as_float(o[k] & 0xffff0000u));
                __builtin_amdgcn_raw_buffer_store_b128(lo, rs_al, off, 0, 0);
            }
        }
    }
}

// Dilated convs of seven taps in launches of many tiles: 256 rows x 128 columns, a wave owning 64 rows of all columns (256 registers, two
// workgroups per CU).  The 128 x 128 tile above reads 8 KB of LDS per wave and 256 cycles of MFMAs, the most a CU delivers; here it is 8 KB per
// 512, with 4 KB of weights.  Weights are the row operand, so that a lane ends with 8 consecutive channels of a column and the
// epilogue needs no LDS.  512 channels, 60 s clip 260 -> 241 us in a call that is waited for (1.37 PFLOP/s; in back-to-back steps at the power
// limit 244 to 258, 1.28 to 1.35); the call 5551 -> 5500.  The same shape for the transposed convs (few k-steps, long epilogues: two workgroups per CU cover them
// less well than three) is slower: 231 -> 242 us, 205 -> 244.
template <int SPAN, int IN>
__global__ __launch_bounds__(256, 2) void conv_tall_kernel(MfmaParams p, StreamGrid sg, bool half_out)
{
    fp16_saturate_on();
    constexpr int NTAPS = 7, TM = 4, TN = 8, MT = 256, NT = 16 * TN;
    constexpr int KX = 64, LDR = KX + 16;                   // stage of a chunk; rows 10 pieces apart: no bank conflicts
    constexpr int SEGS = KX / 8, RPP = 256 / SEGS, X_ITERS = (NT + SPAN + RPP - 1) / RPP, XR = X_ITERS * RPP;
    constexpr int F = 2 * NTAPS, G = F * TN;                // k-steps of 32 in a stage, groups of TM MFMAs
    constexpr int RS = 4;                                   // k-steps of weights in flight
    constexpr int XA = 3, XQ = XA + 1;                      // activation fragments read ahead of their MFMAs
    constexpr int X_BYTES = XR * LDR * 2;
    static_assert(2 * F % RS == 0 && X_ITERS <= 6 && RS / 2 * 16384 <= kWeightSlack, "static ring indices");
    __shared__ __attribute__((aligned(16))) unsigned char smem[2 * X_BYTES];

    const Slot s = p.slots[blockIdx.y];
    const int nrows = __builtin_amdgcn_readfirstlane(s.len * p.r_in);     // (the descriptors must be scalar)
    const int out_lo = max(0, s.crop * p.r_in - p.margin);
    const int out_hi = min(nrows, (s.crop + s.n_int) * p.r_in + p.margin);
    // XCD (x % xm, x / xm) takes every xm-th row tile and every xn-th column tile, as above
    const int xcd = (int)((blockIdx.x + blockIdx.y) & 7u), q8 = (int)(blockIdx.x >> 3);
    const int mtile = xcd % sg.xm + sg.xm * (q8 % sg.mper), ntile = xcd / sg.xm + sg.xn * (q8 / sg.mper);
    const int n0 = out_lo + ntile * NT, m0 = mtile * MT;
    if (n0 >= out_hi) return;                               // (also an empty window: a gated clip)
    const long long rowbase = (long long)__builtin_amdgcn_readfirstlane(s.row0) * p.r_in;

    int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int i = lane & 15, q = lane >> 4;
    const int seg = tid % SEGS, xr0 = tid / SEGS;

    const __amdgpu_buffer_rsrc_t rs_w = weight_rsrc(p.w, p.w_bytes);
    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(p.xa + rowbase * p.cin, (unsigned)nrows * p.cin * 2u);

    // weights as above: this wave's four units are half of a panel of 128 rows, unit u (order 0, 2, 1, 3 in the block) slot l is
    // row 32 (u / 2) + 2 l + u % 2 of the wave's 64
    const int nblocks = p.nchunks * NTAPS;
    const unsigned w_voff = (unsigned)lane * 16u;
    const unsigned w_tile = (unsigned)(2 * mtile + (wave >> 1)) * (unsigned)nblocks * 16384u + (wave & 1) * 8192u;
    u32x4 a[RS][TM];
    auto load_a = [&](int block0, int f, int slot) __attribute__((always_inline)) {          // k-step f from block0 on
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
            a[slot][mi] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, w_voff, w_tile + (unsigned)(block0 + f / 2) * 16384u + ((mi & 1) * 2 + (mi >> 1)) * 2048u + (f & 1) * 1024u, 0);
    };

    const unsigned x_voff = ((unsigned)((n0 + p.tap0 + xr0) * p.cin) + seg * 8u) * 2u;      // may wrap "negative": out of range
    const unsigned x_row_step = (unsigned)(RPP * p.cin) * 2u;
    const int nstages = p.nchunks;                          // even
    u32x4 rx[X_ITERS];
    auto load_x = [&](int stage, int it) __attribute__((always_inline)) {
        rx[it] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, x_voff + (unsigned)(stage * KX) * 2u + it * x_row_step, 0, 0);
    };
    auto store_x = [&](int buf, int it) __attribute__((always_inline)) {
        *reinterpret_cast<u32x4*>(smem + buf * X_BYTES + ((xr0 + it * RPP) * LDR + seg * 8) * 2) = rx[it];
    };
#pragma unroll
    for (int it = 0; it < X_ITERS; ++it) load_x(0, it);
#pragma unroll
    for (int f = 0; f < RS; ++f) load_a(0, f, f);
    // weights are the row operand: registers e of units 2 pr, 2 pr + 1 are rows rb + 32 pr + {0..7} (2 e + unit) of column 16 ni + i
    const int rb = m0 + 64 * wave + 8 * q;
    f32x4 acc[TM][TN];
#pragma unroll
    for (int pr = 0; pr < 2; ++pr) {
        const f32x4 b0 = *reinterpret_cast<const f32x4*>(p.bias + rb + 32 * pr), b1 = *reinterpret_cast<const f32x4*>(p.bias + rb + 32 * pr + 4);
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) {
            acc[2 * pr][ni] = f32x4{b0[0], b0[2], b1[0], b1[2]};
            acc[2 * pr + 1][ni] = f32x4{b0[1], b0[3], b1[1], b1[3]};
        }
    }
#pragma unroll
    for (int it = 0; it < X_ITERS; ++it) store_x(0, it);
    __syncthreads();

    __builtin_amdgcn_s_setprio(1);                          // waves in this loop go first
    const int tap_bytes = p.tap_step * (LDR * 2);
    auto run_stage = [&](int stage_, auto half_, auto last) __attribute__((always_inline)) {
        const int stage = __builtin_amdgcn_readfirstlane(stage_);
        constexpr int half = decltype(half_)::value;
        constexpr bool NEXT = half == 0 || !decltype(last)::value;          // another stage follows
        unsigned at = half * X_BYTES + (i * LDR + q * 8) * 2;
        u32x4 x[XQ];
        auto read_x = [&](int t) __attribute__((always_inline)) {
            const int f = t / TN, ni = t % TN;              // k-step (chunk half ks, tap): the taps of a half are 32 channels apart
            if (t > 0 && t % (2 * TN) == 0) { at += tap_bytes; asm volatile("" : "+v"(at)); }
            x[t % XQ] = *reinterpret_cast<const u32x4*>(smem + at + (16 * ni * LDR + f % 2 * 32) * 2);
        };
#pragma unroll
        for (int t = 0; t < XA; ++t) read_x(t);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < F; ++f) {
            if constexpr (NEXT) {
                // the next stage's activations, two rows of a thread at a time
                if (f >= 4 && f % 4 == 0) {
#pragma unroll
                    for (int it = f / 2 - 2; it < f / 2 && it < X_ITERS; ++it) store_x(half ^ 1, it);
                }
                if (f % 4 == 0) {
#pragma unroll
                    for (int it = f / 2; it < f / 2 + 2 && it < X_ITERS; ++it) load_x(stage + 1, it);
                }
            }
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) {
                const int t = f * TN + ni;
                if (t + XA < G) read_x(t + XA);
#pragma unroll
                for (int mi = 0; mi < TM; ++mi) {
                    const u32x4 w = a[(half * F + f) % RS][mi];
                    if (IN == OP_F16)
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w), __builtin_bit_cast(f16x8, x[t % XQ]), acc[mi][ni], 0, 0, 0);
                    else
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x[t % XQ]), acc[mi][ni], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (NEXT || f + RS < F) load_a(stage * NTAPS, f + RS, (half * F + f) % RS);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (NEXT) __syncthreads();
    };
    int stage = 0;
    for (; stage + 2 < nstages; stage += 2) {
        run_stage(stage, std::integral_constant<int, 0>{}, std::false_type{});
        run_stage(stage + 1, std::integral_constant<int, 1>{}, std::false_type{});
    }
    run_stage(stage, std::integral_constant<int, 0>{}, std::true_type{});
    run_stage(stage + 1, std::integral_constant<int, 1>{}, std::true_type{});
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);

    // ---- epilogue: 8 rows (channels) of a column a lane, 64 bytes in four lanes
    asm volatile("" : "+v"(tid));                           // what the lane's number decides is formed again: nothing of it is held through the loop
    i = tid & 15; q = (tid >> 4) & 3;
    const __amdgpu_buffer_rsrc_t rs_a = make_rsrc(p.ya + rowbase * p.cout, (unsigned)out_hi * p.cout * 2u);
#pragma unroll
    for (int pr = 0; pr < 2; ++pr) {
        const int row = m0 + 64 * wave + 32 * pr + 8 * q;
        float oa[8], ob[8];
#pragma unroll
        for (int e = 0; e < 8; e += 4) {
            const f32x4 va = *reinterpret_cast<const f32x4*>(p.out_alpha + row + e), vb = *reinterpret_cast<const f32x4*>(p.out_inv_beta + row + e);
#pragma unroll
            for (int k = 0; k < 4; ++k) { oa[e + k] = va[k]; ob[e + k] = vb[k]; }
        }
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) {
            __builtin_amdgcn_sched_barrier(0);
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = keep_f32(snake_fast(acc[2 * pr + (e & 1)][ni][e >> 1], oa[e], ob[e]));       // fp32 Snake, then one rounding
            u32x4 o;
            if (half_out) {
#pragma unroll
                for (int k = 0; k < 4; ++k) o[k] = pack_f16x2(v[2 * k], v[2 * k + 1]);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) o[k] = pack_bf16x2(v[2 * k], v[2 * k + 1]);
            }
            __builtin_amdgcn_raw_buffer_store_b128(o, rs_a, (unsigned)((n0 + 16 * ni + i) * p.cout + row) * 2u, 0, 0);
        }
    }
}

template <int TM, int TN, int WM, int WN>
hipError_t launch_tile(const MfmaParams& p, const StreamGrid& sg, int mode, int in_fmt, int emit, dim3 grid, hipStream_t stream)
{
    // Two operand planes (hi + lo) are two MFMAs per k-step against one set of weights, as in the LDS-staged kernel, and twice the
    // LDS per stage.  Whole decodes in us, before (planes alternating per 16 K values, half of every MFMA's K slots zero, with
    // the LDS-staged tile from 256 tiles on) and after: 75 frames 566 -> 511, 250 frames 1231 -> 1204, 750 frames 3249 -> 3225, 1500
    // frames 6410 -> 6439.
    // SC: the more k-steps a stage holds, the deeper the weight ring of the small tiles and the fewer barriers; the chunk
    // count of the layer must be a multiple
    constexpr bool small = TM == 1;
    constexpr int SA = small ? 2 : 1, SR = TN * WN <= 2 ? 8 : TN * WN <= 4 ? 4 : TN * WN <= 6 ? 2 : 1, SU = small ? 4 : TN * WN <= 6 ? 2 : 1, SD = small ? 2 : 1;
#define DEMON_CASE(NTAPS_, SC_, SPAN_, MODE_, IN_, NB_) \
    if (in_fmt == IN_) { \
        hipLaunchKernelGGL((conv_stream_kernel<TM, TN, WM, WN, NTAPS_, SC_, SPAN_, MODE_, IN_, NB_>), grid, dim3(64 * WM * WN), 0, stream, p, sg, emit); \
        return hipGetLastError(); \
    }
    if (mode == MODE_ACT) {
        const int span = (p.ntaps - 1) * p.tap_step;
        if (p.ntaps == 1) {                                 // no rows beyond the columns
            if (p.nchunks % SR == 0) { DEMON_CASE(1, SR, 0, MODE_ACT, OP_BF16, 2) DEMON_CASE(1, SR, 0, MODE_ACT, OP_F16, 2) }
            else { DEMON_CASE(1, 2, 0, MODE_ACT, OP_BF16, 2) DEMON_CASE(1, 2, 0, MODE_ACT, OP_F16, 2) }
        } else if (p.ntaps != 7) { DEMON_CASE(0, SA, MAXSPAN, MODE_ACT, OP_BF16, 2) DEMON_CASE(0, SA, MAXSPAN, MODE_ACT, OP_F16, 2) }
        else if (span <= 6) { DEMON_CASE(7, SA, 6, MODE_ACT, OP_BF16, 2) DEMON_CASE(7, SA, 6, MODE_ACT, OP_F16, 2) }
        else if (span <= 18) { DEMON_CASE(7, SA, 18, MODE_ACT, OP_BF16, 2) DEMON_CASE(7, SA, 18, MODE_ACT, OP_F16, 2) }
        else { DEMON_CASE(7, SA, MAXSPAN, MODE_ACT, OP_BF16, 2) DEMON_CASE(7, SA, MAXSPAN, MODE_ACT, OP_F16, 2) }
    } else if (mode == MODE_RES) {
        if (p.nchunks % SR == 0) { DEMON_CASE(1, SR, 0, MODE_RES, OP_BF16, 2) DEMON_CASE(1, SR, 0, MODE_RES, OP_F16, 2) }
        else { DEMON_CASE(1, 2, 0, MODE_RES, OP_BF16, 2) DEMON_CASE(1, 2, 0, MODE_RES, OP_F16, 2) }
        constexpr int SX = SR >= 4 ? SR / 2 : 1;            // two planes: half the chunks in the same LDS
        if (p.nchunks % SX == 0) { DEMON_CASE(1, SX, 0, MODE_RES, OP_BF16X2, 2) }
        DEMON_CASE(1, 1, 0, MODE_RES, OP_BF16X2, 2)
    } else if (mode == MODE_DOWN) {
        if (p.nchunks == 1) { DEMON_CASE(4, 1, 3, MODE_DOWN, OP_BF16, 1) DEMON_CASE(4, 1, 3, MODE_DOWN, OP_F16, 1) }
        else if (p.nchunks % SD == 0) { DEMON_CASE(4, SD, 3, MODE_DOWN, OP_BF16, 2) DEMON_CASE(4, SD, 3, MODE_DOWN, OP_F16, 2) }
        else { DEMON_CASE(4, 1, 3, MODE_DOWN, OP_BF16, 2) DEMON_CASE(4, 1, 3, MODE_DOWN, OP_F16, 2) }
    } else if (mode == MODE_PART) {
        DEMON_CASE(4, SD, 3, MODE_PART, OP_BF16, 2) DEMON_CASE(4, SD, 3, MODE_PART, OP_F16, 2)
    } else {
        if (p.nchunks == 1) { DEMON_CASE(2, 1, 1, MODE_UP, OP_BF16, 1) DEMON_CASE(2, 1, 1, MODE_UP, OP_F16, 1) }
        else if (p.nchunks % SU == 0) { DEMON_CASE(2, SU, 1, MODE_UP, OP_BF16, 2) DEMON_CASE(2, SU, 1, MODE_UP, OP_F16, 2) }
        else { DEMON_CASE(2, 1, 1, MODE_UP, OP_BF16, 2) DEMON_CASE(2, 1, 1, MODE_UP, OP_F16, 2) }
        if (p.nchunks % 2 == 0) { DEMON_CASE(2, small ? 2 : 1, 1, MODE_UP, OP_BF16X2, 2) }
        DEMON_CASE(2, 1, 1, MODE_UP, OP_BF16X2, 2)
    }
#undef DEMON_CASE
    return hipErrorInvalidValue;
}

// what the kernels' instances assume of a layer
bool stream_conv_ok(const MfmaParams& p, int mode, int in_fmt)
{
    if (p.cout % 8 != 0) return false;
    switch (mode) {
        case MODE_ACT: return (p.ntaps - 1) * p.tap_step <= MAXSPAN && p.nchunks % 2 == 0 && in_fmt != OP_BF16X2;
        case MODE_RES: return p.ntaps == 1 && p.nchunks % 2 == 0;
        case MODE_DOWN: return p.ntaps == 4 && in_fmt != OP_BF16X2;
        case MODE_PART: return p.ntaps == 4 && in_fmt != OP_BF16X2 && p.part && p.nchunks % (2 * kConvParts) == 0;
        default: return p.ntaps == 2;
    }
}

}  // namespace

hipError_t launch_conv_stream(MfmaParams p, int mode, int in_fmt, int emit, int rows, long long ncols, int n_slots, int call_slots, long long max_small, hipStream_t stream)
{
    if (rows % 128 != 0 || ncols < 1 || !stream_conv_ok(p, mode, in_fmt)) return hipErrorInvalidValue;
    // Tile of a launch: the cheapest by (workgroups on the busiest of 256 CUs) x (time of one K step of 32, in ns, with one
    // workgroup on a CU or with several), as measured on the dilated convs of 256 to 1024 channels with 200 to 100000
    // columns.  A CU takes weights in at some 45 bytes per clock, so small tiles are bound by that and large ones by their
    // MFMAs.  Launches of more than `max_small` 128 x 128 tiles take no smaller one (kDown: 128 x 64, unless `max_small` is 0).
    struct Tile { int mt, nt; double alone, shared; };
    static const Tile kFixed[7] = {{32, 32, 25, 26}, {64, 64, 57, 70}, {64, 80, 65, 85}, {64, 96, 73, 97}, {128, 64, 90, 122}, {128, 128, 185, 212}, {256, 128, 335, 368}};
    // Any number of taps: the small tiles have fewer k-steps in flight and the LDS of the largest span.  Measured with 3 to 15 taps
    // (1024-channel dilated conv of 9 taps in us, tiles in this order: 75 frames 49, 32, 34, 37, 40, 56; 250 frames 149, 72, 97, 75, 63,
    // 64; 750 frames 430, 198, 258, 227, 168, 161; 1500 frames 847, 388, 488, 435, 297, 270).
    static const Tile kAny[6] = {{32, 32, 75, 45}, {64, 64, 90, 78}, {64, 80, 100, 115}, {64, 96, 105, 132}, {128, 64, 120, 118}, {128, 128, 177, 190}};
    const bool any = mode == MODE_ACT && p.ntaps != 7 && p.ntaps != 1;
    // Seven taps: the tall tile (conv_tall_kernel) where there is more than one round of its two workgroups per CU: below, it is faster by
    // itself (8 windows of 64 frames, 512 channels: 93 -> 87 us) but not beside the other group's launches (1899 -> 1925 us a call).  From 513
    // to some 640 workgroups in windows it is the other way round: ten windows of 64 frames (620) 108 -> 122 us a launch, the call 2348 -> 2355, which
    // is within the noise.  Calls in us, without / with: 700 frames in one window 2615 / 2581, in 11 windows of 64 2703 / 2666, 800 frames 2880 / 2855 (4 of
    // 200: 2901 / 2868), 1000 3660 / 3624, 1024 in 32 of 32 3920 / 3878, 1536 in 24 of 64 5646 / 5572.
    const bool tall_ok = mode == MODE_ACT && p.ntaps == 7 && rows % 256 == 0 && in_fmt != OP_BF16X2 && (emit == 1 || emit == 3);
    // What a K step costs is not all: the 1x1 and transposed convs have few of them and long epilogues, which the 128 x 128 tile has nothing
    // to cover with where a CU has one workgroup, and which 80 and 96 columns (no power of two) make longer; a transposed conv's
    // 64-row tiles write half runs.  Fitted to the fastest tile of 498 1x1 and 280 transposed launches (13 to 1500 frames, windows of 13
    // to 750): 9.89 -> 9.79 and 9.51 -> 9.39 ms in all (9.69 and 9.34 with the fastest each); transposed conv to 512 channels of a 10 s
    // clip 63 -> 50 us, 1x1 conv of 1024 channels 20 -> 16.  Two operand planes take the same tables, not fitted to them: their calls gain what
    // those of one plane do (3 s window 528 -> 495 us, 10 s clip 1269 -> 1156 with everything else that came with them).
    static const Tile kRes[6] = {{32, 32, 25, 26}, {64, 64, 57, 70}, {64, 80, 65, 90}, {64, 96, 73, 100}, {128, 64, 90, 118}, {128, 128, 245, 190}};
    static const Tile kUp[6] = {{32, 32, 25, 26}, {64, 64, 57, 80}, {64, 80, 65, 95}, {64, 96, 73, 120}, {128, 64, 90, 120}, {128, 128, 240, 190}};
    // Strided convs of up to 512 merged channels: a column is two rows of the activation tile, so 128 columns leave room for two workgroups
    // on a CU and 64 for three, which are faster at any size beyond one round (81 launches: 3.49 -> 3.15 ms; 128 -> 256 channels,
    // 60 s clip by itself, 347 -> 297 us; the whole 60 s encode, two groups at the power limit, does not change).  Longer K loops hide it, in us, 64 /
    // 128 columns, at 48000 columns: 256 merged channels 36 / 38, 384 48 / 50, 512 107 / 110, 640 72 / 71, 768 159 / 154, 1024 203 / 186 and 218 / 200,
    // 1536 298 / 267 (these to 512 channels, 256, 384 and 640 to 256).  A single chunk (64 channels) is bound by its output: 97 us against 117.
    static const Tile kDown[6] = {{32, 32, 25, 26}, {64, 64, 57, 70}, {64, 80, 65, 85}, {64, 96, 73, 97}, {128, 64, 90, 95}, {128, 128, 185, 212}};
    const bool down = mode == MODE_DOWN && p.nchunks > 1 && p.cin <= 512;
    const Tile* kTiles = any ? kAny : down ? kDown : mode == MODE_RES ? kRes : mode == MODE_UP ? kUp : kFixed;
    const bool large = (ncols + 127) / 128 * (rows / 128) * call_slots > max_small;
    int best = 5;
    double cheapest = 0;
    for (int t = large ? (down && max_small > 0 ? 4 : 5) : 0; t < (tall_ok ? 7 : 6); ++t) {
        const long long wgs = (ncols + kTiles[t].nt - 1) / kTiles[t].nt * (rows / kTiles[t].mt) * call_slots * (mode == MODE_PART ? kConvParts : 1);
        if (t == 6 && wgs <= 512) continue;
        const double cost = wgs <= 256 ? kTiles[t].alone : wgs <= 1024 ? (double)((wgs + 255) / 256) * kTiles[t].shared : (wgs / 256.0 + 0.5) * kTiles[t].shared;
        if (cheapest == 0 || cost < cheapest) { cheapest = cost; best = t; }
    }
    const bool tall = best == 6;
    const int mt = kTiles[best].mt, nt = kTiles[best].nt;
    StreamGrid sg;
    const int panels = rows / std::max(128, mt);
    // split of the 8 XCDs over panels and column tiles with the least to read per XCD
    const double w = (double)p.w_bytes, x = (double)ncols * n_slots * (mode == MODE_DOWN ? 2 : 1) * p.cin * 2.0;
    double least = 0;
    sg.xm = 0;
    for (int xm = 1; xm <= (mode == MODE_PART ? 1 : 8); xm *= 2) {
        if (panels % xm != 0) continue;
        const double cost = w / xm + x * xm / 8;
        if (sg.xm == 0 || cost < least) { sg.xm = xm; least = cost; }
    }
    sg.xn = mode == MODE_PART ? 1 : 8 / sg.xm;
    sg.mper = panels / sg.xm * std::max(1, 128 / mt);
    const long long ntiles = ((ncols + nt - 1) / nt + sg.xn - 1) / sg.xn * sg.xn;
    const long long wgs_x = ntiles * (rows / mt) * (mode == MODE_PART ? kConvParts : 1);
    if (wgs_x > 0x7fffffffll) return hipErrorInvalidValue;
    const dim3 grid((unsigned)wgs_x, (unsigned)n_slots);
    if (tall) {
#define DEMON_TALL(SPAN_, IN_) if (in_fmt == IN_ && 6 * p.tap_step <= SPAN_) { \
        hipLaunchKernelGGL((conv_tall_kernel<SPAN_, IN_>), grid, dim3(256), 0, stream, p, sg, emit == 3); \
        return hipGetLastError(); \
    }
        DEMON_TALL(32, OP_BF16) DEMON_TALL(32, OP_F16) DEMON_TALL(MAXSPAN, OP_BF16) DEMON_TALL(MAXSPAN, OP_F16)
#undef DEMON_TALL
        return hipErrorInvalidValue;
    }
    switch (best) {
        case 0: return launch_tile<1, 2, 2, 1>(p, sg, mode, in_fmt, emit, grid, stream);
        case 1: return launch_tile<1, 4, 4, 1>(p, sg, mode, in_fmt, emit, grid, stream);
        case 2: return launch_tile<1, 5, 4, 1>(p, sg, mode, in_fmt, emit, grid, stream);
        case 3: return launch_tile<1, 6, 4, 1>(p, sg, mode, in_fmt, emit, grid, stream);
        case 4: return launch_tile<2, 4, 4, 1>(p, sg, mode, in_fmt, emit, grid, stream);
        default: return launch_tile<2, 8, 4, 1>(p, sg, mode, in_fmt, emit, grid, stream);
    }
}

}  // namespace demon
