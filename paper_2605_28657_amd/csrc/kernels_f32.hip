// fp32 reference-precision path: implicit GEMM on the fp32 MFMA (v_mfma_f32_16x16x4_f32), and a plain kernel for the
// shapes that do not tile.
// Same layer semantics as the bf16 path (decoder layers of the benchmark description):
//   conv  : y[n, o] = b[o] + sum_t sum_i W[o,i,t] x[n + (t - (k-1)/2) d, i]      (x = 0 outside the slot)
//   convT : y[m s - p + phi, o] = b[o] + sum_j sum_i W[i,o,phi + j s] x[m - j, i],  j in {0,1}, p = s/2
//   convS : y[n, o] = b[o] + sum_t sum_i W[o,i,t] x[n s - p + t, i],  t in 0..2s-1, p = s/2   (the encoder's strided conv)
// x is the already activated input: every producer writes, beside the residual stream h, the operand of the layer that
// consumes it (Snake with that layer's parameters), so no layer needs a pass of its own for its Snake.
#include <algorithm>

#include "device_common.h"

namespace demon {

// GEMM rows of a layer: cout for Conv1d, s*cout (row mu = phi*cout + o) for ConvTranspose1d.
static long long gemm_rows(int cout, int stride) { return stride > 0 ? (long long)stride * cout : cout; }

constexpr int F_KC = 32;                     // input channels per stage
// Layers that run on the MFMA kernel: whole 16-row tiles, whole 16-channel groups (the second half of the last 32-channel
// stage may be padding), four consecutive channels per lane.  The others take the plain kernel.
static bool f32_tiles(int cin, int cout, int stride)
{
    return gemm_rows(cout, stride) % 16 == 0 && cin % 16 == 0 && cout % 4 == 0;
}

// Packed weights.  MFMA layout: [row tile of 16][stage = (32-channel chunk, tap)][16-channel group g][lane][4]: lane
// (j = lane % 16, q = lane / 16) holds row j, channels 32 chunk + 16 g + 4 q + {0..3}, which is the operand of four
// consecutive MFMAs (k-slot q of MFMA e is channel 4 q + e; the activations are read in the same order).  Plain layout:
// [tap][cin][M] (M fastest) so that consecutive lanes read consecutive words.
size_t packed_f32_count(int cin, int cout, int ntaps, int stride)
{
    const size_t M = (size_t)gemm_rows(cout, stride);
    if (f32_tiles(cin, cout, stride)) return M * ntaps * ((cin + F_KC - 1) / F_KC) * F_KC;
    return (size_t)ntaps * cin * M;
}

void pack_f32(const float* w, int cin, int cout, int ntaps, int stride, float* dst)
{
    const int M = (int)gemm_rows(cout, stride);
    auto weight = [&](int mu, int i, int t) -> float {
        if (stride == 0) return w[((size_t)mu * cin + i) * ntaps + t];
        const int phi = mu / cout, o = mu - phi * cout;
        return w[((size_t)i * cout + o) * (2 * stride) + phi + t * stride];
    };
    if (!f32_tiles(cin, cout, stride)) {
        for (int t = 0; t < ntaps; ++t)
            for (int i = 0; i < cin; ++i)
                for (int mu = 0; mu < M; ++mu) dst[((size_t)t * cin + i) * M + mu] = weight(mu, i, t);
        return;
    }
    size_t pos = 0;
    for (int mt = 0; mt < M / 16; ++mt)
        for (int c = 0; c < (cin + F_KC - 1) / F_KC; ++c)
            for (int t = 0; t < ntaps; ++t)
                for (int g = 0; g < 2; ++g)
                    for (int lane = 0; lane < 64; ++lane)
                        for (int e = 0; e < 4; ++e) {
                            const int i = c * F_KC + g * 16 + (lane / 16) * 4 + e;
                            dst[pos++] = i < cin ? weight(mt * 16 + lane % 16, i, t) : 0.f;
                        }
}

// ---- MFMA kernel: strided convs, and dilated convs of other kernel sizes or wider spans than the streamed kernel below takes.
// Bound by the fp32 matrix rate (157 TFLOP/s nominal, 154 measured on a library product; 16 of the bf16 rate), at which a
// 16 x 16 x 4 MFMA takes 32 cycles for two 256-byte operands: LDS and L2 bandwidth are no concern, so the weights go
// straight from global memory to registers in fragment order (no LDS, no barrier per tap) and only the activation tile
// is staged, once per 32-channel chunk for all taps.  Four waves of TM x TN accumulator tiles of 16 rows x 16 columns.
// The tile is chosen per launch for the number of CUs it fills (see launch_conv_f32); every tile shape adds in the same
// order -- chunk, tap, 16-channel group, MFMA -- so results do not depend on the choice, nor on the place in a tile.
// All requests are unconditional and through descriptors (out of range where there is nothing to read), so that the compiler
// can count them: a wait for one block of weights leaves the later ones in flight, but for the first stage of a round of PF
// (the compiler leads a round's early end through the loop's own test; a round without one, with the remainder after the loop,
// takes 210 registers instead of 130 and is 4 % slower).  The epilogue takes the accumulators from LDS: sinf is too long to
// unroll, and a dynamic index into registers had put those of the 128 x 128 tile in scratch memory, written back every stage.
// 3 s window of the x1920 stack 3297 -> 2974 us, 2 s clip of the x32 one 153 -> 138, when all layers ran on this kernel.

// A value that every lane holds, in scalar registers: comparisons of 64-bit values are vector instructions, and a descriptor made of
// their results is not scalar (see weight_rsrc).
static __device__ __forceinline__ long long uniform64(long long v)
{
    return (long long)((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)v) |
                       (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32);
}

constexpr int f32_rows_in_registers(int nt) { return nt <= 32 ? 96 : nt <= 64 ? 128 : 192; }      // rows of the next chunk held

template <int TM, int TN, int WM, int WN>
__global__ __launch_bounds__(256) void conv_f32_mfma_kernel(ConvArgs a, int nchunks, int xrows)
{
    static_assert(WM * WN == 4, "four waves");
    constexpr int MT = 16 * TM * WM, NT = 16 * TN * WN, KC = F_KC;
    constexpr int PF = TM * TN >= 16 ? 2 : 4;      // weight stages in flight: a small tile's stage is shorter than an L2 access
    constexpr int XI = f32_rows_in_registers(NT) / 32;      // 32 rows per pass
    extern __shared__ __attribute__((aligned(16))) float xs[];          // [rows][32], 16-byte pieces XOR-swizzled by the row

    const Slot s = a.slots[blockIdx.y];
    const int M = a.cout;
    const long long nrows_in = (long long)s.len * a.r_in;
    // output rows that later layers read: the interior widened by `margin`, clamped to the window
    const long long r_out = a.down > 0 ? a.r_in / a.down : a.r_in;
    const long long out_lo = max(0ll, s.crop * r_out - a.margin);
    const long long out_hi = min(s.len * r_out, (s.crop + s.n_int) * r_out + a.margin);
    const long long n0 = uniform64(out_lo + (long long)blockIdx.x * NT);
    if (n0 >= out_hi) return;                            // (also an empty window: a gated clip)
    const int m0 = blockIdx.z * MT;

    // input row of (column n, tap t): n XS + base + t step
    const int XS = a.down > 0 ? a.down : 1;
    const int step = a.down > 0 ? 1 : a.dil, base = a.down > 0 ? -(a.down / 2) : -((a.ntaps - 1) / 2) * a.dil;
    const long long row0 = n0 * XS + base;               // first staged row (in the window; may be negative)

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN, j = lane & 15, q = lane >> 4;
    const int piece = tid & 7, xr0 = tid >> 3;
    // the tile's rows inside the window: rows outside read as zero
    const long long row_lo = uniform64(max(0ll, row0)), row_hi = uniform64(max(row_lo, min(nrows_in, row0 + xrows)));
    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc((const float*)a.x + ((long long)s.row0 * a.r_in + row_lo) * a.cin,
                                                  (unsigned)(row_hi - row_lo) * (unsigned)a.cin * 4u);
    const int before = (int)(row_lo - row0);             // staged rows before the window; their offsets wrap: out of range

    const int nstages = nchunks * a.ntaps;
    const __amdgpu_buffer_rsrc_t rs_w = weight_rsrc(a.w, (unsigned)M * (unsigned)nstages * (KC * 4u));
    static_assert(PF * 2048u <= kWeightSlack, "stages ahead");
    const unsigned tile_bytes = (unsigned)nstages * 2048u;
    unsigned w_off[TM];
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) w_off[mi] = (unsigned)(m0 / 16 + wm * TM + mi) * tile_bytes + lane * 16u;   // past M: the slack or out of range, not used

    u32x4 wr[PF][TM][2];
    auto load_w = [&](u32x4 (&r)[TM][2], int stage) __attribute__((always_inline)) {
        const unsigned blk = (unsigned)stage * 2048u;
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int g = 0; g < 2; ++g) r[mi][g] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, w_off[mi], blk + g * 1024u, 0);
    };
    auto fetch = [&](int chunk, int row) __attribute__((always_inline)) -> u32x4 {
        const int c = chunk * KC + piece * 4;            // past the last channel: out of range
        return __builtin_amdgcn_raw_buffer_load_b128(rs_x, c < a.cin ? (unsigned)((row - before) * a.cin + c) * 4u : 0xf8000000u, 0, 0);
    };
    u32x4 rx[XI];
    auto load_x = [&](int chunk) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < XI; ++it) rx[it] = fetch(chunk, xr0 + it * 32);
    };
    auto put = [&](int row, u32x4 v) __attribute__((always_inline)) { *reinterpret_cast<u32x4*>(&xs[row * KC + ((piece ^ (row & 7)) * 4)]) = v; };
    auto store_x = [&](int chunk) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < XI; ++it) put(xr0 + it * 32, rx[it]);
        for (int row = xr0 + XI * 32; row < xrows; row += 32) put(row, fetch(chunk, row));
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) {
        const int mu = m0 + (wm * TM + mi) * 16 + 4 * q;
        f32x4 b = {0.f, 0.f, 0.f, 0.f};
        if (mu < M) b = *reinterpret_cast<const f32x4*>(a.bias + mu);
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = b;
    }

    load_x(0);
#pragma unroll
    for (int u = 0; u < PF; ++u) load_w(wr[u], u);
    store_x(0);
    __syncthreads();

    load_x(1);
    int tap = 0, chunk = 0;
    auto body = [&](int stage, int u) __attribute__((always_inline)) {
        if (tap == a.ntaps) {
            tap = 0;
            ++chunk;
            __syncthreads();
            store_x(chunk);
            __syncthreads();
            load_x(chunk + 1);
        }
        const int off = tap * step;
        int row[TN];
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) row[ni] = ((wn * TN + ni) * 16 + j) * XS + off;
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            f32x4 xv[TN];
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) xv[ni] = *reinterpret_cast<const f32x4*>(&xs[row[ni] * KC + (((g * 4 + q) ^ (row[ni] & 7)) * 4)]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int mi = 0; mi < TM; ++mi)
#pragma unroll
                    for (int ni = 0; ni < TN; ++ni)
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(wr[u][mi][g][e]), xv[ni][e], acc[mi][ni], 0, 0, 0);
        }
        load_w(wr[u], stage + PF);
        ++tap;
    };
    for (int stage = 0; stage < nstages; stage += PF)
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            if (stage + u >= nstages) break;
            body(stage + u, u);
        }

    // ---- epilogue: lane (j, q) holds rows 4 q + {0..3} of column j of every accumulator tile
    __syncthreads();                                     // the activation tile has been read
    f32x4* own = reinterpret_cast<f32x4*>(xs) + wave * (TM * TN * 64) + lane;
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) own[(mi * TN + ni) * 64] = acc[mi][ni];
    const long long rowbase_o = (long long)s.row0 * r_out;
    const float* res = (const float*)a.res;
#pragma unroll 1
    for (int i = 0; i < TM * TN; ++i) {
        const int mu = m0 + (wm * TM + i / TN) * 16 + 4 * q;
        const long long n = n0 + (wn * TN + i % TN) * 16 + j;
        if (mu >= M || n >= out_hi) continue;
        const size_t idx = (size_t)(rowbase_o + n) * a.cout + mu;
        f32x4 v = own[i * 64];
        if (res) v += *reinterpret_cast<const f32x4*>(res + idx);
        if (a.y) *reinterpret_cast<f32x4*>((float*)a.y + idx) = v;
        if (a.ya) {
            const f32x4 al = *reinterpret_cast<const f32x4*>(a.out_alpha + mu), ib = *reinterpret_cast<const f32x4*>(a.out_inv_beta + mu);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = snake_precise(v[e], al[e], ib[e]);
            *reinterpret_cast<f32x4*>((float*)a.ya + idx) = v;
        }
    }
}

// ---- Streamed kernel: the dilated and 1x1 convs of seven taps and one, and the transposed convs.
// What bound the kernel above on them: one wave per SIMD waited for the fragments of every 16-channel group and for two barriers a chunk,
// its tiles filled the CUs badly, and the 1x1 convs of the narrow levels moved the branch tensor to memory and back.  Here a wave
// owns 16 rows of TN column tiles; the weights of the next RS groups wait in registers, the fragments of the next group are
// requested between the MFMAs of this one, across the stages too (the only barrier of a stage stands before its last group), and the
// next stage's activations are in the other buffer by then.  TN is chosen per launch so that the rounds of the CUs are full.
// Per launch of a 75-frame window (dilated / 1x1 / transposed), with an event after each, 4 to 5 us: 1024 channels 149 / 37 / 12 -> 119 / 28 / 12 us,
// 512 channels 154 / 36 / 99 -> 133 / 31 / 96, 256 channels 150 / 43 / 100 -> 133 / 34 / 86, 128 channels 143 / 50 / 102 -> 139 / 41 / 91: 93 to 125
// TFLOP/s on the dilated ones where a large library product reaches 153.
// FUSE: a residual unit of 32 or 64 channels in one kernel.  Snake of the accumulators goes to LDS, [column][channel], and is the
// operand of the 1x1 conv: no branch tensor in memory and one launch instead of two (64 channels, 75 frames: 117 as two before, 100
// as two streamed ones, 88).  At 128 channels it is no faster (159 against 163) and at 256 slower (172 against 154): a workgroup that holds
// all channels is alone on its CU, so its Snake and its memory accesses are not covered by another's MFMAs.
// The sums are those of the kernel above, in the same order (chunk, tap, 16-channel group, MFMA), so a value depends neither on the
// tile nor on which kernel computed it.
struct F32Grid { int xm, xn, mper; };        // split of the 8 XCDs over row tiles and column tiles; row tiles of an XCD
struct F32Second {                           // FUSE: the 1x1 conv of the unit and what follows it
    const float* w; const float* bias; const float* res; float* y; float* ya;
    const float* out_alpha; const float* out_inv_beta;
};

// words of LDS: two activation tiles; after the K loop the branch tensor (FUSE), then every lane's own results
constexpr int f32_lds(int span, int nch, int tn, int wm, int wn, bool fuse)
{
    const int rpp = 32 / nch, x = 2 * ((16 * tn * wn + span + rpp - 1) / rpp * rpp) * (F_KC * nch + 4);
    const int m = fuse ? 16 * tn * wn * (16 * wm + 4) : 0, own = tn * 1024;
    return std::max(x, std::max(m, own));
}
// workgroups (waves per SIMD) that its registers and the LDS are meant for
constexpr int f32_occupancy(int tn, int lds) { return std::min(tn <= 4 ? 4 : 3, 163840 / (4 * lds)); }

template <int NTAPS, int SPAN, int NCH, int TN, int WM, int WN, bool FUSE>
__global__ __launch_bounds__(256, f32_occupancy(TN, f32_lds(SPAN, NCH, TN, WM, WN, FUSE))) void conv_f32_stream_kernel(ConvArgs a, F32Second u, F32Grid sg, int nstages)
{
    static_assert(WM * WN == 4, "four waves");
    constexpr int MT = 16 * WM, NT = 16 * TN * WN, KX = F_KC * NCH;
    constexpr int LDR = KX + 4;                             // row of the activation tile: an odd number of pieces, no bank conflicts
    constexpr int SEGS = KX / 4, RPP = 256 / SEGS, X_ITERS = (NT + SPAN + RPP - 1) / RPP, XR = X_ITERS * RPP;
    constexpr int F = 2 * NTAPS * NCH;                      // groups of 16 channels in a stage
    constexpr int RS = NTAPS == 7 ? 7 : F;                  // groups of weights in flight
    constexpr int X_FLOATS = XR * LDR, LDM = MT + 4;
    static_assert(F % RS == 0 && F % 2 == 0 && RS * 1024u <= kWeightSlack, "static indices; groups requested past the layer's end");
    __shared__ __attribute__((aligned(16))) float xs[f32_lds(SPAN, NCH, TN, WM, WN, FUSE)];

    const Slot s = a.slots[blockIdx.y];
    constexpr bool UP = NTAPS == 2;
    const int M = UP ? a.stride * a.cout : a.cout;
    const long long nrows_in = (long long)s.len * a.r_in;
    const long long r_out = UP ? (long long)a.r_in * a.stride : (long long)a.r_in;
    const long long out_lo = max(0ll, s.crop * r_out - a.margin);
    const long long out_hi = min(s.len * r_out, (s.crop + s.n_int) * r_out + a.margin);
    if (out_hi <= out_lo) return;                           // an empty window (a gated clip)
    const long long col_lo = UP ? (out_lo + a.stride / 2) / a.stride : out_lo;
    const long long col_hi = UP ? (out_hi - 1 + a.stride / 2) / a.stride + 1 : out_hi;
    const int xcd = (int)((blockIdx.x + blockIdx.y) & 7u), q8 = (int)(blockIdx.x >> 3);
    const int mtile = xcd % sg.xm + sg.xm * (q8 % sg.mper), ntile = xcd / sg.xm + sg.xn * (q8 / sg.mper);
    const long long n0 = uniform64(col_lo + (long long)ntile * NT);
    if (n0 >= col_hi) return;
    const int m0 = mtile * MT;

    // input row of (column n, tap t): n + base + t step
    const int step = UP ? -1 : a.dil, base = UP ? 0 : -((NTAPS - 1) / 2) * a.dil;
    const int minoff = UP ? -1 : base;
    const long long row0 = n0 + minoff;                     // first staged row (in the window; may be negative)

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN, j = lane & 15, q = lane >> 4;
    const int piece = tid % SEGS, xr0 = tid / SEGS;
    // the tile's rows inside the window: rows outside read as zero
    const long long row_lo = uniform64(max(0ll, row0)), row_hi = uniform64(max(row_lo, min(nrows_in, row0 + XR)));
    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc((const float*)a.x + ((long long)s.row0 * a.r_in + row_lo) * a.cin,
                                                  (unsigned)(row_hi - row_lo) * (unsigned)a.cin * 4u);
    const int before = (int)(row_lo - row0);                // staged rows before the window; their offsets wrap: out of range
    const unsigned tile_bytes = (unsigned)nstages * (F * 1024u);
    const __amdgpu_buffer_rsrc_t rs_w = weight_rsrc(a.w, (unsigned)(M / 16) * tile_bytes);
    const unsigned w_voff = (unsigned)(m0 / 16 + wm) * tile_bytes + lane * 16u;        // past M: the slack or out of range, not used

    u32x4 wr[RS];
    auto load_w = [&](int slot, unsigned group) __attribute__((always_inline)) { wr[slot] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, w_voff, group * 1024u, 0); };
    u32x4 rx[X_ITERS];
    const unsigned x_voff = (unsigned)((xr0 - before) * a.cin + piece * 4) * 4u, x_step = (unsigned)(RPP * a.cin) * 4u;
    auto load_x = [&](int stage) __attribute__((always_inline)) {
        const int c = stage * KX + piece * 4;               // past the last channel: out of range
        const unsigned off = c < a.cin ? x_voff + (unsigned)(stage * KX) * 4u : 0xf8000000u;
#pragma unroll
        for (int it = 0; it < X_ITERS; ++it) rx[it] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, c < a.cin ? off + it * x_step : off, 0, 0);
    };
    auto store_x = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < X_ITERS; ++it) *reinterpret_cast<u32x4*>(&xs[buf + (xr0 + it * RPP) * LDR + piece * 4]) = rx[it];
    };

    load_x(0);
#pragma unroll
    for (int g = 0; g < RS; ++g) load_w(g, g);
    const int mu = m0 + wm * 16 + 4 * q;                    // lane (j, q) holds rows mu + {0..3} of column j of every accumulator tile
    f32x4 acc[TN], b = {0.f, 0.f, 0.f, 0.f};
    if (mu < M) b = *reinterpret_cast<const f32x4*>(a.bias + (UP ? mu % a.cout : mu));
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) acc[ni] = b;
    store_x(0);
    load_x(1);
    __syncthreads();

    u32x4 xv[2][TN];
    const unsigned char* const lds = reinterpret_cast<const unsigned char*>(xs);
    const unsigned x_at = (unsigned)((wn * (16 * TN) + j + base - minoff) * LDR + 4 * q) * 4u;
    const int tap_bytes = step * (LDR * 4);
    unsigned at = x_at;                                     // of the group that is read: one running register
    auto read_x = [&](int ni, int off) __attribute__((always_inline)) -> u32x4 { return *reinterpret_cast<const u32x4*>(lds + at + off + ni * (64 * LDR)); };
    // One group: its MFMAs, a read of the next group's fragments after every fourth (in front of them all, they would leave the
    // matrix core idle while they issue)
    auto group = [&](u32x4 w, const u32x4 (&x)[TN], auto read) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 4 * TN; ++k) {
            const int e = k / TN, ni = k % TN;
            acc[ni] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w[e]), __uint_as_float(x[ni][e]), acc[ni], 0, 0, 0);
            if (k % 4 == 0) read(k / 4);
            __builtin_amdgcn_sched_barrier(0);
        }
        // a use of the whole fragments: taken apart, they would be read as single words
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) asm volatile("" :: "v"(x[ni]));
    };
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) xv[0][ni] = read_x(ni, 0);
    int buf = 0;
#pragma unroll 1
    for (int stage = 0; stage < nstages; ++stage) {
        const int next = X_FLOATS - buf;
#pragma unroll
        for (int f = 0; f < F; ++f) {
            if (f == F - 2) { store_x(next); load_x(stage + 2); }
            int off = 0;
            if (f + 1 == F) {
                __syncthreads();                            // the next stage is complete; nobody reads this one any more
                at = x_at + 4u * next;                           // (after the last stage: read, not used)
            } else {
                off = (f + 1) / (2 * NTAPS) * (4 * F_KC) + (f + 1) % 2 * 64;
                if ((f + 1) % 2 == 0) { at += (f + 1) / 2 % NTAPS == 0 ? -(NTAPS - 1) * tap_bytes : tap_bytes; asm volatile("" : "+v"(at)); }
            }
            group(wr[f % RS], xv[f & 1], [&](int ni) __attribute__((always_inline)) { xv[(f + 1) & 1][ni] = read_x(ni, off); });
            load_w(f % RS, (unsigned)(stage * F + f + RS));
        }
        buf = next;
    }

    if constexpr (FUSE) {
        // ---- Snake on the accumulators (a loop over LDS: sinf is too long to unroll), then the 1x1 conv on [column][channel]
        constexpr int KG = MT / 16;
        const __amdgpu_buffer_rsrc_t rs_p = weight_rsrc(u.w, (unsigned)(MT * MT) * 4u);
        u32x4 wp[KG];
#pragma unroll
        for (int g = 0; g < KG; ++g) wp[g] = __builtin_amdgcn_raw_buffer_load_b128(rs_p, (unsigned)wm * (KG * 1024u) + lane * 16u, g * 1024u, 0);
        float* mid = xs + (wn * (16 * TN) + j) * LDM + mu;
        const f32x4 al = *reinterpret_cast<const f32x4*>(a.out_alpha + mu), ib = *reinterpret_cast<const f32x4*>(a.out_inv_beta + mu);
        b = *reinterpret_cast<const f32x4*>(u.bias + mu);
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) {
            *reinterpret_cast<f32x4*>(mid + ni * 16 * LDM) = acc[ni];
            acc[ni] = b;
        }
#pragma unroll 1
        for (int ni = 0; ni < TN; ++ni) {
            f32x4* const m = reinterpret_cast<f32x4*>(mid + ni * 16 * LDM);
            f32x4 v = *m;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = snake_precise(v[e], al[e], ib[e]);
            *m = v;
        }
        __syncthreads();
        const float* mr = xs + (wn * (16 * TN) + j) * LDM + 4 * q;
        auto read_m = [&](int ni, int g) __attribute__((always_inline)) -> u32x4 { return *reinterpret_cast<const u32x4*>(mr + ni * 16 * LDM + 16 * g); };
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) xv[0][ni] = read_m(ni, 0);
#pragma unroll
        for (int g = 0; g < KG; ++g) {
            group(wp[g], xv[g & 1], [&](int ni) __attribute__((always_inline)) { if (g + 1 < KG) xv[(g + 1) & 1][ni] = read_m(ni, g + 1); });
        }
        __syncthreads();                                    // the branch tensor has been read
    }

    // ---- epilogue: every lane takes its results from LDS in a loop
    f32x4* own = reinterpret_cast<f32x4*>(xs) + wave * (TN * 64) + lane;
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) own[ni * 64] = acc[ni];
    if (mu >= M) return;
    const float* const res = FUSE ? u.res : (const float*)a.res;
    float* const y = FUSE ? u.y : (float*)a.y;
    float* const ya = FUSE ? u.ya : (float*)a.ya;
    const float* const oal = FUSE ? u.out_alpha : a.out_alpha;
    const float* const oib = FUSE ? u.out_inv_beta : a.out_inv_beta;
    const int phi = UP ? mu / a.cout : 0, o = mu - phi * a.cout;
    f32x4 al = {0.f, 0.f, 0.f, 0.f}, ib = al, r = al;
    if (ya) { al = *reinterpret_cast<const f32x4*>(oal + o); ib = *reinterpret_cast<const f32x4*>(oib + o); }
    const long long col = n0 + wn * (16 * TN) + j;          // of the first tile; the tiles are 16 columns apart
    const long long n_step = UP ? 16ll * a.stride : 16ll, idx_step = n_step * a.cout;
    long long n = UP ? col * a.stride - a.stride / 2 + phi : col, idx = ((long long)s.row0 * r_out + n) * a.cout + o;
    if (res && n >= 0 && n < out_hi) r = *reinterpret_cast<const f32x4*>(res + idx);
#pragma unroll 1
    for (int ni = 0; ni < TN; ++ni, n += n_step, idx += idx_step) {
        f32x4 v = own[ni * 64], next = r;
        // the next tile's residual is requested before this one's Snake
        if (res && ni + 1 < TN && n + n_step >= 0 && n + n_step < out_hi) next = *reinterpret_cast<const f32x4*>(res + idx + idx_step);
        if (n >= 0 && n < out_hi) {
            if (res) v += r;
            if (y) *reinterpret_cast<f32x4*>(y + idx) = v;
            if (ya) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = snake_precise(v[e], al[e], ib[e]);
                *reinterpret_cast<f32x4*>(ya + idx) = v;
            }
        }
        r = next;
    }
}

// ---- plain kernel, one thread per output element, for the shapes f32_tiles() turns away (or whose taps span more rows
// than the LDS holds; those weights are packed for the MFMA kernel, hence the two ways to find one).
static __device__ __forceinline__ float f32_weight(const ConvArgs& a, const float* w, bool tiles, int M, int nchunks, int mu, int i, int t)
{
    if (!tiles) return w[((size_t)t * a.cin + i) * M + mu];
    const int c = i / F_KC, g = (i / 16) & 1, q = (i / 4) & 3;
    return w[((((size_t)(mu / 16) * nchunks + c) * a.ntaps + t) * 2 + g) * 256 + (q * 16 + mu % 16) * 4 + (i & 3)];
}

// grid: (ceil(ncols*M/256), n_slots); thread -> (col, mu), mu fastest.
__global__ __launch_bounds__(256) void conv_f32_kernel(ConvArgs a, bool tiles, int nchunks)
{
    const Slot s = a.slots[blockIdx.y];
    const int M = a.stride > 0 ? a.stride * a.cout : a.cout;
    const long long nrows_in = (long long)s.len * a.r_in;
    // output rows that later layers read: the interior widened by `margin`, clamped to the window
    const long long r_out = a.stride > 0 ? (long long)a.r_in * a.stride : a.down > 0 ? a.r_in / a.down : a.r_in;
    const long long out_lo = max(0ll, s.crop * r_out - a.margin);
    const long long out_hi = min(s.len * r_out, (s.crop + s.n_int) * r_out + a.margin);
    if (out_hi <= out_lo) return;                        // an empty window (a gated clip)
    const long long col_lo = a.stride > 0 ? (out_lo + a.stride / 2) / a.stride : out_lo;
    const long long col_hi = a.stride > 0 ? (out_hi - 1 + a.stride / 2) / a.stride + 1 : out_hi;
    const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
    if (e >= (col_hi - col_lo) * M) return;
    const long long col = col_lo + e / M;
    const int mu = (int)(e % M);
    const long long rowbase_in = (long long)s.row0 * a.r_in;
    const float* __restrict__ x = (const float*)a.x;
    const float* __restrict__ w = (const float*)a.w;

    float acc = 0.f;
    const int half = (a.ntaps - 1) / 2;
    for (int t = 0; t < a.ntaps; ++t) {
        const long long r = a.stride > 0 ? col - t : a.down > 0 ? col * a.down - a.down / 2 + t : col + (long long)(t - half) * a.dil;
        if (r < 0 || r >= nrows_in) continue;
        const float* xr = x + (size_t)(rowbase_in + r) * a.cin;
        for (int i = 0; i < a.cin; ++i) acc = fmaf(f32_weight(a, w, tiles, M, nchunks, mu, i, t), xr[i], acc);
    }

    int o = mu;
    long long n = col;
    long long rowbase_out = a.down > 0 ? (long long)s.row0 * r_out : rowbase_in;
    if (a.stride > 0) {
        const int phi = mu / a.cout;
        o = mu - phi * a.cout;
        n = col * a.stride - a.stride / 2 + phi;
        if (n < 0 || n >= nrows_in * a.stride) return;
        rowbase_out = rowbase_in * a.stride;
    }
    float v = acc + a.bias[o];
    const size_t idx = (size_t)(rowbase_out + n) * a.cout + o;
    if (a.res) v += ((const float*)a.res)[idx];
    if (a.y) ((float*)a.y)[idx] = v;
    if (a.ya) ((float*)a.ya)[idx] = snake_precise(v, a.out_alpha[o], a.out_inv_beta[o]);
}

// Split of the XCDs over row tiles and column tiles with the least to read per XCD, and the grid.
static bool f32_stream_grid(const ConvArgs& a, long long M, long long ncols, int mt, int nt, F32Grid* sg, dim3* grid)
{
    const long long mtiles = (M + mt - 1) / mt;
    const double w = (double)M * a.ntaps * a.cin, x = (double)ncols * a.n_slots * a.cin;
    double least = 0;
    sg->xm = 0;
    for (int xm = 1; xm <= 8; xm *= 2) {
        if (mtiles % xm) continue;
        const double cost = w / xm + x * xm / 8;
        if (sg->xm == 0 || cost < least) { sg->xm = xm; least = cost; }
    }
    sg->xn = 8 / sg->xm;
    sg->mper = (int)(mtiles / sg->xm);
    const long long ntiles = ((ncols + nt - 1) / nt + sg->xn - 1) / sg->xn * sg->xn;
    if (ntiles * mtiles > 0x7fffffffll) return false;
    *grid = dim3((unsigned)(ntiles * mtiles), (unsigned)a.n_slots);
    return true;
}

// Column tiles of a wave: those with the least (workgroups on the busiest CU) x (tiles of a wave), times what a tile of that width costs
// beyond its MFMAs.  Measured on a 75-frame window, dilated conv in us, TN 1, 2, 3, 4, 6, 8: 1024 channels 116, 109, 157, 109, 157, 206; 512
// channels 132, 136, 123, 158, 158, 206; 256 channels 134, 126, 140, 137, 125, 160; 128 channels 140, 130, 129, 130, 131, 143.
static int f32_choose(const int* tns, int n, int wn, long long mtiles, long long ncols, long long slots)
{
    int best = 0;
    double least = 0;
    for (int i = 0; i < n; ++i) {
        const int tn = tns[i];
        const long long wgs = (ncols + 16 * tn * wn - 1) / (16 * tn * wn) * mtiles * slots;
        const double cost = (wgs <= 1024 ? (double)((wgs + 255) / 256) : wgs / 256.0 + 0.5) * (tn + 0.1);
        if (best == 0 || cost < least) { best = tn; least = cost; }
    }
    return best;
}

// Columns a launch computes in its longest window.
static long long f32_columns(const ConvArgs& a)
{
    const long long r_out = a.down > 0 ? (long long)a.r_in / a.down : (long long)a.r_in * (a.stride > 0 ? a.stride : 1);
    const long long out_rows = std::min((long long)a.max_int * r_out + 2ll * a.margin, (long long)a.max_len * r_out);
    return a.stride > 0 ? out_rows / a.stride + 2 : out_rows;
}

static bool f32_streams(const ConvArgs& a)
{
    const long long span = (long long)(a.ntaps - 1) * a.dil;
    return f32_tiles(a.cin, a.cout, a.stride) && a.down == 0 &&
           (a.stride > 0 ? a.ntaps == 2 : a.ntaps == 1 || (a.ntaps == 7 && span <= 64)) &&
           (unsigned long long)gemm_rows(a.cout, a.stride) * ((a.cin + F_KC - 1) / F_KC) * a.ntaps * F_KC * 4 < 0xf0000000ull;
}

template <int NTAPS, int SPAN, int NCH>
static hipError_t launch_f32_stream(const ConvArgs& a, hipStream_t stream)
{
    const long long M = gemm_rows(a.cout, a.stride), ncols = f32_columns(a);
    const int nstages = (a.cin + F_KC - 1) / F_KC / NCH;
    const bool narrow = (M + 31) / 32 * 32 < (M + 63) / 64 * 64;        // a 64-row tile would be half empty
    static const int kTn[5] = {1, 2, 3, 4, 6}, kTnNarrow[3] = {1, 2, 4};
    const int mt = narrow ? 32 : 64, wn = narrow ? 2 : 1;
    const int tn = narrow ? f32_choose(kTnNarrow, 3, 2, (M + 31) / 32, ncols, a.n_slots) : f32_choose(kTn, 5, 1, (M + 63) / 64, ncols, a.n_slots);
    F32Grid sg;
    dim3 grid;
    if (!f32_stream_grid(a, M, ncols, mt, 16 * tn * wn, &sg, &grid)) return hipErrorInvalidValue;
    const F32Second none = {};
#define DEMON_F32(TN, WM, WN) if (tn == TN && wn == WN) { \
        hipLaunchKernelGGL((conv_f32_stream_kernel<NTAPS, SPAN, NCH, TN, WM, WN, false>), grid, dim3(256), 0, stream, a, none, sg, nstages); \
        return hipGetLastError(); \
    }
    DEMON_F32(1, 4, 1) DEMON_F32(2, 4, 1) DEMON_F32(3, 4, 1) DEMON_F32(4, 4, 1) DEMON_F32(6, 4, 1)
    DEMON_F32(1, 2, 2) DEMON_F32(2, 2, 2) DEMON_F32(4, 2, 2)
#undef DEMON_F32
    return hipErrorInvalidValue;
}

// A residual unit runs as one kernel where a workgroup holds all its channels (the streamed kernel's comment has the figures).
bool res_unit_f32_fuses(const ConvArgs& d, const ConvArgs& p)
{
    return (d.cout == 32 || d.cout == 64) && d.cin == d.cout && p.cin == d.cout && p.cout == d.cout && d.ntaps == 7 && p.ntaps == 1 && f32_streams(d) && f32_streams(p);
}

// d: the dilated conv (its out_alpha / out_inv_beta: Snake between the convolutions), p: the 1x1 conv.  d.x is read by neighbouring
// tiles: p.ya must be another buffer; p.y may be p.res.
hipError_t launch_res_unit_f32(const ConvArgs& d, const ConvArgs& p, hipStream_t stream)
{
    if (!res_unit_f32_fuses(d, p) || !d.out_alpha || !d.out_inv_beta || p.ya == d.x || p.y == d.x || (!p.y && !p.ya) || (p.ya && (!p.out_alpha || !p.out_inv_beta))) return hipErrorInvalidValue;
    static const int kTn[3] = {1, 2, 3};         // 64 channels, 75 frames, in us: 95, 88, 89; 4 tiles 97, 6 tiles 92, 8 tiles 102
    const int wn = d.cout == 32 ? 2 : 1, tn = f32_choose(kTn, 3, wn, 1, f32_columns(d), d.n_slots);
    const F32Second u = {(const float*)p.w, p.bias, (const float*)p.res, (float*)p.y, (float*)p.ya, p.out_alpha, p.out_inv_beta};
    F32Grid sg;
    dim3 grid;
    if (!f32_stream_grid(d, d.cout, f32_columns(d), d.cout, 16 * tn * wn, &sg, &grid)) return hipErrorInvalidValue;
#define DEMON_F32(TN, WM, WN) if (tn == TN && wn == WN) { \
        if (6 * d.dil <= 24) hipLaunchKernelGGL((conv_f32_stream_kernel<7, 24, 1, TN, WM, WN, true>), grid, dim3(256), 0, stream, d, u, sg, d.cin / F_KC); \
        else hipLaunchKernelGGL((conv_f32_stream_kernel<7, 64, 1, TN, WM, WN, true>), grid, dim3(256), 0, stream, d, u, sg, d.cin / F_KC); \
        return hipGetLastError(); \
    }
    DEMON_F32(1, 2, 2) DEMON_F32(2, 2, 2) DEMON_F32(3, 2, 2) DEMON_F32(1, 4, 1) DEMON_F32(2, 4, 1) DEMON_F32(3, 4, 1)
#undef DEMON_F32
    return hipErrorInvalidValue;
}

// Tile of a launch that the streamed kernel does not take (strided convs, other kernel sizes): each workgroup's four waves take TM x TN
// tiles each on one CU, so a launch lasts about ceil(workgroups / CUs) x TM x TN; the largest tile wins unless a smaller one
// shortens that (factor: the smaller tiles read more weights per MFMA).
hipError_t launch_conv_f32(const ConvArgs& a, hipStream_t stream)
{
    constexpr int kCUs = 256;
    constexpr size_t kMaxLds = 64 * 1024;          // dynamic LDS a launch may ask for without an attribute
    const long long M = gemm_rows(a.cout, a.stride);
    if (a.down > 0 && (a.stride != 0 || a.ntaps != 2 * a.down || a.r_in % a.down != 0 || a.res)) return hipErrorInvalidValue;
    if ((!a.y && !a.ya) || (a.ya && (!a.out_alpha || !a.out_inv_beta))) return hipErrorInvalidValue;
    const long long ncols = f32_columns(a);
    const int nchunks = (a.cin + F_KC - 1) / F_KC;
    const bool tiles = f32_tiles(a.cin, a.cout, a.stride);
    if (f32_streams(a)) {
        if (a.stride > 0) return launch_f32_stream<2, 1, 1>(a, stream);
        if (a.ntaps == 7) return 6 * a.dil <= 24 ? launch_f32_stream<7, 24, 1>(a, stream) : launch_f32_stream<7, 64, 1>(a, stream);
        return nchunks % 2 == 0 ? launch_f32_stream<1, 0, 2>(a, stream) : launch_f32_stream<1, 0, 1>(a, stream);
    }
    const unsigned long long w_bytes = (unsigned long long)M * nchunks * a.ntaps * F_KC * 4;
    if (tiles && a.stride == 0 && w_bytes < 0xf0000000ull) {
        struct Tile { int tm, tn, wm, wn; double factor; };
        static const Tile kTiles[5] = {{4, 4, 2, 2, 1.0}, {2, 2, 2, 2, 1.1}, {2, 2, 1, 4, 1.1}, {1, 2, 4, 1, 1.25}, {1, 1, 2, 2, 1.4}};
        const int xs = a.down > 0 ? a.down : 1;
        const long long span = (long long)(a.ntaps - 1) * (a.down > 0 ? 1 : a.dil);
        int best = -1;
        double best_cost = 0;
        dim3 grid;
        int xrows = 0;
        for (int i = 0; i < 5; ++i) {
            const Tile& t = kTiles[i];
            const int mt = 16 * t.tm * t.wm, nt = 16 * t.tn * t.wn;
            const long long rows = (long long)xs * (nt - 1) + 1 + span;
            if ((size_t)rows * F_KC * 4 > kMaxLds) continue;
            const long long gx = (ncols + nt - 1) / nt, gz = (M + mt - 1) / mt, wgs = gx * gz * a.n_slots;
            if (gx > 0x7fffffffll || gz > 65535) continue;
            const double cost = (double)((wgs + kCUs - 1) / kCUs) * t.tm * t.tn * t.factor;
            if (best < 0 || cost < best_cost) {
                best = i; best_cost = cost; xrows = (int)rows;
                grid = dim3((unsigned)gx, (unsigned)a.n_slots, (unsigned)gz);
            }
        }
        // the activation tile, then the accumulators
        size_t lds = 0;
        if (best >= 0) {
            const Tile& t = kTiles[best];
            lds = std::max((size_t)std::max(xrows, f32_rows_in_registers(16 * t.tn * t.wn)) * F_KC * 4, (size_t)(4 * t.tm * t.tn) * 1024);
        }
        switch (best) {
            case 0: hipLaunchKernelGGL((conv_f32_mfma_kernel<4, 4, 2, 2>), grid, dim3(256), lds, stream, a, nchunks, xrows); return hipGetLastError();
            case 1: hipLaunchKernelGGL((conv_f32_mfma_kernel<2, 2, 2, 2>), grid, dim3(256), lds, stream, a, nchunks, xrows); return hipGetLastError();
            case 2: hipLaunchKernelGGL((conv_f32_mfma_kernel<2, 2, 1, 4>), grid, dim3(256), lds, stream, a, nchunks, xrows); return hipGetLastError();
            case 3: hipLaunchKernelGGL((conv_f32_mfma_kernel<1, 2, 4, 1>), grid, dim3(256), lds, stream, a, nchunks, xrows); return hipGetLastError();
            case 4: hipLaunchKernelGGL((conv_f32_mfma_kernel<1, 1, 2, 2>), grid, dim3(256), lds, stream, a, nchunks, xrows); return hipGetLastError();
            default: break;
        }
    }
    const long long blocks = (ncols * M + 255) / 256;
    if (blocks > 0x7fffffffll) return hipErrorInvalidValue;
    hipLaunchKernelGGL(conv_f32_kernel, dim3((unsigned)blocks, (unsigned)a.n_slots), dim3(256), 0, stream, a, tiles, nchunks);
    return hipGetLastError();
}

}  // namespace demon
