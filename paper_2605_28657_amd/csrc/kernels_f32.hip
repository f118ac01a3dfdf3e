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

// ---- MFMA kernel.
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
// 3 s window of the x1920 stack 3297 -> 2974 us, 2 s clip of the x32 one 153 -> 138.
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
    const int M = a.stride > 0 ? a.stride * a.cout : a.cout;
    const long long nrows_in = (long long)s.len * a.r_in;
    // output rows that later layers read: the interior widened by `margin`, clamped to the window
    const long long r_out = a.stride > 0 ? (long long)a.r_in * a.stride : a.down > 0 ? a.r_in / a.down : (long long)a.r_in;
    const long long out_lo = max(0ll, s.crop * r_out - a.margin);
    const long long out_hi = min(s.len * r_out, (s.crop + s.n_int) * r_out + a.margin);
    if (out_hi <= out_lo) return;                        // an empty window (a gated clip)
    const long long col_lo = a.stride > 0 ? (out_lo + a.stride / 2) / a.stride : out_lo;
    const long long col_hi = a.stride > 0 ? (out_hi - 1 + a.stride / 2) / a.stride + 1 : out_hi;
    const long long n0 = uniform64(col_lo + (long long)blockIdx.x * NT);
    if (n0 >= col_hi) return;
    const int m0 = blockIdx.z * MT;

    // input row of (column n, tap t): n XS + base + t step
    const int XS = a.down > 0 ? a.down : 1;
    const int step = a.stride > 0 ? -1 : a.down > 0 ? 1 : a.dil;
    const int base = a.stride > 0 ? 0 : a.down > 0 ? -(a.down / 2) : -((a.ntaps - 1) / 2) * a.dil;
    const int last = base + (a.ntaps - 1) * step, minoff = min(base, last);
    const long long row0 = n0 * XS + minoff;             // first staged row (in the window; may be negative)

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
        if (mu < M) b = *reinterpret_cast<const f32x4*>(a.bias + mu % a.cout);
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
        const int off = base + tap * step - minoff;
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
        const int phi = a.stride > 0 ? mu / a.cout : 0, o = mu - phi * a.cout;
        const long long col = n0 + (wn * TN + i % TN) * 16 + j;
        const long long n = a.stride > 0 ? col * a.stride - a.stride / 2 + phi : col;
        if (mu >= M || n < 0 || n >= out_hi) continue;
        const size_t idx = (size_t)(rowbase_o + n) * a.cout + o;
        f32x4 v = own[i * 64];
        if (res) v += *reinterpret_cast<const f32x4*>(res + idx);
        if (a.y) *reinterpret_cast<f32x4*>((float*)a.y + idx) = v;
        if (a.ya) {
            const f32x4 al = *reinterpret_cast<const f32x4*>(a.out_alpha + o), ib = *reinterpret_cast<const f32x4*>(a.out_inv_beta + o);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = snake_precise(v[e], al[e], ib[e]);
            *reinterpret_cast<f32x4*>((float*)a.ya + idx) = v;
        }
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

// Tile of a launch: each workgroup's four waves take TM x TN tiles each on one CU, so a launch lasts about
// ceil(workgroups / CUs) x TM x TN; the largest tile wins unless a smaller one shortens that (factor: the smaller tiles
// read more weights per MFMA).  One 3 s window of the x1920 stack: 128 x 128 tiles for the levels of 256 channels and
// below, 64 x 64 and 64 x 32 above them, where 128 x 128 tiles would leave most CUs idle.
hipError_t launch_conv_f32(const ConvArgs& a, hipStream_t stream)
{
    constexpr int kCUs = 256;
    constexpr size_t kMaxLds = 64 * 1024;          // dynamic LDS a launch may ask for without an attribute
    const long long M = gemm_rows(a.cout, a.stride);
    if (a.down > 0 && (a.stride != 0 || a.ntaps != 2 * a.down || a.r_in % a.down != 0 || a.res)) return hipErrorInvalidValue;
    if ((!a.y && !a.ya) || (a.ya && (!a.out_alpha || !a.out_inv_beta))) return hipErrorInvalidValue;
    const long long r_out = a.down > 0 ? (long long)a.r_in / a.down : (long long)a.r_in * (a.stride > 0 ? a.stride : 1);
    const long long out_rows = std::min((long long)a.max_int * r_out + 2ll * a.margin, (long long)a.max_len * r_out);
    const long long ncols = a.stride > 0 ? out_rows / a.stride + 2 : out_rows;
    const int nchunks = (a.cin + F_KC - 1) / F_KC;
    const bool tiles = f32_tiles(a.cin, a.cout, a.stride);
    const unsigned long long w_bytes = (unsigned long long)M * nchunks * a.ntaps * F_KC * 4;
    if (tiles && w_bytes < 0xf0000000ull) {
        struct Tile { int tm, tn, wm, wn; double factor; };
        static const Tile kTiles[5] = {{4, 4, 2, 2, 1.0}, {2, 2, 2, 2, 1.1}, {2, 2, 1, 4, 1.1}, {1, 2, 4, 1, 1.25}, {1, 1, 2, 2, 1.4}};
        const int xs = a.down > 0 ? a.down : 1;
        const long long span = (long long)(a.ntaps - 1) * (a.stride > 0 || a.down > 0 ? 1 : a.dil);
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
