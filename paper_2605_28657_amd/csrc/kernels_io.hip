// Window gather, output head, 16-bit render and the debug tap (HBM-bound kernels).
//
// gather : step 1 of the windowed decode of paper section 3.6 (extend each window by its margins):
//          copies latent frames [lo, hi) of every window into its slot, transposing to time-major.
// head   : Snake -> Conv1d(k, C -> out_channels) -> tanh, the last layer of the decoder.
//          Step 3 (trim the margins, keep the frame-aligned interior, write the interiors side by side into the clip's
//          waveform) is its store address; a kernel of its own for that cost 46 MB of traffic per 60 s clip and a launch (5 us of a
//          0.5 s window).  Only the 16-bit render is a pass of its own.
#include <algorithm>
#include <type_traits>

#include "device_common.h"

namespace demon {

template <typename T> __device__ __forceinline__ float load_act(const T* p);
template <> __device__ __forceinline__ float load_act<float>(const float* p) { return *p; }
template <> __device__ __forceinline__ float load_act<uint16_t>(const uint16_t* p) { return bf16_bits_to_f32(*p); }
template <> __device__ __forceinline__ float load_act<_Float16>(const _Float16* p) { return (float)*p; }

// ---------------------------------------------------------------------------------- gather
// The latent is [clip, channel, frame] (frames fastest), the slots are time-major [frame, channel]: a workgroup moves a
// tile of 32 frames x 16 channels through LDS, reading runs of consecutive frames of one channel and writing runs of
// consecutive channels of one frame.  With `xa` (bf16 path) it writes the first layer's
// MFMA operand directly, snake(latent) in operand format fmt; without it (fp32 path) the same in fp32.
// Bound by latencies: window, latent, parameters and flags are all requested before the first is waited for, two elements a thread.
// (Tiles of 64 x 64, one workgroup for a playback window, went through 16 waits of a load each: 8.1 us for 25 frames, 2.5
// now; 0.5 s window 212.0 -> 206.6 us, 3 s 438 -> 431, 2 s clip of the x32 stack 105.5 -> 100.6.)
constexpr int GATHER_R = 32, GATHER_C = 16;

template <typename T>
__global__ __launch_bounds__(256) void gather_kernel(const T* __restrict__ latent, float* __restrict__ x0,
                                                     uint16_t* __restrict__ xa, int fmt, long long lo_off,
                                                     const float* __restrict__ alpha, const float* __restrict__ inv_beta,
                                                     int c0, int n_frames, const Slot* __restrict__ slots,
                                                     const int* __restrict__ skip, Slot* __restrict__ gated)
{
    fp16_saturate_on();
    constexpr int RS = 256 / GATHER_R, CS = 256 / GATHER_C;           // channels, frames a pass
    __shared__ float tile[GATHER_C][GATHER_R + 1];
    const int cbase = blockIdx.z * GATHER_C, c = cbase + threadIdx.x % GATHER_C;
    const float al = c < c0 ? alpha[c] : 0.f, ib = c < c0 ? inv_beta[c] : 0.f;
    Slot s = slots[blockIdx.y];
    const int r0 = blockIdx.x * GATHER_R;
    const int lane = threadIdx.x % GATHER_R, sub = threadIdx.x / GATHER_R;
    float v[GATHER_C / RS];
#pragma unroll
    for (int u = 0; u < GATHER_C / RS; ++u) {
        const int cc = cbase + sub + u * RS;
        v[u] = cc < c0 && r0 + lane < s.len ? load_act<T>(latent + ((size_t)s.clip * c0 + cc) * n_frames + s.lo + r0 + lane) : 0.f;
    }
    if (skip) {
        // decode gate: the launches after this one read the table that the first workgroup of every window writes here
        if (skip[s.clip] != 0) { s.len = 0; s.n_int = 0; s.crop = 0; }
        if (blockIdx.x == 0 && blockIdx.z == 0 && threadIdx.x == 0) gated[blockIdx.y] = s;
    }
    if (r0 >= s.len) return;
#pragma unroll
    for (int u = 0; u < GATHER_C / RS; ++u) tile[sub + u * RS][lane] = v[u];
    __syncthreads();
    if (c >= c0) return;
#pragma unroll
    for (int u = 0; u < GATHER_R / CS; ++u) {
        const int rr = threadIdx.x / GATHER_C + u * CS, r = r0 + rr;
        if (r >= s.len) break;
        const float raw = tile[threadIdx.x % GATHER_C][rr];
        const size_t idx = ((size_t)s.row0 + r) * c0 + c;
        if (!xa) { x0[idx] = snake_precise(raw, al, ib); continue; }
        const float a = keep_f32(snake_fast(raw, al, ib));
        if (fmt == OP_F16) {
            xa[idx] = __builtin_bit_cast(uint16_t, (_Float16)a);
        } else {
            const uint16_t hi = f32_to_bf16_bits(a);
            xa[idx] = hi;
            if (fmt == OP_BF16X2) xa[lo_off + idx] = f32_to_bf16_bits(a - bf16_bits_to_f32(hi));
        }
    }
}

hipError_t launch_gather(const void* latent, float* x0, int c0, int n_frames, bool bf16,
                         const Slot* slots, int n_slots, int max_len, hipStream_t stream,
                         uint16_t* xa, int xa_fmt, long long xa_lo_off, const float* alpha, const float* inv_beta,
                         const int* skip, Slot* gated)
{
    if (!alpha || !inv_beta || (skip && !gated)) return hipErrorInvalidValue;
    dim3 grid((unsigned)((max_len + GATHER_R - 1) / GATHER_R), (unsigned)n_slots, (unsigned)((c0 + GATHER_C - 1) / GATHER_C));
    if (bf16)
        hipLaunchKernelGGL(gather_kernel<uint16_t>, grid, dim3(256), 0, stream, (const uint16_t*)latent, x0, xa, xa_fmt, xa_lo_off, alpha, inv_beta, c0, n_frames, slots, skip, gated);
    else
        hipLaunchKernelGGL(gather_kernel<float>, grid, dim3(256), 0, stream, (const float*)latent, x0, xa, xa_fmt, xa_lo_off, alpha, inv_beta, c0, n_frames, slots, skip, gated);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------- encoder stem
// First layer of the encoder (the mirror of the head): Conv1d(k, channels -> C) + bias straight from the planar fp32
// waveform of every extended window into the time-major residual stream, and with `ya` the activated operand of the
// next layer as well.  Samples outside the window read as zero (the convolution's zero padding: the window is encoded
// as if it were a whole clip).  Two kernels: on the fp32 MFMA for whole groups of 64 channels and at most 16 taps x channels, a row
// per thread for the others.
constexpr int STEM_MAXK = 15 * 8;                 // taps x channels held in registers

// Row per thread: a thread loads its k x channels samples once (consecutive threads, consecutive samples) and walks the C output
// channels in groups of 8, whose weights are the same for every thread (scalar loads).
template <typename TY, int KCH>
__global__ __launch_bounds__(256) void stem_kernel(const float* __restrict__ wave, TY* __restrict__ y, void* __restrict__ ya_,
                                                   int ya_fmt, const float* __restrict__ w /*[k][ch][C]*/,
                                                   const float* __restrict__ bias, const float* __restrict__ alpha,
                                                   const float* __restrict__ inv_beta, int ch, int C, int k, int S,
                                                   int n_frames, int margin, const Slot* __restrict__ slots)
{
    if (sizeof(TY) == 2) fp16_saturate_on();
    std::conditional_t<sizeof(TY) == 4, float, uint16_t>* __restrict__ ya = static_cast<std::conditional_t<sizeof(TY) == 4, float, uint16_t>*>(ya_);
    const Slot s = slots[blockIdx.y];
    const long long nrows = (long long)s.len * S;
    const long long out_lo = max(0ll, (long long)s.crop * S - margin);
    const long long out_hi = min(nrows, (long long)(s.crop + s.n_int) * S + margin);
    const long long n = out_lo + (long long)blockIdx.x * 256 + threadIdx.x;
    if (n >= out_hi) return;
    const int half = (k - 1) / 2;
    const float* clip = wave + (size_t)s.clip * ch * ((size_t)n_frames * S) + (long long)s.lo * S;
    float xv[KCH];                                 // [tap][channel]
#pragma unroll
    for (int q = 0; q < KCH; ++q) {
        const int t = q / ch, c = q - t * ch;
        const long long m = n + t - half;
        xv[q] = (q < k * ch && m >= 0 && m < nrows) ? clip[(size_t)c * ((size_t)n_frames * S) + m] : 0.f;
    }
    const size_t row = ((size_t)s.row0 * S + n) * C;
    for (int g = 0; g < C / 8; ++g) {
        float acc[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = bias[8 * g + e];
#pragma unroll
        for (int q = 0; q < KCH; ++q) {
            if (q >= k * ch) break;                // uniform
            const float* wt = w + (size_t)q * C + 8 * g;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] = fmaf(wt[e], xv[q], acc[e]);
        }
        const size_t idx = row + 8 * g;
        if constexpr (sizeof(TY) == 4) {
            *reinterpret_cast<float4*>(&y[idx]) = make_float4(acc[0], acc[1], acc[2], acc[3]);
            *reinterpret_cast<float4*>(&y[idx + 4]) = make_float4(acc[4], acc[5], acc[6], acc[7]);
            if (ya) {
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[e] = snake_precise(acc[e], alpha[8 * g + e], inv_beta[8 * g + e]);
                *reinterpret_cast<float4*>(&ya[idx]) = make_float4(acc[0], acc[1], acc[2], acc[3]);
                *reinterpret_cast<float4*>(&ya[idx + 4]) = make_float4(acc[4], acc[5], acc[6], acc[7]);
            }
        } else {
            f16x8 hv;
#pragma unroll
            for (int e = 0; e < 8; ++e) hv[e] = (_Float16)acc[e];
            *reinterpret_cast<f16x8*>(&y[idx]) = hv;
            if (ya) {
                // the next layer's operand is Snake of the STORED value
                u32x4 o;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float a0 = keep_f32(snake_fast((float)hv[2 * q], alpha[8 * g + 2 * q], inv_beta[8 * g + 2 * q]));
                    const float a1 = keep_f32(snake_fast((float)hv[2 * q + 1], alpha[8 * g + 2 * q + 1], inv_beta[8 * g + 2 * q + 1]));
                    o[q] = ya_fmt == OP_F16 ? pack_f16x2(a0, a1) : pack_bf16x2(a0, a1);
                }
                *reinterpret_cast<u32x4*>(&ya[idx]) = o;
            }
        }
    }
}

// Bound by its stores: 64 channels, 7 taps, stereo are 128 bytes out, 8 in and 1.8 kFLOP a row, a third of the stores' time on the fp32 MFMA.
// The kernel above waits for its scalar weight loads and stores 16 bytes of a row at a time, 128 apart.  From there to here, with an event after the launch:
// 60 s clip 246 -> 139 us (3.2 TB/s), 75 frames 29 -> 20; the encodes 6.40 -> 6.27 ms, 477 -> 469 us.
// A wave holds the weights of 64 channels as the row operand of v_mfma_f32_16x16x4 (4 tiles of 16 channels x KS steps of 4 values of
// K = [tap][channel]); the samples of a workgroup's rows lie in LDS, and a lane reads one per step.  Row 4 q + e of tile mi is
// channel 32 (mi / 2) + 8 q + 4 (mi % 2) + e, so that a lane ends with 8 consecutive channels of a row twice and four lanes store 64 bytes of it.
// Sums start at the bias and take the products in the order of K, as above: the same bits.
constexpr int STEM_ROWS = 512, STEM_KCH = 16;     // rows of a workgroup; taps x channels at most

template <typename TY>
__global__ __launch_bounds__(256) void stem_mfma_kernel(const float* __restrict__ wave, TY* __restrict__ y, void* __restrict__ ya_,
                                                        int ya_fmt, const float* __restrict__ w /*[k][ch][C]*/,
                                                        const float* __restrict__ bias, const float* __restrict__ alpha,
                                                        const float* __restrict__ inv_beta, int ch, int C, int k, int S,
                                                        int n_frames, int margin, const Slot* __restrict__ slots)
{
    if (sizeof(TY) == 2) fp16_saturate_on();
    constexpr int KS = STEM_KCH / 4;
    extern __shared__ float xs[];                  // [channel][STEM_ROWS + k - 1]
    std::conditional_t<sizeof(TY) == 4, float, uint16_t>* __restrict__ ya = static_cast<std::conditional_t<sizeof(TY) == 4, float, uint16_t>*>(ya_);
    const Slot s = slots[blockIdx.y];
    const long long nrows = (long long)s.len * S;
    const long long out_lo = max(0ll, (long long)s.crop * S - margin);
    const long long out_hi = min(nrows, (long long)(s.crop + s.n_int) * S + margin);
    const long long n0 = out_lo + (long long)blockIdx.x * STEM_ROWS;
    if (n0 >= out_hi) return;
    const int half = (k - 1) / 2, span = STEM_ROWS + k - 1;
    const float* clip = wave + (size_t)s.clip * ch * ((size_t)n_frames * S) + (long long)s.lo * S;
    for (int c = 0; c < ch; ++c)
        for (int m = threadIdx.x; m < span; m += 256) {
            const long long at = n0 - half + m;
            xs[c * span + m] = at >= 0 && at < nrows ? clip[(size_t)c * ((size_t)n_frames * S) + at] : 0.f;
        }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, i = lane & 15, q = lane >> 4;
    const int cg = blockIdx.z * 64;
    // K value 4 st + q of this lane; past k x ch: 0 x 0
    float a[KS][4];
    int off[KS];
#pragma unroll
    for (int st = 0; st < KS; ++st) {
        const int kk = 4 * st + q, t = kk / ch;
        const bool in = kk < k * ch;
        off[st] = in ? (kk - t * ch) * span + t : 0;
#pragma unroll
        for (int mi = 0; mi < 4; ++mi)
            a[st][mi] = in ? w[(size_t)kk * C + cg + 32 * (mi >> 1) + 8 * (i >> 2) + 4 * (mi & 1) + (i & 3)] : 0.f;
    }
    f32x4 b[4];
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) b[mi] = *reinterpret_cast<const f32x4*>(bias + cg + 32 * (mi >> 1) + 8 * q + 4 * (mi & 1));
    f32x4 al[4], ib[4];
    if (ya) {
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) {
            al[mi] = *reinterpret_cast<const f32x4*>(alpha + cg + 32 * (mi >> 1) + 8 * q + 4 * (mi & 1));
            ib[mi] = *reinterpret_cast<const f32x4*>(inv_beta + cg + 32 * (mi >> 1) + 8 * q + 4 * (mi & 1));
        }
    }
    __syncthreads();
    const int nr = (int)min((long long)STEM_ROWS, out_hi - n0);
    for (int r0 = wv * 16; r0 < nr; r0 += 64) {
        float x[KS];
#pragma unroll
        for (int st = 0; st < KS; ++st) x[st] = 4 * st + q < k * ch ? xs[off[st] + r0 + i] : 0.f;
        f32x4 acc[4];
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) acc[mi] = b[mi];
#pragma unroll
        for (int st = 0; st < KS; ++st)
#pragma unroll
            for (int mi = 0; mi < 4; ++mi) acc[mi] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[st][mi], x[st], acc[mi], 0, 0, 0);
        if (r0 + i >= nr) continue;
        const size_t idx = ((size_t)s.row0 * S + n0 + r0 + i) * C + cg + 8 * q;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            if constexpr (sizeof(TY) == 4) {
                *reinterpret_cast<f32x4*>(&y[idx + 32 * p]) = acc[2 * p];
                *reinterpret_cast<f32x4*>(&y[idx + 32 * p + 4]) = acc[2 * p + 1];
                if (ya) {
#pragma unroll
                    for (int m = 2 * p; m < 2 * p + 2; ++m)
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[m][e] = snake_precise(acc[m][e], al[m][e], ib[m][e]);
                    *reinterpret_cast<f32x4*>(&ya[idx + 32 * p]) = acc[2 * p];
                    *reinterpret_cast<f32x4*>(&ya[idx + 32 * p + 4]) = acc[2 * p + 1];
                }
            } else {
                f16x8 hv;
#pragma unroll
                for (int e = 0; e < 8; ++e) hv[e] = (_Float16)acc[2 * p + e / 4][e % 4];
                *reinterpret_cast<f16x8*>(&y[idx + 32 * p]) = hv;
                if (ya) {
                    // the next layer's operand is Snake of the STORED value
                    u32x4 o;
#pragma unroll
                    for (int e = 0; e < 8; e += 2) {
                        const int m = 2 * p + e / 4;
                        const float a0 = keep_f32(snake_fast((float)hv[e], al[m][e % 4], ib[m][e % 4]));
                        const float a1 = keep_f32(snake_fast((float)hv[e + 1], al[m][e % 4 + 1], ib[m][e % 4 + 1]));
                        o[e / 2] = ya_fmt == OP_F16 ? pack_f16x2(a0, a1) : pack_bf16x2(a0, a1);
                    }
                    *reinterpret_cast<u32x4*>(&ya[idx + 32 * p]) = o;
                }
            }
        }
    }
}

hipError_t launch_stem(const float* wave, void* y, bool y_half, void* ya, int ya_fmt, const float* w, const float* bias,
                       const float* alpha, const float* inv_beta, int ch, int C, int k, int S, int n_frames, int margin,
                       const Slot* slots, int n_slots, int max_len, int max_int, hipStream_t stream)
{
    if (C % 8 != 0 || k < 1 || (k & 1) == 0 || margin < 0 || k * ch > STEM_MAXK) return hipErrorInvalidValue;
    if (ya && (ya_fmt == OP_BF16X2 || !alpha || !inv_beta)) return hipErrorInvalidValue;
    const long long rows = std::min((long long)max_int * S + 2ll * margin, (long long)max_len * S);
    if (C % 64 == 0 && k * ch <= STEM_KCH) {
        const dim3 tiles((unsigned)((rows + STEM_ROWS - 1) / STEM_ROWS), (unsigned)n_slots, (unsigned)(C / 64));
        const size_t lds = (size_t)ch * (STEM_ROWS + k - 1) * sizeof(float);
#define DEMON_STEM(TY_) hipLaunchKernelGGL((stem_mfma_kernel<TY_>), tiles, dim3(256), lds, stream, wave, (TY_*)y, ya, ya_fmt, w, bias, alpha, \
                                           inv_beta, ch, C, k, S, n_frames, margin, slots)
        if (y_half) DEMON_STEM(hres_t); else DEMON_STEM(float);
#undef DEMON_STEM
        return hipGetLastError();
    }
    dim3 grid((unsigned)((rows + 255) / 256), (unsigned)n_slots);
    // stereo with a 7-tap stem holds 14 samples per thread; anything up to 15 taps x 8 channels takes the large form
#define DEMON_STEM(TY_, KCH_) hipLaunchKernelGGL((stem_kernel<TY_, KCH_>), grid, dim3(256), 0, stream, wave, (TY_*)y, ya, ya_fmt, w, bias, alpha, \
                                                 inv_beta, ch, C, k, S, n_frames, margin, slots)
    if (y_half) { if (k * ch <= 16) DEMON_STEM(hres_t, 16); else DEMON_STEM(hres_t, STEM_MAXK); }
    else { if (k * ch <= 16) DEMON_STEM(float, 16); else DEMON_STEM(float, STEM_MAXK); }
#undef DEMON_STEM
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------- encoder: sampling step + trim + scatter
// Last step of the windowed encode: of every window's moments [rows = frames, 2 C0] (mean | log-variance) keep the
// interior frames, write them to moments_out [clip, 2 C0, n_frames] (fp32) and the sampled latent
// z = mean + exp(logvar / 2) eps (the sampling step on the output moments of Table III; eps drawn by the caller, z = mean
// without eps) to latent_out [clip, C0, n_frames] in the path's latent type.  Either output may be absent.
// PARTS: the moments are the sums of the parts that the last convolution's K was cut into (fp32, one rounding to half).
template <typename TM, typename TZ, bool PARTS>
__global__ __launch_bounds__(256) void sample_kernel(TM* __restrict__ m, const float* __restrict__ parts, const float* __restrict__ eps,
                                                     float* __restrict__ moments_out, TZ* __restrict__ latent_out,
                                                     int C0, int n_frames, const Slot* __restrict__ slots)
{
    if (PARTS) fp16_saturate_on();
    const Slot s = slots[blockIdx.y];
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= s.n_int * C0) return;
    const int fi = e / C0, c = e - fi * C0;
    const size_t row = (size_t)s.row0 + s.crop + fi;
    const int f = s.begin + fi;
    float mean, lv;
    if constexpr (PARTS) {
        float a[2][kConvParts];
#pragma unroll
        for (int k = 0; k < kConvParts; ++k)
#pragma unroll
            for (int h = 0; h < 2; ++h) a[h][k] = parts[(row * kConvParts + k) * (2 * C0) + h * C0 + c];
        mean = a[0][0]; lv = a[1][0];
#pragma unroll
        for (int k = 1; k < kConvParts; ++k) { mean += a[0][k]; lv += a[1][k]; }
        const TM hm = (TM)keep_f32(mean), hl = (TM)keep_f32(lv);
        mean = (float)hm; lv = (float)hl;
        if (m) { m[row * (2 * C0) + c] = hm; m[row * (2 * C0) + C0 + c] = hl; }
    } else {
        mean = load_act<TM>(m + row * (2 * C0) + c);
        lv = load_act<TM>(m + row * (2 * C0) + C0 + c);
    }
    if (moments_out) {
        moments_out[((size_t)s.clip * 2 * C0 + c) * n_frames + f] = mean;
        moments_out[((size_t)s.clip * 2 * C0 + C0 + c) * n_frames + f] = lv;
    }
    if (latent_out) {
        const size_t zi = ((size_t)s.clip * C0 + c) * n_frames + f;
        const float z = eps ? fmaf(expf(0.5f * lv), eps[zi], mean) : mean;
        if constexpr (sizeof(TZ) == 2) latent_out[zi] = f32_to_bf16_bits(z);
        else latent_out[zi] = z;
    }
}

hipError_t launch_sample(void* m, const float* parts, bool m_half, const float* eps, float* moments_out, void* latent_out, bool latent_bf16,
                         int C0, int n_frames, const Slot* slots, int n_slots, int max_int, hipStream_t stream)
{
    if (m_half != latent_bf16 || (parts ? !m_half : !m)) return hipErrorInvalidValue;
    dim3 grid((unsigned)(((size_t)max_int * C0 + 255) / 256), (unsigned)n_slots);
#define DEMON_SAMPLE(TM_, TZ_, PARTS_) hipLaunchKernelGGL((sample_kernel<TM_, TZ_, PARTS_>), grid, dim3(256), 0, stream, (TM_*)m, parts, eps, \
                                                          moments_out, (TZ_*)latent_out, C0, n_frames, slots)
    if (parts) DEMON_SAMPLE(_Float16, uint16_t, true);
    else if (m_half) DEMON_SAMPLE(_Float16, uint16_t, false);
    else DEMON_SAMPLE(float, float, false);
#undef DEMON_SAMPLE
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------- head
// Only the interior rows of every window are produced (the halo is trimmed right after).  Rows outside
// the window read as zero (the conv's zero padding at a clip edge); Snake is applied while staging.
//
// Fast kernel (OC output channels, K taps as template arguments): a workgroup owns 256 SPT
// consecutive samples (SPT = 1: 128), each thread SPT of them.  Channels go through LDS in chunks of 16, transposed to
// [channel][row] so that a thread's 4 + K - 1 input rows are consecutive words (three 16-byte reads per
// channel for K = 7) and feed 4*K*OC FMAs; the weights are wave-uniform (scalar loads).  The row
// length LDR = 4 mod 16 keeps both the transposing stores and the reads free of bank conflicts.  SPT = 4 reads
// the fewest LDS words per sample; a launch that would leave CUs idle that way (a few windows) takes SPT = 1, a thread per sample and
// output channel, which adds in the same order.  Such a launch is bound by one workgroup's chain, mostly the precise sines of its rows: 128
// samples a workgroup where it was 256, and a chunk's rows requested together and a chunk ahead where each was waited for in turn.  fp32, 2 s of the x32
// stack 14.8 -> 10.8 us with an event after the launch (requests alone 13.5), the call 100.4 -> 97.2; 3 s window of the x1920 stack 33.8 -> 30.9.
constexpr int HEAD_KC = 16;
constexpr int HEAD_MAXK = 15;
constexpr int HEAD_MAXOC = 8;

template <typename TX, bool FAST, int OC, int K, int HEAD_SPT>
__global__ __launch_bounds__(256) void head_fast_kernel(const TX* __restrict__ x, HeadOut out, bool vec,
                                                        const float* __restrict__ w, const float* __restrict__ bias,
                                                        const float* __restrict__ alpha, const float* __restrict__ inv_beta,
                                                        int cin, int r, const Slot* __restrict__ slots)
{
    constexpr bool SPLIT = HEAD_SPT == 1;                   // a thread per sample and output channel
    constexpr int HEAD_NT = SPLIT ? 256 / OC : 256 * HEAD_SPT, NO = SPLIT ? 1 : OC;
    static_assert(HEAD_NT % 64 == 0, "an output channel per wave");
    constexpr int HEAD_LDR = HEAD_NT + 20;                  // >= HEAD_NT + HEAD_MAXK - 1, = 4 (mod 16)
    __shared__ __attribute__((aligned(16))) float xs[HEAD_KC * HEAD_LDR];
    constexpr int HALF = (K - 1) / 2;
    constexpr int XR = HEAD_NT + K - 1;
    constexpr int NV = (HEAD_SPT + K - 1 + 3) / 4;          // float4 reads per channel
    const Slot s = slots[blockIdx.y];
    const long long nrows = (long long)s.len * r;
    const long long lo = (long long)s.crop * r, hi = (long long)(s.crop + s.n_int) * r;
    const long long n0 = lo + (long long)blockIdx.x * HEAD_NT;
    if (n0 >= hi) return;
    const long long rowbase = (long long)s.row0 * r;
    const int tid = threadIdx.x;
    const int q = tid & 3, r0 = tid >> 2;                   // staging: 4 lanes per row, 4 channels each

    const int sample = SPLIT ? tid % HEAD_NT : HEAD_SPT * tid, o0 = SPLIT ? __builtin_amdgcn_readfirstlane(tid / HEAD_NT) : 0;
    float acc[HEAD_SPT][NO];
#pragma unroll
    for (int i = 0; i < HEAD_SPT; ++i)
#pragma unroll
        for (int o = 0; o < NO; ++o) acc[i][o] = 0.f;

    // every row of a chunk requested before the first is waited for, the next chunk's before this one's sums; rows outside the
    // window are another's (clamped) and become zeros
    constexpr int RP = (XR + 63) / 64;
    using raw_t = std::conditional_t<sizeof(TX) == 4, f32x4, f16x4>;
    raw_t raw[RP];
    f32x4 al, ib;
    auto request = [&](int c0) __attribute__((always_inline)) {
        al = *reinterpret_cast<const f32x4*>(alpha + c0 + 4 * q);
        ib = *reinterpret_cast<const f32x4*>(inv_beta + c0 + 4 * q);
#pragma unroll
        for (int it = 0; it < RP; ++it) {
            const long long n = min(max(n0 - HALF + r0 + 64 * it, 0ll), nrows - 1);
            raw[it] = *reinterpret_cast<const raw_t*>(x + (size_t)(rowbase + n) * cin + c0 + 4 * q);
        }
    };
    request(0);
    for (int c0 = 0; c0 < cin; c0 += HEAD_KC) {
        __syncthreads();
#pragma unroll
        for (int it = 0; it < RP; ++it) {
            const int row = r0 + 64 * it;
            const long long n = n0 - HALF + row;
            if (row >= XR) break;
#pragma unroll
            for (int e = 0; e < 4; ++e) xs[(4 * q + e) * HEAD_LDR + row] = n < 0 || n >= nrows ? 0.f : (float)raw[it][e];
        }
        const f32x4 a = al, b = ib;
        if (c0 + HEAD_KC < cin) request(c0 + HEAD_KC);
        // Snake in place, each thread on what it wrote; one copy of the sine's code
#pragma unroll 1
        for (int row = r0; row < XR; row += 64) {
            if (n0 - HALF + row < 0 || n0 - HALF + row >= nrows) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float* at = &xs[(4 * q + e) * HEAD_LDR + row];
                *at = FAST ? snake_fast(*at, a[e], b[e]) : snake_precise(*at, a[e], b[e]);
            }
        }
        __syncthreads();
#pragma unroll 4
        for (int c = 0; c < HEAD_KC; ++c) {
            float xv[NV * 4];
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const float* src = &xs[c * HEAD_LDR + sample + 4 * i];
                if constexpr (HEAD_SPT == 4) {
                    const float4 t4 = *reinterpret_cast<const float4*>(src);
                    xv[4 * i] = t4.x; xv[4 * i + 1] = t4.y; xv[4 * i + 2] = t4.z; xv[4 * i + 3] = t4.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) xv[4 * i + e] = 4 * i + e < HEAD_SPT + K - 1 ? src[e] : 0.f;
                }
            }
#pragma unroll
            for (int t = 0; t < K; ++t)
#pragma unroll
                for (int o = 0; o < NO; ++o) {
                    const float wv = w[((size_t)t * cin + c0 + c) * OC + o0 + o];
#pragma unroll
                    for (int i = 0; i < HEAD_SPT; ++i) acc[i][o] = fmaf(wv, xv[i + t], acc[i][o]);
                }
        }
    }
    const long long n = n0 + sample, origin = head_origin(out, s, OC, r);
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        const float b = bias[o0 + o];
        float* dst = out.y + (o0 + o) * out.plane + origin + n;
        if (HEAD_SPT == 4 && n + HEAD_SPT <= hi && vec) {
            *reinterpret_cast<float4*>(dst) = make_float4(tanhf(acc[0][o] + b), tanhf(acc[HEAD_SPT / 4][o] + b),
                                                          tanhf(acc[HEAD_SPT / 2][o] + b), tanhf(acc[HEAD_SPT - 1][o] + b));
        } else {
#pragma unroll
            for (int i = 0; i < HEAD_SPT; ++i)
                if (n + i < hi) dst[i] = tanhf(acc[i][o] + b);
        }
    }
}

// Generic kernel (any out_channels <= 8, any odd kernel <= 15, any channel count): one sample per
// thread, channels staged through LDS in chunks of 32.
constexpr int HEADG_NT = 256;
constexpr int HEADG_KC = 32;

template <typename TX, bool FAST>
__global__ __launch_bounds__(256) void head_generic_kernel(const TX* __restrict__ x, HeadOut out,
                                                           const float* __restrict__ w, const float* __restrict__ bias,
                                                           const float* __restrict__ alpha, const float* __restrict__ inv_beta,
                                                           int cin, int oc, int k, int r,
                                                           const Slot* __restrict__ slots)
{
    __shared__ float xs[(HEADG_NT + HEAD_MAXK - 1) * (HEADG_KC + 1)];
    const Slot s = slots[blockIdx.y];
    const long long nrows = (long long)s.len * r;
    const long long lo = (long long)s.crop * r, hi = (long long)(s.crop + s.n_int) * r;
    const long long n0 = lo + (long long)blockIdx.x * HEADG_NT;
    if (n0 >= hi) return;
    const long long rowbase = (long long)s.row0 * r;
    const int half = (k - 1) / 2;
    const int xr = HEADG_NT + k - 1;

    float acc[HEAD_MAXOC];
#pragma unroll
    for (int o = 0; o < HEAD_MAXOC; ++o) acc[o] = 0.f;

    for (int c0 = 0; c0 < cin; c0 += HEADG_KC) {
        const int kc = min(HEADG_KC, cin - c0);
        __syncthreads();
        for (int e = threadIdx.x; e < xr * HEADG_KC; e += 256) {
            const int row = e / HEADG_KC, c = e - row * HEADG_KC;
            const long long n = n0 - half + row;
            float v = 0.f;
            if (c < kc && n >= 0 && n < nrows) {
                v = load_act<TX>(x + (size_t)(rowbase + n) * cin + c0 + c);
                v = FAST ? snake_fast(v, alpha[c0 + c], inv_beta[c0 + c]) : snake_precise(v, alpha[c0 + c], inv_beta[c0 + c]);
            }
            xs[row * (HEADG_KC + 1) + c] = v;
        }
        __syncthreads();
        for (int t = 0; t < k; ++t) {
            const float* xrow = xs + (threadIdx.x + t) * (HEADG_KC + 1);
            const float* wt = w + ((size_t)t * cin + c0) * oc;
            for (int c = 0; c < kc; ++c) {
                const float v = xrow[c];
#pragma unroll
                for (int o = 0; o < HEAD_MAXOC; ++o)
                    if (o < oc) acc[o] = fmaf(wt[c * oc + o], v, acc[o]);
            }
        }
    }
    const long long n = n0 + threadIdx.x, origin = head_origin(out, s, oc, r);
    if (n < hi) {
#pragma unroll
        for (int o = 0; o < HEAD_MAXOC; ++o)
            if (o < oc) out.y[o * out.plane + origin + n] = tanhf(acc[o] + bias[o]);
    }
}

// MFMA head for the bf16 path (half-precision residual stream in, out_channels <= 32).
// GEMM with rows = time, columns = output channel (padded to 32), K = (tap, channel):
//     D[n, o] = sum_t sum_c snake(h[n + t - (K-1)/2, c]) W[o, c, t]
// on v_mfma_f32_32x32x16_f16: operands in IEEE half (their rounding is an order of magnitude below that of
// the bf16 operands elsewhere), fp32 accumulation.  The A operand is the activation tile: whole 128-byte
// rows are read once from HBM, Snake is applied in fp32, the tile sits row-major in LDS and a tap is a row
// offset.  The B operand (the weights, zero beyond out_channels) is packed at create in fragment order and
// staged into LDS once per workgroup.  A lane with column index < out_channels holds the results.
constexpr int HM_NT = 256;                     // rows per sub-tile: 4 waves x 64 rows
constexpr int HM_SUB = 4;                      // sub-tiles per workgroup (the weights are staged once)
constexpr int HM_MAXFRAG = 40;                 // taps * channels / 16

size_t head_mfma_frag_count(int cin, int k) { return (size_t)k * (cin / 16); }

// [tap][k-step][lane][8]: lane (j, h) of k-step ks holds W[o = j][c = 16 ks + 8 h + e][tap], e = 0..7
void pack_head_mfma(const float* w /*[oc][cin][k]*/, int cin, int oc, int k, uint16_t* dst)
{
    size_t pos = 0;
    for (int t = 0; t < k; ++t)
        for (int ks = 0; ks < cin / 16; ++ks)
            for (int lane = 0; lane < 64; ++lane)
                for (int e = 0; e < 8; ++e) {
                    const int j = lane & 31, h = lane >> 5, c = 16 * ks + 8 * h + e;
                    const _Float16 v = (j < oc) ? (_Float16)w[((size_t)j * cin + c) * k + t] : (_Float16)0.f;
                    uint16_t bits;
                    __builtin_memcpy(&bits, &v, 2);
                    dst[pos++] = bits;
                }
}

typedef _Float16 f16x8v __attribute__((ext_vector_type(8)));

// OCP: output channels kept in LDS per weight fragment (8 when oc <= 8, else 32): the other lanes of the fragment are
// zero padding and are not stored, which with the unpadded-weights tile leaves room for three workgroups per CU.
template <int CIN, int OCP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(OCP == 8 ? 3 : 2, OCP == 8 ? 3 : 2)))
void head_mfma_kernel(const _Float16* __restrict__ x, HeadOut out,
                                                        const uint16_t* __restrict__ wfrag, const float* __restrict__ bias,
                                                        const float* __restrict__ alpha, const float* __restrict__ inv_beta,
                                                        int oc, int k, int r, const Slot* __restrict__ slots)
{
    fp16_saturate_on();
    constexpr int LDX = CIN + 8;                           // padded LDS row (halfs)
    constexpr int XR_MAX = HM_NT + HEAD_MAXK - 1;
    constexpr int SEGS = CIN / 8, RPP = 256 / SEGS;
    constexpr int X_ITERS = (XR_MAX + RPP - 1) / RPP;
    constexpr int KS = CIN / 16;
    __shared__ __attribute__((aligned(16))) _Float16 Xs[XR_MAX * LDX];
    __shared__ __attribute__((aligned(16))) uint16_t Ws[HM_MAXFRAG * 2 * OCP * 8];       // [fragment][h][channel < OCP][8 halves]

    const Slot s = slots[blockIdx.y];
    const int nrows = s.len * r;
    const int lo = s.crop * r, hi = (s.crop + s.n_int) * r;
    const int half = (k - 1) / 2;
    const int XR = HM_NT + k - 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = lane & 31, h = lane >> 5;
    const int seg = tid % SEGS, xr0 = tid / SEGS;
    const long long rowbase = (long long)s.row0 * r, origin = head_origin(out, s, oc, r);
    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(x + rowbase * CIN, (unsigned)nrows * CIN * 2u);
    if (lo + (int)blockIdx.x * (HM_NT * HM_SUB) >= hi) return;

    // weights -> LDS once
    {
        const u32x4* src = reinterpret_cast<const u32x4*>(wfrag);             // [fragment][lane = h * 32 + channel][8 halves]
        for (int q = tid; q < k * KS * 2 * OCP; q += 256)
            reinterpret_cast<u32x4*>(Ws)[q] = src[(q / OCP) * 32 + q % OCP];
    }
    float al[8], ib[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) { al[e] = alpha[seg * 8 + e]; ib[e] = inv_beta[seg * 8 + e]; }
    // accumulator register 4g + q of lane (j, h) is output channel 8g + 4h + q: with OCP = 8 only g = 0 holds channels
    constexpr int NB = OCP == 8 ? 4 : 16;
    float b[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        const int c = 8 * (q >> 2) + 4 * h + (q & 3);
        b[q] = (c < oc) ? bias[c] : 0.f;
    }

    // The raw rows of a sub-tile are fetched one sub-tile ahead, so that their latency hides behind the MFMAs and the
    // tanh epilogue of the previous one.  Rows outside the window are out of range of the descriptor and read as
    // zero = the convolution's zero padding.
    u32x4 raw[X_ITERS];
    auto load_rows = [&](int n0) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < X_ITERS; ++it) {
            if (it * RPP >= XR) break;                         // uniform
            raw[it] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, (unsigned)((n0 - half + xr0 + it * RPP) * CIN + seg * 8) * 2u, 0, 0);
        }
    };
    load_rows(lo + (int)blockIdx.x * (HM_NT * HM_SUB));
    for (int sub = 0; sub < HM_SUB; ++sub) {
        const int n0 = lo + ((int)blockIdx.x * HM_SUB + sub) * HM_NT;
        if (n0 >= hi) break;                                   // uniform
        __syncthreads();                                       // the previous sub-tile's reads are done
#pragma unroll
        for (int it = 0; it < X_ITERS; ++it) {
            const int xr = xr0 + it * RPP;
            if (it * RPP >= XR) break;                         // uniform
            if (xr >= XR_MAX) continue;
            const f16x8v hv = __builtin_bit_cast(f16x8v, raw[it]);
            f16x8v ov;
#pragma unroll
            for (int e = 0; e < 8; ++e) ov[e] = (_Float16)keep_f32(snake_fast_half(hv[e], al[e], ib[e]));
            *reinterpret_cast<f16x8v*>(&Xs[xr * LDX + seg * 8]) = ov;
        }
        __syncthreads();
        if (sub + 1 < HM_SUB && n0 + HM_NT < hi) load_rows(n0 + HM_NT);

        f32x16 acc[2];
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[mi][q] = q < NB ? b[q] : 0.f;
        for (int t = 0; t < k; ++t) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                f16x8v bw = {0, 0, 0, 0, 0, 0, 0, 0};
                if (j < OCP) bw = *reinterpret_cast<const f16x8v*>(&Ws[(((t * KS + ks) * 2 + h) * OCP + j) * 8]);
#pragma unroll
                for (int mi = 0; mi < 2; ++mi) {
                    const f16x8v av = *reinterpret_cast<const f16x8v*>(&Xs[(wave * 64 + mi * 32 + j + t) * LDX + ks * 16 + h * 8]);
                    // weights as the row operand: the accumulator tile is [output channel][time]
                    acc[mi] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bw, av, acc[mi], 0, 0, 0);
                }
            }
        }
        // lane (j, h) holds time column j and output channels 8g + 4h + {0..3}: with a few output channels the tanh work
        // sits in the first registers of half of the lanes, and a channel's 32 samples are one contiguous store
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) {
            const int n = n0 + wave * 64 + mi * 32 + j;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if (8 * g >= oc) break;                        // uniform
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int c = 8 * g + 4 * h + q;
                    if (c < oc && n < hi) out.y[c * out.plane + origin + n] = tanhf(acc[mi][4 * g + q]);
                }
            }
        }
    }
}

hipError_t launch_head_mfma(const void* x, const HeadOut& out, const uint16_t* wfrag, const float* bias, const float* alpha,
                            const float* inv_beta, int cin, int oc, int k, int r,
                            const Slot* slots, int n_slots, int max_len, int max_int, hipStream_t stream)
{
    if (oc > 32 || k > HEAD_MAXK || (cin != 64 && cin != 32) || head_mfma_frag_count(cin, k) > HM_MAXFRAG) return hipErrorInvalidValue;
    if ((long long)max_len * r * cin * 2 > 0xf0000000ll) return hipErrorInvalidValue;
    const long long rows = (long long)max_int * r;
    dim3 grid((unsigned)((rows + HM_NT * HM_SUB - 1) / (HM_NT * HM_SUB)), (unsigned)n_slots);
#define DEMON_HEAD(CIN_, OCP_) hipLaunchKernelGGL((head_mfma_kernel<CIN_, OCP_>), grid, dim3(256), 0, stream, (const _Float16*)x, out, wfrag, bias, alpha, inv_beta, oc, k, r, slots)
    if (cin == 64) { if (oc <= 8) DEMON_HEAD(64, 8); else DEMON_HEAD(64, 32); }
    else { if (oc <= 8) DEMON_HEAD(32, 8); else DEMON_HEAD(32, 32); }
#undef DEMON_HEAD
    return hipGetLastError();
}

hipError_t launch_head(const void* x, bool x_half, const HeadOut& out, const float* w, const float* bias, const float* alpha,
                       const float* inv_beta, int cin, int oc, int k, int r,
                       bool fast, const Slot* slots, int n_slots, int max_int, hipStream_t stream)
{
    if (k > HEAD_MAXK || oc > HEAD_MAXOC || (x_half && !fast)) return hipErrorInvalidValue;
    const long long rows = (long long)max_int * r;
    if (oc == 2 && k == 7 && cin % HEAD_KC == 0) {
        const bool few = (rows + 1023) / 1024 * n_slots < 512;        // two 1024-sample workgroups per CU
        const int nt = few ? 128 : 1024;
        // 16-byte stores: rows of a window start at multiples of r in a plane, planes (and clips) are multiples of r apart
        const bool vec = r % 4 == 0 && reinterpret_cast<uintptr_t>(out.y) % 16 == 0;
        dim3 grid((unsigned)((rows + nt - 1) / nt), (unsigned)n_slots);
#define DEMON_HEADF(TX_, FAST_, SPT_) hipLaunchKernelGGL((head_fast_kernel<TX_, FAST_, 2, 7, SPT_>), grid, dim3(256), 0, stream, (const TX_*)x, out, vec, w, bias, alpha, inv_beta, cin, r, slots)
        if (x_half) { if (few) DEMON_HEADF(_Float16, true, 1); else DEMON_HEADF(_Float16, true, 4); }
        else if (fast) { if (few) DEMON_HEADF(float, true, 1); else DEMON_HEADF(float, true, 4); }
        else { if (few) DEMON_HEADF(float, false, 1); else DEMON_HEADF(float, false, 4); }
#undef DEMON_HEADF
        return hipGetLastError();
    }
    dim3 grid((unsigned)((rows + HEADG_NT - 1) / HEADG_NT), (unsigned)n_slots);
    if (x_half)
        hipLaunchKernelGGL((head_generic_kernel<_Float16, true>), grid, dim3(256), 0, stream, (const _Float16*)x, out, w, bias, alpha, inv_beta, cin, oc, k, r, slots);
    else if (fast)
        hipLaunchKernelGGL((head_generic_kernel<float, true>), grid, dim3(256), 0, stream, (const float*)x, out, w, bias, alpha, inv_beta, cin, oc, k, r, slots);
    else
        hipLaunchKernelGGL((head_generic_kernel<float, false>), grid, dim3(256), 0, stream, (const float*)x, out, w, bias, alpha, inv_beta, cin, oc, k, r, slots);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------- 16-bit render
// Crop, stitch and 16-bit render of the window waveforms: q = rint(32767 * clamp(y, -1, 1)) in fp32 (round half to even), channels
// interleaved per sample: pcm[clip][sample][channel].  One thread quantises VEC consecutive samples of all channels.
template <int VEC, int OC>
__global__ __launch_bounds__(256) void stitch_pcm16_kernel(const float* __restrict__ y, int16_t* __restrict__ pcm,
                                                           int oc, int S, int n_frames, long long total_rows,
                                                           const Slot* __restrict__ slots)
{
    const Slot s = slots[blockIdx.y];
    const long long n = (long long)s.n_int * S;
    const long long i = ((long long)blockIdx.x * 256 + threadIdx.x) * VEC;
    if (i >= n) return;
    const float* src = y + ((long long)s.row0 + s.crop) * S + i;
    int16_t* dst = pcm + ((size_t)s.clip * ((size_t)n_frames * S) + (size_t)s.begin * S + i) * oc;
    auto quant = [](float v) -> int16_t {
        v = fminf(fmaxf(v, -1.0f), 1.0f);
        return (int16_t)__float2int_rn(v * 32767.0f);
    };
    if (OC == 2 && VEC == 4) {
        const float4 l = *reinterpret_cast<const float4*>(src);
        const float4 r = *reinterpret_cast<const float4*>(src + total_rows);
        const float lv[4] = {l.x, l.y, l.z, l.w}, rv[4] = {r.x, r.y, r.z, r.w};
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            o[e] = (uint32_t)(uint16_t)quant(lv[e]) | ((uint32_t)(uint16_t)quant(rv[e]) << 16);
        *reinterpret_cast<u32x4*>(dst) = o;
    } else {
        for (int e = 0; e < VEC && i + e < n; ++e)
            for (int c = 0; c < oc; ++c) dst[(size_t)e * oc + c] = quant(src[(size_t)c * total_rows + e]);
    }
}

hipError_t launch_stitch_pcm16(const float* y, int16_t* pcm, int oc, int S, int n_frames, long long total_rows,
                               const Slot* slots, int n_slots, int max_int, hipStream_t stream)
{
    // 16-byte stores need 4 stereo samples per thread at a 16-byte aligned address: S % 4 == 0 keeps every window start aligned
    const bool vec = oc == 2 && (S % 4 == 0) && (total_rows % 4 == 0) &&
                     (reinterpret_cast<uintptr_t>(y) % 16 == 0) && (reinterpret_cast<uintptr_t>(pcm) % 16 == 0);
    const long long per = (long long)max_int * S;
    if (vec) {
        dim3 grid((unsigned)((per / 4 + 255) / 256), (unsigned)n_slots);
        hipLaunchKernelGGL((stitch_pcm16_kernel<4, 2>), grid, dim3(256), 0, stream, y, pcm, oc, S, n_frames, total_rows, slots);
    } else {
        dim3 grid((unsigned)((per + 255) / 256), (unsigned)n_slots);
        hipLaunchKernelGGL((stitch_pcm16_kernel<1, 0>), grid, dim3(256), 0, stream, y, pcm, oc, S, n_frames, total_rows, slots);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------- window table on the device
// The window grid of section 3.6 written by a kernel: window k of a clip covers frames [begin + k window, ...), is
// extended by the halo and clamped to the clip; its workspace rows follow those of the windows before it.  One thread per window; the prefix
// sum over the earlier windows of the clip is a short loop (at most 4096 windows per call).
__global__ __launch_bounds__(256) void plan_slots_kernel(Slot* __restrict__ dst, int n, int per_clip, int clip_frames,
                                                         int n_frames, int fb, int fe, int window, int halo)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int clip = i / per_clip, k = i - clip * per_clip;
    auto extent = [&](int kk, int* lo, int* hi, int* b, int* e) {
        *b = fb + kk * window;
        *e = min(*b + window, fe);
        *lo = max(0, *b - halo);
        *hi = min(n_frames, *e + halo);
    };
    int row = clip * clip_frames;
    for (int kk = 0; kk < k; ++kk) {
        int lo, hi, b, e;
        extent(kk, &lo, &hi, &b, &e);
        row += hi - lo;
    }
    int lo, hi, b, e;
    extent(k, &lo, &hi, &b, &e);
    Slot s;
    s.row0 = row; s.len = hi - lo; s.clip = clip; s.lo = lo; s.crop = b - lo; s.n_int = e - b; s.begin = b; s.pad = 0;
    dst[i] = s;
}

hipError_t launch_plan_slots(Slot* dst, int n_clips, int per_clip, int clip_frames, int n_frames, int frame_begin,
                             int frame_end, int window, int halo, hipStream_t stream)
{
    const long long n = (long long)n_clips * per_clip;
    if (n < 1 || n > 65536) return hipErrorInvalidValue;
    hipLaunchKernelGGL(plan_slots_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, dst, (int)n, per_clip, clip_frames,
                       n_frames, frame_begin, frame_end, window, halo);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------- latent similarity filter
// One workgroup per clip: squared differences accumulate in double in a fixed order (thread-strided partial sums of 16 bytes, then a
// tree over the workgroup), so the result depends neither on scheduling nor on where the latents lie.  mse and the gate go out as fp32 / int.
// Bound by the latency of one workgroup's loads: 16 bytes of each latent at a time, four of them in flight.  The loads claim no more than an
// element's alignment.  64 x 1500 in bf16: single elements 12.2 us, here 7.4 (and from odd addresses, which cost the loads more, 12.4; fp32
// 12.0 and 7.8 from any address).  What is left is arithmetic in double on one CU.
template <typename T>
__global__ __launch_bounds__(1024) void latent_mse_kernel(const T* __restrict__ a, const T* __restrict__ b, long long n,
                                                          float threshold, float* __restrict__ mse, int* __restrict__ unchanged)
{
    __shared__ double part[16];
    constexpr int V = 16 / sizeof(T), U = 4;
    typedef T vec_t __attribute__((ext_vector_type(V)));
    typedef vec_t loose_t __attribute__((aligned(sizeof(T))));
    const T* pa = a + (size_t)blockIdx.x * n;
    const T* pb = b + (size_t)blockIdx.x * n;
    double acc = 0.0;
    auto add = [&](T x, T y) __attribute__((always_inline)) {
        const double d = (double)load_act<T>(&x) - (double)load_act<T>(&y);
        acc += d * d;
    };
    const loose_t* va = reinterpret_cast<const loose_t*>(pa);
    const loose_t* vb = reinterpret_cast<const loose_t*>(pb);
    const long long nv = n / V;
    for (long long i = threadIdx.x; i < nv; i += U * 1024) {
        vec_t x[U] = {}, y[U] = {};
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + u * 1024 < nv) { x[u] = va[i + u * 1024]; y[u] = vb[i + u * 1024]; }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < V; ++e) add(x[u][e], y[u][e]);
    }
    if (const long long i = nv * V + threadIdx.x; i < n) add(pa[i], pb[i]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < 16; ++w) t += part[w];
        const float m = (float)(t / (double)n);
        if (mse) mse[blockIdx.x] = m;
        if (unchanged) unchanged[blockIdx.x] = m < threshold ? 1 : 0;
    }
}

hipError_t launch_latent_mse(const void* a, const void* b, int n_clips, long long n, bool bf16, float threshold,
                             float* mse, int* unchanged, hipStream_t stream)
{
    if (bf16)
        hipLaunchKernelGGL(latent_mse_kernel<uint16_t>, dim3(n_clips), dim3(1024), 0, stream,
                           (const uint16_t*)a, (const uint16_t*)b, n, threshold, mse, unchanged);
    else
        hipLaunchKernelGGL(latent_mse_kernel<float>, dim3(n_clips), dim3(1024), 0, stream,
                           (const float*)a, (const float*)b, n, threshold, mse, unchanged);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------- equal-power crossfade
// out[c][i] = cos(theta_i) * tail[c][i] + sin(theta_i) * head[c][i], theta_i = (pi/2)(i + 1/2)/n.  Element-wise, so out may
// alias head or tail.
__global__ __launch_bounds__(256) void crossfade_kernel(const float* __restrict__ tail, long long tail_stride,
                                                        const float* __restrict__ head, long long head_stride,
                                                        float* out, long long out_stride, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int c = blockIdx.y;
    const float theta = 1.57079632679489662f * (((float)i + 0.5f) / (float)n);
    float sn, cs;
    sincosf(theta, &sn, &cs);
    out[c * out_stride + i] = cs * tail[c * tail_stride + i] + sn * head[c * head_stride + i];
}

hipError_t launch_crossfade(const float* tail, long long tail_stride, const float* head, long long head_stride,
                            float* out, long long out_stride, int n_planes, int n, hipStream_t stream)
{
    dim3 grid((unsigned)((n + 255) / 256), (unsigned)n_planes);
    hipLaunchKernelGGL(crossfade_kernel, grid, dim3(256), 0, stream, tail, tail_stride, head, head_stride, out, out_stride, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------- debug tap
template <typename T>
__global__ __launch_bounds__(256) void to_f32_kernel(const T* __restrict__ x, float* __restrict__ dst, size_t n)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = load_act<T>(x + i);
}

hipError_t launch_to_f32(const void* x, float* dst, size_t n, int src_type, hipStream_t stream)
{
    if (n == 0) return hipSuccess;
    dim3 grid((unsigned)((n + 255) / 256));
    if (src_type == 1) hipLaunchKernelGGL(to_f32_kernel<uint16_t>, grid, dim3(256), 0, stream, (const uint16_t*)x, dst, n);
    else if (src_type == 2) hipLaunchKernelGGL(to_f32_kernel<_Float16>, grid, dim3(256), 0, stream, (const _Float16*)x, dst, n);
    else hipLaunchKernelGGL(to_f32_kernel<float>, grid, dim3(256), 0, stream, (const float*)x, dst, n);
    return hipGetLastError();
}

}  // namespace demon
