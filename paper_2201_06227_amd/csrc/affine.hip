// Affine (asymmetric) uint8 activation codes: the framework's default activation
// code, to which Section 5 of the paper delegates the int8 arithmetic.  From the
// extrema of a tensor, every operation an IEEE fp32 one:
//   hi = max(max x, 0), lo = min(min x, 0)
//   scale = max((hi - lo) / 255, 2^-23);  zp = clamp(0 - rne(lo / scale), 0, 255)
//   q = clamp(rne(x * (1 / scale)) + zp, 0, 255)
// A code is stored as the int8 value q - 128, so the int8 x int8 matrix cores
// contract it unchanged: sum (q - zp) w = sum (q - 128) w + (128 - zp) sum w, and
// the sums of the weight codes (per output channel, and for 3x3 kernels per class
// of border pixel: a window position outside the image holds the real value zero,
// whose centred code is 0, while the contraction reads a stored 0 = code 128
// there) are made once per snapshot by colsum_kernel.
//
// Two launches per quantise point: the extrema as per-workgroup partial results
// (plain stores), then the codes, every workgroup reducing the partial results
// to the same scale and zero point.  HBM-bound: 4 n bytes read twice, n written.
// The output of a ReLU has no negative values, so its extrema are 0 and the
// maximum that the convolution's epilogue keeps anyway: such a point is the code
// pass alone.
#include "common.hpp"

namespace egeria {

namespace {

constexpr int kMinMaxBlocks = 1024;

template <bool BF16>
__global__ __launch_bounds__(256) void minmax_kernel(const void *__restrict__ x, int64_t n, uint32_t *__restrict__ partials,
                                                     uint32_t *__restrict__ reset, int n_reset)
{
    if (blockIdx.x == 0) {               // clears the maximum words of the module's later quantise points
        for (int t = threadIdx.x; t < n_reset * kAmaxWays; t += blockDim.x) reset[(size_t)t * kAmaxStride] = 0u;
    }
    float hi = 0.0f, nlo = 0.0f;       // max(x, 0) and max(-x, 0)
    uint32_t worst = 0;                // largest |x| bit pattern: above 0x7f7fffff for NaN and infinities
    const uint32_t piece = xcd_piece(blockIdx.x, gridDim.x);
    if (!BF16 && ((uintptr_t)x & 15) == 0) {
        const float4 *x4 = (const float4 *)x;
        const int64_t n4 = n >> 2, per = (int64_t)((uint64_t)(n4 + gridDim.x - 1) / gridDim.x), beg = (int64_t)piece * per;
        const int64_t end = beg + per < n4 ? beg + per : n4;
        auto take = [&](const float4 &v) {
            const float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                hi = fmaxf(hi, e[k]);
                nlo = fmaxf(nlo, -e[k]);
                const uint32_t a = abs_bits(e[k]);
                worst = worst > a ? worst : a;
            }
        };
        // four units of a thread in flight (indices clamped: a value seen twice changes no extremum).  A thread's units spread over
        // the whole tensor / this way, us: 1 M values 2.7 / 2.8, 5.2 M 5.3 / 3.9, 12.8 M 10.0 / 8.8, 50 M 28.9 / 28.7, 200 M 144 / 147.
        for (int64_t i = beg + threadIdx.x; i < end; i += 1024) {
            float4 v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = x4[i + 256 * j < end ? i + 256 * j : end - 1];
#pragma unroll
            for (int j = 0; j < 4; ++j) take(v[j]);
        }
        for (int64_t i = piece == 0 ? (n4 << 2) + threadIdx.x : n; i < n; i += 256) {
            const float v = ((const float *)x)[i];
            hi = fmaxf(hi, v);
            nlo = fmaxf(nlo, -v);
            const uint32_t a = abs_bits(v);
            worst = worst > a ? worst : a;
        }
    } else {
        const int64_t first = (int64_t)piece * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
        for (int64_t i = first; i < n; i += stride) {
            const float v = BF16 ? bf16_to_f32(((const uint16_t *)x)[i]) : ((const float *)x)[i];
            hi = fmaxf(hi, v);
            nlo = fmaxf(nlo, -v);
            const uint32_t a = abs_bits(v);
            worst = worst > a ? worst : a;
        }
    }
    // both are non-negative, so their bit patterns order like the values
    uint32_t hb = wave_max_u32(__float_as_uint(hi)), lb = wave_max_u32(__float_as_uint(nlo));
    worst = wave_max_u32(worst);
    __shared__ uint32_t sm[3][4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) { sm[0][wave] = hb; sm[1][wave] = lb; sm[2][wave] = worst; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) {
            sm[0][0] = sm[0][0] > sm[0][w] ? sm[0][0] : sm[0][w];
            sm[1][0] = sm[1][0] > sm[1][w] ? sm[1][0] : sm[1][w];
            sm[2][0] = sm[2][0] > sm[2][w] ? sm[2][0] : sm[2][w];
        }
        const bool bad = sm[2][0] >= 0x7f800000u;
        partials[2 * blockIdx.x] = bad ? 0x7fc00000u : sm[0][0];
        partials[2 * blockIdx.x + 1] = sm[1][0];
    }
}

// [n, c, hw] (channel planes; hw = 1: rows of a matrix) -> codes [n, hw, cp], 16 per store.  HBM-bound; what counts
// is the bytes in flight per thread.  Three forms:
//   kRows    fp32 rows of whole 16-byte units: four 16-byte loads make the 16 codes of a unit
//            (12544 x 256: 12.9 us with a load per value, 5.4 now);
//   kPlanes  fp32 planes of whole 16-byte units: sixteen 16-byte loads (4 pixels x 16 channels) make four units
//            (64 x 1024 x 196: 23.3 -> 16.5 us);
//   kAny     everything else: one load per value (lanes along the pixels, or along the units of a row).
enum AffineForm { kAny = 0, kRows = 1, kPlanes = 2 };

template <bool BF16, int FORM>
__global__ __launch_bounds__(256) void quantize_affine_kernel(const void *__restrict__ x, int64_t n, int64_t c, int64_t hw,
                                                              int64_t cp, const uint32_t *__restrict__ partials, int nb,
                                                              const uint32_t *__restrict__ relu_max, int store_offset, uint8_t *__restrict__ q,
                                                              float *__restrict__ scale_out, int32_t *__restrict__ zp_out,
                                                              uint32_t *__restrict__ flag, int64_t per)
{
    uint32_t hb = 0, lb = 0;
    if (relu_max) {
        hb = relu_max[(threadIdx.x & (kAmaxWays - 1)) * kAmaxStride];
    } else {
        // all candidates requested together (repeats of the last one change nothing)
        uint2 cand[kMinMaxBlocks / 256];
#pragma unroll
        for (int k = 0; k < kMinMaxBlocks / 256; ++k) {
            const int i = (int)threadIdx.x + 256 * k;
            cand[k] = ((const uint2 *)partials)[i < nb ? i : nb - 1];
        }
#pragma unroll
        for (int k = 0; k < kMinMaxBlocks / 256; ++k) {
            hb = hb > cand[k].x ? hb : cand[k].x;
            lb = lb > cand[k].y ? lb : cand[k].y;
        }
    }
    hb = wave_max_u32(hb);
    lb = wave_max_u32(lb);
    __shared__ uint32_t sm[2][4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) { sm[0][wave] = hb; sm[1][wave] = lb; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        hb = hb > sm[0][w] ? hb : sm[0][w];
        lb = lb > sm[1][w] ? lb : sm[1][w];
    }
    const bool bad = hb >= 0x7f800000u || lb >= 0x7f800000u;
    if (bad) hb = lb = 0;
    const float hi = __uint_as_float(hb), lo = -__uint_as_float(lb);
    float scale = __fdiv_rn(__fsub_rn(hi, lo), 255.0f);
    scale = fmaxf(scale, 1.1920928955078125e-07f);
    int zp = 0 - (int)rintf(__fdiv_rn(lo, scale));
    zp = zp < 0 ? 0 : (zp > 255 ? 255 : zp);
    const float inv = __fdiv_rn(1.0f, scale);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        publish(scale, bad, scale_out, nullptr, flag);
        *zp_out = zp;
    }
    auto code_of = [&](float v) {
        int code = (int)rintf(__fmul_rn(v, inv)) + zp;
        code = code < 0 ? 0 : (code > 255 ? 255 : code);
        return (uint32_t)(code - store_offset) & 0xffu;
    };
    const int64_t beg = xcd_piece(blockIdx.x, gridDim.x) * per, first = beg + threadIdx.x, last = beg + per;
    const int64_t upr = cp >> 4;
    if constexpr (FORM == kRows) {
        const int64_t total = n * upr, end = last < total ? last : total;
        const bool narrow = total < (1LL << 32);
        for (int64_t u = first; u < end; u += 256) {
            const int64_t row = narrow ? (int64_t)((uint32_t)u / (uint32_t)upr) : u / upr, c0 = (u - row * upr) * 16;
            const float4 *src = (const float4 *)((const float *)x + row * c);
            float4 v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = src[c0 + 4 * j < c ? (c0 >> 2) + j : 0];
            uint32_t w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)                    // pad channels: the stored byte is zero
                w[j] = c0 + 4 * j < c ? code_of(v[j].x) | code_of(v[j].y) << 8 | code_of(v[j].z) << 16 | code_of(v[j].w) << 24 : 0u;
            *(uint4 *)(q + row * cp + c0) = make_uint4(w[0], w[1], w[2], w[3]);
        }
        return;
    } else if constexpr (FORM == kPlanes) {
        const int64_t pg = hw >> 2, total = n * upr * pg, end = last < total ? last : total;   // groups of four pixels
        const bool narrow = total < (1LL << 32);
        for (int64_t u = first; u < end; u += 256) {
            const int64_t rest = narrow ? (int64_t)((uint32_t)u / (uint32_t)pg) : u / pg, p = (u - rest * pg) * 4;
            const int64_t img = narrow ? (int64_t)((uint32_t)rest / (uint32_t)upr) : rest / upr, ch0 = (rest - img * upr) * 16;
            const float *src = (const float *)x + (img * c + ch0) * hw + p;
            float4 v[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = *(const float4 *)(src + (ch0 + e < c ? e * hw : 0));
            uint32_t w[4][4] = {};
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const bool in = ch0 + e < c;               // pad channels: the stored byte is zero
                const float f[4] = {v[e].x, v[e].y, v[e].z, v[e].w};
#pragma unroll
                for (int k = 0; k < 4; ++k) w[k][e >> 2] |= (in ? code_of(f[k]) : 0u) << (8 * (e & 3));
            }
            uint8_t *dst = q + (img * hw + p) * cp + ch0;
#pragma unroll
            for (int k = 0; k < 4; ++k) *(uint4 *)(dst + k * cp) = make_uint4(w[k][0], w[k][1], w[k][2], w[k][3]);
        }
        return;
    }
    const int64_t total = n * hw * upr, end = last < total ? last : total;
    const bool narrow = total < (1LL << 32);
    for (int64_t u = first; u < end; u += 256) {
        const int64_t line = hw == 1 ? upr : hw;
        const int64_t rest = narrow ? (int64_t)((uint32_t)u / (uint32_t)line) : u / line, at = u - rest * line;
        int64_t img, p, unit;
        if (hw == 1) {
            img = rest;
            unit = at;
            p = 0;
        } else {
            p = at;
            img = narrow ? (int64_t)((uint32_t)rest / (uint32_t)upr) : rest / upr;
            unit = rest - img * upr;
        }
        // unconditional loads (channel clamped, the surplus discarded): loads under a condition are awaited one by one
        float v[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int64_t ch = unit * 16 + e, i = (img * c + (ch < c ? ch : c - 1)) * hw + p;
            v[e] = BF16 ? bf16_to_f32(((const uint16_t *)x)[i]) : ((const float *)x)[i];
        }
        uint32_t w[4] = {};
#pragma unroll
        for (int e = 0; e < 16; ++e) w[e >> 2] |= (unit * 16 + e < c ? code_of(v[e]) : 0u) << (8 * (e & 3));
        *(uint4 *)(q + ((img * hw + p) * cp + unit * 16)) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// One wave per output channel: the sums of its int8 weight codes per window position, combined per border class.
__global__ __launch_bounds__(256) void colsum_kernel(const int8_t *__restrict__ w_q, int32_t out, int32_t taps, int32_t cp,
                                                     int32_t *__restrict__ colsum)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = blockIdx.x * 4 + wave;
    if (n >= out) return;
    int32_t s[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        s[t] = 0;
        if (t < taps) {
            const int8_t *row = w_q + ((int64_t)n * taps + t) * cp;
            for (int k = lane; k < cp; k += 64) s[t] += row[k];
            s[t] = wave_reduce(s[t], [](int a, int b) { return a + b; });
        }
    }
    if (lane != 0) return;
    if (taps == 1) {
        colsum[n] = s[0];
        return;
    }
    for (int cls = 0; cls < 16; ++cls) {
        int32_t v = 0;
#pragma unroll
        for (int kh = 0; kh < 3; ++kh)
#pragma unroll
            for (int kw = 0; kw < 3; ++kw) {
                const bool outside = (kh == 0 && (cls & 1)) || (kh == 2 && (cls & 2)) || (kw == 0 && (cls & 4)) ||
                                     (kw == 2 && (cls & 8));
                if (!outside) v += s[kh * 3 + kw];
            }
        colsum[(int64_t)cls * out + n] = v;
    }
}

}  // namespace

int minmax_blocks(int64_t n)
{
    int64_t b = (n + 4095) / 4096;
    if (b < 1) b = 1;
    return (int)(b > kMinMaxBlocks ? kMinMaxBlocks : b);
}

size_t affine_partial_bytes() { return (size_t)kMinMaxBlocks * 2 * sizeof(uint32_t); }

hipError_t launch_minmax(const void *x, egeria_dtype dt, int64_t n, uint32_t *partials, uint32_t *reset, int n_reset,
                         hipStream_t st)
{
    const dim3 grid((unsigned)minmax_blocks(n)), block(256);
    if (dt == EGERIA_BF16) return launch_k(EGERIA_KERNEL_ABSMAX, minmax_kernel<true>, grid, block, 0, st, x, n, partials, reset, n_reset);
    return launch_k(EGERIA_KERNEL_ABSMAX, minmax_kernel<false>, grid, block, 0, st, x, n, partials, reset, n_reset);
}

hipError_t launch_quantize_affine(const void *x, egeria_dtype dt, int64_t n, int64_t c, int64_t hw, int64_t cp,
                                  const uint32_t *partials, int nb, const uint32_t *relu_max, int store_offset, void *q,
                                  float *scale_out, int32_t *zp_out, uint32_t *flag, hipStream_t st)
{
    // whole 16-byte units of fp32 take the wide forms; bf16, odd rows and planes, and other addresses the general one
    const bool wide = dt == EGERIA_F32 && ((uintptr_t)x & 15) == 0;
    const int form = wide && hw == 1 && (c & 3) == 0 ? kRows : (wide && hw > 1 && (hw & 3) == 0 ? kPlanes : kAny);
    // (one workgroup at least: scale and zero point are still written.)  Rows of codes, spread over the tensor / dealt in order of
    // memory, us: 5.2 M values 6.7 / 5.8, 12.8 M 12.0 / 11.0, 25.7 M 21.4 / 20.9; larger than the L2s together can help with 50 M
    // 36.3 / 37.9, 200 M 186 / 190.
    const UnitShare sh = share_units(n * hw * (cp >> 4) / (form == kPlanes ? 4 : 1));
    const dim3 grid(sh.blocks), block(256);
    auto go = [&](auto kernel) {
        return launch_k(EGERIA_KERNEL_QUANTIZE, kernel, grid, block, 0, st, x, n, c, hw, cp, partials, nb, relu_max, store_offset,
                        (uint8_t *)q, scale_out, zp_out, flag, sh.per);
    };
    if (dt == EGERIA_BF16) return go(quantize_affine_kernel<true, kAny>);
    if (form == kRows) return go(quantize_affine_kernel<false, kRows>);
    if (form == kPlanes) return go(quantize_affine_kernel<false, kPlanes>);
    return go(quantize_affine_kernel<false, kAny>);
}

hipError_t launch_colsum(const int8_t *w_q, int32_t out, int32_t taps, int32_t cp, int32_t *colsum, hipStream_t st)
{
    if (out <= 0) return hipSuccess;
    return launch_k(EGERIA_KERNEL_NONE, colsum_kernel, dim3((unsigned)((out + 3) / 4)), dim3(256), 0, st, w_q, out, taps, cp,
                    colsum);
}

}  // namespace egeria
