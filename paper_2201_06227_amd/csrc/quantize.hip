// Per-tensor symmetric int8 quantisation (Section 4.1 of the paper: the
// reference model is an int8 post-training-quantised snapshot).  Two coalesced
// HBM passes per tensor: an absolute-maximum reduction, then the map to codes.
#include "gelu.hpp"
#include <type_traits>

namespace egeria {

// ---- absolute maximum -------------------------------------------------------------
__device__ __forceinline__ uint32_t max4_bits(float4 v)
{
    uint32_t a = abs_bits(v.x), b = abs_bits(v.y), c = abs_bits(v.z), d = abs_bits(v.w);
    a = a > b ? a : b;
    c = c > d ? c : d;
    return a > c ? a : c;
}

// Each workgroup writes the maximum of its share, a contiguous piece of the tensor, to partials[blk]
// (bit pattern of |x|, so NaN and Inf order above every finite value).
// (workgroup blk of nblks; a device function so that other kernels can carry the pass along.  Workgroup 0's id is a multiple
// of 8.)
template <bool BF16>
__device__ __forceinline__ void absmax_share(const void *__restrict__ xv, int64_t n, uint32_t *__restrict__ partials,
                                             uint32_t *__restrict__ reset, int n_reset, int blk, int nblks)
{
    if (blk == 0) {
        for (int t = threadIdx.x; t < n_reset * kAmaxWays; t += blockDim.x) {
            uint32_t *way = reset + (size_t)(t / kAmaxWays) * kAmaxWays * kAmaxStride + (t % kAmaxWays) * kAmaxStride;
            way[0] = 0u;
            way[1] = 0u;                     // (the second word of a GELU's slot, see GemmArgs::gelu_neg)
        }
        // `reset` is the first atomic slot, kHeaderFixedWords words into the workspace: the header's
        // counter of re-evaluated attention values starts every chain at zero as well
        if (n_reset > 0 && threadIdx.x == 0) reset[kUnsureWord - kHeaderFixedWords] = 0u;
    }
    const uint32_t piece = xcd_piece((uint32_t)blk, (uint32_t)nblks);
    uint32_t m = 0;
    // 16-byte units of the piece, four of a thread's in flight (the last index repeated: a value seen twice changes nothing)
    auto units = [&](int64_t nu, auto unit_max) {
        const int64_t per = (int64_t)((uint64_t)(nu + nblks - 1) / (uint32_t)nblks), beg = (int64_t)piece * per;
        const int64_t end = beg + per < nu ? beg + per : nu;
        for (int64_t i = beg + threadIdx.x; i < end; i += 1024) {
            uint4 v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = ((const uint4 *)xv)[i + 256 * k < end ? i + 256 * k : end - 1];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t a = unit_max(v[k]);
                m = m > a ? m : a;
            }
        }
    };
    if (!BF16) {
        units(n >> 2, [&](const uint4 &v) {
            return max4_bits(make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w)));
        });
    } else {
        units(n >> 3, [&](const uint4 &v) {
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
            uint32_t r = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t lo = (w[j] << 16) & 0x7fffffffu, hi = w[j] & 0x7fff0000u;
                lo = lo > hi ? lo : hi;
                r = r > lo ? r : lo;
            }
            return r;
        });
    }
    // the values after the last whole unit
    if (piece == 0) {
        const int64_t k = (BF16 ? n >> 3 << 3 : n >> 2 << 2) + threadIdx.x;
        if (k < n) {
            const uint32_t a = BF16 ? ((uint32_t)((const uint16_t *)xv)[k] << 16) & 0x7fffffffu : abs_bits(((const float *)xv)[k]);
            m = m > a ? m : a;
        }
    }
    m = wave_max_u32(m);
    __shared__ uint32_t sm[4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) sm[wv] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t a = sm[0] > sm[1] ? sm[0] : sm[1], b = sm[2] > sm[3] ? sm[2] : sm[3];
        partials[blk] = a > b ? a : b;
    }
}

template <bool BF16>
__global__ __launch_bounds__(256) void absmax_kernel(const void *__restrict__ xv, int64_t n,
                                                     uint32_t *__restrict__ partials,
                                                     uint32_t *__restrict__ reset, int n_reset)
{
    absmax_share<BF16>(xv, n, partials, reset, n_reset, (int)blockIdx.x, (int)gridDim.x);
}

int absmax_blocks(int64_t n, egeria_dtype dt)
{
    const int64_t per = dt == EGERIA_F32 ? 4 : 8;
    int64_t blocks = (n / per + 256 * 4 - 1) / (256 * 4);            // about four vectors per thread
    if (blocks < 1) blocks = 1;
    if (blocks > kAbsPartials) blocks = kAbsPartials;
    return (int)blocks;
}

hipError_t launch_absmax(const void *x, egeria_dtype dt, int64_t n, uint32_t *partials, uint32_t *reset,
                         int n_reset, hipStream_t st)
{
    const dim3 grid((unsigned)absmax_blocks(n, dt)), block(256);
    if (dt == EGERIA_F32)
        return launch_k(EGERIA_KERNEL_ABSMAX, absmax_kernel<false>, grid, block, 0, st, x, n, partials, reset, n_reset);
    return launch_k(EGERIA_KERNEL_ABSMAX, absmax_kernel<true>, grid, block, 0, st, x, n, partials, reset, n_reset);
}

template <bool BF16>
__device__ __forceinline__ float load_elem(const void *x, int64_t i)
{
    if (BF16) return bf16_to_f32(((const uint16_t *)x)[i]);
    return ((const float *)x)[i];
}

// The map to codes of a [rows, cols] matrix: unit u = 16 consecutive codes of one row (one
// 16-byte store); this thread takes units first, first + stride, ... below `end` (at most rows * ldq / 16)
template <bool BF16>
__device__ __forceinline__ void quantize_row_units(const void *__restrict__ x, int64_t rows, int64_t cols, int64_t ldq,
                                                   float inv, int8_t *__restrict__ q, int64_t first, int64_t end, int64_t stride)
{
    const int64_t upr = (ldq + 15) >> 4;                     // 16-byte units per row
    const int64_t units = end < rows * upr ? end : rows * upr;
    const bool narrow = units < (1LL << 32);
    const bool vec_ok = BF16 ? ((cols & 7) == 0) : ((cols & 3) == 0);
    int64_t u = first;
    if (!BF16 && cols == ldq && (cols & 15) == 0 && ((uintptr_t)x & 15) == 0 && ((uintptr_t)q & 15) == 0) {
        // fp32 rows without padding are one contiguous run of whole units (cols a multiple of 16, so
        // the last unit ends where the tensor ends): four of a thread's units (sixteen 16-byte loads)
        // in flight together when it has that many (a single workgroup quantising a whole small
        // matrix would otherwise pay one memory round trip per unit)
        const float4 *x4 = (const float4 *)x;
        for (; u + 3 * stride < units; u += 4 * stride) {
            float4 v[4][4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j) v[k][j] = x4[(u + k * stride) * 4 + j];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                uint32_t w[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    w[j] = quant1(v[k][j].x, inv) | (quant1(v[k][j].y, inv) << 8) | (quant1(v[k][j].z, inv) << 16) |
                           (quant1(v[k][j].w, inv) << 24);
                *(uint4 *)(q + ((u + k * stride) << 4)) = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
    }
    for (; u < units; u += stride) {
        const int64_t row = div_u(u, upr, narrow);
        const int64_t c0 = (u - row * upr) << 4;
        const int64_t base = row * cols + c0;
        uint32_t w[4] = {0, 0, 0, 0};
        if (vec_ok && c0 + 16 <= cols) {
            if (!BF16) {
                const float4 *p = (const float4 *)((const float *)x + base);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    float4 v = p[j];
                    w[j] = quant1(v.x, inv) | (quant1(v.y, inv) << 8) | (quant1(v.z, inv) << 16) |
                           (quant1(v.w, inv) << 24);
                }
            } else {
                const uint4 *p = (const uint4 *)((const uint16_t *)x + base);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    uint4 v = p[j];
                    uint32_t s[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        uint32_t lo = quant1(__uint_as_float(s[e] << 16), inv);
                        uint32_t hi = quant1(__uint_as_float(s[e] & 0xffff0000u), inv);
                        int o = j * 8 + e * 2;
                        w[o >> 2] |= (lo << ((o & 3) * 8)) | (hi << (((o + 1) & 3) * 8));
                    }
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (c0 + e < cols) w[e >> 2] |= quant1(load_elem<BF16>(x, base + e), inv) << ((e & 3) * 8);
        }
        int8_t *dst = q + row * ldq + c0;
        if (c0 + 16 <= ldq && (((row * ldq) & 15) == 0)) {
            *(uint4 *)dst = make_uint4(w[0], w[1], w[2], w[3]);
        } else {
            for (int e = 0; e < 16 && c0 + e < ldq; ++e) dst[e] = (int8_t)((w[e >> 2] >> ((e & 3) * 8)) & 0xff);
        }
    }
}

// ---- quantise [rows, cols] -> int8 [rows, ldq] ---------------------------------------
// One thread produces 16 consecutive codes of one row (one 16-byte store).
template <bool BF16>
__global__ __launch_bounds__(256) void quantize_rows_kernel(
    const void *__restrict__ x, int64_t rows, int64_t cols, int64_t ldq,
    const uint32_t *__restrict__ slot, int n_slot, int slot_stride,
    const float *__restrict__ fixed_scale,
    int8_t *__restrict__ q, float *__restrict__ scale_out, float *__restrict__ scale_out2,
    uint32_t *__restrict__ flag, int64_t per, bool flat)
{
    float scale;
    bool bad;
    const int64_t beg = xcd_piece(blockIdx.x, gridDim.x) * per;
    if (!BF16 && flat) {
        // fp32 rows without padding, whole units: one contiguous run.  A thread takes four 16-byte loads 256 units of four
        // values apart, so that every load and store of a wave is contiguous; the first ones go out before the scale
        // is waited for.
        const int64_t n4 = rows * (cols >> 2), end = (beg + per) * 4 < n4 ? (beg + per) * 4 : n4;
        const float4 *x4 = (const float4 *)x;
        float4 v[4];
        const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(q + beg * 16, 0, (int)((end - beg * 4) * 4), kBufferWord);
        auto request = [&](int64_t i) {
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = x4[i + 256 * k < end ? i + 256 * k : end - 1];
        };
        int64_t i = beg * 4 + threadIdx.x;
        request(i);
        const float inv = scales_from(slot, n_slot, slot_stride, fixed_scale, &scale, &bad);
        if (blockIdx.x == 0 && threadIdx.x == 0) publish(scale, bad, scale_out, scale_out2, flag);
        for (;;) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                __builtin_amdgcn_raw_buffer_store_b32(quant1(v[k].x, inv) | (quant1(v[k].y, inv) << 8) | (quant1(v[k].z, inv) << 16) |
                                                          (quant1(v[k].w, inv) << 24),
                                                      rq, (int)(i - beg * 4 + 256 * k) * 4, 0, kThrough);   // (beyond the end: dropped)
            i += 1024;
            if (i - threadIdx.x >= end) break;
            request(i);
        }
        return;
    }
    const float inv = scales_from(slot, n_slot, slot_stride, fixed_scale, &scale, &bad);
    if (blockIdx.x == 0 && threadIdx.x == 0) publish(scale, bad, scale_out, scale_out2, flag);
    quantize_row_units<BF16>(x, rows, cols, ldq, inv, q, beg + threadIdx.x, beg + per, 256);
}

hipError_t launch_quantize_rows(const void *x, egeria_dtype dt, int64_t rows, int64_t cols,
                                int64_t ldq, const uint32_t *slot, int n_slot, int slot_stride,
                                const float *fixed_scale,
                                int8_t *q, float *scale_out, float *scale_out2, uint32_t *flag,
                                hipStream_t st)
{
    const UnitShare sh = share_units(rows * ((ldq + 15) / 16));
    const dim3 grid(sh.blocks), block(256);
    const bool flat = rows > 0 && cols > 0 && cols == ldq && (cols & 15) == 0 && (((uintptr_t)x | (uintptr_t)q) & 15) == 0;
    if (dt == EGERIA_F32)
        return launch_k(EGERIA_KERNEL_QUANTIZE, quantize_rows_kernel<false>, grid, block, 0, st, x, rows, cols, ldq,
                        slot, n_slot, slot_stride, fixed_scale, q, scale_out, scale_out2, flag, sh.per, flat);
    return launch_k(EGERIA_KERNEL_QUANTIZE, quantize_rows_kernel<true>, grid, block, 0, st, x, rows, cols, ldq, slot,
                    n_slot, slot_stride, fixed_scale, q, scale_out, scale_out2, flag, sh.per, false);
}

// ---- quantise [n, c, hw] -> int8 [n, hw, cp] -------------------------------------------
// A workgroup transposes a tile of 64 pixels x 64 channels through LDS: reads
// are contiguous along the pixel axis, writes along the channel axis.
template <bool BF16>
__global__ __launch_bounds__(256) void quantize_nchw_kernel(
    const void *__restrict__ x, int64_t n, int64_t c, int64_t hw, int64_t cp,
    const uint32_t *__restrict__ slot, int n_slot, int slot_stride,
    const float *__restrict__ fixed_scale,
    int8_t *__restrict__ q, float *__restrict__ scale_out, float *__restrict__ scale_out2,
    uint32_t *__restrict__ flag)
{
    float scale;
    bool bad;
    const float inv = scales_from(slot, n_slot, slot_stride, fixed_scale, &scale, &bad);
    if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0)
        publish(scale, bad, scale_out, scale_out2, flag);
    __shared__ uint8_t tile[64][64 + 4];                  // [pixel][channel], padded rows
    const int64_t img = blockIdx.z;
    const int64_t p0 = (int64_t)blockIdx.x * 64, c0 = (int64_t)blockIdx.y * 64;
    const int tp = threadIdx.x & 63, tc = threadIdx.x >> 6;   // pixel lane, channel phase
#pragma unroll 4
    for (int i = 0; i < 16; ++i) {
        const int64_t ch = c0 + tc + 4 * i, p = p0 + tp;
        uint32_t code = 0;
        if (ch < c && p < hw) code = quant1(load_elem<BF16>(x, (img * c + ch) * hw + p), inv);
        tile[tp][tc + 4 * i] = (uint8_t)code;
    }
    __syncthreads();
    // 64 pixels x 4 units of 16 channels = 256 stores of 16 bytes
    const int pix = threadIdx.x >> 2, un = threadIdx.x & 3;
    const int64_t p = p0 + pix, ch0 = c0 + un * 16;
    if (p < hw && ch0 < cp) {
        const uint32_t *src = (const uint32_t *)&tile[pix][un * 16];
        *(uint4 *)(q + (img * hw + p) * cp + ch0) = make_uint4(src[0], src[1], src[2], src[3]);
    }
}

// Same map without the LDS stage, for fp32 input whose pixel count is a
// multiple of 4: a thread owns 4 consecutive pixels x 16 channels (sixteen
// 16-byte loads, lanes along the pixel axis, all in flight together) and
// writes four 16-byte channel groups.
// (this thread takes units first, first + stride, ... below `end`, at most n * cp / 16 * hw / 4)
__device__ __forceinline__ void quantize_nchw_vec_units(const float *__restrict__ x, int64_t n, int64_t c, int64_t hw,
                                                        int64_t cp, float inv, int8_t *__restrict__ q, int64_t first,
                                                        int64_t end, int64_t stride)
{
    const int64_t pq = hw >> 2, cg = cp >> 4;
    const int64_t units = end < n * cg * pq ? end : n * cg * pq;
    const bool narrow = units < (1LL << 32);
    for (int64_t u = first; u < units; u += stride) {
        const int64_t ig = div_u(u, pq, narrow);
        const int64_t p = (u - ig * pq) << 2;
        const int64_t img = div_u(ig, cg, narrow), g = ig - img * cg;
        const int64_t ch0 = g << 4;
        float4 v[16];
#pragma unroll
        for (int e = 0; e < 16; ++e)
            v[e] = ch0 + e < c ? *(const float4 *)(x + (img * c + ch0 + e) * hw + p) : make_float4(0.f, 0.f, 0.f, 0.f);
        uint32_t w[4][4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) w[k][j] = 0;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const uint32_t sh = (e & 3) * 8;
            uint32_t c0 = quant1(v[e].x, inv), c1 = quant1(v[e].y, inv), c2 = quant1(v[e].z, inv), c3 = quant1(v[e].w, inv);
            if (ch0 + e >= c) c0 = c1 = c2 = c3 = 0;                  // pad channels are zero even when inv is not finite
            w[0][e >> 2] |= c0 << sh;
            w[1][e >> 2] |= c1 << sh;
            w[2][e >> 2] |= c2 << sh;
            w[3][e >> 2] |= c3 << sh;
        }
        int8_t *dst = q + (img * hw + p) * cp + ch0;
#pragma unroll
        for (int k = 0; k < 4; ++k) *(uint4 *)(dst + k * cp) = make_uint4(w[k][0], w[k][1], w[k][2], w[k][3]);
    }
}

__global__ __launch_bounds__(256) void quantize_nchw_vec_kernel(
    const float *__restrict__ x, int64_t n, int64_t c, int64_t hw, int64_t cp,
    const uint32_t *__restrict__ slot, int n_slot, int slot_stride,
    const float *__restrict__ fixed_scale,
    int8_t *__restrict__ q, float *__restrict__ scale_out, float *__restrict__ scale_out2,
    uint32_t *__restrict__ flag, int64_t per)
{
    float scale;
    bool bad;
    const float inv = scales_from(slot, n_slot, slot_stride, fixed_scale, &scale, &bad);
    if (blockIdx.x == 0 && threadIdx.x == 0) publish(scale, bad, scale_out, scale_out2, flag);
    const int64_t beg = xcd_piece(blockIdx.x, gridDim.x) * per;
    quantize_nchw_vec_units(x, n, c, hw, cp, inv, q, beg + threadIdx.x, beg + per, 256);
}

// fp32 planes of an odd number of pixels (7x7, 13x13): `group` channels of an image with all their pixels, which lie side by side in
// memory, pass through LDS and come back as pixels x channels.  The loads are whole 16-byte units along memory, whatever the
// length of a plane (a load per value, 49 of 64 lanes at work, took 9.0 us for 50 x 2048 x 49; 6.2 this way).  Rows of the LDS
// tile are padded by a word: lanes hold values four pixels apart, at most four of them fall on one bank.
constexpr int64_t kPlaneMax = 1024;          // pixels of such a plane
__global__ __launch_bounds__(256) void quantize_planes_kernel(
    const float *__restrict__ x, int c, int hw, int cp, int group, uint32_t hw_magic, const uint32_t *__restrict__ slot, int n_slot,
    int slot_stride, const float *__restrict__ fixed_scale, int8_t *__restrict__ q, float *__restrict__ scale_out,
    float *__restrict__ scale_out2, uint32_t *__restrict__ flag)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t turn[];           // [hw][group + 4]
    const uint32_t groups = (uint32_t)((cp + group - 1) / group), piece = xcd_piece(blockIdx.x, gridDim.x);
    const uint32_t img = piece / groups;
    const int ch0 = (int)(piece - img * groups) * group, ld = group + 4, chs = c - ch0 < group ? c - ch0 : group;
    const int n4 = chs > 0 ? chs * hw / 4 : 0;                                // (c is a multiple of 4)
    const float4 *src = (const float4 *)(x + ((int64_t)img * c + ch0) * hw);
    constexpr int NP = 4;
    float4 v[NP];
    auto request = [&](int i) {
#pragma unroll
        for (int k = 0; k < NP; ++k) v[k] = src[i + 256 * k < n4 ? i + 256 * k : n4 - 1];
    };
    if (n4 > 0) request((int)threadIdx.x);
    if (chs < group) {                                                        // pad channels are zero
        for (int i = threadIdx.x; i < hw * ld / 4; i += 256) ((uint32_t *)turn)[i] = 0u;
        __syncthreads();
    }
    float scale;
    bool bad;
    const float inv = scales_from(slot, n_slot, slot_stride, fixed_scale, &scale, &bad);
    if (blockIdx.x == 0 && threadIdx.x == 0) publish(scale, bad, scale_out, scale_out2, flag);
    for (int i = threadIdx.x; i < n4; i += 256 * NP) {
        if (i >= 256 * NP) request(i);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int at = i + 256 * k;
            if (at >= n4) break;
            uint32_t ch = __umulhi((uint32_t)at * 4u, hw_magic), p = (uint32_t)at * 4u - ch * (uint32_t)hw;
            const float e[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                turn[p * (uint32_t)ld + ch] = (uint8_t)quant1(e[j], inv);
                if (++p == (uint32_t)hw) { p = 0; ++ch; }
            }
        }
    }
    __syncthreads();
    const int upp = group / 16;                                               // 16-byte units per pixel: 1, 2 or 4
    for (int u = threadIdx.x; u < hw * upp; u += 256) {
        const int p = u / upp, un = u % upp;
        const uint32_t *w = (const uint32_t *)&turn[p * ld + un * 16];
        if (ch0 + un * 16 < cp) *(uint4 *)(q + ((int64_t)img * hw + p) * cp + ch0 + un * 16) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

hipError_t launch_quantize_nchw(const void *x, egeria_dtype dt, int64_t n, int64_t c, int64_t hw,
                                int64_t cp, const uint32_t *slot, int n_slot, int slot_stride,
                                const float *fixed_scale,
                                int8_t *q, float *scale_out, float *scale_out2, uint32_t *flag,
                                hipStream_t st)
{
    const dim3 grid((unsigned)((hw + 63) / 64), (unsigned)((cp + 63) / 64), (unsigned)n), block(256);
    if (dt == EGERIA_F32 && (hw & 3) == 0 && hw >= 4 && n > 0 && c > 0) {
        const UnitShare sh = share_units(n * (cp >> 4) * (hw >> 2));
        return launch_k(EGERIA_KERNEL_QUANTIZE, quantize_nchw_vec_kernel, dim3(sh.blocks), block, 0, st,
                        (const float *)x, n, c, hw, cp, slot, n_slot, slot_stride, fixed_scale, q, scale_out, scale_out2,
                        flag, sh.per);
    }
    if (dt == EGERIA_F32 && (hw & 3) != 0 && hw > 1 && hw <= kPlaneMax && c > 0 && (c & 3) == 0 && cp < (1 << 30)) {
        const int group = hw <= 64 ? 64 : (hw <= 128 ? 32 : 16);
        const int64_t blocks = n * ((cp + group - 1) / group);
        if (blocks > 0 && blocks < (1 << 24))
            return launch_k(EGERIA_KERNEL_QUANTIZE, quantize_planes_kernel, dim3((unsigned)blocks), block, (size_t)(hw * (group + 4) + 12) & ~(size_t)15, st,
                            (const float *)x, (int)c, (int)hw, (int)cp, group, (uint32_t)(0x100000000ull / (uint64_t)hw) + 1u, slot, n_slot, slot_stride,
                            fixed_scale, q, scale_out, scale_out2, flag);
    }
    if (dt == EGERIA_F32)
        return launch_k(EGERIA_KERNEL_QUANTIZE, quantize_nchw_kernel<false>, grid, block, 0, st, x, n, c, hw, cp, slot,
                        n_slot, slot_stride, fixed_scale, q, scale_out, scale_out2, flag);
    return launch_k(EGERIA_KERNEL_QUANTIZE, quantize_nchw_kernel<true>, grid, block, 0, st, x, n, c, hw, cp, slot,
                    n_slot, slot_stride, fixed_scale, q, scale_out, scale_out2, flag);
}

// ---- small tensors: one workgroup, one launch -----------------------------------------------
// Absolute maximum, scale and codes of a tensor of a few thousand values
// (convolution weights of a narrow layer, a small mini-batch): both passes in
// one workgroup, so the tensor costs one kernel launch instead of two.
// General form [nimg, c, hw] -> int8 [nimg, hw, cp]; a row-major matrix is the
// case hw = 1.
template <bool BF16>
__device__ __forceinline__ void quantize_small_body(const void *__restrict__ x, int nimg, int c, int hw, int cp,
                                                    int8_t *__restrict__ q, float *__restrict__ scale_out,
                                                    uint32_t *__restrict__ flag)
{
    const int total = nimg * c * hw;
    uint32_t m = 0;
    if (!BF16 && ((uintptr_t)x & 15) == 0) {
        // 16-byte loads, four of them requested together
        const float4 *x4 = (const float4 *)x;
        const int n4 = total >> 2;
        int i = threadIdx.x;
        for (; i + 768 < n4; i += 1024) {
            const float4 v0 = x4[i], v1 = x4[i + 256], v2 = x4[i + 512], v3 = x4[i + 768];
            uint32_t a = max4_bits(v0), b = max4_bits(v1), cc = max4_bits(v2), d = max4_bits(v3);
            a = a > b ? a : b;
            cc = cc > d ? cc : d;
            a = a > cc ? a : cc;
            m = m > a ? m : a;
        }
        for (; i < n4; i += 256) {
            const uint32_t a = max4_bits(x4[i]);
            m = m > a ? m : a;
        }
        for (int k = (n4 << 2) + threadIdx.x; k < total; k += 256) {
            const uint32_t a = abs_bits(((const float *)x)[k]);
            m = m > a ? m : a;
        }
    } else {
        for (int i = threadIdx.x; i < total; i += 256) {
            const uint32_t a = abs_bits(load_elem<BF16>(x, i));
            m = m > a ? m : a;
        }
    }
    m = wave_max_u32(m);
    __shared__ uint32_t sm[4];
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = m;
    __syncthreads();
    float scale;
    bool bad;
    const float inv = scales_from(sm, 4, 1, nullptr, &scale, &bad);
    if (threadIdx.x == 0) publish(scale, bad, scale_out, nullptr, flag);
    if (hw == 1) {                                   // rows of a matrix: 16 codes per thread and store
        quantize_row_units<BF16>(x, nimg, c, cp, inv, q, threadIdx.x, (int64_t)nimg * ((cp + 15) >> 4), 256);
        return;
    }
    const int nout = nimg * hw * cp;
    for (int o = threadIdx.x; o < nout; o += 256) {
        const int ch = o % cp, pp = (o / cp) % hw, img = o / (cp * hw);
        uint32_t code = 0;
        if (ch < c) code = quant1(load_elem<BF16>(x, ((int64_t)img * c + ch) * hw + pp), inv);
        q[o] = (int8_t)code;
    }
}

template <bool BF16>
__global__ __launch_bounds__(256) void quantize_small_kernel(const void *__restrict__ x, int nimg, int c, int hw,
                                                             int cp, int8_t *__restrict__ q,
                                                             float *__restrict__ scale_out,
                                                             uint32_t *__restrict__ flag)
{
    quantize_small_body<BF16>(x, nimg, c, hw, cp, q, scale_out, flag);
}

hipError_t launch_quantize_small(const void *x, egeria_dtype dt, int nimg, int c, int hw, int cp, int8_t *q,
                                 float *scale_out, uint32_t *flag, hipStream_t st)
{
    if (dt == EGERIA_F32)
        return launch_k(EGERIA_KERNEL_QUANTIZE, quantize_small_kernel<false>, dim3(1), dim3(256), 0, st, x, nimg, c, hw,
                        cp, q, scale_out, flag);
    return launch_k(EGERIA_KERNEL_QUANTIZE, quantize_small_kernel<true>, dim3(1), dim3(256), 0, st, x, nimg, c, hw, cp,
                    q, scale_out, flag);
}

// ---- a whole snapshot of weight tensors in one or two launches ------------------------------
// Every workgroup finds its tensor in the launch's table (kernel argument) and
// works on a fixed share of it: first the maximum of its share of the values,
// then its share of the 16-byte output units [o][hw][cp / 16].
// (one load per lane and a ballot; walking the table is a chain of scalar loads, up to 32 long)
__device__ __forceinline__ int find_job(const WeightBatch &b, int blk)
{
    const int lane = threadIdx.x & 63;
    const int first = b.job[lane < kWeightBatch ? lane : kWeightBatch - 1].first_block;
    return __popcll(__ballot(lane < b.n && blk >= first)) - 1;     // first_block ascends, job 0 starts at 0
}

__device__ __forceinline__ uint32_t job_share_absmax(const WeightJob &jb, int lb, uint32_t *sm)
{
    const int64_t n_in = (int64_t)jb.o * jb.c * jb.hw;
    const int64_t beg = (int64_t)lb * jb.epb;
    int64_t end = beg + jb.epb;
    if (end > n_in) end = n_in;
    uint32_t m = 0;
    if (!jb.bf16) {
        const float *x = (const float *)jb.x;
        const int64_t n4 = end > beg ? (end - beg) >> 2 : 0;
        const float4 *x4 = (const float4 *)(x + beg);                // epb is a multiple of 8
        int64_t i = threadIdx.x;
        for (; i + 1792 < n4; i += 2048) {                           // eight independent loads in flight
            float4 v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = x4[i + 256 * k];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint32_t a = max4_bits(v[k]);
                m = m > a ? m : a;
            }
        }
        for (; i + 768 < n4; i += 1024) {                            // four
            const float4 v0 = x4[i], v1 = x4[i + 256], v2 = x4[i + 512], v3 = x4[i + 768];
            uint32_t a = max4_bits(v0), b = max4_bits(v1), c = max4_bits(v2), d = max4_bits(v3);
            a = a > b ? a : b;
            c = c > d ? c : d;
            a = a > c ? a : c;
            m = m > a ? m : a;
        }
        if (i < n4) {                                                // at most three strides are left: one round trip
            float4 t[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) t[k] = x4[i + 256 * k < n4 ? i + 256 * k : n4 - 1];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const uint32_t a = i + 256 * k < n4 ? max4_bits(t[k]) : 0u;
                m = m > a ? m : a;
            }
        }
        for (int64_t k = beg + (n4 << 2) + threadIdx.x; k < end; k += 256) {
            const uint32_t a = abs_bits(x[k]);
            m = m > a ? m : a;
        }
    } else {
        // 16-byte loads, four in flight (with a load per value 28.3 M values, both passes, took 124 us, now 52)
        const uint16_t *x = (const uint16_t *)jb.x;
        const int64_t n8 = end > beg ? (end - beg) >> 3 : 0;
        const uint4 *x8 = (const uint4 *)(x + beg);
        for (int64_t i = threadIdx.x; i < n8; i += 1024) {
            uint4 t[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) t[k] = x8[i + 256 * k < n8 ? i + 256 * k : n8 - 1];   // (a repeated unit changes no maximum)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t w[4] = {t[k].x, t[k].y, t[k].z, t[k].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t lo = (w[e] << 16) & 0x7fffffffu, hi = w[e] & 0x7fff0000u;
                    const uint32_t a = lo > hi ? lo : hi;
                    m = m > a ? m : a;
                }
            }
        }
        for (int64_t k = beg + (n8 << 3) + threadIdx.x; k < end; k += 256) {
            const uint32_t a = ((uint32_t)x[k] << 16) & 0x7fffffffu;
            m = m > a ? m : a;
        }
    }
    m = wave_max_u32(m);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = m;
    __syncthreads();
    const uint32_t a = sm[0] > sm[1] ? sm[0] : sm[1], b = sm[2] > sm[3] ? sm[2] : sm[3];
    return a > b ? a : b;
}

// Tensors of one launch report to the same flag word at the same time.
__device__ __forceinline__ void publish_shared(float scale, bool bad, float *scale_out, uint32_t *flag)
{
    *scale_out = scale;
    uint32_t old = *flag;
    for (;;) {
        uint32_t want = (old & 0xffffff00u) == kFlagMagic ? old : kFlagMagic;
        if (bad) want |= kFlagNonFinite;
        if (want == old) break;
        const uint32_t seen = atomicCAS(flag, old, want);
        if (seen == old) break;
        old = seen;
    }
}

__device__ __forceinline__ void job_share_quantize(const WeightJob &jb, int lb, float inv)
{
    const int cpu = jb.cp >> 4;
    const int64_t units = (int64_t)jb.o * jb.hw * cpu;
    const int64_t beg = (int64_t)lb * jb.upb;
    int64_t end = beg + jb.upb;
    if (end > units) end = units;
    const bool rows_vec = jb.hw == 1 && !jb.bf16 && (jb.c & 3) == 0;
    const bool rows_vec8 = jb.hw == 1 && jb.bf16 && (jb.c & 7) == 0;
    const bool narrow = units < (1LL << 32);
    int64_t u = beg + threadIdx.x;
    // sixteen codes of two 16-byte units of bf16 values
    auto codes_of = [&](const uint4 &a, const uint4 &b) {
        const uint32_t s[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            w[j] = quant1(__uint_as_float(s[2 * j] << 16), inv) | (quant1(__uint_as_float(s[2 * j] & 0xffff0000u), inv) << 8) |
                   (quant1(__uint_as_float(s[2 * j + 1] << 16), inv) << 16) | (quant1(__uint_as_float(s[2 * j + 1] & 0xffff0000u), inv) << 24);
        return make_uint4(w[0], w[1], w[2], w[3]);
    };
    if (rows_vec8 && jb.c == jb.cp) {
        const uint4 *x8 = (const uint4 *)jb.x;
        for (; u + 768 < end; u += 1024) {
            uint4 v[4][2];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v[k][0] = x8[(u + 256 * k) * 2];
                v[k][1] = x8[(u + 256 * k) * 2 + 1];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) *(uint4 *)(jb.q + ((u + 256 * k) << 4)) = codes_of(v[k][0], v[k][1]);
        }
    }
    if (rows_vec && jb.c == jb.cp) {
        // rows without padding are one run of whole units: four of a thread's in flight together
        const float4 *x4 = (const float4 *)jb.x;
        for (; u + 768 < end; u += 1024) {
            float4 v[4][4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j) v[k][j] = x4[(u + 256 * k) * 4 + j];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                uint32_t w[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    w[j] = quant1(v[k][j].x, inv) | (quant1(v[k][j].y, inv) << 8) | (quant1(v[k][j].z, inv) << 16) | (quant1(v[k][j].w, inv) << 24);
                *(uint4 *)(jb.q + ((u + 256 * k) << 4)) = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
    }
    for (; u < end; u += 256) {
        const int64_t op = div_u(u, cpu, narrow);         // o * hw + pixel
        const int c0 = (int)(u - op * cpu) << 4;
        const int64_t oc = div_u(op, jb.hw, narrow);
        const int pix = (int)(op - oc * jb.hw);
        uint32_t w[4] = {0, 0, 0, 0};
        if (rows_vec8 && c0 + 16 <= jb.c) {
            const uint4 *p = (const uint4 *)((const uint16_t *)jb.x + oc * jb.c + c0);
            const uint4 r = codes_of(p[0], p[1]);
            w[0] = r.x; w[1] = r.y; w[2] = r.z; w[3] = r.w;
        } else if (rows_vec && c0 + 16 <= jb.c) {
            const float4 *p = (const float4 *)((const float *)jb.x + oc * jb.c + c0);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float4 v = p[j];
                w[j] = quant1(v.x, inv) | (quant1(v.y, inv) << 8) | (quant1(v.z, inv) << 16) | (quant1(v.w, inv) << 24);
            }
        } else {
            // sixteen gathered values, requested together: unconditional loads (a channel beyond c reads
            // channel c - 1 and is dropped), since a load under a per-lane condition is awaited on its own
            float v[16];
            if (jb.bf16) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int ch = c0 + e < jb.c ? c0 + e : jb.c - 1;
                    v[e] = bf16_to_f32(((const uint16_t *)jb.x)[(oc * jb.c + ch) * jb.hw + pix]);
                }
            } else {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int ch = c0 + e < jb.c ? c0 + e : jb.c - 1;
                    v[e] = ((const float *)jb.x)[(oc * jb.c + ch) * jb.hw + pix];
                }
            }
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (c0 + e < jb.c) w[e >> 2] |= quant1(v[e], inv) << ((e & 3) * 8);
        }
        *(uint4 *)(jb.q + (u << 4)) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// PHASE 0: every tensor of the launch fits one workgroup; maximum, scale and codes in one go.
// PHASE 1: per-workgroup maxima -> partials[blockIdx.x].   PHASE 2: scale from the partials, codes.
// Workgroups beyond the table's total_blocks (first launch of a snapshot only) take a share of
// an unrelated maximum pass that the caller wants in the same launch: the mini-batch the
// refreshed reference model is about to run on.
template <int PHASE>
__global__ __launch_bounds__(256) void quantize_weights_kernel(const WeightBatch b, uint32_t *__restrict__ partials,
                                                               uint32_t *__restrict__ flag, int total_blocks,
                                                               const InputMaxJob extra, const InputQuantJob xq)
{
    if ((int)blockIdx.x >= total_blocks) {
        // (the others start at an id that is a multiple of 8: pieces are dealt by XCD)
        const int blk = (int)blockIdx.x - (total_blocks + 7) / 8 * 8;
        if (blk < 0) return;
        if (PHASE == 2 && xq.kind != 0) {
            // second launch: the codes of the mini-batch whose maxima the first launch took
            float scale;
            bool bad;
            const float inv = scales_from(xq.slot, xq.n_slot, 1, nullptr, &scale, &bad);
            if (blk == 0 && threadIdx.x == 0) publish(scale, bad, xq.scale_out, nullptr, xq.flag);
            const int64_t beg = xcd_piece((uint32_t)blk, (uint32_t)xq.nblk) * xq.per, first = beg + threadIdx.x, end = beg + xq.per;
            if (xq.kind == 2) quantize_nchw_vec_units((const float *)xq.x, xq.rows, xq.cols, xq.hw, xq.ldq, inv, xq.q, first, end, 256);
            else if (xq.bf16) quantize_row_units<true>(xq.x, xq.rows, xq.cols, xq.ldq, inv, xq.q, first, end, 256);
            else quantize_row_units<false>(xq.x, xq.rows, xq.cols, xq.ldq, inv, xq.q, first, end, 256);
            return;
        }
        if (PHASE != 2 && extra.q) {
            // a small mini-batch [rows, cols]: maximum, scale and codes by this one workgroup
            if (extra.bf16) quantize_small_body<true>(extra.x, extra.rows, extra.cols, 1, extra.cp, extra.q, extra.scale_out, extra.flag);
            else quantize_small_body<false>(extra.x, extra.rows, extra.cols, 1, extra.cp, extra.q, extra.scale_out, extra.flag);
        } else if (PHASE != 2) {
            if (extra.bf16) absmax_share<true>(extra.x, extra.n, extra.partials, extra.reset, extra.n_reset, blk, extra.nblk);
            else absmax_share<false>(extra.x, extra.n, extra.partials, extra.reset, extra.n_reset, blk, extra.nblk);
        }
        return;
    }
    __shared__ uint32_t sm[4];
    const int j = find_job(b, (int)blockIdx.x);
    const WeightJob &jb = b.job[j];
    const int lb = (int)blockIdx.x - jb.first_block;
    if (PHASE == 1) {
        const uint32_t m = job_share_absmax(jb, lb, sm);
        if (threadIdx.x == 0) partials[blockIdx.x] = m;
        return;
    }
    float scale;
    bool bad;
    float inv;
    if (PHASE == 0) {
        (void)job_share_absmax(jb, lb, sm);
        inv = scales_from(sm, 4, 1, nullptr, &scale, &bad);
    } else {
        inv = scales_from(partials + jb.first_block, jb.nblk, 1, nullptr, &scale, &bad);
    }
    if (lb == 0 && threadIdx.x == 0) publish_shared(scale, bad, jb.scale, flag);
    job_share_quantize(jb, lb, inv);
}

// One scale per output channel: a wave owns channel oc of its tensor, reads the channel's c * hw values once
// with 16-byte loads into registers, takes the maximum, publishes the scale and maps the registers to the
// channel's codes [hw][cp].  No barrier, one launch.
// Bound by HBM (4 or 2 bytes read, 1 written per value).  All of a row's loads are in flight together: NV units
// of EPU values per lane (3 for rows of up to 768 floats, 12 up to 3072; what is longer is read a second time,
// from cache).  A linear layer's codes leave as one 4- or 8-byte store per unit, lanes side by side; where the
// codes of a unit are not neighbours (3x3 kernels, odd row lengths) they are put in place in LDS first and
// leave as 16-byte stores.  Reading 16 neighbouring values per lane with scalar loads (64 cache lines per
// instruction) took 119 us for 28.3 M fp32 values; this form 34 us (4.2 TB/s read + written).  Widths between the two
// counts of units ask for the last unit again (3 of 12 loads of a row of 1024 floats bring new values): still faster,
// the whole call for two encoder layers, before / now, us: hidden 1024 103 / 31, 1280 164 / 38, 2048 420 / 107, 1001 119 / 40.
constexpr int kPcRowLds = 8192;          // bytes of codes of one channel that LDS holds (per wave)

template <bool BF16, int EPU, int NV>
__device__ __forceinline__ void quantize_channel(const WeightJob &jb, int oc, uint8_t *ldsrow, uint32_t *flag, bool first_wave)
{
    using Unit = std::conditional_t<EPU == 1, float, uint4>;
    const int lane = threadIdx.x & 63;
    const int n_row = jb.c * jb.hw, nu = n_row / EPU;             // EPU divides n_row
    const char *row = (const char *)jb.x + (int64_t)oc * n_row * (BF16 ? 2 : 4);
    auto load = [&](int u) -> Unit {
        if constexpr (EPU == 1) return BF16 ? bf16_to_f32(((const uint16_t *)row)[u]) : ((const float *)row)[u];
        else return ((const uint4 *)row)[u];
    };
    auto value = [&](const Unit &v, int e) -> float {
        if constexpr (EPU == 1) return v;
        else {
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
            if (!BF16) return __uint_as_float(w[e]);
            return __uint_as_float((e & 1) ? w[e >> 1] & 0xffff0000u : w[e >> 1] << 16);
        }
    };
    auto unit_max = [&](const Unit &v) {
        uint32_t m = 0;
#pragma unroll
        for (int e = 0; e < EPU; ++e) {
            const uint32_t a = abs_bits(value(v, e));
            m = m > a ? m : a;
        }
        return m;
    };
    Unit v[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = load(lane + 64 * i < nu ? lane + 64 * i : nu - 1);   // (a repeated unit changes no maximum)
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const uint32_t a = unit_max(v[i]);
        m = m > a ? m : a;
    }
    for (int u = lane + 64 * NV; u < nu; u += 64) {
        const uint32_t a = unit_max(load(u));
        m = m > a ? m : a;
    }
    float scale;
    bool bad;
    const float inv = scale_from_bits(wave_max_u32(m), nullptr, &scale, &bad);
    if (lane == 0) {
        if (bad || first_wave) publish_shared(scale, bad, jb.scale + oc, flag);
        else jb.scale[oc] = scale;
    }
    int8_t *q = jb.q + (int64_t)oc * jb.hw * jb.cp;
    const bool direct = EPU > 1 && jb.hw == 1;                    // a row of whole units: its codes are neighbours
    const uint32_t magic = (uint32_t)(0x100000000ull / (uint32_t)jb.hw) + 1u;   // k / hw = mulhi(k, magic) for k * hw < 2^32
    if (!direct && jb.cp != jb.c) {
        for (int o = lane * 16; o < jb.hw * jb.cp; o += 1024) *(uint4 *)(ldsrow + o) = make_uint4(0, 0, 0, 0);
        wave_lds_turn();
    }
    auto emit = [&](const Unit &x, int u) {
        if (direct) {
            uint32_t w[(EPU + 3) / 4];
#pragma unroll
            for (int k = 0; k < (EPU + 3) / 4; ++k) {
                w[k] = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (4 * k + e < EPU) w[k] |= quant1(value(x, 4 * k + e), inv) << (8 * e);
            }
            if constexpr (EPU == 8) *(uint2 *)(q + 8 * u) = make_uint2(w[0], w[1]);
            else *(uint32_t *)(q + 4 * u) = w[0];
        } else {
#pragma unroll
            for (int e = 0; e < EPU; ++e) {
                const uint32_t k = (uint32_t)(u * EPU + e);
                const uint32_t ch = jb.hw == 1 ? k : __umulhi(k, magic);
                ldsrow[(k - ch * (uint32_t)jb.hw) * (uint32_t)jb.cp + ch] = (uint8_t)quant1(value(x, e), inv);
            }
        }
    };
#pragma unroll
    for (int i = 0; i < NV; ++i)
        if (lane + 64 * i < nu) emit(v[i], lane + 64 * i);
    for (int u = lane + 64 * NV; u < nu; u += 64) emit(load(u), u);
    if (direct) {
        for (int c = jb.c + 4 * lane; c < jb.cp; c += 256) *(uint32_t *)(q + c) = 0u;   // pad bytes (jb.c is a multiple of 4)
    } else {
        wave_lds_turn();
        for (int o = lane * 16; o < jb.hw * jb.cp; o += 1024) *(uint4 *)(q + o) = *(const uint4 *)(ldsrow + o);
    }
}

// channels whose codes exceed the LDS row and are not neighbours in memory either: 16 gathered values per lane
template <bool BF16>
__device__ __forceinline__ void quantize_channel_gather(const WeightJob &jb, int oc, uint32_t *flag, bool first_wave)
{
    const int lane = threadIdx.x & 63;
    const int64_t n_row = (int64_t)jb.c * jb.hw, base = (int64_t)oc * n_row;
    uint32_t m = 0;
    for (int64_t k = lane; k < n_row; k += 64) {
        const uint32_t a = abs_bits(load_elem<BF16>(jb.x, base + k));
        m = m > a ? m : a;
    }
    float scale;
    bool bad;
    const float inv = scale_from_bits(wave_max_u32(m), nullptr, &scale, &bad);
    if (lane == 0) {
        if (bad || first_wave) publish_shared(scale, bad, jb.scale + oc, flag);
        else jb.scale[oc] = scale;
    }
    const int cpu = jb.cp >> 4;
    const int64_t units = (int64_t)jb.hw * cpu;
    for (int64_t u = lane; u < units; u += 64) {
        const int pix = (int)(u / cpu), c0 = (int)(u - (int64_t)pix * cpu) << 4;
        uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if (c0 + e < jb.c) w[e >> 2] |= quant1(load_elem<BF16>(jb.x, base + (int64_t)(c0 + e) * jb.hw + pix), inv) << ((e & 3) * 8);
        *(uint4 *)(jb.q + ((int64_t)oc * units + u) * 16) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// lds_row: bytes of LDS per wave
__global__ __launch_bounds__(256) void quantize_weights_pc_kernel(const WeightBatch b, uint32_t *__restrict__ flag, int lds_row)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t rows[];
    const int j = find_job(b, (int)blockIdx.x);
    const WeightJob &jb = b.job[j];
    const int wave = threadIdx.x >> 6;
    const int oc = ((int)blockIdx.x - jb.first_block) * 4 + wave;
    if (oc >= jb.o) return;
    const bool first_wave = blockIdx.x == 0 && wave == 0;          // leaves the flag word initialised
    uint8_t *mine = rows + wave * lds_row;
    const int64_t n_row = (int64_t)jb.c * jb.hw;
    if (n_row == 0) {
        if ((threadIdx.x & 63) == 0) publish_shared(1.0f, false, jb.scale + oc, flag);
        return;
    }
    const bool bf = jb.bf16 != 0;
    const int epu = bf ? 8 : 4;
    const bool whole = n_row % epu == 0 && n_row < (1 << 24);      // rows of whole 16-byte units, 16-byte aligned
    if (whole && jb.hw == 1) {
        if (bf) {
            if (n_row <= 3 * 64 * 8) quantize_channel<true, 8, 3>(jb, oc, mine, flag, first_wave);
            else quantize_channel<true, 8, 12>(jb, oc, mine, flag, first_wave);
        } else {
            if (n_row <= 3 * 64 * 4) quantize_channel<false, 4, 3>(jb, oc, mine, flag, first_wave);
            else quantize_channel<false, 4, 12>(jb, oc, mine, flag, first_wave);
        }
    } else if ((int64_t)jb.hw * jb.cp <= lds_row) {
        if (whole) {
            if (bf) quantize_channel<true, 8, 6>(jb, oc, mine, flag, first_wave);
            else quantize_channel<false, 4, 10>(jb, oc, mine, flag, first_wave);
        } else {
            if (bf) quantize_channel<true, 1, 12>(jb, oc, mine, flag, first_wave);
            else quantize_channel<false, 1, 12>(jb, oc, mine, flag, first_wave);
        }
    } else {
        if (bf) quantize_channel_gather<true>(jb, oc, flag, first_wave);
        else quantize_channel_gather<false>(jb, oc, flag, first_wave);
    }
}

hipError_t launch_quantize_weights_pc(const WeightBatch &b, int total_blocks, uint32_t *flag, hipStream_t st)
{
    // LDS for the tensors that need it (the largest row of codes among those that fit), none for plain matrices
    int lds_row = 0;
    for (int i = 0; i < b.n; ++i) {
        const WeightJob &jb = b.job[i];
        const int64_t row = (int64_t)jb.hw * jb.cp;
        if ((jb.hw > 1 || jb.c % (jb.bf16 ? 8 : 4) != 0) && row <= kPcRowLds && row > lds_row) lds_row = (int)row;
    }
    return launch_k(EGERIA_KERNEL_QUANTIZE, quantize_weights_pc_kernel, dim3((unsigned)total_blocks), dim3(256),
                    (size_t)4 * lds_row, st, b, flag, lds_row);
}

hipError_t launch_quantize_weights(const WeightBatch &b, int total_blocks, bool one_launch, uint32_t *partials,
                                   uint32_t *flag, hipStream_t st, const InputMaxJob *extra, const InputQuantJob *xq)
{
    InputMaxJob ex{};
    InputQuantJob qj{};
    if (extra) ex = *extra;
    if (extra && xq && !one_launch) qj = *xq;               // the codes need the maxima of an earlier launch
    const int others = (total_blocks + 7) / 8 * 8;          // id of the first workgroup that is not the table's
    const dim3 first((unsigned)(ex.nblk ? others + ex.nblk : total_blocks)), second((unsigned)(qj.nblk ? others + qj.nblk : total_blocks)), block(256);
    if (one_launch)
        return launch_k(EGERIA_KERNEL_QUANTIZE, quantize_weights_kernel<0>, first, block, 0, st, b, partials, flag,
                        total_blocks, ex, InputQuantJob{});
    hipError_t e = launch_k(EGERIA_KERNEL_ABSMAX, quantize_weights_kernel<1>, first, block, 0, st, b, partials, flag,
                            total_blocks, ex, InputQuantJob{});
    if (e != hipSuccess) return e;
    return launch_k(EGERIA_KERNEL_QUANTIZE, quantize_weights_kernel<2>, second, block, 0, st, b, partials, flag,
                    total_blocks, InputMaxJob{}, qj);
}

// ---- fused GELU + quantise (gelu.hpp) ----------------------------------------------------
// The GELU output of a Transformer layer's first feed-forward GEMM is consumed
// only by the next quantiser, and its codes must equal those of the fp64
// evaluation rounded to fp32.  GELU is evaluated in fp32 first (cubic pieces from a
// table); a lane falls back to the fp64 form only when the error bound of that
// evaluation leaves two candidate codes (a few elements per 100 000).
__global__ __launch_bounds__(256) void gelu_absmax_exact_kernel(const float *__restrict__ v, int64_t n,
                                                                const uint32_t *__restrict__ vmax,
                                                                uint32_t *__restrict__ exact_absmax)
{
    if (__uint_as_float(reduce_ways(vmax)) >= kGeluShortcutMin) return;   // the shortcut applies: nothing to do
    uint32_t m = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t a = abs_bits(gelu_exact(v[i]));
        m = m > a ? m : a;
    }
    __shared__ uint32_t sm4[4];
    block_atomic_max(m, exact_absmax, sm4);
}

hipError_t launch_gelu_absmax_exact(const float *v, int64_t n, const uint32_t *vmax, uint32_t *exact_absmax,
                                    hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 1023) / 1024;
    if (blocks > 1024) blocks = 1024;
    return launch_k(EGERIA_KERNEL_NONE, gelu_absmax_exact_kernel, dim3((unsigned)blocks), dim3(256), 0, st, v, n, vmax,
                    exact_absmax);
}

__global__ __launch_bounds__(256) void quantize_gelu_rows_kernel(
    const float *__restrict__ v, int64_t rows, int64_t cols, int64_t ldq, const uint32_t *__restrict__ vmax,
    const uint32_t *__restrict__ exact_absmax, int8_t *__restrict__ q, float *__restrict__ scale_out,
    uint32_t *__restrict__ flag, int64_t per)
{
    const float4 entry = kGeluTable[threadIdx.x];
    // absolute maximum of gelu(v): gelu is increasing for v >= 0 and bounded by 0.17 for v < 0
    const float vm = __uint_as_float(reduce_ways(vmax));
    const bool bad = !(vm <= 3.402823466e+38f);
    const float exact = __uint_as_float(reduce_ways(exact_absmax));
    float scale;
    const float inv = gelu_code_scale(vm >= kGeluShortcutMin ? gelu_exact(vm) : exact, bad, &scale);
    if (blockIdx.x == 0 && threadIdx.x == 0) publish(scale, bad, scale_out, nullptr, flag);
    __shared__ float4 tab[256];                    // the table, once per workgroup (256 threads)
    tab[threadIdx.x] = scale_gelu_entry(entry, inv);
    __syncthreads();
    const float room = 0.5f - kGeluErrAbs * inv;
    const int64_t upr = ldq >> 4;
    const int64_t beg = xcd_piece(blockIdx.x, gridDim.x) * per;
    const int64_t units = beg + per < rows * upr ? beg + per : rows * upr;
    const bool narrow = rows * upr < (1LL << 32);
    const bool vec_ok = (cols & 3) == 0;
    // a thread's units are `stride` apart: row and unit within the row advance by stride / upr and stride % upr
    // (one division at the start instead of one per unit)
    const int64_t stride = 256;
    const int64_t first = beg + threadIdx.x;
    const int64_t step_rows = div_u(stride, upr, narrow), step_units = stride - step_rows * upr;
    auto run = [&](auto big_c) {
        constexpr bool BIG = decltype(big_c)::value;
        int64_t row = div_u(first, upr, narrow), cu = first - row * upr;
        for (int64_t u = first; u < units; u += stride) {
            const int64_t c0 = cu << 4;
            const int64_t base = row * cols + c0;
            uint32_t w[4] = {0, 0, 0, 0};
            uint32_t redo = 0;                         // elements that need the fp64 form
            if (vec_ok && c0 + 16 <= cols) {
                const float4 *p = (const float4 *)(v + base);
                float4 x[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) x[j] = p[j];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    bool u0, u1, u2, u3;
                    w[j] = pack_bytes(quant_gelu_fast<BIG>(x[j].x, inv, room, tab, &u0), quant_gelu_fast<BIG>(x[j].y, inv, room, tab, &u1),
                                      quant_gelu_fast<BIG>(x[j].z, inv, room, tab, &u2), quant_gelu_fast<BIG>(x[j].w, inv, room, tab, &u3));
                    redo |= ((u0 ? 1u : 0u) | (u1 ? 2u : 0u) | (u2 ? 4u : 0u) | (u3 ? 8u : 0u)) << (4 * j);
                }
            } else {
                redo = 0xffffu;                        // ragged tail of a row: every element through the loop below
            }
            // one copy of the fp64 code, rolled: the values are re-read (they are in cache)
#pragma unroll 1
            while (redo) {
                const int e = __ffs((int)redo) - 1;
                redo &= redo - 1;
                if (c0 + e >= cols) continue;
                const uint32_t code = settle_gelu(v[base + e], inv);
                const uint32_t sh = (e & 3) * 8, keep = ~(0xffu << sh);
                if ((e >> 2) == 0) w[0] = (w[0] & keep) | (code << sh);
                if ((e >> 2) == 1) w[1] = (w[1] & keep) | (code << sh);
                if ((e >> 2) == 2) w[2] = (w[2] & keep) | (code << sh);
                if ((e >> 2) == 3) w[3] = (w[3] & keep) | (code << sh);
            }
            *(uint4 *)(q + row * ldq + c0) = make_uint4(w[0], w[1], w[2], w[3]);
            row += step_rows;
            cu += step_units;
            if (cu >= upr) { cu -= upr; ++row; }
        }
    };
    // values of kGeluTop and more (where gelu(v) rounds to v and the table ends) only if the tensor's maximum says so
    if (vm >= kGeluTop || bad) run(std::true_type{}); else run(std::false_type{});
}

hipError_t launch_quantize_gelu_rows(const float *v, int64_t rows, int64_t cols, int64_t ldq,
                                     const uint32_t *vmax, const uint32_t *exact_absmax, int8_t *q,
                                     float *scale_out, uint32_t *flag, hipStream_t st)
{
    // (the table costs a workgroup a round trip: two units per thread rather than one where there are many; 16384 x 3072
    // with one 67 us, with two 53)
    const UnitShare sh = share_units(rows * (ldq / 16), 8192);
    return launch_k(EGERIA_KERNEL_QUANTIZE, quantize_gelu_rows_kernel, dim3(sh.blocks), dim3(256), 0, st, v,
                    rows, cols, ldq, vmax, exact_absmax, q, scale_out, flag, sh.per);
}

__global__ __launch_bounds__(256) void gelu_exact_kernel(const float *v, int64_t n, float *y)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        y[i] = gelu_exact(v[i]);
}

hipError_t launch_gelu_exact(const float *v, int64_t n, float *y, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    return launch_k(EGERIA_KERNEL_NONE, gelu_exact_kernel, dim3((unsigned)blocks), dim3(256), 0, st, v, n, y);
}

// The float16 operand of the second feed-forward layer from the first one's fp32 output: float16(fp32(gelu(v))), gelu
// in its fp64 evaluation, as launch_gelu_exact followed by the cast gives it, in one pass and without the fp32
// tensor in between.  Rounding is monotone, so when both ends of the interval that the table's error bound leaves round
// to the same float16 that is the result; the others (about one in 200 for pre-activations of unit size: the
// absolute part of the bound covers many float16 steps near zero) take the fp64 form.  A NaN is looked up as -8,
// where the interval straddles zero, so it takes the fp64 form too.  What bounds it is the table walk and the fp64 forms;
// 4096 x 3072: 19.4 us, against 39.8 (fp64 erf for every value) + 26.5 (cast) before.
__global__ __launch_bounds__(256) void gelu_f16_rows_kernel(const float *__restrict__ v, int64_t rows, int64_t cols, int64_t ldh,
                                                            uint16_t *__restrict__ out, int64_t per)
{
    __shared__ float4 tab[256];
    tab[threadIdx.x] = kGeluTable[threadIdx.x];
    __syncthreads();
    const int64_t upr = ldh >> 3, beg = xcd_piece(blockIdx.x, gridDim.x) * per;
    const int64_t end = beg + per < rows * upr ? beg + per : rows * upr;
    const bool narrow = rows * upr < (1LL << 32);
    for (int64_t u = beg + threadIdx.x; u < end; u += 256) {
        const int64_t row = div_u(u, upr, narrow), c0 = (u - row * upr) * 8, base = row * cols + c0;
        float x[8];
        if ((cols & 3) == 0) {                             // (rows start on 16 bytes, units hold 4 or 8 values)
            const float4 a = *(const float4 *)(v + base), b = *(const float4 *)(v + (c0 + 4 < cols ? base + 4 : base));
            x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
            x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = v[c0 + e < cols ? base + e : base];
        }
        uint32_t w[4] = {0, 0, 0, 0}, redo = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float g = gelu_table<true>(x[e], 1.0f, tab);
            const float err = fmaf(kGeluErrRel + 3.0e-7f, fabsf(g), kGeluErrAbs * 1.001f);
            const uint32_t lo = __builtin_bit_cast(uint16_t, (_Float16)(g - err)), hi = __builtin_bit_cast(uint16_t, (_Float16)(g + err));
            const bool in = c0 + e < cols;                 // pad columns: zero
            w[e >> 1] |= (in ? lo : 0u) << (16 * (e & 1));
            redo |= (in && lo != hi ? 1u : 0u) << e;
        }
        // one copy of the fp64 code, rolled: the values are re-read (they are in cache)
#pragma unroll 1
        while (redo) {
            const int e = __ffs((int)redo) - 1;
            redo &= redo - 1;
            const uint32_t h = __builtin_bit_cast(uint16_t, (_Float16)gelu_exact(v[base + e]));
            const uint32_t sh = 16 * (e & 1), keep = ~(0xffffu << sh);
            if ((e >> 1) == 0) w[0] = (w[0] & keep) | (h << sh);
            if ((e >> 1) == 1) w[1] = (w[1] & keep) | (h << sh);
            if ((e >> 1) == 2) w[2] = (w[2] & keep) | (h << sh);
            if ((e >> 1) == 3) w[3] = (w[3] & keep) | (h << sh);
        }
        *(uint4 *)(out + row * ldh + c0) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

hipError_t launch_gelu_f16_rows(const float *v, int64_t rows, int64_t cols, int64_t ldh, void *out, hipStream_t st)
{
    if (rows * (ldh >> 3) <= 0) return hipSuccess;
    const UnitShare sh = share_units(rows * (ldh >> 3), 8192);
    return launch_k(EGERIA_KERNEL_QUANTIZE, gelu_f16_rows_kernel, dim3(sh.blocks), dim3(256), 0, st, v, rows, cols, ldh,
                    (uint16_t *)out, sh.per);
}

// ---- dequantise ------------------------------------------------------------------------
__global__ __launch_bounds__(256) void dequantize_kernel(const int8_t *__restrict__ q,
                                                         const float *__restrict__ scale, int64_t n,
                                                         float *__restrict__ x)
{
    const float s = *scale;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        x[i] = (float)q[i] * s;
}

hipError_t launch_dequantize(const int8_t *q, const float *scale, int64_t n, float *x, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    return launch_k(EGERIA_KERNEL_NONE, dequantize_kernel, dim3((unsigned)blocks), dim3(256), 0, st, q, scale, n, x);
}

}  // namespace egeria
