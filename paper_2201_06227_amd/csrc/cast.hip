// Reference model at float16 / float32 precision (Section 6.4 of the paper,
// Table 2): operands in the layout the GEMM consumes.  A tensor [n, c, hw]
// (channel-major: a mini-batch of images, a convolution kernel, or with hw = 1
// the rows of a matrix) becomes [n, hw, cpe] of the reference precision, the
// channels rounded to nearest even and padded with zeros to cpe (a whole
// number of 16-byte units).  One thread makes one 16-byte unit; lanes run along
// the pixels of an image (coalesced reads of each channel plane) or, for
// matrices, along the units of a row.
#include "common.hpp"

namespace egeria {

namespace {

// a 16-byte unit of the reference precision from its 8 (float16) or 4 (float32) values, round to nearest even
template <int ET>
__device__ __forceinline__ uint4 pack_unit(const float *v)
{
    union {
        _Float16 h[8];
        float f[4];
        uint4 q;
    } pk;
#pragma unroll
    for (int e = 0; e < (ET == 1 ? 8 : 4); ++e) {
        if constexpr (ET == 1) pk.h[e] = (_Float16)v[e];
        else pk.f[e] = v[e];
    }
    return pk.q;
}

// Three forms; HBM-bound, what counts is that a thread's loads are wide and all in flight together:
//   kRows    fp32 rows of whole 16-byte units (4096 x 768 to float16: 8.9 us with a load per value, 5.6 now);
//   kPlanes  fp32 planes of whole 16-byte units: a thread makes the units of four neighbouring pixels;
//   kAny     everything else, a load per value.
enum CastForm { kAny = 0, kRows = 1, kPlanes = 2 };

template <bool SRC_BF16, int ET, int FORM>
__global__ __launch_bounds__(256) void cast_chlast_kernel(const void *__restrict__ x, int64_t n, int64_t c,
                                                          int64_t hw, int64_t cpe, uint8_t *__restrict__ out,
                                                          float *__restrict__ one, int64_t share)
{
    constexpr int EPU = ET == 1 ? 8 : 4;                  // elements per 16-byte unit
    if (one && blockIdx.x == 0 && threadIdx.x == 0) *one = 1.0f;
    const int64_t upr = cpe / EPU;                        // units per pixel
    const int64_t beg = xcd_piece(blockIdx.x, gridDim.x) * share;
    const int64_t per = hw == 1 ? upr : (FORM == kPlanes ? hw >> 2 : hw);
    const int64_t total = n * upr * (hw == 1 ? 1 : per);
    const int64_t end = beg + share < total ? beg + share : total;
    const __amdgpu_buffer_rsrc_t rows_out = __builtin_amdgcn_make_buffer_rsrc(out + beg * 16, 0, 0x7fffffff, kBufferWord);   // kRows: unit u is the u-th of the output
    const bool narrow = total < (1LL << 32);
    for (int64_t u = beg + threadIdx.x; u < end; u += 256) {
        const int64_t rest = narrow ? (int64_t)((uint32_t)u / (uint32_t)per) : u / per, at = u - rest * per;
        int64_t img = rest, unit = at, p = 0;
        if (hw != 1) {
            img = narrow ? (int64_t)((uint32_t)rest / (uint32_t)upr) : rest / upr;
            unit = rest - img * upr;
            p = FORM == kPlanes ? at * 4 : at;
        }
        const int64_t ch0 = unit * EPU;
        uint4 *dst = (uint4 *)(out + ((img * hw + p) * cpe + ch0) * (ET == 1 ? 2 : 4));
        if constexpr (FORM == kPlanes) {
            const float *src = (const float *)x + (img * c + ch0) * hw + p;
            float4 v[EPU];
#pragma unroll
            for (int e = 0; e < EPU; ++e) v[e] = *(const float4 *)(src + (ch0 + e < c ? e * hw : 0));
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float f[EPU];
#pragma unroll
                for (int e = 0; e < EPU; ++e) f[e] = ch0 + e < c ? (k == 0 ? v[e].x : k == 1 ? v[e].y : k == 2 ? v[e].z : v[e].w) : 0.0f;
                dst[k * upr] = pack_unit<ET>(f);
            }
        } else if constexpr (FORM == kRows) {
            const float4 *src = (const float4 *)((const float *)x + img * c);
            float f[EPU];
            float4 v[EPU / 4];
#pragma unroll
            for (int j = 0; j < EPU / 4; ++j) v[j] = src[ch0 + 4 * j < c ? (ch0 >> 2) + j : 0];
#pragma unroll
            for (int j = 0; j < EPU / 4; ++j) {
                const bool in = ch0 + 4 * j < c;
                f[4 * j] = in ? v[j].x : 0.0f;
                f[4 * j + 1] = in ? v[j].y : 0.0f;
                f[4 * j + 2] = in ? v[j].z : 0.0f;
                f[4 * j + 3] = in ? v[j].w : 0.0f;
            }
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, pack_unit<ET>(f)), rows_out, (int)(u - beg) * 16, 0, kThrough);
        } else {
            float f[EPU];
#pragma unroll
            for (int e = 0; e < EPU; ++e) {                // (unconditional loads, the surplus discarded)
                const int64_t ch = ch0 + e, i = (img * c + (ch < c ? ch : c - 1)) * hw + p;
                f[e] = SRC_BF16 ? bf16_to_f32(((const uint16_t *)x)[i]) : ((const float *)x)[i];
            }
#pragma unroll
            for (int e = 0; e < EPU; ++e)
                if (ch0 + e >= c) f[e] = 0.0f;
            *dst = pack_unit<ET>(f);
        }
    }
}

}  // namespace

hipError_t launch_cast_chlast(const void *x, egeria_dtype dt, int64_t n, int64_t c, int64_t hw, int64_t cpe, int et,
                              void *out, float *one, hipStream_t st)
{
    // whole 16-byte units of fp32 take the wide forms; bf16, odd rows and planes, and other addresses the general one
    const bool wide = dt != EGERIA_BF16 && ((uintptr_t)x & 15) == 0;
    const int form = wide && hw == 1 && (c & 3) == 0 ? kRows : (wide && hw > 1 && (hw & 3) == 0 ? kPlanes : kAny);
    const int64_t total = n * hw * (cpe / (et == 1 ? 8 : 4)) / (form == kPlanes ? 4 : 1);
    const UnitShare sh = share_units(total);               // (one workgroup at least: the 1.0f is still written)
    const dim3 grid(sh.blocks), block(256);
    auto go = [&](auto kernel) { return launch_k(EGERIA_KERNEL_QUANTIZE, kernel, grid, block, 0, st, x, n, c, hw, cpe, (uint8_t *)out, one, sh.per); };
    if (dt == EGERIA_BF16) return et == 1 ? go(cast_chlast_kernel<true, 1, kAny>) : go(cast_chlast_kernel<true, 2, kAny>);
    if (form == kRows) return et == 1 ? go(cast_chlast_kernel<false, 1, kRows>) : go(cast_chlast_kernel<false, 2, kRows>);
    if (form == kPlanes) return et == 1 ? go(cast_chlast_kernel<false, 1, kPlanes>) : go(cast_chlast_kernel<false, 2, kPlanes>);
    return et == 1 ? go(cast_chlast_kernel<false, 1, kAny>) : go(cast_chlast_kernel<false, 2, kAny>);
}

}  // namespace egeria
