// Floating-point glue of a Transformer encoder layer of the reference model:
// under dynamic quantisation (Section 5 of the paper) only the linear layers
// are int8; self-attention and layer norm read and write fp32 tensors.
#include "common.hpp"
#include <type_traits>

namespace egeria {

// ---- y = LN(x + res): one wave per row, evaluated in fp64 and rounded once ----------------
// (its output feeds a quantiser; see the note on the attention kernel)
__global__ __launch_bounds__(256) void layernorm_kernel(const float *__restrict__ x,
                                                        const float *__restrict__ res, int64_t rows,
                                                        int H, const float *__restrict__ gamma,
                                                        const float *__restrict__ beta, double eps,
                                                        float *__restrict__ y,
                                                        uint32_t *__restrict__ absmax_out, uint16_t *__restrict__ y_half)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t row = (int64_t)xcd_piece(blockIdx.x, gridDim.x) * 4 + wave;
    uint32_t amax = 0;
    if (row < rows) {
        const float *xr = x + row * H;
        const float *rr = res ? res + row * H : nullptr;
        double s = 0.0;
        for (int h = lane; h < H; h += 64) s += (double)xr[h] + (rr ? (double)rr[h] : 0.0);
        const double mean = wave_sum(s) / (double)H;
        double q = 0.0;
        for (int h = lane; h < H; h += 64) {
            const double v = ((double)xr[h] + (rr ? (double)rr[h] : 0.0)) - mean;
            q += v * v;
        }
        const double var = wave_sum(q) / (double)H;
        const double rstd = 1.0 / sqrt(var + eps);
        for (int h = lane; h < H; h += 64) {
            const double v = (double)xr[h] + (rr ? (double)rr[h] : 0.0);
            const double gm = gamma ? (double)gamma[h] : 1.0, bt = beta ? (double)beta[h] : 0.0;
            const float o = (float)((v - mean) * rstd * gm + bt);
            y[row * H + h] = o;
            if (y_half) y_half[row * H + h] = __builtin_bit_cast(uint16_t, (_Float16)o);
            const uint32_t ab = abs_bits(o);
            amax = amax > ab ? amax : ab;
        }
    }
    if (absmax_out) {
        __shared__ uint32_t sm4[4];
        block_atomic_max(amax, absmax_out, sm4);
    }
}

// Same, for rows of at most 256*NV floats with H a multiple of 4: the row is
// read once with 16-byte loads and stays in registers (as the exact fp64 sums
// x + res) for the three passes.
template <int NV>
__global__ __launch_bounds__(256) void layernorm_vec_kernel(const float *__restrict__ x,
                                                            const float *__restrict__ res, int64_t rows,
                                                            int H, const float *__restrict__ gamma,
                                                            const float *__restrict__ beta, double eps,
                                                            float *__restrict__ y,
                                                            uint32_t *__restrict__ absmax_out,
                                                            uint16_t *__restrict__ y_half)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row = (int64_t)xcd_piece(blockIdx.x, gridDim.x) * 4 + wave;
    const int nv = H >> 2;
    uint32_t amax = 0;
    if (row < rows) {
        // Every load of the row goes out before the first wait: unconditional, with the index clamped
        // and the value replaced afterwards (a load under a per-lane condition is awaited on its own,
        // and a row would cost a dozen memory round trips instead of one).  Absent operands read x.
        const float4 *xr = reinterpret_cast<const float4 *>(x + row * H);
        const float4 *rr = reinterpret_cast<const float4 *>((res ? res : x) + row * H);
        const float4 *gr = reinterpret_cast<const float4 *>(gamma ? gamma : x + row * H);
        const float4 *br = reinterpret_cast<const float4 *>(beta ? beta : x + row * H);
        const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f), one4 = make_float4(1.f, 1.f, 1.f, 1.f);
        float4 xv[NV], rv[NV], gmv[NV], btv[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int c = lane + 64 * i, cc = c < nv ? c : nv - 1;
            xv[i] = xr[cc];
            rv[i] = rr[cc];
            gmv[i] = gr[cc];
            btv[i] = br[cc];
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const bool in = lane + 64 * i < nv;
            if (!in) xv[i] = zero4;
            if (!in || !res) rv[i] = zero4;
            if (!gamma) gmv[i] = one4;
            if (!beta) btv[i] = zero4;
        }
        float4 o[NV];
        ln_row_vec<NV>(xv, rv, gmv, btv, lane, nv, H, eps, o, amax);
        const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void *)(y + row * H), 0, H * 4, kBufferWord);   // (a unit beyond the row is dropped)
#pragma unroll
        for (int i = 0; i < NV; ++i)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, o[i]), ry, (lane + 64 * i) * 16, 0, kThrough);
        if (y_half) {
            const __amdgpu_buffer_rsrc_t rh = __builtin_amdgcn_make_buffer_rsrc((void *)(y_half + row * H), 0, H * 2, kBufferWord);
            typedef _Float16 v4h __attribute__((ext_vector_type(4)));
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const v4h half = {(_Float16)o[i].x, (_Float16)o[i].y, (_Float16)o[i].z, (_Float16)o[i].w};
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, half), rh, (lane + 64 * i) * 8, 0, kThrough);
            }
        }
    }
    if (absmax_out) {
        __shared__ uint32_t sm4[4];
        block_atomic_max(amax, absmax_out, sm4);
    }
}

static bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

hipError_t launch_layernorm(const float *x, const float *res, int64_t rows, int32_t H,
                            const float *gamma, const float *beta, float eps, float *y,
                            uint32_t *absmax_out, hipStream_t st, uint16_t *y_half)
{
    if (rows <= 0) return hipSuccess;
    const dim3 grid((unsigned)((rows + 3) / 4)), block(256);
    const bool vec = (H % 4) == 0 && H <= 1024 && aligned16(x) && aligned16(res) && aligned16(gamma) &&
                     aligned16(beta) && aligned16(y) && (reinterpret_cast<uintptr_t>(y_half) & 7u) == 0;
    if (vec && H <= 256)
        return launch_k(EGERIA_KERNEL_LAYERNORM, layernorm_vec_kernel<1>, grid, block, 0, st, x, res, rows, (int)H,
                        gamma, beta, (double)eps, y, absmax_out, y_half);
    if (vec && H <= 768)
        return launch_k(EGERIA_KERNEL_LAYERNORM, layernorm_vec_kernel<3>, grid, block, 0, st, x, res, rows, (int)H,
                        gamma, beta, (double)eps, y, absmax_out, y_half);
    if (vec)
        return launch_k(EGERIA_KERNEL_LAYERNORM, layernorm_vec_kernel<4>, grid, block, 0, st, x, res, rows, (int)H,
                        gamma, beta, (double)eps, y, absmax_out, y_half);
    return launch_k(EGERIA_KERNEL_LAYERNORM, layernorm_kernel, grid, block, 0, st, x, res, rows, (int)H, gamma, beta,
                    (double)eps, y, absmax_out, y_half);
}

// ---- multi-head self-attention -----------------------------------------------------------
// Evaluated in fp64 and rounded once to fp32, like the layer norm above: the
// context feeds a quantiser, where a last-bit difference can flip an int8 code
// and the flip is then amplified by every later layer.
//
// A workgroup owns one (batch, head) pair and 64 * QB queries, 16 * QB per wave (QB
// blocks of 16); key / value tiles of 32 rows pass through LDS as fp32 and are
// widened when read.  The products run on v_mfma_f64_16x16x4f64 in the
// transposed form
//     S^T = K Q^T  (keys x queries),      O^T = V^T P^T  (head dim x queries),
// so that a lane always owns one query column (lane = column + 16 * g, register
// r = row 4r + g): the soft-max statistics of a query are an in-lane reduction
// plus two exchanges across g, and the accumulator registers of S^T are,
// unchanged, the B operand of the second product.
typedef double v4d __attribute__((ext_vector_type(4)));
constexpr int kDh = 64;             // head dimension covered (smaller heads are zero padded)
constexpr int kKeyTile = 32;
constexpr int kKVPad = kDh + 4;

template <int QB>
__global__ __launch_bounds__(256) void attention_kernel(const float *__restrict__ qkv, int B, int S,
                                                        int Hd, int heads, int dh, double scale,
                                                        float *__restrict__ ctx,
                                                        uint32_t *__restrict__ absmax_out, uint16_t *__restrict__ ctx_half)
{
    __shared__ __attribute__((aligned(16))) float sKb[2][kKeyTile][kKVPad];   // two stages
    __shared__ __attribute__((aligned(16))) float sVb[2][kKeyTile][kKVPad];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, g = lane >> 4;
    constexpr int QT = 64 * QB;          // queries per workgroup
    const int qtiles = (S + QT - 1) / QT;
    // Each XCD is given a contiguous range of (batch, head, query tile), so that the query tiles of
    // one head, which re-read the same K and V, share an L2.
    const int vid = (int)xcd_piece(blockIdx.x, gridDim.x);
    const int bh = vid / qtiles, qt = vid % qtiles;
    const int bi = bh / heads, hd = bh % heads;
    const int64_t tok0 = (int64_t)bi * S;
    const int64_t ld = 3 * (int64_t)Hd;
    const float *qbase = qkv + hd * dh, *kbase = qbase + Hd, *vbase = qbase + 2 * Hd;

    // query rows as the B operand of S^T = K Q^T: d = 16u + 4g + e (u, e = 0..3).  The loads are
    // unconditional (row and column clamped to valid ones, the value discarded afterwards): loads
    // under a per-lane condition are awaited one by one, sixteen memory round trips before the
    // first key tile instead of one.
    const bool vec4 = (dh & 3) == 0 && (Hd & 3) == 0;
    double qr[QB][16];
    int qidx[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int q = qt * QT + wave * (16 * QB) + qb * 16 + c;
        qidx[qb] = q;
        const float *qrow = qbase + (tok0 + (q < S ? q : S - 1)) * ld;
        float qv[16];
        if (vec4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int d0 = 16 * u + 4 * g;
                const float4 v = *(const float4 *)(qrow + (d0 < dh ? d0 : 0));
                qv[4 * u] = v.x; qv[4 * u + 1] = v.y; qv[4 * u + 2] = v.z; qv[4 * u + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int d = 16 * u + 4 * g + e;
                    qv[4 * u + e] = qrow[d < dh ? d : 0];
                }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int d = 16 * u + 4 * g + e;
                qr[qb][4 * u + e] = (q < S && d < dh) ? (double)qv[4 * u + e] : 0.0;
            }
    }

    v4d o[QB][4];                       // O^T: [query block][16-row block of the head dim]
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r = 0; r < 4; ++r) o[qb][db][r] = 0.0;
    double mrun[QB], lrun[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) { mrun[qb] = -INFINITY; lrun[qb] = 0.0; }

    // Key / value tiles: thread t stages float4 slots t and t + 256 of the
    // 32 x 64 tile (row = slot / 16); the next tile's global loads are issued
    // before the current tile is contracted and land in the other LDS stage.
    float4 pk[2], pv[2];
    auto fetch = [&](int j0) {
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int sl = tid + it * 256, kr = sl >> 4, d = (sl & 15) * 4;
            const int64_t off = (tok0 + j0 + kr) * ld + d;
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b4 = a;
            if (j0 + kr < S) {
                if (vec4 && d + 4 <= dh) {
                    a = *(const float4 *)(kbase + off);
                    b4 = *(const float4 *)(vbase + off);
                } else {
                    float ea[4] = {0.f, 0.f, 0.f, 0.f}, eb[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (d + e < dh) { ea[e] = kbase[off + e]; eb[e] = vbase[off + e]; }
                    a = make_float4(ea[0], ea[1], ea[2], ea[3]);
                    b4 = make_float4(eb[0], eb[1], eb[2], eb[3]);
                }
            }
            pk[it] = a;
            pv[it] = b4;
        }
    };
    auto stash = [&](int stage) {
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int sl = tid + it * 256, kr = sl >> 4, d = (sl & 15) * 4;
            *(float4 *)&sKb[stage][kr][d] = pk[it];
            *(float4 *)&sVb[stage][kr][d] = pv[it];
        }
    };
    fetch(0);
    stash(0);
    __syncthreads();
    int stage = 0;
    for (int j0 = 0; j0 < S; j0 += kKeyTile, stage ^= 1) {
        const bool more = j0 + kKeyTile < S;
        if (more) fetch(j0 + kKeyTile);
        float (*sK)[kKVPad] = sKb[stage];
        float (*sV)[kKVPad] = sVb[stage];

        v4d st[2][QB];                  // [key block][query block]
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int r = 0; r < 4; ++r) st[kb][qb][r] = 0.0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                const float4 kv = *(const float4 *)&sK[kb * 16 + c][16 * u + 4 * g];
                const double k4[4] = {(double)kv.x, (double)kv.y, (double)kv.z, (double)kv.w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb)
                        st[kb][qb] = __builtin_amdgcn_mfma_f64_16x16x4f64(k4[e], qr[qb][4 * u + e], st[kb][qb], 0, 0, 0);
            }
        }
        // register r of st[kb][qb] is key j0 + 16*kb + 4*r + g for this lane's query
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            double mx = -INFINITY;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int key = j0 + kb * 16 + 4 * r + g;
                    st[kb][qb][r] = key >= S ? -INFINITY : st[kb][qb][r] * scale;   // q.k first, then 1/sqrt(dh)
                    mx = fmax(mx, st[kb][qb][r]);
                }
            mx = pair_op<16>(mx, [](double a, double b) { return fmax(a, b); });
            mx = pair_op<32>(mx, [](double a, double b) { return fmax(a, b); });
            const double mnew = fmax(mrun[qb], mx);      // finite: every tile holds at least one key
            const double corr = exp(mrun[qb] - mnew);
            double ps = 0.0;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    st[kb][qb][r] = exp(st[kb][qb][r] - mnew);
                    ps += st[kb][qb][r];
                }
            ps = pair_op<16>(ps, [](double a, double b) { return a + b; });
            ps = pair_op<32>(ps, [](double a, double b) { return a + b; });
            lrun[qb] = lrun[qb] * corr + ps;
            mrun[qb] = mnew;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int r = 0; r < 4; ++r) o[qb][db][r] *= corr;
        }
        // O^T += V^T P^T: step (kb, r) contracts keys 16*kb + 4*r + g, g = 0..3
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int kr = kb * 16 + 4 * r + g;
#pragma unroll
                for (int db = 0; db < 4; ++db) {
                    const double vv = (double)sV[kr][db * 16 + c];
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb)
                        o[qb][db] = __builtin_amdgcn_mfma_f64_16x16x4f64(vv, st[kb][qb][r], o[qb][db], 0, 0, 0);
                }
            }
        if (more) stash(stage ^ 1);
        __syncthreads();
    }

    uint32_t amax = 0;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int q = qidx[qb];
        if (q >= S) continue;
        const int64_t dst = (tok0 + q) * Hd + hd * dh;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int d = db * 16 + 4 * r + g;
                if (d < dh) {
                    const float v = (float)(o[qb][db][r] / lrun[qb]);
                    if (ctx_half) ctx_half[dst + d] = __builtin_bit_cast(uint16_t, (_Float16)v);
                    else ctx[dst + d] = v;
                    const uint32_t ab = abs_bits(v);
                    amax = amax > ab ? amax : ab;
                }
            }
    }
    if (absmax_out) {
        __shared__ uint32_t sm4[4];
        block_atomic_max(amax, absmax_out, sm4);
    }
}

// ---- the same attention in approximate arithmetic on the matrix cores, with certified int8 codes ----------
// Unobserved runs do not need the context as the fp64 evaluation gives it: all that leaves this stage
// is the int8 input of the next GEMM and its scale.  Three launches, for head dims in whole units of 8:
//   1. an approximate attention with fp32 sums: attention_split_kernel (further down: every fp32 product as three float16
//      partial products on the float16 matrix cores).  It stores an approximate context, an error bound E per query of a head
//      and what its workgroups know of the largest value.
//   2. attention_settle_kernel: the tensor's absolute maximum as the fp64 evaluation gives it, from the values that can be it
//      (as a rule one).
//   3. quantize_attention_certify_kernel: the streaming map to codes.  code(x) = clamp(rne(x * inv)) is
//      monotone in x, so an approximate value whose interval [x - E, x + E] maps to one code has that
//      code; the others (a few in ten thousand) are re-evaluated in fp64, a wave per value, by the
//      workgroup that met them.
// Other head sizes take the fp64 kernel at every size.  An approximate kernel in fp32 (here: the structure of the kernel above
// on v_mfma_f32_16x16x4f32, hardware exp2; any head size) gains nothing on them: with the bound that holds for it (below) one
// layer of 64 x 256 tokens x 12 heads of 55 took 1446 us, in fp64 498; with half the bound's lists 572 and 510.  It is left for
// measurement.
// The fp32 kernel's bound of a value x (the split kernel forms its own, per query and tighter, and says what the parts stand
// for): E = 2^-24 * (max|v| of the head * (kErrBase + kErrPerTile * tiles of 32 keys + kErrPerScore * max|score| of the workgroup +
// kErrPerNorm * max|q| of the workgroup * largest norm of a key / sqrt(dh)) + kErrRel |x|).  It is an empirical bound with margin,
// not a proof: bench.py --attention-error measures both kernels against the fp64 kernel on the twelve layers of the
// BERT-base-shaped stack (12.6 M values each) and on inputs whose rounding errors add up.  (With 2 + max|score| / 2 alone the
// error was up to 35 times the bound for tokens that repeat, 2 times for uniform values with scores of 17.)
typedef float v4f __attribute__((ext_vector_type(4)));
constexpr float kErrBase = 3.0f, kErrPerTile = 0.25f, kErrPerScore = 4.0f, kErrPerNorm = 2.5f;
// ... plus a part that grows with the value itself (the drift of the matrix cores' accumulation is
// proportional to the sums it carries): kErrRel * 2^-24 * |x|
constexpr float kErrRel = 12.0f * 5.9604645e-8f;
// error bound of one approximate context value x whose query's bound is err
__device__ __forceinline__ float value_err(float err, float x) { return fmaf(kErrRel, fabsf(x), err); }
struct AttnRecord {
    uint32_t amax_bits;     // largest |approximate context| of the workgroup's 64 queries x head dims
    float err;              // E for those values
};

__global__ __launch_bounds__(256) void attention_fast_kernel(const float *__restrict__ qkv, int B, int S, int Hd,
                                                             int heads, int dh, float scale, float *__restrict__ ctx,
                                                             AttnRecord *__restrict__ rec)
{
    __shared__ __attribute__((aligned(16))) float sKb[2][kKeyTile][kKVPad];
    __shared__ __attribute__((aligned(16))) float sVb[2][kKeyTile][kKVPad];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, g = lane >> 4;
    constexpr int QT = 64;
    const int qtiles = (S + QT - 1) / QT;
    const int vid = (int)xcd_piece(blockIdx.x, gridDim.x);
    const int bh = vid / qtiles, qt = vid % qtiles;
    const int bi = bh / heads, hd = bh % heads;
    const int64_t tok0 = (int64_t)bi * S;
    const int64_t ld = 3 * (int64_t)Hd;
    const float *qbase = qkv + hd * dh, *kbase = qbase + Hd, *vbase = qbase + 2 * Hd;
    const bool vec4 = (dh & 3) == 0 && (Hd & 3) == 0;
    // query rows as the B operand of S^T = K Q^T: lane (c, g) holds dims 16u + 4g + e of query c
    float qr[16];
    const int q = qt * QT + wave * 16 + c;
    {
        const float *qrow = qbase + (tok0 + (q < S ? q : S - 1)) * ld;
        float qv[16];
        if (vec4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int d0 = 16 * u + 4 * g;
                const float4 v = *(const float4 *)(qrow + (d0 < dh ? d0 : 0));
                qv[4 * u] = v.x; qv[4 * u + 1] = v.y; qv[4 * u + 2] = v.z; qv[4 * u + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int d = 16 * u + 4 * g + e;
                    qv[4 * u + e] = qrow[d < dh ? d : 0];
                }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int d = 16 * u + 4 * g + e;
                qr[4 * u + e] = (q < S && d < dh) ? qv[4 * u + e] : 0.0f;
            }
    }
    v4f o[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[db][r] = 0.0f;
    float mrun = -INFINITY, lrun = 0.0f;
    float smax = 0.0f;                  // largest |score| met by this lane
    uint32_t vmax = 0;                  // largest |v| staged by this thread (bit pattern)
    float knorm2 = 0.0f;                // largest squared norm of the keys it staged a part of
    float4 pk[2], pv[2];
    auto fetch = [&](int j0) {
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int sl = tid + it * 256, kr = sl >> 4, d = (sl & 15) * 4;
            const int64_t off = (tok0 + j0 + kr) * ld + d;
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b4 = a;
            if (j0 + kr < S) {
                if (vec4 && d + 4 <= dh) {
                    a = *(const float4 *)(kbase + off);
                    b4 = *(const float4 *)(vbase + off);
                } else {
                    float ea[4] = {0.f, 0.f, 0.f, 0.f}, eb[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (d + e < dh) { ea[e] = kbase[off + e]; eb[e] = vbase[off + e]; }
                    a = make_float4(ea[0], ea[1], ea[2], ea[3]);
                    b4 = make_float4(eb[0], eb[1], eb[2], eb[3]);
                }
            }
            pk[it] = a;
            pv[it] = b4;
        }
    };
    auto stash = [&](int stage) {
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int sl = tid + it * 256, kr = sl >> 4, d = (sl & 15) * 4;
            *(float4 *)&sKb[stage][kr][d] = pk[it];
            *(float4 *)&sVb[stage][kr][d] = pv[it];
            const float n2 = fmaf(pk[it].x, pk[it].x, fmaf(pk[it].y, pk[it].y, fmaf(pk[it].z, pk[it].z, pk[it].w * pk[it].w)));
            knorm2 = fmaxf(knorm2, wave_reduce<8>(n2, [](float a, float b) { return a + b; }));   // the sixteen lanes of a key
            uint32_t a0 = abs_bits(pv[it].x), a1 = abs_bits(pv[it].y), a2 = abs_bits(pv[it].z), a3 = abs_bits(pv[it].w);
            a0 = a0 > a1 ? a0 : a1;
            a2 = a2 > a3 ? a2 : a3;
            a0 = a0 > a2 ? a0 : a2;
            vmax = vmax > a0 ? vmax : a0;
        }
    };
    fetch(0);
    stash(0);
    __syncthreads();
    int stage = 0;
    constexpr float kLog2e = 1.44269504088896340736f;
    for (int j0 = 0; j0 < S; j0 += kKeyTile, stage ^= 1) {
        const bool more = j0 + kKeyTile < S;
        if (more) fetch(j0 + kKeyTile);
        float (*sK)[kKVPad] = sKb[stage];
        float (*sV)[kKVPad] = sVb[stage];
        v4f st[2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r) st[kb][r] = 0.0f;
        // The matrix cores' accumulation is not round-to-nearest over a chain of instructions: measured against
        // fp64, a sum carried through n dependent MFMAs drifts by about n/4 ulp of its size, always towards
        // zero.  Chains are therefore kept short (four instructions from a zero accumulator) and their
        // results are added on the vector ALU, which rounds to nearest: the error of the context dropped
        // from 14 to 4 ulp of the tensor's maximum for 4 % more time.
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                const float4 kv = *(const float4 *)&sK[kb * 16 + c][16 * u + 4 * g];
                const float k4[4] = {kv.x, kv.y, kv.z, kv.w};
                v4f part = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    part = __builtin_amdgcn_mfma_f32_16x16x4f32(k4[e], qr[4 * u + e], part, 0, 0, 0);
#pragma unroll
                for (int r = 0; r < 4; ++r) st[kb][r] += part[r];
            }
        }
        // register r of st[kb] is key j0 + 16 kb + 4 g + r for this lane's query
        float mx = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int key = j0 + kb * 16 + 4 * g + r;
                const float sc = st[kb][r] * scale;
                smax = key < S ? fmaxf(smax, fabsf(sc)) : smax;
                st[kb][r] = key < S ? sc : -INFINITY;
                mx = fmaxf(mx, st[kb][r]);
            }
        mx = pair_op<16>(mx, [](float a, float b) { return fmaxf(a, b); });
        mx = pair_op<32>(mx, [](float a, float b) { return fmaxf(a, b); });
        const float mnew = fmaxf(mrun, mx);
        const float corr = __builtin_amdgcn_exp2f((mrun - mnew) * kLog2e);
        float ps = 0.0f;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                st[kb][r] = __builtin_amdgcn_exp2f((st[kb][r] - mnew) * kLog2e);
                ps += st[kb][r];
            }
        ps = pair_op<16>(ps, [](float a, float b) { return a + b; });
        ps = pair_op<32>(ps, [](float a, float b) { return a + b; });
        lrun = lrun * corr + ps;
        mrun = mnew;
        // this tile's V^T P^T from a zero accumulator (step (kb, r) contracts keys 16 kb + 4 g + r, g = 0..3),
        // then O^T = O^T * corr + tile on the vector ALU
        v4f ot[4];
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r = 0; r < 4; ++r) ot[db][r] = 0.0f;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int kr = kb * 16 + 4 * g + r;
#pragma unroll
                for (int db = 0; db < 4; ++db)
                    ot[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(sV[kr][db * 16 + c], st[kb][r], ot[db], 0, 0, 0);
            }
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r = 0; r < 4; ++r) o[db][r] = fmaf(o[db][r], corr, ot[db][r]);
        if (more) stash(stage ^ 1);
        __syncthreads();
    }

    uint32_t amax = 0;
    if (q < S) {
        float *dst = ctx + (tok0 + q) * Hd + hd * dh;
        const float inv = 1.0f / lrun;
#pragma unroll
        for (int db = 0; db < 4; ++db) {
            const int d = db * 16 + 4 * g;              // registers 0..3: four consecutive head dims
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[r] = o[db][r] * inv;
                const uint32_t ab = abs_bits(v[r]);
                amax = (d + r < dh && ab > amax) ? ab : amax;
            }
            if (vec4 && d + 4 <= dh) {
                *(float4 *)(dst + d) = make_float4(v[0], v[1], v[2], v[3]);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (d + r < dh) dst[d + r] = v[r];
            }
        }
    }
    // the workgroup's record: largest |context| stored, and the error bound of its values
    __shared__ uint32_t red[5][4];
    float qmax = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) qmax = fmaxf(qmax, fabsf(qr[i]));
    const uint32_t kbits = wave_max_u32(__float_as_uint(knorm2)), qbits = wave_max_u32(__float_as_uint(qmax));
    amax = wave_max_u32(amax);
    vmax = wave_max_u32(vmax);
    const uint32_t sbits = wave_max_u32(__float_as_uint(smax));       // non-negative floats order like integers
    if (lane == 0) { red[0][wave] = amax; red[1][wave] = vmax; red[2][wave] = sbits; red[3][wave] = kbits; red[4][wave] = qbits; }
    __syncthreads();
    if (tid == 0) {
        uint32_t a = 0, v = 0, sb = 0, kb = 0, qb = 0;
        for (int w = 0; w < 4; ++w) {
            a = a > red[0][w] ? a : red[0][w];
            v = v > red[1][w] ? v : red[1][w];
            sb = sb > red[2][w] ? sb : red[2][w];
            kb = kb > red[3][w] ? kb : red[3][w];
            qb = qb > red[4][w] ? qb : red[4][w];
        }
        AttnRecord r;
        r.amax_bits = a;
        // (the constant in the norm covers keys whose squares underflow)
        r.err = 5.9604645e-8f * __uint_as_float(v) *
                (kErrBase + kErrPerTile * (float)((S + kKeyTile - 1) / kKeyTile) + kErrPerScore * __uint_as_float(sb) +
                 kErrPerNorm * scale * __uint_as_float(qb) * (__builtin_amdgcn_sqrtf(__uint_as_float(kb)) + 1.0e-18f));
        if (!(r.err <= 3.402823466e+38f)) r.amax_bits = 0x7f800000u;   // non-finite inputs: flagged downstream
        rec[vid] = r;
    }
}

// ---- kernel 1: the approximate attention on the float16 matrix cores, products of fp32 values to 22 bits ----------
// The fp32 matrix instruction runs at 1/16 of the float16 one.  An fp32 value, scaled by a power of two, is the sum of
// two float16 values (the value rounded to 11 bits, the remainder rounded to 11 bits: what is left is at most 2^-23 of
// the value), so a product x * y is four float16 x float16 products, each exact in fp32; the three largest are issued
// (v_mfma_f32_32x32x16_f16, fp32 accumulation), the fourth is at most 2^-22 of the product.  Three bfloat16 parts, which
// need no scale, take six products: 48 instead of 24 matrix instructions per tile, 5.5 instead of 2 vector instructions
// per value split, and the kernel is bound by the sum of the two (64 x 256 tokens x 12 heads, without the norms for the error bound and
// what follows for the maximum: 88 us, with two float16 parts 64).
//   The scale.  float16 reaches from 2^-24 to 2^16: with the largest magnitude scaled to 2^14 .. 2^15, values down to 2^-14
// of it keep their full 22 bits and smaller ones are off by at most 2^-39 of the largest.  K and V are scaled by one power
// of two for the tensor, from the maximum that the QKV GEMM's epilogue leaves behind; a query row by its own; P (at most
// 4, see below) by 2^13.  What the absolute part adds is in the error bound, so that a tensor of very uneven magnitudes
// costs re-evaluations and nothing else.
// Within a chain the small partial products come first, so that the sums carried through most of the chain are
// small against the result (the matrix cores' accumulation drifts with the sums it carries).
// Geometry: a workgroup is four waves x 32 queries of one head; a tile is 32 keys.  S^T = K Q^T and
// O^T = V^T P^T as above, so a lane owns a query column: lane l holds query l % 32 and, of a 32-row
// block, rows 8 (i / 4) + 4 (l / 32) + i % 4 in accumulator register i.  Operands: lane l supplies row
// l % 32 and the 8 values of unit l / 32 of a 16-deep slab.  For the second product the lane's own
// registers 8 s .. 8 s + 7 are its unit of slab s (which keys share a unit is free as long as the V
// operand uses the same assignment), so P never leaves the registers; V is written to LDS transposed,
// as float16 planes [head dim][unit][slot] in that assignment.  K planes are [key][unit] with the units
// xor-rotated by the row; V rows are padded to 80 bytes: all 16-byte operand reads are conflict free.
//   The running maximum of a query is raised only when a tile passes it by more than a factor of 4 (any value near the
// maximum serves a soft-max as its reference), so the sums are rescaled in the first tiles and hardly ever again.
typedef float v16f __attribute__((ext_vector_type(16)));
typedef _Float16 v8hf __attribute__((ext_vector_type(8)));
typedef _Float16 v2hf __attribute__((ext_vector_type(2)));
// (defined further down; the kernel below ends with the exact evaluation of its candidates for the maximum)
__device__ __forceinline__ float context_exact(const float *__restrict__ qkv, int S, int Hd, int heads, int dh, double scale,
                                               uint32_t el, double *red);
template <typename F>
__device__ __forceinline__ void for_each_marked(bool mine, uint64_t *masks, F visit);
constexpr int kSplitQ = 128;             // queries per workgroup
constexpr int kSplitKeys = 32;           // keys per tile
constexpr int kSplitKRow = 128;          // bytes per key row of a K plane (8 units)
constexpr int kSplitVRow = 80;           // bytes per head-dim row of a V plane (4 units + pad)
constexpr int kSplitKPlane = kSplitKeys * kSplitKRow, kSplitVPlane = kDh * kSplitVRow;
constexpr int kSplitStage = 2 * (kSplitKPlane + kSplitVPlane);
// relative errors that make up the error bound of a query's values, in units of 2^-24 (where it is formed, below)
constexpr float kSplitErrBase = 2.5f, kSplitErrPerTile = 0.35f, kSplitErrPerScore = 2.5f, kSplitErrPerNorm = 2.5f;
constexpr float kPScale = 8192.0f;       // scale of P (at most 4) on its way to float16

// What a workgroup of the kernel below knows about the tensor's exact maximum: an upper bound of its own exact values,
// and which of its values can be its largest (as a rule one; with more than kCands it evaluates them itself and has none).
constexpr int kCands = 4;
struct AttnCand {
    float upper;
    uint32_t n;
    uint32_t at[kCands];    // token row * hidden + column
};

// the power of two that brings the largest magnitude (bit pattern) to 2^14 .. 2^15, and its inverse
__device__ __forceinline__ void f16_scale(uint32_t max_bits, float &up, float &down)
{
    const int b = 268 - (int)(max_bits >> 23), e = b > 253 ? 253 : b;
    up = __uint_as_float((uint32_t)e << 23);
    down = __uint_as_float((uint32_t)(254 - e) << 23);
}

struct Split2 {
    v4u h, l;
};
// two floats times s -> float16 pairs, x0 in the low half: a mixed-precision fma per value and part
__device__ __forceinline__ void split_pair(float x0, float x1, float s, uint32_t &h, uint32_t &l)
{
    asm("v_fma_mixlo_f16 %0, %2, %4, 0\n\t"
        "v_fma_mixhi_f16 %0, %3, %4, 0\n\t"
        "v_fma_mixlo_f16 %1, %2, %4, -%0 op_sel_hi:[0,0,1]\n\t"
        "v_fma_mixhi_f16 %1, %3, %4, -%0 op_sel:[0,0,1] op_sel_hi:[0,0,1]"
        : "=&v"(h), "=&v"(l)
        : "v"(x0), "v"(x1), "v"(s));
}
__device__ __forceinline__ Split2 split_eight(const float (&x)[8], float s)
{
    Split2 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint32_t wh, wl;
        split_pair(x[2 * e], x[2 * e + 1], s, wh, wl);
        o.h[e] = wh;
        o.l[e] = wl;
    }
    return o;
}
// The same of values that a matrix instruction reads next: written so that the compiler sees the instructions and keeps
// their distance to it.
__device__ __forceinline__ Split2 split_eight_operand(const float (&x)[8], float s)
{
    Split2 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const v2hf hh = {(_Float16)(x[2 * e] * s), (_Float16)(x[2 * e + 1] * s)};
        uint32_t wh = __builtin_bit_cast(uint32_t, hh);
        asm("" : "+v"(wh));                                      // (else the halves are converted a second time below)
        const v2hf hv = __builtin_bit_cast(v2hf, wh);
        const v2hf ll = {(_Float16)fmaf(x[2 * e], s, -(float)hv[0]), (_Float16)fmaf(x[2 * e + 1], s, -(float)hv[1])};
        o.h[e] = wh;
        o.l[e] = __builtin_bit_cast(uint32_t, ll);
    }
    return o;
}
// the larger of a lane's value and that of the lane 32 away
__device__ __forceinline__ float max_halves(float x) { return pair_op<32>(x, [](float a, float b) { return fmaxf(a, b); }); }

__global__ __launch_bounds__(256, 2) void attention_split_kernel(const float *__restrict__ qkv, int B, int S, int Hd,
                                                                 int heads, int dh, float scale, float *__restrict__ ctx,
                                                                 float *__restrict__ err_q, AttnCand *__restrict__ cands,
                                                                 const uint32_t *__restrict__ max_slot,
                                                                 uint32_t *__restrict__ bound_slot,
                                                                 uint32_t *__restrict__ exact_slot)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * kSplitStage];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = lane & 31, h = lane >> 5;
    const int qblocks = (S + kSplitQ - 1) / kSplitQ;
    const int vid = (int)xcd_piece(blockIdx.x, gridDim.x);
    const int bh = vid / qblocks, qb = vid % qblocks;
    const int bi = bh / heads, hd = bh % heads;
    const int64_t tok0 = (int64_t)bi * S;
    const int64_t ld = 3 * (int64_t)Hd;
    const float *qbase = qkv + hd * dh, *kbase = qbase + Hd, *vbase = qbase + 2 * Hd;

    // the wave's queries: lane (r, h) holds dims 16 sl + 8 h .. + 7 of query r
    const int q = qb * kSplitQ + wave * 32 + r;
    float4 raw[8];
    {
        const float *qrow = qbase + (tok0 + (q < S ? q : S - 1)) * ld;
#pragma unroll
        for (int sl = 0; sl < 4; ++sl) {
            const int d0 = 16 * sl + 8 * h;
            const int dc = d0 < dh ? d0 : 0;                     // head dims come in whole units of 8
            raw[2 * sl] = *(const float4 *)(qrow + dc);
            raw[2 * sl + 1] = *(const float4 *)(qrow + dc + 4);
        }
    }

    // staging.  K: thread t takes unit t % 8 (8 head dims) of key t / 8.  V: lane l of wave w takes head dims
    // 4 (4 w + l % 4) .. + 3 of keys 2 (l / 4) and 2 (l / 4) + 1 (two keys that are neighbours in a unit: one
    // 4-byte LDS word per head dim and plane; a wave's words fall into 64 different banks).
    const int skr = tid >> 3, sku = tid & 7;
    const int svd = 4 * (4 * wave + (lane & 3)), svk = 2 * (lane >> 2);
    const uint32_t koff = (uint32_t)(skr * kSplitKRow + ((sku ^ ((skr >> 1) & 7)) * 16));
    // key k of a tile: slab k / 16, unit 2 (k / 16) + (k / 4) % 2, slot 4 ((k / 8) % 2) + k % 4
    const uint32_t voff = (uint32_t)(svd * kSplitVRow + (2 * (svk >> 4) + ((svk >> 2) & 1)) * 16 + (4 * ((svk >> 3) & 1) + (svk & 3)) * 2);
    float vmax = 0.0f;                  // largest |v| staged by this thread
    float vsq[4] = {0.0f, 0.0f, 0.0f, 0.0f};   // sums of v^2 over the keys it staged, per head dim
    float knorm2 = 0.0f;                // largest squared norm of the keys it staged a part of
    float4 pk[2], pv[2];
    // Loads are unconditional, from clamped addresses: a key beyond S reads the last key's row (its score is
    // masked in the ragged tile, its P is exactly zero), head dims beyond dh read dims 0.. (the query is zero
    // there, and those rows of O^T are never stored).  No zeroing, so nothing waits for a load before its use.
    const float *kfetch = kbase + tok0 * ld + (8 * sku < dh ? 8 * sku : 0);
    const float *vfetch = vbase + tok0 * ld + (svd < dh ? svd : 0);
    auto fetch_k = [&](int j0) {
        const int row = j0 + skr < S ? j0 + skr : S - 1;
        const float *kp = kfetch + (int64_t)row * ld;
        pk[0] = *(const float4 *)kp;
        pk[1] = *(const float4 *)(kp + 4);
    };
    auto fetch_v = [&](int j0) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int row = j0 + svk + e < S ? j0 + svk + e : S - 1;
            pv[e] = *(const float4 *)(vfetch + (int64_t)row * ld);
        }
    };
    fetch_k(0);
    fetch_v(0);

    // the largest |value| of the tensor: the scale of K and V
    const uint32_t mbits = (uint32_t)__builtin_amdgcn_readfirstlane((int)reduce_ways(max_slot));
    float kv_up, kv_down, q_up, q_down;
    f16_scale(mbits, kv_up, kv_down);
    Split2 qs[4];
    float qmax = 0.0f;
    {
        float x[4][8];
#pragma unroll
        for (int sl = 0; sl < 4; ++sl) {
            const bool ok = q < S && 16 * sl + 8 * h < dh;
            const float4 a = raw[2 * sl], b4 = raw[2 * sl + 1];
            const float t[8] = {a.x, a.y, a.z, a.w, b4.x, b4.y, b4.z, b4.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                x[sl][e] = ok ? t[e] : 0.0f;
                qmax = fmaxf(qmax, fabsf(x[sl][e]));
            }
        }
        qmax = max_halves(qmax);
        f16_scale(__float_as_uint(qmax), q_up, q_down);
#pragma unroll
        for (int sl = 0; sl < 4; ++sl) qs[sl] = split_eight_operand(x[sl], q_up);
    }
    auto stash_k = [&](int buf) {
        uint8_t *kst = lds + buf * kSplitStage;
        const float x[8] = {pk[0].x, pk[0].y, pk[0].z, pk[0].w, pk[1].x, pk[1].y, pk[1].z, pk[1].w};
        const Split2 sp = split_eight(x, kv_up);
        *(v4u *)(kst + koff) = sp.h;
        *(v4u *)(kst + kSplitKPlane + koff) = sp.l;
        float n2 = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) n2 = fmaf(x[e], x[e], n2);
        n2 = 8 * sku < dh ? n2 : 0.0f;
        n2 = wave_reduce<4>(n2, [](float a, float b) { return a + b; });     // the eight lanes of a key
        knorm2 = fmaxf(knorm2, n2);
    };
    auto stash_v = [&](int buf) {
        uint8_t *vst = lds + buf * kSplitStage + 2 * kSplitKPlane;
        const float v0[4] = {pv[0].x, pv[0].y, pv[0].z, pv[0].w}, v1[4] = {pv[1].x, pv[1].y, pv[1].z, pv[1].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t wh, wl;
            split_pair(v0[e], v1[e], kv_up, wh, wl);
            uint8_t *dst = vst + voff + e * kSplitVRow;
            *(uint32_t *)dst = wh;
            *(uint32_t *)(dst + kSplitVPlane) = wl;
            vmax = fmaxf(vmax, fmaxf(fabsf(v0[e]), fabsf(v1[e])));
            vsq[e] = fmaf(v0[e], v0[e], fmaf(v1[e], v1[e], vsq[e]));
        }
    };

    // (plane of the K or V operand, plane of the Q or P operand), 0 = high part; the small products come first
    constexpr int ia[3] = {1, 0, 0}, ib[3] = {0, 1, 0};
    const uint32_t ka_off = (uint32_t)(r * kSplitKRow), ka_sw = (uint32_t)((r >> 1) & 7);
    // scaled scores of the tile in K buffer `buf`: register i is key 8 (i / 4) + 4 h + i % 4 of the tile for this
    // lane's query
    auto scores = [&](int buf) {
        const uint8_t *kst = lds + buf * kSplitStage;
        v16f acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
#pragma unroll
        for (int pr = 0; pr < 3; ++pr)
#pragma unroll
            for (int sl = 0; sl < 4; ++sl) {
                const v4u ak = *(const v4u *)(kst + ia[pr] * kSplitKPlane + ka_off + ((((uint32_t)(2 * sl + h)) ^ ka_sw) * 16));
                const v4u bq = ib[pr] == 0 ? qs[sl].h : qs[sl].l;
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8hf, ak), __builtin_bit_cast(v8hf, bq), acc, 0, 0, 0);
            }
        return acc;
    };

    v16f o[2];
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] = 0.0f;
    float mrun = 0.0f, lrun = 0.0f;     // reference of the scaled scores, this lane's share of the sum of P
    float p2run = 0.0f;                 // ... and of the sum of P^2 (for the error bound)
    float smax = 0.0f;                  // largest |scaled score| met by this lane
    const float c2 = scale * 1.44269504088896340736f * q_down * kv_down;   // scaled score -> exponent of 2

    // Software pipeline over the tiles.  Iteration t contracts S(t + 1), turns S(t) into P(t), contracts
    // P(t) V(t) and splits K(t + 2) and V(t + 1) (in registers since the iteration before) into the buffers
    // that S(t) and V(t - 1) have left: the scores of the next tile do not wait for this tile's soft-max, and
    // a tile's loads have a whole iteration to arrive.  One barrier per tile.
    const int ntiles = (S + kSplitKeys - 1) / kSplitKeys;
    stash_k(0);
    stash_v(0);
    fetch_k(kSplitKeys);
    fetch_v(kSplitKeys);
    stash_k(1);
    fetch_k(2 * kSplitKeys);
    __syncthreads();
    v16f sacc = scores(0);
    __syncthreads();                                             // K buffer 0 is rewritten in iteration 0
    // (the loads are unconditional; scores and staging of tiles past the end are skipped under uniform branches)
    auto iteration = [&](int t, auto ragged) {
        const int j0 = t * kSplitKeys;
        v16f snext = sacc;
        if (t + 1 < ntiles) snext = scores((t + 1) & 1);
        // soft-max of tile t
        float mx = sacc[0], mn = sacc[0];                        // keys beyond S repeat the last key's score here
#pragma unroll
        for (int i = 1; i < 16; ++i) { mx = fmaxf(mx, sacc[i]); mn = fminf(mn, sacc[i]); }
        smax = fmaxf(smax, fmaxf(mx, -mn));
        mx = max_halves(mx);
        if (t == 0) {
            mrun = mx;
        } else if (__any((mx - mrun) * c2 > 2.0f)) {
            const float mnew = fmaxf(mrun, mx);
            const float corr = __builtin_amdgcn_exp2f((mrun - mnew) * c2);
            mrun = mnew;
            lrun *= corr;
            p2run *= corr * corr;
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[db][i] *= corr;
        }
        const float shift = -mrun * c2;
        float ps = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            sacc[i] = __builtin_amdgcn_exp2f(fmaf(sacc[i], c2, shift));
            // the ragged last tile: keys beyond S do not count (an infinite score would meet a factor c2 that is zero)
            if constexpr (decltype(ragged)::value) sacc[i] = j0 + 8 * (i >> 2) + 4 * h + (i & 3) < S ? sacc[i] : 0.0f;
            ps += sacc[i];
            p2run = fmaf(sacc[i], sacc[i], p2run);
        }
        lrun += ps;
        // the lane's unit of slab s of P^T: its registers 8 s .. 8 s + 7
        Split2 pp[2];
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) {
            const float x[8] = {sacc[8 * sl], sacc[8 * sl + 1], sacc[8 * sl + 2], sacc[8 * sl + 3],
                                sacc[8 * sl + 4], sacc[8 * sl + 5], sacc[8 * sl + 6], sacc[8 * sl + 7]};
            pp[sl] = split_eight_operand(x, kPScale);
        }
        // this tile's V^T P^T from zero accumulators (two independent chains, one per half of the head dims),
        // then O^T = O^T + tile on the vector ALU
        {
            const uint8_t *vst = lds + (t & 1) * kSplitStage + 2 * kSplitKPlane;
            v16f ot[2];
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) ot[db][i] = 0.0f;
#pragma unroll
            for (int pr = 0; pr < 3; ++pr)
#pragma unroll
                for (int sl = 0; sl < 2; ++sl) {
                    const v4u bp = ib[pr] == 0 ? pp[sl].h : pp[sl].l;
#pragma unroll
                    for (int db = 0; db < 2; ++db) {
                        const v4u av = *(const v4u *)(vst + ia[pr] * kSplitVPlane + (32 * db + r) * kSplitVRow + (2 * sl + h) * 16);
                        ot[db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8hf, av), __builtin_bit_cast(v8hf, bp), ot[db], 0, 0, 0);
                    }
                }
            if (t + 2 < ntiles) stash_k(t & 1);
            if (t + 1 < ntiles) stash_v((t + 1) & 1);
            fetch_k(j0 + 3 * kSplitKeys);
            fetch_v(j0 + 2 * kSplitKeys);
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[db][i] += ot[db][i];
        }
        sacc = snext;
        __syncthreads();
    };
    const int nfull = S / kSplitKeys;
    for (int t = 0; t < nfull; ++t) iteration(t, std::false_type{});
    if (nfull < ntiles) iteration(nfull, std::true_type{});

    __shared__ float red_v[4], red_k[4], red_n[4], red_low[4], red_up[4];
    __shared__ uint32_t n_cand;
    if (tid == 0) n_cand = 0;
    vmax = __uint_as_float(wave_max_u32(__float_as_uint(vmax)));  // non-negative floats order like integers
    knorm2 = __uint_as_float(wave_max_u32(__float_as_uint(knorm2)));
    // the sixteen lanes of a group of head dims, then the largest of all dims
    float vn2 = 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        vsq[e] = pair_op<32>(vsq[e], [](float a, float b) { return a + b; });
        vsq[e] = pair_op<16>(vsq[e], [](float a, float b) { return a + b; });
        vsq[e] += lane_xor<8>(vsq[e]);
        vsq[e] += lane_xor<4>(vsq[e]);
        vn2 = fmaxf(vn2, vsq[e]);
    }
    vn2 = __uint_as_float(wave_max_u32(__float_as_uint(vn2)));
    if (lane == 0) { red_v[wave] = vmax; red_k[wave] = knorm2; red_n[wave] = vn2; }
    // the two halves of a query's sums; the factor that undoes every scale
    lrun += lane_xor<32>(lrun);
    p2run += lane_xor<32>(p2run);
    const float outs = kv_down * (1.0f / kPScale), inv = 1.0f / lrun;
    // register i of block db is head dim 32 db + 8 (i / 4) + 4 h + i % 4 of this lane's query
    float amax = 0.0f;
    float *dst = ctx + (tok0 + (q < S ? q : S - 1)) * Hd + hd * dh;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int d = 32 * db + 8 * g + 4 * h;
            if (d < dh) {                                        // head dims come in whole units of 8
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    o[db][4 * g + e] = o[db][4 * g + e] * inv * outs;
                    amax = fmaxf(amax, fabsf(o[db][4 * g + e]));
                }
                if (q < S) *(float4 *)(dst + d) = make_float4(o[db][4 * g], o[db][4 * g + 1], o[db][4 * g + 2], o[db][4 * g + 3]);
            }
        }
    __syncthreads();
    vmax = fmaxf(fmaxf(red_v[0], red_v[1]), fmaxf(red_v[2], red_v[3]));
    // Error bound of the query's values (the part that grows with a value itself comes on top, value_err).  A value is
    // sum P v / sum P, and every relative error e of a P or a v moves it by at most e sum P |v| / sum P, plus e |x| for its
    // share of the denominator.  Nothing is taken to average out: keys that repeat or lie close together (padding, few
    // distinct tokens) have the same errors.  sum P |v| / sum P is at most the largest |v| of the head and, by Cauchy and
    // Schwarz, sqrt(sum P^2) / sum P times the largest norm of a head dim of V: where the weights are spread over many keys
    // the second one is a third to a half of the first.
    //   e, in units of 2^-24: the splits of V and P, P's own rounding and the exponential (kSplitErrBase); a rounding per tile
    // of the sums that are carried (kSplitErrPerTile); the roundings of the score's sum, which go with the score
    // (kSplitErrPerScore); the splits of Q and K, which go with the root of sum (q k)^2 over the head dims, at most the
    // largest |q| times the largest norm of a key (kSplitErrPerNorm).  The constants are measured, with margin, not proved:
    // bench.py --attention-error sets the error against the bound for two dozen kinds of input (normal, padded, two to eight
    // distinct tokens, values of opposite sign, equal scores up to 300, terms that cancel in the scores) at 8 to 64 dims and 131
    // to 2048 tokens; the worst is 0.71 of it (0.86 over more seeds and 65 to 4096 tokens).  With the P taken to be independent
    // of each other (root of sum P^2 alone) it was 12 times the bound for two tokens and 97 for cancelling terms.  The longer
    // lists cost the quantiser 63 -> 82 us for 64 x 256 tokens x 12 heads (with the maximum settled in it), the norms this kernel
    // 85 -> 88.
    const float M = __uint_as_float(mbits);
    const float sq = max_halves(smax) * c2 * 0.6931472f;         // largest |score| of the query
    auto of_all = [](const float *x) { return fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])); };
    // (the constants cover values whose squares underflow)
    const float kn = __builtin_amdgcn_sqrtf(of_all(red_k)) + 1.0e-18f, vn = __builtin_amdgcn_sqrtf(of_all(red_n)) + 1.1e-19f * (float)S;
    const float spread = fminf(vmax, __builtin_amdgcn_sqrtf(p2run) * inv * vn + max_halves(amax));
    float err = 5.9604645e-8f * (spread * (kSplitErrBase + kSplitErrPerTile * (float)ntiles + kSplitErrPerScore * sq +
                                           scale * qmax * (kSplitErrPerNorm * kn + (float)dh * M * 1.2207031e-4f)) +
                                 M * (float)(S + 2) * 6.1035156e-5f);
    // A bound that is no number: every value of the query is re-evaluated (finite inputs whose scores pass 3e38 only)
    if (!(err <= 3.402823466e+38f)) err = INFINITY;
    if (h == 0 && q < S) err_q[(int64_t)bh * S + q] = err;
    if (!bound_slot) return;                                     // the kernel alone (error measurement)

    // What the workgroup knows about the tensor's exact maximum.  It raises a shared word to a lower bound of its own exact
    // maximum (largest stored |x| minus its error) and leaves an upper bound and the values that reach its own lower
    // bound; the launch that follows evaluates those that reach the tensor's.  (Evaluated here, nearly every workgroup
    // of the first round found its own maximum above all that was reported by then: 21 -> 36 us for 32 x 128 tokens x 12
    // heads, 88 -> 104 for 64 x 256.)
    if (mbits >= 0x7f800000u || mbits == 0) {                    // NaN / Inf: they are the "maximum"; zeros: nothing to find
        if (tid == 0) {
            if (mbits) atomicMax(exact_slot + (blockIdx.x & (kAmaxWays - 1)) * kAmaxStride, 0x7f800000u);
            cands[vid].upper = 0.0f;
            cands[vid].n = 0;
        }
        return;
    }
    // (the factor and the 2^-23 |x| term cover the rounding of this fp32 arithmetic itself)
    const float off = fmaf(amax, 1.2e-7f, value_err(err, amax) * 1.001f);
    float low = 0.0f, up = 0.0f;
    if (q < S) {
        low = fmaxf(amax - off, 0.0f);
        up = amax + off;
        up = up < INFINITY ? up : INFINITY;
    }
    low = __uint_as_float(wave_max_u32(__float_as_uint(low)));
    up = __uint_as_float(wave_max_u32(__float_as_uint(up)));
    if (lane == 0) { red_low[wave] = low; red_up[wave] = up; }
    __syncthreads();
    low = fmaxf(fmaxf(red_low[0], red_low[1]), fmaxf(red_low[2], red_low[3]));
    up = fmaxf(fmaxf(red_up[0], red_up[1]), fmaxf(red_up[2], red_up[3]));
    // bit 16 db + i: that register's value may be as large as floor_v (a NaN counts as anything)
    auto candidates = [&](float floor_v) {
        const float thr = floor_v * (1.0f - 2.0e-6f) - err * 1.001f;
        uint32_t c = 0;
        if (__any(q < S && !(amax < thr))) {
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (32 * db + 8 * (i >> 2) + 4 * h + (i & 3) < dh && !(fabsf(o[db][i]) < thr)) c |= 1u << (16 * db + i);
            if (q >= S) c = 0;
        }
        return c;
    };
    uint32_t cand = candidates(low);
    if (cand) {
        uint32_t at = atomicAdd(&n_cand, (uint32_t)__popc(cand));
        for (uint32_t c = cand; c && at < kCands; c &= c - 1, ++at) {
            const int sl = __ffs((int)c) - 1;
            cands[vid].at[at] = (uint32_t)((tok0 + q) * Hd + hd * dh + 32 * (sl >> 4) + 8 * ((sl & 15) >> 2) + 4 * h + (sl & 3));
        }
    }
    __syncthreads();
    const bool few = n_cand <= kCands;
    if (tid == 0) {
        cands[vid].upper = few ? up : 0.0f;
        cands[vid].n = few ? n_cand : 0;
        atomicMax(bound_slot + (blockIdx.x & (kAmaxWays - 1)) * kAmaxStride, __float_as_uint(low));
    }
    if (few) return;
    // More values than the list holds can be this workgroup's largest (many equal rows): evaluated here, those that reach
    // the largest lower bound reported so far (a stale value only admits more of them)
    const float floor_v = fmaxf(low, __uint_as_float(wave_max_u32(__hip_atomic_load(bound_slot + lane * kAmaxStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))));
    cand = candidates(floor_v);
    __shared__ uint64_t masks[4];
    double *redd = (double *)lds;                                // the stage memory is free now
    const double scale_d = 1.0 / sqrt((double)dh);
    uint32_t best = 0;
    for (int sl = 0; sl < 32; ++sl) {
        if (!__syncthreads_or((cand >> sl) & 1u)) continue;
        for_each_marked(((cand >> sl) & 1u) != 0, masks, [&](int k) {
            const int wk = k >> 6, rk = k & 31, hk = (k >> 5) & 1;
            const int qk = qb * kSplitQ + wk * 32 + rk;
            const int dk = 32 * (sl >> 4) + 8 * ((sl & 15) >> 2) + 4 * hk + (sl & 3);
            const float x = context_exact(qkv, S, Hd, heads, dh, scale_d, (uint32_t)((tok0 + qk) * Hd + hd * dh + dk), redd);
            const uint32_t ab = abs_bits(x);
            best = best > ab ? best : ab;
        });
    }
    if (tid == 0 && best) atomicMax(exact_slot + (blockIdx.x & (kAmaxWays - 1)) * kAmaxStride, best);
}

// The context value of one (query token, head, dim) as the fp64 evaluation defines it:
// scores in fp64 (products summed over the head dims in ascending
// order, then the 1/sqrt(dh) factor), soft-max and the weighted sum of v in fp64, rounded once.  q, k and
// v rows are read from the packed qkv tensor.  Every load is unconditional (indices clamped to valid
// ones, the query zero beyond dh): a load under a condition is awaited on its own, and a key row would
// cost sixteen memory round trips instead of one.
// (kept compact and inlined once per kernel: called as a function it needs scratch memory for the
// caller's registers and ran five times slower)  The whole workgroup of 256 threads evaluates one value, a key per thread.
// Head dims in whole units of 4 floats.  red: 12 + 32 doubles.
__device__ __forceinline__ float context_exact(const float *__restrict__ qkv, int S, int Hd, int heads, int dh, double scale,
                                               uint32_t el, double *red)
{
    const uint32_t mrow = el / (uint32_t)Hd, col = el - mrow * (uint32_t)Hd;
    const uint32_t bi = mrow / (uint32_t)S, hd = col / (uint32_t)dh, dd = col - hd * (uint32_t)dh;
    const int64_t ld = 3 * (int64_t)Hd;
    const float *q = qkv + (int64_t)mrow * ld + hd * dh;
    const float *kb = qkv + (int64_t)bi * S * ld + Hd + hd * dh, *vb = kb + Hd + dd;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int units = dh >> 2;
    // the query row goes through LDS (64 floats behind the waves' sums): every thread needs all of it.
    // Its load and the first block's key and value loads are requested together, before the barriers: the
    // evaluation is a chain of memory round trips, and this takes one out of it.
    float *qs = (float *)(red + 12);
    float4 kv[16];
    float vj = 0.0f;
    auto request = [&](int j0) {
        const int j = j0 + tid;
        const int jj = j < S ? j : S - 1;
        const float *kr = kb + (int64_t)jj * ld;
        vj = vb[(int64_t)jj * ld];
#pragma unroll
        for (int u = 0; u < 16; ++u) kv[u] = *(const float4 *)(kr + 4 * (u < units ? u : units - 1));
    };
    const float qreg = (tid < 64 && tid < dh) ? q[tid] : 0.0f;
    request(0);
    __syncthreads();                                          // an earlier call has finished with red and qs
    if (tid < 64) qs[tid] = qreg;
    __syncthreads();
    double m = -INFINITY, l = 0.0, o = 0.0;
    for (int j0 = 0; j0 < S; j0 += 256) {
        const int j = j0 + tid;
        if (j0) request(j0);
        // a product of two fp32 values is exact in fp64, so each fma below is the multiply and the
        // add of the plain definition, in its order (dims ascending)
        double acc = 0.0;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            if (u < units) {
                const float4 qv = *(const float4 *)&qs[4 * u];
                acc = fma((double)qv.x, (double)kv[u].x, acc);
                acc = fma((double)qv.y, (double)kv[u].y, acc);
                acc = fma((double)qv.z, (double)kv[u].z, acc);
                acc = fma((double)qv.w, (double)kv[u].w, acc);
            }
        }
        const double sc = j < S ? acc * scale : -INFINITY;
        const double cm = wave_max(sc);
        __syncthreads();                                      // red is free (an earlier block, an earlier call)
        if (lane == 0) red[wave] = cm;
        __syncthreads();
        const double mnew = fmax(m, fmax(fmax(red[0], red[1]), fmax(red[2], red[3])));
        const double p = exp(sc - mnew);                 // exp(-inf) = 0 for the keys beyond S
        const double corr = j0 == 0 ? 0.0 : exp(m - mnew);
        const double ps = wave_sum(p), po = wave_sum(p * (double)vj);
        if (lane == 0) { red[4 + wave] = ps; red[8 + wave] = po; }
        __syncthreads();
        l = l * corr + ((red[4] + red[5]) + (red[6] + red[7]));
        o = o * corr + ((red[8] + red[9]) + (red[10] + red[11]));
        m = mnew;
    }
    return (float)(o / l);
}

// Workgroup-uniform walk over the values a predicate marks among 256 consecutive candidates: every thread
// passes its own flag, and `visit(k)` runs, in all threads, for every marked k = 0..255 in ascending order.
template <typename F>
__device__ __forceinline__ void for_each_marked(bool mine, uint64_t *masks, F visit)
{
    const uint64_t b = __ballot(mine);
    __syncthreads();                                          // masks is free
    if ((threadIdx.x & 63) == 0) masks[threadIdx.x >> 6] = b;
    __syncthreads();
    for (int w = 0; w < 4; ++w) {
        uint64_t mask = masks[w];
        while (mask) {
            const int src = __ffsll((long long)mask) - 1;
            mask &= mask - 1;
            visit(w * 64 + src);
        }
    }
}

// The exact maximum from the candidates: a thread per attention workgroup; if that can hold the maximum, the whole workgroup
// evaluates its candidates.  As a rule there is one in the tensor, but equal samples tie, at the same place of each: sixteen
// attention workgroups to a workgroup here share them out.  (With this in the certifying quantiser, where every
// workgroup read all bounds and evaluated all candidates for itself, the time went with the square of the batch: one layer
// of 768 x 12 heads, us, distinct / equal samples of 256 tokens: batch 64 354 / 1010, now 345 / 363;
// 512 2363 / 43187, now 2170 / 2297.)
constexpr int kSettleWorkgroups = 16;      // (a power of two)
__global__ __launch_bounds__(256) void attention_settle_kernel(const float *__restrict__ qkv, const AttnCand *__restrict__ cands,
                                                               int nwg, const uint32_t *__restrict__ bound, int S, int Hd, int heads,
                                                               int dh, double scale, uint32_t *__restrict__ exact)
{
    __shared__ __attribute__((aligned(16))) double red[12 + 32];
    __shared__ uint64_t masks[4];
    __shared__ AttnCand sc[kSettleWorkgroups];
    const int w = blockIdx.x * kSettleWorkgroups + (int)(threadIdx.x & (kSettleWorkgroups - 1));
    const AttnCand mine = cands[w < nwg ? w : nwg - 1];
    const float floor_v = __uint_as_float(reduce_ways(bound));
    if (threadIdx.x < kSettleWorkgroups) sc[threadIdx.x] = mine;
    uint32_t best = 0;
    for_each_marked(threadIdx.x < kSettleWorkgroups && w < nwg && mine.upper >= floor_v && mine.upper > 0.0f, masks, [&](int k) {
        const AttnCand &c = sc[k];
        for (uint32_t e = 0; e < c.n; ++e) {
            const uint32_t ab = abs_bits(context_exact(qkv, S, Hd, heads, dh, scale, c.at[e], red));
            best = best > ab ? best : ab;
        }
    });
    if (threadIdx.x == 0 && best) atomicMax(exact + (blockIdx.x & (kAmaxWays - 1)) * kAmaxStride, best);
}

// The int8 codes of the context under the tensor's exact scale: a workgroup of four waves per (batch element, head), or
// for a share of its tokens where that leaves compute units idle.  It streams over its slice of the approximate context: a
// thread maps 16 consecutive values of a token row (one 16-byte store; WIDE: head size and row length are multiples of
// 16) or a single value.  A value whose interval [x - E, x + E] maps to two codes gets a provisional code
// and goes on the workgroup's list in LDS (token * dh + dim within the head).  After each pass the workgroup re-evaluates
// the listed values in fp64 and overwrites their codes.  A re-evaluation needs all keys of its head (S x dh floats): read
// from global memory per value, that traffic (and the sixteen-byte pieces of 256 different rows each load instruction asks
// for) would bound the whole step.  The workgroup copies the head's keys into LDS, 256 at a
// time, with coalesced loads, and re-evaluates sixteen listed values together from there, on the fp64 matrix cores (rows padded by
// 16 bytes against bank conflicts); only the value columns (one float per key and value) come from global memory.  Up to 256 keys are
// copied once; more are copied for every sixteen values.  What bounds it: a workgroup's chain of round trips (its keys 4 us, codes
// 3, sixteen re-evaluations 5, of which it has one as a rule) and, for many heads, the value columns: a line per key and value
// listed, four to twelve of them per head and 256 tokens.  With a value per wave and its keys spread over the lanes (four values
// in 4 us, two to six times over) it took, us: 24 x 197 tokens x 12 heads 42, now 25; in the stack of 64 x 256 tokens 64, now 47; 8 x
// 384 x 12 49, now 27.  (Eight waves and 128 registers: spills, 30 % longer.)
constexpr int kKeysLds = 256;            // keys a workgroup can hold
constexpr int kKeyRow = kDh + 4;         // floats per key row in LDS (one 16-byte pad)

// true if the approximate value x with error bound err does not settle its code
// (The exact value y lies in [x - e, x + e]; its code is clamp(rne(fl(y * inv))) with fl(y * inv) within
// e * inv + 2^-23 |t| of t = fl(x * inv).  The two codes can differ only if that interval reaches the rounding
// boundary next to t, i.e. |t - rne(t)| + e * inv + 2^-23 |t| >= 1/2; the margins below are a little wider.)
__device__ __forceinline__ bool code_uncertain(float x, float err, float inv)
{
    const float t = x * inv;
    const float reach = fmaf(value_err(err, x) * 1.001f, inv, 2.4e-7f * fabsf(t)) + 1.0e-30f;
    return !(fabsf(t - rintf(t)) + reach < 0.5f);                  // also true for a non-finite bound
}

constexpr int kCertifyThreads = 256;
template <bool WIDE>
__global__ __launch_bounds__(kCertifyThreads, 2) void quantize_attention_certify_kernel(
    const float *__restrict__ qkv, const float *__restrict__ ctx, const float *__restrict__ err_q,
    int S, int Hd, int heads, int dh, int splits, int tokens, double scale, const uint32_t *__restrict__ exact, int8_t *xq, int64_t ldq,
    float *__restrict__ scale_out, uint32_t *__restrict__ flag, uint32_t *__restrict__ unsure_total)
{
    constexpr int NT = kCertifyThreads, NW = NT / 64;
    constexpr int NPRE = 4;                                       // passes whose loads are requested together
    constexpr int TPP = NT / 4;                                   // WIDE: tokens of a pass (four lanes take a token's 64 dims)
    constexpr uint32_t kList = 1024;                              // list entries served per round
    __shared__ uint32_t todo[kList];
    __shared__ uint32_t n_todo, more;
    __shared__ __attribute__((aligned(16))) float ks[kKeysLds * kKeyRow];
    __shared__ double red[NW][16][3];                             // the waves' maximum and sums of sixteen values
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t piece = xcd_piece(blockIdx.x, gridDim.x), bh = piece / (uint32_t)splits, share = piece - bh * (uint32_t)splits;
    const uint32_t bi = bh / (uint32_t)heads, hd = bh - bi * (uint32_t)heads;
    const uint32_t tok0 = bi * (uint32_t)S;
    const int64_t ld = 3 * (int64_t)Hd;
    const float *qb = qkv + (int64_t)tok0 * ld + hd * dh, *kb = qb + Hd, *vb = kb + Hd;
    const uint32_t t0 = share * (uint32_t)tokens, nt = (uint32_t)S - t0 < (uint32_t)tokens ? (uint32_t)S - t0 : (uint32_t)tokens;
    // units of the share: 16-value groups of a token (WIDE), or single columns (the last head also clears the pad columns
    // [Hd, ldq) of its tokens)
    const uint32_t upt = WIDE ? 4u : (uint32_t)dh + (hd + 1u == (uint32_t)heads ? (uint32_t)(ldq - Hd) : 0u);
    const uint32_t passes = WIDE ? (nt + TPP - 1) / TPP : (nt * upt + NT - 1) / NT;
    // this thread's unit of pass p: token of the head, unit of the token; false: none
    auto locate = [&](uint32_t p, uint32_t &t, uint32_t &part) {
        if (WIDE) {
            part = (uint32_t)tid & 3u;
            t = p * TPP + ((uint32_t)tid >> 2);
            const bool ok = t < nt && part * 16u < (uint32_t)dh;
            if (!ok) t = part = 0;
            t += t0;
            return ok;
        }
        const uint32_t u = p * NT + (uint32_t)tid;
        const bool ok = u < nt * upt;
        t = ok ? u / upt : 0u;
        part = ok ? u - t * upt : 0u;
        t += t0;
        return ok;
    };
    float4 v[NPRE][WIDE ? 4 : 1];
    float ev[NPRE];
    auto request = [&](uint32_t p0) {
#pragma unroll
        for (int i = 0; i < NPRE; ++i) {
            uint32_t t, part;
            locate(p0 + i, t, part);
            ev[i] = err_q[(int64_t)bh * S + t];
            if (WIDE) {
                const float4 *p = (const float4 *)(ctx + (int64_t)(tok0 + t) * Hd + hd * (uint32_t)dh + part * 16u);
#pragma unroll
                for (int j = 0; j < 4; ++j) v[i][j] = p[j];
            } else {
                const uint32_t col = hd * (uint32_t)dh + part;
                v[i][0].x = ctx[(int64_t)(tok0 + t) * Hd + (col < (uint32_t)Hd ? col : (uint32_t)Hd - 1u)];
            }
        }
    };
    request(0);
    // keys j0 .. j0 + 255 of the head into LDS: sixteen lanes take a row, four rows per thread in flight (a barrier orders
    // them before any read)
    auto stage_keys = [&](int j0) {
        constexpr int RPB = NT / 16;
        const int nj = S - j0 < kKeysLds ? S - j0 : kKeysLds;
        const int d = (tid & 15) * 4, r = tid >> 4;
        const bool ok = d < dh;
        const float *src = kb + (int64_t)j0 * ld + (ok ? d : 0);
        for (int r0 = 0; r0 < nj; r0 += 4 * RPB) {
            v4f t[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = r0 + i * RPB + r;
                t[i] = *(const v4f *)(src + (int64_t)(row < nj ? row : nj - 1) * ld);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = r0 + i * RPB + r;
                if (ok && row < nj) *(v4f *)&ks[row * kKeyRow + d] = t[i];
            }
        }
    };
    if (S <= kKeysLds) stage_keys(0);
    float sc_f;
    bool bad;
    const float inv = scale_from_bits(reduce_ways(exact), nullptr, &sc_f, &bad);
    if (blockIdx.x == 0 && threadIdx.x == 0) publish(sc_f, bad, scale_out, nullptr, flag);
    uint32_t met = 0;
    // the loop bounds are the same in every thread of the workgroup (barriers inside)
    for (uint32_t p0 = 0; p0 < passes; p0 += NPRE) {
        if (p0) request(p0);
        // provisional codes; pend[i]: which of the unit's values do not settle their code
        uint32_t pend[NPRE], at[NPRE];
#pragma unroll
        for (int i = 0; i < NPRE; ++i) {
            uint32_t t, part;
            pend[i] = 0;
            at[i] = 0;
            if (locate(p0 + i, t, part)) {
                const uint32_t m = tok0 + t;
                const float err = ev[i];
                if (WIDE) {
                    const uint32_t col = hd * (uint32_t)dh + part * 16u;
                    uint32_t w[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float4 x = v[i][j];
                        w[j] = quant1(x.x, inv) | quant1(x.y, inv) << 8 | quant1(x.z, inv) << 16 | quant1(x.w, inv) << 24;
                        pend[i] |= (code_uncertain(x.x, err, inv) ? 1u : 0u) << (4 * j) | (code_uncertain(x.y, err, inv) ? 2u : 0u) << (4 * j) |
                                   (code_uncertain(x.z, err, inv) ? 4u : 0u) << (4 * j) | (code_uncertain(x.w, err, inv) ? 8u : 0u) << (4 * j);
                    }
                    *(uint4 *)(xq + (int64_t)m * ldq + col) = make_uint4(w[0], w[1], w[2], w[3]);
                    at[i] = t * (uint32_t)dh + part * 16u;
                } else {
                    const uint32_t col = hd * (uint32_t)dh + part;
                    uint32_t code = 0;
                    if (col < (uint32_t)Hd) {
                        code = quant1(v[i][0].x, inv);
                        pend[i] = code_uncertain(v[i][0].x, err, inv) ? 1u : 0u;
                    }
                    xq[(int64_t)m * ldq + col] = (int8_t)code;   // pad columns: zero
                    at[i] = t * (uint32_t)dh + part;
                }
                if (bad) pend[i] = 0;
            }
        }
        // rounds: the pending values go on the list (as many as it holds), the workgroup serves the list
        bool again;
        do {
            __syncthreads();                                      // the list of the round before has been served
            if (tid == 0) { n_todo = 0; more = 0; }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NPRE; ++i) {
                while (pend[i]) {
                    const uint32_t slot = atomicAdd(&n_todo, 1u);
                    if (slot >= kList) { more = 1; break; }
                    const int e = __ffs((int)pend[i]) - 1;
                    pend[i] &= pend[i] - 1;
                    todo[slot] = at[i] + (uint32_t)e;
                }
            }
            __syncthreads();                                      // list complete, provisional codes stored
            const uint32_t n = n_todo < kList ? n_todo : kList;
            again = more != 0;
            met += n;
            // Sixteen listed values at a time: S^T = K Q^T on v_mfma_f64_16x16x4f64 as in attention_kernel, lane (c, g) holding, of
            // every 16-key tile, keys 4 r + g of value c's query.  A wave takes every fourth tile with a running maximum
            // of its own; the waves' sums meet at the end.
            const int c = lane & 15, g = lane >> 4;
            for (uint32_t k0 = 0; k0 < n; k0 += 16) {
                const uint32_t k = k0 + (uint32_t)c;
                const uint32_t e = todo[k < n ? k : k0];
                const uint32_t t = e / (uint32_t)dh, d = e - t * (uint32_t)dh;
                double q[16];                                 // dims 16 u + 4 g + i in q[4 u + i]
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int d0 = 16 * u + 4 * g;
                    const float4 x = *(const float4 *)(qb + (int64_t)t * ld + (d0 < dh ? d0 : 0));
                    q[4 * u] = d0 < dh ? (double)x.x : 0.0;
                    q[4 * u + 1] = d0 < dh ? (double)x.y : 0.0;
                    q[4 * u + 2] = d0 < dh ? (double)x.z : 0.0;
                    q[4 * u + 3] = d0 < dh ? (double)x.w : 0.0;
                }
                double m = -INFINITY, l = 0.0, o = 0.0;       // the wave's maximum, this lane's share of its sums
                for (int j0 = 0; j0 < S; j0 += kKeysLds) {    // one round up to 256 keys
                    const int nj = S - j0 < kKeysLds ? S - j0 : kKeysLds;
                    float vj[4][4];                           // the value column at the lane's keys
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int j = 16 * (wave + NW * kk) + 4 * r + g;
                            vj[kk][r] = vb[(int64_t)(j0 + (j < nj ? j : nj - 1)) * ld + d];
                        }
                    if (S > kKeysLds) {
                        __syncthreads();                      // the keys of the round before have been read
                        stage_keys(j0);
                        __syncthreads();
                    }
                    double sc[4][4], mx = -INFINITY;
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) {
                        const int tile = 16 * (wave + NW * kk);
                        v4d acc = {0.0, 0.0, 0.0, 0.0};
                        if (tile < nj) {                      // (uniform)
                            const float *row = &ks[(tile + c < nj ? tile + c : nj - 1) * kKeyRow + 4 * g];
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                const bool in = 16 * u + 4 * g < dh;
                                const float4 kv = *(const float4 *)(row + (in ? 16 * u : -4 * g));
                                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? (double)kv.x : 0.0, q[4 * u], acc, 0, 0, 0);
                                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? (double)kv.y : 0.0, q[4 * u + 1], acc, 0, 0, 0);
                                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? (double)kv.z : 0.0, q[4 * u + 2], acc, 0, 0, 0);
                                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? (double)kv.w : 0.0, q[4 * u + 3], acc, 0, 0, 0);
                            }
                        }
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            sc[kk][r] = tile + 4 * r + g < nj ? acc[r] * scale : -INFINITY;
                            mx = fmax(mx, sc[kk][r]);
                        }
                    }
                    mx = fmax(mx, lane_xor<16>(mx));
                    mx = fmax(mx, lane_xor<32>(mx));
                    const double mnew = fmax(m, mx);
                    if (mnew > -INFINITY) {                   // (a wave may have had no key yet)
                        const double corr = exp(m - mnew);    // 0 in the first round
                        l *= corr;
                        o *= corr;
                        m = mnew;
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const double pr = exp(sc[kk][r] - m);   // exp(-inf) = 0 for the keys beyond S
                                l += pr;
                                o += pr * (double)vj[kk][r];
                            }
                    }
                }
                l += lane_xor<16>(l);
                l += lane_xor<32>(l);
                o += lane_xor<16>(o);
                o += lane_xor<32>(o);
                if (g == 0) { red[wave][c][0] = m; red[wave][c][1] = l; red[wave][c][2] = o; }
                __syncthreads();
                if (tid < 16 && k < n) {
                    double top = red[0][c][0];
#pragma unroll
                    for (int w = 1; w < NW; ++w) top = fmax(top, red[w][c][0]);
                    double ls = 0.0, os = 0.0;
#pragma unroll
                    for (int w = 0; w < NW; ++w) {
                        const double f = exp(red[w][c][0] - top);
                        ls += red[w][c][1] * f;
                        os += red[w][c][2] * f;
                    }
                    xq[(int64_t)(tok0 + t) * ldq + hd * dh + d] = (int8_t)quant1((float)(os / ls), inv);
                }
                __syncthreads();                              // red is free
            }
        } while (again);
    }
    if (tid == 0 && unsure_total && met) atomicAdd(unsure_total, met);
}

static bool attn_aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Scratch of the approximate attention: an error bound per query of a head, then what its workgroups know about the exact
// maximum
static size_t attention_bounds_bytes(int32_t B, int32_t S, int32_t heads) { return align_up((size_t)B * heads * S * 4, 256); }
size_t attention_records_bytes(int32_t B, int32_t S, int32_t heads)
{
    return attention_bounds_bytes(B, S, heads) + align_up((size_t)B * heads * ((S + kSplitQ - 1) / kSplitQ) * sizeof(AttnCand), 256);
}

bool attention_splits(int32_t Hd, int32_t heads) { return ((Hd / heads) & 7) == 0 && (Hd & 3) == 0; }

// cands, bound_slot, exact_slot: null for the kernel alone
static hipError_t launch_attention_approx(const float *qkv, int32_t B, int32_t S, int32_t Hd, int32_t heads, float *ctx,
                                          float *err_q, AttnCand *cands, const uint32_t *max_slot, uint32_t *bound_slot,
                                          uint32_t *exact_slot, hipStream_t st)
{
    const int dh = Hd / heads;
    const int64_t grid = (int64_t)B * heads * ((S + kSplitQ - 1) / kSplitQ);
    return launch_k(EGERIA_KERNEL_ATTENTION, attention_split_kernel, dim3((unsigned)grid), dim3(256), 0, st,
                    qkv, (int)B, (int)S, (int)Hd, (int)heads, dh, (float)(1.0 / sqrt((double)dh)), ctx, err_q, cands,
                    max_slot, bound_slot, exact_slot);
}

// The largest |value| of a tensor into the words of a maximum slot, a workgroup per word (runs have it from the GEMM's epilogue).
__global__ __launch_bounds__(256) void tensor_max_kernel(const float *__restrict__ x, int64_t n, uint32_t *__restrict__ slot)
{
    __shared__ uint32_t sm[4];
    uint32_t m = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += kAmaxWays * 256) {
        const uint32_t a = abs_bits(x[i]);
        m = m > a ? m : a;
    }
    m = wave_max_u32(m);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) m = m > sm[w] ? m : sm[w];
        slot[blockIdx.x * kAmaxStride] = m;
    }
}

// Kernel 1 alone (benchmark instrumentation: its error against the fp64 kernel), on operands scaled as in a run: approximate
// context and the error bound E of every query of a head, fp32 [B, heads, S].  max_slot: scratch, a maximum slot.
hipError_t launch_attention_bounds(const float *qkv, int32_t B, int32_t S, int32_t Hd, int32_t heads, float *ctx,
                                   float *bounds, uint32_t *max_slot, hipStream_t st)
{
    const int dh = Hd / heads;
    const int64_t grid = (int64_t)B * heads * ((S + 63) / 64);
    if (grid <= 0) return hipSuccess;
    if (dh > kDh || !attention_splits(Hd, heads) || grid > 0x7ffffff0LL) return hipErrorInvalidValue;
    if (!attn_aligned16(qkv) || !attn_aligned16(ctx) || !attn_aligned16(bounds)) return hipErrorInvalidValue;
    const hipError_t e = launch_k(EGERIA_KERNEL_NONE, tensor_max_kernel, dim3(kAmaxWays), dim3(256), 0, st, qkv, (int64_t)B * S * 3 * Hd, max_slot);
    if (e != hipSuccess) return e;
    return launch_attention_approx(qkv, B, S, Hd, heads, ctx, bounds, nullptr, max_slot, nullptr, nullptr, st);
}

// The fp32 kernel, any head size: approximate context and a record per 64 queries of a head.
hipError_t launch_attention_fp32(const float *qkv, int32_t B, int32_t S, int32_t Hd, int32_t heads, float *ctx,
                                 void *records, hipStream_t st)
{
    const int dh = Hd / heads;
    const int64_t grid = (int64_t)B * heads * ((S + 63) / 64);
    if (grid <= 0) return hipSuccess;
    if (dh > kDh || grid > 0x7ffffff0LL) return hipErrorInvalidValue;
    if (!attn_aligned16(qkv) || !attn_aligned16(ctx) || !attn_aligned16(records)) return hipErrorInvalidValue;
    return launch_k(EGERIA_KERNEL_ATTENTION, attention_fast_kernel, dim3((unsigned)grid), dim3(256), 0, st, qkv,
                    (int)B, (int)S, (int)Hd, (int)heads, dh, (float)(1.0 / sqrt((double)dh)), ctx,
                    (AttnRecord *)records);
}

hipError_t launch_attention_certified(const float *qkv, int32_t B, int32_t S, int32_t Hd, int32_t heads, float *ctx,
                                      void *records, const uint32_t *max_slot, uint32_t *bound_slot, uint32_t *exact_slot,
                                      int8_t *xq, int64_t ldq, float *scale_out, uint32_t *flag, uint32_t *unsure_total,
                                      hipStream_t st)
{
    const int dh = Hd / heads;
    const int64_t nwg = (int64_t)B * heads * ((S + kSplitQ - 1) / kSplitQ), M = (int64_t)B * S;
    if (nwg <= 0) return hipSuccess;
    // what the kernels assume: heads of at most 64 dims in whole units of 8, 32-bit indices of the context's values, rows that
    // 16-byte vector accesses may touch
    if (dh > kDh || !attention_splits(Hd, heads) || nwg > 0x7ffffff0LL || M * Hd >= (1LL << 32) || ldq < Hd) return hipErrorInvalidValue;
    if (!attn_aligned16(qkv) || !attn_aligned16(ctx) || !attn_aligned16(xq) || !attn_aligned16(records)) return hipErrorInvalidValue;
    float *err_q = (float *)records;
    AttnCand *cands = (AttnCand *)((char *)records + attention_bounds_bytes(B, S, heads));
    const double scale = 1.0 / sqrt((double)dh);
    hipError_t e = launch_attention_approx(qkv, B, S, Hd, heads, ctx, err_q, cands, max_slot, bound_slot, exact_slot, st);
    if (e != hipSuccess) return e;
    e = launch_k(EGERIA_KERNEL_NONE, attention_settle_kernel, dim3((unsigned)((nwg + kSettleWorkgroups - 1) / kSettleWorkgroups)), dim3(256), 0, st,
                 qkv, (const AttnCand *)cands, (int)nwg, (const uint32_t *)bound_slot, (int)S, (int)Hd, (int)heads, dh, scale, exact_slot);
    if (e != hipSuccess) return e;
    const bool wide = (dh & 15) == 0 && (Hd & 15) == 0 && ldq == Hd;
    if ((int64_t)S * (dh + (ldq - Hd)) >= (1LL << 31)) return hipErrorInvalidValue;
    // a workgroup per head; heads are shared out where that leaves compute units idle (a workgroup's fixed part is half its
    // time, so shares of less than 64 tokens do not pay)
    const int64_t all_heads = (int64_t)B * heads;
    int64_t splits = 2 * compute_units() / all_heads;
    if (splits > (S + 63) / 64) splits = (S + 63) / 64;
    if (splits < 1) splits = 1;
    const int tokens = (int)((S + splits - 1) / splits);
    splits = (S + tokens - 1) / tokens;
    if (all_heads * splits > 0x7fffffffLL) return hipErrorInvalidValue;
    auto go = [&](auto kernel) {
        return launch_k(EGERIA_KERNEL_QUANTIZE, kernel, dim3((unsigned)(all_heads * splits)), dim3(kCertifyThreads), 0, st, qkv,
                        (const float *)ctx, (const float *)err_q, (int)S, (int)Hd, (int)heads, dh, (int)splits, tokens, scale,
                        (const uint32_t *)exact_slot, xq, ldq, scale_out, flag, unsure_total);
    };
    return wide ? go(quantize_attention_certify_kernel<true>) : go(quantize_attention_certify_kernel<false>);
}

hipError_t launch_attention(const float *qkv, int32_t B, int32_t S, int32_t Hd, int32_t heads,
                            float *ctx, uint32_t *absmax_out, hipStream_t st, uint16_t *ctx_half)
{
    const int dh = Hd / heads;
    constexpr int QB = 1;               // one 16-query block per wave: ~120 VGPRs, several waves per SIMD
    const int qtiles = (S + 64 * QB - 1) / (64 * QB);
    const int64_t grid = (int64_t)B * heads * qtiles;
    if (grid <= 0) return hipSuccess;
    if (dh > kDh || grid > 0x7ffffff0LL) return hipErrorInvalidValue;
    return launch_k(EGERIA_KERNEL_ATTENTION, attention_kernel<QB>, dim3((unsigned)grid), dim3(256), 0, st, qkv,
                    (int)B, (int)S, (int)Hd, (int)heads, dh, 1.0 / sqrt((double)dh), ctx, absmax_out, ctx_half);
}

}  // namespace egeria
