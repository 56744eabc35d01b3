// int8 x int8 -> int32 GEMM and implicit-GEMM 3x3 convolution on the gfx950
// matrix cores, with the dequantising epilogue fused (the reference model's
// linear and convolution layers, Section 4.1 of the paper).
//
//   acc[m, n] = sum_k a[m, k] * w[n, k]          (both operands K-contiguous)
//   y[m, n]   = act( fma((float)acc, sx*sw, bias[n]) [+ residual] )
//
// One workgroup of 4 (or, for the two largest tiles of big linear layers, 8)
// waves owns a BM x BN tile of the output (256x256 down to 128x32, chosen so
// that the grid still fills the chip).  Per K step of 64 or
// 128 bytes the tile's A and W rows go from global memory straight into a ring
// of LDS stages (buffer loads with the LDS modifier; 16-byte units, rotated by
// an exclusive-or of the row so that the 128-bit operand reads of a wave fall
// on distinct banks): while the matrix cores work on one stage the following
// steps are landing in the others, one barrier per step.  Each wave issues
// v_mfma_i32_32x32x32_i8: lane l supplies 16 consecutive K bytes of row
// (l % 32) at K offset 16 * (l / 32) for A and for W alike, so the product is
// exact whatever the instruction's internal K order is.  Workgroup ids are
// dealt so that each XCD works on a contiguous range of tiles (N fastest) and
// its L2 serves the re-reads of A rows and of the weights.
#include "gelu.hpp"
#include <climits>
#include <type_traits>

namespace egeria {

typedef int v16i __attribute__((ext_vector_type(16)));

// K bytes per step, BK: 128 (one 128-byte cache line of every row per request)
// or 64.  With 64-byte steps each line is fetched half now and half one step
// later; the stage is half as large, so more workgroups or stages fit a CU -
// but a request for half a line costs the L2 -> LDS path as much as one for a
// whole line (measured: 29 against 62 bytes per clock and compute unit), so the
// 64-byte shapes are bound by that path as soon as the matrix cores are fed
// well.  The eight-wave shapes take whole lines, two stages of them, and a
// tile large enough that one workgroup per compute unit keeps two waves on
// every SIMD.
// LDS stages: one being read, the others being filled.  (Three 64-byte stages of the row-owning 64x768 tile fill the 160 KB
// exactly; of 128-byte steps two stages bring as many bytes ahead.)
constexpr int stages_for(int bk) { return bk == 64 ? 3 : 2; }

typedef float v16f __attribute__((ext_vector_type(16)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

// Element type of the two operands (ET): 0 = int8 (int32 sums, the reference
// model's default), 1 = float16, 2 = float32 (fp32 sums; the reference model at
// the higher precisions of the paper's Table 2).  The kernel moves bytes: a
// 16-byte unit is 16, 8 or 4 values of K, and one unit pair per lane feeds one
// MFMA (int8, float16) or four (float32, one value each).
template <int ET>
struct AccOf {
    typedef v16i type;
};
template <>
struct AccOf<1> {
    typedef v16f type;
};
template <>
struct AccOf<2> {
    typedef v16f type;
};
template <int ET>
struct ResOf {
    typedef int8_t type;
};
template <>
struct ResOf<1> {
    typedef _Float16 type;
};
template <>
struct ResOf<2> {
    typedef float type;
};
template <int ET>
__device__ __forceinline__ typename AccOf<ET>::type mma(v4i a, v4i b, typename AccOf<ET>::type c)
{
    if constexpr (ET == 0) {
        return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
    } else if constexpr (ET == 1) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(__int_as_float(a[e]), __int_as_float(b[e]), c, 0, 0, 0);
        return c;
    }
}
__device__ __forceinline__ int32_t acc_bits(int a) { return a; }
__device__ __forceinline__ int32_t acc_bits(float a) { return __float_as_int(a); }

// Workgroups of a tile shape that are meant to share a CU (one wave of each per
// SIMD): the register allocation is held to 512 / that many registers per lane,
// so that one workgroup's epilogue overlaps another's K loop.
constexpr int resident_target(int bm, int bn)
{
    return bm * bn > 256 * 128 ? 1 : (bm * bn > 128 * 128 ? 2 : 3);
}

// What a workgroup does with its sums (EPI)
enum GemmEpilogue {
    kStore = 0,          // y, int8 codes, maxima, observation points
    kLayerNorm = 1,      // the layer norm of its rows (GemmArgs::ln_out)
    kGeluMax = 2,        // nothing but their maximum (gelu_pass 1)
    kGeluCodes = 3       // int8 codes of their GELU (gelu_pass 2)
};
constexpr int kGeluTableBytes = kGeluLines * 8;
// Values of a wave (1024 to 8192 by the tile) that the lines may leave open: a list of 8 bytes each in the stage memory.
constexpr int kGeluList = 512;
// The lines' error in codes from which on the epilogue takes the cubic pieces instead (largest |gelu| below 6 x 10^-3).  The lines
// leave twice that share of the values open, 4 %: the list still holds them, of the largest tile one value in sixteen.  An
// encoder layer, us, lines / pieces, largest |gelu| 8.5 x 10^-3: 151 / 159 (32 x 128 x 768), 475 / 476 (64 x 256), 186 / 195 (24 x 197);
// 3.4 x 10^-3, 7 % left open and, but for the first, lists that overflow: 154 / 159, 524 / 482, 208 / 197.
constexpr float kGeluLinesOpen = 0.02f;

template <int BM, int BN, int WM, int WN, bool CONV, int BK, int ET, int EPI = kStore, int NST = stages_for(BK)>
__global__ __launch_bounds__(64 * WM * WN, EPI == kGeluCodes && BM * BN <= 128 * 128 ? 2 : resident_target(BM, BN)) void gemm_i8_kernel(const GemmArgs g)
{
    typedef typename AccOf<ET>::type acc_t;
    typedef typename ResOf<ET>::type res_t;
    constexpr bool LNF = EPI == kLayerNorm;
    constexpr bool kTurned = EPI == kGeluCodes;      // the transposed product: a lane holds neighbouring columns of one row
    static_assert(BK == 64 || BK == 128, "K step of 64 or 128 bytes");
    constexpr int kBK = BK;
    constexpr int UPR = BK / 16;                 // 16-byte K units per row of a stage
    constexpr int kRowsPerChunk = 64 / UPR;      // rows one load instruction of a wave covers
    constexpr int SWR = 16 / UPR;                // rows that share a rotation of the K units
    constexpr int NSUB = BK / 32;                // 32-byte sub-steps (one MFMA deep) per step
    constexpr int NW = WM * WN, NT = 64 * NW;          // waves and threads per workgroup
    static_assert(NW == 4 || NW == 8, "four or eight waves per workgroup");
    static_assert(BM % kRowsPerChunk == 0 && BN % kRowsPerChunk == 0, "tiles are made of whole chunks");
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int A_CH = BM / kRowsPerChunk, B_CH = BN / kRowsPerChunk; // 1-KiB chunks per K step
    constexpr int A_IT = (A_CH + NW - 1) / NW, B_IT = (B_CH + NW - 1) / NW;         // chunks per wave
    constexpr int STAGE = (BM + BN) * kBK;
    constexpr int NLD = A_IT + B_IT;                                    // loads per wave and K step
    static_assert((NST - 2) * NLD < 64, "outstanding loads must fit the wait counter");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];       // [NST][BM + BN][BK]

    const int tile = (int)xcd_piece(blockIdx.x, gridDim.x);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int wm = wave / WN, wn = wave % WN;
    const int tiles_n = (g.N + BN - 1) / BN;
    const int64_t tile_m = tile / tiles_n;
    const int tile_n = tile % tiles_n;
    const int64_t m0 = tile_m * BM;
    const int n0 = tile_n * BN;
    // epilogue scalars, requested now so that their latency hides behind the K loop
    const float sxv = *g.sx;
    const float s = g.sw_per_n ? 0.0f : sxv * (*g.sw);
    const float rs = g.res_q ? (ET == 0 ? *g.res_scale : 1.0f) : 0.0f;
    float q_inv = 0.0f;                          // multiplier of the optional int8 output
    if constexpr (EPI == kStore) {               // (GELU passes have codes without a static scale)
        if (g.q_out) q_inv = (float)(1.0 / (double)*g.q_scale);
    }
    // affine activation codes: stored codes are q - 128, so 128 - zero point goes back in
    const int zmul = (ET == 0 && g.zp_in) ? 128 - *g.zp_in : 0;
    const int rmul = (ET == 0 && g.zp_res) ? 128 - *g.zp_res : 0;

    // Operands go from global memory straight into LDS (buffer loads with the
    // LDS modifier): one such instruction of a wave fills 1 KiB, lane l writing
    // bytes [16 l, 16 l + 16) of it, i.e. unit l % UPR of row l / UPR of a chunk
    // of 64 / UPR rows (UPR = BK / 16 units per row).  Which 16 bytes of K a
    // lane fetches for that slot is free, so the K units of row r are stored
    // rotated by (r / (16 / UPR)) % UPR (exclusive-or): the 128-bit operand
    // reads of 16 consecutive rows then fall on 16 distinct bank groups.  A lane whose row or K offset
    // is out of range is given an offset beyond the buffer and writes zeros.
    constexpr uint32_t kOob = 0x80000000u;
    auto descriptor = [](const void *p, int64_t bytes) {             // raw buffer: base, no stride, extent, dword format
        const uint64_t a = (uint64_t)p;
        v4i d;
        d[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
        d[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32) & 0xffff);
        d[2] = __builtin_amdgcn_readfirstlane((int)bytes);
        d[3] = 0x00020000;
        return d;
    };
    const v4i rsrc_a = descriptor(g.a, g.a_bytes), rsrc_w = descriptor(g.w, g.w_bytes);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte *)lds;      // LDS address of the stage array
    const int rloc = lane / UPR;                                 // row within the chunk
    // K unit this lane fetches: slot ^ ((row / SWR) % UPR) with row = chunk * (64 / UPR) + rloc and
    // chunk = wave + NW * it; the chunk's share of that is (chunk * 4) % UPR = (wave % 2) * 4 % UPR
    const int unit = (lane % UPR) ^ (((wave_u & 1) * 4 + rloc / SWR) % UPR);
    static_assert(A_CH % 2 == 0 && B_CH % 2 == 0, "a wave's chunks must keep their parity");
    // Byte offset of the lane's row of each chunk (linear) or of its centre pixel (conv).  A row that does not exist starts
    // beyond the buffer, and the K offset is added with saturation, so it stays there: a linear request is one addition.
    uint32_t a_base[A_IT];
    uint32_t a_taps[CONV ? A_IT : 1];            // conv: bit t set if window position t of the pixel lies inside the image
#pragma unroll
    for (int it = 0; it < A_IT; ++it) {
        const int r = ((wave_u + it * NW) % A_CH) * kRowsPerChunk + rloc;
        const int64_t m = m0 + r;
        const bool ok = m < g.M;
        a_base[it] = ok ? (uint32_t)(m * (CONV ? (int64_t)g.cp : g.lda)) : (CONV ? 0u : kOob);
        if constexpr (CONV) {
            // the operand's extent is below 2^31 bytes, so m fits 32 bits (a 64-bit division is a long call)
            const uint32_t mrow = (uint32_t)m / (uint32_t)g.W;
            const int ow = (int)((uint32_t)m - mrow * (uint32_t)g.W), oh = (int)(mrow % (uint32_t)g.H);
            const uint32_t cols = (ow > 0 ? 1u : 0u) | 2u | (ow + 1 < g.W ? 4u : 0u);
            a_taps[it] = !ok ? 0u : (oh > 0 ? cols : 0u) | cols << 3 | (oh + 1 < g.H ? cols << 6 : 0u);
        }
    }
    uint32_t b_base[B_IT];
#pragma unroll
    for (int it = 0; it < B_IT; ++it) {
        const int r = ((wave_u + it * NW) % B_CH) * kRowsPerChunk + rloc;
        b_base[it] = n0 + r < g.N ? (uint32_t)(n0 + r) * (uint32_t)g.kp : kOob;
    }

    // Requests for K step kt into LDS stage `stage`, one 1-KiB chunk per call
    // (idx < A_IT: a chunk of A, else of W).  Every wave issues exactly NLD loads
    // per K step (the waits below count them): where a tile has fewer chunks
    // than that, waves fetch a chunk twice, writing the same bytes.
    struct StepAddr {
        uint32_t k;              // the lane's K offset of the step, beyond any buffer past the end of K
        uint32_t delta, tap;     // conv: what it adds to a centre pixel's offset, and the bit of its window position
    };
    // The row-owning tile: every workgroup streams the whole weight matrix, so all of them would ask the L2 for
    // the same rows at the same time; each starts at a K step of its own instead (integer sums do not depend
    // on the order).  Steps past the end of K stay past the end.
    const int nk_all = (g.kp + kBK - 1) / kBK;
    const int k_rot = LNF ? tile % nk_all : 0;
    // conv, pixels of a K step and more (cp >= BK): the steps come in order, so the window position of a step's first byte
    // (tap_s, which ends at K offset tap_end) is followed with scalars and a lane is at that position or the next one.  Per
    // lane and step a division took some 60 vector instructions and the border tests 8 per request, a thousand clocks of a
    // step whose MFMAs take 130 to 260 (2450 x 512 x 4608, 128x64
    // tiles: 30 -> 22.6 us).
    int tap_s = 0, tap_end = g.cp;
    auto tap_offset = [&](int tap) {             // K offset -> offset from the centre pixel, at window position tap
        const int kh = (tap >= 3 ? 1 : 0) + (tap >= 6 ? 1 : 0);
        return (uint32_t)((((kh - 1) * g.W + (tap - 3 * kh - 1)) - tap) * g.cp);
    };
    auto step_addr = [&](int kt) {
        StepAddr sa;
        if (LNF && kt < nk_all) kt = kt + k_rot < nk_all ? kt + k_rot : kt + k_rot - nk_all;
        const int k0 = kt * kBK + unit * 16;
        const bool k_ok = k0 < g.kp;
        sa.k = k_ok ? (uint32_t)k0 : kOob;
        sa.delta = 0;
        sa.tap = 0;
        if constexpr (CONV) {
            if (g.cp >= kBK) {
                if (kt * kBK >= tap_end) { ++tap_s; tap_end += g.cp; }
                const bool next = k0 >= tap_end;
                sa.delta = (uint32_t)k0 + (next ? tap_offset(tap_s + 1) : tap_offset(tap_s));
                sa.tap = next ? 2u << tap_s : 1u << tap_s;
            } else {
                int tap = 0;                     // k0 / cp, by counting
#pragma unroll
                for (int i = 1; i < 9; ++i) tap += k0 >= i * g.cp ? 1 : 0;
                sa.delta = (uint32_t)k0 + tap_offset(tap);
                sa.tap = 1u << tap;
            }
            sa.tap = k_ok ? sa.tap : 0u;
        }
        return sa;
    };
    auto fetch_one = [&](const StepAddr &sa, int stage, int idx) {
        const uint32_t sA = lds0 + stage * STAGE, sB = sA + BM * kBK;
        if (idx < A_IT) {
            const int it = idx;
            const int chunk = (wave_u + it * NW) % A_CH;
            uint32_t at;
            if constexpr (CONV) at = (a_taps[it] & sa.tap) ? a_base[it] + sa.delta : kOob;
            else at = __builtin_elementwise_add_sat(a_base[it], sa.k);
            load_to_lds_b128(rsrc_a, sA + chunk * 1024, at);
        } else {
            const int it = idx - A_IT;
            const int chunk = (wave_u + it * NW) % B_CH;
            load_to_lds_b128(rsrc_w, sB + chunk * 1024, __builtin_elementwise_add_sat(b_base[it], sa.k));
        }
    };
    auto fetch = [&](int kt, int stage) {
        const StepAddr sa = step_addr(kt);
#pragma unroll
        for (int idx = 0; idx < A_IT + B_IT; ++idx) fetch_one(sa, stage, idx);
    };
    // operand fragments of one 32-byte K sub-step ks: lane l supplies row l % 32, K unit 2 ks + l / 32
    const int frow = lane & 31;
    const int fsw = (frow / SWR) % UPR;
    auto read_frags = [&](int stage, int ks, v4i (&fa)[TM], v4i (&fb)[TN]) {
        const uint8_t *sA = lds + stage * STAGE, *sB = sA + BM * kBK;
        const int koff = ((ks * 2 + (lane >> 5)) ^ fsw) * 16;
#pragma unroll
        for (int i = 0; i < TM; ++i)
            fa[i] = *(const v4i *)&sA[((wm * TM + i) * 32 + frow) * kBK + koff];
#pragma unroll
        for (int j = 0; j < TN; ++j)
            fb[j] = *(const v4i *)&sB[((wn * TN + j) * 32 + frow) * kBK + koff];
    };

    acc_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
    auto mfma_all = [&](const v4i (&fa)[TM], const v4i (&fb)[TN]) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = kTurned ? mma<ET>(fb[j], fa[i], acc[i][j]) : mma<ET>(fa[i], fb[j], acc[i][j]);
    };

    // Software pipeline over a ring of NST LDS stages.  During step kt the
    // matrix cores work on stage kt % NST, K steps kt + 1 .. kt + NST - 2 are
    // landing in the following stages and K step kt + NST - 1 is requested into
    // the stage that step kt - 1 read (every wave has passed the barrier that
    // ended that step).  One barrier per step; a step is two or four 32-byte
    // sub-steps whose operand fragments are double-buffered in registers.
    constexpr int NMF = TM * TN;                 // MFMAs per sub-step
    constexpr int NRD = TM + TN;                 // LDS operand reads per sub-step
    constexpr int kWaitNext = 0x0f70 | (((NST - 2) * NLD) & 0xf) | ((((NST - 2) * NLD) >> 4) << 14);   // vmcnt only
    const int nk = (g.kp + kBK - 1) / kBK;
    v4i fa0[TM], fb0[TN], fa1[TM], fb1[TN];
    if constexpr (EPI == kGeluCodes) {
        // the maximum's words (a way's word per lane, into the stage that is filled last) and the wave's part of the GELU's lines
        static_assert(STAGE >= NW * 1024 && kGeluTableBytes % (4 * 1024) == 0, "a kilobyte per wave, and per request");
        load_to_lds_b128((const uint8_t *)(g.gelu_max + lane * kAmaxStride), lds0 + (NST - 1) * STAGE + wave_u * 1024);
#pragma unroll
        for (int c = 0; c < kGeluTableBytes / 1024 / 4; ++c) {
            const int at = ((wave_u & 3) + 4 * c) * 1024;           // (of eight waves the second four ask for the same)
            load_to_lds_b128((const uint8_t *)kGeluLine + at + lane * 16, lds0 + NST * STAGE + at);
        }
    }
#pragma unroll
    for (int p = 0; p < NST - 1; ++p) fetch(p, p);
    // the scale of the codes, worked out while the first K steps are on their way
    float gelu_vm = 0.0f, gelu_inv = 0.0f;
    if constexpr (EPI == kGeluCodes) {
        __builtin_amdgcn_s_waitcnt(0x0f70 | (((NST - 1) * NLD) & 0xf) | ((((NST - 1) * NLD) >> 4) << 14));
        wave_lds_turn();
        gelu_vm = __uint_as_float(wave_max_u32(*(const uint32_t *)&lds[(NST - 1) * STAGE + wave_u * 1024 + lane * 16]));
        float absmax = gelu_exact(gelu_vm);
        if (gelu_vm < kGeluShortcutMin) {            // uniform, rare
            const uint32_t *way = g.gelu_neg + lane * kAmaxStride;
            const uint32_t below = wave_max_u32(way[0]), above = wave_max_u32(way[1]);
            if (below) absmax = fmaxf(absmax, fabsf(gelu_exact(-__uint_as_float(0x7fffffffu - below))));
            if (above) absmax = fmaxf(absmax, fabsf(gelu_exact(-__uint_as_float(above))));
            if (above > 0x7f800000u) absmax = __uint_as_float(above);    // a NaN among them: no scale is left
        }
        float scale;
        const bool bad = !(gelu_vm <= 3.402823466e+38f);
        gelu_inv = gelu_code_scale(absmax, bad, &scale);
        if (tile == 0 && tid == 0) publish(scale, bad, g.gelu_scale, nullptr, g.flag);
    }
    // which form the epilogue takes: decided while the first K steps are on their way
    int inside = EPI == kStore && m0 + BM <= g.M && n0 + BN <= g.N && !g.acc_out && !g.zp_in && g.ldy < (1 << 20) && g.q_ld < (1 << 20) &&
                 (ET == 0 && BM * BN <= 128 * 128 ? (g.q_out ? g.act == 1 && !g.res_q : g.y != nullptr) : g.y && !g.q_out && !g.res_q);
    inside = __builtin_amdgcn_readfirstlane(inside);
    asm volatile("" : "+s"(inside));
    __builtin_amdgcn_s_waitcnt(kWaitNext);       // K step 0 landed
    __syncthreads();
    read_frags(0, 0, fa0, fb0);
    auto hint = [&]() {                           // one LDS read after each of the first MFMAs
#pragma unroll
        for (int i = 0; i < NMF; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (i < NRD) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
    };
    int st = 0;                                  // stage of K step kt
    for (int kt = 0; kt < nk; ++kt) {            // past the end of K the loads return zeros
        const int st1 = st == NST - 1 ? 0 : st + 1, stl = st == 0 ? NST - 1 : st - 1;
        read_frags(st, 1, fa1, fb1);
        const StepAddr sa = step_addr(kt + NST - 1);
        // the step's requests are spread between its first MFMAs: a burst of them
        // would fill the memory pipeline's queue and stall the wave's MFMA issue
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                acc[i][j] = kTurned ? mma<ET>(fb0[j], fa0[i], acc[i][j]) : mma<ET>(fa0[i], fb0[j], acc[i][j]);
                constexpr int per = (NLD + NMF - 1) / NMF;               // requests after each MFMA
#pragma unroll
                for (int q = 0; q < per; ++q)
                    if ((i * TN + j) * per + q < NLD) fetch_one(sa, stl, (i * TN + j) * per + q);
                if ((i * TN + j) * per < NLD) __builtin_amdgcn_sched_barrier(0);   // keep the MFMA before its requests
            }
        if (NSUB == 4) {
            read_frags(st, 2, fa0, fb0);
            mfma_all(fa1, fb1);
            hint();
            read_frags(st, 3, fa1, fb1);
            mfma_all(fa0, fb0);
            hint();
        }
        __builtin_amdgcn_s_waitcnt(kWaitNext);   // K step kt + 1 landed
        __syncthreads();
        read_frags(st1, 0, fa0, fb0);
        mfma_all(fa1, fb1);
        hint();
        st = st1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the zero-filled K steps past the end

    const int lcol = lane & 31, lrow = (lane >> 5) * 4;
    const int wm_u = __builtin_amdgcn_readfirstlane(wm), wn_u = __builtin_amdgcn_readfirstlane(wn);
    // Running maximum for the next quantiser, kept as a bit pattern so that a
    // NaN or an infinity stays visible.  Non-negative values (after ReLU, or
    // when only positive values are wanted) order like signed integers.
    int32_t amax = 0;
    if constexpr (LNF) {
        // The layer norm of the rows in the same launch: the workgroup owns whole rows (one tile across N).
        // A 32-row block of the fp32 output goes to LDS (the stage memory is free now), then each wave
        // normalises rows of it exactly as layernorm_vec_kernel does with a stored tensor: lane l holds the
        // 16-byte units l, l + 64, ... of the row, and the arithmetic is the shared ln_row_vec.  The residual
        // rows are requested before the barrier, gamma and beta once.
        static_assert(WM == 1 && ET == 0 && !CONV, "whole rows of a linear layer with int8 operands");
        constexpr int YS = BN + 8;                      // floats per row of the block in LDS (pad: the two rows a
                                                        // store instruction writes fall into different banks)
        constexpr int NV = BN / 256, RPW = 32 / NW;     // 16-byte units per lane and row; rows per wave and block
        static_assert(BN % 256 == 0 && 32 % NW == 0, "rows of 256 NV floats, a wave takes whole rows");
        static_assert((size_t)NST * STAGE >= (size_t)32 * YS * 4, "a 32-row block must fit the stage memory");
        float *yt = (float *)lds;
        const int H = g.N, nv = H >> 2;
        const __amdgpu_buffer_rsrc_t rln = __builtin_amdgcn_make_buffer_rsrc((void *)(g.ln_out + m0 * H), 0, BM * H * 4, kBufferWord);
        const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f), one4 = make_float4(1.f, 1.f, 1.f, 1.f);
        float4 gmv[NV], btv[NV];
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int c = lane + 64 * u, cc = c < nv ? c : nv - 1;
            gmv[u] = g.ln_gamma ? reinterpret_cast<const float4 *>(g.ln_gamma)[cc] : one4;
            btv[u] = g.ln_beta ? reinterpret_cast<const float4 *>(g.ln_beta)[cc] : zero4;
        }
        uint32_t amax_u = 0;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            __syncthreads();                            // the stage memory (or the block before) has been read
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int col = (wn_u * TN + j) * 32 + lcol;
                const bool col_ok = col < g.N;
                const float bj = (g.bias && col_ok) ? g.bias[col] : 0.0f;
                const float sj = g.sw_per_n ? (col_ok ? sxv * g.sw[col] : 0.0f) : s;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    yt[(lrow + 8 * (r >> 2) + (r & 3)) * YS + col] = fmaf((float)acc[i][j][r], sj, bj);
            }
            float4 rv[RPW][NV];
#pragma unroll
            for (int k = 0; k < RPW; ++k) {
                const int64_t row = m0 + i * 32 + wave_u + NW * k;
                const float4 *rr = reinterpret_cast<const float4 *>(g.ln_res + (row < g.M ? row : g.M - 1) * H);
#pragma unroll
                for (int u = 0; u < NV; ++u) {
                    const int c = lane + 64 * u;
                    rv[k][u] = rr[c < nv ? c : nv - 1];
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < RPW; ++k) {
                const int lr = wave_u + NW * k;
                const int64_t row = m0 + i * 32 + lr;
                if (row < g.M) {
                    float4 xv[NV], o[NV];
#pragma unroll
                    for (int u = 0; u < NV; ++u) {
                        const int c = lane + 64 * u;
                        const bool in = c < nv;
                        xv[u] = in ? *reinterpret_cast<const float4 *>(&yt[lr * YS + 4 * c]) : zero4;
                        if (!in) rv[k][u] = zero4;
                    }
                    ln_row_vec<NV>(xv, rv[k], gmv, btv, lane, nv, H, g.ln_eps, o, amax_u);
#pragma unroll
                    for (int u = 0; u < NV; ++u) {
                        const int c = lane + 64 * u;
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, o[u]), rln, (int)(c < nv ? (uint32_t)(i * 32 + lr) * (uint32_t)H * 4u + (uint32_t)c * 16u : kOob), 0, kThrough);
                    }
                }
            }
        }
        amax = (int32_t)amax_u;
    } else if constexpr (EPI == kGeluMax) {
        // ---- nothing is stored.  y = fma(sum, s, b) grows (or falls) with the sum, so a column's largest y is that of its largest
        // or its smallest sum.
        float sj[TN], bj[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = n0 + (wn_u * TN + j) * 32 + lcol;
            const bool ok = col < g.N;
            sj[j] = !ok ? 0.0f : (g.sw_per_n ? sxv * g.sw[ok ? col : 0] : s);    // one fp32 multiply
            bj[j] = g.bias && ok ? g.bias[ok ? col : 0] : 0.0f;
        }
        const int rows = (int)(g.M - m0 < BM ? g.M - m0 : BM);                   // valid rows of the tile
        uint32_t worst = 0;                                                      // largest |y| of the two: not finite if any y is not
        auto track = [&](float v) {
            const int32_t bits = (int32_t)__float_as_uint(v);
            amax = amax > bits ? amax : bits;
            worst = worst > abs_bits(v) ? worst : abs_bits(v);
        };
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            int hi = INT_MIN, lo = INT_MAX;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int left = rows - (wm_u * TM + i) * 32;                    // (uniform)
                if (left >= 32) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        hi = hi > acc[i][j][r] ? hi : acc[i][j][r];
                        lo = lo < acc[i][j][r] ? lo : acc[i][j][r];
                    }
                } else if (left > 0) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const bool ok = lrow + 8 * (r >> 2) + (r & 3) < left;
                        const int up = ok ? acc[i][j][r] : INT_MIN, down = ok ? acc[i][j][r] : INT_MAX;
                        hi = hi > up ? hi : up;
                        lo = lo < down ? lo : down;
                    }
                }
            }
            if (lo <= hi) {                             // (a lane may have no row at all)
                track(fmaf((float)hi, sj[j], bj[j]));
                track(fmaf((float)lo, sj[j], bj[j]));
            }
        }
        // (a wave beyond the last row or column has no values)
        if (__builtin_expect(__uint_as_float(wave_max_u32((uint32_t)amax)) < kGeluShortcutMin && wm_u * TM * 32 < rows && n0 + wn_u * TN * 32 < g.N, 0)) {
            uint32_t below = 0, above = 0;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const float v = (wm_u * TM + i) * 32 + lrow + 8 * (r >> 2) + (r & 3) < rows ? fmaf((float)acc[i][j][r], sj[j], bj[j]) : 0.0f;
                        const uint32_t a = abs_bits(v);
                        if (v <= kGeluArgMin) below = below > 0x7fffffffu - a ? below : 0x7fffffffu - a;
                        if (v >= kGeluArgMin && v < 0.0f) above = above > a ? above : a;
                    }
            if (worst >= 0x7f800000u) above = 0x7fc00000u;                              // -infinity, NaN: a NaN
            below = wave_max_u32(below);
            above = wave_max_u32(above);
            uint32_t *way = g.gelu_neg + (blockIdx.x & (kAmaxWays - 1)) * kAmaxStride;
            if (lane == 0 && below) atomicMax(way, below);
            if (lane == 0 && above) atomicMax(way + 1, above);
        }
    } else if constexpr (EPI == kGeluCodes) {
        // ---- codes of gelu(y).  The product is the transposed one, so a lane holds, of every 32x32 block, 16 columns of one row: four
        // times four neighbouring ones, the other half of the wave those between them.  A swap of halves makes 16 neighbours, one
        // store.  Values whose code the lines leave open go on the wave's list (value, place) in the stage memory and
        // are settled side by side afterwards; where they are too many, the cubic pieces leave a thirteenth of them open.  Bound by
        // the vector instructions, 13 a value (16384 x 3072 values: 69 us the launch, 38 the sums alone), about 30 with the
        // pieces.  An encoder layer with its first feed-forward weights times 1 / 10^-3 / 10^-6, us: 64 x 256 x 768 429 / 484 / 550 (fp32
        // tensor and row quantiser 496 / 589 / 676), 32 x 128 x 768 153 / 161 / 177 (171 / 181 / 203).  What is rare is out of line and
        // short (a loop over quarters of a block): cold instructions count, 32 x 128 x 768 178.4 us a step with sixteen values of the
        // pieces unrolled, 177.7 this way.
        static_assert((size_t)NST * STAGE >= (size_t)NW * (kGeluList * 8 + 4096), "the waves' lists must fit the stage memory");
        float2 *lines = (float2 *)&lds[NST * STAGE];
        uint2 *list = (uint2 *)&lds[(uint32_t)wave_u * (uint32_t)((size_t)NST * STAGE / NW)];
        const float room = 0.5f - kGeluLineErr * gelu_inv;
        const int rows = (int)(g.M - m0 < BM ? g.M - m0 : BM);
        const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc((void *)(g.q_out + m0 * g.q_ld), 0, (int)(rows * g.q_ld), 0x00020000);
        const uint32_t q_ld = (uint32_t)g.q_ld;
        const int half = lane >> 5;
#pragma unroll
        for (int c = tid; c < kGeluLines; c += NT) lines[c] = make_float2(lines[c].x * gelu_inv, lines[c].y * gelu_inv);
        __syncthreads();                                // every wave has read its last operands
        // COLS: a scale or a bias per column.  Pad columns are values of 0, settled like the others: the line around 0 is not 0 there.
        auto run = [&](auto cols_c) {
            constexpr bool COLS = decltype(cols_c)::value;
            int n = 0;
            {
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int col0 = n0 + (wn_u * TN + j) * 32;      // register r: column col0 + 8 (r / 4) + 4 half + r % 4
                    float sr[COLS ? 16 : 1], br[COLS ? 16 : 1];
                    sr[0] = s;
                    br[0] = 0.0f;
                    if constexpr (COLS) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int col = col0 + 8 * (r >> 2) + 4 * half + (r & 3), cc = col < g.N ? col : g.N - 1;
                            const float sv = g.sw_per_n ? sxv * g.sw[cc] : s, bv = g.bias ? g.bias[cc] : 0.0f;   // one fp32 multiply
                            sr[r] = col < g.N ? sv : 0.0f;
                            br[r] = col < g.N ? bv : 0.0f;
                        }
                    }
                    const uint32_t c16 = (uint32_t)(col0 + 16 * half) < q_ld ? (uint32_t)(col0 + 16 * half) : kOob;
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        const uint32_t row = (uint32_t)((wm_u * TM + i) * 32 + lcol);    // the lane's row of the tile
                        uint32_t c[16];
                        bool un[16], any = false;
                        auto value = [&](int r) { return fmaf((float)acc[i][j][r], sr[COLS ? r : 0], br[COLS ? r : 0]); };
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            c[r] = quant_gelu_lines(value(r), room, lines, &un[r]);
                            any = any || un[r];
                            if (r == 7) __builtin_amdgcn_sched_barrier(0);               // (sixteen look-ups in flight would spill)
                        }
                        uint32_t w[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) w[q] = pack_bytes(c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]);
                        const auto a = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false), b = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
                        const v4u out = {(unsigned)a[0], (unsigned)a[1], (unsigned)b[0], (unsigned)b[1]};
                        __builtin_amdgcn_raw_buffer_store_b128(out, rq, (int)(c16 == kOob ? kOob : row * q_ld + c16), 0, kThrough);
                        if (__builtin_expect(__ballot(any) != 0, 0)) {
                            float *turn = (float *)(list + kGeluList);       // the block's values, by register and lane
                            uint32_t open = 0;
#pragma unroll
                            for (int r = 0; r < 16; ++r) {
                                turn[r * 64 + lane] = value(r);
                                open |= un[r] ? 1u << r : 0u;
                            }
                            if ((int)row >= rows) open = 0;
                            wave_lds_turn();
#pragma unroll 1
                            while (__ballot(open != 0)) {
                                const int r = __ffs((int)open) - 1, col = col0 + 8 * (r >> 2) + 4 * half + (r & 3);
                                const bool mine = open != 0 && (uint32_t)col < q_ld;
                                const uint64_t m = __ballot(mine);
                                const int at = n + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                                if (mine && at < kGeluList) list[at] = make_uint2(__float_as_uint(turn[r * 64 + lane]), row * q_ld + (uint32_t)col);
                                n += __popcll(m);
                                open &= open - 1;
                            }
                            wave_lds_turn();
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            return n;
        };
        int n = __builtin_amdgcn_readfirstlane(kGeluLineErr * gelu_inv < kGeluLinesOpen ? 0 : kGeluList + 1);
        if (__builtin_expect(n == 0, 1)) n = g.sw_per_n || g.bias ? run(std::true_type{}) : run(std::false_type{});
        if (n == 0) return;                             // (uniform)
        wave_lds_turn();
        __builtin_amdgcn_s_waitcnt(0x0f70);             // the stores above have been performed
        if (__builtin_expect(n <= kGeluList, 1)) {
#pragma unroll 1
            for (int k = lane; k < n; k += 64) {
                const uint2 e = list[k];
                __builtin_amdgcn_raw_buffer_store_b8((uint8_t)settle_gelu(__uint_as_float(e.x), gelu_inv), rq, (int)e.y, 0, 0);
            }
            return;
        }
        // Too many for the list (values on the border of two codes), or lines too coarse for the tensor's scale: every block from
        // its sums with the cubic pieces.  As many blocks at a time as the wave's stage memory holds beside the pieces go there first, so that one
        // loop can take them in turn (the fp64 form's registers beside all of the sums would spill).
        constexpr int kSpan = (int)((size_t)NST * STAGE / NW), kGroup = (kSpan - 4096) / 4096 < TM * TN ? (kSpan - 4096) / 4096 : TM * TN;
        static_assert(kGroup >= 1, "a block's sums and the cubic pieces must fit a wave's share of the stage memory");
        float4 *tab = (float4 *)list;
        int *turn = (int *)(list + kGeluList);
#pragma unroll
        for (int k = 0; k < 4; ++k) tab[lane + 64 * k] = scale_gelu_entry(kGeluTable[lane + 64 * k], gelu_inv);
        const float room3 = 0.5f - kGeluErrAbs * gelu_inv;
        const __amdgpu_buffer_rsrc_t rsw = __builtin_amdgcn_make_buffer_rsrc((void *)g.sw, 0, g.sw_per_n ? g.N * 4 : 0, kBufferWord);
        const __amdgpu_buffer_rsrc_t rbias = __builtin_amdgcn_make_buffer_rsrc((void *)g.bias, 0, g.bias ? g.N * 4 : 0, kBufferWord);
#pragma unroll
        for (int b0 = 0; b0 < TM * TN; b0 += kGroup) {
            wave_lds_turn();
#pragma unroll
            for (int k = 0; k < kGroup; ++k)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (b0 + k < TM * TN) turn[k * 1024 + r * 64 + lane] = acc[(b0 + k) % TM][(b0 + k) / TM][r];
            wave_lds_turn();
#pragma unroll 1
            for (int b = b0; b < b0 + kGroup && b < TM * TN; ++b) {
                int *mine = turn + (b - b0) * 1024 + lane;
                const int col0 = n0 + (wn_u * TN + b / TM) * 32;
                const uint32_t row = (uint32_t)((wm_u * TM + b % TM) * 32 + lcol);
                const uint32_t c16 = (uint32_t)(col0 + 16 * half) < q_ld ? (uint32_t)(col0 + 16 * half) : kOob;
                uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll 1
                for (int q = 0; q < 4; ++q) {
                    const int at = (col0 + 8 * q + 4 * half) * 4;              // (beyond N the loads are 0)
                    uint32_t code[4], open = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float sw = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsw, at, 4 * e, 0));
                        const float bv = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rbias, at, 4 * e, 0));
                        const float v = fmaf((float)mine[(4 * q + e) * 64], g.sw_per_n ? sxv * sw : s, bv);    // one fp32 multiply
                        bool un;
                        code[e] = quant_gelu_fast<true>(v, gelu_inv, room3, tab, &un);
                        open |= un ? 1u << e : 0u;
                        mine[(4 * q + e) * 64] = (int)__float_as_uint(v);
                    }
                    uint32_t word = pack_bytes(code[0], code[1], code[2], code[3]);
                    if ((int)row >= rows) open = 0;
#pragma unroll 1
                    while (__ballot(open != 0)) {
                        const int e = open ? __ffs((int)open) - 1 : 0;
                        const uint32_t exact = settle_gelu(__uint_as_float((uint32_t)mine[(4 * q + e) * 64]), gelu_inv);
                        if (open) word = (word & ~(0xffu << (8 * e))) | exact << (8 * e);
                        open &= open - 1;
                    }
                    w[0] = w[1]; w[1] = w[2]; w[2] = w[3]; w[3] = word;
                }
                const auto a = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false), c = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
                const v4u out = {(unsigned)a[0], (unsigned)a[1], (unsigned)c[0], (unsigned)c[1]};
                __builtin_amdgcn_raw_buffer_store_b128(out, rq, (int)(c16 == kOob ? kOob : row * q_ld + c16), 0, kThrough);
            }
        }
    } else if (inside) {
        // ---- a tile that lies inside the output: stored from the accumulators.  For a fixed register each half of the wave owns
        // 32 neighbouring columns of one row, so every store of y writes two whole 128-byte segments and nothing is tested.
        // Turned through LDS as below, the stores come in bursts with LDS traffic between them, and a wave block of 96
        // columns keeps only 48 of the 64 lanes at work.  Through LDS / this way, us: 200704 x 256 x 64 with a residual 64.4 /
        // 56.4, 50176 x 512 x 128 26.3 / 24.8, 3x3 with int8 output 200704 x 64 x 576 24.8 / 22.8, 12544 x 256 x 2304 18.8 /
        // 18.2; 4096 x 3072 x 768 (128x192) 23.6 / 22.3, 16384 x 3072 x 768 in the encoder stack (256x128) 70.7 / 68.4.  (Naming
        // accumulation registers as the sums' home here splits the allocation of the whole kernel and spills; so do
        // residuals and int8 outputs on tiles above 128x128, which take the form below, as do residuals of the float types.)
        constexpr bool SMALL = ET == 0 && BM * BN <= 128 * 128;
        const bool has_res = SMALL && g.res_q != nullptr;
        if (has_res) {
            // the residual's codes of the tile through LDS (the stage memory is free now): one coalesced pass of 16-byte loads
            constexpr int RU = BN / 16, RIT = (BM * RU + NT - 1) / NT;     // 16-byte units per row, units per thread
            static_assert((size_t)NST * STAGE >= (size_t)BM * BN, "the residual tile must fit the stage memory");
            v4i rv[RIT];
#pragma unroll
            for (int it = 0; it < RIT; ++it) {
                const int u = tid + it * NT < BM * RU ? tid + it * NT : 0;
                rv[it] = *(const v4i *)((const int8_t *)g.res_q + (m0 + u / RU) * g.res_ld + n0 + (u % RU) * 16);
            }
            __syncthreads();                                              // every wave has read its last operands
#pragma unroll
            for (int it = 0; it < RIT; ++it) {
                const int u = tid + it * NT;
                if (u < BM * RU) *(v4i *)&lds[(u / RU) * BN + (u % RU) * 16] = rv[it];
            }
            __syncthreads();
        }
        auto direct = [&](auto relu_c, auto res_c, auto qout_c) {
            constexpr bool RELU = decltype(relu_c)::value, RES = decltype(res_c)::value, QOUT = decltype(qout_c)::value;
            const int32_t keep = RELU || g.amax_pos ? -1 : 0x7fffffff;
            // buffers of the tile's rows: a lane's place in a 32x32 block, and what the block and the register add, in scalars
            const __amdgpu_buffer_rsrc_t ryd = __builtin_amdgcn_make_buffer_rsrc((void *)(g.y + m0 * g.ldy), 0, g.y ? (int)(BM * g.ldy * 4) : 0, kBufferWord);
            const __amdgpu_buffer_rsrc_t rqd = __builtin_amdgcn_make_buffer_rsrc((void *)(g.q_out + m0 * g.q_ld), 0, QOUT ? (int)(BM * g.q_ld) : 0, kBufferWord);
            const int yoff = (int)((uint32_t)(lrow * g.ldy + lcol) * 4u), qoff = QOUT ? (int)(lrow * g.q_ld + lcol) : 0;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int col0 = n0 + (wn_u * TN + j) * 32;
                const float bj = g.bias ? g.bias[col0 + lcol] : 0.0f;
                const float sj = g.sw_per_n ? sxv * g.sw[col0 + lcol] : s;     // one fp32 multiply
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const int row0 = (wm_u * TM + i) * 32;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int rr = 8 * (r >> 2) + (r & 3);
                        float v = fmaf((float)acc[i][j][r], sj, bj);
                        if constexpr (RES) v = v + (float)(int8_t)lds[((wm_u * TM + i) * 32 + lrow + rr) * BN + (wn_u * TN + j) * 32 + lcol] * rs;
                        if (RELU) v = v > 0.0f ? v : 0.0f;
                        if (!QOUT || g.y) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), ryd, yoff, (int)((row0 + rr) * g.ldy + col0) * 4, kThrough);
                        if (QOUT) __builtin_amdgcn_raw_buffer_store_b8((uint8_t)quant1(v, q_inv), rqd, qoff, (int)((row0 + rr) * g.q_ld + col0), kThrough);
                        const int32_t bits = (int32_t)__float_as_uint(v) & keep;
                        amax = amax > bits ? amax : bits;
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        using T = std::true_type;
        using F = std::false_type;
        bool done = false;
        if constexpr (SMALL) {
            done = g.q_out || has_res;
            if (g.q_out) direct(T{}, F{}, T{});
            else if (has_res) { if (g.act == 1) direct(T{}, T{}, F{}); else direct(F{}, T{}, F{}); }
        }
        if (!done) { if (g.act == 1) direct(T{}, F{}, F{}); else direct(F{}, F{}, F{}); }
    } else {
        // ---- everything else: tiles at an edge, affine codes, observed runs.  A wave's sums go through LDS
        // (its own part of the stage memory, no barriers), a 32-row block at a time, and come back as four neighbouring
        // columns of one row per lane: one 16-byte store of y, four packed codes, four residual codes in one load, the
        // columns' scale and bias in registers.  Stores of y are raw buffer stores: what must not be written (rows beyond M,
        // columns beyond N) lies outside the buffer, so edge tiles run straight code as well.
        // (From the accumulators every element of such a tile had to be tested: 4728 x 2304 x 768 took 35.7 us where 4096
        // rows took 20.5; 19.3 this way.)
        constexpr int WC = TN * 32, WS = WC + 8;        // columns of a wave's block; words per row (pad: the two rows a
                                                        // write instruction touches fall into different banks)
        constexpr int LPR = WC / 4, RPI = 64 / LPR;     // lanes per row, rows per instruction (TN = 3: 48 lanes at work)
        constexpr int NP = 32 / RPI;
        static_assert(32 % RPI == 0 && (size_t)NST * STAGE >= (size_t)NW * 32 * WS * 4, "the waves' blocks must fit the stage memory");
        int32_t *yt = (int32_t *)lds + wave_u * 32 * WS;
        const bool zp = ET == 0 && g.zp_in != nullptr, relu = g.act == 1, has_res = g.res_q != nullptr;
        const bool active = lane / LPR < RPI;
        const int row_l = active ? lane / LPR : 0, unit = lane % LPR;   // (an idle lane reads what lanes of row 0 read, in bounds)
        const int wcol = wn_u * WC + 4 * unit, col = n0 + wcol;
        // the four columns' scale, bias and residual multiplier (zero beyond N: what is computed there is zero)
        float sj[4], bj[4], rj[4];
        int zlin[4] = {0, 0, 0, 0};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool ok = col + e < g.N;
            const int ce = ok ? col + e : g.N - 1;
            bj[e] = g.bias ? g.bias[ce] : 0.0f;
            sj[e] = g.sw_per_n ? sxv * g.sw[ce] : s;    // one fp32 multiply
            if (zp && !CONV) zlin[e] = zmul * g.colsum[ce];
            if (!ok) { bj[e] = 0.0f; sj[e] = 0.0f; zlin[e] = 0; }
            rj[e] = ok ? rs : 0.0f;
        }
        const int rows = (int)(g.M - m0 < BM ? g.M - m0 : BM);                    // valid rows of the tile
        // 16-byte stores through a buffer of the tile's rows (32-bit offsets)
        const bool vec = (g.N & 3) == 0 && (g.ldy & 3) == 0 && ((uintptr_t)g.y & 15) == 0 && g.ldy < (1 << 20) && g.res_ld < (1 << 20);
        const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void *)(g.y + m0 * g.ldy), 0, vec && g.y ? (int)(rows * g.ldy * 4) : 0, 0x00020000);
        const uint32_t ycol = active && col < g.N ? (uint32_t)col * 4u : kOob, ystep = (uint32_t)g.ldy * 4u;
        const int32_t keep = relu || g.amax_pos ? -1 : 0x7fffffff;
        __syncthreads();                                // every wave has read its last operands
        // lane l of a 32x32 block holds column l % 32 and rows 8 * (r / 4) + 4 * (l / 32) + r % 4
        auto put = [&](int i) {
            if (i > 0) wave_lds_turn();                 // the block before has been read
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) yt[(lrow + 8 * (r >> 2) + (r & 3)) * WS + j * 32 + lcol] = acc_bits(acc[i][j][r]);
            wave_lds_turn();
        };
        auto get = [&](int p) { return *(const v4i *)&yt[(p * RPI + row_l) * WS + 4 * unit]; };
        int32_t *zp_sum = (int32_t *)lds + NW * 32 * WS;         // affine codes: [16][BN], then a class per row (a launch
        uint8_t *zp_class = (uint8_t *)(zp_sum + 16 * BN);       // that has them brings the LDS for it)
        if (zp && CONV) {
            // the sums of the weight codes of the tile's columns per border class, and the class of every row's pixel
            for (int e = tid; e < 16 * BN; e += NT) {
                const int cls = e / BN, c = n0 + e % BN;
                zp_sum[e] = c < g.N ? zmul * g.colsum[(size_t)cls * g.N + c] : 0;
            }
            for (int e = tid; e < BM; e += NT) {
                const uint32_t m = (uint32_t)(m0 + e), mrow = m / (uint32_t)g.W;
                const int ow = (int)(m - mrow * (uint32_t)g.W), oh = (int)(mrow % (uint32_t)g.H);
                zp_class[e] = (uint8_t)((oh == 0 ? 1 : 0) | (oh == g.H - 1 ? 2 : 0) | (ow == 0 ? 4 : 0) | (ow == g.W - 1 ? 8 : 0));
            }
            __syncthreads();
        }
        // the combinations that forward passes ask for, straight-line
        auto fixed = [&](auto relu_c, auto track_c, auto res_c, auto qout_c, auto zp_c) {
            constexpr bool RELU = decltype(relu_c)::value, TRACK = decltype(track_c)::value, RES = decltype(res_c)::value;
            constexpr bool QOUT = decltype(qout_c)::value, ZP = decltype(zp_c)::value;
            const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc((void *)(g.q_out + m0 * g.q_ld), 0, QOUT ? (int)(rows * g.q_ld) : 0, 0x00020000);
            const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((void *)((const res_t *)g.res_q + m0 * g.res_ld), 0,
                                                                                 RES ? (int)(rows * g.res_ld * (int)sizeof(res_t)) : 0, 0x00020000);
            const uint32_t qcol = active && col < g.q_ld ? (uint32_t)col : kOob;
            const uint32_t rcol = active && col < g.res_ld ? (uint32_t)col * (uint32_t)sizeof(res_t) : kOob;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row0 = (wm_u * TM + i) * 32 + row_l;   // the lane's first row within the tile
                const int left = rows - row0;                    // valid rows from it on
                // four residual values per lane and row, requested before anything is awaited
                v4u rv[RES ? NP : 1];
                if constexpr (RES) {
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
                        const int off = (int)(rcol + (uint32_t)(row0 + p * RPI) * (uint32_t)(g.res_ld * (int)sizeof(res_t)));
                        if constexpr (ET == 0) rv[p][0] = __builtin_amdgcn_raw_buffer_load_b32(rr, off, 0, 0);
                        else if constexpr (ET == 1) {
                            const auto t = __builtin_amdgcn_raw_buffer_load_b64(rr, off, 0, 0);
                            rv[p][0] = t[0];
                            rv[p][1] = t[1];
                        } else rv[p] = __builtin_amdgcn_raw_buffer_load_b128(rr, off, 0, 0);
                    }
                }
                put(i);
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    v4i a = get(p);
                    if constexpr (ZP) {
                        if constexpr (CONV) {
                            const v4i z = *(const v4i *)&zp_sum[zp_class[row0 + p * RPI] * BN + wcol];
#pragma unroll
                            for (int e = 0; e < 4; ++e) a[e] += z[e];
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; ++e) a[e] += zlin[e];
                        }
                    }
                    v4u w;
                    uint32_t codes = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float v = fmaf(ET == 0 ? (float)a[e] : __int_as_float(a[e]), sj[e], bj[e]);
                        if constexpr (RES) {
                            float x;
                            if constexpr (ET == 0) x = (float)((int)(int8_t)(rv[p][0] >> (8 * e)) + (ZP ? rmul : 0));
                            else if constexpr (ET == 1) x = (float)__builtin_bit_cast(_Float16, (uint16_t)(rv[p][e >> 1] >> (16 * (e & 1))));
                            else x = __uint_as_float(rv[p][e]);
                            v = v + x * rj[e];
                        }
                        if (RELU) v = v > 0.0f ? v : 0.0f;
                        w[e] = __float_as_uint(v);
                        if (QOUT) codes |= (col + e < g.N ? quant1(v, q_inv) : 0u) << (8 * e);   // pad columns are zero
                        if (TRACK) {
                            int32_t bits = (int32_t)w[e];
                            if (!RELU) bits &= keep;
                            bits = p * RPI < left ? bits : 0;
                            amax = amax > bits ? amax : bits;
                        }
                    }
                    __builtin_amdgcn_raw_buffer_store_b128(w, ry, (int)(ycol + (uint32_t)(row0 + p * RPI) * ystep), 0, kThrough);
                    if (QOUT) __builtin_amdgcn_raw_buffer_store_b32(codes, rq, (int)(qcol + (uint32_t)(row0 + p * RPI) * (uint32_t)g.q_ld), 0, kThrough);
                }
            }
        };
        // everything else: observed runs, rows that 16-byte stores cannot address, rare combinations
        auto general = [&]() {
            const bool acc16 = (g.N & 3) == 0 && ((uintptr_t)g.acc_out & 15) == 0;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row0 = (wm_u * TM + i) * 32 + row_l;   // the lane's first row within the tile
                // the residual of the block's rows, requested before anything is awaited
                int32_t rcode[ET == 0 ? NP : 1];
                if constexpr (ET == 0) {
                    if (has_res) {
#pragma unroll
                        for (int p = 0; p < NP; ++p) {
                            const bool ok = active && row0 + p * RPI < rows && col < g.res_ld;
                            rcode[p] = *(const int32_t *)(g.res_q + (ok ? (m0 + row0 + p * RPI) * g.res_ld + col : 0));
                        }
                    }
                }
                put(i);
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const int tr = row0 + p * RPI;
                    const int64_t m = m0 + tr;
                    const v4i a4 = get(p);
                    int a[4] = {a4[0], a4[1], a4[2], a4[3]};
                    if constexpr (ET == 0) {
                        if (zp) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) a[e] += CONV ? zp_sum[zp_class[tr] * BN + wcol + e] : zlin[e];
                        }
                    }
                    const bool in = active && tr < rows;
                    if (g.acc_out && in) {              // observed runs: the raw sums
                        int32_t *dst = g.acc_out + m * g.N + col;
                        if (acc16 && col < g.N) *(v4i *)dst = v4i{a[0], a[1], a[2], a[3]};
                        else
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (col + e < g.N) dst[e] = a[e];
                    }
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = fmaf(ET == 0 ? (float)a[e] : __int_as_float(a[e]), sj[e], bj[e]);
                    if (has_res) {
                        if constexpr (ET == 0) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[e] = v[e] + (float)((int)(int8_t)(rcode[p] >> (8 * e)) + rmul) * rj[e];
                        } else {
                            const res_t *res = (const res_t *)g.res_q + (in && col < g.res_ld ? m * g.res_ld + col : 0);   // (rows are padded to whole units)
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[e] = v[e] + (float)res[e] * rj[e];
                        }
                    }
                    v4u w;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float vp = v[e] > 0.0f ? v[e] : 0.0f;
                        v[e] = relu ? vp : v[e];
                        w[e] = __float_as_uint(v[e]);
                        const int32_t bits = in ? (int32_t)w[e] & keep : 0;
                        amax = amax > bits ? amax : bits;
                    }
                    __builtin_amdgcn_raw_buffer_store_b128(w, ry, (int)(ycol + (uint32_t)tr * ystep), 0, 0);   // (no extent unless vec)
                    if (g.y && !vec && in) {
                        float *dst = g.y + m * g.ldy + col;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (col + e < g.N) dst[e] = v[e];
                    }
                    if (g.q_out && in && col < g.q_ld) {         // pad columns of the int8 output are zero
                        uint32_t c4 = 0;
#pragma unroll
                        for (int e = 0; e < 4; ++e) c4 |= (col + e < g.N ? quant1(v[e], q_inv) : 0u) << (8 * e);
                        *(uint32_t *)(g.q_out + m * g.q_ld + col) = c4;
                    }
                }
            }
        };
        using T = std::true_type;
        using F = std::false_type;
        const bool track = g.absmax_out != nullptr, q = g.q_out != nullptr;
        const bool rare = !vec || g.acc_out || (track && (has_res || q || (zp && !relu))) || (q && (!relu || has_res || zp)) || (has_res && !relu);
        if (rare) general();
        else if (zp) {
            if constexpr (ET == 0) {
                if (has_res) fixed(T{}, F{}, T{}, F{}, T{});
                else if (track) fixed(T{}, T{}, F{}, F{}, T{});
                else if (relu) fixed(T{}, F{}, F{}, F{}, T{});
                else fixed(F{}, F{}, F{}, F{}, T{});
            }
        } else if (has_res) fixed(T{}, F{}, T{}, F{}, F{});
        else if (q) { if constexpr (ET == 0) fixed(T{}, F{}, F{}, T{}, F{}); }
        else if (relu) {
            if (track) fixed(T{}, T{}, F{}, F{}, F{}); else fixed(T{}, F{}, F{}, F{}, F{});
        } else {
            if (track) fixed(F{}, T{}, F{}, F{}, F{}); else fixed(F{}, F{}, F{}, F{}, F{});
        }
    }
    if (EPI != kGeluCodes && g.absmax_out) {
        __shared__ uint32_t smw[NW];
        if constexpr (NW == 4) {
            block_atomic_max((uint32_t)amax, g.absmax_out, smw);
        } else {
            const uint32_t v = wave_max_u32((uint32_t)amax);
            if (lane == 0) smw[wave] = v;
            __syncthreads();
            if (tid == 0) {
                uint32_t a = 0;
#pragma unroll
                for (int w = 0; w < NW; ++w) a = smw[w] > a ? smw[w] : a;
                uint32_t *way = g.absmax_out + (blockIdx.x & (kAmaxWays - 1)) * kAmaxStride;
                if (a > __hip_atomic_load(way, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(way, a);
            }
        }
    }
}

template <int BM, int BN, int WM, int WN, int BK, int ET = 0, int EPI = kStore, int NST = stages_for(BK)>
static hipError_t launch_variant(const GemmArgs &g, hipStream_t st)
{
    const int64_t tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
    if (tiles <= 0) return hipSuccess;
    if (tiles > 0x3fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)tiles), block(64 * WM * WN);
    constexpr size_t stages = (size_t)NST * (BM + BN) * BK;
    // affine codes: weight-code sums and row classes behind the epilogue's block
    constexpr size_t affine = ((size_t)WM * 32 * (BN + 8 * WN) + 16 * BN) * 4 + BM, largest = stages > affine ? stages : affine;
    const size_t smem = EPI == kGeluCodes ? stages + kGeluTableBytes : (g.zp_in ? largest : stages);
    hipError_t e;
    const int dev = current_device();
    if (dev < 0) return hipErrorInvalidDevice;
    if (g.conv3x3) {
        if constexpr (EPI != kStore || BM * BN > 256 * 128) {
            return hipErrorInvalidValue;                         // shapes for linear layers only
        } else {
            static bool set[kMaxDevices] = {};                   // the attribute belongs to one device's code object
            if (!set[dev]) {
                e = hipFuncSetAttribute((const void *)gemm_i8_kernel<BM, BN, WM, WN, true, BK, ET, EPI, NST>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)largest);
                if (e != hipSuccess) return e;
                set[dev] = true;
            }
            return launch_k(EGERIA_KERNEL_GEMM, gemm_i8_kernel<BM, BN, WM, WN, true, BK, ET, EPI, NST>, grid, block, smem, st, g);
        }
    }
    static bool set[kMaxDevices] = {};
    if (!set[dev]) {
        e = hipFuncSetAttribute((const void *)gemm_i8_kernel<BM, BN, WM, WN, false, BK, ET, EPI, NST>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)(EPI == kGeluCodes ? stages + kGeluTableBytes : largest));
        if (e != hipSuccess) return e;
        set[dev] = true;
    }
    // (instrumentation: the launch that also normalises its rows is timed with the layer norms, whose bytes bound it)
    return launch_k(EPI == kLayerNorm ? EGERIA_KERNEL_LAYERNORM : EGERIA_KERNEL_GEMM, gemm_i8_kernel<BM, BN, WM, WN, false, BK, ET, EPI, NST>,
                    grid, block, smem, st, g);
}

// ---- 3x3 convolution with at most 16 input channels and at most 32 outputs ----------------
// (the first stages of CIFAR-style ResNets).  The problem is bandwidth bound and
// each output pixel needs only 9 x 16 bytes of input, so there is no LDS stage
// and no barrier: a wave owns 32 consecutive output pixels; lane l reads, for
// K step s, the 16 channel bytes of pixel l % 32 displaced by tap 2s + l / 32
// (half-waves read contiguous 512-byte runs) and the matching 16 weight bytes of
// output channel l % 32; five MFMAs cover the nine taps (the tenth is zero).
__global__ __launch_bounds__(256) void conv3x3_c16_kernel(const GemmArgs g)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int p = lane & 31, h = lane >> 5;
    const uint32_t blk = xcd_piece(blockIdx.x, gridDim.x);
    const int64_t m = ((int64_t)blk * 4 + wave) * 32 + p;
    const bool m_ok = m < g.M;
    // the operand's extent is below 2^31 bytes, so pixel indices fit 32 bits (64-bit division is slow)
    const uint32_t mrow = (uint32_t)m / (uint32_t)g.W;
    const int ow = (int)((uint32_t)m - mrow * (uint32_t)g.W), oh = (int)(mrow % (uint32_t)g.H);
    const float s = (*g.sx) * (g.sw_per_n ? (p < g.N ? g.sw[p] : 0.0f) : *g.sw);   // lane's output channel is p
    const float rs = g.res_q ? *g.res_scale : 0.0f;
    // the residual of the workgroup's 128 pixels (16 bytes each, contiguous): requested now with
    // one 16-byte load per thread, handed to the epilogue through LDS
    __shared__ __attribute__((aligned(16))) uint8_t sres[128 * 16];
    const bool res16 = g.res_q != nullptr && g.res_ld == 16;
    v4i resv = {0, 0, 0, 0};
    if (res16 && threadIdx.x < 128) {
        const int64_t pix = (int64_t)blk * 128 + threadIdx.x;
        if (pix < g.M) resv = *(const v4i *)(g.res_q + pix * 16);
    }
    v4i fa[5], fb[5];
#pragma unroll
    for (int st = 0; st < 5; ++st) {
        const int tap = 2 * st + h;
        const int kh = tap / 3, dh = kh - 1, dw = tap - kh * 3 - 1;
        const bool ok = m_ok && tap < 9 && (unsigned)(oh + dh) < (unsigned)g.H && (unsigned)(ow + dw) < (unsigned)g.W;
        fa[st] = ok ? *(const v4i *)(g.a + (m + (int64_t)dh * g.W + dw) * 16) : v4i{0, 0, 0, 0};
        fb[st] = (p < g.N && tap < 9) ? *(const v4i *)(g.w + (int64_t)p * g.kp + tap * 16) : v4i{0, 0, 0, 0};
    }
    v16i acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0;
#pragma unroll
    for (int st = 0; st < 5; ++st) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[st], fb[st], acc, 0, 0, 0);

    // lane holds output channel p and pixels 8 * (r / 4) + 4 * h + r % 4 of the wave's 32
    const int col = p;
    const bool col_ok = col < g.N;
    const float bc = (g.bias && col_ok) ? g.bias[col] : 0.0f;
    const int64_t mw = ((int64_t)blk * 4 + wave) * 32;
    const float q_inv = g.q_out ? (float)(1.0 / (double)*g.q_scale) : 0.0f;
    if (res16) {
        if (threadIdx.x < 128) *(v4i *)&sres[threadIdx.x * 16] = resv;
        __syncthreads();
    }
    uint32_t amax = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int64_t row = mw + (r >> 2) * 8 + h * 4 + (r & 3);
        if (row >= g.M) continue;
        if (!col_ok) {
            if (g.q_out && col < g.q_ld) g.q_out[row * g.q_ld + col] = 0;     // pad columns of the int8 output
            continue;
        }
        const int a = acc[r];
        if (g.acc_out) g.acc_out[row * g.N + col] = a;
        float v = fmaf((float)a, s, bc);
        if (res16) v = v + (float)(int8_t)sres[(wave * 32 + (r >> 2) * 8 + h * 4 + (r & 3)) * 16 + col] * rs;
        else if (g.res_q) v = v + (float)g.res_q[row * g.res_ld + col] * rs;
        if (g.act == 1) v = v > 0.0f ? v : 0.0f;
        if (g.y) g.y[row * g.ldy + col] = v;
        if (g.q_out) g.q_out[row * g.q_ld + col] = (int8_t)quant1(v, q_inv);
        const uint32_t ab = g.amax_pos ? (v > 0.0f ? __float_as_uint(v) : 0u) : abs_bits(v);
        amax = amax > ab ? amax : ab;
    }
    if (g.absmax_out) {
        __shared__ uint32_t sm4[4];
        block_atomic_max(amax, g.absmax_out, sm4);
    }
}

// ---- the same convolution with the quantiser of its operands folded in -------------------
// A workgroup owns 128 consecutive output pixels.  It reduces the candidate
// maxima of the operand's quantise point to the scale (as every quantise kernel
// does), turns the fp32 values of its pixels and of the W + 1 pixels before and
// after them into int8 codes in LDS (16 bytes per pixel), and the five MFMAs
// of a wave read their operands from there.  The residual of the skip
// connection is either a block of ready codes or, likewise, the block input
// quantised on load.  Workgroup 0 stores the scales for later kernels.
// All global reads of this kernel are raw buffer loads: a request that must not
// happen (a pixel outside the tensor, a channel beyond c, a candidate beyond n) is
// given an offset outside the buffer and returns zero, so no load sits under a
// branch.  (A load under a branch is awaited where the branch ends: one memory
// round trip per load instead of one for all of them.)  Extents are below 2^31.
constexpr uint32_t kNoLoad = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_buffer(const void *p, int64_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float buffer_f32(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}
template <bool BF16>
__device__ __forceinline__ float buffer_elem(__amdgpu_buffer_rsrc_t r, uint32_t index, bool ok)
{
    if (BF16) return __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)(ok ? index * 2 : kNoLoad), 0, 0) << 16);
    return buffer_f32(r, ok ? index * 4 : kNoLoad);
}
// channels [4 gq, 4 gq + 4) of pixel pi of a [n, c, hw] tensor (zeros beyond c and where !ok)
template <bool BF16>
__device__ __forceinline__ float4 plane_values(__amdgpu_buffer_rsrc_t r, int c, uint32_t hw, uint32_t pi, int gq, bool ok)
{
    const uint32_t img = pi / hw, pp = pi - img * hw;                // pixel counts fit 31 bits here: 32-bit division
    const uint32_t base = (img * c + gq * 4) * hw + pp;
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = buffer_elem<BF16>(r, base + e * hw, ok && gq * 4 + e < c);
    return make_float4(v[0], v[1], v[2], v[3]);
}
// item idx of the operand stage: four channels of one of the npix staged pixels.
// Rows of c floats: four consecutive threads share a pixel; channel planes:
// consecutive threads take consecutive pixels of one channel group.
template <int A_SRC>
__device__ __forceinline__ void operand_item(int idx, int npix, int &j, int &gq)
{
    if (A_SRC == 1) { j = idx >> 2; gq = idx & 3; }
    else { gq = idx / npix; j = idx - gq * npix; }
}
template <int A_SRC, bool BF16, bool C16>
__device__ __forceinline__ float4 load_operand_item(__amdgpu_buffer_rsrc_t r, int c, int M, uint32_t hw, int first_pix, int npix, int idx)
{
    int j, gq;
    operand_item<A_SRC>(idx, npix, j, gq);
    const int pi = first_pix + j;
    const bool ok = idx < npix * 4 && pi >= 0 && pi < M;
    if (A_SRC == 1) {
        const uint32_t row = (uint32_t)pi * (uint32_t)c;
        if (C16) {
            const v4u q = __builtin_amdgcn_raw_buffer_load_b128(r, (int)(ok ? (row + gq * 4) * 4 : kNoLoad), 0, 0);
            return make_float4(__uint_as_float(q[0]), __uint_as_float(q[1]), __uint_as_float(q[2]), __uint_as_float(q[3]));
        }
        float t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = buffer_f32(r, (ok && gq * 4 + e < c) ? (row + gq * 4 + e) * 4 : kNoLoad);
        return make_float4(t[0], t[1], t[2], t[3]);
    }
    return plane_values<BF16>(r, c, hw, (uint32_t)pi, gq, ok);
}
// the lane's share of n candidate maxima, `stride` words apart (n <= 512)
__device__ __forceinline__ uint32_t buffer_candidates(const uint32_t *slot, int n, int stride)
{
    const __amdgpu_buffer_rsrc_t r = raw_buffer(slot, n > 0 ? ((int64_t)(n - 1) * stride + 1) * 4 : 0);
    const int lane = threadIdx.x & 63;
    uint32_t v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int i = lane + 64 * k;
        v[k] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)(i < n ? (uint32_t)(i * stride) * 4 : kNoLoad), 0, 0);
    }
    uint32_t bits = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) bits = v[k] > bits ? v[k] : bits;
    return bits;
}
__device__ __forceinline__ uint32_t pack_codes(float4 v, float inv)
{
    return quant1(v.x, inv) | quant1(v.y, inv) << 8 | quant1(v.z, inv) << 16 | quant1(v.w, inv) << 24;
}

// XBF16: the channel planes read (operand of a_src 2, residual of res_src 1) hold bf16; C16 (a_src 1): rows of 16 floats
template <int A_SRC, bool XBF16, bool C16>
__global__ __launch_bounds__(256) void conv3x3_c16_fused_kernel(const GemmArgs g, const ConvFuse z)
{
    // [128][16] residual codes, bias [32], weight scale [32], [128 + 2 (W + 1)][16] operand codes
    extern __shared__ __attribute__((aligned(16))) uint8_t sdyn[];
    uint8_t *sres = sdyn, *sa = sdyn + 128 * 16 + 256;
    float *sbias = (float *)(sdyn + 128 * 16), *ssw = sbias + 32;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int p = lane & 31, h = lane >> 5;
    const int m0 = (int)xcd_piece(blockIdx.x, gridDim.x) * 128, M = (int)g.M;
    const uint32_t hw = (uint32_t)g.H * (uint32_t)g.W;
    const int halo = g.W + 1, npix = 128 + 2 * halo;
    const int xes = XBF16 ? 2 : 4;

    // ---- every request the workgroup depends on goes out before anything is awaited:
    // the first 1024 items of the operand stage (all of it up to 62 pixels of width), the
    // residual, the weights and the candidate maxima
    const __amdgpu_buffer_rsrc_t ra = raw_buffer(z.a_f, A_SRC == 0 ? 0 : (int64_t)M * z.c * (A_SRC == 1 ? 4 : xes));
    constexpr int NB = 4;
    float4 raw[NB];
    if (A_SRC != 0) {
#pragma unroll
        for (int b = 0; b < NB; ++b) raw[b] = load_operand_item<A_SRC, XBF16, C16>(ra, z.c, M, hw, m0 - halo, npix, threadIdx.x + 256 * b);
    }
    // both forms of the residual are requested; the one that is not in use has an empty buffer
    const bool res_planes = z.res_src == 1, res_codes = !res_planes && g.res_q != nullptr;
    const __amdgpu_buffer_rsrc_t rrp = raw_buffer(z.res_f, res_planes ? (int64_t)M * z.res_c * xes : 0);
    const __amdgpu_buffer_rsrc_t rrq = raw_buffer(g.res_q, res_codes ? (int64_t)M * 16 : 0);
    float4 rraw[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int idx = threadIdx.x + 256 * b, gq = idx >> 7, j = idx & 127;
        rraw[b] = plane_values<XBF16>(rrp, z.res_c, hw, (uint32_t)(m0 + j), gq, res_planes && m0 + j < M);
    }
    const int rpi = m0 + (int)(threadIdx.x & 127);
    const v4i rv = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rrq, (int)((res_codes && rpi < M) ? (uint32_t)rpi * 16 : kNoLoad), 0, 0));
    const __amdgpu_buffer_rsrc_t rw = raw_buffer(g.w, g.w_bytes);
    v4i fb[5];
#pragma unroll
    for (int st = 0; st < 5; ++st) {
        const int tap = 2 * st + h;
        fb[st] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(
                                             rw, (int)((p < g.N && tap < 9) ? (uint32_t)(p * g.kp + tap * 16) : kNoLoad), 0, 0));
    }
    // bias and weight scale of output channel t, for threads t < 32 (zero beyond N)
    const __amdgpu_buffer_rsrc_t rb = raw_buffer(g.bias, g.bias ? (int64_t)g.N * 4 : 0);
    const __amdgpu_buffer_rsrc_t rs_w = raw_buffer(g.sw, g.sw_per_n ? (int64_t)g.N * 4 : 4);
    const uint32_t ct = threadIdx.x & 31;
    const float bias_t = buffer_f32(rb, ct * 4), sw_t = buffer_f32(rs_w, g.sw_per_n ? ct * 4 : 0u);
    uint32_t cand_a = 0, cand_r = 0;
    if (A_SRC != 0) cand_a = buffer_candidates(z.a_slot, z.a_nslot, z.a_stride);
    cand_r = buffer_candidates(z.res_slot, res_planes ? z.res_nslot : 0, z.res_stride);

    float scale_a;
    if (A_SRC != 0) {
        bool bad;
        const float inv = scale_from_bits(wave_max_u32(cand_a), z.a_fixed, &scale_a, &bad);
        if (blockIdx.x == 0 && threadIdx.x == 0) publish(scale_a, bad, z.a_scale_out, nullptr, z.flag);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int idx = threadIdx.x + 256 * b;
            int j, gq;
            operand_item<A_SRC>(idx, npix, j, gq);
            if (idx < npix * 4) *(uint32_t *)&sa[j * 16 + gq * 4] = pack_codes(raw[b], inv);
        }
        for (int idx = threadIdx.x + 256 * NB; idx < npix * 4; idx += 256) {       // wide images
            int j, gq;
            operand_item<A_SRC>(idx, npix, j, gq);
            *(uint32_t *)&sa[j * 16 + gq * 4] = pack_codes(load_operand_item<A_SRC, XBF16, C16>(ra, z.c, M, hw, m0 - halo, npix, idx), inv);
        }
    } else {
        scale_a = *g.sx;
    }
    if (threadIdx.x < 32) {
        sbias[threadIdx.x] = bias_t;
        ssw[threadIdx.x] = (int)threadIdx.x < g.N ? sw_t : 0.0f;
    }
    float rs = 0.0f;
    const bool has_res = z.res_src == 1 || g.res_q != nullptr;
    if (z.res_src == 1) {
        bool bad;
        const float inv = scale_from_bits(wave_max_u32(cand_r), z.res_fixed, &rs, &bad);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int idx = threadIdx.x + 256 * b, gq = idx >> 7, j = idx & 127;
            *(uint32_t *)&sres[j * 16 + gq * 4] = pack_codes(rraw[b], inv);
        }
    } else if (g.res_q) {
        rs = *g.res_scale;
        if (threadIdx.x < 128) *(v4i *)&sres[threadIdx.x * 16] = rv;
    }
    __syncthreads();

    const int lp = wave * 32 + p;                                    // the lane's output pixel within the workgroup
    const int m = m0 + lp;
    const bool m_ok = m < M;
    const uint32_t mrow = (uint32_t)m / (uint32_t)g.W;
    const int ow = (int)((uint32_t)m - mrow * (uint32_t)g.W), oh = (int)(mrow % (uint32_t)g.H);
    v4i fa[5];
#pragma unroll
    for (int st = 0; st < 5; ++st) {
        const int tap = 2 * st + h;
        const int kh = tap / 3, dh = kh - 1, dw = tap - kh * 3 - 1;
        const bool ok = m_ok && tap < 9 && (unsigned)(oh + dh) < (unsigned)g.H && (unsigned)(ow + dw) < (unsigned)g.W;
        if (A_SRC != 0) fa[st] = ok ? *(const v4i *)&sa[(lp + halo + dh * g.W + dw) * 16] : v4i{0, 0, 0, 0};
        else fa[st] = ok ? *(const v4i *)(g.a + ((int64_t)m + dh * g.W + dw) * 16) : v4i{0, 0, 0, 0};
    }
    // Weights are the row operand and pixels the column operand, so a lane ends up with 16 output
    // channels of ONE pixel: channels 8 (r / 4) + 4 h + r % 4 in register r, i.e. four groups of four
    // consecutive channels, which go out as 16-byte stores.
    v16i acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0;
#pragma unroll
    for (int st = 0; st < 5; ++st) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[st], fa[st], acc, 0, 0, 0);

    const float q_inv = g.q_out ? (float)(1.0 / (double)*g.q_scale) : 0.0f;
    const int n_out = g.q_out && g.q_ld > g.N ? (int)g.q_ld : g.N;               // channels that receive anything
    const bool vec = g.y && (g.N & 3) == 0 && (g.ldy & 3) == 0 && ((uintptr_t)g.y & 15) == 0;
    uint32_t amax = 0;
#pragma unroll
    for (int gi = 0; gi < 4; ++gi) {
        const int ch0 = 8 * gi + 4 * h;
        if (8 * gi >= n_out) break;                                               // uniform
        if (!m_ok || ch0 >= n_out) continue;
        const float4 b4 = *(const float4 *)&sbias[ch0], w4 = *(const float4 *)&ssw[ch0];
        const float bb[4] = {b4.x, b4.y, b4.z, b4.w}, ww[4] = {w4.x, w4.y, w4.z, w4.w};
        const uint32_t rc = has_res ? *(const uint32_t *)&sres[lp * 16 + (ch0 & 15)] : 0u;
        float v[4];
        uint32_t codes = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float t = fmaf((float)acc[4 * gi + e], scale_a * ww[e], bb[e]);
            if (has_res) t = t + (float)(int8_t)(rc >> (8 * e)) * rs;
            if (g.act == 1) t = t > 0.0f ? t : 0.0f;
            const bool ch_ok = ch0 + e < g.N;
            if (g.absmax_out) {
                const uint32_t ab = g.amax_pos ? (t > 0.0f ? __float_as_uint(t) : 0u) : abs_bits(t);
                amax = (ch_ok && ab > amax) ? ab : amax;
            }
            if (g.q_out) codes |= (ch_ok ? quant1(t, q_inv) : 0u) << (8 * e);     // pad columns of the int8 output are zero
            v[e] = t;
        }
        if (g.y) {
            float *dst = g.y + (int64_t)m * g.ldy + ch0;
            if (vec) {
                *(float4 *)dst = make_float4(v[0], v[1], v[2], v[3]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (ch0 + e < g.N) dst[e] = v[e];
            }
        }
        if (g.q_out && ch0 < g.q_ld) *(uint32_t *)(g.q_out + (int64_t)m * g.q_ld + ch0) = codes;
    }
    if (g.absmax_out) {
        __shared__ uint32_t sm4[4];
        block_atomic_max(amax, g.absmax_out, sm4);
    }
}

hipError_t launch_conv3x3_c16_fused(const GemmArgs &g, const ConvFuse &z, hipStream_t st)
{
    // what the kernel assumes: 16-byte pixels, a residual of 16 codes per pixel at most, no raw-accumulator
    // output, a halo that fits the LDS stage
    if (!g.conv3x3 || g.cp != 16 || g.N < 1 || g.N > 32 || g.kp != 9 * 16 || g.et != 0 || g.acc_out) return hipErrorInvalidValue;
    if (g.W < 1 || g.H < 1 || g.W > kConvFuseMaxWidth || g.M % ((int64_t)g.H * g.W) != 0) return hipErrorInvalidValue;
    if (g.M > 0x7fffffffLL - 2 * (kConvFuseMaxWidth + 1) - 128) return hipErrorInvalidValue;    // 32-bit pixel arithmetic
    if (z.a_src < 0 || z.a_src > 2 || (z.a_src != 0 && (!z.a_f || z.c < 1 || z.c > 16))) return hipErrorInvalidValue;
    if (z.a_src == 0 && (!g.a || !g.sx)) return hipErrorInvalidValue;
    if (z.res_src == 1 && (!z.res_f || z.res_c < 1 || z.res_c > 16 || g.N > 16)) return hipErrorInvalidValue;
    if (z.res_src == 0 && g.res_q && (g.res_ld != 16 || g.N > 16)) return hipErrorInvalidValue;
    const int64_t blocks = (g.M + 127) / 128;
    if (blocks <= 0) return hipSuccess;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const size_t smem = 128 * 16 + 256 + (z.a_src != 0 ? (size_t)(128 + 2 * (g.W + 1)) * 16 : 0);
    const dim3 grid((unsigned)blocks), block(256);
    // what the kernel's 32-bit offsets assume
    if (g.M * 16 * 4 >= (1LL << 31) || g.w_bytes >= (1LL << 31) || z.a_nslot > 512 || z.res_nslot > 512) return hipErrorInvalidValue;
    // XBF16: element type of the planes read (the block input: operand of a_src 2, residual of res_src 1)
    const bool xbf16 = z.a_src == 2 ? z.a_bf16 != 0 : (z.res_src == 1 && z.res_bf16 != 0);
    if (z.a_src == 2 && z.res_src == 1 && (z.a_bf16 != 0) != (z.res_bf16 != 0)) return hipErrorInvalidValue;
#define EG_FUSED(A, B, C) launch_k(EGERIA_KERNEL_GEMM, conv3x3_c16_fused_kernel<A, B, C>, grid, block, smem, st, g, z)
    if (z.a_src == 0) return xbf16 ? EG_FUSED(0, true, false) : EG_FUSED(0, false, false);
    if (z.a_src == 1) {
        if (z.c == 16) return xbf16 ? EG_FUSED(1, true, true) : EG_FUSED(1, false, true);
        return xbf16 ? EG_FUSED(1, true, false) : EG_FUSED(1, false, false);
    }
    return xbf16 ? EG_FUSED(2, true, false) : EG_FUSED(2, false, false);
#undef EG_FUSED
}

// The tile shapes on offer: rows x columns of the output tile, K bytes per
// step, workgroups of that shape that fit a CU together (registers and LDS),
// and the relative cost of a unit of tile area (smaller tiles move more LDS
// and L1 bytes per MFMA).
struct TileShape {
    int bm, bn, bk, resident, waves;
    double penalty;
};
constexpr int kNumShapes = 8, kDeepSmall = 8, kDeepMid = 9, kDeepLarge = 10;
static const TileShape kShapes[kNumShapes + 3] = {
    {256, 128, 64, 2, 4, 1.06},  {128, 192, 64, 2, 4, 1.10}, {128, 128, 64, 3, 4, 1.20},  {128, 128, 128, 2, 4, 1.22},
    {128, 64, 64, 4, 4, 1.40},   {128, 64, 128, 3, 4, 1.38}, {256, 256, 128, 1, 8, 1.00}, {256, 192, 128, 1, 8, 1.02},
    // three stages of whole lines, for layers that bring a compute unit one workgroup or two (chosen by rule, not by price)
    {64, 64, 128, 3, 4, 0.0},    {128, 64, 128, 2, 8, 0.0},  {128, 128, 128, 1, 8, 0.0},
};

template <int ET>
static hipError_t launch_shape(int i, const GemmArgs &g, hipStream_t st)
{
    switch (i) {
    case 0: return launch_variant<256, 128, 2, 2, 64, ET>(g, st);
    case 1: return launch_variant<128, 192, 2, 2, 64, ET>(g, st);
    case 2: return launch_variant<128, 128, 2, 2, 64, ET>(g, st);
    case 3: return launch_variant<128, 128, 2, 2, 128, ET>(g, st);
    case 4: return launch_variant<128, 64, 2, 2, 64, ET>(g, st);
    case 5: return launch_variant<128, 64, 2, 2, 128, ET>(g, st);
    case 6: return launch_variant<256, 256, 2, 4, 128, ET>(g, st);
    case 7: return launch_variant<256, 192, 4, 2, 128, ET>(g, st);
    case kDeepSmall: return launch_variant<64, 64, 2, 2, 128, ET, kStore, 3>(g, st);
    case kDeepMid: return launch_variant<128, 64, 4, 2, 128, ET, kStore, 3>(g, st);
    case kDeepLarge: return launch_variant<128, 128, 2, 4, 128, ET, kStore, 3>(g, st);
    default: return hipErrorInvalidValue;
    }
}

// The two passes of a layer whose output only feeds a GELU (GemmArgs::gelu_pass): nothing or a byte a value is stored, so the
// operands' way into LDS and, in the second pass, vector instructions are what they cost, and large tiles with whole-line K steps
// and eight waves are the fast ones.  A round takes about 3.5 us and 1 us for every 4096 values of a compute unit's tiles (both
// passes of 768 products, us: 256x256 11.4 + 19, 256x192 9.8 + 15.6, two 128x128 7.7 + 11.9, 128x192 10.9 for the second,
// two 64x64 5.9): the shape whose rounds cost least.  us, 128x192 / 128x128 / 256x192 / 256x256: 4096 x 3072 x 768 42.6 / 43.4 / 33.3 /
// 36.5, 4728 rows 54.7 / 46.9 / 55.7 / 42.9, 16384 rows 136 / 121 / 110 / 99, 1920 x 2304 x 576 19.4 / 20.3 / 28.9 / 32.7.
template <int EPI>
static hipError_t launch_gelu(const GemmArgs &g, hipStream_t st)
{
    constexpr struct { int bm, bn, resident; double penalty; } shapes[] = {
        {256, 256, 1, 1.0}, {256, 192, 1, 1.0}, {128, 192, 1, 1.07}, {128, 128, 2, 1.07}, {128, 64, 2, 1.07}, {64, 64, 2, 1.07}};
    int best = 0;
    double best_cost = 0.0;
    for (int i = 0; i < 6; ++i) {
        const int64_t tiles = ((g.M + shapes[i].bm - 1) / shapes[i].bm) * ((g.N + shapes[i].bn - 1) / shapes[i].bn);
        const int64_t slots = (int64_t)compute_units() * shapes[i].resident;
        const double cost = (double)((tiles + slots - 1) / slots) * (shapes[i].bm * shapes[i].bn * shapes[i].resident + 14336) * shapes[i].penalty;
        if (i == 0 || cost < best_cost) {
            best_cost = cost;
            best = i;
        }
    }
    switch (best) {
    case 0: return launch_variant<256, 256, 2, 4, 128, 0, EPI>(g, st);
    case 1: return launch_variant<256, 192, 4, 2, 128, 0, EPI>(g, st);
    case 2: return launch_variant<128, 192, 2, 2, 64, 0, EPI>(g, st);
    case 3: return launch_variant<128, 128, 2, 2, 64, 0, EPI>(g, st);
    case 4: return launch_variant<128, 64, 2, 2, 64, 0, EPI>(g, st);
    default: return launch_variant<64, 64, 2, 2, 128, 0, EPI, 3>(g, st);
    }
}

// Tile choice.  A tile shape is priced by the work the chip does for it,
// padding included: workgroups run in rounds of (compute units) x (workgroups resident
// per CU), a partly filled last round costs as much as a full one, and the
// smaller shapes pay more LDS and L1 traffic per MFMA.  With fp32 outputs the
// epilogue (convert, scale, store) costs as much as the K loop unless K is
// long, so for short K only shapes with two workgroups per CU are considered
// (one is in its K loop while the other stores), and for very short K, where
// the kernel is a stream of stores, only the small shapes.
//   Layers with few tiles come first.  A workgroup alone on its compute unit has nothing to hide its round trips behind: with
// two stages of whole lines every K step waits for the one it requested, 1400 clocks of a 128x64 step; with three stages the
// step takes what LDS needs, 24 KB written at 62 bytes per clock, 48 read at 235 and some 180 clocks of barrier, 770 (a fourth
// stage changes nothing).  Three stages: 64x64 tiles as long as they bring 1.5 workgroups per compute unit, or 2.25 where 128x64
// tiles would start a second round; else 128x64 tiles that fill one round at most; else, from K of 1024 bytes on, 128x128 tiles
// that do.  Two exceptions keep the tile that such sizes have always had, by which tests name them: layers of four 128x64 tiles
// or fewer, where 64x64 makes no difference (257 x 48 x 112 5.2 us with either, 130 x 36 x 64 4.6 / 4.9, 225 x 44 x 432 (3x3)
// 7.3 / 7.6), and linear layers between 4/5 of a round of 128x128 tiles and 7/4 of one of 128x64 tiles, which lose 0.5 to 1.6 us
// with the latter (128x128 / 128x64: 4728 x 768 x 3072 19.8 / 21.3, 7000 x 512 x 1536 13.9 / 14.4, 13500 x 256 x 2048 16.1 / 16.4).
// us, chosen by price / 64x64 / 128x64 / 128x128 with three stages: 2450 x 512 x 2048 12.6 / 8.7 / 9.7 / 12.4, 2000 x 768 x 3072
// 17.3 / 11.8 / 12.0 / 14.9, 128 x 4096 x 4096 20.6 / 11.6 / 13.5 / 17.8, 32 x 512 x 512 5.1 / 4.2 / 5.0 / 6.0, 4480 x 512 x 1024
// 9.6 / 8.5 / 9.0 / 9.2, 4096 x 512 x 2048 13.0 / 11.4 / 9.8 / 12.2, 4096 x 768 x 3072 20.4 / 18.6 / 18.8 / 17.1, 12544 x 256 x
// 2304 (3x3) 18.2 / 21.2 / 17.8 / 16.7; 4096 x 768 x 768 8.5 with all of them; and up to a whole round of
// 128x128 tiles (another run) 4992 x 768 x 3072 22.5 / 24.1 / 22.0 / 20.2, 8000 x 512 x 1536 16.1 / 17.1 / 17.1 / 16.0, 10500 x 260 x
// 2448 (3x3) 21.9 / 26.1 / 21.1 / 19.9.
//   The 128-row ones of these have eight waves: two on a SIMD, one at its operand reads while the other multiplies (four waves /
// eight, us: 4096 x 768 x 3072 20.0 / 18.9, 3000 x 1024 x 4096 23.8 / 22.2, 12544 x 256 x 1024 11.8 / 11.4, 12544 x 256 x 2304 (3x3)
// 18.9 / 17.8, 6468 x 256 x 2304 (3x3) 14.5 / 13.6, 21560 x 128 x 1152 (3x3) 12.8 / 12.0; a fourth stage changes nothing).
static int choose_shape(int64_t M, int32_t N, int64_t kp, bool conv3x3)
{
    const int64_t cu = compute_units(), t64 = ((M + 63) / 64) * ((N + 63) / 64), t128x64 = ((M + 127) / 128) * ((N + 63) / 64),
                  t128 = ((M + 127) / 128) * ((N + 127) / 128);
    if (t128x64 > 4 && (2 * t64 <= 3 * cu || (t128x64 > cu && 4 * t64 <= 9 * cu))) return kDeepSmall;
    if (t128x64 <= cu) return kDeepMid;
    if (t128 <= cu && kp >= 1024) return !conv3x3 && 5 * t128 > 4 * cu && 4 * t128x64 <= 7 * cu ? kDeepMid : kDeepLarge;
    int best = 0;
    double best_cost = 0.0;
    for (int i = 0; i < kNumShapes; ++i) {
        const TileShape &sh = kShapes[i];
        const int64_t tiles = ((M + sh.bm - 1) / sh.bm) * (int64_t)((N + sh.bn - 1) / sh.bn);
        if (sh.waves == 8) {
            // eight waves on one large tile with whole-line K steps: linear layers with a long K.  (With K = 768 they win
            // by 5-10 % when timed alone, where the fp32 output stays in the last-level cache, and lose as much
            // inside an encoder layer, where it goes to HBM and the shapes with two workgroups per compute unit
            // hide more of the store behind the other workgroup's K loop.)  One tile of 256x192 per compute unit, or as
            // much work on fewer compute units: an encoder layer whose second feed-forward layer makes fewer tiles, us
            // with the large tile / with 128x192 or 256x128: 256x192, 176 tiles 464 / 454, 192 485 / 476, 224 496 / 494,
            // 240 521 / 520; 256x256, 200 tiles 619 / 616, 204 663 / 665, 224 882 / 910, 240 727 / 734, 252 753 / 760.
            if (conv3x3 || kp < 2048 || tiles * sh.bm * sh.bn < (int64_t)compute_units() * 256 * 192) continue;
        }
        if (sh.bm * sh.bn > 128 * 128 && kp < 512) continue;       // store bound: many small workgroups in flight
        const int64_t slots = compute_units() * (int64_t)sh.resident;
        const int64_t rounds = (tiles + slots - 1) / slots;
        double cost = (double)rounds * sh.resident * sh.bm * sh.bn * sh.penalty;
        // K of a few steps: the kernel is a stream of fp32 stores, and the more workgroups a CU holds the
        // better they overlap (12544 x 1024 x 256: 128x64 with four per CU 17 us, 128x128 with two 21 us)
        if (kp < 512) cost *= 1.0 + 0.15 * (4 - sh.resident);
        if (best_cost == 0.0 || cost < best_cost) {
            best_cost = cost;
            best = i;
        }
    }
    return best;
}

// K steps in LDS of the kernel that an int8 layer of these sizes runs with (gemm_tile names its output tile).
int gemm_stages(int64_t M, int32_t N, int64_t kp, bool conv3x3)
{
    if (N <= 32) return stages_for(64);
    const int i = choose_shape(M, N, kp, conv3x3);
    return i >= kNumShapes ? 3 : stages_for(kShapes[i].bk);
}

// Output tile and K step of an int8 layer of these sizes, for tests that have to reach a certain shape.
void gemm_tile(int64_t M, int32_t N, int64_t kp, bool conv3x3, int32_t *rows, int32_t *cols, int32_t *k_step)
{
    const TileShape narrow = {128, 32, 64, 0, 4, 0.0}, &sh = N <= 32 ? narrow : kShapes[choose_shape(M, N, kp, conv3x3)];
    *rows = sh.bm;
    *cols = sh.bn;
    *k_step = sh.bk;
}

// The float32 reference precision (bound by its matrix instructions): three tile shapes, chosen by how many tiles the output
// makes.
static hipError_t launch_float32(const GemmArgs &g, hipStream_t st)
{
    const int64_t t128 = ((g.M + 127) / 128) * (int64_t)((g.N + 127) / 128);
    if (t128 >= 512) return launch_variant<128, 128, 2, 2, 64, 2>(g, st);
    return launch_variant<128, 64, 2, 2, 64, 2>(g, st);
}

bool gemm_layernorm_fusable(int32_t N, const void *ln_out, const void *ln_res, const void *gamma, const void *beta)
{
    auto ok16 = [](const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
    return N >= 4 && N <= 768 && (N & 3) == 0 && ln_out && ln_res && ok16(ln_out) && ok16(ln_res) && ok16(gamma) && ok16(beta);
}

// Which layers make their sums twice (GemmArgs::gelu_pass): a second set of sums instead of an fp32 tensor written and read back,
// as long as they are short: up to 1024 products no batch loses by it, beyond that small ones do (large ones would still gain).  An
// encoder layer with three launches / this way, us, tokens x hidden: 4096 x 512 107 / 103, 4096 x 768 147 / 144; 1024 x 1024 85.6 / 86.4,
// 2048 x 1024 121.6 / 121.6, 4096 x 1024 178 / 174, 16384 x 1024 657 / 635; 1024 x 1280 135 / 142, 4096 x 1280 298 / 289, 16384 x 1280
// 996 / 965, 4096 x 1536 374 / 356.  (Rows of codes, padded to 16, stay below 2^22 bytes: launch_gemm_i8 addresses 256 of them with 31 bits.)
bool gemm_gelu_codes(int64_t M, int32_t N, int64_t kp) { return M > 0 && N > 32 && N <= (1 << 22) - 16 && kp <= 1024; }

hipError_t launch_gemm_i8(const GemmArgs &g, hipStream_t st)
{
    if (g.ln_out) {
        // a linear layer and the layer norm of its rows in one launch: 64 whole rows per workgroup
        if (g.et != 0 || g.conv3x3 || g.act || g.res_q || g.q_out || g.acc_out || g.zp_in || g.zp_res) return hipErrorInvalidValue;
        if (!gemm_layernorm_fusable(g.N, g.ln_out, g.ln_res, g.ln_gamma, g.ln_beta)) return hipErrorInvalidValue;
        return launch_variant<64, 768, 1, 8, 64, 0, kLayerNorm>(g, st);
    }
    if (g.gelu_pass) {
        if (g.et != 0 || g.conv3x3 || g.act || g.res_q || g.acc_out || g.zp_in || g.zp_res || !gemm_gelu_codes(g.M, g.N, g.kp))
            return hipErrorInvalidValue;
        if (g.gelu_pass == 1) return g.absmax_out && g.gelu_neg ? launch_gelu<kGeluMax>(g, st) : hipErrorInvalidValue;
        // (256 rows of codes are addressed with 31 bits)
        if (!g.q_out || (g.q_ld & 15) || g.q_ld < g.N || g.q_ld >= (1 << 22) || !g.gelu_max || !g.gelu_neg || !g.gelu_scale) return hipErrorInvalidValue;
        return launch_gelu<kGeluCodes>(g, st);
    }
    if (g.et == 1 || g.et == 2) {
        if (g.q_out || g.absmax_out) return hipErrorInvalidValue;
        if (g.et == 2) return g.N <= 32 ? launch_variant<128, 32, 4, 1, 64, 2>(g, st) : launch_float32(g, st);
        // float16: a byte of K costs what one of int8 does, in the matrix cores and on the way to them, so the same choice
        // (128x128 and 128x64 tiles with 64-byte steps only / now, us: 4096 x 2304 x 768 29 / 26, 4096 x 768 x 3072 38 / 28,
        // 12544 x 256 x 1024 17 / 13.7, 12544 x 256 x 256 (3x3) 33 / 26)
        if (g.N <= 32) return launch_variant<128, 32, 4, 1, 64, 1>(g, st);
        return launch_shape<1>(choose_shape(g.M, g.N, g.kp, g.conv3x3), g, st);
    }
    if (g.conv3x3 && g.cp == 16 && g.N <= 32 && !g.zp_in) {   // (symmetric codes only)
        const int64_t blocks = (g.M + 127) / 128;
        if (blocks <= 0) return hipSuccess;
        if (g.M >= (1LL << 31)) return hipErrorInvalidValue;            // 32-bit pixel arithmetic in the kernel
        return launch_k(EGERIA_KERNEL_GEMM, conv3x3_c16_kernel, dim3((unsigned)blocks), dim3(256), 0, st, g);
    }
    if (g.N <= 32) return launch_variant<128, 32, 4, 1, 64>(g, st);
    return launch_shape<0>(choose_shape(g.M, g.N, g.kp, g.conv3x3), g, st);
}

}  // namespace egeria
