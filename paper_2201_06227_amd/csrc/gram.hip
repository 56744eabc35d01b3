// Training plasticity P = SP_loss(A_T, A_R) (Section 4.2, Eq. 1 of the paper;
// the loss is the cited similarity-preserving loss):
//   Gt = Q Q^T (b x b) for Q = A_T and Q = A_R reshaped to [b, D],
//   rows of Gt divided by their L2 norm, P = ||G_T - G_R||_F^2 / b^2.
//
// P is a squared *difference* of two nearly equal matrices, so forming both
// Gram matrices in fp32 and subtracting loses most of the digits once the
// layer has converged.  The kernels therefore contract
//   W = (T - R)(T + R)^T + (T + R)(T - R)^T     and     B = R R^T
// (T, R the two activations): the Gram difference is exactly W / 2, it is
// obtained to fp32 *relative* accuracy, and G_T's Gram is recovered as
// B + W / 2 in fp64 in the finaliser.
//
// Kernel 1 (gram_kernel): split-K over D.  Samples come in blocks of 32.  A
//   workgroup owns one chunk of D and one pair (p, q) of blocks - both diagonal
//   blocks of W and B and the off-diagonal ones for b <= 64, else one of the
//   3 or 6 pairs with at most one diagonal block - or the single block of b <= 32.
//   Both matrices are symmetric: only blocks p <= q are contracted (7 block
//   products instead of 8 for b = 64, 26 instead of 32 for b = 128).
//   Every fp32 product is formed exactly on the bf16 matrix cores: an fp32
//   value is the sum of three bf16 values (8 + 8 + 8 significant bits, obtained
//   by truncation and exact subtraction), so x * y = sum of nine bf16 x bf16
//   products, each exact in fp32; the six largest are issued
//   (v_mfma_f32_32x32x16_bf16, fp32 accumulation), the three dropped ones sum
//   to less than 2^-21 of the product.  Six bf16 MFMAs cost 0.375 of the eight
//   fp32 MFMAs they replace.
//   Eight waves split the chunk by slabs of 16 features, each with all of the
//   pair's products in its accumulators: a wave streams its own slabs, no
//   barrier until the end.  The raw values go from global memory straight into
//   the wave's stage in LDS (rows of 64 bytes, 16-byte units xor-rotated
//   by the row: conflict-free) and are read back once, in the lane layout of
//   the matrix instruction (row l % 32, eight features of half l / 32), which
//   is the same for both operands; T - R, T + R and the three-way splits are
//   formed in registers, once per value and pair, and never return to LDS.
//   What bounds it: HBM for large D - the stream of 103 MB at b = 64, D = 200704 takes 16 us by itself (5.6 TB/s), the
//   matrix and vector work 12 us beside it, filling and draining six slabs per wave, the final sum over the waves (3 us)
//   and the launch the rest of 27 us - and the L2 -> LDS path for b > 64, where a block of samples is read by up to three
//   pairs.  Before (one 64x64 tile of both products, four waves, operands passed through LDS as nine bf16 planes: 18
//   bytes of LDS writes and 48 of reads per value pair, and one wave per SIMD, which issues a vector instruction
//   every 5 clocks where two waves issue one every 2.9): per score, both launches, us: b = 64, D = 200704 43 -> 34;
//   b = 100, D = 62720 (bf16 T) 54 -> 33; b = 128, D = 16384 27 -> 22; b = 32, D = 98304 (bf16 T) 17.6 -> 13.5.  Rows of
//   odd length in bf16, which are filled element by element: b = 64, D = 200705 124 -> 37, b = 32, D = 98305 31 -> 21.
//   The eight waves' accumulators are added through
//   LDS at the end; the diagonal blocks of W are symmetrised there.
//   Partials are [nsplit][2][b][b] fp32 (W and B, whole rows).
// Kernel 2 (sp_finalize): workgroups own parts of the rows of the b x b
//   matrices.  They sum W and B over the chunks in fp64 and reduce their columns
//   to the sums from which a row's norms and its share of the squared difference
//   follow; the last workgroup to finish adds the shares in index order and writes P.
// A small problem of one block (b <= 32, D <= 512) is finished by kernel 1 itself,
// whose one workgroup has both matrices in LDS: one launch less.
//   Results are bit-reproducible from call to call.
#include "common.hpp"
#include <mutex>
#include <type_traits>

namespace egeria {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr int kSlab = 16;                // features of one matrix instruction
constexpr int kGramWaves = 8;
// LDS of a workgroup: the waves' stages, then the reduction (two blocks of eight waves, their sums) and, for a score
// that the workgroup finishes itself, both matrices.  Kept near 72 KB: other streams' kernels share the CU.
constexpr int kGramReduce = (2 * kGramWaves * 1024 + 2 * 32 * 33) * 4;
constexpr int kGramFused = kGramReduce + 2 * 32 * 33 * 4;
// Slabs (of 16 features) up to which one workgroup does the whole score of at most 32 samples, where slabs are loaded
// straight into LDS and where they are filled element by element (one per wave: every further one is a round trip of
// its own).  Its waves take the slabs one after the other, which soon costs more than the finaliser's launch, us with /
// without: b = 32, D = 256 9.4 / 11, 512 10.4 / 11, 770 12.3 / 11, 1024 12.8 / 11; bf16 T with odd D, D = 65 9.5 /
// 11.5, 129 11.1 / 11.6, 257 12.9 / 11.5, 1001 23 / 11.5.  Two blocks of samples never pay (three products and their
// sums over the waves in one workgroup): b = 33, D = 8 16.0 / 12.5; b = 64, D = 1024 28.7 / 13.6.
constexpr int kFusedSlabs = 32, kFusedFillSlabs = 8;

struct GramPlan {
    int nb;          // blocks of 32 samples
    int npair;       // workgroups (pairs of blocks) per chunk
    int64_t nslab;   // slabs of 16 features in D
    int64_t spc;     // slabs per chunk
    int nsplit;      // chunks of D
    int turns;       // (chunks per XCD) x (pairs)
    int fused;       // one chunk, finished by its workgroup
    int direct;      // whole slabs are loaded straight into LDS (else element by element)
};

static GramPlan plan_gram(int32_t b, int64_t D)
{
    GramPlan p{};
    p.nb = (b + 31) / 32;
    p.npair = p.nb <= 2 ? 1 : (p.nb == 3 ? 3 : 6);
    const int64_t nslab = (D + kSlab - 1) / kSlab;
    p.nslab = nslab;
    // about one workgroup per CU: for b > 32 the registers of its eight waves (160 to 240 per lane) leave no room for a
    // second one, and for smaller b the partials of twice as many cost more than they hide: b = 32, D = 98304 13.2 us
    // against 15.7, b = 64, D = 200704 34 against 44.  At least one slab for every wave.  (The pairs of a chunk share an
    // XCD, so the CUs of an XCD bound the chunks dealt to it.)
    int64_t want = 8 * (compute_units() / 8 / p.npair);
    const int64_t cap = (nslab + kGramWaves - 1) / kGramWaves;
    if (want > cap) want = cap;
    if (want < 1) want = 1;
    p.spc = (nslab + want - 1) / want;
    p.nsplit = (int)((nslab + p.spc - 1) / p.spc);
    p.turns = (p.nsplit + 7) / 8 * p.npair;
    return p;
}

// workspace of the metric: [counter | four sums per workgroup of the finaliser | partials [nsplit][2][b][b] (W, B)]
static int fin_parts(int b);
constexpr int kFinSums = 4;
static size_t off_sums() { return 256; }
static size_t off_partials(int32_t b) { return 256 + align_up((size_t)b * fin_parts(b) * kFinSums * sizeof(double), 256); }

size_t plasticity_partial_bytes(int32_t b, int64_t D)
{
    GramPlan p = plan_gram(b, D);
    return off_partials(b) + align_up((size_t)p.nsplit * 2 * (size_t)b * b * sizeof(float), 256);
}

// The three bf16 parts of eight fp32 values, packed as the 16-byte operand unit
// of the bf16 MFMA.  hi = the value truncated to bf16, mid = the remainder
// truncated, lo = what is left; both subtractions are exact and lo has at most
// eight significant bits, so hi + mid + lo == x exactly.
struct Split8 {
    v4u part[3];     // hi, mid, lo
};
__device__ __forceinline__ uint32_t pack_hi16(float x1, float x0)
{
    return __builtin_amdgcn_perm(__float_as_uint(x1), __float_as_uint(x0), 0x07060302u);
}
// values 2 e and 2 e + 1 of the eight
__device__ __forceinline__ void split_pair(float x0, float x1, int e, Split8 &o)
{
    const float r0 = x0 - __uint_as_float(__float_as_uint(x0) & 0xffff0000u);
    const float r1 = x1 - __uint_as_float(__float_as_uint(x1) & 0xffff0000u);
    const float l0 = r0 - __uint_as_float(__float_as_uint(r0) & 0xffff0000u);
    const float l1 = r1 - __uint_as_float(__float_as_uint(r1) & 0xffff0000u);
    o.part[0][e] = pack_hi16(x1, x0);
    o.part[1][e] = pack_hi16(r1, r0);
    o.part[2][e] = pack_hi16(l1, l0);
}
// acc += a b^T with a in NA parts and b in NB parts (three for fp32, one for a value that is a bf16 value), smallest
// partial products first.  Of nine the three smallest are left out: mid lo and lo mid, each below 2^-22 of the product
// (mid < 2^-7 and lo < 2^-15 of the value), and lo lo.  `after` runs behind every instruction.
template <int NA, int NB, typename F>
__device__ __forceinline__ void mma_parts(const Split8 &a, const Split8 &b, v16f &acc, F after)
{
#pragma unroll
    for (int order = 2; order >= 0; --order)
#pragma unroll
        for (int i = order; i >= 0; --i)
            if (i < NA && order - i < NB) {
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a.part[i]), __builtin_bit_cast(v8bf, b.part[order - i]), acc, 0, 0, 0);
                after();
            }
}

// One tensor's share of a stage: a block of 32 samples x 16 features, as read from memory.
template <int DT>
struct Tile {
    static constexpr int kRow = kSlab * (DT == 0 ? 4 : 2);       // bytes per row
    static constexpr int kBytes = 32 * kRow;
    static constexpr int kUnits = kRow / 16;                     // 16-byte units per row: 4 or 2
    static constexpr int kLoads = kBytes / 1024;                 // load instructions of a wave
    static constexpr int kRowsPerLoad = 64 / kUnits;
    // unit u of row r lies at slot u ^ ((r / (16 / kUnits)) % kUnits) of its row
    static __device__ __forceinline__ int slot(int r, int u) { return u ^ ((r / (16 / kUnits)) % kUnits); }
};

// (fmax would turn the NaN of a non-finite activation into 0)
__device__ __forceinline__ double not_below_zero(double v) { return v < 0.0 ? 0.0 : v; }

// || g / max(|g|, 1e-12) - a / max(|a|, 1e-12) ||^2 for g = a + e from aa = |a|^2, gg = |g|^2, ae = a.e, ee = |e|^2.
// single: rows of one entry (b = 1), which are parallel or opposite; each of the four sums is rounded, so sin^2 of
// the angle would come out as some 1e-16 instead of 0.
__device__ __forceinline__ double row_share(double aa, double gg, double ae, double ee, bool single)
{
    const double nr = sqrt(aa), nt = sqrt(gg);
    if (nr < 1e-12 || nt < 1e-12) {
        const double r = nr < 1e-12 ? 1e-12 : nr, t = nt < 1e-12 ? 1e-12 : nt;
        // |a u + e / t|^2: the large parts of the two rows leave each other in u (0 where both norms are clamped)
        const double u = (r - t) / (t * r);
        return not_below_zero(aa * u * u + 2.0 * (ae * u) / t + ee / (t * t));
    }
    const double c = (aa + ae) / (nr * nt);
    const double s2 = single ? 0.0 * c : not_below_zero(aa * ee - ae * ae) / (aa * gg);      // (0 * NaN stays NaN)
    return c > 0.0 ? 2.0 * s2 / (1.0 + c) : 2.0 - 2.0 * c;
}

// KIND 0: one block (b <= 32); 1: two blocks and all three block products of W and B (b <= 64); 2: two of three
// or four blocks, the off-diagonal products and those of the first block's diagonal if the pair's turn says so.
// LONG: rows whose byte offsets within a block of samples do not fit the 31 bits of a buffer offset (2^24 features and
// more).  Each lane then addresses its 16 bytes with 64 bits; samples beyond b and slabs past the chunk's end repeat valid
// ones (rows beyond b only reach entries that are never stored, a slab past the end is not contracted).  Filled
// element by element, a round trip per slab, 16 x 2^24 fp32 took 2150 us; this form takes 558, 3.9 TB/s.
template <int KIND, int TDT, int RDT, bool LONG>
__global__ __launch_bounds__(64 * kGramWaves, 2) void gram_kernel(const void *__restrict__ at, const void *__restrict__ ar,
                                                                  int b, int64_t D, GramPlan p, int turn0, float *__restrict__ part,
                                                                  uint32_t *__restrict__ counter, float *__restrict__ p_out)
{
    constexpr int NBLK = KIND == 0 ? 1 : 2;                      // blocks of samples
    constexpr int NACC = KIND == 0 ? 1 : (KIND == 1 ? 3 : 2);    // accumulator blocks per matrix: [diag p][off][diag q]
    using TT = Tile<TDT>;
    using TR = Tile<RDT>;
    constexpr int kStage = NBLK * (TT::kBytes + TR::kBytes);
    constexpr int NLD = NBLK * (TT::kLoads + TR::kLoads);        // load instructions of a slab
    static_assert(kGramWaves * kStage <= kGramReduce, "the stages must fit the reduction's LDS");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    // consecutive workgroup ids land on different XCDs: all pairs of one chunk go to the same XCD so that its L2
    // serves the re-reads of that chunk
    const int turn = turn0 + (blockIdx.x >> 3);
    const int chunk = (turn / p.npair) * 8 + (blockIdx.x & 7), pair = turn % p.npair;
    if (blockIdx.x == 0 && threadIdx.x == 0) *counter = 0u;      // ticket of the finaliser
    if (chunk >= p.nsplit) return;
    // pairs of four blocks: (0,1) (1,2) (2,3) (3,0) with the first one's diagonal, (0,2) (1,3) without;
    // of three: (0,1) (1,2) (2,0), each with a diagonal
    const int bp = KIND == 2 ? (pair < p.nb ? pair : pair - p.nb) : 0;
    const int bq = KIND == 2 ? (pair < p.nb ? (pair + 1 == p.nb ? 0 : pair + 1) : bp + 2) : 1;
    const bool diag_p = KIND != 2 || pair < p.nb;
    using slab_t = std::conditional_t<LONG, int64_t, int>;
    const slab_t spc = (slab_t)p.spc, nslab = (slab_t)p.nslab;
    const slab_t slab0 = chunk * spc;
    const slab_t slab1 = slab0 + spc < nslab ? slab0 + spc : nslab;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31, h = lane >> 5;
    uint8_t *stage = lds + wave * kStage;
    const uint32_t stage0 = (uint32_t)(uintptr_t)(lds_byte *)stage;

    // ---- a slab into the wave's stage: [T block p][T block q][R block p][R block q].  One load instruction of the wave
    // fills 1 KiB; which 16 bytes a lane fetches for its slot is free, hence the rotation of the units.  Samples
    // beyond b are given an offset outside the buffer and arrive as zeros.
    constexpr uint32_t kOob = 0x80000000u;
    auto descriptor = [&](const void *base, int64_t row, int es) {
        const uint64_t a = (uint64_t)base + (uint64_t)(row * D * es);
        v4i d;
        d[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
        d[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32) & 0xffff);
        d[2] = 0x7fffffff;                                       // (rows and features are checked here, not by the extent)
        d[3] = 0x00020000;
        return d;
    };
    v4i rt[NBLK], rr[NBLK];
#pragma unroll
    for (int k = 0; k < NBLK; ++k) {
        rt[k] = descriptor(at, 32 * (k == 0 ? bp : bq), TDT == 0 ? 4 : 2);
        rr[k] = descriptor(ar, 32 * (k == 0 ? bp : bq), RDT == 0 ? 4 : 2);
    }
    auto load_tile = [&](auto dt_c, const v4i &rsrc, const void *base, int blk, slab_t slab, bool ok, uint32_t dst, int i) {
        constexpr int DT = decltype(dt_c)::value;
        using T = Tile<DT>;
        const int row = lane / T::kUnits, unit = (lane % T::kUnits) ^ ((row / (16 / T::kUnits)) % T::kUnits);
        const int rl = i * T::kRowsPerLoad + row;
        if constexpr (LONG) {
            const int64_t r64 = 32 * blk + rl < b ? 32 * blk + rl : b - 1;
            load_to_lds_b128((const char *)base + r64 * D * (DT == 0 ? 4 : 2) + (ok ? slab : slab0) * T::kRow + unit * 16, dst + i * 1024);
            return;
        }
        const uint32_t off = ok && 32 * blk + rl < b ? (uint32_t)rl * (uint32_t)(D * (DT == 0 ? 4 : 2)) + (uint32_t)(slab * T::kRow + unit * 16) : kOob;
        load_to_lds_b128(rsrc, dst + i * 1024, off);
    };
    // element by element, with zeros beyond b and D (the last slab of a ragged D; rows that 4-byte accesses cannot address)
    auto fill_tile = [&](auto dt_c, const void *base, int blk, slab_t slab, uint8_t *dst) {
        constexpr int DT = decltype(dt_c)::value;
        using T = Tile<DT>;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int rl = i * 4 + (lane >> 4), f = lane & 15;
            const int64_t row = 32 * blk + rl, k = (int64_t)slab * kSlab + f;
            const bool ok = row < b && k < D;
            const int64_t idx = ok ? row * D + k : 0;
            if (DT == 0) {
                const float v = ((const float *)base)[idx];
                *(float *)(dst + rl * T::kRow + T::slot(rl, f >> 2) * 16 + (f & 3) * 4) = ok ? v : 0.0f;
            } else {
                const uint16_t v = ((const uint16_t *)base)[idx];
                *(uint16_t *)(dst + rl * T::kRow + T::slot(rl, f >> 3) * 16 + (f & 7) * 2) = ok ? v : (uint16_t)0;
            }
        }
    };
    using ct = std::integral_constant<int, TDT>;
    using cr = std::integral_constant<int, RDT>;
    const slab_t last_direct = p.direct ? (slab_t)(D / kSlab) : 0;   // slabs below this one are loaded straight into LDS
    // request q of the NLD of a slab (a slab past the end: no traffic, zeros)
    auto request_one = [&](slab_t slab, slab_t end, int q) {
        constexpr int nt = NBLK * TT::kLoads;
        if (q < nt) {
            const int k = q / TT::kLoads;
            load_tile(ct{}, rt[k], at, k == 0 ? bp : bq, slab, slab < end, stage0 + k * TT::kBytes, q % TT::kLoads);
        } else {
            const int k = (q - nt) / TR::kLoads;
            load_tile(cr{}, rr[k], ar, k == 0 ? bp : bq, slab, slab < end, stage0 + NBLK * TT::kBytes + k * TR::kBytes, (q - nt) % TR::kLoads);
        }
    };
    auto request = [&](slab_t slab, slab_t end) {
#pragma unroll
        for (int q = 0; q < NLD; ++q) request_one(slab, end, q);
    };
    auto fill = [&](slab_t slab) {
        uint8_t *dst = stage;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // the slab before has been read
#pragma unroll
        for (int k = 0; k < NBLK; ++k, dst += TT::kBytes) fill_tile(ct{}, at, k == 0 ? bp : bq, slab, dst);
#pragma unroll
        for (int k = 0; k < NBLK; ++k, dst += TR::kBytes) fill_tile(cr{}, ar, k == 0 ? bp : bq, slab, dst);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
    auto read8 = [&](auto dt_c, const uint8_t *tile, float (&x)[8], v4u &bits) {
        constexpr int DT = decltype(dt_c)::value;
        using T = Tile<DT>;
        const uint8_t *row = tile + r * T::kRow;
        if (DT == 0) {
            const float4 a = *(const float4 *)(row + T::slot(r, 2 * h) * 16), c = *(const float4 *)(row + T::slot(r, 2 * h + 1) * 16);
            x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
            x[4] = c.x; x[5] = c.y; x[6] = c.z; x[7] = c.w;
        } else {
            const v4u a = *(const v4u *)(row + T::slot(r, h) * 16);
            bits = a;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[2 * e] = __uint_as_float(a[e] << 16);
                x[2 * e + 1] = __uint_as_float(a[e] & 0xffff0000u);
            }
        }
    };

    v16f accW[NACC], accB[NACC];
#pragma unroll
    for (int k = 0; k < NACC; ++k)
#pragma unroll
        for (int i = 0; i < 16; ++i) { accW[k][i] = 0.0f; accB[k][i] = 0.0f; }

    // One slab of this wave.  Its raw values and the parts of R are in registers; T's parts are the raw bits where T is
    // bf16 (then W / 2 = D T^T + R D^T is what is summed: D T^T takes three exact partial products and S is not needed).
    constexpr bool TF = TDT == 1;
    constexpr int NR = RDT == 1 ? 1 : 3, NX = TF ? 1 : 3, NY = TF ? NR : 3;
    struct Raw {
        float t[NBLK][8], r[NBLK][8];
        v4u tbits[NBLK];
    };
    auto read_raw = [&](Raw &x) {
#pragma unroll
        for (int k = 0; k < NBLK; ++k) {
            read8(ct{}, stage + k * TT::kBytes, x.t[k], x.tbits[k]);
            v4u unused;
            read8(cr{}, stage + NBLK * TT::kBytes + k * TR::kBytes, x.r[k], unused);
        }
    };
    // The splits come in pieces of one pair of values: piece 4 k + e of block k.
    constexpr int kPieces = 4 * NBLK;
    auto split_r = [&](const Raw &x, int piece, Split8 (&rp)[NBLK]) {
        const int k = piece >> 2, e = piece & 3;
        split_pair(x.r[k][2 * e], x.r[k][2 * e + 1], e, rp[k]);
    };
    // D, and the factor that D multiplies: S = T + R, or T itself
    auto split_d = [&](const Raw &x, int piece, Split8 (&d)[NBLK]) {
        const int k = piece >> 2, e = piece & 3;
        split_pair(x.t[k][2 * e] - x.r[k][2 * e], x.t[k][2 * e + 1] - x.r[k][2 * e + 1], e, d[k]);
    };
    auto split_x = [&](const Raw &x, int piece, Split8 (&o)[NBLK]) {
        const int k = piece >> 2, e = piece & 3;
        if constexpr (TF) o[k].part[0][e] = x.tbits[k][e];
        else split_pair(x.t[k][2 * e] + x.r[k][2 * e], x.t[k][2 * e + 1] + x.r[k][2 * e + 1], e, o[k]);
    };
    auto nothing = [] {};
    auto run = [&](auto diag_c) {
        constexpr bool DG = decltype(diag_c)::value;             // the first block's diagonal products belong to this pair
        constexpr int nRR = NR == 3 ? 6 : 1, nDX = NX == 3 ? 6 : 3, nYD = NY == 3 ? 6 : 3;   // partial products of each kind
        constexpr int kDiag = (DG ? 1 : 0) + (NACC == 3 ? 1 : 0);
        constexpr int mfB = nRR * ((NBLK - 1) + kDiag), mfW = (nDX + nYD) * (NBLK - 1) + kDiag * (nDX + (TF ? nYD : 0));
        auto products_b = [&](const Split8 (&rp)[NBLK], auto after) {
            if constexpr (NBLK == 2) mma_parts<NR, NR>(rp[0], rp[1], accB[1], after);
            if constexpr (DG) mma_parts<NR, NR>(rp[0], rp[0], accB[0], after);
            if constexpr (NACC == 3) mma_parts<NR, NR>(rp[1], rp[1], accB[2], after);
        };
        auto products_w = [&](const Split8 (&rp)[NBLK], const Split8 (&d)[NBLK], const Split8 (&x)[NBLK], auto after) {
            if constexpr (NBLK == 2) mma_parts<3, NX>(d[0], x[1], accW[1], after);
            if constexpr (DG) {
                mma_parts<3, NX>(d[0], x[0], accW[0], after);
                if constexpr (TF) mma_parts<NR, 3>(rp[0], d[0], accW[0], after);
            }
            if constexpr (NBLK == 2) {
                if constexpr (TF) mma_parts<NR, 3>(rp[0], d[1], accW[1], after);
                else mma_parts<3, 3>(x[0], d[1], accW[1], after);
            }
            if constexpr (NACC == 3) {
                mma_parts<3, NX>(d[1], x[1], accW[2], after);
                if constexpr (TF) mma_parts<NR, 3>(rp[1], d[1], accW[2], after);
            }
        };
        // slabs first, first + 8, ... of the chunk: neighbouring waves take neighbouring slabs, i.e. the two halves
        // of a cache line at about the same time
        const slab_t first = slab0 + wave;
        const slab_t end = slab1 < last_direct ? slab1 : last_direct;
        const slab_t n = first < end ? (end - first + kGramWaves - 1) / kGramWaves : 0;
        if (n > 0) {
            // the stage is free again as soon as its raw values are in registers: one slab in registers, the next landing
            // (two stages per wave, i.e. 128 KB in flight per CU instead of 64, made no difference)
            request(first, end);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            Raw cur;
            Split8 rp[NBLK];
            read_raw(cur);
#pragma unroll
            for (int k = 0; k < kPieces; ++k) split_r(cur, k, rp);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            slab_t ahead = first + kGramWaves;
            request(ahead, end);
            // Two steps per slab: the products of B beside the splits of D and S, the products of W beside the split of the
            // next slab's R and the requests for the slab after.  The pieces and the requests are placed between the
            // matrix instructions one by one: left to itself the compiler puts all of one kind first, and the two waves
            // of a SIMD, which start together, wait for the same pipe; a burst of requests holds the wave up.
            for (slab_t i = 0; i < n; ++i) {
                Split8 d[NBLK], x[NBLK], rn[NBLK];
                int m = 0;                                       // (a constant everywhere: the code is straight-line)
                constexpr int perB = (2 * kPieces + mfB - 1) / mfB;
                products_b(rp, [&] {
#pragma unroll
                    for (int q = m * perB; q < (m + 1) * perB && q < 2 * kPieces; ++q) {
                        if (q & 1) split_x(cur, q >> 1, x); else split_d(cur, q >> 1, d);
                    }
                    ++m;
                    __builtin_amdgcn_sched_barrier(0);
                });
                // the next slab has landed (past the last one: zeros, which nothing uses)
                ahead += kGramWaves;
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                read_raw(cur);
                m = 0;
                constexpr int lead = mfW > 8 ? 3 : 0, room = mfW - lead;     // the first instructions cover the LDS reads
                constexpr int perW = (kPieces + room - 1) / room, perL = (NLD + room - 1) / room;
                products_w(rp, d, x, [&] {
                    if (m == lead) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the stage has been read
                    if (m >= lead) {
                        const int j = m - lead;
#pragma unroll
                        for (int q = j * perL; q < (j + 1) * perL && q < NLD; ++q) request_one(ahead, end, q);
#pragma unroll
                        for (int q = j * perW; q < (j + 1) * perW && q < kPieces; ++q) split_r(cur, q, rn);
                    }
                    ++m;
                    __builtin_amdgcn_sched_barrier(0);
                });
#pragma unroll
                for (int k = 0; k < NBLK; ++k) rp[k] = rn[k];
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        // slabs that are filled element by element
        for (slab_t slab = first + n * kGramWaves; slab < slab1; slab += kGramWaves) {
            fill(slab);
            Raw cur;
            Split8 rp[NBLK], d[NBLK], x[NBLK];
            read_raw(cur);
#pragma unroll
            for (int k = 0; k < kPieces; ++k) { split_r(cur, k, rp); split_d(cur, k, d); split_x(cur, k, x); }
            products_b(rp, nothing);
            products_w(rp, d, x, nothing);
        }
    };
    if (diag_p) run(std::true_type{});
    else if constexpr (KIND == 2) run(std::false_type{});

    // ---- the eight waves' sums, one 32x32 block after the other through LDS (the stages are free; the halves of the
    // reduction area alternate, so a block costs two barriers).  Register i of lane l of a block is row
    // 8 (i / 4) + 4 (l / 32) + i % 4, column l % 32.
    float *red = (float *)lds;                                   // [2][waves][16][64]: this block's, the next one's
    float *sum = red + 2 * kGramWaves * 1024;                    // [2][32][33], padded rows
    float *fin = sum + 2 * 32 * 33;                              // fused: W and B, [2][32][33]
    const size_t nelem = (size_t)b * b;
    float *dst = part + (size_t)chunk * 2 * nelem;
    __syncthreads();                                             // every wave has read its last slab
    int turn_ = 0;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
#pragma unroll
        for (int k = 0; k < NACC; ++k) {
            // [diag p][off][diag q]; KIND 0 has the first one only
            if (k == 0 && !diag_p) continue;
            float *rd = red + (turn_ & 1) * kGramWaves * 1024, *sm = sum + (turn_ & 1) * 32 * 33;
            ++turn_;
#pragma unroll
            for (int i = 0; i < 16; ++i) rd[wave * 1024 + i * 64 + lane] = m == 0 ? accW[k][i] : accB[k][i];
            __syncthreads();
#pragma unroll
            for (int e0 = 0; e0 < 1024; e0 += 64 * kGramWaves) {
                const int e = e0 + tid, i = e >> 6;
                float v[kGramWaves];
#pragma unroll
                for (int w = 0; w < kGramWaves; ++w) v[w] = rd[w * 1024 + e];
                float t = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
                if (TF && m == 0) t *= 2.0f;                     // (exact)
                sm[(8 * (i >> 2) + 4 * h + (i & 3)) * 33 + r] = t;
            }
            __syncthreads();
            // whole rows out: block (p, p), (q, q), or (p, q) and its transpose (q, p)
            const int rowb = k == 2 ? bq : bp, colb = k == 0 ? bp : bq;
#pragma unroll
            for (int e0 = 0; e0 < 1024; e0 += 64 * kGramWaves) {
                const int e = e0 + tid, row = e >> 5, col = e & 31;
                const float a = sm[row * 33 + col], c = sm[col * 33 + row];
                const float v = k != 1 && !TF && m == 0 ? a + c : a;    // a diagonal block of (T - R)(T + R)^T: plus its transpose
                const int gr = 32 * rowb + row, gc = 32 * colb + col, tr = 32 * colb + row, tc = 32 * rowb + col;
                if (KIND == 0 && p.fused) {
                    fin[(m * 32 + row) * 33 + col] = v;
                } else {
                    if (gr < b && gc < b) dst[(size_t)m * nelem + (size_t)gr * b + gc] = v;
                    if (k == 1 && tr < b && tc < b) dst[(size_t)m * nelem + (size_t)tr * b + tc] = c;
                }
            }
        }
    }
    if constexpr (KIND == 0) {
        if (!p.fused) return;
        // the whole score: a wave per row, the row's columns in its lanes, shares added in index order
        __syncthreads();
        double *share = (double *)lds;                           // [32][4]
        constexpr int RW = 32 / kGramWaves;                      // rows of a wave, side by side: their sums are chains of exchanges
        double q[4][RW];
#pragma unroll
        for (int k = 0; k < RW; ++k) {
            const int i = wave + kGramWaves * k;
            const bool in = i < b && lane < b;
            const double a = in ? (double)fin[(32 + i) * 33 + (lane < b ? lane : 0)] : 0.0;
            const double e = in ? 0.5 * (double)fin[i * 33 + (lane < b ? lane : 0)] : 0.0, g = a + e;
            q[0][k] = a * a;
            q[1][k] = g * g;
            q[2][k] = a * e;
            q[3][k] = e * e;
        }
#pragma unroll
        for (int k = 0; k < RW; ++k)
#pragma unroll
            for (int m = 0; m < 4; ++m) q[m][k] = wave_sum<16>(q[m][k]);   // (32 columns: no exchange between the halves of the wave)
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < RW; ++k)
                if (wave + kGramWaves * k < b)
#pragma unroll
                    for (int m = 0; m < 4; ++m) share[4 * (wave + kGramWaves * k) + m] = q[m][k];
        }
        __syncthreads();
        if (wave == 0) {
            const double tot = wave_sum(lane < b ? row_share(share[4 * lane], share[4 * lane + 1], share[4 * lane + 2], share[4 * lane + 3], b == 1) : 0.0);
            if (lane == 0) *p_out = (float)(tot / ((double)b * (double)b));
        }
    }
}

// Workgroup (row i, part): columns part * CS .. + CS - 1 of row i.  Its threads form groups of CS lanes, a chunk of the
// partials each, lane j taking column j; W and B are summed over the chunks in fp64 (fixed assignment, fixed order).
// With a = row i of R R^T and e = half of row i of W (so a + e = row i of T T^T) the row's share of P,
// || (a + e) / |a + e| - a / |a| ||^2, follows from four sums over the columns: |a|^2, |a + e|^2, a.e and |e|^2, since
// it is 2 sin^2 / (1 + cos) of the angle between the two rows and sin^2 = (|a|^2 |e|^2 - (a.e)^2) / (|a|^2 |a + e|^2)
// without cancellation where e is small.  The last workgroup to finish adds the parts and the rows in index order.
// Bound by latency: launch, one round trip for the partials (which other XCDs wrote), one for the ticket.  One
// workgroup per row reading 256 chunks of 2 x 256 bytes took 8.5 us for b = 64 (64 of 256 CUs at work, three dependent
// row sums, a fence that writes the L2 back); this form takes 6.
constexpr int kFinThreads = 1024;
static int fin_columns(int b) { return b <= 32 ? 16 : 64; }      // CS
static int fin_parts(int b) { return (b + fin_columns(b) - 1) / fin_columns(b); }

// U: chunks that a thread requests together
template <int CS, int U>
__global__ __launch_bounds__(kFinThreads) void sp_finalize_kernel(const float *__restrict__ part, int nsplit, int b, int parts,
                                                                  double *__restrict__ sums, uint32_t *__restrict__ counter,
                                                                  float *__restrict__ p_out)
{
    constexpr int NW = kFinThreads / 64, G = kFinThreads / CS;
    __shared__ double sm[2][NW][CS];
    __shared__ uint32_t ticket_s;
    const int i = blockIdx.x / parts, pt = blockIdx.x % parts, t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int j = pt * CS + t % CS, grp = t / CS;
    const size_t nelem = (size_t)b * b, cstride = 2 * nelem;
    double aw = 0.0, ab = 0.0;
    const float *p = part + (size_t)i * b + (j < b ? j : b - 1);
    for (int c = grp; c < nsplit; c += U * G) {
        float vw[U], vb[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {                             // (unconditional: a chunk past the end reads the last one)
            const float *pc = p + (size_t)(c + u * G < nsplit ? c + u * G : nsplit - 1) * cstride;
            vw[u] = pc[0];
            vb[u] = pc[nelem];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (c + u * G < nsplit) {
                aw += (double)vw[u];
                ab += (double)vb[u];
            }
    }
    if constexpr (CS == 16) {
        aw += lane_xor<16>(aw);
        ab += lane_xor<16>(ab);
        aw += lane_xor<32>(aw);
        ab += lane_xor<32>(ab);
    }
    if (lane < CS) { sm[0][wave][lane] = aw; sm[1][wave][lane] = ab; }
    __syncthreads();
    if (wave == 0) {
        double q[kFinSums] = {0.0, 0.0, 0.0, 0.0};
        if (lane < CS && j < b) {
            double w = 0.0, a = 0.0;
#pragma unroll
            for (int k = 0; k < NW; ++k) { w += sm[0][k][lane]; a += sm[1][k][lane]; }
            const double e = 0.5 * w, g = a + e;                  // rows of R R^T: a, of T T^T: g
            q[0] = a * a;
            q[1] = g * g;
            q[2] = a * e;
            q[3] = e * e;
        }
#pragma unroll
        for (int k = 0; k < kFinSums; ++k) q[k] = wave_sum<CS / 2>(q[k]);
        if (lane == 0) {
            // device-scope stores (they bypass the XCD's L2), waited for before the ticket is taken: no cache write-back
#pragma unroll
            for (int k = 0; k < kFinSums; ++k)
                __hip_atomic_store(&sums[(size_t)blockIdx.x * kFinSums + k], q[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            ticket_s = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    if (ticket_s != gridDim.x - 1) return;
    double share = 0.0;
    if (t < b) {
        double q[kFinSums] = {0.0, 0.0, 0.0, 0.0};
        for (int k = 0; k < parts; ++k)
#pragma unroll
            for (int m = 0; m < kFinSums; ++m)
                q[m] += __hip_atomic_load(&sums[((size_t)t * parts + k) * kFinSums + m], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        share = row_share(q[0], q[1], q[2], q[3], b == 1);
    }
    __syncthreads();                                              // sm is free
    share = wave_sum(share);
    if (lane == 0) sm[0][wave][0] = share;
    __syncthreads();
    if (t == 0) *p_out = (float)((sm[0][0][0] + sm[0][1][0]) / ((double)b * (double)b));   // waves 0 and 1 hold the rows
}

hipError_t launch_plasticity(const void *a_t, egeria_dtype t_dt, const void *a_r, egeria_dtype r_dt,
                             int32_t b, int64_t D, float *p_out, void *ws_part, hipStream_t st, bool beside)
{
    GramPlan p = plan_gram(b, D);
    const int dev = current_device();
    if (dev < 0) return hipErrorInvalidDevice;
    uint32_t *counter = (uint32_t *)ws_part;
    double *sums = (double *)((char *)ws_part + off_sums());
    float *part = (float *)((char *)ws_part + off_partials(b));
    const int tcode = t_dt == EGERIA_BF16 ? 1 : 0, rcode = r_dt == EGERIA_BF16 ? 1 : 0;
    // straight into LDS: rows that start at 4-byte boundaries, which is what loads with the LDS modifier need
    p.direct = D * (tcode ? 2 : 4) % 4 == 0 && D * (rcode ? 2 : 4) % 4 == 0;
    const bool long_rows = D >= (1LL << 24) - 4096;              // 32 rows of fp32 and a row's own offsets below 2^31 bytes
    p.fused = p.nb == 1 && p.nslab <= (p.direct ? kFusedSlabs : kFusedFillSlabs);
    if (p.fused) {
        p.spc = p.nslab;
        p.nsplit = p.turns = 1;
    }
    // Beside another stream's work: the same chunks (the same bits) in two launches of half the workgroups.  The kernel
    // is bound by HBM either way, and one that sits on every CU keeps the other stream's workgroups waiting.  12-layer
    // stack of 64 x 256 tokens with one launch / two, ms: 6.873 / 6.858 repeated (two runs of a side differ by as much),
    // 6.99 / 6.82 for the first pass on new inputs.
    const int launches = beside && p.turns > 1 ? 2 : 1, width = (p.turns + launches - 1) / launches;
    const dim3 grid((unsigned)(width * 8)), block(64 * kGramWaves);
    const size_t smem = p.fused ? kGramFused : kGramReduce;      // (covers the stages: 8 KB per wave at most)
    hipError_t e = hipSuccess;
#define EGERIA_GRAM(K, T, R, L)                                                                         \
    do {                                                                                               \
        static bool attr_set[kMaxDevices] = {};                                                        \
        if (!attr_set[dev]) {                                                                          \
            e = hipFuncSetAttribute((const void *)gram_kernel<K, T, R, L>, hipFuncAttributeMaxDynamicSharedMemorySize, kGramFused); \
            if (e != hipSuccess) return e;                                                             \
            attr_set[dev] = true;                                                                      \
        }                                                                                              \
        for (int l = 0; l < launches && e == hipSuccess; ++l)                                          \
            e = launch_k(EGERIA_KERNEL_GRAM, gram_kernel<K, T, R, L>, grid, block, smem, st, a_t, a_r, (int)b, D, p, l * width, part, counter, p_out); \
    } while (0)
#define EGERIA_GRAM_DT(K, L)                                                                           \
    do {                                                                                               \
        if (!tcode && !rcode) EGERIA_GRAM(K, 0, 0, L);                                                 \
        else if (tcode && !rcode) EGERIA_GRAM(K, 1, 0, L);                                             \
        else if (!tcode && rcode) EGERIA_GRAM(K, 0, 1, L);                                             \
        else EGERIA_GRAM(K, 1, 1, L);                                                                  \
    } while (0)
#define EGERIA_GRAM_LONG(K)                                                                            \
    do {                                                                                               \
        if (long_rows) EGERIA_GRAM_DT(K, true); else EGERIA_GRAM_DT(K, false);                         \
    } while (0)
    if (p.nb == 1) EGERIA_GRAM_LONG(0);
    else if (p.nb == 2) EGERIA_GRAM_LONG(1);
    else EGERIA_GRAM_LONG(2);
#undef EGERIA_GRAM_LONG
#undef EGERIA_GRAM_DT
#undef EGERIA_GRAM
    if (e != hipSuccess || p.fused) return e;
    const int parts = fin_parts(b);
    auto finish = [&](auto kernel) {
        return launch_k(EGERIA_KERNEL_NONE, kernel, dim3((unsigned)(b * parts)), dim3(kFinThreads), 0, st, (const float *)part,
                        p.nsplit, (int)b, parts, sums, counter, p_out);
    };
    // Few requests beyond the last chunk: b > 96 has 40 of them, where 8 per thread asked for 128.  Whole passes, us, 8 / 4: basic
    // block of 128 x 16 x 32 x 32 44.2 / 43.5, score of 100 x 62720 29.5 / 28.8.  (16 per thread, one round trip for the 256 chunks
    // of b = 64 instead of two, made no difference: bottleneck of 64 x 1024 x 14 x 14 127.2 / 127.0.)
    if (fin_columns(b) == 16) return finish(sp_finalize_kernel<16, 4>);
    return p.nsplit <= 64 ? finish(sp_finalize_kernel<64, 4>) : finish(sp_finalize_kernel<64, 8>);
}

}  // namespace egeria

// ---- the metric for callers that cannot allocate ------------------------------------------
// egeria_plasticity takes its scratch memory (ticket counter, row shares, split-K partials) from a
// workspace the caller allocated.  Code under HIP graph capture, tight serving loops and harnesses
// that forbid allocation have nowhere to get one: egeria_plasticity_noalloc runs the same two
// kernels on a scratch array that lives in the library's own device image.  Each GPU holds its own
// copy of the array, at its own address, until the process ends; `scratch` below is only the
// host-side handle of the symbol, and the device address is looked up once per device.
namespace {
constexpr size_t kScratchBytes = (size_t)16 << 20;      // >= plasticity_partial_bytes(b, D) for every b <= 128 on 256 CUs
std::mutex g_scratch_mutex;
void *g_scratch_ptr[egeria::kMaxDevices] = {};
}  // namespace

// (no `used` attribute: the compiler exports a file-scope static device array that host code names, and
// the runtime finds it by that exported name; marked `used` it stays a local symbol of the code object)
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

// Device address of this GPU's copy of the array (the current device's), looked up on first use.
static hipError_t scratch_address(void **out)
{
    const int dev = egeria::current_device();
    if (dev < 0) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

extern "C" egeria_status egeria_plasticity_noalloc(const void *a_train, egeria_dtype t_dt, const void *a_ref,
                                                   egeria_dtype r_dt, int32_t b, int64_t D, float *p_out, void *stream)
{
    using namespace egeria;
    if (!a_train || !a_ref || !p_out || b < 1 || D < 1) return EGERIA_ERR_INVALID_ARG;
    if (((uintptr_t)a_train & 15u) || ((uintptr_t)a_ref & 15u) || ((uintptr_t)p_out & 3u)) return EGERIA_ERR_INVALID_ARG;
    if ((t_dt != EGERIA_F32 && t_dt != EGERIA_BF16) || (r_dt != EGERIA_F32 && r_dt != EGERIA_BF16))
        return EGERIA_ERR_INVALID_ARG;
    if (b > 128) return EGERIA_ERR_UNSUPPORTED;
    if (plasticity_partial_bytes(b, D) > kScratchBytes) return EGERIA_ERR_UNSUPPORTED;     // beyond the array
    void *ptr = nullptr;
    if (scratch_address(&ptr) != hipSuccess) return EGERIA_ERR_HIP;
    // the kernels take the array's device address as they take the caller's workspace in
    // egeria_plasticity; what must start at zero (the finaliser's ticket) is cleared by the first kernel
    if (launch_plasticity(a_train, t_dt, a_ref, r_dt, b, D, p_out, ptr, (hipStream_t)stream) != hipSuccess)
        return EGERIA_ERR_HIP;
    return EGERIA_OK;
}
