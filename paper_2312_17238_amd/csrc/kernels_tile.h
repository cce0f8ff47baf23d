// Grouped dequantize+GEMM on the matrix cores for batches and prompts, every weight format.
//
// A block multiplies one expert's tokens (or up to TOK of them) with ROWS memory rows.  k_tile<.., TE_BIG>, 2-bit codes (the others have a large
// kernel of their own, kernels_big.h): 8 waves, 256 rows x up to 192 tokens, a wave 64 rows x up to 96 tokens (two waves share each 64 rows).  k_tile<.., 16 or 32>: 128
// rows x up to that many tokens, the units of a set shared by the waves of 64 rows (32, with tiles of 32 tokens and 3 or 4 bits:
// 8 waves a block then fit 128 registers each, four waves a SIMD; 1856 x 5056, 37 tokens, two-level: 26.7 + 19.6 -> 24.2 + 18.2 us,
// larger layers the same as with 4 waves); two blocks per compute unit.
//
// A unit is 64 codes of a row, a set four units: 128 bytes of 4-bit codes, which 8 lanes read in one piece.  Weights
// cross LDS once (v_mfma_f32_32x32x16 wants a row per lane; loaded that way from memory every 16-byte piece would be a
// line of its own to the compute unit's address path: measured 806 us for w1/w3 of a 1024-token prompt, all of it
// that path), the metadata decoded by the thread that stages it.  The order of the contraction is free: lane half hh
// takes the 32 codes at 32 hh of a unit, 16 consecutive bytes, and k-step j of it the activations 32 hh + 8 j .. + 7.
//
// Arithmetic.  A weight is s (q - z) with real z, and with any constant ZC
//     sum_k s (q - z) x  =  sum_groups s (sum_k (q - ZC) x)  +  sum_groups s (ZC - z) X,     X = sum of the group's x.
// 3 and 4 bits, ZC = 4 and 8: a code's bits under the exponent of 64 or 1024 are the fp16 numbers 64 + q and 1024 + q, bias and ZC are
// subtracted packed (codes_centred, nine instructions a word of eight).  q - ZC is exact.  The group's product comes out
// in fp32 and is scaled by the fp32 s with one fused multiply-add per accumulator register; no weight is rounded.
// The subtraction is there for the error.  Codes that enter as 64 + q make the products some fourteen times as large, and the matrix
// cores' roundings with them, which have one sign where the tokens have a mean: the error then grows with the length of the
// contraction (4096 x 14336, 4-bit, below: 4.8e-5, and 24e-5 at a mean of eight deviations; minus the bias's share as a product's
// start, one more matrix instruction, leaves 2.3 to 2.9e-5).  It costs 1 to 3 %: 37 tokens two-level 49.6 -> 50.3 us a step, 16 tokens 3-bit 183.4 -> 184.3 (and
// 1024 tokens 4-bit 1042 -> 1073, 512 tokens 3-bit 605 -> 616 with the large kernel of these formats before k_big).
// (Codes as the subnormal fp16 numbers their bits spell need no exponent, but the matrix cores accumulate products of
// subnormals with fewer bits: 6 % more error in y.)
// Groups of 32 (4 bits, tiles of 16 and 32 tokens): two products of half the length per unit, a lane half or quarter holding its share of either group.
// 2-bit codes (groups of 16; ZC = 1): q - 1 is one of -1, 0, 1, 2 and (q - 1) s is exact in fp16 for an fp16 s, so the
// scaled weight goes in directly; an fp32 s (two-level metadata) goes in as two fp16 numbers, in two products.
// Second term: a contraction over groups instead of codes, on the bf16 matrix instructions.  X and D = s (ZC - z) go in
// whole, cut into three bf16 each: eight k-slots a group (slots3_x, slots3_d) hold all products but that of the third parts.  2-bit
// codes in their large kernel and in tiles of 32: two bf16 each (what is lost is 2^-17 of the term, itself a fraction of the result unless the
// tokens have a mean), the four k-slots (Xh, Xl, Xh, Xl) x (Dh, Dh, Dl, Dl).  Tiles of 16 take steps that the GEMV kernels, whose term is in
// fp32, would else take, and have the slots: whole too (D staged as fp32, cut where it is used; 2-bit, 16 tokens, 167.6 -> 168.4 us a
// step; with tiles of 32 it takes an instruction more, 64 tokens 224 -> 231).  Correcting every group's product in the accumulators instead would double the vector work per group.
// The X come from whoever produced the activations (the gate kernel for h, the w1/w3 epilogue for a), rows padded with zeros
// to a multiple of four groups.
//
// Measured, Mixtral-shaped layer, all 8 experts resident, one step at a time, w1/w3 + w2 in us: 16 tokens 3-bit 115 + 60, 2-bit 116 + 62 (GEMV kernels
// 213 + 103).  What bounds them: no unit is full; a third of the waves' time goes into waits, for a unit's or set's barrier and the activations
// staged for it, and two to four waves a SIMD leave few others to run.  2-bit, 16 tokens: vector unit 59 %, of it a quarter for the metadata.
//
// Error of this arithmetic alone: y of a layer against 64 bits with the activations between the halves rounded to fp16 as
// here (an a close to the middle of two fp16 numbers then falls the other way now and then, which is most of it), one expert of 1024 x 4096
// and of 4096 x 14336, every format (4-bit groups of 64 and 128), two seeds, steps of 16 tokens, of 32 and of as many as a block of the large kernel takes
// (2-bit 192, two-level 128, 3 and 4 bits 128, in k_big).  Normalised tokens of mean 0, as the decode workloads draw them / of a
// mean of a tenth of the deviation / of mean 1 and deviation 1/8, in 1e-5: 4-bit tiles of 16 and 32 0.3 to 1.3 / 0.3 to 2.0 / 0.7 to 2.4, k_big 0.7 to 1.2 / 0.7 to 1.3 / 0.9
// to 1.7 (GEMV kernels 8.6 to 10 / 8.6 to 10 / 14 to 17), 3-bit tiles 0.2 to 1.7 / 0.6 to 1.4 / 0.7 to 3.0, k_big 0.8 to 1.3 / 0.8 to 1.2 / 1.1 to 1.7 (GEMV 17 to 18 / 19 / 41), 2-bit tiles
// of 16 0.6 to 2.0 / 0.7 to 2.2 / 1.1 to 2.4, others 3.5 to 4.6 / 3.4 to 4.4 / 6.4 to 7.3 (GEMV 11 to 12 / 11 / 2.9 to 3.3; the two bf16 of X and D).  With the rounding of a, the error of y at mean 0 is 2.07 to 2.1e-4 (GEMV 2.08 to 2.2e-4).
//
// BIG: of the two waves on a SIMD (same rows, other tokens) one unpacks a unit's codes before it multiplies them, the
// other at the end of the unit before, so that one's vector work runs under the other's matrix work.
//
// MFMA layouts (v_mfma_f32_32x32x16): A lane l = token l%32, k-slots 8*(l/32)..+7; B lane l = memory row l%32, the same
// k-slots; D lane l, register i = token 8*(i/4) + 4*(l/32) + i%4, memory row l%32.
#pragma once
#include "kernels_mfma16.h"
#include <type_traits>

namespace moe {

typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));

constexpr int TE_XCD = 8;                // blocks of one row block go to one XCD, whose L2 then serves its token blocks

struct TeArgs {
    const uint8_t *blob[16];             // device buffers of the launch's experts
    uint32_t experts;                    // ... one bit for each of them
    const uint8_t *pair_expert;          // at most FEW_PAIRS pairs: every pair's expert, and null else
    const int32_t *first;                // k_sort_pairs: expert e's pairs are positions first[e] .. first[e + 1] - 1 of plist
    const uint16_t *plist;               // pair ids (token * top_k + choice), expert by expert, ascending within one
    const float *pair_w;                 // combine weight of every pair
    const uint16_t *act;                 // w1/w3: h [B][K];  w2: a [B*top_k][K]
    const uint2 *xs;                     // sums of act per group: [row of act][xs_stride]
    uint16_t *a;                         // w1/w3: SwiGLU activations [pair][N]
    uint2 *xs_out;                       // ... and their sums
    float *ypart;                        // w2: rows of N, one per pair (k_parts == 1) or per (position, part)
    uint32_t *ytab;
    int32_t K, N, top_k, n_pairs;
    int32_t xs_stride, xs_out_stride;
    uint32_t stride, meta_off, meta2_off, b_off;
    int32_t unit_shift, run_shift;       // group of unit u: u >> unit_shift; run of group g: g >> run_shift
    uint64_t mat_off;
    int32_t units_per_part, k_parts, part_base, row_blocks;
    // w2, other parts where the step's token blocks, all experts' together, turn out fewer than few_below: four bits for every number of
    // blocks, from one up
    int32_t few_below;
    uint64_t few;
    float lift, lower;                   // two-level 2-bit codes: what their scales are multiplied with, and its reciprocal
    uint32_t act_bytes, xs_bytes;        // sizes of the two tables, for the bounds of their loads
};

// ---------------------------------------------------------------------------------------------
// loads
// ---------------------------------------------------------------------------------------------

__device__ __forceinline__ uint32_t bl32(__amdgpu_buffer_rsrc_t r, uint32_t v, int s = 0) { return __builtin_amdgcn_raw_buffer_load_b32(r, (int)v, s, 0); }
__device__ __forceinline__ uint2 bl64(__amdgpu_buffer_rsrc_t r, uint32_t v, int s = 0)
{
    const u32x2_t x = __builtin_amdgcn_raw_buffer_load_b64(r, (int)v, s, 0);
    return make_uint2(x.x, x.y);
}
__device__ __forceinline__ uint4 bl128(__amdgpu_buffer_rsrc_t r, uint32_t v, int s = 0)
{
    const u32x4_t x = __builtin_amdgcn_raw_buffer_load_b128(r, (int)v, s, 0);
    return make_uint4(x.x, x.y, x.z, x.w);
}
constexpr uint32_t TE_NONE = 0x80000000u;    // an offset past every buffer's end: zeros, no request

// Contraction over groups, X and D whole: the eight k-slots of one group, from split3 of X and D (first, second, third
// part): X as (0 1 0 1 0 1 2 2), D as (0 0 1 1 2 2 0 1): all products but that of the third parts.  (Or the other way round.)
__device__ __forceinline__ bf8_t slots3_x(uint2 v)
{
    const u32x4_t r = {v.x, v.x, v.x, v.y};
    return __builtin_bit_cast(bf8_t, r);
}
__device__ __forceinline__ bf8_t slots3_d(uint2 v)
{
    const u32x4_t r = {__builtin_amdgcn_perm(v.x, v.x, 0x01000100u), __builtin_amdgcn_perm(v.x, v.x, 0x03020302u), v.y, v.x};
    return __builtin_bit_cast(bf8_t, r);
}
// 2-bit codes: the k-slots of two groups, X as (h l h l), D as (h h l l)
__device__ __forceinline__ bf8_t slots_x(uint2 v)
{
    const u32x4_t r = {v.x, v.x, v.y, v.y};
    return __builtin_bit_cast(bf8_t, r);
}
__device__ __forceinline__ bf8_t slots_d(uint2 v)
{
    const u32x4_t r = {__builtin_amdgcn_perm(v.x, v.x, 0x01000100u), __builtin_amdgcn_perm(v.x, v.x, 0x03020302u),
                       __builtin_amdgcn_perm(v.y, v.y, 0x01000100u), __builtin_amdgcn_perm(v.y, v.y, 0x03020302u)};
    return __builtin_bit_cast(bf8_t, r);
}

// Eight codes of a word in the 4-bit layout as the fp16 numbers q - ZC, in codes_biased's slots: their bits under the exponent of 1024
// or of 64, and the bias and ZC subtracted.  With 3 bits, bit 3 of a field is not the code's.
struct CentredPatterns { uint32_t m_lo, m_hi, k1024, k64; };
template <int BITS> __device__ __forceinline__ CentredPatterns centred_patterns()
{
    constexpr uint32_t F = (1u << BITS) - 1u;
    CentredPatterns p = {F * 0x00010001u, F * 0x00100010u, 0x64006400u, 0x54005400u};
    asm("" : "+s"(p.m_lo), "+s"(p.m_hi), "+v"(p.k1024), "+v"(p.k64));
    return p;
}
template <int BITS> __device__ __forceinline__ h8_t codes_centred(uint32_t w, const CentredPatterns &p)
{
    constexpr uint32_t C1024 = BITS == 4 ? 0xE408E408u : 0xE404E404u, C64 = BITS == 4 ? 0xD480D480u : 0xD440D440u;      // -1024 - ZC, -64 - ZC
    const uint32_t hi = w >> 8;
    const h2_t r0 = as_h2((w & p.m_lo) | p.k1024) + as_h2(C1024), r1 = as_h2((w & p.m_hi) | p.k64) + as_h2(C64);
    const h2_t r2 = as_h2((hi & p.m_lo) | p.k1024) + as_h2(C1024), r3 = as_h2((hi & p.m_hi) | p.k64) + as_h2(C64);
    h8_t r;
    r[0] = r0.x; r[1] = r0.y; r[2] = r1.x; r[3] = r1.y; r[4] = r2.x; r[5] = r2.y; r[6] = r3.x; r[7] = r3.y;
    return r;
}

// What the format policies know of a matrix: offsets inside a row, units of a row.  Loads of codes address with one
// vector register per thread and a scalar: the slab of rows that a load of the block covers lies wholly inside or outside
// the matrix (rows come in multiples of 64), one outside repeats the last.  A set that reaches past a row's end reads up
// to 96 bytes of what follows the row (at most of the memory behind the expert buffers, which the same allocation holds).
struct TeGeom { uint32_t stride, meta_off, meta2_off, b_off; int32_t unit_shift, run_shift, units; };

// One (scale, zero) per unit, fp16 pair or byte pair and quad: item p = (row p / 4, unit p % 4 of the set).
template <bool META8, int N> struct TeMeta;
template <int N> struct TeMeta<false, N> {
    uint32_t m[N];
    __device__ __forceinline__ void fetch(int i, __amdgpu_buffer_rsrc_t r, uint32_t row, int u, const TeGeom &g) { m[i] = bl32(r, row + g.meta_off + 4u * (uint32_t)(u >> g.unit_shift)); }
    __device__ __forceinline__ void get(int i, float &s, float &z) const { s = lo_half(m[i]); z = hi_half(m[i]); }
};
template <int N> struct TeMeta<true, N> {
    uint32_t m[N];
    uint2 quad[N];
    __device__ __forceinline__ void fetch(int i, __amdgpu_buffer_rsrc_t r, uint32_t row, int u, const TeGeom &g)
    {
        const uint32_t grp = (uint32_t)(u >> g.unit_shift);
        m[i] = __builtin_amdgcn_raw_buffer_load_b16(r, (int)(row + g.meta_off + 2u * grp), 0, 0);
        quad[i] = bl64(r, row + g.meta2_off + 8u * (grp >> g.run_shift));
    }
    __device__ __forceinline__ void get(int i, float &s, float &z) const { decode_meta8(m[i], quad[i], s, z); }
};

// Groups of 32: two (scale, zero) per unit; with two-level metadata both lie in one run (tile_format).
template <bool META8, int N> struct TeMeta2;
template <int N> struct TeMeta2<false, N> {
    uint2 m[N];
    __device__ __forceinline__ void fetch(int i, __amdgpu_buffer_rsrc_t r, uint32_t row, int u, const TeGeom &g) { m[i] = bl64(r, row + g.meta_off + 8u * (uint32_t)u); }
    __device__ __forceinline__ void get(int i, int j, float &s, float &z) const { const uint32_t w = j ? m[i].y : m[i].x; s = lo_half(w); z = hi_half(w); }
};
template <int N> struct TeMeta2<true, N> {
    uint32_t m[N];
    uint2 quad[N];
    __device__ __forceinline__ void fetch(int i, __amdgpu_buffer_rsrc_t r, uint32_t row, int u, const TeGeom &g)
    {
        m[i] = bl32(r, row + g.meta_off + 4u * (uint32_t)u);
        quad[i] = bl64(r, row + g.meta2_off + 8u * (2u * (uint32_t)u >> g.run_shift));
    }
    __device__ __forceinline__ void get(int i, int j, float &s, float &z) const { decode_meta8(m[i] >> (16 * j), quad[i], s, z); }
};

// ---------------------------------------------------------------------------------------------
// format policies.  Stage: what a thread holds of one set on its way to LDS; a row's record in LDS: CODES bytes of
// codes, then (GS) four fp32 scales; D: split zero-point factors, DB bytes per row.  GS: scaled in the accumulators.
// ---------------------------------------------------------------------------------------------

template <int FMT, int ROWS, int THREADS> struct Te;

template <bool META8, int ROWS, int THREADS, int BITS, int G = 1>
struct TeScaled {                        // the part that 4-bit and 3-bit formats share
    static constexpr float ZC = float(1 << (BITS - 1));                  // what the codes are centred on
    static constexpr bool GS = true;
    static constexpr int GPU = G, PLANES = 1, DB = 32 * G;               // groups per unit; bytes of D per row and set
    static constexpr bool LIFTED = false;
    static constexpr int NM = ROWS * 4 / THREADS;
    std::conditional_t<G == 1, TeMeta<META8, NM>, TeMeta2<META8, NM>> meta;
    __device__ __forceinline__ void fetch_meta(__amdgpu_buffer_rsrc_t rs, const TeGeom &g, int row0, int n_rows, int u, bool live, int tid)
    {
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const int r = min(row0 + tid / 4 + i * (THREADS / 4), n_rows - 1);
            meta.fetch(i, rs, live ? (uint32_t)r * g.stride : TE_NONE, min(u + tid % 4, g.units - 1), g);   // a finite scale also for units past the end
        }
    }
    template <int REC, int SOFF>
    __device__ __forceinline__ void commit_meta(uint8_t *rec, uint8_t *d, int tid) const
    {
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            float s, z;
            if constexpr (G == 1) {
                meta.get(i, s, z);
                *reinterpret_cast<float *>(rec + (tid / 4) * REC + (tid % 4) * 4 + SOFF + i * (THREADS / 4) * REC) = s;
                *reinterpret_cast<uint2 *>(d + tid * 8 + i * THREADS * 8) = split3(s * (ZC - z));
            } else {
                float s1, z1;
                meta.get(i, 0, s, z);
                meta.get(i, 1, s1, z1);
                *reinterpret_cast<float2 *>(rec + (tid / 4) * REC + (tid % 4) * 8 + SOFF + i * (THREADS / 4) * REC) = make_float2(s, s1);
                const uint2 d0 = split3(s * (ZC - z)), d1 = split3(s1 * (ZC - z1));
                *reinterpret_cast<uint4 *>(d + tid * 16 + i * THREADS * 16) = make_uint4(d0.x, d0.y, d1.x, d1.y);
            }
        }
    }
};

template <bool META8, int ROWS, int THREADS, int G = 1>
struct Te4 : TeScaled<META8, ROWS, THREADS, 4, G> {
    static constexpr uint32_t BITS = 4;
    static constexpr int SOFF = 128, REC = G == 1 ? 144 : 176, NC = ROWS * 8 / THREADS;
    uint4 c[NC];
    struct Raw { uint4 q; };
    __device__ __forceinline__ void fetch(int h, __amdgpu_buffer_rsrc_t rs, const TeGeom &g, int row0, int n_rows, int u, bool live, int tid)
    {
        constexpr int SLAB = THREADS / 8;
        const uint32_t v = live ? (uint32_t)(tid / 8) * g.stride + (uint32_t)(tid % 8) * 16u : TE_NONE;
#pragma unroll
        for (int i = h * NC / 2; i < (h + 1) * NC / 2; ++i) c[i] = bl128(rs, v, min(row0 + i * SLAB, n_rows - SLAB) * (int)g.stride + u * 32);
        if (h == 1) this->fetch_meta(rs, g, row0, n_rows, u, live, tid);
    }
    __device__ __forceinline__ void commit(int h, uint8_t *rec, uint8_t *d, int, float, int tid) const
    {
        uint8_t *const to = rec + (tid / 8) * REC + (tid % 8) * 16;
#pragma unroll
        for (int i = h * NC / 2; i < (h + 1) * NC / 2; ++i) *reinterpret_cast<uint4 *>(to + i * (THREADS / 8) * REC) = c[i];
        if (h == 1) this->template commit_meta<REC, SOFF>(rec, d, tid);
    }
    // (groups of 32: a lane half takes half of either group)
    static __device__ __forceinline__ void read(Raw &r, const uint8_t *row, int hh, int u)
    {
        if constexpr (G == 1) {
            r.q = *reinterpret_cast<const uint4 *>(row + u * 32 + hh * 16);
        } else {
            const uint2 p = *reinterpret_cast<const uint2 *>(row + u * 32 + hh * 8), q = *reinterpret_cast<const uint2 *>(row + u * 32 + 16 + hh * 8);
            r.q = make_uint4(p.x, p.y, q.x, q.y);
        }
    }
    // words of 8 codes in the 4-bit layout: the lane half's four, or those of quarter kb of the unit
    static __device__ __forceinline__ void words(const Raw &r, uint32_t (&t)[4]) { t[0] = r.q.x; t[1] = r.q.y; t[2] = r.q.z; t[3] = r.q.w; }
    static __device__ __forceinline__ void quarter(const uint8_t *row, int kb, int u, uint32_t (&t)[2])
    {
        if constexpr (G == 1) {
            const uint2 q = *reinterpret_cast<const uint2 *>(row + u * 32 + kb * 8);
            t[0] = q.x; t[1] = q.y;
        } else {                                                         // a quarter of either group
            t[0] = *reinterpret_cast<const uint32_t *>(row + u * 32 + kb * 4);
            t[1] = *reinterpret_cast<const uint32_t *>(row + u * 32 + 16 + kb * 4);
        }
    }
};
template <int R, int T> struct Te<4, R, T> : Te4<false, R, T> {};
template <int R, int T> struct Te<48, R, T> : Te4<true, R, T> {};
template <int R, int T> struct Te<5, R, T> : Te4<false, R, T, 2> {};      // 4-bit codes in groups of 32, and with two-level metadata
template <int R, int T> struct Te<58, R, T> : Te4<true, R, T, 2> {};

// 32 codes of a 3-bit row, from its two regions, as words of the 4-bit layout: one v_bfi each; bit 3 of a field is another word's
struct Codes3 {
    struct Raw { uint2 a; uint32_t b; };
    static __device__ __forceinline__ void words(const Raw &r, uint32_t (&t)[4])
    {
        t[0] = (r.a.x & 0x33333333u) | ((r.b << 2) & ~0x33333333u);
        t[1] = ((r.a.x >> 2) & 0x33333333u) | ((r.b << 1) & ~0x33333333u);
        t[2] = (r.a.y & 0x33333333u) | (r.b & ~0x33333333u);
        t[3] = ((r.a.y >> 2) & 0x33333333u) | ((r.b >> 1) & ~0x33333333u);
    }
};

template <bool META8, int ROWS, int THREADS>
struct Te3 : TeScaled<META8, ROWS, THREADS, 3> {
    static constexpr uint32_t BITS = 3;
    static constexpr int SOFF = 96, REC = 112;
    static_assert(ROWS * 4 == THREADS, "a thread has 16 bytes of region A and 8 of region B");
    uint4 a;
    uint2 b;
    using Raw = Codes3::Raw;
    __device__ __forceinline__ void fetch(int h, __amdgpu_buffer_rsrc_t rs, const TeGeom &g, int row0, int n_rows, int u, bool live, int tid)
    {
        // 64 rows per half block of threads: a load covers two slabs of 64
        const uint32_t row = (uint32_t)(tid / 4 % 64) * g.stride;
        const int at = min(row0 + uniform(tid / 256) * 64, n_rows - 64) * (int)g.stride;
        if (h == 0) {
            a = bl128(rs, live ? row + (uint32_t)(tid % 4) * 16u : TE_NONE, at + u * 16);
        } else {
            b = bl64(rs, live ? row + (uint32_t)(tid % 4) * 8u : TE_NONE, at + (int)g.b_off + u * 8);
            this->fetch_meta(rs, g, row0, n_rows, u, live, tid);
        }
    }
    __device__ __forceinline__ void commit(int h, uint8_t *rec, uint8_t *d, int, float, int tid) const
    {
        if (h == 0) {
            *reinterpret_cast<uint4 *>(rec + (tid / 4) * REC + (tid % 4) * 16) = a;
        } else {
            *reinterpret_cast<uint2 *>(rec + (tid / 4) * REC + (tid % 4) * 8 + 64) = b;
            this->template commit_meta<REC, SOFF>(rec, d, tid);
        }
    }
    static __device__ __forceinline__ void read(Raw &r, const uint8_t *row, int hh, int u)
    {
        r.a = *reinterpret_cast<const uint2 *>(row + u * 16 + hh * 8);
        r.b = *reinterpret_cast<const uint32_t *>(row + 64 + u * 8 + hh * 4);
    }
    static __device__ __forceinline__ void words(const Raw &r, uint32_t (&t)[4]) { Codes3::words(r, t); }
    static __device__ __forceinline__ void quarter(const uint8_t *row, int kb, int u, uint32_t (&t)[2])
    {
        const uint32_t a = *reinterpret_cast<const uint32_t *>(row + u * 16 + kb * 4);
        const uint32_t b = *reinterpret_cast<const uint32_t *>(row + 64 + u * 8 + (kb >> 1) * 4) >> (2 * (kb & 1));
        t[0] = (a & 0x33333333u) | ((b << 2) & ~0x33333333u);
        t[1] = ((a >> 2) & 0x33333333u) | ((b << 1) & ~0x33333333u);
    }
};
template <int R, int T> struct Te<3, R, T> : Te3<false, R, T> {};
template <int R, int T> struct Te<38, R, T> : Te3<true, R, T> {};

// eight codes (half of a 2-bit word) as (q - 1) s: fields of two bits under the exponents of 1024, 256, 64 and 16
struct Patterns2 { uint32_t m[4], k[4]; };
__device__ __forceinline__ Patterns2 patterns2()
{
    Patterns2 p = {{0x00030003u, 0x000C000Cu, 0x00300030u, 0x00C000C0u}, {0x64006400u, 0x5C005C00u, 0x54005400u, 0x4C004C00u}};
    asm("" : "+s"(p.m[0]), "+s"(p.m[1]), "+s"(p.m[2]), "+s"(p.m[3]), "+v"(p.k[0]), "+v"(p.k[1]), "+v"(p.k[2]), "+v"(p.k[3]));
    return p;
}
__device__ __forceinline__ void centred2(uint32_t w, const Patterns2 &p, h2_t (&c)[4])
{
    constexpr uint32_t off[4] = {0xE401E401u, 0xDC04DC04u, 0xD410D410u, 0xCC40CC40u};       // -1025, -257, -65, -17
#pragma unroll
    for (int n = 0; n < 4; ++n) c[n] = as_h2((w & p.m[n]) | p.k[n]) + as_h2(off[n]);
}

// 2-bit codes, groups of 16; record of a unit: (codes, scale) words of its four groups, 32 bytes
template <bool META8, int ROWS, int THREADS>
struct Te2 {
    static constexpr bool GS = false;
    static constexpr uint32_t BITS = 2;
    static constexpr int GPU = 4, PLANES = META8 ? 2 : 1, DB = META8 ? 80 : 0, REC = 144, SOFF = 0;   // one-level: D from the record's (scale, zero)
    static constexpr int NC = ROWS * 8 / THREADS, NA = ROWS * 4 / THREADS;
    // two-level scales are split into two fp16, lifted by the layer's own power of two first (the host chooses it: the
    // largest scale just fits, and the low part of every row's largest is a normal number), the totals lowered at the end
    static constexpr bool LIFTED = META8;
    // D (two-level): one word a group, two bf16 or, with tiles of 16, the fp32 number
    static constexpr bool D2 = ROWS == 256 || THREADS == 256;
    uint4 c[META8 ? NA : NC];
    uint2 mp[META8 ? NA : 1], quad[META8 ? NA : 1];
    struct Raw { uint4 q; };
    __device__ __forceinline__ void fetch(int h, __amdgpu_buffer_rsrc_t rs, const TeGeom &g, int row0, int n_rows, int u, bool live, int tid)
    {
        if constexpr (!META8) {
            constexpr int SLAB = THREADS / 8;
            const uint32_t v = live && u + (tid % 8) / 2 < g.units ? (uint32_t)(tid / 8) * g.stride + (uint32_t)(tid % 8) * 16u : TE_NONE;
#pragma unroll
            for (int i = h * NC / 2; i < (h + 1) * NC / 2; ++i) c[i] = bl128(rs, v, min(row0 + i * SLAB, n_rows - SLAB) * (int)g.stride + u * 32);
        } else {
            const uint32_t row = (uint32_t)(tid / 4 % 64) * g.stride, un = (uint32_t)(tid % 4);
#pragma unroll
            for (int i = h * NA / 2; i < (h + 1) * NA / 2; ++i) {
                const int at = min(row0 + (i * THREADS / 4) + uniform(tid / 256) * 64, n_rows - 64) * (int)g.stride;
                c[i] = bl128(rs, live ? row + un * 16u : TE_NONE, at + u * 16);
                mp[i] = bl64(rs, live ? row + un * 8u : TE_NONE, at + (int)g.meta_off + u * 8);
                quad[i] = bl64(rs, live ? row + 8u * (uint32_t)((min(u + (int)un, g.units - 1) * 4) >> g.run_shift) : TE_NONE, at + (int)g.meta2_off);
            }
        }
    }
    // What lies behind a row's end is no scale, so the records of units there are zeros: not requested (one-level), or set here;
    // valid: units of the set that exist.
    __device__ __forceinline__ void commit(int h, uint8_t *rec, uint8_t *d, int valid, float lift, int tid) const
    {
        if constexpr (!META8) {
            uint8_t *const to = rec + (tid / 8) * REC + (tid % 8) * 16;
#pragma unroll
            for (int i = h * NC / 2; i < (h + 1) * NC / 2; ++i) *reinterpret_cast<uint4 *>(to + i * (THREADS / 8) * REC) = c[i];
        } else {
            const bool in = tid % 4 < valid;
            uint8_t *const to = rec + (tid / 4) * REC + (tid % 4) * 32, *const dd = d + (tid / 4) * DB + (tid % 4) * 16;
#pragma unroll
            for (int i = h * NA / 2; i < (h + 1) * NA / 2; ++i) {
                const uint32_t pr[4] = {mp[i].x, mp[i].x >> 16, mp[i].y, mp[i].y >> 16};
                uint32_t ss[4], dv[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    float s, z;
                    decode_meta8(pr[k], quad[i], s, z);
                    s = in ? s * lift : 0.f;
                    z = in ? z : 0.f;
                    const _Float16 hi = (_Float16)s;
                    const h2_t p = {hi, (_Float16)(s - (float)hi)};
                    ss[k] = __builtin_bit_cast(uint32_t, p);
                    dv[k] = D2 ? split2(s - s * z) : __builtin_bit_cast(uint32_t, s - s * z);
                }
                *reinterpret_cast<uint4 *>(to + i * (THREADS / 4) * REC) = make_uint4(c[i].x, ss[0], c[i].y, ss[1]);
                *reinterpret_cast<uint4 *>(to + i * (THREADS / 4) * REC + 16) = make_uint4(c[i].z, ss[2], c[i].w, ss[3]);
                *reinterpret_cast<uint4 *>(dd + i * (THREADS / 4) * DB) = make_uint4(dv[0], dv[1], dv[2], dv[3]);
            }
        }
    }
    static __device__ __forceinline__ void read(Raw &r, const uint8_t *row, int hh, int u) { r.q = *reinterpret_cast<const uint4 *>(row + u * 32 + hh * 16); }
    // the two groups' D, split in two
    static __device__ __forceinline__ uint2 factors(const uint8_t *row, const uint8_t *drow, int hh, int u)
    {
        if constexpr (META8) return *reinterpret_cast<const uint2 *>(drow + u * 16 + hh * 8);
        Raw r;
        read(r, row, hh, u);
        const float s0 = lo_half(r.q.y), s1 = lo_half(r.q.w);
        return make_uint2(split2(s0 - s0 * hi_half(r.q.y)), split2(s1 - s1 * hi_half(r.q.w)));
    }
    // a quarter of a unit is one group: its two words of weights per plane
    static __device__ __forceinline__ uint2 quarter(const uint8_t *row, int kb, int u, h8_t (&b)[PLANES][2])
    {
        const Patterns2 p = patterns2();
        const uint2 q = *reinterpret_cast<const uint2 *>(row + u * 32 + kb * 8);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            h2_t c[4];
            centred2(k ? q.x >> 8 : q.x, p, c);
#pragma unroll
            for (int pl = 0; pl < PLANES; ++pl) {
                const _Float16 s = as_h2(q.y)[pl];
                const h2_t s2 = {s, s};
                const h2_t v0 = c[0] * s2, v1 = c[1] * s2, v2 = c[2] * s2, v3 = c[3] * s2;
                h8_t x;
                x[0] = v0.x; x[1] = v0.y; x[2] = v1.x; x[3] = v1.y; x[4] = v2.x; x[5] = v2.y; x[6] = v3.x; x[7] = v3.y;
                b[pl][k] = x;
            }
        }
        return q;
    }
    static __device__ __forceinline__ void decode(const Raw &r, h8_t (&b)[PLANES][4])
    {
        const Patterns2 p = patterns2();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t w = k < 2 ? r.q.x : r.q.z, m = k < 2 ? r.q.y : r.q.w;
            h2_t c[4];
            centred2((k & 1) ? w >> 8 : w, p, c);
#pragma unroll
            for (int pl = 0; pl < PLANES; ++pl) {
                const _Float16 s = as_h2(m)[pl];                         // one-level: the pair's scale; two-level: high, low part
                const h2_t s2 = {s, s};
                const h2_t v0 = c[0] * s2, v1 = c[1] * s2, v2 = c[2] * s2, v3 = c[3] * s2;
                h8_t x;
                x[0] = v0.x; x[1] = v0.y; x[2] = v1.x; x[3] = v1.y; x[4] = v2.x; x[5] = v2.y; x[6] = v3.x; x[7] = v3.y;
                b[pl][k] = x;
            }
        }
    }
};
template <int R, int T> struct Te<2, R, T> : Te2<false, R, T> {};
template <int R, int T> struct Te<28, R, T> : Te2<true, R, T> {};

// ---------------------------------------------------------------------------------------------

// MODE: tokens per block at most -- TE_BIG: several tiles of 32; 32 or 16: one tile of that many
constexpr int TE_BIG = 0;

template <int FMT, int MODE> struct TeCfg {
    static constexpr bool BIG = MODE == TE_BIG;
    static constexpr bool SMALL2 = !BIG && (FMT == 2 || FMT == 28);      // 2-bit codes, one tile
    static constexpr int THREADS = SMALL2 && !(MODE == 16 && FMT == 28) ? 256 : 512;
    static constexpr int RG = BIG || (MODE == 32 && !SMALL2) ? 4 : 2, ROWS = BIG ? 256 : 128;     // row groups: RG of RGR rows
    static constexpr int RGR = ROWS / RG;
    static constexpr int KW = THREADS / 64 / RG;                         // waves of a row group (MODE 16, 32: each a share of a set's units)
    static constexpr int WAVES_EU = !BIG && THREADS == 512 && !((FMT == 5 || FMT == 58) && MODE == 32) ? 4 : 2;   // waves per SIMD (groups of 32: LDS for one block a compute unit)
    using F = Te<FMT, ROWS, THREADS>;
    static constexpr int MT = BIG ? (F::PLANES == 1 ? 3 : 2) : 1;                // token tiles of 32 per wave
    static constexpr int TOK = BIG ? 2 * MT * 32 : MODE;
    static constexpr int SU = BIG ? 1 : 4;                               // units of activations per staging step
    static constexpr int PITCH = SU * 128 + 16;                          // staged bytes per token (+16: bank spread)
    static constexpr int NP = TOK * SU * 8 / THREADS;                    // 16-byte pieces per thread and step
    static constexpr int REC = F::REC;
    static constexpr int ABUF = TOK * PITCH, BBUF = ROWS * REC, DBUF = ROWS * F::DB;
    // sums: 16 bytes are four groups, of a set (GS) or of one unit: XQ pieces per token and staging step
    // (8 bytes each; 2-bit codes take only the first four but with tiles of 16)
    static constexpr bool XWHOLE = F::GS || MODE == 16;
    static_assert(!(BIG && F::GS), "3- and 4-bit codes have a large kernel of their own");
    static constexpr int XQ = F::GS ? 2 * F::GPU : SU * 2, XPITCH = F::GS ? 32 * F::GPU : (BIG ? 16 : XQ * (XWHOLE ? 16 : 8) + 16), XBUF = TOK * XPITCH;
    static constexpr int OFF_B = 2 * ABUF, OFF_D = OFF_B + 2 * BBUF, OFF_X = OFF_D + 2 * DBUF, OFF_END = OFF_X + 2 * XBUF;
    static constexpr int OFF_RED = THREADS / 64 * (RGR * MODE * 4);    // MODE 16, 32: behind the waves' partial sums
    static constexpr int ACOLS = ROWS / 2, APITCH = ACOLS * 2 + 16;      // epilogue: fp16 columns of a per token
    static constexpr int OFF_A = BIG ? 0 : OFF_RED, OFF_T = BIG || OFF_END > OFF_RED + TOK * APITCH ? OFF_END : OFF_RED + TOK * APITCH;
    static constexpr int LDS = OFF_T + TOK * 8;
    static_assert(OFF_X >= TOK * APITCH && LDS <= (BIG || F::PLANES == 2 || (F::GPU == 2 && MODE == 32) ? 160 : 80) * 1024, "the epilogue reuses the staging buffers");
};

// token blocks of an expert: one tile of 16 or 32, or up to as many tiles of 32 per block as the large kernel holds
template <int TOK, bool BIG>
__host__ __device__ constexpr int te_token_blocks(int count) { return BIG ? ((count + 31) / 32 + TOK / 32 - 1) / (TOK / 32) : (count + TOK - 1) / TOK; }

// a contraction of `sets` sets in at most `parts` parts
__host__ __device__ inline void te_split(int sets, int parts, int32_t &k_parts, int32_t &units_per_part)
{
    const int per = (sets + parts - 1) / parts;
    units_per_part = per * 4;
    k_parts = (sets + per - 1) / per;
}

// The item of a block.  Items of an XCD: expert by expert, its jobs (row block, part), each job's token blocks next to each other.  How
// many token blocks an expert has is worked out here, from the sorted list's table, so that the launch need not know the routing
// (its grid then covers the most there can be; the blocks too many get none: blob is null).
// Lane e works it out for expert e (a chain of sixteen scalar steps, each behind a load of its arguments, cost 3 us a block).
struct TeItem { const uint8_t *blob; int expert, first, count, tb, job, t, k_parts, units_per_part; };
template <bool W13, class BLOCKS>
__device__ __forceinline__ TeItem te_item(const TeArgs &A, FewPairs &few, BLOCKS &&token_blocks)
{
    const int lane = threadIdx.x & 63;
    TeItem it{};
    it.k_parts = A.k_parts;
    it.units_per_part = A.units_per_part;
    int j = (int)blockIdx.x / TE_XCD, count, first;
    if (A.pair_expert) {
        few.load(A.pair_expert, A.n_pairs);
        count = few.counts();
        first = prefix16(count) - count;
    } else {
        first = A.first[lane & 15];
        count = A.first[(lane & 15) + 1] - first;
    }
    const int blocks = token_blocks(count);
    // tokens that crowd to a few experts: w2's contraction in as many parts as fill the chip then (of the whole step's
    // experts, not the launch's: the order of the sums must not depend on the cache)
    if (!W13 && A.few_below) {
        const int n = __builtin_amdgcn_readlane(prefix16(blocks), 15);
        if (n > 0 && n < A.few_below) {
            te_split((A.K / 64 + 3) / 4, (int)(A.few >> 4 * (n - 1) & 15u), it.k_parts, it.units_per_part);
            it.k_parts = uniform(it.k_parts);
            it.units_per_part = uniform(it.units_per_part);
        }
    }
    const int jobs = A.row_blocks * it.k_parts, per_xcd = (jobs + TE_XCD - 1) / TE_XCD;
    const int tb = lane < 16 && (A.experts >> lane & 1u) ? blocks : 0, items = tb * per_xcd, end = prefix16(items);
    const uint64_t mine = __ballot(lane < 16 && j >= end - items && j < end);
    if (!mine) return it;
    const int e = (int)__builtin_ctzll(mine);
    it.tb = __builtin_amdgcn_readlane(tb, e);
    j -= __builtin_amdgcn_readlane(end - items, e);
    it.job = (j / it.tb) * TE_XCD + (int)blockIdx.x % TE_XCD;
    it.t = j % it.tb;
    if (it.job >= jobs) return it;
    it.expert = e;
    it.first = __builtin_amdgcn_readlane(first, e);
    it.count = __builtin_amdgcn_readlane(count, e);
    it.blob = A.blob[e];
    return it;
}

// The block's pairs and their weights (w2), from its expert's token tok0 on; -1 past the last of n_tok.
template <bool W13, int TOK>
__device__ __forceinline__ void te_pairs(const TeArgs &A, const FewPairs &few, const TeItem &it, int tok0, int n_tok, int32_t *l_pair, float *l_w)
{
    const int tid = threadIdx.x, lane = tid & 63;
    if (A.pair_expert) {
        if (tid < TOK && tid >= n_tok) l_pair[tid] = -1;
        if (uniform(tid >> 6) == 0) {
            int at = -tok0;                                              // a pair's place among its expert's, from the block's first token
#pragma unroll
            for (int c = 0; c < FEW_PAIRS / 64; ++c) {
                const uint64_t m = few.mask(c, it.expert);
                const int k = at + __popcll(m & ((1ull << lane) - 1)), p = c * 64 + lane;
                if (few.e[c] == (uint32_t)it.expert && k >= 0 && k < n_tok) {
                    l_pair[k] = p;
                    l_w[k] = W13 ? 0.f : A.pair_w[p];
                }
                at += __popcll(m);
            }
        }
    } else if (tid < TOK) {
        const int p = tid < n_tok ? (int)A.plist[it.first + tok0 + tid] : -1;
        l_pair[tid] = p;
        l_w[tid] = p >= 0 && !W13 ? A.pair_w[p] : 0.f;
    }
}

// w1/w3: eight columns of a, piece c of a token (pair pr, or none) in row block rb of `cols` columns, and the sums that w2 takes
template <int GPU>
__device__ __forceinline__ void te_copy_out(const TeArgs &A, const u32x4_t &q, int pr, int rb, int cols, int c)
{
    constexpr int XG = 64 / GPU;                                         // columns per sum
    const int colg = rb * cols + c * 8;
    const bool in = colg < A.N;                                          // N is a multiple of 64: a piece is in or out as a whole
    const h2_t ones = {(_Float16)1.f, (_Float16)1.f};
    float xa = __builtin_amdgcn_fdot2(as_h2(q[0]), ones, 0.f, false), xb = __builtin_amdgcn_fdot2(as_h2(q[1]), ones, 0.f, false);
    xa = __builtin_amdgcn_fdot2(as_h2(q[2]), ones, xa, false);
    xb = __builtin_amdgcn_fdot2(as_h2(q[3]), ones, xb, false);
    float xs = in ? xa + xb : 0.f;
    xs += dpp_f<0xB1>(xs);                                               // two lanes: 16 columns
    if constexpr (XG >= 32) xs += dpp_f<0x4E>(xs);
    if constexpr (XG == 64) xs += dpp_f<0x141>(xs);
    if (pr < 0) return;
    if (in) *reinterpret_cast<u32x4_t *>(A.a + (size_t)pr * A.N + colg) = q;
    uint2 *const xo = A.xs_out + (size_t)pr * A.xs_out_stride;
    const int g = colg / XG;
    if (colg % XG == 0 && g < A.xs_out_stride) xo[g] = split3(xs);
    if (c == 0 && (rb + 1) * cols >= A.N)                                // the padding behind the last group that no row block covers
        for (int z = (rb + 1) * cols / XG; z < A.xs_out_stride; ++z) xo[z] = make_uint2(0u, 0u);
}

// w2: the row of ypart that a part's sums of the pair in place `at` of the block's expert go to: the pair's own, or behind the pairs' rows.  The one
// answer for the kernels' stores and for the entry that k_combine finds them by: a step whose tokens crowd has other parts than its launch's arguments.
__device__ __forceinline__ int te_row(const TeArgs &A, const TeItem &it, int pair, int at, int part)
{
    return it.k_parts == 1 ? pair : A.part_base + (it.first + at) * it.k_parts + part;
}

// w2: one block per token block tells k_combine where the rows are
__device__ __forceinline__ void te_rows_told(const TeArgs &A, const TeItem &it, int tok0, int n_tok, int rb, int part, const int32_t *l_pair)
{
    const int tid = threadIdx.x;
    if (rb != 0 || part != 0 || tid >= n_tok) return;
    const int pr = l_pair[tid];
    A.ytab[pr] = y_rows((uint32_t)te_row(A, it, pr, tok0 + tid, 0), (uint32_t)it.k_parts);
}

template <int FMT, bool W13, int MODE>
__global__ __launch_bounds__((TeCfg<FMT, MODE>::THREADS), (TeCfg<FMT, MODE>::WAVES_EU)) void k_tile(TeArgs A)
{
    using C = TeCfg<FMT, MODE>;
    constexpr bool BIG = C::BIG;
    using F = typename C::F;
    constexpr int THREADS = C::THREADS, ROWS = C::ROWS, NP = C::NP, SU = C::SU, PPT = SU * 8;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    int32_t *const l_pair = reinterpret_cast<int32_t *>(lds + C::OFF_T);
    float *const l_w = reinterpret_cast<float *>(l_pair + C::TOK);
    const int tid = threadIdx.x, lane = tid & 63, wv = uniform(tid >> 6), hh = lane >> 5, col = lane & 31;
    const int rg = wv % C::RG, half = wv / C::RG;                        // rows of the wave; token half (BIG) or unit parity

    FewPairs few;
    const TeItem ex = te_item<W13>(A, few, [](int count) { return te_token_blocks<C::TOK, BIG>(count); });
    if (!ex.blob) return;                                                // whole block, before any barrier
    const int k_parts = ex.k_parts, units_per_part = ex.units_per_part, t = ex.t;
    const int rb = ex.job / k_parts, part = ex.job % k_parts;
    constexpr int TILE = BIG ? 32 : MODE;                                // tokens per tile
    const int tiles = (ex.count + TILE - 1) / TILE;
    const int tile0 = t * tiles / ex.tb, n_tiles = (t + 1) * tiles / ex.tb - tile0;
    const int tok0 = tile0 * TILE, n_tok = min(ex.count - tok0, n_tiles * TILE);
    const int n_rows = W13 ? 2 * A.N : A.N, row0 = rb * ROWS;
    const int u0 = part * units_per_part, u1 = min(A.K / 64, u0 + units_per_part);
    // The first sets of weights need no routing: they are requested before the pairs are known.
    const __amdgpu_buffer_rsrc_t w_rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(ex.blob + A.mat_off), 0, n_rows * (int)A.stride, 0x00020000);
    const TeGeom geo = {A.stride, A.meta_off, A.meta2_off, A.b_off, A.unit_shift, A.run_shift, A.K / 64};
    auto fetch_b = [&](F &f, int h, int u) __attribute__((always_inline)) { f.fetch(h, w_rs, geo, row0, n_rows, u < u1 ? u : u0, u < u1, tid); };
    F f0, f1;                                                            // weights on their way to LDS (BIG: f0)
    fetch_b(f0, 0, u0);
    fetch_b(f0, 1, u0);
    if constexpr (!BIG) {
        fetch_b(f1, 0, u0 + 4);
        fetch_b(f1, 1, u0 + 4);
    }
    te_pairs<W13, C::TOK>(A, few, ex, tok0, n_tok, l_pair, l_w);
    __syncthreads();

    // ---------------- staging ----------------
    const __amdgpu_buffer_rsrc_t a_rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(A.act), 0, (int)A.act_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t x_rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint2 *>(A.xs), 0, (int)A.xs_bytes, 0x00020000);
    auto act_row = [&](int tk) __attribute__((always_inline)) { const int p = l_pair[tk]; return W13 ? p / A.top_k : p; };
    uint32_t a_off[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int tk = tid / PPT + i * (THREADS / PPT);
        a_off[i] = tk < n_tok ? (uint32_t)act_row(tk) * (uint32_t)A.K * 2u + (uint32_t)(tid % PPT) * 16u : TE_NONE;
    }
    // sums: piece p of a step is token p / XQ; threads too many request nothing (a repeated piece is a visit of its line as any
    // other), in the large kernel and with 2-bit codes they repeat one (a branch costs those more: 2-bit, 16 tokens, 120 -> 129 us)
    constexpr int XQ = C::XQ, XU = F::GPU;                               // XU: groups per unit
    constexpr bool X_REPEAT = BIG || !F::GS;
    static_assert(C::TOK * XQ <= THREADS && (!X_REPEAT || THREADS % XQ == 0), "one piece per thread");
    const bool x_mine = X_REPEAT || tid < C::TOK * XQ;
    const int xp = tid % (C::TOK * XQ), x_to = C::OFF_X + (xp / XQ) * C::XPITCH + (xp % XQ) * (C::XWHOLE ? 16 : 8);
    const uint32_t x_off = x_mine && xp / XQ < n_tok ? (uint32_t)act_row(xp / XQ) * (uint32_t)A.xs_stride * 8u + (uint32_t)(xp % XQ) * 16u : TE_NONE;
    struct Acts { uint4 a[NP], x; };                                     // activations and sums of one step on their way to LDS
    auto fetch_a = [&](Acts &t, int u) __attribute__((always_inline)) {                                          // units u .. u + SU - 1; zeros from u1 on
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int un = SU == 1 ? u : u + (tid % PPT) / 8;
            t.a[i] = bl128(a_rs, un < u1 ? a_off[i] : TE_NONE, u * 128);
        }
    };
    auto commit_a = [&](const Acts &t, int b) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            *reinterpret_cast<uint4 *>(lds + (tid / PPT) * C::PITCH + (tid % PPT) * 16 + b * C::ABUF + i * (THREADS / PPT) * C::PITCH) = t.a[i];
        }
    };
    auto fetch_x = [&](Acts &t, int u) __attribute__((always_inline)) { t.x = bl128(x_rs, (F::GS ? u : u + xp % XQ / 2) < u1 ? x_off : TE_NONE, u * (XU * 8)); };
    auto commit_x = [&](const Acts &t, int b) __attribute__((always_inline)) {
        if (!X_REPEAT && C::TOK * XQ < THREADS && !x_mine) return;
        if constexpr (C::XWHOLE) *reinterpret_cast<uint4 *>(lds + x_to + b * C::XBUF) = t.x;
        else *reinterpret_cast<uint2 *>(lds + x_to + b * C::XBUF) = make_uint2(t.x.x, t.x.z);
    };
    auto commit_b = [&](const F &f, int h, int b, int u) __attribute__((always_inline)) { f.commit(h, lds + C::OFF_B + b * C::BBUF, lds + C::OFF_D + b * C::DBUF, geo.units - u, A.lift, tid); };

    // Left alone the scheduler moves a step's loads down to just before the LDS stores that wait for them: requests stay
    // above the first mark, stores below the second; everything else may cross.
    auto loads_above = [&]() __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };
    auto stores_below = [&]() __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0x1 | 0x2 | 0x4 | 0x8 | 0x10 | 0x20 | 0x40 | 0x100); };

    // ---------------- multiply ----------------
    const uint8_t *const my_rec = lds + C::OFF_B + (rg * C::RGR + col) * C::REC;      // + 32 rows: the wave's second tile
    const CentredPatterns cp = centred_patterns<F::BITS>();
    // ---------------- epilogue ----------------
    // w1/w3: even columns hold w1's rows, odd ones w3's: SiLU(u) v, rounded to fp16, collected in LDS (put) so that rows of
    // a leave in 16-byte pieces and their sums per group are taken on the way (copy_out).  w2: put stores.
    auto put = [&](float v, int tk, int wrow) __attribute__((always_inline)) {
        if constexpr (F::LIFTED) v *= A.lower;
        if constexpr (W13) {
            const float other = dpp_f<0xB1>(v);
            if ((lane & 1) == 0)
                *reinterpret_cast<uint16_t *>(lds + C::OFF_A + tk * C::APITCH + rg * C::RGR + wrow) = __builtin_bit_cast(uint16_t, (_Float16)silu_mul(v, other));
        } else {
            const int mrow = row0 + rg * C::RGR + wrow;
            const int row = te_row(A, ex, l_pair[tk], tok0 + tk, part);     // outside the branch: inside it the 2-bit large kernel's totals go through scratch
            if (tk < n_tok && mrow < n_rows) A.ypart[(size_t)row * A.N + mrow] = l_w[tk] * v;
        }
    };
    auto copy_out = [&]() __attribute__((always_inline)) {
        if constexpr (W13) {
            __syncthreads();
            constexpr int CPT = C::ACOLS / 8;                            // 16-byte pieces per token
            for (int p = tid; p < n_tiles * TILE * CPT; p += THREADS) {
                const int tk = p / CPT, c = p % CPT;
                te_copy_out<F::GPU>(A, *reinterpret_cast<const u32x4_t *>(lds + C::OFF_A + tk * C::APITCH + c * 16), tk < n_tok ? l_pair[tk] : -1, rb, C::ACOLS, c);
            }
        } else {
            te_rows_told(A, ex, tok0, n_tok, rb, part, l_pair);
        }
    };

    if constexpr (BIG) {
        auto unpack = [&](h8_t (&b)[2][F::PLANES][4], int bb, int u) __attribute__((always_inline)) {
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                typename F::Raw raw;
                F::read(raw, my_rec + bb * C::BBUF + rt * 32 * C::REC, hh, u);
                F::decode(raw, b[rt]);
            }
        };
        // one unit of the wave's NT token tiles (from LDS address src) into the totals; xsrc: the unit's sums
        auto multiply = [&](auto nt_tag, auto &tot, const h8_t (&b)[2][F::PLANES][4], const uint8_t *src, int bb, int u, const uint8_t *xsrc) __attribute__((always_inline)) {
            constexpr int NT = decltype(nt_tag)::value;
            bf8_t d[2];
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) d[rt] = slots_d(F::factors(my_rec + bb * C::BBUF + rt * 32 * C::REC, lds + C::OFF_D + bb * C::DBUF + (rg * C::RGR + rt * 32 + col) * F::DB, hh, u));
#pragma unroll
            for (int mt = 0; mt < NT; ++mt) {
                h8_t a[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) a[k] = *reinterpret_cast<const h8_t *>(src + mt * 32 * C::PITCH + k * 16);
                const uint2 xv = *reinterpret_cast<const uint2 *>(xsrc + mt * 32 * C::XPITCH);
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int pl = 0; pl < F::PLANES; ++pl)
#pragma unroll
                        for (int rt = 0; rt < 2; ++rt) tot[rt][mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[k], b[rt][pl][k], tot[rt][mt], 0, 0, 0);
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) tot[rt][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(slots_x(xv), d[rt], tot[rt][mt], 0, 0, 0);
            }
        };
        auto clear = [&](auto nt_tag, auto &tot) __attribute__((always_inline)) {
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int mt = 0; mt < decltype(nt_tag)::value; ++mt)
#pragma unroll
                    for (int i = 0; i < 16; ++i) tot[rt][mt][i] = 0.f;
        };
        // units one by one: activations double buffered per unit, weights per set
        const int nt0 = (n_tiles + 1) / 2;
        {
            Acts t;
            fetch_a(t, u0);
            fetch_x(t, u0);
            commit_a(t, 0);
            commit_x(t, 0);
            commit_b(f0, 0, 0, u0);
            commit_b(f0, 1, 0, u0);
        }
        __syncthreads();
        auto body = [&](auto nt_tag, auto late_tag) __attribute__((always_inline)) {
            constexpr int NT = decltype(nt_tag)::value;
            constexpr bool LATE = decltype(late_tag)::value;             // unpacks a unit ahead, after its matrix work
            const int tile = LATE ? nt0 : 0;
            f32x16_t tot[2][NT > 0 ? NT : 1];
            clear(nt_tag, tot);
            h8_t b[2][F::PLANES][4];
            if (LATE && NT > 0) unpack(b, 0, 0);
            int bb = 0;
            F f;
            Acts t;
            for (int u = u0; u < u1; u += 4) {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    fetch_a(t, u + s + 1);
                    if (s == 0) fetch_b(f, 0, u + 4);            // weights of the next set in two halves: registers
                    if (s == 1) fetch_b(f, 1, u + 4);
                    fetch_x(t, u + s + 1);
                    loads_above();
                    if constexpr (NT > 0) {
                        if (!LATE) unpack(b, bb, s);
                        multiply(nt_tag, tot, b, lds + (s & 1) * C::ABUF + (tile * 32 + col) * C::PITCH + hh * 64, bb, s,
                                 lds + C::OFF_X + (s & 1) * C::XBUF + (tile * 32 + col) * C::XPITCH + hh * 8);
                        if (LATE) unpack(b, s == 3 ? bb ^ 1 : bb, (s + 1) & 3);
                    }
                    stores_below();
                    commit_a(t, (s & 1) ^ 1);
                    if (s == 0) commit_b(f, 0, bb ^ 1, u + 4);
                    commit_x(t, (s & 1) ^ 1);
                    if (s == 1) commit_b(f, 1, bb ^ 1, u + 4);
                    if (s == 3) bb ^= 1;
                    __syncthreads();
                }
            }
#pragma unroll
            for (int mt = 0; mt < NT; ++mt)
#pragma unroll
                for (int i = 0; i < 16; ++i)
#pragma unroll
                    for (int rt = 0; rt < 2; ++rt) put(tot[rt][mt][i], (tile + mt) * 32 + 8 * (i / 4) + 4 * hh + (i % 4), rt * 32 + col);
            copy_out();
        };
        using std::integral_constant;
        using std::false_type;
        using std::true_type;
        const int nt = half ? n_tiles - nt0 : nt0;               // at most MT
        if (half == 0) {
            if (C::MT == 3 && nt == 3) body(integral_constant<int, C::MT>{}, false_type{});
            else if (nt == 2) body(integral_constant<int, 2>{}, false_type{});
            else body(integral_constant<int, 1>{}, false_type{});
        } else {
            if (C::MT == 3 && nt == 3) body(integral_constant<int, C::MT>{}, true_type{});
            else if (nt == 2) body(integral_constant<int, 2>{}, true_type{});
            else if (nt == 1) body(integral_constant<int, 1>{}, true_type{});
            else body(integral_constant<int, 0>{}, true_type{});
        }
    } else {
        // set by set, the units of a set shared by the waves of a row group; two sets of weights on their way
        constexpr int RROWS = MODE, RT = C::RGR / RROWS, NR = MODE == 32 ? 16 : 4;     // rows of a tile, row tiles of a wave, registers of a tile
        const int rcol = lane % RROWS, kb = lane / RROWS;                // the lane's row of a tile, its half or quarter of a unit
        using Acc = std::conditional_t<MODE == 32, f32x16_t, f32x4_t>;
        auto mm = [&](h8_t a, h8_t b, Acc c) __attribute__((always_inline)) {
            if constexpr (MODE == 32) return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
            else return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
        };
        auto mmb = [&](bf8_t a, bf8_t b, Acc c) __attribute__((always_inline)) {
            if constexpr (MODE == 32) return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
            else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
        };
        Acc tot[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int i = 0; i < NR; ++i) tot[rt][i] = 0.f;
        const uint8_t *const rec0 = lds + C::OFF_B + (rg * C::RGR + rcol) * C::REC;
        // one unit of the wave's rows
        auto unit = [&](int bb, int un) __attribute__((always_inline)) {
            constexpr int KS = MODE == 32 ? 4 : 2;                       // k-steps of a unit
            // k-steps in the order of the lane's codes: its share of the unit, or (groups of 32) of either group
            constexpr int KG = KS / (F::GS ? F::GPU : 1);                // k-steps of a group's product
            const uint8_t *src = lds + bb * C::ABUF + rcol * C::PITCH + un * 128 + kb * (KG * 16);
            h8_t a[KS];
#pragma unroll
            for (int k = 0; k < KS; ++k) a[k] = *reinterpret_cast<const h8_t *>(src + k / KG * 64 + k % KG * 16);
            if constexpr (F::GS) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const uint8_t *rec = rec0 + bb * C::BBUF + rt * RROWS * C::REC;
                    float sc[F::GPU];
#pragma unroll
                    for (int j = 0; j < F::GPU; ++j) sc[j] = *reinterpret_cast<const float *>(rec + F::SOFF + (un * F::GPU + j) * 4);
                    uint32_t t[KS];
                    if constexpr (MODE == 32) {
                        typename F::Raw raw;
                        F::read(raw, rec, kb, un);
                        F::words(raw, t);
                    } else {
                        F::quarter(rec, kb, un, t);
                    }
#pragma unroll
                    for (int j = 0; j < F::GPU; ++j) {
                        Acc g;
#pragma unroll
                        for (int i = 0; i < NR; ++i) g[i] = 0.f;
#pragma unroll
                        for (int k = j * KG; k < (j + 1) * KG; ++k) g = mm(a[k], codes_centred<F::BITS>(t[k], cp), g);
#pragma unroll
                        for (int i = 0; i < NR; ++i) tot[rt][i] = __builtin_fmaf(sc[j], g[i], tot[rt][i]);
                    }
                }
            } else {
                const uint8_t *const xp0 = lds + C::OFF_X + bb * C::XBUF + rcol * C::XPITCH;
                bf8_t xv;
                if constexpr (MODE == 32) xv = slots_x(*reinterpret_cast<const uint2 *>(xp0 + un * 16 + kb * 8));
                else xv = slots3_x(*reinterpret_cast<const uint2 *>(xp0 + un * 32 + kb * 8));          // one group per lane: all of its slots
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const uint8_t *rec = rec0 + bb * C::BBUF + rt * RROWS * C::REC;
                    const uint8_t *drow = lds + C::OFF_D + bb * C::DBUF + (rg * C::RGR + rt * RROWS + rcol) * F::DB;
                    h8_t b[F::PLANES][KS];
                    bf8_t d;
                    if constexpr (MODE == 32) {
                        typename F::Raw raw;
                        F::read(raw, rec, kb, un);
                        F::decode(raw, b);
                        d = slots_d(F::factors(rec, drow, kb, un));
                    } else {
                        const uint2 q = F::quarter(rec, kb, un, b);
                        float v;
                        if constexpr (F::DB > 0) v = *reinterpret_cast<const float *>(drow + un * 16 + kb * 4);
                        else v = lo_half(q.y) - lo_half(q.y) * hi_half(q.y);
                        d = slots3_d(split3(v));
                    }
#pragma unroll
                    for (int k = 0; k < KS; ++k)
#pragma unroll
                        for (int pl = 0; pl < F::PLANES; ++pl) tot[rt] = mm(a[k], b[pl][k], tot[rt]);
                    tot[rt] = mmb(xv, d, tot[rt]);
                }
            }
        };
        // GS: the zero-point term of a set: four groups in one matrix instruction per row tile, or two with tiles of 32
        auto set_term = [&](int bb) __attribute__((always_inline)) {
            constexpr int PER = MODE / 16 * F::GPU / (MODE == 32 ? 2 : 1);
#pragma unroll
            for (int p = 0; p < PER; ++p) {
                const int g = MODE == 32 ? (half * PER + p) * 2 + kb : p * 4 + kb;
                const bf8_t xv = slots3_d(*reinterpret_cast<const uint2 *>(lds + C::OFF_X + bb * C::XBUF + rcol * C::XPITCH + g * 8));
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    tot[rt] = mmb(xv, slots3_x(*reinterpret_cast<const uint2 *>(lds + C::OFF_D + bb * C::DBUF + (rg * C::RGR + rt * RROWS + rcol) * F::DB + g * 8)), tot[rt]);
            }
        };
        // Two sets are on their way, activations as well as weights (one alone takes longer to arrive than a set to multiply)
        Acts t0, t1;
        auto fetch = [&](F &f, Acts &t, int u) __attribute__((always_inline)) {
            fetch_a(t, u);
            fetch_x(t, u);
            for (int h = 0; h < 2; ++h) fetch_b(f, h, u);
        };
        auto commit = [&](const F &f, const Acts &t, int b, int u) __attribute__((always_inline)) {
            commit_a(t, b);
            if constexpr (X_REPEAT) commit_x(t, b);
            for (int h = 0; h < 2; ++h) commit_b(f, h, b, u);
            if constexpr (!X_REPEAT) commit_x(t, b);
        };
        fetch_a(t0, u0);
        fetch_x(t0, u0);
        fetch_a(t1, u0 + 4);
        fetch_x(t1, u0 + 4);
        commit(f0, t0, 0, u0);
        __syncthreads();
        auto set = [&](F &fin, Acts &tin, const F &fout, const Acts &tout, int u, int bb) __attribute__((always_inline)) {
            fetch(fin, tin, u + 8);
            loads_above();
#pragma unroll
            for (int un = 0; un < 4; un += C::KW) unit(bb, un + half);
            if constexpr (F::GS) if (MODE == 32 || half == bb) set_term(bb);
            stores_below();
            commit(fout, tout, bb ^ 1, u + 4);
            __syncthreads();
            if constexpr (!F::GS && F::PLANES == 1) __builtin_amdgcn_sched_barrier(0);   // the next set's work stays behind its own loads: 2-bit, 16 tokens, 173 -> 160 us a step
        };
        for (int u = u0; u < u1; u += 8) {
            set(f0, t0, f1, t1, u, 0);
            set(f1, t1, f0, t0, u + 4, 1);                               // past the end: zeros, one set of work for nothing
        }
        // the waves of a row group hold partial sums of the same outputs: each adds up its share of the row tiles, in the
        // order of the waves
        float *const red = reinterpret_cast<float *>(lds);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int i = 0; i < NR; ++i) red[((wv * RT + rt) * NR + i) * 64 + lane] = tot[rt][i];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RT * NR / C::KW; ++r) {
            const int at = half * (RT * NR / C::KW) + r, rt = at / NR, i = at % NR;
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < C::KW; ++w) v += red[((w * C::RG + rg) * RT * NR + at) * 64 + lane];
            put(v, MODE == 32 ? 8 * (i / 4) + 4 * kb + i % 4 : 4 * kb + i, rt * RROWS + rcol);
        }
        copy_out();
    }
}

}  // namespace moe
