// The large tile kernel for 3- and 4-bit codes: prompts, and batches of more tokens of an expert than a tile of 32.
//
// A block multiplies up to 128 tokens of one expert with 256 memory rows: 8 waves, four row groups of 64 rows times two halves.
// The contraction advances in steps of two units of 64 codes, one unit for either half, so a wave holds 64 rows x 128 tokens and every
// code is unpacked once in the block.  (With the halves sharing the tokens instead, as the kernel before it and the 2-bit one do, each unpacks all of
// its rows' codes: 144 of 340 vector instructions a unit and SIMD where it is 72 of 245.)  At the end either half gives the other one row
// tile's sums, through LDS.  Arithmetic, zero-point term and the order of the additions inside a unit are k_tile's (the head of kernels_tile.h).
//
// Loads go from memory straight to LDS.  One loaded through registers is waited for within the step that requests it, since
// 128 totals, 32 registers of unpacked codes and a product leave none to hold it, and storing it again costs an instruction a piece.  An
// array a buffer: the compiler then knows which requests a read of LDS has to wait for (none: the step before has).  Activations
// are requested a step ahead, piece by piece beside the products (all at once the waves of a compute unit queue for its path to memory
// for 300 to 600 cycles a step: w2 of 1024 tokens 445 -> 392 us), codes and metadata a set (two steps) ahead.  Requests take whole 128-byte
// lines where they can: a line costs that path two cycles, so rows of 64 bytes take twice as long as rows of 128.  Only tiles
// there are get requested (one of nothing takes as long as any other).  The 16-byte pieces of a row are exchanged so that sixteen lanes
// read all 64 banks.
//
// Of the two waves on a SIMD (same rows, other units) one unpacks a step's codes before it multiplies them, the other a set's second step's
// at the end of its first, so that one's vector work runs under the other's matrix work (3950 -> 3730 cycles a step of 128 tokens), which
// goes first (s_setprio; -> 3680).
//
// What bounds it: issue.  A step takes 1480 cycles and 560 for every 32 tokens where an expert's token blocks share its weights, 3350 without any loads at 128; counted with every
// weight read once, 2474 at 32 tokens and 500 for every 32 more.  The matrix cores need 576 for 32 tokens (zero-point term 64), and beside them run 483 vector instructions
// a SIMD at 128 tokens, 281 at 32, at four cycles each while the matrix cores work: 144 unpack, 256 scale.  w1/w3 of 1024 tokens: vector unit 52 %, matrix unit 45 %, waiting 30 %.
// What did not gain: each row tile unpacked under the other's products (4500, spills; 2770 against 2560 where there are registers), a
// product scaled under the next, 16x16x32 instructions (they leave two issue slots free where a 32x32x16 leaves six), codes read ahead of the
// barrier.  With all compute units at work the clock is 2.0 to 2.1 GHz of 2.4.
//
// Measured against that kernel (192 tokens, weights and activations through registers, a barrier a unit), 8 experts 4096 x 14336, w1/w3 + w2, us a launch:
// 4-bit 1024 tokens 705 + 355 -> 590 + 332, 512 tokens 433 + 217 -> 336 + 214, 256 tokens 342 + 163 -> 214 + 110, 128 tokens (32-token kernel 198 +
// 96) 184 + 86; 3-bit 512 tokens 444 + 226 -> 345 + 212; two-level 128 tokens 331 + 157 -> 202 + 100.  (One or two tiles
// of an expert are the 32-token kernel's in large 3-bit layers: 64 tokens, a step 224 us, 264 here.)  What a block does beside its units takes
// 7 us and 2 for every 32 tokens: the pair lookup, the first requests, the halves' sums and SiLU.
#pragma once
#include "kernels_tile.h"

namespace moe {

// 16 bytes a lane from memory to LDS, the lanes' one after the other from `to` on; zeros from past the buffer's end
__device__ __forceinline__ void to_lds(__amdgpu_buffer_rsrc_t r, uint8_t *to, uint32_t v, int s)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)to, 16, (int)v, s, 0, 0);
}
// waits until at most N of the wave's requests are on their way and for its reads and stores of LDS, then for the block's other waves
template <int N> __device__ __forceinline__ void arrive()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | 7 << 4 | (N >> 4) << 14);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Format policies.  CODES: bytes of a set's codes in LDS; NB: requests of a wave for them.
template <int FMT> struct Tb;

template <bool META8> struct Tb4 : TeScaled<META8, 256, 512, 4> {
    static constexpr int BITS = 4, CODES = 256 * 128, NB = 4;
    // 8 rows of 128 bytes a request; piece p of row r lies at p ^ (r / 2 % 8)
    struct Src { uint32_t v; };
    static __device__ __forceinline__ Src src(const TeGeom &g, int wv, int lane)
    {
        return {(uint32_t)(lane / 8) * g.stride + (uint32_t)((lane % 8) ^ (wv % 2 * 4 + lane / 16)) * 16u};
    }
    static __device__ __forceinline__ void request(int i, __amdgpu_buffer_rsrc_t rs, const TeGeom &g, const Src &s, uint8_t *b, int row0, int n_rows, int u, int wv)
    {
        const int at = wv + 8 * i;
        to_lds(rs, b + at * 1024, s.v, min(row0 + at * 8, n_rows - 8) * (int)g.stride + u * 32);
    }
    // half hh of the codes of row r, unit 2 s + half of the set
    struct At {
        int v;
        __device__ __forceinline__ At again() const { int x = v; asm volatile("" : "+v"(x)); return {x}; }
    };
    static __device__ __forceinline__ At at(int r, int hh, int half) { return {r * 128 + (((half * 2 + hh) ^ (r >> 1 & 7)) * 16)}; }
    static __device__ __forceinline__ void words(const uint8_t *b, const At &a, int rt, int s, uint32_t (&t)[4])
    {
        const uint4 q = *reinterpret_cast<const uint4 *>(b + (a.v ^ s * 64) + rt * 32 * 128);
        t[0] = q.x; t[1] = q.y; t[2] = q.z; t[3] = q.w;
    }
};
template <> struct Tb<4> : Tb4<false> {};
template <> struct Tb<48> : Tb4<true> {};

// 3 bits: region A, 64 bytes a row and set (16 rows a request, piece p at p ^ (r / 4 % 4)), behind it region B, 32 bytes (32 rows, p ^ (r / 8 % 2))
template <bool META8> struct Tb3 : TeScaled<META8, 256, 512, 3> {
    static constexpr int BITS = 3, CODES = 256 * 128, NB = 3, B_AT = 256 * 64;     // (256 x 96; the rest is for the halves' sums)
    struct Src { uint32_t a, b; };
    static __device__ __forceinline__ Src src(const TeGeom &g, int, int lane)
    {
        return {(uint32_t)(lane / 4) * g.stride + (uint32_t)((lane % 4) ^ (lane / 16)) * 16u,
                (uint32_t)(lane / 2) * g.stride + (uint32_t)((lane % 2) ^ (lane / 16 % 2)) * 16u + g.b_off};
    }
    static __device__ __forceinline__ void request(int i, __amdgpu_buffer_rsrc_t rs, const TeGeom &g, const Src &s, uint8_t *b, int row0, int n_rows, int u, int wv)
    {
        const int at = wv + 8 * i;
        if (i < 2) to_lds(rs, b + at * 1024, s.a, min(row0 + at * 16, n_rows - 16) * (int)g.stride + u * 16);
        else to_lds(rs, b + B_AT + wv * 1024, s.b, min(row0 + wv * 32, n_rows - 32) * (int)g.stride + u * 8);
    }
    struct At {
        int a, b;
        __device__ __forceinline__ At again() const { int x = a, y = b; asm volatile("" : "+v"(x), "+v"(y)); return {x, y}; }
    };
    static __device__ __forceinline__ At at(int r, int hh, int half)
    {
        return {r * 64 + ((half ^ (r >> 2 & 3)) * 16) + hh * 8, B_AT + r * 32 + (r >> 3 & 1) * 16 + half * 8 + hh * 4};
    }
    static __device__ __forceinline__ void words(const uint8_t *b, const At &a, int rt, int s, uint32_t (&t)[4])
    {
        Codes3::Raw r;
        r.a = *reinterpret_cast<const uint2 *>(b + (a.a ^ s * 32) + rt * 32 * 64);
        r.b = *reinterpret_cast<const uint32_t *>(b + (a.b ^ s * 16) + rt * 32 * 32);
        Codes3::words(r, t);
    }
};
template <> struct Tb<3> : Tb3<false> {};
template <> struct Tb<38> : Tb3<true> {};

struct TbCfg {
    static constexpr int THREADS = 512, ROWS = 256, MT = 4, TOK = MT * 32;
    static constexpr int LDS = 4 * TOK * 128 + 2 * 256 * 128 + 2 * ROWS * 16 + ROWS * 32 + TOK * 32 + TOK * 8;     // what the arrays below add up to
    static_assert(LDS <= 160 * 1024, "one block a compute unit");
};

template <int FMT, bool W13>
__global__ __launch_bounds__(512, 2) void k_big(TeArgs A)
{
    using C = TbCfg;
    using F = Tb<FMT>;
    constexpr int THREADS = C::THREADS, ROWS = C::ROWS, TOK = C::TOK;
    // activations of a step, [half][token][128 bytes, piece p at p ^ (token / 2 % 8)], codes and scales of a set
    __shared__ __attribute__((aligned(16))) uint8_t l_a0[2][TOK * 128], l_a1[2][TOK * 128], l_b0[F::CODES], l_b1[F::CODES], l_s0[ROWS * 16], l_s1[ROWS * 16];
    __shared__ __attribute__((aligned(16))) uint8_t l_d[ROWS * 32], l_x[TOK * 32];        // zero-point factors and sums of activations of a set
    __shared__ int32_t l_pair[TOK];
    __shared__ float l_w[TOK];
    const int tid = threadIdx.x, lane = tid & 63, wv = uniform(tid >> 6), col = lane & 31, hh = lane >> 5;
    const int rg = wv % 4, half = wv / 4;

    FewPairs few;
    const TeItem it = te_item<W13>(A, few, [](int count) { return te_token_blocks<TOK, true>(count); });
    if (!it.blob) return;                                                // whole block, before any barrier
    const int k_parts = it.k_parts, rb = it.job / k_parts, part = it.job % k_parts;
    const int tiles = (it.count + 31) / 32, tile0 = it.t * tiles / it.tb, n_tiles = (it.t + 1) * tiles / it.tb - tile0;
    const int tok0 = tile0 * 32, n_tok = min(it.count - tok0, n_tiles * 32);
    const int n_rows = W13 ? 2 * A.N : A.N, row0 = rb * ROWS;
    const int u0 = part * it.units_per_part, u1 = min(A.K / 64, u0 + it.units_per_part);

    // ---------------- requests ----------------
    // What lies past a row's or a part's end is requested like the rest, as far as the buffer goes: nothing multiplies it, except for the second
    // unit of a step at the end of a row of an odd number of units, whose activations have to be zeros.
    const __amdgpu_buffer_rsrc_t w_rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(it.blob + A.mat_off), 0, n_rows * (int)A.stride, 0x00020000);
    const TeGeom geo = {A.stride, A.meta_off, A.meta2_off, A.b_off, A.unit_shift, A.run_shift, A.K / 64};
    const typename F::Src c_src = F::src(geo, wv, lane);
    auto request_b = [&](uint8_t *b, int u, int i) __attribute__((always_inline)) { F::request(i, w_rs, geo, c_src, b, row0, n_rows, u, wv); };
    F f;
    auto fetch_meta = [&](int u) __attribute__((always_inline)) { f.fetch_meta(w_rs, geo, row0, n_rows, u, true, tid); };
    fetch_meta(u0);                                                      // weights need no routing: requested before the pairs are known
#pragma unroll
    for (int i = 0; i < F::NB; ++i) request_b(l_b0, u0, i);
    te_pairs<W13, TOK>(A, few, it, tok0, n_tok, l_pair, l_w);
    __syncthreads();
    const __amdgpu_buffer_rsrc_t x_rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint2 *>(A.xs), 0, (int)A.xs_bytes, 0x00020000);
    auto act_row = [&](int tk) __attribute__((always_inline)) { const int p = l_pair[tk]; return W13 ? p / A.top_k : p; };
    const int xt = wv % 4 * 32 + lane / 2;                               // 32 tokens a request, four waves one each
    const uint32_t x_off = xt < n_tok ? (uint32_t)act_row(xt) * (uint32_t)A.xs_stride * 8u + (uint32_t)(lane % 2) * 16u : TE_NONE;
    auto request_x = [&](int u) __attribute__((always_inline)) {
        if (wv < 4) to_lds(x_rs, l_x + wv * 1024, x_off, u * 8);
    };
    request_x(u0);
    f.template commit_meta<16, 0>(l_s0, l_d, tid);

    // ---------------- the contraction ----------------
    auto again = [&](int v) __attribute__((always_inline)) { asm volatile("" : "+v"(v)); return v; };     // addresses of eleven arrays, kept, don't fit the registers
    const CentredPatterns cp = centred_patterns<F::BITS>();
    const typename F::At c_at = F::at(rg * 64 + col, hh, half);
    const int a_at = col * 128 + (((hh * 4) ^ (col >> 1 & 7)) * 16), s_at = (rg * 64 + col) * 16 + half * 4;
    const int d_at = (rg * 64 + col) * 32 + half * 16 + hh * 8, x_at = col * 32 + half * 16 + hh * 8;
    auto body = [&](auto nt_tag, auto late_tag) __attribute__((always_inline)) {
        constexpr int NT = decltype(nt_tag)::value;
        constexpr bool LATE = decltype(late_tag)::value;
        // activations: a step's 8 NT requests of 8 tokens, NT a wave, unit by unit
        uint32_t a_off[NT];
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const int tk = (wv + 8 * i) % (4 * NT) * 8 + lane / 8;
            a_off[i] = tk < n_tok ? (uint32_t)act_row(tk) * (uint32_t)A.K * 2u + (uint32_t)((lane % 8) ^ (tk >> 1 & 7)) * 16u : TE_NONE;
        }
        auto request_a = [&](uint8_t (&a)[2][TOK * 128], int u, int i) __attribute__((always_inline)) {
            const int k = (wv + 8 * i) / (4 * NT), at = (wv + 8 * i) % (4 * NT);
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(A.act), 0, u + k < u1 ? (int)A.act_bytes : 0, 0x00020000);
            to_lds(rs, a[0] + k * (TOK * 128) + at * 1024, a_off[i], (u + k) * 128);
        };
#pragma unroll
        for (int i = 0; i < NT; ++i) request_a(l_a0, u0, i);
        arrive<0>();
        float tot[2][NT][16];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int mt = 0; mt < NT; ++mt)
#pragma unroll
                for (int i = 0; i < 16; ++i) tot[rt][mt][i] = 0.f;
        h8_t b[2][4];
        auto unpack = [&](const uint8_t *bs, int s) __attribute__((always_inline)) {
            const typename F::At at = c_at.again();
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                uint32_t t[4];
                F::words(bs, at, rt, s, t);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    b[rt][k] = codes_centred<F::BITS>(t[k], cp);
                    if (LATE) asm volatile("" : "+v"(b[rt][k]));         // here, not behind the barrier
                }
            }
        };
        auto multiply = [&](const uint8_t *as, const uint8_t *ss, int s, auto &&beside) __attribute__((always_inline)) {
            const int sl = again(s_at), al = again(a_at);
            float sc[2];
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) sc[rt] = *reinterpret_cast<const float *>(ss + sl + rt * 32 * 16 + s * 8);
            const uint8_t *const ap[4] = {as + al, as + (al ^ 16), as + (al ^ 32), as + (al ^ 48)};
            h8_t a[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) a[k] = *reinterpret_cast<const h8_t *>(ap[k]);
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int mt = 0; mt < NT; ++mt) {
                h8_t n[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) n[k] = mt + 1 < NT ? *reinterpret_cast<const h8_t *>(ap[k] + (mt + 1) * 32 * 128) : a[k];
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) {
                    beside(mt * 2 + rt);
                    f32x16_t g;
#pragma unroll
                    for (int i = 0; i < 16; ++i) g[i] = 0.f;
#pragma unroll
                    for (int k = 0; k < 4; ++k) g = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[k], b[rt][k], g, 0, 0, 0);
#pragma unroll
                    for (int i = 0; i < 16; ++i) tot[rt][mt][i] = __builtin_fmaf(sc[rt], g[i], tot[rt][mt][i]);
                    __builtin_amdgcn_sched_barrier(0);                   // one product in registers at a time
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) a[k] = n[k];
            }
            __builtin_amdgcn_s_setprio(0);
        };
        // the zero-point term of a set, two of its groups for either half
        auto zero_term = [&]() __attribute__((always_inline)) {
            const int dl = again(d_at), xl = again(x_at);
            bf8_t d[2];
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) d[rt] = slots3_d(*reinterpret_cast<const uint2 *>(l_d + dl + rt * 32 * 32));
#pragma unroll
            for (int mt = 0; mt < NT; ++mt) {
                const bf8_t xv = slots3_x(*reinterpret_cast<const uint2 *>(l_x + xl + mt * 32 * 32));
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) {
                    f32x16_t z;
#pragma unroll
                    for (int i = 0; i < 16; ++i) z[i] = tot[rt][mt][i];
                    z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xv, d[rt], z, 0, 0, 0);
#pragma unroll
                    for (int i = 0; i < 16; ++i) tot[rt][mt][i] = z[i];
                }
            }
        };
        using std::integral_constant;
        // Step s of the set at unit u - 2 s.  Of a set's factors and sums there is one copy: read in its first step, replaced in its second.
        auto step = [&](uint8_t (&a)[2][TOK * 128], uint8_t (&a_nxt)[2][TOK * 128], uint8_t *bs, uint8_t *b_nxt, uint8_t *ss, uint8_t *s_nxt, int u, auto s_tag) __attribute__((always_inline)) {
            constexpr int s = decltype(s_tag)::value;
            if (s == 0) fetch_meta(u + 4);
            else request_x(u + 2);
            // requests beside the products: the activations first, they are waited for at the step's end, the codes at the set's
            constexpr int N = NT + (s == 0 ? F::NB : 0), PER = (N + 2 * NT - 1) / (2 * NT);
            auto beside = [&](int p) __attribute__((always_inline)) {
#pragma unroll
                for (int q = p * PER; q < min((p + 1) * PER, N); ++q) {
                    if (q < NT) request_a(a_nxt, u + 2, q);
                    else request_b(b_nxt, u + 4, q - NT);
                }
            };
            __builtin_amdgcn_sched_barrier(0);
            if (!LATE || s == 0) unpack(bs, s);
            multiply(a[half], ss, s, beside);
            if (s == 0) zero_term();
            if (LATE && s == 0) unpack(bs, 1);
            __builtin_amdgcn_sched_barrier(0);
            if (s == 1) f.template commit_meta<16, 0>(s_nxt, l_d, again(tid));
            arrive<s == 0 ? F::NB : 0>();
            __builtin_amdgcn_sched_barrier(0);
        };
        for (int u = u0; u < u1; u += 8) {
            step(l_a0, l_a1, l_b0, l_b1, l_s0, l_s1, u, integral_constant<int, 0>{});
            if (u + 2 >= u1) break;
            step(l_a1, l_a0, l_b0, l_b1, l_s0, l_s1, u + 2, integral_constant<int, 1>{});
            if (u + 4 >= u1) break;
            step(l_a0, l_a1, l_b1, l_b0, l_s1, l_s0, u + 4, integral_constant<int, 0>{});
            if (u + 6 >= u1) break;
            step(l_a1, l_a0, l_b1, l_b0, l_s1, l_s0, u + 6, integral_constant<int, 1>{});
        }
        arrive<0>();                                                     // nothing is on its way to LDS any more

        // ---------------- the halves' sums: either half gives the other one row tile ----------------
        uint8_t *const mine[4] = {half ? l_b0 : l_a0[0], half ? l_b0 + 16384 : l_a0[1], half ? l_b1 : l_a1[0], half ? l_b1 + 16384 : l_a1[1]};
        uint8_t *const theirs[4] = {half ? l_a0[0] : l_b0, half ? l_a0[1] : l_b0 + 16384, half ? l_a1[0] : l_b1, half ? l_a1[1] : l_b1 + 16384};
        const int ex = rg * 4096 + lane * 4;
        float v[NT][16];
#pragma unroll
        for (int mt = 0; mt < NT; ++mt)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                *reinterpret_cast<float *>(mine[mt] + ex + i * 256) = tot[LATE ? 0 : 1][mt][i];
                v[mt][i] = tot[LATE ? 1 : 0][mt][i];
            }
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < NT; ++mt)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float o = *reinterpret_cast<const float *>(theirs[mt] + ex + i * 256);
                v[mt][i] = LATE ? o + v[mt][i] : v[mt][i] + o;           // (a sum of two is the same either way)
            }
        if constexpr (W13) {
            // even rows are w1's, odd ones w3's: of two registers the even lane finishes the first token, the odd one the second
            __syncthreads();
            uint8_t *const out = l_a0[0];                                // [token][256 bytes, piece p at p ^ (token / 4 % 2)]
            const int cl = rg * 32 + half * 16 + (col >> 1);
            uint8_t *const to = out + (4 * hh + (lane & 1)) * 256 + (((cl >> 3) ^ hh) * 16) + (cl & 7) * 2;
#pragma unroll
            for (int mt = 0; mt < NT; ++mt)
#pragma unroll
                for (int i = 0; i < 16; i += 2) {
                    const bool odd = lane & 1;
                    const float got = dpp_f<0xB1>(odd ? v[mt][i] : v[mt][i + 1]);
                    const float r = silu_mul(odd ? got : v[mt][i], odd ? v[mt][i + 1] : got);
                    *reinterpret_cast<uint16_t *>(to + (mt * 32 + 8 * (i / 4) + i % 4) * 256) = __builtin_bit_cast(uint16_t, (_Float16)r);
                }
            __syncthreads();
            for (int p = tid; p < n_tiles * 32 * 16; p += THREADS) {
                const int tk = p / 16, c = p % 16;
                te_copy_out<1>(A, *reinterpret_cast<const u32x4_t *>(out + tk * 256 + (c ^ (tk >> 2 & 1)) * 16), tk < n_tok ? l_pair[tk] : -1, rb, 128, c);
            }
        } else {
            const int mrow = row0 + rg * 64 + half * 32 + col;
#pragma unroll
            for (int mt = 0; mt < NT; ++mt)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int tk = mt * 32 + 8 * (i / 4) + 4 * hh + i % 4;
                    const int row = te_row(A, it, l_pair[tk], tok0 + tk, part);
                    if (tk < n_tok && mrow < n_rows) A.ypart[(size_t)row * A.N + mrow] = l_w[tk] * v[mt][i];
                }
            te_rows_told(A, it, tok0, n_tok, rb, part, l_pair);
        }
    };
    using std::integral_constant;
    auto both = [&](auto nt_tag) __attribute__((always_inline)) {
        if (half) body(nt_tag, std::true_type{});
        else body(nt_tag, std::false_type{});
    };
    if (n_tiles == 4) both(integral_constant<int, 4>{});
    else if (n_tiles == 3) both(integral_constant<int, 3>{});
    else if (n_tiles == 2) both(integral_constant<int, 2>{});
    else both(integral_constant<int, 1>{});
}

}  // namespace moe
