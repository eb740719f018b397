// BH{m} hash of the LookupFFN forward pass for gfx950 (Sec. 3.2, eq. "block_acdc"):
//   z = x R,  R = prod_{i=1..m} B_i H,  B_i block-diagonal (blocks of 16, 32 or 64), H the
//   Walsh-Hadamard transform scaled by d_pad^(-1/2);  code_j = decimal(sign(z_j)) (Sec. 3.1).
//
// The block-diagonal step is a batch of small dense products over tokens -- the one part of the
// path that is a contraction -- and runs on the matrix cores: per 16-coordinate output tile
// (B^T x^T) with v_mfma_f32_16x16x4f32, 16 tokens along the N dimension.  fp32 MFMA accumulates its
// four products as a chain of fused multiply-adds in ascending k, and chains of MFMAs extend that
// chain, so every output is the same "acc = fma(v_c, B[c][j], acc), c ascending from +0" sequence as a
// plain loop.
//
// Split.  The coordinates of 16 tokens are spread over WPG = d_pad / 256 waves (one wave up to d_pad = 256),
// 256 coordinates = 16 tiles = 64 registers per lane each, so that three waves fit a SIMD.  All of d_pad = 1024 in
// one wave takes 256 data registers and leaves one wave per SIMD, and a lone wave issues one instruction in about
// six clocks (two waves: three).  Measured at d = 768, k = 96, tau = 8, blocks 16 / 32 / 64, one wave against four:
// 16384 tokens 85 / 99 / 131 -> 56 / 70 / 98 us; 128 tokens 72 / 90 / 122 -> 20 / 23 / 30 us; 32768 tokens with
// k = 170, tau = 9 (two projections) and weights, block 64: 576 -> 364 us.
//
// What bounds it: the vector ALU and the fp32 matrix products, whose times add up.  Counters at 32768 tokens, two
// projections, block 64: 524 k clocks of matrix products and 286 k of other vector instructions a SIMD, in 856 k clocks.
// Of the vector instructions of a wave and round two thirds are the butterflies themselves.  At d_pad = 1024 three waves a
// SIMD leave 168 registers: codes only and the window form fit, the weights in registers spill six, outside the factors'
// loop.
//
// Tile layout.  A tile is 16 coordinates x 16 tokens in 4 VGPRs: lane l = (token l % 16, group g = l / 16).
// The product leaves coordinate 4g + r in register r (the MFMA result rows in their own order): strides 1 and
// 2 are register pairs.  A 4 x 4 transpose between lane groups and registers (four row swaps) then makes it
// g + 4r: strides 4 and 8 are register pairs, and register kk is directly the B-operand of k-step kk of the
// next product (k-slot g = coordinate 4*kk + g).
//
// Wave layout.  A wave's 16 tiles are four units of 64 coordinates (whole blocks for every block size).
// Layout A: wave w holds units 4w .. 4w+3; layout B: the unit index has its wave bits and its upper bits
// exchanged (d_pad = 1024: units w, 4+w, 8+w, 12+w), so that the strides that cross waves in A are register
// pairs in B.  Products and strides up to 32 run in either; strides 64 and 128 need A, the ones above B.  The
// exchange is a transpose of (wave, unit) through LDS, the same in both directions, in 16-byte pieces that
// are contiguous over the lanes (no bank conflicts).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "gather_lds_kernel.hpp"
#include "hash_kernel.hpp"

namespace lffn {

constexpr int kBhThreads = 256;
constexpr int kBhWaves = kBhThreads / 64;
constexpr int kBhTok = 16;  // tokens of one MFMA

struct BhArgs {
    const void *x;        // [n][d] fp32, bf16 or IEEE half
    const float *apack;   // packed factors, see bh_pack_kernel
    uint16_t *codes;      // [n][k], or NULL when `packed` is written
    uint32_t *packed;     // packed codes of the staged gather, or NULL
    float *weights;       // weighted variant: gather weights [n][k] (beside `codes`), or NULL
    float *wpk;           // weighted variant: the same table-major, [k][n_pad] (beside `packed`), or NULL
    long long n_pad;
    int packed_shift;     // log2 of the row-piece bytes the packed codes are scaled by
    long long n;
    int d, k, tau, n_factors, P;
    int x_kind;           // element type of x: 0 fp32, 1 bf16, 2 IEEE half
    int x_vec4;           // rows may be read four coordinates at a time (alignment checked by the host)
    float scale;
    int p_per;            // SPLIT: projections per workgroup: grid z covers P; fewer than P only with `codes`
    int cross;            // SPLIT: tables run over from one projection into the next
};

// Shape constants of d_pad = 2^LOG2N.  WINDOW: the weights of a tau other than 4, 8, 16 are formed (z window in LDS).
template <int LOG2N, bool WINDOW>
struct BhShape {
    static constexpr int N = 1 << LOG2N;
    static constexpr int NT = N / 16;               // tiles of a token group
    static constexpr int LT = NT < 16 ? NT : 16;    // tiles in one wave
    static constexpr int NU = LT / 4;               // units of 64 coordinates in one wave
    static constexpr int WPG = NT / LT;             // waves that share a token group
    static constexpr int SETS = kBhWaves / WPG;     // sets of 16 tokens per workgroup
    static constexpr int UPS = WPG > 1 ? 4 / WPG : 0;  // units a wave sends to each other wave
    // exchange phases: 4 / PH tiles of a unit at a time.  One phase has half the barriers, but with the window's other
    // LDS its 48 KB would leave room for two workgroups per compute unit instead of three (32768 tokens, two
    // projections, block 64: 394 against 368 us).
    static constexpr int PH = WINDOW ? 2 : 1;
    static constexpr int TPP = 4 / PH;
    static constexpr int X_BYTES = WPG * (WPG - 1) * UPS * TPP * 1024;  // exchange area of a set
    static constexpr int RUN = N < 256 ? N : 256;   // z window: coordinates per pass
    static constexpr int ZS = RUN + 16 + 1;         // words per token: 16 coordinates before the run; odd stride
};
// LDS of one token set, in words: the exchange area or (at the end of a projection) the z window; the z tail; the bit strings
template <int LOG2N, bool WINDOW>
struct BhLds {
    using S = BhShape<LOG2N, WINDOW>;
    static constexpr int Z = WINDOW ? kBhTok * S::ZS : 0;
    static constexpr int AREA = ((S::X_BYTES / 4 > Z ? S::X_BYTES / 4 : Z) + 3) & ~3;
    static constexpr int TAIL = WINDOW ? kBhTok * 16 : 0;
    __host__ __device__ static int set_words(int P) { return AREA + TAIL + kBhTok * hash_bit_words(P, S::N); }
    __host__ static size_t bytes(int P) { return sizeof(uint32_t) * S::SETS * (size_t)set_words(P); }
};

// Packed factor layout: apack[p][f][o][ii][l][kk], o < N/16 output tiles, ii < b/16 input tiles of
// o's block, l < 64 lanes, kk < 4 k-steps; the element is
//   B_{p,f}[c][j],  c = 16*(first tile of the block + ii) + l/16 + 4*kk,  j = 16*o + l%16
// i.e. exactly the A-operand (row m = l%16, k-slot l/16) of the MFMA that adds input tile ii's
// k-step kk into output tile o.
#if !defined(LFFN_PART) || LFFN_PART == 0  // a plain function: defined by part 0 only of a build in parts
__global__ __launch_bounds__(256) void bh_pack_kernel(const float *bmats, float *apack, int N, int b, long long total)
{
    const int tb = b / 16, nt = N / 16;
    for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (long long)gridDim.x * blockDim.x) {
        const int kk = (int)(idx & 3), l = (int)((idx >> 2) & 63);
        long long rest = idx >> 8;
        const int ii = (int)(rest % tb);
        rest /= tb;
        const int o = (int)(rest % nt);
        const long long pf = rest / nt;  // p * n_factors + f
        const int blk = (16 * o) / b;
        const int c = 16 * (blk * tb + ii) + l / 16 + 4 * kk;
        const int j = 16 * o + l % 16;
        apack[idx] = bmats[((pf * (N / b) + blk) * b + (c - blk * b)) * b + (j - blk * b)];
    }
}
#endif

typedef float mfma_f4 __attribute__((ext_vector_type(4)));

// coordinates 4g + r  ->  g + 4r  (lane group g, register r): a 4 x 4 transpose between lane groups and registers
__device__ __forceinline__ void tile_transpose(float (&t)[4])
{
    // swap16 exchanges (first, odd rows) with (second, even rows); swap32 (first, upper half) with (second, lower half)
    auto s01 = __builtin_amdgcn_permlane16_swap(__float_as_uint(t[0]), __float_as_uint(t[1]), false, false);
    auto s23 = __builtin_amdgcn_permlane16_swap(__float_as_uint(t[2]), __float_as_uint(t[3]), false, false);
    auto s02 = __builtin_amdgcn_permlane32_swap(s01[0], s23[0], false, false);
    auto s13 = __builtin_amdgcn_permlane32_swap(s01[1], s23[1], false, false);
    t[0] = __uint_as_float(s02[0]);
    t[1] = __uint_as_float(s13[0]);
    t[2] = __uint_as_float(s02[1]);
    t[3] = __uint_as_float(s13[1]);
}

__device__ __forceinline__ void reg_butterfly(float &a, float &c)
{
    const float x0 = a, x1 = c;
    a = x0 + x1;
    c = x0 - x1;
}

// strides 1, 2 (coordinate 4g + r in register r), the transpose, strides 4, 8 (coordinate g + 4r)
__device__ __forceinline__ void tile_stages(float (&t)[4])
{
    reg_butterfly(t[0], t[1]);
    reg_butterfly(t[2], t[3]);
    reg_butterfly(t[0], t[2]);
    reg_butterfly(t[1], t[3]);
    tile_transpose(t);
    reg_butterfly(t[0], t[1]);
    reg_butterfly(t[2], t[3]);
    reg_butterfly(t[0], t[2]);
    reg_butterfly(t[1], t[3]);
}

// Reduction over the four lane groups (rows of 16 lanes) of two registers at once: returns a register
// whose even rows hold op over all rows of x and whose odd rows hold op over all rows of y.
template <bool MUL>
__device__ __forceinline__ float reduce_rows(float x, float y)
{
    auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    // s[0] = (x.r0, y.r0, x.r2, y.r2), s[1] = (x.r1, y.r1, x.r3, y.r3)
    const float c = MUL ? __uint_as_float(s[0]) * __uint_as_float(s[1]) : __uint_as_float(s[0]) + __uint_as_float(s[1]);
    auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(c), __float_as_uint(c), false, false);
    // t[0] = (c.r0, c.r1, c.r0, c.r1), t[1] = (c.r2, c.r3, c.r2, c.r3)
    return MUL ? __uint_as_float(t[0]) * __uint_as_float(t[1]) : __uint_as_float(t[0]) + __uint_as_float(t[1]);
}
__device__ __forceinline__ uint32_t or_rows(uint32_t x, uint32_t y)
{
    auto s = __builtin_amdgcn_permlane16_swap(x, y, false, false);
    const uint32_t c = s[0] | s[1];
    auto t = __builtin_amdgcn_permlane32_swap(c, c, false, false);
    return t[0] | t[1];
}

// Workgroup barrier that orders LDS accesses only: vector-memory loads (operands of the next product) stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// LOG2N: d_pad = 2^LOG2N (64 .. 1024); TB = block / 16 (1, 2, 4).
// WMODE: 0 codes only; 1 also the gather weights of the weighted variant (Sec. 4), for tau = 4, 8 or 16 (a
// table then lies inside one tile); 2 the weights of any other tau, formed from z through a window in LDS.
// FEW: no more workgroups than compute units.  A wave is then alone on its SIMD and each operand quad a trip to the L2 or
// beyond: it keeps up to sixteen in flight instead of four and may use any number of registers for them (built for
// d_pad = 1024, block 64).
//
// SPLIT: projections of few tokens go out over workgroups (grid z, p_per each), which ran one after another in one: a table
// that runs over from the projection before is the business of the workgroup it ends in, which hashes that projection too.
// (A form of its own: the bounds of the projections cost a workgroup that has all of them up to 6 %, 20 tokens of 145, k = 12
// 17.3 -> 18.4 us.)
template <int LOG2N, int TB, int WMODE, bool FEW, bool SPLIT>
__global__ __launch_bounds__(kBhThreads, FEW ? 1 : 3) void bh_hash_kernel(BhArgs a)
{
    using L = BhLds<LOG2N, WMODE == 2>;
    using S = typename L::S;
    constexpr int N = S::N, LT = S::LT, NU = S::NU, WPG = S::WPG, UPS = S::UPS;
    constexpr int LQ = LT * TB;                // operand quads (1 KB: one tile product) per wave and factor
    constexpr int D = FEW ? (LQ < 16 ? LQ : 16) : 4;  // quads in flight (with three waves a SIMD 8 cost spills: 1 - 3 us of 20 - 30)
    constexpr bool kEndB = WPG > 1;            // the layout a projection ends in
    static_assert(LT >= TB && LT % TB == 0 && LT % 4 == 0 && LQ % D == 0, "units hold whole blocks");
    extern __shared__ uint32_t lds[];
    const unsigned tid = threadIdx.x;
    const unsigned lane = tid & 63u;
    const unsigned wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned tl = lane & 15u, g = lane >> 4;
    const unsigned set = wave / WPG, w = wave % WPG;  // token set of the workgroup, wave within it
    const int P = a.P;
    const int n_bitw = hash_bit_words(P, N);
    uint32_t *area = lds + set * (unsigned)L::set_words(P);
    float *ztail = reinterpret_cast<float *>(area + L::AREA);   // [16 tokens][16]
    uint32_t *bits = area + L::AREA + L::TAIL;                  // [16 tokens][n_bitw]
    const float scale = a.scale;
    // first token of the set; blocks past one grid row's limit of work-items continue in the next row
    const long long t0 = (((long long)blockIdx.y * gridDim.x + blockIdx.x) * S::SETS + set) * kBhTok;

    // unit u of this wave in layout A (B = false) or B: index of its 64 coordinates
    auto unit_index = [&](bool B, int u) -> unsigned {
        if constexpr (WPG == 1) return (unsigned)u;
        else if constexpr (WPG == 4) return B ? w + 4u * (unsigned)u : 4u * w + (unsigned)u;
        else return B ? (unsigned)(u & 1) + 2u * w + 4u * (unsigned)(u >> 1) : 4u * w + (unsigned)u;
    };
    // Operand stream: quad qi of factor pf, one dwordx4 per lane straight to registers, D quads ahead of its use,
    // across factors and projections.  At d_pad = 1024 no other wave of the workgroup reads it; at 512 two and below four
    // do, which is no loss against the earlier form of the kernel that shared copies in LDS (65536 tokens, one projection,
    // tau = 8, blocks 16 / 32 / 64, that form against this: d = 256 60 / 75 / 105 -> 45 / 58 / 86 us, d = 512
    // 150 / 142 / 201 -> 87 / 116 / 171).
    // the projections emitted here, and the first one hashed
    const int pb = SPLIT ? (int)blockIdx.z * a.p_per : 0, pe = SPLIT && pb + a.p_per < P ? pb + a.p_per : P;
    const int ps = pb > 0 && a.cross ? pb - 1 : pb;
    const unsigned n_pf = (unsigned)(P * a.n_factors);
    constexpr unsigned UB = 4 * TB * 1024;  // operand bytes of a unit
    const __amdgpu_buffer_rsrc_t ops = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.apack), 0, (int)(n_pf * (N / 64) * UB), 0x00020000);
    // one 32-bit byte offset per unit, formed where it is used (left alone the compiler keeps an address per quad)
    auto load_quad = [&](unsigned pf, bool B, int qi) -> u32x4 {
        unsigned off = (pf * (N / 64) + unit_index(B, qi / (4 * TB))) * UB + (unsigned)(qi % (4 * TB) / 4) * 4096u;
        asm volatile("" : "+s"(off));
        return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(ops, (int)(lane * 16u + (qi % 4) * 1024u), (int)off, 0));
    };
    u32x4 ring[D];
#pragma unroll
    for (int i = 0; i < D; ++i) ring[i] = load_quad((unsigned)(ps * a.n_factors), false, i);

    // Transpose of (wave, unit) between layouts A and B
    auto exchange = [&](float (&v)[LT][4]) {
        if constexpr (WPG > 1) {
#pragma unroll
            for (int ph = 0; ph < S::PH; ++ph) {
                lds_barrier();  // the area is free
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const unsigned o = (unsigned)(u / UPS);  // the other wave
                    if (o != w) {
                        uint32_t *q = area + ((o * (WPG - 1) + (w > o ? w - 1 : w)) * UPS + u % UPS) * (S::TPP * 256) + lane * 4u;
#pragma unroll
                        for (int i = 0; i < S::TPP; ++i) {
                            const float *r = v[4 * u + ph * S::TPP + i];
                            *reinterpret_cast<float4 *>(q + i * 256) = make_float4(r[0], r[1], r[2], r[3]);
                        }
                    }
                }
                lds_barrier();
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const unsigned o = (unsigned)(u / UPS);
                    if (o != w) {
                        const uint32_t *q = area + ((w * (WPG - 1) + (o > w ? o - 1 : o)) * UPS + u % UPS) * (S::TPP * 256) + lane * 4u;
#pragma unroll
                        for (int i = 0; i < S::TPP; ++i) {
                            float *r = v[4 * u + ph * S::TPP + i];
                            const float4 f = *reinterpret_cast<const float4 *>(q + i * 256);
                            r[0] = f.x, r[1] = f.y, r[2] = f.z, r[3] = f.w;
                        }
                    }
                }
            }
        }
    };
    // butterflies between units u and u + h of the wave
    auto unit_stage = [&](float (&v)[LT][4], int h) {
#pragma unroll
        for (int u = 0; u < NU; ++u)
            if ((u & h) == 0 && u + h < NU) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) reg_butterfly(v[4 * u + i][r], v[4 * (u + h) + i][r]);
            }
    };

    // The set's rows as a buffer of their own: coordinates past the row and tokens past the batch lie outside it and
    // read as zero, so the loads are straight-line code, all in flight at once (branches per tile made every load
    // wait for the one before: 16 trips to memory).
    const unsigned esz = a.x_kind ? 2u : 4u;
    const bool x_vec4 = a.x_vec4 != 0;
    const long long set_tokens = a.n - t0 < 0 ? 0 : a.n - t0 < kBhTok ? a.n - t0 : kBhTok;
    const __amdgpu_buffer_rsrc_t xs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char *>(static_cast<const char *>(a.x) + (set_tokens ? t0 : 0) * a.d * esz), 0, (int)(set_tokens * a.d * esz), 0x00020000);
    // offset of coordinate c of this lane's token.  The compiler must not see through the lane's first coordinate (taken
    // anew in each load form) nor re-order the offsets: it would keep all forms' offsets and range masks and spill.
    auto hidden = [](unsigned c) -> unsigned {
        asm volatile("" : "+v"(c));
        return c;
    };
    auto x_off = [&](unsigned c) -> unsigned {
        return hidden(c < (unsigned)a.d ? (tl * (unsigned)a.d + c) * esz : 0x80000000u);
    };

    for (int p = ps; p < pe; ++p) {
        // ---- a1: this wave's coordinates of its tokens in layout A, register r of tile i <-> 16*i + g + 4r
        float v[LT][4];
        if (x_vec4 && !a.x_kind) {
            const unsigned cv = hidden(w * 256u + 4u * g);
            // four coordinates 16*i + 4g .. + 3 in one piece, then the transpose
            u32x4 q[LT];
#pragma unroll
            for (int i = 0; i < LT; ++i)
                q[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xs, (int)x_off(cv + 16u * i), 0, 0));
#pragma unroll
            for (int i = 0; i < LT; ++i) {
#pragma unroll
                for (int r = 0; r < 4; ++r) v[i][r] = __uint_as_float(q[i][r]);
                tile_transpose(v[i]);
            }
        } else if (x_vec4) {
            const unsigned cv = hidden(w * 256u + 4u * g);
            uint2 q[LT];
#pragma unroll
            for (int i = 0; i < LT; ++i)
                q[i] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(xs, (int)x_off(cv + 16u * i), 0, 0));
            auto widen = [&](auto kind) {  // one choice of the element type for the whole row
#pragma unroll
                for (int i = 0; i < LT; ++i) {
                    const float2 lo = widen16x2<decltype(kind)::value>(q[i].x), hi = widen16x2<decltype(kind)::value>(q[i].y);
                    v[i][0] = lo.x, v[i][1] = lo.y, v[i][2] = hi.x, v[i][3] = hi.y;
                }
            };
            if (a.x_kind == kElemBF16) widen(std::integral_constant<int, kElemBF16>{});
            else widen(std::integral_constant<int, kElemF16>{});
#pragma unroll
            for (int i = 0; i < LT; ++i) tile_transpose(v[i]);
        } else if (!a.x_kind) {
            const unsigned cs = hidden(w * 256u + g);
#pragma unroll
            for (int i = 0; i < LT; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    v[i][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xs, (int)x_off(cs + 16u * i + 4u * r), 0, 0));
        } else {
            const unsigned cs = hidden(w * 256u + g);
#pragma unroll
            for (int i = 0; i < LT; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    v[i][r] = widen16(__builtin_amdgcn_raw_buffer_load_b16(xs, (int)x_off(cs + 16u * i + 4u * r), 0, 0), a.x_kind);
        }

        bool layB = false;  // uniform: the layout v is in
        for (int f = 0; f < a.n_factors; ++f) {
            const unsigned pf = (unsigned)(p * a.n_factors + f);
            const unsigned pf_next = pf + 1 < n_pf ? pf + 1 : pf;  // after the last factor: harmless re-reads
            const bool next_B = WPG > 1 && f + 1 < a.n_factors;
            // ---- block-diagonal factor on the matrix cores ---------------------------------
            // A wave whose coordinates are all padding (d_pad = 1024, d <= 768) multiplies its zeros like the others: an
            // infinite or NaN entry makes NaN of them.  Passing over its first factor would save little and cost the
            // codes-only and register-weight forms registers they spill (d = 768, 16384 tokens: block 16 50.7 against 48.8 us, block 64
            // weighted 99.3 against 96.7; two projections of tau = 9, block 64, 32768 tokens 363 against 366).
#pragma unroll
            for (int blk = 0; blk < LT / TB; ++blk) {
                mfma_f4 acc[TB];
#pragma unroll
                for (int o = 0; o < TB; ++o) {
                    acc[o] = mfma_f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int ii = 0; ii < TB; ++ii) {
                        const int qi = (blk * TB + o) * TB + ii;
                        const u32x4 cur = ring[qi % D];
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk)
                            acc[o] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                __uint_as_float(cur[kk]), v[blk * TB + ii][kk], acc[o], 0, 0, 0);
                        ring[qi % D] = qi + D < LQ ? load_quad(pf, layB, qi + D) : load_quad(pf_next, next_B, qi + D - LQ);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
#pragma unroll
                for (int o = 0; o < TB; ++o)
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[blk * TB + o][r] = acc[o][r];
            }

            // ---- Walsh-Hadamard transform, ascending stride, then the scale -----------------
#pragma unroll
            for (int i = 0; i < LT; ++i) tile_stages(v[i]);
#pragma unroll
            for (int h = 1; h < 4; h <<= 1)  // strides 16, 32: tiles of a unit
#pragma unroll
                for (int i = 0; i < LT; ++i)
                    if ((i & h) == 0) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) reg_butterfly(v[i][r], v[i + h][r]);
                    }
            if constexpr (WPG == 2) unit_stage(v, 1);  // stride 64 is inside a wave in both layouts
            if (layB) exchange(v);
            if constexpr (WPG != 2) unit_stage(v, 1);
            unit_stage(v, 2);
            if constexpr (WPG > 1) {
                exchange(v);
                if constexpr (WPG == 4) unit_stage(v, 1);
                unit_stage(v, 2);
                layB = true;
            }
#pragma unroll
            for (int i = 0; i < LT; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) v[i][r] = v[i][r] * scale;
        }

        // ---- weighted variant: w_j = |z_j|_1 / prod_b (1 + exp(-2|z_jb|)) (Sec. 4) --------------
        // A tile holds coordinate g + 4r of its 16 in (lane group g, register r): a table of
        // tau = 4 is one register over the four lane groups, tau = 8 two registers, tau = 16 the
        // whole tile.  Four consecutive tables of a unit are reduced together (two pair reductions, one
        // per half of the lane groups) so that lane group g ends with the weight of table g of the four:
        // one store per lane for four tables.  A unit's weights are computed before their stores.
        if constexpr (WMODE == 1) {  // (no table runs over from one projection into the next: ps == pb)
            auto emit = [&](auto tau_c) {
                constexpr int TAU = decltype(tau_c)::value;
                constexpr int TPQ = TAU / 4;    // tiles per group of four tables (1, 2, 4)
                constexpr int NQ = 4 / TPQ;     // groups of four tables in a unit
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    auto az = [&](int i, int r) { return __builtin_fabsf(v[4 * u + i][r]); };
                    auto ez = [&](int i, int r) {  // 1 + exp(-2|z|)
                        return 1.0f + __builtin_amdgcn_exp2f(__builtin_fabsf(v[4 * u + i][r]) * -2.885390082f);
                    };
                    float res[NQ];
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        float sx[2], sy[2], px[2], py[2];  // [half]: tables 2*half (x) and 2*half + 1 (y) of the four
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            if constexpr (TAU == 4) {
                                sx[h] = az(q, 2 * h);
                                px[h] = ez(q, 2 * h);
                                sy[h] = az(q, 2 * h + 1);
                                py[h] = ez(q, 2 * h + 1);
                            } else if constexpr (TAU == 8) {
                                const int i = 2 * q + h;
                                sx[h] = az(i, 0) + az(i, 1);
                                px[h] = ez(i, 0) * ez(i, 1);
                                sy[h] = az(i, 2) + az(i, 3);
                                py[h] = ez(i, 2) * ez(i, 3);
                            } else {
                                const int ix = 2 * h, iy = ix + 1;
                                sx[h] = (az(ix, 0) + az(ix, 1)) + (az(ix, 2) + az(ix, 3));
                                px[h] = (ez(ix, 0) * ez(ix, 1)) * (ez(ix, 2) * ez(ix, 3));
                                sy[h] = (az(iy, 0) + az(iy, 1)) + (az(iy, 2) + az(iy, 3));
                                py[h] = (ez(iy, 0) * ez(iy, 1)) * (ez(iy, 2) * ez(iy, 3));
                            }
                        }
                        // even lane groups get x's total, odd ones y's; groups 0, 1 keep half 0
                        const float s0 = reduce_rows<false>(sx[0], sy[0]), s1 = reduce_rows<false>(sx[1], sy[1]);
                        const float p0 = reduce_rows<true>(px[0], py[0]), p1 = reduce_rows<true>(px[1], py[1]);
                        res[q] = (g < 2 ? s0 : s1) * __builtin_amdgcn_rcpf(g < 2 ? p0 : p1);
                    }
                    const long long t = t0 + tl;
                    const int j0 = p * (N / TAU) + (int)unit_index(kEndB, u) * (64 / TAU) + (int)g;
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        const int j = j0 + 4 * q;
                        if (t < a.n && j < a.k) {
                            if (a.wpk) a.wpk[wpk_index(j, t, a.n_pad)] = res[q];  // the 16 tokens of a lane group are consecutive
                            else a.weights[t * a.k + j] = res[q];
                        }
                    }
                }
            };
            if (a.tau == 8)
                emit(std::integral_constant<int, 8>{});
            else if (a.tau == 16)
                emit(std::integral_constant<int, 16>{});
            else
                emit(std::integral_constant<int, 4>{});
        }

        // ---- weighted variant for any other tau: a table then straddles tiles (and may run from one
        // projection into the next), so z goes through a window in LDS, RUN coordinates of the set's tokens at
        // a time (in layout B unit q of the four waves together are 256 consecutive coordinates); the set's lanes
        // take a (token, table) pair each and form the same sum and product coordinate by coordinate.  A table is
        // handled in the run that holds its last coordinate; the 16 coordinates before a run are kept (across
        // projections too).
        if constexpr (WMODE == 2) {
            constexpr int RUN = S::RUN, ZS = S::ZS, TOK = kBhTok, UPR = WPG == 4 ? 1 : WPG == 2 ? 2 : NU;  // units per run and wave
            float *zw = reinterpret_cast<float *>(area);
            const int tau = a.tau;
            const unsigned st = w * 64u + lane;  // thread of the set
            constexpr unsigned kSetThreads = WPG * 64u;
#pragma unroll
            for (int q = 0; q < N / RUN; ++q) {
                lds_barrier();  // the window is free (exchange, or the last run's readers); the tail is written
#pragma unroll
                for (int uu = 0; uu < UPR; ++uu) {
                    const int u = q * UPR + uu;
                    float *zt = zw + tl * ZS + 16 + g + 64u * unit_index(kEndB, u) - RUN * q;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int r = 0; r < 4; ++r) zt[16 * i + 4 * r] = v[4 * u + i][r];
                }
                if (p - ps + q > 0)
                    for (unsigned e = st; e < TOK * 16u; e += kSetThreads) zw[(e >> 4) * ZS + (e & 15u)] = ztail[e];
                lds_barrier();
                const unsigned lo = (unsigned)(p * N + RUN * q);  // first coordinate of the run in the bit string
                const int jlo = (int)(lo / (unsigned)tau);
                int jhi = (int)((lo + RUN) / (unsigned)tau);
                if (jhi > a.k) jhi = a.k;
                const int ntab = p < pb ? 0 : jhi - jlo;
                for (int idx = (int)st; idx < TOK * ntab; idx += (int)kSetThreads) {
                    // table-major output: the tokens of a table are neighbours; else a token's tables are
                    const int tt = a.wpk ? (idx & 15) : idx / ntab;
                    const int j = jlo + (a.wpk ? idx >> 4 : idx - tt * ntab);
                    const long long tok = t0 + tt;
                    const float *zz = zw + tt * ZS + 16 + (j * tau - (int)lo);  // may start in the tail
                    float sum = 0.0f, q2 = 1.0f;
                    auto term = [&](auto cnt, int b0) {
                        constexpr int C = decltype(cnt)::value;  // coordinates in flight together
                        float az[C], ez[C];
#pragma unroll
                        for (int b = 0; b < C; ++b) az[b] = __builtin_fabsf(zz[b0 + b]);
#pragma unroll
                        for (int b = 0; b < C; ++b) ez[b] = 1.0f + __builtin_amdgcn_exp2f(az[b] * -2.885390082f);  // exp(-2 az) = 2^(-2 az log2 e)
#pragma unroll
                        for (int b = 0; b < C; ++b) sum += az[b], q2 *= ez[b];
                    };
                    int b0 = 0;
                    for (; b0 + 4 <= tau; b0 += 4) term(std::integral_constant<int, 4>{}, b0);
                    if (tau & 2) term(std::integral_constant<int, 2>{}, b0), b0 += 2;
                    if (tau & 1) term(std::integral_constant<int, 1>{}, b0);
                    const float wt = sum * __builtin_amdgcn_rcpf(q2);  // q2 >= 1
                    if (tok < a.n) {
                        if (a.wpk) a.wpk[wpk_index(j, tok, a.n_pad)] = wt;
                        else a.weights[tok * a.k + j] = wt;
                    }
                }
                // the run's last 16 coordinates become the tail of the next run
                for (unsigned e = st; e < TOK * 16u; e += kSetThreads) ztail[e] = zw[(e >> 4) * ZS + RUN + (e & 15u)];
            }
        }

        // ---- a4: sign bits into the tokens' bit strings.  A unit is two words (tiles 2h, 2h + 1); the four lane
        // groups' bits are OR-ed by row swaps, two words at a time: even rows end with word 0, odd rows with word 1
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            uint32_t m[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                m[h] = 0;
#pragma unroll
                for (int hb = 0; hb < 2; ++hb)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        m[h] |= (v[4 * u + 2 * h + hb][r] >= 0.0f ? 1u : 0u) << (16 * hb + 4 * r);
            }
            const uint32_t both = or_rows(m[0] << g, m[1] << g);
            if (g < 2) bits[tl * n_bitw + p * (N / 32) + 2u * unit_index(kEndB, u) + g] = both;
        }
    }
    lds_barrier();

    // ---- codes: code j = bits [j*tau, (j+1)*tau) of the token's string, little-endian ------
    const uint32_t cmask = (1u << a.tau) - 1u;
    auto code_at = [&](unsigned tt, unsigned j) -> uint32_t {
        const uint32_t *bw = bits + tt * n_bitw;
        const unsigned bit = j * (unsigned)a.tau;
        const unsigned wi = bit >> 5, sh = bit & 31u;
        const unsigned long long both = ((unsigned long long)bw[wi + 1] << 32) | bw[wi];
        return (uint32_t)(both >> sh) & cmask;
    };
    const unsigned st = w * 64u + lane;
    constexpr unsigned kSetThreads = WPG * 64u, TOK = kBhTok;
    if (a.packed) {  // token-contiguous: the set's tokens of a word are neighbours
        for (unsigned idx = st; idx < TOK * (unsigned)(a.k / 2); idx += kSetThreads) {
            const unsigned tt = idx % TOK, s = idx / TOK;
            if (t0 + tt < a.n)
                a.packed[(long long)s * a.n_pad + t0 + tt] =
                    (code_at(tt, 2u * s) << a.packed_shift) | (code_at(tt, 2u * s + 1u) << (16 + a.packed_shift));
        }
        // zero the token padding of the packed layout
        for (unsigned s = blockIdx.x; s < (unsigned)(a.k / 2); s += gridDim.x)
            for (long long t = a.n + tid; t < a.n_pad; t += kBhThreads) a.packed[(long long)s * a.n_pad + t] = 0u;
    } else {
        unsigned jb = 0, je = (unsigned)a.k;
        if (pb > 0) jb = (unsigned)(pb * N) / (unsigned)a.tau;
        if (pe < P) je = (unsigned)(pe * N) / (unsigned)a.tau;
        for (unsigned tt = 0; tt < TOK; ++tt) {
            if (t0 + tt >= a.n) break;
            for (unsigned j = jb + st; j < je; j += kSetThreads) a.codes[(t0 + tt) * a.k + j] = (uint16_t)code_at(tt, j);
        }
    }
}

}  // namespace lffn
