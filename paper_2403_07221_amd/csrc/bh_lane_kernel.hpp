// BH{m} hash of few tokens (Sec. 3.2, eq. "block_acdc"; see bh_hash_kernel.hpp for the definition), gfx950.
//
// bh_hash_kernel hands a workgroup sixteen tokens, the width of a matrix product, whatever the batch: 128 tokens of 1024
// coordinates are then eight workgroups on eight compute units, each with the products of sixteen tokens in a chain.  Here a
// workgroup has T = 2 or 4 tokens and a wave of it 64 consecutive coordinates of each, a coordinate to a lane, and the
// products are fused multiply-adds on the vector ALU: lane j forms acc <- fma(v_c, B[c][j], acc), c ascending from +0, the
// sequence that the definition asks for and that the matrix cores' product makes, so the same bits.
//
// What bounds it: the factors.  Every workgroup reads all of them (1 MB for four factors of d_pad = 1024, block 64), and a
// compute unit takes in 47 bytes per clock from its L2, 27 from beyond; T * 64 multiply-adds a lane and factor (1.9 us with
// T = 4 and four waves a SIMD) and the transform stay below that.  So the operands of the next factor are requested as those
// of the present one are used, all of them at once (16 bytes a lane and request), and no barrier waits for them.
//
//   * v_c is the same for the lanes of a block: the sixteen coordinates 16 q .. 16 q + 15 are held by the sixteen lanes of
//     each row, and v_fmac_f32 takes one of them as a DPP operand (row_newbcast), one instruction per multiply-add;
//   * strides 1 .. 8 of the transform are DPP exchanges as in hash_row_kernel.hpp (lane order, negations undone in the
//     multiplier), strides 16 and 32 swap rows and halves between the registers of two tokens;
//   * strides 64 and up cross waves: the coordinates go through LDS into a layout where a block's number is in the low lane
//     bits, and are DPP exchanges again.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "bh_hash_kernel.hpp"
#include "hash_row_kernel.hpp"

namespace lffn {

// LDS of the kernel in words: two arrays of T tokens, each block of 64 coordinates `pitch` words from the next (the reads of
// one offset in every block then fall on all banks), and the last 16 coordinates of the projection before
template <int LOG2N, int T>
struct BhLane {
    static constexpr int N = 1 << LOG2N;
    static constexpr int NB = N / 64;                        // waves, blocks of 64 coordinates
    static constexpr int PITCH = NB > 1 ? 64 + 64 / NB : 64;
    static constexpr int TOKEN = NB * PITCH;
    static constexpr int WORDS = 2 * T * TOKEN + T * 16;
};

// acc[t] += v[t] of lane C of the row * op, for C = C0 .. C0 + 3 in turn (op: one word a coordinate).  The leading s_nop
// covers the two wait states a DPP read needs after a vector write of the same register.
template <int T, int C0>
__device__ __forceinline__ void bh_fma4(float (&acc)[T], const float (&v)[T], float b0, float b1, float b2, float b3)
{
#define LFFN_BH_FMA(a, x, b, c) "v_fmac_f32_dpp %" #a ", %" #x ", %" #b " row_newbcast:%" #c " row_mask:0xf bank_mask:0xf\n\t"
    static_assert(T == 2 || T == 4, "two or four tokens");
    if constexpr (T == 4) {
        asm volatile("s_nop 1\n\t"
                     LFFN_BH_FMA(0, 4, 8, 12) LFFN_BH_FMA(1, 5, 8, 12) LFFN_BH_FMA(2, 6, 8, 12) LFFN_BH_FMA(3, 7, 8, 12)
                     LFFN_BH_FMA(0, 4, 9, 13) LFFN_BH_FMA(1, 5, 9, 13) LFFN_BH_FMA(2, 6, 9, 13) LFFN_BH_FMA(3, 7, 9, 13)
                     LFFN_BH_FMA(0, 4, 10, 14) LFFN_BH_FMA(1, 5, 10, 14) LFFN_BH_FMA(2, 6, 10, 14) LFFN_BH_FMA(3, 7, 10, 14)
                     LFFN_BH_FMA(0, 4, 11, 15) LFFN_BH_FMA(1, 5, 11, 15) LFFN_BH_FMA(2, 6, 11, 15) LFFN_BH_FMA(3, 7, 11, 15)
                     : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3])
                     : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(b0), "v"(b1), "v"(b2), "v"(b3),
                       "n"(C0), "n"(C0 + 1), "n"(C0 + 2), "n"(C0 + 3));
    } else {
        asm volatile("s_nop 1\n\t"
                     LFFN_BH_FMA(0, 2, 4, 8) LFFN_BH_FMA(1, 3, 4, 8) LFFN_BH_FMA(0, 2, 5, 9) LFFN_BH_FMA(1, 3, 5, 9)
                     LFFN_BH_FMA(0, 2, 6, 10) LFFN_BH_FMA(1, 3, 6, 10) LFFN_BH_FMA(0, 2, 7, 11) LFFN_BH_FMA(1, 3, 7, 11)
                     : "+v"(acc[0]), "+v"(acc[1])
                     : "v"(v[0]), "v"(v[1]), "v"(b0), "v"(b1), "v"(b2), "v"(b3), "n"(C0), "n"(C0 + 1), "n"(C0 + 2), "n"(C0 + 3));
    }
#undef LFFN_BH_FMA
}

// exchange of bit BIT of the position in a row: v[t] += s * v[t] of the partner lane (row_exchange16's butterfly, T registers)
template <int BIT, int T>
__device__ __forceinline__ void bh_exchange(float (&v)[T], float s)
{
#define LFFN_BH_X2(ctrl) "s_nop 1\n\tv_fmac_f32_dpp %0, %0, %2 " ctrl " row_mask:0xf bank_mask:0xf\n\tv_fmac_f32_dpp %1, %1, %2 " ctrl " row_mask:0xf bank_mask:0xf"
#pragma unroll
    for (int t = 0; t < T; t += 2) {
        if constexpr (BIT == 0) asm volatile(LFFN_BH_X2("quad_perm:[1,0,3,2]") : "+v"(v[t]), "+v"(v[t + 1]) : "v"(s));
        else if constexpr (BIT == 1) asm volatile(LFFN_BH_X2("quad_perm:[2,3,0,1]") : "+v"(v[t]), "+v"(v[t + 1]) : "v"(s));
        else if constexpr (BIT == 2) asm volatile(LFFN_BH_X2("row_half_mirror") : "+v"(v[t]), "+v"(v[t + 1]) : "v"(s));
        else asm volatile(LFFN_BH_X2("row_ror:8") : "+v"(v[t]), "+v"(v[t + 1]) : "v"(s));
    }
#undef LFFN_BH_X2
}

// strides 16 and 32 of two tokens' registers (lane rows 0 .. 3 hold coordinates 16 row ..): the swaps bring the partners into
// the same lane of the two registers, and back
__device__ __forceinline__ void bh_rows_stage(float &x, float &y)
{
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    float p = __uint_as_float(a[0]), q = __uint_as_float(a[1]);
    reg_butterfly(p, q);
    auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(p), __float_as_uint(q), false, false);
    auto c = __builtin_amdgcn_permlane32_swap(b[0], b[1], false, false);
    p = __uint_as_float(c[0]), q = __uint_as_float(c[1]);
    reg_butterfly(p, q);
    auto d = __builtin_amdgcn_permlane32_swap(__float_as_uint(p), __float_as_uint(q), false, false);
    x = __uint_as_float(d[0]), y = __uint_as_float(d[1]);
}

// LOG2N: d_pad = 2^LOG2N (64 .. 1024); TB = block / 16 (1, 2, 4); T tokens a workgroup; WEIGHTS: the gather weights too.
// Grid x, y: groups of T tokens; grid z: projections, p_per each (as in bh_hash_kernel's SPLIT form).  Codes and weights go
// out in the ABI layout.
template <int LOG2N, int TB, int T, bool WEIGHTS>
__global__ __launch_bounds__(1 << LOG2N) void bh_lane_kernel(BhArgs a)
{
    using L = BhLane<LOG2N, T>;
    constexpr int N = L::N, NB = L::NB, PITCH = L::PITCH, OL = 64 / NB;
    extern __shared__ uint32_t lds[];
    float *cross = reinterpret_cast<float *>(lds);      // [T][TOKEN]: on the way to the strides that cross waves
    float *vals = cross + T * L::TOKEN;                 // [T][TOKEN]: a factor's input; at the end z
    float *ztail = vals + T * L::TOKEN;                 // [T][16]
    const unsigned tid = threadIdx.x, lane = tid & 63u;
    const unsigned w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned row = lane >> 4, rl = lane & 15u;
    const unsigned c16 = rl ^ ((rl & 4u) ? 3u : 0u);    // the coordinate of its row that this lane stands for
    const int P = a.P;
    const long long t0 = ((long long)blockIdx.y * gridDim.x + blockIdx.x) * T;
    if (t0 >= a.n) return;  // the whole workgroup
    // the projections emitted here, and the first one hashed
    const int pb = (int)blockIdx.z * a.p_per, pe = pb + a.p_per < P ? pb + a.p_per : P;
    const int ps = pb > 0 && a.cross ? pb - 1 : pb;

    // a1: coordinate tid of the tokens: a buffer that ends with them, and zero past it and past the row
    const unsigned esz = a.x_kind ? 2u : 4u;
    const long long left = a.n - t0;
    const __amdgpu_buffer_rsrc_t xs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char *>(static_cast<const char *>(a.x) + t0 * a.d * esz), 0, (int)((left < T ? left : T) * a.d * esz), 0x00020000);
    float xr[T];
    if (a.x_kind) {
        unsigned short bits[T];
#pragma unroll
        for (int t = 0; t < T; ++t)
            bits[t] = __builtin_amdgcn_raw_buffer_load_b16(xs, (int)((int)tid < a.d ? ((unsigned)t * (unsigned)a.d + tid) * 2u : 0x80000000u), 0, 0);
#pragma unroll
        for (int t = 0; t < T; ++t) xr[t] = widen16(bits[t], a.x_kind);
    } else {
#pragma unroll
        for (int t = 0; t < T; ++t)
            xr[t] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xs, (int)((int)tid < a.d ? ((unsigned)t * (unsigned)a.d + tid) * 4u : 0x80000000u), 0, 0));
    }

    // operands: 16-byte piece (ii, g) of a lane: B[16 ii + g + 4 kk][j], kk = 0 .. 3, of its column j (bh_pack_kernel's order)
    const unsigned n_pf = (unsigned)(P * a.n_factors);
    constexpr unsigned FB = (unsigned)N * TB * 64u;     // bytes of a factor
    const __amdgpu_buffer_rsrc_t ops = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.apack), 0, (int)(n_pf * FB), 0x00020000);
    const unsigned op_lane = ((4u * w + row) * (TB * 64u) + c16) * 16u;
    u32x4 op[TB][4];
    auto load_op = [&](unsigned pf, int ii) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
            op[ii][g] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(ops, (int)(op_lane + (unsigned)(ii * 1024 + g * 256)), (int)(pf * FB), 0));
    };
#pragma unroll
    for (int ii = 0; ii < TB; ++ii) load_op((unsigned)(ps * a.n_factors), ii);

    // +1 where the lane holds the lower index of an exchange, -1 where the upper: bits of the coordinate in its row, and of the
    // block in the layout for the strides that cross waves (lane = block bits, mapped like c16, and offset bits above them)
    const float s0 = c16 & 1u ? -1.0f : 1.0f, s1 = c16 & 2u ? -1.0f : 1.0f, s2 = c16 & 4u ? -1.0f : 1.0f, s3 = c16 & 8u ? -1.0f : 1.0f;
    const unsigned xl = lane & (unsigned)(NB - 1);
    const unsigned blk = NB >= 8 ? xl ^ ((xl & 4u) ? 3u : 0u) : xl, off = w * OL + lane / NB;
    const float b0 = blk & 1u ? -1.0f : 1.0f, b1 = blk & 2u ? -1.0f : 1.0f, b2 = blk & 4u ? -1.0f : 1.0f, b3 = blk & 8u ? -1.0f : 1.0f;
    const unsigned a_at = w * PITCH + row * 16u + c16;                       // this lane's coordinate, products and strides below 64
    const unsigned x_at = NB > 1 ? blk * PITCH + off : a_at;                 // ... strides 64 and up
    const unsigned neg = __builtin_popcount(NB > 1 ? (off & 15u) ^ (blk << 4) : c16) & 1u;
    const float mul = neg ? -a.scale : a.scale;
    const unsigned v_at = w * PITCH + row / TB * (TB * 16u) + rl;            // first coordinates of this row's block

    for (int p = ps; p < pe; ++p) {
#pragma unroll
        for (int t = 0; t < T; ++t) vals[t * L::TOKEN + w * PITCH + lane] = xr[t];
        lds_barrier();
        float v[T];
        for (int f = 0; f < a.n_factors; ++f) {
            const unsigned pf = (unsigned)(p * a.n_factors + f);
            const unsigned pf_next = pf + 1 < n_pf ? pf + 1 : pf;  // after the last factor: harmless re-reads
            float vq[TB][T];
#pragma unroll
            for (int ii = 0; ii < TB; ++ii)
#pragma unroll
                for (int t = 0; t < T; ++t) vq[ii][t] = vals[t * L::TOKEN + v_at + 16u * ii];
#pragma unroll
            for (int t = 0; t < T; ++t) v[t] = 0.0f;
#pragma unroll
            for (int ii = 0; ii < TB; ++ii) {
                auto word = [&](int g, int kk) { return __uint_as_float(op[ii][g][kk]); };
                bh_fma4<T, 0>(v, vq[ii], word(0, 0), word(1, 0), word(2, 0), word(3, 0));
                bh_fma4<T, 4>(v, vq[ii], word(0, 1), word(1, 1), word(2, 1), word(3, 1));
                bh_fma4<T, 8>(v, vq[ii], word(0, 2), word(1, 2), word(2, 2), word(3, 2));
                bh_fma4<T, 12>(v, vq[ii], word(0, 3), word(1, 3), word(2, 3), word(3, 3));
                load_op(pf_next, ii);
                __builtin_amdgcn_sched_barrier(0);
            }
            bh_exchange<0>(v, s0);
            bh_exchange<1>(v, s1);
            bh_exchange<2>(v, s2);
            bh_exchange<3>(v, s3);
#pragma unroll
            for (int t = 0; t < T; t += 2) bh_rows_stage(v[t], v[t + 1]);
            if constexpr (NB > 1) {
#pragma unroll
                for (int t = 0; t < T; ++t) cross[t * L::TOKEN + a_at] = v[t];
                lds_barrier();  // (and the waves have read their input: it may be overwritten)
#pragma unroll
                for (int t = 0; t < T; ++t) v[t] = cross[t * L::TOKEN + x_at];
                bh_exchange<0>(v, b0);
                if constexpr (NB > 2) bh_exchange<1>(v, b1);
                if constexpr (NB > 4) bh_exchange<2>(v, b2);
                if constexpr (NB > 8) bh_exchange<3>(v, b3);
            }
#pragma unroll
            for (int t = 0; t < T; ++t) vals[t * L::TOKEN + x_at] = v[t] * mul;
            lds_barrier();
        }
        // ---- a4 and the weights (Sec. 4): the tables that end in this projection, one to a thread and token.  The sums and
        // products are formed in the order of bh_hash_kernel's (registers for tau = 4, 8, 16, else one coordinate after
        // another), so a token's weights have the same bits in every batch.
        const int tau = a.tau, lo = p * N;
        const int jlo = lo / tau;
        int jhi = (lo + N) / tau;
        if (jhi > a.k) jhi = a.k;
        const unsigned ntab = p < pb ? 0u : (unsigned)(jhi - jlo);
        for (unsigned idx = tid; idx < T * ntab; idx += NB * 64u) {
            const unsigned t = idx / ntab;
            const int j = jlo + (int)(idx - t * ntab), first = j * tau - lo;  // may be negative: the table began before
            if (t0 + t >= a.n) continue;
            auto z = [&](int b) {
                const int c = first + b;
                return c < 0 ? ztail[t * 16 + 16 + c] : vals[t * L::TOKEN + (c >> 6) * PITCH + (c & 63)];
            };
            uint32_t code = 0;
            auto ez = [](float az) { return 1.0f + __builtin_amdgcn_exp2f(az * -2.885390082f); };  // 1 + exp(-2 az)
            float sum = 0.0f, prod = 1.0f;
            auto tree = [&](auto tau_c) {  // coordinate g + 4 r: r first, then the pairs of g
                constexpr int R = decltype(tau_c)::value / 4;
                float s[4], q[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    float za[R], e[R];
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const float zb = z(g + 4 * r);
                        code |= (zb >= 0.0f ? 1u : 0u) << (g + 4 * r);
                        za[r] = __builtin_fabsf(zb);
                        if constexpr (WEIGHTS) e[r] = ez(za[r]);
                    }
                    if constexpr (WEIGHTS) {
                        if constexpr (R == 1) s[g] = za[0], q[g] = e[0];
                        else if constexpr (R == 2) s[g] = za[0] + za[1], q[g] = e[0] * e[1];
                        else s[g] = (za[0] + za[1]) + (za[2] + za[3]), q[g] = (e[0] * e[1]) * (e[2] * e[3]);
                    }
                }
                if constexpr (WEIGHTS) sum = (s[0] + s[1]) + (s[2] + s[3]), prod = (q[0] * q[1]) * (q[2] * q[3]);
            };
            if (tau == 8) tree(std::integral_constant<int, 8>{});
            else if (tau == 4) tree(std::integral_constant<int, 4>{});
            else if (tau == 16) tree(std::integral_constant<int, 16>{});
            else
                for (int b = 0; b < tau; ++b) {
                    const float zb = z(b);
                    code |= (zb >= 0.0f ? 1u : 0u) << b;
                    if constexpr (WEIGHTS) {
                        const float az = __builtin_fabsf(zb);
                        sum += az, prod *= ez(az);
                    }
                }
            a.codes[(t0 + t) * a.k + j] = (uint16_t)code;
            if constexpr (WEIGHTS) a.weights[(t0 + t) * a.k + j] = sum * __builtin_amdgcn_rcpf(prod);  // prod >= 1
        }
        if (p + 1 < pe) {
            lds_barrier();  // the tail has been read
            if (tid < T * 16u) ztail[tid] = vals[(tid >> 4) * L::TOKEN + (NB - 1) * PITCH + 48 + (tid & 15u)];
            lds_barrier();  // z has been read: the next projection's input may overwrite it
        }
    }
}

}  // namespace lffn
