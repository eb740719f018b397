// Hash of few tokens (Sec. 3.2, eq. "hadamard": z = x R, R = D_1 H D_2 H ...; codes, weights and shares as in hash_kernel.hpp),
// d_pad = 64 .. 1024, for gfx950.
//
// The other hash kernels give a token to a wave, or several, and so a lane 8 to 64 coordinates of a transform whose stages wait for
// one another.  Here a workgroup has T = 2 or 4 tokens, a wave 64 consecutive coordinates of each, a lane one: the layouts and
// exchanges of bh_lane_kernel.hpp, without its products.  The butterflies are the textbook loop's, in ascending stride with the
// same roundings, so the same bits, and weights and shares are formed in hash_kernel's order.
//
// What bounds it: a chain; a round is ten dependent stages and two exchanges through LDS.  1000 tokens of 700,
// k = 97, tau = 7, weights: 8.0 us with a token to a wave, 5.5 here; 512 tokens of 768, k = 170, tau = 9 12.7 / 7.9.  A transform
// takes more instructions than in a wave of its own (a lane's copy for every swap of rows, LDS for every round), so larger
// batches keep the others.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bh_lane_kernel.hpp"
#include "hash_kernel.hpp"

namespace lffn {

// Grid x: groups of T tokens; grid y: projections, p_per each (as in hash_kernel's SPLIT form).  Codes (and weights or shares) go
// out in the ABI layout.  WMODE as in hash_kernel.
template <int LOG2N, int T, int WMODE>
__global__ __launch_bounds__(1 << LOG2N) void hash_lane_kernel(HashArgs a)
{
    using L = BhLane<LOG2N, T>;
    constexpr int N = L::N, NB = L::NB, PITCH = L::PITCH, OL = 64 / NB;
    extern __shared__ uint32_t lds[];
    float *cross = reinterpret_cast<float *>(lds);      // [T][TOKEN]: on the way to the strides that cross waves
    float *vals = cross + T * L::TOKEN;                 // [T][TOKEN]: on the way to the next round; at the end z
    float *ztail = vals + T * L::TOKEN;                 // [T][16]
    const unsigned tid = threadIdx.x, lane = tid & 63u;
    const unsigned w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned row = lane >> 4, rl = lane & 15u;
    const unsigned c16 = rl ^ ((rl & 4u) ? 3u : 0u);    // the coordinate of its row that this lane stands for
    const int P = a.P, R = a.n_rounds;
    const long long t0 = (long long)blockIdx.x * T;
    if (t0 >= a.n) return;  // the whole workgroup
    const int pb = (int)blockIdx.y * a.p_per, pe = pb + a.p_per < P ? pb + a.p_per : P;
    const int ps = pb > 0 && a.cross ? pb - 1 : pb;

    // a1: this lane's coordinate of the tokens: a buffer that ends with them, and zero past it and past the row
    const unsigned mine = w * 64u + row * 16u + c16;
    const unsigned esz = a.x_kind ? 2u : 4u;
    const long long left = a.n - t0;
    const __amdgpu_buffer_rsrc_t xs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char *>(static_cast<const char *>(a.x) + t0 * a.d * esz), 0, (int)((left < T ? left : T) * a.d * esz), 0x00020000);
    auto x_off = [&](int t) { return (int)((int)mine < a.d ? ((unsigned)t * (unsigned)a.d + mine) * esz : 0x80000000u); };
    float xr[T];
    if (a.x_kind) {
        unsigned short bits[T];
#pragma unroll
        for (int t = 0; t < T; ++t) bits[t] = __builtin_amdgcn_raw_buffer_load_b16(xs, x_off(t), 0, 0);
#pragma unroll
        for (int t = 0; t < T; ++t) xr[t] = widen16(bits[t], a.x_kind);
    } else {
#pragma unroll
        for (int t = 0; t < T; ++t) xr[t] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xs, x_off(t), 0, 0));
    }
    const int8_t *diag = a.signs + (size_t)ps * R * N + mine;  // this lane's entry of the next diagonal
    int sg = diag[0];

    // (signs of the exchanges, places in LDS and the multiplier that undoes the negations: see bh_lane_kernel)
    const float s0 = c16 & 1u ? -1.0f : 1.0f, s1 = c16 & 2u ? -1.0f : 1.0f, s2 = c16 & 4u ? -1.0f : 1.0f, s3 = c16 & 8u ? -1.0f : 1.0f;
    const unsigned xl = lane & (unsigned)(NB - 1);
    const unsigned blk = NB >= 8 ? xl ^ ((xl & 4u) ? 3u : 0u) : xl, off = w * OL + lane / NB;
    const float b0 = blk & 1u ? -1.0f : 1.0f, b1 = blk & 2u ? -1.0f : 1.0f, b2 = blk & 4u ? -1.0f : 1.0f, b3 = blk & 8u ? -1.0f : 1.0f;
    const unsigned a_at = w * PITCH + row * 16u + c16;
    const unsigned x_at = NB > 1 ? blk * PITCH + off : a_at;
    const unsigned neg = __builtin_popcount(NB > 1 ? (off & 15u) ^ (blk << 4) : c16) & 1u;
    const float mul = neg ? -a.scale : a.scale;

    for (int p = ps; p < pe; ++p) {
        float v[T];
#pragma unroll
        for (int t = 0; t < T; ++t) v[t] = xr[t];
        for (int rd = 0; rd < R; ++rd) {
            // ---- a2, a3
#pragma unroll
            for (int t = 0; t < T; ++t) v[t] = fxor(v[t], sg < 0 ? 0x80000000u : 0u);
            if (rd + 1 < R || p + 1 < pe) diag += N, sg = diag[0];  // travels meanwhile
            bh_exchange<0>(v, s0);
            bh_exchange<1>(v, s1);
            bh_exchange<2>(v, s2);
            bh_exchange<3>(v, s3);
#pragma unroll
            for (int t = 0; t < T; t += 2) bh_rows_stage(v[t], v[t + 1]);
            if constexpr (NB > 1) {
#pragma unroll
                for (int t = 0; t < T; ++t) cross[t * L::TOKEN + a_at] = v[t];
                lds_barrier();  // (and the waves have read their input of this round: it may be overwritten)
#pragma unroll
                for (int t = 0; t < T; ++t) v[t] = cross[t * L::TOKEN + x_at];
                bh_exchange<0>(v, b0);
                if constexpr (NB > 2) bh_exchange<1>(v, b1);
                if constexpr (NB > 4) bh_exchange<2>(v, b2);
                if constexpr (NB > 8) bh_exchange<3>(v, b3);
            }
#pragma unroll
            for (int t = 0; t < T; ++t) v[t] = v[t] * mul;
            if (NB > 1 || rd + 1 == R) {
#pragma unroll
                for (int t = 0; t < T; ++t) vals[t * L::TOKEN + x_at] = v[t];
                lds_barrier();
                if (rd + 1 < R) {
#pragma unroll
                    for (int t = 0; t < T; ++t) v[t] = vals[t * L::TOKEN + a_at];
                }
            }
        }
        // ---- a4, the weights (Sec. 4) and shares (Sec. 3.1): the tables that end in this projection, one to a thread and token
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
            float sum = 0.0f, q = 1.0f;
            for (int b = 0; b < tau; ++b) {
                const float zb = z(b), az = __builtin_fabsf(zb);
                code |= (zb >= 0.0f ? 1u : 0u) << b;
                if constexpr (WMODE == 1) sum += az;
                if constexpr (WMODE != 0) q *= 1.0f + __builtin_amdgcn_exp2f(az * -2.885390082f);  // exp(-2 az) = 2^(-2 az log2 e)
            }
            const long long e = (t0 + t) * a.k + j;
            a.codes[e] = (uint16_t)code;
            if constexpr (WMODE == 1) a.weights[e] = __fdividef(sum, q);
            if constexpr (WMODE == 2) {
                const float p0 = __fdividef(1.0f, q);
                float *out = a.weights + e * (tau + 1);
                out[0] = p0;
                for (int b = 0; b < tau; ++b) out[1 + b] = p0 * __builtin_amdgcn_exp2f(__builtin_fabsf(z(b)) * -2.885390082f);
            }
        }
        if (p + 1 < pe) {
            lds_barrier();  // the tail has been read
            if (tid < T * 16u) ztail[tid] = vals[(tid >> 4) * L::TOKEN + (NB - 1) * PITCH + 48 + (tid & 15u)];
            lds_barrier();  // z has been read: the next projection may overwrite it
        }
    }
}

}  // namespace lffn
