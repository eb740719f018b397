// Hash and gather of a batch in one launch, one layer of narrow rows, d_pad = 1024 (Sec. 3.1-3.2; see forward_stack_kernel.hpp), gfx950.
//
// forward_stack_kernel gives a token, or two, a workgroup of sixteen waves whatever the row.  A batch of more tokens than a round of
// those goes through them a few at a time, and with few dwords in a row most waves of the gather have none.  Here a token's
// workgroup has a wave to 64 dwords of its row, and the first of them transforms the token as hash1024_kernel does (the same
// round functions, so the same bits): a compute unit holds several, one's transform beside another's gather.
//
// What bounds it: with few tables the transform, some 280 vector instructions and four trips through LDS a round in one wave of each token; with
// many the return of the rows into registers (see stack_gather).  One layer, us a pass, forward_stack_kernel / here, d = 768, tau = 8, three rounds:
// k = 96, 64 wide 600 tokens 11.0 / 6.7, 15834 171 / 43; k = 24, 384 wide 8000 85 / 70; k = 250, 256 wide 5172 207 / 181.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "forward_stack_kernel.hpp"

namespace lffn {

constexpr int kNarrowDwords = 512;  // dwords of a row, and work-items of a workgroup, at most

// LDS: the transpose area, the sign-bit string and the row offsets (each rounded to 16 bytes)
__host__ __device__ inline int narrow_bit_words(int P) { return (hash_bit_words(P, 1024) + 3) & ~3; }
__host__ __device__ inline size_t narrow_lds_bytes(int P, int k) { return ((size_t)kH1024TransposeWords + narrow_bit_words(P) + stack_code_words(k)) * 4; }

template <int R, int KIND>
__global__ __launch_bounds__(kNarrowDwords) void forward_narrow_kernel(StackArgs a)
{
    constexpr int N = 1024, NREG = 16;
    extern __shared__ uint32_t lds[];
    const unsigned tid = threadIdx.x, lane = tid & 63u;
    const int P = a.P;
    uint32_t *tp = lds, *bitw = tp + kH1024TransposeWords;
    const int n_bitw = narrow_bit_words(P), n_off = stack_code_words(a.k);
    uint32_t *rowoff = bitw + n_bitw;
    const long long t = (long long)blockIdx.y * gridDim.x + blockIdx.x;
    if (t >= a.n) return;  // the whole workgroup

    if (__builtin_amdgcn_readfirstlane((int)(tid >> 6)) == 0) {
        H1024Lane L;
        h1024_lane_setup((uint32_t)(uintptr_t)tp, lane, L);
        float xv[NREG];
        h1024_load_row(a.x, t, a.d, a.x_kind, (a.d % 4) == 0, lane, xv);
        for (int p = 0; p < P; ++p) {
            uint32_t sw[R][4];
#pragma unroll
            for (int rd = 0; rd < R; ++rd) {
                const uint4 w = *reinterpret_cast<const uint4 *>(a.signs[0] + ((size_t)p * R + rd) * N + lane * 16);
                sw[rd][0] = w.x, sw[rd][1] = w.y, sw[rd][2] = w.z, sw[rd][3] = w.w;
            }
            float v[NREG];
#pragma unroll
            for (int e = 0; e < NREG; ++e) v[e] = xv[e];
#pragma unroll
            for (int rd = 0; rd < R; ++rd) {
                if (rd + 1 < R) h1024_round<false>(v, sw[rd], L, lane, a.scale);
                else h1024_round<true>(v, sw[rd], L, lane, a.scale);
            }
            h1024_sign_bits(v, lane, bitw, p);
        }
        // the words past the last projection are read with the last code's word and shifted out, never used: cleared
        for (int i = P * (N / 32) + (int)lane; i < n_bitw; i += 64) bitw[i] = 0;
        wave_lds_fence();
        // row offsets; those past k stay 0, a valid row
        for (int j = (int)lane; j < n_off; j += 64)
            rowoff[stack_offset_at(j, n_off)] = j < a.k ? (((uint32_t)j << a.tau) + hash_code_at(bitw, (unsigned)j, a.tau)) * a.row_stride : 0u;
    }
    lds_barrier();

    stack_gather<KIND>(a, a.tables[0], rowoff, n_off, tid, 1, [&](uint32_t, uint32_t col, float acc0, float acc1) { stack_store_y<KIND>(a, t, col, acc0, acc1); });
}

}  // namespace lffn
