// Small-batch forward pass of one layer for d_pad = 64 .. 512, hash and gather in a single launch (plain sum):
// the counterpart of forward_stack_kernel for the narrower rows of small models.
//
// What bounds it: launches.  The two-kernel path runs a hash kernel that fills a corner of the chip, writes the codes
// to memory, and a second kernel that waits for the first to drain; here a workgroup owns a token, its waves
// take the projections in turn (each wave holds the row and transforms it with the generic hash kernel's own
// butterflies, so the same bits), the sign strings meet in LDS, and the waves then sum the k selected rows in table
// order with forward_stack_kernel's gather.  Two launches / this, us a pass: 64 tokens of 64, k = 8 5.6 / 3.7; 64 tokens of 512,
// k = 256 17.9 / 12.8.  Same sequential fp32 sum, bit-equal to the other kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "forward_stack_kernel.hpp"

namespace lffn {

// LDS: the sign-bit string and the row offsets (each rounded to 16 bytes)
__host__ __device__ inline int small_bit_words(int P, int N) { return (hash_bit_words(P, N) + 3) & ~3; }
__host__ __device__ inline size_t small_lds_bytes(int P, int N, int k)
{
    return ((size_t)small_bit_words(P, N) + stack_code_words(k)) * 4;
}

template <int LOG2N, int KIND>
__global__ __launch_bounds__(1024) void forward_small_kernel(StackArgs a)
{
    static_assert(LOG2N >= 6 && LOG2N <= 9, "whole 64-bit masks per register; wider rows take forward_stack_kernel");
    constexpr int N = 1 << LOG2N, NREG = N / 64;
    extern __shared__ uint32_t lds[];
    const unsigned tid = threadIdx.x;
    const unsigned lane = tid & 63u;
    const unsigned wave = tid >> 6, n_waves = blockDim.x >> 6;
    const int P = a.P, R = a.n_rounds;
    uint32_t *bitw = lds;
    const int n_bitw = small_bit_words(P, N);
    uint32_t *rowoff = bitw + n_bitw;
    const int n_off = stack_code_words(a.k);
    const long long t = (long long)blockIdx.y * gridDim.x + blockIdx.x;
    if (t >= a.n) return;  // the whole workgroup

    // a1: the row, coordinate lane + 64 r in register r (as hash_kernel lays it out)
    float xv[NREG];
#pragma unroll
    for (int r = 0; r < NREG; ++r) {
        const int i = (int)lane + 64 * r;
        float f = 0.0f;
        if (i < a.d)
            f = a.x_kind ? widen16(((const uint16_t *)a.x)[t * a.d + i], a.x_kind) : ((const float *)a.x)[t * a.d + i];
        xv[r] = f;
    }
    for (int p = (int)wave; p < P; p += (int)n_waves) {
        float v[NREG];
#pragma unroll
        for (int r = 0; r < NREG; ++r) v[r] = xv[r];
        const int8_t *D = a.signs[0] + (size_t)p * R * N;
        int8_t sg[NREG];
#pragma unroll
        for (int r = 0; r < NREG; ++r) sg[r] = D[lane + 64 * r];
        for (int rd = 0; rd < R; ++rd) {
            // a2, a3: sign diagonal, transform, scale; the next round's signs travel meanwhile
#pragma unroll
            for (int r = 0; r < NREG; ++r) v[r] = fxor(v[r], sg[r] < 0 ? 0x80000000u : 0u);
            if (rd + 1 < R) {
#pragma unroll
                for (int r = 0; r < NREG; ++r) sg[r] = D[(rd + 1) * N + lane + 64 * r];
            }
            fwht_wave<LOG2N, NREG>(v, lane);
#pragma unroll
            for (int r = 0; r < NREG; ++r) v[r] = v[r] * a.scale;
        }
        // a4: the mask of register r is bits [64r, 64r + 64) of this projection
#pragma unroll
        for (int r = 0; r < NREG; ++r) {
            const unsigned long long m = __builtin_amdgcn_ballot_w64(v[r] >= 0.0f);
            if (lane == 0) {
                bitw[p * (N / 32) + 2 * r] = (uint32_t)m;
                bitw[p * (N / 32) + 2 * r + 1] = (uint32_t)(m >> 32);
            }
        }
    }
    // the words past the last projection are read with the last code's word and shifted out, never used: cleared
    for (int i = P * (N / 32) + (int)tid; i < n_bitw; i += (int)blockDim.x) bitw[i] = 0;
    __syncthreads();
    // row offsets; those past k stay 0, a valid row
    for (int j = (int)tid; j < n_off; j += (int)blockDim.x)
        rowoff[stack_offset_at(j, n_off)] = j < a.k ? (((uint32_t)j << a.tau) + hash_code_at(bitw, (unsigned)j, a.tau)) * a.row_stride : 0u;
    __syncthreads();

    stack_gather<KIND>(a, a.tables[0], rowoff, n_off, tid, 1, [&](uint32_t, uint32_t col, float acc0, float acc1) { stack_store_y<KIND>(a, t, col, acc0, acc1); });
}

}  // namespace lffn
