// Small-batch forward pass of LookupFFN for gfx950: hash and gather of one or several chained layers in a
// single launch (Sec. 3.1: z = x (D1 H)(D2 H)(D3 H) -- eq. "hadamard" --, tau-bit sign codes, then
// y = sum_j T_j[code_j] -- eq. "lookup"; layer l+1 takes layer l's y as its x).
//
// With a handful of tokens the two-kernel path spends its time in launches and in a chip that is almost
// empty; here one workgroup owns one token for the whole stack, so nothing leaves the compute unit between
// the hash and the gather, nor between layers:
//   * its sixteen waves transform the row, a coordinate to a lane (see StackLane), and a lane for each table cuts the code out
//     of the coordinates' signs and turns it into the byte offset of the selected row, in LDS;
//   * the waves then sum 64 dwords of the row each over the k tables IN ORDER (stack_gather);
//   * the sum goes to LDS as the next layer's input and, after the last layer, to y.
// The additions are the same sequential fp32 sum per output element as the large-batch gather kernels
// make, so a stack run equals the layer-by-layer loop bit for bit.
//
// What bounds it: a chain, and one compute unit's share of everything in it.  8 tokens through 12 layers of 768 (k = 96, three
// rounds) take 66 us, 5.5 a layer: the transform of 30 dependent stages 1.1 (0.37 a round), a trip to memory and the barriers
// between the steps about 1.4, the 288 KB of a token's rows, at some 95 GB/s, 3.  With the transform in one wave, sixteen
// coordinates to a lane, which took 0.64 a round, and 4-byte fetches a pass took 90 us; 4-byte fetches alone 80.5.
//
// Shapes: d_pad = 1024 (512 < d <= 1024); table set below 2 GiB (32-bit buffer offsets); row-major fp32, bf16
// or IEEE half tables, or the prepared (slice-major, fp32) layout.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "bh_hash_kernel.hpp"
#include "gather_lds_kernel.hpp"
#include "hash_kernel.hpp"

namespace lffn {

constexpr int kStackMaxLayers = 32;
constexpr int kStackChunk = 32;   // the row offsets are rounded up to whole chunks of this many
constexpr int kStackFlight = 8;   // fetches, of four rows each, that a wave keeps on the way

struct StackArgs {
    const void *x;  // [n][d], input of the first layer
    void *y;        // [n][d_out], output of the last layer: fp32, or bf16 / IEEE half when y_kind says so
    int y_kind;
    const int8_t *signs[kStackMaxLayers];  // per layer [P][R][1024]
    const char *tables[kStackMaxLayers];   // per layer, all in the same layout
    long long n;
    long long twos;  // forward_stack_kernel: workgroups that take two tokens; those after them take one
    int d, d_out, k, tau, P, n_layers;
    int n_rounds;  // read by forward_small_kernel; forward_stack_kernel has its own as a template parameter
    int x_kind;  // element type of x: 0 fp32, 1 bf16, 2 IEEE half
    float scale;
    uint32_t row_dwords;  // dwords of one table row
    // byte offset of dword q of row r (r = (j << tau) + code), with b = 4q:
    //   (b >> piece_shift) * slice_stride + (b & ((1 << piece_shift) - 1)) + r * row_stride
    // row-major tables: piece_shift = 31 (the quotient is 0), row_stride = bytes of a row;
    // prepared tables: pieces of 1 << piece_shift bytes, row_stride = the piece, slice_stride = k * rows * piece
    uint32_t piece_shift, row_stride;
    uint32_t slice_stride;
    uint32_t table_bytes;  // extent of one layer's tables
};

__host__ __device__ inline int stack_code_words(int k) { return (k + kStackChunk - 1) / kStackChunk * kStackChunk; }
// LDS, per token: two buffers of a row (exchanges of the transform; the second also holds the layers' rows), a byte for the sign of each
// coordinate of the last two projections, the row offsets
constexpr int kStackThreads = 1024;
constexpr int kStackSignWords = 2 * 1024 / 4;
__host__ __device__ inline size_t stack_lds_bytes(int k, int tokens) { return tokens * ((size_t)2 * 1024 + kStackSignWords + stack_code_words(k)) * 4; }
// The range of P and k of the entry point, and with it what it refuses: 64 KB for a 4 KB transpose area, sign strings, the row
// offsets and two rows, which a form of a wave a token took.  It lies within what this kernel needs, stack_lds_bytes(k, 1) <= 64 KB.
__host__ inline bool stack_range_ok(int P, int k)
{
    return ((size_t)kH1024TransposeWords + ((hash_bit_words(P, 1024) + 3) & ~3) + stack_code_words(k) + 2 * 1024) * 4 <= 64 * 1024;
}

// The row offsets lie in LDS as four lists, of the tables j = 0, 1, 2, 3 modulo 4.
__device__ __forceinline__ int stack_offset_at(int j, int n_off) { return (j & 3) * (n_off >> 2) + (j >> 2); }

// a5: a wave sums 64 dwords (64 fp32 columns, 128 16-bit ones) of the k selected rows, in table order, and hands a lane's dword
// of sums to `store`.
//
// What bounds it: the return of the data into registers, by counters: 20 clocks for the 1 KB of a wave's 16-byte fetch, 10 for
// the 256 bytes of a 4-byte one.  So a fetch takes 16 bytes a lane; that no wave idles and enough is on the way it takes them from
// four rows, those of tables 4m .. 4m + 3, one to each row of 16 lanes, and a transpose between lane rows and registers then gives
// each lane its dword of all four, which it adds in order.  8 tokens through 12 layers (k = 96, 768 wide): 4-byte fetches, 64 a wave
// in flight, 80.5 us a pass, 8-byte ones 82.3, 16-byte ones of one row, sixteen a wave, 67 (and 42 against 34 for two layers of 512 MB of
// tables: three or four of the sixteen waves fetched), this 65.9.
// Which fetches may still be on the way has to be plain to the compiler, or it waits for all (two sets of fetches, the second
// requested and added "if there is one", waited for the first set before the second was requested): the loop requests without a
// condition, rows past k being valid ones that are not added.
template <int KIND, class Store>
__device__ __forceinline__ void stack_gather(const StackArgs &a, const char *tables, const uint32_t *rowoff, int n_off,
                                             unsigned tid, int tokens, Store store)
{
    constexpr int D = kStackFlight;
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(tables), 0, (int)a.table_bytes, 0x00020000);
    const unsigned lane = tid & 63u, g = lane >> 4, i = lane & 15u;
    const int n_m = n_off >> 2;                 // fours of tables (a multiple of D)
    const uint32_t per = (a.row_dwords + 63u) >> 6;  // 64-dword pieces of a row; the waves take those of all tokens in turn
    for (uint32_t unit = __builtin_amdgcn_readfirstlane(tid >> 6); unit < per * (uint32_t)tokens; unit += blockDim.x >> 6) {
        const uint32_t token = tokens == 1 ? 0u : unit / per;
        const uint32_t q0 = (unit - token * per) * 64u;
        const uint32_t *list = rowoff + token * (uint32_t)n_off + g * (unsigned)n_m;
        const uint32_t b = (q0 + 4u * i) * 4u;
        // (a lane past the row reads outside the buffer: zeros, and every lane of the wave stays active)
        const bool in = q0 + 4u * i < a.row_dwords;
        const uint32_t voff = in ? (b >> a.piece_shift) * a.slice_stride + (b & ((1u << a.piece_shift) - 1u)) : 0x80000000u;
        float acc0 = 0.0f, acc1 = 0.0f;
        u32x4 r[D];
        auto issue4 = [&](int m, int u0) {      // fetches of fours m .. m + 3
            const uint4 o = *reinterpret_cast<const uint4 *>(list + m);
            r[u0] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(voff + o.x), 0, 0));
            r[u0 + 1] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(voff + o.y), 0, 0));
            r[u0 + 2] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(voff + o.z), 0, 0));
            r[u0 + 3] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(voff + o.w), 0, 0));
        };
        auto add1 = [&](float w) {
            if constexpr (KIND != 0) {
                const float2 e = widen16x2<KIND == 0 ? 1 : KIND>(__float_as_uint(w));
                acc0 += e.x, acc1 += e.y;
            } else {
                acc0 += w;
            }
        };
        auto add = [&](int u, int n) {          // the first n of four tables
            float t[4] = {__uint_as_float(r[u].x), __uint_as_float(r[u].y), __uint_as_float(r[u].z), __uint_as_float(r[u].w)};
            tile_transpose(t);
#pragma unroll
            for (int x = 0; x < 4; ++x)
                if (x < n) add1(t[x]);
            asm volatile("" : "+v"(acc0), "+v"(acc1));
        };
        if (a.k <= 16) {
            issue4(0, 0);
#pragma unroll
            for (int u = 0; u < 4; ++u) add(u, a.k - 4 * u);
        } else {
            issue4(0, 0);
            issue4(4, 4);
            int m = 0;  // the four in r[0]
            for (; 4 * (m + D) < a.k; m += D) {
#pragma unroll
                for (int u0 = 0; u0 < D; u0 += 4) {
#pragma unroll
                    for (int u = u0; u < u0 + 4; ++u) add(u, 4);
                    issue4(m + D + u0, u0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int u = 0; u < D; ++u) add(u, a.k - 4 * (m + u));
        }
        const uint32_t q = q0 + 4u * i + g;
        if (in) store(token, q * (KIND ? 2u : 1u), acc0, acc1);
    }
}

// column `col` of token t's output (and the next one, for 16-bit rows)
template <int KIND>
__device__ __forceinline__ void stack_store_y(const StackArgs &a, long long t, uint32_t col, float acc0, float acc1)
{
    const size_t e = (size_t)t * a.d_out + col;
    if (a.y_kind == kElemF32) {
        static_cast<float *>(a.y)[e] = acc0;
        if constexpr (KIND != 0) static_cast<float *>(a.y)[e + 1] = acc1;
    } else {
        static_cast<uint16_t *>(a.y)[e] = (uint16_t)narrow16(acc0, a.y_kind);
        if constexpr (KIND != 0) static_cast<uint16_t *>(a.y)[e + 1] = (uint16_t)narrow16(acc1, a.y_kind);
    }
}

// The transform of one row by a workgroup of sixteen waves, a coordinate to a lane.  The 10 R butterfly stages walk through the
// bits of the coordinate in ascending order, again and again; the lanes of a wave hold six consecutive bits (modulo 10), a
// window, and the wave's number the other four, so six stages pass between two exchanges through LDS (four exchanges for
// three rounds).  In window W (its first bit) thread t holds coordinate rotl10(p | row << 4 | wave << 6, W): p the position in
// the row of 16 lanes, mapped to lanes as in hash_row_kernel.hpp, so that the window's first four bits are DPP exchanges, one
// fused multiply-add each, which leave the upper coordinate's value negated; the last two bits are a swap of rows or halves
// with a copy of the register, and exact.  The negations are undone at the end of a round, in the multiplier (scale, the next
// round's sign): a partner's value has the same ones, and rounding does not see them.
template <int R, int T>
struct StackLane {
    static constexpr int kStages = 10 * R;
    static constexpr int window(int stage) { return 6 * (stage / 6) % 10; }
    // bits of the coordinate whose stages in round r are DPP exchanges
    static constexpr unsigned negating(int r)
    {
        unsigned m = 0;
        for (int s = 10 * r; s < 10 * r + 10; ++s)
            if (s % 6 < 4) m |= 1u << (s % 10);
        return m;
    }
    unsigned t;                // p | row << 4 | wave << 6
    float s0, s1, s2, s3;      // +1 where the lane holds the lower coordinate of an exchange, -1 where the upper
    float s4, s5;
    uint32_t buf;              // LDS byte address of the exchange buffers: two of 4 KB for each token

    __device__ __forceinline__ void setup(unsigned tid, uint32_t lds_buf)
    {
        const unsigned rl = tid & 15u, p = rl ^ ((rl & 4u) ? 3u : 0u);
        t = p | (tid & ~15u);
        s0 = p & 1u ? -1.0f : 1.0f, s1 = p & 2u ? -1.0f : 1.0f, s2 = p & 4u ? -1.0f : 1.0f, s3 = p & 8u ? -1.0f : 1.0f;
        s4 = tid & 16u ? -1.0f : 1.0f, s5 = tid & 32u ? -1.0f : 1.0f;
        buf = lds_buf;
    }
    template <int W>
    __device__ __forceinline__ unsigned coord() const
    {
        return W == 0 ? t : ((t << W) | (t >> (10 - W))) & 1023u;
    }
    // Where coordinate i lies in an exchange buffer: the six bits of any window the walk has (0, 6, 2, 8, 4) go to 64 banks.
    static __device__ __forceinline__ uint32_t place(unsigned i) { return (i ^ (i >> 6) ^ ((i & 3u) << 4) ^ ((i >> 8) << 4)) * 4u; }
    template <int W>
    __device__ __forceinline__ __attribute__((address_space(3))) float *at(int b, int token) const
    {
        return reinterpret_cast<__attribute__((address_space(3))) float *>((uintptr_t)(buf + (uint32_t)(2 * token + b) * 4096u + place(coord<W>())));
    }
    // v[i] += s * v[i] of the lane at the other end of the exchange of the position's bit Q
    template <int Q>
    static __device__ __forceinline__ void exchange(float (&v)[T], float s)
    {
#pragma unroll
        for (int i = 0; i < T; ++i) {
            if constexpr (Q == 0) asm volatile("s_nop 1\n\tv_fmac_f32_dpp %0, %0, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf" : "+v"(v[i]) : "v"(s));
            else if constexpr (Q == 1) asm volatile("s_nop 1\n\tv_fmac_f32_dpp %0, %0, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf" : "+v"(v[i]) : "v"(s));
            else if constexpr (Q == 2) asm volatile("s_nop 1\n\tv_fmac_f32_dpp %0, %0, %1 row_half_mirror row_mask:0xf bank_mask:0xf" : "+v"(v[i]) : "v"(s));
            else asm volatile("s_nop 1\n\tv_fmac_f32_dpp %0, %0, %1 row_ror:8 row_mask:0xf bank_mask:0xf" : "+v"(v[i]) : "v"(s));
        }
    }
    // stages S .. 10 R - 1; mul[r]: the multiplier at the end of round r
    template <int S>
    __device__ __forceinline__ void stages(float (&v)[T], const float (&mul)[R]) const
    {
        if constexpr (S < kStages) {
            constexpr int Q = S % 6, W = window(S);
            if constexpr (Q == 0 && S > 0) {
                constexpr int b = (S / 6 - 1) & 1;
#pragma unroll
                for (int i = 0; i < T; ++i) *at<window(S - 1)>(b, i) = v[i];
                lds_barrier();
#pragma unroll
                for (int i = 0; i < T; ++i) v[i] = *at<W>(b, i);
            }
            if constexpr (Q < 4) exchange<Q>(v, Q == 0 ? s0 : Q == 1 ? s1 : Q == 2 ? s2 : s3);
#pragma unroll
            for (int i = 0; i < T; ++i) {
                if constexpr (Q == 4) {         // (even rows twice, odd rows twice)
                    auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i]), false, false);
                    v[i] = __builtin_fmaf(__uint_as_float(x[1]), s4, __uint_as_float(x[0]));
                } else if constexpr (Q == 5) {  // (the lower half twice, the upper half twice)
                    auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i]), false, false);
                    v[i] = __builtin_fmaf(__uint_as_float(x[1]), s5, __uint_as_float(x[0]));
                }
                if constexpr (S % 10 == 9) v[i] *= mul[S / 10];
            }
            stages<S + 1>(v, mul);
        }
    }
    // sign bytes of this thread's coordinates: of the first diagonal, and of the next one where a round ends
    template <int RD = 0>
    __device__ __forceinline__ void load_signs(const int8_t *sg, int (&to)[R]) const
    {
        if constexpr (RD < R) {
            to[RD] = sg[RD * 1024 + (int)coord<RD == 0 ? 0 : window(10 * RD - 1)>()];
            load_signs<RD + 1>(sg, to);
        }
    }
    template <int RD = 0>
    __device__ __forceinline__ void multipliers(const int (&sg)[R], float scale, float (&mul)[R]) const
    {
        if constexpr (RD < R) {
            unsigned neg = __builtin_popcount(coord<window(10 * RD + 9)>() & negating(RD)) & 1u;
            if constexpr (RD + 1 < R) neg ^= sg[RD + 1 < R ? RD + 1 : 0] < 0 ? 1u : 0u;
            mul[RD] = neg ? -scale : scale;
            multipliers<RD + 1>(sg, scale, mul);
        }
    }
};

// T tokens a workgroup: one, or two where there are more tokens than compute units (the kernel's registers leave room for one
// workgroup on each): k = 96, 768 wide, us a pass, one / two: 257 tokens 19.2 / 15.4, 512 26.4 / 24.2; 64 wide 512 10.6 / 9.5.
// Beyond whole rounds of two, a remainder of up to a token a compute unit takes one each: 519 tokens, four layers of 768, k = 170, all in
// twos / so 423 / 353, 626 of 1024, k = 96, tau = 4 94.5 / 77.8.
template <int R, int KIND, int T>
__global__ __launch_bounds__(kStackThreads) void forward_stack_kernel(StackArgs a)
{
    constexpr int N = 1024;
    extern __shared__ uint32_t lds[];
    const unsigned tid = threadIdx.x;
    const int P = a.P;
    // per token: the second exchange buffer, free between two transforms, holds the row; [2048] signs, coordinate c of all
    // projections at c % 2048; the row offsets
    float *row = reinterpret_cast<float *>(lds) + N;
    uint8_t *sign = reinterpret_cast<uint8_t *>(lds + T * 2 * N);
    uint32_t *rowoff = lds + T * (2 * N + kStackSignWords);
    const int n_off = stack_code_words(a.k);
    const long long b = (long long)blockIdx.y * gridDim.x + blockIdx.x;
    const bool both = T == 2 && b < a.twos;
    const long long t0 = T == 1 ? b : both ? 2 * b : a.twos + b;
    if (t0 >= a.n) return;  // the whole workgroup
    const int tokens = both && t0 + 2 <= a.n ? 2 : 1;

#pragma unroll
    for (int i = 0; i < T; ++i)
        for (int j = a.k + (int)tid; j < n_off; j += kStackThreads) rowoff[i * n_off + stack_offset_at(j, n_off)] = 0;  // past k: a valid row
    using Lane = StackLane<R, T>;
    Lane L;
    L.setup(tid, (uint32_t)(uintptr_t)lds);
    // a1: the rows, coordinate t of the first window, zero past d
    const bool in_row = (int)L.t < a.d;
    float x[T];
#pragma unroll
    for (int i = 0; i < T; ++i) {
        x[i] = 0.0f;
        if (in_row && i < tokens) {
            const long long e = (t0 + i) * a.d + (int)L.t;
            x[i] = a.x_kind ? widen16(static_cast<const uint16_t *>(a.x)[e], a.x_kind) : static_cast<const float *>(a.x)[e];
        }
    }
    int sg[R];
    L.load_signs(a.signs[0], sg);

    for (int l = 0; l < a.n_layers; ++l) {
        if (l > 0) {
#pragma unroll
            for (int i = 0; i < T; ++i) x[i] = in_row ? row[i * 2 * N + (int)L.t] : 0.0f;
        }
        for (int p = 0; p < P; ++p) {
            float mul[R], v[T];
            L.multipliers(sg, a.scale, mul);
#pragma unroll
            for (int i = 0; i < T; ++i) v[i] = fxor(x[i], sg[0] < 0 ? 0x80000000u : 0u);
            // the signs of the next projection or layer travel meanwhile: each read of them misses the L2
            if (p + 1 < P) L.load_signs(a.signs[l] + (size_t)(p + 1) * R * N, sg);
            else if (l + 1 < a.n_layers) L.load_signs(a.signs[l + 1], sg);
            L.template stages<0>(v, mul);
#pragma unroll
            for (int i = 0; i < T; ++i)
                sign[2048 * i + (((unsigned)p * N + L.template coord<Lane::window(10 * R - 1)>()) & 2047u)] = v[i] >= 0.0f ? 1 : 0;
            lds_barrier();
            // ---- a4: the tables that end in this projection: bytes j tau .. j tau + tau - 1 of the signs, as bits, to the
            // byte offset of row (j << tau) + code
            const int jlo = p * N / a.tau, jend = (p + 1) * N / a.tau, jhi = jend < a.k ? jend : a.k;
            for (int e = (int)tid; e < T * (jhi - jlo); e += kStackThreads) {
                const int i = T == 1 || e < jhi - jlo ? 0 : 1, j = jlo + e - i * (jhi - jlo);
                const unsigned first = (unsigned)j * (unsigned)a.tau;
                uint32_t bits = 0;
#pragma unroll
                for (int q = 0; q < 5; ++q) {  // four bytes of 0 or 1 -> four bits
                    const uint32_t w = *reinterpret_cast<const uint32_t *>(sign + 2048 * i + (((first & ~3u) + 4u * q) & 2047u));
                    bits |= ((w * 0x01020408u >> 24) & 0xFu) << (4 * q);
                }
                const uint32_t code = (bits >> (first & 3u)) & ((1u << a.tau) - 1u);
                rowoff[i * n_off + stack_offset_at(j, n_off)] = (((uint32_t)j << a.tau) + code) * a.row_stride;
            }
        }
        lds_barrier();

        // ---- a5 ------------------------------------------------------------------------------------
        const bool last = l + 1 == a.n_layers;
        stack_gather<KIND>(a, a.tables[l], rowoff, n_off, tid, tokens, [&](uint32_t i, uint32_t col, float acc0, float acc1) {
            if (last) {
                stack_store_y<KIND>(a, t0 + i, col, acc0, acc1);
            } else {
                row[i * 2 * N + col] = acc0;
                if constexpr (KIND != 0) row[i * 2 * N + col + 1] = acc1;
            }
        });
        lds_barrier();
    }
}

}  // namespace lffn
