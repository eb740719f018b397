// Gather step of the LookupFFN forward pass for gfx950:
//   y[t][:] = sum_{j<k} tables[j][code[t][j]][:]        (Sec. 3.1, eq. "lookup")
// and its weighted form y[t][:] = sum_j w[t][j] * tables[j][code[t][j]][:] (Sec. 4; one fused
// multiply-add per element and table, in table order), and the multi-probe form
//   y[t][:] = sum_j sum_{probe <= tau} p[t][j][probe] * tables[j][code ^ flip(probe)][:]
// (Sec. 3.1, eq. "partial_softmax": the selected row, then the rows one bit away, bit 0 first).
//
// Work decomposition.  A table row is cut into column slices of LPT lanes x 16
// bytes (LPT = "lanes per token"); a wavefront handles 64/LPT tokens of one
// slice: lane = (token within the wave, 16-byte piece within the slice).  Each
// lane walks the k tables in order, fetches its 16 bytes of the selected row
// with one dwordx4 load and adds them into fp32 accumulators -- the same
// sequential fp32 sum per output element as a plain loop over j.
//
// Why slices: one slice of all k tables (k * 2^tau * LPT*16 bytes, 3 MiB for
// k = 96, tau = 8, LPT = 8) fits the 4 MiB L2 of one XCD while a whole table
// set (72 MiB) does not.  Blocks are numbered so that the eight XCDs (block b
// runs on XCD b % 8) each sweep all their tokens for one slice before moving
// to the next one, so after first touch the row fetches are L2 hits instead of
// trips to the Infinity Cache / HBM.
//
// What bounds it: with few tokens the wait for codes and rows, with many the L2.  Codes and weights are read eight at
// a time whatever k is (one by one they cost a wait per table: 1001 tokens, 97 half tables, weighted 60 -> 20 us), and
// a launch of fewer than two full workgroups per compute unit goes out as one-wave workgroups.  The multi-probe form
// keeps eight to sixteen rows in flight across table boundaries (64 tokens, 96 tables, tau = 8: gather 136 -> 57 us
// against three rows at a time; 4096 tokens, tau = 11: 1372 -> 1258 us); the other two take a second set of rows in flight
// (DEEP) where there are too few wavefronts for its registers to matter (2000 tokens weighted 48 -> 55 us with it).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "elem16.hpp"

namespace lffn {

constexpr int kGatherThreads = 256;
constexpr int kGatherWaves = kGatherThreads / 64;  // of a full workgroup; few tokens are launched in one-wave workgroups
constexpr int kXcds = 8;

struct GatherArgs {
    const uint16_t *codes;  // [n][k]
    const float *weights;   // [n][k] for the weighted form, [n][k][1+tau] for the multi-probe form, else NULL
    const char *tables;     // [k][rows][d_out] fp32, bf16 or IEEE half
    void *y;                // [n][d_out] fp32, or bf16 / IEEE half when y_kind says so
    int y_kind;             // 0 fp32, 1 bf16, 2 IEEE half
    long long n;
    int k, tau, d_out;
    int nvec;          // 16-byte pieces per row
    int n_slices;      // ceil(nvec / LPT)
    int n_units;       // n_slices * token_splits; a unit = (slice, contiguous range of token blocks)
    int tb_per_unit;   // token blocks in one unit
    int ntb;           // token blocks in total; a token block = (waves of a workgroup) * (64/LPT) tokens
    int xcd_mode;      // 1: block order is XCD-sliced (see above); 0: plain
    int code_stride;   // codes (and weights, and groups of 1 + tau shares) per token in the arrays; k unless
                       // the launch covers only some of the tables
    int four_rows;     // plain sum: 1: four rows of a token in flight; 0: sixteen
    int accumulate;    // 1: the sums start from what y holds (fp32 y, fp32 rows) instead of zero
    // The 16-byte piece q of row r = (j << tau) + code in slice s sits at
    //   tables + (s / spp) * slice_stride + (s % spp) * LPT*16 + r * row_stride + q*16
    // row-major tables: spp = 1, slice_stride = LPT*16, row_stride = bytes of a row; prepared tables
    // (slice-major, PW bytes per row piece): spp = PW / (LPT*16), slice_stride = k * rows * PW, row_stride = PW.
    uint32_t row_stride;
    uint32_t spp;
    unsigned long long slice_stride;
    int deep;          // few wavefronts: DEEP, 8 or 16; else 0
};

// KIND: element type of the rows (0 fp32, 1 bf16, 2 IEEE half)
template <int KIND>
struct Acc {
    static constexpr int W = KIND ? 8 : 4;  // elements in 16 bytes
    float f[W];
    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int i = 0; i < W; ++i) f[i] = 0.0f;
    }
    // Empty asm that "touches" the accumulators: keeps the compiler from sinking the additions
    // past this point (it otherwise defers them to the loop latch, stretching the live ranges
    // of every fetched row).
    __device__ __forceinline__ void pin()
    {
        asm volatile("" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]));
        if constexpr (KIND != 0) asm volatile("" : "+v"(f[4]), "+v"(f[5]), "+v"(f[6]), "+v"(f[7]));
    }
    // the W elements of 16 bytes of a row, widened exactly
    __device__ __forceinline__ void unpack(const uint4 &r, float (&e)[W]) const
    {
        if constexpr (KIND != 0) {
            const float2 a = widen16x2<KIND == 0 ? 1 : KIND>(r.x), b = widen16x2<KIND == 0 ? 1 : KIND>(r.y),
                         c = widen16x2<KIND == 0 ? 1 : KIND>(r.z), d = widen16x2<KIND == 0 ? 1 : KIND>(r.w);
            e[0] = a.x;
            e[1] = a.y;
            e[2] = b.x;
            e[3] = b.y;
            e[4] = c.x;
            e[5] = c.y;
            e[6] = d.x;
            e[7] = d.y;
        } else {
            e[0] = __uint_as_float(r.x);
            e[1] = __uint_as_float(r.y);
            e[2] = __uint_as_float(r.z);
            e[3] = __uint_as_float(r.w);
        }
    }
    __device__ __forceinline__ void add(const uint4 &r)
    {
        float e[W];
        unpack(r, e);
#pragma unroll
        for (int i = 0; i < W; ++i) f[i] += e[i];
    }
    // acc += w * row, one rounding per element
    __device__ __forceinline__ void fma(const uint4 &r, float w)
    {
        float e[W];
        unpack(r, e);
#pragma unroll
        for (int i = 0; i < W; ++i) f[i] = __builtin_fmaf(w, e[i], f[i]);
    }
};

// Eight consecutive codes of a token.  A token's codes start at any 2-byte boundary (k may be odd), so the 16 bytes
// are one load of that alignment, which the hardware takes.
struct CodeChunk {
    uint32_t c[4];
    __device__ __forceinline__ void load(const uint16_t *codes) { __builtin_memcpy(c, codes, 16); }
    // the first M codes only
    template <int M>
    __device__ __forceinline__ void load_first(const uint16_t *codes)
    {
        c[0] = c[1] = c[2] = c[3] = 0;
        __builtin_memcpy(c, codes, 2 * M);
    }
    // m < 8 codes; the places past them repeat the last one
    __device__ __forceinline__ void load_part(const uint16_t *codes, int m)
    {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            c[u] = codes[2 * u < m ? 2 * u : m - 1] | ((uint32_t)codes[2 * u + 1 < m ? 2 * u + 1 : m - 1] << 16);
    }
    __device__ __forceinline__ uint32_t code(int u) const { return (u & 1) ? (c[u >> 1] >> 16) : (c[u >> 1] & 0xFFFFu); }
    // code 1 becomes code 0, and so on
    __device__ __forceinline__ void next()
    {
#pragma unroll
        for (int u = 0; u < 3; ++u) c[u] = __builtin_amdgcn_alignbit(c[u + 1], c[u], 16);
        c[3] >>= 16;
    }
};

// eight consecutive values from any 4-byte boundary
__device__ __forceinline__ void load_floats8(const float *p, float (&f)[8])
{
    __builtin_memcpy(&f[0], p, 16);
    __builtin_memcpy(&f[4], p + 4, 16);
}

// f(the number `rest`, 1 .. 7, as a constant); nothing for 0
template <class F>
__device__ __forceinline__ void left_over(int rest, F f)
{
    switch (rest) {
        case 1: f(std::integral_constant<int, 1>{}); break;
        case 2: f(std::integral_constant<int, 2>{}); break;
        case 3: f(std::integral_constant<int, 3>{}); break;
        case 4: f(std::integral_constant<int, 4>{}); break;
        case 5: f(std::integral_constant<int, 5>{}); break;
        case 6: f(std::integral_constant<int, 6>{}); break;
        case 7: f(std::integral_constant<int, 7>{}); break;
    }
}

// WMODE: 0 = plain sum, 1 = weighted form, 2 = multi-probe form
// DEEP (plain and weighted; 0, 8 or 16): for few wavefronts, whose registers nobody else needs: DEEP rows more are requested
// before DEEP are added, and codes and weights ahead of the rows before them, so that no request waits for an earlier one's data
// (loads return in order: a code requested behind rows is there only when they are).
template <int KIND, int LPT, int WMODE, int DEEP>
__global__ __launch_bounds__(kGatherThreads) void gather_kernel(GatherArgs a)
{
    constexpr int TPW = 64 / LPT;  // tokens per wave
    const unsigned lane = threadIdx.x & 63u;
    const unsigned wave = threadIdx.x >> 6;

    // ---- block -> (slice, token block) -------------------------------------------------
    const unsigned block = blockIdx.y * gridDim.x + blockIdx.x;  // rows of the grid are a multiple of the XCD count
    int unit, tbl;
    if (a.xcd_mode) {
        const int xcd = (int)(block % kXcds);
        const int q = (int)(block / kXcds);
        unit = (q / a.tb_per_unit) * kXcds + xcd;
        tbl = q % a.tb_per_unit;
    } else {
        unit = (int)(block % (unsigned)a.n_units);
        tbl = (int)(block / (unsigned)a.n_units);
    }
    if (unit >= a.n_units) return;
    const int slice = unit % a.n_slices;
    const int tb = (unit / a.n_slices) * a.tb_per_unit + tbl;
    if (tb >= a.ntb) return;

    const long long t = ((long long)tb * (blockDim.x >> 6) + wave) * TPW + lane / LPT;
    const int vec = slice * LPT + (int)(lane % LPT);
    if (t >= a.n || vec >= a.nvec) return;  // no barrier below: early exit is safe

    const uint16_t *crow = a.codes + t * a.code_stride;
    const char *tcol = a.tables + (size_t)((unsigned)slice / a.spp) * (size_t)a.slice_stride +
                       (size_t)((unsigned)slice % a.spp) * (LPT * 16u) + (size_t)(lane % LPT) * 16u;
    const uint32_t rmask = (1u << a.tau) - 1u;
    const uint32_t row_bytes = a.row_stride;
    const int k = a.k, tau = a.tau;

    auto row = [&](int j, uint32_t code) -> uint4 {
        const uint32_t r = ((uint32_t)j << tau) + (code & rmask);
        return *reinterpret_cast<const uint4 *>(tcol + (unsigned long long)r * row_bytes);
    };

    Acc<KIND> acc;
    acc.zero();
    if constexpr (KIND == 0) {
        if (a.accumulate) {
            const float4 y0 = *reinterpret_cast<const float4 *>(static_cast<const float *>(a.y) +
                                                                 (size_t)t * a.d_out + (size_t)vec * 4);
            acc.f[0] = y0.x, acc.f[1] = y0.y, acc.f[2] = y0.z, acc.f[3] = y0.w;
        }
    }

    // Chunks of eight codes; the k % 8 tables left over are fetched together too, by code for their very number.  One
    // form for any number, which fetched seven rows and added `rest` of them, cost up to 40 % of a pass over few tables:
    // 16384 tokens, 768 wide, tau = 6, that form against this one, us: k = 1 15.1 / 11.1, k = 9 27.8 / 20.5, k = 12
    // 28.1 / 23.3; seven left over gain nothing (k = 15 30.0 / 30.2, weighted 34.5 / 35.6).  Requesting the left-over
    // codes with the last whole chunk instead held them through the loop (72 -> 76, 93 -> 102 registers): k = 100
    // weighted 261 -> 286.
    const int nch = k >> 3, rest = k & 7;
    int done = 0;  // tables summed by the deep form: its whole groups
    if constexpr (DEEP != 0) {
        static_assert(WMODE != 2 && (DEEP == 8 || DEEP == 16), "built for the plain and the weighted sum");
        constexpr int GN = DEEP, NC = GN / 8;  // tables of a group, chunks of their codes
        const float *wrow = WMODE == 1 ? a.weights + t * a.code_stride : nullptr;
        const int ng = k / GN;
        if (ng > 0) {
            CodeChunk cc[2][NC];
            float w[2][GN];
            uint4 r[2][GN];
            auto load_codes = [&](CodeChunk(&c)[NC], int g) {
                const int gc = g < ng ? g : ng - 1;
#pragma unroll
                for (int h = 0; h < NC; ++h) c[h].load(crow + gc * GN + h * 8);
            };
            auto load_weights = [&](float(&f)[GN], int g) {
                if constexpr (WMODE == 1) {
                    const int gc = g < ng ? g : ng - 1;
#pragma unroll
                    for (int h = 0; h < NC; ++h) __builtin_memcpy(&f[h * 8], wrow + gc * GN + h * 8, 32);
                }
            };
            auto issue = [&](int g, const CodeChunk(&c)[NC], uint4(&x)[GN]) {
#pragma unroll
                for (int u = 0; u < GN; ++u) x[u] = row(g * GN + u, c[u >> 3].code(u & 7));
                __builtin_amdgcn_sched_barrier(0);
            };
            auto add = [&](const uint4(&x)[GN], const float(&f)[GN]) {
#pragma unroll
                for (int u = 0; u < GN; ++u) {
                    if constexpr (WMODE == 1) acc.fma(x[u], f[u]);
                    else acc.add(x[u]);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            // group g of the pair (g, g + 1): cur = g & 1; the next group's rows go out before this one is added
            auto turn = [&](auto cur_tag, int g) {
                constexpr int C = decltype(cur_tag)::value, X = C ^ 1;
                load_codes(cc[C], g + 2);
                load_weights(w[X], g + 1);
                if (g + 1 < ng) issue(g + 1, cc[X], r[X]);
                add(r[C], w[C]);
            };
            load_codes(cc[0], 0);
            load_weights(w[0], 0);
            load_codes(cc[1], 1);
            issue(0, cc[0], r[0]);
            for (int g = 0; g < ng; g += 2) {
                turn(std::integral_constant<int, 0>{}, g);
                if (g + 1 < ng) turn(std::integral_constant<int, 1>{}, g + 1);
            }
        }
        done = ng * GN;
    }
    if constexpr (WMODE == 2) {
        // The probes of all tables as one sequence, eight rows at a time, the next eight in flight while these are
        // added: entry q is probe q % (tau + 1) of table q / (tau + 1) and its share is wp[q]; table and probe of an
        // entry are the same in every lane.  Eight codes are held, shifted on by one at every table; the next eight are
        // requested ahead of the rows of the group before the one that runs past them, so that the chain of row
        // addresses holds no wait.
        // Codes read by a running index went through LDS, and refilled at a table they made every row in flight arrive
        // first: gather alone, that form against this, us: 51 tokens, 8 tables, tau = 9 22.3 / 8.8; 2000 tokens, 4 tables,
        // tau = 5 22.3 / 8.7; 64 tokens, 96 tables, tau = 8 73 / 53; 16384 tokens, 17 tables, tau = 6 171 / 167; 1 token, 96
        // tables 59.5 / 60.4, 170 tables 94 / 99.  A load of codes with every group cost 7 to 11 % with many tokens, and no more than 128
        // registers (four waves a SIMD, with spills) 40 %.
        const float *wp = a.weights + t * a.code_stride * (tau + 1);
        const int np = tau + 1, total = k * np;
        const uint32_t np_inv = 65536u / (uint32_t)np + 1u;  // x / np = x * np_inv >> 16 for the x <= 24 below
        auto over_np = [&](int x) -> int { return (int)((uint32_t)x * np_inv >> 16); };
        const bool whole = k >= 8;
        CodeChunk c, nx;             // codes from table j on; the next ones if `fresh`
        bool fresh = false;
        int j = 0, pr = 0;           // next entry to fetch
        int held = whole ? 8 : k;    // first table whose code is not in c
        if (whole) c.load(crow);
        else c.load_part(crow, k);
        uint4 r[2][8];
        float w[2][8];
        auto next_row = [&]() -> uint4 {
            const uint32_t g = c.code(0) & rmask;
            const uint4 x = row(j, g ^ ((1u << pr) >> 1));  // probe 0: the selected row; p: bit p - 1 flipped
            if (++pr == np) {
                pr = 0;
                ++j;
                c.next();
            }
            return x;
        };
        auto take_codes = [&] {
            if (!fresh) return;
            const int first = j + 8 <= k ? j : k - 8;
            c = nx;
            for (int s = j - first; s > 0; --s) c.next();
            held = first + 8;
            fresh = false;
        };
        auto issue = [&](int q, int b) {
            take_codes();
            // the group after this one starts at table j2 and ends in table j3
            const int j2 = j + over_np(pr + 8), j3 = j2 + over_np(pr + 8 - (j2 - j) * np + 7);
            if (j2 < k && (j3 < k ? j3 : k - 1) >= held) {
                nx.load(crow + (j2 + 8 <= k ? j2 : k - 8));
                fresh = true;
            }
            load_floats8(wp + q, w[b]);
#pragma unroll
            for (int u = 0; u < 8; ++u) r[b][u] = next_row();
            __builtin_amdgcn_sched_barrier(0);
        };
        auto add = [&](int b) {
#pragma unroll
            for (int u = 0; u < 8; ++u) acc.fma(r[b][u], w[b][u]);
        };
        // whole groups; inside the loop both requests are unconditional, so that an addition waits for its own rows only
        const int full = total & ~7;
        int q0 = 0;
        if (full) issue(0, 0);
        for (; q0 + 24 <= full; q0 += 16) {
            issue(q0 + 8, 1);
            add(0);
            issue(q0 + 16, 0);
            add(1);
        }
        if (q0 + 16 <= full) {
            issue(q0 + 8, 1);
            add(0);
            add(1);
        } else if (full) {
            add(0);
        }
        if (full < total) take_codes();
        for (int q = full; q < total; ++q) {
            const float wq = wp[q];
            acc.fma(next_row(), wq);
        }
    } else if constexpr (WMODE == 1) {
        const float *wrow = a.weights + t * a.code_stride;
        const int ch0 = DEEP ? done >> 3 : 0;
        if (DEEP ? ch0 < nch : nch) {  // (for the general form `nch > 0` compiles to a loop that is 3 % slower)
            CodeChunk cn;
            float wn[8];
            cn.load(crow + ch0 * 8);
            load_floats8(wrow + ch0 * 8, wn);
            for (int ch = ch0; ch < nch; ++ch) {
                const CodeChunk c = cn;
                float w[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) w[u] = wn[u];
                const int nx = ch + 1 < nch ? ch + 1 : ch;  // next chunk's codes and weights go out first
                cn.load(crow + nx * 8);
                load_floats8(wrow + nx * 8, wn);
                uint4 r[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) r[u] = row(ch * 8 + u, c.code(u));
#pragma unroll
                for (int u = 0; u < 8; ++u) acc.fma(r[u], w[u]);
            }
        }
        left_over(rest, [&](auto m) {
            constexpr int M = decltype(m)::value;
            CodeChunk c;
            float w[M];
            c.template load_first<M>(crow + nch * 8);
            __builtin_memcpy(w, wrow + nch * 8, 4 * M);
            uint4 r[M];
#pragma unroll
            for (int u = 0; u < M; ++u) r[u] = row(nch * 8 + u, c.code(u));
#pragma unroll
            for (int u = 0; u < M; ++u) acc.fma(r[u], w[u]);
        });
    } else {
        auto add_rows = [&](auto m, int j0) {  // tables j0 .. j0 + m - 1, all rows in flight
            constexpr int M = decltype(m)::value;
            CodeChunk c;
            c.template load_first<M>(crow + j0);
            uint4 r[M];
#pragma unroll
            for (int u = 0; u < M; ++u) r[u] = row(j0 + u, c.code(u));
#pragma unroll
            for (int u = 0; u < M; ++u) acc.add(r[u]);
        };
        if (!DEEP && a.four_rows) {
            int j0 = 0;
            for (; j0 + 4 <= k; j0 += 4) add_rows(std::integral_constant<int, 4>{}, j0);
            left_over(k & 3, [&](auto m) { add_rows(m, j0); });
        } else {
            int ch = DEEP ? done >> 3 : 0;
            if (!DEEP && nch >= 2) {
                CodeChunk c0, c1;
                c0.load(crow);
                c1.load(crow + 8);
                for (; ch + 2 <= nch; ch += 2) {
                    const CodeChunk u0 = c0, u1 = c1;
                    // fetch the next two code chunks before the row loads of this pair go out
                    const int nx = ch + 2 <= nch - 2 ? ch + 2 : nch - 2;
                    c0.load(crow + nx * 8);
                    c1.load(crow + nx * 8 + 8);
                    uint4 r[16];
#pragma unroll
                    for (int u = 0; u < 8; ++u) r[u] = row(ch * 8 + u, u0.code(u));
#pragma unroll
                    for (int u = 0; u < 8; ++u) r[8 + u] = row(ch * 8 + 8 + u, u1.code(u));
#pragma unroll
                    for (int u = 0; u < 16; ++u) acc.add(r[u]);
                }
            }
            if (ch < nch) {
                CodeChunk u0;
                u0.load(crow + ch * 8);
                uint4 r[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) r[u] = row(ch * 8 + u, u0.code(u));
#pragma unroll
                for (int u = 0; u < 8; ++u) acc.add(r[u]);
            }
            left_over(rest, [&](auto m) { add_rows(m, nch * 8); });
        }
    }

    // ---- a6: store, streaming (y is written once and not read again here) -------------
    const size_t e = (size_t)t * a.d_out + (size_t)vec * Acc<KIND>::W;
    store_y4(a.y, e, acc.f[0], acc.f[1], acc.f[2], acc.f[3], a.y_kind);
    if constexpr (KIND != 0) store_y4(a.y, e + 4, acc.f[4], acc.f[5], acc.f[6], acc.f[7], a.y_kind);
}

}  // namespace lffn
