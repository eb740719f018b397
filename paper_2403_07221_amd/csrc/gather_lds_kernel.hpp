// LDS-staged gather for tables of 2^7 .. 2^10 rows (k even, fp32 rows; for an odd k the host gives this
// kernel the first k - 1 tables and lets the direct kernel add the last one onto its sums):
//   y[t][:] = sum_{j<k} tables[j][code[t][j]][:]        (Sec. 3.1, eq. "lookup")
//
// With tau = 8 a table has only 256 rows, so a batch of thousands of tokens
// picks every row many times.  A 1024-thread workgroup owns one column slice
// (128 bytes of every row up to tau = 8 or 9, 64 bytes from tau = 8 or 9 on)
// and a chunk of tokens.  Tables are taken one stage at a time: the slice of
// all 2^tau rows of two tables (one table when it fills a 64 KB buffer) is copied
// into LDS once by global_load_lds (memory -> LDS without a
// trip through registers), double-buffered so that stage s+1 streams in while
// stage s is consumed.  Every (token, 16-byte piece) lane then reads its
// selected row from LDS with one ds_read_b128 (the lanes of a token read one
// contiguous row piece) and adds it to its fp32 accumulators.  Each
// output element is still the sequential fp32 sum over j = 0..k-1, so results
// equal the direct kernel's bit for bit, while the L2 -> CU traffic drops from
// one row per (token, table) to one row per (chunk, table, row).
//
// Codes come in the packed layout written by the hash kernel (one 32-bit word
// per token and stage holding both tables' LDS row offsets, token-contiguous).
// The eight lanes of a token would all hold the same word, so the words are
// quad-shared: each lane keeps only those of the token slots i with i % 4 ==
// its position in its quad, and a use takes the word through a DPP quad
// broadcast -- a quarter of the registers and load instructions, one cache
// line per load.
//
// What bounds it (16384 tokens, k = 96, tau = 8, 768 wide; pass of hash and gather): the hand-over of the stages -- a stage's
// copies must land before the barrier, and a build without any row read took as long as the whole (121 us) -- then the
// bank conflicts of the row reads (no copies: 95 us; neither: 57).  So the next stage's copies are the first thing a stage
// issues (spread over its reads: 112 -> 109 us), nothing may wait for them in mid-stage (scratch reloads did: weighted 165 ->
// 141 us, tau = 10 335 -> 291), and a wave's instructions are laid out so that neighbours do not depend on one another (a
// row's address and weight are formed one slot ahead: 109 -> 105.5 us; multi-probe 1030 -> 729).  With the stages brought
// into the L2 ahead of their copies, more slot counts, and the multi-probe form's lagging groups and shares loaded two sweeps
// ahead, pass before and after all of it: plain 118 -> 100, weighted 165 -> 129, multi-probe 899 -> 663 ... 683, 65536 bf16
// tokens 384 -> 328, tau = 10, k = 128, 1024 wide 335 -> 239, 32768 tokens, k = 256, 512 wide 393 -> 285, tau = 9, k = 170, 32768
// tokens, weighted 873 -> 759 us (the last hashes with BH for 398 of it, unchanged).
//
// Weighted form (Sec. 4: y = sum_j w_j T_j[code_j]): the fp32 weights come table-major and
// token-contiguous (wpk[j][n_pad]) and are quad-shared like the code words; each row is
// accumulated with one fused multiply-add per element.
//
// bf16 tables: the staged copy is fp32.  Widening inside this kernel (per stage and workgroup, through
// registers and LDS writes) measured no faster than the direct kernel, and the tables are learned
// constants, so the widening happens once, outside the forward pass: prepare_tables_kernel (below) writes an
// fp32, slice-major copy that this kernel and the direct kernel read.
//
// Work distribution is static and XCD-aware: slice-units are dealt to the
// eight XCDs round-robin (block b runs on XCD b % 8), and the workgroups of
// one XCD split its units' token ranges evenly, so every CU gets one chunk of
// near-equal size and the slice a CU streams stays in its XCD's L2.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "elem16.hpp"

#include <type_traits>

#include "gather_kernel.hpp"
#include "hash_kernel.hpp"

namespace lffn {

constexpr int kLdsThreads = 1024;
// Lanes per token SW (8 or 4): a token group reads one SW*16-byte row piece, the workgroup owns a
// column slice of that width and kLdsThreads / SW token groups.
constexpr int kLdsBufBytes = 64 * 1024;      // one staging buffer (two of them are in use)
constexpr int kLdsMaxTok = 16;               // token slots per lane the packed padding allows for
// f += r, the sums staying in the registers they are in: left to itself the compiler puts a sum where the row was, the
// accumulators wander through the register file and the 16-slot forms spill
__device__ __forceinline__ void add_in_place(float (&f)[4], const uint4 &r)
{
    asm volatile("v_add_f32 %0, %0, %4\n\tv_add_f32 %1, %1, %5\n\tv_add_f32 %2, %2, %6\n\tv_add_f32 %3, %3, %7"
                 : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3])
                 : "v"(r.x), "v"(r.y), "v"(r.z), "v"(r.w));
}

struct GatherLdsArgs {
    const uint32_t *packed;  // [k/2][n_pad] packed codes (see hash_kernel.hpp)
    const float *wpk;        // weighted form: [k][n_pad] weights, table-major (wpk_index); multi-probe form:
                             // [k][1+tau][n_pad] shares.  The token padding [n, n_pad) is never initialised:
                             // slots past a chunk's end multiply it into accumulators that are never stored.
    long long n_pad;
    const char *tables;      // fp32 rows, row-major [k][rows][d_out] or the slice-major prepared layout
    void *y;            // [n][d_out] fp32, or bf16 / IEEE half when y_kind says so
    int y_kind;         // 0 fp32, 1 bf16, 2 IEEE half
    long long n;
    int k, tau, d_out;
    int nvec;           // 16-byte pieces per row
    int n_slices;       // ceil(nvec / lanes per token)
    int token_splits;   // a unit = (slice, one of token_splits equal token ranges)
    int n_units;        // n_slices * token_splits
    int blocks_per_xcd; // gridDim.x / kXcds
    int unit_chunks;    // (not multi-probe) 0, or the chunks of a unit where the workgroups of an XCD divide all chunks of its units
    // Where the piece (slice, table j, row r, 16-byte piece q) lives:
    //   tables + (slice / spp) * slice_stride + (slice % spp) * SW*16 + j * table_stride + r * row_stride + q*16
    // row-major tables: spp = 1, slice_stride = SW*16, row_stride = d_out*4, table_stride = rows * row_stride;
    // prepared tables (one slice of all tables contiguous, PW bytes per row piece): spp = PW / (SW*16),
    // slice_stride = k * rows * PW, row_stride = PW, table_stride = rows * PW.
    uint32_t row_stride;
    uint32_t spp;
    unsigned long long table_stride;
    unsigned long long slice_stride;
};

constexpr int kPrefetchLds = kLdsThreads * 4;  // where the prefetching copies put their bytes

// Multi-probe form: a lane without a table takes its share from this byte offset of a buffer that ends before it (and so gets
// zero): the (1 + tau) * n_pad shares of a table, and a window of 16 token slots past any of them.
constexpr uint32_t kProbesNoTable = 1u << 31;
constexpr uint32_t kProbesWindow = 16 * 256 * 4;

// bytes of LDS the kernel needs: two buffers and that (sw = lanes per token; alternating rows: and one row piece of zeros)
__host__ __device__ inline size_t gather_lds_bytes(int tau, int sw, bool alternating)
{
    if (alternating) return 2 * (size_t)kLdsBufBytes + 16 * (size_t)sw;
    const size_t tbl = ((size_t)16 * sw) << tau;
    return 2 * (2 * tbl <= (size_t)kLdsBufBytes ? 2 * tbl : tbl) + kPrefetchLds;
}

// balanced split of [0, len) into `parts` pieces: start of piece i (32-bit arithmetic only)
__device__ __forceinline__ uint32_t split_at(uint32_t len, uint32_t parts, uint32_t i)
{
    const uint32_t base = len / parts, rem = len - base * parts;
    return base * i + (i < rem ? i : rem);
}

// a pointer that is the same in every lane, in scalar registers whatever the compiler computed it with
__device__ __forceinline__ const char *scalar_ptr(const char *p)
{
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const char *>((uint64_t)hi << 32 | lo);  // (through uint32_t: the builtin's int would be sign-extended)
}

// One global_load_lds_dwordx4: every active lane copies 16 bytes from gbase + voff to LDS byte
// address lds_base + 16 * lane (lds_base and gbase wave-uniform).  Issued through inline asm so
// that the compiler does not serialise later LDS reads of the *other* buffer behind it; the
// caller waits with s_waitcnt vmcnt(0) before the barrier that publishes the buffer.
// The compiler may form gbase in vector registers and read it into scalar ones right before the statement, and it places no
// waits inside: a memory instruction needs five wait states after that, a scalar one none (and a copy one after the write of
// M0).  So a scalar instruction moves the address first, or, WAIT, the five states are waited: faster where the four copies of a
// 64 KB slice go out together (16384 tokens, tau = 10, k = 128, 1024 wide gather 210.7 / 203.8 us), slower elsewhere (16384, tau
// = 8, k = 96, 768 wide 83.6 / 85.8).
template <bool WAIT>
__device__ __forceinline__ void lds_dma16(const char *gbase, uint32_t voff, uint32_t lds_base)
{
    const uint32_t m = __builtin_amdgcn_readfirstlane(lds_base);
    // M0 is written here, so it is named as clobbered: the compiler then keeps none of its own M0
    // values live across the statement (it warns that M0 is a reserved register; that is the point).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    if constexpr (WAIT) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, %2"
                     :
                     : "s"(m), "v"(voff), "s"(scalar_ptr(gbase))
                     : "memory", "m0");
    } else {
        const char *from;
        asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %2, %0"
                     : "=&s"(from)
                     : "s"(m), "v"(voff), "s"(scalar_ptr(gbase))
                     : "memory", "m0");
    }
#pragma clang diagnostic pop
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Four bytes a lane: brings a cache line per lane into the L2 (the LDS bytes are never read; an LDS copy has no destination
// register that would have to be waited for); its address as in lds_dma16.
__device__ __forceinline__ void lds_dma4(const char *gbase, uint32_t voff, uint32_t lds_base)
{
    const uint32_t m = __builtin_amdgcn_readfirstlane(lds_base);
    const char *from;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dword %2, %0"
                 : "=&s"(from)
                 : "s"(m), "v"(voff), "s"(scalar_ptr(gbase))
                 : "memory", "m0");
#pragma clang diagnostic pop
}

// The same as lds_dma16 for the lanes of `lanes` only (every lane is active outside): a lane's 16 bytes go to lds_base + 16 * lane whichever
// others take part.  The mask is set inside the statement: a branch on the lane would make the compiler treat uniform values
// that change beside it as divergent.  (Three moves and s_nop 1 are the five wait states its address may need.)
__device__ __forceinline__ void lds_dma16_lanes(const char *gbase, uint32_t voff, uint32_t lds_base, uint64_t lanes)
{
    const uint32_t m = __builtin_amdgcn_readfirstlane(lds_base);
    uint64_t all;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, exec\n\ts_mov_b64 exec, %4\n\ts_nop 1\n\tglobal_load_lds_dwordx4 %2, %3\n\t"
                 "s_mov_b64 exec, %0"
                 : "=&s"(all)
                 : "s"(m), "v"(voff), "s"(scalar_ptr(gbase)), "s"(lanes)
                 : "memory", "m0");
#pragma clang diagnostic pop
}

// word 3 of a raw buffer resource: 32-bit data format, offsets checked against the byte count
constexpr int kBufferRsrcFlags = 0x00020000;

// Token group g and 16-byte column piece q of thread `tid` (SW lanes per token).  A ds_read_b128 of a wave is served in
// passes of 16 lanes, and a pass is not 16 consecutive lanes: of the eight quads of 32 lanes it takes 0, 3, 5, 6, then
// 1, 2, 4, 7 (found by timing reads of chosen bank patterns).  With the eight lanes of a token in consecutive lanes a pass holds
// halves of four rows and is conflict-free only if two pairs of rows differ in parity; with a token on the quads
// (0, 3), (5, 6), (1, 2) or (4, 7) a pass holds two whole rows and needs one pair to differ: random 128-byte rows are read at
// 170 instead of 144 bytes per clock and compute unit (conflict-free 240).  A token of four lanes is one quad either way.
template <int SW>
__device__ __forceinline__ void read_role(uint32_t tid, uint32_t &g, uint32_t &q)
{
    if constexpr (SW == 8) {
        const uint32_t b0 = tid >> 2, b1 = tid >> 3, b2 = (tid >> 4) & 1u;  // bits of the quad number (b0, b1: bit 0)
        g = (tid >> 5) * 4u + ((b0 ^ b1 ^ b2) & 1u) * 2u + b2;
        q = (b1 & 1u) * 4u + (tid & 3u);
    } else {
        g = tid / SW;
        q = tid % SW;
    }
}

// value of `v` in lane Q of the caller's quad (DPP quad_perm [Q,Q,Q,Q])
template <int Q>
__device__ __forceinline__ float quad_bcast(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), Q * 0x55, 0xF, 0xF, true));
}
__device__ __forceinline__ float quad_bcast(float v, int q)
{
    return q == 0 ? quad_bcast<0>(v) : q == 1 ? quad_bcast<1>(v) : q == 2 ? quad_bcast<2>(v) : quad_bcast<3>(v);
}
__device__ __forceinline__ uint32_t quad_bcast(uint32_t v, int q)
{
    return __float_as_uint(quad_bcast(__uint_as_float(v), q));
}

// FR = 16 KB copy rounds per table slice (one round = every thread copies 16 bytes = G rows): 1, 2, 4.
// Tables per stage TPS: two (FR <= 2: both halves of a code word are consumed in one stage) or one
// (FR = 4: a 64 KB slice fills a buffer; and the multi-probe form; even stages take the low half of the code word, odd stages
// the high half).  SW = lanes per token: 8 (128-byte column slices; tau = 7, 8, 9 <-> FR = 1, 2, 4)
// or 4 (64-byte slices; tau = 8, 9, 10 <-> FR = 1, 2, 4).  The packed codes must be scaled by the LDS row
// stride (gather_lds_shift).
// MODE: 0 plain sum, 1 weighted, 2 multi-probe (Sec. 3.1, eq. "partial_softmax"): every stage is swept
// 1 + tau times, sweep p reading the rows code ^ flip(p) with the shares of probe p
// (wpk[(j * (1 + tau) + p) * n_pad + t]); the staged slice is copied once per stage.
template <int TOK, int FR, int MODE, int SW = 8>
__global__ __launch_bounds__(kLdsThreads) void gather_lds_kernel(GatherLdsArgs a)
{
    constexpr bool WEIGHTED = MODE != 0, PROBES = MODE == 2;
    static_assert(TOK <= kLdsMaxTok, "packed-code padding covers 16 token slots");
    static_assert(FR == 1 || FR == 2 || FR == 4, "table slices of 16, 32 or 64 KB");
    static_assert(SW == 8 || SW == 4, "128- or 64-byte column slices");
    constexpr int TPS = FR <= 2 && !PROBES ? 2 : 1;
    constexpr int G = kLdsThreads / SW;   // token groups per workgroup = rows per copy round
    constexpr uint32_t PIECE = SW * 16u;  // bytes of a row inside the slice
    static_assert(TPS * FR * 16 * 1024 <= kLdsBufBytes, "a stage fits one buffer");
    // Multi-probe form, tables of up to 32 KB: the rows of two consecutive tables alternate in LDS (four tables in all),
    // and half of the token groups of a read pass lag one table behind the others, so that a pass reads one table in each
    // half of the banks (see read_role).  Every group still takes its tables, and their probes, in the same order.  (Over
    // 64-byte rows a pass holds two tokens of each table, which still meet half of the time: 16384 tokens, k = 96, tau = 9
    // 844 us with the lag, 949 without.)
    constexpr bool LAG = PROBES && FR <= 2;
    constexpr uint32_t kLdsShift = (SW == 8 ? 7 : 6) + (LAG ? 1 : 0);  // log2 of the LDS row stride: the codes' scale
    constexpr uint32_t FILLS = LAG ? 2 * FR : TPS * FR;                // copy rounds of a stage
    extern __shared__ uint4 sbuf[];
    const uint32_t tid = threadIdx.x;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t g, q;  // read role: token group, column piece
    read_role<SW>(tid, g, q);
    constexpr uint32_t rows = (uint32_t)G * FR;      // == 1 << a.tau (checked by the host)
    constexpr uint32_t tbl_bytes = rows * PIECE;     // one table slice in LDS
    constexpr uint32_t buf_bytes = tbl_bytes * TPS;  // one buffer (one stage)
    const uint32_t n = (uint32_t)a.n;                // the host uses this kernel only for n < 2^31
    const uint32_t nstages = (uint32_t)a.k / TPS;
    // LDS byte address of the staging area.  It is 0: the multi-probe form flips bits of its rows' addresses and counts them from
    // there, so no __shared__ variable may be added to this kernel (a test of the built library looks).
    const uint32_t lds0 = (uint32_t)(uintptr_t)sbuf;

    // ---- which (unit, token range) pairs does this workgroup own? ---------------------
    const uint32_t xcd = blockIdx.x % kXcds;
    const uint32_t c = blockIdx.x / kXcds;
    const uint32_t Bx = (uint32_t)a.blocks_per_xcd;
    if ((uint32_t)a.n_units <= xcd) return;
    const uint32_t m = ((uint32_t)a.n_units - xcd + kXcds - 1) / kXcds;  // units dealt to this XCD
    uint32_t u_first, u_step, u_end, part, parts;
    // Where whole chunks divide better than token ranges do (65536 tokens in three slices an XCD: three chunks of 16 slots for every
    // workgroup instead of four of 13: bf16 tables, k = 96, pass 347 -> 328 us) a workgroup takes the chunks i_first ... i_end - 1 of
    // the XCD's, and may change slice between.  Not the multi-probe form: the same code made it 2 % slower at 16384 tokens, where
    // it is not taken (683 -> 698 us; its stage loop has no register to spare).
    const uint32_t unit_chunks = PROBES ? 0u : (uint32_t)a.unit_chunks;
    uint32_t i_first = 0, i_end = 0, per_block = 1;
    if (unit_chunks) {
        i_first = split_at(m * unit_chunks, Bx, c);
        i_end = split_at(m * unit_chunks, Bx, c + 1);
        if (i_end <= i_first) return;
        per_block = (m * unit_chunks + Bx - 1) / Bx;
        u_first = i_first / unit_chunks;
        u_step = 1;
        u_end = (i_end - 1) / unit_chunks + 1;
        part = 0;
        parts = 1;
    } else if (m >= Bx) {  // at least one unit per workgroup: take whole units c, c+Bx, ...
        u_first = c;
        u_step = Bx;
        u_end = m;
        part = 0;
        parts = 1;
    } else {        // several workgroups share a unit: split its token range evenly
        u_first = c * m / Bx;
        u_step = 1;
        u_end = u_first + 1;
        const uint32_t first_blk = (u_first * Bx + m - 1) / m;
        const uint32_t next_blk = ((u_first + 1) * Bx + m - 1) / m;
        part = c - first_blk;
        parts = next_blk - first_blk;
    }

    for (uint32_t ui = u_first; ui < u_end; ui += u_step) {
        const uint32_t unit = ui * kXcds + xcd;
        uint32_t slice = unit % (uint32_t)a.n_slices;
        const uint32_t split = unit / (uint32_t)a.n_slices;
        if constexpr (SW == 4) {
            // A 64-byte slice is half of a 128-byte cache line.  Dealt round-robin, the two halves of
            // every line would go to different XCDs and each L2 would fetch the whole line.  With the
            // slice count a multiple of 16 (then slice % 8 is the XCD) the XCD's units 2i and 2i + 1,
            // which run side by side, take the two halves of the same lines instead.
            if ((uint32_t)a.n_slices % 16u == 0u) {
                const uint32_t i = slice / kXcds;
                slice = ((i >> 1) * kXcds + slice % kXcds) * 2u + (i & 1u);
            }
        }
        const uint32_t s0 = split_at(n, (uint32_t)a.token_splits, split);
        const uint32_t s1 = split_at(n, (uint32_t)a.token_splits, split + 1);
        const uint32_t r0 = s0 + split_at(s1 - s0, parts, part), r1 = s0 + split_at(s1 - s0, parts, part + 1);
        if (r1 <= r0) continue;  // uniform over the workgroup
        uint32_t nchunks = (r1 - r0 + G * TOK - 1) / (G * TOK), ch_first = 0, ch_end = nchunks;
        uint32_t share = part, shares = parts;  // of the prefetch below: this workgroup's, of the unit's
        if (unit_chunks) {
            nchunks = unit_chunks;
            ch_first = ui == u_first ? i_first - ui * unit_chunks : 0u;
            ch_end = i_end - ui * unit_chunks < unit_chunks ? i_end - ui * unit_chunks : unit_chunks;
            share = (ch_first + per_block - 1) / per_block;  // (the unit's workgroups in order, nearly)
            shares = (unit_chunks + 2 * per_block - 2) / per_block;
        }

        // Fill role of this thread: LDS bytes 16 tid .. 16 tid + 15 of every copy round, i.e. column piece fq of row
        // tid / SW (of table (tid / SW) % 2 and row tid / (2 SW) where the rows of two tables alternate).
        // Lanes whose piece lies outside the row (ragged last slice) copy piece 0 instead: they
        // never store a result, and this keeps the copy free of divergent control flow.
        // Offsets inside the tables a round touches fit 32 bits (checked by the host).
        const size_t table_stride = (size_t)a.table_stride;
        const uint32_t fq = tid % SW;
        const bool vec_ok = slice * (uint32_t)SW + fq < (uint32_t)a.nvec;
        const uint32_t foff = (tid / (LAG ? 2u * SW : SW)) * a.row_stride + (vec_ok ? fq : 0u) * 16u;
        const char *slice_base = a.tables + (size_t)(slice / a.spp) * (size_t)a.slice_stride +
                                 (size_t)(slice % a.spp) * PIECE;  // uniform
        // copy round idx of stage s into its buffer (idx = table-in-stage * FR + round); with alternating rows a stage is one
        // table, and the lanes whose 16 bytes belong to the other one take no part
        auto fill_piece = [&](uint32_t s, uint32_t idx) {
            if constexpr (LAG) {
                constexpr uint64_t kEven = SW == 8 ? 0x00FF00FF00FF00FFull : 0x0F0F0F0F0F0F0F0Full;
                lds_dma16_lanes(slice_base + (size_t)s * table_stride + (size_t)(idx * (G / 2)) * a.row_stride, foff,
                                lds0 + ((s >> 1) & 1u) * kLdsBufBytes + (idx * kLdsThreads + wave * 64u) * 16u,
                                s & 1u ? ~kEven : kEven);
            } else {
                lds_dma16<FR == 4 && !PROBES>(slice_base + (size_t)(s * TPS + idx / FR) * table_stride + (size_t)(idx % FR * G) * a.row_stride,
                                              foff, lds0 + (s & 1u) * buf_bytes + (idx * kLdsThreads + wave * 64u) * 16u);
            }
        };

        // L2 prefetch role.  The workgroups of a unit stream the same slice in step, so each copy of a stage used to wait for
        // the memory behind the L2.  They share out the lines of the stage kPrefetch stages ahead: 16384 tokens, k = 96, tau = 8
        // pass 106 -> 100 us, weighted 136 -> 129, k = 256, 512 wide 386 -> 361, tau = 10 264 -> 243.  The fewer share a slice the
        // more of its lines each asks for twice, and the copies are bound by such requests, so it takes four workgroups to a unit,
        // or two where the tables are too large to stay in the memory-side cache (256 MB) from one call to the next.
        // Gather, k = 96, without / with it, tables of 700 MB in turn (three sets of tables in turn, which stay there):
        //   one workgroup (29 slices of 128 bytes): 7946 tokens 118 / 204 us (119 / 205), weighted 131 / 225
        //   two (13): 15892 tokens 89.8 / 81.7 (69.2 / 75.2), weighted 109 / 104 (87 / 97), 29798 tokens 105 / 106 (97.2 / 99.8);
        //   of 1024 rows (13 slices of 64 bytes, 164 MB) 51650 tokens 177 / 162, weighted 212 / 204
        //   four (7): 31784 tokens 87.6 / 75.0 (65.5 / 68.5), 59596 tokens 106 / 104 (98.4 / 99.4)
        //   ten (24): 9932 tokens 88.0 / 76.3 (62.4 / 68.4), weighted 105 / 96 (80.5 / 82.1)
        // Stages of 32 KB (tau = 7) wait less for their copies and more for the requests: with seven slots or fewer it pays (16 slices, k =
        // 128, cold 4966 tokens 80.0 / 73.0, warm 57.1 / 59.3; 10926 tokens 87.9 / 81.3), with more only under the weighted sum's
        // loads (19865 tokens 93.5 / 95.9, weighted 126.8 / 123.9; 15892 tokens, eight slots, 86.3 / 85.9, weighted 109.2 / 108.6).
        constexpr bool kPrefetches = !PROBES && (FR >= 2 || TOK <= 7 || (WEIGHTED && TOK >= 10));
        const bool large = (uint64_t)a.k * rows * (uint32_t)a.nvec * 16u >= 128u << 20;
        const uint32_t sharing = unit_chunks ? shares : Bx / m;  // the fewest workgroups of any unit
        constexpr uint32_t kPrefetch = 3;
        const uint32_t rows_a_line = a.row_stride < 128u ? 128u / a.row_stride : 1u;
        const uint32_t tbl_lines = rows / rows_a_line, stage_lines = (uint32_t)TPS * tbl_lines;
        const bool prefetches = kPrefetches && sharing >= (large ? 2u : 4u) && wave * 64u * shares < stage_lines;  // wave-uniform
        uint32_t line = tid * shares + share;
        if (line >= stage_lines) line = share % stage_lines;
        const uint32_t poff = (line / tbl_lines) * (uint32_t)table_stride + (line % tbl_lines) * rows_a_line * a.row_stride;
        auto prefetch = [&](uint32_t s) {
            if (prefetches && s < nstages)
                lds_dma4(slice_base + (size_t)(s * TPS) * table_stride, poff, lds0 + 2u * buf_bytes + wave * 256u);
        };

        const uint32_t len = r1 - r0;
        for (uint32_t ch = ch_first; ch < ch_end; ++ch) {
            const uint32_t c0 = r0 + split_at(len, nchunks, ch), c1 = r0 + split_at(len, nchunks, ch + 1);
            // Token slots.  The lanes of a token group would all hold the same code word and
            // weights, so these are quad-shared: a lane keeps those of the slots 4m + r, r = its
            // position in its quad, in register m, and a use fetches them with a DPP quad broadcast
            // (a quarter of the registers and load instructions).  Slot i of group g is token
            //   c0 + 4G*(i/4) + 4g + i%4   for the full quads of slots (i < 4*(TOK/4)),
            //   c0 + G*i + g               for the remaining TOK % 4 slots,
            // so that register m of a wave's lanes covers consecutive tokens: one or two cache lines
            // per load instruction.  Slots past the chunk end read the codes of later tokens or of the
            // zero padding (always a valid row), add them, and store nothing.
            constexpr int WQ = (TOK + 3) / 4, FQ = TOK / 4;
            // kRun: slot i of group g is token c0 + WQ*(4g + i%4) + i/4 instead, so that a lane's words of a row are neighbours and
            // come with one load of 16 (12) bytes instead of four (three) of 4.  Only with sixteen slots, or twelve and weights: us a
            // pass without / with it, k = 96, 768 wide: 65536 bf16 rows 328.4 / 320.5, weighted 423 / 413; k = 256, 512 wide 32768
            // tokens 287.9 / 286.1, weighted 360 / 353; tau = 9, 43690 tokens weighted 371 / 365; twelve slots (12288 tokens, 1024 wide)
            // 94.1 / 94.9, weighted 113.8 / 112.1.  Where a stage has fewer slots, or slots that fill no whole quad (a second load), the
            // wider load comes back too late: eight slots (8192 tokens) 80.3 / 83.5, weighted 97.6 / 102.8, multi-probe 444 / 478,
            // thirteen 100.6 / 101.3, weighted 129.2 / 132.7; tables of 32 KB stages (tau = 7) 136.9 / 138.6, of 64 KB (tau = 10) 235 / 241.
            constexpr bool kRun = FR == 2 && !PROBES && (TOK == 16 || (TOK == 12 && WEIGHTED));
            constexpr int WL = kRun ? 1 : WQ;  // loads of a word row
            const uint32_t r4 = q & 3u;
            const uint32_t lq_full = (4u * g + r4) * (kRun ? 4u * WQ : 4u);  // byte offset of the lane's token in a full quad register
            const uint32_t lq_tail = (r4 * G + g) * 4u;   // same for the tail register
            // Register mm's dword of the word row at `row` (uniform: the row's word of token c0), `lane_extra` bytes
            // further: a buffer load, whose per-lane part is one 32-bit offset for every row.  (With plain pointers the
            // compiler kept a 64-bit address per row kind and register, 16 of the 128 registers in the 13-slot weighted
            // form, and spilled in the stage loop, where the reload's wait also waited for the row copies just issued.)
            auto load_reg = [&](const char *row, int mm, uint32_t lane_extra, uint32_t bytes) -> uint32_t {
                const __amdgpu_buffer_rsrc_t rs =
                    __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(row), 0, (int)bytes, kBufferRsrcFlags);
                return __builtin_amdgcn_raw_buffer_load_b32(rs, (mm < FQ ? lq_full : lq_tail) + lane_extra, mm * (16 * G), 0);
            };
            // load u (< WL) of the word row at `row` to `to`
            auto load_words = [&](auto(&to)[WQ], const char *row, int u, uint32_t lane_extra, uint32_t bytes) {
                typedef std::remove_reference_t<decltype(to[0])> word_t;
                if constexpr (kRun) {
                    const __amdgpu_buffer_rsrc_t rs =
                        __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(row), 0, (int)bytes, kBufferRsrcFlags);
                    auto put = [&](auto v) {
#pragma unroll
                        for (int m = 0; m < WQ; ++m) to[m] = __builtin_bit_cast(word_t, (uint32_t)v[m]);
                    };
                    if constexpr (WQ == 3) put(__builtin_amdgcn_raw_buffer_load_b96(rs, lq_full + lane_extra, 0, 0));
                    else put(__builtin_amdgcn_raw_buffer_load_b128(rs, lq_full + lane_extra, 0, 0));
                } else {
                    to[u] = __builtin_bit_cast(word_t, load_reg(row, u, lane_extra, bytes));
                }
            };

            Acc<false> acc[TOK];
#pragma unroll
            for (int i = 0; i < TOK; ++i) acc[i].zero();

            auto lds_row = [&](uint32_t at) {
                return *reinterpret_cast<const __attribute__((address_space(3))) u32x4 *>((uintptr_t)at);
            };
            // all LDS reads of the stage are done; the copies into the other buffer have landed (vmcnt 0)
            auto hand_over = [&]() {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
            };

            // stage 0 into buffer 0
#pragma unroll
            for (uint32_t idx = 0; idx < FILLS; ++idx) fill_piece(0, idx);
            uint32_t cr[WQ];
            // load u of the code words of word row `wrow` (one word = two tables)
            auto load_code = [&](uint32_t wrow, int u) {
                load_words(cr, reinterpret_cast<const char *>(a.packed) + ((size_t)wrow * a.n_pad + c0) * 4u, u, 0u, WQ * 16 * G);
            };
#pragma unroll
            for (int u = 0; u < WL; ++u) load_code(0, u);

            if constexpr (!PROBES) {
                uint32_t half[TPS][WQ];  // LDS row offsets, quad-shared, of the stage's tables
                float w[TPS][WQ];        // their weights
                auto split_codes = [&](uint32_t s) {
#pragma unroll
                    for (int mm = 0; mm < WQ; ++mm) {
                        if constexpr (TPS == 2) {
                            half[0][mm] = cr[mm] & 0xFFFFu;
                            half[1][mm] = cr[mm] >> 16;
                        } else {
                            half[0][mm] = (s & 1u) ? cr[mm] >> 16 : cr[mm] & 0xFFFFu;
                        }
                    }
                };
                float wn[TPS][WQ];
                // load u of the weights of table j, the stage's table tt
                auto load_weight = [&](uint32_t j, int tt, int u) {
                    load_words(wn[tt], reinterpret_cast<const char *>(a.wpk) + ((size_t)j * a.n_pad + c0) * 4u, u, 0u, WQ * 16 * G);
                };
                if constexpr (WEIGHTED) {
#pragma unroll
                    for (int tt = 0; tt < TPS; ++tt)
#pragma unroll
                        for (int u = 0; u < WL; ++u) load_weight(tt, tt, u);
                }
                __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
                split_codes(0);
                for (uint32_t ahead = 1; ahead < kPrefetch; ++ahead) prefetch(ahead);
                hand_over();

                for (uint32_t s = 0; s < nstages; ++s) {
                    const bool more = s + 1 < nstages;
                    const uint32_t b = s & 1u, sn = more ? s + 1 : s;
                    const uint32_t qs = lds0 + b * buf_bytes + q * 16u;  // this lane's piece of row 0
                    if constexpr (WEIGHTED) {
#pragma unroll
                        for (int u = 0; u < TPS; ++u)
#pragma unroll
                            for (int mm = 0; mm < WQ; ++mm) w[u][mm] = wn[u][mm];
                    }
                    // Slot i of the stage: token slot i % TOK of table i / TOK.  Reads run D rows ahead of the sums; a read's
                    // address and a row's weight are formed one slot before they are used, so that the instructions of a slot do
                    // not depend on one another (formed where they are used, every slot waited for them).
                    // (16 slots spill with five rows in flight; four slots of one table are all a stage has)
                    constexpr int NS = TPS * TOK, D = TOK > 13 || NS < 5 ? 4 : 5;
                    static_assert(D <= NS, "the first reads stay inside the stage");
                    u32x4 rd[D];
                    auto slot_at = [&](int i) { return quad_bcast(half[i / TOK][(i % TOK) >> 2], (i % TOK) & 3) + qs; };
                    auto slot_w = [&](int i) { return quad_bcast(w[i / TOK][(i % TOK) >> 2], (i % TOK) & 3); };
#pragma unroll
                    for (int i = 0; i < D; ++i) rd[i] = lds_row(slot_at(i) + (uint32_t)(i / TOK) * tbl_bytes);
                    uint32_t at = slot_at(D < NS ? D : 0);
                    float wb = WEIGHTED ? slot_w(0) : 0.0f;
#pragma unroll
                    for (int i = 0; i < NS; ++i) {
                        // vector-memory work of the next stage: its row copies first (they take longest), then its codes and weights
                        if (i < 2 && more) {
#pragma unroll
                            for (uint32_t idx = 0; idx < TPS * FR; ++idx)
                                if (idx % 2 == (uint32_t)i) fill_piece(s + 1, idx);
                        }
                        if (TPS == 2 || (s & 1u)) {
#pragma unroll
                            for (int u = 0; u < WL; ++u)
                                if (2 + u == i) load_code(sn * TPS / 2, u);
                        }
                        if constexpr (WEIGHTED) {
#pragma unroll
                            for (int x = 0; x < TPS * WL; ++x)
                                if ((2 + WL + x) % NS == i) load_weight(sn * TPS + x / WL, x / WL, x % WL);
                        }
                        const u32x4 v = rd[i % D];
                        const uint4 r = make_uint4(v.x, v.y, v.z, v.w);
                        const uint32_t ac = at;
                        const float wc = wb;
                        if (i + D + 1 < NS) at = slot_at(i + D + 1 < NS ? i + D + 1 : 0);
                        if (WEIGHTED && i + 1 < NS) wb = slot_w(i + 1 < NS ? i + 1 : 0);
                        if constexpr (WEIGHTED) {
                            acc[i % TOK].fma(r, wc);
                            acc[i % TOK].pin();
                        } else {
                            add_in_place(acc[i % TOK].f, r);
                        }
                        if (i + D < NS) rd[i % D] = lds_row(ac + (uint32_t)((i + D) / TOK) * tbl_bytes);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): next stage's rows, codes and weights have landed
                    split_codes(sn);
                    prefetch(s + kPrefetch);
                    hand_over();
                }
            } else {
                // ---- multi-probe form: one table a step, 1 + tau sweeps over it ------------------------------
                const uint32_t tau = (uint32_t)a.tau, k = (uint32_t)a.k, lag = LAG ? (tid >> 4) & 1u : 0u;
                const uint32_t nsteps = k + (LAG ? 1u : 0u);
                const uint32_t crow = (uint32_t)a.n_pad * 4u;  // bytes between word rows (host: kProbesPiece)
                // code words of the lane's table t - lag (any valid row where it has none)
                auto load_codes = [&](uint32_t t) {
                    const uint32_t rb = t ? (t - 1u) >> 1 : 0u, ra = (t < k ? t : k - 1u) >> 1;
                    const char *row = reinterpret_cast<const char *>(a.packed) + ((size_t)(LAG ? rb : ra) * a.n_pad + c0) * 4u;
                    const uint32_t extra = LAG && !lag ? (ra - rb) * crow : 0u;
#pragma unroll
                    for (int u = 0; u < WL; ++u) load_words(cr, row, u, extra, (LAG ? crow : 0u) + WQ * 16 * G);
                };
                // Shares.  Row (j, probe) of wpk is row j * (1 + tau) + probe, so the rows of successive sweeps follow one
                // another; `srow_at` is the row of the next sweep to be loaded for the lagging lanes (table 0 in the first step,
                // where they have none) and the others read `crow * (1 + tau)` bytes further.  A lane without a table reads
                // past the end of the buffer, which gives zeros.
                const uint32_t sstep = (tau + 1u) * crow;
                const char *srow_at = reinterpret_cast<const char *>(a.wpk) + (size_t)c0 * 4u;
                uint32_t lt = 0, lp = 0;  // step and probe of the sweep that is loaded next
                uint32_t sx;              // the lane's offset from that row
                const uint32_t sx_first = LAG && lag ? kProbesNoTable : 0u, sx_mid = LAG && !lag ? sstep : 0u,
                               sx_last = LAG && !lag ? kProbesNoTable : 0u;
                auto share_lane = [&]() {
                    const uint32_t first = lt == 0 ? ~0u : 0u, last = lt < k ? 0u : ~0u;  // (masks: a choice between the three
                    sx = (sx_first & first) | (sx_mid & ~(first | last)) | (sx_last & last);  // ends up in scratch memory)
                };
                share_lane();
                static_assert(WQ * 16 * G <= (int)kProbesWindow, "the host keeps this much below kProbesNoTable");
                auto load_share = [&](float(&to)[WQ], int u) { load_words(to, srow_at, u, sx, (LAG ? sstep : 0u) + WQ * 16 * G); };
                auto next_row = [&]() __attribute__((always_inline)) {
                    if (lp < tau) {
                        ++lp;
                        srow_at += crow;
                    } else if (lt + 1 < nsteps) {  // past the last step: its last row again
                        srow_at += LAG && lt == 0 ? crow - (long long)sstep : (long long)crow;
                        lp = 0;
                        ++lt;
                        share_lane();
                    }
                };
                // Four slots: a step is shorter than the memory's latency, and to wait for a share is to wait for every request before
                // it (they return in order), the next table's rows among them.  So a table's shares are all requested a step ahead,
                // after its rows, and nothing waits before the step's end (4966 tokens, k = 48, tau = 7, 512 wide 155 -> 117 us;
                // 123 when a stage was two tables).
                constexpr bool kShort = TOK == 4;
                constexpr int NP = kShort ? __builtin_ctz(rows) + 1 : 1;  // 1 + tau
                float wn[NP][WQ];
                float wA[WQ], wB[WQ];  // shares of this sweep and of the next, then of the one after
                if constexpr (kShort) {
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
                        load_share(wn[p], 0);
                        next_row();
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < WQ; ++u) load_share(wA, u);
                    next_row();
#pragma unroll
                    for (int u = 0; u < WQ; ++u) load_share(wB, u);
                    next_row();
                }
                if (LAG && tid < PIECE / 16) sbuf[2 * kLdsBufBytes / 16 + tid] = make_uint4(0u, 0u, 0u, 0u);  // the zero row
                __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
                hand_over();
                for (uint32_t t = 0; t < nsteps; ++t) {
                    const uint32_t j = t - lag, tn = t + 1 < nsteps ? t + 1 : t;
                    // a group without a table in this step (the first or the last) reads the zero row, whatever the probe
                    const uint32_t in = !LAG || j < k ? ~0u : 0u;
                    const uint32_t base = LAG ? ((j & 2u) << 15) + (j & 1u) * PIECE : (j & 1u) * buf_bytes;
                    const uint32_t lane_base = q * 16u + ((base & in) | (2u * kLdsBufBytes & ~in));
                    uint32_t off[TOK];
#pragma unroll
                    for (int mm = 0; mm < WQ; ++mm) cr[mm] = (cr[mm] >> ((j & 1u) * 16u)) & 0xFFFFu & in;
#pragma unroll
                    for (int i = 0; i < TOK; ++i) off[i] = quad_bcast(cr[i >> 2], i & 3) + lane_base;
                    // Reads run D rows ahead of the sums, into the next sweep; a read's address and a row's share are formed one
                    // slot before they are used, so that the instructions of a slot do not depend on one another.
                    constexpr int D = TOK % 2 ? 2 : 4;  // (2 * TOK is a multiple of it)
                    u32x4 rd[D];
                    auto flip_of = [&](uint32_t pr) { return (pr ? 1u << (kLdsShift + pr - 1u) : 0u) & in; };
                    uint32_t flip = 0u;
                    // PH: the sweep's slot i is in rd[(i + PH) % D]
                    auto sweep = [&](auto ph_tag, uint32_t pr, float(&w)[WQ]) __attribute__((always_inline)) {
                        constexpr int PH = decltype(ph_tag)::value;
                        const uint32_t flip_next = flip_of(pr + 1u);  // after the last sweep: rows that are not added
                        // address of the row the read of slot i fetches
                        auto next_at = [&](int i) { return i + D < TOK ? off[i + D < TOK ? i + D : 0] ^ flip : off[i + D < TOK ? 0 : i + D - TOK] ^ flip_next; };
                        uint32_t at = next_at(0);
                        float wb = quad_bcast(w[0], 0);
#pragma unroll
                        for (int i = 0; i < TOK; ++i) {
                            const u32x4 v = rd[(i + PH) % D];
                            const float wc = wb;
                            if (i + 1 < TOK) wb = quad_bcast(w[(i + 1) >> 2], (i + 1) & 3);
                            const uint32_t ac = at;
                            if (i + 1 < TOK) at = next_at(i + 1);
                            acc[i].fma(make_uint4(v.x, v.y, v.z, v.w), wc);
                            acc[i].pin();
                            rd[(i + PH) % D] = lds_row(ac);
                            if ((i & 3) == 3 || i == TOK - 1) load_share(w, i >> 2);  // two sweeps ahead
                            if (i == TOK - 1 && pr >= 1 && pr <= FILLS && t + 1 < k) fill_piece(t + 1, pr - 1);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        next_row();
                        flip = flip_next;
                    };
                    using ph0 = std::integral_constant<int, 0>;
                    using ph1 = std::integral_constant<int, TOK % D>;
#pragma unroll
                    for (int i = 0; i < D; ++i) rd[i] = lds_row(off[i]);
                    if constexpr (kShort) {
                        float ws[NP];
#pragma unroll
                        for (int p = 0; p < NP; ++p) ws[p] = wn[p][0];
                        uint32_t at = off[0] ^ flip_of(1u);
                        float wb = quad_bcast(ws[0], 0);
#pragma unroll
                        for (int e = 0; e < NP * TOK; ++e) {  // slot i of sweep p
                            constexpr int kShares = 2;        // of a sweep
                            const int p = e / TOK, i = e % TOK, pn = (e + 1) / TOK, in_ = (e + 1) % TOK;
                            if (i == 0 && p < (int)FILLS && t + 1 < k) fill_piece(t + 1, p);
                            if (i == 1 && p == 1) load_codes(tn);
                            if (i >= TOK - kShares && p * kShares + i - (TOK - kShares) < NP) {
                                load_share(wn[p * kShares + i - (TOK - kShares)], 0);
                                next_row();
                            }
                            const u32x4 v = rd[i];
                            const uint32_t ac = at;
                            const float wc = wb;
                            if (e + 1 < NP * TOK) {
                                wb = quad_bcast(ws[pn < NP ? pn : 0], in_);
                                at = off[in_] ^ flip_of(pn + 1u);
                            }
                            acc[i].fma(make_uint4(v.x, v.y, v.z, v.w), wc);
                            acc[i].pin();
                            if (p + 1 < NP) rd[i] = lds_row(ac);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    } else {
                        uint32_t pr = 0;
                        for (; pr < tau; pr += 2) {
                            sweep(ph0{}, pr, wA);
                            sweep(ph1{}, pr + 1, wB);
                        }
                        if (pr == tau) {  // an odd number of sweeps: the sets change places
                            sweep(ph0{}, pr, wA);
#pragma unroll
                            for (int mm = 0; mm < WQ; ++mm) {
                                const float x = wA[mm];
                                wA[mm] = wB[mm];
                                wB[mm] = x;
                            }
                        }
                        load_codes(tn);
                    }
                    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the next table's rows, codes and first shares have landed
                    hand_over();
                }
            }

            {
                // The output addresses are formed here, from a lane index the compiler cannot see through: left
                // alone it computes all TOK of them before the stage loop and keeps them in registers across it.
                uint32_t lt = tid;
                asm volatile("" : "+v"(lt));
                uint32_t sg, sq;
                read_role<SW>(lt, sg, sq);
                const uint32_t svec = slice * (uint32_t)SW + sq;
#pragma unroll
                for (int i = 0; i < TOK; ++i) {
                    const uint32_t t = kRun ? c0 + WQ * (4u * sg + (uint32_t)(i & 3)) + (uint32_t)(i >> 2)
                                     : i < 4 * FQ ? c0 + (4u * G) * (uint32_t)(i >> 2) + 4u * sg + (uint32_t)(i & 3)
                                                  : c0 + (uint32_t)G * (uint32_t)i + sg;
                    if (t >= c1 || svec >= (uint32_t)a.nvec) continue;
                    store_y4(a.y, (size_t)t * a.d_out + (size_t)svec * 4u, acc[i].f[0], acc[i].f[1], acc[i].f[2],
                             acc[i].f[3], a.y_kind);
                }
            }
        }
    }
}

#if !defined(LFFN_PART) || LFFN_PART == 0  // a plain function: defined by part 0 only of a build in parts
// One-time re-layout of the learned tables T_j (Sec. 3.1, eq. "lookup") for the gather kernels: fp32
// elements (bf16 and IEEE half rows widened exactly), slice-major,
//   dst[ps][j][row][PW bytes],  ps < ceil(d_out*4 / PW),
// so that the column slice of ALL tables a workgroup streams is one contiguous run.  Pieces past the end
// of a row (ragged last slice) are zero.  One 16-byte output piece per thread and step.
//   nvec = d_out / 4 (pieces per fp32 row), ppw = PW / 16, n_out = output pieces in total
__global__ __launch_bounds__(256) void prepare_tables_kernel(const void *src, uint4 *dst, int k, int rows, int nvec,
                                                             int ppw, int kind, long long n_out)
{
    for (long long o = (long long)blockIdx.x * blockDim.x + threadIdx.x; o < n_out;
         o += (long long)gridDim.x * blockDim.x) {
        const int p = (int)(o % ppw);
        long long rest = o / ppw;
        const int row = (int)(rest % rows);
        rest /= rows;
        const int j = (int)(rest % k);
        const long long ps = rest / k;
        const long long vec = ps * ppw + p;
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (vec < nvec) {
            const long long piece = ((long long)j * rows + row) * nvec + vec;
            if (kind) {
                const uint2 w = static_cast<const uint2 *>(src)[piece];
                const float2 lo = widen16x2(w.x, kind), hi = widen16x2(w.y, kind);
                v = make_uint4(__float_as_uint(lo.x), __float_as_uint(lo.y), __float_as_uint(hi.x), __float_as_uint(hi.y));
            } else {
                v = static_cast<const uint4 *>(src)[piece];
            }
        }
        dst[o] = v;
    }
}
#endif

}  // namespace lffn
