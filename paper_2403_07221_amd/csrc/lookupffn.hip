// C ABI of the LookupFFN forward pass (declared in include/lookupffn.h): argument
// validation, launch-shape planning and kernel launches.  All arithmetic of the
// method is in hash_kernel.hpp and gather_kernel.hpp.
#include "lookupffn.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "bh_hash_kernel.hpp"
#include "bh_lane_kernel.hpp"
#include "forward_narrow_kernel.hpp"
#include "forward_small_kernel.hpp"
#include "forward_stack_kernel.hpp"
#include "gather_kernel.hpp"
#include "gather_lds_kernel.hpp"
#include "gather_ring_kernel.hpp"
#include "hash_kernel.hpp"
#include "hash_lane_kernel.hpp"
#include "hash_row_kernel.hpp"

// Build parts.  This file compiles whole (LFFN_PART undefined) or as parts that are linked together, so
// that the kernel families compile side by side: part 0 holds the C ABI, the host logic and the hash and
// re-pack kernels; parts 1 .. 14 hold one family of kernel launchers each (declared just below).  No
// kernel is instantiated in two parts.
#ifdef LFFN_PART
#define LFFN_HAS(p) (LFFN_PART == (p))
#else
#define LFFN_HAS(p) 1
#endif

namespace lffn_host {
using namespace lffn;
int hip_fail(hipError_t e, const char *what);  // part 0
int allow_lds(const void *kern, size_t lds);   // part 0
// While an AttrOnly object lives on this thread, the launchers of kernels that need more than 64 KB of LDS
// only register that need with the runtime and launch nothing (lookupffn_init).
bool attr_only();                              // part 0
struct AttrOnly {
    AttrOnly();
    ~AttrOnly();
};
// part 1: the direct gather kernel
int gather_direct_part(int kind, int lpt, const GatherArgs &a, bool probes, dim3 grid, int threads, hipStream_t s);
int gather_direct_load();  // makes the runtime load part 1's code object now (lookupffn_init)
// parts 2, 3, 11: the LDS-staged gather kernel (plain sum; weighted; multi-probe)
int gather_lds_plain_part(int tok, const GatherLdsArgs &a, int fr, int sw, dim3 grid, size_t lds, hipStream_t s);
int gather_lds_weighted_part(int tok, const GatherLdsArgs &a, int fr, int sw, dim3 grid, size_t lds, hipStream_t s);
int gather_lds_probes_part(int tok, const GatherLdsArgs &a, int fr, int sw, dim3 grid, size_t lds, hipStream_t s);
// part 7: the lagged, bank-interleaved staged gather (prepared tables, tau <= 8)
int gather_ring_part(int threads, int tok, const GatherRingArgs &a, dim3 grid, hipStream_t s);
// part 8: hash and gather in one launch: of a few tokens, one or several chained layers, and of one layer of narrow rows
int forward_stack_part(int n_rounds, int kind, const StackArgs &a, dim3 grid, int tokens, size_t lds, hipStream_t s);
int forward_narrow_part(int n_rounds, int kind, const StackArgs &a, dim3 grid, int threads, size_t lds, hipStream_t s);
int forward_small_part(int L, int kind, const StackArgs &a, dim3 grid, int threads, size_t lds, hipStream_t s);
int forward_stack_load();
// parts 9, 10: the hash with a token per row of lanes, d_pad = 1024 (four tokens per wavefront) and 512 (eight)
int hash_row16_part(int n_rounds, bool shares, const HashArgs &a, dim3 grid, size_t lds, hipStream_t s);
int hash_row8_part(int n_rounds, bool shares, const HashArgs &a, dim3 grid, size_t lds, hipStream_t s);
int hash_row16_load();
int hash_row8_load();
// parts 4 .. 6: the BH hash kernel, d_pad = 64 .. 256, 512 and 1024.  wmode: 0 codes only, 1 weights of tau 4, 8, 16, 2 weights
// of any other tau
int bh_lo_part(int L, int wmode, const BhArgs &a, int block, dim3 grid, hipStream_t s);
int bh_512_part(int wmode, const BhArgs &a, int block, dim3 grid, hipStream_t s);
int bh_1024_part(int wmode, const BhArgs &a, int block, dim3 grid, hipStream_t s);
// part 12: blocks of 64 at d_pad = 1024 for grids of no more workgroups than compute units
int bh_few_part(int wmode, const BhArgs &a, dim3 grid, hipStream_t s);
// part 13: BH of few tokens, a coordinate to a lane, two or four tokens to a workgroup
int bh_lane_part(int L, bool weights, int tokens, const BhArgs &a, int block, dim3 grid, hipStream_t s);
int bh_lane_load();
// part 14: the sign-diagonal hash of few tokens, likewise
int hash_lane_part(int L, int tokens, int wmode, const HashArgs &a, dim3 grid, hipStream_t s);
int hash_lane_load();
}  // namespace lffn_host

namespace {

using namespace lffn;
using lffn_host::allow_lds;
using lffn_host::hip_fail;

#define LFFN_HIP(call)                                       \
    do {                                                     \
        hipError_t e_ = (call);                              \
        if (e_ != hipSuccess) return hip_fail(e_, #call);    \
    } while (0)

#if LFFN_HAS(0)
constexpr int kVersion = 100;  // 0.1.0
constexpr int kMaxLog2N = 12;  // d_pad <= 4096
thread_local std::string g_hip_error;
thread_local const char *t_last_gather = "";  // name of the gather kernel this thread's most recent launch used
thread_local const char *t_last_hash = "";    // the same for the hash kernel
thread_local int t_attr_only = 0;
#endif

enum Mode { kPlain = 0, kWeighted = 1, kProbes = 2 };  // what a gather does with a selected row (the staged kernel's MODE)

// token slots the staged gather is built with (64-byte slices: from 6 on)
constexpr int kLdsSlots[] = {4, 6, 7, 8, 10, 12, 13, 14, 16};

// ---------------------------------------------------------------- kernel launchers (templates: every part may use them)
template <int KIND, int LPT>
void launch_gather_t(const GatherArgs &a, bool probes, dim3 grid, int threads, hipStream_t s)
{
    if (probes) {
        hipLaunchKernelGGL((gather_kernel<KIND, LPT, 2, 0>), grid, dim3(threads), 0, s, a);
        return;
    }
    if constexpr (LPT == 4 || LPT == 8 || LPT == 16) {  // the host asks for the deep form with these only
        if (a.deep) {
            if (a.weights && a.deep == 8) {
                hipLaunchKernelGGL((gather_kernel<KIND, LPT, 1, 8>), grid, dim3(threads), 0, s, a);
                return;
            }
            if (a.weights) {
                hipLaunchKernelGGL((gather_kernel<KIND, LPT, 1, 16>), grid, dim3(threads), 0, s, a);
                return;
            }
            if constexpr (KIND == kElemF32) {  // ... and for a plain sum with fp32 rows only
                hipLaunchKernelGGL((gather_kernel<KIND, LPT, 0, 16>), grid, dim3(threads), 0, s, a);
                return;
            }
        }
    }
    if (a.weights)
        hipLaunchKernelGGL((gather_kernel<KIND, LPT, 1, 0>), grid, dim3(threads), 0, s, a);
    else
        hipLaunchKernelGGL((gather_kernel<KIND, LPT, 0, 0>), grid, dim3(threads), 0, s, a);
}

template <int KIND>
int launch_gather_lpt(int lpt, const GatherArgs &a, bool probes, dim3 grid, int threads, hipStream_t s)
{
    switch (lpt) {
        case 1: launch_gather_t<KIND, 1>(a, probes, grid, threads, s); break;
        case 2: launch_gather_t<KIND, 2>(a, probes, grid, threads, s); break;
        case 4: launch_gather_t<KIND, 4>(a, probes, grid, threads, s); break;
        case 8: launch_gather_t<KIND, 8>(a, probes, grid, threads, s); break;
        case 16: launch_gather_t<KIND, 16>(a, probes, grid, threads, s); break;
        case 32: launch_gather_t<KIND, 32>(a, probes, grid, threads, s); break;
        case 64: launch_gather_t<KIND, 64>(a, probes, grid, threads, s); break;
        default: return LFFN_E_UNSUPPORTED;
    }
    return LFFN_OK;
}

template <int TOK, int FR, int MODE, int SW>
int launch_gather_lds_fr(const GatherLdsArgs &a, dim3 grid, size_t lds, hipStream_t s)
{
    auto kern = gather_lds_kernel<TOK, FR, MODE, SW>;
    int rc = allow_lds(reinterpret_cast<const void *>(kern), lds);
    if (rc != LFFN_OK || lffn_host::attr_only()) return rc;
    hipLaunchKernelGGL(kern, grid, dim3(kLdsThreads), lds, s, a);
    return LFFN_OK;
}

// fr = 16 KB copy rounds per table slice, sw = lanes per token (both fixed by the plan).  The multi-probe form takes 128-byte
// slices for tau 7, 8 and 64-byte slices for tau 9, 10.
template <int TOK, int MODE>
int launch_gather_lds_t(const GatherLdsArgs &a, int fr, int sw, dim3 grid, size_t lds, hipStream_t s)
{
    if (sw == 8) {
        if constexpr (MODE != kProbes) {
            if (fr == 4) return launch_gather_lds_fr<TOK, 4, MODE, 8>(a, grid, lds, s);
        }
        if (fr == 2) return launch_gather_lds_fr<TOK, 2, MODE, 8>(a, grid, lds, s);
        if (fr == 1) return launch_gather_lds_fr<TOK, 1, MODE, 8>(a, grid, lds, s);
    } else if (sw == 4 && TOK >= 6) {
        constexpr int T = TOK >= 6 ? TOK : 6;
        if constexpr (MODE != kProbes) {
            if (fr == 1) return launch_gather_lds_fr<T, 1, MODE, 4>(a, grid, lds, s);
        }
        if (fr == 2) return launch_gather_lds_fr<T, 2, MODE, 4>(a, grid, lds, s);
        if (fr == 4) return launch_gather_lds_fr<T, 4, MODE, 4>(a, grid, lds, s);
    }
    return LFFN_E_UNSUPPORTED;
}

// tok: token slots, one of kLdsSlots
template <int MODE>
int launch_gather_lds_mode(int tok, const GatherLdsArgs &a, int fr, int sw, dim3 grid, size_t lds, hipStream_t s)
{
    switch (tok) {
        case 4: return launch_gather_lds_t<4, MODE>(a, fr, sw, grid, lds, s);
        case 6: return launch_gather_lds_t<6, MODE>(a, fr, sw, grid, lds, s);
        case 7: return launch_gather_lds_t<7, MODE>(a, fr, sw, grid, lds, s);
        case 8: return launch_gather_lds_t<8, MODE>(a, fr, sw, grid, lds, s);
        case 10: return launch_gather_lds_t<10, MODE>(a, fr, sw, grid, lds, s);
        case 12: return launch_gather_lds_t<12, MODE>(a, fr, sw, grid, lds, s);
        case 13: return launch_gather_lds_t<13, MODE>(a, fr, sw, grid, lds, s);
        case 14: return launch_gather_lds_t<14, MODE>(a, fr, sw, grid, lds, s);
        case 16: return launch_gather_lds_t<16, MODE>(a, fr, sw, grid, lds, s);
    }
    return LFFN_E_UNSUPPORTED;
}

template <int L, int TB, int WMODE, bool FEW, bool SPLIT>
int launch_bh_s(const BhArgs &a, dim3 grid, hipStream_t s)
{
    auto kern = bh_hash_kernel<L, TB, WMODE, FEW, SPLIT>;
    const bool query = lffn_host::attr_only();
    const size_t lds = query ? 160 * 1024 : BhLds<L, WMODE == 2>::bytes(a.P);
    int rc = allow_lds(reinterpret_cast<const void *>(kern), lds);
    if (rc != LFFN_OK || query) return rc;
    hipLaunchKernelGGL(kern, grid, dim3(kBhThreads), lds, s, a);
    return LFFN_OK;
}

template <int L, int TB, int WMODE, bool FEW>
int launch_bh_k(const BhArgs &a, dim3 grid, hipStream_t s)
{
    // The form for some of the projections also takes all of them where the compiler made it the faster one: d_pad = 1024, weights
    // in registers, blocks of 16 and 32 (k = 96, tau = 8: 4096 tokens 27.3 -> 26.5 us, 32768 tokens, block 16 103.4 -> 101.1).
    if constexpr (L == 10 && WMODE == 1 && TB <= 2) {
        return launch_bh_s<L, TB, WMODE, FEW, true>(a, grid, s);
    } else {
        if (grid.z > 1 || lffn_host::attr_only()) {
            const int rc = launch_bh_s<L, TB, WMODE, FEW, true>(a, grid, s);
            if (rc != LFFN_OK || grid.z > 1) return rc;
        }
        return launch_bh_s<L, TB, WMODE, FEW, false>(a, grid, s);
    }
}

template <int L, int WMODE>
int launch_bh_b(const BhArgs &a, int block, dim3 grid, hipStream_t s)
{
    switch (block) {
        case 16: return launch_bh_k<L, 1, WMODE, false>(a, grid, s);
        case 32: return launch_bh_k<L, 2, WMODE, false>(a, grid, s);
        case 64: return launch_bh_k<L, 4, WMODE, false>(a, grid, s);
    }
    return LFFN_E_UNSUPPORTED;
}

template <int L>
int launch_bh(int wmode, const BhArgs &a, int block, dim3 grid, hipStream_t s)
{
    switch (wmode) {
        case 0: return launch_bh_b<L, 0>(a, block, grid, s);
        case 1: return launch_bh_b<L, 1>(a, block, grid, s);
        case 2: return launch_bh_b<L, 2>(a, block, grid, s);
    }
    return LFFN_E_UNSUPPORTED;
}

}  // namespace

// ---------------------------------------------------------------- the parts' launch functions
namespace lffn_host {

#if LFFN_HAS(1)
int gather_direct_part(int kind, int lpt, const GatherArgs &a, bool probes, dim3 grid, int threads, hipStream_t s)
{
    switch (kind) {
        case kElemF32: return launch_gather_lpt<kElemF32>(lpt, a, probes, grid, threads, s);
        case kElemBF16: return launch_gather_lpt<kElemBF16>(lpt, a, probes, grid, threads, s);
        case kElemF16: return launch_gather_lpt<kElemF16>(lpt, a, probes, grid, threads, s);
    }
    return LFFN_E_DTYPE;
}

int gather_direct_load()
{
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(gather_kernel<kElemF32, 8, 0, 0>));
    return e == hipSuccess ? LFFN_OK : hip_fail(e, "hipFuncGetAttributes(gather_kernel)");
}
#endif

#if LFFN_HAS(2)
int gather_lds_plain_part(int tok, const GatherLdsArgs &a, int fr, int sw, dim3 grid, size_t lds, hipStream_t s)
{
    return launch_gather_lds_mode<kPlain>(tok, a, fr, sw, grid, lds, s);
}
#endif

#if LFFN_HAS(3)
int gather_lds_weighted_part(int tok, const GatherLdsArgs &a, int fr, int sw, dim3 grid, size_t lds, hipStream_t s)
{
    return launch_gather_lds_mode<kWeighted>(tok, a, fr, sw, grid, lds, s);
}
#endif

#if LFFN_HAS(11)
int gather_lds_probes_part(int tok, const GatherLdsArgs &a, int fr, int sw, dim3 grid, size_t lds, hipStream_t s)
{
    return launch_gather_lds_mode<kProbes>(tok, a, fr, sw, grid, lds, s);
}
#endif

#if LFFN_HAS(7)
template <int THREADS, int TOK>
int launch_gather_ring_t(const GatherRingArgs &a, dim3 grid, hipStream_t s)
{
    auto kern = gather_ring_kernel<THREADS, TOK>;
    int rc = allow_lds(reinterpret_cast<const void *>(kern), kRingLdsBytes);
    if (rc != LFFN_OK || attr_only()) return rc;
    hipLaunchKernelGGL(kern, grid, dim3(THREADS), kRingLdsBytes, s, a);
    return LFFN_OK;
}

int gather_ring_part(int threads, int tok, const GatherRingArgs &a, dim3 grid, hipStream_t s)
{
    if (threads == 1024) {
        switch (tok) {
            case 4: return launch_gather_ring_t<1024, 4>(a, grid, s);
            case 8: return launch_gather_ring_t<1024, 8>(a, grid, s);
            case 12: return launch_gather_ring_t<1024, 12>(a, grid, s);
            case 13: return launch_gather_ring_t<1024, 13>(a, grid, s);
            case 14: return launch_gather_ring_t<1024, 14>(a, grid, s);
        }
    } else if (threads == 512) {
        switch (tok) {
            case 8: return launch_gather_ring_t<512, 8>(a, grid, s);
            case 16: return launch_gather_ring_t<512, 16>(a, grid, s);
            case 20: return launch_gather_ring_t<512, 20>(a, grid, s);
            case 24: return launch_gather_ring_t<512, 24>(a, grid, s);
            case 28: return launch_gather_ring_t<512, 28>(a, grid, s);
            case 32: return launch_gather_ring_t<512, 32>(a, grid, s);
        }
    }
    return LFFN_E_UNSUPPORTED;
}
#endif

#if LFFN_HAS(8)
template <int R, int T>
int launch_forward_stack_r(int kind, const StackArgs &a, dim3 grid, size_t lds, hipStream_t s)
{
    switch (kind) {
        case kElemF32: hipLaunchKernelGGL((forward_stack_kernel<R, kElemF32, T>), grid, dim3(kStackThreads), lds, s, a); break;
        case kElemBF16: hipLaunchKernelGGL((forward_stack_kernel<R, kElemBF16, T>), grid, dim3(kStackThreads), lds, s, a); break;
        case kElemF16: hipLaunchKernelGGL((forward_stack_kernel<R, kElemF16, T>), grid, dim3(kStackThreads), lds, s, a); break;
        default: return LFFN_E_DTYPE;
    }
    return LFFN_OK;
}

template <int T>
int launch_forward_stack_t(int n_rounds, int kind, const StackArgs &a, dim3 grid, size_t lds, hipStream_t s)
{
    switch (n_rounds) {
        case 1: return launch_forward_stack_r<1, T>(kind, a, grid, lds, s);
        case 2: return launch_forward_stack_r<2, T>(kind, a, grid, lds, s);
        case 3: return launch_forward_stack_r<3, T>(kind, a, grid, lds, s);
        case 4: return launch_forward_stack_r<4, T>(kind, a, grid, lds, s);
    }
    return LFFN_E_UNSUPPORTED;
}

int forward_stack_part(int n_rounds, int kind, const StackArgs &a, dim3 grid, int tokens, size_t lds, hipStream_t s)
{
    return tokens == 2 ? launch_forward_stack_t<2>(n_rounds, kind, a, grid, lds, s) : launch_forward_stack_t<1>(n_rounds, kind, a, grid, lds, s);
}

template <int R>
int launch_forward_narrow_r(int kind, const StackArgs &a, dim3 grid, int threads, size_t lds, hipStream_t s)
{
    switch (kind) {
        case kElemF32: hipLaunchKernelGGL((forward_narrow_kernel<R, kElemF32>), grid, dim3(threads), lds, s, a); break;
        case kElemBF16: hipLaunchKernelGGL((forward_narrow_kernel<R, kElemBF16>), grid, dim3(threads), lds, s, a); break;
        case kElemF16: hipLaunchKernelGGL((forward_narrow_kernel<R, kElemF16>), grid, dim3(threads), lds, s, a); break;
        default: return LFFN_E_DTYPE;
    }
    return LFFN_OK;
}

int forward_narrow_part(int n_rounds, int kind, const StackArgs &a, dim3 grid, int threads, size_t lds, hipStream_t s)
{
    if (threads < 64 || threads > kNarrowDwords || threads % 64) return LFFN_E_UNSUPPORTED;
    switch (n_rounds) {
        case 1: return launch_forward_narrow_r<1>(kind, a, grid, threads, lds, s);
        case 2: return launch_forward_narrow_r<2>(kind, a, grid, threads, lds, s);
        case 3: return launch_forward_narrow_r<3>(kind, a, grid, threads, lds, s);
        case 4: return launch_forward_narrow_r<4>(kind, a, grid, threads, lds, s);
    }
    return LFFN_E_UNSUPPORTED;
}

template <int L>
int launch_forward_small_l(int kind, const StackArgs &a, dim3 grid, int threads, size_t lds, hipStream_t s)
{
    switch (kind) {
        case kElemF32: hipLaunchKernelGGL((forward_small_kernel<L, kElemF32>), grid, dim3(threads), lds, s, a); break;
        case kElemBF16: hipLaunchKernelGGL((forward_small_kernel<L, kElemBF16>), grid, dim3(threads), lds, s, a); break;
        case kElemF16: hipLaunchKernelGGL((forward_small_kernel<L, kElemF16>), grid, dim3(threads), lds, s, a); break;
        default: return LFFN_E_DTYPE;
    }
    return LFFN_OK;
}

int forward_small_part(int L, int kind, const StackArgs &a, dim3 grid, int threads, size_t lds, hipStream_t s)
{
    if (threads < 64 || threads > 1024 || threads % 64) return LFFN_E_UNSUPPORTED;
    switch (L) {
        case 6: return launch_forward_small_l<6>(kind, a, grid, threads, lds, s);
        case 7: return launch_forward_small_l<7>(kind, a, grid, threads, lds, s);
        case 8: return launch_forward_small_l<8>(kind, a, grid, threads, lds, s);
        case 9: return launch_forward_small_l<9>(kind, a, grid, threads, lds, s);
    }
    return LFFN_E_UNSUPPORTED;
}

int forward_stack_load()
{
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(forward_stack_kernel<3, kElemF32, 1>));
    return e == hipSuccess ? LFFN_OK : hip_fail(e, "hipFuncGetAttributes(forward_stack_kernel)");
}
#endif

#if LFFN_HAS(9) || LFFN_HAS(10)
// WMODE of the lane-row kernel: 0 codes only, 1 weights reduced in registers (tau divides the lanes of a token),
// 2 weights of any tau through the z window, 3 multi-probe shares
inline int row_wmode(const HashArgs &a, bool shares, int lpt)
{
    return shares ? 3 : !(a.weights || a.wpk) ? 0 : lpt % a.tau == 0 ? 1 : 2;
}

template <int MFULL, int WMODE, int LPT>
int launch_hash_row_r(int n_rounds, const HashArgs &a, dim3 grid, size_t lds, hipStream_t s)
{
    switch (n_rounds) {
        case 1: hipLaunchKernelGGL((hash_row_kernel<1, MFULL, WMODE, LPT>), grid, dim3(kRowThreads), lds, s, a); break;
        case 2: hipLaunchKernelGGL((hash_row_kernel<2, MFULL, WMODE, LPT>), grid, dim3(kRowThreads), lds, s, a); break;
        case 3: hipLaunchKernelGGL((hash_row_kernel<3, MFULL, WMODE, LPT>), grid, dim3(kRowThreads), lds, s, a); break;
        case 4: hipLaunchKernelGGL((hash_row_kernel<4, MFULL, WMODE, LPT>), grid, dim3(kRowThreads), lds, s, a); break;
        default: return LFFN_E_UNSUPPORTED;
    }
    return LFFN_OK;
}

// MFULL: the kernel built for one row length, three rounds; else the form with run-time bounds
template <int MFULL, int LPT>
int launch_hash_row_m(int n_rounds, bool shares, const HashArgs &a, dim3 grid, size_t lds, hipStream_t s)
{
    const int wmode = row_wmode(a, shares, LPT);
    if (MFULL != 0) {
        if (wmode == 0) hipLaunchKernelGGL((hash_row_kernel<3, MFULL, 0, LPT>), grid, dim3(kRowThreads), lds, s, a);
        else if (wmode == 1) hipLaunchKernelGGL((hash_row_kernel<3, MFULL, 1, LPT>), grid, dim3(kRowThreads), lds, s, a);
        else if (wmode == 3) hipLaunchKernelGGL((hash_row_kernel<3, MFULL, 3, LPT>), grid, dim3(kRowThreads), lds, s, a);
        else hipLaunchKernelGGL((hash_row_kernel<3, MFULL, 2, LPT>), grid, dim3(kRowThreads), lds, s, a);
        return LFFN_OK;
    }
    return wmode == 0   ? launch_hash_row_r<0, 0, LPT>(n_rounds, a, grid, lds, s)
           : wmode == 1 ? launch_hash_row_r<0, 1, LPT>(n_rounds, a, grid, lds, s)
           : wmode == 3 ? launch_hash_row_r<0, 3, LPT>(n_rounds, a, grid, lds, s)
                        : launch_hash_row_r<0, 2, LPT>(n_rounds, a, grid, lds, s);
}
#endif

#if LFFN_HAS(9)
int hash_row16_part(int n_rounds, bool shares, const HashArgs &a, dim3 grid, size_t lds, hipStream_t s)
{
    // built for the row lengths of the paper's models (d = 768 and 1024, three rounds); any other multiple of
    // 16 in range takes the form with run-time bounds
    if (n_rounds == 3 && a.d == 768) return launch_hash_row_m<48, 16>(3, shares, a, grid, lds, s);
    if (n_rounds == 3 && a.d == 1024) return launch_hash_row_m<64, 16>(3, shares, a, grid, lds, s);
    return launch_hash_row_m<0, 16>(n_rounds, shares, a, grid, lds, s);
}

int hash_row16_load()
{
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(hash_row_kernel<3, 0, 0, 16>));
    return e == hipSuccess ? LFFN_OK : hip_fail(e, "hipFuncGetAttributes(hash_row_kernel, 16 lanes per token)");
}
#endif

#if LFFN_HAS(10)
int hash_row8_part(int n_rounds, bool shares, const HashArgs &a, dim3 grid, size_t lds, hipStream_t s)
{
    if (n_rounds == 3 && a.d == 512) return launch_hash_row_m<64, 8>(3, shares, a, grid, lds, s);  // the paper's small models
    return launch_hash_row_m<0, 8>(n_rounds, shares, a, grid, lds, s);
}

int hash_row8_load()
{
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(hash_row_kernel<3, 0, 0, 8>));
    return e == hipSuccess ? LFFN_OK : hip_fail(e, "hipFuncGetAttributes(hash_row_kernel, 8 lanes per token)");
}
#endif

#if LFFN_HAS(4)
int bh_lo_part(int L, int wmode, const BhArgs &a, int block, dim3 grid, hipStream_t s)
{
    switch (L) {
        case 6: return launch_bh<6>(wmode, a, block, grid, s);
        case 7: return launch_bh<7>(wmode, a, block, grid, s);
        case 8: return launch_bh<8>(wmode, a, block, grid, s);
    }
    return LFFN_E_UNSUPPORTED;
}
#endif

#if LFFN_HAS(5)
int bh_512_part(int wmode, const BhArgs &a, int block, dim3 grid, hipStream_t s) { return launch_bh<9>(wmode, a, block, grid, s); }
#endif

#if LFFN_HAS(6)
int bh_1024_part(int wmode, const BhArgs &a, int block, dim3 grid, hipStream_t s) { return launch_bh<10>(wmode, a, block, grid, s); }
#endif

#if LFFN_HAS(12)
int bh_few_part(int wmode, const BhArgs &a, dim3 grid, hipStream_t s)
{
    switch (wmode) {
        case 0: return launch_bh_k<10, 4, 0, true>(a, grid, s);
        case 1: return launch_bh_k<10, 4, 1, true>(a, grid, s);
        case 2: return launch_bh_k<10, 4, 2, true>(a, grid, s);
    }
    return LFFN_E_UNSUPPORTED;
}
#endif

#if LFFN_HAS(13)
template <int L, int TB, int T>
int launch_bh_lane_t(bool weights, const BhArgs &a, dim3 grid, hipStream_t s)
{
    constexpr size_t lds = BhLane<L, T>::WORDS * 4;
    static_assert(lds <= 64 * 1024, "no LDS beyond what every kernel may use");
    if (weights) hipLaunchKernelGGL((bh_lane_kernel<L, TB, T, true>), grid, dim3(1 << L), lds, s, a);
    else hipLaunchKernelGGL((bh_lane_kernel<L, TB, T, false>), grid, dim3(1 << L), lds, s, a);
    return LFFN_OK;
}

template <int L, int TB>
int launch_bh_lane(bool weights, int tokens, const BhArgs &a, dim3 grid, hipStream_t s)
{
    return tokens == 2 ? launch_bh_lane_t<L, TB, 2>(weights, a, grid, s) : launch_bh_lane_t<L, TB, 4>(weights, a, grid, s);
}

int bh_lane_part(int L, bool weights, int tokens, const BhArgs &a, int block, dim3 grid, hipStream_t s)
{
    switch (L * 100 + block) {
#define LFFN_CASE(l) \
    case l * 100 + 16: return launch_bh_lane<l, 1>(weights, tokens, a, grid, s); \
    case l * 100 + 32: return launch_bh_lane<l, 2>(weights, tokens, a, grid, s); \
    case l * 100 + 64: return launch_bh_lane<l, 4>(weights, tokens, a, grid, s);
        LFFN_CASE(6) LFFN_CASE(7) LFFN_CASE(8) LFFN_CASE(9) LFFN_CASE(10)
#undef LFFN_CASE
    }
    return LFFN_E_UNSUPPORTED;
}

int bh_lane_load()
{
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(bh_lane_kernel<10, 4, 4, true>));
    return e == hipSuccess ? LFFN_OK : hip_fail(e, "hipFuncGetAttributes(bh_lane_kernel)");
}
#endif

#if LFFN_HAS(14)
template <int L, int T>
int launch_hash_lane_t(int wmode, const HashArgs &a, dim3 grid, hipStream_t s)
{
    constexpr size_t lds = BhLane<L, T>::WORDS * 4;
    static_assert(lds <= 64 * 1024, "no LDS beyond what every kernel may use");
    switch (wmode) {
        case 0:  // (codes alone of narrow rows: four tokens only)
            if constexpr (T == 4 || L >= 8) {
                hipLaunchKernelGGL((hash_lane_kernel<L, T, 0>), grid, dim3(1 << L), lds, s, a);
                break;
            }
            return LFFN_E_UNSUPPORTED;
        case 1: hipLaunchKernelGGL((hash_lane_kernel<L, T, 1>), grid, dim3(1 << L), lds, s, a); break;
        case 2: hipLaunchKernelGGL((hash_lane_kernel<L, T, 2>), grid, dim3(1 << L), lds, s, a); break;
        default: return LFFN_E_UNSUPPORTED;
    }
    return LFFN_OK;
}

int hash_lane_part(int L, int tokens, int wmode, const HashArgs &a, dim3 grid, hipStream_t s)
{
    switch (L) {
#define LFFN_CASE(l) case l: return tokens == 2 ? launch_hash_lane_t<l, 2>(wmode, a, grid, s) : launch_hash_lane_t<l, 4>(wmode, a, grid, s);
        LFFN_CASE(6) LFFN_CASE(7) LFFN_CASE(8) LFFN_CASE(9) LFFN_CASE(10)
#undef LFFN_CASE
    }
    return LFFN_E_UNSUPPORTED;
}

int hash_lane_load()
{
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(hash_lane_kernel<10, 4, 1>));
    return e == hipSuccess ? LFFN_OK : hip_fail(e, "hipFuncGetAttributes(hash_lane_kernel)");
}
#endif

#if LFFN_HAS(0)
int hip_fail(hipError_t e, const char *what)
{
    g_hip_error = std::string(what) + ": " + hipGetErrorString(e);
    return LFFN_E_HIP;
}

bool attr_only() { return t_attr_only > 0; }
AttrOnly::AttrOnly() { ++t_attr_only; }
AttrOnly::~AttrOnly() { --t_attr_only; }

// kernels that use more than 64 KB of dynamic LDS must be told so, once per device and kernel
int allow_lds(const void *kern, size_t lds)
{
    static std::mutex mu;
    static std::map<std::pair<int, const void *>, size_t> configured;  // (device, kernel) -> LDS bytes set up
    int dev = 0;
    LFFN_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(mu);
    size_t &have = configured[std::make_pair(dev, kern)];
    if (have < lds) {
        LFFN_HIP(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        have = lds;
    }
    return LFFN_OK;
}
#endif

}  // namespace lffn_host

#if LFFN_HAS(0)  // ================ everything below: host logic and the C ABI ================
namespace {

int log2_pad(int d)
{
    int l = 0;
    while ((1 << l) < d) ++l;
    return l;
}

bool dtype_ok(int t) { return t == LFFN_F32 || t == LFFN_BF16 || t == LFFN_F16; }
static_assert((int)LFFN_F32 == (int)kElemF32 && (int)LFFN_BF16 == (int)kElemBF16 && (int)LFFN_F16 == (int)kElemF16, "the ABI's dtype codes are the kernels' element kinds");
bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }
int gcd(int a, int b) { return b ? gcd(b, a % b) : a; }
int64_t round256(int64_t b) { return (b + 255) & ~int64_t(255); }

// ---------------------------------------------------------------- options
// Tuning knobs (lookupffn_set_option).  Every entry point takes one snapshot at its start, so a
// concurrent lookupffn_set_option can change which kernel the NEXT call runs, never a call in flight.
struct Options {
    int lanes_per_token = 0;  // 0 = default
    int xcd_order = 0;        // 0 = default, 1 = on, -1 = off
    int gather_path = 0;      // 0 = choose, 1 = direct kernel, 2 = the staged kernel whenever the shape allows,
                              // 4 = the ring kernel whenever the shape allows (else as 2)
    int hash_path = 0;        // 0 = choose, 1 = generic kernel only, 2 = no token-per-lane-row kernel, 3 = that kernel for every batch size
    int hash_blocks = 0;      // 0 = default grid cap of the d_pad = 1024 hash kernel
    int slice_lanes = 0;      // 0 = choose, 4 = 64-byte column slices in the staged gather where possible
    int token_slots = 0;      // 0 = choose, else the most token slots per lane of the staged gather
    int ring_threads = 0;     // 0 = choose, 512 / 1024 = workgroup size of the ring gather
    int small_tokens = 0;     // 0 = default, -1 = never: up to this many tokens lookupffn_forward runs as one
                              // hash-and-gather launch (when the shape is that kernel's)
};
// d_pad = 1024, one launch / two, us: k = 96, 768 wide 200 tokens 13.2 / 14.0, 257 16.0 / 15.0, 512 25.0 / 18.4; k = 32, 256 wide, 512 tokens 7.8 /
// 8.5.  Past a token to a compute unit two launches are ahead where the rows are many bytes; the limit is one of tokens alone.
constexpr int kSmallTokensDefault = 512;
std::mutex g_opt_mu;
Options g_opt;
Options options_snapshot()
{
    std::lock_guard<std::mutex> lk(g_opt_mu);
    return g_opt;
}

// ---------------------------------------------------------------- timing
struct Timing {
    std::mutex mu;
    std::atomic<int> on{0};  // bit 0: time hash launches, bit 1: time gather launches
    std::vector<std::pair<hipEvent_t, hipEvent_t>> ev[2];
    std::vector<std::pair<hipEvent_t, hipEvent_t>> pool;
} g_tm;

struct TimedLaunch {
    int which;
    hipStream_t s;
    hipEvent_t a = nullptr, b = nullptr;
    bool on;
    TimedLaunch(int which_, hipStream_t s_, bool counted = true) : which(which_), s(s_), on(counted && ((g_tm.on.load() >> which_) & 1))
    {
        if (!on) return;
        {
            std::lock_guard<std::mutex> lk(g_tm.mu);
            if (!g_tm.pool.empty()) {
                a = g_tm.pool.back().first;
                b = g_tm.pool.back().second;
                g_tm.pool.pop_back();
            }
        }
        if (!a && (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess)) {
            on = false;
            return;
        }
        on = hipEventRecord(a, s) == hipSuccess;
    }
    void done()
    {
        if (!on || !a || !b) return;
        (void)hipEventRecord(b, s);
        std::lock_guard<std::mutex> lk(g_tm.mu);
        g_tm.ev[which].emplace_back(a, b);
    }
};

// ---------------------------------------------------------------- library-owned workspace (workspace == NULL)
// Grow-only: a larger request allocates a new buffer and keeps the old ones until
// lookupffn_release_workspace(), so work already enqueued (or captured) with an old buffer stays valid and
// nothing synchronises.
struct Workspace {
    void *ptr = nullptr;
    size_t bytes = 0;
    std::vector<void *> retired;
};
std::mutex g_ws_mu;
std::map<int, Workspace> g_ws;

int own_workspace(size_t need, void **out)
{
    int dev = 0;
    LFFN_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_ws_mu);
    Workspace &w = g_ws[dev];
    if (w.bytes < need) {
        const size_t sz = (need + (size_t(1) << 20) - 1) & ~((size_t(1) << 20) - 1);
        void *p = nullptr;
        LFFN_HIP(hipMalloc(&p, sz));
        if (w.ptr) w.retired.push_back(w.ptr);
        w.ptr = p;
        w.bytes = sz;
    }
    *out = w.ptr;
    return LFFN_OK;
}

// A call's scratch memory, handed out front to back in 256-byte aligned pieces.
struct Scratch {
    char *base = nullptr;
    int64_t bytes = 0, used = 0;
    template <class T>
    T *take(int64_t n)
    {
        n = round256(n);
        if (!base || used + n > bytes) return nullptr;
        T *p = reinterpret_cast<T *>(base + used);
        used += n;
        return p;
    }
};

// Resolves the (workspace, workspace_bytes) pair of an entry point: the caller's buffer, or the library's.
int get_scratch(void *workspace, int64_t workspace_bytes, int64_t need, Scratch *sc)
{
    if (workspace) {
        if (workspace_bytes < need) return LFFN_E_WORKSPACE;
        if (!aligned(workspace, 256)) return LFFN_E_ALIGN;
        sc->base = static_cast<char *>(workspace);
        sc->bytes = workspace_bytes;
        return LFFN_OK;
    }
    if (need == 0) return LFFN_OK;
    void *p = nullptr;
    int rc = own_workspace((size_t)need, &p);
    if (rc != LFFN_OK) return rc;
    sc->base = static_cast<char *>(p);
    sc->bytes = need;
    return LFFN_OK;
}

// ---------------------------------------------------------------- static scratch (lookupffn_forward_static)
// Device memory that exists from the moment the code object is loaded: the workspace of the entry point
// for callers that cannot allocate.  Every GPU the library runs on holds its own copy until the process
// ends.  The name is a host-side stand-in, not a device address: host code uses the address
// hipGetSymbolAddress returns for the current device (kept per device below), never the name.
constexpr int64_t kStaticScratchBytes = int64_t(16) << 20;
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[kStaticScratchBytes];

std::mutex g_static_mu;
std::map<int, void *> g_static_ptr;  // device -> address of that device's copy of `scratch`

int static_scratch(void **out)
{
    int dev = 0;
    LFFN_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_static_mu);
    auto it = g_static_ptr.find(dev);
    if (it == g_static_ptr.end()) {
        void *p = nullptr;
        LFFN_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || !aligned(p, 256)) return hip_fail(hipErrorInvalidSymbol, "hipGetSymbolAddress(scratch)");
        it = g_static_ptr.emplace(dev, p).first;
    }
    *out = it->second;
    return LFFN_OK;
}

// ---------------------------------------------------------------- tables: row-major or prepared
// Bytes per row piece of the prepared (slice-major) layout: 128 up to tau = 8 (the staged gather's
// 128-byte column slices; its 64-byte form reads half pieces), 64 from tau = 9 on.
int prepared_piece_bytes(int tau) { return tau <= 8 ? 128 : 64; }

struct TableRef {
    const char *p = nullptr;
    int kind = kElemF32;    // element type of the buffer the kernels read (prepared tables are always fp32)
    bool prepared = false;
    int pw = 0;             // prepared: bytes per row piece
    int y_kind = kElemF32;  // storage type of the output rows (LFFN_Y_BF16 / LFFN_Y_F16 in table_dtype)
};

TableRef table_ref(const void *tables, int table_dtype, int tau)
{
    TableRef t;
    t.p = static_cast<const char *>(tables);
    t.prepared = (table_dtype & LFFN_PREPARED) != 0;
    t.kind = t.prepared ? kElemF32 : (table_dtype & 0xFF);  // LFFN_F32 / BF16 / F16 are the kernels' kinds 0 / 1 / 2
    t.pw = t.prepared ? prepared_piece_bytes(tau) : 0;
    t.y_kind = (table_dtype & LFFN_Y_BF16) ? kElemBF16 : (table_dtype & LFFN_Y_F16) ? kElemF16 : kElemF32;
    return t;
}

int64_t prepared_tables_bytes(int k, int tau, int d_out)
{
    const int64_t pw = prepared_piece_bytes(tau);
    const int64_t n_ps = ((int64_t)d_out * 4 + pw - 1) / pw;
    return round256(n_ps * k * (int64_t(1) << tau) * pw);
}

// ---------------------------------------------------------------- validation
int check_hash(const void *x, const int8_t *signs, const uint16_t *codes, int64_t n, int d, int k,
               int tau, int n_rounds, int x_dtype, bool weighted = false)
{
    if (!x || !signs || !codes) return LFFN_E_NULL;
    if (n < 0 || d < 1 || k < 1 || n_rounds < 1) return LFFN_E_SIZE;
    if (tau < 1 || tau > 16) return LFFN_E_TAU;
    if (!dtype_ok(x_dtype)) return LFFN_E_DTYPE;
    if (k > (1 << 20) || n > (int64_t(1) << 40) || n_rounds > 64) return LFFN_E_SIZE;
    if (log2_pad(d) > kMaxLog2N || d > (1 << kMaxLog2N)) return LFFN_E_UNSUPPORTED;
    const int N = 1 << log2_pad(d);
    const int64_t P = ((int64_t)k * tau + N - 1) / N;
    if (P > 4096) return LFFN_E_SIZE;
    if (hash_lds_bytes((int)P, n_rounds, N, weighted) > 64 * 1024) return LFFN_E_UNSUPPORTED;
    if (!aligned(x, x_dtype == LFFN_F32 ? 4 : 2) || !aligned(codes, 2)) return LFFN_E_ALIGN;
    return LFFN_OK;
}

int check_weights(const float *weights)
{
    if (!weights) return LFFN_E_NULL;
    if (!aligned(weights, 4)) return LFFN_E_ALIGN;
    return LFFN_OK;
}

int check_gather(const uint16_t *codes, const void *tables, const void *y, int64_t n, int k, int tau,
                 int d_out, int table_dtype)
{
    if (!codes || !tables || !y) return LFFN_E_NULL;
    if (n < 0 || k < 1 || d_out < 1) return LFFN_E_SIZE;
    if (tau < 1 || tau > 16) return LFFN_E_TAU;
    if ((table_dtype & ~(0xFF | LFFN_PREPARED | LFFN_Y_BF16 | LFFN_Y_F16)) != 0 || !dtype_ok(table_dtype & 0xFF))
        return LFFN_E_DTYPE;
    if ((table_dtype & LFFN_Y_BF16) && (table_dtype & LFFN_Y_F16)) return LFFN_E_DTYPE;
    if (k > (1 << 20) || n > (int64_t(1) << 40) || d_out > (1 << 24)) return LFFN_E_SIZE;
    const int w = (table_dtype & 0xFF) == LFFN_F32 ? 4 : 8;
    if (d_out % w != 0) return LFFN_E_ALIGN;
    const size_t ta = (table_dtype & LFFN_PREPARED) ? 256 : 16;
    const size_t ya = (table_dtype & (LFFN_Y_BF16 | LFFN_Y_F16)) ? 8 : 16;  // four outputs are stored at a time
    if (!aligned(tables, ta) || !aligned(y, ya) || !aligned(codes, 2)) return LFFN_E_ALIGN;
    // row index (j << tau) + code must fit 32 bits
    if (((int64_t)k << tau) > (int64_t(1) << 31)) return LFFN_E_SIZE;
    return LFFN_OK;
}

// ---------------------------------------------------------------- launches
// grid y > 1: the form whose workgroups take some of the projections each (SPLIT), built for widths from 64 on
template <int L, bool SPLIT>
void launch_hash_s(const HashArgs &a, bool probes, dim3 grid, size_t lds, hipStream_t s)
{
    if (probes)
        hipLaunchKernelGGL((hash_kernel<L, 2, SPLIT>), grid, dim3(kHashThreads), lds, s, a);
    else if (a.weights || a.wpk)
        hipLaunchKernelGGL((hash_kernel<L, 1, SPLIT>), grid, dim3(kHashThreads), lds, s, a);
    else
        hipLaunchKernelGGL((hash_kernel<L, 0, SPLIT>), grid, dim3(kHashThreads), lds, s, a);
}

template <int L>
void launch_hash_t(const HashArgs &a, bool probes, dim3 grid, size_t lds, hipStream_t s)
{
    if constexpr (L >= 6) {
        if (grid.y > 1) {
            launch_hash_s<L, true>(a, probes, grid, lds, s);
            return;
        }
    }
    launch_hash_s<L, false>(a, probes, grid, lds, s);
}

template <int R, bool SPLIT>
void launch_hash1024_s(const HashArgs &a, bool probes, dim3 grid, size_t lds, hipStream_t s)
{
    if (probes)
        hipLaunchKernelGGL((hash1024_kernel<R, 2, SPLIT>), grid, dim3(kHashThreads), lds, s, a);
    else if (a.weights || a.wpk)
        hipLaunchKernelGGL((hash1024_kernel<R, 1, SPLIT>), grid, dim3(kHashThreads), lds, s, a);
    else
        hipLaunchKernelGGL((hash1024_kernel<R, 0, SPLIT>), grid, dim3(kHashThreads), lds, s, a);
}

template <int R>
void launch_hash1024_t(const HashArgs &a, bool probes, dim3 grid, size_t lds, hipStream_t s)
{
    if (grid.y > 1) launch_hash1024_s<R, true>(a, probes, grid, lds, s);
    else launch_hash1024_s<R, false>(a, probes, grid, lds, s);
}

// What a hash launch writes: codes[n][k] (and weights[n][k], or shares[n][k][1+tau] with `probes`), or --
// when `codes` is NULL -- the staged gather's packed codes (and table-major weights wpk[k][n_pad]).
struct HashOut {
    uint16_t *codes = nullptr;
    uint32_t *packed = nullptr;
    float *weights = nullptr;  // beside `codes`: [n][k] or [n][k][1+tau]; beside `packed`: wpk[k][n_pad] or [k][1+tau][n_pad]
    bool probes = false;
    int shift = kPackedShift;  // what the packed codes are scaled by: log2 of the staged gather's row-piece bytes
};

// Host-side extent check of one hash launch: every index the kernels form from (n, k, tau, n_pad)
// stays inside the buffers the caller of launch_hash carved out.  `cap_*` are the byte sizes of the
// regions behind out.codes / out.packed / out.weights (0 = unknown: a caller-owned ABI output).
bool hash_extents_ok(const HashOut &o, int64_t n, int k, int tau, int64_t n_pad, int64_t cap_codes,
                     int64_t cap_packed, int64_t cap_weights)
{
    if (o.codes) {
        if (cap_codes && n * k * 2 > cap_codes) return false;
        const int64_t per = o.probes ? (int64_t)k * (tau + 1) : k;
        if (o.weights && cap_weights && n * per * 4 > cap_weights) return false;
        return true;
    }
    // packed[s * n_pad + t], s < k/2, t < n_pad;  wpk[j * n_pad + t], j < k, t < n
    if (n_pad < n) return false;
    if (cap_packed && (int64_t)(k / 2) * n_pad * 4 > cap_packed) return false;
    const int64_t rows = o.probes ? (int64_t)k * (tau + 1) : k;  // [k][1 + tau][n_pad] shares
    if (o.weights && cap_weights && ((rows - 1) * n_pad + n) * 4 > cap_weights) return false;
    return true;
}

int device_cus(int *cus)
{
    static std::mutex mu;
    static std::map<int, int> cache;
    int dev = 0;
    LFFN_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(mu);
    auto it = cache.find(dev);
    if (it == cache.end()) {
        int n = 0;
        LFFN_HIP(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev));
        it = cache.emplace(dev, n).first;
    }
    *cus = it->second;
    return LFFN_OK;
}

// A launch holds fewer than 2^32 work-items along x and wraps beyond, with no error: rows of up to 2^21 workgroups (of up
// to 1024 work-items), of equal length and a multiple of the XCD count; the kernels pass over the workgroups past `blocks`.
// The most that the entry points take is 2^36 workgroups (2^40 tokens, 16 to each), 2^15 rows.
dim3 grid_of(int64_t blocks)
{
    const int64_t most = int64_t(1) << 21;
    if (blocks <= most) return dim3((unsigned)blocks);
    const int64_t rows = (blocks + most - 1) / most;
    return dim3((unsigned)(((blocks + rows - 1) / rows + kXcds - 1) / kXcds * kXcds), (unsigned)rows);
}

// Projections of few tokens over up to `most` workgroups each: returns the groups and sets the projections of one.  A group
// but the first also hashes the projection before its own where tables cross into it.  (For codes in the ABI layout only: a
// word of the packed layout may hold tables of two projections.  Where that costs a staged batch more than staging gains it
// is not staged: staged_from.)
unsigned split_projections(int P, bool cross, int64_t most, int *p_per)
{
    const int64_t groups = most < P ? most : P;
    const int per = groups < 2 ? P : (int)((P + groups - 1) / groups);
    *p_per = per + cross < P ? per : P;
    return (unsigned)((P + *p_per - 1) / *p_per);
}

// Whether hash_row_kernel takes a hash: d_pad = 1024 or 512, up to four rounds, codes alone or with the gather weights (reduced
// in registers when tau divides the lanes of a token: a table is then a run of lanes of one register; else through a z window in
// LDS), or with the multi-probe shares of tau = 8 in the staged gather's layout: a token per row of 16 (8) lanes, four (eight)
// tokens per wavefront, no LDS transposes.  A lane holds every 16th (8th) coordinate: d a multiple of 16 makes "in range" a
// per-register question.
// It needs a batch that gives most SIMDs two waves of tokens to pull ahead; below that one group's latency
// decides and the one-token kernels are faster.  Measured crossovers: d_pad = 1024 about 2048 tokens (4096
// with weights), d_pad = 512 (twice the tokens per wave) about 6000 (10000 with weights); with shares, which the others leave in
// the ABI layout, 1200 (k = 96, d = 768, staged pass of 1500 tokens 229 / 221 us, 4000 243 / 223; d = 512 233 / 228, 8000 404 / 376).
bool hash_row_ok(const int8_t *signs, bool packed, bool weights, bool probes, int64_t n, int d, int k, int tau, int n_rounds,
                 const Options &opt)
{
    const int L = log2_pad(d);
    if ((L != 10 && L != 9) || d % 16 != 0 || n_rounds < 1 || n_rounds > 4 || !aligned(signs, 16)) return false;
    if (probes && (!packed || tau != 8)) return false;
    const int lpt = L == 10 ? 16 : 8;
    const int64_t row_from = probes ? 1536 : lpt == 16 ? (weights ? 4096 : 2048) : (weights ? 12288 : 6144);
    if (!(opt.hash_path == 3 || (opt.hash_path == 0 && n >= row_from))) return false;
    const int P = (int)(((int64_t)k * tau + (1 << L) - 1) >> L);
    return hrow_lds_bytes(P, n_rounds, lpt, weights && lpt % tau != 0) <= 64 * 1024;
}

// Tokens of a workgroup of hash_lane_kernel where it takes the batch of `parts` transforms on a chip that holds `fill` workgroups
// (cus * 1024 / d_pad), else 0.  wmode: 0 codes alone, 1 weights, 2 shares; cross: tables cross into the next projection, which the
// workgroup they end in then hashes too; slow_rows: the others load the rows element by element (d_pad = 1024) or in 16 bits (below).
// Hash alone, three rounds, us, a token to a wave / two tokens a workgroup / four:
//   d = 700, k = 97, tau = 7, weights: 1 token 6.0 / 4.2 / 4.9, 512 7.9 / 4.9 / 5.4, 1000 8.0 / 6.2 / 5.5, 2000 10.7 / 10.5 / 7.7; codes,
//   k = 96, tau = 8: 512 6.0 / 4.7 / 5.4, 2000 8.3 / 9.9 / 7.7, 4000 9.9 / 17.6 / 12.8; shares 512 9.4 / 6.0 / 6.9, 2000 14.5 / 13.2 / 11.0
//   d = 768, k = 170, tau = 9 (two projections), weights: 512 12.7 / 7.9 / 9.2, 1000 12.8 / 9.8 / 9.4, 2000 17.7 / 17.8 / 13.5
//   d = 512, k = 256, tau = 8 (four), weights: 64 5.7 / 4.2 / 4.7, 512 6.9 / 7.4 / 5.7, 1000 11.7 / 12.9 / 9.1
// so two tokens to the second fill (to the fourth where tables cross at d_pad = 1024: two rounds, codes, 512 tokens of 768, k = 170, tau = 9
// 7.6 / 6.9 / 8.0), four to the eighth.  Where the others are ahead, at `f` fills (hash, or a pass 8 wide, us, a token to a wave / here):
//   weights and shares
//     d = 128, one projection: f = 0.5 4.1 / 4.2, 1.5 4.5 / 4.7; twelve that cross, shares: 0.4 5.1 / 5.4
//     two projections that cross, a chain in either kernel: d = 64 weights up to 1.4 longer here between 0.25 and 2, shares up to 2.1 below
//     2, d = 128 0.6 (weights) and 1.4 (shares) below 5, d = 256 shares 0.4
//     three that cross: d = 256 f = 4.5 8.5 / 8.7, shares 10.1 / 11.1 (four and six: 2 ... 7 shorter), d = 512 shares 6 13.1 / 14.8
//   codes alone, whose narrow transforms cost a wave of its own least (whole passes, x and signs from beyond the L2)
//     d = 64: one projection, 64 tokens 3.0 / 3.2, 8192 4.3 / 4.1; twelve 64 3.3 / 3.5, 512 (1.5) 4.9 / 4.1, 2048 (6) 10.6 / 6.7; two to five
//     that cross 0 ... 2.2 longer, seven and up 0.1 longer below 0.5
//     d = 128: one 0.3 ... 1 longer, two 0.1 ... 0.8 (that cross 2); six f = 0.8 3.7 / 4.0, 3 5.6 / 5.2; that cross, up to eleven 1 longer ... 0.6
//     shorter, twelve 0.8 longer below 0.5, 9 12.8 / 12.2
//     d = 256: one 0.2 ... 0.5 longer; two 0.2 ... 0.7 shorter to 3.5, 4 1 longer, that cross 0.4 ... 1.4 longer; three to five 0.2 ... 1.8 shorter to
//     3.5, then 1.2 longer ... 1.5 shorter (three and four that cross up to 2.5 longer), two fp32 rounds as much longer as shorter; six and up 0.2 ... 6 shorter
//     d = 512: 0 ... 3.9 shorter, but for two that cross, two fp32 rounds 0.5 longer (three from 2 to 5 0.5 longer ... 1.8 shorter)
//     d_pad = 1024 from 4 to 8: one, two rounds 0.96 : 1, three 1.02 : 1; two 0.96 : 1, that cross 0.98 and 1.01 : 1; three that cross 1.0
//     ... 1.5 : 1; rows of no multiple of four 1.0 ... 1.2 : 1 in all of these
int hash_lane_tokens(int N, int P, int n_rounds, int wmode, bool cross, bool slow_rows, int64_t parts, int64_t fill)
{
    bool takes;
    const bool chain = parts > (int64_t)P * fill * N / 256;  // more than four tokens a compute unit: the others take projections in turn
    if (wmode != 0) {
        if (P == 2 && cross && N <= 256 && (N < 256 || wmode == 2))
            takes = N < 256 && (parts >= (N == 64 ? 2 : 5) * fill || (N == 64 && wmode == 1 && 4 * parts <= fill));
        else if (N == 128) takes = parts >= (P == 1 ? 2 : cross ? 1 : 0) * fill;
        else takes = !(P == 3 && cross && (N == 256 || (N == 512 && wmode == 2))) || parts <= 4 * fill;
    } else if (N == 64) takes = (cross ? P >= 7 : (int64_t)P * n_rounds >= 9) && 4 * parts >= 3 * fill;
    else if (N == 128) takes = n_rounds >= 3 && (cross ? P >= 12 && chain : P > 2 && parts > 2 * fill && (P >= 6 || parts <= 5 * fill));
    else if (N == 256 && P <= 2) takes = P == 2 && !cross && 2 * parts <= 7 * fill;
    else if (N == 256)
        takes = (n_rounds + slow_rows >= 3 || (P > 3 && !cross)) && (2 * parts <= 7 * fill || (cross ? P > 4 : P > 3 || parts <= 5 * fill));
    else if (N == 512) takes = !(P == 2 && cross && n_rounds + slow_rows < 3);
    else takes = parts <= 4 * fill || slow_rows || (P == 1 ? n_rounds >= 3 : cross && (n_rounds >= 3 || P > 2));
    if (!takes || parts > 8 * fill) return 0;
    if (wmode == 0 && N <= 128) return 4;
    return parts <= (cross && N == 1024 ? 4 : 2) * fill ? 2 : 4;
}

// few_ok: hash_lane_kernel may take the batch (the forward passes; the stand-alone hash keeps the kernels that give a token to a
// wave, and so the one can be held against the others).
int launch_hash(const void *x, const int8_t *signs, const HashOut &out, int64_t n, int d, int k, int tau,
                int n_rounds, int x_dtype, bool few_ok, hipStream_t s, const Options &opt)
{
    const int L = log2_pad(d);
    const int N = 1 << L;
    HashArgs a{};
    a.x = x;
    a.signs = signs;
    a.codes = out.codes;
    a.packed = out.codes ? nullptr : out.packed;
    a.weights = out.codes ? out.weights : nullptr;
    a.wpk = out.codes ? nullptr : out.weights;
    a.n_pad = packed_n_pad(n);
    a.packed_shift = out.shift;
    a.n = n;
    a.d = d;
    a.k = k;
    a.tau = tau;
    a.n_rounds = n_rounds;
    a.P = (int)(((int64_t)k * tau + N - 1) / N);
    a.x_kind = x_dtype;  // LFFN_F32 / BF16 / F16 are the kernels' kinds 0 / 1 / 2
    a.scale = (float)(1.0 / std::sqrt((double)N));
    a.p_per = a.P;
    a.cross = N % tau != 0;
    if (!a.codes && !a.packed) return LFFN_E_NULL;
    const bool row_ok = hash_row_ok(signs, out.packed != nullptr && !out.codes, out.weights != nullptr, out.probes, n, d, k, tau, n_rounds, opt);
    // shares: in the ABI layout, or in the staged gather's from hash_row_kernel alone
    if (out.probes && (!out.weights || (!a.codes && !row_ok))) return LFFN_E_UNSUPPORTED;
    TimedLaunch tl(0, s);
    const int64_t parts = n * a.P;  // transforms
    if (few_ok && a.codes && opt.hash_path == 0 && L >= 6 && L <= 10) {
        int cus = 0;
        int rc = device_cus(&cus);
        if (rc != LFFN_OK) return rc;
        const int64_t fill = (int64_t)cus * (1024 / N);  // workgroups that the chip holds
        const int wmode = out.probes ? 2 : out.weights ? 1 : 0;
        const int tokens = hash_lane_tokens(N, a.P, n_rounds, wmode, a.P > 1 && a.cross, N == 1024 ? d % 4 != 0 : a.x_kind != 0, parts, fill);
        if (tokens) {
            const int64_t groups = (n + tokens - 1) / tokens;
            const unsigned p_groups = a.P > 1 ? split_projections(a.P, a.cross, std::max<int64_t>(1, fill / groups), &a.p_per) : 1u;
            rc = lffn_host::hash_lane_part(L, tokens, wmode, a, dim3((unsigned)groups, p_groups), s);
            if (rc != LFFN_OK) return rc;
            LFFN_HIP(hipGetLastError());
            tl.done();
            t_last_hash = "hash_lane_kernel";
            return LFFN_OK;
        }
    }
    if (row_ok) {
        const int lpt = L == 10 ? 16 : 8;
        // two workgroups per compute unit fill it (two waves per SIMD); a larger batch is worked through in
        // several groups of tokens per wave, the next group's rows in flight during a transform
        int cus = 0;
        int rc = device_cus(&cus);
        if (rc != LFFN_OK) return rc;
        const int64_t groups = (n + 64 / lpt - 1) / (64 / lpt);
        int64_t blocks = (groups + kRowWaves - 1) / kRowWaves;
        const int64_t cap = opt.hash_blocks ? opt.hash_blocks : 2 * (int64_t)cus;
        if (blocks > cap) blocks = cap;
        const size_t lds = hrow_lds_bytes(a.P, n_rounds, lpt, out.weights && lpt % tau != 0);
        rc = lpt == 16 ? lffn_host::hash_row16_part(n_rounds, out.probes, a, dim3((unsigned)blocks), lds, s)
                       : lffn_host::hash_row8_part(n_rounds, out.probes, a, dim3((unsigned)blocks), lds, s);
        if (rc != LFFN_OK) return rc;
        LFFN_HIP(hipGetLastError());
        tl.done();
        t_last_hash = "hash_row_kernel";
        return LFFN_OK;
    }
    // as many workgroups to the projections as leave a SIMD at most two waves
    unsigned p_groups = 1;
    if (a.codes && N >= 64 && a.P > 1) {
        int cus = 0;
        int rc = device_cus(&cus);
        if (rc != LFFN_OK) return rc;
        p_groups = split_projections(a.P, a.cross, 8 * (int64_t)cus / n, &a.p_per);
    }
    // d_pad = 1024 with up to four rounds: the two-layout kernel (needs 16-byte aligned signs, and
    // rows that start on 16-byte boundaries when it loads them as vectors)
    const size_t xrow = (size_t)d * (a.x_kind ? 2 : 4);
    const bool weighted = out.weights != nullptr;
    if (opt.hash_path != 1 && L == 10 && n_rounds <= 4 && aligned(signs, 16) &&
        h1024_lds_bytes(a.P, weighted) <= 64 * 1024 &&
        (d % 4 != 0 || (aligned(x, 16) && xrow % (a.x_kind ? 8 : 16) == 0))) {
        int64_t blocks = (n + kHashWaves - 1) / kHashWaves;
        const int64_t cap = opt.hash_blocks ? opt.hash_blocks : 4096;
        if (blocks > cap) blocks = cap;
        const dim3 grid((unsigned)blocks, p_groups);
        const size_t lds = h1024_lds_bytes(a.P, weighted);
        switch (n_rounds) {
            case 1: launch_hash1024_t<1>(a, out.probes, grid, lds, s); break;
            case 2: launch_hash1024_t<2>(a, out.probes, grid, lds, s); break;
            case 3: launch_hash1024_t<3>(a, out.probes, grid, lds, s); break;
            default: launch_hash1024_t<4>(a, out.probes, grid, lds, s); break;
        }
        LFFN_HIP(hipGetLastError());
        tl.done();
        t_last_hash = "hash1024_kernel";
        return LFFN_OK;
    }
    const size_t lds = hash_lds_bytes(a.P, n_rounds, N, weighted);
    int64_t blocks = (n + kHashWaves - 1) / kHashWaves;
    if (blocks > 2048) blocks = 2048;
    const dim3 grid((unsigned)blocks, p_groups);
    switch (L) {
#define LFFN_CASE(l) case l: launch_hash_t<l>(a, out.probes, grid, lds, s); break;
        LFFN_CASE(0) LFFN_CASE(1) LFFN_CASE(2) LFFN_CASE(3) LFFN_CASE(4) LFFN_CASE(5) LFFN_CASE(6)
        LFFN_CASE(7) LFFN_CASE(8) LFFN_CASE(9) LFFN_CASE(10) LFFN_CASE(11) LFFN_CASE(12)
#undef LFFN_CASE
        default: return LFFN_E_UNSUPPORTED;
    }
    LFFN_HIP(hipGetLastError());
    tl.done();
    t_last_hash = "hash_kernel";
    return LFFN_OK;
}

constexpr int kLdsMinBytes = 84 * 1024;  // more than half of the 160 KB LDS: one workgroup per CU

// Largest number of tokens a workgroup gets in one piece, mirroring the kernel's split.
int64_t lds_tokens_per_block(int64_t n, int n_units, int token_splits, int Bx)
{
    const int m = (n_units + kXcds - 1) / kXcds;  // units of the fullest XCD
    const int64_t unit_tokens = (n + token_splits - 1) / token_splits;
    if (m >= Bx) return unit_tokens;
    const int blocks = Bx / m;  // the unit with the fewest workgroups
    return (unit_tokens + blocks - 1) / blocks;
}

// Whose codes a gather sums by, and in which layout they are before a staged one: a caller's, or this library's own in a forward
// pass, which the hash leaves in the ABI layout (kTurned: two passes turn them around) or writes packed (kPackedInChain: where
// the hash of a direct gather has its projections spread over workgroups).  A gather of a caller's codes takes scratch memory
// to turn them around, which between the lines it did without: it keeps two tokens a row.
enum class Codes { kCallers, kTurned, kPacked, kPackedInChain };

// Four times the tokens a chunk has to have for staging to pay.  A stage costs its copies and at least its fewest slots' row
// reads however few the tokens; the direct kernel costs by the row.  Lines in token slots (kLdsThreads / sw tokens each), where
// the slowest of the shapes measured (k 64 ... 250, 64 ... 1024 wide, prepared and not) draws level; direct / staged, us:
//   multi-probe, tau 8: 1.75 slots (2240 tokens, k = 96, 768 wide 269 / 240, 64 wide 1.15 : 1; 4096 of the first 471 / 236), tau 9
//   and 10: 2.25 (2880 tokens, k = 96, 768 wide, tau 9 551 / 433, tau 10 770 / 495; 64 wide 1.07 and 1.12 : 1)
//   plain, tau 8: 3.75 (4800 tokens, k = 96, 768 wide 73 / 64; k = 64, 256 wide 58.7 / 57.3); weighted 3.25 (4160 82 / 71; 66 / 65)
//   both, tau 9: 2.5 (3200 tokens, k = 170, 768 wide 175 / 133, 64 wide 1.06 : 1), tau 10: 3.25 (6656, k = 96, 512 wide 138 / 114,
//   weighted 198 / 138; k = 64, 1024 wide 99.9 / 98.9)
// Below 64 tables the fill and the hand-over weigh more, an odd one is a launch of its own with codes and weights to turn around
// (multi-probe 2.5 and 2.75 slots; k = 24, 768 wide, 3200 tokens, tau 8 106 / 91; weighted, k = 97, 4160 tokens of 768 98 / 108), and
// copies of 64 bytes from row-major tables are half a line: two tokens a row there, as for tau 7.
// A few tables' codes and shares that are turned around between the two kernels (all but hash_row_kernel's) cost as much as they
// save.  Multi-probe, below ten tables, tau 8 and 9: two tokens a row (tau 9, 768 wide, k = 4 3830 tokens 31 / 46, k = 7 4617 68 / 83, k = 8 3899
// 54 / 64, tau 8, 512 wide 0.9 : 1; tau 9, k = 10 1 : 1 at the line above); below sixteen, tau 8: 3 slots (k = 12, 768
// wide, 3311 51 / 55, k = 10 0.94 : 1 at 2.6, 1 : 1 at 3); below six, tau 10: 4.5 slots (k = 2 0.83 : 1 at 2.8, 1 : 1 at 4.6); an odd
// number below twelve: 3.5 (tau 10, k = 7 0.87 : 1 at 2.9, 1 : 1 at 3.5, tau 9, k = 11 0.83 : 1 and 1 : 1).  What hash_row_kernel writes: 1.1 ... 2 : 1
// from the line above on for k = 2 ... 10.
// In a chain: the hash of a staged batch (in the packed layout) takes the projections in a chain where that of a direct one spreads them
// over workgroups.  BH, d_pad <= 256, four factors, pass, direct / staged: tau 8, k = 96, 768 wide, d = 256, block 64, 4362 tokens 97 / 133,
// d = 64, block 32, 4865 79 / 97, k = 250, d = 128, block 64, 4309 282 / 330: two tokens a row; tau 9, d = 64, block 32, 3586 108 / 128,
// 4210 120 / 115, block 64 4411 135 / 142: 3.5 slots; tau 10, d = 64, block 64, k = 96 4307 219 / 273, k = 170 5304 426 / 429, 512 wide, d = 128
// 6731 116 / 128, k = 80 5215 151 / 168: 4.5 slots, but for blocks of 16 and 32
// of rows of 256 (block 16, two factors, k = 96 5125 203 / 162).  d_pad = 512 spreads them up to 4096 tokens: tau 8, block 32, 536 wide 3575
// 86 / 113, 984 wide 4000 133 / 156, but tau 9 1.1 ... 2 : 1.
// Where an XCD's workgroups have a slice each (an odd number of slices, so that every XCD has all of them) none of them finds its copies
// in the L2, and those past whole turns idle, more than three in eight of them at some widths; the direct kernel is slower where the
// tables go beyond the L2s and half the memory-side cache.  Passes, direct / staged:
//   tau 8, plain: two tokens a row (k = 64, 544 wide 3976 48 / 56, 912 wide 4020 72 / 83); weighted, below 80 MB likewise (k = 64, 712 wide 3489
//   67 / 75, 976 wide 3905 84 / 94), below 140 MB 3.5 slots (0.93 : 1 at 3.3, 1.06 and more from 3.6 on); multi-probe, idle 2.25 (584 wide
//   2004 185 / 208; k = 96, 920 wide, no more than one in ten idle, 2233 361 / 233)
//   tau 9, below 140 MB, idle past a turn: plain and weighted two tokens a row (560 wide 5135 116 / 141, 528 wide 6651 137 / 154; above it 1.1 ... 1.6 : 1:
//   k = 146, 592 wide 7634 457 / 308; idle in the only turn 1 : 1 from the line on, k = 170, 296 wide 7735 293 / 199); multi-probe, idle
//   3.25 (544 wide 2762 269 / 313)
//   tau 10: plain, below 400 MB, 4 slots (720 wide 7636 227 / 234), idle 4.75 (528 wide 7545 266 / 330; above it k = 128, 880 wide 7092 629 / 550);
//   weighted, idle 4.25 (552 wide 8620 224 / 252)
// units: slices of the fullest XCD, for its `per_xcd` workgroups; bytes: of the tables.
int64_t staged_from(Mode mode, int k, int tau, int sw, int rows, bool prepared, Codes codes, int units, int per_xcd, int64_t bytes)
{
    const int64_t two_a_row = 8 * (int64_t)rows, slot = kLdsThreads / sw;
    if (tau == 7 || (sw == 4 && !prepared)) return two_a_row;
    if (codes == Codes::kPackedInChain && sw == 8) return two_a_row;
    if (codes == Codes::kTurned && tau <= 9 && k < 10) return two_a_row;
    int64_t line = two_a_row / slot;  // in quarters of a slot
    const bool small = k < 64 || k % 2;
    const bool chain = codes == Codes::kPackedInChain, turned = codes == Codes::kTurned;
    if (mode == kProbes && turned && k < 12 && (k < 6 || k % 2)) line = k < 6 ? 18 : 14;
    else if (mode == kProbes) line = sw == 8 ? (turned && k < 16 ? 12 : small ? 10 : 7) : (small ? 11 : 9);
    else if (!small) line = sw == 8 ? (mode == kWeighted ? 13 : 15) : tau <= 9 ? (chain ? 14 : 10) : (chain ? 18 : 13);
    const bool alone = 2 * units > per_xcd, idle = alone && 8 * units < 5 * per_xcd * ((units + per_xcd - 1) / per_xcd);
    const bool probes = mode == kProbes, weighted = mode == kWeighted;
    const int mb = (int)(bytes / 1000000);
    int64_t least = 0;
    if (sw == 8) least = probes ? (idle ? 9 : 0) : !alone ? 0 : !weighted || mb < 80 ? 16 : mb < 140 ? 14 : 0;
    else if (tau <= 9) least = !idle || mb >= 140 ? 0 : probes ? 13 : units > per_xcd ? 16 : 0;
    else if (alone && !probes) least = weighted ? (idle ? 17 : 0) : mb >= 400 ? 0 : idle ? 19 : 16;
    return std::min(std::max(line, least) * slot, two_a_row);
}

// Launch shape of the LDS-staged gather for one problem size (no pointers involved).
struct LdsPlan {
    bool use = false;
    GatherLdsArgs a{};
    int tok = 0;
    int sw = 8;     // lanes per token: 8 = 128-byte column slices, 4 = 64-byte ones
    int fr = 1;     // 16 KB copy rounds per table slice
    int shift = 7;  // log2 of the row-piece bytes: what the packed codes are scaled by (the hash kernels and the
                    // re-pack kernel scale by whatever the plan says)
    unsigned grid = 0;
    size_t lds = 0;
    int tail = 0;   // tables left to the direct kernel, which adds them onto the staged kernel's y: 1 when
                    // k is odd (the staged kernel takes its tables in pairs), else 0
};

int plan_gather_lds(int64_t n, int k, int tau, int d_out, const TableRef &T, Mode mode, Codes codes, const Options &opt,
                    LdsPlan *p)
{
    p->use = false;
    if (opt.gather_path == 1) return LFFN_OK;
    if (T.kind) return LFFN_OK;  // the staged kernel reads fp32 rows: 16-bit tables take it once prepared
    const int rows = 1 << tau;
    if (tau < 7 || tau > 10) return LFFN_OK;
    // an odd k: the first k - 1 tables staged, the last one added by the direct kernel, which re-reads the
    // fp32 sums (so not with 16-bit outputs, which are rounded once from the complete sum)
    const int tail = k & 1;
    if (tail && (k < 3 || T.y_kind != 0)) return LFFN_OK;
    // column slices: 128 bytes (8 lanes per token) up to tau = 8; 64 bytes from tau = 9 on (two 512-row
    // tables per stage and half the copy volume per token measured faster than one per stage; tau = 10
    // fits a 64 KB buffer only this way).  The 64-byte form exists for tau >= 8.
    int sw = tau <= 8 ? 8 : 4;
    if (opt.slice_lanes == 4 && tau >= 8) sw = 4;
    if (opt.slice_lanes == 8 && tau <= 9) sw = 8;
    if (mode == kProbes) sw = tau <= 8 ? 8 : 4;  // the multi-probe form is built for these pairings only
    if (T.prepared && sw * 16 > T.pw) sw = T.pw / 16;  // a token's row piece must lie inside one prepared piece
    if (sw == 4 && tau < 8) return LFFN_OK;
    const int groups = kLdsThreads / sw;
    // the kernel indexes tokens and bytes inside one table with 32 bits (the multi-probe form also the bytes between two tables of a
    // batch's shares: kProbesPiece)
    if (n >= (int64_t(1) << 31) - 4096 || (int64_t)rows * d_out * 4 >= (int64_t(1) << 32)) return LFFN_OK;
    int cus = 0;
    int rc = device_cus(&cus);
    if (rc != LFFN_OK) return rc;
    if (cus < kXcds || cus % kXcds != 0) return LFFN_OK;
    GatherLdsArgs &a = p->a;
    a = GatherLdsArgs{};
    a.n = n;
    a.n_pad = packed_n_pad(n);
    a.k = k - tail;
    a.tau = tau;
    a.d_out = d_out;
    const uint32_t row_bytes = (uint32_t)d_out * 4;  // of the fp32 rows the kernel reads
    a.nvec = (int)(row_bytes / 16);
    a.n_slices = (a.nvec + sw - 1) / sw;
    a.token_splits = kXcds / gcd(a.n_slices, kXcds);
    a.n_units = a.n_slices * a.token_splits;
    a.blocks_per_xcd = cus / kXcds;
    if (T.prepared) {
        a.spp = (uint32_t)(T.pw / (sw * 16));
        a.row_stride = (uint32_t)T.pw;
        a.table_stride = (unsigned long long)rows * T.pw;
        a.slice_stride = (unsigned long long)k * rows * T.pw;
    } else {
        a.spp = 1;
        a.row_stride = row_bytes;
        a.table_stride = (unsigned long long)rows * row_bytes;
        a.slice_stride = (unsigned long long)sw * 16;
    }
    const int m = (a.n_units + kXcds - 1) / kXcds, Bx = a.blocks_per_xcd;
    const int64_t tpb = lds_tokens_per_block(n, a.n_units, a.token_splits, Bx);
    int tok_max = 16;
    if (opt.token_slots && opt.token_slots < tok_max) tok_max = opt.token_slots;
    const int64_t nchunks = (tpb + (int64_t)groups * tok_max - 1) / ((int64_t)groups * tok_max);
    const int64_t chunk = (tpb + nchunks - 1) / nchunks;
    if (opt.gather_path < 2 && chunk * 4 < (codes == Codes::kCallers ? 8 * (int64_t)rows : staged_from(mode, k, tau, sw, rows, T.prepared, codes, m, Bx, (int64_t)k * rows * d_out * 4))) return LFFN_OK;
    // the fewest slots built that hold a chunk: a slot without a token costs what any other does
    auto slots_of = [&](int64_t tokens) {
        const int tok = (int)((tokens + groups - 1) / groups);
        for (int built : kLdsSlots)
            if (built >= tok && (sw == 8 || built >= 6)) return built;
        return tok;
    };
    p->tok = slots_of(chunk);
    // Every chunk streams all tables.  Where the workgroups of an XCD take fewer turns when they divide whole chunks instead of token
    // ranges (whose shortest division decides: 32 workgroups over three slices give one of them 10), they do that, unless its
    // slots cost more (a turn's fill and hand-over count as one slot).  65536 bf16 tokens, k = 96, 768 wide, pass 347 -> 328 us.
    const int64_t unit_tokens = (n + a.token_splits - 1) / a.token_splits;
    const int64_t turns = nchunks * (m > Bx ? (m + Bx - 1) / Bx : 1);
    int64_t cost = turns * (p->tok + 1);
    for (int built : kLdsSlots) {
        if (mode == kProbes || built > tok_max || (sw == 4 && built < 6)) continue;
        const int64_t unit_chunks = (unit_tokens + (int64_t)groups * built - 1) / ((int64_t)groups * built);
        if (unit_chunks * m >= (int64_t)1 << 30) continue;
        const int64_t t = (unit_chunks * m + Bx - 1) / Bx;
        const int tok = slots_of((unit_tokens + unit_chunks - 1) / unit_chunks);
        if (t < turns && tok <= tok_max && t * (tok + 1) < cost) {
            cost = t * (tok + 1);
            a.unit_chunks = (int)unit_chunks;
            p->tok = tok;
        }
    }
    p->sw = sw;
    p->fr = rows / groups;
    // log2 of the LDS row stride: the multi-probe form alternates the rows of a stage's two tables
    const bool alternating = mode == kProbes && p->fr <= 2;
    p->shift = (sw == 8 ? 7 : 6) + (alternating ? 1 : 0);
    p->lds = gather_lds_bytes(tau, sw, alternating);
    if (p->lds < (size_t)kLdsMinBytes) p->lds = kLdsMinBytes;
    p->grid = (unsigned)cus;
    p->tail = tail;
    p->use = true;
    return LFFN_OK;
}

// Byte counts of the scratch regions.  The arguments may be anything a caller passes to a size query, so
// the products are formed in 128 bits and a count that no buffer can have saturates at kBytesMax (every
// workspace is then too small, and nothing overflows).
constexpr int64_t kBytesMax = INT64_MAX & ~int64_t(255);
typedef unsigned __int128 u128;
int64_t sat_bytes(u128 b)
{
    b = (b + 255) & ~u128(255);
    return b > (u128)kBytesMax ? kBytesMax : (int64_t)b;
}
int64_t sat_add(int64_t a, int64_t b) { return a > kBytesMax - b ? kBytesMax : a + b; }
u128 n_pad_of(int64_t n) { return n > (int64_t(1) << 60) ? (u128)1 << 61 : (u128)packed_n_pad(n); }
// packed codes of either staged kernel: [k/2][n_pad] words, or the ring kernel's lagged [k/2 + 3][n_pad]
int64_t packed_bytes(int64_t n, int k) { return sat_bytes((u128)ring_code_words(k) * n_pad_of(n) * 4); }
int64_t wpk_bytes(int64_t n, int k) { return sat_bytes((u128)k * n_pad_of(n) * 4); }
int64_t spk_bytes(int64_t n, int k, int tau) { return sat_bytes((u128)k * (u128)(tau + 1) * n_pad_of(n) * 4); }
int64_t abi_codes_bytes(int64_t n, int k) { return sat_bytes((u128)n * (u128)k * 2); }
int64_t abi_weights_bytes(int64_t n, int k, int tau, Mode m)
{
    return m == kPlain ? 0 : sat_bytes((u128)n * (u128)k * (u128)(m == kProbes ? tau + 1 : 1) * 4);
}
// scratch of a stand-alone gather: the staged kernel's packed codes and table-major weights / shares
int64_t gather_ws_bytes(int64_t n, int k, int tau, Mode m)
{
    if (n <= 0 || k < 1) return 0;
    return sat_add(packed_bytes(n, k), m == kWeighted ? wpk_bytes(n, k) : m == kProbes ? spk_bytes(n, k, tau) : 0);
}
// scratch of a forward pass: the hash's ABI-layout outputs and the gather's scratch
int64_t forward_ws_bytes(int64_t n, int k, int tau, Mode m)
{
    if (n <= 0 || k < 1) return 0;
    return sat_add(sat_add(abi_codes_bytes(n, k), abi_weights_bytes(n, k, tau, m)), gather_ws_bytes(n, k, tau, m));
}

int launch_gather_lds(const LdsPlan &p, const uint32_t *packed, const float *wpk, const TableRef &T, void *y,
                      Mode mode, hipStream_t s)
{
    GatherLdsArgs a = p.a;
    a.packed = packed;
    a.wpk = wpk;
    a.tables = T.p;
    a.y = y;
    a.y_kind = T.y_kind;
    // extents the kernel assumes: rows * copy rounds cover a table exactly, the stage fits its buffer,
    // token windows of 16 x 256 tokens past any token stay inside the padded code arrays
    if ((kLdsThreads / p.sw) * p.fr != (1 << a.tau) || a.n_pad < a.n + 16 * 256 || (a.k & 1) || T.kind ||
        (mode != kPlain) != (wpk != nullptr) || !packed)
        return LFFN_E_UNSUPPORTED;
    if (mode == kProbes && (a.tau + 1) * a.n_pad * 4 + kProbesWindow > (long long)kProbesNoTable) return LFFN_E_UNSUPPORTED;
    const dim3 grid(p.grid);
    int rc = LFFN_E_UNSUPPORTED;
    TimedLaunch tl(1, s);
    if (mode == kProbes)
        rc = lffn_host::gather_lds_probes_part(p.tok, a, p.fr, p.sw, grid, p.lds, s);
    else if (mode == kWeighted)
        rc = lffn_host::gather_lds_weighted_part(p.tok, a, p.fr, p.sw, grid, p.lds, s);
    else
        rc = lffn_host::gather_lds_plain_part(p.tok, a, p.fr, p.sw, grid, p.lds, s);
    if (rc != LFFN_OK) return rc;
    LFFN_HIP(hipGetLastError());
    tl.done();
    t_last_gather = "gather_lds_kernel";
    return LFFN_OK;
}

// j_first > 0: only the tables [j_first, k) are summed, onto what y already holds (fp32 y and fp32 rows).
int launch_gather_direct(const uint16_t *codes, const float *weights, const TableRef &T, void *y, int64_t n,
                         int k, int tau, int d_out, Mode mode, hipStream_t s, const Options &opt, int j_first = 0)
{
    const int esz = T.kind ? 2 : 4;
    if (j_first < 0 || j_first >= k || (j_first && (T.kind || T.y_kind))) return LFFN_E_UNSUPPORTED;
    if ((mode != kPlain) != (weights != nullptr)) return LFFN_E_NULL;
    GatherArgs a{};
    a.codes = codes + j_first;
    a.weights = weights ? weights + (size_t)j_first * (mode == kProbes ? tau + 1 : 1) : nullptr;
    a.y = y;
    a.y_kind = T.y_kind;
    a.n = n;
    a.k = k - j_first;
    a.code_stride = k;
    a.accumulate = j_first > 0;
    a.tau = tau;
    a.d_out = d_out;
    const uint32_t row_bytes = (uint32_t)d_out * esz;
    a.nvec = (int)(row_bytes / 16);

    int lpt = opt.lanes_per_token;
    if (lpt == 0) {
        lpt = 8;  // 128-byte slices: one L2 line per (token, table)
        // rows that are no whole number of lines: every piece crosses into a second line, so twice the width halves
        // those, while the slice of all tables still fits an XCD's L2 (1001 tokens, 97 half tables of 128 rows of
        // 1296 bytes: pass 29.7 -> 26.0 us; where the slice does not fit, 96 x 256 rows of 1536 bytes, 139 -> 164 us)
        if (!T.prepared && row_bytes % 128 != 0 && ((int64_t)k << tau) * 256 <= (int64_t)4 << 20) lpt = 16;
        while (lpt > 1 && lpt / 2 >= a.nvec) lpt /= 2;
    }
    if (T.prepared && lpt * 16 > T.pw) lpt = T.pw / 16;  // a token's piece lies inside one prepared piece
    const int tpw = 64 / lpt;
    a.n_slices = (a.nvec + lpt - 1) / lpt;
    if (T.prepared) {
        a.spp = (uint32_t)(T.pw / (lpt * 16));
        a.row_stride = (uint32_t)T.pw;
        a.slice_stride = ((unsigned long long)k << tau) * T.pw;
    } else {
        a.spp = 1;
        a.row_stride = row_bytes;
        a.slice_stride = (unsigned long long)lpt * 16;
    }
    a.tables = T.p + ((size_t)j_first << tau) * a.row_stride;  // row (j << tau) + code of either layout
    int cus = 0;
    int rc = device_cus(&cus);
    if (rc != LFFN_OK) return rc;
    // too few full workgroups to give every compute unit two: one wave a workgroup spreads the same waves wider
    const int64_t full = (n + (int64_t)kGatherWaves * tpw - 1) / ((int64_t)kGatherWaves * tpw);
    const int waves = full * a.n_slices < 2 * (int64_t)cus ? 1 : kGatherWaves;
    const int64_t ntb = (n + (int64_t)waves * tpw - 1) / ((int64_t)waves * tpw);
    if (ntb > (int64_t(1) << 30)) return LFFN_E_SIZE;
    a.ntb = (int)ntb;

    const double table_bytes = (double)k * (double)(1u << tau) * row_bytes;
    // below about 1000 tokens the order makes no difference; 2000 tokens, weighted pass of 96 tables 48 -> 44 us, tau = 11
    // 153 -> 121 us.  Tokens decide, not workgroups: with the 64-byte pieces of prepared tables from tau = 9 on a workgroup has
    // 64 (1664 tokens, k = 170, 512 wide: tau = 10 pass 137 -> 118 us, tau = 9 105 -> 93, weighted 120 -> 109)
    bool xcd = table_bytes > 4.0 * 1024 * 1024 && (full >= 32 || n >= 1000);
    // Rows of a token in flight in the plain sum, sixteen or four.  Sixteen hide the waits of few wavefronts; with many, and a
    // slice of all tables beyond an XCD's L2, four keep the wavefronts closer together in the tables, so more rows are still in
    // the L2.  That pays for rows of 16-bit elements from about nine wavefronts a compute unit on, and for ragged fp32 rows
    // while there are fewer than thirty; whole fp32 lines and prepared tables gain nothing.  Gather, 16 / 4 rows, us:
    //   bf16, k = 170, tau = 9: 504 wide 1500 tokens 28 / 39, 3932 96 / 60, 16384 422 / 394, 40000 1088 / 1220; 512 wide 2000
    //   27 / 36, 8000 118 / 93; k = 128, tau = 10, 1024 wide: 1000 30 / 31, 4000 117 / 87; 97 tables of tau = 8 (3 MiB a
    //   slice), 768 wide 4000 36 / 48
    //   fp32, k = 170, tau = 9: 504 wide 1500 70 / 49, 3000 129 / 111, 8000 356 / 419; 512 wide 4000 112 / 102, 16384 456 /
    //   473; prepared, 768 wide 2500 120 / 141
    const bool beyond_l2 = ((int64_t)k << tau) * lpt * 16 > (int64_t)4 << 20, ragged = row_bytes % 128 != 0;
    const int64_t cu_waves = (n + tpw - 1) / tpw * a.n_slices / cus;
    a.four_rows = mode == kPlain && beyond_l2 && !T.prepared && cu_waves >= 9 &&
                  (T.kind ? !ragged || cu_waves <= 128 : ragged && cu_waves <= 30);
    // The form with thirty-two rows in flight: up to five wavefronts a compute unit (more lose what their registers cost), where
    // the walk through the tables is long enough to show.  Us without / with it:
    //   passes on new tokens, weighted, 768 wide: fp32 k = 48 1 token 9.8 / 9.4, 16 13.0 / 11.9, k = 96 1 token 13.7 / 12.6, 16
    //   18.4 / 15.7, k = 170, tau = 9 1 token 23.3 / 20.8; fp16 k = 48 1 token 9.5 / 9.2, 16 11.6 / 10.8; 256 wide k = 64 1 token
    //   8.4 / 8.4, 16 10.5 / 9.6; plain (BH hash) k = 96 1 token 13.5 / 12.5, 16 19.8 / 17.4
    //   gather alone, the same tokens again and again (the rows of a few then stay in the L2): weighted, fp32, 768 wide, 4 tokens
    //   k = 48 3.8 / 3.9, k = 96 5.7 / 5.8, 64 tokens k = 32 4.7 / 4.3, k = 48 5.5 / 5.1, k = 96 10.4 / 8.2, 344 wide 500 tokens k = 24
    //   5.4 / 5.7, k = 40 6.8 / 6.9; k = 170, tau = 9, 512 wide 256 tokens 27.5 / 22.7, 500 39.4 / 36.7; fp16 768 wide k = 16 1 token
    //   2.8 / 2.8, 500 tokens k = 48 8.0 / 7.1, k = 170 20.5 / 12.9, 1000 21.8 / 18.8, 2000 (eight wavefronts) 33.7 / 35.4
    //   plain, fp32, 768 wide k = 48 8 tokens 3.7 / 3.8, k = 96 7.4 / 6.2, 64 tokens 9.7 / 7.9; 64 wide 64 tokens k = 64 3.8 / 4.0, k = 96
    //   5.9 / 5.6, 8 tokens 4.5 / 4.6; fp16 64 tokens k = 128 9.8 / 10.4
    // From five to eight (fp32 rows seven) sixteen in flight: weighted, fp16, k = 96, 768 wide 1000 tokens 14.8 / 13.4, k = 128,
    // 344 wide 2000 19.1 / 16.6, 3000 (nine) 26.6 / 27.6; fp32, k = 128, 344 wide 1000 tokens 21.0 / 19.4, 1500 (eight) 27.9 /
    // 28.9.
    if (lpt == 4 || lpt == 8 || lpt == 16) {
        if (mode == kWeighted && a.k >= 48) a.deep = cu_waves < 5 ? 16 : cu_waves < (T.kind ? 8 : 7) ? 8 : 0;
        else if (mode == kPlain && !T.kind && a.k >= 96 && cu_waves < 5) a.deep = 16;
    }
    if (opt.xcd_order == 1) xcd = true;
    if (opt.xcd_order == -1) xcd = false;
    a.xcd_mode = xcd;
    int64_t blocks;
    if (xcd) {
        // split the token range so that the number of units is a multiple of the XCD count
        const int splits = kXcds / gcd(a.n_slices, kXcds);
        a.tb_per_unit = (int)((ntb + splits - 1) / splits);
        a.n_units = a.n_slices * splits;
        blocks = (int64_t)(a.n_units / kXcds) * kXcds * a.tb_per_unit;
    } else {
        a.tb_per_unit = (int)ntb;
        a.n_units = a.n_slices;
        blocks = (int64_t)a.n_units * ntb;
    }
    if (blocks > 0x7FFFFFFFLL) return LFFN_E_SIZE;
    const dim3 grid = grid_of(blocks);
    TimedLaunch tl(1, s);
    rc = lffn_host::gather_direct_part(T.kind, lpt, a, mode == kProbes, grid, 64 * waves, s);
    if (rc != LFFN_OK) return rc;
    LFFN_HIP(hipGetLastError());
    tl.done();
    t_last_gather = "gather_kernel";
    return LFFN_OK;
}

// grid of the tiled re-pack kernels: one workgroup per 64 x 64 tile, capped (they stride over the rest)
unsigned repack_grid(int64_t n_rows, int64_t m)
{
    int64_t blocks = ((m + 63) / 64) * ((n_rows + 63) / 64);
    if (blocks > 16384) blocks = 16384;
    return (unsigned)(blocks < 1 ? 1 : blocks);
}

int launch_repack_codes(const uint16_t *codes, uint32_t *packed, int64_t n, int64_t n_pad, int k, int tau,
                        int shift, hipStream_t s)
{
    hipLaunchKernelGGL(repack_codes_kernel, dim3(repack_grid(n_pad, k / 2)), dim3(256), 0, s, codes, packed,
                       (long long)n, (long long)n_pad, k, tau, shift);
    LFFN_HIP(hipGetLastError());
    return LFFN_OK;
}

// ABI weights [n][m] -> table-major [m][n_pad]  (m = k, or k * (1 + tau) for the multi-probe shares)
int launch_repack_weights(const float *weights, float *wpk, int64_t n, int64_t n_pad, int64_t m, hipStream_t s)
{
    hipLaunchKernelGGL(repack_shares_kernel, dim3(repack_grid(n, m)), dim3(256), 0, s, weights, wpk, (long long)n,
                       (long long)n_pad, (long long)m);
    LFFN_HIP(hipGetLastError());
    return LFFN_OK;
}

// Launch shape of the lagged, bank-interleaved staged gather (gather_ring_kernel): prepared tables of up
// to 256 rows, plain sum.
struct RingPlan {
    bool use = false;
    GatherRingArgs a{};
    int threads = 0, tok = 0;
    unsigned grid = 0;
};

int plan_gather_ring(int64_t n, int k, int tau, int d_out, const TableRef &T, Mode mode, const Options &opt,
                     RingPlan *p)
{
    p->use = false;
    // On request only (gather_path 4).  Measured on the RoBERTa-base shape it does not beat the double-buffered
    // staged kernel: its reads are conflict-free, but it pays a barrier and an LDS write per table.
    if (opt.gather_path != 4 || mode != kPlain || !T.prepared || T.pw < 64) return LFFN_OK;
    if (tau < 7 || tau > 8 || k > 480) return LFFN_OK;   // 256-row slices; the re-pack kernel's 64 x k tile fits LDS
    if (n >= (int64_t(1) << 31) - 4096) return LFFN_OK;
    int cus = 0;
    int rc = device_cus(&cus);
    if (rc != LFFN_OK) return rc;
    if (cus < kXcds || cus % kXcds != 0) return LFFN_OK;
    const int rows = 1 << tau;
    GatherRingArgs &a = p->a;
    a = GatherRingArgs{};
    a.n = n;
    a.n_pad = packed_n_pad(n);
    a.k = k;
    a.tau = tau;
    a.d_out = d_out;
    a.nvec = d_out / 4;
    a.n_slices = (a.nvec + 3) / 4;
    a.token_splits = kXcds / gcd(a.n_slices, kXcds);
    a.n_units = a.n_slices * a.token_splits;
    a.blocks_per_xcd = cus / kXcds;
    a.row_stride = (uint32_t)T.pw;
    a.spp = (uint32_t)(T.pw / 64);
    a.table_stride = (uint32_t)(rows * T.pw);
    a.slice_stride = (unsigned long long)k * rows * T.pw;
    // tokens of the fullest workgroup, as the kernel splits them (in units of 16 tokens)
    const int64_t tpb = 16 * lds_tokens_per_block((n + 15) / 16, a.n_units, a.token_splits, a.blocks_per_xcd);
    // workgroup shapes that are built: (threads, token slots), a chunk holds threads / 4 * slots tokens
    static const int shapes[][2] = {{1024, 4}, {1024, 8}, {1024, 12}, {1024, 13}, {1024, 14}, {512, 8}, {512, 16}, {512, 20}, {512, 24}, {512, 28}, {512, 32}};
    int64_t cap_max = 0;
    for (auto &sh : shapes) {
        if (opt.ring_threads && sh[0] != opt.ring_threads) continue;
        if (opt.token_slots && sh[1] > opt.token_slots) continue;
        const int64_t cap = (int64_t)sh[0] / 4 * sh[1];
        if (cap > cap_max) cap_max = cap;
    }
    if (cap_max == 0) return LFFN_OK;
    const int64_t nchunks = (tpb + cap_max - 1) / cap_max;
    const int64_t chunk = ((tpb / 16 + nchunks - 1) / nchunks) * 16;  // tokens of the longest chunk
    // the shape with the fewest slots that holds a chunk; 1024 threads first (more waves to hide latency)
    int best = -1;
    for (int i = 0; i < (int)(sizeof(shapes) / sizeof(shapes[0])); ++i) {
        if (opt.ring_threads && shapes[i][0] != opt.ring_threads) continue;
        if (opt.token_slots && shapes[i][1] > opt.token_slots) continue;
        const int64_t cap = (int64_t)shapes[i][0] / 4 * shapes[i][1];
        if (cap < chunk) continue;
        if (best < 0 || cap < (int64_t)shapes[best][0] / 4 * shapes[best][1]) best = i;
    }
    if (best < 0) return LFFN_OK;
    p->threads = shapes[best][0];
    p->tok = shapes[best][1];
    p->grid = (unsigned)cus;
    p->use = true;
    return LFFN_OK;
}

int launch_gather_ring(const RingPlan &p, const uint16_t *codes, uint32_t *packed, const TableRef &T, void *y,
                       hipStream_t s)
{
    GatherRingArgs a = p.a;
    if (!packed || !T.prepared || a.n_pad < a.n + 16 * 256) return LFFN_E_UNSUPPORTED;
    // codes in the ABI layout -> lagged packed layout (scaled by the 256-byte LDS row stride)
    int64_t blocks = (a.n_pad + 63) / 64;
    if (blocks > 8192) blocks = 8192;
    const size_t tile = (size_t)64 * (a.k | 1) * sizeof(uint16_t);
    TimedLaunch tl(1, s);
    hipLaunchKernelGGL(repack_codes_lag_kernel, dim3((unsigned)blocks), dim3(256), tile, s, codes, packed,
                       (long long)a.n, (long long)a.n_pad, a.k, a.tau, kRingShift);
    LFFN_HIP(hipGetLastError());
    a.packed = packed;
    a.tables = T.p;
    a.y = y;
    a.y_kind = T.y_kind;
    int rc = lffn_host::gather_ring_part(p.threads, p.tok, a, dim3(p.grid), s);
    if (rc != LFFN_OK) return rc;
    LFFN_HIP(hipGetLastError());
    tl.done();
    t_last_gather = "gather_ring_kernel";
    return LFFN_OK;
}

// Tokens that the multi-probe form of the staged gather takes at once: the shares of a table must end before kProbesNoTable.
constexpr int64_t kProbesPiece = int64_t(1) << 25;
static_assert((10 + 1) * packed_n_pad(kProbesPiece) * 4 + kProbesWindow <= kProbesNoTable, "up to tau = 10");

// Gather from ABI-layout codes (and weights / shares): the staged kernel through the re-pack kernels when
// the plan says so and the scratch has room, else the direct kernel.
int gather_from_abi(Mode mode, const uint16_t *codes, const float *weights, const TableRef &T, void *y, int64_t n,
                    int k, int tau, int d_out, const LdsPlan &plan, Scratch *sc, hipStream_t s, const Options &opt)
{
    if (mode == kProbes && plan.use && n > kProbesPiece) {  // nearly equal pieces, one after another through the same scratch
        const int64_t pieces = (n + kProbesPiece - 1) / kProbesPiece;
        const int64_t m = ((n + pieces - 1) / pieces + 127) / 128 * 128;
        for (int64_t t = 0; t < n; t += m) {
            const int64_t len = std::min(m, n - t);
            LdsPlan piece;
            int rc = plan_gather_lds(len, k, tau, d_out, T, mode, Codes::kTurned, opt, &piece);
            if (rc != LFFN_OK) return rc;
            Scratch scratch = *sc;
            rc = gather_from_abi(mode, codes + t * k, weights + t * k * (1 + tau), T,
                                 static_cast<char *>(y) + t * d_out * (T.y_kind ? 2 : 4), len, k, tau, d_out, piece,
                                 &scratch, s, opt);
            if (rc != LFFN_OK) return rc;
        }
        return LFFN_OK;
    }
    RingPlan ring;
    int rrc = plan_gather_ring(n, k, tau, d_out, T, mode, opt, &ring);
    if (rrc != LFFN_OK) return rrc;
    if (ring.use) {
        uint32_t *packed = sc->take<uint32_t>(packed_bytes(n, k));
        if (packed) return launch_gather_ring(ring, codes, packed, T, y, s);
    }
    if (plan.use && aligned(codes, 4)) {
        uint32_t *packed = sc->take<uint32_t>(packed_bytes(n, k));
        float *wpk = mode == kWeighted ? sc->take<float>(wpk_bytes(n, k))
                     : mode == kProbes ? sc->take<float>(spk_bytes(n, k, tau)) : nullptr;
        if (packed && (mode == kPlain || wpk)) {
            int rc = launch_repack_codes(codes, packed, n, plan.a.n_pad, k, tau, plan.shift, s);
            if (rc != LFFN_OK) return rc;
            if (mode != kPlain) {
                rc = launch_repack_weights(weights, wpk, n, plan.a.n_pad, (int64_t)k * (mode == kProbes ? tau + 1 : 1), s);
                if (rc != LFFN_OK) return rc;
            }
            rc = launch_gather_lds(plan, packed, wpk, T, y, mode, s);
            if (rc != LFFN_OK || !plan.tail) return rc;
            rc = launch_gather_direct(codes, weights, T, y, n, k, tau, d_out, mode, s, opt, k - plan.tail);
            t_last_gather = "gather_lds_kernel";  // the one that did all tables but the last
            return rc;
        }
    }
    return launch_gather_direct(codes, weights, T, y, n, k, tau, d_out, mode, s, opt);
}

// ---- BH{m} hash --------------------------------------------------------------------------------
// The BH kernel reduces a table's weight inside one 16-coordinate tile of z (tau = 4, 8, 16); for any other tau it
// forms the weights from z through a window in LDS.
bool bh_weights_in_registers(int tau) { return tau == 4 || tau == 8 || tau == 16; }

// The range of P and tau the BH entry points accept: the bit strings (and the z window) of 64 tokens beside 64 KB.
// The kernel needs less for every shape in it (at most 124 KB).
bool bh_shape_fits(int P, int N, bool window)
{
    const size_t bytes = 64 * 1024 + 256 * (size_t)hash_bit_words(P, N) + (window ? 256 * (size_t)((N < 128 ? N : 128) + 17) : 0);
    return P <= 64 && bytes <= 150 * 1024;
}

int check_bh(const void *x, const float *bmats, int64_t n, int d, int k, int tau, int block, int n_factors,
             int x_dtype, bool weighted = false)
{
    if (!x || !bmats) return LFFN_E_NULL;
    if (n < 0 || d < 1 || k < 1 || n_factors < 1) return LFFN_E_SIZE;
    if (tau < 1 || tau > 16) return LFFN_E_TAU;
    if (!dtype_ok(x_dtype)) return LFFN_E_DTYPE;
    if (k > (1 << 20) || n > (int64_t(1) << 40) || n_factors > 64) return LFFN_E_SIZE;
    const int L = log2_pad(d);
    if (L > 10 || d > 1024) return LFFN_E_UNSUPPORTED;
    const int N = L < 6 ? 64 : 1 << L;  // widths below 64 are not built
    if (L < 6) return LFFN_E_UNSUPPORTED;
    const int b = block & ~LFFN_PREPARED;
    if (b != 16 && b != 32 && b != 64) return LFFN_E_UNSUPPORTED;
    if (b > N) return LFFN_E_SIZE;
    const int64_t P = ((int64_t)k * tau + N - 1) / N;
    if (P > 64 || !bh_shape_fits((int)P, N, weighted && !bh_weights_in_registers(tau))) return LFFN_E_UNSUPPORTED;
    if (!aligned(x, x_dtype == LFFN_F32 ? 4 : 2) || !aligned(bmats, (block & LFFN_PREPARED) ? 256 : 4)) return LFFN_E_ALIGN;
    return LFFN_OK;
}

int64_t bh_pack_bytes(int d, int k, int tau, int block, int n_factors)
{
    const int N = 1 << log2_pad(d);
    const int64_t P = ((int64_t)k * tau + N - 1) / N;
    return round256(P * n_factors * (int64_t)N * block * 4);
}

// The factors in MFMA-operand order (one-time: lookupffn_prepare_bh, or per call into scratch)
int launch_bh_pack(const float *bmats, float *apack, int d, int k, int tau, int block, int n_factors, hipStream_t s)
{
    const int N = 1 << log2_pad(d);
    const int64_t P = ((int64_t)k * tau + N - 1) / N;
    const long long total = (long long)P * n_factors * N * block;
    long long pb = (total + 255) / 256;
    if (pb > 2048) pb = 2048;
    hipLaunchKernelGGL(bh_pack_kernel, dim3((unsigned)pb), dim3(256), 0, s, bmats, apack, N, block, total);
    LFFN_HIP(hipGetLastError());
    return LFFN_OK;
}

// Up to how many transforms, in fills of the chip (cus * 1024 / d_pad: the workgroups that it holds), bh_lane_kernel takes a batch:
// two or four tokens to a workgroup, a wave to 64 coordinates of them.  Hash alone, us, bh_hash_kernel / two tokens a workgroup / four:
//   d = 768, k = 96, tau = 8, weights, block 64: 1 token 29.2 / 13.7 / 15.5, 128 32.4 / 14.6 / 16.5, 512 32.6 / 16.7 / 16.6, 1024
//   32.6 / 29.7 / 17.8, 2048 32.5 / 54.7 / 32.4; block 16: 128 21.1 / 6.6 / 8.5, 2048 21.6 / 20.6 / 15.6, 4096 22.3 / 38.5 / 28.7;
//   codes, block 32: 128 23.9 / 9.2 / 11.0, 2048 23.8 / 30.1 / 20.4, 4096 24.5 / 57.0 / 38.3
//   d = 768, k = 170, tau = 9 (two projections): 128 67.7 / 26.2 / 29.9, 1024 68.1 / 53.9 / 31.8
//   d = 512, k = 256 (four), block 64: 128 32.8 / 10.5 / 10.8, 512 32.8 / 27.8 / 17.6, 1024 32.6 / 48.0 / 30.4, 2048 32.9 / 86.7 / 54.9
//   d = 256, codes, k = 96 (three), block 64: 1800 (5.3 fills) 25.9 / 35.1 / 22.1, 2300 (6.7) 25.8 / 39.9 / 31.1; k = 8, block 16: 8192 (8)
//   15.3 / 15.2 / 12.6
//   d = 64, codes, k = 24 (three), block 64: 2600 (1.9) 10.0 / 12.2 / 9.0, 4096 (3) 10.1 / 16.2 / 11.6
// Every group of tokens reads all factors, n_factors * block KB into a compute unit for each fill, bh_hash_kernel a quarter
// to a sixteenth of that, and it spreads the projections of narrow rows out: the more bytes and the narrower the row, the
// sooner it is ahead.  Fills at the first loss, blocks 16 / 32 / 64, of 1 ... 36 projections, codes and weights: d = 128 one factor
// 8 / 8 / 4.5, two 6 / 4.1 / 4, four 4.1 / 4.1 / 3, sixteen 4.1 / 3.5 / 2.5; d = 64 one 8 / 6 / 2.75, two 5.3 / 3.4 / 2.15, four
// 3 / 2.3 / 2.05, sixteen 2.05 / 2.05 / 1.2.  So a part of the width and one that goes with 1 / bytes, and more where bh_hash_kernel
// forms the weights through its window (d = 64, k = 97, tau = 7, two factors, block 16, 2048 tokens, 5.5 fills 13.7 / 10.3 / 9.4).  d = 256
// first loses at 6.7, and not before 8 with blocks of 16 and 32 or where tables cross into a projection that both then hash
// twice (k = 40, tau = 9, 3500 tokens, block 64 46.6 / 41.8 / 30.0), but for three in a chain (k = 96, block 32, 2300 tokens 19.3 / 23.3 / 21.2).
double bh_lane_most(int N, int P, bool cross, int block, int n_factors, bool window)
{
    if (N >= 512) return block == 64 ? 4 : 8;
    if (N == 256) return (P > 1 && cross) || (P != 3 && block < 64) ? 8 : 6;
    const int bytes = n_factors * block;  // KB a compute unit and fill
    const double most = (N == 128 ? 2.5 : bytes <= 512 ? 1.2 : 1.0) + (window ? 32.0 / block : 0.0) + 100.0 / bytes;
    const double least = bytes > 256 ? 0.0 : N == 64 ? 2.0 : block < 64 ? 4.0 : 0.0;
    return std::min(8.0, std::max(most, least));
}

// Workgroups to the tokens of bh_hash_kernel's grid, and whether it spreads their projections over others with codes in the ABI layout
int64_t bh_token_blocks(int64_t n, int L)
{
    const int wpg = L == 10 ? 4 : L == 9 ? 2 : 1;  // waves that share a token group
    const int64_t per_block = (int64_t)(kBhWaves / wpg) * kBhTok;
    return (n + per_block - 1) / per_block;
}
bool bh_spreads(int64_t n, int d, int k, int tau, int cus)
{
    const int L = log2_pad(d);
    return (int64_t)k * tau > (int64_t(1) << L) && 2 * bh_token_blocks(n, L) <= cus;
}

// Hashes with the packed factors `apack`; `pack_from` != NULL: re-order them from there first.  few_ok: bh_lane_kernel may take
// the batch (the forward passes; the stand-alone hash keeps bh_hash_kernel, and so the one can be held against the other).
int launch_hash_bh(const void *x, const float *pack_from, const float *apack_in, float *apack_scratch,
                   const HashOut &out, int64_t n, int d, int k, int tau, int block, int n_factors, int x_dtype,
                   bool few_ok, hipStream_t s)
{
    const int L = log2_pad(d);
    const int N = 1 << L;
    BhArgs a{};
    a.x = x;
    a.apack = pack_from ? apack_scratch : apack_in;
    a.codes = out.codes;
    a.packed = out.codes ? nullptr : out.packed;
    a.weights = out.codes ? out.weights : nullptr;
    a.wpk = out.codes ? nullptr : out.weights;
    a.n_pad = packed_n_pad(n);
    a.packed_shift = out.shift;
    a.n = n;
    a.d = d;
    a.k = k;
    a.tau = tau;
    a.n_factors = n_factors;
    a.P = (int)(((int64_t)k * tau + N - 1) / N);
    a.x_kind = x_dtype;  // LFFN_F32 / BF16 / F16 are the kernels' kinds 0 / 1 / 2
    a.x_vec4 = d % 4 == 0 && aligned(x, a.x_kind ? 8 : 16);
    a.scale = (float)(1.0 / std::sqrt((double)N));
    if (!a.apack || (!a.codes && !a.packed) || out.probes) return LFFN_E_NULL;
    TimedLaunch tl(0, s);
    if (pack_from) {
        int rc = launch_bh_pack(pack_from, apack_scratch, d, k, tau, block, n_factors, s);
        if (rc != LFFN_OK) return rc;
    }
    int cus = 0, rc = device_cus(&cus);
    if (rc != LFFN_OK) return rc;
    const int64_t fill = (int64_t)cus * (1024 / N);  // workgroups that the chip holds
    if (few_ok && a.codes && (double)(n * a.P) <= bh_lane_most(N, a.P, N % tau != 0, block, n_factors, out.weights && !bh_weights_in_registers(tau)) * (double)fill) {
        const int tokens = n * a.P <= 2 * (int64_t)cus * std::max(1, 256 / N) ? 2 : 4;
        const int64_t groups = (n + tokens - 1) / tokens;
        dim3 grid = grid_of(groups);
        a.p_per = a.P;
        a.cross = N % tau != 0;
        if (a.P > 1) grid.z = split_projections(a.P, a.cross, std::max<int64_t>(1, fill / groups), &a.p_per);
        rc = lffn_host::bh_lane_part(L, out.weights != nullptr, tokens, a, block, grid, s);
        if (rc != LFFN_OK) return rc;
        LFFN_HIP(hipGetLastError());
        tl.done();
        return LFFN_OK;
    }
    const int wmode = !out.weights ? 0 : bh_weights_in_registers(tau) ? 1 : 2;
    const int64_t blocks = bh_token_blocks(n, L);
    dim3 grid = grid_of(blocks);  // a workgroup past the batch does a full hash of no token
    const bool deep_ok = block == 64 && L == 10;
    // as many workgroups to the projections as find a compute unit each (2 tokens: d = 64, block 32, 20 projections pass
    // 77 -> 16 us, d = 256, 6 projections with tables across them 93 -> 40)
    a.p_per = a.P;
    a.cross = N % tau != 0;
    if (a.codes && a.P > 1) grid.z = split_projections(a.P, a.cross, (int64_t)cus / blocks, &a.p_per);
    // With a wave alone on its SIMD the form with more operands in flight is faster at d_pad = 1024 with blocks of 64: the factors
    // come from beyond the L2 wherever a model has more than a few layers.  Hash without / with it, us, k = 96, tau = 8, twelve
    // layers in turn: 1 token 27.8 / 27.5, 128 31.9 / 30.8, weighted 34.2 / 32.4, 4096 tokens 32.4 / 31.7 (passes of 128 tokens,
    // weighted 52.5 / 43.0); three layers in turn, whose factors stay in the L2: 128 tokens 29.1 / 30.5, weighted 31.5 / 32.1, 4096
    // 32.4 / 31.8; k = 170, tau = 9, weighted 128 tokens 75.0 / 67.6 either way.  At other shapes it is not (block 32: 10 tokens
    // 31.1 / 31.4, block 16: 216 tokens of 256 36.3 / 37.1, block 64: 5 tokens of 512 28.7 / 30.4).
    if (deep_ok && blocks * grid.z <= cus) rc = lffn_host::bh_few_part(wmode, a, grid, s);
    else if (L <= 8) rc = lffn_host::bh_lo_part(L, wmode, a, block, grid, s);
    else if (L == 9) rc = lffn_host::bh_512_part(wmode, a, block, grid, s);
    else rc = lffn_host::bh_1024_part(wmode, a, block, grid, s);
    if (rc != LFFN_OK) return rc;
    LFFN_HIP(hipGetLastError());
    tl.done();
    return LFFN_OK;
}

// ---------------------------------------------------------------- the forward pass, all variants
// ---------------------------------------------------------------- the one-launch path for a few tokens
int64_t stack_table_bytes(const TableRef &T, int k, int tau, int d_out)
{
    return T.prepared ? prepared_tables_bytes(k, tau, d_out) : ((int64_t)k << tau) * d_out * (T.kind ? 2 : 4);
}

// Whether forward_stack_kernel takes this shape (checked without a HIP call).
bool stack_shape_ok(const void *x, const int8_t *const *signs, const void *const *tables, int n_layers, int64_t n,
                    int d, int k, int tau, int d_out, int n_rounds, int x_dtype, int table_dtype)
{
    if (log2_pad(d) != 10 || n_rounds > 4 || n_layers < 1 || n_layers > kStackMaxLayers) return false;
    if (n_layers > 1 && d_out != d) return false;
    if (n > 0x7FFFFFFF) return false;
    const bool xb = x_dtype != LFFN_F32;
    const size_t xrow = (size_t)d * (xb ? 2 : 4);
    if (d % 4 == 0 && !(aligned(x, 16) && xrow % (xb ? 8 : 16) == 0)) return false;
    for (int l = 0; l < n_layers; ++l)
        if (!aligned(signs[l], 16)) return false;
    const int P = (int)(((int64_t)k * tau + 1023) / 1024);
    if (!stack_range_ok(P, k)) return false;
    return stack_table_bytes(table_ref(tables[0], table_dtype, tau), k, tau, d_out) < (int64_t(1) << 31);
}

// Whether forward_small_kernel takes this single layer: d_pad 64 .. 512 (any number of rounds, any alignment the
// entry points accept: rows and signs are read element by element) and a table set below 2 GiB.  `by_rate`: leave out
// batches of many or wide rows.  A token's rows come in through one compute unit, a lane to each of up to 1024 dwords, wider rows
// 1024 dwords after another, and every turn of up to 32 rows is a chain of its own however few the tokens.
// Where the lines lie: up to a token to each compute unit all of up to four turns of 4 KB by 32 tables (by more when the tokens and
// tables are many), beyond that while the rows are 40 MiB and one and a half turns; tables that stay in the 256 MiB memory-side cache.
// One launch against two, us a pass (fp32 prepared, tau = 8, d = 512 where not said):
//   k = 8, 64 wide, d = 64: 64 tokens 3.7 / 5.6, 512 3.8 / 5.7; k = 256, 512 wide: 64 12.8 / 17.9, 256 22.7 / 20.9
//   k = 96, 768 wide: 128 tokens 11.1 / 12.1, 192 13.2 / 13.5, 256 15.6 / 14.5, 512 (144 MiB of rows) 24.8 / 18.4
//   512 tokens: d = 256, k = 64, 256 wide 8.5 / 8.9, k = 96 10.8 / 10.6; tau = 7, k = 97, 512 wide (97 MiB) 18.0 / 14.0
//   two turns and more: k = 64, 2048 wide: 1 token 11.3 / 8.4, 128 15.9 / 15.5; k = 96 1 token 13.0 / 9.9; k = 64, 4096 wide, 64 tokens 22.7 / 16.4;
//   k = 8, 6144 wide, 128 tokens 12.0 / 9.2; 300 tokens: k = 8, 2048 wide 9.3 / 8.1, k = 16, 1280 wide 9.3 / 8.4
//   tau = 10, k = 128, 1024 wide (512 MiB of tables, other tokens in every pass): 1 token 16.6 / 12.6, 64 29.6 / 20.7
// The lines were drawn against a slower hash of few tokens and a slower direct gather: where rows are wide, or the tokens near the
// compute units' number and the tables many, two launches are now up to a third shorter.
constexpr int64_t kSmallRowBytes = 40 << 20, kSmallTableBytes = 256 << 20;
bool small_shape_ok(int64_t n, int d, int k, int tau, int d_out, int table_dtype, const void *tables, bool by_rate)
{
    const int L = log2_pad(d);
    if (L < 6 || L > 9 || n > 0x7FFFFFFF) return false;
    const int N = 1 << L;
    const int P = (int)(((int64_t)k * tau + N - 1) / N);
    if (small_lds_bytes(P, N, k) > 64 * 1024) return false;
    const TableRef T = table_ref(tables, table_dtype, tau);
    const int64_t bytes = stack_table_bytes(T, k, tau, d_out);
    if (bytes >= (int64_t(1) << 31)) return false;
    if (!by_rate) return true;
    int cus = 0;
    if (bytes > kSmallTableBytes || device_cus(&cus) != LFFN_OK) return false;
    const int64_t row = (int64_t)d_out * (T.prepared || !T.kind ? 4 : 2);
    const int64_t turns = (row * ((k + kStackChunk - 1) / kStackChunk) + 2048) / 4096;
    if (row > 4096 && !(n <= cus ? turns <= 4 || (k >= 64 && n >= 10 * turns) : turns <= 1)) return false;
    return n <= cus || n * k * row <= kSmallRowBytes;
}

// One launch that reads x and signs and writes y: workgroups run in any order, so y must not lie where another token is
// still to be read from.  In place with rows of one length is fine: a workgroup reads its own row before it writes it.
bool one_launch_overlap_ok(const void *x, const int8_t *signs, const void *y, int64_t n, int d, int k, int tau,
                           int d_out, int n_rounds, int x_dtype, int table_dtype)
{
    const int N = 1 << log2_pad(d);
    const int64_t P = ((int64_t)k * tau + N - 1) / N;
    const int64_t x_row = (int64_t)d * (x_dtype == LFFN_F32 ? 4 : 2);
    const int64_t y_row = (int64_t)d_out * ((table_dtype & (LFFN_Y_BF16 | LFFN_Y_F16)) ? 2 : 4);
    auto apart = [&](const void *p, int64_t bytes) {
        const uintptr_t a = reinterpret_cast<uintptr_t>(p), b = reinterpret_cast<uintptr_t>(y);
        return a + (uintptr_t)bytes <= b || b + (uintptr_t)(n * y_row) <= a;
    };
    return apart(signs, P * n_rounds * N) && (apart(x, n * x_row) || (x == y && x_row == y_row));
}

// Call only with stack_shape_ok(...) (d_pad = 1024) or small_shape_ok(...) true and every argument validated.
int launch_forward_stack(const void *x, const int8_t *const *signs, const void *const *tables, void *y, int64_t n,
                         int d, int k, int tau, int d_out, int n_rounds, int n_layers, int x_dtype, int table_dtype,
                         hipStream_t s)
{
    const TableRef T = table_ref(tables[0], table_dtype, tau);
    StackArgs a{};
    a.x = x;
    a.y = y;
    a.y_kind = T.y_kind;
    for (int l = 0; l < n_layers; ++l) {
        a.signs[l] = signs[l];
        a.tables[l] = static_cast<const char *>(tables[l]);
    }
    a.n = n;
    a.d = d;
    a.d_out = d_out;
    a.k = k;
    a.tau = tau;
    const int L = log2_pad(d), N = 1 << L;
    a.P = (int)(((int64_t)k * tau + N - 1) / N);
    a.n_layers = n_layers;
    a.n_rounds = n_rounds;
    a.x_kind = x_dtype;  // LFFN_F32 / BF16 / F16 are the kernels' kinds 0 / 1 / 2
    a.scale = (float)(1.0 / std::sqrt((double)N));
    const int64_t rows = int64_t(1) << tau;
    if (T.prepared) {
        a.row_dwords = (uint32_t)d_out;
        a.piece_shift = T.pw == 128 ? 7 : 6;
        a.row_stride = (uint32_t)T.pw;
        a.slice_stride = (uint32_t)((int64_t)k * rows * T.pw);
        a.table_bytes = (uint32_t)prepared_tables_bytes(k, tau, d_out);
    } else {
        const int64_t row_bytes = (int64_t)d_out * (T.kind ? 2 : 4);
        a.row_dwords = (uint32_t)(row_bytes / 4);
        a.piece_shift = 31;
        a.row_stride = (uint32_t)row_bytes;
        a.slice_stride = 0;
        a.table_bytes = (uint32_t)((int64_t)k * rows * row_bytes);
    }
    // forward_small_kernel is the call's hash and its gather, and counts as each with its whole duration
    TimedLaunch th(0, s, L != 10), tl(1, s);
    int rc;
    bool narrow = false;
    if (L == 10) {
        // One layer of rows up to 2 KB, more tokens than forward_stack_kernel takes in one round of two to a compute unit: forward_narrow_kernel.
        // That kernel / this, 500 shapes of 513 ... 16384 tokens: 64 ... 256 dwords 1.97 ... 1.42 : 1 (0.97 ... 3.9), 320 1.23 : 1 (0.98 ... 1.67), 512
        // 1.16 : 1 (0.91 ... 1.5), 640 1.0 : 1 (0.82 ... 1.3).
        // Else two tokens to a workgroup where there are more tokens than compute units (and the LDS is what every kernel may use).
        int cus = 0;
        rc = device_cus(&cus);
        if (rc != LFFN_OK) return rc;
        // What is left over from whole rounds of two goes a token to a workgroup where that is one round.
        const int tokens = n > cus && stack_lds_bytes(k, 2) <= 64 * 1024 ? 2 : 1;
        const int64_t left = n % (2 * (int64_t)cus), ones = tokens == 1 ? n : n > 2 * (int64_t)cus && left <= cus ? left : 0;
        a.twos = (n - ones + 1) / 2;
        if ((narrow = n_layers == 1 && n > 2 * (int64_t)cus && a.row_dwords <= kNarrowDwords))
            rc = lffn_host::forward_narrow_part(n_rounds, T.kind, a, grid_of(n), (int)((a.row_dwords + 63) / 64 * 64), narrow_lds_bytes(a.P, k), s);
        else rc = lffn_host::forward_stack_part(n_rounds, T.kind, a, grid_of(a.twos + ones), tokens, stack_lds_bytes(k, tokens), s);
    } else {
        int threads = (int)((a.row_dwords + 63) / 64 * 64);
        if (threads > 1024) threads = 1024;
        threads = std::max(threads, 64 * std::min(a.P, 16));  // a wave per projection
        rc = lffn_host::forward_small_part(L, T.kind, a, grid_of(n), threads, small_lds_bytes(a.P, N, k), s);
    }
    if (rc != LFFN_OK) return rc;
    LFFN_HIP(hipGetLastError());
    tl.done();
    th.done();
    t_last_gather = t_last_hash = narrow ? "forward_narrow_kernel" : L == 10 ? "forward_stack_kernel" : "forward_small_kernel";
    return LFFN_OK;
}

// Hash: the sign-diagonal rounds (`signs`, n_rounds) or the BH factors (`bmats`, block, n_factors).
struct HashSpec {
    const int8_t *signs = nullptr;
    int n_rounds = 0;
    const float *bmats = nullptr;  // row-major factors, or the prepared copy when `bh_prepared`
    int block = 0, n_factors = 0;
    bool bh_prepared = false;
    bool bh() const { return bmats != nullptr; }
};

int64_t forward_need(const HashSpec &h, Mode mode, int64_t n, int d, int k, int tau)
{
    if (n <= 0) return 0;
    const int64_t pack = (h.bh() && !h.bh_prepared) ? bh_pack_bytes(d, k, tau, h.block, h.n_factors) : 0;
    return sat_add(pack, forward_ws_bytes(n, k, tau, mode));
}

int forward_core(const HashSpec &h, Mode mode, const void *x, const void *tables, void *y, int64_t n, int d,
                 int k, int tau, int d_out, int x_dtype, int table_dtype, void *workspace,
                 int64_t workspace_bytes, hipStream_t s)
{
    const uint16_t *stand_in = reinterpret_cast<const uint16_t *>(uintptr_t(256));  // the codes live in scratch
    int rc = h.bh() ? check_bh(x, h.bmats, n, d, k, tau, h.block | (h.bh_prepared ? LFFN_PREPARED : 0), h.n_factors,
                               x_dtype, mode == kWeighted)
                    : check_hash(x, h.signs, stand_in, n, d, k, tau, h.n_rounds, x_dtype, mode != kPlain);
    if (rc != LFFN_OK) return rc;
    if (h.bh() && mode == kProbes) return LFFN_E_UNSUPPORTED;
    rc = check_gather(stand_in, tables, y, n, k, tau, d_out, table_dtype);
    if (rc != LFFN_OK) return rc;
    const int64_t need = forward_need(h, mode, n, d, k, tau);
    Scratch sc;
    if (workspace) {  // a caller's buffer is checked even for an empty batch
        if (workspace_bytes < need) return LFFN_E_WORKSPACE;
        if (!aligned(workspace, 256)) return LFFN_E_ALIGN;
    }
    if (n == 0) return LFFN_OK;
    const Options opt = options_snapshot();
    if (!h.bh() && mode == kPlain && opt.gather_path == 0 && opt.hash_path == 0 && opt.small_tokens >= 0 &&
        n <= (opt.small_tokens ? opt.small_tokens : kSmallTokensDefault) &&
        (stack_shape_ok(x, &h.signs, &tables, 1, n, d, k, tau, d_out, h.n_rounds, x_dtype, table_dtype) ||
         small_shape_ok(n, d, k, tau, d_out, table_dtype, tables, opt.small_tokens == 0)) &&
        one_launch_overlap_ok(x, h.signs, y, n, d, k, tau, d_out, h.n_rounds, x_dtype, table_dtype))
        return launch_forward_stack(x, &h.signs, &tables, y, n, d, k, tau, d_out, h.n_rounds, 1, x_dtype, table_dtype, s);
    rc = get_scratch(workspace, workspace_bytes, need, &sc);
    if (rc != LFFN_OK) return rc;
    const TableRef T = table_ref(tables, table_dtype, tau);
    // a batch that goes in pieces is cut from the ABI layout
    const bool row_shares = mode == kProbes && n <= kProbesPiece && hash_row_ok(h.signs, true, true, true, n, d, k, tau, h.n_rounds, opt);
    Codes codes = k % 2 || (mode == kProbes && !row_shares) ? Codes::kTurned : Codes::kPacked;
    if (h.bh() && d <= (tau <= 8 ? 512 : 256) && codes == Codes::kPacked) {
        int cus = 0;
        rc = device_cus(&cus);
        if (rc != LFFN_OK) return rc;
        if (bh_spreads(n, d, k, tau, cus) && !(tau == 10 && d > 128 && h.block < 64)) codes = Codes::kPackedInChain;
    }
    LdsPlan plan;
    rc = plan_gather_lds(n, k, tau, d_out, T, mode, codes, opt, &plan);
    if (rc != LFFN_OK) return rc;
    float *apack = (h.bh() && !h.bh_prepared) ? sc.take<float>(bh_pack_bytes(d, k, tau, h.block, h.n_factors)) : nullptr;
    if (h.bh() && !h.bh_prepared && !apack) return LFFN_E_WORKSPACE;
    auto run_hash = [&](const HashOut &out) -> int {
        if (h.bh())
            return launch_hash_bh(x, h.bh_prepared ? nullptr : h.bmats, h.bh_prepared ? h.bmats : nullptr, apack, out, n,
                                  d, k, tau, h.block, h.n_factors, x_dtype, true, s);
        return launch_hash(x, h.signs, out, n, d, k, tau, h.n_rounds, x_dtype, true, s, opt);
    };
    // the hash kernels write the staged gather's layout themselves, scaled for its row pieces; multi-probe shares only
    // hash_row_kernel does
    RingPlan ring;
    rc = plan_gather_ring(n, k, tau, d_out, T, mode, opt, &ring);
    if (rc != LFFN_OK) return rc;
    if (!ring.use && plan.use && !plan.tail && (mode != kProbes || row_shares)) {
        HashOut out;
        out.shift = plan.shift;
        out.probes = mode == kProbes;
        const int64_t pb = packed_bytes(n, k), wb = mode == kWeighted ? wpk_bytes(n, k) : mode == kProbes ? spk_bytes(n, k, tau) : 0;
        out.packed = sc.take<uint32_t>(pb);
        out.weights = mode != kPlain ? sc.take<float>(wb) : nullptr;
        if (!out.packed || (mode != kPlain && !out.weights)) return LFFN_E_WORKSPACE;
        if (!hash_extents_ok(out, n, k, tau, plan.a.n_pad, 0, pb, wb)) return LFFN_E_WORKSPACE;
        rc = run_hash(out);
        if (rc != LFFN_OK) return rc;
        return launch_gather_lds(plan, out.packed, out.weights, T, y, mode, s);
    }
    HashOut out;
    const int64_t cb = abi_codes_bytes(n, k), wb = abi_weights_bytes(n, k, tau, mode);
    out.codes = sc.take<uint16_t>(cb);
    out.weights = mode != kPlain ? sc.take<float>(wb) : nullptr;
    out.probes = mode == kProbes;
    if (!out.codes || (mode != kPlain && !out.weights)) return LFFN_E_WORKSPACE;
    if (!hash_extents_ok(out, n, k, tau, plan.a.n_pad, cb, 0, wb)) return LFFN_E_WORKSPACE;
    rc = run_hash(out);
    if (rc != LFFN_OK) return rc;
    return gather_from_abi(mode, out.codes, out.weights, T, y, n, k, tau, d_out, plan, &sc, s, opt);
}

int gather_core(Mode mode, const uint16_t *codes, const float *weights, const void *tables, void *y, int64_t n,
                int k, int tau, int d_out, int table_dtype, void *workspace, int64_t workspace_bytes, hipStream_t s)
{
    int rc = check_gather(codes, tables, y, n, k, tau, d_out, table_dtype);
    if (rc == LFFN_OK && mode != kPlain) rc = check_weights(weights);
    if (rc != LFFN_OK) return rc;
    const int64_t need = gather_ws_bytes(n, k, tau, mode);
    if (workspace) {
        if (workspace_bytes < need) return LFFN_E_WORKSPACE;
        if (!aligned(workspace, 256)) return LFFN_E_ALIGN;
    }
    if (n == 0) return LFFN_OK;
    const Options opt = options_snapshot();
    const TableRef T = table_ref(tables, table_dtype, tau);
    LdsPlan plan;
    rc = plan_gather_lds(n, k, tau, d_out, T, mode, Codes::kCallers, opt, &plan);
    if (rc != LFFN_OK) return rc;
    RingPlan ring;
    rc = plan_gather_ring(n, k, tau, d_out, T, mode, opt, &ring);
    if (rc != LFFN_OK) return rc;
    Scratch sc;
    if (ring.use || (plan.use && aligned(codes, 4))) {  // only the staged kernels need scratch
        rc = get_scratch(workspace, workspace_bytes, need, &sc);
        if (rc != LFFN_OK) return rc;
    }
    return gather_from_abi(mode, codes, weights, T, y, n, k, tau, d_out, plan, &sc, s, opt);
}

HashSpec sign_hash(const int8_t *signs, int n_rounds)
{
    HashSpec h;
    h.signs = signs;
    h.n_rounds = n_rounds;
    return h;
}
HashSpec bh_hash(const float *bmats, int block, int n_factors)
{
    HashSpec h;
    h.bmats = bmats;
    h.block = block & ~LFFN_PREPARED;
    h.n_factors = n_factors;
    h.bh_prepared = (block & LFFN_PREPARED) != 0;
    return h;
}

// stand-alone BH hash (codes, and weights for the weighted variant) into caller buffers
int hash_bh_core(const void *x, const float *bmats, uint16_t *codes, float *weights, bool weighted, int64_t n, int d,
                 int k, int tau, int block, int n_factors, int x_dtype, void *workspace, int64_t workspace_bytes,
                 hipStream_t s)
{
    int rc = check_bh(x, bmats, n, d, k, tau, block, n_factors, x_dtype, weighted);
    if (rc != LFFN_OK) return rc;
    if (!codes || (weighted && !weights)) return LFFN_E_NULL;
    if (!aligned(codes, 2) || (weighted && !aligned(weights, 4))) return LFFN_E_ALIGN;
    const HashSpec h = bh_hash(bmats, block, n_factors);
    const int64_t pb = h.bh_prepared ? 0 : bh_pack_bytes(d, k, tau, h.block, n_factors);
    const int64_t need = pb;
    if (workspace) {
        if (workspace_bytes < need) return LFFN_E_WORKSPACE;
        if (!aligned(workspace, 256)) return LFFN_E_ALIGN;
    }
    if (n == 0) return LFFN_OK;
    Scratch sc;
    rc = get_scratch(workspace, workspace_bytes, need, &sc);
    if (rc != LFFN_OK) return rc;
    float *apack = h.bh_prepared ? nullptr : sc.take<float>(pb);
    if (!h.bh_prepared && !apack) return LFFN_E_WORKSPACE;
    HashOut out;
    out.codes = codes;
    out.weights = weighted ? weights : nullptr;
    return launch_hash_bh(x, h.bh_prepared ? nullptr : bmats, h.bh_prepared ? bmats : nullptr, apack, out, n, d, k,
                          tau, h.block, n_factors, x_dtype, false, s);
}

bool bh_shape_ok(int d, int k, int tau, int block, int n_factors)
{
    return !(d < 1 || d > 1024 || k < 1 || tau < 1 || tau > 16 || block < 1 || n_factors < 1 || n_factors > 64);
}

}  // namespace

extern "C" {

int lookupffn_init(void)
{
    int cus = 0;
    int rc = device_cus(&cus);
    if (rc != LFFN_OK) return rc;
    {
        void *p = nullptr;  // the static scratch array's address on this device
        rc = static_scratch(&p);
        if (rc != LFFN_OK) return rc;
    }
    // code objects are loaded on first use: do that now for the two parts no attribute call below touches
    // (this one: hash, re-pack and prepare kernels; and the direct gather's)
    {
        hipFuncAttributes attr;
        LFFN_HIP(hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(repack_codes_kernel)));
        rc = lffn_host::gather_direct_load();
        if (rc != LFFN_OK) return rc;
    }
    // every kernel that asks for more than 64 KB of dynamic LDS is told so now, so that no later launch
    // has to (the attribute call is not a stream operation and has no place inside a graph capture)
    lffn_host::AttrOnly scope;
    const size_t lds = 160 * 1024;
    GatherLdsArgs ga{};
    BhArgs ba{};
    for (int tok : kLdsSlots)
        for (int fr : {1, 2, 4})
            for (int sw : {4, 8}) {
                for (int part = 0; part < 3; ++part) {
                    rc = part == 0   ? lffn_host::gather_lds_plain_part(tok, ga, fr, sw, dim3(1), lds, nullptr)
                         : part == 1 ? lffn_host::gather_lds_weighted_part(tok, ga, fr, sw, dim3(1), lds, nullptr)
                                     : lffn_host::gather_lds_probes_part(tok, ga, fr, sw, dim3(1), lds, nullptr);
                    if (rc != LFFN_OK && rc != LFFN_E_UNSUPPORTED) return rc;
                }
            }
    rc = lffn_host::hash_row16_load();
    if (rc != LFFN_OK) return rc;
    rc = lffn_host::hash_row8_load();
    if (rc != LFFN_OK) return rc;
    rc = lffn_host::forward_stack_load();
    if (rc != LFFN_OK) return rc;
    rc = lffn_host::bh_lane_load();
    if (rc != LFFN_OK) return rc;
    rc = lffn_host::hash_lane_load();
    if (rc != LFFN_OK) return rc;
    {
        GatherRingArgs ra{};
        for (int threads : {512, 1024})
            for (int tok = 1; tok <= 32; ++tok) {
                rc = lffn_host::gather_ring_part(threads, tok, ra, dim3(1), nullptr);
                if (rc != LFFN_OK && rc != LFFN_E_UNSUPPORTED) return rc;
            }
    }
    for (int wmode = 0; wmode < 3; ++wmode) {
        rc = lffn_host::bh_few_part(wmode, ba, dim3(1), nullptr);
        if (rc != LFFN_OK) return rc;
    }
    for (int block : {16, 32, 64})
        for (int wmode = 0; wmode < 3; ++wmode) {
            for (int L = 6; L <= 8; ++L) {
                rc = lffn_host::bh_lo_part(L, wmode, ba, block, dim3(1), nullptr);
                if (rc != LFFN_OK) return rc;
            }
            for (auto part : {lffn_host::bh_512_part, lffn_host::bh_1024_part}) {
                rc = part(wmode, ba, block, dim3(1), nullptr);
                if (rc != LFFN_OK) return rc;
            }
        }
    return LFFN_OK;
}

int lookupffn_hash(const void *x, const int8_t *signs, uint16_t *codes, int64_t n_tokens, int d, int k,
                   int tau, int n_rounds, int x_dtype, void *hip_stream)
{
    int rc = check_hash(x, signs, codes, n_tokens, d, k, tau, n_rounds, x_dtype);
    if (rc != LFFN_OK || n_tokens == 0) return rc;
    HashOut out;
    out.codes = codes;
    return launch_hash(x, signs, out, n_tokens, d, k, tau, n_rounds, x_dtype, false, static_cast<hipStream_t>(hip_stream),
                       options_snapshot());
}

int lookupffn_hash_weighted(const void *x, const int8_t *signs, uint16_t *codes, float *weights, int64_t n_tokens,
                            int d, int k, int tau, int n_rounds, int x_dtype, void *hip_stream)
{
    int rc = check_hash(x, signs, codes, n_tokens, d, k, tau, n_rounds, x_dtype, true);
    if (rc == LFFN_OK) rc = check_weights(weights);
    if (rc != LFFN_OK || n_tokens == 0) return rc;
    HashOut out;
    out.codes = codes;
    out.weights = weights;
    return launch_hash(x, signs, out, n_tokens, d, k, tau, n_rounds, x_dtype, false, static_cast<hipStream_t>(hip_stream),
                       options_snapshot());
}

int lookupffn_hash_probes(const void *x, const int8_t *signs, uint16_t *codes, float *shares, int64_t n_tokens,
                          int d, int k, int tau, int n_rounds, int x_dtype, void *hip_stream)
{
    int rc = check_hash(x, signs, codes, n_tokens, d, k, tau, n_rounds, x_dtype, true);
    if (rc == LFFN_OK) rc = check_weights(shares);
    if (rc != LFFN_OK || n_tokens == 0) return rc;
    HashOut out;
    out.codes = codes;
    out.weights = shares;
    out.probes = true;
    return launch_hash(x, signs, out, n_tokens, d, k, tau, n_rounds, x_dtype, false, static_cast<hipStream_t>(hip_stream),
                       options_snapshot());
}

int lookupffn_gather(const uint16_t *codes, const void *tables, void *y, int64_t n_tokens, int k, int tau,
                     int d_out, int table_dtype, void *workspace, int64_t workspace_bytes, void *hip_stream)
{
    return gather_core(kPlain, codes, nullptr, tables, y, n_tokens, k, tau, d_out, table_dtype, workspace,
                       workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

int lookupffn_gather_weighted(const uint16_t *codes, const float *weights, const void *tables, void *y,
                              int64_t n_tokens, int k, int tau, int d_out, int table_dtype, void *workspace,
                              int64_t workspace_bytes, void *hip_stream)
{
    return gather_core(kWeighted, codes, weights, tables, y, n_tokens, k, tau, d_out, table_dtype, workspace,
                       workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

int lookupffn_gather_probes(const uint16_t *codes, const float *shares, const void *tables, void *y,
                            int64_t n_tokens, int k, int tau, int d_out, int table_dtype, void *workspace,
                            int64_t workspace_bytes, void *hip_stream)
{
    return gather_core(kProbes, codes, shares, tables, y, n_tokens, k, tau, d_out, table_dtype, workspace,
                       workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

int64_t lookupffn_workspace_bytes_gather(int64_t n_tokens, int k)
{
    return (n_tokens <= 0 || k < 1) ? 0 : gather_ws_bytes(n_tokens, k, 1, kPlain);
}
int64_t lookupffn_workspace_bytes_gather_weighted(int64_t n_tokens, int k)
{
    return (n_tokens <= 0 || k < 1) ? 0 : gather_ws_bytes(n_tokens, k, 1, kWeighted);
}
int64_t lookupffn_workspace_bytes_gather_probes(int64_t n_tokens, int k, int tau)
{
    return (n_tokens <= 0 || k < 1 || tau < 1 || tau > 16) ? 0 : gather_ws_bytes(n_tokens, k, tau, kProbes);
}

int64_t lookupffn_workspace_bytes(int64_t n_tokens, int k)
{
    return (n_tokens <= 0 || k < 1) ? 0 : forward_ws_bytes(n_tokens, k, 1, kPlain);
}
int64_t lookupffn_workspace_bytes_weighted(int64_t n_tokens, int k)
{
    return (n_tokens <= 0 || k < 1) ? 0 : forward_ws_bytes(n_tokens, k, 1, kWeighted);
}
int64_t lookupffn_workspace_bytes_probes(int64_t n_tokens, int k, int tau)
{
    return (n_tokens <= 0 || k < 1 || tau < 1 || tau > 16) ? 0 : forward_ws_bytes(n_tokens, k, tau, kProbes);
}
int64_t lookupffn_workspace_bytes_bh(int64_t n_tokens, int d, int k, int tau, int block, int n_factors)
{
    if (!bh_shape_ok(d, k, tau, block & ~LFFN_PREPARED, n_factors)) return 0;
    const int64_t pack = (block & LFFN_PREPARED) ? 0 : bh_pack_bytes(d, k, tau, block, n_factors);
    return sat_add(pack, n_tokens > 0 ? forward_ws_bytes(n_tokens, k, tau, kPlain) : 0);
}
int64_t lookupffn_workspace_bytes_bh_weighted(int64_t n_tokens, int d, int k, int tau, int block, int n_factors)
{
    if (!bh_shape_ok(d, k, tau, block & ~LFFN_PREPARED, n_factors)) return 0;
    const int64_t pack = (block & LFFN_PREPARED) ? 0 : bh_pack_bytes(d, k, tau, block, n_factors);
    return sat_add(pack, n_tokens > 0 ? forward_ws_bytes(n_tokens, k, tau, kWeighted) : 0);
}

int lookupffn_forward(const void *x, const int8_t *signs, const void *tables, void *y, int64_t n_tokens,
                      int d, int k, int tau, int d_out, int n_rounds, int x_dtype, int table_dtype,
                      void *workspace, int64_t workspace_bytes, void *hip_stream)
{
    return forward_core(sign_hash(signs, n_rounds), kPlain, x, tables, y, n_tokens, d, k, tau, d_out, x_dtype,
                        table_dtype, workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

int lookupffn_forward_stack(const void *x, const int8_t *const *signs, const void *const *tables, void *y,
                            int64_t n_tokens, int d, int k, int tau, int d_out, int n_rounds, int n_layers,
                            int x_dtype, int table_dtype, void *hip_stream)
{
    if (!signs || !tables) return LFFN_E_NULL;
    if (n_layers < 1 || n_layers > kStackMaxLayers) return LFFN_E_SIZE;
    const uint16_t *stand_in = reinterpret_cast<const uint16_t *>(uintptr_t(256));  // no codes leave the kernel
    for (int l = 0; l < n_layers; ++l) {
        int rc = check_hash(x, signs[l], stand_in, n_tokens, d, k, tau, n_rounds, x_dtype);
        if (rc == LFFN_OK) rc = check_gather(stand_in, tables[l], y, n_tokens, k, tau, d_out, table_dtype);
        if (rc != LFFN_OK) return rc;
    }
    if (n_layers > 1 && d_out != d) return LFFN_E_SIZE;
    if (!stack_shape_ok(x, signs, tables, n_layers, n_tokens, d, k, tau, d_out, n_rounds, x_dtype, table_dtype))
        return LFFN_E_UNSUPPORTED;
    if (n_tokens == 0) return LFFN_OK;
    return launch_forward_stack(x, signs, tables, y, n_tokens, d, k, tau, d_out, n_rounds, n_layers, x_dtype,
                                table_dtype, static_cast<hipStream_t>(hip_stream));
}

int64_t lookupffn_static_scratch_bytes(void) { return kStaticScratchBytes; }

int lookupffn_forward_static(const void *x, const int8_t *signs, const void *tables, void *y, int64_t n_tokens,
                             int d, int k, int tau, int d_out, int n_rounds, int x_dtype, int table_dtype,
                             void *hip_stream)
{
    // sizes first (no HIP call yet): a batch whose intermediates do not fit the static array is refused
    if (n_tokens > 0 && k >= 1 && tau >= 1 && tau <= 16 && n_tokens <= (int64_t(1) << 40) && k <= (1 << 20) &&
        forward_ws_bytes(n_tokens, k, tau, kPlain) > kStaticScratchBytes)
        return LFFN_E_WORKSPACE;
    void *ws = reinterpret_cast<void *>(uintptr_t(256));  // stand-in until the arguments have been checked
    if (n_tokens > 0 && x && signs && tables && y) {
        int rc = static_scratch(&ws);
        if (rc != LFFN_OK) return rc;
    }
    return forward_core(sign_hash(signs, n_rounds), kPlain, x, tables, y, n_tokens, d, k, tau, d_out, x_dtype,
                        table_dtype, ws, kStaticScratchBytes, static_cast<hipStream_t>(hip_stream));
}

int lookupffn_forward_weighted(const void *x, const int8_t *signs, const void *tables, void *y, int64_t n_tokens,
                               int d, int k, int tau, int d_out, int n_rounds, int x_dtype, int table_dtype,
                               void *workspace, int64_t workspace_bytes, void *hip_stream)
{
    return forward_core(sign_hash(signs, n_rounds), kWeighted, x, tables, y, n_tokens, d, k, tau, d_out, x_dtype,
                        table_dtype, workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

int lookupffn_forward_probes(const void *x, const int8_t *signs, const void *tables, void *y, int64_t n_tokens,
                             int d, int k, int tau, int d_out, int n_rounds, int x_dtype, int table_dtype,
                             void *workspace, int64_t workspace_bytes, void *hip_stream)
{
    return forward_core(sign_hash(signs, n_rounds), kProbes, x, tables, y, n_tokens, d, k, tau, d_out, x_dtype,
                        table_dtype, workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

int lookupffn_hash_bh(const void *x, const float *bmats, uint16_t *codes, int64_t n_tokens, int d, int k, int tau,
                      int block, int n_factors, int x_dtype, void *workspace, int64_t workspace_bytes,
                      void *hip_stream)
{
    return hash_bh_core(x, bmats, codes, nullptr, false, n_tokens, d, k, tau, block, n_factors, x_dtype, workspace,
                        workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

int lookupffn_hash_bh_weighted(const void *x, const float *bmats, uint16_t *codes, float *weights, int64_t n_tokens,
                               int d, int k, int tau, int block, int n_factors, int x_dtype, void *workspace,
                               int64_t workspace_bytes, void *hip_stream)
{
    if (!weights) return (x && bmats && codes) ? LFFN_E_NULL : LFFN_E_NULL;
    return hash_bh_core(x, bmats, codes, weights, true, n_tokens, d, k, tau, block, n_factors, x_dtype, workspace,
                        workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

int lookupffn_forward_bh(const void *x, const float *bmats, const void *tables, void *y, int64_t n_tokens, int d,
                         int k, int tau, int d_out, int block, int n_factors, int x_dtype, int table_dtype,
                         void *workspace, int64_t workspace_bytes, void *hip_stream)
{
    return forward_core(bh_hash(bmats, block, n_factors), kPlain, x, tables, y, n_tokens, d, k, tau, d_out, x_dtype,
                        table_dtype, workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

int lookupffn_forward_bh_weighted(const void *x, const float *bmats, const void *tables, void *y, int64_t n_tokens,
                                  int d, int k, int tau, int d_out, int block, int n_factors, int x_dtype,
                                  int table_dtype, void *workspace, int64_t workspace_bytes, void *hip_stream)
{
    return forward_core(bh_hash(bmats, block, n_factors), kWeighted, x, tables, y, n_tokens, d, k, tau, d_out,
                        x_dtype, table_dtype, workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

// ---- one-time preparation of the learned constants ------------------------------------------------
int64_t lookupffn_prepared_tables_bytes(int k, int tau, int d_out, int table_dtype)
{
    if (k < 1 || tau < 1 || tau > 16 || d_out < 1 || !dtype_ok(table_dtype)) return 0;
    if (d_out % (table_dtype == LFFN_F32 ? 4 : 8) != 0 || ((int64_t)k << tau) > (int64_t(1) << 31)) return 0;
    return prepared_tables_bytes(k, tau, d_out);
}

int lookupffn_prepare_tables(const void *tables, int k, int tau, int d_out, int table_dtype, void *prepared,
                             int64_t prepared_bytes, void *hip_stream)
{
    if (!tables || !prepared) return LFFN_E_NULL;
    if (k < 1 || d_out < 1 || k > (1 << 20) || d_out > (1 << 24)) return LFFN_E_SIZE;
    if (tau < 1 || tau > 16) return LFFN_E_TAU;
    if (!dtype_ok(table_dtype)) return LFFN_E_DTYPE;
    if (d_out % (table_dtype == LFFN_F32 ? 4 : 8) != 0) return LFFN_E_ALIGN;
    if (((int64_t)k << tau) > (int64_t(1) << 31)) return LFFN_E_SIZE;
    if (!aligned(tables, 16) || !aligned(prepared, 256)) return LFFN_E_ALIGN;
    const int64_t need = prepared_tables_bytes(k, tau, d_out);
    if (prepared_bytes < need) return LFFN_E_WORKSPACE;
    const int pw = prepared_piece_bytes(tau), ppw = pw / 16;
    const int rows = 1 << tau, nvec = d_out / 4;
    const long long n_ps = (nvec + ppw - 1) / ppw;
    const long long n_out = n_ps * k * rows * ppw;
    long long blocks = (n_out + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(prepare_tables_kernel, dim3((unsigned)blocks), dim3(256), 0, static_cast<hipStream_t>(hip_stream),
                       tables, static_cast<uint4 *>(prepared), k, rows, nvec, ppw, table_dtype, n_out);
    LFFN_HIP(hipGetLastError());
    return LFFN_OK;
}

int64_t lookupffn_prepared_bh_bytes(int d, int k, int tau, int block, int n_factors)
{
    if (!bh_shape_ok(d, k, tau, block, n_factors) || (block != 16 && block != 32 && block != 64)) return 0;
    return bh_pack_bytes(d, k, tau, block, n_factors);
}

int lookupffn_prepare_bh(const float *bmats, int d, int k, int tau, int block, int n_factors, void *prepared,
                         int64_t prepared_bytes, void *hip_stream)
{
    if (!prepared) return LFFN_E_NULL;
    const float *stand_in_x = reinterpret_cast<const float *>(uintptr_t(256));
    int rc = check_bh(stand_in_x, bmats, 0, d, k, tau, block, n_factors, LFFN_F32);
    if (rc != LFFN_OK) return rc;
    if (!aligned(prepared, 256)) return LFFN_E_ALIGN;
    if (prepared_bytes < bh_pack_bytes(d, k, tau, block, n_factors)) return LFFN_E_WORKSPACE;
    return launch_bh_pack(bmats, static_cast<float *>(prepared), d, k, tau, block, n_factors,
                          static_cast<hipStream_t>(hip_stream));
}

int lookupffn_release_workspace(void)
{
    std::lock_guard<std::mutex> lk(g_ws_mu);
    int rc = LFFN_OK;
    int cur = 0;
    const bool have_cur = hipGetDevice(&cur) == hipSuccess;
    for (auto &kv : g_ws) {
        if (!kv.second.ptr && kv.second.retired.empty()) continue;
        if (hipSetDevice(kv.first) != hipSuccess || hipDeviceSynchronize() != hipSuccess) rc = LFFN_E_HIP;
        if (kv.second.ptr && hipFree(kv.second.ptr) != hipSuccess) rc = LFFN_E_HIP;
        for (void *p : kv.second.retired)
            if (hipFree(p) != hipSuccess) rc = LFFN_E_HIP;
        kv.second = Workspace();
    }
    if (have_cur) (void)hipSetDevice(cur);
    g_ws.clear();
    return rc;
}

int lookupffn_timing_enable(int mask)
{
    if (mask < 0 || mask > 3) return LFFN_E_SIZE;
    g_tm.on.store(mask);
    return LFFN_OK;
}

int lookupffn_timing_reset(void)
{
    std::lock_guard<std::mutex> lk(g_tm.mu);
    for (auto &v : g_tm.ev) {
        for (auto &p : v) {
            (void)hipEventSynchronize(p.second);
            g_tm.pool.push_back(p);
        }
        v.clear();
    }
    return LFFN_OK;
}

int lookupffn_timing_read(int which, double *total_ms, int64_t *launches)
{
    if (which < 0 || which > 1) return LFFN_E_SIZE;
    if (!total_ms || !launches) return LFFN_E_NULL;
    std::lock_guard<std::mutex> lk(g_tm.mu);
    double sum = 0.0;
    for (auto &p : g_tm.ev[which]) {
        LFFN_HIP(hipEventSynchronize(p.second));
        float ms = 0.0f;
        LFFN_HIP(hipEventElapsedTime(&ms, p.first, p.second));
        sum += ms;
    }
    *total_ms = sum;
    *launches = (int64_t)g_tm.ev[which].size();
    return LFFN_OK;
}

int lookupffn_timing_read_each(int which, double *ms_out, int64_t capacity, int64_t *launches)
{
    if (which < 0 || which > 1 || capacity < 0) return LFFN_E_SIZE;
    if (!launches || (capacity > 0 && !ms_out)) return LFFN_E_NULL;
    std::lock_guard<std::mutex> lk(g_tm.mu);
    int64_t i = 0;
    for (auto &p : g_tm.ev[which]) {
        if (i >= capacity) break;
        LFFN_HIP(hipEventSynchronize(p.second));
        float ms = 0.0f;
        LFFN_HIP(hipEventElapsedTime(&ms, p.first, p.second));
        ms_out[i++] = ms;
    }
    *launches = (int64_t)g_tm.ev[which].size();
    return LFFN_OK;
}

int lookupffn_set_option(const char *key, int value)
{
    if (!key) return LFFN_E_NULL;
    std::lock_guard<std::mutex> lk(g_opt_mu);
    if (!std::strcmp(key, "lanes_per_token")) {
        if (value != 0 && (value < 1 || value > 64 || (value & (value - 1)))) return LFFN_E_SIZE;
        g_opt.lanes_per_token = value;
        return LFFN_OK;
    }
    if (!std::strcmp(key, "hash_path")) {
        if (value < 0 || value > 3) return LFFN_E_SIZE;
        g_opt.hash_path = value;
        return LFFN_OK;
    }
    if (!std::strcmp(key, "hash_blocks")) {
        if (value < 0 || value > 65536) return LFFN_E_SIZE;
        g_opt.hash_blocks = value;
        return LFFN_OK;
    }
    if (!std::strcmp(key, "slice_lanes")) {
        if (value != 0 && value != 4 && value != 8) return LFFN_E_SIZE;
        g_opt.slice_lanes = value;
        return LFFN_OK;
    }
    if (!std::strcmp(key, "ring_threads")) {
        if (value != 0 && value != 512 && value != 1024) return LFFN_E_SIZE;
        g_opt.ring_threads = value;
        return LFFN_OK;
    }
    if (!std::strcmp(key, "small_tokens")) {
        if (value < -1 || value > (1 << 20)) return LFFN_E_SIZE;
        g_opt.small_tokens = value;
        return LFFN_OK;
    }
    if (!std::strcmp(key, "token_slots")) {
        if (value < 0 || value > 32) return LFFN_E_SIZE;
        g_opt.token_slots = value;
        return LFFN_OK;
    }
    if (!std::strcmp(key, "gather_path")) {
        if (value < 0 || value > 4) return LFFN_E_SIZE;
        g_opt.gather_path = value;
        return LFFN_OK;
    }
    if (!std::strcmp(key, "xcd_order")) {
        if (value < -1 || value > 1) return LFFN_E_SIZE;
        g_opt.xcd_order = value;
        return LFFN_OK;
    }
    return LFFN_E_SIZE;
}

const char *lookupffn_strerror(int status)
{
    switch (status) {
        case LFFN_OK: return "success";
        case LFFN_E_NULL: return "a required pointer is NULL";
        case LFFN_E_SIZE: return "a size argument is out of range";
        case LFFN_E_TAU: return "tau must be in [1, 16]";
        case LFFN_E_DTYPE: return "unknown dtype";
        case LFFN_E_ALIGN: return "pointer alignment or d_out granularity not met";
        case LFFN_E_UNSUPPORTED: return "shape not supported by this entry point";
        case LFFN_E_WORKSPACE: return "workspace or output buffer too small";
        case LFFN_E_HIP: return "a HIP call failed";
        default: return "unknown status";
    }
}

const char *lookupffn_last_hip_error(void) { return g_hip_error.c_str(); }

const char *lookupffn_last_gather_kernel(void) { return t_last_gather; }
const char *lookupffn_last_hash_kernel(void) { return t_last_hash; }

int lookupffn_version(void) { return kVersion; }

}  // extern "C"

#endif  // LFFN_HAS(0)
