// Helper workgroups of the GEMM kernels: they fetch operands into a cache ahead of the workgroups
// that work on tiles.
#pragma once

#include <atomic>

#include "tw_mfma.h"

namespace tw {

// Helpers: workgroups on the compute units that got no tile fetch what their XCD's tiles read into
// its L2, ahead of them. A compute unit gets its lines back in the order it asked for them, so
// among lines that come from the L2 every one that comes from HBM holds up all behind it: what the
// weights cost is not their share of the requests but HBM's latency for all of them (a panel
// shared by seven compute units of an XCD comes in at 60 GB/s a unit from HBM and at 105 from the
// caches). Touching lines ahead from the compute units that work on tiles costs the requests it
// saves; from others it is free. us before there were helpers / now, operands from HBM and from the cache: [16 x 8192] x
// [8192 x 1280] 11.6 / 10.0 and 10.6 / 9.2, [64 x 8192] x [8192 x 1280] 14.7 / 11.1 and 11.5 / 10.2; [K x N], whose rows of
// a narrow tile are less than a line: [16 x 4096] x [4096 x 4096] 19.3 / 10.4 and 11.5 / 9.4, [128 x 8192] x [8192 x 2048]
// 34.5 / 19.1 and 21.4 / 19.0. In the counters the same bytes come from beyond the L2 with helpers and without; L2 hits
// and the latency of a request, [16 x 8192] x [8192 x 1280] 46 -> 65 % and 446 -> 292 clocks, [16 x 4096] x [4096 x 4096]
// 59 -> 71 % and 660 -> 509.
//
// They keep `lead` windows (kHelpWindow bytes of K) ahead of a window every `pace` ticks of the
// 100 MHz clock: further ahead they would push out of the 4 MiB what the tiles have yet to read. What the tiles fall
// behind the clock comes on top and grows with K: the clock is a little slower than the tiles are expected to be
// (kHelpPace), and the lead gets smaller by a tenth (kHelpLag) of all that the XCD reads, from kHelpLeadMost to
// kHelpLeadLeast. us with 1.5 MB and 1.15 throughout / so, operands from the cache: [64 x 28672] x [28672 x 4096], stored
// [K x N], 103 / 60 (78 without helpers), [52 x 23680] x [23680 x 3072] 78 / 55 (62), [182 x 17536] x [17536 x 3072],
// [N x K], 53 / 48 (49). 131 sizes with K from 2048 to 10000 against 1.5 MB and 1.15, from the cache and from HBM: 0.998
// and 0.999, 47 with up to 32768 0.951 and 0.981. (0.6 MB throughout: the same, but 7 % slower for [329 x 4816] x
// [4816 x 776]; 0.9 MB 0.998 and 0.998, 0.968 and 0.995; a clock of 0.9, for which the tiles are too slow, or of 1.25:
// level, and 2 to 7 % slower where K is large.)
//
// Where the XCD's share is more than its idle units can fetch, the helpers of all XCDs fetch every
// operand once, for the last-level cache, and keep no pace (ALL).
//
// With kernels of other streams on the device helpers may start when the tiles are done: they must not
// keep the launch from ending (three streams of [2048 x 8192] x [8192 x 3584] took 367 us for a product each, 322
// without helpers and 327 as it is). Workgroup 0, which is dispatched before them, leaves the time it began in a word of the
// launch's own; helpers look there every kHelpLookTicks (not at once: the time may still be that of an earlier
// launch with the word) and leave when the launch's expected time is over. Should two launches with
// the same word ever overlap, some helpers leave early or late; nothing else depends on it.
static constexpr uint32_t kHelpWindow = 1024;
static constexpr uint32_t kHelpWords = 128, kHelpLookTicks = 300;
static __device__ uint32_t tiles_begun[kHelpWords];
// The argument of a launch with helpers: the launch's word (bits 0 to 6), ticks of a window (11 bits) and of
// the lead (13 bits); where the helpers fetch everything, word and expected ticks.
inline uint32_t next_help_word()
{
    static std::atomic<uint32_t> launches{0};
    return launches.fetch_add(1, std::memory_order_relaxed) % kHelpWords;
}
inline uint32_t pack_help(double pace, double lead_ticks)
{
    return static_cast<uint32_t>(pace < 2047.0 ? pace : 2047.0) << 7 |
           static_cast<uint32_t>(lead_ticks < 8191.0 ? lead_ticks : 8191.0) << 18;
}
inline uint32_t pack_help_all(double us) { return static_cast<uint32_t>(us < 160e3 ? us * 100 : 16e6) << 7; }
// By the workgroups with a tile, once
__device__ __forceinline__ void say_begun(uint32_t help)
{
    if (blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(&tiles_begun[help % kHelpWords], static_cast<uint32_t>(__builtin_amdgcn_s_memrealtime()),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
static constexpr double kHelpLeadMost = 1.5e6, kHelpLeadLeast = 0.6e6, kHelpLag = 0.1, kHelpPace = 1.05;
static constexpr double kHelperBytesPerUs = 50e3, kHbmBytesPerUs = 5.3e6;
static constexpr int64_t kHelpFromK = 2048;
// Weights of at least this many bytes are taken to come from HBM: the last-level cache holds 256 MiB, and
// a model's other weights pass through it between two uses of one.
static constexpr int64_t kFromHbmBytes = int64_t(32) << 20;
// What an XCD's tiles, [first, first + count) of the list, read: rows [a_lo, a_hi) of A, and columns
// [c_lo, c_lo + n1) and [0, n2) of B (two runs where its tiles lie in two blocks of tile rows).
struct Operands {
    uint32_t a_lo, a_hi, c_lo, n1, n2;
};
__host__ __device__ inline Operands operands_of(uint32_t first, uint32_t count, uint32_t M, uint32_t N, uint32_t tiles_m,
                                                uint32_t tiles_n, uint32_t group_m, uint32_t BM, uint32_t BN)
{
    const uint32_t tiles = tiles_m * tiles_n;
    if (first >= tiles) return {0, 0, 0, 0, 0};
    const uint32_t last = (first + count < tiles ? first + count : tiles) - 1, per_block = group_m * tiles_n;
    const uint32_t b0 = first / per_block, b1 = last / per_block;
    const auto least = [](uint32_t a, uint32_t b) { return a < b ? a : b; };
    const auto column = [&](uint32_t tile, uint32_t b) { return (tile - b * per_block) / least(group_m, tiles_m - b * group_m); };
    const uint32_t c0 = column(first, b0), c1 = column(last, b1);
    const uint32_t end1 = least((b0 == b1 ? c1 + 1 : tiles_n) * BN, N);
    return {b0 * group_m * BM, least((b1 + 1) * group_m * BM, M), c0 * BN, end1 - c0 * BN,
            b0 == b1 ? 0 : b1 == b0 + 1 ? least((c1 + 1) * BN, N) : N};
}
// One of n_helpers workgroups (of an XCD; ALL: of the launch) of WAVES waves. A wave's load asks for 64 lines, a dword of each.
template <bool B_KN, bool ALL, uint32_t WAVES>
__device__ __forceinline__ void fetch_ahead(const char *A, const char *B, uint32_t N, uint32_t K, const Operands o,
                                            uint32_t helper, uint32_t n_helpers, uint32_t help)
{
    const uint32_t pace = ALL ? 0 : help >> 7 & 0x7ff, lead_ticks = ALL ? 0 : help >> 18 & 0x1fff;
    const int64_t begun = __builtin_amdgcn_s_memrealtime();
    int64_t look = begun + kHelpLookTicks;
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t row_bytes = K * 2, windows = (row_bytes + kHelpWindow - 1) / kHelpWindow;
    const uint32_t expected = ALL ? help >> 7 : pace * windows;
    constexpr uint32_t kRunLines = kHelpWindow / 128, kRows = 64 / kRunLines;  // a load: eight rows of a window
    // B stored [K x N]: a window is kHelpWindow / 2 rows of B, of which a run of columns takes some lines each
    const uint32_t kn_lines1 = (o.n1 * 2 + 127) / 128, kn_lines = kn_lines1 + (o.n2 * 2 + 127) / 128;
    const uint32_t a_loads = (o.a_hi - o.a_lo + kRows - 1) / kRows;
    const uint32_t b_loads = B_KN ? kHelpWindow / 2 * kn_lines / 64 : (o.n1 + o.n2 + kRows - 1) / kRows;
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(A, o.a_hi * row_bytes), rb = make_rsrc(B, K * N * 2);
    for (uint32_t i = wave * n_helpers + helper; i < windows * (a_loads + b_loads); i += WAVES * n_helpers) {
        const uint32_t window = i / (a_loads + b_loads), l = i - window * (a_loads + b_loads);
        int64_t now = __builtin_amdgcn_s_memrealtime();
        if constexpr (!ALL) {
            const int64_t not_before = begun + static_cast<int64_t>(window) * pace - lead_ticks;
            for (; now < not_before; now = __builtin_amdgcn_s_memrealtime()) __builtin_amdgcn_s_sleep(2);
        }
        if (now >= look) {
            if (static_cast<uint32_t>(now) - __hip_atomic_load(&tiles_begun[help % kHelpWords], __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT) > expected)
                return;
            look = now + kHelpLookTicks;
        }
        const uint32_t in_row = window * kHelpWindow + lane % kRunLines * 128;
        uint32_t v;
        if (l < a_loads) {
            const uint32_t row = o.a_lo + l * kRows + lane / kRunLines;
            v = __builtin_amdgcn_raw_buffer_load_b32(ra, in_row < row_bytes ? row * row_bytes + in_row : kOutOfRange, 0, 0);
        } else if constexpr (!B_KN) {
            const uint32_t at = (l - a_loads) * kRows + lane / kRunLines, row = at < o.n1 ? o.c_lo + at : at - o.n1;
            v = __builtin_amdgcn_raw_buffer_load_b32(rb, in_row < row_bytes ? row * row_bytes + in_row : kOutOfRange, 0, 0);
        } else {
            const uint32_t at = (l - a_loads) * 64 + lane, k = at / kn_lines, line = at - k * kn_lines;
            const uint32_t column = line < kn_lines1 ? o.c_lo * 2 + line * 128 : (line - kn_lines1) * 128;
            v = __builtin_amdgcn_raw_buffer_load_b32(rb, (window * (kHelpWindow / 2) + k) * (N * 2) + column, 0, 0);
        }
        asm volatile("" ::"v"(v));
    }
}

// What workgroup `slots` + i of a launch of `slots` workgroups for tiles and some helpers does.
template <bool B_KN, bool ALL, uint32_t WAVES>
__device__ __forceinline__ void help_tiles(const char *A, const char *B, uint32_t M, uint32_t N, uint32_t K, uint32_t tiles_m,
                                           uint32_t tiles_n, uint32_t group_m, uint32_t tiles_per_xcd, uint32_t BM, uint32_t BN,
                                           uint32_t help)
{
    const uint32_t slots = tiles_per_xcd * kXcds;
    if constexpr (ALL) {
        fetch_ahead<B_KN, ALL, WAVES>(A, B, N, K, {0, M, 0, N, 0}, blockIdx.x - slots, gridDim.x - slots, help);
    } else {
        const Operands o = operands_of(blockIdx.x % kXcds * tiles_per_xcd, tiles_per_xcd, M, N, tiles_m, tiles_n, group_m, BM, BN);
        fetch_ahead<B_KN, ALL, WAVES>(A, B, N, K, o, blockIdx.x / kXcds - tiles_per_xcd, gridDim.x / kXcds - tiles_per_xcd, help);
    }
}

}  // namespace tw
