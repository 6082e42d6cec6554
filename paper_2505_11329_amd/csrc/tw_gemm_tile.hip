// bf16 GEMM on small output tiles, for products that the 256-row tiles of
// tw_gemm.hip cannot spread over the device: decode steps (a few rows: the weights
// are read once and that is all the work) and batches of up to a thousand rows or
// so. Same product, same bits: every output is the chain of its K / 32 partial dot
// products (v_mfma_f32_16x16x32_bf16) in the order of increasing k, so K is never
// split, and parallelism comes from the tile shape alone.
//
// What bounds it: what a compute unit can pull into its LDS. Whatever the tile, a
// compute unit takes in 64 to 72 GB/s of operands (90 to 100 requests, 11 to 13 KB,
// in flight, 370 to 420 clocks each, four fifths of them L2 hits; with the weights
// from HBM 43 GB/s over a launch of 12 us), so a tile of BM x BN outputs costs (BM +
// BN) * K * 2 bytes of that, and the best shape is the smallest that still gives
// every compute unit at most one tile. A kernel with the LDS reads and matrix
// instructions taken out ran within 4 to 13 % of the whole. Tried and not kept:
// fetching lines into the L2 ahead of time, each workgroup a share of the panels its
// XCD reads (3 to 20 % slower); rotating the order in which the workgroups of an XCD
// ask for a shared panel's rows (nothing at these sizes).
//
// Measured on MI355X, weights from HBM, us (the 256-row tiles before / these tiles
// without helpers and the rolling K loop / the vendor library): [16 x 8192] x [8192 x
// 3584] 64 / 13.1 / 20 (59 MB of weights: 4.5 TB/s), [16 x 8192] x [8192 x 1280] 46 /
// 11.5 / 20 (with both, on another box, 8.2), [64 x 8192] x [8192 x 3584] 64 / 20.6 / 24,
// [333 x 8192] x [8192 x 3584] 65 / 37 / 45, [512 x 8192] x [8192 x 1280] 73 / 33 / 32.
//
// Shape of a workgroup: WVM x WVN waves own WM x WN blocks of 16 x 16 each; tiles of
// one or two blocks still get four waves, which share the loading. S stages of BK deep
// K steps sit in LDS, filled by 16-byte global-to-LDS loads. Step s: the fragments of
// stage s are in registers; once every wave has them and stage s + 1 has landed (one
// vmcnt wait and one barrier), the stage's LDS takes the loads of step s + S, and the
// reads of stage s + 1's fragments go out between the matrix instructions of stage s
// (15.2 -> 13.7 us at 16 rows against reads first). Waves of a single block, one chain of
// dependent matrix instructions, have a K loop of their own that never waits for all of its
// reads (ROLLS; what bounded those tiles was that chain: 480 clocks for 256 of K, of which
// the matrix instructions take 180 and the loads of a 16 x 16 tile 290, now 300).
// Rows are laid out as in tw_gemm.hip: 16-byte pieces xor-swizzled so that a fragment
// read touches every bank once.
#include <algorithm>
#include <atomic>

#include "tw_help.h"
#include "tw_internal.h"
#include "tw_mfma.h"

namespace tw {

// Waves that only load, beside the ones that multiply (LOADERS). A multiplying wave that also
// loads has the address arithmetic and the loads of a step in the way of its matrix
// instructions, which for a small tile are a chain with one wave to a SIMD: a step of 256 in K of a
// 16 x 16 tile took 600 clocks even with everything in the L2. With waves for each, us, operands from
// the cache / from HBM: [16 x 8192] x [8192 x 1280] 10.5 -> 8.9 / 11.2 -> 10.8; [64 x 8192] x [8192 x 3584]
// (32 x 32) 15.6 -> 14.2 / 21.3 -> 21.2; [K x N]: [1000 x 4096] x [4096 x 3000] (128 x 128) 33.4 -> 30.0. The
// workgroups start later, with twice the waves: 1 to 5 % slower where K is short (see kSmallTiles).
static constexpr int kLoaders = 4;

template <int WM, int WN, int WVM, int WVN, int BK, int S, bool LOADERS>
struct SmallTile {
    static constexpr int kCompute = WVM * WVN;                                          // waves that own outputs
    static constexpr int kWaves = LOADERS ? kLoaders : kCompute < 4 ? 4 : kCompute;      // waves that load
    static constexpr int kThreads = 64 * (LOADERS ? kCompute + kLoaders : kWaves);
    static constexpr int BM = kBlk * WM * WVM, BN = kBlk * WN * WVN;
    static constexpr int kABytes = BM * BK * 2, kBBytes = BN * BK * 2, kStageBytes = kABytes + kBBytes;
    static constexpr int kLdsBytes = S * kStageBytes;
    static constexpr int kALoads = kABytes / 1024 / kWaves, kBLoads = kBBytes / 1024 / kWaves;
    static constexpr int kLoads = kALoads + kBLoads;  // per wave and stage, 1 KiB each
    static_assert(kABytes % (1024 * kWaves) == 0 && kBBytes % (1024 * kWaves) == 0, "whole load instructions");
    static_assert((S - 1) * kLoads < 64, "vmcnt field");
    static_assert(S >= 3 && kLdsBytes <= 160 * 1024, "LDS of one compute unit");
    static_assert(BK == 64 || BK == 128 || BK == 256, "LDS layouts below");
    static constexpr bool kStagedStores = WN == 2 || WN == 4;
    // Whether the last S steps are compiled without loads. Past the end of K there is nothing to
    // load, and an out-of-range load takes its turn in the L1's queue like any other: 16 rows,
    // K = 3584, N = 8192 12.4 -> 12.1 us, 333 rows, K = 8192, N = 3584 38.2 -> 37.5. With three
    // stages there is little to save, and 192 x 128 tiles came out 1 to 3 % slower.
    static constexpr bool kTail = S > 3;
    static_assert(!LOADERS || kTail, "loading waves load nothing past the end of K");
};

// Which shapes have the rolling K loop (see there): those whose waves have one block each, of [K x N] weights with loading
// waves only (short K: 5 % slower). Some short K take the other loop all the same (kShortK).
template <bool B_KN, int WM, int WN, bool LOADERS>
static constexpr bool rolls()
{
    return WM * WN == 1 && (!B_KN || LOADERS);
}

// Position of the 16-byte piece c of row r, of the 2 BK bytes a row takes: two rows of
// 128 bytes share a 256-byte line of all 64 banks (see lds_piece in tw_gemm.hip); rows of
// 256 and 512 bytes are one and two lines, and the sixteen rows a read covers fall on the
// line's sixteen pieces, whichever rows one of its passes takes together.
template <int BK>
__device__ __forceinline__ int swizzled(int r, int c)
{
    return BK == 64 ? (c ^ ((r >> 1) & 7)) : ((c & ~15) | ((c ^ r) & 15));
}

// B stored [K x N]: the stage holds BK rows (k) of BN columns. A transposing read takes,
// per half wave, 32 bytes of eight rows: four consecutive ones of two groups eight rows
// apart. R = 128 / BN rows share a 256-byte line; the other row bits that differ move the
// 32 bytes within the row, so that the eight lie on different banks. (BN = 32: rows r and
// r + 8.)
template <int BN>
__device__ __forceinline__ int kn_swizzle(int r)
{
    if constexpr (BN == 128) return (r & 3) | (((r >> 3) & 1) << 2);
    else if constexpr (BN == 64) return ((r >> 1) & 1) | (((r >> 3) & 1) << 1);
    else return (r >> 3) & 1;
}

template <bool B_KN, int WM, int WN, int SUBS>
struct StageFrags {
    bf16x8 a[SUBS][WM];
    bf16x8 b[B_KN ? 1 : SUBS][B_KN ? 1 : WN];
    u32x2 blo[B_KN ? SUBS : 1][B_KN ? WN : 1], bhi[B_KN ? SUBS : 1][B_KN ? WN : 1];
};

// The arguments are scalars, not a struct: 13 scalar registers' worth, which the wave finds
// loaded when it starts (see the compiler flags), where fetching them was a round trip to
// memory ahead of everything else. Also ahead of the first load stands only what it needs:
// no division that tile_at can spare, the fragment addresses later. (16 rows, K = 1024, N =
// 8192: 5.6 -> 5.1 us; K = 8192, N = 3584: 13.7 -> 13.2; 512 x 4096 x 2048: 15.0 -> 14.7.)
// last_rows: rows of A in the last row of tiles.
template <bool B_KN, int WM, int WN, int WVM, int WVN, int BK, int S, bool LOADERS, bool STREAM_B, bool ROLLS>
__global__ __launch_bounds__((SmallTile<WM, WN, WVM, WVN, BK, S, LOADERS>::kThreads)) void gemm_tile_kernel(
    const char *A, const char *B, char *C, int N, int K, int tiles_m, int tiles_n, int last_rows, int group_m,
    int tiles_per_xcd, uint32_t help)
{
#if defined(__HIP_DEVICE_COMPILE__)  // as in tw_gemm.hip: the host pass needs the launch stub only
    using T = SmallTile<WM, WN, WVM, WVN, BK, S, LOADERS>;
    constexpr int kFilled = ROLLS ? S - 1 : S;  // stages filled ahead of the first step
    constexpr int SUBS = BK / kSubK, NW = T::kWaves, BM = T::BM, BN = T::BN, kRowBytes = BK * 2;
    static_assert(!B_KN || BN == 32 || BN == 64 || BN == 128, "kn_swizzle");
    // Weights that one row of tiles reads once are not worth keeping in the caches (16 rows,
    // K = 8192, N = 3584: 13.7 -> 13.1 us; with three rows of tiles 40 % slower).
    constexpr int kBPolicy = STREAM_B ? kStreamPolicy : 0;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    // (with loading waves only: shapes without helpers came out up to 2 % slower with the branch)
    if (LOADERS && static_cast<int>(blockIdx.x) >= tiles_per_xcd * kXcds)
        return help_tiles<B_KN, false, T::kThreads / 64>(A, B, (tiles_m - 1) * BM + last_rows, N, K, tiles_m, tiles_n, group_m,
                                                         tiles_per_xcd, BM, BN, help);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool computes = wave < T::kCompute;
    const int wave_m = computes ? wave / WVN : 0, wave_n = computes ? wave % WVN : 0;
    const long long row_bytes = K * 2ll, bkn_row_bytes = N * 2ll;
    const int k_tiles = K > 0 ? (K + BK - 1) / BK : 1;
    constexpr uint32_t kPastK = 0x80000000u;  // out of range whatever scalar offset (< 2^31) is added

    const bool loads = !LOADERS || wave >= T::kCompute;
    const int loader = LOADERS ? (loads ? wave - T::kCompute : 0) : wave;  // among the waves that load
    // Load duty: instruction i of this wave fills the 64 pieces from (i * NW + loader) * 64 on.
    constexpr int kRowPieces = kRowBytes / 16, kInstrRows = 64 / kRowPieces;
    constexpr int kStepRows = NW * kInstrRows;                 // rows all waves' instruction i covers
    constexpr int kRepeat = kStepRows % 16 == 0 || BK == 64 ? 1 : 16 / kStepRows;  // instructions after which the swizzle repeats
    static_assert(BK == 64 ? kStepRows % 16 == 0 : 16 % kStepRows == 0 || kStepRows % 16 == 0, "swizzle period");
    const int load_row = loader * kInstrRows + lane / kRowPieces;  // + i * kStepRows
    int load_piece[kRepeat];
#pragma unroll
    for (int q = 0; q < kRepeat; ++q) load_piece[q] = swizzled<BK>(load_row + q * kStepRows, lane % kRowPieces);
    // and of B stored [K x N]
    constexpr int kKnPieces = BN / 8, kKnInstrRows = 64 / kKnPieces;
    static_assert(!B_KN || (NW * kKnInstrRows) % 16 == 0, "the swizzle's row bits do not depend on the instruction");
    const int kn_row = loader * kKnInstrRows + lane / kKnPieces;  // + i * NW * kKnInstrRows
    const int kn_piece = (lane % kKnPieces) ^ (kn_swizzle<BN>(kn_row) << 1);

    for (int w = blockIdx.x; w < tiles_per_xcd * kXcds; w += gridDim.x) {
        const int lin = (w % kXcds) * tiles_per_xcd + w / kXcds;
        if (lin >= tiles_m * tiles_n) continue;
        const TileAt at = tile_at(lin, tiles_m, tiles_n, group_m);
        const long long m0 = static_cast<long long>(at.m) * BM;
        const int n0 = at.n * BN;
        const int rows_a = at.m == tiles_m - 1 ? last_rows : BM;
        const int rows_b = min(BN, N - n0);
        const __amdgpu_buffer_rsrc_t ra = make_rsrc(A + m0 * row_bytes, static_cast<uint32_t>(rows_a * row_bytes));
        const __amdgpu_buffer_rsrc_t rb = make_rsrc(B + n0 * row_bytes, static_cast<uint32_t>(rows_b * row_bytes));
        const uint32_t load_row_off = static_cast<uint32_t>(load_row * row_bytes);
        const uint32_t step_bytes = static_cast<uint32_t>(kStepRows * row_bytes);
        const uint32_t kn_off = n0 + kn_piece * 8 < N
                                    ? static_cast<uint32_t>(kn_row * bkn_row_bytes + (n0 + kn_piece * 8) * 2)
                                    : kPastK;
        const uint32_t kn_step_bytes = static_cast<uint32_t>(NW * kKnInstrRows * bkn_row_bytes);

        f32x4 acc[WM][WN];
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

        // The loads of one K step into one stage: offsets first, then load by load.
        struct Fetch {
            uint32_t off[kRepeat];
            lds_char_ptr_t base;
            __amdgpu_buffer_rsrc_t rbk;
        };
        auto fetch_ctx = [&](int kt, int slot) {
            Fetch c;
            c.base = (lds_char_ptr_t)(lds + slot * T::kStageBytes + loader * 1024);
#pragma unroll
            for (int q = 0; q < kRepeat; ++q) {
                const int k = kt * BK + load_piece[q] * 8;  // K <= 2^22, K steps run S past it at most
                c.off[q] = k < K ? load_row_off + static_cast<uint32_t>(k) * 2 : kPastK;
            }
            if constexpr (B_KN) {
                // rows k0 ... of B through a descriptor of their own: rows past K lie outside it
                const long long k0 = static_cast<long long>(kt) * BK, left = K - k0;
                const int rows_k = static_cast<int>(left < 0 ? 0 : left > BK ? BK : left);
                c.rbk = make_rsrc(B + (left > 0 ? k0 : 0) * bkn_row_bytes, static_cast<uint32_t>(rows_k * bkn_row_bytes));
            } else {
                c.rbk = rb;
            }
            return c;
        };
        auto fetch_one = [&](const Fetch &c, auto i_tag) {
            constexpr int i = decltype(i_tag)::value;
            if constexpr (i < T::kALoads) {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_ptr_t)(c.base + i * NW * 1024), 16, c.off[i % kRepeat],
                                                         step_bytes * i, 0, 0);
            } else {
                constexpr int j = i - T::kALoads;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(c.rbk, (lds_ptr_t)(c.base + T::kABytes + j * NW * 1024), 16,
                                                         B_KN ? kn_off : c.off[j % kRepeat],
                                                         (B_KN ? kn_step_bytes : step_bytes) * j, 0, kBPolicy);
            }
        };
        auto fetch = [&](const Fetch &c) { static_for<T::kLoads>([&](auto i) { fetch_one(c, i); }); };
        uint32_t fa[SUBS], fb[SUBS], fbkn[B_KN ? WN : 1];  // see below
        using F = StageFrags<B_KN, WM, WN, SUBS>;
        constexpr int kPerSub = WM + (B_KN ? 2 * WN : WN);
        constexpr int kReads = SUBS * kPerSub, kMma = SUBS * WM * WN;
        auto read_one = [&](F &f, uint32_t base, auto t_tag) {
            constexpr int t = decltype(t_tag)::value, s = t / kPerSub, i = t % kPerSub;
            if constexpr (i < WM) {
                f.a[s][i] = lds_read16<i * kBlk * kRowBytes>(base + fa[s]);
            } else if constexpr (!B_KN) {
                f.b[s][i - WM] = lds_read16<(i - WM) * kBlk * kRowBytes>(base + fb[s]);
            } else {
                constexpr int j = (i - WM) >> 1, kOff = s * kSubK * BN * 2;
                if constexpr (((i - WM) & 1) == 0) f.blo[s][j] = lds_read_tr8<kOff>(base + fbkn[j]);
                else f.bhi[s][j] = lds_read_tr8<kOff + 4 * BN * 2>(base + fbkn[j]);
            }
        };
        auto read_all = [&](F &f, int slot) {
            const uint32_t base = slot * T::kStageBytes;
            static_for<kReads>([&](auto t) { read_one(f, base, t); });
        };
        // Waits for this wave's LDS reads; the registers they fill pass through, so that no use moves above.
        auto settle = [&](F &f) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int s = 0; s < SUBS; ++s) {
#pragma unroll
                for (int i = 0; i < WM; ++i) asm volatile("" : "+v"(f.a[s][i]));
#pragma unroll
                for (int j = 0; j < WN; ++j) {
                    if constexpr (B_KN) asm volatile("" : "+v"(f.blo[s][j]), "+v"(f.bhi[s][j]));
                    else asm volatile("" : "+v"(f.b[s][j]));
                }
            }
        };
        // the matrix instructions of one stage, and between them the reads of the next one's fragments and (LOADS)
        // the loads of a later stage
        auto multiply = [&](F &cur, F &nxt, int nxt_slot, const Fetch &c, auto loads_tag) {
            constexpr bool LOADS = decltype(loads_tag)::value;
            const uint32_t base = nxt_slot * T::kStageBytes;
            static_for<kMma>([&](auto m_tag) {
                constexpr int m = decltype(m_tag)::value, s = m / (WM * WN), j = m % (WM * WN) / WM, i = m % WM;
                bf16x8 b;
                if constexpr (B_KN) {
                    const u32x4 t = {cur.blo[s][j].x, cur.blo[s][j].y, cur.bhi[s][j].x, cur.bhi[s][j].y};
                    b = __builtin_bit_cast(bf16x8, t);
                } else {
                    b = cur.b[s][j];
                }
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, cur.a[s][i], acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                // the last quarter (few instructions, and none of them a load: the last half) lets them arrive
                constexpr int kReadSlots = LOADERS && kMma < 12 ? kMma / 2 : kMma >= 8 ? kMma * 3 / 4 : kMma;
                static_for<kReads>([&](auto t) {
                    if constexpr (decltype(t)::value * kReadSlots / kReads == m) read_one(nxt, base, t);
                });
                static_for<T::kLoads>([&](auto t) {
                    if constexpr (LOADS && !LOADERS && decltype(t)::value * kMma / T::kLoads == m) fetch_one(c, t);
                });
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        // Waits until at most the loads of the last `newer` stages are outstanding (any number from LIMIT on: of the
        // last LIMIT), then for the same of all waves.
        auto wait_vm = [&](int newer, auto limit_tag) {
            constexpr int LIMIT = decltype(limit_tag)::value;
            if (loads) static_for<LIMIT + 1>([&](auto v) {
                constexpr int n = (LIMIT - decltype(v)::value) * T::kLoads;
                if (decltype(v)::value == 0 ? newer >= LIMIT : decltype(v)::value == LIMIT ? newer <= 0 : newer * T::kLoads == n)
                    __builtin_amdgcn_s_waitcnt(((n >> 4) << 14) | 0x0F70 | (n & 15));
            });
            __builtin_amdgcn_s_barrier();
        };

        // the previous tile's loads have landed and nobody reads LDS any more
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        static_for<kFilled>([&](auto s) {
            if (loads && (!T::kTail || decltype(s)::value < k_tiles)) fetch(fetch_ctx(decltype(s)::value, decltype(s)::value));
        });
        if (LOADERS && help) say_begun(help);
        // Fragment addresses inside a stage; block i lies 16 rows further on. (The lane passes
        // through an asm statement so that all this is computed here, the first loads on their
        // way; with [K x N] weights that made the K loop of 192 x 128 tiles 1 % slower.)
        int at_lane = lane;
        if constexpr (!B_KN) asm volatile("" : "+v"(at_lane));
        const int l15 = at_lane & 15, lgrp = at_lane >> 4;
#pragma unroll
        for (int s = 0; s < SUBS; ++s) {
            const int at = swizzled<BK>(l15, s * 4 + lgrp) * 16;
            fa[s] = (wave_m * kBlk * WM + l15) * kRowBytes + at;
            fb[s] = T::kABytes + (wave_n * kBlk * WN + l15) * kRowBytes + at;
        }
        if constexpr (B_KN) {
            const int a4 = l15 & 3, row = lgrp * 8 + (l15 >> 2);  // see lds_read_tr8
#pragma unroll
            for (int i = 0; i < WN; ++i) {
                const int col = wave_n * kBlk * WN + i * kBlk + 4 * a4;
                fbkn[i] = T::kABytes + row * (BN * 2) + (((col >> 3) ^ (kn_swizzle<BN>(row) << 1)) << 4) + (col & 7) * 2;
            }
        }
        wait_vm(T::kTail ? k_tiles - 1 : S, std::integral_constant<int, kFilled - 1>{});
        if constexpr (ROLLS) {
            // A wave's single block is one chain of matrix instructions, each of which waits for the one before (22
            // clocks), so nothing else may stand in it: fragments are read kAhead sub-steps ahead, from one stage into
            // the next, and waited for by count, never all of them. (So reads are under way where the loop ends, of which the
            // compiler knows nothing: a test follows the built code for uses of their registers.) Once a stage, ahead of its first read of the next
            // one, the waves meet: that has landed, and the stage before this is read and takes the loads of step kt +
            // S - 1 (one stage more in LDS than the other loop, for as many on their way). What bounds a tile now is its
            // intake at the L1's 64 bytes a clock, and weights from HBM. us before / with this, operands from the cache
            // and from HBM: [16 x 8192] x [8192 x 16] 8.8 / 6.4 and 9.0 / 6.6, x [8192 x 1280] 9.3 / 7.0 and 10.0 / 8.2, x
            // [8192 x 3584] 13.5 / 12.2 and 14.5 / 14.2; [64 x 8192] x [8192 x 1280] 10.3 / 8.5 and 11.1 / 10.2; [K x N]
            // [32 x 8192] x [8192 x 1280] 15.6 / 13.0 and 15.9 / 14.8. 180 sizes of 1 to 64 rows: 0.959 and 0.980 (K of two stages to 1024: see
            // kShortK). Reads 3 to 7 sub-steps ahead are level, six and
            // eight stages 1 to 8 % slower from the cache.
            constexpr int kAhead = 4, kBases = 4;
            static_assert(SUBS % kAhead == 0 && (kAhead - 1) * kPerSub < 16, "reads ahead, lgkmcnt field");
            // What the waves that load do at the meeting of step kt. MAIN: a whole stage is to be loaded, and the offsets
            // go on by one (with the waits and ranges of the last steps throughout, loading took longer than multiplying).
            Fetch c = fetch_ctx(S - 2, S - 1);
            int slot = S - 1;
            auto meet = [&](int kt, auto main_tag) {
                if constexpr (decltype(main_tag)::value) {
                    constexpr int n = (S - 3) * T::kLoads;
                    if (loads) __builtin_amdgcn_s_waitcnt(((n >> 4) << 14) | 0x0F70 | (n & 15));  // vmcnt(n)
                    if constexpr (B_KN) {
                        c = fetch_ctx(kt + S - 1, slot);
                    } else {
#pragma unroll
                        for (int q = 0; q < kRepeat; ++q) c.off[q] += kRowBytes;
                        c.base = (lds_char_ptr_t)(lds + slot * T::kStageBytes + loader * 1024);
                    }
                    __builtin_amdgcn_s_barrier();
                } else {
                    wait_vm(k_tiles - 2 - kt, std::integral_constant<int, S - 3>{});
                    c = fetch_ctx(kt + S - 1, slot);
                }
                slot = slot + 1 == S ? 0 : slot + 1;
            };
            if (computes) {
                bf16x8 a[SUBS], b[B_KN ? 1 : SUBS];
                u32x2 blo[B_KN ? SUBS : 1], bhi[B_KN ? SUBS : 1];
                uint32_t at_a[kBases], at_b[kBases];  // in the stage that is read; sub-step s: those of s % 4, and s / 4 lines on
                auto stage = [&](int of) {
                    const uint32_t base = of * T::kStageBytes;
#pragma unroll
                    for (int q = 0; q < kBases; ++q) {
                        at_a[q] = fa[q] + base;
                        at_b[q] = B_KN ? fbkn[0] + base : fb[q] + base;
                    }
                };
                auto read = [&](auto s_tag) {
                    constexpr int s = decltype(s_tag)::value, kOff = s / 4 * 256;
                    a[s] = lds_read16<kOff>(at_a[s % 4]);
                    if constexpr (B_KN) {
                        blo[s] = lds_read_tr8<s * kSubK * BN * 2>(at_b[0]);
                        bhi[s] = lds_read_tr8<s * kSubK * BN * 2 + 4 * BN * 2>(at_b[0]);
                    } else {
                        b[s] = lds_read16<kOff>(at_b[s % 4]);
                    }
                };
                int next = 0;
                auto roll = [&](int kt, auto main_tag) {
                    constexpr bool MAIN = decltype(main_tag)::value;
                    static_for<SUBS>([&](auto s_tag) {
                        constexpr int s = decltype(s_tag)::value, kNewer = (kAhead - 1) * kPerSub;
                        bf16x8 bs;
                        if constexpr (B_KN) {
                            asm volatile("s_waitcnt lgkmcnt(%[n])" : "+v"(a[s]), "+v"(blo[s]), "+v"(bhi[s]) : [n] "n"(kNewer) : "memory");
                            const u32x4 t = {blo[s].x, blo[s].y, bhi[s].x, bhi[s].y};
                            bs = __builtin_bit_cast(bf16x8, t);
                        } else {
                            asm volatile("s_waitcnt lgkmcnt(%[n])" : "+v"(a[s]), "+v"(b[s]) : [n] "n"(kNewer) : "memory");
                            bs = b[s];
                        }
                        acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bs, a[s], acc[0][0], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (s == SUBS - kAhead) {
                            next = next + 1 == S ? 0 : next + 1;
                            stage(next);
                            if constexpr (LOADERS) __builtin_amdgcn_s_barrier();
                            else meet(kt, main_tag);
                        }
                        read(std::integral_constant<int, (s + kAhead) % SUBS>{});
                        if constexpr (!LOADERS && s >= SUBS - kAhead) {
                            static_for<T::kLoads>([&](auto i) {
                                if constexpr (decltype(i)::value * kAhead / T::kLoads == s - (SUBS - kAhead))
                                    if (MAIN || kt + S - 1 < k_tiles) fetch_one(c, i);
                            });
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    });
                };
                stage(0);
                static_for<kAhead>([&](auto s) { read(s); });
                int kt = 0;
                if constexpr (!LOADERS)
                    for (; kt + S < k_tiles; ++kt) roll(kt, std::true_type{});
                for (; kt < k_tiles; ++kt) roll(kt, std::false_type{});
                // (what the last step asked for past the end of K)
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
                for (int s = 0; s < SUBS; ++s) {
                    asm volatile("" ::"v"(a[s]));
                    if constexpr (B_KN) asm volatile("" ::"v"(blo[s]), "v"(bhi[s]));
                    else asm volatile("" ::"v"(b[s]));
                }
            } else {
                int kt = 0;
                for (; kt + S < k_tiles; ++kt) {
                    meet(kt, std::true_type{});
                    fetch(c);
                }
                for (; kt < k_tiles; ++kt) {
                    meet(kt, std::false_type{});
                    if (kt + S - 1 < k_tiles) fetch(c);
                }
            }
        } else {
            F f0, f1;
            if (computes) {
                read_all(f0, 0);
                settle(f0);
            }
            int slot = 0, kt = 0;
            // Step kt, its fragments in cur; those of the next one have arrived in nxt at its end (no read is under way where
            // the control flow branches or joins). MAIN: stage kt + S is loaded meanwhile.
            auto step = [&](F &cur, F &nxt, auto main_tag) {
                constexpr bool MAIN = decltype(main_tag)::value;
                // stage kt + 1 has landed, stage kt is read
                wait_vm(MAIN ? S : k_tiles - 2 - kt, std::integral_constant<int, S - 2>{});
                Fetch c;
                if (loads) c = fetch_ctx(kt + S, slot);
                if constexpr (LOADERS || !MAIN)
                    if (loads && kt + S < k_tiles) fetch(c);
                slot = slot + 1 == S ? 0 : slot + 1;
                ++kt;
                __builtin_amdgcn_sched_barrier(0);
                if (computes) {
                    multiply(cur, nxt, slot, c, main_tag);
                    settle(nxt);
                } else if constexpr (MAIN && !LOADERS) {
                    fetch(c);
                }
            };
            while (kt + (T::kTail ? S + 1 : 0) < k_tiles) {  // (without a tail, a step past an odd end works on zeros)
                step(f0, f1, std::true_type{});
                step(f1, f0, std::true_type{});
            }
            if constexpr (T::kTail) {
                for (;;) {
                    step(f0, f1, std::false_type{});
                    if (kt == k_tiles) break;
                    step(f1, f0, std::false_type{});
                    if (kt == k_tiles) break;
                }
            } else {
                __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): loads past the end
            }
        }
        // A lane holds row l15 and four consecutive columns of each block. Rows past M and
        // columns past N are dropped by the range check.
        const long long c_row_bytes = N * 2;
        const __amdgpu_buffer_rsrc_t rc = make_rsrc(C + m0 * c_row_bytes, static_cast<uint32_t>(rows_a * c_row_bytes));
        if constexpr (T::kStagedStores) {
            // Through LDS, each wave in a region of its own, rows padded by 32 bytes, so that a
            // store covers whole rows of the wave's outputs, written through (as in tw_gemm.hip). The shapes whose stores do
            // not go through LDS keep the default policy: their few bytes leave within the launch either way (sc1: 16 rows,
            // K = 8192, N = 3584 level, 64 x 4096, K = 1024 4.13 -> 4.17 us).
            constexpr int kRowPitch = kBlk * WN * 2 + 32, kRegion = kBlk * WM * kRowPitch;
            constexpr int kPieces = kBlk * WN * 2 / 16, kRowsPerStore = 64 / kPieces;
            static_assert(T::kCompute * kRegion <= T::kLdsBytes, "the waves' regions");
            static_assert(64 % kPieces == 0 && (kBlk * WM) % kRowsPerStore == 0, "whole store instructions");
            __builtin_amdgcn_s_barrier();  // every wave's loads have landed and its fragments are read
            if (computes) {
                const uint32_t region = static_cast<uint32_t>(wave * kRegion);
                const uint32_t w_addr = region + l15 * kRowPitch + lgrp * 8;
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int j = 0; j < WN; ++j) {
                        u32x2 v;
                        v.x = pack_bf16x2(acc[i][j][0], acc[i][j][1]);
                        v.y = pack_bf16x2(acc[i][j][2], acc[i][j][3]);
                        *reinterpret_cast<__attribute__((address_space(3))) u32x2 *>(
                            static_cast<uintptr_t>(w_addr + i * kBlk * kRowPitch + j * kBlk * 2)) = v;
                    }
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
                const int piece_c = lane % kPieces, row_c = lane / kPieces;
                const int n = n0 + wave_n * (kBlk * WN) + piece_c * 8;
                const uint32_t g_off =
                    n < N ? static_cast<uint32_t>((wave_m * (kBlk * WM) + row_c) * c_row_bytes + n * 2) : kPastK;
                const uint32_t r_addr = region + row_c * kRowPitch + piece_c * 16;
                const uint32_t store_rows_bytes = static_cast<uint32_t>(kRowsPerStore * c_row_bytes);
#pragma unroll
                for (int i = 0; i < kBlk * WM / kRowsPerStore; ++i) {
                    const u32x4 v = *reinterpret_cast<__attribute__((address_space(3))) u32x4 *>(
                        static_cast<uintptr_t>(r_addr + i * kRowsPerStore * kRowPitch));
                    __builtin_amdgcn_raw_buffer_store_b128(v, rc, g_off + store_rows_bytes * i, 0, kStorePolicy);  // (no scalar offset: see st())
                }
            }
        } else if (computes) {
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                const int n = n0 + (wave_n * WN + j) * kBlk + lgrp * 4;
#pragma unroll
                for (int i = 0; i < WM; ++i) {
                    u32x2 v;
                    v.x = pack_bf16x2(acc[i][j][0], acc[i][j][1]);
                    v.y = pack_bf16x2(acc[i][j][2], acc[i][j][3]);
                    const uint32_t off =
                        n < N ? static_cast<uint32_t>(((wave_m * WM + i) * kBlk + l15) * c_row_bytes + n * 2) : kPastK;
                    __builtin_amdgcn_raw_buffer_store_b64(v, rc, off, 0, 0);
                }
            }
        }
    }
#endif
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

struct TileLaunch {
    int budget, cus;
    GemmPlace place;
    HelpPlan help;
    int *loading_waves = nullptr;  // not NULL: nothing is launched, but how many waves of a workgroup would only load
};
// LONG_K: from which K on there are loading waves (kNeverLoaders: not for this shape; kEveryK: at every K that it is taken for).
static constexpr int kNeverLoaders = 1 << 30, kLoadersIfHelped = 1 << 29, kEveryK = 0;
// K up to which tiles of 32 rows that could roll and have no loading waves do not, from a second stage on: that loop's one more
// stage in LDS and its meetings cost more there than its chain gains. Time rolling over time not, from the cache and from HBM:
//   32 x 32  K to 128 0.993, 0.992; 200 to 512 1.003 to 1.022, 1.004 to 1.012; 640 and 768 1.015 to 1.020, 1.007; 1024 1.003, 1.003;
//            1152 to 2040 0.985 to 0.96, 1.00
//   32 x 16  K to 512 1.00; 520 to 1024 1.007 to 1.018, 1.001 to 1.014; 1152 to 2040 0.98 to 1.00, 1.00
// 16 x 16 tiles, one wave of which multiplies, roll at every K (0.94 to 0.98, 0.98 to 0.99), 16 x 32 are level.
static constexpr int kShortK = 1024;
// STREAM: whether weights that one row of tiles reads once go past the caches (kStreamPolicy). Of the shapes for up to
// 64 rows only in trains, whose weights come from HBM: us kept / past the caches, from HBM, [40 x 3584] x [3584 x 8192] 14.8 /
// 13.1, 64 rows 17.4 / 15.2, [64 x 1024] x [1024 x 8192] 6.8 / 6.5, but weights that are in the cache do not stay there: 11.2 /
// 12.7 and 11.7 / 15.0. (Several rows of tiles: -14 to +20 % from HBM, +10 to +57 % from the cache.) kStreamAlways: the shape
// is taken for one row of tiles only (left_out).
enum Stream { kKeep, kStream, kStreamInTrains, kStreamAlways };
template <bool B_KN, int WM, int WN, int WVM, int WVN, int BK, int S, int LONG_K, Stream STREAM = kKeep, bool LOADERS = false,
          bool ROLLS = rolls<B_KN, WM, WN, LOADERS>()>
static tw_status launch_tile_t(const tw_gemm_args &g, const TileLaunch &l, hipStream_t stream)
{
    // (eight waves that multiply and four that load leave no registers for a workgroup beside them; weights that
    // one row of tiles reads once each come as fast, from HBM, to the waves that multiply: 32 x 3584, K = 8192 16.1 us, with
    // loading waves 17.2; with helpers they are ahead again)
    const bool one_row = STREAM == kStreamAlways || (STREAM != kKeep && g.M <= kBlk * WM * WVM &&
                                                     (STREAM == kStream || l.place == GemmPlace::kTrain));
    if constexpr (LONG_K < kNeverLoaders && !LOADERS)
        if ((LONG_K == kLoadersIfHelped ? l.help.helpers > 0 : g.K >= LONG_K) && !(l.place == GemmPlace::kBeside && WVM * WVN == 8) &&
            !(one_row && l.help.helpers == 0))
            return launch_tile_t<B_KN, WM, WN, WVM, WVN, BK, S, LONG_K, STREAM, true>(g, l, stream);
    if constexpr (ROLLS && !LOADERS && WVM == 2)
        if (g.K > BK && g.K <= kShortK)
            return launch_tile_t<B_KN, WM, WN, WVM, WVN, BK, S, LONG_K, STREAM, LOADERS, false>(g, l, stream);
    constexpr int STAGES = S + (ROLLS ? 1 : 0);  // (see the K loop)
    using T = SmallTile<WM, WN, WVM, WVN, BK, STAGES, LOADERS>;
    if (l.loading_waves) {
        *l.loading_waves = LOADERS ? T::kWaves : 0;
        return TW_OK;
    }
    const int64_t tiles_m = (g.M + T::BM - 1) / T::BM, tiles_n = (g.N + T::BN - 1) / T::BN;
    // (at kEveryK, what has no loading waves is one row)
    if constexpr ((STREAM == kStream || STREAM == kStreamInTrains) && (LOADERS || LONG_K != kEveryK))
        if (!one_row) return launch_tile_t<B_KN, WM, WN, WVM, WVN, BK, S, LONG_K, kKeep, LOADERS, ROLLS>(g, l, stream);
    if (tiles_m * tiles_n > (int64_t(1) << 30)) return TW_ERR_UNSUPPORTED;
    const int tiles_per_xcd = static_cast<int>((tiles_m * tiles_n + kXcds - 1) / kXcds);
    const int64_t slots = int64_t(tiles_per_xcd) * kXcds;
    // The whole device: a workgroup per tile, as many to a compute unit as fit. Under a
    // budget, and with helpers, one to a compute unit: more than half of its LDS is asked for.
    constexpr int kAloneBytes = T::kLdsBytes > 81 * 1024 ? T::kLdsBytes : 81 * 1024;
    const bool whole = l.budget >= l.cus && l.help.helpers == 0;
    const unsigned grid = static_cast<unsigned>((whole || slots < l.budget ? slots : l.budget) + l.help.helpers * kXcds);
    auto kern = gemm_tile_kernel<B_KN, WM, WN, WVM, WVN, BK, STAGES, LOADERS, STREAM != kKeep, ROLLS>;
    static std::atomic<int> allowed[kMaxDevices];
    TW_TRY(allow_dynamic_lds(reinterpret_cast<const void *>(kern), kAloneBytes, allowed));
    TW_HIP(launch_kernel(kern, dim3(grid), dim3(T::kThreads),
                         static_cast<unsigned>(whole ? T::kLdsBytes : kAloneBytes), stream,
                         static_cast<const char *>(g.A), static_cast<const char *>(g.B), static_cast<char *>(g.C),
                         static_cast<int>(g.N), static_cast<int>(g.K), static_cast<int>(tiles_m),
                         static_cast<int>(tiles_n), static_cast<int>(g.M - (tiles_m - 1) * T::BM),
                         tile_group_m(tiles_m, tiles_per_xcd, T::BM, T::BN, l.budget), tiles_per_xcd,
                         l.help.helpers > 0 ? l.help.packed | next_help_word() : 0u));
    return TW_OK;
}

// From which K a shape has loading waves. Time with them over time without, 96 and 256 tiles, K = 512, 1024, 4096 and 8192
// and some shorter ones, from the cache and from HBM:
//   16 x 16             -7 to -14 % from K = 4096 on, up to +7 % at 512
//   32 x 32             -19 to 0 %, up to +3 % at 1024; [K x N] -12 to +1 %, up to +6 % at 1024
//   64 x 32, 64 x 64    -10 to +2 %, +1 to +5 % up to 1024; 64 x 64 [K x N] 0 to +7 %, but -4 % with helpers
//   96 x 64             -6 to 0 %, up to +2 %; [K x N] -13 to +1 %, +2 to +4 % at 176 and 256
//   96 x 96             -11 to 0 %, up to +2 % at 136
//   96 x 128            -11 to +1 %, +2 to +5 % below 320 (0.2 us, what starting four more waves takes)
//   192 x 64 [K x N]    -10 to 0 %, +2 to +6 % at 512
//   128 x 128 [K x N]   -18 to -4 %, up to +5 % at 512
//   192 x 64, 128 x 128 -7 to +3 %, +1 to +10 % up to 1024: with helpers only, and no size has 192 x 64 with them
// The shapes, smallest first, and what one 64-deep K step of a tile takes when about
// every compute unit has one (us, measured on MI355X at K = 3584 and 8192). Several
// tiles to a compute unit take their times in turn, also where two fit at once. [K x N]
// weights cost two LDS reads a fragment instead of one, and rows of less than 128 bytes
// of them half a request's worth each (tiles of 64 columns and 16 or 32 rows, whole
// lines but half as many workgroups, came out level to 7 % slower than 32 x 32 there).
struct SmallTileShape {
    int rows, cols, k_step;
    float us_nk, us_kn;            // 0: not built for that layout
    float us_help_nk, us_help_kn;  // with helpers (0: none)
    tw_status (*nk)(const tw_gemm_args &, const TileLaunch &, hipStream_t);
    tw_status (*kn)(const tw_gemm_args &, const TileLaunch &, hipStream_t);
};
static const SmallTileShape kSmallTiles[] = {
    {16, 16, 256, 0.075f, 0.0f, 0.051f, 0.0f,
     launch_tile_t<false, 1, 1, 1, 1, 256, 4, 2048, kStream>, nullptr},
    {32, 16, 256, 0.097f, 0.0f, 0.060f, 0.0f,
     launch_tile_t<false, 1, 1, 2, 1, 256, 4, 2048, kStream>, nullptr},
    {16, 32, 256, 0.115f, 0.149f, 0.060f, 0.080f,
     launch_tile_t<false, 1, 1, 1, 2, 256, 4, kLoadersIfHelped, kStreamAlways>, launch_tile_t<true, 1, 1, 1, 2, 256, 4, 2048>},
    {32, 32, 128, 0.132f, 0.150f, 0.078f, 0.102f,
     launch_tile_t<false, 1, 1, 2, 2, 128, 4, 2048, kStream>, launch_tile_t<true, 1, 1, 2, 2, 128, 4, 2048>},
    {48, 32, 128, 0.150f, 0.0f, 0.093f, 0.0f,
     launch_tile_t<false, 3, 1, 1, 2, 128, 4, kEveryK, kStreamInTrains>, nullptr},
    {64, 32, 128, 0.180f, 0.200f, 0.109f, 0.122f,
     launch_tile_t<false, 2, 1, 2, 2, 128, 4, 2048, kStreamInTrains>, launch_tile_t<true, 2, 1, 2, 2, 128, 4, 2048>},
    {64, 64, 128, 0.200f, 0.230f, 0.139f, 0.155f,
     launch_tile_t<false, 2, 2, 2, 2, 128, 4, 2048>, launch_tile_t<true, 2, 2, 2, 2, 128, 4, kLoadersIfHelped>},
    {96, 64, 64, 0.255f, 0.280f, 0.182f, 0.240f,
     launch_tile_t<false, 3, 2, 2, 2, 64, 6, 2048>, launch_tile_t<true, 3, 2, 2, 2, 64, 6, 320>},
    {96, 96, 64, 0.338f, 0.0f, 0.245f, 0.0f,
     launch_tile_t<false, 3, 3, 2, 2, 64, 6, 320>, nullptr},
    {96, 128, 64, 0.405f, 0.430f, 0.260f, 0.290f,
     launch_tile_t<false, 3, 4, 2, 2, 64, 5, 512>, launch_tile_t<true, 3, 4, 2, 2, 64, 5, 512>},
    {192, 64, 64, 0.430f, 0.500f, 0.0f, 0.400f,
     launch_tile_t<false, 3, 2, 4, 2, 64, 4, kNeverLoaders>, launch_tile_t<true, 3, 2, 4, 2, 64, 4, 2048>},
    {128, 128, 64, 0.530f, 0.550f, 0.370f, 0.460f,
     launch_tile_t<false, 2, 4, 4, 2, 64, 4, kLoadersIfHelped>, launch_tile_t<true, 2, 4, 4, 2, 64, 4, 2048>},
    {192, 128, 64, 0.700f, 0.690f, 0.0f, 0.0f,
     launch_tile_t<false, 3, 4, 4, 2, 64, 3, kNeverLoaders>, launch_tile_t<true, 3, 4, 4, 2, 64, 3, kNeverLoaders>},
};

// 48 x 32 takes in 80 rows a step where 64 x 32 takes 96, and as one row of tiles leaves the helpers the compute units that
// two rows of 32 x 32 would use: trains of eight boundaries, us before / streamed / streamed with this shape, 33 rows 216.6 / 212.8
// / 205.0, 40 222.6 / 217.1 / 210.2, 48 234.1 / 229.1 / 222.8 (64 248.5 / 244.6 / 244.3); a boundary of 36 rows 25.6 / 24.6.
// Only where K is enough for helpers, below it is level with 64 x 32; in two rows it gains 6 % from the cache and loses 3 % from
// HBM ([96 x 8192] x [8192 x 3584]). (48 x 16, 64 x 16, 96 x 32 and 128 x 32, streamed: level to 80 % slower; 4 % faster at 80 rows,
// N = 8192.)
//
// Tiles of 16 x 32 are for one row of them: a second reads the weights again, which those of 32 x 32 read once. What
// bounds a decode step's tile is its intake, and of that a 16 x 16 tile spends half on the same 16 rows, a 32 x 32 one a
// quarter on rows that are not there. us before / with them, operands from the cache and from HBM: [16 x 8192] x [8192 x 8192]
// 25.4 / 21.9 and 26.9 / 23.2, [16 x 4096] x [4096 x 6144] 11.8 / 11.0 and 12.1 / 11.4, [16 x 3584] x [3584 x 8192] 10.9 / 10.4
// and 11.4 / 11.2; [K x N], with helpers, [16 x 8192] x [8192 x 3584] 15.4 / 13.6 and 16.5 / 14.6. Time over that with 32 x 32
// tiles, from the cache and from HBM, 789 sizes of up to 16 rows: [N x K] 0.92 and 0.94, [K x N] with helpers 0.76 and 0.86, without
// them K < 2048 0.91 and 1.013, the rest 1.00 and 1.00. Slower are, from HBM, [N x K] at K = 256 (1.01 to 1.03; 1.5 % faster from the
// cache, and K just below is faster from both) and [K x N] up to K = 2040 (to 1.03, of N = 7680 to 1.05: 0.1 us against the 0.1 to
// 1.1 that the cache gains elsewhere); from both, [K x N] whose rows are 16 KB apart, N = 8192, from K = 2560 on (1.03 and 1.006).
static bool left_out(const SmallTileShape &t, int64_t M, int64_t K)
{
    return t.cols == 32 && ((t.rows == 16 && M > 16) || (t.rows == 48 && (M > 48 || K < kHelpFromK)));
}

// A grid's tiles are worked off in turns of one to a compute unit. The launch, the first
// turn's pipeline fill and the last one's stores cost any grid about the same; each
// further turn adds a fill and stores of its own.
double tile_grid_us(int64_t M, int64_t N, int64_t K, int rows, int cols, int k_step, double us_per_step,
                    double us_per_turn, int budget)
{
    const int64_t tiles = ((M + rows - 1) / rows) * ((N + cols - 1) / cols);
    const int64_t turns = (tiles + budget - 1) / budget;
    const int64_t k_steps = (K + k_step - 1) / k_step * (k_step / 64);
    return double(turns) * double(k_steps) * us_per_step + double(turns - 1) * us_per_turn + 4.0;
}

// Helpers for g cut into tiles of shape t: false where they do not pay. A helper gets some 50 KB a us, so
// enough of them to fetch what the XCD with the most to read needs within the product's time, and a
// quarter more; with too few the tiles wait for the helpers (three where eight are needed: 10 to 60 %
// slower than none). Also false where the estimated time does not come below `limit`, before the rest is worked out.
static bool plan_help(const tw_gemm_args &g, const SmallTileShape &t, int budget, double limit, HelpPlan *plan, double *us)
{
    const float per_step = g.b_layout == TW_B_KN ? t.us_help_kn : t.us_help_nk;
    const int64_t max_bytes = int64_t(1) << 31;
    if (per_step == 0.0f || left_out(t, g.M, g.K) || g.K < kHelpFromK || g.N > (1 << 20)) return false;
    if (g.M * g.K * 2 >= max_bytes || g.N * g.K * 2 >= max_bytes) return false;
    const int64_t tiles_m = (g.M + t.rows - 1) / t.rows, tiles_n = (g.N + t.cols - 1) / t.cols;
    const int64_t per_xcd = (tiles_m * tiles_n + kXcds - 1) / kXcds, idle = budget / kXcds - per_xcd;
    if (idle < 1) return false;
    const double from_memory = double(g.M + g.N) * g.K * 2 / kHbmBytesPerUs;
    // Rows that do not start on a line: two lines for every 64 of K, or, in [K x N] weights, of N: there tiles of 64 rows took
    // 1.25 to 1.35 times as long as with whole lines (32 x 32, 192 x 64 and 128 x 128 as long, 96 rows 1.1 to 1.2), and were
    // chosen for an estimate that they did not keep. us before there were helpers / without this / with it, from the
    // cache and from HBM: [34 x 7040] x [7040 x 6344] 23.5 / 33.0 / 22.3 and 33.1 / 32.4 / 32.9, [388 x 3328] x [3328 x 632]
    // 11.1 / 13.4 / 11.5 and 17.3 / 14.5 / 12.6. 200 such sizes, times over those before helpers: 0.938 / 0.922 (the slowest
    // 1.24 / 1.14) and 0.758 / 0.757.
    const double off_line_a = g.K % 64 ? 1.2 : 1.0;
    const double off_line_b = g.b_layout == TW_B_KN && g.N % 64 && t.rows == 64 ? 1.3 : 1.0;
    const double time = std::max(double(per_step) * off_line_a * off_line_b * g.K / 64, from_memory);
    *us = time + 4.0;
    if (*us >= limit) return false;
    const int group_m = tile_group_m(tiles_m, per_xcd, t.rows, t.cols, budget);
    int64_t lines = 0;  // rows of A and columns of B that an XCD reads
    for (int x = 0; x < kXcds; ++x) {
        const Operands o = operands_of(x * per_xcd, per_xcd, g.M, g.N, tiles_m, tiles_n, group_m, t.rows, t.cols);
        lines = std::max<int64_t>(lines, o.a_hi - o.a_lo + o.n1 + o.n2);
    }
    const double needed = double(lines) * g.K * 2 / (time * kHelperBytesPerUs);
    if (needed > 0.85 * idle) return false;
    const int windows = static_cast<int>((g.K * 2 + kHelpWindow - 1) / kHelpWindow);
    const double pace = kHelpPace * time * 100 / windows;
    const double window_bytes = double(lines) * kHelpWindow;
    const double lead = std::max(1.0, std::max(kHelpLeadLeast, kHelpLeadMost - kHelpLag * windows * window_bytes) / window_bytes);
    plan->helpers = static_cast<int>(std::min<int64_t>(idle, int64_t(1.25 * needed) + 1));
    plan->packed = pack_help(pace, pace * lead);
    return true;
}

// The shape of the least estimated time, -1: none for the layout.
int best_small_tile(const tw_gemm_args &g, int budget, GemmPlace place, double *us, HelpPlan *help)
{
    int best = -1;
    *help = {};
    for (int i = 0; i < int(sizeof(kSmallTiles) / sizeof(kSmallTiles[0])); ++i) {
        const SmallTileShape &t = kSmallTiles[i];
        const float per_step = g.b_layout == TW_B_KN ? t.us_kn : t.us_nk;
        if (per_step == 0.0f || left_out(t, g.M, g.K)) continue;
        const double est = tile_grid_us(g.M, g.N, g.K, t.rows, t.cols, t.k_step, per_step, 3.0, budget);
        if (best < 0 || est < *us) {
            best = i;
            *us = est;
        }
    }
    if (best < 0 || place == GemmPlace::kBeside || place == GemmPlace::kWoven) return best;
    // Larger tiles that leave compute units to helpers gain nothing where the operands are in the
    // cache, where [N x K] weights of 59 MB and 64 rows take 19 us with them and 15 without (from HBM
    // 17 and 21): they are taken for a layer's weights, unless small, and for [K x N] weights, which gain more from HBM
    // than they lose from the cache: us before helpers / now, cache and HBM, [128 x 8192] x [8192 x 2048] 21.4 / 19.0 and
    // 34.4 / 19.0, [70 x 8192] x [8192 x 3328] 21.6 / 23.2 and 31.5 / 23.6, [294 x 2560] x [2560 x 1024] 8.3 / 9.7 and 13.4 / 9.9.
    // In a train whose weights together are more than the cache holds, every weight comes from HBM: [333 x 8192] x [8192 x 1280]
    // takes 26.4 without and 21.2 with them. us of a train of eight 70B-class boundaries as a chain of single ones / so, 150 rows
    // 357 / 348, 512 648 / 635, 700 756 / 744, 1500 1286 / 1252, level at 16 to 128 and from 1800 on.
    const bool train = place == GemmPlace::kTrain;
    const bool keep = g.b_layout == TW_B_NK && !train && (place != GemmPlace::kChain || g.N * g.K * 2 < kFromHbmBytes);
    const int only = best;
    const double plain = *us;
    const auto consider = [&](int shape, double limit) {
        HelpPlan plan;
        double est;
        if (!plan_help(g, kSmallTiles[shape], budget, limit, &plan, &est)) return;
        best = shape;
        *us = std::min(est, *us);
        *help = plan;
    };
    consider(only, 1e300);
    for (int i = 0; !keep && i < int(sizeof(kSmallTiles) / sizeof(kSmallTiles[0])); ++i)
        if (i != only) consider(i, std::min((train ? 1.0 : 0.94) * plain, *us));
    return best;
}

void small_tile_size(int shape, int *rows, int *cols)
{
    *rows = kSmallTiles[shape].rows;
    *cols = kSmallTiles[shape].cols;
}

tw_status launch_small_tile(const tw_gemm_args &g, int shape, const HelpPlan &help, int budget, int cus, GemmPlace place,
                            hipStream_t stream)
{
    const SmallTileShape &t = kSmallTiles[shape];
    return (g.b_layout == TW_B_KN ? t.kn : t.nk)(g, {budget, cus, place, help}, stream);
}

int small_tile_loading_waves(const tw_gemm_args &g, int shape, const HelpPlan &help, GemmPlace place)
{
    const SmallTileShape &t = kSmallTiles[shape];
    int waves = 0;
    (g.b_layout == TW_B_KN ? t.kn : t.nk)(g, {0, 0, place, help, &waves}, nullptr);
    return waves;
}

}  // namespace tw
