// Fused reduce over P partials + residual add + RMSNorm for gfx950
// (TokenWeave, arXiv 2505.11329: Section 4.3 and Appendix A, Listing 1).
//
// Per token row: x = (p_0 + ... + p_{P-1}) + residual in fp32; residual_out =
// bf16(x); s = rsqrt(mean(x^2) + eps); out = bf16((x * s) * weight). The paper's
// kernel lets the switch do the sum and re-reads the residual for the second
// loop; here the reading compute unit does the sum and x stays in registers, so
// every input byte is read once and every output byte written once.
//
// Shape of the launch
//   - One workgroup of up to 1024 threads (16 wave64) per compute unit, a persistent
//     grid of `budget` workgroups striding over groups of rows (Listing 1's
//     "token_id = blockIdx.x + iter * gridDim.x"). Each workgroup asks for more
//     than half of a compute unit's LDS, so two can never share one: the grid
//     size IS the number of compute units occupied.
//   - A row wider than a wave is covered by WPR whole waves (2 ... 16), each
//     thread owning VPT 16-byte vector columns (8 bf16); a workgroup handles
//     16/WPR rows per loop trip and is launched with just those waves. A narrower
//     row takes a power-of-two group of lanes. The thread->column map and the
//     reduction tree depend on H only, never on N, the grid or the row's
//     position: the same row gives the same bits in any launch (split or not,
//     any budget).
//   - Loads are software-pipelined two "chunks" deep (a chunk = the P+1 vectors
//     that feed one output vector): the loads of chunk q+2 are issued as soon as
//     chunk q has been summed, before the row's reduction and barrier, so a
//     thread always has P+1 .. 2(P+1) 16-byte loads in flight.
//   - Both outputs of a row are stored together once its scale is known (the new
//     residual stream could go out as soon as a chunk is summed, but loads that
//     are not interleaved with stores come in 1-1.5 % faster); rows of more than
//     16384 elements store it at once, for want of registers.
//   - Row sum of squares: per-thread fp32 FMAs, xor-butterfly across the lanes of
//     a wave (every lane ends with the same bits), and for rows wider than a
//     wave one LDS slot per wave and one barrier; slots are double-buffered by
//     row parity so one barrier per row suffices.
#include <atomic>
#include <type_traits>
#include <utility>

#include "tw_device.h"
#include "tw_internal.h"

namespace tw {

static constexpr int kThreads = 1024;
static constexpr int kWaves = kThreads / 64;
// Dynamic LDS each workgroup requests so that only one fits on a compute unit
// (gfx950 has 160 KiB per CU).
static constexpr unsigned kOccupancyPadBytes = 96 * 1024;

struct FusedParams {
    const void *partials[TW_MAX_P];
    const void *residual;
    const void *weight;
    void *out;
    void *residual_out;
    uint32_t *hw_ids;
    uint32_t n_bytes;      // rows of this launch * H * 2
    uint32_t group_bytes;  // rows_per_iter * H * 2
    uint32_t n_groups;     // ceil(rows / rows_per_iter)
    int hv;                // 16-byte vectors per row
    int P;
    int tpr_log2;          // rows of at most 64 vectors (and the thin kernel): 2^tpr_log2 lanes per row
    int wpr;               // wide kernel, rows wider than a wave: waves per row; else 0
    float eps;
    float inv_h;
};

// The P+1 vectors that feed one output vector, in flight.
template <int PT>
struct Chunk {
    u32x4 v[PT > 0 ? PT + 1 : 1];
};

// Kernels for a P known only at run time, in the place of P: a multiple of the loop's batch, or
// any number (1 to 5 % slower on short launches, for the padding's sign).
static constexpr int kAnyWhole = 0, kAnyPadded = -1;
static constexpr int kWideBatch = 4;

// Adds partials p0 ... p0 + BATCH - 1 to x, all requested at once. PAD: there may be fewer. Past
// the last one a load through a zero-length descriptor fetches nothing and reads as +0.0, and
// what is added is -0.0, the one value that leaves any sum as it is (a sum of -0.0 as well), so
// that a row's bits are those of the kernels without padding. (A branch around the addition in
// its place: up to 25 % slower. Without PAD every partial is live; with the selects left out
// the compiler orders the loads otherwise, 1 to 3 % slower.)
template <int BATCH, bool PAD>
__device__ __forceinline__ void add_batch(const FusedParams &prm, int p0, uint32_t lane_off, uint32_t scalar_off, float (&x)[8])
{
    u32x4 t[BATCH];
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
        const bool live = p0 + i < prm.P;
        t[i] = ld(make_rsrc(prm.partials[live ? p0 + i : 0], live ? prm.n_bytes : 0u), lane_off, scalar_off);
    }
    if (p0 == 0) unpack8(t[0], x); else add8(t[0], x);
#pragma unroll
    for (int i = 1; i < BATCH; ++i) add8(PAD ? t[i] | (p0 + i < prm.P ? 0u : 0x80008000u) : t[i], x);
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>)
template <int... I, typename F>
__device__ __forceinline__ void each_chunk(std::integer_sequence<int, I...>, F &&f)
{
    (f(std::integral_constant<int, I>{}), ...);
}

// How many chunks are kept in flight per thread (register budget: 128 VGPRs).
// (P = 10 and one chunk a row: two buffers would spill.)
template <int PT, int VPT>
constexpr int buffers_in_flight()
{
    return (PT <= 0) ? 1 : (((PT + 1) * 8 + 12 * VPT <= (VPT == 2 ? 100 : 92)) ? 2 : 1);
}

// Helpers of a short launch. A compute unit has some 150 lines of 128 bytes outstanding and gets
// them back in the order it asked, so the one that works on a row waits for HBM once per 150 of
// the row's (P + 1) * H / 64 lines, while the units that got no row idle. The workgroups from
// helper_base() on therefore ask for a row group's lines, a dword of each, all at the same time,
// from the XCD of the workgroup that owns the group (workgroups are dealt to the eight XCDs in turn),
// which then finds all but its first requests in that XCD's L2. Nothing depends on it: a helper
// on another XCD, or a late one, only helps less.
__host__ __device__ __forceinline__ uint32_t helper_base(uint32_t n_groups) { return (n_groups + 7u) & ~7u; }
static constexpr uint32_t kHelperBytes = 64 * 128;  // what one load of a wave asks for
// Loads that ask for a group's rows of the P partials and the residual, and for the weights.
__host__ __device__ __forceinline__ uint32_t helper_pieces(uint32_t group_bytes, int P)
{
    return (group_bytes + kHelperBytes - 1) / kHelperBytes * (P + 2);
}
// tensor(t): partial t, the residual (P), the weights (P + 1).
template <typename F>
__device__ __forceinline__ void help(uint32_t n_groups, uint32_t group_bytes, uint32_t n_bytes, int hv, int P, F &&tensor)
{
    const uint32_t base = helper_base(n_groups);
    if (blockIdx.x < base) return;  // between the last row group and the first helper
    const uint32_t share = (blockIdx.x - base) / base, group = (blockIdx.x - base) - share * base;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const uint32_t piece = share * (blockDim.x >> 6) + wave;
    const uint32_t per_tensor = (group_bytes + kHelperBytes - 1) / kHelperBytes;
    const int t = __builtin_amdgcn_readfirstlane(piece / per_tensor);
    if (group >= n_groups || t > P + 1) return;
    const uint32_t at = (piece - t * per_tensor) * kHelperBytes + lane * 128u;
    const uint32_t off = at >= group_bytes ? kOutOfRange : t <= P ? group * group_bytes + at : at;
    const uint32_t v = __builtin_amdgcn_raw_buffer_load_b32(make_rsrc(tensor(t), t <= P ? n_bytes : hv * 16u), off, 0, 0);
    asm volatile("" ::"v"(v));
}

// OWNERS: empty, or uint32_t: a launch with helpers, and its argument the number of workgroups that
// are none (it arrives in a register with the wave). Launches without have kernels of their own: the
// branch costs them up to 4 %.
template <int PT, int VPT, bool TRACE, bool STREAMED, typename... OWNERS>
__global__ __launch_bounds__(kThreads) void fused_kernel(OWNERS... owners, const FusedParams prm)
{
    if constexpr (sizeof...(OWNERS) > 0)
        if (blockIdx.x >= (owners + ...)) {
            const int P = PT > 0 ? PT : prm.P;
            return help(prm.n_groups, prm.group_bytes, prm.n_bytes, prm.hv, P,
                        [&](int t) { return t < P ? prm.partials[t < P ? t : 0] : t == P ? prm.residual : prm.weight; });
        }
    constexpr bool streamed = STREAMED;  // see st()
    __shared__ float s_wave_sum[2][kWaves];
    constexpr int NB = buffers_in_flight<PT, VPT>();
    constexpr bool KEEP_W = VPT <= 2;     // weights unpacked to fp32 once, else kept packed,
    constexpr bool RELOAD_W = VPT >= 8;  // or (no registers left) re-read through the cache per row
    constexpr bool LATE_RES = VPT <= 2;  // the new residual stream is stored with the output (wide rows: at once, or registers run out)

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int tpr_log2 = prm.tpr_log2;
    // Rows wider than a wave take wpr whole waves each (any number up to 16: the
    // workgroup is launched with just the waves that have columns to work on, an
    // idle wave's out-of-range loads and stores would still cost L1 request
    // slots); narrower rows take a power-of-two group of lanes.
    const int wpr = prm.wpr;
    const int tpr = wpr ? wpr << 6 : 1 << tpr_log2;
    const int row_in_iter = wpr ? __builtin_amdgcn_readfirstlane(wave / wpr) : tid >> tpr_log2;
    const int col0 = wpr ? tid - row_in_iter * tpr : tid & (tpr - 1);
    const int hv = prm.hv;

    if (TRACE && tid == 0) {
        // HW_ID (hwreg 4) and XCC_ID (hwreg 20), all 32 bits of each.
        prm.hw_ids[2 * blockIdx.x] = __builtin_amdgcn_s_getreg(4 | (0 << 6) | (31 << 11));
        prm.hw_ids[2 * blockIdx.x + 1] = __builtin_amdgcn_s_getreg(20 | (0 << 6) | (31 << 11));
    }

    __amdgpu_buffer_rsrc_t r_part[PT > 0 ? PT : 1];
    if constexpr (PT > 0) {
#pragma unroll
        for (int p = 0; p < PT; ++p) r_part[p] = make_rsrc(prm.partials[p], prm.n_bytes);
    }
    const __amdgpu_buffer_rsrc_t r_res = make_rsrc(prm.residual, prm.n_bytes);
    const __amdgpu_buffer_rsrc_t r_out = make_rsrc(prm.out, prm.n_bytes);
    const __amdgpu_buffer_rsrc_t r_res_out = make_rsrc(prm.residual_out, prm.n_bytes);

    // Byte offset of this thread's vector j inside a row group; columns past the
    // end of the row are pushed out of range for good.
    uint32_t lane_off[VPT];
    bool cvalid[VPT];
    u32x4 wv[RELOAD_W ? 1 : VPT];
    float wf[KEEP_W ? VPT : 1][8];
    const __amdgpu_buffer_rsrc_t r_w = make_rsrc(prm.weight, static_cast<uint32_t>(hv) * 16u);
    auto load_w = [&](int j) {
        return __builtin_amdgcn_raw_buffer_load_b128(r_w, cvalid[j] ? (col0 + j * tpr) * 16u : kOutOfRange, 0, 0);
    };
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        const int v = col0 + j * tpr;
        cvalid[j] = v < hv;
        lane_off[j] = static_cast<uint32_t>(row_in_iter * hv + v) * 16u;
        if constexpr (!RELOAD_W) wv[j] = load_w(j);
    }
    // (after the first chunks are requested, so that those do not wait for the weights)
    auto unpack_w = [&] {
        if constexpr (KEEP_W) {
#pragma unroll
            for (int j = 0; j < VPT; ++j) unpack8(wv[j], wf[j]);
        }
    };

    const uint32_t stride = gridDim.x;
    const uint32_t n_groups = prm.n_groups;
    const uint32_t group_bytes = prm.group_bytes;

    // Offset of chunk (group, j); rows past the end of the last group lie past n_bytes.
    auto chunk_off = [&](uint32_t group, int j) -> uint32_t {
        return cvalid[j] ? lane_off[j] + group * group_bytes : kOutOfRange;
    };
    // The loads of one chunk are kept together and in program order (the
    // scheduling barriers): the wait for chunk q must not also wait for q + 1.
    auto issue = [&](Chunk<PT> &c, uint32_t off) {
        if constexpr (PT > 0) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < PT; ++p) c.v[p] = ld(r_part[p], off);
            c.v[PT] = ld(r_res, off);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // x = (p_0 + p_1 + ... + p_{P-1}) + residual, left to right, fp32.
    auto reduce_chunk = [&](const Chunk<PT> &c, uint32_t off, float (&x)[8]) {
        if constexpr (PT > 0) {
            unpack8(c.v[0], x);
#pragma unroll
            for (int p = 1; p < PT; ++p) add8(c.v[p], x);
            add8(c.v[PT], x);
        } else {
            // four at a time (eight at a time measured 4 % slower at P = 12 and 16)
            const u32x4 r = ld(r_res, off);
            for (int p0 = 0; p0 < prm.P; p0 += kWideBatch) add_batch<kWideBatch, PT == kAnyPadded>(prm, p0, off, 0, x);
            add8(r, x);
        }
    };

    // Chunks are numbered q = trip * VPT + j; trip t handles row group
    // blockIdx.x + t * gridDim.x. NB chunk buffers rotate, chunk q sits in buffer
    // q % NB and is refilled with chunk q + NB as soon as it has been summed.
    Chunk<PT> buf[NB];
    int parity = 0;
    // One trip, its first chunk in buffer FIRST. MORE: the row group that the refills past
    // this row reach into exists. (A compile-time choice, hence the copies of the trip below: a
    // load past the end is dropped by the range check but still takes its turn in the L1's
    // request queue, and the last trips have all of them. With such loads, and the weights
    // waited for ahead of the first chunk, 64 rows of 4096 elements, P = 8, on 64 compute units
    // took 8.5 us and take 5.7; 256 rows of 2048 9.0 -> 5.9; 64 rows of 16384 10.5 -> 9.2.)
    auto trip = [&](uint32_t group, auto first_tag, auto more_tag) {
        constexpr int FIRST = decltype(first_tag)::value;
        constexpr bool MORE = decltype(more_tag)::value;
        float x[VPT][8];
        float ss = 0.0f;
        each_chunk(std::make_integer_sequence<int, VPT>{}, [&](auto j_tag) {
            constexpr int j = decltype(j_tag)::value;
            Chunk<PT> &b = buf[(FIRST + j) % NB];
            const uint32_t off = chunk_off(group, j);
            reduce_chunk(b, off, x[j]);
            constexpr int nj = (j + NB) % VPT;
            if constexpr (j + NB < VPT) issue(b, chunk_off(group, nj));
            else if constexpr (MORE) issue(b, chunk_off(group + (VPT == 1 ? NB : 1) * stride, nj));
            if constexpr (!LATE_RES) st(r_res_out, off, pack8(x[j]), streamed);
#pragma unroll
            for (int e = 0; e < 8; ++e) ss = __builtin_fmaf(x[j][e], x[j][e], ss);
        });

        // Row sum of squares: the row's lanes inside this wave, then (rows
        // wider than a wave) the row's waves through LDS.
        ss = wpr ? group_sum(ss, 6) : group_sum(ss, tpr_log2);
        if (wpr) {
            // the row's wave sums, padded with zeros to 16, through a 16-lane butterfly
            if (lane == 0) s_wave_sum[parity][wave] = ss;
            __syncthreads();
            const int k = lane & 15;
            const float part = k < wpr ? s_wave_sum[parity][row_in_iter * wpr + k] : 0.0f;
            ss = group_sum(part, 4);
            parity ^= 1;
        }
        const float s = rsqrtf(ss * prm.inv_h + prm.eps);

#pragma unroll
        for (int j = 0; j < VPT; ++j) {
            float y[8];
            if constexpr (KEEP_W) {
#pragma unroll
                for (int e = 0; e < 8; ++e) y[e] = (x[j][e] * s) * wf[j][e];
            } else {
                float w[8];
                if constexpr (RELOAD_W) unpack8(load_w(j), w);
                else unpack8(wv[j], w);
#pragma unroll
                for (int e = 0; e < 8; ++e) y[e] = (x[j][e] * s) * w[e];
            }
            if constexpr (LATE_RES) st(r_res_out, chunk_off(group, j), pack8(x[j]), streamed);
            st(r_out, chunk_off(group, j), pack8(y), streamed);
        }
    };

    using Zero = std::integral_constant<int, 0>;
    using One = std::integral_constant<int, 1>;
    uint32_t group = blockIdx.x;  // (but for helpers the grid has at most n_groups workgroups)
    if constexpr (VPT == 1 && NB == 2) {
        // two trips ahead: the buffers alternate from trip to trip
        issue(buf[0], chunk_off(group, 0));
        if (group + stride < n_groups) {
            issue(buf[1], chunk_off(group + stride, 0));
            unpack_w();
            while (group + 2 * stride < n_groups) {
                trip(group, Zero{}, std::true_type{});
                group += stride;
                if (group + 2 * stride >= n_groups) {
                    trip(group, One{}, std::false_type{});
                    trip(group + stride, Zero{}, std::false_type{});
                    return;
                }
                trip(group, One{}, std::true_type{});
                group += stride;
            }
            trip(group, Zero{}, std::false_type{});
            trip(group + stride, One{}, std::false_type{});
        } else {
            unpack_w();
            trip(group, Zero{}, std::false_type{});
        }
    } else {
        issue(buf[0], chunk_off(group, 0));
        if constexpr (NB == 2) issue(buf[1], chunk_off(group, 1));
        unpack_w();
        for (; group + stride < n_groups; group += stride) trip(group, Zero{}, std::true_type{});
        trip(group, Zero{}, std::false_type{});
    }
}

// ---------------------------------------------------------------------------
// The same arithmetic in workgroups small enough to sit NEXT TO a GEMM workgroup
// on the same compute unit (256 threads, at most 128 VGPRs, 128 bytes of LDS): the
// "shared" launch mode. Instead of taking a few compute units away from the
// GEMM, the fused kernel is spread thinly over all of them and uses the HBM
// bandwidth the matrix-core-bound GEMM leaves idle. (The two waves per SIMD of a
// GEMM on 256 x 128 tiles hold 2 x 152 of a lane's 512 registers, [K x N] 2 x 160,
// which leaves room for one such wave.)
//
// Bits are identical to fused_kernel's: a thread here plays Q (a row's vectors
// over 256, rounded up: 1 ... 4) of the wide kernel's threads (columns tid,
// tid+256, ...), keeps one sum of squares
// per played thread, and the reduction runs the very same tree (64-lane
// butterfly per played wave, then the 16-lane butterfly over the row's wave
// sums in LDS). Only rows of at most 1024 vectors (H <= 8192) are handled.
// With an even Q two chunks of loads are in flight per thread (chunk c sits in
// buffer c & 1, which needs no run-time index because every row then starts on
// buffer 0), with an odd Q one. Both outputs of a row are stored together once
// its scale is known: a small launch is one wave of workgroups that all run in
// step, and reads that are not interleaved with stores come in faster (a
// 1024-row, H = 8192, P = 8 launch: 33.5 -> 32.2 us with both changes, 256 rows
// 10.6 -> 9.7 us).
//
// What bounds it: HBM from a few thousand rows on; with a row per workgroup what the
// row's compute unit takes in (see help()); in between the chain of round
// trips of one row. Three things lengthened the chain: each output vector's weights
// were asked for on their own, behind the stores of the vector before, so that a row's
// stores went out one round trip after the other; loads past the end, dropped but
// issued; and row sums that went through the LDS, two permutes per vector. Without
// them, us (back-to-back launches, P = 8, H = 8192): 16 rows 5.3 -> 4.5, 64 6.6 -> 5.7,
// 512 17.7 -> 16.7, 1024 32.5 -> 31.7 (5.8 TB/s), 4096 119 -> 116; P = 2, H = 4096: 512 rows
// 5.4 -> 4.4, 2048 15.7 -> 14.8. Every P has its own instance: P = 6, H = 5120, 1531 rows
// 28.2 us with a run-time loop over P in the wide kernel, 25.4 (5.6 TB/s) here.
// ---------------------------------------------------------------------------
static constexpr int kThinThreads = 256;
// The all-at-once form is taken by whole-device launches of at most one workgroup per compute
// unit whose inputs come to at most this many bytes (and P <= kDeepMaxP: registers). Measured
// on MI355X at 16 and 64 rows, H = 8192, 5120, 4096: level to 8 % faster than two chunks at a
// time; at 256 rows of H = 8192 8 % slower: beyond a few MB the requests of a launch queue up.
static constexpr int64_t kDeepInputBytes = 6 << 20;

// DEEP: the form for batches so small that a launch is one round trip to memory
// and back (decode steps, Appendix B): a workgroup has one row group only, every
// chunk of it is requested at once together with the weights, and nothing is
// refilled. It needs ~200 registers, so it is a kernel of its own
// (fused_deep_kernel) without the 128-register bound that lets the other one
// sit beside a GEMM workgroup. Same arithmetic in the same order: same bits.
static constexpr int kDeepMaxP = 8;   // most partials it has registers for
static constexpr int kDeepFirst = 3;  // tensors whose addresses arrive in registers (see fused_deep_kernel)
template <int PT, int Q, bool TRACE, bool STREAMED, bool DEEP>
__device__ __forceinline__ void thin_body(const FusedParams &prm)
{
    constexpr bool streamed = STREAMED;  // see st()
    __shared__ float s_wave_sum[2][kWaves];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int tpr_log2 = prm.tpr_log2;
    const int tpr = 1 << tpr_log2;
    const int hv = prm.hv;
    // Q > 1: the whole workgroup covers one row, thread plays columns tid + 256 q.
    // Q == 1: rows of at most 256 vectors, 256 / tpr of them per workgroup.
    const int row_in_iter = (Q > 1) ? 0 : (tid >> tpr_log2);
    const int col0 = (Q > 1) ? tid : (tid & (tpr - 1));

    if (TRACE && tid == 0) {
        prm.hw_ids[2 * blockIdx.x] = __builtin_amdgcn_s_getreg(4 | (0 << 6) | (31 << 11));
        prm.hw_ids[2 * blockIdx.x + 1] = __builtin_amdgcn_s_getreg(20 | (0 << 6) | (31 << 11));
    }

    // The weights are re-read for every row with ordinary (cached) loads: the
    // streamed tensors are loaded "nt" and do not displace them from the L1, and
    // no LDS is spent on them, which is what lets this workgroup fit beside a GEMM
    // workgroup that uses 144 KiB of it.
    const __amdgpu_buffer_rsrc_t r_w = make_rsrc(prm.weight, static_cast<uint32_t>(hv) * 16u);

    __amdgpu_buffer_rsrc_t r_part[PT > 0 ? PT : 1];
    if constexpr (PT > 0) {
#pragma unroll
        for (int p = 0; p < PT; ++p) r_part[p] = make_rsrc(prm.partials[p], prm.n_bytes);
    }
    const __amdgpu_buffer_rsrc_t r_res = make_rsrc(prm.residual, prm.n_bytes);
    const __amdgpu_buffer_rsrc_t r_out = make_rsrc(prm.out, prm.n_bytes);
    const __amdgpu_buffer_rsrc_t r_res_out = make_rsrc(prm.residual_out, prm.n_bytes);

    // Address of chunk q of a row group: a lane register (the same for every q but the last,
    // which may reach past the row) and a scalar for group and q.
    const int last_col = col0 + (Q - 1) * kThinThreads;
    const uint32_t lane_off = static_cast<uint32_t>(row_in_iter * hv + col0) * 16u;
    const uint32_t lane_off_last = last_col < hv ? lane_off : kPastTensor;
    const uint32_t group_bytes = prm.group_bytes;
    struct Off {
        uint32_t lane, scalar;
    };
    auto chunk_off = [&](uint32_t group, int q) -> Off {
        return {q == Q - 1 ? lane_off_last : lane_off, group * group_bytes + q * (kThinThreads * 16u)};
    };
    auto issue = [&](Chunk<PT> &c, Off off) {
        if constexpr (PT > 0) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < PT; ++p) c.v[p] = ld(r_part[p], off.lane, off.scalar);
            c.v[PT] = ld(r_res, off.lane, off.scalar);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto reduce_chunk = [&](const Chunk<PT> &c, Off off, float (&x)[8]) {
        if constexpr (PT > 0) {
            unpack8(c.v[0], x);
#pragma unroll
            for (int p = 1; p < PT; ++p) add8(c.v[p], x);
            add8(c.v[PT], x);
        } else {
            // eight at a time: a thread here has four times the wide kernel's work per row and
            // fewer waves to hide a round trip behind (four at a time: 10-25 % slower); the
            // padded batch on its own (1 to 3 % faster than padding in every one)
            const u32x4 r = ld(r_res, off.lane, off.scalar);
            int p0 = 0;
            for (; p0 + 8 <= prm.P; p0 += 8) add_batch<8, false>(prm, p0, off.lane, off.scalar, x);
            if (p0 < prm.P) add_batch<8, true>(prm, p0, off.lane, off.scalar, x);
            add8(r, x);
        }
    };

    // This workgroup's row groups: blockIdx.x, blockIdx.x + gridDim.x, ... The
    // workgroups resident at one time then read neighbouring rows of every stream,
    // which the memory system likes better than each workgroup walking a block of
    // its own (4-9 % at 8K rows and more).
    const uint32_t first = blockIdx.x;
    const uint32_t gstride = gridDim.x;
    const uint32_t last = prm.n_groups;
    // Chunks in flight: NB. Chunk (group, q) sits in buffer q % NB and is refilled
    // with the chunk NB further on: the same row's, or the workgroup's next row's;
    // after its last row nothing is fetched.
    constexpr int NB = DEEP ? Q : (Q % 2 == 0 && PT <= 8) ? 2 : 1;  // (registers: 128)
    static_assert(!DEEP || PT > 0, "the run-time loop over P keeps nothing in flight");
    Chunk<PT> buf[NB];
    if constexpr (DEEP) {
        // Tensor by tensor, the ones whose addresses the wave finds in registers first; the asm
        // statement is where the others' addresses are waited for.
        each_chunk(std::make_integer_sequence<int, PT + 1>{}, [&](auto p_tag) {
            constexpr int p = decltype(p_tag)::value;
            __builtin_amdgcn_sched_barrier(0);
            const void *from = p < PT ? prm.partials[p < PT ? p : 0] : prm.residual;
            if constexpr (p >= kDeepFirst) asm volatile("" : "+s"(from));
            const __amdgpu_buffer_rsrc_t r = make_rsrc(from, prm.n_bytes);
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const Off at = chunk_off(first, q);
                buf[q].v[p] = ld(r, at.lane, at.scalar);
            }
        });
        __builtin_amdgcn_sched_barrier(0);
    } else {
        issue(buf[0], chunk_off(first, 0));
        if constexpr (NB >= 2) issue(buf[1], chunk_off(first, 1));
        static_assert(NB <= 2, "chunks issued above");
    }
    u32x4 wv[Q];
    auto load_weights = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        const void *from = prm.weight;
        if constexpr (DEEP) asm volatile("" : "+s"(from));
        const __amdgpu_buffer_rsrc_t r = DEEP ? make_rsrc(from, static_cast<uint32_t>(hv) * 16u) : r_w;
#pragma unroll
        for (int q = 0; q < Q; ++q)
            wv[q] = __builtin_amdgcn_raw_buffer_load_b128(r, q < Q - 1 || last_col < hv ? col0 * 16u : kPastTensor,
                                                          q * (kThinThreads * 16u), 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (DEEP) load_weights();
    constexpr int kAheadOfStores = NB == 1 ? 1 : (PT + 1) * 8 + Q * 12 <= 112 ? 1 : 0;
    int parity = 0;
    // One row group. Loads come back in the order they were issued, and so do stores: the
    // weights are asked for before the next row's chunks, or the output would wait for those,
    // and all together, or each vector of the output would wait for the stores of the one
    // before it. Of two chunks of the next row one goes out after the stores, or both, where
    // the registers do not hold them beside the weights. MORE: the
    // workgroup has another row group. (A compile-time choice: loads past the end would be
    // dropped by the range check, but each still takes its turn in the L1's request queue.)
    auto row_group = [&](uint32_t group, auto more_tag) {
        constexpr bool MORE = decltype(more_tag)::value;
        float x[Q][8];
        float ss[Q];
        each_chunk(std::make_integer_sequence<int, Q>{}, [&](auto q_tag) {
            constexpr int q = decltype(q_tag)::value;
            Chunk<PT> &b = buf[q % NB];
            reduce_chunk(b, chunk_off(group, q), x[q]);
            if constexpr (!DEEP) {
                if constexpr (q + NB < Q) issue(b, chunk_off(group, q + NB));
                if constexpr (q == (Q >= 2 ? Q - 2 : 0)) load_weights();
                if constexpr (MORE && q + NB >= Q && q - Q + NB < kAheadOfStores)
                    issue(b, chunk_off(group + gstride, q + NB - Q));
            }
            float acc = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc = __builtin_fmaf(x[q][e], x[q][e], acc);
            ss[q] = Q > 1 ? group_sum(acc, 6) : group_sum(acc, tpr_log2 < 6 ? tpr_log2 : 6);
        });
        float total = ss[0];
        if (Q > 1 || tpr_log2 > 6) {
            if (lane == 0) {
#pragma unroll
                for (int q = 0; q < Q; ++q) s_wave_sum[parity][wave + q * (kThinThreads / 64)] = ss[q];
            }
            __syncthreads();
            // the played waves' sums, padded with zeros to 16, as in the wide kernel
            const int waves_per_row = (Q > 1) ? Q * (kThinThreads / 64) : tpr >> 6;
            const int k = lane & 15;
            const float part = k < waves_per_row ? s_wave_sum[parity][row_in_iter * waves_per_row + k] : 0.0f;
            total = group_sum(part, 4);
            parity ^= 1;
        }
        const float s = rsqrtf(total * prm.inv_h + prm.eps);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            float w[8], y[8];
            unpack8(wv[q], w);
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = (x[q][e] * s) * w[e];
            const Off at = chunk_off(group, q);
            const uint32_t off = at.lane + at.scalar;  // (see st())
            st(r_res_out, off, pack8(x[q]), streamed);
            st(r_out, off, pack8(y), streamed);
        }
        if constexpr (MORE)
            each_chunk(std::make_integer_sequence<int, NB - kAheadOfStores>{}, [&](auto i_tag) {
                constexpr int c = kAheadOfStores + decltype(i_tag)::value;  // chunk c of the next row
                issue(buf[c], chunk_off(group + gstride, c));
            });
    };
    uint32_t group = first;
    if constexpr (!DEEP)
        for (; group + gstride < last; group += gstride) row_group(group, std::true_type{});
    row_group(group, std::false_type{});
}

template <int PT, int Q, bool TRACE, bool STREAMED>
__global__ __launch_bounds__(kThinThreads) __attribute__((amdgpu_waves_per_eu(4)))
void fused_thin_kernel(const FusedParams prm)
{
    thin_body<PT, Q, TRACE, STREAMED, false>(prm);
}

// The arguments of the form for small batches: a first one of eight words that arrives in scalar
// registers with the wave (an argument of more than fourteen does not), and the rest, a round trip to
// (host) memory away, over which the loads of the first three tensors are on their way. Tensors in the
// order of help(): partials, residual, weights. Two arguments, for the runtime handles each on its own: with
// four, six tensors in registers, 16 rows of 8192, P = 8 took 3.81 us where they take 3.75 (from HBM
// 4.66 / 4.57); a call on the host 2.55 to 2.75 either way, some 0.05 more than with one block that
// the wave has to fetch (which the same launch then took 5.3 us with).
struct DeepRest {
    const void *tensor[kDeepMaxP + 2 - kDeepFirst];
    void *out, *residual_out;
    float eps, inv_h;
};
typedef uint64_t DeepFirst __attribute__((ext_vector_type(4)));  // kDeepFirst tensors and the sizes
template <int PT, int Q>
__global__ __launch_bounds__(kThinThreads) void fused_deep_kernel(DeepFirst first, const DeepRest rest)
{
    auto tensor = [&](int i) -> const void * {
        return reinterpret_cast<const void *>(i == 0 ? first.x : i == 1 ? first.y : first.z);
    };
    const uint64_t shape = first.w;
    FusedParams prm;
    prm.n_bytes = static_cast<uint32_t>(shape);
    prm.hv = shape >> 32 & 0xfff;
    prm.tpr_log2 = shape >> 44 & 0xf;
    prm.n_groups = static_cast<uint32_t>(shape >> 48);
    prm.group_bytes = (Q > 1 ? 1 : kThinThreads >> prm.tpr_log2) * prm.hv * 16u;
    if (blockIdx.x >= prm.n_groups)
        return help(prm.n_groups, prm.group_bytes, prm.n_bytes, prm.hv, PT,
                    [&](int t) { return t < kDeepFirst ? tensor(t) : rest.tensor[t < kDeepFirst ? 0 : t - kDeepFirst]; });
    each_chunk(std::make_integer_sequence<int, PT + 2>{}, [&](auto i_tag) {
        constexpr int i = decltype(i_tag)::value;
        const void *t = i < kDeepFirst ? tensor(i) : rest.tensor[i < kDeepFirst ? 0 : i - kDeepFirst];
        if constexpr (i < PT) prm.partials[i] = t;
        else if constexpr (i == PT) prm.residual = t;
        else prm.weight = t;
    });
    prm.out = rest.out;
    prm.residual_out = rest.residual_out;
    prm.eps = rest.eps;
    prm.inv_h = rest.inv_h;
    thin_body<PT, Q, false, false, true>(prm);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

FusedGeometry fused_geometry(int64_t H)
{
    FusedGeometry g;
    g.hv = static_cast<int>(H / 8);
    int l2 = 0;
    while ((1 << l2) < g.hv && l2 < 10) ++l2;
    g.tpr_log2 = l2;
    if (g.hv <= 64) {  // several rows per wave, or one
        g.vpt = 1;
        g.wpr = 0;
        g.rows_per_iter = kThreads >> l2;
        g.block = kThreads;
        return g;
    }
    const int need = (g.hv + kThreads - 1) / kThreads;  // 1..8
    g.vpt = need <= 1 ? 1 : need <= 2 ? 2 : need <= 4 ? 4 : 8;
    g.wpr = (g.hv + 64 * g.vpt - 1) / (64 * g.vpt);  // 2..16
    g.rows_per_iter = kWaves / g.wpr;
    g.block = g.rows_per_iter * g.wpr * 64;
    return g;
}

int64_t fused_grid_size(int64_t n_rows, const FusedGeometry &g, int budget_wgs)
{
    if (n_rows <= 0) return 0;
    const int64_t groups = (n_rows + g.rows_per_iter - 1) / g.rows_per_iter;
    return groups < budget_wgs ? groups : budget_wgs;
}

tw_status validate_fused(const tw_fused_args &a)
{
    if (a.P < 1 || a.P > TW_MAX_P) return TW_ERR_SHAPE;
    if (a.N < 0 || a.H <= 0) return TW_ERR_SHAPE;
    if (!(a.eps >= 0.0f) || !(a.eps <= 3.402823466e+38f)) return TW_ERR_SHAPE;  // rejects NaN, Inf, < 0
    if (a.H % 8 != 0 || a.H > TW_MAX_H) return TW_ERR_UNSUPPORTED;
    if (a.N > (INT64_MAX / 2) / a.H) return TW_ERR_SHAPE;
    if (!a.weight) return TW_ERR_NULL;
    if (!aligned16(a.weight)) return TW_ERR_ALIGN;
    // The [N x H] tensors of an empty batch have no storage to point at.
    if (a.N == 0) return TW_OK;
    if (!a.partials || !a.residual || !a.out || !a.residual_out) return TW_ERR_NULL;
    for (int p = 0; p < a.P; ++p)
        if (!a.partials[p]) return TW_ERR_NULL;
    if (!aligned16(a.residual) || !aligned16(a.out) || !aligned16(a.residual_out)) return TW_ERR_ALIGN;
    for (int p = 0; p < a.P; ++p)
        if (!aligned16(a.partials[p])) return TW_ERR_ALIGN;

    const uint64_t tensor = static_cast<uint64_t>(a.N) * static_cast<uint64_t>(a.H) * 2u;
    const uint64_t wbytes = static_cast<uint64_t>(a.H) * 2u;
    if (ranges_overlap(a.out, tensor, a.residual_out, tensor)) return TW_ERR_ALIAS;
    const void *outs[2] = {a.out, a.residual_out};
    for (int o = 0; o < 2; ++o) {
        if (ranges_overlap(outs[o], tensor, a.weight, wbytes)) return TW_ERR_ALIAS;
        // residual: only residual_out may coincide with it, and only exactly
        if (ranges_overlap(outs[o], tensor, a.residual, tensor) &&
            !(o == 1 && a.residual_out == a.residual))
            return TW_ERR_ALIAS;
        // partials: only out may coincide with one, and only exactly
        for (int p = 0; p < a.P; ++p)
            if (ranges_overlap(outs[o], tensor, a.partials[p], tensor) &&
                !(o == 0 && a.out == a.partials[p]))
                return TW_ERR_ALIAS;
    }
    return TW_OK;
}

// Partial counts that are traced with the kernel that runs them untraced; the others are
// traced with the run-time loop over P (same grid, same bits).
template <int PT>
static constexpr bool kTracedP = PT == 1 || PT == 2 || PT == 4 || PT == 8;

template <int PT, int VPT>
static tw_status launch_t(const FusedParams &prm, bool trace, bool streamed, int64_t grid, int block, hipStream_t stream)
{
    void (*const plain)(FusedParams) = fused_kernel<PT, VPT, false, false>;
    void (*kern)(FusedParams) = streamed ? static_cast<void (*)(FusedParams)>(fused_kernel<PT, VPT, false, true>) : plain;
    if constexpr (PT <= 0 || kTracedP<PT>)
        if (trace) kern = fused_kernel<PT, VPT, true, false>;
    static std::atomic<int> allowed[4][kMaxDevices];  // a kernel each: plain, streamed, traced, with helpers
    if (grid > prm.n_groups) {
        void (*helped)(uint32_t, FusedParams) = fused_kernel<PT, VPT, false, false, uint32_t>;
        TW_TRY(allow_dynamic_lds(reinterpret_cast<const void *>(helped), static_cast<int>(kOccupancyPadBytes), allowed[3]));
        TW_HIP(launch_kernel(helped, dim3(static_cast<unsigned>(grid)), dim3(static_cast<unsigned>(block)), kOccupancyPadBytes,
                             stream, prm.n_groups, prm));
        return TW_OK;
    }
    TW_TRY(allow_dynamic_lds(reinterpret_cast<const void *>(kern), static_cast<int>(kOccupancyPadBytes),
                             allowed[kern == plain ? 0 : trace ? 2 : 1]));
    TW_HIP(launch_kernel(kern, dim3(static_cast<unsigned>(grid)), dim3(static_cast<unsigned>(block)),
                         kOccupancyPadBytes, stream, prm));
    return TW_OK;
}

template <int PT, int Q>
static tw_status launch_thin_t(const FusedParams &prm, bool trace, bool streamed, int64_t grid,
                               hipStream_t stream)
{
    auto kern = streamed ? fused_thin_kernel<PT, Q, false, true> : fused_thin_kernel<PT, Q, false, false>;
    if constexpr (PT <= 0 || kTracedP<PT>)
        if (trace) kern = fused_thin_kernel<PT, Q, true, false>;
    TW_HIP(launch_kernel(kern, dim3(static_cast<unsigned>(grid)), dim3(kThinThreads), 0u, stream, prm));
    return TW_OK;
}

template <int PT, int Q>
static tw_status launch_deep_t(const FusedParams &prm, int64_t grid, hipStream_t stream)
{
    if constexpr (PT > 0 && PT <= kDeepMaxP) {
        uint64_t t[kDeepMaxP + 2] = {};
        for (int i = 0; i < PT + 2; ++i)
            t[i] = reinterpret_cast<uint64_t>(i < PT ? prm.partials[i < PT ? i : 0] : i == PT ? prm.residual : prm.weight);
        DeepRest rest;
        for (int i = kDeepFirst; i < kDeepMaxP + 2; ++i) rest.tensor[i - kDeepFirst] = reinterpret_cast<const void *>(t[i]);
        rest.out = prm.out;
        rest.residual_out = prm.residual_out;
        rest.eps = prm.eps;
        rest.inv_h = prm.inv_h;
        const uint64_t shape = prm.n_bytes | uint64_t(prm.hv) << 32 | uint64_t(prm.tpr_log2) << 44 | uint64_t(prm.n_groups) << 48;
        TW_HIP(launch_kernel(fused_deep_kernel<PT, Q>, dim3(static_cast<unsigned>(grid)), dim3(kThinThreads), 0u, stream,
                             DeepFirst{t[0], t[1], t[2], shape}, rest));
        return TW_OK;
    }
    return TW_ERR_UNSUPPORTED;
}

// Calls f(integral_constant<int, P>) for P in 1 ... TW_MAX_P.
template <typename F, int... I>
static tw_status with_partials(int P, F &&f, std::integer_sequence<int, I...>)
{
    tw_status s = TW_ERR_UNSUPPORTED;
    (void)((P == I + 1 ? (s = f(std::integral_constant<int, I + 1>{}), true) : false) || ...);
    return s;
}
template <typename F>
static tw_status with_partials(int P, F &&f)
{
    return with_partials(P, static_cast<F &&>(f), std::make_integer_sequence<int, TW_MAX_P>{});
}

template <int PT>
static tw_status launch_thin(const FusedParams &prm, int q, bool trace, bool streamed, bool deep, int64_t grid,
                             hipStream_t s)
{
    if (deep) {
        switch (q) {
        case 1: return launch_deep_t<PT, 1>(prm, grid, s);
        case 2: return launch_deep_t<PT, 2>(prm, grid, s);
        case 3: return launch_deep_t<PT, 3>(prm, grid, s);
        case 4: return launch_deep_t<PT, 4>(prm, grid, s);
        }
        return TW_ERR_UNSUPPORTED;
    }
    switch (q) {
    case 1: return launch_thin_t<PT, 1>(prm, trace, streamed, grid, s);
    case 2: return launch_thin_t<PT, 2>(prm, trace, streamed, grid, s);
    case 3: return launch_thin_t<PT, 3>(prm, trace, streamed, grid, s);
    case 4: return launch_thin_t<PT, 4>(prm, trace, streamed, grid, s);
    }
    return TW_ERR_UNSUPPORTED;
}

// Geometry of the shared (co-resident) mode: 256-thread workgroups, each striding
// over up to eight row groups; enough workgroups that the hardware dispatcher
// balances them over compute units that are busy to different degrees.
struct ThinGeometry {
    int q;              // wide-kernel threads played by one thread (1 ... 4)
    int rows_per_iter;  // rows per row group
};
static ThinGeometry thin_geometry(const FusedGeometry &g)
{
    ThinGeometry t;
    const int tpr = 1 << g.tpr_log2;
    t.q = g.hv > kThinThreads ? (g.hv + kThinThreads - 1) / kThinThreads : 1;
    t.rows_per_iter = tpr >= kThinThreads ? 1 : kThinThreads / tpr;
    return t;
}
static int64_t thin_grid(int64_t n_rows, const ThinGeometry &t, int cus)
{
    const int64_t n_groups = (n_rows + t.rows_per_iter - 1) / t.rows_per_iter;
    int64_t gpw = n_groups / (int64_t(8) * cus);  // row groups per workgroup
    gpw = gpw < 1 ? 1 : gpw > 8 ? 8 : gpw;
    return (n_groups + gpw - 1) / gpw;
}

// Whether a row of VPT vectors per thread and one chunk of PT partials fit the 128 registers of
// a 1024-thread workgroup; where they do not, the run-time loop over P (four loads at a time,
// same order of additions) does.
static constexpr bool wide_fits(int P, int vpt)
{
    return P <= 0 || vpt == 1 || (vpt <= 4 ? P <= 8 : P == 1 || P == 2 || P == 4);
}
template <int PT, int VPT>
static constexpr bool wide_fits()
{
    return wide_fits(PT, VPT);
}

// Where the run-time loop over P is ahead of the kernel made for the P at hand. That one asks
// for all P + 1 vectors of a chunk at once, which pays while a workgroup goes through row after
// row; but its way to the first load is longer (from P = 12 on up to nineteen descriptors do
// not fit the scalar registers, and the small workgroups with 768 vectors a row and more spill
// 100 to 190 of them, at P = 15 and 16 vector registers too). The loop goes through the
// partials a few at a time. Measured on MI355X, launches on rotating buffers.
//
// Wide kernel, loop against instance (tensor_bytes: size of one tensor):
//   - one row group per workgroup: over before anything is pipelined (whole device, P = 3 to 16,
//     512 to 8192 elements: the loop is ahead by 1 to 16 % where half of the device is filled, by 1
//     to 8 % where all of it is; rows of two vectors and more per thread: level to 6 % behind);
//   - rows of one wave and less, from P = 10 on: 3 to 20 %;
//   - from P = 12 on up to two trips, from P = 15 on four: level to 8 %;
//   - many compute units on tensors of 4, 8 or 16 MiB: such tensors lie a power of two apart,
//     and workgroups in step that ask for P + 1 of them at once meet in the same memory
//     channels. 64 compute units, 256 rows of 8192 elements, P = 12: 24.4 us against 27.2, P =
//     16: 29.4 against 34.4 (192 rows: 18.8 against 19.2 and 22.8 against 23.0); all, 4096 rows of
//     2048, P = 7: 31.3 against 34.2, P = 16: 54.8 against 58.6. It fades with the number of
//     trips (64 compute units, 512 rows of 8192, P = 12: 46.6 against 47.7) and with fewer
//     compute units (32, 256 rows of 8192, P = 8 to 14: the loop is 4 to 16 % behind); on 32 and
//     64 MiB either is up to 9 % ahead, from one allocation to another.
static bool wide_loops(int P, const FusedGeometry &g, int64_t grid, uint32_t n_groups, int64_t tensor_bytes)
{
    if (P < 3 || g.vpt != 1) return false;
    if (n_groups <= grid) return true;
    if (P >= 10 && g.wpr == 0) return true;
    if (P >= 12 && n_groups <= grid * (P >= 15 ? 4 : 2)) return true;
    const bool same_channels =
        tensor_bytes >= 4 << 20 && tensor_bytes <= 16 << 20 && (tensor_bytes & (tensor_bytes - 1)) == 0;
    return same_channels && grid >= 64 && P >= (grid >= 256 ? 7 : 10) && n_groups <= grid * (grid / (P >= 12 ? 8 : 16));
}

// The small workgroups, likewise (vectors: of one tensor, over the device's compute units). Rows
// of 256 vectors and fewer, P = 12 to 16: 3 to 10 % (shared mode, 2048 rows of 2048 elements, P =
// 16: 30.7 us against 34.1); wider ones from P = 15 on 3 to 6 % (512 rows of 8192, P = 16: 27.0
// against 28.2), and fewer rows than that 11 to 24 % the other way (one row's chain of round
// trips); at four rows of 8192 to a unit and more level to 6 % the other way.
static bool thin_loops(int P, const FusedGeometry &g, int64_t n_rows, int cus)
{
    const int64_t vectors = n_rows * g.hv;
    const bool narrow = g.hv <= 2 * kThinThreads;
    return P >= (g.hv <= kThinThreads ? 12 : 15) && vectors > int64_t(narrow ? 512 : 1024) * cus &&
           vectors <= int64_t(narrow ? 3072 : 4096) * cus;
}

template <int PT>
static tw_status launch_vpt(const FusedParams &prm, const FusedGeometry &g, bool trace, bool streamed, int64_t grid,
                            hipStream_t s)
{
    switch (g.vpt) {
    case 1: return launch_t<PT, 1>(prm, trace, streamed, grid, g.block, s);
    case 2:
        if constexpr (wide_fits<PT, 2>()) return launch_t<PT, 2>(prm, trace, streamed, grid, g.block, s);
        break;
    case 4:
        if constexpr (wide_fits<PT, 4>()) return launch_t<PT, 4>(prm, trace, streamed, grid, g.block, s);
        break;
    case 8:
        if constexpr (wide_fits<PT, 8>()) return launch_t<PT, 8>(prm, trace, streamed, grid, g.block, s);
        break;
    }
    return TW_ERR_UNSUPPORTED;
}

// Which kernel a launch takes. Shared mode has a kernel for rows of up to 1024 vectors; wider
// rows run on the wide kernel over the whole device. Of a whole-device launch either kernel may
// be the faster one, with the same bits. The small workgroups are placed as compute units fall
// free and have every row in flight at once; the wide kernel works in trips of a row group per
// compute unit, its loads running ahead over the trips. So a last trip that leaves most compute
// units idle costs the wide kernel as much as a full one (2048 elements, P = 8: 1024 rows, one
// full trip, 9.3 us against 10.8 in small workgroups; 1075 rows, two trips, 13.3 against 10.1),
// full trips are its best case, and over many trips the last one no longer counts. Where it is
// taken, by row width and P, from 4300 sizes of 256 to 8192 elements and 51 to 65536 rows
// timed on MI355X in trains of launches on rotating buffers (the kernel chosen is 0.7 % off the
// faster one on average; one number of vectors per compute unit for each kind of row, without a
// look at trips, was 3 % off, and up to 25 % where trips are full):
struct WideFrom {
    int one;   // percent of the compute units that a single trip has to fill
    int full;  // trips, the last of them 92 % full or more
    int any;   // trips, whatever the last one
};
static constexpr int kNever = 1 << 20;
static constexpr WideFrom kWideFrom[5][5] = {
    // P = 1, 2           3, 4                   5 to 8              9 to 11               12 to 16
    {{kNever, kNever, 17}, {85, kNever, 17}, {70, 2, 6}, {85, 2, 6}, {85, 2, 5}},        // rows of up to 64 vectors
    {{kNever, 2, 6}, {85, 2, 6}, {70, 2, 6}, {85, 2, 5}, {85, 2, 5}},                    // 256
    {{kNever, 3, 6}, {kNever, kNever, 9}, {55, kNever, 17}, {55, 3, 6}, {55, 3, 6}},     // 512
    {{kNever, kNever, 7}, {kNever, kNever, 9}, {kNever, kNever, 17}, {kNever, kNever, 13}, {0, kNever, 9}},  // 768
    {{kNever, 4, 6}, {kNever, kNever, 17}, {kNever, kNever, 33}, {kNever, kNever, 33}, {0, 4, 6}},           // 1024
};
static bool takes_thin_kernel(int cu_budget, int cus, const FusedGeometry &g, int64_t n_rows, int P)
{
    if (g.vpt != 1) return false;
    if (cu_budget == TW_CU_SHARED) return true;
    if (resolve_budget(cu_budget, cus) != cus) return false;
    const int width = g.hv <= 64 ? 0 : (g.hv + kThinThreads - 1) / kThinThreads;
    // Few wide rows of more than eight partials: one chunk of registers after another in a thin
    // workgroup, where the wide kernel's waves have one each (64 rows of 8192 elements: P = 12
    // 7.8 us against 6.8, P = 16 9.4 against 8.2).
    if (P > 8 && P < 12 && width >= 3 && n_rows <= cus / 4) return false;
    const WideFrom &w = kWideFrom[width][P <= 2 ? 0 : P <= 4 ? 1 : P <= 8 ? 2 : P <= 11 ? 3 : 4];
    const int64_t groups = (n_rows + g.rows_per_iter - 1) / g.rows_per_iter, trips = (groups + cus - 1) / cus;
    if (trips <= 1) return groups * 100 < int64_t(w.one) * cus;
    return trips < w.any && (trips < w.full || groups * 100 < 92 * trips * cus);
}

// Workgroups of a launch in which each of the n_groups row groups has a workgroup of `waves` waves
// of its own, helpers included (see help()). They are taken where the row groups and all their
// helpers have a compute unit each, and a group's lines are more than a unit can have outstanding.
// Measured on MI355X, us without / with in replayed trains, inputs from HBM: 8192 elements, P = 8: 1 row
// 4.66 / 4.28, 16 rows 5.5 / 4.8, 32 rows 5.9 / 5.1 (from the cache 3.98 / 3.88); past the rule, with an earlier
// form of the kernel, 42 rows 6.22 / 6.12, 64 6.0 / 6.7, 128 7.2 / 8.3. P = 16: 16 rows 7.5 / 6.0, 64 rows 8.3 /
// 7.1 (100 rows, P = 12 7.9 / 8.4); 16384 elements, P = 8: 16 rows 8.6 / 6.9; 512 elements, P = 4, 4 rows, 20 KiB:
// 1.80 / 1.85. (More than one load to a wave, for fewer helpers: 2 to 20 % slower.)
// Calls that put another kernel beside the step have none (fused_grid). Beside a GEMM that a caller put on
// another stream by hand, which no call can know, a launch has to wait until each of its helpers found room: none in
// small workgroups (16 rows of 8192, P = 8, one step at a time beside 2048 x 8192 x 3584 products 25.0 / 23.8), but the
// wide kernel's each take a whole compute unit (P = 16: 54 / 81; 22 before the GEMM had helpers on the units it leaves
// idle). cu_budget, of either call, is for that.
static int64_t grid_with_helpers(uint32_t n_groups, uint32_t group_bytes, int P, int waves, int cus)
{
    if (group_bytes * (P + 1ll) <= 20 * 1024) return n_groups;
    const int64_t shares = (helper_pieces(group_bytes, P) + waves - 1) / waves;
    const int64_t grid = helper_base(n_groups) * (1 + shares);
    return grid <= cus ? grid : n_groups;
}

// What one launch for n_rows rows consists of.
struct FusedGrid {
    int rows_per_group;
    uint32_t n_groups;
    int64_t workers;  // workgroups that work on row groups
    int64_t all;      // and helpers with them (the same where there are none)
    bool deep;        // thin_body's DEEP form
};
static FusedGrid fused_grid(const tw_fused_args &a, const FusedGeometry &g, bool thin, int64_t n_rows, int cus, FusedPlace place,
                            bool trace)
{
    FusedGrid f = {};
    const ThinGeometry tg = thin_geometry(g);
    const int budget = resolve_budget(a.cu_budget, cus);
    f.rows_per_group = thin ? tg.rows_per_iter : g.rows_per_iter;
    f.n_groups = static_cast<uint32_t>((n_rows + f.rows_per_group - 1) / f.rows_per_group);
    f.workers = thin ? thin_grid(n_rows, tg, cus) : fused_grid_size(n_rows, g, budget);
    // one row group per workgroup, at most one workgroup per compute unit, few bytes: the launch is
    // latency-bound, everything is requested at once. Not in shared mode, whose workgroups must fit
    // beside a GEMM's.
    const bool one_each = f.workers == f.n_groups, shared = a.cu_budget == TW_CU_SHARED;
    f.deep = thin && !trace && !shared && a.P <= kDeepMaxP && one_each && f.n_groups <= uint32_t(cus) &&
             n_rows * a.H * 2 * (a.P + 1) <= kDeepInputBytes;
    f.all = f.workers;
    // (the helpers' compute units are idle only if nothing else is meant to run on them)
    if (place == FusedPlace::kAlone && !shared && (f.deep || (!thin && !trace && budget == cus && one_each)))
        f.all = grid_with_helpers(f.n_groups, static_cast<uint32_t>(f.rows_per_group * a.H * 2), a.P,
                                  thin ? kThinThreads / 64 : g.block / 64, cus);
    return f;
}

// Rows a launch addresses (kMaxLaunchBytes per tensor); more go out as consecutive launches on the
// same stream.
static int64_t rows_per_launch(int64_t H, const FusedGeometry &g)
{
    const int64_t rows = kMaxLaunchBytes / (H * 2);
    return rows - rows % g.rows_per_iter;
}

tw_status launch_fused(const tw_fused_args &a, int64_t row_begin, int64_t row_end, uint32_t *hw_ids,
                       int64_t hw_ids_len, hipStream_t stream, FusedPlace place)
{
    if (row_end <= row_begin) return TW_OK;
    int cus = 0;
    TW_TRY(current_cu_count(&cus));
    const FusedGeometry g = fused_geometry(a.H);
    const int budget = resolve_budget(a.cu_budget, cus);
    const bool trace = hw_ids != nullptr;

    const int64_t row_bytes = a.H * 2, most_rows = rows_per_launch(a.H, g);
    if (trace && row_end - row_begin > most_rows) return TW_ERR_UNSUPPORTED;
    const bool thin = takes_thin_kernel(a.cu_budget, cus, g, row_end - row_begin, a.P);
    // outputs that do not fit the last-level cache are stored with the streaming policy (see st());
    // not under a CU budget, where that is 1 % slower
    const bool streamed = 2 * (row_end - row_begin) * row_bytes >= kLastLevelCacheBytes && (thin || budget == cus);
    const int q = thin_geometry(g).q;

    for (int64_t r0 = row_begin; r0 < row_end; r0 += most_rows) {
        const int64_t n_rows = (row_end - r0 < most_rows) ? row_end - r0 : most_rows;
        const FusedGrid f = fused_grid(a, g, thin, n_rows, cus, place, trace);
        if (!thin && f.workers > 1024) return TW_ERR_UNSUPPORTED;  // (no device has as many compute units)
        if (trace && hw_ids_len < f.workers) return TW_ERR_SHAPE;

        FusedParams prm;
        const int64_t off = r0 * row_bytes;
        for (int p = 0; p < TW_MAX_P; ++p)
            prm.partials[p] = p < a.P ? static_cast<const char *>(a.partials[p]) + off : nullptr;
        prm.residual = static_cast<const char *>(a.residual) + off;
        prm.weight = a.weight;
        prm.out = static_cast<char *>(a.out) + off;
        prm.residual_out = static_cast<char *>(a.residual_out) + off;
        prm.hw_ids = hw_ids;
        prm.n_bytes = static_cast<uint32_t>(n_rows * row_bytes);
        prm.group_bytes = static_cast<uint32_t>(f.rows_per_group * row_bytes);
        prm.n_groups = f.n_groups;
        prm.hv = g.hv;
        prm.P = a.P;
        prm.tpr_log2 = g.tpr_log2;
        prm.wpr = g.wpr;
        prm.eps = a.eps;
        prm.inv_h = 1.0f / static_cast<float>(a.H);

        // the run-time loop over P: where it is faster, no specialised kernel has the registers, or none is built to be traced
        const bool traced_p = a.P == 1 || a.P == 2 || a.P == 4 || a.P == 8;
        const bool any_p = (trace && !traced_p) ||
                           (thin ? thin_loops(a.P, g, row_end - row_begin, cus)
                                 : !wide_fits(a.P, g.vpt) || wide_loops(a.P, g, f.workers, f.n_groups, a.N * row_bytes));
        if (thin) {
            if (any_p) TW_TRY((launch_thin<kAnyPadded>(prm, q, trace, streamed, false, f.all, stream)));
            else
                TW_TRY(with_partials(a.P, [&](auto pt) {
                    return launch_thin<decltype(pt)::value>(prm, q, trace, streamed, f.deep, f.all, stream);
                }));
        } else {
            if (any_p && a.P % kWideBatch == 0) TW_TRY((launch_vpt<kAnyWhole>(prm, g, trace, streamed, f.all, stream)));
            else if (any_p) TW_TRY((launch_vpt<kAnyPadded>(prm, g, trace, streamed, f.all, stream)));
            else
                TW_TRY(with_partials(a.P, [&](auto pt) {
                    return launch_vpt<decltype(pt)::value>(prm, g, trace, streamed, f.all, stream);
                }));
        }
    }
    return TW_OK;
}

}  // namespace tw

using namespace tw;

extern "C" {

tw_status tw_reduce_add_rmsnorm(const void *const *partials, const void *residual,
                                const void *weight, float eps, int64_t N, int64_t H, int P,
                                int cu_budget, void *out, void *residual_out, void *stream)
{
    const tw_fused_args a = {partials, residual, weight, eps, N, H, P, cu_budget, out, residual_out};
    TW_TRY(validate_fused(a));
    return launch_fused(a, 0, N, nullptr, 0, static_cast<hipStream_t>(stream));
}

tw_status tw_reduce_add_rmsnorm_traced(const void *const *partials, const void *residual,
                                       const void *weight, float eps, int64_t N, int64_t H, int P,
                                       int cu_budget, void *out, void *residual_out,
                                       uint32_t *hw_ids, int64_t hw_ids_len, void *stream)
{
    const tw_fused_args a = {partials, residual, weight, eps, N, H, P, cu_budget, out, residual_out};
    TW_TRY(validate_fused(a));
    if (!hw_ids) return TW_ERR_NULL;
    if (hw_ids_len < 0) return TW_ERR_SHAPE;
    return launch_fused(a, 0, N, hw_ids, hw_ids_len, static_cast<hipStream_t>(stream));
}

tw_status tw_fused_layout(int64_t H, int *waves_per_row, int *vectors_per_thread, int *rows_per_trip,
                          int *threads_per_workgroup)
{
    if (H <= 0) return TW_ERR_SHAPE;
    if (H % 8 != 0 || H > TW_MAX_H) return TW_ERR_UNSUPPORTED;
    const FusedGeometry g = fused_geometry(H);
    if (waves_per_row) *waves_per_row = g.wpr;
    if (vectors_per_thread) *vectors_per_thread = g.vpt;
    if (rows_per_trip) *rows_per_trip = g.rows_per_iter;
    if (threads_per_workgroup) *threads_per_workgroup = g.block;
    return TW_OK;
}

int64_t tw_fused_grid(int64_t N, int64_t H, int P, int cu_budget)
{
    if (N < 0 || H <= 0 || H % 8 != 0 || H > TW_MAX_H || P < 1 || P > TW_MAX_P) return -1;
    if (N == 0) return 0;
    int cus = 0;
    if (current_cu_count(&cus) != TW_OK) return -1;
    const FusedGeometry g = fused_geometry(H);
    if (takes_thin_kernel(cu_budget, cus, g, N, P) && N * H * 2 <= kMaxLaunchBytes) {
        return thin_grid(N, thin_geometry(g), cus);
    }
    return fused_grid_size(N, g, resolve_budget(cu_budget, cus));
}

tw_status tw_fused_workgroups(int64_t N, int64_t H, int P, int cu_budget, int cus, int beside_other_kernels, int64_t *workers,
                              int64_t *helpers)
{
    if (N < 0 || H <= 0 || P < 1 || P > TW_MAX_P || cus < 1) return TW_ERR_SHAPE;
    if (H % 8 != 0 || H > TW_MAX_H) return TW_ERR_UNSUPPORTED;
    FusedGrid f = {};
    if (N > 0) {
        tw_fused_args a = {};
        a.N = N;
        a.H = H;
        a.P = P;
        a.cu_budget = cu_budget;
        const FusedGeometry g = fused_geometry(H);
        const int64_t most_rows = rows_per_launch(H, g);
        f = fused_grid(a, g, takes_thin_kernel(cu_budget, cus, g, N, P), N < most_rows ? N : most_rows, cus,
                       beside_other_kernels ? FusedPlace::kBeside : FusedPlace::kAlone, false);
    }
    if (workers) *workers = f.workers;
    if (helpers) *helpers = f.all - f.workers;
    return TW_OK;
}

}  // extern "C"
