// What the GEMM kernels share: operand vectors for the matrix cores, LDS reads with
// waits placed by hand, and the walk over output tiles.
#pragma once

#include <stdint.h>

#include <type_traits>
#include <utility>

#include "tw_device.h"

namespace tw {

static constexpr int kXcds = 8;
static constexpr int kBlk = 16;   // rows and columns of one MFMA result block
static constexpr int kSubK = 32;  // K depth of one MFMA

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

typedef __attribute__((address_space(3))) void *lds_ptr_t;
typedef __attribute__((address_space(3))) char *lds_char_ptr_t;

template <int OFF>
__device__ __forceinline__ bf16x8 lds_read16(uint32_t addr)
{
    bf16x8 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
    return v;
}
// gfx950's transposing LDS read. Within each group of 16 lanes, lane 4a+b
// receives, for j = 0..3, the b-th 16-bit element of the 8-byte chunk that lane
// a + 4j points at (lane mapping established with a probe kernel). With lane
// a + 4j pointing at row k0+j, columns 4a..4a+3 of a [k][n] tile, lane d = 4a+b
// ends up with column d of rows k0..k0+3: four consecutive k of one n, which is
// what an MFMA operand register pair holds.
template <int OFF>
__device__ __forceinline__ u32x2 lds_read_tr8(uint32_t addr)
{
    u32x2 v;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
    return v;
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>), unrolled
template <int... I, typename Fn>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, Fn &&f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename Fn>
__device__ __forceinline__ void static_for(Fn &&f)
{
    static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// Tile `lin` of a list ordered in blocks of group_m tile rows, column after column.
struct TileAt {
    int m, n;
};
__device__ __forceinline__ TileAt tile_at(int lin, int tiles_m, int tiles_n, int group_m)
{
    // (a division by a number that is not a constant is a chain of some forty instructions,
    // ahead of a tile's first load: branches spare the ones that few rows of tiles do not need)
    int in_grp = lin, first_tm = 0;
    if (tiles_m > group_m) {
        const int per_group = group_m * tiles_n;
        const int grp = lin / per_group;
        first_tm = grp * group_m;
        in_grp = lin - grp * per_group;
    }
    const int gsz = min(group_m, tiles_m - first_tm);
    if (gsz == 1) return {first_tm, in_grp};
    const int n = in_grp / gsz;
    return {first_tm + in_grp - n * gsz, n};
}

}  // namespace tw
