// Reductions over a wavefront and over the bytes of a word (included inside the
// kernels' namespaces).
#pragma once

// Sum over the 64 lanes, the same in every lane: prefix sums inside the rows of
// 16 lanes, then across rows, by data-parallel moves that are part of the
// additions (an exchange through LDS per step, as __shfl_xor makes, costs a
// step ~100 cycles of latency: a launch's closing reduction 0.9 us).  All
// lanes take part.
template <int CTRL, int ROWS>
__device__ __forceinline__ int add_dpp(int v)
{
    return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, ROWS == 0xF);
}

__device__ __forceinline__ int wave_sum(int v)
{
    v = add_dpp<0x111, 0xF>(v);      // row_shr:1
    v = add_dpp<0x112, 0xF>(v);      // row_shr:2
    v = add_dpp<0x114, 0xF>(v);      // row_shr:4
    v = add_dpp<0x118, 0xF>(v);      // row_shr:8: lane 15 of a row holds its sum
    v = add_dpp<0x142, 0xA>(v);      // row_bcast:15 into rows 1 and 3
    v = add_dpp<0x143, 0xC>(v);      // row_bcast:31 into rows 2 and 3
    return __builtin_amdgcn_readlane(v, 63);
}

// Exclusive prefix sum over the wavefront of per-lane values c < 32, and
// its total: one ballot per bit.
__device__ __forceinline__ uint32_t wave_excl_scan5(uint32_t c, uint32_t& total)
{
    uint32_t pre = 0, tot = 0;
#pragma unroll
    for (uint32_t b = 0; b < 5; ++b) {
        const uint64_t m = __ballot((c >> b) & 1u);
        pre += __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)) << b;
        tot += (uint32_t)__popcll(m) << b;
    }
    total = tot;
    return pre;
}

// 0x01 in every zero byte of x, 0x00 elsewhere (no carry crosses a byte).
__device__ __forceinline__ uint32_t zero_bytes(uint32_t x)
{
    return (~(((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x | 0x7F7F7F7Fu)) >> 7;
}
