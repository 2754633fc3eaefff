// Arm-domain Metropolis pass kernels (included inside the kernels'
// namespace, after the checkerboard sweep, whose one-arm move, table and
// reduction they share).
#pragma once

// ---------------------------------------------------------------------------
// The paper's own parallel partition (Sec. II.C and its figure of layered
// domains), in 2-D: arm a of every cell forms a domain.  A bond index of arm
// a interacts with the three other arms of its cell and with arm a^1 of the
// neighbour in direction a -- none of them in the domain -- so the whole
// domain moves at once, for any L (odd included).  A sweep is four passes,
// one per arm, in an order drawn per step.
//
// Two passes in a row whose arms are not opposite share a launch: the second
// arm's move needs the first one only within its own cell, and neither faces
// the other.  Two orders in three are two such pairs (their third launch is
// empty), the others are one arm, two arms, one arm: three launches instead
// of four.  The launches are short -- a pass took 7.9 us at L = 1025, against
// about 4.8 us for the shortest back-to-back launch -- so their number counts.
// A sweep, with single-arm launches on column pairs (quads at L % 4 == 0) of
// one row per wavefront before: L = 64 20.8 -> 11.8 us, L = 1025 34.8 -> 20.3,
// L = 1024 25.6 -> 17.3, L = 2047 68.2 -> 37.4, L = 4096 102.1 -> 94.1, there
// bound by one Philox block per two moves.
//
// Work layout: a lane owns the quad of columns 4j..4j+3 of `rows` rows (the
// last quad of a row may hold fewer), and a wavefront 64 quads in a row,
// across the ends of lattice rows, so that a row length just above a multiple
// of 256 leaves no wavefront idle.  Two Philox blocks per quad, row and arm,
// one for each column pair: words 0, 1 (proposal, acceptance) for its even
// column, 2, 3 for the odd one.  Per row and lane: four dwords (rows start at
// any address), the facing row's dword, one facing byte, one dword store per
// moved plane.
// ---------------------------------------------------------------------------

// The arms of the sweep at step t in their drawn order, one per nibble: Fisher-Yates on the words of
// Philox(0, t, 0, ORD), position i swapping with i + pick(w_i, 4 - i); pick
// for k = 4 and 2 is a shift, for k = 3 it is w / floor(2^32/3) with the
// NONE draw w = 2^32 - 1 keeping position 1.  The order lives in the nibbles
// of one register.
__device__ __forceinline__ uint32_t domain_order(const LatticeArgs& a, uint32_t t)
{
    const uint4 w = philox(0u, t, 0u, kStreamOrd, a.key0, a.key1);
    uint32_t ord = 0x3210u;
    auto swap = [&ord](uint32_t i, uint32_t j) {
        const uint32_t vi = (ord >> (4 * i)) & 15u, vj = (ord >> (4 * j)) & 15u;
        ord &= ~((15u << (4 * i)) | (15u << (4 * j)));
        ord |= (vj << (4 * i)) | (vi << (4 * j));
    };
    swap(0, w.x >> 30);
    swap(1, 1 + (w.y == 0xFFFFFFFFu ? 0u : w.y / 1431655765u));
    swap(2, 2 + (w.z >> 31));
    return ord;
}

// The n bytes of the quad at column x (offset o of its row, plane offset po)
// of a plane, in the low bytes, zeros above.  RAG: L % 4 != 0, where the last
// quad of a row holds n < 4 columns: read as the row's last dword, shifted, so
// that no access leaves the row.  TINY: L < 4, single bytes.
template <int MODE>
__device__ __forceinline__ uint32_t dom_quad(__amdgpu_buffer_rsrc_t rs, uint32_t o, uint32_t x, uint32_t n, uint32_t po)
{
    if (MODE == 0) return ld32(rs, o + x, po);
    if (MODE == 1) return ld32(rs, o + x - (4 - n), po) >> (8 * (4 - n));
    uint32_t d = 0;
    for (uint32_t k = 0; k < n; ++k) d |= ld8(rs, o + x + k, po) << (8 * k);
    return d;
}

// One arm of the n cells of a quad: d0 the bytes of the moved plane, d1..d3
// of the other three and f of the facing arm, all holding sigma; returns the
// new bytes.  (RAG) moves of columns past the row's end are not counted.
template <int Q, bool RAG>
__device__ __forceinline__ uint32_t dom_move(uint32_t d0, uint32_t d1, uint32_t d2, uint32_t d3, uint32_t f, uint32_t n,
                                             const uint4& wa, const uint4& wb, const uint2* tbl, uint32_t& wsum)
{
    d0 <<= 2, d1 <<= 2, d2 <<= 2, d3 <<= 2, f <<= 2;
    uint32_t s[4], w[4] = {wsum, 0, 0, 0};
#define CVF_DOM_CELL(K, W0, W1)                                                                             \
    {                                                                                                       \
        s[K] = byte4<K>(d0);                                                                                \
        const uint32_t z = (1u << byte4<K>(d1)) + (1u << byte4<K>(d2)) + (1u << byte4<K>(d3)) +             \
                           (8u << byte4<K>(f));                                                             \
        met_arm<Q>(s[K], z, W0, W1, tbl, w[RAG ? K : 0]);                                                   \
    }
    CVF_DOM_CELL(0, wa.x, wa.y)
    CVF_DOM_CELL(1, wa.z, wa.w)
    CVF_DOM_CELL(2, wb.x, wb.y)
    CVF_DOM_CELL(3, wb.z, wb.w)
#undef CVF_DOM_CELL
    wsum = w[0];
    if (RAG) wsum += (n > 1 ? w[1] : 0u) + (n > 2 ? w[2] : 0u) + (n > 3 ? w[3] : 0u);
    return (s[0] >> 2) | ((s[1] >> 2) << 8) | ((s[2] >> 2) << 16) | ((s[3] >> 2) << 24);
}

template <bool RAG>
__device__ __forceinline__ void dom_store(__amdgpu_buffer_rsrc_t rs, uint32_t d, uint32_t voff, uint32_t n, uint32_t po)
{
    if (!RAG || n == 4) {
        st32(rs, d, voff, po);
    } else {
        st8(rs, d & 255u, voff, po);
        if (n > 1) st8(rs, (d >> 8) & 255u, voff + 1, po);
        if (n > 2) st8(rs, (d >> 16) & 255u, voff + 2, po);
    }
}

// MODE 0: L % 4 == 0; 1: other L > 4; 2: L = 2, 3.  Launch `group` 0..2.
template <int Q, int MODE>
__global__ __launch_bounds__(256) void met_domain_kernel(LatticeArgs a, VolArgs va, StepCtl ctl, uint32_t group,
                                                         uint32_t rows)
{
    if (ctl.open && blockIdx.x + 1 == gridDim.x) {
        __shared__ double term[40];
        if (threadIdx.x < 64) open_next(va, term, a.st->view + (ctl.bank ^ 1u));
        return;
    }
    StepView* view = a.st->view + ctl.bank;
    const int skip = view->skip;
    int theta = group == 0 ? view->theta : view->theta2;
    const uint32_t t = view->t_cur;
    if (skip) return;                                      // step limit reached
    if (group == 0 && view->pending) theta = resolve_step(va, view, false, blockIdx.x == 0);
    __shared__ uint2 tbl[32];
    const uint32_t ord = __builtin_amdgcn_readfirstlane(domain_order(a, t));
    // Arms A and B of this launch.  Planes A, B, A^1, B^1 are all four: where
    // only A moves, B is any arm that is not opposite to it.
    const bool split = ((ord ^ (ord >> 4)) & 15u) == 1;    // the first two arms are opposite: 1 + 2 + 1
    const uint32_t at = split ? (group == 0 ? 0u : group == 1 ? 1u : 3u) : 2 * group;
    const bool two = split ? group == 1 : true;
    if (at > 3) return;                                    // 2 + 2: the third launch is empty
    const uint32_t A = (ord >> (4 * at)) & 3u, B = two ? (ord >> (4 * at + 4)) & 3u : A ^ 2u;
    constexpr bool RAG = MODE != 0;
    const uint32_t L = a.L, N = a.N, np = (L + 1) >> 1, quads = (L + 3) >> 2;
    const uint32_t unit = blockIdx.x * 256 + threadIdx.x, band = unit / quads, j = unit - band * quads;
    met_table(a, tbl, theta);
    uint32_t wsum = 0;
    const uint32_t x = 4 * j, n = RAG ? min(4u, L - x) : 4u;
    const uint32_t y0 = band * rows, y1 = min(y0 + rows, L);
    // one of A, B is an x arm (0, 1), the other a y arm (2, 3)
    const bool ax = A < 2;
    const uint32_t X = ax ? A : B, Y = ax ? B : A;
    const uint32_t pa = A * N, pb = B * N, pc = (A ^ 1u) * N, pd = (B ^ 1u) * N;
    const uint32_t xe = X == 0 ? (x + n == L ? 0u : x + n) : (x == 0 ? L - 1 : x - 1);   // column beside the quad
    const __amdgpu_buffer_rsrc_t rs = sigma_rsrc(a.sigma, 4 * N);
    for (uint32_t y = y0; y < y1; ++y) {
        const uint32_t o = y * L;
        const uint32_t fy = Y == 2 ? (y + 1 == L ? 0u : y + 1) : (y == 0 ? L - 1 : y - 1);
        const uint32_t da = dom_quad<MODE>(rs, o, x, n, pa), db = dom_quad<MODE>(rs, o, x, n, pb),
                       dc = dom_quad<MODE>(rs, o, x, n, pc), dd = dom_quad<MODE>(rs, o, x, n, pd);
        const uint32_t e = ld8(rs, o + xe, (X ^ 1u) * N);
        const uint32_t fv = dom_quad<MODE>(rs, fy * L, x, n, (Y ^ 1u) * N);
        const uint32_t own = ax ? dc : dd;                 // plane X ^ 1, this row
        const uint32_t fh = X == 0 ? (own >> 8) | (e << (8 * (n - 1))) : (own << 8) | e;
        const uint32_t blk = x / 2 + np * y;
        uint4 wa = philox(blk, t, A, kStreamDom, a.key0, a.key1);
        uint4 wb = philox(blk + 1, t, A, kStreamDom, a.key0, a.key1);
        const uint32_t na = dom_move<Q, RAG>(da, db, dc, dd, ax ? fh : fv, n, wa, wb, tbl, wsum);
        dom_store<RAG>(rs, na, o + x, n, pa);
        if (two) {
            wa = philox(blk, t, B, kStreamDom, a.key0, a.key1);
            wb = philox(blk + 1, t, B, kStreamDom, a.key0, a.key1);
            const uint32_t nb = dom_move<Q, RAG>(db, na, dc, dd, ax ? fv : fh, n, wa, wb, tbl, wsum);
            dom_store<RAG>(rs, nb, o + x, n, pb);
        }
    }
    met_reduce(wsum, a.slots + (group ? kBankSlots : 0), blockIdx.x);
}
