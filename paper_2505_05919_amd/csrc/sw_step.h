// Swendsen-Wang step kernels (included inside the kernels' namespace).  The step kernels work on kTW x kTH-cell tiles; each
// has a body shared by the single-chain kernel (grid = the chain's tiles) and
// the batched kernel (workgroup -> chain and tile through prefix sums).
#pragma once

// ---------------------------------------------------------------------------
// Swendsen-Wang (Sec. II.D).
// Bond mask per cell: bit 0 covalent +x (arm 0 of c, arm 1 of c+x), bit 1
// covalent +y (arm 2 of c, arm 3 of c+y), bits 2..7 cooperative pairs
// (0,1) (0,2) (0,3) (1,2) (1,3) (2,3).  Link l uses word l of
// Philox(c, t, 0, SWB) for l < 4 and word l-4 of Philox(c, t, 1, SWB).
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool below(uint32_t w, uint64_t thr) { return (uint64_t)w < thr; }

// In-cell components of the 4 arms for each of the 64 cooperative masks:
// 2 bits per arm = smallest arm index of its component.
__device__ void build_incell_lut(uint8_t* lut)
{
    const int pa[6] = {0, 0, 0, 1, 1, 2}, pb[6] = {1, 2, 3, 2, 3, 3};
    if (threadIdx.x < 64) {
        const int m = threadIdx.x;
        int lab[4] = {0, 1, 2, 3};
        for (int it = 0; it < 3; ++it)
            for (int l = 0; l < 6; ++l)
                if (m >> l & 1) {
                    const int mn = min(lab[pa[l]], lab[pb[l]]);
                    lab[pa[l]] = mn;
                    lab[pb[l]] = mn;
                }
        lut[m] = (uint8_t)(lab[0] | lab[1] << 2 | lab[2] << 4 | lab[3] << 6);
    }
}

struct SwBondCtx {
    uint32_t t;
    uint64_t thr_s, thr_e;
    bool cov_on;
};

__device__ __forceinline__ SwBondCtx sw_ctx(const LatticeArgs& a, uint32_t t, int theta)
{
    SwBondCtx k;
    k.t = t;
    k.thr_s = a.tab->sw[0];
    k.thr_e = a.tab->sw[1 + theta];
    k.cov_on = theta == 1 && a.jeff_sign != 0;
    return k;
}

// Bond activation of cell c (link mask): s0..s3 its bond indices, f0 / f2
// the facing arms of its arms 0 and 2 (arm 1 of the +x neighbour, arm 3 of
// the +y neighbour).
__device__ __forceinline__ uint32_t sw_bond_bits(const LatticeArgs& a, const SwBondCtx& k, uint32_t c, uint32_t s0,
                                                 uint32_t s1, uint32_t s2, uint32_t s3, uint32_t f0, uint32_t f2)
{
    const uint4 w0 = philox(c, k.t, 0u, kStreamSwb, a.key0, a.key1);
    const uint4 w1 = philox(c, k.t, 1u, kStreamSwb, a.key0, a.key1);
    uint32_t m = 0;
    if (k.cov_on) {
        const bool e0 = (s0 == f0) == (a.jeff_sign > 0);
        const bool e2 = (s2 == f2) == (a.jeff_sign > 0);
        m |= (e0 && below(w0.x, k.thr_e)) ? 1u : 0u;
        m |= (e2 && below(w0.y, k.thr_e)) ? 2u : 0u;
    }
    m |= (s0 == s1 && below(w0.z, k.thr_s)) ? 4u : 0u;
    m |= (s0 == s2 && below(w0.w, k.thr_s)) ? 8u : 0u;
    m |= (s0 == s3 && below(w1.x, k.thr_s)) ? 16u : 0u;
    m |= (s1 == s2 && below(w1.y, k.thr_s)) ? 32u : 0u;
    m |= (s1 == s3 && below(w1.z, k.thr_s)) ? 64u : 0u;
    m |= (s2 == s3 && below(w1.w, k.thr_s)) ? 128u : 0u;
    return m;
}

// Root of x: follow parents until a self-loop.  label[x] <= x everywhere, so
// the chain strictly decreases and ends.
__device__ __forceinline__ uint32_t find_root(const uint32_t* label, uint32_t x)
{
    uint32_t p = label[x];
    while (p != x) {
        x = p;
        p = label[x];
    }
    return x;
}

// ---------------------------------------------------------------------------
// Tiled Swendsen-Wang step.  A workgroup of kTT threads owns a tile of kTW x
// kTH cells, i.e.
// 4 kTC bond indices with local index v = arm * kTC + ly * kTW + lx, whose
// order is the order of the global flat indices arm * N + y * L + x.
//  sw_tile_kernel         bonds of the tile's cells (mask) and the in-tile
//                         unions in LDS; global labels only where the
//                         tile-crossing links can reach them: border bond
//                         indices (-> their tile root) and the roots of the
//                         components holding one (-> themselves); the old
//                         sigma facing the right and bottom edges; every
//                         bond index's tile-local root (uint16, with the
//                         border flag of its component); then the tile-
//                         crossing links, each united (global union-find)
//                         by the later of the two tiles it joins.
//  sw_flip_tile_kernel    one shift per tile-local component (its cluster
//                         minimum comes from the global labels if the
//                         component touches the border, else it is the
//                         component's own minimum), shifts sigma and
//                         recounts N_HB_raw and N_sigma of the new
//                         configuration.
//  sw_labels_kernel       the full label array, on request.
// ---------------------------------------------------------------------------
constexpr uint32_t kIdx = 4 * kTC - 1;  // local index bits of an LDS label
constexpr uint32_t kBorder = 0x8000u;  // flag on the root of a component that holds a border bond index
static_assert(4 * kTC <= kBorder, "local bond indices must stay below the border flag");
static_assert((4 * kTC & (4 * kTC - 1)) == 0, "kIdx is a bit mask");
static_assert(kTT >= kBorderIdx + kEdgeBytes, "one flip thread per border component and facing arm");
static_assert(kTW == 64, "a wavefront holds one tile row");
static_assert(4 * (kTT / 64) == kTH, "four rows per wavefront cover the tile");

struct TileGeom {
    uint32_t x0, y0, w, h, id;
};

// Tile (bx, by) of a lattice with ncx tiles per row.
__device__ __forceinline__ TileGeom tile_geom(uint32_t L, uint32_t bx, uint32_t by, uint32_t ncx)
{
    TileGeom g;
    g.x0 = bx * kTW;
    g.y0 = by * kTH;
    g.w = min(kTW, L - g.x0);
    g.h = min(kTH, L - g.y0);
    g.id = bx + by * ncx;
    return g;
}

// XCD-aware tile order.  Workgroups are dealt to the eight XCDs in turn
// (workgroup b to XCD b % 8), each with its own L2, and a tile row of one
// plane is 64 bytes, half an L2 line: with tiles in row-major order every
// line would be fetched by two XCDs.  Instead the j-th workgroup of an XCD
// takes tile kTileRun (8 (j / kTileRun) + xcd) + j % kTileRun, so each XCD
// works on runs of kTileRun consecutive tiles and shares lines with other
// XCDs only at the ends of its runs (runs of 8 measured best for 64 x 16
// tiles at L = 1414, against 2, 4, 16, 32 and 64).
constexpr uint32_t kTileXcd = 8, kTileRun = 8;

// The tile of this workgroup in a single-chain launch (gridDim.x x ncy tiles), in the
// XCD-aware order; the last n % (8 kTileRun) tiles, which do not fill a run
// on every XCD, keep their place.
__device__ __forceinline__ TileGeom grid_tile(uint32_t L, uint32_t ncy)
{
    const uint32_t ncx = gridDim.x, n = ncx * ncy;
    const uint32_t b = blockIdx.x + blockIdx.y * ncx;
    uint32_t tile = b;
    if (b < n - n % (kTileXcd * kTileRun)) {
        const uint32_t xcd = b % kTileXcd, j = b / kTileXcd;
        tile = ((j / kTileRun) * kTileXcd + xcd) * kTileRun + j % kTileRun;
    }
    const uint32_t by = tile / ncx;
    return tile_geom(L, tile - by * ncx, by, ncx);
}

__device__ __forceinline__ bool tile_in(const TileGeom& g, uint32_t v)
{
    const uint32_t lc = v % kTC;
    return lc % kTW < g.w && lc / kTW < g.h;
}

__device__ __forceinline__ uint32_t tile_global(const TileGeom& g, uint32_t L, uint32_t N, uint32_t v)
{
    const uint32_t lc = v % kTC;
    return (v / kTC) * N + (g.y0 + lc / kTW) * L + g.x0 + lc % kTW;
}

// The 16 bond indices of a thread: four neighbouring cells of one tile row,
// in each of the four planes.  A tile row is 16 lanes, so the cells to the
// right are the next lane's, and a plane's four sigma are one dword and its
// four local roots two; rows start at even addresses, which wider accesses take.
// Against one bond index per lane and access (16 byte and 16 half-word loads
// or stores, and the new sigma through LDS twice) the flip, with its stores
// written through, went from 19.7 to 15.0 us at L = 1414 and from 8.7 to 6.7 us
// at L = 256; the tile kernel from 25.2 to 24.2 us, of which its 340 VALU
// instructions per cell take 17 at full issue rate.
struct QuadPos {
    uint32_t lx, ly, lc;  // first cell: tile column, tile row, local index (4 threadIdx.x)
    uint32_t c;           // its global index (0 if none is inside)
    uint32_t n;           // cells inside the tile: 0, 2 or 4, for L is even
};
static_assert(kTT * 4 == kTC && kTW == 64, "16 threads per tile row");

__device__ __forceinline__ QuadPos quad_pos(const TileGeom& g, uint32_t L)
{
    QuadPos q;
    q.lc = 4 * threadIdx.x;
    q.lx = q.lc % kTW;
    q.ly = q.lc / kTW;
    q.n = q.ly < g.h && q.lx < g.w ? min(4u, g.w - q.lx) : 0u;
    q.c = q.n ? (g.y0 + q.ly) * L + g.x0 + q.lx : 0u;
    return q;
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// The border bond indices of a tile -- the ends of tile-crossing covalent
// links -- numbered b < 2 kTH + 2 kTW: arm 0 in the last column and arm 1 in
// the first column (row b), arm 2 in the last row and arm 3 in the first row
// (column b); 4 kTC if b names no bond index of a ragged tile.
__device__ __forceinline__ uint32_t border_local(const TileGeom& g, uint32_t b)
{
    if (b < kTH) return b < g.h ? b * kTW + g.w - 1 : 4 * kTC;
    if (b < 2 * kTH) return b - kTH < g.h ? kTC + (b - kTH) * kTW : 4 * kTC;
    if (b < 2 * kTH + kTW) return b - 2 * kTH < g.w ? 2 * kTC + (g.h - 1) * kTW + (b - 2 * kTH) : 4 * kTC;
    return b - 2 * kTH - kTW < g.w ? 3 * kTC + (b - 2 * kTH - kTW) : 4 * kTC;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

__device__ __forceinline__ uint32_t find_root_lds(const uint32_t* lab, uint32_t x)
{
    uint32_t p = lab[x] & kIdx;
    while (p != x) {
        x = p;
        p = lab[x] & kIdx;
    }
    return x;
}

__device__ __forceinline__ void unite_lds(uint32_t* lab, uint32_t a, uint32_t b)
{
    a = find_root_lds(lab, a);
    b = find_root_lds(lab, b);
    while (a != b) {
        if (a > b) {
            const uint32_t tmp = a;
            a = b;
            b = tmp;
        }
        const uint32_t old = atomicMin(lab + b, a);
        if (old == b) return;
        b = find_root_lds(lab, old);
        a = find_root_lds(lab, a);
    }
}

// In-tile components from the link masks mk[i] of cells lc = tid + kTT i:
// the in-cell components (LUT) and the +x links of each row (ballots), then
// the +y links inside the tile (lock-free union-find in LDS);
// finally the roots of components holding a border bond index get kBorder.
// The minimum-index root does not depend on the order of the unions, so
// every kernel that rebuilds the components from the same mask gets the
// same roots.  Expects lut ready; ends with a barrier.
__device__ void tile_components(uint32_t* lab, const uint8_t* lut, const uint32_t (&mk)[kTC / kTT], const TileGeom& g)
{
    const uint32_t lane = threadIdx.x & 63;                // = tile column: a wavefront holds a tile row
#pragma unroll
    for (uint32_t i = 0; i < kTC / kTT; ++i) {
        const uint32_t lc = threadIdx.x + kTT * i, ly = lc / kTW;
        const uint32_t m = mk[i];
        const uint32_t l4 = lut[m >> 2];
        const uint32_t r1 = (l4 >> 2) & 3;                 // arm 0 is always its own in-cell root
        // +x links inside the row: a run of cells joined arm 0 -> arm 1 of the
        // next cell, continued through every cell whose arms 0 and 1 share an
        // in-cell component, is one component whose minimum is arm 0 of the
        // run's first cell.  Found with two ballots; no atomics.
        const uint64_t lnk = __ballot((m & 1) && lane + 1 < g.w);
        const bool in = lane > 0 && ((lnk >> (lane - 1)) & 1);
        const uint64_t brk = __ballot(!(in && r1 == 0));  // bit j: a run starts at column j
        uint32_t e0 = lc;
        uint32_t b_root = 0;
        if (in) {
            const uint64_t upto = lane == 63 ? brk : (brk & ((2ull << lane) - 1));
            const uint64_t before = brk & ((1ull << lane) - 1);
            const uint32_t start = 63 - (uint32_t)__builtin_clzll(upto);
            const uint32_t start_prev = 63 - (uint32_t)__builtin_clzll(before);
            e0 = ly * kTW + start;                         // this cell's arm 0, if the run goes through
            b_root = ly * kTW + start_prev;                // the run that reaches this cell's arm 1
        }
        lab[lc] = e0;
        lab[kTC + lc] = r1 * kTC + lc;
        lab[2 * kTC + lc] = ((l4 >> 4) & 3) * kTC + lc;
        lab[3 * kTC + lc] = ((l4 >> 6) & 3) * kTC + lc;
        if (in && r1 != 0) lab[r1 * kTC + lc] = b_root;    // arm 1's own component joins the run
    }
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < kTC / kTT; ++i) {
        const uint32_t lc = threadIdx.x + kTT * i, ly = lc / kTW;
        if ((mk[i] & 2) && ly + 1 < g.h) unite_lds(lab, 2 * kTC + lc, 3 * kTC + lc + kTW);
    }
    __syncthreads();
    if (threadIdx.x < 2 * (kTW + kTH)) {
        const uint32_t v = border_local(g, threadIdx.x);
        if (v < 4 * kTC) atomicOr(lab + find_root_lds(lab, v), kBorder);
    }
    __syncthreads();
}

__device__ __forceinline__ void tile_masks(const LatticeArgs& a, const TileGeom& g, uint32_t (&mk)[kTC / kTT])
{
#pragma unroll
    for (uint32_t i = 0; i < kTC / kTT; ++i) {
        const uint32_t lc = threadIdx.x + kTT * i, lx = lc % kTW, ly = lc / kTW;
        mk[i] = (lx < g.w && ly < g.h) ? a.mask[(g.y0 + ly) * a.L + g.x0 + lx] : 0u;
    }
}

// Lock-free union of the clusters with roots pu and pv (minimum index wins):
// atomicMin points the larger at the smaller and returns its previous
// parent p; p == the larger means it was a root and the union is done,
// otherwise the pair (smaller, p) is united next, so no connection is lost.
// The larger element of the pair strictly decreases, so the loop ends.
__device__ __forceinline__ void unite_global(uint32_t* label, uint32_t pu, uint32_t pv)
{
    while (pu != pv) {
        if (pu > pv) {
            const uint32_t tmp = pu;
            pu = pv;
            pv = tmp;
        }
        const uint32_t old = atomicMin(label + pv, pu);
        if (old == pv) return;
        pv = old;
    }
}

// lut: 64 bytes, lab: 4 kTC words, act: kEdgeBytes bytes of LDS.
__device__ __forceinline__ void sw_tile_body(const LatticeArgs& a, const VolArgs& va, uint32_t bank, const TileGeom& g,
                                             uint8_t* lut, uint32_t* lab, uint8_t* act)
{
    // Waves of a SIMD issue oldest first; a workgroup that has finished its
    // bonds yields to those still computing theirs, so all tiles reach the
    // latency-bound union phases together (priority 3, 2, 0 by phase).
    __builtin_amdgcn_s_setprio(3);
    const uint32_t L = a.L, N = a.N;
    uint8_t* edge = a.edge + (size_t)g.id * kEdgeBytes;
    // cell i of a thread: tile column lane, tile row wave + W i (wave-uniform),
    // so plane and row offsets are scalar and the loads need no vector address
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool col_in = lane < g.w;
    const uint32_t x = g.x0 + lane;
    const uint32_t vx = col_in ? x : 0u, vxp = col_in ? ((x + 1 == L) ? 0u : x + 1) : 0u;
    const __amdgpu_buffer_rsrc_t rs = buf_rsrc(a.sigma, 4 * N), rm = buf_rsrc(a.mask, N);
    StepView* view = a.st->view + bank;
    if (view->skip) return;
    int theta = view->theta;
    if (view->pending) theta = resolve_step(va, view, true, g.id == 0);
    build_incell_lut(lut);
    const SwBondCtx k = sw_ctx(a, view->t_cur, theta);
    uint32_t mk[kTC / kTT];
#pragma unroll
    for (uint32_t i = 0; i < kTC / kTT; ++i) {
        const uint32_t ly = wave + (kTT / 64) * i;
        uint32_t m = 0;
        if (ly < g.h && col_in) {
            const uint32_t y = g.y0 + ly, row = y * L, rowp = ((y + 1 == L) ? 0u : y + 1) * L;
            const uint32_t s0 = ld8(rs, vx, row), s1 = ld8(rs, vx, N + row), s2 = ld8(rs, vx, 2 * N + row),
                           s3 = ld8(rs, vx, 3 * N + row);
            const uint32_t f0 = ld8(rs, vxp, N + row), f2 = ld8(rs, vx, 3 * N + rowp);
            m = sw_bond_bits(a, k, x + row, s0, s1, s2, s3, f0, f2);
            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)m, rm, (int)vx, (int)row, 0);
            if (lane == g.w - 1) {
                edge[ly] = (uint8_t)f0;
                act[ly] = (uint8_t)(m & 1u);               // the +x link leaving the tile
            }
            if (ly == g.h - 1) {
                edge[kTH + lane] = (uint8_t)f2;
                act[kTH + lane] = (uint8_t)((m >> 1) & 1u);  // the +y link leaving the tile
            }
        }
        mk[i] = m;
    }
    __builtin_amdgcn_s_setprio(2);
    __syncthreads();
    tile_components(lab, lut, mk, g);
    __builtin_amdgcn_s_setprio(0);
    // every bond index: its tile-local root (| flag); flagged roots: a
    // global self-label; border bond indices: a global label of their root.
    // Eight bond indices at a time: their parents, then the parents' entries
    // (a root's entry is the root | flag, so nearly every index is settled by
    // these two reads); the few longer chains are followed in lockstep.
    // Rows past a ragged tile's end hold singletons and are read, not stored.
    const QuadPos qp = quad_pos(g, L);
#pragma unroll
    for (uint32_t h = 0; h < 2; ++h) {
        uint32_t r[8], e[8];
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j) r[j] = lab[(2 * h + (j >> 2)) * kTC + qp.lc + (j & 3)] & kIdx;
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j) e[j] = lab[r[j]];
        for (;;) {
            bool more = false;
#pragma unroll
            for (uint32_t j = 0; j < 8; ++j) more = more || (e[j] & kIdx) != r[j];
            if (!more) break;
#pragma unroll
            for (uint32_t j = 0; j < 8; ++j) {
                r[j] = e[j] & kIdx;                    // unchanged where already settled
                e[j] = lab[r[j]];
            }
        }
#pragma unroll
        for (uint32_t b = 0; b < 2; ++b) {
            const uint32_t p = 2 * h + b;
            const uint32_t* eb = e + 4 * b;
            const __amdgpu_buffer_rsrc_t rl = buf_rsrc(a.lroot + (size_t)p * N, 2 * N);
            if (qp.n == 4) {
                const u32x2 w = {eb[0] | eb[1] << 16, eb[2] | eb[3] << 16};
                if (a.sw_through) __builtin_amdgcn_raw_buffer_store_b64(w, rl, (int)(2 * qp.c), 0, kThrough);
                else __builtin_amdgcn_raw_buffer_store_b64(w, rl, (int)(2 * qp.c), 0, kPlain);
            } else if (qp.n) {
                if (a.sw_through) __builtin_amdgcn_raw_buffer_store_b32(eb[0] | eb[1] << 16, rl, (int)(2 * qp.c), 0, kThrough);
                else __builtin_amdgcn_raw_buffer_store_b32(eb[0] | eb[1] << 16, rl, (int)(2 * qp.c), 0, kPlain);
            }
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j)
                if (j < qp.n && eb[j] == (kBorder | (p * kTC + qp.lc + j))) {
                    // a root other tiles' unions may reach this step: written
                    // through to the device-coherent level (see below)
                    const uint32_t gv = p * N + qp.c + j;
                    __hip_atomic_store(a.label + gv, gv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
        }
    }
    // Tile-crossing links.  Every border bond index gets the global label of
    // its root (the flip follows these chains), and the tile publishes one
    // exchange word per border bond index: the global root of its component,
    // for the ends in the last column and row only if the link leaving there
    // is active (kNoLink otherwise).  Each tile edge has an arrival counter
    // that the two tiles beside it increment once per step (it wraps back to
    // 0); the tile that arrives second unites that edge's active links with
    // the first tile's words.  No tile ever waits for another.
    // Everything one tile reads of another's within this launch -- the
    // exchange words and the label entries the unions' atomicMin acts on --
    // is written and read only with device-scope atomic stores, loads and
    // read-modify-writes, which all act at the device-coherent level (across
    // the XCDs' separate L2 caches); no plain store touches those entries in
    // this launch.  The barrier below waits for this tile's stores to
    // complete before its counter increments are issued, and the other
    // tile's words are read only after its increment was seen.  (Device-scope
    // fences would do the same by writing back and invalidating whole L2
    // caches, which measured four times slower.)
    uint32_t* xw = a.xchg + (size_t)g.id * kBorderIdx;
    if (threadIdx.x < kBorderIdx) {
        const uint32_t b = threadIdx.x;
        const uint32_t v = border_local(g, b);
        uint32_t w = kNoLink;
        if (v < 4 * kTC) {
            const uint32_t gr = tile_global(g, L, N, find_root_lds(lab, v));
            // device-scope store: other tiles' atomicMin may act on this
            // entry (when v is its own root) before the launch ends, and a
            // plain store's dirty L2 line written back later would undo it
            __hip_atomic_store(a.label + tile_global(g, L, N, v), gr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            bool on = true;
            if (b < kTH) on = act[b] != 0;
            else if (b >= 2 * kTH && b < 2 * kTH + kTW) on = act[kTH + (b - 2 * kTH)] != 0;
            w = on ? gr : kNoLink;
        }
        __hip_atomic_store(xw + b, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __builtin_amdgcn_s_waitcnt(0);            // this wave's stores are complete ...
    __syncthreads();                          // ... and so are every wave's, before any increment
    const uint32_t ncx = (L + kTW - 1) / kTW, ncy = (L + kTH - 1) / kTH;
    const uint32_t bx = g.x0 / kTW, by = g.y0 / kTH;
    const uint32_t right = (bx + 1 == ncx ? 0 : bx + 1) + by * ncx, left = (bx == 0 ? ncx - 1 : bx - 1) + by * ncx;
    const uint32_t down = bx + (by + 1 == ncy ? 0 : by + 1) * ncx, up = bx + (by == 0 ? ncy - 1 : by - 1) * ncx;
    uint8_t* second = lut;                    // the in-cell table is dead: four flags
    if (threadIdx.x < 4) {
        // edges: 0 right (counter 2 id), 1 bottom (2 id + 1), 2 left (the left
        // tile's right edge), 3 top (the upper tile's bottom edge)
        const uint32_t e = threadIdx.x;
        const uint32_t c = e == 0 ? 2 * g.id : e == 1 ? 2 * g.id + 1 : e == 2 ? 2 * left : 2 * up + 1;
        second[e] = atomicInc(a.ecnt + c, 1u) == 1u ? 1 : 0;
    }
    __syncthreads();
    if (!(second[0] | second[1] | second[2] | second[3])) return;
    auto word = [](const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    const uint32_t e = threadIdx.x >> 6, pos = threadIdx.x & 63;
    if (e < 4 && second[e]) {
        uint32_t pu = kNoLink, pv = kNoLink;  // pu: the word that carries the link's activity
        if (e == 0 && pos < g.h) {
            pu = word(xw + pos);
            pv = word(a.xchg + (size_t)right * kBorderIdx + kTH + pos);
        } else if (e == 2 && pos < g.h) {
            pu = word(a.xchg + (size_t)left * kBorderIdx + pos);
            pv = word(xw + kTH + pos);
        } else if (e == 1 && pos < g.w) {
            pu = word(xw + 2 * kTH + pos);
            pv = word(a.xchg + (size_t)down * kBorderIdx + 2 * kTH + kTW + pos);
        } else if (e == 3 && pos < g.w) {
            pu = word(a.xchg + (size_t)up * kBorderIdx + 2 * kTH + pos);
            pv = word(xw + 2 * kTH + kTW + pos);
        }
        if (pu != kNoLink) unite_global(a.label, pu, pv);
    }
}

__global__ __launch_bounds__(kTT) void sw_tile_kernel(LatticeArgs a, VolArgs va, StepCtl ctl)
{
    __shared__ uint8_t lut[64];
    __shared__ uint32_t lab[4 * kTC];
    __shared__ uint8_t act[kEdgeBytes];
    sw_tile_body(a, va, ctl.bank, grid_tile(a.L, gridDim.y), lut, lab, act);
}

// LDS of the flip: the compacted roots of the interior components; the shift
// of each root; the new sigma of arm 3; the new sigma facing the right /
// bottom edge; the compacted roots of the border components (at most one per
// border bond index); the two root counts.
struct FlipLds {
    uint16_t roots[4 * kTC];
    uint8_t sh[4 * kTC];
    uint32_t up[kTC / 4];
    __align__(4) uint8_t across[kEdgeBytes];
    uint16_t rootb[kBorderIdx];
    uint32_t nroot, nrootb;
};
static_assert(kTH % 4 == 0, "four columns of the bottom edge's facing arms are one aligned word");

__device__ __forceinline__ void sw_flip_body(const LatticeArgs& a, uint32_t bank, const TileGeom& g, FlipLds& lds)
{
    uint16_t* roots = lds.roots;
    uint8_t* sh = lds.sh;
    uint8_t* across = lds.across;
    uint16_t* rootb = lds.rootb;
    if (threadIdx.x == 0) {
        lds.nroot = 0;
        lds.nrootb = 0;
    }
    const uint32_t L = a.L, N = a.N, q = a.q;
    // entry i: plane i / 4, cell i % 4 of the thread's four
    const uint32_t lane = threadIdx.x & 63;
    const QuadPos qp = quad_pos(g, L);
    const __amdgpu_buffer_rsrc_t rs = buf_rsrc(a.sigma, 4 * N);
    uint32_t os[4], lrp[8];                   // old sigma; local roots | kBorder, two per register
#pragma unroll
    for (uint32_t p = 0; p < 4; ++p) {
        os[p] = 0;
        lrp[2 * p] = lrp[2 * p + 1] = 0;
        const __amdgpu_buffer_rsrc_t rl = buf_rsrc(a.lroot + (size_t)p * N, 2 * N);
        if (qp.n == 4) {
            os[p] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)qp.c, (int)(p * N), 0);
            const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(rl, (int)(2 * qp.c), 0, 0);
            lrp[2 * p] = w.x;
            lrp[2 * p + 1] = w.y;
        } else if (qp.n) {
            os[p] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, (int)qp.c, (int)(p * N), 0);
            lrp[2 * p] = __builtin_amdgcn_raw_buffer_load_b32(rl, (int)(2 * qp.c), 0, 0);
        }
    }
    // the loads above do not depend on the chain state; read it now
    const StepView* view = a.st->view + bank;
    if (view->skip) return;                   // step limit reached (uniform, before any barrier)
    const uint32_t t = view->t_cur;
    if (g.id == 0) {
        if (threadIdx.x == 0) a.st->sw_done = 1;
        // the other bank's recount, of the step before, is dead: the next step
        // adds its own there
        static_assert(kTT >= 2 * kSlots, "one thread per slot of the two recounted values");
        if (threadIdx.x < 2 * kSlots) a.slots[(bank ^ 1u) * kBankSlots + threadIdx.x] = 0;
    }
    auto LR = [&](uint32_t i) { return (lrp[i >> 1] >> (16 * (i & 1))) & 0xFFFFu; };
    // component roots, compacted into an interior and a border list: a lane's
    // slots follow from a prefix sum of the per-lane counts over the
    // wavefront, one LDS atomic per wavefront and list places the wavefront
    // (the order of a list is immaterial: every entry sets its own root's
    // shift)
    // The lane's roots as bits of one register (bit i: entry i is an
    // interior root, bit 16 + i: a border root), so that no per-entry lane
    // masks stay live in SGPRs between the two passes.
    static_assert(4 * kTC / kTT == 16, "16 entries per thread");
    uint32_t rf = 0;
#pragma unroll
    for (uint32_t i = 0; i < 4 * kTC / kTT; ++i) {
        const bool root = (i & 3) < qp.n && (LR(i) & kIdx) == (i >> 2) * kTC + qp.lc + (i & 3);
        const uint32_t bit = ((LR(i) >> 11) & 16u) + i;   // the border flag (bit 15) selects bit 16 + i
        rf |= (root ? 1u : 0u) << bit;
    }
    const uint32_t cnt = (uint32_t)__popc(rf & 0xFFFFu), cntb = (uint32_t)__popc(rf >> 16);
    uint32_t tot, totb;
    uint32_t pos = wave_excl_scan5(cnt, tot), posb = wave_excl_scan5(cntb, totb);
    __syncthreads();                          // counts = 0
    uint32_t base = 0, baseb = 0;
    if (lane == 0) {
        base = atomicAdd(&lds.nroot, tot);
        baseb = atomicAdd(&lds.nrootb, totb);
    }
    pos += (uint32_t)__shfl((int)base, 0);
    posb += (uint32_t)__shfl((int)baseb, 0);
#pragma unroll
    for (uint32_t i = 0; i < 4 * kTC / kTT; ++i) {
        const uint32_t bi = (rf >> i) & 1u, bb = (rf >> (16 + i)) & 1u;
        if (bi) roots[pos] = (uint16_t)LR(i);
        pos += bi;
        if (bb && posb < kBorderIdx) rootb[posb] = (uint16_t)(LR(i) & kIdx);
        posb += bb;
    }
    __syncthreads();
    // One shift per component, drawn at its cluster minimum.  Border
    // components and the facing arms across the right edge (p < kTH) and
    // the bottom edge (column p - kTH) need the global root chain: one job
    // per thread, whose first link is loaded before the interior components
    // (whose minimum is their own root) are drawn, so that the load's
    // latency is hidden behind that arithmetic.
    const uint32_t nr = lds.nroot, nb = min(lds.nrootb, kBorderIdx);
    const uint8_t* edge = a.edge + (size_t)g.id * kEdgeBytes;
    uint32_t x = 0, dst = 0;
    bool live = false;
    if (threadIdx.x < nb) {
        dst = rootb[threadIdx.x];
        x = tile_global(g, L, N, dst);
        live = true;
    } else if (threadIdx.x - nb < kEdgeBytes) {
        const uint32_t p = threadIdx.x - nb;
        dst = 0x10000u | p;
        if (p < kTH) {
            live = p < g.h;
            const uint32_t xx = g.x0 + g.w - 1, yy = g.y0 + p;
            x = N + ((xx + 1 == L) ? 0 : xx + 1) + yy * L;
        } else {
            live = p - kTH < g.w;
            const uint32_t xx = g.x0 + (p - kTH), yy = g.y0 + g.h - 1;
            x = 3 * N + xx + ((yy + 1 == L) ? 0 : yy + 1) * L;
        }
    }
    uint32_t pn = live ? a.label[x] : 0u;
    for (uint32_t j = threadIdx.x; j < nr; j += kTT) {
        const uint32_t e = roots[j];
        const uint32_t w = philox(tile_global(g, L, N, e), t, 0u, kStreamSwf, a.key0, a.key1).x;
        sh[e] = (uint8_t)((w <= a.flip_lim) ? (uint32_t)((double)w * a.flip_invd) : 0u);
    }
    if (live) {
        while (pn != x) {
            x = pn;
            pn = a.label[x];
        }
        const uint32_t w = philox(x, t, 0u, kStreamSwf, a.key0, a.key1).x;
        const uint32_t sft = (w <= a.flip_lim) ? (uint32_t)((double)w * a.flip_invd) : 0u;
        if (dst < 0x10000u) {
            sh[dst] = (uint8_t)sft;
        } else {
            const uint32_t p = dst & 0xFFFFu;
            const uint32_t s = edge[p] + sft;
            across[p] = (uint8_t)(s >= q ? s - q : s);
        }
    }
    __syncthreads();
    // Empty asm, no instruction: the masked roots are recomputed here from
    // the packed registers instead of being kept live (and spilled) across
    // the draws since the compaction.
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) __asm__("" : "+v"(lrp[k]));
    // New sigma, four cells to a word: byte sums stay below 16, and bit 7 of
    // (sum + 128 - q) says whether to take q off.
    const uint32_t one = 0x01010101u, qv = q * one, lift = (128u - q) * one;
    const uint32_t in = qp.n == 4 ? ~0u : (1u << (8 * qp.n)) - 1u;   // bytes of cells inside the tile
    uint32_t ns[4];
#pragma unroll
    for (uint32_t p = 0; p < 4; ++p) {
        uint32_t d = 0;
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) d |= (uint32_t)sh[LR(4 * p + j) & kIdx] << (8 * j);
        uint32_t w = os[p] + (d & in);
        const uint32_t ge = ((w + lift) >> 7) & one;
        w -= ((ge << 3) - ge) & qv;           // 7 in every byte to lower by q (q <= 6)
        ns[p] = w;
        if (qp.n == 4) {
            __builtin_amdgcn_raw_buffer_store_b32(w, rs, (int)qp.c, (int)(p * N), kThrough);
        } else if (qp.n) {
            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)w, rs, (int)qp.c, (int)(p * N), kThrough);
        }
    }
    lds.up[threadIdx.x] = ns[3];
    __syncthreads();
    // Recount of the new configuration: the +x and +y HB pairs and the six
    // in-cell pairs of every cell of the tile.  Bit 3 of (x ^ y) + 7 says
    // that two sigma differ.
    uint32_t f0 = __builtin_amdgcn_alignbyte((uint32_t)__builtin_amdgcn_update_dpp(0, (int)ns[1], 0x101, 0xf, 0xf, true),
                                             ns[1], 1);   // arm 1 one cell on (row_shl:1: the next lane's)
    if (qp.n && qp.lx + qp.n == g.w) {        // the last column faces the next tile
        const uint32_t sft = 8 * (qp.n - 1);
        f0 = (f0 & ~(0xFFu << sft)) | ((uint32_t)across[qp.ly] << sft);
    }
    const uint32_t f2 = qp.ly + 1 < g.h ? lds.up[threadIdx.x + kTW / 4]
                                        : *reinterpret_cast<const uint32_t*>(across + kTH + qp.lx);
    auto differ = [](uint32_t u, uint32_t w) { return ((u ^ w) + 0x07070707u) & 0x08080808u; };
    const uint32_t dh = differ(ns[0], f0) | differ(ns[2], f2) >> 1;
    const uint32_t dc = differ(ns[0], ns[1]) | differ(ns[0], ns[2]) >> 1 | differ(ns[0], ns[3]) >> 2 |
                        differ(ns[1], ns[2]) >> 3 | differ(ns[1], ns[3]) << 1 | differ(ns[2], ns[3]) << 2;
    const int hb = 2 * (int)qp.n - __popc(dh & in), co = 6 * (int)qp.n - __popc(dc & in);
    const int v2[2] = {hb, co};
    block_add<2, kTT>(v2, a.slots + bank * kBankSlots + (g.id & (kSlots - 1)), kSlots);
}

__global__ __launch_bounds__(kTT) __attribute__((amdgpu_waves_per_eu(8, 8))) void sw_flip_tile_kernel(LatticeArgs a, VolArgs va,
                                                                                                    StepCtl ctl)
{
    __shared__ __align__(16) FlipLds lds;
    const uint32_t ncy = gridDim.y - ctl.open;
    if (blockIdx.y == ncy) {                  // opens the next step
        if (blockIdx.x == 0 && threadIdx.x < 64) open_next(va, (double*)&lds, a.st->view + (ctl.bank ^ 1u));
        return;
    }
    sw_flip_body(a, ctl.bank, grid_tile(a.L, ncy), lds);
}

// label[idx] = the minimum of idx's cluster, for every bond index; written
// to out (4N uint32).  Works from the mask and the global labels left by
// either the tiled or the batched step.
__global__ __launch_bounds__(kTT) void sw_labels_kernel(LatticeArgs a, uint32_t* __restrict__ out)
{
    __shared__ uint8_t lut[64];
    __shared__ uint32_t lab[4 * kTC];
    build_incell_lut(lut);
    const uint32_t L = a.L, N = a.N;
    const TileGeom g = grid_tile(L, gridDim.y);
    uint32_t mk[kTC / kTT];
    tile_masks(a, g, mk);
    __syncthreads();
    tile_components(lab, lut, mk, g);
#pragma unroll
    for (uint32_t i = 0; i < 4 * kTC / kTT; ++i) {
        const uint32_t v = threadIdx.x + kTT * i;
        if (!tile_in(g, v)) continue;
        const uint32_t r = find_root_lds(lab, v);
        const uint32_t gr = tile_global(g, L, N, r);
        out[tile_global(g, L, N, v)] = (lab[r] & kBorder) ? find_root(a.label, gr) : gr;
    }
}

// ---------------------------------------------------------------------------
// Batched Swendsen-Wang: the tiled step of every chain of a batch, one launch
// per stage.  Workgroup b belongs to the chain c with start[c] <= b <
// start[c+1] (prefix sums of per-chain tiles) and does
// exactly what the workgroup of that chain's own launch does.
// ---------------------------------------------------------------------------
// Tile of workgroup b of a batch whose chain's tiles are start .. end - 1:
// the XCD-aware order of grid_tile over the workgroups from the first
// multiple of 8 kTileRun at or after start, in whole groups of 8 kTileRun
// (so that b % 8 is the XCD there too); row-major order elsewhere.
__device__ __forceinline__ TileGeom batch_tile(const LatticeArgs& a, uint32_t b, uint32_t start, uint32_t end)
{
    constexpr uint32_t kGroup = kTileXcd * kTileRun;
    const uint32_t ncx = (a.L + kTW - 1) / kTW;
    const uint32_t s8 = (start + kGroup - 1) / kGroup * kGroup;
    uint32_t tile = b - start;
    if (b >= s8 && end >= s8 && b < s8 + (end - s8) / kGroup * kGroup) {
        const uint32_t r = b - s8, xcd = r % kTileXcd, j = r / kTileXcd;
        tile = s8 - start + ((j / kTileRun) * kTileXcd + xcd) * kTileRun + j % kTileRun;
    }
    const uint32_t by = tile / ncx;
    return tile_geom(a.L, tile - by * ncx, by, ncx);
}

__global__ __launch_bounds__(kTT) void sw_tile_batch_kernel(const BatchEntry* __restrict__ ent,
                                                            const uint32_t* __restrict__ tstart, uint32_t count,
                                                            StepCtl ctl)
{
    __shared__ uint8_t lut[64];
    __shared__ uint32_t lab[4 * kTC];
    __shared__ uint8_t act[kEdgeBytes];
    const uint32_t c = batch_chain(tstart, count, blockIdx.x);
    const LatticeArgs a = ent[c].la;
    sw_tile_body(a, ent[c].va, ctl.bank, batch_tile(a, blockIdx.x, tstart[c], tstart[c + 1]), lut, lab, act);
}

__global__ __launch_bounds__(kTT) __attribute__((amdgpu_waves_per_eu(8, 8))) void sw_flip_batch_kernel(
    const BatchEntry* __restrict__ ent, const uint32_t* __restrict__ tstart, uint32_t count, uint32_t total,
    StepCtl ctl)
{
    __shared__ __align__(16) FlipLds lds;
    static_assert(sizeof(FlipLds) >= kSwWaves * 40 * sizeof(double), "the shell terms of each wavefront's step");
    if (blockIdx.x >= total) {                // opens the next step of a chain per wavefront
        const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = open_chain(blockIdx.x - total, w, kSwWaves);
        if (i >= count) return;
        VolArgs v = ent[i].va;
        v.mode = kVolSw;
        v.met_att_add = 0;
        open_next(v, (double*)&lds + 40 * w, v.st->view + (ctl.bank ^ 1u));
        return;
    }
    const uint32_t c = batch_chain(tstart, count, blockIdx.x);
    const LatticeArgs a = ent[c].la;
    sw_flip_body(a, ctl.bank, batch_tile(a, blockIdx.x, tstart[c], tstart[c + 1]), lds);
}
