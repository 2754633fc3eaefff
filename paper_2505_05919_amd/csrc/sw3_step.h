// Swendsen-Wang step of the cubic lattice (included inside cvf3.hip's
// unnamed namespace, Sec. II.D).
//
// Links of cell c: l = 0..2 the covalent link of its +d edge (arm 2d of c
// with arm 2d+1 of the +d neighbour; liquid and eta = 1 only; equal arms for
// J_eff > 0, unequal for J_eff < 0), l = 3..17 the 15 cooperative pairs
// (a, b), a < b, lexicographic (equal arms).  Link l uses word l mod 4 of
// Philox(c, t, l / 4, SWB); bond iff word < 64-bit threshold.  Labels are the
// smallest flat index a N + c of each cluster.
//
// A workgroup owns a tile of TX x TY x TZ cells (the last tile of an axis is
// ragged), T = TX TY TZ, with one or four x-adjacent cells per thread (four:
// the planes are moved as dwords, and at 128^3 the flip's tiles are resident
// all at once).  Bond index (a, lc) has the local index v = a T + lc,
// lc = lx + TX (ly + TY lz), whose order is the order of the flat indices.
// Three launches:
//   sw3_tile_kernel   links, the components inside the tile (in-cell ones from
//                     tables, covalent ones by union-find in LDS), and one
//                     node per face index (below)
//   sw3_union_kernel  the links that cross a tile face, over those nodes
//   sw3_flip_kernel   one shift per component, the new sigma and its recount
// Nodes: a face index is a bond index at the end of a tile-crossing link
// (arm 2d in the last, arm 2d + 1 in the first cell layer of a tile along d).
// It is numbered by its face and its place there, the plus faces first:
// node (x, plus) of tile column bx at (y, z) is bx L^2 + z L + y, and so on;
// F = L^2 (nx + ny + nz) plus nodes, then as many minus nodes.  par[node]
// starts at the representative of its in-tile component, whose key is the
// component's smallest flat index; roots are hooked under the root with the
// smaller key.  Only face indices take part in the global union-find, so its
// arrays are 8 bytes per face index instead of 4 per bond index, and every
// other bond index carries a 16-bit tile-local root.
// Measured at 128^3, 210 K: tiles 52 us (VALU issue and LDS round trips: 2600
// VALU instructions per thread of four cells, 1050 of them draw and test the
// links, and ~47 LDS turns of the unions), crossing links 24 us (memory
// latency), flip and recount 36 us (label chains), 1.38 ms per 10 steps in
// all.  With parents of all bond indices in memory, a find and a Philox block
// per bond index and a separate recount the launches took 33 + 43, 42 and
// 59 + 25 + 5 us, 2.31 ms per 10 steps.
#pragma once

// Components of a cell's six arms under its 15 cooperative links, in three
// table lookups instead of a closure over 36 arm pairs: the partition of arms
// 0..3 from their six links (15 partitions), then arm 4 joins it through its
// four links (52 partitions of five arms), then arm 5 through its five.
struct alignas(4) ArmTables {
    uint8_t four[64];        // links (01)(02)(03)(12)(13)(23) -> partition of arms 0..3
    uint8_t five[16 * 16];   // partition + 16 (links of arm 4) -> partition of arms 0..4
    uint16_t six[52 * 32];   // partition + 52 (links of arm 5) -> root arm of arm k at bits 3(k-1), k = 1..5
};

constexpr ArmTables make_arm_tables()
{
    ArmTables t{};
    // a partition as the smallest arm of each arm's part, three bits per arm
    uint32_t p4[15] = {}, p5[52] = {};
    int n4 = 0, n5 = 0;
    // join arm k's part with the parts of the arms in adj
    auto join = [](uint32_t code, int k, uint32_t adj) {
        int lab[6] = {};
        for (int i = 0; i < k; ++i) lab[i] = (int)((code >> (3 * i)) & 7u);
        lab[k] = k;
        for (int i = 0; i < k; ++i)
            if ((adj >> i) & 1u) {
                const int a = lab[i] < lab[k] ? lab[i] : lab[k], b = lab[i] < lab[k] ? lab[k] : lab[i];
                for (int j = 0; j <= k; ++j)
                    if (lab[j] == b) lab[j] = a;
            }
        uint32_t out = 0;
        for (int i = 0; i <= k; ++i) out |= (uint32_t)lab[i] << (3 * i);
        return out;
    };
    for (uint32_t m = 0; m < 64; ++m) {
        uint32_t code = join(0, 1, m & 1u);
        code = join(code, 2, ((m >> 1) & 1u) | (((m >> 3) & 1u) << 1));
        code = join(code, 3, ((m >> 2) & 1u) | (((m >> 4) & 1u) << 1) | (((m >> 5) & 1u) << 2));
        int id = 0;
        while (id < n4 && p4[id] != code) ++id;
        if (id == n4) p4[n4++] = code;
        t.four[m] = (uint8_t)id;
    }
    for (uint32_t adj = 0; adj < 16; ++adj)
        for (int i = 0; i < n4; ++i) {
            const uint32_t code = join(p4[i], 4, adj);
            int id = 0;
            while (id < n5 && p5[id] != code) ++id;
            if (id == n5) p5[n5++] = code;
            t.five[16 * adj + i] = (uint8_t)id;
        }
    for (uint32_t adj = 0; adj < 32; ++adj)
        for (int i = 0; i < n5; ++i) t.six[52 * adj + i] = (uint16_t)(join(p5[i], 5, adj) >> 3);
    return t;
}

__device__ const ArmTables kArmTables = make_arm_tables();
static_assert(sizeof(ArmTables) % 4 == 0, "copied as words");

// C: cells per thread (4 or 1).
template <int TX_, int TY_, int TZ_, int C_>
struct Tile3 {
    static constexpr uint32_t TX = TX_, TY = TY_, TZ = TZ_, T = TX * TY * TZ;
    // face indices of a full tile on its plus faces: x, y, z
    static constexpr uint32_t FX = TY * TZ, FY = TX * TZ, FZ = TX * TY, NF = FX + FY + FZ;
    static constexpr uint32_t kIdx = 8 * T - 1;            // bits of a local index (6 T < 8 T)
    static constexpr uint32_t C = C_, TT = T / C;          // threads
    static constexpr uint32_t kNoIdx = 6 * T;              // "no bond index"
    uint32_t bx, by, bz, x0, y0, z0, w, h, d, nx, ny, nz;

    // inx, iny: 1 / nx, 1 / ny in single precision (there are fewer than 2^22
    // tiles, so a quotient is off by at most one).
    __device__ __forceinline__ Tile3(uint32_t L, uint32_t tile, uint32_t nx_, uint32_t ny_, float inx, float iny)
        : nx(nx_), ny(ny_), nz((L + TZ - 1) / TZ)
    {
        // uniform over the workgroup, computed in vector registers: back to
        // scalar ones, and everything that follows from them with it
        const uint32_t row = __builtin_amdgcn_readfirstlane(fdiv(tile, nx, inx));
        bx = tile - row * nx;
        bz = __builtin_amdgcn_readfirstlane(fdiv(row, ny, iny));
        by = row - bz * ny;
        x0 = TX * bx;
        y0 = TY * by;
        z0 = TZ * bz;
        w = min(TX, L - x0);
        h = min(TY, L - y0);
        d = min(TZ, L - z0);
    }
    __device__ __forceinline__ static uint32_t fdiv(uint32_t n, uint32_t m, float inv)
    {
        uint32_t r = (uint32_t)((float)n * inv);
        if (r * m > n) --r;
        if ((r + 1) * m <= n) ++r;
        return r;
    }

    // Flat index of the bond index with local index v.
    __device__ __forceinline__ uint32_t flat(uint32_t L, uint32_t N, uint32_t v) const
    {
        const uint32_t lc = v % T;
        return (v / T) * N + (x0 + lc % TX) + L * ((y0 + (lc / TX) % TY) + L * (z0 + lc / (TX * TY)));
    }

    // Face position f < NF (x faces, then y, then z): whether it exists in
    // this tile, and the local indices of the face indices there on the plus
    // and on the minus face.
    __device__ __forceinline__ bool face(uint32_t f, uint32_t& vp, uint32_t& vm) const
    {
        if (f < FX) {
            const uint32_t ly = f % TY, lz = f / TY, lc = TX * (ly + TY * lz);
            vp = lc + w - 1;
            vm = T + lc;
            return ly < h && lz < d;
        }
        if (f < FX + FY) {
            const uint32_t g = f - FX, lx = g % TX, lz = g / TX, lc = lx + TX * TY * lz;
            vp = 2 * T + lc + TX * (h - 1);
            vm = 3 * T + lc;
            return lx < w && lz < d;
        }
        const uint32_t g = f - FX - FY, lx = g % TX, ly = g / TX, lc = lx + TX * ly;
        vp = 4 * T + lc + TX * TY * (d - 1);
        vm = 5 * T + lc;
        return lx < w && ly < h;
    }
    // Plus node of face position f, and the minus node at the other end of its
    // link (on the next tile along the axis); this tile's own minus node is
    // the plus node + F.
    __device__ __forceinline__ uint32_t node(uint32_t L, uint32_t f) const
    {
        const uint32_t L2 = L * L;
        if (f < FX) return bx * L2 + z0 * L + y0 + f % TY + L * (f / TY);
        const bool y = f < FX + FY;
        const uint32_t g = y ? f - FX : f - FX - FY;
        const uint32_t base = y ? (nx + by) * L2 + z0 * L : (nx + ny + bz) * L2 + y0 * L;
        return base + x0 + g % TX + L * (g / TX);
    }
    __device__ __forceinline__ uint32_t nodes(uint32_t L) const { return L * L * (nx + ny + nz); }
    __device__ __forceinline__ uint32_t facing(uint32_t L, uint32_t f, uint32_t plus) const
    {
        const bool wrap = f < FX ? bx + 1 == nx : f < FX + FY ? by + 1 == ny : bz + 1 == nz;
        const uint32_t n = f < FX ? nx : f < FX + FY ? ny : nz;
        return nodes(L) + plus + (wrap ? L * L * (1u - n) : L * L);
    }
    // Node of face position f < 2 NF (NF..: minus faces).
    __device__ __forceinline__ uint32_t node2(uint32_t L, uint32_t f) const
    {
        return f < NF ? node(L, f) : nodes(L) + node(L, f - NF);
    }
};

// Tiles along x and y, and their reciprocals.
struct TileGrid3 {
    uint32_t nx, ny;
    float inx, iny;
};

// The tile of workgroup b of n.  Workgroups are dealt to the eight XCDs in
// turn, and a tile's row of a plane is TX bytes, a fraction of an L2 line:
// the j-th workgroup of an XCD takes tile 8 (8 (j / 8) + xcd) + j % 8, so each
// XCD works on runs of 8 tiles along x that share their lines (the last
// n % 64 tiles keep their place).
__device__ __forceinline__ uint32_t xcd_tile(uint32_t b, uint32_t n)
{
    if (b >= n - n % 64) return b;
    const uint32_t xcd = b % 8, j = b / 8;
    return ((j / 8) * 8 + xcd) * 8 + j % 8;
}

// Unite the components of a and b in LDS (lock-free, smaller index wins):
// both chains are followed in lockstep, one LDS round trip per hop, until
// they meet or both ends are roots; atomicMin then points the larger root at
// the smaller and returns its previous parent (its own index if it still was
// a root), from where the union goes on.  The starting entries are pointed at
// the ancestor reached: they are no roots any more.
__device__ __forceinline__ void lds_join(uint32_t* lab, uint32_t a, uint32_t b)
{
    const uint32_t a0 = a, b0 = b;
    while (a != b) {
        const uint32_t pa = lab[a], pb = lab[b];
        if (pa != a || pb != b) {
            a = pa;
            b = pb;
            continue;
        }
        const uint32_t lo = min(a, b), hi = max(a, b);
        const uint32_t old = atomicMin(lab + hi, lo);
        a = lo;
        b = old == hi ? lo : old;
    }
    if (a0 != a) lab[a0] = a;
    if (b0 != a) lab[b0] = a;
}

constexpr uint16_t kFaceRoot = 0x8000u;   // lroot flag: the component holds a face index (low bits: face position)

// The bytes of a thread's C cells in a plane, from flat cell index c on (C = 4:
// c is a multiple of 4 when L % 4 == 0, of 2 otherwise); n of them belong to
// the row (n even).
template <uint32_t C>
__device__ __forceinline__ uint32_t get_cells(const uint8_t* p, uint32_t c, uint32_t n, bool whole)
{
    if (C == 1) return p[c];
    if (whole) return *(const uint32_t*)(p + c);
    const uint32_t lo = *(const uint16_t*)(p + c);
    return n > 2 ? lo | ((uint32_t)*(const uint16_t*)(p + c + 2) << 16) : lo;
}

// A store written through L2 (see kThrough).
template <class V>
__device__ __forceinline__ void put_through(V* p, V v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

template <uint32_t C>
__device__ __forceinline__ void put_cells(uint8_t* p, uint32_t c, uint32_t n, bool whole, uint32_t v)
{
    if (C == 1) {
        p[c] = (uint8_t)v;
    } else if (whole) {
        *(uint32_t*)(p + c) = v;
    } else {
        *(uint16_t*)(p + c) = (uint16_t)v;
        if (n > 2) *(uint16_t*)(p + c + 2) = (uint16_t)(v >> 16);
    }
}

// C consecutive words of LDS (16-byte aligned for C = 4).
template <uint32_t C>
__device__ __forceinline__ void get_words(const uint32_t* p, uint32_t (&v)[C])
{
    if constexpr (C == 4) {
        const uint4 w = *(const uint4*)p;
        v[0] = w.x;
        v[1] = w.y;
        v[2] = w.z;
        v[3] = w.w;
    } else {
        v[0] = *p;
    }
}

template <uint32_t C>
__device__ __forceinline__ void put_words(uint32_t* p, const uint32_t (&v)[C])
{
    if constexpr (C == 4) *(uint4*)p = make_uint4(v[0], v[1], v[2], v[3]);
    else *p = v[0];
}

// The cells of a thread: the first one in the tile and in the lattice, and
// how many of the C exist.
template <class TL>
struct Cells3 {
    uint32_t lx, ly, lz, lc, x, y, z, c, n;
    bool whole;
    __device__ __forceinline__ Cells3(const TL& g, uint32_t L)
    {
        lc = TL::C * threadIdx.x;
        lx = lc % TL::TX;
        ly = (lc / TL::TX) % TL::TY;
        lz = lc / (TL::TX * TL::TY);
        x = g.x0 + lx;
        y = g.y0 + ly;
        z = g.z0 + lz;
        c = x + L * (y + L * z);
        n = (ly < g.h && lz < g.d && lx < g.w) ? min(TL::C, g.w - lx) : 0u;
        whole = L % 4 == 0;
    }
};

template <class TL>
__global__ __launch_bounds__(TL::TT) void sw3_tile_kernel(Lat3 a, TileGrid3 tg)
{
    constexpr uint32_t T = TL::T, C = TL::C, TT = TL::TT, TX = TL::TX, TY = TL::TY, NF = TL::NF, IDX = TL::kIdx;
    __shared__ __align__(16) uint32_t lab[6 * T];
    const uint32_t L = a.L, N = a.N, L2 = L * L;
    const TL g(L, xcd_tile(blockIdx.x, gridDim.x), tg.nx, tg.ny, tg.inx, tg.iny);
    const Cells3<TL> q(g, L);
    // link: the covalent links of cell j in bits 4 d + j
    uint32_t link = 0, coop[2] = {0, 0}, s[6] = {0, 0, 0, 0, 0, 0}, f[3] = {0, 0, 0}, e[3] = {0, 0, 0};
    {
        const uint32_t* src = reinterpret_cast<const uint32_t*>(&kArmTables);
        for (uint32_t i = threadIdx.x; i < sizeof(ArmTables) / 4; i += TT) lab[i] = src[i];
    }
    if (q.n) {
#pragma unroll
        for (int b = 0; b < 6; ++b) s[b] = get_cells<C>(a.sigma + (size_t)b * N, q.c, q.n, q.whole);
#pragma unroll
        for (int d = 0; d < 3; ++d) e[d] = get_cells<C>(a.eta + (size_t)d * N, q.c, q.n, q.whole);
        // facing arms: +x is this word moved down a byte, with the first byte
        // of the next quad (periodic) above the last cell
        const uint32_t xn = q.x + q.n == L ? q.c + q.n - L : q.c + q.n;
        const uint32_t nx = a.sigma[(size_t)N + xn];
        f[0] = (s[1] >> 8) | (nx << (8 * (q.n - 1)));
        f[1] = get_cells<C>(a.sigma + 3 * (size_t)N, q.y == L - 1 ? q.c + L - L2 : q.c + L, q.n, q.whole);
        f[2] = get_cells<C>(a.sigma + 5 * (size_t)N, q.z == L - 1 ? q.c + L2 - N : q.c + L2, q.n, q.whole);
        const uint32_t t = (uint32_t)a.st->t_cur;
        const int theta = a.st->theta, sgn = a.tab->jeff_sign;
        // word < threshold as word <= threshold - 1 (a threshold is at most
        // 2^32); a zero threshold allows no link
        const uint64_t ts64 = a.tab->sw_sigma, te64 = theta ? a.tab->sw_eff : 0;
        const uint32_t ts = (uint32_t)(ts64 - 1), te = (uint32_t)(te64 - 1);
        const bool coop_on = ts64 != 0, cov_on = te64 != 0 && sgn != 0;
        // links of cell j: of arms 0..3 in bits 0..5, of arm 4 in bits 6..9, of
        // arm 5 in bits 10..14 -- the indices of the tables
#pragma unroll 1
        for (uint32_t j = 0; j < C; ++j) {
            const uint32_t sh = 8 * j;
            uint32_t w[20], v[6];
#pragma unroll
            for (int b = 0; b < 5; ++b) {
                const uint4 r = philox(q.c + j, t, (uint32_t)b, kSwb, a.key0, a.key1);
                w[4 * b] = r.x;
                w[4 * b + 1] = r.y;
                w[4 * b + 2] = r.z;
                w[4 * b + 3] = r.w;
            }
#pragma unroll
            for (int b = 0; b < 6; ++b) v[b] = (s[b] >> sh) & 0xFFu;
            uint32_t on = 0;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const bool eq = v[2 * d] == ((f[d] >> sh) & 0xFFu);
                on |= (cov_on & (eq == (sgn > 0)) & (((e[d] >> sh) & 0xFFu) != 0) & (w[d] <= te)) ? 1u << (4 * d) : 0u;
            }
            uint32_t cm = 0;
            int l = 3;
#pragma unroll
            for (int i = 0; i < 6; ++i)
#pragma unroll
                for (int k = i + 1; k < 6; ++k, ++l) {
                    const uint32_t bit = 1u << (k == 5 ? 10 + i : k == 4 ? 6 + i : i == 0 ? k - 1 : i == 1 ? k + 1 : 5);
                    cm |= ((v[i] == v[k]) & (w[l] <= ts)) ? bit : 0u;
                }
            if (!coop_on) cm = 0;
            coop[j >> 1] |= cm << (16 * (j & 1));
            link |= (j < q.n ? on : 0u) << j;
        }
        // the old sigma facing the plus faces, and whether the link there is active
        const uint32_t last = q.n - 1;
        if (q.lx + q.n == g.w)
            a.edge[g.bx * L2 + q.z * L + q.y] = (uint8_t)(((f[0] >> (8 * last)) & 0xFFu) | (((link >> last) & 1u) << 7));
        if (q.ly == g.h - 1)
            for (uint32_t j = 0; j < q.n; ++j)
                a.edge[(g.nx + g.by) * L2 + q.z * L + q.x + j] =
                    (uint8_t)(((f[1] >> (8 * j)) & 0xFFu) | (((link >> (4 + j)) & 1u) << 7));
        if (q.lz == g.d - 1)
            for (uint32_t j = 0; j < q.n; ++j)
                a.edge[(g.nx + g.ny + g.bz) * L2 + q.y * L + q.x + j] =
                    (uint8_t)(((f[2] >> (8 * j)) & 0xFFu) | (((link >> (8 + j)) & 1u) << 7));
    }
    __syncthreads();
    uint32_t rt[C];                                        // root arm of arm k: bits 3 (k - 1)
    {
        const ArmTables& arms = *reinterpret_cast<const ArmTables*>(lab);
#pragma unroll
        for (uint32_t j = 0; j < C; ++j) {
            const uint32_t cm = coop[j >> 1] >> (16 * (j & 1));
            const uint32_t id5 = arms.five[16 * ((cm >> 6) & 15u) + arms.four[cm & 63u]];
            rt[j] = arms.six[52 * ((cm >> 10) & 31u) + id5];
        }
    }
    __syncthreads();                                       // the tables give way to the labels
    // In-cell roots, and the +x links between the thread's cells: a cell's
    // arm 1 continues the run of the previous cell's arm 0, and so does its
    // arm 0 when both arms are one component; parents point to the run's first
    // cell (arm 0, the smallest index)
    {
        uint32_t e0 = 0, lv[6][C];
#pragma unroll
        for (uint32_t j = 0; j < C; ++j) {
            const uint32_t lc = q.lc + j;
            const bool in_run = j && ((link >> (j - 1)) & 1u);
            const uint32_t r1 = in_run ? e0 : T + lc;
            if (!(in_run && (rt[j] & 7u) == 0)) e0 = lc;
            lv[0][j] = e0;
#pragma unroll
            for (uint32_t k = 1; k < 6; ++k) {
                const uint32_t r = (rt[j] >> (3 * (k - 1))) & 7u;
                lv[k][j] = r == 0 ? e0 : r == 1 ? r1 : r * T + lc;
            }
        }
#pragma unroll
        for (uint32_t k = 0; k < 6; ++k) put_words<C>(lab + k * T + q.lc, lv[k]);
    }
    __syncthreads();
    // Covalent links between the threads' cells.  A +y or +z link whose two
    // ends have the parents of an active link of an earlier cell of the thread
    // is implied by that one.
    if (q.n) {
        if (((link >> (q.n - 1)) & 1u) && q.lx + q.n < g.w) lds_join(lab, q.lc + q.n - 1, T + q.lc + q.n);
#pragma unroll
        for (uint32_t d = 1; d < 3; ++d) {
            if (d == 1 ? q.ly + 1 >= g.h : q.lz + 1 >= g.d) continue;
            const uint32_t u = 2 * d * T + q.lc, v = (2 * d + 1) * T + q.lc + (d == 1 ? TX : TX * TY);
            uint32_t pu[C], pv[C];
            get_words<C>(lab + u, pu);
            get_words<C>(lab + v, pv);
#pragma unroll
            for (uint32_t j = 0; j < C; ++j) {
                bool need = (link >> (4 * d + j)) & 1u;
#pragma unroll
                for (uint32_t k = 0; k < j; ++k)
                    need = need && !(((link >> (4 * d + k)) & 1u) && pu[j] == pu[k] && pv[j] == pv[k]);
                if (need) lds_join(lab, pu[j], pv[j]);
            }
        }
    }
    __syncthreads();
    // Flatten: every entry of the thread's cells to its root, two arms at a
    // time in lockstep (concurrent readers see the old parent or the root).
    uint32_t rp[6][(C + 1) / 2] = {};                      // roots of arm k: two cells in 16-bit halves
    if (q.n) {
#pragma unroll
        for (uint32_t h = 0; h < 3; ++h) {
            uint32_t r[2][C];
#pragma unroll
            for (uint32_t k = 0; k < 2; ++k) {
                get_words<C>(lab + (2 * h + k) * T + q.lc, r[k]);
                if (C == 4 && q.n == 2) {                  // past a ragged row's end: repeat cells that exist
                    r[k][C / 2] = r[k][0];
                    r[k][C - 1] = r[k][0];
                }
            }
            bool more = true;
            while (more) {
                uint32_t en[2][C];
                more = false;
#pragma unroll
                for (uint32_t k = 0; k < 2; ++k)
#pragma unroll
                    for (uint32_t j = 0; j < C; ++j) en[k][j] = lab[r[k][j]];
#pragma unroll
                for (uint32_t k = 0; k < 2; ++k)
#pragma unroll
                    for (uint32_t j = 0; j < C; ++j) {
                        more = more || en[k][j] != r[k][j];
                        r[k][j] = en[k][j];
                    }
            }
#pragma unroll
            for (uint32_t k = 0; k < 2; ++k) {
                put_words<C>(lab + (2 * h + k) * T + q.lc, r[k]);
#pragma unroll
                for (uint32_t j = 0; j < C; ++j) rp[2 * h + k][j / 2] |= r[k][j] << (16 * (j & 1));
            }
        }
    }
    __syncthreads();
    // Face indices: the root of each component that holds one records its
    // largest face position as representative (positions 0..NF-1 on the plus
    // faces, NF..2 NF-1 on the minus faces).  From here on a root's entry is
    // (representative + 1) << 16 | root.
    constexpr uint32_t FT = (NF + TT - 1) / TT;            // face positions per thread
    uint32_t rpl[FT], rmi[FT];                             // roots there, kNoIdx: none
#pragma unroll
    for (uint32_t k = 0; k < FT; ++k) {
        const uint32_t p = threadIdx.x + k * TT;
        uint32_t vp, vm;
        rpl[k] = rmi[k] = TL::kNoIdx;
        if (p < NF && g.face(p, vp, vm)) {
            rpl[k] = lab[vp] & IDX;
            rmi[k] = lab[vm] & IDX;
            atomicMax(lab + rpl[k], ((p + 1) << 16) | rpl[k]);
            atomicMax(lab + rmi[k], ((p + NF + 1) << 16) | rmi[k]);
        }
    }
    __syncthreads();
    if (q.n) {
#pragma unroll
        for (uint32_t k = 0; k < 6; ++k) {
            uint32_t o[(C + 1) / 2] = {};
#pragma unroll
            for (uint32_t j = 0; j < C; ++j) {
                const uint32_t r = (rp[k][j / 2] >> (16 * (j & 1))) & 0xFFFFu, rep = lab[r] >> 16;
                o[j / 2] |= (rep ? (kFaceRoot | (rep - 1)) : r) << (16 * (j & 1));
            }
            uint16_t* dst = a.lroot + (size_t)k * N + q.c;
            if (C == 1) {
                *dst = (uint16_t)o[0];
            } else if (q.whole) {
                put_through((uint64_t*)dst, o[0] | ((uint64_t)o[C / 4] << 32));
            } else {
                *(uint32_t*)dst = o[0];
                if (q.n > 2) *(uint32_t*)(dst + 2) = o[C / 4];
            }
        }
    }
#pragma unroll
    for (uint32_t k = 0; k < FT; ++k) {
        const uint32_t p = threadIdx.x + k * TT;
        if (rpl[k] == TL::kNoIdx) continue;
        const uint32_t F = g.nodes(L), me = g.node(L, p);
        const uint32_t ep = (lab[rpl[k]] >> 16) - 1, em = (lab[rmi[k]] >> 16) - 1;
        a.par[me] = g.node2(L, ep);
        a.par[F + me] = g.node2(L, em);
        if (ep == p) a.key[me] = g.flat(L, N, rpl[k]);
        if (em == p + NF) a.key[F + me] = g.flat(L, N, rmi[k]);
    }
}

// Hook the root with the larger key under the other (CAS on a root's own
// entry): keys strictly decrease along parents, so the root of a finished
// component is the node whose key is the cluster's smallest flat index.  Both
// chains are followed in lockstep, with the keys read beside the parents, so a
// hop costs one memory round trip (finding one root after the other, and the
// keys after both, took 37 us of a 128^3 step).
__device__ __forceinline__ void uf_unite(uint32_t* par, const uint32_t* key, uint32_t u, uint32_t v)
{
    const uint32_t u0 = u, v0 = v;
    while (u != v) {
        const uint32_t pu = par[u], pv = par[v], ku = key[u], kv = key[v];
        if (pu != u || pv != v) {
            u = pu;
            v = pv;
            continue;
        }
        const uint32_t hi = ku > kv ? u : v, lo = ku > kv ? v : u;
        const uint32_t old = atomicCAS(par + hi, hi, lo);
        u = lo;
        v = old == hi ? lo : old;
    }
    if (u0 != u) par[u0] = u;                              // no roots any more: point them at an ancestor
    if (v0 != u) par[v0] = u;
}

// One thread per plus node (face position i < F = L^2 (nx + ny + nz)).  A
// link whose two nodes have the same parents as the active link one place
// lower on the same face is already implied: a parent is an ancestor, so
// equal parents mean the same two components, and the lower link is united
// or itself implied by one lower still.  On a percolating cluster most face
// links repeat a neighbour's pair.
__global__ __launch_bounds__(kBlock) void sw3_union_kernel(Lat3 a, uint32_t nx, uint32_t ny, uint32_t nz)
{
    const uint32_t L = a.L, L2 = L * L, F = L2 * (nx + ny + nz);
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= F || !(a.edge[i] & 0x80u)) return;
    const uint32_t k = udiv(i, L2, a.invL * a.invL), uv = i - k * L2;
    const uint32_t v = udiv(uv, L, a.invL), u = uv - v * L;
    uint32_t nk = k + 1;                                   // the next tile along the axis, periodic
    if (k < nx) nk = nk == nx ? 0 : nk;
    else if (k < nx + ny) nk = nk == nx + ny ? nx : nk;
    else nk = nk == nx + ny + nz ? nx + ny : nk;
    const uint32_t m = F + nk * L2 + uv;
    // everything the tests below need in one round trip
    const uint32_t du = u ? 1u : 0u, dv = v ? L : 0u;
    const uint32_t pu = a.par[i], pv = a.par[m];
    const uint32_t eu = a.edge[i - du], ev = a.edge[i - dv];
    const uint32_t uu = a.par[i - du], uw = a.par[m - du], vu = a.par[i - dv], vw = a.par[m - dv];
    if (u && (eu & 0x80u) && uu == pu && uw == pv) return;
    if (v && (ev & 0x80u) && vu == pu && vw == pv) return;
    uf_unite(a.par, a.key, pu, pv);
}

// Shift of the cluster with label r: pick(word 0 of Philox(r, t, 0, SWF), q),
// NONE -> 0.
__device__ __forceinline__ uint32_t cluster_shift(const Lat3& a, uint32_t r, uint32_t t)
{
    const int k = pick_div(philox(r, t, 0u, kSwf, a.key0, a.key1).x, a.q);
    return k < 0 ? 0u : (uint32_t)k;
}

// One shift per component of the tile: interior components (their own
// smallest index is the label) are compacted into a list and drawn by
// consecutive threads; components with a face index, and the bond indices
// facing the tile's plus faces, follow the node chain to the label.  Then
// the new sigma, and N_HB_raw and N_sigma of the new configuration added to
// the counter slots.
template <class TL>
__global__ __launch_bounds__(TL::TT) __attribute__((amdgpu_waves_per_eu(8, 8))) void sw3_flip_kernel(Lat3 a, TileGrid3 tg)
{
    constexpr uint32_t T = TL::T, C = TL::C, TT = TL::TT, TX = TL::TX, TY = TL::TY, NF = TL::NF;
    // interior roots from the front, representatives from the back: every one
    // of them is another component's, so the two never meet
    __shared__ __align__(4) uint16_t roots[6 * T];
    __shared__ uint8_t sh[6 * T];
    __shared__ uint8_t shf[2 * NF];
    __shared__ uint8_t across[NF];
    __shared__ uint32_t count[2];
    uint8_t* nsg = reinterpret_cast<uint8_t*>(roots);      // the new sigma, once the root list is dead
    const uint32_t L = a.L, N = a.N, q = a.q, tid = threadIdx.x, lane = tid & 63;
    const TL g(L, xcd_tile(blockIdx.x, gridDim.x), tg.nx, tg.ny, tg.inx, tg.iny);
    const Cells3<TL> c4(g, L);
    uint32_t s[6] = {0, 0, 0, 0, 0, 0}, e[3] = {0, 0, 0};
    constexpr uint32_t W = (C + 1) / 2;
    uint32_t lr[6 * W];                                    // 16-bit roots of arm k, two cells per word
#pragma unroll
    for (uint32_t k = 0; k < 6 * W; ++k) lr[k] = TL::kNoIdx * 0x10001u;
    if (c4.n) {
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const uint16_t* src = a.lroot + (size_t)k * N + c4.c;
            if (C == 1) {
                lr[W * k] = *src;
            } else if (c4.whole) {
                const uint2 v = *(const uint2*)src;
                lr[W * k] = v.x;
                lr[W * k + W - 1] = v.y;
            } else {
                lr[W * k] = *(const uint32_t*)src;
                if (c4.n > 2) lr[W * k + W - 1] = *(const uint32_t*)(src + 2);
            }
            s[k] = get_cells<C>(a.sigma + (size_t)k * N, c4.c, c4.n, c4.whole);
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) e[d] = get_cells<C>(a.eta + (size_t)d * N, c4.c, c4.n, c4.whole);
    }
    auto LR = [&](uint32_t k, uint32_t j) { return (lr[W * k + (j >> 1)] >> (16 * (j & 1))) & 0xFFFFu; };
    const uint32_t t = (uint32_t)a.st->t_cur;
    if (tid < 2) count[tid] = 0;
    uint32_t own = 0;                                      // bit 4 k + j: arm k of cell j is an interior root
#pragma unroll
    for (uint32_t k = 0; k < 6; ++k)
#pragma unroll
        for (uint32_t j = 0; j < C; ++j) own |= (LR(k, j) == k * T + c4.lc + j ? 1u : 0u) << (4 * k + j);
    uint32_t tot;
    uint32_t pos = wave_excl_scan5((uint32_t)__popc(own), tot);
    __syncthreads();                                       // counts = 0
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(&count[0], tot);
    pos += (uint32_t)__shfl((int)base, 0, 64);
    while (own) {
        const uint32_t b = (uint32_t)__builtin_ctz(own);
        own &= own - 1;
        roots[pos++] = (uint16_t)((b >> 2) * T + c4.lc + (b & 3u));
    }
    // representatives among the face indices of these cells
    const uint32_t fx = c4.ly + TY * c4.lz, fy = TL::FX + c4.lx + TX * c4.lz, fz = TL::FX + TL::FY + c4.lx + TX * c4.ly;
    auto rep = [&](uint32_t k, uint32_t j, uint32_t p) {
        if (LR(k, j) == (kFaceRoot | p)) roots[6 * T - 1 - atomicAdd(&count[1], 1u)] = (uint16_t)p;
    };
    if (c4.n) {
        if (c4.lx + c4.n == g.w) {
            if (c4.n == C) rep(0, C - 1, fx);
            else rep(0, C / 4, fx);                        // C = 4, n = 2
        }
        if (c4.lx == 0) rep(1, 0, NF + fx);
#pragma unroll
        for (uint32_t j = 0; j < C; ++j) {
            if (c4.ly == g.h - 1) rep(2, j, fy + j);
            if (c4.ly == 0) rep(3, j, NF + fy + j);
            if (c4.lz == g.d - 1) rep(4, j, fz + j);
            if (c4.lz == 0) rep(5, j, NF + fz + j);
        }
    }
    __syncthreads();
    const uint32_t nroot = count[0], nrep = count[1];
    // Label chains: a representative's and that of the bond index facing a
    // plus face position together, so that their hops overlap.
    for (uint32_t i = tid; i < max(nrep, NF); i += TT) {
        const bool mine = i < nrep;
        uint32_t f = 0, x = 0, y = 0, xn = 0, yn = 0, old = 0, vp, vm;
        const bool far = i < NF && g.face(i, vp, vm);
        if (mine) {
            f = roots[6 * T - 1 - i];
            x = g.node2(L, f);
            y = a.par[x];
        }
        if (far) {
            const uint32_t np = g.node(L, i);
            xn = g.facing(L, i, np);
            yn = a.par[xn];
            old = a.edge[np] & 7u;
        }
        while (x != y || xn != yn) {
            x = y;
            xn = yn;
            y = mine ? a.par[x] : 0u;
            yn = far ? a.par[xn] : 0u;
        }
        const uint32_t r = mine ? a.key[x] : 0u, rn = far ? a.key[xn] : 0u;
        if (mine) shf[f] = (uint8_t)cluster_shift(a, r, t);
        if (far) {
            const uint32_t v = old + cluster_shift(a, rn, t);
            across[i] = (uint8_t)(v >= q ? v - q : v);
        }
    }
    for (uint32_t i = tid; i < nroot; i += TT) {
        const uint32_t v = roots[i];
        sh[v] = (uint8_t)cluster_shift(a, g.flat(L, N, v), t);
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < 6; ++k) {
        uint32_t nw = 0;
#pragma unroll
        for (uint32_t j = 0; j < C; ++j) {
            const uint32_t r = LR(k, j);
            if (j < c4.n) {
                const uint32_t v = ((s[k] >> (8 * j)) & 0xFFu) + ((r & kFaceRoot) ? shf[r & 0x7FFFu] : sh[r]);
                nw |= (v >= q ? v - q : v) << (8 * j);
            }
        }
        s[k] = nw;
        if (c4.n) put_cells<C>(a.sigma + (size_t)k * N, c4.c, c4.n, c4.whole, nw);
        put_cells<C>(nsg + k * T, c4.lc, C, true, nw);
    }
    __syncthreads();
    // recount: facing words in the tile or across its plus faces, equal bytes
    // counted four cells at a time
    int cnt[2] = {0, 0};
    if (c4.n) {
        const uint32_t have = c4.n == 4 ? 0x01010101u : (1u << (8 * c4.n)) / 0xFFu;
        const uint32_t nx = c4.lx + c4.n < g.w ? nsg[T + c4.lc + C] : across[fx];
        auto bytes = [](const uint8_t* p) {
            uint32_t v = p[0];
#pragma unroll
            for (uint32_t j = 1; j < C; ++j) v |= (uint32_t)p[j] << (8 * j);
            return v;
        };
        const uint32_t f[3] = {(s[1] >> 8) | (nx << (8 * (c4.n - 1))),
                               c4.ly + 1 < g.h ? get_cells<C>(nsg + 3 * T + c4.lc, TX, 4, true) : bytes(across + fy),
                               c4.lz + 1 < g.d ? get_cells<C>(nsg + 5 * T + c4.lc, TX * TY, 4, true) : bytes(across + fz)};
#pragma unroll
        for (uint32_t d = 0; d < 3; ++d) cnt[0] += __popc(zero_bytes(s[2 * d] ^ f[d]) & ~zero_bytes(e[d]) & have);
#pragma unroll
        for (int i = 0; i < 6; ++i)
#pragma unroll
            for (int j = i + 1; j < 6; ++j) cnt[1] += __popc(zero_bytes(s[i] ^ s[j]) & have);
    }
    __shared__ int part[2][TT / 64];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int sm = wave_sum(cnt[k]);
        if (lane == 0) part[k][tid >> 6] = sm;
    }
    __syncthreads();
    if (tid < 2) {
        int64_t sm = 0;
        for (uint32_t i = 0; i < TT / 64; ++i) sm += part[tid][i];
        if (sm) atomicAdd((unsigned long long*)(a.slots + (size_t)tid * kSlots + blockIdx.x % kSlots),
                          (unsigned long long)sm);
    }
}

// The label of every bond index, on request.  The chain of a face position is
// followed once per tile, by a lane of its own, and its label kept in LDS for
// the cells of its component (every bond index following its own chain took 85
// us at 128^3 and 300 K and 715 at 260^3, this 43 and 304).
template <class TL>
__global__ __launch_bounds__(TL::T) void sw3_labels_kernel(Lat3 a, TileGrid3 tg, uint32_t* __restrict__ out)
{
    constexpr uint32_t T = TL::T, TX = TL::TX, TY = TL::TY, NF = TL::NF;
    __shared__ uint32_t flab[2 * NF];
    const uint32_t L = a.L, N = a.N, tid = threadIdx.x;
    const TL g(L, xcd_tile(blockIdx.x, gridDim.x), tg.nx, tg.ny, tg.inx, tg.iny);
    const uint32_t lx = tid % TX, ly = (tid / TX) % TY, lz = tid / (TX * TY);
    const bool in = lx < g.w && ly < g.h && lz < g.d;
    const uint32_t c = (g.x0 + lx) + L * ((g.y0 + ly) + L * (g.z0 + lz));
    uint32_t lr[6];
#pragma unroll
    for (uint32_t k = 0; k < 6; ++k) lr[k] = in ? a.lroot[(size_t)k * N + c] : 0u;
    for (uint32_t f = tid; f < 2 * NF; f += T) {
        uint32_t vp, vm;
        if (!g.face(f < NF ? f : f - NF, vp, vm)) continue;
        uint32_t x = g.node2(L, f), y = a.par[x];
        while (y != x) {
            x = y;
            y = a.par[x];
        }
        flab[f] = a.key[x];
    }
    __syncthreads();
    if (!in) return;
#pragma unroll
    for (uint32_t k = 0; k < 6; ++k)
        out[(size_t)k * N + c] = (lr[k] & kFaceRoot) ? flab[lr[k] & 0x7FFFu] : g.flat(L, N, lr[k]);
}
