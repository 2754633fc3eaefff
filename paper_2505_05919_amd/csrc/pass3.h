// Arm-domain passes of the cubic lattice (included inside cvf3.hip's unnamed
// namespace, Sec. II.C): arm A of every cell moves once per pass, in the
// order drawn for the step.
//
// A pass reads the other arms of its own cell and arm A^1 of the neighbour in
// direction A.  Consecutive passes of which no two are opposite arms (a and
// a^1) therefore touch nothing that another lane writes: such a group runs in
// one launch, each lane taking its cells through the group's passes with the
// cells' six words in registers.  Six arms in any order make at most four
// groups (a group ends where the next arm's opposite is already in it, and
// there are three pairs), so a step is four launches, of which the last ones
// may find their group empty (two groups in 40 % of the orders, three in 53 %,
// four in 7 %); volume move and order are drawn on the device.  A group of
// three requests 12 bytes per cell and writes 3, against 8 + 1 for each single
// pass.
//
// A lane moves four x-adjacent cells (L % 4 == 2: the last quad of a row has
// two), deciding the four moves of a pass on packed bytes.  Bond indices are
// below 8, so (x ^ y) + 7 has bit 3 set exactly where two bytes differ.
// Measured at 260^3, 300 K: 153 us for the six passes of a step, about 180
// VALU instructions per quad and pass (72 of them the two Philox blocks),
// VALU issue the bound.  One launch per pass, with byte equality counted
// exactly for any byte value and the descriptors of a pass made anew, took
// 187 us at 276 instructions; at 32^3 the launches are the bound, 38 -> 20 us.
#pragma once

// One Philox block per cell pair and arm.  The pair index is the first counter
// word, the arm the third: the first round's product of the pair and the
// second round's product that follows from it are the same for every arm and
// are made once per pair.
struct PhiloxPair {
    uint32_t lo0, hi1, lo1;
};

__device__ __forceinline__ PhiloxPair philox_pair(uint32_t c0, uint32_t c3, uint32_t k1)
{
    PhiloxPair h;
    uint32_t hi0;
    mulhilo(0xD2511F53u, c0, hi0, h.lo0);
    mulhilo(0xCD9E8D57u, hi0 ^ c3 ^ k1, h.hi1, h.lo1);
    return h;
}

// philox(c0, c1, c2, c3, k0, k1) from philox_pair(c0, c3, k1).
__device__ __forceinline__ uint4 philox_rest(const PhiloxPair& h, uint32_t c1, uint32_t c2, uint32_t k0, uint32_t k1)
{
    uint32_t hi, lo, qh, ql;
    mulhilo(0xCD9E8D57u, c2, hi, lo);                     // round 1, uniform
    mulhilo(0xD2511F53u, hi ^ c1 ^ k0, qh, ql);           // round 2, uniform
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
    uint32_t a = h.hi1 ^ (lo ^ k0), b = h.lo1, c = h.lo0 ^ (qh ^ k1), d = ql;
#pragma unroll
    for (int r = 2; r < 10; ++r) {
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
        uint32_t h0, l0, h1, l1;
        mulhilo(0xD2511F53u, a, h0, l0);
        mulhilo(0xCD9E8D57u, c, h1, l1);
        a = __builtin_amdgcn_bitop3_b32(h1, b, k0, 0x96);
        c = __builtin_amdgcn_bitop3_b32(h0, d, k1, 0x96);
        b = l1;
        d = l0;
    }
    return make_uint4(a, b, c, d);
}

// Raw buffer over one plane (N bytes < 2^31): 32-bit lane offsets, base in SGPRs.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(uint8_t* base, uint32_t n)
{
    return __builtin_amdgcn_make_buffer_rsrc(base, (short)0, (int)n, 0x00020000);
}

__device__ __forceinline__ uint32_t bld8(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_amdgcn_raw_buffer_load_b8(r, (int)off, 0, 0);
}

// The four bytes of a quad at off; W: L % 4 == 0, one aligned dword, otherwise
// two halves, the high one repeating the low one where the quad has two cells.
template <bool W>
__device__ __forceinline__ uint32_t bld4(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t n)
{
    if (W) return __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0);
    const uint32_t lo = __builtin_amdgcn_raw_buffer_load_b16(r, (int)off, 0, 0);
    const uint32_t hi = __builtin_amdgcn_raw_buffer_load_b16(r, (int)(n > 2 ? off + 2 : off), 0, 0);
    return lo | (hi << 16);
}

struct Quad3 {
    uint32_t x, y, z, c, n;        // first cell, its flat index, cells (4, or 2 at the end of a row)
};

// Facing bond indices (arm A^1 of the neighbours) and the edges' eta of a
// quad's arm A.  The x arms' words borrow a byte from the next or previous
// quad of the row (periodic).
template <int A, bool W>
__device__ __forceinline__ void pass_load(const Lat3& a, const Quad3& q, const uint32_t (&ow)[6], uint32_t& fw,
                                          uint32_t& ew)
{
    const uint32_t L = a.L, N = a.N, L2 = L * L;
    if (A == 0) {                                         // arm 1 of x+1 .. x+n
        const uint32_t nx = q.x + q.n == L ? q.c + q.n - L : q.c + q.n;
        const uint32_t b = bld8(plane_rsrc(a.sigma + (size_t)N, N), nx);
        fw = W ? __builtin_amdgcn_alignbyte(b, ow[1], 1)
               : q.n == 4 ? (ow[1] >> 8) | (b << 24) : ((ow[1] >> 8) & 0xFFu) | (b << 8);
        ew = bld4<W>(plane_rsrc(a.eta, N), q.c, q.n);
    } else if (A == 1) {                                  // arm 0 of x-1 .. x+n-2
        const uint32_t px = q.x == 0 ? q.c + L - 1 : q.c - 1;
        const __amdgpu_buffer_rsrc_t e0 = plane_rsrc(a.eta, N);
        fw = (ow[0] << 8) | bld8(plane_rsrc(a.sigma, N), px);
        ew = (bld4<W>(e0, q.c, q.n) << 8) | bld8(e0, px);
    } else {
        const uint32_t o = A == 2 ? (q.y == L - 1 ? q.c + L - L2 : q.c + L)
                         : A == 3 ? (q.y == 0 ? q.c + L2 - L : q.c - L)
                         : A == 4 ? (q.z == L - 1 ? q.c + L2 - N : q.c + L2)
                                  : (q.z == 0 ? q.c + N - L2 : q.c - L2);
        fw = bld4<W>(plane_rsrc(a.sigma + (size_t)(A ^ 1) * N, N), o, q.n);
        ew = bld4<W>(plane_rsrc(a.eta + (size_t)(A >> 1) * N, N), (A & 1) ? o : q.c, q.n);
    }
}

// Sums of a lane over its accepted moves, as the packed bytes give them.
struct PassSums {
    uint32_t bits;                 // 8 per accepted move
    uint32_t dc;                   // 64 + 8 dc
    uint32_t ho, hn;               // old / new value unlike the facing one, eta = 1
};

// The moves of arm A of one quad (the oracle's moves, four at a time):
// proposal sigma + 1 + k mod q with k uniform over the q - 1 other states,
// accepted through the table of (theta eta, dh, dc).  LE: the table holds
// thr - 1 (2^32 - 1 for "always"), valid when no threshold is 0, and a move is
// accepted iff word <= entry.
template <int A, int Q, bool LE, bool W>
__device__ __forceinline__ void pass_move(const Lat3& a, const uint32_t* tab, const Quad3& q, uint32_t t, int theta,
                                          const PhiloxPair (&ph)[2], uint32_t (&ow)[6], uint32_t fw, uint32_t ew,
                                          PassSums& sums)
{
    constexpr uint32_t M = Q - 1, kOne = 0x01010101u;
    // M in {3, 5} divides 2^32 - 1: word 2^32 - 1 is no proposal (NONE), and
    // comes out below as k + 1 = q, the old state
    constexpr bool kHasNone = M == 3 || M == 5;
    const uint4 w0 = philox_rest(ph[0], t, (uint32_t)A, a.key0, a.key1);
    const uint4 w1 = philox_rest(ph[1], t, (uint32_t)A, a.key0, a.key1);
    const uint32_t prop[4] = {w0.x, w0.z, w1.x, w1.z}, accw[4] = {w0.y, w0.w, w1.y, w1.w};
    const uint32_t oldw = ow[A];
    uint32_t kw = 0;                                      // k + 1 of the four cells
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t kp = (uint32_t)(((uint64_t)prop[j] * M + ((1ull << 32) + (kHasNone ? M : 0u))) >> 32);
        kw |= kp << (8 * j);
    }
    const uint32_t sum = oldw + kw;                       // sigma + 1 + k <= 2q - 1
    const uint32_t ge = (sum + (16 - Q) * kOne) & (16 * kOne);   // 16 where it reaches q
    const uint32_t nw = sum - ((Q & 4 ? ge >> 2 : 0u) + (Q & 2 ? ge >> 3 : 0u) + (Q & 1 ? ge >> 4 : 0u));
    // 8 per other arm unlike the new (un) and the old (uo) state
    uint32_t un = 0, uo = 0;
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        if (b == A) continue;
        un += ((nw ^ ow[b]) + 7 * kOne) & (8 * kOne);
        uo += ((oldw ^ ow[b]) + 7 * kOne) & (8 * kOne);
    }
    const uint32_t hn = ((nw ^ fw) + 7 * kOne) & (8 * kOne), ho = ((oldw ^ fw) + 7 * kOne) & (8 * kOne);
    const uint32_t dc = uo + 64 * kOne - un;              // 64 + 8 dc, dc in -5..5
    const uint32_t h1 = (ho + 8 * kOne - hn) >> 3;        // dh + 1
    uint32_t e8 = ew << 8;
    __asm__("" : "+v"(e8));                                // no instruction: keeps the next line from becoming a multiply
    const uint32_t eta = e8 - ew;                         // 0xFF where the edge has eta = 1
    const uint32_t gate = theta ? eta : 0u;
    // byte offset of the table entry: 4 dc + 32, + 44 (dh + 1) or + 132 when
    // theta eta = 0 (there dh costs nothing)
    const uint32_t off = (dc >> 1) + ((((h1 << 5) + (h1 << 3) + (h1 << 2)) & gate) | (132 * kOne & ~gate));
    uint32_t acc = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t thr = *(const uint32_t*)((const char*)tab + ((off >> (8 * j)) & 0xFFu));
        const bool ok = LE ? accw[j] <= thr : min(accw[j], 0xFFFFFFFEu) < thr;   // thr = 2^32 - 1 always accepts
        acc |= ok ? 0xFFu << (8 * j) : 0u;
    }
    if (kHasNone && max(max(prop[0], prop[1]), max(prop[2], prop[3])) == 0xFFFFFFFFu) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (prop[j] == 0xFFFFFFFFu) acc &= ~(0xFFu << (8 * j));
    }
    if (!W && q.n == 2) acc &= 0xFFFFu;
    const uint32_t out = (nw & acc) | (oldw & ~acc), counted = acc & eta;
    sums.bits += __popc(acc);
    sums.dc = __builtin_amdgcn_sad_u8(dc & acc, 0u, sums.dc);
    sums.ho += __popc(ho & counted);
    sums.hn += __popc(hn & counted);
    ow[A] = out;
    if (out != oldw) {
        const __amdgpu_buffer_rsrc_t r = plane_rsrc(a.sigma + (size_t)A * a.N, a.N);
        if (W) {
            __builtin_amdgcn_raw_buffer_store_b32(out, r, (int)q.c, 0, cvf::kThrough);
        } else {
            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)out, r, (int)q.c, 0, cvf::kThrough);
            if (q.n > 2) __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(out >> 16), r, (int)q.c + 2, 0, cvf::kThrough);
        }
    }
}

#define CVF3_ARM(arm, f, ...)                     \
    switch (arm) {                                \
    case 0: f<0, __VA_ARGS__; break;              \
    case 1: f<1, __VA_ARGS__; break;              \
    case 2: f<2, __VA_ARGS__; break;              \
    case 3: f<3, __VA_ARGS__; break;              \
    case 4: f<4, __VA_ARGS__; break;              \
    default: f<5, __VA_ARGS__; break;             \
    }

// Quads of a row, and a lane's stride of `step` quads as (quads, rows, planes).
struct PassShape {
    uint32_t per_row, quads;       // quads per row, in all
    uint32_t sj, sy, sz;           // stride between a lane's quads
    double inv_row;                // 1 / per_row
};

constexpr uint32_t kMaxQuadsPerLane = 4;

template <int Q, bool LE, bool W>
__global__ __launch_bounds__(kBlock) void pass3_kernel(Lat3 a_, PassShape sh)
{
    Lat3 a = a_;
    // the group of this launch: passes s0 .. s1 - 1 of the step's order
    const uint32_t ends = a.st->group_end;
    const uint32_t s0 = a.pass ? (ends >> (8 * (a.pass - 1))) & 0xFFu : 0u, s1 = (ends >> (8 * a.pass)) & 0xFFu;
    if (s0 == s1) return;
    // 3 words unused, then [dh + 1][dc + 5] for theta eta = 1, then [dc + 5]
    // for theta eta = 0, then unused ones, so that a move's byte offset (see
    // pass_move) stays inside whatever bytes a kept configuration holds
    __shared__ uint32_t tab[64];
    static_assert(sizeof(tab) > 0xFF, "every byte offset lies in the table");
    if (threadIdx.x >= 3 && threadIdx.x < 47) {
        const uint32_t k = threadIdx.x - 3;
        const uint32_t thr = k < 33 ? (&a.tab->met[1][0][0])[k] : a.tab->met[0][1][k - 33];
        tab[threadIdx.x] = LE ? (thr == 0xFFFFFFFFu ? thr : thr - 1u) : thr;
    }
    const uint32_t ng = s1 - s0;
    const int arm0 = a.st->order[s0], arm1 = a.st->order[min(s0 + 1, 5u)], arm2 = a.st->order[min(s0 + 2, 5u)];
    const uint32_t t = (uint32_t)a.st->t_cur;
    const int theta = a.st->theta;
    const uint32_t L = a.L;
    uint32_t u = blockIdx.x * kBlock + threadIdx.x;
    uint32_t yz = udiv(u, sh.per_row, sh.inv_row), j = u - yz * sh.per_row;
    uint32_t z = udiv(yz, L, a.invL), y = yz - z * L;
    __syncthreads();
    PassSums sums = {0, 0, 0, 0};
    for (; u < sh.quads; u += gridDim.x * kBlock) {
        // Empty asm, no instruction: plane descriptors and round keys are made
        // again in scalar registers where they are used, instead of being kept
        // (and spilled) across the whole loop.
        __asm__ volatile("" : "+s"(a.N), "+s"(a.key0), "+s"(a.key1));
        Quad3 q;
        q.x = 4 * j;
        q.y = y;
        q.z = z;
        q.c = q.x + L * (y + L * z);
        q.n = W || q.x + 4 <= L ? 4u : 2u;
        uint32_t ow[6], f0, e0, f1 = 0, e1 = 0, f2 = 0, e2 = 0;
#pragma unroll
        for (int b = 0; b < 6; ++b) ow[b] = bld4<W>(plane_rsrc(a.sigma + (size_t)b * a.N, a.N), q.c, q.n);
        CVF3_ARM(arm0, pass_load, W>(a, q, ow, f0, e0))
        if (ng > 1) CVF3_ARM(arm1, pass_load, W>(a, q, ow, f1, e1))
        if (ng > 2) CVF3_ARM(arm2, pass_load, W>(a, q, ow, f2, e2))
        const PhiloxPair ph[2] = {philox_pair(q.c / 2, kDom, a.key1), philox_pair(q.c / 2 + 1, kDom, a.key1)};
        CVF3_ARM(arm0, pass_move, Q, LE, W>(a, tab, q, t, theta, ph, ow, f0, e0, sums))
        if (ng > 1) CVF3_ARM(arm1, pass_move, Q, LE, W>(a, tab, q, t, theta, ph, ow, f1, e1, sums))
        if (ng > 2) CVF3_ARM(arm2, pass_move, Q, LE, W>(a, tab, q, t, theta, ph, ow, f2, e2, sums))
        j += sh.sj;
        y += sh.sy;
        z += sh.sz;
        if (j >= sh.per_row) {
            j -= sh.per_row;
            ++y;
        }
        if (y >= L) {
            y -= L;
            ++z;
        }
    }
    // A lane's 48 moves at most (four quads, three passes): d N_sigma in
    // [-240, 240] and d N_HB_raw in [-48, 48], biased into 16-bit halves of one
    // word whose sums over 64 lanes stay below 2^16.
    static_assert(kMaxQuadsPerLane <= 4, "the halves below hold 48 moves per lane");
    const int acc = (int)(sums.bits / 8), dc = ((int)sums.dc - 64 * acc) / 8, dh = (int)sums.ho - (int)sums.hn;
    const uint32_t v = (uint32_t)wave_sum((int)((uint32_t)(dc + 240) | ((uint32_t)(dh + 48) << 16)));
    const int na = wave_sum(acc);
    __shared__ int part[3][kBlock / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
        part[0][wv] = (int)(v >> 16) - 48 * 64;
        part[1][wv] = (int)(v & 0xFFFFu) - 240 * 64;
        part[2][wv] = na;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        int64_t sm = 0;
        for (int i = 0; i < kBlock / 64; ++i) sm += part[threadIdx.x][i];
        if (sm) atomicAdd((unsigned long long*)(a.slots + (size_t)threadIdx.x * kSlots + blockIdx.x % kSlots),
                          (unsigned long long)sm);
    }
}
