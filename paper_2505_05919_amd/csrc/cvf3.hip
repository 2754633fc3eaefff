// CVF water model on the periodic simple-cubic lattice with the eta bond
// constraint (Sec. II.A-C, App. A): device kernels and the cvf3_* C ABI.
//
// One MC step on the caller's stream (Sec. II.B):
//   vol3_kernel   one workgroup: folds the previous step's per-workgroup
//                 counter slots, performs the FP64 volume move, draws the
//                 order of the six arm passes
//   eta3_kernel   one thread per checkerboard cube: Metropolis move of the
//                 cube's eta configuration (one of the nine perfect matchings
//                 of the cube graph marks the eta = 0 edges)
//   pass3_kernel  x4: the six arm passes in the drawn order (the arm-domain
//                 partition of Sec. II.C), grouped so that no two passes of a
//                 launch are opposite arms
// A Swendsen-Wang step (Sec. II.D) replaces the passes by sw3_tile_kernel
// (links, components inside a tile), sw3_union_kernel (tile-crossing links,
// global union-find over the tiles' face indices) and sw3_flip_kernel (cluster
// shifts and the recount).
// Layout: sigma[a*N + c], eta[d*N + c] (edge from c to its +d neighbour),
// c = x + L*(y + L*z); arms 0:+x 1:-x 2:+y 3:-y 4:+z 5:-z.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "cvf.h"
#include "cvf3.h"
#include "dispatch.h"

namespace {

#include "philox.h"
#include "wave.h"

constexpr uint32_t kInit = 0, kVol = 1, kSwb = 3, kSwf = 4, kOrd = 5, kDom = 6, kEta = 7;
constexpr int kSlots = 256;              // counter slots, spread to avoid one hot atomic
constexpr int kAcc = 4;                  // d N_HB_raw, d N_sigma, sigma accepted, eta accepted
constexpr int kRc = 10;                  // recount: N_HB_raw, N_sigma, N_q' (6), eta = 0 edges, spare
constexpr int kRcSpread = 16, kRcBlocks = 1024;
constexpr int kRcState = kRc * kRcSpread;    // word of the recount area where a fold leaves a copy of the state
constexpr int kBlock = 256;

struct Dev3State {
    double  v, u;
    int64_t t_next, t_cur;
    int64_t n_hb_raw, n_coop;
    int64_t met_att, met_acc, eta_att, eta_acc, vol_att, vol_acc;
    int32_t theta;
    uint32_t group_end;       // byte g: passes of the step's order up to the end of pass group g
    int32_t order[6];
    int32_t pad[2];
};
static_assert(sizeof(Dev3State) % 8 == 0 && sizeof(Dev3State) <= 64 * 8, "copied as words, one per lane");

struct Tab3 {
    uint32_t met[2][3][11];   // sigma move: [theta*eta][dh+1][dc+5]
    uint32_t eta[9];          // eta move in the liquid: [dn+4]
    uint32_t match[9];        // perfect matchings of the cube graph (12-bit edge masks, eta = 0)
    uint64_t sw_sigma, sw_eff; // SW bond thresholds floor(p 2^32): cooperative, covalent (liquid)
    int32_t  jeff_sign;        // sign of J_eff
    double   r3[40];          // r3(m), m = 0..36
};

struct Lat3 {
    uint8_t*   sigma;
    uint8_t*   eta;
    Dev3State* st;
    int64_t*   slots;         // [kAcc][kSlots]
    int64_t*   rc;            // recount sums [kRc][kRcSpread], then a copy of the state
    const Tab3* tab;          // device copy
    // Swendsen-Wang only (NULL without it); F plus nodes, see sw3_step.h
    uint32_t*  par;           // [2F] parents of the tile-face nodes
    uint32_t*  key;           // [2F] smallest flat index of a representative's component
    uint16_t*  lroot;         // [6N] tile-local root of every bond index, or its component's face position
    uint8_t*   edge;          // [F] old sigma facing a plus face, bit 7: the link there is active
    uint32_t L, N, h, q;
    uint32_t key0, key1;
    uint32_t pass;
    uint32_t quad;            // 1: L % 4 == 0, quads of four cells; 0: the last quad of a row has two
    uint32_t eta_hb;          // 1: the eta move adds its change of N_HB_raw to the counters
    double   invL, invH, invQ4, Nd, beta, J, P, vHB, dv_max;
    int32_t  do_volume;
};

__device__ __forceinline__ uint32_t udiv(uint32_t n, uint32_t d, double inv)
{
    uint32_t q = (uint32_t)((double)n * inv);
    const int64_t r = (int64_t)n - (int64_t)q * d;
    if (r < 0) --q;
    else if (r >= (int64_t)d) ++q;
    return q;
}


// U_LJ per molecule on the cubic lattice (Sec. II.A): shells m = |n|^2 in
// ascending order, (distance/r0)^6 = v^2 m^3, cutoff 6^6.
__device__ __host__ double lj3(double v, const double* r3)
{
    double s = 0.0;
    for (int m = 1; m <= 36; ++m) {
        const double d6 = (v * v) * (double)(m * m * m);
        if (!(d6 <= 46656.0)) break;
        const double s6 = 1.0 / d6;
        s = s + r3[m] * (s6 * s6 - s6);
    }
    return 2.0 * s;
}

// Uniform draw of {0..k-1} from one word by the exact-block rule (NONE = -1
// when the word falls in the incomplete top block).
__device__ __forceinline__ int pick_div(uint32_t w, uint32_t k)
{
    const uint32_t d = (uint32_t)(4294967296ull / k);
    if ((uint64_t)w >= (uint64_t)k * d) return -1;
    return (int)(w / d);
}

// Corner vtx (bit 0: +x, 1: +y, 2: +z) of cube k: parity k / h^3 sets the
// lowest corner (2i+par, 2j+par, 2l+par).
struct Cube {
    uint32_t x0, y0, z0;
};

__device__ __forceinline__ Cube cube_of(const Lat3& a, uint32_t k)
{
    const uint32_t h3 = a.h * a.h * a.h;
    const uint32_t par = k >= h3 ? 1u : 0u;
    const uint32_t r = k - par * h3;
    const uint32_t jl = udiv(r, a.h, a.invH);
    const uint32_t i = r - jl * a.h;
    const uint32_t l = udiv(jl, a.h, a.invH);
    const uint32_t j = jl - l * a.h;
    return {2 * i + par, 2 * j + par, 2 * l + par};
}

__device__ __forceinline__ uint32_t cell_at(const Lat3& a, const Cube& q, uint32_t vtx)
{
    uint32_t x = q.x0 + (vtx & 1), y = q.y0 + ((vtx >> 1) & 1), z = q.z0 + ((vtx >> 2) & 1);
    x = x == a.L ? 0 : x;
    y = y == a.L ? 0 : y;
    z = z == a.L ? 0 : z;
    return x + a.L * (y + a.L * z);
}

// Ends of cube edge e: axis d = e / 4, r = e % 4 places it along the two
// other axes (lower axis in bit 0).
__device__ __forceinline__ void edge_vtx(int e, uint32_t& lo, uint32_t& hi)
{
    const int d = e >> 2, r = e & 3;
    uint32_t v;
    if (d == 0) v = ((r & 1) << 1) | ((r >> 1) << 2);
    else if (d == 1) v = (r & 1) | ((r >> 1) << 2);
    else v = (r & 1) | ((r >> 1) << 1);
    lo = v;
    hi = v | (1u << d);
}

// ---------------------------------------------------------------------------
// Initial state: sigma of cell c from words 0..3 of Philox(c, 0, 0, INIT) and
// words 0, 1 of Philox(c, 0, 1, INIT); eta of cube k from configuration
// pick(word 0 of Philox(k, 0, 2, INIT), 9), NONE -> 0.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void init3_sigma_kernel(Lat3 a)
{
    const uint32_t c = blockIdx.x * kBlock + threadIdx.x;
    if (c >= a.N) return;
    const uint4 w0 = philox(c, 0u, 0u, kInit, a.key0, a.key1);
    const uint4 w1 = philox(c, 0u, 1u, kInit, a.key0, a.key1);
    const uint32_t w[6] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y};
#pragma unroll
    for (int b = 0; b < 6; ++b) a.sigma[(size_t)b * a.N + c] = (uint8_t)(((uint64_t)w[b] * a.q) >> 32);
}

__global__ __launch_bounds__(kBlock) void init3_eta_kernel(Lat3 a)
{
    const uint32_t k = blockIdx.x * kBlock + threadIdx.x;
    if (k >= a.N / 4) return;
    const uint4 w = philox(k, 0u, 2u, kInit, a.key0, a.key1);
    int m = pick_div(w.x, 9);
    if (m < 0) m = 0;
    const uint32_t mask = a.tab->match[m];
    const Cube q = cube_of(a, k);
#pragma unroll
    for (int e = 0; e < 12; ++e) {
        uint32_t lo, hi;
        edge_vtx(e, lo, hi);
        a.eta[(size_t)(e >> 2) * a.N + cell_at(a, q, lo)] = (uint8_t)(((mask >> e) & 1) ^ 1);
    }
}

__global__ void state3_init_kernel(Lat3 a, double v_init)
{
    for (int i = threadIdx.x; i < kAcc * kSlots; i += blockDim.x) a.slots[i] = 0;
    if (threadIdx.x == 0) {
        Dev3State* s = a.st;
        memset(s, 0, sizeof(*s));
        s->v = v_init;
        s->u = lj3(v_init, a.tab->r3);
        s->theta = v_init < 2.0 ? 1 : 0;
        for (int i = 0; i < 6; ++i) s->order[i] = i;
        s->group_end = 0x06060606u;
    }
}

constexpr int kVolMet = 0, kVolFold = 1, kVolSw = 2;

// ---------------------------------------------------------------------------
// Counter fold + volume move (Sec. II.B step 1) + pass order of the step.
// dH = N (u(v') - u(v)) + P N (v' - v) + (theta' - theta)(P v_HB - J) N_HB_raw
// with words 0, 1 of Philox(0, t, 0, VOL); order: Fisher-Yates over 0..5
// with words 0..3 of Philox(0, t, 0, ORD) and word 0 of Philox(0, t, 1, ORD).
// mode 0: full step opening; mode 1: fold only (clears the recount's sums and
// leaves a copy of the folded state behind them, so that one copy to the host
// brings both).
// ---------------------------------------------------------------------------
// One wavefront: lanes fold the counter slots (kSlots / 64 each), lanes 0-2
// draw the VOL block and the two ORD blocks at once, lanes 1..36 evaluate one
// U_LJ shell term each; lane 0 then sums the terms in ascending shell order
// up to the first shell beyond the cutoff (the order of lj3) and takes the
// decisions.  Every global load (slots, chain state, shell counts) is issued
// before the first store, and the four slot sums share one butterfly.
__global__ __launch_bounds__(64) void vol3_kernel(Lat3 a, int mode)
{
    __shared__ double term[40];
    __shared__ uint32_t words[3][4];
    const int lane = threadIdx.x;
    Dev3State* s = a.st;
    int64_t sl[kAcc][kSlots / 64];
#pragma unroll
    for (int k = 0; k < kAcc; ++k)
#pragma unroll
        for (int j = 0; j < kSlots / 64; ++j) sl[k][j] = a.slots[k * kSlots + j * 64 + lane];
    const uint32_t t = (uint32_t)s->t_next;
    const int64_t t_next = s->t_next;
    const double v0 = s->v, u0 = s->u;
    const int th0 = s->theta;
    const int64_t hb0 = s->n_hb_raw, co0 = s->n_coop, ma0 = s->met_acc, ea0 = s->eta_acc;
    const int64_t matt0 = s->met_att, eatt0 = s->eta_att, vatt0 = s->vol_att, vacc0 = s->vol_acc;
    const double r3 = (lane >= 1 && lane <= 36) ? a.tab->r3[lane] : 0.0;
    constexpr int kWords = sizeof(Dev3State) / 8;
    const int64_t word = lane < kWords ? ((const int64_t*)s)[lane] : 0;
    int64_t r[kAcc];
#pragma unroll
    for (int k = 0; k < kAcc; ++k) {
        r[k] = 0;
#pragma unroll
        for (int j = 0; j < kSlots / 64; ++j) {
            r[k] += sl[k][j];
            a.slots[k * kSlots + j * 64 + lane] = 0;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        int64_t x[kAcc];
#pragma unroll
        for (int k = 0; k < kAcc; ++k) x[k] = __shfl_xor(r[k], o, 64);
#pragma unroll
        for (int k = 0; k < kAcc; ++k) r[k] += x[k];
    }
    if (mode != kVolFold && lane < 3) {
        const uint4 w = philox(0u, t, lane == 2 ? 1u : 0u, lane == 0 ? kVol : kOrd, a.key0, a.key1);
        words[lane][0] = w.x;
        words[lane][1] = w.y;
        words[lane][2] = w.z;
        words[lane][3] = w.w;
    }
    __syncthreads();
    double v1 = 0.0;
    bool inside = false;
    if (mode != kVolFold && a.do_volume) {
        const double u = (double)((int64_t)2 * (int64_t)words[0][0] + 1 - 4294967296LL) * (1.0 / 4294967296.0);
        v1 = v0 + a.dv_max * u;
        inside = v1 >= 1.0;
        if (inside && lane >= 1 && lane <= 36) {
            const double d6 = (v1 * v1) * (double)(lane * lane * lane);
            const double s6 = 1.0 / d6;
            term[lane] = d6 <= 46656.0 ? r3 * (s6 * s6 - s6) : 0.0;
        }
    }
    __syncthreads();
    Dev3State* copy = (Dev3State*)(a.rc + kRcState);
    if (mode == kVolFold) {
        for (int i = lane; i < kRcState; i += 64) a.rc[i] = 0;
        if (lane < kWords) ((int64_t*)copy)[lane] = word;
        __builtin_amdgcn_s_waitcnt(0);                     // before lane 0 writes the folded counters into it
    }
    if (lane != 0) return;
    const int64_t n_hb = hb0 + r[0];
    if (mode == kVolFold) {
        copy->n_hb_raw = n_hb;
        copy->n_coop = co0 + r[1];
        copy->met_acc = ma0 + r[2];
        copy->eta_acc = ea0 + r[3];
    }
    s->n_hb_raw = n_hb;
    s->n_coop = co0 + r[1];
    s->met_acc = ma0 + r[2];
    s->eta_acc = ea0 + r[3];
    if (mode == kVolFold) return;
    if (a.do_volume) {
        s->vol_att = vatt0 + 1;
        if (inside) {
            // all 36 terms read first, then added in ascending m while within
            // the cutoff: the condition is monotone in m, so the terms added
            // and their order are those of the loop that stops at the first
            // shell beyond it
            double tm[36];
#pragma unroll
            for (int m = 1; m <= 36; ++m) tm[m - 1] = term[m];
            double sum = 0.0;
#pragma unroll
            for (int m = 1; m <= 36; ++m) {
                const double d6 = (v1 * v1) * (double)(m * m * m);
                if (d6 <= 46656.0) sum = sum + tm[m - 1];
            }
            const double u1 = 2.0 * sum;
            const int th1 = v1 < 2.0 ? 1 : 0;
            const double dH = (a.Nd * (u1 - u0)) + ((a.P * a.Nd) * (v1 - v0))
                            + (((double)(th1 - th0) * (a.P * a.vHB - a.J)) * (double)n_hb);
            bool acc = dH <= 0.0;
            if (!acc) acc = ((double)words[0][1] + 0.5) * (1.0 / 4294967296.0) < exp(-a.beta * dH);
            if (acc) {
                s->v = v1;
                s->u = u1;
                s->theta = th1;
                s->vol_acc = vacc0 + 1;
            }
        }
    }
    const uint32_t ow[5] = {words[1][0], words[1][1], words[1][2], words[1][3], words[2][0]};
    int ord[6] = {0, 1, 2, 3, 4, 5};
    for (int i = 0; i < 5; ++i) {
        int k = pick_div(ow[i], (uint32_t)(6 - i));
        if (k < 0) k = 0;
        const int tmp = ord[i];
        ord[i] = ord[i + k];
        ord[i + k] = tmp;
    }
    // groups of consecutive passes without opposite arms (at most four)
    uint32_t ends = 0x06060606u, seen = 0, g = 0;
    for (uint32_t i = 0; i < 6; ++i) {
        s->order[i] = ord[i];
        if ((seen >> (ord[i] ^ 1)) & 1u) {
            ends ^= (6u ^ i) << (8 * g++);
            seen = 0;
        }
        seen |= 1u << ord[i];
    }
    s->group_end = ends;
    s->t_cur = t;
    s->t_next = t_next + 1;
    if (mode == kVolMet) {
        s->met_att = matt0 + 6 * (int64_t)a.N;
    } else {                                       // the SW step ends with a full recount
        s->n_hb_raw = 0;
        s->n_coop = 0;
    }
    s->eta_att = eatt0 + a.N / 4;
}

// ---------------------------------------------------------------------------
// eta update (Sec. II.B step 2, App. A): one thread per cube.  Proposal
// pick(w0, 9) of Philox(k, t, 0, ETA) (NONE: no move); dn = change of
// N_HB_raw inside the cube; accepted through the eta table and w1 in the
// liquid, always in the gas.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void eta3_kernel(Lat3 a)
{
    const uint32_t k = blockIdx.x * kBlock + threadIdx.x;
    int cnt[2] = {0, 0};
    if (k < a.N / 4) {
        const uint32_t t = (uint32_t)a.st->t_cur;
        const int theta = a.st->theta;
        const uint4 w = philox(k, t, 0u, kEta, a.key0, a.key1);
        const int m = pick_div(w.x, 9);
        if (m >= 0) {
            const uint32_t mask = a.tab->match[m];
            const Cube q = cube_of(a, k);
            uint32_t cell[8];
#pragma unroll
            for (int v = 0; v < 8; ++v) cell[v] = cell_at(a, q, v);
            int dn = 0;
            uint32_t old = 0;
#pragma unroll
            for (int e = 0; e < 12; ++e) {
                uint32_t lo, hi;
                edge_vtx(e, lo, hi);
                const int d = e >> 2;
                const int eq = a.sigma[(size_t)(2 * d) * a.N + cell[lo]] == a.sigma[(size_t)(2 * d + 1) * a.N + cell[hi]];
                const int eo = a.eta[(size_t)d * a.N + cell[lo]];
                old |= (uint32_t)eo << e;
                const int en = (int)(((mask >> e) & 1) ^ 1);
                dn += (en - eo) * eq;
            }
            bool acc = true;
            if (theta) {
                const uint32_t thr = a.tab->eta[dn + 4];
                acc = thr == 0xFFFFFFFFu || w.y < thr;
            }
            if (acc) {
                cnt[0] = a.eta_hb ? dn : 0;
                cnt[1] = 1;
                const uint32_t neu = (~mask) & 0xFFFu;
                if (neu != old) {
#pragma unroll
                    for (int e = 0; e < 12; ++e) {
                        uint32_t lo, hi;
                        edge_vtx(e, lo, hi);
                        if (((neu ^ old) >> e) & 1)
                            a.eta[(size_t)(e >> 2) * a.N + cell[lo]] = (uint8_t)((neu >> e) & 1);
                    }
                }
            }
        }
    }
    int v4[2] = {cnt[0], cnt[1]};
    // slots: 0 = d N_HB_raw, 3 = eta accepted
    __shared__ int part[2][kBlock / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int j = 0; j < 2; ++j) {
        const int s = wave_sum(v4[j]);
        if (lane == 0) part[j][wv] = s;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        int64_t s = 0;
        for (int i = 0; i < kBlock / 64; ++i) s += part[threadIdx.x][i];
        const int slot = threadIdx.x == 0 ? 0 : 3;
        if (s) atomicAdd((unsigned long long*)(a.slots + (size_t)slot * kSlots + blockIdx.x % kSlots),
                         (unsigned long long)s);
    }
}

// Two cubes per lane (L % 4 == 0): cubes 2i', 2i'+1 of one parity and one
// (j, l) span x = 4i' + par .. 4i' + par + 3, 24 row words of four bytes for
// their 24 edges (for the odd parity at byte addresses; the last lane of a row
// takes its fourth byte from the row's start).  The two cubes' edges are
// compared and gathered on packed words: bit e of the low (high) half of `old`,
// `unlike` and the new mask is edge e of the first (second) cube.  Rows of y and
// z edges belong to one parity and are stored as words, x edges alternate
// between the parities and are stored as bytes.  Each cube's move is the one of
// eta3_kernel.  Bound by the 9 bytes per cell it reads: 34 us at 260^3 (4.7
// TB/s of the bytes read once); cube by cube on single bytes, all even cubes
// before all odd ones, it took 58 us, on packed words in that order 47.5 us.
__device__ __forceinline__ uint32_t load4(const uint8_t* p)
{
    uint32_t v;
    __builtin_memcpy(&v, p, 4);                            // one dword load at any byte address
    return v;
}

// Bits 0 and 1 of edge pairs (x, x + 1), rows k = 0, 1, as bits x + 2k of each half.
__device__ __forceinline__ uint32_t gather4(uint32_t t) { return (t | (t >> 7)) & 0x000F000Fu; }

// Order of the workgroups.  The rows that a cube of one parity reads are, two
// and two, those of cubes of the other parity, and each row is read again for
// the next j or l: workgroups are dealt to the eight XCDs in turn, so workgroup
// b takes part in run b % 8 of `per` blocks (of each parity) and walks it in
// chunks of `chunk` blocks -- about one l -- first the even, then the odd cubes
// of a chunk, while the planes they share are still in that XCD's L2.
struct EtaShape {
    uint32_t per, chunk, blocks;   // blocks per run, per chunk, of one parity in all
};

__global__ __launch_bounds__(kBlock) void eta3_pair_kernel(Lat3 a, EtaShape sh)
{
    const uint32_t run = blockIdx.x % 8, s0 = blockIdx.x / 8;
    const uint32_t ch = s0 / (2 * sh.chunk), in = s0 - 2 * sh.chunk * ch, par = in >= sh.chunk ? 1u : 0u;
    const uint32_t local = sh.chunk * ch + in - par * sh.chunk, blk = run * sh.per + local;
    if (local >= sh.per || blk >= sh.blocks) return;
    // matchings, then the thresholds of dn = -4..4 from word 13 on: dn is in
    // -12..12 whatever a kept eta holds, which stays inside
    __shared__ uint32_t match[32];
    uint32_t* const thr = match + 17;
    if (threadIdx.x < 9) {
        match[threadIdx.x] = a.tab->match[threadIdx.x];
        match[13 + threadIdx.x] = a.tab->eta[threadIdx.x];
    }
    __syncthreads();
    const uint32_t r = blk * kBlock + threadIdx.x;
    int cnt[2] = {0, 0};
    if (r < a.N / 16) {
        const uint32_t L = a.L, N = a.N, h = a.h;
        const uint32_t q4 = L / 4;
        const uint32_t jl = udiv(r, q4, a.invQ4);
        const uint32_t ip = r - jl * q4;
        const uint32_t l = udiv(jl, h, a.invH);
        const uint32_t j = jl - l * h;
        const uint32_t y0 = 2 * j + par, y1 = y0 + 1 == L ? 0u : y0 + 1;
        const uint32_t z0 = 2 * l + par, z1 = z0 + 1 == L ? 0u : z0 + 1;
        const bool wrap = par && 4 * ip + 4 == L;          // the span's last byte is the row's first
        const uint32_t x = 4 * ip + (wrap ? 0u : par);
        const uint32_t row[4] = {L * (y0 + L * z0), L * (y1 + L * z0), L * (y0 + L * z1), L * (y1 + L * z1)};  // dy + 2 dz
        const uint8_t* E[3];
        const uint8_t* S[6];
#pragma unroll
        for (int k = 0; k < 3; ++k) E[k] = a.eta + (size_t)k * N;
#pragma unroll
        for (int k = 0; k < 6; ++k) S[k] = a.sigma + (size_t)k * N;
        // word k of w: its plane and row (dy + 2 dz)
        const uint8_t* const plane[24] = {E[0], E[0], E[0], E[0], S[0], S[0], S[0], S[0], S[1], S[1], S[1], S[1],
                                          E[1], E[1], S[2], S[2], S[3], S[3], E[2], E[2], S[4], S[4], S[5], S[5]};
        constexpr int at[24] = {0, 1, 2, 3, 0, 1, 2, 3, 0, 1, 2, 3,
                                0, 2, 0, 2, 1, 3, 0, 1, 0, 1, 2, 3};
        uint32_t w[24];
#pragma unroll
        for (int k = 0; k < 24; ++k) w[k] = load4(plane[k] + (row[at[k]] + x));   // scalar base, 32-bit lane offset
        if (wrap) {
            uint32_t b[24];
#pragma unroll
            for (int k = 0; k < 24; ++k) b[k] = plane[k][row[at[k]]];
#pragma unroll
            for (int k = 0; k < 24; ++k) w[k] = (w[k] >> 8) | (b[k] << 24);
        }
        const uint32_t t = (uint32_t)a.st->t_cur;
        const int theta = a.st->theta;
        // values are below 8: bit 3 of (u ^ v) + 7 is set where two bytes differ
        auto diff = [](uint32_t u, uint32_t v, uint32_t m) { return ((u ^ v) + 0x07070707u) & m; };
        const uint32_t xm = 0x00080008u, ym = 0x08080808u;
        const uint32_t ux = (diff(w[4], w[8] >> 8, xm) >> 3) | (diff(w[5], w[9] >> 8, xm) >> 2) |
                            (diff(w[6], w[10] >> 8, xm) >> 1) | diff(w[7], w[11] >> 8, xm);
        const uint32_t uy = gather4((diff(w[14], w[16], ym) >> 3) | (diff(w[15], w[17], ym) >> 1));
        const uint32_t uz = gather4((diff(w[20], w[22], ym) >> 3) | (diff(w[21], w[23], ym) >> 1));
        const uint32_t unlike = ux | (uy << 4) | (uz << 8);
        const uint32_t em = 0x00010001u;
        const uint32_t ox = (w[0] & em) | ((w[1] & em) << 1) | ((w[2] & em) << 2) | ((w[3] & em) << 3);
        const uint32_t old = ox | (gather4(w[12] | (w[13] << 2)) << 4) | (gather4(w[18] | (w[19] << 2)) << 8);
        uint32_t neu = old;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const uint32_t k = par * (h * h * h) + 2 * ip + (uint32_t)c + h * jl;
            const uint4 rnd = philox(k, t, 0u, kEta, a.key0, a.key1);
            const int m = pick_div(rnd.x, 9);
            const uint32_t half = 0xFFFu << (16 * c);
            const uint32_t to = (~match[m < 0 ? 0 : m] << (16 * c)) & half, eq = ~unlike & half;
            const int dn = __popc(to & eq) - __popc(old & eq);
            const uint32_t lim = theta ? thr[dn] : 0xFFFFFFFFu;
            const bool acc = m >= 0 && (lim == 0xFFFFFFFFu || rnd.y < lim);
            neu = acc ? (neu & ~half) | to : neu;
            cnt[0] += acc && a.eta_hb ? dn : 0;
            cnt[1] += acc ? 1 : 0;
        }
        const uint32_t chg = neu ^ old;
        if (chg) {
            uint8_t* const e0 = a.eta;
#pragma unroll
            for (int k = 0; k < 4; ++k) {                  // x edges: bytes 0 and 2 of the span
                const uint32_t base = row[k] + 4 * ip + par;
                if ((chg >> k) & 1u) e0[base] = (uint8_t)((neu >> k) & 1u);
                if ((chg >> (16 + k)) & 1u) e0[base + 2] = (uint8_t)((neu >> (16 + k)) & 1u);
            }
#pragma unroll
            for (int d = 1; d < 3; ++d)
#pragma unroll
                for (int k = 0; k < 2; ++k) {              // bits 4 d + 2 k, + 1 of each half: bytes x, x + 1
                    if (!((chg >> (4 * d + 2 * k)) & 0x00030003u)) continue;
                    const uint32_t n = neu >> (4 * d + 2 * k);
                    const uint32_t v = (n & em) | ((n & 0x00020002u) << 7);
                    uint8_t* const p = a.eta + (size_t)d * N;
                    const uint32_t o = d == 1 ? row[2 * k] : row[k];
                    if (!wrap) {
                        __builtin_memcpy(p + (o + x), &v, 4);
                    } else {
                        p[o + x + 1] = (uint8_t)v;
                        p[o + x + 2] = (uint8_t)(v >> 8);
                        p[o + x + 3] = (uint8_t)(v >> 16);
                        p[o] = (uint8_t)(v >> 24);
                    }
                }
        }
    }
    __shared__ int part[2][kBlock / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int sm = wave_sum(cnt[q]);
        if (lane == 0) part[q][wv] = sm;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        int64_t sm = 0;
        for (int i = 0; i < kBlock / 64; ++i) sm += part[threadIdx.x][i];
        const int slot = threadIdx.x == 0 ? 0 : 3;
        if (sm) atomicAdd((unsigned long long*)(a.slots + (size_t)slot * kSlots + blockIdx.x % kSlots),
                          (unsigned long long)sm);
    }
}

#include "pass3.h"
#include "sw3_step.h"

// ---------------------------------------------------------------------------
// Full recount of the configuration (observables): N_HB_raw (eta = 1 edges
// with equal facing sigma), N_sigma (15 pairs per cell), N_q', eta = 0 edges.
// ---------------------------------------------------------------------------
// Exact for any byte values.  At most kRcBlocks workgroups add their sums to
// kRcSpread addresses per counter (with a workgroup per 256 cells and 256
// addresses the recount took 176 us at 260^3, 32 us of which read the lattice).
template <bool W>
__global__ __launch_bounds__(kBlock) void recount3_kernel(Lat3 a, PassShape sh)
{
    int v[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    const uint32_t L = a.L, N = a.N, L2 = L * L;
    for (uint32_t u = blockIdx.x * kBlock + threadIdx.x; u < sh.quads; u += gridDim.x * kBlock) {
        const uint32_t yz = udiv(u, sh.per_row, sh.inv_row), z = udiv(yz, L, a.invL), y = yz - z * L;
        const uint32_t x = 4 * (u - yz * sh.per_row), c = x + L * yz, n = W || x + 4 <= L ? 4u : 2u;
        const uint32_t have = n == 4 ? 0x01010101u : 0x0101u;
        uint32_t s[6], f[3];
#pragma unroll
        for (int b = 0; b < 6; ++b) s[b] = bld4<W>(plane_rsrc(a.sigma + (size_t)b * N, N), c, n);
        const uint32_t nx = bld8(plane_rsrc(a.sigma + (size_t)N, N), x + n == L ? c + n - L : c + n);
        f[0] = n == 4 ? (s[1] >> 8) | (nx << 24) : ((s[1] >> 8) & 0xFFu) | (nx << 8);
        f[1] = bld4<W>(plane_rsrc(a.sigma + 3 * (size_t)N, N), y == L - 1 ? c + L - L2 : c + L, n);
        f[2] = bld4<W>(plane_rsrc(a.sigma + 5 * (size_t)N, N), z == L - 1 ? c + L2 - N : c + L2, n);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const uint32_t off = zero_bytes(bld4<W>(plane_rsrc(a.eta + (size_t)d * N, N), c, n));
            v[0] += __popc(zero_bytes(s[2 * d] ^ f[d]) & ~off & have);
            v[8] += __popc(off & have);
        }
#pragma unroll
        for (int i = 0; i < 6; ++i) {
#pragma unroll
            for (int j = i + 1; j < 6; ++j) v[1] += __popc(zero_bytes(s[i] ^ s[j]) & have);
#pragma unroll
            for (uint32_t k = 0; k < 6; ++k) v[2 + k] += __popc(zero_bytes(s[i] ^ (k * 0x01010101u)) & have);
        }
    }
    __shared__ int part[9][kBlock / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const int sm = wave_sum(v[k]);
        if (lane == 0) part[k][w] = sm;
    }
    __syncthreads();
    if (threadIdx.x < 9) {
        int64_t sm = 0;
        for (int i = 0; i < kBlock / 64; ++i) sm += part[threadIdx.x][i];
        if (sm) atomicAdd((unsigned long long*)(a.rc + threadIdx.x * kRcSpread + blockIdx.x % kRcSpread),
                          (unsigned long long)sm);
    }
}

// N_q' of the current sigma added to out[0..5]: the 6N bytes read as 32-bit
// words; the bytes of w equal to k are the zero bytes of w ^ k 0x01010101,
// counted exactly (no carry crosses a byte) with one popcount.
__global__ __launch_bounds__(kBlock) void counts3_kernel(const uint32_t* __restrict__ words, uint32_t nwords,
                                                         int64_t* out)
{
    int c[6] = {0, 0, 0, 0, 0, 0};
    for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < nwords; i += gridDim.x * kBlock) {
        const uint32_t w = words[i];
#pragma unroll
        for (uint32_t k = 0; k < 6; ++k) c[k] += __popc(zero_bytes(w ^ (k * 0x01010101u)));
    }
    __shared__ int part[6][kBlock / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const int sm = wave_sum(c[k]);
        if (lane == 0) part[k][wv] = sm;
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        int64_t sm = 0;
        for (int i = 0; i < kBlock / 64; ++i) sm += part[threadIdx.x][i];
        if (sm) atomicAdd((unsigned long long*)(out + threadIdx.x), (unsigned long long)sm);
    }
}

inline unsigned blocks_for(uint64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace

// ===========================================================================
// Host side: the cvf3_* C ABI.
// ===========================================================================
struct cvf3_state {
    cvf_params p;
    Lat3       la;
    Tab3       htab;
    Tab3*      dtab;
    uint8_t*   sigma;
    uint8_t*   eta;
    bool       timing;
    bool       sw;
    bool       sw_done;
    bool       le;            // no Metropolis threshold is 0: acceptance is word <= threshold - 1
    std::vector<hipEvent_t> ev[CVF3_K_COUNT];
    int64_t    launches[CVF3_K_COUNT];
    double     total_ms[CVF3_K_COUNT];
};

namespace {

constexpr size_t al256(size_t n) { return (n + 255) & ~(size_t)255; }

// Tiles of a cluster update: 8 x 8 x 4 cells, one per thread, where the chip
// has wavefronts to spare and the latency of a workgroup decides (a step takes
// 44 / 56 / 76 / 97 us at L = 40 / 64 / 80 / 96 and 205 K); 16 x 8 x 8 cells,
// four per thread, from L = 80 (54 / 61 / 76 / 91 us), with fewer face indices
// and wider loads.
using Sw3Big = Tile3<16, 8, 8, 4>;
using Sw3Small = Tile3<8, 8, 4, 1>;
constexpr bool sw3_big(uint64_t L) { return L >= 80; }

// Plus nodes of the tiling (as many minus nodes): a face layer of L^2 per tile
// along each axis.
template <class TL>
constexpr size_t tile_nodes(uint64_t L)
{
    return (size_t)(((L + TL::TX - 1) / TL::TX + (L + TL::TY - 1) / TL::TY + (L + TL::TZ - 1) / TL::TZ) * L * L);
}
constexpr size_t sw3_nodes(uint64_t L) { return sw3_big(L) ? tile_nodes<Sw3Big>(L) : tile_nodes<Sw3Small>(L); }

// What a cluster update keeps for F plus nodes and N cells: parents and keys of
// the nodes, a local root per bond index, a byte per plus node.  A workspace
// has 28 N bytes for it (see cvf3_workspace_bytes): the tiles above have few
// enough faces for that at every L, most nearly at L = 4 with 1584 of 1792 bytes.
constexpr size_t sw3_need(uint64_t L)
{
    return sw3_nodes(L) * (4 * sizeof(uint32_t) + 1) + 6 * L * L * L * sizeof(uint16_t);
}
constexpr size_t sw3_room(uint64_t L)
{
    return al256(L * L * L * sizeof(uint32_t)) + al256(6 * L * L * L * sizeof(uint32_t));
}
constexpr uint64_t kSw3MaxL = 894;                         // 6 N < 2^32
constexpr bool sw3_fits()
{
    for (uint64_t L = 2; L <= kSw3MaxL; L += 2)
        if (sw3_need(L) > sw3_room(L)) return false;
    return true;
}
static_assert(sw3_fits(), "the cluster update's arrays exceed the workspace");

size_t ws3_bytes(const cvf_params* p, int algo_mask)
{
    size_t b = al256(sizeof(Dev3State)) + al256(sizeof(int64_t) * kAcc * kSlots) +
               al256(sizeof(int64_t) * kRc * kSlots) + al256(sizeof(Tab3));
    if (algo_mask & CVF_ALGO_SW) b += sw3_room((uint64_t)p->L);
    return b;
}

// r3(m): integer points on the sphere i^2 + j^2 + k^2 = m, counted as
// octant points with signs (each nonzero coordinate doubles the count).
double sphere_points(int m)
{
    int n = 0;
    for (int i = 0; i * i <= m; ++i)
        for (int j = 0; i * i + j * j <= m; ++j)
            for (int k = 0; i * i + j * j + k * k <= m; ++k)
                if (i * i + j * j + k * k == m) n += (i ? 2 : 1) * (j ? 2 : 1) * (k ? 2 : 1);
    return (double)n;
}

uint32_t thr_of(double beta, double dH)
{
    if (!(dH > 0.0)) return 0xFFFFFFFFu;
    const double acc = exp(-beta * dH);
    if (acc >= 1.0) return 0xFFFFFFFFu;
    const double f = floor(acc * 4294967296.0);
    return f > 4294967294.0 ? 0xFFFFFFFEu : (uint32_t)f;
}

// Perfect matchings of the cube graph, built from its structure: the three
// one-axis matchings (four parallel edges), and for each axis d the two
// faces perpendicular to d each taking one of their two non-d matchings
// where the two faces differ (2 x 3 = 6), sorted by edge mask.
void cube_matchings(uint32_t out[9])
{
    // edge index of the edge along axis d whose other coordinates are (o1, o2)
    auto edge = [](int d, int o_lo, int o_hi) { return 4 * d + o_lo + 2 * o_hi; };
    std::vector<uint32_t> ms;
    for (int d = 0; d < 3; ++d) ms.push_back(0xFu << (4 * d));
    for (int d = 0; d < 3; ++d) {
        const int a1 = d == 0 ? 1 : 0, a2 = d == 2 ? 1 : 2;   // the two other axes, a1 < a2
        // face at coordinate s along d: a 4-cycle, matched along a1 or a2
        for (int f0 = 0; f0 < 2; ++f0) {
            const int f1 = 1 - f0;
            uint32_t m = 0;
            for (int s = 0; s < 2; ++s) {
                const int along = (s == 0 ? f0 : f1) ? a2 : a1;   // axis of this face's two edges
                // the edge along `along` has its d coordinate = s and the remaining axis r in {0,1}
                const int r = 3 - d - along;
                for (int rv = 0; rv < 2; ++rv) {
                    int coord[3] = {0, 0, 0};
                    coord[d] = s;
                    coord[r] = rv;
                    int o[2], n = 0;
                    for (int ax = 0; ax < 3; ++ax)
                        if (ax != along) o[n++] = coord[ax];
                    m |= 1u << edge(along, o[0], o[1]);
                }
            }
            ms.push_back(m);
        }
    }
    for (size_t i = 0; i < ms.size(); ++i)
        for (size_t j = i + 1; j < ms.size(); ++j)
            if (ms[j] < ms[i]) std::swap(ms[i], ms[j]);
    for (int i = 0; i < 9; ++i) out[i] = ms[i];
}

void build_tab3(const cvf_params* p, Tab3* t)
{
    memset(t, 0, sizeof(*t));
    const double Jeff = p->J - p->P * p->vHB;
    for (int th = 0; th < 2; ++th)
        for (int dh = -1; dh <= 1; ++dh)
            for (int dc = -5; dc <= 5; ++dc)
                t->met[th][dh + 1][dc + 5] = thr_of(p->beta, -((double)th * Jeff * (double)dh) - p->Jsigma * (double)dc);
    for (int dn = -4; dn <= 4; ++dn) t->eta[dn + 4] = thr_of(p->beta, -(Jeff * (double)dn));
    cube_matchings(t->match);
    const double xs = p->beta * p->Jsigma, xe = p->beta * fabs(Jeff);
    t->sw_sigma = xs > 0.0 ? (uint64_t)floor(-expm1(-xs) * 4294967296.0) : 0;
    t->sw_eff = xe > 0.0 ? (uint64_t)floor(-expm1(-xe) * 4294967296.0) : 0;
    t->jeff_sign = Jeff > 0.0 ? 1 : (Jeff < 0.0 ? -1 : 0);
    for (int m = 0; m < 40; ++m) t->r3[m] = m <= 36 ? sphere_points(m) : 0.0;
}

int hs(hipError_t e) { return e == hipSuccess ? CVF_OK : CVF_EHIP; }

int validate3(const cvf_params* p)
{
    if (!p) return CVF_EINVAL;
    if (p->L < 2 || p->L > CVF3_MAX_L || (p->L & 1)) return CVF_EINVAL;
    if (p->q < 2 || p->q > 6) return CVF_EINVAL;
    if (!(p->beta >= 0.0) || !std::isfinite(p->beta)) return CVF_EINVAL;
    if (!std::isfinite(p->J) || !std::isfinite(p->Jsigma) || !std::isfinite(p->P) || !std::isfinite(p->vHB))
        return CVF_EINVAL;
    if (!(p->v_init >= 1.0) || !std::isfinite(p->v_init)) return CVF_EINVAL;
    if (!(p->dv_max >= 0.0) || !std::isfinite(p->dv_max)) return CVF_EINVAL;
    if (p->flags & ~(uint32_t)(CVF_NO_VOLUME_MOVE | CVF_KEEP_SIGMA)) return CVF_EINVAL;
    if (p->reserved != 0) return CVF_EINVAL;
    return CVF_OK;
}

using cvf::DispatchEvents;
using cvf::go;

// With timing on: start/stop events that the next launch of this kind
// records on its own dispatch.
DispatchEvents t_events(cvf3_state* st, int kind)
{
    DispatchEvents ev;
    if (!st->timing) return ev;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return ev;
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return ev;
    }
    st->ev[kind].push_back(e0);
    st->ev[kind].push_back(e1);
    ev.start = e0;
    ev.stop = e1;
    return ev;
}

int drain3(cvf3_state* st)
{
    int rc = CVF_OK;
    for (int k = 0; k < CVF3_K_COUNT; ++k) {
        std::vector<hipEvent_t>& v = st->ev[k];
        for (size_t i = 0; i + 1 < v.size(); i += 2) {
            float ms = 0.f;
            if (hipEventSynchronize(v[i + 1]) != hipSuccess || hipEventElapsedTime(&ms, v[i], v[i + 1]) != hipSuccess)
                rc = CVF_EHIP;
            st->launches[k] += 1;
            st->total_ms[k] += ms;
        }
        for (hipEvent_t e : v) (void)hipEventDestroy(e);
        v.clear();
    }
    return rc;
}

template <class TL>
unsigned sw3_tiles(uint32_t L)
{
    return ((L + TL::TX - 1) / TL::TX) * ((L + TL::TY - 1) / TL::TY) * ((L + TL::TZ - 1) / TL::TZ);
}

template <class TL>
TileGrid3 sw3_grid(uint32_t L)
{
    const uint32_t nx = (L + TL::TX - 1) / TL::TX, ny = (L + TL::TY - 1) / TL::TY;
    return {nx, ny, 1.0f / (float)nx, 1.0f / (float)ny};
}

// The three launches of a cluster update over tiles TL.
template <class TL>
hipError_t sw3_update(cvf3_state* st, const Lat3& a, hipStream_t s)
{
    const TileGrid3 tg = sw3_grid<TL>(a.L);
    const dim3 tiles(sw3_tiles<TL>(a.L));
    hipError_t e = go(sw3_tile_kernel<TL>, tiles, dim3(TL::TT), s, t_events(st, CVF3_K_SW_BONDS), a, tg);
    if (e == hipSuccess)
        e = go(sw3_union_kernel, dim3(blocks_for(tile_nodes<TL>(a.L))), dim3(kBlock), s,
               t_events(st, CVF3_K_SW_UNION), a, tg.nx, tg.ny, (a.L + TL::TZ - 1) / TL::TZ);
    if (e == hipSuccess) e = go(sw3_flip_kernel<TL>, tiles, dim3(TL::TT), s, t_events(st, CVF3_K_SW_FLIP), a, tg);
    return e;
}

PassShape quad_shape(const Lat3& a)
{
    PassShape sh = {};
    sh.per_row = (a.L + 3) / 4;
    sh.quads = sh.per_row * a.L * a.L;
    sh.inv_row = 1.0 / (double)sh.per_row;
    return sh;
}

// The recount's sums and the folded chain state, as the host reads them.
struct Recount3 {
    int64_t sums[kRc][kRcSpread];
    Dev3State st;
    int64_t total(int k) const
    {
        int64_t t = 0;
        for (int i = 0; i < kRcSpread; ++i) t += sums[k][i];
        return t;
    }
};
static_assert(offsetof(Recount3, st) == kRcState * sizeof(int64_t), "one copy brings both");
static_assert(sizeof(Recount3) <= kRc * kSlots * sizeof(int64_t), "fits the recount area");

// Folds the counters, recounts the lattice and reads both (synchronises).
int recount3(const Lat3& a, hipStream_t s, Recount3* out)
{
    vol3_kernel<<<1, 64, 0, s>>>(a, kVolFold);
    const PassShape sh = quad_shape(a);
    const unsigned grid = std::min((unsigned)kRcBlocks, blocks_for(sh.quads));
    if (a.quad) recount3_kernel<true><<<grid, kBlock, 0, s>>>(a, sh);
    else recount3_kernel<false><<<grid, kBlock, 0, s>>>(a, sh);
    int rc = hs(hipGetLastError());
    if (rc == CVF_OK) rc = hs(hipMemcpyAsync(out, a.rc, sizeof(Recount3), hipMemcpyDeviceToHost, s));
    if (rc == CVF_OK) rc = hs(hipStreamSynchronize(s));
    return rc;
}

template <int Q, bool LE>
hipError_t pass_launch_q(cvf3_state* st, const Lat3& a, unsigned grid, const PassShape& sh, hipStream_t s)
{
    const DispatchEvents ev = t_events(st, CVF3_K_PASS);
    if (a.quad) return go(pass3_kernel<Q, LE, true>, dim3(grid), dim3(kBlock), s, ev, a, sh);
    return go(pass3_kernel<Q, LE, false>, dim3(grid), dim3(kBlock), s, ev, a, sh);
}

template <int Q>
hipError_t pass_launch_le(cvf3_state* st, const Lat3& a, unsigned grid, const PassShape& sh, hipStream_t s)
{
    return st->le ? pass_launch_q<Q, true>(st, a, grid, sh, s) : pass_launch_q<Q, false>(st, a, grid, sh, s);
}

// Pass group a.pass.  Up to four quads per lane spread a lane's fixed work
// (table load, counter reduction) over more moves; smaller lattices take fewer,
// so that the launch keeps the 2048 workgroups that fill the chip (at L = 130
// a step takes 64 us this way, 76 us with at least 256 workgroups).
hipError_t pass_launch(cvf3_state* st, const Lat3& a, hipStream_t s)
{
    PassShape sh = quad_shape(a);
    const uint32_t one = blocks_for(sh.quads);
    const uint32_t per_lane = std::min(kMaxQuadsPerLane, std::max(1u, one / 2048u));
    const uint32_t grid = (one + per_lane - 1) / per_lane, step = grid * kBlock;
    const uint32_t rows = step / sh.per_row;
    sh.sj = step % sh.per_row;
    sh.sy = rows % a.L;
    sh.sz = rows / a.L;
    switch (a.q) {
    case 2: return pass_launch_le<2>(st, a, grid, sh, s);
    case 3: return pass_launch_le<3>(st, a, grid, sh, s);
    case 4: return pass_launch_le<4>(st, a, grid, sh, s);
    case 5: return pass_launch_le<5>(st, a, grid, sh, s);
    default: return pass_launch_le<6>(st, a, grid, sh, s);
    }
}

}  // namespace

extern "C" {

int validate_algo3(const cvf_params* p, int algo_mask)
{
    if (algo_mask & ~(CVF_ALGO_METROPOLIS | CVF_ALGO_SW)) return CVF_EINVAL;
    if ((algo_mask & CVF_ALGO_SW) && (uint64_t)p->L > kSw3MaxL) return CVF_EINVAL;
    return CVF_OK;
}

int cvf3_workspace_bytes(const cvf_params* p, int algo_mask, size_t* bytes)
{
    if (!bytes) return CVF_EINVAL;
    int rc = validate3(p);
    if (rc == CVF_OK) rc = validate_algo3(p, algo_mask);
    if (rc != CVF_OK) return rc;
    *bytes = ws3_bytes(p, algo_mask);
    return CVF_OK;
}

int cvf3_tables(const cvf_params* p, uint32_t met[2][3][11], uint32_t eta[9], uint32_t match[9])
{
    if (!met || !eta || !match) return CVF_EINVAL;
    const int rc = validate3(p);
    if (rc != CVF_OK) return rc;
    Tab3 t;
    build_tab3(p, &t);
    memcpy(met, t.met, sizeof(t.met));
    memcpy(eta, t.eta, sizeof(t.eta));
    memcpy(match, t.match, sizeof(t.match));
    return CVF_OK;
}

int cvf3_init(const cvf_params* p, int algo_mask, uint8_t* d_sigma, uint8_t* d_eta, void* d_work, size_t work_bytes,
              void* stream, cvf3_state** out)
{
    if (!out) return CVF_EINVAL;
    *out = nullptr;
    int rc = validate3(p);
    if (rc == CVF_OK) rc = validate_algo3(p, algo_mask);
    if (rc != CVF_OK) return rc;
    if (!d_sigma || !d_eta || !d_work) return CVF_EINVAL;
    if (((uintptr_t)d_sigma & 3) || ((uintptr_t)d_eta & 3) || ((uintptr_t)d_work & 255)) return CVF_EINVAL;
    if (work_bytes < ws3_bytes(p, algo_mask)) return CVF_ENOMEM;
    cvf3_state* st = new (std::nothrow) cvf3_state();
    if (!st) return CVF_ENOMEM;
    st->p = *p;
    st->sigma = d_sigma;
    st->eta = d_eta;
    build_tab3(p, &st->htab);
    uint8_t* w = (uint8_t*)d_work;
    Lat3& a = st->la;
    a.sigma = d_sigma;
    a.eta = d_eta;
    a.st = (Dev3State*)w;
    w += al256(sizeof(Dev3State));
    a.slots = (int64_t*)w;
    w += al256(sizeof(int64_t) * kAcc * kSlots);
    a.rc = (int64_t*)w;
    w += al256(sizeof(int64_t) * kRc * kSlots);
    st->dtab = (Tab3*)w;
    a.tab = st->dtab;
    w += al256(sizeof(Tab3));
    st->sw = (algo_mask & CVF_ALGO_SW) != 0;
    a.par = nullptr;
    a.key = nullptr;
    a.lroot = nullptr;
    a.edge = nullptr;
    if (st->sw) {
        const size_t N = (size_t)p->L * p->L * p->L, F = sw3_nodes((uint64_t)p->L);
        a.par = (uint32_t*)w;
        a.key = a.par + 2 * F;
        a.lroot = (uint16_t*)(a.key + 2 * F);
        a.edge = (uint8_t*)(a.lroot + 6 * N);
    }
    a.L = (uint32_t)p->L;
    a.N = a.L * a.L * a.L;
    a.h = a.L / 2;
    a.q = (uint32_t)p->q;
    a.key0 = (uint32_t)p->seed;
    a.key1 = (uint32_t)(p->seed >> 32);
    a.invL = 1.0 / (double)a.L;
    a.invH = 1.0 / (double)a.h;
    a.invQ4 = 1.0 / (double)(a.L / 4 ? a.L / 4 : 1);
    a.Nd = (double)a.N;
    a.beta = p->beta;
    a.J = p->J;
    a.P = p->P;
    a.vHB = p->vHB;
    a.dv_max = p->dv_max;
    a.do_volume = (p->flags & CVF_NO_VOLUME_MOVE) ? 0 : 1;
    a.quad = (a.L % 4 == 0) ? 1u : 0u;
    a.eta_hb = 1;
    st->le = true;
    for (int k = 0; k < 66; ++k)
        if ((&st->htab.met[0][0][0])[k] == 0) st->le = false;
    hipStream_t s = (hipStream_t)stream;
    rc = hs(hipMemcpyAsync(st->dtab, &st->htab, sizeof(Tab3), hipMemcpyHostToDevice, s));
    if (rc == CVF_OK) {
        state3_init_kernel<<<1, kBlock, 0, s>>>(a, p->v_init);
        rc = hs(hipGetLastError());
    }
    if (rc == CVF_OK && !(p->flags & CVF_KEEP_SIGMA)) {
        init3_sigma_kernel<<<blocks_for(a.N), kBlock, 0, s>>>(a);
        init3_eta_kernel<<<blocks_for(a.N / 4), kBlock, 0, s>>>(a);
        rc = hs(hipGetLastError());
    }
    if (rc == CVF_OK) {                              // initial counters from a recount
        Recount3 r;
        rc = recount3(a, s, &r);
        if (rc == CVF_OK) {
            r.st.n_hb_raw = r.total(0);
            r.st.n_coop = r.total(1);
            rc = hs(hipMemcpy(a.st, &r.st, sizeof(r.st), hipMemcpyHostToDevice));
        }
    }
    if (rc != CVF_OK) {
        delete st;
        return rc;
    }
    *out = st;
    return CVF_OK;
}

namespace {

// The eta move of one step: two checkerboard cubes per lane when L % 4 == 0.
hipError_t eta_step(cvf3_state* st, const Lat3& a, hipStream_t s)
{
    const DispatchEvents ev = t_events(st, CVF3_K_ETA);
    if (a.quad) {
        EtaShape sh;
        sh.blocks = blocks_for(a.N / 16);
        sh.per = (sh.blocks + 7) / 8;
        sh.chunk = std::max(1u, std::min(sh.per, (a.h * (a.L / 4) + kBlock / 2) / kBlock));
        const uint32_t chunks = (sh.per + sh.chunk - 1) / sh.chunk;
        return go(eta3_pair_kernel, dim3(8 * chunks * 2 * sh.chunk), dim3(kBlock), s, ev, a, sh);
    }
    return go(eta3_kernel, dim3(blocks_for(a.N / 4)), dim3(kBlock), s, ev, a);
}

}  // namespace

int cvf3_steps(cvf3_state* st, int64_t nsteps, void* stream)
{
    if (!st || nsteps < 0) return CVF_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    Lat3 a = st->la;
    for (int64_t i = 0; i < nsteps; ++i) {
        if (go(vol3_kernel, dim3(1), dim3(64), s, t_events(st, CVF3_K_VOLUME), a, kVolMet) != hipSuccess)
            return CVF_EHIP;
        if (eta_step(st, a, s) != hipSuccess) return CVF_EHIP;
        for (a.pass = 0; a.pass < 4; ++a.pass)
            if (pass_launch(st, a, s) != hipSuccess) return CVF_EHIP;
    }
    return CVF_OK;
}

int cvf3_sw_steps(cvf3_state* st, int64_t nsteps, void* stream)
{
    if (!st || nsteps < 0) return CVF_EINVAL;
    if (!st->sw) return CVF_ESTATE;
    hipStream_t s = (hipStream_t)stream;
    Lat3 a = st->la;
    a.eta_hb = 0;                                          // the flip recounts N_HB_raw
    for (int64_t i = 0; i < nsteps; ++i) {
        if (go(vol3_kernel, dim3(1), dim3(64), s, t_events(st, CVF3_K_VOLUME), a, kVolSw) != hipSuccess)
            return CVF_EHIP;
        if (eta_step(st, a, s) != hipSuccess) return CVF_EHIP;
        const hipError_t e = sw3_big(a.L) ? sw3_update<Sw3Big>(st, a, s) : sw3_update<Sw3Small>(st, a, s);
        if (e != hipSuccess) return CVF_EHIP;
        st->sw_done = true;
    }
    return CVF_OK;
}

int cvf3_labels(cvf3_state* st, uint32_t* d_out, void* stream)
{
    if (!st || !d_out) return CVF_EINVAL;
    if (!st->sw || !st->sw_done) return CVF_ESTATE;
    hipStream_t s = (hipStream_t)stream;
    const Lat3& a = st->la;
    if (sw3_big(a.L)) sw3_labels_kernel<Sw3Big><<<sw3_tiles<Sw3Big>(a.L), Sw3Big::T, 0, s>>>(a, sw3_grid<Sw3Big>(a.L), d_out);
    else sw3_labels_kernel<Sw3Small><<<sw3_tiles<Sw3Small>(a.L), Sw3Small::T, 0, s>>>(a, sw3_grid<Sw3Small>(a.L), d_out);
    return hs(hipGetLastError());
}

int cvf3_state_counts(cvf3_state* st, int64_t* d_counts, void* stream)
{
    if (!st || !d_counts || ((uintptr_t)d_counts & 7)) return CVF_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const uint32_t nwords = (uint32_t)(6ull * st->la.N / 4);
    uint64_t blocks = (nwords + kBlock - 1) / kBlock;
    if (blocks > 4096) blocks = 4096;
    counts3_kernel<<<(unsigned)blocks, kBlock, 0, s>>>((const uint32_t*)st->sigma, nwords, d_counts);
    return hs(hipGetLastError());
}

int cvf3_observables(cvf3_state* st, cvf3_obs* out, void* stream)
{
    if (!st || !out) return CVF_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const Lat3& a = st->la;
    Recount3 r;
    const int rc = recount3(a, s, &r);
    if (rc != CVF_OK) return rc;
    const Dev3State& ds = r.st;
    int64_t tot[kRc];
    for (int k = 0; k < kRc; ++k) tot[k] = r.total(k);
    memset(out, 0, sizeof(*out));
    const double Nd = a.Nd;
    out->step = ds.t_next;
    out->n_hb_raw = tot[0];
    out->n_hb = ds.theta ? tot[0] : 0;
    out->n_coop = tot[1];
    int64_t mx = 0;
    for (int k = 0; k < 6; ++k) {
        out->count[k] = tot[2 + k];
        mx = tot[2 + k] > mx ? tot[2 + k] : mx;
    }
    out->n_eta0 = tot[8];
    out->met_attempted = ds.met_att;
    out->met_accepted = ds.met_acc;
    out->eta_attempted = ds.eta_att;
    out->eta_accepted = ds.eta_acc;
    out->vol_attempted = ds.vol_att;
    out->vol_accepted = ds.vol_acc;
    out->v = ds.v;
    out->V = (Nd * ds.v) + (st->p.vHB * (double)out->n_hb);
    out->H = (((Nd * lj3(ds.v, st->htab.r3)) - (st->p.J * (double)out->n_hb)) - (st->p.Jsigma * (double)out->n_coop)) +
             (st->p.P * out->V);
    out->M = (double)mx / (6.0 * Nd);
    out->consistent = (ds.n_hb_raw == tot[0] && ds.n_coop == tot[1]) ? 1 : 0;
    return CVF_OK;
}

int cvf3_timing_enable(cvf3_state* st, int enable)
{
    if (!st) return CVF_EINVAL;
    const int rc = drain3(st);
    for (int k = 0; k < CVF3_K_COUNT; ++k) {
        st->launches[k] = 0;
        st->total_ms[k] = 0.0;
    }
    st->timing = enable != 0;
    return rc;
}

int cvf3_kernel_times(cvf3_state* st, int kind, int64_t* launches, double* mean_ms)
{
    if (!st || kind < 0 || kind >= CVF3_K_COUNT || !launches || !mean_ms) return CVF_EINVAL;
    const int rc = drain3(st);
    *launches = st->launches[kind];
    *mean_ms = st->launches[kind] ? st->total_ms[kind] / (double)st->launches[kind] : 0.0;
    return rc;
}

int cvf3_destroy(cvf3_state* st)
{
    if (!st) return CVF_EINVAL;
    drain3(st);
    delete st;
    return CVF_OK;
}

}  // extern "C"
