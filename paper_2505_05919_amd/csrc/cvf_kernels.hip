// HIP kernels of libcvf for gfx950 (MI355X).
//
// The lattice kernels are integer-only: uint8 bond indices, uint32 Philox
// words and thresholds, int32 per-lane deltas reduced across the wavefront
// and the workgroup, int64 atomics into spread slots.  The single-wave
// volume kernel is the only floating-point code (FP64, no contraction).
#include "cvf_internal.h"
#include "met_launch.h"

#include <atomic>
#include <type_traits>

namespace cvf {

// Fixed device workspace of the allocation-free entry point
// (cvf_sw_steps_noalloc): every GPU the library runs on holds one copy,
// from module load until the process ends.  Host code never passes this
// name to a kernel or a copy (on the host it is only a stand-in for the
// symbol); it uses the device address from noalloc_scratch().
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

namespace {

constexpr int kBlock = 256;           // 4 wavefronts of 64
constexpr int kMaxBlocks = 8192;      // 256 CUs x 8 waves/SIMD x 4 SIMDs / 4 waves

#include "philox.h"
#include "wave.h"

// floor(j / d) and j mod d for j < 2^32, d < 2^15: one FP64 multiply by the
// reciprocal is at most one too small, never too large; one correction.
__device__ __forceinline__ uint32_t divmod(uint32_t j, uint32_t d, double inv, uint32_t& rem)
{
    uint32_t qt = (uint32_t)((double)j * inv);
    uint32_t r = j - qt * d;
    if (r >= d) {
        ++qt;
        r -= d;
    }
    rem = r;
    return qt;
}


__device__ __forceinline__ int64_t wave_sum64(int64_t v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Sum NV int32 values over the workgroup and add them (as int64) to
// dst[i * stride] (one atomic per value per workgroup).
template <int NV, int BLOCK = kBlock>
__device__ __forceinline__ void block_add(const int (&v)[NV], int64_t* dst, int stride)
{
    __shared__ int part[NV][BLOCK / 64];
    const int tid = threadIdx.x + threadIdx.y * blockDim.x;
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int s = wave_sum(v[i]);
        if (lane == 0) part[i][wave] = s;
    }
    __syncthreads();
    if (tid < NV) {
        int64_t s = 0;
#pragma unroll
        for (int w = 0; w < BLOCK / 64; ++w) s += part[tid][w];
        if (s) atomicAdd((unsigned long long*)(dst + (size_t)tid * stride), (unsigned long long)s);
    }
}

inline unsigned grid_for(uint64_t work)
{
    uint64_t b = (work + kBlock - 1) / kBlock;
    if (b < 1) b = 1;
    if (b > kMaxBlocks) b = kMaxBlocks;
    return (unsigned)b;
}

// ---------------------------------------------------------------------------
// Lennard-Jones lattice energy per molecule (Sec. II.A): hard core r0,
// cutoff 6 r0, square lattice of spacing sqrt(v) r0.  Same operation order as
// the definition: ascending shells m = |n|^2, s = (v m)^-3, 2 sum r2 (s^2-s).
// ---------------------------------------------------------------------------
__device__ double lj_energy(double v, const double* r2)
{
    double s = 0.0;
    for (int m = 1; v * (double)m <= 36.0; ++m) {
        const double d2 = v * (double)m;
        const double s6 = 1.0 / (d2 * d2 * d2);
        s = s + r2[m] * (s6 * s6 - s6);
    }
    return 2.0 * s;
}

// ---------------------------------------------------------------------------
// State initialisation.
// ---------------------------------------------------------------------------
__global__ void state_init_kernel(DevState* st, int64_t* slots, const DevTables* tab, double v_init)
{
    const int i = threadIdx.x;
    for (int k = i; k < 2 * kBankSlots; k += blockDim.x) slots[k] = 0;
    if (i == 0) {
        st->t_next = 0;
        st->n_hb_raw = 0;
        st->n_coop = 0;
        st->met_att = st->met_acc = st->vol_att = st->vol_acc = 0;
        st->v = v_init;
        st->u = lj_energy(v_init, tab->r2);
        st->theta = v_init < 2.0 ? 1 : 0;
        st->sw_done = 0;
        st->stop_at = INT64_MAX;
    }
}

// sigma[a][c] = floor(w_a q / 2^32), (w0..w3) = Philox(c, 0, 0, INIT).
__global__ __launch_bounds__(kBlock) void sigma_init_kernel(LatticeArgs a)
{
    for (uint32_t c = blockIdx.x * kBlock + threadIdx.x; c < a.N; c += gridDim.x * kBlock) {
        const uint4 w = philox(c, 0u, 0u, kStreamInit, a.key0, a.key1);
        a.sigma[c] = (uint8_t)(((uint64_t)w.x * a.q) >> 32);
        a.sigma[(size_t)a.N + c] = (uint8_t)(((uint64_t)w.y * a.q) >> 32);
        a.sigma[2 * (size_t)a.N + c] = (uint8_t)(((uint64_t)w.z * a.q) >> 32);
        a.sigma[3 * (size_t)a.N + c] = (uint8_t)(((uint64_t)w.w * a.q) >> 32);
    }
}

// ---------------------------------------------------------------------------
// Volume move: one wavefront opens a step -- the Metropolis move of v_iso
// (Sec. II.B step 1) with the full dH of Eq. (1) and (3),
//   N (u(v') - u(v)) + P N (v' - v) + (theta(v') - theta(v)) (P v_HB - J) N_HB_raw.
// While theta stays what it is, N_HB_raw drops out and the move needs nothing
// of the sigma update before it.  So only the first step of a call is opened
// by a launch of its own (volume_step, which also folds the counter slots);
// every later one is opened by a workgroup of the last launch of the step
// before it (open_next), beside the sigma update: the launch it saves is
// 4.8 us of a step.  A move that would cross v = 2 is left pending, and the
// step's first launch decides it (resolve_step) from N_HB_raw, which by then
// is complete: every workgroup for itself, the first one writing the result.
// ---------------------------------------------------------------------------
struct VolState {
    int64_t t_next, stop_at, met_att, vol_att, vol_acc;
    double v, u, r2;
    int theta;
};

__device__ __forceinline__ VolState vol_load(const VolArgs& a, int lane)
{
    const DevState* st = a.st;
    VolState s;
    s.t_next = st->t_next;
    s.stop_at = st->stop_at;
    s.met_att = st->met_att;
    s.vol_att = st->vol_att;
    s.vol_acc = st->vol_acc;
    s.v = st->v;
    s.u = st->u;
    s.theta = st->theta;
    s.r2 = lane < 40 ? a.tab->r2[lane] : 0.0;
    return s;
}

// dH of the move and the acceptance through the word w; the same operations
// in the same order wherever a move is decided.
__device__ __forceinline__ bool vol_accept(const VolArgs& a, double v0, double u0, int th0, double v1, double u1, int th1,
                                           int64_t n_hb, uint32_t w)
{
    const double dH = (a.Nd * (u1 - u0)) + ((a.P * a.Nd) * (v1 - v0)) +
                      (((double)(th1 - th0) * (a.P * a.vHB - a.J)) * (double)n_hb);
    return dH <= 0.0 || ((double)w + 0.5) * (1.0 / 4294967296.0) < exp(-a.beta * dH);
}

// Opens the step s.t_next into view, by one wavefront; `term` is 40 doubles of
// LDS.  The shell terms of u(v') are evaluated one per lane and summed by lane
// 0 in ascending shell order, the order of the sequential definition.
// known: n_hb is N_HB_raw; otherwise a move that crosses v = 2 is left
// pending, n_hb being the part of N_HB_raw that is complete now (lane 0's).
__device__ __forceinline__ void open_step(const VolArgs& a, const VolState& s, double* term, StepView* view, bool known,
                                          int64_t n_hb, int lane)
{
    DevState* st = a.st;
    if (s.t_next >= s.stop_at) {                     // step limit: the step's launches do nothing
        if (lane == 0) {
            view->skip = 1;
            view->pending = 0;
        }
        return;
    }
    const uint32_t t = (uint32_t)s.t_next;
    const uint4 w = philox(0u, t, 0u, kStreamVol, a.key0, a.key1);
    const double x = (double)((int64_t)2 * (int64_t)w.x + 1 - 4294967296LL) * (1.0 / 4294967296.0);
    const double v1 = s.v + a.dv_max * x;
    const bool inside = a.do_volume && v1 >= 1.0;
    if (inside && lane >= 1 && lane <= 36) {
        const double d2 = v1 * (double)lane;
        const double s6 = 1.0 / (d2 * d2 * d2);
        term[lane] = s.r2 * (s6 * s6 - s6);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    if (lane != 0) return;
    double v = s.v, u = s.u;
    int th = s.theta, pending = 0;
    int64_t vatt = s.vol_att, vacc = s.vol_acc;
    if (a.do_volume) {
        vatt += 1;
        if (inside) {
            // six shell terms read at a time, then added in ascending m
            // while v' m <= 36 (v' >= 1, so the condition fails past m = 36;
            // it is monotone in m, so the terms added and their order are
            // those of the loop that stops at the first failing m)
            double sum = 0.0;
#pragma unroll 1
            for (int m0 = 1; m0 <= 36; m0 += 6) {
                double tm[6];
#pragma unroll
                for (int k = 0; k < 6; ++k) tm[k] = term[m0 + k];
#pragma unroll
                for (int k = 0; k < 6; ++k)
                    if (v1 * (double)(m0 + k) <= 36.0) sum = sum + tm[k];
            }
            const double u1 = 2.0 * sum;
            const int th1 = v1 < 2.0 ? 1 : 0;
            if (!known && th1 != s.theta) {
                st->pend = {s.v, s.u, v1, u1, n_hb, w.y, s.theta, th1, 0};
                pending = 1;
            } else if (vol_accept(a, s.v, s.u, s.theta, v1, u1, th1, known ? n_hb : 0, w.y)) {
                v = v1;
                u = u1;
                th = th1;
                vacc += 1;
            }
        }
    }
    *view = {0, th, th, t, pending, 0};
    st->t_next = s.t_next + 1;
    st->met_att = s.met_att + a.met_att_add;
    st->vol_att = vatt;
    st->vol_acc = vacc;
    st->v = v;
    st->u = u;
    st->theta = th;
}

// First step of a call, by one wavefront: folds the counter slots of the calls
// before it into the totals and opens the step with N_HB_raw known.  Every
// global load is issued before the first store.  kVolFold: the fold alone,
// and the observables' accumulators cleared for the recount that follows.
__device__ void volume_step(const VolArgs& a, double* term, StepView* view)
{
    constexpr int kPer = 2 * kSlots / 64;
    const int lane = threadIdx.x & 63;
    DevState* st = a.st;
    int64_t sl[3][kPer];
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int b = k / (kSlots / 64), i = k % (kSlots / 64);
            sl[j][k] = a.slots[b * kBankSlots + j * kSlots + i * 64 + lane];
        }
    const VolState s = vol_load(a, lane);
    const int64_t hb0 = st->n_hb_raw, co0 = st->n_coop, macc0 = st->met_acc;
    int64_t r[3] = {0, 0, 0};
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int k = 0; k < kPer; ++k) r[j] += sl[j][k];
    for (int k = lane; k < 2 * kBankSlots; k += 64) a.slots[k] = 0;
    // the three sums in one butterfly: each step's six 32-bit exchanges are
    // issued together and waited for once
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        int64_t x[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) x[j] = __shfl_xor(r[j], o, 64);
#pragma unroll
        for (int j = 0; j < 3; ++j) r[j] += x[j];
    }
    const int64_t n_hb = hb0 + r[0], n_co = co0 + r[1];
    const bool fold = a.mode == kVolFold, stop = fold || s.t_next >= s.stop_at;
    if (fold) {
        DevObs* obs = (DevObs*)((char*)st - kOffState + kOffObs);
        if (lane < kObsAcc) obs->acc[lane] = 0;
        if (lane == 0) obs->arrived = 0;
    }
    if (lane == 0) {
        st->met_acc = macc0 + r[2];
        const bool sw = a.mode == kVolSw && !stop;   // the SW step ends with a full recount
        st->n_hb_raw = sw ? 0 : n_hb;
        st->n_coop = sw ? 0 : n_co;
    }
    if (!fold) open_step(a, s, term, view, true, n_hb, lane);
}

// A later step of a call, opened beside the last launch of the step before it
// by the wavefronts that call this (the first one of the workgroup in a
// single-chain launch).  A pending Metropolis move first takes the slots of
// bank 0, complete since the step's first launch, into the total, so that the
// first launch of the next step finds the rest of N_HB_raw in bank 1 while it
// adds to bank 0 itself.  An SW step's recount lies in one bank.
__device__ void open_next(const VolArgs& a, double* term, StepView* view)
{
    const int lane = threadIdx.x & 63;
    DevState* st = a.st;
    const VolState s = vol_load(a, lane);
    const double far = s.theta ? 2.0 - s.v : s.v - 2.0;
    int64_t n_hb = 0;
    // uniform: the move may cross (it is less than dv_max, and v' is rounded by
    // less than another dv_max where that matters)
    if (a.do_volume && far <= 2.0 * a.dv_max) {
        n_hb = st->n_hb_raw;
        if (a.mode == kVolMet) {
            int64_t r[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                r[j] = 0;
                for (int k = lane; k < kSlots; k += 64) {
                    r[j] += a.slots[j * kSlots + k];
                    a.slots[j * kSlots + k] = 0;
                }
                r[j] = wave_sum64(r[j]);
            }
            n_hb += r[0];
            if (lane == 0) {
                st->n_hb_raw = n_hb;
                st->n_coop += r[1];
                st->met_acc += r[2];
            }
        }
    }
    open_step(a, s, term, view, false, n_hb, lane);
}

// The theta of a pending step, worked out by every wavefront of the step's
// first launch; `commit` (the workgroup that writes it down).
__device__ int resolve_step(const VolArgs& a, StepView* view, bool sw, bool commit)
{
    const int lane = threadIdx.x & 63;
    DevState* st = a.st;
    const PendingMove p = st->pend;
    int64_t n = 0;
    for (int k = lane; k < kSlots; k += 64) n += a.slots[kBankSlots + k] + (sw ? a.slots[k] : 0);
    n = wave_sum64(n) + p.n_hb;
    const bool acc = vol_accept(a, p.v0, p.u0, p.th0, p.v1, p.u1, p.th1, n, p.word);
    const int th = acc ? p.th1 : p.th0;
    if (commit && threadIdx.x == 0) {
        view->theta2 = th;
        if (acc) {
            st->v = p.v1;
            st->u = p.u1;
            st->theta = th;
            st->vol_acc += 1;
        }
    }
    return __builtin_amdgcn_readfirstlane(th);
}

__global__ __launch_bounds__(64) void volume_kernel(VolArgs a)
{
    __shared__ double term[40];
    volume_step(a, term, a.st->view);
}

#include "met_sweep.h"
#include "met_domain.h"

#include "sw_step.h"
#include "recount.h"

// N_q' of the current sigma (q' < 6), added to out[0..5].  The planes are
// read as 32-bit words, four at a time and two such loads in flight per lane:
// with one word at a time 512 workgroups had too few bytes in flight (60 us at
// L = 4096, 195 at L = 8192, 998 at L = 16384; now 35, 80 and 302).
struct Words4 {
    uint32_t w[4];
};

// Adds 28 + the bytes of w other than k to c[k].
__device__ __forceinline__ void count_others(uint32_t w, int (&c)[6])
{
#pragma unroll
    for (uint32_t k = 0; k < 6; ++k) {
        const uint32_t x = w ^ (k * 0x01010101u);
        c[k] += __popc(((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x | 0x7F7F7F7Fu);
    }
}

__global__ __launch_bounds__(kBlock) void state_counts_kernel(const uint32_t* __restrict__ words, uint32_t nwords,
                                                              int64_t* out)
{
    int c[6] = {0, 0, 0, 0, 0, 0}, n = 0;               // n: words counted
    const uint32_t i0 = blockIdx.x * kBlock + threadIdx.x, stride = gridDim.x * kBlock, n4 = nwords / 4;
    auto load = [words](uint32_t i) {                  // 16 bytes, aligned to 4
        Words4 v;
        __builtin_memcpy(&v, words + 4 * (size_t)i, 16);
        return v;
    };
    uint32_t i = i0;
    for (; i + stride < n4; i += 2 * stride, n += 8) {
        const Words4 a = load(i), b = load(i + stride);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            count_others(a.w[j], c);
            count_others(b.w[j], c);
        }
    }
    if (i < n4) {
        const Words4 a = load(i);
#pragma unroll
        for (int j = 0; j < 4; ++j) count_others(a.w[j], c);
        n += 4;
    }
    if (i0 < nwords % 4) {
        count_others(words[4 * n4 + i0], c);
        ++n;
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) c[k] = 32 * n - c[k];
    block_add<6>(c, out, 1);
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------
hipError_t launch_state_init(DevState* st, int64_t* slots, const DevTables* tab, double v_init, hipStream_t s)
{
    state_init_kernel<<<1, 64, 0, s>>>(st, slots, tab, v_init);
    return hipGetLastError();
}

hipError_t launch_sigma_init(const LatticeArgs& a, hipStream_t s)
{
    sigma_init_kernel<<<grid_for(a.N), kBlock, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_volume(const VolArgs& a, hipStream_t s, DispatchEvents ev)
{
    return go(volume_kernel, dim3(1), dim3(64), s, ev, a);
}

// A launch that opens the next step has one more row of workgroups, whose
// first one does it.
template <int Q, bool R, bool LE, int POLICY = kThrough>
hipError_t launch_quad_r(const LatticeArgs& a, const VolArgs& v, StepCtl c, int colour, dim3 grid, hipStream_t s,
                         const DispatchEvents& ev)
{
    if (colour == 0) return go(met_sweep4_kernel<Q, 0, R, LE, POLICY>, grid, dim3(256), s, ev, a, v, c);
    return go(met_sweep4_kernel<Q, 1, R, LE, POLICY>, grid, dim3(256), s, ev, a, v, c);
}

template <int Q>
hipError_t launch_quad(const LatticeArgs& a, const VolArgs& v, StepCtl c, int colour, dim3 grid, hipStream_t s,
                       const DispatchEvents& ev)
{
    if (a.quad == 2 && !met_through(a.L)) {
        if (a.met_le) return launch_quad_r<Q, true, true, kPlain>(a, v, c, colour, grid, s, ev);
        return launch_quad_r<Q, true, false, kPlain>(a, v, c, colour, grid, s, ev);
    }
    if (a.quad == 2) {
        if (a.met_le) return launch_quad_r<Q, true, true>(a, v, c, colour, grid, s, ev);
        return launch_quad_r<Q, true, false>(a, v, c, colour, grid, s, ev);
    }
    if (a.met_le) return launch_quad_r<Q, false, true>(a, v, c, colour, grid, s, ev);
    return launch_quad_r<Q, false, false>(a, v, c, colour, grid, s, ev);
}

hipError_t launch_met_colour(const LatticeArgs& a, const VolArgs& v, StepCtl c, int colour, hipStream_t s,
                             DispatchEvents ev)
{
    const dim3 grid(((a.L + 3) / 4 + 63) / 64, a.row_blocks + c.open);
    switch (a.q) {
    case 2: return launch_quad<2>(a, v, c, colour, grid, s, ev);
    case 3: return launch_quad<3>(a, v, c, colour, grid, s, ev);
    case 4: return launch_quad<4>(a, v, c, colour, grid, s, ev);
    case 5: return launch_quad<5>(a, v, c, colour, grid, s, ev);
    default: return launch_quad<6>(a, v, c, colour, grid, s, ev);
    }
}

__global__ void set_stop_kernel(DevState* st, int64_t stop_at)
{
    if (threadIdx.x == 0) st->stop_at = stop_at;
}

__global__ void tables_init_kernel(DevTables* dst, DevTables src)
{
    const uint32_t* in = (const uint32_t*)&src;
    uint32_t* out = (uint32_t*)dst;
    for (uint32_t i = threadIdx.x; i < sizeof(DevTables) / 4; i += blockDim.x) out[i] = in[i];
}

hipError_t launch_tables_init(DevTables* dst, const DevTables& src, hipStream_t s)
{
    tables_init_kernel<<<1, 64, 0, s>>>(dst, src);
    return hipGetLastError();
}

// Per-device address of `scratch`, taken once per device with that device
// current (each GPU holds its own copy at its own address).
hipError_t noalloc_scratch(void** ptr)
{
    constexpr int kMaxDevices = 64;
    static std::atomic<void*> addr[kMaxDevices];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    void* p = addr[dev].load(std::memory_order_acquire);
    if (!p) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p || ((uintptr_t)p & 255) != 0) return hipErrorInvalidSymbol;
        addr[dev].store(p, std::memory_order_release);
    }
    *ptr = p;
    return hipSuccess;
}

hipError_t launch_set_stop(DevState* st, int64_t stop_at, hipStream_t s)
{
    set_stop_kernel<<<1, 64, 0, s>>>(st, stop_at);
    return hipGetLastError();
}

template <int Q>
hipError_t launch_domain_q(const LatticeArgs& a, const VolArgs& v, StepCtl c, uint32_t group, dim3 grid, uint32_t rows,
                           hipStream_t s, const DispatchEvents& ev)
{
    if (a.L % 4 == 0) return go(met_domain_kernel<Q, 0>, grid, dim3(256), s, ev, a, v, c, group, rows);
    if (a.L > 4) return go(met_domain_kernel<Q, 1>, grid, dim3(256), s, ev, a, v, c, group, rows);
    return go(met_domain_kernel<Q, 2>, grid, dim3(256), s, ev, a, v, c, group, rows);
}

hipError_t launch_met_domain(const LatticeArgs& a, const VolArgs& v, StepCtl c, uint32_t group, hipStream_t s,
                             DispatchEvents ev)
{
    // lanes own column quads; rows per lane for at most 5000 wavefronts, up to
    // 8 (a lane's 10-bit counter fields take 170 moves, a row has up to 8).
    // Measured, us per sweep: one / two rows 20.5 / 21.3 at L = 1025 (4126
    // wavefronts of one row), 19.5 / 20.6 at L = 1128 (4970), 20.6 / 20.8 at
    // L = 1160 (5256), 24.1 / 23.2 at L = 1203 (5657), 22.5 / 23.4 at L = 1300
    // (6602) and 28.7 / 25.4 at L = 1414 (7821); two / four
    // 34.9 / 33.9 at L = 2048; four / eight / sixteen 97.1 / 94.3 / 99.2 at
    // L = 4096
    const uint64_t quads = (a.L + 3) / 4;
    const uint64_t waves = (quads * a.L + 63) / 64;
    const uint32_t rows = (uint32_t)std::min<uint64_t>(8, (waves + 4999) / 5000);
    const uint64_t units = quads * ((a.L + rows - 1) / rows);
    const dim3 grid((uint32_t)((units + 255) / 256) + c.open);
    switch (a.q) {
    case 2: return launch_domain_q<2>(a, v, c, group, grid, rows, s, ev);
    case 3: return launch_domain_q<3>(a, v, c, group, grid, rows, s, ev);
    case 4: return launch_domain_q<4>(a, v, c, group, grid, rows, s, ev);
    case 5: return launch_domain_q<5>(a, v, c, group, grid, rows, s, ev);
    default: return launch_domain_q<6>(a, v, c, group, grid, rows, s, ev);
    }
}

// Quads of four x-adjacent cells.  The observables' sums meet in a few
// addresses, the counter slots are many.
template <bool OBS>
hipError_t recount_launch(const LatticeArgs& a, int64_t* out, int spread, const ObsArgs& o, hipStream_t s)
{
    RecountShape sh;
    sh.per_row = (a.L + 3) / 4;
    sh.quads = sh.per_row * a.L;
    sh.inv_row = 1.0 / (double)sh.per_row;
    const uint32_t blocks = (sh.quads + kBlock - 1) / kBlock;
    const uint32_t most = OBS ? kRecountBlocks : 2048u;
    const uint32_t grid = blocks < most ? blocks : most;
    if (a.L % 4 == 0) recount_kernel<0, OBS><<<grid, kBlock, 0, s>>>(a, sh, out, spread, o);
    else if (a.L > 4) recount_kernel<1, OBS><<<grid, kBlock, 0, s>>>(a, sh, out, spread, o);
    else recount_kernel<2, OBS><<<grid, kBlock, 0, s>>>(a, sh, out, spread, o);
    return hipGetLastError();
}

hipError_t launch_recount(const LatticeArgs& a, int64_t* slots, hipStream_t s)
{
    return recount_launch<false>(a, slots, kSlots, ObsArgs{}, s);
}

hipError_t launch_obs(const LatticeArgs& a, const ObsArgs& o, hipStream_t s)
{
    return recount_launch<true>(a, o.obs->acc, kObsSpread, o, s);
}

hipError_t launch_state_counts(const LatticeArgs& a, int64_t* out, hipStream_t s)
{
    const uint32_t nwords = a.N;                          // 4N bytes
    // at most kRecountBlocks workgroups, whose sums meet in six addresses
    state_counts_kernel<<<grid_for(nwords) < kRecountBlocks ? grid_for(nwords) : kRecountBlocks, kBlock, 0, s>>>(reinterpret_cast<const uint32_t*>(a.sigma), nwords, out);
    return hipGetLastError();
}

hipError_t launch_sw_tiles(const LatticeArgs& a, const VolArgs& v, StepCtl c, hipStream_t s, DispatchEvents ev)
{
    const dim3 grid((a.L + kTW - 1) / kTW, (a.L + kTH - 1) / kTH);
    return go(sw_tile_kernel, grid, dim3(kTT), s, ev, a, v, c);
}

__global__ void sw_counters_init_kernel(uint32_t* ecnt, uint32_t n)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) ecnt[i] = 0;
}

hipError_t launch_sw_counters_init(const LatticeArgs& a, hipStream_t s)
{
    const uint32_t n = 2 * ((a.L + kTW - 1) / kTW) * ((a.L + kTH - 1) / kTH);
    sw_counters_init_kernel<<<grid_for(n), kBlock, 0, s>>>(a.ecnt, n);
    return hipGetLastError();
}

template <int Q>
void launch_batch_q(BatchEntry* ent, const uint32_t* start, uint32_t count, uint32_t total, int colour, int le,
                    StepCtl c, hipStream_t s)
{
    const uint32_t grid = total + (c.open ? open_blocks(count, kMetWaves) : 0u);
    if (le) {
        if (colour == 0) met_batch_kernel<Q, 0, true><<<grid, 64 * kMetWaves, 0, s>>>(ent, ent, start, count, total, c);
        else met_batch_kernel<Q, 1, true><<<grid, 64 * kMetWaves, 0, s>>>(ent, ent, start, count, total, c);
    } else {
        if (colour == 0) met_batch_kernel<Q, 0, false><<<grid, 64 * kMetWaves, 0, s>>>(ent, ent, start, count, total, c);
        else met_batch_kernel<Q, 1, false><<<grid, 64 * kMetWaves, 0, s>>>(ent, ent, start, count, total, c);
    }
}

hipError_t launch_met_batch(BatchEntry* ent, const uint32_t* start, uint32_t count, uint32_t total_blocks, int q,
                            int colour, int le, StepCtl c, hipStream_t s)
{
    switch (q) {
    case 2: launch_batch_q<2>(ent, start, count, total_blocks, colour, le, c, s); break;
    case 3: launch_batch_q<3>(ent, start, count, total_blocks, colour, le, c, s); break;
    case 4: launch_batch_q<4>(ent, start, count, total_blocks, colour, le, c, s); break;
    case 5: launch_batch_q<5>(ent, start, count, total_blocks, colour, le, c, s); break;
    default: launch_batch_q<6>(ent, start, count, total_blocks, colour, le, c, s); break;
    }
    return hipGetLastError();
}

hipError_t launch_volume_batch(BatchEntry* ent, uint32_t count, int mode, hipStream_t s)
{
    volume_batch_kernel<<<count, 64, 0, s>>>(ent, mode);
    return hipGetLastError();
}

hipError_t launch_sw_batch(BatchEntry* ent, const uint32_t* start, uint32_t count, uint32_t total_blocks, int stage,
                           StepCtl c, hipStream_t s)
{
    if (total_blocks == 0) return hipSuccess;
    if (stage == 0) sw_tile_batch_kernel<<<total_blocks, kTT, 0, s>>>(ent, start, count, c);
    else
        sw_flip_batch_kernel<<<total_blocks + (c.open ? open_blocks(count, kSwWaves) : 0u), kTT, 0, s>>>(
            ent, start, count, total_blocks, c);
    return hipGetLastError();
}

hipError_t launch_sw_flip_tiles(const LatticeArgs& a, const VolArgs& v, StepCtl c, hipStream_t s, DispatchEvents ev)
{
    const dim3 grid((a.L + kTW - 1) / kTW, (a.L + kTH - 1) / kTH + c.open);
    return go(sw_flip_tile_kernel, grid, dim3(kTT), s, ev, a, v, c);
}

hipError_t launch_sw_labels(const LatticeArgs& a, uint32_t* out, hipStream_t s)
{
    const dim3 grid((a.L + kTW - 1) / kTW, (a.L + kTH - 1) / kTH);
    sw_labels_kernel<<<grid, kTT, 0, s>>>(a, out);
    return hipGetLastError();
}

}  // namespace cvf
