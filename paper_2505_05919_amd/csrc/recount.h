// Recount of a whole lattice and the observables (included inside the kernels'
// namespace).
#pragma once

// Workgroups of a recount.  Each adds a handful of 64-bit sums to a few
// addresses, ~13 ns per addition to one address: with a workgroup per 256
// cells those additions took 54 us at L = 1024 and 108 us at L = 4096, more
// than reading the lattice.
constexpr uint32_t kRecountBlocks = 512;

struct RecountShape {
    uint32_t per_row, quads;       // quads of four cells per row, in all
    double inv_row;                // 1 / per_row
};

// The n bytes of a quad at p, the others zero.  MODE 0: L % 4 == 0, an aligned
// dword.  1: other L > 4, a dword at any byte address, which the loads take; the
// last quad of a row (n < 4) reads the row's last dword and shifts it, so that
// no access leaves the row.  2: L = 2, 3, single bytes.  (With rows of L % 4 == 2
// in half words and odd rows in single bytes the observables took 1.34 and 2.27
// ms at L = 16382 and 16383, now 0.57; L = 16384 takes 0.55.)
template <int MODE>
__device__ __forceinline__ uint32_t row_bytes(const uint8_t* p, uint32_t n)
{
    if (MODE == 0) return *(const uint32_t*)p;
    uint32_t w = 0;
    if (MODE == 1) {
        __builtin_memcpy(&w, p - (4 - n), 4);
        return w >> (8 * (4 - n));
    }
    for (uint32_t j = 0; j < n; ++j) w |= (uint32_t)p[j] << (8 * j);
    return w;
}

// N_HB_raw and N_sigma of the lattice added to out[0 / 1][spread] (OBS =
// false), or with the state counts to the observables' accumulators, from
// which the workgroup that arrives last writes the record (Eq. (1), (3)).
// Values are counted exactly for any byte.  Bound by reading 4 bytes per cell
// and by ~250 VALU instructions per quad.
template <int MODE, bool OBS>
__global__ __launch_bounds__(kBlock) void recount_kernel(LatticeArgs a, RecountShape sh, int64_t* out, int spread,
                                                         ObsArgs o)
{
    const uint32_t L = a.L;
    const size_t N = a.N;
    const uint8_t* __restrict__ s = a.sigma;
    int v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (uint32_t u = blockIdx.x * kBlock + threadIdx.x; u < sh.quads; u += gridDim.x * kBlock) {
        uint32_t j;
        const uint32_t y = divmod(u, sh.per_row, sh.inv_row, j);
        const uint32_t x = 4 * j, n = min(4u, L - x);
        const uint32_t row = y * L, rowp = (y + 1 == L) ? 0u : row + L;
        const uint8_t* c = s + row + x;
        const uint32_t w[4] = {row_bytes<MODE>(c, n), row_bytes<MODE>(c + N, n),
                               row_bytes<MODE>(c + 2 * N, n), row_bytes<MODE>(c + 3 * N, n)};
        const uint32_t nx = s[N + row + (x + n == L ? 0u : x + n)];       // arm 1 right of the quad
        const uint32_t f0 = (w[1] >> 8) | (nx << (8 * (n - 1)));
        const uint32_t f2 = row_bytes<MODE>(s + 3 * N + rowp + x, n);
        const uint32_t have = 0x01010101u >> (8 * (4 - n));
        v[0] += __popc(zero_bytes(w[0] ^ f0) & have) + __popc(zero_bytes(w[2] ^ f2) & have);
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int q = p + 1; q < 4; ++q) v[1] += __popc(zero_bytes(w[p] ^ w[q]) & have);
        if (OBS) {
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (uint32_t k = 0; k < 6; ++k) v[2 + k] += __popc(zero_bytes(w[p] ^ (k * 0x01010101u)) & have);
        }
    }
    int64_t* dst = out + (blockIdx.x & (spread - 1));
    if (!OBS) {
        const int v2[2] = {v[0], v[1]};
        block_add<2>(v2, dst, spread);
        return;
    }
    block_add<8>(v, dst, spread);
    // The workgroup's additions come before its arrival (the barrier and the
    // arrival's release), and the last workgroup reads the sums after it has
    // seen every arrival (its acquire, which the others do without: it would
    // invalidate the L2 they read the lattice through).  The release costs
    // nothing up to L = 2048 and 3.5 us of 69 at L = 4096; an acquire in every
    // workgroup took 2.5 us at L = 1024 and 5 at L = 4096.
    __syncthreads();
    __shared__ uint32_t last;
    if (threadIdx.x == 0)
        last = __hip_atomic_fetch_add(&o.obs->arrived, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT) + 1 == gridDim.x;
    __syncthreads();
    if (!last || threadIdx.x != 0) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    int64_t acc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        acc[k] = 0;
#pragma unroll
        for (int i = 0; i < kObsSpread; ++i)
            acc[k] += __hip_atomic_load(o.obs->acc + k * kObsSpread + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const DevState* st = a.st;
    cvf_obs& r = o.obs->out;
    r.step = st->t_next;
    r.n_hb_raw = acc[0];
    r.n_hb = st->theta ? acc[0] : 0;
    r.n_coop = acc[1];
    int64_t mx = 0;
    for (int k = 0; k < 6; ++k) {
        r.count[k] = acc[2 + k];
        mx = r.count[k] > mx ? r.count[k] : mx;
    }
    r.met_attempted = st->met_att;
    r.met_accepted = st->met_acc;
    r.vol_attempted = st->vol_att;
    r.vol_accepted = st->vol_acc;
    r.v = st->v;
    r.V = (o.Nd * st->v) + (o.vHB * (double)r.n_hb);
    // st->u is u_LJ(v), summed in the order of lj_energy when v was accepted
    r.H = (((o.Nd * st->u) - (o.J * (double)r.n_hb)) - (o.Jsigma * (double)r.n_coop)) + (o.P * r.V);
    r.M = (double)mx / (4.0 * o.Nd);
    r.consistent = (st->n_hb_raw == acc[0] && st->n_coop == acc[1]) ? 1 : 0;
    r.reserved = 0;
}
