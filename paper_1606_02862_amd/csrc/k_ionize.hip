// Monte Carlo electron-impact ionisation: per-cell electron moments, the
// exact Maxwellian-averaged Lotz rate by 64-point Gauss-Laguerre quadrature
// in FP64, the Philox draw per ion and the append of the new electrons to
// the ion's own supercell.
#include "ionize_step.hpp"

namespace pic {

// ---------------------------------------------------------------- moments
// Nearest-grid-point moments of one species per cell (sum w, sum w u,
// sum w |u|^2) accumulated in FP64 in LDS, one workgroup per supercell, then
// n_e = (sum w / dV) n_ref and kT = m_e c^2 (sum w u^2 / N - |ubar|^2) / 3;
// with mom4, also N = sum w and ubar per cell.
__global__ __launch_bounds__(BLOCK) void k_moments(GridView g, SpeciesView e, double n_ref_over_dv, double* ne,
                                                   double* kT, double* mom4)
{
    __shared__ MomLds m;
    const int sc = blockIdx.x;
    moments_accumulate(e, sc, m);
    const int cell = threadIdx.x;
    moments_store(moments_cell(m, cell, n_ref_over_dv), cell_index(g, sc, cell), ne, kT, mom4);
}

hipError_t launch_moments(const GridView& g, const SpeciesView& e, double n_ref_over_dv, double* ne, double* kT,
                          double* mom4, hipStream_t st)
{
    hipLaunchKernelGGL(k_moments, dim3(g.nsc), dim3(BLOCK), 0, st, g, e, n_ref_over_dv, ne, kT, mom4);
    return hipGetLastError();
}

// The moments of the staged step and, per supercell, the (cell, Z) pairs that
// the rate stage rates and the cell of every ion for the draw.
__global__ __launch_bounds__(BLOCK) void k_moments_pairs(GridView g, SpeciesView e, SpeciesView ion, int z_max,
                                                         PairBuffers pb, double n_ref_over_dv, double* ne, double* kT,
                                                         double* mom4)
{
    __shared__ MomLds m;
    __shared__ PairLds pl;
    const int sc = blockIdx.x, tid = threadIdx.x;
    moments_accumulate(e, sc, m);
    moments_store(moments_cell(m, tid, n_ref_over_dv), cell_index(g, sc, tid), ne, kT, mom4);
    uint16_t* const list = pb.list + (int64_t)sc * pb.cap;
    const int np = pairs_build(ion, sc, z_max, pl, pb.cell,
                               [&](int i, int c, int Z) { list[i] = (uint16_t)(c | Z << 8); });
    pb.info[(int64_t)sc * SC_CELLS + tid] = (uint32_t)pl.off[tid] << PAIR_MASK_BITS | pl.mask[tid];
    if (tid == 0) pb.count[sc] = np;
}

hipError_t launch_moments_pairs(const GridView& g, const SpeciesView& e, const SpeciesView& ion, int z_max,
                                const PairBuffers& pb, double n_ref_over_dv, double* ne, double* kT, double* mom4,
                                hipStream_t st)
{
    if (pb.cap < pair_cap(z_max, ion.cap)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_moments_pairs, dim3(g.nsc), dim3(BLOCK), 0, st, g, e, ion, z_max, pb, n_ref_over_dv, ne, kT,
                       mom4);
    return hipGetLastError();
}

// ---------------------------------------------------------------- exact rate
// The quadrature of every pair, four lanes each: FP64 ALU bound.  Rating the
// pairs instead of the ions divides the work by the ions per cell and state.
__global__ __launch_bounds__(BLOCK) void k_rate_exact(GridView g, PairBuffers pb, IonTables tab, const double* ne,
                                                      const double* kT, const double* gl)
{
    __shared__ GlRule rule;
    const int sc = blockIdx.x;
    const int tid = threadIdx.x;
    load_rule(gl, rule);
    __syncthreads();
    const int n = pb.count[sc];
    const int64_t base = (int64_t)sc * pb.cap;
    rates_of_pairs<BLOCK>(
        n, tab, rule,
        [&](int i, double& t, double& d, int& Z) {
            const int pr = pb.list[base + i];
            const int64_t gi = cell_index(g, sc, pr & 255);
            t = kT[gi];
            d = ne[gi];
            Z = pr >> 8;
        },
        [&](int i, double v) { pb.nu[base + i] = v; });
}

hipError_t launch_rate_exact(const GridView& g, const PairBuffers& pb, const IonTables& tab, const double* ne,
                             const double* kT, const double* gl, hipStream_t st)
{
    hipLaunchKernelGGL(k_rate_exact, dim3(g.nsc), dim3(BLOCK), 0, st, g, pb, tab, ne, kT, gl);
    return hipGetLastError();
}

// Exact ln nu for independent samples (rate evaluation entry point).
__global__ __launch_bounds__(BLOCK) void k_ln_rate_exact(int64_t n, const double* kT, const double* ne,
                                                         const int32_t* Z, IonTables tab, const double* gl,
                                                         double* out)
{
    __shared__ GlRule rule;
    load_rule(gl, rule);
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    if (i >= n) return;
    const int z = Z[i];
    out[i] = (z >= 0 && z < tab.z_max) ? ln_rate_exact(kT[i], ne[i], tab, z, rule) : -INFINITY;
}

hipError_t launch_ln_rate_exact(int64_t n, const double* kT, const double* ne, const int32_t* Z, const IonTables& tab,
                                const double* gl, double* out, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_ln_rate_exact, dim3((unsigned)((n + BLOCK - 1) / BLOCK)), dim3(BLOCK), 0, st, n, kT, ne, Z,
                       tab, gl, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------- draw + append
// Per ion with Z < z_max (counted, striped, at CNT_ACTIVE): its events, then
// one electron per event at the end of the same supercell's electron frames
// (one LDS atomic per ion with events), with the position, momentum and
// weight of the ion; the charge state rises by the events that found a slot.
// With energy loss, w * P_Z of those events goes to the cell's de and the
// supercell's electron count before the appends to old_count.
// CHAIN: max_events > 1 (the instantiation for one event carries no quadrature).
template <bool CHAIN>
__global__ __launch_bounds__(BLOCK) void k_draw_append(GridView g, SpeciesView ion, SpeciesView el, IonTables tab,
                                                       DrawArgs a, PairBuffers pb, DrawBuffers db,
                                                       unsigned long long* counters)
{
    __shared__ GlRule rule;
    __shared__ DrawLds s_d;
    __shared__ uint32_t s_info[SC_CELLS];  // the cells' pairs
    __shared__ double s_first[SC_CELLS * PIC_MAX_ZSTATES];  // first_event of each, sign as in pb.nu
    const int sc = blockIdx.x;
    const int tid = threadIdx.x;
    if (CHAIN) load_rule(db.gl, rule);
    if (tid == 0) s_d = DrawLds{0, 0, 0, 0};
    s_info[tid] = pb.info[(int64_t)sc * SC_CELLS + tid];
    for (int i = tid, np = pb.count[sc]; i < np; i += BLOCK) {
        const double nu = pb.nu[(int64_t)sc * pb.cap + i];
        s_first[i] = copysign(first_event<CHAIN>(fabs(nu), a), nu);
    }
    __syncthreads();
    const int n = ion.count[sc];
    const int ebase = el.count[sc];
    const int room = el.cap - ebase;
    const int64_t base = (int64_t)sc * ion.cap;
    bool full = false;
    int fired = 0, active = 0, fb = 0;
    // chunks of DRAW_PER slots per lane: every load of a chunk is issued
    // before the first decision, so the lanes wait on memory once per chunk
    constexpr int DRAW_PER = 4;
    for (int c0 = 0; c0 < n; c0 += BLOCK * DRAW_PER) {
        int zs[DRAW_PER], cells[DRAW_PER];
        uint32_t ids[DRAW_PER];
#pragma unroll
        for (int k = 0; k < DRAW_PER; ++k) {
            const int t = c0 + k * BLOCK + tid;
            zs[k] = tab.z_max;  // inactive
            cells[k] = 0;
            ids[k] = 0;
            if (t < n) {
                const int64_t p = base + t;
                zs[k] = ion.zs[p];
                cells[k] = pb.cell[p];
                ids[k] = ion.id[p];
            }
        }
#pragma unroll
        for (int k = 0; k < DRAW_PER; ++k) {
            const int Z0 = zs[k];
            const int64_t p = base + c0 + k * BLOCK + tid;
            int nev = 0;
            int64_t gi = 0;
            if (Z0 < tab.z_max) {
                ++active;
                const uint32_t info = s_info[cells[k]];
                const double first = s_first[(info >> PAIR_MASK_BITS) + __popc(info & ((1u << Z0) - 1u))];
                fb += signbit(first) ? 1 : 0;  // rated by the exact fallback
                // the ion's cell, for later events' rates and the energy account only
                if (CHAIN || a.energy_loss) gi = cell_index(g, sc, cells[k]);
                nev = ion_events<CHAIN>(tab, a, ids[k], Z0, fabs(first), CHAIN ? db.kT[gi] : 0.0,
                                        CHAIN ? db.ne[gi] : 0.0, rule);
            }
            const int b = wave_reserve<CHAIN>(nev, &s_d.add);  // every lane of the wave
            if (nev) fired += append_events(ion, el, tab, a, db.de, sc, p, gi, ids[k], Z0, nev, b, ebase, room, full);
        }
    }
    if (full) g.flags[FLAG_CAPACITY] = 1;
    if (fired) atomicAdd(&s_d.fired, fired);
    if (active) atomicAdd(&s_d.active, active);
    if (fb) atomicAdd(&s_d.fb, fb);
    __syncthreads();
    if (tid == 0) draw_finish(el, a, db, sc, ebase, room, s_d, counters);
}

hipError_t launch_draw_append(const GridView& g, const SpeciesView& ion, const SpeciesView& el, const IonTables& tab,
                              const DrawArgs& a, const PairBuffers& pb, const DrawBuffers& b,
                              unsigned long long* counters, hipStream_t st)
{
    if (a.energy_loss && (!b.de || !b.old_count || !b.mom4)) return hipErrorInvalidValue;
    if (a.max_events > 1)
        hipLaunchKernelGGL(k_draw_append<true>, dim3(g.nsc), dim3(BLOCK), 0, st, g, ion, el, tab, a, pb, b, counters);
    else
        hipLaunchKernelGGL(k_draw_append<false>, dim3(g.nsc), dim3(BLOCK), 0, st, g, ion, el, tab, a, pb, b, counters);
    return hipGetLastError();
}

// One ionisation step of one ion species with the exact rate, fused per
// supercell (one workgroup each): the electron moments of its cells in LDS
// (written to the grid as well), the exact rate of each (cell, Z) pair that
// its ions occupy, four lanes each, and for each ion the draw and append of
// its events.  Held to four waves per SIMD with one event (one register more
// and it took 0.35 instead of 0.30 ms on 128^3).
template <bool CHAIN>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(CHAIN ? 3 : 4))) void k_ionize_exact(GridView g, SpeciesView ion, SpeciesView el, IonTables tab,
                                                        DrawArgs a, DrawBuffers db, double n_ref_over_dv, double* ne,
                                                        double* kT, double* mom4, unsigned long long* counters)
{
    __shared__ MomLds mom;
    __shared__ PairLds pl;
    __shared__ uint16_t s_list[SC_CELLS * PIC_MAX_ZSTATES];
    __shared__ double s_nu[SC_CELLS * PIC_MAX_ZSTATES];
    __shared__ GlRule rule;
    __shared__ DrawLds s_d;
    const int sc = blockIdx.x;
    const int tid = threadIdx.x;
    load_rule(db.gl, rule);
    if (tid == 0) s_d = DrawLds{0, 0, 0, 0};
    moments_accumulate(el, sc, mom);  // its barriers also publish the rule and the reset above
    {
        // each thread reads and rewrites only its own cell's column
        const CellMoments cm = moments_cell(mom, tid, n_ref_over_dv);
        moments_store(cm, cell_index(g, sc, tid), ne, kT, mom4);
        mom.acc[0][tid] = cm.ne;
        mom.acc[1][tid] = cm.kT;
    }
    const int np = pairs_build(ion, sc, tab.z_max, pl, nullptr,
                               [&](int i, int c, int Z) { s_list[i] = (uint16_t)(c | Z << 8); });
    rates_of_pairs<BLOCK>(
        np, tab, rule,
        [&](int i, double& t, double& d, int& Z) {
            const int pr = s_list[i], c = pr & 255;
            t = mom.acc[1][c];
            d = mom.acc[0][c];
            Z = pr >> 8;
        },
        [&](int i, double v) { s_nu[i] = v; });
    if constexpr (!CHAIN) {
        __syncthreads();
        for (int i = tid; i < np; i += BLOCK) s_nu[i] = first_event<CHAIN>(s_nu[i], a);
    }
    __syncthreads();
    const int n = ion.count[sc];
    const int ebase = el.count[sc];
    const int room = el.cap - ebase;
    const int64_t base = (int64_t)sc * ion.cap;
    bool full = false;
    int fired = 0, active = 0;
    for (int t0 = 0; t0 < n; t0 += BLOCK) {  // every lane runs every pass (the appends are per wave)
        const int t = t0 + tid;
        const int64_t p = base + t;
        const int Z = t < n ? (int)ion.zs[p] : tab.z_max;
        int nev = 0, cell = 0;
        uint32_t id = 0;
        if (Z < tab.z_max) {
            ++active;
            cell = ion_cell(ion, p);
            const double cne = mom.acc[0][cell], ckT = mom.acc[1][cell];
            const double first = s_nu[pl.off[cell] + __popc(pl.mask[cell] & ((1u << Z) - 1u))];
            id = ion.id[p];
            nev = ion_events<CHAIN>(tab, a, id, Z, first, ckT, cne, rule);
        }
        const int b = wave_reserve<CHAIN>(nev, &s_d.add);
        if (nev) {
            const int64_t gi = a.energy_loss ? cell_index(g, sc, cell) : 0;
            fired += append_events(ion, el, tab, a, db.de, sc, p, gi, id, Z, nev, b, ebase, room, full);
        }
    }
    if (full) g.flags[FLAG_CAPACITY] = 1;
    if (fired) atomicAdd(&s_d.fired, fired);
    if (active) atomicAdd(&s_d.active, active);
    __syncthreads();
    if (tid == 0) draw_finish(el, a, db, sc, ebase, room, s_d, counters);
}

hipError_t launch_ionize_exact(const GridView& g, const SpeciesView& ion, const SpeciesView& el, const IonTables& tab,
                               const DrawArgs& a, const DrawBuffers& db, double n_ref_over_dv, double* ne, double* kT,
                               double* mom4, unsigned long long* counters, hipStream_t st)
{
    if (a.energy_loss && (!db.de || !db.old_count || !mom4)) return hipErrorInvalidValue;
    if (a.max_events > 1)
        hipLaunchKernelGGL(k_ionize_exact<true>, dim3(g.nsc), dim3(BLOCK), 0, st, g, ion, el, tab, a, db, n_ref_over_dv,
                           ne, kT, mom4, counters);
    else
        hipLaunchKernelGGL(k_ionize_exact<false>, dim3(g.nsc), dim3(BLOCK), 0, st, g, ion, el, tab, a, db,
                           n_ref_over_dv, ne, kT, mom4, counters);
    return hipGetLastError();
}

// ---------------------------------------------------------------- counts
// One workgroup adds the striped counters and the electron counts and writes
// four numbers straight to pinned host memory.  Read back instead as copies of
// the counter block, of the per-supercell counts and of the error flags, they
// cost three waits of the host per step: 143 against 87 us for a table step
// on a 40x24x36 box, 500 against 434 us for a surrogate step on 128^3.
constexpr int STATS_NT = 1024;
__global__ __launch_bounds__(STATS_NT) void k_ion_stats(const int32_t* el_count, int nsc, unsigned long long* counters,
                                                        long long* stats)
{
    __shared__ long long part[STATS_NT / 64];
    __shared__ long long striped[3];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    static_assert(CNT_STRIPES == 64, "one wave adds one striped count");
    static_assert(CNT_FIRED == CNT_ACTIVE + 64 && CNT_FBIONS == CNT_FIRED + 64, "stripes in this order");
    long long n = 0;
    for (int t = tid; t < nsc; t += STATS_NT) n += el_count[t];
    long long v = wave < 3 ? (long long)counters[CNT_ACTIVE + tid] : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        n += __shfl_xor(n, o, 64);
        v += __shfl_xor(v, o, 64);
    }
    if (lane == 0) part[wave] = n;
    if (lane == 0 && wave < 3) striped[wave] = v;
    __syncthreads();
    for (int t = tid; t < CNT_WORDS; t += STATS_NT) counters[t] = 0ull;
    if (tid == 0) {
        long long total = 0;
        for (int w = 0; w < STATS_NT / 64; ++w) total += part[w];
        for (int k = 0; k < 3; ++k) stats[k] = striped[k];
        stats[3] = total;
    }
}

hipError_t launch_ion_stats(const int32_t* el_count, int nsc, unsigned long long* counters, long long* stats,
                            hipStream_t st)
{
    hipLaunchKernelGGL(k_ion_stats, dim3(1), dim3(STATS_NT), 0, st, el_count, nsc, counters, stats);
    return hipGetLastError();
}

// ---------------------------------------------------------------- energy loss
// The electrons present before the appends (slots below old_count) of a cell
// with de > 0 and 3/2 N kT > 0: u <- ubar + f (u - ubar),
// f = sqrt(max(0, 1 - de / (3/2 N kT))), in FP64.
__global__ __launch_bounds__(BLOCK) void k_energy_loss(GridView g, SpeciesView el, DrawBuffers db)
{
    const int sc = blockIdx.x;
    const int n = db.old_count[sc];
    const int64_t base = (int64_t)sc * el.cap;
    const int scx = sc % g.ncx, scy = (sc / g.ncx) % g.ncy, scz = sc / (g.ncx * g.ncy);
    for (int t = threadIdx.x; t < n; t += BLOCK) {
        const int64_t p = base + t;
        const Triple<float> r = ld3(el.pos, p);
        const int64_t gi = (int64_t)(scx * SX + (int)r.x) +
                           (int64_t)g.nx * ((scy * SY + (int)r.y) + (int64_t)g.ny * (scz * SZ + (int)r.z));
        const double d = db.de[gi];
        if (!(d > 0.0)) continue;
        const double heat = 1.5 * db.mom4[4 * gi] * db.kT[gi];
        if (!(heat > 0.0)) continue;
        const double f2 = 1.0 - d / heat;
        const double f = f2 > 0.0 ? sqrt(f2) : 0.0;
        const double bx = db.mom4[4 * gi + 1], by = db.mom4[4 * gi + 2], bz = db.mom4[4 * gi + 3];
        const Triple<float> u = ld3(el.mom, p);
        st3(el.mom, p, Triple<float>{(float)(bx + f * ((double)u.x - bx)), (float)(by + f * ((double)u.y - by)),
                                     (float)(bz + f * ((double)u.z - bz))});
    }
}

hipError_t launch_energy_loss(const GridView& g, const SpeciesView& el, const DrawBuffers& b, hipStream_t st)
{
    if (!b.de || !b.old_count || !b.mom4) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_energy_loss, dim3(g.nsc), dim3(BLOCK), 0, st, g, el, b);
    return hipGetLastError();
}

}  // namespace pic
