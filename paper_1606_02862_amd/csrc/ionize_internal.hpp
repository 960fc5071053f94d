// Internal declarations of the Monte Carlo ionisation step and its rate
// paths (exact quadrature, learned surrogate, table): the per-species Lotz
// tables, the draw arguments and buffers, the launchers each kernel file
// provides, and the device-side Lotz rate shared by the kernels.
#pragma once

#include "pic_device.hpp"
#include "rate_log.hpp"

namespace pic {

// ---------------------------------------------------------------- ionisation
constexpr int GL_NODES = 64;                 // Gauss-Laguerre points
constexpr double ME_C2_EV = 510998.95;       // electron rest energy (eV)
constexpr double C_CM_S = 2.99792458e10;     // speed of light (cm/s)
constexpr double LOTZ_A = 4.5e-14;           // Lotz constant (cm^2 eV^2)

// Lotz subshells per charge state Z (subshell 0 the outermost, sp[Z][0] = P[Z]).
struct IonTables {
    double P[PIC_MAX_ZSTATES];                    // ionisation energy of state Z (eV)
    double sp[PIC_MAX_ZSTATES][PIC_LOTZ_SHELLS];  // subshell binding energies (eV)
    double aq[PIC_MAX_ZSTATES][PIC_LOTZ_SHELLS];  // a q (cm^2 eV^2)
    double sb[PIC_MAX_ZSTATES][PIC_LOTZ_SHELLS];  // b
    double sc[PIC_MAX_ZSTATES][PIC_LOTZ_SHELLS];  // c
    int ns[PIC_MAX_ZSTATES];                      // subshells in use
    int z_max;
};

// Ionisation counters (unsigned long long): [CNT_FALLBACK] is the length of
// the fallback list; the active-ion, event and fallback-ion counts are striped
// over CNT_STRIPES words each (supercell sc adds to word sc % CNT_STRIPES) so
// that thousands of workgroups do not serialise on one address; the host sums them.
constexpr int CNT_FALLBACK = 2, CNT_STRIPES = 64;
constexpr int CNT_ACTIVE = 8, CNT_FIRED = CNT_ACTIVE + CNT_STRIPES, CNT_FBIONS = CNT_FIRED + CNT_STRIPES,
              CNT_WORDS = CNT_FBIONS + CNT_STRIPES;

// The rate depends on an ion's cell and charge state only, so a step rates
// the distinct (cell, Z) pairs its ions occupy, not the ions: per supercell,
// pair i holds cell | Z << 8 (cells in order, states ascending in a cell), and
// cell c's pairs start at off(info) and follow the bits of mask(info),
// info = off << PAIR_MASK_BITS | mask.
constexpr int PAIR_MASK_BITS = 16;
static_assert(PIC_MAX_ZSTATES <= PAIR_MASK_BITS, "one mask bit per charge state");
inline int pair_cap(int z_max, int ion_slots) { return SC_CELLS * z_max < ion_slots ? SC_CELLS * z_max : ion_slots; }
struct PairBuffers {
    int cap;             // pairs per supercell: 256 z_max, at most one for each ion slot (pair_cap)
    uint16_t* list;      // [nsc][cap]
    uint32_t* info;      // [nsc][256]
    int32_t* count;      // [nsc]
    uint8_t* cell;       // [nsc][ion.cap]: the cell of every ion with Z < z_max
    double* nu;          // [nsc][cap] rates (1/s); the sign bit marks those of the exact fallback
};

struct DrawArgs {
    uint64_t seed;
    int64_t step;
    int species_index;
    int64_t ion_id_offset;
    int64_t id_base_new;
    double dt_phys;             // dt / omega_p in seconds
    int max_events;             // <= 1: one event per ion; else the waiting-time chain
    int energy_loss;            // 1: accumulate w * P per cell into de
};
// Per-step ionisation buffers the draw and energy-loss kernels share.
struct DrawBuffers {
    const double* ne;           // per cell n_e (cm^-3)
    const double* kT;           // per cell kT_e (eV)
    const double* gl;           // Gauss-Laguerre rule and logarithm table (exact rates)
    const double* mom4;         // per cell N = sum w and mean u (energy loss), or nullptr
    double* de;                 // per cell sum of w * P over the events (energy loss), or nullptr
    int32_t* old_count;         // per supercell electron count before the appends (energy loss), or nullptr
};

// Tabulated rate (PIC_RATE_TABLE): RATE_TABLE_N nodes per charge state,
// uniform in ln kT, covering [RATE_TABLE_TMIN, RATE_TABLE_TMAX] eV.
constexpr int RATE_TABLE_N = 1024;
constexpr double RATE_TABLE_TMIN = 1e-2, RATE_TABLE_TMAX = 1e6;
hipError_t launch_rate_table_build(const IonTables& tab, const double* gl, double* table, hipStream_t st);
// fb_list: one entry per pair, for the pairs outside the table's range
hipError_t launch_rate_table(const GridView& g, const PairBuffers& pb, const IonTables& tab, const double* ne,
                             const double* kT, const double* table, const double* gl,
                             unsigned long long* counters, unsigned long long* fb_list, hipStream_t st);
hipError_t launch_ln_rate_table(int64_t n, const double* kT, const double* ne, const int32_t* Z, const IonTables& tab,
                                const double* table, const double* gl, double* out, hipStream_t st);

// host: the 64-point Gauss-Laguerre rule (nodes; weights through *w)
const double* gauss_laguerre_nodes(const double** w);

// mom4: per cell (sum w, mean ux, uy, uz), or nullptr
hipError_t launch_moments(const GridView& g, const SpeciesView& e, double n_ref_over_dv, double* ne, double* kT,
                          double* mom4, hipStream_t st);
// ... and the (cell, Z) pairs of the ions with Z < z_max
hipError_t launch_moments_pairs(const GridView& g, const SpeciesView& e, const SpeciesView& ion, int z_max,
                                const PairBuffers& pb, double n_ref_over_dv, double* ne, double* kT, double* mom4,
                                hipStream_t st);
hipError_t launch_rate_exact(const GridView& g, const PairBuffers& pb, const IonTables& tab, const double* ne,
                             const double* kT, const double* gl, hipStream_t st);
hipError_t launch_ln_rate_exact(int64_t n, const double* kT, const double* ne, const int32_t* Z, const IonTables& tab,
                                const double* gl, double* out, hipStream_t st);
hipError_t launch_draw_append(const GridView& g, const SpeciesView& ion, const SpeciesView& el, const IonTables& tab,
                              const DrawArgs& a, const PairBuffers& pb, const DrawBuffers& b,
                              unsigned long long* counters, hipStream_t st);
// The step's counts for the host: stats = {active ions, events, fallback ions,
// electrons held} written to pinned host memory, and the counters cleared for
// the next step.
constexpr int ION_STATS = 4;
hipError_t launch_ion_stats(const int32_t* el_count, int nsc, unsigned long long* counters, long long* stats,
                            hipStream_t st);
hipError_t launch_energy_loss(const GridView& g, const SpeciesView& el, const DrawBuffers& b, hipStream_t st);
// The step with the exact rate fused (moments, rate, draw and append per
// supercell in one kernel); ne, kT (and mom4) receive the cell moments as
// the staged step's do.
hipError_t launch_ionize_exact(const GridView& g, const SpeciesView& ion, const SpeciesView& el, const IonTables& tab,
                               const DrawArgs& a, const DrawBuffers& db, double n_ref_over_dv, double* ne, double* kT,
                               double* mom4, unsigned long long* counters, hipStream_t st);

// ---------------------------------------------------------------- surrogate
struct MlpLaunch {
    const float* params;   // FP32 master parameters (PIC_MLP_NPARAM)
    double mu, s;          // target standardisation
    double t_min, t_max, n_min, n_max;
    int act;               // PIC_MLP_SILU or PIC_MLP_RELU
};
struct MlpGen {
    double lt_min, lt_max, ln_min, ln_max;  // log10 ranges of kT (eV) and n_e (cm^-3)
};
struct MlpStep {
    const float* X;        // [n_data][8] features
    const float* t;        // [n_data] standardised targets
    int64_t n_data;
    int batch;             // multiple of 64
    uint64_t draw_seed;    // 0: samples 0..batch-1 in order; else Philox draws
    int64_t step;
    int act;               // PIC_MLP_SILU or PIC_MLP_RELU
};
// fb_list: one entry per pair, for the out-of-range pairs
hipError_t launch_rate_mlp(const GridView& g, const PairBuffers& pb, const IonTables& tab, const MlpLaunch& ml,
                           const double* ne, const double* kT, const double* gl, unsigned long long* counters,
                           unsigned long long* fb_list, hipStream_t st);
// The exact FP64 rate, with the sign bit set, for the counters[CNT_FALLBACK]
// pairs listed in fb_list.
hipError_t launch_rate_fallback(const GridView& g, const PairBuffers& pb, const IonTables& tab, const double* ne,
                                const double* kT, const double* gl, const unsigned long long* fb_list,
                                const unsigned long long* counters, hipStream_t st);
hipError_t launch_ln_rate_mlp(int64_t n, const double* kT, const double* ne, const int32_t* Z, const IonTables& tab,
                              const MlpLaunch& ml, const double* gl, double* out, hipStream_t st);
hipError_t launch_mlp_gen(int64_t n, uint64_t seed, const MlpGen& a, const IonTables& tab, const double* gl, float* X,
                          double* r, hipStream_t st);
hipError_t launch_mlp_standardize(int64_t n, const double* r, double* partial, double* mu_s, float* t, hipStream_t st);
hipError_t launch_mlp_init(uint64_t seed, float* P, float* m, float* v, hipStream_t st);
// A training step's gradient is summed without atomics: each workgroup of
// the step kernel writes its sum (its waves in order) to its own row of a
// partial buffer, MLP_PART_ROWS rows of MLP_PART_STRIDE floats (and its
// squared-error sum to lpart), and the Adam kernel, or launch_mlp_grad, adds
// the rows in row order.  *rows receives the number of rows written.
constexpr int MLP_PART_ROWS = 64;
constexpr int MLP_PART_STRIDE = (PIC_MLP_NPARAM + 63) / 64 * 64;
hipError_t launch_mlp_step(const float* P, const MlpStep& s, float* part, double* lpart, int* rows, hipStream_t st);
// Adam on the master parameters with the summed gradient; *loss = the summed squared error
hipError_t launch_mlp_adam(float* P, const float* part, int rows, const double* lpart, double* loss, float* m, float* v,
                           float lr, float bc1, float bc2, hipStream_t st);
// the summed gradient (PIC_MLP_NPARAM floats) and squared error
hipError_t launch_mlp_grad(const float* part, int rows, const double* lpart, float* grad, double* loss, hipStream_t st);

// Static staging of pic_rate_eval_noalloc (noalloc.hip): one device array per
// GPU, its address taken once per device by noalloc_scratch_setup (with that
// device current) and returned by noalloc_scratch (nullptr before).
struct NoallocStaging {
    double *kT, *ne, *out;
    int32_t* Z;
};
hipError_t noalloc_scratch_setup(int device);
unsigned char* noalloc_scratch(int device);
NoallocStaging noalloc_staging(unsigned char* base);

// ---------------------------------------------------------------- Lotz rate
// What the quadrature reads, in LDS: the rule and the logarithm's table.
struct GlRule {
    double x[GL_NODES], w[GL_NODES];
    double2 lt[LOG_N];
};
constexpr int GL_WORDS = 2 * GL_NODES + 2 * LOG_N;  // doubles of the device copy, in the same order
static_assert(sizeof(GlRule) == GL_WORDS * sizeof(double), "GlRule is the device copy's layout");

// Copies the rule to LDS; a barrier is the caller's.
__device__ inline void load_rule(const double* gl, GlRule& rule)
{
    double* d = reinterpret_cast<double*>(&rule);
    for (int t = threadIdx.x; t < GL_WORDS; t += blockDim.x) d[t] = gl[t];
}

// One subshell (p, a, b, c, q) with E = p + kT x:
//   <sigma v>_j = vbar (a q / (p kT)) e^{-p/kT} sum_k w_k ln(1 + x_k r) (1 - b e^{-c x_k r}),  r = kT / p,
// FP64; the exponential only where b != 0.  The nodes k0, k0 + 4, ... of the sum.
//
// Of the 64 nodes the first GL_SUM are evaluated.  f(x) = ln(1 + x r) is concave
// with f(0) = 0 and so is 1 - b e^{-c x r} from 1 - b >= 0, so each grows by at
// most x_k / x_i from node i to a later node k, and the terms from GL_SUM on
// are at most sum_{k >= GL_SUM} w_k x_k^2 / sum_i w_i x_i^2 = 2^-68 of the sum
// (2^-72 with b = 0) for every r, b and c: 2^-15 of the sum's last place, below
// what FP64 holds of it.
constexpr int GL_SUM = 36;
static_assert(GL_SUM % 4 == 0, "the four partial sums take the nodes evenly");
__host__ __device__ inline double lotz_sum(double r, double b, double c, const GlRule& rule, int k0)
{
    double s = 0.0;
    if (!(rule.x[GL_NODES - 1] * r <= LOG_Y_MAX)) {  // past log1p_pos
        for (int k = k0; k < GL_NODES; k += 4) {
            const double xr = rule.x[k] * r;
            s = fma(rule.w[k] * log1p(xr), b == 0.0 ? 1.0 : 1.0 - b * exp(-c * xr), s);
        }
    } else if (b == 0.0) {
#pragma unroll 9
        for (int k = k0; k < GL_SUM; k += 4) s = fma(rule.w[k], log1p_pos(rule.x[k] * r, rule.lt), s);
    } else {
#pragma unroll 3
        for (int k = k0; k < GL_SUM; k += 4) {
            const double xr = rule.x[k] * r;
            s = fma(rule.w[k] * log1p_pos(xr, rule.lt), 1.0 - b * exp(-c * xr), s);
        }
    }
    return s;
}

// The whole sum by one lane, in the four partial sums that four lanes take: short
// chains of additions, so that the sum is nearer its value than one chain of 64
// terms (mean error, units of 2^-53 of it, kT/p 1e-3 to 1e3: 0.68; one chain 1.68
// with the library log1p, 1.69 with log1p_pos), and the same by either path.
__host__ __device__ inline double lotz_sum4(double r, double b, double c, const GlRule& rule)
{
    double s[4];
#pragma unroll 1
    for (int j = 0; j < 4; ++j) s[j] = lotz_sum(r, b, c, rule, j);
    return (s[0] + s[1]) + (s[2] + s[3]);
}

// sum_j (a_j q_j / p_j) e^{-(p_j - P)/kT} S_j over the subshells of state Z, P = P[Z]:
// the state's <sigma v> is vbar / kT e^{-P/kT} times this.  LANES = 4: a group
// of four consecutive lanes with the same kT and Z, lane j of the group taking
// the nodes j, j + 4, ...; the four partial sums are added so that every lane
// returns the same total.
template <int LANES = 1>
__device__ inline double lotz_shells(double kT, const IonTables& t, int Z, const GlRule& rule)
{
    static_assert(LANES == 1 || LANES == 4, "one lane or a group of four");
    double acc = 0.0;
    for (int j = 0; j < t.ns[Z]; ++j) {
        const double p = t.sp[Z][j];
        double s;
        if constexpr (LANES == 4) {
            s = lotz_sum(kT / p, t.sb[Z][j], t.sc[Z][j], rule, (int)(threadIdx.x & 3));
            s += __shfl_xor(s, 1, 64);
            s += __shfl_xor(s, 2, 64);
        } else {
            s = lotz_sum4(kT / p, t.sb[Z][j], t.sc[Z][j], rule);
        }
        double v = t.aq[Z][j] / p * s;
        if (j > 0) v *= exp(-(p - t.P[Z]) / kT);
        acc += v;
    }
    return acc;
}

__device__ inline double vbar_cm_s(double kT) { return C_CM_S * sqrt(8.0 * kT / (M_PI * ME_C2_EV)); }

// The rate from the shells' sum.
__device__ inline double rate_of_shells(double kT, double ne, const IonTables& t, int Z, double shells)
{
    return ne * vbar_cm_s(kT) / kT * exp(-t.P[Z] / kT) * shells;
}

__device__ inline double rate_exact(double kT, double ne, const IonTables& t, int Z, const GlRule& rule)
{
    if (!(kT > 0.0) || !(ne > 0.0)) return 0.0;
    return rate_of_shells(kT, ne, t, Z, lotz_shells(kT, t, Z, rule));
}

// rate_exact of n pairs by a workgroup: get(i, kT, ne, Z) reads pair i, put(i, nu)
// takes its rate.  Four lanes share a pair's nodes, a wave 16 pairs; it sums the
// shells of up to four such groups (its wave's every NW-th) before lane j of each
// four lanes finishes its pair of group j, so that the prefactor's divisions,
// root and exponential, about 110 FP64 operations, serve 64 pairs and not 16.
template <int NT, class Get, class Put>
__device__ inline void rates_of_pairs(int n, const IonTables& t, const GlRule& rule, Get get, Put put)
{
    constexpr int NW = NT / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane & 3;
    for (int g0 = 16 * wave; g0 < n; g0 += 4 * 16 * NW) {
        double mine = 0.0;
#pragma unroll 1
        for (int q = 0; q < 4; ++q) {
            const int i = g0 + 16 * NW * q + (lane >> 2);
            double kT = 0.0, ne = 0.0;
            int Z = 0;
            if (i < n) get(i, kT, ne, Z);
            if (i < n && kT > 0.0 && ne > 0.0) {  // the same in the pair's four lanes
                const double sum = lotz_shells<4>(kT, t, Z, rule);
                if (q == j) mine = sum;
            }
        }
        const int i = g0 + 16 * NW * j + (lane >> 2);
        if (i < n) {
            double kT, ne;
            int Z;
            get(i, kT, ne, Z);
            put(i, kT > 0.0 && ne > 0.0 ? rate_of_shells(kT, ne, t, Z, mine) : 0.0);
        }
    }
}

__device__ inline double ln_rate_exact(double kT, double ne, const IonTables& t, int Z, const GlRule& rule)
{
    if (!(kT > 0.0) || !(ne > 0.0)) return -INFINITY;
    return log(ne * vbar_cm_s(kT) / kT) - t.P[Z] / kT + log(lotz_shells(kT, t, Z, rule));
}

}  // namespace pic
