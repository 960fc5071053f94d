// Internal structures of the gfx950 particle-in-cell library: device views
// passed to kernels by value, and the launchers each kernel file provides.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/pic.h"

namespace pic {

// Supercell: 8 x 8 x 4 = 256 cells, one 256-lane workgroup (4 wave64) each,
// as in the paper's block-per-supercell mapping.  A frame is 256 slots.
constexpr int SX = PIC_SUPERCELL_X, SY = PIC_SUPERCELL_Y, SZ = PIC_SUPERCELL_Z;
constexpr int SC_CELLS = SX * SY * SZ;
constexpr int BLOCK = 256;
constexpr int MAX_MIGRATE = 4096;  // per supercell, per species, per step

// Largest float below a power of two s (the far face of a supercell).
__host__ __device__ constexpr float below(float s) { return s - s * 0x1p-24f; }
constexpr float XMAX = below((float)SX), YMAX = below((float)SY), ZMAX = below((float)SZ);

// Device error flags (int32 each).
enum Flag { FLAG_CAPACITY = 0, FLAG_MIGRATE = 1, FLAG_CFL = 2, FLAG_NONFINITE = 3, NFLAGS = 4 };

// Views are templated on the real type R of particles, fields and currents:
// float (the default path) or double (the FP64 variant of the PIC cycle).
template <class R> struct Vec4;
template <> struct Vec4<float> { using type = float4; };
template <> struct Vec4<double> { using type = double4; };

template <class R>
struct GridViewT {
    int nx, ny, nz;        // cells
    int ncx, ncy, ncz;     // supercells per axis
    int nsc;               // number of supercells
    int xcd_remap;         // block -> supercell order (sc_of_block): 0 identity, L >= 1 XCD slabs of L z-layers
    R dx, dy, dz, dt;
    R b0x, b0y, b0z;
    R* E;                  // 3 * N, component-major, x fastest
    R* B;
    R* J;
    int32_t* flags;        // NFLAGS, in pinned host memory (kernels store to it on an error only)
    typename Vec4<R>::type* qbuf;  // deposit queue (one per species of a launch): nsc * qcap records of 2 (x0,y0,z0,qw | x1,y1,z1,-)
    int qcap;              // queue slots per supercell (>= every species' frame capacity, in whole frames of a part)
    // PIC_OPT_DETERMINISTIC_J (FP32): 3 * N int64 fixed-point current at the
    // cycle's common scale, which the field update converts (times jinv64) into
    // J and clears; nullptr otherwise
    unsigned long long* J64;
    double jinv64;
};

template <class R>
struct SpeciesViewT {
    // Positions and momenta as triples (element 3 p + d of slot p): one access
    // of 3 values moves a particle's position, at the stream's full rate when
    // the lanes take consecutive slots, and a migrating particle touches 2
    // lines instead of 6.
    R* pos;                 // supercell-relative, in cells: [0,8)x[0,8)x[0,4)
    R* mom;                 // u = gamma v
    R* w;                   // macro weight
    uint32_t* id;
    uint8_t* zs;            // charge state, or nullptr
    int32_t* count;         // particles per supercell
    int cap;                // slots per supercell (multiple of 256)
    // arrival lists: per step parity and destination supercell, cap_in slots of
    // two records {x, y, z, w}, {ux, uy, uz, id (its bits)}
    typename Vec4<R>::type* in;
    uint8_t* izs;
    int32_t* in_count;      // arrivals per parity and supercell (2 * nsc)
    int32_t* holes;         // per source supercell: vacated slots
    int32_t* hole_count;
    int32_t* left;          // per part of a supercell: its leavers' slots (cap_in each), or nullptr
    int parts;              // parts `left` has room for
    int cap_in;
    R charge;               // in e (per unit Z when zs != nullptr)
    R mass;
};

using GridView = GridViewT<float>;
using SpeciesView = SpeciesViewT<float>;
using GridView64 = GridViewT<double>;
using SpeciesView64 = SpeciesViewT<double>;

// Largest value below the far face of a supercell of extent s in type R.
template <class R> __host__ __device__ constexpr R face_below(R s);
template <> __host__ __device__ constexpr float face_below<float>(float s) { return s - s * 0x1p-24f; }
template <> __host__ __device__ constexpr double face_below<double>(double s) { return s - s * 0x1p-53; }

struct Species {
    SpeciesView v;         // FP32 frames (the default path)
    SpeciesView64 v64;     // FP64 frames (the FP64 variant)
    pic_species_t desc;
    int64_t n_init;        // particles at t = 0
    int64_t id_offset;     // first id at t = 0
    double weight;
    double wmax;           // bound of |w| that sets the fixed-point current scale (>= wheld)
    double wheld;          // largest |w| known to be held (init, set, ionisation electrons)
    unsigned long long* jfix;  // 3 * N fixed-point current, FP32 species of several parts (PushItemT), or nullptr
};

// Map a workgroup index to a supercell so that the 8 XCDs (which receive
// workgroups round-robin) each work on one contiguous slab of nsc/8
// supercells and share its guard cells in their own L2.  remap = 0: the
// identity; remap = L >= 1: the slab is L whole z-layers of nxy = ncx*ncy
// supercells (L = 1 also stands for a slab that is not), and within it the
// blocks walk z fastest, so that the neighbours of a supercell along every
// axis, not only x and y, run at about the same time.
__host__ __device__ inline int sc_of_block(int b, int nsc, int nxy, int remap)
{
    if (!remap) return b;
    const int per = nsc >> 3, i = b >> 3;
    return (b & 7) * per + (i % remap) * nxy + i / remap;
}

// ---------------------------------------------------------------- launchers
// The PIC-cycle launchers exist for R = float and R = double.
template <class R>
hipError_t launch_init_species(const GridViewT<R>& g, const SpeciesViewT<R>& s, uint64_t seed, int species_index,
                               int ppc, int64_t id_offset, int pos_index, int pos_ppc, int64_t pos_id_offset,
                               double u_th, const double drift_u[3], int layout, double weight, int z_init,
                               hipStream_t st);
hipError_t launch_zero_f32(float* p, int64_t n, hipStream_t st);
hipError_t launch_zero_f64(double* p, int64_t n, hipStream_t st);
hipError_t launch_zero_i32(int32_t* p, int64_t n, hipStream_t st);
inline hipError_t launch_zero_r(float* p, int64_t n, hipStream_t st) { return launch_zero_f32(p, n, st); }
inline hipError_t launch_zero_r(double* p, int64_t n, hipStream_t st) { return launch_zero_f64(p, n, st); }
// The species of one particle-kernel launch: one, or with parts > 0 (the split
// variant) several that agree in having charge states or not.
// vmax: upper bound of |q w| max(dx,dy,dz) / (dV dt) over the species' particles
// parts: 0 for one workgroup per supercell; else the workgroups of SPLIT_NT
// lanes that share one (the arrivals then absorbed before the launch, apar = -1)
// apar: parity of the arrivals to absorb first (-1: none); wpar: parity the
// leavers of this step are written to
// galerkin: the reduced-order gather along staggered axes (PIC_GATHER_GALERKIN)
// jscale_g: with g.J64, the cycle's common fixed-point scale (2^30 over the
// largest vmax of the cycle's species); each tile is rescaled to it at the flush
// jfix: FP32 without g.J64, parts > 1: 3 * N fixed-point sums at the species' own
// scale (shared by species of one scale) that its tiles are added to instead of
// g.J.  A supercell's current is then one exact integer sum whatever the number
// of its parts; FP32 additions of partial tiles would round each of them.  The
// 64-bit atomics cost 2 to 5 % of a cycle (four cycles of two TSC species on 64
// supercells 230 us, 217 with FP32 ones, 590 with one workgroup per supercell).
template <class R>
struct PushItemT {
    const SpeciesViewT<R>* s;
    double vmax;
    int parts;
    unsigned long long* jfix;
};
template <class R>
hipError_t launch_push(const GridViewT<R>& g, const PushItemT<R>* items, int n, int order, bool galerkin,
                       float jscale_g, int apar, int wpar, hipStream_t st);
// The same as the kernel takes it: the fixed-point scales, and each species' first block.
template <class R>
struct PushSpeciesT {
    SpeciesViewT<R> s;
    R jscale, jinv;
    double jratio;
    unsigned long long* jfix;
    int parts, first;
};
template <class R>
struct PushArgsT {
    PushSpeciesT<R> sp[PIC_MAX_SPECIES];
    int n;
};
constexpr int SPLIT_NT = 512;
// Queue slots a part needs: its share of a full slab, in whole frames.
inline int split_region(int cap, int parts)
{
    const int per = SPLIT_NT * parts;
    return (cap + per - 1) / per * SPLIT_NT;
}
// The parts of a supercell of a species with about n particles per supercell
// (one of nsp that share a launch), 0 for the default variant.  Up to 512
// supercells: the number that makes the fullest CU's work least, its workgroups
// (of 256 CUs) times the frames of each plus 3 for the staging, clearing and
// flush of a tile (fitted to the figures below).  One part is the default's
// work on 512 lanes, better than its 256 for CIC, or for species that share a
// launch.  Measured, two cycles with 16 particles per cell (default
// against 1, 2, 4, 8 parts; us):
//   TSC  16 supercells 155 / 74 (8), 125: 164 / 126 (2), 130 (4), 152 (8),
//        256: 176 / 178 (1), 203 (4), 384: 275 / 279 (1), 240 (2), 640: 374 / 384 (1);
//   CIC  64 supercells 97 / 64 (4), 70 (8), 256: 107 / 96 (1), 640: 165 / 176 (1);
// with 4 per cell TSC 384: 118 / 118 (1), 136 (2).
inline int split_parts(int nsc, int n, int order, int nsp)
{
    constexpr int CUS = 256, TILE = 3;
    if (nsc > 2 * CUS) return 0;
    const int frames = n > SPLIT_NT ? (n + SPLIT_NT - 1) / SPLIT_NT : 1;
    int best = 1;
    int64_t least = INT64_MAX;
    for (int p = 1; p <= frames && (int64_t)nsc * p <= 4 * CUS; ++p) {
        const int64_t cost = ((int64_t)nsc * nsp * p + CUS - 1) / CUS * (TILE + (frames + p - 1) / p);
        if (cost < least) { least = cost; best = p; }
    }
    return best == 1 && order > 1 && nsp == 1 ? 0 : best;
}
// Fixed-point scale of a current tile: 2^30 over the bound vmax of one contribution.
inline float fixed_scale(double vmax)
{
    const float vf = (float)vmax;
    return vf > 0.0f ? 1073741824.0f / vf : 1.0f;
}
template <class R>
hipError_t launch_migrate(const GridViewT<R>& g, const SpeciesViewT<R>& s, int par, hipStream_t st);
template <class R>
hipError_t launch_yee_b(const GridViewT<R>& g, double coef, hipStream_t st);
template <class R>
hipError_t launch_yee_e(const GridViewT<R>& g, double coef, hipStream_t st);
// The fused field update (k_fields.hip), for grids whose field components take up to FUSE_BYTES each.
// Scratch of 3 * N values each: the fields between its two kernels, and the
// current accumulators the deposit adds to, zero between cycles (unused with
// g.J64, whose sums are cleared the same way): Jacc, and n_fix arrays of
// fixed-point sums (PushItemT), each of which times its inv is rounded to FP32 once.
constexpr int64_t FUSE_BYTES = 3 << 20;
template <class R>
struct FieldScratchT {
    R *E, *B, *Jacc;
    unsigned long long* fix[PIC_MAX_SPECIES];
    double inv[PIC_MAX_SPECIES];
    int n_fix;
};
// Species whose arrivals of parity par the tail's first workgroups absorb.
template <class R>
struct MigrateArgsT {
    SpeciesViewT<R> s[PIC_MAX_SPECIES];
    int n, par;
};
// keep_j: write J as well as use it
template <class R>
hipError_t launch_yee_head(const GridViewT<R>& g, const FieldScratchT<R>& f, double dt, bool keep_j, hipStream_t st);
template <class R>
hipError_t launch_yee_tail(const GridViewT<R>& g, const FieldScratchT<R>& f, const MigrateArgsT<R>& mig,
                           double dt, hipStream_t st);

// Particles in id order for the host (k_export.hip).  stats: {largest id,
// duplicate ids seen, particles}, zero before the call.
template <class U>
struct ExportT {
    double *x, *y, *z;
    int64_t* id;
    U *ux, *uy, *uz, *w;
    int32_t* zs;
};
constexpr int EXPORT_CHUNK = 1 << 21;  // particles staged at a time
hipError_t launch_export_stats(const uint32_t* id, const int32_t* count, int nsc, int cap, unsigned long long* stats,
                               hipStream_t st);
int64_t export_words(uint32_t id_max);  // words of the id bits
hipError_t launch_export_rank(const uint32_t* id, const int32_t* count, int nsc, int cap, int64_t words, uint32_t* bits,
                              uint32_t* before, uint32_t* block, uint32_t* perm, unsigned long long* stats, hipStream_t st);
template <class R, class U>
hipError_t launch_export_gather(const GridViewT<R>& g, const SpeciesViewT<R>& s, const uint32_t* perm, int64_t r0, int m,
                                const ExportT<U>& o, hipStream_t st);

// FP64 diagnostics.  partial buffers hold one entry per workgroup.
struct DiagBuffers {
    double* rho;       // N
    double* g0;        // N, Gauss reference
    double* partial;   // scratch for block partial sums / maxima
    int npartial;
    double* rho_prev;  // N, rho before the last cycle (PIC_OPT_CONTINUITY), or nullptr
    double* result;    // small device result vector
};
template <class R>
hipError_t launch_field_energy(const GridViewT<R>& g, const DiagBuffers& d, hipStream_t st);
template <class R>
hipError_t launch_kinetic(const GridViewT<R>& g, const SpeciesViewT<R>& s, const DiagBuffers& d, int slot,
                          hipStream_t st);
template <class R>
hipError_t launch_rho_deposit(const GridViewT<R>& g, const SpeciesViewT<R>& s, int order, double* rho,
                              hipStream_t st);
// mode 0: record G0; mode 1: the reductions, plus the continuity residual
// against d.rho_prev when cont is set
template <class R>
hipError_t launch_gauss(const GridViewT<R>& g, const DiagBuffers& d, double rho_bg, int mode, bool cont, hipStream_t st);

// Result vector layout of the diagnostics.
enum DiagSlot {
    D_WE = 0, D_WB = 1, D_NONFINITE = 2, D_CHARGE = 3, D_RHOMAX = 4, D_GAUSS = 5, D_DIVB = 6,
    D_KIN0 = 8,  // + species index
    D_CONT = 12, D_JMAX = 13,
    D_NSLOTS = 16
};

}  // namespace pic
