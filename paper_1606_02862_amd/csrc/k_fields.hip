// Yee FDTD update on the periodic staggered grid (Yee 1966), the cycle's
// B(dt/2), E(dt), B(dt/2):
//   B -= coef * curl E   (forward differences of E, at the B locations)
//   E += coef * (curl B - J)   (backward differences of B, at the E locations;
//                               J converted from its fixed-point sums first when kept so)
// Each lane takes four x-consecutive cells (nx is a multiple of the supercell
// width, so a group never straddles a row), x fastest, every component row
// read and written in coalesced 4-element vectors; the x differences take
// scalars from the neighbouring groups (wrapped).
//
// Two forms.  Large grids: three passes in place (k_yee_b, k_yee_e, k_yee_b),
// bound by HBM.  Components of up to FUSE_BYTES, bound by launches (5 us each,
// whatever they do): two kernels,
//   head: B1 = B - curl E dt/2 at the group's cells and, computed again, at the
//         neighbours that curl B1 needs; E1 = E + dt (curl B1 - J); B1 and E1 go
//         to scratch, since neighbours still read E and B.  It also writes J from
//         its accumulators and clears them, so the deposit needs no clearing
//         launch of its own;
//   tail: E = E1, B = B1 - curl E1 dt/2; in a call's last cycle also the
//         migration (pic_migrate.hpp), in workgroups of its own, first in the
//         grid so that the field groups run beside them.
// A cycle with its migration is then 3 launches instead of 6 (one species).
// Measured, passes in place against fused, one cycle (us): FP32 16^3 50.9 / 43,
// 64^3 with 7 particles per cell 81 / 73, 96x64x64 107 / 99, 128x96x64
// 169 / 165, 128^3 with 16 equal, 256x256x128 1 % slower (the fused form moves J
// once more); FP64 64^3 118 / 110, 96x64x64 145 / 144, 128x64x64 199 / 205.
#include <type_traits>

#include "pic_migrate.hpp"

namespace pic {

static_assert(SX % 4 == 0, "rows of whole 4-cell groups");

// Four consecutive values, loaded and stored as one 16-byte (FP32) or
// 32-byte (FP64) vector; the offsets used are multiples of 4 elements.
template <class R>
struct Quad {
    R v[4];
};
template <class R> struct VecOf;
template <> struct VecOf<float> { using T = float4; };
template <> struct VecOf<double> { using T = double4; };

template <class R>
__device__ inline Quad<R> ld4(const R* p)
{
    const typename VecOf<R>::T a = *reinterpret_cast<const typename VecOf<R>::T*>(p);
    return Quad<R>{{a.x, a.y, a.z, a.w}};
}
template <class R>
__device__ inline void st4(R* p, const Quad<R>& q)
{
    typename VecOf<R>::T a;
    a.x = q.v[0]; a.y = q.v[1]; a.z = q.v[2]; a.w = q.v[3];
    *reinterpret_cast<typename VecOf<R>::T*>(p) = a;
}

template <class R>
__global__ __launch_bounds__(BLOCK) void k_yee_b(GridViewT<R> g, R cx, R cy, R cz)
{
    const int N = g.nx * g.ny * g.nz;
    const int c = 4 * (blockIdx.x * BLOCK + threadIdx.x);  // first cell of the group
    if (c >= N) return;
    const int i = c % g.nx, j = (c / g.nx) % g.ny, k = c / (g.nx * g.ny);
    const int ip = (i + 4 == g.nx) ? c - i : c + 4;  // first cell of the next group along x
    const int jp = (j + 1 == g.ny) ? c - j * g.nx : c + g.nx;
    const int kp = (k + 1 == g.nz) ? c - k * g.nx * g.ny : c + g.nx * g.ny;
    const R* Ex = g.E;
    const R* Ey = g.E + N;
    const R* Ez = g.E + 2 * N;
    const Quad<R> ex = ld4(Ex + c), ey = ld4(Ey + c), ez = ld4(Ez + c);
    const Quad<R> ex_j = ld4(Ex + jp), ex_k = ld4(Ex + kp), ey_k = ld4(Ey + kp), ez_j = ld4(Ez + jp);
    const R ey_i[4] = {ey.v[1], ey.v[2], ey.v[3], Ey[ip]};  // E_y, E_z one cell up along x
    const R ez_i[4] = {ez.v[1], ez.v[2], ez.v[3], Ez[ip]};
    Quad<R> bx = ld4(g.B + c), by = ld4(g.B + N + c), bz = ld4(g.B + 2 * N + c);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const R curl_x = cy * (ez_j.v[e] - ez.v[e]) - cz * (ey_k.v[e] - ey.v[e]);
        const R curl_y = cz * (ex_k.v[e] - ex.v[e]) - cx * (ez_i[e] - ez.v[e]);
        const R curl_z = cx * (ey_i[e] - ey.v[e]) - cy * (ex_j.v[e] - ex.v[e]);
        bx.v[e] -= curl_x;
        by.v[e] -= curl_y;
        bz.v[e] -= curl_z;
    }
    st4(g.B + c, bx);
    st4(g.B + N + c, by);
    st4(g.B + 2 * N + c, bz);
}

template <class R>
__global__ __launch_bounds__(BLOCK) void k_yee_e(GridViewT<R> g, R cx, R cy, R cz, R coef)
{
    const int N = g.nx * g.ny * g.nz;
    const int c = 4 * (blockIdx.x * BLOCK + threadIdx.x);
    if (c >= N) return;
    const int i = c % g.nx, j = (c / g.nx) % g.ny, k = c / (g.nx * g.ny);
    const int im = (i == 0) ? c + g.nx - 1 : c - 1;  // the cell before the group along x
    const int jm = (j == 0) ? c + (g.ny - 1) * g.nx : c - g.nx;
    const int km = (k == 0) ? c + (g.nz - 1) * g.nx * g.ny : c - g.nx * g.ny;
    const R* Bx = g.B;
    const R* By = g.B + N;
    const R* Bz = g.B + 2 * N;
    const Quad<R> bx = ld4(Bx + c), by = ld4(By + c), bz = ld4(Bz + c);
    const Quad<R> bx_j = ld4(Bx + jm), bx_k = ld4(Bx + km), by_k = ld4(By + km), bz_j = ld4(Bz + jm);
    const R by_i[4] = {By[im], by.v[0], by.v[1], by.v[2]};  // B_y, B_z one cell down along x
    const R bz_i[4] = {Bz[im], bz.v[0], bz.v[1], bz.v[2]};
    Quad<R> jx, jy, jz;
    if (g.J64) {  // PIC_OPT_DETERMINISTIC_J: J from its fixed-point sums (kept in g.J too)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            jx.v[e] = (R)((double)(long long)g.J64[c + e] * g.jinv64);
            jy.v[e] = (R)((double)(long long)g.J64[N + c + e] * g.jinv64);
            jz.v[e] = (R)((double)(long long)g.J64[2 * N + c + e] * g.jinv64);
        }
        st4(g.J + c, jx);
        st4(g.J + N + c, jy);
        st4(g.J + 2 * N + c, jz);
    } else {
        jx = ld4(g.J + c);
        jy = ld4(g.J + N + c);
        jz = ld4(g.J + 2 * N + c);
    }
    Quad<R> ex = ld4(g.E + c), ey = ld4(g.E + N + c), ez = ld4(g.E + 2 * N + c);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const R curl_x = cy * (bz.v[e] - bz_j.v[e]) - cz * (by.v[e] - by_k.v[e]);
        const R curl_y = cz * (bx.v[e] - bx_k.v[e]) - cx * (bz.v[e] - bz_i[e]);
        const R curl_z = cx * (by.v[e] - by_i[e]) - cy * (bx.v[e] - bx_j.v[e]);
        ex.v[e] += curl_x - coef * jx.v[e];
        ey.v[e] += curl_y - coef * jy.v[e];
        ez.v[e] += curl_z - coef * jz.v[e];
    }
    st4(g.E + c, ex);
    st4(g.E + N + c, ey);
    st4(g.E + 2 * N + c, ez);
}

// ---------------------------------------------------------------- fused
// B1 of one component and cell: b - (ca (da) - cb (db)), a B component's curl E
template <class R>
__device__ inline R half_b(R b, R ca, R a1, R a0, R cb, R b1, R b0)
{
    const R curl = ca * (a1 - a0) - cb * (b1 - b0);
    return b - curl;
}

// Block b of n in an order that gives each of the 8 XCDs (which receive
// blocks round-robin) one contiguous range, so that the neighbour rows and
// planes of its groups are in its own L2.
__device__ inline int xcd_range(int b, int n)
{
    const int per = n >> 3, rest = n & 7, x = b & 7;
    return x * per + (x < rest ? x : rest) + (b >> 3);
}

// hx, hy, hz: dt/2 over the cell sizes; cx, cy, cz: dt over them; coef: dt.
// keep_j: also write J (the call's last cycle).
template <class R>
__global__ __launch_bounds__(BLOCK) void k_yee_head(GridViewT<R> g, FieldScratchT<R> f, R hx, R hy, R hz, R cx, R cy,
                                                    R cz, R coef, bool keep_j)
{
    const int N = g.nx * g.ny * g.nz;
    const int c = 4 * (xcd_range(blockIdx.x, gridDim.x) * BLOCK + threadIdx.x);  // first cell of the group
    if (c >= N) return;
    const int i = c % g.nx, j = (c / g.nx) % g.ny, k = c / (g.nx * g.ny);
    const int ip = (i + 4 == g.nx) ? c - i : c + 4;          // first cell of the next group along x
    const int im = (i == 0) ? c + g.nx - 1 : c - 1;          // the cell before the group
    const int P = g.nx * g.ny;
    const int up_y = (j + 1 == g.ny) ? -j * g.nx : g.nx, dn_y = (j == 0) ? (g.ny - 1) * g.nx : -g.nx;
    const int up_z = (k + 1 == g.nz) ? -k * P : P, dn_z = (k == 0) ? (g.nz - 1) * P : -P;
    const R *Ex = g.E, *Ey = g.E + N, *Ez = g.E + 2 * N, *Bx = g.B, *By = g.B + N, *Bz = g.B + 2 * N;
    // E at the group and at its neighbours: suffix y, z one cell up, _y, _z one down
    const Quad<R> ex = ld4(Ex + c), ey = ld4(Ey + c), ez = ld4(Ez + c);
    const Quad<R> exy = ld4(Ex + c + up_y), ezy = ld4(Ez + c + up_y), exz = ld4(Ex + c + up_z), eyz = ld4(Ey + c + up_z);
    const Quad<R> ex_y = ld4(Ex + c + dn_y), ey_y = ld4(Ey + c + dn_y), ez_y = ld4(Ez + c + dn_y);
    const Quad<R> ex_z = ld4(Ex + c + dn_z), ey_z = ld4(Ey + c + dn_z), ez_z = ld4(Ez + c + dn_z);
    const Quad<R> eyz_y = ld4(Ey + c + dn_y + up_z), ezy_z = ld4(Ez + c + dn_z + up_y);
    const Quad<R> bx = ld4(Bx + c), by = ld4(By + c), bz = ld4(Bz + c);
    const Quad<R> bx_y = ld4(Bx + c + dn_y), bz_y = ld4(Bz + c + dn_y), bx_z = ld4(Bx + c + dn_z), by_z = ld4(By + c + dn_z);
    // the scalars beyond the group's ends along x
    const R eyx = Ey[ip], ezx = Ez[ip], ey_yx = Ey[ip + dn_y], ez_zx = Ez[ip + dn_z];
    const R ex_x = Ex[im], ey_x = Ey[im], ez_x = Ez[im], exz_x = Ex[im + up_z], exy_x = Ex[im + up_y];
    const R by_x = By[im], bz_x = Bz[im];
    Quad<R> jx, jy, jz;
    if (g.J64) {  // PIC_OPT_DETERMINISTIC_J: J from its fixed-point sums
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            jx.v[e] = (R)((double)(long long)g.J64[c + e] * g.jinv64);
            jy.v[e] = (R)((double)(long long)g.J64[N + c + e] * g.jinv64);
            jz.v[e] = (R)((double)(long long)g.J64[2 * N + c + e] * g.jinv64);
            g.J64[c + e] = g.J64[N + c + e] = g.J64[2 * N + c + e] = 0ull;
        }
    } else {
        const Quad<R> zero{};
        jx = ld4(f.Jacc + c);
        jy = ld4(f.Jacc + N + c);
        jz = ld4(f.Jacc + 2 * N + c);
        st4(f.Jacc + c, zero);
        st4(f.Jacc + N + c, zero);
        st4(f.Jacc + 2 * N + c, zero);
    }
    if constexpr (std::is_same<R, float>::value) {
        for (int s = 0; s < f.n_fix; ++s) {  // species deposited in several parts
            ulonglong2* const a = reinterpret_cast<ulonglong2*>(f.fix[s]);
            Quad<R>* const j[3] = {&jx, &jy, &jz};
            ulonglong2 v[3][2];
#pragma unroll
            for (int d = 0; d < 3; ++d)
#pragma unroll
                for (int h = 0; h < 2; ++h) v[d][h] = a[(d * N + c) / 2 + h];
#pragma unroll
            for (int d = 0; d < 3; ++d)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    j[d]->v[2 * h] += (R)((double)(long long)v[d][h].x * f.inv[s]);
                    j[d]->v[2 * h + 1] += (R)((double)(long long)v[d][h].y * f.inv[s]);
                    a[(d * N + c) / 2 + h] = make_ulonglong2(0ull, 0ull);
                }
        }
    }
    if (keep_j) {
        st4(g.J + c, jx);
        st4(g.J + N + c, jy);
        st4(g.J + 2 * N + c, jz);
    }
    Quad<R> b1x, b1y, b1z, e1x, e1y, e1z;
    R b1y_x = half_b(by_x, hz, exz_x, ex_x, hx, ez.v[0], ez_x);  // B1_y, B1_z one cell down along x
    R b1z_x = half_b(bz_x, hx, ey.v[0], ey_x, hy, exy_x, ex_x);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const R ez1 = e < 3 ? ez.v[e + 1] : ezx, ey1 = e < 3 ? ey.v[e + 1] : eyx;  // one cell up along x
        b1x.v[e] = half_b(bx.v[e], hy, ezy.v[e], ez.v[e], hz, eyz.v[e], ey.v[e]);
        b1y.v[e] = half_b(by.v[e], hz, exz.v[e], ex.v[e], hx, ez1, ez.v[e]);
        b1z.v[e] = half_b(bz.v[e], hx, ey1, ey.v[e], hy, exy.v[e], ex.v[e]);
        // B1 one cell down along y and z
        const R ey_y1 = e < 3 ? ey_y.v[e + 1] : ey_yx, ez_z1 = e < 3 ? ez_z.v[e + 1] : ez_zx;
        const R b1x_y = half_b(bx_y.v[e], hy, ez.v[e], ez_y.v[e], hz, eyz_y.v[e], ey_y.v[e]);
        const R b1z_y = half_b(bz_y.v[e], hx, ey_y1, ey_y.v[e], hy, ex.v[e], ex_y.v[e]);
        const R b1x_z = half_b(bx_z.v[e], hy, ezy_z.v[e], ez_z.v[e], hz, ey.v[e], ey_z.v[e]);
        const R b1y_z = half_b(by_z.v[e], hz, ex.v[e], ex_z.v[e], hx, ez_z1, ez_z.v[e]);
        const R curl_x = cy * (b1z.v[e] - b1z_y) - cz * (b1y.v[e] - b1y_z);
        const R curl_y = cz * (b1x.v[e] - b1x_z) - cx * (b1z.v[e] - b1z_x);
        const R curl_z = cx * (b1y.v[e] - b1y_x) - cy * (b1x.v[e] - b1x_y);
        e1x.v[e] = ex.v[e] + (curl_x - coef * jx.v[e]);
        e1y.v[e] = ey.v[e] + (curl_y - coef * jy.v[e]);
        e1z.v[e] = ez.v[e] + (curl_z - coef * jz.v[e]);
        b1y_x = b1y.v[e];
        b1z_x = b1z.v[e];
    }
    st4(f.E + c, e1x);
    st4(f.E + N + c, e1y);
    st4(f.E + 2 * N + c, e1z);
    st4(f.B + c, b1x);
    st4(f.B + N + c, b1y);
    st4(f.B + 2 * N + c, b1z);
}

// Blocks [0, mig.n * nsc) migrate one supercell of one species each; the rest
// update fields.
template <class R>
__global__ __launch_bounds__(BLOCK) void k_yee_tail(GridViewT<R> g, FieldScratchT<R> f, MigrateArgsT<R> mig, R hx, R hy,
                                                    R hz)
{
    extern __shared__ int lds[];
    __shared__ int counters[3];
    const int nmig = mig.n * g.nsc;
    if ((int)blockIdx.x < nmig) {
        const int sp = blockIdx.x / g.nsc;
        const int sc = sc_of_block(blockIdx.x - sp * g.nsc, g.nsc, g.ncx * g.ncy, g.xcd_remap);
        fill_supercell<BLOCK>(g, mig.s[sp], sc, mig.par, lds, counters);
        return;
    }
    const int N = g.nx * g.ny * g.nz;
    const int c = 4 * (xcd_range((int)blockIdx.x - nmig, (int)gridDim.x - nmig) * BLOCK + threadIdx.x);
    if (c >= N) return;
    const int i = c % g.nx, j = (c / g.nx) % g.ny, k = c / (g.nx * g.ny);
    const int ip = (i + 4 == g.nx) ? c - i : c + 4;
    const int jp = (j + 1 == g.ny) ? c - j * g.nx : c + g.nx;
    const int kp = (k + 1 == g.nz) ? c - k * g.nx * g.ny : c + g.nx * g.ny;
    const R *Ex = f.E, *Ey = f.E + N, *Ez = f.E + 2 * N;
    const Quad<R> ex = ld4(Ex + c), ey = ld4(Ey + c), ez = ld4(Ez + c);
    const Quad<R> exy = ld4(Ex + jp), exz = ld4(Ex + kp), eyz = ld4(Ey + kp), ezy = ld4(Ez + jp);
    const R eyx = Ey[ip], ezx = Ez[ip];
    Quad<R> bx = ld4(f.B + c), by = ld4(f.B + N + c), bz = ld4(f.B + 2 * N + c);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const R ez1 = e < 3 ? ez.v[e + 1] : ezx, ey1 = e < 3 ? ey.v[e + 1] : eyx;
        bx.v[e] = half_b(bx.v[e], hy, ezy.v[e], ez.v[e], hz, eyz.v[e], ey.v[e]);
        by.v[e] = half_b(by.v[e], hz, exz.v[e], ex.v[e], hx, ez1, ez.v[e]);
        bz.v[e] = half_b(bz.v[e], hx, ey1, ey.v[e], hy, exy.v[e], ex.v[e]);
    }
    st4(g.E + c, ex);
    st4(g.E + N + c, ey);
    st4(g.E + 2 * N + c, ez);
    st4(g.B + c, bx);
    st4(g.B + N + c, by);
    st4(g.B + 2 * N + c, bz);
}

// dt / dx etc. are rounded to R once on the host side of the launch
template <class R>
hipError_t launch_yee_b(const GridViewT<R>& g, double coef, hipStream_t st)
{
    const int N = g.nx * g.ny * g.nz;
    if (g.nx % 4) return hipErrorInvalidValue;
    const R cf = (R)coef;
    hipLaunchKernelGGL(k_yee_b<R>, dim3((N / 4 + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, st, g, cf / g.dx, cf / g.dy,
                       cf / g.dz);
    return hipGetLastError();
}

template <class R>
hipError_t launch_yee_e(const GridViewT<R>& g, double coef, hipStream_t st)
{
    const int N = g.nx * g.ny * g.nz;
    if (g.nx % 4) return hipErrorInvalidValue;
    const R cf = (R)coef;
    hipLaunchKernelGGL(k_yee_e<R>, dim3((N / 4 + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, st, g, cf / g.dx, cf / g.dy,
                       cf / g.dz, cf);
    return hipGetLastError();
}

template <class R>
hipError_t launch_yee_head(const GridViewT<R>& g, const FieldScratchT<R>& f, double dt, bool keep_j, hipStream_t st)
{
    const int N = g.nx * g.ny * g.nz;
    if (g.nx % 4) return hipErrorInvalidValue;
    const R h = (R)(0.5 * dt), cf = (R)dt;
    hipLaunchKernelGGL(k_yee_head<R>, dim3((N / 4 + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, st, g, f, h / g.dx, h / g.dy,
                       h / g.dz, cf / g.dx, cf / g.dy, cf / g.dz, cf, keep_j);
    return hipGetLastError();
}

template <class R>
hipError_t launch_yee_tail(const GridViewT<R>& g, const FieldScratchT<R>& f, const MigrateArgsT<R>& mig,
                           double dt, hipStream_t st)
{
    const int N = g.nx * g.ny * g.nz;
    if (g.nx % 4 || mig.n < 0 || mig.n > PIC_MAX_SPECIES) return hipErrorInvalidValue;
    size_t lds = 0;
    for (int s = 0; s < mig.n; ++s) {
        const size_t need = (size_t)3 * mig.s[s].cap_in * sizeof(int) +
                            ((size_t)mig.s[s].cap_in + 31) / 32 * sizeof(unsigned);
        lds = need > lds ? need : lds;
    }
    const int64_t blocks = (int64_t)mig.n * g.nsc + (N / 4 + BLOCK - 1) / BLOCK;
    const R h = (R)(0.5 * dt);
    hipLaunchKernelGGL(k_yee_tail<R>, dim3((unsigned)blocks), dim3(BLOCK), lds, st, g, f, mig, h / g.dx, h / g.dy,
                       h / g.dz);
    return hipGetLastError();
}

#define PIC_FIELD_INSTANCES(R)                                                                                       \
    template hipError_t launch_yee_b<R>(const GridViewT<R>&, double, hipStream_t);                                   \
    template hipError_t launch_yee_e<R>(const GridViewT<R>&, double, hipStream_t);                                   \
    template hipError_t launch_yee_head<R>(const GridViewT<R>&, const FieldScratchT<R>&, double, bool, hipStream_t); \
    template hipError_t launch_yee_tail<R>(const GridViewT<R>&, const FieldScratchT<R>&, const MigrateArgsT<R>&,     \
                                           double, hipStream_t);
PIC_FIELD_INSTANCES(float)
PIC_FIELD_INSTANCES(double)
#undef PIC_FIELD_INSTANCES

}  // namespace pic
