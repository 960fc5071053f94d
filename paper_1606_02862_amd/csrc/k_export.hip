// Particles of one species in id order, for the host: the device side of
// pic_get_particles.
//
// Ids are distinct and mostly dense, so sorting them is ranking them: a bit
// per id in [0, largest id], a prefix sum of the words' bit counts, and the
// rank of an id is its word's prefix plus the bits below its own.  Three
// passes over the ids and one gather of the particles, in chunks of
// EXPORT_CHUNK so that the staging stays bounded; HBM latency of the scattered
// accesses bounds them (0.2 ms for 0.9 M particles, against 70 ms for the sort
// and gather on one host core).  Duplicate ids (which leave a rank free) are
// reported, and the caller sorts on the host instead, as for ids so sparse that
// their bits would outgrow the particles.
#include "pic_device.hpp"

namespace pic {

// {largest id, duplicates seen, particles} of the species
__global__ __launch_bounds__(BLOCK) void k_export_stats(const uint32_t* id, const int32_t* count, int64_t cap,
                                                        unsigned long long* out)
{
    __shared__ unsigned s_max;
    if (threadIdx.x == 0) s_max = 0u;
    __syncthreads();
    const int n = count[blockIdx.x];
    const uint32_t* p = id + (int64_t)blockIdx.x * cap;
    unsigned m = 0;
    for (int t = threadIdx.x; t < n; t += BLOCK) m = p[t] > m ? p[t] : m;
    if (m) atomicMax(&s_max, m);
    __syncthreads();
    if (threadIdx.x == 0 && n) {
        atomicMax(&out[0], (unsigned long long)s_max);
        atomicAdd(&out[2], (unsigned long long)n);
    }
}

__global__ __launch_bounds__(BLOCK) void k_export_mark(const uint32_t* id, const int32_t* count, int64_t cap,
                                                       uint32_t* bits, unsigned long long* stats)
{
    const int n = count[blockIdx.x];
    const uint32_t* p = id + (int64_t)blockIdx.x * cap;
    for (int t = threadIdx.x; t < n; t += BLOCK) {
        const uint32_t v = p[t], b = 1u << (v & 31);
        if (atomicOr(&bits[v >> 5], b) & b) stats[1] = 1ull;
    }
}

// Bits before each word within its block of EXPORT_WORDS words, and per block.
constexpr int EXPORT_WORDS = 4 * BLOCK;
__global__ __launch_bounds__(BLOCK) void k_export_words(const uint32_t* bits, uint32_t* before, uint32_t* block)
{
    __shared__ unsigned wsum[BLOCK / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t w = (int64_t)blockIdx.x * EXPORT_WORDS + 4 * tid;
    const uint4 v = *reinterpret_cast<const uint4*>(bits + w);
    const unsigned c0 = __popc(v.x), c1 = __popc(v.y), c2 = __popc(v.z), sum = c0 + c1 + c2 + __popc(v.w);
    unsigned incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned u = __shfl_up(incl, o, 64);
        if (lane >= o) incl += u;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    unsigned base = incl - sum, total = 0;
#pragma unroll
    for (int k = 0; k < BLOCK / 64; ++k) {
        if (k < wave) base += wsum[k];
        total += wsum[k];
    }
    *reinterpret_cast<uint4*>(before + w) = make_uint4(base, base + c0, base + c0 + c1, base + c0 + c1 + c2);
    if (tid == 0) block[blockIdx.x] = total;
}

// Exclusive prefix sum of the nb block counts, one workgroup.
__global__ __launch_bounds__(BLOCK) void k_export_scan(uint32_t* block, int nb)
{
    __shared__ unsigned wsum[BLOCK / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    unsigned carry = 0;
    for (int b0 = 0; b0 < nb; b0 += BLOCK) {
        const unsigned v = b0 + tid < nb ? block[b0 + tid] : 0u;
        unsigned incl = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned u = __shfl_up(incl, o, 64);
            if (lane >= o) incl += u;
        }
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        unsigned base = carry + incl - v, total = 0;
#pragma unroll
        for (int k = 0; k < BLOCK / 64; ++k) {
            if (k < wave) base += wsum[k];
            total += wsum[k];
        }
        if (b0 + tid < nb) block[b0 + tid] = base;
        carry += total;
        __syncthreads();  // wsum is rewritten
    }
}

// perm[rank] = slot
__global__ __launch_bounds__(BLOCK) void k_export_rank(const uint32_t* id, const int32_t* count, int64_t cap,
                                                       const uint32_t* bits, const uint32_t* before,
                                                       const uint32_t* block, uint32_t* perm)
{
    const int n = count[blockIdx.x];
    const int64_t base = (int64_t)blockIdx.x * cap;
    for (int t = threadIdx.x; t < n; t += BLOCK) {
        const uint32_t v = id[base + t], w = v >> 5;
        const uint32_t r = block[w / EXPORT_WORDS] + before[w] + __popc(bits[w] & ((1u << (v & 31)) - 1u));
        perm[r] = (uint32_t)(base + t);
    }
}

// Particles of ranks [r0, r0 + m) into the staging arrays of o.
template <class R, class U>
__global__ __launch_bounds__(BLOCK) void k_export_gather(GridViewT<R> g, SpeciesViewT<R> s, const uint32_t* perm, int64_t r0,
                                                         int m, ExportT<U> o)
{
    const int i = blockIdx.x * BLOCK + threadIdx.x;
    if (i >= m) return;
    const uint32_t p = perm[r0 + i];
    const int sc = (int)(p / (uint32_t)s.cap);
    const int scx = sc % g.ncx, scy = (sc / g.ncx) % g.ncy, scz = sc / (g.ncx * g.ncy);
    const Triple<R> r = ld3(s.pos, p), u = ld3(s.mom, p);
    o.x[i] = (double)(scx * SX) + (double)r.x;
    o.y[i] = (double)(scy * SY) + (double)r.y;
    o.z[i] = (double)(scz * SZ) + (double)r.z;
    o.ux[i] = (U)u.x;
    o.uy[i] = (U)u.y;
    o.uz[i] = (U)u.z;
    o.w[i] = (U)s.w[p];
    o.id[i] = (int64_t)s.id[p];
    o.zs[i] = s.zs ? (int32_t)s.zs[p] : 0;
}

hipError_t launch_export_stats(const uint32_t* id, const int32_t* count, int nsc, int cap, unsigned long long* out,
                               hipStream_t st)
{
    hipLaunchKernelGGL(k_export_stats, dim3(nsc), dim3(BLOCK), 0, st, id, count, (int64_t)cap, out);
    return hipGetLastError();
}

int64_t export_words(uint32_t id_max)
{
    const int64_t w = (int64_t)(id_max >> 5) + 1;
    return (w + EXPORT_WORDS - 1) / EXPORT_WORDS * EXPORT_WORDS;
}

hipError_t launch_export_rank(const uint32_t* id, const int32_t* count, int nsc, int cap, int64_t words, uint32_t* bits,
                              uint32_t* before, uint32_t* block, uint32_t* perm, unsigned long long* stats, hipStream_t st)
{
    if (words <= 0 || words % EXPORT_WORDS || (int64_t)nsc * cap > 0xFFFFFFFFLL) return hipErrorInvalidValue;
    const int nb = (int)(words / EXPORT_WORDS);
    const hipError_t e = launch_zero_i32((int32_t*)bits, words, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_export_mark, dim3(nsc), dim3(BLOCK), 0, st, id, count, (int64_t)cap, bits, stats);
    hipLaunchKernelGGL(k_export_words, dim3(nb), dim3(BLOCK), 0, st, bits, before, block);
    hipLaunchKernelGGL(k_export_scan, dim3(1), dim3(BLOCK), 0, st, block, nb);
    hipLaunchKernelGGL(k_export_rank, dim3(nsc), dim3(BLOCK), 0, st, id, count, (int64_t)cap, bits, before, block, perm);
    return hipGetLastError();
}

template <class R, class U>
hipError_t launch_export_gather(const GridViewT<R>& g, const SpeciesViewT<R>& s, const uint32_t* perm, int64_t r0, int m,
                                const ExportT<U>& o, hipStream_t st)
{
    if (m <= 0) return hipSuccess;
    hipLaunchKernelGGL((k_export_gather<R, U>), dim3((m + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, st, g, s, perm, r0, m, o);
    return hipGetLastError();
}

#define PIC_EXPORT_INSTANCES(R, U)                                                                                   \
    template hipError_t launch_export_gather<R, U>(const GridViewT<R>&, const SpeciesViewT<R>&, const uint32_t*, int64_t, \
                                                   int, const ExportT<U>&, hipStream_t);
PIC_EXPORT_INSTANCES(float, float)
PIC_EXPORT_INSTANCES(float, double)
PIC_EXPORT_INSTANCES(double, float)
PIC_EXPORT_INSTANCES(double, double)
#undef PIC_EXPORT_INSTANCES

}  // namespace pic
