// xfer.hip — conversions between the boundary particle layout (linear cell index) and the
// packed cell code used inside the library.
#include "pic_internal.h"

namespace pic {

// All arrays of a species in one launch, four consecutive particles a thread and round: bound by
// memory (a copy per array was five to nine launches, on small boxes 4 us each).  A species' arrays
// start at 16-byte boundaries; a row of a dense array of n particles (off, u, dr) may start at any
// 4-byte one, and its 16-byte accesses carry that alignment.
template <class T>
struct Vec4 {
    typedef T type __attribute__((ext_vector_type(4), aligned(4)));
};
template <class T>
__device__ inline void copy4(T* dst, const T* src, int64_t i, int m)
{
    using V = typename Vec4<T>::type;
    if (m == 4)
        *reinterpret_cast<V*>(dst + i) = *reinterpret_cast<const V*>(src + i);
    else
        for (int k = 0; k < m; k++) dst[i + k] = src[i + k];
}
template <class T>
__device__ inline void load4(T v[4], const T* src, int64_t i, int m)
{
    using V = typename Vec4<T>::type;
    if (m == 4) {
        const V q = *reinterpret_cast<const V*>(src + i);
#pragma unroll
        for (int k = 0; k < 4; k++) v[k] = q[k];
    } else {
        for (int k = 0; k < m; k++) v[k] = src[i + k];
    }
}
template <class T>
__device__ inline void store4(T* dst, const T v[4], int64_t i, int m)
{
    using V = typename Vec4<T>::type;
    if (m == 4)
        *reinterpret_cast<V*>(dst + i) = V{v[0], v[1], v[2], v[3]};
    else
        for (int k = 0; k < m; k++) dst[i + k] = v[k];
}

__global__ __launch_bounds__(kBlock) void particles_in_kernel(Particles to, int64_t n, const int32_t* cell, const float* off,
                                                              const float* u, const uint32_t* id, const float* dr, int dim,
                                                              GridDev G, CellCode cc, int32_t* n_live, uint32_t* err)
{
    const int64_t first = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (first == 0) *n_live = (int32_t)n;
    const int64_t ncell = (int64_t)G.n[0] * G.n[1] * G.n[2];
    const float zero[4] = {0.f, 0.f, 0.f, 0.f};
    for (int64_t i = 4 * first; i < n; i += (int64_t)gridDim.x * kBlock * 4) {
        const int m = n - i < 4 ? (int)(n - i) : 4;
        int32_t c[4] = {};
        load4(c, cell, i, m);
#pragma unroll
        for (int k = 0; k < 4; k++) {
            if (k < m && (c[k] < 0 || (int64_t)c[k] >= ncell)) {
                c[k] = 0;
                atomicOr(err, 8u);
            }
            const uint32_t r = G.div0.div((uint32_t)c[k]), z = G.div1.div(r);
            c[k] = cc.encode((int)((uint32_t)c[k] - r * (uint32_t)G.n[0]), (int)(r - z * (uint32_t)G.n[1]), (int)z);
        }
        store4(to.cell, c, i, m);
#pragma unroll
        for (int d = 0; d < 3; d++) {
            if (d < dim) copy4(to.off[d], off + d * n, i, m);
            copy4(to.u[d], u + d * n, i, m);
            if (to.dr[d]) {
                if (dr)
                    copy4(to.dr[d], dr + d * n, i, m);
                else
                    store4(to.dr[d], zero, i, m);
            }
        }
        if (to.id) {
            uint32_t q[4] = {(uint32_t)i, (uint32_t)i + 1u, (uint32_t)i + 2u, (uint32_t)i + 3u};
            if (id) load4(q, id, i, m);
            store4(to.id, q, i, m);
        }
    }
}

__global__ __launch_bounds__(kBlock) void particles_out_kernel(Particles from, const int32_t* n_live, int32_t* cell, float* off,
                                                               float* u, uint32_t* id, float* dr, int dim, int ndr,
                                                               GridDev G, CellCode cc)
{
    const int64_t n = *n_live;
    const float zero[4] = {0.f, 0.f, 0.f, 0.f};
    for (int64_t i = 4 * ((int64_t)blockIdx.x * kBlock + threadIdx.x); i < n; i += (int64_t)gridDim.x * kBlock * 4) {
        const int m = n - i < 4 ? (int)(n - i) : 4;
        if (cell) {
            int32_t c[4] = {};
            load4(c, from.cell, i, m);
#pragma unroll
            for (int k = 0; k < 4; k++) {
                int x, y, z;
                cc.decode(c[k], x, y, z);
                c[k] = c[k] < 0 ? -1 : x + G.n[0] * (y + G.n[1] * z);
            }
            store4(cell, c, i, m);
        }
#pragma unroll
        for (int d = 0; d < 3; d++) {
            if (off && d < dim) copy4(off + d * n, from.off[d], i, m);
            if (u) copy4(u + d * n, from.u[d], i, m);
            if (dr) {
                if (d < ndr)
                    copy4(dr + d * n, from.dr[d], i, m);
                else
                    store4(dr + d * n, zero, i, m);
            }
        }
        if (id) copy4(id, from.id, i, m);
    }
}

// Plain streaming copy in 16-byte words (the reference kernel of known traffic used to scale
// hardware memory counters).
__global__ __launch_bounds__(kBlock) void copy_kernel(uint4* __restrict__ dst,
                                                      const uint4* __restrict__ src, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

static inline unsigned capped(int64_t n)
{
    const int64_t want = (n + 4 * kBlock - 1) / (4 * kBlock);
    return (unsigned)(want < 1 ? 1 : (want < 8192 ? want : 8192));
}

hipError_t particles_in(const Particles& to, int64_t n, const int32_t* cell, const float* off, const float* u,
                        const uint32_t* id, const float* dr, int dim, const GridDev& G, CellCode cc, int32_t* n_live,
                        uint32_t* err, hipStream_t st)
{
    particles_in_kernel<<<capped(n), kBlock, 0, st>>>(to, n, cell, off, u, id, dr, dim, G, cc, n_live, err);
    return hipGetLastError();
}

hipError_t particles_out(const Particles& from, const int32_t* n_live, int64_t n_upper, int32_t* cell, float* off,
                         float* u, uint32_t* id, float* dr, int dim, int ndr, const GridDev& G, CellCode cc,
                         hipStream_t st)
{
    particles_out_kernel<<<capped(n_upper), kBlock, 0, st>>>(from, n_live, cell, off, u, id, dr, dim, ndr, G, cc);
    return hipGetLastError();
}

hipError_t device_copy16(void* dst, const void* src, int64_t nwords, hipStream_t st)
{
    if (nwords > 0) {
        const int64_t want = (nwords + kBlock - 1) / kBlock;
        const unsigned grid = (unsigned)(want < 256 * 64 ? want : 256 * 64);
        copy_kernel<<<grid, kBlock, 0, st>>>(static_cast<uint4*>(dst), static_cast<const uint4*>(src),
                                             nwords);
    }
    return hipGetLastError();
}

}  // namespace pic
