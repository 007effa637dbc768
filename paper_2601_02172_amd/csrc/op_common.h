// Device helpers shared by the operator kernels.
#pragma once

#include <type_traits>

#include "element.h"

namespace xfft {

__device__ __forceinline__ int wrapi(int a, int n) { return a < 0 ? a + n : (a >= n ? a - n : a); }

// Position of value k (0..23: corner k / 3, component k % 3) of irregular voxel q
// in one half of the corner-force buffer: the 24 values of a voxel are
// contiguous.  The irregular kernels write the values of a run of voxels as one
// stream; a reader takes a whole voxel as six 4-vectors or a corner as three
// adjacent values, from one or two cache lines.
__device__ __forceinline__ uint32_t cut_index(uint32_t q, int k) { return q * 24u + (uint32_t)k; }

// base[i] with a 32-bit byte offset (uniform base pointer + 32-bit lane offset)
template <typename P> __device__ __forceinline__ P &elem(P *base, uint32_t i) {
    using B = typename std::conditional<std::is_const<P>::value, const char, char>::type;
    return *reinterpret_cast<P *>(reinterpret_cast<B *>(base) + (uint32_t)(i * (uint32_t)sizeof(P)));
}

template <typename T>
__device__ __forceinline__ Sym<T> load_ebar(const double *e) {
    T m[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) m[q] = (T)e[q];
    return from_mandel<T>(m);
}

template <typename T>
__device__ __forceinline__ void add_sym(double (&acc)[7], const Sym<T> &s) {
    acc[1] += (double)s.xx; acc[2] += (double)s.yy; acc[3] += (double)s.zz;
    acc[4] += (double)s.yz; acc[5] += (double)s.xz; acc[6] += (double)s.xy;
}

template <typename T>
__device__ __forceinline__ void store_vstress(double *vs, int64_t N, int64_t v, const Sym<T> &s) {
    const double r2 = 1.41421356237309504880;
    vs[0 * N + v] = (double)s.xx; vs[1 * N + v] = (double)s.yy; vs[2 * N + v] = (double)s.zz;
    vs[3 * N + v] = r2 * (double)s.yz; vs[4 * N + v] = r2 * (double)s.xz; vs[5 * N + v] = r2 * (double)s.xy;
}

}  // namespace xfft
