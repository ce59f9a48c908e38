// slices.h -- the one-block sigma_3 kernels of few alpha strings: the source tiles of a
// sigma row dealt to several workgroups.
//
// A workgroup a row leaves most of the chip idle when there are few rows, and they are
// the longer the fewer they are (16 rows of 403 tiles for 1 alpha and 8 beta electrons in
// 16 orbitals).  Workgroup (Ia, y) then takes the y-th run of the tiles; the first adds to
// the sigma row, the others write their sums to scratch, and one more kernel adds these in
// their order, so that results repeat.  Sigma_3 of 1 alpha and 8 beta electrons in 16
// orbitals: FP32 402 -> 46 us (220 on the general kernel), FP64 692 -> 68 (290); of 2 and 6
// in 13: 52 -> 25, 73 -> 37.
#pragma once

#include "internal.h"

#include <algorithm>

namespace cis {

constexpr int kPlaces32 = 512, kPlaces64 = 256;   // workgroups that the chip holds (FP64: at least)

struct SliceTiles {
    int t0, t1;
    __device__ __forceinline__ explicit SliceTiles(int ntile)
        : t0(int(blockIdx.y) * ntile / int(gridDim.y)), t1((int(blockIdx.y) + 1) * ntile / int(gridDim.y)) {}
};

template <typename T>
__device__ __forceinline__ T *slice_row(T *sp, T *part, int Ia, int Na, int ld) {
    return blockIdx.y == 0 ? sp + int64_t(Ia) * ld : part + (int64_t(blockIdx.y - 1) * Na + Ia) * ld;
}

template <typename T>
__global__ __launch_bounds__(256) void k_add_slices(T *sp, const T *part, int64_t n, int more) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n) return;
    T v = sp[i];
    for (int y = 0; y < more; ++y) v += part[int64_t(y) * n + i];
    sp[i] = v;
}

// Slices of a launch over Na rows of ld columns in ntile tiles: workgroups up to `places`, at least four
// tiles each, and sums that fit the scratch.
inline int slices(int Na, int ntile, int ld, size_t es, size_t part_bytes, int places) {
    const size_t row = size_t(Na) * size_t(ld) * es;
    return std::max(1, std::min({places / Na, ntile / 4, int(std::min<size_t>(part_bytes / row, 4096)) + 1}));
}

template <typename T>
hipError_t add_slices(T *sp, const T *part, int64_t n, int ns, hipStream_t s) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || ns == 1) return e;
    hipLaunchKernelGGL((k_add_slices<T>), dim3(unsigned((n + 255) / 256)), dim3(256), 0, s, sp, part, n, ns - 1);
    return hipGetLastError();
}

}  // namespace cis
