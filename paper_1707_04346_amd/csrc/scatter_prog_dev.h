// scatter_prog_dev.h -- the scatter program of scatter_prog.h on the device: one
// wave's lanes run their words of a tile.  The LDS addresses are byte offsets: the
// kernels have dynamic LDS only, which starts at 0, and W lies at its start, so that
// the other arrays' places are the instructions' immediate offsets.
#pragma once

#include "bufio.h"
#include "scatter_prog.h"

namespace cis {

// A workgroup barrier with the wave's LDS accesses complete.  The explicit wait is
// needed: at a barrier that a loop's back edge reaches, the compiler (ROCm 7.2)
// dropped the one that __syncthreads implies.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();
}

template <typename T>
__device__ __forceinline__ T lds_ld(uint32_t off) {
    return *reinterpret_cast<const __attribute__((address_space(3))) T *>(off);
}
template <typename T>
__device__ __forceinline__ void lds_st(uint32_t off, T v) {
    *reinterpret_cast<__attribute__((address_space(3))) T *>(off) = v;
}

// first field of round r
template <int PG>
constexpr int prog_field(int r) {
    int x = kProgs[PG].np * kProgs[PG].ps;
    for (int i = 0; i < r; ++i) x += 1 + kProgs[PG].r[i];
    return x;
}

// A lane's words of a tile for the rounds R0 .. R1 - 1 and the partial round before
// them.  The offsets in them count four-byte elements; FP64 doubles them.
template <typename T, int PG, int R0 = 0, int R1 = kProgs[PG].nr>
struct ProgWords {
    static constexpr int NW = kProgs[PG].words();
    uint32_t q[NW];

    // words of the wave's quarter; voff: (quarter * NW * 64 + lane) * 4
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t voff, int tile) {
        const uint32_t so = uint32_t(tile) * uint32_t(kProgWaves * NW * 64 * 4);
#pragma unroll
        for (int i = 0; i < NW; ++i)
            if (2 * i < prog_field<PG>(0) || (2 * i + 1 >= prog_field<PG>(R0) && 2 * i < prog_field<PG>(R1)))
                q[i] = buffer_ld_u32(r, voff + i * 256u, so);
    }
    template <int I>
    __device__ __forceinline__ uint32_t ref() const {
        if constexpr (sizeof(T) == 4) return I & 1 ? (q[I / 2] >> 16) & 0x7fffu : q[I / 2] & 0x7fffu;
        else return (I & 1 ? q[I / 2] >> 15 : q[I / 2] << 1) & 0xfffeu;
    }
    template <int I>
    __device__ __forceinline__ uint32_t slot() const {
        if constexpr (sizeof(T) == 4) return I & 1 ? q[I / 2] >> 16 : q[I / 2] & 0xffffu;
        else return (I & 1 ? q[I / 2] >> 15 : q[I / 2] << 1) & 0x1fffeu;
    }
    // v with the reference's sign: v_bitop3, a ^ (b & c)
    template <int I>
    __device__ __forceinline__ uint32_t flip(uint32_t v) const {
        return __builtin_amdgcn_bitop3_b32(v, I & 1 ? q[I / 2] : q[I / 2] << 16, 0x80000000u, 0x78);
    }
    template <int I>
    __device__ __forceinline__ float sign(float v) const {
        return __uint_as_float(flip<I>(__float_as_uint(v)));
    }
    template <int I>
    __device__ __forceinline__ double sign(double v) const {
        const unsigned long long u = static_cast<unsigned long long>(__double_as_longlong(v));
        return __longlong_as_double(static_cast<long long>(
            (static_cast<unsigned long long>(flip<I>(uint32_t(u >> 32))) << 32) | uint32_t(u)));
    }
};

// N references from field I on: the loads, then the sum
template <int I, int N, typename W, typename T, int V>
__device__ __forceinline__ void prog_load(const W &w, T (&v)[V]) {
    if constexpr (N > 0) {
        v[I] = lds_ld<T>(w.template ref<I>());
        prog_load<I + 1, N - 1>(w, v);
    }
}
template <int I, int N, typename W, typename T, int V>
__device__ __forceinline__ T prog_sum(const W &w, const T (&v)[V]) {
    if constexpr (N == 1) return w.template sign<I>(v[I]);
    else return prog_sum<I, N / 2>(w, v) + prog_sum<I + N / 2, N - N / 2>(w, v);
}
template <int PG, int R, int END, typename W, typename T, int V>
__device__ __forceinline__ void prog_rounds_load(const W &w, T (&v)[V], uint32_t (&slot)[6]) {
    if constexpr (R < END) {
        constexpr int F = prog_field<PG>(R);
        prog_load<F + 1, kProgs[PG].r[R]>(w, v);
        slot[R] = w.template slot<F>();
        prog_rounds_load<PG, R + 1, END>(w, v, slot);
    }
}
template <int PG, int R, int END, typename W, typename T, int V>
__device__ __forceinline__ void prog_rounds_sum(const W &w, const T (&v)[V], T (&sum)[6]) {
    if constexpr (R < END) {
        sum[R] = prog_sum<prog_field<PG>(R) + 1, kProgs[PG].r[R]>(w, v);
        prog_rounds_sum<PG, R + 1, END>(w, v, sum);
    }
}

// Runs the rounds of a tile's words: SC + mine the byte offset of the lane's scratch
// element, SIG that of the sigma row.  The loads go out together, before the sums.
// (Two waves that share a quarter, each with its own rounds, both write the same partial
// sums, each before it reads them.)
template <uint32_t SC, uint32_t SIG, typename T, int PG, int R0, int R1>
__device__ __forceinline__ void prog_run(const ProgWords<T, PG, R0, R1> &w, uint32_t mine) {
    static_assert(kProgs[PG].np == 1, "one partial round");
    if constexpr (R0 < R1) {
        constexpr int PS = kProgs[PG].ps;
        T v[kProgs[PG].fields()], sum[6], old[6];
        uint32_t slot[6];
        prog_load<0, PS>(w, v);
        __builtin_amdgcn_sched_barrier(0);
        lds_st<T>(mine + SC, prog_sum<0, PS>(w, v));
        prog_rounds_load<PG, R0, R1>(w, v, slot);
#pragma unroll
        for (int i = R0; i < R1; ++i) old[i] = lds_ld<T>(slot[i] + SIG);
        __builtin_amdgcn_sched_barrier(0);
        prog_rounds_sum<PG, R0, R1>(w, v, sum);
#pragma unroll
        for (int i = R0; i < R1; ++i) lds_st<T>(slot[i] + SIG, old[i] + sum[i]);
    }
}

}  // namespace cis
