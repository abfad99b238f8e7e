// grmhd_cell.h -- device functions shared by the kernels that update cells.
#pragma once

#include "grmhd_device.h"
#include "grmhd_internal.h"

namespace grmhd {

// The value of the lane to the left / right (wave-wide shift; the first / last
// lane gets an unspecified one).
__device__ __forceinline__ double from_left(double x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x138, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x138, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double from_right(double x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x130, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x130, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// Memory accesses with a uniform 64-bit base, a 32-bit byte offset per lane and a
// uniform one: the address arithmetic stays in the scalar unit.  NT: streaming.
typedef unsigned uint2v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_at(const double* base)
{
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0xffffffffu, 0x00027000);
}

template <bool NT = false>
__device__ __forceinline__ double buf_load(const double* base, unsigned lane, unsigned uniform = 0)
{
    return __builtin_bit_cast(double,
                              __builtin_amdgcn_raw_buffer_load_b64(buffer_at(base), lane, uniform, NT ? 2 : 0));
}

template <bool NT = false>
__device__ __forceinline__ void buf_store(double* base, unsigned lane, double x)
{
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uint2v, x), buffer_at(base), lane, 0, NT ? 2 : 0);
}

// The kernel's arguments (one struct S), loaded anew: a plane's work uses more
// uniform values than there are scalar registers, and values kept from the
// kernel's start would live in vector registers' lanes, one vector instruction a
// read.
template <class S>
__device__ __forceinline__ S kernel_args()
{
    auto p = (const __attribute__((address_space(4))) S*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    S k;
    __builtin_memcpy(&k, p, sizeof k);
    return k;
}

__device__ __forceinline__ long long cache_index(const Dev& d, int i, int j, int k)
{
    return ((long long)(k + d.g[2]) * d.py + (j + d.g[1])) * d.px + (i + d.g[0]);
}

// Store the primitives of cell (i, j, k) at cache position pc, and at the
// ghost positions whose boundary rule copies this cell, so that the cache
// leaves the kernel with its ghost slabs filled (only the face slabs are
// ghosts: every stencil is 1D).  Periodic: the cell is the image of ghost
// idx + n when idx < g and of ghost idx - n when idx >= n - g.  Outflow
// (zero gradient): the first and last cells fill both ghost layers beside
// them.  Active axes have n >= g, so these are all the images.
template <typename T>
__device__ __forceinline__ void store_prim(const Dev& d, T* __restrict__ P, long long pc, int i, int j,
                                           int k, const double* p)
{
#pragma unroll
    for (int v = 0; v < 9; ++v)
        P[v * d.sv + pc] = (T)p[v];
    const int idx[3] = {i, j, k};
    const long long stride[3] = {1, d.px, (long long)d.px * d.py};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (!d.act[a])
            continue;
        const int n = d.n[a], g = d.g[a];
        const long long st = stride[a];
        if (d.bc[a] == 0) {
            if (idx[a] < g) {
#pragma unroll
                for (int v = 0; v < 9; ++v)
                    P[v * d.sv + pc + n * st] = (T)p[v];
            }
            if (idx[a] >= n - g) {
#pragma unroll
                for (int v = 0; v < 9; ++v)
                    P[v * d.sv + pc - n * st] = (T)p[v];
            }
        } else if (idx[a] == 0 || idx[a] == n - 1) {
            const long long s1 = idx[a] == 0 ? -st : st;
            for (int e = 1; e <= g; ++e)
#pragma unroll
                for (int v = 0; v < 9; ++v)
                    P[v * d.sv + pc + e * s1] = (T)p[v];
        }
    }
}

// Per-thread counts reduced over the wave, one atomic per wave and counter
// into the block's slot (never a returning atomic: waiting on one would also
// wait for the wave's outstanding stores).
__device__ __forceinline__ void count_sums(unsigned long long* cnt_base, int nf, int na, int np,
                                           int nb, int itmax)
{
    unsigned long long* cnt = cnt_base + (size_t)(blockIdx.x % CNT_SLOTS) * CNT_WORDS;
    for (int o = 32; o > 0; o >>= 1) {
        nf += __shfl_xor(nf, o);
        na += __shfl_xor(na, o);
        np += __shfl_xor(np, o);
        nb += __shfl_xor(nb, o);
        itmax = max(itmax, __shfl_xor(itmax, o));
    }
    unsigned long long act = __ballot(1);
    if (__lane_id() == __ffsll((long long)act) - 1) {
        if (nf)
            atomicAdd(&cnt[CNT_FAIL], (unsigned long long)nf);
        if (na)
            atomicAdd(&cnt[CNT_ATM], (unsigned long long)na);
        if (np)
            atomicAdd(&cnt[CNT_PFLOOR], (unsigned long long)np);
        if (nb)
            atomicAdd(&cnt[CNT_FALLBACK], (unsigned long long)nb);
        atomicMax(&cnt[CNT_MAXIT], (unsigned long long)itmax);
    }
}

__device__ __forceinline__ void tally(int flags, int iters, int& nf, int& na, int& np, int& nb, int& itmax)
{
    nf += (flags & FLAG_FAIL) != 0;
    na += (flags & FLAG_ATM) != 0;
    np += (flags & FLAG_PFLOOR) != 0;
    nb += (flags & FLAG_FALLBACK) != 0;
    itmax = max(itmax, iters);
}

}  // namespace grmhd
