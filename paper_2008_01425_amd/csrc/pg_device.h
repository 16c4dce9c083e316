// Device code shared by the kernel files: global accesses, wavefront reductions, the Gram factorisation.
#pragma once
#include <hip/hip_runtime.h>
#include <float.h>

#include "pg_desc.h"

namespace pg {

#define PG_GLOBAL __attribute__((address_space(1)))
// Instruction-scheduling fence: nothing is moved across it.
#define PG_FENCE() __builtin_amdgcn_sched_barrier(0)

// V floats moved by one load / store instruction (128, 64 or 32 bits).
template <int V>
struct VecT {
    typedef float T __attribute__((ext_vector_type(V)));
};

// Loads and stores through explicitly global pointers: parameter buffers are reached through a
// pointer table, so the compiler cannot see that they are global and would emit flat accesses.
template <int V>
__device__ __forceinline__ typename VecT<V>::T ldg(const float *p) {
    return *(const PG_GLOBAL typename VecT<V>::T *)p;
}
template <int V>
__device__ __forceinline__ void stg(float *p, typename VecT<V>::T v) {
    *(PG_GLOBAL typename VecT<V>::T *)p = v;
}
// Four consecutive floats in one 16-byte load at any 4-byte aligned address (global memory
// takes under-aligned vector accesses; rows of a matrix with q % 4 != 0 start at such addresses).
typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ void ld4(const float *p, float (&x)[4]) {
    const float4_any t = *(const PG_GLOBAL float4_any *)p;
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = t[v];
}
// The same with the non-temporal hint when NT.  A pass that rewrites parameters too large for the
// 256 MB memory-side cache leaves that cache full of dirty lines, and the pass after it pays for
// their write-back; streamed past the caches the same pass is faster (plain in-place x *= c over
// 1 GiB: 5.4 -> 6.3 TB/s; over 256 MB, where the cache holds everything: 8.5 -> 6.7).
// ANY: V floats at any 4-byte aligned address (V = 4).
template <int V, bool NT, bool ANY = false>
__device__ __forceinline__ typename VecT<V>::T ldgx(const float *p) {
    if constexpr (ANY) {
        const PG_GLOBAL float4_any *pa = (const PG_GLOBAL float4_any *)p;
        if constexpr (NT) return __builtin_nontemporal_load(pa);
        return *pa;
    }
    if constexpr (NT) return __builtin_nontemporal_load((const PG_GLOBAL typename VecT<V>::T *)p);
    return ldg<V>(p);
}
template <int V, bool NT, bool ANY = false>
__device__ __forceinline__ void stgx(float *p, typename VecT<V>::T v) {
    if constexpr (ANY) {
        if constexpr (NT) __builtin_nontemporal_store((float4_any)v, (PG_GLOBAL float4_any *)p);
        else *(PG_GLOBAL float4_any *)p = v;
    } else {
        if constexpr (NT) __builtin_nontemporal_store(v, (PG_GLOBAL typename VecT<V>::T *)p);
        else stg<V>(p, v);
    }
}
__device__ __forceinline__ float ldg1(const float *p) { return *(const PG_GLOBAL float *)p; }
// The same at a byte offset of 32 bits from a base of the whole wavefront.
__device__ __forceinline__ void ld4_at(const float *base, uint32_t byte_off, float (&x)[4]) {
    const float4_any t = *(const PG_GLOBAL float4_any *)((const PG_GLOBAL char *)base + byte_off);
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = t[v];
}
__device__ __forceinline__ float ld1_at(const float *base, uint32_t byte_off) {
    return *(const PG_GLOBAL float *)((const PG_GLOBAL char *)base + byte_off);
}

// Which tile this work-group takes: the tile list in order, or backwards, so that a pass can start
// on the data the previous pass touched last (still resident in the memory-side cache).
__device__ __forceinline__ int tile_index(int ntiles, int reverse) {
    return reverse ? ntiles - 1 - (int)blockIdx.x : (int)blockIdx.x;
}

// ---- wavefront reductions on the DPP / swizzle network --------------------------------
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v) {
    int lo = __double2loint(v), hi = __double2hiint(v);
    // every lane has a valid source lane under these controls, so no `old` value is needed
    lo = __builtin_amdgcn_mov_dpp(lo, CTRL, 0xf, 0xf, false);
    hi = __builtin_amdgcn_mov_dpp(hi, CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double swizzle_xor16(double v) {
    int lo = __double2loint(v), hi = __double2hiint(v);
    lo = __builtin_amdgcn_ds_swizzle(lo, 0x401f);  // bit mode: and 0x1f, or 0, xor 0x10
    hi = __builtin_amdgcn_ds_swizzle(hi, 0x401f);
    return __hiloint2double(hi, lo);
}
// Sum over the `width` (power of two) consecutive lanes that contain this lane; every lane of
// the group receives the sum.  Lane exchanges: quad permutes (1, 2), mirror within 8 and within
// 16 lanes (each lane of a quad / octet already holds that quad's / octet's sum), swizzle across
// 16, and a cross-half shuffle for 64.
__device__ __forceinline__ double group_sum(double v, int width) {
    if (width > 1) v += dpp_mov<0xB1>(v);   // quad_perm [1,0,3,2]
    if (width > 2) v += dpp_mov<0x4E>(v);   // quad_perm [2,3,0,1]
    if (width > 4) v += dpp_mov<0x141>(v);  // row_half_mirror
    if (width > 8) v += dpp_mov<0x140>(v);  // row_mirror
    if (width > 16) v += swizzle_xor16(v);
    if (width > 32) v += __shfl_xor(v, 32);
    return v;
}

// The same for N values at once, exchange step outermost (one branch per step, not per value).
template <int N>
__device__ __forceinline__ void group_sum_all(double (&v)[N], int width) {
    if (width > 1) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += dpp_mov<0xB1>(v[i]);
    }
    if (width > 2) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += dpp_mov<0x4E>(v[i]);
    }
    if (width > 4) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += dpp_mov<0x141>(v[i]);
    }
    if (width > 8) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += dpp_mov<0x140>(v[i]);
    }
    if (width > 16) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += swizzle_xor16(v[i]);
    }
    if (width > 32) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += __shfl_xor(v[i], 32);
    }
}

// a and b, summed over the two halves of the wavefront: a's sums in the lower half's lanes, b's in the upper's
__device__ __forceinline__ double fold32(double a, double b) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
    const u2 hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// the same over neighbouring rows of 16 lanes: a's sums in the even rows, b's in the odd ones
__device__ __forceinline__ double fold16(double a, double b) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
    const u2 hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

// One thread factors G = R^T R with the dropped-column rule (flags null: not stored); everyone waits for it.
template <int RMAX>
__device__ __forceinline__ void gram_factor(int r, const double *G, double (*sR)[RMAX], int *sDrop,
                                            int32_t *__restrict__ flags) {
    if (threadIdx.x == 0) {
        for (int k = 0; k < r; ++k) {
            const double gkk = G[k * (k + 1) / 2 + k];
            double dk = gkk;
            for (int j = 0; j < k; ++j) {
                double rjk = 0.0;
                if (!sDrop[j]) {
                    double t = G[k * (k + 1) / 2 + j];
                    for (int i = 0; i < j; ++i)
                        if (!sDrop[i]) t -= sR[i][j] * sR[i][k];
                    rjk = t / sR[j][j];
                }
                sR[j][k] = rjk;
                dk -= rjk * rjk;
            }
            double floor2 = 1e-10 * gkk;
            if (floor2 < (double)FLT_MIN) floor2 = (double)FLT_MIN;
            const int dropped = !(dk >= floor2);
            sDrop[k] = dropped;
            sR[k][k] = dropped ? 1.0 : sqrt(dk);
            if (flags) flags[k] = dropped;
        }
    }
    __syncthreads();
}

}  // namespace pg
