// Device helpers shared by the recurrence kernels (sq_kernels.hip,
// sq_tile_kernels.hip): integer and buffer access, wave sums, the node source
// of a launch and the extremes of a Lanczos tridiagonal.
#pragma once

#include <hip/hip_runtime.h>

#include "sq_internal.h"

#include <math.h>

namespace sq {
namespace {

__device__ __forceinline__ int floor_div(int a, int b) {
    int q = a / b;
    return (a % b != 0 && ((a < 0) != (b < 0))) ? q - 1 : q;
}
__device__ __forceinline__ int ceil_div(int a, int b) { return -floor_div(-a, b); }
__device__ __forceinline__ int pmod(int a, int n) {
    int r = a % n;
    return r < 0 ? r + n : r;
}

constexpr unsigned kIdleOffset = 0x7FFFFF00u;  // beyond every buffer: loads read 0, stores drop

// Raw buffer access: SGPR descriptor + one VGPR byte offset + SGPR byte offset,
// so that per-plane addresses stay scalar.  Out-of-range offsets read 0 and
// drop stores (used for idle columns).
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *p, long long bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes, 0x00020000);
}
template <typename T>
__device__ __forceinline__ T bload(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff);
template <>
__device__ __forceinline__ double bload<double>(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
template <>
__device__ __forceinline__ float bload<float>(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
__device__ __forceinline__ void bstore(double v, __amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, voff, soff, 0);
}
__device__ __forceinline__ void bstore(float v, __amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, voff, soff, 0);
}

// Keep a running sum materialised where it is updated.  Without this the
// compiler sinks a chain of per-plane accumulations to its single use after
// the unrolled sweep and keeps every operand live until then.  Emits nothing.
__device__ __forceinline__ void pin(double &x) { asm volatile("" : "+v"(x)); }

// A workgroup-uniform double, moved to SGPRs (VALU ops then take it as their
// scalar operand instead of holding a copy per lane).
__device__ __forceinline__ double uniform(double v) {
    const int lo = __builtin_amdgcn_readfirstlane(__double2loint(v));
    const int hi = __builtin_amdgcn_readfirstlane(__double2hiint(v));
    return __hiloint2double(hi, lo);
}

// The thread index as a value the compiler cannot relate to earlier uses:
// addresses derived from it are formed where they are needed instead of being
// kept live (and spilled) through the unrolled sweeps.
__device__ __forceinline__ int fresh_tid() {
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// Butterfly sum over the 64 lanes.  The lane index is made opaque so that the
// permute addresses are formed here rather than hoisted and kept live (they
// would otherwise occupy registers through the whole sweep).
__device__ __forceinline__ double wave_sum(double v) {
    int lane = (int)__lane_id();
    asm volatile("" : "+v"(lane));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const int src = (lane ^ off) << 2;
        const int lo = __builtin_amdgcn_ds_bpermute(src, __double2loint(v));
        const int hi = __builtin_amdgcn_ds_bpermute(src, __double2hiint(v));
        v += __hiloint2double(hi, lo);
    }
    return v;
}

// SplitMix64 (S. Vigna): first output for a given seed, mapped to [0, 1).
__device__ __forceinline__ double unit_from_seed(unsigned long long seed) {
    unsigned long long z = seed + 0x9E3779B97F4A7C15ULL;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    z = z ^ (z >> 31);
    return (double)(z >> 11) * (1.0 / 9007199254740992.0);
}

__device__ __forceinline__ void node_coords(long long q, int n, int &qi, int &qj, int &qk) {
    qi = (int)(q % n);
    qj = (int)((q / n) % n);
    qk = (int)(q / ((long long)n * n));
}

// Snapshot arguments and work items are read through the constant address
// space: their addresses are workgroup-uniform, so the fields load into SGPRs.
typedef __attribute__((address_space(4))) const RecurrenceArgs *SnapPtr;
typedef __attribute__((address_space(4))) const WorkItem *ItemPtr;

// The nodes a workgroup processes: one static share of snaps[0] (every node
// q0, q0 + qs, ... < q1 of one XCD's range), or items taken from the queue
// until it is empty.
struct WorkSource {
    int round = 0;
    template <typename LdsT>
    __device__ __forceinline__ bool next(const LaunchArgs &K, LdsT &L, int tid, SnapPtr &Ap, long long &q0,
                                         long long &q1, long long &qs) {
        if (!K.items) {
            if (round++) return false;
            Ap = (SnapPtr)K.snaps;
            const long long nd = Ap->nd;
            const int xcd = blockIdx.x & 7, per = gridDim.x >> 3, lw = blockIdx.x >> 3;
            q0 = nd * xcd / 8 + lw;
            q1 = nd * (xcd + 1) / 8;
            qs = per;
            return true;
        }
        __syncthreads();
        if (tid == 0) L.item = atomicAdd(K.counter, 1);
        __syncthreads();
        const int idx = __builtin_amdgcn_readfirstlane(L.item);
        if (idx >= K.n_items) return false;
        const ItemPtr it = (ItemPtr)K.items + idx;
        Ap = (SnapPtr)K.snaps + it->snap;
        q0 = it->q0;
        q1 = it->q1;
        qs = 1;
        return true;
    }
};

__device__ int sturm_count(int k, const double *a, const double *b, double x, double pivmin) {
    int cnt = 0;
    double d = a[0] - x;
    if (fabs(d) < pivmin) d = -pivmin;
    if (d < 0) ++cnt;
    for (int i = 1; i < k; ++i) {
        d = (a[i] - x) - b[i - 1] * b[i - 1] / d;
        if (fabs(d) < pivmin) d = -pivmin;
        if (d < 0) ++cnt;
    }
    return cnt;
}

// Point idx (0..31) of the 32 interior points that split [lo, hi] into 33
// equal parts; the same expression serves the lanes that evaluate the points
// and the lanes that take them over as the new bracket.
__device__ __forceinline__ double split_point(double lo, double hi, int idx) {
    return lo + (hi - lo) * ((double)(idx + 1) / 33.0);
}

// Extreme eigenvalues of the tridiagonal T_k by Sturm counts, on one wave:
// lanes 0-31 bracket the smallest eigenvalue (count target 1), lanes 32-63
// the largest (target k).  A round evaluates the count at 32 interior points
// of the bracket and keeps the sub-interval where it first reaches the
// target, which narrows the bracket 33-fold where bisection halves it.  The
// invariant count(lo) < target <= count(hi) holds throughout; the bracket
// shrinks until no interior point is left (adjacent doubles) and its upper
// end is returned, as with bisection.  out[0] = min, out[1] = max.
__device__ void sturm_extremes(int k, const double *a, const double *b, double *out, int lane) {
    double lo = INFINITY, hi = -INFINITY, bmax2 = 0.0;
    for (int i = 0; i < k; ++i) {
        const double r = (i > 0 ? fabs(b[i - 1]) : 0.0) + (i < k - 1 ? fabs(b[i]) : 0.0);
        lo = fmin(lo, a[i] - r);
        hi = fmax(hi, a[i] + r);
        if (i < k - 1) bmax2 = fmax(bmax2, b[i] * b[i]);
    }
    const double pivmin = 2.2250738585072014e-308 * fmax(bmax2, 1.0);
    const int half = lane >> 5, j = lane & 31;
    const int target = half ? k : 1;
    for (int round = 0; round < 64; ++round) {
        const double x = split_point(lo, hi, j);
        const bool inside = (x > lo) & (x < hi);
        const unsigned long long in_mask = __builtin_amdgcn_ballot_w64(inside);
        if ((unsigned)(half ? in_mask >> 32 : in_mask) == 0u) break;  // uniform per half
        const bool ge = inside ? sturm_count(k, a, b, x, pivmin) >= target : x >= hi;
        const unsigned long long gm = __builtin_amdgcn_ballot_w64(ge);
        const unsigned g32 = (unsigned)(half ? gm >> 32 : gm);
        const int f = g32 ? __builtin_ctz(g32) : 32;  // first point with count >= target
        const double nlo = f > 0 ? split_point(lo, hi, f - 1) : lo;
        const double nhi = f < 32 ? split_point(lo, hi, f) : hi;
        lo = nlo;
        hi = nhi;
    }
    if (j == 0) out[half] = hi;
}

}  // namespace
}  // namespace sq
