// Device helpers shared by the sweep kernels (vi.hip, block.hip).
#pragma once
#include <hip/hip_runtime.h>

namespace morap {
namespace k {

// ---------------------------------------------------------------------------
// neighbourhood blocks
// ---------------------------------------------------------------------------
constexpr int NSLOT = 5;
constexpr int BLK = 32;   // values per agent block

// Sparsity patterns of the blocks (bit 5a + d = entry P[a][d] may be nonzero):
// every entry, or the grid pattern of the host's slot order (slot 0 = stay,
// 1 + a = the cell move a aims at; the N/S moves slip E/W and vice versa).
constexpr uint32_t PAT_DENSE = (1u << 25) - 1;
constexpr uint32_t PAT_GRID = (1u << 0) | (1u << 1) | (1u << 3) | (1u << 4) |        // N: stay, N, E, W
                              (1u << 5) | (1u << 7) | (1u << 8) | (1u << 9) |        // S: stay, S, E, W
                              (1u << 10) | (1u << 11) | (1u << 12) | (1u << 13) |    // E: stay, N, S, E
                              (1u << 15) | (1u << 16) | (1u << 17) | (1u << 19) |    // W: stay, N, S, W
                              (1u << 20);                                            // stay
template <uint32_t PAT>
__device__ __forceinline__ constexpr bool nz(int a, int d) { return (PAT >> (a * NSLOT + d)) & 1u; }

inline uint32_t pattern_for(uint32_t union_pattern) {
    return (union_pattern & ~PAT_GRID) == 0 ? PAT_GRID : PAT_DENSE;
}

// ---------------------------------------------------------------------------
// vector helpers: CPL consecutive columns per lane
// ---------------------------------------------------------------------------
template <class T, int CPL> struct Vec { T v[CPL]; };

template <class T, int CPL>
__device__ __forceinline__ Vec<T, CPL> vload(const T* p) {
    Vec<T, CPL> r;
    if constexpr (CPL == 4 && sizeof(T) == 4) {
        float4 q = *reinterpret_cast<const float4*>(p);
        r.v[0] = q.x; r.v[1] = q.y; r.v[2] = q.z; r.v[3] = q.w;
    } else if constexpr (CPL == 2 && sizeof(T) == 4) {
        float2 q = *reinterpret_cast<const float2*>(p);
        r.v[0] = q.x; r.v[1] = q.y;
    } else if constexpr (CPL >= 2 && sizeof(T) == 8) {
#pragma unroll
        for (int c = 0; c < CPL; c += 2) {
            double2 q = *reinterpret_cast<const double2*>(p + c);
            r.v[c] = q.x; r.v[c + 1] = q.y;
        }
    } else {
#pragma unroll
        for (int c = 0; c < CPL; ++c) r.v[c] = p[c];
    }
    return r;
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// reduce across lanes that hold the same columns: lane bits >= log2(LPS)
template <int LPS>
__device__ __forceinline__ double group_max(double v) {
#pragma unroll
    for (int o = 32; o >= LPS; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// Raise the FP64 maximum stored (as its bit pattern) at p to v >= 0.  The
// current value is read first and the atomic skipped when it is already at
// least v: many workers flush maxima of the same (model, column) pairs, and
// most of them do not raise it, so this keeps atomics on a hot address few.
__device__ __forceinline__ void max_flush(unsigned long long* p, double v) {
    if (!(v > 0.0)) return;
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    // non-negative doubles order like their bit patterns
    if (__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= b) return;
    atomicMax(p, b);
}

// Share [b, e) of n ordered work items for worker idx of count workers on XCD
// xcd.  Workgroups are dealt to the 8 XCDs round-robin by blockIdx.x, so each
// XCD takes one contiguous eighth of the items (neighbouring items share its
// L2) and splits it evenly over its own workers.
__device__ __forceinline__ void xcd_share(int n, int xcd, int idx, int count, int& b, int& e) {
    const int xb = (int)((int64_t)n * xcd / 8), xe = (int)((int64_t)n * (xcd + 1) / 8);
    const int m = xe - xb;
    b = xb + (int)((int64_t)m * idx / count);
    e = xb + (int)((int64_t)m * (idx + 1) / count);
}

}  // namespace k
}  // namespace morap
