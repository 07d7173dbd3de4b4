// Device helpers of the kernels that keep the values of an iteration in LDS
// (resident.hip, instance.hip, staged.hip, rows.hip).
#pragma once
#include "common.h"
#include "kern.h"
#include "once_per_device.h"

#include <type_traits>

namespace morap {
namespace k {

constexpr int MAXW = 8;                       // waves of a workgroup
constexpr int RES_MAX_THREADS = 64 * MAXW;
constexpr int BIG_THREADS = 1024;             // of the kernel for larger products
constexpr int EVAL_BIG_STEPS = 10;            // states per thread of the evaluation of larger products
constexpr int GRID_NNZ = 17;                  // nonzero entries of the grid pattern
constexpr size_t LDS_BYTES = 160 * 1024;      // of a compute unit

// Dynamic LDS beyond 64 KB has to be asked for, once per kernel (whose `granted`
// this is) and device.
template <class F>
void grant_lds(OncePerDevice& granted, F* fn, size_t bytes = LDS_BYTES) {
    int device = 0;
    MORAP_HIP(hipGetDevice(&device));
    granted(device, [&] {
        MORAP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)bytes));
    });
}

// rows of one LDS buffer with ns states per thread (row 0 is the zero row):
// the second buffer lies at this fixed distance, which the 16-bit offset of
// an LDS access reaches
__host__ __device__ constexpr int res_rows(int ns) { return RES_MAX_THREADS * ns + 1; }

// nonzero entries of a sparsity pattern and the place of entry (a, d)
__host__ __device__ constexpr int pat_count(uint32_t pat, int below = 25) {
    int n = 0;
    for (int e = 0; e < below; ++e) n += (pat >> e) & 1u;
    return n;
}

// a value all lanes share, kept in scalar registers
__device__ __forceinline__ float scalar(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double scalar(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}

// a register of its own: values taken out of a wide load otherwise keep the
// whole load's registers, the unused ones among them
__device__ __forceinline__ float own_reg(float v) {
    float r;
    asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}
__device__ __forceinline__ double own_reg(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    unsigned lo, hi;
    asm volatile("v_mov_b32 %0, %1" : "=v"(lo) : "v"((unsigned)b));
    asm volatile("v_mov_b32 %0, %1" : "=v"(hi) : "v"((unsigned)(b >> 32)));
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)b, CTRL, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_ROR4 = 0x124, DPP_ROR8 = 0x128;

// maximum of two values >= 0 (which order like their bits: fmaxf would quiet
// each operand first)
__device__ __forceinline__ float mx(float a, float b) {
    return __builtin_bit_cast(float, max(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b)));
}
__device__ __forceinline__ double mx(double a, double b) { return fmax(a, b); }
__device__ __forceinline__ float max3(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ double max3(double a, double b, double c) { return fmax(fmax(a, b), c); }
// maximum of two values (fmaxf quiets each operand first)
__device__ __forceinline__ float max2(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double max2(double a, double b) { return fmax(a, b); }
// max(a, |b|)
__device__ __forceinline__ float max_abs(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, |%2|" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double max_abs(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, |%2|" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
// (v's low or high half) << SH
template <int SH>
__device__ __forceinline__ unsigned low_row(unsigned v) {
    unsigned r;
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0"
        : "=v"(r) : "s"(SH), "v"(v));
    return r;
}
template <int SH>
__device__ __forceinline__ unsigned high_row(unsigned v) {
    unsigned r;
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1"
        : "=v"(r) : "s"(SH), "v"(v));
    return r;
}

// Maxima of KC per-lane values >= 0 over each row of 16 lanes; afterwards lane
// l holds the maximum of value l % KC.  The values come out of max_abs, whose
// instruction the compiler does not see as one a lane-moving read has to wait
// for: the moves below read selections, and with one value a copy behind the
// two wait states.
template <class T, int KC>
__device__ __forceinline__ T row_max(const T (&v)[KC]) {
    const int lane = threadIdx.x & 63;
    T r;
    if constexpr (KC == 1) {
        T c = v[0];
        asm volatile("s_nop 1" : "+v"(c));
        r = mx(c, dpp<DPP_XOR1>(c));
        r = mx(r, dpp<DPP_XOR2>(r));
    } else if constexpr (KC == 2) {
        const bool odd = lane & 1;
        const T keep = odd ? v[1] : v[0], give = odd ? v[0] : v[1];
        r = mx(keep, dpp<DPP_XOR1>(give));
        r = mx(r, dpp<DPP_XOR2>(r));
    } else {
        const bool odd = lane & 1, high = lane & 2;
        const T a = mx(odd ? v[1] : v[0], dpp<DPP_XOR1>(odd ? v[0] : v[1]));
        const T b = mx(odd ? v[3] : v[2], dpp<DPP_XOR1>(odd ? v[2] : v[3]));
        r = mx(high ? b : a, dpp<DPP_XOR2>(high ? a : b));
    }
    r = mx(r, dpp<DPP_ROR4>(r));
    return mx(r, dpp<DPP_ROR8>(r));
}

template <class T, int KC>
struct Row {
    T v[KC];
};

// KC consecutive values at LDS address addr (the kernels have no LDS but the
// dynamic part, which starts at address 0)
template <class T, int KC>
__device__ __forceinline__ Row<T, KC> lds_get(unsigned addr) {
    using V = T __attribute__((ext_vector_type(KC)));
    const V v = *(__attribute__((address_space(3))) const V*)addr;
    Row<T, KC> r;
#pragma unroll
    for (int c = 0; c < KC; ++c) r.v[c] = v[c];
    return r;
}
template <class T, int KC>
__device__ __forceinline__ void lds_put(unsigned addr, const Row<T, KC>& r) {
    using V = T __attribute__((ext_vector_type(KC)));
    V v;
#pragma unroll
    for (int c = 0; c < KC; ++c) v[c] = r.v[c];
    *(__attribute__((address_space(3))) V*)addr = v;
}

// The maxima of a workgroup from the row maxima its waves left in `part` (four
// rows of four per wave, `stride` values apart), in every lane l for value
// l % 4; nw waves.
template <class T>
__device__ __forceinline__ T part_max(const T* part, int nw, int stride, int ln) {
    T r = 0;
    for (int q = ln >> 2; q < 4 * nw; q += 16) r = mx(r, part[(q * 4 + (ln & 3)) * stride]);
    r = mx(r, dpp<DPP_ROR4>(r));
    r = mx(r, dpp<DPP_ROR8>(r));
    r = mx(r, __shfl_xor(r, 16, 64));
    return mx(r, __shfl_xor(r, 32, 64));
}

// The stop test of one column: its largest change within max(eps, a few units
// in the last place of its largest value), or FP32's rounding floor: no new
// smallest change for stall_sweeps sweeps and within floor |y|.
template <bool F32>
__device__ __forceinline__ bool stop_test(const ResidentArgs& a, double res, double ym, double& best, int& stall,
                                          bool& floor_stop) {
    const double tol = fmax(a.eps, a.unit * ym);
    if (F32 && res > tol) {
        if (res < best) {
            best = res;
            stall = 0;
        } else {
            const int st = stall + 1;
            stall = st;
            floor_stop = st >= a.stall_sweeps && res <= a.floor * ym;
        }
    }
    return res <= tol || floor_stop;
}

// What a workgroup works on: the columns k0 .. k0 + KC - 1 of model m, or (INST)
// instance q.
template <class T, int KC, bool INST>
struct Item {
    bool ok;
    int m, k0, q;
    int64_t pair0, base;
    __device__ __forceinline__ explicit Item(const ResidentArgs& a) {
        if constexpr (INST) {
            ok = true;
            q = a.order[blockIdx.x];
            m = a.inst_model[q];
            k0 = 0;
            pair0 = q;
            base = a.inst_base[q];
        } else {
            // the columns of one product go to one XCD: its records meet in that L2
            const int slot = blockIdx.x >> 3;
            const int mi = slot / a.groups * 8 + (int)(blockIdx.x & 7);
            ok = mi < a.n_models;
            m = ok ? a.order[mi] : 0;
            k0 = slot % a.groups * KC;
            pair0 = (int64_t)m * a.Kp + k0;
            q = 0;
            base = 0;
        }
    }
    __device__ __forceinline__ bool running(const ResidentArgs& a, int c) const {
        return (INST || k0 + c < a.K) && a.pair_sweeps[pair0 + c] == 0;
    }
    __device__ __forceinline__ void weights(const ResidentArgs& a, int c, T& wc, T& wp) const {
        if constexpr (INST) {
            wc = scalar(a.iwc[q]);
            wp = scalar(a.iwp[q]);
        } else {
            const int k = k0 + c < a.K ? k0 + c : 0;
            const double* W = a.W + (int64_t)k * a.d;
            wc = scalar((T)W[m / a.nJ]);
            wp = scalar((T)W[a.nI + m % a.nJ]);
        }
    }
    // place of the value of the product's state l in column c
    __device__ __forceinline__ int64_t place(const ResidentArgs& a, int sb, int l, int c) const {
        return INST ? base + l : (int64_t)(sb + l) * a.Kp + k0 + c;
    }
    __device__ __forceinline__ T start(const ResidentArgs& a, int sb, int l, int c) const {
        if (!INST && k0 + c >= a.K) return 0;   // (the values have no such column where K is small)
        if (a.sweep0 > 0 || (!INST && a.warm)) return static_cast<const T*>(a.x0)[place(a, sb, l, c)];
        if constexpr (INST) {
            // the FP32 solve's values scaled to the instance's weights, where
            // its cost weight is positive (the values scale with the weights)
            if (!a.start0 || !(a.iwc[q] > 0.0)) return 0;
            const int k = a.inst_k[q];
            const float* x = a.start_par[(int64_t)m * a.start_Kp + k] ? a.start1 : a.start0;
            return (double)x[(int64_t)(sb + l) * a.start_Kp + k] * a.iscale[q];
        }
        return 0;
    }
    __device__ __forceinline__ bool stop(const ResidentArgs& a, double res, double ym, double& best, int& stall,
                                         bool& floor_stop) const {
        if constexpr (INST) return res <= a.ieps[q];
        else return stop_test<sizeof(T) == 4>(a, res, ym, best, stall, floor_stop);
    }
    __device__ __forceinline__ void stopped(const ResidentArgs& a, int c, int n, bool floor_stop) const {
        if constexpr (!INST) {
            if (floor_stop) atomicAdd((unsigned long long*)&a.counters[8], 1ull);
            a.final_par[pair0 + c] = 0;
        }
        a.pair_sweeps[pair0 + c] = n;
    }
};

}  // namespace k
}  // namespace morap
