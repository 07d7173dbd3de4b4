// Value iteration with the values resident in LDS (Alg. 3 to its stop for a
// few weight columns of one product, in one workgroup).
//
// Products are independent of each other and so are the columns of a
// product: nothing but the launch ties their sweeps together.  A workgroup
// here takes one product and KC columns, holds both Jacobi iterates of them
// in LDS (at most 64 KB each) and the product itself in registers (every
// thread keeps NS states: their nonzero transition probabilities and the LDS
// rows of their successor slots), and sweeps until every column has met its
// stop test.  A sweep then reads and writes LDS only; there is no launch, no
// stop test over global memory and no list of active tiles per sweep, and a
// column stops the work of its own workgroup only.
//
// The arithmetic of a backup, the change |y - x|, the stop test and the FP32
// rounding floor are those of the batched sweep over the neighbourhood
// blocks, operation by operation, so the values, the stopping sweep of every
// pair and its value at the initial state are the same bits.
#include "common.h"
#include "kern.h"

#include <cfloat>
#include <type_traits>

namespace morap {
namespace k {

namespace {

constexpr int MAXW = 8;                       // waves of a workgroup
constexpr int RES_MAX_THREADS = 64 * MAXW;

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

// waves per SIMD the registers are held to, so that the probabilities of NS
// states fit with room for a step: 128 registers, 168 or 256
__host__ __device__ constexpr int res_waves_per_simd(int bytes, int ns, bool fast) {
    const int need = ns * (bytes / 4) * (fast ? 2 : 3);
    return need <= 6 ? 4 : (need <= 8 ? 3 : 2);
}

}  // namespace

// One product (blockIdx -> model, column group) to its stop.  A wave holds
// the states [w 64 NS, (w + 1) 64 NS) of the product, 64 consecutive ones per
// step; lanes past the last state repeat it in rows of their own.  Sweep n reads buffer (n - 1) & 1
// and writes buffer n & 1 with one barrier; the stop test of sweep n is taken
// by one wave while the others run sweep n + 1, and seen by all behind the
// barrier of n + 1, when buffer n & 1 still holds iterate n: a column's final
// values leave from there, each thread its own states.
template <class T, int KC, int NS, bool FAST>
__global__ void __launch_bounds__(RES_MAX_THREADS, res_waves_per_simd(sizeof(T), NS, FAST))
resident_vi(ResidentArgs a) {
    constexpr uint32_t PAT = FAST ? PAT_GRID : PAT_DENSE;
    constexpr bool UC = FAST;                             // one cost per action
    constexpr int NNZ = pat_count(PAT);
    constexpr int ROWB = sizeof(T) * KC;                  // bytes of an LDS row
    constexpr int SH = ROWB == 4 ? 2 : (ROWB == 8 ? 3 : 4);
    constexpr int BUF = res_rows(NS) * ROWB;              // distance of the two buffers
    constexpr bool want_y = sizeof(T) == 4;               // |y| only bounds the FP32 stop test
    static_assert(BUF <= 65535, "the second buffer must lie within an LDS offset");
    extern __shared__ __align__(16) unsigned char lds[];

    // the columns of one product go to one XCD: its records meet in that L2
    const int slot = blockIdx.x >> 3;
    const int mi = slot / a.groups * 8 + (int)(blockIdx.x & 7);
    if (mi >= a.n_models) return;
    const int m = a.order[mi];
    const int k0 = slot % a.groups * KC;
    const int64_t pair0 = (int64_t)m * a.Kp + k0;
    bool on[KC];
    bool any = false;
#pragma unroll
    for (int c = 0; c < KC; ++c) {
        on[c] = k0 + c < a.K && a.pair_sweeps[pair0 + c] == 0;
        any |= on[c];
    }
    if (!any) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
    const int sb = a.state_base[m], S = a.state_base[m + 1] - sb;
    unsigned char* hdr = lds + BUF + (((nw * 64 * NS + 1) * ROWB + 15) & ~15);
    T* part = reinterpret_cast<T*>(hdr);                               // [2][4 MAXW rows][4][res, |y|]
    // the judge's state per column, kept out of the registers of a sweep
    double* best = reinterpret_cast<double*>(hdr + 2 * 4 * MAXW * 8 * sizeof(T));       // [4] smallest change so far
    int* stall = reinterpret_cast<int*>(best + 4);                                      // [4] sweeps since it was set
    unsigned* flag = reinterpret_cast<unsigned*>(stall + 4);                            // [2] results of the stop test
    // (the kernel has no other LDS: the dynamic part starts at address 0)
    auto get = [&](int buf, unsigned addr) -> Row<T, KC> {
        using V = T __attribute__((ext_vector_type(KC)));
        const V v = *(__attribute__((address_space(3))) const V*)(addr + buf * BUF);
        Row<T, KC> r;
#pragma unroll
        for (int c = 0; c < KC; ++c) r.v[c] = v[c];
        return r;
    };
    auto put = [&](int buf, unsigned addr, const Row<T, KC>& r) {
        using V = T __attribute__((ext_vector_type(KC)));
        V v;
#pragma unroll
        for (int c = 0; c < KC; ++c) v[c] = r.v[c];
        *(__attribute__((address_space(3))) V*)(addr + buf * BUF) = v;
    };

    // the record of every state (they are stored in tile order: each names
    // its state)
    int* where = reinterpret_cast<int*>(lds);
    for (int p = tid; p < S; p += blockDim.x) where[a.rec[(int64_t)(sb + p) * 8 + 7] - sb] = p;
    __syncthreads();
    T P[NS][NNZ], cost[UC ? 1 : NS][5];
    unsigned o01[NS], o23[NS], o4[NS];     // LDS rows of the slots, 16 bits each; o4: accepting slots above
    unsigned acc_steps = 0;                // steps in which a lane of this wave has an accepting slot
    const int own0 = wave * 64 * NS + lane + 1;   // LDS row of the first step's state; step i: + 64 i
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const int l = min(own0 - 1 + 64 * i, S - 1);
        const int32_t* r = a.rec + (int64_t)(sb + where[l]) * 8;
        const int4 r0 = *reinterpret_cast<const int4*>(r), r1 = *reinterpret_cast<const int4*>(r + 4);
        auto place = [&](int s) { return s == a.zero_row ? 0u : (unsigned)(s - sb + 1); };
        o01[i] = place(r0.x) | place(r0.y) << 16;
        o23[i] = place(r0.z) | place(r0.w) << 16;
        const unsigned accm = (unsigned)r1.z & 31u;
        o4[i] = place(r1.x) | accm << 16;
        if (__ballot(accm != 0)) acc_steps |= 1u << i;
        const T* B = static_cast<const T*>(a.ablk) + (int64_t)r1.y * BLK;
        int e = 0;
#pragma unroll
        for (int q = 0; q < NSLOT * NSLOT; ++q)
            if ((PAT >> q) & 1u) P[i][e++] = own_reg(B[q]);
#pragma unroll
        for (int q = 0; q < 5; ++q)
            if (!UC || i == 0) cost[UC ? 0 : i][q] = own_reg(B[25 + q]);
    }
    __syncthreads();   // the buffers take the values now

    T wc[KC], wp[KC];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
        const int k = k0 + c < a.K ? k0 + c : 0;
        const double* W = a.W + (int64_t)k * a.d;
        wc[c] = scalar((T)W[m / a.nJ]);
        wp[c] = scalar((T)W[a.nI + m % a.nJ]);
    }
    // every state of the product has the same action costs: w_c (-cost) once
    T first[UC ? KC : 1][5];
    if constexpr (UC) {
#pragma unroll
        for (int c = 0; c < KC; ++c)
#pragma unroll
            for (int q = 0; q < 5; ++q) first[c][q] = scalar(wc[c] * cost[0][q]);
    }
    T* x0 = static_cast<T*>(a.x0);
    T* x1 = static_cast<T*>(a.x1);
    const bool load = a.warm || a.sweep0 > 0;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        Row<T, KC> v;
#pragma unroll
        for (int c = 0; c < KC; ++c) v.v[c] = load ? x0[(int64_t)(sb + min(own0 - 1 + 64 * i, S - 1)) * a.Kp + k0 + c] : (T)0;
        put(0, (unsigned)(own0 + 64 * i) << SH, v);
    }
    if (tid == 0) {
        Row<T, KC> z;
#pragma unroll
        for (int c = 0; c < KC; ++c) z.v[c] = 0;
        put(0, 0, z);
        put(1, 0, z);
        flag[0] = flag[1] = 0;
    }
    // the stop test is taken by the last wave, whose last steps may be empty
    const bool judge = wave == nw - 1;
    if (want_y && tid < KC) {
        best[tid] = a.best_res[pair0 + tid];
        stall[tid] = a.stall[pair0 + tid];
    }
    unsigned live = 0;   // columns still running
#pragma unroll
    for (int c = 0; c < KC; ++c) live |= on[c] ? 1u << c : 0u;
    unsigned judged = live;   // the same, as the stop test has them (a sweep ahead)
    __syncthreads();

    auto sweep = [&](auto PAR) {
        constexpr int IN = decltype(PAR)::value;
        T r[KC], y[KC];
#pragma unroll
        for (int c = 0; c < KC; ++c) r[c] = y[c] = 0;
        auto fetch = [&](int i, Row<T, KC> (&xv)[NSLOT]) {
            // (opaque: hoisting the unpacked rows out of the sweeps would not
            // leave room for the probabilities)
            asm volatile("" : "+v"(o01[i]), "+v"(o23[i]), "+v"(o4[i]));
            xv[0] = get(IN, low_row<SH>(o01[i]));
            xv[1] = get(IN, high_row<SH>(o01[i]));
            xv[2] = get(IN, low_row<SH>(o23[i]));
            xv[3] = get(IN, high_row<SH>(o23[i]));
            xv[4] = get(IN, low_row<SH>(o4[i]));
        };
        // start of action q's sum in column c: w_c (-cost)
        auto start = [&](int i, int q, int c) -> T {
            if constexpr (UC) return first[c][q];
            else return wc[c] * cost[i][q];
        };
        auto backup = [&](int i, const Row<T, KC> (&xv)[NSLOT], auto ACC) {
            Row<T, KC> old = xv[0];
            if constexpr (!FAST) old = get(IN, (unsigned)(own0 + 64 * i) << SH);
            T rp[5];
            if constexpr (decltype(ACC)::value) {
                // probability reward: the action's mass on accepting slots
                const unsigned accm = o4[i] >> 16;
                int e = 0;
#pragma unroll
                for (int q = 0; q < 5; ++q) {
                    bool first_term = true;
#pragma unroll
                    for (int d = 0; d < NSLOT; ++d)
                        if (nz<PAT>(q, d)) {
                            const T p = (accm >> d & 1) ? P[i][e] : (T)0;
                            rp[q] = first_term ? p : rp[q] + p;
                            first_term = false;
                            ++e;
                        }
                }
            }
            Row<T, KC> out;
#pragma unroll
            for (int c = 0; c < KC; ++c) {
                T v[5];
                int e = 0;
#pragma unroll
                for (int q = 0; q < 5; ++q) {
                    v[q] = start(i, q, c);
                    if constexpr (decltype(ACC)::value) v[q] = fma(wp[c], rp[q], v[q]);
#pragma unroll
                    for (int d = 0; d < NSLOT; ++d)
                        if (nz<PAT>(q, d)) v[q] = fma(P[i][e++], xv[d].v[c], v[q]);
                }
                out.v[c] = max3(max3(v[0], v[1], v[2]), v[3], v[4]);
                r[c] = max_abs(r[c], out.v[c] - old.v[c]);
                if (want_y) y[c] = max_abs(y[c], out.v[c]);
            }
            put(1 - IN, (unsigned)(own0 + 64 * i) << SH, out);
        };
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            Row<T, KC> xv[NSLOT];
            fetch(i, xv);
            if (acc_steps >> i & 1) backup(i, xv, std::true_type{});
            else backup(i, xv, std::false_type{});
        }
        const T rr = row_max<T, KC>(r);
        const T yy = want_y ? row_max<T, KC>(y) : (T)0;
        if ((lane & 15) < 4) {
            T* p = part + ((((1 - IN) * 4 * MAXW) + wave * 4 + (lane >> 4)) * 4 + (lane & 3)) * 2;
            p[0] = rr;
            p[1] = yy;
        }
    };

    // stop test of sweep n, whose iterate is in buffer n & 1
    auto decide = [&](auto PAR, int n) {
        constexpr int CUR = decltype(PAR)::value;
        int ln = lane;
        asm volatile("" : "+v"(ln));   // (as above: no addresses kept over the sweeps)
        T rr = 0, yy = 0;
        for (int q = ln >> 2; q < 4 * nw; q += 16) {
            const T* p = part + ((CUR * 4 * MAXW + q) * 4 + (ln & 3)) * 2;
            rr = mx(rr, p[0]);
            yy = mx(yy, p[1]);
        }
        rr = mx(rr, dpp<DPP_ROR4>(rr));
        rr = mx(rr, dpp<DPP_ROR8>(rr));
        rr = mx(rr, __shfl_xor(rr, 16, 64));
        rr = mx(rr, __shfl_xor(rr, 32, 64));
        if (want_y) {
            yy = mx(yy, dpp<DPP_ROR4>(yy));
            yy = mx(yy, dpp<DPP_ROR8>(yy));
            yy = mx(yy, __shfl_xor(yy, 16, 64));
            yy = mx(yy, __shfl_xor(yy, 32, 64));
        }
        // lane c < KC tests column c
        bool now = false;
        if (ln < KC && (judged >> ln & 1)) {
            const double res = (double)rr, ym = (double)yy;
            const double tol = fmax(a.eps, a.unit * ym);
            bool floor_stop = false;
            if (want_y && res > tol) {
                // the rounding floor: no new smallest change for stall_sweeps sweeps
                if (res < best[ln]) {
                    best[ln] = res;
                    stall[ln] = 0;
                } else {
                    const int st = stall[ln] + 1;
                    stall[ln] = st;
                    floor_stop = st >= a.stall_sweeps && res <= a.floor * ym;
                }
            }
            now = res <= tol || floor_stop;
            if (now) {
                const int64_t i = (int64_t)m * a.Kp + k0 + ln;
                if (floor_stop) atomicAdd((unsigned long long*)&a.counters[8], 1ull);
                a.final_par[i] = 0;
                a.pair_sweeps[i] = n;
                // (a product with states has a live initial state)
                const int s_init = a.init[m] - sb + 1;
                a.c[(int64_t)(k0 + ln) * a.M + m] =
                    (double)reinterpret_cast<const T*>(lds + CUR * BUF + ((unsigned)s_init << SH))[ln];
            }
        }
        const unsigned fresh = (unsigned)__ballot(now);
        judged &= ~fresh;
        if (ln == 0) flag[CUR] = fresh | (judged == 0 ? 0x100u : 0u);
    };

    // final (or, at the end of the launch, current) values of the columns in
    // `cols` from buffer `buf`, each thread its own states
    auto store = [&](T* x, int buf, unsigned cols) {
        int l = own0 - 1;
        asm volatile("" : "+v"(l));   // (as above: no addresses kept over the sweeps)
#pragma clang loop unroll(disable)
        for (int i = 0; i < NS && l < S; ++i, l += 64) {
            const Row<T, KC> v = get(buf, (unsigned)(l + 1) << SH);
#pragma unroll
            for (int c = 0; c < KC; ++c)
                if (cols >> c & 1) x[(int64_t)(sb + l) * a.Kp + k0 + c] = v.v[c];
        }
    };

    // true when the workgroup is done
    auto step = [&](auto PAR, int n) -> bool {
        constexpr int IN = decltype(PAR)::value;
        const bool more = n <= a.sweep1;
        if (more) sweep(PAR);
        __syncthreads();
        const unsigned f = flag[IN];             // the stop test of sweep n - 1
        if (f & 0xffu) {
            store(x0, IN, f & 0xffu);
            live &= ~f;
        }
        if (f & 0x100u) return true;
        if (!more) {
            // the launch ends with columns running: their iterate, and after
            // the last launch of a solve the iterate before it
            store(x0, IN, live);
            if (a.last) store(x1, 1 - IN, live);
            if (judge && lane < KC && (live >> lane & 1)) {
                const int64_t i = (int64_t)m * a.Kp + k0 + lane;
                if (want_y) {
                    a.best_res[i] = best[lane];
                    a.stall[i] = stall[lane];
                }
                if (a.last) a.active[i] = 1;
            }
            return true;
        }
        if (judge) decide(std::integral_constant<int, 1 - IN>{}, n);
        return false;
    };
    for (int n = a.sweep0 + 1;; n += 2) {        // sweep0 and sweep1 are even
        if (step(std::integral_constant<int, 0>{}, n)) return;
        if (step(std::integral_constant<int, 1>{}, n + 1)) return;
    }
}

// ---------------------------------------------------------------------------
// dispatch
// ---------------------------------------------------------------------------
// States a workgroup can hold: 512 per register step.  The grid pattern with
// one cost per action needs 17 probabilities a state (7 steps in FP32, 4 in
// FP64 within 256 registers), the general block 25 and 5 costs (4 and 2).
static int resident_steps(int prec, bool fast) {
    return prec == MORAP_F32 ? (fast ? 7 : 4) : (fast ? 4 : 2);
}

bool has_grid_pattern(uint32_t union_pattern) { return pattern_for(union_pattern) == PAT_GRID; }

int resident_capacity(int prec, bool fast) {
    return res_rows(resident_steps(prec, fast)) - 1;
}

namespace {

template <class T, int KC, int NS, bool FAST>
void launch_res(hipStream_t s, const ResidentArgs& a, int max_states) {
    auto* fn = &resident_vi<T, KC, NS, FAST>;
    constexpr int ROWB = sizeof(T) * KC;
    const int threads = 64 * ((max_states + 64 * NS - 1) / (64 * NS));
    const size_t bytes = (size_t)res_rows(NS) * ROWB + (((size_t)(threads * NS + 1) * ROWB + 15) & ~(size_t)15) +
                         2 * 4 * MAXW * 8 * sizeof(T) + 64;
    MORAP_CHECK(threads <= RES_MAX_THREADS && max_states < res_rows(NS) && bytes <= 160 * 1024, MORAP_E_UNSUPPORTED,
                "a product does not fit the LDS-resident iteration");
    // dynamic LDS beyond 64 KB has to be asked for, once per kernel
    static const hipError_t granted =
        hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    MORAP_HIP(granted);
    const unsigned blocks = 8u * (unsigned)((a.n_models + 7) / 8) * (unsigned)a.groups;
    hipLaunchKernelGGL(fn, dim3(blocks), dim3((unsigned)threads), bytes, s, a);
    MORAP_HIP(hipGetLastError());
}

template <class T, int KC, bool FAST, int MAXNS>
void launch_steps(hipStream_t s, const ResidentArgs& a, int ns, int max_states) {
    if (ns == 1) return launch_res<T, KC, 1, FAST>(s, a, max_states);
    if constexpr (MAXNS >= 2)
        if (ns == 2) return launch_res<T, KC, 2, FAST>(s, a, max_states);
    if constexpr (MAXNS >= 3)
        if (ns == 3) return launch_res<T, KC, 3, FAST>(s, a, max_states);
    if constexpr (MAXNS >= 4)
        if (ns == 4) return launch_res<T, KC, 4, FAST>(s, a, max_states);
    if constexpr (MAXNS >= 7)
        if (ns == 7) return launch_res<T, KC, 7, FAST>(s, a, max_states);
    fail(MORAP_E_UNSUPPORTED, "a product does not fit the LDS-resident iteration");
}

}  // namespace

int resident_class(int states) {
    const int ns = (states + RES_MAX_THREADS - 1) / RES_MAX_THREADS;
    return ns <= 4 ? (ns < 1 ? 1 : ns) : 7;
}

void resident(hipStream_t s, int prec, bool fast, bool wide, int max_states, ResidentArgs a) {
    if (a.n_models <= 0) return;
    const int ns = resident_class(max_states);
    const int kc = !wide ? 1 : (prec == MORAP_F32 ? 4 : 2);
    a.groups = (a.K + kc - 1) / kc;
    if (prec == MORAP_F32) {
        if (fast && wide) launch_steps<float, 4, true, 7>(s, a, ns, max_states);
        else if (fast) launch_steps<float, 1, true, 7>(s, a, ns, max_states);
        else if (wide) launch_steps<float, 4, false, 4>(s, a, ns, max_states);
        else launch_steps<float, 1, false, 4>(s, a, ns, max_states);
    } else {
        if (fast && wide) launch_steps<double, 2, true, 4>(s, a, ns, max_states);
        else if (fast) launch_steps<double, 1, true, 4>(s, a, ns, max_states);
        else if (wide) launch_steps<double, 2, false, 2>(s, a, ns, max_states);
        else launch_steps<double, 1, false, 2>(s, a, ns, max_states);
    }
}

}  // namespace k
}  // namespace morap
