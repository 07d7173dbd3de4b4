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
constexpr int BIG_THREADS = 1024;             // of the kernel for larger products
constexpr int GRID_NNZ = 17;                  // nonzero entries of the grid pattern
constexpr size_t LDS_BYTES = 160 * 1024;      // of a compute unit

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
            bool floor_stop = false;
            now = stop_test<want_y>(a, (double)rr, (double)yy, best[ln], stall[ln], floor_stop);
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
// larger products
// ---------------------------------------------------------------------------
// A product too large for two iterates in LDS and its probabilities in
// registers: one iterate in LDS (up to 160 KB), the new values of a sweep in
// registers until every wave has read the old ones.  Its states are sorted
// by block and padded to steps of 64 states of one block, so that a step's
// probabilities are scalar loads shared by the wave; the LDS rows of a
// state's slots are read from the sorted records every sweep (12 of 16 bytes
// a state, from L2: the columns of a product go to one XCD).  Sorting costs
// up to a step of padding per block and scatters the neighbours' rows over the
// banks; reading the 17 probabilities per lane instead would cost 1.5 (FP32)
// or 3 (FP64) times the LDS traffic of the values themselves.
//
// 24 agents on 32 x 32 .. 128 x 128 grids x 32 tasks, 64 columns, FP32: 0.80
// (4 columns), 0.53 (2) and 0.28 (1) 10^12 state-columns a second against 0.34
// of the batched sweeps on all products of that problem; 37 FP64 columns of 49
// products of up to 2,429 states: 2.3 ms, 10 ms before.
template <class T, int KC, int NS>
__global__ void __launch_bounds__(BIG_THREADS)
resident_big(ResidentArgs a) {
    constexpr int ROWB = sizeof(T) * KC;
    constexpr int SH = ROWB == 4 ? 2 : (ROWB == 8 ? 3 : 4);
    constexpr bool want_y = sizeof(T) == 4;
    constexpr int NW = BIG_THREADS / 64;
    extern __shared__ __align__(16) unsigned char lds[];

    const int slot = blockIdx.x >> 3;
    const int mi = slot / a.groups * 8 + (int)(blockIdx.x & 7);
    if (mi >= a.n_models) return;
    const int m = a.order[mi];
    const int k0 = slot % a.groups * KC;
    const int64_t pair0 = (int64_t)m * a.Kp + k0;
    unsigned live = 0;   // columns still running
#pragma unroll
    for (int c = 0; c < KC; ++c)
        if (k0 + c < a.K && a.pair_sweeps[pair0 + c] == 0) live |= 1u << c;
    if (!live) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sb = a.state_base[m];
    const int pos0 = a.big_base[m], n_steps = (a.big_base[m + 1] - pos0) >> 6;
    // this wave's steps: a contiguous run, so consecutive ones mostly share
    // their block
    const int s_begin = wave * n_steps / NW, cnt = (wave + 1) * n_steps / NW - s_begin;
    using CInt = const __attribute__((address_space(4))) int32_t*;
    using CVal = const __attribute__((address_space(4))) T*;
    const CInt blk = (CInt)(a.big_block + (pos0 >> 6) + s_begin);
    const CVal ablk = (CVal)(static_cast<const T*>(a.grid_blk));
    const uint4* rec = a.big_rec + pos0 + s_begin * 64 + lane;
    unsigned char* hdr = lds + (((n_steps * 64 + 1) * ROWB + 15) & ~15);
    T* part = reinterpret_cast<T*>(hdr);                                     // [4 NW rows][4][res, |y|]
    double* best = reinterpret_cast<double*>(hdr + 4 * NW * 8 * sizeof(T));  // [4] smallest change so far
    int* stall = reinterpret_cast<int*>(best + 4);                           // [4] sweeps since it was set
    unsigned* flag = reinterpret_cast<unsigned*>(stall + 4);
    using V = T __attribute__((ext_vector_type(KC)));
    auto get = [&](unsigned addr) -> Row<T, KC> {
        const V v = *(__attribute__((address_space(3))) const V*)addr;
        Row<T, KC> r;
#pragma unroll
        for (int c = 0; c < KC; ++c) r.v[c] = v[c];
        return r;
    };
    auto put = [&](unsigned addr, const Row<T, KC>& r) {
        V v;
#pragma unroll
        for (int c = 0; c < KC; ++c) v[c] = r.v[c];
        *(__attribute__((address_space(3))) V*)addr = v;
    };

    T wp[KC], first[KC][5];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
        const int k = k0 + c < a.K ? k0 + c : 0;
        const double* W = a.W + (int64_t)k * a.d;
        const T wc = (T)W[m / a.nJ];
        wp[c] = scalar((T)W[a.nI + m % a.nJ]);
        // every state of the product has the same action costs
#pragma unroll
        for (int q = 0; q < 5; ++q) first[c][q] = wc * ablk[(int64_t)blk[-s_begin] * GRID_BLK + GRID_NNZ + q];
    }
    T* x0 = static_cast<T*>(a.x0);
    T* x1 = static_cast<T*>(a.x1);
    const bool load = a.warm || a.sweep0 > 0;
    const unsigned own0 = (unsigned)(s_begin * 64 + lane + 1) << SH;   // LDS row of the first step's state
    for (int i = 0; i < cnt; ++i) {
        const unsigned w = rec[i * 64].w & 0x7fffffffu;
        Row<T, KC> v;
#pragma unroll
        for (int c = 0; c < KC; ++c) v.v[c] = load ? x0[(int64_t)(sb + (int)w) * a.Kp + k0 + c] : (T)0;
        put(own0 + ((unsigned)i << (6 + SH)), v);
    }
    if (tid == 0) {
        Row<T, KC> z;
#pragma unroll
        for (int c = 0; c < KC; ++c) z.v[c] = 0;
        put(0, z);
    }
    if (want_y && tid < KC) {
        best[tid] = a.best_res[pair0 + tid];
        stall[tid] = a.stall[pair0 + tid];
    }
    __syncthreads();

    // the values of the columns in `cols`, each thread its own states
    auto store = [&](T* x, unsigned cols) {
        unsigned own = own0;
        asm volatile("" : "+v"(own));   // (no addresses kept over the sweeps)
        for (int i = 0; i < cnt; ++i) {
            const unsigned w = rec[i * 64].w;
            const Row<T, KC> v = get(own + ((unsigned)i << (6 + SH)));
            if (w >> 31) continue;   // padding
#pragma unroll
            for (int c = 0; c < KC; ++c)
                if (cols >> c & 1) x[(int64_t)(sb + (int)w) * a.Kp + k0 + c] = v.v[c];
        }
    };

    Row<T, KC> out[NS];
    for (int n = a.sweep0 + 1; n <= a.sweep1; ++n) {
        T r[KC], y[KC];
#pragma unroll
        for (int c = 0; c < KC; ++c) r[c] = y[c] = 0;
        uint3 q = *reinterpret_cast<const uint3*>(rec);
        int b = blk[0];
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            if (i < cnt) {
            uint3 qn = q;
            int bn = b;
            if (i + 1 < cnt) {   // the next step's records and block are on their way
                qn = *reinterpret_cast<const uint3*>(rec + (i + 1) * 64);
                bn = blk[i + 1];
            }
            const CVal B = ablk + (int64_t)b * GRID_BLK;
            T P[GRID_NNZ];
#pragma unroll
            for (int e = 0; e < GRID_NNZ; ++e) P[e] = B[e];
            Row<T, KC> xv[NSLOT];
            xv[0] = get(low_row<SH>(q.x));
            xv[1] = get(high_row<SH>(q.x));
            xv[2] = get(low_row<SH>(q.y));
            xv[3] = get(high_row<SH>(q.y));
            xv[4] = get(low_row<SH>(q.z));
            const unsigned accm = q.z >> 16;
            auto backup = [&](auto ACC) {
                T rp[5];
                if constexpr (decltype(ACC)::value) {
                    // probability reward: the action's mass on accepting slots
                    int e = 0;
#pragma unroll
                    for (int act = 0; act < 5; ++act) {
                        bool first_term = true;
#pragma unroll
                        for (int d = 0; d < NSLOT; ++d)
                            if (nz<PAT_GRID>(act, d)) {
                                const T p = (accm >> d & 1) ? P[e] : (T)0;
                                rp[act] = first_term ? p : rp[act] + p;
                                first_term = false;
                                ++e;
                            }
                    }
                }
#pragma unroll
                for (int c = 0; c < KC; ++c) {
                    T v[5];
                    int e = 0;
#pragma unroll
                    for (int act = 0; act < 5; ++act) {
                        v[act] = first[c][act];
                        if constexpr (decltype(ACC)::value) v[act] = fma(wp[c], rp[act], v[act]);
#pragma unroll
                        for (int d = 0; d < NSLOT; ++d)
                            if (nz<PAT_GRID>(act, d)) v[act] = fma(P[e++], xv[d].v[c], v[act]);
                    }
                    out[i].v[c] = max3(max3(v[0], v[1], v[2]), v[3], v[4]);
                    r[c] = max_abs(r[c], out[i].v[c] - xv[0].v[c]);   // slot 0 is the state itself
                    if (want_y) y[c] = max_abs(y[c], out[i].v[c]);
                }
            };
            if (__ballot(accm != 0)) backup(std::true_type{});
            else backup(std::false_type{});
            q = qn;
            b = bn;
            }
        }
        const T rr = row_max<T, KC>(r);
        const T yy = want_y ? row_max<T, KC>(y) : (T)0;
        if ((lane & 15) < 4) {
            T* p = part + ((wave * 4 + (lane >> 4)) * 4 + (lane & 3)) * 2;
            p[0] = rr;
            p[1] = yy;
        }
        // the iterate before the last, of a solve over its limit
        if (a.last && n == a.sweep1) store(x1, live);
        __syncthreads();   // every wave has read the old values
#pragma unroll
        for (int i = 0; i < NS; ++i)
            if (i < cnt) put(own0 + ((unsigned)i << (6 + SH)), out[i]);
        if (wave == NW - 1) {
            int ln = lane;
            asm volatile("" : "+v"(ln));
            T res_t = 0, y_t = 0;
            for (int z = ln >> 2; z < 4 * NW; z += 16) {
                const T* p = part + (z * 4 + (ln & 3)) * 2;
                res_t = mx(res_t, p[0]);
                y_t = mx(y_t, p[1]);
            }
            res_t = mx(res_t, dpp<DPP_ROR4>(res_t));
            res_t = mx(res_t, dpp<DPP_ROR8>(res_t));
            res_t = mx(res_t, __shfl_xor(res_t, 16, 64));
            res_t = mx(res_t, __shfl_xor(res_t, 32, 64));
            if (want_y) {
                y_t = mx(y_t, dpp<DPP_ROR4>(y_t));
                y_t = mx(y_t, dpp<DPP_ROR8>(y_t));
                y_t = mx(y_t, __shfl_xor(y_t, 16, 64));
                y_t = mx(y_t, __shfl_xor(y_t, 32, 64));
            }
            bool now = false;
            if (ln < KC && (live >> ln & 1)) {
                bool floor_stop = false;
                now = stop_test<want_y>(a, (double)res_t, (double)y_t, best[ln], stall[ln], floor_stop);
                if (now) {
                    const int64_t i = (int64_t)m * a.Kp + k0 + ln;
                    if (floor_stop) atomicAdd((unsigned long long*)&a.counters[8], 1ull);
                    a.final_par[i] = 0;
                    a.pair_sweeps[i] = n;
                }
            }
            const unsigned fresh = (unsigned)__ballot(now);
            if (ln == 0) *flag = fresh;
        }
        __syncthreads();
        const unsigned f = *flag;
        if (f) {
            store(x0, f);
            if (tid < KC && (f >> tid & 1))
                a.c[(int64_t)(k0 + tid) * a.M + m] =
                    (double)reinterpret_cast<const T*>(lds + ((unsigned)(a.big_init[m] + 1) << SH))[tid];
            live &= ~f;
            if (!live) return;
        }
    }
    // the launch ends with columns running: their iterate
    store(x0, live);
    if (tid < KC && (live >> tid & 1)) {
        const int64_t i = pair0 + tid;
        if (want_y) {
            a.best_res[i] = best[tid];
            a.stall[i] = stall[tid];
        }
        if (a.last) a.active[i] = 1;
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
    MORAP_CHECK(threads <= RES_MAX_THREADS && max_states < res_rows(NS) && bytes <= LDS_BYTES, MORAP_E_UNSUPPORTED,
                "a product does not fit the LDS-resident iteration");
    // dynamic LDS beyond 64 KB has to be asked for, once per kernel
    static const hipError_t granted =
        hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_BYTES);
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

bool grid_entry(int e) { return (PAT_GRID >> e) & 1u; }

int resident_most_positions() {
    int p = BIG_THREADS * 40;
    while (resident_big_columns(MORAP_F32, p) == 0) p -= 64;
    return p;
}

// Columns a workgroup takes of a larger product of `positions` sorted and
// padded states (0: it does not fit): as many as LDS holds one iterate of,
// at most 4 (FP32) or 2 (FP64), 40 words of new values per thread.
int resident_big_columns(int prec, int positions) {
    const int el = prec == MORAP_F32 ? 4 : 8;
    for (int kc = 16 / el; kc >= 1; kc /= 2) {
        const size_t bytes = (((size_t)positions + 1) * kc * el + 15) / 16 * 16 + 4 * (BIG_THREADS / 64) * 8 * el + 64;
        if (bytes <= LDS_BYTES && positions <= BIG_THREADS * 160 / (el * kc)) return kc;
    }
    return 0;
}

namespace {

template <class T, int KC>
void launch_big(hipStream_t s, const ResidentArgs& a, int max_positions) {
    constexpr int NS = 160 / (sizeof(T) * KC);
    auto* fn = &resident_big<T, KC, NS>;
    const size_t bytes = (((size_t)max_positions + 1) * sizeof(T) * KC + 15) / 16 * 16 +
                         4 * (BIG_THREADS / 64) * 8 * sizeof(T) + 64;
    MORAP_CHECK(max_positions % 64 == 0 && bytes <= LDS_BYTES && max_positions <= BIG_THREADS * NS,
                MORAP_E_UNSUPPORTED, "a product does not fit the LDS-resident iteration");
    static const hipError_t granted =
        hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_BYTES);
    MORAP_HIP(granted);
    const unsigned blocks = 8u * (unsigned)((a.n_models + 7) / 8) * (unsigned)a.groups;
    hipLaunchKernelGGL(fn, dim3(blocks), dim3(BIG_THREADS), bytes, s, a);
    MORAP_HIP(hipGetLastError());
}

}  // namespace

void resident_large(hipStream_t s, int prec, int columns, int max_positions, ResidentArgs a) {
    if (a.n_models <= 0) return;
    a.groups = (a.K + columns - 1) / columns;
    if (prec == MORAP_F32) {
        if (columns == 4) launch_big<float, 4>(s, a, max_positions);
        else if (columns == 2) launch_big<float, 2>(s, a, max_positions);
        else launch_big<float, 1>(s, a, max_positions);
    } else {
        if (columns == 2) launch_big<double, 2>(s, a, max_positions);
        else launch_big<double, 1>(s, a, max_positions);
    }
}

}  // namespace k
}  // namespace morap
