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
#include "resident.h"

#include <cfloat>
#include <type_traits>

namespace morap {
namespace k {

namespace {

// waves per SIMD the registers are held to, so that the probabilities of NS
// states fit with room for a step: 128 registers, 168 or 256
__host__ __device__ constexpr int res_waves_per_simd(int bytes, int ns, bool fast, bool rows) {
    const int need = ns * (bytes / 4) * (fast ? 2 : (rows ? 4 : 3));
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
// With INST an item is a (column, model) instance: FP64, its own two weights
// and stop, values contiguous.  With ROWS the product is given as rows, at most
// five a state of three entries each: these take the place of the block, an LDS
// row and a gather each, in the order given.  48 products of 16 x 16 grids x 8
// tasks, 24 FP32 columns: 0.35 ms; 0.50 streamed (see rows.hip) and 3.7 with the
// batched CSR sweeps.
template <class T, int KC, int NS, bool FAST, bool INST = false, bool ROWS = false>
__global__ void __launch_bounds__(RES_MAX_THREADS, res_waves_per_simd(sizeof(T), NS, FAST, ROWS))
resident_vi(ResidentArgs a) {
    constexpr uint32_t PAT = FAST ? PAT_GRID : PAT_DENSE;
    constexpr bool UC = FAST;                             // one cost per action
    constexpr int NNZ = ROWS ? 15 : pat_count(PAT);
    constexpr int ROWB = sizeof(T) * KC;                  // bytes of an LDS row
    constexpr int SH = ROWB == 4 ? 2 : (ROWB == 8 ? 3 : 4);
    constexpr int BUF = res_rows(NS) * ROWB;              // distance of the two buffers
    constexpr bool want_y = sizeof(T) == 4;               // |y| only bounds the FP32 stop test
    static_assert(BUF <= 65535, "the second buffer must lie within an LDS offset");
    extern __shared__ __align__(16) unsigned char lds[];

    const Item<T, KC, INST> it(a);
    if (!it.ok) return;
    const int m = it.m;
    bool on[KC];
    bool any = false;
#pragma unroll
    for (int c = 0; c < KC; ++c) {
        on[c] = it.running(a, c);
        any |= on[c];
    }
    if (!any) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
    const int sb = a.state_base[m], S = a.state_base[m + 1] - sb;
    unsigned char* hdr = lds + BUF + (((nw * 64 * NS + 1) * ROWB + 15) & ~15);
    T* part = reinterpret_cast<T*>(hdr);                               // [2][4 MAXW rows][4][res, |y|]
    // the stop-test wave's state per column, kept out of the registers of a sweep
    double* best = reinterpret_cast<double*>(hdr + 2 * 4 * MAXW * 8 * sizeof(T));       // [4] smallest change so far
    int* stall = reinterpret_cast<int*>(best + 4);                                      // [4] sweeps since it was set
    unsigned* flag = reinterpret_cast<unsigned*>(stall + 4);                            // [2] results of the stop test
    auto get = [&](int buf, unsigned addr) { return lds_get<T, KC>(addr + buf * BUF); };
    auto put = [&](int buf, unsigned addr, const Row<T, KC>& r) { lds_put<T, KC>(addr + buf * BUF, r); };

    // the record of every state (they are stored in tile order: each names
    // its state)
    int* where = reinterpret_cast<int*>(lds);
    if constexpr (!ROWS)
        for (int p = tid; p < S; p += blockDim.x) where[a.rec[(int64_t)(sb + p) * 8 + 7] - sb] = p;
    __syncthreads();
    T P[NS][NNZ], cost[UC ? 1 : NS][5], reward[ROWS ? NS : 1][5];
    unsigned succ[ROWS ? NS : 1][8];       // LDS rows of the entries, 16 bits each
    unsigned o01[NS], o23[NS], o4[NS];     // LDS rows of the slots, 16 bits each; o4: accepting slots above
    unsigned acc_steps = 0;                // steps in which a lane of this wave has an accepting slot
    const int own0 = wave * 64 * NS + lane + 1;   // LDS row of the first step's state; step i: + 64 i
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const int l = min(own0 - 1 + 64 * i, S - 1);
        if constexpr (ROWS) {
            const int64_t at = (int64_t)a.short_base[m] + l;
            const uint4* q = a.short_rec + at * 2;
            const uint4 q0 = q[0], q1 = q[1];
            const unsigned w[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) succ[i][e] = w[e];
            const T* B = static_cast<const T*>(a.short_val) + at * SHORT_VALUES;
#pragma unroll
            for (int e = 0; e < NNZ; ++e) P[i][e] = own_reg(B[e]);
#pragma unroll
            for (int e = 0; e < 5; ++e) {
                cost[i][e] = own_reg(B[15 + e]);
                reward[i][e] = own_reg(B[20 + e]);
            }
            continue;
        }
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
    for (int c = 0; c < KC; ++c) it.weights(a, c, wc[c], wp[c]);
    // every state of the product has the same action costs: w_c (-cost) once
    T first[UC ? KC : 1][5];
    if constexpr (UC) {
#pragma unroll
        for (int c = 0; c < KC; ++c)
#pragma unroll
            for (int q = 0; q < 5; ++q) first[c][q] = scalar(wc[c] * cost[0][q]);
    }
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        Row<T, KC> v;
#pragma unroll
        for (int c = 0; c < KC; ++c) v.v[c] = it.start(a, sb, min(own0 - 1 + 64 * i, S - 1), c);
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
    const bool stop_wave = wave == nw - 1;
    if (want_y && tid < KC && it.k0 + tid < a.K) {
        best[tid] = a.best_res[it.pair0 + tid];
        stall[tid] = a.stall[it.pair0 + tid];
    }
    unsigned live = 0;   // columns still running
#pragma unroll
    for (int c = 0; c < KC; ++c) live |= on[c] ? 1u << c : 0u;
    unsigned stop_live = live;   // the same, as the stop test has them (a sweep ahead)
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
        auto rows_backup = [&](int i) {
#pragma unroll
            for (int e = 0; e < 8; ++e) asm volatile("" : "+v"(succ[i][e]));   // (as above)
            const Row<T, KC> old = get(IN, (unsigned)(own0 + 64 * i) << SH);
            Row<T, KC> v[5];
#pragma unroll
            for (int q = 0; q < 5; ++q) {
#pragma unroll
                for (int c = 0; c < KC; ++c) v[q].v[c] = wc[c] * cost[i][q] + wp[c] * reward[i][q];
#pragma unroll
                for (int e = 3 * q; e < 3 * q + 3; ++e) {
                    const Row<T, KC> x = get(IN, e & 1 ? high_row<SH>(succ[i][e / 2]) : low_row<SH>(succ[i][e / 2]));
#pragma unroll
                    for (int c = 0; c < KC; ++c) v[q].v[c] = fma(P[i][e], x.v[c], v[q].v[c]);
                }
            }
            Row<T, KC> out;
#pragma unroll
            for (int c = 0; c < KC; ++c) {
                out.v[c] = max3(max3(v[0].v[c], v[1].v[c], v[2].v[c]), v[3].v[c], v[4].v[c]);
                r[c] = max_abs(r[c], out.v[c] - old.v[c]);
                if (want_y) y[c] = max_abs(y[c], out.v[c]);
            }
            put(1 - IN, (unsigned)(own0 + 64 * i) << SH, out);
        };
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            if constexpr (ROWS) {
                rows_backup(i);
                continue;
            }
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
        const T* p = part + CUR * 4 * MAXW * 8;
        const T rr = part_max(p, nw, 2, ln), yy = want_y ? part_max(p + 1, nw, 2, ln) : (T)0;
        // lane c < KC tests column c
        bool now = false;
        if (ln < KC && (stop_live >> ln & 1)) {
            bool floor_stop = false;
            now = it.stop(a, (double)rr, (double)yy, best[ln], stall[ln], floor_stop);
            if (now) {
                it.stopped(a, ln, n, floor_stop);
                // (a product with states has a live initial state)
                const int s_init = a.init[m] - sb + 1;
                if constexpr (!INST)
                    a.c[(int64_t)(it.k0 + ln) * a.M + m] =
                        (double)reinterpret_cast<const T*>(lds + CUR * BUF + ((unsigned)s_init << SH))[ln];
            }
        }
        const unsigned fresh = (unsigned)__ballot(now);
        stop_live &= ~fresh;
        if (ln == 0) flag[CUR] = fresh | (stop_live == 0 ? 0x100u : 0u);
    };

    // final (or, at the end of the launch, current) values of the columns in
    // `cols` from buffer `buf`, each thread its own states
    auto store = [&](void* x, int buf, unsigned cols) {
        int l = own0 - 1;
        asm volatile("" : "+v"(l));   // (as above: no addresses kept over the sweeps)
#pragma clang loop unroll(disable)
        for (int i = 0; i < NS && l < S; ++i, l += 64) {
            const Row<T, KC> v = get(buf, (unsigned)(l + 1) << SH);
#pragma unroll
            for (int c = 0; c < KC; ++c)
                if (cols >> c & 1) static_cast<T*>(x)[it.place(a, sb, l, c)] = v.v[c];
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
            store(a.x0, IN, f & 0xffu);
            live &= ~f;
        }
        if (f & 0x100u) return true;
        if (!more) {
            // the launch ends with columns running: their iterate, and after
            // the last launch of a solve the iterate before it
            store(a.x0, IN, live);
            if constexpr (!INST) {
                if (a.last) store(a.x1, 1 - IN, live);
                if (stop_wave && lane < KC && (live >> lane & 1)) {
                    const int64_t i = it.pair0 + lane;
                    if (want_y) {
                        a.best_res[i] = best[lane];
                        a.stall[i] = stall[lane];
                    }
                    if (a.last) a.active[i] = 1;
                }
            }
            return true;
        }
        if (stop_wave) decide(std::integral_constant<int, 1 - IN>{}, n);
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
// This kernel is FP64's beyond 2,560 states: two columns of the values, new ones in
// registers.  (48 products of 3,143 to 8,319 states, 37 columns: 2.7 ms here, 13.2
// with the batched sweeps.)
template <class T, int KC, int NS, bool INST = false>
__global__ void __launch_bounds__(BIG_THREADS)
resident_big(ResidentArgs a) {
    constexpr int ROWB = sizeof(T) * KC;
    constexpr int SH = ROWB == 4 ? 2 : (ROWB == 8 ? 3 : 4);
    constexpr int NW = BIG_THREADS / 64;
    extern __shared__ __align__(16) unsigned char lds[];

    const Item<T, KC, INST> it(a);
    if (!it.ok) return;
    const int m = it.m;
    unsigned live = 0;   // columns still running
#pragma unroll
    for (int c = 0; c < KC; ++c)
        if (it.running(a, c)) live |= 1u << c;
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
    unsigned* flag = reinterpret_cast<unsigned*>(hdr + 4 * NW * 8 * sizeof(T));
    auto get = [&](unsigned addr) { return lds_get<T, KC>(addr); };
    auto put = [&](unsigned addr, const Row<T, KC>& r) { lds_put<T, KC>(addr, r); };

    T wp[KC], first[KC][5];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
        T wc;
        it.weights(a, c, wc, wp[c]);
        // every state of the product has the same action costs
#pragma unroll
        for (int q = 0; q < 5; ++q) first[c][q] = wc * ablk[(int64_t)(blk[-s_begin] & 0x7fff) * GRID_BLK + GRID_NNZ + q];
    }
    const unsigned own0 = (unsigned)(s_begin * 64 + lane + 1) << SH;   // LDS row of the first step's state
    for (int i = 0; i < cnt; ++i) {
        const unsigned w = rec[i * 64].w & 0xffffu;
        Row<T, KC> v;
#pragma unroll
        for (int c = 0; c < KC; ++c) v.v[c] = it.start(a, sb, (int)w, c);
        put(own0 + ((unsigned)i << (6 + SH)), v);
    }
    if (tid == 0) {
        Row<T, KC> z;
#pragma unroll
        for (int c = 0; c < KC; ++c) z.v[c] = 0;
        put(0, z);
    }
    __syncthreads();

    // the values of the columns in `cols`, each thread its own states
    auto store = [&](void* x, unsigned cols) {
        unsigned own = own0;
        asm volatile("" : "+v"(own));   // (no addresses kept over the sweeps)
        for (int i = 0; i < cnt; ++i) {
            const unsigned w = rec[i * 64].w;
            const Row<T, KC> v = get(own + ((unsigned)i << (6 + SH)));
            if (w >> 31) continue;   // padding
#pragma unroll
            for (int c = 0; c < KC; ++c)
                if (cols >> c & 1) static_cast<T*>(x)[it.place(a, sb, (int)(w & 0xffffu), c)] = v.v[c];
        }
    };

    Row<T, KC> out[NS];
    for (int n = a.sweep0 + 1; n <= a.sweep1; ++n) {
        T r[KC];
#pragma unroll
        for (int c = 0; c < KC; ++c) r[c] = 0;
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
            const CVal B = ablk + (int64_t)(b & 0x7fff) * GRID_BLK;
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
                }
            };
            if (__ballot(accm != 0)) backup(std::true_type{});
            else backup(std::false_type{});
            q = qn;
            b = bn;
            }
        }
        const T rr = row_max<T, KC>(r);
        if ((lane & 15) < 4) part[((wave * 4 + (lane >> 4)) * 4 + (lane & 3)) * 2] = rr;
        // the iterate before the last, of a solve over its limit
        if (!INST && a.last && n == a.sweep1) store(a.x1, live);
        __syncthreads();   // every wave has read the old values
#pragma unroll
        for (int i = 0; i < NS; ++i)
            if (i < cnt) put(own0 + ((unsigned)i << (6 + SH)), out[i]);
        if (wave == NW - 1) {
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const T res_t = part_max(part, NW, 2, ln);
            bool now = false;
            if (ln < KC && (live >> ln & 1)) {
                double best = 0;   // (FP32's)
                int stall = 0;
                bool floor_stop = false;
                now = it.stop(a, (double)res_t, 0.0, best, stall, floor_stop);
                if (now) it.stopped(a, ln, n, floor_stop);
            }
            const unsigned fresh = (unsigned)__ballot(now);
            if (ln == 0) *flag = fresh;
        }
        __syncthreads();
        const unsigned f = *flag;
        if (f) {
            store(a.x0, f);
            if constexpr (!INST)
                if (tid < KC && (f >> tid & 1))
                    a.c[(int64_t)(it.k0 + tid) * a.M + m] =
                        (double)reinterpret_cast<const T*>(lds + ((unsigned)(a.big_init[m] + 1) << SH))[tid];
            live &= ~f;
            if (!live) return;
        }
    }
    // the launch ends with columns running: their iterate
    store(a.x0, live);
    if constexpr (!INST)
        if (a.last && tid < KC && (live >> tid & 1)) a.active[it.pair0 + tid] = 1;
}

// The same in FP32 with the sums on the matrix cores.  v_mfma_f32_4x4x1 takes
// one multiply-add of 16 independent 4 x 4 products: four actions' probabilities
// of a slot (the lanes of a block hold one action each) times the slot's values
// of four states (the lanes of a block hold one state each), so five of them add
// up the four moves of 64 states of one block in slot order, the same bits as 16
// multiply-adds, at 0.6 of their cycles and beside the vector ALU instead of on
// it.  A slot an action does not reach has probability 0 and adds nothing (no
// value overflows: the plan asks for costs within 1e25).  A lane loads its
// action's probabilities where a run of steps of one block begins, a few times
// a sweep; loading them at every step kept the address unit of the vector
// memory half busy, 40 of 78 cycles a step.
//
// 24 agents on 32 x 32 .. 128 x 128 grids x 32 tasks, 64 columns: 0.44 (1 column
// a workgroup), 0.59 (2) and 0.80 (4) 10^12 state-columns a second; with the
// sums on the vector ALU 0.28, 0.53 and 0.80, and 0.34 with the batched sweeps
// on all products of that problem.
using f32x4 = float __attribute__((ext_vector_type(4)));

template <int KC, int NS>
__global__ void __launch_bounds__(BIG_THREADS) big_mfma(ResidentArgs a) {
    constexpr int ROWB = 4 * KC, SH = ROWB == 4 ? 2 : (ROWB == 8 ? 3 : 4);
    constexpr int NW = BIG_THREADS / 64;
    extern __shared__ __align__(16) unsigned char lds[];

    const Item<float, KC, false> it(a);
    if (!it.ok) return;
    const int m = it.m;
    unsigned live = 0;   // columns still running
#pragma unroll
    for (int c = 0; c < KC; ++c)
        if (it.running(a, c)) live |= 1u << c;
    if (!live) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sb = a.state_base[m];
    const int pos0 = a.big_base[m], n_steps = (a.big_base[m + 1] - pos0) >> 6;
    const int s_begin = wave * n_steps / NW, cnt = (wave + 1) * n_steps / NW - s_begin;
    using CVal = const __attribute__((address_space(4))) float*;
    const CVal ablk = (CVal)(static_cast<const float*>(a.grid_blk));
    const char* rec = reinterpret_cast<const char*>(a.big_rec + pos0 + s_begin * 64);
    unsigned char* hdr = lds + (((n_steps * 64 + 1) * ROWB + 15) & ~15);
    float* part = reinterpret_cast<float*>(hdr);                                 // [4 NW rows][4][res, |y|]
    double* best = reinterpret_cast<double*>(hdr + 4 * NW * 8 * sizeof(float));  // [4] smallest change so far
    int* stall = reinterpret_cast<int*>(best + 4);                               // [4] sweeps since it was set
    unsigned* flag = reinterpret_cast<unsigned*>(stall + 4);
    auto get = [&](unsigned addr) { return lds_get<float, KC>(addr); };
    auto put = [&](unsigned addr, const Row<float, KC>& r) { lds_put<float, KC>(addr, r); };

    float wp[KC], stay0[KC];
    f32x4 first[KC];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
        float wc;
        it.weights(a, c, wc, wp[c]);
        // every state of the product has the same action costs
        const CVal cost = ablk + (int64_t)(a.big_block[pos0 >> 6] & 0x7fff) * GRID_BLK + GRID_NNZ;
#pragma unroll
        for (int q = 0; q < 4; ++q) first[c][q] = wc * cost[q];
        stay0[c] = scalar(wc * cost[4]);
    }
    const unsigned own0 = (unsigned)(s_begin * 64 + lane + 1) << SH;   // LDS row of the first step's state
    auto state_word = [&](int i) { return reinterpret_cast<const uint4*>(rec)[i * 64 + lane].w; };
    for (int i = 0; i < cnt; ++i) {
        const unsigned w = state_word(i) & 0xffffu;
        Row<float, KC> v;
#pragma unroll
        for (int c = 0; c < KC; ++c) v.v[c] = it.start(a, sb, (int)w, c);
        put(own0 + ((unsigned)i << (6 + SH)), v);
    }
    if (tid == 0) {
        Row<float, KC> z;
#pragma unroll
        for (int c = 0; c < KC; ++c) z.v[c] = 0;
        put(0, z);
    }
    if (tid < KC && it.k0 + tid < a.K) {
        best[tid] = a.best_res[it.pair0 + tid];
        stall[tid] = a.stall[it.pair0 + tid];
    }
    __syncthreads();

    // the values of the columns in `cols`, each thread its own states
    auto store = [&](void* x, unsigned cols) {
        unsigned own = own0;
        asm volatile("" : "+v"(own));   // (no addresses kept over the sweeps)
        for (int i = 0; i < cnt; ++i) {
            const unsigned w = state_word(i);
            const Row<float, KC> v = get(own + ((unsigned)i << (6 + SH)));
            if (w >> 31) continue;   // padding
#pragma unroll
            for (int c = 0; c < KC; ++c)
                if (cols >> c & 1) static_cast<float*>(x)[it.place(a, sb, (int)(w & 0xffffu), c)] = v.v[c];
        }
    };
    // this lane's action of a block: five slots, the probability to stay
    struct Move {
        f32x4 p;
        float2 q;
    };
    const float* mat = a.grid_mat + (lane & 3) * 8;
    using CInt = const __attribute__((address_space(4))) int32_t*;
    const CInt runs = (CInt)(a.big_block + (pos0 >> 6));

    Row<float, KC> out[NS];
    for (int n = a.sweep0 + 1; n <= a.sweep1; ++n) {
        float r[KC], y[KC];
#pragma unroll
        for (int c = 0; c < KC; ++c) r[c] = y[c] = 0;
        unsigned at = (unsigned)lane * 16;
        asm volatile("" : "+v"(at));   // (no addresses kept over the sweeps)
        // one step and, inside its condition, the next: the registers of what is
        // on its way are renamed from step to step, not copied
        Move mv;
        int run_end = 0;   // first step of the next run of one block
        int k = cnt;
        asm volatile("" : "+s"(k));    // (nor a condition per step)
        // (never past this wave's last step: what follows may be another product's,
        // naming rows that this workgroup's LDS does not have)
        auto record = [&](int i) { return *reinterpret_cast<const uint3*>(rec + min(i, k - 1) * 1024 + at); };
        struct Slots {
            Row<float, KC> v[NSLOT];
        };
        auto gather = [&](const uint3& q) {
            Slots x;
            x.v[0] = get(low_row<SH>(q.x));
            x.v[1] = get(high_row<SH>(q.x));
            x.v[2] = get(low_row<SH>(q.y));
            x.v[3] = get(high_row<SH>(q.y));
            x.v[4] = get(low_row<SH>(q.z));
            return x;
        };
        // (with one or two columns the next step's values are on their way too)
        constexpr bool early = KC < 4;
        auto steps = [&](auto self, auto I, const uint3& q, const uint3& qn, const Slots& x) {
            constexpr int i = decltype(I)::value;
            if (i >= k) return;
            const uint3 q2 = record(i + 2);   // two steps ahead
            Slots xn;
            if constexpr (early) xn = gather(qn);   // (past the last step: its own rows again, not used)
            if (i == run_end) {
                const int run = runs[s_begin + i];
                run_end = (run >> 16) - s_begin;
                const float* b = mat + (run & 0x7fff) * 32;
                mv = Move{*reinterpret_cast<const f32x4*>(b), *reinterpret_cast<const float2*>(b + 4)};
                // (waited for here: the steps without a load wait for less)
                asm volatile("" : "+v"(mv.p), "+v"(mv.q.x), "+v"(mv.q.y));
            }
            const Slots now = early ? x : gather(q);
            const Row<float, KC>(&xv)[NSLOT] = now.v;
            auto slot = [&](int d) { return d < 4 ? mv.p[d] : mv.q.x; };
            constexpr int H = KC == 4 ? 2 : KC;   // columns at a time (registers)
            auto backup = [&](int c0, const f32x4 (&start)[H], const float (&start4)[H]) {
                f32x4 v[H];
                float v4[H];
#pragma unroll
                for (int d = 0; d < NSLOT; ++d)
#pragma unroll
                    for (int c = 0; c < H; ++c)
                        v[c] = __builtin_amdgcn_mfma_f32_4x4x1f32(slot(d), xv[d].v[c0 + c], d == 0 ? start[c] : v[c], 0, 0, 0);
#pragma unroll
                for (int c = 0; c < H; ++c) v4[c] = fma(mv.q.y, xv[0].v[c0 + c], start4[c]);
                // (the maxima below are asm, whose reads of matrix results the
                // compiler does not space)
                if constexpr (H == 2) asm volatile("s_nop 7\n\ts_nop 7" : "+v"(v[0]), "+v"(v[1]));
                else asm volatile("s_nop 7\n\ts_nop 7" : "+v"(v[0]));
#pragma unroll
                for (int c = 0; c < H; ++c) {
                    const float best_v = max3(max3(v[c][0], v[c][1], v[c][2]), v[c][3], v4[c]);
                    out[i].v[c0 + c] = best_v;
                    r[c0 + c] = max_abs(r[c0 + c], best_v - xv[0].v[c0 + c]);   // slot 0 is the state itself
                    y[c0 + c] = max_abs(y[c0 + c], best_v);
                }
            };
            const unsigned accm = q.z >> 16;
            const bool accepts = __ballot(accm != 0) != 0;
            // probability reward: the action's mass on accepting slots
            f32x4 mass = {0.f, 0.f, 0.f, 0.f};
            if (accepts)
#pragma unroll
                for (int d = 0; d < NSLOT; ++d)
                    mass = __builtin_amdgcn_mfma_f32_4x4x1f32(slot(d), accm >> d & 1 ? 1.f : 0.f, mass, 0, 0, 0);
#pragma unroll
            for (int c0 = 0; c0 < KC; c0 += H) {
                f32x4 start[H];
                float start4[H];
#pragma unroll
                for (int c = 0; c < H; ++c) {
                    start[c] = first[c0 + c];
                    start4[c] = stay0[c0 + c];
                }
                if (accepts) {
                    const float mass4 = accm & 1 ? mv.q.y : 0.f;
#pragma unroll
                    for (int c = 0; c < H; ++c) {
#pragma unroll
                        for (int act = 0; act < 4; ++act) start[c][act] = fma(wp[c0 + c], mass[act], start[c][act]);
                        start4[c] = fma(wp[c0 + c], mass4, start4[c]);
                    }
                    backup(c0, start, start4);
                } else {
                    backup(c0, start, start4);
                }
            }
            if constexpr (i + 1 < NS) self(self, std::integral_constant<int, i + 1>{}, qn, q2, xn);
        };
        if (k > 0) {
            const uint3 q = record(0), qn = record(1);
            Slots x;
            if constexpr (early) x = gather(q);
            steps(steps, std::integral_constant<int, 0>{}, q, qn, x);
        }
        const float rr = row_max<float, KC>(r), yy = row_max<float, KC>(y);
        if ((lane & 15) < 4) {
            float* p = part + ((wave * 4 + (lane >> 4)) * 4 + (lane & 3)) * 2;
            p[0] = rr;
            p[1] = yy;
        }
        // the iterate before the last, of a solve over its limit
        if (a.last && n == a.sweep1) store(a.x1, live);
        __syncthreads();   // every wave has read the old values
#pragma unroll
        for (int i = 0; i < NS; ++i)
            if (i < k) put(own0 + ((unsigned)i << (6 + SH)), out[i]);
        if (wave == NW - 1) {
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const float res_t = part_max(part, NW, 2, ln), y_t = part_max(part + 1, NW, 2, ln);
            bool now = false;
            if (ln < KC && (live >> ln & 1)) {
                bool floor_stop = false;
                now = it.stop(a, (double)res_t, (double)y_t, best[ln], stall[ln], floor_stop);
                if (now) it.stopped(a, ln, n, floor_stop);
            }
            const unsigned fresh = (unsigned)__ballot(now);
            if (ln == 0) *flag = fresh;
        }
        __syncthreads();
        const unsigned f = *flag;
        if (f) {
            store(a.x0, f);
            if (tid < KC && (f >> tid & 1))
                a.c[(int64_t)(it.k0 + tid) * a.M + m] =
                    (double)reinterpret_cast<const float*>(lds + ((unsigned)(a.big_init[m] + 1) << SH))[tid];
            live &= ~f;
            if (!live) return;
        }
    }
    // the launch ends with columns running: their iterate
    store(a.x0, live);
    if (tid < KC && (live >> tid & 1)) {
        const int64_t i = it.pair0 + tid;
        a.best_res[i] = best[tid];
        a.stall[i] = stall[tid];
        if (a.last) a.active[i] = 1;
    }
}

// ---------------------------------------------------------------------------
// dispatch
// ---------------------------------------------------------------------------
// States a workgroup can hold: 512 per register step.  The grid pattern with
// one cost per action needs 17 probabilities a state (7 steps in FP32, 5 in
// FP64 within 256 registers), the general block 25 and 5 costs (4 and 2).  A
// fifth FP64 step leaves room for one column (with two it spills 204 bytes):
// 37 columns of products of up to 2,380 states take 2.2 ms so, 2.75 with two
// columns in the larger products' kernel, and an assigned pair's solve at 2,400
// states 0.22 ms, 0.47 there.
static int resident_steps(int prec, bool fast) {
    return prec == MORAP_F32 ? (fast ? 7 : 4) : (fast ? 5 : 2);
}

bool has_grid_pattern(uint32_t union_pattern) { return pattern_for(union_pattern) == PAT_GRID; }

int resident_capacity(int prec, bool fast) {
    return res_rows(resident_steps(prec, fast)) - 1;
}

namespace {

template <class T, int KC, int NS, bool FAST, bool INST, bool ROWS>
void launch_res(hipStream_t s, const ResidentArgs& a, int max_states) {
    auto* fn = &resident_vi<T, KC, NS, FAST, INST, ROWS>;
    constexpr int ROWB = sizeof(T) * KC;
    const int threads = 64 * ((max_states + 64 * NS - 1) / (64 * NS));
    const size_t bytes = (size_t)res_rows(NS) * ROWB + (((size_t)(threads * NS + 1) * ROWB + 15) & ~(size_t)15) +
                         2 * 4 * MAXW * 8 * sizeof(T) + 64;
    MORAP_CHECK(threads <= RES_MAX_THREADS && max_states < res_rows(NS) && bytes <= LDS_BYTES, MORAP_E_UNSUPPORTED,
                "a product does not fit the LDS-resident iteration");
    static OncePerDevice granted;
    grant_lds(granted, fn);
    const unsigned blocks = INST ? (unsigned)a.n_models : 8u * (unsigned)((a.n_models + 7) / 8) * (unsigned)a.groups;
    hipLaunchKernelGGL(fn, dim3(blocks), dim3((unsigned)threads), bytes, s, a);
    MORAP_HIP(hipGetLastError());
}

template <class T, int KC, bool FAST, int MAXNS, bool INST = false, bool ROWS = false>
void launch_steps(hipStream_t s, const ResidentArgs& a, int ns, int max_states) {
    if (ns == 1) return launch_res<T, KC, 1, FAST, INST, ROWS>(s, a, max_states);
    if constexpr (MAXNS >= 2)
        if (ns == 2) return launch_res<T, KC, 2, FAST, INST, ROWS>(s, a, max_states);
    if constexpr (MAXNS >= 3)
        if (ns == 3) return launch_res<T, KC, 3, FAST, INST, ROWS>(s, a, max_states);
    if constexpr (MAXNS >= 4)
        if (ns == 4) return launch_res<T, KC, 4, FAST, INST, ROWS>(s, a, max_states);
    if constexpr (MAXNS >= 5)
        if (ns == 5) return launch_res<T, KC, 5, FAST, INST, ROWS>(s, a, max_states);
    if constexpr (MAXNS >= 7)
        if (ns == 7) return launch_res<T, KC, 7, FAST, INST, ROWS>(s, a, max_states);
    fail(MORAP_E_UNSUPPORTED, "a product does not fit the LDS-resident iteration");
}

}  // namespace

int resident_class(int states) {
    const int ns = (states + RES_MAX_THREADS - 1) / RES_MAX_THREADS;
    return ns <= 5 ? (ns < 1 ? 1 : ns) : 7;
}

// Columns per workgroup of the first kernel: a group, or one where the solve has
// fewer columns than a group (24 x 30 products of 32 x 32 grids, FP32: two
// columns take 0.49 ms one by one, 0.74 as half a group).
static int first_columns(int prec, bool wide, const ResidentArgs& a) {
    const int kc = prec == MORAP_F32 ? 4 : 2;
    return wide && kc <= a.Kp ? kc : 1;
}

void resident(hipStream_t s, int prec, bool fast, bool wide, int max_states, ResidentArgs a) {
    if (a.n_models <= 0) return;
    const int ns = resident_class(max_states);
    if (prec != MORAP_F32 && ns == 5) wide = false;   // (see resident_steps)
    const int kc = first_columns(prec, wide, a);
    wide = kc > 1;
    a.groups = (a.K + kc - 1) / kc;
    if (prec == MORAP_F32) {
        if (fast && wide) launch_steps<float, 4, true, 7>(s, a, ns, max_states);
        else if (fast) launch_steps<float, 1, true, 7>(s, a, ns, max_states);
        else if (wide) launch_steps<float, 4, false, 4>(s, a, ns, max_states);
        else launch_steps<float, 1, false, 4>(s, a, ns, max_states);
    } else {
        if (fast && wide) launch_steps<double, 2, true, 4>(s, a, ns, max_states);
        else if (fast) launch_steps<double, 1, true, 5>(s, a, ns, max_states);
        else if (wide) launch_steps<double, 2, false, 2>(s, a, ns, max_states);
        else launch_steps<double, 1, false, 2>(s, a, ns, max_states);
    }
}

void resident_short(hipStream_t s, int prec, bool wide, int max_states, ResidentArgs a) {
    if (a.n_models <= 0) return;
    const int ns = resident_class(max_states);
    const int kc = first_columns(prec, wide, a);
    wide = kc > 1;
    a.groups = (a.K + kc - 1) / kc;
    if (prec == MORAP_F32) {
        if (wide) launch_steps<float, 4, false, 4, false, true>(s, a, ns, max_states);
        else launch_steps<float, 1, false, 4, false, true>(s, a, ns, max_states);
    } else {
        if (wide) launch_steps<double, 2, false, 2, false, true>(s, a, ns, max_states);
        else launch_steps<double, 1, false, 2, false, true>(s, a, ns, max_states);
    }
}

void resident_inst(hipStream_t s, bool fast, int max_states, ResidentArgs a) {
    if (a.n_models <= 0) return;
    const int ns = resident_class(max_states);
    a.groups = 1;
    if (fast) launch_steps<double, 1, true, 5, true>(s, a, ns, max_states);
    else launch_steps<double, 1, false, 2, true>(s, a, ns, max_states);
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

template <class T, int KC, bool INST = false>
void launch_big(hipStream_t s, const ResidentArgs& a, int max_positions) {
    constexpr int NS = 160 / (sizeof(T) * KC);
    void (*fn)(ResidentArgs);
    if constexpr (sizeof(T) == 4) fn = &big_mfma<KC, NS>;
    else fn = &resident_big<T, KC, NS, INST>;
    const size_t bytes = (((size_t)max_positions + 1) * sizeof(T) * KC + 15) / 16 * 16 +
                         4 * (BIG_THREADS / 64) * 8 * sizeof(T) + 64;
    MORAP_CHECK(max_positions % 64 == 0 && bytes <= LDS_BYTES && max_positions <= BIG_THREADS * NS,
                MORAP_E_UNSUPPORTED, "a product does not fit the LDS-resident iteration");
    static OncePerDevice granted;
    grant_lds(granted, fn);
    const unsigned blocks = INST ? (unsigned)a.n_models : 8u * (unsigned)((a.n_models + 7) / 8) * (unsigned)a.groups;
    hipLaunchKernelGGL(fn, dim3(blocks), dim3(BIG_THREADS), bytes, s, a);
    MORAP_HIP(hipGetLastError());
}

}  // namespace

void resident_large(hipStream_t s, int prec, int columns, int max_positions, ResidentArgs a) {
    if (a.n_models <= 0) return;
    columns = std::min(columns, a.Kp);
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

void resident_inst_large(hipStream_t s, int max_positions, ResidentArgs a) {
    if (a.n_models <= 0) return;
    a.groups = 1;
    launch_big<double, 1, true>(s, a, max_positions);
}

}  // namespace k
}  // namespace morap
