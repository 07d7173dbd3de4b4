// Instances (a column and the model a task is assigned to) after the value
// iteration: the policy of each from its final values, and the fixed-policy
// evaluation of both objectives (Alg. 4), one workgroup per instance with
// what its iterations read and write in LDS.  Instances share nothing, so an
// attractor round or an evaluation sweep costs a barrier instead of a launch
// over all instances, the stop test of all and a look from the host.
//
// 64 columns of 10 x 20 products (1,280 instances of 340 .. 2,400 states): the
// launches side by side, up to 0.19 ms of values, 0.27 of policies and 0.22 of
// evaluation, 0.86 ms in all, where the tiled launches took 6.4 ms.
#include "common.h"
#include "kern.h"
#include "resident.h"

#include <cfloat>
#include <climits>

namespace morap {
namespace k {

// ---------------------------------------------------------------------------
// policies
// ---------------------------------------------------------------------------
// The tau-optimal actions of every state at the instance's values, the ranks
// of the attractor they span (distances to done, relaxed in place to the
// fixed point), and the action choice: among the optimal actions that move
// mass into done or to a lower rank the one that moves most (masses within
// 1e-12 are equal; then the first).  States left unranked get a ten times
// wider tolerance, up to six times, while ranked ones keep their choice and
// are sources at the largest rank so far.  A state lives in one 16-byte LDS
// word: the rows of its slots, the slots its optimal actions reach, those
// actions, and its rank.
// Bound by the latency of the relaxation rounds (one barrier each).
constexpr int POLICY_THREADS = 512;

__global__ void __launch_bounds__(POLICY_THREADS) inst_policy_kernel(InstanceArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];
    uint4* st = reinterpret_cast<uint4*>(lds);
    __shared__ int s_top, s_left;
    const int q = a.order[blockIdx.x], tid = threadIdx.x;
    const int m = a.inst_model[q];
    const int sb = a.state_base[m], S = a.state_base[m + 1] - sb;
    const double* x = a.xi + a.inst_base[q];
    int8_t* mu = a.mu + a.inst_base[q];
    const double w0 = a.iwc[q], w1 = a.iwp[q];
    double tau = a.tau;
    int base = 0, rounds = 0;
    for (int widen = 0;; ++widen) {
        for (int p = tid; p < S; p += POLICY_THREADS) {
            const int32_t* r = a.rec + (int64_t)(sb + p) * 8;
            const int4 r0 = *reinterpret_cast<const int4*>(r), r1 = *reinterpret_cast<const int4*>(r + 4);
            const int own = r1.w - sb;
            if (widen > 0 && (int)st[own].w >= 0) continue;
            const int sc[NSLOT] = {r0.x, r0.y, r0.z, r0.w, r1.x};
            const double* B = a.ablk + (int64_t)r1.y * BLK;
            const unsigned accm = (unsigned)r1.z & 31u, enabled = (unsigned)(r1.z >> 8) & 31u;
            double xv[NSLOT];
            unsigned alive = 0;
#pragma unroll
            for (int d = 0; d < NSLOT; ++d) {
                xv[d] = sc[d] == a.zero_row ? 0.0 : x[sc[d] - sb];
                alive |= sc[d] == a.zero_row ? 0u : 1u << d;
            }
            double Q[5], qmax = -INFINITY;
            unsigned reach[5];   // slots the action moves mass to
#pragma unroll
            for (int act = 0; act < 5; ++act) {
                double v = w0 * B[25 + act], rp = 0.0;
                reach[act] = 0;
#pragma unroll
                for (int d = 0; d < NSLOT; ++d) {
                    const double pr = B[act * NSLOT + d];
                    if (accm >> d & 1) rp += pr;
                    reach[act] |= pr != 0.0 ? 1u << d : 0u;
                }
                if (accm) v = fma(w1, rp, v);
#pragma unroll
                for (int d = 0; d < NSLOT; ++d) v = fma(B[act * NSLOT + d], xv[d], v);
                Q[act] = v;
                if (enabled >> act & 1) qmax = fmax(qmax, v);
            }
            unsigned opt = 0, to = 0;
#pragma unroll
            for (int act = 0; act < 5; ++act)
                if ((enabled >> act & 1) && Q[act] >= qmax - tau) {
                    opt |= 1u << act;
                    to |= reach[act];
                }
            auto row = [&](int d) { return (alive >> d & 1) ? (unsigned)(sc[d] - sb) : 0u; };
            st[own] = make_uint4(row(0) | row(1) << 16, row(2) | row(3) << 16,
                                 row(4) | (to & alive) << 16 | ((to & ~alive) ? 1u << 21 : 0u) | opt << 22, 0xffffffffu);
        }
        if (tid == 0) s_top = s_left = 0;
        __syncthreads();
        // ranks to their fixed point: they only fall, so any order of updates
        // ends at the exact distances
        auto rank_of = [&](unsigned l) {
            return __hip_atomic_load(reinterpret_cast<const int*>(&st[l].w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        };
        int changed;
        do {
            changed = 0;
            for (int it = 0; it < 4; ++it)   // several passes a barrier: most updates are seen without it
                for (int l = tid; l < S; l += POLICY_THREADS) {
                    const uint4 e = st[l];
                    const int cur = (int)e.w;
                    if (cur >= 0 && cur <= base) continue;   // ranked in an earlier phase
                    int cand = (e.z >> 21 & 1) ? base + 1 : INT_MAX;
                    const unsigned rows[NSLOT] = {e.x & 0xffffu, e.x >> 16, e.y & 0xffffu, e.y >> 16, e.z & 0xffffu};
#pragma unroll
                    for (int d = 0; d < NSLOT; ++d)
                        if (e.z >> (16 + d) & 1) {
                            const int rk = rank_of(rows[d]);
                            if (rk >= 0) cand = min(cand, max(rk, base) + 1);
                        }
                    if (cand != INT_MAX && (cur < 0 || cand < cur)) {
                        __hip_atomic_store(reinterpret_cast<int*>(&st[l].w), cand, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                        changed = 1;
                    }
                }
            rounds += 4;
        } while (__syncthreads_or(changed));
        int top = 0, left = 0;
        for (int p = tid; p < S; p += POLICY_THREADS) {
            const int32_t* r = a.rec + (int64_t)(sb + p) * 8;
            const int4 r0 = *reinterpret_cast<const int4*>(r), r1 = *reinterpret_cast<const int4*>(r + 4);
            const int own = r1.w - sb;
            const uint4 e = st[own];
            const int level = (int)e.w;
            if (level < 0) {
                ++left;
                mu[own] = -1;
            }
            if (level <= base) continue;
            top = max(top, level);
            const int sc[NSLOT] = {r0.x, r0.y, r0.z, r0.w, r1.x};
            const double* B = a.ablk + (int64_t)r1.y * BLK;
            const unsigned enabled = (unsigned)(r1.z >> 8) & 31u, opt = e.z >> 22 & 31u;
            unsigned alive = 0, lower = 0;
#pragma unroll
            for (int d = 0; d < NSLOT; ++d)
                if (sc[d] != a.zero_row) {
                    alive |= 1u << d;
                    const int rk = (int)st[sc[d] - sb].w;
                    lower |= rk >= 0 && rk < level ? 1u << d : 0u;
                }
            int best_row = -1;
            double best_m = -1.0;
#pragma unroll
            for (int act = 0; act < 5; ++act) {
                if (!(opt >> act & 1)) continue;
                double live = 0.0, down = 0.0;
                bool done = false, hit = false;
#pragma unroll
                for (int d = 0; d < NSLOT; ++d) {
                    const double pr = B[act * NSLOT + d];
                    if (pr == 0.0) continue;
                    if (alive >> d & 1) live += pr;
                    else done = true;
                    if (lower >> d & 1) {
                        hit = true;
                        down += pr;
                    }
                }
                const double mass = (done ? 1.0 - live : 0.0) + down;
                if ((done || hit) && mass > best_m + 1e-12) {
                    best_m = mass;
                    best_row = __popc(enabled & ((1u << act) - 1u));   // rows are the enabled actions
                }
            }
            mu[own] = (int8_t)best_row;
        }
        if (top) atomicMax(&s_top, top);
        if (left) atomicAdd(&s_left, left);
        __syncthreads();
        base = max(base, s_top);
        const int unranked = s_left;
        if (unranked == 0 || widen == a.widenings) {
            if (tid == 0) {
                if (unranked) atomicAdd((unsigned long long*)&a.counters[0], (unsigned long long)unranked);
                atomicMax((unsigned long long*)&a.counters[1], (unsigned long long)rounds);
            }
            return;
        }
        tau *= 10.0;
        __syncthreads();   // (s_top and s_left are cleared in the next phase)
    }
}

// (1 KB aside for the workgroup's own reductions)
int policy_capacity() { return (int)((LDS_BYTES - 1024) / sizeof(uint4)); }

void inst_policy(hipStream_t s, int max_states, const InstanceArgs& a) {
    if (a.n <= 0) return;
    MORAP_CHECK(max_states <= policy_capacity(), MORAP_E_UNSUPPORTED, "an instance does not fit the policy kernel");
    static OncePerDevice granted;
    grant_lds(granted, &inst_policy_kernel, LDS_BYTES - 1024);
    hipLaunchKernelGGL(inst_policy_kernel, dim3((unsigned)a.n), dim3(POLICY_THREADS), (size_t)max_states * sizeof(uint4), s,
                       a);
    MORAP_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------
// evaluation
// ---------------------------------------------------------------------------
namespace {

// start of state l: the last evaluation's values of the same pair, with
// `from_values` the values its policy was chosen from (as eval_start_kernel)
struct EvalStart {
    double wc, wp;
    const double *xi, *prev;
    bool from_values;
    __device__ EvalStart(const InstanceArgs& a, int q)
        : wc(a.iwc[q]), wp(a.iwp[q]), xi(a.xi + a.inst_base[q]),
          prev(a.prev_src && a.prev_src[q] >= 0 ? a.xe_prev + 2 * a.prev_src[q] : nullptr), from_values(a.from_values != 0) {}
    __device__ __forceinline__ Row<double, 2> at(int l) const {
        Row<double, 2> v;
        v.v[0] = prev ? prev[2 * l] : 0.0;
        v.v[1] = prev ? prev[2 * l + 1] : (from_values ? 1.0 : 0.0);
        if (from_values && wc >= 1e-3) v.v[0] = (xi[l] - wp * v.v[1]) / wc;
        return v;
    }
};

// the chosen action's row of a state: its probabilities per slot, its cost
// and the mass it puts on accepting slots
__device__ __forceinline__ void policy_row(const InstanceArgs& a, const int4& r1, int mu, double (&P)[NSLOT], double& c,
                                           double& acc) {
    unsigned on = (unsigned)(r1.z >> 8) & 31u;
    for (int k = mu; k > 0; --k) on &= on - 1;   // the mu-th enabled action
    const int act = on ? __builtin_ctz(on) : 0;
    const double* B = a.ablk + (int64_t)r1.y * BLK;
    const unsigned accm = (unsigned)r1.z & 31u;
    c = B[25 + act];
    acc = 0.0;
#pragma unroll
    for (int d = 0; d < NSLOT; ++d) {
        P[d] = B[act * NSLOT + d];
        if (accm >> d & 1) acc += P[d];
    }
}

}  // namespace

// Products of up to 512 NS states: both iterates in LDS, NS states' chosen rows
// in the registers of every thread; the scheme of sweeps, stop test (per
// objective, one sweep behind) and final values is the value iteration's.
template <int NS>
__global__ void __launch_bounds__(RES_MAX_THREADS, NS <= 4 ? 4 : 2) eval_resident(InstanceArgs a) {
    constexpr int BUF = res_rows(NS) * 16;
    static_assert(BUF <= 65535, "the second buffer must lie within an LDS offset");
    extern __shared__ __align__(16) unsigned char lds[];
    const int q = a.order[blockIdx.x];
    unsigned live = (a.sweeps[2 * q] == 0 ? 1u : 0u) | (a.sweeps[2 * q + 1] == 0 ? 2u : 0u);
    if (!live) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
    const int m = a.inst_model[q];
    const int sb = a.state_base[m], S = a.state_base[m + 1] - sb;
    const int64_t ib = a.inst_base[q];
    unsigned char* hdr = lds + BUF + (nw * 64 * NS + 1) * 16;
    double* part = reinterpret_cast<double*>(hdr);                        // [2][4 MAXW rows][4]
    unsigned* flag = reinterpret_cast<unsigned*>(hdr + 2 * 4 * MAXW * 4 * 8);   // [2]

    int* where = reinterpret_cast<int*>(lds);
    for (int p = tid; p < S; p += blockDim.x) where[a.rec[(int64_t)(sb + p) * 8 + 7] - sb] = p;
    __syncthreads();
    const int own0 = wave * 64 * NS + lane + 1;   // LDS row of the first step's state; step i: + 64 i
    double P[NS][NSLOT], c0[NS], c1[NS];
    unsigned o01[NS], o23[NS], o4[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const int l = min(own0 - 1 + 64 * i, S - 1);
        const int32_t* r = a.rec + (int64_t)(sb + where[l]) * 8;
        const int4 r0 = *reinterpret_cast<const int4*>(r), r1 = *reinterpret_cast<const int4*>(r + 4);
        auto place = [&](int s) { return s == a.zero_row ? 0u : (unsigned)(s - sb + 1); };
        o01[i] = place(r0.x) | place(r0.y) << 16;
        o23[i] = place(r0.z) | place(r0.w) << 16;
        o4[i] = place(r1.x);
        policy_row(a, r1, a.mu[ib + l], P[i], c0[i], c1[i]);
    }
    __syncthreads();   // the buffers take the values now
    {
        const EvalStart start(a, q);
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const int l = min(own0 - 1 + 64 * i, S - 1);
            Row<double, 2> v;
            if (a.sweep0 > 0) {
                v.v[0] = a.xe[2 * (ib + l)];
                v.v[1] = a.xe[2 * (ib + l) + 1];
            } else {
                v = start.at(l);
            }
            lds_put<double, 2>((unsigned)(own0 + 64 * i) << 4, v);
        }
    }
    if (tid == 0) {
        const Row<double, 2> z = {{0.0, 0.0}};
        lds_put<double, 2>(0, z);
        lds_put<double, 2>(BUF, z);
        flag[0] = flag[1] = 0;
    }
    const bool stop_wave = wave == nw - 1;
    unsigned stop_live = live;
    __syncthreads();

    auto sweep = [&](auto PAR) {
        constexpr int IN = decltype(PAR)::value;
        double r[2] = {0.0, 0.0};
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            asm volatile("" : "+v"(o01[i]), "+v"(o23[i]), "+v"(o4[i]));   // (unpacked anew every sweep)
            Row<double, 2> xv[NSLOT];
            xv[0] = lds_get<double, 2>(low_row<4>(o01[i]) + IN * BUF);
            xv[1] = lds_get<double, 2>(high_row<4>(o01[i]) + IN * BUF);
            xv[2] = lds_get<double, 2>(low_row<4>(o23[i]) + IN * BUF);
            xv[3] = lds_get<double, 2>(high_row<4>(o23[i]) + IN * BUF);
            xv[4] = lds_get<double, 2>(low_row<4>(o4[i]) + IN * BUF);
            const Row<double, 2> old = lds_get<double, 2>(((unsigned)(own0 + 64 * i) << 4) + IN * BUF);
            Row<double, 2> v = {{c0[i], c1[i]}};
#pragma unroll
            for (int d = 0; d < NSLOT; ++d) {
                v.v[0] = fma(P[i][d], xv[d].v[0], v.v[0]);
                v.v[1] = fma(P[i][d], xv[d].v[1], v.v[1]);
            }
            r[0] = max_abs(r[0], v.v[0] - old.v[0]);
            r[1] = max_abs(r[1], v.v[1] - old.v[1]);
            lds_put<double, 2>(((unsigned)(own0 + 64 * i) << 4) + (1 - IN) * BUF, v);
        }
        const double rr = row_max<double, 2>(r);
        if ((lane & 15) < 4) part[((1 - IN) * 4 * MAXW + wave * 4 + (lane >> 4)) * 4 + (lane & 3)] = rr;
    };
    auto store = [&](int buf, unsigned cols) {
        int l = own0 - 1;
        asm volatile("" : "+v"(l));
#pragma clang loop unroll(disable)
        for (int i = 0; i < NS && l < S; ++i, l += 64) {
            const Row<double, 2> v = lds_get<double, 2>(((unsigned)(l + 1) << 4) + buf * BUF);
            if (cols & 1) a.xe[2 * (ib + l)] = v.v[0];
            if (cols & 2) a.xe[2 * (ib + l) + 1] = v.v[1];
        }
    };
    auto step = [&](auto PAR, int n) -> bool {
        constexpr int IN = decltype(PAR)::value;
        const bool more = n <= a.sweep1;
        if (more) sweep(PAR);
        __syncthreads();
        const unsigned f = flag[IN];             // the stop test of sweep n - 1
        if (f) {
            store(IN, f);
            live &= ~f;
        }
        if (!live) return true;
        if (!more) {
            store(IN, live);
            return true;
        }
        if (stop_wave) {
            const double rr = part_max(part + (1 - IN) * 4 * MAXW * 4, nw, 1, lane);
            const bool now = lane < 2 && (stop_live >> lane & 1) && rr <= a.eps;
            if (now) a.sweeps[2 * q + lane] = n;
            const unsigned fresh = (unsigned)__ballot(now);
            stop_live &= ~fresh;
            if (lane == 0) flag[1 - IN] = fresh;
        }
        return false;
    };
    for (int n = a.sweep0 + 1;; n += 2) {        // sweep0 and sweep1 are even
        if (step(std::integral_constant<int, 0>{}, n)) return;
        if (step(std::integral_constant<int, 1>{}, n + 1)) return;
    }
}

// Larger products: one iterate in LDS, the new values in registers until all
// old ones have been read; records and chosen rows come from memory (L2) in
// every sweep, in record order.
__global__ void __launch_bounds__(BIG_THREADS) eval_big(InstanceArgs a) {
    constexpr int NS = EVAL_BIG_STEPS, NW = BIG_THREADS / 64;
    extern __shared__ __align__(16) unsigned char lds[];
    const int q = a.order[blockIdx.x];
    unsigned live = (a.sweeps[2 * q] == 0 ? 1u : 0u) | (a.sweeps[2 * q + 1] == 0 ? 2u : 0u);
    if (!live) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = a.inst_model[q];
    const int sb = a.state_base[m], S = a.state_base[m + 1] - sb;
    const int64_t ib = a.inst_base[q];
    unsigned char* hdr = lds + (S + 1) * 16;
    double* part = reinterpret_cast<double*>(hdr);                           // [4 NW rows][4]
    unsigned* flag = reinterpret_cast<unsigned*>(hdr + 4 * NW * 4 * 8);
    {
        const EvalStart start(a, q);
        for (int l = tid; l < S; l += BIG_THREADS) {
            Row<double, 2> v;
            if (a.sweep0 > 0) {
                v.v[0] = a.xe[2 * (ib + l)];
                v.v[1] = a.xe[2 * (ib + l) + 1];
            } else {
                v = start.at(l);
            }
            lds_put<double, 2>((unsigned)(l + 1) << 4, v);
        }
        if (tid == 0) lds_put<double, 2>(0, Row<double, 2>{{0.0, 0.0}});
    }
    __syncthreads();
    auto store = [&](unsigned cols) {
        for (int l = tid; l < S; l += BIG_THREADS) {
            const Row<double, 2> v = lds_get<double, 2>((unsigned)(l + 1) << 4);
            if (cols & 1) a.xe[2 * (ib + l)] = v.v[0];
            if (cols & 2) a.xe[2 * (ib + l) + 1] = v.v[1];
        }
    };
    Row<double, 2> out[NS];
    unsigned own[NS];
    for (int n = a.sweep0 + 1; n <= a.sweep1; ++n) {
        double r[2] = {0.0, 0.0};
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const int p = tid + i * BIG_THREADS;
            if (p < S) {
                const int32_t* rec = a.rec + (int64_t)(sb + p) * 8;
                const int4 r0 = *reinterpret_cast<const int4*>(rec), r1 = *reinterpret_cast<const int4*>(rec + 4);
                const int sc[NSLOT] = {r0.x, r0.y, r0.z, r0.w, r1.x};
                double P[NSLOT];
                Row<double, 2> v;
                policy_row(a, r1, a.mu[ib + (r1.w - sb)], P, v.v[0], v.v[1]);
#pragma unroll
                for (int d = 0; d < NSLOT; ++d) {
                    const unsigned row = sc[d] == a.zero_row ? 0u : (unsigned)(sc[d] - sb + 1);
                    const Row<double, 2> xv = lds_get<double, 2>(row << 4);
                    v.v[0] = fma(P[d], xv.v[0], v.v[0]);
                    v.v[1] = fma(P[d], xv.v[1], v.v[1]);
                }
                own[i] = (unsigned)(r1.w - sb + 1) << 4;
                const Row<double, 2> old = lds_get<double, 2>(own[i]);
                r[0] = max_abs(r[0], v.v[0] - old.v[0]);
                r[1] = max_abs(r[1], v.v[1] - old.v[1]);
                out[i] = v;
            }
        }
        const double rr = row_max<double, 2>(r);
        if ((lane & 15) < 4) part[(wave * 4 + (lane >> 4)) * 4 + (lane & 3)] = rr;
        __syncthreads();   // every wave has read the old values
#pragma unroll
        for (int i = 0; i < NS; ++i)
            if (tid + i * BIG_THREADS < S) lds_put<double, 2>(own[i], out[i]);
        if (wave == NW - 1) {
            const double top = part_max(part, NW, 1, lane);
            const bool now = lane < 2 && (live >> lane & 1) && top <= a.eps;
            if (now) a.sweeps[2 * q + lane] = n;
            const unsigned fresh = (unsigned)__ballot(now);
            if (lane == 0) *flag = fresh;
        }
        __syncthreads();
        const unsigned f = *flag;
        if (f) {
            store(f);
            live &= ~f;
            if (!live) return;
        }
    }
    store(live);
}

int eval_capacity() {
    return std::min(EVAL_BIG_STEPS * BIG_THREADS, (int)((LDS_BYTES - 4 * (BIG_THREADS / 64) * 4 * 8 - 64) / 16) - 1);
}

template <int NS>
static void launch_eval(hipStream_t s, int max_states, const InstanceArgs& a) {
    const int threads = 64 * ((max_states + 64 * NS - 1) / (64 * NS));
    const size_t bytes = (size_t)res_rows(NS) * 16 + (size_t)(threads * NS + 1) * 16 + 2 * 4 * MAXW * 4 * 8 + 64;
    MORAP_CHECK(threads <= RES_MAX_THREADS && max_states < res_rows(NS) && bytes <= LDS_BYTES, MORAP_E_UNSUPPORTED,
                "an instance does not fit the LDS-resident evaluation");
    static OncePerDevice granted;
    grant_lds(granted, &eval_resident<NS>);
    hipLaunchKernelGGL(eval_resident<NS>, dim3((unsigned)a.n), dim3((unsigned)threads), bytes, s, a);
    MORAP_HIP(hipGetLastError());
}

// register steps of an instance of that many states, 0: the larger form
int eval_class(int states) {
    const int ns = std::max(1, (states + RES_MAX_THREADS - 1) / RES_MAX_THREADS);
    return ns <= 4 ? ns : (ns <= 7 ? 7 : 0);
}

void inst_eval(hipStream_t s, int max_states, const InstanceArgs& a) {
    if (a.n <= 0) return;
    switch (eval_class(max_states)) {
        case 1: return launch_eval<1>(s, max_states, a);
        case 2: return launch_eval<2>(s, max_states, a);
        case 3: return launch_eval<3>(s, max_states, a);
        case 4: return launch_eval<4>(s, max_states, a);
        case 7: return launch_eval<7>(s, max_states, a);
        default: break;
    }
    MORAP_CHECK(max_states <= eval_capacity(), MORAP_E_UNSUPPORTED, "an instance does not fit the LDS-resident evaluation");
    static OncePerDevice granted;
    grant_lds(granted, &eval_big);
    const size_t bytes = (size_t)(max_states + 1) * 16 + 4 * (BIG_THREADS / 64) * 4 * 8 + 64;
    hipLaunchKernelGGL(eval_big, dim3((unsigned)a.n), dim3(BIG_THREADS), bytes, s, a);
    MORAP_HIP(hipGetLastError());
}

}  // namespace k
}  // namespace morap
