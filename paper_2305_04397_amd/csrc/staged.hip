// Stage retirement inside the Jacobi iteration (the staged form of Alg. 3
// that keeps the plain sweep count).
//
// A product's location groups (strongly connected sets of DFA locations)
// form a DAG in which every transition leads to the same or a lower group;
// a state's stage is the height of its group there (0: no lower group).
// The states of each model are split into units, one per stage, lowest
// first, and the sweep kernels run over the units' tiles as over models.
// After every sweep, per (model, column), the units are taken lowest first:
// a unit retires when every lower unit has retired and its own largest
// change in this sweep is within the stop rule; its tiles then leave the
// active list.  A retired unit is no longer written, so its final values
// (in the buffer the sweep just wrote) are copied into the other Jacobi
// buffer before the next sweep writes that buffer's other states: the units
// above it keep reading the same values in every later sweep.
//
// Products that fit a workgroup's LDS run the same iteration there instead
// (staged_vi), all of a product's sweeps in one launch.
#include "common.h"
#include "kern.h"
#include "resident.h"

namespace morap {
namespace k {

// One thread per (model, column) pair.  counters: as the convergence kernel
// ([0] active pairs, [4] backups, [7] state-columns updated), with the
// (unit, column) pairs retired in this sweep appended to a.retired and
// counted in counters[a.slot].
template <class T>
__global__ void __launch_bounds__(256) stage_converge_kernel(StageArgs a) {
    const int64_t n = (int64_t)a.M * a.Kp;
    const int32_t next_sweep = (int32_t)(a.counters[5] + 1);
    unsigned long long bk = 0, sc = 0, cnt = 0;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
        const int m = (int)(t / a.Kp);
        const int k = (int)(t % a.Kp);
        if (k >= a.K) continue;
        bool lower_done = true;
        for (int u = a.unit_base[m]; u < a.unit_base[m + 1]; ++u) {
            const int64_t j = (int64_t)u * a.Kp + k;
            if (!a.active[j]) continue;   // retired earlier (or never live)
            const double r = __longlong_as_double((long long)a.res[j]);
            const double y = __longlong_as_double((long long)a.ymax[j]);
            a.res[j] = 0ull;
            a.ymax[j] = 0ull;
            bk += (unsigned long long)a.rows[u];
            sc += (unsigned long long)a.states[u];
            const double tol = fmax(a.eps, a.unit * y);
            // FP32: a unit whose change has set no new minimum for
            // stall_sweeps sweeps and is within the rounding floor has
            // settled as far as FP32 backups go (as a pair of the plain solve)
            bool floor_stop = false;
            if (a.stall_sweeps > 0 && r > tol) {
                if (r < a.best_res[j]) {
                    a.best_res[j] = r;
                    a.stall[j] = 0;
                } else if (++a.stall[j] >= a.stall_sweeps && r <= a.floor * y) {
                    floor_stop = true;
                }
            }
            if (lower_done && (r <= tol || floor_stop)) {
                if (floor_stop) atomicAdd((unsigned long long*)&a.counters[8], 1ull);
                a.active[j] = 0;
                const unsigned long long p = atomicAdd((unsigned long long*)&a.counters[a.slot], 1ull);
                a.retired[p] = j;
                if (u == a.init_unit[m]) {
                    // the initial state's value is final
                    const int64_t i = (int64_t)m * a.Kp + k;
                    a.c[(int64_t)k * a.M + m] = (double)((const T*)a.x_out)[(int64_t)a.init[m] * a.Kp + k];
                    a.final_par[i] = (uint8_t)a.out_par;
                    a.pair_sweeps[i] = next_sweep;
                }
            } else {
                lower_done = false;
                a.model_active[u] = 1;
                ++cnt;
            }
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        bk += __shfl_xor(bk, o, 64);
        sc += __shfl_xor(sc, o, 64);
        cnt += __shfl_xor(cnt, o, 64);
    }
    __shared__ unsigned long long part[3][4];
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        part[0][w] = cnt;
        part[1][w] = bk;
        part[2][w] = sc;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const unsigned long long v = part[threadIdx.x][0] + part[threadIdx.x][1] + part[threadIdx.x][2] +
                                     part[threadIdx.x][3];
        const int slot = threadIdx.x == 0 ? 0 : (threadIdx.x == 1 ? 4 : 7);
        if (v) atomicAdd((unsigned long long*)&a.counters[slot], v);
    }
}

// The final values of the (unit, column) pairs retired in this sweep, copied
// from the buffer the sweep wrote into the one it read: one workgroup per
// retired pair at a time, its threads over the unit's records (each names
// its state).  The list count of the next sweep starts at 0 here.
template <class T>
__global__ void __launch_bounds__(256) stage_copy_kernel(StageArgs a) {
    if (blockIdx.x == 0 && threadIdx.x == 0) a.counters[a.slot == 9 ? 10 : 9] = 0;
    const int64_t n = a.counters[a.slot];
    for (int64_t e = blockIdx.x; e < n; e += gridDim.x) {
        const int64_t j = a.retired[e];
        const int u = (int)(j / a.Kp);
        const int k = (int)(j % a.Kp);
        for (int tt = a.tile_base[u]; tt < a.tile_base[u + 1]; ++tt) {
            const Tile tl = a.tiles[tt];
            for (int p = tl.s_begin + (int)threadIdx.x; p < tl.s_end; p += blockDim.x) {
                const int64_t g = a.rec[(int64_t)p * 8 + 7];
                ((T*)a.x_in)[g * a.Kp + k] = ((const T*)a.x_out)[g * a.Kp + k];
            }
        }
    }
}

// One product and KC columns to the stop of their last stage: one iterate in
// LDS, the new values of a sweep in registers until every wave has read the
// old ones.  The states lie sorted by (block, stage), padded per block to steps
// of 64 that share their probabilities (scalar loads); sorting by stage first
// would pad every (stage, block) pair, 2.5 times the states at a fifth of the
// cells blocked.  A step runs while a stage of it does in some column: every
// wave takes each NW-th of those steps, listed anew when the lowest running
// stage moves.  A lane whose state has retired in a column keeps its value.
//
// What a stage's stop test needs: in FP64 whether a change was above eps, one
// bit per stage in a register of every lane; in FP32 the largest change and
// value, in registers while a wave's steps stay within one stage, straight to
// LDS from the lanes of a step that spans several.
//
// 8 agents on 24 x 24 grids x 12 tasks of up to 9 locations, 32 FP64 columns:
// 1.8 ms; 14.8 ms with the batched sweeps, whose four launches and stop test
// over memory per sweep (275 of them) cost more than the backups.
template <class T, int KC, int THREADS>
__global__ void __launch_bounds__(THREADS, 4) staged_vi(StagedLdsArgs a) {
    constexpr bool F32 = sizeof(T) == 4;
    constexpr int ROWB = sizeof(T) * KC, SH = ROWB == 4 ? 2 : (ROWB == 8 ? 3 : 4);
    constexpr int NW = THREADS / 64, NS = 160 / ROWB;
    extern __shared__ __align__(16) unsigned char lds[];

    // the columns of one product go to one XCD: its records meet in that L2
    const int slot = blockIdx.x >> 3;
    const int mi = slot / a.groups * 8 + (int)(blockIdx.x & 7);
    if (mi >= a.n_models) return;
    const int m = a.order[mi], k0 = slot % a.groups * KC;
    const int u0 = a.unit_base[m], nst = a.unit_base[m + 1] - u0;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sb = a.state_base[m];
    const int pos0 = a.big_base[m], n_steps = (a.big_base[m + 1] - pos0) >> 6;
    using CInt = const __attribute__((address_space(4))) int32_t*;
    using CVal = const __attribute__((address_space(4))) T*;
    const CInt info = (CInt)(a.big_block + (pos0 >> 6));
    const CVal ablk = (CVal)(static_cast<const T*>(a.grid_blk));
    const uint4* rec = a.big_rec + pos0 + lane;
    unsigned char* hdr = lds + (((n_steps * 64 + 1) * ROWB + 15) & ~15);
    unsigned* top = reinterpret_cast<unsigned*>(hdr);   // FP32: [2][64] largest change, value of (stage, column); FP64: [KC] stages above eps
    unsigned* low = top + 128;                          // lowest running stage of the columns, 8 bits each
    uint16_t* list = reinterpret_cast<uint16_t*>(low + 4) + wave * 64;   // this wave's steps

    // lowest running stage per column (a retired column: all stages)
    unsigned p = 0;
#pragma unroll
    for (int c = 0; c < KC; ++c) {
        int q = nst;
        if (k0 + c < a.K) {
            q = 0;
            while (q < nst && a.unit_sweeps[(int64_t)(u0 + q) * a.Kp + k0 + c] != 0) ++q;
        }
        p |= (unsigned)q << (8 * c);
    }
    p = __builtin_amdgcn_readfirstlane(p);
    auto low_of = [&](int c) { return (int)(p >> (8 * c) & 255u); };
    auto lowest = [&] {
        int q = low_of(0);
#pragma unroll
        for (int c = 1; c < KC; ++c) q = min(q, low_of(c));
        return q;
    };
    int from = lowest();
    if (from >= nst) return;

    T wp[KC], first[KC][5];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
        const int k = k0 + c < a.K ? k0 + c : 0;
        const double* W = a.W + (int64_t)k * a.d;
        const T wc = scalar((T)W[m / a.nJ]);
        wp[c] = scalar((T)W[a.nI + m % a.nJ]);
        // every state of the product has the same action costs
#pragma unroll
        for (int q = 0; q < 5; ++q) first[c][q] = wc * ablk[(int64_t)(info[0] & 0xfffff) * GRID_BLK + GRID_NNZ + q];
    }
    for (int i = tid; i < n_steps * 64; i += THREADS) {
        const int l = (int)(a.big_rec[pos0 + i].w & 0xffffu);
        Row<T, KC> v;
#pragma unroll
        for (int c = 0; c < KC; ++c)
            v.v[c] = a.sweep0 > 0 && k0 + c < a.K ? static_cast<const T*>(a.x0)[(int64_t)(sb + l) * a.Kp + k0 + c] : (T)0;
        lds_put<T, KC>((unsigned)(i + 1) << SH, v);
    }
    if (tid == 0) {
        Row<T, KC> z;
#pragma unroll
        for (int c = 0; c < KC; ++c) z.v[c] = 0;
        lds_put<T, KC>(0, z);
    }
    if (tid < 128) top[tid] = 0;
    // lane s KC + c of the last wave tests stage s of column c
    const int js = lane / KC, jc = lane % KC;
    const bool stop_wave = wave == NW - 1, tests = stop_wave && js < nst && k0 + jc < a.K;
    const int64_t ju = (int64_t)(u0 + min(js, nst - 1)) * a.Kp + k0 + jc;
    const int init_stage = a.init_unit[m] - u0;
    double best = INFINITY;
    int stall = 0;
    if (F32 && tests && a.sweep0 > 0) {
        best = a.best_res[ju];
        stall = a.stall[ju];
    }

    // the steps with a running stage, dealt to the waves
    int mine = 0, cnt = 0;
    auto deal = [&] {
        int total = 0;
        for (int b = 0; b < n_steps; b += 64) {
            const int q = b + lane;
            const bool run = q < n_steps && (int)((unsigned)info[min(q, n_steps - 1)] >> 26) >= from;
            const unsigned long long bal = __ballot(run);
            const int at = total + __popcll(bal & ((1ull << lane) - 1));
            if (run && at % NW == wave) list[at / NW] = (uint16_t)q;
            total += __popcll(bal);
        }
        cnt = __builtin_amdgcn_readfirstlane(total > wave ? (total - wave + NW - 1) / NW : 0);
        __builtin_amdgcn_wave_barrier();
        mine = lane < cnt ? list[lane] : 0;
    };
    deal();
    __syncthreads();

    Row<T, KC> out[NS];
    for (int n = a.sweep0 + 1; n <= a.sweep1; ++n) {
        // FP32: of the wave's current stage; FP64: a bit per stage above eps
        T r[KC], y[KC];
        unsigned above[KC];
        int cur = 0;
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            r[c] = y[c] = 0;
            above[c] = 0;
        }
        auto flush = [&] {
            if constexpr (F32) {
                const T rr = row_max<T, KC>(r), yy = row_max<T, KC>(y);
                if ((lane & 15) < KC) {
                    atomicMax(&top[cur * KC + (lane & 15)], __builtin_bit_cast(unsigned, rr));
                    atomicMax(&top[64 + cur * KC + (lane & 15)], __builtin_bit_cast(unsigned, yy));
                }
#pragma unroll
                for (int c = 0; c < KC; ++c) r[c] = y[c] = 0;
            }
        };
        int step = __builtin_amdgcn_readfirstlane(mine);
        uint4 q = rec[step * 64];
        int inf = info[step];
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            if (i < cnt) {
            uint4 qn = q;
            int in = inf;
            if (i + 1 < cnt) {   // the next step's records and block are on their way
                const int next = __builtin_amdgcn_readlane(mine, i + 1);
                qn = rec[next * 64];
                in = info[next];
                step = next;
            }
            const CVal B = ablk + (int64_t)(inf & 0xfffff) * GRID_BLK;
            const int s_lo = inf >> 20 & 63, s_hi = (int)((unsigned)inf >> 26);
            const int st = (int)(q.w >> 16 & 63u);
            T P[GRID_NNZ];
#pragma unroll
            for (int e = 0; e < GRID_NNZ; ++e) P[e] = B[e];
            Row<T, KC> xv[NSLOT];
            xv[0] = lds_get<T, KC>(low_row<SH>(q.x));
            xv[1] = lds_get<T, KC>(high_row<SH>(q.x));
            xv[2] = lds_get<T, KC>(low_row<SH>(q.y));
            xv[3] = lds_get<T, KC>(high_row<SH>(q.y));
            xv[4] = lds_get<T, KC>(low_row<SH>(q.z));
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
                                const T pr = (accm >> d & 1) ? P[e] : (T)0;
                                rp[act] = first_term ? pr : rp[act] + pr;
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
                    const T best_v = max3(max3(v[0], v[1], v[2]), v[3], v[4]);
                    out[i].v[c] = st < low_of(c) ? xv[0].v[c] : best_v;   // slot 0 is the state itself
                }
            };
            if (__ballot(accm != 0)) backup(std::true_type{});
            else backup(std::false_type{});
            if constexpr (!F32) {
#pragma unroll
                for (int c = 0; c < KC; ++c)
                    above[c] |= fabs(out[i].v[c] - xv[0].v[c]) > a.eps ? 1u << st : 0u;
            } else if (s_lo == s_hi) {
                if (s_lo != cur) {
                    flush();
                    cur = s_lo;
                }
#pragma unroll
                for (int c = 0; c < KC; ++c) {
                    r[c] = max_abs(r[c], out[i].v[c] - xv[0].v[c]);
                    y[c] = max_abs(y[c], out[i].v[c]);
                }
            } else {
#pragma unroll
                for (int c = 0; c < KC; ++c)
                    if (st >= low_of(c)) {
                        atomicMax(&top[st * KC + c], __builtin_bit_cast(unsigned, fabsf((float)(out[i].v[c] - xv[0].v[c]))));
                        atomicMax(&top[64 + st * KC + c], __builtin_bit_cast(unsigned, fabsf((float)out[i].v[c])));
                    }
            }
            q = qn;
            inf = in;
            }
        }
        if constexpr (F32) {
            flush();
        } else {
#pragma unroll
            for (int c = 0; c < KC; ++c) {
                unsigned v = above[c];
#pragma unroll
                for (int o = 32; o >= 1; o >>= 1) v |= (unsigned)__shfl_xor((int)v, o, 64);
                if (lane == 0 && v) atomicOr(&top[c], v);
            }
        }
        __syncthreads();   // every wave has read the old values
#pragma unroll
        for (int i = 0; i < NS; ++i)
            if (i < cnt)
                lds_put<T, KC>((unsigned)(__builtin_amdgcn_readlane(mine, i) * 64 + lane + 1) << SH, out[i]);
        if (stop_wave) {
            bool pass = true, floor_stop = false;
            if (tests && js >= low_of(jc)) {
                if constexpr (F32) {
                    const double res = (double)__builtin_bit_cast(float, top[lane]);
                    const double ym = (double)__builtin_bit_cast(float, top[64 + lane]);
                    top[lane] = top[64 + lane] = 0;
                    const double tol = fmax(a.eps, a.unit * ym);
                    if (res > tol) {
                        if (res < best) {
                            best = res;
                            stall = 0;
                        } else if (++stall >= a.stall_sweeps && res <= a.floor * ym) {
                            floor_stop = true;
                        }
                    }
                    pass = res <= tol || floor_stop;
                } else {
                    pass = !(top[jc] >> js & 1u);
                }
            }
            // a stage retires when it and every lower one pass
            const unsigned long long fail = __ballot(!pass);
            bool retires = false;
            unsigned np = p;
#pragma unroll
            for (int c = 0; c < KC; ++c) {
                unsigned long long f = fail;
                if constexpr (KC > 1) f &= (KC == 2 ? 0x5555555555555555ull : 0x1111111111111111ull) << c;
                const int to = f ? (__ffsll((long long)f) - 1) / KC : nst;
                if (low_of(c) < nst) {
                    if (jc == c && tests && js >= low_of(c) && js < to) retires = true;
                    np = (np & ~(255u << (8 * c))) | (unsigned)to << (8 * c);
                }
            }
            if (retires) {
                a.unit_sweeps[ju] = n;
                if (js == init_stage) a.pair_sweeps[(int64_t)m * a.Kp + k0 + jc] = n;
                if (floor_stop) atomicAdd((unsigned long long*)&a.counters[8], 1ull);
            }
            if (!F32 && lane < KC) top[lane] = 0;
            if (lane == 0) *low = np;
        }
        __syncthreads();
        p = __builtin_amdgcn_readfirstlane(*low);
        const int now = lowest();
        if (now != from) {
            from = now;
            if (from >= nst) break;
            deal();
        }
    }
    // the launch ends with columns running, or all of them are done
    for (int i = tid; i < n_steps * 64; i += THREADS) {
        const unsigned w = a.big_rec[pos0 + i].w;
        if (w >> 31) continue;   // padding
        const Row<T, KC> v = lds_get<T, KC>((unsigned)(i + 1) << SH);
#pragma unroll
        for (int c = 0; c < KC; ++c)
            if (k0 + c < a.K) static_cast<T*>(a.x0)[(int64_t)(sb + (int)(w & 0xffffu)) * a.Kp + k0 + c] = v.v[c];
    }
    if (tid < KC && k0 + tid < a.K)
        a.c[(int64_t)(k0 + tid) * a.M + m] =
            (double)reinterpret_cast<const T*>(lds + ((unsigned)(a.big_init[m] + 1) << SH))[tid];
    if (F32 && tests) {
        a.best_res[ju] = best;
        a.stall[ju] = stall;
    }
}

constexpr int STAGED_HDR = 128 * 4 + 16 + 2 * BIG_THREADS;

// LDS of one iterate of `positions` states and the stop tests' words
static size_t staged_bytes(int prec, int columns, int positions) {
    return ((size_t)(positions + 1) * columns * (prec == MORAP_F32 ? 4 : 8) + 15) / 16 * 16 + STAGED_HDR;
}

int staged_columns(int prec, int positions, int stages) {
    const int el = prec == MORAP_F32 ? 4 : 8;
    if (stages < 1 || (prec != MORAP_F32 && stages > 32)) return 0;
    for (int kc = 16 / el; kc >= 1; kc /= 2)
        if (stages * kc <= 64 && staged_bytes(prec, kc, positions) <= LDS_BYTES &&
            positions <= BIG_THREADS * 160 / (el * kc))
            return kc;
    return 0;
}

// Half the waves where two workgroups then share a compute unit: one computes
// while the other waits at its two barriers a sweep.
int staged_threads(int prec, int columns, int positions) {
    const int el = prec == MORAP_F32 ? 4 : 8;
    return positions <= 512 * 160 / (el * columns) && staged_bytes(prec, columns, positions) <= LDS_BYTES / 2
               ? 512 : BIG_THREADS;
}

template <class T, int KC, int THREADS>
static void launch_staged(hipStream_t s, const StagedLdsArgs& a, int max_positions) {
    auto* fn = &staged_vi<T, KC, THREADS>;
    const size_t bytes = staged_bytes(sizeof(T) == 4 ? MORAP_F32 : MORAP_F64, KC, max_positions);
    MORAP_CHECK(max_positions % 64 == 0 && bytes <= LDS_BYTES && max_positions <= THREADS * 160 / (int)(sizeof(T) * KC),
                MORAP_E_UNSUPPORTED, "a product does not fit the LDS-resident iteration");
    static OncePerDevice granted;
    grant_lds(granted, fn);
    hipLaunchKernelGGL(fn, dim3(8u * (unsigned)((a.n_models + 7) / 8) * (unsigned)a.groups), dim3(THREADS), bytes, s, a);
    MORAP_HIP(hipGetLastError());
}

template <class T, int KC>
static void launch_staged(hipStream_t s, int threads, const StagedLdsArgs& a, int max_positions) {
    if (threads == 512) launch_staged<T, KC, 512>(s, a, max_positions);
    else launch_staged<T, KC, BIG_THREADS>(s, a, max_positions);
}

void staged_lds(hipStream_t s, int prec, int columns, int threads, int max_positions, const StagedLdsArgs& args) {
    StagedLdsArgs a = args;
    if (a.n_models <= 0) return;
    a.groups = (a.K + columns - 1) / columns;
    if (prec == MORAP_F32) {
        if (columns == 4) launch_staged<float, 4>(s, threads, a, max_positions);
        else if (columns == 2) launch_staged<float, 2>(s, threads, a, max_positions);
        else launch_staged<float, 1>(s, threads, a, max_positions);
    } else {
        if (columns == 2) launch_staged<double, 2>(s, threads, a, max_positions);
        else launch_staged<double, 1>(s, threads, a, max_positions);
    }
}

void stage_converge(hipStream_t s, const StageArgs& a) {
    const int64_t n = (int64_t)a.M * a.Kp;
    const unsigned blocks = (unsigned)std::min<int64_t>(256, std::max<int64_t>(1, (n + 255) / 256));
    if (a.prec == MORAP_F32) hipLaunchKernelGGL(stage_converge_kernel<float>, dim3(blocks), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(stage_converge_kernel<double>, dim3(blocks), dim3(256), 0, s, a);
    MORAP_HIP(hipGetLastError());
}

void stage_copy(hipStream_t s, const StageArgs& a) {
    if (a.prec == MORAP_F32) hipLaunchKernelGGL(stage_copy_kernel<float>, dim3(256), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(stage_copy_kernel<double>, dim3(256), dim3(256), 0, s, a);
    MORAP_HIP(hipGetLastError());
}

}  // namespace k
}  // namespace morap
