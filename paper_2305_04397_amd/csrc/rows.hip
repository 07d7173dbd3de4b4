// Value iteration of products given as rows of entries (loaded by the caller,
// or of agents outside the block form) with the values in LDS: a workgroup
// takes one product and KC columns to their stop, as resident_vi does for the
// block form, and adds the terms of a backup in the order of the batched sweep
// over CSR tiles, so values and stopping sweeps are the same bits.  (States of
// at most five rows of three entries take resident_vi itself.)
#include "common.h"
#include "kern.h"
#include "resident.h"

namespace morap {
namespace k {

// Both iterates in LDS.  A wave walks the batches of its slices, a contiguous
// run of memory; rows and entries of a slice are in lockstep and the rewards of
// a row are entries too (the successors of their places are the weights), so a
// place is a gather and KC multiply-adds and the control is scalar.
//
// 48 products of 1,000 states of five rows of three random entries, 24 FP32
// columns, 241 sweeps: 1.6 ms; 15.5 with the batched sweeps.
//
// The batches pass through registers from L2, two ahead; four or six ahead are
// no faster: a wave's batch is a chain of gathers, sums and branches of about
// 600 cycles, which the other waves have to fill.
constexpr int AHEAD = 2;

template <class T, int KC, int THREADS>
__global__ void __launch_bounds__(THREADS) rows_vi(RowsArgs a) {
    constexpr bool F32 = sizeof(T) == 4;
    constexpr int ROWB = sizeof(T) * KC, SH = ROWB == 4 ? 2 : (ROWB == 8 ? 3 : 4);
    constexpr int NW = THREADS / 64;
    using T4 = T __attribute__((ext_vector_type(4)));
    extern __shared__ __align__(16) unsigned char lds[];

    const Item<T, KC, false> it(a);
    if (!it.ok) return;
    const int m = it.m;
    unsigned live = 0;   // columns still running
#pragma unroll
    for (int c = 0; c < KC; ++c)
        if (it.running(a, c)) live |= 1u << c;
    if (!live) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sb = a.state_base[m], S = a.state_base[m + 1] - sb;
    const int sl0 = a.slice[m], n_slices = a.slice[m + 1] - sl0;
    const unsigned buf = (unsigned)(n_slices * 64 + 3) * ROWB;   // distance of the two iterates
    unsigned char* hdr = lds + ((2 * buf + 15) & ~15u);
    T* part = reinterpret_cast<T*>(hdr);                                         // [2][4 NW rows][4][res, |y|]
    double* best = reinterpret_cast<double*>(hdr + 2 * 4 * NW * 8 * sizeof(T));  // [4] smallest change so far
    int* stall = reinterpret_cast<int*>(best + 4);                               // [4] sweeps since it was set
    unsigned* flag = reinterpret_cast<unsigned*>(stall + 4);                     // [2] results of the stop test

    // this wave's slices
    const int s_begin = wave * n_slices / NW, s_end = (wave + 1) * n_slices / NW;
    const int b0 = a.batch[sl0 + s_begin], nb = a.batch[sl0 + s_end] - b0;
    const int32_t* desc = a.desc + b0;
    const uint2* place = a.place + (int64_t)b0 * 64 + lane;
    const T4* value = static_cast<const T4*>(a.value) + (int64_t)b0 * 64 + lane;
    const unsigned own0 = (unsigned)(s_begin * 64 + lane + 1) << SH;

    for (int l = tid; l < n_slices * 64; l += THREADS) {
        Row<T, KC> v;
#pragma unroll
        for (int c = 0; c < KC; ++c) v.v[c] = it.start(a, sb, min(l, S - 1), c);
        lds_put<T, KC>((unsigned)(l + 1) << SH, v);
    }
    if (tid == 0) {
        Row<T, KC> z, wc, wp;
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            z.v[c] = 0;
            it.weights(a, c, wc.v[c], wp.v[c]);
        }
        for (unsigned x : {0u, buf}) {
            lds_put<T, KC>(x, z);
            lds_put<T, KC>(x + ((unsigned)(n_slices * 64 + 1) << SH), wp);
            lds_put<T, KC>(x + ((unsigned)(n_slices * 64 + 2) << SH), wc);
        }
        flag[0] = flag[1] = 0;
    }
    const bool stop_wave = wave == NW - 1;
    if (F32 && tid < KC && it.k0 + tid < a.K) {
        best[tid] = a.best_res[it.pair0 + tid];
        stall[tid] = a.stall[it.pair0 + tid];
    }
    unsigned stop_live = live;   // the running columns, as the stop test has them (a sweep ahead)

    constexpr int NR = AHEAD;
    uint2 at[NR];
    T4 val[NR];
    int d[NR];
    const int run = (nb + NR - 1) / NR * NR;   // ends in empty batches (`none`)
    const int none = a.batch[a.slice[a.M]] - b0;
    int z = 0;
    asm volatile("" : "+v"(z));   // (vector loads: scalar ones would come back in no order among the LDS reads)
    auto load = [&](int i, int b) {
        at[i] = place[(int64_t)b * 64];
        val[i] = value[(int64_t)b * 64];
        d[i] = desc[b + z];
    };
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        load(i, i < nb ? i : none);
    }
    __syncthreads();

    // values of the columns in `cols` from the iterate at `from`, each wave its
    // own slices: nothing waits between a stop's store and the next sweep, which
    // writes that iterate
    auto store = [&](void* x, unsigned from, unsigned cols) {
        for (int l = s_begin * 64 + lane; l < min(s_end * 64, S); l += 64) {
            const Row<T, KC> v = lds_get<T, KC>(from + ((unsigned)(l + 1) << SH));
#pragma unroll
            for (int c = 0; c < KC; ++c)
                if (cols >> c & 1) static_cast<T*>(x)[it.place(a, sb, l, c)] = v.v[c];
        }
    };

    for (int n = a.sweep0 + 1;; ++n) {
        const int par = (n - 1) & 1;                      // the iterate it reads
        const unsigned in = par ? buf : 0, out = par ? 0 : buf;
        const bool more = n <= a.sweep1;
        if (more) {
            T r[KC], y[KC], acc[KC], top[KC];
            unsigned own = own0;
#pragma unroll
            for (int c = 0; c < KC; ++c) {
                r[c] = y[c] = acc[c] = 0;
                top[c] = -INFINITY;
            }
            auto gather = [&](Row<T, KC>(&x)[4], const uint2& q) {
                x[0] = lds_get<T, KC>(in + low_row<SH>(q.x));
                x[1] = lds_get<T, KC>(in + high_row<SH>(q.x));
                x[2] = lds_get<T, KC>(in + low_row<SH>(q.y));
                x[3] = lds_get<T, KC>(in + high_row<SH>(q.y));
            };
            for (int b = 0; b < run; b += NR) {
#pragma unroll
                for (int i = 0; i < NR; ++i) {
                    const int now = __builtin_amdgcn_readfirstlane(d[i]);
                    Row<T, KC> x[4];
                    gather(x, at[i]);
                    const T4 v = val[i];
                    // the batch NR further on, past the end the next sweep's
                    const int next = b + i + NR < run ? b + i + NR : i;
                    load(i, next < nb ? next : none);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
#pragma unroll
                        for (int c = 0; c < KC; ++c) acc[c] = fma(v[u], x[u].v[c], acc[c]);
                        if (now >> u & 1)
#pragma unroll
                            for (int c = 0; c < KC; ++c) {
                                top[c] = max2(top[c], acc[c]);
                                acc[c] = 0;
                            }
                    }
                    if (now & 16) {
                        const Row<T, KC> old = lds_get<T, KC>(in + own);
                        Row<T, KC> w;
#pragma unroll
                        for (int c = 0; c < KC; ++c) {
                            w.v[c] = top[c];
                            r[c] = max_abs(r[c], top[c] - old.v[c]);
                            if (F32) y[c] = max_abs(y[c], top[c]);
                            top[c] = -INFINITY;
                        }
                        lds_put<T, KC>(out + own, w);
                        own += 64 << SH;
                    }
                }
            }
            const T rr = row_max<T, KC>(r);
            const T yy = F32 ? row_max<T, KC>(y) : (T)0;
            if ((lane & 15) < 4) {
                T* w = part + (((1 - par) * 4 * NW + wave * 4 + (lane >> 4)) * 4 + (lane & 3)) * 2;
                w[0] = rr;
                w[1] = yy;
            }
        }
        __syncthreads();
        const unsigned f = flag[par];   // the stop test of sweep n - 1, whose iterate is at `in`
        if (f & 0xffu) {
            store(a.x0, in, f & 0xffu);
            live &= ~f;
        }
        if (f & 0x100u) return;
        if (!more) {
            // the launch ends with columns running: their iterate, and after
            // the last launch of a solve the iterate before it
            store(a.x0, in, live);
            if (a.last) store(a.x1, out, live);
            if (stop_wave && lane < KC && (live >> lane & 1)) {
                const int64_t i = it.pair0 + lane;
                if (F32) {
                    a.best_res[i] = best[lane];
                    a.stall[i] = stall[lane];
                }
                if (a.last) a.active[i] = 1;
            }
            return;
        }
        if (stop_wave) {
            // the stop test of sweep n, while the others run the next one
            const T* w = part + (1 - par) * 4 * NW * 8;
            const T rr = part_max(w, NW, 2, lane), yy = F32 ? part_max(w + 1, NW, 2, lane) : (T)0;
            bool now = false;
            if (lane < KC && (stop_live >> lane & 1)) {
                bool floor_stop = false;
                now = it.stop(a, (double)rr, (double)yy, best[lane], stall[lane], floor_stop);
                if (now) {
                    it.stopped(a, lane, n, floor_stop);
                    a.c[(int64_t)(it.k0 + lane) * a.M + m] =
                        (double)reinterpret_cast<const T*>(lds + out + ((unsigned)(a.init[m] - sb + 1) << SH))[lane];
                }
            }
            const unsigned fresh = (unsigned)__ballot(now);
            stop_live &= ~fresh;
            if (lane == 0) flag[1 - par] = fresh | (stop_live == 0 ? 0x100u : 0u);
        }
    }
}

// The layouts, on the device at upload: the host only measures them.  Laying them
// out on the host, two copies of every value in memory and two over the link, took
// 2.0 of 4.0 ms of loading 48 products of 16 x 16 grids x 8 tasks.
//
// Short rows: one thread a state.
__global__ void __launch_bounds__(256) short_layout_kernel(RowsLayout a) {
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (g >= a.S) return;
    const int m = a.state_model[g];
    if (a.short_base[m] < 0) return;
    const int s0 = a.state_base[m];
    const int64_t at = a.short_base[m] + (g - s0);
    const int r0 = a.state_row[g], nr = a.state_row[g + 1] - r0;
    unsigned w[8] = {};
    double v[SHORT_VALUES] = {};
#pragma unroll
    for (int j = 0; j < 5; ++j) {   // a missing entry at the zero row, a missing row as the first
        const int r = r0 + (j < nr ? j : 0), e = a.row_ptr[r], ne = a.row_ptr[r + 1] - e;
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            if (u >= ne) continue;
            const int p = 3 * j + u;
            w[p / 2] |= (unsigned)(a.col[e + u] - s0 + 1) << (p % 2 * 16);
            v[p] = a.prob[e + u];
        }
        v[15 + j] = a.rew[2 * (int64_t)r];
        v[20 + j] = a.rew[2 * (int64_t)r + 1];
    }
    a.short_rec[2 * at] = make_uint4(w[0], w[1], w[2], w[3]);
    a.short_rec[2 * at + 1] = make_uint4(w[4], w[5], w[6], w[7]);
#pragma unroll
    for (int e = 0; e < SHORT_VALUES; ++e) {
        a.short_val64[at * SHORT_VALUES + e] = v[e];
        a.short_val32[at * SHORT_VALUES + e] = (float)v[e];
    }
}

void lay_out_short(hipStream_t s, const RowsLayout& a) {
    hipLaunchKernelGGL(short_layout_kernel, dim3((unsigned)((a.S + 255) / 256)), dim3(256), 0, s, a);
    MORAP_HIP(hipGetLastError());
}

// Streamed rows: one wave a slice, and one for the empty batch behind the last.
__global__ void __launch_bounds__(64) rows_layout_kernel(RowsLayout a) {
    const int sl = blockIdx.x, lane = threadIdx.x;
    const int64_t b0 = a.batch[sl];
    unsigned p[4] = {0, 0, 0, 0};
    double v[4] = {0, 0, 0, 0};
    int f = 0, bits = 0;   // places of the slice so far; ends of rows in the batch
    auto flush = [&](int extra) {
        const int64_t b = b0 + (f - 1) / 4, at = b * 64 + lane;
        a.place[at] = make_uint2(p[0] | p[1] << 16, p[2] | p[3] << 16);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a.value64[at * 4 + u] = v[u];
            a.value32[at * 4 + u] = (float)v[u];
            p[u] = 0;
            v[u] = 0;
        }
        if (lane == 0) a.desc[b] = bits | extra;
        bits = 0;
    };
    if (sl == a.n_slices) {
        f = 1;
        flush(0);
        return;
    }
    int lo = 0, hi = a.M;   // the slice's model: slice[lo] <= sl < slice[lo + 1]
    while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        if (a.slice[mid] <= sl) lo = mid;
        else hi = mid;
    }
    const int s0 = a.state_base[lo], n = a.state_base[lo + 1] - s0;
    const int g = s0 + min((sl - a.slice[lo]) * 64 + lane, n - 1);
    const int r0 = a.state_row[g], rows = a.state_row[g + 1] - r0;
    const unsigned wp_row = (unsigned)((n + 63) / 64 * 64 + 1);
    auto largest = [](int x) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) x = max(x, __shfl_xor(x, o, 64));
        return x;
    };
    auto put = [&](unsigned row, double x) {   // (the wave's places are in lockstep)
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if ((f & 3) == u) {
                p[u] = row;
                v[u] = x;
            }
        ++f;
    };
    const int most = largest(rows);
    for (int j = 0; j < most; ++j) {
        const int r = r0 + (j < rows ? j : 0), e = a.row_ptr[r], ne = a.row_ptr[r + 1] - e;
        const int len = 2 + largest(ne);
        for (int i = 0; i < len; ++i) {
            if (i < 2) put(wp_row + i, a.rew[2 * (int64_t)r + 1 - i]);
            else if (i - 2 < ne) put((unsigned)(a.col[e + i - 2] - s0 + 1), a.prob[e + i - 2]);
            else put(0, 0);
            const bool last = i + 1 == len;
            if (last) bits |= 1 << ((f - 1) & 3);
            if ((f & 3) == 0 || (last && j + 1 == most)) flush(last && j + 1 == most ? 16 : 0);
        }
    }
}

void lay_out_rows(hipStream_t s, const RowsLayout& a) {
    hipLaunchKernelGGL(rows_layout_kernel, dim3((unsigned)a.n_slices + 1), dim3(64), 0, s, a);
    MORAP_HIP(hipGetLastError());
}

static size_t rows_bytes(int prec, int columns, int states, int threads) {
    const size_t el = prec == MORAP_F32 ? 4 : 8;
    const size_t rows = (size_t)(states + 63) / 64 * 64 + 3;
    return (2 * rows * columns * el + 15) / 16 * 16 + 2 * 4 * (size_t)(threads / 64) * 8 * el + 64;
}

int rows_columns(int prec, int states) {
    for (int kc = prec == MORAP_F32 ? 4 : 2; kc >= 1; kc /= 2)
        if (rows_bytes(prec, kc, states, BIG_THREADS) <= LDS_BYTES) return kc;
    return 0;
}

template <class T, int KC, int THREADS>
static void launch_rows(hipStream_t s, const RowsArgs& a, int max_states) {
    auto* fn = &rows_vi<T, KC, THREADS>;
    const size_t bytes = rows_bytes(sizeof(T) == 4 ? MORAP_F32 : MORAP_F64, KC, max_states, THREADS);
    MORAP_CHECK(bytes <= LDS_BYTES, MORAP_E_UNSUPPORTED, "a product does not fit the LDS-resident iteration");
    static OncePerDevice granted;
    grant_lds(granted, fn);
    hipLaunchKernelGGL(fn, dim3(8u * (unsigned)((a.n_models + 7) / 8) * (unsigned)a.groups), dim3(THREADS), bytes, s, a);
    MORAP_HIP(hipGetLastError());
}

template <class T, int KC>
static void launch_rows(hipStream_t s, const RowsArgs& a, int max_states) {
    if (max_states <= 4 * 64) launch_rows<T, KC, 256>(s, a, max_states);
    else if (max_states <= 8 * 64) launch_rows<T, KC, 512>(s, a, max_states);
    else launch_rows<T, KC, BIG_THREADS>(s, a, max_states);
}

void resident_rows(hipStream_t s, int prec, int columns, int max_states, const RowsArgs& args) {
    RowsArgs a = args;
    if (a.n_models <= 0) return;
    columns = std::min(columns, a.Kp);
    a.groups = (a.K + columns - 1) / columns;
    if (prec == MORAP_F32) {
        if (columns == 4) launch_rows<float, 4>(s, a, max_states);
        else if (columns == 2) launch_rows<float, 2>(s, a, max_states);
        else launch_rows<float, 1>(s, a, max_states);
    } else {
        if (columns == 2) launch_rows<double, 2>(s, a, max_states);
        else launch_rows<double, 1>(s, a, max_states);
    }
}

}  // namespace k
}  // namespace morap
