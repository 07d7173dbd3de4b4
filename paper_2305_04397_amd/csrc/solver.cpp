// Host orchestration of the batched value iteration (Alg. 3 for K weight
// columns at once), policy extraction and per-objective evaluation (Alg. 4)
// of the assigned (column, model) instances.
//
// Precision: an FP32 solve runs FP32 backups (FP64 residual) over every
// (model, column) pair and yields the values that choose the assignment.  The
// evaluation then repeats the value iteration in FP64 from 0, with the same
// stopping rule, on the assigned pairs only (one pair per task and column);
// policies and per-objective values come from those FP64 values.
#include "common.h"

#include <algorithm>
#include <atomic>
#include <chrono>
#include <thread>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <functional>

namespace morap {

// ---------------------------------------------------------------------------
// sweep-kernel variants: kernel family x columns per lane x lanes per state.
// Ids 1-18 are the CSR-tile sweep, 19-36 the same shapes of the
// neighbourhood-block sweep, 37-38 the wave-per-state block sweep with other
// numbers of states in flight, 39-40 the LDS-staged sweep over halo tiles.
// ---------------------------------------------------------------------------
const std::vector<Variant>& variants() {
    static const std::vector<Variant> v = [] {
        std::vector<Variant> out;
        const int pairs[][2] = {{1, 1},  {1, 2},  {2, 1},  {1, 4},  {2, 2},  {4, 1},
                                {1, 8},  {2, 4},  {4, 2},  {1, 16}, {2, 8},  {4, 4},
                                {1, 32}, {2, 16}, {4, 8},  {1, 64}, {2, 32}, {4, 16}};
        int id = 1;
        for (auto& p : pairs) out.push_back({id++, p[0], p[1], std::min(256, 64 * p[1]), SWEEP_CSR, 0});
        for (auto& p : pairs) out.push_back({id++, p[0], p[1], 256, SWEEP_BLOCK, p[1] == 64 ? 4 : 2});
        // the wave-per-state block sweep with 2 and 8 states in flight
        out.push_back({id++, 1, 64, 256, SWEEP_BLOCK, 2});
        out.push_back({id++, 1, 64, 256, SWEEP_BLOCK, 8});
        // the LDS-staged sweep over halo tiles (FP32), 2 and 4 states in flight
        out.push_back({id++, 1, 64, 256, SWEEP_HALO, 2});
        out.push_back({id++, 1, 64, 256, SWEEP_HALO, 4});
        return out;
    }();
    return v;
}

static int kt_of(const Variant& v) { return v.cpl * v.lps; }
static bool uses_halo_tiles(const Variant& v) { return v.kind == SWEEP_HALO; }

static int padded_k(int K) {
    if (K <= 64) {
        int p = 1;
        while (p < K) p <<= 1;
        return std::max(p, 1);
    }
    return (K + 63) / 64 * 64;
}

// candidate variants for a padded width: k-tiles of min(Kp, 64) columns and
// of half that; a restricted solve (few active columns per model) also tries
// narrower k-tiles, which skip the k-tiles without active columns
static std::vector<Variant> candidates(int Kp, bool restricted, bool blocks, bool halo) {
    std::vector<Variant> out;
    const int kt_full = std::min(Kp, 64);
    for (const auto& v : variants()) {
        if (v.kind == SWEEP_BLOCK && !blocks) continue;
        if (v.kind == SWEEP_HALO && !halo) continue;
        const int kt = kt_of(v);
        if (Kp % kt) continue;
        if (kt == kt_full || (kt * 2 == kt_full && kt >= 8) || (restricted && kt >= 8 && kt <= kt_full))
            out.push_back(v);
    }
    return out;
}

static const Variant& variant_by_id(int id) {
    for (const auto& v : variants())
        if (v.id == id) return v;
    fail(MORAP_E_INVALID, "unknown sweep variant id " + std::to_string(id));
}

// ---------------------------------------------------------------------------
// buffers
// ---------------------------------------------------------------------------
static void ensure_scratch(morap_ctx* c, int Kp) {
    const int M = c->hm.M;
    const size_t pairs = (size_t)M * Kp;
    bool moved = false;
    moved |= c->d_wc32.ensure(pairs * 4);
    moved |= c->d_wp32.ensure(pairs * 4);
    moved |= c->d_wc64.ensure(pairs * 8);
    moved |= c->d_wp64.ensure(pairs * 8);
    moved |= c->d_res.ensure(pairs * 8);
    moved |= c->d_ymax.ensure(pairs * 8);
    moved |= c->d_active.ensure(pairs);
    moved |= c->d_pair_mask.ensure(pairs);
    moved |= c->d_pair_sweeps.ensure(pairs * 4);
    moved |= c->d_model_active.ensure(M);
    moved |= c->d_act_models.ensure((size_t)M * 4 + 4);
    moved |= c->d_act_prefix.ensure((size_t)(M + 1) * 4 + 4);
    moved |= c->d_act_tiles.ensure(std::max<size_t>(c->tiles.size(), (size_t)c->n_htiles) * 4 + 4);
    moved |= c->d_best_res.ensure(pairs * 8);
    moved |= c->d_stall.ensure(pairs * 4);
    moved |= c->d_counters.ensure(9 * 8);
    c->h_counters.ensure(9 * 8);
    // a captured sweep graph holds these addresses: it must not replay
    // after any of them moved
    if (moved) ++c->buf_gen;
}

static void ensure_values(morap_ctx* c, ValueSet& vs, int K, int Kp, int prec) {
    const size_t el = prec == MORAP_F32 ? 4 : 8;
    bool moved = false;
    // one row past the last state: the zero row of the block sweep
    moved |= vs.x[0].ensure((size_t)(c->S + 1) * Kp * el);
    moved |= vs.x[1].ensure((size_t)(c->S + 1) * Kp * el);
    moved |= vs.final_par.ensure((size_t)c->hm.M * Kp);
    moved |= vs.c.ensure((size_t)K * c->hm.M * 8);
    if (moved) ++c->buf_gen;
    vs.prec = prec;
    vs.K = K;
    vs.Kp = Kp;
    vs.valid = false;
}

// `halo`: the active tile list is built over the halo tiles (LDS-staged
// sweep) instead of the CSR / block tiles
static k::ConvergeArgs converge_args(morap_ctx* c, ValueSet& vs, const uint8_t* mask, double eps, int out_par,
                                     bool halo) {
    k::ConvergeArgs a{};
    a.res = c->d_res.as<unsigned long long>();
    a.ymax = c->d_ymax.as<unsigned long long>();
    a.active = c->d_active.as<uint8_t>();
    a.final_par = vs.final_par.as<uint8_t>();
    a.pair_sweeps = c->d_pair_sweeps.as<int32_t>();
    a.model_active = c->d_model_active.as<uint8_t>();
    a.c = vs.c.as<double>();
    a.init = c->d_init.as<int32_t>();
    a.mask = mask;
    a.x_out = vs.x[out_par].p;
    a.counters = c->d_counters.as<int64_t>();
    a.M = c->hm.M;
    a.K = vs.K;
    a.Kp = vs.Kp;
    a.prec = vs.prec;
    a.out_par = out_par;
    a.eps = eps;
    // FP32 backups cannot resolve changes below a few units in the last
    // place of the values: stop there too (FP64: the bound is below eps)
    a.unit = vs.prec == MORAP_F32 ? 8.0 * std::ldexp(1.0, -24) : 8.0 * std::ldexp(1.0, -53);
    a.best_res = c->d_best_res.as<double>();
    a.stall = c->d_stall.as<int32_t>();
    a.stall_sweeps = vs.prec == MORAP_F32 ? 64 : 0;
    a.floor = 256.0 * std::ldexp(1.0, -24);
    a.tile_base = halo ? c->d_htile_base.as<int32_t>() : c->d_tile_base.as<int32_t>();
    a.act_models = c->d_act_models.as<int32_t>();
    a.act_prefix = c->d_act_prefix.as<int32_t>();
    a.rows_per_model = c->d_rows_per_model.as<int32_t>();
    a.states_per_model = c->d_states_per_model.as<int32_t>();
    a.csr_bytes = vs.prec == MORAP_F32 ? c->d_csr_bytes32.as<int64_t>() : c->d_csr_bytes64.as<int64_t>();
    a.act_tiles = c->d_act_tiles.as<int32_t>();
    return a;
}

static k::SweepArgs sweep_args(morap_ctx* c, ValueSet& vs, int in_par) {
    k::SweepArgs a{};
    a.tiles = c->d_tiles.as<Tile>();
    a.tile_base = c->d_tile_base.as<int32_t>();
    a.act_models = c->d_act_models.as<int32_t>();
    a.act_prefix = c->d_act_prefix.as<int32_t>();
    a.counters = c->d_counters.as<int64_t>();
    a.state_row = c->d_state_row.as<int32_t>();
    a.row_ptr = c->d_row_ptr.as<int32_t>();
    a.col = c->d_col.as<int32_t>();
    const bool f32 = vs.prec == MORAP_F32;
    a.prob = f32 ? c->d_prob32.p : c->d_prob64.p;
    a.rew = f32 ? c->d_rew32.p : c->d_rew64.p;
    a.wc = f32 ? c->d_wc32.p : c->d_wc64.p;
    a.wp = f32 ? c->d_wp32.p : c->d_wp64.p;
    a.active = c->d_active.as<uint8_t>();
    a.x_in = vs.x[in_par].p;
    a.x_out = vs.x[1 - in_par].p;
    a.res = c->d_res.as<unsigned long long>();
    a.ymax = c->d_ymax.as<unsigned long long>();
    a.Kp = vs.Kp;
    a.rec = c->has_blocks ? c->d_blk_rec.as<int32_t>() : nullptr;
    a.ablk = c->has_blocks ? (f32 ? c->d_blk32.p : c->d_blk64.p) : nullptr;
    a.zero_row = (int32_t)c->S;
    a.pattern = c->hm.blk_pattern;
    a.act_tiles = c->d_act_tiles.as<int32_t>();
    a.htiles = c->has_halo ? c->d_htiles.as<HTile>() : nullptr;
    a.hrec = c->has_halo ? c->d_hrec.as<uint2>() : nullptr;
    a.hlist = c->has_halo ? c->d_hlist.as<int32_t>() : nullptr;
    a.rewk = c->team ? (f32 ? c->d_rewk32.p : c->d_rewk64.p) : nullptr;
    return a;
}

// Persistent grid: as many workgroups as the kernel keeps resident on the
// whole chip at once (a second, partial round of workgroups would double the
// time of a balanced sweep), a multiple of 8 (one share per XCD), and no more
// than the tiles need.
static int persistent_grid(morap_ctx* c, int prec, const Variant& v) {
    const int64_t key = ((int64_t)v.id << 8) | prec;
    int per_cu = 0;
    for (auto& r : c->resident)
        if (r.first == key) per_cu = r.second;
    if (per_cu == 0) {
        per_cu = v.kind == SWEEP_HALO                                   ? k::sweep_halo_resident(v, c->hm.blk_pattern)
                 : v.kind == SWEEP_BLOCK                              ? k::sweep_block_resident(prec, v)
                                                                        : k::sweep_resident(prec, v);
        per_cu = std::max(1, per_cu);
        c->resident.push_back({key, per_cu});
    }
    int g = c->prop.multiProcessorCount * per_cu;
    const int tiles = uses_halo_tiles(v) ? (int)c->n_htiles : (int)c->tiles.size();
    g = std::min(g, (tiles + 7) / 8 * 8);
    return std::max(8, g / 8 * 8);
}

using EventPairs = std::vector<std::pair<hipEvent_t, hipEvent_t>>;

// With time_kernels, every kTimedEvery-th sweep launch of a chunk is timed
// (a uniform sample: its average duration is the launches' average, with a
// quarter of the events in the stream)
constexpr int kTimedEvery = 4;

// per-launch timing events come from a pool: creating and destroying two
// events per sweep costs host time on every launch
static hipEvent_t take_event(morap_ctx* c) {
    if (!c->event_pool.empty()) {
        const hipEvent_t e = c->event_pool.back();
        c->event_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    MORAP_HIP(hipEventCreate(&e));
    return e;
}
static void give_events(morap_ctx* c, const std::pair<hipEvent_t, hipEvent_t>& e) {
    if (e.first) c->event_pool.push_back(e.first);
    if (e.second) c->event_pool.push_back(e.second);
}

// Sampled launch events held by a loop; whatever is still held when the
// scope ends (an error thrown mid-chunk included) goes back to the pool.
struct PooledEvents {
    morap_ctx* c;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> v;
    explicit PooledEvents(morap_ctx* ctx) : c(ctx) {}
    PooledEvents(const PooledEvents&) = delete;
    PooledEvents& operator=(const PooledEvents&) = delete;
    ~PooledEvents() {
        for (auto& e : v) give_events(c, e);
    }
};

// Two HIP events bracketing a timed region, destroyed on every way out of
// the scope that owns them.
struct EventPair {
    hipEvent_t a = nullptr, b = nullptr;
    EventPair() {
        MORAP_HIP(hipEventCreate(&a));
        const hipError_t e = hipEventCreate(&b);
        if (e != hipSuccess) {
            (void)hipEventDestroy(a);
            a = nullptr;
            fail(MORAP_E_HIP, std::string("hipEventCreate: ") + hipGetErrorString(e));
        }
    }
    EventPair(const EventPair&) = delete;
    EventPair& operator=(const EventPair&) = delete;
    ~EventPair() {
        if (a) (void)hipEventDestroy(a);
        if (b) (void)hipEventDestroy(b);
    }
    float elapsed_ms() const {
        float ms = 0;
        MORAP_HIP(hipEventElapsedTime(&ms, a, b));
        return ms;
    }
};

// Optional per-launch log (environment variable MORAP_SWEEP_LOG = file path):
// the autotuner's timings and, for solves run with time_kernels, one line per
// sweep launch with its active tile count and duration.
static FILE* sweep_log() {
    static FILE* f = [] {
        const char* p = std::getenv("MORAP_SWEEP_LOG");
        return p && *p ? std::fopen(p, "a") : nullptr;
    }();
    return f;
}

// Launches that share nothing (products of different sizes take different
// kernels) spread over the context's stream and up to three beside it: one
// after the other on one stream each would wait for the last workgroup of
// the one before (64 columns of 10 x 20 products: 3.18 ms a solve on one
// stream, 2.92 on two, 2.87 on four; a support step of 12 x 24: 42.2 / 37.7 /
// 37.1 ms).  Work enqueued on the stream before the fork is seen by all;
// join() (or the end of the scope) makes the stream wait for them.
struct Fork {
    morap_ctx* c;
    int n;   // streams beside the context's in use
    Fork(morap_ctx* ctx, int launches) : c(ctx), n(std::max(0, std::min(launches - 1, 3))) {
        if (n == 0) return;
        if (!c->fork_event) MORAP_HIP(hipEventCreateWithFlags(&c->fork_event, hipEventDisableTiming));
        for (int i = 0; i < n; ++i) {
            if (!c->side[i]) MORAP_HIP(hipStreamCreateWithFlags(&c->side[i], hipStreamNonBlocking));
            if (!c->join_event[i]) MORAP_HIP(hipEventCreateWithFlags(&c->join_event[i], hipEventDisableTiming));
        }
        const int used = n;
        n = 0;
        MORAP_HIP(hipEventRecord(c->fork_event, c->stream));
        for (int i = 0; i < used; ++i) {
            MORAP_HIP(hipStreamWaitEvent(c->side[i], c->fork_event, 0));
            n = i + 1;
        }
    }
    Fork(const Fork&) = delete;
    Fork& operator=(const Fork&) = delete;
    ~Fork() {
        for (int i = 0; i < n; ++i)   // (an error on the way out: nothing may outlive the call)
            (void)hipStreamSynchronize(c->side[i]);
    }
    hipStream_t stream(int i) const { return i % (n + 1) == 0 ? c->stream : c->side[i % (n + 1) - 1]; }
    // for a launch of that much work: the stream with the least so far (beside:
    // not the context's, where other work goes on)
    hipStream_t least(double work, bool beside = false) {
        int at = beside && n > 0 ? 1 : 0;
        for (int i = at + 1; i <= n; ++i)
            if (load[i] < load[at]) at = i;
        load[at] += work;
        return stream(at);
    }
    double load[4] = {0, 0, 0, 0};
    // what follows on the streams beside the context's waits for all before it
    void barrier() {
        for (int i = 0; i < n; ++i) MORAP_HIP(hipEventRecord(c->join_event[i], c->side[i]));
        for (int i = 0; i < n; ++i)
            for (int j = 0; j < n; ++j)
                if (j != i) MORAP_HIP(hipStreamWaitEvent(c->side[i], c->join_event[j], 0));
    }
    void join() {
        for (int i = 0; i < n; ++i) {
            MORAP_HIP(hipEventRecord(c->join_event[i], c->side[i]));
            MORAP_HIP(hipStreamWaitEvent(c->stream, c->join_event[i], 0));
        }
        n = 0;
    }
};

// Streams for launches in LDS beside a chain of short ones on the context's
// stream.  A process has four hardware queues; with a third stream here and a
// caller's work on the null stream two of them share one, and where that is the
// chain's it waits for whole LDS launches: evaluations of 64 columns of 6 x 8
// products of up to 143,000 states 213 (three) and 208 ms (two), of one column 17.6
// and 12.9; the support step of 12 x 24 42.8 and 39.2 ms.  (A solve with more
// pairs in LDS than fit at once is 1 % faster with three.)
constexpr int kBeside = 2;

// one chunk of `n` sweeps (n even): sweep, converge, compact per sweep;
// `ev` (optional) receives an event pair around every sweep kernel
static void enqueue_chunk(morap_ctx* c, ValueSet& vs, const uint8_t* mask, const Variant& v, double eps, int n,
                          EventPairs* ev = nullptr) {
    const int grid = persistent_grid(c, vs.prec, v);
    const int ktiles = vs.Kp / kt_of(v);
    for (int i = 0; i < n; ++i) {
        const int in_par = i & 1;
        const bool timed = ev && i % kTimedEvery == 0;
        if (timed) {
            if (sweep_log() && ev->size() < 4096) {
                c->h_log.ensure(4096 * 8);
                MORAP_HIP(hipMemcpyAsync(c->h_log.as<int64_t>() + ev->size(), c->d_counters.as<int64_t>() + 1, 8,
                                         hipMemcpyDeviceToHost, c->stream));
            }
            ev->emplace_back(take_event(c), nullptr);
            ev->back().second = take_event(c);
            MORAP_HIP(hipEventRecord(ev->back().first, c->stream));
        }
        if (v.kind == SWEEP_HALO)
            k::sweep_halo(c->stream, vs.prec, v, grid, ktiles, sweep_args(c, vs, in_par));
        else if (v.kind == SWEEP_BLOCK)
            k::sweep_block(c->stream, vs.prec, v, grid, ktiles, sweep_args(c, vs, in_par));
        else
            k::sweep(c->stream, vs.prec, v, grid, ktiles, sweep_args(c, vs, in_par));
        if (timed) MORAP_HIP(hipEventRecord(ev->back().second, c->stream));
        const auto ca = converge_args(c, vs, mask, eps, 1 - in_par, uses_halo_tiles(v));
        k::converge(c->stream, ca);
        k::compact(c->stream, ca);
    }
}

static void reset_solve(morap_ctx* c, ValueSet& vs, const uint8_t* mask, double eps, const Variant& v) {
    const int64_t n = (c->S + 1) * vs.Kp;
    if (vs.prec == MORAP_F32) {
        k::fill_f32(c->stream, vs.x[0].as<float>(), 0.f, n);
        k::fill_f32(c->stream, vs.x[1].as<float>(), 0.f, n);
    } else {
        k::fill_f64(c->stream, vs.x[0].as<double>(), 0.0, n);
        k::fill_f64(c->stream, vs.x[1].as<double>(), 0.0, n);
    }
    k::init_solve(c->stream, converge_args(c, vs, mask, eps, 1, uses_halo_tiles(v)));
}

static void release_graph(morap_ctx* c, int g) {
    if (c->chunk_exec[g]) (void)hipGraphExecDestroy(c->chunk_exec[g]);
    if (c->chunk_graph[g]) (void)hipGraphDestroy(c->chunk_graph[g]);
    c->chunk_exec[g] = nullptr;
    c->chunk_graph[g] = nullptr;
    c->graph_key[g].clear();
}

// run one chunk, replaying a captured graph (slot g) when asked to
static void run_chunk(morap_ctx* c, int g, ValueSet& vs, const uint8_t* mask, const Variant& v, double eps, int n,
                      bool graph, EventPairs* ev) {
    if (!graph || ev) {
        enqueue_chunk(c, vs, mask, v, eps, n, ev);
        return;
    }
    char key[320];
    // the key names everything the captured launches hold: the model upload
    // and the solve buffers (by generation, so a buffer reallocated at an
    // old address still counts as new), the variant and the sizes
    snprintf(key, sizeof key, "%llu/%llu/%d/%d/%d/%d/%d/%.17g/%p/%p/%p/%p/%zu", (unsigned long long)c->load_gen,
             (unsigned long long)c->buf_gen, v.id, vs.K, vs.Kp, vs.prec, n, eps, vs.x[0].p, vs.x[1].p,
             (const void*)mask, vs.c.p, c->tiles.size());
    if (c->graph_key[g] != key) {
        release_graph(c, g);
        MORAP_HIP(hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal));
        try {
            enqueue_chunk(c, vs, mask, v, eps, n);
        } catch (...) {
            hipGraph_t gr = nullptr;
            (void)hipStreamEndCapture(c->stream, &gr);
            if (gr) (void)hipGraphDestroy(gr);
            throw;
        }
        MORAP_HIP(hipStreamEndCapture(c->stream, &c->chunk_graph[g]));
        MORAP_HIP(hipGraphInstantiate(&c->chunk_exec[g], c->chunk_graph[g], nullptr, nullptr, 0));
        c->graph_key[g] = key;
    }
    MORAP_HIP(hipGraphLaunch(c->chunk_exec[g], c->stream));
}

static void read_counters(morap_ctx* c) {
    MORAP_HIP(hipMemcpyAsync(c->h_counters.p, c->d_counters.p, 9 * 8, hipMemcpyDeviceToHost, c->stream));
    MORAP_HIP(hipStreamSynchronize(c->stream));
}

// time 6 sweeps of variant v from a fresh start (autotuner)
static double time_variant(morap_ctx* c, ValueSet& vs, const uint8_t* mask, const Variant& v, double eps) {
    EventPair t;
    reset_solve(c, vs, mask, eps, v);
    enqueue_chunk(c, vs, mask, v, eps, 2);
    MORAP_HIP(hipEventRecord(t.a, c->stream));
    enqueue_chunk(c, vs, mask, v, eps, 6);
    MORAP_HIP(hipEventRecord(t.b, c->stream));
    MORAP_HIP(hipEventSynchronize(t.b));
    return t.elapsed_ms();
}

// autotuner: the fastest candidate variant for (precision, padded width,
// restricted or not), timed on the loaded models and cached on the context
// (`refine`: the masked re-solve of assigned pairs; a mask without it holds the
// models whose values do not fit LDS)
static const Variant& choose_variant(morap_ctx* c, ValueSet& vs, const uint8_t* mask, bool refine, double eps,
                                     int schedule) {
    if (schedule > 0) {
        const Variant& v = variant_by_id(schedule);
        MORAP_CHECK(vs.Kp % kt_of(v) == 0, MORAP_E_INVALID, "variant does not divide the padded column count");
        MORAP_CHECK(v.kind != SWEEP_BLOCK || c->has_blocks, MORAP_E_UNSUPPORTED,
                    "the neighbourhood-block sweep needs products built from agents with at most 5 actions "
                    "and 5 successors per state");
        MORAP_CHECK(v.kind != SWEEP_HALO || (c->has_halo && vs.prec == MORAP_F32), MORAP_E_UNSUPPORTED,
                    "the LDS-staged sweep needs halo tiles (built with the block form) and FP32 values");
        return v;
    }
    const int64_t key = ((int64_t)vs.prec << 40) | ((int64_t)(refine ? 1 : (mask ? 2 : 0)) << 32) | vs.Kp;
    for (auto& t : c->tuned)
        if (t.first == key) return variant_by_id(t.second);
    // The largest products beside products in LDS, not timed (a timing takes a
    // third of a first solve): the LDS-staged kernel with four states in flight
    // where they hold a third of the states (2 x 12 products of up to 140,000
    // states, 87 % of all, 64 columns: 169 ms, 183 with the gather sweep and its
    // hand-over; 20 x 15 products, 43 %: 197 and 210).  Below, few tiles stay active
    // and either will do (27 %: 201 and 199): the wave gather sweep, which hands
    // over to the staged kernel where a check finds under 20 % of the tiles active.
    if (mask && !refine && c->has_halo && vs.prec == MORAP_F32 && vs.Kp % 64 == 0)
        return variant_by_id(c->resident_plan.part[vs.prec].rest_share > 1.0 / 3 ? 40 : 37);
    auto cand = candidates(vs.Kp, refine, c->has_blocks, c->has_halo && vs.prec == MORAP_F32);
    MORAP_CHECK(!cand.empty(), MORAP_E_UNSUPPORTED, "no sweep variant for this column count");
    int best = cand[0].id;
    if (cand.size() > 1) {
        double best_ms = 1e300;
        // the timing covers full sweeps only; a wave-per-state gather sweep
        // also gets the LDS-staged kernel for the last sweeps of a solve
        // (~4 % of its time saved on the 50 x 100 workload), so the others
        // must beat it by 3 %
        const bool tail_possible = !refine && c->has_halo && vs.prec == MORAP_F32 && vs.Kp % 64 == 0;
        for (const auto& v : cand) {
            const bool gets_tail = tail_possible && v.kind == SWEEP_BLOCK && v.cpl == 1 && v.lps == 64;
            const double raw = time_variant(c, vs, mask, v, eps);
            const double ms = raw * (tail_possible && !gets_tail ? 1.03 : 1.0);
            if (sweep_log())
                std::fprintf(sweep_log(), "tune prec=%d mask=%d Kp=%d variant=%d kind=%d cpl=%d lps=%d grid=%d ms=%.4f\n",
                             vs.prec, mask != nullptr, vs.Kp, v.id, v.kind, v.cpl, v.lps,
                             persistent_grid(c, vs.prec, v), raw);
            if (ms < best_ms) {
                best_ms = ms;
                best = v.id;
            }
        }
    }
    c->tuned.push_back({key, best});
    return variant_by_id(best);
}

// Batched value iteration into `vs` until every (masked) pair has converged.
static void swap_buf(DevBuf& a, DevBuf& b) {
    std::swap(a.p, b.p);
    std::swap(a.bytes, b.bytes);
    std::swap(a.meter, b.meter);
}

// For the message of a solve that hit its sweep limit: the first pairs still
// active, each with its two weights and the change between the last two
// iterates (the two value buffers) at its most-changing state.
static std::string describe_active(morap_ctx* c, ValueSet& vs) {
    const int M = c->hm.M, Kp = vs.Kp;
    std::vector<uint8_t> act((size_t)M * Kp);
    MORAP_HIP(hipMemcpy(act.data(), c->d_active.p, act.size(), hipMemcpyDeviceToHost));
    const size_t el = vs.prec == MORAP_F32 ? 4 : 8;
    std::string out;
    int shown = 0;
    for (int m = 0; m < M && shown < 4; ++m)
        for (int k = 0; k < vs.K && shown < 4; ++k) {
            if (!act[(size_t)m * Kp + k]) continue;
            const int32_t s0 = c->hm.state_base[m], s1 = c->hm.state_base[m + 1];
            std::vector<char> b0((size_t)(s1 - s0) * Kp * el + 8), b1(b0.size());
            MORAP_HIP(hipMemcpy(b0.data(), vs.x[0].as<char>() + (size_t)s0 * Kp * el, b0.size() - 8,
                                hipMemcpyDeviceToHost));
            MORAP_HIP(hipMemcpy(b1.data(), vs.x[1].as<char>() + (size_t)s0 * Kp * el, b1.size() - 8,
                                hipMemcpyDeviceToHost));
            double dmax = -1, v0 = 0, v1 = 0;
            int at = -1;
            for (int32_t s = 0; s < s1 - s0; ++s) {
                const size_t i = (size_t)s * Kp + k;
                const double a = el == 4 ? reinterpret_cast<float*>(b0.data())[i] : reinterpret_cast<double*>(b0.data())[i];
                const double b = el == 4 ? reinterpret_cast<float*>(b1.data())[i] : reinterpret_cast<double*>(b1.data())[i];
                if (std::fabs(a - b) > dmax) {
                    dmax = std::fabs(a - b);
                    at = s;
                    v0 = a;
                    v1 = b;
                }
            }
            const int d = n_obj_of(c);
            const int i = m / c->hm.nJ, j = m % c->hm.nJ;
            const double wc = c->team ? 1.0 : c->W[(size_t)k * d + i];
            const double wp = c->team ? 0.0 : c->W[(size_t)k * d + c->hm.nI + j];
            char buf[320];
            std::snprintf(buf, sizeof buf,
                          "%s (model %d, column %d: weights %.9g, %.9g; last change %.6g at state %d, %.9g -> "
                          "%.9g)",
                          shown ? "," : ":", m, k, wc, wp, dmax, at, v0, v1);
            out += buf;
            ++shown;
        }
    return out;
}

// warm: the solve starts from the values prepared in d_xwarm (they become
// the first sweep's input buffer)
// The LDS-staged sweep for the last sweeps of a solve whose kernel is the
// wave-per-state gather sweep: the two give identical values, and once few
// tiles stay active (the last large models) the staged one is faster.
static const Variant* tail_variant(morap_ctx* c, const ValueSet& vs, bool refine, const Variant& v, int schedule) {
    if (refine || schedule != 0 || !c->has_halo || vs.prec != MORAP_F32 || vs.Kp % 64 != 0) return nullptr;
    if (v.kind != SWEEP_BLOCK || v.cpl != 1 || v.lps != 64) return nullptr;
    for (const auto& t : variants())
        if (t.kind == SWEEP_HALO && t.unroll == 2) return &t;
    return nullptr;
}
// switch below this share of the tiles (MORAP_TAIL_PERCENT overrides it,
// 0 never switches)
static int tail_percent() {
    static const int p = [] {
        const char* e = std::getenv("MORAP_TAIL_PERCENT");
        return e && *e ? std::max(0, std::min(100, std::atoi(e))) : 20;
    }();
    return p;
}

// id reported for a solve whose values all stayed in LDS
constexpr int kResidentVariant = 41;

// sweeps of one launch of the LDS-resident iteration: the host looks in
// between, so that a solve that does not converge stays interruptible
constexpr int kResidentSweeps = 4096;

// What a solve reports, in pinned memory behind one synchronisation: the
// sweeps of every pair, the values at the initial states and the counters.
static void read_results(morap_ctx* c, const ValueSet& vs) {
    const size_t ps = (size_t)c->hm.M * vs.Kp * 4, cv = (size_t)vs.K * c->hm.M * 8;
    c->h_pair_sweeps.ensure(ps);
    c->h_c.ensure(cv);
    if (ps + cv <= k::REPORT_BYTES) {
        k::report(c->stream, (int64_t)(ps / 4), c->d_pair_sweeps.as<int32_t>(), c->h_pair_sweeps.as<int32_t>(),
                  (int64_t)(cv / 8), vs.c.as<double>(), c->h_c.as<double>(), c->d_counters.as<int64_t>(),
                  c->h_counters.as<int64_t>());
        MORAP_HIP(hipStreamSynchronize(c->stream));
        return;
    }
    MORAP_HIP(hipMemcpyAsync(c->h_pair_sweeps.p, c->d_pair_sweeps.p, ps, hipMemcpyDeviceToHost, c->stream));
    MORAP_HIP(hipMemcpyAsync(c->h_c.p, vs.c.p, cv, hipMemcpyDeviceToHost, c->stream));
    read_counters(c);
}

static k::ResidentArgs resident_args(morap_ctx* c, ValueSet& vs, const k::ConvergeArgs& ca) {
    const HostModels& hm = c->hm;
    const bool f32 = vs.prec == MORAP_F32;
    k::ResidentArgs a{};
    a.state_base = c->d_state_base.as<int32_t>();
    a.init = c->d_init.as<int32_t>();
    a.rec = c->d_blk_rec.as<int32_t>();
    a.ablk = f32 ? c->d_blk32.p : c->d_blk64.p;
    a.zero_row = (int32_t)c->S;
    const ResidentPlan& plan = c->resident_plan;
    a.grid_blk = f32 ? plan.grid_blk32.p : plan.grid_blk64.p;
    a.grid_mat = plan.grid_mat.as<float>();
    a.big_base = plan.big_base.as<int32_t>();
    a.big_block = plan.big_block.as<int32_t>();
    a.big_rec = plan.big_rec.as<uint4>();
    a.big_init = plan.big_init.as<int32_t>();
    a.W = c->d_weights.as<double>();
    a.nI = hm.nI;
    a.nJ = hm.nJ;
    a.d = hm.nI + hm.nJ;
    a.K = vs.K;
    a.Kp = vs.Kp;
    a.M = hm.M;
    a.x0 = vs.x[0].p;
    a.x1 = vs.x[1].p;
    a.active = ca.active;
    a.final_par = ca.final_par;
    a.pair_sweeps = ca.pair_sweeps;
    a.c = ca.c;
    a.best_res = ca.best_res;
    a.stall = ca.stall;
    a.counters = ca.counters;
    a.eps = ca.eps;
    a.unit = ca.unit;
    a.floor = ca.floor;
    a.stall_sweeps = ca.stall_sweeps;
    return a;
}

// The pairs of the plan's models to their stop with the values in LDS
// (pair_sweeps cleared before), up to `limit` sweeps each; their statistics
// as the batched sweeps count them.  The values land in vs.x[0].
// `beside` runs on the context's stream while the first launches do.
static void run_resident(morap_ctx* c, ValueSet& vs, const ResidentPlan::Part& part, const morap_vi_opts& o,
                         bool warm, int64_t limit, int chunk, Stats& st,
                         const std::function<void()>& beside = nullptr) {
    const HostModels& hm = c->hm;
    const bool f32 = vs.prec == MORAP_F32;
    const ResidentPlan& plan = c->resident_plan;
    k::ResidentArgs a = resident_args(c, vs, converge_args(c, vs, nullptr, o.eps_vi, 0, false));
    a.warm = warm ? 1 : 0;
    // several columns per workgroup share a state's probabilities and rows,
    // unless all pairs run at once anyway: one column each ends sooner then
    const int cus = c->prop.multiProcessorCount;
    const bool wide = (int64_t)part.models.size() * vs.K > 2 * (int64_t)cus;
    PooledEvents held(c);
    int64_t done = 0, running = 0;
    const int32_t* ps = nullptr;
    for (int64_t s0 = 0; s0 < limit; s0 = done) {
        done = std::min<int64_t>(limit, s0 + kResidentSweeps);
        a.sweep0 = (int)s0;
        a.sweep1 = (int)done;
        a.last = done == limit ? 1 : 0;
        // (timed launches one by one)
        Fork fork(c, o.time_kernels ? 1 : (!beside ? (int)part.launches.size()
                                                   : 1 + std::min((int)part.launches.size(), wide ? 3 : kBeside)));
        for (size_t q = 0; q < part.launches.size(); ++q) {
            const auto& l = part.launches[q];
            a.order = plan.order.as<int32_t>() + l.begin;
            a.n_models = l.n;
            if (o.time_kernels) {
                held.v.emplace_back(take_event(c), nullptr);
                held.v.back().second = take_event(c);
                MORAP_HIP(hipEventRecord(held.v.back().first, c->stream));
            }
            double work = 0;   // (the plan lists the larger products first)
            for (int b = l.first; b < l.first + l.n; ++b) {
                const int32_t m = part.models[(size_t)b];
                work += hm.state_base[m + 1] - hm.state_base[m];
            }
            // (FP32 rates with one, two and four columns a workgroup; FP64's are
            // weighed alike)
            const hipStream_t s = fork.least(work * (l.columns == 1 ? 1.8 : (l.columns == 2 ? 1.4 : 1.0)), (bool)beside);
            if (l.rows && l.columns == 0) {
                a.short_base = plan.short_base.as<int32_t>();
                a.short_rec = plan.short_rec.as<uint4>();
                a.short_val = f32 ? plan.short_val32.p : plan.short_val64.p;
                k::resident_short(s, vs.prec, wide, l.max_states, a);
            } else if (l.rows) {
                k::RowsArgs ra{};
                static_cast<k::ResidentArgs&>(ra) = a;
                ra.slice = plan.row_slice.as<int32_t>();
                ra.batch = plan.row_batch.as<int32_t>();
                ra.desc = plan.row_desc.as<int32_t>();
                ra.place = plan.row_place.as<uint2>();
                ra.value = f32 ? plan.row_value32.p : plan.row_value64.p;
                k::resident_rows(s, vs.prec, wide ? l.columns : 1, l.max_states, ra);
            } else if (l.columns > 0) k::resident_large(s, vs.prec, wide ? l.columns : 1, l.max_states, a);
            else k::resident(s, vs.prec, l.fast, wide, l.max_states, a);
            if (o.time_kernels) MORAP_HIP(hipEventRecord(held.v.back().second, c->stream));
        }
        if (beside && s0 == 0) beside();
        fork.join();
        read_results(c, vs);
        ps = c->h_pair_sweeps.as<int32_t>();
        running = 0;
        for (int32_t m : part.models)
            for (int k = 0; k < vs.K; ++k) running += ps[(size_t)m * vs.Kp + k] == 0;
        if (running == 0) break;
    }
    if (running > 0)
        fail(MORAP_E_NOT_CONVERGED, "value iteration: " + std::to_string(running) +
                                        " (model, column) pairs still active after " + std::to_string(limit) +
                                        " sweeps" + describe_active(c, vs));
    const double el = f32 ? 4 : 8;
    int64_t longest = 0;
    for (int32_t m : part.models) {
        int64_t sum = 0, top = 0;
        for (int k = 0; k < vs.K; ++k) {
            const int64_t n = ps[(size_t)m * vs.Kp + k];
            sum += n;
            top = std::max(top, n);
        }
        const int32_t b = hm.state_base[m], e = hm.state_base[m + 1];
        const int64_t rows = hm.state_row[e] - hm.state_row[b];
        const int64_t nnz = hm.row_ptr[hm.state_row[e]] - hm.row_ptr[hm.state_row[b]];
        st.backups += rows * sum;
        st.bytes += (double)top * (4.0 * (e - b) + 4.0 * rows + 4.0 * nnz + el * nnz + 2.0 * el * rows) +
                    2.0 * el * (double)(e - b) * (double)sum;
        longest = std::max(longest, top);
    }
    st.max_pair_sweeps = std::max(st.max_pair_sweeps, longest);
    st.sweeps = std::max<int64_t>(st.sweeps, (longest + chunk - 1) / chunk * chunk);
    st.resident_models = (int)part.models.size();
    if (part.n_rest == 0) {
        st.variant = kResidentVariant;
        if (!c->has_blocks)   // products given as rows: the CSR sweep of that width
            for (const auto& v : variants())
                if (v.kind == SWEEP_CSR && kt_of(v) == std::min(vs.Kp, 64)) {
                    st.variant = v.id;
                    break;
                }
    }
    for (size_t q = 0; q < held.v.size(); ++q) {
        float t = 0;
        MORAP_HIP(hipEventElapsedTime(&t, held.v[q].first, held.v[q].second));
        if (part.n_rest == 0) {
            st.ms_sweep_kernel += t;
            st.sweep_launches += 1;
        }
        if (sweep_log()) {
            const auto& l = part.launches[q % part.launches.size()];
            double work = 0;   // state-columns of the launch's models
            for (int b = l.first; b < l.first + l.n; ++b) {
                const int32_t m = part.models[(size_t)b];
                for (int k = 0; k < vs.K; ++k)
                    work += (double)ps[(size_t)m * vs.Kp + k] * (hm.state_base[m + 1] - hm.state_base[m]);
            }
            std::fprintf(sweep_log(), "resident prec=%d fast=%d columns=%d models=%d states=%d ms=%.4f state_columns=%.4g\n",
                         vs.prec, l.fast, l.columns, l.n, l.max_states, t, work);
        }
    }
}

// The plan of the models whose values stay in LDS in a solve, nullptr with a
// fixed schedule and where the block form or its models are missing.
static const ResidentPlan::Part* resident_part(morap_ctx* c, int prec, const morap_vi_opts& o) {
    const ResidentPlan::Part& part = c->resident_plan.part[prec];
    return c->team || o.schedule != 0 || part.launches.empty() ? nullptr : &part;
}

static void run_vi(morap_ctx* c, int g, ValueSet& vs, const uint8_t* mask, const morap_vi_opts& o, Stats& st,
                   bool warm = false) {
    const bool refine = mask != nullptr;
    const int chunk = std::max(2, (o.check_every + 1) / 2 * 2);
    // products that fit keep their values in LDS; the batched sweeps take the
    // rest (all of them with a fixed schedule)
    const ResidentPlan::Part* part = refine ? nullptr : resident_part(c, vs.prec, o);
    const int64_t limit = ((int64_t)o.max_sweeps + chunk - 1) / chunk * chunk;
    if (part && part->n_rest == 0) {
        EventPair wall;
        if (warm) {
            swap_buf(vs.x[0], c->d_xwarm);
            ++c->buf_gen;   // graphs hold the value buffers' addresses
        } else if (c->resident_plan.unsolved) {
            // (values of models without a live initial state)
            if (vs.prec == MORAP_F32) k::fill_f32(c->stream, vs.x[0].as<float>(), 0.f, (c->S + 1) * vs.Kp);
            else k::fill_f64(c->stream, vs.x[0].as<double>(), 0.0, (c->S + 1) * vs.Kp);
        }
        const int64_t n_W = (int64_t)vs.K * (c->hm.nI + c->hm.nJ);
        k::init_pairs(c->stream, converge_args(c, vs, nullptr, o.eps_vi, 0, false), c->h_weights.as<double>(),
                      c->d_weights.as<double>(), n_W <= k::SMALL_WEIGHTS ? n_W : 0);
        MORAP_HIP(hipEventRecord(wall.a, c->stream));
        run_resident(c, vs, *part, o, warm, limit, chunk, st);
        MORAP_HIP(hipEventRecord(wall.b, c->stream));
        MORAP_HIP(hipEventSynchronize(wall.b));
        st.floor_stops += c->h_counters.as<int64_t>()[8];
        st.ms_vi += wall.elapsed_ms();
        vs.valid = true;
        return;
    }
    if (part) {
        if (c->d_rest_mask.ensure((size_t)c->hm.M * vs.Kp)) ++c->buf_gen;
        k::model_mask(c->stream, c->hm.M, vs.Kp, part->d_rest.as<uint8_t>(), c->d_rest_mask.as<uint8_t>());
        mask = c->d_rest_mask.as<uint8_t>();
    }
    const Variant& v0 = choose_variant(c, vs, mask, refine, o.eps_vi, o.schedule);
    c->last_variant = v0.id;
    const Variant* vt = tail_variant(c, vs, refine, v0, o.schedule);
    const Variant* vp = &v0;   // the kernel of the next chunk
    double bytes_at_switch = -1;
    int64_t sweeps_at_switch = 0;
    EventPair wall;
    reset_solve(c, vs, mask, o.eps_vi, v0);
    if (warm) {
        swap_buf(vs.x[0], c->d_xwarm);
        ++c->buf_gen;   // graphs hold the value buffers' addresses
    } else if (c->team) {
        // a team model starts below its optimum over proper policies (the
        // values of a fixed proper policy), which value iteration then
        // reaches instead of an improper fixed point above it
        k::team_start(c->stream, c->S, vs.K, vs.Kp, n_obj_of(c), c->d_team_w.as<double>(),
                      c->d_team_E.as<double>(), vs.prec, vs.x[0].p);
    }
    MORAP_HIP(hipEventRecord(wall.a, c->stream));
    int64_t launched = 0;
    int64_t* h = c->h_counters.as<int64_t>();
    PooledEvents held(c);
    EventPairs& ev = held.v;
    auto harvest = [&] {
        for (size_t i = 0; i < ev.size(); ++i) {
            auto& e = ev[i];
            float t = 0;
            MORAP_HIP(hipEventElapsedTime(&t, e.first, e.second));
            if (sweep_log() && i < 4096)
                std::fprintf(sweep_log(), "sweep prec=%d mask=%d variant=%d tiles=%lld ms=%.4f\n", vs.prec,
                             mask != nullptr, vp->id, (long long)c->h_log.as<int64_t>()[i], t);
            if (refine) {
                st.ms_sweep_kernel_refine += t;
                st.sweep_launches_refine += 1;
            } else if (vp != &v0) {
                st.ms_sweep_kernel_tail += t;
                st.sweep_launches_tail += 1;
            } else {
                st.ms_sweep_kernel += t;
                st.sweep_launches += 1;
            }
            give_events(c, e);
            e = {nullptr, nullptr};
        }
        ev.clear();
    };
    const size_t el = vs.prec == MORAP_F32 ? 4 : 8;
    const int64_t main_tiles = (int64_t)c->tiles.size();
    int64_t first_tiles = 0;   // active after the first chunk
    auto sweeps = [&] {        // one chunk; true when no pair is active any more
        run_chunk(c, vp == &v0 ? g : 2, vs, mask, *vp, o.eps_vi, chunk, o.use_graph != 0,
                  o.time_kernels ? &ev : nullptr);
        launched += chunk;
        read_counters(c);
        harvest();
        if (h[3] == 0) return true;
        if (first_tiles == 0) first_tiles = h[1];
        if (vt && vp == &v0 && h[1] * 100 < main_tiles * tail_percent()) {
            // the same active models listed over the halo tiles
            bytes_at_switch = (double)h[6] + 2.0 * el * (double)h[7];
            sweeps_at_switch = h[5];
            vp = vt;
            k::relist(c->stream, converge_args(c, vs, mask, o.eps_vi, 0, true));
        }
        if (launched >= o.max_sweeps)
            fail(MORAP_E_NOT_CONVERGED, "value iteration: " + std::to_string(h[3]) +
                                            " (model, column) pairs still active after " +
                                            std::to_string(launched) + " sweeps" + describe_active(c, vs));
        return false;
    };
    bool over = false;
    if (part) {
        // the batched sweeps alone while they fill the device, then (fewer
        // than half of the first tiles active) beside the launches in LDS:
        // 24 agents on 32 x 32 .. 128 x 128 grids x 32 tasks, 64 columns, 203
        // -> 199 ms and, another draw, 184 -> 178 (the LDS kernels leave few
        // compute units to the sweeps until they end)
        while (!over && (first_tiles == 0 || h[1] * 2 > first_tiles)) over = sweeps();
        run_resident(c, vs, *part, o, warm, limit, chunk, st, [&] {
            while (!over) over = sweeps();
        });
    }
    while (!over) over = sweeps();
    MORAP_HIP(hipEventRecord(wall.b, c->stream));
    MORAP_HIP(hipEventSynchronize(wall.b));
    const float ms = wall.elapsed_ms();
    std::vector<int32_t> ps((size_t)c->hm.M * vs.Kp);
    MORAP_HIP(hipMemcpy(ps.data(), c->d_pair_sweeps.p, ps.size() * 4, hipMemcpyDeviceToHost));
    st.backups += h[4];
    st.floor_stops += h[8];
    const double bytes = (double)h[6] + 2.0 * el * (double)h[7];
    if (refine) {
        st.bytes_refine += bytes;
    } else if (bytes_at_switch >= 0) {
        st.bytes += bytes_at_switch;
        st.bytes_tail += bytes - bytes_at_switch;
        st.sweeps_tail += h[5] - sweeps_at_switch;
        st.variant_tail = vt->id;
    } else {
        st.bytes += bytes;
    }
    st.max_pair_sweeps = std::max<int64_t>(st.max_pair_sweeps, *std::max_element(ps.begin(), ps.end()));
    st.ms_vi += ms;
    if (refine) st.variant_refine = v0.id;
    else st.variant = v0.id;
    if (refine) st.polish_sweeps += h[5];
    else st.sweeps = std::max<int64_t>(st.sweeps, h[5]);   // (a solve's own statistics)
    vs.valid = true;
}

// ---------------------------------------------------------------------------
// solve
// ---------------------------------------------------------------------------
static void add_stats(Stats& a, const Stats& b) {
    a.backups += b.backups;
    a.sweeps += b.sweeps;
    a.max_pair_sweeps = std::max(a.max_pair_sweeps, b.max_pair_sweeps);
    a.eval_sweeps += b.eval_sweeps;
    a.polish_sweeps += b.polish_sweeps;
    a.rank_rounds += b.rank_rounds;
    a.floor_stops += b.floor_stops;
    a.bytes += b.bytes;
    a.ms_vi += b.ms_vi;
    a.ms_eval += b.ms_eval;
    a.ms_total += b.ms_total;
    a.ms_sweep_kernel += b.ms_sweep_kernel;
    a.sweep_launches += b.sweep_launches;
    a.bytes_refine += b.bytes_refine;
    a.ms_sweep_kernel_refine += b.ms_sweep_kernel_refine;
    a.sweep_launches_refine += b.sweep_launches_refine;
    a.sweeps_tail += b.sweeps_tail;
    a.sweep_launches_tail += b.sweep_launches_tail;
    a.bytes_tail += b.bytes_tail;
    a.ms_sweep_kernel_tail += b.ms_sweep_kernel_tail;
    a.variant_tail = b.variant_tail ? b.variant_tail : a.variant_tail;
    a.refine_pairs += b.refine_pairs;
    a.refine_columns += b.refine_columns;
    a.variant = b.variant ? b.variant : a.variant;
    a.resident_models = b.variant ? b.resident_models : a.resident_models;
    a.variant_refine = b.variant_refine ? b.variant_refine : a.variant_refine;
}

static void solve_impl(morap_ctx* c, const double* W, int K, const morap_vi_opts& o, double* c_out, Stats& st,
                       const int32_t* warm);
static void evaluate_impl(morap_ctx* c, const int32_t* assign, int K, const morap_vi_opts& o, double* r_out,
                          Stats& st, const int32_t* warm);

// f(false) with the layouts in LDS order; where that runs out of memory which they
// hold, f(true) without them: what fits beside the batched sweeps is not refused
// for them.
template <class F>
static void with_layouts(morap_ctx* c, F&& f) {
    try {
        const LayoutsInUse use(c);
        return f(false);
    } catch (const MorapError& e) {
        if (e.code != MORAP_E_OOM || !drop_layouts(c)) throw;
    }
    f(true);
}

void solve(morap_ctx* c, const double* W, int K, const morap_vi_opts& o, double* c_out, Stats& st,
           const int32_t* warm) {
    Stats local;
    with_layouts(c, [&](bool again) {
        local = Stats();
        // (again: the values a warm start reads may be gone)
        solve_impl(c, W, K, o, c_out, local, again ? nullptr : warm);
    });
    add_stats(st, local);
    add_stats(c->cum, local);
}

static std::vector<double> resolve_pairs(morap_ctx* c, const std::vector<int32_t>& pk,
                                         const std::vector<int32_t>& pm, const morap_vi_opts& o, Stats& st);
static int refine_assignment(morap_ctx* c, const int32_t* assign, int K, const morap_vi_opts& o, Stats& st,
                             int32_t* out);

void evaluate(morap_ctx* c, const int32_t* assign, int K, const morap_vi_opts& o, double* r_out, Stats& st,
              const int32_t* warm, int32_t* refine) {
    Stats local;
    c->eval_prev_valid = c->eval_prev_valid && c->prev_eval_gen == c->load_gen;
    with_layouts(c, [&](bool) {
        local = Stats();
        try {
            evaluate_impl(c, assign, K, o, r_out, local, warm);
            if (refine) {
                std::copy(assign, assign + (size_t)K * c->hm.nJ, refine);
                if (!c->team && c->prec == MORAP_F32 && c->has_blocks && c->last_c64_valid &&
                    refine_assignment(c, assign, K, o, local, refine) > 0) {
                    // again with the new assignment, each instance started from
                    // the first evaluation's values where the pair is unchanged
                    std::vector<int32_t> same(K);
                    for (int k = 0; k < K; ++k) same[k] = k;
                    evaluate_impl(c, refine, K, o, r_out, local, same.data());
                }
            }
        } catch (...) {
            c->eval_prev_valid = false;
            throw;
        }
    });
    add_stats(st, local);
    add_stats(c->cum, local);
}

// rows of W[K][d] on the simplex: finite, >= 0, summing to 1 (1e-9)
static void check_weight_rows(const double* W, int K, int d) {
    for (int k = 0; k < K; ++k) {
        double sum = 0;
        for (int q = 0; q < d; ++q) {
            const double w = W[(size_t)k * d + q];
            MORAP_CHECK(std::isfinite(w) && w >= 0, MORAP_E_INVALID, "weights must be finite and >= 0");
            sum += w;
        }
        MORAP_CHECK(std::fabs(sum - 1.0) <= 1e-9, MORAP_E_INVALID, "weight rows must sum to 1");
    }
}

static void solve_impl(morap_ctx* c, const double* W, int K, const morap_vi_opts& o, double* c_out, Stats& st,
                       const int32_t* warm) {
    MORAP_CHECK(c->loaded, MORAP_E_STATE, "no models loaded");
    MORAP_CHECK(W && K >= 1 && K <= 4096, MORAP_E_INVALID, "need 1 <= K <= 4096 weight vectors");
    MORAP_CHECK(o.precision == MORAP_F32 || o.precision == MORAP_F64, MORAP_E_INVALID, "bad precision");
    MORAP_CHECK(o.eps_vi > 0 && std::isfinite(o.eps_vi), MORAP_E_INVALID, "eps_vi must be > 0");
    MORAP_CHECK(o.max_sweeps >= 1, MORAP_E_INVALID, "max_sweeps must be >= 1");
    const int nI = c->hm.nI, nJ = c->hm.nJ, M = c->hm.M, d = n_obj_of(c);
    check_weight_rows(W, K, d);
    const auto t0 = std::chrono::steady_clock::now();
    const int prec = o.precision;
    const int Kp = padded_k(K);
    // a warm start needs the previous FP32 values in buffers that already
    // fit this solve (they are read in place)
    const size_t need = (size_t)(c->S + 1) * Kp * 4;
    const bool warm_ok = warm && !c->team && prec == MORAP_F32 && c->vmain.valid && c->vmain.prec == MORAP_F32 &&
                         Kp <= c->vmain.Kp && c->vmain.x[0].bytes >= need && c->vmain.x[1].bytes >= need;
    const int Kp_old = c->vmain.Kp, K_old = c->vmain.K;
    // Per pair, the start a x_prev + b from the previous values x_prev, which
    // are (up to the stop rule) the optimal values V = wc_o C + wp_o P of the
    // previous weights, C <= 0 and P in [0, 1] the cost and probability
    // values of the previous optimal policy.  Every start is below the new
    // optimum V', so value iteration climbs to it as from 0 and zero-reward
    // loops (which admit larger fixed points) cannot hold it above:
    //  * probability only now and before: V' = (wp_n / wp_o) V exactly (the
    //    optimal policies do not depend on the scale); a relative 1e-6 below
    //    it covers the previous stop (FP32 stops at 8 2^-24 relative);
    //  * a cost weight now and before: V' >= wc_n C >= (wc_n / wc_o)(V - wp_o),
    //    the previous policy's value without its probability reward;
    //  * otherwise from 0, as Alg. 3.
    std::vector<float> warm_ab;
    if (warm_ok) {
        const std::vector<double>& Wp = c->W;   // the previous solve's weights [K_old][d]
        warm_ab.assign((size_t)M * Kp * 2, 0.f);
        for (int k = 0; k < K; ++k) {
            MORAP_CHECK(warm[k] >= -1 && warm[k] < K_old, MORAP_E_INVALID, "warm-start column out of range");
            if (warm[k] < 0) continue;
            for (int m = 0; m < M; ++m) {
                const int i = m / nJ, j = m % nJ;
                const double wc_n = W[(size_t)k * d + i], wp_n = W[(size_t)k * d + nI + j];
                const double wc_o = Wp[(size_t)warm[k] * d + i], wp_o = Wp[(size_t)warm[k] * d + nI + j];
                double a = 0, b = 0;
                if (wc_n == 0 && wc_o == 0 && wp_o > 0) {
                    a = wp_n / wp_o * (1.0 - 1e-6);
                } else if (wc_n > 0 && wc_o > 0) {
                    a = wc_n / wc_o;
                    b = -a * wp_o;
                }
                warm_ab[((size_t)m * Kp + k) * 2] = (float)a;
                warm_ab[((size_t)m * Kp + k) * 2 + 1] = (float)b;
            }
        }
    }
    c->solved = false;
    c->evaluated = false;
    ensure_scratch(c, Kp);
    c->K = K;
    c->Kp = Kp;
    c->prec = prec;
    c->W.assign(W, W + (size_t)K * d);

    const ResidentPlan::Part* part = resident_part(c, prec, o);
    const bool batched = !part || part->n_rest > 0;   // some models take the batched sweeps
    if (part) {
        c->d_weights.ensure((size_t)K * d * 8);
        c->h_weights.ensure((size_t)K * d * 8);
        std::memcpy(c->h_weights.p, W, (size_t)K * d * 8);
        if (batched || (int64_t)K * d > k::SMALL_WEIGHTS)   // (else with the start of the pairs)
            MORAP_HIP(hipMemcpyAsync(c->d_weights.p, c->h_weights.p, (size_t)K * d * 8, hipMemcpyHostToDevice, c->stream));
    }
    // per-(model, column) weights of the model's two objectives (a team
    // model: its rows are scalarised per column on the device instead, and
    // (1, 0) marks the column in use)
    const size_t nw = batched ? (size_t)M * Kp : 0;
    std::vector<double> wc(nw, 0.0), wp(nw, 0.0);
    std::vector<float> wc32(nw, 0.f), wp32(nw, 0.f);
    for (int m = 0; batched && m < M; ++m) {
        const int i = m / nJ, j = m % nJ;
        for (int k = 0; k < K; ++k) {
            wc[(size_t)m * Kp + k] = c->team ? 1.0 : W[(size_t)k * d + i];
            wp[(size_t)m * Kp + k] = c->team ? 0.0 : W[(size_t)k * d + nI + j];
            wc32[(size_t)m * Kp + k] = (float)wc[(size_t)m * Kp + k];
            wp32[(size_t)m * Kp + k] = (float)wp[(size_t)m * Kp + k];
        }
    }
    if (batched) {
        MORAP_HIP(hipMemcpyAsync(c->d_wc64.p, wc.data(), wc.size() * 8, hipMemcpyHostToDevice, c->stream));
        MORAP_HIP(hipMemcpyAsync(c->d_wp64.p, wp.data(), wp.size() * 8, hipMemcpyHostToDevice, c->stream));
        MORAP_HIP(hipMemcpyAsync(c->d_wc32.p, wc32.data(), wc32.size() * 4, hipMemcpyHostToDevice, c->stream));
        MORAP_HIP(hipMemcpyAsync(c->d_wp32.p, wp32.data(), wp32.size() * 4, hipMemcpyHostToDevice, c->stream));
    }
    if (c->team) {
        // every (row, column)'s reward w[obj[r][0]] rew[r][0] + w[obj[r][1]] rew[r][1]
        const int64_t R = c->hm.state_row.back();
        bool moved = c->d_team_w.ensure((size_t)K * d * 8);
        moved |= c->d_rewk64.ensure((size_t)R * Kp * 8 + 8);
        moved |= c->d_rewk32.ensure((size_t)R * Kp * 4 + 8);
        if (moved) ++c->buf_gen;
        MORAP_HIP(hipMemcpyAsync(c->d_team_w.p, W, (size_t)K * d * 8, hipMemcpyHostToDevice, c->stream));
        k::team_rewards(c->stream, R, K, Kp, d, c->d_team_w.as<double>(), c->d_obj.as<int32_t>(),
                        c->d_rew64.as<double>(), c->d_rewk64.as<double>(), c->d_rewk32.as<float>());
    }
    if (warm_ok) {
        c->d_warm_map.ensure((size_t)K * 4);
        c->d_warm_ab.ensure(warm_ab.size() * 4);
        c->d_xwarm.ensure(need);
        MORAP_HIP(hipMemcpyAsync(c->d_warm_map.p, warm, (size_t)K * 4, hipMemcpyHostToDevice, c->stream));
        MORAP_HIP(hipMemcpyAsync(c->d_warm_ab.p, warm_ab.data(), warm_ab.size() * 4, hipMemcpyHostToDevice,
                                 c->stream));
        k::warm_columns(c->stream, c->S, Kp, K, c->d_warm_map.as<int32_t>(), c->d_state_model.as<int32_t>(),
                        c->d_warm_ab.as<float>(), c->vmain.x[0].as<float>(), c->vmain.x[1].as<float>(),
                        c->vmain.final_par.as<uint8_t>(), Kp_old, c->d_xwarm.as<float>());
    }
    ensure_values(c, c->vmain, K, Kp, prec);
    if (batched || warm_ok) MORAP_HIP(hipStreamSynchronize(c->stream));   // the host vectors go out of scope

    run_vi(c, 0, c->vmain, nullptr, o, st, warm_ok);
    if (c_out && !batched)
        std::memcpy(c_out, c->h_c.p, (size_t)K * M * 8);   // read with the end of the solve
    else if (c_out)
        MORAP_HIP(hipMemcpyAsync(c_out, c->vmain.c.p, (size_t)K * M * 8, hipMemcpyDeviceToHost, c->stream));
    if (batched) MORAP_HIP(hipStreamSynchronize(c->stream));
    st.ms_total += std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    c->solved = true;
}

// ---------------------------------------------------------------------------
// evaluate: FP64 values of the assigned pairs, policy extraction, Alg. 4
// ---------------------------------------------------------------------------
static k::InstArgs inst_args(morap_ctx* c, int n_tiles, int n_inst) {
    k::InstArgs a{};
    a.n_tiles = n_tiles;
    a.n_inst = n_inst;
    a.state_base = c->d_state_base.as<int32_t>();
    a.state_row = c->d_state_row.as<int32_t>();
    a.row_ptr = c->d_row_ptr.as<int32_t>();
    a.col = c->d_col.as<int32_t>();
    a.prob = c->d_prob64.as<double>();
    a.rew = c->d_rew64.as<double>();
    a.to_done = c->d_to_done.as<uint8_t>();
    a.init = c->d_init.as<int32_t>();
    a.cus = c->prop.multiProcessorCount;
    if (c->team) {
        a.rewk = c->d_rewk64.as<double>();
        a.rewk_ld = c->Kp;
        a.row_obj = c->d_obj.as<int32_t>();
        a.inst_obj = c->d_inst_obj.as<int32_t>();
    }
    return a;
}

// widenings of the tie tolerance in policy extraction (tau * 10^k, k <= 6)
constexpr int kTauSteps = 6;

// Stop of the FP64 values a pair's policy is chosen from (R16): eps_vi, or
// 1e-4 eps_vi (not below 1e-12, never above eps_vi) when the scaled cost
// weight vanishes.  Then every action that completes the task as surely as
// the best is optimal, and values stopped at eps_vi differ between such
// actions by their own error, far above the tie tolerance: the greedy
// choice among them is decided by that error and can be an action that
// progresses only through a slip (hundreds of thousands of expected steps,
// which no evaluation finishes).
static double policy_eps(double eps_vi, double wc, double wp) {
    if (wc < 1e-6 && wp > 0) return std::min(eps_vi, std::max(eps_vi * 1e-4, 1e-12));
    return eps_vi;
}

// Host arrays of a set of instances, sent to the device in one copy.
struct InstancePack {
    std::vector<char> bytes;
    template <class T> size_t add(const std::vector<T>& v) {
        const size_t at = (bytes.size() + 15) / 16 * 16;
        bytes.resize(at + v.size() * sizeof(T) + 16);
        if (!v.empty()) std::memcpy(bytes.data() + at, v.data(), v.size() * sizeof(T));
        return at;
    }
    char* send(DevBuf& d, PinnedBuf& h, hipStream_t s) const {
        d.ensure(bytes.size() + 16);
        h.ensure(bytes.size() + 16);
        std::memcpy(h.p, bytes.data(), bytes.size());
        MORAP_HIP(hipMemcpyAsync(d.p, h.p, bytes.size(), hipMemcpyHostToDevice, s));
        return d.as<char>();
    }
};

// Instances (column, model): weights scaled to sum 1, state offsets, and how
// their iterations run: in LDS, one workgroup each (`order`, in launches), or
// over tiles of 256 states of the others.
struct Instances {
    struct Run {
        int begin, n, max_states;
        bool fast, large;
    };
    int n = 0, n_general = 0;
    std::vector<int32_t> k, m, tiles, order;
    std::vector<int64_t> base, init_idx;
    std::vector<double> wc, wp, scale, eps;
    std::vector<uint8_t> resident;
    std::vector<Run> vi;
    int64_t states() const { return base[(size_t)n]; }

    // d_model, ... of the device copy
    const int32_t *d_model = nullptr, *d_k = nullptr, *d_tiles = nullptr, *d_order = nullptr;
    const int64_t *d_base = nullptr, *d_init = nullptr;
    const double *d_wc = nullptr, *d_wp = nullptr, *d_scale = nullptr, *d_eps = nullptr;
    const uint8_t* d_resident = nullptr;

    void build(morap_ctx* c, std::vector<int32_t> ks, std::vector<int32_t> ms, bool policies, const morap_vi_opts& o) {
        const HostModels& hm = c->hm;
        const bool team = c->team;
        const int nI = hm.nI, nJ = hm.nJ, d = nI + nJ;
        k = std::move(ks);
        m = std::move(ms);
        n = (int)k.size();
        base.assign((size_t)n + 1, 0);
        init_idx.assign((size_t)n, -1);
        wc.resize((size_t)n);
        wp.resize((size_t)n);
        scale.assign((size_t)n, 0.0);
        eps.resize((size_t)n);
        resident.assign((size_t)n, 0);
        const bool lds = c->has_blocks && !team;
        // instances that run in LDS by the place of their model in the plan's
        // order (largest first within a launch class)
        const std::vector<int32_t>& rank = c->resident_plan.rank;
        std::vector<int32_t> first(lds ? c->resident_plan.n_order + 2 : 0, 0);
        for (int q = 0; q < n; ++q) {
            const int mq = m[q], i = mq / nJ, j = mq % nJ;
            const int S_m = hm.state_base[mq + 1] - hm.state_base[mq];
            base[q + 1] = base[q] + S_m;
            wc[q] = team ? 1.0 : c->W[(size_t)k[q] * d + i];
            wp[q] = team ? 0.0 : c->W[(size_t)k[q] * d + nI + j];
            const double sum = wc[q] + wp[q];   // policies come from the weights scaled to sum 1
            if (sum > 0) {
                wc[q] /= sum;
                wp[q] /= sum;
                scale[q] = 1.0 / sum;
            }
            eps[q] = policies && !team ? policy_eps(o.eps_vi, wc[q], wp[q]) : o.eps_vi;
            if (hm.init[mq] >= 0) init_idx[q] = base[q] + (hm.init[mq] - hm.state_base[mq]);
            if (S_m == 0) continue;
            if (lds && c->resident_plan.inst_ok[(size_t)mq]) {
                resident[q] = 1;
                ++first[(size_t)rank[(size_t)mq] + 1];
                continue;
            }
            ++n_general;
            for (int b = 0; b < S_m; b += 256) {
                tiles.push_back(q);
                tiles.push_back(b);
            }
        }
        if (!lds) return;
        for (size_t r = 1; r < first.size(); ++r) first[r] += first[r - 1];
        for (const auto& l : c->resident_plan.part[MORAP_F64].launches) {
            const int b = first[(size_t)l.begin], e = first[(size_t)(l.begin + l.n)];
            if (e > b) vi.push_back({b, e - b, l.max_states, l.fast, l.columns > 0});
        }
        order.resize((size_t)first.back());
        for (int q = 0; q < n; ++q)
            if (resident[q]) order[(size_t)first[(size_t)rank[(size_t)m[q]]]++] = q;
    }

    // launches over `order` of instances whose sizes fall in one class
    template <class F>
    std::vector<Run> runs(morap_ctx* c, F&& size_class) const {
        std::vector<Run> out;
        for (int p = 0; p < (int)order.size(); ++p) {
            const int mq = m[(size_t)order[p]];
            const int S_m = c->hm.state_base[mq + 1] - c->hm.state_base[mq];
            if (!out.empty() && size_class(out.back().max_states) == size_class(S_m)) {
                ++out.back().n;
                out.back().max_states = std::max(out.back().max_states, S_m);
            } else {
                out.push_back({p, 1, S_m, false, false});
            }
        }
        return out;
    }

    // everything above (and what `p` already holds) on the device
    char* send(InstancePack& p, DevBuf& d, PinnedBuf& h, hipStream_t s) {
        const size_t at[] = {p.add(m),  p.add(k),  p.add(tiles), p.add(order), p.add(base),    p.add(init_idx),
                             p.add(wc), p.add(wp), p.add(scale), p.add(eps),   p.add(resident)};
        char* b = p.send(d, h, s);
        d_model = reinterpret_cast<int32_t*>(b + at[0]);
        d_k = reinterpret_cast<int32_t*>(b + at[1]);
        d_tiles = reinterpret_cast<int32_t*>(b + at[2]);
        d_order = reinterpret_cast<int32_t*>(b + at[3]);
        d_base = reinterpret_cast<int64_t*>(b + at[4]);
        d_init = reinterpret_cast<int64_t*>(b + at[5]);
        d_wc = reinterpret_cast<double*>(b + at[6]);
        d_wp = reinterpret_cast<double*>(b + at[7]);
        d_scale = reinterpret_cast<double*>(b + at[8]);
        d_eps = reinterpret_cast<double*>(b + at[9]);
        d_resident = reinterpret_cast<uint8_t*>(b + at[10]);
        return b;
    }

    k::InstArgs args(morap_ctx* c) const {
        k::InstArgs a = inst_args(c, (int)(tiles.size() / 2), n);
        a.inst_model = d_model;
        a.inst_k = d_k;
        a.inst_base = d_base;
        a.inst_tiles = d_tiles;
        a.resident = d_resident;
        return a;
    }

    // value iteration in LDS, sweeps s0 + 1 .. s1 of the instances without a
    // stop in `sweeps`, from the FP32 solve's values (after an FP64 solve from 0)
    // (beside: on the streams of that fork other than the context's, not joined)
    void launch_vi(morap_ctx* c, double* x, int32_t* sweeps, int64_t s0, int64_t s1, EventPairs* ev,
                   Fork* beside = nullptr) const {
        k::ResidentArgs a{};
        a.state_base = c->d_state_base.as<int32_t>();
        a.init = c->d_init.as<int32_t>();
        a.rec = c->d_blk_rec.as<int32_t>();
        a.ablk = c->d_blk64.p;
        a.zero_row = (int32_t)c->S;
        a.grid_blk = c->resident_plan.grid_blk64.p;
        a.big_base = c->resident_plan.big_base.as<int32_t>();
        a.big_block = c->resident_plan.big_block.as<int32_t>();
        a.big_rec = c->resident_plan.big_rec.as<uint4>();
        a.big_init = c->resident_plan.big_init.as<int32_t>();
        a.K = 1;
        a.x0 = x;
        a.pair_sweeps = sweeps;
        a.inst_model = d_model;
        a.inst_k = d_k;
        a.inst_base = d_base;
        a.iwc = d_wc;
        a.iwp = d_wp;
        a.ieps = d_eps;
        a.iscale = d_scale;
        if (c->prec == MORAP_F32 && c->vmain.valid) {
            a.start0 = c->vmain.x[0].as<float>();
            a.start1 = c->vmain.x[1].as<float>();
            a.start_par = c->vmain.final_par.as<uint8_t>();
            a.start_Kp = c->vmain.Kp;
        }
        a.sweep0 = (int)s0;
        a.sweep1 = (int)s1;
        std::unique_ptr<Fork> own;
        if (!beside) own.reset(new Fork(c, ev ? 1 : (int)vi.size()));   // (timed launches one by one)
        Fork& fork = beside ? *beside : *own;
        for (size_t q = 0; q < vi.size(); ++q) {
            const Run& r = vi[q];
            a.order = d_order + r.begin;
            a.n_models = r.n;
            if (ev) {
                ev->emplace_back(take_event(c), nullptr);
                ev->back().second = take_event(c);
                MORAP_HIP(hipEventRecord(ev->back().first, c->stream));
            }
            // (an instance's time follows its size: a launch's, its largest one's
            // and how many they are)
            const hipStream_t s =
                fork.least((double)r.max_states * (1.0 + r.n / (double)c->prop.multiProcessorCount), beside != nullptr);
            if (r.large) k::resident_inst_large(s, r.max_states, a);
            else k::resident_inst(s, r.fast, r.max_states, a);
            if (ev) MORAP_HIP(hipEventRecord(ev->back().second, c->stream));
        }
        if (own) own->join();
    }

    // sweeps the value iteration took as the tiled iteration counts them
    // (whole chunks), and the bytes it would have moved; still running: > 0
    int64_t account(morap_ctx* c, const int32_t* sweeps, int chunk, Stats& st) const {
        int64_t longest = 0;
        for (int32_t q : order) {
            const int64_t up = ((int64_t)sweeps[q] + chunk - 1) / chunk * chunk;
            longest = std::max(longest, up);
            // record + own value read + write per state
            st.bytes_refine += (double)up * (double)(base[q + 1] - base[q]) * 48.0;
        }
        return longest;
    }
    int64_t running(const int32_t* sweeps, int width) const {
        int64_t r = 0;
        for (int32_t q : order)
            for (int w = 0; w < width; ++w) r += sweeps[(size_t)q * width + w] == 0;
        return r;
    }
};

static void harvest_refine(morap_ctx* c, EventPairs& ev, Stats& st) {
    for (auto& e : ev) {
        float t = 0;
        MORAP_HIP(hipEventElapsedTime(&t, e.first, e.second));
        st.ms_sweep_kernel_refine += t;
        st.sweep_launches_refine += 1;
        give_events(c, e);
        e = {nullptr, nullptr};
    }
    ev.clear();
}

static void evaluate_impl(morap_ctx* c, const int32_t* assign, int K, const morap_vi_opts& o, double* r_out,
                          Stats& st, const int32_t* warm) {
    MORAP_CHECK(c->solved, MORAP_E_STATE, "morap_evaluate needs a morap_solve first");
    MORAP_CHECK(K == c->K, MORAP_E_INVALID, "K differs from the last morap_solve");
    MORAP_CHECK(assign != nullptr || c->team, MORAP_E_INVALID, "assign is NULL");
    MORAP_CHECK(o.eps_eval > 0 && o.eps_vi > 0 && o.tau >= 0, MORAP_E_INVALID, "bad tolerances");
    const bool team = c->team;
    const int nI = c->hm.nI, nJ = team ? (n_obj_of(c) + 1) / 2 : c->hm.nJ, d = team ? n_obj_of(c) : nI + nJ;
    // A team model has one policy per column; its instances (one per pair of
    // objectives, nJ per column) evaluate that policy's objectives 2p, 2p+1.
    std::vector<int32_t> team_assign;
    if (team) {
        team_assign.assign((size_t)K * nJ, 0);
        assign = team_assign.data();
    }
    const int cap = team ? nJ : std::max(1, (nJ + nI - 1) / nI);
    for (int kk = 0; kk < K; ++kk) {
        std::vector<int> load(nI, 0);
        for (int j = 0; j < nJ; ++j) {
            const int i = assign[(size_t)kk * nJ + j];
            MORAP_CHECK(i >= 0 && i < nI, MORAP_E_INVALID, "assigned agent out of range");
            MORAP_CHECK(++load[i] <= cap, MORAP_E_INVALID, "an agent received more than ceil(|J|/|I|) tasks");
        }
    }
    const auto t0 = std::chrono::steady_clock::now();
    hipStream_t s = c->stream;
    c->evaluated = false;
    // instances (k, m), task-major within each column
    const int n = K * nJ;
    c->assign.assign(assign, assign + (size_t)K * nJ);
    Instances I;
    {
        std::vector<int32_t> ks((size_t)n), ms((size_t)n);
        for (int kk = 0; kk < K; ++kk)
            for (int j = 0; j < nJ; ++j) {
                ks[(size_t)kk * nJ + j] = kk;
                ms[(size_t)kk * nJ + j] = team ? 0 : assign[(size_t)kk * nJ + j] * nJ + j;
            }
        I.build(c, std::move(ks), std::move(ms), true, o);
    }
    c->inst_k = I.k;
    c->inst_m = I.m;
    c->inst_base = I.base;
    const std::vector<int32_t>& tiles = I.tiles;
    const std::vector<double>&iwc = I.wc, &iwp = I.wp, &iscale = I.scale;
    const int64_t NS = I.states();
    const bool lds = !I.order.empty(), general = I.n_general > 0;
    double eps_pol = o.eps_vi;
    for (double e : I.eps) eps_pol = std::min(eps_pol, e);
    c->d_xi.ensure((size_t)NS * 8 + 8);
    c->d_ires.ensure((size_t)2 * n * 8);
    c->d_iactive.ensure((size_t)2 * n);
    c->d_ipar.ensure((size_t)2 * n);
    if (general) {
        c->d_mask.ensure((size_t)NS * 4 + 4);
        c->d_rank.ensure((size_t)NS * 4 + 4);
        c->d_xe[1].ensure((size_t)NS * 16 + 16);
    }
    c->d_mu.ensure((size_t)NS + 4);
    c->d_xe[0].ensure((size_t)NS * 16 + 16);
    c->d_init_val.ensure((size_t)3 * n * 8);
    std::vector<int32_t> iobj;
    if (team) {
        iobj.resize((size_t)2 * n);
        for (int q = 0; q < n; ++q) {
            const int p = q % nJ;
            iobj[2 * q] = 2 * p;
            iobj[2 * q + 1] = 2 * p + 1 < d ? 2 * p + 1 : -1;
        }
        c->d_inst_obj.ensure((size_t)2 * n * 4);
        MORAP_HIP(hipMemcpyAsync(c->d_inst_obj.p, iobj.data(), iobj.size() * 4, hipMemcpyHostToDevice, s));
    }
    // evaluations that start from the previous one's values of the same pair
    std::vector<uint8_t> iwarm(n, 0);
    std::vector<int64_t> prev_src(n, -1);
    if (warm && c->eval_prev_valid && c->prev_per_col == nJ) {
        const int K_prev = (int)(c->prev_inst_m.size() / std::max(1, nJ));
        for (int kk = 0; kk < K; ++kk) {
            const int kp = warm[kk];
            MORAP_CHECK(kp >= -1, MORAP_E_INVALID, "warm-start column out of range");
            if (kp < 0 || kp >= K_prev) continue;
            for (int j = 0; j < nJ; ++j) {
                const int q = kk * nJ + j, qp = kp * nJ + j;
                if (c->prev_inst_m[qp] != c->inst_m[q]) continue;
                iwarm[q] = 1;
                prev_src[q] = c->prev_inst_base[qp];
            }
        }
    }
    InstancePack pack;
    const size_t at_warm = pack.add(iwarm), at_prev = pack.add(prev_src);
    const char* packed = I.send(pack, c->d_inst_pack, c->h_inst_pack, s);
    const uint8_t* d_iwarm = reinterpret_cast<const uint8_t*>(packed + at_warm);
    const k::InstArgs a = I.args(c);
    int64_t* dctr = c->d_counters.as<int64_t>();
    int64_t* h = c->h_counters.as<int64_t>();
    unsigned long long* ires = c->d_ires.as<unsigned long long>();
    uint8_t* iact = c->d_iactive.as<uint8_t>();
    uint8_t* ipar = c->d_ipar.as<uint8_t>();
    const int chunk = std::max(2, (o.check_every + 1) / 2 * 2);

    // Tiles of the instances that still have an active entry (width entries
    // per instance): the sweeps between two host checks launch only these.
    auto live_tiles = [&](const uint8_t* dflags, int width, k::InstArgs& out) {
        std::vector<uint8_t> f((size_t)width * n);
        // (copies on this stream: the null stream's queue can be one that a stream
        // with launches in LDS shares, and would wait for them)
        MORAP_HIP(hipMemcpyAsync(f.data(), dflags, f.size(), hipMemcpyDeviceToHost, s));
        MORAP_HIP(hipStreamSynchronize(s));
        c->h_live_tiles.clear();
        int64_t states = 0;
        for (size_t t = 0; t < tiles.size() / 2; ++t) {
            const int inst = tiles[2 * t];
            bool on = false;
            for (int w = 0; w < width; ++w) on |= f[(size_t)inst * width + w] != 0;
            if (!on) continue;
            c->h_live_tiles.push_back(tiles[2 * t]);
            c->h_live_tiles.push_back(tiles[2 * t + 1]);
            const int m = c->inst_m[inst];
            states += std::min<int64_t>(256, c->hm.state_base[m + 1] - c->hm.state_base[m] - tiles[2 * t + 1]);
        }
        c->d_live_tiles.ensure(c->h_live_tiles.size() * 4 + 8);
        if (!c->h_live_tiles.empty())
            MORAP_HIP(hipMemcpyAsync(c->d_live_tiles.p, c->h_live_tiles.data(), c->h_live_tiles.size() * 4,
                                     hipMemcpyHostToDevice, s));
        out = a;
        out.inst_tiles = c->d_live_tiles.as<int32_t>();
        out.n_tiles = (int)(c->h_live_tiles.size() / 2);
        return states;
    };

    // Values for the policies: FP64 value iteration from 0 on exactly the
    // assigned pairs, with each model's two weights scaled to sum 1.  Scaling
    // leaves the optimal policies unchanged; it keeps the absolute stop test
    // and the tie tolerance meaningful when both weights are tiny (the
    // unscaled iteration then stops after a sweep or two and its greedy
    // policy can take ~1e6 steps to finish).  With the neighbourhood-block
    // form the instances iterate in their own (instance-major) values;
    // otherwise the batched sweep re-solves the marked pairs.
    double* xi = c->d_xi.as<double>();
    // what the iterations in LDS report: sweeps of the values [n] and of the
    // evaluation [2 n], then two counters
    const size_t out_words = (size_t)3 * n + 3;   // (3: room to align the counters)
    c->d_inst_out.ensure(out_words * 4 + 16);
    c->h_inst_out.ensure(out_words * 4 + 16);
    int32_t* vi_sweeps = c->d_inst_out.as<int32_t>();
    int32_t* ev_sweeps = vi_sweeps + n;
    int64_t* inst_ctr = reinterpret_cast<int64_t*>(vi_sweeps + ((size_t)3 * n + 1) / 2 * 2);
    const int32_t* h_sweeps = c->h_inst_out.as<int32_t>();
    const int64_t* h_ctr = reinterpret_cast<const int64_t*>(h_sweeps + ((size_t)3 * n + 1) / 2 * 2);
    const int64_t vi_limit = ((int64_t)o.max_sweeps + chunk - 1) / chunk * chunk;
    auto read_out = [&] {
        MORAP_HIP(hipMemcpyAsync(c->h_inst_out.p, c->d_inst_out.p, out_words * 4 + 16, hipMemcpyDeviceToHost, s));
        MORAP_HIP(hipStreamSynchronize(s));
    };
    const bool warm_values = c->prec == MORAP_F32 && c->vmain.valid;
    if (c->has_blocks && general && !warm_values) k::fill_f64(s, xi, 0.0, NS);
    double* xe0 = c->d_xe[0].as<double>();
    double* xe1 = c->d_xe[1].as<double>();
    int8_t* mu = c->d_mu.as<int8_t>();

    // the instances in LDS: policies, then the first sweeps of the evaluation;
    // all launched before the host looks at how the values ended
    k::InstanceArgs ia{};
    ia.inst_model = I.d_model;
    ia.inst_base = I.d_base;
    ia.state_base = c->d_state_base.as<int32_t>();
    ia.rec = c->d_blk_rec.as<int32_t>();
    ia.ablk = c->d_blk64.as<double>();
    ia.zero_row = (int32_t)c->S;
    ia.iwc = I.d_wc;
    ia.iwp = I.d_wp;
    ia.xi = xi;
    ia.mu = mu;
    ia.tau = o.tau;
    ia.widenings = kTauSteps;
    ia.counters = inst_ctr;
    ia.xe = xe0;
    ia.xe_prev = c->d_xe_prev.as<double>();
    ia.prev_src = reinterpret_cast<const int64_t*>(packed + at_prev);
    ia.from_values = o.eval_start ? 1 : 0;
    ia.sweeps = ev_sweeps;
    ia.eps = o.eps_eval;
    // with larger products beside them, the instances in LDS go through all
    // their steps on other streams while those take theirs on the context's:
    // a support step of 12 agents x 24 tasks whose largest products have 24,000
    // states 43.2 -> 42.0 ms
    std::unique_ptr<Fork> beside;
    auto launch = [&](const std::vector<Instances::Run>& runs, auto&& kernel) {
        std::unique_ptr<Fork> own;
        if (!beside) own.reset(new Fork(c, (int)runs.size()));
        Fork& fork = beside ? *beside : *own;
        for (size_t q = 0; q < runs.size(); ++q) {
            ia.order = I.d_order + runs[q].begin;
            ia.n = runs[q].n;
            kernel(fork.least((double)ia.n * runs[q].max_states, (bool)beside), runs[q].max_states, ia);
        }
        if (own) own->join();
        else beside->barrier();
    };
    // (a policy instance's LDS use follows its size: classes of one, two, four
    // and more workgroups a compute unit)
    const auto policy_runs = I.runs(c, [](int S_m) { return S_m <= 2500 ? 0 : (S_m <= 5000 ? 1 : 2); });
    const auto eval_runs = I.runs(c, [](int S_m) { return k::eval_class(S_m); });
    const int64_t eval_limit = ((int64_t)o.max_sweeps + chunk - 1) / chunk * chunk;
    int64_t esweeps = 0;
    auto policies_and_values = [&] {
        launch(policy_runs, k::inst_policy);
        ia.sweep0 = 0;
        ia.sweep1 = (int)std::min<int64_t>(eval_limit, kResidentSweeps);
        launch(eval_runs, k::inst_eval);
    };
    // Alg. 4 per objective, from 0, or (warm) each instance whose column's
    // previous column had an instance of the same task on the same model from
    // that instance's final values, and (eval_start) from the scalarised
    // values: the evaluation of a proper policy reaches its values from any
    // start, with the same bound on the error at its stop
    if (general) {
        std::vector<int64_t> runs;
        for (int q = 0; q < n; ++q) {
            if (I.resident[q] || !iwarm[q]) continue;
            runs.push_back(I.base[q]);
            runs.push_back(prev_src[q]);
            runs.push_back(I.base[q + 1] - I.base[q]);
        }
        k::fill_f64(s, xe0, 0.0, 2 * NS);
        k::fill_f64(s, xe1, 0.0, 2 * NS);
        if (!runs.empty()) {
            c->d_warm_copy.ensure(runs.size() * 8);
            MORAP_HIP(hipMemcpyAsync(c->d_warm_copy.p, runs.data(), runs.size() * 8, hipMemcpyHostToDevice, s));
            k::copy_runs(s, c->d_warm_copy.as<int64_t>(), (int)(runs.size() / 3), c->d_xe_prev.as<double>(), xe0);
            MORAP_HIP(hipStreamSynchronize(s));   // the host run list goes out of scope
        }
    }
    EventPair vi_wall;
    PooledEvents vi_events(c);
    if (lds) {
        k::fill_i32(s, vi_sweeps, 0, (int64_t)out_words + 4);
        if (general && c->has_blocks && !o.time_kernels) beside.reset(new Fork(c, 1 + kBeside));
        MORAP_HIP(hipEventRecord(vi_wall.a, s));
        I.launch_vi(c, xi, vi_sweeps, 0, std::min<int64_t>(vi_limit, kResidentSweeps),
                    o.time_kernels ? &vi_events.v : nullptr, beside.get());
        MORAP_HIP(hipEventRecord(vi_wall.b, s));
        if (beside) {
            beside->barrier();
            policies_and_values();
        }
    }
    int64_t vsweeps = 0;
    c->last_c64_valid = false;
    if (c->has_blocks && general) {
        c->d_xr.ensure((size_t)NS * 8 + 8);
        double* x0 = xi;
        double* x1 = c->d_xr.as<double>();
        // after an FP32 solve the re-solve starts from its values (scaled to
        // the instance's weights); after an FP64 solve from 0, as Alg. 3
        if (warm_values)
            k::warm_start(s, a, c->vmain.x[0].p, c->vmain.x[1].p, c->vmain.final_par.as<uint8_t>(), c->vmain.Kp, I.d_scale,
                          I.d_wc, x0);
        k::fill_f64(s, x1, 0.0, NS);
        k::set_active(s, n, a, iact, ires, ipar, 1);
        EventPair wall;
        MORAP_HIP(hipEventRecord(wall.a, s));
        k::InstArgs av = a;
        int64_t live_states = 0;
        for (int q = 0; q < n; ++q)
            if (!I.resident[q]) live_states += I.base[q + 1] - I.base[q];
        PooledEvents held(c);
        EventPairs& ev = held.v;
        while (true) {
            for (int i = 0; i < chunk; ++i) {
                const bool even = (i & 1) == 0;
                const bool timed = o.time_kernels && i % kTimedEvery == 0;
                if (timed) {
                    ev.emplace_back(take_event(c), nullptr);
                    ev.back().second = take_event(c);
                    MORAP_HIP(hipEventRecord(ev.back().first, s));
                }
                k::inst_vi_sweep(s, av, c->d_blk_rec.as<int32_t>(), c->d_blk64.as<double>(), I.d_wc, I.d_wp, iact,
                                 even ? x0 : x1, even ? x1 : x0, ires, (int32_t)c->S, c->hm.blk_pattern);
                if (timed) MORAP_HIP(hipEventRecord(ev.back().second, s));
                k::inst_converge(s, n, ires, iact, ipar, even ? 1 : 0, o.eps_vi, dctr, I.d_eps);
            }
            vsweeps += chunk;
            // record + own value read + write per live instance state
            st.bytes_refine += (double)chunk * (double)live_states * 48.0;
            read_counters(c);
            harvest_refine(c, ev, st);
            if (h[0] == 0) break;
            MORAP_CHECK(vsweeps < o.max_sweeps, MORAP_E_NOT_CONVERGED,
                        "value iteration of the assigned pairs: " + std::to_string(h[0]) +
                            " instances still active after " + std::to_string(vsweeps) + " sweeps");
            live_states = live_tiles(iact, 1, av);
        }
        k::select_final(s, a, x0, x1, ipar, 1);
        MORAP_HIP(hipEventRecord(wall.b, s));
        MORAP_HIP(hipEventSynchronize(wall.b));
        st.ms_vi += wall.elapsed_ms();
    } else if (!c->has_blocks) {
        const int M = c->hm.M, Kp = c->Kp;
        std::vector<double> wc((size_t)M * Kp, 0.0), wp((size_t)M * Kp, 0.0);
        for (int kk = 0; kk < K; ++kk)
            for (int m = 0; m < M; ++m) {
                const int i = m / c->hm.nJ, j = m % c->hm.nJ;
                double a0 = team ? 1.0 : c->W[(size_t)kk * d + i], a1 = team ? 0.0 : c->W[(size_t)kk * d + nI + j];
                const double sc = a0 + a1;
                if (sc > 0) {
                    a0 /= sc;
                    a1 /= sc;
                }
                wc[(size_t)m * Kp + kk] = a0;
                wp[(size_t)m * Kp + kk] = a1;
            }
        MORAP_HIP(hipMemcpyAsync(c->d_wc64.p, wc.data(), wc.size() * 8, hipMemcpyHostToDevice, s));
        MORAP_HIP(hipMemcpyAsync(c->d_wp64.p, wp.data(), wp.size() * 8, hipMemcpyHostToDevice, s));
        MORAP_HIP(hipStreamSynchronize(s));   // the host vectors go out of scope
        ensure_values(c, c->vref, K, c->Kp, MORAP_F64);
        uint8_t* pm = c->d_pair_mask.as<uint8_t>();
        k::fill_u8(s, pm, 0, (int64_t)c->hm.M * c->Kp);
        k::mark_pairs(s, a, c->Kp, pm);
        // one stop for the masked batched re-solve: the tightest any pair needs
        morap_vi_opts op = o;
        op.eps_vi = eps_pol;
        run_vi(c, 1, c->vref, pm, op, st);
        k::gather_columns(s, a, MORAP_F64, c->vref.x[0].p, c->vref.x[1].p, c->vref.final_par.as<uint8_t>(),
                          c->vref.Kp, xi);
    }

    EventPair wall;
    MORAP_HIP(hipEventRecord(wall.a, s));
    auto finish_lds = [&] {
        if (beside) {
            beside->join();
            beside.reset();
        } else {
            policies_and_values();
        }
        read_out();
        for (int64_t s0 = kResidentSweeps; I.running(h_sweeps, 1) > 0; s0 += kResidentSweeps) {
            if (s0 < vi_limit) {
                I.launch_vi(c, xi, vi_sweeps, s0, std::min<int64_t>(vi_limit, s0 + kResidentSweeps), nullptr);
                read_out();
            }
            MORAP_CHECK(s0 + kResidentSweeps < vi_limit || I.running(h_sweeps, 1) == 0, MORAP_E_NOT_CONVERGED,
                        "value iteration of the assigned pairs: " + std::to_string(I.running(h_sweeps, 1)) +
                            " instances still active after " + std::to_string(vi_limit) + " sweeps");
            if (I.running(h_sweeps, 1) == 0) {
                // again from the final values
                k::fill_i32(s, ev_sweeps, 0, (int64_t)out_words + 4 - n);
                policies_and_values();
                read_out();
            }
        }
        harvest_refine(c, vi_events.v, st);
        st.ms_vi += vi_wall.elapsed_ms();
        vsweeps = std::max(vsweeps, I.account(c, h_sweeps, chunk, st));
        st.rank_rounds += h_ctr[1];
        if (h_ctr[0] != 0)
            fail(MORAP_E_IMPROPER, std::to_string(h_ctr[0]) + " states cannot reach done through tau-optimal actions");
        for (int64_t s0 = ia.sweep1; I.running(h_sweeps + n, 2) > 0 && s0 < eval_limit; s0 = ia.sweep1) {
            ia.sweep0 = (int)s0;
            ia.sweep1 = (int)std::min<int64_t>(eval_limit, s0 + kResidentSweeps);
            launch(eval_runs, k::inst_eval);
            read_out();
        }
        for (int32_t q : I.order)
            for (int w = 0; w < 2; ++w) {
                const int64_t e = h_sweeps[(size_t)n + 2 * (size_t)q + w];
                esweeps = std::max(esweeps, e > 0 ? (e + chunk - 1) / chunk * chunk : eval_limit);
            }
    };
    if (lds && !beside) finish_lds();

    if (general) {
        // Attractor rounds with the tolerance tau; states left unranked get
        // the tolerance widened tenfold (up to tau * 1e6) while ranked states
        // keep their choice.
        uint32_t* mask = c->d_mask.as<uint32_t>();
        int32_t* rank = c->d_rank.as<int32_t>();
        c->d_ichanged.ensure((size_t)n + 8);
        uint8_t* ichg = c->d_ichanged.as<uint8_t>();
        k::opt_mask(s, a, I.d_wc, I.d_wp, xi, o.tau, mask, rank, mu, false);
        int base = 0, relax_sweeps = 0;
        double tau = o.tau;
        for (int widen = 0;; ++widen) {
            // ranks of this phase: relax to the fixed point (8 sweeps per check,
            // alternating direction; converged when the last sweep changed
            // nothing).  After a round only the tiles of instances that changed
            // in it are relaxed again: ranks spread only inside an instance.
            k::InstArgs ar = a;
            for (int round = 0;; ++round) {
                k::fill_i64(s, dctr, 0, 8);
                k::fill_u8(s, ichg, 0, n);
                for (int i = 0; i < 8; ++i)
                    k::relax_ranks(s, ar, mask, rank, base, (i & 1) != 0, 16, dctr + i, ichg);
                relax_sweeps += 8;
                read_counters(c);
                if (h[7] == 0) break;
                MORAP_CHECK(round < 1000000, MORAP_E_IMPROPER, "attractor ranks did not settle");
                live_tiles(ichg, 1, ar);
            }
            k::fill_i64(s, dctr, 0, 1);
            k::choose_actions(s, a, mask, rank, mu, base, dctr);
            read_counters(c);
            base = std::max<int64_t>(base, h[0]);
            k::fill_i64(s, dctr, 0, 1);
            k::count_unranked(s, a, rank, dctr);
            read_counters(c);
            if (h[0] == 0 || widen == kTauSteps) break;
            tau *= 10.0;
            k::opt_mask(s, a, I.d_wc, I.d_wp, xi, tau, mask, rank, mu, true);
        }
        st.rank_rounds += relax_sweeps;
        if (h[0] != 0)
            fail(MORAP_E_IMPROPER, std::to_string(h[0]) + " states cannot reach done through tau-optimal actions");

        // from the scalarised values the policies were chosen from (R15)
        if (o.eval_start && !team) k::eval_start(s, a, xi, I.d_wc, I.d_wp, d_iwarm, xe0);
        k::set_active(s, n, a, iact, ires, ipar, 2);
        int64_t tiled = 0;
        k::InstArgs ae = a;
        while (true) {
            for (int i = 0; i < chunk; ++i) {
                const bool even = (i & 1) == 0;
                if (c->has_blocks)
                    k::eval_block_sweep(s, ae, c->d_blk_rec.as<int32_t>(), c->d_blk64.as<double>(), mu, iact,
                                        even ? xe0 : xe1, even ? xe1 : xe0, ires, (int32_t)c->S, c->hm.blk_pattern);
                else
                    k::eval_sweep(s, ae, mu, iact, even ? xe0 : xe1, even ? xe1 : xe0, ires);
                k::inst_converge(s, 2 * n, ires, iact, ipar, even ? 1 : 0, o.eps_eval, dctr);
            }
            tiled += chunk;
            read_counters(c);
            if (h[0] == 0 || tiled >= o.max_sweeps) break;
            live_tiles(iact, 2, ae);
        }
        esweeps = std::max(esweeps, tiled);
        k::select_final(s, a, xe0, xe1, ipar, 2);
    }

    if (lds && beside) finish_lds();
    if (c->has_blocks) {
        st.polish_sweeps += vsweeps;
        st.variant_refine = -1;   // instance-major block iteration
    }

    // values at the initial states: of the policy values (an FP32 solve's
    // assignment is checked against them, for the weights of the column, which
    // the re-solve scaled to sum 1) and of both objectives
    double* ival = c->d_init_val.as<double>();
    const bool keep_c64 = c->has_blocks && c->prec == MORAP_F32 && !team;
    if (keep_c64) k::gather_values(s, n, I.d_init, xi, ival);
    k::gather_init(s, n, I.d_init, xe0, ival + n);
    c->h_c.ensure((size_t)3 * n * 8);
    MORAP_HIP(hipMemcpyAsync(c->h_c.p, ival, (size_t)3 * n * 8, hipMemcpyDeviceToHost, s));
    MORAP_HIP(hipEventRecord(wall.b, s));
    MORAP_HIP(hipEventSynchronize(wall.b));
    const float ms = wall.elapsed_ms();
    const double* vals = c->h_c.as<double>() + n;
    if (keep_c64) {
        c->last_c64.resize(n);
        for (int q = 0; q < n; ++q) c->last_c64[q] = iscale[q] > 0 ? c->h_c.as<double>()[q] / iscale[q] : 0.0;
        c->last_c64_valid = true;
    }
    if ((lds && I.running(h_sweeps + n, 2) > 0) || (general && h[0] != 0)) {
        // name the (column, task, objective) entries still running; the
        // policies stay readable through morap_get_policy
        std::vector<uint8_t> still((size_t)2 * n, 0);
        if (general) MORAP_HIP(hipMemcpy(still.data(), iact, still.size(), hipMemcpyDeviceToHost));
        for (int32_t q : I.order)
            for (int w = 0; w < 2; ++w) still[(size_t)2 * q + w] = h_sweeps[(size_t)n + 2 * (size_t)q + w] == 0;
        std::string who;
        int shown = 0;
        for (int q = 0; q < 2 * n && shown < 8; ++q)
            if (still[q]) {
                const int inst = q / 2;
                char buf[256];
                std::snprintf(buf, sizeof buf,
                              " (k=%d, j=%d, %s: model %d, weights %.17g, %.17g, value at the initial state "
                              "now %.6g / %.6g)",
                              inst / nJ, inst % nJ, q % 2 ? "probability" : "cost", c->inst_m[inst], iwc[inst],
                              iwp[inst], vals[2 * inst], vals[2 * inst + 1]);
                who += buf;
                ++shown;
            }
        c->eK = K;
        c->evaluated = true;
        fail(MORAP_E_NOT_CONVERGED,
             "policy evaluation did not converge after " + std::to_string(esweeps) + " sweeps:" + who);
    }
    st.eval_sweeps += esweeps;

    if (r_out) {
        std::fill(r_out, r_out + (size_t)K * d, 0.0);
        for (int kk = 0; kk < K; ++kk)
            for (int j = 0; j < nJ; ++j) {
                const int q = kk * nJ + j;
                if (team) {
                    r_out[(size_t)kk * d + 2 * j] = vals[2 * q];
                    if (2 * j + 1 < d) r_out[(size_t)kk * d + 2 * j + 1] = vals[2 * q + 1];
                    continue;
                }
                r_out[(size_t)kk * d + nI + j] = vals[2 * q + 1];
                r_out[(size_t)kk * d + assign[q]] += vals[2 * q];
            }
    }
    c->eK = K;
    c->evaluated = true;
    // keep the final values and the layout for a warm start of the next one
    std::swap(c->d_xe_prev.p, c->d_xe[0].p);
    std::swap(c->d_xe_prev.bytes, c->d_xe[0].bytes);
    std::swap(c->d_xe_prev.meter, c->d_xe[0].meter);
    c->prev_inst_base = c->inst_base;
    c->prev_inst_m = c->inst_m;
    c->prev_per_col = nJ;
    c->prev_eval_gen = c->load_gen;
    c->eval_prev_valid = true;
    st.ms_eval += ms;
    st.ms_total += std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
}

// ---------------------------------------------------------------------------
// the assignment check after an FP32 solve
// ---------------------------------------------------------------------------
// FP64 value iteration (to eps_vi, instance-major over the block form, from
// the FP32 values) of the (column k, model m) pairs listed; returns each
// pair's value at its model's initial state for the column's own weights.
// Uses buffers of its own: the last evaluation stays readable.
static std::vector<double> resolve_pairs(morap_ctx* c, const std::vector<int32_t>& pk,
                                         const std::vector<int32_t>& pm, const morap_vi_opts& o, Stats& st) {
    hipStream_t s = c->stream;
    Instances I;
    I.build(c, pk, pm, false, o);
    const int n = I.n;
    const int64_t NS = I.states();
    const bool general = I.n_general > 0, lds = !I.order.empty();
    c->d_cand_x0.ensure((size_t)NS * 8 + 8);
    c->d_cand_val.ensure((size_t)n * 8);
    c->d_cand_sweeps.ensure((size_t)n * 4 + 8);
    InstancePack pack;
    I.send(pack, c->d_cand_pack, c->h_cand_pack, s);
    const k::InstArgs a = I.args(c);
    double* x0 = c->d_cand_x0.as<double>();
    const int chunk = std::max(2, (o.check_every + 1) / 2 * 2);
    int64_t sweeps = 0;
    if (lds) {
        const int64_t limit = ((int64_t)o.max_sweeps + chunk - 1) / chunk * chunk;
        int32_t* ps = c->d_cand_sweeps.as<int32_t>();
        c->h_inst_out.ensure((size_t)n * 4 + 16);
        const int32_t* h_ps = c->h_inst_out.as<int32_t>();
        k::fill_i32(s, ps, 0, n);
        for (int64_t s0 = 0; s0 < limit; s0 += kResidentSweeps) {
            I.launch_vi(c, x0, ps, s0, std::min<int64_t>(limit, s0 + kResidentSweeps), nullptr);
            MORAP_HIP(hipMemcpyAsync(c->h_inst_out.p, ps, (size_t)n * 4, hipMemcpyDeviceToHost, s));
            MORAP_HIP(hipStreamSynchronize(s));
            if (I.running(h_ps, 1) == 0) break;
        }
        MORAP_CHECK(I.running(h_ps, 1) == 0, MORAP_E_NOT_CONVERGED,
                    "value iteration of the pairs of the assignment check did not converge");
        Stats ignored;   // (their bytes are not counted)
        sweeps = I.account(c, h_ps, chunk, ignored);
    }
    if (general) {
        c->d_cand_x1.ensure((size_t)NS * 8 + 8);
        c->d_cand_res.ensure((size_t)n * 8);
        c->d_cand_act.ensure((size_t)n);
        c->d_cand_par.ensure((size_t)n);
        double* x1 = c->d_cand_x1.as<double>();
        unsigned long long* res = c->d_cand_res.as<unsigned long long>();
        uint8_t* act = c->d_cand_act.as<uint8_t>();
        uint8_t* par = c->d_cand_par.as<uint8_t>();
        int64_t* dctr = c->d_counters.as<int64_t>();
        int64_t* h = c->h_counters.as<int64_t>();
        k::warm_start(s, a, c->vmain.x[0].p, c->vmain.x[1].p, c->vmain.final_par.as<uint8_t>(), c->vmain.Kp, I.d_scale,
                      I.d_wc, x0);
        k::fill_f64(s, x1, 0.0, NS);
        k::set_active(s, n, a, act, res, par, 1);
        int64_t tiled = 0;
        while (true) {
            for (int i = 0; i < chunk; ++i) {
                const bool even = (i & 1) == 0;
                k::inst_vi_sweep(s, a, c->d_blk_rec.as<int32_t>(), c->d_blk64.as<double>(), I.d_wc, I.d_wp, act,
                                 even ? x0 : x1, even ? x1 : x0, res, (int32_t)c->S, c->hm.blk_pattern);
                k::inst_converge(s, n, res, act, par, even ? 1 : 0, o.eps_vi, dctr);
            }
            tiled += chunk;
            read_counters(c);
            if (h[0] == 0) break;
            MORAP_CHECK(tiled < o.max_sweeps, MORAP_E_NOT_CONVERGED,
                        "value iteration of the pairs of the assignment check did not converge");
        }
        k::select_final(s, a, x0, x1, par, 1);
        sweeps = std::max(sweeps, tiled);
    }
    k::gather_values(s, n, I.d_init, x0, c->d_cand_val.as<double>());
    std::vector<double> out(n);
    MORAP_HIP(hipMemcpyAsync(out.data(), c->d_cand_val.p, (size_t)n * 8, hipMemcpyDeviceToHost, s));
    MORAP_HIP(hipStreamSynchronize(s));
    for (int q = 0; q < n; ++q) out[q] = I.scale[q] > 0 ? out[q] / I.scale[q] : 0.0;
    st.polish_sweeps += sweeps;
    return out;
}

// The assignment of each column was taken on FP32 values c.  Their error on
// the column's assigned pairs, e_k, is known from the FP64 re-solve; every
// unassigned pair whose slack (the value an assignment using it gives up,
// from the optimal duals) is at most 2 e_k could enter a better assignment
// once corrected by that much, so it is re-solved in FP64 too.  The column
// is then assigned again on c with the FP64 values of all these pairs; it
// takes the new assignment when that raises its value by more than 1e-9 of
// it.
// Returns the number of columns that changed (their assignments in out).
static int refine_assignment(morap_ctx* c, const int32_t* assign, int K, const morap_vi_opts& o, Stats& st,
                             int32_t* out) {
    const int nI = c->hm.nI, nJ = c->hm.nJ, M = c->hm.M;
    const auto t0 = std::chrono::steady_clock::now();
    std::vector<double> C((size_t)K * M);
    MORAP_HIP(hipMemcpy(C.data(), c->vmain.c.p, C.size() * 8, hipMemcpyDeviceToHost));   // [K][M]
    // the pairs to re-solve, per column (columns on host threads)
    std::vector<std::vector<int32_t>> cand(K);
    std::atomic<int> next{0};
    auto worker = [&] {
        std::vector<double> slack((size_t)M);
        for (int k; (k = next++) < K;) {
            const double* ck = C.data() + (size_t)k * M;
            double e = 0, cmax = 0;
            for (int j = 0; j < nJ; ++j) {
                const int m = assign[(size_t)k * nJ + j] * nJ + j;
                e = std::max(e, std::fabs(ck[m] - c->last_c64[(size_t)k * nJ + j]));
            }
            for (int m = 0; m < M; ++m) cmax = std::max(cmax, std::fabs(ck[m]));
            const double theta = 2.0 * e + 1e-12 * std::max(1.0, cmax);
            assignment_slack(nI, nJ, ck, slack.data());
            // pairs whose two weights are 0 have the value 0 in any precision
            const double* w = c->W.data() + (size_t)k * (nI + nJ);
            for (int i = 0; i < nI; ++i)
                for (int j = 0; j < nJ; ++j)
                    if (assign[(size_t)k * nJ + j] != i && slack[(size_t)i * nJ + j] <= theta &&
                        w[i] + w[nI + j] > 0)
                        cand[k].push_back(i * nJ + j);
        }
    };
    c->pool.run(host_threads(K), worker);
    std::vector<int32_t> pk, pm;
    for (int k = 0; k < K; ++k)
        for (int32_t m : cand[k]) {
            pk.push_back(k);
            pm.push_back(m);
        }
    st.refine_pairs += (int64_t)pk.size();
    const auto t1 = std::chrono::steady_clock::now();
    if (pk.empty()) return 0;
    const std::vector<double> v = resolve_pairs(c, pk, pm, o, st);
    if (std::getenv("MORAP_PROGRESS"))
        std::fprintf(stderr, "[morap] assignment check: %zu pairs re-solved; slacks %.1f ms, re-solve %.1f ms\n",
                     pk.size(), std::chrono::duration<double, std::milli>(t1 - t0).count(),
                     std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t1).count());
    // c with the FP64 values of the assigned and the re-solved pairs
    for (int k = 0; k < K; ++k)
        for (int j = 0; j < nJ; ++j)
            C[(size_t)k * M + assign[(size_t)k * nJ + j] * nJ + j] = c->last_c64[(size_t)k * nJ + j];
    for (size_t q = 0; q < pk.size(); ++q) C[(size_t)pk[q] * M + pm[q]] = v[q];
    std::vector<int32_t> A((size_t)K * nJ);
    assign_columns(nI, nJ, C.data(), K, A.data(), &c->pool);
    int changed = 0;
    for (int k = 0; k < K; ++k) {
        const double* ck = C.data() + (size_t)k * M;
        double v_old = 0, v_new = 0;
        for (int j = 0; j < nJ; ++j) {
            v_old += ck[assign[(size_t)k * nJ + j] * nJ + j];
            v_new += ck[A[(size_t)k * nJ + j] * nJ + j];
        }
        // gains below 1e-9 of the column's value are under the accuracy of
        // the FP64 values themselves (each stops at eps_vi)
        if (v_new > v_old + 1e-9 * std::max(1.0, std::fabs(v_old))) {
            std::copy(A.begin() + (size_t)k * nJ, A.begin() + (size_t)(k + 1) * nJ, out + (size_t)k * nJ);
            ++changed;
        }
    }
    st.refine_columns += changed;
    return changed;
}

// ---------------------------------------------------------------------------
// stage retirement inside the iteration (the staged form of Alg. 3)
// ---------------------------------------------------------------------------
template <class T>
static void upload_vec(DevBuf& d, const std::vector<T>& h, hipStream_t s) {
    d.ensure(h.size() * sizeof(T) + 16);
    if (!h.empty()) MORAP_HIP(hipMemcpyAsync(d.p, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice, s));
}

// Stage of every state of model m: the location graph has an edge q -> q'
// for every live transition from a state at q to one at q'; its strongly
// connected groups form a DAG, and a group's stage is its height there (0
// for a group with no other group below it).  Every transition therefore
// leads to the same or a lower stage.
static int model_stages(const HostModels& hm, int m, std::vector<int32_t>& stage) {
    const int32_t s0 = hm.state_base[m], s1 = hm.state_base[m + 1];
    std::vector<int32_t> locs;
    for (int32_t g = s0; g < s1; ++g) locs.push_back(hm.states_sq[(size_t)2 * g + 1]);
    std::sort(locs.begin(), locs.end());
    locs.erase(std::unique(locs.begin(), locs.end()), locs.end());
    const int L = (int)locs.size();
    if (L == 0) return 0;
    auto idx = [&](int32_t g) {
        return (int)(std::lower_bound(locs.begin(), locs.end(), hm.states_sq[(size_t)2 * g + 1]) - locs.begin());
    };
    // reachability between locations (a handful per product)
    std::vector<uint8_t> reach((size_t)L * L, 0);
    for (int a = 0; a < L; ++a) reach[(size_t)a * L + a] = 1;
    for (int32_t g = s0; g < s1; ++g) {
        const int a = idx(g);
        for (int32_t r = hm.state_row[g]; r < hm.state_row[g + 1]; ++r)
            for (int32_t e = hm.row_ptr[r]; e < hm.row_ptr[r + 1]; ++e) {
                const int32_t h = hm.col[e];
                MORAP_CHECK(h >= s0 && h < s1, MORAP_E_STATE, "a transition leaves its model");
                reach[(size_t)a * L + idx(h)] = 1;
            }
    }
    for (int q = 0; q < L; ++q)
        for (int a = 0; a < L; ++a)
            if (reach[(size_t)a * L + q])
                for (int b = 0; b < L; ++b)
                    if (reach[(size_t)q * L + b]) reach[(size_t)a * L + b] = 1;
    // heights: a location reaches strictly more locations than every
    // location strictly below it, so count order is a topological order
    std::vector<int> n_reach(L, 0), order(L), height(L, 0);
    for (int a = 0; a < L; ++a)
        for (int b = 0; b < L; ++b) n_reach[a] += reach[(size_t)a * L + b];
    for (int a = 0; a < L; ++a) order[a] = a;
    std::sort(order.begin(), order.end(), [&](int x, int y) { return n_reach[x] < n_reach[y]; });
    int top = 0;
    for (int a : order) {
        for (int b = 0; b < L; ++b)
            if (reach[(size_t)a * L + b] && !reach[(size_t)b * L + a]) height[a] = std::max(height[a], height[b] + 1);
        top = std::max(top, height[a]);
    }
    for (int32_t g = s0; g < s1; ++g) stage[g] = height[idx(g)];
    return top + 1;
}

// The units of every model, and the states of products that fit LDS sorted
// for the kernel that keeps their values there.
static void build_stages(morap_ctx* c) {
    StagedLayout& L = c->staged;
    if (L.gen == c->load_gen) return;
    const HostModels& hm = c->hm;
    const int M = hm.M;
    const int64_t S = hm.S();
    MORAP_CHECK(c->has_blocks, MORAP_E_UNSUPPORTED,
                "stage retirement runs on the neighbourhood-block form (products built by morap_build_products)");
    MORAP_CHECK((int64_t)hm.states_sq.size() == 2 * S, MORAP_E_UNSUPPORTED,
                "stage retirement needs the DFA location of every state");
    L.stage.assign((size_t)S, 0);
    L.unit_base.assign(M + 1, 0);
    L.h_init_unit.assign(M, -1);
    for (int m = 0; m < M; ++m) {
        L.unit_base[m + 1] = L.unit_base[m] + model_stages(hm, m, L.stage);
        if (hm.init[m] >= 0) L.h_init_unit[m] = L.unit_base[m] + L.stage[hm.init[m]];
    }
    const int U = L.unit_base[M];
    L.h_rows.assign(U, 0);
    L.h_states.assign(U, 0);
    L.h_csr.assign(U, 0);
    for (int m = 0; m < M; ++m)
        for (int32_t g = hm.state_base[m]; g < hm.state_base[m + 1]; ++g) {
            const int u = L.unit_base[m] + L.stage[g];
            const int32_t nr = hm.state_row[g + 1] - hm.state_row[g];
            const int64_t nnz = hm.row_ptr[hm.state_row[g + 1]] - hm.row_ptr[hm.state_row[g]];
            L.h_rows[u] += nr;
            L.h_states[u] += 1;
            // state_row + row_ptr + col (int32) + prob and two rewards (FP64)
            L.h_csr[u] += 4 + 4 * (int64_t)nr + 12 * nnz + 16 * (int64_t)nr;
        }
    hipStream_t s = c->stream;
    upload_vec(L.unit_base_d, L.unit_base, s);
    upload_vec(L.init_unit, L.h_init_unit, s);
    L.lds_order.clear();
    L.lds_positions.assign(M, 0);
    std::vector<int32_t> base((size_t)M + 1, 0), block, init((size_t)M, 0);
    std::vector<uint32_t> rec;
    bool fit = k::has_grid_pattern(hm.blk_pattern) && hm.blk_agent.size() / 32 < (1u << 20);
    for (int m = 0; m < M && fit; ++m) {
        if (hm.init[m] < 0) continue;
        fit = hm.blk_plain[(size_t)m] != 0 && L.unit_base[m + 1] - L.unit_base[m] <= 64 &&
              hm.state_base[m + 1] - hm.state_base[m] <= k::resident_most_positions();
        L.lds_order.push_back(m);
    }
    if (fit) {
        const std::vector<SortedStates> sorted = sort_models(hm, L.lds_order, L.stage.data());
        for (int m = 0; m < M; ++m) {
            const SortedStates& x = sorted[(size_t)m];
            block.insert(block.end(), x.block.begin(), x.block.end());
            rec.insert(rec.end(), x.rec.begin(), x.rec.end());
            init[(size_t)m] = x.init;
            L.lds_positions[m] = 64 * (int32_t)x.block.size();
            base[(size_t)m + 1] = base[(size_t)m] + L.lds_positions[m];
        }
        for (int32_t m : L.lds_order) fit = fit && L.lds_positions[m] > 0;
        std::stable_sort(L.lds_order.begin(), L.lds_order.end(),
                         [&](int32_t x, int32_t y) { return L.lds_positions[x] > L.lds_positions[y]; });
    }
    if (!fit) L.lds_order.clear();
    try {
        upload_vec(L.order, L.lds_order, s);
        upload_vec(L.lds_base, base, s);
        upload_vec(L.lds_block, block, s);
        upload_vec(L.lds_rec, rec, s);
        upload_vec(L.lds_init, init, s);
    } catch (const MorapError& e) {
        if (e.code != MORAP_E_OOM) throw;
        // no memory for this layout: the batched sweeps need none of it
        MORAP_HIP(hipStreamSynchronize(s));
        L.drop_lds();
    }
    MORAP_HIP(hipStreamSynchronize(s));
    L.U = U;
    L.gen = c->load_gen;
}

// The records regrouped by unit and the units' tiles (batched sweeps).
static void build_unit_tiles(morap_ctx* c) {
    StagedLayout& L = c->staged;
    if (L.tiles_gen == c->load_gen) return;
    const HostModels& hm = c->hm;
    const int M = hm.M, U = L.U;
    const std::vector<int32_t>& stage = L.stage;
    std::vector<int32_t> live(U, -1);
    for (int m = 0; m < M; ++m)
        for (int u = L.unit_base[m]; u < L.unit_base[m + 1]; ++u) live[u] = hm.init[m] >= 0 ? 0 : -1;
    // records regrouped by unit inside every tile (stable), and the unit
    // tiles, consecutive per unit
    std::vector<int32_t> rec(hm.blk_rec.size());
    std::vector<std::vector<Tile>> per_unit(U);
    for (int m = 0; m < M; ++m) {
        const int nst = L.unit_base[m + 1] - L.unit_base[m];
        std::vector<int> cnt(nst + 1);
        for (int t = c->tile_base[m]; t < c->tile_base[m + 1]; ++t) {
            const Tile& tl = c->tiles[t];
            std::fill(cnt.begin(), cnt.end(), 0);
            for (int p = tl.s_begin; p < tl.s_end; ++p) ++cnt[stage[hm.blk_rec[(size_t)p * 8 + 7]] + 1];
            for (int q = 0; q < nst; ++q) cnt[q + 1] += cnt[q];
            for (int q = 0; q < nst; ++q)
                if (cnt[q + 1] > cnt[q])
                    per_unit[L.unit_base[m] + q].push_back(
                        Tile{L.unit_base[m] + q, tl.s_begin + cnt[q], tl.s_begin + cnt[q + 1], 0});
            for (int p = tl.s_begin; p < tl.s_end; ++p) {
                const int q = stage[hm.blk_rec[(size_t)p * 8 + 7]];
                std::copy(&hm.blk_rec[(size_t)p * 8], &hm.blk_rec[(size_t)p * 8 + 8],
                          &rec[(size_t)(tl.s_begin + cnt[q]++) * 8]);
            }
        }
    }
    std::vector<Tile> tiles;
    std::vector<int32_t> tile_base(U + 1, 0);
    for (int u = 0; u < U; ++u) {
        tile_base[u] = (int32_t)tiles.size();
        tiles.insert(tiles.end(), per_unit[u].begin(), per_unit[u].end());
    }
    tile_base[U] = (int32_t)tiles.size();
    hipStream_t s = c->stream;
    upload_vec(L.tiles, tiles, s);
    upload_vec(L.tile_base, tile_base, s);
    upload_vec(L.rec, rec, s);
    upload_vec(L.rows, L.h_rows, s);
    upload_vec(L.states, L.h_states, s);
    upload_vec(L.csr, L.h_csr, s);
    upload_vec(L.live, live, s);
    MORAP_HIP(hipStreamSynchronize(s));
    L.n_tiles = (int64_t)tiles.size();
    L.tiles_gen = c->load_gen;
}

// What a workgroup takes of model m: columns, and the class of its launch.
struct StagedClass {
    int columns, threads, size;
    bool operator==(const StagedClass& o) const {
        return columns == o.columns && threads == o.threads && size == o.size;
    }
};
static StagedClass staged_class(const StagedLayout& L, int m, int prec, bool wide) {
    const int pos = L.lds_positions[m];
    int columns = k::staged_columns(prec, pos, L.unit_base[m + 1] - L.unit_base[m]);
    if (!wide) columns = std::min(columns, 1);
    StagedClass r{columns, columns ? k::staged_threads(prec, columns, pos) : 0, 0};
    // (a launch's LDS is its largest product's: at most twice the smallest's)
    while (pos >> r.size > 512) ++r.size;
    return r;
}

// Stage retirement with every product's values in LDS, one launch per class of
// products; statistics as the batched sweeps count them.
static void run_staged_lds(morap_ctx* c, ValueSet& vs, const morap_vi_opts& o, bool wide, Stats& st) {
    StagedLayout& L = c->staged;
    const HostModels& hm = c->hm;
    const int M = hm.M, K = vs.K, Kp = vs.Kp, U = L.U;
    hipStream_t s = c->stream;
    const size_t pairs = (size_t)U * Kp;
    L.pair_sweeps.ensure(pairs * 4);
    L.best_res.ensure(pairs * 8);
    L.stall.ensure(pairs * 4);
    L.h_unit_sweeps.ensure(pairs * 4);
    const k::ConvergeArgs ca = converge_args(c, vs, nullptr, o.eps_vi, 0, false);
    EventPair wall;
    MORAP_HIP(hipEventRecord(wall.a, s));
    k::init_pairs(s, ca);
    k::fill_i32(s, L.pair_sweeps.as<int32_t>(), 0, (int64_t)pairs);
    k::StagedLdsArgs a{};
    static_cast<k::ResidentArgs&>(a) = resident_args(c, vs, ca);
    a.big_base = L.lds_base.as<int32_t>();
    a.big_block = L.lds_block.as<int32_t>();
    a.big_rec = L.lds_rec.as<uint4>();
    a.big_init = L.lds_init.as<int32_t>();
    a.best_res = L.best_res.as<double>();
    a.stall = L.stall.as<int32_t>();
    a.unit_base = L.unit_base_d.as<int32_t>();
    a.init_unit = L.init_unit.as<int32_t>();
    a.unit_sweeps = L.pair_sweeps.as<int32_t>();
    struct Launch {
        StagedClass c;
        int begin, n;
    };
    std::vector<Launch> launches;
    for (int b = 0; b < (int)L.lds_order.size(); ++b) {
        const StagedClass q = staged_class(L, L.lds_order[b], vs.prec, wide);
        if (launches.empty() || !(launches.back().c == q)) launches.push_back({q, b, 0});
        ++launches.back().n;
    }
    const int32_t* us = L.h_unit_sweeps.as<int32_t>();
    PooledEvents held(c);
    int64_t done = 0, running = 0;
    for (int64_t s0 = 0; s0 < o.max_sweeps; s0 = done) {
        done = std::min<int64_t>(o.max_sweeps, s0 + kResidentSweeps);
        a.sweep0 = (int)s0;
        a.sweep1 = (int)done;
        Fork fork(c, o.time_kernels ? 1 : (int)launches.size());
        for (size_t q = 0; q < launches.size(); ++q) {
            const Launch& l = launches[q];
            a.order = L.order.as<int32_t>() + l.begin;
            a.n_models = l.n;
            if (o.time_kernels) {
                held.v.emplace_back(take_event(c), nullptr);
                held.v.back().second = take_event(c);
                MORAP_HIP(hipEventRecord(held.v.back().first, s));
            }
            const int positions = L.lds_positions[L.lds_order[l.begin]];   // (the largest product's)
            k::staged_lds(fork.least((double)l.n * positions), vs.prec, l.c.columns, l.c.threads, positions, a);
            if (o.time_kernels) MORAP_HIP(hipEventRecord(held.v.back().second, s));
        }
        fork.join();
        MORAP_HIP(hipMemcpyAsync(L.h_unit_sweeps.p, L.pair_sweeps.p, pairs * 4, hipMemcpyDeviceToHost, s));
        read_results(c, vs);
        running = 0;
        for (int32_t m : L.lds_order)
            for (int u = L.unit_base[m]; u < L.unit_base[m + 1]; ++u)
                for (int k = 0; k < K; ++k) running += us[(size_t)u * Kp + k] == 0;
        if (running == 0) break;
    }
    if (running > 0)
        fail(MORAP_E_NOT_CONVERGED, "value iteration with stage retirement: " + std::to_string(running) +
                                        " (unit, column) pairs still active after " + std::to_string(o.max_sweeps) +
                                        " sweeps");
    MORAP_HIP(hipEventRecord(wall.b, s));
    MORAP_HIP(hipEventSynchronize(wall.b));
    const double el = vs.prec == MORAP_F32 ? 4 : 8;
    int64_t longest = 0;
    for (int32_t m : L.lds_order)
        for (int u = L.unit_base[m]; u < L.unit_base[m + 1]; ++u) {
            int64_t sum = 0, top = 0;
            for (int k = 0; k < K; ++k) {
                const int64_t n = us[(size_t)u * Kp + k];
                sum += n;
                top = std::max(top, n);
            }
            st.backups += L.h_rows[u] * sum;
            st.bytes += (double)L.h_csr[u] * (double)top + 2.0 * el * (double)L.h_states[u] * (double)sum;
            longest = std::max(longest, top);
        }
    // (counted as the batched sweeps are: to the next look at the counters)
    const int64_t check = std::max(2, o.check_every);
    const int64_t looked = std::max<int64_t>((longest + check - 1) / check * check, check);
    st.sweeps += std::min<int64_t>(o.max_sweeps, looked);
    const int32_t* ps = c->h_pair_sweeps.as<int32_t>();
    st.max_pair_sweeps = std::max<int64_t>(st.max_pair_sweeps, *std::max_element(ps, ps + (size_t)M * Kp));
    st.floor_stops += c->h_counters.as<int64_t>()[8];
    st.resident_models = (int)L.lds_order.size();
    st.ms_vi += wall.elapsed_ms();
    for (auto& e : held.v) {
        float t = 0;
        MORAP_HIP(hipEventElapsedTime(&t, e.first, e.second));
        st.ms_sweep_kernel += t;
        st.sweep_launches += 1;
    }
}

// Alg. 3 for K columns with stage retirement: each sweep backs up the
// units still active, then per (model, column) the units are taken lowest
// first and a unit retires when all lower ones have and its own change is
// <= eps_vi; its values are copied into the other buffer.  A pair's value at
// the initial state is final when the initial state's unit retires.
static void solve_staged_impl(morap_ctx* c, const double* W, int K, const morap_vi_opts& o, double* c_out,
                              Stats& st) {
    MORAP_CHECK(c->loaded, MORAP_E_STATE, "no models loaded");
    MORAP_CHECK(!c->team, MORAP_E_UNSUPPORTED, "stage retirement runs on the decentralised products");
    MORAP_CHECK(o.precision == MORAP_F32 || o.precision == MORAP_F64, MORAP_E_INVALID, "bad precision");
    MORAP_CHECK(W && K >= 1 && K <= 4096, MORAP_E_INVALID, "need 1 <= K <= 4096 weight vectors");
    MORAP_CHECK(o.eps_vi > 0 && std::isfinite(o.eps_vi), MORAP_E_INVALID, "eps_vi must be > 0");
    MORAP_CHECK(o.max_sweeps >= 1, MORAP_E_INVALID, "max_sweeps must be >= 1");
    const int nI = c->hm.nI, nJ = c->hm.nJ, M = c->hm.M, d = nI + nJ;
    check_weight_rows(W, K, d);
    const auto t0 = std::chrono::steady_clock::now();
    build_stages(c);
    StagedLayout& L = c->staged;
    const int U = L.U, Kp = padded_k(K), prec = o.precision;
    const size_t el = prec == MORAP_F32 ? 4 : 8;
    // a neighbourhood-block sweep: the one the autotuner chose for plain FP64
    // solves of this width if it is one, else the first with k-tiles of
    // min(Kp, 64) columns (the wave-per-state one where it fits)
    const Variant* v = nullptr;
    if (o.schedule > 0) {
        MORAP_CHECK(o.schedule <= (int)variants().size(), MORAP_E_INVALID, "unknown sweep variant");
        v = &variants()[o.schedule - 1];
        MORAP_CHECK(v->kind == SWEEP_BLOCK && Kp % kt_of(*v) == 0, MORAP_E_UNSUPPORTED,
                    "stage retirement runs a neighbourhood-block sweep whose k-tile divides the padded width");
    } else {
        // (also where some products' plain solves stay in LDS)
        for (int64_t rest : {0, 2})
            for (auto& t : c->tuned)
                if (!v && t.first == (((int64_t)prec << 40) | (rest << 32) | Kp) &&
                    variant_by_id(t.second).kind == SWEEP_BLOCK)
                    v = &variant_by_id(t.second);
        if (!v)
            for (const auto& x : variants())
                if (x.kind == SWEEP_BLOCK && kt_of(x) == std::min(Kp, 64) &&
                    (!v || (x.cpl == 1 && x.lps == 64 && x.unroll == 2)))
                    v = &x;
    }
    MORAP_CHECK(v, MORAP_E_UNSUPPORTED, "no neighbourhood-block sweep for this width");
    hipStream_t s = c->stream;
    c->solved = false;
    c->evaluated = false;
    ensure_scratch(c, Kp);
    c->K = K;
    c->Kp = Kp;
    c->prec = prec;
    c->W.assign(W, W + (size_t)K * d);
    ValueSet& vs = c->vmain;
    ensure_values(c, vs, K, Kp, prec);

    // every live product in LDS, unless the caller fixed the sweep kernel;
    // several columns per workgroup unless all pairs run at once anyway
    const bool wide = (int64_t)L.lds_order.size() * K > 2 * (int64_t)c->prop.multiProcessorCount;
    bool lds = o.schedule == 0 && !L.lds_order.empty() && c->hm.largest_reward <= k::largest_reward(prec);
    for (int32_t m : L.lds_order) lds = lds && staged_class(L, m, prec, wide).columns > 0;
    if (lds) {
        c->d_weights.ensure((size_t)K * d * 8);
        MORAP_HIP(hipMemcpyAsync(c->d_weights.p, W, (size_t)K * d * 8, hipMemcpyHostToDevice, s));
        if (prec == MORAP_F32) k::fill_f32(s, vs.x[0].as<float>(), 0.f, (c->S + 1) * Kp);
        else k::fill_f64(s, vs.x[0].as<double>(), 0.0, (c->S + 1) * Kp);
        run_staged_lds(c, vs, o, wide, st);
        st.variant = v->id;
        if (c_out) std::memcpy(c_out, c->h_c.p, (size_t)K * M * 8);
        st.ms_total += std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
        vs.valid = true;
        c->solved = true;
        return;
    }
    build_unit_tiles(c);
    const size_t pairs = (size_t)U * Kp;
    L.active.ensure(pairs);
    L.res.ensure(pairs * 8);
    L.ymax.ensure(pairs * 8);
    L.wc.ensure(pairs * el);
    L.wp.ensure(pairs * el);
    L.final_par.ensure(pairs);
    L.pair_sweeps.ensure(pairs * 4);
    L.best_res.ensure(pairs * 8);
    L.stall.ensure(pairs * 4);
    L.c_units.ensure((size_t)K * U * 8);
    L.model_active.ensure(U);
    L.act_models.ensure((size_t)U * 4 + 4);
    L.act_prefix.ensure((size_t)(U + 1) * 4 + 4);
    L.act_tiles.ensure((size_t)L.n_tiles * 4 + 4);
    L.retired.ensure(pairs * 8);
    L.counters.ensure(11 * 8);
    {
        std::vector<double> wc(pairs, 0.0), wp(pairs, 0.0);
        for (int m = 0; m < M; ++m) {
            const int i = m / nJ, j = m % nJ;
            for (int u = L.unit_base[m]; u < L.unit_base[m + 1]; ++u)
                for (int k = 0; k < K; ++k) {
                    wc[(size_t)u * Kp + k] = W[(size_t)k * d + i];
                    wp[(size_t)u * Kp + k] = W[(size_t)k * d + nI + j];
                }
        }
        std::vector<float> wc32, wp32;
        if (prec == MORAP_F32) {
            wc32.assign(wc.begin(), wc.end());
            wp32.assign(wp.begin(), wp.end());
        }
        MORAP_HIP(hipMemcpyAsync(L.wc.p, prec == MORAP_F32 ? (const void*)wc32.data() : (const void*)wc.data(),
                                 pairs * el, hipMemcpyHostToDevice, s));
        MORAP_HIP(hipMemcpyAsync(L.wp.p, prec == MORAP_F32 ? (const void*)wp32.data() : (const void*)wp.data(),
                                 pairs * el, hipMemcpyHostToDevice, s));
        MORAP_HIP(hipStreamSynchronize(s));
    }
    const int64_t nx = (c->S + 1) * Kp;
    if (prec == MORAP_F32) {
        k::fill_f32(s, vs.x[0].as<float>(), 0.f, nx);
        k::fill_f32(s, vs.x[1].as<float>(), 0.f, nx);
    } else {
        k::fill_f64(s, vs.x[0].as<double>(), 0.0, nx);
        k::fill_f64(s, vs.x[1].as<double>(), 0.0, nx);
    }
    k::fill_f64(s, vs.c.as<double>(), 0.0, (int64_t)K * M);
    k::fill_u8(s, vs.final_par.as<uint8_t>(), 0, (int64_t)M * Kp);
    k::fill_i32(s, c->d_pair_sweeps.as<int32_t>(), 0, (int64_t)M * Kp);
    k::fill_i64(s, L.counters.as<int64_t>(), 0, 11);

    // the units as models of the active-set machinery
    k::ConvergeArgs ca{};
    ca.res = L.res.as<unsigned long long>();
    ca.ymax = L.ymax.as<unsigned long long>();
    ca.active = L.active.as<uint8_t>();
    ca.final_par = L.final_par.as<uint8_t>();
    ca.pair_sweeps = L.pair_sweeps.as<int32_t>();
    ca.model_active = L.model_active.as<uint8_t>();
    ca.c = L.c_units.as<double>();
    ca.init = L.live.as<int32_t>();
    ca.x_out = vs.x[1].p;
    ca.counters = L.counters.as<int64_t>();
    ca.M = U;
    ca.K = K;
    ca.Kp = Kp;
    ca.prec = prec;
    ca.out_par = 1;
    ca.eps = o.eps_vi;
    // the stop rule of the plain solve (FP32: a few units in the last place,
    // and the rounding floor, R12)
    ca.unit = prec == MORAP_F32 ? 8.0 * std::ldexp(1.0, -24) : 8.0 * std::ldexp(1.0, -53);
    ca.best_res = L.best_res.as<double>();
    ca.stall = L.stall.as<int32_t>();
    ca.tile_base = L.tile_base.as<int32_t>();
    ca.act_models = L.act_models.as<int32_t>();
    ca.act_prefix = L.act_prefix.as<int32_t>();
    ca.rows_per_model = L.rows.as<int32_t>();
    ca.states_per_model = L.states.as<int32_t>();
    ca.csr_bytes = L.csr.as<int64_t>();
    ca.act_tiles = L.act_tiles.as<int32_t>();
    k::init_solve(s, ca);

    k::StageArgs sa{};
    sa.unit_base = L.unit_base_d.as<int32_t>();
    sa.init_unit = L.init_unit.as<int32_t>();
    sa.init = c->d_init.as<int32_t>();
    sa.rows = L.rows.as<int32_t>();
    sa.states = L.states.as<int32_t>();
    sa.active = ca.active;
    sa.res = ca.res;
    sa.ymax = ca.ymax;
    sa.model_active = ca.model_active;
    sa.c = vs.c.as<double>();
    sa.final_par = vs.final_par.as<uint8_t>();
    sa.pair_sweeps = c->d_pair_sweeps.as<int32_t>();
    sa.retired = L.retired.as<int64_t>();
    sa.counters = ca.counters;
    sa.tiles = L.tiles.as<Tile>();
    sa.tile_base = ca.tile_base;
    sa.rec = L.rec.as<int32_t>();
    sa.M = M;
    sa.K = K;
    sa.Kp = Kp;
    sa.eps = o.eps_vi;
    sa.unit = ca.unit;
    sa.prec = prec;
    sa.best_res = ca.best_res;
    sa.stall = ca.stall;
    sa.stall_sweeps = prec == MORAP_F32 ? 64 : 0;
    sa.floor = 256.0 * std::ldexp(1.0, -24);

    k::SweepArgs a = sweep_args(c, vs, 0);
    a.tiles = L.tiles.as<Tile>();
    a.tile_base = ca.tile_base;
    a.act_models = ca.act_models;
    a.act_prefix = ca.act_prefix;
    a.counters = ca.counters;
    a.wc = L.wc.p;
    a.wp = L.wp.p;
    a.active = ca.active;
    a.res = ca.res;
    a.ymax = ca.ymax;
    a.rec = sa.rec;
    a.act_tiles = ca.act_tiles;
    const int grid = persistent_grid(c, prec, *v);
    const int ktiles = Kp / kt_of(*v);
    const int check = std::max(2, o.check_every);
    int64_t h[11] = {0};
    EventPair wall;
    MORAP_HIP(hipEventRecord(wall.a, s));
    for (int n = 0;; ++n) {
        const int in_par = n & 1;
        a.x_in = vs.x[in_par].p;
        a.x_out = vs.x[1 - in_par].p;
        EventPair* ev = nullptr;
        std::unique_ptr<EventPair> timed;
        if (o.time_kernels) {
            timed.reset(new EventPair());
            ev = timed.get();
            MORAP_HIP(hipEventRecord(ev->a, s));
        }
        k::sweep_block(s, prec, *v, grid, ktiles, a);
        if (ev) MORAP_HIP(hipEventRecord(ev->b, s));
        sa.x_in = vs.x[in_par].p;
        sa.x_out = vs.x[1 - in_par].p;
        sa.out_par = 1 - in_par;
        sa.slot = 9 + (n & 1);
        k::stage_converge(s, sa);
        k::stage_copy(s, sa);
        k::compact(s, ca);
        if (ev) {
            MORAP_HIP(hipEventSynchronize(ev->b));
            st.ms_sweep_kernel += ev->elapsed_ms();
            st.sweep_launches += 1;
        }
        if ((n + 1) % check == 0 || n + 1 >= o.max_sweeps) {
            MORAP_HIP(hipMemcpyAsync(h, L.counters.p, sizeof(h), hipMemcpyDeviceToHost, s));
            MORAP_HIP(hipStreamSynchronize(s));
            if (h[3] == 0) break;
            if (n + 1 >= o.max_sweeps)
                fail(MORAP_E_NOT_CONVERGED, "value iteration with stage retirement: " + std::to_string(h[3]) +
                                                " (unit, column) pairs still active after " +
                                                std::to_string(n + 1) + " sweeps");
        }
    }
    MORAP_HIP(hipEventRecord(wall.b, s));
    MORAP_HIP(hipEventSynchronize(wall.b));
    std::vector<int32_t> ps((size_t)M * Kp);
    MORAP_HIP(hipMemcpy(ps.data(), c->d_pair_sweeps.p, ps.size() * 4, hipMemcpyDeviceToHost));
    st.backups += h[4];
    st.sweeps += h[5];
    st.bytes += (double)h[6] + 2.0 * (double)el * (double)h[7];
    st.floor_stops += h[8];
    st.max_pair_sweeps = std::max<int64_t>(st.max_pair_sweeps, *std::max_element(ps.begin(), ps.end()));
    st.ms_vi += wall.elapsed_ms();
    st.variant = v->id;
    if (c_out) MORAP_HIP(hipMemcpy(c_out, vs.c.p, (size_t)K * M * 8, hipMemcpyDeviceToHost));
    st.ms_total += std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    vs.valid = true;
    c->solved = true;
}

void solve_staged(morap_ctx* c, const double* W, int K, const morap_vi_opts& o, double* c_out, Stats& st) {
    Stats local;
    with_layouts(c, [&](bool) {
        local = Stats();
        solve_staged_impl(c, W, K, o, c_out, local);
    });
    add_stats(st, local);
    add_stats(c->cum, local);
}

}  // namespace morap
