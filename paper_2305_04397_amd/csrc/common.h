// Internal declarations of libmorap: context, device arena, error handling,
// kernel launch wrappers.  Not part of the ABI (include/morap.h is).
#pragma once

#include <condition_variable>
#include <exception>
#include <functional>
#include <mutex>
#include <system_error>
#include <thread>
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <memory>
#include <stdexcept>
#include <string>
#include <vector>

#include "../../include/morap.h"

namespace morap {

// ---------------------------------------------------------------------------
// errors: internal code throws MorapError; the ABI layer turns it into a
// return code and keeps the message on the context.
// ---------------------------------------------------------------------------
struct MorapError : std::runtime_error {
    int code;
    MorapError(int c, const std::string& m) : std::runtime_error(m), code(c) {}
};

[[noreturn]] inline void fail(int code, const std::string& msg) { throw MorapError(code, msg); }

#define MORAP_HIP(call)                                                                 \
    do {                                                                                \
        hipError_t e_ = (call);                                                         \
        if (e_ != hipSuccess)                                                           \
            ::morap::fail(MORAP_E_HIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

#define MORAP_CHECK(cond, code, msg) \
    do {                             \
        if (!(cond)) ::morap::fail(code, msg); \
    } while (0)

// ---------------------------------------------------------------------------
// device buffers
// ---------------------------------------------------------------------------
// Device bytes held by a context and its optional budget (0 = none).  The
// context's meter is current on the thread during every call on it, and each
// buffer remembers the meter that paid for it.  Where memory or the budget runs
// out, `reclaim` is asked once to free what the context can do without (true:
// something was freed).
struct AllocMeter {
    int64_t budget = 0, used = 0;
    bool (*reclaim)(void* owner) = nullptr;
    void* owner = nullptr;
    bool reclaimed() { return reclaim && reclaim(owner); }
};
extern thread_local AllocMeter* g_meter;

struct DevBuf {
    void* p = nullptr;
    size_t bytes = 0;
    AllocMeter* meter = nullptr;
    DevBuf() = default;
    DevBuf(const DevBuf&) = delete;
    DevBuf& operator=(const DevBuf&) = delete;
    ~DevBuf() { release(); }
    void release() {
        if (p) (void)hipFree(p);
        if (p && meter) meter->used -= (int64_t)bytes;
        p = nullptr;
        bytes = 0;
        meter = nullptr;
    }
    // (re)allocate when the requested size exceeds the current one; true
    // when the buffer moved.  Over the context's budget: OOM, buffer released.
    bool ensure(size_t n) {
        if (n <= bytes && p) return false;
        release();
        if (n == 0) n = 16;
        AllocMeter* m = g_meter;
        auto over = [&] { return m && m->budget > 0 && m->used + (int64_t)n > m->budget; };
        if (over() && !(m->reclaimed() && !over()))
            fail(MORAP_E_OOM, "device memory budget of " + std::to_string(m->budget) + " bytes exceeded (" +
                                  std::to_string(m->used) + " held, " + std::to_string(n) + " more requested)");
        hipError_t e = hipMalloc(&p, n);
        if (e != hipSuccess && m && m->reclaimed()) {
            (void)hipGetLastError();
            e = hipMalloc(&p, n);
        }
        if (e != hipSuccess) {
            p = nullptr;
            (void)hipGetLastError();   // (reported here, not by the next launch)
            fail(MORAP_E_OOM, "hipMalloc of " + std::to_string(n) + " bytes failed: " + hipGetErrorString(e));
        }
        bytes = n;
        meter = m;
        if (m) m->used += (int64_t)n;
        return true;
    }
    template <class T> T* as() const { return static_cast<T*>(p); }
};

struct PinnedBuf {
    void* p = nullptr;
    size_t bytes = 0;
    ~PinnedBuf() { if (p) (void)hipHostFree(p); }
    void ensure(size_t n) {
        if (n <= bytes && p) return;
        if (p) (void)hipHostFree(p);
        p = nullptr;
        MORAP_HIP(hipHostMalloc(&p, n, hipHostMallocDefault));
        bytes = n;
    }
    template <class T> T* as() const { return static_cast<T*>(p); }
};

// ---------------------------------------------------------------------------
// Host threads of a context, started by their first use and joined with it
// (at most 15).  A pass of queries hands work to them four times; starting 16
// threads each time took as long as the work (16 queries on 10 x 20: 20 ->
// 15 ms).
// ---------------------------------------------------------------------------
class HostPool {
public:
    HostPool() = default;
    HostPool(const HostPool&) = delete;
    HostPool& operator=(const HostPool&) = delete;
    ~HostPool() {
        {
            std::lock_guard<std::mutex> g(mu_);
            stop_ = true;
        }
        wake_.notify_all();
        for (auto& t : threads_) t.join();
    }
    // `worker` on this thread and on up to `threads` - 1 others, which may all
    // find nothing left to do; the first exception is rethrown here.
    void run(int threads, const std::function<void()>& worker) {
        std::unique_lock<std::mutex> call(call_, std::try_to_lock);
        if (threads <= 1 || !call) {   // (in use: alone)
            worker();
            return;
        }
        {
            std::lock_guard<std::mutex> g(mu_);
            try {
                while ((int)threads_.size() < threads - 1) threads_.emplace_back([this] { loop(); });
            } catch (const std::system_error&) {
                // (as many as there are)
            }
            job_ = &worker;
            tickets_ = std::min(threads - 1, (int)threads_.size());
            error_ = nullptr;
        }
        wake_.notify_all();
        std::exception_ptr mine;
        try {
            worker();
        } catch (...) {
            mine = std::current_exception();
        }
        std::unique_lock<std::mutex> g(mu_);
        tickets_ = 0;   // those still asleep are not waited for
        idle_.wait(g, [&] { return running_ == 0; });
        job_ = nullptr;
        if (!mine) mine = error_;
        g.unlock();
        if (mine) std::rethrow_exception(mine);
    }

private:
    void loop() {
        std::unique_lock<std::mutex> g(mu_);
        for (;;) {
            wake_.wait(g, [&] { return stop_ || tickets_ > 0; });
            if (stop_) return;
            --tickets_;
            ++running_;
            const std::function<void()>* job = job_;
            g.unlock();
            std::exception_ptr e;
            try {
                (*job)();
            } catch (...) {
                e = std::current_exception();
            }
            g.lock();
            if (e && !error_) error_ = e;
            if (--running_ == 0) idle_.notify_one();
        }
    }
    std::mutex call_, mu_;
    std::condition_variable wake_, idle_;
    std::vector<std::thread> threads_;
    const std::function<void()>* job_ = nullptr;
    int tickets_ = 0, running_ = 0;
    bool stop_ = false;
    std::exception_ptr error_;
};
inline int host_threads(int n) {
    return std::max(1, std::min<int>(n, (int)std::min(16u, std::thread::hardware_concurrency())));
}

// ---------------------------------------------------------------------------
// host-side model set (concatenated CSR with global indices)
// ---------------------------------------------------------------------------
struct HostModels {
    int nI = 0, nJ = 0, M = 0;
    std::vector<int32_t> state_base;   // [M+1] first global state of each model
    std::vector<int32_t> init;         // [M] global index of the initial state, -1 if done
    std::vector<int32_t> state_row;    // [S+1] global rows
    std::vector<int32_t> row_ptr;      // [R+1] global entries
    std::vector<int32_t> col;          // [N] global states
    std::vector<double>  prob;         // [N]
    std::vector<double>  rew;          // [2R]
    std::vector<uint8_t> to_done;      // [R]
    std::vector<int32_t> states_sq;    // [2S] (agent state, location), may be empty
    // neighbourhood-block form (products built from agents and automata whose
    // agent states have at most 5 actions and 5 distinct successors, the
    // state itself counted): per product state 8 int32
    //   [0..4] global successor state of agent slot d (S = the zero row:
    //          slot unused, or its successor is done), slot 0 = the agent
    //          state itself; [5] index of its agent state's block; [6] bits 0-4: slot
    //          d enters an accepting location, bits 8-12: action a enabled;
    //          [7] the record's own state (records are stored tile by tile,
    //          each tile's in the order the sweep walks it);
    // and per distinct agent-state block 32 values: P[a][d] (a-major, 25), -cost[a] (5), 0, 0,
    // where a disabled action repeats the first enabled one.
    // halo tiles (built with the block form): [4 * tiles] HTile fields, the
    // first tile of each model, per record position (tile by tile) two words
    //   w0 = halo place of slots 0..3 (8 bits each), w1 = slot 4 | accepting
    //   slots << 8 | block << 13   (HALO_MAX = the zero row),
    // and the halo lists (global states)
    std::vector<int32_t> hal_tile, hal_tile_base, hal_list;
    std::vector<uint32_t> hal_rec;
    std::vector<int32_t> blk_rec;      // [8S]
    std::vector<double>  blk_agent;    // [32 * distinct blocks]
    uint32_t blk_pattern = 0;          // bit 5a + d: some block has P[a][d] != 0
    // [M] 1: every action has one cost in all states of the model and slot 0
    // of every state is the state itself
    std::vector<uint8_t> blk_plain;
    // [M] 1: the model's agent lists a successor with probability 0 (the
    // blocks do not tell it from an unused slot; attractor ranks do)
    std::vector<uint8_t> blk_zero_prob;
    double largest_reward = 0;         // magnitude of a cost or probability reward
    int64_t S() const { return (int64_t)state_row.size() - 1; }
    int64_t R() const { return (int64_t)row_ptr.size() - 1; }
    int64_t N() const { return (int64_t)col.size(); }
};

// A tile is a run of consecutive states of one model whose rows and entries
// fit the LDS staging area of the sweep kernel.
struct Tile {
    int32_t model, s_begin, s_end, pad;
};

// A halo tile of the LDS-staged sweep: at most HALO_TILE states of one model
// whose value rows (own states and successors) number at most HALO_MAX.
// Its records are hal_rec[rec_begin .. rec_begin + n), its halo list
// hal_list[halo_begin .. halo_begin + H) (own states first, in record order).
#ifndef MORAP_HALO_TILE
#define MORAP_HALO_TILE 64
#endif
#ifndef MORAP_HALO_MAX
#define MORAP_HALO_MAX 96
#endif
constexpr int HALO_TILE = MORAP_HALO_TILE;
constexpr int HALO_MAX = MORAP_HALO_MAX;   // < 256: halo places are bytes
static_assert(HALO_MAX < 256 && HALO_TILE <= HALO_MAX && HALO_TILE <= 128, "halo tile limits");
struct HTile {
    int32_t model, rec_begin, n, halo_begin;   // n = states | H << 16
};

// sweep-kernel variants: kernel family x columns per lane x lanes per state
enum { SWEEP_CSR = 0, SWEEP_BLOCK = 1, SWEEP_HALO = 2 };
struct Variant {
    int id;        // > 0
    int cpl;       // columns per lane
    int lps;       // lanes per state
    int wg;        // threads per workgroup
    int kind;      // SWEEP_CSR (LDS-staged CSR tiles), SWEEP_BLOCK (neighbourhood blocks) or
                   // SWEEP_HALO (neighbourhood blocks, halo rows staged in LDS)
    int unroll;    // states in flight per lane group (block sweeps)
};

struct Stats {
    int64_t backups = 0, sweeps = 0, max_pair_sweeps = 0, eval_sweeps = 0, polish_sweeps = 0,
            rank_rounds = 0, floor_stops = 0;
    double bytes = 0, ms_vi = 0, ms_eval = 0, ms_total = 0, ms_sweep_kernel = 0;
    int64_t sweep_launches = 0;
    double bytes_refine = 0, ms_sweep_kernel_refine = 0;
    int64_t sweep_launches_refine = 0;
    int variant = 0, variant_refine = 0;
    // the last sweeps of batched solves, run by the LDS-staged kernel
    int64_t sweeps_tail = 0, sweep_launches_tail = 0;
    double bytes_tail = 0, ms_sweep_kernel_tail = 0;
    int variant_tail = 0;
    int resident_models = 0;
    // the assignment check after FP32 solves: pairs re-solved, columns reassigned
    int64_t refine_pairs = 0, refine_columns = 0;
};

// Values of one batched value iteration: two Jacobi buffers [S][Kp], the
// buffer holding each (model, column) pair's result, and the value at every
// model's initial state.
struct ValueSet {
    DevBuf x[2];
    DevBuf final_par;   // [M][Kp] uint8
    DevBuf c;           // [K][M] FP64
    int prec = -1, K = 0, Kp = 0;
    bool valid = false;
};

// The models whose batched value iteration keeps its values in LDS (see the
// kernels), per precision: launches over `order` (models with states, those of
// the kernels' faster form first, each part largest first), and the rest.
// Products too large for the first kernel have their states sorted by block
// and padded to steps of 64 (`rec`: per position the LDS rows of the slots, 16
// bits each -- row 0 is the zero row, row 1 + p position p --, the accepting
// slots, and the state in its product, bit 31 for padding).
struct ResidentPlan {
    struct Launch {
        bool fast;
        bool rows;              // products given as rows of entries: short rows, or streamed (columns > 0)
        int columns;            // > 0: larger products or rows, that many columns per workgroup
        int begin, n, max_states;   // (larger products: positions)
        int first;                  // place of its first model in the part's `models` (which leave out the rest)
    };
    struct Part {
        std::vector<Launch> launches;
        std::vector<int32_t> models;   // of all launches
        std::vector<uint8_t> rest;     // [M] 1: left to the batched sweeps
        int n_rest = 0;
        double rest_share = 0;         // of all states, in those models
        DevBuf d_rest;                 // the same on the device
    };
    std::vector<int32_t> rank;         // [M] place of the model in `order`
    int n_order = 0;
    std::vector<uint8_t> inst_ok;      // [M] 1: an instance's values, policy and evaluation all fit LDS
    DevBuf order, big_base, big_block, big_rec, big_init, grid_blk32, grid_blk64, grid_mat;
    // products given as rows: see RowsArgs
    bool unsolved = false;             // a model with states has none to solve for (its values are 0)
    DevBuf row_slice, row_batch, row_desc, row_place, row_value32, row_value64, short_base, short_rec, short_val32,
        short_val64;
    Part part[2];                      // MORAP_F64, MORAP_F32

    void clear(int M) {   // every model to the batched sweeps
        for (Part& q : part) {
            q.launches.clear();
            q.models.clear();
            q.rest.assign((size_t)M, 0);
            q.n_rest = 0;
            q.rest_share = 0;
        }
        inst_ok.assign((size_t)M, 0);
        unsolved = false;
    }
    size_t drop(int M) {  // the device's memory too: its bytes
        clear(M);
        size_t bytes = 0;
        for (Part& q : part) {
            bytes += q.d_rest.bytes;
            q.d_rest.release();
        }
        for (DevBuf* b : {&order, &big_base, &big_block, &big_rec, &big_init, &grid_blk32, &grid_blk64, &grid_mat, &row_slice,
                          &row_batch, &row_desc, &row_place, &row_value32, &row_value64, &short_base, &short_rec,
                          &short_val32, &short_val64}) {
            bytes += b->bytes;
            b->release();
        }
        return bytes;
    }
};

// Positions of a product's states sorted by block, each block's padded to
// steps of 64 (empty: the product was not sorted, or fits no workgroup).
struct SortedStates {
    std::vector<int32_t> block;    // per step, and << 16 where its run ends; with stages instead its lowest
                                   // << 20 and its highest << 26
    std::vector<uint32_t> rec;     // [4 positions]; with stages: the state's << 16 in word 3
    int32_t init = 0;              // position of the initial state
};
// The models `todo` sorted, [M]; by (block, stage) with `stage` (per state)
std::vector<SortedStates> sort_models(const HostModels& hm, const std::vector<int32_t>& todo, const int32_t* stage);

struct Proposer;  // mlp.hip

// Stage retirement inside the iteration (the staged form of Alg. 3): the
// states of every model split by stage (the height of their location group
// in the product's location DAG) into units, lowest stage first, with the
// neighbourhood-block records reordered inside each tile so that a unit's
// records form runs; the tiles of a unit are consecutive.
struct StagedLayout {
    uint64_t gen = ~0ull;                 // model upload the layout belongs to
    int U = 0;                            // units
    int64_t n_tiles = 0;
    std::vector<int32_t> unit_base;       // [M+1] first unit of each model
    DevBuf tiles, tile_base, rec;         // unit tiles, [U+1], records [8S]
    DevBuf rows, states, csr, live;       // [U] rows, states, CSR bytes (FP64), 0 / -1 (dead model)
    DevBuf unit_base_d, init_unit;        // [M+1], [M] unit of the initial state (-1: done)
    uint64_t tiles_gen = ~0ull;           // the same of the unit tiles (built when the batched sweeps run)
    std::vector<int32_t> stage;           // [S]
    std::vector<int32_t> h_init_unit, h_rows, h_states;   // on the host too
    std::vector<int64_t> h_csr;
    // products whose values stay in LDS: sorted states, and the models by
    // falling number of positions (every live model, or none)
    std::vector<int32_t> lds_order, lds_positions;   // [n], [M]
    DevBuf order, lds_base, lds_block, lds_rec, lds_init;
    size_t drop_lds() {   // the batched sweeps take every model: the bytes freed
        lds_order.clear();
        size_t bytes = 0;
        for (DevBuf* b : {&order, &lds_base, &lds_block, &lds_rec, &lds_init}) {
            bytes += b->bytes;
            b->release();
        }
        return bytes;
    }
    PinnedBuf h_unit_sweeps;
    // solve state
    DevBuf active, res, ymax, wc, wp, final_par, pair_sweeps, best_res, stall;   // [U][Kp]
    DevBuf c_units;                       // [K][U] (cleared at the start, unused)
    DevBuf model_active, act_models, act_prefix, act_tiles, retired, counters;
};

}  // namespace morap

// ---------------------------------------------------------------------------
// the context
// ---------------------------------------------------------------------------
struct morap_ctx {
    morap::AllocMeter meter;                        // first member: outlives every buffer
    int device = 0;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    std::string err;
    hipDeviceProp_t prop{};

    // models
    morap::HostModels hm;
    bool loaded = false;
    int64_t S = 0, R = 0, N = 0;
    int max_rows_per_state = 0;
    bool has_blocks = false;                        // the neighbourhood-block form exists
    morap::DevBuf d_blk_rec, d_blk32, d_blk64;
    bool team = false;                              // a team MDP with per-row objectives is loaded
    int team_nI = 0, team_nJ = 0;                   // its agents and tasks (d = team_nI + team_nJ)
    morap::DevBuf d_obj;                            // [R][2] objective of each reward of a row
    morap::DevBuf d_rewk32, d_rewk64, d_team_w;     // [R][Kp] scalarised rewards, [K][d] weights
    morap::DevBuf d_inst_obj;                       // [instances][2] objectives an instance evaluates
    morap::DevBuf d_team_pi;                        // [S] global row of a fixed proper policy
    morap::DevBuf d_team_E;                         // [S][d] its value per objective (the start of a solve)
    bool has_halo = false;                          // halo tiles exist
    morap::DevBuf d_htiles, d_htile_base, d_hrec, d_hlist;
    int64_t n_htiles = 0;
    morap::DevBuf d_state_row, d_row_ptr, d_col, d_prob32, d_prob64, d_rew32, d_rew64, d_to_done;
    morap::DevBuf d_state_base, d_init;
    morap::DevBuf d_state_model;                    // [S] model of every state
    morap::DevBuf d_xwarm, d_warm_map, d_warm_ab;    // warm start of a solve: values [S+1][Kp], column map,
                                                     // per-pair start a x + b [M][Kp][2]
    morap::DevBuf d_rows_per_model, d_states_per_model;  // [M] int32
    morap::DevBuf d_csr_bytes32, d_csr_bytes64;          // [M] int64: CSR bytes read per sweep

    // tiles of the batched sweep (built for the LDS limits below)
    std::vector<morap::Tile> tiles;
    std::vector<int32_t> tile_base;                 // [M+1] first tile of each model
    morap::DevBuf d_tiles, d_tile_base;

    // solve state (batched value iteration)
    int K = 0, Kp = 0, prec = -1;
    bool solved = false;
    morap::ValueSet vmain;                          // the solve's values (its precision)
    morap::ValueSet vref;                           // FP64 values of the assigned pairs after an FP32 solve
    morap::DevBuf d_pair_mask;                      // [M][Kp] uint8: pairs of a restricted solve
    morap::DevBuf d_wc32, d_wp32, d_wc64, d_wp64;   // [M][Kp]
    morap::DevBuf d_res, d_ymax;                    // [M][Kp] uint64 (bits of FP64)
    morap::DevBuf d_active;                         // [M][Kp] uint8
    morap::DevBuf d_pair_sweeps;                    // [M][Kp] int32
    morap::DevBuf d_model_active;                   // [M] uint8
    morap::DevBuf d_act_models, d_act_prefix;       // compacted active model list
    morap::DevBuf d_act_tiles;                      // the active models' tiles, in order
    morap::DevBuf d_best_res, d_stall;              // [M][Kp] FP32 rounding-floor detection
    morap::DevBuf d_counters;                       // int64 [9] (see the convergence kernel)
    morap::HostPool pool;
    morap::PinnedBuf h_counters;
    morap::PinnedBuf h_log;                         // per-launch tile counts (sweep log)
    std::vector<double> W;                          // [K][d] of the last solve
    int last_variant = 0;
    std::vector<hipEvent_t> event_pool;             // reusable per-launch timing events
    // captured chunks of sweeps: main, FP64 refine, and main again for the
    // sweep kernel of a solve's last, small active sets
    hipGraph_t chunk_graph[3] = {nullptr, nullptr, nullptr};
    hipGraphExec_t chunk_exec[3] = {nullptr, nullptr, nullptr};
    std::string graph_key[3];
    uint64_t load_gen = 0;                          // bumped by every model upload (graph keys)
    uint64_t buf_gen = 0;                           // bumped when a solve buffer moves (graph keys)

    // evaluation state
    int eK = 0;
    bool evaluated = false;
    std::vector<int32_t> assign;                    // [K][nJ]
    std::vector<int32_t> inst_k, inst_m;            // instances (column, model)
    std::vector<int64_t> inst_base;                 // [n_inst+1] state offsets
    morap::DevBuf d_inst_pack, d_inst_out;          // the instances' host arrays; what their LDS iterations report
    morap::PinnedBuf h_inst_pack, h_inst_out;
    morap::DevBuf d_xi;                             // final FP64 values [inst states]
    morap::DevBuf d_ires, d_iactive, d_ipar;        // per (instance, objective)
    morap::DevBuf d_mask, d_rank, d_mu;             // per instance state
    morap::DevBuf d_xe[2];                          // evaluation values [inst states][2]
    // the last evaluation's final values and instance layout (a warm start
    // of the next one)
    morap::DevBuf d_xe_prev, d_warm_copy;
    std::vector<int64_t> prev_inst_base;
    std::vector<int32_t> prev_inst_m;
    int prev_per_col = 0;
    bool eval_prev_valid = false;
    uint64_t prev_eval_gen = 0;
    // FP64 values at the initial states of the assigned pairs of the last
    // evaluation after an FP32 solve (valid when set), and the buffers of
    // the re-solve of other pairs for the assignment check
    std::vector<double> last_c64;
    bool last_c64_valid = false;
    morap::DevBuf d_cand_pack, d_cand_x0, d_cand_x1, d_cand_res, d_cand_act, d_cand_par, d_cand_sweeps, d_cand_val;
    morap::PinnedBuf h_cand_pack;
    morap::DevBuf d_ichanged;                       // per instance: ranks changed in the last round
    morap::DevBuf d_init_val;                       // values at the instances' initial states
    morap::DevBuf d_xr;                             // second buffer of the instance value iteration
    std::vector<int32_t> h_live_tiles;              // instance tiles still active
    morap::DevBuf d_live_tiles;
    std::vector<int8_t> h_mu;                       // policies of the last evaluate

    // streams beside the context's own for launches that share nothing
    // (created when first needed; always joined back before a call returns)
    hipStream_t side[3] = {nullptr, nullptr, nullptr};
    hipEvent_t fork_event = nullptr, join_event[3] = {nullptr, nullptr, nullptr};

    // value iteration with the values in LDS (built per upload)
    morap::ResidentPlan resident_plan;
    int layouts_in_use = 0;                         // > 0: a call builds or reads the layouts in LDS order
    morap::DevBuf d_weights;                        // [K][d] weights of the solve
    morap::DevBuf d_rest_mask;                      // [M][Kp] pairs left to the batched sweeps
    morap::PinnedBuf h_pair_sweeps, h_weights, h_c;

    // units of the stage-retiring solve (built on first use per upload)
    morap::StagedLayout staged;

    // autotuner cache: key (prec, Kp) -> variant id
    std::vector<std::pair<int64_t, int>> tuned;
    // resident workgroups per compute unit: key (variant, prec) -> count
    std::vector<std::pair<int64_t, int>> resident;

    // statistics since the last reset
    morap::Stats cum;

    // proposer
    morap::Proposer* prop_mlp = nullptr;
    std::vector<double> features;

    ~morap_ctx();
};

namespace morap {

// Run f with the context's device current; errors become return codes and
// the message stays on the context (no exception crosses the ABI).
template <class F>
int guarded(morap_ctx* c, F&& f) {
    if (!c) return MORAP_E_INVALID;
    struct MeterScope {   // the context pays for what the call allocates
        AllocMeter* prev;
        explicit MeterScope(AllocMeter* m) : prev(g_meter) { g_meter = m; }
        ~MeterScope() { g_meter = prev; }
    } scope(&c->meter);
    try {
        c->err.clear();
        MORAP_HIP(hipSetDevice(c->device));
        f();
        return MORAP_OK;
    } catch (const MorapError& e) {
        c->err = e.what();
        return e.code;
    } catch (const std::bad_alloc&) {
        c->err = "host allocation failed";
        return MORAP_E_OOM;
    } catch (const std::exception& e) {
        c->err = e.what();
        return MORAP_E_INVALID;
    } catch (...) {
        c->err = "unknown error";
        return MORAP_E_INVALID;
    }
}

// product.cpp
void build_products(morap_ctx* ctx, const morap_agent* agents, int nI, const morap_dfa* tasks, int nJ,
                    const int32_t* const* letters);
void load_models(morap_ctx* ctx, const morap_model* models, int n, int nI, int nJ);
// agent / automaton validation (INVALID on malformed input) and the done
// locations of an automaton (accepting, or no run reaches acceptance)
void check_agent(const morap_agent& a, int i);
void check_dfa(const morap_dfa& t, int j);
std::vector<uint8_t> dfa_done(const morap_dfa& t);
// the team MDP of Def. teamMDP scalarised for one weight vector, as a
// single-objective model (host only): sizes = {S, R, N, init}
void team_model_host(const morap_agent* agents, int n_agents, const morap_dfa* tasks, int n_tasks,
                     const int32_t* const* letters, const double* w, int32_t* sizes, int32_t* state_row,
                     int32_t* row_ptr, int32_t* col, double* prob, double* rew, uint8_t* to_done);
// the team MDP with its d = 2n objectives: per row the two rewards and the
// objective each belongs to (host only)
void team_model_mo_host(const morap_agent* agents, int n_agents, const morap_dfa* tasks, int n_tasks,
                        const int32_t* const* letters, int32_t* sizes, int32_t* state_row, int32_t* row_ptr,
                        int32_t* col, double* prob, double* rew, int32_t* obj, uint8_t* to_done);
// one product on the host (no context, no device): sizes = {S, R, N, init},
// arrays filled where non-NULL
void product_host(const morap_agent* a, const morap_dfa* t, const int32_t* letters, int32_t* sizes,
                  int32_t* state_row, int32_t* row_ptr, int32_t* col, double* prob, double* rew, uint8_t* to_done,
                  int32_t* states);
void upload_models(morap_ctx* ctx, bool team = false);
// Frees the layouts in LDS order, which every solve can do without (the batched
// sweeps take its models until the next upload), unless a call uses them; true
// when there were any.
bool drop_layouts(morap_ctx* ctx);
struct LayoutsInUse {
    morap_ctx* c;
    explicit LayoutsInUse(morap_ctx* ctx) : c(ctx) { ++c->layouts_in_use; }
    LayoutsInUse(const LayoutsInUse&) = delete;
    LayoutsInUse& operator=(const LayoutsInUse&) = delete;
    ~LayoutsInUse() { --c->layouts_in_use; }
};
void load_team_model(morap_ctx* ctx, int n_agents, int n_tasks, const morap_model* model, const int32_t* obj);
// agents, tasks and objectives of the loaded models (a team model: its own)
inline int n_agents_of(const morap_ctx* c) { return c->team ? c->team_nI : c->hm.nI; }
inline int n_tasks_of(const morap_ctx* c) { return c->team ? c->team_nJ : c->hm.nJ; }
inline int n_obj_of(const morap_ctx* c) { return n_agents_of(c) + n_tasks_of(c); }

// solver.cpp
// warm (nullable, [K]): column of the previous solve each column starts from
// (-1: from 0); used when the previous solve was FP32 with at least as many
// padded columns, ignored otherwise
void solve(morap_ctx* ctx, const double* W, int K, const morap_vi_opts& o, double* c_out, Stats& st,
           const int32_t* warm = nullptr);
// the same value iteration with stage retirement inside it (FP64, block form)
void solve_staged(morap_ctx* ctx, const double* W, int K, const morap_vi_opts& o, double* c_out, Stats& st);
// warm (nullable): per column, the column of the previous evaluation whose
// instance of the same task on the same model starts the policy evaluation
// from its final values (-1: from 0, as Alg. 4)
//
// refine (nullable, FP32 solves of block-form products): the assignment
// (assign) is checked against FP64 values -- every pair whose slack lies
// within twice the column's largest FP32 error on its assigned pairs is
// re-solved in FP64, the column is assigned again on the FP64 values, and a
// column whose value rises takes the new assignment, which is then
// evaluated; refine receives the assignment evaluated
void evaluate(morap_ctx* ctx, const int32_t* assign, int K, const morap_vi_opts& o, double* r_out, Stats& st,
              const int32_t* warm = nullptr, int32_t* refine = nullptr);
const std::vector<Variant>& variants();

// assign.cpp
// (pool: host threads to spread the columns over, or null: threads of its own)
void assign_columns(int nI, int nJ, const double* c, int K, int32_t* out, HostPool* pool = nullptr);
// one column's optimal assignment and the slack of every pair against it
std::vector<int32_t> assignment_slack(int nI, int nJ, const double* ck, double* slack);

// qp.cpp
void project_inner(const double* Phi, int m, int d, const double* t, const double* M, double* x,
                   double* lam);
void project_outer(const double* W, const double* R, int n, int d, const double* t, const double* M,
                   double* z);

// query.cpp
void query_batch(morap_ctx* ctx, const double* T, const double* W0, int Q, const double* M,
                 const morap_query_opts& o, morap_query_result* res);

// mlp.hip
void proposer_destroy(Proposer* p);
// device address of the fixed inference scratch, taken once per device
void proposer_scratch_init(int device);

// kernels (vi.hip): launch wrappers
namespace k {
void fill_u8(hipStream_t s, uint8_t* p, uint8_t v, int64_t n);
void fill_i32(hipStream_t s, int32_t* p, int32_t v, int64_t n);
void fill_u64(hipStream_t s, uint64_t* p, uint64_t v, int64_t n);
void fill_f32(hipStream_t s, float* p, float v, int64_t n);
void fill_f64(hipStream_t s, double* p, double v, int64_t n);
void fill_i64(hipStream_t s, int64_t* p, int64_t v, int64_t n);
void to_f32(hipStream_t s, const double* in, float* out, int64_t n);

struct SweepArgs {
    const Tile* tiles;
    const int32_t* tile_base;
    const int32_t* act_models;
    const int32_t* act_prefix;
    const int64_t* counters;
    const int32_t* state_row;
    const int32_t* row_ptr;
    const int32_t* col;
    const void* prob;
    const void* rew;
    const void* wc;
    const void* wp;
    const uint8_t* active;
    const void* x_in;
    void* x_out;
    unsigned long long* res;
    unsigned long long* ymax;
    int Kp;
    const int32_t* rec;     // neighbourhood-block records [8S]
    const void* ablk;       // agent blocks [32 * agent states] (precision of the sweep)
    int32_t zero_row;       // S: the value row that always holds 0
    uint32_t pattern;       // union of the blocks' nonzero (action, slot) entries
    const int32_t* act_tiles;  // global index of every active tile, in order
    const void* rewk;          // team models: scalarised reward of every (row, column) [R][Kp] (nullable)
    const HTile* htiles;       // halo tiles (LDS-staged sweep)
    const uint2* hrec;         // their records
    const int32_t* hlist;      // their halo lists
};
// batched Bellman sweep: variant v, precision prec (MORAP_F32/F64)
void sweep(hipStream_t s, int prec, const Variant& v, int grid, int ktiles, const SweepArgs& a);
void sweep_block(hipStream_t s, int prec, const Variant& v, int grid, int ktiles, const SweepArgs& a);
// workgroups of the variant's kernel that fit one compute unit at once
int sweep_resident(int prec, const Variant& v);
int sweep_block_resident(int prec, const Variant& v);
// LDS-staged sweep over halo tiles (halo.hip): FP32, k-tiles of 64 columns
void sweep_halo(hipStream_t s, int prec, const Variant& v, int grid, int ktiles, const SweepArgs& a);
int sweep_halo_resident(const Variant& v, uint32_t pattern);
int sweep_lds_rows();
int sweep_lds_nnz();
int sweep_tile_states(const Variant& v);

struct ConvergeArgs {
    unsigned long long* res;
    unsigned long long* ymax;
    uint8_t* active;
    uint8_t* final_par;
    int32_t* pair_sweeps;
    uint8_t* model_active;
    double* c;              // [K][M]
    const int32_t* init;    // [M]
    const uint8_t* mask;    // [M][Kp] pairs to solve (nullable: all)
    const void* x_out;      // buffer written by the sweep just finished
    int64_t* counters;
    int M, K, Kp, prec, out_par;
    double eps, unit;       // stop at res <= max(eps, unit * ymax)
    // FP32 rounding floor: a pair whose change has set no new minimum for
    // stall_sweeps sweeps (0: off) and is within floor * ymax stops too
    double* best_res;       // [M][Kp] smallest change so far
    int32_t* stall;         // [M][Kp] sweeps since it was set
    int stall_sweeps;
    double floor;
    const int32_t* tile_base;
    int32_t* act_models;
    int32_t* act_prefix;
    const int32_t* rows_per_model;   // [M] rows (backups per active column)
    const int32_t* states_per_model; // [M] states (value traffic per active column)
    const int64_t* csr_bytes;        // [M] CSR bytes read per sweep of an active model
    int32_t* act_tiles;              // [tiles] global index of every active tile, in order
    int relist;                      // compaction only re-lists the active models (no sweep is counted)
};
void converge(hipStream_t s, const ConvergeArgs& a);
void compact(hipStream_t s, const ConvergeArgs& a);
// the same active models listed over the tiles of a.tile_base (a change of
// sweep kernel between the gather and the LDS-staged tiles)
void relist(hipStream_t s, ConvergeArgs a);
void init_solve(hipStream_t s, const ConvergeArgs& a);
// the same without the active lists: no pair is left to the batched sweeps
// a solve's pair sweeps, values at the initial states and counters to pinned
// memory in one launch
constexpr size_t REPORT_BYTES = (size_t)1 << 20;
void report(hipStream_t s, int64_t n_ps, const int32_t* ps, int32_t* h_ps, int64_t n_c, const double* c, double* h_c,
            const int64_t* counters, int64_t* h_counters);
// (with n_W > 0 it also brings weights over from pinned memory)
void init_pairs(hipStream_t s, const ConvergeArgs& a, const double* from = nullptr, double* W = nullptr,
                int64_t n_W = 0);
constexpr int64_t SMALL_WEIGHTS = 8192;   // (a 2 x 2 problem's solve: 58.8 us, 60.4 with a copy of their own)
// mask[m][k] = flag[m]
void model_mask(hipStream_t s, int M, int Kp, const uint8_t* flag, uint8_t* mask);

// a block of the grid pattern: its 17 nonzero probabilities in (action, slot)
// order, the 5 costs, padding
constexpr int GRID_BLK = 24;

// Value iteration with the values resident in LDS (resident.hip): the sweeps
// sweep0 + 1 .. sweep1 (both even) of the listed models' pairs that have not
// stopped (pair_sweeps 0), each pair to its stop.
struct ResidentArgs {
    const int32_t* order;       // [n_models] models, at most the kernel's states each
    int n_models, groups;       // groups: column groups of a model (set by the launch)
    const int32_t* state_base;  // [M+1]
    const int32_t* init;        // [M]
    const int32_t* rec;         // neighbourhood-block records [8S]
    const void* ablk;           // agent blocks (precision of the solve)
    int32_t zero_row;
    const double* W;            // [K][d] weights
    int nI, nJ, d, K, Kp, M;
    void* x0;                   // [S+1][Kp] start values (warm or sweep0 > 0), final values
    void* x1;                   // after the last launch: iterate before the last, of pairs still running
    uint8_t* active;            // [M][Kp] set for pairs still running after the last launch
    uint8_t* final_par;         // [M][Kp]
    int32_t* pair_sweeps;       // [M][Kp]
    double* c;                  // [K][M] values at the initial states
    double* best_res;           // [M][Kp] FP32 rounding floor, kept between launches
    int32_t* stall;             // [M][Kp]
    int64_t* counters;          // [8]: pairs stopped at the rounding floor
    double eps, unit, floor;
    int stall_sweeps, warm, sweep0, sweep1, last;
    const int32_t* short_base;  // products given as short rows: [M] first of their states, in that layout
    const uint4* short_rec;     // [its states][2] LDS rows of the entries, 16 bits each
    const void* short_val;      // [its states][SHORT_VALUES] (precision of the solve)
    const void* grid_blk;       // compact blocks (precision of the solve), see GRID_BLK
    const float* grid_mat;      // [blocks][4][8] a move's five slots, the probability to stay of the block
    // larger products: states sorted by block, padded to steps of 64
    const int32_t* big_base;    // [M+1] first position (a multiple of 64)
    const int32_t* big_block;   // [positions / 64] block of the step, << 16: first step of the next block's run
    const uint4* big_rec;       // [positions] LDS rows of the slots (see the plan)
    const int32_t* big_init;    // [M] position of the initial state in its product
    // instances (FP64, one column each: see the instance kernels): `order`
    // lists instances, pair_sweeps is per instance, x0 their values
    const int32_t* inst_model;
    const int32_t* inst_k;
    const int64_t* inst_base;
    const double *iwc, *iwp, *ieps;   // weights and stop of every instance
    const double* iscale;             // scale of the start from `start` (with iwc > 0, else from 0)
    const float *start0, *start1;     // an FP32 solve's values (nullable: from 0)
    const uint8_t* start_par;
    int start_Kp;
};
// Products given as rows, 64 consecutive states a slice; the rows and entries
// of a slice in lockstep, every lane its own state's.  A row is its probability
// reward, its cost reward and its entries, as many as the longest of the 64
// lanes has (a shorter one ends in entries of probability 0 at the zero row; a
// state with fewer rows than the slice's most repeats its first).  The rewards
// name two rows behind the product's (rounded up to slices), which hold the
// columns' weights.  Four places make a batch; a slice starts a new one, and an
// empty one lies behind the last.
struct RowsArgs : ResidentArgs {
    const int32_t* slice;       // [M+1] first slice of the model
    const int32_t* batch;       // [slices+1] first batch of the slice
    const int32_t* desc;        // [batches] bits 0-3: a row ends at that place, bit 4: the slice does
    const uint2* place;         // [batches][64] four LDS rows, 16 bits each
    const void* value;          // [batches][64][4] rewards and probabilities
};
// Largest reward of a problem whose values may stay in LDS: at any sweep limit no
// value overflows, so there is no infinity and no NaN to treat as the batched
// sweeps' maxima do (which pass over a NaN and start at minus infinity).
constexpr double largest_reward(int prec) { return prec == MORAP_F32 ? 1e29 : 1e298; }
// columns per workgroup of a product of that many states, 0 if it does not fit
int rows_columns(int prec, int states);
void resident_rows(hipStream_t s, int prec, int columns, int max_states, const RowsArgs& a);
// products given as rows whose states have at most five rows of at most three
// entries (resident_capacity with `fast` false, classes as the block form's)
void resident_short(hipStream_t s, int prec, bool wide, int max_states, ResidentArgs a);
// The layouts of products given as rows, from the arrays of the upload (FP64 and
// the same in FP32).
struct RowsLayout {
    int M, n_slices;
    int64_t S;
    const int32_t *state_base, *state_model, *state_row, *row_ptr, *col;
    const double *prob, *rew;
    const int32_t* short_base;           // [M], -1: not in this layout
    uint4* short_rec;
    double* short_val64;
    float* short_val32;
    const int32_t *slice, *batch;        // as in RowsArgs, and the batches' contents
    int32_t* desc;
    uint2* place;
    double* value64;
    float* value32;
};
void lay_out_short(hipStream_t s, const RowsLayout& a);
void lay_out_rows(hipStream_t s, const RowsLayout& a);
constexpr int SHORT_VALUES = 26;   // probabilities [5][3], cost and probability rewards [5]; one unused
// every block's nonzero entries lie within the grid pattern
bool has_grid_pattern(uint32_t union_pattern);
// largest product (states) the kernel holds; `fast`: every block has the grid
// pattern, every action one cost and slot 0 of every state is the state itself
int resident_capacity(int prec, bool fast);
// register steps (states per thread) of a product of that many states; a
// launch takes models of one class
int resident_class(int states);
// entry e = 5 action + slot of a block belongs to the grid pattern
bool grid_entry(int e);
// largest number of sorted and padded states that fits with one FP32 column
int resident_most_positions();
// the same for instances of products of one class, and of larger products
void resident_inst(hipStream_t s, bool fast, int max_states, ResidentArgs a);
void resident_inst_large(hipStream_t s, int max_positions, ResidentArgs a);
// columns per workgroup of a larger product of that many sorted and padded
// states, 0 if it does not fit
int resident_big_columns(int prec, int positions);
void resident_large(hipStream_t s, int prec, int columns, int max_positions, ResidentArgs a);
// wide: several columns per workgroup (4 in FP32, 2 in FP64), else one
void resident(hipStream_t s, int prec, bool fast, bool wide, int max_states, ResidentArgs a);

// Policies and evaluations of instances in LDS (instance.hip), one workgroup
// per listed instance
struct InstanceArgs {
    const int32_t* order;       // [n] instances of this launch
    int n;
    const int32_t* inst_model;
    const int64_t* inst_base;
    const int32_t* state_base;
    const int32_t* rec;         // neighbourhood-block records
    const double* ablk;         // agent blocks
    int32_t zero_row;
    const double *iwc, *iwp;    // the instance's weights
    const double* xi;           // final values of the instances
    int8_t* mu;                 // policies
    double tau;
    int widenings;              // of the tie tolerance
    int64_t* counters;          // [0] states without a rank, [1] relaxation rounds (largest)
    // evaluation
    double* xe;                 // [instance state][2] values
    const double* xe_prev;      // the last evaluation's values
    const int64_t* prev_src;    // first state of an instance's start there (-1: none; nullable)
    int from_values;            // start from xi
    int32_t* sweeps;            // [2 instances] sweep of the stop, 0: running
    double eps;
    int sweep0, sweep1;
};
int policy_capacity();          // states
void inst_policy(hipStream_t s, int max_states, const InstanceArgs& a);
int eval_capacity();            // states
int eval_class(int states);     // a launch takes instances of one class
void inst_eval(hipStream_t s, int max_states, const InstanceArgs& a);

// stage retirement (staged.hip)
struct StageArgs {
    const int32_t* unit_base;   // [M+1]
    const int32_t* init_unit;   // [M] unit of the initial state, -1 if done
    const int32_t* init;        // [M] initial state
    const int32_t* rows;        // [U] rows (backups per active column)
    const int32_t* states;      // [U] states
    uint8_t* active;            // [U][Kp]
    unsigned long long* res;    // [U][Kp]
    unsigned long long* ymax;   // [U][Kp]
    uint8_t* model_active;      // [U]
    double* c;                  // [K][M] values at the initial states
    uint8_t* final_par;         // [M][Kp]
    int32_t* pair_sweeps;       // [M][Kp] sweep in which the initial state's unit retired
    int64_t* retired;           // [U * Kp] (unit, column) pairs retired in this sweep
    int64_t* counters;          // as the convergence kernel's, [9] / [10] the list counts
    const Tile* tiles;          // unit tiles
    const int32_t* tile_base;   // [U+1]
    const int32_t* rec;         // reordered block records [8S]
    const void* x_out;          // the buffer the sweep wrote (precision prec)
    void* x_in;                 // the buffer it read
    double* best_res;           // [U][Kp] FP32 rounding floor: smallest change so far
    int32_t* stall;             // [U][Kp] sweeps since it was set
    int stall_sweeps;           // 0: no floor stop (FP64)
    double floor;
    int M, K, Kp, out_par, slot, prec;   // slot: 9 or 10, the list count of this sweep
    double eps, unit;
};
// stage retirement with the values in LDS: best_res, stall and unit_sweeps per
// (unit, column), big_block with the stages of a step
struct StagedLdsArgs : ResidentArgs {
    const int32_t* unit_base;   // [M+1]
    const int32_t* init_unit;   // [M]
    int32_t* unit_sweeps;       // [U][Kp] sweep in which the unit retired, 0 before
};
// columns per workgroup of a product of that many positions and stages (0: it
// does not fit), one kernel class per (columns, threads)
int staged_columns(int prec, int positions, int stages);
int staged_threads(int prec, int columns, int positions);
void staged_lds(hipStream_t s, int prec, int columns, int threads, int max_positions, const StagedLdsArgs& a);
void stage_converge(hipStream_t s, const StageArgs& a);
void stage_copy(hipStream_t s, const StageArgs& a);

// instances (polish, policy extraction, evaluation)
struct InstArgs {
    const int32_t* inst_model;
    const int32_t* inst_k;
    const int64_t* inst_base;
    const int32_t* inst_tiles;     // (instance, local state begin) pairs
    int n_tiles;
    int n_inst;
    const int32_t* state_base;
    const int32_t* state_row;
    const int32_t* row_ptr;
    const int32_t* col;
    const double* prob;
    const double* rew;
    const uint8_t* to_done;
    const int32_t* init;
    int cus;                       // compute units (resident-sized grids of the striding kernels)
    // team models (nullable otherwise): FP64 scalarised reward of every
    // (row, column) with its leading dimension, every row's two objectives
    // and the two objectives each instance evaluates (-1: none)
    const double* rewk;
    int rewk_ld;
    const int32_t* row_obj;
    const int32_t* inst_obj;
    const uint8_t* resident;       // [n_inst] instances whose iterations run in LDS (nullable)
};
// team models: one Jacobi sweep of the per-objective evaluation of the fixed
// policy pi (E[s][o], res = max change as FP64 bits), and the start values
// x[s][k] = sum_o W[k][o] E[s][o] minus a margin (FP32 or FP64 x, [S+1][Kp])
void team_eval_sweep(hipStream_t s, int64_t S, int d, const int32_t* pi, const int32_t* row_ptr,
                     const int32_t* col, const double* prob, const double* rew, const int32_t* obj,
                     const double* E_in, double* E_out, unsigned long long* res);
void team_start(hipStream_t s, int64_t S, int K, int Kp, int d, const double* W, const double* E, int prec,
                void* x);
// out[q] = x[idx[q]] (0 where idx[q] < 0): one value per instance state
void gather_values(hipStream_t s, int n, const int64_t* idx, const double* x, double* out);
// runs (dst, src, length) of instance states [.][2] copied from prev to x
void copy_runs(hipStream_t s, const int64_t* runs, int n_runs, const double* prev, double* x);
// evaluation start from the instances' scalarised values xi (iwarm: per
// instance, 1 where its values were warm-started)
void eval_start(hipStream_t s, const InstArgs& a, const double* xi, const double* iwc, const double* iwp,
                const uint8_t* iwarm, double* xe);
// team models: out[r][k] = W[k][obj[r][0]] rew[r][0] + W[k][obj[r][1]] rew[r][1]
void team_rewards(hipStream_t s, int64_t R, int K, int Kp, int d, const double* W, const int32_t* obj,
                  const double* rew, double* out64, float* out32);
void gather_columns(hipStream_t s, const InstArgs& a, int prec, const void* x0, const void* x1,
                    const uint8_t* final_par, int Kp, double* xi);
// start of an FP32 solve from the previous one's final values: out[s][k] =
// a x_prev[s][map[k]] + b (the buffer its pair froze in; ab[m][k] = (a, b))
// where map[k] >= 0 and a != 0, 0 elsewhere (and on the zero row)
void warm_columns(hipStream_t s, int64_t S, int Kp, int K, const int32_t* map, const int32_t* state_model,
                  const float* ab, const float* x0, const float* x1, const uint8_t* final_par, int Kp_old,
                  float* out);
// FP64 start of the instances from the FP32 solve's values, scaled by
// scale[inst] (instances with a zero cost weight start from 0)
void warm_start(hipStream_t s, const InstArgs& a, const void* x0, const void* x1, const uint8_t* final_par, int Kp,
                const double* scale, const double* iwc, double* xi);
// stop test of n entries: residual <= eps, or <= eps_i[i] where eps_i is given
void inst_converge(hipStream_t s, int n, unsigned long long* res, uint8_t* active, uint8_t* par, int out_par,
                   double eps, int64_t* counter, const double* eps_i = nullptr);
void opt_mask(hipStream_t s, const InstArgs& a, const double* wc, const double* wp, const double* x,
              double tau, uint32_t* mask, int32_t* rank, int8_t* mu, bool only_unranked);
void eval_sweep(hipStream_t s, const InstArgs& a, const int8_t* mu, const uint8_t* active,
                const double* x_in, double* x_out, unsigned long long* res);
void count_unranked(hipStream_t s, const InstArgs& a, const int32_t* rank, int64_t* counter);
// attractor ranks as BFS distances (in-place relaxation sweep) and the action
// choice once they are final
void relax_ranks(hipStream_t s, const InstArgs& a, const uint32_t* mask, int32_t* rank, int base, bool reverse,
                 int local, int64_t* changed, uint8_t* inst_changed);
void choose_actions(hipStream_t s, const InstArgs& a, const uint32_t* mask, const int32_t* rank, int8_t* mu,
                    int base, int64_t* max_rank);
// per-instance flags: `width` entries per instance, active when the instance
// has a live initial state
void set_active(hipStream_t s, int n, const InstArgs& a, uint8_t* active, unsigned long long* res,
                uint8_t* par, int width);
// copy the values of entries frozen in buffer 1 into buffer 0
void select_final(hipStream_t s, const InstArgs& a, double* x0, const double* x1, const uint8_t* par,
                  int width);
// pair mask of a restricted solve: mask[m][k] = 1 for the instances' pairs
void mark_pairs(hipStream_t s, const InstArgs& a, int Kp, uint8_t* mask);
// one FP64 value-iteration sweep of instances over the neighbourhood blocks
// (block.hip); residuals per instance
void inst_vi_sweep(hipStream_t s, const InstArgs& a, const int32_t* rec, const double* ablk, const double* wc,
                   const double* wp, const uint8_t* active, const double* x_in, double* x_out,
                   unsigned long long* res, int32_t zero_row, uint32_t pattern);
// one Alg. 4 sweep (both objectives) of instances over the neighbourhood
// blocks (block.hip)
void eval_block_sweep(hipStream_t s, const InstArgs& a, const int32_t* rec, const double* ablk, const int8_t* mu,
                      const uint8_t* active, const double* x_in, double* x_out, unsigned long long* res,
                      int32_t zero_row, uint32_t pattern);
// out[2q + o] = x[2 idx[q] + o] (0 when idx[q] < 0)
void gather_init(hipStream_t s, int n, const int64_t* idx, const double* x, double* out);
}  // namespace k

}  // namespace morap
