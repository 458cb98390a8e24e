// Continuous-batching server of Taylor-Green solves on one GPU.
//
// Admission: a request is admitted when a slot is free and a first-fit block
// of the caller's arena holds its footprint (state, Runge-Kutta register,
// face-trace / interface-flux / forcing workspace, descriptors, a device ring
// of kinetic-energy records).  Admitted solves stay resident until done.
//
// Execution: one host thread and one stream per polynomial order, started with
// the first request of the order.  Each round a thread sets up the admitted
// solves of its order, then advances all it runs by a number of Runge-Kutta
// steps; within a step, the stages of all its solves run in shared launches
// (one k_grad, one batched network launch for the corrected solves, one
// k_resid per stage).  Orders neither wait for each other's rounds nor for
// each other's launches, and overlap on the device.  Requests that arrive
// while others run join them at their order's next round.  Per-solve time
// steps and step counts are independent; nothing is reduced across solves, so
// each result is what the solve computes alone.  After each round the stream
// is synchronised once: kinetic-energy records are collected, non-finite
// solves are failed.  Finished solves are copied out, and their arena blocks
// released, by another thread while the next round is enqueued and runs.
// (Two corrected P=3, two P=6 and two P=8 solves on 4^3, one of each on 8^3:
// 7.6 ms with one thread for all orders, whose rounds waited for the slowest
// order and for the copies, 3.9 so.)
//
// Fallback of the learned part: a corrected solve (network forcing, Eq. (4),
// or Algorithm 1's correction) keeps a copy of its state from the start of
// each round, a state already checked healthy.  At the end of every round its
// state is checked again (finite diagnostics, kinetic energy not above
// (1 + kFallbackKeRise) times the initial value -- the Taylor-Green flow
// decays, so a rise means the forcing is driving it); when that or any of
// the round's kinetic-energy records fails, the solve returns to the copy,
// drops the records after it, and continues from there as the uncorrected
// low-order solve (Eq. (3)), flagged in its status.  A non-finite record of
// an uncorrected solve fails that solve.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <condition_variable>
#include <cstring>
#include <deque>
#include <future>
#include <map>
#include <memory>
#include <mutex>
#include <thread>
#include <vector>

#include "nn_internal.hpp"

namespace dgnn {

constexpr int kHist = 64;    // device KE records per solve between synchronisations
constexpr int kChunk = 16;   // steps per round of the costliest solve of an order
constexpr int kChunkMax = 256;  // steps per round of any solve
constexpr size_t kDiagDoubles = 8;
// finished states go out in chunks, by way of pinned memory: a copy straight
// to pageable memory goes through the runtime's own, one piece after the
// other (15 MB: 0.97 ms to memory that was written before, 1.9 ms to new)
constexpr size_t kStageChunk = 2 << 20;
constexpr int kStageSlots = 4;
constexpr double kFallbackKeRise = 1e-3;   // relative kinetic-energy rise that ends the correction

static double now_s() {
    return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch()).count();
}
static size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Foot {
    size_t q, k, ws, desc, hist, health, ckpt, total;
};

// arena layout of one solve; a corrected solve also holds the state copy of
// its fallback
static Foot foot(const Mesh& m, bool corrected) {
    Foot f;
    const size_t field = a256((size_t)5 * m.E * m.n_p * sizeof(double));
    f.q = 0;
    f.k = field;
    f.ws = 2 * field;
    f.desc = f.ws + a256(ws_layout(m).total);
    f.hist = f.desc + a256(4 * sizeof(SolveDesc));
    f.health = f.hist + a256(kHist * kDiagDoubles * sizeof(double));
    f.ckpt = f.health + a256(kDiagDoubles * sizeof(double));
    f.total = f.ckpt + (corrected ? field : 0);
    return f;
}

static dg_params request_params(const solve_request& r) {
    dg_params p;
    std::memset(&p, 0, sizeof(p));
    p.N = r.N;
    p.P = r.P;
    p.viscous = 1;
    p.L = 2.0 * M_PI;
    p.Re = r.Re;
    p.Mach = r.Mach > 0 ? r.Mach : 0.1;
    p.gamma = 1.4;
    p.Pr = 0.72;
    p.Cs = r.Cs;
    p.Pr_t = 0.6;
    p.p_ref = 1.0 / (p.gamma * p.Mach * p.Mach);
    return p;
}

struct Solve {
    uint64_t id = 0;
    solve_request req;
    Mesh mesh;
    int state = SOLVE_QUEUED;
    int error = 0;
    double t_submit = 0, t_admit = 0, t_done = 0;
    std::atomic<int64_t> steps{0};
    int64_t n_steps = 0;
    double dt = 0;
    size_t off = 0, bytes = 0;
    double* q = nullptr;
    double* k = nullptr;
    char* ws = nullptr;
    SolveDesc* ddesc = nullptr;
    double* hist = nullptr;
    double* health = nullptr;        // diagnostics of the state at the end of a round
    int slot = -1;                   // of the server's slots, while running
    double* records = nullptr;       // pinned: the slot's records read back at the end of a round
    double* ckpt = nullptr;          // corrected solves: state at the start of the round
    bool nn_active = false;          // the correction is applied
    bool fell_back = false;          // continued uncorrected after a failed check
    int64_t fallback_step = 0;
    int64_t ckpt_steps = 0;
    double ke0 = 0.0;
    int par = 0;
    std::vector<double> pending_t;   // times of device records not yet collected
    std::vector<double> ke;          // collected (t, KE) pairs
    std::atomic<bool> inject{false};
};

// first-fit allocator over [0, size) with coalescing
class Arena {
  public:
    void reset(size_t size) {
        free_.clear();
        if (size) free_[0] = size;
    }
    bool alloc(size_t n, size_t& off) {
        for (auto it = free_.begin(); it != free_.end(); ++it)
            if (it->second >= n) {
                off = it->first;
                const size_t rest = it->second - n;
                free_.erase(it);
                if (rest) free_[off + n] = rest;
                return true;
            }
        return false;
    }
    void release(size_t off, size_t n) {
        auto it = free_.emplace(off, n).first;
        auto nx = std::next(it);
        if (nx != free_.end() && it->first + it->second == nx->first) {
            it->second += nx->second;
            free_.erase(nx);
        }
        if (it != free_.begin()) {
            auto pv = std::prev(it);
            if (pv->first + pv->second == it->first) {
                pv->second += it->second;
                free_.erase(it);
            }
        }
    }

  private:
    std::map<size_t, size_t> free_;
};

}  // namespace dgnn

using namespace dgnn;

namespace dgnn {

// the thread of one order
struct Worker {
    int PP = 0;
    std::thread th;
    std::vector<Solve*> inbox;   // admitted, not yet set up (under the server's lock)
    hipStream_t st = nullptr;    // one of the server's, with the first request
    std::deque<Solve*> done;     // finished, not yet copied out (under the server's lock)
    bool delivering = false;     // a thread is at it (likewise)
    std::future<void> delivery;  // that thread
    char* stage = nullptr;       // pinned: kStageSlots chunks of states on their way out
};

// per slot in solve_server::records: a round's kinetic-energy records, then the
// health record
constexpr size_t kRecords = (kHist + 1) * kDiagDoubles;

}  // namespace dgnn

struct solve_server {
    char* base = nullptr;
    size_t bytes = 0;
    int max_slots = 0;
    int device = 0;
    std::mutex mu;
    std::condition_variable cv;
    std::map<uint64_t, std::unique_ptr<Solve>> solves;
    std::deque<Solve*> queue;
    std::vector<int> free_slots; // of max_slots, those no admitted solve holds
    uint64_t next_id = 1;
    bool stop = false;
    Worker workers[dgnn::kMaxPP + 1];
    // What the solves need besides the arena is made with the server, so that
    // its creation fails and not the solves later: a stream for each order,
    // given out in turn as orders come into use (consecutive streams go to
    // different hardware queues), one after them for finished states, and the
    // slots' records.  (A stream for each order's states: the copy of 10 MB
    // took 1 ms longer.)
    hipStream_t streams[DG_MAX_ORDER + 1] = {};
    int streams_used = 0;
    double* records = nullptr;   // pinned
    Arena arena;
    double busy = 0.0;           // time in which some order had a round running
    int in_round = 0;
    double round_t0 = 0.0;
    int64_t batches = 0;
};

namespace dgnn {

// hands queued requests, in their order, to the threads of their orders while
// slots are free; one that finds no room in the arena lets later ones pass
// (lock held)
static void admit_waiting(solve_server* S) {
    for (auto it = S->queue.begin(); it != S->queue.end() && !S->free_slots.empty();) {
        Solve* s = *it;
        size_t off;
        if (!S->arena.alloc(s->bytes, off)) {
            ++it;
            continue;
        }
        s->off = off;
        s->state = SOLVE_RUNNING;
        s->t_admit = now_s();
        s->slot = S->free_slots.back();
        S->free_slots.pop_back();
        s->records = S->records + s->slot * kRecords;
        S->workers[s->mesh.PP].inbox.push_back(s);
        it = S->queue.erase(it);
    }
}

// ends a solve: its state, and its room for others
static void leave(solve_server* S, Solve* s, int state, int code) {
    {
        std::lock_guard<std::mutex> lk(S->mu);
        s->state = state;
        s->error = code;
        s->t_done = now_s();
        S->arena.release(s->off, s->bytes);
        S->free_slots.push_back(s->slot);
        admit_waiting(S);
    }
    S->cv.notify_all();
}

static void fail(solve_server* S, Solve* s, int code) { leave(S, s, SOLVE_FAILED, code); }

static int write_descs(Solve* s, hipStream_t st);
static void stage_desc(const Solve* s, int par, SolveDesc& d);

// admitted solves, first half: pointers, TGV state, its traces and
// diagnostics (which are also the record at t = 0), on their way back
static int admit_begin(solve_server* S, Worker& W, Solve* s) {
    // once more, on this thread's device (solve_submit built it on the caller's)
    const dg_params prm = request_params(s->req);
    Mesh mesh;
    int rc = make_mesh(&prm, mesh);
    if (rc) return rc;
    {
        std::lock_guard<std::mutex> lk(S->mu);
        s->mesh = mesh;
    }
    const Foot f = foot(s->mesh, s->req.use_nn != 0);
    char* p = S->base + s->off;
    s->q = (double*)(p + f.q);
    s->k = (double*)(p + f.k);
    s->ws = p + f.ws;
    s->ddesc = (SolveDesc*)(p + f.desc);
    s->hist = (double*)(p + f.hist);
    s->health = (double*)(p + f.health);
    s->ckpt = s->req.use_nn ? (double*)(p + f.ckpt) : nullptr;
    s->nn_active = s->req.use_nn != 0;
    if ((rc = init_tgv_impl(s->mesh, s->q, W.st))) return rc;
    if ((rc = diag_impl(s->mesh, s->q, s->hist, s->ws, W.st))) return rc;
    if (hipMemcpyAsync(s->records, s->hist, kDiagDoubles * sizeof(double), hipMemcpyDeviceToHost, W.st) != hipSuccess)
        return set_error(DG_EHIP, "admission readback failed");
    SolveDesc d;
    stage_desc(s, 1, d);
    if (launch_traces(s->mesh.PP, d, W.st) != hipSuccess) return set_error(DG_EHIP, "trace launch failed");
    return DG_OK;
}

// second half, with the diagnostics: time step and stage descriptors
static int admit_end(solve_server* S, Worker& W, Solve* s) {
    const double* rec = s->records;
    const double dt0 = stable_dt_from_diag(s->mesh, rec, 0.4);
    if (!(dt0 > 0) || !std::isfinite(dt0)) return set_error(DG_ENONFINITE, "bad initial state");
    s->ke0 = rec[0];
    {
        std::lock_guard<std::mutex> lk(S->mu);
        s->n_steps = (int64_t)std::ceil(s->req.t_end / dt0 - 1e-12);
        if (s->n_steps < 1) s->n_steps = 1;
        s->dt = s->req.t_end / s->n_steps;
    }
    s->pending_t.push_back(0.0);
    s->par = 0;
    s->steps = 0;
    return write_descs(s, W.st);
}

// sets up the admitted solves, with one wait for all of them, and moves those
// that can run to `run`
static void admit(solve_server* S, Worker& W, std::vector<Solve*>& admitted, std::vector<Solve*>& run) {
    if (admitted.empty()) return;
    std::vector<int> rc(admitted.size(), DG_OK);
    for (size_t i = 0; i < admitted.size(); ++i) rc[i] = admit_begin(S, W, admitted[i]);
    const bool back = hipStreamSynchronize(W.st) == hipSuccess;
    for (size_t i = 0; i < admitted.size(); ++i) {
        if (!rc[i] && !back) rc[i] = set_error(DG_EHIP, "admission synchronise failed");
        if (!rc[i]) rc[i] = admit_end(S, W, admitted[i]);
        if (rc[i]) fail(S, admitted[i], rc[i]);
        else run.push_back(admitted[i]);
    }
    admitted.clear();
}

// the stage descriptor of a solve that reads traces `par`
static void stage_desc(const Solve* s, int par, SolveDesc& d) {
    const WsLayout L = ws_layout(s->mesh);
    std::memset(&d, 0, sizeof(SolveDesc));
    d.q = s->q;
    d.k = s->k;
    d.qtr_in = (const double*)(s->ws + (par == 0 ? L.qtr0 : L.qtr1));
    d.qtr_out = (double*)(s->ws + (par == 0 ? L.qtr1 : L.qtr0));
    d.fv = (double*)(s->ws + L.fv);
    d.N = s->mesh.N;
    d.E = s->mesh.E;
    d.dt = s->dt;
    d.ph = s->mesh.ph;
}

// the four stage descriptors of a solve, with the correction while it is
// active: d[par] the stages, d[2 + par] the last stage of a step corrected
// after the step (Algorithm 1), whose update adds dt s(q^n)
static int write_descs(Solve* s, hipStream_t st) {
    const bool post = s->nn_active && s->req.nn_after_step;
    const double* fbuf = s->nn_active ? (const double*)(s->ws + ws_layout(s->mesh).forcing) : nullptr;
    SolveDesc d[4];
    for (int p = 0; p < 4; ++p) {
        stage_desc(s, p & 1, d[p]);
        d[p].forcing = post ? nullptr : fbuf;
        d[p].post = (post && p >= 2) ? fbuf : nullptr;
    }
    if (launch_write_descs(d, 4, s->ddesc, st) != hipSuccess) return set_error(DG_EHIP, "descriptor upload failed");
    return DG_OK;
}

// one Runge-Kutta step of solves of one order, stages batched, enqueued on the
// order's stream
static int step_group(int PP, std::vector<Solve*>& v, hipStream_t st) {
    for (Solve* s : v)
        if (s->inject) {
            static const double nan_val = std::nan("");
            if (hipMemcpyAsync(s->q, &nan_val, sizeof(double), hipMemcpyHostToDevice, st) != hipSuccess)
                return set_error(DG_EHIP, "inject failed");
            if (hipStreamSynchronize(st) != hipSuccess) return set_error(DG_EHIP, "inject sync failed");
            s->inject = false;
        }
    for (int stg = 0; stg < 3; ++stg) {
        for (size_t c0 = 0; c0 < v.size(); c0 += kMaxDescs) {
            const size_t cn = std::min((size_t)kMaxDescs, v.size() - c0);
            DescList dl;
            std::memset(&dl, 0, sizeof(dl));
            int blk = 0;
            for (size_t i = 0; i < cn; ++i) {
                Solve* s = v[c0 + i];
                const bool post = s->nn_active && s->req.nn_after_step;
                dl.d[i] = s->ddesc + s->par + ((post && stg == 2) ? 2 : 0);
                dl.blk[i] = blk;
                blk += s->mesh.E;
            }
            dl.blk[cn] = blk;
            dl.n = (int)cn;
            if (launch_grad(PP, dl, st) != hipSuccess) return set_error(DG_EHIP, "grad launch failed");
            // network forcing of the corrected solves, grouped by model
            std::map<const nn_model*, std::vector<NetTarget>> nets;
            for (size_t i = 0; i < cn; ++i) {
                Solve* s = v[c0 + i];
                if (!s->nn_active) continue;
                if (s->req.nn_after_step && stg != 0) continue;   // s(q^n) once, at the step start
                NetTarget t;
                t.q = s->q;
                t.out = (double*)(s->ws + ws_layout(s->mesh).forcing);
                t.E = s->mesh.E;
                t.blk_begin = 0;
                nets[s->req.model].push_back(t);
            }
            for (auto& nt : nets) {
                int rc = net_forcing_batch(nt.first, PP * PP * PP, nt.second.data(), (int)nt.second.size(), st);
                if (rc) return rc;
            }
            if (launch_resid(PP, dl, kRkA[stg], kRkB[stg], stg == 0, st) != hipSuccess)
                return set_error(DG_EHIP, "resid launch failed");
        }
        for (Solve* s : v) s->par ^= 1;
    }
    for (Solve* s : v) {
        s->steps.fetch_add(1);
        if (s->steps % s->req.ke_every == 0 || s->steps == s->n_steps) {
            if ((int)s->pending_t.size() >= kHist) continue;
            int rc = diag_impl(s->mesh, s->q, s->hist + kDiagDoubles * s->pending_t.size(), s->ws, st);
            if (rc) return rc;
            s->pending_t.push_back(s->steps * s->dt);
        }
    }
    return DG_OK;
}

// cost of one step of a solve, in node-stage units (the network adds about
// as much again at every stage, less when it corrects once per step)
static double step_cost(const Solve* s) {
    return (double)s->mesh.E * s->mesh.n_p * (s->nn_active ? (s->req.nn_after_step ? 1.3 : 2.0) : 1.0);
}

// Steps of one round for each running solve of an order: the costliest takes
// kChunk, and every solve gets about the same device time as that one: a solve
// whose steps cost a k-th as much takes k times the steps (up to kChunkMax),
// so that a small solve batched with large ones does not wait for as many of
// their steps as it needs of its own.  Never past a solve's last step or its
// KE-record capacity.
static std::vector<int64_t> round_plan(const std::vector<Solve*>& run) {
    double cbig = 0.0;
    for (Solve* s : run) cbig = std::max(cbig, step_cost(s));
    std::vector<int64_t> plan;
    for (Solve* s : run) {
        const double n = std::floor(kChunk * cbig / std::max(1.0, step_cost(s)));
        int64_t k = std::max<int64_t>((int64_t)std::min(n, (double)kChunkMax), 1);
        k = std::min<int64_t>(k, s->n_steps - s->steps);
        k = std::min<int64_t>(k, (int64_t)(kHist - 1 - (int)s->pending_t.size()) * s->req.ke_every);
        plan.push_back(std::max<int64_t>(k, 1));
    }
    return plan;
}

static bool record_finite(const double* rec) {
    bool finite = std::isfinite(rec[0]);
    for (int c = 3; c < 8; ++c) finite = finite && std::isfinite(rec[c]);
    return finite;
}

// a corrected solve's state is healthy: finite, kinetic energy not risen
static bool record_healthy(const Solve* s, const double* rec) {
    return record_finite(rec) && rec[0] <= s->ke0 * (1.0 + kFallbackKeRise);
}

// Takes over the round's kinetic-energy records (and, for a corrected solve,
// the end-of-round health record) that the round read back.  Returns true when
// a corrected solve must fall back: its pending records are then dropped,
// except those at or before the state copy it returns to.
static bool collect(solve_server* S, Solve* s) {
    const double* const records = s->records;
    const size_t n = s->pending_t.size();
    const bool check = s->nn_active;
    std::lock_guard<std::mutex> lk(S->mu);
    bool bad = check && !record_healthy(s, records + kHist * kDiagDoubles);
    for (size_t r = 0; r < n && check && !bad; ++r) bad = !record_healthy(s, records + r * kDiagDoubles);
    const double t_ckpt = s->ckpt_steps * s->dt;
    for (size_t r = 0; r < n; ++r) {
        const double* rec = records + r * kDiagDoubles;
        if (bad && s->pending_t[r] > t_ckpt + 0.5 * s->dt) continue;
        if (!bad && !record_finite(rec)) s->error = DG_ENONFINITE;
        s->ke.push_back(s->pending_t[r]);
        s->ke.push_back(rec[0]);
    }
    s->pending_t.clear();
    return bad;
}

// return a corrected solve to the state copy of the round start and continue
// it uncorrected from there
static int fall_back(solve_server* S, Worker& W, Solve* s) {
    s->nn_active = false;
    if (hipMemcpyAsync(s->q, s->ckpt, (size_t)5 * s->mesh.E * s->mesh.n_p * sizeof(double), hipMemcpyDeviceToDevice,
                       W.st) != hipSuccess)
        return set_error(DG_EHIP, "fallback restore failed");
    int rc = write_descs(s, W.st);
    if (rc) return rc;
    s->par = 0;
    SolveDesc d;
    stage_desc(s, 1, d);
    if (launch_traces(s->mesh.PP, d, W.st) != hipSuccess) return set_error(DG_EHIP, "trace launch failed");
    std::lock_guard<std::mutex> lk(S->mu);
    s->steps = s->ckpt_steps;
    s->fell_back = true;
    s->fallback_step = s->ckpt_steps;
    return DG_OK;
}

static hipError_t copy_and_wait(solve_server* S, char* dst, const char* src, size_t n) {
    const hipStream_t st = S->streams[DG_MAX_ORDER];
    const hipError_t e = hipMemcpyAsync(dst, src, n, hipMemcpyDeviceToHost, st);
    return e != hipSuccess ? e : hipStreamSynchronize(st);
}

// Device to pageable host memory, a chunk on its way to pinned memory while
// others go on from there, each in a thread of its own (new pages are what
// takes long: 15 MB in four threads 0.8 ms, in one 1.4).  On a stream of the
// server: a copy on the null stream waits for what the caller has there.
static hipError_t copy_out(solve_server* S, Worker& W, char* dst, const char* src, size_t bytes) {
    if (bytes > kStageChunk && !W.stage &&
        hipHostMalloc((void**)&W.stage, kStageSlots * kStageChunk, hipHostMallocDefault) != hipSuccess)
        W.stage = nullptr;
    if (bytes <= kStageChunk || !W.stage) return copy_and_wait(S, dst, src, bytes);
    std::future<void> going[kStageSlots];   // their destructors wait
    for (size_t at = 0, i = 0; at < bytes; at += kStageChunk, ++i) {
        const size_t slot = i % kStageSlots, n = std::min(kStageChunk, bytes - at);
        char* const piece = W.stage + slot * kStageChunk;
        if (going[slot].valid()) going[slot].wait();
        const hipError_t e = copy_and_wait(S, piece, src + at, n);
        if (e != hipSuccess) return e;
        const auto move = [=] { std::memcpy(dst + at, piece, n); };
        try {
            going[slot] = std::async(std::launch::async, move);
        } catch (const std::exception&) {
            move();
        }
    }
    return hipSuccess;
}

static void finish(solve_server* S, Worker& W, Solve* s) {
    if (s->req.q_out_host && copy_out(S, W, (char*)s->req.q_out_host, (const char*)s->q,
                                      (size_t)5 * s->mesh.E * s->mesh.n_p * sizeof(double)) != hipSuccess)
        return fail(S, s, set_error(DG_EHIP, "copy of the final state failed"));
    if (s->req.ke_host) {
        const size_t pairs = std::min((size_t)s->req.ke_capacity, s->ke.size() / 2);
        std::memcpy(s->req.ke_host, s->ke.data(), pairs * 2 * sizeof(double));
    }
    leave(S, s, SOLVE_DONE, s->error);
}

// copies out what an order has finished until nothing is left
static void deliver_all(solve_server* S, Worker& W) {
    (void)hipSetDevice(S->device);
    while (true) {
        Solve* s;
        {
            std::lock_guard<std::mutex> lk(S->mu);
            W.delivering = !W.done.empty();
            if (!W.delivering) return;
            s = W.done.front();
            W.done.pop_front();
        }
        finish(S, W, s);
    }
}

// Hands a finished solve to the thread that copies results out, started where
// none is at it: beside the next round's enqueueing, which may take as long as
// the round, and beside the round.
static void deliver(solve_server* S, Worker& W, Solve* s) {
    {
        std::lock_guard<std::mutex> lk(S->mu);
        W.done.push_back(s);
        if (W.delivering) return;
        W.delivering = true;
    }
    try {
        W.delivery = std::async(std::launch::async, deliver_all, S, std::ref(W));
    } catch (const std::exception&) {
        deliver_all(S, W);
    }
}

// enqueues one round of the running solves, up to the read-back of its records
static int enqueue_round(solve_server* S, Worker& W, const std::vector<Solve*>& run) {
    int rc = DG_OK;
    const std::vector<int64_t> plan = round_plan(run);
    const int64_t steps = *std::max_element(plan.begin(), plan.end());
    // corrected solves: copy of the (already checked) state the round starts from
    for (Solve* s : run)
        if (s->nn_active) {
            s->ckpt_steps = s->steps;
            if (hipMemcpyAsync(s->ckpt, s->q, (size_t)5 * s->mesh.E * s->mesh.n_p * sizeof(double),
                               hipMemcpyDeviceToDevice, W.st) != hipSuccess)
                return set_error(DG_EHIP, "state copy failed");
        }
    // step n batches every solve that still has steps in this round
    std::vector<Solve*> active;
    for (int64_t n = 0; n < steps; ++n) {
        active.clear();
        for (size_t i = 0; i < run.size(); ++i)
            if (plan[i] > n) active.push_back(run[i]);
        if ((rc = step_group(W.PP, active, W.st))) return rc;
    }
    for (size_t i = 0; i < run.size(); ++i) {
        Solve* s = run[i];
        double* const rec = s->records;
        if (s->nn_active && (rc = diag_impl(s->mesh, s->q, s->health, s->ws, W.st))) return rc;
        if ((!s->pending_t.empty() &&
             hipMemcpyAsync(rec, s->hist, s->pending_t.size() * kDiagDoubles * sizeof(double), hipMemcpyDeviceToHost,
                            W.st) != hipSuccess) ||
            (s->nn_active && hipMemcpyAsync(rec + kHist * kDiagDoubles, s->health, kDiagDoubles * sizeof(double),
                                            hipMemcpyDeviceToHost, W.st) != hipSuccess))
            return set_error(DG_EHIP, "record readback failed");
    }
    std::lock_guard<std::mutex> lk(S->mu);
    S->batches += steps;
    return DG_OK;
}

static void mark_round(solve_server* S, bool begin) {
    std::lock_guard<std::mutex> lk(S->mu);
    const double t = now_s();
    if (begin && S->in_round++ == 0) S->round_t0 = t;
    if (!begin && --S->in_round == 0) S->busy += t - S->round_t0;
}

static void worker_loop(solve_server* S, Worker& W) {
    int broken = DG_OK;
    if (hipSetDevice(S->device) != hipSuccess) broken = set_error(DG_EHIP, "hipSetDevice failed");
    std::vector<Solve*> admitted, run, keep;
    while (true) {
        {
            std::unique_lock<std::mutex> lk(S->mu);
            S->cv.wait(lk, [&] { return S->stop || !W.inbox.empty() || !run.empty(); });
            if (S->stop) break;
            admitted.swap(W.inbox);
        }
        if (broken) {
            for (Solve* s : admitted) fail(S, s, broken);
            admitted.clear();
        }
        admit(S, W, admitted, run);
        if (run.empty()) continue;
        mark_round(S, true);
        int rc = enqueue_round(S, W, run);
        const bool synced = hipStreamSynchronize(W.st) == hipSuccess;
        mark_round(S, false);
        if (!synced && rc == DG_OK) rc = set_error(DG_EHIP, "round synchronise failed");
        keep.clear();
        for (size_t i = 0; i < run.size(); ++i) {
            Solve* s = run[i];
            int err = rc;
            if (err == DG_OK) {
                if (collect(S, s)) {
                    err = fall_back(S, W, s);
                    // what it enqueued before it failed still writes to the block
                    if (err) (void)hipStreamSynchronize(W.st);
                } else {
                    std::lock_guard<std::mutex> lk(S->mu);
                    err = s->error;
                }
            }
            if (err) fail(S, s, err);
            else if (s->steps >= s->n_steps) deliver(S, W, s);
            else keep.push_back(s);
        }
        run.swap(keep);
    }
    (void)hipStreamSynchronize(W.st);
    if (W.delivery.valid()) W.delivery.wait();
    if (W.stage) (void)hipHostFree(W.stage);
}

}  // namespace dgnn

// frees a server whose threads have ended, or were not started
static void destroy(solve_server* S) {
    for (hipStream_t st : S->streams)
        if (st) (void)hipStreamDestroy(st);
    if (S->records) (void)hipHostFree(S->records);
    delete S;
}

extern "C" {

size_t solve_footprint(int32_t P, int32_t N, int32_t use_nn) {
    if (P < DG_MIN_ORDER || P > DG_MAX_ORDER || N < 1 || N > 1024) return 0;
    Mesh m;
    std::memset(&m, 0, sizeof(m));
    m.N = N;
    m.P = P;
    m.PP = P + 1;
    m.E = N * N * N;
    m.n_p = m.PP * m.PP * m.PP;
    m.n_f = m.PP * m.PP;
    return foot(m, use_nn != 0).total;
}

int solve_server_create(void* arena, size_t arena_bytes, int32_t max_slots, solve_server** out) {
    if (!out) return set_error(DG_EINVAL, "null output handle");
    *out = nullptr;
    if (!arena || (((uintptr_t)arena) & 255)) return set_error(DG_EINVAL, "arena must be non-null and 256-byte aligned");
    if (max_slots < 1 || max_slots > 4096) return set_error(DG_EINVAL, "max_slots outside [1, 4096]");
    solve_server* S = new solve_server;
    S->base = (char*)arena;
    S->bytes = arena_bytes & ~(size_t)255;
    S->max_slots = max_slots;
    S->arena.reset(S->bytes);
    for (int i = max_slots; i-- > 0;) S->free_slots.push_back(i);
    if (hipGetDevice(&S->device) != hipSuccess) {
        destroy(S);
        return set_error(DG_EHIP, "hipGetDevice failed");
    }
    for (hipStream_t& st : S->streams)
        if (hipStreamCreateWithFlags(&st, hipStreamNonBlocking) != hipSuccess) {
            st = nullptr;
            destroy(S);
            return set_error(DG_EHIP, "stream creation failed");
        }
    if (hipHostMalloc((void**)&S->records, max_slots * kRecords * sizeof(double), hipHostMallocDefault) != hipSuccess) {
        S->records = nullptr;
        destroy(S);
        return set_error(DG_EHIP, "pinned buffer allocation failed");
    }
    for (int pp = 0; pp <= kMaxPP; ++pp) S->workers[pp].PP = pp;
    *out = S;
    return DG_OK;
}

int solve_submit(solve_server* S, const solve_request* r, uint64_t* id) {
    if (!S || !r || !id) return set_error(DG_EINVAL, "null argument");
    if (!(r->Re > 0) || !(r->t_end > 0) || !std::isfinite(r->t_end) || r->ke_every < 1 || r->Cs < 0)
        return set_error(DG_EINVAL, "invalid request parameters");
    if (r->ke_host && r->ke_capacity < 0) return set_error(DG_EINVAL, "negative KE capacity");
    if (r->nn_after_step != 0 && r->nn_after_step != 1) return set_error(DG_EINVAL, "nn_after_step must be 0 or 1");
    Mesh m;
    dg_params p = request_params(*r);
    int rc = make_mesh(&p, m);
    if (rc) return rc;
    if (r->use_nn) {
        if (!r->model) return set_error(DG_EINVAL, "use_nn without a model");
        if ((rc = net_check_mesh(r->model, m))) return rc;
    }
    const size_t need = foot(m, r->use_nn != 0).total;
    if (need > S->bytes) return set_error(DG_ENOSPC, "request needs %zu bytes, arena holds %zu", need, S->bytes);
    auto s = std::make_unique<Solve>();
    s->req = *r;
    s->mesh = m;
    s->bytes = need;
    s->t_submit = now_s();
    {
        std::lock_guard<std::mutex> lk(S->mu);
        if (S->stop) return set_error(DG_EINVAL, "server is shutting down");
        Worker& W = S->workers[m.PP];
        if (!W.th.joinable()) {
            if (!W.st) W.st = S->streams[S->streams_used++];
            try {
                W.th = std::thread(worker_loop, S, std::ref(W));
            } catch (const std::exception&) {
                return set_error(DG_EHIP, "thread creation failed");
            }
        }
        s->id = S->next_id++;
        *id = s->id;
        S->queue.push_back(s.get());
        S->solves[s->id] = std::move(s);
        admit_waiting(S);
    }
    S->cv.notify_all();
    return DG_OK;
}

int solve_poll(solve_server* S, uint64_t id, solve_status* st) {
    if (!S || !st) return set_error(DG_EINVAL, "null argument");
    std::lock_guard<std::mutex> lk(S->mu);
    auto it = S->solves.find(id);
    if (it == S->solves.end()) return set_error(DG_ENOENT, "unknown request %llu", (unsigned long long)id);
    const Solve* s = it->second.get();
    std::memset(st, 0, sizeof(*st));
    st->state = s->state;
    st->error = s->error;
    st->steps = s->steps;
    st->n_steps = s->n_steps;
    st->ke_count = (int32_t)std::min((size_t)std::max(0, s->req.ke_capacity), s->ke.size() / 2);
    st->fallback = s->fell_back ? 1 : 0;
    st->fallback_step = s->fell_back ? s->fallback_step : -1;
    st->t = s->steps * s->dt;
    st->dt = s->dt;
    st->queue_s = s->state == SOLVE_QUEUED ? 0.0 : s->t_admit - s->t_submit;
    st->latency_s = (s->state == SOLVE_DONE || s->state == SOLVE_FAILED) ? s->t_done - s->t_submit : 0.0;
    st->dof_updates = (int64_t)3 * s->steps * s->mesh.E * s->mesh.n_p;
    return (s->state == SOLVE_DONE || s->state == SOLVE_FAILED) ? DG_OK : DG_EAGAIN;
}

int solve_server_drain(solve_server* S) {
    if (!S) return set_error(DG_EINVAL, "null server");
    std::unique_lock<std::mutex> lk(S->mu);
    S->cv.wait(lk, [&] {
        if (!S->queue.empty()) return false;
        for (auto& kv : S->solves)
            if (kv.second->state == SOLVE_RUNNING) return false;
        return true;
    });
    return DG_OK;
}

int solve_inject_nan(solve_server* S, uint64_t id) {
    if (!S) return set_error(DG_EINVAL, "null server");
    std::lock_guard<std::mutex> lk(S->mu);
    auto it = S->solves.find(id);
    if (it == S->solves.end()) return set_error(DG_ENOENT, "unknown request");
    it->second->inject = true;
    return DG_OK;
}

int solve_server_stats(solve_server* S, double* busy_s, int64_t* batches) {
    if (!S) return set_error(DG_EINVAL, "null server");
    std::lock_guard<std::mutex> lk(S->mu);
    if (busy_s) *busy_s = S->busy + (S->in_round > 0 ? now_s() - S->round_t0 : 0.0);
    if (batches) *batches = S->batches;
    return DG_OK;
}

void solve_server_free(solve_server* S) {
    if (!S) return;
    {
        std::lock_guard<std::mutex> lk(S->mu);
        S->stop = true;
    }
    S->cv.notify_all();
    for (Worker& W : S->workers)
        if (W.th.joinable()) W.th.join();
    destroy(S);
}

}  // extern "C"
