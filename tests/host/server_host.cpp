// The solve server (csrc/server.cpp) on the host alone: the HIP runtime and
// the launches it calls are replaced here, device memory is host memory, and
// every launch and copy is done, or failed, at once.  Each scenario forces one
// condition that a healthy GPU does not show, prints what went wrong and ends
// with the number of complaints.
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <mutex>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "nn_internal.hpp"

using namespace dgnn;

// ------------------------------------------------------------ HIP runtime

struct ihipStream_t {
    std::atomic<int> pending{0};   // operations since the last synchronisation
    std::atomic<int> syncs{0};
};

namespace {

std::mutex g_mu;
int g_bad = 0;
std::set<void*> g_streams, g_pinned;
std::atomic<int> g_null_copies{0};
std::function<bool()> g_fail_stream, g_fail_pinned, g_fail_descs;
std::function<bool(const void*, size_t)> g_fail_to_host;
std::function<void(hipStream_t, const DescList&)> g_on_grad;
std::function<void(hipStream_t, const double*)> g_on_init;
std::function<double(const double*)> g_energy;

void complain(const char* fmt, ...) {
    std::lock_guard<std::mutex> lk(g_mu);
    va_list ap;
    va_start(ap, fmt);
    std::vprintf(fmt, ap);
    va_end(ap);
    std::printf("\n");
    ++g_bad;
}

hipError_t launched(hipStream_t st) {
    if (!st) complain("a launch on the null stream");
    else ++st->pending;
    return hipSuccess;
}

}  // namespace

extern "C" {

hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }

hipError_t hipStreamCreateWithFlags(hipStream_t* st, unsigned) {
    if (g_fail_stream && g_fail_stream()) return hipErrorOutOfMemory;
    *st = new ihipStream_t;
    std::lock_guard<std::mutex> lk(g_mu);
    g_streams.insert(*st);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t st) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_streams.erase(st);   // kept: a scenario may still look at it
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t st) {
    st->pending = 0;
    ++st->syncs;
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    if (g_fail_pinned && g_fail_pinned()) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    std::lock_guard<std::mutex> lk(g_mu);
    g_pinned.insert(*p);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {
    {
        std::lock_guard<std::mutex> lk(g_mu);
        g_pinned.erase(p);
    }
    std::free(p);
    return hipSuccess;
}

static hipError_t copy(void* dst, const void* src, size_t n, hipMemcpyKind kind) {
    if (kind == hipMemcpyDeviceToHost && g_fail_to_host && g_fail_to_host(src, n)) return hipErrorInvalidValue;
    std::memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void* dst, const void* src, size_t n, hipMemcpyKind kind) {
    ++g_null_copies;
    return copy(dst, src, n, kind);
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind kind, hipStream_t st) {
    if (!st) ++g_null_copies;
    else ++st->pending;
    return copy(dst, src, n, kind);
}

}  // extern "C"

// ------------------------------------------------- what the server launches

namespace dgnn {

const double kRkA[3] = {0, 0, 0}, kRkB[3] = {1, 1, 1};

int set_error(int code, const char*, ...) { return code; }

WsLayout ws_layout(const Mesh&) {
    WsLayout L;
    L.qtr0 = 0;
    L.qtr1 = 256;
    L.fv = 512;
    L.forcing = 768;
    L.partial = 1024;
    L.total = 1280;
    return L;
}

int make_mesh(const dg_params* p, Mesh& M) {
    std::memset(&M, 0, sizeof(M));
    M.prm = *p;
    M.N = p->N;
    M.P = p->P;
    M.PP = p->P + 1;
    M.E = p->N * p->N * p->N;
    M.n_p = M.PP * M.PP * M.PP;
    M.n_f = M.PP * M.PP;
    return DG_OK;
}

int init_tgv_impl(const Mesh& m, double* q, hipStream_t st) {
    launched(st);
    if (g_on_init) g_on_init(st, q);
    for (size_t i = 0; i < (size_t)5 * m.E * m.n_p; ++i) q[i] = 1.0 + i;
    return DG_OK;
}

int diag_impl(const Mesh&, const double* q, double* out, char*, hipStream_t st) {
    launched(st);
    for (int c = 0; c < 8; ++c) out[c] = 1.0;
    if (g_energy) out[0] = g_energy(q);
    return DG_OK;
}

double stable_dt_from_diag(const Mesh&, const double*, double) { return 0.1; }

hipError_t launch_traces(int, const SolveDesc&, hipStream_t st) { return launched(st); }
hipError_t launch_write_descs(const SolveDesc* host, int n, SolveDesc* dev, hipStream_t st) {
    if (g_fail_descs && g_fail_descs()) return hipErrorInvalidValue;
    std::memcpy(dev, host, n * sizeof(SolveDesc));
    return launched(st);
}
hipError_t launch_grad(int, const DescList& dl, hipStream_t st) {
    if (g_on_grad) g_on_grad(st, dl);
    return launched(st);
}
hipError_t launch_resid(int, const DescList&, double, double, int, hipStream_t st) { return launched(st); }

int net_check_mesh(const nn_model*, const Mesh&) { return DG_OK; }
int net_forcing_batch(const nn_model*, int, const NetTarget*, int, hipStream_t st) {
    launched(st);
    return DG_OK;
}

}  // namespace dgnn

// ------------------------------------------------------------------ scenarios

namespace {

constexpr size_t kArena = (size_t)512 << 20;

struct Server {
    char* arena;
    solve_server* s = nullptr;
    explicit Server(int slots, size_t bytes = kArena) : arena((char*)std::aligned_alloc(256, bytes)) {
        if (solve_server_create(arena, bytes, slots, &s) != DG_OK) complain("the server was not created");
    }
    ~Server() {
        solve_server_free(s);
        std::free(arena);
        std::lock_guard<std::mutex> lk(g_mu);
        if (!g_streams.empty() || !g_pinned.empty()) {
            std::printf("%zu streams, %zu pinned buffers left\n", g_streams.size(), g_pinned.size());
            ++g_bad;
        }
    }
};

struct Request {
    solve_request r;
    std::vector<double> q;
    uint64_t id = 0;
    // steps of 0.1
    Request(int P, int N, int steps) : q((size_t)5 * N * N * N * (P + 1) * (P + 1) * (P + 1)) {
        std::memset(&r, 0, sizeof(r));
        r.Re = 100;
        r.t_end = 0.1 * steps;
        r.P = P;
        r.N = N;
        r.ke_every = 1;
        r.q_out_host = q.data();
    }
    void submit(Server& S) {
        if (solve_submit(S.s, &r, &id) != DG_OK) complain("request refused");
    }
    solve_status status(Server& S) const {
        solve_status st;
        solve_poll(S.s, id, &st);
        return st;
    }
    bool whole() const {
        for (size_t i = 0; i < q.size(); ++i)
            if (q[i] != 1.0 + i) return false;
        return true;
    }
    void expect_done(Server& S, const char* what) const {
        const solve_status st = status(S);
        if (st.state != SOLVE_DONE || st.error || !whole())
            complain("%s: state %d, error %d, result %s", what, st.state, st.error, whole() ? "whole" : "not whole");
    }
};

bool within_seconds(double s, const std::function<bool()>& f) {
    for (int i = 0; i < 200; ++i) {
        if (f()) return true;
        std::this_thread::sleep_for(std::chrono::duration<double>(s / 200));
    }
    return f();
}

// sizes of a result: one copy, and several pieces (20 MB)
constexpr int kSmallN = 4, kLargeN = 40;

// records are at most this large, results larger
constexpr size_t kRecordBytes = 8192;

// the n-th copy of a finished state fails
void copy_error(int N, int nth) {
    std::atomic<int> seen{0};
    g_fail_to_host = [&](const void*, size_t n) { return n > kRecordBytes && seen++ == nth; };
    Server S(1);
    Request a(1, N, 3), b(1, N, 3);
    a.submit(S);
    b.submit(S);
    solve_server_drain(S.s);
    const solve_status st = a.status(S);
    if (seen <= nth) complain("the copy that fails was not made");
    if (st.state != SOLVE_FAILED || st.error != DG_EHIP)
        complain("copy failed: state %d, error %d", st.state, st.error);
    b.expect_done(S, "the next request");
}

// What the solves need is there once the server is made, or it is not made:
// every stream and pinned buffer of its creation fails in turn, then all of
// them after it.
void create_errors() {
    std::atomic<int> calls{0};
    int fail_at = 0;
    const auto nth = [&] { return calls++ == fail_at; };
    g_fail_stream = g_fail_pinned = nth;
    for (;; ++fail_at) {
        calls = 0;
        char* arena = (char*)std::aligned_alloc(256, 4096);
        solve_server* s = (solve_server*)arena;
        const int rc = solve_server_create(arena, 4096, 40, &s);
        const bool failed = calls > fail_at;
        if (failed && (rc != DG_EHIP || s)) complain("creation %d failed: code %d", fail_at, rc);
        if (!failed && rc != DG_OK) complain("created without a failure: code %d", rc);
        if (s) solve_server_free(s);
        std::free(arena);
        if (!g_streams.empty() || !g_pinned.empty()) complain("creation %d failed: something left", fail_at);
        if (!failed) break;
    }
    if (fail_at == 0) complain("nothing is made with the server");
    g_fail_stream = g_fail_pinned = nullptr;
    Server S(40);
    g_fail_stream = g_fail_pinned = [] { return true; };
    std::vector<Request> r;
    for (int i = 0; i < 40; ++i) r.emplace_back(1 + i % 2, 2 + i % 3, 3 + i);
    r.emplace_back(3, 16, 3);   // a result of several pieces
    for (int P = 4; P <= DG_MAX_ORDER; ++P) r.emplace_back(P, 2, 3);
    for (Request& x : r) x.submit(S);
    solve_server_drain(S.s);
    for (Request& x : r) x.expect_done(S, "without further streams and buffers");
}

// no copy on the null stream, where it would wait for the caller's work
void null_stream() {
    Server S(4);
    Request a(1, kSmallN, 3), b(2, kSmallN, 3), c(1, kLargeN, 2);
    for (Request* r : {&a, &b, &c}) r->submit(S);
    solve_server_drain(S.s);
    for (Request* r : {&a, &b, &c}) r->expect_done(S, "request");
    if (g_null_copies) complain("%d copies on the null stream", g_null_copies.load());
}

// A solve that ends while another of its order goes on is delivered, and its
// slot given to the next request, without waiting for the other's next round:
// the first launch of that round is held until both happened.
void delivery(int N) {
    Server S(2);
    Request a(1, N, 20), b(1, N, 100), next(2, 1, 1);
    std::atomic<bool> submitted{false}, late{false}, held{false};
    std::atomic<int> ended_at{-1};
    g_on_grad = [&](hipStream_t st, const DescList& dl) {
        within_seconds(5, [&] { return submitted.load(); });
        if (dl.n != 1 || held || a.status(S).steps < 20) return;
        int none = -1;
        if (ended_at.compare_exchange_strong(none, st->syncs)) return;   // in the round that ends it
        if (st->syncs == ended_at) return;
        held = true;
        late = !within_seconds(5, [&] {
            return a.status(S).state == SOLVE_DONE && next.status(S).state != SOLVE_QUEUED;
        });
    };
    a.submit(S);
    b.submit(S);
    next.submit(S);
    submitted = true;
    solve_server_drain(S.s);
    g_on_grad = nullptr;
    for (Request* r : {&a, &b, &next}) r->expect_done(S, "request");
    if (!held) complain("no launch after the round in which the first solve ended");
    if (late) complain("the next round began before the finished solve was delivered");
}

// A corrected solve has to fall back, and that fails half-way, with the copy of
// its state already enqueued: its block goes to another order's solve only
// when nothing is pending that writes to it.
void fallback_error() {
    nn_model model;
    Request a(1, kSmallN, 40), b(2, kSmallN, 3);
    a.r.use_nn = 1;
    a.r.model = &model;
    Server S(2, solve_footprint(2, kSmallN, 0));   // one at a time
    std::atomic<hipStream_t> failing{nullptr};
    std::atomic<int> energies{0}, pending{-1};
    g_energy = [&](const double*) { return energies++ ? NAN : 1.0; };
    g_fail_descs = [&] { return energies > 1; };
    g_on_grad = [&](hipStream_t st, const DescList&) { failing = st; };
    g_on_init = [&](hipStream_t st, const double*) {
        if (!failing) return;
        pending = failing.load()->pending.load();
        g_energy = nullptr;   // of the next solve: healthy
        g_fail_descs = nullptr;
        g_on_grad = nullptr;
    };
    a.submit(S);
    b.submit(S);
    solve_server_drain(S.s);
    const solve_status st = a.status(S);
    if (st.state != SOLVE_FAILED || st.error != DG_EHIP) complain("the solve: state %d, error %d", st.state, st.error);
    if (pending < 0) complain("the next solve was not set up");
    if (pending > 0) complain("%d operations pending on a block that was given away", pending.load());
    b.expect_done(S, "the next solve");
}

// requests that are polled from another thread from their submission on
void polling() {
    Server S(3);
    std::vector<Request> r;
    for (int i = 0; i < 12; ++i) r.emplace_back(1 + i % 3, 2, 40);
    for (Request& x : r) {
        x.submit(S);
        for (int n = 0; n < 200; ++n) x.status(S);
    }
    while (true) {
        int done = 0;
        for (Request& x : r) done += x.status(S).state == SOLVE_DONE;
        if (done == (int)r.size()) break;
    }
    for (Request& x : r) x.expect_done(S, "request");
}

int run(const std::string& what) {
    if (what == "copy_error_small") copy_error(kSmallN, 0);
    else if (what == "copy_error_large") copy_error(kLargeN, 2);
    else if (what == "create_errors") create_errors();
    else if (what == "null_stream") null_stream();
    else if (what == "delivery_small") delivery(kSmallN);
    else if (what == "delivery_large") delivery(kLargeN);
    else if (what == "fallback_error") fallback_error();
    else if (what == "polling") polling();
    else complain("no scenario %s", what.c_str());
    return g_bad;
}

}  // namespace

int main(int argc, char** argv) {
    const int bad = run(argc > 1 ? argv[1] : "");
    std::printf("%d complaints\n", bad);
    return bad ? 1 : 0;
}
