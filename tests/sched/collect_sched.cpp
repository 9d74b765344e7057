// Host-only tests of the serving scheduler's collect threads
// (paper_1502_00355_amd/csrc/sl_sched.h): results that take long to fetch hold
// up no step, each is fetched once, and failures and stops in between leave
// nothing behind.  Each scenario prints "ok <name>" or "FAIL <name>: <why>";
// the exit status is the failure count.
#include <cstdio>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "../../paper_1502_00355_amd/csrc/sl_sched.h"

namespace {
thread_local std::string g_err;
}
namespace sl {
void set_error(const std::string& msg) { g_err = msg; }
sl_status fail(sl_status st, const std::string& msg)
{
    g_err = msg;
    return st;
}
}  // namespace sl
extern "C" const char* sl_last_error(void) { return g_err.c_str(); }

namespace {

using sl::sched::StepOutcome;

struct Payload {
    int32_t sweeps = 0;
};

struct Mock {
    using Payload = ::Payload;
    using Req = sl::sched::Request<Payload>;
    int step_us = 1000, collect_us = 40000, fail_step_at = -1;
    std::set<uint64_t> fail_collect;
    std::mutex mu;
    std::set<uint64_t> held, collected;
    int collecting = 0, max_collecting = 0, steps = 0;
    int32_t sweeps = 0;
    std::string bad;

    size_t footprint(const sl_mesh_desc&) { return 1; }
    sl_status admit(Req& q)
    {
        std::lock_guard<std::mutex> lk(mu);
        held.insert(q.id);
        return SL_OK;
    }
    sl_status launch(const std::vector<Req*>& in, bool, int32_t k)
    {
        sweeps = k;
        std::lock_guard<std::mutex> lk(mu);
        for (Req* q : in) {
            q->joined = true;
            if (collected.count(q->id) || q->finishing) bad = "a finished request stepped";
        }
        return SL_OK;
    }
    sl_status wait(const std::vector<Req*>& in, std::vector<StepOutcome>& out)
    {
        std::this_thread::sleep_for(std::chrono::microseconds(step_us));
        if (steps++ == fail_step_at) return sl::fail(SL_EDEVICE, "mock: step failed");
        for (size_t k = 0; k < in.size(); ++k) {
            int32_t& s = in[k]->x.sweeps;
            s = std::min(in[k]->iterations, s + sweeps);
            out[k] = StepOutcome{s < in[k]->iterations, s, s};
        }
        return SL_OK;
    }
    sl_status collect(Req& q, const StepOutcome& o)
    {
        {
            std::lock_guard<std::mutex> lk(mu);
            max_collecting = std::max(max_collecting, ++collecting);
            if (!held.count(q.id)) bad = "collected after its release";
            if (!collected.insert(q.id).second) bad = "collected twice";
        }
        std::this_thread::sleep_for(std::chrono::microseconds(collect_us));
        std::lock_guard<std::mutex> lk(mu);
        --collecting;
        if (fail_collect.count(q.id)) return sl::fail(SL_EDEVICE, "mock: no result");
        for (auto& v : q.result) v = static_cast<double>(q.id);
        q.report.iterations_run = o.sweeps;
        return SL_OK;
    }
    void release(Req& q)
    {
        std::lock_guard<std::mutex> lk(mu);
        held.erase(q.id);
    }
};

struct Run {
    Mock ex;
    sl_server_config cfg{};
    std::unique_ptr<sl::sched::Scheduler<Mock>> core;
    double data[2] = {0, 0};
    Run()
    {
        cfg.hbm_budget_bytes = 1000;
        cfg.max_active = 64;
        cfg.sweeps_per_step = 4;
        cfg.setup_threads = 2;
    }
    void start()
    {
        core = std::make_unique<sl::sched::Scheduler<Mock>>(cfg, ex);
        core->start();
    }
    uint64_t submit(int32_t iters)
    {
        sl_mesh_desc d{};
        d.n_nodes = 3;
        d.coords = data;
        uint64_t id = 0;
        core->submit(d, iters, 0.0, 0.0, &id);
        return id;
    }
    // SL_EBUSY: not done after ten seconds
    sl_status wait(uint64_t id, sl_report* rep, sl_request_times* t, std::vector<double>* x)
    {
        x->assign(6, -1.0);
        for (int k = 0; k < 50000; ++k) {
            const sl_status st = core->poll(id, x->data(), rep, t);
            if (st != SL_EBUSY) return st;
            std::this_thread::sleep_for(std::chrono::microseconds(200));
        }
        return SL_EBUSY;
    }
};

int failures = 0;
void verdict(const char* name, const std::string& why)
{
    if (why.empty()) std::printf("ok %s\n", name);
    else std::printf("FAIL %s: %s\n", name, why.c_str());
    failures += why.empty() ? 0 : 1;
    std::fflush(stdout);
}

void slow_results_hold_up_no_step()
{
    Run r;
    r.start();
    const uint64_t big = r.submit(400);   // 100 steps of 1 ms
    std::vector<uint64_t> small;
    for (int k = 0; k < 30; ++k) small.push_back(r.submit(4));   // 30 results of 40 ms
    sl_report rep{};
    sl_request_times t{};
    std::vector<double> x;
    std::string why;
    const sl_status st = r.wait(big, &rep, &t, &x);
    // done by way of the collect threads' queue: behind at most 15 results each
    if (st != SL_OK || rep.iterations_run != 400) why = "the long request failed";
    else if (t.done_s - t.started_s > 0.9) why = "100 steps took " + std::to_string(t.done_s - t.started_s) + " s";
    for (uint64_t id : small) {
        if (r.wait(id, &rep, &t, &x) != SL_OK) why = "a short request failed";
        for (double v : x)
            if (v != static_cast<double>(id)) why = "a result is not its own";
    }
    r.core->stop();
    if (r.ex.max_collecting > sl::sched::kCollectThreads) why = "too many collected at once";
    if (!r.ex.bad.empty()) why = r.ex.bad;
    if (!r.ex.held.empty()) why = "requests not released";
    verdict("slow_results_hold_up_no_step", why);
}

void failed_results()
{
    Run r;
    r.ex.collect_us = 2000;
    r.ex.fail_collect = {2, 5};
    r.start();
    std::vector<uint64_t> ids;
    for (int k = 0; k < 8; ++k) ids.push_back(r.submit(4 + k));
    std::string why;
    for (uint64_t id : ids) {
        sl_report rep{};
        sl_request_times t{};
        std::vector<double> x;
        const sl_status st = r.wait(id, &rep, &t, &x);
        if (st != (r.ex.fail_collect.count(id) ? SL_EDEVICE : SL_OK)) why = "status " + std::to_string(st);
    }
    r.core->stop();
    if (!r.ex.held.empty()) why = "requests not released";
    verdict("failed_results", why);
}

void stop_with_results_waiting()
{
    Run r;
    r.start();
    std::vector<uint64_t> ids;
    for (int k = 0; k < 40; ++k) ids.push_back(r.submit(4));
    std::this_thread::sleep_for(std::chrono::milliseconds(60));
    r.core->stop();
    std::string why = r.ex.bad;
    if (!r.ex.held.empty()) why = "requests not released";
    verdict("stop_with_results_waiting", why);
}

void failed_step_with_results_waiting()
{
    Run r;
    r.ex.fail_step_at = 20;
    r.start();
    std::vector<uint64_t> small, big;
    for (int k = 0; k < 6; ++k) small.push_back(r.submit(4));
    for (int k = 0; k < 3; ++k) big.push_back(r.submit(4000));
    std::string why;
    sl_report rep{};
    sl_request_times t{};
    std::vector<double> x;
    for (uint64_t id : small)
        if (r.wait(id, &rep, &t, &x) != SL_OK) why = "a finished request lost its result";
    for (uint64_t id : big)
        if (r.wait(id, &rep, &t, &x) != SL_EDEVICE) why = "a request outlived the failed step";
    r.core->stop();
    if (!r.ex.held.empty()) why = "requests not released";
    if (!r.ex.bad.empty()) why = r.ex.bad;
    verdict("failed_step_with_results_waiting", why);
}

}  // namespace

int main()
{
    slow_results_hold_up_no_step();
    failed_results();
    stop_with_results_waiting();
    failed_step_with_results_waiting();
    std::printf("%d failure(s)\n", failures);
    return failures;
}
