// Solves of several independent problems (uneven grids) in one call: a few
// lanes, each a stream and a host thread, take the problems largest first, so
// that small problems' launches fill the GPU beside each other's and beside a
// large one's.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <memory>
#include <string>
#include <system_error>
#include <thread>
#include <utility>
#include <vector>

#include "cp_internal.h"

namespace cp {

namespace {

// Lanes of a device.  More do not help (streams share a few hardware queues,
// and one large problem fills the GPU by itself) and cost: six problems of
// 175 x 128 x 377 took 7.7 ms with six lanes, 5.9 ms one after another.
constexpr int kLanes = 3;

// A pass alone is cut into enough chunks to fill the GPU, at the price of rows
// computed twice; beside others it is cut into half as many (six uneven
// problems: 2.56 ms without, 2.37 with, 2.47 at a third or a quarter), but for
// the pass that leaves the norms, whose sums stay those of a solve alone (2.40).
constexpr int kShare = 2;

// One device's problems, in the order they are taken, and its lanes' streams.
// The streams are kept by the device's first plan (a stream made and destroyed
// for each problem of each call took 130 us a problem).
struct Queue {
    std::vector<int> order;
    std::atomic<int> next{0};
    cylpoisson_plan* keeper = nullptr;
    int lanes = 0;
    std::vector<int> taken[kLanes];  // the problems each lane took, written by that lane alone
};

hipError_t ensure_lanes(cylpoisson_plan* p, int lanes) {
    int prev = 0;
    (void)hipGetDevice(&prev);
    (void)hipSetDevice(p->device);
    hipError_t e = hipSuccess;
    while ((int)p->lanes.size() < lanes && e == hipSuccess) {
        hipStream_t st;
        e = hipStreamCreateWithFlags(&st, hipStreamNonBlocking);
        if (e == hipSuccess) p->lanes.push_back(st);
    }
    (void)hipSetDevice(prev);
    return e;
}

// Each solve runs exactly as alone.
int solve_lanes(cylpoisson_plan* const* plans, const double* const* rho, double* const* phi, int count,
                double tol, hipStream_t s, int* statuses) {
    std::vector<int> res(count, CYLPOISSON_OK);
    std::vector<std::string> msg(count);
    hipEvent_t start = nullptr;
    int status = CYLPOISSON_OK;
    if (hipEventCreateWithFlags(&start, hipEventDisableTiming) != hipSuccess ||
        hipEventRecord(start, s) != hipSuccess) {
        (void)hipGetLastError();
        set_error("batch: cannot order the problems after the caller's stream");
        if (start) (void)hipEventDestroy(start);
        return CYLPOISSON_EHIP;
    }
    std::vector<std::unique_ptr<Queue>> queues;
    for (int i = 0; i < count; ++i) {
        Queue* q = nullptr;
        for (const auto& c : queues)
            if (c->keeper->device == plans[i]->device) q = c.get();
        if (!q) {
            queues.push_back(std::make_unique<Queue>());
            q = queues.back().get();
            q->keeper = plans[i];
        }
        q->order.push_back(i);
    }
    auto nodes = [&](int i) { return (long long)plans[i]->nr * plans[i]->nt * plans[i]->nz; };
    for (const auto& q : queues) {
        std::stable_sort(q->order.begin(), q->order.end(), [&](int a, int b) { return nodes(a) > nodes(b); });
        q->lanes = std::min(kLanes, (int)q->order.size());
        for (int l = 0; l < q->lanes; ++l) q->taken[l].reserve(q->order.size());
        bool ok = ensure_lanes(q->keeper, q->lanes) == hipSuccess;
        for (int l = 0; l < q->lanes && ok; ++l) ok = hipStreamWaitEvent(q->keeper->lanes[l], start, 0) == hipSuccess;
        if (!ok && status == CYLPOISSON_OK) {
            (void)hipGetLastError();
            set_error("batch: cannot create the streams of problem %d", q->order.front());
            status = CYLPOISSON_EHIP;
        }
    }
    if (status == CYLPOISSON_OK) {
        auto lane = [&](Queue* q, int l) {
            hipStream_t st = q->keeper->lanes[l];
            for (int k; (k = q->next.fetch_add(1)) < (int)q->order.size();) {
                const int i = q->order[k];
                q->taken[l].push_back(i);
                res[i] = cylpoisson_solve(plans[i], rho[i], phi[i], tol, st);
                msg[i] = cylpoisson_last_error();
            }
            // the answers' last transforms; if they are lost, so are this lane's
            // answers, and no other's
            const hipError_t e = hipStreamSynchronize(st);
            if (e == hipSuccess) return;
            (void)hipGetLastError();
            for (int i : q->taken[l])
                if (res[i] >= 0) {
                    res[i] = CYLPOISSON_EHIP;
                    msg[i] = std::string("waiting for the answer: ") + hipGetErrorString(e);
                }
        };
        for (const auto& q : queues)
            for (int i : q->order) plans[i]->share = std::min(q->lanes, kShare);
        // the first lane of the first device runs on the caller's thread, and
        // so does one whose thread cannot be started
        std::vector<std::thread> threads;
        std::vector<std::pair<Queue*, int>> here;
        threads.reserve(count);
        here.reserve(count);
        for (const auto& q : queues)
            for (int l = 0; l < q->lanes; ++l) {
                if (q == queues[0] && l == 0) {
                    here.emplace_back(q.get(), l);
                    continue;
                }
                try {
                    threads.emplace_back(lane, q.get(), l);
                } catch (const std::system_error&) {
                    here.emplace_back(q.get(), l);
                }
            }
        for (const auto& h : here) lane(h.first, h.second);
        for (auto& t : threads) t.join();
        for (int i = 0; i < count; ++i) plans[i]->share = 1;
        for (int i = 0; i < count; ++i)
            if (statuses) statuses[i] = res[i];
        // the batch status: the first error, else NOT_CONVERGED if any, else OK
        for (int i = 0; i < count; ++i)
            if (res[i] < 0) {
                set_error("batch problem %d: %s", i, msg[i].c_str());
                status = res[i];
                break;
            }
        if (status == CYLPOISSON_OK)
            for (int i = 0; i < count; ++i)
                if (res[i] == CYLPOISSON_NOT_CONVERGED) {
                    set_error("batch problem %d: %s", i, msg[i].c_str());
                    status = CYLPOISSON_NOT_CONVERGED;
                    break;
                }
    }
    (void)hipEventDestroy(start);
    return status;
}

}  // namespace

}  // namespace cp

using namespace cp;

extern "C" {

int cylpoisson_solve_batch(cylpoisson_plan* const* plans, const double* const* rho, double* const* phi,
                           int count, double tol, void* stream, int* statuses) {
    if (count < 0 || (count > 0 && (!plans || !rho || !phi))) {
        set_error("batch arrays must not be NULL and count must be >= 0");
        return CYLPOISSON_EINVAL;
    }
    for (int i = 0; i < count; ++i)
        for (int j = 0; j < i; ++j)
            if (plans[i] == plans[j] || !plans[i]) {
                set_error("batch entry %d: plans must be distinct and not NULL", i);
                return CYLPOISSON_EINVAL;
            }
    if (count > 0 && !plans[0]) {
        set_error("batch entry 0: plans must be distinct and not NULL");
        return CYLPOISSON_EINVAL;
    }
    if (!(tol > 0.0) || !std::isfinite(tol)) {
        set_error("tol must be a positive finite number");
        return CYLPOISSON_EINVAL;
    }
    return solve_lanes(plans, rho, phi, count, tol, static_cast<hipStream_t>(stream), statuses);
}

}  // extern "C"
