// Which requests of the queue go to the device together, checked on the CPU
// (built against the HIP stand-in of this folder by tests/test_queue_ticks.py).
// Test infrastructure only.  The scheduler's event queries report "not ready"
// while the gate is shut, so nothing the queue has launched ends: what it has
// launched, what still waits and what can be cancelled is then fixed.
//
// Sixteen requests of n = 16,384 (four to a launch) and two of n = 700 after them:
// two launches of long requests, the first of which may have taken whatever had
// arrived, then two of short ones; the other long requests wait, and those can be
// cancelled, the launched ones cannot.  Prints "ok" when everything holds.
#include <math.h>
#include <stdio.h>

#include <atomic>
#include <chrono>
#include <thread>
#include <vector>

#include "geolik.h"

#include <hip/hip_runtime.h>

static std::atomic<bool> gate{false};
hipError_t gated_event_query(hipEvent_t) { return gate.load() ? hipSuccess : hipErrorNotReady; }

static int failures = 0;
#define CHECK(cond, ...)                  \
    do {                                  \
        if (!(cond)) {                    \
            fprintf(stderr, __VA_ARGS__); \
            fputc('\n', stderr);          \
            ++failures;                   \
        }                                 \
    } while (0)

static uint64_t tick_count(lq_queue *q)
{
    uint64_t n = 0;
    lq_tick_stats(q, &n, nullptr, nullptr, nullptr);
    return n;
}

// Ticks launched, once the count has stood still for a while.
static uint64_t settled(lq_queue *q)
{
    uint64_t n = tick_count(q);
    for (int same = 0; same < 50;) {
        std::this_thread::sleep_for(std::chrono::milliseconds(2));
        const uint64_t m = tick_count(q);
        same = m == n ? same + 1 : 0;
        n = m;
    }
    return n;
}

int main()
{
    gl_context *ctx = nullptr;
    if (gl_context_create(0, (size_t)40 << 30, &ctx) != GL_OK) return 2;
    const int64_t big = 16384, small = 700;
    std::vector<double> x(big), y(big, 0.0), z(big, 0.5);
    for (int64_t i = 0; i < big; ++i) x[i] = (double)i;
    uint64_t db = 0, dsm = 0;
    CHECK(gl_dataset_register(ctx, x.data(), y.data(), z.data(), big, &db) == GL_OK, "register");
    CHECK(gl_dataset_register(ctx, x.data(), y.data(), z.data(), small, &dsm) == GL_OK, "register");
    lq_queue *q = nullptr;
    if (lq_create(ctx, nullptr, &q) != GL_OK) return 2;
    const gl_theta th{2.0, 0.1, 0.5};
    std::vector<uint64_t> lg(16), sh(2);
    for (uint64_t &t : lg) CHECK(lq_submit(q, db, th, nullptr, &t) == GL_OK, "submit");
    CHECK(settled(q) == 2, "%lu launches of long requests", (unsigned long)tick_count(q));
    for (uint64_t &t : sh) {
        CHECK(lq_submit(q, dsm, th, nullptr, &t) == GL_OK, "submit");
        settled(q);
    }
    CHECK(tick_count(q) == 4, "%lu launches with the short requests", (unsigned long)tick_count(q));
    CHECK(lq_cancel(q, lg[0]) == GL_EBUSY, "a launched request was cancelled");
    CHECK(lq_cancel(q, lg[15]) == GL_OK, "a waiting request was not cancelled");
    CHECK(lq_cancel(q, sh[0]) == GL_EBUSY, "a launched request was cancelled");
    gl_result r;
    CHECK(lq_wait(q, lg[15], &r, 200000) == GL_ECANCELED, "cancelled");
    CHECK(lq_poll(q, lg[0], &r) == GL_EBUSY, "ended behind the gate");
    gate = true;
    auto l = [&](int64_t n) {
        return -0.5 * 0.25 * (double)n / th.theta1 - 0.5 * (double)n * log(th.theta1) - 0.5 * (double)n * log(2.0 * M_PI);
    };
    for (int i = 0; i < 15; ++i) {
        CHECK(lq_wait(q, lg[i], &r, -1) == GL_OK, "long %d", i);
        CHECK(fabs(r.loglik - l(big)) <= 1e-10 * fabs(l(big)), "l of long %d", i);
    }
    for (int i = 0; i < 2; ++i) {
        CHECK(lq_wait(q, sh[i], &r, -1) == GL_OK, "short %d", i);
        CHECK(fabs(r.loglik - l(small)) <= 1e-10 * fabs(l(small)), "l of short %d", i);
    }
    uint64_t completed = 0;
    int32_t peak = 0;
    lq_stats(q, &completed, nullptr, &peak, nullptr);
    CHECK(completed == 17 && peak == 18, "completed %lu peak %d", (unsigned long)completed, peak);
    // a waiting request's data set may go, and so may the queue
    gate = false;
    for (uint64_t &t : lg) CHECK(lq_submit(q, db, th, nullptr, &t) == GL_OK, "submit");
    settled(q);
    CHECK(gl_dataset_release(ctx, db) == GL_OK, "release");
    CHECK(lq_cancel(q, lg[14]) == GL_OK, "waiting");
    gate = true;
    CHECK(lq_destroy(q) == GL_OK, "destroy");
    CHECK(gl_dataset_release(ctx, dsm) == GL_OK, "release");
    gl_context_destroy(ctx);
    if (failures) return 1;
    printf("ok\n");
    return 0;
}
