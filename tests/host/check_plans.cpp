// CPU checks of the launch plans (host_tables.cpp), built with AddressSanitizer
// and UndefinedBehaviorSanitizer by tests/test_host_plans.py.
#include <stdio.h>
#include <stdlib.h>

#include <vector>

#include "host_tables.h"

using namespace sqz;

static int g_fail = 0;
#define EXPECT(cond, ...)                                   \
    do {                                                    \
        if (!(cond)) {                                      \
            fprintf(stderr, "FAILED %s:%d: ", __FILE__, __LINE__); \
            fprintf(stderr, __VA_ARGS__);                   \
            fprintf(stderr, "\n");                          \
            if (++g_fail > 20) exit(1);                     \
        }                                                   \
    } while (0)

// Sum, parity, bound, and as few launches as these allow.
static void check_plan(const std::vector<int> &plan, int32_t steps, int K, const char *what)
{
    int64_t sum = 0;
    for (int k : plan) {
        EXPECT(k >= 1 && (K < 1 || k <= K), "%s steps %d K %d: a launch of %d", what, steps, K, k);
        sum += k;
    }
    EXPECT(sum == steps, "%s steps %d K %d: %lld steps planned", what, steps, K, (long long)sum);
    EXPECT((plan.size() & 1) == (size_t)(steps & 1), "%s steps %d K %d: parity of %zu launches", what, steps, K, plan.size());
    int64_t n = steps < 1 ? 0 : (K < 1 ? 1 : ((int64_t)steps + K - 1) / K);
    n += (n ^ steps) & 1;
    EXPECT((int64_t)plan.size() == n, "%s steps %d K %d: %zu launches, want %lld", what, steps, K, plan.size(), (long long)n);
}

static void expect_full(int32_t steps, int K, const std::vector<int> &want)
{
    EXPECT(plan_full_launches(steps, K) == want, "full launches, steps %d K %d", steps, K);
}

int main()
{
    for (int K = 0; K <= 40; ++K)
        for (int32_t steps = 0; steps <= 200; ++steps) {
            check_plan(plan_launches(steps, K), steps, K, "equal");
            if (K >= 2) check_plan(plan_full_launches(steps, K), steps, K, "full");
        }
    // a group's launches: no more steps than chosen, the tiles' most without a choice
    for (int chosen : {0, 1, 2, 7, 10})
        for (int full : {0, 15, 27, 31})
            for (int32_t steps = 0; steps <= 200; ++steps)
                for (bool one : {false, true})
                    check_plan(plan_group_launches(steps, chosen, full, one), steps, chosen ? chosen : full, "group");
    EXPECT(plan_group_launches(30, 10, 31, true) == (std::vector<int>{9, 10, 10, 1}), "ten chosen");
    EXPECT(plan_group_launches(30, 0, 31, true) == (std::vector<int>{29, 1}), "none chosen");
    // the tuner times what an untuned run takes, and every choice as it would run
    for (int most : {1, 7, 8, 10})
        for (int full : {0, 15, 27, 31}) {
            const std::vector<GroupChoice> v = group_choices(most, full);
            EXPECT(v[0].chosen == 0 && (full ? v[0].steps == full : v[0].steps > 10), "no choice is timed, full %d", full);
            for (size_t i = 1; i < v.size(); ++i)
                EXPECT(v[i].chosen >= 1 && v[i].chosen <= most && v[i].steps == v[i].chosen, "choice %zu of at most %d", i, most);
            for (const GroupChoice &c : v) {
                const std::vector<int> plan = plan_group_launches(8 * c.steps, c.chosen, full, false);
                for (int k : plan) EXPECT(full ? k == c.steps : k >= c.steps, "choice %d runs %d steps, timed %d", c.chosen, k, c.steps);
            }
        }
    // counts near the largest int32, where steps + K - 1 leaves its range
    for (int K : {0, 1, 15, 27, 31})
        for (int32_t steps : {1 << 30, (1 << 30) + 1, 0x7FFFFFFF - 14, 0x7FFFFFFF}) {
            const int64_t n = launch_count(steps, K);
            EXPECT(n >= 1 && (K < 1 ? n == 1 : n * K >= steps && (n - 1) * K < steps), "launches of %d steps, K %d", steps, K);
            int64_t first = 0, last = 0;
            for (int64_t i = 0; i < n && i < 1000; ++i) {
                first += launch_share(steps, n, i);
                last += launch_share(steps, n, n - 1 - i);
                EXPECT(launch_share(steps, n, i) >= 1 && (K < 1 || launch_share(steps, n, i) <= K), "share of %d steps, K %d", steps, K);
            }
            const int64_t m = n < 1000 ? n : 1000;
            EXPECT(first == steps * m / n && last == steps - steps * (n - m) / n, "shares of %d steps, K %d", steps, K);
        }
    expect_full(4, 3, {3, 1});
    expect_full(5, 3, {3, 1, 1});
    expect_full(7, 3, {3, 3, 1});
    expect_full(8, 3, {3, 3, 1, 1});
    expect_full(9, 3, {3, 3, 3});
    expect_full(2, 3, {1, 1});
    expect_full(6, 4, {4, 2});
    if (g_fail) {
        fprintf(stderr, "%d check(s) failed\n", g_fail);
        return 1;
    }
    printf("launch plans: all checks passed\n");
    return 0;
}
