// TaskPool: every index of every job runs once, whoever comes; jobs of fewer tasks than threads, of slow tasks, and one right after
// the other, so that a worker asked for one job may wake in the next.
#include <chrono>
#include <cstdio>
#include <thread>

#include "zi_io_pool.h"

using namespace zi::host;

struct Job {
    std::atomic<int>* ran;
    std::atomic<int> others{0};
    int slow_us = 0, fail_at = -1;
};
static int task(void* ctx, size_t i, int who)
{
    Job& j = *static_cast<Job*>(ctx);
    j.ran[i].fetch_add(1);
    if (who != 0) j.others.fetch_add(1);
    if (j.slow_us) std::this_thread::sleep_for(std::chrono::microseconds(j.slow_us));
    return (int)i == j.fail_at ? 7 : 0;
}

int main()
{
    std::vector<std::atomic<int>> ran(600);
    for (int threads : {1, 2, 5, 16}) {
        TaskPool pool(threads);
        int helped = 0;
        for (int round = 0; round < 400; ++round)
            for (size_t n : {(size_t)0, (size_t)1, (size_t)2, (size_t)3, (size_t)17, round % 40 ? (size_t)4 : (size_t)600}) {
                for (auto& r : ran) r.store(0);
                Job j{ran.data()};
                j.slow_us = round % 50 == 7 ? 300 : 0;
                j.fail_at = round % 10 == 3 && n > 2 ? 2 : -1;
                const int err = pool.run(n, task, &j);
                for (size_t i = 0; i < ran.size(); ++i)
                    if (ran[i].load() != (i < n ? 1 : 0)) { std::printf("%d threads: task %zu of %zu ran %d times\n", threads, i, n, ran[i].load()); return 1; }
                if (err != (j.fail_at >= 0 ? 7 : 0)) { std::printf("error %d\n", err); return 1; }
                helped += j.others.load();
            }
        if (threads > 1 && helped == 0) { std::printf("%d threads: nobody helped\n", threads); return 1; }
    }
    std::puts("pool jobs ok");
    return 0;
}
