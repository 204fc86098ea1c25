// Prints what the library's rules of dispatch choose (not part of libdq.so): built by tests/test_dispatch_rules.py and run on the CPU.
// "whole": chunks of one tensor, all chunks, and whether sign messages go chunk by chunk.
// "norm": workgroups, padded values and items of one worker's gradient, and whether the pass runs as a stream.
// One line for every number of tiles, workers, width (0: a widths table; "rows": one with a row per worker)
// and kind of reduce: what ur_form_of says.
#include <cstdio>

#include "dq_reduce_core.h"

int main()
{
    const int64_t tiles[] = { 1, 100, 256, 300, 384, 385, 400, 470, 512, 513, 600, 650, 680, 720, 768, 769, 800, 1000, 1024, 1280, 1281, 1366, 1532, 2048, 2500, 3072, 3073, 3200, 4096, 6000, 8192, 16384, 32768 };
    for (int64_t n : tiles)
        for (int M = 1; M <= DQ_MAX_WORKERS; ++M)
            for (int b = 0; b <= 8; ++b)
                for (int update = 0; update < 2; ++update) {
                    dq_plan plan{};
                    plan.padded_elems = n * ur_tile<1>;
                    const ur_form f = ur_form_of(&plan, b, M, update != 0);
                    std::printf("reduce %lld %d %d %d %d %d %d\n", static_cast<long long>(n), M, b, update, f.two ? 2 : 1, f.stream, f.once);
                    if (b != 0) continue;
                    const ur_form r = ur_form_of(&plan, b, M, update != 0, true);
                    std::printf("rows %lld %d %d %d %d %d %d\n", static_cast<long long>(n), M, b, update, r.two ? 2 : 1, r.stream, r.once);
                }
    const int64_t items[] = { 1000, 8191, 8192, 40000 };
    for (int64_t n : items)
        for (int64_t average : { 384, 1152, 2560, 3000, 3583, 3584, 4096 })
            std::printf("norm %lld %lld %lld %d\n", static_cast<long long>(n), static_cast<long long>(n * average), static_cast<long long>(n),
                        dq_norm_streams(n, n * average, n));
    for (int64_t whole : { 0, 18, 32, 49, 50, 51, 100 })
        std::printf("whole %lld 100 %d\n", static_cast<long long>(whole), dq_mostly_whole(whole, 100));
    return 0;
}
