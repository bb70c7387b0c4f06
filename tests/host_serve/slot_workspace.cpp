// Host test of a serving slot's sizes: random matrices (rows, columns and
// chunk sizes over several orders of magnitude, every rate), each of whose
// graphs' plans must fit the workspace its slot is given.  The launch
// planner is compiled in; its kernels are not called.
//
// usage: slot_workspace fit <seed> <count> <most rows> <most values>
//            prints the shapes that fall short, exit status 3 if any
//        slot_workspace size <rate> <rows> <cols> <chunk values>
//            prints the workspace in bytes
#include "planner.hpp"

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>

#include "serve_plan.hpp"

using namespace wh;

int main(int argc, char** argv)
{
    constexpr int kCus = 256;
    const GemvTuning none;
    if (argc == 6 && !strcmp(argv[1], "size")) {
        wh_matrix_desc d{(uint32_t)atoi(argv[3]), (uint32_t)atoi(argv[4]), WH_FMT_ZFP_FIXED_RATE,
                         (uint32_t)atoi(argv[2])};
        const auto chunks = policy::chunk_rows(d.rows, d.cols, (uint64_t)atoll(argv[5]));
        printf("%zu\n", serve_workspace(d, chunks, kCus, none) * sizeof(double));
        return 0;
    }
    if (argc != 6 || strcmp(argv[1], "fit"))
        return 2;
    std::mt19937_64 gen((uint64_t)atoll(argv[2]));
    std::uniform_real_distribution<double> uni(0.0, 1.0);
    const auto log_int = [&](double most) { // 1 .. most, even over the logarithm
        return (uint32_t)std::lround(std::exp(uni(gen) * std::log(std::max(1.0, most))));
    };
    constexpr uint32_t rates[] = {2, 4, 6, 8, 10, 12, 14, 16, 20, 24, 32};
    const double most_rows = atof(argv[4]), most_values = atof(argv[5]);
    int bad = 0;
    for (int i = 0; i < atoi(argv[3]); ++i) {
        wh_matrix_desc d{};
        d.fmt = WH_FMT_ZFP_FIXED_RATE;
        d.rows = log_int(most_rows);
        d.cols = log_int(std::min(262144.0, most_values / d.rows));
        d.rate = rates[(int)(uni(gen) * 11)];
        const uint64_t values = uni(gen) < 0.3 ? 65536ull * log_int(4096) : 1ull << 28;
        auto chunks = policy::chunk_rows(d.rows, d.cols, values);
        if (chunks.size() > 3) // those between are as long as the first
            chunks = {chunks[0], chunks[1], chunks.back()};
        const size_t have = serve_workspace(d, chunks, kCus, none);
        for (const auto& c : chunks)
            for (uint32_t k : policy::kBuckets) {
                const size_t need = serve_plan(d, c, k, kCus, none, have).workspace;
                if (need <= have)
                    continue;
                if (bad++ < 5)
                    fprintf(stderr, "%u x %u rate %u rows [%u, %u) k %u: %zu bytes of %zu\n", d.rows, d.cols, d.rate,
                            c.first, c.second, k, need * 8, have * 8);
            }
    }
    return bad ? 3 : 0;
}
