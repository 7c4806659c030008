// Host driver: runs of one graph planned on several threads at the same time,
// every thread the same schedules in an order of its own, each size the one a
// single thread got.
#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>

#include "fsg.h"

static size_t size_of(const fsg_graph *g, int i)
{
    fsg_params prm;
    memset(&prm, 0, sizeof(prm));
    prm.model = FSG_SIR;
    prm.beta = prm.gamma = 0.1;
    prm.max_steps = 5;
    fsg_schedule s;
    memset(&s, 0, sizeof(s));
    s.tile_edges = 1 + i % 1000;
    s.heavy_threshold = 1 + i / 1000;
    size_t bytes = 0;
    if (fsg_sim_workspace_size(g, &prm, 64, &s, &bytes) != FSG_OK) return 0;
    return bytes;
}

int main()
{
    const int kThreads = 8, kSizes = 4000, n = 6;
    const int64_t ptr[n + 1] = {0, 1, 3, 3, 6, 10, 15};
    const int32_t src[15] = {1, 0, 2, 0, 1, 2, 0, 1, 2, 3, 0, 1, 2, 3, 4};
    for (int rep = 0; rep < 4; ++rep) {
        fsg_graph *one = nullptr, *many = nullptr;
        if (fsg_graph_create(n, 15, ptr, src, &one) || fsg_graph_create(n, 15, ptr, src, &many)) return 1;
        std::vector<size_t> want(kSizes);
        for (int i = 0; i < kSizes; ++i) want[(size_t)i] = size_of(one, i);
        std::vector<int> bad(kThreads, 0);
        std::vector<std::thread> ts;
        for (int t = 0; t < kThreads; ++t)
            ts.emplace_back([&, t] {
                for (int k = 0; k < kSizes; ++k) {
                    const int i = (int)(((long long)k * (2 * t + 7) + 13 * rep) % kSizes);
                    if (size_of(many, i) != want[(size_t)i] || want[(size_t)i] == 0) ++bad[(size_t)t];
                }
            });
        for (auto &t : ts) t.join();
        for (int b : bad)
            if (b) return std::printf("FAIL: %d sizes differ\n", b), 1;
        fsg_graph_destroy(one);
        fsg_graph_destroy(many);
    }
    std::printf("plan threads ok\n");
    return 0;
}
