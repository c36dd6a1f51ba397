// The sample of nodes from which a graph is taken for an unordered mixture of
// element families (host_graph.h): one node of every group, and on structured
// numberings of any line length the share of the sample that lies on given
// planes is the planes' share of the nodes. Exit status 0 on success.
#include <cmath>
#include <cstdio>
#include <vector>

#include "../../paper_1805_03949_amd/csrc/host_graph.h"

using namespace fea::host;

static int failures = 0;

// m^3 nodes, x fastest; nodes with coordinate d in `planes` are the mixed ones.
// The bound is six standard deviations of an independent sample.
static void run(int64_t m, int d, const std::vector<int64_t> &planes)
{
    const int64_t n = m * m * m, groups = (n + kMixedStep - 1) / kMixedStep;
    const int64_t div = d == 0 ? 1 : d == 1 ? m : m * m;
    int64_t hits = 0;
    for (int64_t g = 0; g < groups; ++g) {
        const int64_t v = mixed_sample(g, n);
        if (v < g * kMixedStep || v >= (g + 1) * kMixedStep || v >= n) {
            std::fprintf(stderr, "%lld nodes a line: group %lld gives %lld\n", (long long)m, (long long)g, (long long)v);
            ++failures;
            return;
        }
        for (int64_t p : planes) hits += v / div % m == p;
    }
    const double p = (double)planes.size() / (double)m, got = (double)hits / (double)groups;
    if (std::fabs(got - p) > 6 * std::sqrt(p * (1 - p) / (double)groups)) {
        std::fprintf(stderr, "%lld nodes a line, direction %d: share %.4f of the nodes, %.4f of the sample\n", (long long)m,
                     d, p, got);
        ++failures;
    }
}

int main()
{
    for (int64_t m : {17, 32, 33, 48, 49, 64, 80, 96, 97})
        for (int d = 0; d < 3; ++d) {
            run(m, d, {m / 4, m / 2, 3 * m / 4});
            run(m, d, {16});
            for (int64_t p = 1; p + 16 < m; p += 5) run(m, d, {p, p + 16});
        }
    for (int64_t n = 1; n < 100; ++n)  // the last group is partial
        for (int64_t g = 0; g * kMixedStep < n; ++g)
            if (mixed_sample(g, n) < g * kMixedStep || mixed_sample(g, n) >= n) ++failures;
    return failures ? 1 : 0;
}
