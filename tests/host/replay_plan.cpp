// Host checks of the graphs a purification run launches and of the cache that
// keeps them (plan.hpp).
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <set>

#include "plan.hpp"

using namespace dmp;

#define CHECK(x)                                                \
    do {                                                        \
        if (!(x)) {                                             \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x); \
            std::exit(1);                                       \
        }                                                       \
    } while (0)

int main() {
    for (int n : {1, 1023, 1024, 4095, 4096, 20000}) {
        const int m = iterations_per_sync(n);
        CHECK(m > 0 && m % 2 == 0);
        for (int predicted = 0; predicted <= 204; ++predicted) {
            std::set<int> graphs{m};
            int sum = 0;
            for (int c : replay_plan(m, predicted)) {
                CHECK(c > 0 && c % 2 == 0);
                graphs.insert(c);
                sum += c;
            }
            CHECK(sum == (predicted + 1) / 2 * 2);
            CHECK(graphs.size() <= kGraphsPerSequence);
        }
    }
    // eight sequences run in turn record nothing after their first round
    KeyedCache<int> cache(kGraphCacheCapacity);
    for (int round = 0; round < 3; ++round)
        for (int seq = 0; seq < 8; ++seq) {
            int recorded = 0;
            auto graph = [&](int count) {
                bool made = false;
                CHECK(cache.get_or_create({seq, count}, [] { return std::make_shared<int>(0); }, &made));
                recorded += made ? 1 : 0;
            };
            graph(8);
            for (int c : replay_plan(8, 18 + 8 * seq)) graph(c);
            CHECK(round == 0 || recorded == 0);
        }
    std::printf("replay plan ok\n");
}
