// Prints, for every line "kind S method forced_rb slots count n ..." on standard
// input, the plan of such a purification on digit slices: groups, and of the
// first one the 32-row blocks per tile, the tiles and the parts of its tail.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "plan.hpp"

using namespace dmp;

int main() {
    int kind, S, method, rb, slots, count;
    while (std::scanf("%d %d %d %d %d %d", &kind, &S, &method, &rb, &slots, &count) == 6) {
        std::vector<int> n(count), nocc(count), s(count, S);
        for (int b = 0; b < count; ++b) {
            if (std::scanf("%d", &n[b]) != 1) return 1;
            nocc[b] = n[b] / 2;
        }
        std::vector<GroupPlan> groups;
        plan_groups(count, n.data(), s.data(), dmp_kind(kind), method, rb, groups, nocc.data(), true);
        Carver measure(nullptr);
        for (auto& g : groups) carve_group(measure, g, n.data());
        std::vector<double> dummy(2 * count);
        std::vector<const double*> H(count, dummy.data());
        std::vector<double*> P(count, dummy.data() + count);
        // addresses are stored, never followed
        Carver c(reinterpret_cast<void*>(uintptr_t(1) << 32));
        for (auto& g : groups) carve_group(c, g, n.data());
        GroupHost h;
        build_group(groups[0], H.data(), P.data(), n.data(), nocc.data(), slots, h);
        std::printf("%d %d %d %d\n", int(groups.size()), groups[0].rb, groups[0].ntiles, groups[0].tail.nsplit);
    }
}
