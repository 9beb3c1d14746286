// Host checks of the rule by which a digit split takes its own row maxima.
#include <cstdio>
#include <cstdlib>

#include "plan.hpp"

using namespace dmp;

#define CHECK(x)                                                \
    do {                                                        \
        if (!(x)) {                                             \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x); \
            std::exit(1);                                       \
        }                                                       \
    } while (0)

// An m x n x k product: A by rows, B by columns or by rows.
static bool self(int m, int n, int k, dmp_kind kind, bool b_columns) {
    SplitDesc d[2] = {};
    d[0].R = m;
    d[1].R = n;
    d[0].K = d[1].K = k;
    d[0].KC = d[1].KC = int(chunks_of(k, kind));
    d[1].trans = b_columns ? 1 : 0;
    return split_takes_maxima(d, 2);
}

int main() {
    // short reductions always, long ones never
    CHECK(self(1 << 20, 64, 256, DMP_OZ_INT8, true) && self(1 << 20, 64, 256, DMP_OZ_INT8, false));
    CHECK(self(1 << 20, 64, 128, DMP_OZ_FP16, true));
    CHECK(!self(64, 64, 513, DMP_OZ_INT8, true));
    // between them few rows only
    CHECK(self(4096, 64, 512, DMP_OZ_INT8, true) && !self(8192, 64, 512, DMP_OZ_INT8, true));
    CHECK(self(2048, 64, 512, DMP_OZ_INT8, false) && !self(4096, 64, 512, DMP_OZ_INT8, false));
    CHECK(!self(64, 65536, 512, DMP_OZ_INT8, true) && !self(20000, 128, 400, DMP_MARKIDIS_FP16, true));
    CHECK(self(1024, 64, 512, DMP_OZ_FP16, true) && !self(4096, 64, 512, DMP_OZ_FP16, true));
    CHECK(self(64, 64, 64, DMP_OZ_INT8, true) && self(1024, 1024, 512, DMP_OZ_INT8, true));
    std::printf("split rule ok\n");
}
