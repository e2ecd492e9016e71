// The epsilon rule's run search on a long axis whose prefix sums lose mass: behind
// a large value at the axis's start lie many small ones of just under half a unit in
// the last place of the prefix sums there, between a medium and a second large one.
// The run from the medium to the large one holds the target by its direct sum, whose
// small terms are added to a small sum first; it must not be passed over for a
// longer one because its difference of prefix sums lacks them.
#include <cstdio>
#include <vector>

#include "host_geometry.h"

int main() {
    int fails = 0;
    for (int M : {100, 3000, 30000, 60000}) {
        const int N = 2 * M + 16;
        std::vector<double> m(N, 0.0);
        m[0] = 0.5 + 0x1p-10;
        m[1] = 0x1p-10;
        for (int k = 2; k <= M; ++k) m[k] = 0.49 * 0x1p-53;
        m[M + 1] = 0.5 + 0x1p-6;
        double T = 0.0, mass = 0.0;
        for (int k = 0; k < N; ++k) T += m[k];
        for (int k = 1; k <= M + 1; ++k) mass += m[k];
        double eps = 3.0 * (1.0 - mass / T);   // the run holds the target, by a hair
        for (int k = 0; k < 100 && !((1.0 - eps / 3.0) * T <= mass); ++k) eps += 1e-16;
        int lo = -1, len = -1;
        eps_run(m.data(), N, eps, &lo, &len);
        std::printf("N %d: run of %d points from %d, expected %d from 1\n", N, len, lo, M + 1);
        if (lo != 1 || len != M + 1) ++fails;
    }
    std::printf("long axes: %d failures\n", fails);
    return fails ? 1 : 0;
}
