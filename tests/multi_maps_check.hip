// Host-side checks of the kernels that advance several steps in one launch
// (the same header functions the library uses):
//   * timed_steps: a timing of n steps of a schedule takes whole launches, at
//     least n steps and less than a launch more.
// Prints "ok" and exits 0, or prints the first failure and exits 1.
#include <cstdio>

#include "../paper_1306_6445_amd/csrc/lbm_kernels.hpp"

namespace {

int check_timed_steps()
{
    for (int per : {1, 2, 4})
        for (int64_t n = 1; n <= 70; ++n) {
            const int64_t t = lbm::timed_steps(n, per);
            if (t % per != 0 || t < n || t >= n + per) {
                std::printf("FAIL timed_steps: %lld steps, %d a launch -> %lld\n", (long long)n, per, (long long)t);
                return 1;
            }
        }
    return 0;
}

} // namespace

int main()
{
    if (check_timed_steps()) return 1;
    std::printf("ok\n");
    return 0;
}
