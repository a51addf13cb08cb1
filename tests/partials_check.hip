// Host-side check of the size of the reduction buffers (cg_partials_needed,
// lqs_impl.hpp): for every number of sites and block size a right-hand side's
// share holds what each kernel writes, and is even, so that the pairs of every
// side stand on 16 bytes.  Built and run on the CPU by test_reductions_host.py;
// it launches nothing on a GPU.
#include <cstdio>

#include "lqs_impl.hpp"

using namespace lqs;

int main()
{
    long bad = 0;
    for (int64_t vh = 8; vh < (1 << 20); vh += vh < 4096 ? 8 : 56)
        for (int block : {64, 128, 256, 512}) {
            const int64_t n = cg_partials_needed(vh, block);
            bad += n % 2 != 0 || n < 2 * 1024 || n < (vh + 63) / 64 || n < 2 * ((vh + block - 1) / block);
        }
    std::printf("bad %ld\n", bad);
    return bad != 0;
}
