// Host driver of tests/test_first_zero_cpu.py: the words of the split-K
// counters that each workgroup of the first-layer kernel clears (the statement
// is extracted from conv_direct.hip into first_zero.h by the test), for grids
// up to the largest a launch of 256 threads can have.

#include <cstddef>
#include <cstdio>
#include <map>

struct Dim { unsigned x; };
static Dim blockIdx, gridDim;

// stands for the counters: notes every index written
struct Words {
    std::map<long long, int> *written;
    struct Word {
        Words *w; long long i;
        void operator=(unsigned) { ++(*w->written)[i]; }
    };
    Word operator[](long long i) { return Word{this, i}; }
};
struct Args { int nzero; Words zero; };

static void block(Args &a, int tid)
{
#include "first_zero.h"
}

int main()
{
    const unsigned grids[] = {1, 2, 255, 4096, (1u << 23) - 1, 1u << 23, (1u << 23) + 1, (1u << 24) - 1};
    long runs = 0;
    for (unsigned g : grids)
        for (int nz : {0, 1, 255, 256, 257, 5000}) {
            std::map<long long, int> written;
            Args a{nz, {&written}};
            gridDim.x = g;
            // the first and last workgroups, those around 2^23 and a sample
            // between; every thread of them
            for (unsigned b = 0; b < g; b = (b < 64 || g - b < 64 || (b > (1u << 23) - 8 && b < (1u << 23) + 8)) ? b + 1
                                            : b + 1 + (g - b) / 97) {
                blockIdx.x = b;
                for (int tid = 0; tid < 256; ++tid) block(a, tid);
                ++runs;
            }
            for (const auto &[i, n] : written)
                if (i < 0 || i >= nz || n != 1) {
                    printf("grid %u, %d words: word %lld written %d times\n", g, nz, i, n);
                    return 1;
                }
            if ((long)written.size() != nz) {
                printf("grid %u: %ld of %d words written\n", g, (long)written.size(), nz);
                return 1;
            }
        }
    printf("ok %ld workgroups\n", runs);
    return 0;
}
