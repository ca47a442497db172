// Drives the read-ahead of a batch's results (csrc/read_ahead.h) with host
// memory that runs out: at every allocation of a walk over the results, for
// one time or from there on.  No exception may leave it (its caller is a C
// entry point), and every result must be right.  Exits non-zero otherwise.
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "read_ahead.h"

static long g_left = -1;      // allocations until one fails (< 0: none does)
static bool g_stay = false;   // all further ones fail too

void* operator new(size_t n)
{
    if (g_left == 0 && g_stay) throw std::bad_alloc();
    if (g_left > 0 && --g_left == 0) {
        if (!g_stay) g_left = -1;
        throw std::bad_alloc();
    }
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

using namespace pdhcg;

int main()
{
    // 3000 instances of 100 to 399 variables: some blocks of READ_AHEAD doubles
    const int64_t count = 3000;
    std::vector<int64_t> voff(count + 1, 0), roff(count + 1, 0);
    for (int64_t i = 0; i < count; ++i) {
        voff[i + 1] = voff[i] + 100 + i % 300;
        roff[i + 1] = roff[i] + i % 200;
    }
    int bad = 0;
    std::vector<double> x(400), y(200);
    for (const bool stay : {false, true})
        for (long k = 0; k < 40; ++k) {
            ReadAhead ra;
            g_stay = stay;
            g_left = k == 0 ? -1 : k;
            auto fetch = [&](int64_t a, int64_t b, double* xa, double* ya) {
                if (b > a + 1) std::vector<double> certificates(17);   // as the library's needs for a block
                for (int64_t q = voff[a]; xa && q < voff[b]; ++q) xa[q - voff[a]] = (double)q;
                for (int64_t q = roff[a]; ya && q < roff[b]; ++q) ya[q - roff[a]] = -(double)q;
                return 0;
            };
            auto check = [&](int64_t i, bool wx, bool wy) {
                try {
                    if (ra.get(i, count, voff.data(), roff.data(), wx ? x.data() : nullptr, wy ? y.data() : nullptr, fetch)) ++bad;
                } catch (...) {
                    std::printf("FAILED: an exception left the call (allocation %ld, instance %lld)\n", k, (long long)i);
                    ++bad;
                    return;
                }
                for (int64_t q = voff[i]; wx && q < voff[i + 1]; ++q) bad += x[q - voff[i]] != (double)q;
                for (int64_t q = roff[i]; wy && q < roff[i + 1]; ++q) bad += y[q - roff[i]] != -(double)q;
            };
            for (int64_t i = 0; i < count; ++i) check(i, true, true);
            for (int64_t i = count - 1; i >= 0; i -= 7) check(i, i % 2, true);
            for (int64_t i = 5; i < count; ++i) check(i, true, i % 3 == 0);
            g_left = -1;
        }
    std::printf("read-ahead driver: %d failure(s)\n", bad);
    return bad ? 1 : 0;
}
