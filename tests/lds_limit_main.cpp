// The record of allowed LDS sizes: per kernel and device, from several threads, and beyond its capacity.
#include <stdio.h>

#include <thread>
#include <vector>

#include "lds_limit.hpp"

static int bad = 0;
#define CHECK(c) do { if (!(c)) { ++bad; printf("line %d: %s\n", __LINE__, #c); } } while (0)

int main() {
    static rnn::LdsRecord r;
    static char kernels[4096];
    const void *a = kernels, *b = kernels + 16;
    CHECK(!r.covers(a, 0, 70000));
    r.allowed(a, 0, 70000);
    CHECK(r.covers(a, 0, 70000) && r.covers(a, 0, 65537));
    CHECK(!r.covers(a, 1, 70000));            // the other GPU has a limit of its own
    CHECK(!r.covers(a, 0, 70001));
    CHECK(!r.covers(b, 0, 70000));
    r.allowed(a, 1, 80000);
    r.allowed(a, 1, 66000);                   // a smaller launch does not lower it
    CHECK(r.covers(a, 1, 80000) && r.covers(a, 0, 70000) && !r.covers(a, 0, 80000));
    std::vector<std::thread> threads;
    for (int t = 0; t < 8; ++t)
        threads.emplace_back([t] {
            for (int i = 0; i < 100; ++i) {
                r.allowed(kernels + 32 + 16 * (i % 50), t, 65537u + 1000u * (unsigned)i);
                r.covers(kernels + 32 + 16 * i, (t + 1) % 8, 65537);
            }
        });
    for (auto& t : threads) t.join();
    for (int t = 0; t < 8; ++t)
        for (int i = 50; i < 100; ++i) CHECK(r.covers(kernels + 32 + 16 * (i % 50), t, 65537u + 1000u * (unsigned)i));
    for (int i = 0; i < 2000; ++i) r.allowed(kernels + i, 20, 90000);   // more than it holds
    CHECK(r.covers(a, 0, 70000) && !r.covers(kernels + 1999, 20, 90000));
    printf(bad ? "failed\n" : "ok\n");
    return bad != 0;
}
