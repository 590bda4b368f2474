// Threads that add words to a shared buffer segment by segment and take its fill level between segments, as the blocks of the inverted-list
// kernels do.  One thread leaves every barrier late: only once all others wait at their next barrier (or are done).  Prints the levels
// read that differ from the words added so far, with fill_level and with the level read behind one barrier only.
#include <atomic>
#include <stdio.h>
#include <thread>
#include <vector>
#include "fill_level.h"

static const int THREADS = 4, SEGMENTS = 50;

struct Block {
    std::atomic<unsigned> words{0};
    std::atomic<int> arrived[THREADS];
    Block() { for (auto &a : arrived) a = 0; }
    // (each thread counts its barriers; it passes one when all have arrived at it)
    void sync(int me) {
        const int mine = ++arrived[me];
        for (int t = 0; t < THREADS; ++t) while (arrived[t] < mine) std::this_thread::yield();
        if (me != 0) return;
        for (;;) {  // the late one
            int on = 0;
            for (int t = 1; t < THREADS; ++t) on += arrived[t] > mine ? 1 : 0;
            if (on >= THREADS - 1) return;
            std::this_thread::yield();
        }
    }
};

template <class Level>
static long run(const Level &level) {
    Block b;
    std::atomic<long> wrong{0};
    std::vector<std::thread> all;
    for (int me = 0; me < THREADS; ++me)
        all.emplace_back([&, me] {
            for (int s = 0; s < SEGMENTS; ++s) {
                ++b.words;
                if (level(b, me, s + 1 < SEGMENTS) != (unsigned)(THREADS * (s + 1))) ++wrong;
            }
            b.arrived[me] = 1 << 20;  // (past every barrier)
        });
    for (auto &t : all) t.join();
    return wrong;
}

int main() {
    const long kept = run([](Block &b, int me, bool more) {
        return fill_level([&] { return b.words.load(); }, more, [&] { b.sync(me); });
    });
    const long one_barrier = run([](Block &b, int me, bool) {
        b.sync(me);
        return b.words.load();
    });
    printf("%ld %ld\n", kept, one_barrier);
    return 0;
}
