// The trainer's window of chunks against a device with room for `room` chunks: it holds the frame or a whole
// window where that fits, else at least half of the room (down to the smallest window), asks for no more than an
// eighth over the need, gives up only below the smallest window, and passes other errors on at once.
#include <cstdio>
#include <initializer_list>

#include "train_window.h"

using namespace dpk;

static int check(size_t have, size_t chunks, size_t room)
{
    size_t got = have, calls = 0;
    const size_t need = std::min<size_t>(std::max<size_t>(chunks, 1), TRE_WINDOW), least = std::min<size_t>(need, TRE_WINDOW_MIN);
    const int s = window_alloc(have, chunks, 0, 2, [&](size_t n) {
        ++calls;
        if (n > need + need / 8 || n > (size_t)TRE_WINDOW || n < least) return 9;
        got = 0;   // (the blocks at hand are given back first)
        if (n > room) return 2;
        got = n;
        return 0;
    });
    bool good = calls < 30;
    if (need <= have) good = good && s == 0 && calls == 0 && got == have;
    else if (room >= need) good = good && s == 0 && got >= need;
    else if (room >= least) good = good && s == 0 && got >= least && got <= room && (2 * got >= room || got >= need / 2);
    else good = good && s == 2 && got == 0;
    if (!good) std::printf("have %zu chunks %zu room %zu: status %d got %zu calls %zu\n", have, chunks, room, s, got, calls);
    return good ? 0 : 1;
}

int main()
{
    int bad = 0;
    const std::initializer_list<size_t> sizes = {0, 1, 2, 500, 1023, 1024, 1025, 1151, 1152, 3000, 73800, 83025, 131071, 131072, 131073, 229376, 5000000};
    for (size_t have : sizes)
        for (size_t chunks : sizes)
            for (size_t room : sizes) bad += check(have, chunks, room);
    int calls = 0;
    const int s = window_alloc(0, 100000, 0, 2, [&](size_t) { ++calls; return 7; });
    bad += s != 7 || calls != 1;
    if (!bad) std::printf("window ok\n");
    return bad ? 1 : 0;
}
