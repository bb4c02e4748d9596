// train_window.h -- how many chunks of operand blocks the trainer holds at a time (host logic).
#pragma once
#include <algorithm>
#include <cstddef>

namespace dpk {

// TRE_WINDOW chunks take 8.7 GB (a frame of 12,288 water atoms has 73,800).
constexpr int TRE_WINDOW = 1 << 17, TRE_WINDOW_MIN = 1 << 10;

// Blocks for a frame of `chunks` chunks where `have` are allocated: nothing to do if they hold the frame or
// a whole window; else alloc(n) for an eighth more than needed (the next frame), for what is needed, then half
// as many each time, TRE_WINDOW_MIN at least. alloc returns `ok`, `full` (no memory: fewer are tried) or another
// error, which ends the search.
template <class Status, class Alloc>
Status window_alloc(size_t have, size_t chunks, Status ok, Status full, Alloc&& alloc)
{
    const size_t need = std::min<size_t>(std::max<size_t>(chunks, 1), TRE_WINDOW);
    if (need <= have) return ok;
    for (size_t w = std::min<size_t>(need + need / 8, TRE_WINDOW);; w = w > need ? need : std::max<size_t>(w / 2, TRE_WINDOW_MIN)) {
        const Status s = alloc(w);
        if (s != full || w <= std::min<size_t>(need, TRE_WINDOW_MIN)) return s;
    }
}

}  // namespace dpk
