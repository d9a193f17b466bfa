// The gradient's workspace in one context: what a call takes and when memory is allocated.
#pragma once
#include <cstddef>

namespace gpmppi {

struct GradWorkspace {
    void *p = nullptr;
    std::size_t bytes = 0;
    bool denied = false;   // what was wished for could not be allocated: the samples are taken in chunks that fit
};

// Makes w hold at least g.bytes for the layout g; true on success.  Where that much cannot be
// allocated and is more than `limit` (the most a call may need), g becomes within(limit), the layout of
// the fewest chunks that need no more.  The workspace is kept: later calls take their chunks from it and
// neither free it nor ask for more again.
//   within(n)  the layout of the fewest chunks that need at most n bytes (or the smallest there is)
//   alloc(n)   n bytes or NULL;  release(p) frees them
template <class Layout, class Within, class Alloc, class Release>
bool grad_reserve(GradWorkspace &w, Layout &g, std::size_t limit, Within within, Alloc alloc, Release release) {
    if (g.bytes <= w.bytes) return true;
    if (w.denied) {
        const Layout h = within(w.bytes);
        if (h.bytes <= w.bytes) {
            g = h;
            return true;
        }
    }
    if (w.p) release(w.p);
    w = GradWorkspace{};
    w.p = alloc(g.bytes);
    if (!w.p && g.bytes > limit) {
        g = within(limit);
        w.p = alloc(g.bytes);
        w.denied = w.p != nullptr;
    }
    w.bytes = w.p ? g.bytes : 0;
    return w.p != nullptr;
}

}  // namespace gpmppi
