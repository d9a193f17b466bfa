// grad_reserve with a counting allocator of limited capacity, for tests/test_grad_workspace.py.
// A layout of n chunks needs fixed + (rows + n - 1) / n bytes.
#include "grad_workspace.hpp"

namespace {
struct Layout {
    std::size_t bytes;
    int chunks;
};
struct State {
    gpmppi::GradWorkspace w;
    std::size_t capacity, used, fixed, rows;
    int allocs, frees;
};
Layout layout(const State &s, int n) { return Layout{s.fixed + (s.rows + n - 1) / n, n}; }
}  // namespace

extern "C" {
State *ws_new(std::size_t capacity, std::size_t fixed, std::size_t rows) {
    return new State{{}, capacity, 0, fixed, rows, 0, 0};
}
void ws_delete(State *s) { delete s; }
void ws_capacity(State *s, std::size_t capacity) { s->capacity = capacity; }
int ws_allocs(const State *s) { return s->allocs; }
int ws_frees(const State *s) { return s->frees; }
std::size_t ws_bytes(const State *s) { return s->w.bytes; }
// One call with at most `limit` bytes; returns its chunks, 0 if there is no memory for it.
int ws_call(State *s, std::size_t limit) {
    Layout g = layout(*s, 1);
    const bool ok = gpmppi::grad_reserve(
        s->w, g, limit,
        [&](std::size_t most) {
            int n = 1;
            while (layout(*s, n).bytes > most && n < (int)s->rows) ++n;
            return layout(*s, n);
        },
        [&](std::size_t n) -> void * {
            ++s->allocs;
            if (n > s->capacity) return nullptr;
            s->used = n;
            return s;
        },
        [&](void *) {
            ++s->frees;
            s->used = 0;
        });
    return ok ? g.chunks : 0;
}
}
