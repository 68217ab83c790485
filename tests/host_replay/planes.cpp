// Copies planes through the slots as the library's read-back does, pieces
// becoming ready one after the other, without any memory to be had (operator
// new throws; so does the start of a thread, which needs some): the planes
// arrive whole and nothing is thrown, since the copy runs under a C entry
// point (left out with -DPLANES_NO_STARVE, for sanitizers with an operator new
// of their own).  With memory, and so with helper threads, likewise.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "lbm_planes.h"

static std::atomic<bool> starve{false};
#ifndef PLANES_NO_STARVE
void *operator new(size_t n) {
    if (starve) throw std::bad_alloc();
    if (void *p = malloc(n)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }
#endif

using namespace lbm;

static bool copy_all(int64_t nodes, int64_t piece, int nslots) {
    std::vector<double> out((size_t)6 * nodes, -1.0), slots((size_t)nslots * 6 * piece, -2.0);
    double *outs[6];
    for (int q = 0; q < 6; ++q) outs[q] = out.data() + q * nodes;
    const int64_t pieces = (nodes + piece - 1) / piece;
    auto fill = [&](int64_t p) {  // what the kernel writes: the piece's planes one after the other
        const int64_t o = p * piece, n = std::min(piece, nodes - o);
        double *slot = slots.data() + (p % nslots) * 6 * piece;
        for (int q = 0; q < 6; ++q)
            for (int64_t i = 0; i < n; ++i) slot[q * n + i] = (double)(q * nodes + o + i);
    };
    int64_t filled = 0;
    while (filled < std::min<int64_t>(pieces, nslots)) fill(filled++);
    {
        PlaneCopy copy(outs, slots.data(), 6 * piece, nslots, piece, nodes);
        for (int64_t i = 0; i < pieces; ++i) {
            copy.publish(i + 1);
            if (i == 0) continue;
            copy.finish(i - 1);
            if (filled < pieces) fill(filled++);
        }
        copy.finish(pieces - 1);
    }
    for (int64_t i = 0; i < 6 * nodes; ++i)
        if (out[i] != (double)i) return false;
    return true;
}

int main() {
    const int64_t sizes[][3] = {{1, 1, 1}, {16384, 16384, 1}, {7, 3, 4}, {1000003, 131072, 4}, {600000, 131072, 4}, {131072 * 4, 131072, 4}};
    for (const auto &s : sizes)
        if (!copy_all(s[0], s[1], (int)s[2])) {
            printf("wrong: %lld nodes\n", (long long)s[0]);
            return 1;
        }
    // the same with every allocation failing from the copy's start on
    const int64_t nodes = 1000003, piece = 131072;
    std::vector<double> out((size_t)6 * nodes, -1.0), slots((size_t)4 * 6 * piece);
    double *outs[6];
    for (int q = 0; q < 6; ++q) outs[q] = out.data() + q * nodes;
    try {
        starve = true;
        PlaneCopy copy(outs, slots.data(), 6 * piece, 4, piece, nodes);
        for (int64_t p = 0; p * piece < nodes; ++p) {
            const int64_t o = p * piece, n = std::min(piece, nodes - o);
            for (int64_t i = 0; i < 6 * n; ++i) slots[(p % 4) * 6 * piece + i] = (double)(i / n * nodes + o + i % n);
            copy.publish(p + 1);
            copy.finish(p);
        }
        starve = false;
    } catch (const std::exception &e) {
        starve = false;
        printf("thrown: %s\n", e.what());
        return 1;
    }
    for (int64_t i = 0; i < 6 * nodes; ++i)
        if (out[i] != (double)i) {
            printf("wrong without memory\n");
            return 1;
        }
    printf("identical\n");
    return 0;
}
