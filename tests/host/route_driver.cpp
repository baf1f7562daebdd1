// Which route a launch shape takes, the autotuner's choice between five
// passes and three launches, and which groups one launch must not run (host
// functions of csrc/kernels.h).
#include <cstdio>

#include "../../paper_2506_04489_amd/csrc/kernels.h"

using namespace psp;

static int failures = 0;
#define EXPECT(cond) \
    do { \
        if (!(cond)) { \
            std::printf("line %d: %s\n", __LINE__, #cond); \
            ++failures; \
        } \
    } while (0)

static Shape shape(int N, int tile, bool fused) {
    Shape s;
    for (int p = 0; p < kPasses; ++p) {
        s.plan[p] = fused || !r16_plan_exists(N) ? fused_plan(N, p == 2 ? 2 : p == 1 || p == 3 ? 1 : 0) : 1;
        s.tile[p] = tile;
    }
    return s;
}

int main() {
    for (int N : {8, 32, 36, 96, 108, 128, 256}) {
        // a shape from the table goes by its plans, one set by hand does not
        Shape s = shape(N, 0, true);
        EXPECT(fused_shape(N, s));
        Shape five = s;
        five.five = true;
        EXPECT(!fused_shape(N, five));
        EXPECT(!(five == s) && (five < s) != (s < five));
        // lengths with one plan: both outcomes have the same plans and differ in route
        const Shape pick = shape(N, 1, true);
        const Shape won = route_pick(N, pick, 20.0f, s, 15.0f), lost = route_pick(N, pick, 15.0f, s, 20.0f);
        EXPECT(fused_shape(N, won) && won.tile[0] == 0);
        EXPECT(!fused_shape(N, lost) && lost.five && lost.tile[0] == 1);
        // 0.2% is a draw, which keeps the five passes
        EXPECT(!fused_shape(N, route_pick(N, pick, 10.0f, s, 9.99f)));
        EXPECT(fused_shape(N, route_pick(N, pick, 10.0f, s, 9.97f)));
    }
    // other plans need no flag: they have no three launches
    const Shape other = shape(128, 2, false);
    const Shape kept = route_pick(128, other, 10.0f, shape(128, 0, true), 12.0f);
    EXPECT(kept == other && !kept.five && !fused_shape(128, kept));
    EXPECT(!fused_shape(512, Shape{}) && !fused_shape(216, Shape{}));
    // tiles with half the threads per column and their forms with all of them
    for (int c = 0; c < 3; ++c) {
        const int full[7] = {0, 1, 2, 0, 2, 5, 5};
        for (int t = 0; t < 7; ++t) EXPECT(full_threads(7 * c + t) == 7 * c + full[t]);
    }
    // a u over the rho of another solve, wholly or by one byte, and not over its own
    char b[4096];
    const size_t w = 512;
    EXPECT(!feeds_another({b, b + w}, {b + 2 * w, b + 3 * w}, w));
    EXPECT(feeds_another({b, b + w}, {b + w, b}, w));
    EXPECT(feeds_another({b, b + w}, {b + 2 * w, b + w - 1}, w) && feeds_another({b, b + 2 * w}, {b + 4 * w, b + w - 1}, w));
    EXPECT(!feeds_another({b, b + w}, {b + 4 * w, b + 2 * w}, w) && !feeds_another({b + w, b + 3 * w}, {b, b + 2 * w}, w));
    EXPECT(!feeds_another({b, b + 4 * w}, {b + 8, b + 4 * w + 8}, w));
    EXPECT(feeds_another({b, b}, {b + 8, b + 4 * w}, w));
    EXPECT(!feeds_another({(void *)8, (void *)4096}, {(void *)1024, (void *)2048}, w));
    EXPECT(feeds_another({(void *)8, (void *)4096}, {(void *)1024, (void *)16}, w));
    std::printf("%d failures\n", failures);
    return failures != 0;
}
