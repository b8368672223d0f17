// Host-only checks of the rule that picks a panel's kernel (panel_rule.hpp).  Exit
// status 1 on any failure.
#include <cstdio>
#include <initializer_list>

#include "panel_rule.hpp"

using namespace nebem;

static int failures = 0;
#define CHECK(c)                                             \
    do {                                                     \
        if (!(c)) {                                          \
            std::printf("FAIL line %d: %s\n", __LINE__, #c); \
            ++failures;                                      \
        }                                                    \
    } while (0)

int main()
{
    // on 256 CUs: four workgroups of one wave each, one (FP64) or two (FP32) of four
    const int cap1 = 1024, cap8 = 256, cap4 = 512;
    CHECK(panel_waves(1, 8, cap1, cap8) == 1 && panel_waves(16384, 8, cap1, cap8) == 1);
    CHECK(panel_waves(16385, 8, cap1, cap8) == 4 && panel_waves(65536, 8, cap1, cap8) == 4);
    CHECK(panel_waves(65537, 8, cap1, cap8) == 0);
    CHECK(panel_waves(16384, 4, cap1, cap4) == 1 && panel_waves(16385, 4, cap1, cap4) == 4);
    CHECK(panel_waves(65537, 4, cap1, cap4) == 4 && panel_waves(131072, 4, cap1, cap4) == 4);
    CHECK(panel_waves(131073, 4, cap1, cap4) == 0);
    // never more workgroups than the device holds, or than the lanes have candidates for
    for (int c1 : {0, 100, 1024})
        for (int c4 : {0, 70, 256, 512, 4096})
            for (size_t entry : {size_t(4), size_t(8)})
                for (int rows = 1; rows < 200000; rows += 61) {
                    const int w = panel_waves(rows, entry, c1, c4);
                    if (!w) continue;
                    const int g = (rows + 64 * w - 1) / (64 * w);
                    CHECK(g <= (w == 1 ? c1 : c4) && g <= 64 * panel_key_sets(w, entry));
                    // candidates of both parities, their rows and row c of every panel of an n = rows matrix
                    const size_t W = entry / 4;
                    CHECK(panel_words(rows, (int)W) >= 2 * (W + 1) * g + 2 * g * W * kNB + 2 * W * kNB);
                }
    // a smaller panel of a larger matrix stays within that matrix's words
    for (int n = 64; n < 140000; n += 977)
        for (int rows = n; rows > 0; rows -= 64 * 37) CHECK(panel_words(rows, 2) <= panel_words(n, 2));
    std::printf("%s\n", failures ? "FAIL" : "checks passed");
    return failures != 0;
}
