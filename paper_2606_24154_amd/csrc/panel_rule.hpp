// panel_rule.hpp -- which kernel factors a panel of the LU (host code and sizes
// shared with the kernels, no HIP calls).
#pragma once

#include <cstddef>

namespace nebem {

constexpr int kNB = 64;          // LU panel width
constexpr int kPB = 256;         // rows per workgroup of a panel, or
constexpr int kLoneWaves = 256;  // 64 (one wave) while there are at most this many workgroups

// Candidates that a lane reads in a panel of one launch, and with them its most
// workgroups, 64 per candidate: 512 of 256 FP32 rows are what the device holds at
// once (two per CU by their LDS), 256 of FP64 rows.  (With 256 in FP32 too, panels of
// 65 537 to 131 072 rows went column by column, as those of FP64 that do not fit: the
// mixed solve of n = 100 000 took 8.65 s, with them in one launch 7.56.)
constexpr int panel_key_sets(int waves, size_t entry) { return waves == 4 && entry == 4 ? 8 : 4; }

// Waves per workgroup with which a panel of `rows` rows runs as one launch, 0: one
// launch per column.  cap1, cap4: workgroups of one and of four waves that the device
// holds at once.
inline int panel_waves(int rows, size_t entry, int cap1, int cap4)
{
    const int g1 = (rows + 63) / 64, g4 = (rows + kPB - 1) / kPB;
    if (g1 <= kLoneWaves && g1 <= cap1) return 1;
    return g4 <= cap4 && g4 <= 64 * panel_key_sets(4, entry) ? 4 : 0;
}

// 64-bit words that the panels of a factorisation pass values through, each value
// in word_per_value of them
inline size_t panel_words(int n, int word_per_value)
{
    const int g1 = (n + 63) / 64, g4 = (n + kPB - 1) / kPB;
    const size_t G = (size_t)(g1 < kLoneWaves ? g1 : (g4 > kLoneWaves ? g4 : kLoneWaves));
    return 2 * ((size_t)word_per_value + 1) * G + 2 * (G + 1) * (size_t)word_per_value * kNB;
}

}  // namespace nebem
