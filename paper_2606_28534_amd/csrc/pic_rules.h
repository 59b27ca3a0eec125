// pic_rules.h -- host rules of the launches that can be looked at without a GPU.
#pragma once
#include <cstdint>

namespace pic {

// How a pass moves the particle arrays: cached, cached loads and non-temporal stores, or both
// non-temporal.
enum Access : int { AC_CACHED = 0, AC_STORES = 1, AC_STREAM = 2 };

// In place over more particle data than the 256 MB last-level cache holds, non-temporal streams are
// faster; over less than that they throw away what the next pass finds cached.  The lines, in slots
// in use, and how many of them `slots` reach:
constexpr int64_t kStreamSlots[4] = {10'000'000, 14'000'000, 16'500'000, 21'000'000};
inline int stream_lines(int64_t slots)
{
    int n = 0;
    for (const int64_t line : kStreamSlots) n += slots >= line ? 1 : 0;
    return n;
}

// The FP32 pass's access: of the fused pass with collisions (`coll`) or of a push with or without a
// deposit, with `ppt` particles a thread.  Per step, cached, with non-temporal stores, and with both:
// the fused pass 103.0, 104.5 and 105.5 us at 9e6 particles, 120.6, 118.8 and 117.4 at 1e7, 152, 150 and
// 143 at 1.4e7, 228, 226 and 192 at 2e7, 320, 318 and 267 at 3e7, and with eight a thread 143, 142 and
// 158 at 1.3e7, 196, 165 and 185 at 1.6e7, 253, 228 and 231 at 2.1e7, 284, 275 and 258 at 2.4e7.  The push
// alone (40 of the 44 B) 75.9, 85.4 and 97.4 at 1.3e7, 82.1, 79.4 and 95.8 at 1.4e7, 105.6, 102.5 and
// 115.6 at 1.6e7, 117.9, 115.8 and 115.0 at 1.7e7, 160, 159 and 137 at 2e7, with eight 94.5, 96.1 and 116
// at 1.5e7, 107.7, 102 and 124 at 1.6e7, 162.8, 158 and 153 at 2e7; the pass without collisions turns at
// the same sizes.  A kernel that held more than one form and chose by itself cost every tile (70.5 ->
// 71.7 to 75.4 us a pass at 9.2e6 particles, or folded them into one), so the host chooses, from the
// slots in use as it last saw them (where it waits for the run).  `always` (bit 0 of `nontemporal`)
// streams at any size where the fused pass leaves its candidates to a launch behind it; everywhere
// else small runs lost to it (the pass with candidates inside up to 18%), and the size decides.
inline Access pass32_access(bool coll, bool inside, int ppt, int lines, bool always)
{
    if (always && coll && !inside) return AC_STREAM;
    if (ppt == 4 && coll) return lines >= 1 ? AC_STREAM : AC_CACHED;
    if (ppt == 4) return lines >= 3 ? AC_STREAM : lines >= 2 ? AC_STORES : AC_CACHED;
    return lines >= 4 ? AC_STREAM : lines >= 2 ? AC_STORES : AC_CACHED;
}

// Whether the FP64 push streams.
inline bool pass64_streams(int lines) { return lines >= 1; }

}  // namespace pic
