// Which scoring launches reduce the window's Query states themselves, and how (host code, no GPU).
#pragma once
#include <algorithm>

namespace slim {

// slices: of the (token, head of the group) pairs of an element of the window query, a power of two; 0: the window query has a launch of its own.
// threads: of a workgroup; chunks * slices of them reduce the window, four pairs at a time, the rest of a widened workgroup only waits.
struct WindowPlan { int slices, threads; };

// In the launch, every workgroup reads the whole window and walks its share of the pairs before its first product, so both are bounded: no thread asks for
// its four pairs more than twice (waves are added where there are too few threads), and the windows read are either
//  - few, in a launch whose workgroups all run at once: up to 16 MB of them, 8 MB with more than 32 pairs, whose sums over the slices take longer; or
//  - no more than half of what the workgroup reads in keys, if that is 16 KB at least: then they hide under the keys' way from HBM.
// Replayed as a graph, own launch -> inside (us), bf16 where not said:
//   inside:  scores of 32768 tokens' keys, blocks of 64, 32 / 8 heads of 128, 4 tokens of window 14.5 -> 12.2, 8 tokens 14.6 -> 13.9; 28 / 4 heads, blocks of 128,
//            8 tokens 7.5 -> 7.0; 131072 tokens, blocks of 32, 4 tokens 42.4 -> 39.5; one unit per block of 64, 4 tokens 20.9 -> 15.7 (one wave
//            widened to four); from unit keys 32768 tokens, 4 tokens 6.3 -> 6.2 (16 MB), one unit per block of 64 9.4 -> 5.3, 300 tokens in blocks of 16 8.7 -> 4.5
//   not:     blocks of 8, 8 tokens, 32768 tokens' keys 19.2 -> 31.8, unit keys 10.4 -> 26.6; 131072 tokens' unit keys, blocks of 64, 4 tokens 15.5 -> 19.1; 8 / 1 heads
//            of 64, 131072 tokens, blocks of 64, 8 tokens: keys 10.6 -> 12.4, unit keys 7.4 -> 11.6; 128 pairs, 16 MB 5.2 -> 5.7; 56 pairs, 14 MB 5.6 -> 6.1;
//            keys of 2 KB per workgroup (131072 tokens, 4 / 2 heads of 64, blocks of 8) 11.2 -> 14.0
// Launched one by one the launch that is saved is another 1.5 to 2 us, so the lines lie where the two ways of calling balance.  Unit keys in blocks of 64, 4 tokens, in a graph
// and launched by the host: 24576 tokens (12 MB) 6.2 -> 6.1 and 7.7 -> 6.2, 32768 (16 MB, 4096 waves) 6.2 -> 6.2 and 7.7 -> 6.2, 36864 6.7 -> 7.2 and 7.7 -> 7.3, 49152 6.7 -> 7.3
// and 7.7 -> 7.4, 65536 7.8 -> 9.4 and 7.9 -> 9.4; 28 / 4 heads, 32768 tokens (14 MB, 28 pairs) 5.5 -> 5.9 and 7.6 -> 6.0.  More waves than run at once: blocks of 128, 49152
// tokens (6144 waves, 12 MB) 7.7 -> 8.9 and 7.9 -> 8.9.
constexpr int kWinPairs = 64, kWinRounds = 2;
constexpr long long kWinWaves = 4096;                    // 16 per CU: what certainly runs at once
constexpr long long kWinRead = 16ll << 20, kWinReadMany = 8ll << 20;
constexpr long long kWinKeys = 16ll << 10;

// elems: of the window query; vec: of a 16-byte chunk; group: query heads per kv head; nb workgroups of `waves` waves; key_bytes: of the keys that each
// reads (0: stored unit keys, which are too few to hide anything).
inline WindowPlan window_plan(int elems, int vec, int w, int group, int nb, int waves, long long key_bytes) {
    const WindowPlan own_launch{0, 64 * waves};
    const long long chunks = elems / vec, pairs = (long long)w * group, bytes = pairs * chunks * 16;
    if (elems > 1024 || pairs > kWinPairs) return own_launch;
    int slices = 1;
    while (4 * kWinRounds * slices < pairs) slices *= 2;
    const int threads = (int)std::max<long long>(64 * waves, (chunks * slices + 63) / 64 * 64);
    const bool at_once = threads <= 1024 && (long long)nb * (threads / 64) <= kWinWaves && nb * bytes <= (pairs <= 32 ? kWinRead : kWinReadMany);
    const bool hidden = threads == 64 * waves && key_bytes >= kWinKeys && 2 * bytes <= key_bytes;
    if (!at_once && !hidden) return own_launch;
    while (4 * slices < pairs && 2 * slices * chunks <= threads) slices *= 2;
    return {slices, threads};
}

}   // namespace slim
