// How many workgroups share a tile's pairs (host code, no GPU headers).
#pragma once

#include <stdint.h>

namespace lmkan {

// Microseconds of a launch whose `tiles` are split `split` ways over K pairs.  A workgroup fills a CU and walks
// its pairs one after the other, a slab fill and a barrier each (about 3.5 us), so a launch lasts as many
// such steps as rounds of 256 workgroups times pairs per split, two more per round for the tile's own loads
// and stores.  A forward split beyond the first writes a part of its own that is added up later (part_bytes
// each, moved twice); the input gradient adds atomically and passes 0.
inline double pair_split_us(int64_t rounds, int pairs, int split, int64_t part_bytes)
{
    return 3.5 * (double)rounds * (pairs + 2) + (split - 1) * (double)part_bytes * 2 / 4.9e6 +
           (split > 1 && part_bytes ? 5.0 : 0.0);
}

// Pair splits for a launch of `tiles` workgroups over K pairs.  Few tiles want more splits to have
// work for every CU, and a count a little above a multiple of 256 wastes most of its last round: the
// split is the one with the least time, of those with at least four pairs in each and of `most` at most.
// (500 -> 333 outputs at G = 20 on 5000 rows, 33 tiles of 250 pairs: 8 splits make 264 workgroups and
// two rounds of 32 pairs, 7 make 231 in one round of 36: forward 254 -> 157 us, grad_x 261 -> 212 us.)
// Of the splits with the same pairs in each the smallest is the quickest, so only those are looked at: from
// the one that makes a single round of the chip, or the first that has so few pairs that it could be quicker, to
// where the shares of a full chip and the parts alone take longer than the best.  (Every count from 1 to
// K / 4 in turn took 5 us at 8192 inputs and 70 us at 131070, in every query of a workspace size.)
inline int pair_split_count(int64_t tiles, int K, int64_t part_bytes, int most)
{
    if (most > K / 4) most = K / 4;
    const double part_us = (double)part_bytes * 2 / 4.9e6, shares = 3.5 / 256 * (double)tiles;  // of a step that all CUs take
    const auto pairs_of = [K](int split) { return (K + split - 1) / split; };
    const auto us_of = [&](int split) { return pair_split_us((tiles * split + 255) / 256, pairs_of(split), split, part_bytes); };
    const auto first_with = [K](int pairs) { return (K + pairs - 1) / pairs; };
    int best = 1;
    double best_us = us_of(1);
    if (most < 2) return best;
    const int round = tiles < 128 ? (int)(256 / tiles) : 2, one = first_with(pairs_of(round < most ? round : most));
    if (us_of(one) < best_us) best = one, best_us = us_of(one);
    // (bounds a little lower for rounding; a bound of `few` pairs holds for a single round, more take longer)
    const double few = best_us / (3.5 * 0.999) - 2;
    int split = few < K / 2 ? first_with(pairs_of((int)(K / few))) : 2;
    for (; split <= most; split = first_with(pairs_of(split) - 1)) {
        const double us = us_of(split);
        if (us < best_us || (us == best_us && split < best)) best = split, best_us = us;
        if (0.999 * (shares * (K + 2 * split) + (split - 1) * part_us) > best_us) break;
    }
    return best;
}

}  // namespace lmkan
