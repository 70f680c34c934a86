// launch_rules.h -- how work is cut into launches and workgroups, by sizes
// alone (host code only).
#pragma once
#include <algorithm>
#include <cstdint>

namespace bsmm {

// Output tiles [0, whole) take all of k in one workgroup each, the other
// tiles `splits` parts of `kt_per` k steps (the last one what is left).
struct DenseParts {
    int64_t whole, splits, kt_per;
};

// Fewest parts of k for `tiles` output tiles of `ktiles` k steps on `slots`
// resident workgroups.  An element of a part is one chain of sums, whose error
// grows with the square root of its length, so the parts are never longer than
// about two rounds of workgroups make them (each at least 16 k steps), however
// few parts would be faster.  Errors, and a call by itself, with parts chosen by
// time alone and with these:
//   1900 x 1700 x 2300    FP64 1.15e-15 in 393 us,  6.2e-16 in 411
//   2987 x 618 x 5391     FP64 1.25e-15 in 444 us,  7.2e-16 in 485
//                         FP32 6.5e-7 in 256 us,    3.9e-7 in 289
//   1408 x 1408 x 20,000  FP64 2.4e-15,             1.4e-15
inline int64_t fewest_parts(int64_t tiles, int64_t ktiles, int64_t slots) {
    if (tiles >= slots) return 1;
    return std::max<int64_t>(1, std::min((2 * slots + tiles - 1) / tiles, ktiles / 16));
}

// The part count from `fewest` up with the lowest estimated time, *us.  All
// workgroups take ceil(tiles * S / slots) rounds of ceil(ktiles / S) k steps of
// step_us each (FP64 4, FP32 2), plus about three for a workgroup's start and
// end; S > 1 also writes and reads S partial outputs (tile_bytes each and tile,
// 4.5 TB/s) and takes a launch more.  Each part holds at least eight k steps,
// the partials at most max_bytes.  Two rounds whatever the tile count left the
// last one nearly empty: 1408 x 1408 (121 tiles) with k = 247,808 took 19.0 ms
// in 9 parts (2.13 rounds, three in effect) and takes 15.0 ms in 21.
inline int64_t gemm_splits(int64_t tiles, int64_t ktiles, int64_t slots, int64_t tile_bytes, int64_t max_bytes,
                           double step_us, int64_t fewest, double *us) {
    const int64_t part_bytes = tiles * tile_bytes;
    const int64_t most =
        std::max<int64_t>(1, std::min({ktiles / 8, std::max<int64_t>(64, fewest), max_bytes / part_bytes}));
    const int64_t first = std::min(fewest, most);
    int64_t best = first;
    for (int64_t S = first; S <= most; ++S) {
        const int64_t rounds = (tiles * S + slots - 1) / slots;
        double t = (double)(rounds * ((ktiles + S - 1) / S + 3)) * step_us;
        if (S > 1) t += 2.0 * (double)(S * part_bytes) / 4.5e6 + 8.0;
        if (S == first || t < 0.98 * *us) {
            best = S;
            *us = t;
        }
    }
    return best;
}

// All tiles in parts of k, or the full rounds' tiles whole and only the rest
// in parts (a launch more, about 8 us): N = 3000 (576 tiles, 512 slots) 1.11 ->
// 1.04 ms, N = 6000 (2209) 6.98 -> 6.61, FP32 2900 (529) 0.59 -> 0.54.  Dealing
// the k steps evenly to the workgroups instead filled every round, but put
// neighbours at different k: 1,408 x 1,408 x 247,808 13.9 -> 16.3 ms.
inline DenseParts dense_parts(int64_t tiles, int64_t ktiles, int64_t slots, int64_t tile_bytes, int64_t max_bytes,
                              double step_us) {
    const int64_t rest = tiles % slots;
    double all = 0.0, some = 0.0;
    DenseParts d{0, gemm_splits(tiles, ktiles, slots, tile_bytes, max_bytes, step_us,
                                fewest_parts(tiles, ktiles, slots), &all), ktiles};
    if (rest && rest < tiles) {
        const int64_t r = gemm_splits(rest, ktiles, slots, tile_bytes, max_bytes, step_us, 1, &some);
        some += (double)(tiles / slots * (ktiles + 3)) * step_us + 8.0;
        if (r > 1 && some < 0.98 * all) {
            d.splits = r;
            d.whole = tiles - rest;
        }
    }
    if (d.splits == 1) {
        d.whole = tiles;
        return d;
    }
    d.kt_per = (ktiles + d.splits - 1) / d.splits;
    d.splits = (ktiles + d.kt_per - 1) / d.kt_per;  // no empty part
    return d;
}

// log2 of the entries of a schedule of n runs that go to one XCD in a row: 256
// entries from 16,384 runs on, below that as many as leave each XCD eight
// segments, at least four entries (the largest piece that a wave takes).  With
// 256 always, up to 256 runs all lay on one XCD, and of 4,225 some XCDs had three
// segments and the others two (plans of nine classes, with 256 and so):
//   16 runs of 8 products   49 and 30 us       900 runs of 24      73 and 50 us
//   144 runs of 8           70 and 31          900 runs of 81     195 and 107
//   196 runs of 81         365 and 100       4,225 runs of 32     141 and 130
//   196 runs of 324       1458 and 326       4,225 runs of 81     278 and 240
inline int schedule_segment_bits(int64_t n, int xcds) {
    int bits = 2;
    while (bits < 8 && n >> (bits + 1) >= 8 * xcds) ++bits;
    return bits;
}

}  // namespace bsmm
