// The parts of a batch with host outputs (run_pipeline builds and delivers
// them).
#include "mkf_runtime.hpp"

#include <algorithm>

namespace mkf {

// How a batch whose rows go to the host is built: in parts (ends, in rows),
// each part's rows delivered by the launch that builds the next, so that the
// time is that of the longer of the two plus the first part's build and the
// last one's delivery.  Parts end at blocks of kSeedBlock rows.  Chosen among
// one part and sequences that start with a fraction of the rows and grow (for
// rows that take longer to deliver than to build) or shrink, by the time that
// a model of the launches gives, when it is at least 8 % shorter than that of
// one part.  The model: a build takes `t0` (a wavefront's way through the
// layers) plus `row` a seed, both in proportion to 0.45 + 0.55 of the fullest
// layer's hits over 22,000, and 8/7 of it beside a delivery; a delivery takes
// its bytes, a launch 4 us.  Measured with 6 candidates and seven layers built
// (us): thin cylinders of 22,000 hits 10,240 seeds 50, 200,000 328, of 65,000
// hits 10,240 seeds 102, 50,000 213; disks of 11,000 hits 20,000 seeds 82,
// 40,000 104; deep layers of 5,500 hits 20,000 seeds 86, of 22,000 hits 80,000
// 428.  The number of layers is left out: the build goes as its power of 0.8
// (one layer built 0.2 of seven's time, nine 1.22, thirteen 1.64), but scaled
// so the model, whose density is that of inner layers, gives up parts that pay
// (one event of 50,000 seeds and thirteen layers 520 us in parts, 640 in one;
// 4 x 10,000 on disks 418 and 495) and gains 3 % with one layer (5 x 20,000
// 566 and 549).
std::vector<long long> plan_parts(const std::vector<EventLoad> &loads, const Params &P, double us_per_row)
{
    std::vector<long long> block;   // ends of the blocks
    long long rows = 0;
    double hits = 0.0;
    for (const EventLoad &l : loads) {
        for (int b = kSeedBlock; b < l.seeds; b += kSeedBlock) block.push_back(rows + b);
        rows += l.seeds;
        hits += (double)l.seeds * l.layer_hits;
        if (l.seeds > 0) block.push_back(rows);
    }
    std::vector<long long> best{rows};
    if (rows < 2 * kSeedBlock || us_per_row <= 0.0) return best;
    const double dense = 0.45 + 0.55 * hits / (double)rows / 22000.0;
    const double t0 = dense * (P.geo & 2 ? 58.0 : P.geo & 1 ? 55.0 : 33.0);
    const double row = dense * (1.0 + P.max_cands) / 7.0 * (P.geo & 2 ? 4.6e-3 : P.geo & 1 ? 2.2e-3 : 1.48e-3);
    auto time_of = [&](const std::vector<long long> &ends) {
        double t = 0.0, out = 0.0;
        long long at = 0;
        for (long long e : ends) {
            t += 4.0 + std::max((t0 + row * (double)(e - at)) * (at ? 8.0 / 7.0 : 1.0), out);
            out = us_per_row * (double)(e - at);
            at = e;
        }
        return t + 4.0 + out;
    };
    double best_t = 0.92 * time_of(best);
    for (double first : {0.05, 0.1, 0.2, 0.33, 0.5, 0.62, 0.75})
        for (double growth : {0.5, 1.0, 2.0, 3.0}) {
            std::vector<long long> ends;
            double want = first * (double)rows, size = want;
            for (size_t k = 0; k < block.size() && (int)ends.size() + 1 < kBuildParts; ++k) {
                if ((double)block[k] < want && k + 1 < block.size()) continue;
                ends.push_back(block[k]);
                size = std::max(size * growth, (double)kSeedBlock);
                want = (double)block[k] + size;
            }
            if (ends.empty() || ends.back() < rows) ends.push_back(rows);
            const double t = time_of(ends);
            if (t < best_t) {
                best_t = t;
                best = ends;
            }
        }
    return best;
}

// Work items of the first `rows` rows (whole blocks or events) of a batch.
int items_before(const std::vector<EventLoad> &loads, long long rows, int spi)
{
    long long items = 0;
    for (const EventLoad &l : loads) {
        const long long m = std::min<long long>(l.seeds, rows);
        items += (m + spi - 1) / spi;
        rows -= m;
    }
    return (int)items;
}

}  // namespace mkf
