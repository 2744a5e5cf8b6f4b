// Host-side check of the workgroup id -> (unit, split, XCD) mapping of the bf16 prefill launch and of
// the dense layers' split-K launches (vs_prefill_map.h; there unit = block of output features, split =
// share of the input features), for every (units, splits, number of XCDs) the launch planners can emit:
// every (unit, split) pair is named by exactly one id of the grid, all splits of a unit carry
// ids of one residue modulo the number of XCDs, spare ids name no unit, and units that follow
// one another share a residue as long as that XCD has room; and that an arrival word tells arrivals from one XCD from all others.
#include <cstdio>
#include <vector>

#include "vs_prefill_map.h"

int main() {
    long checked = 0;
    for (int shift = 0; shift <= 4; ++shift) {
        for (int nsplit = 1; nsplit <= 32; ++nsplit) {
            const float inv_nsplit = 1.0f / (float)nsplit;
            for (int units = 1; units <= 1100; units += (units < 300 ? 1 : 37)) {
                const int upx = vs::prefill_units_per_xcd(units, shift);
                const unsigned ids = vs::prefill_grid_ids(units, nsplit, shift);
                if (ids != (unsigned)(upx * nsplit) << shift || upx * (1 << shift) < units) {
                    std::printf("grid too small: units %d nsplit %d shift %d\n", units, nsplit, shift);
                    return 1;
                }
                std::vector<int> seen((size_t)units * nsplit, 0), residue(units, -1);
                for (unsigned id = 0; id < ids; ++id) {
                    const vs::PrefillSlot s = vs::prefill_slot_of_id(id, units, upx, nsplit, inv_nsplit, shift);
                    if (s.xcd != (int)(id & ((1u << shift) - 1u))) { std::printf("residue\n"); return 1; }
                    if (s.unit < 0) continue;
                    if (s.unit >= units || s.split < 0 || s.split >= nsplit) { std::printf("range\n"); return 1; }
                    if (s.unit / upx != s.xcd) { std::printf("unit %d not on XCD %d\n", s.unit, s.xcd); return 1; }
                    ++seen[(size_t)s.unit * nsplit + s.split];
                    if (residue[s.unit] < 0) residue[s.unit] = s.xcd;
                    if (residue[s.unit] != s.xcd) {
                        std::printf("unit %d on two XCDs (units %d nsplit %d shift %d)\n", s.unit, units, nsplit, shift);
                        return 1;
                    }
                }
                for (size_t i = 0; i < seen.size(); ++i)
                    if (seen[i] != 1) {
                        std::printf("(unit, split) %zu named %d times (units %d nsplit %d shift %d)\n", i, seen[i], units,
                                    nsplit, shift);
                        return 1;
                    }
                ++checked;
            }
        }
    }
    // div_small against the integer division over its whole stated range of use
    for (int d = 1; d <= 64; ++d)
        for (int x = 0; x < (1 << 22); x += (x < 70000 ? 1 : 4093))
            if (vs::div_small(x, d, 1.0f / (float)d) != x / d) { std::printf("div_small(%d, %d)\n", x, d); return 1; }
    // Arrival words: n arrivals add up to n times that of XCD x only if all of them came from x (with both sums equal, the
    // squares of the differences to x add up to 0), and nothing runs over into the next field.  Checked for every
    // mixture of up to three XCDs, and for all words of five arrivals.
    auto all_from = [](unsigned word, int n, unsigned x) { return word == (unsigned)n * vs::arrival_of(x); };
    for (int n = 1; n <= 32; ++n)
        for (unsigned x = 0; x < 16; ++x) {
            unsigned word = 0;
            for (int i = 0; i < n; ++i) {
                if (i && (vs::arrivals_in(word) != (unsigned)i || !word)) { std::printf("arrivals\n"); return 1; }
                word += vs::arrival_of(x);
            }
            if (vs::arrivals_in(word) != (unsigned)n || !all_from(word, n, x)) { std::printf("all from %u\n", x); return 1; }
            for (unsigned y = 0; y < 16; ++y)
                for (unsigned z = 0; z < 16; ++z)
                    for (int a = 0; a <= n; ++a)
                        for (int b = 0; a + b <= n; ++b) {
                            const int c = n - a - b;
                            const bool same = (!a || (!b || x == y)) && (!a || !c || x == z) && (!b || !c || y == z);
                            const unsigned w = a * vs::arrival_of(x) + b * vs::arrival_of(y) + c * vs::arrival_of(z);
                            if (vs::arrivals_in(w) != (unsigned)n) { std::printf("count\n"); return 1; }
                            for (unsigned t : {x, y, z})
                                if (!same && all_from(w, n, t)) { std::printf("%u %u %u taken for %u\n", x, y, z, t); return 1; }
                        }
        }
    for (unsigned code = 0; code < (1u << 20); ++code) {
        unsigned w = 0;
        bool same = true;
        for (int i = 0; i < 5; ++i) {
            w += vs::arrival_of(code >> (4 * i) & 15u);
            same = same && (code >> (4 * i) & 15u) == (code & 15u);
        }
        for (unsigned t = 0; t < 16; ++t)
            if (all_from(w, 5, t) != (same && t == (code & 15u))) { std::printf("five arrivals %x\n", code); return 1; }
    }
    std::printf("ok %ld\n", checked);
    return 0;
}
