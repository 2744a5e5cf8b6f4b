// Host-side check of the prefill launch's workgroup map where the first units of every XCD are left whole (vs_prefill_map.h):
// every whole unit is named by one id and every (split unit, split) pair by one, the whole units' ids come first, a unit's
// splits carry ids of one residue, and the split units' places in the partial results are all different and in range.
#include <cstdio>
#include <vector>

#include "vs_prefill_map.h"

int main() {
    long checked = 0;
    for (int shift = 0; shift <= 3; ++shift)
        for (int nsplit = 2; nsplit <= 8; ++nsplit)
            for (int units = 1; units <= 900; units += (units < 80 ? 1 : 29)) {
                const int upx = vs::prefill_units_per_xcd(units, shift);
                for (int whole = 0; whole < upx; whole += (whole < 3 ? 1 : 7)) {
                    const unsigned ids = vs::prefill_grid_ids(units, nsplit, shift, whole);
                    const int parts = (upx - whole) << shift;
                    std::vector<int> seen((size_t)units * nsplit, 0), place(parts, -1);
                    for (unsigned id = 0; id < ids; ++id) {
                        const vs::PrefillSlot s = vs::prefill_slot_of_id(id, units, upx, nsplit, vs::quick_div(nsplit), shift, whole);
                        if (s.unit < 0) continue;
                        const bool is_whole = (int)(id >> shift) < whole;
                        if (s.unit >= units || s.unit / upx != s.xcd || (s.unit % upx < whole) != is_whole ||
                            s.split < 0 || s.split >= (is_whole ? 1 : nsplit)) {
                            std::printf("id %u: unit %d split %d (units %d nsplit %d whole %d)\n", id, s.unit, s.split, units, nsplit, whole);
                            return 1;
                        }
                        ++seen[(size_t)s.unit * nsplit + s.split];
                        if (is_whole) continue;
                        const int part = vs::prefill_part_of_unit(s.unit, s.xcd, whole);
                        if (part < 0 || part >= parts || (place[part] >= 0 && place[part] != s.unit)) { std::printf("place\n"); return 1; }
                        place[part] = s.unit;
                        if (vs::prefill_unit_of_part(part, upx, whole) != s.unit) { std::printf("unit of place %d\n", part); return 1; }
                    }
                    for (int u = 0; u < units; ++u)
                        for (int k = 0; k < nsplit; ++k)
                            if (seen[(size_t)u * nsplit + k] != (u % upx < whole && k ? 0 : 1)) { std::printf("unit %d split %d\n", u, k); return 1; }
                    ++checked;
                }
            }
    // div_by against the integer division: every divisor in use, products up to 2^31
    for (int d = 1; d <= 70000; d += (d < 600 ? 1 : 331))
        for (long x = 0; x * d < (1L << 31); x += (x < 4000 ? 1 : 1 + ((1L << 31) / d) / 5000))
            for (long y : {x, x * d, x * d + d - 1})
                if (y * d < (1L << 31) && vs::div_by((int)y, vs::quick_div(d)) != (int)(y / d)) { std::printf("div_by(%ld, %d)\n", y, d); return 1; }
    std::printf("ok %ld\n", checked);
    return 0;
}
