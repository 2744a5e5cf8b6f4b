// Where the workgroups of a bf16 prefill launch go when the key splits are merged inside the
// kernel; the dense layers' split-K launches place their workgroups the same way (unit = block of
// output features, split = share of the input features).  Shared by the kernels, the launchers
// and a host-side test (plain C++, no HIP types).
//
// The merge goes through the L2 cache that the compute units of one XCD share, so all splits
// of a unit = (KV head, frame, row tile) must run on one XCD; which one does not matter, and it changes: a
// stream's ids start at another XCD once the process has used more streams or a graph.  The hardware deals
// workgroup ids to the XCDs in turn (id mod number of XCDs; read off the device once, and checked again by
// every unit of every launch, see arrival_of).  Unit u therefore takes the ids of one residue x:
//     x = u / units_per_xcd,  j = u % units_per_xcd,  id = x + ((j * nsplit + split) << xcd_shift)
// with units_per_xcd = ceil(units / 2^xcd_shift); consecutive units (the same KV head, whose K/V
// that L2 then holds once) share an XCD.  Ids whose unit does not exist are spare and return.
// (Launches that leave units whole beside split ones use the same map, for that L2 alone: a second kernel merges them.)
#pragma once

#ifdef __HIPCC__
#define VS_HD __host__ __device__ __forceinline__
#else
#define VS_HD inline
#endif

namespace vs {

// floor(x / d) for 0 <= x < 2^22 and d >= 1, given inv_d = 1.0f / d: the float product is within
// one of the quotient, two corrections make it exact.  (A 32-bit integer division costs some
// twenty instructions on the device, and the prologue of the prefill kernel is on its critical
// path.)
VS_HD int div_small(int x, int d, float inv_d) {
    int qd = (int)((float)x * inv_d);
    if (qd * d > x) --qd;
    if ((qd + 1) * d <= x) ++qd;
    return qd;
}

// The same in two scalar instructions: floor(x / d) = floor(2 x m / 2^32) with m = floor(2^31 / d) + 1 worked out by the host,
// exact while 0 <= x and x d < 2^31 (m d exceeds 2^31 by at most d, the product 2 x m / 2^32 the quotient by at most x / 2^31 < 1 / d).
struct QuickDiv {
    unsigned m;
};
VS_HD QuickDiv quick_div(int d) { return QuickDiv{(1u << 31) / (unsigned)d + 1u}; }
VS_HD int div_by(int x, QuickDiv by) { return (int)(((unsigned long long)(2u * (unsigned)x) * by.m) >> 32); }

// What a workgroup on XCD `xcc` adds to its unit's arrival word: itself, its XCD and the square of that, each
// with room for 32 workgroups and 16 XCDs.  With n workgroups in, the word is n * arrival_of(x) if and only if all of
// them ran on XCD x (n numbers whose sum is n x and whose squares' sum is n x^2 are all x).
VS_HD unsigned arrival_of(unsigned xcc) { return 1u | xcc << 6 | (xcc * xcc) << 16; }
VS_HD unsigned arrivals_in(unsigned word) { return word & 63u; }

struct PrefillSlot {
    int unit;   // -1: a spare id
    int split;
    int xcd;    // residue of the id: which XCD of the dealing order it lands on
};

VS_HD int prefill_units_per_xcd(int units, int xcd_shift) { return (units + (1 << xcd_shift) - 1) >> xcd_shift; }

VS_HD unsigned prefill_grid_ids(int units, int nsplit, int xcd_shift, int whole = 0) {
    return (unsigned)(whole + (prefill_units_per_xcd(units, xcd_shift) - whole) * nsplit) << xcd_shift;
}

VS_HD PrefillSlot prefill_slot(unsigned id, int units, int units_per_xcd, int j, int split, int xcd_shift) {
    PrefillSlot s;
    s.xcd = (int)(id & ((1u << xcd_shift) - 1u));
    s.split = split;
    s.unit = s.xcd * units_per_xcd + j;
    if (j >= units_per_xcd || s.unit >= units) s.unit = -1;
    return s;
}

VS_HD PrefillSlot prefill_slot_of_id(unsigned id, int units, int units_per_xcd, int nsplit, float inv_nsplit,
                                     int xcd_shift) {
    const int slot = (int)(id >> xcd_shift), j = div_small(slot, nsplit, inv_nsplit);
    return prefill_slot(id, units, units_per_xcd, j, slot - j * nsplit, xcd_shift);
}

// The first `whole` units of every XCD may be left whole, a workgroup each, which come first; the others are split nsplit ways.
// (whole must be 0 where ids are not dealt by residue: a unit's place below is worked out from the XCD its id says.)
VS_HD PrefillSlot prefill_slot_of_id(unsigned id, int units, int units_per_xcd, int nsplit, QuickDiv by_nsplit, int xcd_shift,
                                     int whole) {
    const int slot = (int)(id >> xcd_shift), behind = slot - whole;
    const int jj = behind < 0 ? behind : div_by(behind, by_nsplit);
    return prefill_slot(id, units, units_per_xcd, whole + jj, behind < 0 ? 0 : behind - jj * nsplit, xcd_shift);
}

// A split unit's place among those that are split: 0 .. (units_per_xcd - whole) * XCDs - 1.
VS_HD int prefill_part_of_unit(int unit, int xcd, int whole) { return unit - whole * (xcd + 1); }
VS_HD int prefill_unit_of_part(int part, int units_per_xcd, int whole) { return part + whole * (part / (units_per_xcd - whole) + 1); }

}  // namespace vs
