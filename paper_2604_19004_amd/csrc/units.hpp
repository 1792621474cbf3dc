// Which unit of rows a workgroup of k_placed_wave has (placed.hip).  Plain C++: also what the host's rules are tested by.
#pragma once

#include <cstdint>

namespace ocean {

constexpr int XCD_COUNT = 8, XCD_UNITS = 8;         // XCDs of the whole chip; neighbouring units that go to one of them
constexpr int UNIT_GROUP = XCD_COUNT * XCD_UNITS;   // units among which the order is changed
constexpr int CUS_PER_XCD = 32;

// The hardware deals workgroups to the XCDs in turn, and each XCD starts those dealt to it in their order.  Where there are eight,
// of every 64 units eight neighbours go to one XCD, whose L2 then has the rows of B (and the lines of A and C) that they share:
// clustered input 1.96 -> 1.93 ms, rectangular 1.240 -> 1.222.  On an XCD units still start in ascending order, so the lowest
// unit that has not finished runs, or is the next that its XCD starts, however few workgroups the chip has room for.  A device of
// fewer XCDs (a partition of the chip) would start them out of order, and a unit that waits for lower ones could keep them from
// starting: there every workgroup has the unit of its own number.
constexpr bool units_by_xcd(int compute_units) { return compute_units == XCD_COUNT * CUS_PER_XCD; }

// The unit of the workgroup that is number `workgroup` of those with units.  (Inlined before anything else: left to the compiler's
// own choice it moved the kernel around it by nine spilled registers, clustered input 1.91 -> 2.00 ms.)
__attribute__((always_inline)) constexpr int64_t unit_of_workgroup(int64_t workgroup, int64_t units, bool by_xcd)
{
    static_assert(XCD_COUNT == 8 && XCD_UNITS == 8, "three bits each");
    const int64_t base = workgroup & ~(int64_t)(UNIT_GROUP - 1);
    if (by_xcd && base + UNIT_GROUP <= units) workgroup = base + (workgroup & 7) * 8 + ((workgroup >> 3) & 7);
    return workgroup;
}

}  // namespace ocean
