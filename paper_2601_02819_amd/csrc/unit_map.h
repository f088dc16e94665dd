// Which workgroup of the sparse attention kernels takes which work unit.  Plain
// arithmetic, so that a host compiler can build it too (the caller defines
// PHSA_HD).
#pragma once

namespace phsa {

struct UnitAt {
  int bg, idx, u;  // u = bg * per_bg + idx, known before the division
};

// Unit of workgroup lin in a grid of R * per_bg (R = B * Hkv; every (b, g) has
// per_bg units reserved, a multiple of 8, and the first ones exist).  The
// dispatcher hands workgroups to the 8 XCDs in turn, so lin mod 8 is the XCD.
// With c = gcd(R, 8), groups of 8 / c XCDs share R / c (b, g) and take their units
// in turn: one (b, g) at a time meets as few L2s as a fair share allows (its
// query rows and dO rows are gathered once per L2), and the XCDs of a group get
// equal parts of it, the long lists of the first blocks and the reserved units
// that do not exist alike.  A contiguous run of units per XCD, which is the same
// where 8 divides R, gave some XCDs only the long lists elsewhere: forward and
// backward 700 + 1768 against 544 + 987 us (2 x 16k, R = 4, the paper's blocks),
// 372 + 957 against 164 + 342 (1 x 16k, R = 1), 547 + 1388 against 562 + 1176 (5 x
// 8k, R = 20, 64-token blocks).  Plain order (every (b, g) over all XCDs): 586 +
// 1032 and 648 + 1307 for the first and the last of these, 274 + 540 against 224 +
// 510 at 1 x 16k, R = 8.  (A prefix over the counts, so that no workgroup is idle:
// no faster.)
PHSA_HD UnitAt unit_at(int lin, int R, int per_bg) {
  const int lg = (R & 7) == 0 ? 3 : (R & 3) == 0 ? 2 : (R & 1) == 0 ? 1 : 0;  // log2 c
  const int x = lin & 7, j = lin >> 3;
  const int item = (j << (3 - lg)) | (x & ((8 >> lg) - 1));  // in the group's order
  const int first = (x >> (3 - lg)) * (R >> lg), y = item / per_bg;
  return {first + y, item - y * per_bg, first * per_bg + item};
}

}  // namespace phsa
