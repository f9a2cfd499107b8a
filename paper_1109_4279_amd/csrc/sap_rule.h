// Which of the two even/odd block solvers is the faster one for several right-hand sides on
// 16-bit storage: the time of a half-sweep on either, from how a launch's work falls on the CUs.
//
// An item of the matrix-core kernel (one block, up to four rhs) takes the same time for one to
// four rhs, so tiles that are not full count as full ones.  Its work-groups do one item each:
// rounds of as many as share a CU (eight wavefronts by registers, and the LDS).  The vector
// kernel (one block, one rhs) runs on four persistent work-groups per CU, of which those
// reside that fit the registers (eight wavefronts) and the LDS; the others follow.  The times of
// a round (us, BF16, 4 MR steps) are fits to 2703 half-sweeps timed on 52 block shapes of 8 to 256
// sites, 32 to 8192 blocks, 2 to 12 rhs:
//   vector          28 + 2.8 a resident wavefront.  Above three full rounds the CUs drift
//                   apart, and a round that only some of them have counts by its share.
//   matrix cores    one work-group per CU 44 with up to four wavefronts, 52 + 1.6 each with
//                   more; a full round of several work-groups 57 + 0.4 a wavefront of each
// By them the pick is at most 3 % behind the vector kernel for blocks without an extent of 16
// and more (20 % for some of 1x1x1x32 and 1x1x1x64), and 0.3 % behind the faster one on average.
// Half-sweeps, vector / matrix cores:
//   4^4     256 blocks 83 / 65 (3 rhs), 94 / 71 (4); 648 blocks 139 / 174 (2), 257 / 204 (4),
//           318 / 365 (5); 1296 blocks 1461 / 1070 (12)
//   2x4^3   256 blocks 47 / 47 (3 rhs), 80 / 49 (4); 648 89 / 98 (2), 155 / 101 (3); 1152 170 / 150 (2)
//   4x3^3   256 blocks 51 / 48 (4 rhs), 79 / 62 (5); 648 93 / 98 (2), 135 / 106 (4), 159 / 173 (5);
//           1152 123 / 150 (2), 179 / 155 (3)
//   8x4x2x2 256 blocks 92 / 90 (5 rhs); 648 94 / 130 (2), 163 / 134 (3), 309 / 263 (6)
//   2^4     256 blocks 38 / 36 (3 rhs), 71 / 38 (6); 2048 140 / 57 (2)
#pragma once

#include <algorithm>

namespace wc {

constexpr int SAP_CU_WAVES = 8;  // wavefronts of either kernel that the registers of a CU hold
constexpr int SAP_EO_PER_CU = 4;  // persistent work-groups of the vector kernel per CU

// work-groups of `waves` wavefronts and `lds` bytes that a CU with lds_max bytes holds
inline int sap_resident(int waves, size_t lds, size_t lds_max) {
  return std::max(1, std::min(SAP_CU_WAVES / waves, int(lds_max / lds)));
}

// the vector kernel with `items` items per CU
inline double sap_vec_us(double items, int resident, int waves) {
  auto rounds = [&](int q) {
    int left[SAP_EO_PER_CU];
    for (int j = 0; j < SAP_EO_PER_CU; ++j) left[j] = (q - j + SAP_EO_PER_CU - 1) / SAP_EO_PER_CU;
    for (double t = 0.0;;) {
      int running = 0;
      for (int& l : left)
        if (l > 0 && running < resident) {
          --l;
          ++running;
        }
      if (!running) return t;
      t += 28.0 + 2.8 * running * waves;
    }
  };
  auto time = [&](int q) {  // (every four items more take the same)
    const int k = q / SAP_EO_PER_CU;
    return k < 2 ? rounds(q) : (k - 1) * rounds(SAP_EO_PER_CU) + rounds(SAP_EO_PER_CU + q % SAP_EO_PER_CU);
  };
  const int q = int(items);
  const double part = items - q;
  if (part == 0.0) return time(q);
  return time(q) + (items >= 3 * SAP_EO_PER_CU ? part : 1.0) * (time(q + 1) - time(q));
}

// the matrix-core kernel with at most `items` items on a CU
inline double sap_mm_us(int items, int resident, int waves) {
  const double one = waves <= 4 ? 44.0 : 52.0 + 1.6 * waves;
  const double full = resident == 1 ? one : 57.0 + 0.4 * waves;
  const int rest = items % resident;
  return items / resident * full + (rest ? one + (full - one) * (rest - 1) / (resident - 1) : 0.0);
}

// Whether `mm_items` items on the matrix cores are faster than `vec_items` on the vector units.
// (Up to two items per CU the vector kernel keeps its operator in registers.)
inline bool sap_mm_faster(long long vec_items, int vec_waves, size_t vec_lds, long long mm_items, int mm_waves,
                          size_t mm_lds, size_t lds_max, int cus) {
  if (mm_lds > lds_max || vec_items <= 2LL * cus) return false;
  return sap_mm_us(int((mm_items + cus - 1) / cus), sap_resident(mm_waves, mm_lds, lds_max), mm_waves) <
         sap_vec_us(double(vec_items) / cus, sap_resident(vec_waves, vec_lds, lds_max), vec_waves);
}

}  // namespace wc
