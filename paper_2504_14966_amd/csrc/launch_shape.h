// Workgroup shapes of the kernels that keep a block of LDS per chain behind records shared by the
// workgroup. Host arithmetic only, with no HIP in it.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace sa {

struct LdsShape {
  int fit;    // chains per workgroup that the LDS holds, at most 16 (0: not even one)
  int waves;  // chains per workgroup of the launch
};

// The launch takes no more chains per workgroup than spread them evenly over the CUs in as many
// passes as the LDS makes necessary (1500 chains: 250 workgroups of 6; in 188 workgroups of 8 a
// quarter of the CUs idled).
inline LdsShape lds_shape(int chains, size_t shared, size_t per, int lim, int cus) {
  if (shared + per > (size_t)lim) return LdsShape{0, 0};
  const int64_t fit = std::min<int64_t>(16, ((int64_t)lim - (int64_t)shared) / (int64_t)per);
  const int64_t passes = (chains + fit * cus - 1) / (fit * cus);
  return LdsShape{(int)fit, (int)((chains + passes * cus - 1) / (passes * cus))};
}

// Whether the LDS gives the delta kernels of fixed-size batches enough chains at once: four per
// CU (one per SIMD), or every chain in one pass. What counts is what the LDS holds, not the
// spread: 1500 chains where five fit go as 500 workgroups of three.
inline bool lds_suffices(const LdsShape &s, int chains, int cus) {
  return s.fit >= 4 || (s.fit > 0 && (int64_t)s.fit * cus >= chains);
}

}  // namespace sa
