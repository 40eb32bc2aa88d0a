// Index arithmetic of walks over rows, in plain C++ (constexpr functions are
// host and device functions both), so that it can be checked on the host at
// sizes of which no graph is built for a test.
#pragma once

#include <cstdint>

namespace hg {

// Positions and row numbers are int32 below 2^31; a walk in strides steps past
// its end, by up to a stride, where an int32 would wrap and never end.
typedef uint32_t row_pos;

// for p = beg, beg + step, ... below end
#define HG_ROW_WALK(p, beg, end, step) \
  for (::hg::row_pos p = (::hg::row_pos)(beg); p < (::hg::row_pos)(end); p += (::hg::row_pos)(step))

}  // namespace hg
