// Entries of a range taken in batches of fixed size, the last batch of which may reach beyond its end.  Entry numbers go up to INT32_MAX, so
// such a place has no sign: up to 2^31 beyond the end of any range it does not wrap around.  Plain C++, so that it can be looked at on
// the host.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define FTC_HD __host__ __device__
#else
#define FTC_HD
#endif

namespace ftc {

// the entry at place e of the range that ends at `end` (not empty), beyond the end its last one
FTC_HD inline int entry_or_last(uint32_t e, int end) { return e < static_cast<uint32_t>(end) ? static_cast<int>(e) : end - 1; }
FTC_HD inline bool entry_in(uint32_t e, int end) { return e < static_cast<uint32_t>(end); }

}  // namespace ftc
