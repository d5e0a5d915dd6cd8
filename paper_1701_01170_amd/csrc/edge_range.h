// Edge positions of a frontier run up to 2^31 - 1; what is added to one of them needs
// more than 32 bits.  Plain C++, so that the host can check it as well.
#pragma once

#include <cstdint>

#if defined(__HIPCC__)
#define GR_RANGE_FN __host__ __device__ inline
#else
#define GR_RANGE_FN inline
#endif

namespace gr {

// First edge of wavefront `wave` in a workgroup's range that starts at `lo`.
GR_RANGE_FN int64_t wave_first_edge(int32_t lo, int wave) { return (int64_t)lo + wave * 64; }

}  // namespace gr
