// Sizes of the thickness-derivative buffers: host arithmetic without HIP, so that
// it also compiles into tests that run without a GPU.
#pragma once
#include <algorithm>

namespace hfd {

// Both buffers only grow over the geometries that a plan is given.  `slots`
// (offsets per table) is the slot count of the derivative spectra and the stride
// of the offset tables; `offsets` the values that the device copy of those
// tables holds.  The number of tables depends on the geometry as well, not on
// n_geom alone (stacks share a table while their offsets fit in it), so a
// geometry with no more offsets per table can still need more of them in all.
struct DerivativeSizes {
    int slots = 0;
    long long offsets = 0;
};

// sizes that hold `tables` tables of at most `most` offsets, from those in hand
inline DerivativeSizes derivative_sizes(DerivativeSizes have, int tables, int most)
{
    DerivativeSizes s;
    s.slots = std::max(have.slots, most);
    s.offsets = std::max(have.offsets, (long long)tables * s.slots);
    return s;
}

// Bytes from the start of a row of the derivative spectra ([slots][6][QY] values)
// that a buffer descriptor reaches: offsets stay below 2^31, as those of the
// tensor table do.  One row per descriptor is what any call needs (more is
// refused); the staged kernel reads the rows kx = 0 and kx = Lx/2 of its packed
// column through one descriptor, so that it takes calls where both fit, and the
// unstaged kernel, with a descriptor per row, takes the others.
constexpr long long kDescriptorBytes = 1LL << 31;
inline bool derivative_rows_fit(int rows, long long slots, long long QY, long long value_bytes)
{
    return rows * slots * 6 * QY * value_bytes < kDescriptorBytes;
}

}  // namespace hfd
