// Bins of the histogram that finds a quantile among the block sums of a large grid.
#ifndef SPION_GRID_BINS_H_
#define SPION_GRID_BINS_H_

#include <hip/hip_runtime.h>

namespace spion {

// Ordered like the values.  One workgroup selects from the cells of the bin that holds the wanted rank, beside the fill, which
// covers for some 16000 of them; 100000 cost 50 us.  So the bins are fine for any scale and sign that the maps may have; to
// an octave: 128 from 2^32 on (a block's sum of scores of 2^-8 in all, where the sums of even maps lie), 64 below, 32 of negative
// values.  Median of 8192 x 8192, block 16, in us, with 32 to an octave throughout, with 128 from 2^32 on and one to an
// octave elsewhere, and so: softmax of band and stripes raised by 4, 163 / 106 / 109; by 6, 146 / 251 / 115; by 8, 132 / 277 / 106.
constexpr int kGridBins = 8192;
constexpr int kGridZeroBin = 63 * 32 + 1;   // -2^63 is the one value of its octave
constexpr int kGridFineFrom = 32;           // the octave
static_assert(kGridZeroBin + 1 + kGridFineFrom * 64 + (63 - kGridFineFrom) * 128 <= kGridBins, "bins of the positive octaves");

__host__ __device__ inline int grid_bin(long long v) {
    if (v == 0) return kGridZeroBin;
    const unsigned long long m = v < 0 ? 0ull - (unsigned long long)v : (unsigned long long)v;
    const int lz = __builtin_clzll(m), octave = 63 - lz;
    const unsigned long long rest = m << lz << 1;   // the bits behind the leading one
    if (v < 0) return kGridZeroBin - 1 - (octave * 32 + (int)(rest >> 59));
    const int first = kGridZeroBin + 1;
    return octave < kGridFineFrom ? first + octave * 64 + (int)(rest >> 58)
                                  : first + kGridFineFrom * 64 + (octave - kGridFineFrom) * 128 + (int)(rest >> 57);
}

}  // namespace spion
#endif
