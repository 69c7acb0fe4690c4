// Integer rules that kernels and launchers share: who writes what, which index is read.  No device code and no HIP types, so
// that the same functions can be compiled and enumerated on the host (tests/test_kernel_rules.py).
#pragma once
#include <stddef.h>

#if defined(__HIPCC__)
#define SSD_HD __host__ __device__ __forceinline__
#else
#define SSD_HD inline
#endif

namespace ssdk {

// 16-row kernels, eight waves: the rows whose RMS scale wave `wave` writes.  Every row of the tile belongs to one wave.
template <typename F> SSD_HD void rows_of_wave(int wave, F&& f)
{
    for (int c = wave; c < 16; c += 8) f(c);
}

// Row of the embedding table that is read for token id `tok`, whatever the id holds: a caller's id, or the 0x7fffffff of a
// row of logits without a maximum.
SSD_HD size_t embed_row(int tok, int V) { return (size_t)(tok < 0 ? 0 : tok < V ? tok : V - 1); }

}  // namespace ssdk
