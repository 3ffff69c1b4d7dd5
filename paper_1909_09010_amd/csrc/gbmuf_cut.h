// gbmuf_cut.h -- which floats the fused kernel loads of a tile [lo, lo + n) that component edges cut, where it loads columns
// in 16 bytes.  Plain arithmetic for the device and, in tests, the host.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define GBMUF_CUT_HD __host__ __device__ __forceinline__
#else
#define GBMUF_CUT_HD inline
#endif

namespace gbmuf {

// The column that starts at element e, a multiple of 4.
struct CutColumn {
    unsigned mine;           // bit c: element e + c is the tile's
    int from;                // its load covers elements [e + from, e + from + 4), all of them the tile's (if any is mine)
};

// A tile that loads of 16 bytes cannot read without floats beside it: it has less than 4, or blocks (2^logB floats) are so
// narrow that one ends less than 4 floats after the tile's begin or begins less than 4 before its end.
GBMUF_CUT_HD bool is_thin(int64_t lo, int n, int logB)
{
    const int64_t last = lo + n - 1;
    return n < 4 || (((lo ^ (lo + 3)) | (last ^ (last - 3))) >> logB) != 0;
}

// Of a tile that is not thin.  Floats beside the tile belong to components that need not be due, or to nobody: they are
// not read.
GBMUF_CUT_HD CutColumn cut_column(int64_t e, int64_t lo, int n)
{
    CutColumn c = {0u, 0};
#pragma unroll
    for (int i = 0; i < 4; ++i) c.mine |= e + i >= lo && e + i < lo + n ? 1u << i : 0u;
    if (c.mine) c.from = e < lo ? static_cast<int>(lo - e) : lo + n - 4 < e ? static_cast<int>(lo + n - 4 - e) : 0;
    return c;
}

}  // namespace gbmuf
