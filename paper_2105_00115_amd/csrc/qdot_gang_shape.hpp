// How many blocks each CG system of a batched launch gets (host side, no GPU
// code).
#pragma once
#include <algorithm>
#include <cstdint>

namespace qd {

// ceil(n / rows) blocks for a system of n rows, at most `most`.
struct GangShape {
    int64_t rows;
    int most;
    int size(int64_t n) const
    {
        return (int)std::max<int64_t>(1, std::min<int64_t>(most, (n + rows - 1) / rows));
    }
};

// Launches that may run at the same time, each on a stream of its own, and
// still never hold all resident blocks in gangs that wait for more: a launch
// has at most one such gang.
constexpr int GANG_LAUNCHES = 8;

// The shape for the S systems of sizes n(0), ..., n(S - 1).  tuned: rows per
// block and the largest gang of the tuned shape.  resident: blocks of the
// launch that are on the chip at once; a gang waits for all of its blocks, so
// none is larger.
//
// The tuned shape suits batches whose gangs fill the chip several times over.
// Systems that it would give fewer blocks than are resident share those out
// evenly: the fewest rows per block, a multiple of `chunk`, at which all gangs
// are resident together.  24 Poisson systems of sides 32 to 512, 60 iterations:
// 14.4 ms with the tuned shape (8192 rows, gangs of at most 16, 185 blocks in
// all), 7.2 ms shared out.  A gang that is shared out gets at most a
// GANG_LAUNCHES-th of the resident blocks, or the tuned most.
template <class Rows>
GangShape gang_shape(Rows &&n, int S, GangShape tuned, int64_t resident, int64_t chunk)
{
    const int all = (int)std::max<int64_t>(1, std::min<int64_t>(resident, INT32_MAX));
    tuned.most = std::min(tuned.most, all);
    const int spread = std::max(all / GANG_LAUNCHES, tuned.most);
    for (int64_t rows = chunk; rows < tuned.rows; rows += chunk) {
        const GangShape g = {rows, spread};
        int64_t blocks = 0;
        for (int s = 0; s < S; s++) blocks += g.size(n(s));
        if (blocks <= resident) return g;
    }
    return tuned;
}

}  // namespace qd
