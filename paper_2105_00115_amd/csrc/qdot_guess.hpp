// Long vectors: when a sample's counts are trusted to select the whole's
// classes (qdot_fused.hip).  The answer decides how much is read, never what
// is returned.
//
// What a wrong guess costs is the sums made for it (2^27 products: 854 us, 700
// where none is made, 381 when it stands; 5e7: 309, 275, 172), so it has to be
// the likelier side by a margin.  Uniform, normal and family B vectors and sums
// that cancel, at six lengths from 2^24 to 2^27: within 1 % of two passes by the
// four-kernel chain (floats 3 %) or up to 1.7 times faster, none slower.
#pragma once
#include <cmath>

#include "qdot_blocks.hpp"

namespace qd {

// Whether the sample's top bin is likely the whole's.  c0, c1, ... are the
// counts of its highest slots, going down; the next slot up would hold about
//   geo   if the ratios of neighbours go on changing as they did,
//   soft  if their logarithms do, as in the tail of a normal law or of its
//         products, which falls ever faster.
// A sample that should have seen four components there and did not has seen
// the end of the range; both estimates have to say so, and the counts must be
// large enough to mean something.  So does a range that ends in a straight
// line (products of two log-uniform factors, sums of two uniform exponents):
// no bend over three slots beyond three standard deviations, and the line
// reaches zero inside the top slot.  Or the whole would not have it either.
__host__ __device__ inline bool top_holds(const unsigned int *h, int top, int up)
{
    const auto c = [&](int i) { return top >= i ? (float)h[top - i] : 0.0f; };
    const float c0 = c(0), c1 = c(1), c2 = c(2), c3 = c(3);
    if (c1 == 0.0f) return c0 >= 4096.0f;
    const float r1 = c0 / c1;
    const float geo = c2 == 0.0f ? c0 * r1 * r1 : c0 * r1 * (r1 * c2 / c1);
    if (ldexpf(geo, up) < 0.02f) return true;
    if (c0 < 32.0f) return false;
    float next = geo;
    if (c0 < c1 && c1 < c2) {
        const float d1 = logf(c1 / c0), d2 = logf(c2 / c1);
        next = fminf(next, c0 * expf(-d1 * d1 / d2));
    }
    if (next >= 4.0f) return true;
    if (!(c3 > c1)) return false;
    const float bend = c1 - 2.0f * c2 + c3, slope = 0.5f * (c3 - c1);
    return bend * bend <= 9.0f * (c1 + 4.0f * c2 + c3) && c1 > 0.5f * slope && c1 < 2.0f * slope;
}

// A slot that the sample saw this often has no neighbour that it missed, and
// its count an error that can be told.
constexpr unsigned int GUESS_SEEN = 16;

// The risks of all slots that are still taken (0.25, in 2^-16).  Over 34 laws
// (log-uniform, uniform, normal, exponential, log-normal, families A and B,
// constants, integers and mixtures), three lengths (2^24, 5e7, 2^27), 6 to 24
// seeds each and six tolerances, 0.2 % of the calls sum for nothing and 41 % by
// classes that stand; by the top and t alone 8 % and 45 %, most of the misses on
// uniform and normal vectors and on sums that cancel.  0.5 gives 0.5 and 41 %.
constexpr int GUESS_RISK = (int)(0.25 * 65536);

// The chance, in 2^-16, that the whole has another class at a slot than the
// sample's count m (cl: ceil(log2 m), 0 for none) selects: that the count it
// stands for lies beyond the next power of two, where that changes the class.
// Certain for rare counts.  score: that of a count of 1 there, plus log2 of the
// sample's inverse share.  m = 0: a slot beside the rare ones, which the whole
// may hold.
__host__ __device__ inline int slot_risk(unsigned int m, int cl, int score, int nonstrict,
                                         int mu_single)
{
    const auto cls = [&](int sigma) {
        const int c = class_of(sigma, nonstrict);
        return mu_single && c == QDOT_DOUBLE ? SINGLE_IN : c;
    };
    const int sigma = score + cl, c = cls(sigma);
    if (m == 0u) return c != QDOT_PERF ? 1 << 16 : 0;
    if (m < GUESS_SEEN) return cls(sigma - 1) != c || cls(sigma + 1) != c ? 1 << 16 : 0;
    const float f = (float)m, above = ldexpf(1.0f, cl), sd = sqrtf(f + 1.0f);
    const auto chance = [&](float d) { return (int)(32768.0f * erfcf(0.70710678f * d / sd)); };
    return (cls(sigma - 1) != c ? chance(f - 0.5f * above) : 0) +
           (cls(sigma + 1) != c ? chance(above - f) : 0);
}

}  // namespace qd
