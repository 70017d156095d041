// Tables with which the encoders find the pattern of least squared error without rating every pattern value by value
// (built on the CPU when a model is uploaded; ecco_rows.h holds the device side).
//
// A value x of a group with scale s is placed on the axis u = x / s by  q = rint(x * (step / s)) + 32768  (16 bits); its
// bin is q >> 8 and its place in the bin q & 255.  For one pattern and one bin the squared distance of u to the nearest
// centroid, less the squared distance to the middle of the bin (which is the same for every pattern), is a concave
// function of u made of straight pieces.  It is replaced by the chord between the bin's ends, moved up by half of the
// largest gap between the two.  A group's squared error under pattern p is then, up to what all patterns share,
//     sum over bins of  n[b] * A[p][b] + m[b] * B[p][b]      n: values in the bin,  m: sum of their places
// with an error of at most  sum of n[b] * E[p][b]: a matrix product of the group's histogram with three tables.
// E holds everything that separates this sum from the FP32 tree sum that decides: half the gap above, the rounding of
// q, of the tables and of m to FP16, of the reconstructed centroids to FP16, and of the FP32 sums themselves.  The
// pattern of least error is therefore always among those whose lower bound does not exceed the least upper bound
// (1.7 of 64 on the weight workloads), and only these are rated exactly.
//
// The second table answers, per pattern and bin, which of two (rarely three) neighbouring centroids can be nearest.  A third
// does so for the min/max selector, which forms no histogram, over bins that are finer around zero (kFineBins).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <vector>

namespace ecco {

constexpr int kSearchBins = 256;
constexpr int kSearchBlocks = 8;        // the matrix product takes the bins 32 at a time
constexpr float kSearchCoefScale = 1024.0f;  // A, B, E are stored times this, in FP16
// the tables hold for scales of at least this (below, the rounding of a reconstructed centroid to a multiple of 2^-24 is
// no longer small against the scale): for other groups the bounds are widened, and the patterns left compared value by value
// (ecco_rows.h)
constexpr float kSearchLeastScale = 0x1p-11f;
// entry of the table of nearest centroids: bits 5:2 the lowest centroid a that can be nearest to a value of the bin
// (the others are a + 1 and, if so marked, a + 2), and two marks
constexpr uint32_t kNearTwo = 1u;   // a + 2 can be nearest as well
constexpr uint32_t kNearWide = 2u;  // more than three: compare with all centroids

// Bins of the min/max selector: t = 2^-7 + kFinePer |u| in FP16, from 2^-7 to below 2, by its four leading mantissa bits -- 16 bins
// to each of 8 octaves, and the sign of u.  Where one channel's magnitude sets the scale (keys) most centroids lie within a few
// hundredths of zero: the uniform bins above, 2^-7 wide, hold midpoints of two pairs there in 97 % of the wavefronts, these
// in none (they are 2^-11 wide at zero, and 2^-4 next to the scale).  The half-precision bits of t with u's sign, shifted right
// by 6, are the place of the pattern's byte: patterns p & 3 lie 128 bytes apart, the signs 512, four patterns 1024.
constexpr int kFineBins = 128;          // per sign
constexpr float kFinePer = 1.988f;      // t stays below 2 with the roundings of build_fine_table
constexpr uint32_t kFineLeast = 0x2000;  // 2^-7 as FP16 bits: bit 13 is set throughout, the place starts at 128
constexpr uint32_t kFineCrowded = 16u;  // entry: more than two candidates, compare with all centroids; else the lower of two

// words of the tables of S patterns
constexpr int search_tiles(int S) { return (S + 15) / 16; }
constexpr size_t search_near_words(int S) { return (size_t)S * (kSearchBins / 4); }                          // a byte per pattern and bin
constexpr size_t search_pair_words(int S) { return (size_t)S * 16; }                                          // (centroid k, centroid k + 1) per pattern
constexpr size_t search_fine_words(int S) { return (size_t)((S + 3) / 4) * (4 * 2 * kFineBins / 4); }          // a byte per pattern, sign and bin
constexpr size_t search_coef_words(int S) { return (size_t)search_tiles(S) * kSearchBlocks * 3 * 64 * 4; }   // A, B, E in matrix-core operand order

// cent: [S][stride] FP16 bits, n_cent ascending centroids each; step: bin axis units per u = 1 (at most 32700)
// Everything is formed in double precision and every rounding is added to E.
namespace search_detail {

inline double half_value(uint16_t h) {
    _Float16 v;
    std::memcpy(&v, &h, 2);
    return (double)v;
}
inline uint16_t half_bits(double d) {
    const _Float16 v = (_Float16)d;
    uint16_t h;
    std::memcpy(&h, &v, 2);
    return h;
}
inline uint16_t half_bits_up(double d) {  // d >= 0: the least FP16 value not below d
    uint16_t h = half_bits(d);
    if (half_value(h) < d) ++h;
    return h;
}

// the squared distance of u to the nearest of n ascending centroids
inline double nearest_sq(const double* c, int n, double u) {
    double best = (u - c[0]) * (u - c[0]);
    for (int k = 1; k < n; ++k) best = std::min(best, (u - c[k]) * (u - c[k]));
    return best;
}

// how far a reconstructed centroid fp16(c s) can lie from c s, in units of s
inline double recon_eps(double c) { return 1.02 * (std::fabs(c) * 0x1p-11 + 0x1p-25 / (double)kSearchLeastScale) + 1e-6; }

// the lowest and the highest of n ascending centroids (off by eps) that can be nearest to a u from lo to hi
inline void candidates(const double* c, const double* eps, int n, double lo, double hi, int& kmin, int& kmax) {
    // the nearest centroid is k when k of the midpoints lie below u; a midpoint is off by its centroids' rounding
    kmin = 0;
    kmax = 0;
    for (int k = 0; k + 1 < n; ++k) {
        const double m = 0.5 * (c[k] + c[k + 1]), off = std::max(eps[k], eps[k + 1]);
        if (m + off < lo) kmin = k + 1;
        if (m - off <= hi) kmax = k + 1;
    }
    // of centroids that round to the same value the lowest counts as nearest, also to values above them
    while (kmin > 0 && c[kmin] - c[kmin - 1] <= 2.0 * (eps[kmin] + eps[kmin - 1])) --kmin;
}

struct Coef {
    uint16_t a, b, e;
};

// one pattern, one bin
inline Coef bin_coef(const double* c, int n, int bin, double step) {
    const double slack = 0.51;  // q is off by half a unit, and by the rounding of step / s
    const double lo = (256.0 * bin - 32768.0 - slack) / step, hi = (256.0 * bin + 255.0 - 32768.0 + slack) / step;
    const double mid = (256.0 * bin + 128.0 - 32768.0) / step, start = (256.0 * bin - 32768.0) / step;
    // h(u) = squared distance to the nearest centroid - (u - mid)^2, concave; its corners lie midway between centroids
    const auto h = [&](double u) { return nearest_sq(c, n, u) - (u - mid) * (u - mid); };
    const double h_lo = h(lo), h_hi = h(hi), slope = (h_hi - h_lo) / (hi - lo);
    double gap = 0.0, far_sq = std::max(nearest_sq(c, n, lo), nearest_sq(c, n, hi));
    for (int k = 0; k + 1 < n; ++k) {
        const double u = 0.5 * (c[k] + c[k + 1]);
        if (u <= lo || u >= hi) continue;
        gap = std::max(gap, h(u) - (h_lo + slope * (u - lo)));
        far_sq = std::max(far_sq, nearest_sq(c, n, u));
    }
    const double a = (h_lo + slope * (start - lo) + 0.5 * gap) * kSearchCoefScale, b = slope / step * kSearchCoefScale;
    Coef r;
    r.a = half_bits(a);
    r.b = half_bits(b);
    double e = 0.5 * gap * kSearchCoefScale + std::fabs(a - half_value(r.a)) + 255.0 * std::fabs(b - half_value(r.b));
    e += (slack + 1.0 / 8.0) * std::fabs(b);  // the place is off by `slack`; m above 2048 is rounded to FP16: by at most 255 n / 2048
    // a reconstructed centroid is fp16(c s): off by 2^-11 |c| and 2^-25 / s in units of s
    const double far = std::sqrt(far_sq), reach = std::max(std::fabs(lo), std::fabs(hi)) + far;
    const double eps = 1.02 * (reach * 0x1p-11 + 0x1p-25 / (double)kSearchLeastScale);
    e += (2.0 * far * eps + 3.0 * eps * eps) * kSearchCoefScale;
    e += 0x1p-14 * (std::fabs(a) + 255.0 * std::fabs(b));  // FP32 accumulation of up to 512 products
    r.e = half_bits_up(std::min(1.01 * e + 1e-6, 60000.0));
    return r;
}

}  // namespace search_detail

inline void build_search_tables(const uint16_t* cent, int stride, int n_cent, int S, double step, uint32_t* near, uint32_t* pair, uint32_t* coef) {
    using namespace search_detail;
    std::vector<Coef> co((size_t)S * kSearchBins);
    uint8_t* nb = reinterpret_cast<uint8_t*>(near);
    for (int p = 0; p < S; ++p) {
        double c[16], eps[16];
        for (int k = 0; k < n_cent; ++k) {
            c[k] = half_value(cent[p * stride + k]);
            eps[k] = recon_eps(c[k]);
        }
        for (int k = 0; k < 16; ++k) {
            const int a = std::min(k, n_cent - 1), b = std::min(k + 1, n_cent - 1);
            pair[p * 16 + k] = (uint32_t)cent[p * stride + a] | ((uint32_t)cent[p * stride + b] << 16);
        }
        for (int bin = 0; bin < kSearchBins; ++bin) {
            co[(size_t)p * kSearchBins + bin] = bin_coef(c, n_cent, bin, step);
            const double lo = (256.0 * bin - 32768.0 - 0.52) / step, hi = (256.0 * bin + 255.0 - 32768.0 + 0.52) / step;
            int kmin, kmax;
            candidates(c, eps, n_cent, lo, hi, kmin, kmax);
            const int range = kmax - kmin;
            nb[p * kSearchBins + bin] = (uint8_t)((range > 1 ? kmin : std::min(kmin, n_cent - 2)) * 4 + (range > 2 ? kNearWide : range == 2 ? kNearTwo : 0u));
        }
    }
    // Operand order of v_mfma_f32_16x16x32_f16 for tiles of 16 patterns: lane l holds column l % 16 and the eight k
    // 8 (l / 16) .. + 7.  Per 32 bins three operands: (B, A) of bins 0..15 (k = 2 bin, 2 bin + 1), (B, A) of bins 16..31,
    // and E, whose k run over the bins that the lane's other two operands hold: 4 (l / 16) .. + 3 and 16 more.
    uint16_t* out = reinterpret_cast<uint16_t*>(coef);
    for (int t = 0; t < search_tiles(S); ++t)
        for (int j = 0; j < kSearchBlocks; ++j)
            for (int op = 0; op < 3; ++op)
                for (int lane = 0; lane < 64; ++lane)
                    for (int i = 0; i < 8; ++i, ++out) {
                        const int p = 16 * t + (lane & 15), g = lane >> 4;
                        const int bin = 32 * j + (op < 2 ? 16 * op + 4 * g + i / 2 : 4 * g + (i & 3) + 16 * (i >> 2));
                        const bool is_a = op < 2 && (i & 1) == 1;
                        if (p >= S) {
                            *out = is_a ? half_bits(60000.0) : 0;  // patterns that do not exist are never near the least
                            continue;
                        }
                        const Coef& r = co[(size_t)p * kSearchBins + bin];
                        *out = op == 2 ? r.e : is_a ? r.a : r.b;
                    }
}

// The min/max selector's table (kFineBins).  t differs from the true 2^-7 + kFinePer |u| by its rounding to FP16, 2^-11 of itself,
// and by that of kFinePer / s: 2^-11 of kFinePer |u|, 2^-10 where the quotient is a subnormal (s above 2^15), and the
// reciprocal's error.
inline void build_fine_table(const uint16_t* cent, int stride, int n_cent, int S, uint32_t* fine) {
    using namespace search_detail;
    uint8_t* out = reinterpret_cast<uint8_t*>(fine);
    for (int p = 0; p < S; ++p) {
        double c[16], eps[16];
        for (int k = 0; k < n_cent; ++k) {
            c[k] = half_value(cent[p * stride + k]);
            eps[k] = recon_eps(c[k]);
        }
        uint8_t* row = out + (size_t)(p >> 2) * (4 * 2 * kFineBins) + (p & 3) * kFineBins;
        for (int bin = 0; bin < kFineBins; ++bin) {
            const auto edge = [](int b) { return std::ldexp(1.0 + (b & 15) / 16.0, (b >> 4) - 7); };
            const double least = std::max(0.0, edge(bin) * (1.0 - 0x1p-10) - 0x1p-7) / kFinePer * (1.0 - 0x1p-9);
            const double most = (edge(bin + 1) * (1.0 + 0x1p-10) - 0x1p-7) / kFinePer * (1.0 + 0x1p-9);
            for (int sign = 0; sign < 2; ++sign) {
                int kmin, kmax;
                candidates(c, eps, n_cent, sign ? -most : least, sign ? -least : most, kmin, kmax);
                row[sign * 4 * kFineBins + bin] = (uint8_t)(kmax - kmin > 1 ? kFineCrowded : std::min(kmin, n_cent - 2));
            }
        }
    }
}

// Whether the min/max selector uses these bins for a model or the uniform ones.  These are the wider ones from u = 0.5 on: patterns that
// crowd centroids there (groups with a common offset, or of two magnitudes) have bins with more than two candidates, and a
// wavefront with a value in one compares all of its values with all centroids.  131072 groups, models fitted to them, 16 patterns:
// offset 1 +- 0.1 42.5 us by these bins, 18.1 us by the uniform ones; two magnitudes, 0.5 +- 0.02 42.2 and 17.8 us.  Where the
// uniform bins have patterns with more than three candidates as well, nothing is gained: two magnitudes, 0.5 +- 0.005 (16 patterns
// crowded here, 13 there) 42.2 and 47.6 us.  Hence the line: a pattern that both bins crowd costs a quarter more by the uniform ones
// (30 us over the 18 us of a model that neither crowds, 24 us by these), and one crowded pattern in sixteen (a wavefront in
// five) costs these what the uniform ones pay for third candidates (2 us for values, 8 us for keys).
inline bool fine_bins_serve(const uint32_t* near, const uint32_t* fine, int S) {
    const uint8_t *n = reinterpret_cast<const uint8_t*>(near), *f = reinterpret_cast<const uint8_t*>(fine);
    int crowded = 0, wide = 0;
    for (int p = 0; p < S; ++p) {
        const uint8_t* row = f + (size_t)(p >> 2) * (4 * 2 * kFineBins) + (p & 3) * kFineBins;
        bool c = false, w = false;
        for (int bin = 0; bin < kFineBins; ++bin) c = c || ((row[bin] | row[4 * kFineBins + bin]) & kFineCrowded) != 0;
        for (int bin = 0; bin < kSearchBins; ++bin) w = w || (n[p * kSearchBins + bin] & kNearWide) != 0;
        crowded += c;
        wide += w;
    }
    return 16 * crowded <= S + 20 * wide;
}

}  // namespace ecco
