// LDS footprint of one front in the factor and sweep kernels. Shared by the
// symbolic analysis (which splits supernodes whose fronts do not fit) and
// the launch code (which sizes dynamic LDS).
#pragma once
#include <algorithm>
#include <cstdint>

#if defined(__HIP__)
#define KKT_HD __host__ __device__
#else
#define KKT_HD
#endif

namespace kkt {

// Panels use an odd leading dimension r|1 in LDS and in HBM (conflict-free
// strided LDS access; the HBM<->LDS copies are contiguous).
// factor: (r|1) x rup16(c) panel of doubles (columns padded to the 16-wide
// matrix-core tile) + r staged relative indices
inline int64_t factor_lds_bytes(int r, int c) {
    const int64_t cp = (c + 15) & ~15;
    return (int64_t)(r | 1) * cp * 8 + (int64_t)r * 4 + 16;
}

// The front kernel's blocked panel: column blocks of 16, each with the rows
// from its diagonal block down (own columns padded to 16, update rows padded
// to 16), 16 doubles per row.
constexpr int kFrontRowStride = 16;
KKT_HD constexpr int64_t blocked_lds_bytes(int r, int c) {
    const int64_t nbc = (c + 15) >> 4, rt = 16 * (nbc + ((r - c + 15) >> 4));
    return 8 * kFrontRowStride * (nbc * rt - 8 * nbc * (nbc - 1));
}
// Fronts that take the blocked panel with maxp panel waves: one wave covers 64
// rows below the diagonal block. Taller fronts stay column-major. (Every front
// so covered that fits 158 KiB by front_lds_bytes fits them blocked too.)
KKT_HD constexpr bool front_blocked(int r, int c, int maxp) {
    return 16 * (((c + 15) >> 4) + ((r - c + 15) >> 4)) <= 16 + 64 * maxp;
}
// what a front of the factor launches reserves (twelve, eight or four waves: four
// or three panel waves); the padding to whole 16-row and 16-column blocks takes
// it up to 5,288 bytes past the front's budget
inline int64_t factor_launch_lds_bytes(int r, int c) {
    return front_blocked(r, c, 4) ? std::max(factor_lds_bytes(r, c), blocked_lds_bytes(r, c)) : factor_lds_bytes(r, c);
}

// what the fronts' budget counts for the sweeps: (r|1) x c panel (padded to an
// even count), r + c vector entries
inline int64_t solve_lds_bytes(int r, int c) { return ((((int64_t)(r | 1) * c + 1) & ~(int64_t)1) + r + c) * 8; }

// what the sweep launches reserve: forward, the solved values (padded to 16
// columns), two vectors of r and the rows past 128;
// backward, the panel (padded to an even count), the update values (padded
// to whole steps of the dot products) and c sums
inline int64_t fwd_lds_bytes(int r, int c) {
    return (((c + 15) & ~15) + 2 * (int64_t)((r + 1) & ~1) + std::max(0, r - 128)) * 8;
}
inline int64_t bwd_lds_bytes(int r, int c) {
    const int g4 = c <= 16 ? 64 : c <= 32 ? 32 : c <= 64 ? 16 : 8;
    return ((((int64_t)(r | 1) * c + 1) & ~(int64_t)1) + ((r - c + g4 - 1) & -g4) + c) * 8;
}
// (levels of many fronts: the triangle with an odd leading dimension, u values
// and the columns' partial sums, 65, 33, 17 or 9 places a column)
inline int64_t bwd_wide_lds_bytes(int r, int c) {
    const int places = c <= 16 ? 65 : c <= 32 ? 33 : c <= 64 ? 17 : 9;
    return ((((int64_t)(c | 1) * c + 1) & ~(int64_t)1) + ((r - c + 1) & ~1) + places * c) * 8;
}

inline int64_t front_lds_bytes(int r, int c) { return std::max(factor_lds_bytes(r, c), solve_lds_bytes(r, c)); }

// A front too tall for the LDS budget even at one column is a large front:
// factored and solved in HBM, in chunks of at most this many columns (the
// sweeps stage its c x c triangle in LDS and solve it with one wave).
constexpr int kLargeFrontCols = 64;

}  // namespace kkt
