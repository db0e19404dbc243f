// Which form of the Brillouin row kernel a launch takes, and how it cuts the rows (host arithmetic only).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>

namespace dirac {

// Threads of a (site, right-hand side): one, one per chirality, or one per colour row, or both (see the kernel).
struct RowForm {
    bool chirality, colour;
};
// form 0: one thread, in FP64 one per chirality; 1: one per chirality and colour row; FP64 only: 2: one per colour row,
// 3: one thread (N_c = 1 and 2, whose sums fit the registers)
inline RowForm row_form(bool fp64, int form) {
    return {form == 1 || (form == 0 && fp64), form == 1 || form == 2};
}
inline bool has_form(bool fp64, int form, int nc) {
    if (!fp64) return form <= 1;
    return form == 0 || (nc == 1 ? form == 3 : form <= (nc == 2 ? 3 : 2));  // N_c = 1: a colour row is the whole
}
constexpr int kMaxWindowEntries = 3;  // entries of a slot of the link window that a lane moves at most

struct RowShape {
    int nc, nv, storage;  // storage: bytes of a vector element (16: FP64)
    int nx;
    int64_t rows;
    bool clover;
};
struct RowPlan {
    int form = -1;  // -1: the direct kernel
    int seg = 0;    // sites per work-group
    int entries = 0;
    double us = 0.0;  // estimate
};

// Estimate.  The kernel takes about start + wave * m microseconds while a CU has m wavefronts of it, the start being the
// latency of the 27 row copies and their barriers: FP32, N_c = 3, 72 us with 1 wavefront per CU, 75 with 8, 101 with 12.  A
// launch is whole rounds of as many work-groups as a CU takes at once (by registers and LDS) and a last round of the
// rest; consecutive rounds overlap by a tenth.  start and wave are fitted to 7000 timings of all forms and segments
// (lattices of 256 to 166320 sites, N_c = 1 to 4, N_v = 1 to 32, three precisions) with a mean error of 6 to 10 %; what
// it picks from them is 1.2 % slower than the best on average.  One table of costs for all N_c, that of N_c = 3, was 9 %
// off: N_c = 2 in FP32 took the split form at 8^3 x 16, N_v = 12 (71 us instead of 50).
constexpr int kDirectForm = 4;
struct RowCost {
    int segmented, whole;  // wavefronts per SIMD that the registers allow, with the row in segments and whole
    double start, wave;
};
inline RowCost row_cost(int storage, int form, int nc) {
    static constexpr RowCost kFp64[4][4] = {{{5, 6, 25.6, 1.23}, {3, 4, 33.2, 2.14}, {3, 3, 52.5, 3.57}, {2, 2, 79.5, 3.22}},
                                            {{}, {4, 4, 28.3, 1.35}, {3, 3, 30.7, 1.57}, {3, 3, 34.3, 1.73}},
                                            {{}, {3, 4, 30.7, 2.15}, {3, 4, 35.4, 2.76}, {3, 4, 48.1, 2.73}},
                                            {{4, 4, 24.7, 1.84}, {2, 2, 59.6, 1.24}, {}, {}}};
    static constexpr RowCost kOther[2][4] = {{{6, 7, 24.1, 1.31}, {4, 4, 35.0, 1.84}, {3, 3, 54.2, 2.58}, {2, 2, 96.7, 0.75}},
                                             {{7, 8, 21.8, 1.33}, {6, 7, 25.1, 1.22}, {5, 5, 29.7, 1.04}, {4, 5, 31.7, 0.97}}};
    // the direct kernel, FP64, FP32 and BF16
    static constexpr RowCost kDirect[3][4] = {{{6, 6, 34.6, 4.12}, {3, 3, 52.6, 8.15}, {2, 2, 70.7, 15.0}, {2, 2, 87.7, 26.2}},
                                              {{6, 6, 40.0, 2.20}, {5, 5, 54.0, 5.10}, {4, 4, 75.0, 8.0}, {3, 3, 99.0, 11.4}},
                                              {{6, 6, 39.4, 1.90}, {5, 5, 58.0, 3.40}, {4, 4, 80.7, 5.95}, {3, 3, 109.0, 7.5}}};
    if (form == kDirectForm) return kDirect[storage == 16 ? 0 : (storage == 8 ? 1 : 2)][nc - 1];
    return storage == 16 ? kFp64[form][nc - 1] : kOther[form][nc - 1];
}
constexpr int kCus = 256;
constexpr std::size_t kCuLds = 160 * 1024;

// Work-groups of w wavefronts that a CU takes by its registers.  Up to four wavefronts pack over the SIMDs (four groups of
// 3 at three per SIMD); 5 to 7 take two places on every SIMD and measured as if a third were lost (one group of 5 or 6
// at three or four per SIMD).
inline int groups_by_registers(int occupancy, int w) {
    return std::max(1, w <= 4 ? 4 * occupancy / w : (occupancy - (w < 8 ? 1 : 0)) / 2);
}

// groups: work-groups of the launch; at_once: of a CU; load: wavefronts of one, weighted
inline double estimate_us(const RowCost& c, double groups, int at_once, double load) {
    const double whole = std::floor(groups / kCus / at_once);
    const double rest = std::ceil(groups / kCus - whole * at_once);
    double us = whole > 0 ? 0.9 * whole * (c.start + c.wave * at_once * load) + 0.1 * c.start : 0.0;
    if (rest > 0) us += c.start + c.wave * rest * load;
    return us;
}

// lds(form, seg): bytes of LDS of a work-group; at most 64 KiB is taken.
template <class Lds>
RowPlan plan_rows(const RowShape& s, Lds&& lds) {
    const bool fp64 = s.storage == 16;
    const int units = s.nc * 4 * s.nv * s.storage / 16;
    RowPlan best;
    for (int form = 0; form < kDirectForm; ++form) {
        const RowForm f = row_form(fp64, form);
        if (!has_form(fp64, form, s.nc) || (f.colour && s.clover)) continue;  // the colour rows carry no clover term
        const int per_site = s.nv * (f.chirality ? 2 : 1) * (f.colour ? s.nc : 1);
        const RowCost c = row_cost(s.storage, form, s.nc);
        for (int d = std::min(s.nx, 512 / per_site); d >= 1; --d) {
            const int n = (s.nx + d - 1) / d;  // segments; the last is moved back to end with the row
            d = (s.nx + n - 1) / n;            // the shortest that many
            const int threads = d * per_site, sites = d + (d == s.nx ? 0 : 2);
            const int entries = (sites * s.nc * s.nc + threads - 1) / threads;
            // at least half a wavefront, and enough threads for the two halo sites and the link window
            if (threads < 32 || (d != s.nx && units > threads) || entries > kMaxWindowEntries) continue;
            const std::size_t bytes = lds(f, d);
            if (bytes > 64 * 1024) continue;
            const int w = (threads + 63) / 64;
            const int at_once = std::min<int>(groups_by_registers(d == s.nx ? c.whole : c.segmented, w),
                                              static_cast<int>(kCuLds / bytes));
            // a wider window costs registers (spilled ones in segments); a copied site a quarter of its threads
            const double wide = entries == 1 ? 1.0 : (d == s.nx ? 1.5 : 2.2);
            const double load = w * wide + 0.25 * sites * per_site / 64;
            const double us = estimate_us(c, static_cast<double>(s.rows) * n, at_once, load);
            if (best.form < 0 || us < best.us) best = {form, d, entries, us};
        }
    }
    // The direct kernel, one thread per (site, right-hand side), by the same estimate (FP64, N_v = 24 at 13 x 14 x 11 x 20:
    // 1.26 ms against 1.62); ahead of the estimate's error in FP32 and BF16, which is larger for few right-hand sides.  Below
    // 8 of them, and in FP32 and BF16 where they are no multiple of 4, its gathers do not coalesce and take up to four
    // times the estimate.
    const RowCost c = row_cost(s.storage, kDirectForm, s.nc);
    const double groups = static_cast<double>(s.rows) * s.nx * s.nv / 64;
    const double ahead = fp64 ? 1.0 : (s.nv >= 16 ? 0.95 : 0.85);
    if (best.form >= 0 && s.nv >= 8 && (fp64 || s.nv % 4 == 0) &&
        estimate_us(c, groups, 4 * c.whole, 1.0) < ahead * best.us)
        return RowPlan{};
    return best;
}

}  // namespace dirac
