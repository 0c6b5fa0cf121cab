// Blinded decryption in one pass per prime (halves_joint_kernel) for every
// size class; the one-lane classes hand the part of a launch that leaves SIMDs
// idle to the lane-group form (kjlanes.hip).  A translation unit of its own,
// so the per-class objects stay as they are.  Its Montgomery products align
// each column (mont.hpp): measured on these kernels' code, that puts their
// multiply-adds at addresses 0 modulo 8.
#define PMK_COLUMN_ALIGN 1
#include "kernels_impl.hpp"

namespace pmk {

namespace {

template <int CB>
int launch_joint_lane_class(const ClassRun &r, hipStream_t s);

// Fold form: blocks as for the plain halves (25 MiB under 2048-bit keys: 27.5 ms with
// Montgomery products, 22.1 ms here).  A small launch runs over lane groups instead
// while each of their waves has a SIMD of its own: eight lanes take 4.6 / 10.0 / 20.5
// ms at 2048 / 3072 / 4096 bits against 5.1 / 17.4 / 40.6 in one lane; four lanes pay
// at 3072 (12.1 ms) and 4096 bits, no longer at 2048 (5.3 ms), two at 4096 where the
// shared tables make two rounds (joint_two_lanes).
template <int CB>
int launch_joint_fold(const ClassRun &r, hipStream_t s) {
    constexpr uint32_t per = fold_lane_block(CB);
    static const FoldBlocks<CB> occ((const void *)halves_joint_kernel<CB>);
    const uint32_t cus = (uint32_t)device_cus();
    uint32_t waves = per * occ.n[per] * cus;
    if (r.grid_cap && r.grid_cap < waves) waves = r.grid_cap;
    if (eight_lanes(CB) && 2 * r.ntiles < waves) {
        uint32_t lane_units = 0;
        const int L = lanes_for_launch(r, 2 * r.ntiles, waves, 4u * cus, joint_lanes_resident, &lane_units);
        if (L > 2 || (L == 2 && joint_two_lanes(r, cus))) return launch_joint_lanes(r, L, 0, 2 * r.ntiles, s);
    }
    if (joint_mont_launch(r, cus)) return launch_joint_mont(r, s);
    if (r.slots_dec < waves) waves = r.slots_dec;
    const uint32_t nw = waves < r.group_tiles ? waves : r.group_tiles;
    const uint32_t grid = occ.resident(nw, waves, cus);
    const uint32_t round = grid / 2 ? grid / 2 : 1;  // groups
    uint32_t full = r.ngroups;
    bool quad = false;
    if (per == 2 && waves >= 2) {
        const uint32_t rest = r.ngroups <= round ? r.ngroups : r.ngroups % round;
        quad = full > rest && 4 * rest <= waves && rest <= (fold_joint_waves(CB) - 1) * cus;
        if (quad || 4 * rest <= 4u * cus) full -= rest;
    }
    const uint64_t slot = 2 * table_words_per_slot(r.cls, 1, r.win);  // two odd-power tables
    auto blocks = [&](uint32_t from, uint32_t to, uint32_t n, uint32_t threads, bool split) {
        hipLaunchKernelGGL(halves_joint_kernel<CB>, dim3(persistent_grid(to - from, n, 0)), dim3(threads), 0, s, r, slot, from,
                           to, split);
        return (int)hipGetLastError();
    };
    int e = 0;
    if (r.group_tiles == 1) {
        e = lone_rounds<CB>(2 * r.ngroups, grid, cus,
                            [&](uint32_t from, uint32_t to) { return blocks(from, to, grid, 64, false); });
        full = r.ngroups;
    } else if (full) {
        e = blocks(0, 2 * full, grid, 64 * nw, false);
    }
    if constexpr (per == 2) {
        if (!e && full < r.ngroups && quad) {
            hipLaunchKernelGGL((halves_quad_kernel<CB, true>), dim3(r.ngroups - full), dim3(256), 0, s, r, slot, 2 * full,
                               2 * r.ngroups);
            e = (int)hipGetLastError();
            full = r.ngroups;
        }
    }
    if (!e && full < r.ngroups) e = blocks(2 * per * full, 2 * per * r.ngroups, waves, 64, true);
    if (e) return e;
    hipLaunchKernelGGL(blind_check_kernel<CB>, dim3(2 * r.ntiles), dim3(64), 0, s, r);
    e = (int)hipGetLastError();
    if (e) return e;
    hipLaunchKernelGGL((fold_finish_kernel<CB, fold_lane(CB).nl, fold_lane(CB).lb>), dim3(2 * r.ntiles), dim3(64), 0, s, r,
                       0u, 0u);
    return (int)hipGetLastError();
}

template <int CB>
int launch_joint_class(const ClassRun &r, hipStream_t s) {
    if constexpr (fold_lane(CB).nl != 0) return launch_joint_fold<CB>(r, s);
    else return launch_joint_lane_class<CB>(r, s);
}

template <int CB>
int launch_joint_lane_class(const ClassRun &r, hipStream_t s) {
    // resident blocks on this device; never more than the r.slots_dec table slots
    // (those of the CRT-halves kernel, which is at least as occupied and capped by
    // the same unit count)
    static const int oj = [] {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void *)halves_joint_kernel<CB>, 64, 0) !=
                hipSuccess ||
            nb < 1)
            nb = 1;
        return nb;
    }();
    const uint32_t ncu = (uint32_t)device_cus();
    const uint32_t resident = (uint32_t)oj * ncu;
    const uint32_t units = 2 * r.ntiles * lanes_half(CB);
    uint32_t grid = persistent_grid(units, r.slots_dec, r.grid_cap);
    if (grid > resident) grid = resident;
    // the part of a launch that leaves SIMDs idle runs in lane groups, as for
    // the plain CRT halves
    uint32_t main_end = units;
    int L = 1;
    if constexpr (lanes_half(CB) == 1) {
        uint32_t res = resident;
        if (r.grid_cap && r.grid_cap < res) res = r.grid_cap;
        if (r.slots_dec < units && r.slots_dec < res) res = r.slots_dec;  // table room
        uint32_t lane_units = 0;
        L = lanes_for_launch(r, units, res, 4u * ncu, joint_lanes_resident, &lane_units);
        main_end = units - lane_units;
    } else {
        if (wide_fill(r, 2 * r.ntiles, lanes_half(CB), 4u * ncu, joint_lanes_resident(r.cls, 2 * lanes_half(CB)))) {
            L = 2 * lanes_half(CB);
            main_end = 0;
        }
    }
    const uint64_t slot = 2 * table_words_per_slot(r.cls, 1, r.win);  // two odd-power tables
    if (main_end) {
        hipLaunchKernelGGL(halves_joint_kernel<CB>, dim3(persistent_grid(main_end, grid, 0)), dim3(64), 0, s, r, slot,
                           0u, main_end, false);
        const int e = (int)hipGetLastError();
        if (e) return e;
    }
    if (main_end == units) return 0;
    if (L == 1) {  // the partial round, one lane per number, in a launch of its own
        hipLaunchKernelGGL(halves_joint_kernel<CB>, dim3(persistent_grid(units - main_end, grid, 0)), dim3(64), 0, s,
                           r, slot, main_end, units, false);
        return (int)hipGetLastError();
    }
    return launch_joint_lanes(r, L, main_end / lanes_half(CB), 2 * r.ntiles, s);
}

}  // namespace

int launch_decrypt_joint(const ClassRun &r, void *stream) {
    if (r.ntiles == 0) return 0;
    hipStream_t s = (hipStream_t)stream;
    switch (r.cls) {
        case 0: return launch_joint_class<128>(r, s);
        case 1: return launch_joint_class<256>(r, s);
        case 2: return launch_joint_class<512>(r, s);
        case 3: return launch_joint_class<1024>(r, s);
        case 4: return launch_joint_class<2048>(r, s);
        case 5: return launch_joint_class<3072>(r, s);
        case 6: return launch_joint_class<4096>(r, s);
        case 7: return launch_joint_class<6144>(r, s);
        case 8: return launch_joint_class<8192>(r, s);
        default: return (int)hipErrorNotSupported;
    }
}

}  // namespace pmk
