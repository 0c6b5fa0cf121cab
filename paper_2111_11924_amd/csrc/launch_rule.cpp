// Which form the CRT halves of a launch take.  Each rule estimates the forms'
// times from the rounds of waves or blocks that the launch makes and takes the
// shortest.  Times in ms, measured on 256 compute units (loads are scaled to the
// device's number of them).
#include <algorithm>

#include "pmk_internal.hpp"

namespace pmk {

namespace {

// Time of `load` (waves, blocks or units) in rounds of `full`, or of `room` where
// the table or the grid limit holds fewer.  A round that leaves SIMDs with fewer waves
// takes less: part[i] up to (i + 1) / N of a full one.
template <int N>
double rounds_ms(uint64_t load, uint64_t full, uint64_t room, const double (&part)[N]) {
    auto one = [&](uint64_t x) { return part[(x * N - 1) / full]; };
    const uint64_t round = std::max<uint64_t>(1, std::min(full, room)), rest = load % round;
    return (double)(load / round) * one(round) + (rest ? one(rest) : 0);
}

// Slots of `slot` words in the launch's table (0 words: not sized yet), at most the
// grid limit.
uint64_t room_of(const ClassRun &r, uint64_t slot) {
    const uint64_t room = r.table_words ? r.table_words / slot : ~0ull;
    return r.grid_cap ? std::min<uint64_t>(room, r.grid_cap) : room;
}

// Fold form in one lane: units of up to nw waves (tiles of a group, modulo one prime),
// `tiles` of them on average.  A group's table takes LDS whatever its tiles: three 3072-bit
// blocks or one 4096-bit block fit a compute unit, so that small groups leave SIMDs idle
// there.
double lane_ms(int bits, uint32_t nw, double tiles, uint64_t units, uint64_t room, uint32_t cus) {
    const uint64_t cu = cus;
    switch (bits) {
        case 1024:
            if (nw == 1) return rounds_ms(units, 8 * cu, room, {1.1, 2.4});
            return rounds_ms(units, 6 * cu, room, {1.1, 1.9, 2.75});
        case 2048:
            if (nw == 1) return rounds_ms(units, 4 * cu, room, {4.4});
            return rounds_ms(units, 4 * cu, room, {4.4, 8.1});
        case 3072: {
            if (nw == 1) return rounds_ms(units, 3 * cu, room, {14.3, 14.3, 15.8});
            // one block per compute unit; two, at first on a few of them
            const double one = 15.2 + 2.7 * std::max(0., tiles - 3),
                         two = 24.4 + 5.1 * std::min(1., std::max(0., tiles - 2)) + 2.5 * std::max(0., tiles - 3);
            const double up = two - one;
            return rounds_ms(units, 2 * cu, room, {one, one, one, one + .77 * up, one + .88 * up, two});
        }
        default: return rounds_ms(units, cu, room, {nw > 3 ? 31.0 : 28.9});
    }
}
// The same, blinded.
double joint_lane_ms(int bits, uint32_t nw, uint64_t units, uint64_t room, uint32_t cus) {
    const uint64_t cu = cus;
    switch (bits) {
        case 1024:
            if (nw == 1) return rounds_ms(units, 8 * cu, room, {1.45, 2.45});
            return rounds_ms(units, 4 * cu, room, {1.45, 2.4});
        case 2048:
            if (nw == 1) return rounds_ms(units, 4 * cu, room, {5.9});
            return rounds_ms(units, 4 * cu, room, {5.9, 11.2});
        case 3072:
            if (nw == 1) return rounds_ms(units, 3 * cu, room, {17.6, 17.6, 20.5});
            if (nw == 2) return rounds_ms(units, 2 * cu, room, {18.5, 29.3});
            if (nw == 3) return rounds_ms(units, 2 * cu, room, {19.5, 35.0});
            return rounds_ms(units, 2 * cu, room, {22.0, 38.7});
        default: return rounds_ms(units, cu, room, {nw > 3 ? 42.8 : (nw > 2 ? 39.0 : 37.5)});
    }
}

// Montgomery products: one lane per number up to 4096 bits, four above.  `busy`: blocks
// of one wave do not land evenly, some SIMDs have two whatever the load (4096 bits in
// the server's rounds: 77 ms for 900 jobs, 43 alone).
double mont_ms(int bits, uint64_t jobs, uint64_t room, bool busy, uint32_t cus) {
    const uint64_t cu = cus;
    switch (bits) {
        case 1024: return rounds_ms(jobs, 12 * cu, room, {busy ? 2.06 : 1.14, busy ? 2.92 : 2.06, 2.92});
        case 2048: return rounds_ms(jobs, 12 * cu, room, {busy ? 11.3 : 5.76, busy ? 16.5 : 11.3, 16.5});
        case 3072: return rounds_ms(jobs, 8 * cu, room, {busy ? 36.0 : 18.8, 36.0});
        case 4096: return rounds_ms(jobs, 8 * cu, room, {busy ? 85.5 : 44.7, 85.5});
        // 4 waves per job; a partial round after a full one runs beside its last waves
        case 6144:
            if (jobs < 2 * cu) return rounds_ms(jobs, 2 * cu, room / 4, {67.0, 111.5});
            return rounds_ms(jobs, 2 * cu, room / 4, {46.0, 66.0, 111.5, 111.5});
        default:
            if (jobs < 2 * cu) return rounds_ms(jobs, 2 * cu, room / 4, {146.0, 154.0, 258.0, 258.0});
            return rounds_ms(jobs, 2 * cu, room / 4, {107.0, 154.0, 258.0, 258.0});
    }
}
double joint_mont_ms(int bits, uint64_t jobs, uint64_t room, uint32_t cus) {
    const uint64_t cu = cus;
    switch (bits) {
        case 1024: return rounds_ms(jobs, 8 * cu, room, {1.64, 2.84});
        case 2048: return rounds_ms(jobs, 8 * cu, room, {7.2, 13.9});
        case 3072: return rounds_ms(jobs, 8 * cu, room, {23.2, 43.8});
        default: return rounds_ms(jobs, 8 * cu, room, {50.6, 50.6, 57.0, 57.0, 107.0, 107.0, 107.0, 107.0});
    }
}

// A number over a block (halves_group_kernel): blocks of 16 chunks modulo one
// prime.  Its chain is 2 to 5 times shorter than the one-lane chain, but it takes
// more of the chip per number.  Up to half a round of resident blocks takes `half`, a
// round `full`; after full rounds the blocks that go on are those that ended first, so that
// a rest of up to one block per compute unit takes `few` or less, a larger one `rest`.
double group_ms(int bits, uint64_t blocks, uint32_t cus) {
    const uint64_t cu = cus;
    auto ms = [&](uint64_t round, double half, double full, double few, double rest) {
        if (blocks <= round) return 2 * blocks <= round ? half : full;
        const uint64_t left = blocks % round;
        const double part = left ? std::min(1., 0.3 + 2. * (double)left / (double)cu) : 0.;
        return (double)(blocks / round) * full + (left > cu ? rest : part * few);
    };
    switch (bits) {
        case 1024: return rounds_ms(blocks, 8 * cu, ~0ull, {0.85, 0.92, 1.14, 1.77});
        case 2048: return ms(4 * cu, 2.7, 3.05, 1.55, 2.6);
        case 3072: return ms(2 * cu, 3.65, 4.5, 3.05, 4.5);
        case 4096: return ms(2 * cu, 6.3, 8.1, 5.1, 8.1);
        case 6144: return ms(cu, 15.4, 15.4, 15.4, 15.4);
        default: return ms(cu, 34.2, 34.2, 34.2, 34.2);
    }
}

// Classes side by side share the chip, each as if all had its blocks: a step of one's blocks runs
// beside the others', there are no rounds (four classes with 36 keys and 71 chunks: 17.4 ms,
// 29.6 where the 4096-bit class counts whole rounds and takes the lane form).
double beside_ms(int bits, uint64_t blocks, uint32_t cus) {
    const double full = (double)cus * (bits < 2048 ? 8 : (bits < 3072 ? 4 : (bits < 6144 ? 2 : 1)));
    const double round = group_ms(bits, (uint64_t)full, cus), x = (double)blocks / full;
    return x <= 1 ? group_ms(bits, blocks, cus) : (0.1 + x) * round;
}

}  // namespace

// The last `groups` groups of the launch's tiles spread over blocks (about as many
// blocks as groups of its average size have).
static double group_rest_ms(const ClassRun &r, uint32_t groups, uint32_t cus) {
    return group_ms(kClassBits[r.cls], 8ull * r.ntiles * groups / r.ngroups, cus);
}

// whether the grid limit holds a block of the group form
static bool group_fits(const ClassRun &r) {
    return !r.grid_cap || r.grid_cap >= (uint32_t)fold_group_block(kClassBits[r.cls]);
}

bool group_rest(const ClassRun &r, uint32_t groups, uint32_t cus) {
    return fold_lane_block(kClassBits[r.cls]) > 2 && r.tail_lanes > 0 && r.fill_lanes > 1 && group_fits(r) &&
           group_rest_ms(r, groups, cus) < lane_ms(kClassBits[r.cls], r.group_tiles, (double)r.ntiles / r.ngroups, 2ull * groups, ~0ull, cus);
}

// The lane form of a launch, its partial round spread over blocks where that is faster.
static double lane_launch_ms(const ClassRun &r, uint64_t room, uint32_t cus) {
    const int bits = kClassBits[r.cls];
    const uint32_t round = std::max(1u, bits > 3072 ? cus / 2 : cus), rest = r.ngroups % round;  // groups (3072, 4096 bits)
    const double tiles = (double)r.ntiles / r.ngroups;
    room /= r.group_tiles;
    if (r.group_tiles > 1 && rest && r.ngroups > round && room >= 2 * round && group_rest(r, rest, cus))
        return lane_ms(bits, r.group_tiles, tiles, 2ull * (r.ngroups - rest), room, cus) + group_rest_ms(r, rest, cus);
    return lane_ms(bits, r.group_tiles, tiles, 2ull * r.ngroups, room, cus);
}

bool mont_launch(const ClassRun &r, uint32_t cus) {
    const int bits = kClassBits[r.cls];
    if (!fold_lane(bits).nl) return false;
    if (!r.fold) return true;
    const uint64_t room = room_of(r, table_words_per_slot(r.cls, 1, r.win));
    return mont_ms(bits, 2ull * r.ntiles, room, r.busy, cus) < lane_launch_ms(r, room, cus);
}

bool group_launch(const ClassRun &r, uint32_t cus) {
    const int bits = kClassBits[r.cls];
    if (!fold_group(bits).nl || !r.fold || r.fill_lanes <= lanes_half(bits) || !group_fits(r)) return false;
    const uint64_t room = room_of(r, table_words_per_slot(r.cls, 1, r.win));
    double other = mont_ms(bits, 2ull * r.ntiles, room, r.busy, cus);
    if (fold_lane(bits).nl) other = std::min(other, lane_launch_ms(r, room, cus));
    const double ms = r.share > 1 ? beside_ms(bits, 2ull * r.parts * r.share, cus)
                      // where tiles have about three of their four parts, some block finds one at each of its steps
                      : group_ms(bits, r.parts > 2 * r.ntiles && 4 * r.parts <= 13 * r.ntiles ? 8ull * r.ntiles : 2ull * r.parts, cus);
    return ms < other;
}

bool fills_chip(const ClassRun &r_, uint32_t classes, uint32_t cus) {
    const int bits = kClassBits[r_.cls];
    ClassRun r = r_;
    r.share = classes;
    if (!fold_group(bits).nl || group_launch(r, cus)) return false;
    r.share = 1;
    const uint64_t waves = group_launch(r, cus) ? 2ull * r.parts * fold_group_block(bits) : 2ull * r.ntiles;
    return waves >= cus;
}

bool joint_mont_launch(const ClassRun &r, uint32_t cus) {
    const int bits = kClassBits[r.cls];
    if (!fold_lane(bits).nl) return false;
    if (!r.fold) return true;
    const uint64_t room = room_of(r, 2 * table_words_per_slot(r.cls, 1, r.win));
    return joint_mont_ms(bits, 2ull * r.ntiles, room, cus) <
           joint_lane_ms(bits, r.group_tiles, 2ull * r.ngroups, room / r.group_tiles, cus);
}

// At 4096 bits 44.8 ms while each of its waves has a SIMD.
bool joint_two_lanes(const ClassRun &r, uint32_t cus) {
    const uint64_t jobs = 2ull * r.ntiles, units = 2ull * r.ngroups;
    return kClassBits[r.cls] == 4096 && 44.8 < std::min(joint_mont_ms(4096, jobs, ~0ull, cus),
                                                        joint_lane_ms(4096, r.group_tiles, units, ~0ull, cus));
}

std::vector<uint64_t> whole_round_cuts(const uint32_t *key_map, uint64_t nchunks, uint32_t nkeys, uint64_t round,
                                       uint32_t group) {
    std::vector<uint64_t> cuts;
    std::vector<uint32_t> cnt(nkeys, 0);
    const uint32_t whole = group * kTile;
    uint64_t tiles = 0, ragged = 0, want = round;
    for (uint64_t i = 0; i < nchunks; ++i) {
        uint32_t &n = cnt[key_map[i]];
        if (n % kTile == 0) ++tiles;
        if (n % whole == 0) ++ragged;
        if (++n % whole == 0) --ragged;
        if (ragged == 0 && tiles == want && i + 1 < nchunks) {
            cuts.push_back(i + 1);
            want = 2 * want + round;  // next slice twice as long
        } else if (tiles > want) {
            want = (tiles / round + 1) * round;  // no cut there: the next round end
        }
    }
    return cuts;
}

}  // namespace pmk
