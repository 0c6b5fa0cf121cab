// Internal layout shared by the host side of the library and its kernels.
#pragma once
#include <stdint.h>

#include <vector>

#if defined(__HIPCC__)
#define PMK_HD __host__ __device__
#else
#define PMK_HD
#endif

namespace pmk {

// Modulus size classes the kernels are instantiated for (kMaxClass: the
// largest one built).  A key of `bits`
// bits runs in the smallest class with at least that many bits: Montgomery
// arithmetic only needs R > 4m, so a smaller modulus fits a larger class.
constexpr int kNumClasses = 9;
constexpr int kClassBits[kNumClasses] = {128, 256, 512, 1024, 2048, 3072, 4096, 6144, 8192};
constexpr int kMaxClass = 8;

PMK_HD constexpr int nl_for(int bits, int lb) { return (bits + 2 + lb - 1) / lb; }

// Radix of the full-size modulus: 28-bit limbs keep every column sum of a
// Montgomery product below 2^64 up to 3072 bits; 4096-bit moduli use 27 bits.
PMK_HD constexpr int lb_full(int bits) { return bits > 3072 ? 27 : 28; }
PMK_HD constexpr int lb_half(int bits) { return lb_full(bits / 2); }

// Lanes per bignum.  Full-size numbers: one lane up to 2048-bit moduli, a
// group of 4 lanes at 3072/4096 bits and of 8 lanes at 6144/8192 bits.  CRT
// halves: one lane up to 2048-bit primes (4096-bit keys), 4 lanes above.
PMK_HD constexpr int lanes_full(int bits) { return bits >= 6144 ? 8 : (bits >= 3072 ? 4 : 1); }
PMK_HD constexpr int lanes_half(int bits) { return bits >= 6144 ? 4 : 1; }
// chunks per tile: 64, one wavefront of one-lane numbers; with L lanes per
// number a tile's exponentiation takes L wavefronts of 64/L chunks each
PMK_HD constexpr int chunks_per_tile(int) { return 64; }
PMK_HD constexpr int round_up(int x, int m) { return (x + m - 1) / m * m; }
// grid of a persistent launch: one wave per unit, at most `slots` (the table
// slots) and at most `cap` when a cap is set
PMK_HD constexpr uint32_t persistent_grid(uint32_t units, uint32_t slots, uint32_t cap) {
    const uint32_t g = units < slots ? units : slots;
    return cap && cap < g ? cap : g;
}

// Default width of the sliding windows of the CRT halves
// (the autotuner may pick another one up to kMaxWin).
PMK_HD constexpr int window_for(int bits) { return bits <= 256 ? 3 : (bits <= 512 ? 4 : 5); }

// Offsets (uint32 words) of one key record of a class.
struct Geom {
    int bits, S, SH;
    int lbf, nlf, lbh, nlh;
    // CRT halves spread over a lane group (2 or 4 lanes per number): nla
    // limbs (a multiple of 4) and the constants of R_A = 2^(lbh nla); for the
    // classes whose halves always run in lane groups these are the nlh-limb ones
    int nla;
    int ew;  // words of the public exponent
    // full-modulus part
    int off_n32, off_nf, off_n0f, off_rrf, off_rrrf, off_onef, off_e, off_ebits, off_kbytes;
    // half records (p then q): m, m0, rr, rrr, one, d, and d2 = m - 1 - d (the
    // exponent of the Fermat inverse of c^d, for blinded decryption), then
    // one, rr, rrr of the lane-group form
    int off_half[2];
    int h_m, h_m0, h_rr, h_rrr, h_one, h_d, h_d2, h_onea, h_rra, h_rrra, h_size;
    int nla8, h_onea8, h_rra8, h_rrra8;  // the same for groups of 8 lanes (nla8 a multiple of 8)
    int off_qinvr;
    int stride;
};

PMK_HD constexpr int pad4(int x) { return (x + 3) & ~3; }

// Every radix-form field starts on a 16-byte boundary and is padded to a
// multiple of 4 limbs, so kernels read it with 128-bit loads.
PMK_HD constexpr Geom make_geom(int bits) {
    Geom g{};
    g.bits = bits;
    g.S = bits / 32;
    g.SH = bits / 64;
    g.lbf = lb_full(bits);
    g.nlf = round_up(nl_for(bits, g.lbf), lanes_full(bits));
    g.lbh = lb_half(bits);
    g.nlh = round_up(nl_for(bits / 2, g.lbh), lanes_half(bits));
    g.ew = 2;
    // lane-group limb counts: nla (a multiple of 4: groups of 2 and 4 lanes)
    // and nla8 (a multiple of 8: groups of 8); the half fields hold the larger,
    // zero-padded, since a lane group reads its K limbs of every field at pos K
    const int nla = lanes_half(bits) > 1 ? g.nlh : round_up(g.nlh, 4);
    const int nla8 = lanes_half(bits) > 1 ? g.nlh : (bits >= 2048 ? round_up(g.nlh, 8) : nla);
    const int pf = pad4(g.nlf), ph = pad4(nla8);
    int o = 0;
    g.off_nf = o; o += pf;
    g.off_rrf = o; o += pf;
    g.off_rrrf = o; o += pf;
    g.off_onef = o; o += pf;
    g.off_n32 = o; o += pad4(g.S);
    g.off_n0f = o; o += 1;
    g.off_e = o; o += g.ew;
    g.off_ebits = o; o += 1;
    g.off_kbytes = o; o += 4;
    // half record: m, rr, rrr, one (radix form), then m0, d
    g.h_m = 0;
    g.h_rr = ph;
    g.h_rrr = 2 * ph;
    g.h_one = 3 * ph;
    g.h_m0 = 4 * ph;
    g.h_d = 4 * ph + 4;
    g.h_d2 = g.h_d + pad4(g.SH);
    g.nla = nla;
    g.nla8 = nla8;
    if (lanes_half(bits) > 1) {  // lane groups already: the same constants
        g.h_onea = g.h_onea8 = g.h_one;
        g.h_rra = g.h_rra8 = g.h_rr;
        g.h_rrra = g.h_rrra8 = g.h_rrr;
        g.h_size = pad4(g.h_d2 + g.SH);
    } else {
        g.h_onea = pad4(g.h_d2 + g.SH);
        g.h_rra = g.h_onea + nla;
        g.h_rrra = g.h_rra + nla;
        g.h_size = g.h_rrra + nla;
        if (nla8 == nla) {
            g.h_onea8 = g.h_onea;
            g.h_rra8 = g.h_rra;
            g.h_rrra8 = g.h_rrra;
        } else {  // 4096 bits: 74 limbs, 76 for 2 and 4 lanes, 80 for 8
            g.h_onea8 = g.h_size;
            g.h_rra8 = g.h_onea8 + nla8;
            g.h_rrra8 = g.h_rra8 + nla8;
            g.h_size = g.h_rrra8 + nla8;
        }
    }
    g.off_half[0] = o; o += g.h_size;
    g.off_half[1] = o; o += g.h_size;
    g.off_qinvr = o; o += ph;
    g.stride = pad4(o);
    return g;
}

// Chunks are grouped into tiles of up to chunks_per_tile chunks that share one
// key, so a wavefront's modulus and exponent are wave-uniform (scalar
// registers, no divergence).  Slot = tile * chunks_per_tile + chunk; a padding
// slot has msg_len 0 and is computed but never written back.
struct ChunkDesc {
    uint64_t msg_off;  // first plaintext byte of the chunk
    uint64_t ct_off;   // first ciphertext byte of the chunk's block
    uint32_t key;      // record index inside the class key table
    uint32_t msg_len;  // plaintext bytes of this chunk (kb - 4, or the remainder); 0 = padding
};

constexpr int kTile = 64;  // bignums per wavefront

// Forms of the CRT halves whose reduction runs on the matrix cores (fold.hpp):
// numbers of nl limbs of lb bits (nl 0: the class has no such form), F = lb nl
// at least 17 bits above the class's largest prime, so that the folded sum stays
// well below 2^F.
struct FoldForm {
    int lb, nl;
};
// a number in one lane (launches that fill the chip)
PMK_HD constexpr FoldForm fold_lane(int bits) {
    switch (bits) {
        case 1024: return {28, 20};
        case 2048: return {29, 36};
        case 3072: return {28, 56};
        case 4096: return {28, 76};
        default: return {0, 0};
    }
}
// its waves per block (tiles of one key that share the prime's table in LDS:
// 7, 21, 51 and 94 KB) and per SIMD (limited by registers: 76 limbs take the
// whole file), and whether a window's entry is copied into LDS ahead of its
// product (where the table leaves room)
PMK_HD constexpr int fold_lane_block(int bits) { return bits >= 3072 ? 4 : 2; }
PMK_HD constexpr int fold_lane_waves(int bits) { return bits >= 4096 ? 1 : (bits >= 2048 ? 2 : 3); }
// the blinded form: its second window spills at three waves per SIMD (25 MB under
// 1024-bit keys: 9.8 / 9.2 ms with two)
PMK_HD constexpr int fold_joint_waves(int bits) { return fold_lane_waves(bits) < 2 ? 1 : 2; }
PMK_HD constexpr bool fold_lane_prefetch(int bits) { return bits <= 2048; }
// a number spread over a block (small launches; the classes above); nl a
// multiple of 4, LB = 28: limbs there carry up to twice 2^lb
PMK_HD constexpr FoldForm fold_group(int bits) {
    switch (bits) {
        case 1024: return {28, 20};
        case 2048: return {28, 40};
        case 3072: return {28, 56};
        case 4096: return {28, 76};
        case 6144: return {28, 112};
        case 8192: return {28, 148};
        default: return {0, 0};
    }
}
// K steps of 64 digits of its MFMAs, and how many of them stay in registers
PMK_HD constexpr int fold_group_steps(int bits) { return (4 * fold_group(bits).nl + 63) / 64; }
PMK_HD constexpr int fold_group_resident(int bits) { return bits > 6144 ? 3 : (bits > 4096 ? 5 : 16); }
PMK_HD constexpr int fold_group_waves(int) { return 2; }  // waves per SIMD
// waves per block
PMK_HD constexpr int fold_group_block(int bits) { return bits <= 1024 ? 1 : (bits <= 2048 ? 2 : (bits <= 4096 ? 4 : (bits <= 6144 ? 7 : 8))); }
// limbs per number of the half buffer: a fold result, or the canonical half
PMK_HD constexpr int half_stride(int bits) {
    const int nlh = make_geom(bits).nlh, a = fold_lane(bits).nl, b = fold_group(bits).nl;
    return a > nlh ? (a > b ? a : b) : (b > nlh ? b : nlh);
}
// Table of one prime (byte offsets): per form the 4 nl start values of the
// accumulators, then the digits of W in operand order.
struct FoldTable {
    uint32_t lane, group, size;
};
PMK_HD constexpr uint32_t fold_lane_bytes(FoldForm f) { return 16u * f.nl + 16u * f.nl * f.nl; }
PMK_HD constexpr FoldTable fold_table(int bits) {
    FoldTable t{};
    t.lane = 0;
    t.group = (uint32_t)round_up((int)fold_lane_bytes(fold_lane(bits)), 256);
    const uint32_t nl = (uint32_t)fold_group(bits).nl;
    t.size = t.group + (uint32_t)round_up((int)(16 * nl + nl / 4 * fold_group_steps(bits) * 1024), 256);
    return t;
}
// Bias of a result row, digit j of limb k: at or above the largest sum of 4 nl
// products of a digit of t_hi with a digit of W < 2^p; a power of two, 0 for rows
// that W does not reach.  Digits of t_hi are at most 128 in size, the top one of
// a limb 2^(lb - 24) + 1 (2^(lb - 23) + 1 where limbs carry up to twice 2^lb).
PMK_HD constexpr uint32_t fold_bias(FoldForm f, int p, int k, int j, bool loose) {
    const int nb = p - f.lb * k < f.lb ? p - f.lb * k : f.lb;  // bits of W in limb k
    if (nb < 8 * j || nb <= 0) return 0;
    const uint64_t w = nb >= 8 * j + 8 && j < 3 ? 128 : (1ull << (nb - 8 * j)) + 1;
    const uint64_t most = (uint64_t)f.nl * (3 * 128 + (1u << (f.lb - (loose ? 23 : 24))) + 2) * w;
    uint64_t b = 1;
    while (b < most) b <<= 1;
    return (uint32_t)b;
}

// Arguments of one class's launches inside a plan.
struct ClassRun {
    int cls;                   // index into kClassBits
    uint32_t count;            // chunks of this class
    uint32_t parts;            // groups of up to 16 of them under one key
    uint32_t share;            // classes whose launches run beside this one's (0 or 1: none)
    bool busy;                 // copies or other kernels may run when the launch starts
    uint32_t ntiles;           // key-uniform tiles of this class
    const uint32_t *keys;      // class key table (device), Geom::stride words per key
    const ChunkDesc *desc;     // ntiles * cpt slot descriptors (device)
    const uint32_t *tile_key;  // ntiles key records (device)
    const uint32_t *groups;    // fold form: ngroups groups of tiles under one key, the first tile and
    uint32_t ngroups;          // the tiles after it in bits 30 and 31 (device);
    uint32_t group_tiles;      // tiles of the largest
    const uint8_t *fold;       // fold tables of the class's keys (two primes each, fold_table); nullptr:
                               // they did not fit, Montgomery forms only
    uint32_t *x32;             // [tile][word < S][chunk < cpt]: packed input words
    uint32_t *y32;             // same shape: result words before unpacking
    uint32_t *half;            // [tile][p, q][limb < half_stride][chunk < cpt]: CRT half results
    uint32_t *table;           // per resident wave: window table scratch
    uint32_t slots_enc;        // wave slots in `table` for the encryption kernel
    uint32_t slots_dec;        // wave slots in `table` for the CRT-halves kernel
    uint64_t table_words;      // words of `table`
    uint32_t *err;             // device error word: bit 0 block out of range, bit 1 blinding factor not invertible
    uint8_t *slot_err;         // optional, per descriptor slot: 1 where unpacking rejected the chunk
    uint32_t grid_cap;         // 0, or the most resident waves a persistent launch may use
    int win;                   // window width of the CRT-halves exponentiation (3..6)
    int fill_lanes;            // lanes per number of the CRT halves of a launch under one round
                               // (one-lane classes 1, 2 or 4; lane-group classes lanes_half or twice it)
    int tail_lanes;            // one-lane classes: the same for the partial round after full ones,
                               // run as a launch of its own; 0: that round stays in the launch
    // blinded PMKRSA (Sec. 3.1, Algorithm 1)
    const uint32_t *fin32;     // encryption: words of a factor v < N the result is multiplied by
                               // (x^e v mod N; tile layout of y32), nullptr = 1; blinded decryption:
                               // the packed c_R blocks
};

constexpr int kMaxWin = 6;
// One-lane classes whose blinded CRT halves also run in groups of 8 lanes (2048-
// to 4096-bit keys, the classes whose record holds the nla8-limb constants), for
// small launches.
PMK_HD constexpr bool eight_lanes(int bits) { return lanes_half(bits) == 1 && bits >= 2048; }

// Limb count and constants (offsets in a half record) of the lane-group form
// with L lanes per number: nla limbs for 2 and 4 lanes, nla8 for 8.
PMK_HD constexpr int lane_limbs(const Geom &g, int L) { return L == 8 ? g.nla8 : g.nla; }
PMK_HD constexpr int lane_one(const Geom &g, int L) { return L == 8 ? g.h_onea8 : g.h_onea; }
PMK_HD constexpr int lane_rr(const Geom &g, int L) { return L == 8 ? g.h_rra8 : g.h_rra; }
PMK_HD constexpr int lane_rrr(const Geom &g, int L) { return L == 8 ? g.h_rrra8 : g.h_rrra; }
// Lanes-per-number settings a class takes: a one-lane class 1, 2 or 4 for
// both forms, and 8 for small launches where eight_lanes; a lane-group class
// its own count L0, or 2 L0 for small launches, and L0 for the tail form.  From
// 1024 bits on a fill count above lanes_half lets a small plain launch run with
// each number over a block (group_launch).
PMK_HD constexpr bool lanes_valid(int bits, int fill, int tail) {
    return lanes_half(bits) == 1
               ? ((fill == 1 || fill == 2 || fill == 4 || (fill == 8 && eight_lanes(bits))) &&
                  (tail == 1 || tail == 2 || tail == 4))
               : ((fill == lanes_half(bits) || fill == 2 * lanes_half(bits)) && tail == lanes_half(bits));
}
PMK_HD constexpr int default_fill_lanes(int bits) {
    return lanes_half(bits) > 1 ? 2 * lanes_half(bits) : (eight_lanes(bits) ? 8 : (bits >= 1024 ? 4 : 1));
}
PMK_HD constexpr int default_tail_lanes(int bits) { return lanes_half(bits) > 1 ? lanes_half(bits) : 1; }

// One persistent launch over the exponentiation work of the 1024- to 4096-bit
// classes of a plan: units (tiles, or job tiles of CRT halves) are numbered
// class by class, largest modulus first, and handed out by an atomic counter.
// The encryption of the 4096- and 3072-bit classes (4 lanes per number) runs
// as one persistent kernel whose waves take work units from a device counter,
// 4096-bit units first.
constexpr int kWideClasses = 2;
constexpr int kClass3072 = 5, kClass4096 = 6;
// class of entry i of the wide batch: 4096 bits, then 3072 bits
constexpr int wide_class(int i) { return kClass4096 - i; }
constexpr bool is_wide_class(int c) { return c == kClass3072 || c == kClass4096; }
struct BatchArgs {
    ClassRun runs[kWideClasses];       // runs[i] is class wide_class(i)
    uint32_t start[kWideClasses + 1];  // first unit of runs[i]; start[2] = total
    uint32_t *counter;                 // next unit to hand out (reset before each launch)
    uint32_t *table;                   // per-block window-table slots
    uint64_t slot_words;               // words per slot
};

// Launchers (kernels.hip).  All asynchronous on `stream`; return hipError_t as int.
int launch_pack(const ClassRun &r, const uint8_t *src, int decrypt, void *stream);
int launch_encrypt(const ClassRun &r, void *stream);
int launch_decrypt_halves(const ClassRun &r, void *stream);
int launch_garner(const ClassRun &r, void *stream);
// fold tables of a class's `count` key records (kfold.hip), two per key; `sums`: a buffer of
// `words` = fold_setup_words words for as long as that runs
uint64_t fold_setup_words(int cls, uint32_t count);
int launch_fold_setup(int cls, const uint32_t *keys, uint32_t count, uint8_t *fold, uint64_t *sums, uint64_t words,
                      void *stream);
inline uint64_t fold_bytes_per_key(int cls) { return 2ull * fold_table(kClassBits[cls]).size; }
// Groups of up to `per` tiles under one key (ClassRun::groups) of a class's
// tiles, appended to out: each key's tiles in the fewest groups, of equal sizes up to one.
// Returns the largest size.
template <typename Vec>
uint32_t tile_groups(const Vec &tile_key, uint32_t ntiles, int per, Vec &out) {
    uint32_t most = 1;
    for (uint32_t t = 0; t < ntiles;) {
        uint32_t n = 1;
        while (t + n < ntiles && tile_key[t + n] == tile_key[t]) ++n;
        for (uint32_t g = (n + per - 1) / per; n; --g) {
            const uint32_t k = (n + g - 1) / g;
            out.push_back(t | (k - 1) << 30);
            if (k > most) most = k;
            t += k;
            n -= k;
        }
    }
    return most;
}
// blinded decryption in one pass per prime: half[h] = (c*)^d_h c_R^(p_h-1-d_h) mod p_h
// with c* at r.x32 and c_R at r.fin32; tables need 2 table_words_per_slot(cls, 1, win)
// words per slot
int launch_decrypt_joint(const ClassRun &r, void *stream);
// Montgomery products in one lane, 1024- to 4096-bit classes: the CRT halves of a
// launch (kmont.inc), blinded decryption (kjmont.hip), and the waves of each that are
// resident on the current device (0: no such form)
PMK_HD constexpr int mont_waves(int bits) { return bits >= 3072 ? 2 : 3; }  // per SIMD, plain halves
int launch_mont(const ClassRun &r, void *stream);
int launch_joint_mont(const ClassRun &r, void *stream);
uint32_t mont_resident(int cls);
uint32_t joint_mont_resident(int cls);
// Job tiles of `r` in full rounds of `resident` one-wave blocks, then the partial
// round as a launch of its own, whose waves spread over the SIMDs; no more blocks
// than the table has slots of `slot` words or the grid limit allows.
template <typename Launch>
int launch_rounds(const ClassRun &r, uint64_t slot, uint32_t resident, Launch launch) {
    uint64_t grid = r.table_words / slot < resident ? r.table_words / slot : resident;
    if (r.grid_cap && r.grid_cap < grid) grid = r.grid_cap;
    if (grid < 1) grid = 1;
    const uint32_t units = 2 * r.ntiles, rest = (uint32_t)(units % grid);
    int e = 0;
    if (units > rest) e = launch((uint32_t)grid, 0u, units - rest);
    if (!e && rest) e = launch(rest, units - rest, units);
    return e;
}
// CRT halves of job tiles [jt_begin, jt_end) in lane groups of L lanes per
// number: the 128- to 512-bit classes with L = 2 or 4 (klanes.hip)
int launch_halves_lanes(const ClassRun &r, int L, uint32_t jt_begin, uint32_t jt_end, void *stream);
// resident waves of that lane-group kernel on the current device (0: no such kernel)
uint32_t lanes_resident(int cls, int L);
// Blinded decryption (one pass per prime) of job tiles [jt_begin, jt_end) in
// lane groups of L lanes (those that joint_lanes_resident knows; a lane-group
// class: twice its own), and that kernel's resident waves, 0 without one (kjlanes.hip)
int launch_joint_lanes(const ClassRun &r, int L, uint32_t jt_begin, uint32_t jt_end, void *stream);
uint32_t joint_lanes_resident(int cls, int L);

// Lanes per number for the part of a one-lane class's CRT launch that leaves
// SIMDs idle (L lanes per number give L times the waves, each with a chain
// about L times shorter).  units: job tiles of the launch; resident: waves of its one-lane
// kernel that fit the chip (already capped by the table slots and grid cap);
// simds: SIMDs of the device; room(cls, L): resident waves of the lane-group
// kernel.  A launch under one round runs wholly in lane groups of r.fill_lanes
// lanes, or of the largest smaller power of two that still gives every
// lane-group wave a SIMD of its own; the partial round after full ones runs
// with r.tail_lanes, or the largest smaller power of two whose waves fit one
// round of the lane-group kernel (1: one lane per number, still as a launch of
// its own; r.tail_lanes 0: no launch of its own).  Returns L and sets
// *lane_units to the job tiles of that last part (0: one launch).
inline int lanes_for_launch(const ClassRun &r, uint32_t units, uint32_t resident, uint32_t simds,
                            uint32_t (*room_of)(int, int), uint32_t *lane_units) {
    *lane_units = 0;
    if (resident == 0) return 1;
    const uint32_t rem = units % resident;
    auto fit = [&](int max_l, uint64_t limit) {
        for (int l = max_l; l >= 2; l /= 2) {
            uint64_t room = room_of(r.cls, l);
            if (limit < room) room = limit;
            if ((uint64_t)r.slots_dec * l < room) room = (uint64_t)r.slots_dec * l;  // table room
            if (r.grid_cap && r.grid_cap < room) room = r.grid_cap;
            if ((uint64_t)rem * l <= room) return l;
        }
        return 1;
    };
    int L = 1;
    if (units < resident) {
        L = fit(r.fill_lanes, simds);
        if (L > 1) *lane_units = rem;
    } else if (rem && r.tail_lanes > 0) {
        // the partial round after full ones runs as a launch of its own: its
        // waves then spread over the SIMDs, where the full rounds' last waves
        // would share them
        L = fit(r.tail_lanes, UINT64_MAX);
        *lane_units = rem;
    }
    return L;
}

// The lane-group classes (6144/8192-bit keys, L0 = lanes_half lanes per
// number): a launch of jt job tiles runs with r.fill_lanes = 2 L0 lanes per
// number when every such wave has a SIMD of its own and fits one round of
// that kernel (room: its resident waves) and the table (two such slots per
// slot of the L0 form).
inline bool wide_fill(const ClassRun &r, uint32_t jt, int L0, uint32_t simds, uint32_t room) {
    if (r.fill_lanes != 2 * L0) return false;
    uint64_t lim = simds < room ? simds : room;
    if ((uint64_t)r.slots_dec * 2 < lim) lim = (uint64_t)r.slots_dec * 2;
    if (r.grid_cap && r.grid_cap < lim) lim = r.grid_cap;
    return (uint64_t)jt * (uint64_t)r.fill_lanes <= lim;
}
// compute units of the current device
int device_cus();
// mode: 0 ciphertext blocks, 1 plaintext chunks (range-checked), 2 whole plaintext
// blocks (range-checked); the checks read the packed input at r.x32 (and r.fin32)
int launch_unpack(const ClassRun &r, uint8_t *dst, int mode, void *stream);
// table words needed per wave slot for a class (decryption: at window width win)
uint64_t table_words_per_slot(int cls, int decrypt, int win);
// resident wave slots the persistent kernels of a class use
uint32_t wave_slots(int cls, int decrypt, int num_cus);
// work units (wavefronts' worth of bignums) of the exponentiation kernels
uint32_t exp_units(int cls, int decrypt, uint32_t ntiles);
// table slots (waves) that a class's CRT-halves launch can use
uint32_t table_units(const ClassRun &r);
// CRT halves of a whole launch with numbers spread over blocks (kgroup.inc): units,
// table words per block, blocks that are resident, and the launch, which leaves
// fold results in r.half; launch_halves_group takes the tiles from that of group
// `first` on (r.groups; 0: all of them)
PMK_HD constexpr uint32_t group_units(uint32_t tiles) { return (tiles + 3) / 4 * 32; }  // parts of jobs, in eights
uint64_t group_slot_words(int cls, int win);
uint32_t group_resident(int cls);
int launch_halves_group(const ClassRun &r, uint32_t first, void *stream);
// Which form a launch takes (launch_rule.cpp), by the forms' estimated times.
// group_launch: CRT halves spread over blocks; mont_launch, joint_mont_launch:
// otherwise, Montgomery products in one lane rather than the fold form (1024 to
// 4096 bits; 6144 and 8192 bits have Montgomery products over 4 lanes); joint_two_lanes:
// of a small blinded launch, two lanes per number rather than either; group_rest: the
// last `groups` groups of tiles after full rounds of the lane form spread over blocks.
bool group_launch(const ClassRun &r, uint32_t cus);
bool mont_launch(const ClassRun &r, uint32_t cus);
bool joint_mont_launch(const ClassRun &r, uint32_t cus);
bool joint_two_lanes(const ClassRun &r, uint32_t cus);
bool group_rest(const ClassRun &r, uint32_t groups, uint32_t cus);
// Whether a class, of `classes` that run side by side, is too large for the group form
// beside the others and holds half of the SIMDs or more by itself.
bool fills_chip(const ClassRun &r, uint32_t classes, uint32_t cus);
// Cuts of a chunk range into slices [0, c_1), [c_1, c_2), ... that give every key only
// whole groups of `group` full tiles and 1, 2, 4, ... rounds of `round` tiles: slicing
// adds no partial round and splits no group (4096 bits, whose rounds need groups of four
// tiles: 256 keys with 256 chunks each, cut into halves of two tiles per key, took 116
// ms, uncut 64), and the copies of one slice overlap the kernels of its neighbours.
std::vector<uint64_t> whole_round_cuts(const uint32_t *key_map, uint64_t nchunks, uint32_t nkeys, uint64_t round,
                                       uint32_t group);
// table words that a class's launches use: plain, and blinded decryption
uint64_t table_words(const ClassRun &r);
uint64_t joint_table_words(const ClassRun &r);
// persistent batched exponentiation (kbatch.hip)
int launch_batch(const BatchArgs &a, uint32_t grid, void *stream);
int launch_counter_reset(uint32_t *counter, void *stream);
uint32_t batch_wave_slots(int num_cus);
// table words per wave slot of the wide batch kernel
uint64_t batch_slot_words();

// primality testing for key generation (kprime.hip); classes 3..6 (1024..4096-bit keys)
int prime_class_ok(int cls);
uint64_t mr_slot_words(int cls, int win);
uint32_t mr_wave_slots(int cls, int num_cus);
int launch_sieve_class(int cls, const uint32_t *cand, uint32_t count, uint32_t *flags, int device, void *stream);
int launch_mr_class(int cls, const uint32_t *cand, uint32_t count, const uint32_t *bases, int rounds, int win,
                    uint32_t *table, uint64_t slot_words, uint32_t grid, uint32_t *result, void *stream);

}  // namespace pmk
